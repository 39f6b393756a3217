"""fp32 forward-only plan with a halo: the halo rows of the projections are
optional in its workspace.  With room for them and without (each tile with halo
senders then forms its own), from the caller's workspace or the library's
static one, the outputs are bitwise the training plan's; a workspace smaller
than the plan without them is refused."""
import numpy as np
import pytest
import torch

import paper_2307_13592_amd as mgn
from paper_2307_13592_amd.runner import Session
from parity import local_inputs, say
from synth import meshes

pytestmark = pytest.mark.gpu


def _rows(n_halo, l):
    return (4 * n_halo * l + 255) // 256 * 256


def _run(s, nbytes, fill=0xff):
    """Outputs with a workspace of nbytes, with NaNs in it and after it."""
    buf = torch.full((nbytes + 4096,), fill, dtype=torch.uint8, device=s.device)
    s.out.fill_(float("nan"))
    mgn.mgn_forward(s.model, s.gs, s.node_feat, s.edge_feat, s.halo, s.out, buf[:nbytes])
    out = s.out.cpu().numpy().copy()
    assert bool((buf[nbytes:] == fill).all()), "wrote past the workspace"
    return out


@pytest.mark.parametrize("l,D", [(64, 2), (64, 3), (128, 2)])
@pytest.mark.parametrize("kind", ["slab", "interior", "all halo", "hub"])
def test_with_and_without_halo_rows(kind, l, D):
    say(f"[infer halo] {kind} l={l} D={D}")
    K = 3
    if kind == "slab":      # halo on one side, few edges
        c = local_inputs(meshes.sector(3, 6, 5, 3, seed=2), 0, l, K, D, 4)
    elif kind == "interior":  # both sides, ragged last tiles
        c = local_inputs(meshes.sector(9, 16, 11, 4, seed=7), 1, l, K, D, 4)
    else:
        m = meshes.hex_lattice(8)
        n, own = m.n_nodes, 200
        part = (np.arange(n) >= own).astype(np.int32)
        if kind == "all halo":  # no edge between owned nodes
            keep = part[m.send] != part[m.recv]
            m.send, m.recv = m.send[keep], m.recv[keep]
        else:  # one owned node receives from every other node (split among waves)
            other = np.setdiff1d(np.arange(n), [77])
            keep = m.recv != 77
            m.send = np.concatenate([m.send[keep], other]).astype(np.int32)
            m.recv = np.concatenate([m.recv[keep], np.full(n - 1, 77)]).astype(np.int32)
        c = local_inputs(m, 0, l, K, D, 4, part)
    args = (l, K, D, "fp32", c["g"], c["nf"], c["ef"], c["halo"], c["params"])
    s = Session(*args)
    want = s.forward().cpu().numpy().copy()
    s.close()
    assert np.isfinite(want).all()
    s = Session(*args, inference=True)
    try:
        full, less = s.ws_bytes, s.ws_bytes - _rows(c["g"]["n_halo"], l)
        for size in (full, full + 4096, full - 256, less):
            assert np.array_equal(_run(s, size), want), f"workspace {size - full:+d} bytes"
        with pytest.raises(mgn.MgnError) as e:
            _run(s, less - 256)
        assert e.value.status == mgn.MGN_E_NOMEM
        s.out.fill_(float("nan"))
        mgn.mgn_forward_noalloc(s.model, s.gs, s.node_feat, s.edge_feat, s.halo, s.out)
        assert np.array_equal(s.out.cpu().numpy(), want), "static workspace"
    finally:
        s.close()


def test_at_the_static_workspace_limit():
    """A graph that fits the static workspace only without the halo rows (9,000
    owned and 20,000 halo nodes, 220,000 edges, l = 128)."""
    say("[infer halo] static workspace limit")
    no, nh, ne, l = 9_000, 20_000, 220_000, 128
    rng = np.random.default_rng(3)
    recv = np.sort(rng.integers(0, no, ne)).astype(np.int32)
    send = rng.integers(0, no + nh, ne).astype(np.int32)
    order = np.lexsort((send, recv))
    send = send[order]
    g = dict(n_owned=no, n_halo=nh, n_edges=ne, row_ptr=np.searchsorted(recv, np.arange(no + 1)).astype(np.int32),
             send=send, trow_ptr=np.concatenate([[0], np.cumsum(np.bincount(send, minlength=no + nh))]).astype(np.int32),
             tedge=np.argsort(send, kind="stable").astype(np.int32))
    m = mgn.mgn_create(l, 2, 2, mgn.MGN_FP32)
    params = (0.08 * rng.standard_normal(mgn.mgn_param_count(m))).astype(np.float32)
    mgn.mgn_destroy(m)
    args = (l, 2, 2, "fp32", g, rng.standard_normal((no, 11)), rng.standard_normal((ne, 4)),
            rng.standard_normal((2, nh, l)), params)
    s = Session(*args)
    want = s.forward().cpu().numpy().copy()
    s.close()
    s = Session(*args, inference=True)
    try:
        limit = mgn.MGN_NOALLOC_WS_MAX
        assert s.ws_bytes <= limit < s.ws_bytes + _rows(nh, l)
        for size in (s.ws_bytes, limit, s.ws_bytes + _rows(nh, l)):
            assert np.array_equal(_run(s, size), want), size
        s.out.fill_(float("nan"))
        mgn.mgn_forward_noalloc(s.model, s.gs, s.node_feat, s.edge_feat, s.halo, s.out)
        assert np.array_equal(s.out.cpu().numpy(), want), "static workspace"
    finally:
        s.close()
