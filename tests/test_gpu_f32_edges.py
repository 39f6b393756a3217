"""The fp32 row-split edge kernels at the sizes where their work split can go
wrong: ranges shorter than a 16-edge tile, exactly one tile, one edge more,
receivers without edges at either end, one receiver over several tiles, and
the smallest graphs (most waves without work); and the forward-only plan at
the static workspace's limit.  Tolerances: see test_gpu_parity."""
import numpy as np
import pytest

from synth import meshes
import paper_2307_13592_amd as mgn
from paper_2307_13592_amd.runner import Session
from parity import local_inputs, rel_err, say
from test_gpu_parity import _case, _with_edges

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("l,D", [(64, 2), (64, 3), (128, 2)])
@pytest.mark.parametrize("edges", [1, 15, 16, 17, 33, "hub", 4097])
def test_ranges(l, D, edges):
    if edges == "hub":  # one receiver with 40 edges, all others without
        m = meshes.hex_lattice(4)
        m.send = np.setdiff1d(np.arange(41), [20]).astype(np.int32)
        m.recv = np.full(40, 20, np.int32)
    else:
        m = meshes.hex_lattice(10 if edges > 100 else 4)
        rng = np.random.default_rng(edges)
        keep = np.zeros(m.n_edges, bool)
        keep[rng.choice(m.n_edges, edges, replace=False)] = True
        m = _with_edges(m, keep)
    _case(f"hex {edges} edges", m, 0, l, 2, D, "fp32")


def test_static_workspace_limit():
    """A graph whose forward-only plan fits the static workspace only without
    the halo rows of the projections runs without them and gives the training
    plan's outputs to fp32 accuracy (1e-5; the latents of the nodes cut off come
    from a float64 encoder here)."""
    say("[f32] static workspace limit")
    mesh = meshes.sector(30, 40, 40, 2, seed=5)
    c = local_inputs(mesh, 0, 128, 1, 2, 3)
    g = c["g"]
    full = Session(128, 1, 2, "fp32", g, c["nf"], c["ef"], c["halo"], c["params"])
    want = full.forward().cpu().numpy().copy()
    full.close()
    # receivers are cut off until the plan without halo rows just fits
    per_edge, per_node = 4 * 128 + 4, 3 * 4 * 128
    rp = g["row_ptr"].astype(np.int64)
    limit = mgn.MGN_NOALLOC_WS_MAX - (1 << 20)
    n = int(np.searchsorted(np.arange(rp.size) * per_node + rp * per_edge, limit)) - 1
    assert n < g["n_owned"], "the mesh is too small for this test"
    ne = int(rp[n])
    # the first n receivers keep their edges; all nodes past them become halo rows
    nl = g["n_owned"] + g["n_halo"]
    send = g["send"][:ne]
    order = np.argsort(send, kind="stable")
    gg = dict(n_owned=n, n_halo=nl - n, n_edges=ne, row_ptr=g["row_ptr"][:n + 1], send=send,
              trow_ptr=np.concatenate([[0], np.cumsum(np.bincount(send, minlength=nl))]).astype(np.int32),
              tedge=order.astype(np.int32))
    # K = 1: the cut-off nodes' latents are their encoder outputs
    v0 = _encode(c, n, g["n_owned"])
    halo = np.concatenate([v0, c["halo"][0]])[None].astype(np.float32)
    s = Session(128, 1, 2, "fp32", gg, c["nf"][:n], c["ef"][:ne], halo, c["params"], inference=True)
    try:
        assert s.ws_bytes <= mgn.MGN_NOALLOC_WS_MAX < s.ws_bytes + 4 * 128 * gg["n_halo"]
        mgn.mgn_forward_noalloc(s.model, s.gs, s.node_feat, s.edge_feat, s.halo, s.out)
        e = rel_err(s.out.cpu().numpy(), want[:n])
        say(f"  outputs against the training plan {e:.2e}")
        assert e < 1e-5
    finally:
        s.close()


def _encode(c, lo, hi):
    """float64 node encoder rows lo..hi of case c (latent 128, depth 2)."""
    import torch
    F = torch.nn.functional
    p = torch.as_tensor(c["params"].astype(np.float64))
    at, t = 0, {}
    for name, kind, shape in c["shapes"][:6]:
        k = int(np.prod(shape))
        t[name] = p[at:at + k].view(*shape)
        at += k
    x = torch.as_tensor(c["nf"][lo:hi].astype(np.float64))
    h = torch.relu(F.linear(x, t["enc_node.lin0.W"], t["enc_node.lin0.b"]))
    y = F.linear(h, t["enc_node.lin1.W"], t["enc_node.lin1.b"])
    return F.layer_norm(y, (128,), t["enc_node.ln.gamma"], t["enc_node.ln.beta"], 1e-5).numpy()
