"""Receivers without edges in long runs, before, between and after those with
edges: the edge kernels zero their rows (agg forward, the receiver sums of
dz_0 backward).  Against the same graph with those nodes spread among the
others, which the oracle comparisons cover, and the time it takes: the zeroing
is shared by all waves, not left to the one whose range of edges the run
adjoins."""
import numpy as np
import pytest

import paper_2307_13592_amd as mgn
from paper_2307_13592_amd.runner import Session
from parity import rel_err, run_gpu, say, segments
import synth
from synth import meshes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,l,D", [("fp32", 64, 2), ("fp32", 128, 2), ("fp32", 64, 3), ("bf16", 64, 2),
                                      ("bf16", 128, 2), ("bf16", 256, 2)])
def test_runs_without_edges(prec, l, D):
    """Renumbering the nodes, the senders' order kept, leaves every node's
    output bit for bit the same, and the parameter gradients to the rounding
    of sums over at most 729 rows and 900 edges in another order (900 x 2^-24
    = 5e-5 of the largest; 1e-4 allowed)."""
    say(f"[edge free] {prec} l={l} D={D}")
    m = meshes.hex_lattice(9)
    n = m.n_nodes
    band = lambda v: ((v >= 200) & (v < 260)) | ((v >= 500) & (v < 530))
    keep = band(m.send) & band(m.recv)
    send, recv = m.send[keep], m.recv[keep]
    rng = np.random.default_rng(5)
    shapes = synth.param_shapes(l, 2, D)
    params = synth.init_params(shapes, 3)
    nf = rng.standard_normal((n, 11)).astype(np.float32)
    ef = rng.standard_normal((send.size, 4)).astype(np.float32)
    d_out = rng.standard_normal((n, 5)).astype(np.float32)
    connected = np.flatnonzero(band(np.arange(n)))
    spread = np.empty(n, np.int64)  # new id of each node: the connected ones every eighth, in their order
    spread[connected] = 3 + 8 * np.arange(connected.size)
    rest = np.setdiff1d(np.arange(n), connected)
    spread[rest] = np.setdiff1d(np.arange(n), spread[connected])
    res = []
    for ids in (np.arange(n), spread):
        g = mgn.mgn_graph_build(ids[send].astype(np.int32), ids[recv].astype(np.int32), np.zeros(n, np.int32), n, 0)
        back = np.argsort(ids)
        c = dict(g=g, nf=nf[back], ef=ef[g["eperm"]], halo=np.zeros((2, 0, l), np.float32), params=params,
                 d_out=d_out[back])
        out, dp, _ = run_gpu(c, l, 2, D, prec)
        res.append((out[ids], dp))
    assert np.isfinite(res[0][0]).all() and np.array_equal(res[0][0], res[1][0])
    e = max(rel_err(res[1][1][sl], res[0][1][sl]) for _, sl in segments(shapes))
    say(f"  parameter gradients {e:.1e}")
    assert e <= 1e-4


@pytest.mark.parametrize("prec,l", [("fp32", 64), ("fp32", 128), ("bf16", 128)])
def test_long_run_is_shared(prec, l):
    """300,000 nodes with edges among the first hundred: a block's edge half
    writes zeros only, so it takes at most a few times what the node half,
    which reads and writes more, takes (with one wave zeroing the run it took
    6.8 ms a launch at l = 128, 22 times as much; shared, a quarter of it)."""
    say(f"[edge free] {prec} l={l}")
    n = 300_000
    send = np.arange(100, dtype=np.int32)
    g = mgn.mgn_graph_build(send, (send + 1) % 100, np.zeros(n, np.int32), n, 0)
    rng = np.random.default_rng(1)
    m = mgn.mgn_create(l, 1, 2, mgn.MGN_BF16 if prec == "bf16" else mgn.MGN_FP32)
    params = (0.05 * rng.standard_normal(mgn.mgn_param_count(m))).astype(np.float32)
    mgn.mgn_destroy(m)
    s = Session(l, 1, 2, prec, g, rng.standard_normal((n, 11)), rng.standard_normal((100, 4)), None, params)
    try:
        d_out = rng.standard_normal((n, 5)).astype(np.float32)
        s.forward()
        s.backward(d_out)
        mgn.mgn_timing_enable(s.model)
        for _ in range(3):
            s.forward()
            s.backward(d_out)
        t = {k: v[0] / 3 for k, v in mgn.mgn_timing_read(s.model).items()}
        say("  " + ", ".join(f"{k} {t[k]:.3f} ms" for k in ("edge_fwd", "node_fwd", "edge_bwd", "node_bwd")))
        assert t["edge_fwd"] < 4 * t["node_fwd"] and t["edge_bwd"] < 4 * t["node_bwd"]
    finally:
        s.close()
