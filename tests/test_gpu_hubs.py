"""fp32 row-split edge kernels on graphs with very large receivers, whose edges
a workgroup's waves share (the sums of a receiver that goes on from one wave to
the next are joined at the end): against the oracle with receivers that span
many waves, several to a workgroup, and one that takes all edges; the
forward-only plan bitwise; and the time of one large receiver.  Tolerances: see
test_gpu_parity."""
import numpy as np
import pytest

import paper_2307_13592_amd as mgn
from paper_2307_13592_amd.runner import Session
from parity import calibrate, compare, local_inputs, oracle_sensitivity, run_gpu, run_oracle, say
from synth import meshes

pytestmark = pytest.mark.gpu


def _mesh(kind):
    m = meshes.hex_lattice(8)
    n = m.n_nodes
    rng = np.random.default_rng(2)
    if kind == "star":  # 65 edges, one more than a wave takes alone on a small graph
        deg = {100: 65}
    elif kind == "star all":
        deg = {250: n - 1}
    elif kind == "many":  # two or three receivers to a workgroup, cut at any edge
        deg = {r: int(rng.integers(60, 131)) for r in range(n)}
    else:  # "mixed": small receivers between large ones of 16, 17 and more tiles, receivers without edges
        deg = {r: int(rng.integers(0, 9)) for r in range(n)}
        deg.update({3: 256, 4: 257, 200: 511, 201: 300, 202: 65, n - 1: 400})
    recv = np.concatenate([np.full(d, r) for r, d in deg.items()])
    send = np.concatenate([rng.permutation(np.setdiff1d(np.arange(n), [r]))[:d] for r, d in deg.items()])
    m.send, m.recv = send.astype(np.int32), recv.astype(np.int32)
    return m


@pytest.mark.parametrize("l,D", [(64, 2), (64, 3), (128, 2)])
@pytest.mark.parametrize("kind", ["star", "star all", "many", "mixed"])
def test_large_receivers(kind, l, D):
    say(f"[hubs] {kind} l={l} D={D}")
    K = 2
    c = local_inputs(_mesh(kind), 0, l, K, D, 3)
    gpu = run_gpu(c, l, K, D, "fp32")
    assert all(np.isfinite(x).all() for x in gpu)
    again = run_gpu(c, l, K, D, "fp32")
    assert all(np.array_equal(x, y) for x, y in zip(gpu, again)), "two runs differ"
    bad = compare(f"hubs {kind} l={l} D={D}", "fp32", c["shapes"], gpu, run_oracle(c, l, K, D),
                  calibrate(c, l, K, D, "fp32", runs=3), sens=oracle_sensitivity(c, l, K, D, "fp32", runs=3))
    assert not bad, bad
    s = Session(l, K, D, "fp32", c["g"], c["nf"], c["ef"], c["halo"], c["params"], inference=True)
    try:
        assert np.array_equal(s.forward().cpu().numpy(), gpu[0]), "forward-only outputs differ"
    finally:
        s.close()


@pytest.mark.parametrize("l", [64, 128])
def test_one_receiver_is_shared(l):
    """16,384 edges into one receiver against the same number into 2,048, which
    is a tile or less for every wave.  A wave alone on the one receiver took
    240 to 390 times as long; eight waves, two to a SIMD, take 48 to 85; 150
    allowed."""
    say(f"[hubs] one receiver l={l}")
    n, E = 16_400, 16_384
    rng = np.random.default_rng(1)
    m = mgn.mgn_create(l, 1, 2, mgn.MGN_FP32)
    params = (0.05 * rng.standard_normal(mgn.mgn_param_count(m))).astype(np.float32)
    mgn.mgn_destroy(m)
    t = {}
    for receivers in (1, 2048):
        if receivers == 1:
            send = 1 + np.arange(E)
        else:  # eight neighbours each
            n = receivers
            send = (np.repeat(np.arange(n), 8) + np.tile(np.arange(1, 9), n)) % n
        g = mgn.mgn_graph_build(send.astype(np.int32), np.repeat(np.arange(receivers, dtype=np.int32), E // receivers),
                                np.zeros(n, np.int32), n, 0)
        s = Session(l, 1, 2, "fp32", g, rng.standard_normal((n, 11)), rng.standard_normal((E, 4)), None, params)
        try:
            d_out = rng.standard_normal((n, 5)).astype(np.float32)
            s.forward()
            s.backward(d_out)
            mgn.mgn_timing_enable(s.model)
            for _ in range(3):
                s.forward()
                s.backward(d_out)
            r = mgn.mgn_timing_read(s.model)
            t[receivers] = {k: r[k][0] / 3 for k in ("edge_fwd", "edge_bwd")}
        finally:
            s.close()
    for k in ("edge_fwd", "edge_bwd"):
        say(f"  {k}: one receiver {t[1][k]:.3f} ms, 2,048 receivers {t[2048][k]:.3f} ms")
    assert all(t[1][k] < 150 * t[2048][k] for k in t[1])
