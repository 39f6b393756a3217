"""The l = 256 layer passes (bf16, from 32,768 edges on): against the oracle at
both depths on a partition with halo, isolated receivers and a ragged tail,
and the plans against each other: the forward-only plan gives the training
plan's outputs bitwise; the
checkpointed plan in chunks on either side of the passes' limit agrees with the
plan that keeps every block (outputs bitwise, gradients to 1e-4: sums over
chunks add in another order)."""
import numpy as np
import pytest

from synth import meshes
from paper_2307_13592_amd.runner import Session
from parity import calibrate, compare, local_inputs, oracle_sensitivity, rel_err, run_gpu, run_oracle, say, segments
from test_gpu_parity import _with_edges

pytestmark = pytest.mark.gpu


def _inputs(K, D):
    m = meshes.sector(20, 16, 36, 4, seed=9)
    m = _with_edges(m, m.recv % 23 != 0)
    c = local_inputs(m, 1, 256, K, D, 3)
    assert 32768 <= c["g"]["n_edges"] < 40000 and c["g"]["n_edges"] % 16
    return c


@pytest.mark.parametrize("D", [2, 3])
def test_wide_against_oracle(D):
    say(f"[wide] oracle D={D}")
    c = _inputs(1, D)
    gpu = run_gpu(c, 256, 1, D, "bf16")
    ref = run_oracle(c, 256, 1, D, bf16=True)
    bad = compare(f"wide D={D}", "bf16", c["shapes"], gpu, ref, calibrate(c, 256, 1, D, "bf16", runs=3),
                  sens=oracle_sensitivity(c, 256, 1, D, "bf16", runs=3))
    assert not bad, bad


def test_wide_node_rows():
    """Node half and node encoder in layer passes (35,937 nodes, a ragged tail)."""
    say("[wide] node rows")
    m = meshes.hex_lattice(33)
    keep = np.zeros(m.n_edges, bool)
    keep[np.random.default_rng(1).choice(m.n_edges, 3001, replace=False)] = True
    c = local_inputs(_with_edges(m, keep), 0, 256, 1, 2, 3)
    gpu = run_gpu(c, 256, 1, 2, "bf16")
    ref = run_oracle(c, 256, 1, 2, bf16=True)
    bad = compare("wide node rows", "bf16", c["shapes"], gpu, ref, calibrate(c, 256, 1, 2, "bf16", runs=2),
                  sens=oracle_sensitivity(c, 256, 1, 2, "bf16", runs=2))
    assert not bad, bad


@pytest.mark.parametrize("D", [2, 3])
def test_wide_plans(D):
    K = 3
    say(f"[wide] plans D={D}")
    c = _inputs(K, D)
    base = run_gpu(c, 256, K, D, "bf16")
    s = Session(256, K, D, "bf16", c["g"], c["nf"], c["ef"], c["halo"], c["params"], inference=True)
    out = s.forward().cpu().numpy().copy()
    s.close()
    assert np.array_equal(out, base[0]), "forward-only outputs differ"
    for chunk in (0, 20000):  # one chunk (layer passes), two (streamed weights in the backward)
        lean = run_gpu(c, 256, K, D, "bf16", recompute=2, chunk_edges=chunk)
        assert np.array_equal(lean[0], base[0]), "checkpointed outputs differ"
        e = max(rel_err(lean[1][sl], base[1][sl]) for _, sl in segments(c["shapes"]))
        say(f"  chunk {chunk}: parameter gradients {e:.1e}, halo {rel_err(lean[2], base[2]):.1e}")
        assert e <= 1e-4 and rel_err(lean[2], base[2]) <= 1e-4
