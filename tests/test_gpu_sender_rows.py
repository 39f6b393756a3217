"""bf16 row-split edge forward: the sender half of the first Linear is formed
per edge from the sender's bf16 row, and stored per node only where a backward
recomputes h_1 from it.  The plans that store it (every block kept,
checkpointing) and those that do not (inference, first-Linear stash) give the
same bits, and the oracle's outputs to the precision's tolerance, on
partitions of a few nodes (less than a tile, ragged last tiles, waves without
edges) and with halo senders."""
import numpy as np
import pytest

from paper_2307_13592_amd.runner import Session
from parity import TOL, local_inputs, rel_err, run_oracle, say
from synth import meshes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("l,D", [(64, 2), (64, 3), (128, 2)])
@pytest.mark.parametrize("nr,nt,nz,parts", [(2, 4, 2, 4), (3, 6, 5, 2), (5, 9, 7, 3)])
def test_plans_agree_on_small_partitions(l, D, nr, nt, nz, parts):
    say(f"[sender rows] sector {nr}x{nt}x{nz}/{parts} l={l} D={D}")
    K = 3
    c = local_inputs(meshes.sector(nr, nt, nz, parts, seed=11), 1, l, K, D, parts)
    outs = []
    for plan in (dict(), dict(inference=True), dict(h1_stash=2), dict(h1_stash=K), dict(recompute=2)):
        s = Session(l, K, D, "bf16", c["g"], c["nf"], c["ef"], c["halo"], c["params"], **plan)
        try:
            outs.append(s.forward().cpu().numpy().copy())
        finally:
            s.close()
        assert np.array_equal(outs[0], outs[-1]), plan
    e = rel_err(outs[0], run_oracle(c, l, K, D, bf16=True)["out"])
    say(f"  out {e:.2e}")
    assert e <= TOL["bf16"]
