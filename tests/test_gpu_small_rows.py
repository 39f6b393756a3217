"""Weight gradients over few rows: node and edge counts around the row steps
of the grouped weight-gradient kernel (16 rows in fp32, 32 in bf16; at least 64
per split), at every latent width, one node and no edges included.
Tolerances: see test_gpu_parity."""
import numpy as np
import pytest

from synth import meshes
from test_gpu_parity import _case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("l,D", [(64, 3), (128, 2), (256, 2)])
@pytest.mark.parametrize("nodes,edges", [(1, 0), (17, 15), (33, 64), (65, 65), (130, 1057)])
def test_small_rows(prec, l, D, nodes, edges):
    m = meshes.hex_lattice(6)
    rng = np.random.default_rng(nodes)
    pair = rng.choice(nodes * nodes, edges, replace=False)
    m.send, m.recv = (pair // nodes).astype(np.int32), (pair % nodes).astype(np.int32)
    m.n_nodes = nodes
    m.coords, m.node_type, m.key = m.coords[:nodes], m.node_type[:nodes], m.key[:nodes]
    m.stream_blocks = [(0, nodes, 0)]
    _case(f"{nodes} nodes {edges} edges", m, 0, l, 1, D, prec)
