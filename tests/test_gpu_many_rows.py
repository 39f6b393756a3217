"""fp32 kernels that only larger partitions reach, against torch_ref's network
in float64 on the device: the 128 x 128 weight-gradient stream kernel (more than
262,144 rows with an odd tail; at latent 256 as four blocks of each layer), and
the latent-64 node projections over more than 8,192 local nodes, with odd
remainders in the owned and in the halo rows.  Among the 10^7 and more ReLU
inputs of such a case some lie within rounding of zero, and one that changes
sides moves a tensor by up to 4e-3; so the parameters keep them away from it
(away_from_zero), and every tensor meets the nominal 1e-4."""
import numpy as np
import pytest
import torch

from parity import away_from_zero, compare, local_inputs, run_gpu, say
from synth import meshes
import torch_ref

pytestmark = pytest.mark.gpu


def _reference(c, l, K, D):
    with torch.device("cuda"):
        model = torch_ref.TorchMGN(l, K, D)
        model.load_flat(c["params"], c["shapes"])
        f64 = lambda a: torch.as_tensor(np.asarray(a, np.float64))
        h = f64(c["halo"]).requires_grad_(True)
        out = model(c["g"], f64(c["nf"]), f64(c["ef"]), h)
        out.backward(f64(c["d_out"]))
        dh = h.grad if h.grad is not None else torch.zeros_like(h)
        return dict(out=out.detach().cpu().numpy(), d_params=model.flat_grad().cpu().numpy(), d_halo=dh.cpu().numpy())


def _check(name, c, l, K, D):
    c = away_from_zero(c, D)
    gpu = run_gpu(c, l, K, D, "fp32")
    assert all(np.isfinite(x).all() for x in gpu)
    bad = compare(name, "fp32", c["shapes"], gpu, _reference(c, l, K, D))
    assert not bad, bad


@pytest.mark.parametrize("l", [128, 256])
def test_weight_gradient_stream(l):
    say(f"[many rows] l={l}")
    m = meshes.hex_lattice(37)  # 295,704 edges
    keep = np.ones(m.n_edges, bool)
    keep[np.random.default_rng(4).choice(m.n_edges, 30_001, replace=False)] = False
    m.send, m.recv = m.send[keep], m.recv[keep]
    assert (1 << 18) < m.n_edges < 270_000 and m.n_edges % 16
    _check(f"fp32 stream l={l}", local_inputs(m, 0, l, 1, 2, 3), l, 1, 2)


@pytest.mark.parametrize("D", [2, 3])
def test_projections_of_many_nodes(D):
    say(f"[many rows] projections l=64 D={D}")
    c = local_inputs(meshes.sector(41, 16, 59, 4, seed=9), 1, 64, 2, D, 3)
    g = c["g"]
    assert g["n_owned"] > 8192 and g["n_owned"] % 16 and g["n_halo"] > 4096 and g["n_halo"] % 16
    _check(f"projections l=64 D={D}", c, 64, 2, D)
