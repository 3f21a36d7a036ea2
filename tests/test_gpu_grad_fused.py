"""The one-pass gradient of the field coefficients (FP32 form) against the
FP64 formula, at the edges of its tiles and blocks: one to 31 terms (one and
two blocks of 16, 33 terms' phase parts), 1 to 64 coils (blocks of 16, 32 and
64), sample and voxel counts off the 16-item chunks, an odd number of voxel
chunks (the last pair half empty), fewer items than a tile, phases past the
raw sine range, and zero data.  Two-part f16 operands give about 2^-21 per
product against a gradient whose terms add incoherently, so the FP32 bar
(1e-4) holds throughout; past 128 revolutions the float32-grade phase itself
is off by up to 2^-21 of the phase bound (about 1e-3 rad at 400 revolutions)
and sets the bar."""
import numpy as np
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu


def reference(d, g):
    a = (d["sens"], d["fields"], d["b0"], d["kcoef"], d["t"])
    out = np.empty((d["K"], d["n_basis"]))
    for b in range(d["n_basis"]):
        z = oracle.apply_E(d["fields"][b].astype(np.float64) * d["rho"].astype(np.complex128), *a)
        out[:, b] = np.imag(np.sum(g.astype(np.complex128) * np.conj(z), axis=0))
    return out


@pytest.mark.parametrize("L,K,G,P,scale,bar", [
    (300, 700, 4, 7, 10.0, 1e-4),
    (16, 16, 1, 1, 10.0, 1e-4),
    (5, 3, 2, 3, 10.0, 1e-4),
    (1000, 333, 16, 16, 10.0, 1e-4),
    (1009, 641, 17, 17, 10.0, 1e-4),
    (530, 258, 32, 20, 10.0, 1e-4),
    (777, 129, 33, 10, 10.0, 1e-4),
    (260, 100, 64, 31, 10.0, 1e-4),
    (4097, 2100, 8, 16, 10.0, 1e-4),
    (400, 300, 6, 9, 900.0, 5e-3),
])
def test_fused_kcoef_gradient(L, K, G, P, scale, bar):
    from paper_2604_09233_amd import nfs

    d = synth.random_problem(L, K, G, P, seed=91, phase_scale=scale)
    # samples of very different size: each is scaled by itself
    g = (d["m"] * np.logspace(0, -6, K)[None, :]).astype(np.complex64)
    gp = nfs.Problem(d["sens"], d["fields"], d["b0"], d["kcoef"], d["t"])
    _, _, gk = nfs.encode_backward(gp, torch.from_numpy(d["rho"]), torch.from_numpy(g), "fp32", False, False, True)
    ref = reference(d, g)
    got = gk.cpu().numpy().astype(np.float64)
    rows = np.linalg.norm(got - ref, axis=1) / np.linalg.norm(ref, axis=1)
    e = np.linalg.norm(got - ref) / np.linalg.norm(ref)
    print(f"fused grad_kcoef L={L} K={K} G={G} P={P}: rel {e:.1e}, median sample {np.median(rows):.1e}")
    assert e < bar
    assert np.median(rows) < bar


def test_fused_kcoef_gradient_zero_and_repeat():
    from paper_2604_09233_amd import nfs

    d = synth.random_problem(500, 400, 5, 16, seed=92)
    gp = nfs.Problem(d["sens"], d["fields"], d["b0"], d["kcoef"], d["t"])
    rho = torch.from_numpy(d["rho"]).cuda()
    m = torch.from_numpy(d["m"]).cuda()
    z = nfs.encode_backward(gp, rho, torch.zeros_like(m), "fp32", False, False, True)[2]
    assert torch.count_nonzero(z) == 0
    z = nfs.encode_backward(gp, torch.zeros_like(rho), m, "fp32", False, False, True)[2]
    assert torch.count_nonzero(z) == 0
    a = nfs.encode_backward(gp, rho, m, "fp32")
    b = nfs.encode_backward(gp, rho, m, "fp32")
    assert all(torch.equal(x, y) for x, y in zip(a, b))


@pytest.mark.parametrize("prec", ["fp16", "bf16"])
@pytest.mark.parametrize("L,K,G,P", [(1000, 700, 4, 16), (333, 257, 16, 17), (900, 500, 21, 9), (700, 300, 32, 5),
                                     (500, 200, 33, 4), (64, 48, 1, 31), (40, 20, 2, 2), (3000, 2000, 15, 16)])
def test_grouped_kcoef_gradient(prec, L, K, G, P):
    """The half-precision forms take several terms per E launch where their
    coils fit 64 virtual ones (groups, a shorter last group, a single last
    term, no group at all): at the operand rounding's bar."""
    from paper_2604_09233_amd import nfs

    d = synth.random_problem(L, K, G, P, seed=93, phase_scale=8.0)
    gp = nfs.Problem(d["sens"], d["fields"], d["b0"], d["kcoef"], d["t"])
    gk = nfs.encode_backward(gp, torch.from_numpy(d["rho"]), torch.from_numpy(d["m"]), prec, False, False, True)[2]
    ref = reference(d, d["m"])
    got = gk.cpu().numpy().astype(np.float64)
    per_term = np.linalg.norm(got - ref, axis=0) / np.linalg.norm(ref, axis=0)
    print(f"grouped grad_kcoef {prec} L={L} K={K} G={G} P={P}: worst term {per_term.max():.1e}")
    assert per_term.max() < 4e-3  # 2e-3 operand bar; single small terms may stand at twice the whole's error
