"""The maxima and the packing in front of the first encode launch, at the edge
between the single launch of small calls (up to 16384 samples and voxels) and
the whole-chip kernels, with the largest phase term, sample value and voxel
value on the last item of each side, 16 to 30 times the others: a maximum that
misses it overflows that item's 16-bit parts (their headroom is 4).  Against
the FP64 formula.  The phase bound is about 300 rad and the phase good to
2^-21 of it (1.4e-4 rad), which sets the FP32 bar; FP16 operands are good to
2^-11 (4.9e-4) each."""
import numpy as np
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,bar", [("fp32", 3e-4), ("fp16", 2e-3)])
@pytest.mark.parametrize("L,K,G,P", [(1, 1, 1, 0), (5, 16384, 3, 2), (5, 16385, 3, 2), (16384, 7, 3, 2),
                                     (16385, 7, 3, 2), (1025, 1031, 33, 16), (300, 4099, 64, 31)])
def test_setup_maxima_and_packing(prec, bar, L, K, G, P):
    from paper_2604_09233_amd import nfs

    d = synth.random_problem(L, K, G, P, seed=17, phase_scale=0.3, b0_hz=1.0)
    d["kcoef"][-1] *= 16
    d["fields"][:, -1] *= 16
    d["t"][-1] *= 16
    d["b0"][-1] *= 16
    d["rho"][-1] *= 30
    d["m"][:, -1] *= 30
    a = (d["sens"], d["fields"], d["b0"], d["kcoef"], d["t"])
    gp = nfs.Problem(*a)
    rho, m = torch.from_numpy(d["rho"]), torch.from_numpy(d["m"])
    x = oracle.apply_EH(d["m"].astype(np.complex128), *a)
    y = oracle.apply_E(d["rho"].astype(np.complex128), *a)
    z = oracle.apply_EH(y, *a)
    for name, got, ref in (("E", nfs.apply_E(gp, rho, prec), y), ("EH", nfs.apply_EH(gp, m, prec), x),
                           ("EHE", nfs.apply_EHE(gp, rho, prec), z)):
        e = np.linalg.norm(got.cpu().numpy() - ref) / np.linalg.norm(ref)
        print(f"setup {name} {prec} L={L} K={K} G={G} P={P}: rel {e:.1e}")
        assert e < bar
