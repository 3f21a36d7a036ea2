"""The two-factor DFT passes at every spacing of the partial sums' groups (none
to three rows added, one to sixteen columns a workgroup, few columns and many).
Against the FP64 FFT: n float32 products per output err by about sqrt(n) 2^-24
each pass, at most 2.7e-6 here, so 1e-5 holds."""
import numpy as np
import pytest
import torch

import oracle.postproc as postproc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(132, 2, 1), (2, 132, 3), (77, 2, 1), (120, 2, 3), (2, 121, 3), (40, 3, 1), (48, 2, 1),
                                  (3, 49, 2), (21, 2, 1), (24, 3, 2), (2, 25, 2), (1024, 2, 2), (1200, 1, 20),
                                  (39, 128, 130), (128, 105, 129), (98, 128, 130), (450, 64, 72), (64, 514, 72),
                                  (16, 784, 40)])
def test_pitches(dims):
    from paper_2604_09233_amd import nfs

    rng = np.random.default_rng(dims)
    L = int(np.prod(dims))
    x = (rng.standard_normal(L) + 1j * rng.standard_normal(L)).astype(np.complex64)
    f = rng.uniform(0, 1, L).astype(np.float32)
    got = nfs.apply_kspace_filter(torch.from_numpy(x), torch.from_numpy(f), dims).cpu().numpy()
    ref = postproc.apply_kspace_filter(x, f, dims)
    e = np.linalg.norm(got - ref) / np.linalg.norm(ref)
    print(f"filter {dims}: rel {e:.1e}")
    assert e < 1e-5
