"""The filter's DFT passes at the edges of the two-factor rule and of its
tiles: lengths with no useful factors (direct sums), the shortest and longest
with two factors, a length whose factors pay only without a long line, ragged
column counts, one axis alone (both passes in one launch) and axes of either
kind in each position.  Against the FP64 FFT: n float32 products per output
err by about sqrt(n) 2^-24 each pass, at most 2.7e-6 here, so 1e-5 holds."""
import numpy as np
import pytest
import torch

import oracle.postproc as postproc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(12, 1, 1), (15, 1, 1), (16, 1, 1), (97, 1, 1), (1, 96, 1), (1, 1, 100), (2031, 1, 1),
                                  (2039, 3, 1), (2048, 1, 1), (1, 2048, 3), (3, 2, 2047), (16, 15, 97), (97, 16, 1),
                                  (35, 33, 18), (18, 13, 36), (1009, 18, 1), (160, 129, 30)])
def test_filter_passes(dims):
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
