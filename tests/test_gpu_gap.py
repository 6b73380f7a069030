"""Global average pooling on its own: one and two planes per wavefront, an odd number of planes, one to four loads each."""
import numpy as np
import pytest

import xl_workloads as W
from oracle import xlo

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,c,h,w", [(91, 91, 7, 7), (91, 91, 8, 9), (91, 91, 13, 13), (91, 91, 14, 14), (3, 7, 1, 1), (3, 7, 8, 8),
                                     (3, 7, 9, 13), (3, 7, 13, 13), (3, 7, 14, 14)])
def test_against_the_oracle(n, c, h, w):
    from paper_2007_06000_amd.session import Session
    wl = W.conv_gap_generic(n, 5, h, w, c, 1, 0, 1)
    x, params = W.make_tensors(wl)
    ref = xlo.forward(wl, x, params)
    print(f"[case] {wl.name} {n} images", flush=True)
    y = Session(wl, x, params).output(False)
    # 5 fp32 multiply-adds per value, then a mean of up to 196 of them in another order
    assert np.linalg.norm(y - ref) <= 2.0 ** -20 * np.linalg.norm(ref)
    assert np.abs(y - ref).max() <= 2.0 ** -18 * np.abs(ref).max()
