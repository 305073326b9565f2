"""The bank builder's quadrant transforms at the edges of their 16 x 16 matrix
tiles: beta S + 1 and beta S / 2 + 1 samples around multiples of 16, the
smallest planes, one plane, planes of very different sizes in one call, against
the FP64 oracle with the bar of the other bank test (FP32 rounding of taps of
at most 1)."""
import numpy as np
import pytest

from oracle import wkernel as WK
from paper_2111_04141_amd import workload as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("beta,base_support,supports", [
    (1, 2, (2,)),
    (1, 2, (2, 4, 14, 16, 30, 32, 64)),
    (2, 3, (3, 7, 8, 15, 16, 17, 31, 33)),
    (3, 4, (4, 10, 6, 64)),
    (8, 2, (2, 3, 4, 5, 64)),
    (30, 1, (1, 2, 17)),
])
def test_bank_shapes(beta, base_support, supports):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2111_04141_amd import api
    base = W.pswf_taps(base_support, beta)
    ws = [37.0 * p for p in range(len(supports))]
    ref, offs = WK.wbank(base, beta, np.array(supports, np.int32), ws, 0.08)
    bank, goffs = api.wkernel_bank(list(supports), ws, beta, torch.from_numpy(base).cuda(), 0.08)
    assert goffs == offs.tolist()
    err = np.max(np.abs(bank.cpu().numpy().astype(np.complex128) - ref))
    print(f"[bank] beta {beta}, supports {supports}: max |error| {err:.2e}", flush=True)
    assert err < 2e-7
