"""Bank planes around and above the beta S = 1024 up to which the cosine products
go: the largest of those, the smallest by transforms (sizes with factors the
library likes and others), both kinds in one call, and builds that overlap on
two streams, against the FP64 oracle with the bar of the other bank tests."""
import numpy as np
import pytest

from oracle import wkernel as WK
from paper_2111_04141_amd import workload as W

pytestmark = pytest.mark.gpu


def _case(beta, base_support, supports):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    base = W.pswf_taps(base_support, beta)
    ws = [29.0 * (p + 1) for p in range(len(supports))]
    ref, offs = WK.wbank(base, beta, np.array(supports, np.int32), ws, 0.05)
    return torch.from_numpy(base).cuda(), ws, ref, offs


@pytest.mark.parametrize("beta,base_support,supports", [
    (64, 2, (16,)),
    (27, 2, (38,)),
    (64, 2, (3, 17, 16, 4)),
    (106, 2, (10, 2)),
    (64, 2, (32,)),
])
def test_large_planes(beta, base_support, supports):
    from paper_2111_04141_amd import api
    base, ws, ref, offs = _case(beta, base_support, supports)
    bank, goffs = api.wkernel_bank(list(supports), ws, beta, base, 0.05)
    assert goffs == offs.tolist()
    err = np.max(np.abs(bank.cpu().numpy().astype(np.complex128) - ref))
    print(f"[bank] beta {beta}, supports {supports}: max |error| {err:.2e}", flush=True)
    assert err < 2e-7


def test_overlapping_builds():
    import torch
    from paper_2111_04141_amd import api
    beta, supports = 37, (30, 2, 30)
    base, ws, ref, _ = _case(beta, 2, supports)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(2)]
    banks = []
    for k in range(6):
        with torch.cuda.stream(streams[k % 2]):
            banks.append(api.wkernel_bank(list(supports), ws, beta, base, 0.05)[0])
    torch.cuda.synchronize()
    for b in banks:
        assert np.max(np.abs(b.cpu().numpy().astype(np.complex128) - ref)) < 2e-7
