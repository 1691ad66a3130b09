"""Buckets of evenly spread keys fit a workgroup.  The run-capacity testing hook
makes a bucket that is collected in runs visible (flag 16): no call, or one of
sixty, on normal keys at a fixed share may need them."""
import sys

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

drt = pytest.importorskip("paper_2109_08219_amd")


@pytest.mark.parametrize("dtype,n,k", [(torch.float32, 1 << 24, 1 << 21), (torch.float64, 1 << 22, 1 << 18)])
def test_even_keys_fit(dtype, n, k):
    g = torch.Generator(device="cuda")
    g.manual_seed(17)
    drt.check()
    drt.set_run_cap(50)
    over = 0
    try:
        for call in range(60):
            x = torch.randn(n, dtype=dtype, device="cuda", generator=g)
            drt.topk_select(x, k)
            try:
                drt.check()
            except drt.DrTopkError as e:
                assert e.flags & 16
                over += 1
    finally:
        drt.set_run_cap(0)
    print("[case] calls with a bucket in runs:", over, file=sys.stderr, flush=True)
    assert over <= 1, over
