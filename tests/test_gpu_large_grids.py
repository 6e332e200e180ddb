"""Token counts whose one launch would pass a limit of the grid: 2^32 threads, 65535 blocks in y."""
import pytest
import torch

from gpu_cases import require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def moe():
    return require_gpu()


def test_combine_of_more_than_2_24_workgroups(moe):
    """256 threads a workgroup, one workgroup a token at 128 columns: more than 2^32 threads."""
    t, h, rows = (1 << 24) + 5, 128, 64
    y = torch.randn((rows, h), device="cuda")
    dest = torch.randint(0, rows, (t, 1), dtype=torch.int32, device="cuda")
    w = torch.rand((t, 1), device="cuda") + 0.5
    out = torch.full((t, h), -7, dtype=torch.int16, device="cuda")
    moe.moe_combine(y, dest, w, out)
    for a in range(0, t, 1 << 21):
        b = min(t, a + (1 << 21))
        want = (w[a:b] * y[dest[a:b, 0].long()]).to(torch.bfloat16)  # one product, rounded in fp32 and once to bf16
        assert torch.equal(out[a:b], want.view(torch.int16)), a
