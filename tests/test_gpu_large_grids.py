"""Token counts whose one launch would pass a limit of the grid: 2^32 threads (more are silently cut), and
the 65536 blocks in y that the device states (this runtime runs more)."""
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


@pytest.mark.parametrize("t", [36800, 37000, 65000, 65200])
def test_combine_on_both_sides_of_the_cached_rows(moe, t):
    """Plain loads for 170 to 300 MB of rows, non-temporal ones below and beyond."""
    h = 1152
    assert (170e6 <= t * h * 4 <= 300e6) == (t in (37000, 65000))
    y = torch.randn((t, h), device="cuda")
    dest = torch.randperm(t, device="cuda").to(torch.int32)[:, None].contiguous()
    w = torch.rand((t, 1), device="cuda") + 0.5
    out = torch.empty((t, h), dtype=torch.int16, device="cuda")
    moe.moe_combine(y, dest, w, out)
    assert torch.equal(out, (w * y[dest[:, 0].long()]).to(torch.bfloat16).view(torch.int16))


def test_quantization_of_2_35_values(moe):
    """16 threads per 128 values: 2^32 threads and more.  104 GB, all ones: code 448 and scale 1 / 448."""
    rows = (1 << 28) + 64
    x = torch.full((rows, 128), 0x3f80, dtype=torch.int16, device="cuda")
    q = torch.zeros((rows, 128), dtype=torch.uint8, device="cuda")
    s = torch.zeros((rows, 1), device="cuda")
    moe.moe_quant_act(x, q, s)
    del x
    one = torch.tensor(1.0) / torch.tensor(448.0)
    for a in range(0, rows, 1 << 24):
        assert bool((q[a:a + (1 << 24)] == 0x7e).all()), a
    assert bool((s == one.item()).all())
    del q, s
    torch.cuda.empty_cache()


def test_router_of_more_than_65535_token_tiles(moe):
    """128-token tiles lie along y: every token's result equals that of a call with fewer tokens."""
    t, h, e = 65535 * 128 + 300, 32, 8
    g = torch.Generator(device="cuda").manual_seed(5)
    x = torch.randn((t, h), generator=g, device="cuda").to(torch.bfloat16)
    w = torch.randn((e, h), generator=g, device="cuda").to(torch.bfloat16)

    def route(x):
        ids = torch.full((len(x), 1), -1, dtype=torch.int32, device="cuda")
        wts = torch.zeros((len(x), 1), device="cuda")
        ws = torch.empty(moe.moe_router_workspace(len(x), h, e), dtype=torch.uint8, device="cuda")
        ws.fill_(0xff)  # partial logits that a call leaves out are NaN
        moe.moe_router(x, w, None, ids, wts, ws=ws)
        return ids, wts

    ids, wts = route(x)
    assert int(ids.min()) >= 0
    step = 1 << 20
    for a in range(0, t, step):
        b = min(t, a + step)
        want = route(x[a:b])
        assert torch.equal(ids[a:b], want[0]) and torch.equal(wts[a:b], want[1]), a
