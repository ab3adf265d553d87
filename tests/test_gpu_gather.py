"""The gather of kept rows at the widths and sizes where its launch changes: one
to eight columns of 64 16-byte pieces and more, rows that are no multiple of 16
bytes, element-wise rows, copies stored in bursts and one column at a time;
byte for byte against X[idx].  lambda = 0 with a supplied Stage II key: X is read
by the gather alone."""
import pytest
import torch

pytestmark = pytest.mark.gpu

DEV = "cuda"

# elements of a row around the edges of a column (512 bf16, 256 fp32), of the
# two-row launches (4096, 2048) and of the element-wise rows (64, 160 elements)
WIDTHS = {torch.bfloat16: [1, 7, 8, 9, 33, 64, 65, 159, 161, 511, 512, 513, 1023, 1025, 1535, 1537, 2048, 2050, 2561, 3072,
                           3577, 3584, 4095, 4096, 4097, 8191, 8193, 12288],
          torch.float32: [1, 3, 4, 5, 63, 65, 161, 255, 256, 257, 513, 1025, 1793, 2047, 2048, 2049, 4097, 6145]}


def check(B, n, D, dtype, K):
    import paper_2607_13500_amd as tr
    print("[case] gather", B, n, D, dtype, K, flush=True)
    g = torch.Generator(device=DEV).manual_seed(D + n)
    X = torch.randint(-32768, 32767, (B * n, D * (1 if dtype == torch.bfloat16 else 2)), generator=g, device=DEV,
                      dtype=torch.int16).view(dtype)
    s = torch.rand(B * n, generator=g, device=DEV)
    r = tr.Reducer(D, D, dtype, lam=0.0, max_images=B, max_tokens=B * n, max_N=n)
    out = torch.zeros(B * K + 2, D, dtype=dtype, device=DEV)       # a row before and after the result stays
    res = r.reduce_given_s(X, s, [n] * B, [K] * B, out=out[1:-1])
    rows = res.idx.long() + torch.arange(B, device=DEV).repeat_interleave(K) * n
    bits = torch.int16 if dtype == torch.bfloat16 else torch.int32
    assert torch.equal(out[1:-1].view(bits), X.view(bits)[rows])
    assert not out[0].view(bits).any() and not out[-1].view(bits).any()
    r.close()


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_gather_every_width(dtype):
    for D in WIDTHS[dtype]:
        check(1, 1100, D, dtype, 37)           # above 1024 tokens the gather is a launch of its own
        check(3, 1100, D, dtype, 211)


@pytest.mark.parametrize("D,dtype", [(33, torch.bfloat16), (160, torch.bfloat16), (63, torch.float32), (1024, torch.bfloat16),
                                     (2048, torch.bfloat16), (4095, torch.bfloat16), (4096, torch.float32)])
def test_gather_every_size(D, dtype):
    e = 2 if dtype == torch.bfloat16 else 4
    for mb in (9, 19, 21, 35, 37, 79, 81, 89, 91, 150):
        rows = int(mb * 1e6 / (D * e))
        B = max(1, rows // 3000)
        check(B, 4000, D, dtype, rows // B if rows // B <= 4000 else 4000)
