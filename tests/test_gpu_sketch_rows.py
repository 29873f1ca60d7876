"""Key sketches written in ranges (a prefill, then appended tokens) against
the whole cache written at once, bit for bit, and against the definition (the
smallest exponent that fits, codes to nearest even) in 64 bits, at the edges of
the rows a workgroup takes (64) and of a lane group's (16)."""
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2602_18750_amd as H
    H.load_library()
    yield


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("B,Hkv,n", [(1, 1, 1), (2, 3, 63), (1, 8, 64), (3, 1, 65), (2, 2, 129), (1, 4, 1000)])
def test_ranges(B, Hkv, n, bits):
    import paper_2602_18750_amd as H
    g = torch.Generator(device=DEV).manual_seed(n)
    k = (torch.randn((B, n, Hkv, 128), generator=g, device=DEV) * 3).to(torch.bfloat16).transpose(1, 2)
    k[0, 0, 0] = 0.0
    whole = H.sketch_keys(k, bits=bits)
    parts = H.new_sketch(B, Hkv, n, DEV, bits=bits)
    cuts = sorted({0, 1, 15, 16, 17, 63, 64, 100, n} & set(range(n + 1)))
    for a, b in zip(cuts[:-1], cuts[1:]):
        H.sketch_keys(k, parts, token_begin=a, token_end=b)
    torch.cuda.synchronize()
    assert torch.equal(whole.codes, parts.codes) and torch.equal(whole.exps, parts.exps)
    qmax = 127 if bits == 8 else 7
    x = k.double()
    amax = x.abs().amax(-1)
    m, e = torch.frexp(amax)
    e = torch.where(m <= qmax / (qmax + 1), e, e + 1) - (7 if bits == 8 else 3)
    e = torch.where(amax > 0, e.clamp(-128, 127), torch.full_like(e, -128))
    assert torch.equal(whole.exps[:, :, :n].int(), e.int())
    c = torch.round(torch.ldexp(x, -e.unsqueeze(-1))).clamp(-qmax, qmax).int()
    if bits == 4:
        c = c.view(B, Hkv, n, 16, 2, 4) + 8
        c = (c[..., 0, :] | (c[..., 1, :] << 4)).flatten(-2)
    assert torch.equal(whole.codes[:, :, :n], c.to(torch.uint8).view(torch.int8))
