"""The scan of long launches (whole 256-token units per wave) against the
general scan, bit for bit.

A batch long enough for the unit scan is scored in one call, then sequence by
sequence, where each call is short and takes the general scan (of 16-bit keys:
more than two units per CU and fewer than 16, so that it is the one with
guarded loads): the logits are the same sums in the same order, so S must not
differ in any bit.  The scan of the shortest calls, which reads through the same
buffer descriptors, is compared with the general one likewise.  The shapes
sit at the edges: exactly as many units as the rule asks for, a last unit with
one token, a padding unit, 1 to 8 heads per KV head, padded and token-major
keys, and a cache past the 32-bit offsets of the unit scan (which then keeps
the general one)."""
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


def _keys(layout, B, Hkv, n, dt, g):
    if layout == "rows":
        k = torch.randn((B, Hkv, n, 128), generator=g, device=DEV, dtype=torch.float32)
        return k.to(dt)
    if layout == "padded":       # 8 elements between rows, 3 rows between heads
        buf = torch.randn((B, Hkv, n + 3, 136), generator=g, device=DEV, dtype=torch.float32).to(dt)
        return buf[:, :, :n, :128]
    if layout == "tokens":       # [B, n, Hkv, D]
        return torch.randn((B, n, Hkv, 128), generator=g, device=DEV, dtype=torch.float32).to(dt).transpose(1, 2)
    # "far": one sequence's rows 512 KiB apart, shared by the whole batch
    sn = 262144
    buf = torch.zeros(n * sn, dtype=dt, device=DEV)
    k = buf.as_strided((1, Hkv, n, 128), (0, 128, sn, 1))
    k.copy_(torch.randn((1, Hkv, n, 128), generator=g, device=DEV).to(dt))
    return buf.as_strided((B, Hkv, n, 128), (0, 128, sn, 1))


@pytest.mark.parametrize("B,Hq,Hkv,n,bits,dtype,layout", [
    (4, 32, 8, 32767, 0, "bf16", "rows"),       # 4096 units, the last token missing
    (4, 32, 8, 32769, 0, "fp16", "padded"),     # a unit of one token and a padding unit
    (7, 40, 8, 20225, 0, "bf16", "tokens"),     # 5 heads per KV head
    (7, 64, 8, 20000, 0, "fp16", "rows"),       # 8 heads: the whole pass
    (5, 28, 4, 60001, 0, "bf16", "rows"),       # 7 heads, odd batch
    (16, 32, 8, 8192, 0, "bf16", "far"),        # offsets past 4 GiB: the general scan
    (16, 32, 8, 8191, 8, "bf16", "rows"),
    (16, 56, 8, 8230, 8, "fp16", "tokens"),
    (8, 32, 8, 8191, 4, "bf16", "rows"),        # 2048 units
    (8, 24, 8, 8193, 4, "fp16", "rows"),
    (8, 8, 8, 8190, 4, "bf16", "padded"),
    (3, 64, 8, 30002, 4, "fp16", "rows"),
])
def test_unit_scan_equals_general_scan(B, Hq, Hkv, n, bits, dtype, layout):
    import paper_2602_18750_amd as H
    dt = torch.bfloat16 if dtype == "bf16" else torch.float16
    g = torch.Generator(device=DEV).manual_seed(n + bits)
    k = _keys(layout, B, Hkv, n, dt, g)
    q = torch.randn((B, Hq, 128), generator=g, device=DEV, dtype=torch.float32).to(dt)
    sk = H.sketch_keys(k, bits=bits) if bits else None
    s_all = H.new_importance(B, 1, n, DEV)
    s_one = H.new_importance(B, 1, n, DEV)
    H.hill_score(q, k, s_all, sketch=sk)
    for b in range(B):
        sb = H.hill.Sketch(sk.codes[b:b + 1], sk.exps[b:b + 1], bits) if bits else None
        H.hill_score(q[b:b + 1], k[b:b + 1], s_one[b:b + 1], sketch=sb)
    torch.cuda.synchronize()
    assert torch.isfinite(s_all).all()
    assert torch.equal(s_all, s_one), "%d tokens differ" % int((s_all != s_one).sum())


@pytest.mark.parametrize("B,Hq,Hkv,n,dtype,layout", [
    (3, 32, 8, 8191, "bf16", "rows"),         # 256 units per sequence, 768 in the batch
    (3, 32, 8, 8193, "fp16", "padded"),       # a unit of one token and a padding unit
    (3, 40, 8, 8225, "bf16", "tokens"),
    (5, 64, 8, 5001, "fp16", "padded"),
    (3, 28, 4, 16001, "bf16", "tokens"),
    (270, 8, 1, 1, "fp16", "rows"),           # two units (one of padding) per sequence, 540 in the batch
    (300, 4, 1, 33, "bf16", "padded"),
])
def test_pair_scan_equals_general_scan(B, Hq, Hkv, n, dtype, layout):
    """Calls of at most two units per CU (512), sequence by sequence, against
    the batch of 513 to 4095 units, which takes the general scan."""
    import paper_2602_18750_amd as H
    dt = torch.bfloat16 if dtype == "bf16" else torch.float16
    g = torch.Generator(device=DEV).manual_seed(n)
    k = _keys(layout, B, Hkv, n, dt, g)
    q = torch.randn((B, Hq, 128), generator=g, device=DEV, dtype=torch.float32).to(dt)
    s_all, s_one = H.new_importance(B, 1, n, DEV), H.new_importance(B, 1, n, DEV)
    H.hill_score(q, k, s_all)
    for b in range(B):
        H.hill_score(q[b:b + 1], k[b:b + 1], s_one[b:b + 1])
    torch.cuda.synchronize()
    assert torch.isfinite(s_all).all()
    assert torch.equal(s_all, s_one), "%d tokens differ" % int((s_all != s_one).sum())
