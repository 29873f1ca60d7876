"""Steps on short rows (one launch selects, attends and writes the outputs)
and the selection alone on rows of up to 32768 tokens (one launch), at the
edges of their ranges.

The step's indices must be the oracle's exact top-k of the step's own S (lower
index first among equal keys, pins first), its output the 64-bit softmax over
them: fp32 sums of k weights that sum to one and logits of 128 products give
(128 + k) * 2^-24 of the largest |V|.  Sizes: one token to one past the
longest row, budgets of one token, the row, and one past the largest list;
rows of equal keys, NaN and infinities; 1 to 9 heads per KV head; per-KV-head
rows; RAW and sketch scores (K gathered) on both sides of their rule; padded
and token-major caches; a streamed sequence that grows past the row limit."""
import numpy as np
import pytest
import torch

from oracle import oracle as O

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2602_18750_amd as H
    H.load_library()
    yield


def _inputs(B, Hq, Hkv, n, dt, seed, layout="rows"):
    g = torch.Generator(device=DEV).manual_seed(seed)

    def cache():
        if layout == "tokens":
            return torch.randn((B, n, Hkv, 128), generator=g, device=DEV).to(dt).transpose(1, 2)
        if layout == "padded":
            return torch.randn((B, Hkv, n + 5, 136), generator=g, device=DEV).to(dt)[:, :, :n, :128]
        return torch.randn((B, Hkv, n, 128), generator=g, device=DEV).to(dt)
    return torch.randn((B, Hq, 128), generator=g, device=DEV).to(dt), cache(), cache(), g


def _check(q, k, v, s, idx, out, ks, sink=0, recent=0):
    B, Hq, _ = q.shape
    Hkv, R = k.shape[1], s.shape[1]
    G = Hq // Hkv
    want = O.topk_pinned(s.cpu().numpy(), ks, sink, recent)
    assert np.array_equal(idx.cpu().numpy(), want)
    for b in range(B):
        for h in range(Hkv):
            rows = idx[b, h if R > 1 else 0].long()
            x = q[b, h * G:(h + 1) * G].double() @ k[b, h, rows].double().T / 128 ** 0.5
            vs = v[b, h, rows].double()
            err = (out[b, h * G:(h + 1) * G].double() - torch.softmax(x, -1) @ vs).abs().max()
            assert err <= (128 + ks) * 2.0 ** -24 * vs.abs().max(), "b %d head %d: %.3g" % (b, h, err)


@pytest.mark.parametrize("B,Hq,Hkv,n,ks,rows,score,layout,pins", [
    (1, 32, 8, 1, 1, "token", "attn", "rows", (0, 0)),
    (2, 4, 4, 3, 2, "token", "attn", "rows", (0, 0)),
    (1, 32, 8, 1021, 204, "token", "attn", "padded", (0, 0)),
    (1, 7, 1, 2047, 1024, "token", "attn", "rows", (4, 64)),
    (3, 16, 8, 2048, 2, "token", "attn", "tokens", (0, 0)),
    (2, 14, 2, 2049, 1, "kvhead", "attn", "rows", (0, 0)),
    (1, 18, 2, 4095, 1023, "token", "attn", "rows", (0, 0)),       # 9 heads: two passes
    (17, 32, 8, 4096, 409, "token", "attn", "rows", (4, 0)),       # 136 KV heads: whole rows of V per workgroup
    (1, 32, 8, 4096, 1025, "token", "attn", "rows", (0, 0)),       # past the longest list
    (1, 32, 8, 4097, 409, "token", "attn", "rows", (0, 0)),        # past the longest row
    (1, 32, 8, 1024, 1024, "token", "attn", "rows", (0, 0)),       # the whole row
    (1, 32, 8, 2000, 256, "token", "int8", "padded", (0, 0)),
    (1, 32, 8, 2000, 257, "token", "int8", "rows", (0, 0)),        # few KV heads gather K for a long list
    (8, 56, 8, 3000, 300, "token", "int4", "tokens", (0, 16)),
    (2, 16, 4, 1500, 150, "kvhead", "raw", "rows", (0, 0)),
    (9, 32, 8, 3333, 1000, "token", "raw", "rows", (0, 0)),
])
def test_step(B, Hq, Hkv, n, ks, rows, score, layout, pins):
    import paper_2602_18750_amd as H
    dt = torch.float16 if (n + ks) % 2 else torch.bfloat16
    q, k, v, _ = _inputs(B, Hq, Hkv, n, dt, n + ks, layout)
    R = 1 if rows == "token" else Hkv
    s = H.new_importance(B, R, n, DEV)
    sk = H.sketch_keys(k, bits=int(score[3:])) if score.startswith("int") else None
    for _ in range(2):
        idx, out = H.hill_step(q, k, v, s, ks, mode="raw" if score == "raw" else "attn", granularity=rows, sketch=sk,
                               n_sink=pins[0], n_recent=pins[1])
        torch.cuda.synchronize()
        _check(q, k, v, s, idx, out, ks, *pins)


@pytest.mark.parametrize("n,ks", [(1000, 300), (4096, 1000), (3001, 7)])
@pytest.mark.parametrize("kind", ["equal", "few", "special", "digits"])
def test_ties_and_special_values(n, ks, kind):
    """S that the step adds to (RAW scores of zero keys add nothing): all
    equal, a few distinct values, NaN / infinities / signed zeros, and keys
    that share their first 12 and 22 bits."""
    import paper_2602_18750_amd as H
    q, k, v, g = _inputs(1, 8, 8, n, torch.bfloat16, n)
    k.zero_()
    s = H.new_importance(1, 1, n, DEV)
    if kind == "equal":
        s.fill_(1.5)
    elif kind == "few":
        s[0, 0] = torch.randint(-2, 3, (n,), generator=g, device=DEV).float()
    elif kind == "special":
        vals = torch.tensor([float("nan"), float("inf"), -float("inf"), 0.0, -0.0, 1.0, -1.0], device=DEV)
        s[0, 0] = vals[torch.randint(0, 7, (n,), generator=g, device=DEV)]
    else:
        low = torch.randint(0, 6, (n,), generator=g, device=DEV) + 1024 * torch.randint(0, 3, (n,), generator=g, device=DEV)
        s[0, 0] = (low.int() + 0x3F900000).view(torch.float32)
    want = O.topk_pinned(s.cpu().numpy(), ks)
    assert np.array_equal(H.hill_topk(s, ks).cpu().numpy(), want)
    idx, _ = H.hill_step(q, k, v, s, ks, mode="raw")
    assert np.array_equal(idx.cpu().numpy(), want)


@pytest.mark.parametrize("rows,n,ks", [(1, 1, 1), (3, 8191, 8191), (2, 8193, 1), (5, 20011, 2001), (1, 32767, 16000),
                                       (2, 32768, 3276), (2, 32769, 3276)])
def test_selection_alone(rows, n, ks):
    import paper_2602_18750_amd as H
    g = torch.Generator(device=DEV).manual_seed(n)
    s = H.new_importance(1, rows, n, DEV)
    s.copy_(torch.randn((1, rows, n), generator=g, device=DEV).mul(8).round() / 8)   # many equal keys
    sink, recent = (min(4, ks), min(n, ks) // 3) if n > 8 else (0, 0)
    idx, val = H.hill_topk(s, ks, granularity="kvhead", with_values=True, n_sink=sink, n_recent=recent)
    want = O.topk_pinned(s.cpu().numpy(), ks, sink, recent)
    assert np.array_equal(idx.cpu().numpy(), want)
    assert torch.equal(val, s.gather(-1, idx.long()))


@pytest.mark.parametrize("streamed", [False, True])
def test_every_stage_is_stamped(streamed):
    """A short row's one launch takes REFINE and MERGE over: their events are
    recorded too, as empty intervals in their places (REFINE not in a streamed
    step, which has no such stage)."""
    import paper_2602_18750_amd as H
    q, k, v, _ = _inputs(1, 32, 8, 1000, torch.bfloat16, 3)
    s, st = H.new_importance(1, 1, 1000, DEV), H.new_stream_state(1, 1, DEV) if streamed else None
    stages, stream = H.hill.STAGES, torch.cuda.current_stream()
    start = [torch.cuda.Event(enable_timing=True) for _ in stages]
    stop = [torch.cuda.Event(enable_timing=True) for _ in stages]
    first = torch.cuda.Event(enable_timing=True)
    for e in start + stop + [first]:
        e.record(stream)
    torch.cuda.synchronize()
    ev = H.HillStepEvents.of([e.cuda_event for e in start], [e.cuda_event for e in stop])
    H.hill_step(q, k, v, s, 100, stream_state=st, events=ev)
    torch.cuda.synchronize()
    at = 0.0
    for name in ["scan", "update"] + ([] if streamed else ["refine"]) + ["select", "merge"]:
        i = stages.index(name)
        a, b = first.elapsed_time(start[i]), first.elapsed_time(stop[i])
        assert 0.0 < a and at <= a + 1e-3 and a <= b + 1e-3, (name, at, a, b)
        at = b


def test_streamed_sequence_grows_past_the_row_limit():
    """The bound that a short row's step writes serves the first longer row."""
    import paper_2602_18750_amd as H
    cap = 4200
    q, k, v, _ = _inputs(1, 32, 8, cap, torch.bfloat16, 9)
    s, s2 = H.new_importance(1, 1, cap, DEV), H.new_importance(1, 1, cap, DEV)
    st = H.new_stream_state(1, 1, DEV)
    for t, n in enumerate([4090, 4093, 4096, 4097, 4097, 4100, 4200]):
        ks = n // 10
        i1, o1 = H.hill_step(q, k, v, s, ks, n_tokens=n, stream_state=st, stream_reset=t == 0)
        i2, o2 = H.hill_step(q, k, v, s2, ks, n_tokens=n)
        torch.cuda.synchronize()
        assert torch.equal(s, s2) and torch.equal(i1, i2) and torch.equal(o1, o2), "n %d" % n
        assert st.view(-1)[2] == n and st.view(-1)[3] == 1
