"""Attention with the heads of a group in the fewest passes (the last one
masked), and lists longer than the batch of rows held in registers, against a
plain 64-bit softmax over the selected rows.

Groups of 3 to 20 heads (one masked pass, whole passes, a masked second and
third), through the fused steps (16-bit logits, RAW and sketch, whose attention
gathers K) and the standalone attention; and a RAW batch of more workgroups
than three per CU whose selection crowds into one chunk (lists of 1, 64, 65,
128, 129 and 400 entries).  Tolerance: fp32 sums of at most k = 400 products
with weights that sum to one and logits of 128 products: (128 + 400) * 2^-24
relative to the largest |V| that is summed, about 3.2e-5 * max|V|."""
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


def _inputs(B, Hq, Hkv, n, dt, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    q = torch.randn((B, Hq, 128), generator=g, device=DEV).to(dt)
    k = torch.randn((B, Hkv, n, 128), generator=g, device=DEV).to(dt)
    v = torch.randn((B, Hkv, n, 128), generator=g, device=DEV).to(dt)
    return q, k, v


def _check(q, k, v, idx, out):
    B, Hq, _ = q.shape
    Hkv = k.shape[1]
    G = Hq // Hkv
    for b in range(B):
        for h in range(Hkv):
            rows = idx[b, h if idx.shape[1] > 1 else 0].long()
            x = q[b, h * G:(h + 1) * G].double() @ k[b, h, rows].double().T / 128 ** 0.5
            vs = v[b, h, rows].double()
            ref = torch.softmax(x, -1) @ vs
            err = (out[b, h * G:(h + 1) * G].double() - ref).abs().max()
            assert err <= (128 + rows.numel()) * 2.0 ** -24 * vs.abs().max(), "b %d head %d: %.3g" % (b, h, err)


@pytest.mark.parametrize("G", [3, 5, 6, 7, 8, 9, 12, 20])
@pytest.mark.parametrize("how", ["step", "raw", "sketch", "kvhead", "streamed", "gather"])
@pytest.mark.parametrize("n", [1500, 4500])   # one launch for a short row; chunks selected and attended by topk_emit
def test_group_sizes(G, how, n):
    import paper_2602_18750_amd as H
    B, Hkv, ks = 2, 2, 250
    dt = torch.float16 if G % 2 else torch.bfloat16
    q, k, v = _inputs(B, G * Hkv, Hkv, n, dt, G)
    R = Hkv if how == "kvhead" else 1
    s = H.new_importance(B, R, n, DEV)
    if how == "gather":
        idx = torch.stack([torch.randperm(n, device=DEV)[:ks] for _ in range(B)]).view(B, 1, ks).int().contiguous()
        out = H.hill_gather_attn(q, k, v, idx)
    else:
        kw = dict(mode="raw" if how == "raw" else "attn", granularity="kvhead" if how == "kvhead" else "token",
                  sketch=H.sketch_keys(k) if how == "sketch" else None)
        if how == "streamed":
            kw["stream_state"] = H.new_stream_state(B, 1, DEV)
            H.hill_step(q, k, v, s, ks, stream_reset=True, **kw)
        idx, out = H.hill_step(q, k, v, s, ks, **kw)
    torch.cuda.synchronize()
    _check(q, k, v, idx, out)


@pytest.mark.parametrize("crowd", [1, 64, 65, 128, 129, 400])
@pytest.mark.parametrize("mode", ["raw", "sketch"])
def test_crowded_chunk(crowd, mode):
    import paper_2602_18750_amd as H
    B, Hkv, n, ks = 13, 8, 4100, 400      # 9 chunks x 13 x 8 workgroups, 50 entries on average
    q, k, v = _inputs(B, 32, Hkv, n, torch.bfloat16, crowd)
    s = H.new_importance(B, 1, n, DEV)
    s[:, 0, 1030:1030 + crowd] = 1e6      # all of them in one 512-token chunk
    idx, out = H.hill_step(q, k, v, s, ks, mode="raw" if mode == "raw" else "attn",
                           sketch=H.sketch_keys(k) if mode == "sketch" else None)
    torch.cuda.synchronize()
    assert int(((idx >= 1024) & (idx < 1536)).sum(-1).min()) >= crowd
    _check(q, k, v, idx, out)
