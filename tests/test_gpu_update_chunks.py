"""The importance update with several chunks per workgroup and the row
histogram in several parts, against the forms they replace.

S of a batch (several chunks per workgroup) must equal, bit for bit, S of its
sequences updated one by one (one chunk per workgroup); the step's selection
must equal the standalone selection of the step's own S (which counts its own
histogram in one part) and that of a step with a stream state.  Shapes: the last workgroup
with fewer chunks, a last chunk of one token, 1, 2 and 4 heads in flight per
wave, 1 to 8 histogram parts, pinned tokens, RAW scores."""
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


@pytest.mark.parametrize("B,Hq,Hkv,n,rows,mode,sink,recent", [
    (1, 32, 8, 4097, "token", "attn", 0, 0),       # 33 workgroups: one part
    (1, 32, 8, 12288, "token", "attn", 0, 0),      # 96: the last size with one
    (1, 32, 8, 12289, "token", "attn", 0, 0),      # 97: two (room for no more)
    (1, 32, 8, 16641, "token", "attn", 4, 64),     # four parts, a last chunk of one token
    (1, 16, 8, 33281, "token", "attn", 0, 0),      # eight parts, 2 heads in flight
    (9, 32, 8, 16385, "token", "attn", 0, 0),      # 129 chunks: two per workgroup, the last with one
    (16, 40, 8, 16200, "token", "attn", 4, 0),     # two per workgroup, 40 heads: two batches
    (3, 28, 4, 20011, "kvhead", "attn", 4, 64),    # 7 heads per row: one in flight
    (2, 64, 8, 40000, "kvhead", "attn", 0, 0),     # 8 heads per row, the statistics launch
    (2, 32, 8, 20000, "token", "raw", 0, 64),      # RAW: one chunk per workgroup, one part
    (2, 32, 8, 9001, "kvhead", "attn", 0, 0),      # several chunks under a streamed bound: 1 head in flight
    (4, 64, 4, 9000, "kvhead", "attn", 4, 0),      # 2
    (16, 16, 4, 9000, "token", "attn", 0, 64),
])
def test_chunks_and_parts(B, Hq, Hkv, n, rows, mode, sink, recent):
    import paper_2602_18750_amd as H
    g = torch.Generator(device=DEV).manual_seed(n)
    q = torch.randn((B, Hq, 128), generator=g, device=DEV).to(torch.bfloat16)
    k = torch.randn((B, Hkv, n, 128), generator=g, device=DEV).to(torch.bfloat16)
    v = torch.randn((B, Hkv, n, 128), generator=g, device=DEV).to(torch.bfloat16)
    R = 1 if rows == "token" else Hkv
    ks = n // 10
    kw = dict(mode=mode, granularity=rows, n_sink=sink, n_recent=recent)
    s, s1, s2 = (H.new_importance(B, R, n, DEV) for _ in range(3))
    s.copy_(torch.exp(torch.randn((B, R, n), generator=g, device=DEV)))
    s1.copy_(s)
    s2.copy_(s)
    idx, out = H.hill_step(q, k, v, s, ks, **kw)
    for b in range(B):
        H.hill_step(q[b:b + 1], k[b:b + 1], v[b:b + 1], s1[b:b + 1], ks, **kw)
    top = H.hill_topk(s, ks, granularity=rows, n_kv_heads=Hkv, n_sink=sink, n_recent=recent)
    torch.cuda.synchronize()
    assert torch.equal(s, s1), "%d tokens differ" % int((s != s1).sum())
    assert torch.equal(idx, top)
    if mode == "attn":
        st = H.new_stream_state(B, R, DEV)
        # the bound from the refine pass, then the streamed selection (calls of more than 196608 tokens, 262144
        # in KV-head rows, take the refine pass again)
        for reset in (True, False):
            i2, o2 = H.hill_step(q, k, v, s2, ks, stream_state=st, stream_reset=reset, **kw)
            if reset:
                torch.cuda.synchronize()
                assert torch.equal(s2, s) and torch.equal(i2, idx) and torch.equal(o2, out)
        H.hill_step(q, k, v, s, ks, **kw)
        top = H.hill_topk(s, ks, granularity=rows, n_kv_heads=Hkv, n_sink=sink, n_recent=recent)
        torch.cuda.synchronize()
        assert torch.equal(s2, s) and torch.equal(i2, top)
