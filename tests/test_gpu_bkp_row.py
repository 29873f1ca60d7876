"""The one-launch pool pass (rows of up to 16384 tokens whose tables allow
vector accesses) against the six-launch pass, which tables with odd strides
take: the same hits, pool bytes, lists and counts over several passes, at the
edges of the groups of eight tokens per access, of the tokens per thread and
of the longest row; saturated counts, pool bytes with stray bits, truncated
lists, no selected tokens, an all-window pool; nothing past the context is
touched."""
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


@pytest.mark.parametrize("B,R,n,k,w,cap,list_cap", [
    (1, 1, 1, 1, 0, 1, 1),
    (2, 3, 7, 3, 1, 4, 7),
    (1, 2, 9, 4, 0, 5, 9),
    (3, 1, 1021, 200, 64, 400, 400),
    (1, 4, 8191, 800, 0, 1600, 100),
    (1, 1, 8192, 0, 819, 1638, 1638),
    (2, 1, 8193, 8193, 100, 3000, 3000),
    (1, 2, 16011, 2000, 2001, 2001, 2001),       # the window fills the pool
    (1, 1, 16377, 3000, 3000, 40000, 16377),     # the pool holds everything
    (2, 1, 16384, 1638, 1638, 3276, 3276),
    (1, 1, 16385, 1638, 1638, 3276, 3276),       # past the limit: six launches both times
])
def test_one_launch_equals_six(B, R, n, k, w, cap, list_cap):
    import paper_2602_18750_amd as H
    g = torch.Generator(device=DEV).manual_seed(n + k)
    ld = (n + 15) // 8 * 8
    a, b = H.BkpState(B, R, ld, DEV), H.BkpState(B, R, ld + 1, DEV)   # odd strides: the six launches
    hits = torch.randint(0, 5, (B, R, ld), generator=g, device=DEV, dtype=torch.int16)
    hits[torch.rand((B, R, ld), generator=g, device=DEV) < 0.05] = -1   # 65535
    hot = torch.randint(0, 256, (B, R, ld), generator=g, device=DEV, dtype=torch.uint8)
    for st in (a, b):
        st.hits[:, :, :ld] = hits
        st.hot[:, :, :ld] = hot
    for step in range(3):
        idx = None
        if k:
            idx = torch.stack([torch.randperm(n, generator=g, device=DEV)[:k] for _ in range(B * R)])
            idx = idx.view(B, R, k).int().contiguous()
        kw = dict(n_tokens=n, n_recent=w, capacity=cap, list_cap=list_cap)
        pa, da, ca = H.bkp_update(a, idx, **kw)
        pb, db, cb = H.bkp_update(b, idx, **kw)
        torch.cuda.synchronize()
        assert torch.equal(ca, cb), "step %d" % step
        assert torch.equal(a.hits[:, :, :ld], b.hits[:, :, :ld]) and torch.equal(a.hot[:, :, :ld], b.hot[:, :, :ld])
        assert torch.equal(a.hits[:, :, n:], hits[:, :, n:]) and torch.equal(a.hot[:, :, n:], hot[:, :, n:])
        for i in range(B):
            for r in range(R):
                np_, nd = (min(int(x), list_cap) for x in ca[i, r])
                assert torch.equal(pa[i, r, :np_], pb[i, r, :np_]) and torch.equal(da[i, r, :nd], db[i, r, :nd])
