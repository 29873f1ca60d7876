"""The order in which a short row's attention adds its partial sums.

V lies in [1, 1.25), so that the rounding of the weights cancels in the
weighted mean and what is left of the output's error is that of the two long
sums (the weighted V and the softmax normaliser).  The same sums are formed
here in fp32, every partial as the kernel forms it (an entry in the lane group
e % P of P = 16 waves times the rows a wave loads at once; the normaliser's in
waves of 64), and the partials then added pairwise.  The GPU's error may exceed
that by what the weights still contribute: their relative rounding of about
2^-22 (logits up to 8 in fp32, exp2) times V's spread of 0.07 over the root of
the effective entries, below 2^-27.  One after another the partials would miss
the bound by a factor of 1.5 and more, which is checked too."""
import numpy as np
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


def _rms(x):
    return float(np.sqrt(np.mean(np.square(x))))


def _pairwise(p):
    while p.shape[-1] > 1:
        h = p.shape[-1] // 2
        p = p[..., :h] + p[..., h:]
    return p[..., 0]


def _serial(p):
    t = np.zeros_like(p[..., 0])
    for i in range(p.shape[-1]):
        t = t + p[..., i]
    return t


def _sums(w, v, parts):
    """fp32 partial sums [head, dim, parts] of w [head, k] times v [k, dim]."""
    p = np.zeros((w.shape[0], v.shape[1], parts), dtype=np.float32)
    for e0 in range(0, w.shape[1], parts):
        n = min(parts, w.shape[1] - e0)
        term = w[:, None, e0:e0 + n].astype(np.float64) * v.T[None, :, e0:e0 + n]
        p[:, :, :n] = (p[:, :, :n].astype(np.float64) + term).astype(np.float32)   # a fused multiply-add
    return p


def _norm(w):
    """fp32 normaliser partials [head, 16]: entry t in wave t / 64."""
    k = w.shape[1]
    x = np.zeros((w.shape[0], 1024), dtype=np.float32)
    x[:, :k] = w
    return _pairwise(x.reshape(-1, 16, 64))


@pytest.mark.parametrize("Hq,Hkv,B,n,ks,parts", [
    (32, 8, 1, 1021, 204, 64),       # half of V's line per workgroup: four rows per load
    (32, 32, 1, 4096, 819, 64),
    (32, 32, 8, 4096, 819, 32),      # whole rows of V: two per load
    (64, 8, 1, 2048, 1000, 64),
])
def test_partial_sums_are_added_pairwise(Hq, Hkv, B, n, ks, parts):
    import paper_2602_18750_amd as H
    g = torch.Generator(device=DEV).manual_seed(n + ks)
    dt = torch.float16
    q = torch.randn((B, Hq, 128), generator=g, device=DEV).to(dt)
    k = torch.randn((B, Hkv, n, 128), generator=g, device=DEV).to(dt)
    v = (1.0 + 0.25 * torch.rand((B, Hkv, n, 128), generator=g, device=DEV)).to(dt)
    s = H.new_importance(B, 1, n, DEV)
    idx, out = H.hill_step(q, k, v, s, ks)
    torch.cuda.synchronize()
    err, pair, serial = [], [], []
    G = Hq // Hkv
    for b in range(min(B, 2)):
        rows = idx[b, 0].long()
        for h in range(Hkv):
            x = (q[b, h * G:(h + 1) * G].double() @ k[b, h, rows].double().T / 128 ** 0.5).cpu().numpy()
            w = np.exp(x - x.max(-1, keepdims=True))
            vs = v[b, h, rows].double().cpu().numpy()
            ref = (w / w.sum(-1, keepdims=True)) @ vs
            err.append(out[b, h * G:(h + 1) * G].double().cpu().numpy() / ref - 1)
            w32 = w.astype(np.float32)
            ref32 = (w32.astype(np.float64) @ vs) / w32.astype(np.float64).sum(-1, keepdims=True)
            po, pl = _sums(w32, vs, parts), _norm(w32)
            pair.append(_pairwise(po) / _pairwise(pl)[:, None] / ref32 - 1)
            serial.append(_serial(po) / _serial(pl)[:, None] / ref32 - 1)
    err, pair, serial = _rms(err), _rms(pair), _rms(serial)
    print("rms error %.3g, pairwise %.3g, serial %.3g" % (err, pair, serial))
    bound = 1.15 * pair + 2.0 ** -27
    assert err <= bound < serial, (err, pair, serial)
