"""The window score where an instance's slots, runs or row slabs are split over
workgroups: every way the plan splits a call, against the definition in float64.

Each score is a mean of softmax terms computed in fp32 (exp2 within 1 ulp, a sum
of at most 2^15 non-negative terms in fixed trees, an fp32 logarithm of the
normaliser), so 2e-5 of the largest score bounds the difference with room."""
import math

import pytest
import torch

from paper_2606_03928_amd import vase

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.fixture(autouse=True)
def _lib(gpu_lib):
    yield
    torch.cuda.synchronize()


def _reference(k, v, q, K, pool):
    n, G, w, d = q.shape
    s = torch.bmm(q.double().reshape(n, G * w, d), k.double().transpose(1, 2).contiguous())
    s = s / math.sqrt(d)
    p = torch.softmax(s, -1)[:, :, :K].mean(1)
    p = torch.nn.functional.pad(p, (pool // 2, pool // 2)).unfold(1, pool, 1).sum(-1) / pool
    lse = torch.logsumexp(s[:, :, :K], -1).view(n, G, w).float()
    vd = v[:, :K].double()
    return p, lse, (vd.amax(-1) - vd.amin(-1)).float()


BF, F32 = torch.bfloat16, torch.float32


@pytest.mark.parametrize("dtype,n,K,B,d,G,w", [
    # bf16: one range although the chip is not full, ranges of one chunk, ranges
    # that do not divide, partials merged four at a time with 1 to 3 left over
    (BF, 400, 96, 8, 64, 2, 16), (BF, 1, 33, 1, 128, 1, 1), (BF, 3, 2000, 77, 128, 4, 65),
    (BF, 8, 545, 32, 64, 8, 33), (BF, 64, 700, 65, 128, 5, 130),
    # fp32: one row, a window one row past a tile and past the rows whose
    # normalisers fit at once, row slabs, runs that do not divide, 24 runs
    (F32, 1, 1, 1, 64, 1, 1), (F32, 2, 31, 2, 128, 3, 11), (F32, 1, 200, 9, 64, 5, 205),
    (F32, 5, 1000, 33, 128, 8, 36), (F32, 40, 127, 64, 64, 1, 97), (F32, 1, 5000, 100, 128, 2, 20),
])
def test_split_scores(dtype, n, K, B, d, G, w):
    g = torch.Generator(device="cpu")
    g.manual_seed(n * K + B + G * w)
    k, v = (torch.randn((n, K + B, d), generator=g).to(dtype).to(DEV) for _ in range(2))
    q = torch.randn((n, G, w, d), generator=g).to(dtype).to(DEV)
    pool = 3 if K > 3 else 1
    want, lse, want_vr = _reference(k, v, q, K, pool)
    status = torch.zeros(1, dtype=torch.int32, device=DEV)
    for lse_win in (None, lse):
        attn, vr = vase.score(k, v, q, K, B, pool, lse_win=lse_win, status=status)
        err = (attn.double() - want).abs().amax(1) / want.amax(1)
        assert err.max().item() < 2e-5
        # the Range of bf16 rows is exact in fp32, that of fp32 rows one rounding
        assert ((vr - want_vr).abs() <= (0 if dtype == BF else 2 ** -23) * want_vr).all()
    assert status.item() == 0
    # a row fault is seen by whichever workgroup merges the row, a value fault
    # by the one that reads it
    q[n - 1, G - 1, w - 1, d - 1] = float("nan")
    v[n - 1, K - 1, 0] = float("inf")
    vase.score(k, v, q, K, B, pool, status=status)
    assert status.item() == vase.STATUS_ROW_NORM | vase.STATUS_VALUE_ROW


@pytest.mark.parametrize("n,K,B,d,G,w", [
    # logits written from the chunk loop, since staged ones would cost the CU a
    # workgroup: one range, several ranges, d = 64; and staged ones of long and of
    # short ranges
    (350, 1000, 53, 128, 5, 9), (206, 3632, 20, 128, 4, 20), (244, 3001, 18, 64, 7, 18),
    (30, 700, 40, 128, 3, 40), (300, 260, 31, 64, 8, 31),
])
def test_split_scores_with_decode_logits(n, K, B, d, G, w):
    g = torch.Generator(device=DEV)
    g.manual_seed(n + K)
    k, v = (torch.randn((n, K + B, d), generator=g, device=DEV).to(BF) for _ in range(2))
    q = torch.randn((n, G, w, d), generator=g, device=DEV).to(BF)
    qd = torch.randn((n, G, d), generator=g, device=DEV).to(BF)
    ident = vase.identity_order(n, K, DEV)
    logits = torch.full((n, G, K + B), float("nan"), device=DEV)
    a0, v0 = vase.score(k, v, q, K, B, 5, ord=ident)
    a1, v1 = vase.score(k, v, q, K, B, 5, ord=ident, q_dec=qd, dec_logits=logits)
    assert torch.equal(a0, a1) and torch.equal(v0, v1)
    # exact products of bf16 values, d of them summed in fp32
    for i in range(0, n, 64):
        qi, kt = qd[i:i + 64].double(), k[i:i + 64].double().transpose(1, 2).contiguous()
        bound = (d + 1) * 2.0 ** -24 * torch.bmm(qi.abs(), kt.abs())
        assert ((logits[i:i + 64].double() - torch.bmm(qi, kt)).abs() <= bound).all()


@pytest.mark.parametrize("n,K,B,G,w", [
    (520, 1000, 64, 4, 128),     # one workgroup per instance pools by itself
    (8, 2048, 128, 2, 128),      # split ranges
    (30, 600, 40, 5, 130),       # two row slabs
])
def test_first_round_scores(n, K, B, G, w):
    # what a whole round selects from, before sampling enters: to the accuracy of a
    # score call (a round's other outputs hang on which keys were sampled)
    d, pool = 128, 7
    g = torch.Generator(device=DEV)
    g.manual_seed(n + K)
    k, v = (torch.randn((n, K + B, d), generator=g, device=DEV) for _ in range(2))
    k[:, :4] *= 10
    k, v = k.to(BF), v.to(BF)
    q = torch.randn((n, G, w, d), generator=g, device=DEV).to(BF)
    qd = torch.randn((n, G, d), generator=g, device=DEV).to(BF)
    want = torch.cat([_reference(k[i:i + 32], v[i:i + 32], q[i:i + 32], K, pool)[0]
                      for i in range(0, n, 32)])
    r = vase.Round(n, K, B, d, G, w, BF, DEV, layout="map")
    r.run(k, v, q, qd, 16, pool, 7, 0, carry=True)
    err = (r.attn.double() - want).norm() / want.norm()
    # a row's normaliser is up to 2^7 in base 2, so its fp32 logarithm is off by up to
    # 2^-18 and a term by 2^-18 ln 2 = 2.6e-6; the means and sums round far less
    assert err.item() < 3e-6


@pytest.mark.parametrize("n,K,B,G,w,scalar", [
    (24, 130, 53, 4, 53, 3.25e-7), (37, 991, 68, 3, 68, 3.66e-7),
])
def test_f32_scores_with_lse_round_like_scalar_products(n, K, B, G, w, scalar):
    # With the persistent normalisers given, the products' rounding is not cancelled by
    # the normaliser's, so these scores show it most.  `scalar` is the error against
    # float64 (mean of the same 8 inputs) of one thread per row with scalar fma; a
    # tenth more is what the order of the sums may add (one chain of MFMAs: 3.79e-7
    # and 4.20e-7)
    d, pool, errs = 128, 5, []
    for seed in range(8):
        g = torch.Generator(device="cpu")
        g.manual_seed(seed)
        k = torch.randn((n, K + B, d), generator=g).to(DEV)
        k[:, :4] *= 10
        q = torch.randn((n, G, w, d), generator=g).to(DEV)
        want, lse, _ = _reference(k, k, q, K, pool)
        attn, _ = vase.score(k, k, q, K, B, pool, lse_win=lse)
        errs.append(((attn.double() - want).norm() / want.norm()).item())
    assert sum(errs) / len(errs) <= 1.1 * scalar


@pytest.mark.parametrize("n,K,B,d,G,w", [(256, 2000, 48, 128, 5, 64), (128, 3000, 64, 128, 8, 100)])
def test_one_range_is_as_accurate_as_several(n, K, B, d, G, w):
    # A call that might be split but takes one range, with rows that look at the first
    # tokens: a single fp32 sum would round every later term to those tokens' last
    # place (2.6e-7 and 3.3e-7; about 1024 workgroups 2.1e-7)
    g = torch.Generator(device="cpu")
    g.manual_seed(n + K)
    k = torch.randn((n, K + B, d), generator=g)
    k[:, :4] *= 10
    k, q = k.to(BF).to(DEV), torch.randn((n, G, w, d), generator=g).to(BF).to(DEV)
    want = torch.cat([_reference(k[i:i + 16], k[i:i + 16], q[i:i + 16], K, 7)[0]
                      for i in range(0, n, 16)])
    attn, _ = vase.score(k, k, q, K, B, 7)
    err = ((attn.double() - want).norm() / want.norm()).item()
    assert err < 2.25e-7, err
