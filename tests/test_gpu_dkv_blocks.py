"""The VaSE-DKV score's split of an instance into blocks of 32-row tiles: at the edges
of tiles, waves and blocks, against the definition in float64."""
import pytest
import torch

from paper_2606_03928_amd import vase

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.fixture(autouse=True)
def _lib(gpu_lib):
    yield
    torch.cuda.synchronize()


@pytest.mark.parametrize("n,K,B,d,G,r", [
    (1, 1, 1, 64, 1, 1), (2, 32, 1, 128, 16, 32), (3, 127, 1, 128, 4, 20), (1, 129, 31, 64, 5, 8),
    (8, 2000, 177, 128, 8, 20),          # blocks of four tiles
    (400, 1030, 10, 64, 2, 31),          # two blocks, the second one tile shorter
    (800, 1100, 5, 128, 3, 17),          # one block, waves with unequal tiles
])
def test_dkv_score_blocks(n, K, B, d, G, r):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(n + K)
    k, v = (torch.randn((n, K + B, d), generator=gen, device=DEV).bfloat16() for _ in range(2))
    q = torch.randn((n, G, d), generator=gen, device=DEV).bfloat16()
    g = vase.dkv_projection(n, d, 7, 3, r=r)
    plain = vase.dkv_score(k, v, g, K, B)
    logits = torch.full((n, G, K + B), float("nan"), device=DEV)
    score = vase.dkv_score(k, v, g, K, B, q_dec=q, dec_logits=logits)
    assert torch.equal(plain, score)
    kd, vd = k[:, :K].double(), v[:, :K].double()
    want = torch.bmm(kd, g.double()).square().sum(-1) * torch.bmm(vd, g.double()).square().sum(-1)
    # every projection is off by at most (2^-16 + (d + 1) 2^-23) sum |g k| (the bf16
    # pair of G, two fp32 sums), a squared norm by twice that over its root sum of
    # squares; the product adds the two
    eps = 2.0 ** -16 + (d + 1) * 2.0 ** -23
    rel = sum(2 * eps * torch.bmm(x.abs(), g.double().abs()).norm(dim=-1) /
              torch.bmm(x, g.double()).norm(dim=-1) for x in (kd, vd)) + (r + 4) * 2.0 ** -23
    assert ((score.double() - want).abs() <= 1.5 * rel * want).all()
    ld = torch.bmm(q.double(), k.double().transpose(1, 2).contiguous())
    ab = torch.bmm(q.double().abs(), k.double().abs().transpose(1, 2).contiguous())
    assert ((logits.double() - ld).abs() <= (d + 1) * 2.0 ** -24 * ab).all()


@pytest.mark.parametrize("n,K,B,d,r", [
    (1, 1, 1, 64, 1), (2, 33, 1, 128, 32), (8, 2000, 48, 64, 20), (400, 1030, 10, 128, 31),
    (800, 1100, 5, 64, 17),
])
def test_dkv_score_f32_blocks(n, K, B, d, r):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(n + K)
    k, v = (torch.randn((n, K + B, d), generator=gen, device=DEV) for _ in range(2))
    g = vase.dkv_projection(n, d, 7, 3, r=r)
    score = vase.dkv_score(k, v, g, K, B)
    kd, vd = k[:, :K].double(), v[:, :K].double()
    want = torch.bmm(kd, g.double()).square().sum(-1) * torch.bmm(vd, g.double()).square().sum(-1)
    # as above with one fp32 sum per projection
    eps = (d + 1) * 2.0 ** -24
    rel = sum(2 * eps * torch.bmm(x.abs(), g.double().abs()).norm(dim=-1) /
              torch.bmm(x, g.double()).norm(dim=-1) for x in (kd, vd)) + (r + 4) * 2.0 ** -23
    assert ((score.double() - want).abs() <= 1.5 * rel * want).all()
    # an infinite element makes its row's score infinite, not a NaN of the padding
    k[0, 0, d - 1] = float("inf")
    assert vase.dkv_score(k, v, g, K, B)[0, 0].item() == float("inf")


@pytest.mark.parametrize("n,K,B,d,G,r", [
    (200, 2300, 10, 64, 2, 20),          # more than 32 tiles a block: blocks of 8 tiles, the last of one
    (385, 2049, 15, 64, 1, 8),           # two blocks would do without the last tile
    (384, 2100, 12, 64, 3, 32),          # the last number of instances with whole rounds of blocks
])
def test_dkv_score_short_blocks(n, K, B, d, G, r):
    test_dkv_score_blocks(n, K, B, d, G, r)


@pytest.mark.parametrize("n,K,B,d,r", [(512, 700, 3, 64, 8), (511, 700, 3, 64, 20)])
def test_dkv_score_f32_rounds(n, K, B, d, r):
    # two rounds of blocks from 512 instances on
    test_dkv_score_f32_blocks(n, K, B, d, r)
