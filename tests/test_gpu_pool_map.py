"""The pooling launch that also applies an order map (vase_score_map when the slots
or the window rows of an instance are split over workgroups): bit for bit the
unpooled per-slot scores put through vase_order_scores, at the edges of its
candidates per thread, with the widest filter and with one candidate."""
import pytest
import torch

from paper_2606_03928_amd import vase

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.fixture(autouse=True)
def _lib(gpu_lib):
    yield
    torch.cuda.synchronize()


SIZES = [(1, 255), (255, 1), (257, 7), (2048, 255), (2049, 7), (8191, 31), (8192, 7)]


# the launch does not depend on the cache type; the small sizes cover fp32
@pytest.mark.parametrize("K,pool,dtype,rows", [
    (K, pool, dtype, rows)
    for dtype, rows in ((torch.bfloat16, 24), (torch.bfloat16, 700), (torch.float32, 24))
    for K, pool in SIZES if dtype == torch.bfloat16 or K <= 2049])
def test_pooling_through_the_map(K, pool, dtype, rows):
    _check(3, K, pool, dtype, rows)


@pytest.mark.parametrize("n,K,pool,rows", [
    # beyond 2^19 candidates one workgroup holds an instance: the last call of the
    # other launch, four and sixteen waves, candidates per thread that do not divide
    (64, 8192, 31, 24), (65, 8192, 255, 24), (65, 8191, 7, 24), (257, 2048, 7, 24),
    (257, 2049, 1, 24), (600, 1001, 13, 520), (2100, 255, 255, 520)])
def test_pooling_of_many_candidates(n, K, pool, rows):
    _check(n, K, pool, torch.bfloat16, rows)


def _check(n, K, pool, dtype, rows):
    B, d = 9, 64
    g = torch.Generator(device="cpu")
    g.manual_seed(K + pool + rows)
    k, v = (torch.randn((n, K + B, d), generator=g).to(dtype).to(DEV) for _ in range(2))
    q = torch.randn((n, 1, rows, d), generator=g).to(dtype).to(DEV)
    ord_map = torch.stack([torch.randperm(K, generator=g) for _ in range(n)]).int().to(DEV)
    attn, vr = vase.score(k, v, q, K, B, pool, ord=ord_map)
    slot_attn, slot_vr = vase.score(k, v, q, K, B, 1)
    want, want_vr = vase.order_scores(slot_attn, ord_map, pool, vrange_phys=slot_vr)
    assert torch.equal(attn, want)
    assert torch.equal(vr, want_vr)
    # without value scores
    only, _ = vase.score(k, v, q, K, B, pool, ord=ord_map, value_kind=vase.VALUE_SKIP)
    assert torch.equal(only, want)
