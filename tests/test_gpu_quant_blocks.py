"""The quantiser's row blocks (32 or 64 rows, by the size of the call) at their edges,
on values whose quotients are often exact ties, with non-finite and constant
groups: codes and parameters against the same IEEE operations in torch."""
import pytest
import torch

from paper_2606_03928_amd import vase

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.fixture(autouse=True)
def _lib(gpu_lib):
    yield
    torch.cuda.synchronize()


@pytest.mark.parametrize("n,K", [(1, 1), (3, 31), (2, 33), (2, 65), (2100, 63), (1100, 65)])
@pytest.mark.parametrize("dtype,d,bits,group", [
    (torch.bfloat16, 128, 4, 32), (torch.bfloat16, 64, 8, 64), (torch.bfloat16, 128, 2, 128),
    (torch.float32, 128, 4, 64), (torch.float32, 64, 8, 32),
])
def test_quant_blocks(dtype, d, bits, group, n, K):
    B, Nv = 3, min(K, 5)
    g = torch.Generator(device="cpu")
    g.manual_seed(K + bits)
    x = torch.randint(-60, 61, (n, K + B, d), generator=g).float()
    x[:, ::3] = torch.randn((n, K + B, d), generator=g)[:, ::3]
    x[0, 0, :group] = 1.5
    if K > 2:
        x[0, 1, 3], x[0, 2, group - 1] = float("nan"), float("inf")
    x = x.to(dtype)
    q = vase.quantize(x.to(DEV), K, B, bits, group, Nv=Nv)
    c = x[:, :K].float().unflatten(-1, (d // group, group))
    # fmin and fmax leave a NaN out; a group's codes are 0 unless its step is above 0
    z = torch.where(c.isnan(), torch.inf, c).amin(-1, keepdim=True)
    hi = torch.where(c.isnan(), -torch.inf, c).amax(-1, keepdim=True)
    step = (hi - z) / float(2 ** bits - 1)
    code = torch.where(step > 0, torch.round((c - z) / step), 0.0).nan_to_num(0.0).to(torch.int64)
    code = code.flatten(-2).view(n, K, -1, 8 // bits)
    packed = sum(code[..., i] << (bits * i) for i in range(8 // bits)).to(torch.uint8)
    assert torch.equal(q["codes"].cpu(), packed)
    assert torch.equal(q["params"].cpu().nan_to_num(7.0), torch.cat([step, z], -1).nan_to_num(7.0))
    back = vase.dequantize(q, K, B, bits, group, dtype).cpu()
    want = torch.addcmul(z.double(), code.view(c.shape).double(), step.double()).float().to(dtype).flatten(-2)
    idx = q["hp_idx"].cpu().long()[:, :, None].expand(n, Nv, d)
    want = want.scatter(1, idx, x[:, :K].gather(1, idx))
    # codes of at most 8 bits times a 24-bit step is exact in 64 bits, the sum with z
    # rounds once more than fma only where it is not: one unit of the last place
    tol = 2.0 ** -7 if dtype == torch.bfloat16 else 2.0 ** -22
    ok = (back[:, :K].double() - want.double()).abs() <= tol * want.double().abs()
    assert (ok | ~want.isfinite()).all()
