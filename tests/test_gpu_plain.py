"""The tiled products on ragged sizes, at token counts where each tiling of the
2:4 product (128 x 128, 256 x 128, 256 x 256) and of the dense ones is chosen:
small integers, whose sums are exact in any order, so that every output is equal
to the product in 64 bits, rounded once."""
import pytest
import torch

import paper_2605_03667_amd as elas

pytestmark = pytest.mark.gpu


def _ints(shape, seed, hi=3):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.randint(0, hi, shape, generator=g, device="cuda").to(torch.bfloat16)


@pytest.mark.parametrize("M,K,N", [(130, 200, 136), (4099, 328, 504), (9001, 200, 520), (16500, 264, 512),
                                   (33001, 136, 256), (65537, 72, 264),
                                   # 256 x 128 tiles with 128 K per step: a half step, one step and a half
                                   (9001, 40, 520), (9001, 136, 520), (15001, 264, 512)])
@pytest.mark.parametrize("layout", [elas.ELAS_B_KN, elas.ELAS_B_NK])
def test_spmm_ragged(M, K, N, layout):
    h = _ints((M, K), M)
    b = _ints((K, N) if layout == elas.ELAS_B_KN else (N, K), N) - 1
    vals, meta = elas.elas_sparsify_24(h, elas.ELAS_SPARSIFY_RAW)
    # the kept entries back in their places
    code = torch.stack((meta & 0xF, meta >> 4), -1).reshape(M, -1)[:, : K // 4].long()
    kept = vals[:, : K // 2].reshape(M, -1, 2)
    s = torch.zeros((M, K // 4, 4), device="cuda", dtype=torch.float64)
    s.scatter_(2, torch.stack((code & 3, code >> 2), -1), kept.double())
    ref = s.reshape(M, K) @ (b if layout == elas.ELAS_B_KN else b.t()).double()
    assert ref.abs().max() <= 2 ** 24
    assert torch.equal(elas.elas_spmm_24(vals, meta, K, b, layout), ref.float().to(torch.bfloat16))


@pytest.mark.parametrize("T,d,F", [(1, 8, 8), (130, 72, 264), (4099, 328, 504), (9001, 264, 136), (33001, 136, 72)])
def test_fullrank_ragged(T, d, F):
    x, w_up, w_down = _ints((T, d), 1) - 1, _ints((F, d), 2) - 1, _ints((d, F), 3) - 1
    h = (x.double() @ w_up.t().double()).clamp_min(0)
    s = (h ** 2).float().to(torch.bfloat16)
    y = s.double() @ w_down.t().double()
    assert h.max() <= 256 and y.abs().max() < 2 ** 24
    o = elas.elas_fullrank_ffn_fwd(x, w_up, w_down)
    assert torch.equal(o["S"], s)
    assert torch.equal(o["y"], y.float().to(torch.bfloat16))
