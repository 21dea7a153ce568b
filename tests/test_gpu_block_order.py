"""The per-die block order of the averaging kernel (order = 1) covers every work item, also when
their number is not a multiple of the 8 dies."""
import pytest
import torch

from paper_2103_03239_amd import binding

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("M,d,P", [(9, 2, 408), (2, 1, 64), (7, 2, 3_000), (16, 2, 2_500), (5, 3, 1_300)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_every_work_item_once(M, d, P, dtype):
    N = M ** d
    gen = torch.Generator(device=DEV)
    gen.manual_seed(P)
    A = torch.randn(N, P, generator=gen, device=DEV).to(dtype)
    B = A.clone()
    print(f"block order M={M} d={d} P={P} {dtype}", flush=True)
    with binding.Moshpit(N, P, M, d, binding.F32 if dtype == torch.float32 else binding.BF16) as m:
        for X, order in ((A, 0), (B, 1)):
            m.bind_state(X)
            m.set_tuning(order=order)
            for t in range(d):
                m.round(t)
        m.sync()
    assert torch.equal(A, B)
