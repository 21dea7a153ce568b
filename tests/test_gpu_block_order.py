"""The per-die block order of the averaging kernel (order = 1) covers every work item, also when
their number is not a multiple of the 8 dies."""
import time

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


@pytest.mark.parametrize("M,P,call", [(32, 3_907, "full"), (32, 3_904, "full"), (24, 6_945, "full"), (16, 15_625, "full"),
                                      (16, 390_625, "chunks"), (24, 200_001, "chunks")])
def test_default_order_of_small_states_and_part_filled_lists(M, P, call):
    """States of up to 24 MiB have too few work items to deal out in eighths, and the list of a
    chunk-index round ends in empty groups: the plain order takes 2/3 of the time or less."""
    X = torch.randn(M * M, P, device=DEV)
    print(f"default order M={M} P={P} {call}", flush=True)

    with binding.Moshpit(M * M, P, M, 2, binding.F32) as m:
        m.bind_state(X)

        def once(order):
            m.set_tuning(order=order)
            m.sync()
            start = time.perf_counter()
            for t in range(16):
                m.round(t) if call == "full" else m.dynamic_round(t, 7)
            m.sync()
            return time.perf_counter() - start

        runs = [(once(-1), once(0)) for _ in range(12)][2:]
    default, plain = (min(r[k] for r in runs) for k in (0, 1))
    print(f"  default {default / 16 * 1e6:.1f} us, plain {plain / 16 * 1e6:.1f}", flush=True)
    assert default <= 1.2 * plain
