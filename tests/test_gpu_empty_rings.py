"""Ring collectives over messages of no elements: every one succeeds, writes
nothing to the outputs, and reports the sends of empty chunks (sparsity 1),
whatever the scratch held before the call."""
import ctypes

import pytest

import oracle as O
from helpers import log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def S():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2607_04676_amd as S
    return S


@pytest.mark.parametrize("dt", [0, 1])
@pytest.mark.parametrize("P", [1, 2, 3, 4, 33])
@pytest.mark.parametrize("fmt,adaptive", [(1, 0), (1, 1), (1, 2), (2, 0), (2, 2)])
def test_collectives_of_no_elements(S, dt, P, fmt, adaptive):
    pol = S.spccl_policy_t(0.6, 0.5, 0.1, 0, adaptive, fmt)
    td = torch.bfloat16 if dt else torch.float32
    # a real address for every rank: an element beside the (empty) array
    bufs = torch.full((2 * P, 64), 7.0, dtype=td, device="cuda")
    send = (ctypes.c_void_p * P)(*[bufs[r].data_ptr() for r in range(P)])
    recv = (ctypes.c_void_p * P)(*[bufs[P + r].data_ptr() for r in range(P)])
    stream = torch.cuda.current_stream().cuda_stream
    scratch = torch.empty(S.spccl_vr_scratch_bytes(P, 0, dt), dtype=torch.uint8, device="cuda")
    rs, ag = P * (P - 1), P
    for name, count in (("spccl_vr_reduce_scatter", rs), ("spccl_vr_all_gather", ag), ("spccl_vr_all_reduce", rs + ag)):
        for fill in (0xFF, 0x00):
            log(f"{name} n=0 P={P} dt={dt} fmt={fmt} adaptive={adaptive} scratch={fill:#x}")
            scratch.fill_(fill)
            tr = (S.spccl_trace_t * max(count, 1))()
            st = getattr(S._lib, name)(send, recv, P, 0, dt, ctypes.byref(pol), scratch.data_ptr(), scratch.numel(), tr,
                                       stream)
            torch.cuda.synchronize()
            assert st == 0, S.spccl_status_string(st)
            assert bool((bufs == 7.0).all())
            gather_only = name == "spccl_vr_all_gather"                  # which does not densify
            steps = [0] * P if gather_only else [k for k in range(P - 1) for _ in range(P)] + [P - 1] * (count - rs)
            for i in range(count):
                assert (tr[i].step, tr[i].rank) == (steps[i], i % P)
                assert tr[i].fmt == (0 if adaptive == 2 and not gather_only else fmt)
                assert tr[i].sigma == 1.0 and tr[i].nnz in (0, O.NNZ_UNKNOWN)
