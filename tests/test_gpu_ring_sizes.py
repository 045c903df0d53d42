"""Rings beyond the sizes of the other tests: dense steps whose pieces span more
than one group of 1024 partitions, the last group ragged (and chunks large
enough for the non-temporal loads), and all-gather hops of two tiles per wave
that forward tiles expanded by the whole block.  Whole outputs, bit for bit."""
import pytest

from helpers import log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def S():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2607_04676_amd as S
    return S


def raw(t):
    return t.view(torch.int16 if t.dtype == torch.bfloat16 else torch.int32)


def filled(n, td, seed, density):
    """Element i nonzero with probability density (a number, or one per tile in turn)."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.randn(n, generator=g, device="cuda")
    d = torch.tensor(density, device="cuda")[(torch.arange(n, device="cuda") // 4096) % len(density)]
    x[torch.rand(n, generator=g, device="cuda") >= d] = 0.0
    x = x.to(td)
    x[raw(x) == (-32768 if td == torch.bfloat16 else -2 ** 31)] = 0.0     # a value rounded to -0.0
    return x


@pytest.mark.parametrize("td", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("adaptive,density", [(2, [0.5]), (1, [0.9]), (1, [0.3])])
def test_ring_of_two_front_groups(S, td, adaptive, density):
    P, m = 2, 1024 * 16384 + 3 * 16384 + 5
    dt = S.SPCCL_BF16 if td == torch.bfloat16 else S.SPCCL_F32
    log(f"ring P={P} m={m} {td} adaptive={adaptive} density={density}")
    x = [filled(P * m, td, 10 + r, density) for r in range(P)]
    recv = [torch.empty_like(x[0]) for _ in range(P)]
    scratch = torch.empty(S.spccl_vr_scratch_bytes(P, m, dt), dtype=torch.uint8, device="cuda").fill_(0xFF)
    tr = S.spccl_vr_all_reduce(x, recv, scratch, S.spccl_policy_t(0.6, 0.5, 0.3, 0, adaptive, S.SPCCL_FMT_PICI))
    # one addition per element, rounded once (both sums are exact in fp32 before rounding to bf16)
    exp = (x[0].float() + x[1].float()).to(td)
    for r in range(P):
        assert torch.equal(raw(recv[r]), raw(exp)), f"rank {r}"
    if density != [0.3]:
        assert any(e[2] == S.SPCCL_FMT_DENSE for e in tr)


@pytest.mark.parametrize("td", [torch.float32, torch.bfloat16])
def test_hops_of_two_tiles_forward_dense_tiles(S, td):
    P, n = 4, 4097 * 4096 + 3
    dt = S.SPCCL_BF16 if td == torch.bfloat16 else S.SPCCL_F32
    log(f"all-gather P={P} n={n} {td}")
    parts = [filled(n, td, 20 + r, [0.01, 0.24, 0.26, 0.6, 1.0, 0.1, 0.5]) for r in range(P)]
    exp = raw(torch.cat(parts))
    scratch = torch.empty(S.spccl_vr_scratch_bytes(P, n, dt), dtype=torch.uint8, device="cuda").fill_(0xFF)
    recv = [torch.full((P * n + 1,), 7.0, dtype=td, device="cuda") for _ in range(P)]
    for off in (0, 1):
        out = [t[off:off + P * n] for t in recv]
        S.spccl_vr_all_gather(parts, out, scratch)
        for r in range(P):
            assert torch.equal(raw(out[r].contiguous()), exp), f"off={off} rank {r}"


@pytest.mark.parametrize("adaptive", [0, 1, 2])
def test_rings_without_a_trace(S, adaptive):
    """The C calls with no trace array: the same results, and status 0."""
    import ctypes
    P, m, dt = 3, 3 * 16384 + 5, S.SPCCL_F32
    x = [filled(P * m, torch.float32, 40 + r, [0.3, 0.01]) for r in range(P)]
    pol = S.spccl_policy_t(0.6, 0.5, 0.3, 0, adaptive, S.SPCCL_FMT_PICI)
    scratch = torch.empty(S.spccl_vr_scratch_bytes(P, P * m, dt), dtype=torch.uint8, device="cuda")
    ptrs = lambda ts: (ctypes.c_void_p * P)(*[t.data_ptr() for t in ts])
    for name, n, out in (("reduce_scatter", P * m, m), ("all_gather", m, P * m), ("all_reduce", P * m, P * m)):
        send = [t[:n] for t in x]
        got, exp = ([torch.full((out,), 7.0, device="cuda") for _ in range(P)] for _ in range(2))
        getattr(S, f"spccl_vr_{name}")(send, exp, scratch, pol)
        st = getattr(S._lib, f"spccl_vr_{name}")(ptrs(send), ptrs(got), P, n, dt, ctypes.byref(pol), scratch.data_ptr(),
                                                 scratch.numel(), None, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert st == 0
        for r in range(P):
            assert torch.equal(raw(got[r]), raw(exp[r])), f"{name} rank {r}"
