"""GPU parity of the expansion around its LDS layouts: tiles with as many
values as one layout holds, one more and one less (1024 and, in bf16, 2048),
in every order of neighbours, alone (decompress, sliced decompress) and while
the message is forwarded (all-gathers), on and off a 128-byte line."""
import numpy as np
import pytest

import workloads as W
from helpers import bits, first_diff, log, to_dev, to_host_bits

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

COUNTS = [1023, 1024, 1025, 2047, 2048, 2049, 41, 0, 4096]


@pytest.fixture(scope="module")
def S():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2607_04676_amd as S
    return S


def neighbours(dtype, tail, seed):
    """Every ordered pair of counts in two neighbouring tiles at an even place (one
    wave's two tiles), then a ragged tile of `tail` elements, half full."""
    counts = [c for a in COUNTS for b in COUNTS for c in (a, b)]
    n = 4096 * len(counts) + tail
    out = W.empty(n, dtype)
    for t, k in enumerate(counts + [tail // 2]):
        m = min(4096, n - 4096 * t)
        out[4096 * t:4096 * t + m] = W.sparse_array(m, k, [83, seed, t], dtype)
    return out


@pytest.mark.parametrize("dtype", [W.F32, W.BF16])
@pytest.mark.parametrize("repeat", [1, 102])
def test_stage_layouts(S, dtype, repeat):
    """repeat 102: enough tiles for two tiles per wave in the gather."""
    dt = S.SPCCL_F32 if dtype == W.F32 else S.SPCCL_BF16
    one = neighbours(dtype, 3001, 0)
    x = np.concatenate([one[:162 * 4096]] * (repeat - 1) + [one])
    n = x.size
    tx, ws = to_dev(x), S.alloc_workspace(n, dt)
    pici, sliced = S.alloc_stream(n, dt), S.alloc_sliced(n, dt)
    S.spccl_compress(tx, pici, ws)
    S.spccl_compress_sliced(tx, sliced, ws)
    for off in (0, 3):
        for what, f, m in (("pici", S.spccl_decompress, pici), ("sliced", S.spccl_decompress_sliced, sliced)):
            log(f"stage layouts {what} {dtype} repeat={repeat} off={off}")
            out = torch.full((n + 64,), 7.0, dtype=tx.dtype, device="cuda")
            f(m, out[off:off + n], ws)
            torch.cuda.synchronize()
            assert S.spccl_read_status(ws) == 0
            got = to_host_bits(out[off:off + n])
            assert np.array_equal(got, bits(x)), first_diff(got, bits(x))
            assert bool((out[off + n:] == 7.0).all()) and bool((out[:off] == 7.0).all())


@pytest.mark.parametrize("dtype", [W.F32, W.BF16])
@pytest.mark.parametrize("form", ["pici", "sliced"])
def test_forwarded_layouts(S, dtype, form):
    """Three hops over four ranks: what a hop writes on is expanded by the next."""
    dt, P = (S.SPCCL_F32 if dtype == W.F32 else S.SPCCL_BF16), 4
    parts = [neighbours(dtype, 3001, r) for r in range(P)]
    n = parts[0].size
    log(f"forwarded layouts {form} {dtype} n={n}")
    send = [to_dev(p) for p in parts]
    recv = [torch.full((P * n,), 7.0, dtype=send[0].dtype, device="cuda") for _ in range(P)]
    if form == "sliced":
        scratch = torch.empty(S.spccl_vr_sliced_scratch_bytes(P, n, dt), dtype=torch.uint8, device="cuda")
        S.spccl_vr_all_gather_sliced(send, recv, scratch)
    else:
        scratch = torch.empty(S.spccl_vr_scratch_bytes(P, n, dt), dtype=torch.uint8, device="cuda")
        S.spccl_vr_all_gather(send, recv, scratch, S.spccl_policy_t(0.6, 0.5, 0.1, 0, 1, S.SPCCL_FMT_PICI))
    torch.cuda.synchronize()
    exp = np.concatenate([bits(p) for p in parts])
    for r in range(P):
        got = to_host_bits(recv[r])
        assert np.array_equal(got, exp), f"rank {r}: {first_diff(got, exp)}"
