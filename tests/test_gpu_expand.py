"""GPU parity of the expansion's line-wise stores: outputs that start anywhere
in a 128-byte line, lengths around its 4 KiB units and tiles, runs of sparse
and dense tiles next to each other (values staged together, tile by tile, or
by column groups), for Pici, COO and sliced messages in both dtypes.  The
elements around the output must keep their values."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from helpers import bits, first_diff, log, to_dev, to_host_bits

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

GUARD = 128


@pytest.fixture(scope="module")
def S():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2607_04676_amd as S
    return S


def mixed(n, dtype, seed):
    """Tiles of alternating density: empty, sparse, around the stage's limits, full."""
    out = W.empty(n, dtype)
    dens = [0.01, 0.1, 0.2495, 0.2505, 0.0, 0.6, 0.01, 1.0, 0.5]
    for t, lo in enumerate(range(0, n, 4096)):
        k = min(4096, n - lo)
        out[lo:lo + k] = W.sparse_array(k, int(round(k * dens[(t + seed) % len(dens)])), [77, seed, t], dtype)
    return out


# one unit and around it, tile edges, several waves' runs
SIZES = [1, 63, 1023, 1025, 2047, 2049, 4095, 4097, 3 * 4096 + 1, 9 * 4096 - 5, 41 * 4096 + 77]


@pytest.mark.parametrize("dtype", [W.F32, W.BF16])
@pytest.mark.parametrize("fmt", ["pici", "coo", "sliced"])
def test_unaligned_outputs(S, dtype, fmt):
    dt = S.SPCCL_F32 if dtype == W.F32 else S.SPCCL_BF16
    line = 32 if dtype == W.F32 else 64                  # elements of a 128-byte line
    for n in SIZES:
        x = mixed(n, dtype, n % 9)
        ws = S.alloc_workspace(n, dt)
        tx = to_dev(x)
        if fmt == "sliced":
            msg = S.alloc_sliced(n, dt)
            S.spccl_compress_sliced(tx, msg, ws, 0.45)   # some slices dense
        else:
            msg = S.alloc_stream(n, dt, fmt=S.SPCCL_FMT_COO if fmt == "coo" else S.SPCCL_FMT_PICI)
            (S.spccl_compress_coo if fmt == "coo" else S.spccl_compress)(tx, msg, ws)
        for off in (0, 1, 3, 8, line // 2 + 1, line - 1):
            log(f"expand {fmt} {dtype} n={n} off={off}")
            big = torch.full((n + 2 * GUARD,), 7.0, dtype=tx.dtype, device="cuda")
            lo = 64 + off
            out = big[lo:lo + n]
            if fmt == "sliced":
                S.spccl_decompress_sliced(msg, out, ws)
            else:
                S.spccl_decompress(msg, out, ws)
            torch.cuda.synchronize()
            assert S.spccl_read_status(ws) == 0
            got = to_host_bits(big)
            exp = to_host_bits(torch.full((n + 2 * GUARD,), 7.0, dtype=tx.dtype))
            exp[lo:lo + n] = bits(x)
            assert np.array_equal(got, exp), f"n={n} off={off}: {first_diff(got, exp)}"


@pytest.mark.parametrize("dtype", [W.F32, W.BF16])
def test_gather_of_odd_parts(S, dtype):
    """Parts of odd length: every part but the first starts inside a line; two
    tiles per wave (the size where the launch switches) as well as one."""
    dt = S.SPCCL_F32 if dtype == W.F32 else S.SPCCL_BF16
    for P, n in [(3, 5 * 4096 + 3), (5, 3413 * 4096 + 1)]:
        log(f"gather P={P} n={n} {dtype}")
        ws = S.alloc_workspace(n, dt)
        xs, ops = [], []
        for q in range(P):
            x = to_dev(mixed(9 * 4096, dtype, q)).repeat(-(-n // (9 * 4096)))[:n].contiguous()
            m = S.alloc_stream(n, dt)
            (S.spccl_encode_dense(x, m) if q == 1 else S.spccl_compress(x, m, ws))
            xs.append(x)
            ops.append(S.operand(m, S.SPCCL_STREAM, S.SPCCL_FMT_DENSE if q == 1 else S.SPCCL_FMT_PICI))
        out = torch.full((P * n,), 7.0, dtype=xs[0].dtype, device="cuda")
        S.spccl_gather_expand(ops, n, dt, out, ws)
        torch.cuda.synchronize()
        assert S.spccl_read_status(ws) == 0
        it = torch.int32 if dtype == W.F32 else torch.int16
        assert torch.equal(out.view(it), torch.cat(xs).view(it))
