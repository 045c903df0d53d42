"""Dense (+) Pici where the merge changes its form with the tile's number of
Pici values: read early (up to 512), merged through a unit of LDS beside the
staged values (up to 768 fp32 or 1536 bf16), row by row from the stage (up to
1792 or 3584), by groups of columns above; each limit, one below and one past
it, and the empty and full tile.  Into a Pici message, a dense array and, for a
sliced operand, a dense array, bit for bit against the oracle.  Where the Pici
operand is absent the dense value passes unchanged: -0.0, NaN, infinities and
subnormals among them."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from helpers import assert_bytes_equal, bits, first_diff, log, to_dev, to_host_bits

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

TILE = 4096
LIMITS = {W.F32: (512, 768, 1792), W.BF16: (512, 1536, 3584)}


@pytest.fixture(scope="module")
def S():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2607_04676_amd as S
    return S


def operands(dtype):
    """a: dense, half full, with special values where b is absent; b: tiles of the counts above."""
    counts = [0, 1, TILE - 1, TILE] + [k + d for k in LIMITS[dtype] for d in (-1, 0, 1)]
    n = len(counts) * TILE
    rng = np.random.default_rng(17)
    a, b = W.sparse_array(n, n // 2, [95, 0], dtype), W.empty(n, dtype)
    for t, k in enumerate(counts):
        b[t * TILE: (t + 1) * TILE] = W.sparse_array(TILE, k, [95, 1, t], dtype)
    for t, k in enumerate(counts):
        assert np.count_nonzero(bits(b[t * TILE: (t + 1) * TILE])) == k
    special = [0x80000000, 0x7FC00001, 0xFF800000, 0x7F800000, 0x00000001, 0x807FFFFF]
    if dtype == W.BF16:
        special = [0x8000, 0x7FC1, 0xFF80, 0x7F80, 0x0001, 0x807F]
    free = np.flatnonzero(bits(b) == 0)
    pick = rng.choice(free, size=free.size // 8, replace=False)
    bits(a)[pick] = np.resize(np.array(special, bits(a).dtype), pick.size)
    both = np.flatnonzero((bits(a) != 0) & (bits(b) != 0))
    sign = bits(a).dtype.type(0x8000 if dtype == W.BF16 else 0x80000000)
    cancel = both[::7]
    bits(b)[cancel] = bits(a)[cancel] ^ sign
    return a, b, n


@pytest.mark.parametrize("dtype", [W.F32, W.BF16])
@pytest.mark.parametrize("out", ["pici", "pici_two_passes", "dense", "sliced_to_dense"])
@pytest.mark.parametrize("order", ["dense_pici", "pici_dense"])
def test_counts_around_each_form(S, dtype, out, order):
    dt = O.BF16 if dtype == W.BF16 else O.F32
    a, b, n = operands(dtype)
    mb = O.compress(b)[0]
    oa, ob = O.Operand.array(a), O.Operand.stream(mb)
    first, second = (oa, ob) if order == "dense_pici" else (ob, oa)
    log(f"merge edges {dtype} {out} {order}")
    ws = S.alloc_workspace(n, dt)
    ta, tm = to_dev(a), torch.from_numpy(mb).cuda()
    pici = lambda t: S.operand(t, S.SPCCL_STREAM, S.SPCCL_FMT_PICI)
    x, y = (S.operand(ta), pici(tm)) if order == "dense_pici" else (pici(tm), S.operand(ta))
    if out.startswith("pici"):
        exp, _ = O.reduce(first, second, n, dt, O.STREAM, O.FMT_PICI)
        got = S.alloc_stream(n, dt).fill_(0x5A)
        prev = S.spccl_set_single_pass_limit(0 if out == "pici_two_passes" else 0xFFFFFFFF)
        try:
            S.spccl_reduce(x, y, pici(got), n, dt, ws)
            torch.cuda.synchronize()
        finally:
            S.spccl_set_single_pass_limit(prev)
        assert S.spccl_read_status(ws) == 0
        assert_bytes_equal(got[:exp.size].cpu().numpy(), exp, f"{out} {order}")
        return
    exp = bits(O.reduce(first, second, n, dt, O.ARRAY))
    got = torch.full((n + 64,), 7.0, dtype=ta.dtype, device="cuda")
    for off in (0, 3):
        to = got[off:off + n]
        if out == "dense":
            S.spccl_reduce(x, y, S.operand(to), n, dt, ws)
        else:
            sl = S.alloc_sliced(n, dt)
            S.spccl_compress_sliced(to_dev(b), sl, ws)
            S.spccl_reduce_sliced(ta, sl, to, ws, out_sliced=False)
        torch.cuda.synchronize()
        assert S.spccl_read_status(ws) == 0
        assert np.array_equal(to_host_bits(to), exp), f"off={off}: {first_diff(to_host_bits(to), exp)}"
