"""The expansion where its launch changes form with the size: fp32 outputs above
64 MiB (rows stored as they are walked) with tiles of every density side by
side, aligned to a line and not, either side of 96 MiB (unaligned outputs go
back to whole lines) and of 128 and 256 MiB (all do, in between), from one message,
several parts, COO, dense and sliced streams; bf16 where a pair of tiles per
wave replaces one.  Whole outputs bit for bit, and the elements around them."""
import pytest

from helpers import log
from test_gpu_ring_sizes import filled, raw

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

MIX = [0.01, 0.1, 0.2495, 0.2505, 0.0, 0.6, 0.01, 1.0, 0.5, 0.12, 0.13]
MIB_F32, MIB_BF16 = 1 << 18, 1 << 19
# fp32: 64 MiB (lines), one element more, a tile more, 96, 128 and 256 MiB and a little more
CASES = [(torch.float32, n) for n in (64 * MIB_F32, 64 * MIB_F32 + 1, 64 * MIB_F32 + 4097, 96 * MIB_F32, 96 * MIB_F32 + 1,
                                      128 * MIB_F32, 128 * MIB_F32 + 3, 256 * MIB_F32 + 5)]
# bf16: 5120 tiles (one per wave), one more (pairs), 10240 (pairs) and one more (one per wave)
CASES += [(torch.bfloat16, 4096 * t - 7) for t in (5120, 5121, 10240, 10241)]


@pytest.fixture(scope="module")
def S():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2607_04676_amd as S
    return S


def check(out, exp, off, what):
    n = exp.numel()
    assert torch.equal(raw(out[off:off + n]), raw(exp)), what
    rest = torch.cat([out[:off], out[off + n:]])
    assert bool((rest == 7.0).all()), what


@pytest.mark.parametrize("td,n", CASES)
def test_forms_by_size(S, td, n):
    dt = S.SPCCL_BF16 if td == torch.bfloat16 else S.SPCCL_F32
    x = filled(n, td, 5, MIX)
    ws = S.alloc_workspace(n, dt)
    out = torch.empty(n + 128, dtype=td, device="cuda")
    for fmt in ("pici", "coo", "dense", "sliced"):
        log(f"expand {fmt} {td} n={n}")
        if fmt == "sliced":
            msg = S.alloc_sliced(n, dt)
            S.spccl_compress_sliced(x, msg, ws, 0.45)               # some slices dense
        else:
            msg = S.alloc_stream(n, dt, fmt=S.SPCCL_FMT_COO if fmt == "coo" else S.SPCCL_FMT_PICI)
            if fmt == "dense":
                S.spccl_encode_dense(x, msg)
            else:
                (S.spccl_compress_coo if fmt == "coo" else S.spccl_compress)(x, msg, ws)
        for off in (0, 1, 64):
            out.fill_(7.0)
            (S.spccl_decompress_sliced if fmt == "sliced" else S.spccl_decompress)(msg, out[off:off + n], ws)
            assert S.spccl_read_status(ws) == 0
            check(out, x, off, f"{fmt} off={off}")
        del msg


@pytest.mark.parametrize("P,n", [(3, 22 * MIB_F32 + 9), (2, 33 * MIB_F32), (5, 30 * MIB_F32 + 1), (4, 66 * MIB_F32)])
def test_parts_stored_by_rows(S, P, n):
    """Totals above 64 MiB: parts that start on a line and parts that do not,
    one of them a dense message and one a plain array."""
    log(f"gather fp32 P={P} n={n}")
    dt, ws = S.SPCCL_F32, S.alloc_workspace(n, S.SPCCL_F32)
    xs = [filled(n, torch.float32, 30 + q, MIX[q:] + MIX[:q]) for q in range(P)]
    ops = []
    for q, x in enumerate(xs):
        if q == 1:
            ops.append(S.operand(x))
            continue
        m = S.alloc_stream(n, dt)
        (S.spccl_encode_dense(x, m) if q == 2 else S.spccl_compress(x, m, ws))
        ops.append(S.operand(m, S.SPCCL_STREAM, S.SPCCL_FMT_DENSE if q == 2 else S.SPCCL_FMT_PICI))
    out = torch.full((P * n + 128,), 7.0, device="cuda")
    S.spccl_gather_expand(ops, n, dt, out[64:64 + P * n], ws)
    assert S.spccl_read_status(ws) == 0
    check(out, torch.cat(xs), 64, f"P={P}")
