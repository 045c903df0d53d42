"""GPU parity of the dense streams (dense (+) dense, dense encoding) at their
edges: lengths around a vector and a block's 16 KiB range, operands and outputs
that start at any element (each its own offset), in place, message operands and
outputs; and the collectives' dense paths over chunks of odd length."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from helpers import bits, first_diff, log, to_dev, to_host_bits

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def S():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2607_04676_amd as S
    return S


@pytest.mark.parametrize("dtype", [W.F32, W.BF16])
def test_dense_dense_offsets(S, dtype):
    dt = S.SPCCL_F32 if dtype == W.F32 else S.SPCCL_BF16
    chunk = 16384 // (4 if dtype == W.F32 else 2)
    for n in (1, 7, 9, 1023, chunk - 1, chunk + 1, 3 * chunk + 5):
        a, b = W.sparse_array(n, -(-n // 2), [91, n, 0], dtype), W.sparse_array(n, -(-n // 2), [91, n, 1], dtype)
        b[: n // 4] = a[: n // 4]
        if dtype == W.F32:
            b[: n // 4] *= -1                               # cancellations
        else:
            b[: n // 4] ^= np.uint16(0x8000)
        exp = O.reduce(O.Operand.array(a), O.Operand.array(b), n, dt, O.ARRAY)
        ws = S.alloc_workspace(n, dt)
        for oa, ob, oo in ((0, 0, 0), (1, 2, 3), (8, 0, 7), (5, 5, 5)):
            log(f"dense+dense n={n} {dtype} offsets {oa} {ob} {oo}")
            td = to_dev(a).dtype
            pa, pb, po = (torch.full((n + 64,), 7.0, dtype=td, device="cuda") for _ in range(3))
            pa[oa:oa + n], pb[ob:ob + n] = to_dev(a), to_dev(b)
            S.spccl_reduce(S.operand(pa[oa:oa + n]), S.operand(pb[ob:ob + n]), S.operand(po[oo:oo + n]), n, dt, ws)
            assert S.spccl_read_status(ws) == 0
            got = to_host_bits(po[oo:oo + n])
            assert np.array_equal(got, bits(exp)), first_diff(got, bits(exp))
            rest = torch.cat([po[:oo], po[oo + n:]])
            assert bool((rest == 7.0).all())
            S.spccl_reduce(S.operand(pa[oa:oa + n]), S.operand(pb[ob:ob + n]), S.operand(pa[oa:oa + n]), n, dt, ws)
            assert np.array_equal(to_host_bits(pa[oa:oa + n]), bits(exp))          # in place
        # messages: encoded from an odd offset, added into a message
        ma, mb, mo = (S.alloc_stream(n, dt) for _ in range(3))
        big = torch.zeros(n + 3, dtype=to_dev(a).dtype, device="cuda")
        big[3:] = to_dev(a)
        S.spccl_encode_dense(big[3:], ma)
        S.spccl_encode_dense(to_dev(b), mb)
        msg = lambda t: S.operand(t, S.SPCCL_STREAM, S.SPCCL_FMT_DENSE)
        S.spccl_reduce(msg(ma), msg(mb), msg(mo), n, dt, ws)
        h = S.spccl_read_header(mo)
        assert S.spccl_read_status(ws) == 0 and h["format"] == S.SPCCL_FMT_DENSE and h["n"] == n
        got = to_host_bits(mo[48:48 + n * big.element_size()].view(big.dtype))
        assert np.array_equal(got, bits(exp)), first_diff(got, bits(exp))


@pytest.mark.parametrize("dtype", [W.F32, W.BF16])
@pytest.mark.parametrize("adaptive", [0, 1, 2])
def test_rings_of_odd_chunks(S, dtype, adaptive):
    """Forwarded messages of every format and parity of hop, chunks that start
    anywhere in a line: the all-reduce equals the oracle's, canonical and sliced."""
    dt = S.SPCCL_F32 if dtype == W.F32 else S.SPCCL_BF16
    for P, m in ((3, 4097), (4, 3 * 16384 + 5)):
        log(f"rings P={P} m={m} {dtype} adaptive={adaptive}")
        n = P * m
        x = [W.sparse_array(n, n // 3, [92, r, m], dtype) for r in range(P)]
        tx = [to_dev(v) for v in x]
        pol = S.spccl_policy_t(0.6, 0.5, 0.3, 0, adaptive, S.SPCCL_FMT_PICI)
        acc = [None] * P
        for c in range(P):
            lo, hi = c * m, (c + 1) * m
            v = x[(c + 1) % P][lo:hi]
            for k in range(2, P + 1):
                v = O.reduce(O.Operand.array(v), O.Operand.array(x[(c + k) % P][lo:hi]), m, dt, O.ARRAY)
            acc[c] = v
        exp = bits(np.concatenate(acc))
        recv = [torch.empty_like(tx[0]) for _ in range(P)]
        scratch = torch.empty(S.spccl_vr_scratch_bytes(P, m, dt), dtype=torch.uint8, device="cuda").fill_(0xFF)
        for _ in range(2):
            S.spccl_vr_all_reduce(tx, recv, scratch, pol)
            for r in range(P):
                assert np.array_equal(to_host_bits(recv[r]), exp), f"rank {r}: {first_diff(to_host_bits(recv[r]), exp)}"
        scratch = torch.empty(S.spccl_vr_sliced_scratch_bytes(P, m, dt), dtype=torch.uint8, device="cuda").fill_(0xFF)
        S.spccl_vr_all_reduce_sliced(tx, recv, scratch, pol)
        for r in range(P):
            assert np.array_equal(to_host_bits(recv[r]), exp), f"sliced rank {r}: {first_diff(to_host_bits(recv[r]), exp)}"
