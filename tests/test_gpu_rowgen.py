"""The generic decoder's frame-per-workgroup kernel against the oracle: short
and long codes, matrices of one to several rounds of rows, row weights across
sign words, every branch count and message mode, ragged frame counts, and a
matrix on either side of its LDS limit (above it the one-lane-per-frame kernel
runs).  The parity bar of tests/helpers.compare_with_oracle."""
import numpy as np
import pytest

import oracle
from tests.helpers import compare_with_oracle, ensure_built

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

PRIM = {3: 0b1011, 4: 0b10011, 5: 0b100101, 6: 0b1000011, 7: 0b10001001}


@pytest.fixture(scope="module")
def B():
    b = ensure_built()
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return b


def run(B, m, t, H, nb, mode, F, max_iter, seed, amp=1.0):
    c = B.Code(m, PRIM[m], t)
    oc = oracle.Code(m, PRIM[m], t)
    p = B.Pcm.from_dense(c, H if H is not None else oc.Hstd)
    H = p.dense()
    dec = B.Decoder(c, p, n_branches=nb, mode=mode, alpha=0.75, max_iter=max_iter, flags=B.FORCE_GENERIC)
    rng = np.random.default_rng(seed)
    ld = 64 if c.N <= 64 else 128
    x = np.zeros((F, ld), np.float32)
    x[:, :c.N] = amp * (3.0 + 3.0 * rng.standard_normal((F, c.N)))
    d_o = rng.integers(0, B.shift_period(c.N), F).astype(np.uint8)
    bits, iters, flg, tr = dec.decode(torch.from_numpy(x).cuda(), torch.from_numpy(d_o).cuda(), trace=True)
    torch.cuda.synchronize()
    words = B.unpack_bits(bits.cpu().numpy().view(np.uint64), c.N)
    res = oracle.decode_batch(H, oc.Hstd, x, d_o, nb, 0.75, max_iter, mode, threads=8, trace=True)
    one = (H, oc.Hstd, x, d_o, nb, 0.75) if mode == oracle.R1 else None
    compare_with_oracle(words, iters.cpu().numpy(), flg.cpu().numpy(), tr.cpu().numpy(), *res, onestep=one)


@pytest.mark.parametrize("mode", [oracle.R1, oracle.R2, oracle.R3])
@pytest.mark.parametrize("nb", [1, 3, 9])
@pytest.mark.parametrize("m,t", [(3, 1), (4, 2), (5, 3), (6, 5), (7, 4), (7, 1)])
def test_standard_matrices(B, m, t, nb, mode):
    run(B, m, t, None, nb, mode, 67, 4, seed=100 * m + 10 * t + nb)


@pytest.mark.parametrize("F", [1, 2, 130])
@pytest.mark.parametrize("m,t,rows,nb,mode", [(6, 5, 48, 9, oracle.R1), (7, 10, 90, 9, oracle.R1),
                                              (7, 10, 65, 3, oracle.R2), (6, 3, 70, 9, oracle.R3)])
def test_own_matrices(B, m, t, rows, nb, mode, F):
    c = B.Code(m, PRIM[m], t)
    H = B.Pcm.build(c, target_rows=rows, seed=3).dense()
    run(B, m, t, H, nb, mode, F, 5, seed=rows + F)


@pytest.mark.parametrize("copies,mode", [(7, oracle.R1), (8, oracle.R1), (2, oracle.R3), (4, oracle.R3)])
def test_both_sides_of_the_lds_limit(B, copies, mode):
    """122 rows repeated: 854 rows fit 64 KB of records in restart mode, 976 do
    not; with edge memory 244 rows fit and 488 do not."""
    c = B.Code(6, PRIM[6], 5)
    H = np.tile(B.Pcm.build(c, target_rows=122, seed=1).dense(), (copies, 1))
    run(B, 6, 5, H, 9, mode, 40, 3, seed=copies)
