"""Kernels that default calls of the tests' sizes do not reach, against the
oracle: the lane-per-frame kernels of the redundancy sweep's matrices, whose
small calls run the row-parallel kernel, and the one-lane-per-frame generic
kernel, which runs matrices whose state does not fit the frame-per-workgroup
form."""
import numpy as np
import pytest

import oracle
import synth
from tests.helpers import compare_with_oracle, ensure_built, oracle_code, oracle_hopt

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

PRIM = {6: 0b1000011, 7: 0b10001001}


@pytest.fixture(scope="module")
def B():
    return ensure_built()


def decode(B, dec, llr, d_o):
    bits, iters, flg, tr = dec.decode(torch.from_numpy(llr).cuda(), torch.from_numpy(d_o).cuda(), trace=True)
    torch.cuda.synchronize()
    return (B.unpack_bits(bits.cpu().numpy().view(np.uint64), dec.N), iters.cpu().numpy(), flg.cpu().numpy(),
            tr.cpu().numpy())


@pytest.mark.parametrize("name,rows", [("bch63_36", 27), ("bch63_36", 32), ("bch63_36", 47), ("bch63_36", 269),
                                       ("bch63_36", 316), ("bch127_78", 49), ("bch127_78", 65)])
def test_lane_kernels_of_the_redundancy_sweep(B, name, rows):
    d = B.CODE_DEFS[name]
    c = B.Code(d.m, d.prim, d.t)
    p = B.Pcm.build(c, target_rows=rows, seed=1)
    H, oc = oracle_hopt(name, rows), oracle_code(name)
    dec = B.Decoder(c, p, n_branches=9, max_iter=8, flags=B.SMALL_NEVER)
    F = 64 * 3 + 11
    assert dec.running_kernel(F) == "spec_%s_m%d_b9" % (name, rows)
    fr = synth.frames(name, F, 4.0, seed=19)
    res = oracle.decode_batch(H, oc.Hstd, fr.llr, fr.d_o, 9, 0.75, 8, oracle.R1, threads=8, trace=True)
    compare_with_oracle(*decode(B, dec, fr.llr, fr.d_o), *res, onestep=(H, oc.Hstd, fr.llr, fr.d_o, 9, 0.75))


# the standard matrix repeated until its state does not fit, alpha divided by the
# repeats, so that the sums are those of one copy
@pytest.mark.parametrize("m,t,copies,nb,mode", [
    (7, 10, 14, 9, oracle.R1), (7, 10, 5, 9, oracle.R2), (7, 10, 5, 9, oracle.R3), (7, 10, 15, 3, oracle.R2),
    (7, 10, 15, 3, oracle.R3), (6, 5, 36, 9, oracle.R1), (6, 5, 20, 9, oracle.R2), (6, 5, 20, 9, oracle.R3)])
def test_generic_kernel_of_large_matrices(B, m, t, copies, nb, mode):
    c, oc = B.Code(m, PRIM[m], t), oracle.Code(m, PRIM[m], t)
    H = np.tile(np.asarray(oc.Hstd, np.uint8), (copies, 1))
    alpha = 0.75 / copies
    dec = B.Decoder(c, B.Pcm.from_dense(c, H), n_branches=nb, mode=mode, alpha=alpha, max_iter=3)
    assert dec.running_kernel(70) == "generic"
    rng = np.random.default_rng(copies)
    x = np.zeros((70, 64 if c.N <= 64 else 128), np.float32)
    x[:, :c.N] = 3.0 + 3.0 * rng.standard_normal((70, c.N))
    d_o = rng.integers(0, B.shift_period(c.N), 70).astype(np.uint8)
    res = oracle.decode_batch(H, oc.Hstd, x, d_o, nb, alpha, 3, mode, threads=8, trace=True)
    one = (H, oc.Hstd, x, d_o, nb, alpha) if mode == oracle.R1 else None
    compare_with_oracle(*decode(B, dec, x, d_o), *res, onestep=one)
