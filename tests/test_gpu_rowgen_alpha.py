"""Generic decoder, restart messages, with normalisation factors that are not
positive and finite: negative ones against the oracle (the parity bar of
tests/helpers.compare_with_oracle), zero and infinite ones on inputs whose
posteriors are exact."""
import numpy as np
import pytest

import oracle
from tests.helpers import compare_with_oracle, ensure_built

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("alpha", [-0.5, -1.25, 0.0, float("inf"), -float("inf")])
@pytest.mark.parametrize("nb", [1, 3, 9])
@pytest.mark.parametrize("m,prim,t", [(6, 0b1000011, 3), (7, 0b10001001, 4)])
def test_restart_mode(m, prim, t, nb, alpha):
    B = ensure_built()
    c, oc = B.Code(m, prim, t), oracle.Code(m, prim, t)
    dec = B.Decoder(c, B.Pcm.standard(c), n_branches=nb, alpha=alpha, max_iter=4, flags=B.FORCE_GENERIC)
    F, ld = 90, 64 if c.N <= 64 else 128
    rng = np.random.default_rng(nb)
    x = np.zeros((F, ld), np.float32)
    x[:, :c.N] = 3.0 + 3.0 * rng.standard_normal((F, c.N))
    d_o = rng.integers(0, B.shift_period(c.N), F).astype(np.uint8)
    bits, iters, flg, tr = dec.decode(torch.from_numpy(x).cuda(), torch.from_numpy(d_o).cuda(), trace=True)
    torch.cuda.synchronize()
    words = B.unpack_bits(bits.cpu().numpy().view(np.uint64), c.N)
    res = oracle.decode_batch(oc.Hstd, oc.Hstd, x, d_o, nb, alpha, 4, oracle.R1, threads=8, trace=True)
    if np.isfinite(alpha):
        compare_with_oracle(words, iters.cpu().numpy(), flg.cpu().numpy(), tr.cpu().numpy(), *res,
                            onestep=(oc.Hstd, oc.Hstd, x, d_o, nb, alpha))
    else:  # every sum is infinite or NaN: the same in both precisions
        assert np.array_equal(words, res[0])
        assert np.array_equal(iters.cpu().numpy(), res[1])
        assert np.array_equal(flg.cpu().numpy().astype(bool), res[2].astype(bool))
