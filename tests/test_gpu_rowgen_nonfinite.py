"""Generic decoder on LLRs that are infinite, erased (zero) or NaN: hard
decisions with errors and erasures, whose posteriors are 0, infinite or NaN in
every precision, so that words, iteration counts and flags equal the oracle's."""
import numpy as np
import pytest

import oracle
import synth
from tests.helpers import ensure_built, oracle_code

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def inputs(name, F, kind):
    """Infinite hard decisions of noisy frames, a tenth of them erased or NaN."""
    rng = np.random.default_rng(7)
    x = synth.frames(name, F, 2.0, seed=17).llr
    hard = np.where(x < 0, -1.0, 1.0).astype(np.float32) * np.float32(np.inf)
    other = {"hard": hard, "erased": np.zeros_like(hard),
             "nan": np.where(rng.random(x.shape) < 0.5, np.float32(np.nan), -np.float32(np.nan))}[kind]
    return np.where(rng.random(x.shape) < 0.1, other, hard).astype(np.float32)


@pytest.mark.parametrize("kind", ["hard", "erased", "nan"])
@pytest.mark.parametrize("mode", [oracle.R1, oracle.R2, oracle.R3])
@pytest.mark.parametrize("nb", [1, 3, 9])
@pytest.mark.parametrize("name", ["bch63_45", "bch127_99"])
def test_equals_oracle(name, nb, mode, kind):
    B = ensure_built()
    d = B.CODE_DEFS[name]
    c, oc = B.Code(d.m, d.prim, d.t), oracle_code(name)
    dec = B.Decoder(c, B.Pcm.standard(c), n_branches=nb, mode=mode, max_iter=4, flags=B.FORCE_GENERIC)
    F = 150
    x = inputs(name, F, kind)
    d_o = np.random.default_rng(3).integers(0, B.shift_period(c.N), F).astype(np.uint8)
    bits, iters, flg, _ = dec.decode(torch.from_numpy(x).cuda(), torch.from_numpy(d_o).cuda())
    torch.cuda.synchronize()
    words = B.unpack_bits(bits.cpu().numpy().view(np.uint64), c.N)
    res = oracle.decode_batch(oc.Hstd, oc.Hstd, x, d_o, nb, 0.75, 4, mode, threads=8)
    assert np.array_equal(words, res[0])
    assert np.array_equal(iters.cpu().numpy(), res[1])
    assert np.array_equal(flg.cpu().numpy().astype(bool), np.asarray(res[2]).astype(bool))
