"""The one-wave kernels of N = 127 and the grouped ones of N = 63 on calls of
many frames a lane against the row-parallel kernel on the same frames in small
calls, bit for bit."""
import numpy as np
import pytest

import synth
from tests.helpers import HO_ROWS, ensure_built

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def B():
    b = ensure_built()
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return b


@pytest.mark.parametrize("F,ebn0", [(60_001, 1.0), (150_000, 4.0)])
@pytest.mark.parametrize("name", ["bch127_64", "bch127_78", "bch127_99", "bch63_36", "bch63_45"])
def test_equals_small_calls(B, name, F, ebn0):
    d = B.CODE_DEFS[name]
    c = B.Code(d.m, d.prim, d.t)
    p = B.Pcm.build(c, target_rows=HO_ROWS[name], seed=1)
    dec = B.Decoder(c, p, n_branches=9, max_iter=8)
    fr = synth.frames(name, 20_000, ebn0, seed=51)
    rep = -(-F // 20_000)
    llr = torch.from_numpy(fr.llr).cuda().repeat(rep, 1)[:F].contiguous()
    d_o = torch.from_numpy(np.random.default_rng(5).integers(0, B.shift_period(c.N), F,
                                                              dtype=np.uint8)).cuda()
    trace = F < 70_000
    big = dec.decode(llr, d_o, trace=trace)
    n = 16_384
    for f0 in range(0, F, n):
        small = dec.decode(llr[f0:f0 + n], d_o[f0:f0 + n], trace=trace)
        torch.cuda.synchronize()
        for a, b in zip(big, small):
            if a is not None:
                assert torch.equal(a[f0:f0 + n].view(torch.uint8), b.view(torch.uint8))
