"""Small calls of specialised one-branch decoders against the specialised kernel
on LLRs that are infinite, erased, NaN or about to overflow, and with
normalisation factors of either sign: bit for bit, NaN posteriors as one value."""
import numpy as np
import pytest

import synth
from tests.helpers import ensure_built

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def inputs(name, F, kind):
    rng = np.random.default_rng(7)
    x = synth.frames(name, F, 2.0, seed=17).llr
    with np.errstate(over="ignore"):
        hard = np.where(x < 0, -1.0, 1.0).astype(np.float32) * np.float32(np.inf)
        some = rng.random(x.shape) < 0.1
        x = {"channel": x, "hard": hard, "erased": np.where(some, np.float32(0), hard),
             "some": np.where(some, hard, x), "huge": x * np.float32(5e37),
             "nan": np.where(some, np.where(hard < 0, -np.float32(np.nan), np.float32(np.nan)), x)}[kind]
    x = np.ascontiguousarray(x, dtype=np.float32)
    x[:, 63:] = 0.0
    return torch.from_numpy(x).cuda()


@pytest.mark.parametrize("alpha", [0.75, 0.0, -0.5, float("inf")])
@pytest.mark.parametrize("kind", ["channel", "hard", "erased", "some", "huge", "nan"])
@pytest.mark.parametrize("name", ["bch63_36", "bch63_45"])
def test_equals_specialised_kernel(name, kind, alpha):
    B = ensure_built()
    d = B.CODE_DEFS[name]
    c = B.Code(d.m, d.prim, d.t)
    p = B.Pcm.standard(c)
    kw = dict(n_branches=1, mode=B.MODE_EXTRINSIC, max_iter=6, alpha=alpha)
    llr = inputs(name, 300, kind)
    a = B.Decoder(c, p, **kw).decode(llr, trace=True)
    b = B.Decoder(c, p, flags=B.SMALL_NEVER, **kw).decode(llr, trace=True)
    torch.cuda.synchronize()
    for u, v in zip(a[:3], b[:3]):
        assert torch.equal(u, v)
    assert np.array_equal(a[3].cpu().numpy(), b[3].cpu().numpy(), equal_nan=True)
