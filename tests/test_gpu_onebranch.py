"""Small calls of specialised one-branch decoders, which a frame-per-workgroup
kernel takes, against the specialised kernel, bit for bit: on both sides of the
limit of 64 frames per CU, channel frames and frames with ties and infinities."""
import numpy as np
import pytest

import synth
from tests.helpers import ensure_built

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def B():
    b = ensure_built()
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return b


@pytest.mark.parametrize("kind", ["channel", "equal", "zeros", "inf"])
@pytest.mark.parametrize("F", [1, 65, 0])
@pytest.mark.parametrize("name", ["bch63_36", "bch63_45"])
def test_equals_specialised_kernel(B, name, F, kind):
    d = B.CODE_DEFS[name]
    c = B.Code(d.m, d.prim, d.t)
    p = B.Pcm.standard(c)
    if F == 0:
        F = torch.cuda.get_device_properties(0).multi_processor_count * 64
    kw = dict(n_branches=1, mode=B.MODE_EXTRINSIC, max_iter=6)
    new, old = B.Decoder(c, p, **kw), B.Decoder(c, p, flags=B.SMALL_NEVER, **kw)
    assert new.specialized and old.specialized
    rng = np.random.default_rng(F)
    if kind == "channel":
        x = synth.frames(name, F, 2.0, seed=71).llr
    else:
        mag = {"equal": np.full((F, 64), 1.5), "zeros": rng.choice([0.0, 2.0], size=(F, 64)),
               "inf": rng.choice([1.0, 3.0, np.inf], p=[0.6, 0.38, 0.02], size=(F, 64))}[kind]
        x = (rng.choice([-1.0, 1.0], size=(F, 64)) * mag).astype(np.float32)
        x[:, 63] = 0.0
    llr = torch.from_numpy(np.ascontiguousarray(x)).cuda()
    a, b = new.decode(llr, trace=True), old.decode(llr, trace=True)
    torch.cuda.synchronize()
    for u, v in zip(a[:3], b[:3]):
        assert torch.equal(u, v)
    ta, tb = a[3].cpu().numpy(), b[3].cpu().numpy()
    assert np.array_equal(ta, tb, equal_nan=True)
