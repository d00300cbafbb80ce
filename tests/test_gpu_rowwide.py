"""The row-parallel kernel on both sides of one frame per CU (twelve waves a
frame up to there, three beyond) against the lane-per-frame kernels, bit for
bit: frames with ties, zeros and infinities, and mixed calls."""
import numpy as np
import pytest

from tests.helpers import HO_ROWS, ensure_built

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def B():
    b = ensure_built()
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return b


def make(B, name, **kw):
    d = B.CODE_DEFS[name]
    c = B.Code(d.m, d.prim, d.t)
    return B.Decoder(c, B.Pcm.build(c, target_rows=HO_ROWS[name], seed=1), n_branches=9, max_iter=8, **kw)


def frames(names, F, kind, prec, ld=128):
    rng = np.random.default_rng(9)
    mag = {"equal": np.full((F, ld), 1.5), "zeros": rng.choice([0.0, 2.0], size=(F, ld)),
           "inf": rng.choice([1.0, 3.0, np.inf], p=[0.6, 0.38, 0.02], size=(F, ld))}[kind]
    x = (rng.choice([-1.0, 1.0], size=(F, ld)) * mag).astype(np.float32)
    if prec:
        x = np.clip(np.rint(x * 60), -128, 127).astype(np.int8)
    return torch.from_numpy(x).cuda(), torch.from_numpy(rng.integers(0, 256, F, dtype=np.uint8)).cuda()


def run(dec, llr, d_o, code=None):
    F, W = len(d_o), 2 if code is not None else dec.W64
    o = [torch.zeros((F, W), dtype=torch.int64, device="cuda"), torch.zeros(F, dtype=torch.uint8, device="cuda"),
         torch.zeros(F, dtype=torch.uint8, device="cuda")]
    ws = torch.empty(dec.workspace_size(F), dtype=torch.uint8, device="cuda")
    if code is None:
        dec.decode_into(llr, d_o, *o, workspace=ws)
    else:
        dec.decode_into(code, llr, d_o, *o, ws)
    torch.cuda.synchronize()
    return o


@pytest.mark.parametrize("over", [0, 1])
@pytest.mark.parametrize("kind", ["equal", "zeros", "inf"])
@pytest.mark.parametrize("name,prec", [("bch63_45", 0), ("bch63_36", 0), ("bch127_64", 0), ("bch127_78", 0),
                                       ("bch127_99", 0), ("bch63_36", 1), ("bch127_99", 1)])
def test_equals_lane_kernels(B, name, prec, kind, over):
    F = torch.cuda.get_device_properties(0).multi_processor_count + over
    x, d_o = frames([name], F, kind, prec)
    got = run(make(B, name, precision=prec), x, d_o)
    want = run(make(B, name, precision=prec, flags=B.SMALL_NEVER), x, d_o)
    for a, b in zip(got, want):
        assert torch.equal(a, b)


@pytest.mark.parametrize("F", [1, 5, 200])
@pytest.mark.parametrize("names", [["bch63_36", "bch63_45"], ["bch127_64", "bch63_36", "bch127_99"]])
def test_mixed_calls(B, names, F):
    x, d_o = frames(names, F, "inf", 0)
    code = torch.arange(F, device="cuda").remainder(len(names)).to(torch.uint8)
    got = run(B.MixedDecoder([make(B, n) for n in names]), x, d_o, code)
    for c, n in enumerate(names):
        m = code == c
        if bool(m.any()):
            want = run(make(B, n, flags=B.SMALL_NEVER), x[m].contiguous(), d_o[m])
            assert torch.equal(got[0][m][:, :want[0].shape[1]], want[0])
            assert torch.equal(got[1][m], want[1]) and torch.equal(got[2][m], want[2])
