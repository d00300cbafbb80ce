"""The row-parallel kernel against the lane-per-frame kernels on LLRs that are
infinite, erased, NaN or about to overflow, whose posteriors turn NaN: words,
iteration counts and flags bit for bit, NaN posteriors as one value, both sides
of one frame per CU, alone and in a mixed call."""
import numpy as np
import pytest

import synth
from tests.helpers import HO_ROWS, ensure_built

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
KINDS = ["hard", "erased", "some", "half", "huge", "nan", "all_nan"]


@pytest.fixture(scope="module")
def B():
    return ensure_built()


def make(B, name, **kw):
    d = B.CODE_DEFS[name]
    c = B.Code(d.m, d.prim, d.t)
    return B.Decoder(c, B.Pcm.build(c, target_rows=HO_ROWS[name], seed=1), n_branches=9, max_iter=8, **kw)


def inputs(name, F, kind, seed=7):
    rng = np.random.default_rng(seed)
    N = int(name[3:].split("_")[0])
    x = synth.frames(name, F, 2.0, seed=seed).llr
    with np.errstate(over="ignore"):
        hard = np.where(x < 0, -1.0, 1.0).astype(np.float32) * np.float32(np.inf)
        nan = np.where(hard < 0, -np.float32(np.nan), np.float32(np.nan))
        some, half = rng.random(x.shape) < 0.1, rng.random(x.shape) < 0.5
        x = {"hard": hard, "erased": np.where(some, np.float32(0), hard), "some": np.where(some, hard, x),
             "half": np.where(half, hard, x), "huge": x * np.float32(5e37), "nan": np.where(some, nan, x),
             "all_nan": nan}[kind]
    x = np.ascontiguousarray(x, dtype=np.float32)
    x[:, N:] = 0.0
    return (torch.from_numpy(x).cuda(),
            torch.from_numpy(rng.integers(0, {63: 21, 127: 42}[N], F).astype(np.uint8)).cuda())


@pytest.mark.parametrize("F", [90, 400])
@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("name", ["bch63_45", "bch63_36", "bch127_64", "bch127_78", "bch127_99"])
def test_equals_lane_kernels(B, name, kind, F):
    llr, d_o = inputs(name, F, kind)
    a = make(B, name).decode(llr, d_o, trace=True)
    for flags in (B.SMALL_NEVER, B.SMALL_ALWAYS):
        b = make(B, name, flags=flags).decode(llr, d_o, trace=True)
        torch.cuda.synchronize()
        for u, v in zip(a[:3], b[:3]):
            assert torch.equal(u, v)
        assert np.array_equal(a[3].cpu().numpy(), b[3].cpu().numpy(), equal_nan=True)


@pytest.mark.parametrize("kind", KINDS)
def test_mixed_call_decodes_as_alone(B, kind):
    names = ["bch63_36", "bch63_45", "bch127_64", "bch127_99"]
    F = 500
    idx = np.random.default_rng(2).integers(0, len(names), F)
    llr = torch.zeros((F, 128), device="cuda")
    d_o = torch.zeros(F, dtype=torch.uint8, device="cuda")
    parts = []
    for c, n in enumerate(names):
        at = torch.from_numpy(np.nonzero(idx == c)[0]).cuda()
        x, d = inputs(n, len(at), kind, seed=c)
        llr[at, :x.shape[1]], d_o[at] = x, d
        parts.append((at, make(B, n, flags=B.SMALL_NEVER).decode(x, d)))
    got = B.MixedDecoder([make(B, n) for n in names]).decode(torch.from_numpy(idx.astype(np.uint8)).cuda(), llr, d_o)
    torch.cuda.synchronize()
    for at, want in parts:
        assert torch.equal(got[0][at][:, :want[0].shape[1]], want[0])
        assert torch.equal(got[1][at], want[1]) and torch.equal(got[2][at], want[2])
