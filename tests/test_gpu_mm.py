"""The fixed-point kernel with its sums on the matrix cores against the
lane-per-frame kernels it stands in for: words, iteration counts, flags and
every iteration's posterior, from its smallest calls on.  All values are
integers and every sum is exact, so no tolerance is needed."""
import numpy as np
import pytest

import synth
from tests.helpers import HO_ROWS, ensure_built

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
CODES = ["bch127_64", "bch127_99", "bch63_36"]


@pytest.fixture(scope="module")
def B():
    b = ensure_built()
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return b


def make(B, name, **kw):
    d = B.CODE_DEFS[name]
    c = B.Code(d.m, d.prim, d.t)
    p = B.Pcm.build(c, target_rows=HO_ROWS[name], seed=1)
    return B.Decoder(c, p, n_branches=9, max_iter=kw.pop("max_iter", 8), precision=B.FIX8, **kw)


def smallest(name):
    """Frames of the kernel's smallest call: the row-parallel kernel takes those
    up to 92 per CU of N = 127, the waves of N = 63 those up to 2400."""
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    return n_cu * 92 + 1 if name.startswith("bch127") else n_cu * 2400


def frames(name, F, ebn0, seed):
    """int8 frames: 20000 drawn, repeated with other offsets."""
    fr = synth.frames(name, 20000, ebn0, seed=seed)
    q = np.clip(np.rint(fr.llr * 4.0), -127, 127).astype(np.int8)
    rep = -(-F // len(q))
    rng = np.random.default_rng(seed)
    return (torch.from_numpy(np.tile(q, (rep, 1))[:F]).cuda(),
            torch.from_numpy(rng.integers(0, 256, F, dtype=np.uint8)).cuda())  # taken modulo d_p


def outputs(dec, F):
    return (torch.zeros((F, dec.W64), dtype=torch.int64, device="cuda"), torch.zeros(F, dtype=torch.uint8, device="cuda"),
            torch.zeros(F, dtype=torch.uint8, device="cuda"))


def run(dec, llr, d_o):
    o = outputs(dec, len(d_o))
    ws = torch.empty(dec.workspace_size(len(d_o)), dtype=torch.uint8, device="cuda")
    dec.decode_into(llr, d_o, *o, workspace=ws)
    torch.cuda.synchronize()
    return o


def same(a, b):
    torch.cuda.synchronize()
    for x, y in zip(a, b):
        assert torch.equal(x, y)


@pytest.mark.parametrize("ebn0,iters", [(1.0, 8), (4.5, 3)])
@pytest.mark.parametrize("name", CODES)
def test_equals_lane_kernels(B, name, ebn0, iters):
    F = smallest(name)
    q, d_o = frames(name, F, ebn0, seed=31)
    d_o = d_o % B.shift_period(int(name[3:].split("_")[0]))  # decode() refuses more
    a = make(B, name, max_iter=iters).decode(q, d_o, trace=True)
    b = make(B, name, max_iter=iters, flags=B.SMALL_NEVER).decode(q, d_o, trace=True)
    same(a, b)


@pytest.mark.parametrize("kind", ["equal", "zeros", "saturated", "uniform"])
@pytest.mark.parametrize("name", CODES)
def test_adversarial_frames(B, name, kind):
    F, N = smallest(name) + 5, int(name[3:].split("_")[0])
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    lo, hi = {"equal": (9, 10), "zeros": (0, 2), "saturated": (126, 129), "uniform": (0, 129)}[kind]
    mag = torch.randint(lo, hi, (F, N + 1), generator=g, device="cuda", dtype=torch.int16)
    sgn = torch.randint(0, 2, (F, N + 1), generator=g, device="cuda", dtype=torch.int16) * 2 - 1
    q = (mag * sgn).clamp(-128, 127).to(torch.int8)
    d_o = torch.randint(0, 256, (F,), generator=g, device="cuda", dtype=torch.int16).to(torch.uint8)
    same(run(make(B, name), q, d_o), run(make(B, name, flags=B.SMALL_NEVER), q, d_o))


@pytest.mark.parametrize("ld,skew", [(127, 0), (127, 3), (128, 1), (132, 4), (130, 2)])
def test_row_strides_and_alignment(B, ld, skew):
    name, F = "bch127_99", 30011
    q, d_o = frames(name, F, 3.0, seed=33)
    # the last row ends with its last coordinate
    buf = torch.zeros(F * ld + skew - (ld - 127), dtype=torch.int8, device="cuda")
    rows = torch.as_strided(buf, (F, 127), (ld, 1), skew)
    rows.copy_(q[:, :127])
    dec = make(B, name)
    o = outputs(dec, F)
    ws = torch.empty(dec.workspace_size(F), dtype=torch.uint8, device="cuda")
    L = B.lib()
    rc = L.bch_nms_decode_batch(dec.h, rows.data_ptr(), ld, F, d_o.data_ptr(), o[0].data_ptr(), o[1].data_ptr(),
                                o[2].data_ptr(), None, ws.data_ptr(), ws.numel(),
                                torch.cuda.current_stream().cuda_stream)
    assert rc == 0
    same(o, run(make(B, name, flags=B.SMALL_NEVER), q, d_o))


@pytest.mark.parametrize("flags,waves", [("CHUNK_BUCKETS", 0), ("UNPACKED16", 1)])
def test_ranges_and_grids(B, flags, waves):
    """Chunked ranges of the prepass, and a grid of one wave a CU."""
    name, F = "bch127_64", (1 << 20) + 77
    q, d_o = frames(name, F, 4.0, seed=35)
    dec = make(B, name, flags=getattr(B, flags))
    if waves:
        dec.set_tuning(waves)
    same(run(dec, q, d_o), run(make(B, name, flags=B.SMALL_NEVER), q, d_o))


def test_mixed_per_code(B):
    """A mixed call that runs a kernel per code selects its frames from the mix."""
    F = 700_000
    names = ["bch127_64", "bch127_99", "bch63_36"]
    decs = [make(B, n, flags=B.NO_MIXED_KERNEL) for n in names]
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    code = torch.randint(0, 3, (F,), generator=g, device="cuda", dtype=torch.int16).to(torch.uint8)
    q = torch.zeros((F, 128), dtype=torch.int8, device="cuda")
    d_o = torch.zeros(F, dtype=torch.uint8, device="cuda")
    for c, n in enumerate(names):
        m = code == c
        x, o = frames(n, int(m.sum()), 3.0, seed=37 + c)
        q[m, :x.shape[1]] = x
        d_o[m] = o
    mix = B.MixedDecoder(decs)
    got = mix.decode(code, q, d_o)
    for c, n in enumerate(names):
        m = code == c
        want = run(make(B, n, flags=B.SMALL_NEVER), q[m].contiguous(), d_o[m])
        same((got[0][m][:, :want[0].shape[1]], got[1][m], got[2][m]), want)
