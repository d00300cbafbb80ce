"""The row-parallel kernel (a frame per workgroup, small calls) against the
lane-per-frame kernels it stands in for: words, iteration counts, flags and
every iteration's posterior bit for bit, on both code lengths and precisions,
one frame to several hundred, channel and adversarial frames, and mixed
calls.  Its sums are formed in the same order, so no tolerance is needed."""
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


def make(B, name, rows, **kw):
    d = B.CODE_DEFS[name]
    c = B.Code(d.m, d.prim, d.t)
    p = B.Pcm.build(c, target_rows=rows, seed=1)
    return B.Decoder(c, p, n_branches=9, max_iter=kw.pop("max_iter", 8), **kw)


def same(a, b):
    torch.cuda.synchronize()
    for x, y in zip(a, b):
        assert torch.equal(x.view(torch.uint8), y.view(torch.uint8))


@pytest.mark.parametrize("F", [1, 2, 63, 321])
@pytest.mark.parametrize("name,rows,prec", [
    ("bch63_45", 33, 0), ("bch63_36", 122, 0), ("bch63_36", 316, 0), ("bch63_36", 27, 0), ("bch127_64", 72, 0),
    ("bch127_78", 57, 0), ("bch127_99", 33, 0), ("bch63_45", 33, 1), ("bch63_36", 122, 1), ("bch127_64", 72, 1),
    ("bch127_99", 33, 1)])
def test_equals_lane_kernels(B, name, rows, prec, F):
    for ebn0, alpha, iters in ((1.0, 0.75, 8), (4.5, 0.6, 3)):
        new = make(B, name, rows, precision=prec, alpha=alpha, max_iter=iters)
        old = make(B, name, rows, precision=prec, alpha=alpha, max_iter=iters, flags=B.SMALL_NEVER)
        fr = synth.frames(name, F, ebn0, seed=90 + F)
        llr = torch.from_numpy(fr.llr).cuda()
        if prec:
            q = torch.empty(llr.shape, dtype=torch.int8, device="cuda")
            B.quantize_llr(llr, new.N, 4.0, q)
            llr = q
        d_o = torch.from_numpy(fr.d_o).cuda()
        same(new.decode(llr, d_o, trace=True), old.decode(llr, d_o, trace=True))


@pytest.mark.parametrize("kind", ["equal", "zeros", "subnormal", "inf"])
@pytest.mark.parametrize("name", ["bch63_36", "bch127_99"])
def test_adversarial_frames(B, name, kind):
    spec = synth.code(name)
    F = 130
    rng = np.random.default_rng(5)
    x = np.zeros((F, spec.ld), np.float32)
    sgn = rng.choice([-1.0, 1.0], size=(F, spec.N))
    mag = {"equal": np.full((F, spec.N), 1.5), "zeros": rng.choice([0.0, -0.0, 2.0], size=(F, spec.N)),
           "subnormal": rng.choice([1e-42, 3e-40, 1e-38], size=(F, spec.N)),
           "inf": rng.choice([1.0, 3.0, np.inf], p=[0.6, 0.38, 0.02], size=(F, spec.N))}[kind]
    x[:, :spec.N] = sgn * mag
    llr = torch.from_numpy(x).cuda()
    # offsets past d_p are taken modulo d_p by every kernel
    d_o = torch.from_numpy(np.arange(F, dtype=np.uint8) * 2).cuda()
    outs = []
    for flags in (0, B.SMALL_NEVER):
        dec = make(B, name, HO_ROWS[name], flags=flags)
        o = (torch.zeros((F, dec.W64), dtype=torch.int64, device="cuda"), torch.zeros(F, dtype=torch.uint8, device="cuda"),
             torch.zeros(F, dtype=torch.uint8, device="cuda"))
        ws = torch.empty(dec.workspace_size(F), dtype=torch.uint8, device="cuda")
        dec.decode_into(llr, d_o, *o, workspace=ws)
        outs.append(o)
    same(*outs)


@pytest.mark.parametrize("name", ["bch63_45", "bch127_99"])
def test_both_sides_of_the_size_limit(B, name):
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    lim = n_cu * (224 if name == "bch63_45" else 128)
    fr = synth.frames(name, lim + 1, 4.0, seed=3)
    llr, d_o = torch.from_numpy(fr.llr).cuda(), torch.from_numpy(fr.d_o).cuda()
    dec = make(B, name, HO_ROWS[name])
    a = dec.decode(llr[:lim], d_o[:lim])[:3]
    b = dec.decode(llr, d_o)[:3]
    same(a, [x[:lim] for x in b])


@pytest.mark.parametrize("names,prec", [
    (["bch63_36", "bch63_45", "bch127_64", "bch127_99"], 0), (["bch127_64", "bch127_99", "bch63_36"], 1),
    (["bch63_45", "bch63_36"], 0), (["bch127_99"], 0)])
def test_mixed_equals_other_paths(B, names, prec):
    F, ld = 700, (128 if any("127" in n for n in names) else 64)
    rng = np.random.default_rng(8)
    idx = rng.integers(0, len(names) + 1, F).astype(np.uint8)  # some frames name no decoder
    llr = np.zeros((F, ld), np.float32)
    d_o = rng.integers(0, 21, F).astype(np.uint8)
    for c, n in enumerate(names):
        sel = np.nonzero(idx == c)[0]
        x = synth.frames(n, len(sel), 2.5, seed=c + 1).llr
        llr[sel, :x.shape[1]] = x
    x = torch.from_numpy(llr).cuda()
    if prec:
        x = torch.clamp(torch.round(4.0 * x), -127, 127).to(torch.int8)
    idx_d, d_o_d = torch.from_numpy(idx).cuda(), torch.from_numpy(d_o).cuda()
    outs = []
    for flags in (0, B.MIXED_KERNEL, B.NO_MIXED_KERNEL):
        mix = B.MixedDecoder([make(B, n, HO_ROWS[n], precision=prec, flags=flags) for n in names])
        o = (torch.full((F, 2), -7, dtype=torch.int64, device="cuda"), torch.full((F,), 77, dtype=torch.uint8, device="cuda"),
             torch.full((F,), 77, dtype=torch.uint8, device="cuda"))
        ws = torch.empty(mix.workspace_size(F), dtype=torch.uint8, device="cuda")
        mix.decode_into(idx_d, x, d_o_d, *o, ws)
        outs.append(o)
    same(outs[0], outs[1])
    same(outs[0], outs[2])
    assert bool((outs[0][1][torch.from_numpy(idx == len(names)).cuda()] == 77).all())
