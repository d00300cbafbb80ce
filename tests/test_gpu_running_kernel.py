"""Which kernel a call runs: running_kernel names the one that the dispatch
takes, and the tests that compare a stand-in kernel with the one registered do
run the stand-in at their sizes."""
import pytest

from tests.helpers import HO_ROWS, ensure_built

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def B():
    return ensure_built()


def make(B, name, rows=None, **kw):
    d = B.CODE_DEFS[name]
    c = B.Code(d.m, d.prim, d.t)
    p = B.Pcm.standard(c) if rows == 0 else B.Pcm.build(c, target_rows=rows or HO_ROWS[name], seed=1)
    return B.Decoder(c, p, n_branches=kw.pop("n_branches", 9), **kw)


def cus():
    return torch.cuda.get_device_properties(0).multi_processor_count


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("name", ["bch63_45", "bch63_36", "bch127_64", "bch127_99"])
def test_row_parallel(B, name, prec):
    dec = make(B, name, precision=prec)
    assert dec.running_kernel(1) == dec.running_kernel(cus()) == "rowpar_wide"
    assert dec.running_kernel(cus() + 1) == dec.running_kernel(2 * cus()) == "rowpar"
    reg = "spec_%s_m%d_b9" % (name, HO_ROWS[name]) + ("_fix8" if prec else "")
    big = dec.running_kernel(3_999_999)
    assert big == (reg + "_mm" if prec and name != "bch63_45" else reg)
    flags = [B.SMALL_ALWAYS, B.SMALL_NEVER] + ([B.PACKED16] if prec else [])
    for f in flags:
        d = make(B, name, precision=prec, flags=f)
        for F in (1, 2 * cus(), 4_000_000):
            assert d.running_kernel(F) == d.kernel_name(F) and d.running_kernel(F).startswith(reg)


def test_matrices_of_the_redundancy_sweep(B):
    """Their tables fit the three-wave form; two have too many rounds for the wide one."""
    for name, rows, wide in [("bch63_36", 27, True), ("bch63_36", 47, True), ("bch63_36", 269, False),
                             ("bch63_36", 316, False), ("bch127_78", 49, True), ("bch127_78", 65, True)]:
        dec = make(B, name, rows)
        assert dec.running_kernel(1) == ("rowpar_wide" if wide else "rowpar")
        assert dec.running_kernel(2 * cus()) == "rowpar"
        assert dec.running_kernel(1_000_000) == "spec_%s_m%d_b9" % (name, rows)


def test_generic(B):
    for kw in (dict(), dict(mode=B.MODE_MEMORY), dict(mode=B.MODE_EXTRINSIC), dict(n_branches=1), dict(n_branches=3)):
        dec = make(B, "bch63_36", flags=B.FORCE_GENERIC, **kw)
        assert dec.running_kernel(1) == dec.running_kernel(10 ** 8) == "rowgen" and dec.kernel_name(1) == "generic"
    one = make(B, "bch63_36", 0, n_branches=1, mode=B.MODE_EXTRINSIC)
    reg = "spec_bch63_36_m27_b1_ext"
    assert one.running_kernel(1) == one.running_kernel(64 * cus()) == "rowgen"
    assert one.running_kernel(64 * cus() + 1) == one.kernel_name(1) == reg
    for kw in (dict(flags=B.SMALL_NEVER), dict(alpha=0.0), dict(alpha=-0.5), dict(alpha=float("inf"))):
        dec = make(B, "bch63_36", 0, n_branches=1, mode=B.MODE_EXTRINSIC, **kw)
        assert dec.running_kernel(1) == reg
    assert make(B, "bch63_36", n_branches=3).running_kernel(1) == "spec_bch63_36_m122_b3"


def test_mixed(B):
    names = ["bch63_36", "bch63_45", "bch127_64", "bch127_99"]
    fused = "mix_63_36_m122_63_45_m33_127_64_m72_127_99_m33"
    mix = B.MixedDecoder([make(B, n) for n in names])
    assert mix.running_kernel(1) == mix.running_kernel(cus()) == "rowpar_wide"
    assert mix.running_kernel(cus() + 1) == "rowpar"
    assert mix.running_kernel(1_000_000) == mix.kernel_name(1) == fused
    assert mix.running_kernel(3_000_000) == "per-code"
    for f, want in ((B.MIXED_KERNEL, fused), (B.NO_MIXED_KERNEL, "per-code")):
        m = B.MixedDecoder([make(B, n, flags=f) for n in names])
        assert m.running_kernel(1) == m.kernel_name(1) == want


@pytest.mark.parametrize("name,rows,prec,per_cu", [
    ("bch127_64", 72, 0, 92), ("bch127_78", 57, 0, 92), ("bch127_99", 33, 0, 92), ("bch127_64", 72, 1, 92),
    ("bch127_99", 33, 1, 84), ("bch63_45", 33, 0, 224), ("bch63_36", 122, 0, 224), ("bch63_36", 122, 1, 208),
    ("bch63_36", 27, 0, 76), ("bch63_36", 32, 0, 88), ("bch63_36", 47, 0, 100), ("bch63_36", 269, 0, 208),
    ("bch63_36", 316, 0, 188)])
def test_both_sides_of_the_row_parallel_line(B, name, rows, prec, per_cu):
    """The kernels on either side, and that they give the same frames."""
    F = per_cu * cus()
    dec = make(B, name, rows, precision=prec)
    assert dec.running_kernel(F) == "rowpar" and dec.running_kernel(F + 1).startswith("spec_%s_m%d" % (name, rows))
    N = dec.N
    g = torch.Generator(device="cuda")
    g.manual_seed(per_cu)
    llr = 2.0 + 2.5 * torch.randn((F + 1, 64 if N <= 64 else 128), generator=g, device="cuda")
    if prec:
        llr = torch.clamp(torch.round(4.0 * llr), -127, 127).to(torch.int8)
    d_o = torch.randint(0, B.shift_period(N), (F + 1,), generator=g, device="cuda").to(torch.uint8)
    a = dec.decode(llr[:F].contiguous(), d_o[:F].contiguous())
    b = dec.decode(llr, d_o)
    torch.cuda.synchronize()
    for x, y in zip(a[:3], b[:3]):
        assert torch.equal(x, y[:F])


def test_line_of_fewer_iterations(B):
    """The short codes leave the row-parallel kernel earlier, the long ones do not."""
    for it, per_cu in ((1, 56), (2, 56), (4, 96), (6, 160), (8, 224), (20, 224)):
        dec = make(B, "bch63_36", max_iter=it)
        assert dec.running_kernel(per_cu * cus()) == "rowpar"
        assert dec.running_kernel(per_cu * cus() + 1) == "spec_bch63_36_m122_b9"
        dec = make(B, "bch127_64", max_iter=it)
        assert dec.running_kernel(92 * cus()) == "rowpar"


@pytest.mark.parametrize("names,prec,per_cu,past", [
    (["bch127_64"], 0, 92, "per-code"), (["bch127_99"], 1, 84, "per-code"), (["bch63_36"], 0, 224, "per-code"),
    (["bch127_64", "bch127_99", "bch63_36"], 0, 192, "mix_127_64_m72_127_99_m33_63_36_m122"),
    (["bch127_64", "bch127_99", "bch63_36"], 1, 192, "mix_127_64_m72_127_99_m33_63_36_m122_fix8"),
    (["bch127_64", "bch127_99"], 0, 256, "per-code"), (["bch127_64", "bch127_99"], 1, 192, "per-code"),
    (["bch63_36", "bch63_45"], 0, 256, "per-code"),
    (["bch63_36", "bch63_45", "bch127_64", "bch127_99"], 0, 256, "mix_63_36_m122_63_45_m33_127_64_m72_127_99_m33"),
    (["bch63_36", "bch63_45", "bch127_64", "bch127_99"], 1, 256, "per-code")])
def test_both_sides_of_the_mixed_line(B, names, prec, per_cu, past):
    F = per_cu * cus()
    mix = B.MixedDecoder([make(B, n, precision=prec) for n in names])
    assert mix.running_kernel(F) == "rowpar" and mix.running_kernel(F + 1) == past
    g = torch.Generator(device="cuda")
    g.manual_seed(per_cu)
    llr = 2.0 + 2.5 * torch.randn((F + 1, mix.ld), generator=g, device="cuda")
    if prec:
        llr = torch.clamp(torch.round(4.0 * llr), -127, 127).to(torch.int8)
    idx = torch.randint(0, len(names) + 1, (F + 1,), generator=g, device="cuda").to(torch.uint8)  # some name no code
    d_o = torch.randint(0, 21, (F + 1,), generator=g, device="cuda").to(torch.uint8)
    a = mix.decode(idx[:F].contiguous(), llr[:F].contiguous(), d_o[:F].contiguous())
    b = mix.decode(idx, llr, d_o)
    torch.cuda.synchronize()
    for x, y in zip(a, b):
        assert torch.equal(x, y[:F])
