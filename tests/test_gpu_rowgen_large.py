"""Calls of the generic decoder past the work-items that one dispatch counts in
32 bits (a frame per workgroup of 64 threads: 2^26 frames; of 128 threads: 2^25),
against a small call of the same frames."""
import pytest

from tests.helpers import ensure_built

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("m,prim,t,ld,F", [(3, 0b1011, 1, 8, (1 << 26) + 70), (7, 0b10001001, 1, 127, (1 << 25) + 70)])
def test_more_frames_than_a_dispatch_holds(m, prim, t, ld, F):
    B = ensure_built()
    c = B.Code(m, prim, t)
    dec = B.Decoder(c, B.Pcm.standard(c), n_branches=9, max_iter=2, flags=B.FORCE_GENERIC)
    n = 4099  # frames repeat with this period, which divides no launch size
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    llr = 2.0 + 2.0 * torch.randn((n, ld), generator=g, device="cuda")
    d_o = torch.randint(0, B.shift_period(c.N), (n,), generator=g, device="cuda").to(torch.uint8)
    want = dec.decode(llr, d_o)
    big = torch.empty((F, ld), device="cuda")
    off = torch.empty(F, dtype=torch.uint8, device="cuda")
    for f0 in range(0, F, 1024 * n):
        k = min(1024 * n, F - f0)
        big[f0:f0 + k] = llr.repeat(-(-k // n), 1)[:k]
        off[f0:f0 + k] = d_o.repeat(-(-k // n))[:k]
    out = (torch.full((F, dec.W64), -1, dtype=torch.int64, device="cuda"),
           torch.zeros(F, dtype=torch.uint8, device="cuda"), torch.full((F,), 7, dtype=torch.uint8, device="cuda"))
    dec.decode_into(big, off, *out)
    torch.cuda.synchronize()
    for got, ref in zip(out, want[:3]):
        for f0 in range(0, F, 1024 * n):
            k = min(1024 * n, F - f0)
            assert torch.equal(got[f0:f0 + k], ref.repeat(*([-(-k // n)] + [1] * (ref.dim() - 1)))[:k])
