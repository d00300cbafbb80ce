"""The quantiser's four-at-a-time form against the element-wise one, and the
bucketing prepass past one step of its scan (1024 blocks of 2048 frames)."""
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


@pytest.mark.parametrize("scale", [4.0, 0.5, float("inf")])
@pytest.mark.parametrize("F,N,ld,ldq", [(1, 63, 64, 64), (77, 127, 128, 128), (1000, 127, 132, 136), (300, 63, 128, 64),
                                        (50, 4, 4, 8), (51, 5, 8, 8), (9, 1, 4, 4)])
def test_quantise_equals_element_wise(B, F, N, ld, ldq, scale):
    rng = np.random.default_rng(F + N)
    x = rng.normal(0, 20, (F, ld)).astype(np.float32)
    x[rng.random(x.shape) < 0.2] = rng.choice([0.125, -0.125, 0.49999997, -1.0, 0.0, -0.0, np.inf, -np.inf, np.nan, 1e30])
    llr = torch.from_numpy(x).cuda()
    q = torch.full((F, ldq), 99, dtype=torch.int8, device="cuda")
    B.quantize_llr(llr, N, scale, q)  # groups of four
    buf = torch.full((F * ldq + 1,), 99, dtype=torch.int8, device="cuda")
    r = buf[1:].view(F, ldq)          # an odd address: element by element
    B.quantize_llr(llr, N, scale, r)
    torch.cuda.synchronize()
    assert torch.equal(q, r) and not bool(q[:, N:].any())


@pytest.mark.parametrize("F,chunked", [(2048, 0), (2049, 0), (1024 * 2048, 0), (1024 * 2048 + 1, 0), (2_500_000, 1)])
def test_every_frame_decoded_once(B, F, chunked):
    """Frames repeat with period 20000, so their results do."""
    d = B.CODE_DEFS["bch63_45"]
    c = B.Code(d.m, d.prim, d.t)
    p = B.Pcm.build(c, target_rows=HO_ROWS["bch63_45"], seed=1)
    dec = B.Decoder(c, p, n_branches=9, max_iter=4, flags=B.SMALL_NEVER | (B.CHUNK_BUCKETS if chunked else 0))
    n = 20_000
    fr = synth.frames("bch63_45", n, 4.0, seed=81)
    idx = torch.arange(F, device="cuda").remainder(n)
    llr, d_o = torch.from_numpy(fr.llr).cuda(), torch.from_numpy(fr.d_o).cuda()
    want = dec.decode(llr, d_o)
    out = (torch.full((F, dec.W64), -1, dtype=torch.int64, device="cuda"),
           torch.zeros(F, dtype=torch.uint8, device="cuda"), torch.full((F,), 7, dtype=torch.uint8, device="cuda"))
    ws = torch.empty(dec.workspace_size(F), dtype=torch.uint8, device="cuda")
    dec.decode_into(llr[idx].contiguous(), d_o[idx].contiguous(), *out, workspace=ws)
    torch.cuda.synchronize()
    for a, b in zip(out, want):
        assert torch.equal(a, b[idx])
