"""Device OSD of hard decisions of infinite reliability, with errors, erasures and
finite positions among them, against the host OSD, bit for bit: the parity-side
kernel and the generator-side one of codes with N - K > 64."""
import numpy as np
import pytest

from tests.helpers import ensure_built

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

PRIM = {6: 0b1000011, 7: 0b10001001}


@pytest.mark.parametrize("m,t", [(6, 3), (6, 5), (7, 4), (7, 10), (7, 11), (7, 14)])
@pytest.mark.parametrize("p_inf,p_zero", [(1.0, 0.0), (0.9, 0.1), (0.5, 0.0), (0.02, 0.0)])
def test_equals_host_osd(m, t, p_inf, p_zero):
    B = ensure_built()
    c = B.Code(m, PRIM[m], t)
    dec = B.Decoder(c, B.Pcm.standard(c), n_branches=1, mode=B.MODE_EXTRINSIC, max_iter=2)
    rng = np.random.default_rng(m + t)
    F = 200
    x = (1.5 + 2.0 * rng.standard_normal((F, 64 if c.N <= 64 else 128))).astype(np.float32)
    u = rng.random(x.shape)
    x = np.where(u < p_inf, np.copysign(np.float32(np.inf), x), np.where(u < p_inf + p_zero, np.float32(0), x))
    x = np.ascontiguousarray(x, dtype=np.float32)
    for order in (0, 1, 2):
        bits = torch.full((F, dec.W64), -3, dtype=torch.int64, device="cuda")
        dec.osd_into(torch.from_numpy(x).cuda(), order, bits)
        torch.cuda.synchronize()
        assert np.array_equal(bits.cpu().numpy(), B.osd_decode(c, x, order).view(np.int64)), order
