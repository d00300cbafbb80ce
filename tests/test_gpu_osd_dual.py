"""Device OSD by the parity side (codes with N - K <= 64) against the host OSD,
bit for bit: every instance of the kernel (tiles of basis positions, depth),
short codes, orders 0 to 2, ties, infinite reliabilities, skipped frames and
mixed calls with and without a code that needs the generator-side kernel."""
import numpy as np
import pytest

from tests.helpers import ensure_built

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

PRIM = {3: 0b1011, 4: 0b10011, 5: 0b100101, 6: 0b1000011, 7: 0b10001001}
# (m, t): N - K <= 32 with up to 3, 4, 7, 8 tiles; 33..64 with 3, 4, 5, 7; short codes; N - K > 64
CODES = [(6, 5), (6, 2), (7, 4), (7, 2), (6, 7), (7, 10), (7, 7), (7, 6), (5, 3), (4, 2), (3, 1), (3, 3), (7, 11)]


@pytest.fixture(scope="module")
def B():
    b = ensure_built()
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return b


def make(B, m, t):
    c = B.Code(m, PRIM[m], t)
    return c, B.Decoder(c, B.Pcm.standard(c), n_branches=1, mode=B.MODE_EXTRINSIC, max_iter=2)


def frames(N, n, seed):
    """n noisy frames, n integer-valued (ties), a few flat, zero and infinite ones."""
    rng = np.random.default_rng(seed)
    x = (2.0 + 2.5 * rng.standard_normal((2 * n, N))).astype(np.float32)
    x[n:] = np.round(x[n:])
    flat = np.where(rng.random((6, N)) < 0.5, -2.5, 2.5).astype(np.float32)
    flat[0] = 0.0
    inf = x[:6].copy()
    inf[rng.random((6, N)) < 0.1] = np.inf
    inf[:, 0] = -np.inf
    big = x[:4] * np.float32(1e30)
    tiny = x[:4] * np.float32(1e-40)
    return np.concatenate([x, flat, inf, big, tiny]).astype(np.float32)


@pytest.mark.parametrize("m,t", CODES)
def test_equals_host_osd(B, m, t):
    c, dec = make(B, m, t)
    ld = 64 if c.N <= 64 else 128
    x = frames(c.N, 60, seed=10 * m + t)
    llr = np.zeros((x.shape[0], ld), np.float32)
    llr[:, :c.N] = x
    dev = torch.from_numpy(llr).cuda()
    skip = (np.arange(len(llr)) % 7 == 3).astype(np.uint8)
    for order in (0, 1, 2):
        bits = torch.full((len(llr), dec.W64 + 1), -3, dtype=torch.int64, device="cuda")
        dec.osd_into(dev, order, bits, skip=torch.from_numpy(skip).cuda())
        torch.cuda.synchronize()
        got = bits.cpu().numpy()
        ref = np.full((len(llr), dec.W64), -3, np.int64).view(np.uint64)
        B.osd_decode(c, llr, order, skip=skip, bits=ref)
        assert np.array_equal(got[:, :dec.W64], ref.view(np.int64)), order
        assert (got[:, dec.W64:] == -3).all() and (got[skip != 0] == -3).all()


@pytest.mark.parametrize("codes", [[(6, 5), (7, 10), (7, 4)], [(7, 4), (6, 5), (7, 11)], [(5, 3)]])
def test_mixed_equals_host_osd(B, codes):
    pairs = [make(B, m, t) for m, t in codes]
    rng = np.random.default_rng(4)
    F = 300
    idx = rng.integers(0, len(codes) + 1, F).astype(np.uint8)  # some frames name no code
    llr = (1.5 + 2.0 * rng.standard_normal((F, 128))).astype(np.float32)
    bits = torch.full((F, 2), -3, dtype=torch.int64, device="cuda")
    mix = B.MixedDecoder([d for _, d in pairs])
    mix.osd_into(torch.from_numpy(idx).cuda(), torch.from_numpy(llr).cuda(), 2, bits)
    torch.cuda.synchronize()
    got = bits.cpu().numpy()
    for k, (c, d) in enumerate(pairs):
        sel = np.nonzero(idx == k)[0]
        ref = B.osd_decode(c, llr[sel], 2)
        assert np.array_equal(got[sel][:, :d.W64], ref.view(np.int64))
    assert (got[idx == len(codes)] == -3).all()


def test_more_frames_than_waves(B):
    """A wave looks at 64 frames ahead in strides of the grid; failures sparse
    and clustered."""
    c, dec = make(B, 6, 5)
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    F = n_cu * 64 * 64 + 12345
    rng = np.random.default_rng(9)
    rows = np.unique(np.concatenate([np.arange(150), rng.integers(0, F, 150), [F - 1, n_cu * 64, n_cu * 64 * 64]]))
    llr = torch.zeros((F, 64), device="cuda")
    x = np.zeros((len(rows), 64), np.float32)
    x[:, :63] = 1.5 + 2.0 * rng.standard_normal((len(rows), 63))
    at = torch.from_numpy(rows).cuda()
    llr[at] = torch.from_numpy(x).cuda()
    skip = torch.ones(F, dtype=torch.uint8, device="cuda")
    skip[at] = 0
    bits = torch.full((F, 1), -3, dtype=torch.int64, device="cuda")
    dec.osd_into(llr, 2, bits, skip=skip)
    torch.cuda.synchronize()
    assert np.array_equal(bits[at].cpu().numpy(), B.osd_decode(c, x, 2).view(np.int64))
    assert int((bits != -3).sum()) <= len(rows) and int((bits == -3).sum()) == F - len(rows)
