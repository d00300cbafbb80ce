"""Row signs from the syndrome bits of one dual codeword (gen_spec.Dual): the
generated dual_bits and the rows' masks, run here on random sign strings,
against the parity of each row's signs, at every cyclic shift the kernels use."""
import re

import numpy as np
import pytest

from paper_2412_20828_amd import gen_spec
from tests.helpers import oracle_code, oracle_hopt


def run_dual_bits(src, S):
    """The generated assignments with Python's integers."""
    env = {"S": [int(x) for x in S], "Z": [0] * 4}
    for line in re.findall(r"(?:const uint32_t )?(e\d+|Z\[\d\]) = (.*);", src):
        expr = re.sub(r"__builtin_amdgcn_alignbit\((\w+), (\w+), (\d+)\)",
                      r"((((\1 << 32) | \2) >> \3) & 0xffffffff)", line[1])
        exec("%s = (%s) & 0xffffffff" % (line[0], expr), env)
    return env["Z"]


@pytest.mark.parametrize("name,rows", [("bch127_64", 72), ("bch127_78", 57), ("bch127_99", 33), ("bch63_36", 122),
                                       ("bch63_45", 33)])
def test_row_signs(name, rows):
    H, c = oracle_hopt(name, rows), oracle_code(name)
    N, n = H.shape[1], c.N - c.K
    dual = gen_spec.Dual(H, n)
    src = dual.source()
    rng = np.random.default_rng(5)
    mats = gen_spec.shift_matrices(H, {63: 21, 127: 42}[N])
    for _ in range(6):
        neg = rng.integers(0, 2, N)
        S = [0] * ((N + 31) // 32)
        for i in range(N):
            S[i >> 5] = (S[i >> 5] << 1 | int(neg[i])) & 0xFFFFFFFF
        Z = run_dual_bits(src, S)
        for Hs in mats:
            for row in Hs:
                masks = dual.masks(np.nonzero(row)[0].tolist())
                got = sum(bin(z & m).count("1") for z, m in zip(Z, masks)) & 1
                assert got == int(neg[row == 1].sum()) & 1


def test_syndrome_bits_vanish_on_codewords_only():
    """All bits of Z zero exactly where the standard matrix's syndrome is."""
    c = oracle_code("bch127_99")
    dual = gen_spec.Dual(oracle_hopt("bch127_99", 33), c.N - c.K)
    src = dual.source()
    rng = np.random.default_rng(6)
    for k in range(20):
        w = np.zeros(c.N, int)
        for g in np.nonzero(rng.integers(0, 2, c.K))[0]:  # a codeword: shifts of the generator
            w ^= np.roll(_generator_row(c), g)
        if k % 2:
            w[rng.integers(0, c.N)] ^= 1
        S = [0] * 4
        for i in range(c.N):
            S[i >> 5] = (S[i >> 5] << 1 | int(w[i])) & 0xFFFFFFFF
        zero = not any(run_dual_bits(src, S)[:(dual.n + 31) // 32])
        assert zero == (not (np.asarray(c.Hstd) @ w % 2).any()) == (k % 2 == 0)


def _generator_row(c):
    """A codeword whose shifts span the code: the least-degree one."""
    H = np.asarray(c.Hstd, int)
    M = H[:, :c.N - c.K + 1].copy()  # N - K + 1 first columns have one dependency
    piv, r = [], 0
    for j in range(M.shape[1]):
        p = next((i for i in range(r, len(M)) if M[i, j]), None)
        if p is None:
            free = j
            continue
        M[[r, p]] = M[[p, r]]
        for i in range(len(M)):
            if i != r and M[i, j]:
                M[i] ^= M[r]
        piv.append(j)
        r += 1
    w = np.zeros(c.N, int)
    w[free] = 1
    for i, j in enumerate(piv):
        w[j] = M[i, free]
    return w


def test_rows_outside_the_dual_code_are_refused():
    H = oracle_hopt("bch127_99", 33)
    dual = gen_spec.Dual(H, 28)
    with pytest.raises(ValueError, match="outside"):
        dual.masks([0, 1, 2])
    with pytest.raises(ValueError, match="spans"):
        gen_spec.Dual(H, 29)
