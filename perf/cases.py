"""The decode work that users of this library have it do, as cases to time.

Each case is one pass through the public Python entry points on frames that sit
in device memory: random information bits, systematic encoding, BPSK over AWGN
at the stated Eb/N0, LLR = 2 y / sigma^2, every frame with its random cyclic
offset.  The kinds:

  decode   Decoder.decode_into with outputs and workspace kept by the program
  soft     Decoder.decode(trace=True): the decision and the posterior of every
           iteration, buffers made by the call
  fixed    the int8 front end and decoder: draw_offsets on the device,
           quantize_llr, decode_into
  hybrid   decode_into, then order-2 OSD of the frames that did not converge
  mixed    the device work of one service step: frames of four codes in one
           MixedDecoder call, then order-2 OSD of the failures

Codes, matrices, Eb/N0 ranges, iteration limits and sizes are those of
bench.py and the tests: calls of one frame to the seven-point sweep of
1,000,000 frames per point.
"""
import functools
import math

import numpy as np
import torch

from paper_2412_20828_amd import binding as B

DEV = "cuda:0"
# rows of H_o with a kernel of their own (Table 1's dimensions)
ROWS = {"bch63_36": 122, "bch63_45": 33, "bch127_64": 72, "bch127_78": 57, "bch127_99": 33}
SERVE = ["bch63_36", "bch63_45", "bch127_64", "bch127_99"]  # the service's codes, in its order
MODES = {"restart": B.MODE_RESTART, "memory": B.MODE_MEMORY, "extrinsic": B.MODE_EXTRINSIC}


def _case(kind, code, frames, lo, hi, rows=None, branches=9, mode="restart", iters=8, int8=False):
    return {"kind": kind, "code": code, "rows": ROWS.get(code, 0) if rows is None else rows, "frames": frames,
            "lo": lo, "hi": hi, "branches": branches, "mode": mode, "iters": iters, "int8": int8}


def listed():
    out = []

    def add(name, *a, **k):
        out.append({"name": name, **_case(*a, **k)})

    # one code block arrives and its word is wanted: the smallest call
    add("one_frame", "decode", "bch127_64", 1, 3.0, 3.0)
    # a control message of a few hundred short blocks
    add("packet63", "decode", "bch63_45", 193, 3.0, 3.0)
    # posteriors of every iteration for a soft-output receiver or a study
    add("soft127", "soft", "bch127_64", 1021, 3.0, 3.0)
    # the fixed-point receiver from float LLRs to words, a service-sized batch
    add("fixed127", "fixed", "bch127_99", 4096, 4.0, 4.0, int8=True)
    # ordinary batches of both lengths
    add("batch127", "decode", "bch127_64", 16384, 3.0, 3.0)
    add("batch63", "decode", "bch63_36", 50021, 3.0, 3.0)
    # one step of the continuous-batching service, mixed codes with OSD-2
    add("mixed_step", "mixed", "serve", 8192, 2.0, 5.0)
    # the hybrid decoder on the code with the largest OSD search
    add("hybrid127", "hybrid", "bch127_99", 20011, 3.0, 3.0)
    # a matrix of the user's own (48 rows): no kernel was compiled for it
    add("own_matrix63", "decode", "bch63_36", 20000, 3.0, 3.0, rows=48)
    # plain min-sum on the standard matrix, the usual baseline of a study
    add("plain127", "decode", "bch127_64", 10007, 3.0, 3.0, rows=0, branches=1, mode="extrinsic", iters=12)
    # an error-rate point in fixed point
    add("point127_int8", "decode", "bch127_99", 4000000, 4.0, 4.0, int8=True)
    # an error-rate sweep of seven points in one call: the largest
    add("sweep127", "decode", "bch127_64", 7000000, 2.0, 5.0)
    return out


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode", "decode", "decode", "soft", "fixed", "hybrid", "mixed", "own", "own", "plain"])
    e = rng.uniform(2.0, 5.0)
    spread = rng.random() < 0.3  # Eb/N0 drawn per frame instead of one value
    lo, hi = (2.0, 5.0) if spread else (e, e)
    code = rng.choice(sorted(ROWS))
    if kind == "decode":
        int8 = code != "bch127_78" and rng.random() < 0.35
        return _case("decode", code, _log(rng, 1, 3000000), lo, hi, int8=int8)
    if kind == "soft":
        return _case("soft", code, _log(rng, 1, 5000), lo, hi)
    if kind == "fixed":
        code = rng.choice(SERVE)
        return _case("fixed", code, _log(rng, 1, 500000), lo, hi, int8=True)
    if kind == "hybrid":
        return _case("hybrid", code, _log(rng, 1, 100000), lo, hi)
    if kind == "mixed":
        return _case("mixed", "serve", _log(rng, 1, 65536), 2.0, 5.0)
    if kind == "own":
        mode = rng.choice(["restart", "restart", "memory", "extrinsic"])
        base = 27 if code == "bch63_36" else (18 if code == "bch63_45" else (28 if code == "bch127_99" else 63))
        rows = base + 8 + rng.randrange(0, 40)
        while rows in (ROWS[code], 47, 49, 57, 65):
            rows += 1
        branches = rng.choice([9, 9, 3, 1])
        return _case("decode", code, _log(rng, 1, 20000 if mode == "restart" else 4000), lo, hi, rows=rows,
                     branches=branches, mode=mode)
    return _case("decode", code, _log(rng, 1, 20000), lo, hi, rows=0, branches=1, mode="extrinsic", iters=12)


# what a user's program builds once and keeps: codes, matrices, decoders

@functools.lru_cache(maxsize=None)
def _code(name):
    d = B.CODE_DEFS[name]
    return B.Code(d.m, d.prim, d.t)


@functools.lru_cache(maxsize=None)
def _pcm(name, rows):
    return B.Pcm.standard(_code(name)) if rows == 0 else B.Pcm.build(_code(name), target_rows=rows, seed=1)


@functools.lru_cache(maxsize=None)
def _decoder(name, rows, branches, mode, iters, int8):
    return B.Decoder(_code(name), _pcm(name, rows), n_branches=branches, mode=MODES[mode], alpha=0.75,
                     max_iter=iters, precision=B.FIX8 if int8 else B.FP32)


@functools.lru_cache(maxsize=None)
def _generator(name):
    return torch.from_numpy(_code(name).export()[1].astype(np.float32)).to(DEV)


def _rng(case, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed((seed * 1000003 + case["frames"]) & 0x7FFFFFFF)
    return g


def _channel(name, F, ld, lo, hi, g):
    """[F][ld] LLRs of F random codewords and their offsets d_o."""
    code = _code(name)
    G = _generator(name)
    llr = torch.zeros((F, ld), dtype=torch.float32, device=DEV)
    for f0 in range(0, F, 1000000):
        n = min(1000000, F - f0)
        msg = torch.randint(0, 2, (n, code.K), generator=g, device=DEV).to(torch.float32)
        cw = torch.remainder(msg @ G, 2.0)
        e = lo + (hi - lo) * torch.rand((n, 1), generator=g, device=DEV)
        s2 = 1.0 / (2.0 * (code.K / code.N) * torch.pow(10.0, e / 10.0))
        y = (1.0 - 2.0 * cw) + torch.sqrt(s2) * torch.randn((n, code.N), generator=g, device=DEV)
        llr[f0:f0 + n, :code.N] = (2.0 / s2) * y
    d_o = torch.randint(0, B.shift_period(code.N), (F,), generator=g, device=DEV).to(torch.uint8)
    return llr, d_o


def _ld(N):
    return 64 if N <= 64 else 128


def _outputs(F, W64):
    return (torch.zeros((F, W64), dtype=torch.int64, device=DEV), torch.zeros(F, dtype=torch.uint8, device=DEV),
            torch.zeros(F, dtype=torch.uint8, device=DEV))


def prepare(case, seed):
    F, kind = case["frames"], case["kind"]
    g = _rng(case, seed)
    if kind == "mixed":
        decs = [_decoder(n, ROWS[n], 9, "restart", case["iters"], False) for n in SERVE]
        mix = B.MixedDecoder(decs)
        idx = torch.randint(0, len(SERVE), (F,), generator=g, device=DEV).to(torch.uint8)
        llr = torch.zeros((F, mix.ld), dtype=torch.float32, device=DEV)
        d_o = torch.zeros(F, dtype=torch.uint8, device=DEV)
        for c, n in enumerate(SERVE):
            x, d = _channel(n, F, mix.ld, case["lo"], case["hi"], g)
            llr[idx == c], d_o[idx == c] = x[idx == c], d[idx == c]
        ws = torch.empty(max(1, mix.workspace_size(F)), dtype=torch.uint8, device=DEV)
        return {"kind": kind, "mix": mix, "idx": idx, "llr": llr, "d_o": d_o, "ws": ws, "out": _outputs(F, mix.W64)}
    code = _code(case["code"])
    llr, d_o = _channel(case["code"], F, _ld(code.N), case["lo"], case["hi"], g)
    dec = _decoder(case["code"], case["rows"], case["branches"], case["mode"], case["iters"], case["int8"])
    st = {"kind": kind, "dec": dec, "llr": llr, "d_o": d_o, "seed": seed}
    if kind == "soft":
        return st
    st["ws"] = torch.empty(max(1, dec.workspace_size(F)), dtype=torch.uint8, device=DEV)
    st["out"] = _outputs(F, dec.W64)
    if case["int8"]:
        st["q"] = torch.empty(llr.shape, dtype=torch.int8, device=DEV)
        if kind == "decode":
            B.quantize_llr(llr, code.N, 4.0, st["q"])
            st["llr"] = st["q"]
    return st


def run(state):
    kind = state["kind"]
    llr, d_o = state["llr"], state["d_o"]
    if kind == "soft":
        return state["dec"].decode(llr, d_o, trace=True)
    bits, iters, flags = state["out"]
    if kind == "mixed":
        mix = state["mix"]
        mix.decode_into(state["idx"], llr, d_o, bits, iters, flags, state["ws"])
        mix.osd_into(state["idx"], llr, 2, bits, skip=flags)
        return bits, iters, flags
    dec = state["dec"]
    if kind == "fixed":
        B.draw_offsets(dec.N, state["seed"], 7, 0, llr.shape[0], out=d_o)
        B.quantize_llr(llr, dec.N, 4.0, state["q"])
        dec.decode_into(state["q"], d_o, bits, iters, flags, workspace=state["ws"])
        return state["q"], d_o, bits, iters, flags
    dec.decode_into(llr, d_o, bits, iters, flags, workspace=state["ws"])
    if kind == "hybrid":
        dec.osd_into(llr, 2, bits, skip=flags)
    return bits, iters, flags


# mean iterations a frame of these ranges runs (stopping included), for work()
MEAN_ITERS = 4.0


def work(case):
    F = case["frames"]
    if case["kind"] == "mixed":
        parts = [_case("decode", n, F / len(SERVE), case["lo"], case["hi"]) for n in SERVE]
        ws = [work(p) for p in parts]
        return {"bytes": sum(w["bytes"] for w in ws), "flops": sum(w["flops"] for w in ws)}
    code = _code(case["code"])
    N, K, W = code.N, code.K, (code.N + 63) // 64
    pcm = _pcm(case["code"], case["rows"])
    nb = case["branches"]
    in_bytes = N * (1 if case["int8"] and case["kind"] == "decode" else 4) + 1
    nbytes = in_bytes + 8 * W + 2
    if case["kind"] == "fixed":
        nbytes += N
    if case["kind"] == "soft":
        nbytes += MEAN_ITERS * N * 4
    # per edge: minimum search 3, sign 1, selection and sign 2, sum 1
    ops = 7.0 * nb * pcm.E + 2.0 * nb * (pcm.M + N) + 2.0 * (N - K) * W
    return {"bytes": F * nbytes, "flops": F * MEAN_ITERS * ops}


def exact(case, seed):
    """The posteriors of the soft case in 64 bits: Algorithm 1 with restarted
    messages, nine branches.  The other outputs are decisions and counts."""
    if case["kind"] != "soft":
        return None
    name, F, T = case["code"], case["frames"], case["iters"]
    code = _code(name)
    llr, d_o = _channel(name, F, _ld(code.N), case["lo"], case["hi"], _rng(case, seed))
    N, dp = code.N, B.shift_period(code.N)
    H = torch.from_numpy(_pcm(name, case["rows"]).dense().astype(np.float64)).to(DEV)
    Hs = torch.from_numpy(code.export()[2].astype(np.float64)).to(DEV)
    y = llr[:, :N].to(torch.float64)
    out = torch.zeros((F, T, llr.shape[1]), dtype=torch.float64, device=DEV)
    live = torch.ones(F, dtype=torch.bool, device=DEV)
    j = torch.arange(N, device=DEV)
    rows = [torch.nonzero(H[r])[:, 0] for r in range(H.shape[0])]
    for t in range(T):
        total = torch.zeros_like(y)
        for s in range(3):
            for a in (1, 2, (N + 1) // 2):
                # branch (s, p) reads Y[j] = y[a (j - s d_p - d_o) mod N]
                pos = (a * (j[None, :] - s * dp - d_o.to(torch.int64)[:, None])) % N
                Y = torch.gather(y, 1, pos)
                mag, neg = Y.abs(), Y < 0
                c2v = torch.zeros_like(Y)
                for cols in rows:
                    m = mag[:, cols]
                    two = torch.topk(m, 2, dim=1, largest=False)
                    sel = torch.where(two.indices[:, 0:1] == torch.arange(len(cols), device=DEV)[None, :],
                                      two.values[:, 1:2], two.values[:, 0:1])
                    ng = neg[:, cols]
                    sign = 1.0 - 2.0 * ((ng.sum(1, keepdim=True) % 2).to(torch.float64))
                    c2v[:, cols] += sign * (1.0 - 2.0 * ng.to(torch.float64)) * sel
                total.scatter_add_(1, pos, c2v)
        yn = y + 0.75 * total / 9.0
        out[live, t, :N] = yn[live]
        y = torch.where(live[:, None], yn, y)
        hard = (y < 0).to(torch.float64)
        live = live & ((hard @ Hs.T) % 2 != 0).any(1)
    return None, None, None, out
