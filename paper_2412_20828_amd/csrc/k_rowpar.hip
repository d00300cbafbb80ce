// Row-parallel enhanced-NMS decoder for small and middle batches: restart
// message mode, nine branches, one workgroup of three waves per frame
// (Algorithm 1 of Section III-B, eqs. 2-5).
//
// The lane-per-frame kernels run an iteration of 64 frames in the time one
// wave needs for a type's three row functions, about 58 us for the 127-bit
// codes however few frames there are.  Here a frame's rows and coordinates
// are spread over the lanes instead.  Wave p owns automorphism type p; with
// B_p[k] = y[a_p (k - d_o) mod N] the input of its shift 0, branch (p, s)
// reads B_p[i - s d_p].  Per iteration, in wave p:
//   1. lane = coordinate k: |B_p[k]| to the extended input (cells x = k + 2 d_p
//      and, wrapped, x - N), so that branch s reads column i at cell
//      i - s d_p + 2 d_p with no reduction; the signs become a ballot word;
//   2. lane = row (s, r) of the 3 M rows, 64 a round: min1, min2 of its cells
//      and the parity of its signs to the row's record {sign | min1, min2};
//   3. lane = coordinate: the c2v of its rows, shift by shift, rows ascending,
//      selected with med3(min1, min2, min1 + min2 - |B_p[k]|) and summed;
//   4. after the only barrier of the iteration: each wave takes the three
//      types' sums at its coordinates, forms y^(t), and has the input of its
//      next iteration in registers; the syndrome is tested on each type's own
//      ordering of the word (the automorphisms preserve the code), so the
//      three waves reach the same decision without exchanging it.
// Cells and records are named by tables (rowpar.h) that depend on neither the
// frame nor d_o, so frames need no bucketing and a call is one launch of one
// workgroup per frame, handed out by the hardware as others end.  The sums are
// formed in the order of the lane-per-frame kernels: the results are theirs
// bit for bit.
//
// What bounds it: VALU issue.  An iteration of BCH(127,64) takes 2,900 VALU
// instructions of a frame's three waves (6 per edge in step 3, 3.7 in step 2:
// unpacking an address, the search), issued at 1.1 per CU-cycle with the LDS
// 57% busy: 1.15-1.35 us per frame-iteration and CU, twice the lane-per-frame
// kernels' figure at full load, but from the first frame on.  One frame at
// 3 dB: 39 us against 451; 4,096 frames: 173 against 470; the mixed call of
// 8,192 frames over four codes: 165 against 1,425.
// Forms measured and not taken (16,384 frames of (127,64)): records of 12 or
// 16 bytes with min1 + min2 and the sign as a factor save one and two
// instructions an edge, but 96- and 128-bit LDS reads cost more than that
// (723 and 672 us against 602); two and four frames side by side in a
// workgroup share addresses, but idle slots and fewer waves take it back (656
// and 768 against 615); eight records of a step in flight instead of four
// cost registers, and with them waves, for N = 127 (1,142 against 1,073 us at
// 32,768 frames) and pay for N = 63 (398 against 418).
#include <hip/hip_runtime.h>

#include "rowpar.h"

namespace bch {
namespace {

constexpr int WAVE = 64;
constexpr int TYPES = 3;
constexpr int B = 9;

__device__ __forceinline__ uint32_t med3i(uint32_t a, uint32_t b, uint32_t c)
{
    return __float_as_uint(__builtin_amdgcn_fmed3f(__uint_as_float(a), __uint_as_float(b), __uint_as_float(c)));
}

// ordering of a wave's own LDS traffic: LDS operations of a wave complete in
// order, so only the compiler has to keep them so
__device__ __forceinline__ void wave_order()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

struct StepWord {
    uint32_t x, y, z;
};

// a x mod N for the multipliers a_0 = 1, a_1 = 2, a_2 = (N + 1) / 2 (0 <= x < N)
__device__ __forceinline__ int times(int p, int x, int N)
{
    const int dbl = 2 * x >= N ? 2 * x - N : 2 * x;
    const int hlf = (x & 1) ? (x + N) >> 1 : x >> 1;
    return p == 0 ? x : (p == 1 ? dbl : hlf);
}

template <int NK, bool FIX8>
__device__ __forceinline__ void decode_frame(const RowParArgs &A, const RowParTab &tb, int64_t f, char *lds, int p,
                                             int lane)
{
    const int N = tb.N, M = tb.M, dp = tb.dp;
    const int ext = N + 2 * dp;
    const int ext_pad = (ext + 4) & ~3;
    const int nrec = 3 * M + 2;
    constexpr int US = NK * WAVE;  // sums of one type
    char *Eb = lds + 4 * p * ext_pad;
    char *Rb = lds + 4 * TYPES * ext_pad + 8 * p * nrec;
    float *Ubase = reinterpret_cast<float *>(lds + 4 * TYPES * ext_pad + 8 * TYPES * nrec);
    float *E = reinterpret_cast<float *>(Eb);
    const int d_o = (int)A.d_o[f] % dp;
    // ---- this lane's coordinates k = lane, lane + 64
    float y[NK];
    int u[NK], src[NK][TYPES];
    bool in[NK];
#pragma unroll
    for (int j = 0; j < NK; j++) {
        in[j] = lane + j * WAVE < N;
        const int kk = in[j] ? lane + j * WAVE : 0;
        u[j] = times(p, kk >= d_o ? kk - d_o : kk - d_o + N, N);
#pragma unroll
        for (int q = 0; q < TYPES; q++) {
            // type q holds coordinate u at k_q = a_q^-1 u + d_o (a_1 a_2 = 1 mod N)
            const int kq = times(q == 0 ? 0 : TYPES - q, u[j], N) + d_o;
            src[j][q] = q * US + (kq >= N ? kq - N : kq);
        }
        if (FIX8)
            y[j] = in[j] ? (float)static_cast<const int8_t *>(A.llr)[f * A.ld + u[j]] : 1.0f;
        else
            y[j] = in[j] ? static_cast<const float *>(A.llr)[f * A.ld + u[j]] + 0.0f : 1.0f;
    }
    // ---- parity rows of the syndrome, one or two per lane
    uint64_t hs[2][NK];
#pragma unroll
    for (int r = 0; r < 2; r++)
#pragma unroll
        for (int w = 0; w < NK; w++) {
            const int row = lane + r * WAVE;
            hs[r][w] = row < tb.msyn ? tb.hsyn[row * NK + w] : 0ull;
        }
    if (lane == 0) {
        E[ext] = __builtin_inff();
        *reinterpret_cast<uint2 *>(Rb + 8 * (3 * M)) = make_uint2(0u,0u);
    }
    const float scale = tb.alpha / (float)B;
    for (int t = 1;; t++) {
        // ---- 1. input of the type
        uint64_t W[NK];
        float a[NK];
#pragma unroll
        for (int j = 0; j < NK; j++) {
            const int k = lane + j * WAVE;
            W[j] = __ballot(in[j] && (__float_as_uint(y[j]) >> 31));
            a[j] = FIX8 ? fminf(fabsf(y[j]), 127.0f) : __builtin_canonicalizef(fabsf(y[j]));
            if (in[j]) {
                E[k + 2 * dp] = a[j];
                if (k >= N - 2 * dp)
                    E[k + 2 * dp - N] = a[j];
            }
        }
        wave_order();
        // ---- 2. rows
        {
            const StepWord *sp = reinterpret_cast<const StepWord *>(tb.steps);
            StepWord nx = sp[lane];
            for (int q = 0; q < tb.n_rounds; q++) {
                const int ns = __builtin_amdgcn_readfirstlane(tb.rounds[q]);
                const uint4 mk = tb.mask[q * WAVE + lane];
                const uint32_t slot = tb.slot[q * WAVE + lane];
                uint32_t u1 = 0x7f800000u, u2 = 0x7f800000u;
#pragma unroll 2
                for (int e = 0; e < ns; e++) {
                    const StepWord st = nx;
                    sp += WAVE;
                    nx = sp[lane];
                    uint32_t v[6];
                    v[0] = *reinterpret_cast<const uint32_t *>(Eb + (st.x & 0xffffu));
                    v[1] = *reinterpret_cast<const uint32_t *>(Eb + (st.x >> 16));
                    v[2] = *reinterpret_cast<const uint32_t *>(Eb + (st.y & 0xffffu));
                    v[3] = *reinterpret_cast<const uint32_t *>(Eb + (st.y >> 16));
                    v[4] = *reinterpret_cast<const uint32_t *>(Eb + (st.z & 0xffffu));
                    v[5] = *reinterpret_cast<const uint32_t *>(Eb + (st.z >> 16));
                    const uint32_t ma = min(min(v[0], v[1]), v[2]), sa = med3i(v[0], v[1], v[2]);
                    const uint32_t mb = min(min(v[3], v[4]), v[5]), sb = med3i(v[3], v[4], v[5]);
                    u2 = min(med3i(u1, ma, mb), min(min(u2, sa), sb));
                    u1 = min(min(u1, ma), mb);
                }
                uint32_t par = ((uint32_t)W[0] & mk.x) ^ ((uint32_t)(W[0] >> 32) & mk.y);
                if (NK == 2)
                    par ^= ((uint32_t)W[NK - 1] & mk.z) ^ ((uint32_t)(W[NK - 1] >> 32) & mk.w);
                const uint32_t sg = (uint32_t)__builtin_popcount(par) << 31;
                const float m1 = __uint_as_float(u1), m2 = __uint_as_float(u2);
                uint2 rec;
                if (FIX8) {
                    // min1 and the signed c2v (3 m + 2) >> 2 of min1, min2
                    const float q1 = floorf(__builtin_fmaf(m1, 0.75f, 0.5f));
                    const float q2 = floorf(__builtin_fmaf(m2, 0.75f, 0.5f));
                    const int c1 = sg ? -(int)q1 : (int)q1, c2 = sg ? -(int)q2 : (int)q2;
                    rec = make_uint2(u1, ((uint32_t)c1 & 0xffffu) | ((uint32_t)c2 << 16));
                } else {
                    rec = make_uint2(u1 | sg, u2);
                }
                *reinterpret_cast<uint2 *>(Rb + slot) = rec;
            }
        }
        wave_order();
        // ---- 3. c2v sums of the coordinates
        float *U = Ubase + (t & 1) * TYPES * US;
        {
            float T[NK];
            int Ti[NK];
            uint2 nx[NK];
            const uint2 *rp = tb.recs;
#pragma unroll
            for (int j = 0; j < NK; j++) {
                T[j] = 0.0f;
                Ti[j] = 0;
                nx[j] = rp[lane + j * WAVE];
            }
            // the first n of a chunk's records
            auto add = [&](const uint2 *id, int n) {
                uint2 rc[NK][kRpRecs];
#pragma unroll
                for (int j = 0; j < NK; j++) {
                    const uint32_t at[kRpRecs] = {id[j].x & 0xffffu, id[j].x >> 16, id[j].y & 0xffffu, id[j].y >> 16};
#pragma unroll
                    for (int e = 0; e < kRpRecs; e++)
                        rc[j][e] = *reinterpret_cast<const uint2 *>(Rb + at[e]);
                }
#pragma unroll
                for (int e = 0; e < kRpRecs; e++) {
                    if (e >= n)
                        break;
#pragma unroll
                    for (int j = 0; j < NK; j++) {
                        const uint2 r = rc[j][e];
                        if (FIX8) {
                            const int pk = (int)r.y;
                            Ti[j] += r.x == __float_as_uint(a[j]) ? pk >> 16 : (int)(int16_t)pk;
                        } else {
                            const float s1 = __uint_as_float(r.x), m1 = fabsf(s1), m2 = __uint_as_float(r.y);
                            T[j] += __builtin_copysignf(__builtin_amdgcn_fmed3f(m1, m2, (m1 + m2) - a[j]), s1);
                        }
                    }
                }
            };
            const int whole = tb.n_recs / kRpRecs;
#pragma unroll(NK == 1 ? 2 : 1)
            for (int c = 0; c < whole; c++) {
                uint2 id[NK];
                rp += NK * WAVE;
#pragma unroll
                for (int j = 0; j < NK; j++) {
                    id[j] = nx[j];
                    nx[j] = rp[lane + j * WAVE];
                }
                add(id, kRpRecs);
            }
            switch (tb.n_recs % kRpRecs) {
            case 1: add(nx, 1); break;
            case 2: add(nx, 2); break;
            case 3: add(nx, 3); break;
            }
#pragma unroll
            for (int j = 0; j < NK; j++)
                U[p * US + lane + j * WAVE] = FIX8 ? (float)Ti[j] : T[j];
        }
        __syncthreads();
        // ---- 4. merge in type order, posterior, decision, syndrome
        uint64_t w[NK];
#pragma unroll
        for (int j = 0; j < NK; j++) {
            const float s = (U[src[j][0]] + U[src[j][1]]) + U[src[j][2]];
            float yn;
            if (FIX8) {
                // branch sum sgn(y) s; average sign(s) ((|s| + B/2) / B)
                const int q = ((int)fabsf(s) + B / 2) / B;
                const float qs = __uint_as_float(__float_as_uint((float)q) ^
                                                 ((__float_as_uint(s) ^ __float_as_uint(y[j])) & 0x80000000u));
                yn = fminf(fmaxf(y[j] + qs, -32767.0f), 32767.0f);
            } else {
                const float d = scale * s;
                yn = y[j] + __uint_as_float(__float_as_uint(d) ^ (__float_as_uint(y[j]) & 0x80000000u));
            }
            y[j] = in[j] ? yn : 1.0f;
            w[j] = __ballot(in[j] && (__float_as_uint(yn) >> 31));
            if (A.trace && p == 0 && in[j]) {
                const int64_t at = (f * tb.max_iter + (t - 1)) * A.ld + u[j];
                if (FIX8)
                    static_cast<int32_t *>(A.trace)[at] = (int32_t)yn;
                else
                    static_cast<float *>(A.trace)[at] = yn;
            }
        }
        uint32_t odd = 0;
#pragma unroll
        for (int r = 0; r < 2; r++) {
            uint64_t x = hs[r][0] & w[0];
            if (NK == 2)
                x ^= hs[r][NK - 1] & w[NK - 1];
            odd |= (uint32_t)__popcll(x);
        }
        const bool ok = __ballot(odd & 1u) == 0ull;
        if (ok || t >= tb.max_iter) {
            if (p == 0) {
                // type 0 holds y_u at k = u + d_o: rotate the word down by d_o
                uint64_t o[NK];
                if (NK == 1) {
                    o[0] = d_o ? (w[0] >> d_o) | (w[0] << (N - d_o)) : w[0];
                    if (N < 64)
                        o[0] &= (1ull << N) - 1ull;
                } else {
                    const unsigned __int128 v = ((unsigned __int128)w[NK - 1] << 64) | w[0];
                    unsigned __int128 r = d_o ? (v >> d_o) | (v << (N - d_o)) : v;
                    if (N < 128)
                        r &= ((unsigned __int128)1 << N) - 1;
                    o[0] = (uint64_t)r;
                    o[NK - 1] = (uint64_t)(r >> 64);
                }
                if (lane == 0) {
#pragma unroll
                    for (int j = 0; j < NK; j++)
                        A.bits[f * A.bits_ld + j] = o[j];
                    A.iters[f] = (uint8_t)t;
                    A.flags[f] = ok ? 1 : 0;
                }
            }
            return;
        }
    }
}

// LEN: words of the codes' vectors (1: N <= 64, 2: N > 64, 0: a mix of both)
template <int LEN, bool FIX8>
__global__ void __launch_bounds__(TYPES *WAVE) rowpar_decode(RowParArgs A)
{
    extern __shared__ __align__(16) char lds[];
    const int p = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
    const int lane = threadIdx.x % WAVE;
    const int64_t f = blockIdx.x;
    const int c = A.code_idx ? __builtin_amdgcn_readfirstlane((int)A.code_idx[f]) : 0;
    if (c >= A.n_codes)
        return;
    const RowParTab &tb = A.tab[c];
    if (LEN == 2 || (LEN == 0 && tb.N > WAVE))
        decode_frame<2, FIX8>(A, tb, f, lds, p, lane);
    else
        decode_frame<1, FIX8>(A, tb, f, lds, p, lane);
}

template <bool FIX8>
void launch(const RowParArgs &a, int len, size_t lds, hipStream_t stream)
{
    const dim3 grid((unsigned)a.F), block(TYPES * WAVE);
    if (len == 1)
        hipLaunchKernelGGL((rowpar_decode<1, FIX8>), grid, block, lds, stream, a);
    else if (len == 2)
        hipLaunchKernelGGL((rowpar_decode<2, FIX8>), grid, block, lds, stream, a);
    else
        hipLaunchKernelGGL((rowpar_decode<0, FIX8>), grid, block, lds, stream, a);
}

}  // namespace

hipError_t launch_rowpar(const RowParArgs &a, int fix8, hipStream_t stream)
{
    if (a.F < 1 || a.n_codes < 1 || a.n_codes > kRpMaxCodes || a.F > (int64_t)0x7fffffff)
        return hipErrorInvalidValue;
    size_t lds = 0;
    bool one = false, two = false;
    for (int c = 0; c < a.n_codes; c++) {
        const size_t n = rowpar_lds_bytes(a.tab[c].N, a.tab[c].M, a.tab[c].dp);
        lds = n > lds ? n : lds;
        (a.tab[c].N > WAVE ? two : one) = true;
    }
    if (lds > kRpMaxLds)
        return hipErrorInvalidValue;
    const int len = one && two ? 0 : (two ? 2 : 1);
    if (fix8)
        launch<true>(a, len, lds, stream);
    else
        launch<false>(a, len, lds, stream);
    return hipGetLastError();
}

}  // namespace bch
