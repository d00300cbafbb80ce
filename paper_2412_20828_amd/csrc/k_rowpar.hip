// Row-parallel enhanced-NMS decoder for small and middle batches: restart
// message mode, nine branches, one workgroup of three waves per frame (twelve
// in the smallest calls, decode_wide; Algorithm 1 of Section III-B, eqs. 2-5).
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
// bit for bit.  A frame with a NaN posterior searches its rows in their order too
// (rowsearch.h).
//
// What bounds it: VALU issue.  An iteration of BCH(127,64) takes 2,900 VALU
// instructions of a frame's three waves (6 per edge in step 3, 3.7 in step 2:
// unpacking an address, the search), issued at 1.0 per CU-cycle with the LDS
// 51-59% busy: 1.15-1.35 us per frame-iteration and CU, twice the lane-per-frame
// kernels' figure at full load, but from the first frame on.  One frame at
// 3 dB: 39 us against 451 (decode_wide 25); 4,096 frames: 173 against 470; the mixed call of
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

#include <algorithm>

#include "rowpar.h"
#include "rowsearch.h"

namespace bch {
namespace {

constexpr int WAVE = 64;
constexpr int TYPES = 3;
constexpr int B = 9;

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

// a lane's coordinates k = lane, lane + 64 in type p: y, the coordinate u of the
// code, and where the three types' sums of it are
template <int NK, bool FIX8>
__device__ __forceinline__ void coordinates(const RowParArgs &A, int N, int p, int64_t f, int d_o, int lane, float *y,
                                            int *u, int (*src)[TYPES], bool *in)
{
    constexpr int US = NK * WAVE;  // sums of one type
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
}

// parity rows of the syndrome, one or two per lane
template <int NK>
__device__ __forceinline__ void parity_rows(const RowParTab &tb, int lane, uint64_t (*hs)[NK])
{
#pragma unroll
    for (int r = 0; r < 2; r++)
#pragma unroll
        for (int w = 0; w < NK; w++) {
            const int row = lane + r * WAVE;
            hs[r][w] = row < tb.msyn ? tb.hsyn[row * NK + w] : 0ull;
        }
}

// the input of the type: magnitudes to the extended cells, signs to W
template <int NK, bool FIX8>
__device__ __forceinline__ void type_input(float *E, int N, int dp, int lane, const float *y, const bool *in, uint64_t *W,
                                           float *a)
{
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
}

// six more entries of a row's search
__device__ __forceinline__ void search_step(const char *Eb, const StepWord &st, uint32_t &u1, uint32_t &u2)
{
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

// the two least of a row of n <= MAX steps
template <int MAX>
__device__ __forceinline__ uint2 search_row(const char *Eb, const StepWord *st, int n)
{
    uint32_t u1 = 0x7f800000u, u2 = 0x7f800000u;
#pragma unroll
    for (int e = 0; e < MAX; e++)
        if (e < n)
            search_step(Eb, st[e], u1, u2);
    return make_uint2(u1, u2);
}

template <int NK, bool FIX8>
__device__ __forceinline__ uint2 row_record(const uint64_t *W, const uint4 &mk, uint2 u);

// a posterior of the frame is NaN (past its end they are 1): its rows take
// ordered_row.  Every wave holds the whole frame and finds the same
template <int NK, bool FIX8>
__device__ __forceinline__ bool has_nan(const float *y)
{
    return !FIX8 && __builtin_amdgcn_ballot_w64(__builtin_isunordered(y[0], y[NK - 1])) != 0ull;
}

// the two least of a row by its columns mk of the type's input, k at E[k + 2 d_p]
template <int NK, bool FIX8>
__device__ __forceinline__ uint2 ordered_row(const uint64_t *W, const float *E, int dp, uint4 mk)
{
    // opaque: what depends on the mask alone would be formed ahead of the iterations, and spill
    __asm__ volatile("" : "+v"(mk.x), "+v"(mk.y), "+v"(mk.z), "+v"(mk.w));
    uint64_t lo = (uint64_t)mk.y << 32 | mk.x, hi = (uint64_t)mk.w << 32 | mk.z;
    const uint2 u = ordered_search(__popcll(lo) + (NK == 2 ? __popcll(hi) : 0), [&]() {
        const bool first = NK == 1 || lo != 0ull;
        const uint64_t m = first ? lo : hi;
        lo &= first ? lo - 1ull : ~0ull;
        hi &= first ? ~0ull : hi - 1ull;
        return __float_as_uint(E[__builtin_ctzll(m) + (first ? 0 : WAVE) + 2 * dp]);
    });
    uint2 r = row_record<NK, FIX8>(W, mk, u);
    // a row of NaNs: its sign multiplies them there, which leaves theirs
    r.x &= u.x > 0x7f800000u ? 0x7fffffffu : ~0u;
    return r;
}

template <int NK, bool FIX8>
__device__ __forceinline__ uint2 row_record(const uint64_t *W, const uint4 &mk, uint2 u)
{
    const uint32_t u1 = u.x, u2 = u.y;
    uint32_t par = ((uint32_t)W[0] & mk.x) ^ ((uint32_t)(W[0] >> 32) & mk.y);
    if (NK == 2)
        par ^= ((uint32_t)W[NK - 1] & mk.z) ^ ((uint32_t)(W[NK - 1] >> 32) & mk.w);
    const uint32_t sg = (uint32_t)__builtin_popcount(par) << 31;
    if (!FIX8)
        return make_uint2(u1 | sg, u2);
    // min1 and the signed c2v (3 m + 2) >> 2 of min1, min2
    const float q1 = floorf(__builtin_fmaf(__uint_as_float(u1), 0.75f, 0.5f));
    const float q2 = floorf(__builtin_fmaf(__uint_as_float(u2), 0.75f, 0.5f));
    const int c1 = sg ? -(int)q1 : (int)q1, c2 = sg ? -(int)q2 : (int)q2;
    return make_uint2(u1, ((uint32_t)c1 & 0xffffu) | ((uint32_t)c2 << 16));
}

// the c2v of record r at a coordinate of magnitude a
template <bool FIX8>
__device__ __forceinline__ void add_record(const uint2 &r, float a, float &T, int &Ti)
{
    if (FIX8) {
        const int pk = (int)r.y;
        Ti += r.x == __float_as_uint(a) ? pk >> 16 : (int)(int16_t)pk;
    } else {
        const float s1 = __uint_as_float(r.x), m1 = fabsf(s1), m2 = __uint_as_float(r.y);
        T += __builtin_copysignf(__builtin_amdgcn_fmed3f(m1, m2, (m1 + m2) - a), s1);
    }
}

// the types' sums in type order, the posterior, and its signs
template <int NK, bool FIX8>
__device__ __forceinline__ void posterior(const RowParArgs &A, const RowParTab &tb, int64_t f, int t, bool trace,
                                          float scale, const float *U, const int *u, const int (*src)[TYPES],
                                          const bool *in, float *y, uint64_t *w)
{
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
        if (A.trace && trace && in[j]) {
            const int64_t at = (f * tb.max_iter + (t - 1)) * A.ld + u[j];
            if (FIX8)
                static_cast<int32_t *>(A.trace)[at] = (int32_t)yn;
            else
                static_cast<float *>(A.trace)[at] = yn;
        }
    }
}

template <int NK>
__device__ __forceinline__ bool syndrome_zero(const uint64_t (*hs)[NK], const uint64_t *w)
{
    uint32_t odd = 0;
#pragma unroll
    for (int r = 0; r < 2; r++) {
        uint64_t x = hs[r][0] & w[0];
        if (NK == 2)
            x ^= hs[r][NK - 1] & w[NK - 1];
        odd |= (uint32_t)__popcll(x);
    }
    return __ballot(odd & 1u) == 0ull;
}

// outputs of a frame from type 0, which holds y_u at k = u + d_o: its word
// rotated down by d_o
template <int NK>
__device__ __forceinline__ void write_frame(const RowParArgs &A, int N, int64_t f, int d_o, int t, bool ok, int lane,
                                            const uint64_t *w)
{
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
    float y[NK];
    int u[NK], src[NK][TYPES];
    bool in[NK];
    coordinates<NK, FIX8>(A, N, p, f, d_o, lane, y, u, src, in);
    uint64_t hs[2][NK];
    parity_rows<NK>(tb, lane, hs);
    if (lane == 0) {
        E[ext] = __builtin_inff();
        *reinterpret_cast<uint2 *>(Rb + 8 * (3 * M)) = make_uint2(0u,0u);
    }
    const float scale = tb.alpha / (float)B;
    for (int t = 1;; t++) {
        // ---- 1. input of the type
        uint64_t W[NK];
        float a[NK];
        type_input<NK, FIX8>(E, N, dp, lane, y, in, W, a);
        wave_order();
        // ---- 2. rows
        if (__builtin_expect(has_nan<NK, FIX8>(y), 0)) {
            for (int q = 0; q < tb.n_rounds; q++) {
                const uint4 mk = tb.mask[q * WAVE + lane];
                *reinterpret_cast<uint2 *>(Rb + tb.slot[q * WAVE + lane]) = ordered_row<NK, FIX8>(W, E, dp, mk);
            }
        } else {
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
                    search_step(Eb, st, u1, u2);
                }
                *reinterpret_cast<uint2 *>(Rb + slot) = row_record<NK, FIX8>(W, mk, make_uint2(u1, u2));
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
                    for (int j = 0; j < NK; j++)
                        add_record<FIX8>(rc[j][e], a[j], T[j], Ti[j]);
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
        posterior<NK, FIX8>(A, tb, f, t, p == 0, scale, U, u, src, in, y, w);
        const bool ok = syndrome_zero<NK>(hs, w);
        if (ok || t >= tb.max_iter) {
            if (p == 0)
                write_frame<NK>(A, N, f, d_o, t, ok, lane, w);
            return;
        }
    }
}

// The smallest calls, a workgroup a CU: kRpWide waves a type.  Steps of
// decode_frame, with what the time of one frame hangs on taken apart: the
// rounds of step 2 go to the type's waves, the coordinates of step 3 to its
// first NK, at the price of a second barrier; the tables are read once a frame
// into registers (RowParTab::wide: they fit); and the records of step 3 are
// read eight ahead of their use.  Sums keep their order (a record past a
// list's end adds +0, and no partial sum is -0).  Type p is every third wave,
// so that the waves of step 3 are on different SIMDs.  One frame of (127,64), 3
// dB, eight iterations: 23.1 us against 37.5.  Measured and not taken: steps 1
// and 4 in the type's first wave alone, with a third barrier (32.7), and steps
// of the search read ahead (29.6): both spill.
template <int NK, bool FIX8>
__device__ __forceinline__ void decode_wide(const RowParArgs &A, const RowParTab &tb, int64_t f, char *lds, int p, int g,
                                            int lane)
{
    constexpr int G = kRpWide;
    constexpr int S2 = NK == 1 ? kRpWideSteps2 : 0;  // steps of a second round
    const int N = tb.N, M = tb.M, dp = tb.dp;
    const int ext = N + 2 * dp;
    const int ext_pad = (ext + 4) & ~3;
    const int nrec = 3 * M + 2;
    constexpr int US = NK * WAVE;
    char *Eb = lds + 4 * (p * G + g) * ext_pad;  // the wave's own copy
    char *Rb = lds + 4 * TYPES * G * ext_pad + 8 * p * nrec;
    float *Ubase = reinterpret_cast<float *>(lds + 4 * TYPES * G * ext_pad + 8 * TYPES * nrec);
    float *E = reinterpret_cast<float *>(Eb);
    // ---- tables
    const int ka = g < NK ? lane + g * WAVE : lane;  // coordinate of step 3
    uint2 id[kRpWideRecs / kRpRecs];
    const int n8 = g < NK ? (tb.n_recs + 7) / 8 : 0;
#pragma unroll
    for (int c = 0; c < kRpWideRecs / kRpRecs; c++)
        id[c] = c / 2 < n8 ? tb.recs[c * US + ka] : make_uint2(0u, 0u);
    // the wave's rounds g and g + G: steps, sign masks, places of the records
    StepWord sa[kRpWideSteps], sb[S2 + 1];
    uint4 mka = make_uint4(0u, 0u, 0u, 0u), mkb = mka;
    uint32_t slota = 0u, slotb = 0u;
    int na = 0, nb = 0;
    {
        int ata = 0, atb = 0, n = 0;
        for (int q = 0; q < tb.n_rounds; q++) {
            const int r = __builtin_amdgcn_readfirstlane(tb.rounds[q]);
            if (q == g) {
                ata = n;
                na = r;
            }
            if (S2 && q == g + G) {
                atb = n;
                nb = r;
            }
            n += r;
        }
        const StepWord *sp = reinterpret_cast<const StepWord *>(tb.steps) + lane;
#pragma unroll
        for (int e = 0; e < kRpWideSteps; e++)
            sa[e] = e < na ? sp[(ata + e) * WAVE] : StepWord{0u, 0u, 0u};
#pragma unroll
        for (int e = 0; e < S2; e++)
            sb[e] = e < nb ? sp[(atb + e) * WAVE] : StepWord{0u, 0u, 0u};
        if (na) {
            mka = tb.mask[g * WAVE + lane];
            slota = tb.slot[g * WAVE + lane];
        }
        if (S2 && nb) {
            mkb = tb.mask[(g + G) * WAVE + lane];
            slotb = tb.slot[(g + G) * WAVE + lane];
        }
    }
    const int d_o = (int)A.d_o[f] % dp;
    float y[NK];
    int u[NK], src[NK][TYPES];
    bool in[NK];
    coordinates<NK, FIX8>(A, N, p, f, d_o, lane, y, u, src, in);
    uint64_t hs[2][NK];
    parity_rows<NK>(tb, lane, hs);
    if (lane == 0) {
        E[ext] = __builtin_inff();
        *reinterpret_cast<uint2 *>(Rb + 8 * (3 * M)) = make_uint2(0u, 0u);
    }
    const float scale = tb.alpha / (float)B;
    for (int t = 1;; t++) {
        // table words opaque: unpacked outside the loop they would fill the registers
#pragma unroll
        for (int c = 0; c < kRpWideRecs / kRpRecs; c++)
            __asm__ volatile("" : "+v"(id[c].x), "+v"(id[c].y));
#pragma unroll
        for (int e = 0; e < kRpWideSteps; e++)
            __asm__ volatile("" : "+v"(sa[e].x), "+v"(sa[e].y), "+v"(sa[e].z));
#pragma unroll
        for (int e = 0; e < S2; e++)
            __asm__ volatile("" : "+v"(sb[e].x), "+v"(sb[e].y), "+v"(sb[e].z));
        // ---- 1. input of the type, in each of its waves
        uint64_t W[NK];
        float a[NK];
        type_input<NK, FIX8>(E, N, dp, lane, y, in, W, a);
        wave_order();
        // ---- 2. rows
        if (__builtin_expect(has_nan<NK, FIX8>(y), 0)) {
            if (na)
                *reinterpret_cast<uint2 *>(Rb + slota) = ordered_row<NK, FIX8>(W, E, dp, mka);
            if (S2 && nb)
                *reinterpret_cast<uint2 *>(Rb + slotb) = ordered_row<NK, FIX8>(W, E, dp, mkb);
        } else {
            if (na)
                *reinterpret_cast<uint2 *>(Rb + slota) =
                    row_record<NK, FIX8>(W, mka, search_row<kRpWideSteps>(Eb, sa, na));
            if (S2 && nb)
                *reinterpret_cast<uint2 *>(Rb + slotb) = row_record<NK, FIX8>(W, mkb, search_row<S2>(Eb, sb, nb));
        }
        __syncthreads();
        // ---- 3. c2v sums of the coordinates
        float *U = Ubase + (t & 1) * TYPES * US;
        if (g < NK) {
            const float am = g == 0 ? a[0] : a[NK - 1];
            float T = 0.0f;
            int Ti = 0;
            uint2 rc[2][8];
            auto fetch = [&](uint2 *r, const uint2 *i) {
#pragma unroll
                for (int h = 0; h < 2; h++) {
                    r[4 * h] = *reinterpret_cast<const uint2 *>(Rb + (i[h].x & 0xffffu));
                    r[4 * h + 1] = *reinterpret_cast<const uint2 *>(Rb + (i[h].x >> 16));
                    r[4 * h + 2] = *reinterpret_cast<const uint2 *>(Rb + (i[h].y & 0xffffu));
                    r[4 * h + 3] = *reinterpret_cast<const uint2 *>(Rb + (i[h].y >> 16));
                }
            };
            fetch(rc[0], id);
#pragma unroll
            for (int c = 0; c < kRpWideRecs / 8; c++)
                if (c < n8) {
                    if (c + 1 < kRpWideRecs / 8 && c + 1 < n8)
                        fetch(rc[(c + 1) % 2], id + 2 * (c + 1));
#pragma unroll
                    for (int e = 0; e < 8; e++)
                        add_record<FIX8>(rc[c % 2][e], am, T, Ti);
                }
            U[p * US + ka] = FIX8 ? (float)Ti : T;
        }
        __syncthreads();
        // ---- 4. merge, posterior, decision, syndrome, in each wave
        uint64_t w[NK];
        posterior<NK, FIX8>(A, tb, f, t, p == 0 && g == 0, scale, U, u, src, in, y, w);
        const bool ok = syndrome_zero<NK>(hs, w);
        if (ok || t >= tb.max_iter) {
            if (p == 0 && g == 0)
                write_frame<NK>(A, N, f, d_o, t, ok, lane, w);
            return;
        }
    }
}

// LEN: words of the codes' vectors (1: N <= 64, 2: N > 64, 0: a mix of both);
// G: waves a type
template <int LEN, bool FIX8, int G>
__global__ void __launch_bounds__(TYPES *G *WAVE) rowpar_decode(RowParArgs A)
{
    extern __shared__ __align__(16) char lds[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
    const int lane = threadIdx.x % WAVE;
    const int64_t f = blockIdx.x;
    const int c = A.code_idx ? __builtin_amdgcn_readfirstlane((int)A.code_idx[f]) : 0;
    if (c >= A.n_codes)
        return;
    const RowParTab &tb = A.tab[c];
    const bool two = LEN == 2 || (LEN == 0 && tb.N > WAVE);
    if constexpr (G == 1) {
        if (two)
            decode_frame<2, FIX8>(A, tb, f, lds, wave, lane);
        else
            decode_frame<1, FIX8>(A, tb, f, lds, wave, lane);
    } else {
        if (two)
            decode_wide<2, FIX8>(A, tb, f, lds, wave % TYPES, wave / TYPES, lane);
        else
            decode_wide<1, FIX8>(A, tb, f, lds, wave % TYPES, wave / TYPES, lane);
    }
}

template <bool FIX8, int G>
void launch(const RowParArgs &a, int len, size_t lds, hipStream_t stream)
{
    const dim3 grid((unsigned)a.F), block(TYPES * G * WAVE);
    if (len == 1)
        hipLaunchKernelGGL((rowpar_decode<1, FIX8, G>), grid, block, lds, stream, a);
    else if (len == 2)
        hipLaunchKernelGGL((rowpar_decode<2, FIX8, G>), grid, block, lds, stream, a);
    else
        hipLaunchKernelGGL((rowpar_decode<0, FIX8, G>), grid, block, lds, stream, a);
}

}  // namespace

bool rowpar_is_wide(const RowParArgs &a)
{
    bool wide = a.wide != 0;
    for (int c = 0; c < a.n_codes; c++) {
        const RowParTab &t = a.tab[c];
        wide = wide && t.wide && rowpar_lds_bytes(t.N, t.M, t.dp, kRpWide) <= kRpMaxLds;
    }
    return wide;
}

hipError_t launch_rowpar(const RowParArgs &a, int fix8, hipStream_t stream)
{
    if (a.F < 1 || a.n_codes < 1 || a.n_codes > kRpMaxCodes || a.F > (int64_t)0x7fffffff)
        return hipErrorInvalidValue;
    const bool wide = rowpar_is_wide(a);
    size_t lds = 0;
    bool one = false, two = false;
    for (int c = 0; c < a.n_codes; c++) {
        const RowParTab &t = a.tab[c];
        lds = std::max(lds, rowpar_lds_bytes(t.N, t.M, t.dp, wide ? kRpWide : 1));
        (t.N > WAVE ? two : one) = true;
    }
    if (lds > kRpMaxLds)
        return hipErrorInvalidValue;
    const int len = one && two ? 0 : (two ? 2 : 1);
    if (wide && fix8)
        launch<true, kRpWide>(a, len, lds, stream);
    else if (wide)
        launch<false, kRpWide>(a, len, lds, stream);
    else if (fix8)
        launch<true, 1>(a, len, lds, stream);
    else
        launch<false, 1>(a, len, lds, stream);
    return hipGetLastError();
}

}  // namespace bch
