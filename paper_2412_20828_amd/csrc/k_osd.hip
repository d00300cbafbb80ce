// Order-p ordered statistics decoding on the device (Section II-B), the second
// stage of the hybrid decoder run next to the NMS kernels: one wave per frame,
// frames whose skip byte is set are left alone.
//
// Per frame, exactly the host algorithm:
//   1. reliabilities r_u = |L_u| and hard decisions z;
//   2. positions ordered by reliability, descending, ties by index (each
//      lane counts how many positions precede its own);
//   3. most reliable basis by greedy Gaussian elimination on the generator
//      rows in that column order (row k of the working matrix sits in lane
//      k mod 64, slot k / 64; a row swap moves data between lanes);
//   4. base candidate c0 = sum of the rows whose basis decision is 1;
//   5. candidates c0 + (up to p rows), in the order weight 0, weight 1
//      (ascending), weight 2 (lexicographic); cost = sum of r over the
//      positions where the candidate disagrees with z, in FP64, ascending
//      position; the first candidate of least cost wins.
// The candidates are spread over the lanes and scored in two passes.  The
// first uses r quantised to 16 bits (q_u = round(r_u 2^s), s per frame), an
// integer weighted popcount over bit-planes of q that the wave builds with
// ballots; each candidate's quantised cost is within 63.5 units of 2^s times
// its exact cost, and it is kept in LDS (written and read by the same lane):
// as a word for up to KEEP_MAX candidates, else as a half-word saturated at
// 65535, which the second pass recomputes only when the threshold below
// reaches 65535.  The second pass computes the exact FP64 cost of every
// candidate whose quantised cost is within 128 units of the smallest,
// which includes every candidate of least exact cost, and the wave picks the
// least exact cost, then the first candidate.  The result is therefore the
// host's.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "kernels.h"

namespace bch {
namespace {

constexpr int WAVE = 64;

__device__ __forceinline__ uint32_t rd(uint32_t v, int l) { return __builtin_amdgcn_readlane(v, l); }
// old with lane l's value replaced by v
__device__ __forceinline__ uint32_t wr(uint32_t v, int l, uint32_t old)
{
    return (int)threadIdx.x == l ? v : old;
}

// candidate key -> rows: key 0 = c0, 1..K = one row, then the pairs in
// lexicographic order.  Only for keys below 1 + K + K (K - 1) / 2.
__device__ __forceinline__ void key_rows(int key, int K, int &k1, int &k2)
{
    k1 = -1;
    k2 = -1;
    if (key == 0)
        return;
    if (key <= K) {
        k1 = key - 1;
        return;
    }
    int p = key - 1 - K;
    int a = 0;
    while (p >= K - 1 - a) {  // ends at a <= K - 2 for a valid key
        p -= K - 1 - a;
        a++;
    }
    k1 = a;
    k2 = a + 1 + p;
}

// rows of key, given those of key - WAVE (valid keys only)
__device__ __forceinline__ void next_rows(int key, int K, int &k1, int &k2)
{
    if (key <= K) {
        k1 = key - 1;
        k2 = -1;
        return;
    }
    if (k2 < 0) {
        key_rows(key, K, k1, k2);
        return;
    }
    k2 += WAVE;
    while (k2 >= K) {  // carry into the next row(s); stays below K - 1 for a valid key
        const int over = k2 - K;
        k1++;
        k2 = k1 + 1 + over;
    }
}

// pass-1 costs kept in LDS as words up to this many candidates (9 KB; every
// order-2 search with K <= 67); larger searches keep saturated half-words
// (at most 16.5 KB for K = 128): a word each, 20 KB for K = 99, cut the
// resident waves per CU and measured slower than recomputing.
constexpr int KEEP_MAX = 2304;

// candidates of an order-p search over K basis rows (p = 0, 1 or 2)
__host__ __device__ inline int n_candidates(int order, int K)
{
    return order <= 0 ? 1 : (order == 1 ? 1 + K : 1 + K + K * (K - 1) / 2);
}

__global__ void __launch_bounds__(WAVE) osd_kernel(OsdArgs A)
{
    extern __shared__ uint32_t qv[];  // [n_candidates] quantised costs of pass 1
    __shared__ float r[128];
    __shared__ uint32_t rowl[128][4];  // working generator rows after elimination
    __shared__ int mrb[128];
    const int lane = threadIdx.x;
    const int N = A.N, K = A.K;
    for (int64_t f = blockIdx.x; f < A.F; f += gridDim.x) {
        if ((A.skip && A.skip[f]) || (A.code_idx && A.code_idx[f] != A.which))
            continue;
        const float *L = A.llr + f * A.ld;
        const bool in0 = lane < N, in1 = lane + WAVE < N;
        const float l0 = in0 ? L[lane] : 0.0f, l1 = in1 ? L[lane + WAVE] : 0.0f;
        const float r0 = fabsf(l0), r1 = fabsf(l1);
        const uint64_t z0 = __ballot(in0 && l0 < 0.0f), z1 = __ballot(in1 && l1 < 0.0f);
        r[lane] = r0;
        r[lane + WAVE] = r1;
        __syncthreads();
        // ---- rank of each position: higher reliability first, ties by index
        int rk0 = 0, rk1 = 0;
        for (int j = 0; j < N; j++) {
            const float rj = r[j];
            rk0 += (rj > r0 || (rj == r0 && j < lane)) ? 1 : 0;
            rk1 += (rj > r1 || (rj == r1 && j < lane + WAVE)) ? 1 : 0;
        }
        // ---- greedy elimination; row k in lane k & 63, slot k >> 6
        uint32_t a[4], b[4];
#pragma unroll
        for (int w = 0; w < 4; w++) {
            a[w] = lane < K ? A.G[lane * 4 + w] : 0u;
            b[w] = lane + WAVE < K ? A.G[(lane + WAVE) * 4 + w] : 0u;
        }
        int piv = 0;
        for (int pos = 0; pos < N && piv < K; pos++) {
            // the column of rank pos (one lane holds it)
            const uint64_t m0 = __ballot(in0 && rk0 == pos), m1 = __ballot(in1 && rk1 == pos);
            // (ranks are distinct, so one lane matches; the masks only keep a
            // malformed input inside the arrays)
            const int col = (m0 ? __builtin_ctzll(m0) : WAVE + __builtin_ctzll(m1 | (1ull << 63))) & 127;
            const int cw = (col >> 5) & 3;
            const uint32_t cb = 1u << (col & 31);
            const uint64_t h0 = __ballot(lane < K && lane >= piv && (a[cw] & cb));
            const uint64_t h1 = __ballot(lane + WAVE < K && lane + WAVE >= piv && (b[cw] & cb));
            if (!h0 && !h1)
                continue;
            const int k0 = h0 ? __builtin_ctzll(h0) : WAVE + __builtin_ctzll(h1);
            uint32_t pr[4];
#pragma unroll
            for (int w = 0; w < 4; w++)
                pr[w] = k0 < WAVE ? rd(a[w], k0) : rd(b[w], k0 - WAVE);
            if (k0 != piv) {
                uint32_t qr[4];
#pragma unroll
                for (int w = 0; w < 4; w++)
                    qr[w] = piv < WAVE ? rd(a[w], piv) : rd(b[w], piv - WAVE);
#pragma unroll
                for (int w = 0; w < 4; w++) {
                    if (k0 < WAVE)
                        a[w] = wr(qr[w], k0, a[w]);
                    else
                        b[w] = wr(qr[w], k0 - WAVE, b[w]);
                    if (piv < WAVE)
                        a[w] = wr(pr[w], piv, a[w]);
                    else
                        b[w] = wr(pr[w], piv - WAVE, b[w]);
                }
            }
            if (lane < K && lane != piv && (a[cw] & cb)) {
#pragma unroll
                for (int w = 0; w < 4; w++)
                    a[w] ^= pr[w];
            }
            if (lane + WAVE < K && lane + WAVE != piv && (b[cw] & cb)) {
#pragma unroll
                for (int w = 0; w < 4; w++)
                    b[w] ^= pr[w];
            }
            if (lane == 0)
                mrb[piv] = col;
            piv++;
        }
        // ---- rows to LDS, base candidate c0 and d0 = c0 + z
#pragma unroll
        for (int w = 0; w < 4; w++) {
            if (lane < K)
                rowl[lane][w] = a[w];
            if (lane + WAVE < K)
                rowl[lane + WAVE][w] = b[w];
        }
        __syncthreads();
        uint32_t c[4] = {0u, 0u, 0u, 0u};
        if (lane < K) {
            const int m = mrb[lane];
            if (((m < WAVE ? z0 : z1) >> (m & 63)) & 1ull)
#pragma unroll
                for (int w = 0; w < 4; w++)
                    c[w] ^= a[w];
        }
        if (lane + WAVE < K) {
            const int m = mrb[lane + WAVE];
            if (((m < WAVE ? z0 : z1) >> (m & 63)) & 1ull)
#pragma unroll
                for (int w = 0; w < 4; w++)
                    c[w] ^= b[w];
        }
#pragma unroll
        for (int w = 0; w < 4; w++)
            for (int s = 1; s < WAVE; s <<= 1)
                c[w] ^= __shfl_xor(c[w], s);
        const uint32_t zw[4] = {(uint32_t)z0, (uint32_t)(z0 >> 32), (uint32_t)z1, (uint32_t)(z1 >> 32)};
        uint32_t d0[4];
#pragma unroll
        for (int w = 0; w < 4; w++)
            d0[w] = __builtin_amdgcn_readfirstlane(c[w] ^ zw[w]);
        // ---- quantised reliabilities and their bit-planes
        float mx = fmaxf(r0, r1);
        for (int s = 1; s < WAVE; s <<= 1)
            mx = fmaxf(mx, __shfl_xor(mx, s));
        // no scale holds an infinite reliability: pass 2 then takes every candidate
        const bool finite = mx < __builtin_inff();
        const int sc = finite && mx > 0.0f ? 14 - ilogbf(mx) : 0;  // every q below 2^15
        const uint32_t q0 = finite ? (uint32_t)rintf(ldexpf(r0, sc)) : 0u;
        const uint32_t q1 = finite ? (uint32_t)rintf(ldexpf(r1, sc)) : 0u;
        uint32_t pl[16][4];
#pragma unroll
        for (int bp = 0; bp < 16; bp++) {
            const uint64_t p0 = __ballot(in0 && ((q0 >> bp) & 1u)), p1 = __ballot(in1 && ((q1 >> bp) & 1u));
            pl[bp][0] = (uint32_t)p0;
            pl[bp][1] = (uint32_t)(p0 >> 32);
            pl[bp][2] = (uint32_t)p1;
            pl[bp][3] = (uint32_t)(p1 >> 32);
        }
        auto qcost = [&](const uint32_t *x) {
            uint32_t t = 0u;
#pragma unroll
            for (int bp = 0; bp < 16; bp++) {
                const uint32_t n = __builtin_popcount(x[0] & pl[bp][0]) + __builtin_popcount(x[1] & pl[bp][1]) +
                                   __builtin_popcount(x[2] & pl[bp][2]) + __builtin_popcount(x[3] & pl[bp][3]);
                t += n << bp;
            }
            return t;
        };
        const int nk = n_candidates(A.order, K);
        // pass 1: least quantised cost
        uint32_t qmin = 0xffffffffu;
        {
            int k1 = -1, k2 = -1;
            if (lane < nk)
                key_rows(lane, K, k1, k2);
            for (int key = lane; key < nk; key += WAVE) {
                uint32_t x[4];
#pragma unroll
                for (int w = 0; w < 4; w++)
                    x[w] = d0[w] ^ (k1 >= 0 ? rowl[k1][w] : 0u) ^ (k2 >= 0 ? rowl[k2][w] : 0u);
                const uint32_t qc = qcost(x);
                if (A.keep_costs == 1)
                    qv[key] = qc;
                else
                    reinterpret_cast<uint16_t *>(qv)[key] = (uint16_t)(qc < 65535u ? qc : 65535u);
                qmin = qc < qmin ? qc : qmin;
                if (key + WAVE < nk)
                    next_rows(key + WAVE, K, k1, k2);
            }
        }
        for (int s = 1; s < WAVE; s <<= 1) {
            const uint32_t o = __shfl_xor(qmin, s);
            qmin = o < qmin ? o : qmin;
        }
        const uint32_t thr = finite ? qmin + 128u : 0xffffffffu;
        // pass 2: exact FP64 cost of the candidates near the least
        double best = 0.0;
        int bkey = 0x7fffffff;
        {
            int k1 = -1, k2 = -1;
            if (lane < nk)
                key_rows(lane, K, k1, k2);
            for (int key = lane; key < nk; key += WAVE) {
                // the stored cost, or 65535 for "at least 65535"
                const uint32_t st = A.keep_costs == 1 ? qv[key] : reinterpret_cast<const uint16_t *>(qv)[key];
                const bool sat = A.keep_costs != 1 && st == 65535u;
                bool near = sat ? thr >= 65535u : st <= thr;
                uint32_t x[4];
                if (near) {
#pragma unroll
                    for (int w = 0; w < 4; w++)
                        x[w] = d0[w] ^ (k1 >= 0 ? rowl[k1][w] : 0u) ^ (k2 >= 0 ? rowl[k2][w] : 0u);
                    if (sat)
                        near = qcost(x) <= thr;
                }
                if (near) {
                    double d = 0.0;
#pragma unroll
                    for (int w = 0; w < 4; w++) {
                        uint32_t v = x[w];
                        while (v) {
                            d += (double)r[w * 32 + __builtin_ctz(v)];
                            v &= v - 1u;
                        }
                    }
                    if (bkey == 0x7fffffff || d < best) {
                        best = d;
                        bkey = key;
                    }
                }
                if (key + WAVE < nk)
                    next_rows(key + WAVE, K, k1, k2);
            }
        }
        for (int s = 1; s < WAVE; s <<= 1) {
            const double ob = __shfl_xor(best, s);
            const int ok = __shfl_xor(bkey, s);
            if (ok != 0x7fffffff && (bkey == 0x7fffffff || ob < best || (ob == best && ok < bkey))) {
                best = ob;
                bkey = ok;
            }
        }
        if (lane == 0) {
            int k1 = -1, k2 = -1;
            key_rows(bkey, K, k1, k2);
            uint32_t out[4];
#pragma unroll
            for (int w = 0; w < 4; w++)
                out[w] = d0[w] ^ zw[w] ^ (k1 >= 0 ? rowl[k1][w] : 0u) ^ (k2 >= 0 ? rowl[k2][w] : 0u);
            uint64_t *dst = A.bits + f * A.bits_ld;
            dst[0] = (uint64_t)out[0] | ((uint64_t)out[1] << 32);
            if (N > 64)
                dst[1] = (uint64_t)out[2] | ((uint64_t)out[3] << 32);
        }
        __syncthreads();
    }
}

// ---- codes with N - K <= 64 --------------------------------------------------
//
// osd_kernel above is bound by its VALU work: for (127,99) 99 elimination steps
// and 4,951 candidates of 130 instructions each, 32 us a frame and CU.  It
// stays for codes with N - K > 64, whose columns do not fit a 64-bit word.
//
// The same decisions from the parity side.  The positions outside the most
// reliable basis are the greedy basis of the parity-check columns taken in
// ascending order of reliability (the bases of a matroid and of its dual are
// complements), so N - K pivots are eliminated instead of K, on columns: a lane
// holds the column of two positions as N - K bits, a pivot column is read into
// scalar registers, and every column with the pivot's bit set takes the others.
// Afterwards the column of basis position j says which of the N - K dependent
// positions flip with it, and the columns where z = 1 add to the base
// candidate's disagreement d0 on the dependent positions.
//
// A candidate flips basis positions i and j and dependent positions
// d0 + x_i + x_j.  With S = 1 - 2 x in {1, -1} and w_b = (1 - 2 d0_b) q_b, twice its
// quantised cost is 2 q_i + 2 q_j - sum_b w_b S_ib S_jb up to a constant: one
// K x K product over N - K, on the matrix cores in int8 with w_b split into
// 254 h + l (two products, exact in 32 bits).  q = rint(16000 r / 2^e) with 2^e
// the power of two at or below the largest r: each term is within 0.502 of
// its scaled value, a candidate has at most N - K + 2 terms, so every candidate
// of least exact cost lies within 2.008 (N - K + 2) of the least doubled
// quantised cost.  The candidates within 2 (N - K + 2) + 8 are scored in FP64,
// ascending position, as the host scores them; if a reliability is infinite,
// all are.  Each lane keeps its two least costs; if a second one is near as
// well (ties), all costs are formed once more and every near candidate scored.
//
// Bound now by VALU issue, about 4,000 cycles a frame and CU: ranking 650
// instructions, elimination 25 a pivot, the cost update 5 per 64 candidates.
// Measured, order 2 on the failed frames of 20,011 at 3 dB (us, before / now):
// (127,64) 674 / 98, (127,78) 732 / 82, (127,99) 1441 / 79, (63,36) 118 / 25;
// 2,000,000 frames of (127,64) with 0.1% failed: 615 / 83.  Five waves per
// SIMD with a few spilled registers beat three without (79 against 94 for
// (127,99)); a grid of 64 waves per CU beats 16 (91 against 129: a wave's
// share of failed frames varies, and later waves fill in).

using i32x4 = __attribute__((__vector_size__(4 * sizeof(int)))) int;

constexpr int Q_MAX = 32000;
// Doubled "reliability" of the rows past K.  A doubled cost of two real positions
// is below 68 Q_MAX = 2,176,000 in magnitude (64 terms and two of 2 q), so with two
// of these added it is below 2^23, and with an eight-bit index beside it below
// 2^31.  A candidate with a pad costs Q_PAD more than the one without it, which is
// a candidate of lower weight, so that no pad comes within the threshold.
constexpr int Q_PAD = 1 << 21;

struct DualLds {
    float r[128];
    uint64_t x[128];     // [basis index] dependent positions that flip with it
    int q2[128];         // [basis index] 2 q
    int bpos[128];       // [basis index] position
    int ord[128];        // position of each rank
    int ppos[64];        // [row] dependent position
    int w[64];           // [row] -(1 - 2 d0_b) q_b
    uint32_t byte[4][16];  // h, -h, l, -l of w, a byte per row
};

// Lane (g, i) = (lane / 16, lane % 16) of a tile of 16 basis positions: rows
// [NB g, NB g + NB) of position i as bytes, S and the two halves of w S.
template <int KD>
struct Tile {
    static constexpr int NB = KD / 4, ND = NB / 4;
    uint32_t s[ND], h[ND], l[ND];
};

// wp: h, -h, l, -l of the lane's rows; x: the position's column
template <int KD>
__device__ __forceinline__ Tile<KD> make_tile(const uint32_t wp[4][KD / 16], const uint64_t *x, int g)
{
    Tile<KD> t;
    const uint32_t bits = KD == 32 ? (uint32_t) reinterpret_cast<const uint8_t *>(x)[g]
                                   : (uint32_t) reinterpret_cast<const uint16_t *>(x)[g];
#pragma unroll
    for (int d = 0; d < Tile<KD>::ND; d++) {
        // four bits to the low bits of four bytes
        const uint32_t m = (((bits >> (4 * d)) & 15u) * 0x204081u) & 0x01010101u;
        t.s[d] = __builtin_amdgcn_perm(0u, 0x0000ff01u, m);
        const uint32_t sel = (m << 2) | 0x03020100u;
        t.h[d] = __builtin_amdgcn_perm(wp[1][d], wp[0][d], sel);
        t.l[d] = __builtin_amdgcn_perm(wp[3][d], wp[2][d], sel);
    }
    return t;
}

template <int KD>
__device__ __forceinline__ i32x4 mfma(const uint32_t *a, const uint32_t *b, i32x4 c)
{
    if constexpr (KD == 32) {
        const long x = (long)((uint64_t)a[0] | ((uint64_t)a[1] << 32));
        const long y = (long)((uint64_t)b[0] | ((uint64_t)b[1] << 32));
        return __builtin_amdgcn_mfma_i32_16x16x32_i8(x, y, c, 0, 0, 0);
    } else {
        const i32x4 x = {(int)a[0], (int)a[1], (int)a[2], (int)a[3]};
        const i32x4 y = {(int)b[0], (int)b[1], (int)b[2], (int)b[3]};
        return __builtin_amdgcn_mfma_i32_16x16x64_i8(x, y, c, 0, 0, 0);
    }
}

__device__ __forceinline__ int wave_min(int v)
{
#pragma unroll
    for (int s = 1; s < WAVE; s <<= 1) {
        const int o = __shfl_xor(v, s);
        v = o < v ? o : v;
    }
    return v;
}

// positions where candidate key disagrees with z.  Keys order as the
// candidates do: weight << 14 | i << 7 | j.
__device__ __forceinline__ void disagreement(const DualLds &D, uint64_t d0, int key, uint64_t m[2])
{
    const int wt = key >> 14, i = (key >> 7) & 127, j = key & 127;
    m[0] = m[1] = 0ull;
    uint64_t d = d0;
    if (wt >= 1) {
        d ^= D.x[i];
        const int u = D.bpos[i];
        m[u >> 6] |= 1ull << (u & 63);
    }
    if (wt == 2) {
        d ^= D.x[j];
        const int u = D.bpos[j];
        m[u >> 6] |= 1ull << (u & 63);
    }
    while (d) {
        const int u = D.ppos[__builtin_ctzll(d)];
        d &= d - 1ull;
        const uint64_t bit = 1ull << (u & 63);
        m[0] |= u < WAVE ? bit : 0ull;
        m[1] |= u < WAVE ? 0ull : bit;
    }
}

__device__ __forceinline__ double exact_cost(const DualLds &D, uint64_t d0, int key)
{
    uint64_t m[2];
    disagreement(D, d0, key, m);
    double d = 0.0;
#pragma unroll
    for (int w = 0; w < 2; w++)
        while (m[w]) {
            d += (double)D.r[w * WAVE + __builtin_ctzll(m[w])];
            m[w] &= m[w] - 1ull;
        }
    return d;
}

// one frame; NT tiles of 16 basis positions, KD = 32 or 64 >= N - K
template <int NT, int KD>
__device__ __forceinline__ void osd_dual(const OsdArgs &A, const OsdCode &C, int64_t f, DualLds &D)
{
    const int lane = threadIdx.x;
    const int N = C.N, K = C.K, P = N - K;
    const float *L = A.llr + f * A.ld;
    const bool in0 = lane < N, in1 = lane + WAVE < N;
    const float l0 = in0 ? L[lane] : 0.0f, l1 = in1 ? L[lane + WAVE] : 0.0f;
    const float r0 = fabsf(l0), r1 = fabsf(l1);
    uint64_t c0 = in0 ? C.hcol[lane] : 0ull, c1 = in1 ? C.hcol[lane + WAVE] : 0ull;
    const uint64_t z0 = __ballot(in0 && l0 < 0.0f), z1 = __ballot(in1 && l1 < 0.0f);
    D.r[lane] = r0;
    D.r[lane + WAVE] = r1;
    // ---- rank of each position: higher reliability first, ties by index, on
    // the bit patterns (the order of non-negative floats).  Strictly greater
    // ones are counted first; the ranks then sum to N (N - 1) / 2 unless some tie.
    const int b0 = (int)__float_as_uint(r0), b1 = (int)__float_as_uint(r1);
    int rk0 = 0, rk1 = 0;
    const int n0 = N < WAVE ? N : WAVE;
#pragma unroll 8
    for (int j = 0; j < n0; j++) {
        const int rj = __builtin_amdgcn_readlane(b0, j);
        rk0 += rj > b0 ? 1 : 0;
        rk1 += rj > b1 ? 1 : 0;
    }
#pragma unroll 8
    for (int j = 0; j < N - WAVE; j++) {
        const int rj = __builtin_amdgcn_readlane(b1, j);
        rk0 += rj > b0 ? 1 : 0;
        rk1 += rj > b1 ? 1 : 0;
    }
    int sum = (in0 ? rk0 : 0) + (in1 ? rk1 : 0);
#pragma unroll
    for (int s = 1; s < WAVE; s <<= 1)
        sum += __shfl_xor(sum, s);
    if (__builtin_amdgcn_readfirstlane(sum) != N * (N - 1) / 2) {
        for (int j = 0; j < n0; j++) {
            const int rj = __builtin_amdgcn_readlane(b0, j);
            rk0 += rj == b0 && j < lane ? 1 : 0;
            rk1 += rj == b1 ? 1 : 0;
        }
        for (int j = 0; j < N - WAVE; j++)
            rk1 += __builtin_amdgcn_readlane(b1, j) == b1 && j < lane ? 1 : 0;
    }
    if (in0)
        D.ord[rk0] = lane;
    if (in1)
        D.ord[rk1] = lane + WAVE;
    D.w[lane] = 0;
    for (int k = K + lane; k < 16 * NT; k += WAVE) {
        D.x[k] = 0ull;
        D.q2[k] = Q_PAD;
    }
    __syncthreads();
    const int o0 = D.ord[lane & 127], o1 = D.ord[(lane + WAVE) & 127];
    // ---- greedy elimination, least reliable position first
    uint64_t open = P == 64 ? ~0ull : (1ull << P) - 1ull;  // rows without a pivot
    uint64_t pr0 = 0ull, pr1 = 0ull;                       // ranks of the pivots
    auto pivot = [&](int pos) -> bool {
        uint64_t v;
        if (pos < WAVE)
            v = (uint64_t)rd((uint32_t)c0, pos) | (KD == 64 ? (uint64_t)rd((uint32_t)(c0 >> 32), pos) << 32 : 0ull);
        else
            v = (uint64_t)rd((uint32_t)c1, pos - WAVE) |
                (KD == 64 ? (uint64_t)rd((uint32_t)(c1 >> 32), pos - WAVE) << 32 : 0ull);
        const uint64_t m = v & open;
        if (!m)
            return false;
        const int b = __builtin_ctzll(m);
        const uint64_t bit = 1ull << b;
        open ^= bit;
        v ^= bit;
        uint32_t s0, s1;
        if (KD == 32 || b < 32) {
            s0 = (uint32_t)((int)((uint32_t)c0 << (31 - b)) >> 31);
            s1 = (uint32_t)((int)((uint32_t)c1 << (31 - b)) >> 31);
        } else {
            s0 = (uint32_t)((int)((uint32_t)(c0 >> 32) << (63 - b)) >> 31);
            s1 = (uint32_t)((int)((uint32_t)(c1 >> 32) << (63 - b)) >> 31);
        }
        const uint32_t vl = (uint32_t)v, vh = (uint32_t)(v >> 32);
        if (KD == 32) {
            c0 ^= s0 & vl;
            c1 ^= s1 & vl;
        } else {
            c0 ^= (uint64_t)(s0 & vl) | ((uint64_t)(s0 & vh) << 32);
            c1 ^= (uint64_t)(s1 & vl) | ((uint64_t)(s1 & vh) << 32);
        }
        return true;
    };
    for (int t = N - 1; t >= WAVE && open; t--)
        if (pivot(__builtin_amdgcn_readlane(o1, t - WAVE)))
            pr1 |= 1ull << (t - WAVE);
    for (int t = N - 1 < WAVE ? N - 1 : WAVE - 1; t >= 0 && open; t--)
        if (pivot(__builtin_amdgcn_readlane(o0, t)))
            pr0 |= 1ull << t;
    // ---- d0: sum of the columns where z = 1
    uint64_t d0;
    {
        const uint64_t v = ((z0 >> lane) & 1ull ? c0 : 0ull) ^ ((z1 >> lane) & 1ull ? c1 : 0ull);
        uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
#pragma unroll
        for (int s = 1; s < WAVE; s <<= 1) {
            lo ^= __shfl_xor(lo, s);
            if (KD == 64)
                hi ^= __shfl_xor(hi, s);
        }
        d0 = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)lo) |
             (KD == 64 ? (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)hi) << 32 : 0ull);
    }
    // ---- quantised reliabilities; basis and dependent positions to LDS
    float mx = fmaxf(r0, r1);
#pragma unroll
    for (int s = 1; s < WAVE; s <<= 1)
        mx = fmaxf(mx, __shfl_xor(mx, s));
    const bool finite = mx < __builtin_inff();
    const int e = finite && mx > 0.0f ? -ilogbf(mx) : 0;
    auto quant = [&](float r) { return (int)fminf(rintf(ldexpf(r, e) * 16000.0f), (float)Q_MAX); };
    auto place = [&](int u, float r, int rk, uint64_t c) {
        const bool dep = ((rk < WAVE ? pr0 >> rk : pr1 >> (rk - WAVE)) & 1ull) != 0ull;
        const int q = quant(r);
        if (dep) {
            const int b = __builtin_ctzll(c) & 63;  // c is a unit vector
            D.ppos[b] = u;
            D.w[b] = (d0 >> b) & 1ull ? q : -q;
        } else {
            const uint64_t lo = rk < WAVE ? pr0 & ((1ull << rk) - 1ull) : pr0;
            const uint64_t hi = rk < WAVE ? 0ull : pr1 & ((1ull << (rk - WAVE)) - 1ull);
            const int k = (rk - __popcll(lo) - __popcll(hi)) & 127;
            D.x[k] = c;
            D.q2[k] = 2 * q;
            D.bpos[k] = u;
        }
    };
    if (in0)
        place(lane, r0, rk0, c0);
    if (in1)
        place(lane + WAVE, r1, rk1, c1);
    __syncthreads();
    {
        const int w = D.w[lane];
        const int h = (int)rintf((float)w * (1.0f / 254.0f)), l = w - 254 * h;
        uint8_t *by = reinterpret_cast<uint8_t *>(D.byte);
        by[lane] = (uint8_t)h;
        by[64 + lane] = (uint8_t)-h;
        by[128 + lane] = (uint8_t)l;
        by[192 + lane] = (uint8_t)-l;
    }
    __syncthreads();
    // ---- pass 1: doubled quantised costs; each lane keeps its two least, with
    // an index: 4 (tile pair) + k, ONE + tile for one position, BASE for none
    constexpr int NB = KD / 4, ND = NB / 4, ONE = 144, BASE = 152;
    const int g = lane >> 4, li = lane & 15;
    uint32_t wp[4][ND];
#pragma unroll
    for (int k = 0; k < 4; k++)
#pragma unroll
        for (int d = 0; d < ND; d++)
            wp[k][d] = D.byte[k][g * ND + d];
    int m1 = 0x7fffffff, m2 = 0x7fffffff;
    auto put = [&](int cost, int idx) {
        const int v = cost * 256 + idx;
        const int hi = m1 > v ? m1 : v;
        m2 = m2 < hi ? m2 : hi;
        m1 = m1 < v ? m1 : v;
    };
    const i32x4 nil = {0, 0, 0, 0};
    {
        int sum = 0;
#pragma unroll
        for (int d = 0; d < ND; d++) {
            const int h = __builtin_amdgcn_sdot4((int)wp[0][d], 0x01010101, 0, false);
            sum += 254 * h + __builtin_amdgcn_sdot4((int)wp[2][d], 0x01010101, 0, false);
        }
        sum += __shfl_xor(sum, 16);
        sum += __shfl_xor(sum, 32);
        if (lane == 0)
            put(sum, BASE);
    }
    uint32_t S[NT][ND];  // the tiles' S, kept for the rows before them
#pragma unroll
    for (int i = NT - 1; i >= 0; i--) {
        const Tile<KD> a = make_tile<KD>(wp, &D.x[16 * i + li], g);
        int sh = 0, sl = 0;
#pragma unroll
        for (int d = 0; d < ND; d++) {
            S[i][d] = a.s[d];
            sh = __builtin_amdgcn_sdot4((int)a.h[d], 0x01010101, sh, false);
            sl = __builtin_amdgcn_sdot4((int)a.l[d], 0x01010101, sl, false);
        }
        int one = 254 * sh + sl;
        one += __shfl_xor(one, 16);
        one += __shfl_xor(one, 32);
        if (A.order >= 1 && g == 0)
            put(one + D.q2[16 * i + li], ONE + i);
        if (A.order >= 2) {
            const i32x4 qi = *reinterpret_cast<const i32x4 *>(&D.q2[16 * i + 4 * g]);
#pragma unroll
            for (int j = i; j < NT; j++) {
                const int n = i * NT - i * (i - 1) / 2 + j - i;
                const i32x4 h = mfma<KD>(a.h, S[j], nil);
                const i32x4 l = mfma<KD>(a.l, S[j], nil);
                const int qj = D.q2[16 * j + li];
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    const int c = 254 * h[k] + l[k] + qi[k] + qj;
                    put(i == j && 4 * g + k >= li ? 2 * Q_PAD : c, 4 * n + k);  // i < j only
                }
            }
            __builtin_amdgcn_sched_barrier(0);  // else every product starts at once and spills
        }
    }
    const int thr = finite ? (wave_min(m1) >> 8) + 2 * (P + 2) + 8 : 0x7fffffff;
    // ---- pass 2: exact cost of the candidates near the least
    double bc = 0.0;
    int bk = 0x7fffffff;
    auto score = [&](int key) {
        const double d = exact_cost(D, d0, key);
        if (bk == 0x7fffffff || d < bc || (d == bc && key < bk)) {
            bc = d;
            bk = key;
        }
    };
    if (__ballot((m2 >> 8) <= thr) == 0ull) {
        // at most one candidate a lane
        const int idx = m1 & 255;
        int key = 0;
        bool in = (m1 >> 8) <= thr;
        if (idx < ONE) {
            int n = idx >> 2, i = 0;
            while (n >= NT - i && i < NT - 1) {
                n -= NT - i;
                i++;
            }
            const int p = 16 * i + 4 * g + (idx & 3), q = 16 * (i + n) + li;
            in = in && p < q && q < K;
            key = (2 << 14) | ((p & 127) << 7) | (q & 127);
        } else if (idx < BASE) {
            const int p = 16 * (idx - ONE) + li;
            in = in && p < K;
            key = (1 << 14) | ((p & 127) << 7);
        }
        if (in)
            score(key);
    } else {
        // ties: every candidate's cost once more
        const int nt = (K + 15) / 16;
        for (int i = A.order >= 1 ? -1 : nt; i < nt; i++) {
            // i = -1: the base candidate and single positions, as products with
            // the zero column
            Tile<KD> a;
            i32x4 qi = nil;
            if (i < 0) {
#pragma unroll
                for (int d = 0; d < ND; d++) {
                    a.h[d] = wp[0][d];
                    a.l[d] = wp[2][d];
                }
            } else {
                a = make_tile<KD>(wp, &D.x[16 * i + li], g);
                qi = *reinterpret_cast<const i32x4 *>(&D.q2[16 * i + 4 * g]);
            }
            if (i >= 0 && A.order < 2)
                break;
            for (int j = i < 0 ? 0 : i; j < nt; j++) {
                const Tile<KD> b = make_tile<KD>(wp, &D.x[16 * j + li], g);
                const i32x4 h = mfma<KD>(a.h, b.s, nil);
                const i32x4 l = mfma<KD>(a.l, b.s, nil);
                const int q = 16 * j + li, qj = D.q2[q & 127];
                uint32_t near = 0u;
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    const int c = 254 * h[k] + l[k] + qi[k] + qj, p = 16 * i + 4 * g + k;
                    const bool in = i < 0 ? k == 0 && g == 0 && q < K : p < q && q < K;
                    near |= (in && c <= thr ? 1u : 0u) << k;
                }
                while (near) {
                    const int k = __builtin_ctz(near);
                    near &= near - 1u;
                    score(i < 0 ? (1 << 14) | (q << 7) : (2 << 14) | ((16 * i + 4 * g + k) << 7) | q);
                }
            }
        }
        if (lane == 0)
            score(0);
    }
#pragma unroll
    for (int s = 1; s < WAVE; s <<= 1) {
        const double oc = __shfl_xor(bc, s);
        const int ok = __shfl_xor(bk, s);
        if (ok != 0x7fffffff && (bk == 0x7fffffff || oc < bc || (oc == bc && ok < bk))) {
            bc = oc;
            bk = ok;
        }
    }
    uint64_t m[2];
    disagreement(D, d0, __builtin_amdgcn_readfirstlane(bk), m);
    if (lane == 0) {
        uint64_t *dst = A.bits + f * A.bits_ld;
        dst[0] = z0 ^ m[0];
        if (N > WAVE)
            dst[1] = z1 ^ m[1];
    }
    __syncthreads();
}

// V < 0: any code of the mix; else the one code's variant
constexpr int kVariants = 8;

template <int V>
__device__ __forceinline__ void osd_variant(const OsdArgs &A, const OsdCode &C, int64_t f, DualLds &D)
{
    constexpr int nt[kVariants] = {3, 4, 7, 8, 3, 4, 5, 7};
    osd_dual<nt[V], (V < 4 ? 32 : 64)>(A, C, f, D);
}

template <int V>
__global__ void __launch_bounds__(WAVE) __attribute__((amdgpu_waves_per_eu(5))) osd_dual_kernel(OsdArgs A)
{
    __shared__ DualLds D;
    const int lane = threadIdx.x;
    const int64_t G = gridDim.x;
    for (int64_t base = blockIdx.x; base < A.F; base += G * WAVE) {
        // this wave's next 64 frames: which of them to decode
        const int64_t mine = base + G * lane;
        int c = -1;
        if (mine < A.F && !(A.skip && A.skip[mine]))
            c = A.code_idx ? (int)A.code_idx[mine] : 0;
        uint64_t todo = __ballot(c >= 0 && c < A.n_codes);
        while (todo) {
            const int k = __builtin_ctzll(todo);
            todo &= todo - 1ull;
            const int64_t f = base + G * k;
            const OsdCode &C = A.code[__builtin_amdgcn_readlane(c, k)];
            if constexpr (V >= 0) {
                osd_variant<V>(A, C, f, D);
            } else {
                switch (C.variant) {
                case 0: osd_variant<0>(A, C, f, D); break;
                case 1: osd_variant<1>(A, C, f, D); break;
                case 2: osd_variant<2>(A, C, f, D); break;
                case 3: osd_variant<3>(A, C, f, D); break;
                case 4: osd_variant<4>(A, C, f, D); break;
                case 5: osd_variant<5>(A, C, f, D); break;
                case 6: osd_variant<6>(A, C, f, D); break;
                case 7: osd_variant<7>(A, C, f, D); break;
                }
            }
        }
    }
}

}  // namespace

// the variant (tiles of 16 basis positions, depth) for a code, or -1
int osd_variant_of(int N, int K)
{
    const int P = N - K, nt = (K + 15) / 16;
    if (N > 128 || K < 1 || P < 1 || P > 64)
        return -1;
    if (P <= 32)
        return nt <= 3 ? 0 : (nt <= 4 ? 1 : (nt <= 7 ? 2 : (nt <= 8 ? 3 : -1)));
    return nt <= 3 ? 4 : (nt <= 4 ? 5 : (nt <= 5 ? 6 : (nt <= 7 ? 7 : -1)));
}

hipError_t launch_osd_dual(const OsdArgs &A, int n_cu, hipStream_t stream)
{
    if (A.F < 1)
        return hipSuccess;
    if (A.n_codes < 1 || A.n_codes > kOsdMaxCodes)
        return hipErrorInvalidValue;
    int v = A.code[0].variant;
    for (int c = 0; c < A.n_codes; c++) {
        if (A.code[c].variant < 0 || A.code[c].variant >= kVariants || A.code[c].hcol == nullptr)
            return hipErrorInvalidValue;
        if (A.code[c].variant != v)
            v = -1;
    }
    int64_t grid = (int64_t)n_cu * 64;
    if (grid > A.F)
        grid = A.F;
    const dim3 g((unsigned)grid), b(WAVE);
    switch (v) {
    case 0: hipLaunchKernelGGL(osd_dual_kernel<0>, g, b, 0, stream, A); break;
    case 1: hipLaunchKernelGGL(osd_dual_kernel<1>, g, b, 0, stream, A); break;
    case 2: hipLaunchKernelGGL(osd_dual_kernel<2>, g, b, 0, stream, A); break;
    case 3: hipLaunchKernelGGL(osd_dual_kernel<3>, g, b, 0, stream, A); break;
    case 4: hipLaunchKernelGGL(osd_dual_kernel<4>, g, b, 0, stream, A); break;
    case 5: hipLaunchKernelGGL(osd_dual_kernel<5>, g, b, 0, stream, A); break;
    case 6: hipLaunchKernelGGL(osd_dual_kernel<6>, g, b, 0, stream, A); break;
    case 7: hipLaunchKernelGGL(osd_dual_kernel<7>, g, b, 0, stream, A); break;
    default: hipLaunchKernelGGL(osd_dual_kernel<-1>, g, b, 0, stream, A); break;
    }
    return hipGetLastError();
}

hipError_t launch_osd(const OsdArgs &args, int n_cu, hipStream_t stream)
{
    OsdArgs A = args;
    if (A.N > 128 || A.K > 128 || A.K < 1)
        return hipErrorInvalidValue;
    int64_t grid = (int64_t)n_cu * 16;
    if (grid > A.F)
        grid = A.F;
    if (grid < 1)
        return hipSuccess;
    const int nk = n_candidates(A.order, A.K);
    A.keep_costs = nk <= KEEP_MAX ? 1 : 2;
    const size_t lds = (A.keep_costs == 1 ? sizeof(uint32_t) : sizeof(uint16_t)) * (size_t)nk;
    hipLaunchKernelGGL(osd_kernel, dim3((unsigned)grid), dim3(WAVE), lds, stream, A);
    return hipGetLastError();
}

}  // namespace bch
