// Generic decoder: normalized min-sum decoding of any parity-check matrix in
// any of the three message-memory modes with 1, 3 or 9 branches, one workgroup
// per frame (one wave for N <= 64, two above), rows and coordinates over the
// lanes, index lists from tables made with the decoder (rowpar.h).
//
// Per iteration:
//   1. lane = coordinate u: |y_u| (or y_u, with edge memory) to each type's
//      extended input, in which branch (s, p) reads column i at cell
//      i + (2 - s) d_p; the signs of the whole word to both waves; the
//      syndrome of the last iteration's word;
//   2. lane = row (s, r), rounds of 64 rows of one type dealt to the waves:
//      restart mode finds min1, min2 and the sign parity of the row's cells;
//      with edge memory each v2c message is formed first, from the row's own
//      last messages (alpha min1, alpha min2, the argmin's position and a sign
//      bit per position, all a row's messages) and, in the literal mode, the
//      branch's last sums;
//   3. lane = coordinate: the c2v of its rows over the branches in order, rows
//      ascending, then y^(t).
// The sums have the order of the one-lane-per-frame kernel (k_generic.hip), and
// the results are the same bit for bit, of posteriors that are infinite or NaN
// too.  Message state lives in LDS; that kernel moves every edge's message
// through device memory, runs a frame's edges one after another and needs 64
// frames to fill a wave.  It stays for matrices whose records or state do not fit
// 64 KB of LDS or 16-bit offsets (rowgen_stride bytes a row, shift and type:
// nine branches from 874 rows (N = 127) or 892 (N = 63) in restart mode; extrinsic
// messages from 437 or 446 with rows of up to 30 entries, 291 or 297 of up to 90;
// literal memory 18 to 53 rows earlier; three branches with edge memory from
// about 860 to 900 with rows of more than 30; one branch never) and for restart messages with an infinite or NaN alpha.
//
// What bounds it: VALU issue and LDS reads (3.7 and 7 vector instructions an
// edge in steps 2 and 3 of restart mode, about 14 and 13 with edge memory;
// counted: 0.55 instructions per CU-cycle and the LDS 31% busy on 20,000 frames of
// (63,36) with 48 rows, 0.84 and 36% on 10,007 of plain (127,64)).
// Measured at 3 dB, us a call, one-lane-per-frame kernel / this one:
//   (63,36), 48 rows, 9 branches       1 frame 5415 / 35, 20,000: 14,705 / 224,
//                                      200,000: 59,210 / 1,629
//   (127,64), 100 rows, 9 branches     1: 45,647 / 108, 20,000: 46,832 / 994
//   (127,64) standard, plain NMS       1: 11,450 / 74, 10,007: 15,131 / 379,
//                                      200,000: 145,475 / 6,064
//   (63,45), 40 rows, 9, literal memory  4,000: 40,320 / 211
//   (127,99), 50 rows, 9, extrinsic      4,000: 107,128 / 782
// One wave (N <= 64) or two a frame, not one a type: the sums of step 3 run over
// the shifts first, so only the coordinates can be spread there.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "kernels.h"
#include "rowpar.h"
#include "rowsearch.h"

namespace bch {
namespace {

constexpr int WAVE = 64;

// all LDS traffic of the workgroup before this point is seen after it
template <int NK>
__device__ __forceinline__ void sync()
{
    if (NK > 1) {
        __syncthreads();
    } else {
        // one wave, whose LDS operations complete in order
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
}

struct StepWord {
    uint32_t x, y, z;
};

// a x mod N for the multipliers 1, 2, (N + 1) / 2 (0 <= x < N)
__device__ __forceinline__ int times(int p, int x, int N)
{
    const int dbl = 2 * x >= N ? 2 * x - N : 2 * x;
    const int hlf = (x & 1) ? (x + N) >> 1 : x >> 1;
    return p == 0 ? x : (p == 1 ? dbl : hlf);
}

// Extrinsic messages of a one-branch decoder that stands in for a specialised
// kernel: a row's entries in the order of that kernel (nms_spec_ext.inc), its
// signs the sign bits and its argmin the last entry equal to the least, as there.
// n <= 5 table steps from sp, ord: the position of the row's k-th column at [k][lane].
__device__ __forceinline__ void ordered_row(const StepWord *sp, const uint8_t *ord, int n, int w, int lane, const char *Eb,
                                            float alpha, char *rec)
{
    const float a1 = reinterpret_cast<const float *>(rec)[0], a2 = reinterpret_cast<const float *>(rec)[1];
    const uint32_t arg = reinterpret_cast<const uint32_t *>(rec)[2], old = reinterpret_cast<const uint32_t *>(rec)[3];
    const int last = kRpCols * n - 1;
    // v of the row's k-th column, at position e
    auto entry = [&](int k, int &e) {
        e = ord[k * WAVE + lane];
        const uint32_t st = reinterpret_cast<const uint32_t *>(sp + (e / kRpCols) * WAVE + lane)[e % kRpCols / 2];
        const float own = (uint32_t)e == arg ? a2 : a1;
        const float y = *reinterpret_cast<const float *>(Eb + (e & 1 ? st >> 16 : st & 0xffffu));
        return y - __uint_as_float(__float_as_uint(own) ^ ((old >> (last - e)) << 31));
    };
    int k = 0;
    uint32_t ng = 0u;
    const uint2 u = ordered_search(w, [&]() {
        int e;
        const uint32_t v = __float_as_uint(entry(k++, e));
        ng |= (v >> 31) << (last - e);
        return v & 0x7fffffffu;
    });
    uint32_t at = 0xffu;
#pragma unroll 1
    for (k = 0; k < w; k++) {
        int e;
        if ((__float_as_uint(entry(k, e)) & 0x7fffffffu) == u.x)
            at = (uint32_t)e;
    }
    const uint32_t par = (uint32_t)__builtin_popcount(ng) << 31;
    reinterpret_cast<uint32_t *>(rec)[0] = __float_as_uint(alpha * __uint_as_float(u.x)) ^ par;
    reinterpret_cast<uint32_t *>(rec)[1] = __float_as_uint(alpha * __uint_as_float(u.y)) ^ par;
    reinterpret_cast<uint32_t *>(rec)[2] = at;
    reinterpret_cast<uint32_t *>(rec)[3] = ng;
}

// ORD: extrinsic messages in the place of a specialised kernel; a kernel of its
// own, as the ordered search takes registers
template <int NK, int MODE, bool ORD>
__global__ void __launch_bounds__(NK *WAVE) rowgen_decode(GenericArgs A, RowGenTab tb)
{
    extern __shared__ __align__(16) char lds[];
    constexpr bool MEM = MODE != BCH_MODE_RESTART;
    const int N = A.N, M = A.M, ns = tb.ns, np = tb.np, dp = tb.dp;
    const int tid = threadIdx.x, lane = tid % WAVE;
    const int wv = __builtin_amdgcn_readfirstlane(tid / WAVE);
    const int64_t f = blockIdx.x;
    const int ext = N + (ns - 1) * dp;
    const int ext_pad = (ext + 4) & ~3;
    const int rec_type = tb.stride * (ns * M + 2);  // bytes of a type's records
    uint64_t *words = reinterpret_cast<uint64_t *>(lds);
    float *E = reinterpret_cast<float *>(lds + 32);
    char *Rb = lds + 32 + 4 * np * ext_pad;
    float *S = reinterpret_cast<float *>(Rb + np * rec_type);  // literal mode: [branch][cell] last sums
    const float *llr = static_cast<const float *>(A.llr) + f * A.ld;
    const int d_o = tb.offsets ? (int)A.d_o[f] % dp : 0;
    const bool in = tid < N;
    const float chan = in ? llr[tid] + 0.0f : 1.0f;
    float y = chan;
    // k of this coordinate in each type, and the coordinates at k = lane, lane + 64
    int kp[3], up[3][NK];
#pragma unroll
    for (int p = 0; p < 3; p++) {
        const int k = times(p == 0 ? 0 : 3 - p, in ? tid : 0, N) + d_o;
        kp[p] = k >= N ? k - N : k;
#pragma unroll
        for (int j = 0; j < NK; j++) {
            const int kk = lane + j * WAVE < N ? lane + j * WAVE : 0;
            up[p][j] = times(p, kk >= d_o ? kk - d_o : kk - d_o + N, N);
        }
    }
    uint64_t hs[2][NK];
#pragma unroll
    for (int r = 0; r < 2; r++)
#pragma unroll
        for (int w = 0; w < NK; w++) {
            const int row = lane + r * WAVE;
            hs[r][w] = row < A.msyn ? A.hsyn[row * NK + w] : 0ull;
        }
    if (tid < np)
        E[tid * ext_pad + ext] = __builtin_inff();
    if (MEM) {
        for (int i = tid; i < np * rec_type / 4; i += NK * WAVE)
            reinterpret_cast<uint32_t *>(Rb)[i] = 0u;
        if (MODE == BCH_MODE_MEMORY)
            for (int i = tid; i < np * ns * ext_pad; i += NK * WAVE)
                S[i] = 0.0f;
    } else if (tid < np) {
        *reinterpret_cast<uint2 *>(Rb + tid * rec_type + 8 * ns * M) = make_uint2(0u, 0u);
    }
    const float invB = (float)A.B;
    for (int t = 0;; t++) {
        // ---- 1. signs and inputs; syndrome and end of the frame
        {
            // the specialised kernels decide on the sign bit, of a NaN too
            const uint64_t w = __ballot(in && (ORD ? (int)__float_as_uint(y) < 0 : y < 0.0f));
            const bool odd_frame = ORD && __ballot(in && !(fabsf(y) < __builtin_inff())) != 0ull;
            if (NK > 1 && lane == 0)
                words[wv] = w;
            if (in)
                for (int p = 0; p < np; p++) {
                    // a NaN is no minimum of its rows and no least entry, as +inf is;
                    // the medians of the search would return one of the others for it
                    const float e = MEM ? y : fminf(fabsf(y), __builtin_inff());
                    float *dst = E + p * ext_pad + kp[p];
                    dst[(ns - 1) * dp] = e;
                    if (kp[p] >= N - (ns - 1) * dp)
                        dst[(ns - 1) * dp - N] = e;
                }
            sync<NK>();
            uint64_t W[NK];
#pragma unroll
            for (int k = 0; k < NK; k++)
                W[k] = NK > 1 ? words[k] : w;
            if (t > 0) {
                uint32_t odd = 0;
#pragma unroll
                for (int r = 0; r < 2; r++) {
                    uint64_t x = hs[r][0] & W[0];
                    if (NK == 2)
                        x ^= hs[r][NK - 1] & W[NK - 1];
                    odd |= (uint32_t)__popcll(x);
                }
                const bool ok = __ballot(odd & 1u) == 0ull;
                if (ok || t >= A.max_iter) {
                    if (tid == 0) {
#pragma unroll
                        for (int k = 0; k < NK; k++)
                            A.bits[f * NK + k] = W[k];
                        A.iters[f] = (uint8_t)t;
                        A.flags[f] = ok ? 1 : 0;
                    }
                    return;
                }
            }
            // ---- 2. rows: round (p, q) on wave (p n_rounds + q) mod NK
            for (int p = 0; p < np; p++) {
                const char *Eb = reinterpret_cast<const char *>(E + p * ext_pad);
                char *Rp = Rb + p * rec_type;
                uint32_t sw[2 * NK];  // sign word of the type's shift-0 input
                if (!MEM) {
#pragma unroll
                    for (int j = 0; j < NK; j++) {
                        const int u = up[p][j];
                        const uint64_t x = NK > 1 && u >= WAVE ? W[NK - 1] : W[0];
                        const uint64_t b = __ballot(lane + j * WAVE < N && ((x >> (u & 63)) & 1ull));
                        sw[2 * j] = (uint32_t)b;
                        sw[2 * j + 1] = (uint32_t)(b >> 32);
                    }
                }
                const StepWord *sp = reinterpret_cast<const StepWord *>(tb.steps);
                for (int q = 0; q < tb.n_rounds; q++) {
                    const int n = __builtin_amdgcn_readfirstlane(tb.rounds[q]);
                    if (NK > 1 && (p * tb.n_rounds + q) % NK != wv) {
                        sp += n * WAVE;
                        continue;
                    }
                    char *rec = Rp + tb.slot[q * WAVE + lane];
                    if constexpr (ORD) {
                        if (odd_frame) {
                            const uint4 mk = tb.mask[q * WAVE + lane];
                            const size_t step = sp - reinterpret_cast<const StepWord *>(tb.steps);  // WAVE words a step
                            ordered_row(sp, tb.order + kRpCols * step, n, __popc(mk.x) + __popc(mk.y), lane, Eb, A.alpha,
                                        rec);
                            sp += n * WAVE;
                            continue;
                        }
                    }
                    StepWord nx = sp[lane];
                    if constexpr (!MEM) {
                        const uint4 mk = tb.mask[q * WAVE + lane];
                        uint32_t u1 = 0x7f800000u, u2 = 0x7f800000u;
#pragma unroll 2
                        for (int e = 0; e < n; e++) {
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
                        uint32_t par = (sw[0] & mk.x) ^ (sw[1] & mk.y);
                        if (NK == 2)
                            par ^= (sw[2 * NK - 2] & mk.z) ^ (sw[2 * NK - 1] & mk.w);
                        *reinterpret_cast<uint2 *>(rec) = make_uint2(u1 | (uint32_t)__builtin_popcount(par) << 31, u2);
                    } else {
                        const float a1 = reinterpret_cast<const float *>(rec)[0];
                        const float a2 = reinterpret_cast<const float *>(rec)[1];
                        const uint32_t arg = reinterpret_cast<const uint32_t *>(rec)[2];
                        uint32_t *sg = reinterpret_cast<uint32_t *>(rec) + 3;
                        // literal mode: the sums of branch (s, p) of this lane's row
                        const char *Sb = nullptr;
                        if (MODE == BCH_MODE_MEMORY) {
                            const int row = (int)tb.slot[q * WAVE + lane] / tb.stride;
                            const int s = row / M < ns ? row / M : 0;
                            Sb = reinterpret_cast<const char *>(S + (s * np + p) * ext_pad);
                        }
                        float min1 = __builtin_inff(), min2 = __builtin_inff();
                        uint32_t at = 0xffu, ng = 0u, par = 0u, old = 0u;
                        for (int e = 0; e < n; e++) {
                            const StepWord st = nx;
                            sp += WAVE;
                            nx = sp[lane];
                            const int left = kRpCols * n - kRpCols * e, w = kRpCols * e / kRgSigns;
                            if (kRpCols * e % kRgSigns == 0)
                                old = sg[w] << (32 - (left < kRgSigns ? left : kRgSigns));
                            const uint32_t ad[6] = {st.x & 0xffffu, st.x >> 16, st.y & 0xffffu,
                                                    st.y >> 16,     st.z & 0xffffu, st.z >> 16};
#pragma unroll
                            for (int k = 0; k < 6; k++) {
                                float v = *reinterpret_cast<const float *>(Eb + ad[k]);
                                const float own = (uint32_t)(kRpCols * e + k) == arg ? a2 : a1;
                                v -= __uint_as_float(__float_as_uint(own) ^ (old & 0x80000000u));
                                old <<= 1;
                                if (MODE == BCH_MODE_MEMORY)
                                    v += *reinterpret_cast<const float *>(Sb + ad[k]);
                                const float m = fabsf(v);
                                if (m < min1) {
                                    min2 = min1;
                                    min1 = m;
                                    at = (uint32_t)(kRpCols * e + k);
                                } else if (m < min2) {
                                    min2 = m;
                                }
                                const uint32_t neg = v < 0.0f ? 1u : 0u;
                                ng = (ng << 1) | neg;
                                par ^= neg;
                            }
                            if (kRpCols * (e + 1) % kRgSigns == 0 || e == n - 1) {
                                sg[w] = ng;
                                ng = 0u;
                            }
                        }
                        const uint32_t sp1 = par << 31;
                        reinterpret_cast<uint32_t *>(rec)[0] = __float_as_uint(A.alpha * min1) ^ sp1;
                        reinterpret_cast<uint32_t *>(rec)[1] = __float_as_uint(A.alpha * min2) ^ sp1;
                        reinterpret_cast<uint32_t *>(rec)[2] = at;
                    }
                }
            }
        }
        sync<NK>();
        // ---- 3. c2v sums over the branches, y^(t)
        {
            float T = 0.0f;
            const float a = fabsf(y);
            const int n = NK * WAVE;
            const uint32_t *list = tb.recs;
            for (int s = 0; s < ns; s++) {
                const int cnt = tb.seg[s];
                for (int p = 0; p < np; p++) {
                    const char *Rp = Rb + p * rec_type;
                    const int k = kp[p];
                    if constexpr (!MEM) {
                        const uint2 *rp = reinterpret_cast<const uint2 *>(list);
                        uint2 nx = rp[k];
                        auto add = [&](uint2 id, int m) {
                            const uint32_t at[kRpRecs] = {id.x & 0xffffu, id.x >> 16, id.y & 0xffffu, id.y >> 16};
                            uint2 rc[kRpRecs];
#pragma unroll
                            for (int e = 0; e < kRpRecs; e++)
                                rc[e] = *reinterpret_cast<const uint2 *>(Rp + at[e]);
#pragma unroll
                            for (int e = 0; e < kRpRecs; e++) {
                                if (e >= m)
                                    break;
                                // row sign and magnitude; the sign of y_u comes in below
                                const float s1 = __uint_as_float(rc[e].x), m1 = fabsf(s1);
                                const float am = A.alpha * (a == m1 ? __uint_as_float(rc[e].y) : m1);
                                // alpha may be negative: flip, not set, the sign
                                T += __uint_as_float(__float_as_uint(am) ^ (__float_as_uint(s1) & 0x80000000u));
                            }
                        };
                        const int whole = cnt / kRpRecs;
#pragma unroll 2
                        for (int c = 0; c < whole; c++) {
                            const uint2 id = nx;
                            rp += n;
                            nx = rp[k];
                            add(id, kRpRecs);
                        }
                        switch (cnt % kRpRecs) {
                        case 1: add(nx, 1); break;
                        case 2: add(nx, 2); break;
                        case 3: add(nx, 3); break;
                        }
                    } else {
                        const uint32_t *rp = list;
                        float own = 0.0f;  // literal mode: the branch's sum
                        uint32_t nx = rp[k];
#pragma unroll 4
                        for (int c = 0; c < cnt; c++) {
                            const uint32_t id = nx;
                            rp += n;
                            nx = rp[k];
                            const char *rec = Rp + (id & 0xffffu);
                            const float2 am = *reinterpret_cast<const float2 *>(rec);
                            const uint32_t arg = *reinterpret_cast<const uint32_t *>(rec + 8);
                            const uint32_t bit = id >> 24;
                            const uint32_t sg = *reinterpret_cast<const uint32_t *>(rec + 12 + 4 * (bit >> 5));
                            const float m = ((id >> 16) & 0xffu) == arg ? am.y : am.x;
                            const float c2v = __uint_as_float(__float_as_uint(m) ^ ((sg >> (bit & 31u)) << 31));
                            T += c2v;
                            if (MODE == BCH_MODE_MEMORY)
                                own += c2v;
                        }
                        if (MODE == BCH_MODE_MEMORY && in) {
                            // cell of column i = k + s d_p mod N in branch (s, p)
                            int i = k + s * dp;
                            i = i >= N ? i - N : i;
                            S[(s * np + p) * ext_pad + i + (ns - 1 - s) * dp] = own;
                        }
                    }
                }
                list += MEM ? (cnt + 1) * n : (cnt + kRpRecs - 1) / kRpRecs * 2 * n + 2 * n;
            }
            if (in) {
                const float avg = ORD ? T : T / invB;
                if (MODE == BCH_MODE_RESTART)
                    // T holds the row signs only: sgn(y_u) is common to all its terms
                    y = y + __uint_as_float(__float_as_uint(avg) ^ (y < 0.0f ? 0x80000000u : 0u));
                else
                    y = (MODE == BCH_MODE_EXTRINSIC ? chan : y) + avg;
                if (A.trace)
                    A.trace[(f * A.max_iter + t) * A.ld_trace + tid] = y;
            }
        }
    }
}

template <int NK>
void launch(const GenericArgs &a, const RowGenTab &t, size_t lds, hipStream_t stream)
{
    const dim3 grid((unsigned)a.F), block(NK * WAVE);
    switch (a.mode) {
    case BCH_MODE_RESTART:
        hipLaunchKernelGGL((rowgen_decode<NK, BCH_MODE_RESTART, false>), grid, block, lds, stream, a, t);
        break;
    case BCH_MODE_MEMORY:
        hipLaunchKernelGGL((rowgen_decode<NK, BCH_MODE_MEMORY, false>), grid, block, lds, stream, a, t);
        break;
    default:
        if (NK == 1 && t.order)
            hipLaunchKernelGGL((rowgen_decode<1, BCH_MODE_EXTRINSIC, true>), grid, block, lds, stream, a, t);
        else
            hipLaunchKernelGGL((rowgen_decode<NK, BCH_MODE_EXTRINSIC, false>), grid, block, lds, stream, a, t);
        break;
    }
}

}  // namespace

hipError_t launch_rowgen(const GenericArgs &args, const RowGenTab &t, hipStream_t stream)
{
    const size_t lds = rowgen_lds_bytes(t, args.N, args.M, args.mode);
    if (args.F < 1 || lds > kRpMaxLds || args.msyn > 2 * WAVE)
        return hipErrorInvalidValue;
    // a dispatch counts its work-items, 64 or 128 a frame, in 32 bits: more
    // frames take several launches
    GenericArgs a = args;
    for (int64_t done = 0; done < args.F; done += a.F) {
        a.F = std::min(args.F - done, (int64_t)kRgLaunchFrames);
        a.llr = static_cast<const float *>(args.llr) + done * args.ld;
        a.d_o = args.d_o ? args.d_o + done : nullptr;
        a.bits = args.bits + done * args.W64;
        a.iters = args.iters + done;
        a.flags = args.flags + done;
        a.trace = args.trace ? args.trace + done * args.max_iter * args.ld_trace : nullptr;
        if (a.N > WAVE)
            launch<2>(a, t, lds, stream);
        else
            launch<1>(a, t, lds, stream);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess)
            return e;
    }
    return hipSuccess;
}

}  // namespace bch
