// Bucketing prepass of the specialised decoder: frames are grouped by their
// random cyclic offset d_o so that a wave's 64 frames share every branch
// permutation.  Counting sort without global atomics:
//   1. each block of BLK frames counts its frames per bucket;
//   2. a workgroup per bucket scans its per-block counts (per-block offsets, total);
//   3. each block sums the totals (bucket starts; the first block writes the bucket
//      slices [cursor, end)) and places its frames at its offsets plus their rank inside the
//      block (LDS counters).
// Frames keep their input order inside a (block, bucket) up to the LDS-atomic
// ranks; no result depends on that order (every frame is decoded on its own).
// With a code index, either only the frames of one code of a mixed batch are
// taken, or (mixed-code kernels) every frame of codes 0..n_codes-1 goes to
// bucket base[code] + d_o mod d_p of its code.
#include <hip/hip_runtime.h>

#include "mix_launch.h"
#include "spec_launch.h"

namespace bch {

namespace {

constexpr int MAXB = 512;
constexpr int BLK = 2048;   // frames per counting block
constexpr int TPB = 256;    // threads per counting block
constexpr int SCAN = 1024;  // threads of a scan workgroup

// which frames go to which bucket: one code (code_idx null, or the frames
// with code_idx == code), bucket (f ranges / F) nofs + d_o mod dp (offset 0
// when !use; nofs = dp, or 1 when !use); or, with n_codes > 0, every frame of
// code c < n_codes to bucket base[c] + d_o mod dps[c]
struct BucketMap {
    const uint8_t *code_idx;
    int code, dp, use, nofs, ranges;
    int64_t F;
    int n_codes;
    int base[MIX_MAXC + 1];
    int dps[MIX_MAXC];
};

// bucket of frame f, or -1 if the map does not take it
__device__ __forceinline__ int bucket_of(const uint8_t *d_o, int64_t f, const BucketMap &m)
{
    if (m.n_codes > 0) {
        const int c = m.code_idx[f];
        return c < m.n_codes ? m.base[c] + (int)d_o[f] % m.dps[c] : -1;
    }
    if (m.code_idx && m.code_idx[f] != m.code)
        return -1;
    const int r = m.ranges > 1 ? (int)((f >> kRangeChunkLog2) % m.ranges) : 0;
    return r * m.nofs + (m.use ? (int)d_o[f] % m.dp : 0);
}

__global__ void __launch_bounds__(TPB) bucket_count(const uint8_t *__restrict__ d_o, BucketMap m, int64_t F,
                                                    int nb, int *__restrict__ blk_hist)
{
    __shared__ int h[MAXB];
    for (int i = threadIdx.x; i < nb; i += TPB)
        h[i] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * BLK;
    for (int k = threadIdx.x; k < BLK; k += TPB) {
        const int64_t f = base + k;
        if (f < F) {
            const int b = bucket_of(d_o, f, m);
            if (b >= 0)
                atomicAdd(&h[b], 1);
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < nb; i += TPB)
        blk_hist[(size_t)blockIdx.x * nb + i] = h[i];
}

// inclusive prefix over a wave's lanes
__device__ __forceinline__ int wave_prefix(int v, int lane)
{
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int t = __shfl_up(v, off);
        if (lane >= off)
            v += t;
    }
    return v;
}

// a workgroup per bucket: offsets of the blocks inside it, and its total.
// Latency bounds it: one workgroup for all buckets, 64 blocks of one a step,
// took 88 and 165 us at 4 and 7 million frames; 1024 blocks a step and the
// buckets side by side take 5 and 9
__global__ void __launch_bounds__(SCAN) bucket_scan(int *__restrict__ blk_hist, int nblk, int nb, BucketWs w)
{
    __shared__ int sums[2][SCAN / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, d = blockIdx.x;
    int carry = 0, turn = 0;
    for (int b0 = 0; b0 < nblk; b0 += SCAN, turn ^= 1) {
        const int b = b0 + tid;
        const int c = b < nblk ? blk_hist[(size_t)b * nb + d] : 0;
        const int v = wave_prefix(c, lane);
        if (lane == 63)
            sums[turn][wave] = v;
        __syncthreads();
        int before = carry;
#pragma unroll
        for (int k = 0; k < SCAN / 64; k++) {
            before += k < wave ? sums[turn][k] : 0;
            carry += sums[turn][k];
        }
        if (b < nblk)
            blk_hist[(size_t)b * nb + d] = before + v - c;
    }
    if (tid == 0)
        w.counts[d] = carry;
}

__global__ void __launch_bounds__(TPB) bucket_place(const uint8_t *__restrict__ d_o, BucketMap m, int64_t F,
                                                    int nb, const int *__restrict__ blk_off, BucketWs w)
{
    __shared__ int h[MAXB];
    // bucket starts: every block sums the totals, the first one writes the slices
    if (threadIdx.x < 64) {
        int start = 0;
        for (int i0 = 0; i0 < nb; i0 += 64) {
            const int i = i0 + threadIdx.x;
            const int c = i < nb ? w.counts[i] : 0;
            const int v = wave_prefix(c, threadIdx.x);
            if (i < nb) {
                h[i] = start + v - c + blk_off[(size_t)blockIdx.x * nb + i];
                if (blockIdx.x == 0) {
                    w.cursor[i] = start + v - c;
                    w.end[i] = start + v;
                }
            }
            start += __shfl(v, 63);
        }
    }
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * BLK;
    for (int k = threadIdx.x; k < BLK; k += TPB) {
        const int64_t f = base + k;
        if (f < F) {
            const int b = bucket_of(d_o, f, m);
            if (b >= 0) {
                const int pos = atomicAdd(&h[b], 1);
                w.order[pos] = (int)f;
            }
        }
    }
}

size_t align16(size_t x) { return (x + 15) & ~(size_t)15; }

int64_t n_blocks(int64_t F) { return (F + BLK - 1) / BLK; }

}  // namespace

size_t bucket_ws_bytes(int64_t F, int nb)
{
    const size_t head = align16(sizeof(int) * 3 * (size_t)nb);
    const size_t hist = align16(sizeof(int) * (size_t)n_blocks(F) * nb);
    return head + hist + align16((size_t)F * sizeof(int));
}

BucketWs bucket_ws_carve(void *ws, int64_t F, int nb)
{
    BucketWs w;
    char *p = static_cast<char *>(ws);
    int *h = reinterpret_cast<int *>(p);
    w.counts = h;
    w.cursor = h + nb;
    w.end = h + 2 * nb;
    p += align16(sizeof(int) * 3 * (size_t)nb);
    w.blk_hist = reinterpret_cast<int *>(p);
    p += align16(sizeof(int) * (size_t)n_blocks(F) * nb);
    w.order = reinterpret_cast<int *>(p);
    return w;
}

static hipError_t run_bucketing(const uint8_t *d_o, const BucketMap &m, int64_t F, int nb, const BucketWs &w,
                                hipStream_t stream)
{
    if (nb < 1 || nb > MAXB || F <= 0)
        return hipErrorInvalidValue;
    const int nblk = (int)n_blocks(F);
    hipLaunchKernelGGL(bucket_count, dim3(nblk), dim3(TPB), 0, stream, d_o, m, F, nb, w.blk_hist);
    hipLaunchKernelGGL(bucket_scan, dim3(nb), dim3(SCAN), 0, stream, w.blk_hist, nblk, nb, w);
    hipLaunchKernelGGL(bucket_place, dim3(nblk), dim3(TPB), 0, stream, d_o, m, F, nb, w.blk_hist, w);
    return hipGetLastError();
}

hipError_t launch_bucketing(const uint8_t *d_o, const uint8_t *code_idx, int code, int64_t F, int dp,
                            int use_offsets, int ranges, const BucketWs &w, hipStream_t stream)
{
    BucketMap m{};
    m.code_idx = code_idx;
    m.code = code;
    m.dp = dp;
    m.use = use_offsets;
    m.nofs = use_offsets ? dp : 1;
    if (ranges < 1 || ranges > kRangeXcds)
        return hipErrorInvalidValue;
    m.ranges = ranges;
    m.F = F;
    m.n_codes = 0;
    return run_bucketing(d_o, m, F, m.ranges * m.nofs, w, stream);
}

hipError_t launch_bucketing_mixed(const uint8_t *d_o, const uint8_t *code_idx, int n_codes, const int *dps,
                                  int64_t F, const BucketWs &w, hipStream_t stream)
{
    if (n_codes < 1 || n_codes > MIX_MAXC || code_idx == nullptr)
        return hipErrorInvalidValue;
    BucketMap m{};
    m.code_idx = code_idx;
    m.n_codes = n_codes;
    m.base[0] = 0;
    for (int c = 0; c < n_codes; c++) {
        m.dps[c] = dps[c];
        m.base[c + 1] = m.base[c] + dps[c];
    }
    return run_bucketing(d_o, m, F, m.base[n_codes], w, stream);
}

}  // namespace bch
