// Row-parallel decoder: one workgroup per frame, lanes over the check rows and
// then over the coordinates, every index list read from tables made once per
// decoder.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <vector>

#include "internal.h"

namespace bch {

constexpr int kRpMaxCodes = 8;   // codes of one launch (a mixed batch)
constexpr int kRpCols = 6;       // columns of a row per table step
constexpr int kRpRecs = 4;       // row records of a coordinate per table step
// the smallest calls: waves of a type, and the tables whose parts its lanes hold
// in registers (steps of a wave's first and second round, records of a coordinate)
constexpr int kRpWide = 4;
constexpr int kRpWideSteps = 8;
constexpr int kRpWideSteps2 = 4;
constexpr int kRpWideRecs = 128;
constexpr size_t kRpMaxLds = 65536;  // LDS of one workgroup; a larger matrix does not use the kernel

// One code's tables (device pointers into one allocation) and parameters.
struct RowParTab {
    const uint32_t *steps;   // [step][64][3]: six 16-bit byte offsets into the extended input of a type
    const uint32_t *rounds;  // [round]: steps of the round
    const uint4 *mask;       // [round][64]: the row's columns as bits of the shift-0 sign word
    const uint32_t *slot;    // [round][64]: byte offset of the row's record
    const uint2 *recs;       // [chunk][64 NK]: four 16-bit byte offsets of row records
    const uint64_t *hsyn;    // [msyn][ceil(N/64)] standard parity-check rows
    int n_rounds, n_recs;        // n_recs: records of a coordinate (the longest list)
    int N, M, dp, msyn;
    int max_iter;
    float alpha;
    int wide;                    // the tables fit decode_wide's registers
};

struct RowParArgs {
    const void *llr;          // [F][ld] float32, or int8
    int64_t ld;
    int64_t F;
    const uint8_t *d_o;       // [F]
    const uint8_t *code_idx;  // [F] or null (every frame: tab[0])
    uint64_t *bits;           // [F][bits_ld]
    int64_t bits_ld;
    uint8_t *iters;           // [F]
    uint8_t *flags;           // [F]
    void *trace;              // [F][max_iter][ld] float32 / int32, or null (one code only)
    int n_codes;
    int wide;                 // kRpWide waves a type instead of one
    RowParTab tab[kRpMaxCodes];
};

// Host image of a code's tables; offsets in bytes into `data`.
struct RowParImage {
    std::vector<uint8_t> data;
    size_t steps = 0, rounds = 0, mask = 0, slot = 0, recs = 0, order = 0;
    int n_rounds = 0, n_recs = 0;
    int seg[3] = {0, 0, 0};  // generic kernels: records of a coordinate in shift s (the longest list)
    int sign_words = 0;      // words of a row's message signs
    bool wide = false;       // RowParTab::wide
};

// Tables of the nine-branch restart-mode decode of matrix p; false if an
// offset would not fit its 16 bits.
bool build_rowpar(const Pcm &p, RowParImage &out);

// LDS bytes of one workgroup on this code, with `waves` waves a type
size_t rowpar_lds_bytes(int N, int M, int dp, int waves);

// ---- generic decoder (k_rowgen.hip): any matrix, 1, 3 or 9 branches, all
// message modes.  The sums run over the shifts, then the types, so a
// coordinate's records are listed shift by shift.  With edge memory
// (memory = true) a list entry is a 32-bit word: byte offset of the row's
// state | the entry's position in the row << 16 | (32 word + bit) << 24 of the
// position's sign.
constexpr int kRgSigns = 30;  // positions (five table steps) whose signs share a word
constexpr int kRgLaunchFrames = 1 << 24;  // frames of one launch (below 2^32 work-items of 128 threads a frame)

struct RowGenTab {
    const uint32_t *steps;
    const uint32_t *rounds;
    const uint4 *mask;
    const uint32_t *slot;
    const uint32_t *recs;    // restart: uint2 chunks of four 16-bit offsets; else 32-bit entries
    int n_rounds;
    int seg[3];
    int stride;              // bytes of a row's record or state
    int ns, np;              // shifts and types
    int dp;                  // shift period, 0 for one branch
    int offsets;             // d_o is used (more than one branch)
    const uint8_t *order;    // [step][kRpCols][64]: position in the order read of a row's columns, ascending (a decoder
                             // that stands in for a specialised one-branch kernel), or null
};

bool build_rowgen(const Pcm &p, int n_branches, bool memory, bool ordered, RowParImage &out);
int rowgen_stride(const RowParImage &im, bool memory);
size_t rowgen_lds_bytes(const RowGenTab &t, int N, int M, int mode);

struct GenericArgs;
hipError_t launch_rowgen(const GenericArgs &a, const RowGenTab &t, hipStream_t stream);

hipError_t launch_rowpar(const RowParArgs &a, int fix8, hipStream_t stream);
// launch_rowpar runs kRpWide waves a type on these codes
bool rowpar_is_wide(const RowParArgs &a);

}  // namespace bch
