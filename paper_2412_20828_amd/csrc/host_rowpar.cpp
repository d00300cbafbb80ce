// Index tables of the row-parallel decoder (see k_rowpar.hip for how they are
// read).  Made once per decoder, on the host.
#include <algorithm>
#include <cstring>

#include "rowpar.h"

namespace bch {

namespace {

constexpr int kLanes = 64;
constexpr int kBanks = 32;  // LDS banks of four bytes that half a wave reads in one cycle

size_t append(std::vector<uint8_t> &d, const void *src, size_t n)
{
    d.resize((d.size() + 255) & ~(size_t)255);
    const size_t at = d.size();
    d.resize(at + n);
    std::memcpy(d.data() + at, src, n);
    return at;
}

// Order in which the 64 lanes of a round read their cells, so that the lanes
// of each half wave hit distinct LDS banks at every step as far as possible.
// The two least values of a row do not depend on the order.  Greedy, step by
// step: each lane takes, of its cells left, one whose bank is free (or whose
// very cell is read by another lane, which costs nothing), preferring the
// bank that its half wave still has to read most often.
void order_cells(std::vector<std::vector<int>> &cells, int steps, int pad)
{
    for (int half = 0; half < 2; half++) {
        std::vector<std::vector<int>> left(kLanes / 2), out(kLanes / 2);
        int need[kBanks] = {0};
        for (int l = 0; l < kLanes / 2; l++) {
            left[l] = cells[half * (kLanes / 2) + l];
            for (int c : left[l])
                need[c % kBanks]++;
        }
        for (int e = 0; e < steps; e++) {
            int used[kBanks];          // distinct cells of the bank read in this step
            int first[kBanks];
            std::fill(used, used + kBanks, 0);
            std::fill(first, first + kBanks, -1);
            for (int k = 0; k < kLanes / 2; k++) {
                const int l = (k + 5 * e) % (kLanes / 2);
                const int spare = steps - e - (int)left[l].size();  // steps this lane may still sit out
                int best = -1;
                long score = 0;
                for (size_t i = 0; i < left[l].size(); i++) {
                    const int c = left[l][i], b = c % kBanks;
                    const int cost = first[b] == c ? 0 : used[b];
                    const long s = -1000L * cost + need[b];
                    if (best < 0 || s > score) {
                        best = (int)i;
                        score = s;
                    }
                }
                if (best < 0 || (spare > 0 && score < -500)) {
                    out[l].push_back(pad);
                    continue;
                }
                const int c = left[l][best], b = c % kBanks;
                if (first[b] != c) {
                    used[b]++;
                    first[b] = c;
                }
                need[b]--;
                left[l].erase(left[l].begin() + best);
                out[l].push_back(c);
            }
        }
        for (int l = 0; l < kLanes / 2; l++)
            cells[half * (kLanes / 2) + l] = out[l];
    }
}

}  // namespace

size_t rowpar_lds_bytes(int N, int M, int dp)
{
    const size_t ext = (size_t)((N + 2 * dp + 4) & ~3);
    const size_t us = N > kLanes ? 2 * kLanes : kLanes;
    return 4 * 3 * ext + 8 * 3 * (size_t)(3 * M + 2) + 4 * 2 * 3 * us;
}

bool build_rowpar(const Pcm &p, RowParImage &out)
{
    const int N = p.N, M = p.M, dp = shift_period(N);
    const int ext = N + 2 * dp;  // cells of a type's extended input; cell ext is the pad (+inf)
    if (8 * (3 * M + 2) > 65535)
        return false;
    struct Item {
        int s, r, w;
    };
    std::vector<Item> items;
    for (int s = 0; s < 3; s++)
        for (int r = 0; r < M; r++)
            items.push_back({s, r, p.rows[r].weight()});
    // rows of like weight share a round, which then takes the steps of its heaviest row
    std::stable_sort(items.begin(), items.end(), [](const Item &a, const Item &b) { return a.w > b.w; });
    const int R = (int)(items.size() + kLanes - 1) / kLanes;
    std::vector<uint32_t> steps, rounds, mask, slot;
    for (int q = 0; q < R; q++) {
        std::vector<std::vector<int>> cells(kLanes);
        int w = 0;
        for (int l = 0; l < kLanes; l++) {
            const size_t t = (size_t)q * kLanes + l;
            uint32_t mk[4] = {0, 0, 0, 0};
            int sl = 3 * M + 1;  // idle lanes write a record nobody reads
            if (t < items.size()) {
                const Item &it = items[t];
                sl = it.s * M + it.r;
                for (int i = 0; i < N; i++)
                    if (p.rows[it.r].get(i)) {
                        cells[l].push_back(i - it.s * dp + 2 * dp);
                        const int k = ((i - it.s * dp) % N + N) % N;
                        mk[k >> 5] |= 1u << (k & 31);
                    }
                w = std::max(w, it.w);
            }
            mask.insert(mask.end(), mk, mk + 4);
            slot.push_back((uint32_t)(8 * sl));
        }
        const int ns = (w + kRpCols - 1) / kRpCols;
        order_cells(cells, ns * kRpCols, ext);
        for (int e = 0; e < ns; e++)
            for (int l = 0; l < kLanes; l++)
                for (int h = 0; h < kRpCols / 2; h++) {
                    const uint32_t a = 4u * cells[l][e * kRpCols + 2 * h];
                    const uint32_t b = 4u * cells[l][e * kRpCols + 2 * h + 1];
                    steps.push_back(a | (b << 16));
                }
        rounds.push_back((uint32_t)ns);
    }
    // one more step: the kernel reads a step ahead
    steps.insert(steps.end(), 3 * kLanes, 0u);
    // records of coordinate k in the order of the sums: shift 0's rows, 1's, 2's
    const int nk = N > kLanes ? 2 : 1;
    std::vector<std::vector<int>> lists(nk * kLanes);
    size_t most = 0;
    for (int k = 0; k < N; k++) {
        for (int s = 0; s < 3; s++)
            for (int r = 0; r < M; r++)
                if (p.rows[r].get((k + s * dp) % N))
                    lists[k].push_back(s * M + r);
        most = std::max(most, lists[k].size());
    }
    const int C = (int)(most + kRpRecs - 1) / kRpRecs;
    std::vector<uint32_t> recs;
    for (int c = 0; c < C + 1; c++)
        for (int k = 0; k < nk * kLanes; k++)
            for (int h = 0; h < kRpRecs / 2; h++) {
                uint32_t v[2];
                for (int j = 0; j < 2; j++) {
                    const size_t e = (size_t)c * kRpRecs + 2 * h + j;
                    v[j] = 8u * (uint32_t)(e < lists[k].size() ? lists[k][e] : 3 * M);  // 3 M: the zero record
                }
                recs.push_back(v[0] | (v[1] << 16));
            }
    out.data.clear();
    out.steps = append(out.data, steps.data(), steps.size() * 4);
    out.rounds = append(out.data, rounds.data(), rounds.size() * 4);
    out.mask = append(out.data, mask.data(), mask.size() * 4);
    out.slot = append(out.data, slot.data(), slot.size() * 4);
    out.recs = append(out.data, recs.data(), recs.size() * 4);
    out.n_rounds = R;
    out.n_recs = (int)most;
    return true;
}

}  // namespace bch
