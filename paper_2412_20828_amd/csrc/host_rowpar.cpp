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

size_t rowpar_lds_bytes(int N, int M, int dp, int waves)
{
    const size_t ext = (size_t)((N + 2 * dp + 4) & ~3);
    const size_t us = N > kLanes ? 2 * kLanes : kLanes;
    return 4 * 3 * waves * ext + 8 * 3 * (size_t)(3 * M + 2) + 4 * 2 * 3 * us;
}

namespace {

// Rounds of 64 rows (s, r), s < ns: steps, masks and record slots.  stride:
// bytes of a record; where: if not null, receives each row's columns in the
// order read, [s * M + r][position] (the pad cell for a lane that sits out).
// ordered (one branch): also the positions of a row's columns, ascending.
void build_rounds(const Pcm &p, int ns, int dp, int stride, bool ordered, RowParImage &out,
                  std::vector<std::vector<int>> *where)
{
    const int N = p.N, M = p.M;
    const int ext = N + (ns - 1) * dp;  // cells of a type's extended input; cell ext is the pad (+inf)
    struct Item {
        int s, r, w;
    };
    std::vector<Item> items;
    for (int s = 0; s < ns; s++)
        for (int r = 0; r < M; r++)
            items.push_back({s, r, p.rows[r].weight()});
    // rows of like weight share a round, which then takes the steps of its heaviest row
    std::stable_sort(items.begin(), items.end(), [](const Item &a, const Item &b) { return a.w > b.w; });
    const int R = (int)(items.size() + kLanes - 1) / kLanes;
    std::vector<uint32_t> steps, rounds, mask, slot;
    std::vector<uint8_t> order;
    if (where)
        where->assign(ns * M, {});
    for (int q = 0; q < R; q++) {
        std::vector<std::vector<int>> cells(kLanes);
        int w = 0;
        for (int l = 0; l < kLanes; l++) {
            const size_t t = (size_t)q * kLanes + l;
            uint32_t mk[4] = {0, 0, 0, 0};
            int sl = ns * M + 1;  // idle lanes write a record nobody reads
            if (t < items.size()) {
                const Item &it = items[t];
                sl = it.s * M + it.r;
                for (int i = 0; i < N; i++)
                    if (p.rows[it.r].get(i)) {
                        cells[l].push_back(i + (ns - 1 - it.s) * dp);
                        const int k = ((i - it.s * dp) % N + N) % N;
                        mk[k >> 5] |= 1u << (k & 31);
                    }
                w = std::max(w, it.w);
            }
            mask.insert(mask.end(), mk, mk + 4);
            slot.push_back((uint32_t)(stride * sl));
        }
        const int n = (w + kRpCols - 1) / kRpCols;
        order_cells(cells, n * kRpCols, ext);
        for (int e = 0; e < n; e++)
            for (int l = 0; l < kLanes; l++)
                for (int h = 0; h < kRpCols / 2; h++) {
                    const uint32_t a = 4u * cells[l][e * kRpCols + 2 * h];
                    const uint32_t b = 4u * cells[l][e * kRpCols + 2 * h + 1];
                    steps.push_back(a | (b << 16));
                }
        for (int k = 0; ordered && k < n * kRpCols; k++)
            for (int l = 0; l < kLanes; l++) {
                std::vector<int> c;
                for (int x : cells[l])
                    if (x != ext)
                        c.push_back(x);
                std::sort(c.begin(), c.end());
                const bool in = k < (int)c.size();
                order.push_back(in ? (uint8_t)(std::find(cells[l].begin(), cells[l].end(), c[k]) - cells[l].begin()) : 0);
            }
        rounds.push_back((uint32_t)n);
        out.sign_words = std::max(out.sign_words, (n * kRpCols + kRgSigns - 1) / kRgSigns);
        if (where)
            for (int l = 0; l < kLanes && (size_t)q * kLanes + l < items.size(); l++) {
                const Item &it = items[(size_t)q * kLanes + l];
                (*where)[it.s * M + it.r] = cells[l];
            }
    }
    // one more step: the kernel reads a step ahead
    steps.insert(steps.end(), 3 * kLanes, 0u);
    out.steps = append(out.data, steps.data(), steps.size() * 4);
    out.rounds = append(out.data, rounds.data(), rounds.size() * 4);
    out.mask = append(out.data, mask.data(), mask.size() * 4);
    out.slot = append(out.data, slot.data(), slot.size() * 4);
    if (ordered)
        out.order = append(out.data, order.data(), order.size());
    out.n_rounds = R;
}

// Chunks of four 16-bit record offsets, [chunk][coordinate], zero records past
// a list's end; one chunk more than the longest list, which the kernel reads ahead.
int append_lists(const std::vector<std::vector<int>> &lists, int stride, int zero, std::vector<uint32_t> &recs)
{
    size_t most = 0;
    for (const auto &l : lists)
        most = std::max(most, l.size());
    const int C = (int)(most + kRpRecs - 1) / kRpRecs;
    for (int c = 0; c < C + 1; c++)
        for (const auto &l : lists)
            for (int h = 0; h < kRpRecs / 2; h++) {
                uint32_t v[2];
                for (int j = 0; j < 2; j++) {
                    const size_t e = (size_t)c * kRpRecs + 2 * h + j;
                    v[j] = (uint32_t)(stride * (e < l.size() ? l[e] : zero));
                }
                recs.push_back(v[0] | (v[1] << 16));
            }
    return (int)most;
}

}  // namespace

bool build_rowpar(const Pcm &p, RowParImage &out)
{
    const int N = p.N, M = p.M, dp = shift_period(N);
    constexpr int kRec = 8;
    if (kRec * (3 * M + 2) > 65535)
        return false;
    out = RowParImage();
    build_rounds(p, 3, dp, kRec, false, out, nullptr);
    // records of coordinate k in the order of the sums: shift 0's rows, 1's, 2's
    std::vector<std::vector<int>> lists(N > kLanes ? 2 * kLanes : kLanes);
    for (int k = 0; k < N; k++)
        for (int s = 0; s < 3; s++)
            for (int r = 0; r < M; r++)
                if (p.rows[r].get((k + s * dp) % N))
                    lists[k].push_back(s * M + r);
    std::vector<uint32_t> recs;
    out.n_recs = append_lists(lists, kRec, 3 * M, recs);
    out.recs = append(out.data, recs.data(), recs.size() * 4);
    out.wide = out.n_rounds <= (N > kLanes ? 1 : 2) * kRpWide && out.n_recs <= kRpWideRecs;
    for (int q = 0; q < out.n_rounds; q++) {
        const uint32_t n = reinterpret_cast<const uint32_t *>(out.data.data() + out.rounds)[q];
        out.wide = out.wide && (int)n <= (q < kRpWide ? kRpWideSteps : kRpWideSteps2);
    }
    return true;
}

int rowgen_stride(const RowParImage &im, bool memory)
{
    return memory ? 4 * ((3 + im.sign_words + 1) & ~1) : 8;
}

bool build_rowgen(const Pcm &p, int n_branches, bool memory, bool ordered, RowParImage &out)
{
    const int N = p.N, M = p.M, ns = n_branches > 1 ? 3 : 1, dp = n_branches > 1 ? shift_period(N) : 0;
    out = RowParImage();
    // the stride of a row's state depends on its steps, known from the heaviest row
    int w = 0;
    for (const Row &r : p.rows)
        w = std::max(w, r.weight());
    out.sign_words = ((w + kRpCols - 1) / kRpCols * kRpCols + kRgSigns - 1) / kRgSigns;
    const int stride = rowgen_stride(out, memory);
    if ((long)stride * (ns * M + 2) > 65535)
        return false;
    std::vector<std::vector<int>> where;
    build_rounds(p, ns, dp, stride, ordered, out, &where);
    const int n = N > kLanes ? 2 * kLanes : kLanes;
    std::vector<uint32_t> recs;
    for (int s = 0; s < ns; s++) {
        std::vector<std::vector<int>> lists(n), pos(n);
        size_t most = 0;
        for (int k = 0; k < N; k++) {
            const int i = (k + s * dp) % N;
            for (int r = 0; r < M; r++)
                if (p.rows[r].get(i)) {
                    const std::vector<int> &c = where[s * M + r];
                    const int e = (int)(std::find(c.begin(), c.end(), i + (ns - 1 - s) * dp) - c.begin());
                    // sign of position e: bit `last - e` of its word, whose positions end at `last`
                    const int word = e / kRgSigns, last = std::min(kRgSigns * (word + 1), (int)c.size()) - 1;
                    lists[k].push_back(s * M + r);
                    pos[k].push_back(e | (32 * word + last - e) << 8);
                }
            most = std::max(most, lists[k].size());
        }
        out.seg[s] = (int)most;
        if (!memory) {
            append_lists(lists, stride, ns * M, recs);
            continue;
        }
        for (size_t e = 0; e < most + 1; e++)
            for (int k = 0; k < n; k++) {
                const bool in = e < lists[k].size();
                recs.push_back((uint32_t)(stride * (in ? lists[k][e] : ns * M)) | (uint32_t)(in ? pos[k][e] : 0) << 16);
            }
    }
    out.recs = append(out.data, recs.data(), recs.size() * 4);
    return true;
}

size_t rowgen_lds_bytes(const RowGenTab &t, int N, int M, int mode)
{
    const size_t ext = (size_t)((N + (t.ns - 1) * t.dp + 4) & ~3);
    size_t n = 32 + 4 * t.np * ext + (size_t)t.stride * t.np * (t.ns * M + 2);
    if (mode == BCH_MODE_MEMORY)
        n += 4 * (size_t)t.np * t.ns * ext;
    return n;
}

}  // namespace bch
