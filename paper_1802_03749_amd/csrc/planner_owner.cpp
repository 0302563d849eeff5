// Host plans of the owner kernels: a hierarchical plan's blocks without an
// order between them.  Every point that a loop increments belongs to one of
// the blocks that touch it, and that block evaluates every element around
// the point; elements on a border between blocks are evaluated by each
// block that owns one of their points.  No point is then written by two
// blocks, so a sweep is one launch of blocks that neither wait nor colour.
#include <algorithm>
#include <cstdint>
#include <cstdlib>
#include <exception>
#include <initializer_list>
#include <memory>
#include <new>
#include <thread>

#include "internal.hpp"

namespace um {

namespace {

// Launch order of nb blocks in G = 8 or the caller's number of XCD groups:
// the k-th workgroup takes the next block of id range k mod G (G equal
// ranges), or, once that range is used up, of the range with most left.
std::vector<int32_t> interleaved_blocks(int32_t nb, int32_t G) {
    std::vector<int32_t> order(nb), next(G), end(G);
    for (int32_t g = 0; g < G; ++g) {
        // ids b with floor(b * G / nb) == g
        next[g] = int32_t((int64_t(g) * nb + G - 1) / G);
        end[g] = int32_t((int64_t(g + 1) * nb + G - 1) / G);
    }
    for (int32_t k = 0; k < nb; ++k) {
        int32_t g = k % G;
        if (next[g] == end[g])
            for (int32_t h = 0; h < G; ++h)
                if (end[h] - next[h] > end[g] - next[g]) g = h;
        order[k] = next[g]++;
    }
    return order;
}

// The same over windows of 8 * 32 consecutive blocks: each XCD takes 32
// neighbouring blocks and all of them stay in one part of the mesh.
std::vector<int32_t> windowed_blocks(int32_t nb) {
    constexpr int32_t X = 8, B = 32;
    std::vector<int32_t> order(nb);
    for (int32_t k = 0; k < nb; ++k) {
        const int32_t w = k / (X * B) * (X * B), i = k - w;
        order[k] = w + X * B <= nb ? w + i % X * B + i / X : k;
    }
    return order;
}

// Length of the run of consecutive ids that starts the sorted list's first n.
int32_t leading_run(const std::vector<int32_t> &v, size_t n) {
    size_t r = n > 0;
    while (r < n && v[r] == v[r - 1] + 1) ++r;
    return int32_t(r);
}

// Moves the sorted list's longest run to its front; returns its length.
int32_t longest_run_first(std::vector<int32_t> &v) {
    size_t best = 0, len = 0;
    for (size_t i = 0; i < v.size();) {
        size_t j = i + 1;
        while (j < v.size() && v[j] == v[j - 1] + 1) ++j;
        if (j - i > len) {
            best = i;
            len = j - i;
        }
        i = j;
    }
    std::rotate(v.begin(), v.begin() + best, v.begin() + best + len);
    return int32_t(len);
}

// Consecutive workgroups go to the 8 XCDs in turn, each with its own L2, so
// neighbouring blocks, which stage each other's border points, are dealt 8
// apart: one eighth of the blocks to each XCD where the sweep's data stay in
// the 256 MB last-level cache (edge loop, 1200x600 cells: 19.2 us, in windows
// 19.6, in plain order 22.7), in windows where they stream from memory
// (2400x1200: 73.1 us, in eighths 76.4, in plain order 76.4).
std::vector<int32_t> launch_order(int32_t nb, const um_plan_opts &o, int64_t bytes) {
    if (o.xcd_groups > 1) return interleaved_blocks(nb, o.xcd_groups);
    return bytes > 256000000 ? windowed_blocks(nb) : interleaved_blocks(nb, 8);
}

// The owners of a map's points, and the elements around each point.
struct Around {
    int32_t D = 0;                       // incidences held per point
    std::vector<int32_t> own_off, own;   // per block: its points, ascending
    std::vector<int32_t> inc;            // [points][D]: arity * element + slot, ascending
    std::vector<uint8_t> deg;            // how many of them
    std::vector<int32_t> owner;          // per point, -1 if no block touches it

    // Owner of a point: the first of the blocks that touch it or, where that
    // leaves the blocks' points in fewer runs of consecutive ids, the last.
    // False if a point has more incidences than the largest of `sizes`.
    bool build(const Map &m, int64_t P, const std::vector<int32_t> &blk_off,
               std::initializer_list<int32_t> sizes) {
        const int32_t nb = int32_t(blk_off.size()) - 1;
        const int64_t k = m.arity;
        if (k * int64_t(blk_off[nb]) > int64_t(INT32_MAX)) return false;
        std::vector<int32_t> first(P), last(P);
        bool full = true;
        for (auto size = sizes.begin(); full && size != sizes.end(); ++size) {
            D = *size;
            full = false;
            inc.resize(size_t(P) * D);
            deg.assign(P, 0);
            std::fill(first.begin(), first.end(), -1);
            for (int32_t b = 0; b < nb && !full; ++b)
                for (int64_t i = k * blk_off[b]; i < k * blk_off[b + 1]; ++i) {
                    const int32_t p = m.table[i];
                    if (first[p] < 0) first[p] = b;
                    last[p] = b;
                    full = deg[p] == D;
                    if (full) break;
                    inc[size_t(p) * D + deg[p]++] = int32_t(i);
                }
        }
        if (full) return false;
        int64_t breaks = 0;
        for (int64_t p = 1; p < P; ++p)
            if (first[p] >= 0 && first[p - 1] >= 0)
                breaks += (last[p] != last[p - 1]) - (first[p] != first[p - 1]);
        own_off.assign(nb + 1, 0);
        if (breaks < 0)
            for (int64_t p = 0; p < P; ++p)
                if (first[p] >= 0) first[p] = last[p];
        owner.swap(first);
        for (int64_t p = 0; p < P; ++p)
            if (owner[p] >= 0) own_off[owner[p] + 1]++;
        for (int32_t b = 0; b < nb; ++b) own_off[b + 1] += own_off[b];
        own.resize(own_off[nb]);
        std::vector<int32_t> fill(own_off.begin(), own_off.end() - 1);
        for (int64_t p = 0; p < P; ++p)
            if (owner[p] >= 0) own[fill[owner[p]]++] = int32_t(p);
        return true;
    }
};

// Per cell, bit k set if a boundary edge (nodes a, b; its cell) is the cell's
// side from node k to node k + 1; false if one is none of its cell's sides or
// two are the same.
bool far_sides(const std::vector<int32_t> &b2c, const std::vector<int32_t> &b2n,
               const int32_t *c2n, int64_t C, std::vector<uint8_t> &far) {
    far.assign(C, 0);
    for (size_t e = 0; e < b2c.size(); ++e) {
        const int32_t *n = c2n + 4 * int64_t(b2c[e]);
        int k = 0;
        while (k < 4 && (n[k] != b2n[2 * e] || n[(k + 1) & 3] != b2n[2 * e + 1])) ++k;
        if (k == 4 || far[b2c[e]] >> k & 1) return false;
        far[b2c[e]] |= uint8_t(1 << k);
    }
    return true;
}

uint16_t *zeroed(int64_t n) {
    void *p = std::calloc(size_t(std::max<int64_t>(n, 1)), sizeof(uint16_t));
    if (!p) throw std::bad_alloc();
    return static_cast<uint16_t *>(p);
}

// One side of an owned cell: staged positions of the neighbour and of the
// nodes a, b (the normal of (a, b) points out of the cell), slot of the cell.
struct Side {
    uint32_t h, a, b, slot;
};

// Arranges the n sides around the cell (side k from corner k to corner k + 1
// mod 4) as s[0..3], missing ones with h = NO_CELL; false if they don't fit.
bool arrange(const Side *side, int32_t n, Side s[4], uint32_t corner[4]) {
    if (n > 4) return false;
    // usually each side's end is the start of one that follows in the list or
    // closes the ring: follow them from the first
    for (int32_t c = 0; c < 4; ++c) s[c] = Side{NO_CELL, 0, 0, 0};
    corner[0] = corner[1] = corner[2] = corner[3] = 0;
    if (n == 4) {
        int32_t at = 0, left = 0xE, k = 0;  // sides 1..3 are still to be placed
        for (; k < 4; ++k) {
            s[k] = side[at];
            corner[k] = side[at].a;
            if (k == 3) break;
            const uint32_t end = side[at].b;
            int32_t j = 1;
            while (j < 4 && !((left >> j & 1) && side[j].a == end)) ++j;
            if (j == 4) break;
            left &= ~(1 << j);
            at = j;
        }
        if (k == 3 && s[3].b == corner[0]) return true;
    }
    bool used[4] = {false, false, false, false};
    int32_t first = 0;
    // start where no side ends, if there is such a place
    for (int32_t i = 0; i < n; ++i) {
        bool ends = false;
        for (int32_t j = 0; j < n; ++j) ends |= j != i && side[j].b == side[i].a;
        if (!ends) {
            first = i;
            break;
        }
    }
    int32_t k = 0, at = n > 0 ? first : -1, placed = 0;
    for (int32_t c = 0; c < 4; ++c) {
        s[c] = Side{NO_CELL, 0, 0, 0};
        corner[c] = 0;
    }
    bool set[4] = {false, false, false, false};
    auto put = [&](int32_t c, uint32_t v) {
        c &= 3;
        if (set[c] && corner[c] != v) return false;
        set[c] = true;
        corner[c] = v;
        return true;
    };
    while (placed < n) {
        if (at < 0) {  // the next side starts anew, one corner further
            ++k;
            for (int32_t j = 0; j < n && at < 0; ++j)
                if (!used[j]) at = j;
        }
        if (k > 3 || !put(k, side[at].a) || !put(k + 1, side[at].b)) return false;
        s[k++] = side[at];
        used[at] = true;
        ++placed;
        int32_t next = -1;
        for (int32_t j = 0; j < n && next < 0; ++j)
            if (!used[j] && side[j].a == side[at].b) next = j;
        at = next;
    }
    return true;
}

// Places the n sides at the corners they run between, and the boundary
// sides' marks; false if a side is none of those or taken.
bool place(const Side *side, int32_t n, uint8_t far, uint32_t far_pos, const uint32_t corner[4],
           Side s[4]) {
    for (int k = 0; k < 4; ++k) s[k] = Side{far >> k & 1 ? far_pos : NO_CELL, 0, 0, 0};
    for (int32_t i = 0; i < n; ++i) {
        int k = 0;
        while (k < 4 && (corner[k] != side[i].a || corner[(k + 1) & 3] != side[i].b)) ++k;
        if (k == 4 || s[k].h != NO_CELL) return false;
        s[k] = side[i];
    }
    return true;
}

// Runs work(b0, b1) over [0, nb) in as many ranges as threads are worth it
// for E elements, each on its own thread; the largest result.
template <typename F>
auto in_ranges(int32_t nb, int64_t E, F work) {
    using R = decltype(work(0, 0));
    const int64_t most = std::min<int64_t>(8, std::thread::hardware_concurrency());
    const int32_t n = int32_t(std::max<int64_t>(1, std::min<int64_t>({most, nb, E / 10000})));
    std::vector<R> got(n, R{});
    std::vector<std::exception_ptr> failed(n);
    auto part = [&](int32_t i) {
        try {
            got[i] = work(int32_t(int64_t(i) * nb / n), int32_t(int64_t(i + 1) * nb / n));
        } catch (...) {
            failed[i] = std::current_exception();
        }
    };
    std::vector<std::thread> threads;
    for (int32_t i = 1; i < n; ++i) {
        try {
            threads.emplace_back(part, i);
        } catch (const std::exception &) {  // no more threads to be had
            part(i);
        }
    }
    part(0);
    for (std::thread &t : threads) t.join();
    for (const std::exception_ptr &e : failed)
        if (e) std::rethrow_exception(e);
    return *std::max_element(got.begin(), got.end());
}

}  // namespace

void build_owner_plan(const Ctx &ctx, const EdgeArgs &ea, const um_plan_opts &o, HostPlan &hp,
                      const StepArgs *sa) {
    const Map &mc = ctx.maps[ea.map_c];
    const Map &mn = ctx.maps[ea.map_n];
    const int64_t C = ctx.sets[mc.to].size, N = ctx.sets[mn.to].size;
    const int64_t E = int64_t(mc.table.size()) / 2;
    const int32_t nb = int32_t(hp.blk_off.size()) - 1;
    OwnerPlan &op = hp.owner;
    op = OwnerPlan{};
    if (nb <= 0) return;

    Around ar;
    if (!ar.build(mc, C, hp.blk_off, {4, 4 * MAX_SIDE_QUADS})) return;
    op.quads = ar.D / 4;
    const auto &[D, own_off, own, inc, deg, owner] = ar;
    const int32_t *rows_c2n = nullptr;
    std::vector<uint8_t> far;  // per cell: which sides are boundary edges'
    if (sa) {
        if (int64_t(own.size()) != C || op.quads != 1) return;
        rows_c2n = ctx.maps[sa->map_c2n].table.data();
        if (!far_sides(ctx.maps[sa->map_c].table, ctx.maps[sa->map_n].table, rows_c2n, C, far))
            return;
    }

    const int64_t w = ea.dtype == UM_F64 ? 8 : 4;
    const std::vector<int32_t> order =
        launch_order(nb, o, C * (5 * w + 32 + 12) + N * 2 * w);
    std::vector<int32_t> pos_of(nb);
    op.rec.resize(nb);
    int64_t rows = 0;
    for (int32_t k = 0; k < nb; ++k) {
        pos_of[order[k]] = k;
        op.rec[k].word_off = int32_t(rows);
        op.rec[k].n_own = own_off[order[k] + 1] - own_off[order[k]];
        rows += op.rec[k].n_own;
        op.n_own_max = std::max(op.n_own_max, op.rec[k].n_own);
    }
    std::vector<std::vector<int32_t>> items(nb), shared(nb);
    enum Result { OK = 0, NO_RING = 1, TOO_LARGE = 2 };
    // the records, listed ids and side words of blocks [b0, b1)
    auto plan_range = [&](int32_t b0, int32_t b1, bool ring) -> Result {
        // staged position + 1 of a point; 0 elsewhere, so that a thread only
        // touches its own blocks' part of the arrays
        const std::unique_ptr<uint16_t, void (*)(void *)> cm(zeroed(C), std::free),
            nm(zeroed(N), std::free);
        uint16_t *const cpos = cm.get(), *const npos = nm.get();
        std::vector<int32_t> cells, nodes;
        Side s[4 * MAX_SIDE_QUADS], g[4];
        uint32_t corner[4];
        for (int32_t b = b0; b < b1; ++b) {
            const int32_t k = pos_of[b];
            OwnRec &r = op.rec[k];
            cells.assign(own.begin() + own_off[b], own.begin() + own_off[b + 1]);
            nodes.clear();
            for (int32_t c : cells) cpos[c] = 1;
            for (int32_t i = 0; i < r.n_own; ++i)
                for (int32_t a = 0; a < deg[cells[i]]; ++a) {
                    const int64_t here = inc[size_t(cells[i]) * D + a], there = here ^ 1;
                    const int32_t h = mc.table[there];
                    if (!cpos[h]) {
                        cpos[h] = 1;
                        cells.push_back(h);
                    }
                    for (int64_t t : {here, there})
                        if (!npos[mn.table[t]]) {
                            npos[mn.table[t]] = 1;
                            nodes.push_back(mn.table[t]);
                        }
                }
            if (sa)
                for (int32_t i = 0; i < 4 * (sa->own_adt ? int32_t(cells.size()) : r.n_own); ++i) {
                    const int32_t n = rows_c2n[4 * int64_t(cells[i / 4]) + i % 4];
                    if (!npos[n]) {
                        npos[n] = 1;
                        nodes.push_back(n);
                    }
                }
            std::sort(cells.begin() + r.n_own, cells.end());
            std::sort(nodes.begin(), nodes.end());
            r.nc = int32_t(cells.size());
            r.nn = int32_t(nodes.size());
            if (r.nc > MAX_OWNER_POINTS || r.nn > MAX_OWNER_POINTS) return TOO_LARGE;
            const bool lists = o.explicit_lists != 0;
            r.c_run = lists ? 0 : leading_run(cells, r.n_own);
            r.n_run = lists ? 0 : longest_run_first(nodes);
            r.c_start = r.n_own ? cells[0] : 0;
            r.n_start = r.nn ? nodes[0] : 0;
            for (int32_t i = 0; i < r.nc; ++i) cpos[cells[i]] = uint16_t(i + 1);
            for (int32_t i = 0; i < r.nn; ++i) npos[nodes[i]] = uint16_t(i + 1);
            for (int32_t i = 0; i < r.n_own; ++i) {
                int32_t n = 0;
                for (; n < deg[cells[i]]; ++n) {
                    // the normal of (a, b) points out of the edge's cell 0
                    const int64_t here = inc[size_t(cells[i]) * D + n], there = here ^ 1;
                    s[n] = Side{cpos[mc.table[there]] - 1u, npos[mn.table[here]] - 1u,
                                npos[mn.table[there]] - 1u, uint32_t(here & 1)};
                }
                if (ring) {
                    if (sa) {
                        for (int j = 0; j < 4; ++j)
                            corner[j] = npos[rows_c2n[4 * int64_t(cells[i]) + j]] - 1u;
                        if (!place(s, n, far[cells[i]], uint32_t(r.nc), corner, g)) return NO_RING;
                    } else if (!arrange(s, n, g, corner)) {
                        return NO_RING;
                    }
                    uint32_t *w = &op.words[3 * size_t(r.word_off) + i];
                    w[0] = g[0].h | g[1].h << 10 | g[2].h << 20 | g[0].slot << 30 | g[1].slot << 31;
                    w[r.n_own] =
                        g[3].h | corner[0] << 10 | corner[1] << 20 | g[2].slot << 30 | g[3].slot << 31;
                    w[2 * r.n_own] = corner[2] | corner[3] << 10;
                    if (sa && std::any_of(s, s + n, [&](const Side &t) {
                            return owner[cells[t.h]] != b;
                        })) {
                        shared[k].push_back(cells[i]);
                        w[2 * r.n_own] |= uint32_t(shared[k].size()) << 20;
                    }
                } else {
                    uint32_t *w = &op.words[(size_t(r.word_off) + i) * D];
                    for (int32_t j = 0; j < D; ++j)
                        w[j] = j < n ? s[j].h | s[j].a << 10 | s[j].b << 20 | s[j].slot << 30
                                     : NO_SIDE;
                }
            }
            // explicit ids: cells past the run, padded to a whole wavefront,
            // then nodes past theirs
            std::vector<int32_t> &it = items[k];
            it.assign(cells.begin() + r.c_run, cells.end());
            it.resize((it.size() + 63) / 64 * 64, 0);
            r.node_item = int32_t(it.size());
            it.insert(it.end(), nodes.begin() + r.n_run, nodes.end());
            r.n_items = int32_t(it.size());
            if (sa && sa->own_adt)
                for (int32_t i = r.n_own; i < r.nc; ++i) {
                    for (int j = 0; j < 4; ++j)
                        corner[j] = npos[rows_c2n[4 * int64_t(cells[i]) + j]] - 1u;
                    it.push_back(int32_t(corner[0] << 10 | corner[1] << 20));
                    it.push_back(int32_t(corner[2] | corner[3] << 10));
                }
            for (int32_t c : cells) cpos[c] = 0;
            for (int32_t n : nodes) npos[n] = 0;
        }
        return OK;
    };
    Result res = op.quads == 1 ? OK : NO_RING;
    for (bool ring : {true, false}) {
        if (ring ? res != OK : sa != nullptr) continue;
        op.ring = ring;
        op.words.assign(size_t(rows) * (ring ? 3 : D), 0u);
        res = in_ranges(nb, E, [&](int32_t b0, int32_t b1) { return plan_range(b0, b1, ring); });
        if (res != NO_RING) break;
    }
    int32_t lanes = op.n_own_max;  // a lane per owned cell, or per cell whose adt it evaluates
    for (int32_t k = 0; k < nb; ++k) {
        const OwnRec &r = op.rec[k];
        op.id_stride = std::max(op.id_stride, int32_t(items[k].size()));
        if (sa && sa->own_adt) lanes = std::max(lanes, r.nc);
        op.lds = std::max(op.lds, owner_lds_bytes(ea.dtype, r.nc + (sa ? 1 : 0), r.nn));
    }
    if (res != OK || op.lds > (o.lds_limit_bytes > 0 ? o.lds_limit_bytes : ctx.lds_limit)) {
        op = OwnerPlan{};
        return;
    }
    op.ids.assign(size_t(nb) * op.id_stride, 0);
    for (int32_t k = 0; k < nb; ++k) {
        std::copy(items[k].begin(), items[k].end(), op.ids.begin() + size_t(k) * op.id_stride);
        op.rec[k].own_off = int32_t(op.shared.size());
        op.shared.insert(op.shared.end(), shared[k].begin(), shared[k].end());
    }
    op.threads = std::max(64, (lanes + 63) / 64 * 64);
    op.use = true;
}

// Elements of a dataflow hex loop above which its waiting kernel is the faster
// one.  A brick of 8x8x4 elements evaluates 405 to 441 for its 256 nodes.  On
// small meshes that costs less than waiting for eight block colours in turn; on
// large ones the chain is hidden and the extra evaluations are not.  One sweep
// in us, waiting -> owner kernel, MIN colouring, 256 elements per block unless
// stated:
//   AoS, barrier rounds: 24^3 elements 25.3 -> 6.0 (RECOLOUR), 104^3 52.2 -> 41.6,
//     120^3 73.7 -> 61.5, 124^3 81.9 -> 77.3 (128 per block 101 -> 84), but 128^3
//     73.4 -> 75.5.  Blocks of 512 were refused below 2,000,000 elements for what
//     they stage; the bricks of 128^3 are not, and would gain.
//   AoS, LDS atomics, whose single round makes a shorter chain: 104^3 48.8 -> 42.0,
//     116^3 58.1 -> 56.3 (320 per block 61.2 -> 62.3), 120^3 64.6 -> 62.2 (320:
//     64.9 -> 68.7), 124^3 68.5 -> 76.6 (128: 83.3 -> 84.1; but 64: 107 -> 91).
//   SoA data wait longer: 124^3 88.8 -> 79.8, LDS atomics 80.5 -> 79.8.
//   Blocks that are chunks of the RCM order evaluate up to 3.9 elements per
//     element (64 per block; larger ones stage too much): AoS 80^3 61.9 -> 44.3,
//     104^3 92.7 -> 92.3, 112^3 111 -> 115, 124^3 147 -> 167; LDS atomics 88^3
//     58.8 -> 58.2, 96^3 69.8 -> 74.3; SoA 104^3 99.4 -> 97.1.
// As launches the colours cost more at every size and in every order: 24^3 59.0
// -> 5.9, 96^3 110 -> 33.4, 124^3 144 -> 77, 160^3 258 -> 189 (chunks, 64 per
// block: 124^3 194 -> 169, 160^3 382 -> 362).
static int64_t waiting_from(bool redundant, bool few_rounds, int32_t block_size) {
    if (redundant) return few_rounds ? 800000 : 1200000;
    return few_rounds && block_size >= 128 ? 1600000 : 2000000;
}

// The same for the hex loop: nodes are owned, a block evaluates every element
// around its nodes.
void build_owner_plan_hex(const Ctx &ctx, const HexArgs &ha, const um_plan_opts &o,
                          HostPlan &hp) {
    const Map &m = ctx.maps[ha.map];
    const int64_t N = ctx.sets[m.to].size, E = hp.n_elem;
    const int32_t nb = int32_t(hp.blk_off.size()) - 1;
    OwnerPlan &op = hp.owner;
    op = OwnerPlan{};
    if (nb <= 0) return;
    const bool flow = o.schedule == UM_SCHED_DATAFLOW;
    const bool few_rounds = ha.layout == UM_AOS && o.tcmode == UM_TC_LDS_ATOMIC;
    if (flow && E > waiting_from(false, few_rounds, o.block_size)) return;
    Around ar;
    if (!ar.build(m, N, hp.blk_off, {8, MAX_NODE_ELEMENTS})) return;
    const auto &[D, own_off, own, inc, deg, owner] = ar;
    for (uint8_t n : deg) op.quads = std::max<int32_t>(op.quads, n);

    const std::vector<int32_t> order = launch_order(nb, o, N * 72 + E * 24);
    std::vector<int32_t> pos_of(nb);
    op.rec.resize(nb);
    op.counts.reserve(own.size());
    int64_t owned = 0;
    for (int32_t k = 0; k < nb; ++k) {
        const int32_t b = order[k];
        pos_of[b] = k;
        op.rec[k].own_off = int32_t(owned);
        op.rec[k].n_own = own_off[b + 1] - own_off[b];
        op.n_own_max = std::max(op.n_own_max, op.rec[k].n_own);
        owned += op.rec[k].n_own;
    }
    op.counts.resize(owned);
    std::vector<std::vector<int32_t>> items(nb);
    std::vector<std::vector<uint32_t>> words(nb);
    // the records, listed ids and elements of blocks [b0, b1): 0, or 1 if one
    // of them is too large
    auto plan_range = [&](int32_t b0, int32_t b1) -> int32_t {
        const std::unique_ptr<uint16_t, void (*)(void *)> nm(zeroed(N), std::free);
        uint16_t *const npos = nm.get();
        std::vector<int32_t> nodes, elems;
        std::vector<uint8_t> seen;
        for (int32_t b = b0; b < b1; ++b) {
            const int32_t k = pos_of[b];
            OwnRec &r = op.rec[k];
            nodes.assign(own.begin() + own_off[b], own.begin() + own_off[b + 1]);
            elems.clear();
            for (int32_t n : nodes)
                for (int32_t a = 0; a < deg[n]; ++a) elems.push_back(inc[size_t(n) * D + a] / 8);
            std::sort(elems.begin(), elems.end());
            elems.erase(std::unique(elems.begin(), elems.end()), elems.end());
            for (int32_t n : nodes) npos[n] = 1;
            for (int32_t e : elems)
                for (int a = 0; a < 8; ++a) {
                    const int32_t n = m.table[8 * int64_t(e) + a];
                    if (!npos[n]) {
                        npos[n] = 1;
                        nodes.push_back(n);
                    }
                }
            std::sort(nodes.begin() + r.n_own, nodes.end());
            r.nc = int32_t(nodes.size());
            r.nn = int32_t(elems.size());
            if (r.nc > MAX_OWNER_POINTS || r.nn > 1024) return 1;
            r.c_run = o.explicit_lists != 0 ? 0 : leading_run(nodes, r.n_own);
            r.c_start = r.n_own ? nodes[0] : 0;
            for (int32_t i = 0; i < r.nc; ++i) npos[nodes[i]] = uint16_t(i + 1);
            for (int32_t i = 0; i < r.n_own; ++i) op.counts[r.own_off + i] = deg[nodes[i]];
            std::vector<uint32_t> &w = words[k];
            w.assign(4 * size_t(r.nn), 0u);
            seen.assign(r.n_own, 0);
            for (int32_t i = 0; i < r.nn; ++i)
                for (int a = 0; a < 8; ++a) {
                    const uint32_t t = npos[m.table[8 * int64_t(elems[i]) + a]] - 1u;
                    w[4 * i + a / 3] |= t << (10 * (a % 3));
                    if (t < uint32_t(r.n_own)) w[4 * i + 3] |= uint32_t(seen[t]++) << (4 * a);
                }
            std::vector<int32_t> &it = items[k];
            it.assign(nodes.begin() + r.c_run, nodes.end());
            r.n_items = int32_t(it.size());
            for (int32_t n : nodes) npos[n] = 0;
        }
        return 0;
    };
    const int32_t res = in_ranges(nb, 8 * E, plan_range);
    int64_t rows = 0;
    int32_t lanes = 64;
    for (int32_t k = 0; k < nb; ++k) {
        OwnRec &r = op.rec[k];
        r.word_off = int32_t(rows);
        rows += r.nn;
        op.id_stride = std::max(op.id_stride, r.n_items);
        op.lds = std::max(op.lds, hex_owner_lds_bytes(r.nc, r.n_own, op.quads));
        lanes = std::max({lanes, r.nn, r.n_own});
    }
    op.threads = (lanes + 63) / 64 * 64;
    const bool slow = flow && E > waiting_from(2 * rows > 5 * E, few_rounds, o.block_size);
    if (res != 0 || slow || op.threads > 1024 || rows > int64_t(INT32_MAX) ||
        op.lds > (o.lds_limit_bytes > 0 ? o.lds_limit_bytes : ctx.lds_limit)) {
        op = OwnerPlan{};
        return;
    }
    op.words.reserve(4 * size_t(rows));
    op.ids.assign(size_t(nb) * op.id_stride, 0);
    for (int32_t k = 0; k < nb; ++k) {
        op.words.insert(op.words.end(), words[k].begin(), words[k].end());
        std::copy(items[k].begin(), items[k].end(), op.ids.begin() + size_t(k) * op.id_stride);
    }
    op.use = true;
}

}  // namespace um
