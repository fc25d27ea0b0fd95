// Host-side checks of the library's own host code, built with AddressSanitizer
// and UndefinedBehaviorSanitizer (host pass only, no device code): the
// population tables of the update, the tiling of tensors and of blocks, the
// int8 row divisor, the geometry of quantized blocks, the launches of the step
// kernels, and every argument check that fails before the device is touched.
// The library source is compiled into this translation unit, so its internal
// (anonymous-namespace) routines are reachable; each is compared with a plain
// reference written here.  Prints "ok" and exits 0, or names the first
// failure and exits 1.
#include "../../paper_2608_17310_amd/csrc/esopt.hip"

#include <cstdio>
#include <random>

namespace {

int g_failures = 0;

void check(bool ok, const char* what) {
    if (!ok && g_failures++ < 20) std::printf("FAIL: %s\n", what);
}

// Population tables: distinct seeds in order of first appearance, members
// grouped by seed in member order.
void test_member_tables(std::mt19937_64& rng) {
    for (int trial = 0; trial < 400; ++trial) {
        const uint32_t n = trial < 4 ? uint32_t(trial == 3 ? ES_MAX_MEMBERS : trial + 1)
                                     : uint32_t(1 + rng() % ES_MAX_MEMBERS);
        const uint64_t pool = 1 + rng() % (trial % 3 == 0 ? 4 : n + 3);   // repeats likely
        std::vector<uint64_t> seeds(n);
        std::vector<int32_t> signs(n);
        for (uint32_t i = 0; i < n; ++i) {
            seeds[i] = (rng() % pool) * 0x9E3779B97F4A7C15ull;              // spread over 64 bits
            signs[i] = (rng() & 1) ? 1 : -1;
        }
        MemberTables t;
        build_member_tables(seeds.data(), signs.data(), n, t);
        // reference: first appearances by a quadratic scan
        std::vector<uint64_t> distinct;
        for (uint32_t i = 0; i < n; ++i) {
            bool seen = false;
            for (uint64_t d : distinct) seen |= (d == seeds[i]);
            if (!seen) distinct.push_back(seeds[i]);
        }
        check(t.n_distinct == distinct.size(), "member tables: distinct count");
        uint32_t pos = 0;
        for (uint32_t d = 0; d < t.n_distinct && d < distinct.size(); ++d) {
            const uint64_t key = uint64_t(t.din[d].k0) | (uint64_t(t.din[d].k1) << 32);
            check(key == distinct[d], "member tables: distinct order");
            check(t.din[d].first == pos, "member tables: CSR offsets");
            uint32_t expect_count = 0;
            for (uint32_t i = 0; i < n; ++i) {
                if (seeds[i] != distinct[d]) continue;
                check(t.min[pos + expect_count].reward_index == i, "member tables: member order");
                check(t.min[pos + expect_count].sign == signs[i], "member tables: signs");
                ++expect_count;
            }
            check(t.din[d].count == expect_count, "member tables: counts");
            pos += expect_count;
        }
        check(pos == n, "member tables: every member once");
    }
}

// Tiling: every element in exactly one tile, tiles sorted full-then-tail,
// full tiles whole and on tile-sized address boundaries.
void test_tiling(std::mt19937_64& rng) {
    const uint64_t tile = uint64_t(kDefaultThreads) * kDefaultGroups * kGroupElems;
    std::vector<es_tile_info_t> out;
    for (int trial = 0; trial < 600; ++trial) {
        const uint64_t addr = (rng() % (uint64_t(1) << 40)) & ~uint64_t(trial % 4 == 0 ? 1 : 15);
        const uint64_t numel = trial % 5 == 0 ? rng() % 20 : rng() % (5 * tile + 3);
        const uint32_t off8 = trial % 7 == 0 ? uint32_t(rng() % (1u << 31)) : 0u;
        uint64_t n = 0;
        check(es_tile_layout(addr, numel, off8, nullptr, 0, &n) == ES_OK, "tile layout: count");
        out.assign(n + 1, es_tile_info_t{});
        uint64_t n2 = 0;
        check(es_tile_layout(addr, numel, off8, out.data(), n, &n2) == ES_OK && n2 == n,
              "tile layout: list");
        std::vector<uint8_t> cover(numel, 0);
        bool tails = false;
        for (uint64_t i = 0; i < n; ++i) {
            const es_tile_info_t& ti = out[i];
            const uint64_t base = 8 * uint64_t(off8);
            check(ti.elem0 >= base && ti.end <= base + numel && ti.elem0 < ti.end,
                  "tile layout: tile inside the tensor");
            if (ti.full) {
                check(!tails, "tile layout: full tiles first");
                check(ti.end - ti.elem0 == tile, "tile layout: full tile size");
                check((addr + 2 * (ti.elem0 - base)) % (2 * tile) == 0,
                      "tile layout: full tile on an address boundary");
            } else {
                tails = true;
                check(ti.end - ti.elem0 <= tile, "tile layout: tail tile size");
            }
            for (uint64_t e = ti.elem0; e < ti.end && e - base < numel; ++e) ++cover[e - base];
        }
        bool once = true;
        for (uint8_t c : cover) once &= (c == 1);
        check(once, "tile layout: every element in exactly one tile");
        // a short output array receives only `cap` entries
        if (n > 1) {
            es_tile_info_t one[1];
            check(es_tile_layout(addr, numel, off8, one, 1, &n2) == ES_OK && n2 == n,
                  "tile layout: capped output");
        }
    }
    uint64_t n = 0;
    check(es_tile_layout(1, 10, 0, nullptr, 0, &n) == ES_ERR_ALIGN, "tile layout: odd address");
    check(es_tile_layout(0, 10, 0, nullptr, 0, nullptr) == ES_ERR_INVALID_ARG,
          "tile layout: null count");
    check(es_tile_layout(0, uint64_t(1) << 61, 0, nullptr, 0, &n) == ES_ERR_INVALID_ARG,
          "tile layout: above 2^60");
    check(es_tile_layout(0, 10, 0, nullptr, 5, &n) == ES_ERR_INVALID_ARG,
          "tile layout: null output with a capacity");
}

// Block tiling (es_plan_create_blocks): every element of a block lies in
// exactly one tile, at its own address, and the index the kernels give it is
// its whole-tensor index (row0 + i) row_len + col0 + j.  The kernels take a
// group's index at its first element (tile start + a multiple of 8) and
// count on from there: the descriptor's element itself for a contiguous
// layout, rows_index through the row map for a strided piece.
struct BlockCheck {
    const es_block_t& b;
    uintptr_t addr;
    uint64_t numel;
    std::vector<uint8_t>* cover;           // null: sampled check only
    uint64_t expected(uint64_t local) const {
        return (b.row0 + local / b.cols) * b.row_len + b.col0 + local % b.cols;
    }
    // element e of a tile: its address gives its place in the block
    void element(const DevTile& d, const DevRows* m, uint64_t e) {
        const uintptr_t a = reinterpret_cast<uintptr_t>(d.data) + 2 * e;
        check(a >= addr && (a - addr) / 2 < numel, "block tiling: address inside the block");
        if (a < addr || (a - addr) / 2 >= numel) return;
        const uint64_t local = (a - addr) / 2;
        if (cover) ++(*cover)[local];
        const uint64_t g = d.elem0 + ((e - d.elem0) & ~uint64_t(7));
        const uint64_t n = m ? rows_index(m->n0, m->skip, m->magic, m->shift, g) + (e - g)
                             : e;
        check(n == expected(local), "block tiling: whole-tensor index");
        if (m) check(e < (uint64_t(1) << 31), "block tiling: piece index below 2^31");
        // a strided tile's high word is its row map's
        if (m) check((n >> 34) == m->hi, "block tiling: high word of a strided tile");
        // the counter's high word is taken per tile for a contiguous layout
        if (!m) check((d.elem0 >> 34) == (e >> 34), "block tiling: uniform high word");
    }
    void tiles(const std::vector<DevTile>& v, const std::vector<DevRows>* rows, bool full,
               uint64_t tile, bool sampled) {
        for (size_t i = 0; i < v.size(); ++i) {
            const DevTile& d = v[i];
            const DevRows* m = rows ? &(*rows)[i] : nullptr;
            check(d.elem0 < d.limit && d.limit - d.elem0 <= tile, "block tiling: tile size");
            if (full) {
                check(d.limit - d.elem0 == tile, "block tiling: full tile size");
                check((reinterpret_cast<uintptr_t>(d.data) + 2 * d.elem0) % (2 * tile) == 0,
                      "block tiling: full tile on an address boundary");
            }
            check(d.elem0 % 8 == 0 || d.aligned16 == 0, "block tiling: group starts");
            if (sampled) {
                for (uint64_t e : {d.elem0, d.elem0 + 7, (d.elem0 + d.limit) / 2, d.limit - 1})
                    if (e < d.limit) element(d, m, e);
            } else {
                for (uint64_t e = d.elem0; e < d.limit; ++e) element(d, m, e);
            }
        }
    }
};

void test_block_tiling(std::mt19937_64& rng) {
    const uint64_t tile = uint64_t(kDefaultThreads) * kDefaultGroups * kGroupElems;
    int strided_seen = 0, row_by_row_seen = 0, high_word_cuts = 0;
    for (int trial = 0; trial < 280; ++trial) {
        es_block_t b{};
        const int kind = trial % 7;
        if (kind == 0) {                                  // one row, any length
            b.rows = 1;
            b.cols = rng() % (3 * tile);
            b.row_len = b.cols + rng() % 5000;
            b.col0 = rng() % (b.row_len - b.cols + 1);
            b.row0 = rng() % 1000;
            const uint64_t first = b.row0 * b.row_len + b.col0;
            b.col0 -= std::min(b.col0, first % 8);        // first index a multiple of 8
            if ((b.row0 * b.row_len + b.col0) % 8 != 0) b.row0 = 0, b.col0 = 0;
        } else if (kind == 1) {                           // whole rows, any row length
            b.cols = b.row_len = 1 + rng() % 3000;
            b.rows = 1 + rng() % 60;
            b.row0 = 8 * (rng() % 1000);
        } else if (kind == 5) {                           // rows 2^32 or more apart
            b.cols = 8 * (1 + rng() % 40);
            b.row_len = (uint64_t(1) << 32) + 8 * (rng() % 1000) + b.cols;
            b.rows = 2 + rng() % 6;
            b.row0 = rng() % 1000;
            b.col0 = 8 * (rng() % 100);
        } else if (kind == 6) {                           // rows just under 2^32 apart: the
            b.cols = 8 * (1 + rng() % 8);                 // index passes a multiple of 2^34
            b.row_len = (uint64_t(1) << 32) - 8 * (rng() % 1000);   // every ~4 rows
            b.rows = 2 + rng() % 100;
            b.row0 = rng() % 50;
            b.col0 = 8 * (rng() % 100);
        } else {                                          // column / 2-D shards
            b.cols = 8 * (1 + rng() % (kind == 2 ? 4 : 700));
            b.row_len = b.cols + 8 * (1 + rng() % 2000);
            b.col0 = 8 * (rng() % ((b.row_len - b.cols) / 8 + 1));
            b.rows = 2 + rng() % (kind == 2 ? 3000 : 150);
            // some blocks straddle whole-tensor element 2^34
            b.row0 = kind == 4 ? (uint64_t(1) << 34) / b.row_len - b.rows / 2 : rng() % 100000;
        }
        const uintptr_t addr =
            uintptr_t(0x100000000000ull + (rng() % (uint64_t(1) << 40))) &
            ~uintptr_t(trial % 5 == 0 ? 1 : 15);
        b.data = reinterpret_cast<void*>(addr);
        b.tensor_id = uint32_t(trial);
        check(block_geometry_error(b).empty(), "block tiling: generated geometry is valid");
        PlanTiles t;
        tile_block(b, tile, t);
        check(t.rows_full.size() == t.rfull.size() && t.rows_tail.size() == t.rtail.size(),
              "block tiling: one row map per strided tile");
        const bool contiguous = b.rows == 1 || b.cols == b.row_len;
        check(!contiguous || t.rfull.empty() && t.rtail.empty(),
              "block tiling: contiguous blocks take the plain layout");
        strided_seen += !t.rfull.empty() || !t.rtail.empty();
        for (size_t i = 1; i < t.rows_tail.size(); ++i)
            high_word_cuts += t.rows_tail[i].hi != t.rows_tail[i - 1].hi &&
                              t.rtail[i].elem0 == t.rtail[i - 1].limit;
        row_by_row_seen += kind == 5 && t.rfull.empty() && t.rtail.empty() && !t.tail.empty();
        const uint64_t numel = b.rows * b.cols;
        std::vector<uint8_t> cover(numel, 0);
        BlockCheck c{b, addr, numel, &cover};
        c.tiles(t.full, nullptr, true, tile, false);
        c.tiles(t.tail, nullptr, false, tile, false);
        c.tiles(t.rfull, &t.rows_full, true, tile, false);
        c.tiles(t.rtail, &t.rows_tail, false, tile, false);
        bool once = true;
        for (uint8_t k : cover) once &= (k == 1);
        check(once, "block tiling: every element in exactly one tile");
    }
    check(strided_seen > 100 && row_by_row_seen > 20 && high_word_cuts > 200,
          "block tiling: every layout exercised");

    // a block of more than 2^31 elements is cut into pieces of whole rows:
    // sampled elements of every tile, and the tiles' sizes add up
    es_block_t b{};
    b.rows = 3000;
    b.cols = uint64_t(1) << 20;
    b.row_len = b.cols + 5120;
    b.col0 = 2560;
    b.row0 = 17;
    b.data = reinterpret_cast<void*>(uintptr_t(0x200000000000ull + 4096));
    PlanTiles t;
    tile_block(b, tile, t);
    uint64_t total = 0;
    for (const auto* v : {&t.full, &t.tail, &t.rfull, &t.rtail})
        for (const DevTile& d : *v) total += d.limit - d.elem0;
    check(total == b.rows * b.cols, "block tiling: pieces add up to the block");
    check(t.full.empty() && t.tail.empty(), "block tiling: pieces are strided");
    std::vector<uint64_t> n0s;
    for (const DevRows& m : t.rows_full) n0s.push_back(m.n0);
    std::sort(n0s.begin(), n0s.end());
    n0s.erase(std::unique(n0s.begin(), n0s.end()), n0s.end());
    check(n0s.size() == 2, "block tiling: two pieces of 2048 and 952 rows");
    BlockCheck c{b, reinterpret_cast<uintptr_t>(b.data), b.rows * b.cols, nullptr};
    c.tiles(t.rfull, &t.rows_full, true, tile, true);
    c.tiles(t.rtail, &t.rows_tail, false, tile, true);
}

// Row divisor: exact for every j < 2^31 (boundaries of every row, and random j).
void test_row_divisor(std::mt19937_64& rng) {
    std::vector<uint32_t> rows = {8, 16, 24, 64, 1000, 1024, 5120, 17408, 151936, 1u << 20,
                                  (1u << 30) + 8, 0x7FFFFFF8u};
    for (int i = 0; i < 200; ++i) rows.push_back(8 * uint32_t(1 + rng() % (1u << 27)));
    for (uint32_t r : rows) {
        uint32_t magic = 0, shift = 0;
        row_divisor(r, magic, shift);
        auto q = [&](uint32_t j) {
            return uint32_t((uint64_t(j) * magic) >> 32) >> shift;
        };
        bool ok = true;
        for (uint64_t k = 0; k * r < (uint64_t(1) << 31) && k < 4096; ++k) {
            const uint64_t j = k * r;
            ok &= q(uint32_t(j)) == k;
            if (j > 0) ok &= q(uint32_t(j - 1)) == k - 1;
        }
        const uint32_t top = 0x7FFFFFFFu;
        ok &= q(top) == top / r;
        ok &= q(top - top % r) == top / r;
        for (int t = 0; t < 2000; ++t) {
            const uint32_t j = uint32_t(rng() % (uint64_t(1) << 31));
            ok &= q(j) == j / r;
        }
        check(ok, "row divisor: exact below 2^31");
    }
}

// Quantized blocks: the geometry rules of es_qblock_t against a plain
// statement of them, and for every accepted block the kernels' index map
// n0 + j + (j / cols) skip (the division as the device computes it) against
// the whole-tensor index (row0 + i) row_len + col0 + c, j = i cols + c.
void test_qblock_geometry(std::mt19937_64& rng) {
    const uint64_t lim = uint64_t(1) << 31;
    auto pick = [&](uint64_t hi) { return hi == 0 ? 0 : rng() % hi; };
    int accepted = 0;
    for (int t = 0; t < 20000; ++t) {
        es_qblock_t b{};
        const int scale = int(rng() % 4);
        const uint64_t grain = (rng() % 4 == 0) ? 1 : 16;
        b.row_len = grain * (1 + pick(scale == 3 ? (uint64_t(1) << 27) : 4096 / grain));
        b.cols = 1 + pick(b.row_len + 2);
        b.col0 = pick(b.row_len + 1);
        if (rng() % 4 != 0) {                   // mostly blocks the rules allow
            b.cols = std::max<uint64_t>(16, (b.cols / 16) * 16);
            b.col0 = (b.col0 / 16) * 16;
            if (b.col0 + b.cols > b.row_len) b.col0 = b.row_len >= b.cols ? (b.row_len - b.cols) / 16 * 16 : 0;
        }
        b.rows = pick(scale == 0 ? 3 : scale == 1 ? 64 : (uint64_t(1) << 16));
        b.row0 = pick(scale == 3 ? (uint64_t(1) << 5) : (uint64_t(1) << 12));
        if (rng() % 8 == 0) b.rows = (uint64_t(1) << 40) + pick(5);
        QSpec spec{};
        const std::string err = qblock_geometry(b, spec);
        // the rules, stated plainly (products kept below 2^64 by the ranges above)
        const uint64_t n = (b.rows == 0 || b.cols == 0) ? 0
                           : (b.rows < lim && b.cols < lim) ? b.rows * b.cols : lim;
        bool ok = n < lim;
        if (ok && n > 0) {
            const uint64_t first = b.row0 * b.row_len + b.col0;
            const uint64_t end = (b.row0 + b.rows - 1) * b.row_len + b.col0 + b.cols;
            const bool strided = b.rows > 1 && b.cols < b.row_len;
            ok = b.col0 + b.cols <= b.row_len && end < lim && first % 16 == 0 &&
                 (!strided || (b.cols % 16 == 0 && b.row_len % 16 == 0));
        }
        check(ok == err.empty(), "qblock geometry: accepted exactly when the rules hold");
        if (!ok || n == 0) continue;
        ++accepted;
        check(spec.numel == n, "qblock geometry: numel");
        uint32_t cmagic = 0, cshift = 0;
        if (spec.skip != 0) row_divisor(uint32_t(spec.cols), cmagic, cshift);
        bool map_ok = true;
        for (int k = 0; k < 64; ++k) {
            const uint64_t j = k < 2 ? (k == 0 ? 0 : n - 1) : pick(n);
            uint64_t got = spec.n0 + j;
            if (spec.skip != 0)
                got += uint64_t((uint32_t((uint64_t(uint32_t(j)) * cmagic) >> 32) >> cshift)) *
                       spec.skip;
            const uint64_t exp = (b.row0 + j / b.cols) * b.row_len + b.col0 + j % b.cols;
            map_ok &= got == exp && exp < lim;
        }
        check(map_ok, "qblock geometry: index map");
    }
    check(accepted > 5000, "qblock geometry: enough accepted blocks");
}

// The launches of the one-step workgroups: the order over the XCDs is a
// permutation, every step of every tile is taken by exactly one workgroup and no
// workgroup is without one, whatever the tail tiles' lengths (also when a pass
// is cut into several launches), and every launch stays below 2^32 lanes
// whatever the plan's size.
struct StepCover {
    uint64_t n_full;
    uint32_t full_shift;
    std::vector<TileDesc> tiles;                 // the full ones, then the tails
    TailIndex index;
    std::vector<std::vector<uint8_t>> taken;     // steps of every tile taken so far
    bool ok;
    StepCover(uint64_t full, uint32_t tile_elems, int groups, const std::vector<uint32_t>& tails)
        : n_full(full), full_shift(full_tile_shift(tile_elems, groups)) {
        for (uint64_t t = 0; t < full; ++t) tiles.push_back(TileDesc{nullptr, 0, tile_elems, 0, 0, 0});
        for (uint32_t n : tails) tiles.push_back(TileDesc{nullptr, 0, n, 0, 0, 0});
        index = index_tails(tiles.data() + full, tails.size());
    }
    uint64_t steps_of(uint64_t t) const {
        return t < n_full ? uint64_t(1) << full_shift : (tiles[t].len + kTailStep - 1) / kTailStep;
    }
    void reset() {
        ok = true;
        taken.assign(tiles.size(), {});
        for (uint64_t t = 0; t < taken.size(); ++t) taken[t].assign(steps_of(t), 0);
    }
    // the launch as launch_steps passes it to the kernels
    void launch(uint64_t first, uint64_t full, uint32_t step0, uint32_t grid) {
        const StepShape sh{full_shift, static_cast<uint32_t>(step0), n_full - first, index};
        for (uint64_t i = 0; i < grid; ++i) {
            const StepItem it = step_item(i, full, sh, tiles.data() + first);
            const uint64_t tile = first + it.tile;
            if (tile >= taken.size() || it.full != (tile < n_full) ||
                it.part >= taken[tile].size())
                ok = false;
            else
                ++taken[tile][it.part];
        }
    }
    bool once() const {
        bool good = ok;
        for (const auto& t : taken)
            for (uint8_t c : t) good &= c == 1;
        return good;
    }
};

void test_step_launches(std::mt19937_64& rng) {
    for (uint64_t n : {512ull, 1024ull, 512ull * 37}) {
        std::vector<uint8_t> seen(n, 0);
        bool ok = true;
        for (uint64_t i = 0; i < n; ++i) {
            const uint64_t j = xcd_run_item(i);
            ok &= j < n && !seen[j];
            if (j < n) seen[j] = 1;
        }
        check(ok, "step launches: the order over the XCDs is a permutation");
    }
    for (int trial = 0; trial < 300; ++trial) {
        const uint32_t tile = trial % 3 == 0 ? 8192 : 65536;
        const uint64_t n_full = trial % 5 == 0 ? 0 : rng() % 300;
        const uint64_t n_tail = trial % 7 == 0 ? 0 : rng() % (trial % 11 == 0 ? 70000 : 300);
        // tails of one length or of any, or short ones with longer ones among
        // them or at one end
        std::vector<uint32_t> tails;
        const int kind = trial % 6;
        const uint32_t same = 1 + rng() % tile;
        for (uint64_t t = 0; t < n_tail; ++t) {
            const bool longer = kind == 2 ? rng() % 50 == 0
                                : kind == 3 ? t + 1 == n_tail
                                : kind == 4 ? t == 0
                                            : t < n_tail / 2;
            tails.push_back(kind == 0   ? same
                            : kind == 1 ? 1 + rng() % tile
                            : longer    ? tile - rng() % 4096
                                        : 1 + rng() % 64);
        }
        StepCover c(n_full, tile, trial % 2 == 0 ? 2 : 4, tails);
        uint64_t needed = 0;
        for (uint64_t t = 0; t < c.tiles.size(); ++t) needed += c.steps_of(t);
        for (const uint64_t cap : {kMaxStepGrid, uint64_t(1000), uint64_t(16)}) {
            c.reset();
            uint64_t launches = 0, items = 0;
            for_step_launches(n_full, c.index.n_steps, c.full_shift,
                              [&](uint64_t first, uint64_t full, uint32_t step0, uint32_t grid) {
                                  check(grid > 0 && grid <= cap, "step launches: grid");
                                  c.launch(first, full, step0, grid);
                                  ++launches;
                                  items += grid;
                                  return ES_OK;
                              }, cap);
            check(c.once(), "step launches: every step once");
            check(items == needed, "step launches: no workgroup without a step");
            check(cap != kMaxStepGrid || launches <= 1, "step launches: one for a small plan");
            check(launches >= items / cap, "step launches: cut at the cap");
        }
    }
    // up to and beyond the card's memory: aligned plans, unaligned ones (all
    // tails) and the smallest tiles
    for (const uint64_t elems : {(uint64_t(1) << 36) - 1, uint64_t(1) << 36,
                                 (uint64_t(1) << 36) + 65536, uint64_t(1) << 37,
                                 uint64_t(160) << 30})
        for (const uint64_t tile : {8192ull, 65536ull})
            for (const int groups : {2, 4})
                for (const bool aligned : {true, false}) {
                    const uint64_t n_full = aligned ? elems / tile : 0;
                    const uint64_t n_steps = aligned ? 3 : (elems + kTailStep - 1) / kTailStep;
                    const uint32_t shift = full_tile_shift(tile, groups);
                    uint64_t f = 0, t = 0;
                    for_step_launches(
                        n_full, n_steps, shift,
                        [&](uint64_t first, uint64_t full, uint32_t step0, uint32_t grid) {
                            check(uint64_t(grid) * kStepThreads < (uint64_t(1) << 32),
                                  "step launches: below 2^32 lanes");
                            check(first == f && step0 == t, "step launches: in order");
                            const uint64_t tail_items = grid - (full << shift);
                            check(tail_items == 0 || f + full == n_full,
                                  "step launches: the full tiles first");
                            f += full;
                            t += tail_items;
                            return ES_OK;
                        });
                    check(f == n_full && t == n_steps, "step launches: every step");
                }
    // quantized plans up to the card's memory, with the fewest and the most codes
    // per workgroup: legal launches
    for (const uint64_t tile : {16384ull, 65536ull})
        for (const uint64_t codes : {uint64_t(5000), uint64_t(1) << 30, uint64_t(320) << 30}) {
            const uint64_t part = qsteps_per_workgroup(codes, tile, 256) * uint64_t(kQStepCodes);
            uint32_t shift = 0;
            while ((part << shift) < tile) ++shift;
            check(part << shift == tile, "step launches: a quantized tile's steps");
            for (const bool aligned : {true, false}) {
                const uint64_t n_full = aligned ? codes / tile : 0;
                const uint64_t n_steps = (codes - n_full * tile + part - 1) / part;
                uint64_t f = 0, t = 0;
                for_step_launches(n_full, n_steps, shift,
                                  [&](uint64_t first, uint64_t full, uint32_t step0,
                                      uint32_t grid) {
                                      check(uint64_t(grid) * kStepThreads < (uint64_t(1) << 32) &&
                                                first == f && step0 == t,
                                            "step launches: quantized");
                                      f += full;
                                      t += grid - (full << shift);
                                      return ES_OK;
                                  });
                check(f == n_full && t == n_steps, "step launches: every quantized step");
            }
        }
    // and their tails: every code beyond a tensor's full tiles in one step of the
    // entry that a lookup of the step finds (the last one not beyond it), none empty
    for (int trial = 0; trial < 60; ++trial) {
        const uint32_t n = 1 + rng() % 200;
        const uint64_t tile = trial % 2 ? 16384 : 65536, part = kQStepCodes << (rng() % 3);
        std::vector<esq::DevQTensor> tab(n + 1);
        uint64_t n_full = 0;
        for (uint32_t i = 0; i < n; ++i) {
            tab[i].numel = uint32_t(rng() % 5 == 0 ? 0 : rng() % (trial % 3 ? 400000 : 100));
            tab[i].first_full = n_full;
            n_full += rng() % 2 ? tab[i].numel / tile : 0;       // aligned or not
        }
        tab[n].first_full = n_full;
        index_qtails(tab.data(), n, tile, part);
        std::vector<uint64_t> next(n);
        for (uint32_t i = 0; i < n; ++i) next[i] = (tab[i + 1].first_full - tab[i].first_full) * tile;
        bool ok = true;
        for (uint32_t j = 0; j < tab[n].first_step; ++j) {
            uint32_t t = 0;
            for (uint32_t i = 0; i < n; ++i)
                if (tab[i].first_step <= j) t = i;
            const uint64_t full = (tab[t + 1].first_full - tab[t].first_full) * tile;
            const uint64_t e0 = full + (j - tab[t].first_step) * part;
            ok &= e0 == next[t] && e0 < tab[t].numel;
            next[t] = std::min<uint64_t>(e0 + part, tab[t].numel);
        }
        for (uint32_t i = 0; i < n; ++i) ok &= next[i] == tab[i].numel;
        check(ok, "step launches: quantized tails");
    }
}

// A quantized member's coefficient is finite for every sigma a call takes.
void test_qmember() {
    for (const float sigma : {1e-3f, 2.8e38f, 2.9e38f, std::numeric_limits<float>::max()})
        for (const int32_t sign : {1, -1}) {
            const float w = qmember(7, sign, sigma).w_k;
            const double exact = sign * double(sigma) * kSqrt2Ln2Double;
            check(std::isfinite(w) && (w > 0) == (sign > 0), "quantized member: finite");
            check(std::abs(exact) > 3.4e38 || std::abs(w - exact) <= std::abs(exact) * 0x1p-24,
                  "quantized member: coefficient");
        }
}

// Argument checks that must fail before any device access.
void test_validation() {
    const uint64_t seeds[3] = {1, 2, 3};
    const int32_t signs[3] = {1, -1, 1}, bad_signs[3] = {1, 0, 1};
    es_update_opts_t o{5e-4f, 1e-3f, 1e-8f, 0u, 0u};
    const float* fake = reinterpret_cast<const float*>(uintptr_t(0x1000));
    check(validate_update("t", seeds, signs, fake, 3, &o) == ES_OK, "validate: good call");
    check(validate_update("t", nullptr, signs, fake, 3, &o) == ES_ERR_INVALID_ARG, "validate: seeds");
    check(validate_update("t", seeds, bad_signs, fake, 3, &o) == ES_ERR_INVALID_ARG, "validate: signs");
    check(validate_update("t", seeds, signs, fake, 0, &o) == ES_ERR_INVALID_ARG, "validate: n = 0");
    check(validate_update("t", seeds, signs, fake, ES_MAX_MEMBERS + 1, &o) == ES_ERR_INVALID_ARG,
          "validate: n too large");
    es_update_opts_t bad = o;
    bad.flags = 64;
    check(validate_update("t", seeds, signs, fake, 3, &bad) == ES_ERR_INVALID_ARG, "validate: flags");
    bad = o;
    bad.alpha = NAN;
    check(validate_update("t", seeds, signs, fake, 3, &bad) == ES_ERR_INVALID_ARG, "validate: alpha");
    check(std::string(es_last_error()) == "t: alpha not finite", "validate: message");
    check(es_update(nullptr, seeds, signs, fake, 3, &o, nullptr, nullptr, nullptr) ==
              ES_ERR_INVALID_ARG, "es_update: null plan");
    check(es_update_noalloc(nullptr, seeds, signs, fake, 3, &o, nullptr, nullptr, nullptr) ==
              ES_ERR_INVALID_ARG, "es_update_noalloc: null plan");

    es_plan_t* plan = reinterpret_cast<es_plan_t*>(uintptr_t(0xdead));
    check(es_plan_create(nullptr, 1, &plan) == ES_ERR_INVALID_ARG && plan == nullptr,
          "plan create: null list");
    alignas(16) static uint16_t buf[64];
    es_tensor_t ts[3] = {{buf, 8, 0, 0}, {buf + 8, 8, 0, 0}, {buf + 16, 8, 2, 0}};
    check(es_plan_create(ts, 2, &plan) == ES_ERR_INVALID_ARG, "plan create: duplicate ids");
    ts[1].tensor_id = 1;
    ts[1].data = buf + 4;
    check(es_plan_create(ts, 2, &plan) == ES_ERR_INVALID_ARG, "plan create: overlap");
    ts[1].data = reinterpret_cast<uint8_t*>(buf + 20) + 1;
    check(es_plan_create(ts, 2, &plan) == ES_ERR_ALIGN, "plan create: odd address");
    ts[1].data = nullptr;
    check(es_plan_create(ts, 2, &plan) == ES_ERR_INVALID_ARG, "plan create: null data");
    ts[1].data = buf + 20;
    ts[1].numel = uint64_t(1) << 61;
    check(es_plan_create(ts, 2, &plan) == ES_ERR_INVALID_ARG, "plan create: too large");
    check(es_plan_create(ts, 0, &plan) == ES_ERR_INVALID_ARG, "plan create: no tensors");
    check(es_plan_create(ts, 1, nullptr) == ES_ERR_INVALID_ARG, "plan create: null output");

    alignas(16) static int8_t codes[64];
    alignas(4) static float scales[8];
    es_qtensor_t qt[2] = {{codes, scales, 16, 8, 0}, {codes + 16, scales, 16, 8, 0}};
    es_qplan_t* qp = nullptr;
    check(es_qplan_create(qt, 2, &qp) == ES_ERR_INVALID_ARG, "qplan create: duplicate ids");
    qt[1].tensor_id = 1;
    qt[1].row = 12;
    check(es_qplan_create(qt, 2, &qp) == ES_ERR_INVALID_ARG, "qplan create: row");
    qt[1].row = 8;
    qt[1].data = codes + 8;
    check(es_qplan_create(qt, 2, &qp) == ES_ERR_INVALID_ARG, "qplan create: overlap");
    qt[1].data = codes + 16;
    qt[1].scales = reinterpret_cast<const float*>(reinterpret_cast<const char*>(scales) + 2);
    check(es_qplan_create(qt, 2, &qp) == ES_ERR_ALIGN, "qplan create: scales alignment");
    qt[1].scales = scales;
    qt[1].numel = uint64_t(1) << 31;
    check(es_qplan_create(qt, 2, &qp) == ES_ERR_INVALID_ARG, "qplan create: numel");

    check(es_perturb(nullptr, 1, 1, 1e-3f, nullptr) == ES_ERR_INVALID_ARG, "perturb: null plan");
    check(es_swap(nullptr, 1, 1, 1e-3f, 2, 1, 1e-3f, nullptr) == ES_ERR_INVALID_ARG, "swap: null");
    check(es_zscore(nullptr, 4, 1e-8f, nullptr, nullptr, nullptr) == ES_ERR_INVALID_ARG, "zscore");
    check(es_hbm_calibrate(nullptr, 1 << 17, 1, nullptr, nullptr) == ES_ERR_INVALID_ARG,
          "calibrate: null");
    check(es_hbm_calibrate(buf, 1 << 17, 7, nullptr, nullptr) == ES_ERR_INVALID_ARG,
          "calibrate: mode");
    check(es_philox_words(1, 0, 0, 0, 4, nullptr, nullptr) == ES_ERR_INVALID_ARG, "words: null");
    check(es_normals(1, 0, 0, 4, nullptr, nullptr) == ES_ERR_INVALID_ARG, "normals: null");
    for (int code = -6; code <= 0; ++code) check(es_strerror(code) != nullptr, "strerror");

    check(std::isnan(es_sigma_cosine(1e-3, 1e-4, 5, 4)), "sigma: t > T");
    check(std::isnan(es_sigma_cosine(1e-3, 1e-4, 0, 0)), "sigma: T = 0");
    check(es_sigma_cosine(1e-3, 1e-4, 0, 100) == 1e-3, "sigma: t = 0");
    check(es_sigma_cosine(1e-3, 1e-4, 100, 100) == 1e-4, "sigma: t = T");
}

}  // namespace

int main() {
    std::mt19937_64 rng(20261202);
    test_member_tables(rng);
    test_tiling(rng);
    test_block_tiling(rng);
    test_row_divisor(rng);
    test_qblock_geometry(rng);
    test_step_launches(rng);
    test_qmember();
    test_validation();
    if (g_failures) {
        std::printf("%d failures\n", g_failures);
        return 1;
    }
    std::printf("ok\n");
    return 0;
}
