// Host-and-device geometry of the tilings (Sec. 3.1 tiles of size B; Sec. 4.2 per-head shapes,
// Eq. 7): the per-head table the kernels read and the pure host arithmetic that fills it.
// Plain C++ with no HIP types, so that host tools and CPU tests can include it on its own.
#pragma once

#include <stdint.h>

#include <algorithm>
#include <array>
#include <vector>

namespace veda {

// Per-head geometry, one entry per head, in device memory (plan->d_heads).
//
// 128-token tiles are handled as two 64-slot halves: a tile of extents (ot,oh,ow) is cut across
// its slowest axis of extent > 1, so that slots 0-63 are one half and slots 64-127 the other, and
// the two halves are tiles 2o and 2o+1 of an "inner" geometry (grp = 2).  There pt,ph,pw are
// the extents of a half, (ht,hh,hw) the token offset of the second half inside the whole tile,
// and nt,nh,nw still count whole tiles.  For 64-token tiles grp = 1, (ot,oh,ow) = (pt,ph,pw)
// and the offsets are zero.
struct HeadGeom {
    int32_t pt, ph, pw;      // extents of one 64-slot tile (or half tile)
    int32_t nt, nh, nw;      // grid of whole tiles (ceil)
    int32_t n_tiles;         // number of 64-slot tiles: grp*nt*nh*nw
    int32_t tile_off;        // first global tile index of this head
    int64_t score_off;       // first score element of this head (per batch)
    int32_t score_blk_off;   // first 128x128 score block of this head
    int32_t score_blk_dim;   // ceil(n_tiles / 128)
    int32_t ot, oh, ow;      // extents of a whole tile
    int32_t ht, hh, hw;      // token offset of the second half inside a whole tile
    int32_t grp;             // 64-slot tiles per whole tile: 1 or 2
    // Partners are neighbours along pair_ax (0 = t, 1 = h, 2 = w: the axis along which a tile is thinnest, so
    // its neighbour is the closest one and keeps the most similar key tiles): the attention kernels take full query tiles two at a
    // time along it (attn_items; a last layer without a partner goes with the next lines'), and merged lists' work items
    // are partners or one without (pair_tiles).  pair_ax = 3: the two halves of a 128-token tile.
    int32_t pair_ax;
    int32_t n_pairs;         // merged lists' work items (pairs and partnerless tiles) of this head
    int32_t log_pw, log_phw; // log2 of pw and of ph*pw (extents multiply to 64, so each is a power of two)
};

// Extents and tile grid of one head: shape = (p_t,p_h,p_w) of a whole tile, grp = 1 or 2.
// Offsets (tile_off, score_*), pair_ax and n_pairs are left to the caller.
inline void head_extents(HeadGeom& g, const int32_t* shape, int grp, int T, int H, int W) {
    g.ot = shape[0]; g.oh = shape[1]; g.ow = shape[2];
    g.pt = g.ot; g.ph = g.oh; g.pw = g.ow;
    g.ht = g.hh = g.hw = 0;
    g.grp = grp;
    if (grp == 2) {   // cut across the slowest axis of extent > 1 (a product of 128: it is even)
        if (g.ot > 1) { g.pt = g.ot / 2; g.ht = g.pt; }
        else if (g.oh > 1) { g.ph = g.oh / 2; g.hh = g.ph; }
        else { g.pw = g.ow / 2; g.hw = g.pw; }
    }
    for (g.log_pw = 0; (1 << g.log_pw) < g.pw; ++g.log_pw) {}
    for (g.log_phw = g.log_pw; (1 << g.log_phw) < g.ph * g.pw; ++g.log_phw) {}
    g.nt = (T + g.ot - 1) / g.ot;
    g.nh = (H + g.oh - 1) / g.oh;
    g.nw = (W + g.ow - 1) / g.ow;
    g.n_tiles = (int32_t)((int64_t)grp * g.nt * g.nh * g.nw);
}

// Anchor token of 64-slot tile i: the token of its slot 0, from which a kernel finds the tile's
// rows in token order.  Every whole tile starts inside the grid, so its slot 0 is a real token;
// the second half of a 128-token tile may lie wholly outside a ragged grid (no real slot at
// all): such a half is anchored at the first half's token instead, so that the address formed
// from the anchor always stays inside the tensor (the rows fetched for it are masked anyway).
inline int32_t tile_anchor_token(const HeadGeom& g, int32_t i, int T, int H, int W) {
    const int o = g.grp == 2 ? i >> 1 : i, half = g.grp == 2 ? (i & 1) : 0;
    const int tw = o % g.nw, th = (o / g.nw) % g.nh, tt = o / (g.nw * g.nh);
    int64_t t = (int64_t)tt * g.ot + half * g.ht, h = (int64_t)th * g.oh + half * g.hh,
            w = (int64_t)tw * g.ow + half * g.hw;
    if (t >= T || h >= H || w >= W) { t -= half * g.ht; h -= half * g.hh; w -= half * g.hw; }
    return (int32_t)((t * H + h) * W + w);
}

// The tables below are those of 64-slot tiles: a plan of whole 128-token tiles has none, its halves' plan has them.
inline bool slots_64(const HeadGeom& g) { return (int64_t)g.pt * g.ph * g.pw == 64; }

// Real slots of 64-slot tile i: bit l is set if slot l lies inside the grid.
inline uint64_t tile_real_slots(const HeadGeom& g, int32_t i, int T, int H, int W) {
    const int o = g.grp == 2 ? i >> 1 : i, half = g.grp == 2 ? (i & 1) : 0;
    const int tw = o % g.nw, th = (o / g.nw) % g.nh, tt = o / (g.nw * g.nh);
    auto inside = [](int first, int extent, int size) { return std::max(0, std::min(extent, size - first)); };
    const int rt = inside(tt * g.ot + half * g.ht, g.pt, T), rh = inside(th * g.oh + half * g.hh, g.ph, H),
              rw = inside(tw * g.ow + half * g.hw, g.pw, W);
    if (rt == g.pt && rh == g.ph && rw == g.pw) return ~0ull;
    uint64_t mask = 0;
    for (int t = 0; rw > 0 && t < rt; ++t)
        for (int h = 0; h < rh; ++h) mask |= (rw == 64 ? ~0ull : (1ull << rw) - 1ull) << ((t * g.ph + h) * g.pw);
    return mask;
}

// Whether two heads' tiles are the same ones.
inline bool same_tiles(const HeadGeom& a, const HeadGeom& b) {
    return a.ot == b.ot && a.oh == b.oh && a.ow == b.ow && a.grp == b.grp && a.pair_ax == b.pair_ax;
}

// That of every tile, heads in order.
inline std::vector<uint64_t> tile_real_table(const std::vector<HeadGeom>& heads, int T, int H, int W) {
    std::vector<uint64_t> real;
    if (!slots_64(heads[0])) return real;
    for (size_t h = 0; h < heads.size(); ++h) {
        const HeadGeom& g = heads[h];
        const size_t at = real.size();
        real.resize(at + g.n_tiles);
        if (h > 0 && same_tiles(g, heads[h - 1])) std::copy(real.begin() + (at - g.n_tiles), real.begin() + at, real.begin() + at);
        else for (int32_t i = 0; i < g.n_tiles; ++i) real[at + i] = tile_real_slots(g, i, T, H, W);
    }
    return real;
}

// What a workgroup of the attention kernels (four wavefronts of 32 query rows) computes: up to four query tiles of one
// head, visited together.  A tile with more than 32 real rows takes two wavefronts, a thin one at a ragged edge of the
// grid (32 rows or fewer: its second wavefront would have none) takes one, so four thin tiles share a workgroup where two full
// ones do.  Built once per plan: which tiles share depends on the geometry alone.
struct AttnItem {
    int32_t head;      // -1: nothing to do (a die with fewer items than others)
    int32_t n_tiles;   // 1..4
    int32_t tile[4];   // head-local query tiles; places beyond n_tiles repeat the first
    uint32_t waves;    // byte w: wavefront w's place in tile[] | kItemSecond | kItemIdle
    int32_t partners;  // bit 0: the tiles in places 0 and 1 are partners that take one form of products (fp32), bit 1: those in 2 and 3
};
constexpr uint32_t kItemSecond = 4u;   // rows 32-63 of its tile, not 0-31
constexpr uint32_t kItemIdle = 8u;     // no rows

// How many full tiles, or thin ones, share a workgroup.  The more do, the fewer key tiles are loaded and the more steps a
// workgroup's walk has (1.1-1.3 times a list's length for two full tiles, 1.3-2.0 for four thin ones).
struct AttnShare {
    int full, thin;
    bool partners = false;   // tiles stay with their partners along pair_ax (pair_tiles), whatever else shares their workgroup
};

// Appends head h's items: those of more than two tiles, which have the most steps, before the others, each kind ordered by
// its first tile.  Returns the number of the former.  Full tiles are paired along pair_ax (line by line; the odd ones out
// with those of the next lines), thin ones taken four at a time by 2x2x2 blocks of the tile grid, so that tiles that share a
// workgroup are neighbours, whose kept lists agree most.  At most two items of a head have wavefronts to spare (more where partners
// stay together: a thin tile with a full one, or a pair of thin ones left over).
inline size_t attn_items_of_head(const HeadGeom& g, int32_t h, int T, int H, int W, AttnShare share, std::vector<AttnItem>& items) {
    const size_t first = items.size();
    auto add = [&](const int32_t* tiles, int n, int full, int partners = 0) {   // the first `full` of them take two wavefronts
        AttnItem it = {h, n, {0, 0, 0, 0}, 0u, partners};
        for (int t = 0; t < 4; ++t) it.tile[t] = tiles[t < n ? t : 0];
        // which of a tile's wavefronts comes first alternates: the second one of an edge tile has less to do, and is then
        // not on the same SIMD in every workgroup
        uint32_t place[4] = {kItemIdle, kItemIdle, kItemIdle, kItemIdle};
        int w = 0;
        const uint32_t flip = (items.size() - first) & 1;
        for (int t = 0; t < n; ++t) {
            if (t < full) {
                place[w++] = (uint32_t)t | (flip ? kItemSecond : 0u);
                place[w++] = (uint32_t)t | (flip ? 0u : kItemSecond);
            } else {
                place[w++] = (uint32_t)t;
            }
        }
        for (w = 0; w < 4; ++w) it.waves |= place[w] << (8 * w);
        items.push_back(it);
    };
    if (g.pair_ax == 3) {   // the two halves of a 128-token tile keep one list between them
        for (int32_t o = 0; o < g.n_tiles / 2; ++o) {
            const int32_t both[2] = {2 * o, 2 * o + 1};
            add(both, 2, 2);
        }
        return 0;
    }
    const int cnt[3] = {g.nt, g.nh, g.nw}, stride[3] = {g.nh * g.nw, g.nw, 1}, ax = g.pair_ax;
    std::vector<int32_t> odd, thin;
    std::vector<std::array<int32_t, 2>> thin_pairs;   // partners, both thin
    auto is_thin = [&](int32_t t) { return __builtin_popcountll(tile_real_slots(g, t, T, H, W)) <= 32; };
    for (int32_t i = 0; i < g.n_tiles; ++i) {
        if (i / stride[ax] % cnt[ax] != 0) continue;
        if (share.partners) {
            for (int c = 0; c < cnt[ax]; c += 2) {
                const int32_t pair[2] = {i + c * stride[ax], i + (c + 1) * stride[ax]};
                if (c + 1 == cnt[ax]) (is_thin(pair[0]) ? thin : odd).push_back(pair[0]);
                else if (is_thin(pair[0]) && is_thin(pair[1])) thin_pairs.push_back({pair[0], pair[1]});
                else add(pair, 2, 2, 1);
            }
            continue;
        }
        int32_t held = -1;
        for (int c = 0; c < cnt[ax]; ++c) {
            const int32_t t = i + c * stride[ax];
            if (is_thin(t)) {
                thin.push_back(t);
            } else if (share.full == 1) {
                add(&t, 1, 1);
            } else if (held < 0) {
                held = t;
            } else {
                const int32_t pair[2] = {held, t};
                add(pair, 2, 2);
                held = -1;
            }
        }
        if (held >= 0) odd.push_back(held);
    }
    for (size_t i = 0; i + 1 < odd.size(); i += 2) add(&odd[i], 2, 2);
    auto block = [&](int32_t i) {
        const int64_t w = i % g.nw, hh = i / g.nw % g.nh, t = i / (g.nw * g.nh);
        return ((((t / 2) * g.nh + hh / 2) * g.nw + w / 2) * 2 + t % 2) * 4 + hh % 2 * 2 + w % 2;
    };
    std::sort(thin.begin(), thin.end(), [&](int32_t a, int32_t b) { return block(a) < block(b); });
    std::sort(thin_pairs.begin(), thin_pairs.end(), [&](const auto& a, const auto& b) { return block(a[0]) < block(b[0]); });
    for (size_t i = 0, n; i < thin_pairs.size(); i += n) {
        n = share.thin == 4 && i + 1 < thin_pairs.size() ? 2 : 1;
        add(thin_pairs[i].data(), (int)(2 * n), 0, n == 2 ? 3 : 1);   // pairs lie one behind the other
    }
    if (odd.size() % 2) {   // a last full tile takes along what would not fill a workgroup
        int32_t tiles[3] = {odd.back(), 0, 0};
        int n = 1;
        for (size_t over = share.thin == 4 && thin.size() % 4 < 3 ? thin.size() % 4 : 0; over > 0; --over) {
            tiles[n++] = thin.back();
            thin.pop_back();
        }
        add(tiles, n, 1);
    }
    for (size_t i = 0; i < thin.size(); i += share.thin) add(&thin[i], (int)std::min<size_t>(share.thin, thin.size() - i), 0);
    std::sort(items.begin() + first, items.end(), [](const AttnItem& a, const AttnItem& b) {
        return (a.n_tiles > 2) != (b.n_tiles > 2) ? a.n_tiles > 2 : a.tile[0] < b.tile[0];
    });
    return (size_t)std::count_if(items.begin() + first, items.end(), [](const AttnItem& a) { return a.n_tiles > 2; });
}

// Shares of n items for each die.  Those that n leaves over go to the first dies, of the items dealt from the last die on to the last; in
// calls of few workgroups to the dies with the fewest so far: to the same ones for every head they left one die twice the others' work.
// Whole calls: 36 heads of 9 tiles, d = 128, fp32, one tile kept 75.7 -> 64.6 us, five kept 116.5 -> 90.3, bf16 55.2 -> 49.2.  (In calls of many
// workgroups nothing to gain, and what dies share of the heads in progress changes: 8 heads of 624 in fp32 5 % slower.)
inline std::vector<size_t> die_shares(size_t n, const std::vector<std::vector<AttnItem>>& per, bool from_last, bool few) {
    std::vector<size_t> order(per.size()), share(per.size(), n / per.size());
    for (size_t x = 0; x < order.size(); ++x) order[x] = from_last ? order.size() - 1 - x : x;
    if (few) std::stable_sort(order.begin(), order.end(), [&](size_t a, size_t b) { return per[a].size() < per[b].size(); });
    for (size_t i = 0; i < n % per.size(); ++i) ++share[order[i]];
    return share;
}

// The launch table: workgroup i runs on die i % dies, and die x takes the x-th part of every head's items of either kind, heads
// in order (all dies then work on the same head at the same time, whose K and V stay in the memory-side cache, and the
// workgroups that share an L2 hold neighbouring query tiles).  Dies with fewer items end with empty ones.
inline std::vector<AttnItem> attn_items(const std::vector<HeadGeom>& heads, int T, int H, int W, int dies, AttnShare sharing) {
    std::vector<std::vector<AttnItem>> per(dies);
    std::vector<AttnItem> items;
    size_t most = 0, many = 0;
    if (!slots_64(heads[0])) return items;
    for (size_t h = 0; h < heads.size(); ++h) {
        if (h > 0 && same_tiles(heads[h], heads[h - 1])) {
            for (AttnItem& it : items) it.head = (int32_t)h;
        } else {
            items.clear();
            many = attn_items_of_head(heads[h], (int32_t)h, T, H, W, sharing, items);
        }
        const size_t n[2] = {many, items.size() - many};
        size_t at = 0;
        for (int kind = 0; kind < 2; ++kind) {
            const std::vector<size_t> shares = die_shares(n[kind], per, kind == 0, sharing.thin != 4);
            for (int i = 0; i < dies; ++i) {
                const int x = kind ? i : dies - 1 - i;
                per[x].insert(per[x].end(), items.begin() + at, items.begin() + at + shares[x]);
                at += shares[x];
                most = std::max(most, per[x].size());
            }
        }
    }
    const AttnItem none = {-1, 0, {0, 0, 0, 0}, 0u, 0};
    std::vector<AttnItem> table(most * dies, none);
    for (int x = 0; x < dies; ++x)
        for (size_t i = 0; i < per[x].size(); ++i) {
            AttnItem it = per[x][i];
            // Workgroups 32 apart on a die tend to share a compute unit: where two wavefronts or fewer have rows they are not
            // the same ones, so not on the same SIMDs, in both.
            int live = 0;
            for (int w = 0; w < 4; ++w) live += (it.waves >> (8 * w) & kItemIdle) == 0u;
            const uint32_t turn = live <= 2 ? (uint32_t)(i / 32 * live % 4) * 8u : 0u;
            if (turn) it.waves = it.waves << turn | it.waves >> (32u - turn);
            table[i * dies + x] = it;
        }
    return table;
}

// What a workgroup of the target scores computes where all query tiles are asked for: consecutive query tiles of one head, as
// many as have 128 real rows between them (four wavefronts of 32, packed: a wavefront may hold rows of several tiles).
constexpr int kHeatTiles = 8;   // at most
struct HeatItem {
    int32_t head, first, n;   // n = 0: nothing to do (a die with fewer items than others)
};
inline std::vector<HeatItem> heat_items(const std::vector<HeadGeom>& heads, int T, int H, int W, int dies, int most_tiles) {
    std::vector<std::vector<HeatItem>> per(dies);
    std::vector<HeatItem> items;
    size_t most = 0;
    if (!slots_64(heads[0])) return items;
    for (size_t h = 0; h < heads.size(); ++h) {
        const HeadGeom& g = heads[h];
        const bool same = h > 0 && same_tiles(g, heads[h - 1]);
        if (!same) items.clear();
        int rows = 0;
        for (int32_t i = 0; i < g.n_tiles && !same; ++i) {
            const int more = __builtin_popcountll(tile_real_slots(g, i, T, H, W));
            const bool fits = g.grp == 2 ? i % 2 == 1 : rows + more <= 128 && !items.empty() && items.back().n < most_tiles;
            if (fits) {
                ++items.back().n;
                rows += more;
            } else {
                items.push_back({0, i, 1});
                rows = more;
            }
        }
        for (HeatItem& it : items) it.head = (int32_t)h;
        const size_t n = items.size();
        size_t at = 0;
        for (int x = 0; x < dies; ++x) {
            const size_t share = n / dies + ((size_t)x < n % dies ? 1 : 0);
            per[x].insert(per[x].end(), items.begin() + at, items.begin() + at + share);
            at += share;
            most = std::max(most, per[x].size());
        }
    }
    std::vector<HeatItem> table(most * dies, HeatItem{0, 0, 0});
    for (int x = 0; x < dies; ++x)
        for (size_t i = 0; i < per[x].size(); ++i) table[i * dies + x] = per[x][i];
    return table;
}

// Work split of the target scores over a list of n query tiles, in any order: entries of one head, the next in
// the list, share a workgroup: two full tiles, four thin ones (32 real rows or fewer), or a last full one and two thin ones;
// workgroup p takes the p-th such item, head by head.  Items are formed inside windows of
// kListWindow entries, so that a workgroup's look at the list is bounded (a longer list loses at most one partner per
// head and window).  A window of m entries has at most one partnerless entry per head, hence this many workgroups
// at most (those past the last item have nothing to do).
constexpr int kListWindow = 4096;
// f full and t thin entries of a head make no more items than pairs.
constexpr int list_items(int f, int t) { return (f + 1) / 2 + ((f & 1) ? (t > 2 ? (t + 1) / 4 : 0) : (t + 3) / 4); }
constexpr int64_t list_window_blocks(int64_t m, int heads) { return (m + (heads < m ? heads : m)) / 2; }
constexpr int64_t list_blocks(int64_t n, int heads) {
    return n / kListWindow * list_window_blocks(kListWindow, heads) + list_window_blocks(n % kListWindow, heads);
}

}  // namespace veda
