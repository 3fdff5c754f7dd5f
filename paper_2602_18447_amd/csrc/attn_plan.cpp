// Host side of the attention planner: the choice of the key-range pieces from a simulated schedule, the counts the
// launches need, and a host twin of the device list builder.  Plain C++ (no HIP), see attn_plan.h.
#include "attn_plan.h"

#include <algorithm>
#include <cmath>
#include <vector>

namespace cs {

void attn_plan_capacity(const AttnTune &tune, int64_t max_T, int64_t max_B, int G, int Hkv, int64_t *max_tiles,
                        int64_t *max_items) {
    int64_t tiles = (int64_t)Hkv * ((G * max_T + ATTN_BM - 1) / ATTN_BM + max_B);
    *max_tiles = tiles;
    *max_items = 3 * tiles + 4 * tune.target_items;     // candidates that need more are not considered
}

namespace {
struct UnitShape { int tiles, nc; };
struct Candidate { int cpi, equalize; };

UnitPlan shape_plan(const UnitShape &t, Candidate cd) {
    UnitPlan p;
    p.n_qt = t.tiles; p.nc_max = t.nc;       // n_qt holds Hkv * n_qt here (Hkv = 1 in the calls below)
    int n = t.nc > cd.cpi ? plan_ceil_div(t.nc, cd.cpi) : 1;
    bool clamped = n > ATTN_MAX_SPLIT;
    p.n_split = clamped ? ATTN_MAX_SPLIT : n;
    p.piece = (cd.equalize || clamped) ? plan_ceil_div(std::max(t.nc, 1), p.n_split) : cd.cpi;
    return p;
}

// The model of the planner: an item costs its chunks and a fixed part - filling the pipeline, loading q, writing the result (rows of the
// output, or fp32 partial results) - and a workgroup alone on its CU runs through its chunks, not its fixed part, 1.4 times as fast as one of
// two.  Units: the time a workgroup takes for one chunk while its CU holds two (about 2 us).  The constants are those with the smallest loss
// against the fastest of all candidates over 63 measured batches (1 - 128 traces, contexts to 16384, steps of 8 - 300 tokens, with and
// without shared contexts, 150 - 19000 tokens in all), all with 12 q heads on 2 kv heads: there a layer takes 0.4 % longer than with the best candidate on
// average, 3.4 % at worst, which says how well it fits and no more.  On 200 other batches (random ones of the same ranges on five head
// layouts, attention and little else in a layer) it is 3.0 % on average and 18 % at worst: 1.8 with 12/2 heads, 2.2 with 40/8, 2.6, 3.9 and 4.4 with 32/8, 16/8 and 8/8.  0.9 points of that are the
// choice of the loop; the rest is mostly tiles of few rows, whose keys no other tile reads: such a batch is bound by its stream of keys, and cutting 200 to 256
// of them in two gains nothing.  (6 and 8 chunk-times, all of an item 1.5 times as fast alone, 4 for the merge, longer pieces only: 4.2 and 41 % there; it left tiles
// whole that cover half the chip - 12 candidates on contexts of 1211 - 2890, 1317 tokens: 243 us a layer, 221 in pieces.)
constexpr float ITEM_OVERHEAD_WHOLE = 14.0f, ITEM_OVERHEAD_PIECE = 12.5f;

// Items, partial slots and the largest per-XCD item count of a candidate; lens (optional) receives the
// per-XCD items in dispatch order.  Same arithmetic as the list builder.
void candidate_counts(const std::vector<UnitShape> &tr, Candidate cd, int64_t n_tiles, int64_t work_total,
                      AttnPlanCounts *r, std::vector<AttnItemCost> *lens /* [8] */) {
    r->n_items = 0; r->n_part_slots = 0; r->max_xcd_items = 0;
    int tile_lo[9] = {0}, seg_base[9] = {0};
    int tile_base = 0, rest_base = 0;
    long long work_base = 0;
    std::vector<UnitPlan> plans;
    plans.reserve(tr.size());
    for (const UnitShape &t : tr) {
        UnitPlan p = shape_plan(t, cd);
        plans.push_back(p);
        plan_xcd_starts(p, 1, tile_base, rest_base, work_base, work_total, tile_lo, seg_base);
        r->n_items += (int64_t)t.tiles * p.n_split;
        if (p.n_split > 1) r->n_part_slots += (int64_t)t.tiles * p.n_split;
        tile_base += t.tiles; rest_base += t.tiles * (p.n_split - 1);
        work_base += (long long)t.tiles * t.nc;
    }
    tile_lo[8] = (int)n_tiles;
    seg_base[8] = (int)r->n_items;
    for (int x = 0; x < 8; ++x) r->max_xcd_items = std::max<int64_t>(r->max_xcd_items, seg_base[x + 1] - seg_base[x]);
    if (!lens) return;
    std::vector<AttnItemCost> rest_lens[8];
    for (int x = 0; x < 8; ++x) {
        lens[x].reserve((size_t)r->max_xcd_items);
        rest_lens[x].reserve((size_t)r->max_xcd_items);
    }
    int ti = 0;
    for (size_t i = 0; i < tr.size(); ++i)
        for (int j = 0; j < tr[i].tiles; ++j, ++ti) {
            int x = 7;
            while (x > 0 && tile_lo[x] > ti) --x;
            const UnitPlan &p = plans[i];
            const float ov = p.n_split > 1 ? ITEM_OVERHEAD_PIECE : ITEM_OVERHEAD_WHOLE;
            lens[x].push_back({(float)std::min(p.piece, p.nc_max), ov});
            for (int sp = 1; sp < p.n_split; ++sp)
                rest_lens[x].push_back({(float)std::max(0, std::min(p.piece, p.nc_max - sp * p.piece)), ov});
        }
    for (int x = 0; x < 8; ++x) lens[x].insert(lens[x].end(), rest_lens[x].begin(), rest_lens[x].end());
}

// Makespan of the item list of the busiest XCD.
double simulate(const std::vector<AttnItemCost> *lens, int slots, double enough) {
    int x_busy = 0;
    double most = -1;
    for (int x = 0; x < 8; ++x) {
        double w = 0;
        for (const AttnItemCost &c : lens[x]) w += c.chunks + c.fixed;
        if (w > most) { most = w; x_busy = x; }
    }
    return attn_plan_makespan(lens[x_busy].data(), (int64_t)lens[x_busy].size(), slots, enough);
}
}  // namespace

// In chunk-times (the time a workgroup takes for one chunk while its CU holds two workgroups).  An XCD has slots / 8 workgroup slots, two per
// CU; items are handed out in list order as slots free up.  A workgroup that has its CU to itself runs faster, which decides the value of a last
// round that does not fill the chip.  A makespan of enough or more is not followed to its end (two workgroups a CU get most done, so the work
// bounds it from below).
double attn_plan_makespan(const AttnItemCost *q, int64_t n, int slots, double enough) {
    constexpr double ALONE = 1.4;
    const int n_cu = std::max(1, slots / 16);
    double work = 0;
    for (int64_t i = 0; i < n; ++i) work += q[i].chunks + q[i].fixed;
    if (work / (2 * n_cu) >= enough) return 1e300;
    struct Cu { double rem[2], chunks[2], at; int busy; };         // remaining work (down to chunks it is the fixed part; < 0: empty) at time at
    std::vector<Cu> cus((size_t)n_cu, Cu{{-1.0, -1.0}, {0.0, 0.0}, 0.0, 0});
    std::vector<double> change((size_t)n_cu, 1e300);     // of a CU: an item done, or the fixed part of one that is alone
    int64_t next = 0;
    auto speed = [&](const Cu &c, int s) { return c.busy == 1 && c.rem[s] <= c.chunks[s] ? ALONE : 1.0; };
    auto take = [&](Cu &c) {
        const int s = c.rem[0] < 0 ? 0 : 1;
        c.chunks[s] = q[next].chunks;
        c.rem[s] = c.chunks[s] + q[next].fixed;
        ++c.busy;
        ++next;
    };
    auto schedule = [&](int i) {
        const Cu &c = cus[i];
        double t = 1e300;
        for (int s = 0; s < 2; ++s)
            if (c.rem[s] >= 0) t = std::min(t, c.at + (c.busy == 1 && c.rem[s] > c.chunks[s] ? c.rem[s] - c.chunks[s] : c.rem[s] / speed(c, s)));
        change[i] = t;
    };
    // Items are handed out in list order as slots free up, emptier CUs first (the dispatcher spreads workgroups over the CUs).
    for (int round = 0; round < 2; ++round)
        for (int i = 0; i < n_cu && next < n; ++i) take(cus[i]);
    for (int i = 0; i < n_cu; ++i) schedule(i);
    double now = 0.0;
    std::vector<int> freed;
    for (;;) {
        int i = 0;
        for (int k = 1; k < n_cu; ++k)
            if (change[k] < change[i]) i = k;
        if (change[i] == 1e300) break;
        if (change[i] >= enough) return 1e300;
        now = change[i];
        // What counts as no time: more than rounding leaves of the item whose end now is (some 1e-16 of now), or that item would stay
        // in its slot with a rest too short to move now, and the loop would not end (makespans from about 1e7 chunk-times on).
        const double none = std::max(1e-9, 1e-12 * now);
        freed.clear();
        for (int k = i; k < n_cu; ++k) {                 // (items of the same length end together)
            if (change[k] > now + none) continue;
            Cu &c = cus[k];
            const double step[2] = {(now - c.at) * speed(c, 0), (now - c.at) * speed(c, 1)};
            c.at = now;
            for (int s = 0; s < 2; ++s)
                if (c.rem[s] >= 0) {
                    const bool fixed = c.rem[s] > c.chunks[s];
                    c.rem[s] -= step[s];
                    if (fixed && std::abs(c.rem[s] - c.chunks[s]) < none) c.rem[s] = c.chunks[s];
                    if (c.rem[s] <= none) { c.rem[s] = -1.0; --c.busy; }
                }
            freed.push_back(k);
        }
        for (int busy = 0; busy < 2; ++busy)
            for (int k : freed)
                if (cus[k].busy == busy && next < n) take(cus[k]);
        for (int k : freed) schedule(k);
    }
    return now;
}

// Choice of the pieces: equal pieces with a split factor 1..4 of the average tile, or front-loaded pieces of the chunks' share of 480, 420,
// 360, 300 or 240 slots (fewer slots: less to merge, and room for the pieces that tiles of uneven length leave over); the
// candidate with the smallest simulated makespan plus the cost of its merge pass wins.  The merge pass is a launch plus the partial results it
// reads back, 64 KiB written and read per piece: measured 26 us for 1536 pieces and 90 us for about 4000 - 0.011 chunk-times per piece.
AttnPlanCounts attn_plan_counts(const AttnTune &tune, const int32_t *h_cu, const int32_t *h_plens, int B, int T,
                                const int32_t *h_group_start, int n_units, int G, int Hkv, int last_only, int64_t max_part_slots) {
    AttnPlanCounts r = {};
    if (!h_group_start || last_only) n_units = B;
    std::vector<UnitShape> tr;
    tr.reserve(n_units);
    int64_t total = 0, n_tiles = 0;
    int nc_longest = 0;
    for (int i = 0; i < n_units; ++i) {
        AttnUnit u = plan_unit(h_cu, h_plens, h_group_start, n_units, i, B, T, 1 << 30, last_only);
        UnitPlan p = unit_plan(u, G, 1 << 30, 1, last_only);
        tr.push_back({Hkv * p.n_qt, p.nc_max});
        total += (int64_t)Hkv * p.n_qt * p.nc_max;
        n_tiles += (int64_t)Hkv * p.n_qt;
        if (p.n_qt > 0) nc_longest = std::max(nc_longest, p.nc_max);
        r.part_rows = std::max(r.part_rows, last_only ? G : (int)std::min<int64_t>((int64_t)G * u.S_tot, ATTN_BM));
    }
    r.part_rows = std::min((r.part_rows + 31) / 32 * 32, ATTN_BM);
    r.n_tiles = n_tiles;
    r.total_chunks = total;
    double avg = n_tiles > 0 ? (double)total / (double)n_tiles : 1.0;
    int64_t slots = tune.target_items;
    int64_t cap_items = 3 * n_tiles + 4 * slots;
    std::vector<Candidate> cands;
    auto equal_cpi = [&](int sp) { return sp == 1 ? (1 << 30) : std::max<int>(tune.min_chunks, (int)((avg + sp - 1) / sp)); };
    auto front_cpi = [&](double f) { return std::max<int>(tune.min_chunks, (int)std::ceil(f * (double)total / (double)slots)); };
    if (tune.force_split >= 1 && tune.force_split <= 4) cands.push_back({equal_cpi(tune.force_split), 1});
    else if (tune.force_split == 5) cands.push_back({front_cpi(1.07), 0});
    else {
        for (int sp = 1; sp <= 4; ++sp) {
            if (sp > 1 && avg / sp < tune.min_chunks) break;
            cands.push_back({equal_cpi(sp), 1});
        }
        for (double f : {1.07, 1.22, 1.43, 1.71, 2.14})
            if (front_cpi(f) < nc_longest) cands.push_back({front_cpi(f), 0});
    }
    for (size_t i = 1; i < cands.size();) {              // (short lists: several clamp to min_chunks)
        const bool again = std::any_of(cands.begin(), cands.begin() + i, [&](const Candidate &c) { return c.cpi == cands[i].cpi && c.equalize == cands[i].equalize; });
        if (again) cands.erase(cands.begin() + i);
        else ++i;
    }
    double best = 1e300;
    Candidate pick = {1 << 30, 1};
    for (size_t i = 0; i < cands.size(); ++i) {
        AttnPlanCounts c = {};
        std::vector<AttnItemCost> lens[8];
        candidate_counts(tr, cands[i], n_tiles, total, &c, lens);
        if ((c.n_items > cap_items || c.n_part_slots > max_part_slots) && cands.size() > 1 && cands[i].cpi != (1 << 30)) continue;
        const double merge = c.n_part_slots > 0 ? 3.0 + 0.011 * (double)c.n_part_slots : 0.0;
        const double even = c.n_part_slots > 0 ? 1.01 : 1.0;     // (whole tiles where it makes no difference)
        const double est = even * (simulate(lens, (int)slots, best / even - merge) + merge);
        if (est < best) { best = est; pick = cands[i]; }
    }
    r.chunks_per_item = pick.cpi;
    r.equalize = pick.equalize;
    candidate_counts(tr, pick, n_tiles, total, &r, nullptr);
    return r;
}

void attn_plan_host(const int32_t *cu, const int32_t *plens, const int32_t *group_start, int n_units, int B, int T,
                    int max_L, int G, int Hkv, int cpi, int equalize, int last_only, int max_tiles, int max_items,
                    AttnTile *tiles, AttnItem *items, int32_t *counts) {
    if (!group_start || last_only) n_units = B;
    // pass 0 adds up the chunks (the XCD cuts depend on the total), pass 1 places the cuts, pass 2 writes the lists
    long long work_total = 0;
    int tile_lo[9] = {0}, seg_base[9] = {0};
    int total_tiles = 0, total_rest = 0;
    for (int pass = 0; pass < 3; ++pass) {
        int tile_base = 0, rest_base = 0, slot_base = 0;
        long long work_base = 0;
        for (int i = 0; i < n_units; ++i) {
            AttnUnit u = plan_unit(cu, plens, group_start, n_units, i, B, T, max_L, last_only);
            UnitPlan p = unit_plan(u, G, cpi, equalize, last_only);
            int my_tiles = Hkv * p.n_qt;
            if (pass == 1) plan_xcd_starts(p, Hkv, tile_base, rest_base, work_base, work_total, tile_lo, seg_base);
            if (pass == 2)
                plan_emit_unit(cu, T, u, G, Hkv, p, tile_base, rest_base, slot_base, tile_lo, seg_base, last_only, max_tiles,
                               max_items, tiles, items);
            tile_base += my_tiles;
            rest_base += my_tiles * (p.n_split - 1);
            slot_base += p.n_split > 1 ? my_tiles * p.n_split : 0;
            work_base += (long long)my_tiles * p.nc_max;
        }
        if (pass == 0) work_total = work_base;
        if (pass == 1) { tile_lo[8] = tile_base; seg_base[8] = tile_base + rest_base; }
        total_tiles = tile_base;
        total_rest = rest_base;
    }
    counts[0] = std::min(total_tiles, max_tiles);
    counts[1] = std::min(total_tiles + total_rest, max_items);
    for (int x = 0; x < 9; ++x) counts[2 + x] = std::min(seg_base[x], max_items);
}

}  // namespace cs
