// Host-side checker, meant to be built with AddressSanitizer and UBSan (no GPU needed): drives the attention
// planner (attn_plan.h / attn_plan.cpp) and the library's host arithmetic that sizes and carves device memory
// (workspace layout, split-K planes, validators, through the C ABI) over the five benchmark shapes and a few
// thousand seeded random batches, and checks the properties whose violation would become an out-of-bounds access
// on the device: every index in range, every key range covered exactly once, slices disjoint.
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <sstream>
#include <string>
#include <utility>
#include <vector>

#include "../../include/confspec.h"
#include "../../include/confspec_ops.h"
#include "../../include/confspec_static.h"
#include "attn_plan.h"
#include "kernels.h"

static int g_fail = 0;
#define CHECK(cond, ...)                                                         \
    do {                                                                         \
        if (!(cond)) {                                                           \
            if (++g_fail <= 20) { printf("FAIL %s:%d %s  ", __FILE__, __LINE__, #cond); printf(__VA_ARGS__); printf("\n"); } \
        }                                                                        \
    } while (0)

struct Batch {
    std::vector<int32_t> cu, plens, groups;   // groups empty = every trace on its own
    int B() const { return (int)plens.size(); }
    int T() const { return cu.back(); }
};

// One plan (all rows or last rows) of one batch: counts from the host planner, lists from the host twin of the
// device builder, then the invariants.
static void check_plan(const cs::AttnTune &tune, const Batch &b, int G, int Hkv, int last_only, const char *what) {
    const int B = b.B(), T = b.T();
    const int32_t *gs = b.groups.empty() ? nullptr : b.groups.data();
    const int n_units = b.groups.empty() ? B : (int)b.groups.size() - 1;
    cs::AttnPlanCounts pc = cs::attn_plan_counts(tune, b.cu.data(), b.plens.data(), B, T, gs, n_units, G, Hkv, last_only);
    int64_t cap_tiles = 0, cap_items = 0;
    cs::attn_plan_capacity(tune, T, B, G, Hkv, &cap_tiles, &cap_items);
    // the planner's own choice always fits the workspace bound; a forced split factor may not (the pass then refuses
    // the call with CONFSPEC_E_WORKSPACE before anything is launched)
    CHECK(pc.n_tiles <= cap_tiles && (pc.n_items <= cap_items || tune.force_split != 0),
          "%s: plan %lld tiles %lld items exceeds capacity %lld / %lld", what, (long long)pc.n_tiles, (long long)pc.n_items,
          (long long)cap_tiles, (long long)cap_items);
    // a limit on the partial results is kept, and changes nothing where the plan keeps it already
    for (int64_t limit : {(int64_t)0, pc.n_part_slots / 2, pc.n_part_slots}) {
        const cs::AttnPlanCounts lc = cs::attn_plan_counts(tune, b.cu.data(), b.plens.data(), B, T, gs, n_units, G, Hkv, last_only, limit);
        CHECK((lc.n_part_slots <= limit || tune.force_split != 0) && (limit < pc.n_part_slots || (lc.chunks_per_item == pc.chunks_per_item && lc.equalize == pc.equalize)),
              "%s: %lld partial slots with a limit of %lld, %lld without", what, (long long)lc.n_part_slots, (long long)limit, (long long)pc.n_part_slots);
    }
    // exact-size arrays with guard entries behind them: a write past the counted size is an ASan error
    std::vector<cs::AttnTile> tiles((size_t)std::max<int64_t>(pc.n_tiles, 1));
    std::vector<cs::AttnItem> items((size_t)std::max<int64_t>(pc.n_items, 1));
    for (auto &it : items) it.tile = -7;
    int32_t counts[11];
    int max_L = 0;
    for (int v : b.plens) max_L = std::max(max_L, v);
    cs::attn_plan_host(b.cu.data(), b.plens.data(), gs, n_units, B, T, max_L, G, Hkv, pc.chunks_per_item, pc.equalize, last_only,
                       (int)pc.n_tiles, (int)pc.n_items, tiles.data(), items.data(), counts);
    CHECK(counts[0] == pc.n_tiles && counts[1] == pc.n_items, "%s: builder wrote %d tiles %d items, planner counted %lld / %lld", what,
          counts[0], counts[1], (long long)pc.n_tiles, (long long)pc.n_items);
    CHECK(counts[2] == 0 && counts[10] == pc.n_items, "%s: XCD ranges do not span the item list", what);
    int64_t max_seg = 0;
    for (int x = 0; x < 8; ++x) {
        CHECK(counts[2 + x] <= counts[3 + x], "%s: XCD %d range is negative", what, x);
        max_seg = std::max<int64_t>(max_seg, counts[3 + x] - counts[2 + x]);
    }
    CHECK(max_seg == pc.max_xcd_items, "%s: largest XCD range %lld, planner said %lld", what, (long long)max_seg, (long long)pc.max_xcd_items);
    // per tile: pieces cover [0, nc) exactly once, in order of part slots; indices in range
    std::vector<std::vector<std::pair<int, int>>> cover((size_t)pc.n_tiles);
    std::vector<char> slot_used((size_t)std::max<int64_t>(pc.n_part_slots, 1), 0);
    for (int64_t i = 0; i < pc.n_items; ++i) {
        const cs::AttnItem &it = items[(size_t)i];
        CHECK(it.tile >= 0 && it.tile < pc.n_tiles, "%s: item %lld never written or tile %d out of range", what, (long long)i, it.tile);
        if (it.tile < 0 || it.tile >= pc.n_tiles) continue;
        const cs::AttnTile &t = tiles[(size_t)it.tile];
        CHECK(it.b0 == t.b0 && it.c == t.c && it.row0 == t.row0 && it.b_end == t.b_end, "%s: item / tile mismatch", what);
        CHECK(it.b0 >= 0 && it.b0 < it.b_end && it.b_end <= B && it.c >= 0 && it.c < Hkv, "%s: unit [%d, %d) head %d", what, it.b0, it.b_end, it.c);
        int rows = G * (b.cu[it.b_end] - b.cu[it.b0]);
        CHECK(it.row0 >= 0 && it.row0 < rows, "%s: row0 %d of %d rows", what, it.row0, rows);
        CHECK(it.chunk_begin >= 0 && it.chunk_begin <= it.chunk_end, "%s: chunk range [%d, %d)", what, it.chunk_begin, it.chunk_end);
        if (t.n_splits > 1) {
            CHECK(it.part_slot >= t.part_base && it.part_slot < t.part_base + t.n_splits && it.part_slot < pc.n_part_slots,
                  "%s: part slot %d (base %d, %d pieces, %lld slots)", what, it.part_slot, t.part_base, t.n_splits, (long long)pc.n_part_slots);
            if (it.part_slot >= 0 && it.part_slot < pc.n_part_slots) {
                CHECK(!slot_used[(size_t)it.part_slot], "%s: part slot %d used twice", what, it.part_slot);
                slot_used[(size_t)it.part_slot] = 1;
            }
        } else {
            CHECK(it.part_slot == -1, "%s: unsplit tile with part slot %d", what, it.part_slot);
        }
        cover[(size_t)it.tile].push_back({it.chunk_begin, it.chunk_end});
    }
    for (int64_t ti = 0; ti < pc.n_tiles; ++ti) {
        const cs::AttnTile &t = tiles[(size_t)ti];
        auto &cv = cover[(size_t)ti];
        CHECK((int)cv.size() == t.n_splits, "%s: tile %lld has %zu items, %d pieces", what, (long long)ti, cv.size(), t.n_splits);
        std::sort(cv.begin(), cv.end());
        // the chunks this tile must see, computed here from the definition
        int L = b.plens[t.b0], S_tot = b.cu[t.b_end] - b.cu[t.b0];
        int n_pc = (L + 63) / 64, need;
        if (last_only) {
            need = n_pc + (S_tot + 63) / 64;
            CHECK(t.b_end == t.b0 + 1 && t.row0 == (S_tot - 1) * G, "%s: last-row tile of trace %d at row %d", what, t.b0, t.row0);
        } else {
            int r_last = std::min(t.row0 + 127, G * S_tot - 1);
            int tok_lo = b.cu[t.b0] + t.row0 / G, tok_hi = b.cu[t.b0] + r_last / G;
            int tr = t.b0;
            while (b.cu[tr + 1] <= tok_lo) ++tr;          // trace of the tile's first row
            need = n_pc + (tok_hi - b.cu[tr] + 1 + 63) / 64;
            CHECK(t.row0 % 128 == 0, "%s: tile row0 %d", what, t.row0);
        }
        int at = 0;
        for (auto &p : cv) {
            CHECK(p.first == at || p.first == p.second, "%s: tile %lld pieces leave a gap or overlap at chunk %d (next piece [%d, %d))", what,
                  (long long)ti, at, p.first, p.second);
            if (p.second > p.first) at = p.second;
        }
        CHECK(at == need, "%s: tile %lld covered up to chunk %d, needs %d", what, (long long)ti, at, need);
    }
    // every row of every unit belongs to exactly one tile per kv head
    if (!last_only) {
        int64_t rows_total = 0, rows_tiled = 0;
        for (int u = 0; u < n_units; ++u) {
            int b0 = gs ? gs[u] : u, b1 = gs ? gs[u + 1] : u + 1;
            rows_total += (int64_t)Hkv * G * (b.cu[b1] - b.cu[b0]);
        }
        for (auto &t : tiles)
            if (pc.n_tiles > 0) rows_tiled += std::min(128, G * (b.cu[t.b_end] - b.cu[t.b0]) - t.row0);
        CHECK(rows_total == rows_tiled, "%s: %lld rows, %lld in tiles", what, (long long)rows_total, (long long)rows_tiled);
    }
}

// The schedule of attn_plan_makespan from its definition: every slot moved at every event.
static double plain_makespan(const std::vector<cs::AttnItemCost> &q, int n_cu) {
    struct Slot { double fixed = 0, chunks = 0; bool busy = false; };
    std::vector<Slot> sl(2 * (size_t)n_cu);
    size_t next = 0;
    double now = 0;
    for (;;) {
        for (int busy = 0; busy < 2; ++busy)                                // emptier CUs first
            for (int c = 0; c < n_cu; ++c)
                while (next < q.size() && sl[2 * c].busy + sl[2 * c + 1].busy <= busy) {
                    Slot &s = sl[2 * c + (sl[2 * c].busy ? 1 : 0)];
                    s.fixed = q[next].fixed;
                    s.chunks = q[next++].chunks;
                    s.busy = true;
                }
        double dt = 1e300;
        for (int c = 0; c < n_cu; ++c) {
            const double speed = sl[2 * c].busy + sl[2 * c + 1].busy == 1 ? 1.4 : 1.0;
            for (int i = 0; i < 2; ++i)
                if (const Slot &s = sl[2 * c + i]; s.busy) dt = std::min(dt, s.fixed > 0 ? s.fixed : s.chunks / speed);
        }
        if (dt == 1e300) return now;
        now += dt;
        for (int c = 0; c < n_cu; ++c) {
            const double speed = sl[2 * c].busy + sl[2 * c + 1].busy == 1 ? 1.4 : 1.0;
            for (int i = 0; i < 2; ++i) {
                Slot &s = sl[2 * c + i];
                if (!s.busy) continue;
                (s.fixed > 0 ? s.fixed : s.chunks) -= s.fixed > 0 ? dt : dt * speed;
                if (s.fixed > 0 && s.fixed < 1e-9) s.fixed = 0;
                if (s.fixed == 0 && s.chunks < 1e-9) s.busy = false;
            }
        }
    }
}

static Batch uniform_batch(int B, int L, int S) {
    Batch b;
    b.cu.push_back(0);
    for (int i = 0; i < B; ++i) { b.plens.push_back(L); b.cu.push_back(b.cu.back() + S); }
    return b;
}

static void check_library(const confspec_model_cfg &cfg, const Batch &b, const char *what) {
    confspec_ctx *ctx = nullptr;
    int rc = confspec_create(&cfg, 0, &ctx);
    CHECK(rc == CONFSPEC_OK && ctx, "%s: create rc %d", what, rc);
    if (!ctx) return;
    size_t ws = 0, need = 0;
    CHECK(confspec_workspace_bytes(ctx, b.T(), b.B(), 0, &ws) == CONFSPEC_OK && ws % 256 == 0 && ws > 0, "%s: workspace %zu", what, ws);
    // the device pointers are never dereferenced by the calls below; any non-null value passes the null checks
    const int32_t *dev = reinterpret_cast<const int32_t *>(uintptr_t(0x1000));
    confspec_batch cb = {b.B(), b.T(), dev, dev, dev, b.cu.data(), b.plens.data()};
    CHECK(confspec_static_scratch_need(ctx, &cb, &need) == CONFSPEC_OK && need % 256 == 0 && need <= ws,
          "%s: exact layout %zu vs bound %zu", what, need, ws);
    // slices of both layouts: aligned, inside the total, disjoint
    for (int exact = 0; exact < 2; ++exact) {
        size_t off[64], len[64];
        int32_t n = 64;
        size_t total = 0;
        rc = confspec_op_workspace_slices(ctx, b.T(), b.B(), exact ? &cb : nullptr, off, len, &n, &total);
        CHECK(rc == CONFSPEC_OK && n > 10 && n <= 64, "%s: slices rc %d n %d", what, rc, n);
        if (rc != CONFSPEC_OK) continue;
        CHECK(total == (exact ? need : ws), "%s: slices total %zu", what, total);
        std::vector<std::pair<size_t, size_t>> v;
        for (int i = 0; i < n; ++i) {
            CHECK(off[i] % 256 == 0 && off[i] + len[i] <= total, "%s: slice %d [%zu, +%zu) of %zu", what, i, off[i], len[i], total);
            if (len[i]) v.push_back({off[i], len[i]});
        }
        std::sort(v.begin(), v.end());
        for (size_t i = 1; i < v.size(); ++i)
            CHECK(v[i - 1].first + v[i - 1].second <= v[i].first, "%s: slices overlap at %zu", what, v[i].first);
        // the slices of passes over few rows: inside the total, clear of each other, and behind every slice that such passes
        // share with the others (those in front of the attention plan, of which the last is the activations' slice)
        size_t few_off[16], few_len[16], from = 0;
        const int n_few = confspec_few_row_slices(ctx, b.T(), b.B(), exact ? &cb : nullptr, few_off, few_len, &from, &total);
        CHECK(n_few == 0 || n_few == 8, "%s: %d few-row slices", what, n_few);
        CHECK((n_few > 0) == (cfg.dtype == CONFSPEC_DTYPE_BF16 && cfg.n_layers > 0 && cfg.n_q_heads / cfg.n_kv_heads <= cs::FEW_MAX_G &&
                              (!exact || b.T() <= cs::SK_MAX_ROWS)), "%s: %d few-row slices", what, n_few);
        std::vector<std::pair<size_t, size_t>> f;
        for (int i = 0; i < n_few; ++i) {
            CHECK(few_off[i] % 256 == 0 && few_off[i] >= from && few_off[i] + few_len[i] <= total, "%s: few-row slice %d [%zu, +%zu)", what, i, few_off[i],
                  few_len[i]);
            if (few_len[i]) f.push_back({few_off[i], few_len[i]});
        }
        std::sort(f.begin(), f.end());
        for (size_t i = 1; i < f.size(); ++i)
            CHECK(f[i - 1].first + f[i - 1].second <= f[i].first, "%s: few-row slices overlap at %zu", what, f[i].first);
        for (int i = 0, before = 0; n_few && i < n; ++i) {
            before += off[i] + len[i] <= from;
            CHECK(off[i] >= from || off[i] + len[i] <= from, "%s: slice %d crosses %zu", what, i, from);
            if (i == n - 1) CHECK(before == 16, "%s: %d slices in front of the few-row ones", what, before);
        }
    }
    // split-K planes: the bytes asked for are a whole number (2..64) of [M, N] fp32 planes, or none
    const int qw = cfg.n_q_heads * cfg.head_dim, kw = cfg.n_kv_heads * cfg.head_dim;
    const int shapes[4][2] = {{qw + 2 * kw, cfg.d_model}, {cfg.d_model, qw}, {2 * cfg.d_ffn, cfg.d_model}, {cfg.d_model, cfg.d_ffn}};
    for (int M : {1, 7, b.B(), 128, 129, 300, b.T()})
        for (auto &s : shapes)
            for (int terms = 1; terms <= 3; ++terms) {
                size_t bytes = confspec_op_gemm_scratch_bytes(ctx, M, s[0], s[1], terms);
                size_t plane = (size_t)M * s[0] * 4;
                CHECK(bytes % plane == 0 && (bytes == 0 || (bytes / plane >= 2 && bytes / plane <= 64)), "%s: split-K bytes %zu for M %d N %d K %d", what,
                      bytes, M, s[0], s[1]);
            }
    // validators: malformed batches are rejected before anything else is touched
    std::vector<int32_t> bad_cu = b.cu;
    bad_cu[1] = bad_cu[0];                                   // an empty suffix
    confspec_batch bad = cb;
    bad.h_cu_suffix = bad_cu.data();
    CHECK(confspec_static_scratch_need(ctx, &bad, &need) == CONFSPEC_E_OUT_OF_RANGE, "%s: empty suffix accepted", what);
    bad = cb;
    bad.T = b.T() + 1;
    CHECK(confspec_static_scratch_need(ctx, &bad, &need) == CONFSPEC_E_OUT_OF_RANGE, "%s: wrong T accepted", what);
    confspec_destroy(ctx);
}

// The planner on measured batches (profiles/attention_plans_of_random_batches.txt says how they are written): its pick's time against
// the best plan with either loop, per head layout and in all.
static int replay(const char *path) {
    FILE *f = fopen(path, "r");
    if (!f) { printf("cannot open %s\n", path); return 1; }
    std::vector<std::pair<std::string, std::vector<double>>> losses = {{"all", {}}};
    std::string line;
    for (int c; (c = fgetc(f)) != EOF;) {
        if (c != '\n') { line += (char)c; continue; }
        if (line.empty() || line[0] == '#') { line.clear(); continue; }
        std::istringstream in(line);
        line.clear();
        int hq, hkv, group;
        std::string word;
        in >> hq >> hkv >> group >> word;
        Batch b;
        b.cu.push_back(0);
        while (in >> word && word != "|") {
            int L = 0, S = 0, n = 1;
            if (sscanf(word.c_str(), "%d:%d*%d", &L, &S, &n) < 2) return 1;
            for (; n > 0; --n) { b.plens.push_back(L); b.cu.push_back(b.cu.back() + S); }
        }
        double t[2][9], best = 1e300;
        for (auto &loop : t) {
            for (double &v : loop) { in >> v; best = std::min(best, v); }
            in >> word;
        }
        for (int i = 0; group > 1 && i <= b.B(); i += group) b.groups.push_back(i);
        const cs::AttnTune tune;
        const int G = hq / hkv, n_units = group > 1 ? b.B() / group : b.B();
        auto plan = [&](const cs::AttnTune &tn) {
            return cs::attn_plan_counts(tn, b.cu.data(), b.plens.data(), b.B(), b.T(), group > 1 ? b.groups.data() : nullptr, n_units, G, hkv, 0);
        };
        const cs::AttnPlanCounts pick = plan(tune);
        int found = -1;
        for (int k = 0; k < 9 && found < 0; ++k) {
            cs::AttnTune forced = tune;
            const int shares[5] = {512, 449, 383, 320, 256};       // (pieces of 1.07 times the chunks' share of these)
            forced.force_split = std::min(k + 1, 5);
            if (k >= 4) forced.target_items = shares[k - 4];
            const cs::AttnPlanCounts p = plan(forced);
            if (p.n_items == pick.n_items && (p.chunks_per_item == pick.chunks_per_item || p.n_part_slots == 0)) found = k;
        }
        CHECK(found >= 0, "%d/%d, %d traces: the pick of %lld items, %d chunks each, was not measured", hq, hkv, b.B(), (long long)pick.n_items, pick.chunks_per_item);
        if (found < 0) continue;
        const double loss = t[pick.total_chunks / pick.n_items < cs::ATTN_STAGED_BELOW ? 0 : 1][found] / best - 1;
        const std::string layout = std::to_string(hq) + "/" + std::to_string(hkv);
        losses[0].second.push_back(loss);
        if (losses.back().first != layout) losses.push_back({layout, {}});
        losses.back().second.push_back(loss);
    }
    fclose(f);
    for (auto &[name, v] : losses) {
        double sum = 0;
        for (double x : v) sum += x;
        printf("%s: %zu batches, mean loss %.4f, worst %.4f\n", name.c_str(), v.size(), sum / (double)v.size(), *std::max_element(v.begin(), v.end()));
    }
    return g_fail ? 1 : 0;
}

int main(int argc, char **argv) {
    if (argc > 1) return replay(argv[1]);
    cs::AttnTune tune;
    const confspec_model_cfg draft = {28, 1536, 12, 2, 128, 8960, 151936, 1e6f, 1e-6f, CONFSPEC_DTYPE_BF16};
    const confspec_model_cfg target = {64, 5120, 40, 8, 128, 27648, 152064, 1e6f, 1e-6f, CONFSPEC_DTYPE_BF16};
    // the benchmark shapes
    struct Named { const char *name; Batch b; int G, Hkv; const confspec_model_cfg *cfg; };
    std::vector<Named> named;
    named.push_back({"config 2", uniform_batch(32, 2048, 96), 6, 2, &draft});
    named.push_back({"config 3", uniform_batch(64, 8192, 128), 6, 2, &draft});
    {
        std::mt19937 rng(1004);
        Batch b;
        b.cu.push_back(0);
        for (int i = 0; i < 128; ++i) {
            b.plens.push_back(512 + (int)(rng() % (16384 - 512 + 1)));
            b.cu.push_back(b.cu.back() + 32 + (int)(rng() % 225));
        }
        named.push_back({"config 4 (same ranges)", b, 6, 2, &draft});
    }
    named.push_back({"config 5", uniform_batch(16, 4096, 96), 5, 8, &target});
    named.push_back({"one-token batch", uniform_batch(32, 2048, 1), 6, 2, &draft});
    for (auto &nb : named) {
        check_plan(tune, nb.b, nb.G, nb.Hkv, 0, nb.name);
        check_plan(tune, nb.b, nb.G, nb.Hkv, 1, nb.name);
        check_library(*nb.cfg, nb.b, nb.name);
    }
    // seeded random batches: head groupings, lengths on and around page / chunk / tile borders, shared-context groups,
    // every planner setting
    std::mt19937 rng(20260218);
    const int special[] = {0, 1, 15, 16, 17, 63, 64, 65, 127, 128, 129, 255, 256, 257, 1023, 1024, 4095, 4096, 16384};
    const int heads[][2] = {{6, 2}, {1, 8}, {5, 8}, {2, 2}, {12, 1}, {4, 4}, {3, 3}};
    for (int iter = 0; iter < 4000; ++iter) {
        Batch b;
        int B = 1 + (int)(rng() % (iter % 50 == 0 ? 300 : 24));
        b.cu.push_back(0);
        for (int i = 0; i < B; ++i) {
            int L = (rng() & 1) ? special[rng() % 19] : (int)(rng() % 3000);
            int S = (rng() % 5 == 0) ? 1 : 1 + (int)(rng() % 300);
            b.plens.push_back(L);
            b.cu.push_back(b.cu.back() + S);
        }
        if (iter % 3 == 0) {          // groups of consecutive traces with one context length
            b.groups.push_back(0);
            while (b.groups.back() < B) {
                int w = 1 + (int)(rng() % 5);
                int lo = b.groups.back(), hi = std::min(B, lo + w);
                for (int i = lo + 1; i < hi; ++i) b.plens[i] = b.plens[lo];
                b.groups.push_back(hi);
            }
        }
        const int *h = heads[rng() % 7];
        cs::AttnTune t = tune;
        t.force_split = (int)(rng() % 6);
        t.min_chunks = 1 + (int)(rng() % 8);
        t.target_items = 64 << (rng() % 5);
        char what[64];
        snprintf(what, sizeof what, "random batch %d", iter);
        check_plan(t, b, h[0], h[1], 0, what);
        check_plan(t, b, h[0], h[1], 1, what);
        if (iter % 200 == 0) check_library(draft, b, what);
    }
    // the planner's schedule against the plain one, and its early end: with a bound it says the makespan, or that it is not below the bound
    for (int iter = 0; iter < 3000; ++iter) {
        const int slots = 16 << (rng() % 6), n = 1 + (int)(rng() % (iter % 4 ? 3 * (slots / 8) : 400)), kinds = 1 + (int)(rng() % 6);
        float len[6];
        for (float &l : len) l = (float)(rng() % (iter % 3 ? 60 : 400));
        std::vector<cs::AttnItemCost> q;
        for (int i = 0; i < n; ++i) q.push_back({iter % 2 ? (float)(rng() % 100) : len[rng() % kinds], rng() % 3 ? 12.5f : 14.0f});
        if (iter % 5 == 0) std::sort(q.begin(), q.end(), [](const auto &a, const auto &b) { return a.chunks > b.chunks; });
        const double want = plain_makespan(q, std::max(1, slots / 16)), got = cs::attn_plan_makespan(q.data(), n, slots, 1e300);
        CHECK(std::abs(got - want) <= 1e-6 * want, "schedule %d: %d items on %d slots take %.9g, plain %.9g", iter, n, slots, got, want);
        for (double f : {0.3, 0.99, 1.0, 1.01, 2.0}) {
            const double e = cs::attn_plan_makespan(q.data(), n, slots, f * got);
            CHECK(f > 1 ? e == got : e == 1e300, "schedule %d: bound of %.9g, makespan %.9g, result %.9g", iter, f * got, got, e);
        }
    }
    // tiling of the few-row projections: a kernel for it, the rows covered, tiles that divide the columns, every k-tile in
    // exactly one slice, no more cut tiles than there are arrival counters, planes sized for the slices and growing with the rows
    for (int iter = 0; iter < 60000; ++iter) {
        int epi = iter % 3, K = 64 * (1 + (int)(rng() % 600)), n_ct = 1 + (int)(rng() % (iter % 2 ? 12000 : 300)), M = 1 + (int)(rng() % 128);
        if (iter < 24) {
            const int shapes[8][2] = {{1536, 128}, {1536, 96}, {1536, 1120}, {8960, 96}, {5120, 448}, {5120, 320}, {5120, 3456}, {27648, 320}};
            K = shapes[iter / 3][0]; n_ct = shapes[iter / 3][1];
        }
        const cs::SkinnyPlan p = cs::skinny_plan(epi, M, K, n_ct);
        const int nk = K / 64;
        bool ok = cs::skinny_has_kernel(epi, p) && p.mb >= 1 && p.ms >= 1 && p.mb * p.ms * 16 >= M && (p.ms - 1) * p.mb * 16 < M && p.ct >= 1 &&
                  n_ct % p.ct == 0 && p.S >= 1 && p.S <= nk && (p.S == 1 || (epi == cs::SK_EPI_RESID && n_ct / p.ct * p.ms <= 256));
        int covered = 0;
        for (int sl = 0; ok && sl < p.S; ++sl) {
            int k0 = (int)((long)sl * nk / p.S), k1 = (int)((long)(sl + 1) * nk / p.S);
            ok = k1 > k0 && k0 == covered;
            covered = k1;
        }
        ok = ok && covered == nk;
        size_t pb = cs::skinny_plane_bytes(epi, M, K, n_ct);
        ok = ok && pb >= (p.S > 1 ? (size_t)p.S * 16 * p.mb * p.ms * n_ct * 16 * 4 : 0) && pb <= cs::skinny_plane_bytes(epi, 128, K, n_ct);
        if (!ok && ++g_fail <= 20)
            printf("skinny_plan(epi=%d, M=%d, K=%d, n_ct=%d) -> mb=%d ms=%d ct=%d S=%d planes=%zu\n", epi, M, K, n_ct, p.mb, p.ms, p.ct, p.S, pb);
    }
    // pieces of the few-row attention: the whole context covered, and a partial result for every workgroup of a tile that
    // has several pieces
    for (int iter = 0; iter < 20000; ++iter) {
        const bool one = iter & 1;
        cs::FewAttn a = {};
        a.n_tiles = 1 + (int)(rng() % (iter % 3 ? 300 : 20));
        a.Hkv = 1 + (int)(rng() % 8);
        a.max_L = (int)(rng() % (iter % 5 ? 5000 : 140000));
        cs::few_attn_pieces(a, one);
        const int of_context = a.pieces - (one || a.fold ? 0 : 1);
        CHECK(a.wave_pages >= 1 && of_context >= 1 && (int64_t)of_context * a.wave_pages * 8 * 16 >= a.max_L &&
              (a.pieces == 1 || (int64_t)a.n_tiles * a.Hkv * a.pieces <= cs::FEW_RECORDS),
              "few_attn_pieces(n_tiles=%d, Hkv=%d, max_L=%d, one=%d) -> pieces=%d wave_pages=%d fold=%d", a.n_tiles, a.Hkv, a.max_L, one,
              a.pieces, a.wave_pages, a.fold);
    }
    // split-K planes of a projection: a pass of fewer rows never asks for more than the workspace laid out for more rows holds
    for (int iter = 0; iter < 20000; ++iter) {
        const cs::GemmTune g{};
        const int N = 32 * (1 + (int)(rng() % (iter % 2 ? 1800 : 200))), K = 64 * (1 + (int)(rng() % 500));
        const int max_M = 1 + (int)(rng() % (iter % 3 ? 2200 : 20000)), M = 1 + (int)(rng() % max_M);
        CHECK(cs::gemm_splitk_bytes(g, M, N, K) <= cs::gemm_splitk_max_bytes(g, max_M, N, K) &&
              (size_t)cs::gemm_splitk_factor(g, M, N, K) * M * N * 4 <= std::max((size_t)M * N * 4, cs::gemm_splitk_bytes(g, M, N, K)),
              "split-K planes of M=%d, N=%d, K=%d exceed those of up to %d rows", M, N, K, max_M);
    }
    // few k-tiles: at most 32 rows are cut into shorter slices than a whole tile row is
    for (int M : {1, 31, 32, 33, 128})
        for (int max_M : {M, 128, 129, 2000})
            for (int N : {128, 512, 1536, 24576})
                for (int nk = 1; nk <= 16; ++nk)
                    for (int short_tile : {0, 1}) {
                        cs::GemmTune g{};
                        g.short_tile = short_tile;
                        CHECK(M > max_M || cs::gemm_splitk_bytes(g, M, N, nk * 64) <= cs::gemm_splitk_max_bytes(g, max_M, N, nk * 64),
                              "split-K planes of M=%d, N=%d, K=%d exceed those of up to %d rows (short_tile %d)", M, N, nk * 64, max_M, short_tile);
                    }
    // launch-shape settings reach every tile: a band height that is set is taken, and "never split" changes nothing else
    for (int iter = 0; iter < 20000; ++iter) {
        cs::GemmTune g{}, never{};
        never.splitk = 1;
        g.group_m = 1 + (int)(rng() % 100);
        const int tm = 1 + (int)(rng() % 80), tn = 1 + (int)(rng() % 200);
        CHECK(cs::gemm_band_rows(g, 64, 128, 73728, tm, tn) == std::min(g.group_m, tm), "group_m %d of %d tile rows is not taken", g.group_m, tm);
        const int M = 1 + (int)(rng() % 12000), N = 128 * (1 + (int)(rng() % 300)), K = 64 * (1 + (int)(rng() % 500)), epi = (int)(rng() % 4);
        const cs::GemmPlan a = cs::gemm_plan(never, M, N, K, epi, false, true), b = cs::gemm_plan(cs::GemmTune{}, M, N, K, epi, false, false);
        CHECK(a.splits == 1 && b.splits == 1 && a.feed == b.feed, "never split: M=%d, N=%d, K=%d, epilogue %d on feed tile %d, without scratch on %d", M, N, K, epi,
              a.feed, b.feed);
    }
    // the GPU tests of gemm_feed_kernel reach every tile, whole and in slices, with these shapes (tests/test_gpu_gemm_feed.py)
    struct Whole { int M, N, K, feed, feed_swiglu; };
    for (const Whole &w : {Whole{33, 128, 64, 1, 2}, {64, 256, 128, 1, 2}, {65, 384, 192, 1, 2}, {129, 512, 832, 1, 2}, {255, 2048, 320, 1, 2}, {1290, 2048, 128, 3, 3},
                           {2040, 2048, 448, 3, 3}, {1921, 2048, 192, 3, 3}, {2600, 2048, 576, 4, 4}, {257, 4096, 1024, 2, 2}, {200, 17920, 448, 4, 4}, {7937, 1536, 576, 5, 0},
                           {10753, 1536, 192, 0, 0}, {18606, 1536, 320, 0, 0}, {1, 128, 64, 0, 0}, {8, 33024, 320, 0, 0}, {32, 32768, 192, 0, 0}})
        for (int epi : {cs::EPI_STORE_F32, cs::EPI_RESID_F32, cs::EPI_SWIGLU})
            for (int terms : {1, 2}) {
                const cs::GemmPlan p = cs::gemm_plan(cs::GemmTune{}, w.M, w.N, w.K * terms, epi, false, false);
                CHECK(p.splits == 1 && p.feed == (epi == cs::EPI_SWIGLU ? w.feed_swiglu : w.feed), "M=%d, N=%d, K=%d, epilogue %d: feed tile %d, %d slices", w.M, w.N,
                      w.K * terms, epi, p.feed, p.splits);
            }
    struct Cut { int epi, M, N, K, feed, splits; };   // epi -1: store, residual and SwiGLU
    for (const Cut &c : {Cut{-1, 33, 256, 1664, 1, 6}, {-1, 65, 3072, 2432, 2, 5}, {-1, 66, 3072, 2944, 3, 8}, {-1, 641, 3072, 2816, 4, 3}, {-1, 769, 3072, 4224, 5, 4},
                         {cs::EPI_ROPE, 74, 2048, 512, 1, 1}, {cs::EPI_ROPE, 257, 2048, 512, 1, 1}, {cs::EPI_ROPE, 2041, 2048, 512, 3, 1}, {cs::EPI_ROPE, 2600, 2048, 512, 4, 1},
                         {cs::EPI_ROPE, 641, 1536, 768, 2, 1}, {cs::EPI_ROPE, 65, 1536, 1792, 1, 5}, {cs::EPI_ROPE, 65, 3072, 2816, 2, 5}, {cs::EPI_ROPE, 66, 3072, 3328, 3, 9},
                         {cs::EPI_ROPE, 641, 3072, 2816, 4, 3}, {cs::EPI_ROPE, 769, 3072, 4096, 5, 4}})
        for (int epi : {cs::EPI_STORE_F32, cs::EPI_RESID_F32, cs::EPI_SWIGLU, cs::EPI_ROPE})
            if (c.epi < 0 ? epi != cs::EPI_ROPE : epi == c.epi) {
                const cs::GemmPlan p = cs::gemm_plan(cs::GemmTune{}, c.M, c.N, c.K, epi, false, true);
                CHECK(p.feed == c.feed && p.splits == c.splits, "M=%d, N=%d, K=%d, epilogue %d: feed tile %d, %d slices",
                      c.M, c.N, c.K, epi, p.feed, p.splits);
            }
    for (const auto &[d, F] : {std::pair{2048, 6144}, {2176, 6144}, {4224, 4096}, {6144, 16384}})
        for (int M : {100, 768, 769})
            CHECK(cs::gemm_plan(cs::GemmTune{}, M, d, F, cs::EPI_RESID_F32, true, true).splits > 1, "down projection %d x %d x %d is not cut", M, d, F);
    if (g_fail) { printf("host_check: %d check(s) failed\n", g_fail); return 1; }
    printf("host_check: ok\n");
    return 0;
}
