// Runs the repack and the kernels that write the prefill FFN's tables on the CPU
// (hip/hip_runtime.h here) over exactly sized buffers, for residency maps with and without shared slots, and
// checks what the FFN kernels will read: the groups, their items and the gathered rows.
#include "../../paper_2608_21614_amd/csrc/repack.hip"
#include "../../paper_2608_21614_amd/csrc/ffn.hip"

using namespace saem;

#define CHECK(cond, ...)                                     \
    do {                                                     \
        if (!(cond)) {                                       \
            printf("%s:%d: %s: ", __FILE__, __LINE__, #cond); \
            printf(__VA_ARGS__);                             \
            printf("\n");                                    \
            exit(1);                                         \
        }                                                    \
    } while (0)

static std::mt19937 rng(7);
static int pick(int lo, int hi) { return std::uniform_int_distribution<int>(lo, hi)(rng); }

struct Case {
    Shape s;
    int resident;  // experts with a slot in range (more than slots: some share one)
    int dropped;   // pairs whose id is outside [0, E)
};

// A heap array of exactly n elements (AddressSanitizer guards its ends), filled with v.
template <typename T>
static std::unique_ptr<T[]> filled(size_t n, T v) {
    std::unique_ptr<T[]> p(new T[n]);
    std::fill(p.get(), p.get() + n, v);
    return p;
}

static int shapes_seen[kFShapes];  // fp32: phases that took each item shape

static void run(const Case& c) {
    const Shape& s = c.s;
    const int P = s.T * s.k, H = s.H;
    printf("T %d H %d E %d F %d k %d S %d Fs %d slots %d %s, %d resident, %d dropped\n", s.T, H, s.E, s.F, s.k, s.S, s.Fs,
           s.slots, s.bf16 ? "bf16" : "f32", c.resident, c.dropped);

    // ids: distinct experts per token; slots: the first ones distinct, then shared
    auto ids = filled<int32_t>(P, 0);
    std::vector<int> e_all(s.E);
    for (int e = 0; e < s.E; ++e) e_all[e] = e;
    for (int t = 0; t < s.T; ++t) {
        std::shuffle(e_all.begin(), e_all.end(), rng);
        for (int j = 0; j < s.k; ++j) ids[t * s.k + j] = e_all[j];
    }
    for (int i = 0; i < c.dropped; ++i) ids[pick(0, P - 1)] = i % 2 ? -1 : s.E + i;
    auto slot = filled<int32_t>(s.E, -1);
    std::shuffle(e_all.begin(), e_all.end(), rng);
    for (int i = 0; i < c.resident; ++i) slot[e_all[i]] = i < s.slots ? i : pick(0, s.slots - 1);

    // x[t][h] names its element, so that a gathered piece can be told
    const size_t elt = s.bf16 ? 2 : 4;
    auto x = filled<uint8_t>((size_t)s.T * H * elt, 0);
    for (size_t i = 0; i < (size_t)s.T * H; ++i) {
        if (s.bf16) reinterpret_cast<uint16_t*>(x.get())[i] = (uint16_t)(1 + i % 65535);
        else reinterpret_cast<uint32_t*>(x.get())[i] = (uint32_t)(1 + i);
    }
    auto gate = filled<float>(P, 0.f);
    for (int q = 0; q < P; ++q) gate[q] = (float)q;

    // repack, with the offloaded rows, against a plain stable sort
    auto counts = filled<int32_t>(s.E, -9), seg = filled<int32_t>(s.E, -9), perm = filled<int32_t>(P, -9);
    auto inv = filled<int32_t>(P, -9), nres = filled<int32_t>(1, -9);
    auto off_rows = filled<uint8_t>((size_t)P * H * elt, 0xEE);
    auto off_w = filled<float>(P, -1.f);
    launch_repack(s, ids.get(), slot.get(), counts.get(), seg.get(), perm.get(), inv.get(), nres.get(), x.get(), gate.get(),
                  off_rows.get(), off_w.get(), nullptr);
    std::vector<int> order, want_counts(s.E, 0), want_seg(s.E, 0);
    int want_nres = 0;
    for (int pass = 0; pass < 2; ++pass) {
        for (int e = 0; e < s.E; ++e) {
            if (is_resident(slot[e], s.slots) != (pass == 0)) continue;
            want_seg[e] = (int)order.size();
            for (int q = 0; q < P; ++q)
                if (ids[q] == e) order.push_back(q);
            want_counts[e] = (int)order.size() - want_seg[e];
        }
        if (pass == 0) want_nres = (int)order.size();
    }
    CHECK(nres[0] == want_nres, "%d, not %d", nres[0], want_nres);
    for (int e = 0; e < s.E; ++e) CHECK(counts[e] == want_counts[e] && seg[e] == want_seg[e], "expert %d", e);
    for (int p = 0; p < P; ++p) CHECK(perm[p] == (p < (int)order.size() ? order[p] : -1), "packed row %d", p);
    for (int q = 0; q < P; ++q) CHECK(ids[q] >= 0 && ids[q] < s.E ? perm[inv[q]] == q : inv[q] == -1, "pair %d", q);
    const std::vector<uint8_t> untouched(H * elt, 0xEE);
    auto check_off = [&]() {
        for (int i = 0; i < P; ++i) {
            const bool row = want_nres + i < (int)order.size();  // else left as it was
            CHECK(off_w[i] == (row ? gate[order[want_nres + i]] : -1.f), "offloaded gate %d", i);
            const uint8_t* want = row ? x.get() + (size_t)(order[want_nres + i] / s.k) * H * elt : untouched.data();
            CHECK(memcmp(off_rows.get() + (size_t)i * H * elt, want, H * elt) == 0, "offloaded row %d", i);
        }
    };
    check_off();
    if (s.T <= 64) return;

    // the prefill FFN's preparation, on buffers of the workspace's sizes
    std::fill(off_rows.get(), off_rows.get() + (size_t)P * H * elt, 0xEE);
    std::fill(off_w.get(), off_w.get() + P, -1.f);
    const size_t meta_bytes = ffn_tile_meta_bytes(s);
    if (!s.bf16) CHECK(meta_bytes <= (size_t)s.T * s.E * 4, "the scores' room holds the tables");
    auto meta = filled<int32_t>(meta_bytes / 4, 0x5A5A5A5A), claim = filled<int32_t>(ffn_tile_claim_bytes(s) / 4, 77);
    auto xg = filled<uint16_t>((size_t)ffn_gather_rows(s) * H, 0xDEAD);
    FfnArgs a;
    a.x = x.get(); a.perm = perm.get(); a.counts = counts.get(); a.seg_start = seg.get(); a.expert_slot = slot.get();
    a.xg = xg.get(); a.tmeta = meta.get(); a.tclaim = claim.get();
    a.w13 = a.w2 = a.ws13 = a.ws2 = x.get();  // only addresses are taken
    a.Fa = max(s.F, s.Fs);
    a.ks = 1;
    a.topk_w = gate.get(); a.n_res = nres.get(); a.off_rows = off_rows.get(); a.off_w = off_w.get();
    launch_ffn_prepare(s, a, nullptr);
    check_off();
    for (int i = 0; i < 16; ++i) CHECK(claim[i * kTClaimPitch] == 0, "claim counter %d", i);

    // the active resident experts that can run: at most one per slot and pair
    const int max_routed = max_routed_groups(s), max_groups = max_routed + s.S;
    std::vector<int> active;
    for (int e = 0; e < s.E; ++e)
        if (is_resident(slot[e], s.slots) && counts[e] > 0 && (int)active.size() < max_routed) active.push_back(e);
    const int ng = (int)active.size() + s.S;
    const TileGroup* groups = reinterpret_cast<const TileGroup*>(meta.get() + kTHeader);
    const TileItem* tab = reinterpret_cast<const TileItem*>(groups + max_groups);
    const int32_t* pre = reinterpret_cast<const int32_t*>(groups + max_groups);
    if (!s.bf16) CHECK(meta[2] == ng, "%d groups, not %d", meta[2], ng);

    // row blocks of the gathered copy and of the activations, in the active list's order
    std::vector<int> blk(active.size() + 1, 0);
    for (size_t i = 0; i < active.size(); ++i) blk[i + 1] = blk[i] + (counts[active[i]] + 15) / 16;
    const int rb = blk.back(), tb16 = (s.T + 15) / 16;

    std::vector<int> seen(ng, 0), group_rows(max_groups, 0), group_fg(max_groups, 0);
    for (int o = 0; o < ng; ++o) {
        const TileGroup& g = groups[o];
        int which = -1;
        if (g.wsel < 0) {
            const int sh = -g.wsel - 1;
            CHECK(sh < s.S && g.count == s.T && g.rowbase == P + sh * s.T, "shared group %d", o);
            if (s.bf16) CHECK(g.blk == rb + sh * tb16, "shared group %d", o);
            which = (int)active.size() + sh;
        } else {
            for (size_t i = 0; i < active.size(); ++i)
                if (seg[active[i]] == g.rowbase && counts[active[i]] == g.count) which = (int)i;
            CHECK(which >= 0 && g.wsel == slot[active[which]], "group %d: slot %d, row %d, %d rows", o, g.wsel, g.rowbase,
                  g.count);
            if (s.bf16) CHECK(g.blk == blk[which], "group %d", o);
        }
        CHECK(seen[which]++ == 0, "group %d twice", o);
        CHECK(o == 0 || groups[o - 1].count >= g.count, "group %d out of order", o);
        group_rows[o] = g.count;
        group_fg[o] = g.wsel < 0 ? s.Fs : s.F;
    }

    // every weight tile of every group meets every token tile once, in either phase
    for (int ph = 0; ph < 2; ++ph) {
        const int shape = s.bf16 ? 0 : meta[3 + ph];
        CHECK(shape >= 0 && shape < kFShapes, "phase %d: shape %d", ph, shape);
        const int tn = s.bf16 ? kTN : shape_rows(shape), wr = shape_weights(shape);
        if (!s.bf16) ++shapes_seen[shape];
        std::vector<int> first(ng + 1, 0);
        for (int o = 0; o < ng; ++o)
            first[o + 1] = first[o] + weight_tiles(H, group_fg[o], ph == 1, wr) * ((group_rows[o] + tn - 1) / tn);
        CHECK(meta[ph] == first[ng], "phase %d: %d items, not %d", ph, meta[ph], first[ng]);
        if (s.bf16) CHECK(first[ng] <= tiled_items(s, ph == 1), "phase %d: %d items", ph, first[ng]);
        if (!s.bf16) {
            for (int o = 0; o < ng; ++o) CHECK(pre[ph * max_groups + o] == first[o], "phase %d, group %d", ph, o);
            continue;
        }
        const TileItem* items = tab + (ph ? tiled_items(s, false) : 0);
        for (int o = 0; o < ng; ++o) {
            const int nwt = weight_tiles(H, group_fg[o], ph == 1, wr), ntt = (group_rows[o] + tn - 1) / tn;
            std::vector<int> hit(nwt * ntt, 0);
            for (int i = first[o]; i < first[o + 1]; ++i) {
                const int g = items[i].gt & 511, tt = items[i].gt >> 9, wt = items[i].wt;
                CHECK(g == o && wt >= 0 && wt < nwt && tt < ntt, "phase %d, item %d: group %d, tiles %d %d", ph, i, g, wt, tt);
                CHECK(hit[wt * ntt + tt]++ == 0, "phase %d, item %d twice", ph, i);
            }
        }
    }

    // the gathered rows
    auto row = [&](int block, int r, int t) {
        for (int h = 0; h < H; ++h) {
            const size_t at = ((size_t)block * (H / 32) + h / 32) * 512 + 8 * (r + 16 * (h % 32 / 8)) + h % 8;
            const uint16_t want = t < 0 ? 0 : reinterpret_cast<uint16_t*>(x.get())[(size_t)t * H + h];
            CHECK(xg[at] == want, "block %d row %d column %d", block, r, h);
        }
    };
    if (s.bf16) {
        for (size_t i = 0; i < active.size(); ++i)
            for (int b = blk[i]; b < blk[i + 1]; ++b)
                for (int r = 0; r < 16; ++r) {
                    const int n = 16 * (b - blk[i]) + r;
                    row(b, r, n < counts[active[i]] ? perm[seg[active[i]] + n] / s.k : -1);
                }
        for (int b = 0; s.S > 0 && b < tb16; ++b)
            for (int r = 0; r < 16; ++r) row(rb + b, r, 16 * b + r < s.T ? 16 * b + r : -1);
    }
}

// The persistent FFN kernels take every item once, from the claim queues and without them.
static void check_queues() {
    for (int n = 1; n <= 3000; n += n < 600 ? 1 : 7) {
        std::vector<int> hit(n, 0);
        for (int x = 0; x < 8; ++x)
            for (int q = 0;; ++q) {
                const int it = claimed_item(q, x);
                if (it >= n) break;  // and so are all that follow in the queue
                CHECK(it >= 0 && hit[it]++ == 0 && claimed_item(q + 1, x) > it, "%d of %d items", it, n);
            }
        CHECK(std::count(hit.begin(), hit.end(), 1) == n, "%d items", n);
        const int cus = 256;
        for (int run : {0, (n + 7) / 8}) {
            if (n > cus) break;
            std::fill(hit.begin(), hit.end(), 0);
            int per_xcd[8] = {};
            for (int wg = 0; wg < cus; ++wg) {
                const int it = few_item(wg / 8, wg % 8, run);
                if (it < n) ++hit[it], ++per_xcd[wg % 8];
            }
            CHECK(std::count(hit.begin(), hit.end(), 1) == n, "%d items, one per CU", n);
            CHECK(*std::max_element(per_xcd, per_xcd + 8) <= (n / 64 + 1) * 8, "%d items spread unevenly", n);
        }
    }
}

int main() {
    check_queues();
    // T, H, E, F, k, S, Fs, slots, bf16; resident, dropped
    std::vector<Case> cases;
    for (int bf16 = 0; bf16 < 2; ++bf16) {
        cases.push_back({{65, 64, 1, 64, 1, 8, 64, 1, bf16}, 1, 0});          // the tightest tables in fp32
        cases.push_back({{70, 64, 12, 128, 3, 0, 0, 5, bf16}, 5, 0});         // one expert a slot
        cases.push_back({{70, 192, 12, 128, 3, 2, 64, 5, bf16}, 12, 0});      // twelve experts share five slots
        cases.push_back({{300, 64, 64, 64, 8, 1, 128, 1, bf16}, 64, 0});      // all in one slot
        cases.push_back({{150, 64, 256, 64, 8, 8, 64, 256, bf16}, 256, 0});  // the most groups
        cases.push_back({{150, 64, 256, 64, 8, 8, 64, 40, bf16}, 256, 5});    // the most experts, shared slots
        cases.push_back({{66, 64, 200, 64, 1, 0, 0, 150, bf16}, 200, 0});     // fewer pairs than slots
        cases.push_back({{80, 64, 6, 64, 2, 0, 0, 0, bf16}, 0, 3});           // no slot at all
        cases.push_back({{600, 128, 3, 192, 2, 1, 64, 2, bf16}, 3, 7});       // several token tiles
    }
    for (int i = 0; i < 12; ++i) {
        Case c;
        Shape& s = c.s;
        s.E = pick(1, 40);
        s.T = i % 4 == 3 ? pick(1, 64) : pick(65, 400);
        s.H = 64 * pick(1, 4);
        s.F = 64 * pick(1, 5);
        s.k = pick(1, min(s.E, 8));
        s.S = pick(0, 2);
        s.Fs = s.S ? 64 * pick(1, 3) : 0;
        s.slots = pick(0, s.E);
        s.bf16 = i / 4 & 1;
        c.resident = s.slots ? pick(0, s.E) : 0;
        c.dropped = pick(0, 3);
        cases.push_back(c);
    }
    for (size_t i = 0; i < cases.size(); ++i) {
        emu_cus = i % 4 == 0 ? 1 : (i % 4 == 1 ? 256 : 8);  // small cases take each item shape
        run(cases[i]);
    }
    for (int i = 0; i < kFShapes; ++i) CHECK(shapes_seen[i] > 0, "item shape %d", i);
    printf("tables ok\n");
    return 0;
}
