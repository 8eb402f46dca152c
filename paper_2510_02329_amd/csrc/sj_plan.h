// Launch shapes of the projections: which kernel, how many n-tiles and waves a workgroup has, into how many K-slices and row
// groups a product is cut, and how large the buffer of the partial sums has to be.  Plain host arithmetic without HIP, so that it can
// be checked over all shapes on a machine without a GPU.
#pragma once
#include <algorithm>
#include <cstddef>
#include <vector>

namespace sj {

constexpr int RING_CW = 8;         // waves of the LDS-ring kernel, which interleave K
constexpr int ROWS_MT = 9;         // row tiles per launch (144 rows)

// Up to two row tiles (32 rows) the few-row kernel (every wave fetches its own operand fragments) is the faster
// one (gate/up of the 70B shape at 24 rows: 179 us against 262 us); from three on the loader-wave kernels.
constexpr int FEW_ROWS = 32;

// Shape of a split-K projection launch: NT n-tiles and `waves` waves per workgroup, `split` K-slices
// across workgroups (summed by the consumer), `depth` k-steps in the few-row kernel's load ring.  The chip has
// 256 CUs and these kernels are a single wave of workgroups long, so a launch whose workgroup count is not a
// multiple of 256 leaves CUs idle for its whole duration: plan_partial takes, among the first tile groupings
// the kernel is instantiated for, the one that wastes the fewest workgroup slots, every wave keeping at least
// 8 k-steps; tune_plans then measures that choice against the other shapes on the model's own weights.
// waves == RING_WAVES selects the LDS-ring kernel (eight waves, each with a ring of its own); `depth` is then that ring's 1 KB fragments.
struct GemmPlan { int nt = 4, waves = 4, split = 1, depth = 2; };
constexpr int RING_WAVES = 10;                 // (a mark: the other kernels have 4 or 8)
constexpr int RING_ROWS = FEW_ROWS;
constexpr int RING_PACK_ROWS = 8;              // both operand planes in one product
constexpr int RING_TWO = 9;                    // rings of up to this depth leave room for two workgroups a CU (160 KB of LDS)
constexpr int RING_MOST = 19;                  // fragments of a ring (and n-tiles x row tiles of a reduction) that one workgroup's LDS holds

// operand fragments of a k-step
constexpr int ring_operand(bool pack, int planes, int row_tiles) { return pack ? 1 : planes * row_tiles; }

// Can the LDS-ring kernel run this product in this launch shape?  bf16 with one or two operand planes, up to two row tiles, whole groups of
// n-tiles, K-slices of whole k-blocks (8 k-steps), as many as its ring holds in part, and LDS for the rings and for the reduction.
inline bool ring_fits(const GemmPlan& p, int ntiles, int ksteps, int rows, int planes, bool bf16) {
    if (p.waves != RING_WAVES || !bf16 || planes > 2 || rows > RING_ROWS) return false;
    if (p.nt < 1 || p.split < 1 || p.depth < 1 || ntiles % p.nt || ksteps % (RING_CW * p.split)) return false;
    const int mt = rows > 16 ? 2 : 1, per = p.nt + ring_operand(planes == 2 && rows <= RING_PACK_ROWS, planes, mt), d = std::max(p.depth, per);
    return ksteps / RING_CW / p.split >= (d + per - 1) / per && d <= RING_MOST && p.nt * mt <= RING_MOST;
}

// The shapes the split-K projections are instantiated for: (n-tiles, waves, ring depth) of the register-ring kernel - the second list
// for one and two operand planes only - and (n-tiles, ring depth in fragments) of the LDS-ring kernel.
#define SJ_FEW_PARTIAL_SHAPES(X) X(4, 4, 2) X(4, 4, 4) X(3, 8, 2) X(6, 4, 2) X(1, 8, 2)
#define SJ_FEW_PARTIAL_SHAPES_2(X) X(5, 4, 2) X(8, 8, 2) X(4, 8, 2) X(8, 4, 2) X(3, 4, 4) X(2, 4, 4) X(2, 4, 2) X(2, 8, 2)
#define SJ_RING_PARTIAL_SHAPES(X) X(1, 4) X(1, 9) X(2, 4) X(2, 9) X(3, 4) X(3, 9) X(4, 4) X(4, 9) X(3, 18) X(4, 18) X(5, 18) X(8, 18)

// Is there a kernel for exactly this split-K launch?  The consumer adds p.split K-slices, so no other shape may stand in for it.
inline bool partial_fits(const GemmPlan& p, int ntiles, int ksteps, int rows, int planes, bool bf16) {
    if (p.waves == RING_WAVES) {
#define SJ_IS(NT, D) if (p.nt == NT && p.depth == D) return ring_fits(p, ntiles, ksteps, rows, planes, bf16);
        SJ_RING_PARTIAL_SHAPES(SJ_IS)
#undef SJ_IS
        return false;
    }
    if (p.nt < 1 || ntiles % p.nt) return false;
#define SJ_IS(NT, WV, D) if (p.nt == NT && p.waves == WV && p.depth == D) return true;
    SJ_FEW_PARTIAL_SHAPES(SJ_IS)
    if (planes <= 2) { SJ_FEW_PARTIAL_SHAPES_2(SJ_IS) }
#undef SJ_IS
    return false;
}

// The same for the gate / up projection and the LM head with few rows, which have no K-slices: (n-tiles, waves, ring depth) of the
// register-ring kernel (LM head: depth 2), (n-tiles, ring depth) of the LDS-ring kernel.
#define SJ_FEW_GATE_UP_SHAPES(X) X(7, 8, 2) X(8, 8, 2) X(1, 8, 2)
#define SJ_FEW_GATE_UP_SHAPES_2(X) X(4, 8, 2) X(4, 4, 2) X(2, 8, 2) X(2, 4, 2) X(7, 8, 3) X(7, 8, 4) X(8, 8, 4)
#define SJ_RING_GATE_UP_SHAPES(X) X(1, 4) X(1, 9) X(2, 4) X(2, 9) X(4, 4) X(4, 9) X(7, 18) X(8, 18)
#define SJ_FEW_LOGITS_SHAPES(X) X(8, 4, 2) X(2, 8, 2)
#define SJ_FEW_LOGITS_SHAPES_2(X) X(8, 8, 2) X(4, 8, 2) X(4, 4, 2)
#define SJ_RING_LOGITS_SHAPES(X) X(2, 4) X(2, 9) X(4, 4) X(4, 9) X(8, 9) X(8, 18)
// and for the projections that close a sub-layer in their epilogue
#define SJ_RING_RESID_SHAPES(X) X(1, 4) X(1, 9) X(2, 4) X(2, 9) X(4, 4) X(4, 9)

// Is there a kernel for exactly this launch?
#define SJ_IS_RING(NT, D) if (p.nt == NT && p.depth == D) return ring_fits(p, ntiles, ksteps, rows, planes, bf16);
#define SJ_IS_FEW(NT, WV, D) if (p.nt == NT && p.waves == WV && p.depth == D) return true;
inline bool gate_up_fits(const GemmPlan& p, int ntiles, int ksteps, int rows, int planes, bool bf16) {
    if (p.split != 1 || p.nt < 1 || ntiles % p.nt) return false;
    if (p.waves == RING_WAVES) { SJ_RING_GATE_UP_SHAPES(SJ_IS_RING) return false; }
    SJ_FEW_GATE_UP_SHAPES(SJ_IS_FEW)
    if (planes <= 2) { SJ_FEW_GATE_UP_SHAPES_2(SJ_IS_FEW) }
    return false;
}
inline bool logits_fits(const GemmPlan& p, int ntiles, int ksteps, int rows, int planes, bool bf16) {
    if (p.split != 1 || p.nt < 1 || ntiles % p.nt) return false;
    if (p.waves == RING_WAVES) { SJ_RING_LOGITS_SHAPES(SJ_IS_RING) return false; }
    SJ_FEW_LOGITS_SHAPES(SJ_IS_FEW)
    if (planes <= 2) { SJ_FEW_LOGITS_SHAPES_2(SJ_IS_FEW) }
    return false;
}
#undef SJ_IS_RING
#undef SJ_IS_FEW

// Rule shape of a split-K projection of up to 8 rows on the LDS-ring kernel (two planes: the measured case), or waves = 0
// when no shape fits; from 9 rows on: ring_rule_partial_rows.  Fewest idle workgroup slots first (256 CUs, one round); among those at least two n-tiles per
// workgroup (with one, the operand is as much traffic as the weights) and two K-slices, else four, else one, else
// eight (measured on 4096 x 4096, 4096 x 14336 and 6144 x 4096: the middle of the range wins, and fewer slices are
// less work for the kernel that adds them).
inline GemmPlan ring_rule_partial(int ntiles, int ksteps) {
    static const int nts[] = {2, 3, 4, 8, 1}, splits[] = {2, 4, 1, 8};
    GemmPlan best;
    best.waves = 0;
    double best_waste = 1e30;
    for (int split : splits)
        for (int nt : nts) {
            GemmPlan p;
            p.nt = nt; p.waves = RING_WAVES; p.split = split; p.depth = RING_TWO;
            if (!partial_fits(p, ntiles, ksteps, 1, 2, true)) p.depth = 4;
            if (!partial_fits(p, ntiles, ksteps, 1, 2, true)) continue;
            const int wgs = ntiles / nt * split;
            const double waste = (double)((wgs + 255) / 256 * 256) / wgs + (nt == 1 ? 0.25 : 0.0);
            if (waste < best_waste - 1e-9) { best = p; best_waste = waste; }
        }
    return best;
}
// Who adds a split-K product's K-slices: attention, in its prologue (QKV), or what closes the sub-layer (O, down).
enum class Sums { attention, closing };

// The longest chain of a split-K launch: k-steps that one accumulator adds up before the waves' and slices' sums meet.
inline int partial_chain(const GemmPlan& p, int ksteps) {
    const int lanes = (p.waves == RING_WAVES ? RING_CW : p.waves) * p.split;
    return (ksteps + lanes - 1) / lanes;
}
inline GemmPlan plan_partial(int ntiles, int ksteps, bool one_row_tile);

// The same from 9 rows on, where a k-step has one operand fragment per plane and row tile: whole rounds of 256 workgroups, and few fragments for a
// wave to read (with one row tile an operand fragment counts twice: it comes from the L2 each time), tiles left to the reduction and K-slices (their
// sums are written and read).  QKV_SLICES: slices of QKV, which attention adds (1B, 12 rows: 12.7 us with two, 13.8 with four).  us of the shapes that
// fill the chip, n-tiles x slices:
//   8B, 20 rows: down 4 x 4 21.6, 8 x 8 22.1; QKV 3 x 2 11.4, 3 x 4 12.6;   70B, 24 rows: O 4 x 2 24.8, 8 x 4 28.6; down 8 x 4 72.3, 4 x 2 75.5;
//   1B, 12 rows: O 1 x 2 4.4; down 2 x 4 8.6, 4 x 8 9.1; QKV (192 workgroups) 2 x 2 5.2, 1 x 1 6.1.
// (Back to back; in a step these launches take 1 - 3 us more.)  With two row tiles an operand fragment counts once: any weight from 0.4 to 1.3 has the
// faster of the measured shapes of O and down of 8B and 70B, 2 has O of 70B in 8 x 4.
// QKV's sums are rounded into the cache: it has at least the slices that keep a chain no longer than the register-ring kernel's rule has it (8 - 15 k-steps
// while eight slices allow that; four slices for the 70B shape from 9 rows on, where two would do for the stream).  O and down have no such bound, as the
// rule there never had: their sums stay fp32, and longer chains leave the same error (70B shape, 24 rows, 64 inputs, hidden states against 64 bits,
// relative to the register-ring kernel: O in two slices 1.002 +- 0.017, in four 1.002 +- 0.017).
constexpr int QKV_SLICES = 2;
inline GemmPlan ring_rule_partial_rows(int ntiles, int ksteps, int rows, int planes, Sums sums) {
    GemmPlan best;
    best.waves = 0;
    double best_cost = 1e30;
    const int mt = rows > 16 ? 2 : 1, nb = ring_operand(false, planes, mt), chain = partial_chain(plan_partial(ntiles, ksteps, true), ksteps);
    int most = sums == Sums::attention ? QKV_SLICES : 8;
    for (int split = 1; split <= most; split *= 2) {
        if (sums == Sums::attention && partial_chain(GemmPlan{1, RING_WAVES, split, 0}, ksteps) > chain) {
            most = std::min(8, std::max(most, split * 2));
            continue;
        }
        for (int nt : {1, 2, 3, 4, 5, 8}) {
            const int wgs = ntiles / nt * split, to_cu = (wgs + 255) / 256;
            GemmPlan p;
            p.nt = nt; p.waves = RING_WAVES; p.split = split; p.depth = wgs <= 256 && nt >= 3 ? 18 : RING_TWO;
            if (!partial_fits(p, ntiles, ksteps, rows, planes, true)) p.depth = RING_TWO;
            if (!partial_fits(p, ntiles, ksteps, rows, planes, true)) p.depth = 4;
            if (!partial_fits(p, ntiles, ksteps, rows, planes, true)) continue;
            const double cost = 256.0 * to_cu / wgs * (to_cu * ((double)ksteps / RING_CW / split * (nt + (mt == 2 ? 1 : 2) * nb) + 4 * nt * mt + 8) + 6 * split);
            if (cost < best_cost - 1e-9) { best = p; best_cost = cost; }
        }
    }
    return best;
}
// Gate / up on that kernel: 8 or 7 n-tiles where they make whole rounds of one workgroup a CU (8B, 70B: 7), else two, two workgroups a CU (1B,
// one row: 2 n-tiles 13.0 us, 4 of them 14.8 - 18; 8B, 6 rows: 7 of them 37.4, 4 of them 41.0).
inline GemmPlan ring_rule_gate_up(int ntiles, int ksteps, int rows, int planes) {
    for (int nt : {8, 7, 2, 4, 1})
        for (int depth : {18, RING_TWO, 4}) {
            const GemmPlan p{nt, RING_WAVES, 1, depth};
            if (nt >= 7 && (ntiles / nt) % 256) continue;
            if (gate_up_fits(p, ntiles, ksteps, rows, planes, true)) return p;
        }
    return GemmPlan{4, 0, 1, 0};
}
// LM head on it: four n-tiles, two workgroups a CU; two for short rows of packed operand (1B, one row: 2 n-tiles 76.7 us, 4 of them 85.8; 8B, 6 rows:
// 164 with 4, 169 - 177 with 2); eight from 17 rows on (8B, 20 rows: 191, 4 of them 196).
inline GemmPlan ring_rule_logits(int ntiles, int ksteps, int rows, int planes) {
    const bool two = ksteps <= 64 && planes == 2 && rows <= RING_PACK_ROWS;
    for (int nt : {rows > 16 ? 8 : two ? 2 : 4, 4, 2})
        for (int depth : {nt == 8 ? 18 : RING_TWO, 4}) {
            const GemmPlan p{nt, RING_WAVES, 1, depth};
            if (logits_fits(p, ntiles, ksteps, rows, planes, true)) return p;
        }
    return GemmPlan{8, 0, 1, 0};
}

// Small matrices (small models): a launch is over as soon as its longest workgroup, so every n-tile gets one of its own, its eight waves
// share K (LM head: two n-tiles).  With the shapes of the large ones, 8 or 4 n-tiles to a workgroup on a dozen workgroups: fp32 step of
// d 256, 2 layers, 5 rows: gate / up 7.8 -> 4.1 us, LM head 7.3 -> 4.7, down 7.9 -> 4.5; whole step 129 -> 108 - 112 (the draw's one launch
// among it); bf16, d 512: step of 4 layers, 30 rows 314 -> 224, draft block of 8 layers, one row 1663 -> 1440.
constexpr int SMALL_TILES = 128;
inline GemmPlan rule_gate_up(int ntiles, int planes) {
    GemmPlan p;
    p.waves = 8; p.split = 1; p.depth = 2;
    p.nt = 1;
    if (ntiles < 2 * SMALL_TILES) return p;
    // the n-tiles that leave the fewest workgroup slots of a round of the chip empty, the most of those (8B shape, 1792 tiles: 7; 1B, 1024
    // tiles: 4 - with 8, on half of the CUs, a decode's gate / up takes 17.0 us instead of 14.6; three planes have no kernel of 4)
    double best = 1e30;
    for (int nt : {8, 7, 4}) {
        if (ntiles % nt || (nt == 4 && planes > 2)) continue;
        const int wgs = ntiles / nt;
        const double waste = (double)((wgs + 255) / 256 * 256) / wgs;
        if (waste < best - 1e-9) { best = waste; p.nt = nt; }
    }
    return p;
}
inline GemmPlan rule_logits(int ntiles) { return ntiles < 8 * SMALL_TILES ? GemmPlan{2, 8, 1, 2} : GemmPlan{8, 4, 1, 2}; }

inline GemmPlan plan_partial(int ntiles, int ksteps, bool one_row_tile) {
    static const int cand[3][2] = {{4, 4}, {3, 8}, {6, 4}};
    GemmPlan best;
    if (!one_row_tile) {
        // loader-wave kernel: 8 n-tiles per workgroup, one workgroup per CU; as many K-slices (at most 8, of at
        // least 8 k-steps each) as fit one round of the chip - a second, partly filled round costs a whole one
        const int groups = (ntiles + 7) / 8;
        best.nt = 8; best.waves = 8;
        best.split = std::max(1, std::min({8, 256 / std::max(groups, 1), ksteps / 8}));
        return best;
    }
    if (ntiles < SMALL_TILES) {
        best.nt = 1; best.waves = 8;
        while (best.split < 4 && ntiles * best.split * 2 <= 256 && ksteps / (8 * best.split * 2) >= 8) best.split *= 2;
        return best;
    }
    double best_waste = 1e30;
    for (const auto& c : cand) {
        if (ntiles % c[0]) continue;
        int split = 1;
        while (split < 8 && ksteps / (c[1] * split * 2) >= 8) split *= 2;
        const int wgs = ntiles / c[0] * split;
        const double waste = (double)((wgs + 255) / 256 * 256) / wgs;
        if (waste < best_waste - 1e-9) { best.nt = c[0]; best.waves = c[1]; best.split = split; best_waste = waste; }
    }
    // short K-slices (at most 8 k-steps per wave): a deeper register ring puts the whole slice in flight
    best.depth = (best.nt == 4 && best.waves == 4 && ksteps / (best.split * 4) <= 8) ? 4 : 2;
    return best;
}

// The launch of a split-K projection with at most 32 rows: the plan, or, where its kernel does not take these rows or planes (a prompt
// chunk can have more rows than the plan was made for), the register-ring kernel's rule shape, which is always instantiated.
inline GemmPlan resolve_partial(const GemmPlan& p, int ntiles, int ksteps, int rows, int planes, bool bf16) {
    return partial_fits(p, ntiles, ksteps, rows, planes, bf16) ? p : plan_partial(ntiles, ksteps, true);
}

// The same for the gate / up projection and the LM head.  (The LM head's statistics are laid out for the n-tiles of the launch: whoever
// reads them goes by what this returned.)
inline GemmPlan resolve_gate_up(const GemmPlan& p, int ntiles, int ksteps, int rows, int planes, bool bf16) {
    return gate_up_fits(p, ntiles, ksteps, rows, planes, bf16) ? p : rule_gate_up(ntiles, planes);
}
inline GemmPlan resolve_logits(const GemmPlan& p, int ntiles, int ksteps, int rows, int planes, bool bf16) {
    return logits_fits(p, ntiles, ksteps, rows, planes, bf16) ? p : rule_logits(ntiles);
}

// The rules over both kernels; the LDS-ring kernel up to `ring_rows` rows.
inline GemmPlan rule_partial(int ntiles, int ksteps, int rows, int planes, bool bf16, int ring_rows, Sums sums) {
    if (bf16 && planes <= 2 && rows <= ring_rows) {
        const GemmPlan r = rows <= RING_PACK_ROWS ? ring_rule_partial(ntiles, ksteps) : ring_rule_partial_rows(ntiles, ksteps, rows, planes, sums);
        if (r.waves) return r;
    }
    return plan_partial(ntiles, ksteps, true);
}
inline GemmPlan rule_gate_up(int ntiles, int ksteps, int rows, int planes, bool bf16, int ring_rows) {
    if (bf16 && planes <= 2 && rows <= ring_rows) {
        const GemmPlan r = ring_rule_gate_up(ntiles, ksteps, rows, planes);
        if (r.waves) return r;
    }
    return rule_gate_up(ntiles, planes);
}
inline GemmPlan rule_logits(int ntiles, int ksteps, int rows, int planes, bool bf16, int ring_rows) {
    if (bf16 && planes <= 2 && rows <= ring_rows) {
        const GemmPlan r = ring_rule_logits(ntiles, ksteps, rows, planes);
        if (r.waves) return r;
    }
    return rule_logits(ntiles);
}

// A shape made (by the rule or the measurement) for one row count speaks for others with as many operand fragments to a k-step: one packed, one
// row tile, two.  A draft block of 12 sequences runs 12 rows on an object made for blocks of 60: in the shapes of 32 rows, or what stood in
// for those that do not take 12, its QKV and O took 7.2 us each; in the rule's for 12 rows 5.2 and 4.9.
inline int few_class(int rows) { return rows <= RING_PACK_ROWS ? 0 : rows <= 16 ? 1 : 2; }
inline GemmPlan few_partial_plan(const GemmPlan& made, int made_rows, int ntiles, int ksteps, int rows, int planes, bool bf16, int ring_rows, Sums sums) {
    return resolve_partial(few_class(rows) == few_class(made_rows) ? made : rule_partial(ntiles, ksteps, rows, planes, bf16, ring_rows, sums), ntiles, ksteps, rows, planes, bf16);
}
inline GemmPlan few_gate_up_plan(const GemmPlan& made, int made_rows, int ntiles, int ksteps, int rows, int planes, bool bf16, int ring_rows) {
    return resolve_gate_up(few_class(rows) == few_class(made_rows) ? made : rule_gate_up(ntiles, ksteps, rows, planes, bf16, ring_rows), ntiles, ksteps, rows, planes, bf16);
}
inline GemmPlan few_logits_plan(const GemmPlan& made, int made_rows, int ntiles, int ksteps, int rows, int planes, bool bf16, int ring_rows) {
    return resolve_logits(few_class(rows) == few_class(made_rows) ? made : rule_logits(ntiles, ksteps, rows, planes, bf16, ring_rows), ntiles, ksteps, rows, planes, bf16);
}

// Shapes that the start-up measurement tries for a split-K projection with at most 32 rows.
inline std::vector<GemmPlan> partial_candidates(int ntiles, int ksteps, int rows, int planes, bool bf16) {
    std::vector<GemmPlan> cands;
    auto offer = [&](int nt, int waves, int depth) {
        for (int split = 1; split <= 8; split *= 2) {
            GemmPlan p;
            p.nt = nt; p.waves = waves; p.split = split; p.depth = depth;
            const long long wgs = (long long)ntiles / nt * split;
            if (!partial_fits(p, ntiles, ksteps, rows, planes, bf16)) continue;
            if (split == 1 && ntiles < SMALL_TILES && nt == 1 && waves != RING_WAVES) {   // the rule's shape of a small matrix, where it starts from a ring
                cands.push_back(p);
                continue;
            }
            if (wgs < 128 || wgs > 4096) continue;
            const int kpw = ksteps / (waves * split);       // k-steps of a wave of the register-ring kernel
            if (waves != RING_WAVES && (kpw < 4 || (depth == 4 && kpw > 8))) continue;
            cands.push_back(p);
        }
    };
#define SJ_OFFER(NT, WV, D) offer(NT, WV, D);
    SJ_FEW_PARTIAL_SHAPES(SJ_OFFER)
    SJ_FEW_PARTIAL_SHAPES_2(SJ_OFFER)
#undef SJ_OFFER
#define SJ_OFFER(NT, D) offer(NT, RING_WAVES, D);
    SJ_RING_PARTIAL_SHAPES(SJ_OFFER)
#undef SJ_OFFER
    return cands;
}

// Those of them that may take the place of `rule`, the rule's shape.  QKV: of no more K-slices, since the measurement does not see the attention
// launches that add them (1B, 1 row, a draft block: 8 slices 4642 us, 4 slices 4529 - 4580), and from 9 rows on of no longer chains than the rule's
// bound.  `closes`: on the LDS-ring kernel.
inline std::vector<GemmPlan> measured_partials(const GemmPlan& rule, int ntiles, int ksteps, int rows, int planes, bool bf16, Sums sums, bool closes) {
    std::vector<GemmPlan> cands = partial_candidates(ntiles, ksteps, rows, planes, bf16);
    const int chain = std::max(partial_chain(rule, ksteps), partial_chain(plan_partial(ntiles, ksteps, true), ksteps));
    auto out = [&](const GemmPlan& p) {
        return (sums == Sums::attention && (p.split > rule.split || (rows > RING_PACK_ROWS && partial_chain(p, ksteps) > chain))) || (closes && p.waves != RING_WAVES);
    };
    cands.erase(std::remove_if(cands.begin(), cands.end(), out), cands.end());
    return cands;
}

// Row tiles of a row group of the loader-wave kernel: the smallest group that holds all rows, or, with more rows than the largest
// holds, the one of the two largest that pads them least (equal: fewer groups).  The kernel spends matrix and L2 time on
// every tile of a group: 126 rows in groups of 144 (score block of 6 x 21, 8B shape): QKV / O / down 30.6 us, LM head 348, in
// one group of 128: 29.3, 325; 509 rows, 4 x 144 against 4 x 128: gate / up 277 -> 249 us.
// planes: bf16 operand planes, 0 = fp32 storage, whose folded accumulators leave registers for 144 rows (and groups of 256 or 288 were
// the slower ones: 252 rows, d 1024: 962 -> 572 us, 500 rows 1195 -> 882).  Three planes: the 18 operand fragments that the stages in
// LDS hold are six row tiles (8B shape cut to 3 layers, 45 / 144 / 288 rows: 1018 / 2937 / 7087 us with compute waves that loaded the
// operand themselves, in groups of 144; 823 / 1533 / 2582 so).
inline int row_tiles(int planes, int rows) {
    static const int lists[4][4] = {{4, 4, 4, 9}, {4, 9, 16, 18}, {4, 6, 8, 9}, {4, 4, 5, 6}};
    const int* rt = lists[planes];
    for (int i = 0; i < 4; ++i)
        if (rows <= rt[i] * 16) return rt[i];
    auto padded = [&](int t) { return (rows + t * 16 - 1) / (t * 16) * t; };
    return padded(rt[2]) < padded(rt[3]) ? rt[2] : rt[3];
}

// K-slices of a split-K projection on the loader-wave kernel, which works in groups of `group` rows.  One group: the
// rule's (one round of the chip).  With several, the groups fill the chip by themselves and every further slice costs a
// write and a read of the partials: the slice count (never above the rule's) with the least estimated time, in units of
// one k-step of a workgroup (0.58 us on two-plane operands) - rounds of 256 workgroups x (k-steps of a slice + 5 for ramp
// and epilogue) + the partials' bytes at 4 TB/s.
inline int rows_split(int rule, int ntiles, int ksteps, int rows, int planes) {
    const int group = row_tiles(planes, rows) * 16;
    if (rows <= group) return rule;
    const int rgroups = (rows + group - 1) / group, wgs = (ntiles + 7) / 8 * rgroups;
    int best = 1;
    double best_cost = 1e30;
    for (int s = 1; s <= rule; ++s) {
        const double rounds = (wgs * s + 255) / 256;
        const double cost = rounds * ((double)ksteps / s + 5.0) + (double)s * rgroups * group * ntiles * 16 * 8 / 4e12 / 0.58e-6;
        if (cost < best_cost - 1e-9) { best = s; best_cost = cost; }
    }
    return best;
}
// fp32 elements of the partials of a projection with up to `rows` rows, for every plane count, since a cache object's can be changed
// between steps (slices and group depend on the rows in steps of 16; another plane count has other groups, and fewer groups can
// mean more slices), and for any few-row plan the start-up measurement may pick (at most 8 K-slices)
inline size_t part_elems(int rule, int N, int ksteps, int rows) {
    size_t most = (size_t)8 * std::min(rows, FEW_ROWS) * N;
    for (int planes = 0; planes <= 3; ++planes)
        for (int r = 0; r < rows; r += 16) {
            const int upto = std::min(r + 16, rows);
            most = std::max(most, (size_t)rows_split(rule, N / 16, ksteps, upto, planes) * upto * N);
        }
    return most;
}

// Row tiles of a row group of the large-tile gate / up kernel (gemm_tile_kernel: bf16, two planes, 16 n-tiles a workgroup), 0: not taken.
// One workgroup to a CU, so its tiles have to come in nearly whole rounds of 256.  us of that kernel / of the loader-wave kernel:
//   8B shape (4096 -> 2 x 14336), rows 260 / 320 / 380 / 440 / 509 (224 tiles): 150 / 171, 150 / 226, 179 / 228, 207 / 298, 238 / 296;
//   220 rows (112 tiles): 165 / 138; 576 (336 tiles, a second round a third full): 307 / 343;
//   70B (8192 -> 2 x 28672), rows 160 / 320 / 576 (224, 448, 672 tiles): 340 / 537, 590 / 759, 920 / 1044;
//   1B (2048 -> 2 x 8192), rows 160 / 380 / 509 / 576 (64, 128, 128, 192 tiles): 63 / 37, 78 / 66, 100 / 71, 82 / 80.
constexpr int TILE_NT = 16;
constexpr int TILE_WGS = 256;
inline int tile_rows(int rows, int ntiles) {
    if (rows <= ROWS_MT * 16) return 0;
    const int groups = (rows + 255) / 256, rt = std::max(10, ((rows + 15) / 16 + groups - 1) / groups + 1) / 2 * 2;
    const int tiles = (ntiles + TILE_NT - 1) / TILE_NT * groups, rounds = (tiles + TILE_WGS - 1) / TILE_WGS;
    return tiles * 100 >= rounds * TILE_WGS * (rounds > 1 ? 65 : 80) ? rt : 0;
}

// The same for the LM head, on one operand plane or two: row tiles of a row group of the large-tile kernel, 0: not taken.  Row groups are
// as few as LDS allows (16 row tiles of two planes, 18 of one) and of nearly equal size.  us of one layer and the head, or of a head
// alone (one plane), with the loader-wave kernel / with this one:
//   8B shape, rows 64 / 81 / 96 / 144 / 154 / 224: 463 / 459, 525 / 502, 535 / 506, 1367 / 1331 (4 layers), 896 / 686, 931 / 809;
//   head alone, rows 64 / 80 / 128 / 192 / 288 / 360 / 576: 262 / 281, 292 / 286, 326 / 302, 360 / 317, 425 / 394, 605 / 555, 708 / 638;
//   1B, rows 64 / 96 / 192 / 320: 284 / 280, 328 / 308, 512 / 415, 721 / 615; 70B, rows 64 / 96 / 144 / 192: 903 / 889, 1096 / 1039, 1315 / 1236, 1861 / 1524;
//   48 rows: 432 / 442 (8B), 261 / 278 (head alone).
// Row groups of an odd number of tiles leave one half of the waves a tile less.  From nine tiles of two planes on, where the products bound a
// k-step, that beats a padded even group; padded / odd, 8B and 1B shapes, one layer and the head: 5 tiles 488 / 491, 294 / 299, 7 tiles 541 / 541,
// 324 / 327, 9 tiles 602 / 593, 363 / 362, 11 tiles 709 / 690, 391 / 381, 13 tiles 770 / 757, 427 / 422, 15 tiles 833 / 817, 462 / 454.  On one plane
// it makes no difference: 5 to 15 tiles 286 / 285, 293 / 293, 297 / 299, 300 / 302, 318 / 319, 335 / 335.
// Gate / up of the 70B shape on these small row groups: 96 and 144 rows 0 %, 99 rows 2 % of a layer and head: not taken.
constexpr int TILE_STAT = 4;                   // n-tiles of a wave, and of a softmax statistic
inline int tile_logits(int rows, int ntiles, int planes) {
    if (rows <= 64 || planes < 1 || planes > 2) return 0;
    const int tiles = (rows + 15) / 16, most = planes == 2 ? 16 : 18, groups = (tiles + most - 1) / most, per = (tiles + groups - 1) / groups;
    const int rt = planes == 2 && per >= 9 ? per : (per + 1) / 2 * 2;              // the sizes gemm_tile launches
    const int wgs = (ntiles + TILE_NT - 1) / TILE_NT * groups, rounds = (wgs + TILE_WGS - 1) / TILE_WGS;
    return wgs * 100 >= rounds * TILE_WGS * (rounds > 1 ? 65 : 80) ? rt : 0;
}

// A projection that closes a sub-layer (O, down) with the residual add in its epilogue (EPI_RESID; no K-slices): one launch
// instead of two.  Without slices a workgroup has one n-tile (two, four where that fills the chip) and reads as much operand as
// weights, so it pays up to 8 rows, where both planes are one packed fragment: 8B shape, 6 rows: down 20.3 -> 21.0 us, O 8.5 ->
// 8.7, the norm launches (4.7 us each) gone, step 3.45 -> 3.30 ms; 1B draft, 1 row: 5.18 -> 4.85 ms a block.  At 12 and 20 rows
// (operand twice and four times the weights) steps took 8 % and 11 % longer.  nt = 0: not taken.
inline GemmPlan resid_plan(int N, int K, int kstep, int rows, int planes, bool bf16, int ring_rows) {
    GemmPlan p;
    p.nt = 0;
    const int ntiles = N / 16, ksteps = K / kstep, nt = ntiles > 512 ? 4 : ntiles > 256 ? 2 : 1;
    if (rows > RING_PACK_ROWS || planes > 2 || ntiles % nt) return p;
    p.nt = nt; p.split = 1;
    p.waves = RING_WAVES;
    for (int depth : {RING_TWO, 4}) {
        p.depth = depth;
        if (rows <= ring_rows && ring_fits(p, ntiles, ksteps, rows, planes, bf16)) return p;
    }
    p.waves = 8; p.depth = 2;
    return p;
}
}  // namespace sj
