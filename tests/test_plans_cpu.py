"""The launch-shape rules of the projections, over model shapes, row counts and operand planes, on the CPU."""
from tests.plan_check import run_program, shapes_array

PARTIALS = shapes_array() + r"""
// a cache object of `rows` rows may launch any smaller number, with any number of operand planes
int main() {
    long bad = 0, checked = 0;
    for (const auto& s : shapes)
        for (int kstep : {32, 16}) {
            const int prod[3][2] = {{s[1], s[0]}, {s[0], s[2]}, {s[0], s[3]}};      // N, K of QKV, O, down
            for (const auto& p : prod) {
                const int N = p[0], ksteps = p[1] / kstep;
                if (ksteps < 1) continue;
                const int rule = plan_partial(N / 16, ksteps, false).split;
                size_t need = 0;
                for (int rows = 1; rows <= 4200; ++rows) {
                    for (int planes = 0; planes <= 3; ++planes) need = std::max(need, (size_t)rows_split(rule, N / 16, ksteps, rows, planes) * rows * N);
                    if (rows % 7 && rows % 16 && rows % 9) continue;
                    ++checked;
                    if (part_elems(rule, N, ksteps, rows) < need && bad++ < 10)
                        printf("N %d, %d k-steps, %d rows: %zu elements, %zu needed\n", N, ksteps, rows, part_elems(rule, N, ksteps, rows), need);
                }
            }
        }
    printf("%ld of %ld too small\n", bad, checked);
}
"""


def test_partials_of_every_launch_fit_their_buffer(tmp_path):
    out = run_program(tmp_path, PARTIALS)
    assert out.splitlines()[-1].startswith("0 of "), out

LAUNCHES = shapes_array() + r"""
// what a split-K projection of at most 32 rows may be launched as: the rule shapes, whatever the measurement tries, and their stand-ins
int main() {
    long bad = 0, checked = 0;
    for (const auto& s : shapes)
        for (int kstep : {32, 16})
            for (int rows = 1; rows <= 32; ++rows)
                for (int planes = 1; planes <= 3; ++planes) {
                    const bool bf16 = kstep == 32;
                    if (!bf16 && planes > 1) continue;
                    const int prod[3][2] = {{s[1], s[0]}, {s[0], s[2]}, {s[0], s[3]}};      // N, K of QKV, O, down
                    for (const auto& p : prod) {
                        const int ntiles = p[0] / 16, ksteps = p[1] / kstep;
                        auto see = [&](const char* what, const GemmPlan& q) {
                            ++checked;
                            // a kernel, and every K-slice written: none is empty
                            if ((!partial_fits(q, ntiles, ksteps, rows, planes, bf16) || q.split > std::max(ksteps, 1)) && bad++ < 10)
                                printf("%s: %d tiles, %d k-steps, %d rows, %d planes: {%d, %d, %d, %d}\n", what, ntiles, ksteps, rows, planes, q.nt, q.waves, q.split, q.depth);
                        };
                        see("rule", plan_partial(ntiles, ksteps, true));
                        GemmPlan ring = ring_rule_partial(ntiles, ksteps);
                        if (ring.waves && bf16 && planes <= 2 && rows <= 8) see("ring rule", ring);
                        // the rule over both kernels, with the ring's limit of rows anywhere, and a plan made for any class of rows
                        const Sums sums = &p == prod ? Sums::attention : Sums::closing;
                        for (int ring_rows : {0, 8, 20, RING_ROWS}) {
                            see("rule over both kernels", rule_partial(ntiles, ksteps, rows, planes, bf16, ring_rows, sums));
                            for (int made : {1, 8, 9, 16, 17, 32})
                                see("plan of a class", few_partial_plan(rule_partial(ntiles, ksteps, made, planes, bf16, ring_rows, sums), made, ntiles, ksteps, rows, planes, bf16, ring_rows, sums));
                        }
                        for (const GemmPlan& q : partial_candidates(ntiles, ksteps, rows, planes, bf16)) see("candidate", q);
                        // plans of other row and plane counts, as a prompt chunk or a changed plane count finds them
                        if (ring.waves) see("resolved ring rule", resolve_partial(ring, ntiles, ksteps, rows, planes, bf16));
                        for (int r2 : {1, 8, 12, 24})
                            for (const GemmPlan& q : partial_candidates(ntiles, ksteps, r2, bf16 ? 2 : 1, bf16))
                                see("resolved candidate", resolve_partial(q, ntiles, ksteps, rows, planes, bf16));
                    }
                }
    printf("%ld of %ld without a kernel\n", bad, checked);
}
"""


def test_every_split_k_launch_is_an_instantiated_shape(tmp_path):
    """The consumer adds the plan's K-slices: a launch in another shape would leave some of them from an earlier product."""
    out = run_program(tmp_path, LAUNCHES)
    assert out.splitlines()[-1].startswith("0 of "), out


TILES = shapes_array() + r"""
int main() {
    long bad = 0, taken = 0;
    for (const auto& s : shapes)
        for (int rows = 1; rows <= 4200; ++rows) {
            const int ntiles = 2 * s[3] / 16, rt = tile_rows(rows, ntiles);
            if (!rt) continue;
            ++taken;
            // an instantiated size whose groups hold all rows, none of them empty, with a k-step pair to work on
            const int groups = (rows + rt * 16 - 1) / (rt * 16);
            const bool known = rt == 10 || rt == 12 || rt == 14 || rt == 16;
            if ((!known || rows <= ROWS_MT * 16 || groups * rt * 16 < rows || (groups - 1) * rt * 16 >= rows || s[0] % 64) && bad++ < 10)
                printf("%d rows, %d tiles: %d\n", rows, ntiles, rt);
        }
    printf("%ld of %ld large-tile launches wrong\n", bad, taken);
}
"""


def test_large_tile_launches_hold_their_rows(tmp_path):
    out = run_program(tmp_path, TILES).splitlines()[-1]
    assert out.startswith("0 of ") and not out.startswith("0 of 0 "), out


FEW = shapes_array() + r"""
// what the gate / up projection and the LM head of at most 32 rows are launched as: the rule's shapes, its ring shapes, and plans that were made for
// another row or plane count
int main() {
    long bad = 0, checked = 0;
    for (const auto& s : shapes)
        for (int vocab : {1024, 4096, 4992, 16256, 16384, 32000, 128256})
            for (int rows = 1; rows <= 32; ++rows)
                for (int planes = 0; planes <= 3; ++planes) {                 // 0: fp32
                    const bool bf16 = planes > 0;
                    const int spl = bf16 ? planes : 1, ksteps = s[0] / (bf16 ? 32 : 16), gu = 2 * s[3] / 16, lm = vocab / 16;
                    auto see = [&](const char* what, const GemmPlan& q, int ntiles, bool fits) {
                        ++checked;
                        if (!fits && bad++ < 10)
                            printf("%s: %d tiles, %d k-steps, %d rows, %d planes: {%d, %d, %d, %d}\n", what, ntiles, ksteps, rows, planes, q.nt, q.waves, q.split, q.depth);
                    };
                    auto gate_up = [&](const char* what, const GemmPlan& q) { see(what, q, gu, gate_up_fits(q, gu, ksteps, rows, spl, bf16)); };
                    auto logits = [&](const char* what, const GemmPlan& q) { see(what, q, lm, logits_fits(q, lm, ksteps, rows, spl, bf16)); };
                    // a residual epilogue leaves operands that its consumers scale, for at most 8 rows and two planes
                    for (int K : {s[2], s[3]}) {
                        const GemmPlan q = resid_plan(s[0], K, bf16 ? 32 : 16, rows, spl, bf16, RING_PACK_ROWS);
                        see("residual", q, s[0] / 16, !q.nt || (rows <= 8 && planes <= 2));
                    }
                    // no K-slices; an instantiated shape of either kernel
                    for (int K : {s[2], s[3]})
                        for (int ring_rows : {0, RING_PACK_ROWS, RING_ROWS}) {
                            const GemmPlan q = resid_plan(s[0], K, bf16 ? 32 : 16, rows, spl, bf16, ring_rows);
                            bool known = q.waves == 8 && (q.nt == 1 || q.nt == 2 || q.nt == 4);
#define SJ_KNOWN(NT, D) if (q.waves == RING_WAVES && q.nt == NT && q.depth == D) known = ring_fits(q, s[0] / 16, K / 32, rows, spl, bf16);
                            SJ_RING_RESID_SHAPES(SJ_KNOWN)
#undef SJ_KNOWN
                            see("residual", q, s[0] / 16, !q.nt || (rows <= 8 && planes <= 2 && q.split == 1 && known));
                        }
                    gate_up("gate/up rule", rule_gate_up(gu, spl));
                    logits("LM head rule", rule_logits(lm));
                    for (int ring_rows : {0, 8, 20, RING_ROWS}) {
                        gate_up("gate/up rule over both kernels", rule_gate_up(gu, ksteps, rows, spl, bf16, ring_rows));
                        logits("LM head rule over both kernels", rule_logits(lm, ksteps, rows, spl, bf16, ring_rows));
                        for (int made : {1, 8, 9, 16, 17, 32}) {
                            gate_up("gate/up plan of a class", few_gate_up_plan(rule_gate_up(gu, ksteps, made, spl, bf16, ring_rows), made, gu, ksteps, rows, spl, bf16, ring_rows));
                            logits("LM head plan of a class", few_logits_plan(rule_logits(lm, ksteps, made, spl, bf16, ring_rows), made, lm, ksteps, rows, spl, bf16, ring_rows));
                        }
                    }
                    for (int nt : {1, 2, 4, 7, 8})
                        for (int waves : {4, 8, RING_WAVES})
                            for (int depth : {2, 3, 4, 8}) {
                                gate_up("gate/up resolved", resolve_gate_up(GemmPlan{nt, waves, 1, depth}, gu, ksteps, rows, spl, bf16));
                                logits("LM head resolved", resolve_logits(GemmPlan{nt, waves, 1, depth}, lm, ksteps, rows, spl, bf16));
                            }
                    for (int nt : {1, 2, 4, 7, 8})
                        for (int waves : {4, 8, RING_WAVES})
                            for (int depth : {9, 18}) {
                                gate_up("gate/up resolved", resolve_gate_up(GemmPlan{nt, waves, 1, depth}, gu, ksteps, rows, spl, bf16));
                                logits("LM head resolved", resolve_logits(GemmPlan{nt, waves, 1, depth}, lm, ksteps, rows, spl, bf16));
                            }
                }
    printf("%ld of %ld without a kernel\n", bad, checked);
}
"""


def test_every_gate_up_and_lm_head_launch_is_an_instantiated_shape(tmp_path):
    """A shape without a kernel would run as another one: timed, and reported, under the wrong name."""
    out = run_program(tmp_path, FEW)
    assert out.splitlines()[-1].startswith("0 of "), out


CHAINS = shapes_array() + r"""
// split-K products of 9 to 32 rows: what the rule takes for a row count, what a plan of another class of rows becomes, and what the measurement may
// put in the rule's place
int main() {
    long bad = 0, checked = 0;
    for (const auto& s : shapes)
        for (int rows = RING_PACK_ROWS + 1; rows <= FEW_ROWS; ++rows)
            for (int planes = 1; planes <= 2; ++planes) {
                const int prod[3][2] = {{s[1], s[0]}, {s[0], s[2]}, {s[0], s[3]}};      // N, K of QKV, O, down
                for (const auto& p : prod) {
                    const int ntiles = p[0] / 16, ksteps = p[1] / 32;
                    const Sums sums = &p == prod ? Sums::attention : Sums::closing;
                    const int longest = partial_chain(plan_partial(ntiles, ksteps, true), ksteps);
                    auto see = [&](const char* what, const GemmPlan& q) {
                        ++checked;
                        if (((sums == Sums::attention && partial_chain(q, ksteps) > longest) || !partial_fits(q, ntiles, ksteps, rows, planes, true)) && bad++ < 10)
                            printf("%s: %d tiles, %d k-steps, %d rows, %d planes: {%d, %d, %d, %d}\n", what, ntiles, ksteps, rows, planes, q.nt, q.waves, q.split, q.depth);
                    };
                    const GemmPlan rule = rule_partial(ntiles, ksteps, rows, planes, true, RING_ROWS, sums);
                    see("rule", rule);
                    for (int made : {1, 12, 32}) {
                        const GemmPlan other = rule_partial(ntiles, ksteps, made, planes, true, RING_ROWS, sums);
                        if (few_class(made) != few_class(rows)) see("another class", few_partial_plan(other, made, ntiles, ksteps, rows, planes, true, RING_ROWS, sums));
                    }
                    for (bool closes : {false, true})
                        for (const GemmPlan& q : measured_partials(rule, ntiles, ksteps, rows, planes, true, sums, closes)) {
                            see("measured", q);
                            if (sums == Sums::attention && q.split > rule.split && bad++ < 10) printf("QKV of %d slices, the rule has %d\n", q.split, rule.split);
                            // where the sub-layers are closed in the products' launches, a shape of another kernel would bring the norm's launch back
                            if (closes && q.waves != RING_WAVES && bad++ < 10) printf("not on the LDS rings: {%d, %d, %d, %d}\n", q.nt, q.waves, q.split, q.depth);
                        }
                }
            }
    printf("%ld of %ld wrong\n", bad, checked);
}
"""


def test_few_row_qkv_sums_are_no_longer_than_the_register_rings(tmp_path):
    """Fewer K-slices are longer fp32 sums: no QKV launch of 9 to 32 rows, whose sums are rounded into the cache, adds more k-steps in one
    accumulator than the register-ring kernel's rule does, by the rule or by the start-up measurement."""
    out = run_program(tmp_path, CHAINS)
    assert out.splitlines()[-1].startswith("0 of "), out


HEADS = r"""
int main() {
    long bad = 0, taken = 0;
    for (int ntiles = 32; ntiles <= 9600; ntiles += ntiles < 1024 ? 8 : 248)
        for (int rows = 1; rows <= 4200; ++rows)
            for (int planes = 0; planes <= 3; ++planes) {
                const int rt = tile_logits(rows, ntiles, planes);
                if (!rt) continue;
                ++taken;
                // an instantiated size whose groups hold all rows, none of them empty, and whole statistics of a row
                const int groups = (rows + rt * 16 - 1) / (rt * 16);
                const bool known = (rt % 2 == 0 && rt >= 6 && rt <= 16) || (planes == 2 && rt % 2 && rt >= 9 && rt <= 15) || (planes == 1 && rt == 18);
                if ((!known || rows <= 64 || planes < 1 || planes > 2 || groups * rt * 16 < rows || (groups - 1) * rt * 16 >= rows || ntiles % TILE_STAT) && bad++ < 10)
                    printf("%d rows, %d tiles, %d planes: %d\n", rows, ntiles, planes, rt);
            }
    printf("%ld of %ld large-tile heads wrong\n", bad, taken);
}
"""


def test_large_tile_heads_hold_their_rows(tmp_path):
    out = run_program(tmp_path, HEADS).splitlines()
    assert out[-1].startswith("0 of ") and not out[-1].startswith("0 of 0 "), out
