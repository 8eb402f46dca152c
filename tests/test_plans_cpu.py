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
                    for (int planes = 1; planes <= 3; ++planes) need = std::max(need, (size_t)rows_split(rule, N / 16, ksteps, rows, planes) * rows * N);
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
