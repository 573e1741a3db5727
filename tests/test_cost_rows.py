"""The bandwidth rows of the collapsed hierarchy: written down from the factors, as built from the devices under every unit."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2110_10548_amd", "csrc")
CODE = r"""
#include "p2_plan.cpp"
#include <cstdio>
using namespace p2;

// every placement of the axes, every set of reduce axes, every set of forms
int main(int argc, char** argv) {
    std::vector<int32_t> card, axes;
    int a = 1;
    for (; argv[a][0] != '/'; ++a) card.push_back(std::atoi(argv[a]));
    for (++a; a < argc; ++a) axes.push_back(std::atoi(argv[a]));
    const int n = (int)card.size(), m = (int)axes.size();
    p2_hierarchy h = {n, card.data(), nullptr, nullptr};
    std::string err;
    int64_t count = 0;
    if (enumerate_placements(&h, axes.data(), m, nullptr, 0, &count, err) != P2_OK) return 2;
    std::vector<int32_t> places((size_t)count * n * m);
    if (enumerate_placements(&h, axes.data(), m, places.data(), count, &count, err) != P2_OK) return 2;
    std::vector<Plan> kept;
    long rows = 0, shared = 0;
    for (int64_t p = 0; p < count; ++p)
        for (unsigned mask = 1; mask < (1u << m); ++mask)
            for (unsigned forms = 1; forms < 8; ++forms) {
                std::vector<int32_t> reduce;
                for (int i = 0; i < m; ++i) if (mask >> i & 1u) reduce.push_back(i);
                p2_options opt = {};
                opt.form_mask = forms;
                Plan pl;
                if (make_plan(&h, axes.data(), m, &places[(size_t)p * n * m], reduce.data(), (int)reduce.size(), 1, &opt, false, pl, err) != P2_OK) return 2;
                Plan general = pl;
                build_cost_tables(pl);
                number_collapsed(general, general.local_of, general.replica_of);
                for (size_t t = 0; t < pl.patterns.size(); ++t) {
                    build_cost_rows(general, general.patterns[t]);
                    const Pattern &x = pl.patterns[t], &y = general.patterns[t];
                    if (x.row_ptr != y.row_ptr || x.row_level != y.row_level || x.entries != y.entries) return 1;
                    rows += (long)x.row_level.size();
                }
                for (const Plan& q : kept) {
                    if (!same_cost_rows(pl, q)) continue;
                    ++shared;
                    if (q.patterns.size() != pl.patterns.size()) return 1;
                    for (size_t t = 0; t < q.patterns.size(); ++t)
                        if (pl.patterns[t].row_ptr != q.patterns[t].row_ptr || pl.patterns[t].entries != q.patterns[t].entries) return 1;
                }
                if (kept.size() < 64) kept.push_back(pl);
            }
    std::printf("%ld %ld\n", rows, shared);
    return 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("no host compiler")
    at = tmp_path_factory.mktemp("rows")
    (at / "rows.cpp").write_text(CODE)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", CSRC, str(at / "rows.cpp"), "-o", str(at / "rows")], check=True)
    return str(at / "rows")


@pytest.mark.parametrize("card,axes", [([2, 4], [2, 4]), ([4, 2, 4], [4, 8]), ([3, 4, 6], [6, 12]), ([2, 1, 6], [2, 6]), ([4, 8, 8], [4, 8, 8]), ([5, 1], [1, 5]),
                                       ([2, 3, 2, 4], [6, 8]), ([2, 2, 2, 2, 4], [4, 16])])
def test_rows_from_the_factors(program, card, axes):
    out = subprocess.run([program, *map(str, card), "/", *map(str, axes)], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stderr
    rows, shared = map(int, out.stdout.split())
    assert rows > 0 and shared > 0
