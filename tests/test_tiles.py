"""Index arithmetic of the kernels' tiles (csrc/w2v_tiles.h), compiled for the host: no lane reads outside its row."""
import os
import subprocess
import textwrap

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1606_07822_amd", "csrc")


def run_host(tmp_path, body):
    src, exe = tmp_path / "t.cpp", str(tmp_path / "t")
    src.write_text('#include "w2v_tiles.h"\n#include <cstdint>\n#include <cstdio>\n#include <vector>\n'
                   "using namespace w2v;\n" + textwrap.dedent(body))
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-fsanitize=undefined",
                           "-fno-sanitize-recover=undefined", "-I" + CSRC, str(src), "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr


@pytest.mark.parametrize("lo,hi", [(1, 64), (65, 512), (513, 1024)])
def test_loglik_reads_stay_in_the_row_and_cover_it(tmp_path, lo, hi):
    run_host(tmp_path, f"""
        int main() {{
            for (int dim = {lo}; dim <= {hi}; ++dim) {{
                const int stride = (dim + 3) / 4 * 4;   // the smallest that is accepted
                int i = 0;
                while (dim > kLoglikTiles[i].columns) ++i;
                const LoglikTiles t = kLoglikTiles[i];
                std::vector<int> seen(dim, 0);
                for (int c0 = 0; c0 < (t.panels ? dim : 1); c0 += t.tiles * 64)
                    for (int n = 0; n < t.tiles; ++n)
                        for (int lane = 0; lane < 64; ++lane) {{
                            const int at = quad_column(t.full, c0, n, lane, dim);
                            if (at < 0 || at % 4 || at + 4 > stride) {{
                                std::printf("dim %d tile %d lane %d reads %d..%d\\n", dim, n, lane, at, at + 3);
                                return 1;
                            }}
                            const int col = c0 + n * 64 + lane / 4 * 4;
                            if (n < t.full && col >= dim) return 2;   // its columns are not masked
                            if (lane % 4 == 0)
                                for (int k = col; k < col + 4 && k < dim; ++k) seen[k] += at == col;
                        }}
                for (int k = 0; k < dim; ++k)
                    if (seen[k] != 1) return 3;
            }}
            return 0;
        }}
    """)


def test_search_steps_cover_ranges_of_any_length(tmp_path):
    run_host(tmp_path, """
        int main() {
            for (int64_t n : {int64_t(1), int64_t(63), int64_t(64), int64_t(65), int64_t(1) << 20, (int64_t(1) << 31) - 65,
                              (int64_t(1) << 31) - 64, (int64_t(1) << 31) - 1})
                for (int64_t lo : {int64_t(0), int64_t(1), (int64_t(1) << 31) - 1 - n}) {
                    if (lo < 0 || lo + n > (int64_t(1) << 31) - 1) continue;
                    const int64_t step = probe_step(static_cast<int32_t>(lo), static_cast<int32_t>(lo + n));
                    // 64 probes reach the range's end, and no fewer steps do
                    if (step < 1 || 64 * step < n || 64 * (step - 1) >= n) {
                        std::printf("lo %lld n %lld step %lld\\n", (long long)lo, (long long)n, (long long)step);
                        return 1;
                    }
                }
            return 0;
        }
    """)
