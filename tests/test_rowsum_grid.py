"""CPU test: no row sum launches a grid of 2^32 threads or more, and every row
tile has a finish counter."""
import subprocess


def test_row_tiles_fit_a_grid(tmp_path):
    from paper_2604_22242_amd import build
    src = tmp_path / "lanes.hip"
    src.write_text(
        '#include <cstdio>\n#include "fx_kernels.hpp"\nusing namespace fx;\n'
        "int main() {\n"
        "  int bad = 0;\n"
        "  for (int64_t rows : {1ll, 7ll, 8ll, 63ll, 100ll, 1000ll, 4097ll, 16383ll, 16384ll, 32769ll, 65536ll, 100003ll,\n"
        "                       262144ll, 1048576ll, 3000001ll, 1ll << 30, 1ll << 31, (1ll << 32) + 8, 1ll << 34})\n"
        "    for (int64_t cols : {1ll, 2ll, 3ll, 17ll, 64ll, 1000ll})\n"
        "      for (int elem : {2, 4, 8})\n"
        "        for (int vec = 1; vec * elem <= 16; vec *= 2)\n"
        "          for (int block = 64; block <= 512; block += 64) {\n"
        "            if (rows < vec) continue;\n"
        "            const int rl = rowsum_lanes(rows, cols, vec, elem, block);\n"
        "            const int64_t tiles = ceil_div(rows, (int64_t)rl * vec);\n"
        "            // lanes divide the block and the rows of a tile its finish\n"
        "            bool ok = rl >= 1 && block % rl == 0 && (rl <= 64 ? 64 % rl == 0 : true);\n"
        "            if (rows / vec * 1 < (1ll << 32) - block) ok = ok && tiles * block < (1ll << 32);\n"
        "            launch L{block, 1, vec * elem, 4};\n"
        "            ok = ok && (int64_t)workspace_for(FX_R_ROWSUM, rows, cols, L, elem, vec).counter_bytes >= 4 * tiles;\n"
        '            if (!ok) { ++bad; std::printf("%lld x %lld elem %d vec %d block %d: %d lanes\\n", (long long)rows,\n'
        "                                          (long long)cols, elem, vec, block, rl); }\n"
        "          }\n"
        "  return bad != 0;\n}\n")
    exe = tmp_path / "lanes"
    subprocess.check_call([build.HIPCC] + build.CFLAGS + [str(src), "-L" + build.HERE, "-l:libfx.so",
                                                         "-Wl,-rpath," + build.HERE, "-o", str(exe)])
    p = subprocess.run([str(exe)], capture_output=True, text=True)
    assert p.returncode == 0, p.stdout
