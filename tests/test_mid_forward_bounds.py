"""What the forward of small and mid-sized batches asks memory for, walked on the CPU with the very functions
the kernel forms its addresses with (csrc/gram_mid_rows.h, compiled by the host compiler): entries of the row
list and bytes of A for the rows of every tile and every slab.  A caller's list may hold just the U items, and a
caller's matrix of hidden activations just their rows: nothing behind either is read."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

WALK = r"""
#include <cstdio>
#include <initializer_list>
#include "gram_mid_rows.h"
using namespace gram;
int main()
{
    const int items[] = {1, 2, 31, 32, 33, 63, 64, 65, 100, 127, 128, 129, 300, 1000, 1281};
    const int widths[] = {8, 64, 72, 136, 264, 1536};
    long reads = 0;
    for (int tile : {64, 128})                          // rows of a tile
        for (int U : items)
            for (int k : widths) {
                const uint32_t a_bytes = (uint32_t)U * k * 2;           // identity list: row j of A
                for (int j = 0; j < (U + tile - 1) / tile * tile; ++j) {        // rows of the tiles that start below U
                    const int e = mid_list_entry(j, U);
                    if (e < 0 || e >= U) return std::printf("list entry %d of %d\n", e, U), 1;
                    for (int xk = 0; xk < 64; xk += 8) {
                        const uint32_t row = mid_row_offset(j, U, false, (uint32_t)e, (uint32_t)k, (uint32_t)xk);
                        if (mid_row_offset(j, U, true, (uint32_t)e, (uint32_t)k, (uint32_t)xk) != kPastEnd) return 2;
                        for (int k0 = 0; k0 < (k + 63) / 64 * 64 + 6 * 64; k0 += 64) {      // and the slabs past the end
                            const uint32_t at = mid_slab_offset(row, k0, xk, k);
                            if (j >= U || k0 + xk >= k) {
                                if (at != kPastEnd) return std::printf("row %d of %d at element %d of %d\n", j, U, k0 + xk, k), 3;
                            } else if (at != ((uint32_t)j * k + k0 + xk) * 2 || at + 16 > a_bytes) {
                                return std::printf("byte %u of %u\n", at, a_bytes), 4;
                            } else {
                                ++reads;
                            }
                        }
                    }
                }
            }
    std::printf("%ld\n", reads);
    return 0;
}
"""


def test_nothing_behind_the_items_is_read(tmp_path):
    src, exe = tmp_path / "walk.cpp", tmp_path / "walk"
    src.write_text(WALK)
    inc = os.path.join(ROOT, "paper_2204_04179_amd", "csrc")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-I", inc, str(src), "-o", str(exe)])
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
    widths, items = (8, 64, 72, 136, 264, 1536), (1, 2, 31, 32, 33, 63, 64, 65, 100, 127, 128, 129, 300, 1000, 1281)
    assert int(out.stdout) == 2 * sum(u * k // 8 for u in items for k in widths)      # every chunk of the items' rows, once


def test_the_kernel_uses_these_functions():
    with open(os.path.join(ROOT, "paper_2204_04179_amd", "csrc", "gram_gemm.hip")) as f:
        src = f.read()
    body = src[src.index("void encode_mid_tile("):src.index("// ---- C[M,N] = A[M,K] . B[N,K]^T")]
    assert "uniq[jj]" in body and "zero_ids[jj]" in body and "jj = mid_list_entry(" in body
    assert body.count("mid_row_offset(") == 1 and body.count("mid_slab_offset(") == 1
    assert "rows_max" not in body          # the only bound is the number of items on the device


def test_the_kernel_of_square_tiles_uses_them_too():
    with open(os.path.join(ROOT, "paper_2204_04179_amd", "csrc", "gram_gemm.hip")) as f:
        src = f.read()
    body = src[src.index("void k_encode_square("):src.index("// How many row tiles of 256 are taken whole.")]
    assert "uniq[j]" in body and "zero_ids[j]" in body and "j = mid_list_entry(" in body
    assert body.count("mid_row_offset(") == 1 and body.count("mid_slab_offset(") == 1
    assert "rows_max" not in body
    # every load's offset is the lane's own, which the range check covers
    loads = [line for line in body.splitlines() if "load_to_lds(" in line]
    assert len(loads) == 2 and all(", 0u, to_" in line for line in loads)
