"""What the 256-row contraction asks memory for along K, walked on the CPU with the very functions the kernel forms its
addresses with (csrc/gram_mid_rows.h, compiled by the host compiler).  A caller's matrix of hidden activations may end with the
items' rows, and features and weights end where they end: no slab reads behind a row, and what the slabs multiply is every
element of K once, in order."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

WALK = r"""
#include <cstdio>
#include "gram_mid_rows.h"
using namespace gram;
int main()
{
    long reads = 0;
    for (int k = 32; k <= 1664; k += 32) {
        const int slabs = (k + kBigSlab - 1) / kBigSlab;
        int next = 0;                                   // element of K that is to be multiplied next
        for (int slab = 0; slab < slabs + 3; ++slab) {  // and the slabs past the end
            const int k0 = big_slab_start(slab < slabs ? slab : slabs - 1, k);
            for (int chunk = 0; chunk < 8; ++chunk) {   // chunks of 8 elements: rows of A, and of a K-contiguous B
                const int at = k0 + big_slab_part(chunk, 8, k) * 8;
                if (at < 0 || at + 8 > k) return std::printf("K %d slab %d chunk %d: element %d\n", k, slab, chunk, at), 1;
                ++reads;
            }
            for (int row = 0; row < kBigSlab; ++row) {  // rows of W [k, n]
                // (a lane of a wave loads row 8 wave + {0 .. 3} and, by the same offset, the one four below)
                const int at = k0 + big_slab_part(row & ~4, 1, k) + (row & 4);
                if (at < 0 || at >= k) return std::printf("K %d slab %d row %d: row %d\n", k, slab, row, at), 2;
            }
            if (slab >= slabs) continue;
            for (int step = 0; step < (slab == big_half_slab(k) ? 32 : 64); step += 8, next += 8) {
                if (k0 + big_slab_part(step / 8, 8, k) * 8 != next) return std::printf("K %d slab %d step %d\n", k, slab, step), 3;
                for (int i = 0; i < 8; ++i)
                    if (k0 + big_slab_part((step + i) & ~4, 1, k) + ((step + i) & 4) != next + i) return 4;
            }
        }
        if (next != k) return std::printf("K %d: %d multiplied\n", k, next), 5;
    }
    std::printf("%ld\n", reads);
    return 0;
}
"""


def _tile_source():
    with open(os.path.join(ROOT, "paper_2204_04179_amd", "csrc", "gram_gemm.hip")) as f:
        src = f.read()
    return src[src.index("void gemm_nt_tile("):src.index("// One tile per block, of 256 rows or")]


def test_nothing_behind_k_is_read(tmp_path):
    src, exe = tmp_path / "walk.cpp", tmp_path / "walk"
    src.write_text(WALK)
    inc = os.path.join(ROOT, "paper_2204_04179_amd", "csrc")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-I", inc, str(src), "-o", str(exe)])
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
    assert int(out.stdout) == sum(((k + 63) // 64 + 3) * 8 for k in range(32, 1665, 32))


def test_the_kernel_uses_these_functions():
    body = _tile_source()
    assert body.count("big_slab_start(") == 2 and body.count("big_slab_part(") == 3 and body.count("big_half_slab(") == 1
    # the offsets of a load: the lane's, which big_slab_part enters, and the slab's start, nothing else along K
    loads = body[body.index("#define GRAM_LOAD_A("):body.index("#define GRAM_READ_A(")]
    assert "TK" not in loads and "load_to_lds(rs_, oa[H][g_], so_," in loads and "load_to_lds(pa[H][g_] + k_," in loads


def test_the_epilogue_waits_for_every_load_to_its_stages():
    """The stages of the main loop become the epilogue's: each wave has waited for all its loads to them before its last
    barrier of the loop, whatever else it has requested since."""
    body = _tile_source()
    slab = body[body.index("#define GRAM_SLAB("):body.index("// (subtracting) the targets")]
    # subtracting, last slab: wait for all, then the targets, and no load to the stages behind that
    at = slab.index("if (epi_subtracts(EPI) && (SL) == last) {")
    end = slab.index("} else {", at)
    assert slab.index("wait_loads<0>();", at) < slab.index("GRAM_AUX(0)", at) < end
    assert "GRAM_LOAD" not in slab[at:end] and "GRAM_LOAD" not in slab[slab.index("wait_lds();", end):]
    # the other forms: wait for all behind the loop
    tail = body[body.index("if (sl == last) GRAM_SLAB("):]
    assert tail.index("if (!epi_subtracts(EPI)) wait_loads<0>();") < tail.index("__syncthreads()") and "wait_loads<" not in tail[tail.index("__syncthreads()"):]


def test_stores_are_bounded_by_their_own_offset():
    """The range check of a raw buffer access is only sure to cover the lane's offset, so the row of a store or of the
    activation beside it stands in that, and the scalar offset is zero."""
    import re
    body = _tile_source()
    calls = re.findall(r"raw_buffer_(?:load|store)_b32\((.*)\);", body)
    assert len(calls) == 3
    for args in calls:
        assert re.search(r"rs[CX], below\(at\[j\], .*\), 0, 0$", args), args
    assert body.count("add_sat(from, ") == 2
