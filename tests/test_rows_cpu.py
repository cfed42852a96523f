"""Row arithmetic of the kernels, compiled for the host: what a wavefront that summarises several small blocks reads lies in the rows
of its own blocks, also where the sequence is longer than the cache has blocks for or where its range of blocks ends early."""
import ctypes
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2512_02337_amd", "csrc")


def test_rows_of_small_blocks(tmp_path):
    src = tmp_path / "rows.cpp"
    src.write_text('#include "rows.h"\nextern "C" int row(int t, int L, int end, int B) { return specpv::row_below(t, L, end, B); }\n')
    lib = str(tmp_path / "rows.so")
    subprocess.run(["g++", "-shared", "-fPIC", "-O1", "-I" + CSRC, str(src), "-o", lib], check=True)
    row = ctypes.CDLL(lib).row
    for B, per in ((16, 4), (32, 2), (8, 4), (64, 2)):   # rows of a block, blocks of a wavefront
        for max_blocks in (1, 2, 3, 5, 8):
            for L in sorted({1, B - 1, B, B + 1, max_blocks * B - 1, max_blocks * B, max_blocks * B + 1, (max_blocks + 3) * B, (max_blocks + 9) * B + 5}):
                nb = min((L + B - 1) // B, max_blocks)
                for end in range(1, nb + 1):
                    for i0 in range(end):
                        for x in range(per * B):
                            r = row(i0 * B + x, L, end, B)
                            assert i0 * B <= r < min(L, end * B)
                            if x < B * min(per, end - i0) and i0 * B + x < L:
                                assert r == i0 * B + x
    # the largest cache
    assert row((1 << 30) + 7, 2 ** 31 - 1, 1 << 26, 16) == (1 << 30) - 1
    # and the kernel goes by it
    text = open(os.path.join(CSRC, "summarize.h")).read()
    body = text[text.index("void summarize_small("):]
    assert body.count("load_keys<") == 1 and "row_below(t0 + x * RPP + rsub, L, end, N * RPP)" in body[body.index("load_keys<"):]
