"""The matrix-core column kernels in the library are those that a plan can reach.

They are built per (log2 of the rows, steps of four sources). A plan is accepted when the
scalar form's staging of its digits fits the 160 KB of LDS, count * 2^log_r * 64 * 8 bytes,
and the matrix form takes 4 sources and more, up to 32.
"""
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_column_kernels_built_and_reachable():
    with open(os.path.join(ROOT, "paper_2603_16692_amd", "libks.so"), "rb") as f:
        names = f.read()
    # the flag forces the matrix form for fewer sources too, hence from one on
    reach = {(log_r, -(-count // 4)) for log_r in range(6) for count in range(1, 33)
             if count * (1 << log_r) * 64 * 8 <= 160 * 1024}
    for kernel in (b"k_modup_cols_mx", b"k_moddown_cols_mx"):
        built = {(int(r), int(nm)) for r, nm in re.findall(kernel + rb"ILi(\d+)ELi(\d+)E", names)}
        assert built == reach, (kernel, sorted(built - reach), sorted(reach - built))
