"""Dispatch rules that need only sizes (csrc/fn_rules.h), compiled with the host
compiler and checked over their ranges."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2401_10287_amd", "csrc")


def _run(tmp_path, body):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    src, exe = tmp_path / "rules.cc", tmp_path / "rules"
    src.write_text('#include <stdio.h>\n#include "fn_rules.h"\nusing namespace fn;\nint main()\n{\n%s\nreturn 0;\n}\n' % body)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    return [[int(v) for v in line.split()] for line in subprocess.run([str(exe)], check=True, capture_output=True,
                                                                      text=True).stdout.splitlines()]


def test_weight_gradient_splits(tmp_path):
    """A wave's FP32 sum (a quarter of a split's rows) runs over at most 512 rows, or,
    where the 64 splits of the partial sums' buffer (32 for the product that forms two
    weight blocks) do not reach, over no more than 1/64 of the rows, at every width."""
    out = _run(tmp_path, """
    const int rows[] = {1, 7, 255, 256, 300, 2048, 2049, 5000, 8192, 12345, 32768, 32769, 49152, 81920, 163840, 1000003};
    const int widths[] = {32, 64, 256, 384, 512, 1024};
    for (int R : rows)
        for (int w : widths)
            for (int tile = 32; tile <= 64; tile *= 2)
                for (int two = 1; two <= 2; ++two) {
                    const int n = (w + tile - 1) / tile, tiles = two * n * n;
                    printf("%d %d %d\\n", R, tiles, (int)tn_product_splits(R, tiles, 64 / two));
                }""")
    assert len(out) == 16 * 24
    for rows, tiles, splits in out:
        assert 1 <= splits <= 64
        wave = -(-(-(-rows // splits)) // 4)
        assert wave <= max(512, -(-rows // 64)), (rows, tiles, splits)


def test_weight_gradient_workgroups(tmp_path):
    """Every (split, tile) has one workgroup, and of the eight XCDs, to which workgroups
    are dealt in turn, none has more than 1.8 times its share (nine splits: two on one),
    unless it has a workgroup per CU at most."""
    out = _run(tmp_path, """
    const int tiles[] = {1, 3, 16, 32, 33, 64, 256, 512};
    const int splits[] = {1, 2, 3, 4, 5, 7, 8, 9, 13, 16, 25, 64};
    for (int t : tiles)
        for (int S : splits)
            for (int b = 0; b < tn_grid(S, t); ++b)
                printf("%d %d %d %d %d\\n", t, S, b % 8, tn_block(b, S, t).sp, tn_block(b, S, t).tile);""")
    cases = {}
    for t, s, xcd, sp, tile in out:
        if sp < s and tile < t:
            cases.setdefault((t, s), []).append((xcd, sp, tile))
    assert len(cases) == 96
    for (t, s), work in cases.items():
        assert sorted(w[1:] for w in work) == [(sp, tile) for sp in range(s) for tile in range(t)]
        per = [sum(w[0] == x for w in work) for x in range(8)]
        assert max(per) <= max(32, 1.8 * s * t / 8 + 1), (t, s, per)


def test_determinant_kernel_choice(tmp_path):
    """The direction-per-lane kernel where it was measured to be the faster one, the wave
    per determinant elsewhere: (electrons of the spin, of both, nuclei, FP64, lanes)."""
    cases = [(2, 4, 1, 0, 0), (3, 3, 32, 0, 1), (7, 7, 32, 0, 1), (8, 8, 2, 0, 0), (8, 10, 20, 0, 0), (8, 10, 1, 0, 1),
             (8, 15, 20, 0, 1), (9, 9, 1, 0, 0), (9, 11, 2, 0, 0), (9, 12, 2, 0, 1), (9, 12, 20, 0, 0), (9, 18, 20, 0, 1),
             (10, 10, 2, 0, 1), (10, 10, 20, 0, 0), (10, 12, 32, 0, 0), (10, 20, 20, 0, 1), (11, 20, 2, 0, 0),
             (8, 8, 20, 1, 1), (10, 10, 32, 1, 1), (11, 11, 2, 1, 0)]
    out = _run(tmp_path, "\n".join('printf("%%d\\n", (int)det_lanes_fl(%d, %d, %d, %d));' % c[:4] for c in cases))
    assert [v[0] for v in out] == [c[4] for c in cases]


def test_walking_layer_batches(tmp_path):
    """The walking stream layer only for batches where it was measured to be the faster
    one: (walkers, walkers of a round, 16-row blocks of an electron, six products, walks)."""
    cases = [(141, 256, 3, 0, 1), (140, 256, 3, 0, 0), (300, 256, 3, 0, 1), (218, 256, 2, 0, 1), (217, 256, 2, 0, 0),
             (300, 256, 2, 0, 0), (4096, 256, 4, 0, 1), (72, 128, 3, 1, 0), (82, 128, 3, 1, 1), (143, 128, 3, 1, 1),
             (72, 128, 4, 1, 0), (85, 128, 4, 1, 0), (92, 128, 4, 1, 1), (128, 128, 4, 1, 1), (143, 128, 4, 1, 0),
             (154, 128, 4, 1, 1), (1000, 128, 4, 1, 1), (1024, 128, 2, 1, 0)]
    out = _run(tmp_path, "\n".join('printf("%%d\\n", (int)walk_batch(%d, %d, %d, %d));' % c[:4] for c in cases))
    assert [v[0] for v in out] == [c[4] for c in cases]
