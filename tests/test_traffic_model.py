"""The per-cell access counts printed in the paper's Table
tab:memory_references (Section 4.1) reproduced by the traffic formulas."""
import itertools
import os
import re

import pytest

from paper_2510_00998_amd import traffic

GOLDEN = os.path.join(os.path.dirname(__file__), "golden", "memory_references.txt")


def _rows():
    out = {}
    for line in open(GOLDEN):
        line = line.strip()
        if not line or line.startswith("#"):
            continue
        parts = line.split()
        out[(int(parts[0]), parts[1])] = [float(x) for x in parts[2:]]
    return out


@pytest.mark.parametrize("d", [2, 3])
def test_table_counts(d):
    rows = _rows()
    for i, p in enumerate(range(1, 11)):
        assert traffic.words_vanilla(d, p) == rows[(d, "vanilla")][i]
        assert traffic.words_facet(d, p) == rows[(d, "facet")][i]
        assert traffic.words_facet_exit(d, p) == rows[(d, "facet_exit")][i]
        r = traffic.words_vanilla(d, p) / traffic.words_facet(d, p)
        assert abs(r - rows[(d, "reduction")][i]) <= 0.0051
        r = traffic.words_vanilla(d, p) / traffic.words_facet_exit(d, p)
        assert abs(r - rows[(d, "reduction_exit")][i]) <= 0.0051


def test_exact_sweep_bytes_tends_to_per_cell_model():
    # interior cells dominate for large n: bytes/cell -> words_fused_sweep
    d, p, n = 3, 4, 400
    per_cell = traffic.sweep_bytes(d, n, p, 1) / n ** d
    assert abs(per_cell / traffic.words_fused_sweep(d, p) - 1) < 0.01
    # 32^3, Q4, FP64: 3 * 4.096e6 * 8 B of cell data + 95232 facets * 200 words * 8 B
    assert traffic.sweep_bytes(3, 32, 4, 8) == (3 * 32 ** 3 * 125 + 3 * 32 * 32 * 31 * 200) * 8


HEADER = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2510_00998_amd", "csrc",
                      "dg_kernels.hpp")


def test_block_tables_are_the_kernels():
    src = open(HEADER).read()
    cpp = {}
    for key, row in re.findall(r"(case \d+|default): return ([^;]*);", src.split("constexpr Brick brick(")[1]
                               .split("\n}")[0]):
        br = [tuple(int(v) for v in b.split(",")) for b in re.findall(r"Brick\{([^}]*)\}", row)]
        p = 8 if key == "default" else int(key.split()[1]) - 1
        if len(br) == 1:
            cpp[p] = (br[0],) * 3
        else:
            half_only = row.startswith("V == 1 ?")  # else V == 0 ? full : other
            assert half_only or row.startswith("V == 0 ?")
            cpp[p] = (br[1], br[0], br[1]) if half_only else (br[0], br[1], br[1])
    assert cpp == traffic.BRICKS
    rows = re.search(r"line\[2\]\[8\] = \{\{([^}]*)\}, \{([^}]*)\}\}", src)
    for size, row in zip((4, 8), rows.groups()):
        assert tuple(eval(v) for v in row.split(",")) == traffic.RUN_BRICKS[size]


def _exchanged_by_walking(n, brick):
    """Facets between two bricks, counted cell by cell."""
    count = 0
    for x in itertools.product(range(n), repeat=3):
        for k in range(3):
            if x[k] + 1 < n and x[k] // brick[k] != (x[k] + 1) // brick[k]:
                count += 1
    return count


@pytest.mark.parametrize("p,n", [(1, 9), (2, 7), (4, 11), (5, 8), (8, 6)])
@pytest.mark.parametrize("shape", [0, 1, 2, 3])
def test_exchanged_facets(p, n, shape):
    brick = (1, 1, 1) if shape == 3 else traffic.BRICKS[p][shape]
    assert traffic.exchanged_facets(3, n, p, shape) == _exchanged_by_walking(n, brick)


def test_moved_bytes():
    # Q4 32^3 in bricks of 5 x 2 x 2: 32^2 (6 + 15 + 15) facets of 50 values a side, written and read
    f = 32 * 32 * 36
    cells = 32 ** 3 * 125
    assert traffic.sweep_bytes(3, 32, 4, 8, moved=True) == (3 * cells + f * 200) * 8
    assert traffic.project_bytes(3, 32, 4, 8, moved=True) == (cells + f * 100) * 8
    assert traffic.apply_bytes(3, 32, 4, 8, moved=True) == (2 * cells + f * 100) * 8
    # runs of cells (2D, 16-bit storage, small meshes) exchange every facet
    for d, n, p, size in ((2, 64, 3, 8), (3, 48, 5, 2), (3, 8, 4, 8)):
        assert traffic.sweep_bytes(d, n, p, size, moved=True) == traffic.sweep_bytes(d, n, p, size)
    # a batch's half bricks
    half = {4: 1}
    f = 32 * 32 * (6 + 15 + 31)
    assert traffic.sweep_bytes(3, 32, 4, 8, moved=True, shapes=half) == (3 * cells + f * 200) * 8
    assert traffic.vcycle_bytes(3, 32, 4, 4, moved=True) < traffic.vcycle_bytes(3, 32, 4, 4)
