"""Writes choice_table.h: the library's measured configuration choice, distilled
from the tuner database shipped with the package, in two tables: one for rows that are
no whole 16-byte loads (FP64: n, lda or ldb odd; FP32: not multiples of 4; the direct-load
configurations had three stages when the database was measured and took only whole
ones), one for rows that are (consulted by the library only where its preference list
names a two-stage configuration).

For each dtype, row class and cell (floor(log2 m), floor(log2 n), floor(log2 k)) with
m, n, k in [64, 16384], the cell's configuration is the registered one with the
highest weighted mean log relative speed (TFLOP/s over the shape's best) over the
database's training shapes (the tuner's 'train', 'train2' and 'aligned' sets) of that class in
the cell (weight 1) and in the 26 cells around it (weight NEIGHBOUR_WEIGHT: a cell
holds only a few shapes of a class, and speeds change smoothly from one octave to
the next); the held-out shapes stay out, so they can score the table.  Run from the
repository root:

    python -m paper_1706_10086_amd.csrc.gen_choice_table
"""
from __future__ import annotations

import collections
import math
import os

HERE = os.path.dirname(os.path.abspath(__file__))
OUT = os.path.join(HERE, "choice_table.h")
LO, HI = 6, 14          # log2 range of the table's cells (m, n, k in [64, 16384])


def three_stage_ineligible(dtype: int, n: int, k: int) -> bool:
    """Rows of A (lda = k) or B (ldb = n) that are not whole 16-byte loads."""
    epu = 2 if dtype == 0 else 4
    return n % epu != 0 or k % epu != 0


def cell_of(m: int, n: int, k: int):
    return tuple(int(math.floor(math.log2(x))) for x in (m, n, k))


def registered_configs() -> dict:
    """{dtype: set of configuration tuples} the library registers: the hand
    entries of gemm_tiled.hip and the tuning-grid selection (gen_grid)."""
    from paper_1706_10086_amd.csrc import gen_grid
    return {dt: gen_grid.hand_configs(dt) | set(gen_grid.selection(dt)) for dt in (0, 1)}


NEIGHBOUR_WEIGHT = 0.5


def build_table(records, train_shapes, whole_rows: bool = False, allowed=None):
    """{dtype: {cell: cfg tuple}} from compact-database records, for shapes whose
    rows are (whole_rows) or are not whole 16-byte loads; only
    configurations in ``allowed[dtype]`` (default: the registered ones) measured on
    every such training shape compete."""
    import itertools
    allowed = registered_configs() if allowed is None else allowed
    per_shape = collections.defaultdict(dict)
    for r in records:
        if tuple(r["cfg"]) not in allowed.get(r["dtype"], ()):
            continue
        per_shape[(r["dtype"], r["m"], r["n"], r["k"])][tuple(r["cfg"])] = r["tflops"]
    # per dtype and cell: summed log relative speeds and shape counts per configuration
    sums = collections.defaultdict(lambda: collections.defaultdict(lambda: [0.0, 0]))
    for (dt, m, n, k), v in per_shape.items():
        if (m, n, k) not in train_shapes or three_stage_ineligible(dt, n, k) == whole_rows:
            continue
        best = max(v.values())
        acc = sums[(dt, cell_of(m, n, k))]
        for cfg, t in v.items():
            acc[cfg][0] += math.log(t / best)
            acc[cfg][1] += 1
    table = collections.defaultdict(dict)
    for dt in sorted({d for d, _ in sums}):
        for cell in itertools.product(range(LO, HI + 1), repeat=3):
            tot = collections.defaultdict(lambda: [0.0, 0.0])
            shapes = 0.0
            for d in itertools.product((-1, 0, 1), repeat=3):
                nb = (dt, tuple(a + b for a, b in zip(cell, d)))
                if nb not in sums:
                    continue
                w = 1.0 if d == (0, 0, 0) else NEIGHBOUR_WEIGHT
                nmax = max(x[1] for x in sums[nb].values())
                shapes += w * nmax
                for cfg, (lsum, cnt) in sums[nb].items():
                    tot[cfg][0] += w * lsum
                    tot[cfg][1] += w * cnt
            if shapes == 0:
                continue
            # only configurations measured on every shape around the cell compete
            cand = [(x[0] / x[1], cfg) for cfg, x in tot.items() if x[1] >= shapes - 1e-9]
            if cand:
                table[dt][cell] = max(cand)[1]
    return table


def build_tables(records, train_shapes):
    allowed = registered_configs()
    return {w: build_table(records, train_shapes, bool(w), allowed) for w in (0, 1)}


def training_shapes() -> set:
    """The database's training shapes: the tuner's 'train', 'train2' and 'aligned'
    sets."""
    from paper_1706_10086_amd import tune
    return set(tune.shape_set("train")) | set(tune.shape_set("train2")) | \
        set(tune.shape_set("aligned"))


def render(tables) -> str:
    """tables: {whole_rows (0/1): {dtype: {cell: cfg}}}."""
    lines = [
        "// Generated by gen_choice_table.py from data/tune_db.json.gz; do not edit.",
        "// Measured configuration choice per (dtype, rows16, floor(log2 m), floor(log2 n),",
        f"// floor(log2 k)) cell, m, n, k in [{2 ** LO}, {2 ** HI}]; rows16: whether the rows",
        "// are whole 16-byte loads.  Each cell names the configuration measured fastest",
        "// on the tuner's shapes of that class in and around the cell (weighted mean log",
        "// relative speed).",
        "#pragma once",
        "#include <stdint.h>",
        "",
        "namespace mgemm {",
        "",
        "struct ChoiceCell {",
        "    int8_t dtype, rows16, lm, ln, lk;",
        "    int16_t bm, bn, bk, waves, ept, dbuf, occ;",
        "};",
        "",
        f"constexpr int CHOICE_LOG2_LO = {LO};",
        f"constexpr int CHOICE_LOG2_HI = {HI};",
        "",
        "static const ChoiceCell kChoiceCells[] = {",
    ]
    count = 0
    for dt in (0, 1):
        for w in (0, 1):
            for (lm, ln, lk), c in sorted(tables[w].get(dt, {}).items()):
                lines.append("    {%d, %d, %d, %d, %d, %d, %d, %d, %d, %d, %d, %d}," %
                             ((dt, w, lm, ln, lk) + c))
                count += 1
    lines += ["};", "", f"constexpr int CHOICE_CELLS = {count};", "", "}  // namespace mgemm", ""]
    return "\n".join(lines)


def main() -> None:
    from paper_1706_10086_amd import tune
    db = tune.load_compact(os.path.join(os.path.dirname(HERE), "data", "tune_db.json.gz"))
    text = render(build_tables(db.records, training_shapes()))
    with open(OUT, "w") as f:
        f.write(text)
    print(f"wrote {OUT}")


if __name__ == "__main__":
    main()
