"""Which product the planner takes, by default and with its tuning variables (host only)."""
from tests import planner as PL


def ladder(G, a, c, i, dtype=PL.F32, compute="bf16x3", **kw):
    """G x (G a^2 x G c^2 x G i0 i1) of abcd,cdij->abij."""
    return PL.line("abcd,cdij->abij", (G,), "++--", (a, a, c, c), "++--", (c, c) + i, dtype, compute, **kw)


def test_wide_split_bf16_tiles_where_they_were_measured_faster():
    # (product, columns of the tile, 0 for the plan's own product)
    cases = [(ladder(8, 24, 24, (6, 6)), 288),            # 553 us on the plan's own product, 407 on the tile
             (ladder(12, 24, 24, (6, 6)), 288),           # 2284, 1779
             (ladder(8, 24, 24, (5, 5)), 224),            # 556, 348
             (ladder(8, 24, 24, (4, 6)), 192),            # 518, 332
             (ladder(8, 32, 32, (8, 8)), 0),              # 1555, 1753
             (PL.line("abcd,cdij->abij", (8,), "++--", (37, 40, 12, 8), "++--", (12, 8, 4, 7), PL.F32, "bf16x3"), 0),   # 184, 225
             (PL.line("abcd,cdij->abij", (12,), "++--", (19, 32, 4, 4), "++--", (4, 4, 3, 8), PL.F32, "bf16x3"), 0),    # 133, 156
             (PL.line("abcd,cdij->abij", (8,), "++--", (26, 33, 10, 8), "++--", (10, 8, 4, 7), PL.F32, "bf16x3"), 0),   # 115, 149
             (ladder(8, 24, 0, (6, 6)), 0)]               # no contracted index at all
    got = PL.plans([ln for ln, _ in cases])
    assert [p["wide_bn"] for p in got] == [bn for _, bn in cases]
