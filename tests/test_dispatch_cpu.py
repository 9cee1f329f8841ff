"""Which product the planner takes, by default and with its tuning variables (host only)."""
import random

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


def test_in_place_and_steps_share_k_out_alike():
    # stream-K cuts K where its tile, its loads' width and its workgroups per CU say: the three
    # steps must have the in-place product's, so that both sum the same ranges
    rng = random.Random(11)
    forms = [("abcd,cdij->abij", "++--", "++--"), ("klab,klij->abij", "--++", "++--"), ("ak,kb->ab", "+-", "+-"),
             ("ka,kb->ab", "-+", "+-"), ("abk,ki->abi", "++-", "+-"), ("ak,ik->ai", "+-", "-+")]
    # (two that ran 128 x 64 in place against 96 x 96 in steps, then random ones)
    cases = [("abcd,cdij->abij", (8,), "++--", (25, 9, 15, 20), "++--", (15, 20, 3, 3), PL.F64, "f64"),
             ("abcd,cdij->abij", (8,), "++--", (3, 4, 16, 14), "++--", (16, 14, 29, 6), PL.F32, "f32")]
    for _ in range(3000):
        sub, su, sv = rng.choice(forms)
        tu, tv = sub.split("->")[0].split(",")
        pair = len(tu) == 2
        d = {c: rng.randint(1, 900) if pair and rng.random() < .7 else 4 * rng.randint(1, 250) if pair
             else rng.choice([rng.randint(1, 40), 2 * rng.randint(1, 20)]) for c in dict.fromkeys(tu + tv)}
        dt, comp = rng.choice([(PL.F64, "f64"), (PL.F32, "f32"), (PL.C128, "f64"), (PL.C64, "f32"), (PL.F32, "bf16x3")])
        cases.append((sub, (rng.choice([1, 2, 3, 4, 6, 8]),), su, tuple(d[c] for c in tu), sv, tuple(d[c] for c in tv), dt,
                      comp))
    got = PL.plans([PL.line(*c) for c in cases] + [PL.line(*c, steps=True) for c in cases])
    cut = 0
    for c, a, b in zip(cases, got, got[len(cases):]):
        if a["any"] < 0 or a["wide_bn"]:
            continue
        # a tile's launch takes 128 x 64 where the first one has no kernel for 4-byte loads
        def runs(p):
            tile = p["any"] if p["ch16"] else max(p["any"], 1)
            wgs = 3 if tile == 2 else 2 if c[-1] == "bf16x3" or (tile == 1 and not p["ch16"]) else 3
            return tile, wgs
        assert a["ch16"] or a["any"] > 0, c               # the planner's choice is the tile that runs
        assert a["sk"] == b["sk"] and a["chunk"] == b["chunk"] and a["any"] == b["any"], c
        if a["sk"]:
            cut += 1
            assert runs(a) == runs(b), c
    assert cut > 100


def test_tile_names_that_restrict_nothing():
    # an unknown or empty name, or one of another compute mode's tiles, leaves the default choice
    mm = lambda dt, comp, G=8, M=500, K=1000, N=600: PL.line("ak,kb->ab", (G,), "+-", (M, K), "++", (K, N), dt, comp)
    f64 = [mm(PL.F64, "f64", 9, 500, 500, 500), mm(PL.C128, "f64"), mm(PL.C64, "f32")]
    bf = [ladder(8, 24, 24, (6, 6)), mm(PL.F32, "bf16x3"), ladder(2, 9, 5, (3, 4))]
    want, want_bf = PL.plans(f64), PL.plans(bf)
    assert all(p["any"] >= 0 for p in want) and want_bf[0]["wide_bn"] and all(p["any"] >= 0 for p in want_bf[1:])
    for name in ("", "no-such-tile", "bw256x288sk", "a128x128s2"):
        assert PL.plans(f64, SYMT_GEMM_TILE=name) == want, name
    for name in ("", "no-such-tile", "a96x96s2", "d96x96s2", "tallk"):
        assert [(p["any"], p["wide_bn"]) for p in PL.plans(bf, SYMT_GEMM_TILE=name)] == \
            [(p["any"], p["wide_bn"]) for p in want_bf], name
    # names of other tiles of the same compute mode keep these products out
    for name in ("96x96", "d128x128s2", "rows", "tallk"):
        assert all(p["any"] < 0 for p in PL.plans(f64, SYMT_GEMM_TILE=name)), name
    for name in ("b128x128k32", "bd128x256s3", "bw256x256s2"):
        assert all(p["any"] < 0 and not p["wide_bn"] for p in PL.plans(bf, SYMT_GEMM_TILE=name)), name


def test_complex_products_stay_where_in_place_was_measured_slower():
    # (G, contracted blocks, u's other blocks, v's other blocks): the in-place product, or not
    km = lambda G, kl, ab, ij, dt: PL.line("klab,klij->abij", (G,), "--++", kl + ab, "++--", kl + ij, dt,
                                           "f32" if dt == PL.C64 else "f64")
    ak = lambda G, kl, ab, ij, dt: PL.line("abkl,klij->abij", (G,), "++--", ab + kl, "++--", kl + ij, dt,
                                           "f32" if dt == PL.C64 else "f64")
    slower = [km(6, (2, 16), (44, 36), (8, 38), PL.C64),      # 1471 us before, 1616 in place
              km(4, (4, 8), (38, 32), (48, 37), PL.C64),      # 1383, 1533
              km(4, (16, 20), (39, 20), (24, 40), PL.C128)]   # 7782, 8283
    faster = [km(3, (16, 20), (20, 12), (13, 10), PL.C64),    # 3 x (720 x 1920 x 780): 156, 112
              ak(2, (4, 8), (27, 11), (26, 43), PL.C64),      # 2 x (594 x 128 x 4472): 47, 26
              ak(2, (4, 8), (27, 11), (26, 43), PL.C128)]     # 56, 38
    assert [p["any"] >= 0 for p in PL.plans(slower + faster)] == [False] * 3 + [True] * 3


def test_split_bf16_products_take_planes_or_in_place_as_measured():
    # (layout, G, M, K, N): us on planes, us on the in-place or wide tile
    planes = [("ak", 4, 7937, 160, 1613),     # 149, 198 (in place)
              ("ak", 16, 4096, 128, 449),     # 93, 113
              ("ka", 16, 1940, 96, 1405),     # 129, 155
              ("ak", 4, 3648, 32, 2970),      # 90, 238 (256-column tiles under stream-K)
              ("ak", 16, 2592, 256, 1631),    # 274, 412
              ("ak", 8, 7840, 256, 2963)]     # 683, 946
    in_place = [("ak", 4, 958, 199, 1701),    # 88, 42
                ("ak", 2, 3072, 174, 1363),   # 103, 50
                ("ak", 4, 2011, 193, 1472),   # 100, 61
                ("ka", 4, 2848, 416, 576),    # 91, 41
                ("ka", 16, 128, 64, 176128)]  # 1207, 804
    def line(form, G, M, K, N):
        return PL.line("ak,kb->ab" if form == "ak" else "ka,kb->ab", (G,), "+-" if form == "ak" else "-+",
                       (M, K) if form == "ak" else (K, M), "++", (K, N), PL.F32, "bf16x3")
    got = PL.plans([line(*c) for c in planes + in_place])
    assert [(p["any"] >= 0, p["wide_bn"]) for p in got] == [(False, 0)] * len(planes) + [(True, 0)] * len(in_place)


ROWS = 64     # GemmChoice::tile of the row-streaming product


def test_rows_along_n_where_w_is_contiguous():
    def line(sub, su, sv, G, d, dt):
        tu, tv = sub.split("->")[0].split(",")
        return PL.line(sub, (G,), su, [d[c] for c in tu], sv, [d[c] for c in tv], dt, "f64" if dt in (PL.F64, PL.C128) else "f32")
    # (us on tiles, us on rows)
    rows = [line("ak,kb->ab", "+-", "++", 4, dict(a=32, k=32, b=524288), PL.F32),           # 255, 111
            line("ka,bk->ba", "-+", "++", 6, dict(a=29, k=55, b=381895), PL.F64),           # 786, 354
            line("ak,kb->ba", "+-", "++", 1, dict(a=23, k=7, b=361591), PL.F32)]            # 42, 18
    tiles = [line("ka,ijk->jai", "-+", "+++", 8, dict(a=63, k=63, i=337, j=72), PL.F32),    # 969, 1441
             line("ka,ijk->jai", "-+", "+++", 6, dict(a=32, k=33, i=172, j=45), PL.F64),    # 94, 121
             line("ak,kb->ba", "+-", "++", 4, dict(a=51, k=57, b=168664), PL.F32),          # 154, 193
             line("ak,kb->ab", "+-", "++", 4, dict(a=47, k=26, b=207855), PL.C64),          # 448, 700
             line("ak,kb->ab", "+-", "++", 6, dict(a=62, k=16, b=389338), PL.C128)]         # 1691, 1897
    got = PL.plans(rows + tiles)
    assert [p["tile"] == ROWS for p in got] == [True] * len(rows) + [False] * len(tiles)
    # the three steps take the same product
    steps = PL.plans([ln.rsplit(" ", 1)[0] + " " + str(int(ln.rsplit(" ", 1)[1]) | PL.STEPS) for ln in rows + tiles])
    assert [p["tile"] for p in steps] == [p["tile"] for p in got]
    # (many columns of few rows stay off the in-place tiles as well: 2916 us, 4493)
    few, = PL.plans([line("ak,ijkl->aijl", "+-", "++++", 6, dict(a=7, k=8, i=25, j=129, l=23), PL.C64)])
    assert few["tile"] != ROWS and few["any"] < 0


TALLK = 65    # GemmChoice::tile of the long-K product


def test_the_gpu_tests_reach_their_kernels():
    """Forced names that do not apply are ignored, and the GPU tests of a kernel then pass on
    another: the planner takes each of their cases as they mean it."""
    from tests import test_gpu_any as any_layout
    from tests import test_gpu_rows_swapped as rows
    from tests import test_gpu_subgroup_direct as subgroup
    from tests import test_gpu_tallk_vec as tallk
    from tests import test_gpu_wide_sk as wide
    real, every = ((PL.F64, "f64"), (PL.F32, "f32")), ((PL.F64, "f64"), (PL.F32, "f32"), (PL.C128, "f64"), (PL.C64, "f32"))

    def lines(cases, dt, comp):
        return [PL.line(sub, g, cu, du, cv, dv, dt, comp) for sub, g, cu, cv, du, dv in cases]
    for sk in ("0", "1"):
        layouts = set()
        for i, tile in enumerate(("a96x96s2", "a128x64s2", "a64x64s2")):
            for dt, comp in every:
                got = PL.plans(lines(any_layout.CASES, dt, comp), SYMT_GEMM_TILE=tile, SYMT_GEMM_SK=sk)
                # (without whole 16-byte chunks the first tile's launch runs the second)
                assert [p["any"] for p in got] == [i if p["ch16"] else max(i, 1) for p in got], (tile, dt, sk)
                layouts |= {(p["am"], p["cb"], p["ch16"]) for p in got}
        assert layouts >= {(0, 0, 0), (0, 0, 1), (1, 0, 0), (1, 0, 1), (0, 1, 1), (2, 1, 0), (2, 1, 1)}
        for i, tile in enumerate(("a128x128s2", "a128x64s2", "a64x64s2")):
            got = PL.plans(lines(any_layout.CASES, PL.F32, "bf16x3"), SYMT_GEMM_TILE=tile, SYMT_GEMM_SK=sk)
            assert [p["any"] for p in got] == [i if p["ch16"] else max(i, 1) for p in got], (tile, sk)
            assert all(p["sk"] == int(sk) for p in got)
    for bn in (192, 224, 256, 288):
        got = PL.plans(lines(wide.CASES, PL.F32, "bf16x3"), SYMT_GEMM_TILE=f"bw256x{bn}sk")
        assert [p["wide_bn"] for p in got] == [bn] * len(got)
    for dt, comp in every + ((PL.F32, "bf16x3"),):
        got = PL.plans([PL.line(sub, (G,), cu, du, cv, dv, dt, comp, cv=2, hu=hu, hv=hv)
                        for sub, G, cu, cv, du, dv, hu, hv in subgroup.CASES])
        assert all(p["direct"] and p["slices"] for p in got), (dt, comp)
    for dt, comp in real:
        assert all(p["tile"] == ROWS for p in PL.plans(lines(rows.CASES, dt, comp), SYMT_GEMM_TILE="rows"))
        assert all(p["tile"] == TALLK for p in PL.plans(lines(tallk.CASES, dt, comp), SYMT_GEMM_TILE="tallk"))
