"""Input types and layouts that a GO table holds no tuned shape of borrow those
of a sibling: fp16 and bf16 each other's of the same layout, any type its
untransposed ones, then the other 16-bit type's untransposed ones.  They bind
their own type's kernels of the same tile and grid cap (the closest tile where
their catalogue has none), and the plan still reports fallback = 1: nothing was
tuned for them.  Host-only contexts."""
import pytest

from paper_2409_02227_amd import gdy

TYPES = {"f16": 1, "bf16": 2, "fp8": 3, "f32": 4}
CLASSES = ["64x64_w2x2_d4_c0", "128x128_w2x2_d2_c128", "128x128_w2x2_d2_c64", "64x64_w2x2_d4_c32",
           "256x256_w2x4_d2_c0"]
PARTS = ["128x128_w2x2_d2_c0", "64x64_w2x2_d4_c0", "256x256_w2x4_d2_c0"]  # under 128, 64 and 32 CUs


def table(path, rows, classes=CLASSES, parts=PARTS):
    """rows: (type, layout, m, n, k)."""
    lines = ["gdy-go-table 2", "device host cus 256", "catalogue 0"]
    for dt, lay, m, n, k in rows:
        lines.append(f"entry {TYPES[dt]} {int(lay[0] == 't')} {int(lay[1] == 't')} {(m - 1).bit_length()} {n} {k} 1 " +
                     " ".join(f"{dt}_{lay}_{c}" for c in classes + parts))
    path.write_text("\n".join(lines) + "\n")
    return gdy.Context(-1, table=str(path))


def desc(dt, lay, m, n, k, slot=0):
    d = gdy.GemmDesc()
    ta, tb = int(lay[0] == "t"), int(lay[1] == "t")
    d.m, d.n, d.k = m, n, k
    d.a_type = d.b_type = TYPES[dt]
    d.c_type = {1: 1, 2: 2, 3: 2, 4: 4}[TYPES[dt]]
    d.trans_a, d.trans_b = ta, tb
    d.lda, d.ldb, d.ldc = (m if ta else k), (k if tb else n), n
    base = (slot + 1) << 40
    d.a, d.b, d.c = base, base + (1 << 38), base + (2 << 38)
    d.scale_a = d.scale_b = 1.0
    d.variant = -1
    return d


def bound(t, dt, lay, classes=True):
    """(names bound for the CD classes, or under the CU budgets, and the plans' fallback flags): GO groups of 1, 2, 4, 8
    and 16 copies of one shape whose K does not split, or CU partitions of 2, 4 and 8."""
    names, flags = [], set()
    for s in ([1, 2, 4, 8, 16] if classes else [2, 4, 8]):
        p = t.plan([desc(dt, lay, 512, 1024, 1024, j) for j in range(s)], mode="go" if classes else "cu_partition_rc",
                   forced_cd=0 if classes else s)
        assert set(p["split_of"][:s]) == {1} and len(set(p["variant_of"][:s])) == 1
        v = t.variant(p["variant_of"][0])
        assert v["dtype"] == TYPES[dt] and (v["trans_a"], v["trans_b"]) == (int(lay[0] == "t"), int(lay[1] == "t"))
        names.append(v["name"])
        flags.add(p["fallback"])
    return names, flags


@pytest.mark.parametrize("dt,lay,source", [
    ("f16", "nt", ("bf16", "nt")), ("bf16", "nn", ("f16", "nn")), ("f16", "tn", ("bf16", "tn")),  # the other 16-bit type's
    ("fp8", "nt", ("fp8", "nn")), ("f16", "nt", ("f16", "nn")), ("bf16", "tt", ("bf16", "nn")),   # the untransposed ones
    ("f16", "tt", ("bf16", "nn"))])                                                              # the other's untransposed
def test_tile_and_cap_of_the_sibling(tmp_path, dt, lay, source):
    t = table(tmp_path / "t.table", [source + (512, 1024, 1024)])
    names, flags = bound(t, dt, lay)
    assert names == [f"{dt}_{lay}_{c}" for c in CLASSES] and flags == {1}
    names, flags = bound(t, dt, lay, classes=False)
    assert names == [f"{dt}_{lay}_{c}" for c in PARTS] and flags == {1}
    names, flags = bound(t, *source)  # the tuned type and layout itself
    assert names == [f"{source[0]}_{source[1]}_{c}" for c in CLASSES] and flags == {0}
    assert bound(t, *source, classes=False)[1] == {0}


def test_own_shapes_are_not_replaced(tmp_path):
    """One tuned shape of its own, however far, and a type borrows nothing; the other types' entries do not mix in."""
    far = ["16x64_w1x4_m16_c0"] * 5
    lines = (tmp_path / "a.table", tmp_path / "b.table")
    table(lines[0], [("bf16", "nt", 512, 1024, 1024)])
    table(lines[1], [("f16", "nt", 16, 65536, 65536)], far, far[:3])
    both = lines[0].read_text() + lines[1].read_text().splitlines()[-1] + "\n"
    (tmp_path / "both.table").write_text(both)
    t = gdy.Context(-1, table=str(tmp_path / "both.table"))
    assert bound(t, "f16", "nt") == ([f"f16_nt_{c}" for c in far], {0})
    assert bound(t, "bf16", "nt") == ([f"bf16_nt_{c}" for c in CLASSES], {0})


def test_closest_tile_where_the_catalogue_has_none(tmp_path):
    """Transposed A has fewer tiles: the closest one (in octaves of rows and columns; the catalogue's first of equals),
    direct for direct, caps kept."""
    t = table(tmp_path / "t.table", [("bf16", "nn", 512, 1024, 1024)],
              ["32x128_w1x4_d4_c0", "64x128_w2x2_d4_c128", "128x256_w2x2_d3_c64", "256x256_w4x4_d2_c32",
               "128x128_w2x2_d4_c0"])
    names, flags = bound(t, "bf16", "tn")
    assert flags == {1}
    # 32 x 128 is two octaves from 128 x 128 and from 64 x 64, 64 x 128 one octave from both: 128 x 128 comes first;
    # 128 x 256 is one octave from 128 x 128 and from 256 x 256, which comes first; the others have their own tiles
    assert names == [f"bf16_tn_{c}" for c in ("128x128_w2x2_d2_c0", "128x128_w2x2_d2_c128", "256x256_w2x4_d2_c64",
                                              "256x256_w2x4_d2_c32", "128x128_w2x2_d2_c0")]


def test_nothing_to_borrow(tmp_path):
    """fp32 and fp8 borrow from no other type: the isolated heuristic."""
    t = table(tmp_path / "t.table", [("bf16", "nn", 512, 1024, 1024)])
    h = gdy.Context(-1)
    for dt in ("f32", "fp8"):
        for lay in ("nn", "nt", "tn", "tt"):
            d = desc(dt, lay, 512, 1024, 1024)
            assert t.isolated_variant(d) == h.isolated_variant(d)
            assert t.plan([d], mode="go")["fallback"] == 1
    # a group of one tuned and one untuned member reports it too
    p = t.plan([desc("bf16", "nn", 512, 1024, 1024, 0), desc("bf16", "nt", 512, 1024, 1024, 1)], mode="selector")
    assert p["fallback"] == 1


def test_isolated_kernels_of_batches_and_fp32(tmp_path):
    """A lone batch or fp32 GEMM of a borrowed layout runs the isolated heuristic's kernel, a lone 16-bit or fp8 GEMM the
    borrowed one without its grid cap; in a group all bind the borrowed kernels of its class."""
    capped = ["64x64_w2x2_m32_c128", "128x128_w2x2_m32_c64"] + ["64x64_w2x2_m32_c32"] * 3
    h = gdy.Context(-1)
    for dt in ("f16", "fp8", "f32"):
        t = table(tmp_path / f"{dt}.table", [(dt, "nn", 512, 1024, 1024)], capped, [c.replace("_c128", "_c0") for c in capped[:3]])
        one, many = desc(dt, "nt", 512, 1024, 512), desc(dt, "nt", 512, 1024, 512)
        many.batch, many.stride_a, many.stride_b, many.stride_c = 4, 512 * 512, 1024 * 512, 512 * 1024
        for d, heuristic in ((one, dt == "f32"), (many, True)):
            vid = t.isolated_variant(d)
            for mode in ("sequential", "selector", "default"):
                p = t.plan([d], mode=mode)
                assert p["variant_of"][0] == vid and p["fallback"] == 1
            if heuristic:
                assert vid == h.isolated_variant(d)
            else:
                assert t.variant(vid)["name"] == f"{dt}_nt_64x64_w2x2_m32_c0"
            pair = [d, desc(dt, "nt", 512, 1024, 512, 1)]
            pair[1].batch, pair[1].stride_a, pair[1].stride_b, pair[1].stride_c = d.batch, d.stride_a, d.stride_b, d.stride_c
            p = t.plan(pair, mode="go")
            assert {t.variant(v)["name"] for v in p["variant_of"][:2]} == {f"{dt}_nt_128x128_w2x2_m32_c64"}
            assert p["fallback"] == 1
        # the type's tuned layout keeps its caps and its batches
        own = desc(dt, "nn", 512, 1024, 512)
        assert t.variant(t.isolated_variant(own))["name"] == f"{dt}_nn_64x64_w2x2_m32_c128"


def test_features_describe_the_entry(tmp_path):
    """The predictor's features are of the borrowed entry's kernels, also where the GEMM alone runs the heuristic's: a
    group forms as its kernels were tuned to."""
    t = table(tmp_path / "t.table", [("f32", "nn", 512, 1024, 1024)], ["128x128_w2x2_m32_c0"] + ["64x64_w2x2_m32_c0"] * 4,
              ["64x64_w2x2_m32_c0"] * 3)
    d = desc("f32", "nt", 512, 1024, 512)
    assert t.variant(t.isolated_variant(d))["name"] != "f32_nt_128x128_w2x2_m32_c0"
    f = t.features(d)
    assert list(f[:4]) == [512, 1024, 512, 32] and f[6] == 128  # 4 x 8 tiles of 128 x 128, 8 x 16 of 64 x 64
