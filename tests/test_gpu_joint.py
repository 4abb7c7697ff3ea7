"""Joint launches (csrc/go_kernel_u.h go_gemm_joint, go_kernel_p.h
go_gemm_p_joint): a group whose GEMMs bind several kernels of one type runs
them in one grid.  Each GEMM's result equals, bit for bit, its run alone on
the kernel the plan names, over layouts, tiles, alignments, split K and adds;
and the oracle's."""
import numpy as np
import pytest

import paper_2409_02227_amd  # noqa: F401  (sets GPU_MAX_HW_QUEUES before HIP starts)

torch = pytest.importorskip("torch")

from paper_2409_02227_amd import gdy, inputs  # noqa: E402
from paper_2409_02227_amd.inputs import GemmSpec  # noqa: E402
from tests.gpu_helpers import check, check_add, gemm_of, out_codes, reset_outputs  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = gdy.Context(0)  # no table: GO binds every GEMM to its isolated heuristic
    yield c
    c.close()


SHAPES = [("nn", 300, 1000, 520, 0), ("nt", 77, 512, 1024, 0), ("nt", 1000, 640, 512, 1), ("nn", 16, 1024, 4096, 0),
          ("tn", 256, 300, 200, 0), ("tt", 130, 128, 384, 8), ("nn", 1, 700, 333, 3), ("nt", 33, 257, 2048, 0),
          ("tn", 513, 515, 1040, 1), ("nn", 260, 260, 64, 0)]


# (layout, m, n, k, pad, kernel): every tile of the joint kernel in the layouts that have it, wider tiles that run as
# those, operands of any alignment, K tails, split K on four tile sizes, and 256 x 256 kernels, which join short
# groups as 128 x 128 tiles (with operands that take copies and that do not)
MIXED = [("nn", 300, 1000, 520, 0, "128x128_w2x2_m32"), ("nt", 77, 512, 1024, 0, "64x128_w1x4_m32"),
         ("nt", 1000, 640, 512, 1, "64x64_w2x2_m32"), ("nn", 16, 1024, 8192, 0, "16x64_w1x4_m16"),
         ("nn", 40, 1024, 8192, 0, "64x64_w2x2_m32"), ("nt", 33, 257, 8192, 3, "32x128_w1x4_m32"),
         ("nn", 130, 512, 8192, 0, "128x128_w2x2_m32"), ("nn", 1, 700, 333, 3, "16x256_w1x4_m16"),
         ("tn", 256, 300, 200, 0, "128x128_w2x2_m32"), ("tt", 130, 128, 384, 8, "64x64_w2x2_m32"),
         ("tn", 513, 515, 1040, 1, "256x256_w2x4_m32"), ("nn", 260, 260, 64, 0, "64x256_w1x4_m32"),
         ("nt", 200, 333, 1040, 0, "256x128_w2x2_m32"), ("nn", 90, 640, 512, 0, "32x256_w1x4_m32"),
         ("tt", 17, 40, 96, 0, "16x64_w1x4_m16"), ("nn", 700, 512, 1024, 0, "256x256_w2x4_m32")]


@pytest.mark.parametrize("dt", ["bf16", "f16", "fp8", "f32"])
@pytest.mark.parametrize("order", [1, -1])
def test_mixed_tiles_in_one_launch(ctx, tmp_path, dt, order):
    """GO under a table that binds each of 16 GEMMs to a kernel of its own tile
    and layout: a dispatch per kernel, one launch, each result that of its
    kernel alone bit for bit and within the oracle's bound."""
    rows = MIXED[::order]
    t = gdy.Context(0, table=bound_table(tmp_path / "mixed.table", ctx, [(dt,) + r[:4] for r in rows], [r[5] for r in rows]))
    try:
        mats = [inputs.materialize(GemmSpec(m, n, k, dt, int(lay[0] == "t"), int(lay[1] == "t"), seed=9400 + i, pad_a=pad,
                                            pad_b=pad, name=f"{dt}_{lay}_{m}x{n}x{k}"))
                for i, (lay, m, n, k, pad, _) in enumerate(rows)]
        gemms = [gemm_of(m) for m in mats]
        reset_outputs(mats)
        plan = t.execute(gemms, mode="go", want_plan=True)
        torch.cuda.synchronize()
        assert [t.variant(v)["name"] for v in plan["variant_of"][:16]] == [f"{dt}_{r[0]}_{r[5]}_c0" for r in rows]
        assert set(plan["stream_of"]) == {-1} and plan["n_dispatches"] == 15  # two members share 128 x 128 nn
        assert len({t.dispatch_map(gemms, mode="go", dispatch=d)["grid"] for d in range(15)}) == 1
        split = {r[5].split("_")[0] for r, x in zip(rows, plan["split_of"]) if x > 1}
        assert split >= {"16x64", "64x64", "32x128", "128x128"}, split
        for m in mats:
            check(m, label="joint")
        same_bits_alone(t, mats, plan)
    finally:
        t.close()


@pytest.mark.parametrize("dt", ["bf16", "f16", "fp8", "f32"])
@pytest.mark.parametrize("count", [2, 5, 10])
def test_bits_and_values(ctx, dt, count):
    """Groups of dispatches of named kernels (FORCED_GROUPED: one launch each,
    on pool streams), and the joint GO launch of the isolated heuristics."""
    mats = [inputs.materialize(GemmSpec(m, n, k, dt, int(lay[0] == "t"), int(lay[1] == "t"), seed=9500 + i, pad_a=pad,
                                        pad_b=pad, name=f"{dt}_{lay}_{m}x{n}x{k}"))
            for i, (lay, m, n, k, pad) in enumerate(SHAPES[:count])]
    # kernels of every tile and both families, named one by one
    names = ["128x128_w2x2_m32", "64x64_w2x2_m32", "256x256_w2x4_m32", "16x64_w1x4_m16"]
    for rnd in range(len(names)):
        vids = [ctx.find(f"{dt}_{SHAPES[i][0]}_{names[(i + rnd) % len(names)]}_c0") for i in range(count)]
        assert min(vids) >= 0
        alone = []
        for m, v in zip(mats, vids):
            reset_outputs([m])
            ctx.execute([gemm_of(m, v)], mode="forced")
            torch.cuda.synchronize()
            check(m, label="alone")
            alone.append(out_codes(m).copy())
        reset_outputs(mats)
        ctx.execute([gemm_of(m, v) for m, v in zip(mats, vids)], mode="forced_grouped")
        torch.cuda.synchronize()
        for m, ref in zip(mats, alone):
            assert np.array_equal(out_codes(m), ref), m.spec.name
    reset_outputs(mats)
    plan = ctx.execute([gemm_of(m) for m in mats], mode="go", want_plan=True)
    torch.cuda.synchronize()
    got = [out_codes(m).copy() for m in mats]
    for m, v, bits in zip(mats, plan["variant_of"], got):
        check(m, label="go")
        reset_outputs([m])
        ctx.execute([gemm_of(m, v)], mode="forced")
        torch.cuda.synchronize()
        assert np.array_equal(out_codes(m), bits), (m.spec.name, ctx.variant(v)["name"])


def test_table_bound_kernels_join(ctx, tmp_path):
    """GO under a table that binds each GEMM to a kernel of another tile and
    layout: one stream, and the bits of each kernel run alone; an add rides
    along."""
    rows = [("nn", 300, 1024, 512, "64x64_w2x2_d4"), ("nt", 77, 512, 1024, "128x128_w2x2_d2"),
            ("nt", 1000, 640, 512, "256x256_w2x4_d2"), ("nn", 16, 1024, 4096, "32x128_w1x4_d4"),
            ("tn", 256, 304, 256, "256x256_w2x4_d2"), ("nn", 40, 2048, 2048, "64x256_w1x4_d3"),
            ("nn", 512, 512, 192, "256x128_w2x2_d3"), ("tt", 128, 128, 384, "64x64_w2x2_d4")]
    lines = ["gdy-go-table 2", f"device gfx950 cus {ctx.cus()}", f"catalogue {ctx.catalogue_hash():016x}"]
    mats = []
    for i, (lay, m, n, k, name) in enumerate(rows):
        ta, tb = int(lay[0] == "t"), int(lay[1] == "t")
        lines.append(f"entry 2 {ta} {tb} {(m - 1).bit_length()} {n} {k} 1 " + " ".join([f"bf16_{lay}_{name}_c0"] * 5))
        mats.append(inputs.materialize(GemmSpec(m, n, k, "bf16", ta, tb, seed=9600 + i, name=f"{lay}_{m}x{n}x{k}")))
    path = tmp_path / "joint.table"
    path.write_text("\n".join(lines) + "\n")
    t = gdy.Context(0, table=str(path))
    try:
        add = inputs.materialize_add(200, 1000, "bf16", seed=4)
        reset_outputs(mats)
        add.c_full.fill_(float("nan"))
        plan = t.execute([gemm_of(m) for m in mats] + [gdy.Add(add.a, add.b, add.c)], mode="go", want_plan=True)
        torch.cuda.synchronize()
        assert [t.variant(v)["name"] for v in plan["variant_of"][:8]] == [f"bf16_{r[0]}_{r[4]}_c0" for r in rows]
        assert plan["fallback"] == 0 and set(plan["stream_of"]) == {-1}  # a short group: one launch
        check_add(add)
        got = [out_codes(m).copy() for m in mats]
        for m, v, bits in zip(mats, plan["variant_of"], got):
            check(m, label="joint")
            reset_outputs([m])
            t.execute([gemm_of(m, v)], mode="forced")
            torch.cuda.synchronize()
            assert np.array_equal(out_codes(m), bits), m.spec.name
    finally:
        t.close()


def bound_table(path, ctx, rows, name):
    """A GO table that binds each row (type, layout, m, n, k) to the kernel `name` of its type and layout (a list: each
    to its own)."""
    names = [name] * len(rows) if isinstance(name, str) else name
    lines = ["gdy-go-table 2", f"device gfx950 cus {ctx.cus()}", f"catalogue {ctx.catalogue_hash():016x}"]
    codes = {"f16": 1, "bf16": 2, "fp8": 3, "f32": 4}
    for (dt, lay, m, n, k), kernel in zip(rows, names):
        ta, tb = int(lay[0] == "t"), int(lay[1] == "t")
        lines.append(f"entry {codes[dt]} {ta} {tb} {(m - 1).bit_length()} {n} {k} 1 " +
                     " ".join([f"{dt}_{lay}_{kernel}_c0"] * 5))
    path.write_text("\n".join(lines) + "\n")
    return str(path)


def same_bits_alone(t, mats, plan):
    got = [out_codes(m).copy() for m in mats]
    for m, v, bits in zip(mats, plan["variant_of"], got):
        reset_outputs([m])
        t.execute([gemm_of(m, v)], mode="forced")
        torch.cuda.synchronize()
        assert np.array_equal(out_codes(m), bits), m.spec.name


@pytest.mark.parametrize("dt,k", [("bf16", 1032), ("f16", 1088), ("fp8", 2064)])
@pytest.mark.parametrize("layouts", [("nt", "tn"), ("nn", "nn"), ("tt", "tn")])
def test_wide_tiles_for_128_row_kernels(ctx, tmp_path, dt, k, layouts):
    """Large groups bound to 128 x 128 kernels run on the 256 x 256 one: one
    launch of a quarter of the tiles, the bits of the kernels alone."""
    rows = [(dt, lay, 2048, 4096 - 16 * i, k) for i, lay in enumerate(layouts)]
    t = gdy.Context(0, table=bound_table(tmp_path / "wide.table", ctx, rows, "128x128_w2x2_m32"))
    try:
        mats = [inputs.materialize(GemmSpec(m, n, kk, dt, int(lay[0] == "t"), int(lay[1] == "t"), seed=9800 + i,
                                            name=f"{dt}_{lay}_{m}x{n}x{kk}"))
                for i, (_, lay, m, n, kk) in enumerate(rows)]
        gemms = [gemm_of(m) for m in mats]
        reset_outputs(mats)
        plan = t.execute(gemms, mode="go", want_plan=True)
        torch.cuda.synchronize()
        assert set(plan["stream_of"]) == {-1}
        assert t.dispatch_map(gemms, mode="go")["grid"] <= 256 + 8
        same_bits_alone(t, mats, plan)
    finally:
        t.close()


@pytest.mark.parametrize("dt", ["bf16", "fp8"])
@pytest.mark.parametrize("m,n,half", [(1300, 4096, True), (513, 12288, True), (2048, 1024, True), (1024, 2048, True),
                                      (3900, 4096, False), (2100, 8192, False), (4096, 4096, False)])
def test_half_rows(ctx, tmp_path, dt, m, n, half):
    """256 x 256 launches that do not fill the chip cut their tile rows in two
    (whole, short and one-row last tiles), others do not: tiles of 256 CUs' worth
    once (256) or 9 x 32 of them, where halves would take longer.  The bits are
    those of the 128 x 128 kernel."""
    k = 1040  # not split on either kernel
    rows = [(dt, "nn", m, n, k)]
    mat = inputs.materialize(GemmSpec(m, n, k, dt, 0, 0, seed=9900 + m, name=f"{dt}_{m}x{n}x{k}"))
    got = {}
    for name in ("256x256_w2x4_m32", "128x128_w2x2_m32"):
        t = gdy.Context(0, table=bound_table(tmp_path / f"{name}.table", ctx, rows, name))
        try:
            reset_outputs([mat])
            vid = t.find(f"{dt}_nn_{name}_c0") if name[0] == "1" else None
            plan = t.execute([gemm_of(mat) if vid is None else gemm_of(mat, vid)],
                             mode="go" if vid is None else "forced", want_plan=True)
            torch.cuda.synchronize()
            got[name] = out_codes(mat).copy()
            assert plan["split_of"][0] == 1
            if name[0] == "2":
                assert t.dispatch_map([gemm_of(mat)], mode="go")["grid"] == -(-m // (128 if half else 256)) * -(-n // 256)
        finally:
            t.close()
    assert np.array_equal(*got.values())


@pytest.mark.parametrize("dt,lay,kernel", [(dt, lay, kernel) for dt, lay in (("bf16", "nn"), ("f16", "nt"), ("fp8", "nn"))
                                           for kernel in ("256x128_w2x2_m32", "128x256_w2x2_m32", "128x128_w2x2_d4")] +
                         [("bf16", "tn", "256x128_w2x2_m32")])
def test_lone_dispatches_on_wide_tiles(ctx, tmp_path, dt, lay, kernel):
    """A lone dispatch of 256 x 128, 128 x 256 or four-stage 128 x 128 tiles runs
    on 256 x 256 ones where its own would take longer, with the same bits."""
    m, n, k = 1990, 3088, 1152
    t = gdy.Context(0, table=bound_table(tmp_path / "lone.table", ctx, [(dt, lay, m, n, k)], kernel))
    try:
        ta, tb = int(lay[0] == "t"), int(lay[1] == "t")
        mat = inputs.materialize(GemmSpec(m, n, k, dt, ta, tb, seed=9950, pad_a=-(m if ta else k) % 16,
                                          name=f"{dt}_{lay}_{m}x{n}x{k}"))
        reset_outputs([mat])
        plan = t.execute([gemm_of(mat)], mode="go", want_plan=True)
        torch.cuda.synchronize()
        assert t.variant(plan["variant_of"][0])["name"] == f"{dt}_{lay}_{kernel}_c0"
        assert t.dispatch_map([gemm_of(mat)], mode="go")["grid"] == 16 * 13  # 128-row tiles
        check(mat, label="wide")
        same_bits_alone(t, [mat], plan)
    finally:
        t.close()
