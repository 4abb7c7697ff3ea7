"""Every work item of every dispatch is computed exactly once: the host's
dispatch map (gdy_dispatch_map runs the kernels' own workgroup-to-work
mapping on the launch blocks gdy_execute builds) over random submissions
in every execution mode, including XCD-placed fused dispatches.  Host-only
context; no GPU."""
import collections
import os

import numpy as np
import pytest

from paper_2409_02227_amd import gdy, inputs

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
TABLE = os.path.join(ROOT, "paper_2409_02227_amd", "tables", "gfx950.table")
MODES = ("sequential", "default", "go", "selector", "forced_grouped", "cu_partition_go")


def _desc(m, n, k, dtype, slot, ta=0, tb=0, batch=0, op=0):
    d = gdy.GemmDesc()
    d.m, d.n, d.k = m, n, k
    d.a_type = d.b_type = dtype
    d.c_type = {1: 1, 2: 2, 3: 2, 4: 4}[dtype]
    d.trans_a, d.trans_b = ta, tb
    d.lda, d.ldb, d.ldc = (m if ta else k) or 1, (k if tb else n) or 1, n
    if op:
        d.lda = d.ldb = n
    base = (slot + 1) << 40
    d.a, d.b, d.c = base, base + (1 << 38), base + (2 << 38)
    d.scale_a = d.scale_b = 1.0
    d.variant = -1
    d.op = op
    if batch:
        d.batch = batch
        d.stride_a, d.stride_b, d.stride_c = d.lda * (k if ta else m), d.ldb * (n if tb else k), n * m
    return d


def _check_cover(ctx, descs, mode, forced=0):
    p = ctx.plan(descs, mode=mode, forced_cd=forced)
    placed = 0
    for d in range(p["n_dispatches"]):
        m = ctx.dispatch_map(descs, mode=mode, forced_cd=forced, dispatch=d)
        members = [i for i in range(len(descs)) if p["dispatch_of"][i] == d]
        assert sorted(i for i in range(len(descs)) if m["items"][i] > 0) == \
            sorted(i for i in members if m["items"][i] > 0)
        cov = collections.Counter()
        xcds = collections.defaultdict(set)
        for b in range(m["grid"]):
            g = m["gemm"][b]
            if g < 0:
                continue
            assert g in members and m["stride"][b] > 0
            t = m["first"][b]
            while t < m["items"][g]:
                cov[(g, t)] += 1
                xcds[g].add(b % 8)
                t += m["stride"][b]
        for g in members:
            got = [cov[(g, t)] for t in range(m["items"][g])]
            assert got == [1] * m["items"][g], (mode, d, g)
        assert sum(cov.values()) == sum(m["items"][g] for g in members)
        if len(members) >= 2 and max(len(x) for x in xcds.values()) < 8:
            placed += 1
    return p, placed


def test_layer_share_is_placed_on_few_xcds():
    """The tensor-sliced layer share's fused dispatch: every tile once, each
    GEMM's tiles on at most 4 of the 8 XCDs (all 8 before placement), and
    every XCD holds the same work (tiles x (K tiles + 1)) within 1%."""
    ctx = gdy.Context(-1, table=TABLE if os.path.exists(TABLE) else None)
    specs = inputs.layer_share()
    descs = [_desc(s.m, s.n, s.k, 2, i) for i, s in enumerate(specs)]
    for mode in ("selector", "go"):
        p, placed = _check_cover(ctx, descs, mode)
        if p["n_dispatches"] != 1:
            continue
        m = ctx.dispatch_map(descs, mode=mode, dispatch=0)
        on = collections.defaultdict(set)
        work = [0] * 8
        for b in range(m["grid"]):
            g = m["gemm"][b]
            if g >= 0:
                on[g].add(b % 8)
                v = ctx.variant(p["variant_of"][g])
                work[b % 8] += -(-specs[g].k // v["bk"]) + 1
        assert all(len(x) <= 4 for x in on.values()), dict(on)
        assert max(work) <= 1.01 * min(work), work


def test_every_dispatch_covers_its_work_once():
    ctx = gdy.Context(-1, table=TABLE if os.path.exists(TABLE) else None)
    rng = np.random.default_rng(17)
    placed_total = 0
    for _ in range(60):
        n = int(rng.integers(1, 12))
        descs = []
        for i in range(n):
            if rng.random() < 0.1:
                descs.append(_desc(int(rng.integers(1, 300)), int(rng.integers(1, 700)), 0, 2, i, op=1))
                continue
            dtype = int(rng.choice([1, 2, 3, 4]))
            ta, tb = [(0, 0), (0, 1), (1, 0), (1, 1)][int(rng.integers(4))]
            m = int(rng.choice([1, 16, 100, 512, 1000, 4096]))
            nn = int(rng.choice([64, 300, 1024, 4096, 8192]))
            k = int(rng.choice([64, 1000, 1024, 8192]))
            batch = int(rng.choice([0, 0, 0, 3]))
            descs.append(_desc(m, nn, k, dtype, i, ta, tb, batch))
        for mode in MODES:
            for forced in ((0, 2) if mode in ("go", "forced_grouped") else (0,)):
                if mode == "forced_grouped":
                    for d in descs:
                        d.variant = ctx.isolated_variant(d)
                _, placed = _check_cover(ctx, descs, mode, forced)
                placed_total += placed
    assert placed_total > 0  # some fused dispatches were placed


@pytest.mark.parametrize("dtype,name,tile_k", [(3, "fp8", 128), (2, "bf16", 64)])
def test_placement_counts_the_k_tiles_that_run(dtype, name, tile_k):
    """Names of the one 256 x 256 kernel that state K tiles of 64 and of 128
    bytes share a dispatch: members of one K weigh the same, so XCDs hold equal
    work.  Four members of 8 x 32 tiles of one K: 128 tiles on each XCD.  Random
    sets: the busiest XCD is within 3% of its share on average (a cut falls
    on whole tile columns); 10-17% when K tiles were counted by name."""
    ctx = gdy.Context(-1)
    kern = [ctx.find(f"{name}_nn_256x256_{s}_c0") for s in ("w2x4_d4h", "w2x4_d2", "w2x2_d4h", "w2x2_d2")]

    def work(sizes, variants):
        descs = [_desc(m, n, k, dtype, j) for j, (m, n, k) in enumerate(sizes)]
        for d, v in zip(descs, variants):
            d.variant = v
        assert ctx.plan(descs, mode="forced_grouped")["n_dispatches"] == 1
        m = ctx.dispatch_map(descs, mode="forced_grouped", dispatch=0)
        out = np.zeros(8)
        for b, g in enumerate(m["gemm"][:m["grid"]]):
            if g >= 0:
                out[b % 8] += sizes[g][2] // tile_k + 1
        return out

    w = work([(2048, 8192, 4096)] * 4, kern)
    assert w.min() == w.max() == 128 * (4096 // tile_k + 1)
    rng = np.random.default_rng(5)
    over = []
    for _ in range(40):
        u = int(rng.integers(2, 13))
        sizes = [tuple(int(rng.choice(c)) for c in ((512, 1024, 2048), (2048, 4096, 8192), (2048, 4096, 8192)))
                 for _ in range(u)]
        w = work(sizes, [kern[int(rng.integers(2))] for _ in range(u)])
        over.append(w.max() / w.mean() - 1)
    assert np.mean(over) < 0.03, np.mean(over)


def test_half_rows_count_the_cus_of_the_stream(tmp_path):
    """256 x 256 kernels cut their tile rows in two where the tiles do not fill
    the CUs of the stream they run on: 8 x 8 tiles of (2048, 2048) do not fill
    256 CUs (0.6 of a tile's time on 128 half tiles against 1), but a quarter
    of them: 64 tiles on 64 CUs take 1, 128 half tiles 0.6 * 128 / 64 + 0.3.
    2 x 8 tiles of (512, 2048) fill neither."""
    name = "bf16_nn_256x256_w2x4_d2_c0"
    lines = ["gdy-go-table 2", "device host cus 256", "catalogue 0"]
    lines += [f"entry 2 0 0 {m.bit_length() - 1} 2048 1024 1 " + " ".join([name] * 8) for m in (2048, 512)]
    path = tmp_path / "half.table"
    path.write_text("\n".join(lines) + "\n")
    ctx = gdy.Context(-1, table=str(path))
    for m, whole_gpu, quarter in ((2048, 128, 64), (512, 32, 32)):
        descs = [_desc(m, 2048, 1024, 2, j) for j in range(4)]
        assert ctx.dispatch_map(descs, mode="sequential", dispatch=0)["grid"] == whole_gpu
        for mode in ("cu_partition", "cu_partition_go", "cu_partition_rc"):
            p = ctx.plan(descs, mode=mode, forced_cd=4)
            assert [ctx.variant(v)["name"] for v in p["variant_of"][:4]] == [name] * 4
            for d in range(4):
                assert ctx.dispatch_map(descs, mode=mode, forced_cd=4, dispatch=d)["grid"] == quarter


@pytest.mark.parametrize("kernel,m,k,own,runs", [
    # (600, 4096, K) on 256 x 128 tiles: 3 x 32 of 0.72 of a 256 x 256 tile's time at once; 128-row halves: 5 x 16 of
    # 0.6 < 0.9 * 0.72
    ("256x128_w2x2_d3", 600, 1024, 96, 80),
    ("256x128_w2x2_d3", 600, 960, 96, 96),      # short K keeps its kernel
    # (2048, 4096, K) on 128 x 128 tiles of four stages, one to a CU: 512 take 2 * 0.42 + 0.21 = 1.05, 16 x 16 halves 0.6
    ("128x128_w2x2_d4", 2048, 1024, 512, 256),
    ("128x128_w2x2_d2", 2048, 1024, 512, 512),  # all 512 resident: 0.64, and 0.6 > 0.9 * 0.64
    ("128x128_w2x2_d2", 4096, 1024, 1024, 256),  # 0.32 * 4 + 0.32 = 1.6 against 256 whole tiles: 1
])
def test_lone_dispatch_is_priced_on_its_own_tiles(tmp_path, kernel, m, k, own, runs):
    """GO binds one kernel; the launch keeps its tiles or runs 256 x 256 ones,
    by the estimate of what each would take (256 CUs)."""
    name = f"bf16_nn_{kernel}_c0"
    path = tmp_path / "lone.table"
    path.write_text(f"gdy-go-table 2\ndevice host cus 256\ncatalogue 0\nentry 2 0 0 11 4096 1024 1 {' '.join([name] * 5)}\n")
    ctx = gdy.Context(-1, table=str(path))
    d = _desc(m, 4096, k, 2, 0)
    assert ctx.variant(ctx.plan([d], mode="go")["variant_of"][0])["name"] == name
    assert ctx.dispatch_map([d], mode="sequential")["grid"] == own
    assert ctx.dispatch_map([d], mode="go")["grid"] == runs
