"""The 256 x 256 kernel of two alternating wave groups (csrc/go_kernel_p.h)
where it can go wrong: its loops over 256-row and over 128-row tiles at one K
tile and the first few ring turns, tile edges in M and N, C rows with and
without 8-byte alignment, and a grid-capped (persistent) run whose workgroups
walk several tiles.  Every element against the oracle."""
import pytest

import paper_2409_02227_amd  # noqa: F401  (sets GPU_MAX_HW_QUEUES before HIP starts)

torch = pytest.importorskip("torch")

from paper_2409_02227_amd import gdy, inputs  # noqa: E402
from paper_2409_02227_amd.inputs import GemmSpec  # noqa: E402
from tests.gpu_helpers import check, gemm_of, reset_outputs  # noqa: E402

pytestmark = pytest.mark.gpu

ES = {"bf16": 2, "f16": 2, "fp8": 1}


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = gdy.Context(0)
    yield c
    c.close()


def run_forced(ctx, mats, vids):
    reset_outputs(mats)
    plan = ctx.execute([gemm_of(m, v) for m, v in zip(mats, vids)], mode="forced_grouped", want_plan=True)
    torch.cuda.synchronize()
    return plan


def spec(dt, lay, m, n, k, seed, pad_c=0, batch=0):
    """Operand rows padded to 16 bytes, as the direct kernels need them."""
    ta, tb = int(lay[0] == "t"), int(lay[1] == "t")
    q = 16 // ES[dt]
    return GemmSpec(m, n, k, dt, ta, tb, seed=seed, name=f"{dt}_{lay}_{m}x{n}x{k}", pad_a=-(m if ta else k) % q,
                    pad_b=-(k if tb else n) % q, pad_c=pad_c, batch=batch)


@pytest.mark.parametrize("rows", [128, 256])
@pytest.mark.parametrize("dt,lay", [("bf16", "nn"), ("bf16", "nt"), ("f16", "nn"), ("fp8", "nn"), ("fp8", "nt"),
                                    ("bf16", "tn"), ("fp8", "tt")])
def test_edges(ctx, dt, lay, rows):
    """Both loops, which differ in copy order, LDS layout and stages: launches
    this small run 128-row tiles, those of a grid-capped variant 256-row ones
    (and 128-row ones where the last tile row holds at most 128 rows)."""
    vid = ctx.find(f"{dt}_{lay}_256x256_w2x4_d2_c{0 if rows == 128 else 32}")
    bk = ctx.variant(vid)["bk"]
    for i, (m, n, nk, pad_c) in enumerate([
            (1, 1, 1, 0), (127, 255, 2, 0), (128, 256, 3, 0), (129, 257, 4, 4), (255, 8, 5, 3), (256, 513, 1, 0),
            (257, 130, 6, 1), (384, 300, 7, 0), (385, 264, 2, 8), (640, 7, 9, 0), (200, 260, 1, 0), (511, 33, 8, 0),
            (450, 257, 3, 5), (256, 256, 2, 0)]):
        mat = inputs.materialize(spec(dt, lay, m, n, nk * bk, 8100 + i, pad_c))
        assert run_forced(ctx, [mat], [vid])["variant_of"][0] == vid
        assert ctx.dispatch_map([gemm_of(mat, vid)], mode="forced_grouped")["items"][0] == -(-m // rows) * -(-n // 256)
        check(mat, label=mat.spec.name)


@pytest.mark.parametrize("dt,lay", [("bf16", "nn"), ("fp8", "nt")])
def test_workgroups_that_walk_several_tiles(ctx, dt, lay):
    """32 workgroups over 3 x (3 x 9) tiles of a batch: whole and 128-row
    tiles follow each other in one workgroup, and results equal the uncapped
    run's bit for bit."""
    v0, v32 = (ctx.find(f"{dt}_{lay}_256x256_w2x4_d2_c{c}") for c in (0, 32))
    mat = inputs.materialize(spec(dt, lay, 600, 2200, 3 * ctx.variant(v0)["bk"], 8200, 0, batch=3))
    run_forced(ctx, [mat], [v0])
    whole = mat.c.clone()
    run_forced(ctx, [mat], [v32])
    assert bool((mat.c == whole).all())
    check(mat, label="capped")
