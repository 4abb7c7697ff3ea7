"""Split-K planes of direct kernels of 64 and more rows leave through LDS, 64 rows at a
time (csrc/go_kernel_u.h): rows that end inside a half of 64, at its edge and one
past it, columns that end inside a tile, N that is no multiple of four (stored
from the accumulators), batches, and members of one dispatch with different runs.
Every element against the oracle."""
import pytest

import paper_2409_02227_amd  # noqa: F401  (sets GPU_MAX_HW_QUEUES before HIP starts)

torch = pytest.importorskip("torch")

from paper_2409_02227_amd import gdy, inputs  # noqa: E402
from paper_2409_02227_amd.inputs import GemmSpec  # noqa: E402
from tests.gpu_helpers import check, gemm_of, reset_outputs  # noqa: E402

pytestmark = pytest.mark.gpu

KERNELS = [("bf16", "nn", "64x64_w2x2_d4"), ("bf16", "nt", "64x128_w2x2_d4"), ("f16", "nn", "64x256_w1x4_d3"),
           ("bf16", "tn", "128x128_w2x2_d2"), ("fp8", "nt", "128x128_w2x2_d4"), ("fp8", "nn", "64x64_w2x2_d4"),
           ("fp8", "nn", "64x128_w1x4_m32"), ("f32", "nt", "128x128_w2x2_m32")]  # the last two: from the accumulators


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = gdy.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("dt,lay,kernel", KERNELS)
def test_plane_edges(ctx, dt, lay, kernel):
    ta, tb = int(lay[0] == "t"), int(lay[1] == "t")
    vid = ctx.find(f"{dt}_{lay}_{kernel}_c0")
    k = {"f32": 2048, "fp8": 8192}.get(dt, 4096)
    q = 16 // {"bf16": 2, "f16": 2, "fp8": 1, "f32": 4}[dt]
    for i, (m, n, batch) in enumerate([(1, 4, 0), (63, 260, 0), (64, 256, 0), (65, 132, 0), (128, 68, 2), (130, 262, 0),
                                       (200, 516, 0), (193, 301, 2)]):
        spec = GemmSpec(m, n, k, dt, ta, tb, seed=9300 + i, name=f"{dt}_{lay}_{m}x{n}x{k}_{kernel}",
                        pad_a=-(m if ta else k) % q, pad_b=-(k if tb else n) % q, batch=batch)
        mat = inputs.materialize(spec)
        reset_outputs([mat])
        plan = ctx.execute([gemm_of(mat, vid)], mode="forced", want_plan=True)
        torch.cuda.synchronize()
        assert plan["variant_of"][0] == vid and plan["split_of"][0] > 1
        check(mat, label=spec.name)


def test_members_of_different_runs(ctx):
    """Members of one dispatch with runs of different lengths beside an unsplit one."""
    vid = ctx.find("bf16_nn_128x128_w2x2_d2_c0")
    mats = [inputs.materialize(GemmSpec(m, n, k, "bf16", seed=9350 + i, name=f"{m}x{n}x{k}"))
            for i, (m, n, k) in enumerate([(200, 520, 8192), (128, 256, 2112), (65, 1032, 4160), (1024, 1024, 1024)])]
    reset_outputs(mats)
    plan = ctx.execute([gemm_of(m, vid) for m in mats], mode="forced_grouped", want_plan=True)
    torch.cuda.synchronize()
    assert plan["n_dispatches"] == 1 and min(plan["split_of"][:3]) > 1 and plan["split_of"][3] == 1
    for m in mats:
        check(m, label=m.spec.name)
