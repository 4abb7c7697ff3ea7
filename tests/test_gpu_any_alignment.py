"""The kernels for operands of any size and alignment (csrc/go_kernel_u.h):
copies and register loads must put the same operand into LDS.  Row pitches of
every residue, bases off by one element, K tails inside a 16-byte chunk, split
K runs with a tail, M and N at tile edges.  Every stored element that is not
part of an operand (row padding, and what lies before and behind it) is NaN, so
a chunk that is not cut off at K shows.  Every element against the oracle."""
import numpy as np
import pytest

import paper_2409_02227_amd  # noqa: F401  (sets GPU_MAX_HW_QUEUES before HIP starts)

torch = pytest.importorskip("torch")

from paper_2409_02227_amd import gdy, inputs  # noqa: E402
from paper_2409_02227_amd.inputs import GemmSpec  # noqa: E402
from tests.gpu_helpers import check, gemm_of, reset_outputs  # noqa: E402

pytestmark = pytest.mark.gpu

NAN = {"bf16": 0x7fc0, "f16": 0x7e00, "fp8": 0x7f, "f32": 0x7fc00000}
RAW = {"bf16": np.int16, "f16": np.int16, "fp8": np.uint8, "f32": np.int32}


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = gdy.Context(0)
    yield c
    c.close()


def materialize(spec, shift):
    """inputs.materialize with NaN codes in the row padding and around the
    operands, whose bases lie `shift` elements past a 256-byte boundary."""
    mat = inputs.materialize(spec)
    for which in ("a", "b"):
        r, c = spec.stored_shape(which)
        ld = spec.ld(which)
        codes = mat.host[which].reshape(r, ld)
        codes[:, c:] = NAN[spec.dtype]
        ring = np.full(256 + shift + r * ld + 256, NAN[spec.dtype], dtype=codes.dtype)
        ring[256 + shift:256 + shift + r * ld] = codes.reshape(-1)
        t = getattr(mat, which)
        dev = torch.from_numpy(ring.view(RAW[spec.dtype])).cuda().view(t.dtype)
        setattr(mat, which, dev[256 + shift:256 + shift + r * ld].view(r, ld)[:, :c])
    return mat


FORMS = [  # m, n, k, padding of A's, B's and C's rows, shift of the bases (elements)
    (1, 1, 1, 0, 0, 0, 0), (17, 33, 8, 0, 0, 0, 0), (65, 127, 24, 8, 8, 4, 0), (130, 70, 64, 16, 0, 0, 0),
    (31, 257, 72, 0, 1, 0, 0), (129, 64, 136, 0, 0, 1, 1), (63, 65, 127, 1, 0, 3, 0), (16, 200, 129, 3, 5, 0, 3),
    (260, 31, 200, 0, 0, 2, 8), (40, 300, 333, 2, 2, 0, 2), (100, 100, 1000, 0, 3, 7, 5)]


@pytest.mark.parametrize("dt", ["bf16", "f16", "fp8", "f32"])
@pytest.mark.parametrize("lay", ["nn", "nt", "tn", "tt"])
def test_forms(ctx, dt, lay):
    names = ["64x64_w2x2_m32", "128x128_w2x2_m32", "16x64_w1x4_m16"]
    if lay[0] == "n":
        names += ["32x128_w1x4_m32", "256x256_w2x4_m32"]
    for i, (m, n, k, pa, pb, pc, shift) in enumerate(FORMS):
        spec = GemmSpec(m, n, k, dt, int(lay[0] == "t"), int(lay[1] == "t"), seed=9100 + i,
                        name=f"{dt}_{lay}_{m}x{n}x{k}_{pa}_{pb}_{pc}_{shift}", pad_a=pa, pad_b=pb, pad_c=pc)
        mat = materialize(spec, shift)
        for name in names:
            vid = ctx.find(f"{dt}_{lay}_{name}_c0")
            reset_outputs([mat])
            plan = ctx.execute([gemm_of(mat, vid)], mode="forced_grouped", want_plan=True)
            torch.cuda.synchronize()
            assert plan["variant_of"][0] == vid
            check(mat, label=name)


@pytest.mark.parametrize("dt,lay", [("bf16", "nn"), ("f16", "tn"), ("fp8", "nt"), ("f32", "nn")])
def test_split_runs_with_a_tail(ctx, dt, lay):
    """K of several split runs whose last one ends inside a chunk."""
    vid = ctx.find(f"{dt}_{lay}_64x64_w2x2_m32_c0")
    k = 33 * ctx.variant(vid)["bk"] + 13
    for pad in (0, 3, 16):
        spec = GemmSpec(70, 90, k, dt, int(lay[0] == "t"), int(lay[1] == "t"), seed=9300 + pad,
                        name=f"split_{dt}_{lay}_{pad}", pad_a=pad, pad_b=pad)
        mat = materialize(spec, pad % 4)
        reset_outputs([mat])
        plan = ctx.execute([gemm_of(mat, vid)], mode="forced_grouped", want_plan=True)
        torch.cuda.synchronize()
        assert plan["split_of"][0] == 2
        check(mat, label=spec.name)


@pytest.mark.parametrize("dt", ["bf16", "fp8"])
def test_batch_items_at_every_alignment(ctx, dt):
    """Items of a batch whose stride is odd: each starts at another byte of a
    dword, and the last element of an item may be the first of its dword."""
    for lay, m, n, k in (("nn", 33, 50, 64), ("nt", 20, 65, 31), ("tt", 40, 32, 33)):
        for pad_item in (1, 2, 3):
            spec = GemmSpec(m, n, k, dt, int(lay[0] == "t"), int(lay[1] == "t"), seed=9400 + pad_item, batch=5,
                            pad_item=pad_item, name=f"items_{dt}_{lay}_{pad_item}")
            mat = inputs.materialize(spec)
            for name in ("64x64_w2x2_m32", "16x64_w1x4_m16"):
                reset_outputs([mat])
                ctx.execute([gemm_of(mat, ctx.find(f"{dt}_{lay}_{name}_c0"))], mode="forced_grouped")
                torch.cuda.synchronize()
                check(mat, label=name)
