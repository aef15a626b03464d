"""Default launches of a call against launches of a set chunk size: the 256 x 256
correlation of every frame is the one that units of the default's former size
select (one kernel, or three passes for a last unit below the threshold), so
the spectra are equal and only the order of FP64 sums may differ."""
import numpy as np
import pytest
import torch

from tests.test_gpu_window import spots, t

pytestmark = pytest.mark.gpu

# FP64 sums of at most 2^17 terms in another order, relative to the peak, over
# a curvature that is above 1e-3 of it for these spots
TOL_PX = 1e-9


# 192 MB by 256 x 256 frame: two FP32 half spectra, and for the split precisions
# a 32-bit word per pixel and a complex value per row
SPECTRA = 2 * 256 * 129 * 8
FP32_UNIT = (192 << 20) // SPECTRA
SPLIT_UNIT = (192 << 20) // (SPECTRA + 256 * 256 * 4 + 256 * 8)


@pytest.mark.parametrize("prec,unit,count,ny,nx", [
    ("fp32", FP32_UNIT, 100, 256, 256),   # one unit below the threshold
    ("fp32", FP32_UNIT, 481, 256, 256),   # 381 in one kernel, 100 in passes
    ("fp32", FP32_UNIT, 762, 256, 256),   # units that are whole
    ("fp32", FP32_UNIT, 961, 256, 256),   # a quarter over a default launch, and one frame
    ("bf16x2", SPLIT_UNIT, 360, 256, 256),
    ("bf16x2", SPLIT_UNIT, 1000, 256, 256),
    ("fp32", 95, 100, 512, 512),
    ("fp32", 764, 965, 128, 256),
    ("fp64", 188, 200, 256, 256)])
@pytest.mark.parametrize("streams", [1, 2])
def test_default_launches_match_units(prec, unit, count, ny, nx, streams):
    print(f"case: {count} frames of {ny}x{nx}, {prec}, units of {unit}, {streams} streams", flush=True)
    from paper_2310_08770_amd import Tracker, decode
    fr, ref = spots(5, ny, nx, 3.0, 900.0, 30.0, 5)
    fr = t(np.round(fr).astype(np.uint16))
    frames = [fr[i % 5] for i in range(count)]
    tr = Tracker(upsample=37, precision=prec, streams=streams)
    tr.set_reference(t(ref))
    got = decode(tr.track(frames, [0] * count))
    tr.set_plan(ny, nx, chunk=unit)
    want = decode(tr.track(frames, [0] * count))
    torch.cuda.synchronize()
    assert np.array_equal(got["p"], want["p"]) and np.array_equal(got["status"], want["status"])
    assert np.max(np.abs(got["d"] - want["d"])) < TOL_PX
    tr.close()
