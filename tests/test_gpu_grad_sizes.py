"""Adjoint at sizes and frame counts where its kernels split the work
differently, with several references in one call, against the FP64 oracle."""
import numpy as np
import pytest
import torch

from oracle import ccpt_oracle as O
from tests.test_gpu_window import spots, t

pytestmark = pytest.mark.gpu

# The FP32 transforms err by a few 1e-6 of an image's maximum, and the inverse
# Hessian of these spots amplifies an error of the forward pass by less than 100.
TOL = 1e-3


def check(n, count, nrefs, mode, runs=False):
    """`count` frames that repeat two per reference; references in turn, or in
    runs of equal length."""
    from paper_2310_08770_amd import Tracker, decode
    m = O.MODE_CCU if mode == "ccu" else O.MODE_CCSN
    made = [spots(2, n, n, 1.9 if n < 32 else 3.0, 900.0 + 70 * r, 30.0, 17 * n + r) for r in range(nrefs)]
    refs = [a[1].astype(np.float32) for a in made]
    ids = np.arange(count) * nrefs // count if runs else np.arange(count) % nrefs
    which = np.arange(count) // nrefs % 2
    frames = np.stack([made[r][0][w] for r, w in zip(ids, which)]).astype(np.float32)
    rng = np.random.Generator(np.random.PCG64(n + count))
    gd = rng.standard_normal((nrefs, 2, 2))
    gp = rng.standard_normal((nrefs, 2)) * 1e-6
    tr = Tracker(mode=mode, upsample=37, eps=200.0)
    tr.set_reference([t(r) for r in refs])
    fr = t(frames)
    ids_l = [int(i) for i in ids]
    res = tr.track(fr, ids_l)
    gf, gr = tr.track_grad(fr, res, t(gd[ids, which]), t(gp[ids, which]), ref_ids=ids_l)
    only_f = tr.track_grad(fr, res, t(gd[ids, which]), t(gp[ids, which]), want_ref=False, ref_ids=ids_l)[0]
    only_r = tr.track_grad(fr, res, t(gd[ids, which]), t(gp[ids, which]), want_frames=False, ref_ids=ids_l)[1]
    torch.cuda.synchronize()
    assert torch.equal(gf, only_f) and torch.equal(gr, only_r)
    gf = gf.cpu().numpy().reshape(count, n, n)
    gr = gr.cpu().numpy().reshape(nrefs, n, n)
    d = decode(res)["d"]
    tr.close()
    for r in range(nrefs):
        tot = np.zeros((n, n))
        for w in range(2):
            mine = np.flatnonzero((ids == r) & (which == w))
            if mine.size == 0:
                continue
            o = O.track(frames[mine[0]], refs[r].astype(np.float64), 37, mode=m, eps=200.0)
            assert np.max(np.abs(d[mine] - o["d"])) < 1e-3
            gI, gE = O.adjoint(frames[mine[0]], refs[r].astype(np.float64), o, gd[r, w], gp[r, w], mode=m, eps=200.0)
            tot += gE * mine.size
            assert np.max(np.abs(gf[mine] - gI)) <= TOL * np.max(np.abs(gI)), (r, w)
        assert np.max(np.abs(gr[r] - tot)) <= TOL * np.max(np.abs(tot)), r


@pytest.mark.parametrize("n", [108, 162, 324])
def test_sizes_that_8_does_not_divide(n):
    print(f"case: adjoint {n}x{n}", flush=True)
    check(n, 3, 1, "ccu")


@pytest.mark.parametrize("mode", ["ccu", "ccsn"])
@pytest.mark.parametrize("n,count,nrefs,runs", [
    (16, 1, 1, False), (24, 17, 1, False), (54, 16, 2, False), (64, 67, 3, True),
    (128, 33, 2, True), (128, 33, 2, False), (144, 130, 1, False), (192, 3, 1, False),
    (192, 129, 2, True), (162, 258, 1, False), (256, 18, 1, False),
    (512, 31, 2, False)])
def test_runs_and_rounds(n, count, nrefs, runs, mode):
    # one frame; a run and one more; references in turn (runs of 8 and 9) and in
    # runs; a launch of the one-kernel path, of the passes, and of both; frames
    # that fill more than one chunk of the workspace
    print(f"case: adjoint {n}x{n}, {count} frames, {nrefs} references, {mode}", flush=True)
    check(n, count, nrefs, mode, runs)
