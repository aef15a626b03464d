"""Replacing a context's references: buffers taken over by references of the
same shape, sets that grow, shrink and change shape, every pixel type and row
pitch, and refusals that leave the old set in force.  Each set must give the
bits that a fresh context gives."""
import numpy as np
import pytest
import torch

from tests.test_gpu_window import spots, t

pytestmark = pytest.mark.gpu


def image(a, dtype, pad):
    b = np.full((a.shape[0], a.shape[1] + pad), 3, dtype)
    b[:, :a.shape[1]] = a
    return t(b)[:, :a.shape[1]]


@pytest.mark.parametrize("mode,prec", [("ccu", "fp32"), ("ccsn", "fp32"), ("ccu", "fp64")])
def test_sets_replace_each_other(mode, prec):
    from paper_2310_08770_amd import CcptError, Tracker
    print(f"case: {mode} {prec}", flush=True)
    sets = [[(64, 1)], [(64, 2)], [(64, 2), (48, 3)], [(48, 3), (64, 1), (64, 4)], [(48, 5)], [(64, 2)]]
    made = {}
    for s in sets:
        for n, k in s:
            made.setdefault((n, k), spots(3, n, n, 3.0, 400.0 + 90 * k, 20.0, 31 * n + k))
    tr = Tracker(mode=mode, upsample=20, precision=prec)

    def results(tracker, s):
        out = []
        for i, (n, k) in enumerate(s):
            fr = t(made[n, k][0].astype(np.float32))
            out.append(tracker.track(fr, [i] * 3).cpu().numpy())
        return out

    for s in sets:
        refs = [image(np.round(made[n, k][1]), dt, 0) for (n, k), dt in
                zip(s, (np.float32, np.uint16, np.float64))]
        tr.set_reference(refs)
        fresh = Tracker(mode=mode, upsample=20, precision=prec)
        fresh.set_reference(refs)
        for a, b in zip(results(tr, s), results(fresh, s)):
            assert np.array_equal(a, b), s
        fresh.close()
        # refused sets leave this one in force
        before = results(tr, s)
        bad = made[64, 2][1].astype(np.float32)
        bad[7, 9] = np.nan
        with pytest.raises(CcptError):
            tr.set_reference([refs[0], t(bad)])
        if mode == "ccsn":
            bad[7, 9] = -200.0
            with pytest.raises(CcptError):
                tr.set_reference([t(bad)])
        assert all(np.array_equal(a, b) for a, b in zip(before, results(tr, s)))
    tr.close()


def test_long_batches_share_the_record_layout():
    """A stacked batch of 16 or more frames is described in one pass over the
    records: the same fields as frame by frame, views and ids included."""
    from paper_2310_08770_amd import Tracker
    print("case: roi records", flush=True)
    fr, ref = spots(20, 32, 32, 2.5, 500.0, 20.0, 5)
    x = t(np.ascontiguousarray(np.pad(fr, ((0, 0), (0, 2), (0, 3)))).astype(np.float32))[1:, :32, :32]
    tr = Tracker(upsample=20)
    tr.set_reference([t(ref.astype(np.float32)), t((2 * ref).astype(np.float32))])
    ids = [i % 2 for i in range(19)]
    for v, k in ((x, ids), (x, None), (x[::2], None), (x[:17], torch.tensor(ids[:17]))):
        a, n = tr.rois(v, k)
        b, m = tr.rois(list(v), None if k is None else list(k))
        assert n == m
        for i in range(n):
            assert all(getattr(a[i], f) == getattr(b[i], f) for f in ("data", "ny", "nx", "pitch", "dtype",
                                                                      "ref_id")), i
    whole = tr.track(x, ids).cpu().numpy()
    one = np.concatenate([tr.track(x[i:i + 1], ids[i:i + 1]).cpu().numpy() for i in range(19)])
    d = np.dtype([("d", "<f8", (2,)), ("rest", "u1", (56,))])
    assert np.max(np.abs(whole.reshape(-1).view(d)["d"] - one.reshape(-1).view(d)["d"])) <= 1e-12
    tr.close()
