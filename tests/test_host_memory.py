"""Calls on a card that has no room: what they report, and that the calls after
them are as if they had not been made."""
import ctypes

import pytest
import torch

from tests._host import host, host_lib  # noqa: F401

E_NOREF, E_NOMEM, E_HIP = -3, -6, -4


def refused(call, codes=(E_NOMEM,)):
    from paper_2310_08770_amd import CcptError
    with pytest.raises(CcptError) as e:
        call()
    assert e.value.code in codes, e.value


def frames(count, n):
    return [torch.zeros(n, n)] * count, [0] * count


def test_a_refused_workspace_is_not_the_next_calls_error(host):
    tr = host.tracker()
    tr.set_reference([torch.ones(512, 512), torch.ones(16, 16)], stream=0)
    small = [torch.zeros(16, 16)]
    tr.track(small, [1], stream=0)
    host.limit(host.live() + (4 << 20))
    refused(lambda: tr.track(*frames(200, 512), stream=0))  # default and small launches alike
    tr.track(small, [1], stream=0)
    refused(lambda: tr.track(*frames(200, 512), stream=0))
    host.limit(2**63)
    host.launches()
    tr.track(*frames(200, 512), stream=0)
    assert host.launches()


def test_a_refused_reference_is_not_the_next_calls_error(host):
    tr = host.tracker()
    host.limit(host.live())
    refused(lambda: tr.set_reference(torch.ones(64, 64), stream=0), (E_NOMEM, E_HIP))
    host.limit(2**63)
    tr.set_reference(torch.ones(64, 64), stream=0)
    tr.track(*frames(3, 64), stream=0)
    host.limit(host.live())
    refused(lambda: tr.set_reference(torch.ones(512, 512), stream=0), (E_NOMEM, E_HIP))
    host.limit(2**63)
    tr.set_reference(torch.ones(64, 64), stream=0)
    tr.track(*frames(3, 64), stream=0)


def test_refused_buffers_of_other_calls(host):
    tr = host.tracker()
    tr.set_reference(torch.ones(64, 64), stream=0)
    fr = torch.zeros(5, 64, 64)
    fwd = tr.track(fr, stream=0)
    g = torch.ones(5, 2, dtype=torch.float64)
    calls = [lambda: tr.track_grad(fr, fwd, g, stream=0), lambda: tr.fisher(torch.ones(64, 64), stream=0),
             lambda: tr.mean_aligned(torch.zeros(300, 64, 64), torch.zeros(300, 72, dtype=torch.uint8), stream=0),
             lambda: tr.track_update(fr[0], 0.1, stream=0), lambda: tr.autotune(64, 20000, stream=0)]
    for call in calls:
        host.limit(host.live())
        refused(call, (E_NOMEM, E_HIP))
        host.limit(2**63)
        tr.track(fr, stream=0)
        call()


# 192 MB by a 512 x 512 frame's two FP32 half spectra
SMALL = (192 << 20) // (2 * 512 * 257 * 8)


def counts(host):
    return [l[2] for l in host.launches()]


def test_smaller_launches_without_room_and_default_ones_with_it(host):
    tr = host.tracker()
    tr.set_reference(torch.ones(512, 512), stream=0)
    call = frames(200, 512)
    tr.track(call[0][:1], [0], stream=0)
    assert counts(host) == [1]
    host.limit(host.live() + (300 << 20))
    tr.track(*call, stream=0)
    assert counts(host) == [SMALL, SMALL, 200 - 2 * SMALL]
    # the call succeeded: no error is left of the workspace it did without
    assert host.lib.ccpt_last_error(tr._h, None, 0) == 0
    # the same room: not asked again
    asked = host.asked()
    for _ in range(3):
        tr.track(*call, stream=0)
        assert counts(host) == [SMALL, SMALL, 200 - 2 * SMALL]
    assert host.asked() == asked
    # more room while the stream is captured: allocations have to wait
    host.limit(2**63)
    graph = ctypes.c_void_p()
    host.lib.hipStreamBeginCapture(None, 0)
    tr.track(*call, stream=0)
    host.lib.hipStreamEndCapture(None, ctypes.byref(graph))
    host.lib.hipGraphDestroy(graph)
    assert host.asked() == asked
    # and after it: the default launches again
    tr.track(*call, stream=0)
    assert counts(host) == [200]
    assert host.lib.ccpt_last_error(tr._h, None, 0) == 0


def test_a_workspace_in_hand_is_used(host):
    # a larger call was refused; one that fits what the context has is not affected
    tr = host.tracker()
    tr.set_reference(torch.ones(512, 512), stream=0)
    tr.track(*frames(150, 512), stream=0)
    assert counts(host) == [150]
    host.limit(host.live() + (1 << 20))
    tr.track(*frames(200, 512), stream=0)  # refused; the small launches' workspace instead
    assert counts(host) == [SMALL, SMALL, 200 - 2 * SMALL]
    host.limit(2**63)
    tr.track(*frames(150, 512), stream=0)
    assert counts(host) == [150]
    tr.track(*frames(200, 512), stream=0)
    assert counts(host) == [200]


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_tables_are_whole_or_absent(host, precision):
    # each allocation of the first set_reference refused in turn, then the same call
    from paper_2310_08770_amd import CcptError
    k = 0
    while True:
        k += 1
        tr = host.tracker(precision=precision)
        host.refuse(k)
        try:
            tr.set_reference(torch.ones(64, 64), stream=0)
        except CcptError as e:
            assert e.code in (E_NOMEM, E_HIP)
        else:
            break
        tr.set_reference(torch.ones(64, 64), stream=0)
        tr.track(*frames(3, 64), stream=0)
        assert not host.no_tables(), k
    assert k > 5


def test_a_context_makes_the_grid_table_it_reads(host):
    m = 1536  # grid points per axis: 16 floats each in FP32, 24 doubles in FP64
    for precision, grid in (("fp32", m * 16 * 4), ("fp64", m * 24 * 8)):
        tr = host.tracker(precision=precision, upsample=1024)
        before = host.live()
        tr.set_reference(torch.ones(16, 16), stream=0)
        assert grid <= host.live() - before < grid + (32 << 10)


def test_a_set_that_fails_leaves_no_part_of_it(host):
    # two larger references, each allocation refused in turn: a caller that still
    # holds the old set sizes its gradient arrays by it
    fr = torch.zeros(3, 512, 512)
    g = torch.ones(3, 2, dtype=torch.float64)
    fwd = torch.zeros(3, 72, dtype=torch.uint8)
    k = 0
    while True:
        k += 1
        tr = host.tracker()
        tr.set_reference(torch.ones(16, 16), stream=0)
        host.refuse(k)
        try:
            tr.set_reference([torch.ones(512, 512), torch.ones(512, 512)], stream=0)
        except Exception:
            host.refuse(0)
            # (the old set, of another size, or none)
            refused(lambda: tr.track_grad(fr, fwd, g, stream=0), (E_NOREF, -1))
        else:
            break
    assert k > 5
