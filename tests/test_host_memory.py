"""Calls on a card that has no room: what they report, and that the calls after
them are as if they had not been made."""
import pytest
import torch

from tests._host import host, host_lib  # noqa: F401

E_NOMEM, E_HIP = -6, -4


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
