"""Calls on several streams of one GPU that share the library's work buffers: queued without a
wait between them they give what serial calls give, bit for bit."""
import dataclasses

import pytest

from paper_1607_01650_amd import configs as C

from helpers import need_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    return need_gpu()


def _overlapped(torch, calls, rounds=12):
    """Each call's results from serial runs, and from `rounds` runs queued on a stream each."""
    ref = [c() for c in calls]
    streams = [torch.cuda.Stream() for _ in calls]
    torch.cuda.synchronize()
    got = []
    for _ in range(rounds):
        for k, c in enumerate(calls):
            with torch.cuda.stream(streams[k]):
                got.append((k, c()))
    torch.cuda.synchronize()
    for k, out in got:
        assert all(torch.equal(a, b) for a, b in zip(out, ref[k]))


@pytest.mark.parametrize("mode", [0, 1])
def test_pls_on_two_streams(torch, mode):
    from paper_1607_01650_amd import dect
    gen = torch.Generator(device="cuda").manual_seed(3)
    calls = []
    for k, n in ((0, 512), (1, 448)):
        xh, xl = (torch.rand((n, n), generator=gen, device="cuda") * s + o
                  for s, o in ((0.005, 0.02), (0.008, 0.03)))
        p = dataclasses.replace(C.PlsParams(), gamma=(1.0, 1e-4)[mode] * (k + 1), tol=1e-12, mode=mode,
                                max_iter=8)  # (fewer than the iterations between the host's looks)
        calls.append(lambda xh=xh, xl=xl, p=p: dect.pls_decompose(xh, xl, p, report=False)[:2])
    calls.append(lambda: (dect.pls_edge_weights(xl, 0.2, 0.1),))
    _overlapped(torch, calls)


def test_edge_weights3_on_two_streams(torch):
    from paper_1607_01650_amd import dect
    gen = torch.Generator(device="cuda").manual_seed(4)
    xs = [torch.rand((24, 130, 100 + 30 * k), generator=gen, device="cuda") for k in range(2)]
    _overlapped(torch, [lambda x=x: (dect.pls_edge_weights3(x, 0.2, 0.1),) for x in xs])
