"""Calls of two threads on one device, each on a stream and with arrays of its own:
streams, lengths, headers and values equal those of the same calls in one thread."""
import threading

import pytest

from tests.gpu_common import gpu

pytestmark = pytest.mark.gpu


def _calls(torch, mgc, x, whole):
    """One round of calls that read results or headers back, and what they return."""
    s = mgc.compress(x, 1e-3)
    h = mgc.hx_compress(whole)
    z = mgc.zfp_compress(x, 8.0)
    y = mgc.decompress(s)
    return [s, h, z, y, mgc.hx_decompress(h), mgc.zfp_decompress(z), mgc.header_info(s), mgc.hx_header(h)]


def test_two_threads_on_two_streams():
    torch, mgc = gpu()
    gen = torch.Generator(device="cuda").manual_seed(3)
    shapes = [(65, 66, 67), (130, 90)]
    xs = [torch.randn(s, device="cuda", generator=gen).cumsum(0) for s in shapes]
    ints = [torch.randint(-50, 50 * (k + 1), (70000 + 5000 * k,), device="cuda", dtype=torch.int32, generator=gen)
            for k in range(2)]
    wrong, got = [], [[], []]
    torch.cuda.synchronize()

    def work(k):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for _ in range(20):
                    got[k].append(_calls(torch, mgc, xs[k], ints[k]))
                torch.cuda.current_stream().synchronize()
        except Exception as e:  # noqa: BLE001
            wrong.append("thread %d: %s" % (k, e))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    [t.start() for t in threads]
    [t.join() for t in threads]
    assert not wrong, wrong
    for k in range(2):
        ref = _calls(torch, mgc, xs[k], ints[k])
        for r in got[k]:
            for a, b in zip(r, ref):
                assert torch.equal(a, b) if torch.is_tensor(a) else a == b
