"""The instance count of a synchronous binning on its way to the host: refused while the
stream is being captured without harm to the capture, and read back right by contexts that
come and go on several threads and streams."""
import threading

import pytest

from tests.gpu_util import log
from tests.test_gpu_bin_refused import _case

pytestmark = pytest.mark.gpu


def test_refused_under_capture_and_the_capture_goes_on():
    import torch
    from paper_2411_09156_amd._lib import GESR_ERR_HIP, GesrError
    log("[gpu] synchronous binning under capture")
    n = 5000
    rast, sp = _case(n, [(200, 150)])
    want = rast.forward(sp)
    proj, m_cap = want["proj"], want["bins"]["m_cap"]
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        rast.bin(proj, n, m_cap=m_cap, sync=False)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for static in (False, True):
            with pytest.raises(GesrError, match="captured") as err:
                rast.bin(proj, n, m_cap=m_cap, static_scratch=static)
            assert err.value.status == GESR_ERR_HIP
        bins = rast.bin(proj, n, m_cap=m_cap, sync=False)
    for _ in range(3):
        for k in ("val_sorted", "ranges", "worklist", "counters"):
            bins[k].zero_()
        graph.replay()
        torch.cuda.synchronize()
        again = rast.bin(proj, n, m_cap=m_cap)
        assert again["M"] == want["bins"]["M"]
        listed = int(again["counters"][3])
        assert torch.equal(bins["val_sorted"][:listed], again["val_sorted"][:listed])
        for k in ("ranges", "worklist", "counters"):
            assert torch.equal(bins[k], again[k]), k


def test_contexts_on_threads_and_streams_read_their_own_counts():
    import torch
    log("[gpu] counts read back on six threads")
    cases = [(700, [(90, 70)]), (3000, [(200, 150)]), (5000, [(333, 215), (64, 48)])]
    want = []
    for n, sizes in cases:
        rast, sp = _case(n, sizes)
        want.append(rast.forward(sp))
    torch.cuda.synchronize()
    assert len({f["bins"]["M"] for f in want}) == len(cases)
    errors = []

    def work(k):
        try:
            n, sizes = cases[k % len(cases)]
            ref = want[k % len(cases)]
            stream = torch.cuda.Stream()
            with torch.cuda.stream(stream):
                for _ in range(12):
                    rast, sp = _case(n, sizes)  # a context per pass, destroyed with it
                    f = rast.forward(sp)
                    assert f["bins"]["M"] == ref["bins"]["M"]
                    stream.synchronize()
                    assert torch.equal(f["image"], ref["image"])
                    del rast, f
        except Exception as e:  # noqa: BLE001 (told to the main thread)
            errors.append((k, repr(e)))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(6)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
