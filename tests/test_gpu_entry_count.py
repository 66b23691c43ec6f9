"""The host entry count of tgs_bin, read back while the rest of the stream is
being built: exact counts from several threads on their own streams, more calls
at once than the library keeps read-back slots, with streams equal to a
single-threaded call's; a count above the capacity is an error in every order;
a stream that is being captured is refused and stays usable."""
import ctypes
import threading

import numpy as np
import pytest
import torch

import oracle
import scenes

pytestmark = pytest.mark.gpu

tg = pytest.importorskip("paper_2609_03613_amd")
from paper_2609_03613_amd import _lib as L  # noqa: E402


def scene(n, seed, W=160, H=128):
    dev = torch.device("cuda:0")
    splats, info = scenes.random_splats(n, W, H, seed=seed)
    cam = scenes.camera(np.eye(3), np.zeros(3), 100.0, 100.0, W / 2, H / 2, W, H)
    M = oracle.count_entries(scenes.info_rects(info))
    return torch.as_tensor(splats).to(dev), torch.as_tensor(info.view(np.int32)).to(dev), cam, M


@pytest.mark.parametrize("threads", [2, 20])
def test_counts_from_threads_and_streams(threads):
    work = [scene(200 + 137 * i, i) for i in range(threads)]
    want = []
    for s, i, cam, M in work:
        b = tg.Renderer(cam, tg.Params(), device=s.device).bin(s, i)
        want.append(b.pairs[:M].clone())
    torch.cuda.synchronize()
    got, errors = [None] * threads, []
    gate = threading.Barrier(threads)

    def run(k):
        try:
            s, i, cam, M = work[k]
            stream = torch.cuda.Stream()
            with torch.cuda.stream(stream):
                r = tg.Renderer(cam, tg.Params(), device=s.device)
                gate.wait(30)
                for _ in range(5):
                    b = r.bin(s, i)
                    assert b.num_entries == M
                stream.synchronize()
                got[k] = b.pairs[:M].clone()
                stream.synchronize()
        except BaseException as e:  # noqa: BLE001 (reported below)
            errors.append(e)

    ts = [threading.Thread(target=run, args=(k,)) for k in range(threads)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not errors
    for a, b in zip(got, want):
        assert torch.equal(a, b)


@pytest.mark.parametrize("order", ["binned", "global"])
@pytest.mark.parametrize("n", [0, 1, 900])
def test_count_against_the_capacity(order, n):
    s, i, cam, M = scene(n, 3) if n else (torch.zeros((0, 16), device="cuda:0"),
                                          torch.zeros((0, 4), dtype=torch.int32, device="cuda:0"), scene(1, 3)[2], 0)
    r = tg.Renderer(cam, tg.Params(), device=s.device)
    o = {"global": L.ORDER_GLOBAL, "binned": L.ORDER_BINNED}[order]
    for cap, expect in ((M, 0), (M - 1, L.TGS_ERR_CAPACITY), (0, L.TGS_ERR_CAPACITY if M else 0)):
        if cap < 0:
            continue
        b = r._new_binned(o, cap)
        ws = r._workspace(o, n, cap)
        m = ctypes.c_int64(-1)
        pr = L.Projected(s.data_ptr() or None, i.data_ptr() or None, n)
        st = L.lib().tgs_bin(ctypes.byref(pr), ctypes.byref(r.ccam), ctypes.byref(r.cparams), o,
                             ctypes.c_void_p(ws.data_ptr()), ws.numel(), ctypes.byref(b.c()), ctypes.byref(m),
                             ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
        assert st == expect
        assert m.value == M
        torch.cuda.synchronize()
        assert int(b.counters[0]) == M and int(b.counters[2]) == (1 if M > cap else 0)


def test_captured_stream_is_refused():
    s, i, cam, M = scene(500, 9)
    r = tg.Renderer(cam, tg.Params(), device=s.device)
    r.bin(s, i)  # buffers
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    keep = torch.zeros(1, device=s.device)
    with torch.cuda.graph(g):
        keep.add_(1.0)
        with pytest.raises(tg.TileGSError):
            r.bin(s, i)
    g.replay()
    assert r.bin(s, i).num_entries == M
    torch.cuda.synchronize()
    assert float(keep) == 1.0
