"""Device memory of closed scenes, kept for the next ones: scenes made in turn and from two threads at once compute what
the first scene of a process computes, and the memory is bounded and given back."""
import threading

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2306_06946_amd.scenes import make_scene  # noqa: E402

pytestmark = pytest.mark.gpu

CONFIGS = ["tiny", "medium"]


def _wh(sc, count, stream=None):
    from paper_2306_06946_amd import icr
    pick = np.asarray(sc["candidates"])[:: max(1, len(sc["candidates"]) // count)].astype(np.int32)
    stream = stream or torch.cuda.current_stream()
    with torch.cuda.stream(stream):
        s = icr.Scene(stream.cuda_stream)
        s.assemble(sc)
        s.factor()
        WH = torch.zeros(9 * len(pick) ** 2, dtype=torch.float64, device="cuda")
        s.build_WH(torch.from_numpy(pick).cuda(), WH)
        out = WH.cpu().numpy()
        s.close()
    return out


def _free():
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


@pytest.mark.parametrize("counts", [(40, 160), (160, 40)], ids=str)
def test_reused_memory(counts):
    from paper_2306_06946_amd import icr
    scs = [make_scene(c) for c in CONFIGS]
    icr.release_idle()
    want = {}
    for sc in scs:
        for n in counts:
            want[id(sc), n] = _wh(sc, n)
            icr.release_idle()
    for _ in range(2):
        for n in counts:
            for sc in scs:
                assert np.array_equal(_wh(sc, n), want[id(sc), n])
    got, errs = [], []

    def work(k):
        try:
            st = torch.cuda.Stream()
            for i in range(6):
                sc, n = scs[(i + k) % 2], counts[(i // 2 + k) % 2]
                got.append(np.array_equal(_wh(sc, n, st), want[id(sc), n]))
        except Exception as e:   # noqa: BLE001 - reported by the assert below
            errs.append(e)

    ts = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    [t.start() for t in ts]
    [t.join() for t in ts]
    assert not errs and len(got) == 12 and all(got)


def test_bounded_and_given_back():
    from paper_2306_06946_amd import icr
    sc = make_scene("tiny")
    _wh(sc, 40)
    icr.release_idle()
    base = _free()
    live = []
    for _ in range(14):   # 14 scenes with room for 1200 contacts each: about 0.5 GB of contact work space a scene
        s = icr.Scene()
        s.assemble(sc)
        s.factor()
        s.reserve(1200)
        live.append(s)
    held = base - _free()
    assert held > 5 << 30
    [s.close() for s in live]
    kept = base - _free()
    assert 0 < kept <= (4 << 30) + (256 << 20)
    icr.release_idle()
    assert base - _free() <= 256 << 20
