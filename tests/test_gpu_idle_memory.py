"""Device memory of closed scenes, kept for the next ones: scenes made in turn and from two threads at once compute what
the first scene of a process computes, and the memory is bounded and given back."""
import threading
import time

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


def test_close_waits_for_every_stream():
    """A closed scene's memory goes to the next scene, so closing waits for work that may use it: on the scene's stream,
    on the one it had before, and on one the library never saw."""
    from paper_2306_06946_amd import icr
    sc = make_scene("tiny")
    streams = [torch.cuda.Stream() for _ in range(3)]
    for busy in range(3):
        s = icr.Scene(streams[0].cuda_stream)
        s.assemble(sc)
        s.factor()
        s.set_stream(streams[1].cuda_stream)
        torch.cuda.synchronize()
        done = torch.cuda.Event()
        with torch.cuda.stream(streams[busy]):
            torch.cuda._sleep(100_000_000)
            done.record()
        s.close()
        assert done.query(), busy


@pytest.mark.parametrize("mode", ["global", "thread_local"])
def test_close_and_reuse_beside_a_capture(mode):
    """Another thread closes scenes, takes their memory and gives it back while a graph is captured."""
    from paper_2306_06946_amd import icr
    sc = make_scene("tiny")
    x, y = torch.ones(1000, device="cuda"), torch.zeros(1000, device="cuda")
    y.add_(x)
    y.zero_()

    def scene():
        s = icr.Scene(torch.cuda.Stream().cuda_stream)
        s.assemble(sc)
        s.factor()
        return s

    live = [scene() for _ in range(3)]
    torch.cuda.synchronize()
    graph, stream, errs = torch.cuda.CUDAGraph(), torch.cuda.Stream(), []

    def work():
        try:
            for s in live:
                s.close()
            icr.release_idle()
        except Exception as e:   # noqa: BLE001 - reported by the assert below
            errs.append(e)

    with torch.cuda.stream(stream):
        graph.capture_begin(capture_error_mode=mode)
        y.add_(x)
        t = threading.Thread(target=work)
        t.start()
        t.join()
        y.add_(x)
        graph.capture_end()
    torch.cuda.synchronize()
    assert not errs
    for k in range(1, 4):
        graph.replay()
        torch.cuda.synchronize()
        assert float(y[0]) == 2.0 * k


def test_idle_memory_goes_when_its_time_is_up_also_beside_a_capture():
    from paper_2306_06946_amd import icr
    sc = make_scene("tiny")
    x, y = torch.ones(1000, device="cuda"), torch.zeros(1000, device="cuda")
    y.add_(x)
    y.zero_()
    icr.release_idle()
    base = _free()
    s = icr.Scene()
    s.assemble(sc)
    s.factor()
    s.reserve(1200)
    closed = time.monotonic()
    s.close()
    kept = base - _free()
    assert kept > 256 << 20
    graph, stream = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    time.sleep(max(0.0, closed + 9.5 - time.monotonic()))
    with torch.cuda.stream(stream):
        graph.capture_begin()   # in the mode that forbids most calls of every thread
        y.add_(x)
        time.sleep(max(0.0, closed + 11.5 - time.monotonic()))
        y.add_(x)
        graph.capture_end()
    torch.cuda.synchronize()
    assert base - _free() < kept // 4
    for k in range(1, 4):
        graph.replay()
        torch.cuda.synchronize()
        assert float(y[0]) == 2.0 * k


STEPS = {   # scene, options of its steps
    "fast": ("medium", dict(graph=False)),
    "graph": ("medium", dict()),
    "standard": ("tiny", dict(standard=True)),
    "per constraint": ("tiny", dict(per_constraint=True)),
    "mixed": ("medium", "mixed"),
    "pairs": ("stacked_small", dict()),
}


@pytest.mark.parametrize("kind", STEPS)
def test_steps_on_used_memory(kind):
    """A time step gives the same bits on memory that other scenes' steps left as on fresh memory."""
    from paper_2306_06946_amd import icr
    cfg, opts = STEPS[kind]
    opts = dict(precision=icr.FP32_IR) if opts == "mixed" else opts

    def run(cfg, opts, poison=False):
        sc = make_scene(cfg)
        s = icr.scene_from_dict(sc)
        for _ in range(2):
            s.step(sc["obstacle"], sc["n_contacts"], 3, 20, 0.0, 8, report=False, **opts)
        q, v, _ = s.get_state()
        r = s.step_results(sc["n_contacts"], with_WH=True)
        out = [x.cpu() for x in (q, v, *r.values())]
        if poison:
            s.set_state(torch.full_like(q, float("nan")), torch.full_like(v, float("nan")), 0.0)
        s.close()
        return out

    print(f"[gpu] used memory {kind}", flush=True)
    icr.release_idle()
    want = run(cfg, opts)
    icr.release_idle()
    for other in STEPS:   # every kind's buffers, some of them of this scene's sizes
        c, o = STEPS[other]
        run(c, dict(precision=icr.FP32_IR) if o == "mixed" else o, poison=True)
    for a, b in zip(run(cfg, opts), want):
        assert torch.equal(a, b)
