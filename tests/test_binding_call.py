"""The native way from a Python call to the library (_amap_call): what it hands over, and what it leaves to ctypes.  The library is
replaced by functions that write down what they were given, so no GPU is needed."""
import ctypes as C

import pytest

from paper_2002_12798_amd import binding as B

V, I64 = C.c_void_p, C.c_int64
TABLE = C.POINTER(V)


class Tensor:
    def __init__(self, at):
        self.at = at

    def data_ptr(self):
        if isinstance(self.at, Exception):
            raise self.at
        return self.at


@pytest.fixture
def call():
    """The extension bound to recorders; the real entry points afterwards."""
    seen = []

    def recorder(name, *types):
        def f(*args):
            seen.append((name, *[[a[i] for i in range(2)] if isinstance(a, TABLE) else a for a in args]))
            return 0
        return C.CFUNCTYPE(C.c_int, *types)(f)

    fs = [recorder("execute", TABLE, V, V, V), recorder("multi", TABLE, TABLE, TABLE, C.c_int, V), recorder("fused", V, V, V, I64, V, V),
          recorder("store", V, V, V, I64, V, V, V), recorder("mapped", V, V, V, V, V, V, V), recorder("gather", TABLE, V, V, V, I64, V, V, V)]
    B._call.library(*(C.cast(f, V).value for f in fs))
    B._call.seen = seen
    yield B._call
    L = B.raw
    B._call.library(*(C.cast(f, V).value for f in (L.amap_execute, L.amap_execute_multi, L.amap_gemm_fused, L.amap_gemm_fused_store,
                                                   L.amap_gemm_mapped, L.amap_gemm_gather)))


def _map(*shapes, ops=()):
    m = B.amap_compose(list(shapes), 2, list(ops))
    B._reads(m)
    return m


def test_what_is_handed_over(call):
    m, two = _map((8, 16)), _map((8, 16), (8, 16), ops=[("concat", 0)])
    top = (1 << 63) + 16
    assert call.execute(m, [Tensor(64)], Tensor(top), 7) == 0
    assert call.execute(two, (Tensor(64), Tensor(128)), Tensor(256), 0) == 0
    assert call.execute_multi([m, two], [Tensor(64), Tensor(128)], [Tensor(256), Tensor(512)], 7) == 0
    assert call.gemm(64, m, 128, None, 24, None, 256, 7) == 0
    assert call.gemm(64, m, 128, None, 24, two, 256, 7) == 0
    assert call.gemm(64, m, 128, two, 0, None, 256, 7) == 0
    assert call.gather([64, None], two, 128, None, 24, None, 256, 7) == 0
    assert call.seen == [
        ("execute", [64, None], top, m._at, 7), ("execute", [64, 128], 256, two._at, None),
        ("multi", [64, 128], [256, 512], [m._at, two._at], 2, 7),
        ("fused", 64, m._at, 128, 24, 256, 7), ("store", 64, m._at, 128, 24, two._at, 256, 7), ("mapped", 64, m._at, 128, two._at, None, 256, 7),
        ("gather", [64, None], two._at, 128, None, 24, None, 256, 7)]


@pytest.mark.parametrize("bad", [b"bytes", "text", 1.5, 1 << 64, Tensor(1.5), Tensor(RuntimeError("no storage")), object()], ids=lambda v: type(v).__name__)
def test_what_is_left_to_ctypes(call, bad):
    m, two = _map((8, 16)), _map((8, 16), (8, 16), ops=[("concat", 0)])
    x, out = Tensor(64), Tensor(128)
    calls = [lambda: call.execute(m, [bad], out, 0), lambda: call.execute(m, [x], bad, 0), lambda: call.execute(m, [x], out, bad),
             lambda: call.execute(bad, [x], out, 0), lambda: call.execute(m, bad, out, 0),
             lambda: call.execute(two, [x], out, 0),                                             # a source missing
             lambda: call.execute(m, [x] * 17, out, 0), lambda: call.execute(m, iter([x]), out, 0),
             lambda: call.execute(B.amap_compose([(8, 16)], 2, []), [x], out, 0),                # its sources not asked for yet
             lambda: call.execute_multi([m, two], [x, x], [out], 0), lambda: call.execute_multi([m, bad], [x], [out, out], 0),
             lambda: call.gemm(bad, m, 64, None, 8, None, 128, 0), lambda: call.gemm(64, m, bad, None, 8, None, 128, 0),
             lambda: call.gemm(64, m, 64, bad, 8, None, 128, 0), lambda: call.gemm(64, m, 64, None, bad, None, 128, 0),
             lambda: call.gemm(64, m, 64, None, 8, bad, 128, 0), lambda: call.gemm(64, m, 64, None, 8, None, 128, bad),
             lambda: call.gather([bad], m, 64, None, 8, None, 128, 0), lambda: call.gather([64], bad, 64, None, 8, None, 128, 0)]
    for k, f in enumerate(calls):
        assert f() == -1, k
    assert call.seen == []


def test_the_current_stream_before_and_after_cuda_is_initialised(call):
    from paper_2002_12798_amd import device
    ready = []
    try:
        call.torch(lambda dev: 1000 + dev, lambda: 3, lambda: bool(ready))
        assert call.current_stream() is None and call.execute(_map((8, 16)), [Tensor(64)], Tensor(128), None) == -1
        ready.append(1)
        assert call.current_stream() == 1003
        assert call.execute(_map((8, 16)), [Tensor(64)], Tensor(128), None) == 0 and call.seen[-1][-1] == 1003
    finally:
        import torch
        call.torch(device._raw_stream, device._get_device, torch.cuda.is_initialized)


def test_a_map_given_back_is_not_handed_over(call):
    m = _map((8, 16))
    m.__del__()
    assert call.execute(m, [Tensor(64)], Tensor(128), 0) == -1 and call.gemm(64, m, 64, None, 8, None, 128, 0) == -1 and call.seen == []


def test_a_map_that_leaves_the_list_while_it_is_asked(call):
    """The list's reference may be the last one: the map lives until both of its attributes are read."""
    asked = []

    class Leaves:
        @property
        def _at(self):
            maps.clear()
            asked.append("_at")
            return 64

        @property
        def _reads(self):
            asked.append("_reads")

        def __del__(self):
            asked.append("gone")

    maps = [Leaves()]
    assert call.execute_multi(maps, [Tensor(64)], [Tensor(128)], 0) == -1
    assert asked == ["_at", "_reads", "gone"] and call.seen == []


def test_no_output_is_none(call):
    """An output that is not there is the caller's mistake and raised as one, in a call of one map and of several."""
    from paper_2002_12798_amd import device
    m, x = _map((8, 16)), Tensor(64)
    for outs in ([None], [x, None], [None, x]):   # (one more than there are maps is looked at too)
        assert call.execute_multi([m], [x], outs, 0) == -1
        with pytest.raises(AttributeError):
            device.execute_multi([m], [x], outs, stream=0)
    assert call.seen == []


@pytest.mark.parametrize("stop", [KeyboardInterrupt, SystemExit])
def test_an_interrupt_is_not_taken_for_a_call_to_leave(call, stop):
    """What ends the program passes through; a data_ptr() that raised it is not asked again."""
    from paper_2002_12798_amd import device

    class Stops(Tensor):
        def data_ptr(self):
            self.at -= 1
            if self.at == 63:
                raise stop
            return self.at

    m, x = _map((8, 16)), Tensor(128)
    calls = [lambda: device.execute(m, [Stops(64)], x, stream=0), lambda: device.execute(m, [x], Stops(64), stream=0),
             lambda: device.execute_multi([m], [Stops(64)], [x], stream=0), lambda: device.execute_multi([m], [x], [Stops(64)], stream=0)]
    for f in calls:
        with pytest.raises(stop):
            f()

    def stopped(*args):
        raise stop

    try:
        for fs in ((lambda dev: 1000, lambda: 3, stopped), (lambda dev: 1000, stopped, lambda: True), (stopped, lambda: 3, lambda: True)):
            call.torch(*fs)
            with pytest.raises(stop):
                call.execute(m, [x], x, None)
            with pytest.raises(stop):
                call.current_stream()
    finally:
        import torch
        call.torch(device._raw_stream, device._get_device, torch.cuda.is_initialized)
    assert call.seen == []


def test_only_maps_hold_a_map_s_address(call):
    """What is given back: a map's address with the map; a graph has none, before and after."""
    layout = B.LayoutGraph()
    graph = B.GraphDME([("input", (8, 16))], [0], 2)
    for owner in (layout, graph):
        owner.__del__()
        assert owner._h is None and not hasattr(owner, "_at")
