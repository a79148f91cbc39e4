"""Plain row pieces as small kernel arguments: one piece of up to five loops, up to three pieces of four that differ in where they read
and write.  The host replay compares the decode of every piece that has such a form (test_plan_replay.py walks random maps through
it); here whole launches walked on the CPU, and on the GPU those on both sides of each limit, bit for bit against the oracle."""
import os
import subprocess

import numpy as np
import pytest

from oracle import oracle
from paper_2002_12798_amd import binding as B

T, R, S = "transpose", "reshape", "slice"
ONE = [
    # source shape, element size, chain, small argument; loops counted after those that continue one another are one
    ((64, 64), 4, [], True),                                                          # one loop
    ((3, 5, 7, 8), 2, [(T, (0, 2, 1, 3))], True),                                     # rows of one vector
    ((2, 3, 5, 7, 16), 4, [(T, (3, 2, 1, 0, 4))], True),                              # five loops
    ((2, 3, 2, 5, 3, 16), 4, [(T, (4, 3, 2, 1, 0, 5))], False),                       # six
    ((9, 33, 64), 2, [(S, 1, 1, 32, 1)], True),                                       # an origin in the source
    ((9, 33, 64), 2, [(S, 0, 8, -1, -1)], False),                                     # backwards
    ((1, 40), 4, [("tile", 0, 9)], True),                                             # a loop that stands still in the source
    ((700, 8, 3072), 2, [(T, (1, 0, 2))], False),                                     # 34 MB
]


@pytest.fixture(scope="module")
def replay(tmp_path_factory):
    """The library's launch of the kernel, walked on the CPU (rows_few_replay.cpp)."""
    import torch
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    exe = str(tmp_path_factory.mktemp("few") / "rows_few_replay")
    rt_dirs = [os.path.join(os.path.dirname(torch.__file__), "lib"), "/opt/rocm/lib"]
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-Wno-unknown-pragmas", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I", os.path.join(root, "include"), "-I", os.path.join(root, "paper_2002_12798_amd", "csrc"),
                    os.path.join(root, "tests", "rows_few_replay.cpp"), "-o", exe, B.LIB_PATH, "-rdynamic", "-Wl,--allow-shlib-undefined"]
                   + [f"-Wl,-rpath,{d}" for d in [os.path.dirname(B.LIB_PATH)] + rt_dirs], check=True)
    env = dict(os.environ, LD_LIBRARY_PATH=":".join(rt_dirs + [os.environ.get("LD_LIBRARY_PATH", "")]))

    def run(es, kernel, *maps):
        r = subprocess.run([exe, str(es), kernel, *maps], capture_output=True, text=True, env=env, timeout=120)
        assert (r.returncode, r.stdout.strip()) == (0, "OK"), (r.stdout, r.stderr)
    return run


@pytest.mark.parametrize("es", [2, 4])
@pytest.mark.parametrize("kernel, maps", [
    # pieces of whole workgroups, of one vector more and less, of less than one; outputs in any order in memory
    ("few", ["4,8,8,64,12,0"]), ("few", ["5,7,3,24,02,0"]), ("few", ["1,1,1,16,--,0"]),
    ("few", ["4,8,8,64,12,0", "4,8,8,64,12,1", "4,8,8,64,12,2"]), ("few", ["5,7,3,24,02,2", "5,7,3,24,02,0", "5,7,3,24,02,1"]),
    ("few", ["1,1,257,8,--,1", "1,1,257,8,--,0"]), ("few", ["3,5,17,8,01,0", "3,5,17,8,01,1", "3,5,17,8,01,2"]), ("few", ["1,1,1,16,--,2", "1,1,1,16,--,1", "1,1,1,16,--,0"]),
    # as many vectors, but in another order; four pieces
    ("other", ["6,6,6,64,12,0", "6,6,6,64,01,1"]), ("other", ["6,6,6,64,12,0", "6,6,6,64,12,1", "6,6,6,64,02,2"]), ("other", ["4,8,8,64,12,0", "4,8,8,64,--,1"]),
    ("other", [f"2,3,4,16,12,{i}" for i in range(4)]),
])
def test_the_launch_replayed(replay, kernel, maps, es):
    replay(es, kernel, *maps)


def _run(shapes, es, chains, dsts=None):
    """The outputs of one execute or execute_multi call, in a buffer with guards, and the oracle's."""
    import torch
    from paper_2002_12798_amd import device
    rng = np.random.default_rng(11)
    src = rng.integers(0, 1 << (8 * es), shapes, dtype=np.uint64).astype({2: np.uint16, 4: np.uint32}[es])
    maps = [B.amap_compose([shapes], es, c) for c in chains]
    for m in maps:
        assert B.amap_plan_selfcheck(m) == 0
    outs, room = [], []
    for m in maps:
        n = int(np.prod(B.dst_shape(m)))
        pad = 512 // es
        buf = torch.full((n + 2 * pad,), 0x5A5A, dtype={2: torch.int16, 4: torch.int32}[es], device="cuda")
        outs.append(buf[pad:pad + n].view(B.dst_shape(m)))
        room.append((buf, pad, n))
    x = device.to_device(src)
    print(f"[gpu] rows, small argument: {shapes} {chains}", flush=True)
    if len(maps) == 1:
        device.execute(maps[0], [x], outs[0])
    else:
        device.execute_multi(maps, [x], outs)
    torch.cuda.synchronize()
    for (buf, pad, n), out, chain in zip(room, outs, chains):
        assert (buf[:pad] == 0x5A5A).all() and (buf[pad + n:] == 0x5A5A).all()
        assert np.array_equal(device.to_host(out), oracle.run_chain([src], chain) if chain else src)


@pytest.mark.gpu
@pytest.mark.parametrize("shape, es, chain, few", ONE)
def test_one_piece(shape, es, chain, few, monkeypatch, capfd):
    monkeypatch.setenv("AMAP_PLAN_TRACE", "1")
    capfd.readouterr()
    _run(shape, es, [chain])
    lines = [x for x in capfd.readouterr().err.splitlines() if x.startswith("amap launch")]
    assert len(lines) == 1 and lines[0].endswith("few loops") == few, lines


def heads(b, s, n, h, d):
    return (b, s, n * h * d), [[(R, (b, s, n, h, d)), (T, (2, 0, 3, 1, 4)), (S, 0, t, t + 1, 1), (R, (b, h, s, d))] for t in range(n)]


@pytest.mark.gpu
@pytest.mark.parametrize("args, es, few", [((2, 33, 3, 4, 32), 4, True), ((3, 70, 2, 5, 24), 2, True), ((1, 1, 3, 1, 8), 2, True),
                                           ((2, 40, 4, 2, 16), 2, False),                       # four outputs
                                           ((8, 1000, 3, 12, 64), 2, False)])                   # 36 MB
def test_alike_pieces(args, es, few, monkeypatch, capfd):
    monkeypatch.setenv("AMAP_PLAN_TRACE", "1")
    capfd.readouterr()
    _run(*(lambda shape, chains: (shape, es, chains))(*heads(*args)))
    lines = [x for x in capfd.readouterr().err.splitlines() if x.startswith("amap launch")]
    assert len(lines) == 1 and lines[0].endswith("few loops") == few, lines


@pytest.mark.gpu
def test_pieces_that_are_not_alike(monkeypatch, capfd):
    shape = (6, 40, 64)
    monkeypatch.setenv("AMAP_PLAN_TRACE", "1")
    capfd.readouterr()
    _run(shape, 4, [[(T, (1, 0, 2))], [(S, 0, 0, 3, 1), (T, (1, 0, 2))]])
    lines = [x for x in capfd.readouterr().err.splitlines() if x.startswith("amap launch")]
    assert len(lines) == 1 and not lines[0].endswith("few loops"), lines
