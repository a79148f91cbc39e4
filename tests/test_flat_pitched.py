"""Transposing maps whose dst rows begin an odd number of elements apart, further than they are long (channels padded or joined
to an odd number): column-blocked flat tiles that store row by row.  On the CPU every lane of the planned launches is replayed,
on the GPU the result is compared with the oracle, bit for bit."""
import numpy as np
import pytest

from oracle import oracle
from paper_2002_12798_amd import binding as B


def tokens(b, c, s, lo, hi, pad):
    return [(b, c, s, s)], [("transpose", (0, 2, 3, 1)), ("reshape", (b, s * s, c)), ("slice", 1, lo, hi, 1), ("pad", (0, 0, 0), (0, 0, pad), 9)]


CASES = [
    tokens(3, 24, 35, 153, 1072, 1),                 # an odd number of positions, cropped
    tokens(2, 24, 32, 128, 896, 1),                  # source rows of whole vectors
    tokens(1, 8, 8, 0, 64, 1),                       # one block of 64 rows, the fewest columns
    tokens(2, 130, 10, 2, 67, 3),                    # several blocks of columns, 65 rows
    tokens(1, 75, 17, 0, 289, 2),                    # odd rows, pitch 77
    ([(2, 16, 10, 9)], [("transpose", (0, 2, 3, 1)), ("pad", (0, 0, 0, 1), (0, 0, 0, 0), 5)]),             # dst begins at element 1
    ([(2, 24, 12, 11), (2, 33, 12, 11)], [("concat", 1), ("transpose", (0, 2, 3, 1))]),                   # two sources, pitch 57
    ([(2, 40, 70)], [("transpose", (0, 2, 1)), ("pad", (0, 1, 0), (0, 0, 5), 1)]),                          # 70 rows per batch point
    ([(130, 64)], [("transpose", (1, 0)), ("slice", 0, 63, -1, -1), ("pad", (0, 0), (0, 1), 0)]),         # rows walked backwards
]


ODD_ROWS = (0, 4)   # source rows that begin at odd elements: 2-byte elements keep their forms
NOT_FLAT = 8        # (a source walked backwards)


def _planned(case, es, monkeypatch, capfd):
    shapes, ops = CASES[case]
    monkeypatch.setenv("AMAP_PLAN_TRACE", "1")
    monkeypatch.setenv("AMAP_FLAT", "2")   # also where a call is small enough to do without
    capfd.readouterr()
    m = B.amap_compose(shapes, es, ops)
    err = capfd.readouterr().err
    monkeypatch.delenv("AMAP_PLAN_TRACE")
    monkeypatch.delenv("AMAP_FLAT")
    return shapes, ops, m, err


@pytest.mark.parametrize("es", [2, 4])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_replay(case, es, monkeypatch, capfd):
    _, _, m, err = _planned(case, es, monkeypatch, capfd)
    assert ("flat-blocked-dst" in err.split("plan: begin")[-1]) == (case != NOT_FLAT and (es == 4 or case not in ODD_ROWS))
    assert B.amap_plan_selfcheck(m) == 0 and B.amap_check_cover(m) == (0, 0)


@pytest.mark.parametrize("es, channels, size, batch, pad, blocked", [
    # MB of dst in pieces that begin at any element
    (4, (17, 96), 16, 6, (0, 0), ()), (4, (17, 96), 16, 7, (0, 0), (17, 96)),               # 0.75
    (4, (64,), 16, 11, (1, 1), ()), (4, (64,), 16, 12, (1, 1), (64,)),                      # the same, 66 elements apart
    (4, (31, 127), 14, 7, (0, 0), ()), (4, (31, 127), 14, 8, (0, 0), (127,)),               # the piece of 127 channels alone
    (4, (57, 24), 8, 97, (0, 3), ()), (4, (57, 24), 8, 98, (0, 3), (24,)),                  # less than that, but 2 of dst in all
    (2, (64, 97), 16, 12, (0, 0), ()), (2, (64, 97), 16, 13, (0, 0), (64, 97)),             # 1
    (2, (192,), 16, 10, (1, 1), ()), (2, (192,), 16, 11, (1, 1), (192,)),
    (2, (31, 129), 16, 15, (0, 0), ()), (2, (31, 129), 16, 16, (0, 0), (129,)),
    (2, (8, 9), 56, 64, (0, 0), ()), (2, (12, 13), 56, 128, (0, 0), ()),                    # few columns to a block, however large
    (2, (14, 15), 56, 46, (0, 0), ()), (2, (14, 15), 56, 47, (0, 0), (14, 15)),             # 8
    (2, (16, 17), 56, 14, (0, 0), ()), (2, (16, 17), 56, 16, (0, 0), (16, 17)),             # 3.1 and 3 for 16 and 17 columns
    (2, (24, 25), 56, 6, (0, 0), ()), (2, (24, 25), 56, 7, (0, 0), (24, 25)),               # 2.1 and 2 for 24 and 25
    (2, (32, 33), 10, 150, (0, 0), ()), (2, (32, 33), 10, 170, (0, 0), (32, 33)),           # as 25 and 26: blocks of 100 rows and 28 empty ones
    (2, (8, 255), 28, 4, (0, 0), (255,)),
])
def test_small_calls_keep_their_forms(es, channels, size, batch, pad, blocked, monkeypatch, capfd):
    monkeypatch.setenv("AMAP_PLAN_TRACE", "1")
    capfd.readouterr()
    m = B.amap_compose([(batch, c, size, size) for c in channels], es,
                       [("concat", 1), ("transpose", (0, 2, 3, 1)), ("pad", (0, 0, 0, pad[0]), (0, 0, 0, pad[1]), 0)])
    lines = [line.split() for line in capfd.readouterr().err.split("plan: begin")[-1].splitlines()[1:]]
    got = sorted(int(line[-1].split("=")[1]) // (batch * size * size) for line in lines if line[2] == "flat-blocked-dst")
    assert got == sorted(blocked)
    assert batch > 20 or B.amap_plan_selfcheck(m) == 0


def test_fewer_rows_than_a_block_keep_their_forms(monkeypatch, capfd):
    monkeypatch.setenv("AMAP_PLAN_TRACE", "1")
    capfd.readouterr()
    B.amap_compose([(3, 64, 7, 9)], 2, [("transpose", (0, 2, 3, 1)), ("pad", (0, 0, 0, 0), (0, 0, 0, 1), 0)])
    assert "flat" not in capfd.readouterr().err.split("begin (2")[-1]


@pytest.mark.gpu
@pytest.mark.parametrize("es", [2, 4])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_against_the_oracle(case, es, monkeypatch, capfd):
    import torch
    from paper_2002_12798_amd import device
    device.require_gpu()
    shapes, ops, m, _ = _planned(case, es, monkeypatch, capfd)
    rng = np.random.default_rng(40 + case)
    srcs = [rng.integers(0, 1 << (8 * es), s, dtype=np.uint64).astype({2: np.uint16, 4: np.uint32}[es]) for s in shapes]
    print(f"[gpu] pitched {shapes} {ops} es={es}", flush=True)
    dst = device.empty_dst(m, fill=0x5A5A)
    device.execute(m, [device.to_device(s) for s in srcs], dst)
    torch.cuda.synchronize()
    assert np.array_equal(device.to_host(dst), oracle.run_chain(srcs, ops))
