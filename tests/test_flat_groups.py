"""Images joined along the channels and made channels-last whose tile would move 4-byte vectors (an odd number of positions, or of
pairs of 2-byte ones): one tile over all pieces, or a flat tile per piece where their workgroups keep the chip busy or are small.
On the CPU the planned form and its replay, on the GPU the result against the oracle, bit for bit."""
import numpy as np
import pytest

from oracle import oracle
from paper_2002_12798_amd import binding as B


def joined(b, channels, h, w):
    return [(b, c, h, w) for c in channels], [("concat", 1), ("transpose", (0, 2, 3, 1))]


CASES = [
    # chain, element size, flat pieces?
    (joined(1, (64, 64), 15, 15), 4, False),              # 2 workgroups of 57.6 KB
    (joined(23, (64, 64), 15, 15), 4, False),             # 46
    (joined(24, (64, 64), 15, 15), 4, True),              # 48
    (joined(4, (192, 64), 17, 17), 4, False),             # 32, 37 KB each
    (joined(6, (192, 64), 17, 17), 4, True),              # 48
    (joined(1, (24, 64), 7, 7), 4, True),                 # 12.5 KB: however few
    (joined(8, (24, 40), 7, 7), 4, False),                # 7.8 KB: a single wavefront each
    (joined(8, (64, 64), 15, 10), 2, False),              # 16 of 19 KB
    (joined(55, (64, 64), 14, 25), 2, False),             # 110
    (joined(56, (64, 64), 14, 25), 2, True),              # 112
    (joined(1, (64, 32), 7, 14), 2, True),                # 12.5 KB
]


def _forms(case, capfd, monkeypatch):
    (shapes, ops), es, _ = CASES[case]
    monkeypatch.setenv("AMAP_PLAN_TRACE", "1")
    capfd.readouterr()
    m = B.amap_compose(shapes, es, ops)
    err = capfd.readouterr().err
    monkeypatch.delenv("AMAP_PLAN_TRACE")
    return m, {line.split()[2] for line in err.split("plan: begin")[-1].splitlines()[1:]}


@pytest.mark.parametrize("case", range(len(CASES)))
def test_form_and_replay(case, capfd, monkeypatch):
    m, forms = _forms(case, capfd, monkeypatch)
    assert forms == ({"flat-src"} if CASES[case][2] else {"tile"})
    assert B.amap_plan_selfcheck(m) == 0 and B.amap_check_cover(m) == (0, 0)
    monkeypatch.setenv("AMAP_FLAT", "2")                  # wherever they apply
    m, forms = _forms(case, capfd, monkeypatch)
    assert forms == {"flat-src"} and B.amap_plan_selfcheck(m) == 0


@pytest.mark.gpu
@pytest.mark.parametrize("case", [1, 2, 5, 6, 7])
def test_against_the_oracle(case, capfd, monkeypatch):
    import torch
    from paper_2002_12798_amd import device
    device.require_gpu()
    (shapes, ops), es, _ = CASES[case]
    rng = np.random.default_rng(70 + case)
    srcs = [rng.integers(0, 1 << (8 * es), s, dtype=np.uint64).astype({2: np.uint16, 4: np.uint32}[es]) for s in shapes]
    want = oracle.run_chain(srcs, ops)
    for flat in ("1", "2"):
        monkeypatch.setenv("AMAP_FLAT", flat)
        m, forms = _forms(case, capfd, monkeypatch)
        print(f"[gpu] groups {shapes} es={es} {forms}", flush=True)
        dst = device.empty_dst(m, fill=0x5A5A)
        device.execute(m, [device.to_device(s) for s in srcs], dst)
        torch.cuda.synchronize()
        assert np.array_equal(device.to_host(dst), want)
