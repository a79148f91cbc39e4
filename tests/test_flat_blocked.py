"""Column-blocked flat tiles (rows too long for LDS, or towards a dst that offers no vectors): row counts from the smallest
to more than a block, columns around whole blocks and slots, both directions, both element sizes.  The plans are replayed
on the CPU lane by lane; on the GPU the result is the oracle's bit for bit."""
import numpy as np
import pytest

from oracle import oracle
from paper_2002_12798_amd import binding as B
from paper_2002_12798_amd import synth

T2 = [("transpose", (1, 0))]
NCHW, NHWC, PAD = [("transpose", (0, 3, 1, 2))], [("transpose", (0, 2, 3, 1))], [("pad", (0, 1, 1, 0), (0, 1, 1, 0), 7)]

CASES = [
    # source shape, element size, chain
    ((2, 47, 47, 24), 2, NCHW), ((2, 47, 47, 16), 2, NCHW), ((1, 55, 55, 48), 2, NCHW), ((1, 59, 59, 72), 2, NCHW),
    ((2, 33, 33, 48), 4, NCHW), ((1, 41, 41, 20), 4, NCHW), ((1, 33, 33, 68), 4, NCHW),
    ((1, 48, 47, 47), 2, NHWC + PAD), ((1, 72, 59, 59), 2, NHWC + PAD), ((1, 24, 33, 33), 4, NHWC + PAD),
    # dst without vectors: odd row and column counts around a block of 64 x 64 (4-byte: 64 x 32) and around slots of 8 (4)
    ((63, 16 + 1), 2, T2), ((64 + 1, 64 + 1), 2, T2), ((64 + 7, 127), 2, T2), ((128 + 9, 63), 2, T2), ((193, 2 * 64 + 3), 2, T2),
    ((33, 65), 4, T2), ((3 * 32 + 1, 67), 4, T2), ((31, 17), 4, T2),
    ((3, 7, 7, 64), 2, NCHW + [("pad", (0, 1, 0, 0), (0, 0, 0, 0), 0)]),
]


def _blocked(shape, es, ops, monkeypatch, capfd):
    capfd.readouterr()
    monkeypatch.setenv("AMAP_PLAN_TRACE", "1")
    m = B.amap_compose([shape], es, ops)
    monkeypatch.delenv("AMAP_PLAN_TRACE")
    return m, "flat-blocked" in capfd.readouterr().err


@pytest.mark.parametrize("case", range(len(CASES)))
def test_replay(case, monkeypatch, capfd):
    m, blocked = _blocked(*CASES[case], monkeypatch, capfd)
    assert blocked                                # the form under test is the planned one
    assert B.amap_plan_selfcheck(m) == 0


@pytest.mark.gpu
@pytest.mark.parametrize("case", range(len(CASES) + 1))
def test_against_the_oracle(case, monkeypatch, capfd):
    import torch
    from paper_2002_12798_amd import device
    device.require_gpu()
    # the last one: 16 rows would fit LDS, blocked because the piece is larger than a third of the last-level cache
    shape, es, ops = CASES[case] if case < len(CASES) else ((64, 35, 35, 288), 2, NCHW)
    print(f"[gpu] blocked flat tiles {shape} {es} {ops}", flush=True)
    m, blocked = _blocked(shape, es, ops, monkeypatch, capfd)
    assert blocked
    src = synth.random_bits(shape, es, 300 + case)
    dst = device.empty_dst(m, fill=-1)
    device.execute(m, [device.to_device(src)], dst)
    torch.cuda.synchronize()
    assert np.array_equal(device.to_host(dst), oracle.run_chain([src], ops))
