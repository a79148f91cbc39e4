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


def _planned(shapes, es, ops, monkeypatch, capfd):
    """The map and the forms its copy pieces are planned in."""
    capfd.readouterr()
    monkeypatch.setenv("AMAP_PLAN_TRACE", "1")
    m = B.amap_compose(shapes, es, ops)
    monkeypatch.delenv("AMAP_PLAN_TRACE")
    lines = [line.split()[2] for line in capfd.readouterr().err.splitlines() if line.startswith("amap plan:")]
    last = max(i for i, form in enumerate(lines) if form == "begin")   # the plan of the whole chain
    return m, lines[last + 1:]


def _blocked(shape, es, ops, monkeypatch, capfd):
    m, forms = _planned([shape], es, ops, monkeypatch, capfd)
    return m, any(form.startswith("flat-blocked") for form in forms)


# Towards a contiguous dst, rows of which 16 fit LDS: 16 rows at a time where that gives every compute unit two workgroups and
# the whole call is resident at once, else blocked.  Both sides of both lines, with 4, 3 and 2 workgroups to a compute unit.
ROWS16 = [
    ((127, 35, 35, 64), 2, "flat-blocked-dst"), ((128, 35, 35, 64), 2, "flat-dst"),       # 508, 512 blocks
    ((256, 35, 35, 64), 2, "flat-dst"), ((257, 35, 35, 64), 2, "flat-blocked-dst"),       # 1024, 1028: four of 39200 bytes fit
    ((60, 35, 35, 264), 2, "flat-dst"), ((61, 35, 35, 264), 2, "flat-blocked-dst"),       # a half-empty block counts: 1020, 1037
    ((96, 39, 39, 128), 2, "flat-dst"), ((97, 39, 39, 128), 2, "flat-blocked-dst"),       # 768, 776: three
    ((64, 41, 41, 128), 2, "flat-dst"), ((65, 41, 41, 128), 2, "flat-blocked-dst"),       # 512, 520: three of 53792, but LDS goes in steps
    ((64, 27, 27, 192), 4, "flat-dst"), ((65, 27, 27, 192), 4, "flat-blocked-dst"), ((96, 29, 29, 96), 4, "flat-blocked-dst"),
]


@pytest.mark.parametrize("shape, es, form", ROWS16)
def test_rows_per_block_towards_a_contiguous_dst(shape, es, form, monkeypatch, capfd):
    assert _planned([shape], es, NCHW, monkeypatch, capfd)[1] == [form]


def test_rows_per_block_look_at_the_whole_call(monkeypatch, capfd):
    join = [("concat", 0)] + NCHW
    assert _planned([(64, 35, 35, 128)] * 2, 2, join, monkeypatch, capfd)[1] == ["flat-dst"] * 2                 # 512 blocks each
    assert _planned([(64, 35, 35, 128)] * 3, 2, join, monkeypatch, capfd)[1] == ["flat-blocked-dst"] * 3


@pytest.mark.parametrize("case", range(len(CASES)))
def test_replay(case, monkeypatch, capfd):
    m, blocked = _blocked(*CASES[case], monkeypatch, capfd)
    assert blocked                                # the form under test is the planned one
    assert B.amap_plan_selfcheck(m) == 0


@pytest.mark.gpu
@pytest.mark.parametrize("case", range(len(CASES) + 2))
def test_against_the_oracle(case, monkeypatch, capfd):
    import torch
    from paper_2002_12798_amd import device
    device.require_gpu()
    # the last two: 16 rows would fit LDS, blocked because not all blocks of 16 would be resident at once; 16 rows at a time
    shape, es, ops = (CASES + [((64, 35, 35, 288), 2, NCHW), ((64, 41, 41, 128), 2, NCHW)])[case]
    print(f"[gpu] blocked flat tiles {shape} {es} {ops}", flush=True)
    m, blocked = _blocked(shape, es, ops, monkeypatch, capfd)
    assert blocked == (case <= len(CASES))
    src = synth.random_bits(shape, es, 300 + case)
    dst = device.empty_dst(m, fill=-1)
    device.execute(m, [device.to_device(src)], dst)
    torch.cuda.synchronize()
    assert np.array_equal(device.to_host(dst), oracle.run_chain([src], ops))
