"""Branches of the GEMM kernel on smaller tiles beyond the forms of test_gemm_ring.py: runs of A along k of every kind of
length, with two and with more digits of k; the tiles between 32 x 64 and 128 x 128.  On the CPU the host replay, on the GPU bit for bit against the general kernel,
which adds the same products in the same order."""
import numpy as np
import pytest

from paper_2002_12798_amd import binding as B
from paper_2002_12798_amd import synth
from tests.test_gemm_ring import FORMS, _replay, conv, dev, merge  # noqa: F401  (dev: fixture)


def three_digits(g, h, s, d):
    """[g,h,s,d] as [s, h * g * d]: k has three digits that no two of merge."""
    return [(g, h, s, d)], [("transpose", (2, 1, 0, 3)), ("reshape", (s, h * g * d))]


RUNS = [
    # whole runs only in a step (16, 32), a part of one left over (24, 40, 48), a run longer than a step (72, 80, 120)
    *[(merge(2, 64 // np.gcd(d, 64), 45, d), 136) for d in (16, 24, 32, 40, 48, 72, 80, 120)],
    (three_digits(5, 4, 70, 16), 72),
    (three_digits(2, 4, 133, 80), 264),
    (three_digits(3, 8, 50, 24), 64),
    (three_digits(2, 4, 1800, 80), 1160),   # 128 x 128 tiles of 8 wavefronts
    (three_digits(2, 4, 3200, 80), 3080),   # and of 4
]


@pytest.mark.parametrize("case", range(len(RUNS)))
def test_replay_of_short_runs(case, monkeypatch, capfd):
    (shapes, ops), n = RUNS[case]
    a = B.amap_compose(shapes, 2, ops)
    k = B.dst_shape(a)[1]
    wt = B.amap_compose([(n, k)], 2, [("transpose", (1, 0))])
    monkeypatch.setenv("AMAP_PLAN_TRACE", "1")
    for w in (None, wt):
        capfd.readouterr()
        assert _replay(a, n, w) == (B.AMAP_OK, 0)
        assert "runs shorter than a step" in capfd.readouterr().err


def _against_general(dev, shapes, a, n, w_map, monkeypatch, capfd, seed, expect, out_map=None):  # noqa: F811
    import torch
    m, k = B.dst_shape(a)
    rng = np.random.default_rng(seed)
    srcs = [dev.to_device(synth.f32_to_bf16_bits(rng.standard_normal(s).astype(np.float32))) for s in shapes]
    w = synth.f32_to_bf16_bits((rng.standard_normal((n, k) if w_map else (k, n)) * 0.05).astype(np.float32))
    w = dev.to_device(w)

    def run():
        out = torch.full(B.dst_shape(out_map) if out_map else (m, n), 0x5A5A, dtype=torch.int16, device="cuda")
        B.amap_gemm_gather([t.data_ptr() for t in srcs], a, w.data_ptr(), w_map, n, out_map, out.data_ptr(), 0)
        torch.cuda.synchronize()
        return dev.to_host(out)

    monkeypatch.setenv("AMAP_PLAN_TRACE", "1")
    capfd.readouterr()
    got = run()
    said = capfd.readouterr().err
    assert expect in said
    monkeypatch.setenv("AMAP_GEMM_TILE256", "0")
    general = run()
    assert "256 x 128 tiles" in capfd.readouterr().err
    assert np.array_equal(got, general)
    return said


@pytest.mark.gpu
@pytest.mark.parametrize("case", range(len(RUNS)))
def test_short_runs_against_the_general_kernel(dev, case, monkeypatch, capfd):  # noqa: F811
    (shapes, ops), n = RUNS[case]
    a = B.amap_compose(shapes, 2, ops)
    k = B.dst_shape(a)[1]
    for w in (None, B.amap_compose([(n, k)], 2, [("transpose", (1, 0))])):
        print(f"[gpu] short runs {shapes} N={n} w={'nk' if w else 'kn'}", flush=True)
        assert _replay(a, n, w) == (B.AMAP_OK, 0)
        _against_general(dev, shapes, a, n, w, monkeypatch, capfd, 900 + case, "runs shorter than a step")
        monkeypatch.undo()


TILES = [
    # chain -> [M,K], N, weight along k, what the plan says: every instance, partial tiles in M and N, few and many k-steps
    *[(merge(1, 16, 518, 128), 264, w, "32 x 64 per workgroup of 2") for w in (False, True)],
    *[(merge(3, 20, 111, 80), 264, w, "32 x 64 per workgroup of 2") for w in (False, True)],          # in short runs
    *[(merge(1, 20, 2341, 64), 760, w, "64 x 128 per workgroup of 4") for w in (False, True)],
    *[(merge(5, 20, 469, 80), 760, w, "64 x 128 per workgroup of 4") for w in (False, True)],
    (merge(3, 16, 1300, 64), 3336, False, "128 x 128 per workgroup of 8"),                            # more than three per unit
    *[(merge(3, 4, 1500, 80), 1160, w, "128 x 128 per workgroup of 8") for w in (False, True)],       # between one and two per unit, in short runs
    (conv(40, [320], 12), 72, False, "64 x 64 per workgroup of 4"),                                   # A along m
    (conv(7, [96, 128, 256, 128], 12), 136, False, "64 x 64 per workgroup of 4"),                     # gathered
    (conv(16, [256], 28), 120, False, "64 x 128 per workgroup of 4"),
    (conv(11, [96, 32, 32, 96], 28), 264, False, "64 x 128 per workgroup of 4"),
    (conv(2, [288], 4), 8, False, "64 x 64 per workgroup of 4"),                                      # smaller than a tile
]


@pytest.mark.parametrize("case", range(len(TILES)))
def test_replay_of_tiles(case, monkeypatch, capfd):
    (shapes, ops), n, along_k, expect = TILES[case]
    a = B.amap_compose(shapes, 2, ops)
    m, k = B.dst_shape(a)
    w = B.amap_compose([(n, k)], 2, [("transpose", (1, 0))]) if along_k else None
    store = B.amap_compose([(m, n)], 2, [("reshape", (m, n // 8, 8)), ("transpose", (1, 0, 2))])
    monkeypatch.setenv("AMAP_PLAN_TRACE", "1")
    for out_map in (None, store):
        capfd.readouterr()
        assert _replay(a, n, w, out_map) == (B.AMAP_OK, 0)
        assert expect in capfd.readouterr().err


def _routes(cases, monkeypatch, capfd):
    """For each product, with the weight along n and along k: what its plan says of tile, A and W, and of the shape beyond its tile."""
    monkeypatch.setenv("AMAP_PLAN_TRACE", "1")
    for (shapes, ops), n, *_ in cases:
        a = B.amap_compose(shapes, 2, ops)
        k = B.dst_shape(a)[1]
        for w in (None, B.amap_compose([(n, k)], 2, [("transpose", (1, 0))])):
            capfd.readouterr()
            _replay(a, n, w)
            line = [x for x in capfd.readouterr().err.splitlines() if x.startswith("amap gemm: ring")]
            parts = line[0].split(", ") if line else []
            yield ", ".join(parts[1:4] + parts[6:]) if parts else None


def test_the_cases_reach_every_instance(monkeypatch, capfd):
    from tests.test_gemm_ring_few import CASES
    seen = set(_routes(FORMS + RUNS + TILES + CASES, monkeypatch, capfd)) - {None}
    tile = {t: f"{t} per workgroup of {w} wavefronts" for t, w in (("32 x 64", 2), ("64 x 64", 4), ("64 x 128", 4), ("128 x 128", 4))}
    wide8, short, decoded = "128 x 128 per workgroup of 8 wavefronts", " in runs shorter than a step", " in runs shorter than a step (k decoded)"
    few = [(tile["32 x 64"], ", 2 more load"), (tile["64 x 64"], ", 4 more load"), (wide8, ", four stages"),
           ("192 x 128 per workgroup of 8 wavefronts", "")]
    alone = [(t, "") for t in (tile["64 x 64"], tile["64 x 128"], tile["128 x 128"], wide8)]
    want = {f"{t}, A along k{runs}, W along {w}{more}" for t, more in few + alone for runs in ("", short) for w in "nk"}
    want |= {f"{t}, A along k{decoded}, W along {w}" for t in (tile["64 x 64"], tile["128 x 128"], wide8) for w in "nk"}
    want |= {f"{tile[t]}, A along m{g}, W along n" for t in ("64 x 64", "64 x 128", "128 x 128") for g in ("", " gathered")}
    want |= {f"{tile['128 x 128']}, A along m{g}, W along k" for g in ("", " gathered")}
    want |= {f"{tile['128 x 128']}, A along k gathered, W along {w}" for w in "nk"}
    assert seen == want


def test_runs_of_one_length_are_carried_and_others_decoded(monkeypatch, capfd):
    """The first eight cases of RUNS merge heads (k has two digits), the others have three."""
    for i, route in enumerate(_routes(RUNS, monkeypatch, capfd)):
        assert "in runs shorter than a step" in route and ("(k decoded)" in route) == (i // 2 >= 8)


@pytest.mark.parametrize("m, k, n, expect", [
    # 128 x 128 tiles of the busiest compute unit: 8 wavefronts for up to two, four and eight from K = 768 on, six from 960, more from 1024
    (2682, 1024, 3072, "128 x 128 per workgroup of 8"),     # 1.97
    (2778, 1024, 3072, "128 x 128 per workgroup of 4"),     # 2.06
    (4185, 768, 3072, "128 x 128 per workgroup of 8"),      # 3.09
    (4194, 512, 3072, "128 x 128 per workgroup of 4"),
    (5595, 1024, 3072, "128 x 128 per workgroup of 4"),     # 4.13
    (7164, 960, 3072, "128 x 128 per workgroup of 8"),      # 5.25
    (7164, 896, 3072, "128 x 128 per workgroup of 4"),
    (8442, 1024, 3072, "128 x 128 per workgroup of 4"),     # 6.19
    (10216, 768, 3072, "128 x 128 per workgroup of 8"),     # 7.5
    (11262, 960, 3072, "128 x 128 per workgroup of 4"),     # 8.25
    (11262, 1024, 3072, "128 x 128 per workgroup of 8"),
    # 64 x 128 tiles from K = 640 on, above one and a half per unit from K = 384 on
    (1305, 512, 3072, "64 x 128 per workgroup of 4"),       # 1.97
    (1305, 320, 3072, "64 x 64 per workgroup of 4"),
    (396, 512, 4096, "64 x 64 per workgroup of 4"),
    (396, 640, 4096, "64 x 128 per workgroup of 4"),
    # and below K = 1280 from two thirds of a tile per unit on
    (448, 704, 3072, "64 x 64 per workgroup of 4"),         # 0.66
    (450, 704, 3072, "64 x 128 per workgroup of 4"),        # 0.75
    (338, 1216, 3072, "64 x 64 per workgroup of 4"),        # 0.56
    (338, 1280, 3072, "64 x 128 per workgroup of 4"),
])
def test_the_rule_for_the_tile(m, k, n, expect, monkeypatch, capfd):
    """(blocks of rows that are no whole 256: not for the 256 x 256 tiles)"""
    b = 2 if m % 2 == 0 else 3
    shapes, ops = merge(b, k // 64, m // b, 64)
    a = B.amap_compose(shapes, 2, ops)
    monkeypatch.setenv("AMAP_PLAN_TRACE", "1")
    capfd.readouterr()
    assert _replay(a, n)[0] == B.AMAP_OK
    assert expect in capfd.readouterr().err


@pytest.mark.gpu
@pytest.mark.parametrize("case", range(len(TILES)))
def test_tiles_against_the_general_kernel(dev, case, monkeypatch, capfd):  # noqa: F811
    (shapes, ops), n, along_k, expect = TILES[case]
    a = B.amap_compose(shapes, 2, ops)
    m, k = B.dst_shape(a)
    w = B.amap_compose([(n, k)], 2, [("transpose", (1, 0))]) if along_k else None
    store = B.amap_compose([(m, n)], 2, [("reshape", (m, n // 8, 8)), ("transpose", (1, 0, 2))])
    for out_map in (None, store):
        print(f"[gpu] tiles {shapes} N={n} w={'nk' if along_k else 'kn'} store={out_map is not None}", flush=True)
        assert _replay(a, n, w, out_map) == (B.AMAP_OK, 0)
        _against_general(dev, shapes, a, n, w, monkeypatch, capfd, 700 + case, expect, out_map)
        monkeypatch.undo()
