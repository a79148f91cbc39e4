"""Products with at most one tile to a compute unit: wavefronts that only load (32 x 64 and 64 x 64 tiles), four stages of 128 x 128, tiles of
192 x 128, and stores through the caches where rows or runs are no whole 64-byte pieces.  On the CPU the host replay, on the GPU bit for bit against the
general kernel, which adds the same products in the same order."""
import pytest

from paper_2002_12798_amd import binding as B
from tests.test_gemm_ring import _replay, conv, dev, merge  # noqa: F401  (dev: fixture)
from tests.test_gemm_ring_shapes import _against_general

CASES = [
    # chain -> [M,K], N, what the plan says of tile and wavefronts; partial tiles, whole runs of A and runs shorter than a step
    (merge(1, 8, 250, 32), 264, "32 x 64", "2 more load"),          # the fewest steps: four, all issued before the first is awaited
    (merge(1, 10, 250, 32), 264, "32 x 64", "2 more load"),         # five, in a ring of five stages: one issued behind a barrier
    (merge(1, 8, 250, 64), 264, "32 x 64", "2 more load"),          # eight, the fewest in whole runs
    (merge(1, 14, 64, 64), 520, "32 x 64", "2 more load"),          # eight tiles of 64 x 64, the fewest with K from 896 on
    (merge(2, 12, 63, 80), 1000, "32 x 64", "2 more load"),         # rows of 2000 bytes
    (merge(2, 20, 500, 64), 1000, "64 x 64", "4 more load"),        # 256 tiles, one to each unit
    (merge(2, 16, 500, 80), 1000, "64 x 64", "4 more load"),
    (merge(4, 8, 275, 64), 1928, "128 x 128", "four stages"),       # 144 tiles, just over half the units
    (merge(4, 8, 275, 80), 1928, "128 x 128", "four stages"),
    (merge(8, 20, 512, 64), 1000, "128 x 128", "four stages"),      # 256 tiles
    (merge(5, 8, 300, 64), 3000, "192 x 128", ""),                  # eight steps in a ring of three stages, 192 tiles
    (merge(5, 8, 300, 80), 3000, "192 x 128", ""),
    (merge(2, 12, 1150, 64), 2304, "192 x 128", ""),                # 216 tiles
]


def _maps(case):
    (shapes, ops), n, tile, more = CASES[case]
    a = B.amap_compose(shapes, 2, ops)
    m, k = B.dst_shape(a)
    wt = B.amap_compose([(n, k)], 2, [("transpose", (1, 0))])
    store = B.amap_compose([(m, n)], 2, [("reshape", (m, n // 8, 8)), ("transpose", (1, 0, 2))])
    return shapes, a, n, wt, store, f"amap gemm: ring, {tile} per workgroup", f" {m} x {n} x {k}{', ' if more else ''}{more}"


def _is(err, tile, end):
    """Whether the one line of a product's plan says of the tile, and of the shape beyond it, what the case does."""
    line = [x for x in err.splitlines() if x.startswith("amap gemm: ")]
    return len(line) == 1 and line[0].startswith(tile) and line[0].endswith(end)


@pytest.mark.parametrize("case", range(len(CASES)))
def test_replay(case, monkeypatch, capfd):
    _, a, n, wt, store, tile, end = _maps(case)
    monkeypatch.setenv("AMAP_PLAN_TRACE", "1")
    for w, out_map in ((None, None), (wt, None), (wt, store)):
        capfd.readouterr()
        assert _replay(a, n, w, out_map) == (B.AMAP_OK, 0)
        assert _is(capfd.readouterr().err, tile, end)


@pytest.mark.gpu
@pytest.mark.parametrize("case", range(len(CASES)))
def test_against_the_general_kernel(dev, case, monkeypatch, capfd):  # noqa: F811
    shapes, a, n, wt, store, tile, end = _maps(case)
    for w, out_map in ((None, None), (wt, None), (None, store)):
        print(f"[gpu] few tiles {shapes} N={n} w={'nk' if w else 'kn'} store={out_map is not None}", flush=True)
        assert _replay(a, n, w, out_map) == (B.AMAP_OK, 0)
        assert _is(_against_general(dev, shapes, a, n, w, monkeypatch, capfd, 1300 + case, tile, out_map), tile, end)
        monkeypatch.undo()


THROUGH, PAST = ", C through the caches, ", ", C past the caches, "


@pytest.mark.parametrize("m, n, heads, kind", [(333, 1000, None, THROUGH), (333, 1024, None, PAST), (333, 992, None, PAST), (333, 1008, None, THROUGH),
                                               (16384, 1000, None, THROUGH), (16784, 1000, None, PAST),   # 33.5 MB: just over 32 MB
                                               # a mapped store: the length of its runs, whatever N is
                                               (330, 1024, 8, THROUGH), (330, 1024, 80, THROUGH), (330, 1024, 32, PAST), (16896, 1024, 16, PAST)])
def test_the_kind_of_store(m, n, heads, kind, monkeypatch, capfd):
    """Rows or runs of no whole 64-byte pieces go through the caches while the product fits them."""
    n -= n % (heads or 1)
    a = B.amap_compose([(m, 64)], 2, [])
    out_map = B.amap_compose([(m, n)], 2, [("reshape", (m, n // heads, heads)), ("transpose", (1, 0, 2))]) if heads else None
    monkeypatch.setenv("AMAP_PLAN_TRACE", "1")
    capfd.readouterr()
    assert _replay(a, n, None, out_map) == (B.AMAP_OK, 0)
    assert kind in capfd.readouterr().err


@pytest.mark.parametrize("n", [120, 128])
def test_the_kind_of_store_along_m(n, monkeypatch, capfd):
    """A product whose A runs along m is stored past the caches, whatever its rows."""
    shapes, ops = conv(9, [64], 8)
    monkeypatch.setenv("AMAP_PLAN_TRACE", "1")
    capfd.readouterr()
    assert _replay(B.amap_compose(shapes, 2, ops), n) == (B.AMAP_OK, 0)
    err = capfd.readouterr().err
    assert "A along m" in err and PAST in err


@pytest.mark.gpu
@pytest.mark.parametrize("m, k, n, tile256, kind", [(333, 64, 1000, "", THROUGH), (16800, 64, 1000, "", PAST),   # more than 32 MB
                                                    # partial 256 x 256 tiles, at any size; whole ones have one kind
                                                    (300, 128, 1000, "1", THROUGH), (300, 128, 1024, "1", PAST), (512, 128, 512, "1", PAST)])
def test_rows_of_no_whole_pieces(dev, m, k, n, tile256, kind, monkeypatch, capfd):  # noqa: F811
    a = B.amap_compose([(m, k)], 2, [])
    monkeypatch.setenv("AMAP_GEMM_TILE256", tile256)
    print(f"[gpu] rows of no whole pieces {m} x {k} x {n}", flush=True)
    said = _against_general(dev, [(m, k)], a, n, None, monkeypatch, capfd, 1400, "256 x 256 tiles" if tile256 else "amap gemm: ring")
    assert kind in said


# A along m: few tiles of a short walk, on either side of 512 rows
CONV = [(conv(8, [64], 8), 120, "128 x 128"), (conv(9, [64], 8), 160, "64 x 64"), (conv(17, [96, 32], 8), 64, "64 x 64"), (conv(50, [64], 12), 120, "64 x 128"),
        # rows of no whole 64-byte pieces: narrower tiles only where two tiles of 64 would share what one of 128 holds
        (conv(245, [32], 4), 200, "64 x 64"), (conv(2, [128], 28), 360, "64 x 64"), (conv(10, [128], 12), 136, "64 x 64"), (conv(49, [64], 4), 120, "64 x 128")]


@pytest.mark.parametrize("case", range(len(CONV)))
def test_replay_along_m(case, monkeypatch, capfd):
    (shapes, ops), n, tile = CONV[case]
    a = B.amap_compose(shapes, 2, ops)
    m = B.dst_shape(a)[0]
    store = B.amap_compose([(m, n)], 2, [("reshape", (m, n // 8, 8)), ("transpose", (1, 0, 2))])
    monkeypatch.setenv("AMAP_PLAN_TRACE", "1")
    for out_map in (None, store):
        capfd.readouterr()
        assert _replay(a, n, None, out_map) == (B.AMAP_OK, 0)
        assert f"ring, {tile} per workgroup of 4 wavefronts, A along m" in capfd.readouterr().err


@pytest.mark.gpu
@pytest.mark.parametrize("case", range(len(CONV)))
def test_along_m_against_the_general_kernel(dev, case, monkeypatch, capfd):  # noqa: F811
    (shapes, ops), n, tile = CONV[case]
    a = B.amap_compose(shapes, 2, ops)
    print(f"[gpu] few tiles along m {shapes} N={n}", flush=True)
    _against_general(dev, shapes, a, n, None, monkeypatch, capfd, 1500 + case, f"ring, {tile} per workgroup")
