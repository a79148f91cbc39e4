"""The GEMM kernel on smaller tiles (amap_gemm_ring.hip).  On the CPU: the host replay of every form it takes (runs of A
along k or m, whole or shorter than a k-step, gathered sources, both weight forms, a mapped store) walks every load, every
LDS read and every store with the kernel's own address functions.  On the GPU: bit for bit against the general kernel,
which adds the same products in the same order, and against the oracle."""
import ctypes as C

import numpy as np
import pytest

from oracle import oracle
from paper_2002_12798_amd import binding as B
from paper_2002_12798_amd import synth


def _replay(a, n, w=None, out_map=None):
    f = B.raw.amap_gemm_ring_selfcheck
    f.argtypes = [C.c_void_p, C.c_void_p, C.c_int64, C.c_void_p, C.POINTER(C.c_int64)]
    errors = C.c_int64(-1)
    st = f(a.handle, w.handle if w else None, n, out_map.handle if out_map else None, C.byref(errors))
    return st, errors.value


def merge(b, h, s, d):
    """The heads of [b,h,s,d] as the matrix of their rows."""
    return [(b, h, s, d)], [("transpose", (0, 2, 1, 3)), ("reshape", (b * s, h * d))]


def conv(b, channels, size):
    """[b,c,size,size] branches as the [b*size*size, sum c] matrix of a pointwise convolution."""
    join = [("concat", 1)] if len(channels) > 1 else []
    return ([(b, c, size, size) for c in channels],
            join + [("transpose", (0, 2, 3, 1)), ("reshape", (b * size * size, sum(channels)))])


FORMS = [
    # (source shapes, chain -> [M,K]), N: every kernel shape, tile edges, remainders, one k-step, many k-steps
    (merge(1, 7, 64, 64), 64),                                       # 64 x 64 tiles, exactly one
    (merge(1, 16, 70, 64), 120),                                     # partial tiles in M and N
    (merge(3, 8, 33, 80), 136),                                      # runs of 80 (k decoded per lane), blocks of 33 rows
    (merge(2, 8, 50, 32), 72),                                       # runs of 32
    (([(1, 64)], []), 8),                                            # one row, one k-step, one vector of n
    (([(133, 640)], [("slice", 0, 5, 133, 1), ("slice", 1, 64, 640, 1)]), 200),   # base offset, rows longer than K
    (([(700, 448)], [("slice", 0, 699, -1, -1)]), 264),              # rows walked backwards
    (([(64, 448)], [("repeat", 0, 4)]), 64),                         # a source row read by four rows
    (([(1800, 448)], []), 1160),                                     # 128 x 128 tiles of 8 wavefronts
    (merge(81, 8, 37, 64), 3080),                                    # of 4 wavefronts
    (conv(2, [64], 8), 64),                                          # runs along m
    (conv(3, [32, 96, 40 + 24], 12), 264),                           # gathered, partial tiles
    (conv(1, [32], 4), 8),                                           # smaller than a tile each way, one k-step
    (([(256, 64), (256, 128), (256, 64)], [("concat", 1)]), 136),    # gathered along k
    (([(200, 64)] * 8, [("concat", 1)]), 72),                        # eight sources
    (([(512, 128)], []), 256),                                       # two k-steps in a ring of three stages
    (([(200, 192)], []), 136),                                       # as many as stages
    (merge(2, 4, 256, 64), 512),                                     # four
    (merge(9, 8, 200, 80), 1160),                                    # runs of 80 on 128 x 128 tiles of four stages
    (merge(16, 8, 200, 80), 3080),                                   # and of 4 wavefronts
    (conv(3, [64, 128, 64], 12), 264),                               # gathered along m, ranges for either weight
]


def _stays_general(case, w_along_k):
    """With the weight along k a step is 64 long: K and the ranges of the gathered sources must be whole numbers of it."""
    shapes, ops = FORMS[case][0]
    ranges = [s[1] for s in shapes] if len(shapes) > 1 else [B.dst_shape(B.amap_compose(shapes, 2, ops))[1]]
    return w_along_k and any(r % 64 for r in ranges)


def _maps(case):
    (shapes, ops), n = FORMS[case]
    a = B.amap_compose(shapes, 2, ops)
    m, k = B.dst_shape(a)
    wt = B.amap_compose([(n, k)], 2, [("transpose", (1, 0))])
    wn = B.amap_compose([(k, n + 8)], 2, [("slice", 1, 8, n + 8, 1)])    # row-major behind an offset, rows longer than N
    store = B.amap_compose([(m, n)], 2, [("reshape", (m, n // 8, 8)), ("transpose", (1, 0, 2))])
    return shapes, ops, a, m, k, n, wt, wn, store


@pytest.mark.parametrize("case", range(len(FORMS)))
def test_replay(case):
    _, _, a, _, k, n, wt, wn, store = _maps(case)
    for w, out_map in ((None, None), (wt, None), (wn, store)):
        st, errors = _replay(a, n, w, out_map)
        if _stays_general(case, w is wt):
            assert st == B.AMAP_E_UNSUPPORTED
            continue
        assert (st, errors) == (B.AMAP_OK, 0), (w is wt, out_map is not None)


def test_forms_reach_every_kernel_shape(monkeypatch, capfd):
    """Tile, wavefronts and stages, A along m or k, gathered, in short runs, W along n or k (every instance there is: test_gemm_ring_shapes.py)."""
    monkeypatch.setenv("AMAP_PLAN_TRACE", "1")
    capfd.readouterr()
    for case in range(len(FORMS)):
        _, _, a, _, _, n, wt, wn, _ = _maps(case)
        for w in (wt, wn):
            _replay(a, n, w)
    lines = [line.split(", ") for line in capfd.readouterr().err.splitlines() if line.startswith("amap gemm: ring")]
    seen = {", ".join(line[1:4] + line[6:]) for line in lines}
    small, wide8, wide4 = ("64 x 64 per workgroup of 4 wavefronts", "128 x 128 per workgroup of 8 wavefronts", "128 x 128 per workgroup of 4 wavefronts")
    want = {f"{t}, A along k{runs}, W along {w}" for t in (small, wide4) for runs in ("", " in runs shorter than a step") for w in "nk"}
    want |= {f"{wide8}, A along k, W along {w}" for w in "nk"} | {f"{wide8}, A along k in runs shorter than a step, W along {w}, four stages" for w in "nk"}
    want |= {f"{wide4}, A along {a}, W along {w}" for a in ("m", "m gathered", "k gathered") for w in "nk"}
    assert seen == want


def test_replay_of_random_forms():
    rng = np.random.default_rng(29)
    taken = 0
    for _ in range(60):
        b, h, s = int(rng.integers(1, 4)), int(rng.integers(1, 9)), int(rng.integers(1, 90))
        d = int(rng.choice([16, 24, 32, 64, 80, 128]))
        n = 8 * int(rng.integers(1, 40))
        along_m = rng.random() >= 0.5
        if along_m:
            shapes, ops = conv(b, [32 * int(rng.integers(1, 5)) for _ in range(h % 4 + 1)], 4 * int(rng.integers(1, 6)))
        else:
            shapes, ops = merge(b, 4 * h, s, d)
        a = B.amap_compose(shapes, 2, ops)
        m, k = B.dst_shape(a)
        out_map = B.amap_compose([(m, n)], 2, [("slice", 0, m - 1, -1, -1)]) if rng.random() < 0.5 else None
        w = B.amap_compose([(n, k)], 2, [("transpose", (1, 0))]) if rng.random() < 0.5 else None
        step = 32 if along_m and w is None else 64
        whole = all(r % step == 0 for r in ([shape[1] for shape in shapes] if along_m else [k]))
        st, errors = _replay(a, n, w, out_map)
        assert st == (B.AMAP_OK if whole else B.AMAP_E_UNSUPPORTED), (shapes, ops, n)
        assert st != B.AMAP_OK or errors == 0, (shapes, ops, n, errors)
        taken += whole
    assert taken >= 40


def test_products_of_the_other_kernels_have_no_ring_replay(monkeypatch):
    for shapes, ops, n in [([(200, 72)], [], 128),                       # K is no multiple of 64
                           ([(256, 136)], [("pad", (0, 0), (0, 56), 0)], 256),
                           ([(8192, 1024)], [], 4096)]:                  # fills the chip with 256 x 256 tiles
        assert _replay(B.amap_compose(shapes, 2, ops), n)[0] == B.AMAP_E_UNSUPPORTED
    monkeypatch.setenv("AMAP_GEMM_TILE256", "1")
    assert _replay(B.amap_compose([(512, 128)], 2, []), 256)[0] == B.AMAP_E_UNSUPPORTED   # 256 x 256 when asked for


@pytest.mark.parametrize("m, k, n", [(512, 128, 256), (8, 128, 8), (33, 256, 512), (1000, 384, 1000), (1024, 384, 1024), (512, 448, 1024)])
def test_few_tiles_of_few_k_steps_run_on_small_tiles(m, k, n):
    """Up to 16 tiles of 256 x 256 leave almost the whole chip idle, however short their walk along k."""
    a, wt = B.amap_compose([(m, k)], 2, []), B.amap_compose([(n, k)], 2, [("transpose", (1, 0))])
    assert _replay(a, n) == (B.AMAP_OK, 0) and _replay(a, n, wt) == (B.AMAP_OK, 0)


def test_the_switch_for_256_x_256_tiles(monkeypatch):
    """AMAP_GEMM_TILE256=1 gives the 256 x 256 kernel every product it takes, and no other."""
    few_tiles = B.amap_compose([(1800, 448)], 2, [])
    shapes, ops = conv(2, [64], 8)
    along_m = B.amap_compose(shapes, 2, ops)
    assert _replay(few_tiles, 1160) == (B.AMAP_OK, 0) and _replay(along_m, 64) == (B.AMAP_OK, 0)
    monkeypatch.setenv("AMAP_GEMM_TILE256", "1")
    assert _replay(few_tiles, 1160)[0] == B.AMAP_E_UNSUPPORTED
    assert _replay(along_m, 64) == (B.AMAP_OK, 0)


def test_one_store_map_used_by_several_threads():
    """The reverse of a store map is made at its first use and kept with it: the first uses race here."""
    import threading
    a = B.amap_compose([(300, 448)], 2, [])
    for _ in range(20):
        store = B.amap_compose([(300, 136)], 2, [("reshape", (300, 17, 8)), ("transpose", (1, 0, 2))])
        got = []
        threads = [threading.Thread(target=lambda: got.append(_replay(a, 136, None, store))) for _ in range(4)]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        assert got == [(B.AMAP_OK, 0)] * 4


@pytest.fixture(scope="module")
def dev():
    from paper_2002_12798_amd import device
    device.require_gpu()
    return device


@pytest.mark.gpu
@pytest.mark.parametrize("case", range(len(FORMS)))
def test_against_the_general_kernel_and_the_oracle(dev, case, monkeypatch, capfd):
    import torch
    shapes, ops, a, m, k, n, wt, wn, store = _maps(case)
    rng = np.random.default_rng(5100 + case)
    srcs = [synth.f32_to_bf16_bits(rng.standard_normal(s).astype(np.float32)) for s in shapes]
    w = synth.f32_to_bf16_bits((rng.standard_normal((k, n)) * 0.05).astype(np.float32))
    d_srcs = [dev.to_device(s) for s in srcs]
    d_w = [dev.to_device(w), dev.to_device(np.ascontiguousarray(w.T)), dev.to_device(np.concatenate([w[:, :8], w], axis=1))]
    rows = np.arange(m) if 2 * m * k * n < 1e9 else np.unique(np.concatenate([np.arange(0, m, 61), np.arange(m - 9, m)]))
    a_bits = np.ascontiguousarray((oracle.run_chain(srcs, ops) if ops else srcs[0])[rows])
    want = synth.bf16_bits_to_f32(oracle.gemm_bf16(a_bits, w)).astype(np.float64)
    # per element: K additions in fp32, each to one unit in the last place, 2^-23 sum |a w|, against the oracle's sums in 64 bits;
    # then one rounding to bf16 on either side, 2^-8 of the value
    sums = np.abs(synth.bf16_bits_to_f32(a_bits)).astype(np.float64) @ np.abs(synth.bf16_bits_to_f32(w)).astype(np.float64)
    bound = k * 2.0 ** -23 * sums + 2.0 ** -8 * np.abs(want)
    for w_map, d, out_map in ((None, d_w[0], None), (wt, d_w[1], None), (wn, d_w[2], store)):
        if _stays_general(case, w_map is wt):
            continue
        assert _replay(a, n, w_map, out_map) == (B.AMAP_OK, 0)

        def run():
            out = torch.full(B.dst_shape(out_map) if out_map else (m, n), 0x5A5A, dtype=torch.int16, device="cuda")
            B.amap_gemm_gather([t.data_ptr() for t in d_srcs], a, d.data_ptr(), w_map, n, out_map, out.data_ptr(), 0)
            torch.cuda.synchronize()
            return dev.to_host(out)

        print(f"[gpu] ring gemm case {case}: {shapes} {ops} N={n} w={'nk' if w_map is wt else 'kn'} store={out_map is not None}", flush=True)
        monkeypatch.setenv("AMAP_PLAN_TRACE", "1")
        capfd.readouterr()
        got = run()
        assert "amap gemm: ring" in capfd.readouterr().err           # the kernel under test is the one that ran
        monkeypatch.setenv("AMAP_GEMM_TILE256", "0")
        general = run()
        assert "256 x 128 tiles" in capfd.readouterr().err
        monkeypatch.delenv("AMAP_GEMM_TILE256")
        monkeypatch.delenv("AMAP_PLAN_TRACE")
        assert np.array_equal(got, general)                          # the same products in the same order
        g = synth.bf16_bits_to_f32(got).astype(np.float64)
        if out_map:
            g = g.transpose(1, 0, 2).reshape(m, n)
        assert (np.abs(g[rows] - want) <= bound + 2.0 ** -8 * np.abs(g[rows])).all()
