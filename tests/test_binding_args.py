"""Device addresses and streams are integers (or None): anything ctypes would turn into the address of host memory is refused
by the binding before the library, let alone the GPU, sees it."""
import ctypes as C

import pytest

from paper_2002_12798_amd import binding as B

BAD = [b"bytes", "text", (C.c_char * 16)(), C.c_void_p(16), 1.5]


@pytest.mark.parametrize("bad", BAD, ids=lambda v: type(v).__name__)
def test_only_integers_are_addresses(bad):
    m = B.amap_compose([(64, 64)], 2, [])
    x, w, out = 1 << 20, 2 << 20, 3 << 20   # never reached: every call below has one bad argument
    calls = [
        lambda: B.amap_execute([x], bad, m), lambda: B.amap_execute([x], out, m, bad), lambda: B.amap_execute([x], bad, m, 0, 1),
        lambda: B.amap_execute_kernel([x], out, m, bad, 1), lambda: B.amap_execute_multi([x], [out], [m], bad),
        lambda: B.amap_gemm_fused(bad, m, w, 64, out), lambda: B.amap_gemm_fused(x, m, bad, 64, out),
        lambda: B.amap_gemm_fused(x, m, w, 64, bad), lambda: B.amap_gemm_fused(x, m, w, 64, out, bad),
        lambda: B.amap_gemm_fused_store(x, m, w, 64, m, bad), lambda: B.amap_gemm_fused_store(bad, m, w, 64, m, out),
        lambda: B.amap_gemm_mapped(x, m, bad, m, None, out), lambda: B.amap_gemm_mapped(x, m, w, m, m, bad),
        lambda: B.amap_gemm_gather([x], m, bad, None, 64, None, out), lambda: B.amap_gemm_gather([x], m, w, None, 64, None, out, bad),
    ]
    for k, call in enumerate(calls):
        with pytest.raises(TypeError):
            call()
            pytest.fail(f"call {k} took {bad!r}")
