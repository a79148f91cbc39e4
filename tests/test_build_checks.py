"""The build refuses a library whose kernels lost registers to scratch, hold static LDS they do not know of, or keep fewer
wavefronts per SIMD than the map kernels need."""
import glob
import os
import subprocess
import sys
import sysconfig

import pytest

from paper_2002_12798_amd import binding, build

PIECES = "_ZN12_GLOBAL__N_118amap_pieces_kernelILi{}ELi2ELb0EEEvN8amap_dev10LaunchArgsEPc"
RING = "_ZN12_GLOBAL__N_121amap_gemm_ring_kernelINS_5ShapeILi64ELi64EEEEE"


def _remarks(name, vgprs, occupancy, scratch=0, lds=0):
    fields = [f"Function Name: {name}", f"    VGPRs: {vgprs}", f"    ScratchSize [bytes/lane]: {scratch}",
              f"    Occupancy [waves/SIMD]: {occupancy}", f"    LDS Size [bytes/block]: {lds}"]
    return "\n".join(f"k.hip:1:1: remark: {f} [-Rpass-analysis=kernel-resource-usage]" for f in fields)


@pytest.mark.parametrize("remarks, wrong", [
    (_remarks(PIECES.format(2), 66, 7), None),
    (_remarks(PIECES.format(2), 74, 6), "wavefronts"),
    (_remarks(PIECES.format(4), 78, 6), None),
    (_remarks(PIECES.format(2), 66, 7, scratch=16), "scratch"),
    (_remarks(PIECES.format(2), 66, 7, lds=512), None),
    (_remarks(RING, 118, 4), None),
    (_remarks(RING, 118, 4, lds=512), "static LDS"),
])
def test_check_usage(remarks, wrong):
    found = build.check_usage(build.kernel_usage(remarks))
    assert len(found) == (wrong is not None)
    assert wrong is None or wrong in found[0]


def test_the_extension_is_for_one_python():
    """Its name says for which: another one does not load what it would misread."""
    assert build.CALL.endswith(sysconfig.get_config_var("EXT_SUFFIX")) and len(sysconfig.get_config_var("EXT_SUFFIX")) > len(".so")
    assert os.path.realpath(binding._call.__file__) == os.path.realpath(build.CALL)
    assert glob.glob(os.path.join(os.path.dirname(build.CALL), "_amap_call.so")) == []


WITHOUT = """
import sys
sys.modules["paper_2002_12798_amd._amap_call"] = None
from paper_2002_12798_amd import binding as B, device

class Tensor:
    shape = (64, 24)
    def __init__(self, at): self.at = at
    def data_ptr(self): return self.at

seen = []
def recorder(name):
    def f(*args):
        seen.append((name, [x if x is None or type(x) is int else x.value if hasattr(x, "value") else list(x) for x in args]))
        return 0
    return f
B._execute = recorder("execute")
for name in ("amap_execute_multi", "amap_gemm_fused", "amap_gemm_gather"):
    setattr(B._L, name, recorder(name))
m, x, y = B.amap_compose([(8, 64)], 2, []), Tensor(64), Tensor(128)
assert device.execute(m, [x], y, stream=7) is y and device.execute_multi([m], [x], [y], stream=7) == [y]
assert device.gemm_fused(x, m, Tensor(96), out=y, stream=7) is y
B.amap_gemm_gather([64], m, 96, None, 24, None, 128, 7)
h = m.handle.value
assert seen == [("execute", [[64], 128, h, 7]), ("amap_execute_multi", [[64], [128], [h], 1, 7]), ("amap_gemm_fused", [64, h, 96, 24, 128, 7]),
                ("amap_gemm_gather", [[64], h, 96, None, 24, None, 128, 7])], seen
"""


def test_without_the_extension_calls_go_through_ctypes():
    """(The library is replaced by functions that write down what they were given.)"""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-W", "always", "-c", WITHOUT], cwd=root, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "through ctypes" in r.stderr, r.stderr


def test_a_build_without_python_s_headers(monkeypatch, tmp_path, capfd):
    """The library is what has to be built; an extension that cannot be is left out, an old one too."""
    monkeypatch.setattr(build, "CALL", str(tmp_path / "_amap_call.x.so"))
    (tmp_path / "_amap_call.x.so").write_bytes(b"old")
    monkeypatch.setattr(sysconfig, "get_path", lambda name: str(tmp_path))
    assert build.build_call() is None and not os.path.exists(build.CALL)
    assert "Python.h" in capfd.readouterr().err


@pytest.mark.parametrize("rows, columns, waves, compiles", [(64, 64, 8, True), (192, 128, 8, True), (64, 64, 6, False), (192, 128, 12, True), (128, 128, 6, False),
                                                            (64, 128, 32, False)])
def test_a_tile_that_its_wavefronts_cannot_store_does_not_compile(rows, columns, waves, compiles, tmp_path):
    """Whole passes over the tile's rows: others would leave the last ones unwritten, or store none."""
    unit = tmp_path / "store.hip"
    unit.write_text(f'#include "amap_gemm_ring.hpp"\ntemplate struct amap_gemm::RingStore<{rows}, {columns}, {waves}>;\n')
    r = subprocess.run(["hipcc", "-x", "hip", "--offload-host-only", "-std=c++17", "-fsyntax-only", "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC,
                        str(unit)], capture_output=True, text=True, timeout=300)
    assert (r.returncode == 0) == compiles, r.stderr
    assert compiles or "every row of the tile" in r.stderr
