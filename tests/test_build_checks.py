"""The build refuses a library whose kernels lost registers to scratch, hold static LDS they do not know of, or keep fewer
wavefronts per SIMD than the map kernels need."""
import glob
import os
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
