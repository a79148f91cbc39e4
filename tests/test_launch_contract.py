"""What the library asks of the HIP runtime around a launch, from a C caller that stands in for the runtime (no GPU)."""
import os
import subprocess

import pytest

from paper_2002_12798_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def caller(tmp_path_factory):
    import torch
    exe = str(tmp_path_factory.mktemp("launch") / "launch_contract")
    rt_dirs = [os.path.join(os.path.dirname(torch.__file__), "lib"), "/opt/rocm/lib"]
    subprocess.run(["gcc", "-std=c99", "-Wall", "-Wextra", "-Werror", "-I", os.path.join(ROOT, "include"),
                    os.path.join(ROOT, "tests", "launch_contract.c"), "-o", exe, B.LIB_PATH, "-rdynamic", "-Wl,--allow-shlib-undefined"]
                   + [f"-Wl,-rpath,{d}" for d in [os.path.dirname(B.LIB_PATH)] + rt_dirs], check=True)
    env = dict(os.environ, AMAP_PLAN_TRACE="1", LD_LIBRARY_PATH=":".join(rt_dirs + [os.environ.get("LD_LIBRARY_PATH", "")]))

    def run(mode):
        r = subprocess.run([exe, mode], capture_output=True, text=True, env=env, timeout=120)
        assert (r.returncode, r.stdout.strip()) == (0, "OK"), (r.stdout, r.stderr)
        return r.stderr.splitlines()
    return run


def test_lds_is_reserved_on_every_device(caller):
    """A kernel's attribute belongs to the device that was current when it was set."""
    caller("devices")


def test_errors_of_other_calls_pass_through(caller):
    caller("errors")


def test_a_failed_look_up_leaves_no_error(caller):
    """The kernel's handle is a short cut: without it the launch goes by the kernel's address."""
    caller("lookup")


def test_a_stream_of_another_device(caller):
    """The stream says where a call runs, whichever device is current."""
    caller("streams")


def test_the_trace_names_the_kernel_that_runs(caller):
    lines, traced = [x for x in caller("names") if not x.startswith("amap plan")], []
    for said, ran in zip(lines[::2], lines[1::2]):
        assert said.startswith("amap launch: ") and ran.startswith("ran "), (said, ran)
        traced.append(said.removeprefix("amap launch: ").split(",")[0])
        assert traced[-1] in ran, (said, ran)
    rows, few, multi = "amap_rows_kernel", "amap_rows_few_kernel", "amap_rows_multi_kernel"
    assert len(lines) == 16 and traced[:5] == [few, rows, few, multi, multi] and len(set(traced)) >= 5, traced
