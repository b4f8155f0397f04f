"""Host side of the C ABI sources on the CPU: tests/host/*.cpp includes a
source of the library with its kernel launches replaced by recorders, so the
choice of kernels, their tiling and the host's own state can be checked
without a device."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    """program(name) compiles tests/host/<name>.cpp (host code only) once."""
    if shutil.which("hipcc") is None:
        pytest.skip("no hipcc")
    built, where = {}, tmp_path_factory.mktemp("host")

    def build(name):
        if name not in built:
            obj, exe = str(where / (name + ".o")), str(where / name)
            subprocess.run(["hipcc", "--offload-host-only", "--offload-arch=gfx950", "-x", "hip",
                            "-std=c++17", "-O1", "-w", "-I", os.path.join(ROOT, "include"), "-c",
                            os.path.join(HERE, "host", name + ".cpp"), "-o", obj], check=True)
            subprocess.run(["hipcc", obj, "-o", exe, "-lpthread"], check=True)
            built[name] = exe
        return built[name]

    def run(name, *args):
        r = subprocess.run([build(name), *map(str, args)], capture_output=True, text=True,
                           timeout=120)
        assert r.returncode == 0, (r.returncode, r.stderr)
        return [line.split() for line in r.stdout.splitlines()]
    return run


def test_refused_two_step_launch_falls_back_to_whole_single_steps(program):
    """200 x 100 nodes in single-step tiles of 64 x 4: 4 columns, 100 tiles."""
    assert program("lattice_steps", "refused") == [["1", "1", "4", "100", "1", "1"]]
