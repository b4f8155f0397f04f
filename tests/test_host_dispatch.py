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
            # (the device code that the object refers to is not there)
            subprocess.run(["hipcc", obj, "-o", exe, "-lpthread",
                            "-Wl,--unresolved-symbols=ignore-all"], check=True)
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


CAVITY, CHANNEL, MILL, DUCT, COUETTE = ((1, 1, 1, 2), (3, 4, 1, 1), (0, 0, 0, 0), (0, 0, 1, 1),
                                        (2, 1, 0, 0))
F64, F32, BF16, F16 = range(4)
ONE_BY_ONE = -1


@pytest.mark.parametrize("nx,ny,sides,storage,mask,shape,share", [
    # small: the lowest blocks that fit, whatever the mask
    (32, 32, CAVITY, F64, 0, 0, 1.0), (256, 256, CAVITY, F32, 1, 1, 1.0),
    (251, 251, MILL, F64, 0, 1, 1.0), (300, 300, CAVITY, F16, 1, 2, 1.0),
    (384, 384, CAVITY, F32, 0, 1, 1.0), (400, 400, CAVITY, F16, 1, 1, 1.0),
    # FP64 where two of the two-step tiles stand for one
    (128, 128, CAVITY, F64, 0, 0, 1.0), (64, 64, CAVITY, F64, 1, 0, 0.4),
    (64, 64, MILL, F64, 1, 0, 1.0), (64, 1000, CAVITY, F64, 0, ONE_BY_ONE, 0),
    (64, 1500, MILL, F64, 0, ONE_BY_ONE, 0), (64, 1500, CHANNEL, F64, 0, 1, 1.0),
    (64, 1000, CAVITY, F32, 0, 2, 1.0), (70, 1000, CAVITY, F64, 0, 2, 1.0),
    # larger: the ring's work
    (1024, 1024, CAVITY, F32, 0, 3, 1.0), (1024, 1024, CAVITY, F64, 1, 3, 0.5),
    (1024, 1024, MILL, F64, 1, 3, 0.15), (512, 512, CAVITY, F64, 1, 3, 0.15),
    (4096, 4096, CAVITY, F32, 0, 4, 1.0), (2048, 2048, CAVITY, F64, 0, 3, 0.5),
    (180, 2000, CAVITY, F32, 0, ONE_BY_ONE, 0), (190, 1500, CHANNEL, F16, 0, ONE_BY_ONE, 0),
    (180, 1000, MILL, F64, 0, ONE_BY_ONE, 0), (200, 2000, CAVITY, F64, 0, 3, 0.5),
    (250, 1025, CAVITY, F32, 0, 3, 1.0),
    # FP64 in partly empty tiles
    (129, 1025, MILL, F64, 0, ONE_BY_ONE, 0), (129, 1025, CHANNEL, F64, 1, 3, 1.0),
    (129, 2000, MILL, F64, 0, 3, 0.15), (16, 4000, COUETTE, F64, 0, ONE_BY_ONE, 0),
    (80, 4000, COUETTE, F64, 0, ONE_BY_ONE, 0), (116, 4000, COUETTE, F64, 0, 3, 0.15),
    (129, 1025, CAVITY, F32, 1, 3, 0.05), (16, 4000, CAVITY, F32, 1, 3, 0.05), (450, 450, CAVITY, F64, 0, 3, 0.15),
    # FP32 periodic in cache
    (1500, 1500, MILL, F32, 1, 3, 0.2), (1500, 1500, CAVITY, F32, 1, 3, 1.0),
    (2048, 2048, DUCT, F32, 1, 4, 1.0),
    # 16 bits
    (128, 128, MILL, F16, 0, ONE_BY_ONE, 0), (1024, 1024, CAVITY, BF16, 1, 3, 0.05),
    (1500, 1500, CAVITY, F16, 0, ONE_BY_ONE, 0), (1500, 1500, CAVITY, F16, 1, ONE_BY_ONE, 0),
    (4096, 4096, CAVITY, F16, 0, 4, 0.05), (1600, 750, CHANNEL, F16, 0, ONE_BY_ONE, 0),
    (1600, 750, CHANNEL, F16, 1, 4, 0.25), (400, 3000, CHANNEL, F16, 0, 4, 0.25),
    (300, 4000, CHANNEL, F16, 1, ONE_BY_ONE, 0), (2400, 1041, CHANNEL, F16, 0, 4, 0.25),
    (4096, 1024, CHANNEL, F16, 1, 4, 0.25),
    # never
    (15, 400, CAVITY, F32, 0, ONE_BY_ONE, 0), (4000, 15, CAVITY, F64, 0, ONE_BY_ONE, 0),
])
def test_two_step_shape(program, nx, ny, sides, storage, mask, shape, share):
    """Where two steps per launch were measured slower the lattice steps one by
    one; the share of rows near solid nodes up to which they pay."""
    (got,) = program("lattice_steps", "shape", nx, ny, *sides, storage, mask)
    assert (int(got[0]), float(got[1])) == (shape, share)


def test_fields_read_by_two_threads_have_staging_of_their_own(program):
    """Two threads inside lbm_batch_fields of one batch at the same time: two
    exports, to different memory, and no copy from memory given back."""
    assert program("batch_host", "fields") == [["2", "1", "0"]]


def test_two_step_items_are_built_for_runs_that_use_them(program):
    """Runs of one and two steps, and windows without two plain steps in a row,
    build no list; a list stays until the cases or the shape change."""
    got = [list(map(int, r)) for r in program("batch_host", "items", 100, 1, 2, 3, 100, 2, 50,
                                              -100, 1, 100)]
    runs, (every_item, out_of_order, even) = got[:-1], got[-1]
    shapes, uploads = [r[0] for r in runs], [r[2] for r in runs]
    s = shapes[2]
    assert s >= 0 and shapes == [-1, -1, s, s, -1, s, s, -1, s]
    assert uploads == [2, 2, 3, 2, 2, 2, 3, 2, 2]
    assert runs[3][1] == runs[5][1] > runs[6][1]
    assert (every_item, out_of_order, even) == (1, 0, 1)
    assert [int(r[0]) for r in program("batch_host", "items", 3, 3, 30)[:2]] == [-1, -1]
    assert [int(r[0]) for r in program("batch_host", "items", 4, 3)[:1]] == [s]


@pytest.mark.parametrize("nx,allocs,live", [(100, 3, 0), (200, 1, 1), (4000, 1, 1), (10000, 3, 0)])
def test_staging_is_kept_where_it_pays(program, nx, allocs, live):
    """Three reads of nx x 300 nodes: from 1 to 64 MB one allocation that stays."""
    assert program("batch_host", "staging", nx) == [[str(allocs), str(live)]]


@pytest.mark.parametrize("storage,cases,shape", [
    # one block per compute unit, two rounds of them
    (F64, [(4, 64, 64, CAVITY, 0)], 0), (F64, [(16, 64, 64, CAVITY, 0)], 2),
    (F64, [(20, 64, 64, CAVITY, 0)], 1), (F32, [(14, 100, 100, MILL, 3)], 1),
    # tiles away from the sides: none, a quarter, many
    (F64, [(200, 64, 64, CAVITY, 0)], ONE_BY_ONE), (F32, [(30, 116, 116, CAVITY, 0)], ONE_BY_ONE),
    (F64, [(20, 128, 128, CAVITY, 0)], 3), (F32, [(20, 512, 512, CAVITY, 0)], 4),
    (F64, [(20, 400, 100, CHANNEL, 0)], 3),
    # the ring's work beyond 2048 tiles
    (F64, [(30, 128, 128, CAVITY, 0)], 3), (F64, [(76, 128, 128, CAVITY, 0)], ONE_BY_ONE),
    (F32, [(76, 128, 128, MILL, 0)], ONE_BY_ONE), (F64, [(102, 128, 256, DUCT, 0)], ONE_BY_ONE),
    (F64, [(41, 180, 180, CAVITY, 0)], 3), (F32, [(102, 128, 256, DUCT, 0)], 4),
    (F64, [(85, 256, 64, CHANNEL, 0)], 3),
    # solids in every tile
    (F64, [(60, 400, 400, CAVITY, 41)], 3), (F32, [(20, 200, 200, CAVITY, 41)], 3),
    # a lattice narrower than 16 nodes
    (F32, [(4, 64, 64, CAVITY, 0), (1, 15, 64, CAVITY, 0)], ONE_BY_ONE),
])
def test_two_step_shape_of_batches(program, storage, cases, shape):
    args = [v for n, nx, ny, sides, every in cases for v in (n, nx, ny, *sides, every)]
    assert program("batch_host", "shape", storage, *args) == [[str(shape)]]


@pytest.mark.parametrize("n,h,w,cin,cout,kernel", [
    # LDS holds a tile of 32 columns, only one of 16, none
    (16, 64, 64, 352, 32, "tile"), (16, 64, 64, 384, 96, "tile"), (4, 9, 9, 416, 32, "tile"),
    (16, 64, 64, 640, 64, "tile"), (2, 64, 64, 576, 128, "tile"),
    (16, 64, 64, 704, 64, "conv_fwd32_kernel"), (1, 256, 256, 1024, 32, "conv_fwd_kernel"),
    (16, 64, 63, 704, 64, "conv_fwd_kernel"), (1, 3, 5, 1216, 64, "conv_fwd_kernel"),
])
def test_wide_convolutions(program, n, h, w, cin, cout, kernel):
    """Many input channels: a tile wherever one fits, else the 64-pixel wave
    tiles from 65536 pixels on (64 output channels)."""
    (launch,) = program("unet_launches", "fwd", n, h, w, cin, cout)
    assert launch[0] == kernel


@pytest.mark.parametrize("n,h,w,cin,cout,kernel", [
    # few blocks: tiles, however empty
    (500, 1, 1, 32, 32, "tile"), (125, 4, 4, 64, 64, "tile"), (300, 2, 3, 256, 64, "tile"),
    # many small images: without tiles, the large form from 65536 pixels on
    (2000, 1, 1, 32, 32, "conv_fwd_kernel"), (4096, 1, 1, 128, 128, "conv_fwd_kernel"),
    (4096, 2, 2, 256, 256, "conv_fwd_kernel"), (1333, 3, 3, 96, 32, "conv_fwd_kernel"),
    (4096, 4, 4, 64, 64, "conv_fwd32_kernel"), (5000, 4, 4, 96, 32, "conv_fwd32_kernel"),
    (16250, 1, 16, 128, 128, "conv_fwd32_kernel"), (937, 8, 8, 32, 128, "conv_fwd_kernel"),
    # a smaller tile
    (3209, 9, 9, 128, 128, "tile"), (1015, 16, 16, 64, 64, "tile"), (1024, 4, 4, 64, 64, "tile"),
    (4062, 8, 8, 64, 64, "tile"), (899, 17, 17, 64, 64, "tile"),
    # the sizes of the network
    (16, 128, 128, 32, 32, "tile"), (16, 16, 16, 256, 256, "tile"), (2048, 16, 16, 256, 256, "tile"),
])
def test_many_small_images(program, n, h, w, cin, cout, kernel):
    (launch,) = program("unet_launches", "fwd", n, h, w, cin, cout)
    assert launch[0] == kernel


@pytest.mark.parametrize("n,h,w,blocks", [
    (64, 1, 1, 1), (65, 1, 1, 2), (25, 2, 2, 1), (9, 4, 4, 1), (10, 4, 4, 2), (4, 7, 7, 1),
    (2, 8, 8, 2), (8, 1, 16, 1), (2, 7, 40, 2), (3, 40, 7, 4), (1, 16, 16, 1),
])
def test_small_images_share_the_tiles_of_a_weight_gradient(program, n, h, w, blocks):
    """Blocks for 32 x 32 channels: the power of two up to the pixel tiles."""
    tile, _ = program("unet_launches", "bwdw", n, h, w, 32, 32)
    assert tile[:3] == ["wgrad_tile_kernel", str(blocks), "1"]


@pytest.mark.parametrize("n,h,w,cin,cout,floats", [
    (1, 16, 16, 32, 32, 9 * 1024 + 32), (1, 16, 16, 16, 32, 0), (1, 16, 16, 32, 8, 0),
    (2, 3, 5, 0, 32, 0), (0, 16, 16, 32, 32, 0),
])
def test_scratch_of_a_weight_gradient(program, n, h, w, cin, cout, floats):
    """Channel counts that the gradient refuses need none (and end no process)."""
    assert program("unet_launches", "work", n, h, w, cin, cout) == [[str(floats)]]
