"""Two plain steps in one launch against the same steps one by one: a call of
n steps pairs them, n calls of one step never do, and the states must be the
same bit for bit (same arithmetic and the same storage rounding between the
steps), for every side kind, storage and launch shape of the two-step kernel
(chosen by size)."""
import numpy as np
import pytest

from workloads import hartmann_force

pytestmark = pytest.mark.gpu

PERIODIC, WALL, LID, INLET, OUTLET = 0, 1, 2, 3, 4
CAVITY = (WALL, WALL, WALL, LID)
CHANNEL = (INLET, OUTLET, WALL, WALL)


@pytest.fixture(scope="module", autouse=True)
def lbm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1806_10251_amd import lbm as L
    L.load()
    return L


def pair(nx, ny, sides, storage, mask=None, force=None, **kw):
    from paper_1806_10251_amd import lbm
    p = dict(nu=0.03, gamma=0.6, u_lid=0.05, u_in_max=0.03, check_every=1000, storage=storage)
    p.update(kw)
    out = []
    rng = np.random.default_rng(5)
    y, x = np.mgrid[0:ny, 0:nx]
    start = (1 + 1e-3 * np.sin(0.3 * x + 0.1 * y), 0.01 * np.sin(0.2 * y), 0.01 * rng.random((ny, nx)))
    for _ in range(2):
        lat = lbm.Lattice(nx, ny, sides, solid=mask, **p)
        if force is not None:
            lat.set_force_field(*force)
        lat.init_fields(*start)
        out.append(lat)
    return out


def same_after(nx, ny, sides, storage, steps=7, **kw):
    print("[gpu-case] two-step", nx, ny, sides, storage, sorted(kw), flush=True)
    a, b = pair(nx, ny, sides, storage, **kw)
    a.step(steps)
    for _ in range(steps):
        b.step(1)
    assert a.steps == b.steps == steps
    mask = kw.get("mask")
    fluid = np.ones((ny, nx), bool) if mask is None else np.asarray(mask) == 0
    fa, fb = a.populations(), b.populations()
    assert np.isfinite(fa[:, fluid]).all()
    np.testing.assert_array_equal(fa[:, fluid], fb[:, fluid])
    # the other lattice holds the step before: the mean of the last two agrees
    a.average_last_two()
    b.average_last_two()
    np.testing.assert_array_equal(a.populations()[:, fluid], b.populations()[:, fluid])
    # and the next steps start from consistent boundary slots and history
    a.step(3)
    for _ in range(3):
        b.step(1)
    for p, q in zip(a.fields(), b.fields()):
        np.testing.assert_array_equal(p, q)


def obstacles(nx, ny):
    m = np.zeros((ny, nx), np.uint8)
    m[ny // 3:ny // 3 + max(3, ny // 6), nx // 4:nx // 4 + 5] = 1
    m[ny - 4:ny - 2, nx // 2:nx // 2 + 7] = 1
    m[0:2, nx // 3] = 1          # on the south side
    m[ny // 2, nx - 9] = 1       # a single node
    return m


@pytest.mark.parametrize("storage", ["f64", "f32", "bf16", "f16"])
@pytest.mark.parametrize("sides", [CAVITY, CHANNEL, (PERIODIC,) * 4, (PERIODIC, PERIODIC, WALL, LID),
                                   (LID, WALL, PERIODIC, PERIODIC),
                                   (INLET, OUTLET, PERIODIC, PERIODIC)])
@pytest.mark.parametrize("solid", [False, True])
def test_every_side_kind(sides, storage, solid):
    nx, ny = 123, 37
    same_after(nx, ny, sides, storage, mask=obstacles(nx, ny) if solid else None)


@pytest.mark.parametrize("nx,ny", [(16, 16), (58, 22), (59, 23), (61, 17), (116, 52), (1000, 16)])
@pytest.mark.parametrize("sides", [CAVITY, (PERIODIC,) * 4, CHANNEL])
def test_tile_edges(nx, ny, sides):
    same_after(nx, ny, sides, "f32")


@pytest.mark.parametrize("nx,ny,storage", [
    (230, 190, "f64"), (330, 310, "f64"), (401, 390, "f32"),   # 6- and 10-row tiles, two rounds
    (700, 333, "f64"), (650, 640, "f32"), (900, 700, "bf16"),  # two rows per wavefront
    (1930, 1901, "f32"), (4100, 1101, "f16"),                  # four, beyond the last-level cache
])
def test_launch_shapes(nx, ny, storage):
    same_after(nx, ny, CHANNEL, storage, steps=5, mask=obstacles(nx, ny))
    same_after(nx, ny, CAVITY, storage, steps=5)


@pytest.mark.parametrize("kw", [dict(gi_correct=0), dict(drho_stencil=1), dict(fx=1e-5, fy=-2e-5),
                                dict(force=True)])
def test_options(kw):
    nx, ny = 100, 41
    if kw.pop("force", False):
        kw["force"] = hartmann_force(nx, ny, 1e-5, 2.0)
    for sides in (CHANNEL, (PERIODIC, PERIODIC, WALL, WALL)):
        same_after(nx, ny, sides, "f64", **kw)


@pytest.mark.parametrize("check_every", [1, 2, 3, 4, 5, 7, 100])
def test_windows_and_checkpoints(check_every, tmp_path):
    """Captured windows of any length (their lattice swaps are odd or even),
    residuals, and a checkpoint in the middle of a pair."""
    from paper_1806_10251_amd import lbm
    print("[gpu-case] two-step windows", check_every, flush=True)
    nx, ny = 90, 45
    kw = dict(nu=0.03, gamma=0.6, u_in_max=0.03, check_every=check_every, storage="f16")
    m = obstacles(nx, ny)
    a = lbm.Lattice(nx, ny, CHANNEL, solid=m, **kw)
    b = lbm.Lattice(nx, ny, CHANNEL, solid=m, **kw)
    for n in (201, 13, 2 * check_every, 3):
        a.step(n)
        for _ in range(n):
            b.step(1)
        if a.steps >= check_every:
            assert a.residual == b.residual and a.mass == b.mass
    a.save(tmp_path / "c")
    c = lbm.Lattice(nx, ny, CHANNEL, solid=m, **kw)
    c.load_checkpoint(tmp_path / "c")
    c.step(9)
    b.step(9)
    for p, q in zip(c.fields(), b.fields()):
        np.testing.assert_array_equal(p, q)


def batch_of(shapes, storage, check_every, masks):
    from paper_1806_10251_amd import lbm
    grids = [lbm.make_grid(nx, ny, s) for nx, ny, s in shapes]
    params = [lbm.make_params(nu=0.02 + 0.002 * i, gamma=0.5, u_lid=0.05, u_in_max=0.03,
                              storage=storage, check_every=check_every)
              for i in range(len(shapes))]
    b = lbm.Batch(grids, masks, params)
    lats = [lbm.Lattice(nx, ny, s, solid=m, nu=0.02 + 0.002 * i, gamma=0.5, u_lid=0.05,
                        u_in_max=0.03, storage=storage, check_every=check_every)
            for i, ((nx, ny, s), m) in enumerate(zip(shapes, masks))]
    for i, (nx, ny, _) in enumerate(shapes):
        y, x = np.mgrid[0:ny, 0:nx]
        start = (1 + 1e-3 * np.sin(0.3 * x), 0.01 * np.sin(0.2 * y), 0.01 * np.cos(0.1 * x + y))
        b.init_fields(i, *start)
        lats[i].init_fields(*start)
    return b, lats


# one entry per launch shape of a batch, and one that stays step by step
BATCHES = {
    "2 rows": [(40, 31, CAVITY), (16, 16, (PERIODIC,) * 4), (90, 33, CHANNEL)],
    "6 rows": [(64, 64, CAVITY)] * 6 + [(130, 61, CHANNEL), (59, 23, (PERIODIC, PERIODIC, WALL, LID))],
    "10 rows": [(190, 200, CHANNEL)] * 2 + [(190, 200, CAVITY)],
    "two rows per wavefront": [(400, 260, CHANNEL)] * 2 + [(300, 210, CAVITY)] * 2 + [(40, 20, CAVITY)],
    "beyond the last-level cache": [(1100, 900, CHANNEL)] * 3 + [(1000, 1000, CAVITY)],
    "step by step": [(64, 64, CAVITY)] * 30,
    "narrow": [(15, 40, CAVITY), (40, 31, CAVITY)],
}


@pytest.mark.parametrize("storage", ["f32", "f64"])
@pytest.mark.parametrize("key", BATCHES)
def test_batch_launch_shapes(key, storage):
    shapes = BATCHES[key]
    masks = [obstacles(nx, ny) if i % 2 == 0 and min(nx, ny) > 25 else None
             for i, (nx, ny, _) in enumerate(shapes)]
    print("[gpu-case] two-step batch", key, storage, flush=True)
    b, lats = batch_of(shapes, storage, 10, masks)
    for n in (7, 24, 30, 2, 1):   # partial windows, whole ones, odd starts
        b.run(0.0, n)
        for i, (nx, ny, _) in enumerate(shapes):
            for _ in range(n):
                lats[i].step(1)
            fluid = np.ones((ny, nx), bool) if masks[i] is None else masks[i] == 0
            for p, q in zip(b.fields(i, ny, nx), lats[i].fields()):
                np.testing.assert_array_equal(np.asarray(p)[fluid], np.asarray(q)[fluid])


@pytest.mark.parametrize("check_every", [1, 2, 3, 5, 8, 9])
def test_batch_windows(check_every):
    """Windows of odd and even lattice swaps, cases that retire at different
    checks, and a later run that takes them up again."""
    shapes = [(40, 31, CAVITY), (33, 40, CAVITY), (90, 33, CHANNEL)]
    b, lats = batch_of(shapes, "f64", check_every, [None] * 3)
    n = 3 * check_every
    b.run(0.0, n)
    for lat in lats:
        for _ in range(n):
            lat.step(1)
    for lat in lats:                  # the first check at which a run retires cases
        for _ in range(2 * check_every):
            lat.step(1)
    res = sorted(lat.residual for lat in lats)
    assert res[0] < res[1]
    done = b.run(0.5 * (res[0] + res[1]), 5 * check_every)
    more = b.run(0.0, check_every + 1)
    assert len(set(int(d) for d in done)) > 1
    for i, (nx, ny, _) in enumerate(shapes):
        for _ in range(int(done[i]) + int(more[i]) - 2 * check_every):
            lats[i].step(1)
        for p, q in zip(b.fields(i, ny, nx), lats[i].fields()):
            np.testing.assert_array_equal(np.asarray(p), np.asarray(q))


@pytest.mark.parametrize("nx,ny", [(200, 190), (700, 333)])
def test_changes_of_storage_and_launch_shape(nx, ny):
    """Storage and launch shape change in the middle of a run of a lattice with a
    mask: the two-step shape and its marks are chosen again."""
    from paper_1806_10251_amd import lbm
    print("[gpu-case] two-step changes", nx, ny, flush=True)
    m = obstacles(nx, ny)
    a, b = pair(nx, ny, CHANNEL, "f64", mask=m)
    shapes = lbm.launch_shapes()

    def both(n):
        a.step(n)
        for _ in range(n):
            b.step(1)
        for p, q in zip(a.fields(), b.fields()):
            np.testing.assert_array_equal(p, q)

    both(5)
    for storage in ("f32", "f16", "f32", "f64"):
        a.set_storage(storage)
        b.set_storage(storage)
        both(6)
    for shape in ((8, 2), (4, 1)):
        assert shape in shapes
        a.set_launch(*shape)
        b.set_launch(*shape)
        both(7)


def test_steps_on_a_stream_of_the_caller():
    """Lattices and a batch on streams of their own, their steps queued in turn."""
    import torch
    from paper_1806_10251_amd import lbm
    print("[gpu-case] two-step streams", flush=True)
    a, b = pair(123, 90, CAVITY, "f32", mask=obstacles(123, 90))
    c, d = pair(250, 61, CHANNEL, "f64")
    streams = [torch.cuda.Stream() for _ in range(3)]
    a.set_stream(streams[0])
    c.set_stream(streams[1])
    bat, lats = batch_of([(64, 64, CAVITY), (90, 33, CHANNEL)], "f32", 10, [None, None])
    bat.set_stream(streams[2])
    for n in (3, 8, 25):
        a.step(n)
        c.step(n)
        bat.run(0.0, n)
    for one in (b, d, *lats):
        for _ in range(36):
            one.step(1)
    got = [a.fields(), c.fields(), bat.fields(0, 64, 64), bat.fields(1, 33, 90)]
    for p, q in zip(got, (b, d, *lats)):
        for x, y in zip(p, q.fields()):
            np.testing.assert_array_equal(x, y)


def test_fp64_batch_beyond_the_last_level_cache():
    """FP64 keeps two rows per wavefront whatever the size: three lattices of
    1600 x 1000 hold 0.7 GB."""
    shapes = [(1600, 1000, CHANNEL), (1600, 1000, CAVITY), (1600, 1000, (PERIODIC,) * 4)]
    print("[gpu-case] two-step batch, FP64 beyond the cache", flush=True)
    masks = [obstacles(1600, 1000), None, None]
    b, lats = batch_of(shapes, "f64", 10, masks)
    for n in (7, 16):
        b.run(0.0, n)
        for i, (nx, ny, _) in enumerate(shapes):
            for _ in range(n):
                lats[i].step(1)
            fluid = np.ones((ny, nx), bool) if masks[i] is None else masks[i] == 0
            for p, q in zip(b.fields(i, ny, nx), lats[i].fields()):
                np.testing.assert_array_equal(np.asarray(p)[fluid], np.asarray(q)[fluid])


@pytest.mark.parametrize("nx,ny,sides,storage", [
    (180, 700, CAVITY, "f32"), (190, 800, CHANNEL, "f16"), (129, 1025, (PERIODIC,) * 4, "f64"),
    (64, 1000, CAVITY, "f64"), (512, 512, CAVITY, "f64"),
])
def test_lattices_around_the_rule(nx, ny, sides, storage):
    """Lattices that step one by one by the rule on their tiles, and one whose mask
    (a third of the nodes solid) decides it."""
    m = None
    if nx == ny:
        m = (np.random.default_rng(9).random((ny, nx)) > 0.66).astype(np.uint8)
    same_after(nx, ny, sides, storage, steps=5, mask=m)
