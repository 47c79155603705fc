"""How much device memory a step's emitter queue takes, from the library's own host code on a runtime
of plain memory (tests/host_runtime.c; no GPU needed): where no launch shape is set, no more than the
shape 8 x 2048 takes or a slot per particle and 2^20 more, however short the tiles are; and sfq_reserve
holds the queue of every step within its limits without holding more than that."""
import os
import subprocess

import pytest

from paper_2301_07684_amd import sfq

HERE = os.path.dirname(os.path.abspath(__file__))
DEPTH, LOCAL = 0, 1
PLANE_WAVE = 2
FORMS = [(DEPTH, 0), (LOCAL, 0), (LOCAL, 1)]  # decision, beyond LCFA
ENTRY = {(DEPTH, 0): 48, (LOCAL, 0): 56, (LOCAL, 1): 72}
LAYOUTS = ["1x4096", "20x4096", "500x4096", "1000x4096", "4000000x1,100x4095", "3000x64",
           "8000000x1,1x4095", "2000x4000,300000x1", "50000x100,17x3000", "9000000x1,5x4000",
           "8388607x1", "65536x1", "1003x2"]


@pytest.fixture(scope="module")
def runtime(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("rt") / "host_runtime")
    lib = os.path.dirname(sfq.LIB_PATH)
    subprocess.check_call(
        ["gcc", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
         "-I" + os.path.join(HERE, "..", "include"), "-rdynamic",
         os.path.join(HERE, "host_runtime.c"), "-o", exe, "-L" + lib, "-lsfq",
         "-Wl,-rpath," + lib, "-Wl,--unresolved-symbols=ignore-in-shared-libs"])

    def run(form, shape, *actions, limit=0, field=0):
        args = [*form, *(shape or (0, 0)), limit, field]
        r = subprocess.run([exe, *map(str, args), *actions], capture_output=True, text=True,
                           timeout=60)
        assert r.returncode == 0, r.stdout + r.stderr
        return [tuple(map(int, line.split())) for line in r.stdout.splitlines()]

    return run


def particles(layout):
    return sum(int(n) * int(k) for n, k in (part.split("x") for part in layout.split(",")))


def books(n, tiles):
    """The queue's bytes beside its entries: 52 a block and 16 a chunk (at least 256 particles, or
    what a tile ends with), and some alignment."""
    return 68 * (n // 256 + 2 * tiles) + 4096


@pytest.mark.parametrize("field", [0, PLANE_WAVE])
@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("layout", LAYOUTS)
def test_short_tiles_do_not_multiply_the_queue(runtime, form, layout, field):
    n = particles(layout)
    tiles = sum(int(part.split("x")[1]) for part in layout.split(","))
    (st, fixed, _, _), = runtime(form, (8, 2048), "step:" + layout, field=field)
    assert st == 0
    most = max(fixed, (n + (1 << 20)) * ENTRY[form] + books(n, tiles))
    (st, held, _, _), = runtime(form, None, "step:" + layout, field=field)
    assert st == 0 and held <= most
    (st, _, plan, _), = runtime(form, None, "plan:" + layout, field=field)
    assert st == 0 and plan <= most + tiles * 300 + 4096


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("limits", ["8388608:4096", "1200000:2", "1000:1", "20000000:300"])
def test_reserve_holds_what_it_may_need(runtime, form, limits):
    n, tiles = map(int, limits.split(":"))
    steps = []
    for layout in LAYOUTS + [f"{n}x1", f"{n // 2}x2", f"{max(n // tiles, 1)}x{tiles}",
                             f"{n // 2}x1,1x{tiles - 1}", "1x1", "700x1"]:
        if particles(layout) <= n and \
                sum(int(part.split("x")[1]) for part in layout.split(",")) <= tiles:
            steps.append("step:" + layout)
    for field in (0, 1, PLANE_WAVE):
        first, *rest = runtime(form, None, "reserve:" + limits, *steps, field=field)
        assert first[0] == 0 and len(rest) == len(steps) >= 2
        assert all(st == 0 and held == first[1] for st, held, _, _ in rest)
    fixed = runtime(form, (8, 2048), "reserve:" + limits)[0][1]
    assert first[1] <= max(fixed, (min(n, 1 << 23) + (1 << 20)) * ENTRY[form] + books(n, tiles))


OUT_OF_MEMORY = 3


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("field", [0, PLANE_WAVE])
def test_short_memory(runtime, form, field):
    """Where the picked shape's queue does not fit the device and that of 8 x 2048 does, the step, the
    plan and the reservation use the latter."""
    step, plan, reserve = "step:8300000x1", "plan:8300000x1", "reserve:8300000:1"
    picked, = runtime(form, None, step, field=field)
    fixed, = runtime(form, (8, 2048), step, field=field)
    assert fixed[1] < picked[1] and (picked[0], picked[3]) == (0, 4053 if form[1] else 2027)
    limit = (fixed[2] + picked[2]) // 2
    st, held, _, grid = runtime(form, None, step, step, limit=limit, field=field)[1]
    assert (st, grid) == (0, 2048) and held == fixed[1]
    (st, held, _, grid), small = runtime(form, None, plan, "step:1000x1", limit=limit, field=field)
    assert (st, grid) == (0, 2048) and (small[0], small[3]) == (0, 4)
    res = runtime(form, None, reserve, step, "step:65536x1", limit=limit, field=field)
    assert [r[0] for r in res] == [0, 0, 0] and len({r[1] for r in res}) == 1


def test_refused_memory_leaves_nothing_behind(runtime):
    """A step refused for lack of memory is refused by itself: the handle's next steps, which fit, work
    and are shaped as before."""
    for action in ("step:", "plan:", "reserve:"):
        res = runtime((DEPTH, 0), None, action + ("2000000:1" if action == "reserve:" else "2000000x1"),
                      "step:1000x1", limit=20_000_000)
        assert [r[0] for r in res] == [OUT_OF_MEMORY, 0] and res[1][3] == 4


def test_unset_shape(runtime):
    """A handle whose shape was set picks again after sfq_auto_launch."""
    res = runtime((DEPTH, 0), (8, 2048), "step:65536x1", "auto:", "step:65536x1", "step:2000000x1")
    assert [r[0] for r in res] == [0, 0, 0, 0]
    assert [r[3] for r in res] == [33, 33, 257, 489]


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("layout", ["9000000x1", "16777216x2", "200000000x1", "1000x4096",
                                    "50000x100,17x3000", "9000000x1,5x4000"])
def test_resident_blocks_hold_as_many_emitters(runtime, form, layout):
    """The resident blocks of a picked shape are fewer than those of 8 x 2048; their queue holds as
    many entries, so that no more shares are deferred."""
    for field in (0, 1, PLANE_WAVE):
        (st, held, _, grid), = runtime(form, None, "step:" + layout, field=field)
        (_, fixed, _, blocks), = runtime(form, (8, 2048), "step:" + layout, field=field)
        assert st == 0 and grid < blocks
        # beside the entries: 52 bytes a block and 16 a chunk, some alignment, and what does not divide
        # by the slices
        chunks = particles(layout) // 2048 + 4096
        assert held >= fixed - 64 * blocks - 16 * chunks - 4 * grid * ENTRY[form]
