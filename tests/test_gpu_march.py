"""The register-march plans (and the default plan, which takes them where they
apply) against the direct plan, bit for bit: every plan forms each cell by the
same arithmetic, so the fields must be equal at the edges of tiles, of lanes
and of z chunks, for every face rule the plans take, whatever is left of a
step count, and the calls they refuse must fall back."""
import numpy as np
import pytest

from paper_1004_0480_amd import rd
from paper_1004_0480_amd import workloads as W

pytestmark = pytest.mark.gpu

MIRROR, PERIODIC = ("mirror", 0.0), ("periodic", 0.0)
GHOST, HELD = ("ghost", 0.7), ("held", 0.6)
# x-, x+, y faces, z faces
FACES = {"mirror": (MIRROR, MIRROR, MIRROR, MIRROR), "periodic": (PERIODIC, PERIODIC, PERIODIC, PERIODIC),
         "ghost_lo": (GHOST, MIRROR, MIRROR, PERIODIC), "ghost_hi": (MIRROR, GHOST, PERIODIC, MIRROR)}
# several rows in a wave; ragged rows; a row per wave; the fewest lanes; rows
# longer than a workgroup takes whole; the fewest rows and planes; one cell past
# a lane
SHAPES = [(9, 37, 64), (7, 40, 101), (20, 23, 256), (6, 33, 29), (5, 11, 2060), (4, 5, 260), (6, 9, 385), (6, 70, 24), (4, 9, 5),
          (5, 7, 1)]


def spec_of(model, shape, faces):
    s = (W.diffusion_spec() if model == "diffusion" else W.brusselator_spec() if model == "brusselator" else
         W.turing_spec() if model == "turing" else W.pollutant_spec(shape, 5, ns=int(model[-1]), nsrc=40))
    if model == "diffusion":
        s.K = [[1.0, 0.7, 0.4]]
    xl, xh, y, z = faces
    s.bc = [[xl, xh, y, y, z, z] for _ in range(s.ns)]
    return s


def run(spec, shape, fields, storage, steps, plan=None, chunk=0, rounding=None):
    import torch
    g = rd.Grid(shape, spec.ns, spec.h, storage, stream=torch.cuda.Stream() if chunk else None)
    g.set_model(spec)
    if rounding is not None:
        g.set_rounding("stochastic", rounding)
    if plan is not None or chunk:
        g.set_plan(**dict(plan or {}, graph_chunk=chunk))
    for s, f in enumerate(fields):
        g.write(s, f)
    for n in steps:
        g.step(n)
    got, used = g.read_all(np.float32), g.plan()
    g.close()
    return got, used


def same(a, b):
    return all(np.array_equal(x, y) for x, y in zip(a, b))


def fields_of(shape, ns, seed):
    rng = np.random.default_rng(seed)
    return [rng.random(shape) + 0.5 for _ in range(ns)]


@pytest.mark.parametrize("storage", ["f32", "bf16"])
@pytest.mark.parametrize("model,shapes", [("diffusion", [(1, 8, 2), (1, 16, 2), (1, 8, 3), (1, 16, 3), (1, 8, 4)]),
                                          ("brusselator", [(1, 8, 2), (1, 16, 2), (2, 8, 2)]),
                                          ("pollutant4", [(1, 8, 2), (2, 8, 2)]),
                                          ("pollutant3", [(1, 16, 2)]), ("pollutant1", [(1, 8, 4)])])
def test_march_plans_bitwise(model, shapes, storage):
    for shape in SHAPES:
        for name, faces in FACES.items():
            spec = spec_of(model, shape, faces)
            f = fields_of(shape, spec.ns, 3)
            ref, _ = run(spec, shape, f, storage, [7], dict(kernel="direct"))
            for ry, w, k in shapes:
                for cz in (0, 3):
                    plan = dict(kernel="march", vx=4, ry=ry, waves=w, prefetch=k, cz=cz, order=cz & 1)
                    if name == "periodic" and shape[2] % 4 and shape[2] > 256:
                        # whole rows only (a halo lane cannot hold a ragged
                        # wrap): too few rows fit some shapes
                        try:
                            got, used = run(spec, shape, f, storage, [7], plan)
                        except rd.RDError as e:
                            assert e.code == rd.EINVAL
                            continue
                    else:
                        got, used = run(spec, shape, f, storage, [7], plan)
                    assert used["kernel"] == 8
                    assert same(got, ref), (model, shape, name, plan)


def test_march_graphs_split_calls_and_left_steps():
    shape = (12, 30, 100)
    spec = spec_of("diffusion", shape, FACES["mirror"])
    f = fields_of(shape, 1, 4)
    for k, w in ((4, 8), (3, 16), (2, 8)):
        plan = dict(kernel="march", vx=4, ry=1, waves=w, prefetch=k, cz=5)
        ref, _ = run(spec, shape, f, "f32", [33], dict(kernel="direct"))
        for chunk in (0, 2, 6, 10):
            for calls in ([33], [1, 2, 3, 5, 22]):
                got, _ = run(spec, shape, f, "f32", calls, plan, chunk)
                assert same(got, ref), (k, chunk, calls)


@pytest.mark.parametrize("storage", ["f32", "bf16", "f16"])
def test_default_plan_bitwise(storage):
    """Every kind of face, also those the register march refuses (the default
    plan then falls back), mixed between fields and passes, on small and odd
    grids."""
    one = [[MIRROR] * 6, [PERIODIC] * 6, [HELD, MIRROR] + [MIRROR] * 4, [MIRROR] * 4 + [HELD, GHOST],
           [MIRROR, MIRROR, GHOST, MIRROR, MIRROR, MIRROR], [GHOST, GHOST] + [PERIODIC] * 4]
    for shape in ((1, 1, 1), (2, 3, 40), (5, 2, 33), (3, 4, 28), (9, 21, 130), (30, 33, 37)):
        for model in ("diffusion", "brusselator", "pollutant4"):
            for i, bc in enumerate(one):
                spec = spec_of(model, shape, FACES["mirror"])
                # the last field of a model with several takes other rules
                spec.bc = [list(bc) for _ in range(spec.ns)]
                if spec.ns > 1 and i % 2:
                    spec.bc[-1] = list(one[(i + 1) % len(one)])
                f = fields_of(shape, spec.ns, 5)
                ref, _ = run(spec, shape, f, storage, [5], dict(kernel="direct"))
                got, used = run(spec, shape, f, storage, [5])
                assert same(got, ref), (shape, model, i, used)


@pytest.mark.parametrize("storage,rounding", [("f32", None), ("bf16", None), ("bf16", 5)])
def test_front_march_bitwise(storage, rounding):
    for shape in SHAPES + [(2, 9, 388), (3, 64, 32)]:
        for za, zb, k2 in ((HELD, MIRROR, 0.0), (MIRROR, GHOST, 0.5), (GHOST, HELD, 0.0)):
            spec = W.front_spec()
            spec.params = dict(spec.params, k2=k2)
            spec.bc[0][4], spec.bc[1][5] = za, zb
            f = [0.5 * x for x in fields_of(shape, 3, 6)]
            ref, _ = run(spec, shape, f, storage, [3], dict(kernel="direct"), rounding=rounding)
            for ry, w in ((2, 8), (1, 8), (1, 16)):
                for cz in (0, 3):
                    plan = dict(kernel="fused", vx=0, ry=ry, waves=w, prefetch=1, cz=cz)
                    if rounding is not None and shape[2] % 4:
                        with pytest.raises(rd.RDError):
                            run(spec, shape, f, storage, [1], plan, rounding=rounding)
                        continue
                    got, _ = run(spec, shape, f, storage, [3], plan, rounding=rounding)
                    assert same(got, ref), (shape, za, zb, plan)
            got, _ = run(spec, shape, f, storage, [3], rounding=rounding)
            assert same(got, ref), (shape, za, zb, "default plan")


def test_march_refusals():
    def refused(spec, shape, storage="f32", **plan):
        g = rd.Grid(shape, spec.ns, spec.h, storage)
        g.set_model(spec)
        with pytest.raises(rd.RDError) as e:
            g.set_plan(**plan)
        assert e.value.code == rd.EINVAL and "slab" not in str(e.value)
        with pytest.raises(rd.RDError, match="slab shape not available"):
            g.set_plan(kernel="block", vx=3)
        g.step(1)
        g.close()

    p = dict(kernel="march", vx=4, ry=1, waves=8, prefetch=2)
    mirror = FACES["mirror"]
    refused(spec_of("diffusion", (8, 8, 64), (HELD, MIRROR, MIRROR, MIRROR)), (8, 8, 64), **p)
    refused(spec_of("diffusion", (8, 8, 64), (MIRROR, MIRROR, GHOST, MIRROR)), (8, 8, 64), **p)
    refused(spec_of("diffusion", (8, 8, 64), mirror), (8, 8, 64), **dict(p, vx=2))
    refused(spec_of("diffusion", (8, 8, 64), mirror), (8, 8, 64), **dict(p, prefetch=5))
    refused(spec_of("diffusion", (1, 8, 64), mirror), (1, 8, 64), **p)      # fewer planes than steps
    refused(spec_of("diffusion", (8, 8, 64), mirror), (8, 8, 64), "f16", **p)
    rk = spec_of("diffusion", (8, 8, 64), mirror)
    rk.integrator = "rk2"
    refused(rk, (8, 8, 64), **p)

def test_march_plan_gives_way_to_later_settings():
    """A register-march plan that was set by name (as from autotune) and does
    not take a rounding, integrator or face set later gives way while it
    cannot run, and comes back."""
    shape, mirror = (8, 8, 64), FACES["mirror"]
    p = dict(kernel="march", vx=4, ry=1, waves=8, prefetch=2)
    spec = spec_of("brusselator", shape, mirror)
    rk, held = spec_of("brusselator", shape, mirror), spec_of("brusselator", shape, (HELD,) + mirror[1:])
    rk.integrator = "rk2"
    f = fields_of(shape, 2, 8)
    g = rd.Grid(shape, 2, spec.h, "bf16")
    g.set_model(spec)
    g.set_plan(**p)
    assert g.plan()["kernel"] == 8
    for other, rounding in ((spec, 1), (rk, None), (held, None)):
        g.set_model(other)
        if rounding is not None:
            g.set_rounding("stochastic", rounding)
        assert g.plan()["kernel"] != 8
        for s, x in enumerate(f):
            g.write(s, x)
        g.step(3)
        assert same(g.read_all(np.float32), run(other, shape, f, "bf16", [3], dict(kernel="direct"), rounding=rounding)[0])
        if rounding is not None:
            g.set_rounding("nearest")
            assert g.plan()["kernel"] == 8
    g.set_model(spec)
    assert g.plan()["kernel"] == 8
    g.close()


@pytest.mark.parametrize("storage", ["f32", "bf16"])
def test_batched_march_bitwise(storage):
    """Grids of a batch against the same grids alone: even and odd step counts
    and ticks, rows inside a wave, across waves and ragged, all faces; and a
    batch with a grid the register march does not take."""
    import torch
    cases = [("diffusion", (32, 32, 32), "mirror", 9), ("brusselator", (20, 33, 64), "periodic", 6),
             ("diffusion", (5, 40, 101), "periodic", 7), ("brusselator", (33, 17, 48), "ghost_lo", 1),
             ("diffusion", (48, 48, 48), "ghost_hi", 0), ("brusselator", (9, 130, 140), "mirror", 4)]
    held = ("diffusion", (12, 20, 40), (HELD, MIRROR, MIRROR, MIRROR), 5)
    for extra in ((), (held,)):
        for chunk in (1, 3, 4, 20):
            stream = torch.cuda.Stream()
            b = rd.Batch(8, 1 << 34, storage, stream=stream)
            grids, refs = [], []
            for model, shape, faces, steps in tuple(cases) + extra:
                spec = spec_of(model, shape, FACES[faces] if isinstance(faces, str) else faces)
                f = fields_of(shape, spec.ns, steps)
                refs.append(run(spec, shape, f, storage, [steps], dict(kernel="direct"))[0])
                g = rd.Grid(shape, spec.ns, spec.h, storage, stream=stream)
                g.set_model(spec)
                for s, x in enumerate(f):
                    g.write(s, x)
                b.add(g, steps)
                grids.append(g)
            done = []
            while len(done) < len(grids):
                done += b.step(chunk)
            for g, ref in zip(grids, refs):
                assert same(g.read_all(np.float32), ref), (g.shape, chunk, len(extra))
            b.close()
            for g in grids:
                g.close()


@pytest.mark.parametrize("storage", ["f32", "bf16"])
@pytest.mark.parametrize("model", ["diffusion", "brusselator", "turing"])
def test_march19_plans_bitwise(model, storage):
    """The 19-point march (an LDS plan with vx = 0, whose ry is the whole-row
    worth of a tile): rows of one tile and of several, of every lane count,
    ragged ends and all faces; left steps; and the default plan, which also has
    to take the grids that the march refuses."""
    for shape in SHAPES + [(3, 31, 56), (8, 29, 57), (5, 18, 240), (6, 4, 256)]:
        for name, faces in dict(FACES, held=(HELD, MIRROR, MIRROR, MIRROR), ghost_y=(MIRROR, MIRROR, GHOST, MIRROR)).items():
            spec = spec_of(model, shape, faces)
            spec.stencil = 19
            spec.K = [[max(k)] * 3 for k in spec.K]
            f = fields_of(shape, spec.ns, 9)
            ref, _ = run(spec, shape, f, storage, [5], dict(kernel="direct"))
            got, used = run(spec, shape, f, storage, [5])
            assert same(got, ref), (model, shape, name, used)
            if name in ("held", "ghost_y") or (name == "periodic" and shape[2] % 4):
                assert (used["kernel"], used["vx"]) != (rd.KERNEL["lds"], 0)
                continue
            assert (used["kernel"], used["vx"]) == (rd.KERNEL["lds"], 0)
            g = rd.Grid(shape, spec.ns, spec.h, storage)
            g.set_model(spec)
            plans = []
            for k in (1, 2):
                for ry in range(1, 33):
                    try:
                        g.set_plan(kernel="lds", vx=0, ry=ry, waves=8, prefetch=k, cz=3)
                        plans.append(g.plan())
                    except rd.RDError as e:
                        assert e.code == rd.EINVAL
            g.close()
            assert {p["prefetch"] for p in plans} == {1, 2}
            for plan in plans:
                got, _ = run(spec, shape, f, storage, [2, 3], dict(plan, kernel="lds"))
                assert same(got, ref), (model, shape, name, plan)


def test_tuning_one_class_of_faces_leaves_the_other_its_plans():
    """Autotuning a grid whose faces no register march takes does not keep grids
    of its shape from theirs, nor the other way round; and a tuned march that
    gives way to a rounding it does not take is followed by a plan that does."""
    mirror = FACES["mirror"]
    for first, shape in (("held", (22, 26, 68)), ("mirror", (24, 26, 68))):
        spec = {"held": spec_of("brusselator", shape, (HELD,) + mirror[1:]), "mirror": spec_of("brusselator", shape, mirror)}
        f = fields_of(shape, 2, 4)
        used = {}
        for name in (first, "mirror" if first == "held" else "held"):
            g = rd.Grid(shape, 2, 1.0, "bf16")
            g.set_model(spec[name])
            for s, x in enumerate(f):
                g.write(s, x)
            if name == first:
                g.set_plan(**dict(g.autotune(4), graph_chunk=0))
            used[name] = g.plan()
            g.step(5)
            got = g.read_all(np.float32)
            assert same(got, run(spec[name], shape, f, "bf16", [5], dict(kernel="direct"))[0])
            if name == first == "mirror":
                g.set_rounding("stochastic", 3)
                assert g.plan()["kernel"] != 8
            g.close()
        assert used["held"]["kernel"] != 8
        if first == "held":
            assert used["mirror"]["kernel"] == 8


def test_held_faces_borrow_no_ring():
    """A 7-point ring that was timed on a grid with mirror faces is not lent to
    one with held faces, where it is slower than the default plan."""
    mirror = FACES["mirror"]
    for model, shape, storage in (("brusselator", (192, 192, 192), "f32"), ("pollutant4", (100, 101, 725), "bf16")):
        plans = []
        for faces in (mirror, (HELD,) + mirror[1:]):
            spec = spec_of(model, shape, faces)
            g = rd.Grid(shape, spec.ns, 1.0, storage)
            g.set_model(spec)
            for s in range(spec.ns):
                g.write(s, np.full(shape, 0.5, np.float32))
            if faces is mirror:
                g.autotune(4)
            plans.append(g.plan()["kernel"])
            g.close()
        assert plans[1] not in (4, 5, 7), (model, plans)


def test_march19_orders_bitwise():
    """Both tile orders of the 19-point march, with left-over launches, on grids
    of several tiles along every axis."""
    for shape in ((13, 70, 300), (21, 65, 57), (9, 40, 64)):
        spec = W.turing_spec()
        f = fields_of(shape, 2, 12)
        ref, _ = run(spec, shape, f, "f32", [5], dict(kernel="direct"))
        g = rd.Grid(shape, 2, spec.h, "f32")
        g.set_model(spec)
        plans = []
        for k in (1, 2):
            for ry in range(1, 33):
                try:
                    g.set_plan(kernel="lds", vx=0, ry=ry, waves=8, prefetch=k, cz=4, order=1)
                    plans.append(g.plan())
                except rd.RDError as e:
                    assert e.code == rd.EINVAL
        g.close()
        assert {p["prefetch"] for p in plans} == {1, 2} and all(p["order"] == 1 for p in plans)
        for plan in plans:
            got, _ = run(spec, shape, f, "f32", [2, 3], dict(plan, kernel="lds"))
            assert same(got, ref), (shape, plan)


def check_single_steps_of_a_large_field(spec, shape, stencil_march, storage="f32"):
    """A grid whose buffers pass the last cache (256 MB), by default plan: calls
    that leave one step, directly and in graphs, from both parities; then a
    Runge-Kutta model on the same grid, whose stage arguments the left-over
    launch borrows."""
    import torch
    rng = np.random.default_rng(8)
    f = [(rng.random(shape, dtype=np.float32) + np.float32(0.5)) for _ in range(spec.ns)]
    rk = W.ModelSpec(**dict(vars(spec), integrator="rk2"))

    def sequence(plan, chunk):
        g = rd.Grid(shape, spec.ns, spec.h, storage, stream=torch.cuda.Stream())
        g.set_model(spec)
        g.set_plan(**dict(plan, graph_chunk=chunk))
        used = g.plan()
        for s, x in enumerate(f):
            g.write(s, x)
        out = []
        for n in (1, 2, 5, 1):
            g.step(n)
            out.append([x[::7].copy() for x in g.read_all(np.float32)])
        g.set_model(rk)
        g.step(3)
        out.append(g.read_all(np.float32))
        g.set_model(spec)
        g.step(3)
        out.append(g.read_all(np.float32))
        g.close()
        return out, used

    ref, _ = sequence(dict(kernel="direct"), 0)
    for chunk in (0, 2, 6):
        got, used = sequence(dict(kernel="auto"), chunk)
        assert (used["kernel"], used["vx"]) == ((rd.KERNEL["lds"], 0) if stencil_march else (rd.KERNEL["march"], 4))
        for i, (a, b) in enumerate(zip(got, ref)):
            assert same(a, b), (chunk, i)


@pytest.mark.parametrize("model", ["diffusion", "pollutant1"])
def test_single_steps_of_a_large_field(model):
    shape = (322, 280, 330)
    assert 2 * 384 * shape[0] * shape[1] * 4 > 256 << 20
    check_single_steps_of_a_large_field(spec_of(model, shape, FACES["ghost_lo" if model != "diffusion" else "mirror"]), shape,
                                        False)


@pytest.mark.parametrize("storage", ["f32", "bf16"])
def test_march_tables_of_long_chunks(storage):
    """A march looks the wind and the source planes up 64 planes at a time: one
    chunk over all planes, with sources on both sides of every refill, on the
    planes next to the faces and in between."""
    for nz in (62, 63, 64, 65, 66, 130):
        shape = (nz, 9, 40)
        zs = sorted(z for z in {0, 1, 2, 31, 59, 60, 61, 62, 63, 64, 65, 66, 67, 123, 124, 125, 126, 127, 128, 129, nz - 2, nz - 1}
                    if z < nz)
        rng = np.random.default_rng(nz)
        cells = np.array([(z * 9 + rng.integers(9)) * 40 + rng.integers(40) for z in zs for _ in range(2)], dtype=np.int64)
        for model, plans in (("pollutant1", [(1, 8, 2), (1, 8, 3), (1, 16, 3), (1, 8, 4)]), ("pollutant4", [(1, 8, 2), (2, 8, 2)])):
            for name in ("mirror", "periodic"):
                spec = spec_of(model, shape, FACES[name])
                spec.sources = (cells, (np.arange(len(cells)) % spec.ns).astype(np.int32), 1.0 + np.arange(len(cells)) / 8.0)
                spec.wind = np.linspace(0.1, 4.0, nz)
                f = fields_of(shape, spec.ns, nz)
                ref, _ = run(spec, shape, f, storage, [9], dict(kernel="direct"))
                for ry, w, k in plans:
                    for cz in (0, 61):
                        plan = dict(kernel="march", vx=4, ry=ry, waves=w, prefetch=k, cz=cz)
                        got, used = run(spec, shape, f, storage, [9], plan)
                        assert used["kernel"] == 8 and same(got, ref), (nz, model, name, plan)


@pytest.mark.parametrize("model,storage", [("diffusion", "f32"), ("turing", "f32"), ("diffusion", "bf16")])
def test_single_steps_of_a_large_19_point_field(model, storage):
    shape = {"diffusion": (300, 300, 384) if storage == "f32" else (460, 300, 504), "turing": (152, 300, 384)}[model]
    spec = spec_of(model, shape, FACES["mirror"])
    spec.stencil = 19
    spec.K = [[max(k)] * 3 for k in spec.K]
    assert 2 * spec.ns * (-(-shape[2] // 64) * 64) * shape[0] * shape[1] * (4 if storage == "f32" else 2) > 256 << 20
    check_single_steps_of_a_large_field(spec, shape, True, storage)


def test_default_plans_of_few_rows():
    """Grids on which a march's tiles hold few rows: long ragged periodic rows,
    few rows of a large grid, a 19-point sheet of one row. The default is the
    plan it was without a march, which a plan set by name may still take."""
    cases = [("brusselator", 7, (20, 90, 725), "block", (1, 16, 2)), ("pollutant4", 7, (1024, 2, 1024), "block", (1, 8, 2)),
             ("turing", 19, (256, 1, 256), "lds", None), ("diffusion", 19, (3, 1, 30000), "direct", None)]
    for model, stencil, shape, kind, march in cases:
        spec = spec_of(model, shape, FACES["periodic" if model == "brusselator" else "mirror"])
        spec.stencil = stencil
        if stencil == 19:
            spec.K = [[max(k)] * 3 for k in spec.K]
        f = fields_of(shape, spec.ns, 14)
        ref, _ = run(spec, shape, f, "f32", [4], dict(kernel="direct"))
        got, used = run(spec, shape, f, "f32", [4])
        assert (used["kernel"], used["vx"] > 0 or kind == "direct") == (rd.KERNEL[kind], True) and same(got, ref), (model, shape, used)
        if march:
            ry, w, k = march
            got, used = run(spec, shape, f, "f32", [4], dict(kernel="march", vx=4, ry=ry, waves=w, prefetch=k))
            assert used["kernel"] == 8 and same(got, ref)


@pytest.mark.parametrize("storage", ["f32", "bf16"])
def test_batches_that_return_to_the_ring(storage):
    """Batches whose members' rows leave a march few rows to store, alone and
    with others, even and odd ticks and single steps, between ticks that march:
    the same bits as alone."""
    import torch
    ragged = ("brusselator", (6, 20, 389), "periodic", 7)
    small = ("diffusion", (16, 32, 32), "mirror", 4)
    for cases in ((ragged, ("brusselator", (5, 18, 405), "periodic", 3)), (ragged,) + (small,) * 5, (ragged, small)):
        for chunk in (1, 3, 4):
            stream = torch.cuda.Stream()
            b = rd.Batch(8, 1 << 34, storage, stream=stream)
            grids, refs = [], []
            for i, (model, shape, faces, steps) in enumerate(cases):
                spec = spec_of(model, shape, FACES[faces])
                f = fields_of(shape, spec.ns, steps + i)
                refs.append(run(spec, shape, f, storage, [steps], dict(kernel="direct"))[0])
                g = rd.Grid(shape, spec.ns, spec.h, storage, stream=stream)
                g.set_model(spec)
                for s, x in enumerate(f):
                    g.write(s, x)
                b.add(g, steps)
                grids.append(g)
            done = []
            while len(done) < len(grids):
                done += b.step(chunk)
            for g, ref in zip(grids, refs):
                assert same(g.read_all(np.float32), ref), (g.shape, chunk)
            b.close()
            for g in grids:
                g.close()


def test_single_steps_of_a_large_batch():
    """A batch of two FP32 fields beyond the last cache, stepped one step and
    three steps a tick: both forms of the launch, from either parity."""
    import torch
    shape = (256, 256, 258)
    spec = spec_of("brusselator", shape, FACES["mirror"])
    rng = np.random.default_rng(3)
    f = [rng.random(shape, dtype=np.float32) + np.float32(0.5) for _ in range(2)]
    ref = [x[::5] for x in run(spec, shape, f, "f32", [6], dict(kernel="direct"))[0]]
    for ticks in ((1,) * 6, (3, 1, 1, 1), (1, 3, 2)):
        stream = torch.cuda.Stream()
        b = rd.Batch(1, 1 << 34, "f32", stream=stream)
        g = rd.Grid(shape, 2, spec.h, "f32", stream=stream)
        g.set_model(spec)
        for s, x in enumerate(f):
            g.write(s, x)
        b.add(g, 6)
        done = [b.step(n) for n in ticks][-1]
        assert len(done) == 1
        assert same([x[::5] for x in g.read_all(np.float32)], ref), ticks
        b.close()
        g.close()
