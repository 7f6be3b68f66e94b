"""GPU tests of the kernels' dispatch edges: each rule that picks a kernel or a
launch shape, at the sizes on both sides of its line, against the oracle."""
import numpy as np
import pytest

from oracle import dp45, sd
from oracle import fields as F
from oracle import potential
from paper_2406_16064_amd import inputs

from _util import field_err, gpu_params, oracle_params, representable, to_dev

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

PAR = dict(Ms=5.8e5, A=1.5e-11, D=3e-3, Ku=8e5, u=(0.2, -0.3, 1.0), H=(3e4, -2e4, 2e5), alpha=0.3)


@pytest.fixture(scope="module")
def mm():
    if not torch.cuda.is_available():
        pytest.fail("GPU test run without a GPU")
    from paper_2406_16064_amd import mm as m
    return m


def _m(mesh, seed):
    return inputs.random_unit(*mesh[:3], np.random.default_rng(seed))


@pytest.mark.parametrize("ny", [64, 65, 95, 97])
def test_error_norm_over_many_workgroups_fp64(mm, ny):
    """The step decision gathers one workgroup a row here: up to 64 at the
    instance, beyond that over 32 arrival slots (65 and 97: one slot holds one
    more than the others, 95: one less).  Four attempts of two instances, so
    that each finds the slots as the one before left them; the error norm of
    every attempt against the oracle's."""
    mesh = (16, ny, 1, 2e-9, 2e-9, 2e-9)
    plan = mm.Plan(mesh, "f64", terms=F.ALL_TERMS, max_batch=2)
    gp, op = gpu_params(mm, PAR, F.ALL_TERMS), oracle_params(PAR, F.ALL_TERMS)
    kern = F.DemagKernel(F.Mesh(*mesh))
    f = lambda y: F.llg_rhs(y, F.Mesh(*mesh), op, kern)
    mo = [_m(mesh, 11), _m(mesh, 12)]
    md = to_dev(np.stack(mo), torch.float64)
    st = mm.new_states(2, h=2e-14)
    ost = [dp45.State(h=2e-14), dp45.State(h=2e-14)]
    for _ in range(4):
        plan.rk45_step([gp, gp], md, st)
        for b in range(2):
            mo[b], acc = dp45.step(f, mo[b], ost[b])
            assert bool(st[b].last_accepted) == acc
            assert abs(st[b].last_err - ost[b].last_err) <= 1e-9 * max(1.0, ost[b].last_err)
            assert field_err(md[b].cpu().numpy(), mo[b]) <= 1e-12


@pytest.mark.parametrize("prec,tol", [("f32", 1e-5), ("f64", 1e-11)])
@pytest.mark.parametrize("mesh", [(20, 128, 2), (9, 128, 3), (16, 128, 4), (10, 256, 2), (6, 256, 3), (5, 512, 2),
                                  (8, 256, 4), (6, 512, 3), (12, 127, 2), (12, 128, 5)])
def test_fused_yz_planes(mm, mesh, prec, tol):
    """Fields of small 3-D meshes on both sides of the fused y and z passes:
    nz = 2 to 4 with 128, 256 and 512 rows (fused while a kx fits 64 KB of LDS),
    a length and a plane count that keep the separate passes.  Two instances."""
    mesh = mesh + (3e-9, 2e-9, 2.5e-9)
    plan = mm.Plan(mesh, prec, terms=F.ALL_TERMS, max_batch=2)
    gp, op = gpu_params(mm, PAR, F.ALL_TERMS), oracle_params(PAR, F.ALL_TERMS)
    kern = F.DemagKernel(F.Mesh(*mesh))
    m = [representable(_m(mesh, s), plan.dtype) for s in (21, 22)]
    H = plan.effective_field([gp, gp], to_dev(np.stack(m), plan.dtype)).double().cpu().numpy()
    for b in range(2):
        assert field_err(H[b], F.effective_field(m[b], F.Mesh(*mesh), op, kern)) <= tol


def test_fused_yz_batch_with_films_fp64(mm):
    """A batch whose films and fused planes share one y launch (Py = 256), next
    to a mesh with the separate passes: each trajectory against the oracle's."""
    meshes = [(12, 128, 1, 2e-9, 2e-9, 2e-9), (10, 128, 2, 2e-9, 2e-9, 2e-9), (10, 20, 2, 2e-9, 2e-9, 2e-9)]
    batch = mm.Batch(meshes, "f64")
    gp, op = gpu_params(mm, PAR, F.ALL_TERMS), oracle_params(PAR, F.ALL_TERMS)
    which = [1, 0, 2, 1]
    m0 = [_m(meshes[k], 30 + i) for i, k in enumerate(which)]
    md = [to_dev(m, torch.float64) for m in m0]
    t_end = 8e-14
    batch.run([dict(mesh_id=k, params=gp, m=md[i], t_end=t_end, state=mm.new_states(1, h=2e-14, h_max=2e-14)[0])
               for i, k in enumerate(which)])
    for i, k in enumerate(which):
        mesh = F.Mesh(*meshes[k])
        kern = F.DemagKernel(mesh)
        mo = dp45.run(lambda y: F.llg_rhs(y, mesh, op, kern), m0[i], dp45.State(h=2e-14, h_max=2e-14), t_end=t_end)
        assert np.max(np.abs(md[i].cpu().numpy() - mo)) <= 1e-9


@pytest.mark.parametrize("steps", [1, 7, 8, 9, 17, 70])
def test_run_submits_the_attempts_it_needs_fp64(mm, steps):
    """A run of `steps` equal steps, submitted one by one (up to 63 expected) or
    in graphs of eight and a rest (70), against as many single attempts: the
    same kernels, so the same bits, and no attempt more or less."""
    mesh = (16, 12, 1, 2e-9, 2e-9, 2e-9)
    gp = gpu_params(mm, PAR, F.ALL_TERMS)
    plan = mm.Plan(mesh, "f64", terms=F.ALL_TERMS)
    m0 = inputs.add_noise(inputs.s_state(*mesh[:4]), 1e-2, np.random.default_rng(5))
    h = 1e-14
    a, b = to_dev(m0, torch.float64), to_dev(m0, torch.float64)
    sa, sb = mm.new_states(1, h=h, h_max=h), mm.new_states(1, h=h, h_max=h)
    for t_end in (steps * h, 2 * steps * h):
        plan.rk45_run(gp, a, sa, t_end=t_end)
        for _ in range(steps):  # one attempt a call, to the same end (the last step is what is left to it)
            plan.rk45_run(gp, b, sb, t_end=t_end, max_steps=1, check=False)
        assert sa[0].n_accept == sb[0].n_accept == round(t_end / h) and sa[0].n_reject == 0
        assert torch.equal(a, b)


@pytest.mark.parametrize("n", [1, 12, 60])
def test_parameter_tables_follow_every_call(mm, n):
    """The device tables are sent when their bytes change (one kernel argument,
    several, and a copy for 60 instances): parameters, arrays, batch sizes and
    streams changed from call to call on one plan, each result bit for bit that
    of a fresh plan."""
    mesh = (8, 6, 1, 2e-9, 2e-9, 2e-9)
    plan = mm.Plan(mesh, "f64", terms=F.ALL_TERMS, max_batch=n)
    m = [to_dev(np.stack([_m(mesh, 50 + 100 * k + i) for i in range(n)]), torch.float64) for k in range(2)]
    side = torch.cuda.Stream()

    def pars(seed):
        r = np.random.default_rng(seed)
        return [gpu_params(mm, dict(PAR, Ms=r.uniform(4e5, 9e5), A=r.uniform(5e-12, 2e-11)), F.ALL_TERMS)
                for _ in range(n)]

    for seed, k, nb, other in ((1, 0, n, False), (1, 0, n, False), (1, 1, n, False), (2, 1, n, False), (1, 0, 1, False),
                               (1, 0, n, True), (1, 0, n, False), (2, 0, n, True)):
        p = pars(seed)[:nb]
        fresh = mm.Plan(mesh, "f64", terms=F.ALL_TERMS, max_batch=n).llg_rhs(p, m[k][:nb])
        torch.cuda.synchronize()
        with torch.cuda.stream(side if other else torch.cuda.current_stream()):
            got = plan.llg_rhs(p, m[k][:nb])
        torch.cuda.synchronize()
        assert torch.equal(got, fresh)


LENGTHS = (16, 24, 32, 36, 48, 54, 64, 72, 96, 108, 128, 144, 162, 192, 216, 256, 288, 324, 384, 432, 512, 576, 648,
           768, 864, 972)


def _smooth(n):
    for q in (2, 3):
        while n % q == 0:
            n //= q
    return n == 1


def _short_rows(L):
    """The smallest n whose padded length is L (2n where that is 3-smooth, else the smallest 3-smooth >= 2n - 1)."""
    def padded(n):
        return 2 * n if _smooth(2 * n) else next(P for P in range(2 * n - 1, 4 * n) if _smooth(P))
    return next(n for n in range(2, L // 2 + 1) if padded(n) == L)


@pytest.mark.parametrize("prec,tol", [("f32", 1e-5), ("f64", 1e-11)])
@pytest.mark.parametrize("L", LENGTHS)
def test_compiled_lengths(mm, L, prec, tol):
    """Every compiled transform length against the oracle: rows with Lx = L
    (whole, and one cell short of it where the row still pads to 2 L), columns
    with Py = L (half of it, and the shortest that pads to it), as films, fused
    planes (nz = 2) and separate passes (nz = 5)."""
    gp, op = gpu_params(mm, PAR, F.ALL_TERMS), oracle_params(PAR, F.ALL_TERMS)
    sizes = [(L, 5, 1), (L - 1, 3, 1), (6, L // 2, 1), (6, _short_rows(L), 1), (5, L // 2, 2), (4, _short_rows(L), 5)]
    for k, n in enumerate(sizes):
        mesh = n + (3e-9, 2e-9, 2.5e-9)
        plan = mm.Plan(mesh, prec, terms=F.ALL_TERMS)
        if k in (2, 3, 4, 5):
            assert plan.padded()[1] == L
        m = representable(_m(mesh, 60 + k), plan.dtype)
        H = plan.effective_field(gp, to_dev(m, plan.dtype)).double().cpu().numpy()
        kern = F.DemagKernel(F.Mesh(*mesh))
        assert field_err(H, F.effective_field(m, F.Mesh(*mesh), op, kern)) <= tol, n


@pytest.mark.parametrize("n", [24, 81, 100, 128, 162, 200])
def test_compiled_rows_in_stages_fp64(mm, n):
    """Dormand-Prince attempts (stage kernels with the next forward x pass, the
    error pass) on rows of compiled and other lengths, in the default launch shape
    and with one to four cells a thread: every trajectory against the oracle's."""
    mesh = (n, 6, 1, 2e-9, 2e-9, 2e-9)
    gp, op = gpu_params(mm, PAR, F.ALL_TERMS), oracle_params(PAR, F.ALL_TERMS)
    kern = F.DemagKernel(F.Mesh(*mesh))
    m0 = [_m(mesh, 70 + i) for i in range(2)]
    mo = [dp45.run(lambda y: F.llg_rhs(y, F.Mesh(*mesh), op, kern), m, dp45.State(h=1e-14, h_max=1e-14), t_end=3e-14)
          for m in m0]
    for nt, ty in ((None, None), (64, 1), (128, 2), (256, 4)):
        plan = mm.Plan(mesh, "f64", terms=F.ALL_TERMS, max_batch=2)
        if ty:
            try:
                plan.set_shapes(dict(ty_x=ty, nt_i=nt))
            except mm.MMError:
                continue
        md = to_dev(np.stack(m0), torch.float64)
        st = mm.new_states(2, h=1e-14, h_max=1e-14)
        plan.rk45_run([gp, gp], md, st, t_end=3e-14)
        assert np.max(np.abs(md.cpu().numpy() - np.stack(mo))) <= 1e-9


@pytest.mark.parametrize("nz", [17, 18, 19, 24])
def test_lane_pair_z_of_36_and_48_points(mm, nz):
    """The FP32 lane-pair z transforms of 36 and 48 points (full and short
    columns) and FP64's pass through LDS at the same lengths."""
    for prec, tol in (("f32", 1e-5), ("f64", 1e-11)):
        mesh = (10, 9, nz, 3e-9, 2e-9, 2.5e-9)
        plan = mm.Plan(mesh, prec, terms=F.ALL_TERMS)
        assert plan.padded()[2] == (36 if nz < 19 else 48)
        gp, op = gpu_params(mm, PAR, F.ALL_TERMS), oracle_params(PAR, F.ALL_TERMS)
        m = representable(_m(mesh, 80 + nz), plan.dtype)
        H = plan.effective_field(gp, to_dev(m, plan.dtype)).double().cpu().numpy()
        assert field_err(H, F.effective_field(m, F.Mesh(*mesh), op, F.DemagKernel(F.Mesh(*mesh)))) <= tol


@pytest.mark.parametrize("n", [1, 2, 5])
@pytest.mark.parametrize("nx", [8, 256, 257])
def test_sd_step_inside_the_update_fp64(mm, nx, n):
    """Steepest descent of two instances whose update takes the step itself (one
    and 256 workgroups an instance) and of 257 workgroups, where a kernel of its
    own does: the state and the last step, after odd and even iterations."""
    mesh = (nx, 256, 1, 2e-9, 2e-9, 2e-9) if nx > 8 else (nx, 8, 1, 2e-9, 2e-9, 2e-9)
    plan = mm.Plan(mesh, "f64", terms=F.ALL_TERMS, max_batch=2)
    ps = [dict(PAR, alpha=0.5), dict(PAR, Ms=8e5, Ku=2e5, alpha=0.5)]
    rng = np.random.default_rng(90)
    m0 = np.array([0.0, 0.0, 1.0]).reshape(3, 1, 1, 1) + 0.3 * rng.normal(size=(2, 3, *mesh[2::-1]))
    m0 /= np.linalg.norm(m0, axis=1, keepdims=True)
    md = to_dev(m0, torch.float64)
    tau = plan.sd_run([gpu_params(mm, p, F.ALL_TERMS) for p in ps], md, n, 1e-7, 1e-10, 1e-3)
    kern = F.DemagKernel(F.Mesh(*mesh))
    for b, p in enumerate(ps):
        op = oracle_params(p, F.ALL_TERMS)
        mo, taus = sd.run(lambda y: F.effective_field(y, F.Mesh(*mesh), op, kern), m0[b].copy(), n, 1e-7, 1e-10, 1e-3)
        assert np.max(np.linalg.norm(md[b].cpu().numpy() - mo, axis=0)) <= 1e-9
        assert abs(tau[b] - taus[-1]) <= 1e-9 * taus[-1]


@pytest.mark.parametrize("prec,tol", [("f32", 1e-5), ("f64", 1e-11)])
@pytest.mark.parametrize("L", [1152, 1296, 1458, 1536, 1728, 1944])
def test_compiled_columns_beyond_1024(mm, L, prec, tol):
    """Fields of films and two-plane meshes whose y columns take the longer
    compiled transforms, full (2 ny = L) and short (3-D columns of 1944 points
    are refused)."""
    for mesh in ((6, L // 2, 1), (5, L // 2 - 2, 1), (4, L // 2, 2), (9, L // 2 - 1, 3)):
        mesh = mesh + (2e-9, 3e-9, 2.5e-9)
        if L == 1944 and mesh[2] > 1:
            with pytest.raises(mm.MMError):
                mm.Plan(mesh, prec, terms=F.ALL_TERMS)
            continue
        plan = mm.Plan(mesh, prec, terms=F.ALL_TERMS)
        assert plan.padded()[1] == L
        gp, op = gpu_params(mm, PAR, F.ALL_TERMS), oracle_params(PAR, F.ALL_TERMS)
        m = representable(_m(mesh, L), plan.dtype)
        H = plan.effective_field(gp, to_dev(m, plan.dtype)).double().cpu().numpy()
        assert field_err(H, F.effective_field(m, F.Mesh(*mesh), op, F.DemagKernel(F.Mesh(*mesh)))) <= tol


def test_long_columns_in_a_batch_fp64(mm):
    """A batch of two long column lengths (films and separate passes) and a short
    one: each trajectory against the oracle's."""
    meshes = [(8, 600, 1, 2e-9, 2e-9, 2e-9), (6, 648, 2, 2e-9, 2e-9, 2e-9), (6, 760, 1, 2e-9, 2e-9, 2e-9),
              (10, 64, 1, 2e-9, 2e-9, 2e-9)]
    batch = mm.Batch(meshes, "f64")
    gp, op = gpu_params(mm, PAR, F.ALL_TERMS), oracle_params(PAR, F.ALL_TERMS)
    which = [0, 1, 2, 3, 0]
    m0 = [_m(meshes[k], 95 + i) for i, k in enumerate(which)]
    md = [to_dev(m, torch.float64) for m in m0]
    t_end = 4e-14
    batch.run([dict(mesh_id=k, params=gp, m=md[i], t_end=t_end, state=mm.new_states(1, h=2e-14, h_max=2e-14)[0])
               for i, k in enumerate(which)])
    for i, k in enumerate(which):
        mesh = F.Mesh(*meshes[k])
        kern = F.DemagKernel(mesh)
        mo = dp45.run(lambda y: F.llg_rhs(y, mesh, op, kern), m0[i], dp45.State(h=2e-14, h_max=2e-14), t_end=t_end)
        assert np.max(np.abs(md[i].cpu().numpy() - mo)) <= 1e-9


@pytest.mark.parametrize("prec,tol", [("f32", 1e-5), ("f64", 1e-11)])
@pytest.mark.parametrize("nx,rows", [(128, 1), (127, 4), (256, 2), (512, 4), (512, 1), (509, 2), (1024, 2)])
def test_potential_rows(mm, nx, rows, prec, tol):
    """The scalar-potential route's inverse x of the compiled rows at the rows a
    workgroup of the launch shape, which long rows take at most two of outside
    the integrators, with a short last tile: field and dm/dt, and two attempts in
    FP64 (the Runge-Kutta epilogues keep the shape's rows)."""
    mesh = (nx, 9, 2, 3e-9, 2e-9, 2.5e-9)
    local = F.EXCHANGE | F.DMI | F.ANIS | F.ZEEMAN
    plan = mm.Plan(mesh, prec, terms=local | mm.DEMAG_POTENTIAL)
    try:
        plan.set_shapes(dict(ty_x=rows, nt_i=512, ty_f=1))
    except mm.MMError:
        pytest.skip("four FP64 rows of 512 points exceed LDS")
    gp, op = gpu_params(mm, PAR, local | mm.DEMAG_POTENTIAL), oracle_params(PAR, local | F.DEMAG)
    m = representable(_m(mesh, 97), plan.dtype)
    kern = potential.PotentialKernel(F.Mesh(*mesh), P=tuple(plan.padded()[::-1]))
    field = lambda y: potential.effective_field(y, F.Mesh(*mesh), op, kern)
    md = to_dev(m, plan.dtype)
    Href = field(m)
    assert field_err(plan.effective_field(gp, md).double().cpu().numpy(), Href) <= tol
    k = F.llg_rhs_from_field(m, Href, op)
    assert field_err(plan.llg_rhs(gp, md).double().cpu().numpy(), k) <= tol
    if prec == "f64":
        st, ost, mo = mm.new_states(1, h=2e-14), dp45.State(h=2e-14), m
        for _ in range(2):
            plan.rk45_step([gp], md, st)
            mo, acc = dp45.step(lambda y: F.llg_rhs_from_field(y, field(y), op), mo, ost)
            assert bool(st[0].last_accepted) == acc
        assert field_err(md.cpu().numpy(), mo) <= 1e-10


@pytest.mark.parametrize("prec,tol", [("f32", 1e-5), ("f64", 1e-10)])
@pytest.mark.parametrize("nx,rows", [(127, 4), (256, 8), (512, 1), (512, 2), (512, 4), (509, 4), (1024, 2)])
def test_potential_energy_rows(mm, nx, rows, prec, tol):
    """Energies of two instances on the scalar-potential route at the rows a
    workgroup of the launch shape, long rows in fours among them (one partial sum
    a workgroup, counted by the shape where they are summed), with a short last
    tile: each instance against the oracle, to the field's bar of the sum of its
    terms, and the same again after a field of the same plan (in twos)."""
    mesh = (nx, 9, 2, 3e-9, 2e-9, 2.5e-9)
    local = F.EXCHANGE | F.DMI | F.ANIS | F.ZEEMAN
    plan = mm.Plan(mesh, prec, terms=local | mm.DEMAG_POTENTIAL, max_batch=2)
    plan.set_shapes(dict(ty_x=rows, nt_i=512, ty_f=1))
    gp, op = gpu_params(mm, PAR, local | mm.DEMAG_POTENTIAL), oracle_params(PAR, local | F.DEMAG)
    m = [representable(_m(mesh, s), plan.dtype) for s in (98, 99)]
    kern = potential.PotentialKernel(F.Mesh(*mesh), P=tuple(plan.padded()[::-1]))
    md = to_dev(np.stack(m), plan.dtype)
    E = plan.energy([gp, gp], md)
    for b in range(2):
        Eref = potential.energies(m[b], F.Mesh(*mesh), op, kern)
        assert np.all(np.abs(E[b] - Eref) <= tol * np.sum(np.abs(Eref))), (E[b], Eref)
    plan.effective_field([gp, gp], md)
    assert np.array_equal(plan.energy([gp, gp], md), E)


def test_potential_energy_default_rows_fp32(mm):
    """A slab whose default shape takes four rows a workgroup: the demag energy of
    two instances against the FP64 sum over the cells of m . H from the field call
    (H to 1e-5 of its largest value), and no other term."""
    mesh = (512, 256, 16, 5e-9, 5e-9, 5e-9)
    plan = mm.Plan(mesh, "f32", terms=mm.DEMAG_POTENTIAL, max_batch=2)
    assert plan.shapes()["ty_x"] == 4
    gp = gpu_params(mm, PAR, mm.DEMAG_POTENTIAL)
    md = to_dev(np.stack([_m(mesh, s) + np.array([0.0, 0.0, w]).reshape(3, 1, 1, 1) for s, w in ((1, 2.0), (2, -1.0))]),
                plan.dtype)
    md /= md.norm(dim=1, keepdim=True)
    E = plan.energy([gp, gp], md)
    H = plan.effective_field([gp, gp], md)
    V = mesh[3] * mesh[4] * mesh[5]
    c = -0.5 * 4e-7 * np.pi * PAR["Ms"] * V
    for b in range(2):
        mh = md[b].double() * H[b].double()
        ref = c * float(mh.sum())
        bar = 1e-5 * abs(c) * float(H[b].double().norm(dim=0).max()) * md[b, 0].numel()
        assert abs(E[b][1] - ref) <= bar and abs(ref) > 100 * bar
        assert np.all(E[b][[0, 2, 3, 4]] == 0.0)


@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_mixed_batch_has_the_bits_of_each_mesh_alone(mm, prec):
    """A batch whose launch has 512 threads, so that rows of a power of two take the
    compiled inverse x with four rows a workgroup beside a length with threes:
    three steps of every instance bit for bit those of a plan of its mesh."""
    meshes = [(256, 256, 1, 2e-9, 2e-9, 2e-9), (96, 96, 1, 2e-9, 2e-9, 2e-9), (128, 64, 2, 2e-9, 2e-9, 2e-9)]
    batch = mm.Batch(meshes, prec)
    gp = gpu_params(mm, PAR, F.ALL_TERMS)
    plans = [mm.Plan(m, prec, terms=F.ALL_TERMS) for m in meshes]
    which = [i % 3 for i in range(48)]
    m0 = [to_dev(_m(meshes[k], 200 + i), plans[k].dtype) for i, k in enumerate(which)]
    md = [m.clone() for m in m0]
    state = lambda: mm.new_states(1, h=1e-14, h_max=1e-14)
    batch.run([dict(mesh_id=k, params=gp, m=md[i], t_end=3e-14, state=state()[0]) for i, k in enumerate(which)])
    for i in (0, 1, 2, 45, 46, 47):
        plans[which[i]].rk45_run(gp, m0[i], state(), t_end=3e-14)
        assert torch.equal(m0[i], md[i]), i


def test_long_runs_follow_the_material_form_fp64(mm):
    """Two runs of 99 steps (graphs of eight attempts) on one plan and one array, the
    first with cell material and torques, the second uniform, and the other way
    round: the second has the bits of a fresh plan's."""
    mesh = (32, 24, 3, 3e-9, 2.5e-9, 2e-9)
    general = F.ALL_TERMS | mm.CELLS | mm.STT_SOT
    cells = lambda v: np.full(mesh[2::-1], v)

    def plan():
        p = mm.Plan(mesh, "f64", terms=general)
        p.set_cells(0, cells(6e5), cells(1.3e-11), cells(1e-3))
        return p

    run = lambda p, q, m: p.rk45_run(q, m, mm.new_states(1, h=2e-15, h_max=2e-15), t_end=99 * 2e-15)
    m0 = to_dev(_m(mesh, 7), torch.float64)
    qs = [mm.make_params(terms=general, a_J=5e7, p=(0, 1, 0), **PAR), mm.make_params(terms=F.ALL_TERMS, **PAR)]
    for first, second in (qs, qs[::-1]):
        p, m, ref = plan(), m0.clone(), m0.clone()
        run(p, first, m)
        m.copy_(m0)
        run(p, second, m)
        run(plan(), second, ref)
        assert torch.equal(m, ref)
