"""The Gauss-Seidel sweeps' special cases: robot rows with and without room
for their data beside the contact list (and more of them than lanes), and more
groups of free-body rows than lanes.

The room for a robot row's data depends on the contact caps, the arithmetic
does not, so a step under generous caps and one under caps that just fit the
scenes' contacts agree bit for bit.
"""
import numpy as np
import pytest

import oracle
import scenegen as sg
from _grad import GRAD_TOL, compare, oracle_vjp_smooth, scene_vectors
from _parity import errors, fp32_sensitivity, same_contacts

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _ms():
    import paper_2412_13211_amd as ms
    return ms


def _crowded(depth, n=6, seed=3):
    """Robots standing `depth` of the way into furniture, beside doors,
    drawers and objects."""
    b = sg.make(5, n, seed=seed)
    st = sg.split_state(b.state0, n, b.n_free, b.n_aux)
    for s in range(n):
        box = b.static_box[b.static_off[s] + s]
        st["q"][s, 0:2] += depth * (box[0:2] - st["q"][s, 0:2])
        # an object against the robot's base
        f = b.free_off[s]
        st["free"][f, 0:2] = st["q"][s, 0:2] + 0.35
    b.state0[:] = sg.join_state(st["q"], st["qd"], st["free"], st["aux"])
    return b


def _run(ms, b, ccap, rcap):
    mb = ms.MsBatch(b, contact_cap=ccap, robot_contact_cap=rcap)
    mb.enable_debug(True)
    rf, bf = mb.enable_forces()
    x = torch.as_tensor(b.state0).cuda()
    u = torch.as_tensor(b.controls(0)).cuda()
    out = mb.step(x, u)
    torch.cuda.synchronize()
    d = mb.debug_contacts()
    return out.cpu().numpy(), rf.cpu().numpy(), bf.cpu().numpy(), d, mb.status()


@pytest.mark.parametrize("depth", [0.0, 0.15, 0.25, 0.35])
def test_robot_rows_independent_of_their_room(depth):
    ms = _ms()
    b = _crowded(depth)
    wide = _run(ms, b, 640, 300)
    nc, nr = int(wide[3][..., 0].max()), int(wide[3][..., 1].max())
    print(f"[robot rows] depth {depth}: up to {nc} contacts, {nr} of the robot", flush=True)
    assert not np.any(wide[4] & (ms.MS_ST_OVERFLOW | ms.MS_ST_ROBOT_OVERFLOW))
    # joint-limit rows share the contact cap
    tight = _run(ms, b, nc + 4, max(nr, 1))
    assert not np.any(tight[4] & (ms.MS_ST_OVERFLOW | ms.MS_ST_ROBOT_OVERFLOW))
    for a, c in zip(wide[:3], tight[:3]):
        assert np.array_equal(a.view(np.uint32), c.view(np.uint32))


def _sphere_floor(pgs_iters=10, n_sub=4):
    """58 spheres on the floor in touching rows: 58 floor groups and 54 pairs."""
    rng = np.random.default_rng(5)
    objs = []
    for i in range(58):
        r = 0.05
        row, col = divmod(i, 15)
        objs.append(sg.sphere_object(r, float(rng.uniform(0.1, 1.0)),
                                     (col * (2 * r + 1e-3), row * 0.3, r + float(rng.uniform(-2e-4, 2e-4))),
                                     vel=tuple(rng.normal(0, 0.05, 3)), angvel=tuple(rng.normal(0, 0.2, 3))))
    return sg.custom_batch([sg.empty_model()], [dict(free=objs, planes=[(0.0, 0.0, 1.0, 0.0)])], h=0.002,
                           n_sub=n_sub, pgs_iters=pgs_iters, contact_cap=160)


def test_more_groups_than_lanes():
    ms = _ms()
    b = _sphere_floor()
    o = oracle.Oracle(b)
    x = b.state0.astype(np.float64)
    u = np.zeros((1, 16))
    mb = ms.MsBatch(b)
    mb.enable_debug(True)
    xg = mb.step(torch.as_tensor(b.state0).cuda(), torch.zeros((1, 16), device="cuda")).cpu().numpy()
    xo, d = o.step(x, u, debug=True)
    assert d["n_contacts"].min() > 64
    assert same_contacts(d, mb.debug_contacts()).all()
    pe, ve = errors(o, b, xo, xg.astype(np.float64))
    ps, vs = fp32_sensitivity(o, b, x, u)
    pf, vf = errors(o, b, xo, o.step_f32(x, u))
    # the repository's one-step parity bars
    assert pe.max() <= max(1e-5, 10 * ps.max(), 4 * pf.max()), pe
    assert ve.max() <= max(1e-4, 10 * vs.max(), 4 * vf.max()), ve


def _vjp(mb, b, g):
    x = torch.as_tensor(b.state0).cuda()
    u = torch.as_tensor(np.ascontiguousarray(b.controls(0))).cuda()
    gx, gu = mb.step_backward(x, u, torch.as_tensor(g.astype(np.float32)).cuda())
    torch.cuda.synchronize()
    return gx.cpu().numpy().astype(np.float64), gu.cpu().numpy().astype(np.float64)


def _check_gradient(ms, b, **caps):
    """The wavefront adjoint against the oracle's, on its smooth components
    (the repository's gradient bar), and twice the same bit for bit."""
    o = oracle.Oracle(b)
    x = b.state0.astype(np.float64)
    u = np.asarray(b.controls(0), np.float64)
    g = np.random.default_rng(2).normal(size=x.size)
    ref, mask, scale = oracle_vjp_smooth(o, b, x, u, g)
    mb = ms.MsBatch(b, backward=True, **caps)
    first = _vjp(mb, b, g)
    second = _vjp(mb, b, g)
    assert all(np.array_equal(p, q) for p, q in zip(first, second))
    err = compare(ref, mask, scale, scene_vectors(b, *first))
    print(f"[gradient] {b.name}: rel err {np.array2string(err, precision=2)}, smooth "
          f"{np.mean([m.mean() for m in mask]):.2f}", flush=True)
    assert np.all(err <= GRAD_TOL), err


@pytest.mark.parametrize("iters", [1, 2, 10])
def test_gradient_more_groups_than_lanes(iters):
    _check_gradient(_ms(), _sphere_floor(pgs_iters=iters, n_sub=2))


@pytest.mark.parametrize("depth", [0.0, 0.1])
def test_gradient_robot_rows(depth):
    """Robot contacts with furniture, doors, drawers and objects."""
    b = _crowded(depth)
    st = sg.split_state(b.state0, b.n_scenes, b.n_free, b.n_aux)
    rng = np.random.default_rng(4)
    st["qd"][:, :15] = rng.normal(0.0, 0.1, st["qd"][:, :15].shape)
    st["free"][:, 2] -= rng.uniform(0.0, 2e-4, b.n_free)
    st["free"][:, 8:11] = rng.normal(0.0, 0.02, (b.n_free, 3))
    st["free"][:, 12:15] = rng.normal(0.0, 0.05, (b.n_free, 3))
    st["aux"][:, 0] += rng.uniform(1e-4, 1e-3, b.n_aux)
    b.state0[:] = sg.join_state(st["q"], st["qd"], st["free"], st["aux"])
    _check_gradient(_ms(), b)


@pytest.mark.parametrize("cfg,n", [(1, 2), (2, 3), (5, 5)])
def test_large_batches_step_like_small_ones(cfg, n):
    """Batches past the line of the instantiation with more scenes per CU: the
    same scenes many times over give bit for bit the small batch's results."""
    ms = _ms()
    small = sg.make(cfg, n)
    reps = (12 * torch.cuda.get_device_properties(0).multi_processor_count) // n + 1
    rows = np.tile(np.arange(n), reps)
    b = _repeat(small, rows)
    out = {}
    for name, batch in (("small", small), ("large", b)):
        mb = ms.MsBatch(batch)
        mb.set_schedule(ms.MS_SCHED_PERSISTENT | ms.MS_SCHED_CULL | ms.MS_SCHED_STAGE_STATIC)
        x = torch.as_tensor(batch.state0).cuda()
        u = torch.as_tensor(np.ascontiguousarray(small.controls(0)[rows] if name == "large" else small.controls(0))).cuda()
        y = mb.step(mb.step(x, u), u).cpu().numpy()
        out[name] = sg.split_state(y, batch.n_scenes, batch.n_free, batch.n_aux)
    nf, na = small.n_free, small.n_aux
    want = out["small"]
    got = out["large"]
    for k in ("q", "qd", "free", "aux"):
        w = np.ascontiguousarray(np.concatenate([want[k]] * reps)).view(np.uint32)
        assert np.array_equal(np.ascontiguousarray(got[k]).view(np.uint32), w), k


def _repeat(b, rows):
    """The scenes `rows` of a batch, one after the other."""
    import dataclasses

    def gather(off):
        off = np.asarray(off, np.int64)
        n = off[rows + 1] - off[rows]
        new = np.zeros(len(rows) + 1, np.int64)
        np.cumsum(n, out=new[1:])
        return new.astype(np.int32), np.repeat(off[rows] - new[:-1], n) + np.arange(new[-1])
    S = len(rows)
    st = sg.split_state(b.state0, b.n_scenes, b.n_free, b.n_aux)
    fo, fi = gather(b.free_off)
    so, si = gather(b.static_off)
    po, pi = gather(b.plane_off)
    ao, ai = gather(b.aux_off)
    kw = {k: getattr(b, k)[fi] for k in ("free_type", "free_size", "free_mass", "free_inertia")}
    kw.update({k: getattr(b, k)[ai] for k in ("aux_type", "aux_rot", "aux_pos", "aux_axis", "aux_box", "aux_mass",
                                              "aux_inertia", "aux_limit")})
    return dataclasses.replace(
        b, n_scenes=S, scene_model=b.scene_model[rows], scene_hold=b.scene_hold[rows], free_off=fo, static_off=so,
        plane_off=po, aux_off=ao, static_box=b.static_box[si], plane=b.plane[pi],
        state0=sg.join_state(st["q"][rows], st["qd"][rows], st["free"][fi], st["aux"][ai]), **kw)


@pytest.mark.parametrize("ccap,rcap", [(700, 24), (700, 200), (None, 1)])
def test_caps_past_the_adjoint_block(ccap, rcap):
    """Contact caps whose adjoint workspace is past the LDS block (None: the
    largest cap the forward step takes, where its dynamics scratch lies in the
    contact list's place): the same step and gradient bit for bit as with caps
    that fit."""
    ms = _ms()
    b = sg.make(2, 6)
    x = torch.as_tensor(b.state0).cuda()
    u = torch.as_tensor(b.controls(0)).cuda()
    g = torch.as_tensor(np.random.default_rng(3).normal(size=b.state0.size).astype(np.float32)).cuda()
    if ccap is None:
        for ccap in range(2100, 1500, -1):
            try:
                ms.MsBatch(b, contact_cap=ccap, robot_contact_cap=rcap).step(x, u)
                break
            except ms.MsError:
                pass
        print(f"[largest caps] {ccap} contacts, {rcap} of the robot", flush=True)
        assert ccap > 1800
    got = []
    for cc, rc in ((64, rcap if rcap < 24 else 24), (ccap, rcap)):
        mb = ms.MsBatch(b, contact_cap=cc, robot_contact_cap=rc, backward=True)
        y = mb.step(x, u)
        gx, gu = mb.step_backward(x, u, g)
        torch.cuda.synchronize()
        assert not np.any(mb.status())
        got.append([t.cpu().numpy() for t in (y, gx, gu)])
    for a, c in zip(*got):
        assert np.array_equal(a.view(np.uint32), c.view(np.uint32))


def test_force_outputs_at_the_largest_cap():
    """The contact-force step in an LDS block near the limit (dynamics before the
    contact list): states and forces as with a small cap, bit for bit, into the
    steps where the robots push bodies."""
    ms = _ms()
    b = sg.make(2, 32)
    got = []
    for cc in (64, *range(2100, 1900, -1)):
        x = torch.as_tensor(b.state0).cuda()
        try:
            mb = ms.MsBatch(b, contact_cap=cc, robot_contact_cap=16)
            fr, fb = mb.enable_forces()
            out = []
            for t in range(7):
                x = mb.step(x, torch.as_tensor(b.controls_for(t)).cuda())
                torch.cuda.synchronize()
                assert not np.any(mb.status())
                out.append([v.cpu().numpy() for v in (x, fr, fb)])
        except ms.MsError:
            continue
        got.append(out)
        if len(got) == 2:
            break
    print(f"[largest cap with forces] {cc}", flush=True)
    assert len(got) == 2 and np.any(got[0][-1][2])
    for step in zip(*got):
        for a, c in zip(*step):
            assert np.array_equal(a.view(np.uint32), c.view(np.uint32))


def _moving(depth, n=6):
    """_crowded with moving robots, objects, doors and drawers."""
    b = _crowded(depth, n)
    st = sg.split_state(b.state0, n, b.n_free, b.n_aux)
    rng = np.random.default_rng(4)
    st["qd"][:, :15] = rng.normal(0.0, 0.1, st["qd"][:, :15].shape)
    st["free"][:, 2] -= rng.uniform(0.0, 2e-4, b.n_free)
    st["free"][:, 8:11] = rng.normal(0.0, 0.02, (b.n_free, 3))
    st["free"][:, 12:15] = rng.normal(0.0, 0.05, (b.n_free, 3))
    st["aux"][:, 0] += rng.uniform(1e-4, 1e-3, b.n_aux)
    b.state0[:] = sg.join_state(st["q"], st["qd"], st["free"], st["aux"])
    return b


@pytest.mark.parametrize("depth,ccap,rcap", [(0.1, 658, 24), (0.1, 627, 32), (0.1, 376, 96), (0.1, 153, 153),
                                             (0.25, 282, 120)])
def test_reverse_from_a_record_without_a_tape_buffer(depth, ccap, rcap):
    """The largest contact caps whose adjoint block held one wavefront's arrays: a
    kept record is reversed without a tape buffer, bit for bit as with small
    caps."""
    ms = _ms()
    b = _moving(depth)
    x, u = torch.as_tensor(b.state0).cuda(), torch.as_tensor(b.controls(0)).cuda()
    g = torch.as_tensor(np.random.default_rng(3).normal(size=b.state0.size).astype(np.float32)).cuda()
    got = []
    for cc, rc in ((120, 80), (ccap, rcap)):
        mb = ms.MsBatch(b, contact_cap=cc, robot_contact_cap=rc)
        mb.enable_debug(True)
        mb.step(x, u)
        robot = mb.debug_contacts()[..., 1].max()
        assert (robot > 64) == (depth == 0.25) and robot >= 20
        rec = mb.new_record()
        y = mb.step_record(x, u, rec)
        gx, gu = mb.step_backward_recorded(x, u, rec, g)
        torch.cuda.synchronize()
        assert not np.any(mb.status() & (ms.MS_ST_OVERFLOW | ms.MS_ST_ROBOT_OVERFLOW | ms.MS_ST_NONFINITE))
        got.append([t.cpu().numpy() for t in (y, gx, gu)])
    for a, c in zip(*got):
        assert np.array_equal(a.view(np.uint32), c.view(np.uint32))


def _sphere_chains(counts, lone, pgs_iters=10, n_sub=2):
    """Per entry of `counts` a scene with a row of that many touching spheres on the
    floor (n floor groups, n - 1 pairs), and `lone` spheres apart."""
    scenes = []
    for s, n in enumerate(counts):
        rng = np.random.default_rng(s)
        at = [(i * 0.101, 0.0) for i in range(n)] + [(i * 0.3, 1.0) for i in range(lone)]
        scenes.append(dict(free=[sg.sphere_object(0.05, float(rng.uniform(0.1, 1.0)),
                                                  (x, y, 0.05 + float(rng.uniform(-2e-4, 2e-4))),
                                                  vel=tuple(rng.normal(0, 0.05, 3)), angvel=tuple(rng.normal(0, 0.2, 3)))
                                 for x, y in at], planes=[(0.0, 0.0, 1.0, 0.0)]))
    return sg.custom_batch([sg.empty_model()], scenes, h=0.002, n_sub=n_sub, pgs_iters=pgs_iters, contact_cap=160)


def _boxes(nx, ny, nz, seed=0):
    """Touching boxes on the floor, stacked: rows of a body broken by its neighbours'."""
    rng = np.random.default_rng(seed)
    out = []
    for k in range(nz):
        for j in range(ny):
            for i in range(nx):
                out.append(sg.box_object((0.05, 0.05, 0.05), 0.5, (i * 0.1001, j * 0.1001, 0.05 + 0.1 * k - float(rng.uniform(0, 2e-4))),
                                         vel=tuple(rng.normal(0, 0.02, 3)), angvel=tuple(rng.normal(0, 0.05, 3))))
    return dict(free=out, planes=[(0.0, 0.0, 1.0, 0.0)])


@pytest.mark.parametrize("counts,lone", [((31, 32, 33), 0), ((31, 32, 33), 1), ((32, 33, 34), 24), ((3, 57, 58), 0)])
def test_group_counts_about_the_lanes(counts, lone):
    """2 n - 1 + lone groups, about 64 and more: the repository's one-step parity bars."""
    ms = _ms()
    b = _sphere_chains(counts, lone)
    o = oracle.Oracle(b)
    x, u = b.state0.astype(np.float64), np.zeros((len(counts), 16))
    mb = ms.MsBatch(b)
    mb.enable_debug(True)
    xg = mb.step(torch.as_tensor(b.state0).cuda(), torch.as_tensor(u.astype(np.float32)).cuda()).cpu().numpy()
    xo, d = o.step(x, u, debug=True)
    assert d["n_contacts"][:, 0].tolist() == [2 * n - 1 + lone for n in counts]
    assert same_contacts(d, mb.debug_contacts()).all()
    pe, ve = errors(o, b, xo, xg.astype(np.float64))
    ps, vs = fp32_sensitivity(o, b, x, u)
    pf, vf = errors(o, b, xo, o.step_f32(x, u))
    assert pe.max() <= max(1e-5, 10 * ps.max(), 4 * pf.max()), pe
    assert ve.max() <= max(1e-4, 10 * vs.max(), 4 * vf.max()), ve


@pytest.mark.parametrize("what", ["boxes", "spheres"])
def test_forms_agree_on_many_groups(what):
    """Scenes with few and with hundreds of groups: the plain step, the one for
    large batches, the recording one and the ones for LDS blocks near the limit
    give the same bits."""
    ms = _ms()
    if what == "boxes":
        scenes, cap = [_boxes(1, 1, 2), _boxes(2, 2, 1), _boxes(1, 1, 12), _boxes(5, 5, 1), _boxes(3, 3, 2),
                       _boxes(4, 2, 3)], 720
        small = sg.custom_batch([sg.empty_model()], scenes, h=0.005, n_sub=2, pgs_iters=10, contact_cap=cap)
    else:
        small, cap = _sphere_chains((3, 28, 34), 2), 80
    n = small.n_scenes
    reps = (12 * torch.cuda.get_device_properties(0).multi_processor_count) // n + 1
    large = _repeat(small, np.tile(np.arange(n), reps))
    got = {}
    for name, b, c in (("plain", small, cap), ("large", large, cap), ("tight", small, 1500)):
        mb = ms.MsBatch(b, contact_cap=c, robot_contact_cap=1)
        if what == "spheres" and name == "large":
            assert 163840 // (mb.sizes.lds + 1024) > 6
        x = torch.as_tensor(b.state0).cuda()
        u = torch.zeros((b.n_scenes, 16), device="cuda")
        mb.enable_debug(name == "plain")
        y = mb.step(mb.step(x, u), u)
        torch.cuda.synchronize()
        assert not np.any(mb.status())
        if name == "plain":
            nc = mb.debug_contacts()[..., 0]
            assert nc.max() > 64 and nc.min() < 64
        z = mb.step_record(mb.step(x, u), u, mb.new_record()) if name != "large" else y
        for v in (y, z):
            st = sg.split_state(v.cpu().numpy(), b.n_scenes, b.n_free, b.n_aux)["free"]
            got.setdefault(name, []).append(np.ascontiguousarray(st).view(np.uint32))
    want = got["plain"][0]
    for name, vs in got.items():
        for v in vs:
            assert np.array_equal(v, np.concatenate([want] * reps) if name == "large" else want), name


@pytest.mark.parametrize("counts,lone", [((31, 32, 33), 1), ((32, 33), 24), ((57, 58), 0)])
def test_gradient_group_counts_about_the_lanes(counts, lone):
    _check_gradient(_ms(), _sphere_chains(counts, lone))


def _arm_beside(n, cap=160):
    """An arm leaning onto the floor and onto the first of n touching spheres."""
    rng = np.random.default_rng(7)
    q = np.zeros(16)
    q[:7] = rng.normal(0.0, 0.05, 7)
    q[1] = 1.8
    free = [sg.sphere_object(0.05, float(rng.uniform(0.1, 1.0)), (1.1, 0.101 * i, 0.05 + float(rng.uniform(-2e-4, 2e-4))),
                             vel=tuple(rng.normal(0, 0.05, 3)), angvel=tuple(rng.normal(0, 0.2, 3))) for i in range(n)]
    scene = dict(q=q, qd=np.concatenate([rng.normal(0.0, 0.2, 7), np.zeros(9)]), free=free,
                 planes=[(0.0, 0.0, 1.0, 0.0)])
    return sg.custom_batch([sg.arm7_model(np.random.default_rng(1))], [scene], h=0.002, n_sub=2, pgs_iters=10,
                           contact_cap=cap)


@pytest.mark.parametrize("n", [20, 40])
def test_gradient_many_groups_beside_a_robot(n):
    """Robot rows beside few and many groups: the gradient against the oracle's, and
    the same bits from the form for LDS blocks near the limit."""
    ms = _ms()
    b = _arm_beside(n)
    _check_gradient(ms, b)
    g = np.random.default_rng(2).normal(size=b.state0.size)
    robot, got = [], []
    for cap in (160, 570):
        mb = ms.MsBatch(b, contact_cap=cap, backward=True)
        mb.enable_debug(True)
        mb.step(torch.as_tensor(b.state0).cuda(), torch.zeros((1, 16), device="cuda"))
        robot.append(mb.debug_contacts()[..., 1].max())
        got.append(_vjp(mb, b, g))
    assert min(robot) > 0
    assert all(np.array_equal(p, q) for p, q in zip(*got))


def test_gradient_of_piles():
    """Hundreds of groups of boxes against the reference adjoint, which takes the
    rows one after the other, and the same bits from a small block and from one
    near the limit.  (The last pile, at rest on redundant contacts, has no gradient
    to compare: its sweeps sit on kinks, and float64 gives another one.)"""
    ms = _ms()
    scenes = [_boxes(1, 1, 2), _boxes(1, 1, 14), _boxes(4, 2, 1), _boxes(3, 2, 2)]
    b = sg.custom_batch([sg.empty_model()], scenes, h=0.005, n_sub=2, pgs_iters=10, contact_cap=360)
    g = np.random.default_rng(2).normal(size=b.state0.size)
    got = []
    for cap, flags in ((360, 0), (720, 0), (360, ms.MS_SCHED_BWD_REFERENCE)):
        mb = ms.MsBatch(b, contact_cap=cap, robot_contact_cap=1, backward=True)
        mb.set_schedule(ms.MS_SCHED_CULL | ms.MS_SCHED_STAGE_STATIC | flags)
        mb.enable_debug(True)
        mb.step(torch.as_tensor(b.state0).cuda(), torch.zeros((b.n_scenes, 16), device="cuda"))
        assert not np.any(mb.status()) and mb.debug_contacts()[..., 0].max() > 100
        got.append(_vjp(mb, b, g))
    assert all(np.array_equal(p, q) for p, q in zip(*got[:2]))
    mine, ref = (scene_vectors(b, *v) for v in (got[0], got[2]))
    err = [np.linalg.norm(p - q) / np.linalg.norm(q) for p, q in zip(mine[:3], ref)]
    print(f"[piles] rel err {np.array2string(np.array(err), precision=2)}", flush=True)
    assert max(err) <= GRAD_TOL, err


@pytest.mark.parametrize("kept", [False, True])
@pytest.mark.parametrize("depth,ccap,rcap", [(0.15, 900, 200), (0.25, 1200, 120)])
def test_caps_past_the_adjoint_block_in_a_mixed_batch(depth, ccap, rcap, kept):
    """Caps past the adjoint's LDS block, in a batch where some scenes' robot contacts
    fit the layout that runs in LDS (eight of them) and others' do not: those go to
    the lane kernel, from a kept record and from one it makes itself in the buffer
    that then is the lane kernel's workspace."""
    ms = _ms()
    few = _moving(depth)
    rows = np.tile(np.arange(6), 12)
    b = _repeat(few, rows)
    x = torch.as_tensor(b.state0).cuda()
    u = torch.as_tensor(np.ascontiguousarray(few.controls(0)[rows])).cuda()
    g = torch.as_tensor(np.random.default_rng(3).normal(size=b.state0.size).astype(np.float32)).cuda()

    def grads(cc, rc, flags=0):
        mb = ms.MsBatch(b, contact_cap=cc, robot_contact_cap=rc, backward=True)
        mb.set_schedule(ms.MS_SCHED_CULL | flags)
        mb.enable_debug(True)
        mb.step(x, u)
        robot = mb.debug_contacts()[..., 1].max(1)
        if kept and not flags:
            rec = mb.new_record()
            mb.step_record(x, u, rec)
            gx, gu = mb.step_backward_recorded(x, u, rec, g)
        else:
            gx, gu = mb.step_backward(x, u, g)
        torch.cuda.synchronize()
        assert not np.any(mb.status() & (ms.MS_ST_OVERFLOW | ms.MS_ST_ROBOT_OVERFLOW))
        return robot, scene_vectors(b, gx.cpu().numpy().astype(np.float64), gu.cpu().numpy().astype(np.float64))

    robot, mixed = grads(ccap, rcap)
    assert np.sum(robot > 8) >= 20 and np.sum((robot <= 8) & (robot > 0)) >= 10
    _, wave = grads(220, 100)      # every scene in LDS
    _, lane = grads(220, 100, ms.MS_SCHED_BWD_REFERENCE)
    for s in range(b.n_scenes):
        want = lane[s] if robot[s] > 8 else wave[s]
        assert np.array_equal(mixed[s], want), (s, robot[s])


@pytest.mark.parametrize("depth", [0.25, 0.35])
def test_robot_rows_past_the_lanes(depth):
    """More robot rows than lanes, with room for their data and without."""
    ms = _ms()
    b = _crowded(depth)
    wide = _run(ms, b, 640, 300)
    nc, nr = int(wide[3][..., 0].max()), int(wide[3][..., 1].max())
    assert nr > 64
    tight = _run(ms, b, nc + 4, nr)
    # the tight layout has room for the data of a few rows only: past the
    # contact list fewer floats than one block, past the Jacobian rows none
    # (their block is the larger one), and the spheres' centres
    assert 4 * 17 < 76 and 48 * nr > 1600 and 5 * int(b.model_nsph.max()) // 76 < 10
    assert not np.any(tight[4] & (ms.MS_ST_OVERFLOW | ms.MS_ST_ROBOT_OVERFLOW))
    for a, c in zip(wide[:3], tight[:3]):
        assert np.array_equal(a.view(np.uint32), c.view(np.uint32))


@pytest.mark.parametrize("depth,tight", [(0.1, False), (0.15, False), (0.15, True)])
def test_large_batches_with_robot_contacts_step_like_small_ones(depth, tight):
    """The instantiation with more scenes per CU on scenes whose robots push
    furniture, doors, drawers and objects, with room for the robot rows' data and
    without."""
    ms = _ms()
    small = _moving(depth)
    n = small.n_scenes
    u = small.controls(0)
    mb = ms.MsBatch(small)
    mb.enable_debug(True)
    x = torch.as_tensor(small.state0).cuda()
    for _ in range(2):
        x = mb.step(x, torch.as_tensor(u).cuda())
        torch.cuda.synchronize()
        assert not np.any(mb.status())
    want = sg.split_state(x.cpu().numpy(), n, small.n_free, small.n_aux)
    mb.step(torch.as_tensor(small.state0).cuda(), torch.as_tensor(u).cuda())
    d = mb.debug_contacts()
    nc, nr = int(d[..., 0].max()), int(d[..., 1].max())
    assert np.sum(d[..., 1].max(1) > 8) >= 2 and nr > (24 if depth > 0.1 else 16)
    caps = dict(contact_cap=nc + 8, robot_contact_cap=nr) if tight else {}
    reps = (12 * torch.cuda.get_device_properties(0).multi_processor_count) // n + 1
    rows = np.tile(np.arange(n), reps)
    large = _repeat(small, rows)
    for flags in (0, ms.MS_SCHED_PERSISTENT):
        mb = ms.MsBatch(large, **caps)
        assert 163840 // (mb.sizes.lds + 1024) > 6
        mb.set_schedule(flags | ms.MS_SCHED_CULL | ms.MS_SCHED_STAGE_STATIC)
        x, ul = torch.as_tensor(large.state0).cuda(), torch.as_tensor(np.ascontiguousarray(u[rows])).cuda()
        x = mb.step(mb.step(x, ul), ul)
        got = sg.split_state(x.cpu().numpy(), large.n_scenes, large.n_free, large.n_aux)
        assert not np.any(mb.status())
        for k in ("q", "qd", "free", "aux"):
            w = np.ascontiguousarray(np.concatenate([want[k]] * reps)).view(np.uint32)
            assert np.array_equal(np.ascontiguousarray(got[k]).view(np.uint32), w), k


def test_gradient_robot_rows_past_the_lanes():
    """More robot rows than lanes in reverse, against the oracle's gradient on its
    smooth components."""
    import dataclasses
    b = dataclasses.replace(_moving(0.25), contact_cap=120, robot_contact_cap=80)
    ms = _ms()
    mb = ms.MsBatch(b)
    mb.enable_debug(True)
    mb.step(torch.as_tensor(b.state0).cuda(), torch.as_tensor(b.controls(0)).cuda())
    assert mb.debug_contacts()[..., 1].max() > 64
    _check_gradient(ms, b)
