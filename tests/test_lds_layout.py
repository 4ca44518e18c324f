"""What fits a workgroup's LDS block.  The step's two wavefronts keep culling
masks, dynamics scratch and the contact list side by side; a block that would
not hold them shares the space as one wavefront's phases in turn did, so every
scene and contact cap that fitted that way fits."""
import ctypes as C
import dataclasses

import numpy as np
import pytest

import paper_2412_13211_amd as ms
import scenegen as sg

LDS = 163840  # bytes of a workgroup


def one_wavefront_block(bodies, boxes, cap, robot_cap, spheres, staged=True, force=False):
    """Bytes of a scene's block with all phases in turn in one wavefront."""
    up4 = lambda n: (n + 3) // 4 * 4
    targets = 8 + boxes + 4 + bodies                       # planes, boxes, joints, bodies
    chunks = -(-targets // 64)
    n = up4(5 * 16 + 16 * 9 + 16 * 3 + 16 * 6 + 16 * 16)   # the robot
    n += 4 * spheres + up4(37 * (bodies + 1)) + 4 * 32     # spheres, bodies, joints
    n += up4(6 * boxes) if staged else 0
    n += 8 * 4 + up4((8 * bodies + 1) // 2)                # planes, owners
    masks = up4(max(bodies, 16) * chunks * 2) + max(bodies, 16) * 4
    dynamics = 16 * 11 + 2 * 16 * 6 + 16 * 16 + 16 + 16 * 17
    n += max(up4(17 * cap) + max(48 * robot_cap, masks), dynamics)  # contacts, robot rows
    n += up4((6 * cap + 5 + 1) // 2)                       # schedule
    n += up4(max(targets, (5 + bodies) * -(-cap // 64) * 2))
    n += up4(5 * bodies) if force else 0
    return 4 * n


def furnished(b, boxes):
    """The batch with `boxes` furniture boxes in every scene: its own and small
    ones overhead."""
    off, out = [0], []
    for s in range(b.n_scenes):
        own = b.static_box[b.static_off[s]:b.static_off[s + 1]][:boxes]
        k = np.arange(boxes - len(own))
        more = np.zeros((len(k), 6), np.float32)
        more[:, 0], more[:, 1], more[:, 2] = 0.1 * (k % 64) - 3.2, 0.1 * (k // 64 % 64) - 3.2, 4.0 + 0.1 * (k // 4096)
        more[:, 3:] = 0.02
        out += [own, more]
        off.append(off[-1] + boxes)
    return dataclasses.replace(b, static_off=np.array(off, np.int32), static_box=np.concatenate(out))


def _block(b, bodies, boxes, cap, robot_cap):
    """ms_query_sizes of one scene of the batch with these sizes (furniture staged)."""
    scene = dataclasses.replace(
        b, n_scenes=1, free_off=np.array([0, bodies], np.int32), free_type=np.zeros(bodies, np.int32),
        free_size=np.full((bodies, 3), 0.1, np.float32), free_mass=np.ones(bodies, np.float32),
        free_inertia=np.ones((bodies, 3), np.float32), static_off=np.array([0, boxes], np.int32),
        static_box=np.ones((boxes, 6), np.float32))
    d = ms.make_desc(scene, contact_cap=cap, robot_contact_cap=robot_cap)
    sd, keep = ms.make_scene_desc(scene)
    sz = ms.Sizes()
    assert ms.lib().ms_query_sizes(C.byref(d), C.byref(sd), C.byref(sz)) == 0
    return sz.lds


def _batch():
    b = sg.make(2, 1)
    assert b.n_aux == 0
    return b


@pytest.mark.parametrize("bodies,boxes,cap", [(17, 4000, 400), (17, 4504, 256), (32, 4144, 256), (58, 3616, 256),
                                              (8, 60, 1858), (1, 0, 1915), (40, 4300, 123)])
def test_blocks_that_fitted_still_fit(bodies, boxes, cap):
    b = _batch()
    n = one_wavefront_block(bodies, boxes, cap, min(24, cap), int(b.model_nsph.max()))
    assert n <= LDS
    assert _block(b, bodies, boxes, cap, min(24, cap)) <= LDS


def test_blocks_over_the_range():
    """Random sizes near the limit: the largest cap of one wavefront fits."""
    b = _batch()
    spheres = int(b.model_nsph.max())
    rng = np.random.default_rng(0)
    tried = 0
    while tried < 400:
        bodies, boxes = int(rng.integers(1, 59)), int(rng.integers(0, 6000))
        share = rng.uniform(0, 1)
        fits = lambda cap: one_wavefront_block(bodies, boxes, cap, max(int(share * cap), 1), spheres) <= LDS
        if not fits(1):
            continue
        lo, hi = 1, 4096
        while lo < hi:
            mid = (lo + hi + 1) // 2
            lo, hi = (mid, hi) if fits(mid) else (lo, mid - 1)
        assert _block(b, bodies, boxes, lo, max(int(share * lo), 1)) <= LDS, (bodies, boxes, lo, share)
        tried += 1


@pytest.mark.parametrize("cfg,tape", [(1, 6879744), (2, 8242176), (3, 16018944), (5, 8605696)])
def test_tape_holds_no_more_than_the_lane_adjoint_needs(cfg, tape):
    """The tape buffer of 70 scenes, a lane of the reference adjoint each (in
    wavefronts of 64): its contact adjoint record takes 16 floats."""
    b = sg.make(cfg, 70)
    d = ms.make_desc(b)
    sd, keep = ms.make_scene_desc(b)
    sz = ms.Sizes()
    assert ms.lib().ms_query_sizes(C.byref(d), C.byref(sd), C.byref(sz)) == 0
    assert sz.tape <= tape


@pytest.mark.gpu
@pytest.mark.parametrize("boxes,staged", [(600, True), (4000, True), (9000, False), (22000, False)])
@pytest.mark.parametrize("force", [False, True])
def test_steps_at_the_largest_cap_with_many_boxes(boxes, staged, force):
    """Bit for bit the step under a small cap, for robots among furniture, doors,
    drawers and objects, with a record or with force outputs."""
    torch = pytest.importorskip("torch")
    from test_gpu_sweeps import _crowded
    b = furnished(_crowded(0.1), boxes)
    bodies, spheres, rcap = int(np.diff(b.free_off).max()), int(b.model_nsph.max()), 24
    cap = max(c for c in range(1, 2100)
              if one_wavefront_block(bodies, boxes, c, min(rcap, c), spheres, staged, force) <= LDS)
    x0, u = torch.as_tensor(b.state0).cuda(), torch.as_tensor(b.controls(0)).cuda()
    got = []
    for c, stage in ((40, 0), (cap, ms.MS_SCHED_STAGE_STATIC if staged else 0)):
        mb = ms.MsBatch(b, contact_cap=c, robot_contact_cap=min(rcap, c))
        mb.set_schedule(ms.MS_SCHED_CULL | stage)
        mb.enable_debug(True)
        out = list(mb.enable_forces()) if force else []
        x, robot = x0, []
        for _ in range(3):
            x = mb.step(x, u)
            torch.cuda.synchronize()
            assert not np.any(mb.status())
            robot.append(int(mb.debug_contacts()[..., 1].max()))
        assert max(robot) > 8, robot
        if not force:
            out.append(mb.step_record(x, u, mb.new_record()))
        got.append([v.cpu().numpy() for v in [x] + out])
    print(f"[lds] {boxes} boxes, {'staged' if staged else 'in memory'}: {cap} contacts", flush=True)
    assert not force or np.any(got[0][2])
    for p, q in zip(*got):
        assert np.array_equal(p.view(np.uint32), q.view(np.uint32))
