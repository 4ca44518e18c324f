"""The spawn check with the robot's culling against the test of every (robot
sphere, target) pair: the same answer for every scene, at robot placements
from deep inside the furniture to far outside the room, with furniture staged
in LDS or not, and with contact lists too short for the hits."""
import numpy as np
import pytest

import scenegen as sg

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cfg,scenes", [(1, 3), (2, 70), (3, 65)])
@pytest.mark.parametrize("spread", [0.05, 0.5, 8.0])
@pytest.mark.parametrize("rcap", [None, 1])
def test_spawn_check_culled_equals_every_pair(cfg, scenes, spread, rcap):
    import paper_2412_13211_amd as ms
    b = sg.make(cfg, scenes)
    if rcap is not None:
        b.robot_contact_cap = rcap
    rng = np.random.default_rng(cfg)
    x = b.state0.copy()
    st = sg.split_state(x, b.n_scenes, b.n_free, b.n_aux)
    st["q"][:, 0:2] += rng.normal(0, spread, (scenes, 2))
    st["q"][:, 2] += rng.normal(0, 1.0, scenes)
    st["q"][:, 3:13] += rng.normal(0, 0.2, (scenes, 10))
    xg = torch.as_tensor(x.astype(np.float32)).cuda()
    got = {}
    for stage in (0, ms.MS_SCHED_STAGE_STATIC):
        for cull in (0, ms.MS_SCHED_CULL):
            mb = ms.MsBatch(b)
            mb.set_schedule(stage | cull)
            got[stage, cull] = mb.spawn_check(xg).cpu().numpy()
    want = got[0, 0]
    for k, v in got.items():
        assert np.array_equal(v, want), k


def _odd(kind, b, st, rng):
    """Scenes whose bounding volumes do not cover what the pair test accepts."""
    if kind == "plane":        # normals of length 3: the pair test's gap is three times the distance
        b.plane[:] *= 3.0
    elif kind == "quat":       # quaternions of norm 0.6: boxes larger than their half extents
        st["free"][:, 4:8] *= 0.6
    elif kind == "door":
        b.aux_rot[:] *= 0.6
    elif kind == "far":        # an ulp there is 4 mm
        at = np.float32(40000.0)
        b.static_box[:, 0] += at
        st["free"][:, 0] += at
        st["q"][:, 0] += at
        b.aux_pos[:, 0] += at
        b.plane[:, 3] += b.plane[:, 0] * at
    elif kind == "long":       # beams: half extents past the levers the bounds take
        b.free_size[:, 0] = np.where(b.free_type == sg.FREE_BOX, 40.0, b.free_size[:, 0])
        st["free"][:, 2] += 0.5


@pytest.mark.parametrize("kind", ["plain", "plane", "quat", "door", "far", "long"])
def test_spawn_check_holds_where_bounds_do_not(kind):
    """Plane normals that are not unit vectors, quaternions that are not, distant
    scenes and long bodies: culled or not, the check answers as the test of every
    pair; and robots that collide and robots that do not both occur."""
    import paper_2412_13211_amd as ms
    hits = scenes = 0
    for seed in range(4):
        b = sg.make(5, 96, seed=seed)
        rng = np.random.default_rng(seed)
        st = sg.split_state(b.state0.copy(), b.n_scenes, b.n_free, b.n_aux)
        st["q"][:, 0:2] += rng.normal(0, 1.5, (b.n_scenes, 2))
        st["q"][:, 3:13] += rng.normal(0, 0.2, (b.n_scenes, 10))
        _odd(kind, b, st, rng)
        x = torch.as_tensor(sg.join_state(st["q"], st["qd"], st["free"], st["aux"]).astype(np.float32)).cuda()
        got = {}
        for stage in (0, ms.MS_SCHED_STAGE_STATIC):
            for cull in (0, ms.MS_SCHED_CULL):
                mb = ms.MsBatch(b)
                mb.set_schedule(stage | cull)
                got[stage, cull] = mb.spawn_check(x).cpu().numpy()
        want = got[0, 0]
        for k, v in got.items():
            assert np.array_equal(v, want), (seed, k, np.flatnonzero(v != want))
        hits += int(want.sum())
        scenes += want.size
    print(f"[spawn] {kind}: {hits} of {scenes} collide", flush=True)
    assert 0 < hits < scenes
