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
