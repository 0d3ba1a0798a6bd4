"""The contact search's near map (one bit per cell: can a tip here touch a target at all)
against a search over every target in float64.

One straight step (no steering, no noise) puts each tip at a known place: most within 2% of a
contact sphere, spread over every direction, the rest anywhere, with targets on map-cell
boundaries, on walls and in corners.  The tips read back are compared, so only the FP32 distance
itself is uncertain: coordinates up to L carry at most L 2^-24 each, which moves a distance by at
most 4 L 2^-24, and the FP32 sums and products move it by at most R 2^-22.  A cone whose outcome
hangs on less than that is left out; at most a tenth may be."""
import numpy as np
import pytest

from paper_1405_3331_amd import binding as B
from paper_1405_3331_amd import scenarios as S

pytestmark = pytest.mark.gpu

CASES = [  # grid, contact radius, targets
    ((64, 48), 1.0, 40), ((64, 48), 0.01, 40), ((64, 48), 30.0, 3), ((2100, 30), 0.4, 500),
    ((333, 517), 2.5, 4096), ((24, 20, 18), 1.0, 60), ((24, 20, 18), 0.02, 60),
    ((24, 20, 18), 9.0, 4), ((300, 12, 9), 0.7, 400), ((130, 131, 70), 1.5, 4096),
]


@pytest.mark.parametrize("block", [1, 0])
@pytest.mark.parametrize("n,R,n_targets", CASES)
def test_contacts_against_every_target(n, R, n_targets, block):
    dim = len(n)
    if dim == 3 and block == 0:
        pytest.skip("a volume has one path")
    print(f"[gpu] {n} R={R} targets={n_targets} block={block}", flush=True)
    rng = np.random.default_rng(5)
    L = np.array(n, dtype=np.float64)
    sc = S.make_scenario("near map", dim, n, 1.0, 0.15, ((1.0, 0.01, 1.0),), 1, (1.0, 1.0), 0, 0,
                         contact_radius=R, turn_gain=0.0, noise_sigma=0.0, step_len=0.25, seed=5)
    # targets: anywhere; on map-cell boundaries; on walls (some in corners)
    cell = max(R, L.max() / (2048 if dim == 2 else 256))
    targets = rng.random((n_targets, dim)) * L
    on_edge = rng.random((n_targets, dim)) < 0.3
    targets = np.where(on_edge, np.minimum(np.round(targets / cell) * cell, L), targets)
    wall = rng.random((n_targets, dim)) < 0.05
    targets = np.where(wall, np.where(rng.random((n_targets, dim)) < 0.5, 0.0, L), targets)
    # tips after the step: near a contact sphere, or anywhere
    m = 6000
    u = rng.normal(size=(m, dim))
    u /= np.linalg.norm(u, axis=1, keepdims=True)
    tips = targets[rng.integers(0, n_targets, m)] + u * (R * rng.uniform(0.98, 1.02, (m, 1)))
    tips = np.where(rng.random((m, 1)) < 0.15, rng.random((m, dim)) * L, tips)
    tips = np.clip(tips, 0.6, L - 0.6)   # neither end of the step meets a wall
    h = rng.normal(size=(m, dim))
    h /= np.linalg.norm(h, axis=1, keepdims=True)
    f32 = lambda v: np.asarray(v, dtype=np.float32).astype(np.float64)
    sc.target_pos = f32(targets)
    sc.cone_pos = f32(tips - 0.25 * h)
    sc.cone_dir = f32(np.arctan2(h[:, 1], h[:, 0]) if dim == 2 else h)
    with B.Simulation(sc, block_steps=block) as sim:
        sim.step(1)
        got = sim.cones()
    pos = got["pos"].astype(np.float64)
    slack = 4.0 * L.max() * 2.0 ** -24 + R * 2.0 ** -22
    status, target = np.zeros(m, dtype=np.int64), np.full(m, -1, dtype=np.int64)
    sure = np.ones(m, dtype=bool)
    for at in range(0, m, 500):
        d = np.linalg.norm(pos[at:at + 500, None, :] - sc.target_pos[None], axis=2)
        two = np.sort(d, axis=1)[:, :2]
        hit = two[:, 0] < R
        status[at:at + 500] = hit
        target[at:at + 500] = np.where(hit, np.argmin(d, axis=1), -1)
        sure[at:at + 500] = (np.abs(two[:, 0] - R) > slack) & \
            (~hit | (two[:, 1] - two[:, 0] > 2.0 * slack))
    assert sure.mean() > 0.9 and status[sure].any() and not status[sure].all()
    np.testing.assert_array_equal(got["status"][sure], status[sure])
    np.testing.assert_array_equal(got["target"][sure], target[sure])
