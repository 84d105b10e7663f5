"""GPU parity tests of the shared-world task (the whole population as agents of one world) against
oracle/forage.py.  The world's arithmetic is binary32 by definition, so a step from a given state
with given actions is compared bit for bit; so is a whole roll-out whose policies ignore their
observations (constant actions).  With observation-driven policies the fp32 policy output differs
from the oracle's in the last bits, so one step is compared at 1e-6 and longer horizons
statistically (a flipped nearest neighbour is a legitimate, discontinuous difference)."""
import numpy as np
import pytest

from oracle import forage
from workloads import CONFIGS, configs as wc, generators as gen
from tests.util import dev, host

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SEED = 20220509


@pytest.fixture(scope="module")
def evo():
    import paper_2202_05008_amd as e
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return e


def _cp(w):
    return (w["dt"], w["thrust"], w["drag"], w["vmax"], w["radius"], float(w["n_food"]), float(w["n_poison"]))


def _task(evo, w, worlds, pop, pd=None, generation=3, seed=SEED, kind=None):
    kind = evo.EVO_TASK_FORAGE if kind is None else kind
    make = lambda work: evo.make_task_desc(kind, n_rollouts=worlds, reset_seed=seed,
                                           generation=generation, cp=_cp(w), work=work)
    if pd is None:
        return make(None)
    n = evo.rollout_workspace_bytes(make(None), pd, pop)
    assert n > 0
    return make(torch.empty(n, dtype=torch.uint8, device="cuda"))


def _bits(a):
    a = np.ascontiguousarray(a)
    return a.view(np.uint32) if a.dtype == np.float32 else a


@pytest.mark.parametrize("pop,worlds,n_food,n_poison,radius", [(130, 3, 5, 7, 0.0625), (1024, 5, 24, 24, 0.03125),
                                                               (2, 1, 1, 1, 0.25), (77, 8, 100, 156, 0.015625),
                                                               (2500, 2, 24, 24, 0.03125),
                                                               (4800, 1, 24, 24, 0.03125)])   # the most that fit
def test_one_step_from_a_given_state_is_bit_exact(evo, pop, worlds, n_food, n_poison, radius):
    w = dict(forage.WORLD_DEFAULT, n_food=n_food, n_poison=n_poison, radius=radius)
    n_items = n_food + n_poison
    rng = np.random.default_rng(pop * 31 + worlds)
    pos = rng.random((worlds, pop, 2), dtype=np.float32)
    vel = (rng.random((worlds, pop, 2), dtype=np.float32) - np.float32(0.5)) * np.float32(2 * w["vmax"])
    act = (rng.standard_normal((worlds, pop, 2)) * 1.2).astype(np.float32)
    counts = rng.integers(0, 6, size=(worlds, n_items)).astype(np.int32)
    # special cases: agents on top of each other (distance 0, index tie-break), on the walls and heading
    # out, and sitting on items of their world (touches)
    if pop >= 16:
        pos[:, 5] = pos[:, 3]
        pos[:, 9] = pos[:, 3]
        pos[:, 7] = (0.0, 1.0)
        vel[:, 7] = (-w["vmax"], w["vmax"])
        act[:, 7] = (-1.0, 1.0)
        for r in range(worlds):
            items = forage.item_positions(SEED, 3, r, counts[r])
            pos[r, 10:10 + min(4, n_items)] = items[:min(4, n_items)]
            pos[r, 14] = items[-1] + np.float32(radius / 2)
            vel[r, 10:15] = 0
            act[r, 10:15] = 0
    td = _task(evo, w, worlds, pop)
    f32, i32 = torch.float32, torch.int32
    obs = torch.empty(worlds, pop, 8, dtype=f32, device="cuda")
    npos, nvel = torch.empty(worlds, pop, 2, dtype=f32, device="cuda"), torch.empty(worlds, pop, 2, dtype=f32, device="cuda")
    reward = torch.full((worlds, pop), 99, dtype=i32, device="cuda")
    hit = torch.full((worlds, n_items), 99, dtype=i32, device="cuda")
    evo.evo_forage_step(td, pop, dev(pos), dev(vel), dev(counts), dev(act), obs, npos, nvel, reward, hit)
    touched = 0
    for r in range(worlds):
        items = forage.item_positions(SEED, 3, r, counts[r])
        want_obs = forage.observe(pos[r], vel[r], items, n_food)
        p, v, rew, h = forage.step(pos[r], vel[r], act[r], items, n_food, w)
        assert np.array_equal(_bits(host(obs)[r]), _bits(want_obs)), "observations of world %d" % r
        assert np.array_equal(_bits(host(npos)[r]), _bits(p)), "positions of world %d" % r
        assert np.array_equal(_bits(host(nvel)[r]), _bits(v)), "velocities of world %d" % r
        assert np.array_equal(host(reward)[r], rew), "rewards of world %d" % r
        assert np.array_equal(host(hit)[r], h.astype(np.int32)), "hits of world %d" % r
        touched += int(np.abs(rew).sum())
    assert touched > 0 or pop < 16, "the case must exercise touches"


def _params_constant_action(pop, dims, rng):
    """Zero weights, the output bias as the action (no output activation): policies that ignore what they see."""
    P = wc.mlp_param_count(dims)
    params = np.zeros((pop, P), dtype=np.float32)
    params[:, -2:] = (rng.random((pop, 2), dtype=np.float32) - np.float32(0.5)) * np.float32(3.0)
    return params


def _run_state(evo, td, pd, params, pop, worlds, n_items, steps, solo=False):
    f32, i32 = torch.float32, torch.int32
    pos = torch.empty(worlds, pop, 2, dtype=f32, device="cuda")
    vel = torch.empty(worlds, pop, 2, dtype=f32, device="cuda")
    reward = torch.empty(worlds, pop, dtype=i32, device="cuda")
    counts = torch.empty((worlds, pop, n_items) if solo else (worlds, n_items), dtype=i32, device="cuda")
    evo.evo_forage_state(td, pd, params, pop, steps, pos, vel, reward, counts)
    fit = torch.empty(pop, dtype=f32, device="cuda")
    evo.rollout(td, pd, params, pop, steps, fit)
    return host(pos), host(vel), host(reward), host(counts), host(fit)


@pytest.mark.parametrize("pop,worlds,H,steps", [(150, 3, 16, 61), (64, 1, 32, 40), (34, 6, 64, 35)])
def test_whole_rollout_with_constant_actions_is_bit_exact(evo, pop, worlds, H, steps):
    w = dict(forage.WORLD_DEFAULT, n_food=9, n_poison=6, radius=0.0625)
    dims, acts = (8, H, H, 2), (evo.EVO_ACT_TANH, evo.EVO_ACT_RELU, evo.EVO_ACT_NONE)
    params = _params_constant_action(pop, dims, np.random.default_rng(H))
    pd = evo.make_policy_desc(evo.EVO_POLICY_MLP, dims, acts)
    td = _task(evo, w, worlds, pop, pd)
    pos, vel, reward, counts, fit = _run_state(evo, td, pd, dev(params), pop, worlds, 15, steps)
    want_fit, total, details = forage.rollout(params, dims, acts, SEED, 3, worlds, steps, w, return_details=True)
    for r in range(worlds):
        assert np.array_equal(_bits(pos[r]), _bits(details[r][0])), "positions of world %d" % r
        assert np.array_equal(_bits(vel[r]), _bits(details[r][1])), "velocities of world %d" % r
        assert np.array_equal(counts[r], details[r][2]), "item book of world %d" % r
    assert np.array_equal(reward, total)
    assert np.abs(total).sum() > 20 and max(d[2].max() for d in details) >= 2, "items must be eaten, some twice"
    np.testing.assert_allclose(fit, want_fit, rtol=1e-6, atol=0)


def _random_policies(pop, dims, scale, seed):
    P = wc.mlp_param_count(dims)
    return (np.random.default_rng(seed).standard_normal((pop, P)) * scale).astype(np.float32)


@pytest.mark.parametrize("H,acts", [(32, (1, 1, 1)), (16, (2, 1, 0)), (64, (1, 2, 1))])
def test_one_step_with_the_policy_in_the_loop(evo, H, acts):
    pop, worlds = 200, 2
    w = dict(forage.WORLD_DEFAULT, radius=0.0625)
    dims = (8, H, H, 2)
    params = _random_policies(pop, dims, 0.5, H)
    pd = evo.make_policy_desc(evo.EVO_POLICY_MLP, dims, acts)
    td = _task(evo, w, worlds, pop, pd)
    pos, vel, reward, counts, fit = _run_state(evo, td, pd, dev(params), pop, worlds, 48, 1)
    _, total, details = forage.rollout(params, dims, acts, SEED, 3, worlds, 1, w, return_details=True)
    for r in range(worlds):
        np.testing.assert_allclose(vel[r], details[r][1], rtol=0, atol=1e-7)
        np.testing.assert_allclose(pos[r], details[r][0], rtol=0, atol=1e-7)
    assert np.array_equal(reward, total)
    assert np.abs(vel).max() > 1e-3, "the policies must act"


def test_short_horizon_with_the_policy_in_the_loop(evo):
    pop, worlds, steps = 256, 2, 20
    w = dict(forage.WORLD_DEFAULT, radius=0.0625)
    dims, acts = (8, 32, 32, 2), (1, 1, 1)
    params = _random_policies(pop, dims, 0.5, 11)
    pd = evo.make_policy_desc(evo.EVO_POLICY_MLP, dims, acts)
    td = _task(evo, w, worlds, pop, pd)
    pos, vel, reward, counts, fit = _run_state(evo, td, pd, dev(params), pop, worlds, 48, steps)
    want_fit, total, details = forage.rollout(params, dims, acts, SEED, 3, worlds, steps, w, return_details=True)
    want_pos = np.stack([d[0] for d in details])
    close = np.abs(pos - want_pos).max(axis=-1) < 1e-5
    assert close.mean() > 0.97, "agents off the oracle's path: %d of %d" % ((~close).sum(), close.size)
    assert (reward == total).mean() > 0.97
    assert np.abs(total).sum() > 10


def test_long_horizon_population_statistics(evo):
    """300 steps with observation-driven policies: single trajectories part ways (a nearest neighbour that
    flips is a discontinuity), the population's statistics do not: the two fitness vectors have the same mean
    within sampling error and are strongly rank-correlated (what an agent collects is mostly its policy's doing)."""
    from scipy.stats import spearmanr
    pop, worlds, steps = 128, 4, 300
    w = dict(forage.WORLD_DEFAULT, radius=0.0625)
    dims, acts = (8, 32, 32, 2), (1, 1, 1)
    params = _random_policies(pop, dims, 0.7, 23)
    pd = evo.make_policy_desc(evo.EVO_POLICY_MLP, dims, acts)
    td = _task(evo, w, worlds, pop, pd)
    pos, vel, reward, counts, fit = _run_state(evo, td, pd, dev(params), pop, worlds, 48, steps)
    want = forage.rollout(params, dims, acts, SEED, 3, worlds, steps, w)
    sem = np.sqrt((want.var() + fit.var()) / pop)
    assert abs(fit.mean() - want.mean()) < 4 * sem + 0.05, (fit.mean(), want.mean(), sem)
    assert abs(np.abs(fit).mean() - np.abs(want).mean()) < 0.25 * np.abs(want).mean() + 0.1
    rho = spearmanr(fit, want).correlation
    assert rho > 0.5, rho


def test_full_size_constant_actions_and_properties(evo):
    """The benchmark's configuration (1024 agents, 8 worlds, H = 32): 40 steps of policies that ignore
    their observations bit for bit against the oracle, then the full 500 steps with random policies:
    repeatable, whole-number rewards, everyone inside the square."""
    c = CONFIGS["forage"]
    w = wc.world_dict(c.world)
    n_items = w["n_food"] + w["n_poison"]
    pd = evo.make_policy_desc(evo.EVO_POLICY_MLP, c.dims, c.acts)
    td = _task(evo, w, c.n_rollouts, c.pop, pd)
    acts_none = (1, 1, 0)
    pd_none = evo.make_policy_desc(evo.EVO_POLICY_MLP, c.dims, acts_none)
    params = _params_constant_action(c.pop, c.dims, np.random.default_rng(1))
    pos, vel, reward, counts, fit = _run_state(evo, td, pd_none, dev(params), c.pop, c.n_rollouts, n_items, 40)
    want_fit, total, details = forage.rollout(params, c.dims, acts_none, SEED, 3, c.n_rollouts, 40, w, return_details=True)
    for r in range(c.n_rollouts):
        assert np.array_equal(_bits(pos[r]), _bits(details[r][0])) and np.array_equal(counts[r], details[r][2])
    assert np.array_equal(reward, total) and np.abs(total).sum() > 100
    params = dev(_random_policies(c.pop, c.dims, 0.3, 5))
    a = _run_state(evo, td, pd, params, c.pop, c.n_rollouts, n_items, c.steps)
    b = _run_state(evo, td, pd, params, c.pop, c.n_rollouts, n_items, c.steps)
    for x, y in zip(a, b):
        assert np.array_equal(_bits(x), _bits(y)), "two runs of the same roll-out differ"
    pos, vel, reward, counts, fit = a
    assert pos.min() >= 0 and pos.max() <= 1 and np.abs(vel).max() <= w["vmax"]
    np.testing.assert_array_equal(fit * c.n_rollouts, reward.sum(axis=0).astype(np.float32))
    assert counts.min() > 0, "over 500 steps every item of every world is eaten at some point"


@pytest.mark.parametrize("solo", [False, True])
@pytest.mark.parametrize("radius", [2.0, 1e19, 2e19, float("inf")])      # 2e19 and more: the square is infinite in binary32
def test_a_radius_over_the_whole_square_touches_every_item_and_no_empty_slot(evo, solo, radius):
    """Item lists that fill no chunk of slots: every agent touches every item in every step, in the whole episode as in the
    single step, and the hits and counts behind a world's items stay those of the next world."""
    pop, worlds, steps, food, poison = 9, 3, 4, 5, 2
    w = dict(forage.WORLD_DEFAULT, n_food=food, n_poison=poison, radius=radius)
    dims, acts = (8, 16, 16, 2), (1, 1, 0)
    pd = evo.make_policy_desc(evo.EVO_POLICY_MLP, dims, acts)
    params = dev(_params_constant_action(pop, dims, np.random.default_rng(2)))
    td = _task(evo, w, worlds, pop, pd, kind=evo.EVO_TASK_FORAGE_SOLO if solo else None)
    pos, vel, reward, counts, fit = _run_state(evo, td, pd, params, pop, worlds, food + poison, steps, solo=solo)
    assert (reward == steps * (food - poison)).all() and (fit == steps * (food - poison)).all()
    assert (counts == steps).all()
    if not solo:
        i32, f32 = torch.int32, torch.float32
        out = [torch.empty(worlds, pop, n, dtype=f32, device="cuda") for n in (8, 2, 2)]
        rew = torch.empty(worlds, pop, dtype=i32, device="cuda")
        hit = torch.full((worlds + 1, food + poison), 99, dtype=i32, device="cuda")
        zero = torch.zeros(worlds, pop, 2, dtype=f32, device="cuda")
        evo.evo_forage_step(td, pop, dev(pos), zero, dev(counts), zero, *out, rew, hit[:worlds])
        assert (host(rew) == food - poison).all() and (host(hit)[:worlds] == 1).all() and (host(hit)[worlds] == 99).all()


def _state(evo, td, pd, params, pop, worlds, n_items, steps, wait_ticks=None, form=None, expect=None, **fail):
    """The state after an episode; form, fail: evo_forage_state_form's, and how every world must have been played."""
    out = dict(pos=torch.empty(worlds, pop, 2, dtype=torch.float32, device="cuda"),
               vel=torch.empty(worlds, pop, 2, dtype=torch.float32, device="cuda"),
               reward=torch.empty(worlds, pop, dtype=torch.int32, device="cuda"),
               counts=torch.empty(worlds, n_items, dtype=torch.int32, device="cuda"))
    if form is not None:
        forms = torch.full((worlds,), 99, dtype=torch.int32, device="cuda")
        evo.evo_forage_state_form(td, pd, params, pop, steps, form, forms=forms, **out, **fail)
        assert expect is None or (forms == expect).all(), (forms.unique().tolist(), form, fail)
    elif wait_ticks is None:
        evo.evo_forage_state(td, pd, params, pop, steps, **out)
    else:
        evo.evo_forage_state_bounded(td, pd, params, pop, steps, wait_ticks, **out)
    return out


# agents per workgroup 32 (H = 64: 8), 64 lanes of candidates, items in chunks of 32 per list (256 items: nine chunks)
@pytest.mark.parametrize("pop,worlds,H,steps,n_food,n_poison,acts",
                         [(2, 1, 16, 9, 1, 1, (1, 1, 1)), (32, 3, 32, 9, 32, 32, (1, 1, 1)), (33, 3, 32, 9, 33, 32, (1, 1, 1)),
                          (64, 2, 16, 12, 9, 6, (1, 2, 0)), (129, 2, 32, 9, 5, 7, (0, 0, 0)), (8, 2, 64, 9, 24, 24, (1, 1, 1)),
                          (9, 4, 64, 9, 33, 223, (2, 1, 1)), (300, 4, 64, 12, 32, 33, (1, 1, 1)), (1000, 8, 32, 12, 24, 24, (1, 1, 1)),
                          (1090, 7, 16, 9, 1, 255, (1, 1, 1)), (64, 130, 32, 5, 24, 24, (1, 1, 1)),
                          (700, 5, 64, 5, 24, 24, (1, 1, 1)), (4800, 1, 32, 5, 24, 24, (1, 1, 1))])
def test_the_episode_in_one_launch_is_the_episode_step_by_step(evo, pop, worlds, H, steps, n_food, n_poison, acts):
    """Whole episodes with observation-driven policies: where every wait is given up the worlds are played again by the
    step kernel's code, and both give the same bits (stacked agents and agents in corners among them: a wide thrust
    drives many into the walls).  A workspace full of another call's words changes nothing.  So do a launch per step, and
    waits that end in vain in the middle of the episode, with the other workgroups of the world a step ahead."""
    w = dict(forage.WORLD_DEFAULT, n_food=n_food, n_poison=n_poison, radius=0.0625, thrust=0.25, vmax=2.0)
    pd = evo.make_policy_desc(evo.EVO_POLICY_MLP, (8, H, H, 2), acts)
    params = dev(_random_policies(pop, (8, H, H, 2), 0.5, pop + H))
    td = _task(evo, w, worlds, pop, pd)
    n_items = n_food + n_poison
    one = _state(evo, td, pd, params, pop, worlds, n_items, steps)
    again = _state(evo, td, pd, params, pop, worlds, n_items, steps, 0)
    after = _state(evo, td, pd, params, pop, worlds, n_items, steps)
    for k in one:
        assert torch.equal(one[k], again[k]), k
        assert torch.equal(one[k], after[k]), k
    assert pop < 32 or int(one["counts"].sum()) > 0, "items must be eaten"
    forms = [dict(form=1, expect=1), dict(form=2, expect=0)]
    for step in (1, 2, steps // 2, steps - 1):
        forms += [dict(form=1, expect=2, fail_step=step, fail_items=items) for items in (0, 1)]
    forms += [dict(form=1, expect=2, fail_step=steps, fail_items=1), dict(form=1, expect=1, fail_step=steps, fail_items=0)]
    for how in forms:
        other = _state(evo, td, pd, params, pop, worlds, n_items, steps, **how)
        assert all(torch.equal(one[k], other[k]) for k in one), how
    fit = torch.empty(pop, dtype=torch.float32, device="cuda")
    evo.rollout(td, pd, params, pop, steps, fit)
    assert np.array_equal(host(fit), host(one["reward"]).sum(axis=0).astype(np.float32) / np.float32(worlds))


# (agents, worlds, H, steps): the size of a control loop and of the benchmark; a step or two; few agents in many worlds
@pytest.mark.parametrize("pop,worlds,H,steps,one", [(1024, 8, 32, 40, 1), (64, 8, 64, 40, 1), (8, 256, 32, 40, 1), (64, 512, 32, 12, 1),
                                                    (4800, 1, 32, 2, 1), (1024, 8, 32, 1, 0), (64, 8, 16, 2, 0), (8, 1, 32, 2, 0),
                                                    (8, 2048, 32, 40, 0), (2, 4096, 16, 20, 0), (512, 64, 64, 20, 0)])
def test_a_rollout_takes_the_form_that_is_faster(evo, pop, worlds, H, steps, one):
    """At these sizes the two forms differ by 10 % and more: the roll-out's own choice is the faster, with the same bits."""
    w = dict(forage.WORLD_DEFAULT, radius=0.0625)
    pd = evo.make_policy_desc(evo.EVO_POLICY_MLP, (8, H, H, 2), (1, 1, 1))
    params = dev(_random_policies(pop, (8, H, H, 2), 0.5, pop + H))
    td = _task(evo, w, worlds, pop, pd)
    own = _state(evo, td, pd, params, pop, worlds, 48, steps, form=0, expect=one)
    other = _state(evo, td, pd, params, pop, worlds, 48, steps, form=2 if one else 1, expect=1 - one)
    assert all(torch.equal(own[k], other[k]) for k in own)


def _ms(run):
    best = float("inf")
    for _ in range(3):
        start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        start.record()
        run()
        end.record()
        end.synchronize()
        best = min(best, start.elapsed_time(end))
    return best


def test_an_episode_that_is_given_up_does_not_collapse(evo):
    """Where other work holds the chip, worlds are played again by as many workgroups as there are, not by one for four
    worlds: 8 times the episode here, and 220 with one for four."""
    pop, worlds, steps = 1024, 8, 100
    w = dict(forage.WORLD_DEFAULT, radius=0.0625)
    pd = evo.make_policy_desc(evo.EVO_POLICY_MLP, (8, 32, 32, 2), (1, 1, 1))
    params = dev(_random_policies(pop, (8, 32, 32, 2), 0.5, 3))
    td = _task(evo, w, worlds, pop, pd)
    one = _ms(lambda: _state(evo, td, pd, params, pop, worlds, 48, steps, form=1))
    again = _ms(lambda: _state(evo, td, pd, params, pop, worlds, 48, steps, 0))
    assert again < 20 * one, (again, one)


def test_later_launches_of_an_episode_that_is_given_up_do_not_wait(evo):
    """128 launches of 32 worlds: the first one's wait ends in vain after 0.2 ms, and the others leave at once (each waiting
    0.2 ms of its own, they took 26 ms)."""
    pop, worlds, steps = 64, 4096, 2
    w = dict(forage.WORLD_DEFAULT, radius=0.0625)
    pd = evo.make_policy_desc(evo.EVO_POLICY_MLP, (8, 64, 64, 2), (1, 1, 1))
    params = dev(_random_policies(pop, (8, 64, 64, 2), 0.5, 3))
    td = _task(evo, w, worlds, pop, pd)
    want = _state(evo, td, pd, params, pop, worlds, 48, steps, form=2, expect=0)
    got = _state(evo, td, pd, params, pop, worlds, 48, steps, form=1, expect=2, fail_step=1, fail_items=0)
    assert all(torch.equal(want[k], got[k]) for k in want)
    assert _ms(lambda: _state(evo, td, pd, params, pop, worlds, 48, steps, form=1, fail_step=1, fail_items=0)) < 13


def test_one_launch_episodes_on_two_streams(evo):
    """Each launch fills the chip: they take turns, whatever stream they are on, and no world is given up."""
    w = dict(forage.WORLD_DEFAULT, radius=0.0625)
    pd = evo.make_policy_desc(evo.EVO_POLICY_MLP, (8, 16, 16, 2), (1, 1, 1))
    pop, worlds, steps = 1024, 8, 20
    params = [dev(_random_policies(pop, (8, 16, 16, 2), 0.5, s)) for s in (1, 2)]
    tds = [_task(evo, w, worlds, pop, pd) for _ in range(2)]
    want = [_state(evo, td, pd, p, pop, worlds, 48, steps) for td, p in zip(tds, params)]
    streams = [torch.cuda.Stream() for _ in range(2)]
    torch.cuda.synchronize()
    got = [[], []]
    for _ in range(4):
        for i, s in enumerate(streams):
            with torch.cuda.stream(s):
                out, forms = _state(evo, tds[i], pd, params[i], pop, worlds, 48, steps), torch.empty(worlds, dtype=torch.int32, device="cuda")
                evo.evo_forage_state_form(tds[i], pd, params[i], pop, steps, 1, forms=forms, **out)
                got[i].append(dict(out, forms=forms))
    torch.cuda.synchronize()
    for g in got[0] + got[1]:
        assert (g.pop("forms") == 1).all(), "a launch met the other stream's on the chip"
    for i in range(2):
        for g in got[i]:
            assert all(torch.equal(g[k], want[i][k]) for k in g)


@pytest.mark.parametrize("H,acts", [(16, (2, 1, 0)), (32, (0, 2, 1)), (64, (1, 2, 0)), (64, (1, 1, 1))])
def test_a_recorded_episode_is_the_one_launch_episode(evo, H, acts):
    """Into a graph the steps are recorded one by one; its replays give the bits of the one launch."""
    pop, worlds, steps = 70, 3, 11
    w = dict(forage.WORLD_DEFAULT, radius=0.0625, thrust=0.25, vmax=2.0)
    pd = evo.make_policy_desc(evo.EVO_POLICY_MLP, (8, H, H, 2), acts)
    params = dev(_random_policies(pop, (8, H, H, 2), 0.5, H))
    td = _task(evo, w, worlds, pop, pd)
    want = _state(evo, td, pd, params, pop, worlds, 48, steps, form=1, expect=1)
    got = {k: torch.empty_like(v) for k, v in want.items()}
    forms = torch.empty(worlds, dtype=torch.int32, device="cuda")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        evo.evo_forage_state_form(td, pd, params, pop, steps, 1, forms=forms, **got)
    for _ in range(3):
        for t in (*got.values(), forms):
            t.zero_()
        graph.replay()
        assert (forms == 0).all() and all(torch.equal(want[k], got[k]) for k in want)
        assert all(torch.equal(v, want[k]) for k, v in _state(evo, td, pd, params, pop, worlds, 48, steps, form=1, expect=1).items())


def test_errors_are_reported(evo):
    w = forage.WORLD_DEFAULT
    good = evo.make_policy_desc(evo.EVO_POLICY_MLP, (8, 32, 32, 2), (1, 1, 1))
    fit = torch.empty(64, dtype=torch.float32, device="cuda")
    params = torch.zeros(64, wc.mlp_param_count((8, 32, 32, 2)), dtype=torch.float32, device="cuda")
    td = _task(evo, w, 2, 64, good)
    for dims in [(8, 32, 16, 2), (5, 32, 32, 2), (8, 48, 48, 2), (8, 32, 32, 1)]:
        bad = evo.make_policy_desc(evo.EVO_POLICY_MLP, dims, (1, 1, 1))
        with pytest.raises(evo.EvoError):
            evo.rollout(td, bad, params, 64, 5, fit)
    with pytest.raises(evo.EvoError):                    # no workspace
        evo.rollout(_task(evo, w, 2, 64), good, params, 64, 5, fit)
    with pytest.raises(evo.EvoError):                    # no poison
        evo.rollout(_task(evo, dict(w, n_poison=0), 2, 64), good, params, 64, 5, fit)
    big = torch.zeros(6000, params.shape[1], dtype=torch.float32, device="cuda")
    with pytest.raises(evo.EvoError):                    # more agents than the staging area holds
        evo.rollout(_task(evo, w, 2, 6000, good), good, big, 6000, 5, torch.empty(6000, dtype=torch.float32, device="cuda"))
    evo.rollout(td, good, params, 64, 5, fit)            # and the good case still runs
    assert torch.isfinite(fit).all()


# ---- the single-agent form: every member alone in its own copy of each world, one launch per episode ----

@pytest.mark.parametrize("pop,worlds,H,steps,n_food,n_poison", [(13, 3, 16, 60, 9, 6), (8, 1, 32, 45, 24, 24),
                                                                 (5, 6, 64, 35, 3, 40), (1, 1, 32, 30, 1, 1)])
def test_solo_rollout_with_constant_actions_is_bit_exact(evo, pop, worlds, H, steps, n_food, n_poison):
    w = dict(forage.WORLD_DEFAULT, n_food=n_food, n_poison=n_poison, radius=0.125)
    dims, acts = (8, H, H, 2), (evo.EVO_ACT_TANH, evo.EVO_ACT_RELU, evo.EVO_ACT_NONE)
    params = _params_constant_action(pop, dims, np.random.default_rng(H + pop))
    pd = evo.make_policy_desc(evo.EVO_POLICY_MLP, dims, acts)
    td = _task(evo, w, worlds, pop, pd, kind=evo.EVO_TASK_FORAGE_SOLO)
    n_items = n_food + n_poison
    pos, vel, reward, counts, fit = _run_state(evo, td, pd, dev(params), pop, worlds, n_items, steps, solo=True)
    want_fit, total, details = forage.rollout_solitary(params, dims, acts, SEED, 3, worlds, steps, w, return_details=True)
    for m in range(pop):
        for r in range(worlds):
            assert np.array_equal(_bits(pos[r, m]), _bits(details[m][r][0][0])), "position of member %d, world %d" % (m, r)
            assert np.array_equal(_bits(vel[r, m]), _bits(details[m][r][1][0]))
            assert np.array_equal(counts[r, m], details[m][r][2]), "item book of member %d, world %d" % (m, r)
    assert np.array_equal(reward, total)
    assert counts.sum() > 0 or n_items < 10, "items must be eaten"
    np.testing.assert_allclose(fit, want_fit, rtol=1e-6, atol=0)


def test_solo_policy_in_the_loop(evo):
    pop, worlds = 24, 2
    w = dict(forage.WORLD_DEFAULT, radius=0.0625)
    dims, acts = (8, 32, 32, 2), (1, 1, 1)
    params = _random_policies(pop, dims, 0.5, 31)
    pd = evo.make_policy_desc(evo.EVO_POLICY_MLP, dims, acts)
    td = _task(evo, w, worlds, pop, pd, kind=evo.EVO_TASK_FORAGE_SOLO)
    pos, vel, reward, counts, fit = _run_state(evo, td, pd, dev(params), pop, worlds, 48, 1, solo=True)
    _, total, details = forage.rollout_solitary(params, dims, acts, SEED, 3, worlds, 1, w, return_details=True)
    want_pos = np.stack([np.stack([details[m][r][0][0] for m in range(pop)]) for r in range(worlds)])
    want_vel = np.stack([np.stack([details[m][r][1][0] for m in range(pop)]) for r in range(worlds)])
    np.testing.assert_allclose(pos, want_pos, rtol=0, atol=1e-7)
    np.testing.assert_allclose(vel, want_vel, rtol=0, atol=1e-7)
    assert np.array_equal(reward, total) and np.abs(vel).max() > 1e-3
    # 25 steps: most members still on the oracle's path (a flipped nearest item is a legitimate discontinuity)
    pos, vel, reward, counts, fit = _run_state(evo, td, pd, dev(params), pop, worlds, 48, 25, solo=True)
    _, total, details = forage.rollout_solitary(params, dims, acts, SEED, 3, worlds, 25, w, return_details=True)
    want_pos = np.stack([np.stack([details[m][r][0][0] for m in range(pop)]) for r in range(worlds)])
    close = np.abs(pos - want_pos).max(axis=-1) < 1e-5
    assert close.mean() > 0.9 and (reward == total).mean() > 0.9


def test_solo_full_size_properties(evo):
    """1024 members x 8 worlds x 500 steps in one launch: repeatable bit for bit, inside the square, whole-number
    rewards; members with the same policy get the same result (their worlds are identical)."""
    c = CONFIGS["forage"]
    w = wc.world_dict(c.world)
    n_items = w["n_food"] + w["n_poison"]
    pd = evo.make_policy_desc(evo.EVO_POLICY_MLP, c.dims, c.acts)
    td = _task(evo, w, c.n_rollouts, c.pop, pd, kind=evo.EVO_TASK_FORAGE_SOLO)
    host_params = _random_policies(c.pop, c.dims, 0.3, 5)
    host_params[1::2] = host_params[0::2]                  # pairs of identical policies
    params = dev(host_params)
    a = _run_state(evo, td, pd, params, c.pop, c.n_rollouts, n_items, c.steps, solo=True)
    b = _run_state(evo, td, pd, params, c.pop, c.n_rollouts, n_items, c.steps, solo=True)
    for x, y in zip(a, b):
        assert np.array_equal(_bits(x), _bits(y)), "two runs of the same roll-out differ"
    pos, vel, reward, counts, fit = a
    assert pos.min() >= 0 and pos.max() <= 1 and np.abs(vel).max() <= w["vmax"]
    np.testing.assert_array_equal(fit * c.n_rollouts, reward.sum(axis=0).astype(np.float32))
    assert np.array_equal(reward[:, 0::2], reward[:, 1::2]) and np.array_equal(_bits(pos[:, 0::2]), _bits(pos[:, 1::2]))
    assert counts.sum() > 0 and np.array_equal(counts[:, :, :w["n_food"]].sum(axis=2) - counts[:, :, w["n_food"]:].sum(axis=2), reward)
