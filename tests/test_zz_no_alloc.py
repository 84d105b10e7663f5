"""rollout_static_scratch: the roll-out for callers that cannot allocate (its workspace is a fixed array in
the library's device image) gives, through the C ABI, what rollout gives with a caller-owned workspace --
bit for bit, since the kernels are the same -- on calls in a row of which the later ones are smaller; it
refuses a task whose workspace exceeds the array before launching anything."""
import numpy as np
import pytest
import torch

from workloads import generators as gen

from util import dev, host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def evo():
    import paper_2202_05008_amd as evo
    return evo


def _both(evo, kind, pd, params, pop, **task):
    td = evo.make_task_desc(kind, **task)
    need = evo.rollout_workspace_bytes(td, pd, pop)
    assert 0 < need <= evo.rollout_static_scratch_bytes()
    work = torch.empty(need, dtype=torch.uint8, device="cuda")
    td_own = evo.make_task_desc(kind, work=work, **task)
    want = torch.full((pop,), np.nan, dtype=torch.float32, device="cuda")
    got = torch.full((pop,), np.nan, dtype=torch.float32, device="cuda")
    evo.rollout(td_own, pd, params, pop, 1, want)
    evo.rollout_static_scratch(td, pd, params, pop, 1, got)        # work_dev is NULL here
    torch.cuda.synchronize()
    assert np.isfinite(host(want)).all()
    assert torch.equal(got, want)
    return host(got)


def test_static_scratch_matches_rollout_on_calls_in_a_row(evo):
    from oracle import policy as opolicy, tasks as otasks
    # a ConvNet classification (partial loss sums per member and chunk), then a smaller one
    pd = evo.make_policy_desc(evo.EVO_POLICY_CONVNET, (28, 8, 16, 10))
    P = evo.policy_param_count(pd)
    for pop, B, seed in ((12, 150, 1), (4, 13, 2)):
        params = gen.random_params(50 + seed, pop, P, 0.1)
        img, y = gen.mnist_shaped_batch(60 + seed, 1, B)
        fit = _both(evo, evo.EVO_TASK_CLASSIFY, pd, dev(params), pop, B=B, obs=dev(img), target=dev(y))
        ref = otasks.classify_fitness(opolicy.convnet_forward(params, img), y)
        assert np.abs(fit - ref).max() <= 1e-5 * np.abs(ref).max()
    # the sphere (partial sums per member and slice of the parameters): large, then small
    for pop, P in ((64, 1 << 16), (6, 4099)):
        params = gen.random_params(70, pop, P, 1.0)
        xs = gen.sphere_target(71, P)
        fit = _both(evo, evo.EVO_TASK_SPHERE, None, dev(params), pop, P=P, target=dev(xs))
        ref = otasks.sphere_fitness(params, xs)
        assert np.abs(fit - ref).max() <= 1e-5 * np.abs(ref).max()
    # an fp32 MLP classification, and back to the first shape: stale contents of the shared array do not matter
    pdm = evo.make_policy_desc(evo.EVO_POLICY_MLP, (16, 32, 4), (1, 0))
    x, y = gen.class_blobs(80, 300, 16, 4)
    _both(evo, evo.EVO_TASK_CLASSIFY, pdm, dev(gen.random_params(81, 10, 676, 0.3)), 10, B=300, obs=dev(x),
          target=dev(y))
    params = gen.random_params(51, 12, evo.policy_param_count(pd), 0.1)
    img, y = gen.mnist_shaped_batch(61, 1, 150)
    _both(evo, evo.EVO_TASK_CLASSIFY, pd, dev(params), 12, B=150, obs=dev(img), target=dev(y))


def test_static_scratch_refuses_what_does_not_fit(evo):
    P, pop = 1 << 20, 16384
    td = evo.make_task_desc(evo.EVO_TASK_SPHERE, P=P, target=torch.zeros(16, device="cuda"))
    assert evo.rollout_workspace_bytes(td, None, pop) > evo.rollout_static_scratch_bytes()
    fake = torch.zeros(16, device="cuda")
    with pytest.raises(evo.EvoError) as e:
        evo.rollout_static_scratch(td, None, fake, pop, 1, torch.zeros(pop, device="cuda"))
    assert e.value.code == -3 and "built-in scratch" in str(e.value)


_COUNTS = r"""
static int (*real)(void**, unsigned);
static int count;
void set_real(void* f) { real = (int (*)(void**, unsigned))f; }
int events_created(void) { return count; }
int hipEventCreateWithFlags(void** event, unsigned flags) { ++count; return real(event, flags); }
"""
_PROGRAM = r"""
import ctypes, sys
stub = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)      # before anything that brings the runtime's own
import torch
import paper_2202_05008_amd as evo
evo.make_policy_desc(evo.EVO_POLICY_MLP, (8, 32, 32, 2), (1, 1, 1))
from paper_2202_05008_amd import _lib
_lib.load()
paths = {l.split()[-1] for l in open("/proc/self/maps") if "libamdhip64" in l}
assert len(paths) == 1, paths
real = ctypes.CDLL(paths.pop()).hipEventCreateWithFlags
stub.set_real(ctypes.cast(real, ctypes.c_void_p))
pop, worlds, steps = 64, 8, 40
pd = evo.make_policy_desc(evo.EVO_POLICY_MLP, (8, 32, 32, 2), (1, 1, 1))
params = torch.randn(pop, evo.policy_param_count(pd), device="cuda")
cp = (0.0625, 0.015625, 0.875, 0.25, 0.0625, 24, 24)
task = dict(n_rollouts=worlds, reset_seed=3, cp=cp)
td = evo.make_task_desc(evo.EVO_TASK_FORAGE, **task)
work = torch.empty(evo.rollout_workspace_bytes(td, pd, pop), dtype=torch.uint8, device="cuda")
got, again, want = (torch.full((pop,), float("nan"), device="cuda") for _ in range(3))
torch.cuda.synchronize()
before = stub.events_created()
evo.rollout_static_scratch(td, pd, params, pop, steps, got)
assert stub.events_created() == before, "the entry point that allocates nothing created an event"
evo.rollout(evo.make_task_desc(evo.EVO_TASK_FORAGE, work=work, **task), pd, params, pop, steps, want)
assert stub.events_created() == before + 1, "rollout orders its one launches by an event"
evo.rollout_static_scratch(td, pd, params, pop, steps, again)
assert stub.events_created() == before + 1
torch.cuda.synchronize()
assert torch.isfinite(want).all() and torch.equal(got, want) and torch.equal(again, want)
print("created nothing")
"""


def test_static_scratch_creates_no_event(tmp_path):
    """A forage episode in one launch: the event that orders such launches is rollout's to create.  In a process of its
    own, where the runtime's routine is counted and nothing has run before."""
    import os
    import subprocess
    import sys
    (tmp_path / "counts.c").write_text(_COUNTS)
    stub = str(tmp_path / "libcounts.so")
    subprocess.run(["gcc", "-shared", "-fPIC", "-o", stub, str(tmp_path / "counts.c")], check=True)
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", _PROGRAM, stub], capture_output=True, text=True, timeout=100, cwd=root)
    assert r.returncode == 0 and "created nothing" in r.stdout, (r.stdout, r.stderr)
