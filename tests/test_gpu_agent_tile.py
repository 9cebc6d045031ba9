"""The agent kernels of agent.hip, on calls that the register-resident plans
refuse, against the oracle, with the library's profile showing which kernel
ran.  First the tile form of their Z/V phase (slices read from global memory),
shapes chosen to reach each of its cases:

  - a row side longer than one block of 12 rows (20, 15 and 16 rows), with
    one and with two row factors (block boundaries inside the second factor);
  - several 32-column chunks per context (42 columns) and a ragged last chunk;
  - an odd column count (the pair's second column is the padding column);
  - a rank-0 row side (V only) and two column factors;
  - soft observations (the per-context log-likelihood tensors);
  - a window longer than one context chunk of the Z/V scratch (T = 100);
  - FPI on steps whose slices exceed one step's LDS staging, with a slice of
    598 or 1122 rows taking one dot product per thread beside tiled ones, its
    update by segments of lanes and by waves.

Then the staged and untiled forms.  What makes the resident plans refuse a
call: more than 8 factors (here factors of two states that no list names),
factors of more than 64 states, more than 16 modalities, a window too long for
their LDS, FPI with more than four maximal lists or steps beyond a workgroup's
registers.  The same lists without that are run too, on the resident kernels.
"""
import numpy as np
import pytest

from paper_2607_17855_amd import bi, synth
import oracle
from agent_plan import plan_of_handle
from test_gpu_parity import check_invariants

pytestmark = pytest.mark.gpu
TOL = 1e-5

TILE, RESIDENT, STREAMED = "agent_window_tile", "agent_window_resident", "agent_window_streamed"
FILTER_TILE, FILTER_RESIDENT = "agent_filter_tile", "agent_filter_resident"


def _nine(n, U):
    """The factors with others of two states behind them, nine in all."""
    return n + [2] * (9 - len(n)), U + [1] * (9 - len(n))


CASES = [
    # (n, U, K, deps, b, T, per_agent): the slices of one context exceed what
    # the window's LDS staging takes, so the window kernels of agent.hip read
    # them from global memory
    ([20, 6, 7], [2, 1, 3], [5, 3, 4], [[0, 1, 2], [1], [0, 2]], 6, 12, True),
    ([3, 5, 4, 6], [1, 2, 2, 1], [4, 3], [[0, 1, 2, 3], [2, 3]], 5, 30, True),
    ([4, 4, 30], [2, 2, 1], [6], [[0, 1, 2]], 4, 20, False),
    ([20, 6, 7], [2, 1, 3], [5, 3, 4], [[0, 1, 2], [1], [0, 2]], 3, 100, True),
]
KERNEL = [RESIDENT] * 3 + [TILE]
# the first three with nine factors
CASES += [(*_nine(n, U), *rest) for n, U, *rest in CASES[:3]]
KERNEL += [TILE] * 3


def _torch():
    import torch
    return torch


def _workload(case, iters):
    n, U, K, deps, b, T, per_agent = CASES[case]
    rng = np.random.Generator(np.random.PCG64(1300 + case))
    model = synth.make_model(rng, n, U, K, deps, b if per_agent else 1, 0.7, 1.0, uniform_D=False)
    obs, act = synth.sample_sequences(rng, model, b, T)
    return synth.Workload(f"tile{case}", ["vmp", "mmp"], model, obs, act, iters)


def _dev(x):
    return _torch().from_numpy(np.ascontiguousarray(x)).cuda()


def _profiled(pm, call, *args):
    """The call's result and the names of the kernels it ran."""
    bi.bi_profile_begin()
    q = call(*args)
    _torch().cuda.synchronize()
    return q.cpu().numpy(), set(bi.bi_profile_end())


@pytest.mark.parametrize("case", range(len(CASES)))
@pytest.mark.parametrize("algo", ["vmp", "mmp"])
def test_tile_vs_oracle(case, algo):
    torch = _torch()
    w = _workload(case, 16 if case in (0, 4) else 3)
    print(f"[gpu] {w.name} {algo} b={w.b} T={w.T} iters={w.iters}", flush=True)
    pm = bi.PackedModel(w.model, bi.BI_DENSE_A)
    try:
        assert pm.path(w.b, w.T, algo) == "agent"
        q, names = _profiled(pm, pm.infer, algo, _dev(w.obs), _dev(w.act), w.iters)
        assert names == {KERNEL[case]}, names
        check_invariants(w, q)
        ref = oracle.infer(algo, w.model, w.obs, w.act, w.iters)
        err = float(np.abs(q - ref).max())
        print(f"[gpu]   tile vs oracle {err:.3e}", flush=True)
        assert err <= TOL
        # fixed summation order: the same call gives the same bits
        q2 = pm.infer(algo, _dev(w.obs), _dev(w.act), w.iters)
        torch.cuda.synchronize()
        assert np.array_equal(q, q2.cpu().numpy())
    finally:
        pm.close()


# FPI reads a step's slices from global memory when they exceed what one
# step's LDS staging takes: the tile form then serves the modalities of at
# most 96 rows, one dot product per thread the taller ones (mixed).
FPI_CASES = [
    # (n, K, deps, b, T): every modality tiled (a 30 x 700 slice)
    ([30, 25, 28], [3, 4], [[0, 1, 2], [2]], 3, 4),
    # a 598 x 31 slice (one dot product per thread) beside tiled ones
    ([23, 26, 31], [3, 4, 5], [[0, 1, 2], [0, 2], [1]], 3, 4),
    # the same forms (40 x 868; 1122 x 35) beyond a workgroup's registers
    ([40, 28, 31], [3, 4], [[0, 1, 2], [2]], 3, 4),
    ([33, 34, 35], [3, 4, 5], [[0, 1, 2], [0, 2], [1]], 3, 4),
]
FPI_KERNEL = [(FILTER_RESIDENT, STREAMED)] * 2 + [(FILTER_TILE, STREAMED)] * 2
# the first two with nine factors
FPI_CASES += [(_nine(n, [])[0], *rest) for n, *rest in FPI_CASES[:2]]
FPI_KERNEL += [(FILTER_TILE, TILE)] * 2


@pytest.mark.parametrize("case", range(len(FPI_CASES)))
@pytest.mark.parametrize("algo", ["fpi", "vmp", "mmp"])
def test_tile_large_slices(case, algo):
    n, K, deps, b, T = FPI_CASES[case]
    rng = np.random.Generator(np.random.PCG64(1360 + case))
    model = synth.make_model(rng, n, [2] * len(n), K, deps, b, 0.7, 1.0, uniform_D=False)
    obs, act = synth.sample_sequences(rng, model, b, T)
    w = synth.Workload(f"tile_large{case}", [algo], model, obs, act, 4)
    print(f"[gpu] {w.name} {algo} b={w.b} T={w.T}", flush=True)
    pm = bi.PackedModel(w.model, bi.BI_DENSE_A)
    try:
        q, names = _profiled(pm, pm.infer, algo, _dev(w.obs), _dev(w.act), w.iters)
        assert names == {FPI_KERNEL[case][algo != "fpi"]}, names
        check_invariants(w, q)
        ref = oracle.infer(algo, w.model, w.obs, w.act, w.iters)
        err = float(np.abs(q - ref).max())
        print(f"[gpu]   tile vs oracle {err:.3e}", flush=True)
        assert err <= TOL
        if algo == "fpi" and case >= 2:   # observation vectors through the same form
            so = synth.soft_obs(rng, w.obs, w.model.K, confidence=0.5)
            q, names = _profiled(pm, pm.infer_soft, algo, _dev(so), _dev(w.act), w.iters)
            assert names == {FILTER_TILE, "soft_ll"}, names
            ref = oracle.infer_soft(algo, w.model, so.astype(np.float64), w.act, w.iters)
            assert float(np.abs(q - ref).max()) <= TOL
    finally:
        pm.close()


# The other forms: (n, U, K, deps, b, T), the forms of FPI and of the windows
# ("" where a resident kernel runs).
FORMS = {
    "nine_factors_short": (*_nine([5, 4, 3], [2, 1, 2]), [4, 3, 2], [[0, 1], [1, 2], [2]], 4, 6, "lds", "lds_short"),
    "nine_factors": (*_nine([12, 5], [2, 3]), [4, 3], [[0, 1], [0]], 4, 6, "lds", "lds"),
    "long_factor": ([70, 3], [2, 1], [4, 3], [[0, 1], [0]], 3, 5, "lds", "lds"),
    "many_modalities": ([6, 4], [2, 2], [2] * 17, [[0, 1], [0], [1]] * 5 + [[0, 1]] * 2, 3, 5, "global", "global"),
    "five_lists": ([5, 4, 6, 3, 4, 5], [2, 1, 2, 1, 2, 1], [3] * 5, [[0, 1], [1, 2], [2, 3], [3, 4], [4, 5]], 3, 6,
                   "lds", ""),
}


@pytest.mark.parametrize("algo", ["fpi", "vmp", "mmp"])
@pytest.mark.parametrize("name", list(FORMS))
def test_other_forms_vs_oracle(name, algo):
    n, U, K, deps, b, T, *form = FORMS[name]
    form = form[algo != "fpi"]
    rng = np.random.Generator(np.random.PCG64(1380 + list(FORMS).index(name)))
    model = synth.make_model(rng, n, U, K, deps, b, 0.7, 1.0, uniform_D=False)
    obs, act = synth.sample_sequences(rng, model, b, T)
    w = synth.Workload(f"form_{name}", [algo], model, obs, act, 8)
    print(f"[gpu] {w.name} {algo} b={w.b} T={w.T}", flush=True)
    pm = bi.PackedModel(w.model, bi.BI_DENSE_A)
    try:
        plan = plan_of_handle(pm.handle, b, T, algo)
        assert plan.get("src", "") == form, plan
        q, names = _profiled(pm, pm.infer, algo, _dev(w.obs), _dev(w.act), w.iters)
        assert names == {plan["kernel"]}, names
        check_invariants(w, q)
        err = float(np.abs(q - oracle.infer(algo, w.model, w.obs, w.act, w.iters)).max())
        prior = synth.random_prior(rng, w.model.n, w.b, p_zero=0.3)
        qp = pm.infer(algo, _dev(w.obs), _dev(w.act), 5, prior=_dev(prior), damping=0.6).cpu().numpy()
        errp = float(np.abs(qp - oracle.infer(algo, w.model, w.obs, w.act, 5, prior=prior, damping=0.6)).max())
        print(f"[gpu]   vs oracle {err:.3e}, prior and damping {errp:.3e}", flush=True)
        assert err <= TOL and errp <= TOL
    finally:
        pm.close()


@pytest.mark.parametrize("case", [0, 4])
@pytest.mark.parametrize("algo", ["vmp", "mmp"])
def test_tile_soft_observations(algo, case):
    torch = _torch()
    w = _workload(case, 3)
    so = synth.soft_obs(np.random.Generator(np.random.PCG64(1350)), w.obs, w.model.K, confidence=0.5)
    print(f"[gpu] {w.name} soft {algo} b={w.b} T={w.T}", flush=True)
    pm = bi.PackedModel(w.model, bi.BI_DENSE_A)
    try:
        q, names = _profiled(pm, pm.infer_soft, algo, _dev(so), _dev(w.act), w.iters)
        assert names == {KERNEL[case], "soft_ll"}, names
        check_invariants(w, q)
        ref = oracle.infer_soft(algo, w.model, so.astype(np.float64), w.act, w.iters)
        err = float(np.abs(q - ref).max())
        print(f"[gpu]   tile soft vs oracle {err:.3e}", flush=True)
        assert err <= TOL
        # one-hot vectors reproduce the integer call bit for bit
        qs = pm.infer_soft(algo, _dev(synth.one_hot_obs(w.obs, w.model.K)), _dev(w.act), w.iters)
        qi = pm.infer(algo, _dev(w.obs), _dev(w.act), w.iters)
        torch.cuda.synchronize()
        assert np.array_equal(qs.cpu().numpy(), qi.cpu().numpy())
    finally:
        pm.close()
