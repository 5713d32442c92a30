"""The single pass's two kernels (plans of few rounds, plans of many) at the
sizes where a tile, a block or a float4 ends: the same layers alone in a plan
and among ten thousand small ones, each against the oracle and against each
other bit for bit (tiles and summation order do not depend on the plan)."""

import numpy as np
import pytest

import gpu_harness as H
from paper_1904_00962_amd import _lib

pytestmark = pytest.mark.gpu

# float4s, 1024-element blocks, tiles of 8 and 10 blocks, and layers of several
# tiles whose last block is whole, ragged, or a lone element; each tile count
# with blocks missing from some of its tiles
SIZES = [1, 2, 3, 4, 5, 7, 1020, 1023, 1024, 1025, 1027, 4096, 8191, 8192, 8193, 10239, 10240,
         10241, 36864, 5 * 8192 + 1026, 7 * 10240 + 1, 100003, 64 * 8192, 300 * 1024 + 4]
FILLERS = 10400
QUICK_ROUNDS = 10


def _rounds(plan, sizes):
    cus = H.torch_cuda().cuda.get_device_properties(0).multi_processor_count
    groups = _lib.lamb_plan_tiles(plan)[2]
    *_, round_width, _ = _lib.lamb_tile_schedule(sizes, 4 * cus, groups)
    return _lib.lamb_plan_tiles(plan)[1] / round_width


@pytest.mark.parametrize("path", ["auto", "wide"])
@pytest.mark.parametrize("variant,g_dtype,norm,eps", [
    ("lamb", "f32", "l2", 1e-6), ("lamb", "bf16", "l2", 0.0), ("nn-lamb", "bf16", "l1", 1e-8),
    ("n-lamb", "f32", "linf", 0.0), ("lars", "bf16", "l2", 0.0), ("lars", "f32", "l1", 0.0)])
def test_short_and_long_plans_agree(path, variant, g_dtype, norm, eps):
    torch = H.torch_cuda()
    algo = "lars" if variant == "lars" else "lamb"
    rng = np.random.default_rng(77)
    n = len(SIZES)
    fill = [1 + 37 * k % 61 for k in range(FILLERS)]
    xs = [(rng.standard_normal(s) * 0.05).astype(np.float32) for s in SIZES + fill]
    grads = [[(rng.standard_normal(s) * 1e-3 + 2e-3).astype(np.float32) for s in SIZES + fill]
             for _ in range(2)]
    wd = [k % 2 == 0 for k in range(n + FILLERS)]
    states = []
    for sizes in (SIZES, SIZES + fill):
        k = len(sizes)
        pair = H.Pair(xs[:k], wd[:k], g_dtype, algo, oracle_subset=range(n), path=path)
        assert (_rounds(pair.plan, sizes) <= QUICK_ROUNDS) == (k == n)
        for t in range(1, 3):
            hg = pair.set_grads([torch.from_numpy(g) for g in grads[t - 1][:k]])
            hp = _lib.lamb_hparams_init(variant, step=t, lr=1e-2, eps=eps, norm=norm)
            tol = pair.ratio_tolerances(hp, hg)
            ref = H.step_ex_both(pair, hp, hg)
            pair.compare(ref, "%s %s plan t=%d" % (variant, "long" if k > n else "short", t), tol)
        state = pair.X[:n] + pair.M[:n] + (pair.V[:n] if pair.V is not None else [])
        states.append([s.clone() for s in state] + [pair.ratio[:n].clone()])
        pair.close()
    for a, b in zip(*states):
        assert torch.equal(a, b)


@pytest.mark.parametrize("path", ["auto", "wide"])
@pytest.mark.parametrize("n,quick", [(3000, True), (11000, False)])
def test_ragged_layers_in_successive_rounds(path, n, quick):
    """Layers of 1 to 1023 elements that end in every wave of the workgroup,
    round after round, on both kernels: against the oracle, and bit for bit
    against the same layers in plans of one round (x, m, v, bf16 copies)."""
    torch = H.torch_cuda()
    rng = np.random.default_rng(n)
    sizes = [int(4 * k + e) for k, e in zip(rng.integers(0, 256, n), rng.integers(1, 4, n))]
    xs = [(rng.standard_normal(s) * 0.05).astype(np.float32) for s in sizes]
    gs = [(rng.standard_normal(s) * 1e-3 + 2e-3).astype(np.float32) for s in sizes]
    hp = _lib.lamb_hparams_init("lamb", step=1, lr=1e-2)
    step = 1000  # layers of a plan of one round

    def run(lo, hi, subset):
        pair = H.Pair(xs[lo:hi], [True] * (hi - lo), "f32", "lamb", oracle_subset=subset,
                      path=path)
        copies = [torch.zeros(s + 8, dtype=torch.bfloat16, device="cuda") for s in sizes[lo:hi]]
        _lib.lamb_plan_set_bf16_copies(pair.plan, [c.data_ptr() for c in copies])
        rounds = _rounds(pair.plan, sizes[lo:hi])
        hg = pair.set_grads([torch.from_numpy(g) for g in gs[lo:hi]])
        tol = pair.ratio_tolerances(hp, hg)
        ref = H.step_ex_both(pair, hp, hg)
        pair.compare(ref, "%d ragged layers from %d" % (hi - lo, lo), tol)
        state = [torch.cat([t.float() for t in part]) for part in (pair.X, pair.M, pair.V, copies)]
        pair.close()
        return state, rounds

    whole, rounds = run(0, n, range(0, n, 43))
    assert rounds >= 2 and (rounds <= QUICK_ROUNDS) == quick
    parts = [run(lo, lo + step, []) for lo in range(0, n, step)]
    assert all(r <= 1 for _, r in parts)
    for k, a in enumerate(whole):
        assert torch.equal(a, torch.cat([p[0][k] for p in parts]))
