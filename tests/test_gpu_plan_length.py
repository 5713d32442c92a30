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


class _Copies:
    """A bf16 copy of every layer: the SIZES layers' between guard bands of 8
    elements, the fillers' in slots of 64."""

    GUARD = -3.0

    def __init__(self, pair):
        torch = H.torch_cuda()
        sizes = [x.numel() for x in pair.X]
        n = len(SIZES)
        self.bands = [torch.full((s + 16,), self.GUARD, dtype=torch.bfloat16, device="cuda")
                      for s in sizes[:n]]
        self.fill = torch.full((max(1, len(sizes) - n), 64), self.GUARD, dtype=torch.bfloat16,
                               device="cuda")
        self.pair = pair
        _lib.lamb_plan_set_bf16_copies(
            pair.plan, [b.data_ptr() + 16 for b in self.bands] +
            [self.fill.data_ptr() + 128 * k for k in range(len(sizes) - n)])

    def check(self):
        """Every copy is its x rounded; nothing around it was written."""
        torch = H.torch_cuda()
        for x, b in zip(self.pair.X, self.bands):
            assert torch.equal(b[8:-8], x.to(torch.bfloat16)), x.numel()
            assert bool((b[:8] == self.GUARD).all()) and bool((b[-8:] == self.GUARD).all())
        want = torch.full_like(self.fill, self.GUARD)
        for k, x in enumerate(self.pair.X[len(SIZES):]):
            want[k, :x.numel()] = x.to(torch.bfloat16)
        assert torch.equal(self.fill, want)


def _plan_state(pair):
    return [t.clone() for t in pair.X + pair.M + (pair.V if pair.V is not None else [])]


def _equal(a, b):
    return len(a) == len(b) and all(H.torch_cuda().equal(p, q) for p, q in zip(a, b))


def _options_inputs(long, seed):
    rng = np.random.default_rng(seed)
    sizes = SIZES + ([1 + 37 * k % 61 for k in range(FILLERS)] if long else [])
    xs = [(rng.standard_normal(s) * 0.05).astype(np.float32) for s in sizes]
    grads = [[(rng.standard_normal(s) * 1e-3 + 2e-3).astype(np.float32) for s in sizes]
             for _ in range(3)]
    return sizes, xs, grads, [k % 2 == 0 for k in range(len(sizes))]


@pytest.mark.parametrize("long", [False, True])
@pytest.mark.parametrize("captured", [False, True])
@pytest.mark.parametrize("path,variant,g_dtype", [("auto", "lamb", "bf16"), ("wide", "lars", "f32"),
                                                  ("wide", "nn-lamb", "bf16")])
def test_copies_skips_and_replays(path, variant, g_dtype, captured, long):
    """Both kernels with bf16 copies and skip_nonfinite, eager or replayed from a
    graph: a step, a step skipped for a NaN in one layer (the last of the plan,
    then the first), a step, a step. A skipped one reports it and writes nothing;
    the others match the oracle, and each copy is its layer's x."""
    torch = H.torch_cuda()
    algo = "lars" if variant == "lars" else "lamb"
    n = len(SIZES)
    sizes, xs, grads, wd = _options_inputs(long, 91)
    # (replays repeat one step number)
    hp = _lib.lamb_hparams_init(variant, step=2, lr=1e-2, skip_nonfinite=1)
    pair = H.Pair(xs, wd, g_dtype, algo, oracle_subset=range(n), path=path)
    try:
        assert (_rounds(pair.plan, sizes) > QUICK_ROUNDS) == long
        copies = _Copies(pair)
        verdict = torch.full((1,), 7, dtype=torch.int32, device="cuda")

        def step():
            _lib.lamb_step_ex(pair.plan, hp, torch.cuda.current_stream().cuda_stream,
                              pair.ratio.data_ptr(), pair.norms.data_ptr(), verdict.data_ptr())

        graph = None
        for t, nan_layer in enumerate([None, len(sizes) - 1, None, 0, None]):
            gs = [torch.from_numpy(g.copy()) for g in grads[t % 3]]
            if nan_layer is not None:
                gs[nan_layer][-1] = float("nan")
            hg = pair.set_grads(gs)
            tol = None if nan_layer is not None else pair.ratio_tolerances(hp, hg)
            before = _plan_state(pair)
            torch.cuda.synchronize()
            if captured and t == 1:
                side = torch.cuda.Stream()
                side.wait_stream(torch.cuda.current_stream())
                graph = torch.cuda.CUDAGraph()
                with torch.cuda.graph(graph, stream=side):
                    step()
                torch.cuda.synchronize()
            if graph is not None:
                graph.replay()
            else:
                step()
            torch.cuda.synchronize()
            label = "%s %s t=%d" % (variant, "long" if long else "short", t)
            if nan_layer is not None:
                assert int(verdict) == 1, label
                assert _equal(before, _plan_state(pair)), label
            else:
                assert int(verdict) == 0, label
                pair.compare(H.step_ex_both_oracle(pair, hp, hg), label, tol)
            copies.check()
        _lib.lamb_plan_check(pair.plan)
    finally:
        pair.close()


@pytest.mark.parametrize("long", [False, True])
@pytest.mark.parametrize("path", ["auto", "wide"])
def test_abandoned_wait_on_both_kernels(path, long, monkeypatch):
    """With a budget of one poll a wait gives up (every workgroup still exits):
    the plan reports it and its later steps write nothing, the copies included;
    a plan with the normal budget steps on."""
    torch = H.torch_cuda()
    n = len(SIZES)
    sizes, xs, grads, wd = _options_inputs(long, 92)
    hp = _lib.lamb_hparams_init("lamb", step=1, lr=1e-2)
    out = lambda p: (p.ratio.data_ptr(), p.norms.data_ptr())  # noqa: E731
    monkeypatch.setenv("LAMB_MI355X_SPIN_LIMIT", "1")
    pair = H.Pair(xs, wd, "f32", "lamb", oracle_subset=range(n), path=path)
    monkeypatch.delenv("LAMB_MI355X_SPIN_LIMIT")
    try:
        assert (_rounds(pair.plan, sizes) > QUICK_ROUNDS) == long
        copies = _Copies(pair)
        pair.set_grads([torch.from_numpy(g) for g in grads[0]])
        _lib.lamb_step_ex(pair.plan, hp, 0, *out(pair))
        with pytest.raises(_lib.LambError) as e:
            _lib.lamb_plan_check(pair.plan)
        assert e.value.status == _lib.LAMB_ESYNC
        before = _plan_state(pair) + [b.clone() for b in copies.bands + [copies.fill]]
        _lib.lamb_step_ex(pair.plan, hp, 0, *out(pair))
        torch.cuda.synchronize()
        assert _equal(before, _plan_state(pair) + copies.bands + [copies.fill])
    finally:
        pair.close()
    pair = H.Pair(xs, wd, "f32", "lamb", oracle_subset=range(n), path=path)
    try:
        hg = pair.set_grads([torch.from_numpy(g) for g in grads[0]])
        tol = pair.ratio_tolerances(hp, hg)
        pair.compare(H.step_ex_both(pair, hp, hg), "after a give-up", tol)
        _lib.lamb_plan_check(pair.plan)
    finally:
        pair.close()
