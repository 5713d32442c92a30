"""The finalize in one kernel (no tensor of more than eight segments, and not
too many tensors) and in two, at the sizes where a segment or the one-kernel
range ends: the same tensors alone and beside a wider one, or among thousands,
each against the oracle and against each other bit for bit (the order of every
sum is the same). And the planless step's table, at the tensor counts where a
batch of it ends."""

import numpy as np
import pytest

import gpu_harness as H
from paper_1904_00962_amd import _lib

pytestmark = pytest.mark.gpu

CHUNK = 8
SEG = 2048 * CHUNK           # elements of a segment
SIZES = [1, 7, 8, 255 * CHUNK, SEG - 1, SEG, SEG + 1, 4 * SEG, 4 * SEG + 1, 5 * SEG + 9,
         8 * SEG - 8, 8 * SEG]
WIDER = 8 * SEG + 1


@pytest.mark.parametrize("variant,norm,skip", [("lamb", "l2", 0), ("lamb", "l1", 1),
                                               ("n-lamb", "linf", 0), ("lars", "l2", 1)])
@pytest.mark.parametrize("call", ["step", "split"])
def test_one_kernel_equals_two(call, variant, norm, skip):
    torch = H.torch_cuda()
    algo = "lars" if variant == "lars" else "lamb"
    rng = np.random.default_rng(5)
    # skip: the moment pass's chunks, and so the segments, are eight times as long
    sizes = [s * (8 if skip else 1) for s in SIZES + [WIDER]]
    xs = [(rng.standard_normal(s) * 0.05).astype(np.float32) for s in sizes]
    gs = [(rng.standard_normal(s) * 1e-3 + 2e-3).astype(np.float32) for s in sizes]
    n = len(SIZES)
    states = []
    for k in (n, n + 1):
        pair = H.Pair(xs[:k], [i % 2 == 0 for i in range(k)], "f32", algo, chunk_elems=CHUNK,
                      path="two-pass")
        hg = pair.set_grads([torch.from_numpy(g) for g in gs[:k]])
        hp = _lib.lamb_hparams_init(variant, step=1, lr=1e-2, norm=norm, skip_nonfinite=skip)
        tol = pair.ratio_tolerances(hp, hg)
        if call == "step":
            ref = H.step_ex_both(pair, hp, hg)
        else:
            totals = torch.zeros(2 * k + 1, dtype=torch.float64, device="cuda")
            _lib.lamb_step_partials(pair.plan, hp, 0, totals.data_ptr())
            _lib.lamb_step_finish(pair.plan, hp, 0, totals.data_ptr(), pair.ratio.data_ptr(),
                                  pair.norms.data_ptr(), 0)
            ref = H.step_ex_both_oracle(pair, hp, hg)
        torch.cuda.synchronize()
        pair.compare(ref, "%s %s %d tensors" % (call, variant, k), tol)
        states.append([s.clone() for s in pair.X[:n] + pair.M[:n]] +
                      [pair.ratio[:n].clone(), pair.norms[:2 * n].clone()])
        pair.close()
    for a, b in zip(*states):
        assert torch.equal(a, b)


@pytest.mark.parametrize("norm", ["l2", "linf"])
def test_any_number_of_tensors(norm):
    """Tensors of one segment among a few, in one kernel of four teams a tensor;
    among thousands, in one kernel of one team; beside one of two segments, in
    two kernels."""
    torch = H.torch_cuda()
    rng = np.random.default_rng(6)
    first = [1, 9, 2047 * CHUNK, SEG]
    xs, states = [], []
    for tail in ([300, 4 * SEG], [7] * 3000, [7] * 3000 + [SEG + 1]):
        sizes = first + tail
        while len(xs) < len(first):
            xs.append((rng.standard_normal(first[len(xs)]) * 0.05).astype(np.float32))
        here = xs + [(rng.standard_normal(s) * 0.05).astype(np.float32) for s in tail]
        subset = list(range(len(first))) + [len(sizes) - 2, len(sizes) - 1]
        pair = H.Pair(here, [True] * len(sizes), "f32", "lamb", chunk_elems=CHUNK,
                      oracle_subset=subset, path="two-pass")
        hg = pair.set_grads([torch.full((s,), 1e-3) for s in sizes])
        hp = _lib.lamb_hparams_init("lamb", step=1, lr=1e-2, norm=norm)
        tol = pair.ratio_tolerances(hp, hg)
        pair.compare(H.step_ex_both(pair, hp, hg), "%s, %d tensors" % (norm, len(sizes)), tol)
        n = len(first)
        states.append([s.clone() for s in pair.X[:n] + pair.M[:n]] +
                      [pair.ratio[:n].clone(), pair.norms[:2 * n].clone()])
        pair.close()
    for other in states[1:]:
        for a, b in zip(states[0], other):
            assert torch.equal(a, b)


@pytest.mark.parametrize("n", [1, 81, 82, 83, 165])
def test_static_table_batches(n):
    torch = H.torch_cuda()
    rng = np.random.default_rng(n)
    sizes = [1 + 977 * k % 4099 for k in range(n - 1)] + [600001]
    xs = [(rng.standard_normal(s) * 0.05).astype(np.float32) for s in sizes]
    gs = [(rng.standard_normal(s) * 1e-3).astype(np.float32) for s in sizes]
    results = []
    for static in (False, True):
        pair = H.Pair(xs, [i % 3 != 0 for i in range(n)], "f32", "lamb", path="two-pass")
        pair.set_grads([torch.from_numpy(g) for g in gs])
        hp = _lib.lamb_hparams_init("lamb", step=1, lr=1e-2)
        out = pair.ratio.data_ptr(), pair.norms.data_ptr()
        if static:
            rows = [(x.data_ptr(), g.data_ptr(), m.data_ptr(), v.data_ptr(), x.numel(), int(w))
                    for x, g, m, v, w in zip(pair.X, pair.G, pair.M, pair.V, pair.wd)]
            _lib.lamb_step_static(rows, _lib.LAMB_GRAD_F32, hp, 0, 0, *out)
        else:
            _lib.lamb_step_ex(pair.plan, hp, 0, *out)
        torch.cuda.synchronize()
        results.append([t.clone() for t in pair.X + pair.M + pair.V + [pair.ratio, pair.norms]])
        pair.close()
    for a, b in zip(*results):
        assert torch.equal(a, b)
