"""A target entry that is NaN, or infinite where the sums take it to NaN, gives NaN
and the numeric error flag on every path and width, and such circuits never count
as the best of a search."""
import numpy as np
import pytest
import torch

from paper_1809_11134_amd import inputs, qe

pytestmark = pytest.mark.gpu

PATHS = {"fp32": qe.PATH_FP32, "reg": qe.PATH_FP32_REG, "lds": qe.PATH_FP32_LDS, "dense": qe.PATH_DENSE,
         "bf16": qe.PATH_MFMA_BF16, "fp16_raw": qe.PATH_MFMA_FP16_RAW}


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    qe.load()
    return torch.device("cuda", 0)


def targets(rng, n, count):
    """Permutation targets; the second has a NaN off its diagonal, the third an
    infinite diagonal entry."""
    N = 1 << n
    T = np.stack([np.eye(N)[rng.permutation(N)] for _ in range(count)]).astype(np.complex128)
    T[1, 0, N - 1] = np.nan
    T[2] = np.eye(N)
    T[2, 1, 1] = np.inf
    return T


def check(f, bad=(1, 2)):
    nan = torch.isnan(f).cpu().numpy()
    assert sorted(np.nonzero(nan)[0]) == sorted(bad)
    assert qe.device_errors() == qe.DEVERR_NUMERIC


@pytest.mark.parametrize("path,n", [(p, n) for p in [*PATHS, "fp64", "angles"]
                                    for n in ((5, 6) if "16" in p else (2, 3, 4, 5, 6))])   # (MFMA: 5 and 6)
@pytest.mark.parametrize("B", [3, 1030])
def test_evaluation(dev, n, path, B):
    rng = np.random.default_rng(n)
    L = 9
    g = inputs.random_circuits(rng, B, n, L, inputs.LIB_NCV)
    g[2] = 0                                   # (the identity keeps the infinity on the diagonal)
    T = torch.from_numpy(targets(rng, n, B)).to(dev)
    gd = torch.from_numpy(g.view(np.int16)).to(dev)
    args = dict(n=n, L=L, target_stride=4 ** n)
    qe.device_errors()
    if path == "fp64":
        f = qe.eval_fitness_fp64(gd, T, **args)[0]
    elif path == "angles":
        f = qe.eval_fitness(gd, T, angles=torch.zeros_like(gd, dtype=torch.int32), **args)[0]
    else:
        f = qe.eval_fitness(gd, T, path=PATHS[path], **args)[0]
    check(f)


@pytest.mark.parametrize("B", [12, 4100])
@pytest.mark.parametrize("workspace", [True, False])
def test_mixed_widths(dev, B, workspace):
    rng = np.random.default_rng(B)
    L, nq = 7, (3 + np.arange(B) % 4).astype(np.int8)
    T = [targets(rng, n, 3) for n in range(3, 7)]
    base = np.cumsum([0] + [t.size for t in T])
    which = np.where(np.arange(B) < 12, np.arange(B) // 4, 0)     # each width: good, NaN, infinite
    toff = base[nq - 3] + which * 4 ** nq.astype(np.int64)
    g = np.concatenate([inputs.random_circuits(rng, 1, int(n), L, inputs.LIB_NCV) for n in nq])
    g[8:12] = 0
    qe.device_errors()
    f = qe.eval_fitness(torch.from_numpy(g.reshape(-1).view(np.int16)).to(dev),
                        torch.from_numpy(np.concatenate([t.reshape(-1) for t in T])).to(dev),
                        nq=torch.from_numpy(nq).to(dev), goff=torch.arange(0, B * L + 1, L, dtype=torch.int32, device=dev),
                        toff=torch.from_numpy(toff).to(dev), target_stride=None, workspace=workspace)[0]
    check(f, range(4, 12))


@pytest.mark.parametrize("lds", [0, 1])
@pytest.mark.parametrize("n,lib,P", [(3, qe.LIB_NCV, 8), (4, qe.LIB_NCV, 8), (5, qe.LIB_NCV, 8), (5, qe.LIB_ISING, 8),
                                     (6, qe.LIB_NCV, 8), (6, qe.LIB_NCV, 300)])
def test_searches(dev, lds, n, lib, P):
    rng = np.random.default_rng(n)
    saved = {(c, k): qe.get_schedule_lib(n, c, k) for c in (0, 1) for k in (0, 1, 2)}
    try:
        if n >= 4:
            qe.set_schedule(n, lds)
        T = torch.from_numpy(targets(rng, n, 3)).to(dev)
        T[2, 0, 0] = float("nan")
        qe.device_errors()
        ctx = qe.Context(n, lib, qe.ALG_QEQEA, 12, P, 3, prob_mutation=0.2, seed=n)
        ctx.set_targets(T)
        out = ctx.sample_eval(0)
        check(out[-1], range(P, 3 * P))
        ctx.update(0, None, out[1], out[-1], angles=out[2] if lib == qe.LIB_ISING else None)
        check(ctx.generation(1), range(P, 3 * P))
        best = ctx.state("best_f").reshape(3, -1)
        assert best[0].max().item() >= 0 and best[1:].max().item() == -1
        assert [ctx.get_best(i, with_fp64=False)[1] for i in (1, 2)] == [-1, -1]
        ctx.close()
        if lib == qe.LIB_NCV:
            ga = qe.Context(n, lib, qe.ALG_GA, 12, P, 3, seed=n)
            ga.set_targets(T)
            check(ga.generation(0), range(P, 3 * P))
            ga.close()
    finally:
        for (c, k), v in saved.items():
            qe.set_schedule_lib(n, c, k, *v)
