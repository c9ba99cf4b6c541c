"""Layouts of the fused sampling kernel that meet only in large contexts: the
shared-slot search together with the register kernels of widths 4 to 6, lengths of
one chunk and more (chunks after the first are sampled before the gates run and
committed afterwards), and width 6 with a column per lane over the Ising library.
Fused results equal the step-by-step ones, or the LDS-staged kernel's, bit for bit."""
import numpy as np
import pytest
import torch

from paper_1809_11134_amd import inputs, qe

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    qe.load()
    return torch.device("cuda", 0)


def targets(oracle, dev, n, I, seed):
    rng = np.random.default_rng(seed)
    few = [oracle.unitary(n, inputs.random_target_gates(rng, n, 9, permutation=True)) for _ in range(3)]
    return torch.from_numpy(np.stack(few)).to(dev)[torch.arange(I, device=dev) % 3]


@pytest.mark.parametrize("n,lib,I,P,L,cpb", [(4, qe.LIB_NCV, 260, 31, 70, 1), (4, qe.LIB_NCV, 260, 31, 70, 4),
                                             (4, qe.LIB_ISING, 140, 29, 130, 1),
                                             (5, qe.LIB_ISING, 140, 62, 66, 1), (5, qe.LIB_NCV, 300, 15, 129, 4),
                                             (6, qe.LIB_NCV, 220, 49, 51, 1), (6, qe.LIB_NCV, 240, 33, 70, 1),
                                             (6, qe.LIB_ISING, 220, 49, 51, 1)])
def test_search_with_register_kernels(dev, oracle, n, lib, I, P, L, cpb):
    assert I * P * L > 524288
    saved = {(c, k): qe.get_schedule_lib(n, c, k) for c in (0, 1) for k in (0, 1, 2)}
    try:
        for c in (0, 1):
            qe.set_schedule_ex(n, c, 0, 4 if n == 6 else 1, cpb)
        T = targets(oracle, dev, n, I, n)
        runs = []
        for fused in (True, False):
            ctx = qe.Context(n, lib, qe.ALG_QEQEA, L, P, I, prob_mutation=0.3, seed=L)
            ctx.set_targets(T)
            for gen in range(3):
                if fused:
                    f = ctx.generation(gen)
                else:
                    slots, g, *a = ctx.sample(gen)
                    a = a[0] if lib == qe.LIB_ISING else None
                    f = ctx.eval_population(g, angles=a)
                    ctx.update(gen, slots, g, f, angles=a)
            runs.append([f] + [ctx.state(k) for k in ("theta", "qutrit", "best_f", "best_theta", "best_qutrit")])
            ctx.close()
        for x, y in zip(*runs):
            assert torch.equal(x, y)
    finally:
        for (c, k), v in saved.items():
            qe.set_schedule_lib(n, c, k, *v)
    assert qe.device_errors() == 0


@pytest.mark.parametrize("lib,P", [(qe.LIB_ISING, 1023), (qe.LIB_ISING, 1024), (qe.LIB_NCV, 639), (qe.LIB_NCV, 640)])
@pytest.mark.parametrize("L", [40, 64, 70])
def test_width_6_layouts(dev, oracle, lib, P, L):
    T = targets(oracle, dev, 6, 1, 6)
    ctx = qe.Context(6, lib, qe.ALG_QEQEA, L, P, prob_mutation=0.3, seed=P + L)
    ctx.set_targets(T)
    for gen in (0, 1):
        ctx.generation(gen)
    slots, g, *a = ctx.sample(2)
    a = a[0] if lib == qe.LIB_ISING else None
    out = ctx.sample_eval(2)
    assert torch.equal(out[0], slots) and torch.equal(out[1], g)
    if a is not None:
        assert torch.equal(out[2], a)
    assert torch.equal(out[-1], ctx.eval_population(g, angles=a))
    lds = qe.eval_fitness(g, T, n=6, L=L, target_stride=0, path=qe.PATH_FP32_LDS, angles=a)[0]
    assert torch.equal(out[-1], lds)
    ctx.close()
    assert qe.device_errors() == 0


@pytest.mark.parametrize("n,P,L", [(4, 9, 64), (5, 9, 90), (5, 90, 200), (6, 9, 200), (6, 220, 70)])
def test_exact_values_end_in_registers(dev, oracle, n, P, L):
    # the bodies for exact values and the end of their reach (36 CV gates), register
    # schedule set; targets of units, with one other entry (the first or the last
    # looked at), of no zero at all
    N, rng = 1 << n, np.random.default_rng(n)
    T = np.stack([np.eye(N)[rng.permutation(N)].astype(np.complex128) for _ in range(3)] +
                 [1j ** rng.integers(0, 4, (N, N))])
    T[1], T[2] = np.eye(N), np.eye(N)
    T[1, 0, 0], T[2, N - 1, N - 1] = np.exp(0.3j), 0.75
    T = torch.from_numpy(T).to(dev)
    saved = {(c, k): qe.get_schedule_lib(n, c, k) for c in (0, 1) for k in (0, 1, 2)}
    try:
        qe.set_schedule(n, 0)
        ctx = qe.Context(n, qe.LIB_NCV, qe.ALG_QEQEA, L, P, 4, prob_mutation=0.3, seed=L)
        ctx.set_targets(T)
        for gen in range(2):
            slots, g, f = ctx.sample_eval(gen)
            for i in range(4):
                one = g.view(4, P, L)[i].contiguous()
                want = qe.eval_fitness(one, T[i].to(torch.complex64), n=n, L=L, target_stride=0, path=qe.PATH_FP32_LDS)[0]
                assert torch.equal(f.view(4, P)[i], want), i
            ctx.update(gen, slots, g, f)
        ctx.close()
    finally:
        for (c, k), v in saved.items():
            qe.set_schedule_lib(n, c, k, *v)
    assert qe.device_errors() == 0
