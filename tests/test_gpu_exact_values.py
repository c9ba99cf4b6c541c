"""Sampled {I, NOT, CNOT, CV, CV+} circuits on targets of 0, +-1 and +-i take gate
bodies with fewer operations while nothing can be rounded (up to 36 gates CV or CV+):
the fused kernel leaves the bits that the evaluation of the same circuits leaves,
at lengths whose circuits stay below that count, straddle it and pass it after a
whole chunk, and with targets of other values between populations of exact ones."""
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


def targets(oracle, n, I):
    rng = np.random.default_rng(n)
    N, out = 1 << n, []
    for i in range(I):
        U = oracle.unitary(n, inputs.random_target_gates(rng, n, 10, permutation=True)).astype(np.complex128)
        if i % 4 == 1:
            U = U * (1j ** rng.integers(0, 4, N))            # signs and units, also -0.0 parts
        if i % 4 == 2:
            U = U * np.exp(0.3j * np.arange(N))              # other values
        if i % 4 == 3:
            U = 1j ** rng.integers(0, 4, (N, N))             # no zero at all: the largest sums
        out.append(U)
    return np.stack(out)


@pytest.mark.parametrize("n,P", [(4, 7), (4, 300), (5, 7), (5, 64), (6, 7), (6, 300)])
@pytest.mark.parametrize("L", [20, 64, 90, 200])
def test_fused_equals_evaluation(dev, oracle, n, P, L):
    I = 6
    T = torch.from_numpy(targets(oracle, n, I)).to(dev)
    ctx = qe.Context(n, qe.LIB_NCV, qe.ALG_QEQEA, L, P, I, prob_mutation=0.3, seed=L)
    ctx.set_targets(T)
    cvs = []
    for gen in range(2):
        out = ctx.sample_eval(gen)
        gates, f = out[1], out[-1]
        assert torch.equal(f, ctx.eval_population(gates))
        per = f.view(I, P)
        for i in range(I):
            g = gates.view(I, P, L)[i].contiguous()
            assert torch.equal(qe.eval_fitness(g, T[i].to(torch.complex64), n=n, L=L, target_stride=0)[0], per[i])
        cvs.append(((gates.view(-1, L) & 15) >= 3).sum(1))
        ctx.update(gen, out[0], gates, f)
    ctx.close()
    cvs = torch.cat(cvs)
    assert (L != 20 or cvs.max() <= 36) and (L != 200 or cvs.max() > 36)
    assert qe.device_errors() == 0
