"""Arguments that the binding converts (gates in 32 bits, angles in 64, a strided
fitness) live until the call is launched: no later conversion of the same call may
take their memory.  The same results as with arguments that need no conversion."""
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


@pytest.mark.parametrize("P,L", [(64, 16), (50, 40)])
def test_calls_of_a_search(dev, oracle, P, L):
    n, k = 4, 4
    rng = np.random.default_rng(P)
    T = torch.from_numpy(oracle.unitary(n, inputs.random_target_gates(rng, n, 6, permutation=True))[None]).to(dev)
    runs = []
    for convert in (False, True):
        ctx = qe.Context(n, qe.LIB_ISING, qe.ALG_QEQEA, L, P, prob_mutation=0.3, seed=P)
        ctx.set_targets(T)
        slots, g, a = ctx.sample(0)
        f = ctx.eval_population(g, angles=a)
        if convert:
            torch.cuda.synchronize()
            torch.cuda.empty_cache()                 # (the next allocations come from the call's own frees)
            wide = torch.stack([f, torch.zeros_like(f)], 1)
            g, a, f = g.to(torch.int32), a.to(torch.int64) & 0xFFFFFFFF, wide[:, 0]
            assert torch.equal(ctx.eval_population(g, angles=a), f)
        out = ctx.elite_recheck(g, f, k, angles=a)
        ctx.update(0, slots, g, f, angles=a)
        runs.append([*out, ctx.get_best(0, with_angles=True)] + [ctx.state(s) for s in ("theta", "qutrit", "best_f")])
        ctx.close()
    for x, y in zip(*runs):
        assert torch.equal(x, y) if torch.is_tensor(x) else x == y
