"""The register-resident kernels (widths 4 to 6) give the bits of the LDS-staged
ones: the same operations on every element and the same order of the
reduction.  Every library, lengths around the chunks of 64 gates, circuits
without gates, and the QEQEA loop's whole encoding; the tolerance is none."""
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


@pytest.fixture()
def schedule():
    saved = {(n, c, k): qe.get_schedule_lib(n, c, k) for n in range(4, 7) for c in (0, 1) for k in (0, 1, 2)}

    def use(n, lds, cpb=4):
        for c in (0, 1):
            qe.set_schedule_ex(n, c, lds, 4 if n == 6 else 1, 1 if n == 6 else cpb)
    yield use
    for (n, c, k), v in saved.items():
        qe.set_schedule_lib(n, c, k, *v)


def circuits(rng, lib, B, n, L):
    if lib in ("ncv", "ht"):
        return inputs.random_circuits(rng, B, n, L, inputs.LIB_NCV if lib == "ncv" else inputs.LIB_HT_NCV), None
    return inputs.random_ising_circuits(rng, B, n, L, discrete_frac=0.5 if lib == "both" else 0.0)


@pytest.mark.parametrize("n", [4, 5, 6])
@pytest.mark.parametrize("lib", ["ncv", "ht", "ising", "both"])
@pytest.mark.parametrize("L", [1, 40, 64, 65, 150])
def test_same_bits_as_lds_kernel(dev, schedule, n, lib, L):
    rng = np.random.default_rng(10 * n + L)
    B = 71
    g, a = circuits(rng, lib, B, n, L)
    gd = torch.from_numpy(g.view(np.int16)).to(dev)
    ad = None if a is None else torch.from_numpy(a.view(np.int32)).to(dev)
    T = qe.build_unitary(torch.from_numpy(circuits(rng, "ht", 1, n, 20)[0].view(np.int16)).to(dev), n, 20)
    out = []
    for lds in (1, 0):
        schedule(n, lds)
        out.append(qe.eval_fitness(gd, T, n=n, L=L, target_stride=0, want_g=True, want_delta=True, angles=ad))
    for x, y in zip(*out):
        assert torch.equal(x, y)
    assert qe.device_errors() == 0


@pytest.mark.parametrize("n", [4, 5, 6])
def test_empty_and_uneven_circuits(dev, schedule, n):
    rng = np.random.default_rng(n)
    lens = np.array([0, 3, 0, 64, 1, 0, 130])
    goff = torch.from_numpy(np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)).to(dev)
    g = torch.from_numpy(inputs.random_circuits(rng, 1, n, int(lens.sum()), 1)[0].view(np.int16)).to(dev)
    T = qe.build_unitary(g[3:23].reshape(1, 20).contiguous(), n, 20)
    out = []
    for lds in (1, 0):
        schedule(n, lds)
        out.append(qe.eval_fitness(g, T, n=n, goff=goff, target_stride=0)[0])
    assert torch.equal(*out)


@pytest.mark.parametrize("n,lib", [(4, qe.LIB_NCV), (5, qe.LIB_NCV), (6, qe.LIB_NCV), (4, qe.LIB_ISING),
                                   (5, qe.LIB_ISING), (6, qe.LIB_ISING)])
@pytest.mark.parametrize("L", [40, 70])
def test_qeqea_loop_same_bits(dev, oracle, schedule, n, lib, L):
    P, I, seed = 33, 2, 500 + n
    rng = np.random.default_rng(seed)
    T = np.stack([oracle.unitary(n, inputs.random_target_gates(rng, n, 10, permutation=True)) for _ in range(I)])
    runs = []
    for lds, cpb in ((1, 4), (0, 4), (0, 1)):
        schedule(n, lds, cpb)
        ctx = qe.Context(n, lib, qe.ALG_QEQEA, L, P, I, prob_mutation=0.3, seed=seed)
        ctx.set_targets(torch.from_numpy(T).to(dev))
        fs = [ctx.generation(g).clone() for g in range(3)]
        runs.append(fs + list(ctx.sample_eval(3)) + [ctx.state(k) for k in ("theta", "qutrit", "best_f")])
        ctx.close()
    for r in runs[1:]:
        for x, y in zip(r, runs[0]):
            assert torch.equal(x, y)
    assert qe.device_errors() == 0
