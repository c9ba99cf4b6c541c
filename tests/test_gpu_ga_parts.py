"""The GA update splits a population over workgroups: population sizes around
the ends of its shares (one child, an odd last child, more pairs than one
workgroup takes, the largest population) and generations whose weights are all
zero, bit for bit against the oracle's update, teacher-forced; and the circuits
that a re-check without gates takes after another call wrote the genomes."""
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


@pytest.mark.parametrize("P,L,I", [(1, 7, 3), (2, 1, 2), (3, 33, 2), (64, 36, 5), (65, 36, 3), (257, 20, 1),
                                   (2047, 9, 1), (4096, 20, 1), (4095, 3, 2)])
def test_update_matches_oracle(dev, oracle, P, L, I):
    n, lib, seed = 3, 1, 900 + P
    rng = np.random.default_rng(seed)
    ctx = qe.Context(n, lib, qe.ALG_GA, L, P, I, seed=seed, ga_gene_mutation_prob=0.1)
    ctx.set_targets(torch.from_numpy(np.stack([oracle.unitary(n, inputs.random_target_gates(rng, n, 6, 1))
                                               for _ in range(I)])).to(dev))
    for gen in range(3):
        _, g = ctx.sample(gen)
        # fitness with ties, zeros and a NaN; generation 2: all zero
        f = rng.choice(np.array([0.0, 0.25, 0.5, 0.731, 1e-9], np.float32), size=(I, P))
        f[0, P // 2] = np.nan
        if gen == 2:
            f[:] = 0.0
        genomes = g.cpu().numpy().view(np.uint16).reshape(I, P, L)
        ctx.update(gen, None, g, torch.from_numpy(f.reshape(-1)).to(dev))
        _, got = ctx.sample(gen + 1)
        got = got.cpu().numpy().view(np.uint16).reshape(I, P, L)
        for i in range(I):
            want = oracle.ga_update_at(n, lib, L, P, i, seed, gen, float(np.float32(0.9)),
                                       float(np.float32(0.1)), f[i], genomes[i])
            assert np.array_equal(got[i], want), (gen, i)
    ctx.close()


def test_recheck_keeps_the_last_generation(dev, oracle):
    n, P, L, k = 4, 48, 12, 5
    rng = np.random.default_rng(3)
    T = torch.from_numpy(oracle.unitary(n, inputs.random_target_gates(rng, n, 6, 0))[None]).to(dev)
    ctx = qe.Context(n, qe.LIB_NCV, qe.ALG_GA, L, P, seed=5)
    ctx.set_targets(T)
    blob = ctx.checkpoint()
    for overwrite in ("nothing", "update", "restore"):
        ctx.restore(blob)
        f = ctx.generation(0)
        g = ctx.state("genomes0").reshape(P, L)          # generation 0's circuits
        want = ctx.elite_recheck(g, f, k)
        if overwrite == "update":
            ctx.update(1, None, ctx.sample(1)[1], f)     # writes genomes0
        elif overwrite == "restore":
            ctx.run_graph(0, 3, None)
            f = ctx.generation(3)
            g = ctx.state("genomes1").reshape(P, L)
            want = ctx.elite_recheck(g, f, k)
            ctx.restore(blob)
        got = ctx.elite_recheck(None, f, k)
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1]), overwrite
    ctx.close()
