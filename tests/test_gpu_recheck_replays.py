"""The circuits that a GA re-check without gates takes are those of the last
generation that ran on the stream, also when the calls were captured: graphs of
single generations replayed in any order, one captured re-check after each, and a
captured update that writes over the genomes.  Population sizes with one child, an
odd last child and several workgroups; uniform and mixed populations."""
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


def captured(fn):
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        out = fn()
    return g, out


@pytest.mark.parametrize("mixed,P", [(False, 1), (False, 2), (False, 33), (False, 700), (True, 33), (True, 64)])
def test_recheck_follows_replays(dev, oracle, mixed, P):
    rng = np.random.default_rng(P)
    k, widths, lengths = min(P, 5), [3, 5, 4], [9, 30, 70]
    if mixed:
        ctx = qe.Context(0, qe.LIB_NCV, qe.ALG_GA, 0, P, seed=P, ga_gene_mutation_prob=0.1, widths=widths,
                         lengths=lengths)
    else:
        widths = [4, 4]
        ctx = qe.Context(4, qe.LIB_NCV, qe.ALG_GA, 12, P, 2, seed=P, ga_gene_mutation_prob=0.1)
    ctx.set_targets(torch.cat([torch.from_numpy(oracle.unitary(n, inputs.random_target_gates(rng, n, 6, 0))).reshape(-1)
                               for n in widths]).to(dev))
    f = torch.empty(ctx.circuits, dtype=torch.float32, device=dev)
    for gen in (0, 1):                               # (modules loaded before the captures)
        ctx.generation(gen, f)
    gates = ctx.sample(2)[1]
    ctx.elite_recheck(None, f, k)
    torch.cuda.synchronize()
    runs = [captured(lambda p=p: ctx.generation(2 + p, f))[0] for p in (0, 1)]
    recheck, got = captured(lambda: ctx.elite_recheck(None, f, k))
    update, _ = captured(lambda: ctx.update(3, None, gates, f))      # (writes the genomes of parity 0)
    for p in (0, 1, 0, 0, 1, 1, 0):
        circuits = ctx.sample(2 + p)[1].clone()
        runs[p].replay()
        want = ctx.elite_recheck(circuits, f, k)
        recheck.replay()
        torch.cuda.synchronize()
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1]), p
        eager = ctx.elite_recheck(None, f, k)
        assert torch.equal(eager[1], want[1]), p
        if p == 0:
            update.replay()
            eager = ctx.elite_recheck(None, f, k)
            assert torch.equal(eager[1], want[1])
    # and the library's own graph, whose last generation has the other parity
    hist = torch.empty((3, ctx.circuits), dtype=torch.float32, device=dev)
    for first in (0, 1):
        ctx.run_graph(first, 2)
        circuits = ctx.sample(first)[1].clone()      # (three generations from here on)
        ctx.run_graph(first, 1, hist[:1])
        want = ctx.elite_recheck(circuits, hist[0], k)
        got1 = ctx.elite_recheck(None, hist[0], k)
        assert torch.equal(got1[1], want[1]), first
    ctx.close()
