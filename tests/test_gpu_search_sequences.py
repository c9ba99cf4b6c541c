"""Contexts with the shared-slot search (more than 524288 entries) keep the words and
mutation decisions of two generations.  Sequences in which they go stale: skipped and
repeated generations, graph replays between single generations, a fused first half
completed either way, a step-by-step update that writes the decisions of another
generation's words over, checkpoints restored in mid-sequence.  Fitness and encoding
equal those of step-by-step calls, which use no words, bit for bit."""
import numpy as np
import pytest
import torch

from paper_1809_11134_amd import inputs, qe

pytestmark = pytest.mark.gpu
FIELDS = ("theta", "qutrit", "best_f", "best_theta", "best_qutrit")


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    qe.load()
    return torch.device("cuda", 0)


class Search:
    """One context, and the fitness of each generation run."""

    def __init__(self, dev, oracle, lib, pm=0.4, n=3, I=512, P=33, L=32):
        rng = np.random.default_rng(11)
        few = torch.from_numpy(np.stack([oracle.unitary(n, inputs.random_target_gates(rng, n, 8, permutation=True))
                                         for _ in range(4)])).to(dev)
        assert I * P * L > 524288
        self.ctx = qe.Context(n, lib, qe.ALG_QEQEA, L, P, I, prob_mutation=pm, seed=77)
        self.ctx.set_targets(few[torch.arange(I, device=dev) % 4])
        self.dev, self.ising, self.f = dev, lib == qe.LIB_ISING, []

    def steps(self, *gens):
        for gen in gens:
            slots, g, *a = self.ctx.sample(gen)
            a = a[0] if self.ising else None
            f = self.ctx.eval_population(g, angles=a)
            self.ctx.update(gen, slots, g, f, angles=a)
            self.f.append(f)
        return self

    def one(self, *gens):
        self.f += [self.ctx.generation(gen) for gen in gens]
        return self

    def graph(self, first, count):
        hist = torch.empty((count, self.ctx.circuits), dtype=torch.float32, device=self.dev)
        self.ctx.run_graph(first, count, hist)
        self.f += list(hist)
        return self

    def halves(self, gen, with_slots):
        slots, g, *rest = self.ctx.sample_eval(gen)
        self.ctx.update(gen, slots if with_slots else None, g, rest[-1], angles=rest[0] if self.ising else None)
        self.f.append(rest[-1])
        return self

    def decisions(self):
        return self.ctx.state("mutation_masks").reshape(2, -1)

    def same(self, other):
        assert len(self.f) == len(other.f)
        for j, (x, y) in enumerate(zip(self.f, other.f)):
            assert torch.equal(x, y), j
        for k in FIELDS:
            assert torch.equal(self.ctx.state(k), other.ctx.state(k)), k
        self.ctx.close()
        other.ctx.close()
        assert qe.device_errors() == 0


LIBS = pytest.mark.parametrize("lib", [qe.LIB_NCV, qe.LIB_ISING])


@LIBS
def test_search_is_active(dev, oracle, lib):
    # its update leaves the next generation's decisions (the others leave that mask empty)
    s = Search(dev, oracle, lib).one(0)
    assert s.decisions()[1].any() and not torch.equal(*s.decisions())
    s.steps(2)                       # (writes the decisions of generation 2 over those of 0)
    want = s.decisions()[0].clone()
    t = Search(dev, oracle, lib).one(1)
    assert torch.equal(t.decisions()[0], want)
    small = Search.__new__(Search)
    small.ctx = qe.Context(3, lib, qe.ALG_QEQEA, 32, 32, 512, prob_mutation=0.4, seed=77)
    small.ctx.set_targets(torch.eye(8, dtype=torch.complex128, device=dev).repeat(512, 1, 1))
    small.ctx.generation(0)
    assert small.decisions()[0].any() and not small.decisions()[1].any()
    for c in (s, t, small):
        c.ctx.close()


@LIBS
def test_calls_in_one_sequence(dev, oracle, lib):
    a = Search(dev, oracle, lib)
    a.graph(0, 2).halves(2, False).one(3).halves(5, False).graph(6, 2).graph(10, 1).one(11, 13).halves(14, True)
    a.one(15).graph(15, 3).one(2, 4)
    b = Search(dev, oracle, lib)
    b.steps(0, 1, 2, 3, 5, 6, 7, 10, 11, 13, 14, 15, 15, 16, 17, 2, 4)
    a.same(b)


@LIBS
def test_step_overwrites_other_words_decisions(dev, oracle, lib):
    # generation 3 leaves the words and decisions of 4; the step-by-step update of 2
    # writes its own decisions in their place, and 4 has to search again; likewise
    # with a graph, and with the step of the very generation whose words are there
    a = Search(dev, oracle, lib)
    a.one(3).steps(2).one(4).one(5).steps(8).graph(6, 2).steps(8).one(9).one(10)
    b = Search(dev, oracle, lib)
    b.steps(3, 2, 4, 5, 8, 6, 7, 8, 9, 10)
    a.same(b)


@LIBS
def test_restore_in_mid_sequence(dev, oracle, lib):
    a = Search(dev, oracle, lib).one(0, 1, 2)
    blob = a.ctx.checkpoint()
    a.one(3, 4)
    a.ctx.restore(blob)              # (words of 5 and 4 stay; 3's are gone)
    a.one(3).one(4)
    _, g, *rest = a.ctx.sample_eval(5)
    a.ctx.restore(blob)              # (between the halves: the second is refused)
    with pytest.raises(qe.QeError) as refused:
        a.ctx.update(5, None, g, rest[-1], angles=rest[0] if a.ising else None)
    assert refused.value.status == qe.QE_ERR_STATE
    a.graph(3, 2).steps(5).one(6)
    b = Search(dev, oracle, lib).steps(0, 1, 2)
    mid = b.ctx.checkpoint()
    b.steps(3, 4)
    b.ctx.restore(mid)
    b.steps(3, 4)
    b.ctx.restore(mid)
    b.steps(3, 4, 5, 6)
    a.same(b)
