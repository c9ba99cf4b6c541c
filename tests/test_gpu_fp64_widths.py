"""FP64 evaluations, unitaries and re-checks on the register-resident and
one-entry-per-lane kernels: every width, discrete and angled gates, lengths
around the chunks of 64, part-filled workgroups, malformed circuits; FP64
against the oracle within 1e-12 (the bar of the other FP64 tests: a few
hundred roundings of 1e-16), FP32 unitaries within 1e-5."""
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


def circuits(rng, n, B, L, angled):
    if angled:
        return inputs.random_ising_circuits(rng, B, n, L, discrete_frac=0.4)
    return inputs.random_circuits(rng, B, n, L, 1), None


def on(dev, g, a):
    return (torch.from_numpy(g.view(np.int16)).to(dev),
            None if a is None else torch.from_numpy(a.view(np.int32)).to(dev))


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 6])
@pytest.mark.parametrize("angled", [False, True])
@pytest.mark.parametrize("L", [1, 33, 64, 65, 140])
def test_fitness_and_unitary(dev, oracle, n, angled, L):
    rng = np.random.default_rng(100 * n + L)
    B = 6
    g, a = circuits(rng, n, B, L, angled)
    T = oracle.unitary(n, inputs.random_target_gates(rng, n, 9, 1))
    gd, ad = on(dev, g, a)
    f, gg, d = qe.eval_fitness_fp64(gd, torch.from_numpy(T).to(dev), n=n, L=L, target_stride=0, want_g=True,
                                    want_delta=True, angles=ad)
    U64 = qe.build_unitary(gd, n, L, precision=1, angles=ad).cpu().numpy()
    U32 = qe.build_unitary(gd, n, L, precision=0, angles=ad).cpu().numpy()
    for b in range(B):
        kw = {} if a is None else dict(angles=a[b])
        ref = oracle.fitness(n, g[b], T, **kw)
        U = oracle.unitary(n, g[b], **kw)
        assert abs((1 - f[b].item()) ** 2 - (1 - ref[0]) ** 2) <= 1e-12
        assert abs(gg[b].item() - ref[1]) <= 1e-12 and abs(d[b].item() - ref[2]) <= 1e-12 * (1 << n)
        assert np.abs(U64[b] - U).max() <= 1e-12
        assert np.abs(U32[b] - U).max() <= 1e-5
    assert qe.device_errors() == 0


@pytest.mark.parametrize("n", [2, 3, 4, 5, 6])
def test_malformed_circuits(dev, n):
    L = 5
    g = np.zeros((6, L), np.uint16)
    g[:, 1] = inputs.desc(inputs.H, 0)
    g[2, 3] = inputs.desc(inputs.CV, 0, 0)                     # control == target
    g[4, 4] = inputs.desc(inputs.NOT, n)                       # no such wire
    gd, _ = on(dev, g, None)
    T = torch.eye(1 << n, dtype=torch.complex128, device=dev)
    f, _, _ = qe.eval_fitness_fp64(gd, T, n=n, L=L, target_stride=0)
    assert torch.isnan(f).cpu().tolist() == [False, False, True, False, True, False]
    assert qe.device_errors() == qe.DEVERR_DESC
    for precision in (0, 1):
        U = torch.view_as_real(qe.build_unitary(gd, n, L, precision=precision))
        bad = torch.isnan(U).reshape(6, -1)
        assert bad.all(1).cpu().tolist() == [False, False, True, False, True, False]
        assert bad.any(1).cpu().tolist() == bad.all(1).cpu().tolist()
        assert qe.device_errors() == qe.DEVERR_DESC


@pytest.mark.parametrize("n,lib", [(2, qe.LIB_NCV), (3, qe.LIB_ISING), (4, qe.LIB_ISING), (5, qe.LIB_ISING),
                                   (6, qe.LIB_NCV), (6, qe.LIB_ISING)])
@pytest.mark.parametrize("mode", [qe.FIT_EQ11, qe.FIT_PHASE_INSENSITIVE])
def test_elite_recheck(dev, oracle, n, lib, mode):
    L, P, I, k = 70, 21, 3, 5                                   # 15 circuits: part-filled workgroups
    rng = np.random.default_rng(n)
    T = np.stack([oracle.unitary(n, inputs.random_target_gates(rng, n, 7, permutation=True)) for _ in range(I)])
    ctx = qe.Context(n, lib, qe.ALG_QEQEA, L, P, I, seed=n, fitness_mode=mode)
    ctx.set_targets(torch.from_numpy(T).to(dev))
    out = ctx.sample_eval(0)
    g, f = out[1], out[-1]
    ang = out[2] if lib == qe.LIB_ISING else None
    idx, f64 = ctx.elite_recheck(g, f, k, angles=ang)
    gh = g.cpu().numpy().view(np.uint16).reshape(I, P, L)
    ah = None if ang is None else ang.cpu().numpy().view(np.uint32).reshape(I, P, L)
    for i in range(I):
        for e in range(k):
            c = int(idx[i, e])
            kw = {} if ah is None else dict(angles=ah[i, c])
            ref = (oracle.fitness if mode == qe.FIT_EQ11 else oracle.fitness_pi)(n, gh[i, c], T[i], **kw)
            ref = ref[0] if hasattr(ref, "__len__") else ref
            assert abs((1 - f64[i, e].item()) ** 2 - (1 - ref) ** 2) <= 1e-12
    ctx.close()
