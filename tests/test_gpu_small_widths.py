"""Widths 1 to 3: the gates that act are gathered at the start of each chunk of 64.
Chunks with none, with all 64 and with gaps at either end, lengths around the chunks,
discrete and angled gates; FP32 within 1e-5 of the oracle (fitness near 1 keeps its
accuracy by the residual form) and FP64 within 1e-12, the bars of the other tests."""
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


@pytest.mark.parametrize("n", [1, 2, 3])
@pytest.mark.parametrize("angled", [False, True])
@pytest.mark.parametrize("L", [1, 2, 63, 64, 65, 128, 130])
def test_gaps(dev, oracle, n, angled, L):
    rng = np.random.default_rng(1000 * n + L)
    B = 9
    if angled:
        g, a = inputs.random_ising_circuits(rng, B, n, L, discrete_frac=0.5)
    else:
        g, a = inputs.random_circuits(rng, B, n, L, inputs.LIB_HT_NCV), None
    g = np.array(g)
    g[0] = 0                                           # nothing acts
    g[1, ::2] = 0
    g[2, : L // 2] = 0
    g[3, L // 2:] = 0
    g[4, :64] = 0
    g[5, 0] = g[5, -1] = 0
    g[6, rng.random(L) < 0.9] = 0                      # (7, 8: every gate)
    T = oracle.unitary(n, inputs.random_target_gates(rng, n, 7, 1 if n > 1 else None, permutation=n == 1))
    gd = torch.from_numpy(g.view(np.int16)).to(dev)
    ad = None if a is None else torch.from_numpy(np.array(a).view(np.int32)).to(dev)
    Td = torch.from_numpy(T).to(dev)
    args = dict(n=n, L=L, target_stride=0, want_g=True, want_delta=True, angles=ad)
    f32 = qe.eval_fitness(gd, Td, **args)
    f64 = qe.eval_fitness_fp64(gd, Td, **args)
    U = qe.build_unitary(gd, n, L, precision=1, angles=ad).cpu().numpy()
    for b in range(B):
        kw = {} if a is None else dict(angles=a[b])
        ref = oracle.fitness(n, g[b], T, **kw)
        assert abs(f32[0][b].item() - ref[0]) <= 1e-5
        assert abs((1 - f64[0][b].item()) ** 2 - (1 - ref[0]) ** 2) <= 1e-12
        assert abs(f64[1][b].item() - ref[1]) <= 1e-12
        assert np.abs(U[b] - oracle.unitary(n, g[b], **kw)).max() <= 1e-12
    assert qe.device_errors() == 0
