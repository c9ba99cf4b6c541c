"""Rounding error of the FP64 fitness sums.  One column of the product holds all of
its energy, so that the order in which a lane adds its own terms shows.  The
uniform-width kernels may be no further from the exact sum than the one-workgroup
kernel of mixed-width batches, which adds at most four terms in series at width 5
and a binary tree above them (16 in series are 1.19 times as far off there).  The
margin of 1.1 is for the scatter of two root mean squares over 4096 samples, 2 %."""
import numpy as np
import pytest
import torch

from paper_1809_11134_amd import qe

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    qe.load()
    return torch.device("cuda", 0)


@pytest.mark.parametrize("n", [4, 5, 6])
def test_error_of_the_sums(dev, n):
    rng = np.random.default_rng(n)
    B, N = 4096, 1 << n
    # row c of the target is column c of the product; large entries, so that the
    # rest of the residual (N - 1 ones) does not hide their sum's error
    rows = 1e4 * (rng.uniform(0.5, 1, (B, N)) * np.exp(2j * np.pi * rng.uniform(size=(B, N))))
    c = rng.integers(0, N, B)
    T = torch.zeros((B, N, N), dtype=torch.complex128, device=dev)
    T[torch.arange(B, device=dev), torch.from_numpy(c).to(dev)] = torch.from_numpy(rows).to(dev)
    gates = torch.zeros((B, 1), dtype=torch.int16, device=dev)
    m = rows.view(np.float64).reshape(B, N, 2).astype(np.longdouble)
    energy = (m ** 2).sum(2)
    diag = energy[np.arange(B), c]
    off = energy.sum(1) - diag
    exact = ((np.sqrt(diag) - 1) ** 2 + (N - 1) + off) / 2
    _, _, uniform = qe.eval_fitness_fp64(gates, T, n=n, L=1, target_stride=N * N, want_delta=True)
    _, _, mixed = qe.eval_fitness_fp64(gates.reshape(-1), T, goff=torch.arange(B + 1, dtype=torch.int32, device=dev),
                                       nq=torch.full((B,), n, dtype=torch.int8, device=dev),
                                       target_stride=N * N, want_delta=True)

    def rms(d):
        e = (d.cpu().numpy().astype(np.longdouble) - exact) / exact
        return float(np.sqrt((e ** 2).mean()) / 2.0 ** -53)
    u, x = rms(uniform), rms(mixed)
    print(f"n={n}: {u:.3f} against {x:.3f} units of 2^-53")
    assert u <= 1.1 * x
    assert qe.device_errors() == 0
