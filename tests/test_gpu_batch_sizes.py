"""Batch sizes at which the evaluation takes another layout: width 6 with a column
per lane from 640 circuits on (1024 with angles), mixed widths with one circuit per
workgroup from 4096 on and the sort's general loop above 16384.  Same operations
and order either way, so the results are the same bits; malformed widths included."""
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


@pytest.mark.parametrize("angled", [False, True])
@pytest.mark.parametrize("B", [639, 640, 1023, 1024])
@pytest.mark.parametrize("L", [48, 130])
def test_width_6(dev, angled, B, L):
    rng = np.random.default_rng(B + L)
    a = None
    if angled:
        g, a = inputs.random_ising_circuits(rng, B, 6, L, discrete_frac=0.5)
        a = torch.from_numpy(np.ascontiguousarray(a).view(np.int32)).to(dev)
    else:
        g = inputs.random_circuits(rng, B, 6, L, inputs.LIB_HT_NCV)
    g = torch.from_numpy(np.ascontiguousarray(g).view(np.int16)).to(dev)
    T = qe.build_unitary(torch.from_numpy(inputs.random_circuits(rng, 1, 6, 20, 1).view(np.int16)).to(dev), 6, 20)
    args = dict(n=6, L=L, target_stride=0, want_g=True, want_delta=True, angles=a)
    for x, y in zip(qe.eval_fitness(g, T, **args), qe.eval_fitness(g, T, path=qe.PATH_FP32_LDS, **args)):
        assert torch.equal(x, y)
    assert qe.device_errors() == 0


@pytest.mark.parametrize("B", [4095, 4096, 16384, 16385])
def test_mixed(dev, B):
    rng = np.random.default_rng(B)
    nq = rng.integers(1, 7, size=B).astype(np.int8)
    lens = rng.integers(0, 40, size=B)
    lens[rng.integers(0, B, 5)] = 140
    goff = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    gates = np.zeros(int(goff[-1]), np.uint16)
    owner = np.repeat(nq, lens)
    for n in range(1, 7):
        m = owner == n
        gates[m] = inputs.random_circuits(rng, 1, n, int(m.sum()), inputs.LIB_HT_NCV)[0]
    T = [qe.build_unitary(torch.from_numpy(inputs.random_circuits(rng, 1, n, 8, 1).view(np.int16)).to(dev), n, 8,
                          precision=0).reshape(-1) for n in range(1, 7)]
    off = np.cumsum([0] + [t.numel() for t in T])
    toff = off[nq - 1].astype(np.int64)
    bad = np.array([0, B // 2, B - 1])
    nq[bad] = [0, 9, -3]
    args = dict(nq=torch.from_numpy(nq).to(dev), goff=torch.from_numpy(goff).to(dev),
                toff=torch.from_numpy(toff).to(dev), target_stride=None, want_g=True, want_delta=True)
    gd = torch.from_numpy(gates.view(np.int16)).to(dev)
    out = [qe.eval_fitness(gd, torch.cat(T), workspace=w, **args) for w in (True, False)]
    torch.cuda.synchronize()
    assert qe.device_errors() & qe.DEVERR_WIDTH
    for x, y in zip(*out):
        x, y = x.cpu().numpy(), y.cpu().numpy()
        assert np.array_equal(x, y, equal_nan=True)
        assert np.isnan(x[bad]).all() and np.isnan(x).sum() == len(bad)
