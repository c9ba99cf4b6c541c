"""Searches whose circuits are longer than what the schedules were tuned on change
their layout by length and number of circuits, unless a schedule was set.  On either
side of each line: the table's choice, the register-resident and the LDS-staged
schedule leave the same fitness and encoding, bit for bit."""
import os
import subprocess
import sys

import pytest
import torch

from paper_1809_11134_amd import inputs, qe

SHAPES = [(4, 2047, 129), (4, 2048, 128), (4, 2048, 129), (5, 512, 64), (5, 512, 65), (5, 513, 65), (5, 513, 129),
          (6, 639, 128), (6, 639, 129), (6, 640, 129), (5, 16, 1000)]


def generations(n, P, L):
    dev = torch.device("cuda", 0)
    g = torch.tensor([[inputs.desc(inputs.CNOT, 0, 1), inputs.desc(inputs.NOT, n - 1)]], dtype=torch.int16, device=dev)
    ctx = qe.Context(n, qe.LIB_NCV, qe.ALG_QEQEA, L, P, prob_mutation=0.3, seed=n + P + L)
    ctx.set_targets(qe.build_unitary(g, n, 2))
    out = [ctx.generation(0), ctx.generation(1)] + [ctx.state(k) for k in ("theta", "qutrit", "best_f")]
    ctx.close()
    return out


def main():
    # (in a process of its own: schedules once set stay set)
    default = {s: generations(*s) for s in SHAPES}
    for lds in (0, 1):
        for n in (4, 5, 6):
            qe.set_schedule(n, lds)
        for s in SHAPES:
            assert all(torch.equal(x, y) for x, y in zip(default[s], generations(*s))), (s, lds)
            print(*s, lds, flush=True)
    assert qe.device_errors() == 0


@pytest.mark.gpu
def test_same_bits_at_the_lines():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-u", os.path.abspath(__file__)], capture_output=True, text=True, timeout=100,
                       env=dict(os.environ, PYTHONPATH=root))
    assert r.returncode == 0, r.stdout[-500:] + r.stderr[-2000:]
    assert len(r.stdout.splitlines()) == 2 * len(SHAPES)


if __name__ == "__main__":
    main()
