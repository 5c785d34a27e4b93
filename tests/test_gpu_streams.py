"""The streams of a Green's-function call.

A context on a stream of its own that does not synchronise with the null stream runs two chains
of batches while a kernel spins on the null stream (for about 0.4 s).  In a child process:
a process's streams share four hardware queues, and this one has three.
"""
import os
import subprocess
import sys

import numpy as np
import pytest

from seeded_inputs import SUPERCELLS

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def main():
    import time

    import torch

    import paper_1802_02854_amd as ftk
    print("chains beside the null stream", flush=True)
    ctx = ftk.Context(0, allocator="torch")
    h = ftk.Hamiltonian(ctx, ftk.plan_layout(ftk.honeycomb_cluster(*SUPERCELLS[16]))[0], -1.0, 0.1)
    st = ftk.TypicalStates(h, seed=2, n_vectors=1, betas=[0.0], E_b=None, eps=None, L=8, M=4, n_steps=8)

    def spectrum():
        return ftk.Spectrum(h, st, q_xy=[(0.0, 0.0)], omega=np.linspace(-3, 3, 20), eta=0.1, n_steps=9, rhs_block=1,
                            alpha_mask=4).raw()[0]

    def spin(cycles):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        torch.cuda._sleep(int(cycles))
        b.record()
        return a, b

    want = spectrum()
    a, b = spin(1e6)
    torch.cuda.synchronize()
    cycles = 1e6 * 400.0 / a.elapsed_time(b)
    a, b = spin(cycles)
    t0 = time.perf_counter()
    got = spectrum()
    took, spinning = time.perf_counter() - t0, not b.query()
    torch.cuda.synchronize()
    assert a.elapsed_time(b) < 5000
    assert spinning and took < 0.2, f"the call took {took:.3f} s"
    assert np.array_equal(got, want)


@pytest.mark.gpu
def test_chains_do_not_wait_for_the_null_stream():
    print("chains beside the null stream", flush=True)
    env = dict(os.environ, PYTHONPATH=ROOT + os.pathsep + os.environ.get("PYTHONPATH", ""))
    r = subprocess.run([sys.executable, "-u", os.path.abspath(__file__)], env=env, cwd=ROOT, timeout=100)
    assert r.returncode == 0


if __name__ == "__main__":
    main()
