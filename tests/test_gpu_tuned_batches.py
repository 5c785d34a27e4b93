"""Spectra and pairs under a tuning record of one sequence per launch, bit for bit with the
batches asked for in turn (which kernel timing keeps)."""
import json

import numpy as np
import pytest

from seeded_inputs import SUPERCELLS

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,shells", [(16, 1), (16, 24), (18, 8), (20, 2), (20, 8)])
def test_a_record_of_single_sequences(tmp_path, monkeypatch, N, shells):
    """3 to 72 sequences (batches of 2 to 32, sizes the block layout has no kernel for among
    them) for rhs_block 0 and 1, read from a tuning file."""
    import torch

    import paper_1802_02854_amd as ftk
    print(f"tuned batches N={N} shells={shells}", flush=True)
    n_omega = 29 + shells  # a key of this test's own
    arch = torch.cuda.get_device_properties(0).gcnArchName.replace(":", "_")
    record = tmp_path / "tune.json"
    record.write_text(json.dumps({f"{arch}/N{N}/w{n_omega}/graph": [1, 1000.0, 0, 0, -1]}))
    monkeypatch.setenv("FTK_TUNE_CACHE", str(record))
    ctx = ftk.Context(0)
    cl = ftk.plan_layout(ftk.honeycomb_cluster(*SUPERCELLS[N]))[0]
    h = ftk.Hamiltonian(ctx, cl, -1.0, 0.1)
    assert h.autotune(n_omega) == (1, 1000.0), "the record was not read"
    st = ftk.TypicalStates(h, seed=4, n_vectors=1, betas=[0.0], E_b=None, eps=None, L=24, M=4, n_steps=8)
    omega = np.linspace(-3, 3, n_omega)
    q = ftk.honeycomb_momenta(*SUPERCELLS[N])[1]
    op_a = np.stack([ftk.momentum_operator(cl, 0, q)])
    op_b = np.stack([ftk.momentum_operator(cl, 1, q)])

    def both(rhs):
        sp = ftk.Spectrum(h, st, q_xy=[(0.0, 0.0)], omega=omega, eta=0.1, n_steps=7, rhs_block=rhs, shells=(0, shells))
        out = [*sp.raw(), sp.norms()]
        if shells == 1:  # 24 shells, 96 sequences
            out += ftk.PairSpectrum(h, st, op_a=op_a, op_b=op_b, omega=omega, eta=0.1, n_steps=5, rhs_block=rhs).raw()
        return out

    ctx.set_timing(True)
    want = both(1)
    ctx.set_timing(False)
    for rhs in (0, 1):
        for x, y in zip(both(rhs), want):
            assert np.array_equal(x, y)
    assert np.abs(want[0]).max() > 0
