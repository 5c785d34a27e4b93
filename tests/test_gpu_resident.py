"""Whole-sequence kernels of small clusters against the per-step kernels, bit for bit.

The per-step kernels are pinned to the oracle (test_gpu_parity.py); forcing a form of H v
selects them.  Inner products are the double nearest the exact sum in both, so every
coefficient and every output must agree exactly.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch

    import paper_1802_02854_amd as ftk
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return ftk, ftk.Context(0), torch


def _ring(ftk, N):
    """A ring of N sites (any N) with chords to the second and third neighbours (36 bonds at
    N = 12, past the 32 of one parity word), bond types in turn."""
    ij = sorted({(min(i, (i + d) % N), max(i, (i + d) % N)) for d in (1, 2, 3) for i in range(N)})
    xy = np.stack([np.cos(np.arange(N)), np.sin(1.7 * np.arange(N))], axis=1)
    return ftk.Cluster(N, np.array([b[0] for b in ij], np.int32), np.array([b[1] for b in ij], np.int32),
                       (np.arange(len(ij)) % 3).astype(np.int8), xy)


def _both(ftk, fn):
    """fn() on the resident path and on the per-step kernels."""
    out = [fn()]
    ftk.set_tuning("hv_variant", 0)
    try:
        out.append(fn())
    finally:
        ftk.set_tuning("hv_variant", -1)
    return out


@pytest.mark.parametrize("N", [6, 7, 8, 9, 10, 11, 12, 13, 14])
def test_resident_sequences_match_per_step(env, N):
    """Spectra (fixed length, one step, truncated) and operator pairs at every resident size."""
    ftk, ctx, torch = env
    print(f"resident N={N}", flush=True)
    cl = _ring(ftk, N)
    h = ftk.Hamiltonian(ctx, cl, -1.0, 0.13)
    g = torch.Generator(device="cuda")
    g.manual_seed(N)
    draws = torch.view_as_complex(torch.randn(1, 1 << N, 2, dtype=torch.float64, device="cuda", generator=g))
    st = ftk.TypicalStates(h, seed=0, n_vectors=1, betas=[0.5], E_b=None, eps=None, L=3, M=4, n_steps=12, gaussians=draws)
    qs = [(0.0, 0.0), (0.7, -0.4)]
    n = min(40, (1 << N) // 2)  # no breakdown
    for omega, eta, steps, tol, shells in ((np.linspace(-3, 3, 130), 0.3, n, 0.0, (0, 3)),
                                           (np.linspace(-2, 2, 5), 0.3, 1, 0.0, (1, 2)),
                                           (np.linspace(-3, 3, 600), 1.0, n, 1e-2, (0, 3))):
        def spectrum():
            sp = ftk.Spectrum(h, st, q_xy=qs, omega=omega, eta=eta, n_steps=steps, rhs_block=1, resid_tol=tol,
                              shells=shells)
            return [sp.raw(), sp.norms(), [sp.lanczos(0, 0, m, a, q) for m in range(3) for a in range(3) for q in range(2)]]
        a, b = _both(ftk, spectrum)
        assert np.array_equal(a[0][0], b[0][0]) and np.array_equal(a[0][1], b[0][1]) and np.array_equal(a[1], b[1])
        for (al, be), (al2, be2) in zip(a[2], b[2]):
            assert np.array_equal(al, al2) and np.array_equal(be, be2)
        assert np.abs(a[0][0]).max() > 0
    assert any(len(al) < n for al, _ in a[2]), "the truncated run never stopped early"

    op_a = np.stack([ftk.momentum_operator(cl, 0, qs[1]), ftk.momentum_operator(cl, 2, qs[0])])
    op_b = np.stack([ftk.momentum_operator(cl, 1, qs[1]), ftk.momentum_operator(cl, 0, qs[0])])
    a, b = _both(ftk, lambda: ftk.PairSpectrum(h, st, op_a=op_a, op_b=op_b, omega=np.linspace(-3, 3, 33), eta=0.2,
                                               n_steps=n, rhs_block=1).raw())
    for x, y in zip(a, b):
        assert np.array_equal(x, y)


def test_resident_breakdown_and_many_shifts(env):
    """Sequences that exhaust their Krylov space (three separate bonds have four
    energies) end at the same step, and more sequences and shifts than one workgroup's share
    give the per-step results."""
    ftk, ctx, torch = env
    print("resident breakdown", flush=True)
    cl = ftk.Cluster(6, np.array([0, 2, 4], np.int32), np.array([1, 3, 5], np.int32), np.zeros(3, np.int8),
                     np.arange(12.0).reshape(6, 2))
    h = ftk.Hamiltonian(ctx, cl, -1.0, 0.0)
    st = ftk.TypicalStates(h, seed=3, n_vectors=2, betas=[0.0, 1.0], E_b=None, eps=None, L=40, M=4, n_steps=30)
    a, b = _both(ftk, lambda: (lambda sp: [sp.raw(), [sp.lanczos(1, 1, m, 2, 0) for m in range(40)]])(
        ftk.Spectrum(h, st, q_xy=[(0.0, 0.0)], omega=np.linspace(-3, 3, 1100), eta=0.4, n_steps=90, rhs_block=1)))
    steps = [len(al) for al, _ in a[1]]
    assert min(steps) < 90
    assert steps == [len(al) for al, _ in b[1]]
    for (al, be), (al2, be2) in zip(a[1], b[1]):
        assert np.array_equal(al, al2) and np.array_equal(be, be2)
    assert np.array_equal(a[0][0], b[0][0]) and np.array_equal(a[0][1], b[0][1])


@pytest.mark.parametrize("N,nb", [(6, 0), (9, 5), (12, 1), (13, 7), (14, 64)])
def test_resident_filter_runs_match_per_step(env, N, nb):
    """Filtered states of several vectors and anchors (blocks of pass 2 of every size, shell
    moments, per-shell truncation) from the resident filter runs and the per-step ones."""
    ftk, ctx, torch = env
    print(f"resident filter N={N} nb={nb}", flush=True)
    h = ftk.Hamiltonian(ctx, _ring(ftk, N), -1.0, 0.07)
    n = 23
    for tol in (0.0, 0.5):
        def states():
            st = ftk.TypicalStates(h, seed=5, n_vectors=2, betas=[0.0, 0.4, 1.5], E_b=None, eps=None, L=11, M=4, n_steps=n,
                                   block_steps=nb, shell_moments=True, resid_tol=tol)
            return [*st.scalars(), *st.moments(), *st.window(),
                    *[x for s in range(2) for a in range(3) for x in st.lanczos(s, a)],
                    *[st.shell(s, a, m).cpu().numpy() for s in range(2) for a in range(3) for m in (0, 5, 10)]]
        for x, y in zip(*_both(ftk, states)):
            assert np.array_equal(x, y)


def test_more_sequences_than_a_grid_has_rows(env):
    """70656 sequences of 6 sites in one call (a grid's y extent ends at 65535) against the
    same in three calls."""
    ftk, ctx, torch = env
    print("resident rows", flush=True)
    cl = ftk.honeycomb_cluster((1, 1), (-1, 2))
    h = ftk.Hamiltonian(ctx, cl, -1.0, 0.1)
    st = ftk.TypicalStates(h, seed=6, n_vectors=23, betas=[0.0], E_b=None, eps=None, L=256, M=2, n_steps=6)
    qs = [(0.0, 0.0), (0.7, -0.4), (1.1, 0.3), (-0.2, 0.9)]

    def spectrum(first, n):
        sp = ftk.Spectrum(h, st, q_xy=qs, omega=np.array([-0.4, 0.9]), eta=0.2, n_steps=3, rhs_block=1, shells=(first, n))
        return sp.raw()[0][:, :, first:first + n], sp.work()[1]

    whole, n_seq = spectrum(0, 256)
    assert n_seq > 65535
    parts = [spectrum(f, n)[0] for f, n in ((0, 100), (100, 100), (200, 56))]
    assert np.array_equal(whole, np.concatenate(parts, axis=2)) and np.abs(whole).max() > 0


@pytest.mark.parametrize("N", [4, 5, 6, 7, 8])
def test_every_rhs_block_of_the_smallest_clusters(env, N):
    """Batches of 2 to 16 sequences whose entries together are fewer than a wavefront of the block
    layout takes (4 to 8 sites on the per-step kernels), against one sequence at a time."""
    ftk, ctx, torch = env
    print(f"smallest clusters N={N}", flush=True)
    ij = [(i, i + 1) for i in range(N - 1)]
    cl = ftk.Cluster(N, np.array([b[0] for b in ij], np.int32), np.array([b[1] for b in ij], np.int32),
                     (np.arange(N - 1) % 3).astype(np.int8), np.stack([np.arange(N) * 1.0, np.sin(np.arange(N))], axis=1))
    h = ftk.Hamiltonian(ctx, cl, -1.0, 0.3)
    st = ftk.TypicalStates(h, seed=2, n_vectors=1, betas=[0.0], E_b=None, eps=None, L=6, M=4, n_steps=6)
    ftk.set_tuning("hv_variant", 0)
    try:
        out = [ftk.Spectrum(h, st, q_xy=[(0.2, 0.1)], omega=np.linspace(-2, 2, 11), eta=0.3, n_steps=5, rhs_block=B).raw()
               for B in (1, 0, 2, 4, 8, 16)]
    finally:
        ftk.set_tuning("hv_variant", -1)
    assert np.isfinite(out[0][0]).all() and np.abs(out[0][0]).max() > 0
    for g, r in out[1:]:
        assert np.array_equal(g, out[0][0]) and np.array_equal(r, out[0][1])
