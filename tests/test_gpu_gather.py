"""H v with one element per thread, all rows in one launch, and the two-launch Lanczos step
built on it, bit for bit against the forms they stand in for."""
import numpy as np
import pytest

from seeded_inputs import SUPERCELLS

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch

    import paper_1802_02854_amd as ftk
    return ftk, ftk.Context(0), torch


def _forced(ftk, mode, f):
    ftk.set_tuning("hv_variant", mode)
    try:
        return f()
    finally:
        ftk.set_tuning("hv_variant", -1)


@pytest.mark.parametrize("N,rows,pad,layout", [(6, 3, 5, False), (8, 1, 0, True), (12, 5, 64, False), (16, 3, 7, False),
                                               (18, 2, 0, True)])
def test_rows_in_one_launch(env, N, rows, pad, layout):
    """Rows a padded stride apart; the padding of the output is left alone."""
    ftk, ctx, torch = env
    print(f"gather rows N={N} rows={rows}", flush=True)
    cl = ftk.honeycomb_cluster(*SUPERCELLS[N])
    h = ftk.Hamiltonian(ctx, ftk.plan_layout(cl)[0] if layout else cl, -1.0, 0.1)
    v = torch.randn(rows, (1 << N) + pad, dtype=torch.complex128, generator=torch.Generator().manual_seed(N)).cuda()
    v = v[:, :1 << N]

    def apply():
        base = torch.full((rows, (1 << N) + pad), 7.0 + 0j, dtype=torch.complex128, device="cuda")
        h.apply(v, out=base[:, :1 << N])
        torch.cuda.synchronize()
        return base.cpu()
    a = apply()
    for mode in (1, 2, 3):  # as many of them as the size has
        assert torch.equal(a, _forced(ftk, mode, apply))
    if pad:
        assert bool((a[:, 1 << N:] == 7.0).all())
    assert bool((a[:, :1 << N].abs().sum(1) > 0).all())


@pytest.mark.parametrize("N,B,n,tol", [(16, 1, 1, 0.0), (16, 1, 14, 0.0), (16, 8, 9, 0.0), (16, 4, 40, 1e-3), (18, 2, 7, 0.0)])
def test_two_launch_steps(env, N, B, n, tol):
    """Green's sequences, the last batch ragged, and the filter runs before them."""
    ftk, ctx, torch = env
    print(f"pairs N={N} B={B} n={n} tol={tol}", flush=True)
    cl = ftk.plan_layout(ftk.honeycomb_cluster(*SUPERCELLS[N]))[0]

    def run():
        h = ftk.Hamiltonian(ctx, cl, -1.0, 0.1)
        st = ftk.TypicalStates(h, seed=3, n_vectors=1, betas=[0.0, 1.0], E_b=None, eps=None, L=3, M=4, n_steps=11)
        sp = ftk.Spectrum(h, st, q_xy=[(0.0, 0.0)], omega=np.linspace(-3, 3, 30), eta=0.3, n_steps=n, rhs_block=B,
                          resid_tol=tol, alpha_mask=3)
        return (*st.scalars(), *sp.raw(), sp.norms())
    two = run()
    for x, y in zip(two, _forced(ftk, 3, run)):
        assert np.array_equal(x, y)
    assert np.abs(two[-2]).max() > 0


@pytest.mark.parametrize("N", [13, 14])
def test_few_and_many_sequences(env, N):
    """More sequences than run in lockstep (one workgroup each) and few, each row the same."""
    ftk, ctx, torch = env
    print(f"few N={N}", flush=True)
    ij = sorted({(min(i, (i + d) % N), max(i, (i + d) % N)) for d in (1, 2, 3) for i in range(N)})
    cl = ftk.Cluster(N, np.array([b[0] for b in ij], np.int32), np.array([b[1] for b in ij], np.int32),
                     (np.arange(len(ij)) % 3).astype(np.int8), np.arange(2.0 * N).reshape(N, 2) ** 0.5)
    h = ftk.Hamiltonian(ctx, cl, -1.0, 0.07)
    st = {}
    for nv in (17, 2):  # 34 filter sequences, 4
        st[nv] = ftk.TypicalStates(h, seed=4, n_vectors=nv, betas=[0.0, 0.8], E_b=None, eps=None, L=9, M=4, n_steps=8,
                                   block_steps=3)
    for s in range(2):
        for a in range(2):
            for x, y in zip(st[17].lanczos(s, a), st[2].lanczos(s, a)):
                assert np.array_equal(x, y)
            for m in (0, 4, 8):
                assert np.array_equal(st[17].shell(s, a, m).cpu().numpy(), st[2].shell(s, a, m).cpu().numpy())
    kw = dict(q_xy=[(0.3, 0.1)], omega=np.linspace(-3, 3, 40), eta=0.2, n_steps=21, rhs_block=1)
    many = ftk.Spectrum(h, st[2], **kw)  # 2 x 2 x 9 x 3 = 108
    few = ftk.Spectrum(h, st[2], shells=(3, 2), **kw)  # 24
    for s in range(2):
        for a in range(2):
            for al in range(3):
                for x, y in zip(many.lanczos(s, a, 3, al, 0), few.lanczos(s, a, 3, al, 0)):
                    assert np.array_equal(x, y)
    assert np.array_equal(many.raw()[0][:, :, 3], few.raw()[0][:, :, 3]) and np.abs(few.raw()[0]).max() > 0


@pytest.mark.parametrize("N,L,shells", [(8, 12, (2, 3)), (16, 4, (1, 1))])
def test_cocg_batches(env, N, L, shells):
    """Shifted COCG sequences in lockstep, the last batch ragged: the rows of another batching
    and of the form with work vectors, spectra and operator pairs."""
    ftk, ctx, torch = env
    print(f"cocg batches N={N}", flush=True)
    cl = ftk.honeycomb_cluster(*SUPERCELLS[N])
    h = ftk.Hamiltonian(ctx, cl, -1.0, 0.1)
    st = ftk.TypicalStates(h, seed=6, n_vectors=1, betas=[0.3], E_b=None, eps=None, L=L, M=4, n_steps=10)
    kw = dict(omega=np.linspace(-2, 2, 600), eta=0.3, n_steps=25, solver="cocg")
    qs = [(0.0, 0.0), (0.4, 0.2)]

    def spectrum(shells=None):
        sp = ftk.Spectrum(h, st, q_xy=qs, shells=shells, seed_tol=1e-3, **kw)
        return sp.raw(), [sp.cocg(0, 0, m, a, q) for m in range(shells[0], sum(shells)) for a in range(3) for q in (0, 1)] \
            if shells else [sp.cocg(0, 0, m, a, q) for m in range(L) for a in range(3) for q in (0, 1)]
    op_a = np.stack([ftk.momentum_operator(cl, 0, qs[1])])
    op_b = np.stack([ftk.momentum_operator(cl, 2, qs[0])])

    def pair():
        return ftk.PairSpectrum(h, st, op_a=op_a, op_b=op_b, **kw).raw()
    many, few = spectrum(), spectrum(shells)  # 8 sites: 72 sequences, 18
    other, pairs = _forced(ftk, 1, spectrum), (pair(), _forced(ftk, 1, pair))
    for x, y in zip(many[0], other[0]):
        assert np.array_equal(x, y)
    for m, o in zip(many[1], other[1]):
        assert m[3] == o[3] and all(np.array_equal(x, y) for x, y in zip(m[:3], o[:3]))
    for m, o in zip(many[1][shells[0] * 6:], few[1]):
        assert m[3] == o[3] and all(np.array_equal(x, y) for x, y in zip(m[:3], o[:3]))
    for x, y in zip(*pairs):
        assert np.array_equal(x, y)
    assert np.abs(many[0][0]).max() > 0 and np.abs(pairs[0][0]).max() > 0


@pytest.mark.parametrize("N,M,n,L", [(8, 2, 6, 9), (8, 64, 150, 300), (14, 6, 37, 11), (18, 4, 9, 17)])
def test_shells_do_not_depend_on_their_number(env, N, M, n, L):
    """Shell coefficients in one go and in slabs of their work space (300 shells of 64 contour
    points and 150 steps), whole and partial shell groups, both widths of the accumulation;
    8 sites also against the host's coefficients on the regenerated Krylov basis."""
    ftk, ctx, torch = env
    print(f"shells N={N} L={L}", flush=True)
    cl = ftk.honeycomb_cluster(*SUPERCELLS[N])
    h = ftk.Hamiltonian(ctx, cl, -1.0, 0.1)
    few = 5
    kw = dict(seed=8, n_vectors=1, betas=[0.2], E_b=-3.0, eps=0.02, M=M, n_steps=n, block_steps=6)
    a = ftk.TypicalStates(h, L=L, **kw)
    b = ftk.TypicalStates(h, L=few, **kw)
    for m in range(few):
        assert torch.equal(torch.view_as_real(a.shell(0, 0, m)), torch.view_as_real(b.shell(0, 0, m)))
    al, be = a.lanczos(0, 0)
    assert np.abs(a.shell(0, 0, L - 1).cpu().numpy()).max() > 0
    if N == 8:
        # all shells lie in the Krylov space of the first steps: sum_k c_k <v_j|v_k> = c_j
        c = ftk.filter_coefficients(al, be, 1.0, -3.0, 0.02, L, M)
        n2 = np.array([float((a.shell(0, 0, m).abs() ** 2).sum()) for m in range(L)])
        ratio = n2 / np.maximum((np.abs(np.asarray(c).reshape(L, -1)[:, :len(al)]) ** 2).sum(1), 1e-300)
        if n < 20:  # before the basis loses orthogonality, eps per step and term
            assert np.allclose(ratio, ratio[0], rtol=1e-11)


@pytest.mark.parametrize("nv,betas", [(1, [0.0, 0.7]), (3, [0.4])])
def test_filter_runs_side_by_side(env, nv, betas):
    """16 sites: the filter sequences of several (vector, anchor) pairs in lockstep, in groups
    of two where the memory allowance asks for it, against one after the other."""
    ftk, ctx, torch = env
    print(f"side by side nv={nv}", flush=True)
    h = ftk.Hamiltonian(ctx, ftk.plan_layout(ftk.honeycomb_cluster(*SUPERCELLS[16]))[0], -1.0, 0.1)

    def states(nb):
        st = ftk.TypicalStates(h, seed=9, n_vectors=nv, betas=betas, E_b=None, eps=None, L=7, M=4, n_steps=105,
                               block_steps=nb, shell_moments=True)
        sa = [(s, a) for s in range(nv) for a in range(len(betas))]
        return [*st.scalars(), *st.moments(), *st.window(), *[x for p in sa for x in st.lanczos(*p)],
                *[st.shell(*p, m).cpu().numpy() for p in sa for m in range(7)]]
    two = [states(10), states(100)]  # 100: two pairs to a group
    for one in (two[1], _forced(ftk, 3, lambda: states(10))):
        for x, y in zip(two[0], one):
            assert np.array_equal(x, y)
