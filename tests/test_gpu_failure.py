"""Failure paths of the C-ABI that need the device: non-finite numbers reach the
library as FTK_ENUMERIC (a numeric check on the host side of the call, no device
fault), and the context keeps working afterwards."""
import ctypes

import numpy as np
import pytest

from seeded_inputs import SUPERCELLS, gaussian_vector

pytestmark = pytest.mark.gpu

FTK_ENUMERIC = -4


@pytest.fixture(scope="module")
def env():
    import torch

    import paper_1802_02854_amd as ftk
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    ctx = ftk.Context(0)
    h = ftk.Hamiltonian(ctx, ftk.honeycomb_cluster(*SUPERCELLS[12]), -1.0, 0.1)
    return ftk, torch, ctx, h


def _states(ftk, torch, h, g):
    G = torch.from_numpy(np.ascontiguousarray(g).view(np.complex128)).to("cuda").reshape(1, -1)
    return ftk.TypicalStates(h, seed=1, n_vectors=1, betas=[0.0, 1.0], E_b=-2.0, eps=0.1, L=8, M=8, n_steps=12,
                             gaussians=G)


@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf])
def test_non_finite_start_vector_is_enumeric(env, bad):
    """A start vector with one NaN or infinite entry: FTK_ENUMERIC through the C-ABI with a
    message; nothing else happens on the device."""
    ftk, torch, ctx, h = env
    print(f"non-finite start vector {bad}", flush=True)
    g = gaussian_vector(5, 0, 12)
    g[2 * 777 + 1] = bad
    with pytest.raises(ftk.FTKError) as e:
        _states(ftk, torch, h, g)
    assert e.value.status == FTK_ENUMERIC
    assert "norm" in str(e.value)


def test_overflowing_start_vector_is_enumeric(env):
    """Finite entries whose squared norm overflows: FTK_ENUMERIC, not a silent Inf."""
    ftk, torch, ctx, h = env
    g = gaussian_vector(6, 0, 12) * 1e300
    with pytest.raises(ftk.FTKError) as e:
        _states(ftk, torch, h, g)
    assert e.value.status == FTK_ENUMERIC


def test_context_usable_after_numeric_error(env):
    """After the failures above the same context and Hamiltonian give a normal result."""
    ftk, torch, ctx, h = env
    st = _states(ftk, torch, h, gaussian_vector(7, 0, 12))
    ln, nm, em, ep = st.scalars()
    assert np.isfinite(ln).all() and np.isfinite(nm).all() and (nm >= 0).all()
    sp = ftk.Spectrum(h, st, q_xy=[(0.0, 0.0)], omega=np.linspace(-2, 2, 9), eta=0.1, n_steps=12, alpha_mask=4)
    g, r = sp.raw()
    assert np.isfinite(g).all()


def test_direct_c_call_status(env):
    """The raw C entry point returns the status code itself (no Python exception layer)."""
    ftk, torch, ctx, h = env
    from paper_1802_02854_amd import _lib
    g = gaussian_vector(8, 0, 12)
    g[0] = np.nan
    G = torch.from_numpy(g.view(np.complex128)).to("cuda")
    betas = np.array([0.0])
    E_b = np.array([-2.0])
    eps = np.array([0.1])
    p = _lib.TsParamsC(1, 0, 1, betas.ctypes.data, 1, E_b.ctypes.data, eps.ctypes.data, 4, 8, 6, 0.0,
                       G.data_ptr(), 0, 0.0, 0.0, 0)
    out = ctypes.c_void_p()
    rc = _lib.lib().ftk_typical_states(h.handle, ctypes.byref(p), ctypes.byref(out))
    assert rc == FTK_ENUMERIC and not out.value
    assert b"norm" in _lib.lib().ftk_last_error()


# -------------------------------------------------------------------------
class _Pool:
    """A context whose device memory comes from a pool of `limit` bytes (a caller's allocator)."""

    def __init__(self, ftk, torch, limit):
        from paper_1802_02854_amd import _lib
        self.lib, self.limit, self.held, self.refused = _lib, limit, {}, 0

        def alloc(n, _user):
            if sum(t.numel() for t in self.held.values()) + n > self.limit:
                self.refused += 1
                return None
            t = torch.empty(int(n), dtype=torch.uint8, device="cuda")
            self.held[t.data_ptr()] = t
            return t.data_ptr()

        def free(p, _user):
            torch.cuda.synchronize()
            del self.held[p]

        self._cb = _lib.ALLOC_FN(alloc), _lib.FREE_FN(free)
        self.handle = ctypes.c_void_p()
        _lib.call("ftk_ctx_create_with_allocator", 0, None, *self._cb, None, ctypes.byref(self.handle))

    def close(self):
        self.lib.lib().ftk_ctx_destroy(self.handle)


@pytest.mark.parametrize("N,states_mib,spectra_mib", [(8, 6, 2), (12, 24, 12), (14, 56, 32)])
def test_small_clusters_fit_a_small_pool(env, N, states_mib, spectra_mib):
    """A pool that holds the results and the vectors of a sequence or two: 12 (vector, anchor)
    pairs, their spectra (fixed and truncated) and pairs of operators, as from a pool without
    that limit.  Per vector of 2^N entries: 12 x 8 shells stay, a filter run takes 64 + 8."""
    ftk, torch, ctx, _ = env
    print(f"small pool N={N}", flush=True)
    cl = ftk.honeycomb_cluster(*SUPERCELLS[N])
    out = []
    for limit in (states_mib << 20, 1 << 40):
        pool = _Pool(ftk, torch, limit)
        h = ftk.Hamiltonian(pool, cl, -1.0, 0.1)
        st = ftk.TypicalStates(h, seed=3, n_vectors=4, betas=[0.0, 0.5, 1.0], E_b=None, eps=None, L=8, M=16, n_steps=70)
        if limit < 1 << 40:  # the shells, and room for a few sequences
            pool.limit = 12 * 8 * (16 << N) + (spectra_mib << 20)
        res = [*st.scalars()]
        for tol in (0.0, 1e-2):
            sp = ftk.Spectrum(h, st, q_xy=[(0.0, 0.0)], omega=np.linspace(-2, 2, 9), eta=0.3, n_steps=20, rhs_block=1,
                              resid_tol=tol)
            res += [*sp.raw(), sp.norms()]
        ops = [np.stack([ftk.momentum_operator(cl, a, (0.7, -0.4))]) for a in (0, 1)]
        res += ftk.PairSpectrum(h, st, op_a=ops[0], op_b=ops[1], omega=np.linspace(-2, 2, 5), eta=0.3, n_steps=12,
                                rhs_block=1).raw()
        out.append(res)
        assert (pool.refused > 0) == (limit < 1 << 40)
        st.close(), h.close(), pool.close()
        assert not pool.held
    for a, b in zip(*out):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("N", [8, 16])
def test_handles_outlive_their_context(env, N):
    """A Hamiltonian and states used and destroyed after their context was."""
    ftk, torch, _, _ = env
    print(f"destroy order N={N}", flush=True)
    ctx = ftk.Context(0)
    h = ftk.Hamiltonian(ctx, ftk.honeycomb_cluster(*SUPERCELLS[N]), -1.0, 0.1)
    st = ftk.TypicalStates(h, seed=1, n_vectors=1, betas=[0.0], E_b=None, eps=None, L=4, M=4, n_steps=8)
    v = ftk.random_vector(ctx, 3, 0, N)
    w, phi = h.apply(v).cpu(), st.shell(0, 0, 2).cpu()
    ctx.close()
    others = [ftk.Context(0) for _ in range(64)]  # its memory, were it free, has other owners now
    assert torch.equal(h.apply(v).cpu(), w) and torch.equal(st.shell(0, 0, 2).cpu(), phi)
    st.close(), h.close()
    del others
