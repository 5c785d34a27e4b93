"""Two chains of batches on two streams against one chain, bit for bit."""
import numpy as np
import pytest

from seeded_inputs import SUPERCELLS

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,B,alloc", [(16, 1, None), (16, 4, "torch"), (16, 32, None), (18, 16, None), (20, 4, None)])
def test_two_chains_match_one(N, B, alloc):
    """One to three rounds of two batches, with ragged last ones, against the batches asked for
    in one chain, which kernel timing keeps."""
    import torch

    import paper_1802_02854_amd as ftk
    print(f"chains N={N} B={B}", flush=True)
    ctx = ftk.Context(0, allocator=alloc)
    cl = ftk.plan_layout(ftk.honeycomb_cluster(*SUPERCELLS[N]))[0]
    h = ftk.Hamiltonian(ctx, cl, -1.0, 0.1)
    L = {1: 7, 4: 6, 16: 16, 32: 23}[B]
    st = ftk.TypicalStates(h, seed=2, n_vectors=1, betas=[0.0], E_b=None, eps=None, L=L, M=4, n_steps=8)
    alpha = 4 if B == 1 else 7
    res = []
    for timing in (False, True, False):
        ctx.set_timing(timing)
        for _ in range(2):
            sp = ftk.Spectrum(h, st, q_xy=[(0.0, 0.0)], omega=np.linspace(-3, 3, 40), eta=0.1, n_steps=9, rhs_block=B,
                              alpha_mask=alpha)
            res.append((*sp.raw(), sp.norms()))
            # the caller's own work between the calls
            torch.zeros(1 << 20, device="cuda").add_(1.0)
    ctx.set_timing(False)
    for r in res[1:]:
        for x, y in zip(res[0], r):
            assert np.array_equal(x, y)
    assert np.abs(res[0][0]).max() > 0


@pytest.mark.parametrize("N,B,rows", [(16, 4, 3), (16, 4, 9), (20, 1, 1), (20, 1, 3)])
def test_every_batch_is_timed_as_a_whole(N, B, rows):
    """Kernel timing counts one replayed loop per batch, the first and an only one included, and no
    single steps."""
    import paper_1802_02854_amd as ftk
    print(f"timed batches N={N} B={B} rows={rows}", flush=True)
    ctx = ftk.Context(0)
    h = ftk.Hamiltonian(ctx, ftk.plan_layout(ftk.honeycomb_cluster(*SUPERCELLS[N]))[0], -1.0, 0.1)
    st = ftk.TypicalStates(h, seed=2, n_vectors=1, betas=[0.0], E_b=None, eps=None, L=9, M=4, n_steps=8)
    ctx.set_timing(True)
    ftk.Spectrum(h, st, q_xy=[(0.0, 0.0)], omega=np.linspace(-3, 3, 20), eta=0.1, n_steps=9, rhs_block=B, alpha_mask=4,
                 shells=(0, rows))
    ctx.set_timing(False)
    blocks, ms = ctx.kernel_time("lanczos_block")
    assert blocks == -(-rows // B) and ms > 0
    assert ctx.kernel_time("lanczos_step") == (0, 0.0)


@pytest.mark.parametrize("N,B,rows", [(16, 32, 24), (18, 8, 8), (20, 1, 3)])
def test_a_call_allocates_a_few_times(N, B, rows):
    """A call of two chains takes its memory in a few pieces (results, the vectors of each chain): every
    hipMalloc and hipFree of such buffers costs a good part of a millisecond."""
    import ctypes

    import torch

    import paper_1802_02854_amd as ftk
    from paper_1802_02854_amd import _lib
    print(f"allocations N={N} B={B}", flush=True)
    held, calls = {}, [0]

    class Counted:
        def __init__(self):
            def alloc(n, _user):
                calls[0] += 1
                t = torch.empty(int(n), dtype=torch.uint8, device="cuda")
                held[t.data_ptr()] = t
                return t.data_ptr()

            def free(p, _user):
                torch.cuda.synchronize()
                del held[p]

            self._cb = _lib.ALLOC_FN(alloc), _lib.FREE_FN(free)
            self.handle = ctypes.c_void_p()
            _lib.call("ftk_ctx_create_with_allocator", 0, None, *self._cb, None, ctypes.byref(self.handle))

    ctx = Counted()
    h = ftk.Hamiltonian(ctx, ftk.plan_layout(ftk.honeycomb_cluster(*SUPERCELLS[N]))[0], -1.0, 0.1)
    st = ftk.TypicalStates(h, seed=2, n_vectors=1, betas=[0.0], E_b=None, eps=None, L=24, M=4, n_steps=8)
    before = calls[0]
    ftk.Spectrum(h, st, q_xy=[(0.0, 0.0)], omega=np.linspace(-3, 3, 20), eta=0.1, n_steps=9, rhs_block=B, alpha_mask=4,
                 shells=(0, rows))
    assert calls[0] - before <= 4
    st.close(), h.close()
    _lib.lib().ftk_ctx_destroy(ctx.handle)
    assert not held
