"""The device bounds checks where clusters of 6 to 14 sites run, and in the H v forms that
only a tuning key selects there.

A child process on the debug library (libftkw_check.so) must report no violation and give the
release library's results bit for bit.  That the resident kernels state their indices at all is
read off their preprocessed source.
"""
import os
import re
import shutil
import subprocess
import sys

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1802_02854_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="needs hipcc")
def test_resident_kernels_state_their_indices():
    """Start-vector gathers (12), own entries (14), LDS partners (15) and carried vectors (16) of
    the debug build's resident kernels are checked; the release build has none of it."""
    def source(*flags):
        r = subprocess.run([HIPCC, "-x", "hip", "--offload-arch=gfx950", "--offload-device-only", "-std=c++17", "-E", "-P",
                            *flags, os.path.join(CSRC, "resident.hip")], capture_output=True, text=True, check=True)
        return r.stdout
    text = source("-DFTK_DEVICE_CHECKS")
    sites = [int(x) for x in re.findall(r"ftk::dchk\(.*?, \((\d+)\)\)", text)]
    assert set(sites) >= {12, 14, 15, 16} and sites.count(14) == 2 and sites.count(15) == 4
    assert "dchk" not in source()


def workload(ftk, torch, ctx):
    out = {}

    def ring(N):
        ij = sorted({(min(i, (i + d) % N), max(i, (i + d) % N)) for d in (1, 2) for i in range(N)})
        xy = np.stack([np.cos(np.arange(N)), np.sin(1.7 * np.arange(N))], axis=1)
        return ftk.Cluster(N, np.array([b[0] for b in ij], np.int32), np.array([b[1] for b in ij], np.int32),
                           (np.arange(len(ij)) % 3).astype(np.int8), xy)

    omega = np.linspace(-3, 3, 41)
    for N in (6, 7, 9, 10, 11, 12, 13, 14):
        h = ftk.Hamiltonian(ctx, ring(N), -1.0, 0.1)
        st = ftk.TypicalStates(h, seed=N, n_vectors=1, betas=[0.0, 0.7], E_b=None, eps=None, L=12, M=4, n_steps=12,
                               block_steps=5)
        out[f"nm{N}"] = st.scalars()[1]
        for tol in (0.0, 1e-2):  # 72 sequences: past the few that run in lockstep
            sp = ftk.Spectrum(h, st, q_xy=[(0.3, 0.1)], omega=omega, eta=0.3, n_steps=20, rhs_block=1, resid_tol=tol)
            out[f"g{N}_{tol}"] = sp.raw()[0]
        op = [np.stack([ftk.momentum_operator(ring(N), a, (0.3, 0.1))]) for a in (0, 1)]
        out[f"pair{N}"] = ftk.PairSpectrum(h, st, op_a=op[0], op_b=op[1], omega=omega, eta=0.3, n_steps=9,
                                           rhs_block=1).raw()[0]
        print(f"  resident N={N}", flush=True)
    for N, variant in ((12, 1), (13, 2), (16, 2)):
        h = ftk.Hamiltonian(ctx, ring(N), -1.0, 0.1)
        ftk.set_tuning("hv_variant", variant)
        try:
            out[f"hv{N}"] = h.apply(ftk.random_vector(ctx, 5, 0, N)).cpu().numpy()
        finally:
            ftk.set_tuning("hv_variant", -1)
    return out


def _child(path):
    import torch

    import paper_1802_02854_amd as ftk
    assert ftk.LIB_PATH.endswith("libftkw_check.so"), ftk.LIB_PATH
    ctx = ftk.Context(0)
    compiled, v, _, _ = ctx.device_checks(clear=True)
    assert compiled and v == 0
    out = workload(ftk, torch, ctx)
    out["violations"] = np.array(ctx.device_checks()[1:])
    np.savez(path, **out)


@pytest.mark.gpu
def test_resident_kernels_stay_in_bounds(tmp_path):
    import torch

    import paper_1802_02854_amd as ftk
    path = str(tmp_path / "checked.npz")
    print("resident checks: child on the debug library", flush=True)
    env = dict(os.environ, FTK_LIBRARY="check", PYTHONPATH=ROOT + os.pathsep + os.environ.get("PYTHONPATH", ""))
    r = subprocess.run([sys.executable, "-u", os.path.abspath(__file__), path], env=env, cwd=ROOT, timeout=300)
    assert r.returncode == 0
    got = dict(np.load(path))
    assert list(got.pop("violations")) == [0, 0, 0]
    print("resident checks: the same workload on the release library", flush=True)
    ref = workload(ftk, torch, ftk.Context(0))
    assert sorted(ref) == sorted(got)
    for k in ref:
        assert np.array_equal(ref[k], got[k]), k


if __name__ == "__main__":
    _child(sys.argv[1])
