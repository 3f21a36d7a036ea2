"""Operators in a workspace smaller than nfs_workspace_bytes asks for: down to
the size with the solves' split counts (what every operator once took, and
what a solve's workspace holds) a call runs with fewer splits and stays inside
it; below that it is refused.  Against the FP64 formulas at each precision's
usual bars."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu
BAR = {"fp32": 1e-4, "fp16": 2e-3, "bf16": 4e-3}


def _size(h, pr, op, prec, n_iter=0):
    from paper_2604_09233_amd import nfs

    n = ctypes.c_size_t()
    assert nfs.lib().nfs_workspace_bytes(h, ctypes.byref(pr.st), nfs.OPS[op], nfs.PRECISIONS[prec], n_iter, 0,
                                         ctypes.byref(n)) == 0
    return n.value


def _least(pr, prec):
    """Sizes of E, EH and EHE in a context whose shapes are pinned to the solves'
    (of bf16 for fp32: same operand sizes, no room for the one-pass gradient)."""
    from paper_2604_09233_amd import nfs

    prec = "bf16" if prec == "fp32" else prec
    L, p = nfs.lib(), nfs.PRECISIONS[prec]
    h = ctypes.c_void_p()
    assert L.nfs_create(ctypes.byref(h), 0) == 0
    for op in (0, 1):
        mt, ns = ctypes.c_int(), ctypes.c_int()
        assert L.nfs_tuned_shape(h, ctypes.byref(pr.st), p, op, ctypes.byref(mt), ctypes.byref(ns)) == 0
        assert L.nfs_set_shape(h, ctypes.byref(pr.st), p, op, mt.value, ns.value) == 0
    out = {op: _size(h, pr, op, prec) for op in ("E", "EH", "EHE")}
    assert L.nfs_destroy(h) == 0
    return out


@pytest.mark.parametrize("prec", ["fp32", "fp16", "bf16"])
@pytest.mark.parametrize("L,K,G,P", [(4200, 5000, 12, 5), (3000, 2500, 20, 3), (700, 9000, 33, 17), (2100, 300, 4, 0),
                                     (40, 30, 2, 20)])
def test_operators_in_a_smaller_workspace(prec, L, K, G, P):
    from paper_2604_09233_amd import nfs

    d = synth.random_problem(L, K, G, P, seed=31, phase_scale=10.0)
    a = (d["sens"], d["fields"], d["b0"], d["kcoef"], d["t"])
    pr = nfs.Problem(*a)
    h, lib, p = nfs.context(0), nfs.lib(), nfs.PRECISIONS[prec]
    rho, m = torch.from_numpy(d["rho"]).cuda(), torch.from_numpy(d["m"]).cuda()
    least, cg = _least(pr, prec), _size(h, pr, "CG", prec)
    y = oracle.apply_E(d["rho"].astype(np.complex128), *a)
    x = oracle.apply_EH(d["m"].astype(np.complex128), *a)
    gk = np.stack([np.imag(np.sum(d["m"] * np.conj(oracle.apply_E(d["fields"][b] * d["rho"].astype(np.complex128), *a)),
                                  axis=0)) for b in range(P)], 1) if P else None
    ref = dict(E=y, EH=x, EHE=oracle.apply_EH(y, *a), BACK=gk)

    def call(op, nbytes):
        ws = torch.full((nbytes + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
        off = (-ws.data_ptr()) % 256
        out = torch.empty((G, K) if op == "E" else (K, P) if op == "BACK" else L, device="cuda",
                          dtype=torch.float32 if op == "BACK" else torch.complex64)
        v = lambda t: ctypes.c_void_p(t.data_ptr())  # noqa: E731
        w = (p, ctypes.c_void_p(ws.data_ptr() + off), nbytes, pr._stream())
        if op == "BACK":
            rc = lib.nfs_encode_backward(h, ctypes.byref(pr.st), v(rho), v(m), None, None, v(out), *w)
        else:
            f = dict(E=lib.nfs_apply_E, EH=lib.nfs_apply_EH, EHE=lib.nfs_apply_EHE)[op]
            rc = f(h, ctypes.byref(pr.st), v(m if op == "EH" else rho), v(out), *w)
        assert torch.all(ws[off + nbytes:] == 0x5A)
        return rc, out.cpu().numpy()

    for op in ("E", "EH", "EHE", "BACK") if P else ("E", "EH", "EHE"):
        kind = "EHE" if op == "BACK" else op
        full = _size(h, pr, kind, prec)
        for n in {full, (full + least[kind]) // 512 * 256, least[kind], max(cg, least[kind])}:
            rc, got = call(op, n)
            e = np.linalg.norm(got - ref[op]) / np.linalg.norm(ref[op]) if rc == 0 else np.nan
            print(f"{op} {prec} L={L} K={K} G={G} P={P}: {n} of {full} bytes, rc {rc}, rel {e:.1e}")
            assert rc == 0 and e < BAR[prec]


def test_less_than_the_solves_counts_is_refused():
    from paper_2604_09233_amd import nfs

    d = synth.random_problem(4200, 5000, 12, 0, seed=32)
    pr = nfs.Problem(*(d[k] for k in ("sens", "fields", "b0", "kcoef", "t")))
    ws = torch.empty(1 << 26, dtype=torch.uint8, device="cuda")
    off = (-ws.data_ptr()) % 256
    v = lambda t: ctypes.c_void_p(t.data_ptr())  # noqa: E731
    rho = torch.zeros(4200, dtype=torch.complex64, device="cuda")
    for op, n in _least(pr, "fp16").items():
        f = dict(E=nfs.lib().nfs_apply_E, EH=nfs.lib().nfs_apply_EH, EHE=nfs.lib().nfs_apply_EHE)[op]
        out = torch.empty(12 * 5000, dtype=torch.complex64, device="cuda")
        src = out if op == "EH" else rho
        assert f(nfs.context(0), ctypes.byref(pr.st), v(src), v(out.clone()), nfs.PRECISIONS["fp16"],
                 ctypes.c_void_p(ws.data_ptr() + off), n - 256, pr._stream()) == nfs.NFS_EWORKSPACE
