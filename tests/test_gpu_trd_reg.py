"""Register-resident tridiagonalisation at the edges of its configurations: orders around every
change of columns per lane, of waves per matrix and of one to several workgroups, odd orders (the
exchange words' alignment) and several matrices at once.

The reduction is backward stable in fp32: the computed spectrum is that of a matrix within a few
sqrt(n) 2^-24 ||C|| of the Gram (measured 0.5 to 3e-7), asserted at 1e-6; eigenvectors satisfy
||C u - lambda u|| within 1e-5 ||C||, thirty times that.
"""
import threading

import numpy as np
import pytest
import torch

import paper_2607_12550_amd as J
from gpu_util import compress, ctx, device_cells, note, workspace

pytestmark = pytest.mark.gpu


def _cells(T, n):
    rng = np.random.default_rng(T)
    k = rng.standard_normal((4, T, 8)) @ rng.standard_normal((8, 64))
    return [k + 0.3 * (i + 1) * rng.standard_normal((4, T, 64)) for i in range(n)]


def _gram(x):
    X2 = x.transpose(1, 0, 2).reshape(x.shape[1], -1)
    return X2 @ X2.T


@pytest.mark.parametrize("T", [1, 2, 3, 63, 64, 65, 128, 129, 255, 256, 257, 273, 384, 385, 522, 576, 577, 768, 769, 1001, 1024])
def test_spectrum_and_factor(T):
    n = 3 if T < 700 else 2
    xs, ex, desc = device_cells(_cells(T, n), "f32")
    ws = workspace(desc, n)
    note("jolt_spectrum T", T, "cells", n)
    E, lam, _ = J.jolt_spectrum(ctx(), desc, xs, None, None, ws)
    r = min(16, T)
    compress(xs, desc, [J.Params(r, 8, 4, 32, J.JOLT_FACTOR_F32, 0, i) for i in range(n)], dict(reuse=1), ws)
    for c in range(n):
        C = _gram(ex[c])
        want = np.linalg.eigvalsh(C)[::-1]
        got = np.asarray(lam)[c][:T]
        assert np.abs(got - np.maximum(want, 0)).max() <= 1e-6 * want[0]
        U = torch.empty((T, r), device="cuda")
        J.jolt_debug_export(ctx(), 0, c, U)
        U = U.cpu().numpy().astype(np.float64)
        assert np.abs(C @ U - U * got[:r]).max() <= 1e-5 * want[0]
        assert np.abs(U.T @ U - np.eye(r)).max() <= 1e-5


# batches in registers of more workgroups than the chip holds at once (512, 320), and batches of
# more rounds than stay there, which go to one workgroup per matrix
@pytest.mark.parametrize("T, n", [(450, 64), (700, 20), (300, 72), (577, 50)])
def test_batches_larger_than_the_chip(T, n):
    """Spectra spread over batches of several rounds of workgroups, every matrix a differently
    scaled copy of one of two, match the oracle's (a mix-up between matrices would show)."""
    base = _cells(T, 2)
    lam0 = [np.linalg.eigvalsh(_gram(x.astype(np.float32).astype(np.float64)))[::-1] for x in base]
    scale = [1.0 + i / 64.0 for i in range(n)]
    xs, ex, desc = device_cells([base[i % 2] * scale[i] for i in range(n)], "f32")
    note("jolt_spectrum T", T, "cells", n)
    lam = np.array(J.jolt_spectrum(ctx(), desc, xs, None, None, workspace(desc, n))[1])
    for i in range(n):
        # 1e-6 for the reduction and 2^-23 for the rounding of the scaled copies
        want = lam0[i % 2] * scale[i] ** 2
        assert np.abs(lam[i][:T] - np.maximum(want, 0)).max() <= 1.2e-6 * want[0], i


def test_exchange_that_gives_up_is_reported():
    """A wait bound of zero (JOLT_DBG_BULGE_SPIN, forced from the host) ends the exchange between
    workgroups at its first unanswered poll; every wave still ends normally and the call reports
    JOLT_E_NOCONV, as for the bulge chase.  The default bound succeeds again."""
    xs, ex, desc = device_cells(_cells(300, 2), "f32")
    c2 = J.jolt_create(0)
    try:
        ws = workspace(desc, 2)
        J.jolt_debug_set(c2, J.JOLT_DBG_BULGE_SPIN, 0)
        note("exact spectrum, exchange forced to give up")
        with pytest.raises(J.JoltError) as e:
            J.jolt_spectrum(c2, desc, xs, None, None, ws)
        assert e.value.code == J.JOLT_E_NOCONV
        J.jolt_debug_set(c2, J.JOLT_DBG_BULGE_SPIN, 1 << 24)
        E, lam, _ = J.jolt_spectrum(c2, desc, xs, None, None, ws)
        want = np.linalg.eigvalsh(_gram(ex[0]))[::-1]
        assert np.abs(np.asarray(lam)[0][:300] - want).max() <= 1e-6 * want[0]
    finally:
        J.jolt_destroy(c2)


@pytest.mark.parametrize("T", [257, 400, 577, 768, 769, 1024])
def test_matrices_left_to_one_workgroup(T):
    """JOLT_DBG_TRD_GATHER = 0 leaves every matrix whose workgroups would have to run at once to
    the one-workgroup reduction: spectra and factors meet the same bounds (the spectra are not
    those of the register kernel bit for bit, so that the setting cannot have gone unnoticed)."""
    xs, ex, desc = device_cells(_cells(T, 2), "f32")
    ws = workspace(desc, 2)
    c2 = J.jolt_create(0)
    try:
        note("jolt_spectrum T", T, "in registers, then left")
        E, default, _ = J.jolt_spectrum(c2, desc, xs, None, None, ws)
        default = np.array(default)
        J.jolt_debug_set(c2, J.JOLT_DBG_TRD_GATHER, 0)
        E, lam, _ = J.jolt_spectrum(c2, desc, xs, None, None, ws)
        r = 16
        p = [J.Params(r, 8, 4, 32, J.JOLT_FACTOR_F32, 0, i) for i in range(2)]
        blobs = [torch.zeros(J.jolt_compressed_size(desc, q), dtype=torch.uint8, device="cuda") for q in p]
        J.jolt_compress(c2, desc, xs, p, dict(reuse=1), ws, blobs)
        assert np.any(np.array(lam) != default)
        for c in range(2):
            C = _gram(ex[c])
            want = np.linalg.eigvalsh(C)[::-1]
            got = np.asarray(lam)[c][:T]
            assert np.abs(got - np.maximum(want, 0)).max() <= 1e-6 * want[0]
            U = torch.empty((T, r), device="cuda")
            J.jolt_debug_export(c2, 0, c, U)
            U = U.cpu().numpy().astype(np.float64)
            assert np.abs(C @ U - U * got[:r]).max() <= 1e-5 * want[0]
            assert np.abs(U.T @ U - np.eye(r)).max() <= 1e-5
        for bad in (-1, (1 << 24) + 1):
            with pytest.raises(J.JoltError):
                J.jolt_debug_set(c2, J.JOLT_DBG_TRD_GATHER, bad)
    finally:
        J.jolt_destroy(c2)


def test_two_contexts_side_by_side():
    """Two contexts reduce batches of more workgroups than the chip holds at the same time, each
    from a thread and on a stream of its own: both succeed with the spectra that the same call
    gives alone (to the bound of both reductions, as a matrix may be left to one workgroup)."""
    T, n = 300, 48
    base = _cells(T, 2)
    xs, ex, desc = device_cells([base[i % 2] * (1.0 + i / 64.0) for i in range(n)], "f32")
    alone = np.array(J.jolt_spectrum(ctx(), desc, xs, None, None, workspace(desc, n))[1])
    want = np.linalg.eigvalsh(_gram(ex[n - 1]))[::-1]
    assert np.abs(alone[n - 1][:T] - want).max() <= 1e-6 * want[0]
    torch.cuda.synchronize()
    got, failed = {}, []

    def work(k):
        try:
            c2, st = J.jolt_create(0), torch.cuda.Stream()
            ws = workspace(desc, n)
            torch.cuda.synchronize()
            for rep in range(4):
                note("two contexts, thread", k, "pass", rep)
                got[k, rep] = np.array(J.jolt_spectrum(c2, desc, xs, None, None, ws, stream=st)[1])
            J.jolt_destroy(c2)
        except Exception as e:      # reported by the test below, not lost with the thread
            failed.append(e)

    threads = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failed and len(got) == 8
    for lam in got.values():
        assert (np.abs(lam - alone).max(axis=1) <= 2e-6 * alone[:, 0]).all()
