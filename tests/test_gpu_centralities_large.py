"""Vertex measures around the size at which the trace is summed by the whole GPU, against numpy in
64 bits; calls whose outputs cannot hold the partial sums (none given, or in place over the
diagonal) give the same measures.

Tolerance: the trace is a sum of n positive terms through trees of depth at most 16 + 12 + 10, so
its relative error is below 38 units of 2^-53; each measure adds a handful of operations: 1e-13.
"""
import ctypes

import numpy as np
import pytest
import torch

from paper_2006_13679_amd import api

pytestmark = pytest.mark.gpu
TOL = 1e-13


def _want(d):
    n, tr = len(d), float(np.sum(d.astype(np.longdouble)))
    far = n * d + tr
    return dict(farness=far, closeness=(n - 1) / far, nrwb=1.0 / n + tr / ((n - 1) * far), trace=tr, kirchhoff=n * tr)


@pytest.mark.parametrize("n", [16383, 16384, 16385, 20480, 20481, 1_000_003])
def test_measures(n):
    d = np.random.default_rng(n).random(n) + 0.01
    got, want = api.centralities(torch.from_numpy(d).cuda()), _want(d)
    for key in ("farness", "closeness", "nrwb"):
        np.testing.assert_allclose(got[key].cpu().numpy(), want[key], rtol=TOL, atol=0)
    assert abs(got["trace"] - want["trace"]) <= TOL * want["trace"]
    assert abs(got["kirchhoff"] - want["kirchhoff"]) <= TOL * want["kirchhoff"]


@pytest.mark.parametrize("outputs", ["none", "in place", "in place and one more"])
def test_outputs_that_cannot_hold_partial_sums(outputs):
    n = 40_001
    d = np.random.default_rng(1).random(n) + 0.01
    want = _want(d)
    diag = torch.from_numpy(d).cuda()
    clo = torch.empty_like(diag)
    sc = torch.empty(2, dtype=torch.float64, device="cuda")
    ptr = lambda t: None if t is None else ctypes.c_void_p(t.data_ptr())  # noqa: E731
    far = None if outputs == "none" else diag
    close = clo if outputs.endswith("more") else None
    rc = api.lib().ustd_centralities(n, ptr(diag), ptr(far), ptr(close), None, ptr(sc),
                                     ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == api.OK
    torch.cuda.synchronize()
    assert abs(float(sc[0]) - want["trace"]) <= TOL * want["trace"]
    if far is not None:
        np.testing.assert_allclose(diag.cpu().numpy(), want["farness"], rtol=TOL, atol=0)
    if close is not None:
        np.testing.assert_allclose(clo.cpu().numpy(), want["closeness"], rtol=TOL, atol=0)
