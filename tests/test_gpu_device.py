"""Device functions on their own (tests/device/probe.hip, built with the
library): the rounding of the FP32 operand form, which adds up in the energy of
a large system but hides in that of a small one."""
import ctypes

import numpy as np
import pytest

from paper_2506_04055_amd.build import probe_lib

pytestmark = pytest.mark.gpu

U = 2.0 ** -24


@pytest.fixture(scope="module")
def probe():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return ctypes.CDLL(probe_lib())


def dev(a):
    import torch
    return torch.as_tensor(np.ascontiguousarray(a)).cuda()


def ptr(t):
    return ctypes.c_void_p(t.data_ptr())


def unbiased(label, err, ref, terms):
    """The mean error of sums of `terms` products is that of rounding to nearest: each of the roundings is below U of the
    running sum and takes either sign, so the mean over n sums stays within five of its standard deviations U sqrt(terms / n)
    (relative to the sums' RMS; the running sums are no larger than the results on the average)."""
    m, s = err.mean() / np.sqrt((ref ** 2).mean()), np.sqrt((err ** 2).mean() / (ref ** 2).mean())
    tol = 5 * U * np.sqrt(terms / err.size)
    print(f"[measured] {label}: mean error {m:+.1e} (tol {tol:.1e}), rms {s:.1e}", flush=True)
    assert abs(m) <= tol
    assert s <= U * np.sqrt(terms)


@pytest.mark.parametrize("kind", ["centred", "positive", "shifted"])
def test_fp32_products_are_rounded_not_cut(probe, kind):
    n, K = 2048, 128
    rng = np.random.default_rng(5)
    a, b = rng.normal(size=(n, 16, K)) / np.sqrt(K), rng.normal(size=(n, 16, K))
    if kind == "positive":
        a, b = abs(a), abs(b)
    if kind == "shifted":       # the shape of SiLU's outputs
        b = np.where(b > 0, b, 0.1 * b)
    A, B, D = dev(a.astype(np.float32)), dev(b.astype(np.float32)), dev(np.zeros((n, 16, 16), np.float32))
    print(f"[case] products {kind}", flush=True)
    assert probe.probe_products(ptr(A), ptr(B), ptr(D), n) == 0
    ref = A.double().cpu().numpy() @ B.double().cpu().numpy().transpose(0, 2, 1)
    unbiased(f"products {kind}", D.double().cpu().numpy() - ref, ref, K)


@pytest.mark.parametrize("K", [20, 8, 6])
@pytest.mark.parametrize("der", [0, 1])
def test_fp32_filter_is_rounded_not_cut(probe, K, der):
    n, rc = 4096, 5.0
    rng = np.random.default_rng(6)
    A, c = rng.normal(size=(384, K)).astype(np.float32) / np.float32(np.sqrt(K)), rng.normal(size=384).astype(np.float32)
    r = rng.uniform(0.9, rc, n).astype(np.float32)
    dA, dc, dr = dev(A), dev(c), dev(r)
    e, w = dev(np.zeros((n, 32), np.float32)), dev(np.zeros((n, 96), np.float32))
    print(f"[case] filter K={K} der={der}", flush=True)
    assert probe.probe_filter(K, ptr(dA), ptr(dc), ptr(dr), ctypes.c_float(rc), n // 16, der, ptr(e), ptr(w)) == 0
    rows = (np.arange(96) // 32) * 128 + np.arange(96) % 32
    W = np.concatenate([c[rows, None], A[rows]], 1).astype(np.float64)
    ref = e[:, :K + 1].double().cpu().numpy() @ W.T
    unbiased(f"filter K={K} der={der}", w.double().cpu().numpy() - ref, ref, K + 1)


def test_edge_sigmoid_is_divided(probe):
    x = np.concatenate([np.linspace(-80, 80, 400001), np.random.default_rng(7).normal(size=400000),
                        [-1000.0, 1000.0, -100.0, 100.0, 0.0, -np.inf, np.inf, np.nan]]).astype(np.float32)
    X, O = dev(x), dev(np.zeros((x.size, 4), np.float32))
    print("[case] sigmoid", flush=True)
    assert probe.probe_sigmoid(ptr(X), x.size, ptr(O)) == 0
    d, s, silu, dsilu = O.cpu().numpy().T
    with np.errstate(all="ignore"):
        want = (np.float32(1) / d).astype(np.float32)
    print(f"[measured] sigmoid: {(s[:-8] != want[:-8]).mean():.1e} of the quotients differ", flush=True)
    assert np.array_equal(s, want, equal_nan=True)
    # the limits, and what an argument that is no number gives
    assert np.array_equal(silu[-8:-3], [0, 1000, 0, 100, 0]) and np.array_equal(dsilu[-8:-3], [0, 1, 0, 1, 0.5])
    assert silu[-2] == np.inf and not np.isfinite(silu[-3]) and np.isnan(silu[-1]) and np.isnan(dsilu[-1])


@pytest.mark.parametrize("rc", [5.0, 4.7, 6.0])
def test_edge_phase(probe, rc):
    r = np.linspace(0, rc, 1000001).astype(np.float32)
    r = r[r <= np.float32(rc)]
    R, O = dev(r), dev(np.zeros((r.size, 2), np.float32))
    print(f"[case] phase rc={rc}", flush=True)
    assert probe.probe_phase(ptr(R), r.size, ctypes.c_float(rc), ptr(O)) == 0
    th = np.pi * r.astype(np.float64) / np.float64(np.float32(rc))
    err = O.double().cpu().numpy() - np.stack([np.sin(th), np.cos(th)], 1)
    print(f"[measured] phase rc={rc}: mean error of sin, cos {err.mean(0)}, max {abs(err).max():.1e}", flush=True)
    # no offset beyond the series' truncation (2e-9); the series' last sums and the result are rounded once each
    assert abs(err.mean(0)).max() <= 2.5e-9
    assert abs(err).max() <= 2 * U


@pytest.mark.parametrize("F", [64, 128])
def test_row_offsets_at_their_limit(probe, F):
    """The largest system whose rows are reached by 32-bit offsets, and the first that is not."""
    probe.probe_wide.argtypes = [ctypes.c_long, ctypes.c_int]
    n = (2 ** 32 - 1) // (12 * F)
    assert n < 2 ** 24 and not probe.probe_wide(n, F) and probe.probe_wide(n + 1, F)
    assert probe.probe_wide(2 ** 24, 16) and not probe.probe_wide(2 ** 24 - 1, 16)
    rng = np.random.default_rng(1)
    for ld in (F, 3 * F):
        row = np.concatenate([[0, n - 1], rng.integers(0, n, 10000)]).astype(np.int32)
        f = np.concatenate([[0, ld - 1], rng.integers(0, ld, 10000)]).astype(np.int32)
        R, Fe, O = dev(row), dev(f), dev(np.zeros(row.size, np.int64))
        print(f"[case] row offsets F={F} ld={ld}", flush=True)
        assert probe.probe_row_offset(ptr(R), ptr(Fe), row.size, ld, ptr(O)) == 0
        want = 4 * (row.astype(np.int64) * ld + f)
        assert want.max() < 2 ** 32 and np.array_equal(O.cpu().numpy(), want)


@pytest.mark.parametrize("F,K", [(64, 8), (128, 20)])
@pytest.mark.parametrize("adjoint", [0, 1])
def test_message_rows_by_either_offset(probe, F, K, adjoint):
    import torch
    n, rc = 173, 5.0
    rng = np.random.default_rng(2)
    deg = rng.integers(0, 70, n)
    deg[:3] = [0, 16, 70]
    rowc = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    E = int(rowc[-1])
    r = rng.uniform(1.0, rc, E)
    d = rng.normal(size=(E, 3))
    geom = np.concatenate([d / np.linalg.norm(d, axis=1, keepdims=True) * r[:, None], r[:, None]], 1).astype(np.float32)
    rows = lambda *shape: rng.normal(size=shape).astype(np.float32)  # noqa: E731
    host = [rowc, rng.integers(0, n, E).astype(np.int32), geom, rows(n, 3 * F), rows(n, 3 * F), rows(n, F), rows(n, 3 * F),
            rows(n, F), rows(n, 3 * F), rows(3 * F, K), rows(3 * F), rng.integers(0, 3, n).astype(np.int8)]
    data = [dev(h) for h in host]
    ins = (ctypes.c_void_p * len(data))(*[t.data_ptr() for t in data])
    res = []
    for wide in (0, 1):
        out = [torch.zeros(n, 3 * F, device="cuda"), torch.zeros(n, 3 * F, device="cuda"), torch.zeros(E, 4, device="cuda")]
        outs = (ctypes.c_void_p * 3)(*[t.data_ptr() for t in out])
        queue = torch.zeros(2048, dtype=torch.int32, device="cuda")
        torch.cuda.synchronize()
        print(f"[case] message F={F} adjoint={adjoint} wide={wide}", flush=True)
        assert probe.probe_message(wide, adjoint, F, n, ctypes.c_float(rc), 1, ins, outs, ptr(queue)) == 0
        res.append([t.cpu().numpy() for t in out])
    assert all(np.array_equal(a, b) for a, b in zip(*res))
    assert np.abs(res[0][1]).max() > 0 and (not adjoint or np.abs(res[0][2]).max() > 0)
