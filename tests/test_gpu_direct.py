"""GPU tests of the direct route's kernels (csrc/direct.hip) at the sizes where they can go wrong:
edges of the 32-key blocks and of the row tiles, feature counts around the 16-feature steps and the
compiled step counts, column tiles and passes of v, row tiles split over work-groups, powers of two
that differ by far more than fp16 holds, what two fp16 terms do not hold at all (opposed queries and
keys, small weights beside large values, values and denominators far apart), and elements that are
not finite; and of the direct backward likewise.

Tolerance: 2e-5 of a row's largest entry.  z is a ratio of sums of positive weights (PRF, elu + 1):
its error is at most twice the relative error of a weight phi(q).phi(k) c plus that of a value.  A
weight carries the errors of two phi (the exponent, of size up to 2^5, is rounded to 2^-24 of its
terms in each of d / 16 partial sums of the projection: below 2^-19 in all), three products per
term (2^-22) and fp32 sums over m features (2^-24 sqrt(m)): below 2^-17 = 7.6e-6; doubled, 1.5e-5.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2106_12566_amd import synth
from parity_util import rownorm_err, sample_rows, to_gpu

pytestmark = pytest.mark.gpu

TOL = 2e-5


def _check(lib, d, nprf=False, features="prf", causal=False, rows=64):
    wl = d["workload"]
    B, H, n = wl.B, d["H"], wl.n
    W = None if features == "elu" else d["W"]
    print(f"direct {wl.name} {wl.qkv_dtype} {wl.bias} {features} nprf={nprf}", flush=True)
    q, k, v = (to_gpu(d[x], wl.qkv_dtype) for x in ("q", "k", "v"))
    z = lib.attention_fwd(q, k, v, to_gpu(d["b"]), None if W is None else to_gpu(W), nprf=nprf, features=features,
                          route="direct", causal=causal).cpu().numpy()
    assert np.all(np.isfinite(z))
    sel = sample_rows(B, H, n, min(rows, B * H * n), seed=n, extra=[(0, 0, i) for i in (31, 32, 127, 128) if i < n])
    ref, _ = oracle.attention_rows(d["q"], d["k"], d["v"], d["b"], W, sel, nprf=nprf, kind=features)
    err = rownorm_err(np.stack([z[s] for s in sel]), ref)
    print(f"  row-normwise error {err:.3e}", flush=True)
    assert err <= TOL, err
    return z


@pytest.mark.parametrize("B,H,n,d,m,dt,bias", [
    (1, 1, 1, 1, 1, "f32", "normal"),
    (1, 2, 31, 8, 16, "f32", "causal"),
    (2, 1, 32, 31, 17, "bf16", "normal"),
    (1, 2, 33, 32, 33, "f32", "decay"),
    (1, 1, 127, 33, 64, "f32", "causal"),
    (3, 1, 129, 64, 65, "bf16", "causal"),
    (1, 8, 257, 65, 97, "f32", "normal"),      # two column passes; XCD order of the work-groups
    (1, 1, 640, 128, 129, "f32", "decay"),     # four column tiles, 12 k steps, d = 128
    (1, 2, 500, 100, 200, "bf16", "normal"),   # 16 k steps
    (1, 1, 300, 63, 256, "f32", "causal"),     # 16 k steps, fp32 values, columns not a multiple of 4
    (1, 1, 2049, 64, 128, "f32", "normal"),    # row tiles split into parts
    (1, 1, 3000, 40, 48, "bf16", "causal"),    # parts of unequal spans
    (2, 16, 1000, 64, 128, "f32", "decay"),
])
def test_direct_edges(gpu_lib, B, H, n, d, m, dt, bias):
    _check(gpu_lib, synth.custom(B, H, n, d, m, seed=5 + n, qkv_dtype=dt, bias=bias), causal=bias == "causal")


@pytest.mark.parametrize("features,n,d,m", [("trf", 130, 20, 15), ("trf", 333, 64, 128), ("elu", 200, 33, 33),
                                            ("elu", 90, 128, 128), ("prf", 70, 96, 40)])
def test_direct_feature_maps(gpu_lib, features, n, d, m):
    _check(gpu_lib, synth.custom(1, 2, n, d, m, seed=n, bias="decay", bias_sigma=0.3), nprf=True, features=features)


def test_direct_powers_far_apart(gpu_lib):
    """Keys and queries whose sizes differ by far more than fp16 holds inside one 32-key block (phi(k)
    from 2^-103 to 2^7), and the values of one block from the others' (within a block:
    test_direct_values_far_apart): each position's features carry a power of their own, so the
    first rows of a causal mask, which see only small ones, keep their accuracy (row 0 is v_0
    whatever its weight).  The exponents of phi reach 2^7 here, where their rounding is eight times
    that of the other tests."""
    B, H, n, d, m = 1, 1, 200, 16, 32
    dd = synth.custom(B, H, n, d, m, seed=9, bias="causal", qk_scale=0.5)
    for i in range(0, n, 7):
        dd["k"][..., i, :] *= 6.0
        dd["q"][..., i, :] *= 3.0
    dd["k"][..., 0, :] = 2.0
    dd["v"][..., 64:96, :] *= 2.0 ** 30
    z = gpu_lib.attention_fwd(*(to_gpu(dd[x]) for x in ("q", "k", "v", "b", "W")), route="direct",
                              causal=True).cpu().numpy()
    ref, _ = oracle.attention(dd["q"], dd["k"], dd["v"], dd["b"], dd["W"])
    assert np.all(np.isfinite(z))
    np.testing.assert_allclose(z[0, 0, 0], dd["v"][0, 0, 0], rtol=1e-6)
    err = rownorm_err(z, ref)
    print(f"powers far apart: {err:.3e}", flush=True)
    assert err <= 8 * TOL, err


@pytest.mark.parametrize("n,d,m,offset,kw", [
    (100, 64, 64, -85.5, {}), (70, 20, 16, -86.0, {}), (1300, 40, 128, -85.5, {}),
    (100, 64, 40, -85.5, {"features": "trf", "nprf": True}), (150, 33, 8, -86.0, {"features": "trf", "nprf": True}),
    (100, 48, 48, -85.5, {"features": "elu"}),
])
def test_direct_weights_small(gpu_lib, n, d, m, offset, kw):
    """A bias near the end of fp32's range (c = exp(b) of 2^-123): z does not depend on the scale of c."""
    dd = synth.custom(1, 2, n, d, m, seed=n, bias="normal", bias_sigma=0.2)
    dd["b"] = (dd["b"] + np.float32(offset)).astype(np.float32)
    print(f"weights small n={n} d={d} m={m} {kw}", flush=True)
    z = gpu_lib.attention_fwd(*(to_gpu(dd[x]) for x in ("q", "k", "v", "b", "W")), route="direct", **kw).cpu().numpy()
    ref, _ = oracle.attention(dd["q"], dd["k"], dd["v"], dd["b"], dd["W"], nprf=kw.get("nprf", False),
                              kind=kw.get("features", "prf"))
    err = rownorm_err(z, ref)
    print(f"  {err:.3e}", flush=True)
    # (c itself is an fp32 number of 2^-123 and up, normal: rounded to 2^-24)
    assert err <= TOL, err


@pytest.mark.parametrize("mask", ["causal", "window"])
def test_direct_keys_hidden(gpu_lib, mask):
    """Keys whose features are 2^-117 beside one, in their block but hidden from the first rows, that is
    2^11: the rows that see only the small ones keep them."""
    n, d, m = 80, 16, 32
    dd = synth.custom(1, 1, n, d, m, seed=17, bias="normal", bias_sigma=0.3, qk_scale=0.3)
    t = np.arange(-(n - 1), n)
    dd["b"][:, t > 0] = -np.inf
    if mask == "window":
        dd["b"][:, t < -3] = -np.inf
    W = dd["W"][0].astype(np.float64)
    u = np.zeros(d)
    u[0] = 1.0
    for j in range(5):
        # |k|^2 / 2 - max_l w_l.k = 81 (e^-81 is 2^-117)
        g = float(np.max(W @ u))
        dd["k"][0, 0, j] = ((g + np.sqrt(g * g + 2 * 81.0)) * u).astype(np.float32)
        dd["k"][0, 0, j, 1:] += 0.01 * (j + 1)
    dd["k"][0, 0, 5] = (W[3] * (np.sqrt(2 * 8.5) / np.linalg.norm(W[3]))).astype(np.float32)
    ref, _ = oracle.attention(dd["q"], dd["k"], dd["v"], dd["b"], dd["W"])
    z = gpu_lib.attention_fwd(*(to_gpu(dd[x]) for x in ("q", "k", "v", "b", "W")), route="direct",
                              causal=True).cpu().numpy()
    assert np.all(np.isfinite(z))
    err = rownorm_err(z, ref)
    print(f"keys hidden {mask}: {err:.3e}", flush=True)
    # (exponents of phi near 2^7, as in test_direct_powers_far_apart)
    assert err <= 8 * TOL, err


@pytest.mark.parametrize("dt,features", [("f32", "prf"), ("bf16", "prf"), ("f32", "trf")])
def test_direct_weights_far_apart(gpu_lib, dt, features):
    """Rows in which a small weight meets a large value: entries of P 2^24 to 2^40 below the row's largest
    in the block, with values as much larger, count as much in z as the others.  Positive weights and
    values: element by element."""
    n, d, m = 96, 64, 64
    dd = synth.custom(1, 2, n, d, m, seed=23, qkv_dtype=dt, bias="normal", bias_sigma=0.2)
    v = 1.0 + np.random.default_rng(23).random((1, 2, n, d))
    t = np.arange(-(n - 1), n)
    dd["b"] = dd["b"].copy()
    # row i weighs key j by 2^(e_{j - i}); values grow with j as the weights fall
    dd["b"] += (-t * np.log(2.0) * 1.25).astype(np.float32)
    v = (v * 2.0 ** (1.25 * np.arange(n))[:, None]).astype(np.float32)
    if dt == "bf16":
        v = torch.from_numpy(v).to(torch.bfloat16).float().numpy()
    dd["v"] = v
    # (TRF of unit rows that are nearly alike: S = phi(q).phi(k) is near its largest, m of the amplitudes' product)
    nprf = features == "trf"
    if nprf:
        dd["q"], dd["k"] = (np.float32(1.0) + np.float32(0.1) * dd[x] for x in ("q", "k"))
    ref, _ = oracle.attention(dd["q"], dd["k"], v, dd["b"], dd["W"], nprf=nprf, kind=features)
    z = gpu_lib.attention_fwd(to_gpu(dd["q"], dt), to_gpu(dd["k"], dt), to_gpu(v, dt), to_gpu(dd["b"]), to_gpu(dd["W"]),
                              route="direct", nprf=nprf, features=features).cpu().numpy()
    err = float(np.max(np.abs(z - ref) / np.abs(ref)))
    print(f"weights far apart {dt}: {err:.3e}", flush=True)
    assert err <= TOL, err


@pytest.mark.parametrize("dt,n,d,features,nprf,bias", [
    ("bf16", 100, 64, "prf", False, "causal"), ("f32", 100, 64, "prf", False, "causal"),
    ("bf16", 70, 33, "trf", True, "decay"), ("f32", 200, 128, "elu", False, "causal"),
    ("bf16", 2100, 24, "prf", True, "causal"),  # row tiles in parts
])
def test_direct_values_far_apart(gpu_lib, dt, n, d, features, nprf, bias):
    """Values within one 32-key block whose sizes differ by more than fp16 terms with one power hold, by
    key and by column: each is in the results of the rows that see it.  Weights and values are
    positive (TRF under NPRF: nearly), so every element of z is a sum without cancellation and TOL,
    a bound on the relative error of each weight and value, holds element by element."""
    m = d if features == "elu" else 32
    dd = synth.custom(1, 2, n, d, m, seed=n + d, qkv_dtype=dt, bias=bias, bias_sigma=0.3)
    rng = np.random.default_rng([n, d])
    v = 1.0 + rng.random((1, 2, n, d))
    v[..., ::3] *= 2.0 ** -36  # whole columns
    for j, e in ((5, 40), (17, -33), (37, 44), (50, 30), (n - 2, 35)):
        v[:, :, j] *= 2.0 ** e
    v = v.astype(np.float32)
    if dt == "bf16":
        v = torch.from_numpy(v).to(torch.bfloat16).float().numpy()
    dd["v"] = v
    q, k, vv, b = to_gpu(dd["q"], dt), to_gpu(dd["k"], dt), to_gpu(v, dt), to_gpu(dd["b"])
    W = None if features == "elu" else to_gpu(dd["W"])
    print(f"values far apart {dt} n={n} d={d} {features}", flush=True)
    z = gpu_lib.attention_fwd(q, k, vv, b, W, nprf=nprf, features=features, route="direct",
                              causal=bias == "causal").cpu().numpy()
    ref, _ = oracle.attention(dd["q"], dd["k"], v, dd["b"], None if W is None else dd["W"], nprf=nprf, kind=features)
    if bias == "causal":  # row 0 is v_0, row 4 does not see the large values behind it
        np.testing.assert_allclose(z[:, :, 0], v[:, :, 0], rtol=TOL)
    rel = np.abs(z - ref) / np.abs(ref)
    err = float(np.max(rel))
    print(f"  elementwise {err:.3e} at {np.unravel_index(np.argmax(rel), rel.shape)}", flush=True)
    assert err <= TOL, err


@pytest.mark.parametrize("dt,n,d,parts", [("f32", 100, 64, False), ("bf16", 160, 40, False), ("f32", 2100, 24, True)])
def test_direct_values_not_finite(gpu_lib, dt, n, d, parts):
    """An infinite or NaN value reaches its column of the rows that see it and nothing else."""
    dd = synth.custom(1, 1, n, d, 32, seed=n, qkv_dtype=dt, bias="causal")
    q, k, v, b, W = (to_gpu(dd[x], dt) if x in "qkv" else to_gpu(dd[x]) for x in ("q", "k", "v", "b", "W"))
    clean = gpu_lib.attention_fwd(q, k, v, b, W, route="direct", causal=True).cpu().numpy()
    vi = v.clone()
    j0, j1, j2 = n // 3, n // 2, n - 2
    vi[0, 0, j0, 3] = float("inf")
    vi[0, 0, j1, 5] = float("-inf")
    vi[0, 0, j2, 7] = float("nan")
    z = gpu_lib.attention_fwd(q, k, vi, b, W, route="direct", causal=True).cpu().numpy()
    want = np.zeros_like(clean, dtype=bool)
    want[0, 0, j0:, 3] = want[0, 0, j1:, 5] = want[0, 0, j2:, 7] = True
    assert np.all(z[0, 0, j0:, 3] == np.inf) and np.all(z[0, 0, j1:, 5] == -np.inf)
    assert np.all(np.isnan(z[0, 0, j2:, 7]))
    # elsewhere only the elements themselves left the sums, where no row sees them: equal to 2e-5
    scale = np.max(np.abs(clean), axis=-1, keepdims=True)
    assert np.max(np.where(want, 0.0, np.abs(np.where(want, 0.0, z) - clean)) / scale) <= TOL


@pytest.mark.parametrize("dt,d,m,n", [("f32", 64, 130, 200), ("bf16", 33, 20, 40), ("f32", 128, 64, 129)])
def test_features_not_finite(gpu_lib, dt, d, m, n):
    """An infinite or enormous element of x, or of W, reaches the features it is in: phi = 0 where
    W x - |x|^2 / 2 is -inf, NaN only where the formula's terms are of both signs."""
    dd = synth.custom(1, 1, n, d, m, seed=d, qkv_dtype=dt)
    x, W = dd["q"].copy(), dd["W"].copy()
    W[W == 0] = 0.1
    clean = gpu_lib.feature_map(to_gpu(x, dt), to_gpu(W)).cpu().numpy()
    big = float(np.float32(3.3895e38))  # (bf16's largest)
    for j, v in ((3, np.inf), (n - 1, -np.inf), (35, big), (7, np.nan)):
        x[0, 0, j, d - 2] = v
    if dt == "bf16":
        x = torch.from_numpy(x).to(torch.bfloat16).float().numpy()
    xt = torch.from_numpy(x).to(torch.bfloat16).cuda() if dt == "bf16" else to_gpu(x)
    phi = gpu_lib.feature_map(xt, to_gpu(W)).cpu().numpy()
    up = W[0, :, d - 2] > 0
    assert np.all(np.isnan(phi[0, 0, 3, up])) and np.all(phi[0, 0, 3, ~up] == 0)
    assert np.all(np.isnan(phi[0, 0, n - 1, ~up])) and np.all(phi[0, 0, n - 1, up] == 0)
    assert np.all(np.isnan(phi[0, 0, 7]))
    assert np.all((phi[0, 0, 35] == 0) | ((np.abs(W[0, :, d - 2]) > 1) & np.isnan(phi[0, 0, 35])))
    rest = np.setdiff1d(np.arange(n), [3, 7, 35, n - 1])
    np.testing.assert_allclose(phi[:, :, rest], clean[:, :, rest], rtol=TOL)
    W[0, 5, 1] = -np.inf
    got = gpu_lib.feature_map(to_gpu(dd["q"], dt), to_gpu(W)).cpu().numpy()
    want = np.where(dd["q"][..., 1:2] > 0, 0.0, np.where(dd["q"][..., 1:2] < 0, np.inf, np.nan))[..., 0]
    np.testing.assert_array_equal(got[..., 5], want.astype(np.float32))
    others = [l for l in range(m) if l != 5]
    np.testing.assert_allclose(got[..., others], clean[..., others], rtol=TOL)
    # a key whose every feature is zero has no weight
    W = -np.abs(dd["W"]).astype(np.float32)
    W[W == 0] = -0.1
    k, kz = dd["k"].copy(), dd["k"].copy()
    k[0, 0, 9, 0], kz[0, 0, 9, 0] = np.inf, 1e4
    kt = torch.from_numpy(k).to(torch.bfloat16).cuda() if dt == "bf16" else to_gpu(k)
    z = gpu_lib.attention_fwd(to_gpu(dd["q"], dt), kt, to_gpu(dd["v"], dt), to_gpu(dd["b"]), to_gpu(W), route="direct")
    ref, _ = oracle.attention(dd["q"], kz, dd["v"], dd["b"], W)
    assert rownorm_err(z.cpu().numpy(), ref) <= TOL


def _opposed(d, scale, kind, mask, n=200, m=128, dt="f32"):
    """Queries and keys for which every product phi_l(q) phi_l(k) a row sums pairs a large feature with
    one far below its position's largest: k = -q, a common direction with `kind`'s share of noise, or
    independent draws (where a mask leaves a row few keys, some rows see only such ones)."""
    dd = synth.custom(1, 2, n, d, m, seed=d + int(100 * scale) + n, qkv_dtype=dt)
    rng = np.random.default_rng([n, d, int(100 * scale)])
    draw = lambda *shape: (scale * rng.standard_normal(shape)).astype(np.float32)
    q = draw(1, 2, n, d)
    if kind == "opposite":
        k = -q
    elif kind == "aligned":
        u = draw(1, 2, 1, d)
        q, k = u + 0.1 * q, -u + 0.1 * draw(1, 2, n, d)
    else:
        k = draw(1, 2, n, d)
    if dt == "bf16":
        q, k = (torch.from_numpy(x).to(torch.bfloat16).float().numpy() for x in (q, k))
    dd["q"], dd["k"] = np.ascontiguousarray(q), np.ascontiguousarray(k)
    t = np.arange(-(n - 1), n)
    if mask == "causal":
        dd["b"][:, t > 0] = -np.inf
    elif mask == "window":
        dd["b"][:, np.abs(t) > 2] = -np.inf
    return dd


OPPOSED = [
    (64, 0.8, "aligned", "none", 200, 128, "f32"), (64, 1.0, "aligned", "none", 130, 128, "f32"),
    (64, 1.0, "aligned", "causal", 200, 64, "bf16"), (64, 1.0, "aligned", "window", 97, 200, "f32"),
    (128, 0.6, "aligned", "none", 200, 128, "f32"), (128, 0.6, "aligned", "causal", 33, 256, "bf16"),
    (64, 0.8, "opposite", "window", 200, 128, "f32"), (64, 1.0, "opposite", "causal", 160, 16, "f32"),
    (64, 1.2, "random", "causal", 300, 128, "f32"), (64, 1.2, "random", "window", 300, 128, "bf16"),
    (31, 1.0, "aligned", "none", 129, 40, "f32"), (64, 1.0, "aligned", "none", 2050, 128, "f32"),  # (row tiles in parts)
]


@pytest.mark.parametrize("d,scale,kind,mask,n,m,dt", OPPOSED)
def test_direct_opposed(gpu_lib, d, scale, kind, mask, n, m, dt):
    """Rows whose S is below what two fp16 terms hold: they keep the accuracy of the others, on the
    default route too.  Exponents of phi are up to 2^6 to 2^7 here (norms up to d^(1/2) and more), up to
    twice those that TOL is derived from; the rows are the exact features' (fp32 sums over d), so
    the bound is 2 TOL."""
    dd = _opposed(d, scale, kind, mask, n, m, dt)
    print(f"opposed d={d} scale={scale} {kind} {mask} n={n} m={m} {dt}", flush=True)
    q, k, v, b, W = (to_gpu(dd[x], dt) if x in "qkv" else to_gpu(dd[x]) for x in ("q", "k", "v", "b", "W"))
    ref, _ = oracle.attention(dd["q"], dd["k"], dd["v"], dd["b"], dd["W"])
    for route in ("auto", "direct"):
        z = gpu_lib.attention_fwd(q, k, v, b, W, route=route, causal=mask == "causal").cpu().numpy()
        assert np.all(np.isfinite(z))
        err = rownorm_err(z, ref)
        print(f"  {route}: {err:.3e}", flush=True)
        assert err <= 2 * TOL, err


@pytest.mark.parametrize("B,H,n,d,m,dt", [(1, 12, 64, 64, 64, "f32"), (2, 4, 300, 64, 128, "f32"), (1, 3, 17, 16, 7, "f32"),
                                          (1, 8, 777, 40, 50, "bf16"), (1, 16, 1500, 64, 64, "f32")])
def test_backward_causal_hint(gpu_lib, B, H, n, d, m, dt):
    """Under a causal mask, on the default route, the hint that states it changes no gradient: both calls
    within the direct products' bound (test_direct_backward) of 64 bits."""
    dd = synth.custom(B, H, n, d, m, seed=31 + n, qkv_dtype=dt, bias="causal")
    G = np.random.default_rng([31, n]).standard_normal((B, H, n, d)).astype(np.float32)
    args = (*(to_gpu(dd[x], dt) for x in ("q", "k", "v")), to_gpu(dd["b"]), to_gpu(dd["W"]), to_gpu(G))
    print(f"backward causal B={B} H={H} n={n} d={d} m={m} {dt}", flush=True)
    ref = oracle.attention_grad(dd["q"], dd["k"], dd["v"], dd["b"], dd["W"], G)
    for hint in (True, False):
        got = gpu_lib.attention_bwd(*args, with_db=True, causal=hint)
        for name, g, r in zip(("dq", "dk", "dv", "db"), got, ref):
            err = np.linalg.norm(g.cpu().numpy() - r) / np.linalg.norm(r)
            print(f"  hint={hint} {name}: {err:.3e}", flush=True)
            assert err <= TOL, (hint, name, err)


BWD_CASES = [
    # n, d, m: 32-position blocks and row tiles (128 and 256 rows); d + 1 contracted columns around the
    # compiled 3, 5 and 9 steps of 16; column tiles and passes; feature counts around 64, 128 and 256
    (1, 4, 4, "f32", "normal", False), (33, 31, 64, "f32", "causal", True), (127, 32, 65, "bf16", "normal", False),
    (129, 47, 20, "f32", "decay", False), (257, 48, 128, "f32", "causal", False), (300, 64, 129, "bf16", "decay", False),
    (255, 79, 256, "f32", "normal", True), (130, 80, 33, "f32", "causal", False), (520, 128, 200, "f32", "decay", False),
    (1025, 64, 64, "bf16", "causal", False),
]


def _bwd_check(lib, dd, dt, G, what, tol=TOL, **kw):
    print(what, flush=True)
    args = (*(to_gpu(dd[x], dt) for x in ("q", "k", "v")), to_gpu(dd["b"]), to_gpu(dd["W"]), to_gpu(G))
    got = lib.attention_bwd(*args, with_db=True, **kw)
    ref = oracle.attention_grad(dd["q"], dd["k"], dd["v"], dd["b"], dd["W"], G, nprf=kw.get("nprf", False))
    errs = {}
    for name, g, r in zip(("dq", "dk", "dv", "db"), got, ref):
        g = g.cpu().numpy().astype(np.float64)
        assert np.all(np.isfinite(g)), name
        errs[name] = np.linalg.norm(g - r) / np.linalg.norm(r)
    print("  " + " ".join(f"{k} {e:.3e}" for k, e in errs.items()), flush=True)
    assert max(errs.values()) <= tol, errs


@pytest.mark.parametrize("power,dt,bias", [(-60, "f32", "normal"), (-45, "bf16", "causal"), (45, "f32", "causal"), (60, "bf16", "normal")])
def test_direct_backward_value_scale(gpu_lib, power, dt, bias):
    """Gradients do not depend on the scale of the values (dv), or by that factor (the others)."""
    n, d, m = 150, 64, 64
    dd = synth.custom(2, 2, n, d, m, seed=3, qkv_dtype=dt, bias=bias)
    dd["v"] = (dd["v"] * 2.0 ** power).astype(np.float32)
    G = np.random.default_rng(3).standard_normal((2, 2, n, d)).astype(np.float32)
    _bwd_check(gpu_lib, dd, dt, G, f"value scale 2^{power} {dt} {bias}", route="direct")


@pytest.mark.parametrize("d,n,m,bias", [(64, 200, 64, "normal"), (64, 130, 128, "causal"), (30, 100, 200, "normal")])
def test_direct_backward_denominators_far_apart(gpu_lib, d, n, m, bias):
    """Rows of one block whose denominators (in units of their queries) differ by 2^20 and more: every
    third query opposes the keys, which share a direction."""
    dd = synth.custom(1, 2, n, d, m, seed=5, bias=bias, qk_scale=0.1)
    rng = np.random.default_rng([5, n])
    u = rng.standard_normal((1, 2, 1, d)).astype(np.float32)
    u *= 3.6 / np.linalg.norm(u, axis=-1, keepdims=True)
    dd["k"] = (dd["k"] + u).astype(np.float32)
    sign = np.where(np.arange(n) % 3 == 1, -1.0, 1.0)[:, None]
    dd["q"] = (dd["q"] + sign * u).astype(np.float32)
    G = rng.standard_normal((1, 2, n, d)).astype(np.float32)
    _bwd_check(gpu_lib, dd, "f32", G, f"denominators far apart d={d} n={n} m={m} {bias}", route="direct")


@pytest.mark.parametrize("d,scale,kind,mask,n,m,dt", OPPOSED[:11] + [(128, 0.6, "aligned", "none", 600, 256, "f32")])
def test_direct_backward_opposed(gpu_lib, d, scale, kind, mask, n, m, dt):
    """The four gradients where the forward's rows are not held by two fp16 terms, on the default route and
    with the gradients of other heads beside them.  Bound: that of test_direct_opposed, twice for
    the features on both sides of a product."""
    dd = _opposed(d, scale, kind, mask, n, m, dt)
    # head 0: ordinary queries and keys; both heads of a second batch entry like head 1
    for x in ("q", "k", "v"):
        dd[x] = np.concatenate([dd[x], dd[x][:, ::-1]], axis=0)
    other = synth.custom(1, 1, n, d, m, seed=7, qkv_dtype=dt)
    dd["q"][0, 0], dd["k"][0, 0] = other["q"][0, 0], other["k"][0, 0]
    G = np.random.default_rng([n, d]).standard_normal((2, 2, n, d)).astype(np.float32)
    _bwd_check(gpu_lib, dd, dt, G, f"backward opposed d={d} scale={scale} {kind} {mask} n={n} m={m} {dt}", tol=4 * TOL)


@pytest.mark.parametrize("n,d,m,dt,bias,nprf", BWD_CASES)
def test_direct_backward(gpu_lib, n, d, m, dt, bias, nprf):
    """The gradients of the direct products against the fp64 chain rule.  Tolerance 2e-5 of a
    gradient's norm, per head: the terms' errors are those of z above, and sums of either sign are
    measured against the gradient's norm.  Where the exact gradient vanishes (one key, n = 1) terms of
    the size scale = max|dz| max|[v, 1]| max|W| cancel, a handful of them each rounded to 2^-24 of
    it: an absolute 2^-21 scale, TOL times the floor 2^-5 scale."""
    B, H = 2, 2
    dd = synth.custom(B, H, n, d, m, seed=71 + n, qkv_dtype=dt, bias=bias)
    G = np.random.default_rng([71, n]).standard_normal((B, H, n, d)).astype(np.float32)
    print(f"direct backward n={n} d={d} m={m} {dt} {bias} nprf={nprf}", flush=True)
    q, k, v = (to_gpu(dd[x], dt) for x in ("q", "k", "v"))
    args = (q, k, v, to_gpu(dd["b"]), to_gpu(dd["W"]), to_gpu(G))
    got = gpu_lib.attention_bwd(*args, nprf=nprf, with_db=True, route="direct")
    ref = oracle.attention_grad(dd["q"], dd["k"], dd["v"], dd["b"], dd["W"], G, nprf=nprf)
    scale = float(np.max(np.abs(G)) * max(1.0, np.max(np.abs(dd["v"]))) * np.max(np.abs(dd["W"])))
    for name, g, r in zip(("dq", "dk", "dv", "db"), got, ref):
        g = g.cpu().numpy().astype(np.float64)
        assert np.all(np.isfinite(g)), name
        err = np.linalg.norm(g - r) / max(np.linalg.norm(r), 2.0 ** -5 * scale)
        print(f"  {name}: {err:.3e}", flush=True)
        assert err <= TOL, (name, err)
    # without the bias gradient dv comes from another kernel: the same values up to rounding
    dv = gpu_lib.attention_bwd(*args, nprf=nprf, route="direct")[2].cpu().numpy()
    assert np.linalg.norm(dv - got[2].cpu().numpy()) <= 2e-6 * np.linalg.norm(ref[2])


def test_backward_workspace_of_the_transforms(gpu_lib):
    """A workspace sized for the transforms (KRPE_ROUTE_FFT's query) serves a call on any route, which then
    has the transforms' bits; one byte less is refused."""
    B, H, n, d, m = 1, 2, 4000, 8, 16  # (the direct products need more)
    dd = synth.custom(B, H, n, d, m, seed=8)
    G = np.random.default_rng(8).standard_normal((B, H, n, d)).astype(np.float32)
    args = (*(to_gpu(dd[x]) for x in ("q", "k", "v", "b", "W")), to_gpu(G))
    lib = gpu_lib.load()
    small = int(lib.krpe_attention_bwd_workspace(B, H, n, d, m, gpu_lib.ROUTE_FFT))
    assert small < int(lib.krpe_attention_bwd_workspace(B, H, n, d, m, 0))
    want = gpu_lib.attention_bwd(*args, with_db=True, route="fft")
    ws = torch.empty(small, dtype=torch.uint8, device="cuda")
    for route in ("fft", "auto"):
        got = gpu_lib.attention_bwd(*args, workspace=ws, with_db=True, route=route)
        for g, w in zip(got, want):
            assert torch.norm(g - w) <= 2e-4 * torch.norm(w), route
    with pytest.raises(gpu_lib.KrpeError):
        gpu_lib.attention_bwd(*args, workspace=ws[:-1], with_db=True)
