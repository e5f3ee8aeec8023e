"""GPU compress / decompress vs the FP64 oracle.

* bins: bit-identical for L-inf (min and max are exact); within 1e-14 for L2
  (the sum of squares is accumulated in a different order);
* quantised integers: equal to the oracle's except at bin-boundary ties
  (at most 1e-6 of the points, each off by one);
* when all integers agree the whole stream is byte-identical (Huffman,
  layout and header are bit-exact);
* the error bound holds for the GPU reconstruction, and each side decodes the
  other's stream;
* edge cases: constant, empty, squeezed axes, L = 0, NaN input, corrupt
  streams, outlier-capacity retry.
"""
import numpy as np
import pytest

import oracle
import synthetic
from oracle import Hierarchy
from oracle.quantize import from_symbols
from oracle.stream import decode_symbols, parse_header
from tests.gpu_common import assert_stream_matches_oracle, gpu, to_bytes

pytestmark = pytest.mark.gpu


def _field(shape, dtype, seed):
    if len(shape) == 3 and seed % 2 == 0:
        return synthetic.bumps(shape, seed, dtype=dtype)
    return synthetic.grf(shape, seed, dtype=dtype)


def _bound_ok(u, v, rel, norm):
    x = u.astype(np.float64)
    e = v.astype(np.float64) - x
    if norm == "linf":
        return np.max(np.abs(e)) <= rel * (x.max() - x.min())
    return np.sqrt(np.sum(e * e)) <= rel * np.sqrt(np.sum(x * x))


def _check_parity(u, rel, norm, mode="rel"):
    torch, mgc = gpu()
    blob = mgc.compress(torch.from_numpy(u).cuda(), rel, norm, mode)
    g = to_bytes(blob)
    r = oracle.compress(u, rel, norm, mode)
    hg, hr = parse_header(g), parse_header(r)
    for key in ("L", "N", "n_chunks", "D", "shape", "S", "C", "flags"):
        assert hg[key] == hr[key], key
    if norm == "linf":
        assert np.array_equal(hg["q"], hr["q"])
        assert hg["tau"] == hr["tau"] and hg["tau_eff"] == hr["tau_eff"]
    else:
        assert np.allclose(hg["q"], hr["q"], rtol=1e-14, atol=0)
    kg = from_symbols(*decode_symbols(g))
    kr = from_symbols(*decode_symbols(r))
    diff = np.nonzero(kg != kr)[0]
    assert len(diff) <= 1e-6 * u.size + 1
    assert np.all(np.abs(kg[diff] - kr[diff]) == 1)
    if len(diff) == 0 and norm == "linf":
        assert g == r, "identical integers must give an identical stream"
    # reconstructions: GPU of its own stream, GPU of the oracle stream, oracle of GPU stream
    v = mgc.decompress(blob).cpu().numpy()
    assert v.shape == u.shape and v.dtype == u.dtype
    assert _bound_ok(u, v, rel, norm)
    rdev = torch.from_numpy(np.frombuffer(r, dtype=np.uint8).copy()).cuda()
    v2 = mgc.decompress(rdev).cpu().numpy()
    v2_ref = oracle.decompress(r)
    tol = 1e-12 * float(np.max(np.abs(u))) + (np.spacing(np.float32(np.max(np.abs(u))))
                                              if u.dtype == np.float32 else 0.0)
    assert np.max(np.abs(v2.astype(np.float64) - v2_ref)) <= tol
    assert _bound_ok(u, oracle.decompress(g), rel, norm)
    return len(g)


@pytest.mark.parametrize("shape", [(65, 65, 65), (30, 41, 12), (40, 33, 17), (9, 5, 4),
                                   (33, 20), (257,), (2, 2, 2), (1, 7, 1), (3, 5)])
@pytest.mark.parametrize("rel", [1e-2, 1e-3, 1e-4])
def test_linf_f32(shape, rel):
    u = _field(shape, np.float32, 2 if len(shape) == 3 else 3)
    _check_parity(u, rel, "linf")


@pytest.mark.parametrize("shape", [(65, 65, 65), (129, 70), (300,)])
@pytest.mark.parametrize("norm", ["linf", "l2"])
def test_f64_and_l2(shape, norm):
    u = _field(shape, np.float64, 5)
    _check_parity(u, 1e-3, norm)
    _check_parity(u.astype(np.float32), 1e-4, norm)


def test_absolute_mode():
    u = _field((33, 33, 33), np.float32, 4)
    _check_parity(u, 0.01, "linf", "abs")


def test_constant_empty_and_scalar():
    torch, mgc = gpu()
    c = np.full((20, 7), 3.5, dtype=np.float32)
    b = mgc.compress(torch.from_numpy(c).cuda(), 1e-3)
    assert to_bytes(b) == oracle.compress(c, 1e-3)
    assert np.array_equal(mgc.decompress(b).cpu().numpy(), c)
    e = np.zeros((0, 5), dtype=np.float64)
    b = mgc.compress(torch.from_numpy(e).cuda(), 1e-3)
    assert to_bytes(b) == oracle.compress(e, 1e-3)
    assert mgc.decompress(b).shape == (0, 5)
    s = np.array([1.25], dtype=np.float64)
    b = mgc.compress(torch.from_numpy(s).cuda(), 1e-3)
    assert mgc.decompress(b).cpu().numpy()[0] == 1.25


def test_rejects_nan_and_bad_bound():
    torch, mgc = gpu()
    u = np.ones((16, 16), dtype=np.float32)
    u[3, 4] = np.nan
    with pytest.raises(mgc.MgcError) as e:
        mgc.compress(torch.from_numpy(u).cuda(), 1e-3)
    assert e.value.name == "EINVAL"
    with pytest.raises(mgc.MgcError) as e:
        mgc.compress(torch.ones(8, 8, device="cuda"), -1.0)
    assert e.value.name == "EINVAL"


def test_rejects_corrupt_streams():
    torch, mgc = gpu()
    u = _field((33, 33, 33), np.float32, 3)
    blob = mgc.compress(torch.from_numpy(u).cuda(), 1e-3)
    with pytest.raises(mgc.MgcError) as e:
        mgc.decompress(blob[: blob.numel() - 16])
    assert e.value.name == "EFORMAT"
    bad = blob.clone()
    bad[0] = bad[0] ^ 0xFF
    with pytest.raises(mgc.MgcError):
        mgc.decompress(bad)


def test_decompress_stream_at_word_offsets():
    """A compressed stream copied 4, 12 or 36 bytes past an aligned address
    reconstructs the same array, bit for bit."""
    torch, mgc = gpu()
    u = _field((65, 33, 47), np.float32, 5)
    blob = mgc.compress(torch.from_numpy(u).cuda(), 1e-3)
    ref = mgc.decompress(blob)
    n = blob.numel()
    for off in (4, 12, 36):
        print("case: offset", off, flush=True)
        buf = torch.zeros(n + 64, dtype=torch.uint8, device="cuda")
        buf[off:off + n] = blob
        assert bool(torch.equal(mgc.decompress(buf[off:off + n]), ref)), off


def test_outlier_capacity_retry():
    torch, mgc = gpu()
    u = _field((65, 65, 65), np.float32, 3)
    x = torch.from_numpy(u).cuda()
    full = to_bytes(mgc.compress(x, 1e-5))
    hd = parse_header(full)
    assert hd["n_outliers"] > 10
    small = to_bytes(mgc.compress(x, 1e-5, outlier_cap=8))   # overflows, then retries
    assert small == full


def test_repeat_calls_are_deterministic():
    torch, mgc = gpu()
    u = _field((129, 129, 65), np.float32, 3)
    x = torch.from_numpy(u).cuda()
    a = to_bytes(mgc.compress(x, 1e-3))
    b = to_bytes(mgc.compress(x, 1e-3))
    assert a == b


def test_streamed_level_kernel_matches_tiled():
    """Levels of >= 2^25 points use the z-streamed decomposition kernel; the
    tiled kernel (forced candidate 1) must give the same stream and the same
    FP64 coefficients, bit for bit."""
    torch, mgc = gpu()
    gen = torch.Generator(device="cuda").manual_seed(17)
    x = torch.randn((65, 513, 1025), generator=gen, device="cuda", dtype=torch.float32)
    x += torch.linspace(-3.0, 3.0, 1025, device="cuda")
    streamed = mgc.compress(x, 1e-3)
    coeff_s = mgc.decompose(x)
    mgc.set_tuning("dec_f32", 1)
    try:
        tiled = mgc.compress(x, 1e-3)
        coeff_t = mgc.decompose(x)
    finally:
        mgc.set_tuning("dec_f32", -1)
    assert streamed.numel() == tiled.numel() and bool((streamed == tiled).all())
    assert bool((coeff_s == coeff_t).all())
    # the streamed recomposition restriction: exact inversion without
    # quantisation, and the decompressed field within the bound
    back = mgc.recompose(coeff_s, tuple(x.shape), dtype=torch.float64)
    err = torch.max(torch.abs(back - x.double())).item()
    assert err <= 1e-12 * torch.max(torch.abs(x)).item()
    y = mgc.decompress(streamed)
    tau = 1e-3 * (x.max() - x.min()).item()
    assert torch.max(torch.abs(y.double() - x.double())).item() <= tau


@pytest.mark.parametrize("rel", [1e-2, 1e-3, 1e-4])
def test_full_size_513(rel):
    """The benchmark's configuration: 513^3 FP32 |k|^-3 field."""
    torch, mgc = gpu()
    u = _grf513()
    x = torch.from_numpy(u).cuda()
    blob = mgc.compress(x, rel)
    v = mgc.decompress(blob).cpu().numpy()
    assert _bound_ok(u, v, rel, "linf")
    g = to_bytes(blob)
    hd = parse_header(g)
    h = Hierarchy(u.shape)
    assert hd["L"] == h.L == 9
    # sampled finest-level integers against the oracle, one by one
    idx = np.random.default_rng(1).choice(u.size, 2000, replace=False)
    pos, c = oracle.transform.finest_coefficients_at(u.astype(np.float64), h, idx)
    _, tau_eff = oracle.error_budget(u, rel, "linf", "rel")
    q = oracle.level_bins(h, tau_eff, "linf")
    assert np.array_equal(hd["q"], q)
    k_ref = np.rint(c * (1.0 / q[h.L])).astype(np.int64)
    chunks = np.unique(pos // hd["C"])
    sym, opos, oval = decode_symbols(g, hd, chunks=chunks)
    k = sym[pos] - 32768
    esc = sym[pos] == 0
    if np.any(esc):
        where = np.searchsorted(opos.astype(np.int64), pos[esc])
        k[esc] = oval[where]
    mism = np.count_nonzero(k != k_ref)
    assert mism <= 1e-6 * u.size
    assert np.all(np.abs(k - k_ref) <= 1)


_CACHE = {}


def _grf513():
    if "u" not in _CACHE:
        _CACHE["u"] = synthetic.grf((513, 513, 513), 2)
    return _CACHE["u"]


def _cfg3(name):
    key = "cfg3_" + name
    if key not in _CACHE:
        if name == "sin8193":
            _CACHE[key] = synthetic.sinusoids((8193, 8193), 3)
        else:
            _CACHE[key] = synthetic.grf((300, 400, 500), 4)
    return _CACHE[key]


@pytest.mark.parametrize("name,norm,rel", [("sin8193", "linf", 1e-4), ("sin8193", "l2", 1e-3),
                                           ("grf300", "linf", 1e-4), ("grf300", "l2", 1e-3)])
def test_full_size_fp64_and_non_dyadic(name, norm, rel):
    """8193^2 FP64 plane waves and a 300x400x500 FP32 |k|^-3 field."""
    torch, mgc = gpu()
    u = _cfg3(name)
    x = torch.from_numpy(u).cuda()
    blob = mgc.compress(x, rel, norm)
    v = mgc.decompress(blob).cpu().numpy()
    assert v.dtype == u.dtype and _bound_ok(u, v, rel, norm)
    g = to_bytes(blob)
    hd = parse_header(g)
    h = Hierarchy(u.shape)
    assert hd["L"] == h.L
    _, tau_eff = oracle.error_budget(u, rel, norm, "rel")
    q = oracle.level_bins(h, tau_eff, norm)
    if norm == "linf":
        assert np.array_equal(hd["q"], q)
    else:
        assert np.allclose(hd["q"], q, rtol=1e-13, atol=0)
    # sampled finest-level integers (with the stream's own bins)
    idx = np.random.default_rng(2).choice(u.size, 2000, replace=False)
    pos, c = oracle.transform.finest_coefficients_at(u.astype(np.float64), h, idx)
    k_ref = np.rint(c * (1.0 / hd["q"][h.L])).astype(np.int64)
    chunks = np.unique(pos // hd["C"])
    sym, opos, oval = decode_symbols(g, hd, chunks=chunks)
    k = sym[pos] - 32768
    esc = sym[pos] == 0
    if np.any(esc):
        where = np.searchsorted(opos.astype(np.int64), pos[esc])
        k[esc] = oval[where]
    assert np.count_nonzero(k != k_ref) <= 1e-6 * u.size
    assert np.all(np.abs(k - k_ref) <= 1)


@pytest.mark.parametrize("shape,dtype", [((325, 322, 321), "float32"), ((322, 326, 323), "float64")])
@pytest.mark.parametrize("share", [0.0, 0.002, 0.4])
def test_streamed_level_equals_tiled_with_escapes(shape, dtype, share):
    """The z-streamed finest level against the tiled one (forced candidate 1),
    axes of odd and even length, with no, some and many escaped values (the
    block's list stays empty, is flushed now and then, and overflows): equal
    streams, since escaped values are placed by rank."""
    torch, mgc = gpu()
    gen = torch.Generator(device="cuda").manual_seed(5)
    x = torch.randn(shape, device="cuda", generator=gen).cumsum(0).cumsum(1).cumsum(2) * 1e-3
    spike = torch.rand(shape, device="cuda", generator=gen) < share
    x = torch.where(spike, torch.randn(shape, device="cuda", generator=gen) * 300.0, x).to(getattr(torch, dtype))
    n = x.numel()
    a = mgc.compress(x, 1e-3, mode="abs", outlier_cap=n)
    kind = "dec_f32" if dtype == "float32" else "dec_f64"
    mgc.set_tuning(kind, 1)
    try:
        b = mgc.compress(x, 1e-3, mode="abs", outlier_cap=n)
    finally:
        mgc.set_tuning(kind, -1)
    assert torch.equal(a, b)
    y = mgc.decompress(a)
    assert torch.max(torch.abs(y.double() - x.double())).item() <= 1e-3


@pytest.mark.parametrize("dtype", ["float32", "float64"])
@pytest.mark.parametrize("shape,share", [((2897, 2897), 0.0), ((2898, 2899), 1e-3),
                                         ((16385, 513), 0.05), ((514, 16400), 0.3),
                                         ((2049, 2050), 0.01)])
def test_streamed_rows_equal_tiled_with_escapes(shape, share, dtype):
    """2-axis levels streamed along the rows (2^23 points and more down, 2^22
    back) against the tiled decomposition (forced candidate 1): equal streams
    with no, some and many escaped values, axes of odd and even length; and the
    streamed way back meets the bound, its error in FP64 that of rounding."""
    torch, mgc = gpu()
    gen = torch.Generator(device="cuda").manual_seed(6)
    x = torch.randn(shape, device="cuda", generator=gen).cumsum(0).cumsum(1) * 1e-3
    spike = torch.rand(shape, device="cuda", generator=gen) < share
    x = torch.where(spike, torch.randn(shape, device="cuda", generator=gen) * 300.0, x).to(getattr(torch, dtype))
    n = x.numel()
    a = mgc.compress(x, 1e-3, mode="abs", outlier_cap=n)
    kind = "dec_f32" if dtype == "float32" else "dec_f64"
    mgc.set_tuning(kind, 1)
    try:
        b = mgc.compress(x, 1e-3, mode="abs", outlier_cap=n)
    finally:
        mgc.set_tuning(kind, -1)
    assert torch.equal(a, b)
    assert torch.max(torch.abs(mgc.decompress(a).double() - x.double())).item() <= 1e-3
    if dtype == "float64":
        back = mgc.recompose(mgc.decompose(x), shape)
        assert torch.max(torch.abs(back - x)).item() <= 1e-11 * float(x.abs().max())


@pytest.mark.parametrize("shape", [(3, 600, 601), (600, 3, 602), (601, 602, 3), (4, 513, 520),
                                   (129, 130, 131), (130, 129, 64), (1025, 1024), (1024, 1025),
                                   (3, 16500, 22), (65, 16500)])
@pytest.mark.parametrize("share", [0.0, 0.02])
def test_streamed_interpolation_holds_bound_and_inverts(shape, share):
    """Levels of 2^20 points and more go back through the streamed
    interpolation: both kinds of axis ends, one and several blocks and segments
    a column, escaped values absent and present, both output types; FP64
    coefficients invert to rounding."""
    torch, mgc = gpu()
    gen = torch.Generator(device="cuda").manual_seed(7)
    x = torch.randn(shape, device="cuda", generator=gen, dtype=torch.float64) * 1e-2
    spike = torch.rand(shape, device="cuda", generator=gen) < share
    x = torch.where(spike, torch.randn(shape, device="cuda", generator=gen, dtype=torch.float64) * 300.0, x)
    for y in (x, x.float()):
        a = mgc.compress(y, 1e-3, mode="abs", outlier_cap=y.numel())
        assert torch.max(torch.abs(mgc.decompress(a).double() - y.double())).item() <= 1e-3
    back = mgc.recompose(mgc.decompose(x), shape)
    assert torch.max(torch.abs(back - x)).item() <= 1e-11 * float(x.abs().max())


@pytest.mark.parametrize("shape,share", [((257, 258, 259), 0.0), ((258, 257, 256), 1e-4),
                                         ((3, 2400, 2401), 0.02), ((2400, 3, 2402), 0.3),
                                         ((2401, 2402, 3), 0.0), ((4, 2049, 2050), 0.3),
                                         ((2050, 4, 2049), 1e-4), ((2050, 2049, 4), 0.02)])
def test_column_restriction_holds_bound_and_inverts(shape, share):
    """3-axis levels of 2^24 points and more: columns of wavefronts with both
    kinds of axis ends, partial strips and columns, one and many segments; no
    escaped value in a plane, some, more than are searched together."""
    torch, mgc = gpu()
    gen = torch.Generator(device="cuda").manual_seed(8)
    x = torch.randn(shape, device="cuda", generator=gen, dtype=torch.float64) * 1e-2
    spike = torch.rand(shape, device="cuda", generator=gen) < share
    x = torch.where(spike, torch.randn(shape, device="cuda", generator=gen, dtype=torch.float64) * 300.0, x)
    for y in (x, x.float()):
        a = mgc.compress(y, 1e-3, mode="abs", outlier_cap=y.numel())
        assert torch.max(torch.abs(mgc.decompress(a).double() - y.double())).item() <= 1e-3
    back = mgc.recompose(mgc.decompose(x), shape)
    assert torch.max(torch.abs(back - x)).item() <= 1e-11 * float(x.abs().max())


@pytest.mark.parametrize("dtype", ["float32", "float64"])
@pytest.mark.parametrize("shape,share", [((162, 163, 161), 0.0), ((161, 162, 164), 1e-4),
                                         ((3, 1200, 1201), 0.02), ((1200, 3, 1202), 0.3),
                                         ((1201, 1202, 3), 0.0), ((4, 1025, 1050), 0.3),
                                         ((1026, 4, 1049), 1e-4), ((1050, 1025, 4), 0.02)])
def test_columns_equal_tiled_with_escapes(shape, share, dtype):
    """3-axis levels of 2^22 points and more, columns of wavefronts, against the
    tiled decomposition (forced candidate 1): equal streams for both kinds of
    axis ends, partial strips and columns, one and many segments, and no, some
    and many escaped values (the list stays empty, is handed over now and then,
    every plane)."""
    torch, mgc = gpu()
    gen = torch.Generator(device="cuda").manual_seed(9)
    x = torch.randn(shape, device="cuda", generator=gen) * 1e-2
    spike = torch.rand(shape, device="cuda", generator=gen) < share
    x = torch.where(spike, torch.randn(shape, device="cuda", generator=gen) * 300.0, x).to(getattr(torch, dtype))
    n = x.numel()
    a = mgc.compress(x, 1e-3, mode="abs", outlier_cap=n)
    kind = "dec_f32" if dtype == "float32" else "dec_f64"
    mgc.set_tuning(kind, 1)
    try:
        b = mgc.compress(x, 1e-3, mode="abs", outlier_cap=n)
    finally:
        mgc.set_tuning(kind, -1)
    assert torch.equal(a, b)


@pytest.mark.parametrize("shape", [(33, 34, 35), (130, 70), (3000,)])
def test_mostly_escaped_values_match_oracle(shape):
    """Noise at a bound that escapes most values: every tile's list overflows."""
    torch, mgc = gpu()
    u = np.random.default_rng(9).standard_normal(shape)
    blob = to_bytes(mgc.compress(torch.from_numpy(u).cuda(), 1e-7, mode="abs"))
    ref = oracle.compress(u, 1e-7, mode="abs")
    assert oracle.parse_header(ref)["n_outliers"] > 0.5 * u.size
    assert_stream_matches_oracle(blob, ref, "linf")


# 3-axis levels from 2^20 points (interpolation) and 2^24 (restriction) on and
# 2-axis ones from 2^20 and 2^22 on: both kinds of axis ends, partial strips, columns
# and segments; no escaped value, some, more of a plane than are searched together
@pytest.mark.parametrize("shape,share", [((257, 258, 259), 0.0), ((258, 257, 256), 1e-4), ((3, 2400, 2401), 0.02),
                                         ((2401, 2402, 3), 0.3), ((2050, 4, 2049), 1e-3), ((101, 102, 103), 0.01),
                                         ((2897, 2898), 1e-3), ((2050, 2049), 0.3), ((1030, 1025), 0.0),
                                         ((16385, 513), 0.05), ((64528, 65), 0.01)])
def test_way_back_streamed_equals_tiled(shape, share):
    """Decompression and recomposition of large levels against the tiled kernels
    (forced candidate 1): equal values, from symbols and from FP64 coefficients, in
    both output types."""
    torch, mgc = gpu()
    gen = torch.Generator(device="cuda").manual_seed(11)
    x = torch.randn(shape, device="cuda", generator=gen, dtype=torch.float64) * 1e-2
    spike = torch.rand(shape, device="cuda", generator=gen) < share
    x = torch.where(spike, torch.randn(shape, device="cuda", generator=gen, dtype=torch.float64) * 300.0, x)
    streams = [mgc.compress(y, 1e-3, mode="abs", outlier_cap=y.numel()) for y in (x, x.float())]
    c = mgc.decompose(x)

    def back():
        return [mgc.decompress(s) for s in streams] + [mgc.recompose(c, shape, t) for t in (torch.float64, torch.float32)]

    a = back()
    mgc.set_tuning("rec", 1)
    try:
        b = back()
    finally:
        mgc.set_tuning("rec", -1)
    for u, v in zip(a, b):
        assert torch.equal(u, v)


def _spiked(torch, shape, nodes, dtype, seed=12):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.randn(shape, device="cuda", generator=gen, dtype=torch.float64) * 1e-2
    x.reshape(-1)[nodes] = 300.0 + torch.rand(len(nodes), device="cuda", generator=gen, dtype=torch.float64)
    return x.to(dtype)


# escaped values too few for an index of their records and enough for one, in
# clusters and alone, at both ends of the stream; arrays whose index has an entry
# every 64 positions and one every few hundred
@pytest.mark.parametrize("shape", [(40, 41, 42), (700, 33), (161, 162, 163), (3000,)])
def test_escaped_values_found_through_their_index(shape):
    torch, mgc = gpu()
    n = int(np.prod(shape))
    rng = np.random.default_rng(n)
    below = above = 0
    for spikes in (1, 4, 9, 11, 13, 16, 25, 60, 300, min(n // 3, 40000)):
        nodes = np.unique(np.concatenate([[0, n - 1], rng.integers(0, n, spikes), n // 2 + np.arange(min(spikes, 40))]))
        x = _spiked(torch, shape, torch.from_numpy(nodes).cuda(), torch.float64)
        s = mgc.compress(x, 1e-3, mode="abs", outlier_cap=n)
        esc = parse_header(to_bytes(s[:1024].contiguous()) + bytes(8))["n_outliers"]
        below, above = below + (0 < esc < 128), above + (esc >= 128)
        assert torch.max(torch.abs(mgc.decompress(s) - x)).item() <= 1e-3, (spikes, esc)
    assert above and (below or len(shape) > 2)


def test_one_in_a_hundred_escaped_values_cost_little_on_the_way_back():
    """The level kernels of 150 x 200 x 250 with 1 % of the values escaped against none:
    a search through all records for each made them take eight times as long."""
    torch, mgc = gpu()
    shape = (150, 200, 250)
    n = int(np.prod(shape))
    nodes = torch.from_numpy(np.random.default_rng(1).choice(n, n // 100, replace=False)).cuda()

    def us(x):
        s = mgc.compress(x, 1e-3, mode="abs", outlier_cap=n)
        mgc.decompress(s)
        mgc.profile_enable(True)
        mgc.profile_reset()
        for _ in range(5):
            mgc.decompress(s)
        r = mgc.profile_read()
        mgc.profile_enable(False)
        return sum(r[k][1] for k in ("rec_restrict[finest]", "rec_interp[finest]")) / 5 * 1e3

    a, b = us(_spiked(torch, shape, nodes[:0], torch.float32)), us(_spiked(torch, shape, nodes, torch.float32))
    print("finest level back: %.1f us without, %.1f us with escaped values" % (a, b))
    assert b <= 5 * a


def test_escaped_values_of_thin_arrays_cost_little_on_the_way_back():
    """Columns of 1449 x 1449 x 17 with 10 % of the values escaped against none: lanes
    past the end of the rows looked up values too, 36 times the time."""
    torch, mgc = gpu()
    shape = (1449, 1449, 17)
    n = int(np.prod(shape))
    nodes = torch.from_numpy(np.random.default_rng(2).choice(n, n // 10, replace=False)).cuda()

    def us(x):
        s = mgc.compress(x, 1e-3, mode="abs", outlier_cap=n)
        y = mgc.decompress(s)
        assert torch.max(torch.abs(y - x)).item() <= 1e-3
        mgc.profile_enable(True)
        mgc.profile_reset()
        for _ in range(3):
            mgc.decompress(s, out=y)
        ms = mgc.profile_read()["rec_restrict[finest]"][1]
        mgc.profile_enable(False)
        return ms / 3 * 1e3

    a, b = us(_spiked(torch, shape, nodes[:0], torch.float32)), us(_spiked(torch, shape, nodes, torch.float32))
    print("restriction of the finest level: %.1f us without, %.1f us with escaped values" % (a, b))
    assert b <= 14 * a
