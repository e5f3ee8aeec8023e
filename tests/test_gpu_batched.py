"""Batched form: one graph launch compresses many arrays of uneven shapes.

* every array's stream is bit-identical to the plain mgc_compress stream of
  the same array and outlier capacity, in graph and in eager mode, for every
  candidate of every autotuner kind (outputs may not depend on tile shapes);
* graph replays with new data and new bounds stay identical to plain calls;
* constant, empty, non-finite and overflowing arrays get the plain path's
  trivial streams or statuses; an overflowing array is compressed again with
  the capacity the batch reported;
* the 256-array batch (axes from {33, 65, 129, 257}, relative L-inf bounds
  from {1e-2, 1e-3, 1e-4}, bump and |k|^-3 fields) matches plain calls array
  by array and every reconstruction holds its bound;
* every batched stream of the small mixed batch equals the FP64 oracle's
  stream of the same array and request, byte for byte (oracle.compress), for
  relative and absolute L-inf and relative L2 bounds; a slice of the
  256-array batch is compared with the oracle in test_gpu_oracle_fullsize.py;
* small arrays of the batch decode with the FP64 oracle's decoder too.
"""
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest

import oracle
import synthetic
from tests.gpu_common import assert_stream_matches_oracle, gpu, to_bytes

pytestmark = pytest.mark.gpu

SMALL = [  # (shape, dtype, kind, bound)
    ((33, 17, 20), np.float32, "bumps", 1e-3),
    ((65, 65, 65), np.float32, "grf", 1e-2),
    ((40, 33, 17), np.float64, "grf", 1e-4),
    ((17, 17, 17), np.float64, "bumps", 1e-3),
    ((100, 3), np.float32, "grf", 1e-3),
    ((257,), np.float64, "grf", 1e-4),
    ((9, 5, 4), np.float32, "bumps", 1e-2),
    ((2, 2, 2), np.float32, "grf", 1e-3),
    ((33, 20), np.float32, "bumps", 1e-4),
    ((1, 30, 1), np.float64, "grf", 1e-3),
]


def _field(shape, dtype, kind, seed):
    if kind == "bumps":
        return synthetic.bumps(shape, seed, dtype=dtype)
    return synthetic.grf(shape, seed, dtype=dtype)


def _inputs(torch, seed=11):
    return [torch.from_numpy(_field(s, d, k, seed + i)).cuda() for i, (s, d, k, _) in enumerate(SMALL)]


def _assert_same_as_plain(mgc, xs, bounds, streams, norm="linf", mode="rel", cap=0):
    for j, (x, b, got) in enumerate(zip(xs, bounds, streams)):
        ref = mgc.compress(x, b, norm, mode, outlier_cap=cap)
        assert got.numel() == ref.numel(), "array %d: %d vs %d bytes" % (j, got.numel(), ref.numel())
        assert bool((got == ref).all()), "array %d differs from the plain stream" % j


@pytest.mark.parametrize("norm,mode", [("linf", "rel"), ("l2", "rel"), ("linf", "abs")])
@pytest.mark.parametrize("flags", [0, 1])
def test_batched_equals_plain(norm, mode, flags):
    torch, mgc = gpu()
    xs = _inputs(torch)
    bounds = [b for (_, _, _, b) in SMALL]
    out = mgc.compress_batched(xs, bounds, norm, mode, flags=flags)
    _assert_same_as_plain(mgc, xs, bounds, out, norm, mode)


@pytest.mark.parametrize("norm,mode", [("linf", "rel"), ("l2", "rel"), ("linf", "abs")])
def test_batched_streams_equal_oracle(norm, mode):
    torch, mgc = gpu()
    xs = _inputs(torch, seed=51)
    bounds = [b for (_, _, _, b) in SMALL]
    if mode == "abs":
        bounds = [b * 2.0 for b in bounds]
    out = mgc.compress_batched(xs, bounds, norm, mode)
    for j, (x, bd) in enumerate(zip(xs, bounds)):
        u = x.cpu().numpy()
        ref = oracle.compress(u, bd, norm, mode)
        print("case: array", j, u.shape, u.dtype, norm, mode, flush=True)
        assert_stream_matches_oracle(to_bytes(out[j]), ref, norm)


def test_every_tuning_candidate_gives_the_same_streams():
    torch, mgc = gpu()
    xs = _inputs(torch, seed=21)
    bounds = [b for (_, _, _, b) in SMALL]
    ref = [mgc.compress(x, b) for x, b in zip(xs, bounds)]
    b = mgc.Batch([x.shape for x in xs], [x.dtype for x in xs])
    try:
        for kind in mgc.TUNE_KINDS:
            n_cand, _ = mgc.tuning_info(kind)
            for c in range(n_cand):
                mgc.set_tuning(kind, c)
                b.run(xs, bounds)
                got = b.streams()
                assert mgc.tuning_info(kind)[1] == c
                # tile shapes never change a result; Thomas candidates 1 and 2
                # select the serial sweeps, so the reference is the plain call
                # under the same candidate
                want = ref
                if kind.startswith("thomas") and c > 0:
                    want = [mgc.compress(x, bd) for x, bd in zip(xs, bounds)]
                for j in range(len(xs)):
                    assert bool((got[j] == want[j]).all()), "kind %s candidate %d array %d" % (kind, c, j)
                # plain calls use the forced candidate too
                for j in (1, 2, 3):
                    plain = mgc.compress(xs[j], bounds[j])
                    assert bool((plain == want[j]).all()), "plain: kind %s candidate %d" % (kind, c)
            mgc.set_tuning(kind, -1)
    finally:
        for kind in mgc.TUNE_KINDS:
            mgc.set_tuning(kind, -1)


def test_graph_replay_with_new_data_and_bounds():
    torch, mgc = gpu()
    shapes = [s for (s, _, _, _) in SMALL]
    dtypes = [torch.float32 if d == np.float32 else torch.float64 for (_, d, _, _) in SMALL]
    b = mgc.Batch(shapes, dtypes)
    for rep, seed in enumerate([31, 32, 33]):
        xs = _inputs(torch, seed)
        bounds = [bd * (1 + rep) for (_, _, _, bd) in SMALL]
        b.run(xs, bounds)
        got = b.streams()
        _assert_same_as_plain(mgc, xs, bounds, [g.clone() for g in got])


def test_trivial_and_failing_arrays():
    torch, mgc = gpu()
    good = torch.from_numpy(synthetic.grf((33, 33, 33), 5)).cuda()
    const = torch.full((9, 9, 9), 1.5, dtype=torch.float32, device="cuda")
    empty = torch.empty((0, 5), dtype=torch.float32, device="cuda")
    bad = torch.from_numpy(synthetic.bumps((17, 17), 6)).cuda()
    bad[3, 4] = float("nan")
    xs = [good, const, empty, bad]
    bounds = [1e-3, 1e-3, 1e-3, 1e-3]
    b = mgc.Batch([x.shape for x in xs], [x.dtype for x in xs])
    b.run(xs, bounds)
    torch.cuda.synchronize()
    status = b.status.cpu().tolist()
    assert status == [0, 0, 0, 1]
    sizes = b.sizes.cpu().tolist()
    for j in range(3):
        got = b.out[b.offsets[j]: b.offsets[j] + sizes[j]]
        ref = mgc.compress(xs[j], bounds[j])
        assert bool((got == ref).all()), "array %d" % j
    with pytest.raises(mgc.MgcError):
        b.streams()


def test_overflow_is_reported_and_recompressed():
    torch, mgc = gpu()
    x_over = torch.from_numpy(synthetic.grf((65, 65, 65), 7)).cuda()
    x_ok = torch.from_numpy(synthetic.bumps((33, 33, 33), 8)).cuda()
    xs = [x_ok, x_over]
    bounds = [1e-2, 1e-6]
    b = mgc.Batch([x.shape for x in xs], [x.dtype for x in xs], outlier_cap=16)
    b.run(xs, bounds)
    torch.cuda.synchronize()
    status = b.status.cpu().tolist()
    sizes = b.sizes.cpu().tolist()
    assert status[1] == 3 and sizes[1] > 16
    got = b.streams()
    assert bool((got[0] == mgc.compress(x_ok, 1e-2, outlier_cap=16)).all())
    assert bool((got[1] == mgc.compress(x_over, 1e-6, outlier_cap=int(sizes[1]))).all())


def test_small_arrays_decode_with_the_oracle():
    torch, mgc = gpu()
    xs = _inputs(torch, seed=41)
    bounds = [b for (_, _, _, b) in SMALL]
    out = mgc.compress_batched(xs, bounds)
    for j, (x, bd) in enumerate(zip(xs, bounds)):
        if x.numel() > 40000:
            continue
        u = x.cpu().numpy().astype(np.float64)
        back = oracle.decompress(to_bytes(out[j]))
        tau = bd * (u.max() - u.min())
        assert np.max(np.abs(back - u)) <= tau, "array %d" % j


@pytest.fixture(scope="module")
def batch256():
    specs = synthetic.batch_specs(256, seed=5)
    with ThreadPoolExecutor(8) as ex:
        fields = list(ex.map(synthetic.field_from_spec, specs))
    return specs, fields


def test_batch_of_256_matches_plain_and_holds_bounds(batch256):
    torch, mgc = gpu()
    specs, fields = batch256
    xs = [torch.from_numpy(u).cuda() for u in fields]
    bounds = [s["bound"] for s in specs]
    b = mgc.Batch([x.shape for x in xs], [x.dtype for x in xs])
    b.run(xs, bounds)
    got = b.streams()
    info = None
    worst = 0.0
    for j, (x, u, bd) in enumerate(zip(xs, fields, bounds)):
        ref = mgc.compress(x, bd)
        assert got[j].numel() == ref.numel() and bool((got[j] == ref).all()), "array %d" % j
        info = mgc.header_info(got[j])
        y = mgc.decompress(got[j], info=info)
        tau = bd * (float(u.max()) - float(u.min()))
        err = torch.max(torch.abs(y.double() - x.double())).item()
        worst = max(worst, err / tau)
        assert err <= tau, "array %d: error %.3g above %.3g" % (j, err, tau)
    print("256 arrays: worst error / bound = %.3f" % worst)


def test_long_lines_equal_plain():
    """Arrays whose coarse lines exceed 512 (strided) and 1024 (contiguous)
    values: window sweeps, block rows and moves between the grid buffers, one
    and two per level, beside short arrays in one batch."""
    torch, mgc = gpu()
    shapes = [(1100, 60), (60, 2100), (1030, 1030, 3), (2200, 2100), (33, 33, 33), (1100, 4, 1100)]
    gen = torch.Generator(device="cuda").manual_seed(8)
    xs = [torch.randn(s, device="cuda", generator=gen, dtype=torch.float64).cumsum(0).cumsum(-1) for s in shapes]
    xs = [x.float() if j % 2 else x for j, x in enumerate(xs)]
    got = mgc.compress_batched(xs, [1e-3] * len(xs), flags=mgc.BATCH_NO_TUNE)
    for x, g in zip(xs, got):
        assert torch.equal(g, mgc.compress(x, 1e-3))


@pytest.mark.parametrize("n", [96, 97])
def test_codebooks_spread_and_whole_equal_plain(n):
    """Up to 96 arrays sort their leaves and assign their codes on many blocks,
    more of them in one workgroup each: the plain call's streams either way."""
    torch, mgc = gpu()
    gen = torch.Generator(device="cuda").manual_seed(n)
    xs = [torch.randn((17 + k % 5, 9 + k % 3, 12), device="cuda", generator=gen) for k in range(n)]
    bounds = [10.0 ** -(1 + k % 4) for k in range(n)]
    got = mgc.compress_batched(xs, bounds, flags=mgc.BATCH_NO_TUNE)
    for x, b, s in zip(xs, bounds, got):
        assert torch.equal(s, mgc.compress(x, b))


# the largest array's size decides how many arrays have their codebooks built on
# many blocks: the last number that has and the first that has not, arrays without
# values and without a codebook among them
@pytest.mark.parametrize("side,n", [(17, 1), (25, 8), (25, 9), (33, 24), (33, 25), (65, 48), (65, 49)])
def test_codebook_forms_by_size_equal_plain(side, n):
    torch, mgc = gpu()
    gen = torch.Generator(device="cuda").manual_seed(side + n)
    xs = [torch.randn((side, side, side) if k == 0 else (5 + k % 9, 20, 17), device="cuda", generator=gen).cumsum(0)
          for k in range(n)]
    if n > 4:
        xs[2] = torch.zeros((0, 5), device="cuda")
        xs[3] = torch.full((6, 7), 2.5, device="cuda")
    bounds = [10.0 ** -(1 + k % 4) for k in range(n)]
    got = mgc.compress_batched(xs, bounds, flags=mgc.BATCH_NO_TUNE)
    for x, b, s in zip(xs, bounds, got):
        assert torch.equal(s, mgc.compress(x, b))
