"""The rules that choose between two kernels by size (csrc/routes.hpp), on the CPU.
What each side took is beside the rule; here is which one a call takes."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2503_06322_amd", "csrc")
PROGRAM = """
#include "routes.hpp"
using namespace mgc;
struct Level {
  int64_t nf[3], nc[3];
  explicit Level(const int64_t* n) {
    for (int k = 0; k < 3; ++k) nf[k] = n[k], nc[k] = n[k] > 1 ? n[k] / 2 + 1 : 1;
  }
};
extern "C" {
int dec_columns(const int64_t* n, int f32) {
  const Level l(n);
  return dec_takes_columns(l.nf, l.nc, f32);
}
int dec_rows(const int64_t* n) {
  const Level l(n);
  return dec_streams_rows(l.nf, l.nc);
}
int rec_rows(const int64_t* n) {
  const Level l(n);
  return rec_streams_rows(l.nf, l.nc);
}
int batch_spread(int arrays, int64_t most) { return batch_spreads_codebooks(arrays, most); }
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    out = tmp_path_factory.mktemp("routes")
    (out / "r.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-Wall", "-Werror", "-I" + CSRC, "-o", str(out / "r.so"),
                    str(out / "r.cpp")], check=True)
    return ctypes.CDLL(str(out / "r.so"))


# (FP32, FP64): columns of wavefronts where they were the faster side, tiles where
# the contiguous axis leaves their lanes idle or there are too few points
@pytest.mark.parametrize("shape,f32,f64", [
    ((513, 513, 17), 0, 0), ((497, 497, 17), 0, 0), ((1025, 1025, 17), 1, 0), ((683, 683, 9), 0, 0),
    ((1449, 1449, 5), 1, 0), ((2897, 2897, 3), 1, 0), ((820, 820, 25), 0, 0), ((1096, 1096, 25), 1, 0),
    ((513, 513, 33), 1, 0), ((1025, 1025, 33), 1, 1), ((320, 320, 41), 1, 0), ((640, 640, 41), 1, 1),
    ((513, 513, 65), 1, 1), ((513, 513, 129), 1, 1), ((17, 513, 513), 1, 1), ((3, 2049, 1025), 1, 1),
    ((150, 200, 250), 1, 1), ((162, 163, 161), 1, 1), ((161, 162, 164), 1, 1), ((300, 400, 500), 1, 1),
    ((257, 257, 257), 1, 1), ((513, 513, 513), 1, 1), ((129, 129, 129), 0, 0), ((75, 100, 125), 0, 0)])
def test_decomposition_columns(rules, shape, f32, f64):
    n = (ctypes.c_int64 * 3)(*shape)
    assert (rules.dec_columns(n, 1), rules.dec_columns(n, 0)) == (f32, f64)


# (decomposition, restriction): streamed along the rows where that was the faster side
@pytest.mark.parametrize("shape,dec,rec", [
    ((130000, 65), 0, 1), ((66000, 129), 0, 1), ((33000, 257), 1, 1), ((16384, 513), 1, 1), ((8193, 8193), 1, 1),
    ((123362, 34), 0, 0), ((254201, 33), 0, 0), ((64528, 65), 0, 1), ((4097, 4097), 1, 1), ((2049, 2049), 0, 1),
    ((17, 1 << 20), 1, 1), ((2047, 2047), 0, 0)])
def test_rows_streamed(rules, shape, dec, rec):
    n = (ctypes.c_int64 * 3)(1, *shape)
    assert (rules.dec_rows(n), rules.rec_rows(n)) == (dec, rec)


# codebooks on many blocks up to a number of arrays that grows with the largest one
@pytest.mark.parametrize("side,few,many", [(9, 0, 1), (17, 0, 1), (25, 8, 9), (33, 24, 25), (65, 48, 49), (129, 72, 73),
                                           (257, 96, 97), (513, 96, 97)])
def test_codebooks_of_a_batch(rules, side, few, many):
    most = ctypes.c_int64(side ** 3)
    assert (few == 0 or rules.batch_spread(few, most)) and not rules.batch_spread(many, most)
    assert not rules.batch_spread(1, ctypes.c_int64(0))
