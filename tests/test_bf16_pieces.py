"""The splitting of fp32 operands into three bf16 pieces (csrc/bf16_pieces.h), compiled for the host: the pieces add up to the value
exactly, and the products of pieces that are left out stay below one fp32 rounding (2^-24 of the product; 2^-34 for the product of the two
last pieces) and have no preferred sign.

Bound of the mean: over N random pairs the left-out part has a standard deviation of at most 2^-24 of the product, so its mean is within
5 * 2^-24 / sqrt(N) of zero (truncated pieces give +0.6 * 2^-24 on average and up to 2^-21)."""
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROBE = r'''
#define __host__
#define __device__
#define __forceinline__ inline
#include "bf16_pieces.h"
#include <cstdio>
int main(int, char** argv) {
  FILE* f = fopen(argv[1], "rb");
  FILE* o = fopen(argv[2], "wb");
  float v[2];
  while (fread(v, 4, 2, f) == 2) {
    uint32_t p[3];
    moqe::cut3_pair(v[0], v[1], p[0], p[1], p[2]);
    fwrite(p, 4, 3, o);
  }
  fclose(o);
  return 0;
}
'''


def _pieces(values, tmp_path):
    src, exe, fin, fout = tmp_path / "probe.cpp", tmp_path / "probe", tmp_path / "in", tmp_path / "out"
    src.write_text(PROBE)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "paper_2508_09204_amd", "csrc"), "-o", str(exe), str(src)], check=True)
    values.astype(np.float32).tofile(fin)
    subprocess.run([str(exe), str(fin), str(fout)], check=True)
    p = np.fromfile(fout, dtype=np.uint32).reshape(-1, 3)
    lo = (p << 16).astype(np.uint32).view(np.float32)
    hi = (p & np.uint32(0xffff0000)).astype(np.uint32).view(np.float32)
    return np.stack([lo, hi], axis=1).reshape(-1, 3).astype(np.float64)


def _values(kind, n, rng):
    if kind == "normal":
        return rng.standard_normal(n).astype(np.float32)
    if kind == "one_sign":
        return (1.0 + rng.random(n)).astype(np.float32)
    if kind == "exponents":
        return (np.ldexp(1.0 + rng.random(n), rng.integers(-100, 120, n)) * rng.choice([-1.0, 1.0], n)).astype(np.float32)
    # mantissas at the edges of a piece: a few low bits beside the halves of bits 8 and 16
    m = (1 << 23) + sum((rng.integers(0, 2, n) << b) for b in (0, 1, 6, 7, 8, 14, 15, 16, 22)) - rng.integers(0, 2, n)
    return np.ldexp(m.astype(np.float64), -23).astype(np.float32)


@pytest.mark.parametrize("kind", ["normal", "one_sign", "exponents", "edges"])
def test_pieces_are_exact_and_what_is_left_out_is_one_rounding(kind, tmp_path):
    n = 1 << 17
    v = _values(kind, n, np.random.default_rng(5))
    v = v[np.abs(v) > 2.0 ** -100]
    v = v[:len(v) // 2 * 2]
    p = _pieces(v, tmp_path)
    v64 = v.astype(np.float64)
    assert np.array_equal(p.sum(axis=1), v64)
    a, b, va, vb = p[0::2], p[1::2], v64[0::2], v64[1::2]
    left = (a[:, 1] * b[:, 2] + a[:, 2] * b[:, 1] + a[:, 2] * b[:, 2]) / (va * vb)
    assert np.abs(left).max() <= 2.0 ** -24 + 2.0 ** -34
    if kind != "edges":
        assert abs(left.mean()) <= 5 * 2.0 ** -24 / np.sqrt(len(left))
