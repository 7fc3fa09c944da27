"""The closed-form pair intervals of the tilted and hybrid policies (compiled for
the host from the kernels' own header) against the oracle's estimator, which
compares the retained ranks one by one: every pair of surfaces whose counters
sit on the edges of the policies' rings (0, powers of two and their
neighbours, the top of the 32-bit range), close together and far apart, for
lower bounds of one to more ranks than a surface holds."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

import oracle

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2405_03605_amd", "csrc")

SOURCE = r"""
#include "ga_mrca_pairs.hpp"
using namespace ga;
static uint64_t word(const uint32_t* D, int x, int words) {
  return D[x * words] | (words > 1 ? (uint64_t)D[x * words + 1] << 32 : 0);
}
extern "C" void pairs(const uint32_t* T, const uint32_t* D, const uint32_t* S, const uint32_t* E,
                      int n, int sites, int bits, int policy, uint32_t kc, uint32_t* L,
                      uint32_t* U) {
  const int words = sites * bits / 32;
  for (int x = 0; x < n; ++x)
    for (int y = 0; y < n; ++y) {
      const uint64_t d = word(D, x, words) ^ word(D, y, words);
      Interval r;
      if (policy == 2) {
        const uint32_t e = E[x] > E[y] ? E[x] : E[y];
        const uint32_t na = (T[x] >> 1) + (T[x] & 1), nb = (T[y] >> 1) + (T[y] & 1);
        const uint32_t m = na < nb ? na : nb, shared = m ? ((m - 1) >> e) + 1 : 0;
        uint32_t s[2] = {0, 0};
        for (uint32_t j = 0; j < shared; ++j) {
          s[0] |= ((S[x] >> (j << (e - E[x]))) & 1u) << j;
          s[1] |= ((S[y] >> (j << (e - E[y]))) & 1u) << j;
        }
        r = hybrid_interval(T[x], T[y], s[0], s[1], e, shared, (uint32_t)(d >> 32), kc);
      } else if (sites == 64) {
        r = tilted2_interval(T[x], T[y], even_bits(d), even_bits(d >> 1), kc);
      } else {
        r = tilted_interval(T[x], T[y], bits == 2 ? even_bits(d) | even_bits(d >> 1) : (uint32_t)d,
                            kc);
      }
      L[x * n + y] = r.lower;
      U[x * n + y] = r.upper;
    }
}
"""


@pytest.fixture(scope="module")
def pairs(tmp_path_factory):
    d = tmp_path_factory.mktemp("pairs")
    src, so = str(d / "pairs.cpp"), str(d / "pairs.so")
    with open(src, "w") as fh:
        fh.write(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=all",
                    "-fPIC", "-shared", "-I" + CSRC, src, "-o", so], check=True,
                   capture_output=True, timeout=120)
    return ctypes.CDLL(so).pairs


def site_walk(r, s):
    """Site of rank r on 2^s sites under the steady policy."""
    n = 1 << s
    if r < n:
        return r
    e = r.bit_length() - s
    return site_walk(((2 * ((r >> e) - n // 2) + 1) << (e - 1)), s)


def steady_halves(T, D):
    """The steady half of each hybrid surface in rank order, and its epoch."""
    S, E = [], []
    for t, (lo, _) in zip(T.tolist(), D.tolist()):
        nh = (t + 1) // 2
        e = max(0, (nh - 1).bit_length() - 5) if nh else 0
        count = ((nh - 1) >> e) + 1 if nh else 0
        S.append(sum(((lo >> site_walk(j << e, 5)) & 1) << j for j in range(count)))
        E.append(e)
    return np.array(S, np.uint32), np.array(E, np.uint32)


def counters():
    out = {0, 1, 2, 3, 4, 5, 6, 7, (1 << 32) - 1, (1 << 32) - 2, 3 << 30, (3 << 30) + 1}
    for b in (3, 5, 6, 10, 16, 30, 31):
        out |= {(1 << b) - 2, (1 << b) - 1, 1 << b, (1 << b) + 1, (3 << b) >> 1}
    rng = np.random.default_rng(9)
    out |= {int(x) for x in rng.integers(0, 1 << 32, 12)}
    base = int(rng.integers(2000, 100000))
    out |= {base + int(x) for x in rng.integers(0, 70, 24)}
    return np.array(sorted(out), dtype=np.uint32)


@pytest.mark.parametrize("sites,bits,policy", [(32, 1, 1), (64, 1, 1), (32, 2, 1), (64, 1, 2)])
@pytest.mark.parametrize("kc", [1, 2, 5, 33, 70])
def test_pair_intervals_match_oracle(pairs, sites, bits, policy, kc):
    words = sites * bits // 32
    rng = np.random.default_rng(100 * sites + 10 * bits + policy)
    T = counters()
    # every counter three times, with unrelated fields and with a few flips
    T = np.concatenate([T, T, T])
    D = rng.integers(0, 1 << 32, (T.size, words), dtype=np.uint64).astype(np.uint32)
    third = T.size // 3
    flips = (rng.integers(0, 1 << 32, (third, words), dtype=np.uint64) &
             rng.integers(0, 1 << 32, (third, words), dtype=np.uint64) &
             rng.integers(0, 1 << 32, (third, words), dtype=np.uint64)).astype(np.uint32)
    D[third:2 * third] = D[0] ^ flips
    D[2 * third:] = D[1]
    n = T.size
    S, E = steady_halves(T, D) if policy == 2 else (np.zeros(n, np.uint32),) * 2
    L, U = np.empty((n, n), np.uint32), np.empty((n, n), np.uint32)
    p = lambda a: a.ctypes.data_as(ctypes.c_void_p)  # noqa: E731
    pairs(p(T), p(D), p(S), p(E), n, sites, bits, policy, ctypes.c_uint32(kc), p(L), p(U))
    L0, U0 = oracle.mrca_interval_matrix(T, D, sites, kc, bits, policy=policy)
    assert np.array_equal(U, U0)
    assert np.array_equal(L, L0)
