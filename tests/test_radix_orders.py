"""The autotuner's radix orders (csrc/hp_radix.hpp): the planner's own order first,
every order a factorisation of the length, the register radices up to the
largest among them, prime factors above it in front."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2301_01145_amd", "csrc")

MAIN = r"""
#include <cstdio>
#include <cstdlib>
#include "hp_radix.hpp"
int main(int argc, char** argv) {
  const int top = std::atoi(argv[1]);
  for (int L = 1; L <= 1024; ++L) {
    // the planner's order here: the prime factors
    std::vector<int> own;
    for (int f = 2, r = L; r > 1; ++f)
      while (r % f == 0) own.push_back(f), r /= f;
    if (own.size() > 8) own.clear();
    for (const auto& o : hp::radix_orders(L, top, 8, own)) {
      std::printf("%d", L);
      for (int r : o) std::printf(" %d", r);
      std::printf("\n");
    }
  }
}
"""


def primes(n):
    out, f = [], 2
    while n > 1:
        while n % f == 0:
            out.append(f)
            n //= f
        f += 1
    return out


@pytest.mark.parametrize("top", [10, 16])
def test_orders(top, tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if not cxx:
        pytest.skip("no host compiler")
    (tmp_path / "main.cpp").write_text(MAIN)
    subprocess.run([cxx, "-std=c++17", "-O1", "-I", CSRC, str(tmp_path / "main.cpp"), "-o", str(tmp_path / "orders")],
                   check=True)
    text = subprocess.run([str(tmp_path / "orders"), str(top)], check=True, capture_output=True, text=True).stdout
    by_length = {}
    for line in text.splitlines():
        L, *o = map(int, line.split())
        by_length.setdefault(L, []).append(o)
    for L, orders in by_length.items():
        p = primes(L)
        if len(p) <= 8:
            assert orders[0] == p
        assert len({tuple(o) for o in orders}) == len(orders) <= 14
        nbig = sum(f > top for f in p)
        for o in orders:
            prod = 1
            for r in o:
                prod *= r
            assert prod == L and 1 <= len(o) <= 8
        for o in orders[1:]:
            assert all(r > top for r in o[:nbig]) and all(2 <= r <= top for r in o[nbig:])
    assert sorted(by_length) == list(range(2, 1025))
    # the splits of the fewest stages are among them
    assert ([16, 15] if top == 16 else [8, 6, 5]) in by_length[240]
    assert ([16, 16] if top == 16 else [8, 8, 4]) in by_length[256]
    assert by_length[254][-1][0] == 127
