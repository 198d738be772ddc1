"""Which gradient forms the autotuner tries for a batch (csrc/nr_autotune.hpp, built
with g++ against the library)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2509_06924_amd")

MAIN = r"""
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "nr_autotune.hpp"
int main(int argc, char** argv) {  // precision, then the items' layer counts
  std::vector<int64_t> row_off{0};
  for (int k = 2; k < argc; ++k) row_off.push_back(row_off.back() + atoi(argv[k]) + 2);
  nr_batch_desc d{};
  d.precision = atoi(argv[1]);
  d.n_items = argc - 2;
  d.row_off = row_off.data();
  for (const auto& c : nr::form_candidates(&d))
    printf("%d:%d ", c.first == NR_NUM_BUCKETS ? -1 : nr_bucket_lmax(c.first), c.second);
}
"""


@pytest.fixture(scope="module")
def candidates(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    import paper_2509_06924_amd as nr
    nr._n.lib()  # built
    tmp = tmp_path_factory.mktemp("autotune")
    src, exe = str(tmp / "main.cpp"), str(tmp / "main")
    with open(src, "w") as f:
        f.write(MAIN)
    r = subprocess.run([gxx, "-std=c++17", "-I", os.path.join(ROOT, "include"),
                        "-I", os.path.join(PKG, "csrc"), src, os.path.join(PKG, "libnr.so"),
                        "-Wl,-rpath," + PKG, "-Wl,--allow-shlib-undefined", "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]

    def run(precision, *layers):
        out = subprocess.run([exe, str(precision), *map(str, layers)], capture_output=True,
                             text=True, check=True).stdout
        return [tuple(map(int, c.split(":"))) for c in out.split()]
    return run, nr.NR_F64, nr.NR_F32, nr._n.NR_VARIANT_STORE, nr._n.NR_VARIANT_RECOMPUTE


def test_forms_tried(candidates):
    run, F64, F32, S, R = candidates
    assert run(F64, 0, 1, 4) == [(1, S), (1, R), (4, S), (4, R)]
    assert run(F32, 8, 3) == [(4, S), (4, R), (8, S), (8, R)]
    # one of two forms by default beyond the store form's depths, in FP64 only
    assert run(F64, 20, 33) == [(20, R), (36, R)]
    assert run(F32, 20, 33) == []
    # deep stacks: the last bucket's entry names their scan
    assert run(F64, 500) == [(40, R)] and run(F32, 500) == []
