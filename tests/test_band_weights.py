"""The band weights of the tree build's large nodes, in the kernel's 32-bit sums
(on the CPU: a node whose sums could wrap has more rows than a test can hold)."""
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2107_03368_amd", "csrc")
BITS, BINS, BANDS = 4096, 256, 32


@pytest.fixture(scope="module")
def weight_shift(tmp_path_factory):
    d = tmp_path_factory.mktemp("band_weight")
    (d / "main.cpp").write_text('#include <stdio.h>\n#include <stdlib.h>\n#include "band_weight.h"\n'
                                "int main(int n, char **v) {\n"
                                "    for (int i = 1; i < n; i++)\n"
                                '        printf("%u\\n", qd::band_weight_shift((uint32_t)strtoul(v[i], 0, 10)));\n}\n')
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, str(d / "main.cpp"), "-o", str(d / "main")], check=True)
    return lambda m: int(subprocess.run([str(d / "main"), str(m)], check=True, capture_output=True, text=True).stdout)


def _bands(counts, m, wshift):
    """A band for every count, as big_band_kernel finds it when every bit is banded."""
    shift = max(0, 24 - (32 - int(m).bit_length()))
    bins = np.zeros(BINS, np.uint32)
    for c in counts[counts > 0]:
        bins[c >> shift] += np.uint32((int(c) >> wshift) + 1)
    end = np.cumsum(bins, dtype=np.uint32)
    run, total = (end - bins).astype(np.uint64), max(1, int(end[-1]))
    f = (run * np.uint64(4 * BANDS // 2) // np.uint64(total)).astype(np.int64)
    band = np.where(f < BANDS // 2, f, np.minimum(BANDS - 1, BANDS // 2 + (f - BANDS // 2) // 3)) % BANDS
    return band[counts >> shift]


@pytest.mark.parametrize("m", [2_049, 2**27 - 1, 2**27, 2**28 - 1, 2**28, 280_000_000, 540_000_000, 2**32 - 2])
def test_sums_fit_and_bands_follow_the_counts(weight_shift, m):
    wshift = weight_shift(m)
    assert BITS * ((m >> wshift) + 1) < 2**32
    rng = np.random.default_rng(m)
    for counts in (np.full(BITS, m), np.concatenate([np.full(2_048, m // 2), np.full(2_048, m)]),
                   rng.integers(1, m + 1, BITS), (m * rng.random(BITS) ** 0.2).astype(np.int64),
                   np.repeat(np.linspace(1, m, 64).astype(np.int64), 64)):
        counts = np.sort(counts.astype(np.int64))
        assert np.all(np.diff(_bands(counts, m, wshift)) >= 0)


def test_small_nodes_keep_their_weights(weight_shift):
    assert all(weight_shift(m) == 8 for m in (1, 255, 2_049, 1_000_000, 2**27 - 1))
