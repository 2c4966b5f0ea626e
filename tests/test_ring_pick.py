"""The tile that the linear layers pick, from the rule itself (gemm_ring.h) compiled for the host: two blocks of 128 x 128 per compute unit
are taken with GELU only, where their rounds fill the chip; a last round of a few deep blocks is not given away as if it were a part of one."""
import os
import subprocess

import pytest

SOURCE = r"""
#include <cstdio>
#include <cstdlib>
#include "gemm_ring.h"
int main(int argc, char** argv) {
  for (int i = 1; i + 3 < argc; i += 4) {
    const int64_t m = atoll(argv[i]), n = atoll(argv[i + 1]), k = atoll(argv[i + 2]);
    const dllava::RingTile* t = dllava::ring_pick(
        k, 0, [&](const dllava::RingTile& c) -> int64_t { return c.id == 10 ? 0 : dllava::ceil_div(m, 32 * c.jt) * dllava::ceil_div(n, 32 * c.fi); },
        atoi(argv[i + 3]) == 1);
    printf("%d\n", t->id);
  }
}
"""


@pytest.fixture(scope="module")
def pick(tmp_path_factory):
    from paper_2412_00876_amd import build
    d = tmp_path_factory.mktemp("pick")
    (d / "pick.hip").write_text(SOURCE)
    r = subprocess.run([build.HIPCC, *build.COMMON, *build.HIP_FLAGS, "--offload-host-only", "-O1", str(d / "pick.hip"), "-o", str(d / "pick")],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]

    def run(*shapes):
        out = subprocess.run([str(d / "pick"), *(str(v) for s in shapes for v in s)], capture_output=True, text=True, check=True).stdout
        return [int(x) for x in out.split()]

    return run


def test_deep_layers_of_little_more_than_a_round(pick):
    """4096 features with GELU, 11008 wide: 544, 576 and 1056 tiles of 128 x 128 (221, 220 and 358 us, 256 x 160 149, 156 and 293)."""
    assert pick((2100, 4096, 11008, 1), (2304, 4096, 11008, 1), (4200, 4096, 11008, 1)) == [5, 5, 5]
    assert 12 not in pick(*((m, 4096, k, 1) for k in (4096, 11008) for m in range(2100, 9000, 100)))


def test_many_tiles_of_short_rows_with_gelu(pick):
    """512 wide, 2048 features, the image predictor's: 9216 to 23040 rows (11520: 39 us, 256 x 192 42.6)."""
    assert pick(*((m, 2048, 512, 1) for m in (9216, 11520, 16000, 18432, 23040))) == [12] * 5
    assert 12 not in pick(*((m, 2048, 512, a) for m in range(64, 24000, 500) for a in (0, 2)))
    assert 12 not in pick(*((m, 2048, 512, 1) for m in range(64, 4097, 64)))   # at most one round
