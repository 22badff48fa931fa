"""The order in which a launch deals its tiles out (grid_of, decode_block), on the CPU: a small host program built
from the header prints the grids, and the decoding is done here with plain divisions."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = """
#include <cstdio>
#include "s2attn_launch.h"
int main() {
  int T, n, share, slots, crowded;
  while (scanf("%d %d %d %d %d", &T, &n, &share, &slots, &crowded) == 5) {
    const s2::Grid g = s2::grid_of(T, n, share, slots, crowded);
    printf("%d %d %d %d\\n", g.blocks, g.deal.bundle, g.deal.il, s2::interleave_for(T, slots));
  }
}
"""
# tiles of a sequence, sequences, neighbours that share K and V, workgroup slots of an XCD, the four-wave forward's grid
GRIDS = [(T, n, share, slots, crowded) for slots, crowded in ((32, 0), (64, 0), (64, 1), (96, 0), (128, 0)) for T in (1, 2, 3, 4, 5, 6, 7, 8, 11, 12, 14, 16, 22, 43, 100)
         for n, share in ((1, 1), (8, 1), (12, 2), (24, 8), (56, 8), (80, 4), (104, 1), (144, 1), (160, 1), (200, 1), (344, 2),
                          (376, 1), (520, 2), (608, 2), (1216, 4), (3000, 3), (8200, 1))]


@pytest.fixture(scope="module")
def grids(tmp_path_factory):
    d = tmp_path_factory.mktemp("grid")
    (d / "grid.hip").write_text(SOURCE)
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "--offload-arch=gfx950", "-std=c++17", "-w",
                    "-I", os.path.join(ROOT, "paper_2309_12307_amd", "csrc"), str(d / "grid.hip"), "-o", str(d / "grid")], check=True)
    text = "\n".join(" ".join(map(str, g)) for g in GRIDS)
    out = subprocess.run([str(d / "grid")], input=text, capture_output=True, text=True, check=True).stdout
    return list(zip(GRIDS, (tuple(map(int, l.split())) for l in out.splitlines())))


def test_every_tile_once(grids):
    for (T, n, share, slots, crowded), (blocks, bundle, il, want) in grids:
        if blocks > 200000:
            continue
        seen = set()
        for block in range(blocks):
            slot = block // 8
            chunk, within = divmod(slot, T * il)
            rank, x = divmod(within, il)
            y = chunk * il + x
            seq = (y // bundle * 8 + block % 8) * bundle + y % bundle
            if seq < n:
                assert (seq, rank) not in seen
                seen.add((seq, rank))
        assert len(seen) == n * T, (T, n, share, slots)


def test_last_walks_are_full(grids):
    """The last walk of an XCD is three quarters full, or at least as full as with the shortest walks; sequences of few
    tiles make do with half (the four-wave forward's with five eighths)."""
    for (T, n, share, slots, crowded), (blocks, bundle, il, want) in grids:
        each = -(-(n // bundle) // 8) * bundle
        if each <= want:
            assert il == each
            continue
        assert want <= il <= 2 * want
        fill = lambda x: ((each - 1) % x + 1) / x
        assert fill(il) >= min(0.75, fill(want)), (T, each, want, il)
        if T > 6 or (T > 4 and (each >= 2 * want or not crowded)):
            assert fill(il) >= 0.75 or all(fill(x) < 0.75 for x in range(want, 2 * want + 1)), (T, each, want, il)
