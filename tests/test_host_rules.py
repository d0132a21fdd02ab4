"""CPU checks of layouts and rules in the library's sources, compiled for the
host only."""
import os
import subprocess

import pytest

from paper_2604_25459_amd import build


def _syntax(text, tmp_path):
    """Compiles `text` (host side, no code written) against the sources; returns the compiler's messages."""
    src = str(tmp_path / "t.hip")
    with open(src, "w") as f:
        f.write(text)
    r = subprocess.run([build.HIPCC, *build.FLAGS, "--offload-host-only", "-fsyntax-only", src], capture_output=True,
                       text=True)
    return r.returncode, r.stderr


@pytest.mark.parametrize("ts", [8, 16])
def test_lidar_quadratics_are_aligned_for_16_byte_reads(ts, tmp_path):
    rc, err = _syntax(f"""
#include <stddef.h>
#include "k_lidar.hip"
using Lds = gsr::LidarLds<{ts}>;
static_assert(offsetof(Lds, quad) % 16 == 0 && sizeof(Lds::quad[0]) % 16 == 0, "misaligned");
""", tmp_path)
    assert rc == 0, err


def test_lowest_bit_is_defined_for_every_mask(tmp_path):
    """Undefined results are no constant expressions: the mask without a bit,
    which every ray's walk ends with, has to have a value too."""
    rc, err = _syntax("""
#include "gsr_internal.h"
constexpr bool every_bit()
{
    for (uint32_t k = 0; k < 32; ++k)
        if (gsr::lowest_bit(1u << k) != k || gsr::lowest_bit(0xFFFFFFFFu << k) != k) return false;
    return true;
}
static_assert(every_bit(), "lowest set bit");
static_assert(gsr::lowest_bit(0u) == 31u, "an empty mask");
""", tmp_path)
    assert rc == 0, err


def test_tile_scan_fits_lds_for_images_of_any_sides(tmp_path):
    """Two images of one launch, each of at most 15,000 tiles and 1,024 tile
    columns and rows: the scan's LDS holds the tile differences of both and, with
    the 4,160 bytes of the kernel's own, no more than a CU has."""
    rc, err = _syntax("""
#include "gsr_internal.h"
constexpr bool fits(long ax, long ay, long bx, long by)
{
    const long t_max = ax * ay > bx * by ? ax * ay : bx * by, ty_max = ay > by ? ay : by;
    const long lds = (long)gsr::tile_scan_lds((int)t_max, (int)ty_max);
    return lds >= 4 * (ax + 1) * ay && lds >= 4 * (bx + 1) * by && lds + 4160 <= 160 * 1024;
}
constexpr long most(long side) { return side * 1024 <= 15000 ? 1024 : 15000 / side; }
constexpr bool all()
{
    for (long a = 1; a <= 1024; a += a < 64 ? 1 : 31)
        for (long b = 1; b <= 1024; b += b < 64 ? 1 : 31)
            if (!fits(a, most(a), most(b), b) || !fits(most(a), a, b, most(b))) return false;
    return true;
}
static_assert(all() && fits(200, 1, 1, 200) && fits(200, 63, 63, 200), "k_tile_scan");
""", tmp_path)
    assert rc == 0, err
