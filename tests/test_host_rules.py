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


def _run(text, tmp_path):
    """Builds `text` as a host program (what it does not call may stay
    undefined) and returns its exit status and output."""
    src, obj, exe = (str(tmp_path / f) for f in ("t.hip", "t.o", "t"))
    with open(src, "w") as f:
        f.write(text)
    subprocess.run([build.HIPCC, *build.FLAGS, "--offload-host-only", "-c", src, "-o", obj], check=True,
                   capture_output=True)
    subprocess.run([build.HIPCC, "-o", exe, obj, "-Wl,--unresolved-symbols=ignore-all"], check=True, capture_output=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    return r.returncode, r.stdout


def test_totals_without_a_device_address_are_not_taken_as_allocated(tmp_path):
    """The device address of a working set's pinned totals is refused twice and
    then given: every call reports what it got, and none leaves the kernels an
    address that is not one."""
    rc, out = _run("""
#include <stdio.h>
#include <stdlib.h>
#include <hip/hip_runtime.h>
static int refuse = 2, held = 0;
static hipError_t fake_alloc(void** p, size_t n, unsigned) { *p = malloc(n); ++held; return hipSuccess; }
static hipError_t fake_free(void* p) { free(p); --held; return hipSuccess; }
static hipError_t fake_address(void** d, void* h, unsigned)
{
    if (refuse-- > 0) return hipErrorInvalidValue;
    *d = h;
    return hipSuccess;
}
#define hipHostMalloc(p, n, f) fake_alloc(p, n, f)
#define hipHostFree(p) fake_free(p)
#define hipHostGetDevicePointer(d, h, f) fake_address(d, h, f)
#include "gsr_api.cpp"
int main()
{
    gsr::Workspace* ws = new gsr::Workspace();      // not destroyed: no device
    for (int k = 0; k < 4; ++k) {
        const hipError_t e = gsr::alloc_totals(*ws);
        if ((e == hipSuccess) != (k >= 2) || (e == hipSuccess) != (ws->d_total != nullptr)) return printf("call %d\\n", k), 1;
        if (held != (k >= 2 ? 1 : 0)) return printf("held %d after call %d\\n", held, k), 1;
    }
    return 0;
}
""", tmp_path)
    assert rc == 0, out


def test_segment_offsets_stay_within_half_of_the_row_lists(tmp_path):
    """Level-2 segments over launches of every row count, list length and
    width: their offsets take at most half the bytes of the row lists that they
    divide, and images of up to 128 tile columns keep the numbers of segments
    that the launch's waves ask for."""
    rc, out = _run("""
#include <stdio.h>
#include "gsr_internal.h"
int main()
{
    long many = 0;
    for (uint64_t rows = 1; rows <= 40000; rows = rows * 5 / 4 + 1)
        for (uint64_t per = 0; per <= 4000000; per = per * 3 / 2 + 1)
            for (int tx = 1; tx <= 1024; tx = tx * 2 + (tx > 100)) {
                const int s = gsr::row_segments(rows, rows * per, tx), narrow = gsr::row_segments(rows, rows * per, 1);
                const bool ok = s >= 1 && s <= gsr::kMaxRowSegs && s <= narrow && (tx > 128 || s == narrow) &&
                                (s == 1 || (uint64_t)s * tx * 4 * rows <= rows * per * 8 / 2);
                if (!ok) return printf("rows %lu entries %lu tx %d: %d segments\\n", rows, per, tx, s), 1;
                many += s > 1;
            }
    return many < 1000;
}
""", tmp_path)
    assert rc == 0, out


def test_tile_pass_blocks_stay_within_the_memory_budget(tmp_path):
    """Chunk plans over scenes, image sides and budgets: smaller tile-pass
    blocks are planned only as far as their row counts fit the chunk's budget
    beside what the estimate counts, all of them where there is room, and a
    served request is charged for the blocks of any launch that it ends up in."""
    rc, out = _run("""
#include <stdio.h>
#include "gsr_api.cpp"
using namespace gsr;
int main()
{
    gsr_ctx* ctx = new gsr_ctx();           // neither is destroyed: no device
    SceneRes* sc = new SceneRes();
    const int sides[][2] = {{640, 480}, {128, 96}, {1920, 1080}, {112, 8192}, {8192, 112}};
    long refined = 0, bounded = 0;
    for (const long n : {1l, 5000l, 300000l, 3000000l})
        for (const auto& wh : sides)
            for (const int images : {1, 7, 64}) {
                sc->dev.n = n;
                std::vector<ImageInfo> imgs((size_t)images);
                for (ImageInfo& im : imgs) {
                    im.tiles_x = (wh[0] + 15) / 16;
                    im.tiles_y = (wh[1] + 15) / 16;
                }
                const size_t one = image_bytes_estimate(sc, wh[0], wh[1], 16), all = one * (size_t)images;
                const size_t coarse = (size_t)tile_blocks_of(n, kTileGauss) * (size_t)imgs[0].tiles_y * 4 * (size_t)images;
                const int want = tile_items_for((uint64_t)n, (uint64_t)images, imgs[0].tiles_x, imgs[0].tiles_y);
                for (const size_t spare : {(size_t)0, (size_t)4096, all / 256, all}) {
                    const ChunkPlan p = plan_chunks(ctx, sc, imgs, false, 0, 48, (int64_t)(all + spare));
                    const size_t rows = (size_t)p.tile_blocks * (size_t)p.ty_max * 4 * (size_t)p.chunk;
                    if (p.chunk != images || p.tile_blocks != tile_blocks_of(n, p.tile_items)) return printf("plan\\n"), 1;
                    if (rows > coarse + spare) return printf("n %ld side %d: %zu over\\n", n, wh[0], rows - coarse - spare), 1;
                    if (spare == all && p.tile_items != want) return printf("n %ld side %d: %d items\\n", n, wh[0], p.tile_items), 1;
                    refined += p.tile_items < kTileGauss;
                    bounded += p.tile_items > want;
                }
                // charged by the request's own images: a larger launch has no smaller blocks
                for (const int with : {images, 3 * images + 1}) {
                    const int items = tile_items_for((uint64_t)n, (uint64_t)with, imgs[0].tiles_x, imgs[0].tiles_y);
                    const size_t rows = (size_t)tile_blocks_of(n, items) * (size_t)imgs[0].tiles_y * 4;
                    if (rows > coarse / (size_t)images + image_block_bytes(sc, wh[0], wh[1], 16, images)) return printf("charge\\n"), 1;
                }
            }
    return !(refined > 20 && bounded > 20);
}
""", tmp_path)
    assert rc == 0, out
