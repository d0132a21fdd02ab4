// Internal declarations shared by the HIP kernels and the host runtime of
// libgsr (batched 3D Gaussian Splatting for rigid-body environments).
//
// Every file of the library is compiled with -ffp-contract=off: the binning
// arithmetic (projection, culls, radius, tile rectangle, depth key) is
// specified operation by operation in IEEE binary32 so that sort keys and tile
// lists are reproducible bit for bit.  Kernels that want fused multiply-adds
// (the rasteriser) call fmaf() explicitly.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "gsr.h"

namespace gsr {

constexpr uint32_t kInvalidKey = 0xFFFFFFFFu;  // depth-key slot of a culled Gaussian
constexpr int kMaxShDegree = 3;

// Attribute storage formats of a resident scene.
enum Storage : int { kF32 = 0, kF16 = 1, kBF16 = 2 };

// Per-image description inside one launch (device resident).  Images of one
// launch may come from several render requests: every image carries its own
// input offsets and output pointers.
struct ImageInfo {
    int width, height;
    int tiles_x, tiles_y;
    float fx, fy, cx, cy, near_plane;
    float guard_x, guard_y;   // Jacobian clamp of x/z, y/z: 1.3 * ((0.5 W) / fx), same in y (binary32)
    uint32_t key_tile_base;   // first global tile id of the image in its request (sort keys)
    const float* viewmat;     // the image's world->camera [R | t] in the caller's viewmat array
    const float* poses;       // the image's env body poses [B][7] in the caller's pose array (null without bodies)
    float bg[3];              // background colour of the image's request
    int attach_body;          // -1: viewmat is world->camera; b: viewmat is body-b->camera
    float* out_rgb;           // first pixel of the image: [H][W][3] or null
    float* out_depth;         // [H][W]
    float* out_alpha;         // [H][W] or null
    uint32_t* out_work;       // [H][W][2] (visited entries, blended Gaussians) or null
    void* out_obs;            // observation epilogue output [H][W][3] (u8 or half) or null
    const float* obs_gain;    // per-image parameters (indexed by obs_idx) or null
    const float* obs_contrast;
    const float* obs_bright;
    int obs_fmt;              // GSR_OBS_U8 / GSR_OBS_F16
    uint32_t obs_idx;         // c * E + e within the image's request
    // LiDAR images (kind 1 angular, 2 heightmap grid, 3 listed rays): width x height rays, range ->
    // out_depth, hit -> out_alpha
    int kind;                 // 0 camera, 1 angular LiDAR, 2 heightmap grid, 3 listed rays
    float az0, az_step;       // kind 1: ray azimuths az0 + (c + 0.5) az_step
    const float* elev;        // kind 1: device [height] beam elevations, ascending; kind 3: [2][height]
                              // smallest, then largest elevation of each band (both ascending)
    float gx0, gy0, gdx, gdy; // kind 2: ray (r, c) starts at (gx0 + (c + 0.5) gdx, gy0 + (r + 0.5) gdy, 0), along -z
    const float* ray_az;      // kind 3: device [height][width] azimuths, ascending within each band
    const float* ray_el;      // kind 3: device [height][width] elevations
    const uint32_t* ray_perm; // kind 3: device [height][width] caller's index of each ray (output position)
    const float* ray_tile_az; // kind 3: device [2][tiles_y][tiles_x] smallest, then largest azimuth of each
                              // ray tile (both ascending along a tile row)
};

// Resident scene, device pointers.
struct SceneDev {
    int64_t n;            // Gaussians
    int64_t n_pad;        // plane stride (n rounded up to 64)
    int degree;           // SH degree 0..3
    int storage;          // Storage
    int n_bodies;
    int sh_chunks;        // 16-byte chunks of SH per Gaussian
    const float4* pos;    // [n] (x, y, z, opacity); means are always float32
    const void* rot;      // F32: float4 quaternion [n]; F16/BF16: uint4 = 8 halves (qw qx qy qz sx sy sz 0) [n]
    const float4* scale;  // F32 only: (sx, sy, sz, 0) [n]
    const void* sh;       // planes [sh_chunks][n_pad] of 16 bytes
    const int* body_off;  // [n_bodies + 1] (int32): [0, off[0]) static, body b = [off[b], off[b+1])
};

// Segment of the chunk that shares one camera slot (uniform resolution).
struct RasterSeg {
    uint32_t first_image;  // first chunk-local image
    uint32_t n_images;
    uint32_t tiles_per_image;
};
constexpr int kMaxSegs = 8;
constexpr int kRect4MaxTiles = 255;

// Streaming store of 16 bytes: non-temporal, for whole cache lines of a
// stream that is read back only after it has left L2 and the Infinity Cache
// (the projection's records, written 1 KB per wave instruction).  Scattered
// or partial-line streams keep ordinary stores, which L2 combines.
__device__ __forceinline__ void store_stream(float4* p, float4 v)
{
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    const f32x4 w = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(w, reinterpret_cast<f32x4*>(p));
}

// Tile rectangle [x0, x1) x [y0, y1) of entry k in either format.
__device__ __forceinline__ void put_rect(void* a, int rect4, size_t k, uint32_t x0, uint32_t x1, uint32_t y0,
                                         uint32_t y1)
{
    if (rect4) static_cast<uint32_t*>(a)[k] = x0 | (x1 << 8) | (y0 << 16) | (y1 << 24);
    else static_cast<uint2*>(a)[k] = make_uint2(x0 | (x1 << 16), y0 | (y1 << 16));
}
// Raw entry k (the u32 in .x for the packed format), decoded by decode_rect.
__device__ __forceinline__ uint2 raw_rect(const void* a, int rect4, size_t k)
{
    return rect4 ? make_uint2(static_cast<const uint32_t*>(a)[k], 0u) : static_cast<const uint2*>(a)[k];
}
__device__ __forceinline__ void decode_rect(uint2 r, int rect4, uint32_t* x0, uint32_t* x1, uint32_t* y0,
                                            uint32_t* y1)
{
    if (rect4) {
        *x0 = r.x & 0xFFu;
        *x1 = (r.x >> 8) & 0xFFu;
        *y0 = (r.x >> 16) & 0xFFu;
        *y1 = r.x >> 24;
    } else {
        *x0 = r.x & 0xFFFFu;
        *x1 = r.x >> 16;
        *y0 = r.y & 0xFFFFu;
        *y1 = r.y >> 16;
    }
}

// Per-chunk device buffers and sizes handed to the kernels.
struct ChunkDev {
    uint64_t n;                // Gaussians of the scene (dense row length)
    int n_img;
    int t_max;                 // largest tile count of an image in the chunk
    int sort_blocks;           // depth-sort blocks per image (pass 0: ceil(n / kSortItems))
    int tile_blocks;           // tile-pass blocks per image (ceil(n / tile_items))
    int tile_items;            // depth-ordered Gaussians per tile-pass block (level 1: one wave each)
    const ImageInfo* img;      // [n_img]
    float* xform;              // [n_img][n_bodies + 1][16]
    // What the projection writes per (image, Gaussian).  Cameras: in slots, the
    // visible Gaussians of each 64 consecutive ones (a wave's) packed to the
    // front of the 64 slots, in index order, so slots order like indices; the
    // ids of the sort and of the lists are slots, and `vmask` maps them back.
    // LiDAR: a Gaussian's slot is its index.
    uint32_t* keyz;            // [n_img][n] depth bits or kInvalidKey
    uint2* rect;               // [n_img][n] tile rectangle (format: rect4 below)
    float4* rec;               // [n_img][n][3] raster records ([..][4] for LiDAR)
    uint64_t* vmask;           // [n_img][ceil(n / 64)] visible Gaussians of each 64 (debug runs; else null)
    uint32_t* sk[2];           // depth-sort keys, ping-pong [n_img][n]
    uint32_t* sv[2];           // depth-sort values (Gaussian ids); sorted result in sv[0]
    uint2* srect;              // [n_img][n] tile rectangle of the j-th depth-ordered Gaussian
    uint32_t* sort_hist;       // [n_img][sort_blocks][512]
    uint32_t* kmm;             // [n_img][kKmmStride]: smallest visible key rounded down to 512, largest
    uint32_t* kblk;            // [n_img][sort_blocks][2] smallest, largest visible key of each pass-0 block
    uint32_t* vis_count;       // [n_img] visible Gaussians V_i
    int32_t* tile_hist;       // [n_img][(tx_max + 1) (ty_max + 1)] 2D difference array of tile counts
    uint32_t* tile_range;      // [n_img][t_max][2] local [start, end)
    uint32_t* pair_count;      // [n_img] P_i
    uint32_t* longest;         // [n_img] entries of the image's longest tile list (LiDAR; else null)
    uint64_t* pair_base;       // [n_img + 2] exclusive prefix of P_i, total pairs, total visible
    uint32_t* pairs;           // [total pairs] Gaussian id per (tile, depth)-sorted entry
    int ty_max;                // largest tile-row count of an image in the chunk
    int tx_max;                // largest tile-column count
    // Rectangle format of rect / srect: 1 = one u32 per entry, bytes (x0, x1, y0,
    // y1), used when every image has at most kRect4MaxTiles tiles per axis; 0 =
    // one uint2 per entry (x0 | x1 << 16, y0 | y1 << 16).
    int rect4;
    uint32_t* row_hist;        // [n_img][tile_blocks][ty_max] per-block row counts, then offsets
    uint32_t* row_range;       // [n_img][ty_max][2] local [start, end) of each tile-row list
    uint32_t* row_count;       // [n_img] R_i (entries of all row lists)
    uint64_t* row_base;        // [n_img + 1] exclusive prefix of R_i
    uint2* rows;               // [total row entries] (Gaussian id, x0 | x1 << 16) per (row, depth)-sorted entry
    uint32_t* err;             // device word of the context: kErr* bits set by a kernel that meets an entry its
                               // inputs cannot contain (checked by the host at every chunk; poisons the context)
    // List capacity of the chunk (entries of `pairs` and `rows`).  k_image_scan
    // compares the chunk's totals with them and sets *ovf; an overflowed chunk
    // writes no lists and is composited by the fallback rasteriser, which
    // filters each tile's list from the depth-ordered Gaussians instead.
    uint64_t cap_pairs, cap_rows;
    uint32_t* ovf;             // device word of the workspace: 1 = this chunk's lists do not fit
    // pinned host memory of the workspace, written by k_image_scan: the chunk's
    // totals and the consistency bits (pairs, row entries, visible Gaussians,
    // bits, longest tile list; null where the host does not wait for them), and a
    // word set to 1 when a chunk overflowed
    uint64_t* host_totals;
    uint32_t* host_ovf;
    uint32_t* fallback_counter;   // kXcds tile counters of the fallback rasteriser, zeroed by k_image_scan (or null)
    unsigned long long* acc;   // device accumulators of the context: visible Gaussians, pairs, row entries
};

// Bits of ChunkDev::err.
constexpr uint32_t kErrListEntry = 1u;    // a tile list held a Gaussian id >= n
constexpr uint32_t kErrSortSlot = 2u;     // a depth-sort rank or offset fell outside its segment
constexpr uint32_t kErrRowEntry = 4u;     // a depth-ordered id >= n reached the tile-row expansion

// Depth sort geometry.
// Words per image of ChunkDev::kmm (smallest and largest visible key).
constexpr int kKmmStride = 2;
constexpr int kSortBlock = 256;
constexpr int kSortIpt = 16;
constexpr int kSortItems = kSortBlock * kSortIpt;   // 4096 items per block
// Tile pass geometry: k_tile_hist counts kTileGauss depth-ordered Gaussians per
// block; level 1 places `tile_items` of them per wave (tile_items_for).
constexpr int kTileGauss = 4096;
constexpr int kTileItemsMin = 128;
constexpr int kLevel1Waves = 16384;
// Items per level-1 wave: a wave walks its items in dependent groups of 64, so
// a launch of few images is cut into more, shorter waves until it has about
// kLevel1Waves of them (a single 640x480 image of 300k Gaussians: one wave per
// 4096 items took 201 us with 74 waves on the chip, 256 items 29 us; 128
// instead of 256 as the least takes 5 us more off its 283 us, twice the waves
// 1 % off 64 images of 320x240 and 1.6 % off 64 rosette scans).  Large
// launches keep 4096: every block starts and ends its row lists with partial
// lines, and the scan of block offsets grows with the blocks.  The rows counted
// per block also have to fit the LDS of k_tile_hist beside its tile counts.
inline int tile_items_for(uint64_t n, uint64_t n_img, int tx_max, int ty_max)
{
    int items = kTileGauss;
    while (items > kTileItemsMin && n * n_img / (uint64_t)items < (uint64_t)kLevel1Waves &&
           ((size_t)(tx_max + 1) * (ty_max + 1) + (size_t)(2 * kTileGauss / items) * (ty_max + 1)) * 4 <= 60 * 1024)
        items /= 2;
    return items;
}
inline int tile_blocks_of(int64_t n, int tile_items)
{
    return (int)std::max<int64_t>(1, (n + tile_items - 1) / tile_items);
}
// Level 2 runs one wave per (image, tile row, segment).  A launch that has
// kLevel2Rows tile rows takes each as one segment: an extra segment costs a
// count pass over its entries.  Fewer rows are cut into kLevel2Waves segments of
// at least kRowSegEntries entries: the entries are in depth order, so a row's
// first segments hold the widest rectangles and take several times as long as
// its last ones, and short segments keep the launch from waiting for those (512
// scans of 32 x 1024 rays, 1024 rows: 3.6 ms with 16 segments per row, 2.1 with
// 128).  A launch that would stay below kLevel2FewWaves waves takes segments of
// down to kRowSegEntriesFew entries: there the longest wave is what it waits for
// (with 256 entries below 4096 waves and with 128 below 32768: one 128x96 image
// 130.5 and 122.8 us, one 640x480 290 and 285, 64 rosette scans 1.85 and 1.71 ms;
// 64 entries cost 37 images of 317x203 2 %).
constexpr int kRowSegEntries = 512;
constexpr int kRowSegEntriesFew = 128;
constexpr int kLevel2Rows = 16384;
constexpr int kLevel2Waves = 131072;
constexpr int kLevel2FewWaves = 32768;
constexpr int kMaxRowSegs = 128;
// Segments per tile-row list of a launch with n_rows tile rows of row_total
// entries in all, at most tx_max tiles each.  A segment also has at least as
// many entries as its row has tiles: its offsets (a word per tile) then take at
// most half the memory of its entries (two words each), whatever the images' width.
constexpr int row_segments(uint64_t n_rows, uint64_t row_total, int tx_max)
{
    if (n_rows == 0 || n_rows >= (uint64_t)kLevel2Rows) return 1;
    const uint64_t per_row = row_total / n_rows, tx = (uint64_t)tx_max;
    uint64_t segs = per_row / std::max<uint64_t>(kRowSegEntries, tx), waves = kLevel2Waves;
    if (n_rows * std::max<uint64_t>(segs, 1) < (uint64_t)kLevel2FewWaves) {
        segs = per_row / std::max<uint64_t>(kRowSegEntriesFew, tx);
        waves = kLevel2FewWaves;
    }
    segs = std::min(segs, (waves + n_rows - 1) / n_rows);
    return (int)std::max<uint64_t>(1, std::min<uint64_t>(kMaxRowSegs, segs));
}

// LDS of k_tile_scan for an image's tile differences ([tiles_y][tiles_x + 1]
// words) of a chunk's largest image.  Not tx_max x ty_max: those may come from
// different images, and a wide and a tall one of 200 tiles each would take more
// than the 160 KB there are.  An image has at most 15,000 tiles, 1,024 rows.
constexpr size_t tile_scan_lds(int t_max, int ty_max) { return ((size_t)t_max + (size_t)ty_max) * 4; }

// ------------------------------------------------------------ launchers
// All launchers enqueue on `stream` and return hipGetLastError().
hipError_t launch_compose(const SceneDev& s, const ChunkDev& c, hipStream_t stream);
hipError_t launch_project(const SceneDev& s, const ChunkDev& c, int ts, float cutoff, int img_per_thread,
                          hipStream_t stream);
hipError_t launch_depth_sort(const SceneDev& s, const ChunkDev& c, hipStream_t stream);
// Tile and tile-row histograms, ranges, image bases (before the host reads the
// totals), and the order of the tiles where p asks for one.
struct RasterParams;
hipError_t launch_tile_count(const SceneDev& s, const ChunkDev& c, const RasterParams& p, hipStream_t stream);
// LiDAR: projection into the ray grid (keys = centre distance, conservative
// angular tile rectangles, 64-byte whitening and cone records) and per-ray compositing.
hipError_t launch_project_lidar(const SceneDev& s, const ChunkDev& c, int ts, int ipt, hipStream_t stream);

// Stable two-level scatter: depth-ordered Gaussians -> tile-row lists -> tile lists.
// schedule 0: both levels as stable expansions (two slots per lane, ranks
// from per-bucket lane masks); 1: by transposed ranks (a 64 x 64 bit transpose
// gives each bucket lane its items, each item places itself in its buckets).
// Both give identical lists.
// n_seg: segments per tile-row list (seg_off: n_img * ty_max * n_seg * tx_max
// words of scratch when n_seg > 1).
hipError_t launch_tile_scatter(const SceneDev& s, const ChunkDev& c, int schedule, int n_seg, uint32_t* seg_off,
                               hipStream_t stream);
struct RasterParams {
    int ts;                  // tile side: 8, 16 or 32
    int batch;               // records staged in LDS per round
    int persistent;          // 1: persistent workgroups pulling tiles from `counter`
    int count_work;          // 1: images carry out_work (counting instantiation)
    int persistent_blocks;   // workgroups of the persistent launch
    uint32_t* counter;       // device tile counters, one per XCD (persistent launch)
    int n_segs;
    RasterSeg segs[kMaxSegs];
    uint32_t n_blocks;
    uint64_t entries;        // LiDAR: of the chunk's tile lists, and of the longest of them
    uint64_t longest;
    uint32_t* order;         // heavy-first order of each XCD's part (k_image_scan_order), or null: as they come
};
// Launches of more than kOrderTilesMin tiles (up to that all are resident at
// once: five workgroups per CU) and at most kOrderTilesMax take their tiles
// heavy first.  Above, image and tile no longer fit a word of 16 bits each, the
// ordering blocks would have more than eight tiles a thread, and the longest tile
// is a small part of the launch: scans of 32 x 1024 rays over 300k Gaussians take
// 23.1 us each in launches of 480 and of 512 (65,536 tiles), 23.0 of 513 and of
// 520, 22.7 of 640.
constexpr uint32_t kOrderTilesMin = 1280;
constexpr uint32_t kOrderTilesMax = 65536;
// Launches whose tiles hold at most kShortList entries on average: their time is
// what a tile sets up.  Their images are not dealt out by list entries (a ranking
// that takes 0.04 us an image), and LiDAR launches of more tiles than are resident
// at once take a kernel of fewer culling steps, unless some list is long
// (kShortLongest).  With the dealing and the full kernel, and without: 512 scans of
// 32 x 1024 rays over 500, 2,000, 4,000 and 8,000 Gaussians 509, 579, 614 and 737
// us and 345, 430, 496 and 684, the last of about 90 entries a tile; 1,024 of
// 16 x 360 over 2,000 and 8,000 438 and 667, and 364 and 666; 1,000 images of 64x64
// over 2,000 299 and 261.  40 heightmaps of 16 tiles, resident at once, lose 4 %
// with the smaller kernel, and one list of 4,000 entries takes it 0.2 ms longer;
// with lines at 256 and 1,024 entries the times above differ by less than 1 %.
constexpr uint64_t kShortList = 96;
constexpr uint64_t kShortLongest = 512;
__host__ __device__ inline bool short_lists(uint64_t entries, uint32_t n_blocks)
{
    return entries <= kShortList * n_blocks;
}
hipError_t launch_raster_lidar(const SceneDev& s, const ChunkDev& c, const RasterParams& p, hipStream_t stream);
hipError_t launch_raster(const SceneDev& s, const ChunkDev& c, const RasterParams& p, hipStream_t stream);
// Fallback compositing of a chunk whose lists overflowed (a persistent grid
// that exits at once when the chunk's lists fit; its tile counters are
// ChunkDev::fallback_counter).
hipError_t launch_raster_fallback(const SceneDev& s, const ChunkDev& c, const RasterParams& p, hipStream_t stream);

// Scene upload: convert caller float32 attributes to resident storage.
hipError_t launch_scene_convert(int storage, int64_t n, int64_t n_pad, int degree, const float* means,
                                const float* scales, const float* quats, const float* opac, const float* sh,
                                float4* pos, void* rot, float4* scale, void* sh_planes, hipStream_t stream);

// Debug: 64-bit keys and Gaussian indices of one image from its sorted pairs.
hipError_t launch_debug_keys(const ChunkDev& c, int image, uint64_t n, const uint32_t* pairs, uint64_t n_pairs,
                             uint64_t* keys_out, uint32_t* ids_out, hipStream_t stream);
// Debug: the projections' reciprocal or square root (GSR_ROOT_*) of the values with the bits first, first + 1, ...
hipError_t launch_debug_roots(int root, uint32_t first, uint32_t count, float* out, hipStream_t stream);
// Index of the k-th set bit of m (k < popcount(m)).
__host__ __device__ inline uint32_t select_bit(uint64_t m, uint32_t k)
{
    for (; k > 0; --k) m &= m - 1;
    return (uint32_t)__builtin_ctzll(m);
}

// Index of the lowest set bit of m, 31 for m = 0.
__host__ __device__ constexpr uint32_t lowest_bit(uint32_t m)
{
    return (uint32_t)__builtin_ctz(m | 0x80000000u);
}

// Workgroups of a launch are handed to the chip's 8 XCDs round-robin by
// linear id, and each XCD has its own L2.  xcd_remap renumbers linear id b of
// a G-workgroup launch so that each XCD runs one contiguous range of logical
// ids: neighbouring work (the tiles or blocks of one image) then shares one
// L2 instead of being fetched into all eight.  A bijection of [0, G).
constexpr int kXcds = 8;

__host__ __device__ inline uint32_t xcd_remap(uint32_t b, uint32_t G)
{
    const uint32_t q = G / kXcds, r = G % kXcds, x = b % kXcds, k = b / kXcds;
    return x * q + (x < r ? x : r) + k;
}

// The k-th tile of part x of a chunk's tiles cut into `parts` parts (the XCDs
// that have workgroups): chunk-local image and tile in it.  Each segment is
// cut into contiguous ranges by itself, its remainder dealt out from where the
// last segment's ended, so that parts differ by at most one tile in all and
// every part gets its share of every image size.  One cut through all segments
// gave the first XCD the images of the first: the 256 wrist views of 128x128
// before 256 head views of 640x480 kept it busy to 13.9 ms, the others to 10.5.
__host__ __device__ inline void tile_of(const RasterParams& p, uint32_t x, uint32_t k, uint32_t parts, int* image,
                                        uint32_t* tile)
{
    uint32_t from = 0;                  // part that takes the segment's first extra tile
    RasterSeg seg = p.segs[0];
    uint32_t rel;
    for (int s = 0;;) {
        const uint32_t n = seg.n_images * seg.tiles_per_image, q = n / parts, r = n % parts;
        const uint32_t xs = x >= from ? x - from : x + parts - from;
        const uint32_t count = q + (xs < r ? 1u : 0u);
        rel = xs * q + (xs < r ? xs : r) + k;
        if (++s == p.n_segs || k < count) break;
        k -= count;
        from += r;
        if (from >= parts) from -= parts;
        seg = p.segs[s];
    }
    const uint32_t io = rel / seg.tiles_per_image;
    *image = (int)(seg.first_image + io);
    *tile = rel - io * seg.tiles_per_image;
}

// The tile of workgroup b of a launch of p.n_blocks workgroups, one per tile.
__device__ __forceinline__ void tile_of_block(const RasterParams& p, uint32_t b, int* image, uint32_t* tile)
{
    if (p.order) {
        // (at most 65,536 tiles: both fit 16 bits)
        const uint32_t v = p.order[xcd_remap(b, p.n_blocks)];
        *image = (int)(v >> 16);
        *tile = v & 0xFFFFu;
        return;
    }
    tile_of(p, b % (uint32_t)kXcds, b / (uint32_t)kXcds, (uint32_t)kXcds, image, tile);
}

}  // namespace gsr
