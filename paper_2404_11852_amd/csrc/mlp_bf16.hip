// Feature Gathering + Feature Computation (Sec. II-B) with the MLP in BF16
// on MFMA (FP32 accumulation), in ray order or, on dense grids, in voxel
// order from LDS-staged bricks (Sec. IV-A).
#include "mlp_common.h"

namespace cic {

// BF16 compute: the view-encoding inputs of every ray with live samples,
// rounded to BF16 (the rounding the MLP kernel applies to its inputs).  Row of
// a ray: for each lane half 15 values and a zero; half 0: the direction and
// the 12 sines, half 1: the 12 cosines and three ones (layer 0's bias).  Four
// threads per ray, three encoding arguments each.
__global__ __launch_bounds__(256) void k_ray_encode_bf16(RenderBufs b)
{
    __shared__ __attribute__((aligned(16))) __bf16 rows[64][32];   // stored 16 bytes per thread
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t ray = t >> 2;
    const int q = (int)(t & 3);
    const bool live = ray < b.n && b.count[ray] != 0;
    __bf16 *row = rows[threadIdx.x >> 2];
    if (live) {
        float d[3], x[7];
#pragma unroll
        for (int a = 0; a < 3; ++a) d[a] = b.rays_d[3 * ray + a];
        encode_group(d, q, x);
        row[q < 3 ? q : 15] = (__bf16)x[0];   // (the fourth thread's is the pad, 0)
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            row[3 + 3 * q + k] = (__bf16)x[1 + 2 * k];
            row[16 + 3 * q + k] = (__bf16)x[2 + 2 * k];
        }
        row[16 + 12 + q] = (__bf16)(q < 3 ? 1.0f : 0.0f);
    }
    __syncthreads();
    if (live) *(u4_t *)(b.enc + ray * 16 + 4 * q) = *(const u4_t *)(row + 8 * q);
}

void launch_ray_encode_bf16(const RenderBufs &b, hipStream_t s)
{
    if (b.n == 0) return;
    const int64_t threads = 4 * b.n;
    hipLaunchKernelGGL(k_ray_encode_bf16, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, s, b);
}

// ---------------------------------------------------------------------------
// Voxel order with LDS-staged bricks (the memory-centric rendering of Sec.
// IV-A): workgroups claim segments of up to kTileSeg samples of one brick of
// 8^3 voxels, stage the brick's 9^3 vertices x 12 feature channels in LDS
// (44 KB as float32) together with the segment's per-sample records (record
// index, ray, voxel fractions and cell within the brick, 24 B per sample),
// and then run the MLP batches from LDS.  Each feature vertex is read from
// the grid once per segment instead of by every sample near it, and the
// dependent loads that locate a sample (its record, its ray, the ray's
// origin and direction) are issued by the whole workgroup at once.
// ---------------------------------------------------------------------------
// Launch shapes.  The gathering kernel (ray order): 8 wavefronts per CU (two
// per SIMD), 64 samples per batch, the next batch's gather among this batch's
// MFMAs.  The brick kernels: 16 wavefronts of 32 samples, whose batches come
// from LDS and are short between the segments' barriers.
constexpr int kRayWaves8 = 8;
constexpr int kBfWaves = 16;                  // wavefronts per workgroup of the brick kernels
constexpr int kBfBatch = 32;                  // samples per wavefront batch there
constexpr int kTileThreads = kBfWaves * 64;   // threads of a workgroup there

constexpr int kFTileV = kBrick + 1;
// Brick tile: channel ch of vertex (lx, ly, lz) at
// ch * kFTileS + lx * kFTileSX + ly * kFTileSY + lz * kFTileSZ.  One gather
// instruction reads one channel of the 32 samples' corner for either lane half,
// six channels apart; the samples of a batch lie along one or two rays through
// the brick, so their cells are near neighbours.  The strides were chosen for
// few LDS bank collisions (64 banks) of a gather by 16 samples and four lane
// groups, three channels apart, and not measured again for this one: there the
// channel stride puts the lane groups 16 banks apart, so two cells collide when
// their offsets differ by a multiple of 16 words.  Among cell steps of at
// most 2 per axis, 10 do so with the dense x stride of 81 (+-(1, 0, -1) among
// them: 80 words) and 6 with the x stride of 102 (+-(1, 1, 1): 112 words,
// and +-(0, 2, -2) as before).  Estimated on
// voxel-ordered samples of an 800x800 view: 1.35 distinct words per bank per
// instruction against 1.82 for the dense 9 x 81 x 752 layout; the 8-view
// pass measured 0.5-1.2% faster over three runs (bank conflicts are not what
// bounds the batches).
#ifndef CIC_TILE_SZ
#define CIC_TILE_SZ 1
#endif
#ifndef CIC_TILE_SY
#define CIC_TILE_SY 9
#endif
#ifndef CIC_TILE_SX
#define CIC_TILE_SX 102
#endif
#ifndef CIC_TILE_CS
#define CIC_TILE_CS 912
#endif
constexpr int kFTileSZ = CIC_TILE_SZ, kFTileSY = CIC_TILE_SY, kFTileSX = CIC_TILE_SX, kFTileS = CIC_TILE_CS;
constexpr int kFTileMax = 11 * kFTileS + (kFTileV - 1) * (kFTileSX + kFTileSY + kFTileSZ);   // largest index
constexpr int kFTileFloats = (kFTileMax + 4) & ~3;
constexpr bool tile_layout_injective()
{
    bool used[kFTileFloats] = {};
    for (int ch = 0; ch < 12; ++ch)
        for (int x = 0; x < kFTileV; ++x)
            for (int y = 0; y < kFTileV; ++y)
                for (int z = 0; z < kFTileV; ++z) {
                    const int i = ch * kFTileS + x * kFTileSX + y * kFTileSY + z * kFTileSZ;
                    if (used[i]) return false;
                    used[i] = true;
                }
    return true;
}
static_assert(tile_layout_injective(), "brick tile layout puts two values in one word");
// Segment records in LDS (structure of arrays, kTileSeg entries each):
// record index, ray, three voxel fractions, packed cell (lx | ly << 4 | lz << 8).
constexpr int kSegWords = 6 * kTileSeg;

// origin vertex of a brick (kept in registers by the callers)
struct BrickBase {
    int x, y, z;
};
__device__ __forceinline__ BrickBase brick_base(const GridK &g, int64_t brick)
{
    const int bz = (int)(brick % g.nb2), by = (int)((brick / g.nb2) % g.nb1);
    const int bx = (int)(brick / ((int64_t)g.nb2 * g.nb1));
    return BrickBase{kBrick * bx, kBrick * by, kBrick * bz};
}

template <typename T>
__device__ void load_feature_tile(const GridK &g, const BrickBase base, float *tile)
{
    const T *feat = (const T *)g.features;
    for (int e = threadIdx.x; e < kFTileV * kFTileV * kFTileV * 3; e += blockDim.x) {
        const int vtx = e / 3, part = e - 3 * vtx;
        const int lz = vtx % kFTileV, ly = (vtx / kFTileV) % kFTileV, lx = vtx / (kFTileV * kFTileV);
        const int vx = base.x + lx, vy = base.y + ly, vz = base.z + lz;
        const int tv = lx * kFTileSX + ly * kFTileSY + lz * kFTileSZ;
        f4_t v = f4_t{0.f, 0.f, 0.f, 0.f};
        if (vx < g.r0 && vy < g.r1 && vz < g.r2) {
            const int64_t off = vertex_index(g, vx, vy, vz) * 12 + 4 * part;
#pragma unroll
            for (int c = 0; c < 4; ++c) v[c] = ldv(feat, off + c);
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) tile[(4 * part + c) * kFTileS + tv] = v[c];
    }
}

// Features 3q..3q+2 of a sample in cell (lx, ly, lz) of the staged brick
// (same interpolation order as the gather from the grid).
__device__ __forceinline__ void tile_gather3(const float *tile, int lx, int ly, int lz, const float fr[3], int q,
                                             float x[3])
{
    const int sx = kFTileSX, sy = kFTileSY, sz = kFTileSZ;
    const float *t = tile + lx * kFTileSX + ly * kFTileSY + lz * kFTileSZ + 3 * q * kFTileS;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const float *u = t + c * kFTileS;
        const float v000 = u[0], v001 = u[sz], v010 = u[sy], v011 = u[sy + sz];
        const float v100 = u[sx], v101 = u[sx + sz], v110 = u[sx + sy], v111 = u[sx + sy + sz];
        const float c00 = lerpf(v000, v001, fr[2]), c01 = lerpf(v010, v011, fr[2]);
        const float c10 = lerpf(v100, v101, fr[2]), c11 = lerpf(v110, v111, fr[2]);
        const float c0 = lerpf(c00, c01, fr[1]), c1 = lerpf(c10, c11, fr[1]);
        x[c] = lerpf(c0, c1, fr[0]);
    }
}

// The segment's per-sample records into LDS (every thread of the workgroup;
// same voxel computation as the march, so the cell and fractions are the
// ones the gather from the grid would use).
__device__ void stage_segment(const GridK &g, const RenderBufs &b, uint32_t start, int n, const BrickBase base,
                              uint32_t *seg)
{
    for (int e = threadIdx.x; e < n; e += blockDim.x) {
        const uint32_t rec = b.perm[start + e];
        SampleRay r;
        load_sample_ray(b, b.rec_ray[rec], b.rec_k[rec], r);
        int i0[3];
        float fr[3], tk;
        sample_voxel(r.o, r.d, r.tn, r.delta, r.k, g, i0, fr, tk);
        seg[e] = rec;
        seg[kTileSeg + e] = r.ray;
        seg[2 * kTileSeg + e] = __float_as_uint(fr[0]);
        seg[3 * kTileSeg + e] = __float_as_uint(fr[1]);
        seg[4 * kTileSeg + e] = __float_as_uint(fr[2]);
        seg[5 * kTileSeg + e] =
            (uint32_t)(i0[0] - base.x) | ((uint32_t)(i0[1] - base.y) << 4) | ((uint32_t)(i0[2] - base.z) << 8);
    }
}

// Claim the next segment (up to kTileSeg samples of one brick) for this
// workgroup.  The segment list is split into kXcds contiguous ranges, one
// per XCD, each drained through its own counter: the workgroups sharing an
// L2 then work through neighbouring bricks (and the rays crossing them)
// instead of the whole chip's in-flight window.  Thread 0 claims the
// segment, finds its brick in the segment table and publishes it in LDS
// (a binary search over the segment offsets per claim measured 1.5% slower
// for the whole stage; claiming the next segment while the current one's
// batches run, with batches handed out through an LDS counter, measured the
// same as this); returns false once this XCD's range is exhausted (every
// workgroup of the XCD then ends).  Large bricks are shared by several
// workgroups, each staging the brick's tile.
// With dense brick tiles, segments are claimed kClaimRun consecutive ones at
// a time, so a brick's segments tend to follow each other in one workgroup,
// which then keeps the brick's staged tile (reuse set) instead of loading it
// again (measured on the 8-view pass: 24.4 ms one at a time, 24.1 ms in runs
// of 2, 23.9 ms in runs of 8).  The multi-level boxes depend on each
// segment's samples, so those segments are claimed one at a time.
#ifndef CIC_CLAIM_RUN
#define CIC_CLAIM_RUN 8
#endif
constexpr int kClaimRun = CIC_CLAIM_RUN;
struct TileWork {
    int64_t brick;
    uint32_t start, end;
    int reuse;   // the staged tile is already this brick's
};
// the claiming thread's state: next index of its current run, the run's end, the brick in the tile
struct ClaimState {
    uint64_t next, end;
    int64_t tile_brick;
};
template <int RUN>
__device__ __forceinline__ bool claim_segment(const RenderBufs &b, TileWork *slot, ClaimState &cs, TileWork &w)
{
    __syncthreads();   // every wave is done with the previous segment and tile
    if (threadIdx.x == 0) {
        const int xcd = blockIdx.x % kXcds;
        const uint64_t nseg = b.seg_off[b.n_bricks];
        const uint64_t hi = nseg * (xcd + 1) / kXcds;
        if (cs.next >= cs.end) {
            cs.next = nseg * xcd / kXcds + atomicAdd(b.work_ctr + xcd, (uint32_t)RUN);
            cs.end = min(cs.next + RUN, hi);
        }
        TileWork t{-1, 0u, 0u, 0};
        if (cs.next < cs.end) {
            const uint64_t k = cs.next++;
            const uint32_t brick = b.seg_brick[k];   // from the segment table
            const uint32_t bstart = brick == 0 ? 0u : b.brick_off[brick - 1], bend = b.brick_off[brick];
            t.brick = brick;
            t.start = bstart + ((uint32_t)k - b.seg_off[brick]) * (uint32_t)kTileSeg;
            t.end = min(bend, t.start + (uint32_t)kTileSeg);
            t.reuse = (int64_t)brick == cs.tile_brick;
            cs.tile_brick = brick;
        }
        *slot = t;
    }
    __syncthreads();
    w = *slot;
    return w.brick >= 0;
}

// ---------------------------------------------------------------------------
// Voxel order with the multi-level encoding (hierarchical encodings, Sec.
// IV-A): the segments are still those of the density grid's bricks.  For each
// segment the workgroup stages its samples' records (record index, ray and
// float32 position) and reduces, per level, the bounding box of the cells the
// samples fall in.  Levels are then taken coarse to fine: a level whose box
// of vertices fits the LDS left over and holds no more vertices than the
// segment's gathers would request (8 per sample) is loaded into LDS once and
// its samples interpolate from there; the other levels (typically the finest,
// whose box is large against the samples that use it) are gathered from the
// table per sample, the plain data flow.  Either way a vertex's value is the
// table's, so the features equal the ray-order gather bit for bit.
// ---------------------------------------------------------------------------
// Level staging rule: 0 = levels whose box fits and holds at most 8 vertices
// per sample of the segment; 1 = the densely stored levels only, when they
// fit; 2 = every level that fits.
#ifndef CIC_HASH_STAGE
#define CIC_HASH_STAGE 0
#endif
constexpr int kHSegWords = 5 * kTileSeg;   // record, ray, position x, y, z
constexpr int kHTileBytes = 66 * 1024;     // LDS for the staged levels' vertices

// one staged vertex: the level's 3 features and a pad, in the table's type
template <typename T> struct HashVtx;
template <> struct HashVtx<float> {
    typedef float type __attribute__((ext_vector_type(4)));
};
template <> struct HashVtx<__half> {
    typedef _Float16 type __attribute__((ext_vector_type(4)));
};

struct HashSegInfo {
    float pmin[kBfWaves][3], pmax[kBfWaves][3];   // per wavefront: bounds of its samples' positions
    int lo[4][3], hi[4][3];   // per level: lowest and highest cell of the segment's samples
    int ext[4][3];            // vertices per axis of the staged box (hi - lo + 2)
    int off[4];               // first staged vertex of the level, -1: gathered from the table
};

__device__ __forceinline__ float wave_min_f(float v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fminf(v, __shfl_xor(v, o, kWave));
    return v;
}
__device__ __forceinline__ float wave_max_f(float v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, kWave));
    return v;
}

// Records of the segment's samples into LDS, and each wavefront's bounds of
// their positions.  A level's cell index along an axis is a non-decreasing
// function of that coordinate (subtract, scale by a positive factor, floor,
// clamp, each monotonic in float32), so the cells of the extreme coordinates
// bound every sample's cells exactly.
__device__ void stage_segment_hash(const GridK &g, const RenderBufs &b, uint32_t start, int n, uint32_t *seg,
                                   HashSegInfo &h)
{
    float mn[3] = {INFINITY, INFINITY, INFINITY}, mx[3] = {-INFINITY, -INFINITY, -INFINITY};
    constexpr int kIter = (kTileSeg + kTileThreads - 1) / kTileThreads;
#pragma unroll
    for (int k = 0; k < kIter; ++k) {
        // out-of-range threads repeat the last sample (its cells do not widen the bounds)
        const int e = (int)threadIdx.x + k * kTileThreads;
        const uint32_t rec = b.perm[start + min(e, n - 1)];
        SampleRay r;
        load_sample_ray(b, b.rec_ray[rec], b.rec_k[rec], r);
        float xp[3];
        sample_position(r, xp);
        if (e < n) {
            seg[e] = rec;
            seg[kTileSeg + e] = r.ray;
#pragma unroll
            for (int a = 0; a < 3; ++a) seg[(2 + a) * kTileSeg + e] = __float_as_uint(xp[a]);
        }
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            mn[a] = fminf(mn[a], xp[a]);
            mx[a] = fmaxf(mx[a], xp[a]);
        }
    }
    const int wave = threadIdx.x / kWave;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const float lo = wave_min_f(mn[a]), hi = wave_max_f(mx[a]);
        if (lane_id() == 0) {
            h.pmin[wave][a] = lo;
            h.pmax[wave][a] = hi;
        }
    }
}

// Where the batches find a level's staged box (off < 0: not staged).
struct LevelTile {
    int off, lo[3], sy, sx;   // sy = ez, sx = ey * ez
};

// Which levels the segment stages, and where (one thread).
template <typename T>
__device__ void plan_hash_levels(const GridK &g, int n, HashSegInfo &h, LevelTile *lt)
{
    constexpr int64_t vb = sizeof(typename HashVtx<T>::type);
    float pmin[3], pmax[3];
    for (int a = 0; a < 3; ++a) {
        pmin[a] = h.pmin[0][a];
        pmax[a] = h.pmax[0][a];
        for (int w = 1; w < kBfWaves; ++w) {
            pmin[a] = fminf(pmin[a], h.pmin[w][a]);
            pmax[a] = fmaxf(pmax[a], h.pmax[w][a]);
        }
    }
    int64_t used = 0;
    for (int l = 0; l < 4; ++l) {
        float fr[3];
        hash_cell(g, l, pmin, h.lo[l], fr);
        hash_cell(g, l, pmax, h.hi[l], fr);
        int64_t nv = 1;
        for (int a = 0; a < 3; ++a) {
            h.ext[l][a] = h.hi[l][a] - h.lo[l][a] + 2;
            nv *= h.ext[l][a];
        }
        const bool want = CIC_HASH_STAGE == 0 ? nv <= 8 * (int64_t)n : CIC_HASH_STAGE == 1 ? g.hdense[l] != 0 : true;
        if (want && used + nv * vb <= kHTileBytes) {
            h.off[l] = (int)(used / vb);
            used += nv * vb;
        } else {
            h.off[l] = -1;
        }
        lt[l] = LevelTile{h.off[l], {h.lo[l][0], h.lo[l][1], h.lo[l][2]}, h.ext[l][2], h.ext[l][1] * h.ext[l][2]};
    }
}

// The staged levels' vertex boxes from the tables into LDS (vertex (dx, dy,
// dz) of the box at off + (dx * ey + dy) * ez + dz).
// The staged boxes are contiguous in level order, so staged vertex t is
// vertex t - off[l] of the level l whose range holds t; each thread loads
// kHLoads of them with independent loads before storing any.
constexpr int kHLoads = 8;
template <typename T>
__device__ void load_hash_tiles(const GridK &g, const HashSegInfo &h, typename HashVtx<T>::type *tile)
{
    typedef typename HashVtx<T>::type V;
    typedef decltype(V{}[0]) E;
    int end[4], tot = 0;
#pragma unroll
    for (int l = 0; l < 4; ++l) {
        if (h.off[l] >= 0) tot = h.off[l] + h.ext[l][0] * h.ext[l][1] * h.ext[l][2];
        end[l] = tot;
    }
    for (int t0 = threadIdx.x; t0 < tot; t0 += kHLoads * kTileThreads) {
        float x[kHLoads][3];
#pragma unroll
        for (int u = 0; u < kHLoads; ++u) {
            const int t = min(t0 + u * kTileThreads, tot - 1);   // past the end: reload the last vertex
            const int l = t < end[0] ? 0 : t < end[1] ? 1 : t < end[2] ? 2 : 3;
            const int v = t - h.off[l], ey = h.ext[l][1], ez = h.ext[l][2];
            const int dz = v % ez, dy = (v / ez) % ey, dx = v / (ez * ey);
            const T *tab = (const T *)g.htab + (size_t)l * ((size_t)g.hmask + 1) * 3;
            load_entry3(tab, hash_entry(g, l, (uint32_t)(h.lo[l][0] + dx), (uint32_t)(h.lo[l][1] + dy),
                                        (uint32_t)(h.lo[l][2] + dz)),
                        x[u]);
        }
#pragma unroll
        for (int u = 0; u < kHLoads; ++u) {
            const int t = t0 + u * kTileThreads;
            if (t < tot) tile[t] = V{(E)x[u][0], (E)x[u][1], (E)x[u][2], (E)0.0f};
        }
    }
}

// Level q's 3 features of a sample at position xp: from the staged box when
// the level is staged, else gathered from the table.
template <typename T>
__device__ __forceinline__ void hash_level3_tiled(const GridK &g, const LevelTile &lt,
                                                  const typename HashVtx<T>::type *tile, int q, const float xp[3],
                                                  float x[3])
{
    int i0[3];
    float fr[3], v[8][3];
    hash_cell(g, q, xp, i0, fr);
    if (lt.off >= 0) {
        const int base = lt.off + (i0[0] - lt.lo[0]) * lt.sx + (i0[1] - lt.lo[1]) * lt.sy + (i0[2] - lt.lo[2]);
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const auto w = tile[base + ((c >> 2) & 1) * lt.sx + ((c >> 1) & 1) * lt.sy + (c & 1)];
#pragma unroll
            for (int f = 0; f < 3; ++f) v[c][f] = (float)w[f];
        }
    } else {
        hash_corners<T>(g, q, i0, v);
    }
    lerp3_corners(v, fr, x);
}

// ---------------------------------------------------------------------------
// Layers.  Inputs and activations are rounded to BF16 (round to nearest even),
// products accumulate in FP32 on v_mfma_f32_32x32x16_bf16, 32 samples on the N
// axis: lane (h, j) holds rows 8 (r / 4) + 4 h + r % 4 of sample j's 32-row
// result tile and supplies 8 of a chunk's 16 reduction slots, so a result tile
// becomes two input chunks of the next layer once the weights' columns are
// permuted alike.  Layer 0 takes 24 slots per lane half: features 6h .. 6h+5,
// the half's 15 encoding values and 3 pads.  Its bias rides on the encoding's
// three ones: the weights hold the three BF16 parts of the float32 bias, whose
// sum is the bias exactly, so the layer reads no bias from LDS.  The 3-wide
// output layer runs on 4x4x4 MFMA, whose B operand is four activations of the
// lane's own sample.  Every kernel below runs the same sums in the same order
// for a sample, so ray and voxel order give the same bits.
// ---------------------------------------------------------------------------
typedef short s4_t __attribute__((ext_vector_type(4)));

// LDS layout in 16-byte fragments, then floats
constexpr int kBfW0 = 0;                           // [t 4][c 3][lane 64]
constexpr int kBfW1 = kBfW0 + 4 * 3 * 64;          // [t 4][c 8][lane 64]
constexpr int kBfW2 = kBfW1 + 4 * 8 * 64;          // [t 4][i 4][h 2][ch 4] of 4 BF16
constexpr int kBfFrags = kBfW2 + 4 * 4 * 2 * 4 / 2;
constexpr int kBfB1 = 0, kBfB2 = 128, kBfFloats = 132;
constexpr int kLdsBf16 = kBfFrags * 16 + kBfFloats * 4;
static_assert(kLdsBf16 + (kFTileFloats + kSegWords) * 4 <= 160 * 1024 - 1024, "brick tile kernel LDS");
static_assert(kLdsBf16 + kHSegWords * 4 + kHTileBytes <= 160 * 1024 - 2048, "level box kernel LDS");

// (every load goes out before the first conversion: a small launch waits for
// one round trip to memory here)
template <int THREADS>
__device__ void stage_weights_bf16(const cic_mlp &m, bf8_t *frag, float *fl)
{
    constexpr int kN0 = 4 * 3 * 64, kIt0 = (kN0 + THREADS - 1) / THREADS, kN1 = 4 * 8 * 64, kIt1 = kN1 / THREADS;
    static_assert(kN1 % THREADS == 0 && THREADS >= 512, "whole rounds of W1 fragments, one W2 entry per thread");
    const int tid = threadIdx.x;
    float w0[kIt0][8], w1[kIt1][8], b0[kIt0];
#pragma unroll
    for (int k = 0; k < kIt1; ++k) {
        const int i = tid + k * THREADS, l = i & 63, c = (i >> 6) & 7, t = i >> 9;
        const float *src = m.w1 + (32 * t + (l & 31)) * 128;
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e) w1[k][4 * u + e] = src[x_hid(c, l >> 5, 4 * u) + e];
    }
#pragma unroll
    for (int k = 0; k < kIt0; ++k) {
        const int i = min(tid + k * THREADS, kN0 - 1), l = i & 63, c = (i >> 6) % 3, t = i / 192;
        const int row = 32 * t + (l & 31), h = l >> 5;
        b0[k] = m.b0[row];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int s = 8 * c + e;   // slot: features, then encoding values 15h + s - 6
            w0[k][e] = m.w0[row * 39 + (s < 6 ? 6 * h + s : 12 + min(15 * h + s - 6, 26))];
        }
    }
    const int ch2 = (tid >> 2) & 3, h2 = (tid >> 4) & 1;
    const int row2 = 32 * ((tid >> 7) & 3) + 8 * ((tid >> 5) & 3) + 4 * h2 + (tid & 3);
    const float v2 = m.w2[min(ch2, 2) * 128 + row2], vb1 = m.b1[tid & 127], vb2 = m.b2[min(tid & 3, 2)];
#pragma unroll
    for (int k = 0; k < kIt1; ++k) {
        bf8_t v;
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = (__bf16)w1[k][e];
        frag[kBfW1 + tid + k * THREADS] = v;
    }
#pragma unroll
    for (int k = 0; k < kIt0; ++k) {
        const int i = tid + k * THREADS, l = i & 63, c = (i >> 6) % 3, h = l >> 5;
        bf8_t v;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int s = 8 * c + e, part = 15 * h + s - 6 - 27;
            const float w = s >= 6 && part >= 0 ? bf16_part(b0[k], part) : w0[k][e];   // the bias's parts are exact
            v[e] = (__bf16)(s < 21 ? w : 0.f);
        }
        if (i < kN0) frag[kBfW0 + i] = v;
    }
    if (tid < 512) ((__bf16 *)(frag + kBfW2))[tid] = (__bf16)(ch2 < 3 ? v2 : 0.f);
    if (tid < 128) fl[kBfB1 + tid] = vb1;
    if (tid < 4) fl[kBfB2 + tid] = tid < 3 ? vb2 : 0.f;
}

// ReLU of BF16 values as 16-bit integers: a negative BF16 (sign bit set) is
// a negative int16, so max(bits, 0) zeroes exactly the negatives (and -0).
// Rounding to BF16 preserves sign, so this equals rounding after the ReLU.
__device__ __forceinline__ uint32_t relu_bf2(uint32_t v)
{
    typedef short s2_t __attribute__((ext_vector_type(2)));
    s2_t s = __builtin_bit_cast(s2_t, v);
    s[0] = s[0] > 0 ? s[0] : (short)0;
    s[1] = s[1] > 0 ? s[1] : (short)0;
    return __builtin_bit_cast(uint32_t, s);
}

// rows r .. r + 3 of a result tile as four BF16 activations
__device__ __forceinline__ void act4(const f16_t &a, int r, uint32_t &lo, uint32_t &hi)
{
    lo = relu_bf2(pack_bf2(a[r], a[r + 1]));
    hi = relu_bf2(pack_bf2(a[r + 2], a[r + 3]));
}

// The network on NT groups of 32 samples; a wavefront's working set.
template <int NT>
struct BfNet {
    const bf8_t *w0f, *w1f;
    const s4_t *w2f;
    const float *b1;
    f16_t acc[2][NT];    // a result tile and the one before it
    bf8_t hb[NT][8];     // the first hidden layer's activations
    f4_t out[NT][2];     // channels 0..2 in rows 0..2, even and odd row groups

    __device__ __forceinline__ BfNet(const bf8_t *frag, const float *fl, int lane)
        : w0f(frag + kBfW0 + lane), w1f(frag + kBfW1 + lane),
          w2f((const s4_t *)(frag + kBfW2) + (lane >> 5) * 4 + (lane & 3)), b1(fl + kBfB1 + 4 * (lane >> 5))
    {
    }
    // layer 0, tile t (xin: features and encoding in three chunks)
    __device__ __forceinline__ void layer0(int t, const bf8_t (&xin)[NT][3])
    {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const bf8_t a = w0f[(t * 3 + c) * 64];
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                if (c == 0)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[t & 1][nt][r] = 0.f;
                acc[t & 1][nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, xin[nt][c], acc[t & 1][nt], 0, 0, 0);
            }
        }
    }
    // ReLU and rounding of tile t: input chunks 2t, 2t + 1 of layer 1
    __device__ __forceinline__ void activate(int t)
    {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int hh = 0; hh < 2; ++hh) {
                uint32_t w[4];
                act4(acc[t & 1][nt], 8 * hh, w[0], w[1]);
                act4(acc[t & 1][nt], 8 * hh + 4, w[2], w[3]);
                hb[nt][2 * t + hh] = __builtin_bit_cast(bf8_t, u4_t{w[0], w[1], w[2], w[3]});
            }
    }
    // layer 1, tile t, chunk c
    __device__ __forceinline__ void layer1(int t, int c, const bf8_t a)
    {
        if (c == 0) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const f4_t z = *(const f4_t *)(b1 + 32 * t + 8 * i);
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                    for (int r = 0; r < 4; ++r) acc[t & 1][nt][4 * i + r] = z[r];
            }
        }
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
            acc[t & 1][nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, hb[nt][c], acc[t & 1][nt], 0, 0, 0);
    }
    // rows 4i .. 4i + 3 of tile t into the output layer
    __device__ __forceinline__ void output(int t, int i)
    {
        const s4_t w = w2f[(4 * t + i) * 8];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            uint32_t lo, hi;
            act4(acc[t & 1][nt], 4 * i, lo, hi);
            typedef uint32_t u2_t __attribute__((ext_vector_type(2)));
            const f4_t z = f4_t{0.f, 0.f, 0.f, 0.f};
            out[nt][i & 1] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(w, __builtin_bit_cast(s4_t, u2_t{lo, hi}),
                                                                     t == 0 && i < 2 ? z : out[nt][i & 1], 0, 0, 0);
        }
    }
    __device__ __forceinline__ float logit(int nt, int ch, float b2) const
    {
        float p = out[nt][0][ch] + out[nt][1][ch];
        p += __shfl_xor(p, 32, kWave);
        return p + b2;
    }
};

// layer 0's input chunks of a sample: its 6 features and its ray's half row
__device__ __forceinline__ void bf_inputs(const float x[6], const u4_t e0, const u4_t e1, bf8_t xin[3])
{
    xin[0] = __builtin_bit_cast(bf8_t, u4_t{pack_bf2(x[0], x[1]), pack_bf2(x[2], x[3]), pack_bf2(x[4], x[5]), e0[0]});
    xin[1] = __builtin_bit_cast(bf8_t, u4_t{e0[1], e0[2], e0[3], e1[0]});
    xin[2] = __builtin_bit_cast(bf8_t, u4_t{e1[1], e1[2], e1[3], 0u});
}

// Samples gathered from the grid or the tables: ray order, or voxel order
// through the permutation.  Persistent, one workgroup per CU; its wavefronts
// claim batches of 64 samples from an LDS counter.  As in the FP32 kernel, the
// next batch's records, gathers and interpolation sit between this batch's
// layer-1 MFMAs; 64 samples share each weight fragment read from LDS, which 32
// would read at the LDS's full rate.  800x800 frame over a float16 grid with 36
// M live samples: 2.36 -> 1.77 ms (the matrix power limit of the 46,000
// operations per sample that the padded tiles execute is 1.43 ms), multi-level
// encoding 2.45 -> 2.16 ms.  The brick kernel with the same 32-row tiles: 5.04
// -> 4.90 ms per pass of 95 M samples of eight views, 51 ps per sample against 49
// here and 39 at that limit: it is held by its staging between barriers.
template <typename T, bool HASH>
__global__ __launch_bounds__(kRayWaves8 * 64) __attribute__((amdgpu_waves_per_eu(2, 2))) void
k_mlp_fwd_bf16_gather(GridK g, cic_mlp m, RenderBufs b, int voxel)
{
    constexpr int NT = 2, kBatch = 32 * NT;
    extern __shared__ __attribute__((aligned(16))) float lds_raw[];   // 16-byte fragments
    __shared__ uint32_t claimed;
    bf8_t *frag = (bf8_t *)lds_raw;
    float *fl = lds_raw + kBfFrags * 4;
    stage_weights_bf16<kRayWaves8 * 64>(m, frag, fl);
    if (threadIdx.x == 0) claimed = kRayWaves8;
    __syncthreads();

    const int lane = lane_id(), h = lane >> 5, j = lane & 31;
    const uint32_t total = b.offsets[b.n];
    const BatchRange br = xcd_batches(((int64_t)total + kBatch - 1) / kBatch, kRayWaves8, 0);
    const uint32_t bfirst = (uint32_t)br.first, bstride = (uint32_t)br.stride;
    const uint32_t bcount = br.end > br.first ? (uint32_t)(br.end - br.first) : 0u;   // relative to bfirst
    auto batch_of = [&](uint32_t k) -> uint32_t { return (k / kRayWaves8) * bstride + k % kRayWaves8; };
    // (a lane past the last sample works on sample 0: in-bounds inputs, no
    // branches around the loads; its colour is not stored)
    auto record_of = [&](uint32_t bt, int nt) -> uint32_t {
        const uint32_t s = (bfirst + bt) * kBatch + 32 * nt + j;
        const uint32_t sv = bt < bcount && s < total ? s : 0;
        return voxel ? b.perm[sv] : sv;
    };
    uint32_t bt = batch_of(threadIdx.x / kWave);
    if (bt >= bcount) return;

    BfNet<NT> net(frag, fl, lane);
    const f4_t b2 = *(const f4_t *)(fl + kBfB2);
    uint32_t crec[NT], nrec[NT], nray[NT];
    int nk[NT];
    float xp[NT][3];
    Gather<T, HASH> gt;
    float x[6];
    bf8_t xin[NT][3];
    u4_t enc[NT][2];
    auto load_enc = [&](int nt, uint32_t ray) {
        const u4_t *e = (const u4_t *)(b.enc + (int64_t)ray * 16 + 8 * h);
        enc[nt][0] = e[0];
        enc[nt][1] = e[1];
    };
    auto position = [&](int nt, uint32_t ray, int k) {
        SampleRay r;
        load_sample_ray(b, ray, k, r);
        sample_position(r, xp[nt]);
    };
    auto inputs = [&](int nt) {
        bf_inputs(x, enc[nt][0], enc[nt][1], xin[nt]);
        // (keeps the interpolation here, among the MFMAs, and not moved down
        // to its use)
        asm volatile("" : "+v"(xin[nt][0]));
    };
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        crec[nt] = record_of(bt, nt);
        const uint32_t ray = b.rec_ray[crec[nt]];
        position(nt, ray, b.rec_k[crec[nt]]);
        load_enc(nt, ray);
        gt.issue(g, xp[nt], h);
#pragma unroll
        for (int k = 0; k < 6; ++k) x[k] = gt.feature(k);
        inputs(nt);
    }
    for (;;) {
        uint32_t claim = 0;
        if (lane == 0) claim = atomicAdd(&claimed, 1u);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t <= 4; ++t) {
            if (t < 4) net.layer0(t, xin);
            if (t > 0) net.activate(t - 1);
            interleave_mfma<6>();
            __builtin_amdgcn_sched_barrier(0);
        }
        const uint32_t nbt = batch_of(__builtin_amdgcn_readfirstlane(claim));
        bf8_t a = net.w1f[0];
        static_for<32>([&](auto step) {
            constexpr int t = step / 8, c = step % 8;
            const bf8_t an = net.w1f[(step + 1 < 32 ? step + 1 : step) * 64];
            net.layer1(t, c, a);
            a = an;
            // what else happens during these MFMAs
            if constexpr (t > 0 && (c & 1)) net.output(t - 1, c >> 1);
            if constexpr (t == 0 && c == 0) {
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) nrec[nt] = record_of(nbt, nt);
            }
            if constexpr (t == 0 && c == 2) {
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    nray[nt] = b.rec_ray[nrec[nt]];
                    nk[nt] = b.rec_k[nrec[nt]];
                }
            }
            if constexpr (t == 1 && c == 0) {
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    position(nt, nray[nt], nk[nt]);
                    load_enc(nt, nray[nt]);
                }
            }
            if constexpr (t == 1 && c == 6) gt.issue(g, xp[0], h);
            if constexpr (t == 2 && c >= 2 && c < 5) {
                x[2 * (c - 2)] = gt.feature(2 * (c - 2));
                x[2 * (c - 2) + 1] = gt.feature(2 * (c - 2) + 1);
            }
            if constexpr (t == 2 && c == 5) {
                inputs(0);
                gt.issue(g, xp[1], h);
            }
            if constexpr (t == 3 && c >= 3 && c < 6) {
                x[2 * (c - 3)] = gt.feature(2 * (c - 3));
                x[2 * (c - 3) + 1] = gt.feature(2 * (c - 3) + 1);
            }
            if constexpr (t == 3 && c == 6) inputs(1);
            interleave_mfma<NT>();
            __builtin_amdgcn_sched_barrier(0);
        });
#pragma unroll
        for (int i = 0; i < 4; ++i) net.output(3, i);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const float p0 = net.logit(nt, 0, b2[0]), p1 = net.logit(nt, 1, b2[1]), p2 = net.logit(nt, 2, b2[2]);
            if ((bfirst + bt) * kBatch + 32 * nt + j < total && h == 0) {
                float *out = b.rec_c + 3 * (int64_t)crec[nt];
                out[0] = sigmoid_hw(p0);
                out[1] = sigmoid_hw(p1);
                out[2] = sigmoid_hw(p2);
            }
            crec[nt] = nrec[nt];
        }
        if (nbt >= bcount) return;
        bt = nbt;
    }
}

// TILE: 1 = voxel order with the brick's features staged in LDS (dense
// grids); 2 = voxel order with the segment's multi-level encoding boxes
// staged in LDS.
template <typename T, int TILE>
__global__ __launch_bounds__(kBfWaves * 64) void k_mlp_fwd_bf16(GridK g, cic_mlp m, RenderBufs b)
{
    typedef typename HashVtx<T>::type HV;
    extern __shared__ __attribute__((aligned(16))) float lds_raw[];   // 16-byte fragments
    bf8_t *frag = (bf8_t *)lds_raw;
    float *fl = lds_raw + kBfFrags * 4;
    float *tile = lds_raw + kBfFrags * 4 + kBfFloats;    // TILE 1: the brick's features
    // the segment's records
    uint32_t *seg = TILE == 1 ? (uint32_t *)(tile + kFTileFloats) : (uint32_t *)tile;
    HV *htile = (HV *)(seg + kHSegWords);                // TILE 2: the staged level boxes
    __shared__ TileWork seg_slot;
    __shared__ HashSegInfo hinfo;
    __shared__ LevelTile ltab[4];
    stage_weights_bf16<kTileThreads>(m, frag, fl);
    __syncthreads();

    const int lane = lane_id(), h = lane >> 5, j = lane & 31;
    const int wave = threadIdx.x / 64;

    // one batch: positions s0 + j below send in the staged segment
    auto batch = [&](int s0, int send) {
        // wave priority raised at each layer (measured: MLP stage 27.0 -> 26.7 ms)
        __builtin_amdgcn_s_setprio(0);
        const int s = s0 + j;
        const bool valid = s < send;
        // (a lane past the batch's last sample works on the segment's first)
        const int sv = valid ? s : 0;
        const int64_t rec = (int64_t)seg[sv];
        const uint32_t ray = seg[kTileSeg + sv];
        const u4_t *er = (const u4_t *)(b.enc + (int64_t)ray * 16 + 8 * h);
        const u4_t e0 = er[0], e1 = er[1];
        const float p[3] = {__uint_as_float(seg[2 * kTileSeg + sv]), __uint_as_float(seg[3 * kTileSeg + sv]),
                            __uint_as_float(seg[4 * kTileSeg + sv])};
        float x[6];
        if constexpr (TILE == 2) {
            hash_level3_tiled<T>(g, ltab[2 * h], htile, 2 * h, p, x);
            hash_level3_tiled<T>(g, ltab[2 * h + 1], htile, 2 * h + 1, p, x + 3);
        } else {
            const uint32_t cell = seg[5 * kTileSeg + sv];
            const int lx = (int)(cell & 15u), ly = (int)((cell >> 4) & 15u), lz = (int)(cell >> 8);
            tile_gather3(tile, lx, ly, lz, p, 2 * h, x);
            tile_gather3(tile, lx, ly, lz, p, 2 * h + 1, x + 3);
        }
        BfNet<1> net(frag, fl, lane);
        bf8_t xin[1][3];
        bf_inputs(x, e0, e1, xin[0]);
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int t = 0; t <= 4; ++t) {
            if (t < 4) net.layer0(t, xin);
            if (t > 0) net.activate(t - 1);
            __builtin_amdgcn_sched_barrier(0);
        }
        __builtin_amdgcn_s_setprio(2);
#pragma unroll
        for (int t = 0; t <= 4; ++t) {
            if (t < 4) {
#pragma unroll
                for (int c = 0; c < 8; ++c) net.layer1(t, c, net.w1f[(t * 8 + c) * 64]);
            }
            if (t > 0) {
#pragma unroll
                for (int i = 0; i < 4; ++i) net.output(t - 1, i);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        __builtin_amdgcn_s_setprio(3);
        const f4_t b2 = *(const f4_t *)(fl + kBfB2);
        const float p0 = net.logit(0, 0, b2[0]), p1 = net.logit(0, 1, b2[1]), p2 = net.logit(0, 2, b2[2]);
        if (valid && h == 0) {
            float *out = b.rec_c + 3 * rec;
            out[0] = sigmoid_hw(p0);
            out[1] = sigmoid_hw(p1);
            out[2] = sigmoid_hw(p2);
        }
    };

    TileWork w;
    ClaimState cs{0, 0, -1};   // used by thread 0 only
    while (claim_segment<TILE == 1 ? kClaimRun : 1>(b, &seg_slot, cs, w)) {
        const int n = (int)(w.end - w.start);
        if constexpr (TILE == 2) {
            stage_segment_hash(g, b, w.start, n, seg, hinfo);
            __syncthreads();
            if (threadIdx.x == 0) plan_hash_levels<T>(g, n, hinfo, ltab);
            __syncthreads();
            load_hash_tiles<T>(g, hinfo, htile);
        } else {
            const BrickBase base = brick_base(g, w.brick);
            if (!w.reuse) load_feature_tile<T>(g, base, tile);
            stage_segment(g, b, w.start, n, base, seg);
        }
        __syncthreads();
        const int nb = (n + kBfBatch - 1) / kBfBatch;
        for (int bi = wave; bi < nb; bi += kBfWaves) batch(bi * kBfBatch, n);
    }
}

#ifndef CIC_VOXEL_TILE
#define CIC_VOXEL_TILE 1
#endif
template <typename T, int TILE>
static void launch_bf16_tile(const GridK &g, const cic_mlp &m, const RenderBufs &b, hipStream_t s)
{
    const int lds = kLdsBf16 + (TILE == 1 ? (kFTileFloats + kSegWords) * 4 : kHSegWords * 4 + kHTileBytes);
    static bool attr_set = false;
    if (!attr_set) {
        (void)hipFuncSetAttribute((const void *)k_mlp_fwd_bf16<T, TILE>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                  lds);
        attr_set = true;
    }
    launch_brick_segments(b, kTileSeg, true, s);
    launch_fill_u32(b.work_ctr, 0u, kXcds, s);
    // at least one workgroup per XCD range of segments
    const int grid = std::max(num_cus(b), kXcds);
    hipLaunchKernelGGL((k_mlp_fwd_bf16<T, TILE>), dim3(grid), dim3(kBfWaves * 64), lds, s, g, m, b);
}

template <typename T, bool HASH>
static void launch_bf16_gather(const GridK &g, const cic_mlp &m, const RenderBufs &b, bool voxel, hipStream_t s)
{
    static bool attr_set = false;
    if (!attr_set) {
        (void)hipFuncSetAttribute((const void *)k_mlp_fwd_bf16_gather<T, HASH>,
                                  hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBf16);
        attr_set = true;
    }
    hipLaunchKernelGGL((k_mlp_fwd_bf16_gather<T, HASH>), dim3(num_cus(b)), dim3(kRayWaves8 * 64), kLdsBf16, s, g, m, b,
                       voxel ? 1 : 0);
}

template <typename T>
void launch_mlp_forward_bf16(const GridK &g, const cic_mlp &m, const RenderBufs &b, bool voxel, hipStream_t s)
{
    if (CIC_VOXEL_TILE && voxel) {
        if (g.hlevels == 0) launch_bf16_tile<T, 1>(g, m, b, s);
        else launch_bf16_tile<T, 2>(g, m, b, s);
    } else if (g.hlevels) {
        launch_bf16_gather<T, true>(g, m, b, voxel, s);
    } else {
        launch_bf16_gather<T, false>(g, m, b, voxel, s);
    }
}

template void launch_mlp_forward_bf16<float>(const GridK &, const cic_mlp &, const RenderBufs &, bool, hipStream_t);
template void launch_mlp_forward_bf16<__half>(const GridK &, const cic_mlp &, const RenderBufs &, bool, hipStream_t);

}  // namespace cic
