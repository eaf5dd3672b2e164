// Adjoint of the rendering quadrature, the MLP and the trilinear gathers.
//
// With C = sum_k w_k c_k + T_stop bg, w_k = T_k (1 - e^{-sigma_k delta}) and
// T_{k+1} = T_k e^{-sigma_k delta}, the derivative with respect to the
// density of live sample k is
//   dC/dsigma_k = delta (T_{k+1} c_k - R_k),  R_k = sum_{j>k} w_j c_j + T_stop bg,
// (every later weight and the background term scale with T_{k+1}), the
// expected distance gives delta (T_{k+1} t_k - D_k) with D_k = sum_{j>k} w_j t_j,
// and the opacity 1 - T_stop gives delta T_stop.  dC/dc_k = w_k.
//
// Kernels (one backward pass over a chunk of rays, after the march and the
// bucketing):
//  - k_mlp_adjoint: per 16-sample batch (ray order), the forward recomputed
//    on chip (its colours c_k kept for the next kernel), the MLP backward
//    from dL/dc_k = w_k dL/dC (the 12 feature gradients written per sample)
//    and the weight-gradient outer products accumulated per workgroup, the
//    backward's products on split float16; k_mlp_adjoint_f32 repeats in
//    float32 the workgroups whose values the split cannot hold;
//    k_wgrad_apply adds the workgroups' partials in a fixed order
//    (deterministic).
//  - k_bwd_composite: one wavefront per ray walks its live samples from the
//    back, 64 at a time, with a reverse wavefront scan for R_k and D_k; it
//    writes dL/draw per sample.
//  - k_fgrad_seg, k_fgrad_gather: the feature and raw-density gradients of
//    each brick segment summed per tile vertex on chip, then added to the
//    grids per vertex in a fixed order (no atomics).
#include <algorithm>

#include "mlp_common.h"

namespace cic {

// Reverse inclusive scan (sum over lanes >= this lane).
__device__ __forceinline__ float wave_rev_incl_scan(float v)
{
    const int l = lane_id();
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const float u = __shfl_down(v, off, kWave);
        if (l + off < kWave) v += u;
    }
    return v;
}

__global__ __launch_bounds__(256) void k_bwd_composite(GridK g, OptsK op, RenderBufs b, BackwardBufs bb)
{
    const int lane = lane_id();
    const int64_t ray = (int64_t)blockIdx.x * 4 + (threadIdx.x / kWave);
    if (ray >= b.n) return;
    const uint32_t cnt = b.count[ray];
    if (cnt == 0) return;
    const uint32_t off = b.offsets[ray];
    const RayInfo inf = b.info[ray];
    const float gr[3] = {bb.d_rgb[3 * ray], bb.d_rgb[3 * ray + 1], bb.d_rgb[3 * ray + 2]};
    const float gd = bb.d_depth_t ? bb.d_depth_t[ray] : 0.f;
    const float ga = bb.d_acc ? bb.d_acc[ray] : 0.f;
    float o[3], d[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        o[a] = b.rays_o[3 * ray + a];
        d[a] = b.rays_d[3 * ray + a];
    }
    const float *dens = (const float *)g.density;
    float carry[3] = {inf.t_stop * op.bg[0], inf.t_stop * op.bg[1], inf.t_stop * op.bg[2]};
    float carry_d = 0.f;
    const int nch = (int)((cnt + kWave - 1) / kWave);
    for (int chn = nch - 1; chn >= 0; --chn) {
        const uint32_t j = (uint32_t)chn * kWave + lane;
        const bool act = j < cnt;
        float w = 0.f, T = 0.f, c[3] = {0.f, 0.f, 0.f}, tk = 0.f;
        int i0[3] = {0, 0, 0};
        float fr[3] = {0.f, 0.f, 0.f};
        if (act) {
            const int64_t r = (int64_t)off + j;
            w = b.rec_w[r];
            T = b.rec_t[r];
            c[0] = b.rec_c[3 * r];
            c[1] = b.rec_c[3 * r + 1];
            c[2] = b.rec_c[3 * r + 2];
            sample_voxel(o, d, inf.tn, inf.delta, b.rec_k[r], g, i0, fr, tk);
        }
        float R[3], incl[3];
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) {
            incl[ch] = wave_rev_incl_scan(w * c[ch]);
            R[ch] = carry[ch] + (incl[ch] - w * c[ch]);
        }
        const float incl_d = wave_rev_incl_scan(w * tk);
        const float D = carry_d + (incl_d - w * tk);
        if (act) {
            const int64_t r = (int64_t)off + j;
            const float Tn = T - w;   // T_{k+1} = T_k (1 - alpha_k)
            float ds = 0.f;
#pragma unroll
            for (int ch = 0; ch < 3; ++ch) ds = fmaf(gr[ch], fmaf(Tn, c[ch], -R[ch]), ds);
            ds = fmaf(gd, fmaf(Tn, tk, -D), ds);
            ds = fmaf(ga, inf.t_stop, ds);
            ds *= inf.delta;
            const float raw = trilerp1(dens, g, i0, fr, 1, 0);
            const float draw = ds * sigmoidf(raw + g.shift);
            bb.rec_draw[r] = draw;   // added per brick segment with the feature gradients
        }
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) carry[ch] += __shfl(incl[ch], 0, kWave);
        carry_d += __shfl(incl_d, 0, kWave);
    }
}

void launch_backward_composite(const GridK &g, const OptsK &o, const RenderBufs &b, const BackwardBufs &bb,
                               hipStream_t s)
{
    if (b.n == 0) return;
    hipLaunchKernelGGL(k_bwd_composite, dim3((unsigned)((b.n + 3) / 4)), dim3(256), 0, s, g, o, b, bb);
}

static int num_cus_b()
{
    int dev = 0, n = 0;
    (void)hipGetDevice(&dev);
    (void)hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev);
    return n > 0 ? n : 256;
}

// Feature and density gradients in two steps, without atomics on floats.
// The brick-ordered samples are cut into segments of at most kFgSeg samples
// of one brick (a brick crossed by many rays gets several segments, which
// keeps the workgroups' loads even).  k_fgrad_seg: one workgroup per
// segment stages its samples (voxel fractions and the 13 gradient channels:
// 12 features, raw density) in LDS, counting-sorted by cell of the brick
// (one integer LDS atomic per sample), and then each thread sums, for its
// vertices of the brick's 9x9x9-vertex tile, the trilinear shares of the
// samples in the up-to-8 cells around the vertex, and stores the tile row
// into the segment's slot.  k_fgrad_gather: one workgroup per brick over the
// vertices it owns (its 8^3 lower corner block, and the grid's last vertex
// layer for the last brick of an axis); a vertex on a brick's lower face also
// lies in the lower neighbours' tiles, so each vertex adds the slots of every
// segment of the bricks containing it, in ascending brick and segment order,
// to the gradient grids.
constexpr int kTileV = kBrick + 1;
constexpr int kTileCh = 13;
constexpr int kTileFloats = kTileV * kTileV * kTileV * kTileCh;
constexpr int kCells = kBrick * kBrick * kBrick;
static_assert(kTileFloats == kFgTileFloats, "brick tile size");

// Exclusive scan of cnt[0..kCells) in place by 256 threads (tmp: 4 words).
__device__ __forceinline__ void cell_scan(int *cnt, int *tmp)
{
    static_assert(kCells == 512, "two cells per thread");
    const int t = threadIdx.x, lane = t & (kWave - 1);
    const int a = cnt[2 * t], c = cnt[2 * t + 1];
    int incl = a + c;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const int v = __shfl_up(incl, d, kWave);
        if (lane >= d) incl += v;
    }
    if (lane == kWave - 1) tmp[t / kWave] = incl;
    __syncthreads();
    int excl = incl - (a + c);
    for (int w = 0; w < t / kWave; ++w) excl += tmp[w];
    cnt[2 * t] = excl;
    cnt[2 * t + 1] = excl + a;
}

// Latency and the vector ALUs decide (68% busy): the segment's brick is found
// 256 candidates at a time, a sample's place in the sorted order is its cell's
// start plus the rank that counting it returned (so its row is written once, in
// place), and a vertex goes through its up-to-8 cells in one loop over four
// runs (cells adjacent in z are adjacent in the order).  2.07 M samples in 8000
// bricks: 172 us; 233 with a binary search, a second pass of atomics for the
// order, sample data read through it, and a loop per cell.
__global__ __launch_bounds__(256) void k_fgrad_seg(GridK g, RenderBufs b, BackwardBufs bb)
{
    constexpr int kPer = kFgSeg / 256;   // samples per thread
    // row of a sample: fractions and raw density, features 0-3, 4-7, 8-11 (64-byte
    // rows: 172 us, one array per channel 184, the quads rotated by row to spread
    // them over the banks 178)
    __shared__ f4_t rows[kFgSeg][4];
    __shared__ int cnt[kCells + 1], tmp[4];
    const uint32_t k = blockIdx.x;
    if (k >= b.seg_off[b.n_bricks]) return;   // uniform per block
    // brick: the last index with seg_off[brick] <= k (seg_off[0] is 0)
    int64_t brick = 0, width = b.n_bricks;
    while (width > 1) {
        const int64_t step = (width + 255) / 256, at = brick + threadIdx.x * step;
        const int below = __syncthreads_count(threadIdx.x * step < width && b.seg_off[at] <= k);
        const int64_t end = brick + width;
        brick += (below - 1) * step;
        width = min(step, end - brick);
    }
    const uint32_t start = (brick == 0 ? 0u : b.brick_off[brick - 1]) + (k - b.seg_off[brick]) * (uint32_t)kFgSeg;
    const int n = (int)(min(b.brick_off[brick], start + (uint32_t)kFgSeg) - start);
    for (int c = threadIdx.x; c <= kCells; c += blockDim.x) cnt[c] = 0;
    __syncthreads();
    const int bz = (int)(brick % g.nb2), by = (int)((brick / g.nb2) % g.nb1), bx = (int)(brick / ((int64_t)g.nb2 * g.nb1));
    const int base[3] = {kBrick * bx, kBrick * by, kBrick * bz};
    float fr[kPer][3], val[kPer][kTileCh];
    int cell[kPer], rank[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int e = threadIdx.x + 256 * u;
        if (e >= n) continue;
        const uint32_t rec = b.perm[start + (uint32_t)e];
        const uint32_t ray = b.rec_ray[rec];
        const float *df = bb.rec_df + (int64_t)rec * 12;
#pragma unroll
        for (int f = 0; f < 12; ++f) val[u][f] = df[f];
        val[u][12] = bb.rec_draw[rec];
        const RayInfo inf = b.info[ray];
        float o[3], d[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            o[a] = b.rays_o[3 * (int64_t)ray + a];
            d[a] = b.rays_d[3 * (int64_t)ray + a];
        }
        int i0[3];
        float tk;
        sample_voxel(o, d, inf.tn, inf.delta, b.rec_k[rec], g, i0, fr[u], tk);
        cell[u] = ((i0[0] - base[0]) * kBrick + (i0[1] - base[1])) * kBrick + (i0[2] - base[2]);
        rank[u] = atomicAdd(&cnt[cell[u]], 1);
    }
    __syncthreads();
    cell_scan(cnt, tmp);
    if (threadIdx.x == 0) cnt[kCells] = n;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        if ((int)threadIdx.x + 256 * u >= n) continue;
        const int p = cnt[cell[u]] + rank[u];
        rows[p][0] = f4_t{fr[u][0], fr[u][1], fr[u][2], val[u][12]};
#pragma unroll
        for (int c = 0; c < 3; ++c)
            rows[p][c + 1] = f4_t{val[u][4 * c], val[u][4 * c + 1], val[u][4 * c + 2], val[u][4 * c + 3]};
    }
    __syncthreads();
    // each tile vertex sums the shares of the samples in its up-to-8 cells
    float *slot = bb.seg_tiles + (int64_t)k * kTileFloats;
    for (int vtx = threadIdx.x; vtx < kTileV * kTileV * kTileV; vtx += blockDim.x) {
        const int vz = vtx % kTileV, vy = (vtx / kTileV) % kTileV, vx = vtx / (kTileV * kTileV);
        float acc[kTileCh];
#pragma unroll
        for (int f = 0; f < kTileCh; ++f) acc[f] = 0.f;
        // run r = 2 (cx - vx + 1) + (cy - vy + 1): the cells (cx, cy, vz - 1) and (cx, cy, vz); their
        // samples begin at p[r], the second cell's at mid[r], and end after len[r]
        const int z0 = max(vz - 1, 0), z1 = min(vz, kBrick - 1);
        int p[4], mid[4], upto[4], total = 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int cx = vx - 1 + (r >> 1), cy = vy - 1 + (r & 1);
            const bool in = cx >= 0 && cx < kBrick && cy >= 0 && cy < kBrick;
            const int c = in ? (cx * kBrick + cy) * kBrick : 0;
            p[r] = cnt[c + z0];
            mid[r] = vz == kBrick ? cnt[c + kBrick] : cnt[c + vz];
            upto[r] = total;   // samples before this run
            total += in ? cnt[c + z1 + 1] - p[r] : 0;
        }
        for (int i = 0; i < total; ++i) {
            const int r = i < upto[1] ? 0 : i < upto[2] ? 1 : i < upto[3] ? 2 : 3;
            const int e = i + (r == 0 ? p[0] : r == 1 ? p[1] - upto[1] : r == 2 ? p[2] - upto[2] : p[3] - upto[3]);
            const int m = r == 0 ? mid[0] : r == 1 ? mid[1] : r == 2 ? mid[2] : mid[3];
            // the vertex is the cell's lower corner along an axis (weight 1 - fr) or its upper one (fr)
            const f4_t s = rows[e][0];
            const float wx = r & 2 ? 1.f - s[0] : s[0];
            const float wy = r & 1 ? 1.f - s[1] : s[1];
            const float wz = e >= m ? 1.f - s[2] : s[2];
            const float w = wx * wy * wz;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const f4_t v = rows[e][c + 1];
#pragma unroll
                for (int f = 0; f < 4; ++f) acc[4 * c + f] = fmaf(w, v[f], acc[4 * c + f]);
            }
            acc[12] = fmaf(w, s[3], acc[12]);
        }
#pragma unroll
        for (int f = 0; f < kTileCh; ++f) slot[vtx * kTileCh + f] = acc[f];
    }
}

// Bricks along one axis whose tiles contain vertex coordinate x (nb bricks).
__device__ __forceinline__ void tile_bricks(int x, int nb, int &lo, int &hi)
{
    hi = min(x / kBrick, nb - 1);
    lo = (x % kBrick == 0 && x > 0) ? x / kBrick - 1 : x / kBrick;
    lo = min(lo, hi);
}

__global__ __launch_bounds__(256) void k_fgrad_gather(GridK g, int nb0, RenderBufs b, BackwardBufs bb)
{
    const int64_t brick = blockIdx.x;
    const int nb1 = g.nb1, nb2 = g.nb2;
    const int bz = (int)(brick % nb2), by = (int)((brick / nb2) % nb1), bx = (int)(brick / ((int64_t)nb2 * nb1));
    // nothing to add unless this brick or a lower neighbour has samples (uniform per block)
    bool any = false;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        const int x = bx - ((c >> 2) & 1), y = by - ((c >> 1) & 1), z = bz - (c & 1);
        if (x >= 0 && y >= 0 && z >= 0) {
            const int64_t nbk = ((int64_t)x * nb1 + y) * nb2 + z;
            any = any || b.seg_off[nbk + 1] > b.seg_off[nbk];
        }
    }
    if (!any) return;
    const int rr[3] = {g.r0, g.r1, g.r2}, nbs[3] = {nb0, nb1, nb2}, bc[3] = {bx, by, bz};
    int lo[3], cnt[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        lo[a] = kBrick * bc[a];
        const int hi = bc[a] == nbs[a] - 1 ? rr[a] - 1 : lo[a] + kBrick - 1;
        cnt[a] = hi - lo[a] + 1;
    }
    const int n = cnt[0] * cnt[1] * cnt[2];
    for (int e = threadIdx.x; e < n; e += blockDim.x) {
        const int z = lo[2] + e % cnt[2], y = lo[1] + (e / cnt[2]) % cnt[1], x = lo[0] + e / (cnt[2] * cnt[1]);
        int xl, xh, yl, yh, zl, zh;
        tile_bricks(x, nb0, xl, xh);
        tile_bricks(y, nb1, yl, yh);
        tile_bricks(z, nb2, zl, zh);
        float acc[kTileCh];
#pragma unroll
        for (int f = 0; f < kTileCh; ++f) acc[f] = 0.f;
        bool hit = false;
        for (int cx = xl; cx <= xh; ++cx)
            for (int cy = yl; cy <= yh; ++cy)
                for (int cz = zl; cz <= zh; ++cz) {
                    const int64_t cb = ((int64_t)cx * nb1 + cy) * nb2 + cz;
                    const uint32_t k0 = b.seg_off[cb], k1 = b.seg_off[cb + 1];
                    const int loc = ((x - kBrick * cx) * kTileV + (y - kBrick * cy)) * kTileV + (z - kBrick * cz);
                    for (uint32_t k = k0; k < k1; ++k) {
                        hit = true;
                        const float *t = bb.seg_tiles + (int64_t)k * kTileFloats + loc * kTileCh;
#pragma unroll
                        for (int f = 0; f < kTileCh; ++f) acc[f] += t[f];
                    }
                }
        if (!hit) continue;
        const int64_t vi = vertex_index(g, x, y, z);
#pragma unroll
        for (int f = 0; f < 12; ++f) bb.d_features[vi * 12 + f] += acc[f];
        bb.d_density[vi] += acc[12];
    }
}

void launch_feature_grads_bricks(const GridK &g, const RenderBufs &b, const BackwardBufs &bb, hipStream_t s)
{
    if (b.n_bricks == 0) return;
    launch_brick_segments(b, kFgSeg, false, s);
    const int64_t max_seg = fg_max_segments(b.n_bricks, b.n * (int64_t)b.n_samples);
    hipLaunchKernelGGL(k_fgrad_seg, dim3((unsigned)max_seg), dim3(256), 0, s, g, b, bb);
    const int nb0 = (int)(b.n_bricks / ((int64_t)g.nb1 * g.nb2));
    hipLaunchKernelGGL(k_fgrad_gather, dim3((unsigned)b.n_bricks), dim3(256), 0, s, g, nb0, b, bb);
}

// ---------------------------------------------------------------------------
// MLP adjoint, fused: per batch of 16 live samples (ray order) a wavefront
// recomputes the forward (full 40-wide layer-0 input, FP32 MFMA: the ReLU
// masks have to be those of float32 arithmetic), forms the output-logit
// gradient from dL/dc_k = w_k g, and runs the backward: dp1 = [h2 > 0]
// (W2^T dlogit) on the vector ALUs, dh1 = W1^T dp1, dp0 = [h1 > 0] dh1 and the
// feature gradient (W0^T dp0)[0:12].  Nothing of it leaves the chip except the
// 12 feature gradients per sample (for the brick-segment tiles).  Ray order
// fixes which samples each workgroup sums, so the MLP gradients are the same
// bits on every call (in brick order the bucketing's atomic cursors would
// decide it).  The weight gradients are sums over samples of outer products,
//   P0 = dp0^T [x|1] (dW0, db0), P1 = dp1^T h1 (dW1),
//   P2 = dl^T h2 (dW2), and the sums of dp1 (db1) and dl (db2).
//
// Arithmetic.  Everything after the forward multiplies values split into two
// float16 parts, v = hi + lo, as hi hi + hi lo + lo hi on float16 MFMA (16 times
// the float32 rate), summed in float32.  Every factor is scaled by a power of
// two first, to a largest value in [2^14, 2^15) (dp1 below 3 2^14, mostly near
// 2^11); a remainder is then exact to 2^-25, 2^-39 of the largest value that
// shares its scale, and a normal float16 number down to 2^-17 of it:
//  - in the products that stay with a sample (dp1 -> dh1 -> dp0 -> the feature
//    gradients) dp1 and dp0 have scales of that sample, by its dlogit and its
//    largest dp0, so its feature gradients do not depend on any other sample;
//  - W1 has one scale, W0 one per feature;
//  - in the products over samples (the weight gradients) the workgroup's 128
//    samples of a step have one for dp1 and one for dp0, and the activations and
//    the direction one each and the features one per channel, by the largest so
//    far.  What a sample's dlogit (its dp0) is below the step's largest, 2^-d, is
//    carried half by each of its two factors, so that entries to which only such
//    samples add keep float32's bits down to d = 30.  From step to step the sums
//    are brought to the new scale, which is exact.
// k_mlp_adjoint_f32 does a workgroup's share again where the scales do not hold
// a value (dlogit or dp0 from about 2^100, inputs and activations from 2^51,
// infinities, NaN), where its rays' upstream gradients are more than 2^36
// apart, or W1's rows and columns more than 2^17, multiplied, in their largest
// entries (at 2^20 feature gradients are off by 3e-7 in place of 2e-7).
// Gradient error against 64 bits, rms over seeds, float32 products -> these:
// 3000 rays of 96 samples dW0 8.3e-7 -> 5.1e-7, dW1 7.3e-7 -> 4.3e-7, dW2 9.5e-7
// -> 1.8e-7, features 6.1e-7 both (the float32 sums over all samples were rounded
// 4 to 12 times as often); 100 rays of 8: dW0 2.1e-7 -> 1.8e-7, dW1 1.9e-7 both.
// With one scale for all that a workgroup met (1.90 ms), feature gradients of
// rays 2^-24 below others were off by 1% and rows of dW0 by 7%.
//
// Layout.  The products over samples want the samples along a lane's words,
// the forward leaves them along the lanes: a product with the identity (exact)
// transposes each 16x16 tile.  P2 and db1 then stay within the wavefront.  P0
// and P1 are cut into 32x32 tiles, three per wavefront, in registers for the
// workgroup's lifetime; the wavefronts take turns writing their batch's
// transposed columns into one of two LDS blocks, while all of them add the
// other one's 16 samples to their tiles.  LDS: the forward's weight fragments
// (92.6 KB, W1 padded for its transposed reads, which are split after the
// read), W0^T fragments (8 KB), the blocks (56 KB).
//
// Bound.  2.07 M samples, 8192 rays: 2.67 ms with float32 products and one row
// block of float32 rows, 2.10 so.  Of the 1.90 ms with one scale per workgroup
// the matrix cores were busy 48% (two thirds of that with the recomputed forward,
// whose float32 MFMA no vector instruction runs beside), the vector ALUs 28%, and
// a third of the wavefronts' time were waits (halves of the workgroup half a step
// apart, so that one's forward runs beside the other's backward, took the same
// time).
// ---------------------------------------------------------------------------
constexpr int kAdjWaves = 8;
// LDS in floats: the forward's weights, W0^T fragments for the feature
// gradients, then two blocks, each 27 16-column tiles of 16 samples (dp1 8, h1
// 8, dp0 8, x 3) and an unused one, W0's scales and the step's maxima.
typedef F32Lds AdjLds;
constexpr int kTH1 = 8, kTDP0 = 16, kTX = 24, kTiles = 27;
constexpr int kAOffW0T = AdjLds::kSize;                 // [part 2][s 4][lane 64][4 words]
constexpr int kAOffBlocks = kAOffW0T + 8 * 64 * 4;
constexpr int kBlock = (kTiles + 1) * 256;   // [32 columns][part 2][8 samples h][column 32][4 words]
constexpr int kAOffS0 = kAOffBlocks + 2 * kBlock;   // [16] W0's scales taken out again, per feature
constexpr int kAOffTops = kAOffS0 + 16;             // [wave 8][16] the step's largest values
constexpr int kALds = kAOffTops + 128;
static_assert(kAOffBlocks % 4 == 0 && kBlock % 4 == 0 && kAOffS0 % 4 == 0, "16-byte alignment");
static_assert(kALds * 4 <= 160 * 1024, "LDS");

typedef uint32_t u2_t __attribute__((ext_vector_type(2)));
typedef _Float16 h4_t __attribute__((ext_vector_type(4)));

// A 16x16 tile from sample-major registers (lane l holds columns 4 (l / 16) ..
// + 3 of sample l % 16) to column-major ones (column l % 16 of samples 4 (l /
// 16) .. + 3): a product with the identity, which is exact.
__device__ __forceinline__ h4_t as_h4(uint32_t a, uint32_t b) { return __builtin_bit_cast(h4_t, u2_t{a, b}); }

__device__ __forceinline__ u2_t transpose16(u2_t v, h4_t identity)
{
    const f4_t t = __builtin_amdgcn_mfma_f32_16x16x16f16(__builtin_bit_cast(h4_t, v), identity,
                                                         f4_t{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
    h4_t r;
#pragma unroll
    for (int e = 0; e < 4; ++e) r[e] = (_Float16)t[e];
    return __builtin_bit_cast(u2_t, r);
}

// v0 and v1 times `scale` into a float16 and a float16 remainder each
__device__ __forceinline__ void split_pair(float v0, float v1, float scale, uint32_t &hi, uint32_t &lo)
{
    h2_t a, b;
    v0 *= scale;
    v1 *= scale;
    a[0] = (_Float16)v0;
    a[1] = (_Float16)v1;
    hi = __builtin_bit_cast(uint32_t, a);
    asm("" : "+v"(hi));   // one packed conversion, not two more single ones for the remainders
    a = __builtin_bit_cast(h2_t, hi);
    // v - hi (exact), rounded to float16: one mixed-precision multiply-add each,
    // which the compiler does not use where it knows the factor to be -1 (the
    // kernel 1.95 -> 1.91 ms)
    float minus = -1.f;
    asm("" : "+s"(minus));
    b[0] = (_Float16)fmaf((float)a[0], minus, v0);
    b[1] = (_Float16)fmaf((float)a[1], minus, v1);
    lo = __builtin_bit_cast(uint32_t, b);
}

// the same of four values, transposed: the first parts in words 0 and 1, the
// remainders in words 2 and 3
__device__ __forceinline__ u4_t split_transpose(f4_t v, float scale, h4_t identity)
{
    u2_t hi, lo;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        uint32_t x, y;
        split_pair(v[2 * e], v[2 * e + 1], scale, x, y);
        hi[e] = x;
        lo[e] = y;
    }
    hi = transpose16(hi, identity);
    lo = transpose16(lo, identity);
    return u4_t{hi[0], hi[1], lo[0], lo[1]};
}

// the largest of a value over the four lanes j, j + 16, j + 32, j + 48, in each of them
__device__ __forceinline__ uint32_t across_rows_max(uint32_t v)
{
    const auto a = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    v = max((uint32_t)a[0], (uint32_t)a[1]);
    const auto b = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return max((uint32_t)b[0], (uint32_t)b[1]);
}

// both float16 of a word times f
__device__ __forceinline__ uint32_t scale_h2(uint32_t v, float f)
{
    const h2_t a = __builtin_bit_cast(h2_t, v), b = {(_Float16)f, (_Float16)f};
    return __builtin_bit_cast(uint32_t, a * b);
}

// the largest of a value over the 16 lanes of a row, in each of them
__device__ __forceinline__ uint32_t row_max(uint32_t v)
{
    v = max_dpp<0x121>(v);   // row_ror:1, 2, 4, 8
    v = max_dpp<0x122>(v);
    v = max_dpp<0x124>(v);
    return max_dpp<0x128>(v);
}

// 2^k, k in [-126, 126]
__device__ __forceinline__ float pow2(int k) { return __int_as_float((127 + min(max(k, -126), 126)) << 23); }
// k with 2^k top in [2^to, 2^(to + 1)) (for zero more than any limit)
__device__ __forceinline__ int exp_to(uint32_t top, int to) { return to + 127 - (int)(top >> 23); }
__device__ __forceinline__ int clamp_exp(int k, int lim) { return min(max(k, -lim), lim); }

// half (rounded up, at most 30) of the powers of two between a value and the largest (0 for zero)
__device__ __forceinline__ int half_below(uint32_t v, uint32_t top)
{
    return v ? min(((int)(top >> 23) - (int)(v >> 23) + 1) >> 1, 30) : 0;
}

constexpr int kXExp = 14;     // of the encoding's sines and cosines and the constant 1
// limits of the exponents of a gradient and of what it is multiplied with (their sums are powers of two)
constexpr int kGradExp = 90, kActExp = 36;
constexpr int kStepExp = 60;            // a step's gradient exponent above the smallest so far
constexpr int kRaySpread = 36;          // largest ratio of its rays' upstream gradients, 2^this
constexpr float kAdjSpread = 0x1p17f;   // largest product of the ratios of W1's rows' and of its columns' largest entries

__device__ __forceinline__ uint32_t abs_bits(float v) { return __float_as_uint(v) & 0x7fffffffu; }

// P0's column slot 16 u + 4 g + e is chunk 4 u + e of lane group g; the slots of
// a wavefront's 32x32 tile
__device__ __forceinline__ int slot_chunk(int wave, int lane)
{
    return 8 * (wave & 1) + 4 * ((lane >> 4) & 1) + (lane & 3);
}
__device__ __forceinline__ int slot_group(int lane) { return (lane >> 2) & 3; }

// The layer-0 inputs of a lane group q that depend on the ray alone, once per
// ray, in the rows that the forward pass uses for z0 (8192 rays: 5 us; per
// sample they are three sincosf a lane: the adjoint 1.91 -> 1.87 ms): row of a
// ray: [q 4][8], 7 used.
__global__ __launch_bounds__(256) void k_ray_encode(RenderBufs b)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, ray = t >> 2;
    if (ray >= b.n) return;
    const float d[3] = {b.rays_d[3 * ray], b.rays_d[3 * ray + 1], b.rays_d[3 * ray + 2]};
    float x[7];
    encode_group(d, (int)(t & 3), x);
    f4_t *row = (f4_t *)b.z0 + 2 * t;
    row[0] = f4_t{x[0], x[1], x[2], x[3]};
    row[1] = f4_t{x[4], x[5], x[6], 0.f};
}

// Two wavefronts per SIMD: a wavefront holds its batch's columns (108 VGPRs)
// and its sums (57) between its turns at the blocks.  (Sums of a step in
// registers of their own, to be added at its end, spill: 2.96 ms a training step
// of 8192 rays against 2.87.)
__global__ __launch_bounds__(kAdjWaves * 64) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_mlp_adjoint(
    GridK g, cic_mlp m, RenderBufs b, BackwardBufs bb)
{
    extern __shared__ __attribute__((aligned(16))) float lds[];
    // Powers of two (exact; taken out again where gradients leave the kernel):
    // s1 of W1, and W0's feature columns', s0
    float *blocks = lds + kAOffBlocks;
    float s1, s0;   // (s0 of the feature that this thread stages)
    int e_s1, e_w2;    // of s1, and of W2 / s1
    bool bad;          // a value left the range of the split
    {
        const int tid = threadIdx.x, lane = lane_id(), wave = tid / kWave;
        // max|W2|, |W1| (whole, row tid / 4, column tid % 128), W0's features wave / 2 + 4 k; the weights' sum
        uint32_t w2 = 0, w1, row = 0, col = 0, f0[3], lo, rows_lo;
        float sum = 0.f;
        if (tid < 384) sum = fabsf(m.w2[tid]);
        w2 = wave_max_last(__float_as_uint(sum));
#pragma unroll
        for (int i = 0; i < 128 * 128; i += kAdjWaves * 64) {
            const float w = fabsf(m.w1[i + tid]);
            col = max(col, __float_as_uint(w));
            sum += w;
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
#pragma unroll
            for (int e = 0; e < 4; ++e) row = max(row, abs_bits(m.w1[4 * (8 * tid + i) + e]));
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const float w = fabsf(m.w0[(tid & 127) * 39 + (tid >> 7) + 4 * k]);
            f0[k] = wave_max_last(__float_as_uint(w));
            sum += w;
        }
        row = max(row, (uint32_t)__shfl_xor((int)row, 1, kWave));
        row = max(row, (uint32_t)__shfl_xor((int)row, 2, kWave));
        uint32_t *cols = (uint32_t *)blocks + 256;
        cols[tid] = col;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 4; ++k) col = max(col, cols[(tid & 127) + 128 * k]);
        w1 = wave_max_last(row);
        lo = ~wave_max_last(~(col ? col : 0x7f800000u));
        rows_lo = ~wave_max_last(~(row ? row : 0x7f800000u));
#pragma unroll
        for (int off = kWave / 2; off > 0; off >>= 1) sum += __shfl_xor(sum, off, kWave);
        uint32_t *red = (uint32_t *)blocks;   // [wave][8]
        if (lane == kWave - 1) {
            red[8 * wave] = w1;
            red[8 * wave + 1] = lo;
            red[8 * wave + 2] = w2;
            red[8 * wave + 3] = __float_as_uint(sum);
#pragma unroll
            for (int k = 0; k < 3; ++k) red[8 * wave + 4 + k] = f0[k];
            red[8 * wave + 7] = rows_lo;
        }
        __syncthreads();
        sum = 0.f;
        for (int w = 0; w < kAdjWaves; ++w) {
            w1 = max(w1, red[8 * w]);
            lo = min(lo, red[8 * w + 1]);
            rows_lo = min(rows_lo, red[8 * w + 7]);
            w2 = max(w2, red[8 * w + 2]);
            sum += __uint_as_float(red[8 * w + 3]);
        }
        w1 = __builtin_amdgcn_readlane(w1, kWave - 1);
        w2 = __builtin_amdgcn_readlane(w2, kWave - 1);
        lo = __builtin_amdgcn_readlane(lo, kWave - 1);
        rows_lo = __builtin_amdgcn_readlane(rows_lo, kWave - 1);
        e_s1 = clamp_exp(exp_to(w1, 14), 60);
        s1 = pow2(e_s1);
        e_w2 = exp_to(w2, 6) + e_s1;
        // (the sum is not finite where a weight is not)
        bad = __builtin_amdgcn_readfirstlane(!(sum < 0x1p50f) || e_w2 < -94 ||
                                             (w1 && !(__uint_as_float(w1) / __uint_as_float(lo) *
                                                          (__uint_as_float(w1) / __uint_as_float(rows_lo)) <=
                                                      kAdjSpread)));
#pragma unroll
        for (int k = 0; k < 3; ++k) f0[k] = max(red[16 * (wave >> 1) + 4 + k], red[16 * (wave >> 1) + 12 + k]);
        __syncthreads();
        // W0's scale per feature: f % 4 is its wavefront pair, f / 4 its k
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const int e0 = clamp_exp(exp_to(f0[k], 14), 60);
            if ((tid & 127) == 0) lds[kAOffS0 + (tid >> 7) + 4 * k] = pow2(-e0);
        }
        if (tid < 4) lds[kAOffS0 + 12 + tid] = 1.f;
        __syncthreads();
        s0 = 1.f / lds[kAOffS0 + min(tid & 15, 11)];
    }
    stage_weights_f32(m, lds, s1);
    // W0^T's fragments: lane l, word e: feature l % 16 (rows 12 .. of the
    // product are not used), unit 32 s + 16 (e / 4) + 4 (l / 16) + e % 4
    if (threadIdx.x < 256) {
        const int l = threadIdx.x & 63, s = threadIdx.x >> 6;
        u4_t hi, lo;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            float w[2];
#pragma unroll
            for (int u = 0; u < 2; ++u)
                w[u] = m.w0[(32 * s + 16 * (e >> 1) + 4 * (l >> 4) + 2 * (e & 1) + u) * 39 + min(l & 15, 11)];
            uint32_t x, y;
            split_pair(w[0], w[1], s0, x, y);
            hi[e] = x;
            lo[e] = y;
        }
        ((u4_t *)(lds + kAOffW0T))[threadIdx.x] = hi;
        ((u4_t *)(lds + kAOffW0T))[256 + threadIdx.x] = lo;
    }
    __syncthreads();   // (the row blocks' memory is free from here on)
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);

    // this workgroup's batches: the XCD's contiguous range, interleaved over
    // its workgroups and wavefronts; every wavefront runs the same number of
    // steps (the row-block turns are workgroup-wide)
    const int64_t total = (int64_t)b.offsets[b.n];
    const int64_t nbatch = (total + 15) / 16;
    const int xcd = blockIdx.x % kXcds, slot = blockIdx.x / kXcds, nslots = gridDim.x / kXcds;
    const int64_t per = (nbatch + kXcds - 1) / kXcds;
    const int64_t lo = xcd * per, hi = lo + per < nbatch ? lo + per : nbatch;
    const int64_t first = lo + (int64_t)slot * kAdjWaves, stride = (int64_t)nslots * kAdjWaves;
    const int64_t steps = !bad && hi > first ? (hi - first + stride - 1) / stride : 0;   // (bad: the weights)

    // this wavefront's share of the sums (see the turns)
    f16_t acc0, acc1[2];
    f4_t acc2[2];        // rows 0..2: P2, row 3: db1, of unit 64 u + lane
    float acc4 = 0.f;    // db2, channel q
    uint32_t g_hi = 0, g_lo = 0x7f800000u;   // largest and smallest (but zero) upstream gradient of this lane's rays
#pragma unroll
    for (int r = 0; r < 16; ++r) acc0[r] = acc1[0][r] = acc1[1][r] = 0.f;
    acc2[0] = acc2[1] = f4_t{0.f, 0.f, 0.f, 0.f};

    // exponents of the sums' scales (see the steps), eb and e0 with their smallest so far
    int eb = kGradExp, e0 = kGradExp, eb_low = kGradExp, e0_low = kGradExp, e1 = kActExp, ed = kActExp;
    int ef[3] = {kActExp, kActExp, kActExp};
    int ec = kActExp;   // that of the inputs in this lane's column of P0

    for (int64_t st = 0; st < steps; ++st) {
        // (the lane's LDS addresses are formed anew in each step: kept over the
        // loop they would take the registers of the batch)
        int lane = lane_id();
        asm volatile("" : "+v"(lane));
        const int q = lane >> 4, j = lane & 15;
        const f2_t *w0f = (const f2_t *)(lds + AdjLds::kW0);
        const f4_t *w2l = (const f4_t *)(lds + AdjLds::kW2);
        const h8_t *w0t = (const h8_t *)(lds + kAOffW0T) + lane;
        // this lane's W1 fragment in block 0 (block k at + k * kW1Block floats)
        const float *w1f = lds + AdjLds::w1(0, lane);
        const int64_t bt = first + st * stride + wave;
        const int64_t s = bt * 16 + j;
        const bool valid = bt < hi && s < total;
        // ray order; a lane past the end works on sample 0 (in-bounds inputs,
        // no branches around the loads) with a zero logit gradient, so it
        // adds nothing to the weight gradients and stores nothing
        const uint32_t rec = valid ? (uint32_t)s : 0u;
        float x[10];
        const uint32_t ray = b.rec_ray[rec];
        {
            const f4_t *row = (const f4_t *)b.z0 + 2 * (4 * (int64_t)ray + q);
            const f4_t e0 = row[0], e1 = row[1];
            SampleRay r;
            load_sample_ray(b, ray, b.rec_k[rec], r);
            int i0[3];
            float fr[3], tk;
            sample_voxel(r.o, r.d, r.tn, r.delta, r.k, g, i0, fr, tk);
#pragma unroll
            for (int c = 0; c < 3; ++c) x[c] = trilerp1((const float *)g.features, g, i0, fr, 12, 3 * q + c);
            x[3] = e0[0];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                x[4 + c] = e0[1 + c];
                x[7 + c] = e1[c];
            }
        }
        // forward: layer 0 (40 -> 128)
        f4_t h1[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) h1[t] = *(const f4_t *)(lds + AdjLds::kB0 + 16 * t + 4 * q);
#pragma unroll
        for (int c2 = 0; c2 < 5; ++c2) {
            f2_t a[8];
#pragma unroll
            for (int t = 0; t < 8; ++t) a[t] = w0f[(t * 5 + c2) * 64 + lane];
#pragma unroll
            for (int e = 0; e < 2; ++e)
#pragma unroll
                for (int t = 0; t < 8; ++t)
                    h1[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[t][e], x[2 * c2 + e], h1[t], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int t = 0; t < 8; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) h1[t][r] = relu_bits(h1[t][r]);
        // layer 1 (128 -> 128)
        f4_t h2[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) h2[t] = *(const f4_t *)(lds + AdjLds::kB1 + 16 * t + 4 * q);
        {
            f4_t a[4], an[4];
#pragma unroll
            for (int tt = 0; tt < 4; ++tt) a[tt] = *(const f4_t *)(w1f + (tt * 8 + 0) * AdjLds::kW1Block);
#pragma unroll
            for (int c4 = 0; c4 < 8; ++c4) {
#pragma unroll
                for (int tg = 0; tg < 2; ++tg) {
                    const int step = c4 * 2 + tg, nx = step + 1 < 16 ? step + 1 : step;
                    const int nc4 = nx >> 1, ntg = nx & 1;
#pragma unroll
                    for (int tt = 0; tt < 4; ++tt)
                        an[tt] = *(const f4_t *)(w1f + ((4 * ntg + tt) * 8 + nc4) * AdjLds::kW1Block);
#pragma unroll
                    for (int rr = 0; rr < 4; ++rr)
#pragma unroll
                        for (int tt = 0; tt < 4; ++tt)
                            h2[4 * tg + tt] =
                                __builtin_amdgcn_mfma_f32_16x16x4f32(a[tt][rr], h1[c4][rr], h2[4 * tg + tt], 0, 0, 0);
#pragma unroll
                    for (int tt = 0; tt < 4; ++tt) a[tt] = an[tt];
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
#pragma unroll
        for (int t = 0; t < 8; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) h2[t][r] = relu_bits(h2[t][r]);
        // output layer on the vector ALUs (every lane group ends with the
        // three sums), sigmoid, and the logit gradient from dL/dc
        float p0 = 0.f, p1 = 0.f, p2 = 0.f;
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const f4_t wa = w2l[(q * 3 + 0) * 8 + t], wb = w2l[(q * 3 + 1) * 8 + t], wc = w2l[(q * 3 + 2) * 8 + t];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                p0 = fmaf(wa[r], h2[t][r], p0);
                p1 = fmaf(wb[r], h2[t][r], p1);
                p2 = fmaf(wc[r], h2[t][r], p2);
            }
        }
        p0 += __shfl_xor(p0, 16, kWave);
        p1 += __shfl_xor(p1, 16, kWave);
        p2 += __shfl_xor(p2, 16, kWave);
        p0 += __shfl_xor(p0, 32, kWave);
        p1 += __shfl_xor(p1, 32, kWave);
        p2 += __shfl_xor(p2, 32, kWave);
        // dL/dc_k = w_k g (g = dL/dC of the sample's ray); the colour is kept
        // for the compositing adjoint, which runs next
        float dl[3];
        {
            const float pp[3] = {p0, p1, p2};
            const float w = b.rec_w[rec];
            uint32_t g = 0;
#pragma unroll
            for (int ch = 0; ch < 3; ++ch) {
                const float c = sigmoid_hw(pp[ch] + lds[AdjLds::kB2 + ch]);
                const float gr = valid ? bb.d_rgb[3 * (int64_t)ray + ch] : 0.f;
                g = max(g, abs_bits(gr));
                const float dc = valid ? w * gr : 0.f;
                dl[ch] = dc * c * (1.f - c);
                acc4 += q == ch ? dl[ch] : 0.f;
                if (valid && q == ch) b.rec_c[3 * (int64_t)rec + ch] = c;
            }
            g_hi = max(g_hi, g);
            g_lo = min(g_lo, g ? g : g_lo);
        }
        // Exponents.  Of the sample: es, its dlogit's with W2's (its dp1 is at most
        // 3 2^7 2^7).  Of this batch, for P2: ep of its largest dlogit, e2 of its
        // second activations; sh2 is half of what the sample's dlogit is below.
        uint32_t dl_top = 0, dl_batch;
        int es, ep, e2, sh2;
        {
            uint32_t v = 0;
#pragma unroll
            for (int ch = 0; ch < 3; ++ch) dl_top = max(dl_top, abs_bits(dl[ch]));
#pragma unroll
            for (int t = 0; t < 8; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) v = max(v, __float_as_uint(h2[t][r]));   // (not negative)
            dl_batch = __builtin_amdgcn_readlane(wave_max_last(dl_top), kWave - 1);
            es = clamp_exp(exp_to(dl_top, 6) + e_w2, 120);
            sh2 = half_below(dl_top, dl_batch);
            ep = exp_to(dl_batch, 14);
            // (h2 is times s1 here; 2^-(ep + e2) takes both out)
            e2 = exp_to(__builtin_amdgcn_readlane(wave_max_last(v), kWave - 1), 14) + e_s1;
            // (what is not finite has the largest bits)
            bad |= ep < -kGradExp || e2 < -kActExp;
            ep = clamp_exp(ep, kGradExp);
            e2 = clamp_exp(e2, kActExp);
        }
        h4_t identity, replicate;   // [k = 4 q + e][n = j]: k == n, k == n % 4
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            identity[e] = (_Float16)(4 * q + e == j ? 1.f : 0.f);
            replicate[e] = (_Float16)(4 * q + e == (j & 3) ? 1.f : 0.f);
        }
        // dp1 = [h2 > 0] (W2^T dl); and this batch's P2 and db1 within the
        // wavefront: per 16 units a product of dl^T (rows 4 (t % 4) + channel,
        // the rest zero, so four tiles share an accumulator) and the transposed h2
        u4_t dp1h[4], dp1l[4];   // dp1's parts, tiles 2 s and 2 s + 1 in word pairs
        {
            const float p2 = pow2(ep + sh2);
            const u4_t dt = split_transpose(f4_t{dl[0], dl[1], dl[2], 0.f}, p2, replicate);
            const float scale = pow2(es), scale2 = pow2(e2 - e_s1 - sh2);
#pragma unroll
            for (int ch = 0; ch < 3; ++ch) dl[ch] *= scale;
            f4_t sum[2];
            sum[0] = sum[1] = f4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const f4_t wa = w2l[(q * 3 + 0) * 8 + t], wb = w2l[(q * 3 + 1) * 8 + t], wc = w2l[(q * 3 + 2) * 8 + t];
                f4_t v;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float u = fmaf(wa[r], dl[0], fmaf(wb[r], dl[1], wc[r] * dl[2]));
                    v[r] = h2[t][r] > 0.f ? u : 0.f;
                }
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    uint32_t hi, lo;
                    split_pair(v[2 * e], v[2 * e + 1], 1.f, hi, lo);
                    dp1h[t >> 1][2 * (t & 1) + e] = hi;
                    dp1l[t >> 1][2 * (t & 1) + e] = lo;
                }
                const u4_t ht = split_transpose(h2[t], scale2, identity);
                const bool mine = (j >> 2) == (t & 3);
                const h4_t dh = as_h4(mine ? dt[0] : 0u, mine ? dt[1] : 0u);
                const h4_t dlo = as_h4(mine ? dt[2] : 0u, mine ? dt[3] : 0u);
                f4_t &a = sum[t >> 2];
                a = __builtin_amdgcn_mfma_f32_16x16x16f16(dlo, as_h4(ht[0], ht[1]), a, 0, 0, 0);
                a = __builtin_amdgcn_mfma_f32_16x16x16f16(dh, as_h4(ht[2], ht[3]), a, 0, 0, 0);
                a = __builtin_amdgcn_mfma_f32_16x16x16f16(dh, as_h4(ht[0], ht[1]), a, 0, 0, 0);
                if (t & 1) __builtin_amdgcn_sched_barrier(0);
            }
            const float out = pow2(-(ep + e2));
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int r = 0; r < 3; ++r) acc2[u][r] = fmaf(sum[u][r], out, acc2[u][r]);
        }
        // dh1 = W1^T dp1 (A fragments of W1^T read from the forward's W1
        // layout and split here), dp0 = [h1 > 0] dh1
        f4_t dp0[8];   // times 2^es
        {
            // lane l needs W1[16 c4 + 4 (l / 16) + rr][16 ti + l % 16]: float
            // l % 4 of lane 16 g + 4 (l / 16) + rr of block (c4, ti), g =
            // (l % 16) / 4; the next step's eight values are read while this
            // step's are split
            const float *w1l = lds + AdjLds::w1(0, 16 * (j >> 2) + 4 * q) + (lane & 3);
            float a[8], an[8];
            auto read8 = [&](int idx, float w[8]) {
                const int ti = idx >> 2, s = idx & 3;
#pragma unroll
                for (int e = 0; e < 8; ++e) w[e] = w1l[((2 * s + (e >> 2)) * 8 + ti) * AdjLds::kW1Block + (e & 3) * 4];
            };
            read8(0, a);
#pragma unroll
            for (int ti = 0; ti < 8; ++ti) {
                f4_t d = f4_t{0.f, 0.f, 0.f, 0.f}, dlow = d;
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const int idx = 4 * ti + s;
                    read8(idx + 1 < 32 ? idx + 1 : idx, an);
                    u4_t hi, lo;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        uint32_t x, y;
                        split_pair(a[2 * e], a[2 * e + 1], 1.f, x, y);
                        hi[e] = x;
                        lo[e] = y;
                    }
                    const h8_t wh = __builtin_bit_cast(h8_t, hi), wl = __builtin_bit_cast(h8_t, lo);
                    const h8_t ph = __builtin_bit_cast(h8_t, dp1h[s]), pl = __builtin_bit_cast(h8_t, dp1l[s]);
                    dlow = __builtin_amdgcn_mfma_f32_16x16x32_f16(wl, ph, dlow, 0, 0, 0);
                    dlow = __builtin_amdgcn_mfma_f32_16x16x32_f16(wh, pl, dlow, 0, 0, 0);
                    d = __builtin_amdgcn_mfma_f32_16x16x32_f16(wh, ph, d, 0, 0, 0);
#pragma unroll
                    for (int e = 0; e < 8; ++e) a[e] = an[e];
                    __builtin_amdgcn_sched_barrier(0);
                }
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    dp0[ti][r] = h1[ti][r] > 0.f ? d[r] + dlow[r] : 0.f;
            }
        }
        // feature gradient (W0^T dp0)[0:12] of the sample (ray order); dp0 scaled by
        // the sample's largest, 2^e0s
        uint32_t dp0_top;   // the sample's largest dp0 (without 2^es)
        {
            uint32_t v = 0;
#pragma unroll
            for (int t = 0; t < 8; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) v = max(v, abs_bits(dp0[t][r]));
            v = across_rows_max(v);
            dp0_top = __float_as_uint(__uint_as_float(v) * pow2(-es));
            const int e0s = clamp_exp(exp_to(v, 14), 120);
            const float scale = pow2(e0s);
            f4_t df = f4_t{0.f, 0.f, 0.f, 0.f}, low = df;
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                u4_t hi, lo;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const f4_t &d = dp0[2 * s + (e >> 1)];
                    uint32_t x, y;
                    split_pair(d[2 * (e & 1)], d[2 * (e & 1) + 1], scale, x, y);
                    hi[e] = x;
                    lo[e] = y;
                }
                const h8_t wh = w0t[s * 64], wl = w0t[(4 + s) * 64];
                const h8_t ph = __builtin_bit_cast(h8_t, hi), pl = __builtin_bit_cast(h8_t, lo);
                low = __builtin_amdgcn_mfma_f32_16x16x32_f16(wl, ph, low, 0, 0, 0);
                low = __builtin_amdgcn_mfma_f32_16x16x32_f16(wh, pl, low, 0, 0, 0);
                df = __builtin_amdgcn_mfma_f32_16x16x32_f16(wh, ph, df, 0, 0, 0);
            }
            const f4_t unscale = *(const f4_t *)(lds + kAOffS0 + 4 * q);
            const float fs = pow2(-es), f0 = pow2(-e0s);
#pragma unroll
            for (int r = 0; r < 4; ++r) df[r] = (df[r] + low[r]) * unscale[r] * f0 * fs;
            if (valid && q < 3) *(f4_t *)(bb.rec_df + (int64_t)rec * 12 + 4 * q) = df;
        }
        // Weight gradients.  Exponents of the step's 128 samples by their largest
        // values, eb of dp1 (the dlogit's with W2's) and e0 of dp0, and of all samples
        // so far, e1 of h1, ed of the direction and ef of this lane's features; sh
        // and sh0: half of what the sample's dlogit and dp0 are below the largest.
        // The sums are brought to the step's scale.
        int sh, sh0;
        {
            uint32_t *tops = (uint32_t *)(lds + kAOffTops);
            uint32_t v = 0;
#pragma unroll
            for (int t = 0; t < 8; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) v = max(v, __float_as_uint(h1[t][r]));
            const u4_t tw = {dl_batch, wave_max_last(v), wave_max_last(dp0_top), wave_max_last(abs_bits(x[3]))};
            if (lane == kWave - 1) *(u4_t *)(tops + 16 * wave) = tw;
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const uint32_t f = row_max(abs_bits(x[k]));
                if (j == 0) tops[16 * wave + 4 + 3 * q + k] = f;
            }
            __syncthreads();
            uint32_t w = 0;   // the lane % 16-th value's largest
#pragma unroll
            for (int k = 0; k < kAdjWaves; ++k) w = max(w, tops[16 * k + j]);
            // this lane's column of P0 and its three features (a lane without a feature's column takes the direction's)
            const int c = slot_chunk(wave, lane), gr = slot_group(lane);
            const uint32_t wc = (uint32_t)__shfl((int)w, c < 3 ? 4 + 3 * gr + c : 3, kWave);
            uint32_t wf[3];
#pragma unroll
            for (int k = 0; k < 3; ++k) wf[k] = (uint32_t)__shfl((int)w, 4 + 3 * q + k, kWave);
            const uint32_t dl_all = __builtin_amdgcn_readlane(w, 0), dp0_all = __builtin_amdgcn_readlane(w, 2);
            sh = half_below(dl_top, dl_all);
            sh0 = half_below(dp0_top, dp0_all);
            const int was1 = eb + e1, was0 = e0 + ec;
            eb = exp_to(dl_all, 6) + e_w2 - e_s1;   // (without W1's s1)
            e0 = exp_to(dp0_all, 14);
            e1 = min(e1, exp_to(__builtin_amdgcn_readlane(w, 1), 14));
            ed = min(ed, exp_to(__builtin_amdgcn_readlane(w, 3), 14));
            bad |= min(eb, e0) < -kGradExp || min(e1, ed) < -kActExp;
            eb = max(min(eb, kGradExp), -kGradExp);
            e0 = max(min(e0, kGradExp), -kGradExp);
            eb_low = min(eb_low, eb);
            e0_low = min(e0_low, e0);
            eb = min(eb, eb_low + kStepExp);
            e0 = min(e0, e0_low + kStepExp);
            e1 = max(e1, -kActExp);
            ed = max(ed, -kActExp);
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                ef[k] = min(ef[k], exp_to(wf[k], 14));
                bad |= ef[k] < -kActExp;
                ef[k] = max(ef[k], -kActExp);
            }
            ec = c < 3 || (c == 3 && gr < 3) ? max(min(ec, exp_to(wc, 14)), -kActExp) : kXExp;
            const float f1 = pow2(eb + e1 - was1), f0 = pow2(e0 + ec - was0);
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                acc1[0][r] *= f1;
                acc1[1][r] *= f1;
                acc0[r] *= f0;
            }
        }
        // this batch's columns: split and transposed
        u4_t cols[kTiles];
        {
            const float c1 = pow2(min(max(eb + e_s1 - es + sh, -24), 0)), c0 = pow2(e0 - es + sh0), ch = pow2(e1 - sh);
            const float cd = pow2(ed - sh0), cx = pow2(kXExp - sh0);
            const h2_t one2 = {(_Float16)pow2(kXExp - sh), (_Float16)0.f};
            const u2_t ones = transpose16(u2_t{0u, __builtin_bit_cast(uint32_t, one2) << 16}, replicate);
            f4_t sum[2];   // db1
            sum[0] = sum[1] = f4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int t = 0; t < kTiles; ++t) {
                if (t < kTH1) {
                    // (in float16: what that cuts off is no more than what a remainder does)
                    u2_t hi, lo;
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        hi[e] = scale_h2(dp1h[t >> 1][2 * (t & 1) + e], c1);
                        lo[e] = scale_h2(dp1l[t >> 1][2 * (t & 1) + e], c1);
                    }
                    hi = transpose16(hi, identity);
                    lo = transpose16(lo, identity);
                    cols[t] = u4_t{hi[0], hi[1], lo[0], lo[1]};
                    const bool mine = j == 4 * (t & 3) + 3;   // (the fourth row of four)
                    const h4_t one = as_h4(mine ? ones[0] : 0u, mine ? ones[1] : 0u);
                    f4_t &a = sum[t >> 2];
                    a = __builtin_amdgcn_mfma_f32_16x16x16f16(one, as_h4(lo[0], lo[1]), a, 0, 0, 0);
                    a = __builtin_amdgcn_mfma_f32_16x16x16f16(one, as_h4(hi[0], hi[1]), a, 0, 0, 0);
                } else if (t < kTDP0) {
                    cols[t] = split_transpose(h1[t - kTH1], ch, identity);
                } else if (t < kTX) {
                    cols[t] = split_transpose(dp0[t - kTDP0], c0, identity);
                } else {
                    f4_t v;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int c = 4 * (t - kTX) + r;
                        if (c < 3) v[r] = x[c] * pow2(ef[c] - sh0);
                        else if (c == 3) v[r] = q < 3 ? x[3] * cd : cx;   // (1 in the padding slot)
                        else v[r] = c < 10 ? x[c] * cx : 0.f;
                    }
                    cols[t] = split_transpose(v, 1.f, identity);
                }
                if ((t & 3) == 3) __builtin_amdgcn_sched_barrier(0);
            }
            const float out = pow2(-(eb + kXExp));
#pragma unroll
            for (int u = 0; u < 2; ++u) acc2[u][3] = fmaf(sum[u][3], out, acc2[u][3]);
        }
        auto write_block = [&](float *blk) {
#pragma unroll
            for (int t = 0; t < kTiles; ++t) {
                u2_t *dst = (u2_t *)(blk + (t >> 1) * 512 + ((q >> 1) * 32 + (t & 1) * 16 + j) * 4 + (q & 1) * 2);
                dst[0] = u2_t{cols[t][0], cols[t][1]};
                dst[128] = u2_t{cols[t][2], cols[t][3]};
            }
        };
        // The wavefronts take turns at the two row blocks: turn t works on
        // wavefront t's while wavefront t + 1 writes the other.
        // P1: rows 32 (wave / 2) .., columns 64 (wave % 2) .. as two 32x32
        // tiles; P0: rows 32 (wave / 2) .., column slots 32 (wave % 2) ..
        const int ta = wave >> 1, tb = 4 + 2 * (wave & 1), tc = 8 + (wave >> 1), td = 12 + (wave & 1);
        if (wave == 0) write_block(blocks);
#pragma unroll 1
        for (int turn = 0; turn < kAdjWaves; ++turn) {
            __syncthreads();   // this turn's block is written, the other one consumed
            if (wave == turn + 1) write_block(blocks + ((turn + 1) & 1) * kBlock);
            const float *blk = blocks + (turn & 1) * kBlock + lane * 4;
            auto frag = [&](int tile, int part) {
                return *(const h8_t *)(blk + tile * 512 + part * 256);
            };
            const h8_t ah = frag(ta, 0), al = frag(ta, 1);
            const h8_t ch = frag(tb, 0), cl = frag(tb, 1), dh = frag(tb + 1, 0), dlo = frag(tb + 1, 1);
            const h8_t eh = frag(tc, 0), el = frag(tc, 1), xh = frag(td, 0), xl = frag(td, 1);
            acc1[0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(al, ch, acc1[0], 0, 0, 0);
            acc1[1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(al, dh, acc1[1], 0, 0, 0);
            acc0 = __builtin_amdgcn_mfma_f32_32x32x16_f16(el, xh, acc0, 0, 0, 0);
            acc1[0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, cl, acc1[0], 0, 0, 0);
            acc1[1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, dlo, acc1[1], 0, 0, 0);
            acc0 = __builtin_amdgcn_mfma_f32_32x32x16_f16(eh, xl, acc0, 0, 0, 0);
            acc1[0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, ch, acc1[0], 0, 0, 0);
            acc1[1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, dh, acc1[1], 0, 0, 0);
            acc0 = __builtin_amdgcn_mfma_f32_32x32x16_f16(eh, xh, acc0, 0, 0, 0);
        }
    }
    // the workgroup's partial
    const int lane = lane_id(), q = lane >> 4, j = lane & 15;
    float *out = bb.partials + (int64_t)blockIdx.x * kPartialFloats;
    const float out1 = pow2(-(eb + e1)), out0 = pow2(-(e0 + ec));
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int row = 32 * (wave >> 1) + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3), col = lane & 31;
#pragma unroll
        for (int u = 0; u < 2; ++u)
            out[kPart1 + row * 128 + 64 * (wave & 1) + 32 * u + col] = acc1[u][r] * out1;
        const int c = slot_chunk(wave, lane), g = slot_group(lane), src = c < 10 ? l0_input(c, g) : 0;
        if (c < 10) out[row * 48 + (src >= 0 ? src : 39)] = acc0[r] * out0;
    }
    // the others added up over the wavefronts in order
#pragma unroll
    for (int off = 8; off > 0; off >>= 1) acc4 += __shfl_xor(acc4, off, kWave);
    __syncthreads();   // the row blocks are consumed
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int r = 0; r < 4; ++r) blocks[wave * 516 + r * 128 + 64 * u + lane] = acc2[u][r];
    if (j == 0) blocks[wave * 516 + 512 + q] = acc4;
    __syncthreads();
    for (int i = threadIdx.x; i < 515; i += kAdjWaves * 64) {
        float v = 0.f;
#pragma unroll
        for (int k = 0; k < kAdjWaves; ++k) v += blocks[k * 516 + i];
        out[kPart2 + i] = v;
    }
    // rays whose gradients are so far apart that the halves of it that each factor carries cost bits
    {
        const uint32_t hi = __builtin_amdgcn_readlane(wave_max_last(g_hi), kWave - 1);
        const uint32_t lo = ~(uint32_t)__builtin_amdgcn_readlane(wave_max_last(~g_lo), kWave - 1);
        if (lane == 0) {
            ((uint32_t *)lds)[kAOffTops + wave] = hi;
            ((uint32_t *)lds)[kAOffTops + kAdjWaves + wave] = lo;
        }
        __syncthreads();
        uint32_t h = 0, l = 0x7f800000u;
        for (int k = 0; k < kAdjWaves; ++k) {
            h = max(h, ((uint32_t *)lds)[kAOffTops + k]);
            l = min(l, ((uint32_t *)lds)[kAOffTops + kAdjWaves + k]);
        }
        bad |= (int)(h >> 23) - (int)(l >> 23) > kRaySpread;
    }
    const int redo = __syncthreads_or(bad);
    if (threadIdx.x == 0) out[kRedoFlag] = redo ? 1.f : 0.f;
}

// ---------------------------------------------------------------------------
// The same in float32 throughout, for the workgroups that met a value outside
// the split's range (the flag in their partial): the same batches, every
// output overwritten.  Each wavefront owns some of the 105 16x16 output tiles
//   P0 = dp0^T [x|1|h1[0:8]]   (128 x 48: dW0 and, in column 39, db0)
//   P1 = dp1^T h1              (128 x 128: dW1)
//   P2 = dl^T h2               (16 x 128: dW2 in rows 0..2)
//   P3 = dp1^T [x|1][32:48]    (128 x 16: db1 in column 7)
//   P4 = dl^T [x|1][32:48]     (16 x 16: db2 in column 7)
// on FP32 MFMA; the wavefronts take turns writing their batch's per-sample
// rows [x|1, h1, h2, dp0, dlogit, dp1] into one LDS row block, and after each
// write every wavefront adds that block's 16 samples to its tiles.
// ---------------------------------------------------------------------------
constexpr int kWgTiles = 24 + 64 + 8 + 8 + 1;
constexpr int kAdjTPW = (kWgTiles + kAdjWaves - 1) / kAdjWaves;
// Row of the LDS block: the staged vectors at the offsets below, padded so
// that an MFMA operand read (16 consecutive columns of 4 consecutive rows)
// puts the 64 lanes on 64 distinct banks (row stride 16 mod 64 words).
constexpr int kAdjRow = kStDP1 + 128 + 24;
static_assert(kAdjRow % 64 == 16, "adjoint LDS row stride");
constexpr int kFOffW0T = AdjLds::kSize;                  // [c4 8][lane 64][4]
constexpr int kFOffRows = kFOffW0T + 8 * 64 * 4;        // [16][kAdjRow]
constexpr int kFLds = kFOffRows + 16 * kAdjRow;

struct WgTile {
    int a_col, b_col, out;   // row columns of A and B, offset in the partial
    int ld, rows, col;       // row length of the partial's matrix, rows it has; >= 0: its only column
};

__device__ __forceinline__ WgTile wg_tile(int t)
{
    if (t < 24) {
        const int mt = t / 3, nt = t % 3;
        return {kStDP0 + 16 * mt, kStX + 16 * nt, (16 * mt) * 48 + 16 * nt, 48, 16, -1};
    }
    t -= 24;
    if (t < 64) {
        const int mt = t / 8, nt = t % 8;
        return {kStDP1 + 16 * mt, kStH1 + 16 * nt, kPart1 + (16 * mt) * 128 + 16 * nt, 128, 16, -1};
    }
    t -= 64;
    if (t < 8) return {kStDL, kStH2 + 16 * t, kPart2 + 16 * t, 128, 3, -1};
    t -= 8;
    if (t < 8) return {kStDP1 + 16 * t, kStX + 32, kPart3 + 16 * t, 1, 16, 7};
    return {kStDL, kStX + 32, kPart4, 1, 3, 7};
}

// Two wavefronts per SIMD: a wavefront holds its batch's h1, h2, dp0, dp1
// (128 VGPRs) and its output tiles (56) between its turns at the row block.
__global__ __launch_bounds__(kAdjWaves * 64) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_mlp_adjoint_f32(
    GridK g, cic_mlp m, RenderBufs b, BackwardBufs bb)
{
    extern __shared__ __attribute__((aligned(16))) float lds[];
    float *out = bb.partials + (int64_t)blockIdx.x * kPartialFloats;
    if (out[kRedoFlag] == 0.f) return;   // uniform per block
    stage_weights_f32(m, lds, 1.f);
    for (int i = threadIdx.x; i < 8 * 64 * 4; i += blockDim.x) {
        const int rr = i & 3, l = (i >> 2) & 63, c4 = i >> 8;
        const int col = l & 15;
        lds[kFOffW0T + i] = col < 12 ? m.w0[(16 * c4 + 4 * (l >> 4) + rr) * 39 + col] : 0.f;
    }
    __syncthreads();
    const int lane = lane_id(), q = lane >> 4, j = lane & 15;
    const int wave = threadIdx.x / 64;
    const f2_t *w0f = (const f2_t *)(lds + AdjLds::kW0);
    const f4_t *w2l = (const f4_t *)(lds + AdjLds::kW2);
    const f4_t *w0t = (const f4_t *)(lds + kFOffW0T);
    // this lane's W1 fragment in block 0 (block k at + k * kW1Block floats)
    const float *w1f = lds + AdjLds::w1(0, lane);
    float *rows = lds + kFOffRows;

    // this workgroup's batches: the XCD's contiguous range, interleaved over
    // its workgroups and wavefronts; every wavefront runs the same number of
    // steps (the row-block turns are workgroup-wide)
    const int64_t total = (int64_t)b.offsets[b.n];
    const int64_t nbatch = (total + 15) / 16;
    const int xcd = blockIdx.x % kXcds, slot = blockIdx.x / kXcds, nslots = gridDim.x / kXcds;
    const int64_t per = (nbatch + kXcds - 1) / kXcds;
    const int64_t lo = xcd * per, hi = lo + per < nbatch ? lo + per : nbatch;
    const int64_t first = lo + (int64_t)slot * kAdjWaves, stride = (int64_t)nslots * kAdjWaves;
    const int64_t steps = hi > first ? (hi - first + stride - 1) / stride : 0;

    f4_t acc[kAdjTPW];
#pragma unroll
    for (int i = 0; i < kAdjTPW; ++i) acc[i] = f4_t{0.f, 0.f, 0.f, 0.f};

    for (int64_t st = 0; st < steps; ++st) {
        const int64_t bt = first + st * stride + wave;
        const int64_t s = bt * 16 + j;
        const bool valid = bt < hi && s < total;
        // ray order; a lane past the end works on sample 0 (in-bounds inputs,
        // no branches around the loads) with a zero logit gradient, so it
        // adds nothing to the weight gradients and stores nothing
        const uint32_t rec = valid ? (uint32_t)s : 0u;
        float x[10];
        sample_inputs(g, b, rec, q, x);
        // forward: layer 0 (40 -> 128)
        f4_t h1[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) h1[t] = *(const f4_t *)(lds + AdjLds::kB0 + 16 * t + 4 * q);
#pragma unroll
        for (int c2 = 0; c2 < 5; ++c2) {
            f2_t a[8];
#pragma unroll
            for (int t = 0; t < 8; ++t) a[t] = w0f[(t * 5 + c2) * 64 + lane];
#pragma unroll
            for (int e = 0; e < 2; ++e)
#pragma unroll
                for (int t = 0; t < 8; ++t)
                    h1[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[t][e], x[2 * c2 + e], h1[t], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int t = 0; t < 8; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) h1[t][r] = relu_bits(h1[t][r]);
        // layer 1 (128 -> 128)
        f4_t h2[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) h2[t] = *(const f4_t *)(lds + AdjLds::kB1 + 16 * t + 4 * q);
        {
            f4_t a[4], an[4];
#pragma unroll
            for (int tt = 0; tt < 4; ++tt) a[tt] = *(const f4_t *)(w1f + (tt * 8 + 0) * AdjLds::kW1Block);
#pragma unroll
            for (int c4 = 0; c4 < 8; ++c4) {
#pragma unroll
                for (int tg = 0; tg < 2; ++tg) {
                    const int step = c4 * 2 + tg, nx = step + 1 < 16 ? step + 1 : step;
                    const int nc4 = nx >> 1, ntg = nx & 1;
#pragma unroll
                    for (int tt = 0; tt < 4; ++tt)
                        an[tt] = *(const f4_t *)(w1f + ((4 * ntg + tt) * 8 + nc4) * AdjLds::kW1Block);
#pragma unroll
                    for (int rr = 0; rr < 4; ++rr)
#pragma unroll
                        for (int tt = 0; tt < 4; ++tt)
                            h2[4 * tg + tt] =
                                __builtin_amdgcn_mfma_f32_16x16x4f32(a[tt][rr], h1[c4][rr], h2[4 * tg + tt], 0, 0, 0);
#pragma unroll
                    for (int tt = 0; tt < 4; ++tt) a[tt] = an[tt];
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
#pragma unroll
        for (int t = 0; t < 8; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) h2[t][r] = relu_bits(h2[t][r]);
        // output layer on the vector ALUs (every lane group ends with the
        // three sums), sigmoid, and the logit gradient from dL/dc
        float p0 = 0.f, p1 = 0.f, p2 = 0.f;
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const f4_t wa = w2l[(q * 3 + 0) * 8 + t], wb = w2l[(q * 3 + 1) * 8 + t], wc = w2l[(q * 3 + 2) * 8 + t];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                p0 = fmaf(wa[r], h2[t][r], p0);
                p1 = fmaf(wb[r], h2[t][r], p1);
                p2 = fmaf(wc[r], h2[t][r], p2);
            }
        }
        p0 += __shfl_xor(p0, 16, kWave);
        p1 += __shfl_xor(p1, 16, kWave);
        p2 += __shfl_xor(p2, 16, kWave);
        p0 += __shfl_xor(p0, 32, kWave);
        p1 += __shfl_xor(p1, 32, kWave);
        p2 += __shfl_xor(p2, 32, kWave);
        // dL/dc_k = w_k g (g = dL/dC of the sample's ray); the colour is kept
        // for the compositing adjoint, which runs next
        float dl[3];
        {
            const float pp[3] = {p0, p1, p2};
            const float w = b.rec_w[rec];
            const uint32_t ray = b.rec_ray[rec];
#pragma unroll
            for (int ch = 0; ch < 3; ++ch) {
                const float c = sigmoid_hw(pp[ch] + lds[AdjLds::kB2 + ch]);
                const float dc = valid ? w * bb.d_rgb[3 * (int64_t)ray + ch] : 0.f;
                dl[ch] = dc * c * (1.f - c);
                if (valid && q == ch) b.rec_c[3 * (int64_t)rec + ch] = c;
            }
        }
        // dp1 = [h2 > 0] (W2^T dl), for output tile t
        auto dp1_tile = [&](int t) {
            const f4_t wa = w2l[(q * 3 + 0) * 8 + t], wb = w2l[(q * 3 + 1) * 8 + t], wc = w2l[(q * 3 + 2) * 8 + t];
            f4_t v;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float u = fmaf(wa[r], dl[0], fmaf(wb[r], dl[1], wc[r] * dl[2]));
                v[r] = h2[t][r] > 0.f ? u : 0.f;
            }
            return v;
        };
        // dh1 = W1^T dp1 (A fragments of W1^T read from the forward's W1
        // layout), dp0 = [h1 > 0] dh1
        f4_t dp0[8];
#pragma unroll
        for (int ti = 0; ti < 8; ++ti) dp0[ti] = f4_t{0.f, 0.f, 0.f, 0.f};
        // kept in registers through the weight-gradient turns below (32 more
        // live registers, some spilled, against recomputing it, W2 reads from
        // LDS included, inside the writing wavefront's turn, where every other
        // wavefront waits: fused adjoint 2.91 -> 2.64 ms per 8192-ray step)
        f4_t dp1[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) dp1[t] = dp1_tile(t);
        {
            // lane l needs W1[16 c4 + 4 (l / 16) + rr][16 ti + l % 16]: float
            // l % 4 of lane 16 g + 4 (l / 16) + rr of block (c4, ti), g =
            // (l % 16) / 4; the next (ti, c4) step's four values are read
            // while this step's MFMAs run
            const float *w1l = lds + AdjLds::w1(0, 16 * ((lane & 15) >> 2) + 4 * (lane >> 4)) + (lane & 3);
            float a[4], an[4];
#pragma unroll
            for (int rr = 0; rr < 4; ++rr) a[rr] = w1l[rr * 4];
#pragma unroll
            for (int idx = 0; idx < 64; ++idx) {
                const int ti = idx >> 3, c4 = idx & 7;
                const int nx = idx + 1 < 64 ? idx + 1 : idx, nti = nx >> 3, nc4 = nx & 7;
#pragma unroll
                for (int rr = 0; rr < 4; ++rr) an[rr] = w1l[(nc4 * 8 + nti) * AdjLds::kW1Block + rr * 4];
#pragma unroll
                for (int rr = 0; rr < 4; ++rr)
                    dp0[ti] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[rr], dp1[c4][rr], dp0[ti], 0, 0, 0);
#pragma unroll
                for (int rr = 0; rr < 4; ++rr) a[rr] = an[rr];
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int ti = 0; ti < 8; ++ti)
#pragma unroll
            for (int r = 0; r < 4; ++r) dp0[ti][r] = h1[ti][r] > 0.f ? dp0[ti][r] : 0.f;
        // feature gradient (W0^T dp0)[0:12] of the sample (ray order)
        {
            f4_t df = f4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int c4 = 0; c4 < 8; ++c4) {
                const f4_t a = w0t[c4 * 64 + lane];
#pragma unroll
                for (int rr = 0; rr < 4; ++rr) df = __builtin_amdgcn_mfma_f32_16x16x4f32(a[rr], dp0[c4][rr], df, 0, 0, 0);
            }
            if (valid && q < 3) *(f4_t *)(bb.rec_df + (int64_t)rec * 12 + 4 * q) = df;
        }
        // weight gradients: the wavefronts take turns at the row block
        for (int turn = 0; turn < kAdjWaves; ++turn) {
            __syncthreads();   // the previous block is consumed
            if (wave == turn) {
                float *row = rows + j * kAdjRow;
#pragma unroll
                for (int c = 0; c < 10; ++c) {
                    const int src = l0_input(c, q);
                    row[kStX + (src >= 0 ? src : 39)] = src >= 0 ? x[c] : 1.0f;
                }
#pragma unroll
                for (int t = 0; t < 8; ++t) {
                    *(f4_t *)(row + kStH1 + 16 * t + 4 * q) = h1[t];
                    *(f4_t *)(row + kStH2 + 16 * t + 4 * q) = h2[t];
                    *(f4_t *)(row + kStDP0 + 16 * t + 4 * q) = dp0[t];
                    *(f4_t *)(row + kStDP1 + 16 * t + 4 * q) = dp1[t];
                }
                *(f4_t *)(row + kStDL + 4 * q) = q == 0 ? f4_t{dl[0], dl[1], dl[2], 0.f} : f4_t{0.f, 0.f, 0.f, 0.f};
            }
            __syncthreads();
            // per owned tile, the block's 16 samples in four k-steps (one
            // address pair per tile, the k-step offsets immediate); the
            // compiler may start the next tiles' operand reads during these
            // MFMAs (with a scheduling barrier per tile the adjoint kernel
            // took 3.02 against 2.94 ms per 8192-ray step)
            const float *rl = rows + (lane >> 4) * kAdjRow + (lane & 15);
#pragma unroll
            for (int i = 0; i < kAdjTPW; ++i) {
                const int t = wave + kAdjWaves * i;
                if (t < kWgTiles) {
                    const WgTile w = wg_tile(t);
                    const float *pa = rl + w.a_col, *pb = rl + w.b_col;
#pragma unroll
                    for (int kk = 0; kk < 16; kk += 4)
                        acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(pa[kk * kAdjRow], pb[kk * kAdjRow], acc[i], 0, 0,
                                                                      0);
                }
            }
        }
    }
#pragma unroll
    for (int i = 0; i < kAdjTPW; ++i) {
        const int t = wave + kAdjWaves * i;
        if (t < kWgTiles) {
            const WgTile w = wg_tile(t);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = 4 * (lane >> 4) + r, col = lane & 15;
                if (row < w.rows && (w.col < 0 || col == w.col))
                    out[w.out + row * w.ld + (w.col < 0 ? col : 0)] = acc[i][r];
            }
        }
    }
}

// Sum the per-block partials in block order and add into the gradients.
// Sum of the per-block partials of every weight-gradient entry, added to the
// gradient.  A block takes 64 consecutive outputs; its 16 groups of 64
// threads sum contiguous ranges of blocks (coalesced over the outputs), and
// the group sums are added in group order: a fixed order, so the result is
// deterministic.
constexpr int kApplyOut = 64, kApplyGroups = 16;

__device__ __forceinline__ bool wgrad_entry(int e, int &src, float *&dst, const BackwardBufs &bb)
{
    if (e < 128 * 39) {
        src = (e / 39) * 48 + e % 39;
        dst = bb.d_w0 + e;
    } else if (e < 128 * 39 + 128) {
        const int o = e - 128 * 39;
        src = o * 48 + 39;
        dst = bb.d_b0 + o;
    } else if (e < 128 * 39 + 128 + 128 * 128) {
        const int k = e - (128 * 39 + 128);
        src = kPart1 + k;
        dst = bb.d_w1 + k;
    } else if (e < 128 * 39 + 128 + 128 * 128 + 3 * 128) {
        const int k = e - (128 * 39 + 128 + 128 * 128);
        src = kPart2 + k;
        dst = bb.d_w2 + k;
    } else if (e < 128 * 39 + 128 + 128 * 128 + 3 * 128 + 128) {
        const int o = e - (128 * 39 + 128 + 128 * 128 + 3 * 128);
        src = kPart3 + o;
        dst = bb.d_b1 + o;
    } else if (e < 128 * 39 + 128 + 128 * 128 + 3 * 128 + 128 + 3) {
        const int ch = e - (128 * 39 + 128 + 128 * 128 + 3 * 128 + 128);
        src = kPart4 + ch;
        dst = bb.d_b2 + ch;
    } else {
        return false;
    }
    return true;
}

__global__ __launch_bounds__(kApplyOut * kApplyGroups) void k_wgrad_apply(const float *partials, int nblk,
                                                                          BackwardBufs bb)
{
    __shared__ float part[kApplyGroups][kApplyOut];
    const int o = threadIdx.x % kApplyOut, grp = threadIdx.x / kApplyOut;
    const int e = blockIdx.x * kApplyOut + o;
    int src = 0;
    float *dst = nullptr;
    const bool ok = wgrad_entry(e, src, dst, bb);
    const int per = (nblk + kApplyGroups - 1) / kApplyGroups;
    const int b0 = grp * per, b1 = min(nblk, b0 + per);
    float sum = 0.f;
    if (ok)
        for (int blk = b0; blk < b1; ++blk) sum += partials[(int64_t)blk * kPartialFloats + src];
    part[grp][o] = sum;
    __syncthreads();
    if (grp == 0 && ok) {
        float t = 0.f;
#pragma unroll
        for (int k = 0; k < kApplyGroups; ++k) t += part[k][o];
        *dst += t;
    }
}

void launch_mlp_adjoint(const GridK &g, const cic_mlp &m, const RenderBufs &b, const BackwardBufs &bb, hipStream_t s)
{
    const int lds = kALds * (int)sizeof(float), lds_f32 = kFLds * (int)sizeof(float);
    static bool attr_set = false;
    if (!attr_set) {
        (void)hipFuncSetAttribute((const void *)k_mlp_adjoint, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        (void)hipFuncSetAttribute((const void *)k_mlp_adjoint_f32, hipFuncAttributeMaxDynamicSharedMemorySize, lds_f32);
        attr_set = true;
    }
    const int nblk = std::min(num_cus_b(), kWgBlocks);
    hipLaunchKernelGGL(k_ray_encode, dim3((unsigned)((4 * b.n + 255) / 256)), dim3(256), 0, s, b);
    hipLaunchKernelGGL(k_mlp_adjoint, dim3(nblk), dim3(kAdjWaves * 64), lds, s, g, m, b, bb);
    hipLaunchKernelGGL(k_mlp_adjoint_f32, dim3(nblk), dim3(kAdjWaves * 64), lds_f32, s, g, m, b, bb);
    const int n_out = 128 * 39 + 128 + 128 * 128 + 3 * 128 + 128 + 3;
    hipLaunchKernelGGL(k_wgrad_apply, dim3((n_out + kApplyOut - 1) / kApplyOut), dim3(kApplyOut * kApplyGroups), 0, s,
                       (const float *)bb.partials, nblk, bb);
}

}  // namespace cic
