// Ray marching, live-sample compaction, voxel-order bucketing and the final
// per-ray accumulation of the rendering quadrature.
//
// March: one wavefront per ray, 64 samples per step (one per lane).  Each
// lane finds its sample's voxel, skips it if unoccupied, interpolates the
// raw density, applies softplus and forms the optical depth sigma*delta.  A
// wavefront inclusive scan of the optical depths gives every lane its
// transmittance T_k = exp(-(carry + exclusive sum)); the first lane whose
// T_k falls below the threshold ends the ray (ballot + find-first-set).
// Live samples (occupied, before termination) are written to per-ray slots
// with their weight w_k = T_k (1 - exp(-sigma_k delta)); sum w_k t_k is a
// wavefront tree sum.  The MLP stage later reads the compacted live samples;
// the per-ray reduction sums w_k c_k in sample order, so results do not
// depend on the order in which the MLP stage visits samples.
#include "kernels.h"

namespace cic {

constexpr int kRayWaves = 4;   // rays (wavefronts) per 256-thread block

// ln(u) for finite u >= 1/2 (the only inputs below whose result is used):
// the hardware log2 times ln 2 rounded to float (3e-9 relative), without the
// library's denormal scaling and extended-precision product
__device__ __forceinline__ float ln_hw(float u)
{
    return __builtin_amdgcn_logf(u) * 0.693147182f;
}

// e^x for x <= 15 (no overflow to guard): 2^(x log2 e) on the hardware exp2,
// the rounding error of the product x log2 e (and of log2 e itself) carried
// as a first-order correction e^lo ~ 1 + lo ln 2 (within 1.2e-7 relative
// when exp2 is correctly rounded)
__device__ __forceinline__ float exp_hw(float x)
{
    constexpr float kL = 1.44269502162933349609375f;    // log2(e) rounded to float
    constexpr float kLlo = 1.925963033500011079e-8f;    // log2(e) - kL
    const float hi = x * kL;
    const float lo = fmaf(x, kLlo, fmaf(x, kL, -hi));
    const float eh = __builtin_amdgcn_exp2f(hi);
    return fmaf(eh, lo * 0.693147182f, eh);
}

// softplus(x) = log(1 + e^x) (x + e^-x above 15), with log1p(e) taken as
// log(u) e / (u - 1), u = 1 + e: Goldberg's form, accurate to a few ulp when
// the logarithm is (3.1e-7 relative over x <= 15 with the hardware exp2, log2
// and reciprocal correctly rounded), where the library's log1pf spends about
// a hundred instructions per call
__device__ __forceinline__ float softplus_fast(float x)
{
    const bool big = x > 15.0f;
    const float e = exp_hw(big ? -x : x), u = 1.0f + e;
    const float l = u == 1.0f ? e : ln_hw(u) * (e * __builtin_amdgcn_rcpf(u - 1.0f));
    return big ? x + e : l;
}

// Opacity 1 - e^-s of optical depth s >= 0: directly where e^-s <= 1/2, and
// in Kahan's form (1 - u) s / -log(u), u = e^-s, near s = 0, where the
// subtraction would cancel (2.4e-7 relative, from the hardware exp2 and log2)
__device__ __forceinline__ float opacity_fast(float s)
{
    const float u = __expf(-s);
    const float k = u == 1.0f ? s : (1.0f - u) * s * __builtin_amdgcn_rcpf(-ln_hw(u));
    return u > 0.5f ? k : 1.0f - u;
}

// Wavefront inclusive prefix sum on DPP lane moves (no LDS round trips):
// within each row of 16 lanes, shifts by 1, 2, 4 and 8 (a lane without a
// source adds 0); then rows 1 and 3 add the last lane of rows 0 and 2, and
// rows 2 and 3 add lane 31.
template <int CTRL, int ROW_MASK, bool BOUND_ZERO>
__device__ __forceinline__ float dpp_add(float v)
{
    return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROW_MASK, 0xf, BOUND_ZERO));
}
__device__ __forceinline__ float wave_incl_scan_dpp(float v)
{
    v = dpp_add<0x111, 0xf, true>(v);    // row_shr:1
    v = dpp_add<0x112, 0xf, true>(v);    // row_shr:2
    v = dpp_add<0x114, 0xf, true>(v);    // row_shr:4
    v = dpp_add<0x118, 0xf, true>(v);    // row_shr:8
    v = dpp_add<0x142, 0xa, false>(v);   // row_bcast:15 into rows 1, 3
    v = dpp_add<0x143, 0xc, false>(v);   // row_bcast:31 into rows 2, 3
    return v;
}
// the value of the lane below (0 in lane 0): wave_shr:1
__device__ __forceinline__ float wave_shr1(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x138, 0xf, 0xf, true));
}


// March of one ray by a wavefront.  Bound by the vector L1's lookups (about
// one per CU and cycle: the 64 samples of a step lie in as many cells, so
// every corner row is a cache line of its own) and its vector instructions
// together: what is the same for a ray stays in scalar registers (its data,
// its slots' bases), indexes are 32 bits, and a step with no occupied sample
// ends after the lookup.  800x800 frame (160^3, 256 samples, float32) 645 ->
// 568 us, pass of 2^21 rays over a float16 grid 1.60 -> 1.35 ms.  Fewer
// instructions alone do not help (the box intervals computed beforehand,
// one ray per thread: 23% fewer, and 8% slower), nor do several rays per
// wavefront (4: +7%, 8: +20%) or an eighth of the image per XCD (+55%: the
// rows through the scene have most of the work).
template <typename T>
__device__ __forceinline__ void march_ray(const GridK &g, const OptsK &op, const RenderBufs &b, int64_t ray, int lane)
{
    const int N = op.n_samples;
    float o[3], d[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        o[a] = b.rays_o[3 * ray + a];
        d[a] = b.rays_d[3 * ray + a];
    }
    float tn, tf;
    const bool hit = ray_box(o, d, g, tn, tf);
    const float delta = (tf - tn) / (float)N;
    if (!hit) {
        if (lane == 0) {
            b.count[ray] = 0;
            b.info[ray] = RayInfo{tn, 0.f, 1.f, 0.f};
        }
        return;
    }
    const float thr = op.et_threshold;
    uint16_t *slot_k = b.slot_k + ray * (int64_t)N;
    float *slot_w = b.slot_w + ray * (int64_t)N;
    float *slot_t = b.slot_t ? b.slot_t + ray * (int64_t)N : nullptr;
    float carry = 0.f, depth = 0.f, t_stop = -1.f;
    uint32_t count = 0;
    for (int base = 0; base < N; base += kWave) {
        const int k = base + lane;
        const bool valid = k < N;
        float s = 0.f, tk = 0.f;
        bool occ = false;
        if (valid) {
            int i0[3];
            float fr[3];
            sample_voxel(o, d, tn, delta, k, g, i0, fr, tk);
            occ = g.occ ? (g.occ[cell_index32(g, i0)] != 0) : true;
            if (occ) s = softplus_fast(density_at<T>(g, i0, fr) + g.shift) * delta;
        }
        if (!__builtin_amdgcn_ballot_w64(occ)) {
            // no sample of the step is occupied: nothing to add, and every
            // transmittance is the carried one
            const float Tc = __expf(-carry);
            if (thr > 0.f && Tc < thr) {
                t_stop = Tc;
                break;
            }
            continue;
        }
        const float incl = wave_incl_scan_dpp(s);
        const float excl = wave_shr1(incl);
        const float Tk = __expf(-(carry + excl));
        const uint64_t tmask = __builtin_amdgcn_ballot_w64(valid && thr > 0.f && Tk < thr);
        const int first = tmask ? __builtin_ctzll(tmask) : kWave;
        const bool live = valid && occ && lane < first;
        const float w = live ? Tk * opacity_fast(s) : 0.f;
        const uint64_t lmask = __builtin_amdgcn_ballot_w64(live);
        if (live) {
            const uint32_t below = __builtin_amdgcn_mbcnt_lo((uint32_t)lmask, 0u);
            const uint32_t pos = count + __builtin_amdgcn_mbcnt_hi((uint32_t)(lmask >> 32), below);
            // (32-bit byte offsets from the ray's uniform bases)
            *(uint16_t *)((char *)slot_k + 2u * pos) = (uint16_t)k;
            *(float *)((char *)slot_w + 4u * pos) = w;
            if (slot_t) *(float *)((char *)slot_t + 4u * pos) = Tk;
        }
        count += (uint32_t)__builtin_popcountll(lmask);
        depth += __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wave_incl_scan_dpp(w * tk)), kWave - 1));
        if (first < kWave) {
            t_stop = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(Tk), first));
            break;
        }
        carry += __int_as_float(__builtin_amdgcn_readlane(__float_as_int(incl), kWave - 1));
    }
    if (t_stop < 0.f) t_stop = __expf(-carry);
    if (lane == 0) {
        b.count[ray] = count;
        b.info[ray] = RayInfo{tn, delta, t_stop, depth};
    }
}

// COUNTED: a device-counted pass, which strides over its rays (a loop costs the
// others 12%: 1.35 -> 1.51 ms per 95 M samples)
template <typename T, bool COUNTED>
__global__ __launch_bounds__(256) void k_march(GridK g, OptsK op, RenderBufs b)
{
    const int lane = lane_id();
    const int64_t first = (int64_t)blockIdx.x * kRayWaves + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    if constexpr (!COUNTED) {
        if (first < b.n) march_ray<T>(g, op, b, first, lane);
    } else {
        const int64_t n = min((int64_t)*b.n_active, b.n);
        // rays that the pass does not have: no samples
        for (int64_t r = n + (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < b.n;
             r += (int64_t)gridDim.x * blockDim.x) {
            b.count[r] = 0;
            b.info[r] = RayInfo{0.f, 0.f, 1.f, 0.f};
        }
        for (int64_t ray = first; ray < n; ray += (int64_t)gridDim.x * kRayWaves) march_ray<T>(g, op, b, ray, lane);
    }
}

// March of a tile of 8 x 8 pixels by a wavefront, one ray per lane (whole
// image rows of large frames).  The lanes' samples of one step lie in a handful
// of neighbouring cells, so a gather is a few cache lines instead of one per
// lane, a step is skipped when none of the 64 rays needs it, and the box
// intervals cost one lane each.  The sums are those of k_march bit for bit:
// its scan of a 64-sample chunk adds within rows of 16 samples by steps of 1,
// 2, 4 and 8 and then the rows' ends, which a lane follows here on 16
// registers (prefix16, and the row constants below); the chunk's depth sum is
// the same tree.  Live samples are collected in LDS per lane and row, then
// written 16 per ray at a time.  Bound by its vector instructions (89% of its
// cycles, half of them the lookups' positions).  800x800 frame of a 160^3 grid
// with empty space 582 -> 335 us, 1000x900 926 -> 464-512; smaller frames see
// kMarchTileMin.  Caller's rays stay with
// k_march: 64 consecutive rays of one image row are faster here (640,000: 564
// -> 442 us), but rays that are not neighbours up to 1.8 times slower.
constexpr int kTileRow = 16;

// Inclusive prefixes of 16 values: rows of k_march's scan.
__device__ __forceinline__ void prefix16(float x[kTileRow])
{
#pragma unroll
    for (int off = 1; off < kTileRow; off <<= 1)
#pragma unroll
        for (int i = kTileRow - 1; i >= off; --i) x[i] += x[i - off];
}

// Rays: the pixels of `rows` image rows of `width` (row-major).
template <typename T>
__global__ __launch_bounds__(256) void k_march_tile(GridK g, OptsK op, RenderBufs b, int width, int rows)
{
    __shared__ float sw[kRayWaves][kWave][kTileRow + 1];
    __shared__ uint16_t sk[kRayWaves][kWave][kTileRow + 2];
    const int lane = lane_id(), wv = threadIdx.x / kWave;
    const int tile = (int)blockIdx.x * kRayWaves + __builtin_amdgcn_readfirstlane(wv), tx = (width + 7) / 8;
    const int px = (tile % tx) * 8 + (lane & 7), py = (tile / tx) * 8 + (lane >> 3);
    if (tile / tx * 8 >= rows) return;
    const bool have = px < width && py < rows;
    const uint32_t ray = (uint32_t)(py * width + px);   // at most 2^21 rays
    float o[3] = {0.f, 0.f, 0.f}, d[3] = {0.f, 0.f, 0.f}, tn = 0.f, tf = 0.f;
    bool hit = false;
    if (have) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            o[a] = b.rays_o[3 * (int64_t)ray + a];
            d[a] = b.rays_d[3 * (int64_t)ray + a];
        }
        hit = ray_box(o, d, g, tn, tf);
    }
    const int N = op.n_samples;
    const float delta = hit ? (tf - tn) / (float)N : 0.f;
    const float thr = op.et_threshold;
    // sample_voxel of sample k0 + i
    auto row_voxel = [&](float kf0, int i, int i0[3], float fr[3]) {
        const float tk = tn + (kf0 + ((float)i + 0.5f)) * delta;
        float x[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) x[a] = o[a] + tk * d[a];
        locate(x, g, i0, fr);
    };
    float carry = 0.f, depth = 0.f, t_stop = 1.f;
    uint32_t count = 0;
    bool run = hit;   // still marching
    for (int base = 0; base < N && __builtin_amdgcn_ballot_w64(run); base += kWave) {
        float a0 = 0.f, a2 = 0.f, l31 = 0.f;   // row 0's and row 2's sums, the first two rows' sum
        float last = 0.f;                      // inclusive sum of the sample before
        float dsum[4] = {0.f, 0.f, 0.f, 0.f};  // the rows' depth sums
#pragma unroll 1
        for (int row = 0; row < 4; ++row) {
            const int k0 = base + row * kTileRow;
            if (k0 >= N) break;
            const float kf0 = (float)k0;   // (k0 + i + 1/2 is exact, also as the sum of kf0 and i + 1/2)
            // which of the row's samples are occupied
            uint32_t m = 0;
            if (run) {
                const uint32_t valid = N - k0 >= kTileRow ? 0xffffu : (1u << (N - k0)) - 1u;
                if (g.occ) {
                    uint8_t by[kTileRow];
#pragma unroll
                    for (int i = 0; i < kTileRow; ++i) {
                        int i0[3];
                        float fr[3];
                        row_voxel(kf0, i, i0, fr);
                        by[i] = g.occ[cell_index32(g, i0)];
                    }
#pragma unroll
                    for (int i = 0; i < kTileRow; ++i) m |= by[i] ? 1u << i : 0u;
                    m &= valid;
                } else {
                    m = valid;
                }
            }
            float rowsum = 0.f;   // this row's own inclusive end
            if (__builtin_amdgcn_ballot_w64(m != 0)) {
                float s[kTileRow], x[kTileRow];
#pragma unroll
                for (int q = 0; q < kTileRow; q += 4) {
                    const uint32_t mq = (m >> q) & 15u;
#pragma unroll
                    for (int i = 0; i < 4; ++i) s[q + i] = 0.f;
                    if (!__builtin_amdgcn_ballot_w64(mq != 0)) continue;
                    if (mq) {
                        // the four samples' gathers go out together (an
                        // unoccupied one's is in bounds and unused)
                        float raw[4];
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            int i0[3];
                            float fr[3];
                            row_voxel(kf0, q + i, i0, fr);
                            raw[i] = density_at<T>(g, i0, fr);
                        }
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            s[q + i] = (mq >> i) & 1u ? softplus_fast(raw[i] + g.shift) * delta : 0.f;
                    }
                }
#pragma unroll
                for (int i = 0; i < kTileRow; ++i) x[i] = s[i];
                prefix16(x);
                rowsum = x[kTileRow - 1];
                float wt[kTileRow];
                uint32_t nrow = 0;
#pragma unroll
                for (int i = 0; i < kTileRow; ++i) {
                    // inclusive sum of the sample before: rows 1 and 3 add the
                    // row before them, rows 2 and 3 the first two
                    float excl = last;
                    if (i > 0) excl = row == 0 ? x[i - 1] : row == 1 ? x[i - 1] + a0 : row == 2 ? x[i - 1] + l31
                                                                                               : (x[i - 1] + a2) + l31;
                    const float Tk = __expf(-(carry + excl));
                    if (run && k0 + i < N && thr > 0.f && Tk < thr) {
                        t_stop = Tk;
                        run = false;
                    }
                    const bool live = run && ((m >> i) & 1u);
                    const float tk = tn + (kf0 + ((float)i + 0.5f)) * delta;
                    const float w = live ? Tk * opacity_fast(s[i]) : 0.f;
                    wt[i] = w * tk;
                    if (live) {
                        sw[wv][lane][nrow] = w;
                        sk[wv][lane][nrow] = (uint16_t)(k0 + i);
                        ++nrow;
                    }
                }
#pragma unroll
                for (int off = 1; off < kTileRow; off <<= 1)
#pragma unroll
                    for (int i = 0; i < kTileRow; i += 2 * off) wt[i] += wt[i + off];
                dsum[row] = wt[0];
                // the rows' samples to their slots: 16 lanes per ray
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int it = 0; it < kWave / 4; ++it) {
                    const int rr = it * 4 + (lane >> 4), e = lane & 15;
                    const uint32_t nr = __shfl(nrow, rr, kWave), at = __shfl(count, rr, kWave);
                    const int64_t slot = (int64_t)__shfl(ray, rr, kWave) * N + at + (uint32_t)e;
                    if ((uint32_t)e < nr) {
                        b.slot_w[slot] = sw[wv][rr][e];
                        b.slot_k[slot] = sk[wv][rr][e];
                    }
                }
                __builtin_amdgcn_wave_barrier();
                count += nrow;
            } else if (run && thr > 0.f) {
                // an empty row adds nothing, and all its transmittances are one
                const float Tc = __expf(-(carry + last));
                if (Tc < thr) {
                    t_stop = Tc;
                    run = false;
                }
            }
            if (row == 0) {
                a0 = last = rowsum;
            } else if (row == 1) {
                l31 = last = rowsum + a0;
            } else if (row == 2) {
                a2 = rowsum;
                last = rowsum + l31;
            } else {
                last = (rowsum + a2) + l31;
            }
        }
        depth += (dsum[3] + dsum[2]) + (dsum[1] + dsum[0]);
        carry += last;
    }
    if (run) t_stop = __expf(-carry);
    if (have) {
        b.count[ray] = count;
        b.info[ray] = RayInfo{tn, delta, t_stop, depth};
    }
}

// Fewest pixels that march in tiles: below, too few wavefronts are left, and the
// longest decide.  Less so without an occupancy grid, where the rays' lengths are
// alike.  us in tiles and one wavefront per ray (96^3 and 160^3 grids): 450x450
// 223 / 187 and 242 / 241, without occupancy 173 / 167 and 193 / 232; 512x512 291
// / 252 and 306 / 296, without 186 / 210 and 208 / 286; 640x480 302 / 305 and 319
// / 352, without 209 / 252 and 232 / 348.
constexpr int64_t kMarchTileMinOcc = 300000, kMarchTileMin = 250000;

template <typename T>
void launch_march(const GridK &g, const OptsK &o, const RenderBufs &b, int width, hipStream_t s)
{
    if (b.n == 0) return;
    if (width > 0 && b.n >= (g.occ ? kMarchTileMinOcc : kMarchTileMin)) {
        const int rows = (int)(b.n / width), tiles = ((width + 7) / 8) * ((rows + 7) / 8);
        hipLaunchKernelGGL(k_march_tile<T>, dim3((unsigned)((tiles + kRayWaves - 1) / kRayWaves)), dim3(256), 0, s, g,
                           o, b, width, rows);
        return;
    }
    const dim3 blocks = ray_grid(b, kRayWaves);
    if (b.n_active) hipLaunchKernelGGL((k_march<T, true>), blocks, dim3(256), 0, s, g, o, b);
    else hipLaunchKernelGGL((k_march<T, false>), blocks, dim3(256), 0, s, g, o, b);
}
template void launch_march<float>(const GridK &, const OptsK &, const RenderBufs &, int, hipStream_t);
template void launch_march<__half>(const GridK &, const OptsK &, const RenderBufs &, int, hipStream_t);

// Head-of-run detection for equal consecutive keys among the first `active`
// lanes: returns the mask of run heads; run length of a head lane is the
// distance to the next head (or to `active`).
__device__ __forceinline__ uint64_t run_heads(uint32_t key, bool active)
{
    const uint32_t prev = __shfl_up(key, 1, kWave);
    const bool head = active && (lane_id() == 0 || prev != key);
    return __ballot(head);
}

__device__ __forceinline__ int run_length(uint64_t heads, int active)
{
    const int l = lane_id();
    const uint64_t above = (l == kWave - 1) ? 0ull : (heads & ~((2ull << l) - 1ull));
    const int next = above ? (__ffsll((unsigned long long)above) - 1) : active;
    return next - l;
}

// Compaction: the live samples' rays and sample indices from the per-ray slots
// to consecutive records (the weights stay in the slots), and in voxel mode a
// brick key per sample and each run of equal bricks added to counts[brick].
// Bound by the latency of dependent loads, so a wavefront takes several rays:
// lane l loads ray l's header, and a ray's slots are loaded before the ray
// before it is stored (as far as the compiler knows the stores could alias
// the slots, so it would not move the loads up by itself).
//
// Ray order: RAYS rays per wavefront, the first 128 slots of all of them in
// flight together.  1, 4 or 8 by the number of rays, since small passes need
// the wavefronts and large ones the loads (us with 1 / 4 / 8 rays per
// wavefront, and with one whose loads all follow each other: 64x64 frame
// 3.7 / 5.5 / 8.2, 4.2; 30,000 rays 7.3 / 7.9 / 10.1, 8.6; 333x257 15.8 /
// 13.4 / 15.2, 22.5; 450x400 30.9 / 24.7 / 26.1, 46.8; 800x800 - / 97.6 /
// 95.8, 171).
template <int RAYS> __device__ __forceinline__ void compact_rays(const RenderBufs &b, int64_t ray0)
{
    const int lane = lane_id();
    uint32_t lc = 0, lo = 0;
    if (lane < RAYS && ray0 + lane < b.n) {
        lc = b.count[ray0 + lane];
        lo = b.offsets[ray0 + lane];
    }
    uint32_t cnt[RAYS], off[RAYS];
    uint16_t ka[RAYS], kb[RAYS];
#pragma unroll
    for (int r = 0; r < RAYS; ++r) {
        cnt[r] = __builtin_amdgcn_readlane(lc, r);
        off[r] = __builtin_amdgcn_readlane(lo, r);
        // (a lane past the count reads the ray's first slot, which is in bounds)
        const uint16_t *sk = b.slot_k + min(ray0 + r, b.n - 1) * (int64_t)b.n_samples;
        ka[r] = sk[(uint32_t)lane < cnt[r] ? lane : 0];
        kb[r] = sk[(uint32_t)lane + kWave < cnt[r] ? lane + kWave : 0];
    }
#pragma unroll
    for (int r = 0; r < RAYS; ++r) {
        if (cnt[r] == 0) continue;
        uint32_t *rr = b.rec_ray + off[r];
        uint16_t *rk = b.rec_k + off[r];
        const uint32_t ray = (uint32_t)(ray0 + r);
        if ((uint32_t)lane < cnt[r]) {
            rr[lane] = ray;
            rk[lane] = ka[r];
        }
        if ((uint32_t)lane + kWave < cnt[r]) {
            rr[lane + kWave] = ray;
            rk[lane + kWave] = kb[r];
        }
        const uint16_t *sk = b.slot_k + (int64_t)ray * b.n_samples;
        for (uint32_t j = 2 * kWave + lane; j < cnt[r]; j += kWave) {
            rr[j] = ray;
            rk[j] = sk[j];
        }
    }
}

template <int RAYS, bool COUNTED> __global__ __launch_bounds__(256) void k_compact(RenderBufs b)
{
    const int64_t wave = (int64_t)blockIdx.x * kRayWaves + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    if constexpr (COUNTED) {
        const int64_t n = min((int64_t)*b.n_active, b.n), stride = (int64_t)gridDim.x * kRayWaves;
        for (int64_t w = wave; w * RAYS < n; w += stride) compact_rays<RAYS>(b, w * RAYS);
    } else {
        if (wave * RAYS < b.n) compact_rays<RAYS>(b, wave * RAYS);
    }
}

// Voxel mode, up to 64 rays ray0, ray0 + stride, .. of one wavefront: the next
// ray's first 64 slots are loaded before this ray's are worked through.
__device__ __forceinline__ void compact_rays_voxel(const GridK &g, const RenderBufs &b, int64_t ray0, int stride,
                                                   int nrays, uint32_t *counts)
{
    const int lane = lane_id();
    const int64_t mine = ray0 + (int64_t)lane * stride;
    uint32_t lc = 0, loff = 0;
    RayInfo linf{};
    float lo[3] = {}, ld[3] = {};
    if (lane < nrays) {
        lc = b.count[mine];
        loff = b.offsets[mine];
        linf = b.info[mine];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            lo[a] = b.rays_o[3 * mine + a];
            ld[a] = b.rays_d[3 * mine + a];
        }
    }
    auto lane_f = [](float v, int l) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l)); };
    auto first_slots = [&](uint64_t todo) -> uint32_t {
        const int r = todo ? __builtin_ctzll(todo) : 0;
        const uint32_t cnt = __builtin_amdgcn_readlane(lc, r);
        const uint16_t *sk = b.slot_k + (ray0 + (int64_t)r * stride) * (int64_t)b.n_samples;
        return sk[(uint32_t)lane < cnt ? lane : 0];
    };
    uint64_t todo = __builtin_amdgcn_ballot_w64(lc != 0);
    uint32_t kn = todo ? first_slots(todo) : 0u;
    while (todo) {
        const int r = __builtin_ctzll(todo);
        todo &= todo - 1;
        uint32_t kc = kn;
        if (todo) kn = first_slots(todo);
        const int64_t ray = ray0 + (int64_t)r * stride;
        const uint32_t cnt = __builtin_amdgcn_readlane(lc, r), off = __builtin_amdgcn_readlane(loff, r);
        const float tn = lane_f(linf.tn, r), delta = lane_f(linf.delta, r);
        const float o[3] = {lane_f(lo[0], r), lane_f(lo[1], r), lane_f(lo[2], r)};
        const float d[3] = {lane_f(ld[0], r), lane_f(ld[1], r), lane_f(ld[2], r)};
        const int64_t slots = ray * (int64_t)b.n_samples;
        for (uint32_t j0 = 0; j0 < cnt; j0 += kWave) {
            const uint32_t j = j0 + lane;
            const bool act = j < cnt;
            uint32_t key = 0xffffffffu;
            if (act) {
                if (j0) kc = b.slot_k[slots + j];
                b.rec_ray[off + j] = (uint32_t)ray;
                b.rec_k[off + j] = (uint16_t)kc;
                if (b.rec_w) {   // the adjoint's
                    b.rec_w[off + j] = b.slot_w[slots + j];
                    b.rec_t[off + j] = b.slot_t[slots + j];
                }
                int i0[3];
                float fr[3], tk;
                sample_voxel(o, d, tn, delta, (int)kc, g, i0, fr, tk);
                key = brick_of(g, i0);
                b.rec_key[off + j] = key;
            }
            const int active = (int)min(cnt - j0, (uint32_t)kWave);
            const uint64_t heads = run_heads(key, act);
            if ((heads >> lane) & 1ull) atomicAdd(&counts[key], (uint32_t)run_length(heads, active));
        }
    }
}

__global__ __launch_bounds__(256) void k_compact_voxel(GridK g, RenderBufs b)
{
    const int64_t ray = (int64_t)blockIdx.x * kRayWaves + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    if (ray < b.n) compact_rays_voxel(g, b, ray, 1, 1, b.brick_off);
}

// Voxel mode with an LDS histogram of the bricks: a block compacts `rays`
// consecutive rays, counting their runs in LDS, and then adds each brick it
// touched to the global count once.  The rays of a block cross largely the
// same bricks, so this takes far fewer device-wide atomics than one per run,
// and neighbouring rays' runs do not queue at the same counter.  With fewer
// rays per block in smaller passes the histogram pays down to about 2000 rays
// (compaction + scatter: 333x257 frame of a 97x113x81 grid 471 -> 44 us,
// 240x180 of 160^3 126 -> 42, 64x64 of 64^3 31 -> 11; 8192 training rays,
// which are not neighbours, 38 -> 36 us); below that it is not measured to.
constexpr int kHistBins = 16384;   // largest brick count of the LDS path (64 KB)
constexpr int64_t kHistMin = 2048;   // fewest rays of the LDS path
// 16 wavefronts per block: the rays' dependent load chains overlap across
// wavefronts (measured on eight 800x800 views with 256 rays per block:
// compaction + sort 6.5 ms with 4 wavefronts per block, 4.9 ms with 8, 4.7 ms
// with 16).  Mean pass of those views, 95 M samples: 488 us, 687 when each ray's
// loads began after the ray before it and the weights were copied too.
constexpr int kHistThreads = 1024;
// Rays per block: 256 where that still gives 512 blocks, else fewer, down to
// one per wavefront; 0 = the per-run global atomics.
static int hist_rays(const RenderBufs &b)
{
    if (b.n_bricks > kHistBins || b.n < kHistMin) return 0;
    int r = 256;
    while (r > kHistThreads / kWave && b.n < (int64_t)r * 512) r >>= 1;
    return r;
}

__global__ __launch_bounds__(kHistThreads) void k_compact_hist(GridK g, RenderBufs b, int rays)
{
    extern __shared__ uint32_t hist[];
    for (int64_t i = threadIdx.x; i < b.n_bricks; i += blockDim.x) hist[i] = 0u;
    __syncthreads();
    const int64_t ray0 = (int64_t)blockIdx.x * rays;
    const int64_t ray1 = ray0 + rays < b.n ? ray0 + rays : b.n;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), stride = kHistThreads / kWave;
    const int mine = (int)((ray1 - ray0) - wave + stride - 1) / stride;   // this wavefront's rays, at most 16
    if (mine > 0) compact_rays_voxel(g, b, ray0 + wave, stride, mine, hist);
    __syncthreads();
    for (int64_t i = threadIdx.x; i < b.n_bricks; i += blockDim.x) {
        const uint32_t c = hist[i];
        if (c) atomicAdd(&b.brick_off[i], c);
    }
}

void launch_compact(const GridK &g, const RenderBufs &b, bool voxel_keys, hipStream_t s)
{
    if (b.n == 0) return;
    auto grid = [&](int64_t per) { return dim3((unsigned)((b.n + per - 1) / per)); };
    if (voxel_keys) {
        const int rays = hist_rays(b);
        if (rays)
            hipLaunchKernelGGL(k_compact_hist, grid(rays), dim3(kHistThreads), b.n_bricks * sizeof(uint32_t), s, g, b,
                               rays);
        else hipLaunchKernelGGL(k_compact_voxel, grid(kRayWaves), dim3(256), 0, s, g, b);
        return;
    }
    // rays per wavefront (of a device-counted pass only few exist: 4, which is near the
    // best for the 20,000 to 200,000 of an 800x800 target's holes)
    const int rays = b.n < 32768 ? 1 : b.n < 262144 || b.n_active ? 4 : 8;
    const dim3 blocks = ray_grid(b, kRayWaves * rays), block(256);
    if (b.n_active) {
        if (rays == 1) hipLaunchKernelGGL((k_compact<1, true>), blocks, block, 0, s, b);
        else hipLaunchKernelGGL((k_compact<4, true>), blocks, block, 0, s, b);
        return;
    }
    if (rays == 1) hipLaunchKernelGGL((k_compact<1, false>), blocks, block, 0, s, b);
    else if (rays == 4) hipLaunchKernelGGL((k_compact<4, false>), blocks, block, 0, s, b);
    else hipLaunchKernelGGL((k_compact<8, false>), blocks, block, 0, s, b);
}

// Bucket scatter: brick_off holds the exclusive scan of brick counts and is
// advanced as a cursor; each run of equal bricks takes one atomic.
__global__ __launch_bounds__(256) void k_brick_scatter(RenderBufs b)
{
    const int lane = lane_id();
    const int64_t ray = (int64_t)blockIdx.x * kRayWaves + (threadIdx.x / kWave);
    if (ray >= b.n) return;
    const uint32_t cnt = b.count[ray];
    if (cnt == 0) return;
    const uint32_t off = b.offsets[ray];
    for (uint32_t j0 = 0; j0 < cnt; j0 += kWave) {
        const uint32_t j = j0 + lane;
        const bool act = j < cnt;
        const uint32_t key = act ? b.rec_key[off + j] : 0xffffffffu;
        const int active = (int)min(cnt - j0, (uint32_t)kWave);
        const uint64_t heads = run_heads(key, act);
        uint32_t base = 0;
        if ((heads >> lane) & 1ull) base = atomicAdd(&b.brick_off[key], (uint32_t)run_length(heads, active));
        // head of my run = highest head at or below my lane
        const uint64_t upto = heads & ((lane == kWave - 1) ? ~0ull : ((2ull << lane) - 1ull));
        const int head = upto ? (63 - __clzll((long long)upto)) : 0;
        const uint32_t hb = __shfl(base, head, kWave);
        if (act) b.perm[hb + (uint32_t)(lane - head)] = off + j;
    }
}

// LDS-histogram scatter over the same blocks of rays, whose
// samples are one contiguous range of records: count the block's samples
// per brick in LDS, reserve each touched brick's share of the global cursor
// with one atomic, then hand out positions from the LDS cursors (one LDS
// atomic per run of equal bricks).  Bound by the latency of the keys' loads: with
// four chunks' keys in flight a pass of 95 M samples takes 305 us, one by one 399.
__global__ __launch_bounds__(kHistThreads) void k_brick_scatter_hist(RenderBufs b, int rays)
{
    extern __shared__ uint32_t hist[];
    const int lane = lane_id(), wave = threadIdx.x / kWave, nwaves = blockDim.x / kWave;
    for (int64_t i = threadIdx.x; i < b.n_bricks; i += blockDim.x) hist[i] = 0u;
    __syncthreads();
    const int64_t ray0 = (int64_t)blockIdx.x * rays;
    const int64_t ray1 = ray0 + rays < b.n ? ray0 + rays : b.n;
    const uint32_t s0 = b.offsets[ray0], s1 = b.offsets[ray1];
    constexpr int kAhead = 4;
    const uint32_t stride = (uint32_t)nwaves * kWave;
    auto load_keys = [&](uint32_t w0, uint32_t key[kAhead]) {
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const uint32_t sidx = w0 + u * stride + lane;
            key[u] = sidx < s1 ? b.rec_key[sidx] : 0xffffffffu;
        }
    };
    for (uint32_t w0 = s0 + (uint32_t)wave * kWave; w0 < s1; w0 += kAhead * stride) {
        uint32_t key[kAhead];
        load_keys(w0, key);
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const uint32_t at = w0 + u * stride;
            if (at >= s1) break;
            const uint64_t heads = run_heads(key[u], at + lane < s1);
            if ((heads >> lane) & 1ull)
                atomicAdd(&hist[key[u]], (uint32_t)run_length(heads, (int)min(s1 - at, (uint32_t)kWave)));
        }
    }
    __syncthreads();
    for (int64_t i = threadIdx.x; i < b.n_bricks; i += blockDim.x) {
        const uint32_t c = hist[i];
        if (c) hist[i] = atomicAdd(&b.brick_off[i], c);
    }
    __syncthreads();
    for (uint32_t w0 = s0 + (uint32_t)wave * kWave; w0 < s1; w0 += kAhead * stride) {
        uint32_t key[kAhead];
        load_keys(w0, key);
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const uint32_t at = w0 + u * stride;
            if (at >= s1) break;
            const bool act = at + lane < s1;
            const uint64_t heads = run_heads(key[u], act);
            uint32_t base = 0;
            if ((heads >> lane) & 1ull)
                base = atomicAdd(&hist[key[u]], (uint32_t)run_length(heads, (int)min(s1 - at, (uint32_t)kWave)));
            const uint64_t upto = heads & ((lane == kWave - 1) ? ~0ull : ((2ull << lane) - 1ull));
            const int head = upto ? (63 - __clzll((long long)upto)) : 0;
            const uint32_t hb = __shfl(base, head, kWave);
            if (act) b.perm[hb + (uint32_t)(lane - head)] = at + lane;
        }
    }
}

void launch_brick_scatter(const RenderBufs &b, hipStream_t s)
{
    if (b.n == 0) return;
    const int rays = hist_rays(b);
    if (rays) {
        const unsigned blocks = (unsigned)((b.n + rays - 1) / rays);
        hipLaunchKernelGGL(k_brick_scatter_hist, dim3(blocks), dim3(kHistThreads), b.n_bricks * sizeof(uint32_t), s, b,
                           rays);
        return;
    }
    const unsigned blocks = (unsigned)((b.n + kRayWaves - 1) / kRayWaves);
    hipLaunchKernelGGL(k_brick_scatter, dim3(blocks), dim3(256), 0, s, b);
}

__global__ void k_fill_u32(uint32_t *p, uint32_t v, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}
__global__ void k_fill_u64(uint64_t *p, uint64_t v, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}
static unsigned fill_blocks(int64_t n)
{
    int64_t b = (n + 255) / 256;
    return (unsigned)(b < 1 ? 1 : (b > 8192 ? 8192 : b));
}
void launch_fill_u32(uint32_t *p, uint32_t v, int64_t n, hipStream_t s)
{
    if (n > 0) hipLaunchKernelGGL(k_fill_u32, dim3(fill_blocks(n)), dim3(256), 0, s, p, v, n);
}
void launch_fill_u64(uint64_t *p, uint64_t v, int64_t n, hipStream_t s)
{
    if (n > 0) hipLaunchKernelGGL(k_fill_u64, dim3(fill_blocks(n)), dim3(256), 0, s, p, v, n);
}
__global__ void k_fill_u8(uint8_t *p, uint8_t v, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}
// Segments per brick (ceil(count / kTileSeg)) into seg_off, then their
// exclusive scan: brick k owns segments seg_off[k] .. seg_off[k+1]-1.
__global__ void k_brick_segments(RenderBufs b, uint32_t seg)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= b.n_bricks) return;
    const uint32_t start = k == 0 ? 0u : b.brick_off[k - 1], end = b.brick_off[k];
    b.seg_off[k] = (end - start + seg - 1u) / seg;
}

// Brick of every segment: brick k writes its own segments' entries.
__global__ void k_segment_bricks(RenderBufs b)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= b.n_bricks) return;
    for (uint32_t q = b.seg_off[k]; q < b.seg_off[k + 1]; ++q) b.seg_brick[q] = (uint32_t)k;
}

void launch_brick_segments(const RenderBufs &b, int seg, bool table, hipStream_t s)
{
    if (b.n_bricks > 0)
        hipLaunchKernelGGL(k_brick_segments, dim3((unsigned)((b.n_bricks + 255) / 256)), dim3(256), 0, s, b,
                           (uint32_t)seg);
    launch_exclusive_scan(b.seg_off, b.seg_off, b.brick_tmp, b.n_bricks, s);   // also writes the total
    if (table && b.seg_brick && seg == kTileSeg && b.n_bricks > 0)
        hipLaunchKernelGGL(k_segment_bricks, dim3((unsigned)((b.n_bricks + 255) / 256)), dim3(256), 0, s, b);
}

void launch_fill_u8(uint8_t *p, uint8_t v, int64_t n, hipStream_t s)
{
    if (n > 0) hipLaunchKernelGGL(k_fill_u8, dim3(fill_blocks(n)), dim3(256), 0, s, p, v, n);
}

// Per-ray accumulation: rgb = sum_k w_k c_k + T_stop bg, depth_t,
// acc = 1 - T_stop; frame mode converts to z-depth with the void rule.  One
// wavefront per ray: lanes read consecutive live samples (coalesced) and a
// butterfly sum combines them in a fixed order, so the result does not
// depend on the order in which the MLP stage produced the colours.
// Per-ray accumulation, four rays per wavefront (16 lanes each): lane l of a
// ray's group sums w_k c_k over its live samples l, l + 16, l + 32, ... in
// order, then a 16-lane butterfly adds the lanes' partial sums (a fixed
// order, so the result is deterministic and the same in every sample order
// of the MLP stage).  The four rays' loads go out together, which is what a
// stage bound by the latency of its dependent loads needs (measured on eight
// 800x800 views: 1.55 ms with 16 lanes per ray, 1.82 with 8, 1.64 with 32,
// 2.37 with a wavefront per ray), and four samples of each lane with them (mean
// pass of those views, 95 M samples: 349 -> 325 us, 4.7 TB/s of the samples' 16
// bytes).
constexpr int kReduceLanes = 16;
constexpr int kReduceRays = kRayWaves * (kWave / kReduceLanes);   // rays per 256-thread block

// Sum over the 16 lanes of a DPP row, every lane getting it: rotations of
// the row by 8, 4, 2 and 1 lanes (DPP lane moves, no LDS round trips).
__device__ __forceinline__ float group16_sum(float v)
{
    static_assert(kReduceLanes == 16, "one ray per DPP row");
    v = dpp_add<0x128, 0xf, false>(v);   // row_ror:8
    v = dpp_add<0x124, 0xf, false>(v);   // row_ror:4
    v = dpp_add<0x122, 0xf, false>(v);   // row_ror:2
    v = dpp_add<0x121, 0xf, false>(v);   // row_ror:1
    return v;
}

__device__ __forceinline__ void reduce_ray(const RenderBufs &b, const OptsK &op, float *rgb, float *depth, float *acc,
                                           const int32_t *out_map, const cic_camera &cam, int frame, int64_t ray, int sub)
{
    const uint32_t cnt = b.count[ray], off = b.offsets[ray];
    float r = 0.f, gg = 0.f, bb = 0.f;
    const float *ws = b.slot_w + ray * (int64_t)b.n_samples;
    for (uint32_t j0 = (uint32_t)sub; j0 < cnt; j0 += 4 * kReduceLanes) {
        // four samples' loads in flight (one past the count re-reads the first and adds nothing)
        float w[4], c[4][3];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t j = j0 + u * kReduceLanes < cnt ? j0 + u * kReduceLanes : j0;
            const float *p = b.rec_c + 3 * ((int64_t)off + j);
            w[u] = ws[j];
#pragma unroll
            for (int ch = 0; ch < 3; ++ch) c[u][ch] = p[ch];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const bool in = j0 + u * kReduceLanes < cnt;
            r = in ? fmaf(w[u], c[u][0], r) : r;
            gg = in ? fmaf(w[u], c[u][1], gg) : gg;
            bb = in ? fmaf(w[u], c[u][2], bb) : bb;
        }
    }
    r = group16_sum(r);
    gg = group16_sum(gg);
    bb = group16_sum(bb);
    if (sub != 0) return;
    const RayInfo inf = b.info[ray];
    const float ts = inf.t_stop;
    const int64_t out = out_map ? (int64_t)out_map[ray] : ray;
    rgb[3 * out + 0] = fmaf(ts, op.bg[0], r);
    rgb[3 * out + 1] = fmaf(ts, op.bg[1], gg);
    rgb[3 * out + 2] = fmaf(ts, op.bg[2], bb);
    const float a = 1.0f - ts;
    if (acc) acc[out] = a;
    if (frame) {
        float dz = INFINITY;
        if (a >= op.void_acc) {
            const float *d = b.rays_d + 3 * ray;
            const float cosang = fmaf(d[0], cam.c2w[2], fmaf(d[1], cam.c2w[6], d[2] * cam.c2w[10]));
            dz = inf.depth_t / a * cosang;
        }
        depth[out] = dz;
    } else {
        depth[out] = inf.depth_t;
    }
}

__global__ __launch_bounds__(256) void k_reduce(RenderBufs b, OptsK op, float *rgb, float *depth, float *acc,
                                                const int32_t *out_map, cic_camera cam, int frame,
                                                unsigned long long *n_eval, int64_t *n_masked)
{
    const int sub = (int)(threadIdx.x % kReduceLanes);
    const uint32_t n_act = b.n_active ? min(*b.n_active, (uint32_t)b.n) : (uint32_t)b.n;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        if (n_eval) atomicAdd(n_eval, (unsigned long long)b.offsets[b.n]);
        if (n_masked) *n_masked = (int64_t)n_act;
    }
    for (int64_t ray = (int64_t)blockIdx.x * kReduceRays + (threadIdx.x / kReduceLanes); ray < (int64_t)n_act;
         ray += (int64_t)gridDim.x * kReduceRays)
        reduce_ray(b, op, rgb, depth, acc, out_map, cam, frame, ray, sub);
}

void launch_reduce(const RenderBufs &b, const OptsK &o, float *rgb, float *depth, float *acc,
                   const int32_t *out_map, const cic_camera *frame_cam, int64_t *n_eval, int64_t *n_masked,
                   hipStream_t s)
{
    cic_camera cam{};
    if (frame_cam) cam = *frame_cam;
    hipLaunchKernelGGL(k_reduce, ray_grid(b, kReduceRays), dim3(256), 0, s, b, o, rgb, depth, acc,
                       out_map, cam, frame_cam ? 1 : 0, (unsigned long long *)n_eval, n_masked);
}

// Pixel rays; pixel index from pix (int64), pix32 (int32) or identity.
__global__ __launch_bounds__(256) void k_generate_rays(cic_camera cam, int64_t n, int64_t base, const int64_t *pix,
                                                       const int32_t *pix32, const uint32_t *n_active, float *o,
                                                       float *d)
{
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= n) return;
    if (n_active && (uint64_t)r >= *n_active) return;
    const int64_t p = pix ? pix[r] : (pix32 ? (int64_t)pix32[r] : base + r);
    float oo[3], dd[3];
    pixel_ray(cam, (int)(p % cam.width), (int)(p / cam.width), oo, dd);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        o[3 * r + a] = oo[a];
        d[3 * r + a] = dd[a];
    }
}

void launch_generate_rays(const cic_camera &cam, int64_t n, int64_t base, const int64_t *pix, const int32_t *pix32,
                          const uint32_t *n_active, float *o, float *d, hipStream_t s)
{
    if (n == 0) return;
    hipLaunchKernelGGL(k_generate_rays, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, cam, n, base, pix, pix32,
                       n_active, o, d);
}

// Occupancy: a voxel is occupied iff any vertex has raw + shift > thr
// (thr = log(expm1(occ_sigma)) rounded to float32 on the host).  One
// wavefront tests the 64 vertices from z0 in the vertex rows y and y + 1 of
// kOccX + 1 consecutive x (all its loads go out together), as one 64-bit mask
// per x; the voxels' bytes are ORs of neighbouring masks and their shifts.  A
// row's vertices are loaded twice rather than eight times, coalesced, with no
// division per voxel.  Bound by the read of the density (160^3 float32: 16.4
// MB and 4.0 MB of bytes written: 8.3 us, before 18.7; float16 10.2 and 21.4).
constexpr int kOccX = 8;           // voxels per wavefront along x (2: 12.0 us, 4: 9.2, 8: 8.3)
constexpr int kOccZ = kWave - 1;   // and along z

template <typename T>
__global__ __launch_bounds__(256) void k_build_occupancy(GridK g, float thr, uint8_t *occ, uint32_t nx, uint32_t nz)
{
    const uint32_t c1 = g.r1 - 1, c2 = g.r2 - 1;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(blockIdx.x * 4u + threadIdx.x / kWave);
    const uint32_t xg = wave / (c1 * nz), y = (wave / nz) % c1, z0 = (wave % nz) * kOccZ;
    if (xg >= nx) return;
    const int lane = lane_id();
    const uint32_t z = min(z0 + (uint32_t)lane, (uint32_t)g.r2 - 1u), x0 = xg * kOccX;
    const T *dens = (const T *)g.density;
    float v[kOccX + 1][2];
#pragma unroll
    for (int i = 0; i <= kOccX; ++i) {
        const T *row = dens + ((int64_t)min(x0 + i, (uint32_t)g.r0 - 1u) * g.r1 + y) * g.r2;
        v[i][0] = ldv(row, z);
        v[i][1] = ldv(row, z + (uint32_t)g.r2);
    }
    uint64_t m[kOccX + 1];
#pragma unroll
    for (int i = 0; i <= kOccX; ++i)
        m[i] = __builtin_amdgcn_ballot_w64(v[i][0] + g.shift > thr || v[i][1] + g.shift > thr);
    if (lane >= kOccZ || z0 + (uint32_t)lane >= c2) return;
#pragma unroll
    for (int i = 0; i < kOccX; ++i) {
        if (x0 + i >= (uint32_t)g.r0 - 1u) break;
        const uint64_t any = m[i] | m[i + 1];
        occ[((int64_t)(x0 + i) * c1 + y) * c2 + z] = (uint8_t)(((any | any >> 1) >> lane) & 1u);
    }
}

template <typename T>
void launch_build_occupancy(const GridK &g, float thr, uint8_t *occ, hipStream_t s)
{
    const uint32_t nx = (uint32_t)(g.r0 - 1 + kOccX - 1) / kOccX, nz = (uint32_t)(g.r2 - 1 + kOccZ - 1) / kOccZ;
    const uint64_t waves = (uint64_t)nx * (uint64_t)(g.r1 - 1) * nz;   // at most 2^22
    hipLaunchKernelGGL(k_build_occupancy<T>, dim3((unsigned)((waves + 3) / 4)), dim3(256), 0, s, g, thr, occ, nx, nz);
}
template void launch_build_occupancy<float>(const GridK &, float, uint8_t *, hipStream_t);
template void launch_build_occupancy<__half>(const GridK &, float, uint8_t *, hipStream_t);

}  // namespace cic
