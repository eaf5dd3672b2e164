// Feature Gathering + Feature Computation (Sec. II-B) for the compacted live
// samples: trilinear gather of the 12 feature channels, the view-direction
// encoding, and the 39 -> 128 -> 128 -> 3 MLP on MFMA, for float32 compute.
//
// Arithmetic.  The matrix cores run float16 products 16 times as fast as
// float32 ones, so the hidden layers split both operands into two float16
// parts, v = hi + lo / 2^11 (22 significand bits and a sign between them),
// and sum three products, hi hi, hi lo and lo hi, in float32.  The remainders
// are kept times 2^11, so they are normal float16 values wherever the first
// part is one; weights are scaled by powers of two to use float16's range,
// and a sample whose features or activations leave it (65504, after the
// scaling of layer 0) is computed again with float32 products.  The low products
// have their own accumulators, so the high ones are rounded 8 times over a
// 128-long sum where a float32 chain rounds 128 times.  Colour error against
// 64 bits, rms over 300,000 single-sample rays: 2.80e-8, and 2.90e-8 for the
// float32 MFMA chain that this replaced; features x 30: 4.73e-8 and 4.82e-8;
// W0 x 30: 9.8e-8 and 1.16e-7; W1 x 8: 5.8e-8 and 6.6e-8 (three BF16 parts
// and six products, the exact split, were less exact, 3.06e-8, because one
// accumulator takes 48 roundings, and 1.4 times as slow).
//
// Bound.  Matrix power: with the matrix cores 62% busy the card lowers its
// clock to 1.8 GHz (2.37 GHz under float32 MFMA at 85%), which is the busy
// rate times clock that a library BF16 product reaches here too (1.2
// PFLOP/s).  MLP stage of an 800x800 frame with 36 M live samples: 9.9 -> 4.0 ms.
//
// Layout.  The MLP runs transposed, H^T = W X^T, so that samples sit on the
// MFMA's N axis (32 samples per wavefront batch): the result tile of one
// layer (lane l holds rows 8 (r / 4) + 4 (l / 32) + r % 4 of sample l % 32) is
// the B operand of the next layer once the reduction index is permuted the
// same way in the weights.  Activations never leave registers; weights are
// staged once per workgroup in LDS in per-lane fragment order, so every A
// operand is one contiguous, conflict-free ds_read_b128.  32x32 tiles rather
// than 16x16: each fragment serves 32 samples (LDS reads are the next limit)
// and a sample's cell is located by two lanes instead of four.  The output
// layer runs on 4x4x1 float32 MFMA, whose B operand is the lane's own
// activation.
//
// Schedule.  Persistent: one 8-wavefront workgroup per CU (two per SIMD at
// 232 VGPRs; 12 wavefronts spill, 8.4 against 4.7 ms per frame).  Within a
// batch the vector work (splitting the activations, the output layer, and
// the next batch's records, gathers and interpolation) sits between the
// layer-1 MFMAs: 3.5% faster than the same order left to the compiler.
#include "mlp_common.h"

namespace cic {

constexpr int kFwdWaves = 8;    // wavefronts of the CU's one workgroup
constexpr int kFwdBatch = 32;   // samples per wavefront batch

// LDS in 16-byte fragments, then floats
constexpr int kXW1 = 0;                          // [part 2][t 4][c 8][lane 64]
constexpr int kXW0 = kXW1 + 2 * 4 * 8 * 64;      // [t 4][s 3][lane 64]
constexpr int kXFrags = kXW0 + 4 * 3 * 64;
constexpr int kXB1 = 0, kXW2 = 128;              // [128]; [t 4][i 4][h 2][ch 4][r 4]
constexpr int kXB2 = kXW2 + 512, kXFloats = kXB2 + 4;
constexpr int kXLdsBytes = std::max(kXFrags * 16 + kXFloats * 4, F32Lds::kSize * 4);
constexpr float kLoScale = 2048.f;               // the low parts are kept times 2^11

// v0, v1 into a float16 and a second float16 that holds the remainder times
// 2^11 (the remainder is exact in float32; times 2^11 it is a normal float16
// wherever the first part is)
__device__ __forceinline__ void split2(float v0, float v1, uint32_t &hi, uint32_t &lo)
{
    h2_t a, b;
    a[0] = (_Float16)v0;
    a[1] = (_Float16)v1;
    hi = __builtin_bit_cast(uint32_t, a);
    asm("" : "+v"(hi));   // one packed conversion, not two more single ones for the remainders
    a = __builtin_bit_cast(h2_t, hi);
    b[0] = (_Float16)fmaf((float)a[0], -kLoScale, v0 * kLoScale);
    b[1] = (_Float16)fmaf((float)a[1], -kLoScale, v1 * kLoScale);
    lo = __builtin_bit_cast(uint32_t, b);
}

// 2^k, k in [-100, 100], that puts a weight block's largest magnitude `top`
// into [2^to, 2^(to + 1)) (1 where the block is zero)
__device__ __forceinline__ int block_exp(float top, int to)
{
    return top > 0.f ? min(max(to + 127 - (int)(__float_as_uint(top) >> 23), -100), 100) : 0;
}

// Largest of a value over the block (red: one float per wavefront and block
// maximum; a barrier before its next use is the caller's).
__device__ __forceinline__ float block_max(float v, float *red)
{
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) v = fmaxf(v, __shfl_xor(v, off, kWave));
    if (lane_id() == 0) red[threadIdx.x / kWave] = v;
    __syncthreads();
    for (int k = 0; k < (int)blockDim.x / kWave; ++k) v = fmaxf(v, red[k]);
    return v;
}

// Weights into LDS in fragment order.  W0's feature columns are scaled by the
// power of two 2^e0 that puts their largest entry in [1, 2) (the per-ray
// direction terms with them), W1 by the one that puts its largest entry in
// [2^14, 2^15) before the split (so both parts use float16's range), b1 by
// both; W2 by the inverse of both, which the ReLUs let through exactly.
// Returns e0.  Every load goes out before the first barrier (a SpaRW target's
// MLP stage 215 -> 209 us against loading between the barriers).
__device__ int stage_weights_split(const cic_mlp &m, float *lds)
{
    h8_t *w1 = (h8_t *)lds + kXW1;
    h8_t *w0 = (h8_t *)lds + kXW0;
    float *fl = lds + kXFrags * 4;
    constexpr int kT = kFwdWaves * 64, kN = 4 * 8 * 64, kIt = kN / kT, kN0 = 4 * 3 * 64, kIt0 = (kN0 + kT - 1) / kT;
    static_assert(kN % kT == 0 && kT == 512, "one W2 entry and the W1 fragments per thread");
    const int tid = threadIdx.x;
    f4_t w[kIt][2];
    float v0[kIt0][8], top1 = 0.f, top0 = 0.f;
#pragma unroll
    for (int k = 0; k < kIt; ++k) {
        const int i = tid + k * kT, l = i & 63, c = (i >> 6) & 7, t = i >> 9;
        const float *src = m.w1 + (32 * t + (l & 31)) * 128;
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e) w[k][u][e] = src[x_hid(c, l >> 5, 4 * u) + e];
    }
#pragma unroll
    for (int k = 0; k < kIt0; ++k) {
        const int i = min(tid + k * kT, kN0 - 1), l = i & 63, s = (i >> 6) % 3, t = i / 192;
#pragma unroll
        for (int e = 0; e < 8; ++e) v0[k][e] = m.w0[(32 * t + (l & 31)) * 39 + 6 * (l >> 5) + (8 * s + e) % 6];
    }
    const int ch2 = (tid >> 2) & 3, h2 = (tid >> 4) & 1;
    const int row2 = 32 * (tid >> 7) + 8 * ((tid >> 5) & 3) + 4 * h2 + (tid & 3);
    const float v2 = m.w2[min(ch2, 2) * 128 + row2], vb1 = m.b1[tid & 127], vb2 = m.b2[min(tid & 3, 2)];
#pragma unroll
    for (int k = 0; k < kIt; ++k)
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e) top1 = fmaxf(top1, fabsf(w[k][u][e]));
#pragma unroll
    for (int k = 0; k < kIt0; ++k)
#pragma unroll
        for (int e = 0; e < 8; ++e) top0 = fmaxf(top0, fabsf(v0[k][e]));
    // (the two reductions' floats lie where the fragments come later)
    top0 = block_max(top0, fl);
    top1 = block_max(top1, fl + 16);
    __syncthreads();
    const int e0 = block_exp(top0, 0), e1 = block_exp(top1, 14);
    const float s0 = ldexpf(1.f, e0), s1 = ldexpf(1.f, e1);
#pragma unroll
    for (int k = 0; k < kIt0; ++k) {
        const int i = tid + k * kT, s = (i >> 6) % 3;
        h8_t v;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            // products: high x high, high / 2^11 x (low times 2^11), low x high
            const int p = (8 * s + e) / 6;
            const float a = v0[k][e] * s0;
            const _Float16 hi = (_Float16)a;
            v[e] = p == 0 ? hi : p == 1 ? (_Float16)((float)hi * (1.f / kLoScale)) : p == 2 ? (_Float16)(a - (float)hi)
                                                                                           : (_Float16)0.f;
        }
        if (i < kN0) w0[i] = v;
    }
#pragma unroll
    for (int k = 0; k < kIt; ++k) {
        u4_t hi, lo;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            uint32_t a, b;
            split2(w[k][e >> 1][2 * (e & 1)] * s1, w[k][e >> 1][2 * (e & 1) + 1] * s1, a, b);
            hi[e] = a;
            lo[e] = b;
        }
        w1[tid + k * kT] = __builtin_bit_cast(h8_t, hi);
        w1[kN + tid + k * kT] = __builtin_bit_cast(h8_t, lo);
    }
    fl[kXW2 + tid] = ch2 < 3 ? ldexpf(v2, -(e0 + e1)) : 0.f;
    if (tid < 128) fl[kXB1 + tid] = ldexpf(vb1, e0 + e1);
    if (tid < 4) fl[kXB2 + tid] = tid < 3 ? vb2 : 0.f;
    return e0;
}

// Per-ray direction term of layer 0: z0[ray][o] = 2^e0 (b0[o] + sum_i
// W0[o][12+i] pe_i) over the 27 direction inputs (d, sin, cos), once per ray
// with live samples (float32, scaled as the MLP scales W0; used in either
// order).  A block stages the inputs of RAYS rays in LDS (one sincosf per
// argument gives both its sine and cosine input), and each of its 128 threads
// then forms output o for every ray with its 27 weights held in registers.
// The weight rows (whose first 12 entries give e0) and the rays are loaded
// together, before the first barrier.  64 rays per block amortise the weight
// reads in large passes; small ones, and the holes of a warped frame, take 16,
// so that the launch spreads over the chip (4096 rays: 19.4 -> 7.3 us; 85,581: 16 per block 22.7, 64 27.3;
// 640,000: 110 and 90).
template <int RAYS, bool COUNTED>
__global__ __launch_bounds__(128) void k_ray_embed(cic_mlp m, RenderBufs b, float *z0)
{
    __shared__ __attribute__((aligned(16))) float pe[RAYS][28];
    __shared__ uint32_t live[RAYS];
    __shared__ float red[2];
    const int o = threadIdx.x;
    // (a device-counted pass, the holes of a warped frame, has rays up to its count)
    const int64_t n = COUNTED ? min((int64_t)*b.n_active, b.n) : b.n;
    if ((int64_t)blockIdx.x * RAYS >= n) return;
    float w[39];
#pragma unroll
    for (int i = 0; i < 39; ++i) w[i] = m.w0[o * 39 + i];
    const float bias = m.b0[o];
    int e0 = 0;
    const int64_t first = (int64_t)blockIdx.x * RAYS;
    for (int64_t base = first; base < n; base += (int64_t)gridDim.x * RAYS) {
        if (base != first) __syncthreads();   // the rays before are done with
        for (int r = threadIdx.x; r < RAYS; r += 128) live[r] = base + r < n ? b.count[base + r] : 0u;
        // entries 0..2: the direction; argument k = 4c + octave (k < 12): sine at
        // 3 + k, cosine at 15 + k (also for rays without live samples: their
        // entries are not used)
        for (int e = threadIdx.x; e < RAYS * 15; e += 128) {
            const int r = e / 15, i = e % 15;
            if (base + r >= n) continue;
            const float *d = b.rays_d + 3 * (base + r);
            if (i < 3) {
                pe[r][i] = d[i];
            } else {
                const int k = i - 3, c = k >> 2, oc = k & 3;
                float sn, cs;
                sincosf(ldexpf(d[c], oc), &sn, &cs);
                pe[r][3 + k] = sn;
                pe[r][15 + k] = cs;
            }
        }
        if (base == first) {
            float top = 0.f;
#pragma unroll
            for (int i = 0; i < 12; ++i) top = fmaxf(top, fabsf(w[i]));
            e0 = block_exp(block_max(top, red), 0);   // its barrier also covers pe and live
        } else {
            __syncthreads();
        }
        for (int r = 0; r < RAYS; ++r) {
            if (!live[r]) continue;
            float acc = bias;
#pragma unroll
            for (int i = 0; i < 27; ++i) acc = fmaf(w[12 + i], pe[r][i], acc);
            z0[(base + r) * 128 + o] = ldexpf(acc, e0);
        }
        if constexpr (!COUNTED) break;   // one group per block
    }
}

template <int RAYS, bool COUNTED>
static void launch_embed(const cic_mlp &m, const RenderBufs &b, hipStream_t s)
{
    hipLaunchKernelGGL((k_ray_embed<RAYS, COUNTED>), ray_grid(b, RAYS), dim3(128), 0, s, m, b, b.z0);
}

void launch_ray_embed(const cic_mlp &m, const RenderBufs &b, hipStream_t s)
{
    if (b.n == 0 || m.compute != CIC_F32) return;
    if (b.n_active) launch_embed<16, true>(m, b, s);
    else if (b.n < 131072) launch_embed<16, false>(m, b, s);
    else launch_embed<64, false>(m, b, s);
}

// float32 MFMA for the samples whose features or activations leave the range of
// the split: 16 samples per step of a wavefront, 16x16x4 products as in the
// adjoint's recomputed forward, the weights staged anew over the split's.
// Bound by the float32 products: a call of 1.6 M samples takes 0.37 ms, 0.94 when
// all of them come here (13.0 with a wavefront per sample on the vector ALUs,
// which read W1 from memory for each).
template <typename T, bool HASH>
__device__ __forceinline__ void colours_f32(const GridK &g, const RenderBufs &b, const float *lds, uint32_t rec,
                                            bool write, int e0)
{
    typedef F32Lds L;
    const int lane = lane_id(), q = lane >> 4;
    const f2_t *w0f = (const f2_t *)(lds + L::kW0);
    const f4_t *w2l = (const f4_t *)(lds + L::kW2);
    const float *w1f = lds + L::w1(0, lane);   // (block k at + k * kW1Block floats)
    SampleRay r;
    load_sample_ray(b, b.rec_ray[rec], b.rec_k[rec], r);
    float x[3];
    {
        Gather<T, HASH> gt;
        float xp[3], f[6];
        sample_position(r, xp);
        gt.issue(g, xp, q >> 1);
#pragma unroll
        for (int k = 0; k < 6; ++k) f[k] = gt.feature(k);
#pragma unroll
        for (int c = 0; c < 3; ++c) x[c] = q & 1 ? f[3 + c] : f[c];
    }
    f4_t h1[8], h2[8];
    const float *zr = b.z0 + (int64_t)r.ray * 128 + 4 * q;
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        const f4_t z = *(const f4_t *)(zr + 16 * t);
#pragma unroll
        for (int e = 0; e < 4; ++e) h1[t][e] = ldexpf(z[e], -e0);
        h2[t] = *(const f4_t *)(lds + L::kB1 + 16 * t + 4 * q);
    }
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int t = 0; t < 8; ++t)
            h1[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(w0f[(t * 5 + (c >> 1)) * 64 + lane][c & 1], x[c], h1[t], 0, 0, 0);
#pragma unroll
    for (int c4 = 0; c4 < 8; ++c4) {
#pragma unroll
        for (int tg = 0; tg < 2; ++tg) {
            f4_t a[4];
#pragma unroll
            for (int tt = 0; tt < 4; ++tt) a[tt] = *(const f4_t *)(w1f + ((4 * tg + tt) * 8 + c4) * L::kW1Block);
#pragma unroll
            for (int rr = 0; rr < 4; ++rr) {
                const float h = relu_bits(h1[c4][rr]);
#pragma unroll
                for (int tt = 0; tt < 4; ++tt)
                    h2[4 * tg + tt] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[tt][rr], h, h2[4 * tg + tt], 0, 0, 0);
            }
        }
    }
    float p[3] = {0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 8; ++t)
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) {
            const f4_t w = w2l[(q * 3 + ch) * 8 + t];
#pragma unroll
            for (int e = 0; e < 4; ++e) p[ch] = fmaf(w[e], relu_bits(h2[t][e]), p[ch]);
        }
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) {
        p[ch] += __shfl_xor(p[ch], 16, kWave);
        p[ch] += __shfl_xor(p[ch], 32, kWave);
    }
    if (write && q < 3) b.rec_c[3 * (int64_t)rec + q] = sigmoid_hw(pick3(q, p[0], p[1], p[2]) + lds[L::kB2 + q]);
}

constexpr uint32_t kRedo = 0x7fc0c0deu;   // a NaN that marks a colour to be redone

template <typename T, bool HASH>
__global__ __launch_bounds__(kFwdWaves * 64) __attribute__((amdgpu_waves_per_eu(kFwdWaves / 4, kFwdWaves / 4))) void
k_mlp_fwd_f32(GridK g, cic_mlp m, RenderBufs b, int voxel)
{
    extern __shared__ __attribute__((aligned(16))) float lds[];
    __shared__ uint32_t claimed;
    const int e0 = stage_weights_split(m, lds);
    if (threadIdx.x == 0) claimed = kFwdWaves;
    __syncthreads();

    const int lane = lane_id(), h = lane >> 5, j = lane & 31;
    const int wave = threadIdx.x / 64;
    const uint32_t total = b.offsets[b.n];
    const BatchRange br = xcd_batches(((int64_t)total + kFwdBatch - 1) / kFwdBatch, kFwdWaves, 0);
    // The workgroup's k-th batch; its wavefronts claim them one by one (two
    // wavefronts of a SIMD do not share its issue slots evenly: with fixed
    // shares the favoured one ran out of batches early and left the other to
    // run alone for the last sixth of the kernel).
    const uint32_t bfirst = (uint32_t)br.first, bstride = (uint32_t)br.stride;
    const uint32_t bcount = br.end > br.first ? (uint32_t)(br.end - br.first) : 0u;   // relative to bfirst
    auto batch_of = [&](uint32_t k) -> uint32_t { return (k / kFwdWaves) * bstride + k % kFwdWaves; };
    // Record of this lane's sample of batch bt (a lane past the last sample
    // works on sample 0: in-bounds inputs, no branches around the loads; its
    // colour is not stored).
    auto record_of = [&](uint32_t bt) -> uint32_t {
        const uint32_t s = (bfirst + bt) * kFwdBatch + j;
        const uint32_t sv = bt < bcount && s < total ? s : 0;
        return voxel ? b.perm[sv] : sv;
    };
    const float *fl = lds + kXFrags * 4;
    const h8_t *w0f = (const h8_t *)lds + kXW0 + lane;
    const h8_t *w1f = (const h8_t *)lds + kXW1 + lane;

    bool redo = false;
    uint32_t bt = batch_of(wave), nbt = 0;
    if (bt < bcount) {
        uint32_t crec = record_of(bt), nrec = 0, nray = 0;
        int nk = 0;
        SampleRay cur;
        load_sample_ray(b, b.rec_ray[crec], b.rec_k[crec], cur);
        Gather<T, HASH> gt;
        {
            float xp[3];
            sample_position(cur, xp);
            gt.issue(g, xp, h);
        }
        // the features and, once split, their parts: pair k in xhi[k] and xlo[k]
        float x[6];
        uint32_t xhi[3], xlo[3];
        bool bad;
        auto split_features = [&]() {
            const float lo3 = fabsf(x[0]) + fabsf(x[1]) + fabsf(x[2]), hi3 = fabsf(x[3]) + fabsf(x[4]) + fabsf(x[5]);
            bad = !(lo3 + hi3 < 65504.f);
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                split2(x[2 * k], x[2 * k + 1], xhi[k], xlo[k]);
                // (keeps the interpolation and the split here, among the MFMAs,
                // and not moved down to their use)
                asm volatile("" : "+v"(xhi[k]), "+v"(xlo[k]));
            }
        };
#pragma unroll
        for (int k = 0; k < 6; ++k) x[k] = gt.feature(k);
        split_features();

        f16_t acc0[4];         // layer 0
        f16_t acch[2], accl[2];   // layer 1, one 32-row tile and the one before it: high products, low ones times 2^11
        h8_t hb[2][8];         // the first activations' parts
        f4_t out[2];           // the output layer's sums: channels 0..2 in rows 0..2
        // layer 0 on top of the per-ray direction term (every record's ray has
        // live samples, so its row is written); word w of the 3 x 4 input words is
        // feature pair w % 3 of product w / 3 (the weights' staging lists them)
        auto load_z0 = [&]() {
            const float *zr = b.z0 + (int64_t)cur.ray * 128 + 4 * h;
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const f4_t z = *(const f4_t *)(zr + 32 * t + 8 * i);
#pragma unroll
                    for (int r = 0; r < 4; ++r) acc0[t][4 * i + r] = z[r];
                }
        };
        auto layer0_step = [&](int s) {
            u4_t v;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int w = 4 * s + e;
                v[e] = w / 3 == 3 ? 0u : w / 3 == 1 ? xlo[w % 3] : xhi[w % 3];
            }
            const h8_t xin = __builtin_bit_cast(h8_t, v);
#pragma unroll
            for (int t = 0; t < 4; ++t)
                acc0[t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(w0f[(t * 3 + s) * 64], xin, acc0[t], 0, 0, 0);
        };
        // ReLU and split of the 16 units of chunk c
        auto split_chunk = [&](int c) {
            u4_t hi, lo;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                uint32_t u, v;
                const int r = 8 * (c & 1) + 2 * e;
                split2(relu_bits(acc0[c >> 1][r]), relu_bits(acc0[c >> 1][r + 1]), u, v);
                hi[e] = u;
                lo[e] = v;
            }
            hb[0][c] = __builtin_bit_cast(h8_t, hi);
            hb[1][c] = __builtin_bit_cast(h8_t, lo);
        };
        // 4 of tile t's 16 rows per lane into the output layer: a 4x4x1 MFMA adds
        // W2's entries of one row (lane l supplies channel l % 4) times the lane's
        // own activation, in place of three multiply-adds and three times the
        // weight reads
        auto output_rows = [&](int t, int i) {
            const f4_t w = *(const f4_t *)(fl + kXW2 + ((4 * t + i) * 2 + h) * 16 + (lane & 3) * 4);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float hv = relu_bits(fmaf(accl[t & 1][4 * i + r], 1.f / kLoScale, acch[t & 1][4 * i + r]));
                out[r & 1] = __builtin_amdgcn_mfma_f32_4x4x1f32(w[r], hv, out[r & 1], 0, 0, 0);
            }
        };
        auto finish = [&](uint32_t bt_, uint32_t rec, bool bad_) {
            const f4_t b2 = *(const f4_t *)(fl + kXB2);
            float p[3];
#pragma unroll
            for (int ch = 0; ch < 3; ++ch) {
                p[ch] = out[0][ch] + out[1][ch];
                p[ch] += __shfl_xor(p[ch], 32, kWave);
                p[ch] += b2[ch];
            }
            const bool valid = (bfirst + bt_) * kFwdBatch + j < total;
            bad_ = bad_ || !(fabsf(p[0]) + fabsf(p[1]) + fabsf(p[2]) < INFINITY);
            const uint64_t bm = __ballot(bad_ && valid);
            redo = redo || bm != 0;
            const bool mine = (((bm | (bm >> 32)) >> j) & 1u) != 0;
            if (valid && h == 0) {
                float *o = b.rec_c + 3 * (int64_t)rec;
                o[0] = mine ? __uint_as_float(kRedo) : sigmoid_hw(p[0]);
                o[1] = sigmoid_hw(p[1]);
                o[2] = sigmoid_hw(p[2]);
            }
        };

        load_z0();
#pragma unroll
        for (int s = 0; s < 3; ++s) layer0_step(s);

        for (;;) {
            bool cbad = bad;
            __builtin_amdgcn_sched_barrier(0);
            out[0] = out[1] = f4_t{0.f, 0.f, 0.f, 0.f};
            uint32_t claim = 0;
            if (lane == 0) claim = atomicAdd(&claimed, 1u);
            split_chunk(0);
            h8_t a[2], an[2];
#pragma unroll
            for (int p = 0; p < 2; ++p) a[p] = w1f[p * 2048];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < 4; ++t) {
#pragma unroll
                for (int c = 0; c < 8; ++c) {
                    f16_t &ah = acch[t & 1], &al = accl[t & 1];
                    if (c == 0) {
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const f4_t z = *(const f4_t *)(fl + kXB1 + 32 * t + 8 * i + 4 * h);
#pragma unroll
                            for (int r = 0; r < 4; ++r) {
                                ah[4 * i + r] = z[r];
                                al[4 * i + r] = 0.f;
                            }
                        }
                    }
                    const int nx = t * 8 + c + 1 < 32 ? t * 8 + c + 1 : t * 8 + c;
#pragma unroll
                    for (int p = 0; p < 2; ++p) an[p] = w1f[p * 2048 + nx * 64];
                    ah = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[0], hb[0][c], ah, 0, 0, 0);
                    al = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[0], hb[1][c], al, 0, 0, 0);
                    al = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[1], hb[0][c], al, 0, 0, 0);
#pragma unroll
                    for (int p = 0; p < 2; ++p) a[p] = an[p];
                    // what else happens during these MFMAs
                    if (t == 0 && c < 7) split_chunk(c + 1);
                    if (t == 0 && c == 1) {
                        nbt = batch_of(__builtin_amdgcn_readfirstlane(claim));
                        nrec = record_of(nbt);
                    }
                    if (t == 0 && c == 7) {
                        nray = b.rec_ray[nrec];
                        nk = b.rec_k[nrec];
                    }
                    if (t == 1 && c == 4) load_sample_ray(b, nray, nk, cur);
                    // an activation beyond float16's range makes every low sum of its sample infinite or NaN
                    if (t == 1 && c == 1) cbad = cbad || !(fabsf(accl[0][0]) < INFINITY);
                    if (t > 0 && (c & 1)) output_rows(t - 1, c >> 1);
                    if (t == 2 && c == 2) {
                        float xp[3];
                        sample_position(cur, xp);
                        gt.issue(g, xp, h);
                    }
                    if (t == 3 && c >= 1 && c < 7) x[c - 1] = gt.feature(c - 1);
                    if (t == 3 && c == 7) split_features();
                    interleave_mfma<3>();
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            load_z0();
#pragma unroll
            for (int i = 0; i < 4; ++i) output_rows(3, i);
            __builtin_amdgcn_sched_barrier(0);
            finish(bt, crec, cbad);
            if (nbt >= bcount) break;
            bt = nbt;
            crec = nrec;
#pragma unroll
            for (int s = 0; s < 3; ++s) layer0_step(s);
        }
    }
    if (!__syncthreads_or(redo)) return;
    // (every wavefront is past the barrier, so the split's weights are done with)
    stage_weights_f32(m, lds, 1.f);
    __syncthreads();
    for (uint32_t k = wave;; k += kFwdWaves) {
        const uint32_t rbt = batch_of(k);
        if (rbt >= bcount) break;
        for (uint32_t s0 = (bfirst + rbt) * kFwdBatch, end = s0 + kFwdBatch; s0 < end && s0 < total; s0 += 16) {
            const uint32_t s = min(s0 + (lane & 15), total - 1), rec = voxel ? b.perm[s] : s;
            const bool marked = __float_as_uint(b.rec_c[3 * (int64_t)rec]) == kRedo;
            if (__builtin_amdgcn_ballot_w64(marked)) colours_f32<T, HASH>(g, b, lds, rec, marked, e0);
        }
    }
}

template <typename T, bool HASH>
static void launch_fwd(const GridK &g, const cic_mlp &m, const RenderBufs &b, bool voxel, hipStream_t s)
{
    static bool attr_set = false;   // per process; the attribute is per kernel
    if (!attr_set) {
        (void)hipFuncSetAttribute((const void *)k_mlp_fwd_f32<T, HASH>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                  kXLdsBytes);
        attr_set = true;
    }
    hipLaunchKernelGGL((k_mlp_fwd_f32<T, HASH>), dim3(num_cus(b)), dim3(kFwdWaves * 64), kXLdsBytes, s, g, m, b,
                       voxel ? 1 : 0);
}

// FP32, in either order, uses the per-ray direction table (b.z0 must be
// filled by launch_ray_embed first): in voxel order the samples of a ray
// within a brick are consecutive, so the table rows stay cached (the same rows
// without the table cost 13% on eight 800x800 views), and both orders then
// give the same bits.  The BF16 kernel reads a
// per-ray BF16 encoding table instead.
template <typename T>
void launch_mlp_forward(const GridK &g, const cic_mlp &m, const RenderBufs &b, bool voxel, hipStream_t s)
{
    if (m.compute == CIC_BF16) {
        launch_mlp_forward_bf16<T>(g, m, b, voxel, s);
        return;
    }
    if (g.hlevels) launch_fwd<T, true>(g, m, b, voxel, s);
    else launch_fwd<T, false>(g, m, b, voxel, s);
}

template void launch_mlp_forward<float>(const GridK &, const cic_mlp &, const RenderBufs &, bool, hipStream_t);
template void launch_mlp_forward<__half>(const GridK &, const cic_mlp &, const RenderBufs &, bool, hipStream_t);

}  // namespace cic
