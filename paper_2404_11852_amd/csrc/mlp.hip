// Feature Gathering + Feature Computation (Sec. II-B) for the compacted live
// samples: trilinear gather of the 12 feature channels, the view-direction
// encoding, and the 39 -> 128 -> 128 -> 3 MLP on MFMA, for float32 compute.
//
// Arithmetic.  The matrix cores run 16-bit products 16 times as fast as float32
// ones.  Layer 0 splits both operands into three BF16 parts, which have
// float32's range and together its 24 bits, and sums the six products above
// 2^-24 of the whole on top of the ray's float32 direction term, whatever the
// magnitudes of features and weights are.  Layer 1 splits both operands into
// two float16 parts, v = hi + lo / 2^11 (22 significand bits and a sign between
// them), and sums three products, hi hi, hi lo and lo hi, in float32.  The
// remainders are kept times 2^11, so they are normal float16 values wherever
// the first part is one, which is down to 2^-28 of the largest value: the
// activations are scaled by a power of two for each sample, by a bound of its
// own, and W1 by one for its largest entry.  The low products have their own
// accumulators, so the high ones are rounded 8 times over a 128-long sum where
// a float32 chain rounds 128 times.  The output layer is float32.
//
// Float32 products instead, for whole calls: where W1's rows and its columns (the
// hidden units on either side) differ by more than 2^26, multiplied, in their
// largest entries, so that small entries may decide a sum; where a weight is not
// finite or beyond 2^60.  And for single samples: features and weights whose products are
// beyond 2^100, an output that is not finite.
//
// Colour error against 64 bits, rms over 300,000 single-sample rays: 2.82e-8,
// and 2.90e-8 for a float32 MFMA chain; features x 30: 4.35e-8 and 4.82e-8; W0 x
// 30: 1.02e-7 and 1.16e-7; W1 x 8: 5.9e-8 and 6.6e-8 (BF16 parts in both layers
// were less exact, 3.06e-8, because one accumulator takes 48 roundings, and 1.4
// times as slow).  Layer 0 in two float16 parts, with one power of two for all of
// W0, took 8 of 116 products less (kernel 3.88 against 4.25 ms per 800x800
// frame), but lost features, weights and units that are small beside others:
// errors from 1e-6 (a channel 2^10 smaller) to all of it.
//
// Bound.  Matrix power: with the matrix cores 62% busy the card lowers its
// clock to 1.8 GHz (2.37 GHz under float32 MFMA at 85%), which is the busy
// rate times clock that a library BF16 product reaches here too (1.2
// PFLOP/s).  MLP stage of an 800x800 frame with 36 M live samples: 9.9 -> 4.3 ms.
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
// 236 VGPRs; 12 wavefronts spill, 8.4 against 4.7 ms per frame).  Within a
// batch the vector work (splitting the activations, the output layer, and
// the next batch's records, gathers and interpolation) sits between the
// layer-1 MFMAs: 3.5% faster than the same order left to the compiler.  The next
// batch's layer 0 goes out before this one's outputs are written (1%).
#include "mlp_common.h"

namespace cic {

constexpr int kFwdWaves = 8;    // wavefronts of the CU's one workgroup
constexpr int kFwdBatch = 32;   // samples per wavefront batch

// LDS in 16-byte fragments, then floats
constexpr int kXW1 = 0;                          // [part 2][t 4][c 8][lane 64]
constexpr int kL0Steps = 5;                      // 36 of 40 slots per lane half: 6 products of 6 features
constexpr int kXW0 = kXW1 + 2 * 4 * 8 * 64;      // [t 4][s 5][lane 64]
constexpr int kXFrags = kXW0 + 4 * kL0Steps * 64;
constexpr int kXB1 = 0, kXW2 = 128;              // [128]; [t 4][i 4][h 2][ch 4][r 4]
constexpr int kXB2 = kXW2 + 512;
constexpr int kXTop = kXB2 + 4;                  // [h 2][8]: see stage_weights_split
constexpr int kXFloats = kXTop + 16;
constexpr int kXLdsBytes = std::max(kXFrags * 16 + kXFloats * 4, F32Lds::kSize * 4);
constexpr float kLoScale = 2048.f;               // the low parts are kept times 2^11

// v0 and v1 times `scale` (a power of two) into a float16 and a second float16
// that holds the remainder times 2^11 (the remainder is exact in float32; times
// 2^11 it is a normal float16 wherever the first part is)
__device__ __forceinline__ void split2(float v0, float v1, float scale, uint32_t &hi, uint32_t &lo)
{
    h2_t a, b;
    a[0] = (_Float16)(v0 * scale);
    a[1] = (_Float16)(v1 * scale);
    hi = __builtin_bit_cast(uint32_t, a);
    asm("" : "+v"(hi));   // one packed conversion, not two more single ones for the remainders
    a = __builtin_bit_cast(h2_t, hi);
    b[0] = (_Float16)fmaf((float)a[0], -kLoScale, v0 * (scale * kLoScale));
    b[1] = (_Float16)fmaf((float)a[1], -kLoScale, v1 * (scale * kLoScale));
    lo = __builtin_bit_cast(uint32_t, b);
}

// v0 and v1 into three BF16 parts each (every remainder is exact in float32)
__device__ __forceinline__ void split3(float v0, float v1, uint32_t part[3])
{
#pragma unroll
    for (int p = 0; p < 3; ++p) {
        uint32_t w = pack_bf2(v0, v1);
        asm("" : "+v"(w));
        part[p] = w;
        v0 -= __uint_as_float(w << 16);
        v1 -= __uint_as_float(w & 0xffff0000u);
    }
}

// Layer 0's products, the small ones first: which part of the weight, which of the feature
__host__ __device__ constexpr int l0_wpart(int p) { return p == 0 ? 2 : p == 2 || p == 3 ? 1 : 0; }
__host__ __device__ constexpr int l0_xpart(int p) { return p == 1 ? 2 : p == 2 || p == 4 ? 1 : 0; }

constexpr float kWMax = 0x1p60f;    // largest weight of the split path, and W1's largest at least 2^-60
constexpr float kSpread = 0x1p26f;  // largest product of the ratios of its rows' and of its columns' largest entries

// Weights into LDS in fragment order.  W1 is scaled by the power of two 2^e1
// that puts its largest entry in [2^14, 2^15) before the split (so both parts
// use float16's range).  For the samples' scales, kXTop of lane half h: the
// largest weight of each of its 6 features, the largest sum of a row's weights
// of d (the half's seventh), and that of its other direction weights and bias.
// Returns e1, or kPlain where the call runs on float32 products (see the top of
// the file).  Every load goes out before the first barrier (a SpaRW target's
// MLP stage 215 -> 209 us against loading between the barriers).
constexpr int kPlain = 1000;
__device__ int stage_weights_split(const cic_mlp &m, float *lds)
{
    h8_t *w1 = (h8_t *)lds + kXW1;
    __bf16 *w0 = (__bf16 *)((h8_t *)lds + kXW0);
    float *fl = lds + kXFrags * 4;
    constexpr int kT = kFwdWaves * 64, kN = 4 * 8 * 64, kIt = kN / kT;
    static_assert(kN % kT == 0 && kT == 512, "one W2 entry, three of W0 and the W1 fragments per thread");
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    f4_t w[kIt][2];
#pragma unroll
    for (int k = 0; k < kIt; ++k) {
        const int i = tid + k * kT, l = i & 63, c = (i >> 6) & 7, t = i >> 9;
        const float *src = m.w1 + (32 * t + (l & 31)) * 128;
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e) w[k][u][e] = src[x_hid(c, l >> 5, 4 * u) + e];
    }
    // W0: features (tid >> 7) + 4k of row tid & 127; a quarter of the direction weights and bias of row tid >> 2
    float v0[3], vd[7];
#pragma unroll
    for (int k = 0; k < 3; ++k) v0[k] = m.w0[(tid & 127) * 39 + (tid >> 7) + 4 * k];
#pragma unroll
    for (int e = 0; e < 7; ++e) {
        const int i = (tid & 3) * 7 + e;
        vd[e] = fabsf(*(i < 27 ? m.w0 + (tid >> 2) * 39 + 12 + i : m.b0 + (tid >> 2)));
    }
    const int ch2 = (tid >> 2) & 3, h2 = (tid >> 4) & 1;
    const int row2 = 32 * (tid >> 7) + 8 * ((tid >> 5) & 3) + 4 * h2 + (tid & 3);
    const float v2 = m.w2[min(ch2, 2) * 128 + row2], vb1 = m.b1[tid & 127], vb2 = m.b2[min(tid & 3, 2)];
    // Maxima as integers, which order positive floats (NaN above all).  W1: per
    // row over a fragment's 8 columns, combined below, and per column over the
    // lane's rows, then over lanes.
    uint32_t col[8] = {}, dir, rest, f0[3];
#pragma unroll
    for (int k = 0; k < kIt; ++k) {
        uint32_t row = 0;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const uint32_t a = __float_as_uint(fabsf(w[k][e >> 2][e & 3]));
            row = max(row, a);
            col[e] = max(col[e], a);
        }
        ((uint32_t *)w1)[(wave * kIt + k) * 64 + lane] = row;   // (where the fragments come later)
    }
    {
        float d = 0.f, r = 0.f;
#pragma unroll
        for (int e = 0; e < 7; ++e) {
            if ((tid & 3) == 0 && e < 3) d += vd[e];
            else r += vd[e];
        }
        r += __shfl_xor(r, 1, kWave);
        r += __shfl_xor(r, 2, kWave);
        dir = wave_max_last(__float_as_uint(d));
        rest = wave_max_last(__float_as_uint(r));
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) f0[k] = wave_max_last(__float_as_uint(fabsf(v0[k])));
    // largest of the weights that only have to be within kWMax
    uint32_t any = wave_max_last(max(__float_as_uint(fabsf(v2)), __float_as_uint(fabsf(vb1))));
    uint32_t hi = 0, lo = 0x7f800000u;   // largest and smallest (but zero) of the columns, hi later of the rows too
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        // (lanes 31 and 63 end with the maxima of their 32 lanes, the others with some of them)
        uint32_t v = col[e];
        v = max_dpp<0x111>(v);   // row_shr:1, 2, 4, 8
        v = max_dpp<0x112>(v);
        v = max_dpp<0x114>(v);
        v = max_dpp<0x118>(v);
        v = max_dpp<0x142>(v);   // row_bcast:15
        hi = max(hi, v);
        if ((lane & 31) == 31 && v) lo = min(lo, v);
    }
    uint32_t *red = (uint32_t *)fl;   // [wave][8]
    if (lane == 63) {
        red[wave * 8 + 2] = dir;
        red[wave * 8 + 3] = rest;
#pragma unroll
        for (int k = 0; k < 3; ++k) red[wave * 8 + 4 + k] = f0[k];
        red[wave * 8 + 7] = any;
    }
    __syncthreads();
    if (tid < 128) {
        uint32_t row = 0;
#pragma unroll
        for (int c = 0; c < 8; ++c)
#pragma unroll
            for (int h = 0; h < 2; ++h)
                row = max(row, ((const uint32_t *)w1)[(c * kIt + (tid >> 5)) * 64 + 32 * h + (tid & 31)]);
        hi = max(hi, row);
        const uint32_t rows_lo = ~wave_max_last(~(row ? row : 0x7f800000u));
        if (lane == 63) red[64 + wave] = rows_lo;
    }
    hi = wave_max_last(hi);
    lo = ~wave_max_last(~lo);
    if (lane == 63) {
        red[wave * 8] = hi;
        red[wave * 8 + 1] = lo;
    }
    __syncthreads();
    hi = dir = rest = any = 0;
    lo = 0x7f800000u;
#pragma unroll
    for (int k = 0; k < kFwdWaves; ++k) {
        hi = max(hi, red[k * 8]);
        lo = min(lo, red[k * 8 + 1]);
        dir = max(dir, red[k * 8 + 2]);
        rest = max(rest, red[k * 8 + 3]);
#pragma unroll
        for (int u = 4; u < 8; ++u) any = max(any, red[k * 8 + u]);
    }
    // feature f's two wavefronts are 2 (f % 4) and the next, word f / 4
    const int f = 6 * ((tid >> 3) & 1) + (tid & 7);
    const uint32_t feat = (tid & 7) < 6 ? max(red[(f & 3) * 16 + 4 + (f >> 2)], red[(f & 3) * 16 + 12 + (f >> 2)])
                                        : (tid & 7) == 6 ? dir : rest;
    __syncthreads();
    const uint32_t rows_lo = min(red[64], red[65]);
    const float top = __uint_as_float(hi), all = __uint_as_float(max(max(hi, any), max(dir, rest)));
    const float spread = top / __uint_as_float(lo) * (top / __uint_as_float(rows_lo));
    if (!(all <= kWMax) || (hi && !(top >= 1.f / kWMax && spread <= kSpread))) return kPlain;
    const int e1 = hi ? 14 + 127 - (int)(hi >> 23) : 0;
    const float s1 = ldexpf(1.f, e1);
    // layer 0's slot of feature ff of half h in product p: 6 p + ff, 8 of them per step
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const int ft = (tid >> 7) + 4 * k, h = ft >= 6, row = tid & 127;
#pragma unroll
        for (int p = 0; p < 6; ++p) {
            const int slot = 6 * p + ft - 6 * h;
            w0[(((row >> 5) * kL0Steps + (slot >> 3)) * 64 + 32 * h + (row & 31)) * 8 + (slot & 7)] =
                (__bf16)bf16_part(v0[k], l0_wpart(p));
        }
    }
    if (tid < 256)   // the last four slots of the last step
        *(uint64_t *)(w0 + (((tid >> 6) * kL0Steps + kL0Steps - 1) * 64 + lane) * 8 + 4) = 0;
#pragma unroll
    for (int k = 0; k < kIt; ++k) {
        u4_t h, l;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            uint32_t a, b;
            split2(w[k][e >> 1][2 * (e & 1)], w[k][e >> 1][2 * (e & 1) + 1], s1, a, b);
            h[e] = a;
            l[e] = b;
        }
        w1[tid + k * kT] = __builtin_bit_cast(h8_t, h);
        w1[kN + tid + k * kT] = __builtin_bit_cast(h8_t, l);
    }
    fl[kXW2 + tid] = ch2 < 3 ? v2 : 0.f;
    if (tid < 128) fl[kXB1 + tid] = vb1;
    if (tid < 4) fl[kXB2 + tid] = tid < 3 ? vb2 : 0.f;
    if (tid < 16) fl[kXTop + tid] = __uint_as_float(feat);
    return e1;
}

// Per-ray direction term of layer 0: z0[ray][o] = b0[o] + sum_i W0[o][12+i] pe_i
// over the 27 direction inputs (d, sin, cos), once per ray with live samples
// (float32; used in either order).  A block stages the inputs of RAYS rays in
// LDS (one sincosf per argument gives both its sine and cosine input), and each
// of its 128 threads then forms output o for every ray with its 27 weights held
// in registers.  The weight rows and the rays are loaded together, before the
// first barrier.  64 rays per block amortise the weight reads in large passes;
// small ones, and the holes of a warped frame, take 16, so that the launch
// spreads over the chip (4096 rays: 64 per block 16.6 us, 16 per block 7.2).
template <int RAYS, bool COUNTED>
__global__ __launch_bounds__(128) void k_ray_embed(cic_mlp m, RenderBufs b, float *z0)
{
    __shared__ __attribute__((aligned(16))) float pe[RAYS][28];
    __shared__ uint32_t live[RAYS];
    const int o = threadIdx.x;
    // (a device-counted pass, the holes of a warped frame, has rays up to its count)
    const int64_t n = COUNTED ? min((int64_t)*b.n_active, b.n) : b.n;
    if ((int64_t)blockIdx.x * RAYS >= n) return;
    float w[27];
#pragma unroll
    for (int i = 0; i < 27; ++i) w[i] = m.w0[o * 39 + 12 + i];
    const float bias = m.b0[o];
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
        __syncthreads();
        for (int r = 0; r < RAYS; ++r) {
            if (!live[r]) continue;
            float acc = bias;
#pragma unroll
            for (int i = 0; i < 27; ++i) acc = fmaf(w[i], pe[r][i], acc);
            z0[(base + r) * 128 + o] = acc;
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

// float32 MFMA for the samples that leave the range of the split, or for all of
// them where the weights do: 16 samples per step of a wavefront, 16x16x4 products as in the
// adjoint's recomputed forward, the weights staged anew over the split's.
// Bound by the float32 products: a call of 1.6 M samples takes 0.37 ms, 0.87 when
// all of them come here (13.0 with a wavefront per sample on the vector ALUs,
// which read W1 from memory for each).
// ahead(k): the loads of the next step's samples, in three rounds, each of which
// uses the one before (an 800x800 frame whose every sample comes here: 11.87 ms
// without, 11.37 so; 10.88 with four wavefronts per SIMD, which the split's
// registers do not leave).
template <typename T, bool HASH, typename Ahead>
__device__ __forceinline__ void colours_f32(const GridK &g, const RenderBufs &b, const float *lds, uint32_t rec,
                                            const SampleRay &r, bool write, const Ahead &ahead)
{
    typedef F32Lds L;
    const int lane = lane_id(), q = lane >> 4;
    const f2_t *w0f = (const f2_t *)(lds + L::kW0);
    const f4_t *w2l = (const f4_t *)(lds + L::kW2);
    const float *w1f = lds + L::w1(0, lane);   // (block k at + k * kW1Block floats)
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
        h1[t] = *(const f4_t *)(zr + 16 * t);
        h2[t] = *(const f4_t *)(lds + L::kB1 + 16 * t + 4 * q);
    }
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int t = 0; t < 8; ++t)
            h1[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(w0f[(t * 5 + (c >> 1)) * 64 + lane][c & 1], x[c], h1[t], 0, 0, 0);
    // (the wavefront that is further through its step wins the matrix unit)
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int c4 = 0; c4 < 8; ++c4) {
        if (c4 % 2 == 0 && c4 < 6) ahead(c4 / 2);
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
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    __builtin_amdgcn_s_setprio(0);
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
    const int e1 = stage_weights_split(m, lds);
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
    const bf8_t *w0f = (const bf8_t *)lds + kXW0 + lane;
    const h8_t *w1f = (const h8_t *)lds + kXW1 + lane;

    const bool plain = e1 == kPlain;   // (the same in every workgroup)
    bool redo = plain;
    uint32_t bt = batch_of(wave), nbt = 0;
    if (!plain && bt < bcount) {
        const float inv_s1 = ldexpf(1.f, -e1);
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
        // the features and, once split, their parts: pair k's in xp3[k]
        float x[6];
        uint32_t xp3[3][3];
        bool bad;
        // A sample's power of two puts a bound of its first activations, the sum
        // of the magnitudes of layer 0's terms, in [2^14, 2^15): what float32
        // arithmetic rounds them by is relative to that sum too.  unscale takes
        // it and W1's out again.
        float scale, unscale, nscale, nunscale;
        auto split_features = [&]() {
            const f4_t t0 = *(const f4_t *)(fl + kXTop + 8 * h), t1 = *(const f4_t *)(fl + kXTop + 8 * h + 4);
            const float top[6] = {t0[0], t0[1], t0[2], t0[3], t1[0], t1[1]};
            float sum = 0.f;
#pragma unroll
            for (int k = 0; k < 6; ++k) sum = fmaf(fabsf(x[k]), top[k], sum);
            sum += __shfl_xor(sum, 32, kWave);
            sum += fmaf(fmaxf(fmaxf(fabsf(cur.d[0]), fabsf(cur.d[1])), fabsf(cur.d[2])), t1[2], t1[3]);
            bad = !(sum < 0x1p100f);
            const int e = max(14 + 2 * 127 - (__float_as_int(sum) >> 23), 127 - 100);
            nscale = __int_as_float(min(e, 127 + 60) << 23);
            nunscale = __int_as_float((2 * 127 - min(e, 127 + 60)) << 23) * inv_s1;
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                split3(x[2 * k], x[2 * k + 1], xp3[k]);
                // (keeps the interpolation and the split here, among the MFMAs,
                // and not moved down to their use)
                asm volatile("" : "+v"(xp3[k][0]), "+v"(xp3[k][1]), "+v"(xp3[k][2]));
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
        // live samples, so its row is written); word w of the 5 x 4 input words is
        // feature pair w % 3 of product w / 3
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
                v[e] = w / 3 < 6 ? xp3[w % 3][l0_xpart(w / 3)] : 0u;
            }
            const bf8_t xin = __builtin_bit_cast(bf8_t, v);
#pragma unroll
            for (int t = 0; t < 4; ++t)
                acc0[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w0f[(t * kL0Steps + s) * 64], xin, acc0[t], 0, 0, 0);
        };
        // ReLU and split of the 16 units of chunk c
        auto split_chunk = [&](int c) {
            u4_t hi, lo;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                uint32_t u, v;
                const int r = 8 * (c & 1) + 2 * e;
                split2(relu_bits(acc0[c >> 1][r]), relu_bits(acc0[c >> 1][r + 1]), scale, u, v);
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
            const f4_t b1 = *(const f4_t *)(fl + kXB1 + 32 * t + 8 * i + 4 * h);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float sum = fmaf(accl[t & 1][4 * i + r], 1.f / kLoScale, acch[t & 1][4 * i + r]);
                const float hv = relu_bits(fmaf(sum, unscale, b1[r]));
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
        for (int s = 0; s < kL0Steps; ++s) layer0_step(s);

        for (;;) {
            const bool cbad = bad;
            scale = nscale;
            unscale = nunscale;
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
                    if (c == 0)
#pragma unroll
                        for (int r = 0; r < 16; ++r) ah[r] = al[r] = 0.f;
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
#pragma unroll
            for (int s = 0; s < kL0Steps; ++s) layer0_step(s);
            finish(bt, crec, cbad);
            __builtin_amdgcn_sched_barrier(0);
            if (nbt >= bcount) break;
            bt = nbt;
            crec = nrec;
        }
    }
    if (!__syncthreads_or(redo)) return;
    // (every wavefront is past the barrier, so the split's weights are done with)
    stage_weights_f32(m, lds, 1.f);
    __syncthreads();
    // step u of this wavefront: half of its batch u / 2; its first sample, or total past the last
    auto step_start = [&](uint32_t u) -> uint32_t {
        const uint32_t rbt = batch_of(wave + (u >> 1) * kFwdWaves);
        return rbt < bcount ? min((bfirst + rbt) * kFwdBatch + 16 * (u & 1), total) : total;
    };
    auto step_record = [&](uint32_t s0) -> uint32_t {
        const uint32_t s = min(s0 + (lane & 15), total - 1);
        return voxel ? b.perm[s] : s;
    };
    uint32_t s0 = step_start(0), u = 0;
    if (s0 >= total) return;
    uint32_t rec = step_record(s0);
    SampleRay cur;
    load_sample_ray(b, b.rec_ray[rec], b.rec_k[rec], cur);
    while (s0 < total) {   // (the starts grow)
        const uint32_t n0 = step_start(++u);
        uint32_t nrec = 0, nray = 0;
        int nk = 0;
        SampleRay next;
        auto ahead = [&](int k) {
            if (k == 0) nrec = step_record(n0);
            if (k == 1) {
                nray = b.rec_ray[nrec];
                nk = b.rec_k[nrec];
            }
            if (k == 2) load_sample_ray(b, nray, nk, next);
        };
        const bool marked = plain || __float_as_uint(b.rec_c[3 * (int64_t)rec]) == kRedo;
        if (__builtin_amdgcn_ballot_w64(marked)) {
            colours_f32<T, HASH>(g, b, lds, rec, cur, marked, ahead);
        } else {
#pragma unroll
            for (int k = 0; k < 3; ++k) ahead(k);
        }
        s0 = n0;
        rec = nrec;
        cur = next;
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
