// Device helpers shared by the FP32 and BF16 MLP kernels: the per-sample
// inputs of layer 0 (trilinear feature gather or multi-level encoding, and
// the view-direction encoding) and the persistent grids' size.
#pragma once
#include <type_traits>
#include <utility>

#include "kernels.h"

namespace cic {

typedef float f4_t __attribute__((ext_vector_type(4)));
typedef float f2_t __attribute__((ext_vector_type(2)));
typedef float f16_t __attribute__((ext_vector_type(16)));
typedef _Float16 h8_t __attribute__((ext_vector_type(8)));
typedef _Float16 h2_t __attribute__((ext_vector_type(2)));
typedef uint32_t u4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf8_t __attribute__((ext_vector_type(8)));

// Input index (0..38, or -1 for padding) of chunk c for lane group q.
__host__ __device__ __forceinline__ int l0_input(int c, int q)
{
    if (c < 3) return 3 * q + c;
    if (c == 3) return q < 3 ? 12 + q : -1;
    const int jj = (c - 4) >> 1, p = 3 * q + jj;
    return ((c - 4) & 1) ? 27 + p : 15 + p;
}

__device__ __forceinline__ float pick3(int i, float a, float b, float c) { return i == 0 ? a : (i == 1 ? b : c); }

// float32 weights in LDS (in floats), pre-permuted into per-lane MFMA
// fragment order (the adjoint's recomputed forward): W0 [t 8][c2 5][lane 64][2]
// (lane l of output tile t holds row 16t + l%16 at the inputs of chunks 2*c2,
// 2*c2+1 of lane group l/16), W1 [t 8][c4 8][lane 64][4] (row 16t + l%16,
// columns 16*c4 + 4*(l/16) + r), W2 [q 4][ch 3][t 8][r 4] (column 16t + 4q + r
// of output row ch), biases.  4 floats after every 16 lanes of a W1 block keep
// the fragment reads conflict-free, and put a read of W1 transposed (lane l
// taking row 16 c4 + 4 (l/16) + rr, column 16 ti + l%16) on 64 distinct banks
// instead of 16.  W1 and its bias are held times the power of two s1, W2
// divided by it (exact, and without effect on the outputs).
struct F32Lds {
    static constexpr int kW1Block = 272;
    static constexpr int kW0 = 0;
    static constexpr int kW1 = kW0 + 8 * 5 * 64 * 2;
    static constexpr int kW2 = kW1 + 64 * kW1Block;
    static constexpr int kB0 = kW2 + 4 * 3 * 8 * 4;
    static constexpr int kB1 = kB0 + 128;
    static constexpr int kB2 = kB1 + 128;
    static constexpr int kSize = kB2 + 4;
    // first float of lane `lane` of W1 block (t * 8 + c4)
    __host__ __device__ static constexpr int w1(int blk, int lane)
    {
        return kW1 + blk * kW1Block + 4 * (lane + (lane >> 4));
    }
};

__device__ __forceinline__ void stage_weights_f32(const cic_mlp &m, float *lds, float s1)
{
    typedef F32Lds L;
    const int nt = blockDim.x;
    for (int i = threadIdx.x; i < 8 * 10 * 64; i += nt) {
        const int l = i & 63, c = (i >> 6) % 10, t = i / 640;
        const int row = 16 * t + (l & 15), src = l0_input(c, l >> 4);
        lds[L::kW0 + ((t * 5 + (c >> 1)) * 64 + l) * 2 + (c & 1)] = src >= 0 ? m.w0[row * 39 + src] : 0.f;
    }
    for (int i = threadIdx.x; i < 8 * 32 * 64; i += nt) {
        const int l = i & 63, c = (i >> 6) & 31, t = i >> 11;
        const int row = 16 * t + (l & 15), col = 16 * (c >> 2) + 4 * (l >> 4) + (c & 3);
        lds[L::w1(t * 8 + (c >> 2), l) + (c & 3)] = m.w1[row * 128 + col] * s1;
    }
    for (int i = threadIdx.x; i < 384; i += nt) {
        const int q = i / 96, ch = (i / 32) % 3, t = (i / 4) % 8, r = i & 3;
        lds[L::kW2 + i] = m.w2[ch * 128 + 16 * t + 4 * q + r] * (1.f / s1);
    }
    for (int i = threadIdx.x; i < 128; i += nt) {
        lds[L::kB0 + i] = m.b0[i];
        lds[L::kB1 + i] = m.b1[i] * s1;
    }
    if (threadIdx.x < 3) lds[L::kB2 + threadIdx.x] = m.b2[threadIdx.x];
}

// View-encoding inputs of lane group q (layer-0 chunks 3-9): direction
// component q (q = 3 pads with 0), then sin and cos of encoding pairs
// p = 3q..3q+2, p = 4*component + octave.
__device__ __forceinline__ void encode_group(const float d[3], int q, float x[7])
{
    x[0] = q < 3 ? pick3(q, d[0], d[1], d[2]) : 0.f;
#pragma unroll
    for (int jj = 0; jj < 3; ++jj) {
        const int p = 3 * q + jj;
        const float a = ldexpf(pick3(p >> 2, d[0], d[1], d[2]), p & 3);
        float sn, cs;
        sincosf(a, &sn, &cs);
        x[1 + 2 * jj] = sn;
        x[2 + 2 * jj] = cs;
    }
}

// The ray data a sample's gather needs: its ray, sample index, interval
// start and step, origin and direction.
struct SampleRay {
    uint32_t ray;
    int k;
    float tn, delta;
    float o[3], d[3];
};

__device__ __forceinline__ void load_sample_ray(const RenderBufs &b, uint32_t ray, int k, SampleRay &r)
{
    r.ray = ray;
    r.k = k;
    const RayInfo inf = b.info[ray];
    r.tn = inf.tn;
    r.delta = inf.delta;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        r.o[a] = b.rays_o[3 * (int64_t)ray + a];
        r.d[a] = b.rays_d[3 * (int64_t)ray + a];
    }
}

// Sample position o + t_k d in float32 (the march's sample point).
__device__ __forceinline__ void sample_position(const SampleRay &r, float xp[3])
{
    const float tk = sample_t(r.tn, r.delta, r.k);
#pragma unroll
    for (int a = 0; a < 3; ++a) xp[a] = r.o[a] + tk * r.d[a];
}

// Layer-0 inputs of one sample of a dense float32 grid for this lane's group
// q of four (the adjoint): features 3q .. 3q+2 and the group's encoding.
__device__ __forceinline__ void sample_inputs(const GridK &g, const RenderBufs &b, int64_t rec, int q, float x[10])
{
    SampleRay r;
    load_sample_ray(b, b.rec_ray[rec], b.rec_k[rec], r);
    int i0[3];
    float fr[3], tk;
    sample_voxel(r.o, r.d, r.tn, r.delta, r.k, g, i0, fr, tk);
#pragma unroll
    for (int c = 0; c < 3; ++c) x[c] = trilerp1((const float *)g.features, g, i0, fr, 12, 3 * q + c);
    encode_group(r.d, q, x + 3);
}

// Features 6h .. 6h+5 of one sample (lane half h): issue() sends the loads of
// the 8 corners, feature() interpolates one of them, in two steps so that a
// batch's work fits between the loads and their use.  Dense grids: corner c
// (x bit 2, y bit 1, z bit 0), 6 consecutive channels.  Multi-level encoding:
// levels 2h and 2h + 1, 3 features each.
template <typename T, bool HASH>
struct Gather {
    static constexpr bool kHalf = sizeof(T) == 2;
    static constexpr int kWords = kHalf ? (HASH ? 4 : 3) : 6;   // 32-bit words per corner
    uint32_t raw[8][kWords];
    float fr[HASH ? 2 : 1][3];
    uint32_t odd;   // float16 tables: parity of each entry, bit 8 * level + corner

    // xp: the sample's position
    __device__ __forceinline__ void issue(const GridK &g, const float xp[3], int h)
    {
        if constexpr (HASH) {
            odd = 0;
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                // level 2h + u (its parameters selected, not indexed by lane)
                const int N = h ? g.hN[2 + u] : g.hN[u], dense = h ? g.hdense[2 + u] : g.hdense[u];
                float scale[3];
#pragma unroll
                for (int a = 0; a < 3; ++a) scale[a] = h ? g.hscale[2 + u][a] : g.hscale[u][a];
                int i0[3];
                hash_cell_n(g.lo, N, scale, xp, i0, fr[u]);
                const T *tab = (const T *)g.htab + (size_t)(2 * h + u) * ((size_t)g.hmask + 1) * 3;
#pragma unroll
                for (int c = 0; c < 8; ++c) {
                    const uint64_t e = hash_entry_n(N, dense, g.hmask, (uint32_t)(i0[0] + ((c >> 2) & 1)),
                                                    (uint32_t)(i0[1] + ((c >> 1) & 1)), (uint32_t)(i0[2] + (c & 1)));
                    if constexpr (kHalf) {
                        // the two aligned words that hold the entry's 6 bytes (see load_entry3)
                        const uint32_t *w = (const uint32_t *)((const char *)tab + ((e * 6) & ~(uint64_t)3));
                        raw[c][2 * u] = w[0];
                        raw[c][2 * u + 1] = w[1];
                        odd |= ((uint32_t)e & 1u) << (8 * u + c);
                    } else {
                        const uint32_t *w = (const uint32_t *)tab + e * 3;
#pragma unroll
                        for (int k = 0; k < 3; ++k) raw[c][3 * u + k] = w[k];
                    }
                }
            }
        } else {
            int i0[3];
            locate(xp, g, i0, fr[0]);
            constexpr int kRec = 12 * (int)sizeof(T);
            const int64_t sy = (int64_t)g.r2 * kRec, sx = (int64_t)g.r1 * sy;
            const char *p = (const char *)g.features + vertex_index(g, i0[0], i0[1], i0[2]) * kRec + h * (kRec / 2);
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const uint32_t *w =
                    (const uint32_t *)(p + ((c >> 2) & 1) * sx + ((c >> 1) & 1) * sy + (c & 1) * kRec);
#pragma unroll
                for (int k = 0; k < kWords; ++k) raw[c][k] = w[k];
            }
        }
    }

    __device__ __forceinline__ float value(int c, int k) const
    {
        if constexpr (!kHalf) {
            return __uint_as_float(raw[c][k]);
        } else if constexpr (!HASH) {
            const uint32_t w = raw[c][k >> 1];
            return __half2float(__ushort_as_half((unsigned short)((k & 1) ? w >> 16 : w & 0xffffu)));
        } else {
            const int u = k / 3, f = k % 3;
            const uint32_t a = raw[c][2 * u], b = raw[c][2 * u + 1], sh = ((odd >> (8 * u + c)) & 1u) * 16u;
            const uint32_t w = f < 2 ? __builtin_amdgcn_alignbit(b, a, sh) : b >> sh;
            return __half2float(__ushort_as_half((unsigned short)(f == 1 ? w >> 16 : w & 0xffffu)));
        }
    }

    __device__ __forceinline__ float feature(int k) const
    {
        const float *f = fr[HASH ? k / 3 : 0];
        const float c00 = lerpf(value(0, k), value(1, k), f[2]), c01 = lerpf(value(2, k), value(3, k), f[2]);
        const float c10 = lerpf(value(4, k), value(5, k), f[2]), c11 = lerpf(value(6, k), value(7, k), f[2]);
        return lerpf(lerpf(c00, c01, f[1]), lerpf(c10, c11, f[1]), f[0]);
    }
};

// f(0), f(1), .. f(N - 1) with compile-time arguments (a loop whose body is as
// long as a batch's exceeds the compiler's unrolling limit)
template <int... I, typename F>
__device__ __forceinline__ void static_for_seq(std::integer_sequence<int, I...>, const F &f)
{
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F> __device__ __forceinline__ void static_for(const F &f)
{
    static_for_seq(std::make_integer_sequence<int, N>{}, f);
}

// Alternates the instructions before it, back to the last barrier: N times one MFMA,
// then up to 8 vector and a few memory instructions that fit in its shadow.
template <int N>
__device__ __forceinline__ void interleave_mfma()
{
#pragma unroll
    for (int u = 0; u < N; ++u) {
        __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);     // MFMA
        __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);   // LDS reads
        __builtin_amdgcn_sched_group_barrier(0x2, 8, 0);     // vector ALU
        __builtin_amdgcn_sched_group_barrier(0x20, 4, 0);    // global loads
    }
}

// hidden unit of slot e of chunk c (16 units) for lane half h: the rows that
// the lane half holds of the 32-row result tile c / 2
__host__ __device__ __forceinline__ int x_hid(int c, int h, int e)
{
    return 16 * c + 8 * (e >> 2) + 4 * h + (e & 3);
}

// part p of float32 b split into three BF16 values b0 + b1 + b2 = b (each
// remainder is exact in float32, and the last has at most 8 significant bits)
__device__ __forceinline__ float bf16_part(float b, int p)
{
    const float hi = (float)(__bf16)b, r1 = b - hi;
    const float mid = (float)(__bf16)r1, r2 = r1 - mid;
    return p == 0 ? hi : p == 1 ? mid : r2;
}

__device__ __forceinline__ uint32_t pack_bf2(float a, float b)
{
    typedef __bf16 bf2_t __attribute__((ext_vector_type(2)));
    bf2_t v;
    v[0] = (__bf16)a;
    v[1] = (__bf16)b;
    return __builtin_bit_cast(uint32_t, v);
}

template <int CTRL> __device__ __forceinline__ uint32_t max_dpp(uint32_t v)
{
    // (a lane without a source takes 0: one instruction)
    return max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, true));
}

// the wavefront's largest value, in its last lane
__device__ __forceinline__ uint32_t wave_max_last(uint32_t v)
{
    v = max_dpp<0x111>(v);   // row_shr:1, 2, 4, 8
    v = max_dpp<0x112>(v);
    v = max_dpp<0x114>(v);
    v = max_dpp<0x118>(v);
    v = max_dpp<0x142>(v);   // row_bcast:15, 31
    return max_dpp<0x143>(v);
}

// Output sigmoid from the hardware base-2 exponential and reciprocal:
// 1 / (1 + 2^(-x log2 e)), within about 1e-6 relative of the correctly
// rounded value for |x| < 20 (the rounding of x log2 e dominates), in 4
// instructions where the library's expf and IEEE division take about 25.
__device__ __forceinline__ float sigmoid_hw(float x)
{
    return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.44269504088896341f * x));
}

inline int num_cus(const RenderBufs &b)
{
    if (b.grid_cus > 0) return b.grid_cus;
    int dev = 0, n = 0;
    (void)hipGetDevice(&dev);
    (void)hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev);
    return n > 0 ? n : 256;
}

}  // namespace cic
