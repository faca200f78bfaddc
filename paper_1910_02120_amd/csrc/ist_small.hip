// All k local steps of a small network in one launch: one workgroup per subnet.
//
// A subnet of a few ten thousand weights at a batch of some dozen samples is microseconds of arithmetic for one
// compute unit, but a step is 2 t + 2 dependent launches of about 4.5 us each (t layers).  Here the subnet's weights,
// biases, activations and gradients live in the 160 KB LDS of one compute unit for the whole call: weights are read
// once and written once, every step reads its mini-batch (requested during the step before), and what used to be a launch
// is a workgroup barrier.
//
// Products run on 16 x 16 MFMA tiles (a hidden layer of 64 neurons and 32 samples is 8 of them: enough for the 16 waves
// of the workgroup) from LDS arrays [row][column] with zero padding up to the k-step unit (16 values in f32: four
// 16x16x4 products, lane group q taking k = 4 q + e in product e so that a k-contiguous operand is one 16-byte read;
// 32 values in bf16).  Row pitches are an odd multiple of 16 bytes: no bank conflict in any of the three directions.
//
// Measured (us per step, before -> now): two subnets of 64-64-64-10, 32 samples, f32: 31 -> 9.4; three subnets of
// 75-111-73-12, 50 samples, bf16: 48 -> 13.  What bounds it: of the 20,600 cycles of a step of the former 7,000 are its f32
// matrix products (one compute unit per subnet), the rest is the chain of 8 phases - descriptor and LDS latency, tile
// epilogues of a few dozen instructions, barriers.  8 or 12 waves instead of 16 measure the same.
#include "ist_internal.h"
#include "ist_mfma.h"

#include <algorithm>
#include <type_traits>

namespace ist {

namespace small {

constexpr int kWaves = 16, kThreads = 64 * kWaves;
constexpr int kXRegs = 8;   // 64-value pieces of the next mini-batch a wave holds in registers


// k-step unit: fragments of 16 rows (or columns) and U values of k
template <typename D> struct Unit;
template <> struct Unit<F32> {
    static constexpr int U = 16;
    struct Frag { float v[4]; };
    // [row][k] array: a lane's first byte for rows r0 .. r0 + 15; unit u lies kStep * u further on
    static constexpr int kStep = 64;
    __device__ static inline const unsigned char *kc_base(const unsigned char *m, int pitch, int r0, int lane)
    {
        return m + __umul24(r0 + (lane & 15), pitch) + 16 * (lane >> 4);
    }
    __device__ static inline Frag kc(const unsigned char *p)
    {
        const float4 x = *reinterpret_cast<const float4 *>(p);
        return Frag{{x.x, x.y, x.z, x.w}};
    }
    // [k][col] array: columns c0 .. c0 + 15; unit u lies U * pitch * u further on
    __device__ static inline const unsigned char *ks_base(const unsigned char *m, int pitch, int c0, int lane)
    {
        return m + __umul24(4 * (lane >> 4), pitch) + (c0 + (lane & 15)) * 4;
    }
    __device__ static inline Frag ks(const unsigned char *p, int pitch)
    {
        Frag f;
#pragma unroll
        for (int e = 0; e < 4; ++e) f.v[e] = *reinterpret_cast<const float *>(p + e * pitch);
        return f;
    }
    // operands exchanged: lane l ends up with row l % 16 of a and columns 4 (l / 16) .. + 3 of b
    __device__ static inline f32x4 mma(const Frag &a, const Frag &b, f32x4 c)
    {
#pragma unroll
        for (int e = 0; e < 4; ++e) c = __builtin_amdgcn_mfma_f32_16x16x4f32(b.v[e], a.v[e], c, 0, 0, 0);
        return c;
    }
    __device__ static inline f32x4 ld4(const unsigned char *p)
    {
        const float4 x = *reinterpret_cast<const float4 *>(p);
        return f32x4{x.x, x.y, x.z, x.w};
    }
    __device__ static inline void st4(unsigned char *p, f32x4 v) { *reinterpret_cast<float4 *>(p) = make_float4(v[0], v[1], v[2], v[3]); }
};
template <> struct Unit<BF16> {
    static constexpr int U = 32;
    struct Frag { bf16x8 v; };
    static constexpr int kStep = 64;
    __device__ static inline const unsigned char *kc_base(const unsigned char *m, int pitch, int r0, int lane)
    {
        return m + __umul24(r0 + (lane & 15), pitch) + 16 * (lane >> 4);
    }
    __device__ static inline Frag kc(const unsigned char *p) { return Frag{*reinterpret_cast<const bf16x8 *>(p)}; }
    // transposing reads: 16 lanes supply four k rows of 16 columns, lane q of them receives column q
    __device__ static inline const unsigned char *ks_base(const unsigned char *m, int pitch, int c0, int lane)
    {
        const int q = lane & 15;
        return m + __umul24(8 * (lane >> 4) + (q >> 2), pitch) + (c0 + 4 * (q & 3)) * 2;
    }
    __device__ static inline Frag ks(const unsigned char *p, int pitch)
    {
        typedef s16x4 __attribute__((address_space(3))) * lds_ptr;
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(p));
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(p + 4 * pitch));
        return Frag{__builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7))};
    }
    __device__ static inline f32x4 mma(const Frag &a, const Frag &b, f32x4 c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(b.v, a.v, c, 0, 0, 0);
    }
    __device__ static inline f32x4 ld4(const unsigned char *p)
    {
        const uint2 x = *reinterpret_cast<const uint2 *>(p);
        return f32x4{__uint_as_float(x.x << 16), __uint_as_float(x.x & 0xffff0000u), __uint_as_float(x.y << 16),
                     __uint_as_float(x.y & 0xffff0000u)};
    }
    __device__ static inline void st4(unsigned char *p, f32x4 v)
    {
        *reinterpret_cast<uint2 *>(p) = make_uint2(f32x2_to_bf16x2(v[0], v[1]), f32x2_to_bf16x2(v[2], v[3]));
    }
};

// i / n for the tile counts that fit in LDS (i, n < 1024), m = ceil(2^20 / n)
__device__ inline int tile_row(int i, int m) { return (int)((unsigned)i * (unsigned)m >> 20); }

enum Layout { KC, KS };   // operand stored [row][k] or [k][row]

// one 16 x 16 tile: sum over nu units of a (rows r0 ..) times b (columns c0 ..).  The LDS reads of several units are
// issued before the first of their products (left alone, the compiler waits for each unit's reads in turn).
template <typename D, Layout LA, Layout LB>
__device__ inline f32x4 tile(const unsigned char *a, int pa, int r0, const unsigned char *b, int pb, int c0, int nu, int lane)
{
    using T = Unit<D>;
    const unsigned char *qa = LA == KC ? T::kc_base(a, pa, r0, lane) : T::ks_base(a, pa, r0, lane);
    const unsigned char *qb = LB == KC ? T::kc_base(b, pb, c0, lane) : T::ks_base(b, pb, c0, lane);
    const int sa = LA == KC ? T::kStep : T::U * pa, sb = LB == KC ? T::kStep : T::U * pb;
    f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
    auto group = [&](auto count) {
        constexpr int G = decltype(count)::value;
        typename T::Frag fa[G], fb[G];
#pragma unroll
        for (int u = 0; u < G; ++u) {
            if constexpr (LA == KC) fa[u] = T::kc(qa + u * T::kStep); else fa[u] = T::ks(qa + u * sa, pa);
            if constexpr (LB == KC) fb[u] = T::kc(qb + u * T::kStep); else fb[u] = T::ks(qb + u * sb, pb);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < G; ++u) acc = T::mma(fa[u], fb[u], acc);
        qa += G * sa;
        qb += G * sb;
    };
    for (; nu >= 4; nu -= 4) group(std::integral_constant<int, 4>{});
    if (nu & 2) group(std::integral_constant<int, 2>{});
    if (nu & 1) group(std::integral_constant<int, 1>{});
    return acc;
}

// sum / maximum over the G lanes (16 or 64) of a row group, in every lane of it: rotations inside rows of 16 lanes, then
// (G = 64) across the rows
template <bool MAX> __device__ inline float combine(float x, float y) { return MAX ? fmaxf(x, y) : x + y; }
template <int G, bool MAX> __device__ inline float group_reduce(float v)
{
    auto ror = [](float x, auto ctl) {
        return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), decltype(ctl)::value, 0xF, 0xF, true));
    };
    v = combine<MAX>(v, ror(v, std::integral_constant<int, 0x128>{}));   // row_ror:8, 4, 2, 1
    v = combine<MAX>(v, ror(v, std::integral_constant<int, 0x124>{}));
    v = combine<MAX>(v, ror(v, std::integral_constant<int, 0x122>{}));
    v = combine<MAX>(v, ror(v, std::integral_constant<int, 0x121>{}));
    if (G == 64) {
        v = combine<MAX>(v, __shfl_xor(v, 16));
        v = combine<MAX>(v, __shfl_xor(v, 32));
    }
    return v;
}

// Loss and dz_t of the rows of one mini-batch, G lanes per row; dz_t takes the place of the row's logits.  N classes, Np
// columns of dz_t (zeros from N on); rows B .. Bz - 1 (padding of the 16-row tiles) become zero gradients.
template <typename D, int G>
__device__ inline void loss_rows(unsigned char *top, int pitch, const int32_t *Y, float *row_loss, int B, int Bz, int N, int Np)
{
    using E = typename D::T;
    constexpr int RPW = 64 / G;   // rows a wave handles together
    const int gl = (threadIdx.x & 63) % G, sub = (threadIdx.x & 63) / G, wave = threadIdx.x >> 6;
    const float invB = 1.0f / (float)B;
    for (int b0 = wave * RPW; b0 < Bz; b0 += kWaves * RPW) {
        const int b = b0 + sub;
        const bool in = b < B;
        unsigned char *row = top + (b < Bz ? b : b0) * pitch;
        const float *z = reinterpret_cast<const float *>(row);
        const int label = in ? Y[b] : -1;
        float mx = -INFINITY;
        for (int c = gl; c < N; c += G) mx = fmaxf(mx, z[c]);
        mx = group_reduce<G, true>(mx);
        float se = 0.0f;
        for (int c = gl; c < N; c += G) se += __expf(z[c] - mx);
        se = group_reduce<G, false>(se);
        const float zl = label >= 0 && label < N ? z[label] : mx, inv = 1.0f / se;
        for (int c = gl; c < Np; c += G) {   // (a wave's LDS accesses stay in order: what is overwritten was read)
            const float zc = z[c];
            __builtin_amdgcn_wave_barrier();
            if (b < Bz)
                reinterpret_cast<E *>(row)[c] =
                    D::cvt(in && c < N ? (__expf(zc - mx) * inv - (c == label ? 1.0f : 0.0f)) * invB : 0.0f);
            __builtin_amdgcn_wave_barrier();
        }
        if (in && gl == 0) row_loss[b] = __logf(se) + mx - zl;
    }
}

template <typename D>
__global__ __launch_bounds__(kThreads) void k_small_steps(SmallArgs a)
{
    using E = typename D::T;
    using T = Unit<D>;
    constexpr int ES = D::kBytes;
    __shared__ __attribute__((aligned(256))) unsigned char lds[kSmallLds];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int g = blockIdx.x, t = a.t, B = a.B;
    const int bt = (B + 15) / 16, bu = (B + T::U - 1) / T::U;   // 16-row tiles and k-step units of the batch
    const int top_pitch = a.layer[t - 1].pz;
    unsigned char *const X = lds + a.off_x;
    int32_t *const Y = reinterpret_cast<int32_t *>(lds + a.off_y);
    float *const row_loss = reinterpret_cast<float *>(lds + a.off_loss);

    // ---- everything in LDS starts as zero (padding stays zero), then the weights and biases ----
    for (int i = threadIdx.x; i < a.lds_bytes / 16; i += kThreads) reinterpret_cast<uint4 *>(lds)[i] = uint4{0, 0, 0, 0};
    __syncthreads();
#pragma unroll 1
    for (int l = 0; l < t; ++l) {
        const SmallLayer L = a.layer[l];
        const E *W = static_cast<const E *>(L.W) + (int64_t)g * L.R * L.C;
        for (int c = lane; c < L.C; c += 64)
            for (int r = wave; r < L.R; r += 4 * kWaves) {   // four rows requested together
                E v[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) v[u] = r + u * kWaves < L.R ? W[(int64_t)(r + u * kWaves) * L.C + c] : E(0);
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (r + u * kWaves < L.R) *reinterpret_cast<E *>(lds + L.off_w + (r + u * kWaves) * L.pw + c * ES) = v[u];
            }
        if (L.bias)
            for (int r = threadIdx.x; r < L.R; r += kThreads)
                reinterpret_cast<E *>(lds + L.off_b)[r] = static_cast<const E *>(L.bias)[(int64_t)g * L.R + r];
    }

    // ---- mini-batches: pieces of 64 values, wave w takes pieces w, w + 16, ... ----
    const int N0 = a.layer[0].C, xcpr = (N0 + 63) / 64, xpieces = B * xcpr;
    E xr[kXRegs];
    int32_t yr = 0;
    auto x_rows = [&](int j) { return static_cast<const E *>(a.x) + ((int64_t)g * a.stride_s + (int64_t)j * a.stride_k) * N0; };
    auto x_request = [&](int j) {
        const E *xb = x_rows(j);
#pragma unroll
        for (int i = 0; i < kXRegs; ++i) {
            if (kWaves * i >= xpieces) break;
            const int q = wave + kWaves * i, b = tile_row(q, a.mx), c = (q - b * xcpr) * 64 + lane;
            xr[i] = (q < xpieces && c < N0) ? xb[(int64_t)b * N0 + c] : E(0);
        }
        if ((int)threadIdx.x < B) yr = a.y[(int64_t)g * a.stride_s + (int64_t)j * a.stride_k + threadIdx.x];
    };
    auto x_store = [&](int j) {
#pragma unroll
        for (int i = 0; i < kXRegs; ++i) {
            if (kWaves * i >= xpieces) break;
            const int q = wave + kWaves * i, b = tile_row(q, a.mx), c = (q - b * xcpr) * 64 + lane;
            if (q < xpieces && c < N0) *reinterpret_cast<E *>(X + b * a.px + c * ES) = xr[i];
        }
        const E *xb = x_rows(j);   // a mini-batch of more than 16 * kXRegs pieces: the rest straight from memory
        for (int q0 = wave + kWaves * kXRegs; q0 < xpieces; q0 += 4 * kWaves) {
            E v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int q = q0 + u * kWaves, b = q / xcpr, c = (q - b * xcpr) * 64 + lane;
                v[u] = q < xpieces && c < N0 ? xb[(int64_t)b * N0 + c] : E(0);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int q = q0 + u * kWaves, b = q / xcpr, c = (q - b * xcpr) * 64 + lane;
                if (q < xpieces && c < N0) *reinterpret_cast<E *>(X + b * a.px + c * ES) = v[u];
            }
        }
        if ((int)threadIdx.x < B) Y[threadIdx.x] = yr;
        for (int b = kThreads + (int)threadIdx.x; b < B; b += kThreads)
            Y[b] = a.y[(int64_t)g * a.stride_s + (int64_t)j * a.stride_k + b];
    };
    x_request(0);
    x_store(0);
    __syncthreads();

    // W_l <- W_l - lr dz_l^T h_{l-1}: this wave's tiles i, i + 16, ... of layer l; i ends as the index into what comes next
    auto update = [&](int l, int &i) {
        const SmallLayer L = a.layer[l];
        const int ct = (L.C + 15) / 16, n = ct * ((L.R + 15) / 16);
        const unsigned char *h = l ? lds + a.layer[l - 1].off_h : X;
        const int ph = l ? a.layer[l - 1].ph : a.px;
        for (; i < n; i += kWaves) {
            const int q = tile_row(i, L.mc), r0 = 16 * q, c0 = 16 * (i - q * ct);
            const f32x4 d = tile<D, KS, KS>(lds + L.off_dz, L.pz, r0, h, ph, c0, bu, lane);
            unsigned char *p = lds + L.off_w + (r0 + (lane & 15)) * L.pw + (c0 + 4 * (lane >> 4)) * ES;
            f32x4 w = T::ld4(p);
#pragma unroll
            for (int e = 0; e < 4; ++e) w[e] -= L.lr * d[e];
            T::st4(p, w);
        }
        i -= n;
    };

    for (int j = 0; j < a.k; ++j) {
        // ---- forward ----
#pragma unroll 1
        for (int l = 0; l < t; ++l) {
            const SmallLayer L = a.layer[l];
            const unsigned char *h = l ? lds + a.layer[l - 1].off_h : X;
            const int ph = l ? a.layer[l - 1].ph : a.px;
            const int rt = (L.R + 15) / 16, nu = (L.C + T::U - 1) / T::U;
            for (int i = wave; i < bt * rt; i += kWaves) {
                const int q = tile_row(i, L.mr), b0 = 16 * q, r0 = 16 * (i - q * rt);
                const f32x4 z = tile<D, KC, KC>(h, ph, b0, lds + L.off_w, L.pw, r0, nu, lane);
                const int row = b0 + (lane & 15), col = r0 + 4 * (lane >> 4);
                const f32x4 bv = T::ld4(lds + L.off_b + col * ES);
                f32x4 o;
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = fmaf(L.alpha, z[e], bv[e]);
                if (l == t - 1) {
                    Unit<F32>::st4(lds + L.off_dz + row * L.pz + col * 4, o);   // logits (fp32) where dz_t will stand
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[e] = o[e] > 0.0f ? o[e] : 0.0f;
                    T::st4(lds + L.off_h + row * L.ph + col * ES, o);
                }
            }
            __syncthreads();
        }
        if (j + 1 < a.k) x_request(j + 1);
        {
            const int N = a.layer[t - 1].R, Np = (N + T::U - 1) / T::U * T::U;
            unsigned char *top = lds + a.layer[t - 1].off_dz;
            if (Np <= 32) loss_rows<D, 16>(top, top_pitch, Y, row_loss, B, 16 * bt, N, Np);
            else loss_rows<D, 64>(top, top_pitch, Y, row_loss, B, 16 * bt, N, Np);
        }
        __syncthreads();
        // ---- back through the layers; the update of layer l + 1 shares a phase with the step through layer l ----
#pragma unroll 1
        for (int l = t - 1; l >= 1; --l) {
            const SmallLayer L = a.layer[l];
            const unsigned char *h = lds + a.layer[l - 1].off_h;
            unsigned char *dz = lds + a.layer[l - 1].off_dz;
            const int ph = a.layer[l - 1].ph, pz = a.layer[l - 1].pz;
            const int ct = (L.C + 15) / 16, nu = (L.R + T::U - 1) / T::U, n = bt * ct;
            int i = wave;
            for (; i < n; i += kWaves) {
                const int q = tile_row(i, L.mc), b0 = 16 * q, c0 = 16 * (i - q * ct);
                const f32x4 d = tile<D, KC, KS>(lds + L.off_dz, L.pz, b0, lds + L.off_w, L.pw, c0, nu, lane);
                const int row = b0 + (lane & 15), col = c0 + 4 * (lane >> 4);
                const f32x4 hv = T::ld4(h + row * ph + col * ES);
                f32x4 o;
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = hv[e] > 0.0f ? L.alpha * d[e] : 0.0f;
                T::st4(dz + row * pz + col * ES, o);
            }
            i -= n;
            if (l + 1 < t) update(l + 1, i);
            if (l == t - 1 && wave == kWaves - 1 && a.loss_out) {   // mean of the row losses
                float s = 0.0f;
                for (int b = lane; b < B; b += 64) s += row_loss[b];
#pragma unroll
                for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
                if (lane == 0) a.loss_out[(int64_t)g * a.k + j] = s / (float)B;
            }
            __syncthreads();
        }
        // ---- the remaining updates (layers 2 and 1) and all biases ----
        {
            int i = wave;
#pragma unroll 1
            for (int l = 1; l >= 0; --l) update(l, i);
            int job = kWaves - 1 - wave;   // 64 columns a job, from the wave that has the fewest tiles
#pragma unroll 1
            for (int l = 0; l < t; ++l) {
                const SmallLayer L = a.layer[l];
                const int jobs = L.bias ? (L.R + 63) / 64 : 0;
                for (; job < jobs; job += kWaves) {
                    const int r = job * 64 + lane;
                    if (r >= L.R) continue;
                    const unsigned char *p0 = lds + L.off_dz + r * ES;
                    float s = 0.0f;
                    int b = 0;
                    for (; b + 16 <= B; b += 16) {   // sixteen rows' reads in flight
                        float v[16];
#pragma unroll
                        for (int u = 0; u < 16; ++u) v[u] = D::ld(reinterpret_cast<const E *>(p0 + (b + u) * L.pz));
#pragma unroll
                        for (int u = 0; u < 16; ++u) s += v[u];
                    }
                    for (; b < B; ++b) s += D::ld(reinterpret_cast<const E *>(p0 + b * L.pz));
                    E *p = reinterpret_cast<E *>(lds + L.off_b) + r;
                    *p = D::cvt(D::up(*p) - a.lr * s);
                }
                job -= jobs;
            }
        }
        __syncthreads();
        if (j + 1 < a.k) {
            x_store(j + 1);
            __syncthreads();
        }
    }

    // ---- weights and biases back ----
#pragma unroll 1
    for (int l = 0; l < t; ++l) {
        const SmallLayer L = a.layer[l];
        E *W = static_cast<E *>(L.W) + (int64_t)g * L.R * L.C;
        for (int r = wave; r < L.R; r += kWaves)
            for (int c = lane; c < L.C; c += 64)
                W[(int64_t)r * L.C + c] = *reinterpret_cast<const E *>(lds + L.off_w + r * L.pw + c * ES);
        if (L.bias)
            for (int r = threadIdx.x; r < L.R; r += kThreads)
                static_cast<E *>(L.bias)[(int64_t)g * L.R + r] = reinterpret_cast<const E *>(lds + L.off_b)[r];
    }
}

}  // namespace small

// LDS layout for a batch of a.B samples; false if the subnet does not fit.
static bool small_layout(SmallArgs &a, int esz)
{
    const int U = esz == 2 ? 32 : 16;
    auto up = [](int64_t x, int64_t m) { return (x + m - 1) / m * m; };
    int64_t off = 0;
    auto take = [&](int64_t bytes) { const int64_t o = off; off = up(off + bytes, 16); return (int32_t)std::min<int64_t>(o, kSmallLds); };
    const int64_t Bp = up(a.B, U);
    a.px = (int32_t)up((int64_t)a.layer[0].C, U) * esz + 16;
    a.off_x = take(Bp * a.px);
    for (int l = 0; l < a.t; ++l) {
        SmallLayer &L = a.layer[l];
        const int64_t Rp = up(L.R, U), Cp = up(L.C, U);
        if (Rp > kSmallLds || Cp > kSmallLds) return false;
        L.mr = (int32_t)(((1 << 20) + (L.R + 15) / 16 - 1) / ((L.R + 15) / 16));
        L.mc = (int32_t)(((1 << 20) + (L.C + 15) / 16 - 1) / ((L.C + 15) / 16));
        L.pw = (int32_t)(Cp * esz + 16);
        L.off_w = take(Rp * L.pw);
        L.off_b = take(Rp * esz);
        L.ph = (int32_t)(Rp * esz + 16);
        L.pz = (int32_t)((l == a.t - 1 ? Rp * 4 : Rp * esz) + 16);   // the top layer's rows hold fp32 logits first
        L.off_h = l == a.t - 1 ? 0 : take(Bp * L.ph);
        L.off_dz = take(Bp * L.pz);
        if (off > kSmallLds) return false;
    }
    const int32_t cpr = (a.layer[0].C + 63) / 64;
    a.mx = ((1 << 20) + cpr - 1) / cpr;
    a.off_y = take(4 * (int64_t)a.B);
    a.off_loss = take(4 * (int64_t)a.B);
    a.lds_bytes = (int32_t)off;
    return off <= kSmallLds;
}

// Every shape that fits was measured faster than the launch per product: 70 random ones (2 .. 4 layers, 1 .. 8 subnets,
// 8 .. 230 samples, 9 .. 155 KB of LDS, 10 steps) by factors of 2.1 .. 6.9, the least near the LDS limit in f32.  More
// subnets than compute units queue up behind each other, which the per-product launches do not: two rounds of
// workgroups are allowed, the least of those factors.
bool small_steps_fit(SmallArgs &a, int dtype)
{
    if (a.t > kSmallLayers || a.B < 1 || a.G > 2 * 256) return false;
    return small_layout(a, dtype == IST_BF16 ? 2 : 4);
}

hipError_t launch_small_steps(const SmallArgs &a, int dtype, hipStream_t st)
{
    double w = 0.0;
    for (int l = 0; l < a.t; ++l) w += (double)a.layer[l].R * a.layer[l].C;
    const double esz = dtype == IST_BF16 ? 2.0 : 4.0;
    tag_kernel(dtype == IST_BF16 ? "k_small_steps_bf16" : "k_small_steps_f32", 0.0,
               a.G * esz * (2.0 * w + (double)a.k * a.B * a.layer[0].C));
    const dim3 grid((unsigned)a.G), block(small::kThreads);
    if (dtype == IST_BF16) hipLaunchKernelGGL(small::k_small_steps<BF16>, grid, block, 0, st, a);
    else hipLaunchKernelGGL(small::k_small_steps<F32>, grid, block, 0, st, a);
    return hipGetLastError();
}

}  // namespace ist
