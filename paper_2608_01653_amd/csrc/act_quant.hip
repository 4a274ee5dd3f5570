// Activation transform + per-sample absmax + INT8 quantization (steps a2-a4).
//
// The input of one sample is a flat fp32 array of E = h*w*c elements (NHWC).
// With c % b == 0 every Hadamard block (b consecutive channels of one pixel) is
// b-aligned in the flat array, so the kernel tiles the array into "items" of
// I = max(64, b) consecutive floats without looking at pixel boundaries.
//
// One quad (4 lanes) owns one item.  Lane t of the quad holds the channels
// c = 16*i + 4*t + j (j = 0..3 inside a float4, i = 0..I/16-1): bits 0-1 of
// the channel index are inside a float4, bits 2-3 are the lane, bits 4+ are the
// register index.  Loads are 64 contiguous bytes per quad per instruction.
//
// Two kernels:
//   absmax_kernel: transform, max |S| per sample (one value per block, into the
//   sample's slots).
//   quant_kernel : transform again, quantize with s = fl32(A / 127), store codes.
// When the producer of x already computed A (next_absmax of the convolution),
// only quant_kernel runs and x is read once.
#include <mutex>
#include <type_traits>

#include "hatq_device.h"
#include "hatq_launch.h"

// Scratch of the no-allocation entry point: the per-sample absmax of the
// two-pass quantization for callers that cannot allocate.  Every GPU the
// library runs on holds its own copy until the process ends.  In host code the
// name is a stand-in, not a device address: the address comes from
// hipGetSymbolAddress, looked up once per device (scratch_absmax below).
static __device__ __align__(256) float scratch[hatq::kNoAllocMaxSamples * hatq::kAbsSlots];

namespace hatq {

__global__ void fill_u32_kernel(uint32_t *p, int n, uint32_t v) {
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) p[i] = v;
}

namespace {

constexpr int kThreads = 256;
constexpr int kQuadsPerBlock = kThreads / 4;
template <int B>
__device__ __forceinline__ void load_item(const float *xs, int64_t base, int64_t E, int t,
                                          float (&v)[4 * ItemShape<B>::R]) {
    constexpr int R = ItemShape<B>::R;
    constexpr int I = ItemShape<B>::I;
    const bool full = base + I <= E;
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const int64_t off = base + 16 * i + 4 * t;
        float4 f = make_float4(0.f, 0.f, 0.f, 0.f);
        if (full || off < E) f = *reinterpret_cast<const float4 *>(xs + off);
        v[4 * i + 0] = f.x;
        v[4 * i + 1] = f.y;
        v[4 * i + 2] = f.z;
        v[4 * i + 3] = f.w;
    }
}

// The reductions (absmax, min/max, range): blocks of RT threads, f(item) for
// every item of a sample the quad takes, its values in registers; the loads of U items
// are issued before the first is used.  From the sample's end (FWD: from its
// beginning); launch shapes below.
template <int B, int RT, int U, bool FWD, typename F>
__device__ __forceinline__ void for_items(const float *xs, int64_t E, int t, F &&f) {
    constexpr int I = ItemShape<B>::I, R = ItemShape<B>::R;
    const int64_t items = (E + I - 1) / I, step = (int64_t)gridDim.x * (RT / 4);
    int64_t it = (int64_t)blockIdx.x * (RT / 4) + (threadIdx.x >> 2);
    for (; it + (U - 1) * step < items; it += U * step) {
        float v[U][4 * R];
#pragma unroll
        for (int u = 0; u < U; ++u) load_item<B>(xs, (FWD ? it + u * step : items - 1 - it - u * step) * I, E, t, v[u]);
#pragma unroll
        for (int u = 0; u < U; ++u) f(v[u]);
    }
    if constexpr (U > 1) {
        for (; it < items; it += step) {
            float v[4 * R];
            load_item<B>(xs, (FWD ? it : items - 1 - it) * I, E, t, v);
            f(v);
        }
    }
}

// Maximum over the block of each thread's N values, one atomic per value and
// block: out[k] holds the address of value k.  own: the block is the only one that
// writes there, and the memory need not hold anything before.
template <int RT, int N>
__device__ __forceinline__ void block_max(const float (&m)[N], float *const (&out)[N], bool own = false) {
    __shared__ float red[N][RT / 64];
    // (the values' lane exchanges side by side: one after the other they were 0.3 us
    // of a small launch)
    float wm[N];
#pragma unroll
    for (int k = 0; k < N; ++k) wm[k] = wave_max(m[k]);
    if ((threadIdx.x & 63) == 0) {
#pragma unroll
        for (int k = 0; k < N; ++k) red[k][threadIdx.x >> 6] = wm[k];
    }
    __syncthreads();
    if (threadIdx.x < N) {
        float b = red[threadIdx.x][0];
#pragma unroll
        for (int w = 1; w < RT / 64; ++w) b = fmaxf(b, red[threadIdx.x][w]);
        float *dst = out[0];
#pragma unroll
        for (int k = 1; k < N; ++k) dst = threadIdx.x == k ? out[k] : dst;
        if (own) *dst = b;
        else atomic_max_nonneg(dst, b);
    }
}

// Maximum of a sample's slots (at most 64, non-negative): a slot per lane; read one
// after the other they took 3 us before a block's first load.
__device__ __forceinline__ float slots_max(const float *p, int slots) {
    if (slots == 1) return *p;
    const int lane = threadIdx.x & 63;
    return wave_max(lane < slots ? p[lane] : 0.0f);
}

template <int B, int RT, int U, bool FWD>
__global__ void __launch_bounds__(RT) absmax_kernel(const float *__restrict__ x, int64_t E,
                                                    float *__restrict__ absmax, int own) {
    // from the end of the batch: the codes pass then reads from its beginning,
    // where this pass's last reads are still in the 256 MB memory-side cache
    const int n = FWD ? blockIdx.y : gridDim.y - 1 - blockIdx.y, t = threadIdx.x & 3;
    float m[1] = {0.0f};
    for_items<B, RT, U, FWD>(x + (int64_t)n * E, E, t, [&](auto &v) {
        fwht_item<B>(v, t);
#pragma unroll
        for (float e : v) m[0] = fmaxf(m[0], fabsf(e));
    });
    block_max<RT, 1>(m, {absmax + (int64_t)n * kAbsSlots + blockIdx.x % kAbsSlots}, own != 0);
}

// The same for blocks of 1 (no transform): max |x| over the sample read as
// float4 (E % 4 == 0), four loads per thread in flight per iteration.
template <int RT>
__global__ void __launch_bounds__(RT) absmax_flat_kernel(const float *__restrict__ x, int64_t E,
                                                         float *__restrict__ absmax, int own) {
    const int n = gridDim.y - 1 - blockIdx.y;   // from the end, as absmax_kernel
    const int64_t E4 = E >> 2;
    const float4 *xs = reinterpret_cast<const float4 *>(x + (int64_t)n * E) + (E4 - 1);
    const int64_t stride = (int64_t)gridDim.x * RT;
    int64_t i = (int64_t)blockIdx.x * RT + threadIdx.x;
    auto m4 = [](float m, const float4 &f) {
        return fmaxf(fmaxf(fmaxf(m, fabsf(f.x)), fabsf(f.y)), fmaxf(fabsf(f.z), fabsf(f.w)));
    };
    float m = 0.0f;
    for (; i + 3 * stride < E4; i += 4 * stride) {
        const float4 a = xs[-i], b = xs[-i - stride], c = xs[-i - 2 * stride], d = xs[-i - 3 * stride];
        m = m4(m4(m4(m4(m, a), b), c), d);
    }
    for (; i < E4; i += stride) m = m4(m, xs[-i]);
    const float mm[1] = {m};
    block_max<RT, 1>(mm, {absmax + (int64_t)n * kAbsSlots + blockIdx.x % kAbsSlots}, own != 0);
}

// Items per quad per loop iteration (all their loads issued before first use).
#ifndef HATQ_QUANT_UN
#define HATQ_QUANT_UN 1
#endif
template <int B>
struct QuantUnroll {
    // two items in flight per quad: the untransformed 3-channel image's two-pass
    // quantization 80.5 -> 77.3 us; with blocks of 64, 178 -> 182 us
    static constexpr int UN = B == 1 ? 2 : HATQ_QUANT_UN;
};

// Quantize one transformed item (s = act scale, r = fl(1/s)) and store its codes.
// cc > 0: codes in the chunk-major layout of a sample of cc channels (items of
// 64 channels, cc % 64 == 0): the item of pixel p, channels 64m .. 64m + 63, goes
// to ((m * (E / cc)) + p) * 64.
template <int B>
__device__ __forceinline__ void quant_store_item(const float (&vin)[4 * ItemShape<B>::R], int8_t *qs, int64_t base,
                                                 int64_t E, int t, float s, float r, bool fast_ok, float sigma,
                                                 int cc) {
    constexpr int R = ItemShape<B>::R;
    constexpr int I = ItemShape<B>::I;
    static_assert(R % 4 == 0, "groups of four words");
    const float rs = sigma * r;
    uint32_t u[4 * R];
    bool near = !fast_ok;
#pragma unroll
    for (int k = 0; k < 4 * R; ++k) {
        const float tq = clamp127(vin[k] * rs);
        const float uf = tq + HATQ_MAGIC;
        const float kf = uf - HATQ_MAGIC;
        near |= fabsf(tq - kf) > HATQ_NEAR_TIE;
        u[k] = __float_as_uint(uf);
    }
    if (near) {
#pragma unroll
        for (int k = 0; k < 4 * R; ++k) {
            const float q = rintf(clamp127((sigma * vin[k]) / s));
            u[k] = __float_as_uint(q + HATQ_MAGIC);
        }
    }
    const bool full = base + I <= E;
    if (full) {
        // Word i of lane t holds channels 16i + 4t .. +3.  A 4 x 4 transpose of
        // words inside the quad (two DPP swap stages) gives lane t channels
        // 64g + 16t .. +15 of each group g of four words, so every lane stores
        // 16 contiguous bytes and the wave 1 KB per group.
#pragma unroll
        for (int g = 0; g < R / 4; ++g) {
            int w[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int k = 4 * (4 * g + i);
                w[i] = (int)pack_low_bytes(u[k], u[k + 1], u[k + 2], u[k + 3]);
            }
            int x[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) x[i] = __builtin_amdgcn_mov_dpp(w[i ^ 1], 0xB1, 0xF, 0xF, true);   // lane ^ 1
#pragma unroll
            for (int i = 0; i < 4; ++i) w[i] = ((t ^ i) & 1) ? x[i] : w[i];
#pragma unroll
            for (int i = 0; i < 4; ++i) x[i] = __builtin_amdgcn_mov_dpp(w[i ^ 2], 0x4E, 0xF, 0xF, true);   // lane ^ 2
#pragma unroll
            for (int i = 0; i < 4; ++i) w[i] = ((t ^ i) & 2) ? x[i] : w[i];
            int8_t *dst = qs + base + 64 * g + 16 * t;
            if (I == 64 && cc > 0) {
                const int64_t p = base / cc;
                dst = qs + (((base - p * cc) >> 6) * (E / cc) + p) * 64 + 16 * t;
            }
            // (xq need only be 4-byte aligned and a sample's E only a multiple
            // of 4; base is a multiple of 64, so the sample's start decides,
            // uniformly for the block)
            if ((reinterpret_cast<uintptr_t>(qs) & 15) == 0) {
                // streaming store: the codes are read by the next convolution,
                // not by this kernel, so they bypass the caches on the way out
                // (782 -> 716 us on the 805 M-element tensor)
                __builtin_nontemporal_store(v4i{w[0], w[1], w[2], w[3]}, reinterpret_cast<v4i *>(dst));
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) reinterpret_cast<int *>(dst)[i] = w[i];
            }
        }
        return;
    }
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const int64_t off = base + 16 * i + 4 * t;
        if (off < E)
            *reinterpret_cast<uint32_t *>(qs + off) = pack_low_bytes(u[4 * i], u[4 * i + 1], u[4 * i + 2], u[4 * i + 3]);
    }
}

template <int B>
__global__ void __launch_bounds__(kThreads) quant_kernel(const float *__restrict__ x, int64_t E,
                                                         const float *__restrict__ absmax,
                                                         int8_t *__restrict__ xq,
                                                         float *__restrict__ act_scale, int cc, int slots, int stride) {
    constexpr int I = ItemShape<B>::I;
    constexpr int R = ItemShape<B>::R;
    constexpr int UN = QuantUnroll<B>::UN;
    // Sample order: when the batch splits evenly over the 8 XCDs, the window
    // convolution that usually produced x gave XCD k the samples k g .. k g +
    // g - 1 (g = n / 8) and finished their last ones last, so the launch takes
    // samples last-finished first and reads each from its end: its first reads
    // meet the lines most recently written, still in the 256 MB memory-side
    // cache (layer 3's 201 M-element input: 188 -> 181 us).  After this call's
    // own absmax pass (stride > 1), which reads from the end of the batch, the
    // beginning is what was read last.  Any order gives the same codes.
    const int ns = gridDim.y;
    int n = blockIdx.y;
    const bool rev = ns % 8 == 0 && stride == 1;
    if (rev) {
        const int g = ns / 8, j = g - 1 - n / 8, k = n % 8;
        n = k * g + j;
    }
    const float *xs = x + (int64_t)n * E;
    int8_t *qs = xq + (int64_t)n * E;
    const int t = threadIdx.x & 3;
    // the sample's absmax: one value (given), or the maximum of its slots
    const float s = act_scale_from_absmax(slots_max(absmax + (int64_t)n * stride, slots));
    if (blockIdx.x == 0 && threadIdx.x == 0) act_scale[n] = s;
    const float r = 1.0f / s;
    // The fast path needs r and every t finite and normal-range; a scale below
    // 2^-125 or above 2^125 takes the exact division for every element.
    const bool fast_ok = s >= 0x1p-125f && s <= 0x1p125f;
    const int64_t items = (E + I - 1) / I;
    const int64_t step = (int64_t)gridDim.x * kQuadsPerBlock;
    for (int64_t it0 = (int64_t)blockIdx.x * kQuadsPerBlock * UN + (threadIdx.x >> 2); it0 < items;
         it0 += step * UN) {
        float v[UN][4 * R];
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const int64_t it = it0 + u * kQuadsPerBlock;
            if (it < items) load_item<B>(xs, (rev ? items - 1 - it : it) * I, E, t, v[u]);
        }
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const int64_t it = it0 + u * kQuadsPerBlock;
            if (it >= items) break;
            const float sigma = fwht_item<B>(v[u], t);
            quant_store_item<B>(v[u], qs, (rev ? items - 1 - it : it) * I, E, t, s, r, fast_ok, sigma, cc);
        }
    }
}

// ---- affine quantization (Eq. affine_q, Eq. uniform_q) ----------------------
// Signed grid [-128, 127].  amax[k] = max(max S, 0), amax[n + k] = max(-min S, 0)
// (both non-negative, so the order-preserving atomic serves both).
template <int B, int RT, int U, bool FWD>
__global__ void __launch_bounds__(RT) minmax_kernel(const float *__restrict__ x, int64_t E,
                                                    float *__restrict__ amax) {
    const int k = FWD ? blockIdx.y : gridDim.y - 1 - blockIdx.y, t = threadIdx.x & 3;
    float m[2] = {0.0f, 0.0f};   // max(S, 0) and max(-S, 0)
    for_items<B, RT, U, FWD>(x + (int64_t)k * E, E, t, [&](auto &v) {
        const float sigma = fwht_item<B>(v, t);
#pragma unroll
        for (float e : v) {
            const float sv = sigma * e;
            m[0] = fmaxf(m[0], sv);
            m[1] = fmaxf(m[1], -sv);
        }
    });
    block_max<RT, 2>(m, {amax + k, amax + gridDim.y + k});
}

// s = fl32(fl32(hi + lo) / 255) and z = clamp(rne(fl32(lo / s)) - 128) for a
// nonzero range (hi + lo = xmax' - xmin'), else s = 1, z = 0.
__device__ __forceinline__ void affine_params(float hi, float lo, float &s, int &z) {
    const float r = hi + lo;
    s = 1.0f;
    z = 0;
    if (r > 0.0f) {
        s = r / 255.0f;
        z = (int)rintf(lo / s) - 128;
        z = z < -128 ? -128 : (z > 127 ? 127 : z);
    }
}

// Codes q = clamp(rne(fl32(S / s)) + z, -128, 127), IEEE division per element.
template <int B>
__global__ void __launch_bounds__(kThreads) quant_affine_kernel(const float *__restrict__ x, int64_t E,
                                                                const float *__restrict__ amax,
                                                                int8_t *__restrict__ xq, float *__restrict__ act_scale,
                                                                int32_t *__restrict__ act_zero) {
    constexpr int I = ItemShape<B>::I;
    constexpr int R = ItemShape<B>::R;
    const int k = blockIdx.y;
    const float *xs = x + (int64_t)k * E;
    int8_t *qs = xq + (int64_t)k * E;
    const int t = threadIdx.x & 3;
    float s;
    int z;
    affine_params(amax[k], amax[gridDim.y + k], s, z);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        act_scale[k] = s;
        act_zero[k] = z;
    }
    const float zf = (float)z;
    const int64_t items = (E + I - 1) / I;
    for (int64_t it = (int64_t)blockIdx.x * kQuadsPerBlock + (threadIdx.x >> 2); it < items;
         it += (int64_t)gridDim.x * kQuadsPerBlock) {
        float v[4 * R];
        load_item<B>(xs, it * I, E, t, v);
        const float sigma = fwht_item<B>(v, t);
        uint32_t u[4 * R];
#pragma unroll
        for (int r = 0; r < 4 * R; ++r) {
            const float q = __builtin_amdgcn_fmed3f(rintf((sigma * v[r]) / s) + zf, -128.0f, 127.0f);
            u[r] = (uint32_t)(int32_t)q;
        }
        const int64_t base = it * I;
        const bool full = base + I <= E;
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const int64_t off = base + 16 * i + 4 * t;
            if (full || off < E)
                *reinterpret_cast<uint32_t *>(qs + off) = pack_low_bytes(u[4 * i], u[4 * i + 1], u[4 * i + 2], u[4 * i + 3]);
        }
    }
}

// ---- range-expansion profiling (Eq. hadamard_sensitivity) -------------------
// One read of x gives both maxima of each sample: max |x| (into amax[k]) and
// max |S| of the same butterfly the quantizer applies (into amax[n + k]).
template <int B, int RT, int U>
__global__ void __launch_bounds__(RT) range_kernel(const float *__restrict__ x, int64_t E,
                                                   float *__restrict__ amax) {
    const int k = blockIdx.y, t = threadIdx.x & 3;
    float m[2] = {0.0f, 0.0f};   // max |x| and max |S|
    for_items<B, RT, U, false>(x + (int64_t)k * E, E, t, [&](auto &v) {
#pragma unroll
        for (float e : v) m[0] = fmaxf(m[0], fabsf(e));
        fwht_item<B>(v, t);
#pragma unroll
        for (float e : v) m[1] = fmaxf(m[1], fabsf(e));
    });
    block_max<RT, 2>(m, {amax + k, amax + gridDim.y + k});
}

// Channels not a multiple of the block (or a ragged sample): one thread per
// (pixel, block), zero channels past C, the same ascending-bit butterfly in
// registers.
template <int B>
__global__ void __launch_bounds__(kThreads) range_pad_kernel(const float *__restrict__ x, int64_t P, int C,
                                                             float *__restrict__ amax) {
    const int k = blockIdx.y;
    const float *xs = x + (int64_t)k * P * C;
    const int nblk = (C + B - 1) / B;
    float mx = 0.0f, mh = 0.0f;
    for (int64_t u = (int64_t)blockIdx.x * kThreads + threadIdx.x; u < P * nblk; u += (int64_t)gridDim.x * kThreads) {
        const int64_t px = u / nblk;
        const int c0 = (int)(u - px * nblk) * B;
        float v[B];
#pragma unroll
        for (int j = 0; j < B; ++j) {
            v[j] = c0 + j < C ? xs[px * C + c0 + j] : 0.0f;
            mx = fmaxf(mx, fabsf(v[j]));
        }
#pragma unroll
        for (int h = 1; h < B; h <<= 1)
#pragma unroll
            for (int j = 0; j < B; ++j) {
                if (j & h) continue;
                const float a = v[j], c = v[j + h];
                v[j] = a + c;
                v[j + h] = a - c;
            }
#pragma unroll
        for (int j = 0; j < B; ++j) mh = fmaxf(mh, fabsf(v[j]));
    }
    mx = wave_max(mx);
    mh = wave_max(mh);
    __shared__ float red[2][kThreads / 64];
    if ((threadIdx.x & 63) == 0) {
        red[0][threadIdx.x >> 6] = mx;
        red[1][threadIdx.x >> 6] = mh;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        float b = red[threadIdx.x][0];
#pragma unroll
        for (int w = 1; w < kThreads / 64; ++w) b = fmaxf(b, red[threadIdx.x][w]);
        atomic_max_nonneg(amax + (threadIdx.x ? gridDim.y : 0) + k, b);
    }
}

// The indicator of each sample: max|S|^2 > b max|x|^2, exact in fp64 (the
// orthonormal transform is S / sqrt(b)); the expanding samples are counted.
__global__ void expansion_flags_kernel(const float *__restrict__ amax, int n, int b, int32_t *flags,
                                       int32_t *count) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    const double mx = amax[k], mh = amax[n + k];
    const int f = mh * mh > (double)b * (mx * mx);
    if (flags) flags[k] = f;
    if (count && f) atomicAdd(count, 1);
}

// Elementwise path for b <= 2 when E is not a multiple of 4 (float4 alignment
// of every sample cannot be assumed).  Element pairs never straddle a pixel
// because c % b == 0.
template <int B, bool QUANT>
__global__ void __launch_bounds__(kThreads) scalar_kernel(const float *__restrict__ x, int64_t E,
                                                          float *__restrict__ absmax,
                                                          int8_t *__restrict__ xq,
                                                          float *__restrict__ act_scale) {
    const int n = blockIdx.y;
    const float *xs = x + (int64_t)n * E;
    float s = 1.0f;
    if constexpr (QUANT) {
        s = act_scale_from_absmax(absmax[n]);
        if (blockIdx.x == 0 && threadIdx.x == 0) act_scale[n] = s;
    }
    float m = 0.0f;
    const int64_t groups = E / B;
    for (int64_t g = (int64_t)blockIdx.x * kThreads + threadIdx.x; g < groups;
         g += (int64_t)gridDim.x * kThreads) {
        float v[B];
#pragma unroll
        for (int j = 0; j < B; ++j) v[j] = xs[g * B + j];
        if constexpr (B == 2) {
            const float a = v[0], c = v[1];
            v[0] = a + c;
            v[1] = a - c;
        }
#pragma unroll
        for (int j = 0; j < B; ++j) {
            if constexpr (QUANT) xq[(int64_t)n * E + g * B + j] = (int8_t)(int)rintf(clamp127(v[j] / s));
            else m = fmaxf(m, fabsf(v[j]));
        }
    }
    if constexpr (!QUANT) {
        m = wave_max(m);
        if ((threadIdx.x & 63) == 0) atomic_max_nonneg(absmax + n, m);
    }
}

// Blocks per sample: enough for the work, at most `total` over the whole batch.
// Blocks of the quantization kernels over the whole batch (measured on the
// 805 M-element layer-2-shaped tensor: 16384 -> 32768 blocks 801 -> 782 us,
// 65536 no faster; on the 201 M-element one, blocks of 64, single read:
// 32768 -> 65536 blocks 175 -> 167 us NHWC, 178 -> 175 us chunk-major).
#ifndef HATQ_QUANT_GRID
#define HATQ_QUANT_GRID 65536
#endif
int grid_x(int64_t work_units, int per_block, int n, int total = HATQ_QUANT_GRID) {
    int64_t want = (work_units + per_block - 1) / per_block;
    int64_t cap = (total + n - 1) / n;
    if (cap < 1) cap = 1;
    if (want > cap) want = cap;
    return (int)(want < 1 ? 1 : want);
}

// Launch shapes of the reductions.  They are bound by memory, or, for small samples,
// by their start and end: the blocks end in one atomic per value on an address that
// all blocks of a sample share (or its slots), some 7 ns each, one after the other.
// So up to order 128 at most 512 blocks of 1024 threads (two per CU) over the batch;
// with up to 4096 blocks of 256 (2048 for min/max and range) the range pass of one 50 MB
// sample of order 64 took 33 us, now 17, the absmax and codes passes 37, now 25.  Small
// samples take fewer threads: range of 3.1 MB 8.4 (256), 7.5 (512), 7.6 us (1024).  The
// orders 192 and 320 (48 and 80 values per lane) hold fewer waves per CU, and with 1024
// threads most of them wait for the slowest: absmax and codes of order 192, 12.6 MB, 15.0
// (256), 15.6 (512), 18.0 us (1024), 64 samples of 1.8 MB 56 / 57 / 67; order 320, 32
// samples of 2.9 MB 65 / 75 / 81.
// Blocks per sample: one per RT / 4 items, `total` over the whole batch at most, none
// left over for a round of their own (513 blocks of order 128 over three samples of
// 98 MB: range 61 us, 510: 57).
constexpr int kRedGrid = 512;
int red_blocks(int64_t work_units, int per_block, int n, int total = kRedGrid) {
    const int64_t want = (work_units + per_block - 1) / per_block, cap = total / n > 0 ? total / n : 1;
    return (int)(want < 1 ? 1 : want < cap ? want : cap);
}

// The reduction before a codes pass of an order of 192 or 320, a batch that fits the
// XCDs' L2s: blocks of 256 threads from the beginning, as the codes pass has them, so
// that each block finds its items in its own L2 (order 192, 24 MB: 20 us, 22-23 with
// any other shape; up to order 128 the shapes above are faster, 20 against 16).
template <int B>
bool red_mapped(int n, int64_t E) {
    return B > 128 && (int64_t)n * E <= (int64_t)7 << 20;
}

// The minimum and maximum or range pass: f(threads, U, FWD) and the blocks per sample.
template <int B, typename F>
void red_launch(int n, int64_t items, bool mapped, F &&f) {
    using std::integral_constant;
    constexpr integral_constant<int, 1> one{};
    constexpr integral_constant<int, 2> two{};
    constexpr std::true_type fwd{};
    constexpr std::false_type rev{};
    if constexpr (B <= 128) {
        if (items < 16384) {
            constexpr int RT = B == 128 ? 256 : 512;
            // (many samples, whose maxima lie on several cache lines: more blocks)
            const int blocks = red_blocks(items, RT / 4, n, n < 128 ? kRedGrid : 1024 * 1024 / RT);
            if ((int64_t)blocks * (RT / 4) >= items) f(integral_constant<int, RT>{}, one, rev, blocks);
            else f(integral_constant<int, RT>{}, two, rev, blocks);
        } else {
            f(integral_constant<int, 1024>{}, two, rev, red_blocks(items, 256, n));
        }
    } else {
        if (mapped) f(integral_constant<int, 256>{}, one, fwd, red_blocks(items, 64, n, 1 << 20));
        else if (B == 192 && items >= 12288) f(integral_constant<int, 512>{}, one, rev, red_blocks(items, 128, n));
        else f(integral_constant<int, 256>{}, one, rev, red_blocks(items, 64, n));
    }
}

// A sample of few floats goes to at most kAbsSlots blocks, each with a slot of its
// own: the slots need no clearing, one launch less (1-2 us on the GPU and as much on
// the host).  Order 64, 0.8 MB 8.4 us without, 6.7 with, 3.1 MB 9.0 / 8.4, 7.1 MB 10.2 /
// 11.3; untransformed 9.4 MB 10.0 / 9.4; order 320, 1.3 MB 20.4 / 18.7, 32 samples of 2.9
// MB 65 / 72.
template <int B>
bool red_own(int n, int64_t E) {
    return E <= (B == 1 ? 1 << 21 : B <= 192 || n < 16 ? 1 << 20 : 3 << 17);
}

template <int B, int RT, bool FWD = false>
void launch_absmax(const float *x, int n, int64_t E, float *ws, int blocks, int own, hipStream_t st) {
    if constexpr (B == 1) absmax_flat_kernel<RT><<<dim3(blocks, n), RT, 0, st>>>(x, E, ws, own);
    else absmax_kernel<B, RT, B <= 128 ? 2 : 1, FWD><<<dim3(blocks, n), RT, 0, st>>>(x, E, ws, own);
}

template <int B>
hipError_t launch_vector(const float *x, int n, int64_t E, const float *absmax_in, float *ws_absmax,
                         int8_t *xq, float *act_scale, hipStream_t st, int c64 = 0) {
    constexpr int I = ItemShape<B>::I;
    const int64_t items = (E + I - 1) / I;
    const float *A = absmax_in;
    int slots = 1;
    if (!A && red_own<B>(n, E)) {
        // a quad with at most two items (four of order 320, whose blocks of more threads
        // do not pay): fewer threads
        const bool few = items <= (B == 192 ? 2048 : 2 * 64 * kAbsSlots);
        constexpr int SMALL = B <= 64 ? 512 : 256, LARGE = B <= 128 ? 1024 : B == 192 ? 512 : 256;
        slots = red_blocks(items, (few ? SMALL : LARGE) / 4, 1, kAbsSlots);
        if (few) launch_absmax<B, SMALL>(x, n, E, ws_absmax, slots, 1, st);
        else launch_absmax<B, LARGE>(x, n, E, ws_absmax, slots, 1, st);
        A = ws_absmax;
    } else if (!A) {
        slots = kAbsSlots;
        fill_u32_kernel<<<1, 256, 0, st>>>(reinterpret_cast<uint32_t *>(ws_absmax), n * kAbsSlots, 0u);
        if constexpr (B == 1)   // (with the fewest registers: twice the blocks, four float4 per thread at least)
            launch_absmax<B, 1024>(x, n, E, ws_absmax, red_blocks(E / 4, 4096, n, 2 * kRedGrid), 0, st);
        else if constexpr (B <= 128)
            launch_absmax<B, 1024>(x, n, E, ws_absmax, red_blocks(items, 256, n), 0, st);
        else if (red_mapped<B>(n, E))
            launch_absmax<B, 256, true>(x, n, E, ws_absmax, red_blocks(items, 64, n, 1 << 20), 0, st);
        else if constexpr (B == 192)
            launch_absmax<B, 512>(x, n, E, ws_absmax, red_blocks(items, 128, n, 2 * kRedGrid), 0, st);
        else
            launch_absmax<B, 256>(x, n, E, ws_absmax, red_blocks(items, 64, n, 8 * kRedGrid), 0, st);
        A = ws_absmax;
    }
    dim3 grid(grid_x(items, kQuadsPerBlock * QuantUnroll<B>::UN, n), n);
    quant_kernel<B><<<grid, kThreads, 0, st>>>(x, E, A, xq, act_scale, c64, slots, absmax_in ? 1 : kAbsSlots);
    return hipGetLastError();
}

template <int B>
hipError_t launch_scalar(const float *x, int n, int64_t E, const float *absmax_in, float *ws_absmax,
                         int8_t *xq, float *act_scale, hipStream_t st) {
    dim3 grid(grid_x(E / B, kThreads, n), n);
    const float *A = absmax_in;
    if (!A) {
        fill_u32_kernel<<<1, 256, 0, st>>>(reinterpret_cast<uint32_t *>(ws_absmax), n, 0u);
        scalar_kernel<B, false><<<dim3(grid_x(E / B, kThreads, n, 2048), n), kThreads, 0, st>>>(x, E, ws_absmax,
                                                                                              nullptr, nullptr);
        A = ws_absmax;
    }
    scalar_kernel<B, true><<<grid, kThreads, 0, st>>>(x, E, const_cast<float *>(A), xq, act_scale);
    return hipGetLastError();
}

template <int B>
hipError_t launch_range_b(const float *x, int n, int64_t P, int C, float *amax, hipStream_t st) {
    const int64_t E = P * C;
    if (C % B == 0 && E % 4 == 0) {
        constexpr int I = ItemShape<B>::I;
        const int64_t items = (E + I - 1) / I;
        red_launch<B>(n, items, false, [&](auto rt, auto u, auto, int blocks) {
            constexpr int RT = decltype(rt)::value;
            range_kernel<B, RT, decltype(u)::value><<<dim3(blocks, n), RT, 0, st>>>(x, E, amax);
        });
    } else if constexpr (kron_q(B) == 0) {
        const int64_t units = P * ((C + B - 1) / B);
        range_pad_kernel<B><<<dim3(grid_x(units, kThreads, n, 2048), n), kThreads, 0, st>>>(x, P, C, amax);
    } else {
        return hipErrorInvalidValue;   // Kronecker orders: whole blocks only
    }
    return hipGetLastError();
}

template <int B>
hipError_t launch_affine_b(const float *x, int n, int64_t E, float *ws, int8_t *xq, float *act_scale,
                           int32_t *act_zero, hipStream_t st) {
    constexpr int I = ItemShape<B>::I;
    const int64_t items = (E + I - 1) / I;
    fill_u32_kernel<<<1, 256, 0, st>>>(reinterpret_cast<uint32_t *>(ws), 2 * n, 0u);
    red_launch<B>(n, items, red_mapped<B>(n, E), [&](auto rt, auto u, auto fwd, int blocks) {
        constexpr int RT = decltype(rt)::value;
        minmax_kernel<B, RT, decltype(u)::value, decltype(fwd)::value><<<dim3(blocks, n), RT, 0, st>>>(x, E, ws);
    });
    quant_affine_kernel<B><<<dim3(grid_x(items, kQuadsPerBlock, n), n), kThreads, 0, st>>>(x, E, ws, xq, act_scale,
                                                                                          act_zero);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_act_quant_affine(const float *x, int n, int64_t E, int hblock, float *ws, int8_t *xq,
                                   float *act_scale, int32_t *act_zero, hipStream_t st) {
    if (E % 4 != 0) return hipErrorInvalidValue;
    switch (hblock) {
        case 1: return launch_affine_b<1>(x, n, E, ws, xq, act_scale, act_zero, st);
        case 2: return launch_affine_b<2>(x, n, E, ws, xq, act_scale, act_zero, st);
        case 4: return launch_affine_b<4>(x, n, E, ws, xq, act_scale, act_zero, st);
        case 8: return launch_affine_b<8>(x, n, E, ws, xq, act_scale, act_zero, st);
        case 16: return launch_affine_b<16>(x, n, E, ws, xq, act_scale, act_zero, st);
        case 32: return launch_affine_b<32>(x, n, E, ws, xq, act_scale, act_zero, st);
        case 64: return launch_affine_b<64>(x, n, E, ws, xq, act_scale, act_zero, st);
        case 128: return launch_affine_b<128>(x, n, E, ws, xq, act_scale, act_zero, st);
        case 192: return launch_affine_b<192>(x, n, E, ws, xq, act_scale, act_zero, st);
        case 320: return launch_affine_b<320>(x, n, E, ws, xq, act_scale, act_zero, st);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_range_expansion(const float *x, int n, int64_t P, int C, int hblock, float *amax, int32_t *flags,
                                  int32_t *count, hipStream_t st) {
    fill_u32_kernel<<<1, 256, 0, st>>>(reinterpret_cast<uint32_t *>(amax), 2 * n, 0u);
    hipError_t e;
    switch (hblock) {
        case 1: e = launch_range_b<1>(x, n, P, C, amax, st); break;
        case 2: e = launch_range_b<2>(x, n, P, C, amax, st); break;
        case 4: e = launch_range_b<4>(x, n, P, C, amax, st); break;
        case 8: e = launch_range_b<8>(x, n, P, C, amax, st); break;
        case 16: e = launch_range_b<16>(x, n, P, C, amax, st); break;
        case 32: e = launch_range_b<32>(x, n, P, C, amax, st); break;
        case 64: e = launch_range_b<64>(x, n, P, C, amax, st); break;
        case 128: e = launch_range_b<128>(x, n, P, C, amax, st); break;
        case 192: e = launch_range_b<192>(x, n, P, C, amax, st); break;
        case 320: e = launch_range_b<320>(x, n, P, C, amax, st); break;
        default: return hipErrorInvalidValue;
    }
    if (e != hipSuccess) return e;
    expansion_flags_kernel<<<(n + 255) / 256, 256, 0, st>>>(amax, n, hblock, flags, count);
    return hipGetLastError();
}

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
float *g_scratch[kMaxDevices] = {};

// The current device's copy of `scratch`, looked up on the first call on that
// device (with it current) and kept.
hipError_t scratch_absmax(float **out) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        g_scratch[dev] = static_cast<float *>(p);
    }
    *out = g_scratch[dev];
    return hipSuccess;
}

}  // namespace

hipError_t launch_act_quant_noalloc(const float *x, int n, int64_t E, int hblock, int8_t *xq, float *act_scale,
                                    hipStream_t st) {
    if (n <= 0 || n > kNoAllocMaxSamples) return hipErrorInvalidValue;
    float *ws = nullptr;
    const hipError_t e = scratch_absmax(&ws);
    if (e != hipSuccess) return e;
    // the two-pass path writes the slots that it reads (small samples) or clears
    // all n * kAbsSlots with a fill kernel before its atomics
    return launch_act_quant(x, n, E, hblock, nullptr, ws, xq, act_scale, st);
}

hipError_t launch_act_quant(const float *x, int n, int64_t E, int hblock, const float *absmax_in,
                            float *ws_absmax, int8_t *xq, float *act_scale, hipStream_t st, int c64) {
    if (c64 > 0) {
        // items of 64 channels, one chunk each
        if (c64 % 64 != 0 || E % c64 != 0) return hipErrorInvalidValue;
        switch (hblock) {
            case 1: return launch_vector<1>(x, n, E, absmax_in, ws_absmax, xq, act_scale, st, c64);
            case 2: return launch_vector<2>(x, n, E, absmax_in, ws_absmax, xq, act_scale, st, c64);
            case 4: return launch_vector<4>(x, n, E, absmax_in, ws_absmax, xq, act_scale, st, c64);
            case 8: return launch_vector<8>(x, n, E, absmax_in, ws_absmax, xq, act_scale, st, c64);
            case 16: return launch_vector<16>(x, n, E, absmax_in, ws_absmax, xq, act_scale, st, c64);
            case 32: return launch_vector<32>(x, n, E, absmax_in, ws_absmax, xq, act_scale, st, c64);
            case 64: return launch_vector<64>(x, n, E, absmax_in, ws_absmax, xq, act_scale, st, c64);
            default: return hipErrorInvalidValue;
        }
    }
    if (E % 4 != 0) {
        if (hblock == 1) return launch_scalar<1>(x, n, E, absmax_in, ws_absmax, xq, act_scale, st);
        return launch_scalar<2>(x, n, E, absmax_in, ws_absmax, xq, act_scale, st);
    }
    switch (hblock) {
        case 1: return launch_vector<1>(x, n, E, absmax_in, ws_absmax, xq, act_scale, st);
        case 2: return launch_vector<2>(x, n, E, absmax_in, ws_absmax, xq, act_scale, st);
        case 4: return launch_vector<4>(x, n, E, absmax_in, ws_absmax, xq, act_scale, st);
        case 8: return launch_vector<8>(x, n, E, absmax_in, ws_absmax, xq, act_scale, st);
        case 16: return launch_vector<16>(x, n, E, absmax_in, ws_absmax, xq, act_scale, st);
        case 32: return launch_vector<32>(x, n, E, absmax_in, ws_absmax, xq, act_scale, st);
        case 64: return launch_vector<64>(x, n, E, absmax_in, ws_absmax, xq, act_scale, st);
        case 128: return launch_vector<128>(x, n, E, absmax_in, ws_absmax, xq, act_scale, st);
        case 192: return launch_vector<192>(x, n, E, absmax_in, ws_absmax, xq, act_scale, st);
        case 320: return launch_vector<320>(x, n, E, absmax_in, ws_absmax, xq, act_scale, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace hatq
