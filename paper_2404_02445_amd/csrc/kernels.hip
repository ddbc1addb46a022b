// Bandwidth-bound kernels of the sliced forward pass (gfx950, wave64):
// input layout conversion, pooling, layer norm, embeddings, attention and the
// raw boundary copy.  Accesses are 16-byte vectors along the contiguous
// (channel / feature) dimension wherever the shape allows; reductions are
// wave-level butterflies (no atomics, so results are reproducible).
#include "internal.h"

namespace mopar {

template <typename T> struct Vec;   // 16-byte vector of T
template <> struct Vec<__bf16> { static constexpr int N = 8; };
template <> struct Vec<float> { static constexpr int N = 4; };

__device__ __forceinline__ float to_f(__bf16 v) {
    return __uint_as_float(static_cast<unsigned>(__builtin_bit_cast(unsigned short, v)) << 16);
}
__device__ __forceinline__ float to_f(float v) { return v; }

template <typename T> __device__ __forceinline__ T from_f(float v) { return static_cast<T>(v); }

// Sum over the wave, the same value in every lane: within each row of 16 lanes a butterfly of
// DPP moves (partners 1 and 2 apart, then the mirrored half, then the mirrored row: each step
// adds a lane's partial to its partner's, so all lanes of a row agree), then the four row sums
// are read out and added in row order.
__device__ __forceinline__ float dpp_add(float v, int ctrl_sel) {
    int m = 0;
    switch (ctrl_sel) {   // DPP controls must be compile-time constants
        case 0: m = __builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xF, 0xF, false); break;   // quad [1,0,3,2]
        case 1: m = __builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x4E, 0xF, 0xF, false); break;   // quad [2,3,0,1]
        case 2: m = __builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x141, 0xF, 0xF, false); break;  // row half mirror
        default: m = __builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x140, 0xF, 0xF, false); break; // row mirror
    }
    return v + __int_as_float(m);
}
__device__ __forceinline__ float wave_sum(float v) {
    v = dpp_add(v, 0);
    v = dpp_add(v, 1);
    v = dpp_add(v, 2);
    v = dpp_add(v, 3);
    const float r0 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 0));
    const float r1 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 16));
    const float r2 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 32));
    const float r3 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 48));
    return (r0 + r1) + (r2 + r3);
}

static inline unsigned blocks_for(int64_t n, int per_block) {
    int64_t b = (n + per_block - 1) / per_block;
    return static_cast<unsigned>(b < 1 ? 1 : b);
}

// ---------------------------------------------------------------------------
// NCHW float32 (model input) -> NHWC in the model dtype, channels padded to cs.
// One thread per pixel: C strided reads (coalesced across neighbouring w),
// cs-wide contiguous 16-byte writes.  Sizes below 2^31 elements (host-checked).
// ---------------------------------------------------------------------------
template <typename T>
__global__ void nchw_to_nhwc_kernel(const float* __restrict__ x, T* __restrict__ y, int n, int c, int h, int w,
                                    int cs) {
    constexpr int V = Vec<T>::N;
    const int pix = blockIdx.x * blockDim.x + threadIdx.x;
    const int hw = h * w;
    if (pix >= n * hw) return;
    const int img = pix / hw, r = pix - img * hw;
    const float* src = x + static_cast<int64_t>(img) * c * hw + r;
    T* dst = y + static_cast<int64_t>(pix) * cs;
    for (int c0 = 0; c0 < cs; c0 += V) {           // cs is a multiple of V
        // every channel slot loads (padding slots re-read channel c - 1), so the loads go out
        // together instead of one branch and one wait per channel
        float f[V];
#pragma unroll
        for (int i = 0; i < V; ++i) f[i] = src[static_cast<int64_t>(min(c0 + i, c - 1)) * hw];
        uint4 out;
        T* o = reinterpret_cast<T*>(&out);
#pragma unroll
        for (int i = 0; i < V; ++i) o[i] = from_f<T>(c0 + i < c ? f[i] : 0.0f);
        *reinterpret_cast<uint4*>(dst + c0) = out;
    }
}

hipError_t launch_nchw_to_nhwc(const float* x, void* y, int n, int c, int h, int w, int cs, int dtype,
                               hipStream_t s) {
    const int64_t pix = static_cast<int64_t>(n) * h * w;
    if (pix * cs >= (int64_t(1) << 31) || cs % (dtype == MOPAR_BF16 ? 8 : 4) != 0) return hipErrorInvalidValue;
    if (dtype == MOPAR_BF16)
        launch_kernel(nchw_to_nhwc_kernel<__bf16>, dim3(blocks_for(pix, 256)), dim3(256), 0, s, x,
                           static_cast<__bf16*>(y), n, c, h, w, cs);
    else
        launch_kernel(nchw_to_nhwc_kernel<float>, dim3(blocks_for(pix, 256)), dim3(256), 0, s, x,
                           static_cast<float*>(y), n, c, h, w, cs);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Max pool, NHWC: one thread per (output pixel, 16-byte channel group).
// Window positions outside the image count as -inf.  KW > 0 fixes the window
// size at compile time; every position then loads (an outside one re-reads a
// clamped pixel and is ignored), so all the window's loads issue together.
// Sizes below 2^31 elements (host-checked): 32-bit index math.
// ---------------------------------------------------------------------------
template <typename T, int KW>
__global__ void maxpool_kernel(const T* __restrict__ x, T* __restrict__ y, int n, int h, int w, int c, int kr,
                               int stride, int pad, int ho, int wo) {
    constexpr int V = Vec<T>::N;
    const int k = KW > 0 ? KW : kr;
    const int groups = c / V;
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n * ho * wo * groups) return;
    const int pix = t / groups, g = t - pix * groups;
    const int img = pix / (ho * wo), rem = pix - img * (ho * wo);
    const int oy = rem / wo, ox = rem - oy * wo;
    float m[V];
#pragma unroll
    for (int i = 0; i < V; ++i) m[i] = -INFINITY;
    if constexpr (KW > 0) {
        uint4 raw[KW * KW];
#pragma unroll
        for (int r = 0; r < KW; ++r)
#pragma unroll
            for (int q = 0; q < KW; ++q) {
                const int iy = min(max(oy * stride - pad + r, 0), h - 1);
                const int ix = min(max(ox * stride - pad + q, 0), w - 1);
                raw[r * KW + q] = *reinterpret_cast<const uint4*>(x + ((img * h + iy) * w + ix) * c + g * V);
            }
#pragma unroll
        for (int r = 0; r < KW; ++r)
#pragma unroll
            for (int q = 0; q < KW; ++q) {
                const int iy = oy * stride - pad + r, ix = ox * stride - pad + q;
                const bool in = static_cast<unsigned>(iy) < static_cast<unsigned>(h) &&
                                static_cast<unsigned>(ix) < static_cast<unsigned>(w);
                const T* e = reinterpret_cast<const T*>(&raw[r * KW + q]);
#pragma unroll
                for (int i = 0; i < V; ++i) m[i] = fmaxf(m[i], in ? to_f(e[i]) : -INFINITY);
            }
    } else {
        for (int r = 0; r < k; ++r) {
            const int iy = oy * stride - pad + r;
            for (int q = 0; q < k; ++q) {
                const int ix = ox * stride - pad + q;
                if (static_cast<unsigned>(iy) >= static_cast<unsigned>(h) ||
                    static_cast<unsigned>(ix) >= static_cast<unsigned>(w))
                    continue;
                const uint4 raw = *reinterpret_cast<const uint4*>(x + ((img * h + iy) * w + ix) * c + g * V);
                const T* e = reinterpret_cast<const T*>(&raw);
#pragma unroll
                for (int i = 0; i < V; ++i) m[i] = fmaxf(m[i], to_f(e[i]));
            }
        }
    }
    uint4 out;
    T* o = reinterpret_cast<T*>(&out);
#pragma unroll
    for (int i = 0; i < V; ++i) o[i] = from_f<T>(m[i]);
    *reinterpret_cast<uint4*>(y + pix * c + g * V) = out;
}

template <typename T>
static void maxpool_launch(const void* x, void* y, int n, int h, int w, int c, int k, int stride, int pad, int ho,
                           int wo, hipStream_t s) {
    const int64_t total = static_cast<int64_t>(n) * ho * wo * (c / Vec<T>::N);
    const T* xp = static_cast<const T*>(x);
    T* yp = static_cast<T*>(y);
    if (k == 3)
        launch_kernel((maxpool_kernel<T, 3>), dim3(blocks_for(total, 256)), dim3(256), 0, s, xp, yp, n, h, w, c, k,
                           stride, pad, ho, wo);
    else if (k == 2)
        launch_kernel((maxpool_kernel<T, 2>), dim3(blocks_for(total, 256)), dim3(256), 0, s, xp, yp, n, h, w, c, k,
                           stride, pad, ho, wo);
    else
        launch_kernel((maxpool_kernel<T, 0>), dim3(blocks_for(total, 256)), dim3(256), 0, s, xp, yp, n, h, w, c, k,
                           stride, pad, ho, wo);
}

hipError_t launch_maxpool(const void* x, void* y, int n, int h, int w, int c, int k, int stride, int pad, int ho,
                          int wo, int dtype, hipStream_t s) {
    if (static_cast<int64_t>(n) * h * w * c >= (int64_t(1) << 31)) return hipErrorInvalidValue;
    // the kernel moves whole 16-byte channel groups: a channel count off the granule is refused
    if (c % (dtype == MOPAR_BF16 ? 8 : 4) != 0) return hipErrorInvalidValue;
    if (dtype == MOPAR_BF16)
        maxpool_launch<__bf16>(x, y, n, h, w, c, k, stride, pad, ho, wo, s);
    else
        maxpool_launch<float>(x, y, n, h, w, c, k, stride, pad, ho, wo, s);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Global average pool, NHWC -> [N][C].  A block owns one image and 8 channel
// chunks (16 bytes each); its 256 threads are 8 chunks x 32 pixel slices.
// Slice s sums pixels s, s + 32, ... in order (fp32); the 32 slice sums are
// then added in slice order and divided once: a fixed order, so the result
// is reproducible.  Channel counts that are not a whole number of chunks use
// one thread per channel, summing pixels in order.
// ---------------------------------------------------------------------------
constexpr int AP_SLICES = 32, AP_CHUNKS = 8;

template <typename T>
__global__ __launch_bounds__(256) void avgpool_kernel(const T* __restrict__ x, T* __restrict__ y, int hw, int c) {
    constexpr int V = Vec<T>::N;
    __shared__ float part[AP_SLICES][AP_CHUNKS * V];
    const int img = blockIdx.y;
    const int chunk = threadIdx.x % AP_CHUNKS, slice = threadIdx.x / AP_CHUNKS;
    const int c0 = (blockIdx.x * AP_CHUNKS + chunk) * V;
    float sum[V];
#pragma unroll
    for (int i = 0; i < V; ++i) sum[i] = 0.0f;
    if (c0 < c) {
        const T* p = x + static_cast<int64_t>(img) * hw * c + c0;
        for (int px = slice; px < hw; px += AP_SLICES) {
            const uint4 raw = *reinterpret_cast<const uint4*>(p + static_cast<int64_t>(px) * c);
            const T* e = reinterpret_cast<const T*>(&raw);
#pragma unroll
            for (int i = 0; i < V; ++i) sum[i] += to_f(e[i]);
        }
    }
#pragma unroll
    for (int i = 0; i < V; ++i) part[slice][chunk * V + i] = sum[i];
    __syncthreads();
    if (threadIdx.x < AP_CHUNKS * V) {
        const int ch = blockIdx.x * AP_CHUNKS * V + threadIdx.x;
        if (ch < c) {
            float s = 0.0f;
            for (int sl = 0; sl < AP_SLICES; ++sl) s += part[sl][threadIdx.x];
            y[static_cast<int64_t>(img) * c + ch] = from_f<T>(s / static_cast<float>(hw));
        }
    }
}

template <typename T>
__global__ void avgpool_channel_kernel(const T* __restrict__ x, T* __restrict__ y, int n, int hw, int c) {
    const int64_t t = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (t >= static_cast<int64_t>(n) * c) return;
    const int64_t img = t / c;
    const int ch = static_cast<int>(t - img * c);
    const T* p = x + img * hw * c + ch;
    float s = 0.0f;
    for (int i = 0; i < hw; ++i) s += to_f(p[static_cast<int64_t>(i) * c]);
    y[t] = from_f<T>(s / static_cast<float>(hw));
}

template <typename T>
static void avgpool_launch(const void* x, void* y, int n, int hw, int c, hipStream_t s) {
    constexpr int V = Vec<T>::N;
    if (c % V == 0) {
        const dim3 grid((c / V + AP_CHUNKS - 1) / AP_CHUNKS, n);
        launch_kernel(avgpool_kernel<T>, grid, dim3(256), 0, s, static_cast<const T*>(x), static_cast<T*>(y), hw, c);
    } else {
        launch_kernel(avgpool_channel_kernel<T>, dim3(blocks_for(static_cast<int64_t>(n) * c, 256)), dim3(256), 0, s,
                           static_cast<const T*>(x), static_cast<T*>(y), n, hw, c);
    }
}

hipError_t launch_avgpool(const void* x, void* y, int n, int hw, int c, int dtype, hipStream_t s) {
    if (dtype == MOPAR_BF16)
        avgpool_launch<__bf16>(x, y, n, hw, c, s);
    else
        avgpool_launch<float>(x, y, n, hw, c, s);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Layer norm over rows of F <= 64 * LN_MAXV elements: one wave per row, the
// row held in registers, mean then centred variance by wave butterflies.
// When F is a whole number of 16-byte chunks each lane holds whole chunks
// (chunk lane + 64 j), read and written as vectors, and the kernel instance
// keeps MV floats per lane -- just the row's chunks, so fewer registers and
// more resident waves; otherwise element lane + 64 i, MV = LN_MAXV.
// ---------------------------------------------------------------------------
constexpr int LN_MAXV = 32;

// column of register i of this lane
template <typename T, bool VEC>
__device__ __forceinline__ int ln_col(int lane, int i) {
    constexpr int V = Vec<T>::N;
    return VEC ? (lane + 64 * (i / V)) * V + i % V : lane + 64 * i;
}

template <typename T, bool VEC, int MV>
__device__ __forceinline__ void ln_row(float (&v)[MV], int f, int lane, const T* g, const T* b, float eps,
                                       T* out) {
    constexpr int V = Vec<T>::N;
    // gamma and beta go out before the reductions, so their latency overlaps the row's
    uint4 gr[VEC ? MV / V : 1], br[VEC ? MV / V : 1];
    if constexpr (VEC) {
#pragma unroll
        for (int j = 0; j < MV / V; ++j) {
            const int c0 = min((lane + 64 * j) * V, f - V);   // in range; unused past f
            gr[j] = *reinterpret_cast<const uint4*>(g + c0);
            br[j] = *reinterpret_cast<const uint4*>(b + c0);
        }
    }
    float s = 0.0f;
#pragma unroll
    for (int i = 0; i < MV; ++i)
        if (ln_col<T, VEC>(lane, i) < f) s += v[i];
    const float mean = wave_sum(s) / static_cast<float>(f);
    float q = 0.0f;
#pragma unroll
    for (int i = 0; i < MV; ++i)
        if (ln_col<T, VEC>(lane, i) < f) {
            const float d = v[i] - mean;
            q += d * d;
        }
    const float var = wave_sum(q) / static_cast<float>(f);
    const float inv = 1.0f / sqrtf(var + eps);
    if constexpr (VEC) {
#pragma unroll
        for (int j = 0; j < MV / V; ++j) {
            const int c0 = (lane + 64 * j) * V;
            if (c0 >= f) continue;
            const T* ge = reinterpret_cast<const T*>(&gr[j]);
            const T* be = reinterpret_cast<const T*>(&br[j]);
            uint4 o;
            T* oe = reinterpret_cast<T*>(&o);
#pragma unroll
            for (int e = 0; e < V; ++e) oe[e] = from_f<T>((v[j * V + e] - mean) * inv * to_f(ge[e]) + to_f(be[e]));
            *reinterpret_cast<uint4*>(out + c0) = o;
        }
    } else {
#pragma unroll
        for (int i = 0; i < MV; ++i) {
            const int col = lane + i * 64;
            if (col < f) out[col] = from_f<T>((v[i] - mean) * inv * to_f(g[col]) + to_f(b[col]));
        }
    }
}

// v[i] = a[col] (+ c[col]) for this lane's columns (zeros past f)
template <typename T, bool VEC, int MV>
__device__ __forceinline__ void ln_load(const T* a, const T* c, int f, int lane, float (&v)[MV]) {
    constexpr int V = Vec<T>::N;
    if constexpr (VEC) {
        // Every lane loads (a lane past f re-reads the last chunk and keeps zeros): per-lane
        // branches around the loads would make each chunk wait for the previous one.
        uint4 ar[MV / V], cr[MV / V];
#pragma unroll
        for (int j = 0; j < MV / V; ++j) {
            const int cc = min((lane + 64 * j) * V, f - V);
            ar[j] = *reinterpret_cast<const uint4*>(a + cc);
            cr[j] = c ? *reinterpret_cast<const uint4*>(c + cc) : make_uint4(0, 0, 0, 0);
        }
#pragma unroll
        for (int j = 0; j < MV / V; ++j) {
            const bool ok = (lane + 64 * j) * V < f;
            const T* ae = reinterpret_cast<const T*>(&ar[j]);
            const T* ce = reinterpret_cast<const T*>(&cr[j]);
#pragma unroll
            for (int e = 0; e < V; ++e) v[j * V + e] = ok ? to_f(ae[e]) + (c ? to_f(ce[e]) : 0.0f) : 0.0f;
        }
    } else {
#pragma unroll
        for (int i = 0; i < MV; ++i) {
            const int col = lane + i * 64;
            v[i] = col < f ? to_f(a[col]) + (c ? to_f(c[col]) : 0.0f) : 0.0f;
        }
    }
}

template <typename T, bool VEC, int MV>
__global__ void layernorm_kernel(const T* __restrict__ x, const T* __restrict__ res, const T* __restrict__ g,
                                 const T* __restrict__ b, T* __restrict__ y, int64_t rows, int f, float eps) {
    const int lane = threadIdx.x & 63;
    const int64_t row = static_cast<int64_t>(blockIdx.x) * (blockDim.x / 64) + (threadIdx.x >> 6);
    if (row >= rows) return;
    float v[MV];
    ln_load<T, VEC, MV>(x + row * f, res ? res + row * f : nullptr, f, lane, v);
    ln_row<T, VEC, MV>(v, f, lane, g, b, eps, y + row * f);
}

// go(kernel) with the row kernel instance for f columns: 16-byte chunks when f allows, with as
// many per lane as the row needs (fewer registers, more resident waves), else one element
// per lane and step
template <typename T, template <typename, bool, int> class K, typename Go>
static void ln_instance(int f, Go&& go) {
    constexpr int V = Vec<T>::N;
    if (f % V != 0) return go(K<T, false, LN_MAXV>::fn);
    switch ((f + 64 * V - 1) / (64 * V)) {
        case 1: return go(K<T, true, V>::fn);
        case 2: return go(K<T, true, 2 * V>::fn);
        case 3: return go(K<T, true, 3 * V>::fn);
        case 4: return go(K<T, true, 4 * V>::fn);
        default: return go(K<T, true, LN_MAXV>::fn);
    }
}
template <typename T, bool VEC, int MV>
struct LnK { static constexpr auto fn = layernorm_kernel<T, VEC, MV>; };

template <typename T>
static void layernorm_launch(const void* x, const void* res, const void* g, const void* b, void* y, int64_t rows,
                             int f, float eps, hipStream_t s) {
    const T *xp = static_cast<const T*>(x), *rp = static_cast<const T*>(res);
    const T *gp = static_cast<const T*>(g), *bp = static_cast<const T*>(b);
    ln_instance<T, LnK>(f, [&](auto kern) {
        launch_kernel(kern, dim3(blocks_for(rows, 4)), dim3(256), 0, s, xp, rp, gp, bp, static_cast<T*>(y), rows, f,
                      eps);
    });
}

hipError_t launch_layernorm(const void* x, const void* res, const void* g, const void* b, void* y, int64_t rows,
                            int f, float eps, int dtype, hipStream_t s) {
    if (f < 1 || f > 64 * LN_MAXV) return hipErrorInvalidValue;   // a row lives in one wave's registers
    if (dtype == MOPAR_BF16)
        layernorm_launch<__bf16>(x, res, g, b, y, rows, f, eps, s);
    else
        layernorm_launch<float>(x, res, g, b, y, rows, f, eps, s);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// BERT embedding: v = tok[id] + pos[s] + type[0], then layer norm (one wave
// per token).
// ---------------------------------------------------------------------------
template <typename T, bool VEC, int MV>
__global__ void embed_bert_kernel(const int32_t* __restrict__ ids, const T* __restrict__ tok,
                                  const T* __restrict__ pos, const T* __restrict__ type, const T* __restrict__ g,
                                  const T* __restrict__ b, T* __restrict__ y, int64_t rows, int seq, int vocab, int f,
                                  float eps) {
    const int lane = threadIdx.x & 63;
    const int64_t row = static_cast<int64_t>(blockIdx.x) * (blockDim.x / 64) + (threadIdx.x >> 6);
    if (row >= rows) return;
    const int sidx = static_cast<int>(row % seq);
    const T* tr = tok + static_cast<int64_t>(min(max(ids[row], 0), vocab - 1)) * f;   // ids clamped to the table
    const T* pr = pos + static_cast<int64_t>(sidx) * f;
    float v[MV];
    ln_load<T, VEC, MV>(tr, pr, f, lane, v);
    float t[MV];
    ln_load<T, VEC, MV>(type, nullptr, f, lane, t);
#pragma unroll
    for (int i = 0; i < MV; ++i) v[i] += t[i];
    ln_row<T, VEC, MV>(v, f, lane, g, b, eps, y + row * f);
}

template <typename T, bool VEC, int MV>
struct EmbK { static constexpr auto fn = embed_bert_kernel<T, VEC, MV>; };

template <typename T>
static void embed_bert_launch(const int32_t* ids, const void* tok, const void* pos, const void* type, const void* g,
                              const void* b, void* y, int64_t rows, int seq, int vocab, int f, float eps,
                              hipStream_t s) {
    const T *tp = static_cast<const T*>(tok), *pp = static_cast<const T*>(pos), *yp = static_cast<const T*>(type);
    const T *gp = static_cast<const T*>(g), *bp = static_cast<const T*>(b);
    ln_instance<T, EmbK>(f, [&](auto kern) {
        launch_kernel(kern, dim3(blocks_for(rows, 4)), dim3(256), 0, s, ids, tp, pp, yp, gp, bp, static_cast<T*>(y),
                      rows, seq, vocab, f, eps);
    });
}

hipError_t launch_embed_bert(const int32_t* ids, const void* tok, const void* pos, const void* type, const void* g,
                             const void* b, void* y, int batch, int seq, int vocab, int f, float eps, int dtype,
                             hipStream_t s) {
    const int64_t rows = static_cast<int64_t>(batch) * seq;
    if (vocab < 1 || f < 1 || f > 64 * LN_MAXV) return hipErrorInvalidValue;
    if (dtype == MOPAR_BF16)
        embed_bert_launch<__bf16>(ids, tok, pos, type, g, b, y, rows, seq, vocab, f, eps, s);
    else
        embed_bert_launch<float>(ids, tok, pos, type, g, b, y, rows, seq, vocab, f, eps, s);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Plain embedding gather: one thread per 16-byte chunk of an output row.
// ---------------------------------------------------------------------------
// one block per token: the id is one (scalar) load per block, then the row's 16-byte chunks
// (an id outside [0, vocab) reads the nearest valid row instead of memory past the table)
__global__ __launch_bounds__(128) void embed_kernel(const int32_t* __restrict__ ids, const uint4* __restrict__ table,
                                                    uint4* __restrict__ y, int chunks, int vocab) {
    const int64_t row = blockIdx.x;
    const uint4* src = table + static_cast<int64_t>(min(max(ids[row], 0), vocab - 1)) * chunks;
    uint4* dst = y + row * chunks;
    for (int c = threadIdx.x; c < chunks; c += 128) dst[c] = src[c];
}

hipError_t launch_embed(const int32_t* ids, const void* table, void* y, int64_t n, int f, int vocab, int dtype,
                        hipStream_t s) {
    const int chunks = static_cast<int>(f * dtype_size(dtype) / 16);
    if (n >= (int64_t(1) << 31) || vocab < 1) return hipErrorInvalidValue;
    if (n == 0) return hipSuccess;
    launch_kernel(embed_kernel, dim3(static_cast<unsigned>(n)), dim3(128), 0, s, ids, static_cast<const uint4*>(table),
                  static_cast<uint4*>(y), chunks, vocab);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// float32 attention on the matrix cores (v_mfma_f32_16x16x4_f32), head dim 64, seq <= 128.  One block
// per (batch, head, 64-query tile), a wave per 16 queries; K and V of the head sit in LDS as float32.
// The k index of an MFMA may run over its operands' elements in any order that both share, so the
// fragments are whole 16-byte reads: S^T = K Q^T takes dim 16 g + s in step s for lane group g = lane / 16,
// O^T = V^T P^T key 16 t + 4 g + e in step (t, e), which is where S^T left the probabilities of that key --
// they stay in registers -- and row i of its dim tile d stands for dim 4 i + d.  Every product and sum is
// float32, the softmax runs over all keys at once, keys past seq have probability 0 (their V rows are
// zero).  4 x 77 tokens, 12 heads: 64.6 us as one thread per query row on the vector ALUs, 8.6 us here (the
// MFMAs of a block take 2.2 us).
// ---------------------------------------------------------------------------
constexpr int ATT_D = 64;
constexpr int ATT_MAXS = 128;
constexpr int ATT_LD = ATT_D + 4;          // float row stride: neighbouring rows start 4 banks apart

typedef float f32x4_t __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(256) void attention_f32_kernel(const float* __restrict__ qkv, float* __restrict__ y, int seq,
                                                            int heads, float scale) {
    __shared__ __attribute__((aligned(16))) float ks[ATT_MAXS * ATT_LD];
    __shared__ __attribute__((aligned(16))) float vs[ATT_MAXS * ATT_LD];
    constexpr int NT = ATT_MAXS / 16;
    const int qtiles = (seq + 63) / 64;
    const int qt = blockIdx.x % qtiles, bh = blockIdx.x / qtiles, b = bh / heads, h = bh % heads;
    const int f = heads * ATT_D;
    const int64_t row3 = 3 * static_cast<int64_t>(f);
    const float* base = qkv + static_cast<int64_t>(b) * seq * row3 + h * ATT_D;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lr = lane & 15, g = lane >> 4;
    const int nt = (seq + 15) / 16;            // key tiles
    const f32x4_t zero = {0.f, 0.f, 0.f, 0.f};

    // this lane's query row, dims 16 g .. 16 g + 15 (a row past seq reads the last one; it is not stored)
    const int q = qt * 64 + wave * 16 + lr;
    const float* qr = base + static_cast<int64_t>(min(q, seq - 1)) * row3 + 16 * g;
    f32x4_t qf[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) qf[i] = *reinterpret_cast<const f32x4_t*>(qr + 4 * i);
    // K and V rows, 16 bytes a thread, up to the last key tile's end (zeros past seq)
    for (int i0 = 0; i0 < nt * 16 * 16; i0 += 4 * 256) {
        f32x4_t kv[4], vv[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = i0 + u * 256 + threadIdx.x, r = min(i >> 4, seq - 1);
            const float* src = base + static_cast<int64_t>(r) * row3 + f + (i & 15) * 4;
            kv[u] = *reinterpret_cast<const f32x4_t*>(src);
            vv[u] = *reinterpret_cast<const f32x4_t*>(src + f);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = i0 + u * 256 + threadIdx.x, r = i >> 4;
            if (r < nt * 16) {
                *reinterpret_cast<f32x4_t*>(ks + r * ATT_LD + (i & 15) * 4) = r < seq ? kv[u] : zero;
                *reinterpret_cast<f32x4_t*>(vs + r * ATT_LD + (i & 15) * 4) = r < seq ? vv[u] : zero;
            }
        }
    }
    __syncthreads();
    if (qt * 64 + wave * 16 >= seq) return;    // (no barrier follows)

    // S^T: this lane ends with keys 16 t + 4 g + e of query lr
    f32x4_t s[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        s[t] = zero;
        if (t >= nt) continue;
        const float* kr = ks + (t * 16 + lr) * ATT_LD + 16 * g;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const f32x4_t kf = *reinterpret_cast<const f32x4_t*>(kr + 4 * i);
#pragma unroll
            for (int e = 0; e < 4; ++e) s[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[e], qf[i][e], s[t], 0, 0, 0);
        }
    }
    float mx = -INFINITY;
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            s[t][e] *= scale;
            if (t * 16 + 4 * g + e < seq) mx = fmaxf(mx, s[t][e]);
        }
    mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    float sum = 0.0f;
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            s[t][e] = t * 16 + 4 * g + e < seq ? __expf(s[t][e] - mx) : 0.0f;
            sum += s[t][e];
        }
    sum += __shfl_xor(sum, 16, 64);
    sum += __shfl_xor(sum, 32, 64);
    // O^T: this lane ends with dims 16 g + 4 e + d of query lr
    f32x4_t o[4] = {zero, zero, zero, zero};
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        if (t >= nt) continue;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const f32x4_t vf = *reinterpret_cast<const f32x4_t*>(vs + (t * 16 + 4 * g + e) * ATT_LD + 4 * lr);
#pragma unroll
            for (int d = 0; d < 4; ++d) o[d] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[d], s[t][e], o[d], 0, 0, 0);
        }
    }
    if (q >= seq) return;
    const float inv = 1.0f / sum;
    float* out = y + (static_cast<int64_t>(b) * seq + q) * f + h * ATT_D + 16 * g;
#pragma unroll
    for (int e = 0; e < 4; ++e)
        *reinterpret_cast<f32x4_t*>(out + 4 * e) = f32x4_t{o[0][e] * inv, o[1][e] * inv, o[2][e] * inv, o[3][e] * inv};
}

// ---------------------------------------------------------------------------
// bf16 attention on the matrix cores.  One block per (batch, head, 64-query
// tile), four waves of 16 query rows.  Q, K (row-major) and V (transposed,
// [dim][key]) are staged in LDS with padded rows so the 16 lanes of an MFMA
// fragment hit distinct banks.  S = Q K^T accumulates in fp32
// (v_mfma_f32_16x16x32_bf16, key fragment first so each lane holds four
// consecutive keys of one query row); the row max and sum are butterflies over
// the four lanes that share a row; P = exp(scale * (S - max)) goes to LDS as
// bf16 and O = P V runs on the matrix cores again; O is divided by the row sum
// in fp32 and stored.  Keys past seq are masked to -inf (zero K / V rows),
// queries past seq are computed on zero rows and not stored.
// ---------------------------------------------------------------------------
constexpr int AM_Q = 64, AM_K = 128, AM_D = 64;
constexpr int AM_LD = AM_D + 8;     // bf16 row stride of Q and K (144 bytes)
constexpr int AM_LP = AM_K + 8;     // bf16 row stride of V^T and P (272 bytes)

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));

__device__ __forceinline__ bf16x8_t lds8(const __bf16* p) { return *reinterpret_cast<const bf16x8_t*>(p); }

__global__ __launch_bounds__(256) void attention_mfma_kernel(const __bf16* __restrict__ qkv, __bf16* __restrict__ y,
                                                             int seq, int heads, float scale, int n_tiles) {
    // P reuses the Q and K space once S = Q K^T is done (45 KB in all: three blocks per CU)
    static_assert(4 * 16 * AM_LP <= (AM_Q + AM_K) * AM_LD, "P fits where Q and K were");
    __shared__ __attribute__((aligned(16))) __bf16 sqk[(AM_Q + AM_K) * AM_LD];
    __shared__ __attribute__((aligned(16))) __bf16 svt[AM_D * AM_LP];
    __bf16* const sq = sqk;
    __bf16* const sk = sqk + AM_Q * AM_LD;
    __bf16* const sp = sqk;
    // The XCDs take blocks round-robin: number the tiles so that each XCD runs a contiguous
    // range, and the query tiles of one (batch, head) -- which read the same K and V -- run
    // on the same XCD at about the same time, K and V coming from its L2 after the first.
    const int qtiles = (seq + AM_Q - 1) / AM_Q;
    const int tiles = gridDim.x;                       // a multiple of 8 (padded by the launcher)
    const int ti = static_cast<int>(blockIdx.x % 8) * (tiles / 8) + static_cast<int>(blockIdx.x / 8);
    if (ti >= n_tiles) return;
    const int qt = ti % qtiles, bh = ti / qtiles;
    const int b = bh / heads, h = bh % heads;
    const int f = heads * AM_D;
    const int64_t row3 = 3 * static_cast<int64_t>(f);
    const __bf16* base = qkv + static_cast<int64_t>(b) * seq * row3 + h * AM_D;
    const int q0 = qt * AM_Q;
    const uint4 zero4 = make_uint4(0, 0, 0, 0);
    // stage: 8 chunks of 8 dims per row
    for (int i = threadIdx.x; i < AM_Q * 8; i += 256) {
        const int r = i >> 3, c = i & 7, q = q0 + r;
        const uint4 v = q < seq ? *reinterpret_cast<const uint4*>(base + q * row3 + c * 8) : zero4;
        *reinterpret_cast<uint4*>(&sq[r * AM_LD + c * 8]) = v;
    }
    // every key row of the tile is staged (zeros past seq), so the products below run over all
    // AM_K keys with no data-dependent branches; the softmax masks keys >= seq.  A thread takes
    // two adjacent keys, so each V^T word it writes holds both (keys 2p, 2p + 1 of one dim).
    unsigned* svt32 = reinterpret_cast<unsigned*>(svt);
    for (int i = threadIdx.x; i < AM_K / 2 * 8; i += 256) {
        const int kp = i >> 3, c = i & 7, r0 = 2 * kp;
        uint4 k0 = zero4, k1 = zero4, v0 = zero4, v1 = zero4;
        if (r0 < seq) {
            k0 = *reinterpret_cast<const uint4*>(base + r0 * row3 + f + c * 8);
            v0 = *reinterpret_cast<const uint4*>(base + r0 * row3 + 2 * f + c * 8);
        }
        if (r0 + 1 < seq) {
            k1 = *reinterpret_cast<const uint4*>(base + (r0 + 1) * row3 + f + c * 8);
            v1 = *reinterpret_cast<const uint4*>(base + (r0 + 1) * row3 + 2 * f + c * 8);
        }
        *reinterpret_cast<uint4*>(&sk[r0 * AM_LD + c * 8]) = k0;
        *reinterpret_cast<uint4*>(&sk[(r0 + 1) * AM_LD + c * 8]) = k1;
        const unsigned a[4] = {v0.x, v0.y, v0.z, v0.w}, b[4] = {v1.x, v1.y, v1.z, v1.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            svt32[((c * 8 + 2 * e) * AM_LP) / 2 + kp] = (a[e] & 0xffffu) | (b[e] << 16);
            svt32[((c * 8 + 2 * e + 1) * AM_LP) / 2 + kp] = (a[e] >> 16) | (b[e] & 0xffff0000u);
        }
    }
    __syncthreads();

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int lr = lane & 15, lg = lane >> 4;          // fragment row, k group
    // S = Q K^T for query rows wave*16 .. +15
    f32x4_t sacc[AM_K / 16];
#pragma unroll
    for (int t = 0; t < AM_K / 16; ++t) sacc[t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < AM_D / 32; ++ks) {
        const bf16x8_t qa = lds8(&sq[(wave * 16 + lr) * AM_LD + ks * 32 + lg * 8]);
#pragma unroll
        for (int t = 0; t < AM_K / 16; ++t) {
            const bf16x8_t kb = lds8(&sk[(t * 16 + lr) * AM_LD + ks * 32 + lg * 8]);
            sacc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kb, qa, sacc[t], 0, 0, 0);
        }
    }
    // softmax over the keys of row lr: this lane holds keys 16 t + 4 lg + e
    float mx = -INFINITY;
#pragma unroll
    for (int t = 0; t < AM_K / 16; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int key = t * 16 + lg * 4 + e;
            if (key >= seq) sacc[t][e] = -INFINITY;
            mx = fmaxf(mx, sacc[t][e]);
        }
    mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    __syncthreads();                                   // every wave is done with Q and K: P goes there
    float sum = 0.0f;
    __bf16* prow = &sp[(wave * 16 + lr) * AM_LP];
#pragma unroll
    for (int t = 0; t < AM_K / 16; ++t) {
        float pe[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            pe[e] = sacc[t][e] == -INFINITY ? 0.0f : __expf(scale * (sacc[t][e] - mx));
            sum += pe[e];
        }
        const __bf16 pb[4] = {(__bf16)pe[0], (__bf16)pe[1], (__bf16)pe[2], (__bf16)pe[3]};
        *reinterpret_cast<uint2*>(&prow[t * 16 + lg * 4]) = *reinterpret_cast<const uint2*>(pb);
    }
    sum += __shfl_xor(sum, 16, 64);
    sum += __shfl_xor(sum, 32, 64);
    __syncthreads();                                   // P rows written before their fragment reads
    // O = P V: dims 16 dt + 4 lg + e of row lr
    f32x4_t oacc[AM_D / 16];
#pragma unroll
    for (int dt = 0; dt < AM_D / 16; ++dt) oacc[dt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < AM_K / 32; ++ks) {
        const bf16x8_t pa = lds8(&sp[(wave * 16 + lr) * AM_LP + ks * 32 + lg * 8]);
#pragma unroll
        for (int dt = 0; dt < AM_D / 16; ++dt) {
            const bf16x8_t vb = lds8(&svt[(dt * 16 + lr) * AM_LP + ks * 32 + lg * 8]);
            oacc[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vb, pa, oacc[dt], 0, 0, 0);
        }
    }
    const int q = q0 + wave * 16 + lr;
    if (q >= seq) return;
    const float inv = 1.0f / sum;
    __bf16* out = y + (static_cast<int64_t>(b) * seq + q) * f + h * AM_D;
#pragma unroll
    for (int dt = 0; dt < AM_D / 16; ++dt) {
        const __bf16 ob[4] = {(__bf16)(oacc[dt][0] * inv), (__bf16)(oacc[dt][1] * inv), (__bf16)(oacc[dt][2] * inv),
                              (__bf16)(oacc[dt][3] * inv)};
        *reinterpret_cast<uint2*>(out + dt * 16 + lg * 4) = *reinterpret_cast<const uint2*>(ob);
    }
}

hipError_t launch_attention(const void* qkv, void* y, int batch, int seq, int heads, float scale, int dtype,
                            hipStream_t s) {
    if (seq < 1 || seq > AM_K) return hipErrorInvalidValue;
    if (dtype == MOPAR_BF16) {
        const int n_tiles = batch * heads * ((seq + AM_Q - 1) / AM_Q);
        launch_kernel(attention_mfma_kernel, dim3((n_tiles + 7) / 8 * 8), dim3(256), 0, s,
                      static_cast<const __bf16*>(qkv), static_cast<__bf16*>(y), seq, heads, scale, n_tiles);
    } else {
        launch_kernel(attention_f32_kernel, dim3(batch * heads * ((seq + 63) / 64)), dim3(256), 0, s,
                      static_cast<const float*>(qkv), static_cast<float*>(y), seq, heads, scale);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Raw copy (the lossless boundary codec) and zero fill, 16-byte vectors with a
// byte tail.
// ---------------------------------------------------------------------------
__global__ void copy_kernel(const uint4* __restrict__ src, uint4* __restrict__ dst, int64_t n16) {
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n16;
         i += static_cast<int64_t>(gridDim.x) * blockDim.x)
        dst[i] = src[i];
}
__global__ void copy_tail_kernel(const unsigned char* src, unsigned char* dst, int64_t n) {
    const int64_t i = threadIdx.x;
    if (i < n) dst[i] = src[i];
}
__global__ void fill_kernel(uint4* __restrict__ dst, int64_t n16, unsigned v) {
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n16;
         i += static_cast<int64_t>(gridDim.x) * blockDim.x)
        dst[i] = make_uint4(v, v, v, v);
}
__global__ void fill_tail_kernel(unsigned char* dst, int64_t n, unsigned char v) {
    const int64_t i = threadIdx.x;
    if (i < n) dst[i] = v;
}

static unsigned stream_blocks(int64_t n16) {
    int64_t b = (n16 + 255) / 256;
    if (b > 256 * 16) b = 256 * 16;     // grid-stride beyond 16 blocks per CU
    return static_cast<unsigned>(b < 1 ? 1 : b);
}

hipError_t launch_copy(const void* src, void* dst, size_t bytes, hipStream_t s) {
    const int64_t n16 = static_cast<int64_t>(bytes / 16);
    if (n16 > 0)
        launch_kernel(copy_kernel, dim3(stream_blocks(n16)), dim3(256), 0, s, static_cast<const uint4*>(src),
                           static_cast<uint4*>(dst), n16);
    const int64_t tail = static_cast<int64_t>(bytes % 16);
    if (tail)
        launch_kernel(copy_tail_kernel, dim3(1), dim3(16), 0, s,
                           static_cast<const unsigned char*>(src) + n16 * 16,
                           static_cast<unsigned char*>(dst) + n16 * 16, tail);
    return hipGetLastError();
}

hipError_t launch_fill_bytes(void* p, size_t bytes, unsigned char value, hipStream_t s) {
    const int64_t n16 = static_cast<int64_t>(bytes / 16);
    if (n16 > 0)
        launch_kernel(fill_kernel, dim3(stream_blocks(n16)), dim3(256), 0, s, static_cast<uint4*>(p), n16,
                      0x01010101u * value);
    const int64_t tail = static_cast<int64_t>(bytes % 16);
    if (tail)
        launch_kernel(fill_tail_kernel, dim3(1), dim3(16), 0, s, static_cast<unsigned char*>(p) + n16 * 16, tail,
                      value);
    return hipGetLastError();
}

hipError_t launch_fill_zero(void* p, size_t bytes, hipStream_t s) { return launch_fill_bytes(p, bytes, 0, s); }

// ---------------------------------------------------------------------------
// One autoencoder codec layer whose input width is not a whole number of 16-byte
// chunks (the matrix-core GEMM streams 16-byte chunks of every row, so it needs
// that width on the granule): y[p][o] = b[o] + sum_c w[o][c] x[p][c], one thread
// per (position, output channel), the sum over c in ascending order in float32.
// Such layers are tiny (a few channels per position), so the vector ALUs serve.
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void codec_narrow_kernel(const T* __restrict__ x, const T* __restrict__ w,
                                                           const T* __restrict__ b, T* __restrict__ y,
                                                           unsigned total, int cin, int cout) {
    const unsigned i = blockIdx.x * 256u + threadIdx.x;
    if (i >= total) return;
    const unsigned p = i / static_cast<unsigned>(cout);
    const int o = static_cast<int>(i - p * static_cast<unsigned>(cout));
    const T* xr = x + static_cast<int64_t>(p) * cin;
    const T* wr = w + static_cast<int64_t>(o) * cin;
    float acc = b ? to_f(b[o]) : 0.0f;
    for (int c = 0; c < cin; ++c) acc += to_f(wr[c]) * to_f(xr[c]);
    y[i] = from_f<T>(acc);
}

hipError_t launch_codec_narrow(const void* x, const void* w, const void* b, void* y, int64_t positions, int cin,
                               int cout, int dtype, hipStream_t s) {
    const int64_t total = positions * cout;
    if (total <= 0) return hipSuccess;
    if (total >= (int64_t(1) << 31)) return hipErrorInvalidValue;   // 32-bit thread index
    const dim3 grid(blocks_for(total, 256));
    if (dtype == MOPAR_BF16)
        launch_kernel(codec_narrow_kernel<__bf16>, grid, dim3(256), 0, s, static_cast<const __bf16*>(x),
                      static_cast<const __bf16*>(w), static_cast<const __bf16*>(b), static_cast<__bf16*>(y),
                      static_cast<unsigned>(total), cin, cout);
    else
        launch_kernel(codec_narrow_kernel<float>, grid, dim3(256), 0, s, static_cast<const float*>(x),
                      static_cast<const float*>(w), static_cast<const float*>(b), static_cast<float*>(y),
                      static_cast<unsigned>(total), cin, cout);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// First-layer 7x7, stride-2 convolution of an NCHW float32 image of at most four channels (gfx950, bf16
// results), with the 3x3, stride-2, padding-1 max pool that follows it in the same pass.
//
// As three passes (a channels-last bf16 copy, an implicit GEMM, the pool) the layer reads and writes
// its 112 x 112 x 64 activation through memory, and the GEMM works on K = 7 x 7 x 8 with 245 of 392
// products on padding channels.  Here a block owns an 8 x 8 tile of pooled pixels (without the pool a
// 16 x 16 tile of conv pixels) and 64 output channels: the input patch goes to LDS once as bf16,
// four channels a pixel, and the contraction runs over k = (tap row r, tap column 0..7, channel 0..3),
// 32 wide per tap row with the eighth column's weights zero.  The eight k values of an MFMA
// fragment lane are two neighbouring pixels of the patch: one aligned 16-byte LDS read, no im2col.
// Each wave keeps the weights of its 32 channels in registers (14 fragments) and takes every other
// 16-pixel row tile.  The conv tile is rounded to bf16 in LDS, as the unfused op stores it, and pooled
// there, so the results equal the conv followed by the pool bit for bit.  The conv pixels on tile
// borders are computed twice (289 for 256).
//
// ResNet-50's stem at batch 32 (224 x 224): 75 us as three kernels, 34.8 us here; at batch 8 33.6 -> 11.5 us.
// It is bound by the latency of a block's phases (patch, weights, MFMAs, pool) with three blocks per
// CU: 1568 blocks, two rounds of 768 and 32 more.  Loads under branches cost most of it before they
// went through buffer resources (52 us), weights read in fragment order 3 us more.
// ---------------------------------------------------------------------------
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

constexpr int STEM_K = 7;                    // window
constexpr int STEM_LD = 64 + 8;              // bf16 row stride of the conv tile in LDS (spreads rows over the banks)

struct StemParams {
    const float* x;      // [n][c][h][w]
    const __bf16* w;     // [cout][7][7][8], channels past c zero
    const __bf16* b;     // [cout] or null
    __bf16* y;           // POOL: [n][ph][pw][ldc], else [n][ch][cw][ldc]
    int c, h, wd, pad;
    int ch, cw;          // conv output
    int ph, pw;          // pool output
    int cout, ldc, act;
    int tiles, tx;       // tiles per image, per tile row
};

__device__ __forceinline__ float act_of(float v, int act) {
    if (act == MOPAR_ACT_RELU) return v > 0.0f ? v : 0.0f;
    return v;
}
__device__ __forceinline__ float bf_lo(unsigned w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf_hi(unsigned w) { return __uint_as_float(w & 0xffff0000u); }

constexpr unsigned kOOB = 0x80000000u;   // past every resource here
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const void* base, unsigned bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), static_cast<short>(0), static_cast<int>(bytes), 0x00020000);
}

template <bool POOL>
__global__ __launch_bounds__(256) void stem_kernel(const StemParams p) {
    constexpr int TC = POOL ? 17 : 16;           // conv tile edge
    constexpr int NPIX = TC * TC, MT = (NPIX + 15) / 16;
    constexpr int PR = 2 * (TC - 1) + STEM_K;        // patch rows
    constexpr int PW = 2 * (TC - 1) + STEM_K + 1;    // patch columns (even; the last one meets zero weights)
    constexpr int PPIX = PR * PW, LPT = (PPIX + 255) / 256;
    __shared__ __attribute__((aligned(16))) u32x2 patch[PPIX];
    // the conv tile; before it, the 64 channels' weights as [channel][tap row][8 columns][4 channels]
    __shared__ __attribute__((aligned(16))) __bf16 conv[NPIX * STEM_LD];
    static_assert(sizeof(conv) >= 64 * STEM_K * 8 * sizeof(u32x2), "weights fit where the conv tile goes");
    u32x2* const wl = reinterpret_cast<u32x2*>(conv);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int img = blockIdx.x / p.tiles, t = blockIdx.x - img * p.tiles;
    const int ty = t / p.tx, tx = t - ty * p.tx;
    const int n0 = blockIdx.y * 64;
    // first conv pixel of the tile (with the pool, its window's corner: -1 at the image's edge)
    const int cy0 = POOL ? 16 * ty - 1 : 16 * ty, cx0 = POOL ? 16 * tx - 1 : 16 * tx;
    const int iy0 = 2 * cy0 - p.pad, ix0 = 2 * cx0 - p.pad;

    // the patch: all loads of a thread go out together, then the conversions (zeros outside the image)
    // (through a buffer resource: an offset past it reads zeros, where a branch around each load would make
    // every load wait for the one before it)
    const unsigned plane = static_cast<unsigned>(p.h) * static_cast<unsigned>(p.wd);
    const auto xr = rsrc(p.x + static_cast<int64_t>(img) * p.c * plane, static_cast<unsigned>(p.c) * plane * 4u);
    float v[LPT][4];
#pragma unroll
    for (int i = 0; i < LPT; ++i) {
        const int q = tid + 256 * i, r = q / PW, cc = q - r * PW;
        const int iy = iy0 + r, ix = ix0 + cc;
        const bool in = q < PPIX && static_cast<unsigned>(iy) < static_cast<unsigned>(p.h) &&
                        static_cast<unsigned>(ix) < static_cast<unsigned>(p.wd);
        const unsigned off = in ? static_cast<unsigned>(iy * p.wd + ix) * 4u : kOOB;
#pragma unroll
        for (int ch = 0; ch < 4; ++ch)           // (the scalar offset is not part of the range check)
            v[i][ch] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xr, static_cast<int>(ch < p.c ? off : kOOB),
                                                                                      static_cast<int>(ch * plane * 4u), 0));
    }

    // the weights of channels n0 .. n0 + 63, first four channels of each tap: whole lines of the (contiguous)
    // weight rows (fragments read straight from memory touch 16 rows per load: 3 us per block)
    constexpr int WPT = (64 * STEM_K * STEM_K + 255) / 256;
    u32x2 wv[WPT];
    const int wmax = (p.cout - n0) * (STEM_K * STEM_K) - 1;
#pragma unroll
    for (int i = 0; i < WPT; ++i) {
        const int q = min(min(tid + 256 * i, 64 * STEM_K * STEM_K - 1), wmax);
        wv[i] = *reinterpret_cast<const u32x2*>(p.w + (static_cast<int64_t>(n0) * STEM_K * STEM_K + q) * 8);
    }
    const int wn = wave & 1, wm = wave >> 1;
    const auto br = rsrc(p.b, p.b ? static_cast<unsigned>(p.cout) * 2u : 0u);
    float bias[2][4];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int n = n0 + wn * 32 + j * 16 + (lane >> 4) * 4 + e;
            bias[j][e] = bf_lo(static_cast<unsigned short>(
                __builtin_amdgcn_raw_buffer_load_b16(br, n < p.cout ? 2 * n : static_cast<int>(kOOB), 0, 0)));
        }

#pragma unroll
    for (int i = 0; i < LPT; ++i) {
        const int q = tid + 256 * i;
        if (q < PPIX)
            patch[q] = __builtin_bit_cast(u32x2, bf16x4{(__bf16)v[i][0], (__bf16)v[i][1], (__bf16)v[i][2], (__bf16)v[i][3]});
    }
#pragma unroll
    for (int i = 0; i < WPT; ++i) {
        const int q = tid + 256 * i, n = q / (STEM_K * STEM_K), rc = q - n * (STEM_K * STEM_K), r = rc / STEM_K;
        if (q < 64 * STEM_K * STEM_K) wl[(n * STEM_K + r) * 8 + rc - r * STEM_K] = wv[i];
    }
    for (int q = tid; q < 64 * STEM_K; q += 256) wl[q * 8 + 7] = u32x2{0u, 0u};
    __syncthreads();
    // this wave's weights: channels n0 + 32 wn + 16 j + l % 16, k of tap row r: columns 2 (l / 16) and + 1
    u32x4 wf[2][STEM_K];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < STEM_K; ++r)
            wf[j][r] = *reinterpret_cast<const u32x4*>(wl + ((wn * 32 + j * 16 + (lane & 15)) * STEM_K + r) * 8 + 2 * (lane >> 4));
    __syncthreads();

    // conv pixels 16 mt + l % 16 (past the tile: the last one again), weight fragment first: a lane ends
    // with four consecutive channels of one pixel; the next row tile's fragments are read under the MFMAs
    auto read = [&](int mt, u32x4 (&af)[STEM_K]) {
        const int px = min(mt * 16 + (lane & 15), NPIX - 1), oy = px / TC, ox = px - oy * TC;
        const u32x2* src = patch + (2 * oy) * PW + 2 * ox + 2 * (lane >> 4);
#pragma unroll
        for (int r = 0; r < STEM_K; ++r) af[r] = *reinterpret_cast<const u32x4*>(src + r * PW);
    };
    // the eighth column is no tap: its pixel counts as zero, or an infinity or NaN there would reach the sum
    const unsigned tap8 = (lane >> 4) == 3 ? 0u : ~0u;
    auto compute = [&](int mt, u32x4 (&af)[STEM_K]) {
        f32x4 acc[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[j] = f32x4{bias[j][0], bias[j][1], bias[j][2], bias[j][3]};
#pragma unroll
        for (int r = 0; r < STEM_K; ++r) af[r][2] &= tap8, af[r][3] &= tap8;
#pragma unroll
        for (int r = 0; r < STEM_K; ++r)
#pragma unroll
            for (int j = 0; j < 2; ++j)
                acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wf[j][r]),
                                                                 __builtin_bit_cast(bf16x8, af[r]), acc[j], 0, 0, 0);
        const int px = mt * 16 + (lane & 15);
        if (px >= NPIX) return;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            bf16x4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = (__bf16)act_of(acc[j][e], p.act);
            *reinterpret_cast<bf16x4*>(&conv[px * STEM_LD + wn * 32 + j * 16 + (lane >> 4) * 4]) = o;
        }
    };
    u32x4 a0[STEM_K], a1[STEM_K];
    read(wm, a0);
    for (int mt = wm; mt < MT; mt += 4) {
        if (mt + 2 < MT) read(mt + 2, a1);
        compute(mt, a0);
        if (mt + 2 >= MT) break;
        if (mt + 4 < MT) read(mt + 4, a0);
        compute(mt + 2, a1);
    }
    __syncthreads();

    if constexpr (POOL) {
        // 64 pooled pixels x 8 chunks of 8 channels; window pixels outside the conv's output are skipped
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int q = tid + 256 * i, chunk = q & 7, pix = q >> 3, py = pix >> 3, px = pix & 7;
            const int oy = 8 * ty + py, ox = 8 * tx + px, n = n0 + chunk * 8;
            if (oy >= p.ph || ox >= p.pw || n >= p.cout) continue;
            float m[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) m[e] = -INFINITY;
#pragma unroll
            for (int r = 0; r < 3; ++r)
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    const int ly = 2 * py + r, lx = 2 * px + c;
                    const bool in = static_cast<unsigned>(cy0 + ly) < static_cast<unsigned>(p.ch) &&
                                    static_cast<unsigned>(cx0 + lx) < static_cast<unsigned>(p.cw);
                    const u32x4 u = *reinterpret_cast<const u32x4*>(&conv[(ly * TC + lx) * STEM_LD + chunk * 8]);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        m[2 * e] = fmaxf(m[2 * e], in ? bf_lo(u[e]) : -INFINITY);
                        m[2 * e + 1] = fmaxf(m[2 * e + 1], in ? bf_hi(u[e]) : -INFINITY);
                    }
                }
            bf16x8 o;
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] = (__bf16)m[e];
            *reinterpret_cast<bf16x8*>(p.y + ((static_cast<int64_t>(img) * p.ph + oy) * p.pw + ox) * p.ldc + n) = o;
        }
    } else {
        for (int q = tid; q < NPIX * 8; q += 256) {
            const int chunk = q & 7, pix = q >> 3, oy = 16 * ty + (pix >> 4), ox = 16 * tx + (pix & 15), n = n0 + chunk * 8;
            if (oy >= p.ch || ox >= p.cw || n >= p.cout) continue;
            *reinterpret_cast<u32x4*>(p.y + ((static_cast<int64_t>(img) * p.ch + oy) * p.cw + ox) * p.ldc + n) =
                *reinterpret_cast<const u32x4*>(&conv[pix * STEM_LD + chunk * 8]);
        }
    }
}

}  // namespace

// (GELU keeps the general path: its formula lives with the GEMM's epilogues)
bool stem_ok(int dtype, int c, int kh, int kw, int stride, int cout, int64_t ldc, int64_t out_off, int act, bool res) {
    return dtype == MOPAR_BF16 && c <= 4 && kh == STEM_K && kw == STEM_K && stride == 2 && cout % 8 == 0 && ldc % 8 == 0 &&
           out_off % 8 == 0 && act != MOPAR_ACT_GELU && !res;
}

hipError_t launch_stem(const float* x, const void* w, const void* b, void* y, int n, int c, int h, int wd, int pad, int ch,
                       int cw, int ph, int pw, int cout, int64_t ldc, int act, bool pool, hipStream_t s) {
    StemParams p{};
    p.x = x;
    p.w = static_cast<const __bf16*>(w);
    p.b = static_cast<const __bf16*>(b);
    p.y = static_cast<__bf16*>(y);
    p.c = c, p.h = h, p.wd = wd, p.pad = pad, p.ch = ch, p.cw = cw, p.ph = ph, p.pw = pw;
    p.cout = cout, p.ldc = static_cast<int>(ldc), p.act = act;
    const int oh = pool ? ph : ch, ow = pool ? pw : cw, edge = pool ? 8 : 16;
    const int64_t tyn = (oh + edge - 1) / edge, txn = (ow + edge - 1) / edge, blocks = tyn * txn * n;
    if (int64_t(c) * h * wd * 4 >= (int64_t(1) << 31) || c < 1 || c > 4) return hipErrorInvalidValue;
    if (blocks >= (int64_t(1) << 31) || (cout + 63) / 64 > 65535) return hipErrorInvalidValue;
    p.tiles = static_cast<int>(tyn * txn), p.tx = static_cast<int>(txn);
    const dim3 grid(static_cast<unsigned>(blocks), static_cast<unsigned>((cout + 63) / 64));
    if (pool)
        launch_kernel(stem_kernel<true>, grid, dim3(256), 0, s, p);
    else
        launch_kernel(stem_kernel<false>, grid, dim3(256), 0, s, p);
    return hipGetLastError();
}

size_t dtype_size(int dtype) { return dtype == MOPAR_BF16 ? 2 : 4; }

}  // namespace mopar
