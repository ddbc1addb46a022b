// MFMA GEMMs for gfx950: the resource-dominant operators (conv as implicit GEMM
// over NHWC activations, linear layers), the boundary autoencoder and the
// LSTM's products.  gemm_kernel, which this comment describes, takes any of them;
// gemm_pp_kernel takes large bf16 products and convs, conv3_halo_kernel small 3x3
// convs (each described at its place).
//
//   C[m, n] = epilogue( sum_k A[m, k] * B[n, k] )
//
// A is [M][K]: a dense row-major matrix or the im2col view of an NHWC image
// (k runs over (r, s, c) with c fastest).  B is [N][K] row-major.
//
// Horizontal sub-slicing (the k equal-size sub-slices of an RD operator): a
// block's sub-slice index selects output columns [lo, hi) and weight rows
// [lo, hi), split as mopar_subslice_range does; each sub-slice is tiled on its
// own and masked at hi (gemm_pp_kernel's tiles run across the edges instead).
// What fixes the arithmetic -- the kernel and so the MFMA shape, the order of the
// k steps, the split-K boundaries (in 64-element units), whether the waves of a
// block share out K, the blocks that float32 sums are made of and the order
// partial sums are added -- is a function of the op alone ((M, N, K), dtype, conv
// geometry), never of the sub-slice count; the rest of a tile's shape and the stage
// depth may follow the sub-slice.  So every output element goes through the same
// fp32 operations whatever k is: sub-sliced output equals the unsplit output bit
// for bit.
//
// Data path.  Operands stream from HBM straight into LDS with buffer_load_dwordx4
// ... lds (16 bytes per lane, no VGPR staging), NS stages deep; a stage holds one
// sub-stage (one per wave on the K-split tiles) and costs one barrier.  A
// sub-stage holds 64 bf16 (32 float) of k for
// every row: 128 bytes, one cache line.  Each load instruction fetches 8 whole rows
// (the DMA writes lane l's 16 bytes to slot l of a 1 KB LDS block); lanes take the
// chunks of a row in XOR-swizzled order (chunk (l % 8) ^ row), so the ds_read_b128
// of an MFMA fragment -- 16 rows, one chunk each -- hits distinct banks.  Each
// operand is a raw buffer resource: a lane's offset is fixed at set-up, the k
// advance of dense operands is a scalar offset, and out-of-range chunks (image
// padding, the K tail) use an offset past the resource, which writes zeros without
// a memory access -- every lane issues the same loads, so the wait counts are
// exact.  The waves run v_mfma_f32_16x16x32_bf16 (bf16) or v_mfma_f32_16x16x4_f32
// (fp32) on their wave tile, with the weight fragment as the first operand: each
// lane ends up holding four consecutive output columns of one row.  The
// accumulators start at the bias (loaded before the operand stages); the epilogue
// stages the fp32 tile through LDS so that each thread finishes whole 8-column
// chunks (residual, activation, one 16-byte store), except that tiles of 32
// columns or fewer store straight from the MFMA layout; the LSTM cell works on the
// MFMA layout directly.
//
// Blocks are numbered so that the eight XCDs (which take blocks round-robin)
// each receive a contiguous run of tiles, grouped eight m-tiles at a time so
// that the blocks an XCD runs together share A rows and B rows in its L2.
#include <type_traits>

#include "internal.h"

namespace mopar {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void* lds_ptr_t;
typedef const __attribute__((address_space(1))) void* gptr_t;

template <typename T> struct Elt;
template <> struct Elt<__bf16> { static constexpr int EPC = 8; };   // elements per 16-byte chunk
template <> struct Elt<float> { static constexpr int EPC = 4; };

// 32 zero bytes: the source of absent epilogue operands.
__device__ __attribute__((aligned(16))) const unsigned int kZeroChunk[8] = {0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u};

// Raw buffer resources: word 3 of the descriptor (32-bit data format) and the lane offset
// that lies past every resource (operand sizes are below 2^31 bytes) and so reads zeros.
constexpr int kRsrcWord3 = 0x00020000;
// m tiles per group in the XCD-local block order
constexpr int kGroupM = 8;
constexpr unsigned kOOB = 0x80000000u;

// Touch every 64-byte line of a kernel's BYTES of arguments at entry: their scalar-cache misses
// then overlap in one wait instead of arriving phase by phase as fields are first used.
template <size_t BYTES>
__device__ __forceinline__ void touch_kernargs() {
    const auto* ka = (const __attribute__((address_space(4))) unsigned*)(__builtin_amdgcn_kernarg_segment_ptr());
    unsigned x = 0;
#pragma unroll
    for (int o = 0; o < static_cast<int>(BYTES / 4); o += 16) x |= ka[o];
    asm volatile("" ::"s"(x));
}

// f(std::integral_constant<int, i>) for i = 0 .. N-1, unrolled at compile time
template <int N, typename F, int I = 0>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<N, F, I + 1>(static_cast<F&&>(f));
    }
}

__device__ __forceinline__ float ld_f(const __bf16* p, int64_t i) {
    unsigned short u = reinterpret_cast<const unsigned short*>(p)[i];
    return __uint_as_float(static_cast<unsigned>(u) << 16);
}
__device__ __forceinline__ float ld_f(const float* p, int64_t i) { return p[i]; }

// whether q is aligned to a whole vector of four elements (8 bytes for bf16, 16 for float)
template <typename T>
__device__ __forceinline__ bool aligned4(const T* q) { return (reinterpret_cast<uintptr_t>(q) & (4 * sizeof(T) - 1)) == 0; }

// four consecutive elements (vector load when the address is aligned)
template <typename T>
__device__ __forceinline__ void ld4(const T* p, int64_t i, int nvalid, float* v) {
    if constexpr (sizeof(T) == 2) {
        if (nvalid == 4 && aligned4(p + i)) {
            const uint2 r = *reinterpret_cast<const uint2*>(p + i);
            v[0] = __uint_as_float(r.x << 16);
            v[1] = __uint_as_float(r.x & 0xffff0000u);
            v[2] = __uint_as_float(r.y << 16);
            v[3] = __uint_as_float(r.y & 0xffff0000u);
            return;
        }
    } else {
        if (nvalid == 4 && aligned4(p + i)) {
            const f32x4 r = *reinterpret_cast<const f32x4*>(p + i);
            v[0] = r[0], v[1] = r[1], v[2] = r[2], v[3] = r[3];
            return;
        }
    }
    for (int q = 0; q < 4; ++q) v[q] = q < nvalid ? ld_f(p, i + q) : 0.0f;
}

__device__ __forceinline__ float sigmoidf_(float v) { return 1.0f / (1.0f + __expf(-v)); }

// erf by formula 7.1.26 of Abramowitz and Stegun's Handbook of Mathematical Functions (absolute
// error at most 1.5e-7): erf(x) = 1 - t (a1 + t (a2 + t (a3 + t (a4 + t a5)))) e^(-x^2) with
// t = 1 / (1 + p x) for x >= 0, odd in x.  Branch-free (the hardware reciprocal and exponential,
// about 1 ulp each, and five multiply-adds), where the library's erf takes several times the
// instructions and branches on |x|: in GELU epilogues it cost a quarter of BERT-base's FFN1
// (9.5 of 39.7 us).  The error is far below the rounding of GELU's result to bf16 and, relative
// to the output's scale, below float32's.
__device__ __forceinline__ float erf_as(float x) {
    const float ax = __builtin_fabsf(x);
    const float t = __builtin_amdgcn_rcpf(1.0f + 0.3275911f * ax);
    const float poly =
        t * (0.254829592f + t * (-0.284496736f + t * (1.421413741f + t * (-1.453152027f + t * 1.061405429f))));
    return __builtin_copysignf(1.0f - poly * __expf(-ax * ax), x);
}

__device__ __forceinline__ float act_f(float v, int act) {
    if (act == MOPAR_ACT_RELU) return v > 0.0f ? v : 0.0f;
    if (act == MOPAR_ACT_GELU) return 0.5f * v * (1.0f + erf_as(v * 0.70710678118654752f));
    return v;
}

// four consecutive elements to c + idx (vector store when the address is aligned: a branch
// written into a concatenated tensor may start at any channel)
template <typename T>
__device__ __forceinline__ void store4(T* c, int64_t idx, const float* v, int nvalid) {
    if constexpr (sizeof(T) == 2) {
        if (nvalid == 4 && aligned4(c + idx)) {
            const bf16x4 o = {(__bf16)v[0], (__bf16)v[1], (__bf16)v[2], (__bf16)v[3]};
            *reinterpret_cast<bf16x4*>(c + idx) = o;
            return;
        }
    } else {
        if (nvalid == 4 && aligned4(c + idx)) {
            *reinterpret_cast<f32x4*>(c + idx) = f32x4{v[0], v[1], v[2], v[3]};
            return;
        }
    }
    for (int q = 0; q < nvalid; ++q) c[idx + q] = static_cast<T>(v[q]);
}

// eight consecutive elements as raw bits (one 16-byte load for bf16, two for float32)
template <typename T> struct Raw8 { uint4 w[sizeof(T) / 2]; };

__device__ __forceinline__ bool aligned16(const void* q) { return (reinterpret_cast<uintptr_t>(q) & 15) == 0; }

template <typename T>
__device__ __forceinline__ void unpack8(const Raw8<T>& r, float (&v)[8]) {
    if constexpr (sizeof(T) == 2) {
        const unsigned w[4] = {r.w[0].x, r.w[0].y, r.w[0].z, r.w[0].w};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            v[2 * q] = __uint_as_float(w[q] << 16);
            v[2 * q + 1] = __uint_as_float(w[q] & 0xffff0000u);
        }
    } else {
        const unsigned w[8] = {r.w[0].x, r.w[0].y, r.w[0].z, r.w[0].w, r.w[1].x, r.w[1].y, r.w[1].z, r.w[1].w};
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = __uint_as_float(w[q]);
    }
}

// v[0..7] = p[i..i+7] for the first nvalid elements, 0 after them (and everywhere when p is null)
template <typename T>
__device__ __forceinline__ void load8(const T* p, int64_t i, int nvalid, float (&v)[8]) {
    if (p && nvalid == 8 && aligned16(p + i)) {
        unpack8<T>(*reinterpret_cast<const Raw8<T>*>(p + i), v);
        return;
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = (p && q < nvalid) ? ld_f(p, i + q) : 0.0f;
}

// four consecutive elements as raw bits (8 bytes for bf16, 16 for float)
template <typename T> struct Raw4Sel { using type = uint4; };
template <> struct Raw4Sel<__bf16> { using type = uint2; };
template <typename T> using Raw4 = typename Raw4Sel<T>::type;

// the 4 elements at q (8-byte aligned for bf16, 16 for float), or zeros from the zero page when
// q is null: one unconditional load either way
template <typename T>
__device__ __forceinline__ Raw4<T> load_raw4(const T* q, const void* zero_page) {
    // through a global-address-space pointer, so it is a global (not flat) load
    const void* src = q ? static_cast<const void*>(q) : zero_page;
    Raw4<T> r;
    if constexpr (sizeof(T) == 2) {
        const unsigned long long v = *(const __attribute__((address_space(1))) unsigned long long*)(src);
        r.x = static_cast<unsigned>(v);
        r.y = static_cast<unsigned>(v >> 32);
    } else {
        typedef unsigned w4_t __attribute__((ext_vector_type(4)));
        const w4_t v = *(const __attribute__((address_space(1))) w4_t*)(src);
        r.x = v[0], r.y = v[1], r.z = v[2], r.w = v[3];
    }
    return r;
}
template <typename T>
__device__ __forceinline__ void unpack4(const Raw4<T>& r, float (&v)[4]) {
    if constexpr (sizeof(T) == 2) {
        v[0] = __uint_as_float(r.x << 16);
        v[1] = __uint_as_float(r.x & 0xffff0000u);
        v[2] = __uint_as_float(r.y << 16);
        v[3] = __uint_as_float(r.y & 0xffff0000u);
    } else {
        v[0] = __uint_as_float(r.x), v[1] = __uint_as_float(r.y), v[2] = __uint_as_float(r.z), v[3] = __uint_as_float(r.w);
    }
}
// the 4 floats at q (16-byte aligned), or zeros from the zero page when q is null: one
// unconditional global load either way
__device__ __forceinline__ f32x4 load_f32x4(const float* q, const void* zero_page) {
    const void* src = q ? static_cast<const void*>(q) : zero_page;
    return *(const __attribute__((address_space(1))) f32x4*)(src);
}

// p[i .. i+nvalid-1] (zeros after them, and everywhere when p is null), element by element
template <typename T>
__device__ __forceinline__ void ld4_or_zero(const T* p, int64_t i, int nvalid, float (&v)[4]) {
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = (p && q < nvalid) ? ld_f(p, i + q) : 0.0f;
}

// the 16 (bf16) or 32 (float) bytes at q, or zeros from the zero page when q is null: one
// unconditional load either way
template <typename T>
__device__ __forceinline__ Raw8<T> load_raw8(const T* q, const void* zero_page) {
    // through a global-address-space pointer, so it is a global (not flat) load
    typedef unsigned w4_t __attribute__((ext_vector_type(4)));
    const auto* src = (const __attribute__((address_space(1))) w4_t*)(q ? static_cast<const void*>(q) : zero_page);
    Raw8<T> r;
#pragma unroll
    for (int h = 0; h < static_cast<int>(sizeof(T)) / 2; ++h) {
        const w4_t v = src[h];
        r.w[h] = make_uint4(v[0], v[1], v[2], v[3]);
    }
    return r;
}

template <typename T>
__device__ __forceinline__ void store8(T* c, int64_t idx, const float (&v)[8], int nvalid) {
    if (nvalid == 8 && aligned16(c + idx)) {
        if constexpr (sizeof(T) == 2) {
            const bf16x8 o = {(__bf16)v[0], (__bf16)v[1], (__bf16)v[2], (__bf16)v[3],
                              (__bf16)v[4], (__bf16)v[5], (__bf16)v[6], (__bf16)v[7]};
            *reinterpret_cast<bf16x8*>(c + idx) = o;
        } else {
            *reinterpret_cast<f32x4*>(c + idx) = f32x4{v[0], v[1], v[2], v[3]};
            *reinterpret_cast<f32x4*>(c + idx + 4) = f32x4{v[4], v[5], v[6], v[7]};
        }
        return;
    }
    for (int q = 0; q < nvalid; ++q) c[idx + q] = static_cast<T>(v[q]);
}

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

// LDS fragment reads.  They are issued as inline asm so the compiler does not
// treat them as readers of the in-flight LDS DMA (it would otherwise drain every
// outstanding global_load_lds before each read, collapsing the pipeline to one
// stage); completion is awaited explicitly with lds_wait(), and pin() ties each
// value to that wait so no use can be scheduled above it.
__device__ __forceinline__ u32x4 lds_read16(unsigned addr) {
    u32x4 v;
    asm volatile("ds_read_b128 %0, %1" : "=v"(v) : "v"(addr));
    return v;
}
// One 16-byte chunk per lane from the raw buffer [base, base + size) at byte offset voff + soff
// (soff wave-uniform) into LDS slot lane of the 1 KB block at dst; an offset voff >= size
// writes zeros.  (The resource is built here, in a plain device function, and not in the
// kernel templates.)
__device__ __forceinline__ void buffer_load_lds(const void* base, unsigned size, lds_ptr_t dst, unsigned voff,
                                                unsigned soff) {
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), static_cast<short>(0),
                                                                      static_cast<int>(size), kRsrcWord3);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, dst, 16, voff, soff, 0, 0);
}

template <int OFF>
__device__ __forceinline__ u32x4 lds_read16_at(unsigned addr) {
    static_assert(OFF >= 0 && OFF < 65536, "ds offset");
    u32x4 v;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF));
    return v;
}
__device__ __forceinline__ void lds_wait() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }
template <int N>
__device__ __forceinline__ void lds_wait_until() {
    static_assert(N >= 0 && N <= 15, "lgkmcnt range");
    asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(N) : "memory");
}
__device__ __forceinline__ void pin(u32x4& v) { asm volatile("" : "+v"(v)); }

// wait until at most `r` of this wave's stages (L loads each) are still in flight
template <int L>
__device__ __forceinline__ void wait_stages(int r) {
    switch (r) {
        case 0: asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); break;
        case 1: asm volatile("s_waitcnt vmcnt(%0)" ::"n"(L) : "memory"); break;
        case 2: asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * L) : "memory"); break;
        case 3: asm volatile("s_waitcnt vmcnt(%0)" ::"n"(3 * L) : "memory"); break;
        case 4: asm volatile("s_waitcnt vmcnt(%0)" ::"n"(4 * L < 63 ? 4 * L : 63) : "memory"); break;
        case 5: asm volatile("s_waitcnt vmcnt(%0)" ::"n"(5 * L < 63 ? 5 * L : 63) : "memory"); break;
        case 6: asm volatile("s_waitcnt vmcnt(%0)" ::"n"(6 * L < 63 ? 6 * L : 63) : "memory"); break;
        default: asm volatile("s_waitcnt vmcnt(%0)" ::"n"(7 * L < 63 ? 7 * L : 63) : "memory"); break;
    }
}

// Waves a SIMD has to hold: the conv form of the float32 128 x 128 tiles keeps two blocks on a CU (its block sums took
// it to 136 registers, one block: 3x3 convs over 32 x 56 x 56 x 128 292 us with two, 330 with one).
template <typename T, int BM, int BN, bool CONV>
constexpr int min_waves() { return sizeof(T) == 4 && BM == 128 && BN == 128 && CONV ? 4 : 1; }

// KS > 1: the KS waves of a block share one wave tile (the whole block tile) and split K
// instead: a stage holds KH = KS sub-stages and wave w computes sub-stage w of each, so the
// serial K loop is KS times shorter; the waves' sums are added in wave order at the end.
template <typename T, int BM, int BN, int WM, int WN, int NS, int KH, int KS, bool CONV>
__global__ __launch_bounds__(WM * WN * KS * 64, (min_waves<T, BM, BN, CONV>())) void gemm_kernel(const GemmParams p) {
    constexpr int EPC = Elt<T>::EPC;
    constexpr int BK = 8 * EPC;                 // K elements per sub-stage: two 32-wide (bf16) k steps
    constexpr int TM = BM / WM, TN = BN / WN;   // wave tile
    constexpr int FM = TM / 16, FN = TN / 16;   // 16x16 MFMA tiles per wave
    constexpr int NBA = BM / 16 * 2, NBB = BN / 16 * 2;
    constexpr int NBLK = NBA + NBB;             // 1 KB fragment blocks per stage
    constexpr int NW = WM * WN * KS, NT = NW * 64;   // waves and threads per block
    constexpr int LA = (NBA + NW - 1) / NW, LB = (NBB + NW - 1) / NW;   // load slots per wave
    constexpr int LMIN = NBA / NW + NBB / NW;   // loads per sub-stage issued by every wave
    constexpr int STAGE = NBLK * 64;            // uint4 per sub-stage
    constexpr int SSTAGE = KH * STAGE;          // uint4 per stage: KH sub-stages, one barrier
    static_assert((NW == 4 || NW == 8) && FM >= 1 && FN >= 1 && NS >= 2 && NS <= 9 && LMIN >= 1, "tile");
    static_assert(KH == 1 || KH == 2 || KH == 4, "sub-stages per stage");
    static_assert(KS == KH && (KS == 1 || (WM == 1 && WN == 1)), "K split across waves: one sub-stage per wave");
    static_assert((NS - 2) * LMIN * KH <= 63, "vmcnt range");

    constexpr int LDT = BN + 4;                 // fp32 row stride of the staged output tile (padded)
    constexpr int TILE_U4 = (KS * BM * LDT + 3) / 4;   // staged output tile(s), one per K-split wave
    constexpr int LDS_U4 = NS * SSTAGE > TILE_U4 ? NS * SSTAGE : TILE_U4;
    __shared__ uint4 lds[LDS_U4];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // scalar: load blocks are wave-uniform
    const int wt = KS > 1 ? 0 : wave;           // wave-tile index
    const int kw = KS > 1 ? wave : 0;           // K-split index
    const int wm = wt / WN, wn = wt % WN;

    // --- block -> (m tile, split, sub-slice, n tile), XCD-grouped -------------------------
    // (all divisions by launch constants go through precomputed multipliers)
    touch_kernargs<sizeof(GemmParams)>();
    const unsigned t = (blockIdx.x % 8) * static_cast<unsigned>(p.g_per_xcd) + blockIdx.x / 8;
    if (t >= static_cast<unsigned>(p.g_total)) return;
    // within an XCD's run, tiles go in groups of GM m-tiles x every column (split, sub-slice,
    // n-tile), m fastest: the blocks resident together share both A rows and B rows in L2
    constexpr int GM = kGroupM;
    const unsigned group = p.g_div_group.div(t);
    const unsigned within = t - group * static_cast<unsigned>(GM * p.g_cols);
    const bool last = static_cast<int>(group) == (p.g_mt - 1) / GM;   // the last group may be short
    const unsigned gm = last ? static_cast<unsigned>(p.g_mt - group * GM) : GM;
    const unsigned colu = last ? p.g_div_last.div(within) : within / GM;
    const int mti = static_cast<int>(group * GM + (within - colu * gm));
    const unsigned c1 = p.g_div_nt.div(colu);
    const int nti = static_cast<int>(colu - c1 * static_cast<unsigned>(p.g_nt));
    const unsigned c2 = p.g_div_ksub.div(c1);
    const int j = static_cast<int>(c1 - c2 * static_cast<unsigned>(p.ksub));
    const int split = static_cast<int>(c2);

    const int q = p.g_q, rr = p.g_rr;
    const int n_lo = j * q + min(j, rr), n_hi = (j + 1) * q + min(j + 1, rr);
    const int n0 = n_lo + nti * BN;
    if (n0 >= n_hi) return;                     // block-uniform, before any barrier
    // rows fit in 32 bits (M <= 2^31 - 256, checked at launch); output offsets are 64-bit
    const int Mi = static_cast<int>(p.M);
    const int m0 = mti * BM;

    // this split's sub-stages [u0, u1): boundaries in BK units, whatever KH is
    const int nk = p.g_nk;
    const int u0 = static_cast<int>(p.g_div_splits.div(static_cast<unsigned>(nk * split)));
    const int u1 = static_cast<int>(p.g_div_splits.div(static_cast<unsigned>(nk * (split + 1))));
    const int nst = (u1 - u0 + KH - 1) / KH;    // stages; sub-stages past u1 re-read u0, run no MFMA

    // --- operand loads ----------------------------------------------------------------------
    // Each operand is read through a raw buffer resource: a lane's chunk address is a fixed
    // per-lane byte offset (VGPR) plus a per-sub-stage offset that only the scalar unit
    // advances (dense operands), and a lane whose offset is kOOB -- past the resource's size
    // -- writes zeros to LDS without touching memory (image padding, K tail).
    // Load block blk of a sub-stage covers 8 rows x 128 bytes (whole cache lines): lane l
    // loads row 8 * blk + l / 8, k chunk cl = (l % 8) ^ (l / 8) -- the XOR swizzle that keeps
    // the fragment reads conflict-free -- into LDS slot l of the block.  Wave w loads A blocks
    // w, w + NW, ... and B blocks w, w + NW, ...: slots are fixed at compile time, and only a
    // last, partial round of slots tests the wave index.
    const int cl = (lane & 7) ^ (lane >> 3);    // this lane's chunk of every sub-stage, 0..7
    // Rows past M (A) or past the sub-slice (B) load a real row (the last valid one) instead:
    // the products they feed are never stored.
    // Dense A and B: voff = byte offset of (row, chunk cl of sub-stage 0).  Conv A: voff =
    // offset of the window's top-left pixel (two's complement when the window starts in the
    // padding), with the window corner (hb, wb) for the bounds test.
    unsigned voffA[LA], voffB[LB];
    int hb[LA], wb[LA];
#pragma unroll
    for (int i = 0; i < LA; ++i) {
        const int blk = min(wave + NW * i, NBA - 1);
        const int m = m0 + blk * 8 + (lane >> 3);
        const int mc = m < Mi ? m : Mi - 1;
        hb[i] = wb[i] = 0;
        if constexpr (CONV) {
            // M < 2^31, so the pixel decode runs in 32 bits with precomputed divisors
            const unsigned mu = static_cast<unsigned>(mc);
            const unsigned img = p.div_hw.div(mu);
            const unsigned rem = mu - img * static_cast<unsigned>(p.out_h * p.out_w);
            const unsigned ho = p.div_w.div(rem), wo = rem - ho * static_cast<unsigned>(p.out_w);
            hb[i] = static_cast<int>(ho) * p.stride - p.pad;
            wb[i] = static_cast<int>(wo) * p.stride - p.pad;
            const int pix = (static_cast<int>(img) * p.img_h + hb[i]) * p.img_w + wb[i];
            voffA[i] = static_cast<unsigned>(pix) * static_cast<unsigned>(p.cs * sizeof(T));
        } else {
            // (A spans less than 2^31 bytes, so the offset of row mc fits in 32 bits)
            voffA[i] = static_cast<unsigned>(mc) * static_cast<unsigned>(p.lda * sizeof(T)) + static_cast<unsigned>(cl * 16);
        }
    }
#pragma unroll
    for (int i = 0; i < LB; ++i) {
        const int blk = min(wave + NW * i, NBB - 1);
        const int n = n0 + blk * 8 + (lane >> 3);
        const int nc = n < n_hi ? n : n_hi - 1;
        voffB[i] = static_cast<unsigned>(nc) * static_cast<unsigned>(p.K * sizeof(T)) + static_cast<unsigned>(cl * 16);
    }

    // im2col coordinates (tap row, tap column, channel) of this lane's chunk, advanced
    // incrementally by one sub-stage: BK = (dqr * kw + dqc) * cs + dc elements
    int tr = 0, tcol = 0, tci = 0;
    const int dqr = p.dqr, dqc = p.dqc, dc = p.dc;
    if (CONV) {
        const unsigned k = static_cast<unsigned>(u0 * BK + cl * EPC);
        const unsigned tap = p.div_cs.div(k);
        tci = static_cast<int>(k - tap * static_cast<unsigned>(p.cs));
        const unsigned r = p.div_kw.div(tap);
        tr = static_cast<int>(r);
        tcol = static_cast<int>(tap - r * static_cast<unsigned>(p.kw));
    }
    auto advance = [&]() {
        tci += dc;
        const int carry = tci >= p.cs ? 1 : 0;
        tci -= carry * p.cs;
        tcol += dqc + carry;                    // < 2 kw: one wrap at most
        tr += dqr;
        if (tcol >= p.kw) {
            tcol -= p.kw;
            ++tr;
        }
    };

    // Loads of sub-stage kt (conv coordinates must be those of kt) into LDS at dst.  A dead
    // sub-stage (past the split: its MFMAs are skipped) re-reads sub-stage u0, so that every
    // sub-stage issues the same loads and the wait counts stay exact.
    const int ktail = (p.K % BK) ? nk - 1 : nk;   // the one sub-stage whose chunks may pass K
    auto issue = [&](int kt, uint4* dst, bool live) {
        const int ku = live ? kt : u0;
        const unsigned soff = static_cast<unsigned>(ku) * (BK * sizeof(T));
        const bool tail = ku == ktail;          // uniform
        const bool kin = !tail || ku * BK + cl * EPC < p.K;
        const unsigned koff = CONV ? static_cast<unsigned>(((tr * p.img_w + tcol) * p.cs + tci) * sizeof(T)) : 0u;
#pragma unroll
        for (int i = 0; i < LA; ++i) {
            if (NBA % NW != 0 && i == LA - 1 && wave + NW * i >= NBA) break;   // wave-uniform
            unsigned v;
            if constexpr (CONV) {
                const bool ok = kin && static_cast<unsigned>(hb[i] + tr) < static_cast<unsigned>(p.img_h) &&
                                static_cast<unsigned>(wb[i] + tcol) < static_cast<unsigned>(p.img_w);
                v = ok ? voffA[i] + koff : kOOB;
            } else {
                v = kin ? voffA[i] : kOOB;
            }
            buffer_load_lds(p.A, p.a_bytes, (lds_ptr_t)(dst + (wave + NW * i) * 64), v, CONV ? 0u : soff);
        }
#pragma unroll
        for (int i = 0; i < LB; ++i) {
            if (NBB % NW != 0 && i == LB - 1 && wave + NW * i >= NBB) break;
            buffer_load_lds(p.B, p.b_bytes, (lds_ptr_t)(dst + (NBA + wave + NW * i) * 64), kin ? voffB[i] : kOOB, soff);
        }
    };
    // stage st: sub-stages u0 + st * KH + h into buffer buf, conv coordinates advanced past them
    auto issue_stage = [&](int st, int buf) {
#pragma unroll
        for (int h = 0; h < KH; ++h) {
            const int kt = u0 + st * KH + h;
            issue(kt, &lds[buf * SSTAGE + h * STAGE], kt < u1);
            if (CONV) advance();
        }
    };

    f32x4 acc[FM][FN];
#pragma unroll
    for (int a = 0; a < FM; ++a)
#pragma unroll
        for (int b = 0; b < FN; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};

    // --- epilogue set-up ---------------------------------------------------------------------
    // MFMA layout: lane holds row mrow[a], columns ncol[b]..+3
    int mrow[FM];
    int ncol[FN], nval[FN];
#pragma unroll
    for (int a = 0; a < FM; ++a) mrow[a] = m0 + wm * TM + a * 16 + (lane & 15);
#pragma unroll
    for (int b = 0; b < FN; ++b) {
        ncol[b] = n0 + wn * TN + b * 16 + (lane >> 4) * 4;
        nval[b] = max(0, min(4, n_hi - ncol[b]));
    }
    // chunk layout (everything else): thread owns 8 consecutive columns c0..c0+7 of tile
    // rows cr, cr + RPP, ...; after the staging through LDS each chunk is one 16-byte store
    constexpr int CPR = BN / 8, RPP = NT / CPR, NCH = (BM + RPP - 1) / RPP;
    const int cc = threadIdx.x % CPR, cr = threadIdx.x / CPR;
    const int c0 = n0 + cc * 8;
    const int cval = max(0, min(8, n_hi - c0));
    const bool direct = p.splits == 1 && p.epi == EPI_STD;   // this block finishes its outputs
    // A direct launch starts its accumulators at bias + second bias.  Their raw bits (MFMA
    // layout: 4 columns per lane and fragment) are loaded here, before the operand stages, and
    // added after the prologue: the latency hides under the first stage's.  Each is one load
    // per lane, from the zero page when absent; partial column groups are read element by
    // element up front.  With K split across waves only wave 0 starts from them.  (The residual is added in the epilogue, in
    // the chunk layout whose 16-byte loads cover whole lines: in the MFMA layout its 8-byte
    // loads were measured slower.)
    const T* biasp = static_cast<const T*>(p.bias);
    const T* bias2p = static_cast<const T*>(p.bias2);
    const T* resp = static_cast<const T*>(p.res);
    const bool init_here = direct && (KS == 1 || kw == 0);
    // (Loads whose results a path never reads would leave their registers pending there, and
    // the compiler would then drain every load in flight, operand stages included, when it
    // reuses those registers inside the K loop: each of these loads is issued only under the
    // wave-uniform condition under which it is added.)
    Raw4<T> rb[FN], rb2[FN];
    bool bfast[FN];
    float bslow[FN][4];                         // partial groups: summed bias, read up front
#pragma unroll
    for (int b = 0; b < FN; ++b) {
        bfast[b] = nval[b] == 4;
        if (init_here) {
            rb[b] = load_raw4<T>(bfast[b] && biasp ? biasp + ncol[b] : nullptr, kZeroChunk);
            rb2[b] = load_raw4<T>(bfast[b] && bias2p ? bias2p + ncol[b] : nullptr, kZeroChunk);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) bslow[b][e] = 0.0f;
        // (element loads under a per-lane branch: done before any operand load is in flight,
        // since the wait they need would otherwise drain the operand stages too)
        if (init_here && !bfast[b]) {
            float bv[4], b2v[4];
            ld4_or_zero<T>(biasp, ncol[b], nval[b], bv);
            ld4_or_zero<T>(bias2p, ncol[b], nval[b], b2v);
#pragma unroll
            for (int e = 0; e < 4; ++e) bslow[b][e] = bv[e] + b2v[e];
        }
    }
    // An LSTM step starts wave 0's accumulators at the gate pre-activations gx (fp32, loaded
    // here in the same way): the epilogue then only applies the cell.
    const bool lstm_here = p.epi == EPI_LSTM && (KS == 1 || kw == 0);
    f32x4 rgx[FM][FN];
    if (lstm_here) {
#pragma unroll
        for (int a = 0; a < FM; ++a)
#pragma unroll
            for (int b = 0; b < FN; ++b) {
                const bool ok = mrow[a] < Mi && nval[b] == 4;
                rgx[a][b] = load_f32x4(ok ? p.gx + static_cast<int64_t>(mrow[a]) * p.ldgx + ncol[b] : nullptr, kZeroChunk);
            }
    }

    // prologue: NS-1 stages in flight (coordinates then stand at stage NS - 1); stages past
    // the split re-read its first sub-stage, and are issued anyway so that the loads in flight
    // at this point do not depend on the path
#pragma unroll
    for (int s = 0; s < NS - 1; ++s) issue_stage(s, s);

    if (lstm_here) {
#pragma unroll
        for (int a = 0; a < FM; ++a)
#pragma unroll
            for (int b = 0; b < FN; ++b) acc[a][b] = rgx[a][b];
    }
    if (init_here) {
#pragma unroll
        for (int b = 0; b < FN; ++b) {
            float bv[4], b2v[4];
            unpack4<T>(rb[b], bv);
            unpack4<T>(rb2[b], b2v);
#pragma unroll
            for (int a = 0; a < FM; ++a)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[a][b][e] = bfast[b] ? bv[e] + b2v[e] : bslow[b][e];
        }
    }
    // The accumulators now hold values computed from loads; pinning them here makes the
    // compiler settle those loads once, before the K loop.  (Otherwise it treats the
    // accumulators as possibly pending loads inside the loop and waits there for every load
    // in flight, the operand stages just issued included.)
#pragma unroll
    for (int a = 0; a < FM; ++a)
#pragma unroll
        for (int b = 0; b < FN; ++b) asm volatile("" : "+v"(acc[a][b]));

    // LDS byte addresses of this lane's MFMA fragments (row l % 16 of a 16-row block, chunk
    // 4 * ks + l / 16) in stage buffer 0, sub-stage 0, for the wave's first A and B rows;
    // the other fragments sit at compile-time offsets from them
    const unsigned lds0 = static_cast<unsigned>(reinterpret_cast<size_t>((lds_ptr_t)(&lds[0])));
    unsigned fa[2], fb[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        const unsigned f = lds0 + ((((lane >> 3) & 1) * 64 + (lane & 7) * 8 + ((ks * 4 + (lane >> 4)) ^ (lane & 7))) * 16);
        fa[ks] = f + ((wm * TM) >> 3) * 1024;
        fb[ks] = f + (NBA + ((wn * TN) >> 3)) * 1024;
    }
    auto read_frags = [&](unsigned sbase, int ks, u32x4 (&af)[FM], u32x4 (&bf)[FN]) {
        const unsigned ab = sbase + fa[ks], bb = sbase + fb[ks];
        static_for<FM>([&](auto a) { af[a] = lds_read16_at<a * 2048>(ab); });
        static_for<FN>([&](auto b) { bf[b] = lds_read16_at<b * 2048>(bb); });
    };
    // float32 sums in blocks of 128 of k (64 per wave where the waves split K), added up in order: a rounding
    // error that grows with the number of blocks plus the length of one instead of with K (a float32
    // BERT-base layer on 4 x 77 tokens: 7.0e-7 of the result without, 3.2e-7 with).  They cost 2 to 3 % of a large
    // product (8192 x 768 -> 3072 290 -> 297 us) and were 7 % on wave tiles of one MFMA tile (3x3 convs over 32 x 64
    // x 64 x 16 13.6 -> 14.6 us), which add a block's sum to the total under the next block's first MFMAs, from zero;
    // on larger wave tiles that costs registers, and with them a CU's second block.
    constexpr bool BLOCKED = sizeof(T) == 4, MERGED = BLOCKED && FM * FN == 1;
    f32x4 total[BLOCKED ? FM : 1][BLOCKED ? FN : 1];
    if constexpr (BLOCKED) {
#pragma unroll
        for (int a = 0; a < FM; ++a)
#pragma unroll
            for (int b = 0; b < FN; ++b) total[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    auto flush = [&](int a, int b) {
        if constexpr (BLOCKED) total[a][b] += acc[a][b], acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
    };
    auto block_ends = [&](int st) { return BLOCKED && st > 0 && st % (KS == 1 ? 4 : 2) == 0; };   // before stage st
    auto mfmas = [&](u32x4 (&af)[FM], u32x4 (&bf)[FN], auto next_block) {
#pragma unroll
        for (int a = 0; a < FM; ++a)
#pragma unroll
            for (int b = 0; b < FN; ++b) {
                if constexpr (sizeof(T) == 2) {
                    acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                        __builtin_bit_cast(bf16x8, bf[b]), __builtin_bit_cast(bf16x8, af[a]), acc[a][b], 0, 0, 0);
                } else {
                    const f32x4 av = __builtin_bit_cast(f32x4, af[a]);
                    const f32x4 bv = __builtin_bit_cast(f32x4, bf[b]);
                    if constexpr (decltype(next_block)::value) flush(a, b);
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(bv[e], av[e], acc[a][b], 0, 0, 0);
                }
            }
    };

    // the first k step of stage st (block-uniform choice)
    auto mfmas_first = [&](int st, u32x4 (&af)[FM], u32x4 (&bf)[FN]) {
        if (MERGED && block_ends(st))
            mfmas(af, bf, std::true_type{});
        else
            mfmas(af, bf, std::false_type{});
    };
    auto flush_all = [&]() {
#pragma unroll
        for (int a = 0; a < FM; ++a)
#pragma unroll
            for (int b = 0; b < FN; ++b) flush(a, b);
    };
    for (int st = 0; st < nst; ++st) {
        const int buf = st % NS;
        const int later = min(NS - 2, nst - 1 - st);   // stages issued after this one
        if (!MERGED && block_ends(st)) flush_all();
        wait_stages<LMIN * KH>(later);                 // this wave's share of stage st has landed
        __builtin_amdgcn_s_barrier();                  // every wave's share has; stage st-1 fully consumed
        if (st + NS - 1 < nst) issue_stage(st + NS - 1, (st + NS - 1) % NS);
        const unsigned sbase = buf * SSTAGE * 16;
        u32x4 a0[FM], b0[FN], a1[FM], b1[FN];
        if constexpr (KS > 1) {
            // this wave's sub-stage of the stage (uniform skip when it lies past the split)
            if (u0 + st * KH + kw >= u1) continue;
            const unsigned hb = sbase + kw * STAGE * 16;
            read_frags(hb, 0, a0, b0);
            lds_wait();
#pragma unroll
            for (int a = 0; a < FM; ++a) pin(a0[a]);
#pragma unroll
            for (int b = 0; b < FN; ++b) pin(b0[b]);
            read_frags(hb, 1, a1, b1);
            mfmas_first(st, a0, b0);
        } else if constexpr (FM + FN <= 3) {
            // thin wave tiles: both k steps' fragment reads go out together; LDS reads complete
            // in order, so once at most FM + FN are outstanding the first step's have landed
            read_frags(sbase, 0, a0, b0);
            read_frags(sbase, 1, a1, b1);
            lds_wait_until<FM + FN>();
#pragma unroll
            for (int a = 0; a < FM; ++a) pin(a0[a]);
#pragma unroll
            for (int b = 0; b < FN; ++b) pin(b0[b]);
            mfmas_first(st, a0, b0);
            __builtin_amdgcn_sched_barrier(0);         // keep these MFMAs ahead of the next wait
        } else {
            // wide wave tiles: holding both steps' fragments would cost the registers that
            // keep two blocks per CU resident; the second step's reads follow the first's wait
            read_frags(sbase, 0, a0, b0);
            lds_wait();
#pragma unroll
            for (int a = 0; a < FM; ++a) pin(a0[a]);
#pragma unroll
            for (int b = 0; b < FN; ++b) pin(b0[b]);
            read_frags(sbase, 1, a1, b1);
            mfmas_first(st, a0, b0);
        }
        lds_wait();
#pragma unroll
        for (int a = 0; a < FM; ++a) pin(a1[a]);
#pragma unroll
        for (int b = 0; b < FN; ++b) pin(b1[b]);
        mfmas(a1, b1, std::false_type{});
    }

    if constexpr (BLOCKED) {
        flush_all();
#pragma unroll
        for (int a = 0; a < FM; ++a)
#pragma unroll
            for (int b = 0; b < FN; ++b) acc[a][b] = total[a][b];
    }

    // --- epilogue --------------------------------------------------------------------------
    // The fp32 tile goes through LDS (row-major, padded rows; one copy per K-split wave,
    // added in wave order when read back).
    float* tile = reinterpret_cast<float*>(lds);
    auto stage_tile = [&]() {
        __syncthreads();                      // every wave is done with the operand stages
#pragma unroll
        for (int a = 0; a < FM; ++a)
#pragma unroll
            for (int b = 0; b < FN; ++b) {
                const int row = wm * TM + a * 16 + (lane & 15), col = wn * TN + b * 16 + (lane >> 4) * 4;
                *reinterpret_cast<f32x4*>(tile + (kw * BM + row) * LDT + col) = acc[a][b];
            }
        __syncthreads();
    };
    auto tile4 = [&](int row, int col) {
        f32x4 v = *reinterpret_cast<const f32x4*>(tile + row * LDT + col);
#pragma unroll
        for (int w = 1; w < KS; ++w) v += *reinterpret_cast<const f32x4*>(tile + (w * BM + row) * LDT + col);
        return v;
    };
    if constexpr (KS > 1) {
        stage_tile();
        // the summed tile back in the MFMA layout, for the row tiles this wave finishes
#pragma unroll
        for (int a = 0; a < FM; ++a)
#pragma unroll
            for (int b = 0; b < FN; ++b)
                if (a % KS == kw) acc[a][b] = tile4(a * 16 + (lane & 15), b * 16 + (lane >> 4) * 4);
    }
    if (p.epi == EPI_LSTM) {
        // gates i, f, g, o of unit n / 4 (n is a multiple of 4 and the whole group is valid),
        // gx already in the sums; with K split across waves, wave w finishes row tiles
        // a = w (mod KS)
        float cprev[FM][FN];
#pragma unroll
        for (int a = 0; a < FM; ++a)
#pragma unroll
            for (int b = 0; b < FN; ++b) {
                const bool ok = a % KS == kw && mrow[a] < Mi && nval[b] == 4;
                const int64_t mm = ok ? mrow[a] : 0;
                const int nn = ok ? ncol[b] : 0;
                cprev[a][b] = p.cstate[mm * (p.N >> 2) + (nn >> 2)];
            }
#pragma unroll
        for (int a = 0; a < FM; ++a)
#pragma unroll
            for (int b = 0; b < FN; ++b) {
                if (a % KS != kw || mrow[a] >= Mi || nval[b] != 4) continue;
                const f32x4 v = acc[a][b];
                const float c = sigmoidf_(v[1]) * cprev[a][b] + sigmoidf_(v[0]) * tanhf(v[2]);
                const int u = ncol[b] >> 2;
                p.cstate[static_cast<int64_t>(mrow[a]) * (p.N >> 2) + u] = c;
                static_cast<T*>(p.C)[static_cast<int64_t>(mrow[a]) * p.ldc + u] = static_cast<T>(sigmoidf_(v[3]) * tanhf(c));
            }
        return;
    }

    // Narrow tiles (32 columns or fewer) store straight from the MFMA layout: a lane's four
    // consecutive columns are one 8-byte (bf16) store, and the LDS round trip costs more than
    // the shorter stores save (measured).
    if constexpr (KS == 1 && BN <= 32) {
        if (direct) {
#pragma unroll
            for (int a = 0; a < FM; ++a)
#pragma unroll
                for (int b = 0; b < FN; ++b) {
                    if (mrow[a] >= Mi || nval[b] == 0) continue;
                    const int64_t idx = static_cast<int64_t>(mrow[a]) * p.ldc + ncol[b];
                    float v[4], rv[4] = {0.f, 0.f, 0.f, 0.f};
                    if (resp) ld4<T>(resp, idx, nval[b], rv);
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = act_f(acc[a][b][e] + rv[e], p.act);
                    if (p.out_f32)
                        store4<float>(static_cast<float*>(p.C), idx, v, nval[b]);
                    else
                        store4<T>(static_cast<T*>(p.C), idx, v, nval[b]);
                }
            return;
        }
    }
    // Otherwise every thread owns whole 8-column chunks of the staged tile: full-line stores.
    if constexpr (KS == 1) stage_tile();
    auto tile8 = [&](int r, float (&v)[8]) {
        const f32x4 lo = tile4(r, cc * 8), hi = tile4(r, cc * 8 + 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = lo[e], v[4 + e] = hi[e];
    };
    if (direct) {
        // bias is already in the sums: residual, activation, store.  The residual chunks of
        // all this thread's rows go out together before any is used (a load under each row's
        // own conditions would wait for the one before it); partial or unaligned chunks are
        // read element by element when used.
        Raw8<T> rraw[NCH];
        bool rfast[NCH];
        if (resp) {
#pragma unroll
            for (int i = 0; i < NCH; ++i) {
                const int r = cr + i * RPP;
                const int m = m0 + r;
                const int64_t idx = static_cast<int64_t>(m) * p.ldc + c0;
                rfast[i] = r < BM && m < Mi && cval == 8 && aligned16(resp + idx);
                rraw[i] = load_raw8<T>(rfast[i] ? resp + idx : nullptr, kZeroChunk);
            }
        }
#pragma unroll
        for (int i = 0; i < NCH; ++i) {
            const int r = cr + i * RPP;
            const int m = m0 + r;
            if (r >= BM || m >= Mi || cval == 0) continue;
            float v[8], rsd[8];
            tile8(r, v);
            const int64_t idx = static_cast<int64_t>(m) * p.ldc + c0;
            if (resp && rfast[i])
                unpack8<T>(rraw[i], rsd);
            else
                load8<T>(resp, idx, resp ? cval : 0, rsd);
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = act_f(v[e] + rsd[e], p.act);
            if (p.out_f32)
                store8<float>(static_cast<float*>(p.C), idx, v, cval);
            else
                store8<T>(static_cast<T*>(p.C), idx, v, cval);
        }
        return;
    }

    // split-K: this block's partial sums; splitk_reduce_kernel adds them up in split order
    float* part = p.partial + static_cast<int64_t>(split) * p.M * p.N;
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
        const int r = cr + i * RPP;
        const int m = m0 + r;
        if (r >= BM || m >= Mi || cval == 0) continue;
        float v[8];
        tile8(r, v);
        store8<float>(part, static_cast<int64_t>(m) * p.N + c0, v, cval);
    }
}

// ---------------------------------------------------------------------------
// Large bf16 products (see pp_tile): 256 x 256 or 128 x 128 block tiles on v_mfma_f32_32x32x16_bf16,
// eight waves in two groups that take turns on the matrix units.
//
// Waves 0-3 (one per SIMD) own the upper 128 rows of the tile, waves 4-7 the lower ones, each a
// 128 x 64 part (8 accumulator tiles, 128 registers).  A 64-wide k tile is worked in two phases,
// the upper and the lower half of the wave's rows (A0, A1) against all its columns, 16 MFMAs each.
// A phase is a memory step (fragment reads from LDS, operand loads) and an MFMA step with a barrier
// after each, and the second group runs one step behind the first: while one wave of a SIMD
// multiplies, the other reads and loads, so neither the LDS reads nor the issue of the loads (which
// hold a wave for ~50 cycles each) leave the matrix unit idle.  A step costs a few tens of
// instructions and a barrier whatever it does, so the phases are as large as the registers allow
// (four phases of 8 MFMAs, with longer load distances: 877 against 785 us on 8192 x 8192 x 8192).
//
// Each operand's stage is two 16 KB halves, two stages in LDS (128 KB).  A0 and both halves of B are
// read in the first phase and reloaded for the k tile after next in the second; A1 is read in the
// second and reloaded in the first of the next k tile: at the end of every memory step the loads
// the next one needs are a k tile old (~2300 cycles) and the eight issued since stay in flight.
//
// Products with too few 256-wide tiles to fill the CUs take 128 x 128 ones: a wave owns 64 x 32, a k tile is
// one phase of 8 MFMAs, a stage 32 KB, and four stages ring through the same 128 KB, the loads three k
// tiles ahead (a k tile takes 0.4-0.5 us; gemm_kernel's 128 x 64 tiles 0.6-1 us).
//
// A block runs up to kPPChunk tiles; the load stream goes on into the next tile during the last k
// tiles of the current one, so set-up and first-stage latency are paid once per block (but for the conv forms of 256
// x 256 tiles, which keep 1 to 17 registers in scratch: they reload them at a change of tile behind a wait for
// every load in flight).  The 32
// blocks an XCD runs at a time work on 32 consecutive tiles of its run, in groups of 8 m tiles
// that share operand rows in its L2.  The results turn through 4 KB of LDS per wave so that a store
// covers whole rows of the wave's part (128 bytes of bf16 or float32 a row; straight from the accumulators
// a row got 32 bytes a store: 8192 x 1024 -> 32000 492 -> 473 us, 8000 x 1024 -> 31001 571 -> 530).
//
// Arithmetic: acc = sum over k in 16-wide steps in ascending order from zero, then + (bias +
// bias2), + residual, activation: a function of the op alone, so tiles run across the edges of
// sub-slices (a sub-slice narrower than a tile would leave the rest of it empty: 4096 x 768 -> 2304 in
// 8 sub-slices of 288 columns took 27.1 us with two tiles each, 23.6 us so).
//
// What bounds it: with 16 of the 256 CUs busy a k tile takes 0.94 us (the MFMAs alone 0.87 us at
// 2.36 GHz); with all of them 1.5 us, the clock the chip holds under that load (8192 x 8192 x 8192: 778-800
// us, with a zero operand 629 us; independent MFMAs alone: 1950 TFLOP/s on random data, 2490 on zeros).  Measured
// against the kernels it replaced (128 x 128 tiles of gemm_kernel, and four waves of 128 x 128 with
// one stage of prefetch for the largest products): 8192 x 1024 -> 32000 580 -> 472 us, VGG-16's
// 3x3 convs over 56 x 56 x 256 at batch 16 75 -> 56 us, 8192 x 256 -> 8002 188 -> 72 us.  Not kept: four phases
// per k tile (above), waiting for the reads after the barrier instead of before it (931 against 877
// us), all eight waves in step with the next k step read under each (847 against 803 us), stores
// with the non-temporal policy (694 against 514 us), blocks started apart so that their stores
// do not meet (531 against 520 us), 4 m tiles per group (531 against 514 us).
// ---------------------------------------------------------------------------
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
constexpr int kPPChunk = 4;        // most tiles of one block
constexpr int kPPGroupM = 8;       // m tiles per group in the block order

__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_rsrc(const void* base, int bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), static_cast<short>(0), bytes, kRsrcWord3);
}
// the low (0) or high (1) bf16 of a word
__device__ __forceinline__ float bf16_of(unsigned w, int hi) { return __uint_as_float(hi ? w & 0xffff0000u : w << 16); }

// epilogues: bf16 results in whole aligned groups of eight columns, without and with a residual,
// float32 results (no residual or activation), and bf16 results of any width and alignment
enum { PP_BF16 = 0, PP_RES = 1, PP_F32 = 2, PP_ANY = 3 };
// eight bf16 at any address (the hardware takes unaligned 16-byte accesses)
__device__ __forceinline__ u32x4 load_any16(const void* q) {
    u32x4 v;
    __builtin_memcpy(&v, __builtin_assume_aligned(q, 2), 16);
    return v;
}
__device__ __forceinline__ void store_any16(void* q, u32x4 v) { __builtin_memcpy(__builtin_assume_aligned(q, 2), &v, 16); }

template <int TILE, bool CONV, int EPI, int ACT>
__global__ __launch_bounds__(512, 2) void gemm_pp_kernel(const GemmParams p) {
    using T = __bf16;
    constexpr int TM = TILE / 2, TN = TILE / 4;          // a wave's part of C
    constexpr int IA = TM / 32, NJ = TN / 32;            // its 32 x 32 tiles
    constexpr int HALVES = TILE / 128;                   // 128-row halves of an operand's stage
    constexpr unsigned HALF = 16384, STAGE = 2 * HALVES * HALF, RING = 131072;   // bytes: a stage holds A0 (A1) B0 (B1)
    constexpr unsigned STG = 4096;                       // bytes per wave to turn 32 rows of results in
    __shared__ uint4 lds[(RING + 8 * STG) / 16];
    touch_kernargs<sizeof(GemmParams)>();
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave >> 2, wn = wave & 3;
    const int lrow = lane & 31, lhalf = lane >> 5;

    // --- the block's tiles: j-th is number first + 32 j of its XCD's run -------------------------
    const int t_lo = static_cast<int>(blockIdx.x & 7) * p.g_per_xcd;
    const int t_end = min(p.g_per_xcd, p.g_total - t_lo);
    const int li = static_cast<int>(blockIdx.x >> 3);
    int t_next = (li >> 5) * 32 * p.g_chunk + (li & 31);
    const int t_last = min(t_end, ((li >> 5) + 1) * 32 * p.g_chunk);
    struct Tile { int m0, n0; };
    auto take = [&](Tile& tl) __attribute__((always_inline)) -> bool {   // the next tile of the block
        if (t_next >= t_last) return false;
        const unsigned t = static_cast<unsigned>(t_lo + t_next);
        t_next += 32;
        const unsigned group = p.g_div_group.div(t);
        const unsigned within = t - group * static_cast<unsigned>(kPPGroupM * p.g_nt);
        const bool last = static_cast<int>(group) == (p.g_mt - 1) / kPPGroupM;
        const unsigned gm = last ? static_cast<unsigned>(p.g_mt - group * kPPGroupM) : kPPGroupM;
        const unsigned nti = last ? p.g_div_last.div(within) : within / kPPGroupM;
        tl.n0 = __builtin_amdgcn_readfirstlane(static_cast<int>(nti) * TILE);
        tl.m0 = __builtin_amdgcn_readfirstlane(static_cast<int>(group * kPPGroupM + (within - nti * gm)) * TILE);
        return true;
    };
    Tile cur, ahead;
    if (!take(cur)) return;                    // block-uniform, before any barrier
    ahead = cur;
    bool live = true;                          // the load stream still has a tile

    // --- operand loads ------------------------------------------------------------------------
    // A half is 16 blocks of 1 KB (8 rows x 128 bytes); wave w loads blocks w and w + 8.  Chunk c of
    // row r sits at place c ^ (r % 8) ^ (bit 4 of r): the 32-row fragment reads are then free of bank
    // conflicts (a read serves lanes 0-3, 12-15, 20-23, 24-27 together, then 4-11, 16-19, 28-31;
    // without bit 4 two of each group's rows meet in a bank: 292 against 510 B/ns per CU).  Row r of A half i is tile row 128 (r / 64) + 64 i + r % 64, row r
    // of B half j tile column 64 (r / 32) + 32 j + r % 32: each wave's part of C is contiguous.
    const int Mi = static_cast<int>(p.M);
    const int nk = p.g_nk;                     // >= 2 (checked at launch)
    const int ktail = (p.K % 64) ? nk - 1 : nk;
    const int cl = (lane & 7) ^ (lane >> 3) ^ ((wave >> 1) & 1);
    // Offsets of this lane's loads [half][slot]; a lane or tile with nothing to load holds kOOB.
    // Dense: va, vb + 128 bytes per k tile (the scalar offset).  Conv: a k tile lies in one tap; vw is
    // the offset of the window's corner (counted from a_lead bytes before A, so never negative), vmask
    // has a bit per tap inside the image, va = vw or kOOB for the current tap, and the scalar offset is
    // that of the tap's pixel and channel.
    u32x4 va = {}, vb = {}, vw = {}, vmask = {};   // element 2 half + slot
    const unsigned a_lead = CONV ? static_cast<unsigned>((p.pad * p.img_w + p.pad) * p.cs * 2) : 0u;
    const unsigned char* const a_base = static_cast<const unsigned char*>(p.A) - a_lead;
    const unsigned a_size = p.a_bytes + a_lead;
    int ikt = 0, tap = 0, tcol = 0, tch = 0;   // k tile of the load stream; conv: its tap, tap column, first channel
    unsigned koff_a = 0, koff_b = 0;           // its scalar offsets
    unsigned lds_dst = static_cast<unsigned>(wave) * 64u;   // where this wave's loads go, in uint4 (stage 0 or 1)
    auto offsets = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int h = 0; h < HALVES; ++h)
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const int r = (wave + 8 * s) * 8 + (lane >> 3);
                const int m = min(ahead.m0 + (r >> 6) * TM + h * 64 + (r & 63), Mi - 1);
                const int n = min(ahead.n0 + (r >> 5) * TN + h * 32 + (r & 31), p.N - 1);
                if constexpr (CONV) {
                    const unsigned mu = static_cast<unsigned>(m);
                    const unsigned img = p.div_hw.div(mu);
                    const unsigned rem = mu - img * static_cast<unsigned>(p.out_h * p.out_w);
                    const unsigned ho = p.div_w.div(rem), wo = rem - ho * static_cast<unsigned>(p.out_w);
                    const int hb = static_cast<int>(ho) * p.stride - p.pad, wb = static_cast<int>(wo) * p.stride - p.pad;
                    vw[2 * h + s] = static_cast<unsigned>((static_cast<int>(img) * p.img_h + hb) * p.img_w + wb) *
                                   static_cast<unsigned>(p.cs * 2) + static_cast<unsigned>(cl * 16) + a_lead;
                    unsigned mask = 0;
                    for (int tr = 0, bit = 0; tr < p.kh; ++tr)
                        for (int tc = 0; tc < p.kw; ++tc, ++bit)
                            if (static_cast<unsigned>(hb + tr) < static_cast<unsigned>(p.img_h) &&
                                static_cast<unsigned>(wb + tc) < static_cast<unsigned>(p.img_w))
                                mask |= 1u << bit;
                    vmask[2 * h + s] = mask;
                    va[2 * h + s] = (mask & 1u) ? vw[2 * h + s] : kOOB;
                } else {
                    va[2 * h + s] = static_cast<unsigned>(m) * static_cast<unsigned>(p.lda * 2) + static_cast<unsigned>(cl * 16);
                }
                vb[2 * h + s] = static_cast<unsigned>(n) * static_cast<unsigned>(p.K * 2) + static_cast<unsigned>(cl * 16);
            }
    };
    auto load_a = [&](auto h) __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < 2; ++s)
            buffer_load_lds(a_base, a_size, (lds_ptr_t)(lds + lds_dst + h * (HALF / 16) + s * 512), va[2 * h + s], koff_a);
    };
    auto load_b = [&](auto h) __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < 2; ++s)
            buffer_load_lds(p.B, p.b_bytes, (lds_ptr_t)(lds + lds_dst + (HALVES + h) * (HALF / 16) + s * 512), vb[2 * h + s], koff_b);
    };
    // the load stream to the next k tile: of the same tile, or the first of the block's next one
    auto stream_next = [&]() __attribute__((always_inline)) {
        lds_dst = (lds_dst + STAGE / 16) & (RING / 16 - 1);
        koff_b += 128;
        koff_a += 128;
        ++ikt;
        if (ikt == nk) {
            ikt = tap = tcol = tch = 0;
            koff_a = koff_b = 0;
            live = live && take(ahead);
            if (live) {
                offsets();
            } else {
                va = vb = u32x4{kOOB, kOOB, kOOB, kOOB};
                vmask = u32x4{};
            }
        } else if constexpr (CONV) {
            tch += 64;
            if (tch == p.cs) {                 // the next tap
                tch = 0;
                ++tap;
                if (++tcol == p.kw) {
                    tcol = 0;
                    koff_a += static_cast<unsigned>((p.img_w - p.kw) * p.cs * 2);
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) va[e] = ((vmask[e] >> tap) & 1u) ? vw[e] : kOOB;
            }
        } else {
            if (ikt == ktail) {                // chunks past K
                const bool past = ikt * 64 + cl * 8 >= p.K;
#pragma unroll
                for (int e = 0; e < 4; ++e) va[e] = past ? kOOB : va[e], vb[e] = past ? kOOB : vb[e];
            }
        }
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;

    offsets();
    if constexpr (TILE == 256) {               // prologue: k tile 0, and k tile 1 but for A1
        load_b(I0{});
        load_b(I1{});
        load_a(I0{});
        load_a(I1{});
        stream_next();
        load_b(I0{});
        load_b(I1{});
        load_a(I0{});
    } else {                                   // k tiles 0, 1 and 2
#pragma unroll
        for (int u = 0; u < 3; ++u) {
            if (u) stream_next();
            load_b(I0{});
            load_a(I0{});
        }
    }

    // --- fragments ------------------------------------------------------------------------------
    // lane's 16 bytes of k step kk (16 wide): row l % 32 of a 32-row tile, chunk 2 kk + l / 32
    const unsigned lds0 = static_cast<unsigned>(reinterpret_cast<size_t>((lds_ptr_t)(&lds[0])));
    unsigned fa[4], fb[4];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
        const unsigned f = lds0 + (lrow >> 3) * 1024 + (lrow & 7) * 128 + (((2 * kk + lhalf) ^ (lrow & 7) ^ (lrow >> 4)) << 4);
        fa[kk] = f + wm * 8192;
        fb[kk] = f + wn * 4096;
    }
    u32x4 af[2][4], bf[NJ][4];
    f32x16 acc[HALVES][2][NJ];                 // [A half][row tile][B half]
    unsigned roff = 0;                         // stage the fragments come from, in bytes
    bool stored = false;                       // the block has stored a tile, with a known number of stores per wave
    // An MFMA step, after the reads and loads of its memory step: wait for the reads and for the loads
    // that the next memory step reads, the eight issued since staying in flight (in a tile's first
    // k tile the previous tile's stores lie between them)
    constexpr int STORES = IA * NJ * (EPI == PP_F32 ? 4 : 2);
    auto mfma_step = [&](auto i, auto first) __attribute__((always_inline)) {
        if (decltype(first)::value && stored)
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(8 + STORES) : "memory");
        else
            asm volatile("s_waitcnt vmcnt(8) lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
            pin(af[0][kk]), pin(af[1][kk]);
            if constexpr (i == 0) {
#pragma unroll
                for (int j = 0; j < NJ; ++j) pin(bf[j][kk]);
            }
        }
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int j = 0; j < NJ; ++j)
                    acc[i][a][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, bf[j][kk]),
                                                                           __builtin_bit_cast(bf16x8, af[a][kk]), acc[i][a][j], 0, 0, 0);
        __builtin_amdgcn_s_setprio(0);
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_barrier();
    };
    auto read_a = [&](auto h) __attribute__((always_inline)) {
        static_for<4>([&](auto kk) __attribute__((always_inline)) {
            af[0][kk] = lds_read16_at<h * HALF>(fa[kk] + roff);
            af[1][kk] = lds_read16_at<h * HALF + 4096>(fa[kk] + roff);
        });
    };
    auto read_b = [&]() __attribute__((always_inline)) {
        static_for<4>([&](auto kk) __attribute__((always_inline)) {
            static_for<NJ>([&](auto j) __attribute__((always_inline)) { bf[j][kk] = lds_read16_at<(HALVES + j) * HALF>(fb[kk] + roff); });
        });
    };
    auto ktile = [&](auto first) __attribute__((always_inline)) {
        read_b();
        read_a(I0{});
        if constexpr (TILE == 256) {
            load_a(I1{});
            stream_next();
            mfma_step(I0{}, first);
            read_a(I1{});
            load_b(I0{});
            load_b(I1{});
            load_a(I0{});
            roff ^= STAGE;
            mfma_step(I1{}, first);
        } else {
            stream_next();
            load_b(I0{});
            load_a(I0{});
            roff = (roff + STAGE) & (RING - 1);
            mfma_step(I0{}, first);
        }
    };

    asm volatile("s_waitcnt vmcnt(8)" ::: "memory");    // what the first phase of k tile 0 reads
    __builtin_amdgcn_s_barrier();
    if (wave >= 4) __builtin_amdgcn_s_barrier();        // the second group runs one step behind
    for (;;) {
#pragma unroll
        for (int i = 0; i < HALVES; ++i)
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int j = 0; j < NJ; ++j)
#pragma unroll
                    for (int e = 0; e < 16; ++e) acc[i][a][j][e] = 0.0f;
        ktile(std::true_type{});
        for (int kt = 1; kt < nk; ++kt) ktile(std::false_type{});
        // --- epilogue: rows m0 + TM wm + 32 ia + l % 32, columns n0 + TN wn + 32 j + 8 g + 4 (l / 32) .. + 3
        const int nb = cur.n0 + wn * TN;
        // Results turn through LDS, 32 rows at a time in this wave's own space, so that a store covers whole
        // rows of the wave's part: CPR 16-byte chunks a row, chunk c of row r at place c ^ (r % CPR).
        constexpr int CPR = EPI == PP_F32 ? 8 : TN * 2 / 16, SROWS = 64 / CPR;   // (float32: one column tile at a time)
        const unsigned stg = lds0 + RING + static_cast<unsigned>(wave) * STG;
        auto put = [&](int chunk, int half8, auto v) __attribute__((always_inline)) {   // lane's 8 (16) bytes of its row
            const unsigned a = stg + static_cast<unsigned>(lrow * CPR + (chunk ^ (lrow & (CPR - 1)))) * 16u + static_cast<unsigned>(half8 * 8);
            if constexpr (sizeof(v) == 8)
                asm volatile("ds_write_b64 %0, %1" ::"v"(a), "v"(v) : "memory");
            else
                asm volatile("ds_write_b128 %0, %1" ::"v"(a), "v"(v) : "memory");
        };
        const int sc = lane & (CPR - 1), sr = lane / CPR;
        auto get = [&](u32x4 (&w)[32 / SROWS]) __attribute__((always_inline)) {   // chunk sc of rows sr, sr + SROWS, ...
            static_for<32 / SROWS>([&](auto i) __attribute__((always_inline)) {
                const int r = sr + i * SROWS;
                w[i] = lds_read16(stg + static_cast<unsigned>(r * CPR + (sc ^ (r & (CPR - 1)))) * 16u);
            });
            lds_wait();
#pragma unroll
            for (int i = 0; i < 32 / SROWS; ++i) pin(w[i]);
        };
        if constexpr (EPI != PP_ANY) {
            // results and residual go through buffer resources: a row or group that is not stored gets an
            // offset past the end, so every lane issues the same stores
            const auto crs = buffer_rsrc(p.C, static_cast<int>(p.c_bytes));
            const auto rrs = buffer_rsrc(p.res, p.res ? static_cast<int>(p.c_bytes) : 0);
            // the wave's columns of bias, through the scalar cache: a vector load would be waited for
            // behind the operand loads in flight (groups past the end re-read the last one)
            u32x2 rb[NJ][4], rb2[NJ][4];
            auto group_bias = [&](const void* base, int n) __attribute__((always_inline)) -> u32x2 {
                const auto* src = (const __attribute__((address_space(4))) unsigned char*)(base ? base : kZeroChunk);
                const u32x4 q = *(const __attribute__((address_space(4))) u32x4*)(src + (base ? min(n, p.N - 8) * 2 : 0));
                return u32x2{lhalf ? q[2] : q[0], lhalf ? q[3] : q[1]};
            };
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    rb[j][g] = group_bias(p.bias, nb + j * 32 + g * 8);
                    if constexpr (EPI == PP_F32) rb2[j][g] = group_bias(p.bias2, nb + j * 32 + g * 8);
                }
            // byte offsets: row + column, either past the result when it is not stored (results span less
            // than 2^31 bytes: 0x7fffffff plus any row, and 2^31 plus any column, lie past it)
            constexpr unsigned ESZ = EPI == PP_F32 ? 4u : 2u;
            auto row_off = [&](int ia, int r) __attribute__((always_inline)) -> unsigned {
                const int m = cur.m0 + wm * TM + ia * 32 + r;
                return m < Mi ? static_cast<unsigned>(m) * static_cast<unsigned>(p.ldc * ESZ) : kOOB;
            };
            // residual: the group of eight columns a lane loads, 2 gp (lanes 0-31) or 2 gp + 1 (32-63)
            unsigned col_off[NJ][2];
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int g = 0; g < 2; ++g) {
                    const int n = nb + j * 32 + (2 * g + lhalf) * 8;
                    col_off[j][g] = n < p.N ? static_cast<unsigned>(n) * ESZ : 0x7fffffffu;
                }
            // the staged 32 rows to C: chunk sc (16 bytes from column byte col) of rows sr, sr + SROWS, ...
            auto flush_rows = [&](int ia, unsigned col) __attribute__((always_inline)) {
                u32x4 w[32 / SROWS];
                get(w);
#pragma unroll
                for (int i = 0; i < 32 / SROWS; ++i) {
                    __builtin_amdgcn_raw_buffer_store_b128(w[i], crs, static_cast<int>(row_off(ia, sr + i * SROWS) + col), 0, 0);
                }
            };
            auto chunk_off = [&](int n) __attribute__((always_inline)) -> unsigned {
                return n < p.N ? static_cast<unsigned>(n) * ESZ : 0x7fffffffu;
            };
            u32x4 rr[NJ][2];
            auto load_res = [&](unsigned row) __attribute__((always_inline)) {
#pragma unroll
                for (int j = 0; j < NJ; ++j)
#pragma unroll
                    for (int gp = 0; gp < 2; ++gp)
                        rr[j][gp] = __builtin_amdgcn_raw_buffer_load_b128(rrs, static_cast<int>(row + col_off[j][gp]), 0, 0);
            };
            auto store_bf16 = [&]() __attribute__((always_inline)) {
                static_for<IA>([&](auto ia) __attribute__((always_inline)) {
                    if constexpr (EPI == PP_RES) load_res(row_off(ia, lrow));
#pragma unroll
                    for (int j = 0; j < NJ; ++j)
#pragma unroll
                        for (int gp = 0; gp < 2; ++gp) {
                            float rs[2][4] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
                            if constexpr (EPI == PP_RES) {
                                const u32x4 q = rr[j][gp];
                                const u32x2 s0 = __builtin_amdgcn_permlane32_swap(q[0], q[2], false, false);
                                const u32x2 s1 = __builtin_amdgcn_permlane32_swap(q[1], q[3], false, false);
#pragma unroll
                                for (int h = 0; h < 2; ++h)
                                    rs[h][0] = bf16_of(s0[h], 0), rs[h][1] = bf16_of(s0[h], 1), rs[h][2] = bf16_of(s1[h], 0),
                                    rs[h][3] = bf16_of(s1[h], 1);
                            }
                            u32x2 pk[2];
#pragma unroll
                            for (int h = 0; h < 2; ++h) {
                                const int g = 2 * gp + h;
                                float v[4];
#pragma unroll
                                for (int e = 0; e < 4; ++e) {
                                    v[e] = acc[ia / 2][ia % 2][j][4 * g + e] + bf16_of(rb[j][g][e / 2], e & 1);
                                    if constexpr (EPI == PP_RES) v[e] += rs[h][e];
                                    v[e] = act_f(v[e], ACT);
                                }
                                pk[h] = __builtin_bit_cast(u32x2, bf16x4{(__bf16)v[0], (__bf16)v[1], (__bf16)v[2], (__bf16)v[3]});
                            }
                            put(4 * j + 2 * gp, lhalf, pk[0]);
                            put(4 * j + 2 * gp + 1, lhalf, pk[1]);
                        }
                    lds_wait();
                    flush_rows(ia, chunk_off(nb + sc * 8));
                    __builtin_amdgcn_sched_barrier(0);
                });
            };
            if constexpr (EPI == PP_F32) {
                static_for<IA>([&](auto ia) __attribute__((always_inline)) {
#pragma unroll
                    for (int j = 0; j < NJ; ++j) {
#pragma unroll
                        for (int g = 0; g < 4; ++g) {
                            u32x4 v;
#pragma unroll
                            for (int e = 0; e < 4; ++e) v[e] = __float_as_uint(acc[ia / 2][ia % 2][j][4 * g + e] +
                                                       (bf16_of(rb[j][g][e / 2], e & 1) + bf16_of(rb2[j][g][e / 2], e & 1)));
                            put(2 * g + lhalf, 0, v);
                        }
                        lds_wait();
                        flush_rows(ia, chunk_off(nb + j * 32 + sc * 4));
                    }
                    __builtin_amdgcn_sched_barrier(0);
                });
            } else {
                store_bf16();
            }
        } else {
            // Whole groups of eight columns move as unaligned 16-byte accesses, the last, partial one
            // element by element (only the last column tile has it).
            const T* const biasp = static_cast<const T*>(p.bias);
            const T* const resp = static_cast<const T*>(p.res);
            T* const C = static_cast<T*>(p.C);
            const bool tail = cur.n0 + TILE > p.N;
            u32x2 rb[NJ][4];
            const auto brs = buffer_rsrc(biasp, biasp ? p.N * 2 : 0);
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int o = (nb + j * 32 + g * 8 + lhalf * 4) * 2;
                    if (tail) {
                        unsigned h[4];
#pragma unroll
                        for (int e = 0; e < 4; ++e) h[e] = static_cast<unsigned short>(__builtin_amdgcn_raw_buffer_load_b16(brs, o + 2 * e, 0, 0));
                        rb[j][g] = u32x2{h[0] | (h[1] << 16), h[2] | (h[3] << 16)};
                    } else {
                        rb[j][g] = u32x2{0u, 0u};
                        if (biasp) rb[j][g] = *(const __attribute__((address_space(1))) u32x2*)(reinterpret_cast<const char*>(biasp) + o);
                    }
                }
            static_for<IA>([&](auto ia) __attribute__((always_inline)) {
                const int m = cur.m0 + wm * TM + ia * 32 + lrow;
                const int64_t row = static_cast<int64_t>(min(m, Mi - 1)) * p.ldc;
#pragma unroll
                for (int j = 0; j < NJ; ++j)
#pragma unroll
                    for (int gp = 0; gp < 2; ++gp) {
                        const int n = nb + j * 32 + (2 * gp + lhalf) * 8;
                        const int nv = m < Mi ? p.N - n : 0;           // 8 or more: a whole group
                        u32x4 q = {};
                        if (resp) {
                            if (nv >= 8) {
                                q = load_any16(resp + row + n);
                            } else if (nv > 0) {
                                unsigned h[8];
#pragma unroll
                                for (int e = 0; e < 8; ++e) h[e] = e < nv ? __builtin_bit_cast(unsigned short, resp[row + n + e]) : 0u;
                                q = u32x4{h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16)};
                            }
                        }
                        const u32x2 r0 = __builtin_amdgcn_permlane32_swap(q[0], q[2], false, false);
                        const u32x2 r1 = __builtin_amdgcn_permlane32_swap(q[1], q[3], false, false);
                        u32x2 pk[2];
#pragma unroll
                        for (int h = 0; h < 2; ++h) {
                            const int g = 2 * gp + h;
                            float v[4];
#pragma unroll
                            for (int e = 0; e < 4; ++e)
                                v[e] = act_f((acc[ia / 2][ia % 2][j][4 * g + e] + bf16_of(rb[j][g][e / 2], e & 1)) +
                                                 bf16_of(e < 2 ? r0[h] : r1[h], e & 1), ACT);
                            pk[h] = __builtin_bit_cast(u32x2, bf16x4{(__bf16)v[0], (__bf16)v[1], (__bf16)v[2], (__bf16)v[3]});
                        }
                        put(4 * j + 2 * gp, lhalf, pk[0]);
                        put(4 * j + 2 * gp + 1, lhalf, pk[1]);
                    }
                lds_wait();
                u32x4 w[32 / SROWS];
                get(w);
#pragma unroll
                for (int i = 0; i < 32 / SROWS; ++i) {
                    const int ms = cur.m0 + wm * TM + ia * 32 + sr + i * SROWS, n = nb + sc * 8;
                    const int nv = ms < Mi ? p.N - n : 0;              // 8 or more: a whole group
                    T* const dst = C + static_cast<int64_t>(min(ms, Mi - 1)) * p.ldc + n;
                    if (nv >= 8) {
                        store_any16(dst, w[i]);
                    } else if (nv > 0) {
#pragma unroll
                        for (int e = 0; e < 7; ++e)
                            if (e < nv) reinterpret_cast<unsigned short*>(dst)[e] = static_cast<unsigned short>(w[i][e / 2] >> (16 * (e & 1)));
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            });
        }
        stored = EPI != PP_ANY;   // (there the number of stores issued depends on the lanes: counted as none)
        // the load stream has at least begun the next tile (it runs two k tiles ahead, or three)
        if (!live) break;
        cur = ahead;
    }
    if (wave < 4) __builtin_amdgcn_s_barrier();         // the second group's last step
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");    // no load into LDS outlives the block
}

// Split-K finish: sum the partials in split order, then the usual epilogue.
template <typename T>
__global__ void splitk_reduce_kernel(const GemmParams p) {
    touch_kernargs<sizeof(GemmParams)>();
    // one thread per 4 columns of a row; M * ceil(N / 4) < 2^31 (checked at launch)
    const unsigned groups = static_cast<unsigned>(p.N + 3) / 4;
    const unsigned t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= static_cast<unsigned>(p.M) * groups) return;
    const unsigned mu = p.r_div_groups.div(t);
    const int64_t m = mu;
    const int n = static_cast<int>(t - mu * groups) * 4;
    const int nvalid = min(4, p.N - n);
    // bias, second bias and residual go out first, so their latency overlaps the partials'
    float bias[4] = {0.f, 0.f, 0.f, 0.f}, bias2[4] = {0.f, 0.f, 0.f, 0.f}, rsd[4] = {0.f, 0.f, 0.f, 0.f};
    if (p.bias) ld4(static_cast<const T*>(p.bias), n, nvalid, bias);
    if (p.bias2) ld4(static_cast<const T*>(p.bias2), n, nvalid, bias2);
    if (p.res) ld4(static_cast<const T*>(p.res), m * p.ldc + n, nvalid, rsd);
    float v[4] = {0.f, 0.f, 0.f, 0.f};
    const int64_t plane = p.M * static_cast<int64_t>(p.N);
    const float* src = p.partial + m * p.N + n;
    if (nvalid == 4 && (p.N & 3) == 0) {
        f32x4 part[16];                       // splits <= 16: all loads in flight together
#pragma unroll
        for (int s = 0; s < 16; ++s)
            if (s < p.splits) part[s] = *reinterpret_cast<const f32x4*>(src + s * plane);
#pragma unroll
        for (int s = 0; s < 16; ++s)
            if (s < p.splits)
                for (int e = 0; e < 4; ++e) v[e] += part[s][e];
    } else {
        for (int s = 0; s < p.splits; ++s)
            for (int e = 0; e < nvalid; ++e) v[e] += src[s * plane + e];
    }
    for (int q = 0; q < 4; ++q) v[q] = act_f((v[q] + (bias[q] + bias2[q])) + rsd[q], p.act);
    const int64_t idx = m * p.ldc + n;
    if (p.out_f32)
        store4<float>(static_cast<float*>(p.C), idx, v, nvalid);
    else
        store4<T>(static_cast<T*>(p.C), idx, v, nvalid);
}

// ---------------------------------------------------------------------------
// 3x3 convolutions (stride 1, padding 1) over bf16 images of 64 to 512 channels
// (multiples of 64) and at most 56 x 56 pixels, patch-staged.  The implicit
// GEMM above fetches every input pixel once per tap (nine times); here a block
// owns a TH x 8 tile of output pixels of one image (8 x 8 in use) and BN output
// channels of one sub-slice, and for each 64-channel chunk it stages the
// (TH + 2) x 10 input patch around its tile (one pixel of halo each way, zeros
// outside the image) once, with the nine taps' weight rows, then forms all nine
// taps' A fragments from that patch in LDS (about a sixth of the A bytes; the
// win is largest on narrow sub-slices, whose A traffic dominates).  Images of
// more than two chunks take two chunk buffers, the next chunk's loads going out
// before the current chunk's products (64 KB of LDS per block; with fewer chunks
// one buffer, which leaves room for more resident blocks: measured faster on
// ResNet-50's stages 1 and 2, 7.7-8.9 us against 10.8-14.1 us).  Loads use the same whole-line, XOR-swizzled layout as
// above (patch pixels and weight rows in place of tile rows).  The k order is
// chunk, then tap, then the two 32-wide steps; it depends only on the op, not
// on BN, TH or the sub-slice, so sub-sliced and unsplit launches agree bit for
// bit.  TH / 2 waves each take two tile rows (16 pixels) by BN columns; the
// accumulators start at the bias and the epilogue stores from the MFMA layout
// (residual, activation).
// ---------------------------------------------------------------------------
constexpr int HTW = 8;                       // output tile width; its height TH is a parameter

bool conv_halo_ok(int dtype, int kh, int kw, int stride, int pad, int cs, int n_out, int out_h, int out_w, int64_t m) {
    // Small convs only: at most 2^31 multiply-adds (M x N x K; each of ResNet-50's stride-1 3x3
    // convs at batch 8 is 0.92 G).  On those the implicit GEMM's large tiles leave CUs idle or need split-K and
    // a second launch.  On larger ones the patch, re-read for every 16 output channels, and the small tiles lose to it;
    // and over images above 56 x 56.  Measured in four sub-slices (us, here / the implicit GEMM's best tiles), both
    // sides of the line: 128 channels over 28 x 28, batch 8 7.6 / 10.4, 16 (1.8 G) 12.0 / 12.8, 24 (2.8 G) 16.5 / 13.9; 256 over
    // 14 x 14, batch 8 8.3 / 13.2, 16 15.3 / 17.2, 24 22.1 / 19.0, 32 28.2 / 19.2; 512 over 7 x 7, batch 8 12.4 / 14.2, 16 13.6 / 17.0, 24
    // 23.3 / 23.2, 32 26.0 / 24.4, 64 50.7 / 33.5.  64 channels over 56 x 56 are ahead past it too (batch 8 8.2 / 10.2, 32 22.2 / 33.4), and the
    // GEMM is ahead before it where 8 x 8 tiles fit badly (10 x 10 of 256 channels, batch 16 14.9 / 13.3) or blocks are
    // few (512 over 14 x 14, batch 1 11.3 / 10.8).
    if (!(dtype == MOPAR_BF16 && kh == 3 && kw == 3 && stride == 1 && pad == 1 && cs % 64 == 0 && cs <= 512 &&
          n_out >= 1 && n_out <= 512 && out_h >= 7 && out_w >= 7 && int64_t(out_h) * out_w <= 56 * 56 && m >= 0 &&
          m < (int64_t(1) << 31)))
        return false;
    // (the checks above bound the product below 2^53)
    return m * n_out * (int64_t(kh) * kw * cs) <= (int64_t(1) << 31);
}

template <int BN, int TH, int NBUF>
__global__ __launch_bounds__(TH * HTW / 16 * 64) void conv3_halo_kernel(const GemmParams p) {
    using T = __bf16;
    constexpr int NW = TH * HTW / 16;           // waves: 16 tile pixels (two tile rows) each
    constexpr int PW = HTW + 2, PIX = (TH + 2) * PW;   // patch width, pixels
    constexpr int HPBLK = (PIX + 7) / 8;        // patch load blocks of 8 pixels
    constexpr int FN = BN / 16;
    constexpr int BPT = BN / 8;                 // weight load blocks per tap
    constexpr int NBB = 9 * BPT;                // weight load blocks per chunk
    constexpr int LP = (HPBLK + NW - 1) / NW, LB = (NBB + NW - 1) / NW;   // load slots per wave
    // NBUF chunk buffers: patch blocks, weight blocks and, with two buffers, one block for the
    // load slots past the last block (a wave whose share ends early still issues LP + LB loads,
    // of zeros, there, so that every wave's wait count is the same)
    static_assert(NBUF == 1 || NBUF == 2, "chunk buffers");
    constexpr int CHB = HPBLK + NBB + (NBUF == 2 ? 1 : 0);
    __shared__ uint4 lds[NBUF * CHB * 64];
    touch_kernargs<sizeof(GemmParams)>();
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

    // block -> (image, spatial tile, sub-slice, n tile); the blocks that share a patch are
    // consecutive, and each XCD runs a contiguous range of them
    const unsigned t = (blockIdx.x % 8) * static_cast<unsigned>(p.g_per_xcd) + blockIdx.x / 8;
    if (t >= static_cast<unsigned>(p.g_total)) return;
    const unsigned tile = p.g_div_group.div(t);
    const unsigned col = t - tile * static_cast<unsigned>(p.g_cols);
    const unsigned j = p.g_div_nt.div(col);
    const int nti = static_cast<int>(col - j * static_cast<unsigned>(p.g_nt));
    const unsigned img = p.h_div_tiles.div(tile);
    const unsigned tin = tile - img * static_cast<unsigned>(p.h_tiles);
    const unsigned tyi = p.h_div_tx.div(tin);
    const int oh0 = static_cast<int>(tyi) * TH, ow0 = static_cast<int>(tin - tyi * static_cast<unsigned>(p.h_tx)) * HTW;
    const int jj = static_cast<int>(j);
    const int n_lo = jj * p.g_q + min(jj, p.g_rr), n_hi = (jj + 1) * p.g_q + min(jj + 1, p.g_rr);
    const int n0 = n_lo + nti * BN;
    if (n0 >= n_hi) return;                     // block-uniform, before any barrier

    // loads of chunk q: patch block b covers pixels 8b .. 8b + 7 (pixel pp at patch row pp / 10,
    // column pp % 10), weight block b covers rows 8 (b % BPT) .. +7 of tap b / BPT; lane l takes
    // entity 8b + l / 8, chunk cl = (l % 8) ^ (l / 8); a chunk's byte offset adds 128 q
    const int cl = (lane & 7) ^ (lane >> 3);
    const unsigned pix_bytes = static_cast<unsigned>(p.cs) * 2u;
    unsigned voffP[LP], voffB[LB];
#pragma unroll
    for (int i = 0; i < LP; ++i) {
        const int pp = 8 * min(wave + NW * i, HPBLK - 1) + (lane >> 3);
        const int ih = oh0 - 1 + pp / PW, iw = ow0 - 1 + pp % PW;
        const bool in = pp < PIX && static_cast<unsigned>(ih) < static_cast<unsigned>(p.img_h) &&
                        static_cast<unsigned>(iw) < static_cast<unsigned>(p.img_w);
        voffP[i] = in ? (static_cast<unsigned>((static_cast<int>(img) * p.img_h + ih) * p.img_w + iw)) * pix_bytes +
                            static_cast<unsigned>(cl * 16)
                      : kOOB;
    }
#pragma unroll
    for (int i = 0; i < LB; ++i) {
        const int b = min(wave + NW * i, NBB - 1);
        const int tap = b / BPT, n = min(n0 + (b % BPT) * 8 + (lane >> 3), n_hi - 1);
        voffB[i] = static_cast<unsigned>(n) * static_cast<unsigned>(p.K * 2) + static_cast<unsigned>(tap) * pix_bytes +
                   static_cast<unsigned>(cl * 16);
    }

    // epilogue set-up (MFMA layout): this lane's tile pixel and four columns per n fragment
    const int pix = wave * 16 + (lane & 15);
    const int oh = oh0 + (pix >> 3), ow = ow0 + (pix & 7);
    const bool row_ok = oh < p.out_h && ow < p.out_w;
    const int64_t row = (static_cast<int64_t>(img) * p.out_h + oh) * p.out_w + ow;
    int ncol[FN], nval[FN];
    f32x4 acc[FN];
#pragma unroll
    for (int b = 0; b < FN; ++b) {
        ncol[b] = n0 + b * 16 + (lane >> 4) * 4;
        nval[b] = max(0, min(4, n_hi - ncol[b]));
        float bv[4], b2v[4];
        ld4_or_zero<T>(static_cast<const T*>(p.bias), ncol[b], nval[b], bv);
        ld4_or_zero<T>(static_cast<const T*>(p.bias2), ncol[b], nval[b], b2v);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[b][e] = bv[e] + b2v[e];
    }

    const int nq = p.cs / 64;
    // chunk qc's loads into buffer buf (LP + LB per wave, always)
    auto issue = [&](int qc, int buf) __attribute__((always_inline)) {
        const unsigned soff = static_cast<unsigned>(qc) * 128u;
        uint4* const base = &lds[buf * CHB * 64];
#pragma unroll
        for (int i = 0; i < LP; ++i) {
            const int b = wave + NW * i;        // wave-uniform
            const bool dead = HPBLK % NW != 0 && b >= HPBLK;
            if (NBUF == 1 && dead) break;
            buffer_load_lds(p.A, p.a_bytes, (lds_ptr_t)(base + (dead ? CHB - 1 : b) * 64), dead ? kOOB : voffP[i], soff);
        }
#pragma unroll
        for (int i = 0; i < LB; ++i) {
            const int b = wave + NW * i;
            const bool dead = NBB % NW != 0 && b >= NBB;
            if (NBUF == 1 && dead) break;
            buffer_load_lds(p.B, p.b_bytes, (lds_ptr_t)(base + (dead ? CHB - 1 : HPBLK + b) * 64), dead ? kOOB : voffB[i],
                            soff);
        }
    };
    static_assert(LP + LB <= 63, "the wait below counts the next chunk's loads");
    if constexpr (NBUF == 2) issue(0, 0);
    for (int qc = 0; qc < nq; ++qc) {
        if constexpr (NBUF == 2) {
            // the next chunk goes out before this one is waited for; its loads are the last issued
            if (qc + 1 < nq) {
                issue(qc + 1, (qc + 1) & 1);
                asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LP + LB) : "memory");
            } else {
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            }
        } else {
            if (qc > 0) __syncthreads();        // the previous chunk's fragments have been read
            issue(qc, 0);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        }
        __builtin_amdgcn_s_barrier();           // every wave's share of chunk qc has landed
        const unsigned lds0 =
            static_cast<unsigned>(reinterpret_cast<size_t>((lds_ptr_t)(&lds[(NBUF == 2 ? qc & 1 : 0) * CHB * 64])));
#pragma unroll
        for (int tap = 0; tap < 9; ++tap) {
            const int pp = ((pix >> 3) + tap / 3) * PW + (pix & 7) + tap % 3;
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                const int ch = 4 * ks + (lane >> 4);
                u32x4 af = lds_read16(lds0 + static_cast<unsigned>(pp * 128 + ((ch ^ (pp & 7)) << 4)));
                u32x4 bf[FN];
#pragma unroll
                for (int b = 0; b < FN; ++b) {
                    const int nb = b * 16 + (lane & 15);
                    bf[b] = lds_read16(lds0 + static_cast<unsigned>((HPBLK * 64 + (tap * BN + nb) * 8 + (ch ^ (nb & 7))) * 16));
                }
                lds_wait();
                pin(af);
#pragma unroll
                for (int b = 0; b < FN; ++b) {
                    pin(bf[b]);
                    acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, bf[b]),
                                                                   __builtin_bit_cast(bf16x8, af), acc[b], 0, 0, 0);
                }
            }
        }
        if constexpr (NBUF == 2) __syncthreads();   // chunk qc's buffer is read before chunk qc + 2 reuses it
    }

    if (!row_ok) return;
    const T* resp = static_cast<const T*>(p.res);
#pragma unroll
    for (int b = 0; b < FN; ++b) {
        if (nval[b] == 0) continue;
        const int64_t idx = row * p.ldc + ncol[b];
        float v[4], rv[4] = {0.f, 0.f, 0.f, 0.f};
        if (resp) ld4<T>(resp, idx, nval[b], rv);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = act_f(acc[b][e] + rv[e], p.act);
        if (p.out_f32)
            store4<float>(static_cast<float*>(p.C), idx, v, nval[b]);
        else
            store4<T>(static_cast<T*>(p.C), idx, v, nval[b]);
    }
}

template <int BN, int TH, int NBUF>
static hipError_t launch_halo(const GemmParams& params, int width, hipStream_t st) {
    GemmParams p = params;
    const int64_t nt = (width + BN - 1) / BN;
    const int ty = (p.out_h + TH - 1) / TH, tx = (p.out_w + HTW - 1) / HTW;
    const int64_t imgs = p.M / (static_cast<int64_t>(p.out_h) * p.out_w);
    const int64_t total = imgs * ty * tx * p.ksub * nt;
    if (total >= (int64_t(1) << 31) / 8 || static_cast<int64_t>(ty) * tx * p.ksub * nt >= (int64_t(1) << 31))
        return hipErrorInvalidValue;
    p.g_total = static_cast<int>(total);
    p.g_per_xcd = static_cast<int>((total + 7) / 8);
    p.g_nt = static_cast<int>(nt);
    p.g_cols = static_cast<int>(nt * p.ksub);
    p.g_q = p.N / p.ksub;
    p.g_rr = p.N % p.ksub;
    p.g_div_group = FastDiv(static_cast<unsigned>(p.g_cols));
    p.g_div_nt = FastDiv(static_cast<unsigned>(nt));
    p.h_tiles = ty * tx;
    p.h_tx = tx;
    p.h_div_tiles = FastDiv(static_cast<unsigned>(ty * tx));
    p.h_div_tx = FastDiv(static_cast<unsigned>(tx));
    const int64_t grid = (total + 7) / 8 * 8;
    launch_kernel(conv3_halo_kernel<BN, TH, NBUF>, dim3(static_cast<unsigned>(grid)), dim3(TH * HTW / 16 * 64), 0, st,
                  p);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Tile selection.  Tiles of gemm_kernel with the same number of waves along K share the K
// loop and give the same bits, so a choice among them may follow the sub-slice width.
// What changes bits (pp_tile, conv_halo_ok, gemm_splits, and K shared out over the waves: up to 64 rows,
// and f32_small_tiles) depends on the op alone.
// ---------------------------------------------------------------------------

constexpr int kCUs = 256;

// Whether a float32 product runs on 32 x 16 tiles with K split over the waves: at most 16 64 x 64 tiles (a batch-1
// CNN's later convs and its classifier), whose serial K loop counts as much as a block's MFMA time (64 x 768 -> 768 11.5 us on
// 64 x 64 tiles with four splits, 6.7 here).  Up to 16 rows and over 2048 of k the 16 x 64 tiles with more splits
// are faster from 9 tiles on (16 x 4096 -> 1024 8.4 there, 9.2 here; -> 512 8.2 there, 7.8 here).  Over 64 rows, up to 16
// columns and 128 of k, four stages, there is too little K to share out: 64 x 16 tiles (3x3 convs over 32 x 32 x 4 -> 16
// 3.8 there, 4.2 here; 1024 x 100 -> 10 4.3, 4.6; past it the sums shared out are the more exact ones, 1.2e-7 against
// 2.0e-7 of the result at 144 of k, and as fast: 1024 x 144 -> 16 4.4, 4.5).
bool f32_small_tiles(int64_t M, int N, int K) {
    const int64_t tiles = ((M + 63) / 64) * ((N + 63) / 64);
    return tiles <= 16 && !(M <= 16 && K > 2048 && tiles > 8) && !(M > 64 && N <= 16 && K <= 128);
}

int gemm_splits(int64_t M, int N, int K, int dtype, int epi) {
    if (epi != EPI_STD || M * ((N + 3) / 4) >= (int64_t(1) << 31)) return 1;
    const int bk = dtype == MOPAR_BF16 ? 64 : 32;
    const int64_t nk = (K + bk - 1) / bk;
    const int64_t tiles = ((M + 63) / 64) * ((N + 63) / 64);   // reference tiling, independent of k
    // the reduce pass costs about as much as a dozen k stages: split only long K loops
    if (nk < 24) return 1;
    int s = 1;
    auto split = [&](int most, auto fits) {
        while (s < most && nk / (2 * s) >= 4 && fits(2 * s)) s *= 2;
        return s;
    };
    if (dtype == MOPAR_BF16) return split(16, [&](int64_t sp) { return tiles * sp < 2 * kCUs; });
    // float32 is MFMA-bound: splits pay while they put idle CUs to work (us by number of splits, 1 / 2 / 4 / 8).
    if (f32_small_tiles(M, N, K)) {
        // 32 x 16 tiles, three rounds of blocks: 1 x 1024 -> 256 7.6 / 7.1 / 6.1 / 5.7, 100 x 4608 -> 512 (128 blocks) 23.6 /
        // 15.5 / 13.3 / 14.9, 77 (96 blocks) 23.6 / 15.4 / 13.2 / 11.9; one split under 1024 of k (64 x 768 -> 768 6.7 / 7.2 / 7.5),
        // and up to there where the reduce pass has no whole groups of four columns (1024 x 1024 -> 10 8.5 / 8.8 / 9.0 / 10.8)
        const int64_t blocks = ((M + 31) / 32) * ((N + 15) / 16);
        if (nk < 32 || (N % 4 != 0 && nk == 32)) return 1;
        return split(16, [&](int64_t sp) { return blocks * sp <= 3 * kCUs; });
    }
    // 16 x 64 tiles, one round: 16 x 1024 -> 4096 11.3 / 9.5 / 8.1 / 11.0, 1 x 1024 -> 1088 11.2 / 9.2 / 7.5 / 7.0
    if (M <= 16) return split(16, [&](int64_t sp) { return tiles * sp <= kCUs; });
    if (M <= 64) {
        // tiles of 32 x 16 up to 192 blocks of 64 x 64, which up to 1024 of k need no splits (64 x 768 -> 2304 8.5 / 9.7 /
        // 13.1, 64 x 1024 -> 1088 7.8 / 9.0 / 8.4); past it half a round of the larger ones (64 x 2048 -> 1088 12.3 / 12.2 / 10.7 /
        // 13.2, 64 x 3072 -> 2304 23.9 / 20.1 / 23.5, 64 x 3072 -> 6144 33.9 / 39.9), and four splits where they
        // are one round (33 x 4096 -> 4096 31.2 / 33.6 / 28.7)
        if (nk <= 32) return 1;
        if (M > 32 && nk > 64 && tiles > 48 && tiles <= 64) return 4;
        return split(16, [&](int64_t sp) { return tiles * sp < kCUs / 2; });
    }
    // 64 x 64 tiles, one round: 77 x 768 -> 768 (24 tiles) 18.7 / 13.0 / 9.7, 308 x 768 -> 768 (60) 18.9 / 13.9 / 11.6 / 13.4,
    // 77 x 768 -> 2304 (72) 18.9 / 13.7 / 14.1, 512 x 1024 -> 1024 (128) 24.1 / 19.1 / 20.7, 308 x 768 -> 2304 (180) 19.3 / 22.5.
    // From 1536 of k on also into a second round: 768 x 2048 -> 768 (144) 44.4 / 42.4 / 44.7, 512 x 3072 -> 768 (96) 64.4 / 37.4 /
    // 35.2; at 1536 the same (34.3 / 34.3 / 36.6).  More than eight are slower (77 x 3072 -> 768 14.0, with sixteen 14.8)
    return split(8, [&](int64_t sp) { return tiles * sp <= (nk > 48 ? 2 * kCUs - 1 : kCUs); });
}

template <typename T, int BM, int BN, int WM, int WN, int NS, int KH = 1, int KS = 1>
static hipError_t launch_cfg(const GemmParams& params, int width, hipStream_t st) {
    GemmParams p = params;
    const int64_t mt = (p.M + BM - 1) / BM, nt = (width + BN - 1) / BN;
    const int64_t total = mt * nt * p.ksub * p.splits;
    if (total >= (int64_t(1) << 31) / kGroupM) return hipErrorInvalidValue;
    p.g_mt = static_cast<int>(mt);
    p.g_nt = static_cast<int>(nt);
    p.g_total = static_cast<int>(total);
    p.g_per_xcd = static_cast<int>((total + 7) / 8);
    p.g_cols = static_cast<int>(nt * p.ksub * p.splits);
    p.g_nk = (p.K + 8 * Elt<T>::EPC - 1) / (8 * Elt<T>::EPC);
    p.g_q = p.N / p.ksub;
    p.g_rr = p.N % p.ksub;
    p.g_div_group = FastDiv(static_cast<unsigned>(kGroupM * p.g_cols));
    const int last = static_cast<int>(mt - (mt - 1) / kGroupM * kGroupM);   // m tiles in the last group
    p.g_div_last = FastDiv(static_cast<unsigned>(last));
    p.g_div_nt = FastDiv(static_cast<unsigned>(nt));
    p.g_div_ksub = FastDiv(static_cast<unsigned>(p.ksub));
    p.g_div_splits = FastDiv(static_cast<unsigned>(p.splits));
    if (p.conv) {
        const int bk = 8 * Elt<T>::EPC, dq = bk / p.cs;
        p.dc = bk - dq * p.cs;
        p.dqr = dq / p.kw;
        p.dqc = dq - p.dqr * p.kw;
        p.div_cs = FastDiv(static_cast<unsigned>(p.cs));
        p.div_kw = FastDiv(static_cast<unsigned>(p.kw));
    }
    const int64_t grid = (total + 7) / 8 * 8;
    const dim3 block(WM * WN * KS * 64);
    if (p.conv)
        launch_kernel((gemm_kernel<T, BM, BN, WM, WN, NS, KH, KS, true>), dim3(static_cast<unsigned>(grid)), block, 0,
                      st, p);
    else
        launch_kernel((gemm_kernel<T, BM, BN, WM, WN, NS, KH, KS, false>), dim3(static_cast<unsigned>(grid)), block, 0,
                      st, p);
    return hipGetLastError();
}

// The tile of gemm_pp_kernel for an (M, N, K) product (0: gemm_kernel's tiles are faster): a function of the
// product alone, never of the sub-slice count, so that all sub-slice launches of an operator run the same arithmetic
// (a tile may hold columns of several sub-slices).  A block fills a CU, so the lines lie at the share of the
// CUs that the last round of tiles leaves idle.  Measured against gemm_kernel's tiles (us, here / there).
// 256: 4096 x 768 -> 2304, 144 tiles, 23.6 / 30.9; -> 3072, 192 tiles, 25.0 / 30.3; 3x3 convs over 56 x 56 x 256,
// 147 tiles, 56 / 68.5, 98 tiles, 52.5 / 43.9; 8192 x 1024 -> 1024, 128 tiles, 26.6 / 24.1; in two rounds 600 x
// 1024 -> 25047, 294 tiles, 63.4 / 55.9, 5612 x 512 -> 3526, 308 tiles, 0.85 of there, convs of 311 to 320 tiles
// 0.86 (1x1, K 512) to 1.06 (3x3, K 576) of there, of 328 tiles 0.88, 8192 x 768 -> 3072, 384 tiles, 45.6 / 54.5;
// 8229 x 312 -> 8000, 1056 tiles, 73 / 94.
// Rows past M count too: gemm_kernel holds two 128 x 128 tiles a CU, so a product whose 128 x 128 tiles take
// no more rounds of 512 than its 256 x 256 tiles take of 256 stays there: 384 x 1024 -> 18000, 423 of 512, 25.5 / 22.7,
// 96 x 1024 -> 48000, 375, 27.4 / 21.5, 288 x 1024 -> 40000 in two rounds, 939 of 1024, 46.8 / 41.3; and
// 320 x 1024 -> 22000, 516, 0.82 of there, 256 x 1024 -> 40000, 626, 26.9 / 35.4.
// 128, one round: the conv over 56 x 56 x 256, 196 tiles, 28.9 / 34.9, over 28 x 28 x 512, 196
// tiles, 45.8 / 56.6, over 112 x 112 x 128, 196 tiles, 20.3 / 23.5; 2048 x 1024 -> 1024, 128 tiles, 12.3 / 11.7; few
// rows too, whose time is the weights': 1 x 256 -> 18000 6.2 / 8.2, 1 x 1024 -> 32000 14.0 / 15.6, 17 x 1024 -> 18000
// 12.4 / 16.2, 64 x 1024 -> 32000 15.4 / 20.6, 128 x 1024 -> 18000 13.0 / 14.7.  gemm_kernel's 128 x 64 tiles in one
// round are faster still (6314 x 4096 -> 278, 250 of them, 35.5 / 31.9; 6588 x 768 -> 267, 260, 0.79 of there).
// 128 in more rounds: 17 to 64 rows, whose other tiles split K (64 x 1024 -> 40000 23.3 / 28.2, 17 x 512 -> 48000
// 15.3 / 18.6); else only short K, 75 % of the rounds: 8192 x 256 -> 1024 12.3 / 14.2, 257 x 256 -> 18000, 423 tiles, 10.8 /
// 11.8, 16 x 512 -> 56000 15.7 / 20.1, 7209 x 512 -> 798, 399, 0.85 of there (65 x 512 -> 56000 16.0 / 15.3, 8192 x 1024 -> 1024
// 25.0 / 24.1, the conv over 56 x 56 x 256, 392 tiles, 50 / 44, 1 x 1024 -> 40000 22.8 / 20.2); past 256 of k 90 % where
// gemm_kernel's tiles are 128 wide: 8192 x 512 -> 1024, 512 tiles, 16.2 / 17.3, 256 x 512 -> 32000, 500, 0.99 of there, 129 x
// 512 -> 28000, 438, 1.02, -> 25000, 392, 1.04.
int pp_tile_size(int64_t M, int N, int K) {
    if (K < 256) return 0;
    const int64_t tiles = ((M + 255) / 256) * ((N + 255) / 256), rounds = (tiles + kCUs - 1) / kCUs;
    const int64_t small = ((M + 127) / 128) * ((N + 127) / 128), srounds = (small + kCUs - 1) / kCUs;
    if (N >= 192 && small > 2 * kCUs * rounds &&
        (rounds == 1 ? tiles >= 140 : tiles * 10 >= rounds * kCUs * 6))
        return 256;
    if (N < 96 || ((M + 127) / 128) * ((N + 63) / 64) <= kCUs) return 0;
    if (srounds == 1) return small >= 140 ? 128 : 0;
    if (M > 16 && M <= 64) return 128;
    const bool wide = M > 64 && (N + 127) / 128 * 128 * int64_t(10) <= N * int64_t(11);
    const int share = K > 256 && wide ? 90 : 75;
    return K <= 512 && small * 100 >= srounds * kCUs * share && (M <= 64 || M > 128) ? 128 : 0;
}

// The tile of an operator that runs on gemm_pp_kernel (0: it does not)
static int pp_tile(const GemmParams& p) {
    // (the output span is addressed with 32-bit offsets, below the out-of-range offset 2^31)
    const int64_t c_span = ((p.M - 1) * p.ldc + p.N) * (p.out_f32 ? 4 : 2);
    if (p.thin || p.epi != EPI_STD || p.splits != 1 || c_span >= (int64_t(1) << 31)) return 0;
    // float32 results and second biases: the LSTM's input projection only
    if (p.out_f32 && (p.conv || p.res || p.act != MOPAR_ACT_NONE || p.N % 8 != 0 || p.ldc % 8 != 0)) return 0;
    if (p.bias2 && !p.out_f32) return 0;
    // a 64-wide k tile of a conv lies in one tap, and a tap has a bit of a 32-bit mask; the operand and
    // the rows of padding before it are addressed together
    if (p.conv && (p.cs % 64 != 0 || p.kh * p.kw > 32 || p.pad >= p.img_w ||
                   int64_t(p.a_bytes) + (int64_t(p.pad) * p.img_w + p.pad) * p.cs * 2 >= (int64_t(1) << 31)))
        return 0;
    return pp_tile_size(p.M, p.N, p.K);
}

template <int TILE>
static hipError_t launch_pp(const GemmParams& params, hipStream_t st) {
    GemmParams p = params;
    p.c_bytes = static_cast<uint32_t>(((p.M - 1) * p.ldc + p.N) * (p.out_f32 ? 4 : 2));
    const int64_t mt = (p.M + TILE - 1) / TILE, nt = (p.N + TILE - 1) / TILE;
    const int64_t total = mt * nt;
    if (total >= (int64_t(1) << 31) / kPPGroupM) return hipErrorInvalidValue;
    p.g_mt = static_cast<int>(mt);
    p.g_nt = static_cast<int>(nt);
    p.g_total = static_cast<int>(total);
    p.g_per_xcd = static_cast<int>((total + 7) / 8);
    p.g_nk = (p.K + 63) / 64;
    p.g_div_group = FastDiv(static_cast<unsigned>(kPPGroupM * p.g_nt));
    const int last = static_cast<int>(mt - (mt - 1) / kPPGroupM * kPPGroupM);
    p.g_div_last = FastDiv(static_cast<unsigned>(last));
    if (p.g_nk < (TILE == 256 ? 2 : 3)) return hipErrorInvalidValue;
    // tiles per block: one round of 32 blocks per XCD where that is at most kPPChunk tiles each
    const int rounds = (p.g_per_xcd + 31) / 32;
    p.g_chunk = rounds < kPPChunk ? rounds : kPPChunk;
    const int per = 32 * p.g_chunk;
    const unsigned grid = static_cast<unsigned>((p.g_per_xcd + per - 1) / per * 32 * 8);
    // whole aligned groups of eight columns everywhere
    const bool regular = p.N % 8 == 0 && p.ldc % 8 == 0 &&
                         ((reinterpret_cast<uintptr_t>(p.C) | reinterpret_cast<uintptr_t>(p.res) |
                           reinterpret_cast<uintptr_t>(p.bias) | reinterpret_cast<uintptr_t>(p.bias2)) & 15) == 0;
    if (p.out_f32 && (!regular || p.conv)) return hipErrorInvalidValue;   // see pp_tile
    const dim3 g(grid), b(512);
    auto go_act = [&](auto conv, auto epi) {
        constexpr bool C = decltype(conv)::value;
        constexpr int E = decltype(epi)::value;
        if (p.act == MOPAR_ACT_RELU)
            launch_kernel(gemm_pp_kernel<TILE, C, E, MOPAR_ACT_RELU>, g, b, 0, st, p);
        else if (p.act == MOPAR_ACT_GELU)
            launch_kernel(gemm_pp_kernel<TILE, C, E, MOPAR_ACT_GELU>, g, b, 0, st, p);
        else
            launch_kernel(gemm_pp_kernel<TILE, C, E, MOPAR_ACT_NONE>, g, b, 0, st, p);
    };
    auto go = [&](auto conv) {
        constexpr bool C = decltype(conv)::value;
        if (!regular)
            go_act(conv, std::integral_constant<int, PP_ANY>{});
        else if (p.out_f32)
            launch_kernel(gemm_pp_kernel<TILE, false, PP_F32, MOPAR_ACT_NONE>, g, b, 0, st, p);
        else if (p.res)
            go_act(conv, std::integral_constant<int, PP_RES>{});
        else
            go_act(conv, std::integral_constant<int, PP_BF16>{});
    };
    if (p.conv)
        go(std::true_type{});
    else
        go(std::false_type{});
    return hipGetLastError();
}

// Whether a bf16 product of more than 64 rows takes 32 x 32 tiles, four times as many, for its `blocks` 64 x 64
// ones: while those leave at least a quarter of the CUs idle (us, 64 x 64 / 32 x 32 tiles: 1600 x 1024 -> 256, 100
// blocks, 7.8 / 6.7; 1024 x 768 -> 768, 192, 6.9 / 6.5; 3136 x 1024 -> 256, 196, 8.1 / 8.5; 900 x 1024 -> 1024, 240,
// 8.2 / 8.7; 3136 x 512 -> 512, 392, 7.4 / 9.1).
bool tiles_32x32(int64_t blocks) { return blocks * 4 <= kCUs * 3; }

// Whether a product of 17 to 64 rows takes 32 x 16 tiles, eight times as many, for its `blocks` 64 x 64 ones
// (us, 64 x 64 / 32 x 16 tiles).  bf16: under 128 blocks (33 x 768 -> 6000, 94 blocks, 8.0 / 5.7; 64 x 1024 -> 8000, 125,
// 8.8 / 9.3, 64 x 512 -> 8000 7.3 / 7.1; 64 x 512 -> 12000, 188, 7.5 / 8.2).  float32, whose 64 x 64 tiles pay most for the
// block sums: up to 32 rows always (17 x 512 -> 7000 15.3 / 7.0, -> 20000 29.0 / 13.9), above while those leave a quarter
// of their rounds idle (64 x 512 -> 9216, 144 blocks, 16.2 / 13.3; -> 12000, 188, 16.4 / 15.0; -> 16000, 250, 17.0 /
// 20.2; -> 20000, 313, 31.2 / 24.6).
bool tiles_32x16(int64_t M, int64_t blocks, bool bf16) {
    if (bf16) return blocks < kCUs / 2;
    return M <= 32 || blocks * 4 <= (blocks + kCUs - 1) / kCUs * kCUs * 3;
}

template <typename T>
static hipError_t dispatch(const GemmParams& p, hipStream_t st) {
    const int width = (p.N + p.ksub - 1) / p.ksub;   // widest sub-slice
    if constexpr (sizeof(T) == 2) {
        const int tile = pp_tile(p);
        if (tile) return tile == 256 ? launch_pp<256>(p, st) : launch_pp<128>(p, st);
    }
    if (sizeof(T) == 4 && p.epi == EPI_STD && f32_small_tiles(p.M, p.N, p.K))
        return launch_cfg<T, 32, 16, 1, 1, 2, 4, 4>(p, width, st);
    // few rows: the four waves split K (four 64-wide sub-stages per stage) instead of the tile
    if (p.M <= 16) return launch_cfg<T, 16, 64, 1, 1, 3, 4, 4>(p, width, st);
    // the LSTM step: 32 x 16 tiles (twice the blocks of 64 x 16, less LDS each) measured
    // fastest, alone and beside other streams' kernels
    if (p.epi == EPI_LSTM) return launch_cfg<T, 32, 16, 1, 1, 2, 4, 4>(p, width, st);
    if (p.M <= 64 && tiles_32x16(p.M, (width + 63) / 64 * p.ksub * p.splits, sizeof(T) == 2))
        return launch_cfg<T, 32, 16, 1, 1, 2, 4, 4>(p, width, st);
    if (p.M <= 64) {
        if (width >= 64) return launch_cfg<T, 64, 64, 1, 1, 2, 4, 4>(p, width, st);
        return launch_cfg<T, 64, 16, 1, 1, 3, 4, 4>(p, width, st);
    }
    const int64_t mt = (p.M + 127) / 128;
    auto blocks = [&](int64_t bm_tiles, int bn) { return bm_tiles * ((width + bn - 1) / bn) * p.ksub * p.splits; };
    // a codec layer with at most 128 output columns whose 64-row tiles would not give every
    // compute unit a block: 32 x 32 tiles (measured about 20 % faster on such encoders, cold)
    if (p.thin && width <= 128 && blocks((p.M + 63) / 64, width >= 64 ? 64 : 32) < kCUs)
        return launch_cfg<T, 32, 32, 2, 2, 4>(p, width, st);
    // float32 is MFMA-bound, rows past M cost as much as any: 64-row tiles where 128-row ones would leave more
    // than a tenth of theirs empty (308 x 768 -> 3072: 32.6 us on 128 x 64 tiles, 21.7 us on 64 x 64)
    if (sizeof(T) == 4 && width >= 64 && mt * 128 * 10 > p.M * 11) return launch_cfg<T, 64, 64, 2, 4, 4>(p, width, st);
    // 128-wide tiles unless they would leave more than a tenth of the columns they cover empty
    const bool w128 = width >= 128 && (width + 127) / 128 * 128 * 10 <= width * 11;
    if (w128 && blocks(mt, 128) >= kCUs) return launch_cfg<T, 128, 128, 2, 4, 2>(p, width, st);
    if (width >= 64 && blocks(mt, 64) >= kCUs) return launch_cfg<T, 128, 64, 4, 2, 3>(p, width, st);
    if (sizeof(T) == 2 && width >= 64 && !p.thin && tiles_32x32(blocks((p.M + 63) / 64, 64)))
        return launch_cfg<T, 32, 32, 2, 2, 4>(p, width, st);
    if (width >= 64) return launch_cfg<T, 64, 64, 2, 4, 4>(p, width, st);
    if (width >= 32) {
        if (blocks(mt, 32) >= kCUs) return launch_cfg<T, 128, 32, 4, 2, 3>(p, width, st);
        return launch_cfg<T, 64, 32, 4, 2, 4>(p, width, st);
    }
    // 16-column sub-slices: 64 x 16 tiles measured faster than 128 x 16 at every grid size tried
    return launch_cfg<T, 64, 16, 4, 1, 4>(p, width, st);
}

hipError_t launch_gemm(const GemmParams& params, int dtype, hipStream_t stream) {
    GemmParams p = params;
    if (p.splits < 1) p.splits = 1;
    if (p.ksub < 1) p.ksub = 1;
    if (p.conv) {
        p.div_hw = FastDiv(static_cast<unsigned>(p.out_h * p.out_w));
        p.div_w = FastDiv(static_cast<unsigned>(p.out_w));
    }
    if (p.M <= 0 || p.N <= 0) return hipSuccess;
    if (p.M > (int64_t(1) << 31) - 256) return hipErrorInvalidValue;   // rows are 32-bit in the kernel
    // operands are read through buffer resources with 32-bit byte offsets, and offset 2^31
    // must lie past both of them
    const int64_t esz = dtype == MOPAR_BF16 ? 2 : 4;
    const int64_t a_bytes = p.conv ? p.M / (int64_t(p.out_h) * p.out_w) * p.img_h * p.img_w * p.cs * esz
                                   : p.M * p.lda * esz;
    const int64_t b_bytes = int64_t(p.N) * p.K * esz;
    if (a_bytes >= (int64_t(1) << 31) || b_bytes >= (int64_t(1) << 31)) return hipErrorInvalidValue;
    p.a_bytes = static_cast<uint32_t>(a_bytes);
    p.b_bytes = static_cast<uint32_t>(b_bytes);
    // the reduce keeps every split's partial in flight at once, for at most 16 splits
    if (p.splits < 1 || p.splits > 16 || (p.splits > 1 && (!p.partial || p.epi != EPI_STD)))
        return hipErrorInvalidValue;
    if (p.conv && conv_halo_ok(dtype, p.kh, p.kw, p.stride, p.pad, p.cs, p.N, p.out_h, p.out_w, p.M)) {
        if (p.splits != 1 || p.epi != EPI_STD) return hipErrorInvalidValue;
        // 16-column tiles at every width (measured at least as fast as 32 on 32-wide sub-slices)
        const int width = (p.N + p.ksub - 1) / p.ksub;
        return p.cs / 64 > 2 ? launch_halo<16, 8, 2>(p, width, stream) : launch_halo<16, 8, 1>(p, width, stream);
    }
    hipError_t e = dtype == MOPAR_BF16 ? dispatch<__bf16>(p, stream) : dispatch<float>(p, stream);
    if (e != hipSuccess || p.splits == 1) return e;
    const int64_t n = p.M * ((p.N + 3) / 4);
    if (n >= (int64_t(1) << 31)) return hipErrorInvalidValue;
    p.r_div_groups = FastDiv(static_cast<unsigned>((p.N + 3) / 4));
    const unsigned blocks = static_cast<unsigned>((n + 255) / 256);
    if (dtype == MOPAR_BF16)
        launch_kernel(splitk_reduce_kernel<__bf16>, dim3(blocks), dim3(256), 0, stream, p);
    else
        launch_kernel(splitk_reduce_kernel<float>, dim3(blocks), dim3(256), 0, stream, p);
    return hipGetLastError();
}

}  // namespace mopar
