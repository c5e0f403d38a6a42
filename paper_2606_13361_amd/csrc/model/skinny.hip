// skinny.hip -- matrix products of a few rows (2 .. 48 tokens: a question over
// a cached document), y[T][N] = x[T][K] w[N][K]^T, on the matrix cores.
//
// What bounds them: reading the weights once, and the tokens' rows once per
// compute unit.  A decoder layer of the 4B geometry moves 202 MB of weights for 24
// tokens, 32 us at the 6.3 TB/s that a streaming read reaches; the arithmetic is a
// tenth of that; and as every workgroup needs all of x, L2 delivers more bytes of x
// than of weights (down product, 256 workgroups of 10 outputs: 120 MB of x to 50 MB
// of weights, 18 us).
//
// The waves of a workgroup split K: each streams its part of the tile's weight rows
// through a ring of its own in LDS, 64 elements (one 128-byte line of 16 rows, 2 KB)
// a stage, by direct loads that it alone waits for.  (Loaded straight into the
// operand layout, 16 bytes from each of 16 rows per instruction, the same bytes took
// three times as long: the address path takes neighbouring lanes' addresses one by
// one.)  The tokens are the other operand, v_mfma_f32_16x16x32 with 16 weight rows
// by 16 tokens.  The waves' partial sums meet in LDS in wave order.
//
//   skinny_reg_kernel    the normalized input (QKV, gate/up), K = 256 S: a wave's
//                        share of the tokens stays in registers for all tiles of
//                        its workgroup, 16 outputs or fewer each; the tokens come
//                        packed in operand order from the norm.  pair: a tile is 8
//                        gate rows and their 8 up rows, the epilogue stores
//                        silu(g) * u with g and u rounded to the element format
//                        first
//   skinny_split_kernel  the residual products (O, down): K in four parts, so that a
//                        workgroup of 1/256 of the weights covers four times the
//                        outputs and reads a quarter of x, which streams through
//                        the ring with the weights; the four partial sums are added
//                        by residual_kernel, which the O product shares with the
//                        next norm
//
// Measured (24 tokens, bf16, hidden 2560, one layer over 3774 cached tokens, kernel
// times), library products with their norm and activation launches -> these: QKV
// 3.5 + 12.5 -> 3.7 + 11.8 us, O 13.4 -> 6.2, gate/up 4.0 + 25 + 4.5 -> 4.0 + 21.7,
// down 20 -> 13 + 3.7; the layer 100 -> 81.5 us, with 5 tokens 114 -> 69.7, with 40
// 112 -> 90.8.
#include "skinny.hpp"

#include <type_traits>

#include "attn_common.hpp"
#include "silu.hpp"

namespace kvr {
namespace model {
namespace {

using namespace dev;

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int NWV = 8;             // skinny_reg_kernel
constexpr int THREADS = 64 * NWV;
constexpr int SWV = 4;             // skinny_split_kernel
constexpr int RT = 3;              // its 16-row tiles per workgroup
constexpr int64_t kCus = 256;
constexpr int WST = 2048;          // bytes of a weight stage: 16 rows x 128
constexpr int XST = 1024;          // bytes of a tokens' stage per group of eight: 2 steps x 512
constexpr int LDS_MAX = 160 * 1024;

template <class E>
__device__ __forceinline__ f32x4 mfma16(u32x4 a, u32x4 b, f32x4 c) {
    if constexpr (std::is_same<E, Bf16>::value)
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(a), as_bf16x8(b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0,
                                                      0, 0);
}

// 16-byte chunk c of weight row m of a stage sits in slot c ^ wswz(m): 16 lanes
// reading one chunk of the 16 rows touch every bank once
__device__ __forceinline__ int wswz(int m) { return (m >> 1) & 7; }

// The weight row that row m of a tile is: outputs past the tile or past N repeat
// its last one (loaded, never stored).
template <bool PAIR>
__device__ __forceinline__ int64_t weight_row(const SkinnyParams &p, int64_t n0, int m) {
    const int last = (int)min((int64_t)p.rows, p.N - n0) - 1;
    if (PAIR) return n0 + min(m & 7, last) + (m >> 3) * p.N;
    return n0 + min(m, last);
}

// vmcnt holds 63; rings deep enough to exceed it do not exist
constexpr int left(int n, int per) { return n * per < 63 ? n * per : 63; }
// s_waitcnt for "every load but the last n * PER of this wave has landed" (stores
// in between only make it wait longer)
template <int PER>
__device__ __forceinline__ void wait_left(int n) {
    switch (n) {
        case 0: wait_vmcnt<0>(); break;
        case 1: wait_vmcnt<left(1, PER)>(); break;
        case 2: wait_vmcnt<left(2, PER)>(); break;
        case 3: wait_vmcnt<left(3, PER)>(); break;
        case 4: wait_vmcnt<left(4, PER)>(); break;
        case 5: wait_vmcnt<left(5, PER)>(); break;
        case 6: wait_vmcnt<left(6, PER)>(); break;
        default: wait_vmcnt<left(7, PER)>(); break;
    }
}

// Column tile c's sums over the eight waves, in wave order, and their outputs:
// lane (token j of the tile, kg) holds outputs 4 kg .. 4 kg + 3.
template <class E, int CT, bool PAIR>
__device__ __forceinline__ void finish(const SkinnyParams &p, const f32x4 *buf, int c, int64_t n0, int lane) {
    const int kg = lane >> 4;
    const int t = 16 * c + (lane & 15);
    f32x4 s = buf[c * 64 + lane];
#pragma unroll
    for (int w = 1; w < NWV; ++w) s += buf[(w * CT + c) * 64 + lane];
    uint16_t *y = p.y + (int64_t)t * p.N + n0 + 4 * kg;
    if constexpr (PAIR) {
        float a[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float up = __shfl_xor(s[r], 32);        // the up rows of lanes kg = 0, 1
            const float g = E::lo(E::pack2(s[r], 0.f)), u = E::lo(E::pack2(up, 0.f));
            a[r] = silu(g) * u;
        }
        if (kg >= 2 || t >= p.T) return;
        u32x2 v;                                          // tiles of 8 outputs of N = 8 i: 8-byte aligned
        v[0] = E::pack2(a[0], a[1]);
        v[1] = E::pack2(a[2], a[3]);
        *(u32x2 *)y = v;
    } else {
        if (t >= p.T) return;
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (4 * kg + r < p.rows && n0 + 4 * kg + r < p.N) y[r] = (uint16_t)(E::pack2(s[r], 0.f) & 0xffffu);
    }
}

// dma16 with the non-temporal hint: a layer's weights are read once and come back
// after more bytes than any cache holds (a decoder layer over 24 tokens 81.4 -> 74.5
// us with it, over 5 tokens 67.9 -> 63.3, over 40 90.7 -> 82.9).
__device__ __forceinline__ void dma16_nt(const void *src, const void *lds_dst) {
    const uint32_t lds = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void *)lds_dst;
    asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, off nt" ::"s"(lds), "v"(src) : "m0");
}

// Two loads of a weight stage: lane -> row 8 i + lane / 8, slot lane % 8
template <bool PAIR>
struct WSrc {
    uint64_t a[2];
    __device__ __forceinline__ void point(const SkinnyParams &p, int64_t n0, int64_t k0, int lane) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int m = 8 * i + (lane >> 3);
            a[i] = (uint64_t)(uintptr_t)(p.w + weight_row<PAIR>(p, n0, m) * p.K + k0) + 16u * ((lane & 7) ^ wswz(m));
        }
    }
    __device__ __forceinline__ void load(int stage, const unsigned char *dst) const {
#pragma unroll
        for (int i = 0; i < 2; ++i) dma16_nt((const void *)(a[i] + (uint64_t)stage * 128), dst + 1024 * i);
    }
};

__device__ __forceinline__ u32x4 wfrag(const unsigned char *st, int h, int lane) {   // step h of a stage
    const int m = lane & 15, c = 4 * h + (lane >> 4);
    return *(const u32x4 *)(st + m * 128 + 16 * (c ^ wswz(m)));
}

// Elements from a step's packed rows to the lane's 8 of column tile c (token 16 c +
// lane % 16, k group lane / 16); groups past the last repeat it, never stored.
__device__ __forceinline__ int xlane(int c, int ht, int lane) {
    const int u = min(2 * c + ((lane >> 3) & 1), ht - 1);
    return ((u * 4 + (lane >> 4)) * 8 + (lane & 7)) * 8;
}

// K = 256 S.  The workgroup walks tiles blockIdx.x, + gridDim.x, ... as one stream
// of stages.
template <class E, int CT, int S, bool PAIR>
__global__ __launch_bounds__(THREADS) void skinny_reg_kernel(const SkinnyParams p) {
    constexpr int NR = CT == 1 ? 8 : CT == 2 ? 7 : 6;      // ring slots
    constexpr int SPT = S / 2;                             // a wave's stages per tile
    __shared__ __attribute__((aligned(1024))) unsigned char ring[NWV * NR * WST];
    __shared__ f32x4 buf[2][NWV * CT * 64];
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63;
    const int64_t tiles = (p.N + p.rows - 1) / p.rows;
    const int mine = (int)((tiles - blockIdx.x + gridDim.x - 1) / gridDim.x);   // this workgroup's tiles
    const int total = mine * SPT;
    unsigned char *slots = ring + wave * NR * WST;

    // the loads' cursor, NR - 1 stages ahead of the products
    WSrc<PAIR> src;
    int ci = 0, cq = 0;
    int64_t ctile = blockIdx.x;
    auto issue = [&]() {
        if (ci >= total) return;
        if (cq == 0) src.point(p, ctile * p.rows, 32 * S * wave, lane);
        src.load(cq, slots + (ci % NR) * WST);
        ++ci;
        if (++cq == SPT) {
            cq = 0;
            ctile += gridDim.x;
        }
    };
    for (int i = 0; i < NR - 1; ++i) issue();
    u32x4 x[CT][S];
    const int ht = (p.T + 7) >> 3;
#pragma unroll
    for (int c = 0; c < CT; ++c) {
        const uint16_t *xc = p.x + (int64_t)wave * S * ht * 256 + xlane(c, ht, lane);
#pragma unroll
        for (int s = 0; s < S; ++s) x[c][s] = *(const u32x4 *)(xc + s * ht * 256);
    }
    // the compiler's wait for the tokens lands here (with it the first stages'),
    // and none in the loop, where only the direct loads are counted
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
        for (int c = 0; c < CT; ++c) asm volatile("" ::"v"(x[c][s]));

    int i = 0;
    for (int n = 0; n < mine; ++n) {
        f32x4 acc[CT];
#pragma unroll
        for (int c = 0; c < CT; ++c) acc[c] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int q = 0; q < SPT; ++q, ++i) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // stage i - 1 has been read
            issue();                                       // into its slot
            wait_left<2>(min(NR - 1, total - 1 - i));
            const unsigned char *st = slots + (i % NR) * WST;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const u32x4 w = wfrag(st, h, lane);
#pragma unroll
                for (int c = 0; c < CT; ++c) acc[c] = mfma16<E>(w, x[c][2 * q + h], acc[c]);
            }
        }
        f32x4 *b = buf[n & 1];
#pragma unroll
        for (int c = 0; c < CT; ++c) b[(wave * CT + c) * 64 + lane] = acc[c];
        // LDS only: the weights stay in flight.  The barrier also says that the
        // other buffer, read by finish() a tile ago, may be written
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if (wave < CT) finish<E, CT, PAIR>(p, b, wave, (blockIdx.x + (int64_t)n * gridDim.x) * p.rows, lane);
    }
}

// Workgroup (output group, quarter of K): RT 16-row tiles of p.rows outputs together
// (rows past the group or past N repeat its last one), SWV waves over the quarter's
// stages.  A stage holds the tiles' weights, then the tokens: 8 rows x 128 bytes per
// group of eight, laid out like the weight rows.
template <class E, int HT>
__global__ __launch_bounds__(64 * SWV) void skinny_split_kernel(const SkinnyParams p) {
    constexpr int CT = (HT + 1) / 2;
    constexpr int SLOT = RT * WST + HT * XST;
    constexpr int NR = LDS_MAX / (SWV * SLOT) < 5 ? LDS_MAX / (SWV * SLOT) : 5;   // 5, 5, 4, 4, 3, 3
    constexpr int PER = 2 * RT + HT;                       // loads of a stage
    __shared__ __attribute__((aligned(1024))) unsigned char ring[SWV * NR * SLOT];
    static_assert(SWV * RT * CT * 1024 <= SWV * NR * SLOT, "the sums do not fit the ring");
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63;
    const int f = blockIdx.x % kSplitK;
    const int64_t n0 = (int64_t)(blockIdx.x / kSplitK) * p.rows;
    const int last = (int)min((int64_t)p.rows, p.N - n0) - 1;
    const int stages = p.K / 64;
    const int fs0 = (int)((int64_t)stages * f / kSplitK), fs1 = (int)((int64_t)stages * (f + 1) / kSplitK);
    const int s0 = fs0 + (fs1 - fs0) * wave / SWV, total = fs0 + (fs1 - fs0) * (wave + 1) / SWV - s0;
    unsigned char *slots = ring + wave * NR * SLOT;

    // load i: rows 8 i + lane / 8 (weights, then tokens), slot lane % 8
    uint64_t a[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int m = 8 * i + (lane >> 3);
        const bool wt = i < 2 * RT;
        const int64_t row = wt ? n0 + min(m, last) : min(m - 16 * RT, p.T - 1);
        a[i] = (uint64_t)(uintptr_t)((wt ? p.w : p.x) + row * p.K + (int64_t)s0 * 64) + 16u * ((lane & 7) ^ wswz(m & 15));
    }
    auto issue = [&](int i) {
        if (i >= total) return;
        unsigned char *d = slots + (i % NR) * SLOT;
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            if (u < 2 * RT) dma16_nt((const void *)(a[u] + (uint64_t)i * 128), d + 1024 * u);
            else dma16((const void *)(a[u] + (uint64_t)i * 128), d + 1024 * u);
        }
    };
    for (int i = 0; i < NR - 1; ++i) issue(i);
    f32x4 acc[RT][CT];
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int c = 0; c < CT; ++c) acc[r][c] = (f32x4){0.f, 0.f, 0.f, 0.f};
    // tokens' fragments: row 16 c + lane % 16; a tile's rows past the last group
    // repeat its first eight, never stored
    int xo[CT][2];
#pragma unroll
    for (int c = 0; c < CT; ++c) {
        const int t = lane & 15;
        const int row = 16 * c + (2 * c + (t >> 3) < HT ? t : t & 7);
#pragma unroll
        for (int h = 0; h < 2; ++h) xo[c][h] = RT * WST + row * 128 + 16 * ((4 * h + (lane >> 4)) ^ wswz(row & 15));
    }
    for (int i = 0; i < total; ++i) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // stage i - 1 has been read
        issue(i + NR - 1);                                 // into its slot
        wait_left<PER>(min(NR - 1, total - 1 - i));
        const unsigned char *st = slots + (i % NR) * SLOT;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            u32x4 x[CT];
#pragma unroll
            for (int c = 0; c < CT; ++c) x[c] = *(const u32x4 *)(st + xo[c][h]);
#pragma unroll
            for (int r = 0; r < RT; ++r) {
                const u32x4 w = wfrag(st + r * WST, h, lane);
#pragma unroll
                for (int c = 0; c < CT; ++c) acc[r][c] = mfma16<E>(w, x[c], acc[r][c]);
            }
        }
    }
    __syncthreads();                                       // the rings are no longer read
    f32x4 *b = (f32x4 *)ring;
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int c = 0; c < CT; ++c) b[((wave * RT + r) * CT + c) * 64 + lane] = acc[r][c];
    __syncthreads();
    for (int u = wave; u < RT * CT; u += SWV) {
        const int r = u / CT, c = u % CT;
        const int t = 16 * c + (lane & 15), m = 16 * r + 4 * (lane >> 4);
        f32x4 v = b[u * 64 + lane];
#pragma unroll
        for (int w = 1; w < SWV; ++w) v += b[(w * RT * CT + u) * 64 + lane];
        if (t < p.T && m <= last)                          // groups of four outputs: whole or none (p.rows, N % 4 == 0)
            *(f32x4 *)(p.part + ((int64_t)f * p.T + t) * p.N + n0 + m) = v;
    }
}

// One workgroup per token: the residual add of the partial sums, then the norm
// into packed rows (see skinny.hpp).
constexpr int PT = 512;
template <class E>
__global__ __launch_bounds__(PT) void residual_kernel(uint16_t *h, const float *part, const uint16_t *ln, uint16_t *xp,
                                                      int K, int T, float eps) {
    constexpr int MAXC = 1;                                // 8-element chunks of a row per thread: K <= 4096
    static_assert(MAXC * PT * 8 >= 4096, "row width");
    __shared__ float red[PT / 64];
    const int t = blockIdx.x, i = threadIdx.x;
    const bool act = i < K / 8;
    uint16_t *hr = h + (int64_t)t * K + 8 * i;
    u32x4 v = {0, 0, 0, 0}, g = {0, 0, 0, 0};
    if (act) {
        v = *(const u32x4 *)hr;
        if (ln) g = *(const u32x4 *)(ln + 8 * i);
        if (part) {
            float4 s[2] = {make_float4(0.f, 0.f, 0.f, 0.f), make_float4(0.f, 0.f, 0.f, 0.f)};
#pragma unroll
            for (int f = 0; f < kSplitK; ++f)
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const float4 a = *(const float4 *)(part + ((int64_t)f * T + t) * K + 8 * i + 4 * q);
                    s[q].x += a.x; s[q].y += a.y; s[q].z += a.z; s[q].w += a.w;
                }
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                v[2 * q] = E::pack2(E::lo(v[2 * q]) + s[q].x, E::hi(v[2 * q]) + s[q].y);
                v[2 * q + 1] = E::pack2(E::lo(v[2 * q + 1]) + s[q].z, E::hi(v[2 * q + 1]) + s[q].w);
            }
            *(u32x4 *)hr = v;
        }
    }
    if (!ln) return;
    float ss = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float a = E::lo(v[e]), b = E::hi(v[e]);
        ss = __builtin_fmaf(a, a, ss);
        ss = __builtin_fmaf(b, b, ss);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o);
    if ((i & 63) == 0) red[i >> 6] = ss;
    __syncthreads();
    float tot = 0.f;
#pragma unroll
    for (int w = 0; w < PT / 64; ++w) tot += red[w];
    const float inv = 1.0f / sqrtf(tot / (float)K + eps);
    if (!act) return;
#pragma unroll
    for (int e = 0; e < 4; ++e)
        v[e] = E::pack2(E::lo(v[e]) * inv * E::lo(g[e]), E::hi(v[e]) * inv * E::hi(g[e]));
    const int ht = (T + 7) >> 3;
    *(u32x4 *)(xp + ((((int64_t)(i >> 2) * ht + (t >> 3)) * 4 + (i & 3)) * 8 + (t & 7)) * 8) = v;
}

template <class E, int CT, bool PAIR>
void launch_reg(const SkinnyParams &p, hipStream_t s) {
    const int64_t tiles = (p.N + p.rows - 1) / p.rows;
    const dim3 grid((unsigned)(tiles < kCus ? tiles : kCus)), th(THREADS);
    if (p.K == 2048) hipLaunchKernelGGL((skinny_reg_kernel<E, CT, 8, PAIR>), grid, th, 0, s, p);
    else if (p.K == 2560) hipLaunchKernelGGL((skinny_reg_kernel<E, CT, 10, PAIR>), grid, th, 0, s, p);
    else hipLaunchKernelGGL((skinny_reg_kernel<E, CT, 16, PAIR>), grid, th, 0, s, p);
}

template <class E, bool PAIR>
void launch_reg_e(const SkinnyParams &p, hipStream_t s) {
    const int ct = (p.T + 15) / 16;
    if (ct == 1) launch_reg<E, 1, PAIR>(p, s);
    else if (ct == 2) launch_reg<E, 2, PAIR>(p, s);
    else launch_reg<E, 3, PAIR>(p, s);
}

template <class E>
void launch_split_e(const SkinnyParams &p, hipStream_t s) {
    const dim3 grid((unsigned)((p.N + p.rows - 1) / p.rows * kSplitK)), th(64 * SWV);
    switch (token_groups(p.T)) {
        case 1: hipLaunchKernelGGL((skinny_split_kernel<E, 1>), grid, th, 0, s, p); break;
        case 2: hipLaunchKernelGGL((skinny_split_kernel<E, 2>), grid, th, 0, s, p); break;
        case 3: hipLaunchKernelGGL((skinny_split_kernel<E, 3>), grid, th, 0, s, p); break;
        case 4: hipLaunchKernelGGL((skinny_split_kernel<E, 4>), grid, th, 0, s, p); break;
        case 5: hipLaunchKernelGGL((skinny_split_kernel<E, 5>), grid, th, 0, s, p); break;
        default: hipLaunchKernelGGL((skinny_split_kernel<E, 6>), grid, th, 0, s, p); break;
    }
}

}  // namespace

hipError_t launch_skinny_norm(SkinnyParams p, bool pair, bool f16, hipStream_t s) {
    // outputs per tile: as many tiles per compute unit as full tiles need, evenly
    // filled (6144 outputs: 512 tiles of 12); pairs: 8
    const int64_t rounds = (p.N + 16 * kCus - 1) / (16 * kCus);
    p.rows = pair ? 8 : (int32_t)((p.N + kCus * rounds - 1) / (kCus * rounds));
    if (pair) {
        if (f16) launch_reg_e<F16, true>(p, s);
        else launch_reg_e<Bf16, true>(p, s);
    } else {
        if (f16) launch_reg_e<F16, false>(p, s);
        else launch_reg_e<Bf16, false>(p, s);
    }
    return hipGetLastError();
}

hipError_t launch_skinny_split(SkinnyParams p, bool f16, hipStream_t s) {
    // one workgroup per compute unit and round: groups of outputs, a multiple of 8,
    // at most RT tiles (2560 outputs: 64 groups of 40)
    const int64_t groups = kCus / kSplitK;
    const int64_t rounds = (p.N + 16 * RT * groups - 1) / (16 * RT * groups);
    p.rows = (int32_t)((p.N + 8 * groups * rounds - 1) / (8 * groups * rounds) * 8);
    if (f16) launch_split_e<F16>(p, s);
    else launch_split_e<Bf16>(p, s);
    return hipGetLastError();
}

hipError_t launch_residual(uint16_t *h, const float *part, const uint16_t *ln, uint16_t *xp, int T, int K, float eps,
                           bool f16, hipStream_t s) {
    if (f16) hipLaunchKernelGGL(residual_kernel<F16>, dim3(T), dim3(PT), 0, s, h, part, ln, xp, K, T, eps);
    else hipLaunchKernelGGL(residual_kernel<Bf16>, dim3(T), dim3(PT), 0, s, h, part, ln, xp, K, T, eps);
    return hipGetLastError();
}

}  // namespace model
}  // namespace kvr
