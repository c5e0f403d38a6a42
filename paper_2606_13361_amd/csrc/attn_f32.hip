// attn_f32.hip -- the fp32 member of the attention family: the same rows,
// segments and causal offset as the 16-bit kernels, computed entirely in fp32
// (fp32 matrix instructions; the hardware's 2^x, within an ulp, for the weights), for
// inputs whose tolerance is 1e-5.
//
// What bounds it: the fp32 matrix rate, 256 flops per clock and CU.  A
// workgroup is 8 waves (two per SIMD) that all hold the same 16 * NCT query
// rows and split the keys: wave w takes the 16-key stages w, w + 8, ... of the
// tile's keys, straight from memory into registers (a K or V row reaches its
// lanes in 16-byte pieces; the next stage's pieces are requested as the current
// ones are used up), so the key loop has no barrier and no LDS.  The eight
// (m, l, O) meet in LDS at the end.
//
// Transposed products as in the 16-bit kernels, on v_mfma_f32_16x16x4_f32
// (lane l: column l % 16, k group kg = l / 16):
//   S^T[key][row] = K Q^T     lane (key, kg) reads head dims 16c + 4 kg .. +3 of
//                             its key; product e of chunk c uses dim 16c + 4 kg + e
//   O^T[d][row] += V^T P^T    the score accumulator register e of a lane is the
//                             weight of key 4 kg + e: the operand of product e as
//                             it stands; lane (m, kg) reads dims MT m .. MT m + MT - 1
//                             of key 4 kg + e, MT = D / 16
//
// Row tiles: 16 rows (NCT = 1) give twice the workgroups, 32 rows (NCT = 2) read
// every key once for two column tiles; the caller takes 32 once there are 512 of
// them (two rounds of the part).
//
// Measured against the vector-ALU kernel this one replaces (64 rows per
// workgroup, the keys one after another), 32 / 8 heads, d = 128: 24 tokens over
// 945 cached rows 438 -> 28 us (48 workgroups: the bound is their own 14 us of
// matrix time), prefill 1000 491 -> 114 us, 4000 4257 -> 1274 us (103 TFLOP/s of
// the 157 peak); one token over 700 rows 372 -> 24 us.  Error against 64 bits
// (2-norm) at the first shape 7.4e-7 -> 2.8e-7; with 16 times larger scores 8.9e-7 ->
// 8.2e-7 (1.24e-6 with scores of two chains).
#include <type_traits>

#include "attn_common.hpp"

namespace kvr {
namespace {

using dev::rope_rot;

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int NW = 8;              // waves per workgroup
constexpr int THREADS = 64 * NW;
constexpr int SK = 16;             // keys per stage

__device__ __forceinline__ int find_segment_f32(const AttnParams &p, int tile) {
    int lo = 0, hi = p.n_seg - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (p.seg_tile0[mid] <= tile) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// the four lanes l, l^16, l^32, l^48 of a query row
__device__ __forceinline__ float row_max(float x) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return dev::pair_max(fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1])));
}
__device__ __forceinline__ float row_sum(float x) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return dev::pair_sum(__uint_as_float(a[0]) + __uint_as_float(a[1]));
}

// e^t for t <= 0.  (t log2(e) is rounded: that moves a weight by |t| 2^-24 of itself, at
// most 2e-8 of the row's largest.)
__device__ __forceinline__ float exp_neg(float t) { return __builtin_amdgcn_exp2f(t * 1.44269504f); }

template <int D, int NCT>
__global__ __launch_bounds__(THREADS) void attn_f32_kernel(const AttnParams p) {
    constexpr int ROWS = 16 * NCT;
    constexpr int NC = D / 16;         // 16-byte pieces of a K row per lane
    constexpr int MT = D / 16;         // 16-row tiles of O^T
    constexpr int Q4 = MT / 4;         // 16-byte pieces of a V row per lane
    constexpr int UNITS = MT * NCT;    // (column tile, 16-byte piece of O) pairs of the merge
    __shared__ float4 obuf[NW][UNITS][64];
    __shared__ float mbuf[NW][NCT][16], lbuf[NW][NCT][16];

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63;
    const int j = lane & 15;
    const int kg = lane >> 4;

    int b = blockIdx.x;
    const int g = b % p.n_kv_heads;
    b /= p.n_kv_heads;
    const int tile_lin = p.reverse ? (p.tiles_total - 1 - b) : b;
    const int seg = find_segment_f32(p, tile_lin);
    const int rt = tile_lin - p.seg_tile0[seg];
    const int tok0 = p.seg_tok0[seg];
    const int n_tok = p.seg_tok0[seg + 1] - tok0;
    const int G = p.group;
    const int R = G * n_tok;
    const int row0 = rt * ROWS;
    const int row_last = min(row0 + ROWS, R) - 1;
    const int64_t npre = p.n_prefix;
    const int64_t ke = npre + row_last / G + 1;     // keys any row here may see
    const int64_t k_full = npre + row0 / G + 1;     // keys every row here sees
    const int nst = (int)((ke + SK - 1) / SK);

    bool valid[NCT];
    int tok[NCT], head[NCT];
    int64_t pos[NCT];
    f32x4 q[NCT][NC], o[NCT][MT];
    float m_run[NCT], l_run[NCT];
#pragma unroll
    for (int c = 0; c < NCT; ++c) {
        const int r = row0 + 16 * c + j;
        valid[c] = r < R;
        tok[c] = valid[c] ? r / G : 0;
        head[c] = g * G + (valid[c] ? r % G : 0);
        pos[c] = valid[c] ? npre + tok[c] : -1;
        m_run[c] = -INFINITY;
        l_run[c] = 0.f;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) o[c][mt] = (f32x4){0.f, 0.f, 0.f, 0.f};
        const float *qrow = (const float *)p.q + ((int64_t)(tok0 + tok[c]) * p.n_q_heads + head[c]) * D + 4 * kg;
#pragma unroll
        for (int i = 0; i < NC; ++i) q[c][i] = valid[c] ? *(const f32x4 *)(qrow + 16 * i) : (f32x4){0.f, 0.f, 0.f, 0.f};
        // RoPE (prefill, readers): dim i < D/2 pairs with dim i + D/2, which the
        // same lane holds NC/2 pieces further
        if (p.rope && valid[c]) {
            const float *cs = p.rope + pos[c] * D + 8 * kg;
#pragma unroll
            for (int i = 0; i < NC / 2; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    float y1, y2;
                    rope_rot(q[c][i][e], q[c][i + NC / 2][e], cs[32 * i + 2 * e], cs[32 * i + 2 * e + 1], y1, y2);
                    q[c][i][e] = y1;
                    q[c][i + NC / 2][e] = y2;
                }
        }
    }

    const float scale = p.scale;
    const float *kc = (const float *)p.kc + (int64_t)g * p.cap * D;
    const float *vc = (const float *)p.vc + (int64_t)g * p.cap * D;
    const int64_t nstride = p.new_tok_stride;
    const float *kn = (const float *)p.kn + (int64_t)tok0 * nstride + p.new_head_stride * g;
    const float *vn = (const float *)p.vn + (int64_t)tok0 * nstride + p.new_head_stride * g;
    // row of a key; keys past the end repeat the last one (masked, and their V
    // pieces zeroed before use)
    auto row = [&](const float *cache, const float *fresh, int64_t key) {
        const int64_t k = key < ke ? key : ke - 1;
        return k < npre ? cache + k * D : fresh + (k - npre) * nstride;
    };

    f32x4 kf[NC], vf[4][Q4];
    const float *kp;
    const float *vp[4];
    auto point = [&](int t) {                       // this lane's rows of stage t
        const int64_t key0 = (int64_t)t * SK;
        kp = row(kc, kn, key0 + j) + 4 * kg;
#pragma unroll
        for (int e = 0; e < 4; ++e) vp[e] = row(vc, vn, key0 + 4 * kg + e) + MT * j;
    };
    auto kload = [&](int i) { kf[i] = *(const f32x4 *)(kp + 16 * i); };
    auto vload = [&](int e, int h) { vf[e][h] = *(const f32x4 *)(vp[e] + 4 * h); };

    // one stage; `more`: request stage t + NW's pieces as this one's are used up
    auto stage = [&](int t, auto more_tag) {
        constexpr bool more = decltype(more_tag)::value;
        const int64_t key0 = (int64_t)t * SK;
        if constexpr (more) point(t + NW);
        // a score is four chains of D / 4 products, added in pairs: in two chains the
        // longer sums put the outputs of peaked rows up to 1.6 times further off
        float w[NCT][4];
#pragma unroll
        for (int c = 0; c < NCT; ++c) {
            f32x4 s[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) s[e] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int i = 0; i < NC; ++i) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    s[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[i][e], q[c][i][e], s[e], 0, 0, 0);
                if constexpr (more) {
                    if (c == NCT - 1) kload(i);
                }
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) w[c][e] = (s[0][e] + s[1][e]) + (s[2][e] + s[3][e]);
        }
        const bool masked = key0 + SK > k_full;
#pragma unroll
        for (int c = 0; c < NCT; ++c) {
#pragma clang fp contract(off)
            // the product is rounded before m is taken off, so that the largest
            // score's weight is exactly 1 however large the scores are
            float mx = -INFINITY;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float x = w[c][e] * scale;
                w[c][e] = masked && key0 + 4 * kg + e > pos[c] ? -INFINITY : x;
                mx = fmaxf(mx, w[c][e]);
            }
            const float m_new = fmaxf(m_run[c], row_max(mx));
            const float m_use = m_new == -INFINITY ? 0.f : m_new;   // nothing visible so far
            const float alpha = exp_neg(m_run[c] - m_use);
            m_run[c] = m_new;
            float sum = 0.f;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                w[c][e] = exp_neg(w[c][e] - m_use);
                sum += w[c][e];
            }
            if (__ballot(alpha != 1.f)) {
                l_run[c] *= alpha;
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int i = 0; i < 4; ++i) o[c][mt][i] *= alpha;
            }
            l_run[c] += sum;
        }
        if (key0 + SK > ke) {                       // ragged end: no key there (0 * its repeated row)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (key0 + 4 * kg + e >= ke)
#pragma unroll
                    for (int h = 0; h < Q4; ++h) vf[e][h] = (f32x4){0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int c = 0; c < NCT; ++c)
                    o[c][mt] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[e][mt / 4][mt % 4], w[c][e], o[c][mt], 0, 0, 0);
            if constexpr (more) {
#pragma unroll
                for (int h = 0; h < Q4; ++h) vload(e, h);
            }
        }
    };

    if (wave < nst) {
        point(wave);
#pragma unroll
        for (int i = 0; i < NC; ++i) kload(i);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int h = 0; h < Q4; ++h) vload(e, h);
        int t = wave;
        for (; t + NW < nst; t += NW) stage(t, std::true_type{});
        stage(t, std::false_type{});
    }

    // ---- the eight waves' (m, l, O): lane (row j, kg) holds O dims
    // MT (4 kg + i) + mt, posted in pieces of four dims; unit u = (column tile,
    // piece) is summed by wave u % 8 over the waves in order, scaled to the
    // common maximum, and stored
#pragma unroll
    for (int c = 0; c < NCT; ++c) {
        const float l = row_sum(l_run[c]);
        if (kg == 0) {
            mbuf[wave][c][j] = m_run[c];
            lbuf[wave][c][j] = l;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int h = 0; h < Q4; ++h)
                obuf[wave][c * MT + i * Q4 + h][lane] =
                    make_float4(o[c][4 * h][i], o[c][4 * h + 1][i], o[c][4 * h + 2][i], o[c][4 * h + 3][i]);
    }
    __syncthreads();
    for (int u = wave; u < UNITS; u += NW) {
        const int c = u / MT, piece = u % MT;
        float M = -INFINITY;
#pragma unroll
        for (int x = 0; x < NW; ++x) M = fmaxf(M, mbuf[x][c][j]);
        float l = 0.f;
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int x = 0; x < NW; ++x) {
            const float mx = mbuf[x][c][j];
            const float a = mx == -INFINITY ? 0.f : exp_neg(mx - M);   // a wave without keys
            const float4 v = obuf[x][u][lane];
            l = __builtin_fmaf(a, lbuf[x][c][j], l);
            acc[0] = __builtin_fmaf(a, v.x, acc[0]);
            acc[1] = __builtin_fmaf(a, v.y, acc[1]);
            acc[2] = __builtin_fmaf(a, v.z, acc[2]);
            acc[3] = __builtin_fmaf(a, v.w, acc[3]);
        }
        const int r = row0 + 16 * c + j;
        if (r >= R) continue;
        const float inv = 1.f / l;
        float *orow = (float *)p.out + ((int64_t)(tok0 + r / G) * p.n_q_heads + g * G + r % G) * D;
        *(float4 *)(orow + MT * 4 * kg + 4 * piece) = make_float4(acc[0] * inv, acc[1] * inv, acc[2] * inv, acc[3] * inv);
    }
}

template <int D>
hipError_t launch_d(const AttnParams &p, int grid, hipStream_t s) {
    if (p.row_tile == 16) hipLaunchKernelGGL((attn_f32_kernel<D, 1>), dim3(grid), dim3(THREADS), 0, s, p);
    else hipLaunchKernelGGL((attn_f32_kernel<D, 2>), dim3(grid), dim3(THREADS), 0, s, p);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_attn_f32(const AttnParams &p, int head_dim, int grid, hipStream_t s) {
    return head_dim == 128 ? launch_d<128>(p, grid, s) : launch_d<64>(p, grid, s);
}

}  // namespace kvr
