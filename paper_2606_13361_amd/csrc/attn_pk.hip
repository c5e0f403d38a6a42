// attn_pk.hip -- prefill of short documents, 16-bit: the two-group kernel
// (attn_pp.hip) with the keys split between its groups.
//
// A prefill's longest row tile sees every key, and with 256-row tiles a short
// document has fewer of them than the part has compute units: the call takes
// as long as its longest tile.  Here a workgroup is 128 query rows of one kv
// head; both groups (waves 0-3 and 4-7, one wave of each on every SIMD) hold the
// same rows, group A runs the even 64-key tiles and group B the odd ones, and
// the two (m, l, O) meet in LDS at the end.  The tile's steps are those of the
// two-group kernel, written out again for this one's schedule and both head dims,
//   GEMM(t)  O += V_{t-2} P_{t-2}  and  S_t = K_t Q^T
//   SOFT(t)  mask, weights, reference maximum
// one per barrier-separated phase, GEMM(t) in phase t and SOFT(t) in phase t + 1:
// in every phase one group multiplies and the other runs its softmax, as there,
// but a tile takes one phase instead of two.
//
// K and V tiles have rings of four slots each.  In phase t every wave issues its
// share of K(t + 3) and V(t + 1): K(t) is read in phase t, V(t) in phase t + 2, so
// both are issued three phases before their use, into the slots whose last
// readers finished in phase t - 1.  Rows are unpadded with swizzled 16-byte
// chunks (conflict-free K reads and transposing V reads).
//
// What bounds it: the phase (softmax issue and matrix products sharing the
// SIMDs), and per workgroup about 7 us of query rows, first tiles and epilogue;
// a phase moves twice the two-group kernel's bytes from L2 into LDS, and a
// workgroup's fixed time covers half the rows, so long documents stay there.
// Measured against the kernels that served these sizes: 945 tokens (32 / 8 heads,
// d = 128) 30.8 -> 23.3 us, 255 14.9 -> 12.3; 2047 tokens (16 / 2 heads, d = 64)
// 42.8 -> 29.3.  At d = 64 a build for two workgroups per compute unit (128
// registers) spills.
#include <type_traits>

#include "attn_common.hpp"

namespace kvr {
namespace {

using namespace dev;

constexpr int KEYS = 64;
constexpr int NS = 4;                      // ring slots of K, and of V
constexpr int PK_THREADS = 512;

template <int D>
struct Geo {
    static constexpr int ROWB = D * 2;             // bytes of a K/V row
    static constexpr int CH = ROWB / 16;           // its 16-byte chunks: 16 or 8
    static constexpr int TILE = KEYS * ROWB;       // 16 or 8 KB
    static constexpr int LPT = TILE / 8192;        // 1 KB loads per wave and tile: 2 or 1
    static constexpr int RPL = 64 / CH;            // rows of one load: 4 or 8
    static constexpr int MT = D / 32;
    static constexpr int HALF_MT = MT / 2;
    // 16 consecutive rows' chunk c covers every bank once, and so do the four
    // rows x 64 bytes of half a transposing read
    __device__ static __forceinline__ int swz(int row) {
        return D == 128 ? ((row >> 2) & 3) | ((row & 3) << 2) : ((row >> 2) & 3) | (((row >> 1) & 1) << 2);
    }
};

template <class E, int D>
__global__ __launch_bounds__(PK_THREADS) void attn_pk_kernel(const AttnParams p) {
    using T = Geo<D>;
    __shared__ __attribute__((aligned(1024))) unsigned char smem[2 * NS * T::TILE];

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int gw = wave >> 2;                       // group: 0 = A (even tiles), 1 = B
    const int lane = tid & 63;
    const int j = lane & 31;
    const int grp = lane >> 5;

    // ---- work: kv head fastest, longest row tiles first
    const int G = p.group;
    const int g = blockIdx.x % p.n_kv_heads;
    const int tile_lin = p.tiles_total - 1 - blockIdx.x / p.n_kv_heads;
    const int R = G * p.seg_tok0[1];
    const int row0 = tile_lin * kRowsPK;
    const int row_last = min(row0 + kRowsPK, R) - 1;
    const int ke = row_last / G + 1;                // keys any row here may see
    const int n = (ke + KEYS - 1) / KEYS;

    const int wrow0 = row0 + 32 * (wave & 3);
    const int r = wrow0 + j;
    const bool valid = r < R;
    const int tok = valid ? r / G : 0;
    const int head = g * G + (valid ? r % G : 0);
    const int pos = valid ? tok : -1;
    const bool act = wrow0 < R;
    const int k_full = act ? wrow0 / G + 1 : 0;     // keys every row of this wave sees

    u32x4 qf[D / 16];
    {
        const uint16_t *qrow = (const uint16_t *)p.q + ((int64_t)tok * p.n_q_heads + head) * D;
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks)
            qf[ks] = valid ? *(const u32x4 *)(qrow + 16 * ks + 8 * grp) : (u32x4){0, 0, 0, 0};
        if (p.rope && valid) rope_q_frag<E, D>(qf, p.rope + (int64_t)pos * D, grp);
    }

    // ---- loads: wave w moves rows 8w .. 8w + 7 of a K or V tile, RPL rows per
    // instruction; lane -> row, LDS slot lane % CH, global chunk slot ^ swz(row)
    const int64_t nstride_b = p.new_tok_stride * 2;
    const uint64_t kn_a = (uint64_t)(uintptr_t)p.kn + (uint64_t)p.new_head_stride * 2 * g;
    const uint64_t vn_a = (uint64_t)(uintptr_t)p.vn + (uint64_t)p.new_head_stride * 2 * g;
    int lrow[T::LPT];
    uint32_t lchunk[T::LPT], loff[T::LPT];
#pragma unroll
    for (int i = 0; i < T::LPT; ++i) {
        lrow[i] = 8 * wave + T::RPL * i + lane / T::CH;
        lchunk[i] = 16u * (uint32_t)((lane % T::CH) ^ T::swz(lrow[i]));
        loff[i] = (uint32_t)lrow[i] * (uint32_t)nstride_b + lchunk[i];
    }
    // one tile's loads of a step: the base of a whole tile (on = 1); otherwise (no
    // tile left, or the ragged last one, loaded row by row just before) the same
    // instructions run with no lane enabled
    struct Src {
        uint64_t base;
        int lds, on;
    };
    auto lds_of = [&](int v, int t) { return (v * NS + t % NS) * T::TILE + 8 * wave * T::ROWB; };
    auto plan = [&](int v, int t) {
        const uint64_t a = v ? vn_a : kn_a;
        const bool have = t < n, whole = have && (t + 1) * KEYS <= ke;
        if (have && !whole) {
            // rows past the end repeat row ke - 1 (beyond every causal bound, masked)
#pragma unroll
            for (int i = 0; i < T::LPT; ++i) {
                const int key = min(t * KEYS + lrow[i], ke - 1);
                dma16((const void *)(a + (uint64_t)key * (uint64_t)nstride_b + lchunk[i]),
                      smem + lds_of(v, t) + 1024 * i);
            }
        }
        Src f;
        f.base = whole ? a + (uint64_t)t * KEYS * (uint64_t)nstride_b : a;
        f.lds = whole ? lds_of(v, t) : 0;
        f.on = whole ? 1 : 0;
        return f;
    };
    auto issue = [&](const Src &f, int i) { dma16_s_if(f.base, loff[i], smem + f.lds + 1024 * i, f.on); };
    struct Step {
        Src k, v;
    };
    auto plan_step = [&](int phi) {
        Step s;
        s.k = plan(0, phi + 3);
        s.v = plan(1, phi + 1);
        return s;
    };
    auto step_load = [&](const Step &s, int q) {    // loads 0 .. 2 LPT - 1 of a step
        if (q < T::LPT) issue(s.k, q);
        else issue(s.v, q - T::LPT);
    };
    auto load_all = [&](const Step &s) {
#pragma unroll
        for (int q = 0; q < 2 * T::LPT; ++q) step_load(s, q);
    };

    // ---- read maps
    uint32_t ka[D / 16];
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks)
        ka[ks] = (uint32_t)j * T::ROWB + 16u * (uint32_t)((2 * ks + grp) ^ T::swz(j));
    const int l16 = lane & 15;
    const int g16 = lane >> 4;
    uint32_t va[2][T::MT];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int mt = 0; mt < T::MT; ++mt) {
            const int row = 8 * h + 4 * (g16 >> 1) + (l16 >> 2);
            const int chunk = (32 * mt + 16 * (g16 & 1) + 4 * (l16 & 3)) / 8;
            va[h][mt] = (uint32_t)row * T::ROWB + 16u * (uint32_t)(chunk ^ T::swz(row)) + 8u * (uint32_t)(l16 & 1);
        }

    RowState<D> rs;
    rs.zero();
    const float c2 = p.scale_log2;
    f32x16 s[2];
    u32x4 pf[2][2];
#pragma unroll
    for (int st = 0; st < 2; ++st) {
#pragma unroll
        for (int i = 0; i < 16; ++i) s[st][i] = 0.f;
        pf[st][0] = pf[st][1] = (u32x4){0, 0, 0, 0};
    }
    auto kslot = [&](int t) { return smem + (t % NS) * T::TILE; };
    auto vslot = [&](int t) { return smem + (NS + t % NS) * T::TILE; };
    auto kfrag = [&](const unsigned char *b, int st, int ks) {
        return *(const u32x4 *)(b + ka[ks] + 32 * st * T::ROWB);
    };
    auto vfrag = [&](const unsigned char *vs_, int idx) {   // PV product idx = (st, kk, mt)
        const int st = idx / (2 * T::MT), kk = idx / T::MT % 2, mt = idx % T::MT;
        const unsigned char *b = vs_ + (32 * st + 16 * kk) * T::ROWB;
        const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4 *)(b + va[0][mt]));
        const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4 *)(b + va[1][mt]));
        const u32x2 lo2 = __builtin_bit_cast(u32x2, lo);
        const u32x2 hi2 = __builtin_bit_cast(u32x2, hi);
        return (u32x4){lo2[0], lo2[1], hi2[0], hi2[1]};
    };
    auto pv = [&](const u32x4 &a, int idx) {
        const int st = idx / (2 * T::MT), kk = idx / T::MT % 2, mt = idx % T::MT;
        rs.o[mt] = E::mfma(a, pf[st][kk], rs.o[mt]);
    };
    auto s_zero = [&]() {
#pragma unroll
        for (int st = 0; st < 2; ++st)
#pragma unroll
            for (int i = 0; i < 16; ++i) s[st][i] = 0.f;
    };
    auto gemm_s = [&](int t) {                      // the group's first tile
        const unsigned char *kb = kslot(t);
        s_zero();
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks)
#pragma unroll
            for (int st = 0; st < 2; ++st) s[st] = E::mfma(kfrag(kb, st, ks), qf[ks], s[st]);
    };
    auto gemm_pv = [&](int t) {                     // after the group's last tile
        const unsigned char *vb = vslot(t);
#pragma unroll
        for (int idx = 0; idx < 4 * T::MT; ++idx) pv(vfrag(vb, idx), idx);
    };
    constexpr int NCH = D / 16;                     // chunks of 2 S and 2 PV products
    auto gemm = [&](int t, const Step &ld) {
        const unsigned char *kb = kslot(t), *vb = vslot(t - 2);
        s_zero();
        u32x4 k0 = kfrag(kb, 0, 0), k1 = kfrag(kb, 1, 0), v0 = vfrag(vb, 0), v1 = vfrag(vb, 1);
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            u32x4 nk0, nk1, nv0, nv1;
            if (c + 1 < NCH) {
                nk0 = kfrag(kb, 0, c + 1);
                nk1 = kfrag(kb, 1, c + 1);
                nv0 = vfrag(vb, 2 * c + 2);
                nv1 = vfrag(vb, 2 * c + 3);
            }
            s[0] = E::mfma(k0, qf[c], s[0]);
            pv(v0, 2 * c);
            s[1] = E::mfma(k1, qf[c], s[1]);
            pv(v1, 2 * c + 1);
            if (c & 1) step_load(ld, c >> 1);
            __builtin_amdgcn_sched_barrier(0);
            if (c + 1 < NCH) {
                k0 = nk0; k1 = nk1; v0 = nv0; v1 = nv1;
            }
        }
    };
    static_assert(NCH / 2 == 2 * T::LPT, "one load per two chunks");
    // SOFT(t), as in the two-group kernel
    auto soft = [&](int t, const Step &ld) {
        const int k0 = t * KEYS;
        if (k0 + KEYS > k_full) {
            const int lim = max(-1, min(pos - k0, KEYS));
#pragma unroll
            for (int st = 0; st < 2; ++st)
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int o = 32 * st + 8 * (i >> 2) + 4 * grp + (i & 3);
                    s[st][i] = o > lim ? -INFINITY : s[st][i];
                }
        }
        auto exps = [&](auto loads) {
            float lsum[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int st = 0; st < 2; ++st)
#pragma unroll
                for (int i = 0; i < 16; i += 2) {
                    const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[st][i], c2, -rs.m));
                    const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[st][i + 1], c2, -rs.m));
                    lsum[(i >> 1) & 3] += p0 + p1;
                    pf[st][i >> 3][(i & 7) >> 1] = E::pack2(p0, p1);
                    if constexpr (decltype(loads)::value) {
                        constexpr int per = 2 / T::LPT;                  // a load every `per` half sub-tiles
                        const int at = 2 * st + (i >> 3);
                        if ((i & 7) == 6 && at % per == per - 1) step_load(ld, at / per);
                    }
                }
            return (lsum[0] + lsum[1]) + (lsum[2] + lsum[3]);
        };
        float part = exps(std::true_type{});
        if (__ballot(!(part <= kSlackSum) || part > kSignificance * (rs.l + part))) {
            float v[32];
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                v[i] = s[0][i];
                v[16 + i] = s[1][i];
            }
#pragma unroll
            for (int w = 16; w >= 1; w >>= 1)
#pragma unroll
                for (int i = 0; i < w; ++i) v[i] = fmaxf(v[i], v[i + w]);
            const float mx = pair_max(v[0]) * c2;
            const float pmax = __builtin_amdgcn_exp2f(mx - rs.m);
            const bool sig = mx > rs.m && pmax > kSignificance * pair_sum(rs.l + part);
            const bool need = mx > rs.m + (sig ? 0.f : kRescaleSlack);
            if (__ballot(need)) {
                move_reference(rs, need ? mx : rs.m);
                part = exps(std::false_type{});
            }
        }
        rs.l += part;
    };

    // ---- phases 0 .. n + 1.  Phase phi needs K(phi) and V(phi - 2), both issued in
    // phase phi - 3 or before (the prologue counts as phases -3 .. -1): what the
    // two phases before phi issued may still be in flight.  The count below is
    // of the tiles they really loaded (a wave's loads land in issue order).
    constexpr int LPT = T::LPT;
    auto sync = [&](int phi) {
        __builtin_amdgcn_sched_barrier(0);
        if (phi == 0) {
            if (n >= 3) wait_vmcnt<3 * LPT>();      // K(1), K(2), V(0)
            else wait_vmcnt<0>();
        } else if (phi + 2 < n) wait_vmcnt<4 * LPT>();
        else if (phi + 1 < n) wait_vmcnt<3 * LPT>();
        else if (phi < n) wait_vmcnt<2 * LPT>();
        else if (phi == n) wait_vmcnt<LPT>();
        else wait_vmcnt<0>();
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    {
        auto first = [&](int v, int t) {
            const Src f = plan(v, t);
            if (f.on)
#pragma unroll
                for (int i = 0; i < LPT; ++i) issue(f, i);
        };
        first(0, 0);
        if (n > 1) first(0, 1);
        if (n > 2) first(0, 2);
        first(1, 0);
    }
    // one use of the Q fragments: the compiler's wait for their loads lands here
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) asm volatile("" ::"v"(qf[ks]));

    // K/V rows of the workgroup's own tokens (first query row here) into the
    // cache, from the ring: they are the last keys, within the last four tiles
    auto copy_cache = [&]() {
        if (!p.kc_out) return;
        const int own_lo = (row0 + G - 1) / G, own_hi = row_last / G;
        const int n_copy = own_hi >= own_lo ? (own_hi - own_lo + 1) * 2 * T::CH : 0;
        unsigned char *kc = (unsigned char *)p.kc_out + ((int64_t)g * p.cap) * T::ROWB;
        unsigned char *vc = (unsigned char *)p.vc_out + ((int64_t)g * p.cap) * T::ROWB;
        constexpr int NT = PK_THREADS / 2;
        for (int base = tid & (NT - 1); base < n_copy; base += 4 * NT) {
            u32x4 v[4];
            u32x4 *dp[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int idx = min(base + u * NT, n_copy - 1);   // past the end: re-read, not stored
                const int tk = own_lo + idx / (2 * T::CH);
                const int half = idx / T::CH & 1;                 // 0: K row, 1: V row
                const int c = idx % T::CH;
                const int rr = tk & (KEYS - 1);
                v[u] = *(const u32x4 *)((half ? vslot(tk / KEYS) : kslot(tk / KEYS)) + rr * T::ROWB + 16 * (c ^ T::swz(rr)));
                dp[u] = (u32x4 *)((half ? vc : kc) + (int64_t)tk * T::ROWB + 16 * c);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (base + u * NT < n_copy) *dp[u] = v[u];
        }
    };
    auto multiply = [&](auto f) {
        __builtin_amdgcn_s_setprio(1);
        f();
        __builtin_amdgcn_s_setprio(0);
    };
    // phase phi of the group's tile steps; a wave without rows only loads
    if (gw == 1) {                                  // group A has tile 0 meanwhile
        sync(0);
        load_all(plan_step(0));
    }
    int t = gw;
    if (t < n) {
        sync(t);
        if (act) multiply([&]() { gemm_s(t); });
        load_all(plan_step(t));
        sync(t + 1);
        {
            const Step ld = plan_step(t + 1);
            if (act) soft(t, ld);
            else load_all(ld);
        }
        for (t += 2; t < n; t += 2) {
            sync(t);
            {
                const Step ld = plan_step(t);
                if (act) multiply([&]() { gemm(t, ld); });
                else load_all(ld);
            }
            sync(t + 1);
            {
                const Step ld = plan_step(t + 1);
                if (act) soft(t, ld);
                else load_all(ld);
            }
        }
        sync(t);                                    // n or n + 1
        if (act) multiply([&]() { gemm_pv(t - 2); });
    } else {                                        // n = 1: group B has no tile
        sync(1);
    }
    if (t == n) {                                   // the other group's last product is one phase later
        sync(n + 1);
        copy_cache();
    }
    __syncthreads();                                // the rings are no longer read

    // ---- the two groups' (m, l, O) of the same rows: each posts the half of the
    // head dims that the other one finishes, scaled to the larger m and added (A
    // then B), and stores its half of the output rows through LDS
    constexpr int XB = 64 * 16 * 4 * T::HALF_MT;    // bytes a wave posts: 16 HALF_MT floats a lane
    float4 *mine = (float4 *)(smem + wave * XB), *theirs = (float4 *)(smem + (wave ^ 4) * XB);
    float *ml = (float *)(smem + 8 * XB);           // [8 waves][m, l][64 lanes]
    const float l_row = pair_sum(rs.l);
    auto post = [&](int m0) {
#pragma unroll
        for (int mt = 0; mt < T::HALF_MT; ++mt)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4)
                mine[(4 * mt + q4) * 64 + lane] = make_float4(rs.o[m0 + mt][4 * q4], rs.o[m0 + mt][4 * q4 + 1],
                                                              rs.o[m0 + mt][4 * q4 + 2], rs.o[m0 + mt][4 * q4 + 3]);
    };
    if (gw == 0) post(T::HALF_MT);
    else post(0);
    ml[wave * 128 + lane] = rs.m;
    ml[wave * 128 + 64 + lane] = l_row;
    __syncthreads();
    constexpr int OPITCH = T::ROWB / 2 + 16;        // half a row of output
    static_assert(8 * XB + 8 * 128 * 4 + 8 * 32 * OPITCH <= 2 * NS * T::TILE, "merge buffers exceed the rings");
    if (act) {
        const float m1 = ml[(wave ^ 4) * 128 + lane], l1 = ml[(wave ^ 4) * 128 + 64 + lane];
        const float M = fmaxf(rs.m, m1);
        const float a0 = __builtin_amdgcn_exp2f(rs.m - M), a1 = __builtin_amdgcn_exp2f(m1 - M);
        const float l = gw == 0 ? __builtin_fmaf(a1, l1, a0 * l_row) : __builtin_fmaf(a0, l_row, a1 * l1);
        const float inv = l > 0.f ? 1.f / l : 0.f;
        unsigned char *ob = smem + 8 * XB + 8 * 128 * 4 + wave * 32 * OPITCH;
        auto finish = [&](int m0) {
#pragma unroll
            for (int mt = 0; mt < T::HALF_MT; ++mt)
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4) {
                    const float4 x = theirs[(4 * mt + q4) * 64 + lane];
                    const float e[4] = {x.x, x.y, x.z, x.w};
                    float y[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const float o = rs.o[m0 + mt][4 * q4 + i];
                        y[i] = (gw == 0 ? __builtin_fmaf(a1, e[i], a0 * o) : __builtin_fmaf(a0, o, a1 * e[i])) * inv;
                    }
                    u32x2 v;
                    v[0] = E::pack2(y[0], y[1]);
                    v[1] = E::pack2(y[2], y[3]);
                    *(u32x2 *)(ob + j * OPITCH + 2 * (32 * mt + 8 * q4 + 4 * grp)) = v;
                }
        };
        if (gw == 0) finish(0);
        else finish(T::HALF_MT);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // this wave's half rows are in LDS
        constexpr int HC = T::CH / 2;               // chunks of half a row: 8 or 4
        constexpr int RPS = 64 / HC;                // rows of one store
        u32x4 v[32 / RPS];
#pragma unroll
        for (int i = 0; i < 32 / RPS; ++i) v[i] = *(const u32x4 *)(ob + (RPS * i + lane / HC) * OPITCH + 16 * (lane % HC));
#pragma unroll
        for (int i = 0; i < 32 / RPS; ++i) {
            const int rw = wrow0 + RPS * i + lane / HC;
            if (rw < R) {
                uint16_t *orow = (uint16_t *)p.out + ((int64_t)(rw / G) * p.n_q_heads + g * G + rw % G) * D;
                *(u32x4 *)(orow + gw * (D / 2) + 8 * (lane % HC)) = v[i];
            }
        }
    }
}

}  // namespace

hipError_t launch_attn_pk(const AttnParams &p, int head_dim, bool f16, int grid, hipStream_t s) {
    if (head_dim == 128) {
        if (f16) hipLaunchKernelGGL((attn_pk_kernel<F16, 128>), dim3(grid), dim3(PK_THREADS), 0, s, p);
        else hipLaunchKernelGGL((attn_pk_kernel<Bf16, 128>), dim3(grid), dim3(PK_THREADS), 0, s, p);
    } else {
        if (f16) hipLaunchKernelGGL((attn_pk_kernel<F16, 64>), dim3(grid), dim3(PK_THREADS), 0, s, p);
        else hipLaunchKernelGGL((attn_pk_kernel<Bf16, 64>), dim3(grid), dim3(PK_THREADS), 0, s, p);
    }
    return hipGetLastError();
}

}  // namespace kvr
