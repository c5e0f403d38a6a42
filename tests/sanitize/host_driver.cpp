// Drives the host side of libkvr (kvr_api.hip, artifact.hip: argument
// validation, split planning, workspace layouts, artifact headers) under
// AddressSanitizer and UndefinedBehaviorSanitizer, without a GPU.  The kernel
// launchers are replaced by stubs that count their calls and fail, so a call
// with valid arguments ends in KVR_ERR_DEVICE without touching a device; a
// rejected call must reach no launcher at all.  Device pointers are fake
// aligned integers and are never dereferenced on the host.
#include <math.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>

#include <vector>

#include "kvr.h"
#include "kvr_internal.hpp"

static int g_launches = 0;
static int64_t g_nsplit = -1, g_chunk = -1;   // the split plan the last continuation launch got
static int g_pp_bad = 0;                       // many-readers launches whose plan broke an invariant
static int g_pp_split = 0, g_pp_whole = 0;     // many-readers launches checked: split last round or not
static int64_t g_pp_grid = -1, g_pp_tail0 = -1, g_pp_rows = -1;

static int g_long = 0, g_long_bad = 0, g_long_split = 0;   // long continuations on the two-group kernel
static size_t g_ws_given = (size_t)1 << 60;                // workspace bytes of the running call, where they are checked
static char g_kernel = 0;                                  // the last attention launch: 's'taged, 'p' two-group, 'k'ey-split
static int g_pre = 0, g_pre_bad = 0;                       // 16-bit prefills whose tiles were checked

namespace kvr {
// a prefill's row tiles cover its rows, and the grid its tiles and kv heads
static void check_prefill(const AttnParams &p, int64_t tile, int grid, char kernel) {
    const int64_t rows = (int64_t)p.group * p.seg_tok0[1], tiles = (rows + tile - 1) / tile;
    if (p.n_seg != 1 || p.seg_tok0[0] != 0 || p.tiles_total != tiles || (int64_t)grid != tiles * p.n_kv_heads) {
        ++g_pre_bad;
        fprintf(stderr, "prefill plan: kernel %c heads %d/%d rows %ld tiles %d grid %d\n", kernel, p.n_q_heads, p.n_kv_heads,
                (long)rows, p.tiles_total, grid);
    }
    ++g_pre;
    g_kernel = kernel;
}
hipError_t launch_attn_bf16(const AttnParams &p, int head_dim, int mode, bool, int grid, hipStream_t) {
    ++g_launches;
    if (mode == kModePrefill) {
        check_prefill(p, kRowsBf16, grid, 's');
        if (head_dim != 64) ++g_pre_bad;
    } else if (mode == kModeContinue) g_kernel = 's';
    return hipErrorUnknown;
}
hipError_t launch_attn_pk(const AttnParams &p, int, bool, int grid, hipStream_t) {
    ++g_launches; check_prefill(p, kRowsPK, grid, 'k'); return hipErrorUnknown;
}
hipError_t launch_merge_bf16(const MergeParams &, int, bool, hipStream_t) { ++g_launches; return hipErrorUnknown; }
// many readers on the two-group kernel: the packed plan must cover its tiles
// with whole workgroups (split tiles ns times), and split partial rows must
// number the rows from the first split tile to the end of the launch
hipError_t launch_attn_pp(const AttnParams &p, int mode, bool, int grid, hipStream_t) {
    ++g_launches;
    if (mode == kModeReaders) {
        const int64_t ns = p.nsplit, tiles = p.tiles_total, t0 = p.tail_tile0;
        const int64_t rows = (int64_t)p.group * ((int64_t)p.seg_tok0[p.n_seg] - p.seg_tok0[0]);
        bool ok = ns >= 1 && ns <= 16 && t0 >= 0 && t0 <= tiles && tiles == (rows + kRowsPP - 1) / kRowsPP &&
                  (int64_t)grid == (t0 + (tiles - t0) * ns) * p.n_kv_heads;
        if (ns > 1) ok = ok && t0 < tiles && p.ws && p.rows_total == rows - t0 * kRowsPP && kRowsPP % p.group == 0;
        else ok = ok && t0 == tiles;
        if (!ok) ++g_pp_bad;
        ++(ns > 1 ? g_pp_split : g_pp_whole);
        g_pp_grid = grid; g_pp_tail0 = t0; g_pp_rows = p.rows_total;
    } else if (mode == kModeContinue) {
        // one reader: every tile whole, or every tile in nsplit shares of at least one
        // key tile, whose partials fit the workspace of the call; 32-bit products
        const int64_t ns = p.nsplit, tiles = p.tiles_total, rows = (int64_t)p.group * p.seg_tok0[1];
        const int64_t key_tiles = (p.n_prefix + p.seg_tok0[1] + kKeyTile - 1) / kKeyTile;
        bool ok = p.n_seg == 1 && p.seg_tok0[0] == 0 && tiles == (rows + kRowsPP - 1) / kRowsPP && ns >= 1 &&
                  ns <= kMaxSplits && ns <= p.n_prefix / kKeyTile && ns * key_tiles <= 0x7fffffff &&
                  p.tail_tile0 == (ns > 1 ? 0 : tiles) && (int64_t)grid == tiles * ns * p.n_kv_heads && rows > kContMaxRows;
        if (ns > 1) ok = ok && p.ws && p.rows_total == rows && (size_t)ns * p.n_kv_heads * rows * 130 * 4 <= g_ws_given;
        if (!ok) { ++g_long_bad; fprintf(stderr, "long plan: heads %d/%d rows %ld prefix %ld splits %ld tiles %ld given %zu\n", p.n_q_heads, p.n_kv_heads, (long)rows, (long)p.n_prefix, (long)ns, (long)tiles, g_ws_given); }
        ++g_long;
        g_long_split += ns > 1;
        g_kernel = 'p';
    } else {
        check_prefill(p, kRowsPP, grid, 'p');
    }
    return hipErrorUnknown;
}
hipError_t launch_attn_rows(const AttnParams &p, bool, int, hipStream_t) {
    ++g_launches; g_nsplit = p.nsplit; g_chunk = p.chunk; return hipErrorUnknown;
}
hipError_t launch_attn_cont(const AttnParams &p, int, bool, bool, int, hipStream_t) {
    ++g_launches; g_nsplit = p.nsplit; g_chunk = p.chunk; return hipErrorUnknown;
}
hipError_t launch_quantize(const QuantParams &, hipStream_t) { ++g_launches; return hipErrorUnknown; }
hipError_t launch_attn_f32(const AttnParams &, int, int, hipStream_t) { ++g_launches; return hipErrorUnknown; }
hipError_t launch_append(const AppendParams &, hipStream_t) { ++g_launches; return hipErrorUnknown; }
hipError_t launch_rope(const RopeParams &, int, int, hipStream_t) { ++g_launches; return hipErrorUnknown; }
hipError_t launch_rope_table(float *, int, double, int64_t, hipStream_t) { ++g_launches; return hipErrorUnknown; }
}  // namespace kvr

static void *const A = (void *)(uintptr_t)0x10000;    // 16-byte aligned fake device pointer
static void *const MIS = (void *)(uintptr_t)0x10008;  // 8-byte aligned only
static const float *const AF = (const float *)A;
static int fails = 0;

#define EXPECT(expr, want)                                                                              \
    do {                                                                                                \
        const int before_ = g_launches;                                                                 \
        const int got_ = (int)(expr);                                                                   \
        if (got_ != (want)) {                                                                           \
            fprintf(stderr, "line %d: %s = %d, want %d\n", __LINE__, #expr, got_, (int)(want));       \
            ++fails;                                                                                    \
        }                                                                                               \
        if ((want) != KVR_OK && (want) != KVR_ERR_DEVICE && g_launches != before_) {                    \
            fprintf(stderr, "line %d: %s launched after a rejection\n", __LINE__, #expr);              \
            ++fails;                                                                                    \
        }                                                                                               \
    } while (0)

static kvr_desc desc(int hq = 32, int hkv = 8, int d = 128, int dt = KVR_BF16, int64_t cap = 4096) {
    kvr_desc x;
    memset(&x, 0, sizeof x);
    x.n_q_heads = hq; x.n_kv_heads = hkv; x.head_dim = d; x.dtype = dt; x.capacity = cap; x.scale = 0.f;
    return x;
}

static uint64_t rng = 0x2545f4914f6cdd1dull;
static uint64_t next() { rng ^= rng << 13; rng ^= rng >> 7; rng ^= rng << 17; return rng; }
static int64_t pick(const int64_t *v, int n) { return v[next() % (uint64_t)n]; }

static void fixed_cases() {
    kvr_desc d = desc();
    const size_t big = (size_t)1 << 40;
    // descriptors
    EXPECT(kvr_prefill(nullptr, A, A, A, 4, A, A, A, nullptr), KVR_ERR_NULL);
    kvr_desc bad = desc(); bad.dtype = 7;
    EXPECT(kvr_prefill(&bad, A, A, A, 4, A, A, A, nullptr), KVR_ERR_DTYPE);
    bad = desc(); bad.n_q_heads = 30;
    EXPECT(kvr_continue(&bad, A, A, A, A, A, 8, 4, A, A, big, nullptr), KVR_ERR_SHAPE);
    bad = desc(); bad.head_dim = 96;
    EXPECT(kvr_cache_append(&bad, A, A, 4, A, A, 0, nullptr), KVR_ERR_SHAPE);
    bad = desc(); bad.reserved = 1;
    EXPECT(kvr_prefill(&bad, A, A, A, 4, A, A, A, nullptr), KVR_ERR_SHAPE);
    bad = desc(); bad.scale = NAN;
    EXPECT(kvr_prefill(&bad, A, A, A, 4, A, A, A, nullptr), KVR_ERR_SHAPE);
    bad = desc(); bad.capacity = -1;
    EXPECT(kvr_prefill(&bad, A, A, A, 4, A, A, A, nullptr), KVR_ERR_SHAPE);
    // lengths, capacity, pointers, alignment
    EXPECT(kvr_prefill(&d, A, A, A, -1, A, A, A, nullptr), KVR_ERR_SHAPE);
    EXPECT(kvr_prefill(&d, A, A, A, 4097, A, A, A, nullptr), KVR_ERR_CAPACITY);
    EXPECT(kvr_prefill(&d, nullptr, nullptr, nullptr, 0, nullptr, nullptr, nullptr, nullptr), KVR_OK);
    EXPECT(kvr_prefill(&d, MIS, A, A, 4, A, A, A, nullptr), KVR_ERR_ALIGN);
    EXPECT(kvr_prefill(&d, A, A, A, 4, A, nullptr, A, nullptr), KVR_ERR_NULL);
    EXPECT(kvr_continue(&d, A, A, A, A, A, -1, 4, A, A, big, nullptr), KVR_ERR_SHAPE);
    EXPECT(kvr_continue(&d, A, A, A, A, A, 4097, 4, A, A, big, nullptr), KVR_ERR_CAPACITY);
    EXPECT(kvr_continue(&d, nullptr, nullptr, nullptr, A, A, 8, 0, nullptr, nullptr, 0, nullptr), KVR_OK);
    const size_t need = kvr_workspace_bytes(&d, 4096, 24, 1);
    EXPECT(need > 0, 1);
    EXPECT(kvr_continue(&d, A, A, A, A, A, 4096, 24, A, A, need - 1, nullptr), KVR_ERR_WORKSPACE);
    EXPECT(kvr_continue(&d, A, A, A, A, A, 4096, 24, A, nullptr, need, nullptr), KVR_ERR_NULL);
    EXPECT(kvr_continue(&d, A, A, A, A, A, 4096, 24, A, MIS, need, nullptr), KVR_ERR_ALIGN);
    EXPECT(kvr_continue(&d, A, A, A, A, A, 4096, 24, A, A, need, nullptr), KVR_ERR_DEVICE);   // reaches a stub
    EXPECT(kvr_continue_append(&d, A, A, A, A, A, 4090, 24, A, A, big, nullptr), KVR_ERR_CAPACITY);
    EXPECT(kvr_cache_append(&d, A, A, 10, A, A, 4090, nullptr), KVR_ERR_CAPACITY);
    EXPECT(kvr_cache_append(&d, A, A, -1, A, A, 0, nullptr), KVR_ERR_SHAPE);
    // readers: cu_seqlens checks
    const int32_t cu_ok[4] = {0, 5, 5, 12}, cu_dec[3] = {0, 7, 3}, cu_first[3] = {2, 4, 6};
    EXPECT(kvr_continue_batched(&d, A, A, A, cu_dec, 2, A, A, 100, A, A, big, nullptr), KVR_ERR_SHAPE);
    EXPECT(kvr_continue_batched(&d, A, A, A, cu_first, 2, A, A, 100, A, A, big, nullptr), KVR_ERR_SHAPE);
    EXPECT(kvr_continue_batched(&d, A, A, A, nullptr, 3, A, A, 100, A, A, big, nullptr), KVR_ERR_NULL);
    EXPECT(kvr_continue_batched(&d, A, A, A, cu_ok, 3, A, A, 5000, A, A, big, nullptr), KVR_ERR_CAPACITY);
    EXPECT(kvr_continue_batched(&d, A, A, A, cu_ok, 3, A, A, 100, A, A, big, nullptr), KVR_ERR_DEVICE);
    {
        // 64 readers, 8424 tokens over 3774: 132 tiles per kv head, the last 4 split 8 ways
        std::vector<int32_t> cu64(65, 0);
        const int step[4] = {120, 140, 131, 135};
        for (int i = 1; i <= 64; ++i) cu64[i] = cu64[i - 1] + step[i % 4];
        cu64[64] = 8424;
        kvr_desc dr = desc(32, 8, 128, KVR_BF16, 4096);
        const size_t wsr = kvr_workspace_bytes(&dr, 3774, 8424, 64);
        EXPECT(wsr == (size_t)8 * 8 * 928 * 130 * 4, 1);
        EXPECT(kvr_continue_batched(&dr, A, A, A, cu64.data(), 64, A, A, 3774, A, A, wsr - 1, nullptr),
               KVR_ERR_WORKSPACE);
        EXPECT(kvr_continue_batched(&dr, A, A, A, cu64.data(), 64, A, A, 3774, A, A, wsr, nullptr), KVR_ERR_DEVICE);
        EXPECT(g_pp_grid == (128 + 4 * 8) * 8 * 1 && g_pp_tail0 == 128 && g_pp_rows == 928, 1);
    }
    // int8 artifact
    kvr_desc f32 = desc(32, 8, 128, KVR_F32);
    EXPECT(kvr_quantize_cache(&f32, A, A, 10, A, A, (float *)A, nullptr), KVR_ERR_DTYPE);
    EXPECT(kvr_continue_q8(&d, A, A, A, A, A, nullptr, 100, 4, A, A, big, nullptr), KVR_ERR_NULL);
    // RoPE
    kvr_rope r;
    r.cos_sin = AF; r.n_pos = 64;
    EXPECT(kvr_rope_table(96, 1e6, 10, (float *)A, nullptr), KVR_ERR_SHAPE);
    EXPECT(kvr_rope_table(128, -1.0, 10, (float *)A, nullptr), KVR_ERR_POSITION);
    EXPECT(kvr_prefill_rope(&d, &r, A, A, A, 65, A, A, A, nullptr), KVR_ERR_POSITION);
    EXPECT(kvr_continue_rope(&d, &r, A, A, A, A, A, 60, 8, 1, A, A, big, nullptr), KVR_ERR_POSITION);
    EXPECT(kvr_continue_rope(&d, nullptr, A, A, A, A, A, 60, 4, 1, A, A, big, nullptr), KVR_ERR_NULL);
    EXPECT(kvr_continue_batched_rope(&d, &r, A, A, A, cu_ok, 3, A, A, 60, A, A, big, nullptr), KVR_ERR_POSITION);
    EXPECT(kvr_rope_apply(&d, &r, A, 4, 0, 0, A, nullptr), KVR_ERR_SHAPE);
    // artifact: header round trip with L = 0 (no copies), then every corrupted field
    std::vector<unsigned char> host(KVR_ARTIFACT_HEADER_BYTES + 64);
    const void *kcs[2] = {A, A};
    void *kcd[2] = {A, A};
    int64_t L_out = -5;
    EXPECT(kvr_artifact_save(&d, "qwen3-4b", 2, 0, kcs, kcs, host.data(), host.size(), nullptr), KVR_OK);
    EXPECT(kvr_artifact_load(&d, "qwen3-4b", 2, host.data(), host.size(), kcd, kcd, &L_out, nullptr), KVR_OK);
    EXPECT(L_out == 0, 1);
    EXPECT(kvr_artifact_load(&d, "qwen3-8b", 2, host.data(), host.size(), kcd, kcd, &L_out, nullptr),
           KVR_ERR_MISMATCH);
    EXPECT(kvr_artifact_load(&d, "qwen3-4b", 3, host.data(), host.size(), kcd, kcd, &L_out, nullptr),
           KVR_ERR_MISMATCH);
    EXPECT(kvr_artifact_load(&d, "qwen3-4b", 2, host.data(), KVR_ARTIFACT_HEADER_BYTES - 1, kcd, kcd, &L_out,
                             nullptr),
           KVR_ERR_WORKSPACE);
    char long_id[200];
    memset(long_id, 'x', sizeof long_id - 1);
    long_id[sizeof long_id - 1] = 0;
    EXPECT(kvr_artifact_save(&d, long_id, 2, 0, kcs, kcs, host.data(), host.size(), nullptr), KVR_ERR_SHAPE);
    for (size_t off = 0; off < KVR_ARTIFACT_HEADER_BYTES; ++off) {
        std::vector<unsigned char> h2(host);
        h2[off] ^= 0x5a;
        const int st = kvr_artifact_load(&d, "qwen3-4b", 2, h2.data(), h2.size(), kcd, kcd, &L_out, nullptr);
        // the reserved tail of the header is ignored; every other byte is checked
        if (st != KVR_OK && st != KVR_ERR_MISMATCH && st != KVR_ERR_CAPACITY && st != KVR_ERR_WORKSPACE) {
            fprintf(stderr, "corrupted header byte %zu: status %d\n", off, st);
            ++fails;
        }
    }
}

// Random descriptors, lengths and reader tables through every entry point:
// whatever the status, the sanitizers watch the host arithmetic.
static void fuzz() {
    const int heads[] = {1, 2, 3, 4, 8, 16, 32, 64, 4096, 5000, 0, -3};
    const int dims[] = {64, 128, 96, 0};
    const int64_t caps[] = {0, 1, 64, 4096, 40000, 1LL << 20, (int64_t)1 << 31, -1};
    const int64_t lens[] = {0, 1, 2, 31, 32, 33, 63, 64, 65, 96, 255, 3774, 32768, 1LL << 20, (int64_t)1 << 31,
                            (int64_t)1 << 40, -1, -7};
    for (int it = 0; it < 20000; ++it) {
        kvr_desc d = desc();
        d.n_kv_heads = heads[next() % 12];
        d.n_q_heads = d.n_kv_heads * (int)(1 + next() % 8);
        if (next() % 8 == 0) d.n_q_heads = heads[next() % 12];
        d.head_dim = dims[next() % 4];
        d.dtype = (int)(next() % 4);
        d.capacity = pick(caps, 8);
        const int64_t Lp = pick(lens, 18), S = pick(lens, 18);
        const int32_t n = (int32_t)(next() % 140);
        std::vector<int32_t> cu(n + 1);
        cu[0] = 0;
        for (int32_t i = 1; i <= n; ++i) cu[i] = cu[i - 1] + (int32_t)(next() % 300);
        if (n > 0 && next() % 16 == 0) cu[next() % (n + 1)] = -(int32_t)(next() % 5);
        const size_t ws = kvr_workspace_bytes(&d, Lp, S, 1);
        const size_t wsn = kvr_workspace_bytes(&d, Lp, n > 0 ? cu[n] : 0, n);
        const size_t wsr = kvr_workspace_bytes_rope(&d, Lp, S, 1);
        const size_t wsrn = kvr_workspace_bytes_rope(&d, Lp, n > 0 ? cu[n] : 0, n);
        const size_t big = (size_t)1 << 50;
        kvr_rope r;
        r.cos_sin = AF;
        r.n_pos = pick(lens, 18);
        (void)kvr_prefill(&d, A, A, A, Lp, A, A, A, nullptr);
        (void)kvr_continue(&d, A, A, A, A, A, Lp, S, A, A, next() % 2 ? ws : big, nullptr);
        (void)kvr_continue_append(&d, A, A, A, A, A, Lp, S, A, A, ws, nullptr);
        (void)kvr_continue_batched(&d, A, A, A, cu.data(), n, A, A, Lp, A, A, wsn, nullptr);
        (void)kvr_cache_append(&d, A, A, S, A, A, Lp, nullptr);
        (void)kvr_q8_bytes(&d);
        (void)kvr_quantize_cache(&d, A, A, Lp, A, A, (float *)A, nullptr);
        (void)kvr_continue_q8(&d, A, A, A, A, A, AF, Lp, S, A, A, ws, nullptr);
        (void)kvr_prefill_rope(&d, &r, A, A, A, Lp, A, A, A, nullptr);
        (void)kvr_continue_rope(&d, &r, A, A, A, A, A, Lp, S, (int32_t)(next() % 2), A, A, wsr, nullptr);
        (void)kvr_continue_batched_rope(&d, &r, A, A, A, cu.data(), n, A, A, Lp, A, A, wsrn, nullptr);
        (void)kvr_rope_apply(&d, &r, A, S, (int32_t)(next() % 40) - 2, Lp, A, nullptr);
        (void)kvr_artifact_bytes(&d, (int32_t)(next() % 40) - 2, Lp);
    }
}

// The split plan of the continuation, as the kernels receive it: splits of
// whole 64-key tiles, no more splits than 256-key pieces of the prefix, the
// last one non-empty and
// ending at the prefix end -- or, for a prefix at most 32 - S keys past a
// multiple of the split count x 128 keys, chunks of a multiple of 128 keys
// whose last split also takes the few remaining keys.
static void split_plans() {
    const int64_t cap = 40200;
    kvr_desc e = desc(32, 8, 128, KVR_BF16, cap);
    void *P = (void *)(uintptr_t)0x100000;
    const int64_t lens[] = {256, 300, 1000, 3774, 4096, 8191, 16384, 16387, 16400, 32768, 32769, 32775,
                            32790, 32799, 32800, 32900, 40000};
    const int64_t sfx[] = {1, 2, 8, 12, 24, 31, 32, 33, 64, 96};
    int planned = 0;
    for (int64_t L : lens)
        for (int64_t S : sfx) {
            if (L + S > cap) continue;
            const size_t ws = kvr_workspace_bytes(&e, L, S, 1);
            g_nsplit = g_chunk = -1;
            const int st = kvr_continue(&e, P, P, P, P, P, L, S, P, P, ws, nullptr);
            if (st != KVR_ERR_DEVICE) { fprintf(stderr, "plan L=%ld S=%ld: status %d\n", (long)L, (long)S, st); ++fails; continue; }
            if (g_nsplit <= 1) continue;
            ++planned;
            const int64_t n = g_nsplit, c = g_chunk;
            const bool tiles = c % 64 == 0 && n <= (L + 255) / 256 && (n - 1) * c < L;
            const bool covers = n * c >= L || (c % 128 == 0 && L - n * c + S <= 32);
            if (!tiles || !covers) {
                fprintf(stderr, "plan L=%ld S=%ld: %ld splits of %ld keys\n", (long)L, (long)S, (long)n, (long)c);
                ++fails;
            }
        }
    if (planned < 50) { fprintf(stderr, "only %d split plans checked\n", planned); ++fails; }
}

// Continuations of more than 96 rows per kv head, over head counts, lengths and
// token counts: the plans' invariants (checked in the stubs), and the route of calls
// that measured clearly faster on one kernel.
static void long_plans() {
    void *P = (void *)(uintptr_t)0x100000;
    const int heads[][2] = {{32, 8}, {8, 8}, {12, 3}, {64, 8}, {16, 16}, {32, 32}, {4, 1}, {16, 2}, {40, 8}, {28, 4}, {5, 5}, {96, 1}};
    const int64_t lens[] = {1, 255, 256, 300, 1000, 4000, 16000, 32000, 200000, ((int64_t)1 << 29) - 500, (int64_t)1 << 29,
                            ((int64_t)1 << 30) - 100, (int64_t)1 << 31};
    const int64_t rows[] = {97, 128, 129, 256, 257, 600, 1024, 2047, 2048, 2049, 5000, 20000};
    for (const auto &h : heads)
        for (int64_t L : lens)
            for (int64_t r : rows)
                for (int dt : {KVR_BF16, KVR_F16}) {
                    const kvr_desc d = desc(h[0], h[1], 128, dt, (int64_t)1 << 32);
                    const int64_t S = (r * h[1] + h[0] - 1) / h[0];
                    g_ws_given = kvr_workspace_bytes(&d, L, S, 1);
                    EXPECT(kvr_continue(&d, P, P, P, P, P, L, S, P, P, g_ws_given, nullptr), KVR_ERR_DEVICE);
                    g_ws_given = kvr_workspace_bytes(&d, L, S, 1);
                    if (g_ws_given <= KVR_NOALLOC_SCRATCH_BYTES && g_ws_given == 0)   // no device scratch needed
                        EXPECT(kvr_continue_noalloc(&d, P, P, P, P, P, L, S, P, nullptr), KVR_ERR_DEVICE);
                }
    struct Route { int hq, hkv; int64_t L, S; char want; };
    const Route routes[] = {
        // us staged, two-group
        {4, 1, 300, 512, 's'},      // 24.9, 31.1
        {4, 1, 16000, 64, 's'},     // 24.2, 28.9
        {16, 2, 1000, 256, 's'},    // 23.6, 29.9
        {12, 1, 16384, 24, 's'},    // 21.4, 26.3
        {12, 3, 16000, 48, 's'},    // 28.0, 30.7
        {32, 8, 4000, 100, 's'},    // 25.6, 28.2
        {32, 8, 300, 64, 's'},      // 14.3, 20.0
        {32, 8, 64, 600, 's'},      // 22.5, 25.6
        {32, 8, 7001, 517, 'p'},    // 128.9, 87.6
        {32, 8, 20000, 300, 'p'},   // 187.2, 116.0
        {32, 8, 2000, 500, 'p'},    // 51.3, 44.7
        {32, 8, 1000, 1024, 'p'},   // 74.2, 60.5
        {8, 8, 4000, 768, 'p'},     // 58.5, 38.3
        {4, 1, 20000, 1500, 'p'},   // 150.9, 80.2
        {4, 1, 8297, 161, 's'},     // 21.8, 25.0
        {8, 8, 953, 517, 's'},      // 28.8, 31.3
        {12, 3, 1643, 385, 's'},    // 29.7, 31.8
        {16, 2, 8789, 111, 's'},    // 28.4, 30.6
        {4, 1, 32763, 122, 's'},    // 32.3, 33.7
        {32, 8, 459, 660, 'p'},     // 48.2, 39.0
        {32, 8, 8497, 156, 's'},    // 40.8, 45.0
        {64, 8, 17504, 66, 's'},    // 62.5, 65.8
        {32, 8, 3221, 143, 'p'},    // 36.1, 31.7
    };
    for (const Route &r : routes) {
        const kvr_desc d = desc(r.hq, r.hkv, 128, KVR_BF16, 40000);
        g_kernel = 0;
        g_ws_given = kvr_workspace_bytes(&d, r.L, r.S, 1);
        EXPECT(kvr_continue(&d, P, P, P, P, P, r.L, r.S, P, P, g_ws_given, nullptr), KVR_ERR_DEVICE);
        if (g_kernel != r.want) {
            fprintf(stderr, "%d/%d heads, %ld over %ld: kernel %c, want %c\n", r.hq, r.hkv, (long)r.S, (long)r.L, g_kernel, r.want);
            ++fails;
        }
    }
    g_ws_given = (size_t)1 << 60;
    if (g_long_bad) { fprintf(stderr, "%d long continuations broke a plan invariant\n", g_long_bad); ++fails; }
    if (g_long_split < 200 || g_long - g_long_split < 100) {
        fprintf(stderr, "only %d split and %d whole long plans checked\n", g_long_split, g_long - g_long_split);
        ++fails;
    }
}

// 16-bit prefills over head counts and lengths: the tiles of the kernel they run on
// (checked in the stubs), and the route of calls that measured faster on one kernel.
static void prefill_plans() {
    void *P = (void *)(uintptr_t)0x100000;
    const int heads[][2] = {{32, 8}, {8, 8}, {12, 3}, {64, 8}, {128, 8}, {512, 8}, {4, 1}, {16, 2}, {5, 5}, {96, 1}, {14, 2}};
    const int64_t lens[] = {1, 2, 31, 33, 64, 65, 127, 129, 255, 257, 449, 513, 600, 945, 1200, 1473, 2047, 2049, 4097, 9000, 40000};
    int seen[3] = {0, 0, 0};
    for (const auto &h : heads)
        for (int64_t L : lens)
            for (int hd : {64, 128})
                for (int dt : {KVR_BF16, KVR_F16}) {
                    const kvr_desc d = desc(h[0], h[1], hd, dt, L);
                    g_kernel = 0;
                    EXPECT(kvr_prefill(&d, P, P, P, L, P, P, P, nullptr), KVR_ERR_DEVICE);
                    if (g_kernel == (hd == 64 ? 's' : 'p')) ++seen[hd == 64];
                    else if (g_kernel == 'k') ++seen[2];
                    else { fprintf(stderr, "prefill %d/%d d=%d L=%ld: kernel %c\n", h[0], h[1], hd, (long)L, g_kernel); ++fails; }
                }
    struct Route { int hq, hkv, hd; int64_t L; char want; };
    const Route routes[] = {
        // us whole tiles, key-split
        {32, 8, 64, 29, 's'},       // 4.8, 6.0
        {32, 32, 64, 157, 's'},     // 7.0, 7.9
        {128, 8, 64, 247, 's'},     // 8.8, 9.8
        {64, 8, 64, 321, 's'},      // 9.8, 10.3
        {16, 2, 64, 600, 'k'},      // 14.7, 13.7
        {16, 2, 64, 2047, 'k'},     // 42.8, 29.3
        {64, 8, 64, 1000, 's'},     // 25.1, 26.1
        {32, 8, 128, 1, 'p'},       // 5.0, 6.1
        {16, 16, 128, 20, 'p'},     // 5.5, 6.5
        {1024, 64, 128, 7, 'p'},    // 7.8, 8.1
        {32, 8, 128, 50, 'k'},      // 8.7, 8.1
        {16, 16, 128, 125, 'k'},    // 11.5, 10.9
        {128, 8, 128, 317, 'p'},    // 17.1, 18.2
        {512, 8, 128, 77, 'p'},     // 12.2, 16.4
        {256, 8, 128, 173, 'p'},    // 13.9, 17.8
        {96, 8, 128, 466, 'p'},     // 21.3, 22.1
        {128, 8, 128, 251, 'k'},    // 15.1, 13.4
        {80, 8, 128, 457, 'k'},     // 21.0, 18.4
        {64, 8, 128, 701, 'k'},     // 25.6, 23.8
        {32, 8, 128, 945, 'k'},     // 30.8, 23.3
        {32, 8, 128, 1797, 'k'},    // 49.9, 44.4
        {64, 8, 128, 900, 'p'},     // 35.6, 36.8
    };
    for (const Route &r : routes) {
        const kvr_desc d = desc(r.hq, r.hkv, r.hd, KVR_BF16, r.L);
        g_kernel = 0;
        EXPECT(kvr_prefill(&d, P, P, P, r.L, P, P, P, nullptr), KVR_ERR_DEVICE);
        if (g_kernel != r.want) {
            fprintf(stderr, "prefill %d/%d d=%d L=%ld: kernel %c, want %c\n", r.hq, r.hkv, r.hd, (long)r.L, g_kernel, r.want);
            ++fails;
        }
    }
    if (g_pre_bad || g_pre < 900) { fprintf(stderr, "%d of %d prefills broke a plan invariant\n", g_pre_bad, g_pre); ++fails; }
    if (seen[0] < 50 || seen[1] < 50 || seen[2] < 50) { fprintf(stderr, "prefill kernels seen: %d %d %d\n", seen[0], seen[1], seen[2]); ++fails; }
}

int main() {
    if (kvr_abi_version() != KVR_ABI_VERSION) {
        fprintf(stderr, "ABI version mismatch\n");
        return 1;
    }
    for (int s = -1; s < 12; ++s)
        if (!kvr_strerror(s) || !kvr_strerror(s)[0]) ++fails;
    fixed_cases();
    split_plans();
    long_plans();
    prefill_plans();
    fuzz();
    if (g_pp_bad) {
        fprintf(stderr, "%d many-readers launches broke a plan invariant\n", g_pp_bad);
        ++fails;
    }
    if (g_pp_split < 20 || g_pp_whole < 20) {
        fprintf(stderr, "only %d split and %d whole many-readers plans checked\n", g_pp_split, g_pp_whole);
        ++fails;
    }
    if (fails) {
        fprintf(stderr, "%d checks failed\n", fails);
        return 1;
    }
    printf("host driver: all checks passed (%d stub launches; many-readers plans: %d split, %d whole)\n", g_launches,
           g_pp_split, g_pp_whole);
    return 0;
}
