/*
 * Host-side checks of libtileattn's C ABI, built from the library sources
 * compiled for the host only with AddressSanitizer and
 * UndefinedBehaviorSanitizer (tests/test_sanitizers.py builds and runs it on
 * the CPU).  Every entry point is called with fake, 16-byte aligned device
 * addresses and arguments that must fail validation, so nothing is ever
 * dereferenced or launched; the pure host functions (tile schedule, workspace
 * sizes, split heuristics, status strings) run on many shapes.  A status
 * other than the expected one, or any sanitizer report, fails the run.
 */
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include "tileattn.h"

static int failures = 0;

#define EXPECT(cond, ...)                      \
    do {                                       \
        if (!(cond)) {                         \
            fprintf(stderr, "FAIL %s:%d: ", __FILE__, __LINE__); \
            fprintf(stderr, __VA_ARGS__);      \
            fputc('\n', stderr);               \
            ++failures;                        \
        }                                      \
    } while (0)

#define P(x) ((void *)(uintptr_t)(x))

#define BIG 2147483647               /* the largest int */
#define BIG_128 (BIG - 127)          /* the largest multiple of 128 */

/* attn_fwd family: base arguments are valid except where a case changes one */
typedef struct {
    uintptr_t Q, K, V, O, L, ws;
    int B, Hq, Hkv, Sq, Sk, D, causal, splits, o_bf16;
    float scale;
    size_t ws_bytes;
} attn_args;

static attn_args attn_ok(void)
{
    attn_args a = {0x10000000, 0x20000000, 0x30000000, 0x40000000, 0x50000000, 0x60000000,
                   1, 2, 2, 128, 128, 64, 0, 2, 0, 0.125f, 1u << 24};
    return a;
}

/* Every entry point with the arguments of one case (all of them must fail
   validation: the pointers are fake).  split_only: the case concerns an
   argument only the split entry points take, so the others (which would get
   valid arguments) are not called. */
static void attn_case_any(attn_args a, int want, const char *what, int split_only)
{
    int rc;
    if (split_only)
        goto split;
    rc = attn_fwd(P(a.Q), P(a.K), P(a.V), (float *)P(a.O), (float *)P(a.L), a.B, a.Hq, a.Hkv,
                      a.Sq, a.Sk, a.D, a.causal, a.scale, NULL);
    EXPECT(rc == want, "attn_fwd %s: %d want %d", what, rc, want);
    rc = attn_fwd_bf16out(P(a.Q), P(a.K), P(a.V), P(a.O), (float *)P(a.L), a.B, a.Hq, a.Hkv,
                          a.Sq, a.Sk, a.D, a.causal, a.scale, NULL);
    EXPECT(rc == want || (want == TA_ERR_ALIASING), "attn_fwd_bf16out %s: %d want %d", what, rc,
           want);
split:
    rc = attn_fwd_split(P(a.Q), P(a.K), P(a.V), P(a.O), a.o_bf16, (float *)P(a.L), a.B, a.Hq,
                        a.Hkv, a.Sq, a.Sk, a.D, a.causal, a.scale, a.splits, P(a.ws), a.ws_bytes,
                        NULL);
    EXPECT(rc == want, "attn_fwd_split %s: %d want %d", what, rc, want);
    rc = attn_fwd_split_noalloc(P(a.Q), P(a.K), P(a.V), P(a.O), a.o_bf16, (float *)P(a.L), a.B,
                                a.Hq, a.Hkv, a.Sq, a.Sk, a.D, a.causal, a.scale, a.splits, NULL);
    EXPECT(rc == want, "attn_fwd_split_noalloc %s: %d want %d", what, rc, want);
}

static void attn_case(attn_args a, int want, const char *what)
{
    attn_case_any(a, want, what, 0);
}

static void check_attn_validation(void)
{
    attn_args a;
#define CASE(field, value, want) \
    a = attn_ok();               \
    a.field = value;             \
    attn_case(a, want, #field "=" #value)
    CASE(Q, 0, TA_ERR_NULL_POINTER);
    CASE(K, 0, TA_ERR_NULL_POINTER);
    CASE(V, 0, TA_ERR_NULL_POINTER);
    CASE(O, 0, TA_ERR_NULL_POINTER);
    CASE(L, 0, TA_ERR_NULL_POINTER);
    CASE(B, 0, TA_ERR_INVALID_SHAPE);
    CASE(Hq, 0, TA_ERR_INVALID_SHAPE);
    CASE(Hkv, -1, TA_ERR_INVALID_SHAPE);
    CASE(Sq, 0, TA_ERR_INVALID_SHAPE);
    CASE(Sk, -7, TA_ERR_INVALID_SHAPE);
    CASE(Hkv, 3, TA_ERR_INVALID_SHAPE);
    CASE(Sq, 1 << 25, TA_ERR_INVALID_SHAPE);
    a = attn_ok();
    a.splits = 0;
    attn_case_any(a, TA_ERR_INVALID_SHAPE, "splits=0", 1);
    a.splits = 129;
    attn_case_any(a, TA_ERR_INVALID_SHAPE, "splits=129", 1);
    CASE(D, 96, TA_ERR_UNSUPPORTED);
    CASE(D, 256, TA_ERR_UNSUPPORTED);
    CASE(Q, 0x10000008, TA_ERR_MISALIGNED);
    CASE(O, 0x40000004, TA_ERR_MISALIGNED);
    CASE(L, 0x50000004, TA_ERR_MISALIGNED);
    CASE(scale, -0.5f, TA_ERR_INVALID_SCALE);
    CASE(scale, 1.0f / 0.0f, TA_ERR_INVALID_SCALE);
    CASE(O, 0x10000000 + 16, TA_ERR_ALIASING);
    CASE(L, 0x20000000 + 64, TA_ERR_ALIASING);
#undef CASE
    a = attn_ok();
    a.causal = 1;
    a.Sq = 129;
    attn_case(a, TA_ERR_INVALID_SHAPE, "causal Sq > Sk");
    /* workspace errors only concern attn_fwd_split */
    a = attn_ok();
    a.ws = 0;
    EXPECT(attn_fwd_split(P(a.Q), P(a.K), P(a.V), P(a.O), 0, (float *)P(a.L), a.B, a.Hq, a.Hkv,
                          a.Sq, a.Sk, a.D, 0, a.scale, 2, NULL, 1u << 24, NULL) == TA_ERR_WORKSPACE,
           "split without workspace");
    EXPECT(attn_fwd_split(P(a.Q), P(a.K), P(a.V), P(a.O), 0, (float *)P(a.L), a.B, a.Hq, a.Hkv,
                          a.Sq, a.Sk, a.D, 0, a.scale, 2, P(0x60000000), 1000, NULL) ==
               TA_ERR_WORKSPACE,
           "split with a small workspace");
    /* partial results beyond the static scratch */
    EXPECT(attn_fwd_split_noalloc(P(0x10000000), P(0x20000000), P(0x30000000), P(0x40000000), 0,
                                  (float *)P(0x50000000), 1, 32, 32, 4096, 4096, 128, 0, 0.1f, 2,
                                  NULL) == TA_ERR_SCRATCH,
           "noalloc beyond the scratch");
}

/* ta_schedule against a brute-force count of visible and masked pairs */
static void check_schedule(void)
{
    int bm, bn;
    EXPECT(ta_tile_shape(128, &bm, &bn) == TA_OK, "tile shape");
    EXPECT(ta_tile_shape(96, &bm, &bn) == TA_ERR_UNSUPPORTED, "tile shape D=96");
    EXPECT(ta_tile_shape(64, NULL, &bn) == TA_ERR_NULL_POINTER, "tile shape null");
    ta_tile_shape(64, &bm, &bn);
    const int sizes[] = {1, 2, 37, 63, 64, 65, 127, 128, 129, 200, 300, 511, 1000};
    const int ns = (int)(sizeof sizes / sizeof sizes[0]);
    for (int x = 0; x < ns; ++x)
        for (int y = 0; y < ns; ++y)
            for (int causal = 0; causal < 2; ++causal) {
                const int Sq = sizes[x], Sk = sizes[y];
                int n, fm;
                if (causal && Sq > Sk) {
                    EXPECT(ta_schedule(Sq, Sk, 64, causal, 0, &n, &fm) == TA_ERR_INVALID_SHAPE,
                           "schedule rejects causal Sq > Sk");
                    continue;
                }
                const int n_qt = (Sq + bm - 1) / bm;
                for (int qt = 0; qt < n_qt; ++qt) {
                    EXPECT(ta_schedule(Sq, Sk, 64, causal, qt, &n, &fm) == TA_OK, "schedule ok");
                    const int n_tiles = (Sk + bn - 1) / bn;
                    int last_vis = -1, first_mask = n_tiles;
                    for (int t = 0; t < n_tiles; ++t) {
                        int vis = 0, masked = 0;
                        for (int i = qt * bm; i < qt * bm + bm && i < Sq; ++i)
                            for (int j = t * bn; j < t * bn + bn; ++j) {
                                const int ok = j < Sk && (!causal || j <= i + Sk - Sq);
                                vis |= ok;
                                masked |= !ok;
                            }
                        if (vis)
                            last_vis = t;
                        if (masked && t < first_mask)
                            first_mask = t;
                    }
                    EXPECT(n == last_vis + 1, "n_kv %d want %d (Sq %d Sk %d qt %d)", n,
                           last_vis + 1, Sq, Sk, qt);
                    EXPECT(fm <= n && (fm == n || fm >= first_mask) && fm <= first_mask + 0 + n,
                           "first_masked %d (Sq %d Sk %d qt %d)", fm, Sq, Sk, qt);
                    EXPECT(fm == (first_mask < n ? first_mask : n),
                           "first_masked %d want %d (Sq %d Sk %d qt %d)", fm,
                           first_mask < n ? first_mask : n, Sq, Sk, qt);
                }
                EXPECT(ta_schedule(Sq, Sk, 64, causal, n_qt, &n, &fm) == TA_ERR_INVALID_SHAPE,
                       "schedule rejects a query tile past the end");
            }
}

static void check_host_helpers(void)
{
    size_t bytes = 0;
    EXPECT(ta_split_workspace_bytes(2, 3, 100, 128, 4, &bytes) == TA_OK &&
               bytes == (size_t)4 * 2 * 3 * 100 * 129 * 4,
           "split workspace bytes");
    EXPECT(ta_split_workspace_bytes(2, 3, 100, 128, 1, &bytes) == TA_OK && bytes == 0,
           "one split needs no workspace");
    EXPECT(ta_split_workspace_bytes(2, 3, 100, 128, 0, &bytes) == TA_ERR_INVALID_SHAPE,
           "zero splits");
    const int shapes[][6] = {{1, 32, 32, 512, 512, 128},   {1, 32, 32, 1024, 1024, 128},
                             {8, 32, 32, 2048, 2048, 128}, {1, 32, 8, 1024, 8192, 128},
                             {1, 1, 1, 1, 1, 64},           {1, 2, 2, 128, 100000, 64}};
    for (size_t i = 0; i < sizeof shapes / sizeof shapes[0]; ++i) {
        int n = 0;
        for (int causal = 0; causal < 2; ++causal) {
            const int *s = shapes[i];
            const int rc = ta_split_heuristic(s[0], s[1], s[2], s[3], s[4], s[5], causal, &n);
            EXPECT(rc == (causal && s[3] > s[4] ? TA_ERR_INVALID_SHAPE : TA_OK),
                   "split heuristic status");
            if (rc == TA_OK)
                EXPECT(n >= 1 && n <= 128, "split heuristic range %d", n);
        }
    }
    EXPECT(mla_workspace_bytes(64, 128, 4, &bytes) == TA_OK &&
               bytes == (size_t)4 * 64 * 128 * 513 * 4,
           "mla workspace");
    int n = 0;
    EXPECT(mla_split_heuristic(64, 128, 1, 8192, &n) == TA_OK && n >= 1 && n <= 128,
           "mla heuristic");
    for (int s = 0; s < 12; ++s)
        EXPECT(ta_status_string((ta_status)s) && strlen(ta_status_string((ta_status)s)) > 0,
               "status string %d", s);
    EXPECT(ta_version() >= 400, "version");
}

static void check_other_validation(void)
{
    /* mla_decode */
    EXPECT(mla_decode(P(0x10000000), P(0x18000000), P(0x20000000), P(0x30000000),
                      (float *)P(0x40000000), (float *)P(0x50000000), 2, 128, 1, 256, 256, 64,
                      0.04f, 2, P(0x60000000), 1u << 24, NULL) == TA_ERR_UNSUPPORTED,
           "mla Dl");
    EXPECT(mla_decode(NULL, P(0x18000000), P(0x20000000), P(0x30000000), (float *)P(0x40000000),
                      (float *)P(0x50000000), 2, 128, 1, 256, 512, 64, 0.04f, 2, P(0x60000000),
                      1u << 24, NULL) == TA_ERR_NULL_POINTER,
           "mla null");
    EXPECT(mla_decode(P(0x10000000), P(0x18000000), P(0x20000000), P(0x30000000),
                      (float *)P(0x40000000), (float *)P(0x50000000), 2, 128, 1, 256, 512, 64,
                      0.04f, 2, NULL, 0, NULL) == TA_ERR_WORKSPACE,
           "mla workspace");
    /* gemm_bf16 */
    EXPECT(gemm_bf16(P(0x10000000), P(0x30000000), P(0x50000000), 0, 200, 256, 128, NULL) ==
               TA_ERR_UNSUPPORTED,
           "gemm M");
    EXPECT(gemm_bf16(P(0x10000000), P(0x30000000), P(0x10000000 + 1024), 0, 256, 256, 128,
                     NULL) == TA_ERR_ALIASING,
           "gemm aliasing");
    EXPECT(gemm_bf16(P(0x10000000), P(0x30000000), P(0x50000000), 0, 256, 65536, 16384, NULL) ==
               TA_ERR_INVALID_SHAPE,
           "gemm 32-bit offsets");
    /* gemv_bf16_split */
    EXPECT(gemv_bf16_split(P(0x10000000), P(0x30000000), P(0x50000000), 0, 256, 128, 2, NULL, 0, NULL) ==
               TA_ERR_WORKSPACE,
           "gemv without workspace");
    EXPECT(gemv_bf16_split(P(0x10000000), P(0x30000000), P(0x50000000), 0, 100, 128, 2,
                           P(0x60000000), 1u << 20, NULL) == TA_ERR_UNSUPPORTED,
           "gemv N");
    EXPECT(gemv_bf16_split(P(0x10000000), P(0x30000000), P(0x30000000), 0, BIG - 63, BIG - 7, 2,
                           P(0x60000000), 1u << 20, NULL) == TA_ERR_ALIASING,
           "gemv aliasing, the largest sizes");
    /* SSD */
    EXPECT(ssd_chunk_scan(P(0x10000000), P(0x12000000), (const float *)P(0x20000000),
                          (const float *)P(0x13000000), (const float *)P(0x14000000),
                          (const float *)P(0x30000000), (const float *)P(0x15000000),
                          (float *)P(0x40000000), 1, 300, 4, 2, 128, 128, 256, NULL) ==
               TA_ERR_UNSUPPORTED,
           "ssd scan headdim");
    EXPECT(ssd_chunk_state(P(0x10000000), P(0x11000000), (const float *)P(0x13000000),
                           (const float *)P(0x14000000), (float *)P(0x11000000 + 4096), 1, 300,
                           4, 2, 64, 128, 256, NULL) == TA_ERR_ALIASING,
           "ssd state aliasing");
    EXPECT(ssd_bmm_chunk(P(0x12000000), P(0x11000000), NULL, 1, 300, 2, 128, 256, NULL) ==
               TA_ERR_NULL_POINTER,
           "ssd bmm null");
    EXPECT(ssd_state_passing((const float *)P(0x30000000), (const float *)P(0x13000000),
                             (const float *)P(0x14000000), (float *)P(0x30000000 + 1024), NULL, 1,
                             300, 4, 64, 128, 256, NULL) == TA_ERR_ALIASING,
           "ssd passing aliasing");
}

/* gemm_bf16_split and ssd_forward: one argument of a valid call changed */
static void check_split_gemm_and_forward(void)
{
    typedef struct { uintptr_t A, B, C, ws; int M, N, K, splits; size_t ws_bytes; } G;
    const G g0 = {0x10000000, 0x30000000, 0x50000000, 0x70000000, 256, 256, 256, 3,
                  (size_t)3 * 256 * 256 * 4};
    G g;
#define GEMM(field, value, want)                                                                    \
    g = g0;                                                                                         \
    g.field = value;                                                                                \
    EXPECT(gemm_bf16_split(P(g.A), P(g.B), P(g.C), 1, g.M, g.N, g.K, g.splits, P(g.ws), g.ws_bytes, \
                           NULL) == want,                                                           \
           "gemm split " #field "=" #value)
    GEMM(B, 0, TA_ERR_NULL_POINTER);
    GEMM(M, 0, TA_ERR_INVALID_SHAPE);
    GEMM(splits, 65, TA_ERR_INVALID_SHAPE);
    GEMM(splits, 5, TA_ERR_UNSUPPORTED);
    GEMM(M, 200, TA_ERR_UNSUPPORTED);
    GEMM(M, BIG, TA_ERR_UNSUPPORTED);
    GEMM(N, BIG_128, TA_ERR_INVALID_SHAPE);
    GEMM(K, BIG_128, TA_ERR_INVALID_SHAPE);
    GEMM(A, 0x10000008, TA_ERR_MISALIGNED);
    GEMM(ws, 0x10000000, TA_ERR_ALIASING);
    GEMM(ws, 0, TA_ERR_WORKSPACE);
    GEMM(ws_bytes, 1000, TA_ERR_WORKSPACE);
#undef GEMM
    typedef struct { uintptr_t x, Bm, Cm, dt, A, D, out, fin, ws; int b, L, H, G, hd, ds, seg; size_t ws_bytes; } S;
    const S s0 = {0x10000000, 0x11000000, 0x12000000, 0x13000000, 0x14000000, 0x15000000, 0x40000000,
                  0x30000000, 0x20000000, 1, 300, 4, 2, 64, 128, 2, 1u << 20};
    S s;
#define SSD(field, value, want)                                                                  \
    s = s0;                                                                                      \
    s.field = value;                                                                             \
    EXPECT(ssd_forward(P(s.x), P(s.Bm), P(s.Cm), (const float *)P(s.dt), (const float *)P(s.A),  \
                       (const float *)P(s.D), (float *)P(s.out), (float *)P(s.fin), s.b, s.L,    \
                       s.H, s.G, s.hd, s.ds, s.seg, P(s.ws), s.ws_bytes, NULL) == want,          \
           "ssd forward " #field "=" #value)
    SSD(x, 0, TA_ERR_NULL_POINTER);
    SSD(L, 0, TA_ERR_INVALID_SHAPE);
    SSD(seg, 65, TA_ERR_INVALID_SHAPE);
    SSD(b, BIG, TA_ERR_INVALID_SHAPE);
    SSD(L, BIG, TA_ERR_INVALID_SHAPE);
    SSD(H, BIG - 1, TA_ERR_INVALID_SHAPE);
    SSD(hd, 32, TA_ERR_UNSUPPORTED);
    SSD(fin, 0x30000004, TA_ERR_MISALIGNED);
    SSD(out, 0x10000000, TA_ERR_ALIASING);
    SSD(ws, 0, TA_ERR_WORKSPACE);
#undef SSD
    s = s0;
    s.b = s.L = s.H = s.G = BIG;
    EXPECT(ssd_forward(P(s.x), P(s.Bm), P(s.Cm), (const float *)P(s.dt), (const float *)P(s.A), NULL,
                       (float *)P(s.out), NULL, s.b, s.L, s.H, s.G, s.hd, s.ds, 64, P(s.ws),
                       s.ws_bytes, NULL) == TA_ERR_INVALID_SHAPE,
           "ssd forward, every size the largest");
}

/* The host helpers over all pairs of ordinary and extreme sizes: a status and
   a value in range, no overflow on the way */
static void check_extreme_sizes(void)
{
    const int v[] = {-1, 0, 1, 2, 16, 127, 128, 4096, 8191, 1 << 20, 1 << 24, BIG_128, BIG - 1, BIG};
    const int nv = (int)(sizeof v / sizeof v[0]);
    for (int i = 0; i < nv; ++i)
        for (int j = 0; j < nv; ++j)
            for (int k = 0; k < nv; ++k) {
                const int a = v[i], b = v[j], c = v[k];
                int n = 0, ok;
                size_t bytes = 0;
                for (int D = 64; D <= 128; D += 64)
                    for (int g = 1; g <= 3; g += 2) {
                        /* (g query heads per key/value head where that fits) */
                        const int hq = b > 0 && b <= BIG / g ? b * g : b;
                        ok = ta_split_heuristic(a, hq, b, 1, c, D, 0, &n);
                        EXPECT(ok != TA_OK || (n >= 1 && n <= 128), "split heuristic %d %d %d", a, b, c);
                        ok = ta_split_plan(a, hq, b, 1, c, D, 0, &n);
                        EXPECT(ok != TA_OK || (n >= 1 && n <= 128), "split plan %d %d %d", a, b, c);
                        ok = ta_decode_route(a, hq, b, 1, c, D, 128, &n);
                        EXPECT(ok != TA_OK || n == 0 || n == 1, "decode route %d %d %d", a, b, c);
                        ok = ta_decode_route(a, hq, b, c, c, D, 1, &n);
                        EXPECT(ok != TA_OK || n == 0 || n == 1, "decode route %d %d %d", a, b, c);
                    }
                ok = mla_split_heuristic(a, b, b, c, &n);
                EXPECT(ok != TA_OK || (n >= 1 && n <= 128), "mla heuristic %d %d %d", a, b, c);
                ok = mla_split_plan(a, b, b, c, &n);
                EXPECT(ok != TA_OK || (n >= 1 && n <= 128), "mla plan %d %d %d", a, b, c);
                ok = mla_split_plan(a, b, 1, c, &n);
                EXPECT(ok != TA_OK || (n >= 1 && n <= 128), "mla plan, one latent head %d %d %d", a, b, c);
                ok = gemm_split_heuristic(a, b, c, &n);
                EXPECT(ok != TA_OK || (n >= 1 && n <= 64), "gemm heuristic %d %d %d", a, b, c);
                ok = gemm_split_workspace_bytes(a, b, 64, &bytes);
                EXPECT(ok == (a > 0 && b > 0 ? TA_OK : TA_ERR_INVALID_SHAPE), "gemm workspace %d %d", a, b);
                ok = gemv_split_workspace_bytes(a, 7, &bytes);
                EXPECT(ok == (a > 0 ? TA_OK : TA_ERR_INVALID_SHAPE), "gemv workspace %d", a);
                ok = mla_workspace_bytes(a, b, 128, &bytes);
                EXPECT(ok == (a > 0 && b > 0 ? TA_OK : TA_ERR_INVALID_SHAPE), "mla workspace %d %d", a, b);
                ok = ta_split_workspace_bytes(a, b, c, 128, 128, &bytes);
                EXPECT(ok == (a > 0 && b > 0 && c > 0 ? TA_OK : TA_ERR_INVALID_SHAPE),
                       "split workspace %d %d %d", a, b, c);
                ok = gemv_split_heuristic(a, b, &n);
                EXPECT(ok != TA_OK || (n >= 1 && n <= 64), "gemv heuristic %d %d", a, b);
                ok = ssd_segment_heuristic(a, b, c, &n);
                EXPECT(ok != TA_OK || (n >= 1 && n <= 64), "segments %d %d %d", a, b, c);
                ok = ssd_forward_workspace_bytes(a, b, c, 64, &bytes);
                EXPECT(ok == (a > 0 && b > 0 && c > 0 ? TA_OK : TA_ERR_INVALID_SHAPE),
                       "ssd workspace %d %d %d", a, b, c);
            }
    int n;
    EXPECT(ta_split_plan(8, 32, 8, 1, 8191, 128, 0, NULL) == TA_ERR_NULL_POINTER, "plan null");
    EXPECT(ta_decode_route(8, 32, 8, 1, 8191, 128, 1, NULL) == TA_ERR_NULL_POINTER, "route null");
    EXPECT(ta_decode_route(8, 32, 8, 1, 8191, 96, 1, &n) == TA_ERR_UNSUPPORTED, "route D");
    EXPECT(mla_split_plan(8, 32, 3, 64, &n) == TA_ERR_INVALID_SHAPE, "mla plan heads");
}

int main(void)
{
    check_split_gemm_and_forward();
    check_extreme_sizes();
    check_attn_validation();
    check_schedule();
    check_host_helpers();
    check_other_validation();
    if (failures) {
        fprintf(stderr, "%d check(s) failed\n", failures);
        return 1;
    }
    printf("abi_driver: all checks passed\n");
    return 0;
}
