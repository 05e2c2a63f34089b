// Limits of the host planner (make_plan, plain C++, no device), for a build
// with AddressSanitizer and UndefinedBehaviorSanitizer: with a cap on the
// workspace (the static scratch) default host blocks fit it whenever one
// segment does, and a caller's own tiling is bounded and sized by what the
// caller gave, not by the default segment length.
#include <stdio.h>
#include <string.h>

#include <initializer_list>

#include "../../paper_2512_23068_amd/csrc/pgf_plan.h"

static int failures = 0;

static pgf_params sizes(int64_t B, int64_t D, int64_t N, int64_t K, int order = 1) {
    pgf_params p;
    memset(&p, 0, sizeof(p));
    p.batch = B; p.seqlen = 131072; p.d_inner = D; p.d_state = N; p.n_dirs = K; p.order = order;
    return p;
}

static void fail(const char *what, const pgf_params &p) {
    printf("%s: order %d B %ld D %ld N %ld K %ld seg %d chunk_segs %d\n", what, p.order, (long)p.batch,
           (long)p.d_inner, (long)p.d_state, (long)p.n_dirs, p.seg_len, p.chunk_segs);
    ++failures;
}

int main() {
    long fitted = 0;
    for (int order : {1, 2, 3})
        for (int64_t B : {1, 3, 128})
            for (int64_t D : {1, 16, 77, 128, 1000, 1536, 2048, 5120, 8192, 65536})
                for (int64_t N : {4, 8, 16, 32, 64})
                    for (int64_t K : {1, 2, 4, 8})
                        for (int seg : {0, 16, 32, 128, 256, 1024})
                            for (int var = 0; var < 4; ++var)
                                for (size_t cap : {(size_t)PGF_SCRATCH_BYTES, (size_t)64 << 20}) {
                                    pgf_params p = sizes(B, D, N, K, order);
                                    p.seg_len = seg;
                                    p.delta_flows = order == 3 && K == 2;
                                    p.A_im = var == 1 ? (const float *)16 : nullptr;   // tested for NULL only
                                    p.dt_rank = var == 2 ? 48 : 0;
                                    p.in_dtype = var == 3;
                                    pgf::Plan q;
                                    if (pgf::make_plan(&p, &q, cap) != PGF_OK || q.seg == 0) continue;
                                    if (q.ws.total <= cap) {
                                        ++fitted;
                                        continue;
                                    }
                                    // only where a single segment does not fit either
                                    p.chunk_segs = 1;
                                    pgf::Plan one;
                                    if (pgf::make_plan(&p, &one, cap) == PGF_OK && one.ws.total <= cap) {
                                        p.chunk_segs = 0;
                                        fail("default block beyond the cap", p);
                                    }
                                }
    // chunk_segs beside the default segment length is bounded as 256-step
    // segments of D channels: 2^30 elements
    for (int64_t D : {1024, 1025, 1536, 2048})
        for (int64_t N : {4, 16})
            for (int dt = 0; dt < 2; ++dt) {
                pgf_params p = sizes(1, D, N, 1);
                p.in_dtype = dt;
                p.chunk_segs = 4096;
                pgf::Plan q;
                const int want = D <= 1024 ? PGF_OK : PGF_ERR_INVALID_ARG;
                if (pgf::make_plan(&p, &q) != want) fail("bound of chunk_segs", p);
            }
    // a given segment length: three rounds of 1024 resident blocks, as whole
    // rounds, within 512 MiB and 4096 segments
    const struct { int64_t B, D, N, K; int seg, segs; } given[] = {
        {1, 1, 4, 1, 16, 3072}, {1, 1536, 16, 1, 64, 512}, {1, 1536, 16, 1, 128, 512}, {1, 1536, 16, 1, 256, 512},
        {1, 77, 16, 8, 16, 1536}, {2, 1000, 16, 1, 32, 384}, {3, 77, 16, 1, 128, 1024},
    };
    for (const auto &c : given) {
        pgf_params p = sizes(c.B, c.D, c.N, c.K);
        p.seg_len = c.seg;
        pgf::Plan q;
        if (pgf::make_plan(&p, &q) != PGF_OK || q.chunk_segs != c.segs || q.chunk_len != (int64_t)c.segs * c.seg) {
            printf("(%d segments) ", q.chunk_segs);
            fail("block of a given segment length", p);
        }
    }
    // linear attention: a given chunk_segs beside the default segment length is
    // bounded as 128-step segments (2^30 elements), sequential blocks where
    // blocks of 4096 state entries fill the GPU, and cut where the chosen
    // length is longer; a given length keeps three rounds of those blocks
    const struct { int64_t H, DK, DV; int seg, segs, rc; int64_t len; } la[] = {
        {1, 16, 64, 0, 4096, PGF_OK, 4096 * 64},    {1, 16, 2048, 0, 4096, PGF_OK, 524288},
        {1, 16, 4096, 0, 4096, PGF_ERR_INVALID_ARG, 0}, {2, 16, 4096, 0, 1024, PGF_OK, 262144},
        {6, 16, 4096, 0, 256, PGF_OK, 262144},      {64, 16, 4096, 0, 64, PGF_OK, 262144},
        {64, 16, 4096, 0, 65, PGF_ERR_INVALID_ARG, 0}, {256, 64, 64, 0, 4, PGF_OK, 16384},
        {1, 16, 64, 16, 0, PGF_OK, 3072 * 16},      {32, 64, 64, 128, 0, PGF_OK, 96 * 128},
        {8, 16, 128, 64, 0, PGF_OK, 768 * 64},      {1, 64, 64, 16, 4096, PGF_OK, 4096 * 16},
    };
    for (const auto &c : la) {
        pgf_la_params p;
        memset(&p, 0, sizeof(p));
        p.batch = 1; p.heads = c.H; p.seqlen = 131072; p.d_key = c.DK; p.d_value = c.DV; p.n_dirs = 1;
        p.seg_len = c.seg; p.chunk_segs = c.segs;
        pgf::LaPlan q;
        const int rc = pgf::make_la_plan(&p, &q);
        if (rc != c.rc || (rc == PGF_OK && q.chunk_len != c.len)) {
            printf("linear attention: H %ld DK %ld DV %ld seg %d chunk_segs %d: rc %d block %ld\n", (long)c.H,
                   (long)c.DK, (long)c.DV, c.seg, c.segs, rc, rc == PGF_OK ? (long)q.chunk_len : 0L);
            ++failures;
        }
    }
    printf("%ld plans fit their cap, %d failures\n", fitted, failures);
    return failures ? 1 : 0;
}
