// Host-only check of the wide batched plans over a grid of shapes: token
// slots, groups, down chunks within the row list, regions in order, and the
// whole plan within the workspace that the shape asks for.
#include <algorithm>
#include <cstdio>

#include "ts_plan.h"

using namespace ts;

static int fail(const char *what, int B, int H, int I, int E) {
    std::printf("FAIL %s B=%d H=%d I=%d E=%d\n", what, B, H, I, E);
    return 1;
}

static const char *check(const BatchPlan &p, int B, int H, int I, size_t limit) {
    if (!p.wide || p.batch != B) return "wide";
    if (p.total > limit) return "workspace";
    if ((long long)p.vpe * p.tok < B || (p.vpe - 1) * p.tok >= B || p.groups != p.experts * p.vpe) return "groups";
    if (p.hpad < H || p.hpad % kBxKQuant || p.ntiles != (I + kBxRows - 1) / kBxRows) return "tiles";
    const int cw = wd_slice_cols(p.tok, p.parts);
    if (p.nslices * cw < H || (p.nslices - 1) * cw >= H) return "slices";
    if (p.tpc < 1 || p.tpc > wd_down_tiles(p.tok, p.parts)) return "down chunk";
    if ((long long)p.nchunks * p.tpc < p.ntiles || (long long)(p.nchunks - 1) * p.tpc >= p.ntiles) return "chunks cover";
    const size_t G = (size_t)p.groups, T = (size_t)p.ntiles, P = (size_t)p.parts;
    const size_t offs[] = {p.off_gcount, p.off_tslot, p.off_xhl, p.off_cnt, p.off_arow, p.off_hfrag,
                           p.off_gmask, p.off_amask, p.off_partial, p.off_union, p.total};
    const size_t need[] = {G * 4, (size_t)B * p.top_k * 8, std::max(G * P * p.tok, (size_t)B * P) * p.hpad * 2,
                           G * T * 8, G * T * kBxRows, G * T * P * p.tok * kBxRows * 2, G * T * p.tok * 4,
                           G * T * p.tok * 4, G * p.tok * (size_t)p.nchunks * H * 4, 16};
    for (int k = 0; k < 10; ++k)
        if (offs[k] % 256 || offs[k] + need[k] > offs[k + 1]) return "regions";
    return nullptr;
}

int main() {
    long taken = 0;
    for (int B = 1; B <= kMaxBatch; B += B < 20 ? 1 : 13)
        for (int H : {8, 200, 1032, 4096, 8192})
            for (int I : {1, 33, 700, 5003, 14336, 100000})
                for (int dc : {0, 1, 64}) {
                    ts_tune_set("down_chunks", dc);
                    BatchPlan p;
                    if (plan_wide_ffn(B, H, I, TS_F32, &p)) return fail("fp32", B, H, I, 1);
                    if (plan_wide_ffn(B, H, I, TS_BF16, &p)) {
                        ++taken;
                        const char *w = check(p, B, H, I, ts_ffn_workspace_bytes(B, H, I, TS_BF16));
                        if (w || B <= kWdMinTokens || p.parts != 2) return fail(w ? w : "ffn", B, H, I, 1);
                    } else if (B > 64 && H == 4096 && I >= 700) return fail("refused", B, H, I, 1);
                    for (int E : {1, 3, 8, 64})
                        for (int K : {1, 2, 8}) {
                            if (K > E || !plan_wide_moe(B, H, I, E, K, TS_BF16, &p)) continue;
                            ++taken;
                            const char *w = check(p, B, H, I, ts_moe_workspace_bytes(B, H, I, E, K, TS_BF16) -
                                                                  2 * align_up256((size_t)B * K * 4));
                            if (w || B <= kBxMaxTokens || p.parts != 3) return fail(w ? w : "moe", B, H, I, E);
                        }
                }
    ts_tune_set("down_chunks", 0);
    if (taken < 1000) return fail("plans taken", (int)taken, 0, 0, 0);
    std::printf("ok\n");
    return 0;
}
