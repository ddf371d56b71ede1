// Host-only check of the wide and the fp32-exact batched plans over a grid of
// shapes: token slots, groups, down chunks within the row list, regions in
// order, and the whole plan within the workspace that the shape asks for;
// shapes that have to be taken; both sides of the size rule's lines.
#include <algorithm>
#include <cstdio>
#include <initializer_list>

#include "ts_plan.h"

using namespace ts;

static int fail(const char *what, int B, int H, int I, int E) {
    std::printf("FAIL %s B=%d H=%d I=%d E=%d\n", what, B, H, I, E);
    return 1;
}

// Regions in order and large enough, tiles and chunks covering.
static const char *check(const BatchPlan &p, int B, int H, int I, size_t limit, int slice_cols, int max_tiles) {
    if (p.batch != B || p.hidden != H || p.inter != I) return "sizes";
    if (p.total > limit) return "workspace";
    if ((long long)p.vpe * p.tok < B || (p.vpe - 1) * p.tok >= B || p.groups != p.experts * p.vpe) return "groups";
    if (p.bpad != p.tok || p.ntiles != (I + kBxRows - 1) / kBxRows) return "tiles";
    const bool f32 = p.mode == kBxF32;
    const int quant = f32 ? kBxKQuant / 2 : kBxKQuant;
    if (p.hpad < H || p.hpad % quant || p.hpad - H >= quant) return "hidden padding";
    if (p.parts != (p.mode == kBxBf16x3 ? 3 : 2)) return "parts";  // (an fp32 value takes the room of two)
    if (p.nslices * slice_cols < H || (p.nslices - 1) * slice_cols >= H) return "slices";
    if (p.tpc < 1 || p.tpc > max_tiles) return "down chunk";
    if ((long long)p.nchunks * p.tpc < p.ntiles || (long long)(p.nchunks - 1) * p.tpc >= p.ntiles) return "chunks cover";
    const size_t G = (size_t)p.groups, T = (size_t)p.ntiles, P = (size_t)p.parts;
    // bytes of x as the kernels read it: per group, k-step of 64 bytes of a row and 1 KB fragment (router's split:
    // per token), packed three-part operands in two fragments
    const size_t nks = (size_t)p.hpad * (f32 ? 4 : 2) / 64;
    const size_t nx = f32 ? p.tok / 16 : (p.tok == 8 ? (P + 1) / 2 : P * p.tok / 16);
    const size_t offs[] = {p.off_gcount, p.off_tslot, p.off_xhl, p.off_cnt, p.off_arow, p.off_hfrag,
                           p.off_gmask, p.off_amask, p.off_partial, p.off_union, p.total};
    const size_t need[] = {G * 4, (size_t)B * p.top_k * 8, std::max(G * nks * nx * 1024, (size_t)B * P * p.hpad * 2),
                           G * T * 8, G * T * kBxRows, G * T * P * p.tok * kBxRows * 2, G * T * p.tok * 4,
                           G * T * p.tok * 4, G * p.tok * (size_t)p.nchunks * H * 4, 16};
    for (int k = 0; k < 10; ++k)
        if (offs[k] % 256 || offs[k] + need[k] > offs[k + 1]) return "regions";
    return nullptr;
}

static const char *check_wide(const BatchPlan &p, int B, int H, int I, size_t limit) {
    if (!p.wide || p.rows) return "wide";
    if (p.vpe > 1 && p.experts == 1 && !wd_many_groups(p.tok, p.parts)) return "several groups";
    return check(p, B, H, I, limit, wd_slice_cols(p.tok, p.parts), wd_down_tiles(p.tok, p.parts));
}

static const char *check_exact(const BatchPlan &p, int B, int H, int I, size_t limit, ts_dtype dt) {
    if (p.mode != (dt == TS_F32 ? kBxF32 : kBxBf16x3)) return "mode";
    if (p.rows != (dt == TS_F32 && p.experts == 1 && p.top_k == 1 && B <= kRowsMaxTokens)) return "row streams";
    if (p.wide) return dt == TS_BF16 && p.experts == 1 && p.tok == 64 ? check_wide(p, B, H, I, limit) : "wide";
    if (dt == TS_F32 ? p.tok != 16 && p.tok != 32 : p.tok != 8 && p.tok != 16) return "slots";
    return check(p, B, H, I, limit, kBxSliceCols, bx_down_tiles(p.tok));
}

static size_t moe_limit(int B, int H, int I, int E, int K, ts_dtype dt) {
    return ts_moe_workspace_bytes(B, H, I, E, K, dt) - 2 * align_up256((size_t)B * K * 4);
}

int main() {
    long ffn = 0, moe = 0, exact = 0;
    for (int B = 1; B <= kMaxBatch; B += B < 20 ? 1 : 13)
        for (int H : {8, 200, 1032, 4096, 8192})
            for (int I : {1, 33, 700, 5003, 14336, 100000})
                for (int dc : {0, 1, 64}) {
                    ts_tune_set("down_chunks", dc);
                    BatchPlan p;
                    if (plan_wide_ffn(B, H, I, TS_F32, &p)) return fail("fp32", B, H, I, 1);
                    if (plan_wide_ffn(B, H, I, TS_BF16, &p)) {
                        ++ffn;
                        const char *w = check_wide(p, B, H, I, ts_ffn_workspace_bytes(B, H, I, TS_BF16));
                        if (w || B <= kWdMinTokens || p.parts != 2) return fail(w ? w : "ffn", B, H, I, 1);
                    } else if (B > 64 && H == 4096 && I >= 700) return fail("refused", B, H, I, 1);
                    for (int E : {1, 3, 8, 64})
                        for (int K : {1, 2, 8}) {
                            if (K > E) continue;
                            if (plan_wide_moe(B, H, I, E, K, TS_BF16, &p)) {
                                ++moe;
                                const char *w = check_wide(p, B, H, I, moe_limit(B, H, I, E, K, TS_BF16));
                                if (w || B <= kBxMaxTokens || p.parts != 3) return fail(w ? w : "moe", B, H, I, E);
                            }
                            if (H <= 4096 && plan_exact(B, H, I, E, K, TS_F32, moe_limit(B, H, I, E, K, TS_F32), &p)) {
                                ++exact;
                                const char *w = check_exact(p, B, H, I, moe_limit(B, H, I, E, K, TS_F32), TS_F32);
                                if (w || B < 2) return fail(w ? w : "exact moe", B, H, I, E);
                            }
                        }
                    for (ts_dtype dt : {TS_F32, TS_BF16}) {
                        const size_t limit = ts_ffn_workspace_bytes(B, H, I, dt);
                        if (!plan_exact(B, H, I, 1, 1, dt, limit, &p)) continue;
                        ++exact;
                        const char *w = check_exact(p, B, H, I, limit, dt);
                        if (w || B < 2) return fail(w ? w : "exact ffn", B, H, I, 1);
                    }
                }
    ts_tune_set("down_chunks", 0);
    if (ffn < 1000 || moe < 1000 || exact < 2000) {
        std::printf("FAIL plans taken: ffn %ld moe %ld exact %ld\n", ffn, moe, exact);
        return 1;
    }

    // MoE shapes that have to be taken (the last rows: those that the GPU tests run)
    const int must[][5] = {{128, 4096, 14336, 8, 2}, {65, 4096, 14336, 8, 2}, {256, 4096, 14336, 16, 2},
                           {128, 2048, 7000, 4, 2}, {130, 520, 1205, 2, 2}, {200, 1032, 700, 4, 2},
                           {256, 264, 1300, 8, 4}, {128, 4096, 700, 4, 2}, {130, 4104, 665, 2, 2},
                           {65, 3592, 640, 2, 2}, {65, 8, 600, 2, 2}, {130, 256, 1040, 2, 1}};
    for (const auto &m : must) {
        BatchPlan p;
        if (!plan_wide_moe(m[0], m[1], m[2], m[3], m[4], TS_BF16, &p)) return fail("must be taken", m[0], m[1], m[2], m[3]);
    }

    // both sides of the size rule's lines: {batch, hidden, inter, experts, top_k, fp32, pays}
    const int lines[][7] = {{3, 2048, 4097, 1, 1, 1, 0}, {3, 2048, 6500, 1, 1, 1, 1},     // fp32, 32 MB and more
                            {2, 4096, 12000, 1, 1, 1, 0}, {2, 4096, 12300, 1, 1, 1, 1},   // two tokens
                            {6, 1024, 5000, 1, 1, 1, 0}, {8, 1024, 5000, 1, 1, 1, 1},     // one round (240), two (320 workgroups)
                            {9, 2048, 3500, 1, 1, 1, 0}, {10, 2048, 3500, 1, 1, 1, 1},    // (252, 280)
                            {24, 512, 3500, 1, 1, 1, 0}, {40, 512, 3500, 1, 1, 1, 1},     // below 12 MB
                            {18, 2048, 3600, 1, 1, 0, 0}, {19, 2048, 3600, 1, 1, 0, 1},   // bf16
                            {65, 512, 1792, 2, 1, 0, 0}, {128, 512, 1792, 4, 2, 0, 1},    // MoE
                            {10, 4096, 1792, 4, 1, 1, 0}, {11, 4096, 1792, 4, 1, 1, 1},
                            {4, 4096, 14336, 8, 2, 1, 0}, {4, 4096, 14336, 8, 2, 0, 0}};  // (no reading saved)
    for (const auto &l : lines)
        if (exact_pays(l[0], l[1], l[2], l[3], l[4], l[5] ? TS_F32 : TS_BF16) != (l[6] == 1))
            return fail("size rule", l[0], l[1], l[2], l[3]);
    std::printf("ok\n");
    return 0;
}
