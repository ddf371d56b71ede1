// Gate + up of a few tokens with fp32 weights (gfx950): the row stream of the
// single-token kernel for up to T tokens at once.
//
// The matrix-core kernel (bx_gate_up) reads its weights in 16-row operands
// and x as fragments from L2, and its fp32 products run at a quarter of the
// columns' use with 4 tokens.  Here every wave streams whole rows, as
// ffn_pipe does, and the tokens' x sit in LDS: a lane's 16-byte chunks of two
// rows meet the same x values, so a value read from LDS serves two rows, and
// a lane chains its share of a row, the wave's 64 sums meeting in wave_sum
// (the single-token kernel's products and chains).  Open rows' W_up loads
// follow the gate rows of the same wave without a barrier.  The result
// leaves in the batched layout: per 32-neuron tile the active rows as slots
// with their Combined records, for bx_down_f32.  Measured at 6 tokens,
// hidden 2052, inter 5003: 23.0 us against 4.4 + 30.8 with bx_prep +
// bx_gate_up; hidden 4096, inter 14336: 78.5 against 4.4 + 87.5 (409 MB of
// rows, 5.2 TB/s).  With bf16 weights the two extra unpacking operations per
// pair and twice the products per byte make it VALU-bound at 4 tokens (44 us
// against 40.5 + 4.3), so it serves fp32 only.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "ts_bx.h"
#include "ts_device.h"
#include "ts_plan.h"
#include "ts_runtime.h"
#include "turbosparse.h"

namespace ts {

namespace {
constexpr int kRowThreads = 512;
constexpr int kRowWaves = kRowThreads / 64;
constexpr uint32_t kRowOob = 0xFFFFFFF0u;  // past any matrix here: zeros, no traffic
}  // namespace

// One workgroup: `tiles` (1 or 2) 32-neuron tiles; wave w takes rows w, w + 8,
// ... two at a time.  A row is read in nseg segments of 64 NC chunks.
template <int T, int NC>
__global__ __launch_bounds__(kRowThreads, 2) void bx_rows(BxArgs a, int nseg, int tiles) {
    constexpr int TOK = 16;             // slots of a Combined record (bx_down_f32<16>)
    constexpr int MAXCH = 2 * 64 * NC;  // chunks per row at most (two segments)
    constexpr int RW = 2 * kBxRows;     // rows per workgroup at most
    __shared__ f32x4 s_x[T][MAXCH];
    __shared__ float s_g[RW][T], s_u[RW][T];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int H = a.H, nch = H / 4;
    const int tile0 = blockIdx.x * tiles, r0 = tile0 * kBxRows;
    const int nrow = min(tiles * kBxRows, a.I - r0);
    const int ng = a.B;
    const float thr = gate_threshold(a.act, a.tau);
    const uint32_t Hb = (uint32_t)H * 4u;
    const size_t base = (size_t)r0 * Hb;
    const uint32_t tbytes = (uint32_t)nrow * Hb;
    const __amdgpu_buffer_rsrc_t rg = make_rsrc(static_cast<const char *>(a.wg) + base, tbytes);
    const __amdgpu_buffer_rsrc_t ru = make_rsrc(static_cast<const char *>(a.wu) + base, tbytes);

    // work items of this wave: gate pairs in order, then pairs of open rows
    struct Item {
        int ra, rb, up, seg;  // tile-local rows (-1: none)
    };
    const int nown = wave < nrow ? (nrow - wave + kRowWaves - 1) / kRowWaves : 0;  // rows wave, wave + 8, ...
    int gnext = 0;         // next gate row (own index)
    uint32_t open = 0u;    // own rows with an open gate whose W_up row is not requested yet
    auto pick = [&](const Item &last) {
        Item n{-1, -1, 0, 0};
        if (last.ra >= 0 && last.seg + 1 < nseg) {
            n = last;
            ++n.seg;
        } else if (gnext < nown) {
            n.ra = wave + kRowWaves * gnext;
            n.rb = gnext + 1 < nown ? n.ra + kRowWaves : -1;
            gnext += 2;
        } else if (open) {
            n.up = 1;
            n.ra = wave + kRowWaves * (__ffs((int)open) - 1);
            open &= open - 1u;
            if (open) {
                n.rb = wave + kRowWaves * (__ffs((int)open) - 1);
                open &= open - 1u;
            }
        }
        return n;
    };
    u32x4 w[2][2][NC];
    auto issue = [&](int s, const Item &n) {
        const __amdgpu_buffer_rsrc_t rs = n.up ? ru : rg;
#pragma unroll
        for (int k = 0; k < NC; ++k) {
            const int c = n.seg * (64 * NC) + 64 * k + lane;
            const uint32_t cb = 16u * (uint32_t)c;
            w[s][0][k] = ld_buf_stream(rs, n.ra >= 0 && c < nch ? (uint32_t)n.ra * Hb + cb : kRowOob);
            w[s][1][k] = ld_buf_stream(rs, n.rb >= 0 && c < nch ? (uint32_t)n.rb * Hb + cb : kRowOob);
        }
    };
    Item cur = pick(Item{-1, -1, 0, 0});
    issue(0, cur);

    // x into LDS (zero past the batch; chunks past the row end meet zero weights)
    for (int t = 0; t < T; ++t)
        for (int c = tid; c < nseg * 64 * NC; c += kRowThreads)
            s_x[t][c] = t < a.B && c < nch ? *reinterpret_cast<const f32x4 *>(a.x + (size_t)t * H + 4 * c)
                                           : f32x4{0.f, 0.f, 0.f, 0.f};
    if (blockIdx.x == 0) {
        for (int t = tid; t < a.B; t += kRowThreads) {
            a.tslot[t * 2] = 0;
            a.tslot[t * 2 + 1] = t;
        }
        if (tid == 0) a.gcount[0] = a.B;
    }
    __syncthreads();

    float d[2][T];
    auto compute = [&](int s, const Item &n) {
        if (n.seg == 0) {
#pragma unroll
            for (int t = 0; t < T; ++t) d[0][t] = d[1][t] = 0.f;
        }
#pragma unroll
        for (int k = 0; k < NC; ++k) {
            const int c = n.seg * (64 * NC) + 64 * k + lane;
            const f32x4 fa = __builtin_bit_cast(f32x4, w[s][0][k]), fb = __builtin_bit_cast(f32x4, w[s][1][k]);
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const f32x4 x = s_x[t][c];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    d[0][t] = fmaf(fa[e], x[e], d[0][t]);
                    d[1][t] = fmaf(fb[e], x[e], d[1][t]);
                }
            }
        }
        if (n.seg + 1 < nseg) return;
        // the row's sums; a gate row that some token opens asks for its W_up row
        float(*dst)[T] = n.up ? s_u : s_g;
        bool oa = false, ob = false;
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const float va = wave_sum(d[0][t]), vb = wave_sum(d[1][t]);
            oa |= va > thr && t < ng;
            ob |= vb > thr && t < ng;
            if (lane == 0) {
                dst[n.ra][t] = va;
                if (n.rb >= 0) dst[n.rb][t] = vb;
            }
        }
        if (!n.up) {
            // (wave-uniform values: every lane holds the same sums)
            const uint32_t ia = (uint32_t)(n.ra / kRowWaves);
            uint32_t m = (a.dense || oa) ? 1u << ia : 0u;
            if (n.rb >= 0 && (a.dense || ob)) m |= 1u << (ia + 1u);
            open |= (uint32_t)__builtin_amdgcn_readfirstlane((int)m);
        }
    };
    // two register slots in turn; the next item's loads are in flight while
    // one is computed (an empty item loads nothing)
    bool more = cur.ra >= 0;
    while (more) {
        const Item n1 = pick(cur);
        issue(1, n1);
        if (cur.ra >= 0) compute(0, cur);
        cur = pick(n1);
        issue(0, cur);
        if (n1.ra >= 0) compute(1, n1);
        more = cur.ra >= 0 || open != 0u || gnext < nown;
    }
    __syncthreads();

    // ---- per tile (one wave each): open and active rows, Combined records
    if (wave >= tiles || tile0 + wave >= a.ntiles) return;
    const size_t tix = (size_t)(tile0 + wave);
    const int r = wave * kBxRows + (lane & 31);
    const bool in = lane < kBxRows && r < nrow;
    bool op = false, ac = false;
    float h[T];
    const int rr = in ? r : 0;
#pragma unroll
    for (int t = 0; t < T; ++t) {
        const float g = s_g[rr][t], u = s_u[rr][t];  // (s_u: only of rows some token opens)
        const bool o = in && t < ng && g > thr;
        const bool on = o && combined_nonzero(a.act, u);
        h[t] = on ? combined_value(a.act, a.tau, g, u) : 0.f;
        op |= o;
        ac |= on;
        if (a.want_masks) {
            const uint64_t mo = __ballot(o), ma = __ballot(on);
            if (lane == 0) {
                a.gmask[tix * TOK + t] = (uint32_t)mo;
                a.amask[tix * TOK + t] = (uint32_t)ma;
            }
        }
    }
    if (a.want_masks)
        for (int t = T + lane; t < TOK; t += 64) {
            a.gmask[tix * TOK + t] = 0u;
            a.amask[tix * TOK + t] = 0u;
        }
    const uint32_t om = (uint32_t)__ballot(a.dense ? in : op), am = (uint32_t)__ballot(a.dense ? in : ac);
    const int na = __popc(am);
    if ((am >> (lane & 31)) & 1u && lane < kBxRows) {
        const int slot = __popc(am & ((1u << lane) - 1u));
        f32x4 *dst = reinterpret_cast<f32x4 *>(a.hfrag) + (tix * kBxRows + slot) * (TOK / 4);
#pragma unroll
        for (int q = 0; q < TOK / 4; ++q) {
            f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (4 * q + e < T) v[e] = h[4 * q + e < T ? 4 * q + e : 0];
            dst[q] = v;
        }
    }
    if (lane < kBxRows)  // an empty tile lists row 0 (always < I), never used
        a.arow[tix * kBxRows + lane] = na > 0 ? (uint8_t)nth_set_bit(am, lane < na ? lane : 0) : (uint8_t)0;
    if (lane == 0) {
        a.cnt[tix * 2] = __popc(om);
        a.cnt[tix * 2 + 1] = na;
    }
}

namespace {

// Chunks per lane: a lane's chunks past its segment are loads of nothing, but
// their products are issued, so rows of five or six chunks have forms of their
// own (6 tokens, hidden 2052 25.4 us against 28.7 in the form of eight, 8
// tokens 26.3 against 34.9; six chunks, hidden 3072, 8 tokens 29.8 against
// 36.0); three or seven round up (a 64th to an 8th of the widest hidden).
template <int T>
void launch_rows_t(const BatchPlan &p, const BxArgs &a, hipStream_t st) {
    const int nch = p.hidden / 4;
    const int nseg = nch > 512 ? 2 : 1;
    const int nc = ((nch + nseg - 1) / nseg + 63) / 64;  // chunks per lane and segment, at most 8
    // two tiles per workgroup where that still fills the chip
    const int tiles = p.ntiles >= 2 * 224 ? 2 : 1;
    const dim3 grid((unsigned)((p.ntiles + tiles - 1) / tiles)), b(kRowThreads);
    if (nc <= 2) launch("batch_gate_up", bx_rows<T, 2>, grid, b, st, a, nseg, tiles);
    else if (nc <= 4) launch("batch_gate_up", bx_rows<T, 4>, grid, b, st, a, nseg, tiles);
    else if (nc <= 5) launch("batch_gate_up", bx_rows<T, 5>, grid, b, st, a, nseg, tiles);
    else if (nc <= 6) launch("batch_gate_up", bx_rows<T, 6>, grid, b, st, a, nseg, tiles);
    else launch("batch_gate_up", bx_rows<T, 8>, grid, b, st, a, nseg, tiles);
}

}  // namespace

// Tokens: the products of a slot past the batch are issued as well.  A form of
// six serves 5 and 6 tokens (hidden 4096, 6 tokens 36.6 us against 40.5 in the
// form of eight, 512 x 14000 15.6 against 18.4).
void launch_rows(const BatchPlan &p, const BxArgs &a, hipStream_t st) {
    if (p.batch <= 4) launch_rows_t<4>(p, a, st);
    else if (p.batch <= 6) launch_rows_t<6>(p, a, st);
    else launch_rows_t<8>(p, a, st);
}

}  // namespace ts
