// Device-side pieces shared by the batched kernels (ts_batch.hip: up to 64
// token slots per group, ts_rows.hip: a few fp32 tokens, ts_wide.hip: wide
// batches).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "ts_device.h"
#include "ts_plan.h"

namespace ts {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ f32x4 mfma_bf16(const u32x4 a, const u32x4 b, const f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c,
                                                   0, 0, 0);
}

// Shape constants per token-slot count TOK (8, 16, 32, 64).  A k-step is 64
// bytes of a weight row (32 bf16 or 16 fp32 elements): one 16-byte chunk per
// lane of a 16-row operand in every mode.
template <int TOK, int M = kBxBf16x2>
struct Bx {
    static constexpr bool F32 = M == kBxF32;
    static constexpr int ESZ = F32 ? 4 : 2;              // bytes per weight element
    static constexpr int P = F32 ? 1 : (M == kBxBf16x3 ? 3 : 2);
    static constexpr bool PACK = TOK == 8;               // two parts share one 16-column tile
    static_assert(!(PACK && F32), "fp32 operands: 16 or more token slots");
    static constexpr int NT = PACK ? 1 : TOK / 16;       // 16-token accumulator tiles
    static constexpr int NX = PACK ? (P + 1) / 2 : P * NT;  // operand fragments per k-step (x or Combined)
    static constexpr int REC = F32 ? TOK * 4 : P * TOK * 2; // bytes of a slot's Combined record
    // k-steps per batch of gate / up loads (default; measured: 2 at 8 token
    // slots, 4 at 16, 2 past that, where deeper rings spill)
    static constexpr int KS = PACK ? 2 : (NX <= 2 ? 4 : 2);
    static constexpr int D = 2;                     // gate / up batches in flight per wave (default)
    static constexpr int DD = 2;                    // down blocks in flight per wave (default)
};

// Part p (< P, run-time) of v, without a branch.
template <int P>
__device__ __forceinline__ uint32_t bf16_sel(float v, int p) {
    uint32_t out = 0;
#pragma unroll
    for (int q = 0; q < P; ++q) {
        const uint32_t b = bf16_take<P>(v);
        out = q == p ? b : out;
    }
    return out;
}

struct BxArgs {
    const float *x;          // [tokens][H] (already offset to the pass's first token)
    const void *wg, *wu, *wd;
    size_t expert_stride;    // elements per expert matrix (0: one weight set)
    int B, H, I, G, K, bpad, hpad, ntiles, nslices, nchunks, tpc;
    int vpe;                 // groups per weight set: group g uses weight set g / vpe
    const int32_t *topk;     // [B][K] routed experts, or null (FFN)
    const float *topw;       // [B][K] routing weights, or null
    int32_t *gcount;         // [G]
    int32_t *tslot;          // [B][K][2] (group, slot) of each routed token
    uint16_t *xhl;           // x fragments [G][k-steps][NX][64 lanes][16 bytes] (MFMA operand order)
    int32_t *cnt;            // [G][ntiles][2] |union G|, |union A|
    uint8_t *arow;           // [G][ntiles][32] row within the tile of each active slot (slot 0's past |union A|)
    uint16_t *hfrag;         // [G][ntiles][32 slots][P][bpad] Combined per active slot in P bf16 parts
                             // (kBxF32: [32 slots][bpad] fp32)
    uint32_t *gmask;         // [G][ntiles][bpad] open-gate rows of the tile per token
    uint32_t *amask;         // [G][ntiles][bpad] active rows of the tile per token
    float *partial;          // [G][bpad][nchunks][H]
    float *out;              // [tokens][H]
    int want_masks;
    int dense;               // 1: every row is taken (the dense comparator)
    const uint16_t *xtok;    // or null: every token's x in P bf16 parts, token-major (the MoE router's
                             // split: per token xchunks chunks of 8 values, P 16-byte pieces each at xs_pos)
    int xchunks;
    int act;                 // activation (gate_threshold and the two functions beside it)
    float tau;
};

constexpr uint32_t kPadRow = 0xFFFFFFFFu;  // row-list padding of the down kernels

// Gate + up of a few tokens with fp32 weights by row streams (ts_rows.hip).
void launch_rows(const BatchPlan &p, const BxArgs &a, hipStream_t st);

// The wide kernels (ts_wide.hip) of one call: x fragments and group tables
// (without a routing table), gate + up, down.
void launch_wide_prep(const BatchPlan &p, const BxArgs &a, hipStream_t st);
void launch_wide_gate_up(const BatchPlan &p, const BxArgs &a, hipStream_t st);
void launch_wide_down(const BatchPlan &p, const BxArgs &a, hipStream_t st);

// Group g's token list (MoE): the tokens routed to expert g / vpe, entries
// [r0, r0 + TOK) of that expert's ascending list, by one wave scanning the
// (token, rank) pairs in token-major order; s_tok[slot] = token, -1 past the
// count.  With `tables`, also the group's token count and the (group, slot)
// of each of its routed pairs (for the reduce and the report).  Returns the
// count (on every lane).
template <int TOK>
__device__ __forceinline__ int bx_list_group(const BxArgs &a, int g, int lane, int *s_tok, bool tables) {
    const int np = a.B * a.K;
    const int e = g / a.vpe, r0 = (g - e * a.vpe) * TOK;
    int base = 0;
    for (int p0 = 0; p0 < np; p0 += 64) {
        const int p = p0 + lane;
        const bool mine = p < np && a.topk[p] == e;
        const uint64_t m = __ballot(mine);
        const int rank = base + lane_prefix(m, lane) - r0;  // rank within this group
        if (mine && rank >= 0 && rank < TOK) {
            s_tok[rank] = p / a.K;
            if (tables) {
                a.tslot[p * 2] = g;
                a.tslot[p * 2 + 1] = rank;
            }
        }
        base += __popcll(m);
    }
    const int n = min(max(base - r0, 0), TOK);
    for (int sl = n + lane; sl < TOK; sl += 64) s_tok[sl] = -1;
    if (tables && lane == 0) a.gcount[g] = n;
    return n;
}

// A down workgroup's row list: the active rows of `ntc` tiles from tile
// index tbase, tile after tile, as (tile within the chunk) << 10 | slot << 5
// | row, padded with kPadRow to whole blocks of KB rows; s_pre (ntc + 1) is
// scratch.  Returns the number of blocks; ends with a barrier.
template <int THREADS, int KB>
__device__ __forceinline__ int bx_list_rows(const BxArgs &a, size_t tbase, int ntc, int *s_pre, uint32_t *s_ent) {
    const int tid = threadIdx.x, lane = tid & 63;
    if (tid < 64) {  // wave 0 scans the tiles' active counts
        int base = 0;
        for (int t = 0; t < ntc; t += 64) {
            const int v = t + lane < ntc ? a.cnt[(tbase + t + lane) * 2 + 1] : 0;
            int inc = v;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int u = __shfl_up(inc, o, 64);
                if (lane >= o) inc += u;
            }
            if (t + lane < ntc) s_pre[t + lane] = base + inc - v;
            base += __shfl(inc, 63, 64);
        }
        if (lane == 0) s_pre[ntc] = base;
    }
    __syncthreads();
    const int total = s_pre[ntc];
    const int nblk = (total + KB - 1) / KB;
    for (int e = tid; e < ntc * kBxRows; e += THREADS) {
        const int t = e / kBxRows, s = e % kBxRows;
        const int base = s_pre[t];
        if (s < s_pre[t + 1] - base)
            s_ent[base + s] = ((uint32_t)t << 10) | ((uint32_t)s << 5) | (uint32_t)(a.arow[tbase * kBxRows + e] & 31);
    }
    for (int e = total + tid; e < nblk * KB; e += THREADS) s_ent[e] = kPadRow;
    __syncthreads();
    return nblk;
}

// Position of the n-th (from 0) set bit of m, by halving with population
// counts; n < popcount(m) (otherwise some position in 0..31).
__device__ __forceinline__ int nth_set_bit(uint32_t m, int n) {
    int pos = 0;
#pragma unroll
    for (int w = 16; w >= 1; w >>= 1) {
        const int c = __popc(m & ((1u << w) - 1u));
        if (n >= c) {
            n -= c;
            m >>= w;
            pos += w;
        }
    }
    return pos;
}

}  // namespace ts
