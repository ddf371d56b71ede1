// Batched activation-sparse dReLU FFN for gfx950 where a weight set has many
// tokens: workgroup-tiled matrix-core kernels whose operands are shared
// through LDS by all waves of a workgroup.
//
// The kernels of ts_batch.hip let every wave contract its own quarter of the
// hidden dimension for all rows and tokens of a workgroup: no barrier in the
// K loop, but each wave holds every accumulator, so a workgroup takes at
// most 64 rows x 64 tokens, and more tokens mean another pass over the
// weights.  Here the eight waves split the workgroup's rows and tokens, the
// K loop stages both operands in LDS once per workgroup (double buffered,
// the next stages' loads in registers), and:
//   wd_gate_up   a workgroup takes NB neurons' W_gate and W_up rows together
//                against up to TOK tokens: one pass over the x fragments for
//                both matrices, gate and up of a neuron end in the same
//                lane, and Combined leaves the kernel as in ts_batch.hip
//                (active rows of each 32-row tile as slots).  Every W_up row
//                is read: with this many tokens nearly every row is open for
//                one of them (at 20% open gates 99.9% of the rows at 32
//                tokens).
//   wd_down      per (group, chunk of tiles, column slice): K blocks of 32
//                listed active rows; W_down_t rows and Combined records are
//                both neuron-major, so both operands are read back from LDS
//                with transposing reads (ds_read_b64_tr_b16).
// x and Combined enter as P bf16 parts: 2 (16 significant bits) or 3 (all
// 24 bits of the fp32 value: products as exact as fp32 ones).
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "ts_bx.h"
#include "ts_device.h"
#include "ts_plan.h"
#include "ts_runtime.h"
#include "turbosparse.h"

namespace ts {

namespace {

constexpr int kWdThreads = 512;

// Past every buffer resource here (matrices are below 4 GB): a load there
// returns zeros and touches no memory.
constexpr uint32_t kWdOob = 0xFFFFFFF0u;

template <bool STREAM>
__device__ __forceinline__ u32x4 wd_ld(__amdgpu_buffer_rsrc_t r, uint32_t off) {
    if constexpr (STREAM) return ld_buf_stream(r, off);
    else return ld_buf_cached(r, off);
}

// 16-byte chunk c of 128-byte LDS row r sits at this position: 16 rows of a
// fragment read spread over all banks.
__device__ __forceinline__ int wd_swz(int r, int c) { return r * 8 + (c ^ ((r >> 1) & 7)); }

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

// MFMA operand (lane (lm, lq): eight k's of column lm) out of a k-major LDS
// tile: two transposing reads, each giving the 16 lanes of one lq four k
// rows x 16 columns; `p` is the tile's column 0 of the fragment, `pitch` in
// elements.  Lane group lq takes k rows 4 lq .. 4 lq + 3 and 16 + 4 lq ..
// (both operands alike, so every product pairs the same k): the rows of one
// read are consecutive and, with rows padded by 32 bytes, spread over all
// banks.
__device__ __forceinline__ u32x4 wd_tr_frag(const uint16_t *p, int pitch, int lane) {
    const int lm = lane & 15, lq = lane >> 4;
    const uint16_t *q = p + (4 * lq + (lm >> 2)) * pitch + 4 * (lm & 3);
    typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
    const s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(q));
    const s16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(q + 16 * pitch));
    return __builtin_bit_cast(u32x4, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
}

// Workgroup barrier that orders LDS only (global loads stay in flight).
__device__ __forceinline__ void wd_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Instruction order of a half stage that reads the next k-step's operands
// (R LDS reads) while M matrix instructions contract the present one, and
// writes W chunks of the next stage: spread over each other.  Left alone the
// compiler moves every read next to its use, and the reads' time adds to the
// matrix instructions' instead of hiding behind them.
template <int R, int W, int M>
__device__ __forceinline__ void wd_spread() {
    constexpr int PER = R > 0 && (M - W) / R > 0 ? (M - W) / R : 1;
#pragma unroll
    for (int i = 0; i < R; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);  // LDS read
        __builtin_amdgcn_sched_group_barrier(0x008, PER, 0);  // matrix
    }
#pragma unroll
    for (int i = 0; i < W; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);  // LDS write
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
}

// The same for a half stage of N operand fragments with G matrix
// instructions each: the reads follow the instructions, so a fragment's
// register is free for the next k-step's by the time that is read.
template <int R, int W, int N, int G, int I = 0>
__device__ __forceinline__ void wd_roll() {
    if constexpr (I < N) {
        constexpr int READS = (I + 1) * R / N - I * R / N;
        constexpr int WRITES = 2 * I < N ? 0 : (2 * I + 2 - N) * W / N - (2 * I - N) * W / N;  // the later half
        __builtin_amdgcn_sched_group_barrier(0x008, G, 0);
        if constexpr (READS > 0) __builtin_amdgcn_sched_group_barrier(0x100, READS, 0);
        if constexpr (WRITES > 0) __builtin_amdgcn_sched_group_barrier(0x200, WRITES, 0);
        wd_roll<R, W, N, G, I + 1>();
    } else {
        __builtin_amdgcn_sched_barrier(0);
    }
}

}  // namespace

// x of every group's token slots as MFMA operand fragments in P parts (the
// FFN: group g holds tokens [g TOK, (g + 1) TOK)); fragment P nt + part of
// k-step ks, lane (lm, lq): the 8 values at k = 32 ks + 8 lq of token slot
// 16 nt + lm.  One thread per (group, k-step, n-tile, lane): one read of x,
// P fragments written.
template <int TOK, int P>
__global__ __launch_bounds__(256) void wd_prep(BxArgs a) {
    constexpr int NTT = TOK / 16;
    const int nks = a.hpad / 32;
    if (blockIdx.x == 0) {
        for (int t = threadIdx.x; t < a.B; t += 256) {
            a.tslot[t * 2] = t / TOK;
            a.tslot[t * 2 + 1] = t % TOK;
        }
        for (int g = threadIdx.x; g < a.G; g += 256) a.gcount[g] = min(TOK, a.B - g * TOK);
    }
    const int idx = blockIdx.x * 256 + threadIdx.x;
    if (idx >= a.G * nks * NTT * 64) return;
    const int lane = idx & 63, lm = lane & 15, lq = lane >> 4;
    const int nt = (idx >> 6) % NTT;
    const int ks = (idx >> 6) / NTT % nks;
    const int g = (idx >> 6) / (NTT * nks);
    const int t = g * TOK + 16 * nt + lm;
    const int k0 = ks * 32 + 8 * lq;
    float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (t < a.B && k0 < a.H) {  // H is a multiple of 8, so all 8 are in range
        const f32x4 *src = reinterpret_cast<const f32x4 *>(a.x + (size_t)t * a.H + k0);
        const f32x4 p = src[0], q = src[1];
        v[0] = p.x; v[1] = p.y; v[2] = p.z; v[3] = p.w;
        v[4] = q.x; v[5] = q.y; v[6] = q.z; v[7] = q.w;
    }
    u32x4 *dst = reinterpret_cast<u32x4 *>(a.xhl) + (((size_t)g * nks + ks) * (P * NTT) + P * nt) * 64 + lane;
#pragma unroll
    for (int p = 0; p < P; ++p) {
        uint32_t o[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint32_t b0 = bf16_take<P>(v[2 * e]), b1 = bf16_take<P>(v[2 * e + 1]);
            o[e] = b0 | (b1 << 16);
        }
        dst[p * 64] = u32x4{o[0], o[1], o[2], o[3]};
    }
}

// ---------------------------------------------------------------------------
// Gate + up for NB neurons x TOK token slots per workgroup: 2 NB weight rows
// (gate rows first) and the x fragments of 64 hidden elements per stage.
// Waves: 4 along the neurons x 2 along the tokens; a wave's gate and up
// m-tiles are of the same neurons.  D stages of loads are in flight in
// registers besides the two LDS buffers.  STREAM: non-temporal weight loads
// (off where several groups share a weight set: the second group's read of a
// tile then hits in L2, since both run on one XCD).
// QSPLIT: the sums of the hidden dimension's quarters are added in
// bx_gate_up's order, (q0 + q1) + (q2 + q3): the same bits.  QSEQ (128
// slots): one after another, which holds one total besides the running sums.
// A single chain over the hidden dimension rounds more: error against 64 bits
// at hidden 4096 / 8192 4.92e-6 / 5.00e-6, in quarters 4.88e-6 / 4.91e-6 (as
// the passes of 64 tokens), for 103 -> 107 us at 256 tokens of the Mistral
// shape, 69.5 -> 71.5 at 128.  ROLL: the totals leave room for one register
// slot of x fragments, not two (wd_roll).
template <int TOK, int P, int NB, int D, bool GATHER, bool STREAM, bool AHEAD>
__global__ __launch_bounds__(kWdThreads, 2) void wd_gate_up(BxArgs a) {
    constexpr int KS = 2;                       // 32-wide k-steps per stage
    constexpr int NX = P * TOK / 16;            // x fragments per k-step
    constexpr int NA = 2 * NB * 8 / kWdThreads; // weight chunks per thread and stage
    constexpr int XCH = KS * NX * 64;           // x chunks per stage
    constexpr int NXL = (XCH + kWdThreads - 1) / kWdThreads;
    constexpr int MN = NB / 64;                 // neuron m-tiles per wave
    constexpr int NT = TOK / 32;                // token n-tiles per wave
    constexpr int NW = NB / kBxRows;            // 32-row tiles per workgroup
    constexpr bool QSPLIT = TOK <= 64 && P == 2;
    constexpr bool QSEQ = TOK > 64, ROLL = QSEQ && NB == 128;
    constexpr int ABUF = 2 * NB * 8, BBUF = XCH;  // 16-byte units per LDS buffer
    constexpr int SH = NB * P * TOK / 8;          // 16-byte units of the Combined staging
    constexpr int LDS = 2 * (ABUF + BBUF) > SH ? 2 * (ABUF + BBUF) : SH;
    static_assert(NA % 2 == 0 && NB % 64 == 0 && TOK % 32 == 0, "gate and up halves, whole wave tiles");
    __shared__ u32x4 s_lds[LDS];
    __shared__ uint32_t s_open[NW], s_act[NW];
    __shared__ uint32_t s_gm[NW][TOK], s_am[NW][TOK];
    __shared__ int s_tok[GATHER ? TOK : 1];
    __shared__ int s_ng;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lm = lane & 15, lq = lane >> 4;
    const int wm = wave >> 1, wn = wave & 1;
    const int nwt = (a.ntiles + NW - 1) / NW;  // workgroup tiles per group
    int g, wt;
    if constexpr (GATHER) {
        g = bx_group_at(blockIdx.x / nwt, a.G, a.vpe);
        wt = blockIdx.x % nwt;
    } else {
        // groups share the weight set: all groups of a tile on one XCD
        // (the dispatcher hands workgroup b to XCD b % 8), one after another
        const int q = blockIdx.x % 8, r = blockIdx.x / 8;
        g = r % a.G;
        wt = 8 * (r / a.G) + q;
        if (wt >= nwt) return;
    }
    const int tile0 = wt * NW;
    const int nsub = min(NW, a.ntiles - tile0);
    const size_t tix0 = (size_t)g * a.ntiles + tile0;
    int ng;
    if constexpr (GATHER) {
        if (wave == 0) {
            const int n = bx_list_group<TOK>(a, g, lane, s_tok, wt == 0);
            if (lane == 0) s_ng = n;
        }
        __syncthreads();
        ng = s_ng;
    } else {
        ng = a.gcount[g];
    }
    if (ng == 0) {
        if (tid < 2 * nsub) a.cnt[tix0 * 2 + tid] = 0;
        if (a.want_masks)
            for (int s = tid; s < nsub * TOK; s += kWdThreads) {
                a.gmask[tix0 * TOK + s] = 0;
                a.amask[tix0 * TOK + s] = 0;
            }
        return;
    }
    if (tid < NW) {
        s_open[tid] = 0u;
        s_act[tid] = 0u;
    }
    for (int e = tid; e < NW * TOK; e += kWdThreads) {
        (&s_gm[0][0])[e] = 0u;
        (&s_am[0][0])[e] = 0u;
    }

    const int H = a.H, r0 = tile0 * kBxRows;
    const uint32_t mbytes = (uint32_t)a.I * (uint32_t)H * 2u;
    const size_t eoff = (size_t)(g / a.vpe) * a.expert_stride;
    const __amdgpu_buffer_rsrc_t rwg = make_rsrc(reinterpret_cast<const uint16_t *>(a.wg) + eoff, mbytes);
    const __amdgpu_buffer_rsrc_t rwu = make_rsrc(reinterpret_cast<const uint16_t *>(a.wu) + eoff, mbytes);
    const int nst = a.hpad / (32 * KS);  // a multiple of 16 (kBxKQuant)

    // this thread's weight chunks: LDS row 64 j + tid / 8, chunk tid % 8
    const int ac = tid & 7, ar = tid >> 3;
    uint32_t aoff[NA];
#pragma unroll
    for (int j = 0; j < NA; ++j) {
        const int row = 64 * (j % (NA / 2)) + ar;
        aoff[j] = 2u * (uint32_t)min(r0 + row, a.I - 1) * (uint32_t)H + 16u * (uint32_t)ac;
    }
    // x chunks: linear in the group's fragments, or gathered from the
    // token-major split (pieces at xs_pos)
    const u32x4 *xb = reinterpret_cast<const u32x4 *>(a.xhl) + (size_t)g * (a.hpad / 32) * NX * 64;
    const __amdgpu_buffer_rsrc_t rx =
        GATHER ? make_rsrc(a.xtok, (uint32_t)a.B * (uint32_t)a.xchunks * 16u * P)
               : make_rsrc(xb, (uint32_t)(a.hpad / 32) * NX * 1024u);
    uint32_t xoff[NXL];
#pragma unroll
    for (int j = 0; j < NXL; ++j) {
        const int idx = tid + kWdThreads * j;
        xoff[j] = kWdOob;
        if (idx < XCH) {
            if constexpr (GATHER) {
                const int l = idx & 63, f = (idx >> 6) % NX, s = (idx >> 6) / NX;
                const int tk = s_tok[16 * (f / P) + (l & 15)];
                if (tk >= 0)
                    xoff[j] = ((uint32_t)tk * (uint32_t)a.xchunks * P + (uint32_t)xs_pos(4 * s + (l >> 4), f % P, P)) * 16u;
            } else {
                if (16 * ((idx >> 6) % NX / P) < ng) xoff[j] = 16u * (uint32_t)idx;
            }
        }
    }
    constexpr uint32_t XSTEP = GATHER ? KS * 4 * 16 * P : XCH * 16;  // bytes per stage

    u32x4 ra[D][NA], rb[D][NXL];
    // MoE, rows above 6 KB (padded to 8 KB): every workgroup starts at another
    // fold of the hidden dimension.  In step, all would read the same 128-byte
    // column of rows that far apart, and how many memory channels that meets
    // depends on where the weights lie.  8 experts, 128 tokens, over several
    // allocations, without / with: 4096 x 14336 392 to 466 / 374 to 386 us,
    // 4096 x 7168 204 to 237 / 192 to 194, 3584 x 7168 205 / 196, 8192 x 3584
    // 199 to 212 / 186.  Shorter rows: 4 experts of 2048 x 7000 102 to 109 /
    // 109, but 8 of 2048 x 7168 125 to 136 / 117 to 125 and 3072 x 7168 169 /
    // 163; 1024 x 7168 the same.  The FFN (one weight set) gained nothing: 32
    // tokens 43.2 / 45.8 us, 256 tokens 102.4 / 104.9.
    const int rot = GATHER && nst >= 64 ? 8 * ((int)(blockIdx.x / 8) % (nst / 8)) : 0;
    auto issue = [&](int d, int lst) {
        int st = lst;
        if constexpr (GATHER) {
            st += rot;
            st -= st >= nst ? nst : 0;
        }
        // (a stage past the last one loads nothing)
        const bool kin = (!GATHER || lst < nst) && st * 64 + 8 * ac < H;
#pragma unroll
        for (int j = 0; j < NA; ++j)
            ra[d][j] = wd_ld<STREAM>(j < NA / 2 ? rwg : rwu, kin ? aoff[j] + 128u * (uint32_t)st : kWdOob);
#pragma unroll
        for (int j = 0; j < NXL; ++j)
            rb[d][j] = ld_buf_cached(rx, xoff[j] != kWdOob ? xoff[j] + XSTEP * (uint32_t)st : kWdOob);
    };
    auto stash = [&](int d, int buf) {
        u32x4 *sa = s_lds + buf * ABUF, *sb = s_lds + 2 * ABUF + buf * BBUF;
#pragma unroll
        for (int j = 0; j < NA; ++j) sa[wd_swz(64 * j + ar, ac)] = ra[d][j];
#pragma unroll
        for (int j = 0; j < NXL; ++j)
            if (XCH % kWdThreads == 0 || tid + kWdThreads * j < XCH) sb[tid + kWdThreads * j] = rb[d][j];
    };
    // P == 3 (fp32-exact operands): the high parts' sums apart from the small
    // lower ones (cgl, cul), so those do not round the large sum
    constexpr bool LO = P == 3;
    f32x4 cg[MN][NT], cu[MN][NT], cgl[LO ? MN : 1][LO ? NT : 1], cul[LO ? MN : 1][LO ? NT : 1];
    auto clear = [&]() {
#pragma unroll
        for (int m = 0; m < MN; ++m)
#pragma unroll
            for (int n = 0; n < NT; ++n) cg[m][n] = cu[m][n] = f32x4{0.f, 0.f, 0.f, 0.f};
    };
    // operand fragments of k-step s in register slot s: the reads of the next
    // k-step are in flight while one is contracted
    u32x4 fa[2][2 * MN], fb[2][NT * P];
    // the wave's n-tiles are wn, wn + 2, ...; the first NACT hold tokens
    auto load = [&](int buf, int s, auto nac) {
        constexpr int NACT = decltype(nac)::value;
        const u32x4 *sa = s_lds + buf * ABUF, *sb = s_lds + 2 * ABUF + buf * BBUF;
        if constexpr (NACT > 0) {
#pragma unroll
            for (int m = 0; m < MN; ++m) {
                const int row = (wm * MN + m) * 16 + lm;
                fa[s][2 * m] = sa[wd_swz(row, 4 * s + lq)];
                fa[s][2 * m + 1] = sa[wd_swz(NB + row, 4 * s + lq)];
            }
        }
#pragma unroll
        for (int n = 0; n < NACT; ++n)
#pragma unroll
            for (int p = 0; p < P; ++p) fb[s][P * n + p] = sb[(s * NX + P * (2 * n + wn) + p) * 64 + lane];
    };
    auto contract = [&](int s, auto nac) {
        constexpr int NACT = decltype(nac)::value;
#pragma unroll
        for (int n = 0; n < NACT; ++n)
#pragma unroll
            for (int p = 0; p < P; ++p)
#pragma unroll
                for (int m = 0; m < MN; ++m) {
                    f32x4 &g = LO && p ? cgl[LO ? m : 0][LO ? n : 0] : cg[m][n];
                    f32x4 &v = LO && p ? cul[LO ? m : 0][LO ? n : 0] : cu[m][n];
                    g = mfma_bf16(fa[s][2 * m], fb[s][P * n + p], g);
                    v = mfma_bf16(fa[s][2 * m + 1], fb[s][P * n + p], v);
                }
    };
    static_assert(KS == 2, "a register slot per k-step of a stage");

    constexpr int U = D > 2 ? D : 2;
    static_assert(4 % U == 0, "a quarter's stages (a multiple of 4) in whole rounds");
    clear();
#pragma unroll
    for (int d = 0; d < D; ++d) issue(d, d);
    stash(0, 0);
    issue(0, D);
    wd_barrier();
    // stage st of the ring slot (st mod D): its buffer is contracted, then
    // the next stage goes from registers to the other buffer and its slot
    // takes a later stage (loads past the last stage are out of range: zeros)
    auto steps_n = [&](int s0, int s1, auto nac) {
        constexpr int NACT = decltype(nac)::value;
        constexpr int R = NACT ? 2 * MN + NACT * P : 0, M = 2 * MN * NACT * P;  // (of a k-step)
        if (AHEAD && (QSEQ || s0 == 0)) load(0, 0, nac);
        for (int st = s0; st < s1; st += U) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if constexpr (!AHEAD) load(u & 1, 0, nac);
                load(u & 1, 1, nac);
                contract(0, nac);
                if constexpr (!AHEAD) contract(1, nac);
                stash((u + 1) % D, (u + 1) & 1);
                issue((u + 1) % D, st + u + 1 + D);
                if constexpr (AHEAD && ROLL && NACT > 0) wd_roll<R, NA + NXL, NACT * P, 2 * MN>();
                else if constexpr (AHEAD) wd_spread<R, NA + NXL, M>();
                wd_barrier();
                if constexpr (AHEAD) {
                    __builtin_amdgcn_sched_barrier(0);
                    load((u + 1) & 1, 0, nac);
                    contract(1, nac);
                    if constexpr (ROLL && NACT > 0) wd_roll<R, 0, NACT * P, 2 * MN>();
                    else wd_spread<R, 0, M>();
                }
            }
        }
    };
    // n-tiles without tokens are left out (rounded up to 0, 1, 2 or 4 tiles)
    const int nact = max(0, ((ng + 15) / 16 - wn + 1) / 2);
    auto steps = [&](int s0, int s1) {
        if constexpr (NT == 1) return steps_n(s0, s1, std::integral_constant<int, 1>{});
        if constexpr (NT >= 4) {
            if (nact > 2) return steps_n(s0, s1, std::integral_constant<int, 4>{});
        }
        if constexpr (NT >= 2) {
            if (nact > 1) return steps_n(s0, s1, std::integral_constant<int, 2>{});
        }
        if (nact > 0) return steps_n(s0, s1, std::integral_constant<int, 1>{});
        return steps_n(s0, s1, std::integral_constant<int, 0>{});
    };
    if constexpr (LO) {
        // the high parts' sum folded every FS stages of 64 elements: shorter
        // chains of roundings, so that the error is no larger than that of
        // the single-token kernels, whose chain is a lane's 1/64 of a row.
        // Against theirs, 6% open gates, every 8 / 4 / 2 stages: hidden 1024
        // 1.33 / 1.07 / 0.86, 2048 1.19 / 0.90 / 0.74, 4096 0.95 / 0.72 / 0.63;
        // a fold every 4 stages costs 3.5 us of 53 (ReLU, 32 tokens)
        const int FS = H >= 4096 ? 8 : (H >= 2048 ? 4 : 2);
        f32x4 tg[MN][NT], tu[MN][NT];
#pragma unroll
        for (int m = 0; m < MN; ++m)
#pragma unroll
            for (int n = 0; n < NT; ++n) tg[m][n] = tu[m][n] = cgl[m][n] = cul[m][n] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int s0 = 0; s0 < nst; s0 += FS) {
            clear();
            steps(s0, s0 + FS);
#pragma unroll
            for (int m = 0; m < MN; ++m)
#pragma unroll
                for (int n = 0; n < NT; ++n) tg[m][n] += cg[m][n], tu[m][n] += cu[m][n];
        }
#pragma unroll
        for (int m = 0; m < MN; ++m)
#pragma unroll
            for (int n = 0; n < NT; ++n) cg[m][n] = tg[m][n] + cgl[m][n], cu[m][n] = tu[m][n] + cul[m][n];
    } else if constexpr (QSPLIT) {
        f32x4 tg[MN][NT], tu[MN][NT], t2g[MN][NT], t2u[MN][NT];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (q) clear();
            steps(q * (nst / 4), (q + 1) * (nst / 4));
#pragma unroll
            for (int m = 0; m < MN; ++m)
#pragma unroll
                for (int n = 0; n < NT; ++n) {
                    if (q == 0) tg[m][n] = cg[m][n], tu[m][n] = cu[m][n];
                    else if (q == 1) tg[m][n] += cg[m][n], tu[m][n] += cu[m][n];
                    else if (q == 2) t2g[m][n] = cg[m][n], t2u[m][n] = cu[m][n];
                    else {
                        cg[m][n] = tg[m][n] + (t2g[m][n] + cg[m][n]);
                        cu[m][n] = tu[m][n] + (t2u[m][n] + cu[m][n]);
                    }
                }
        }
    } else {
        f32x4 tg[MN][NT], tu[MN][NT];
#pragma unroll
        for (int m = 0; m < MN; ++m)
#pragma unroll
            for (int n = 0; n < NT; ++n) tg[m][n] = tu[m][n] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int q = 0; q < 4; ++q) {
            clear();
            steps(q * (nst / 4), (q + 1) * (nst / 4));
#pragma unroll
            for (int m = 0; m < MN; ++m)
#pragma unroll
                for (int n = 0; n < NT; ++n) tg[m][n] += cg[m][n], tu[m][n] += cu[m][n];
        }
#pragma unroll
        for (int m = 0; m < MN; ++m)
#pragma unroll
            for (int n = 0; n < NT; ++n) cg[m][n] = tg[m][n], cu[m][n] = tu[m][n];
    }

    // ---- open gates, active rows: lane (lm, lq), register i holds neuron
    // 16 (wm MN + m) + 4 lq + i, token slot 16 (2 n + wn) + lm
    const float thr = gate_threshold(a.act, a.tau);
    uint32_t abits[MN];  // this lane's active (neuron i, n) pairs: bit 4 n + i
#pragma unroll
    for (int m = 0; m < MN; ++m) {
        uint32_t ob = 0, ab = 0, obits = 0;
        abits[m] = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const bool in = r0 + (wm * MN + m) * 16 + 4 * lq + i < a.I;
            uint64_t mo = 0, ma = 0;
#pragma unroll
            for (int n = 0; n < NT; ++n) {
                const bool tin = 16 * (2 * n + wn) + lm < ng;
                const float gv = cg[m][n][i], uv = cu[m][n][i];
                const bool op = in && tin && gv > thr;
                const bool on = op && combined_nonzero(a.act, uv);
                if (a.dense ? in : op) obits |= 1u << (4 * n + i);
                if (a.dense ? in : on) abits[m] |= 1u << (4 * n + i);
                mo |= __ballot(a.dense ? in : op);
                ma |= __ballot(a.dense ? in : on);
                cg[m][n][i] = on ? combined_value(a.act, a.tau, gv, uv) : 0.f;
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if ((mo >> (16 * q)) & 0xFFFFull) ob |= 1u << (4 * q + i);
                if ((ma >> (16 * q)) & 0xFFFFull) ab |= 1u << (4 * q + i);
            }
        }
        const int mt = wm * MN + m, sh = 16 * (mt & 1);
        if (lane == 0) {
            atomicOr(&s_open[mt >> 1], ob << sh);
            atomicOr(&s_act[mt >> 1], ab << sh);
        }
        if (a.want_masks) {
#pragma unroll
            for (int n = 0; n < NT; ++n) {
                const int t = 16 * (2 * n + wn) + lm;
                atomicOr(&s_gm[mt >> 1][t], ((obits >> (4 * n)) & 15u) << (sh + 4 * lq));
                atomicOr(&s_am[mt >> 1][t], ((abits[m] >> (4 * n)) & 15u) << (sh + 4 * lq));
            }
        }
    }
    __syncthreads();

    // ---- Combined of every active row into its slot (its rank in the tile)
    uint16_t *sh16 = reinterpret_cast<uint16_t *>(s_lds);
#pragma unroll
    for (int m = 0; m < MN; ++m) {
        const int mt = wm * MN + m;
        const uint32_t am = s_act[mt >> 1];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int b = 16 * (mt & 1) + 4 * lq + i;
            if ((am >> b) & 1u) {
                const int slot = __popc(am & ((1u << b) - 1u));
                uint16_t *dst = sh16 + ((mt >> 1) * kBxRows + slot) * (P * TOK);
#pragma unroll
                for (int n = 0; n < NT; ++n) {
                    const int t = 16 * (2 * n + wn) + lm;
                    float v = cg[m][n][i];
#pragma unroll
                    for (int p = 0; p < P; ++p) {
                        dst[p * TOK + t] = (uint16_t)bf16_take<P>(v);
                    }
                }
            }
        }
    }
    __syncthreads();
    constexpr int RC = P * TOK / 8;  // 16-byte chunks per record
    for (int h = 0; h < nsub; ++h) {
        const uint32_t am = s_act[h];
        const int na = __popc(am);
        u32x4 *hdst = reinterpret_cast<u32x4 *>(a.hfrag) + (tix0 + h) * (kBxRows * RC);
        for (int e = tid; e < na * RC; e += kWdThreads) hdst[e] = s_lds[h * kBxRows * RC + e];
        if (tid < kBxRows)  // an empty tile lists row 0 (always < I), never used
            a.arow[(tix0 + h) * kBxRows + tid] = na > 0 ? (uint8_t)nth_set_bit(am, tid < na ? tid : 0) : (uint8_t)0;
        if (tid == 0) {
            a.cnt[(tix0 + h) * 2] = __popc(s_open[h]);
            a.cnt[(tix0 + h) * 2 + 1] = na;
        }
        if (a.want_masks)
            for (int t = tid; t < TOK; t += kWdThreads) {
                a.gmask[(tix0 + h) * TOK + t] = s_gm[h][t];
                a.amask[(tix0 + h) * TOK + t] = s_am[h][t];
            }
    }
}

// ---------------------------------------------------------------------------
// Down: workgroup (group, chunk of tiles, slice of CW columns) x all token
// slots.  The chunk's active rows are listed as in bx_down and cut into K
// blocks of 32; a block's W_down_t rows and Combined records go through LDS
// (rows padded by 32 bytes, so a transposing read's four rows start on
// different banks).  Waves: WC along the columns x 8 / WC along the tokens.
template <int TOK, int P, int CW, int WC, int KS, int D, int MAXT, bool STREAM, bool AHEAD>
__global__ __launch_bounds__(kWdThreads, 2) void wd_down(BxArgs a) {
    constexpr int WT = 8 / WC;
    constexpr int NC = CW / 16 / WC, NT = TOK / 16 / WT;  // tiles per wave
    constexpr int KB = KS * kBxRows;                          // listed rows per block
    constexpr int WCH = KB * CW / 8, HCH = KB * P * TOK / 8;  // 16-byte chunks per block
    constexpr int NW = WCH / kWdThreads, NH = (HCH + kWdThreads - 1) / kWdThreads;
    constexpr int WP = CW + 16, HP = P * TOK + 16;  // LDS row pitches (elements)
    static_assert(KS <= 2 && WCH % kWdThreads == 0 && NC >= 1 && NT >= 1, "whole chunks per thread");
    __shared__ __attribute__((aligned(16))) uint16_t s_w[2][KB * WP], s_h[2][KB * HP];
    __shared__ uint32_t s_ent[(MAXT + KS - 1) * kBxRows];  // (tile within the chunk) << 10 | slot << 5 | row, or kPadRow
    __shared__ int s_pre[MAXT + 1];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lm = lane & 15, lq = lane >> 4;
    const int wc = wave % WC, wtk = wave / WC;
    // Work item (group, chunk, slice): the slices of a (group, chunk) pair on
    // one XCD (its Combined records and list in one L2); for groups sharing
    // a weight set (a.topk null) all groups of a chunk as well (its rows).
    const int share = a.topk ? 1 : a.vpe;
    const int nitem = a.nslices * share, npairs = a.G / share * a.nchunks;
    const int q = blockIdx.x % 8, r = blockIdx.x / 8;
    const int j8 = r / nitem, it = r % nitem;
    const int pair = 8 * j8 + ((q - j8) & 7);
    if (pair >= npairs) return;
    const int slice = it % a.nslices;
    const int chunk = pair % a.nchunks;
    const int gs = pair / a.nchunks;
    const int g = a.topk ? bx_group_at(gs, a.G, a.vpe) : gs * share + it / a.nslices;
    const int ng = a.gcount[g];
    if (ng == 0) return;
    const int H = a.H;
    const int t0 = chunk * a.tpc;
    const int ntc = min(a.tpc, a.ntiles - t0);
    const size_t tbase = (size_t)g * a.ntiles + t0;

    const int nblk = bx_list_rows<kWdThreads, KB>(a, tbase, ntc, s_pre, s_ent);

    const uint16_t *wde = reinterpret_cast<const uint16_t *>(a.wd) + (size_t)(g / a.vpe) * a.expert_stride;
    const __amdgpu_buffer_rsrc_t rwd = make_rsrc(wde, (uint32_t)a.I * (uint32_t)H * 2u);
    const __amdgpu_buffer_rsrc_t rh =
        make_rsrc(a.hfrag + tbase * (kBxRows * P * TOK), (uint32_t)ntc * (kBxRows * P * TOK * 2u));
    const int col0 = slice * CW;

    u32x4 rw[D][NW], rr[D][NH];
    auto issue = [&](int d, int b) {
        const bool bin = b < nblk;
#pragma unroll
        for (int j = 0; j < NW; ++j) {
            const int idx = tid + kWdThreads * j, row = idx / (CW / 8), c = col0 + 8 * (idx % (CW / 8));
            const uint32_t e = bin ? s_ent[b * KB + row] : kPadRow;
            const uint32_t n = (uint32_t)(t0 + (int)(e >> 10)) * kBxRows + (e & 31u);
            rw[d][j] = wd_ld<STREAM>(rwd, e != kPadRow && c < H ? (n * (uint32_t)H + (uint32_t)c) * 2u : kWdOob);
        }
#pragma unroll
        for (int j = 0; j < NH; ++j) {
            const int idx = tid + kWdThreads * j, row = idx / (P * TOK / 8), c = idx % (P * TOK / 8);
            const bool in = bin && (HCH % kWdThreads == 0 || idx < HCH);
            const uint32_t e = in ? s_ent[b * KB + row] : kPadRow;
            rr[d][j] = ld_buf_cached(rh, e != kPadRow ? (e >> 5) * (P * TOK * 2u) + 16u * (uint32_t)c : kWdOob);
        }
    };
    auto stash = [&](int d, int buf) {
#pragma unroll
        for (int j = 0; j < NW; ++j) {
            const int idx = tid + kWdThreads * j;
            *reinterpret_cast<u32x4 *>(&s_w[buf][idx / (CW / 8) * WP + 8 * (idx % (CW / 8))]) = rw[d][j];
        }
#pragma unroll
        for (int j = 0; j < NH; ++j) {
            const int idx = tid + kWdThreads * j;
            if (HCH % kWdThreads == 0 || idx < HCH)
                *reinterpret_cast<u32x4 *>(&s_h[buf][idx / (P * TOK / 8) * HP + 8 * (idx % (P * TOK / 8))]) = rr[d][j];
        }
    };
    constexpr bool LO = P == 3;  // the lower parts' sums apart, as in wd_gate_up
    f32x4 acc[NC][NT], accl[LO ? NC : 1][LO ? NT : 1];
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int n = 0; n < NT; ++n) acc[c][n] = accl[LO ? c : 0][LO ? n : 0] = f32x4{0.f, 0.f, 0.f, 0.f};
    // fragments of k-step s of a stage in register slot `slot`
    u32x4 wf[2][NC], hf[2][NT * P];
    // the wave's n-tiles are wtk, wtk + WT, ...
    auto load = [&](int buf, int s, int slot, auto nac) {
        constexpr int NACT = decltype(nac)::value;
        if constexpr (NACT > 0) {
#pragma unroll
            for (int c = 0; c < NC; ++c)
                wf[slot][c] = wd_tr_frag(&s_w[buf][s * kBxRows * WP + 16 * (wc * NC + c)], WP, lane);
        }
#pragma unroll
        for (int n = 0; n < NACT; ++n)
#pragma unroll
            for (int p = 0; p < P; ++p)
                hf[slot][P * n + p] =
                    wd_tr_frag(&s_h[buf][s * kBxRows * HP + p * TOK + 16 * (n * WT + wtk)], HP, lane);
    };
    auto contract = [&](int slot, auto nac) {
        constexpr int NACT = decltype(nac)::value;
#pragma unroll
        for (int n = 0; n < NACT; ++n)
#pragma unroll
            for (int p = 0; p < P; ++p)
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    f32x4 &v = LO && p ? accl[LO ? c : 0][LO ? n : 0] : acc[c][n];
                    v = mfma_bf16(wf[slot][c], hf[slot][P * n + p], v);
                }
    };
    // The sums are folded into totals every FB blocks (256 listed rows): a
    // chain of roundings spans those, not the whole chunk (two parts, 256
    // tokens: 4.88e-6 instead of 4.93e-6; three parts, a chunk of 7000 active
    // rows: 1.8e-7 instead of 4.2e-7, the single-token kernels' 1.8e-7).  It
    // costs 2 us of 65 at 128 slots and nothing elsewhere.
    constexpr int U = D > 2 ? D : 2, FB = 8 / KS;
    static_assert(FB % U == 0, "whole rounds between folds");
    f32x4 tot[NC][NT];
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int n = 0; n < NT; ++n) tot[c][n] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto blocks = [&](auto nac) {
        constexpr int NACT = decltype(nac)::value;
        constexpr int R = NACT ? 2 * (NC + NACT * P) : 0, M = NC * NACT * P;  // (of a k-step)
        auto spread = [&]() {
            if constexpr (TOK == 128 && NACT > 0) wd_roll<R, 0, NACT * P, NC>();
            else wd_spread<R, 0, M>();
        };
        if constexpr (AHEAD) load(0, 0, 0, nac);
        for (int b0 = 0; b0 < nblk; b0 += FB) {
            const int b1 = min(nblk, b0 + FB);
            for (int b = b0; b < b1; b += U) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if (b + u < nblk) {  // uniform over the workgroup
                        if constexpr (AHEAD && KS == 2) {
                            load(u & 1, 1, 1, nac);
                            contract(0, nac);
                            spread();
                        } else if constexpr (!AHEAD) {
#pragma unroll
                            for (int s = 0; s < KS; ++s) {
                                load(u & 1, s, s, nac);
                                contract(s, nac);
                            }
                        }
                        stash((u + 1) % D, (u + 1) & 1);
                        issue((u + 1) % D, b + u + 1 + D);
                        wd_barrier();
                        if constexpr (AHEAD) {
                            __builtin_amdgcn_sched_barrier(0);
                            load((u + 1) & 1, 0, KS == 2 ? 0 : (u + 1) & 1, nac);
                            contract(KS == 2 ? 1 : u & 1, nac);
                            spread();
                        }
                    }
                }
            }
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int n = 0; n < NACT; ++n) tot[c][n] += acc[c][n], acc[c][n] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    };
    if (nblk > 0) {
#pragma unroll
        for (int d = 0; d < D; ++d) issue(d, d);
        stash(0, 0);
        issue(0, D);
        wd_barrier();
        // n-tiles without tokens are left out, as in wd_gate_up
        const int nact = max(0, ((ng + 15) / 16 - wtk + WT - 1) / WT);
        if (NT >= 4 && nact > 2) blocks(std::integral_constant<int, NT >= 4 ? 4 : NT>{});
        else if (NT >= 2 && nact > 1) blocks(std::integral_constant<int, NT >= 2 ? 2 : NT>{});
        else if (nact > 0) blocks(std::integral_constant<int, 1>{});
        else blocks(std::integral_constant<int, 0>{});
    }
    // lane (lm, lq): columns 4 lq .. 4 lq + 3 of a 16-column tile, token lm
#pragma unroll
    for (int n = 0; n < NT; ++n) {
        const int t = 16 * (n * WT + wtk) + lm;
        if (t < ng) {
            float *prow = a.partial + (((size_t)g * TOK + t) * a.nchunks + chunk) * H;
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                const int col = col0 + 16 * (wc * NC + c) + 4 * lq;
                if (col < H)
                    *reinterpret_cast<f32x4 *>(prow + col) = LO ? tot[c][n] + accl[LO ? c : 0][LO ? n : 0] : tot[c][n];
            }
        }
    }
}

// ---------------------------------------------------------------------------

namespace {

template <int TOK, int P, int NB, int D, bool AHEAD>
void launch_wide_gate(const BatchPlan &p, const BxArgs &a, hipStream_t st) {
    const int nwt = (p.ntiles + NB / kBxRows - 1) / (NB / kBxRows);
    const dim3 grid((unsigned)((nwt + 7) / 8 * 8 * p.groups));
    if constexpr (wd_many_groups(TOK, P)) {
        if (p.groups > 1) {
            launch("batch_gate_up", wd_gate_up<TOK, P, NB, D, false, false, AHEAD>, grid, dim3(kWdThreads), st, a);
            return;
        }
    }
    launch("batch_gate_up", wd_gate_up<TOK, P, NB, D, false, true, AHEAD>, grid, dim3(kWdThreads), st, a);
}

template <int TOK, int P, int NB, int D, bool AHEAD>
void launch_wide_gate_moe(const BatchPlan &p, const BxArgs &a, hipStream_t st) {
    const int nwt = (p.ntiles + NB / kBxRows - 1) / (NB / kBxRows);
    launch("batch_gate_up", wd_gate_up<TOK, P, NB, D, true, true, AHEAD>, dim3((unsigned)(p.groups * nwt)), dim3(kWdThreads),
           st, a);
}

template <int TOK, int P, int CW, int WC, int KS, int D, int MAXT, bool AHEAD>
void launch_wide_down_cw(const BatchPlan &p, const BxArgs &a, hipStream_t st) {
    const int share = a.topk ? 1 : p.vpe;
    const dim3 dgrid((unsigned)((p.groups / share * p.nchunks + 7) / 8 * 8 * p.nslices * share));
    if constexpr (wd_many_groups(TOK, P)) {
        if (share > 1) {
            launch("batch_down", wd_down<TOK, P, CW, WC, KS, D, MAXT, false, AHEAD>, dgrid, dim3(kWdThreads), st, a);
            return;
        }
    }
    launch("batch_down", wd_down<TOK, P, CW, WC, KS, D, MAXT, true, AHEAD>, dgrid, dim3(kWdThreads), st, a);
}

}  // namespace

void launch_wide_prep(const BatchPlan &p, const BxArgs &a, hipStream_t st) {
    const dim3 grid((unsigned)((p.groups * (p.hpad / 32) * (p.tok / 16) * 64 + 255) / 256));
    if (p.parts == 3) {
        launch("batch_prep", wd_prep<64, 3>, grid, dim3(256), st, a);
        return;
    }
    switch (p.tok) {
    case 32: launch("batch_prep", wd_prep<32, 2>, grid, dim3(256), st, a); break;
    case 64: launch("batch_prep", wd_prep<64, 2>, grid, dim3(256), st, a); break;
    default: launch("batch_prep", wd_prep<128, 2>, grid, dim3(256), st, a); break;
    }
}

// Stages in flight, rows and columns per workgroup as measured on the
// Mistral shape (gate + up / down in us): 32 tokens 43 / 25.5 (bx_gate_up64
// and bx_down 58.0 / 28.8), 64 tokens 52 / 33 (85.8 / 42.7), 256 tokens
// 107 / 67 (four passes of 64: 327 / 168).  More stages in flight changed
// nothing (gate + up) or lost (down, two stages: 41 at 64 tokens, 79 at 256);
// with 128 neurons and 128 slots a second stage does not fit the registers
// (spills in the loop: 157 us).
// At 128 slots a workgroup takes 64 neurons where 128 leave fewer than 192
// workgroups for the 256 compute units: 128 tokens, 110 -> 71 us (two groups,
// 224 workgroups of 128 neurons: each x stage serves twice the weights, 107
// us against 128 with 64).
// Operands a k-step ahead (the last flag): 256 tokens 115 -> 102 us; not at
// 32 slots (131 registers leave one workgroup per unit instead of two) nor in
// the MoE form (spills).
void launch_wide_gate_up(const BatchPlan &p, const BxArgs &a, hipStream_t st) {
    if (p.parts == 3 && a.topk) launch_wide_gate_moe<64, 3, 128, 1, false>(p, a, st);
    else if (p.parts == 3) launch_wide_gate<64, 3, 64, 1, true>(p, a, st);
    else if (p.tok == 128 && p.groups * p.ntiles < 4 * 192) launch_wide_gate<128, 2, 64, 2, true>(p, a, st);
    else if (p.tok == 128) launch_wide_gate<128, 2, 128, 1, true>(p, a, st);
    else if (p.tok == 64) launch_wide_gate<64, 2, 64, 2, true>(p, a, st);
    else launch_wide_gate<32, 2, 64, 4, false>(p, a, st);
}

void launch_wide_down(const BatchPlan &p, const BxArgs &a, hipStream_t st) {
    if (p.parts == 3) launch_wide_down_cw<64, 3, 256, 4, 1, 2, wd_down_tiles(64, 3), true>(p, a, st);
    else if (p.tok == 128) launch_wide_down_cw<128, 2, 256, 4, 2, 1, wd_down_tiles(128, 2), true>(p, a, st);
    else if (p.tok == 64) launch_wide_down_cw<64, 2, 128, 4, 2, 1, wd_down_tiles(64, 2), true>(p, a, st);
    else launch_wide_down_cw<32, 2, 128, 8, 2, 1, wd_down_tiles(32, 2), true>(p, a, st);
}

}  // namespace ts
