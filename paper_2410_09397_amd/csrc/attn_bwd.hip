// Fused backward kernels for d <= 256 (the regime where a d x d working set fits on chip; d = 256
// runs with one wave per SIMD and up to 512 registers per lane):
//   dQ      : one workgroup owns a block of 128 queries and streams key tiles; its prologue also
//             forms delta = rowsum(dO o O) (second matrix form of p, App. B.4) for those queries
//   dK, dV  : one workgroup owns a block of 64 keys and streams query tiles
//   calls of few blocks run both kinds of blocks side by side in one launch (bwd_both_kernel), with delta from a small
//   launch in front (bwd_rows_kernel), short ones alone, with delta formed in every block (bwd_short_kernel); blocks that
//   have a CU to themselves get eight waves, two groups that take the tiles in turn (bwd_*_eight_kernel); the rules are in
//   attn_rules.hpp and attn_common.hpp.  delta_kernel serves the large-d path
// Per tile pair this is the inner body of the paper's large-cache phase-2 algorithm (App. D):
// q = dO h^T, A = S A_2^T, f = exp(A) / l, p = f o q - diag(v) f, followed by the three
// products that use f and p.  The resident operand is the owned block, so dK/dV (resp. dQ)
// accumulate in registers with no atomics and no n x n matrix ever leaves the chip.
#include <type_traits>

#include "attn_common.hpp"
#include "attn_internal.hpp"
#include "attn_rules.hpp"

namespace attn {

// --------------------------------------------------------------------------------- delta
// min(d / 8, 64) consecutive lanes share one row (16-byte chunks; a lane takes every 64th chunk when
// the row has more than 64); the row sum is a shuffle reduction inside that lane group.  d / 8 must
// be a power of two.
__global__ void __launch_bounds__(kThreads) delta_kernel(FusedParams p, int d) {
    const int cpr = d >> 3;             // chunks per row
    const int lpr = cpr < 64 ? cpr : 64;  // lanes per row
    const long rows = (long)p.batch * p.heads * p.n;
    const long f = (long)blockIdx.x * kThreads + threadIdx.x;
    const long r = f / lpr;
    const int c = (int)(f % lpr);
    float acc = 0.f;
    if (r < rows) {
        const int bh = (int)(r / p.n), i = (int)(r % p.n);
        const long off = (long)(bh / p.heads) * p.stride_b + (long)(bh % p.heads) * p.stride_h + (long)i * p.stride_n;
        for (int cc = c; cc < cpr; cc += lpr) {
            const bf16x8 o = *reinterpret_cast<const bf16x8*>(p.O + off + cc * 8);
            const bf16x8 g = *reinterpret_cast<const bf16x8*>(p.dO + off + cc * 8);
#pragma unroll
            for (int t = 0; t < 8; ++t) acc += (float)o[t] * (float)g[t];
        }
    }
    for (int m = lpr >> 1; m >= 1; m >>= 1) acc += __shfl_xor(acc, m, 64);
    if (r < rows && c == 0) p.delta[r] = acc;
}

// --------------------------------------------------------------------------- block order
// order[r] = the block with the r-th longest list (ties: lower index first).  Workgroups are
// dispatched in index order, so taking the long lists first keeps the tail of a launch short
// when the lists of a block mask differ in length, and workgroups that run at the same time walk
// through the streamed blocks together (their re-reads then hit in L2).  Two steps: the list
// lengths that count (entries the causal rule removes do not), then one thread per block ranks
// its length against all others (nblk^2 comparisons).
__global__ void __launch_bounds__(kThreads) block_len_kernel(const int32_t* ptr_all, const int32_t* idx, int nblk,
                                                            int causal, int column_lists, int32_t* len_all) {
    const int i = blockIdx.x * kThreads + threadIdx.x;
    if (i >= nblk) return;
    const int32_t* ptr = ptr_all + (long)blockIdx.y * (nblk + 1);  // mask blockIdx.y
    int32_t* len = len_all + (long)blockIdx.y * nblk;
    const int first = ptr[i];
    int count = ptr[i + 1] - first;
    if (causal) {
        if (column_lists) count -= causal_col_skip(idx, first, count, i);
        else count = causal_row_entries(idx, first, count, i);
    }
    len[i] = count;
}
__global__ void __launch_bounds__(kThreads) block_order_kernel(const int32_t* len_all, int nblk, int32_t* order_all) {
    const int i = blockIdx.x * kThreads + threadIdx.x;
    if (i >= nblk) return;
    const int32_t* len = len_all + (long)blockIdx.y * nblk;
    int32_t* order = order_all + (long)blockIdx.y * nblk;
    const int mine = len[i];
    int rank = 0;
    for (int k = 0; k < nblk; ++k) {
        const int other = len[k];
        rank += (other > mine || (other == mine && k < i)) ? 1 : 0;
    }
    order[rank] = i;
}

// Both steps, for the row lists and the column lists of a mask, in one launch when a mask has at most
// kOrderFusedBlocks blocks: workgroup (mask, kind) keeps the lengths in LDS and ranks them there (four small
// launches in front of the backward kernels cost as much as 2 % of a block-sparse call).
constexpr int kOrderFusedBlocks = 256;
struct OrderParams {
    const int32_t *row_ptr, *col_idx, *col_ptr, *row_idx;
    int32_t *order_q, *order_k;
    int nblk, causal;
};
// kind 0: row lists (query blocks), 1: column lists (key blocks)
__device__ __forceinline__ void rank_blocks(const OrderParams& p, int mask, int kind, int32_t* len) {
    const int nblk = p.nblk, causal = p.causal;
    const int32_t* ptr = (kind ? p.col_ptr : p.row_ptr) + (long)mask * (nblk + 1);
    const int32_t* idx = kind ? p.row_idx : p.col_idx;
    int32_t* order = (kind ? p.order_k : p.order_q) + (long)mask * nblk;
    for (int i = threadIdx.x; i < nblk; i += kThreads) {
        const int first = ptr[i];
        int count = ptr[i + 1] - first;
        if (causal) {
            if (kind) count -= causal_col_skip(idx, first, count, i);
            else count = causal_row_entries(idx, first, count, i);
        }
        len[i] = count;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < nblk; i += kThreads) {
        const int mine = len[i];
        int rank = 0;
        for (int k = 0; k < nblk; ++k) {
            const int other = len[k];
            rank += (other > mine || (other == mine && k < i)) ? 1 : 0;
        }
        order[rank] = i;
    }
}
__global__ void __launch_bounds__(kThreads) block_order_fused_kernel(OrderParams p, int first_kind) {
    __shared__ int32_t len[kOrderFusedBlocks];
    rank_blocks(p, blockIdx.x, first_kind + blockIdx.y, len);
}

// v = rowsum(dO o O) of a row (0 past n) by two lanes, 32 apart, in the order of the dQ kernel.
template <int D>
__device__ __forceinline__ float row_dot(const FusedParams& p, long base, int row, int h) {
    float dsum = 0.f;
    if (row < p.n) {
        const long off = base + (long)row * p.stride_n + 8 * h;
        bf16x8 o[D / 16], g[D / 16];
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks) {
            o[ks] = *reinterpret_cast<const bf16x8*>(p.O + off + 16 * ks);
            g[ks] = *reinterpret_cast<const bf16x8*>(p.dO + off + 16 * ks);
        }
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks)
#pragma unroll
            for (int e = 0; e < 8; ++e) dsum += (float)o[ks][e] * (float)g[ks][e];
    }
    return dsum + __shfl_xor(dsum, 32, 64);
}

// What the two halves of the backward need when they run side by side: v = rowsum(dO o O), and the block orders of the
// masks (`orders` workgroups: both kinds of a mask one after the other).  Two lanes per row with the sum in the dQ kernel's order, so that the
// bits of v do not depend on which of the two formed it.
template <int D>
__global__ void __launch_bounds__(kThreads) bwd_rows_kernel(FusedParams p, OrderParams op, int orders) {
    __shared__ int32_t len[kOrderFusedBlocks];
    if ((int)blockIdx.x < orders) {
        rank_blocks(op, blockIdx.x >> 1, blockIdx.x & 1, len);
        return;
    }
    const int lane = threadIdx.x & 63, h = lane >> 5;
    const long rows = (long)p.batch * p.heads * p.n;
    const long r = ((long)(blockIdx.x - orders) * (kThreads / 64) + (threadIdx.x >> 6)) * 32 + (lane & 31);
    const int bh = r < rows ? (int)(r / p.n) : 0;
    const long base = (long)(bh / p.heads) * p.stride_b + (long)(bh % p.heads) * p.stride_h;
    const float dsum = row_dot<D>(p, base, r < rows ? (int)(r - (long)bh * p.n) : p.n, h);
    if (r < rows && h == 0) p.delta[r] = dsum;
}

// ------------------------------------------------------------------------------- dK, dV
// A workgroup owns 64 keys and streams 64-query tiles; per tile its 4 waves work in two phases:
//   phase 1: wave (wk, wx) computes S^T and dP^T for key half wk and query half wx, with the
//            resident K / V fragments as A operands (lane <-> query, so lse2 and delta are
//            per-lane scalars), then P and dS go to LDS as bf16 tiles [query][key];
//   phase 2: wave (wk, wx) accumulates dV^T (wx = 0) or dK^T (wx = 1) for the d-half wk and all
//            64 keys over the 64 queries, as a block of accumulators in which every fragment
//            read from LDS feeds two MFMAs; P / dS (B operands) and dO^T / Q^T (A operands)
//            are all read with transposing LDS loads.
// Keeping K, V and both gradients of 128 keys in the registers of one workgroup instead (no LDS
// round trip for P and dS) needs more than 256 registers per lane at d = 128, i.e. one wave per
// SIMD; that variant was measured at 60 % of this one's speed at d = 128 and 91 % at d = 64.
// Wave priorities per phase: the two waves that share a SIMD compete for one matrix pipe and
// fall into step; ranking phase 1 above phase 2 above the exponentials lets one of them run ahead
// (measured: 2 % faster than without priorities, 3 % faster than with the exponentials in the middle).
constexpr int kPrioPhase1 = 3, kPrioSoftmax = 0, kPrioPhase2 = 1;
template <int D, int NG = 1, bool OWN = false>
__device__ __forceinline__ void dkdv_block(const FusedParams& p, char* lds, int bh, int j) {
    constexpr int BR = 64, BC = 64, KS = D / 16, MT = D / 32;
    constexpr int kTileBytes = BR * D * 2;
    constexpr int kStageBytes = 2 * kTileBytes;
    constexpr int kPBytes = BC * BR * 2;

    // NG = 2: two groups of four waves, each with stages and P / dS tiles of its own, take the streamed tiles in turn (eight_waves_bwd)
    const int group = NG == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / kThreads);
    char* smem = lds + group * (2 * kStageBytes + 2 * kPBytes);
    const int tid = threadIdx.x % kThreads, lane = tid & 63, h = lane >> 5, l32 = lane & 31;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave index within the group, uniform
    const int wk = w & 1, wx = w >> 1;
    if (p.order) {
        j = 2 * p.order[(long)bh * p.order_stride + (j >> 1)] + (j & 1);
        if (j * BC >= p.n) return;
    }
    const long base = (long)(bh / p.heads) * p.stride_b + (long)(bh % p.heads) * p.stride_h;
    const long ld = p.stride_n;
    const int j0 = j * BC;
    const float* lse_g = p.LSE + (long)bh * p.n;
    const float* delta_g = p.delta + (long)bh * p.n;

    int n_it, t0 = 0, lp0 = 0;
    if (p.list_ptr) {
        const int32_t* lptr = p.list_ptr + (long)bh * p.list_stride;  // this (batch, head)'s mask
        lp0 = lptr[j0 / 128];
        int entries = lptr[j0 / 128 + 1] - lp0;
        if (p.causal) {
            const int skip = causal_col_skip(p.list_idx, lp0, entries, j0 / 128);
            lp0 += skip;
            entries -= skip;
        }
        n_it = entries * (128 / BR);
    } else {
        t0 = p.causal ? j0 / BR : 0;
        n_it = (p.n + BR - 1) / BR - t0;
    }
    const int n_all = n_it;
    if constexpr (NG > 1) n_it = (n_all - group + NG - 1) / NG;  // this group's tiles: every NG-th, from `group` on
    auto tile_start = [&](int it) -> int { return tile_start_row<BR>(p.list_idx, lp0, t0, NG * it + group); };

    // phase-2 role of this wave: wx = 0 accumulates dV^T (from P and dO^T), wx = 1 dK^T (from dS
    // and Q^T), each for all 64 keys and the half wk of d: a 2 x 2 block of accumulators, so that
    // every fragment read from LDS feeds two MFMAs
    constexpr int MH = MT / 2;
    f32x16 acc[MH][2];
#pragma unroll
    for (int m = 0; m < MH; ++m)
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[m][kt][i] = 0.f;

    const float c = p.scale * kLog2e;
    // Row i0 + 32 wx + l32 of the tile being fetched.  The loaded values are not touched until
    // the next iteration, so nothing waits on the copies in flight behind them.
    float lse_raw = 0.f, delta_raw = 0.f;
    bool row_ok = false;
    TileLoader<D, BR> loader;
    loader.init(tid, ld);
    auto fetch_rows = [&](int i0) {
        const int q = i0 + 32 * wx + l32;
        row_ok = q < p.n;
        lse_raw = lse_g[min(q, p.n - 1)];
        if constexpr (!OWN) delta_raw = delta_g[min(q, p.n - 1)];
    };
    auto fetch = [&](int i0, int stage_off) {
        char* s = smem + stage_off;
        loader.load(p.Q + base, ld, i0, p.n, s, tid);
        loader.load(p.dO + base, ld, i0, p.n, s + kTileBytes, tid);
        fetch_rows(i0);
    };
    // The resident K and V rows come through the second stage, which is free until the first tile is worked on: read straight from
    // memory as operands, every load takes 16 bytes from each of 64 places, and a workgroup stood 3 to 5 us in front of its first tile.
    // Rows past n repeat the last row; their gradients are not stored.  The gradients leave through LDS as well (8-byte pieces of 32 rows
    // before).  us of the kernel, before -> now: d = 64 b4 h16 n2048 158 -> 154   d = 128 b2 h16 n1024 causal 28.6 -> 26.0,
    // b2 h32 n8192 causal 2157 -> 2108   d = 256 h8 n1000 37.3 -> 32.9, b2 h23 n97 causal 14.9 -> 10.5
    int i0_next = n_it > 0 ? tile_start(0) : 0;
    loader.load(p.K + base, ld, j0, p.n, smem + kStageBytes, tid);  // (every group for itself)
    loader.load(p.V + base, ld, j0, p.n, smem + kStageBytes + kTileBytes, tid);
    if (n_it > 0) fetch(i0_next, 0);
    // OWN: v = rowsum(dO o O) of every query that these keys see, formed here (with the bits of bwd_rows_kernel) and kept behind the stages
    float* own_delta = reinterpret_cast<float*>(lds + NG * (2 * kStageBytes + 2 * kPBytes));
    if constexpr (OWN)
        for (int r0 = BR * t0 + 32 * (w + 4 * group); r0 < p.n; r0 += 32 * 4 * NG) {
            const float v = row_dot<D>(p, base, r0 + l32, h);
            if (h == 0 && r0 + l32 < p.n) own_delta[r0 + l32] = v;
        }
    FragOffsets<D> fo;    // Q / dO tiles
    FragOffsets<BC> fp;   // P / dS tiles
    fo.init(lane);
    fp.init(lane);
    wait_direct_loads();
    __syncthreads();
    bf16x8 kf[KS], vf[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        kf[ks] = fo.frag(smem, kStageBytes, 32 * wk, ks);
        vf[ks] = fo.frag(smem, kStageBytes + kTileBytes, 32 * wk, ks);
    }
    lds_barrier();  // (the first tile's copies go into that stage)
    constexpr int kPOff = 2 * kStageBytes, kDsOff = kPOff + kPBytes;
    // This lane's 8-byte slot of group g in the [query][key] tiles: p_wr ^ (g << 4).  The two
    // 8-byte halves of a chunk swap places in odd rows: rows 2k and 2k+1 share their swizzle
    // term and are 128 bytes apart, so without the swap the 16 lanes that write together would
    // hit every bank twice.  The transposed reads apply the same swap per lane.
    const int p_wr = tile_off<BC>(32 * wx + l32, 4 * wk) + 8 * (h ^ (l32 & 1));
    fp.tr0 ^= (((lane & 15) >> 2) & 1) << 3;
    // Address registers of everything this wave reads from or writes to LDS, relative to the
    // stage (all wave-dependent tile choices folded in): a fetch is then a register plus an
    // immediate, with no vector arithmetic in the loop.
    //   q_rm[ks]     Q rows 32 wx + l32 (phase 1; the dO tile is kTileBytes further)
    //   a_tr[m][.]   phase-2 A operand: dO^T (wx = 0) or Q^T (wx = 1), columns 32 (MH wk + m) ..
    //   b_tr[kt][.]  phase-2 B operand: P (wx = 0) or dS (wx = 1), keys 32 kt ..
    //   p_slot[g]    this lane's slot in the P tile (the dS tile is kPBytes further)
    int q_rm[KS], a_tr[MT / 2][2], b_tr[2][2], p_slot[4];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) q_rm[ks] = fo.rm(ks) + 32 * wx * (D * 2);
#pragma unroll
    for (int half = 0; half < 2; ++half) {
#pragma unroll
        for (int m = 0; m < MT / 2; ++m) a_tr[m][half] = fo.tr((MT / 2) * wk + m, half) + (wx == 0 ? kTileBytes : 0);
#pragma unroll
        for (int kt = 0; kt < 2; ++kt) b_tr[kt][half] = fp.tr(kt, half) + (wx == 0 ? kPOff : kDsOff);
    }
#pragma unroll
    for (int g = 0; g < 4; ++g) p_slot[g] = kPOff + (p_wr ^ (g << 4));
    // One streamed query tile (two barriers).  `masked` selects the copy of phase 1 that applies
    // the causal bound.
    auto tile = [&](auto stage_off, int it, int i0, bool skip, auto masked) {
        const float lse_cur = row_ok ? lse_raw * kLog2e : __builtin_inff();
        const float delta_cur = row_ok ? (OWN ? own_delta[i0 + 32 * wx + l32] : delta_raw) : 0.f;
        const int q_off = stage_off;  // Q tile; the dO tile follows it
        // The copies of the next tile go into the stage that was last read before barrier B of the
        // previous tile.  In the mask-free body they are issued one by one between the MFMAs of
        // phase 1 (a wave that issues all of them at once waits until the copy path, 64 B per
        // cycle and CU, has taken them: ~750 cycles per tile in front of the first MFMA; 1.5 % faster).
        bool spread = false;
        const __bf16* next_q = nullptr;
        const __bf16* next_g = nullptr;
        char* next_stage = smem + (kStageBytes - q_off);
        if (it + 1 < n_it) {
            i0_next = tile_start(it + 1);
            spread = !decltype(masked)::value && !skip && i0_next + BR <= p.n;
            if (spread) {
                next_q = p.Q + base + (long)i0_next * ld;
                next_g = p.dO + base + (long)i0_next * ld;
                loader.hold(next_q);
                loader.hold(next_g);
                fetch_rows(i0_next);
            } else {
                fetch(i0_next, kStageBytes - q_off);
            }
        }
        __builtin_amdgcn_s_setprio(kPrioPhase1);
        if (!skip) {
            // ---- phase 1: S^T, dP^T for (key half wk) x (query half wx); the resident K / V
            // fragments serve as A operands, so a lane holds one query and lse2 / delta are scalars
            f32x16 s, dp;
#pragma unroll
            for (int i = 0; i < 16; ++i) { s[i] = 0.f; dp[i] = 0.f; }
            {
                // Q and dO fragments are requested kAhead k-steps before the MFMAs that use them
                // (left to itself the compiler requests each pair right in front of its MFMAs and
                // every pair waits out the LDS latency: measured 3 % slower)
                constexpr int kAhead = 2;
                bf16x8 fq[KS], fg[KS];
#pragma unroll
                for (int ks = 0; ks < kAhead; ++ks) {
                    fq[ks] = FragOffsets<D>::read(smem, q_rm[ks], q_off);
                    fg[ks] = FragOffsets<D>::read(smem, q_rm[ks], q_off + kTileBytes);
                }
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {  // two independent accumulation chains, interleaved
                    __builtin_amdgcn_sched_barrier(0);
                    if (ks + kAhead < KS) {
                        fq[ks + kAhead] = FragOffsets<D>::read(smem, q_rm[ks + kAhead], q_off);
                        fg[ks + kAhead] = FragOffsets<D>::read(smem, q_rm[ks + kAhead], q_off + kTileBytes);
                    }
                    s = mfma32(kf[ks], fq[ks], s);
                    dp = mfma32(vf[ks], fg[ks], dp);
                    if (spread) {  // 2 kInst copies over KS k-steps: one per step for d = 64 and 128
                        constexpr int kPer = TileLoader<D, BR>::kInst;
                        static_assert(2 * kPer == KS, "one copy per k-step");
                        if (ks < kPer) loader.load_one(ks, next_q, next_stage);
                        else loader.load_one(ks - kPer, next_g, next_stage + kTileBytes);
                    }
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_setprio(kPrioSoftmax);
            // key j0 + 32 wk + 8g + 4h + r is visible to this lane's query iff 8g + r <= lim
            // (the masked body also serves unpaired tiles of unmasked runs)
            const int lim = p.causal ? i0 + 32 * wx + l32 - j0 - 32 * wk - 4 * h : 0x7fffffff;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                float pv[4], dsv[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int i = 4 * g + r;
                    float v = __builtin_amdgcn_exp2f(s[i] * c - lse_cur);
                    if constexpr (decltype(masked)::value) v = (8 * g + r > lim) ? 0.f : v;
                    pv[r] = v;
                    dsv[r] = v * (dp[i] - delta_cur);
                }
                // [query][key] tiles: four consecutive keys of this lane's query
                u32x2 a, b;
                a[0] = pack_bf16(pv[0], pv[1]);
                a[1] = pack_bf16(pv[2], pv[3]);
                b[0] = pack_bf16(dsv[0], dsv[1]);
                b[1] = pack_bf16(dsv[2], dsv[3]);
                *reinterpret_cast<u32x2*>(smem + p_slot[g]) = a;
                *reinterpret_cast<u32x2*>(smem + p_slot[g] + kPBytes) = b;
            }
        }
        lds_barrier();  // P, dS visible; the tile copies for the next iteration stay in flight
        __builtin_amdgcn_s_setprio(kPrioPhase2);
        if (!skip) {
            // ---- phase 2: dV^T = dO^T P (wx = 0) or dK^T = Q^T dS (wx = 1) for d half wk over the
            // 64 queries and 64 keys
            bf16x8 at[2][MH], bt[2][2];
            auto request = [&](int ks) {
#pragma unroll
                for (int m = 0; m < MH; ++m)
                    at[ks & 1][m] = FragOffsets<D>::read_t(smem, a_tr[m][0], a_tr[m][1], 16 * ks, q_off);
#pragma unroll
                for (int kt = 0; kt < 2; ++kt)
                    bt[ks & 1][kt] = FragOffsets<BC>::read_t(smem, b_tr[kt][0], b_tr[kt][1], 16 * ks);
            };
            request(0);
#pragma unroll
            for (int ks = 0; ks < BR / 16; ++ks) {  // fragments of the next 16 queries requested ahead
                if (ks + 1 < BR / 16) request(ks + 1);
#pragma unroll
                for (int m = 0; m < MH; ++m)
#pragma unroll
                    for (int kk = 0; kk < 2; ++kk) {
                        // boustrophedon order: consecutive MFMAs share an operand (A, then B, then A);
                        // with both operands changing between the second and third one the kernel
                        // measured 3 % slower
                        const int kt = (m & 1) ? 1 - kk : kk;
                        acc[m][kt] = mfma32(at[ks & 1][m], bt[ks & 1][kt], acc[m][kt]);
                    }
            }
        }
        wait_direct_loads();
        __syncthreads();
    };
    // Query tiles come in ascending order: under the causal rule the ones that straddle the
    // diagonal (or lie wholly above it) are the first, then everything is visible.  The visible
    // ones go two at a time through a body whose LDS stage offsets are compile-time constants;
    // the masked body (run-time stage) also takes the tile that makes the pairs start at an even
    // index and the one left over at the end.
    int it = 0;
    for (; it < n_it; ++it) {
        const int i0 = i0_next;
        if (!(p.causal && i0 < j0 + BC - 1) && !(it & 1)) break;
        tile((it & 1) * kStageBytes, it, i0, i0 + BR - 1 < j0, std::true_type{});
    }
    for (; it + 2 <= n_it; it += 2) {
        tile(std::integral_constant<int, 0>{}, it, i0_next, false, std::false_type{});
        tile(std::integral_constant<int, kStageBytes>{}, it + 1, i0_next, false, std::false_type{});
    }
    for (; it < n_it; ++it) tile((it & 1) * kStageBytes, it, i0_next, false, std::true_type{});

    if constexpr (NG > 1) {
        static_assert(NG == 2, "one group hands its sums to the other");
        if (n_it < (n_all + 1) / 2) {  // (the barriers of the tile that the first group has more)
            lds_barrier();
            __syncthreads();
        }
        auto slot = [&](int m, int kt, int q) { return reinterpret_cast<f32x4*>(lds) + (((w * MH + m) * 2 + kt) * 4 + q) * 64 + lane; };
        if (group == 1) {
#pragma unroll
            for (int m = 0; m < MH; ++m)
#pragma unroll
                for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        *slot(m, kt, q) = f32x4{acc[m][kt][4 * q], acc[m][kt][4 * q + 1], acc[m][kt][4 * q + 2], acc[m][kt][4 * q + 3]};
        }
        __syncthreads();
        if (group == 0) {
#pragma unroll
            for (int m = 0; m < MH; ++m)
#pragma unroll
                for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const f32x4 other = *slot(m, kt, q);
#pragma unroll
                        for (int e = 0; e < 4; ++e) acc[m][kt][4 * q + e] += other[e];
                    }
        }
    }

    const float f = wx == 0 ? 1.f : p.scale;
    typedef RowStage<D> Rows;
    constexpr int kGradBytes = 2 * Rows::kBytes;  // 64 rows: dV, then dK
    constexpr int kSlots = NG > 1 ? 4 * MH * 2 * 4096 : 0;
    static_assert(kSlots + 2 * kGradBytes <= NG * (2 * kStageBytes + 2 * kPBytes), "the stages are free after the last tile");
    char* rows = lds + kSlots;
    if (group == 0) {
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)  // accumulator column: key j0 + 32 kt + l32
#pragma unroll
        for (int m = 0; m < MH; ++m)
#pragma unroll
            for (int g = 0; g < 4; ++g)
                Rows::put(rows + wx * kGradBytes + kt * Rows::kBytes, 4 * (MH * wk + m) + g,
                          u32x2{pack_bf16(acc[m][kt][4 * g + 0] * f, acc[m][kt][4 * g + 1] * f),
                                pack_bf16(acc[m][kt][4 * g + 2] * f, acc[m][kt][4 * g + 3] * f)},
                          lane);
    }
    __syncthreads();
    const long out = base + (long)j0 * ld;
    Rows::template store<64, 4 * NG>(rows, p.dV + out, ld, p.n - j0, lane, 4 * group + w);
    Rows::template store<64, 4 * NG>(rows + kGradBytes, p.dK + out, ld, p.n - j0, lane, 4 * group + w);
}

template <int D>
__global__ void __launch_bounds__(kThreads, D <= 128 ? 2 : 1) bwd_dkdv_kernel(FusedParams p) {
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    // with an order list the grid has both halves of every 128-key block (the last one may lie
    // past n) and the blocks come longest list first
    const int key_blocks = p.order ? 2 * ((p.n + 127) / 128) : (p.n + 63) / 64;
    int bh, j;
    decode_block_causal(blockIdx.x, key_blocks, p.batch * p.heads, p.resident, bh, j);
    dkdv_block<D>(p, smem, bh, j);
}

// ----------------------------------------------------------------------------------- dQ
// Wave w owns queries i0 + 32w .. +31: their Q and dO rows stay in registers as B operands.
// Per key tile (64 keys, two halves T):
//   S^T[T] = K_T Q_w^T, dP^T[T] = V_T dO_w^T        accumulator: lane <-> query, register <-> key
//   dS^T = P^T (dP^T - delta)                        per-lane scalars lse2, delta
//   dQ_w^T += K_T^T dS^T                             K^T from transposed LDS reads
// SPLIT = 2: the block has 64 queries and wave (wq, wk) takes queries 32 wq .. +31 with key half wk of every tile; the two
// sums of a query meet in LDS at the end.
// OWN: delta is formed here and left in the workspace; else it is read from there.
template <int D, int SPLIT, bool OWN, int NG = 1>
__device__ __forceinline__ void dq_block(const FusedParams p, char* lds, int bh, int blk) {
    static_assert(NG == 1 || SPLIT == 2, "two groups: blocks of 64 queries");
    constexpr int BR = 128 / SPLIT, BC = 64, KS = D / 16, MT = D / 32;
    constexpr int NT = 2 / SPLIT;  // 32-key halves of a tile per wave
    constexpr int kTileBytes = BC * D * 2;
    constexpr int kStageBytes = 2 * kTileBytes;

    // group of four waves, each with stages of its own; the key tiles take turns (see dkdv_block)
    const int group = NG == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / kThreads);
    char* smem = lds + group * ((OWN && SPLIT == 2 ? 5 : 4) * kTileBytes);
    const int tid = threadIdx.x % kThreads, lane = tid & 63, h = lane >> 5, l32 = lane & 31;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave index within the group, uniform
    const int wq = SPLIT == 1 ? w : w & 1, wk = SPLIT == 1 ? 0 : w >> 1;
    const int q_blocks = (p.n + BR - 1) / BR;
    // longest rows first: under the causal rule the last blocks, under a block mask by the order list
    const int ib = p.order ? SPLIT * p.order[(long)bh * p.order_stride + blk / SPLIT] + blk % SPLIT
                           : (p.causal ? q_blocks - 1 - blk : blk);
    const long base = (long)(bh / p.heads) * p.stride_b + (long)(bh % p.heads) * p.stride_h;
    const long ld = p.stride_n;
    const int i0 = ib * BR;
    const int w0 = i0 + 32 * wq;  // first query of this wave

    int n_it, lp0 = 0;
    if (p.list_ptr) {  // block lists are per 128 queries
        const int32_t* lptr = p.list_ptr + (long)bh * p.list_stride;  // this (batch, head)'s mask
        const int lb = ib / SPLIT;
        lp0 = lptr[lb];
        int entries = lptr[lb + 1] - lp0;
        if (p.causal) entries = causal_row_entries(p.list_idx, lp0, entries, lb);
        n_it = entries * (128 / BC);
    } else {
        const int k_end = p.causal ? min(p.n, i0 + BR) : p.n;
        n_it = (k_end + BC - 1) / BC;
    }
    const int n_all = n_it;
    if constexpr (NG > 1) n_it = (n_all - group + NG - 1) / NG;
    auto tile_start = [&](int it) -> int { return tile_start_row<BC>(p.list_idx, lp0, 0, NG * it + group); };

    // K and V tiles go straight from global memory into the LDS stage that was last read one
    // iteration ago; rows past n repeat the last row and are masked below.
    TileLoader<D, BC> loader;
    loader.init(tid, ld);
    auto fetch = [&](int j0, int stage) {
        char* s = smem + stage * kStageBytes;
        loader.load(p.K + base, ld, j0, p.n, s, tid);
        loader.load(p.V + base, ld, j0, p.n, s + kTileBytes, tid);
    };
    // Resident operands: 32 queries per wave.  Their rows come through LDS (read straight from memory as operands, every load takes 16
    // bytes from each of 64 places): blocks of 64 queries through the second stage and, for O, a tile behind the stages, while the first
    // tile arrives in the first; of 128 queries Q and dO through both stages, then O while the first tile arrives.  Rows past n repeat the
    // last row; nothing of theirs is stored.  dQ leaves through LDS as well.  us of the kernel, before -> now: d = 64
    // b4 h16 n2048 103 -> 103, causal h12 n2048 25.7 -> 23.6   d = 128 b2 h16 n1024 causal 26.1 -> 23.7, b2 h32 n8192 causal 1383 -> 1357   d = 256
    // h8 n1000 39.1 -> 35.6, b2 h23 n97 causal 13.8 -> 11.9
    const int q = w0 + l32;
    const bool ok = q < p.n;
    const float lse2 = ok ? p.LSE[(long)bh * p.n + q] * kLog2e : __builtin_inff();
    float dl = 0.f;
    if constexpr (!OWN) {
        if (ok) dl = p.delta[(long)bh * p.n + q];
    }
    FragOffsets<D> lane_offsets;
    lane_offsets.init(lane);
    FragAddrs<D> fo;
    fo.init(lane_offsets);
    bf16x8 qf[KS], gf[KS];
    int j0_next = n_it > 0 ? tile_start(0) : 0;
    // delta = rowsum(dO o O) of this lane's query: the dO fragments are at hand, the O row is
    // read once here (and nowhere else in the backward); the two lane halves hold the two
    // halves of every 16-element chunk.  The dK / dV kernel, which runs after this one,
    // takes delta from the workspace.
    auto form_delta = [&](int o_off) {
        float dsum = 0.f;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const bf16x8 of = fo.frag(smem, o_off, 32 * wq, ks);
#pragma unroll
            for (int e = 0; e < 8; ++e) dsum += (float)of[e] * (float)gf[ks][e];
        }
        dsum += __shfl_xor(dsum, 32, 64);
        if (ok) dl = dsum;
        if (ok && h == 0 && wk == 0 && group == 0) p.delta[(long)bh * p.n + q] = dsum;
    };
    auto read_operands = [&](int q_off, int g_off) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            qf[ks] = fo.frag(smem, q_off, 32 * wq, ks);
            gf[ks] = fo.frag(smem, g_off, 32 * wq, ks);
        }
    };
    if constexpr (SPLIT == 2) {
        loader.load(p.Q + base, ld, i0, p.n, smem + kStageBytes, tid);
        loader.load(p.dO + base, ld, i0, p.n, smem + kStageBytes + kTileBytes, tid);
        if constexpr (OWN) loader.load(p.O + base, ld, i0, p.n, smem + 2 * kStageBytes, tid);
        if (n_it > 0) fetch(j0_next, 0);
        wait_direct_loads();
        __syncthreads();
        read_operands(kStageBytes, kStageBytes + kTileBytes);
        if constexpr (OWN) form_delta(2 * kStageBytes);
    } else {
        TileLoader<D, BR> rows;  // a stage holds 128 rows
        rows.init(tid, ld);
        rows.load(p.Q + base, ld, i0, p.n, smem + kStageBytes, tid);
        rows.load(p.dO + base, ld, i0, p.n, smem, tid);
        wait_direct_loads();
        __syncthreads();
        read_operands(kStageBytes, 0);
        lds_barrier();
        if constexpr (OWN) rows.load(p.O + base, ld, i0, p.n, smem + kStageBytes, tid);
        if (n_it > 0) fetch(j0_next, 0);
        wait_direct_loads();
        __syncthreads();
        if constexpr (OWN) form_delta(kStageBytes);
    }
    lds_barrier();  // (the first tile's copies go into the second stage)
    settle(lse2);
    settle(dl);

    f32x16 dq[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int i = 0; i < 16; ++i) dq[mt][i] = 0.f;

    const float c = p.scale * kLog2e;
    // -delta of this lane's query in all 16 registers of an accumulator block: the dP^T chains start
    // from it (C operand of their first MFMA), so dP^T - delta costs no vector instruction per tile.
    // Not at d = 64: there the kernel is built for four workgroups per CU (128 registers) and the
    // 16 extra registers would spill (measured: 12 -> 332 bytes of scratch per lane, four times slower).
    constexpr bool kDeltaInAcc = D >= 128;
    f32x16 ndl;
#pragma unroll
    for (int i = 0; i < 16; ++i) ndl[i] = kDeltaInAcc ? -dl : 0.f;
    if constexpr (SPLIT > 1) fo.shift_rows(32 * wk);

    // One streamed tile.  `masked` selects the copy of the body that applies the causal / tail
    // bound; the other copy has no mask arithmetic at all.
    // Wave priorities per phase (see the forward kernel): score MFMAs, then the dQ MFMAs, the
    // exponentials last.
    constexpr int kPrioScores = 2, kPrioSoftmax = 0, kPrioDq = 1;
    auto tile = [&](auto stage_off, int j0, auto masked) {
        const int k_off = stage_off;  // K tile; the V tile follows it
        // the two 32-key halves one after the other: half the score registers live at a time
#pragma unroll
        for (int T = 0; T < NT; ++T) {
            __builtin_amdgcn_s_setprio(kPrioScores);
            f32x16 st, dpt = ndl;
#pragma unroll
            for (int i = 0; i < 16; ++i) st[i] = 0.f;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {  // independent accumulation chains, interleaved
                const bf16x8 kfr = fo.frag(smem, k_off, 32 * T, ks);
                const bf16x8 vfr = fo.frag(smem, k_off + kTileBytes, 32 * T, ks);
                st = mfma32(kfr, qf[ks], st);
                dpt = mfma32(vfr, gf[ks], dpt);
            }
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_setprio(kPrioSoftmax);
            bf16x8 dsb[2], kt[2][MT];
            // key j0 + 32T + 8g + 4h + r is visible iff 8g + r <= lim (one per-lane bound)
            const int lim = (p.causal ? min(q, p.n - 1) : p.n - 1) - j0 - 32 * (T + wk) - 4 * h;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                float pv = __builtin_amdgcn_exp2f(st[i] * c - lse2);
                if constexpr (decltype(masked)::value) pv = (8 * (i >> 2) + (i & 3) > lim) ? 0.f : pv;
                dpt[i] = kDeltaInAcc ? pv * dpt[i] : pv * (dpt[i] - dl);
            }
#pragma unroll
            for (int ss = 0; ss < 2; ++ss) dsb[ss] = acc_to_operand(dpt, ss);
            __builtin_amdgcn_s_setprio(kPrioDq);
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) kt[0][mt] = fo.frag_t(smem, k_off, mt, 32 * T);
#pragma unroll
            for (int ss = 0; ss < 2; ++ss) {  // K^T fragments of the next 16 keys requested ahead
                if (ss == 0) {
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) kt[1][mt] = fo.frag_t(smem, k_off, mt, 32 * T + 16);
                }
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) dq[mt] = mfma32(kt[ss][mt], dsb[ss], dq[mt]);
            }
            __builtin_amdgcn_sched_barrier(0);  // the next half starts after this one is issued
        }
    };
    // Tiles come in ascending key order, so those that need the bound (they straddle the
    // diagonal or the end of the sequence) are the last ones.  Mask-free tiles go two at a time
    // through a body whose LDS stage offsets are compile-time constants (fragment addresses are
    // then a precomputed register plus an immediate); the rest takes the masked body with a
    // run-time stage.  Waves may leave the first loop at different tiles; both loops run the same
    // fetches and barriers.
    constexpr int kWaveKeys = 32 * NT;  // keys of a tile that a wave looks at, from j0 + 32 wk on
    auto needs_mask = [&](int j0) {
        return (p.causal && (j0 + 32 * wk + kWaveKeys - 1 > w0)) || (j0 + 32 * wk + kWaveKeys > p.n);
    };
    int it = 0;
    for (; it + 2 <= n_it; it += 2) {
        const int ja = j0_next, jb = tile_start(it + 1);
        if (needs_mask(ja) || needs_mask(jb)) break;
        j0_next = jb;
        fetch(jb, 1);
        tile(std::integral_constant<int, 0>{}, ja, std::false_type{});
        wait_direct_loads();
        __syncthreads();
        if (it + 2 < n_it) {
            j0_next = tile_start(it + 2);
            fetch(j0_next, 0);
        }
        tile(std::integral_constant<int, kStageBytes>{}, jb, std::false_type{});
        wait_direct_loads();
        __syncthreads();
    }
    for (; it < n_it; ++it) {
        const int j0 = j0_next;
        if (it + 1 < n_it) {
            j0_next = tile_start(it + 1);
            fetch(j0_next, (it + 1) & 1);
        }
        // causal: this wave's last query precedes its first key of the tile -> nothing visible
        if (!(p.causal && (w0 + 31 < j0 + 32 * wk))) tile((it & 1) * kStageBytes, j0, std::true_type{});
        wait_direct_loads();
        __syncthreads();
    }

    if constexpr (NG > 1) {
        if (n_it < (n_all + 1) / 2) __syncthreads();  // (the barrier of the tile that the first group has more)
        auto slot = [&](int mt, int q) { return reinterpret_cast<f32x4*>(lds) + ((w * MT + mt) * 4 + q) * 64 + lane; };
        if (group == 1) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4) *slot(mt, q4) = f32x4{dq[mt][4 * q4], dq[mt][4 * q4 + 1], dq[mt][4 * q4 + 2], dq[mt][4 * q4 + 3]};
        }
        __syncthreads();
        if (group == 0) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4) {
                    const f32x4 other = *slot(mt, q4);
#pragma unroll
                    for (int e = 0; e < 4; ++e) dq[mt][4 * q4 + e] += other[e];
                }
        }
        __syncthreads();
    }
    constexpr int MW = MT / SPLIT;  // 32-column groups of dQ that a wave writes, from MW wk on
    if constexpr (SPLIT > 1) {
        // each of the two waves of a query hands the other the half of its sum that the other writes; the stages are
        // free (every wave is past the last barrier of the loop)
        auto slot = [&](int wave, int mt, int g) { return reinterpret_cast<f32x4*>(smem) + ((wave * MW + mt) * 4 + g) * 64 + lane; };
        auto send = [&](auto first) {
#pragma unroll
            for (int mt = 0; mt < MW; ++mt)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const f32x16& a = dq[decltype(first)::value + mt];
                    *slot(w, mt, g) = f32x4{a[4 * g], a[4 * g + 1], a[4 * g + 2], a[4 * g + 3]};
                }
        };
        auto meet = [&](auto first) {
#pragma unroll
            for (int mt = 0; mt < MW; ++mt)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const f32x4 b = *slot(w ^ 2, mt, g);
#pragma unroll
                    for (int r = 0; r < 4; ++r) dq[mt][4 * g + r] = dq[decltype(first)::value + mt][4 * g + r] + b[r];
                }
        };
        if (group == 0) {
            if (wk == 0) send(std::integral_constant<int, MW>{});
            else send(std::integral_constant<int, 0>{});
        }
        __syncthreads();
        if (group == 1) return;
        if (wk == 0) meet(std::integral_constant<int, 0>{});
        else meet(std::integral_constant<int, MW>{});
    }
    // (a wave's own rows and columns: nothing to wait for but its own writes; behind the slots of the two sums)
    typedef RowStage<32 * MW> Rows;
    constexpr int kSlots = SPLIT > 1 ? 4 * MW * 4096 : 0;
    static_assert(kSlots + 4 * Rows::kBytes <= 2 * kStageBytes, "the stages are free after the last tile");
    int out_lane = lane;  // formed again here, so that no address is carried through the loop (d = 64 has no register to spare)
    asm volatile("" : "+v"(out_lane));
    char* mine = smem + kSlots + w * Rows::kBytes;
#pragma unroll
    for (int mt = 0; mt < MW; ++mt)
#pragma unroll
        for (int g = 0; g < 4; ++g)
            Rows::put(mine, 4 * mt + g,
                      u32x2{pack_bf16(dq[mt][4 * g + 0] * p.scale, dq[mt][4 * g + 1] * p.scale),
                            pack_bf16(dq[mt][4 * g + 2] * p.scale, dq[mt][4 * g + 3] * p.scale)},
                      out_lane);
    Rows::store(mine, p.dQ + base + (long)w0 * ld + 32 * MW * wk, ld, p.n - w0, out_lane);
}

constexpr int dq_per_cu(int d) { return d == 64 ? 4 : d == 128 ? 2 : 1; }
constexpr int dq_split_per_cu(int d) { return d == 64 ? 3 : dq_per_cu(d); }  // (130 registers at d = 64)

template <int D, int QT>  // QT: 32-query tiles per wave
__global__ void __launch_bounds__(kThreads, dq_per_cu(D)) bwd_dq_kernel(FusedParams p) {
    static_assert(QT == 1, "two tiles per wave do not leave two waves per SIMD");
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    int bh, blk;
    decode_block_causal(blockIdx.x, (p.n + 127) / 128, p.batch * p.heads, p.resident, bh, blk);
    dq_block<D, 1, true>(p, smem, bh, blk);
}

template <int D>
__global__ void __launch_bounds__(kThreads, dq_split_per_cu(D)) bwd_dq_split_kernel(FusedParams p) {
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    int bh, blk;
    decode_block_causal(blockIdx.x, p.order ? 2 * ((p.n + 127) / 128) : (p.n + 63) / 64, p.batch * p.heads, p.resident, bh, blk);
    dq_block<D, 2, true>(p, smem, bh, blk);
}

// Both halves of the backward side by side: for every 128 rows two blocks of 64 queries (SPLIT = 2) or one of 128 (dQ), and two of
// 64 keys (dK, dV).  The same blocks as in the two kernels, so the same bits; v comes from bwd_rows_kernel for both.
template <int D, int SPLIT>
__global__ void __launch_bounds__(kThreads, D <= 128 ? 2 : 1) bwd_both_kernel(FusedParams pq, FusedParams pk) {
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    int bh, rank;
    if constexpr (SPLIT == 2) {
        const int blocks = pq.order ? 2 * ((pq.n + 127) / 128) : (pq.n + 63) / 64;
        decode_block_causal(blockIdx.x, 2 * blocks, pq.batch * pq.heads, pq.resident, bh, rank);
        if (rank & 1) dq_block<D, 2, false>(pq, smem, bh, rank >> 1);
        else dkdv_block<D>(pk, smem, bh, rank >> 1);
    } else {
        const int blocks = 3 * ((pq.n + 127) / 128);
        decode_block_causal(blockIdx.x, blocks, pq.batch * pq.heads, pq.resident, bh, rank);
        const int r = rank % 3, k = 2 * (rank / 3) + r - 1;
        if (r == 0) dq_block<D, 1, false>(pq, smem, bh, rank / 3);
        else if (pk.order || 64 * k < pk.n) dkdv_block<D>(pk, smem, bh, k);
    }
}

// The same, and each half alone, with eight waves for blocks of 64 queries and of 64 keys: see eight_waves_bwd
template <int D>
__global__ void __launch_bounds__(2 * kThreads, 2) bwd_dkdv_eight_kernel(FusedParams p) {
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    const int key_blocks = p.order ? 2 * ((p.n + 127) / 128) : (p.n + 63) / 64;
    int bh, j;
    decode_block_causal(blockIdx.x, key_blocks, p.batch * p.heads, p.resident, bh, j);
    dkdv_block<D, 2>(p, smem, bh, j);
}
template <int D>
__global__ void __launch_bounds__(2 * kThreads, 2) bwd_dq_eight_kernel(FusedParams p) {
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    int bh, blk;
    decode_block_causal(blockIdx.x, p.order ? 2 * ((p.n + 127) / 128) : (p.n + 63) / 64, p.batch * p.heads, p.resident, bh, blk);
    dq_block<D, 2, true, 2>(p, smem, bh, blk);
}
template <int D>
__global__ void __launch_bounds__(2 * kThreads, 2) bwd_both_eight_kernel(FusedParams pq, FusedParams pk) {
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    const int blocks = pq.order ? 2 * ((pq.n + 127) / 128) : (pq.n + 63) / 64;
    int bh, rank;
    decode_block_causal(blockIdx.x, 2 * blocks, pq.batch * pq.heads, pq.resident, bh, rank);
    if (rank & 1) dq_block<D, 2, false, 2>(pq, smem, bh, rank >> 1);
    else dkdv_block<D, 2>(pk, smem, bh, rank >> 1);
}

// The whole backward of a short call in one launch: every block forms the row sums it needs (see own_rows; the query blocks leave theirs in the
// workspace as they do for bwd_dkdv_kernel, though nothing reads them here).
template <int D, int NG>
__global__ void __launch_bounds__(NG * kThreads, D <= 128 ? 2 : 1) bwd_short_kernel(FusedParams p) {
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    int bh, rank;
    decode_block_causal(blockIdx.x, 2 * ((p.n + 63) / 64), p.batch * p.heads, p.resident, bh, rank);
    if (rank & 1) dq_block<D, 2, true, NG>(p, smem, bh, rank >> 1);
    else dkdv_block<D, NG, true>(p, smem, bh, rank >> 1);
}

// Workgroups per CU of bwd_both_kernel and bwd_dkdv_kernel (their LDS and registers).
constexpr int both_per_cu(int d) { return d == 64 ? 3 : d == 128 ? 2 : 1; }

// Whether dQ and dK / dV run in one launch of `grid` workgroups, with v formed by a small launch in front.  One launch instead of two dependent ones
// fills the CUs that the first leaves idle while its last blocks run, and a call with fewer blocks than CUs takes the longer of the
// two instead of their sum; the price is the launch in front (3 to 4 us) and, at d = 64, three workgroups per CU for dQ instead of four.
// With lists of equal length the two launches fill the chip as evenly as one, so there all blocks have to fit at once; causal
// and masked lists leave a tail per launch, which is worth it up to four rounds (six at d = 64).  us of the backward, two launches -> one:
//   full     d64  h8 n333 (causal) 17.0 -> 12.5   h4 n1500 45 -> 28   h12 n2048 69 -> 64     h16 n2048 (beyond) 75 -> 89
//            d128 h8 n700 34 -> 21     h8 n2048 79 -> 69     h16 n2048 (beyond) 125 -> 132    h16 n4096 (beyond) 428 -> 488
//            d256 h8 n1000 77 -> 45    h6 n2048 (beyond) 139 -> 146     h20 n3000 (beyond) 722 -> 760
//   causal   d64  h16 n2048 57 -> 48   h64 n2048 153 -> 149     d256 h8 n4096 345 -> 278   h24 n2048 243 -> 235
//            d128 h32 n1024 56 -> 50   h16 n4096 259 -> 241     h48 n2048 (four rounds and a half) 202 -> 204   h32 n4096 (beyond) 459 -> 482
//   10 %     d128 h16 n4096 110 -> 84  h16 n8192 (beyond) 250 -> 248   h16 n16384 (beyond) 818 -> 870   d64 h16 n8192 156 -> 136   h32 n8192 (beyond) 271 -> 260
inline bool side_by_side(long grid, int d, bool uneven) {
    return grid <= 256L * both_per_cu(d) * (!uneven ? 1 : d == 64 ? 6 : 4);
}

// ------------------------------------------------------------------------------ launchers
void launch_delta(const FusedParams& p, int d, hipStream_t stream) {
    const long lanes = (long)p.batch * p.heads * p.n * (d / 8 < 64 ? d / 8 : 64);
    hipLaunchKernelGGL(delta_kernel, dim3((unsigned)((lanes + kThreads - 1) / kThreads)), dim3(kThreads), 0, stream, p, d);
}

template <int D>
static hipError_t launch_bwd(const FusedParams& p, const int32_t* csr_ptr, const int32_t* csr_idx,
                             const int32_t* csc_ptr, const int32_t* csc_idx, hipStream_t stream, bool dq_only,
                             int32_t* order_scratch, int onepass_keys, float* dq_acc, bool dkdv_only) {
    const int bh = p.batch * p.heads;
    const bool onepass = onepass_keys != 0 && !dq_only;

    constexpr int kv_lds = 2 * (2 * 64 * D * 2) + 2 * 64 * 64 * 2;  // two stages of Q, dO; P and dS
    const int blocks128 = (p.n + 127) / 128;
    const bool split = few_blocks(blocks128 * bh, dq_per_cu(D), p.causal && !p.mask_form);
    const long both_grid = (long)bh * (split ? 2 * (csr_ptr ? 2 * blocks128 : (p.n + 63) / 64) : 3 * blocks128);
    const bool both = p.may_join && !onepass && !dq_only && !dkdv_only && side_by_side(both_grid, D, p.causal || csr_ptr);
    const bool eight = D <= 128 && split && eight_waves_bwd(p.causal != 0, p.mask_form, p.n, bh);
    const int groups = eight ? 2 : 1;
    const int q_lds = groups * (split ? 5 : 4) * (64 * D * 2);  // two stages of K, V; blocks of 64 queries: and their O rows
    void (*dq_fn)(FusedParams) = split ? bwd_dq_split_kernel<D> : bwd_dq_kernel<D, 1>;
    void (*dkdv_fn)(FusedParams) = bwd_dkdv_kernel<D>;
    void (*both_fn)(FusedParams, FusedParams) = split ? bwd_both_kernel<D, 2> : bwd_both_kernel<D, 1>;
    if constexpr (D <= 128) {
        if (eight) {
            dq_fn = bwd_dq_eight_kernel<D>;
            dkdv_fn = bwd_dkdv_eight_kernel<D>;
            both_fn = bwd_both_eight_kernel<D>;
        }
    }
    const dim3 block((unsigned)(groups * kThreads));
    hipError_t e = hipSuccess;
    // (a gradient that takes the place of O: key blocks of the short kernel would read O beside the blocks that write it)
    const bool o_stays = p.O != p.dQ && p.O != p.dK && p.O != p.dV;
    if (both && split && o_stays && own_rows(p.causal != 0, p.n, D, both_grid, csr_ptr != nullptr)) {
        void (*fn)(FusedParams) = bwd_short_kernel<D, 1>;
        if constexpr (D == 64) {
            if (eight) fn = bwd_short_kernel<D, 2>;
        }
        const int kv = groups * kv_lds + kOwnRows * (int)sizeof(float), lds = kv > q_lds ? kv : q_lds;
        e = allow_lds(fn, lds);
        if (e != hipSuccess) return e;
        FusedParams ps = p;
        if (p.causal) ps.resident = causal_resident((int)both_grid, D == 64 && !eight ? both_per_cu(D) : 1);
        hipLaunchKernelGGL(fn, dim3((unsigned)both_grid), block, lds, stream, ps);
        return hipGetLastError();
    }
    if (both) {
        e = allow_lds(both_fn, groups * kv_lds);
    } else if (!onepass) {
        e = allow_lds(dkdv_fn, groups * kv_lds);
        if (e == hipSuccess) e = allow_lds(dq_fn, q_lds);
    }
    if (e != hipSuccess) return e;
    OrderParams op = {csr_ptr, csr_idx, csc_ptr, csc_idx, nullptr, nullptr, blocks128, p.causal};
    const int masks = p.list_stride ? bh : 1;  // one mask per (batch, head), or one for all
    if (order_scratch && csr_ptr && csc_ptr && masks <= 65535) {  // (grid.y limit; beyond it: ascending order)
        op.order_q = order_scratch;
        op.order_k = order_scratch + (long)masks * blocks128;
        int32_t* len = order_scratch + 2L * masks * blocks128;
        const dim3 og((unsigned)((blocks128 + kThreads - 1) / kThreads), (unsigned)masks);
        const bool want_q = !onepass && !dkdv_only, want_k = !dq_only;
        if (blocks128 <= kOrderFusedBlocks) {
            if (!both && (want_q || want_k))
                hipLaunchKernelGGL(block_order_fused_kernel, dim3((unsigned)masks, want_q && want_k ? 2u : 1u),
                                   dim3(kThreads), 0, stream, op, want_q ? 0 : 1);
        } else {
            if (want_q) {
                hipLaunchKernelGGL(block_len_kernel, og, dim3(kThreads), 0, stream, csr_ptr, csr_idx, blocks128, p.causal, 0, len);
                hipLaunchKernelGGL(block_order_kernel, og, dim3(kThreads), 0, stream, len, blocks128, op.order_q);
            }
            if (want_k) {
                hipLaunchKernelGGL(block_len_kernel, og, dim3(kThreads), 0, stream, csc_ptr, csc_idx, blocks128, p.causal, 1, len);
                hipLaunchKernelGGL(block_order_kernel, og, dim3(kThreads), 0, stream, len, blocks128, op.order_k);
            }
        }
    }
    FusedParams pq = p, pk = p;
    pq.list_ptr = csr_ptr;
    pq.list_idx = csr_idx;
    pq.order = op.order_q;
    pk.list_ptr = csc_ptr;
    pk.list_idx = csc_idx;
    pk.order = op.order_k;
    pq.order_stride = pk.order_stride = p.list_stride ? blocks128 : 0;
    if (onepass) return launch_bwd_onepass(D, onepass_keys, pk, dq_acc, stream);
    // with an order list both halves of every 128-row block (the last one may lie past n: it writes nothing)
    const int halves = op.order_k ? 2 * blocks128 : (p.n + 63) / 64;
    if (both) {
        const int orders = op.order_q && blocks128 <= kOrderFusedBlocks ? 2 * masks : 0;
        const long rows = (long)bh * p.n;
        const unsigned grid = (unsigned)((split ? 2 * halves : 3 * blocks128) * bh);  // (both_grid, or a little less without orders)
        if (p.causal && !csr_ptr) pq.resident = causal_resident((int)grid, eight ? 1 : both_per_cu(D));
        hipLaunchKernelGGL(bwd_rows_kernel<D>, dim3((unsigned)(orders + (rows + kThreads / 2 - 1) / (kThreads / 2))), dim3(kThreads), 0, stream,
                           p, op, orders);
        hipLaunchKernelGGL(both_fn, dim3(grid), block, groups * kv_lds, stream, pq, pk);
        return hipGetLastError();
    }
    const int q_blocks = split ? halves : blocks128;
    if (p.causal && !csr_ptr) pq.resident = causal_resident(q_blocks * bh, eight ? 1 : split ? dq_split_per_cu(D) : dq_per_cu(D));
    // One query tile per wave and two workgroups per CU.  (QT = 2, i.e. one wave per SIMD with every
    // LDS fragment feeding two MFMAs, halves the LDS traffic but measured 20 % slower at d = 128:
    // with a single wave per SIMD the softmax arithmetic no longer overlaps another wave's MFMAs.)
    if (!dkdv_only)
        hipLaunchKernelGGL(dq_fn, dim3((unsigned)(q_blocks * bh)), block, q_lds, stream, pq);
    if (dq_only) return hipGetLastError();
    if (p.causal && !csc_ptr) pk.resident = causal_resident(halves * bh, eight ? 1 : both_per_cu(D));
    hipLaunchKernelGGL(dkdv_fn, dim3((unsigned)(halves * bh)), block, groups * kv_lds, stream, pk);
    return hipGetLastError();
}

hipError_t launch_bwd_fused(int d, const FusedParams& p, const int32_t* csr_ptr, const int32_t* csr_idx,
                            const int32_t* csc_ptr, const int32_t* csc_idx, hipStream_t stream, bool dq_only,
                            int32_t* order_scratch, int onepass_keys, float* dq_acc, bool dkdv_only) {
    switch (d) {
        case 64: return launch_bwd<64>(p, csr_ptr, csr_idx, csc_ptr, csc_idx, stream, dq_only, order_scratch, onepass_keys, dq_acc, dkdv_only);
        case 128: return launch_bwd<128>(p, csr_ptr, csr_idx, csc_ptr, csc_idx, stream, dq_only, order_scratch, onepass_keys, dq_acc, dkdv_only);
        case 256: return launch_bwd<256>(p, csr_ptr, csr_idx, csc_ptr, csc_idx, stream, dq_only, order_scratch, 0, nullptr, dkdv_only);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace attn
