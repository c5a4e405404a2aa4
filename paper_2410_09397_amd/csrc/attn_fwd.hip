// Fused forward for d <= 256 (d = 256: one wave per SIMD): O = diag(l)^{-1} exp(scale Q K^T) V and LSE = log l (forward
// definition, Sec. 3.1; A, l, f, O of App. B.4), evaluated per block of 128 queries with a
// running maximum so that no n x n matrix is formed.  The paper gives no forward algorithm;
// the streaming-softmax tiling is prior art, the kernel is written for gfx950.
#include <type_traits>

#include "attn_common.hpp"
#include "attn_internal.hpp"

namespace attn {

// The Q rows of a wave, 32 from q0 on, as operands: through `lds`, which only this wave uses (read straight from memory every load takes
// 16 bytes from each of 64 places), as O leaves through LDS in whole rows (fwd_finish; 8-byte pieces of 32 rows before).  us, straight -> through LDS:
// d = 64 b4 h16 n2048 84.9 -> 82.6   d = 128 b2 h16 n1024 causal 19.9 -> 18.7, h11 n700 14.2 -> 13.3, b2 h32 n8192 causal 1086 -> 1075   d = 256 h8 n1000 29.1 -> 27.2
// The way through LDS is 0.3 us in front of the first tile and behind the last, which a causal call of few blocks shows where its last block, the longest, has
// few rows to read and write.  So in the kernels of short calls
//   d = 64 (64 queries) and 256: a wave that the end of the sequence cuts reads its rows straight from memory and writes its O so (kCutRowsStraight; rows past
//     n are 0 then, else they repeat the last row; nothing of theirs is stored).  us, causal, all through LDS -> those straight: d = 64 h46 n337 7.7 -> 7.5,
//     h26 n580 9.9 -> 9.6 (full h64 n512 9.6 -> 9.7)   d = 256 b2 h29 n284 22.7 -> 21.1, h26 n580 31.7 -> 30.4.  With 128 queries at d = 64 the two ways need 12 bytes of scratch.
//   d = 128 (64 queries): the Q rows are requested in front of the first tile, not behind it, and read while it is on its way (kQueriesFirst).  us, behind -> in
//     front: causal h46 n337 10.2 -> 10.0, h58 n284 9.4 -> 9.1, h12 n721 14.3 -> 14.2, h16 n1900 29.6 -> 29.5; full h6 n200 7.4 -> 7.3, h30 n460 14.3 -> 14.5.  (Cut rows straight
//     there: h16 n1900 30.5 -> 30.7; with 128 queries h34 n2982 full 171 -> 176.)
template <int D, int SPLIT>
constexpr bool kCutRowsStraight = D == 256 || (D == 64 && SPLIT == 2);
template <int D, int SPLIT>
constexpr bool kQueriesFirst = D == 128 && SPLIT == 2;
// first_tile: requests the copies of the first tile (kCopies of them, or none); called here if kQueriesFirst
template <int D, int SPLIT, int kCopies, typename FirstTile>
__device__ __forceinline__ void load_queries(const FusedParams& p, long base, int q0, char* lds, const FragOffsets<D>& offsets, int lane,
                                             bf16x8 (&qf)[D / 16], FirstTile first_tile) {
    const long ld = p.stride_n;
    if (!kCutRowsStraight<D, SPLIT> || q0 + 32 <= p.n) {
        TileLoader<D, 32, 1> rows;
        rows.init(lane, ld);
        if constexpr (kCutRowsStraight<D, SPLIT>) rows.load(p.Q + base + (long)q0 * ld, lds);
        else rows.load(p.Q + base, ld, q0, p.n, lds, lane);
        if constexpr (kQueriesFirst<D, SPLIT>) {
            first_tile();
            // (a block without a tile has no use for its queries; what is still on its way to LDS is waited for before the next barrier)
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kCopies) : "memory");
        } else {
            wait_direct_loads();
        }
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks) qf[ks] = offsets.frag(lds, 0, 0, ks);
    } else {
        const int q = q0 + (lane & 31), h = lane >> 5;
        const bf16x8 zero = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks) {
            qf[ks] = zero;
            if (q < p.n) qf[ks] = *reinterpret_cast<const bf16x8*>(p.Q + base + (long)q * ld + 16 * ks + 8 * h);
        }
    }
}

// The end of a query block: O / l and LSE of wave (wq, wk)'s 32 queries, from w0 on.  SPLIT > 1: SPLIT waves hold a part of the keys each; of the
// 4 MT groups of four registers of O each writes MG, from MG wk on, and hands the others theirs through LDS, whose stages are
// free (every wave is past the last barrier of the loop).
template <int D, int SPLIT, int kLdsBytes>
__device__ __forceinline__ void fwd_finish(const FusedParams& p, char* smem, long base, int bh, int w0, int wq, int wk, f32x16 (&o)[D / 32],
                                           float m_run, float l_run) {
    constexpr int MT = D / 32, MG = 4 * MT / SPLIT;
    const int lane = threadIdx.x & 63, h = lane >> 5, q = w0 + (lane & 31);
    float l = l_run + __shfl_xor(l_run, 32, 64);
    if constexpr (SPLIT > 1) {
        float* ml = reinterpret_cast<float*>(smem + 2 * SPLIT * (SPLIT - 1) * MG * 64 * 16);  // [wave][2][64]
        // groups of wave `from` for the wave with key part `to`: [wave][SPLIT - 1][MG][64 lanes] x 16 bytes
        auto slot = [&](int from, int to, int g) {
            const int part = to - (to > from / 2 ? 1 : 0);
            return reinterpret_cast<f32x4*>(smem) + ((from * (SPLIT - 1) + part) * MG + g) * 64 + lane;
        };
        static_for<SPLIT>([&](auto to) {
            if (wk == decltype(to)::value) return;
#pragma unroll
            for (int g = 0; g < MG; ++g) {
                constexpr int first = decltype(to)::value * MG;
                const f32x16& a = o[(first + g) / 4];
                const int r = 4 * ((first + g) % 4);
                *slot(wq + 2 * wk, decltype(to)::value, g) = f32x4{a[r], a[r + 1], a[r + 2], a[r + 3]};
            }
        });
        ml[(wq + 2 * wk) * 128 + lane] = m_run;
        ml[(wq + 2 * wk) * 128 + 64 + lane] = l;
        __syncthreads();
        float m_part[SPLIT], m = m_run;
#pragma unroll
        for (int k = 0; k < SPLIT; ++k) {
            m_part[k] = ml[(wq + 2 * k) * 128 + lane];
            m = __builtin_elementwise_maximum(m, m_part[k]);
        }
        const float m_use = m == -__builtin_inff() ? 0.f : m;
        l = 0.f;
#pragma unroll
        for (int k = 0; k < SPLIT; ++k) {
            m_part[k] = __builtin_amdgcn_exp2f(m_part[k] - m_use);  // the factor of that part
            l += ml[(wq + 2 * k) * 128 + 64 + lane] * m_part[k];
        }
        const float f_mine = __builtin_amdgcn_exp2f(m_run - m_use);
        m_run = m;
        static_for<SPLIT>([&](auto mine) {
            if (wk != decltype(mine)::value) return;
#pragma unroll
            for (int g = 0; g < MG; ++g) {
                constexpr int first = decltype(mine)::value * MG;
                const f32x16& a = o[(first + g) / 4];
                const int r = 4 * ((first + g) % 4);
                f32x4 s = f32x4{a[r], a[r + 1], a[r + 2], a[r + 3]} * f_mine;
#pragma unroll
                for (int k = 0; k < SPLIT; ++k)
                    if (k != decltype(mine)::value) s += *slot(wq + 2 * k, decltype(mine)::value, g) * m_part[k];
#pragma unroll
                for (int e = 0; e < 4; ++e) o[g / 4][4 * (g % 4) + e] = s[e];
            }
        });
    }
    const float inv = l > 0.f ? 1.f / l : 0.f;
    if (h == 0 && wk == 0 && q < p.n)
        p.LSEout[(long)bh * p.n + q] = l > 0.f ? (m_run + __builtin_amdgcn_logf(l)) * kLn2 : -__builtin_inff();
    if constexpr (kCutRowsStraight<D, SPLIT>)
        if (w0 + 32 > p.n) {  // (see load_queries)
            if (q < p.n) {
                __bf16* row = p.Oout + base + (long)q * p.stride_n;
#pragma unroll
                for (int g = 0; g < MG; ++g)
                    *reinterpret_cast<u32x2*>(row + 8 * (MG * wk + g) + 4 * h) =
                        u32x2{pack_bf16(o[g / 4][4 * (g % 4) + 0] * inv, o[g / 4][4 * (g % 4) + 1] * inv),
                              pack_bf16(o[g / 4][4 * (g % 4) + 2] * inv, o[g / 4][4 * (g % 4) + 3] * inv)};
            }
            return;
        }
    // (a wave's own rows and columns: nothing to wait for but its own writes; behind the slots of the other parts)
    typedef RowStage<8 * MG> Rows;
    constexpr int kWaves = 4 * (SPLIT > 1 ? SPLIT / 2 : 1);
    constexpr int kSlots = SPLIT > 1 ? 2 * SPLIT * (SPLIT - 1) * MG * 64 * 16 + kWaves * 512 : 0;
    static_assert(kSlots + kWaves * Rows::kBytes <= kLdsBytes, "the stages are free after the last tile");
    int out_lane = lane;  // formed again here, so that no address is carried through the loop (d = 64 has no register to spare)
    asm volatile("" : "+v"(out_lane));
    char* mine = smem + kSlots + (SPLIT > 1 ? wq + 2 * wk : wq) * Rows::kBytes;
#pragma unroll
    for (int g = 0; g < MG; ++g)  // 8 columns each, from MG wk on
        Rows::put(mine, g,
                  u32x2{pack_bf16(o[g / 4][4 * (g % 4) + 0] * inv, o[g / 4][4 * (g % 4) + 1] * inv),
                        pack_bf16(o[g / 4][4 * (g % 4) + 2] * inv, o[g / 4][4 * (g % 4) + 3] * inv)},
                  out_lane);
    Rows::store(mine, p.Oout + base + (long)w0 * p.stride_n + 8 * MG * wk, p.stride_n, p.n - w0, out_lane);
}

// Wave w owns queries i0 + 32w .. +31 (Q rows resident in registers as B operands).
// Per key tile (64 keys, two halves T):
//   S^T[T] = K_T Q_w^T                 accumulator: lane <-> query, register <-> key
//   m, l   : running row maximum and sum, one scalar per lane (both lane halves of a query
//            see the same maximum; their partial sums are added at the end)
//   O_w^T += V_T^T P^T                 V^T from transposed LDS reads, P^T straight from registers
// Workgroups per CU: 4 at d = 64 (128 registers per lane; measured 5-6 % faster than 3 per CU at 134
// registers on a grid of 1024 workgroups), 2 at d = 128.
// SPLIT = 2: the block has 64 queries and wave (wq, wk) takes queries 32 wq .. +31 with key half wk of every tile; each wave keeps
// a maximum, a sum and an O of its own, and the two of a query meet in LDS at the end.
template <int D, int SPLIT>
__device__ __forceinline__ void fwd_block(const FusedParams p, char* smem) {
    constexpr int BR = 128 / SPLIT, BC = 64, KS = D / 16, MT = D / 32;
    constexpr int NT = 2 / SPLIT;  // 32-key halves of a tile per wave
    constexpr int kTileBytes = BC * D * 2;

    const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, l32 = lane & 31;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave index, uniform
    const int wq = SPLIT == 1 ? w : w & 1, wk = SPLIT == 1 ? 0 : w >> 1;
    const int q_blocks = (p.n + BR - 1) / BR;
    int bh, blk;
    decode_block_causal(blockIdx.x, q_blocks, p.batch * p.heads, p.resident, bh, blk);
    const int ib = p.causal ? q_blocks - 1 - blk : blk;  // causal: longest rows first
    const long base = (long)(bh / p.heads) * p.stride_b + (long)(bh % p.heads) * p.stride_h;
    const long ld = p.stride_n;
    const int i0 = ib * BR;

    int n_it, lp0 = 0;
    if (p.list_ptr) {
        const int32_t* lptr = p.list_ptr + (long)bh * p.list_stride;  // this (batch, head)'s mask
        const int lb = ib / SPLIT;  // the lists are per 128 rows
        lp0 = lptr[lb];
        int entries = lptr[lb + 1] - lp0;
        if (p.causal) entries = causal_row_entries(p.list_idx, lp0, entries, lb);
        n_it = entries * (128 / BC);
    } else {
        const int k_end = p.causal ? min(p.n, i0 + BR) : p.n;
        n_it = (k_end + BC - 1) / BC;
    }
    auto tile_start = [&](int it) -> int { return tile_start_row<BC>(p.list_idx, lp0, 0, it); };

    // K and V tiles go straight from global memory into the LDS stage that was last read one
    // iteration ago; rows past n repeat the last row and are masked below.
    TileLoader<D, BC> loader;
    loader.init(tid, ld);
    // [K stage 0][K stage 1][V stage 0][V stage 1]: every fetch of a fragment is a register plus an immediate of 16 bits
    auto fetch = [&](int j0, int stage) {
        char* s = smem + stage * kTileBytes;
        loader.load(p.K + base, ld, j0, p.n, s, tid);
        loader.load(p.V + base, ld, j0, p.n, s + 2 * kTileBytes, tid);
    };
    // the Q rows come through a piece of the second stage that only this wave reads; their latency and that of the first tile overlap
    int j0_next = n_it > 0 ? tile_start(0) : 0;
    auto first_tile = [&] {
        if (n_it > 0) fetch(j0_next, 0);
    };
    if constexpr (!kQueriesFirst<D, SPLIT>) first_tile();

    const int q = i0 + 32 * wq + l32;
    FragOffsets<D> lane_offsets;
    lane_offsets.init(lane);
    bf16x8 qf[KS];
    load_queries<D, SPLIT, 2 * TileLoader<D, BC>::kInst>(p, base, i0 + 32 * wq, smem + (w < 2 ? 1 : 3) * kTileBytes + (w & 1) * (32 * D * 2), lane_offsets, lane, qf,
                                                         first_tile);

    f32x16 o[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[mt][i] = 0.f;
    float m_run = -__builtin_inff();  // running maximum of scale * log2(e) * s
    float l_run = 0.f;                // this lane's share of sum exp2(scaled s - m_run)

    // Scores are kept raw in the accumulators and scaled inside the exponential: with
    // cs = |scale| log2(e) > 0 the row maximum commutes with the scaling.  A negative scale is
    // moved into Q (sign flip of the resident fragments), a zero scale becomes a denormal-sized
    // positive one so that masked (-inf) scores stay -inf.
    const float cs = fmaxf(fabsf(p.scale) * kLog2e, 1.17549435e-38f);
    if (p.scale < 0.f) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            u32x4 v = __builtin_bit_cast(u32x4, qf[ks]);
            v ^= 0x80008000u;
            qf[ks] = __builtin_bit_cast(bf16x8, v);
        }
    }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) settle(qf[ks]);
    FragAddrs<D> fo;
    fo.init(lane_offsets);
    if constexpr (SPLIT > 1) fo.shift_rows(32 * wk);
    fo.shift_transposed(2 * kTileBytes);
    wait_direct_loads();
    __syncthreads();

    // One streamed tile; `masked` selects the copy of the body that applies the causal / tail bound.
    // Wave priorities: the two waves that share a SIMD tend to fall into step (they compete for
    // the same matrix pipe, so both reach the end of a phase, and its LDS latency, together).
    // Ranking the phases - score MFMAs first, then the PV MFMAs, the exponentials last - lets one
    // wave run ahead while the other fills the gaps (measured: 5-7 % faster at d = 128).
    constexpr int kPrioScores = 2, kPrioSoftmax = 0, kPrioPV = 1;
    auto tile = [&](auto stage_off, int j0, auto masked) {
        const int k_off = stage_off;  // of the stage among those of K, and of V
        __builtin_amdgcn_s_setprio(kPrioScores);
        f32x16 st[NT];
#pragma unroll
        for (int T = 0; T < NT; ++T)
#pragma unroll
            for (int i = 0; i < 16; ++i) st[T][i] = 0.f;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int T = 0; T < NT; ++T) st[T] = mfma32(fo.frag(smem, k_off, 32 * T, ks), qf[ks], st[T]);
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_setprio(kPrioSoftmax);
        if constexpr (decltype(masked)::value) {
            // key j0 + 32T + 8g + 4h + r is visible iff 32T + 8g + r <= lim (one per-lane bound)
            const int lim = (p.causal ? min(q, p.n - 1) : p.n - 1) - j0 - 32 * wk - 4 * h;
#pragma unroll
            for (int T = 0; T < NT; ++T)
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    st[T][i] = (32 * T + 8 * (i >> 2) + (i & 3) > lim) ? -__builtin_inff() : st[T][i];
        }
        // maximum (IEEE-754-2019, v_maximum3_f32) instead of fmaxf: for fmaxf the compiler first
        // canonicalises every accumulator value (one extra VALU instruction each, for signalling
        // NaNs).  Two chains of three-input maxima over the 32 values of this lane.
        float mx;
        if constexpr (NT == 2) {
            float mxa = max3(st[0][0], st[0][1], st[0][2]), mxb = max3(st[1][0], st[1][1], st[1][2]);
#pragma unroll
            for (int i = 3; i < 15; i += 2) {
                mxa = max3(mxa, st[0][i], st[0][i + 1]);
                mxb = max3(mxb, st[1][i], st[1][i + 1]);
            }
            mx = max3(mxa, mxb, __builtin_elementwise_maximum(st[0][15], st[1][15]));
        } else {
            float mxa = max3(st[0][0], st[0][1], st[0][2]), mxb = max3(st[0][3], st[0][4], st[0][5]);
#pragma unroll
            for (int i = 6; i < 14; i += 4) {
                mxa = max3(mxa, st[0][i], st[0][i + 1]);
                mxb = max3(mxb, st[0][i + 2], st[0][i + 3]);
            }
            mx = max3(mxa, mxb, __builtin_elementwise_maximum(st[0][14], st[0][15]));
        }
        // The reference point m_run of the exponentials only has to be close to the row maximum,
        // not equal to it: it moves (and O, l are rescaled) only when the maximum has grown by
        // more than kSlack, so p = exp2(s - m_run) stays below 2^kSlack and the final O / l and
        // m_run + log2(l) are unchanged.  After the first tiles of a row this almost never
        // happens, which saves the 16 MT + 1 multiplications per lane and tile of the rescaling.
        // Whether it has to move is seen from each lane's own scores; the two halves of a row meet only then.
        // (The exchange between the halves sat in the chain of every tile; the forward alone: d = 128 h16 n1900 causal 32.5 -> 30.5 us,
        // b2 h16 n1024 causal 21.3 -> 19.9, b2 h32 n8192 causal 1057 -> 1047; d = 64 b4 h16 n2048 84.1 -> 82.4.)
        constexpr float kSlack = 8.f;
        if (__builtin_amdgcn_ballot_w64(mx * cs > m_run + kSlack) != 0) {  // also the first finite maximum after -inf
            mx = __builtin_elementwise_maximum(mx, __shfl_xor(mx, 32, 64));
            const float cand = mx * cs;
            const float m_new = cand > m_run + kSlack ? cand : m_run;
            const float alpha = __builtin_amdgcn_exp2f(m_run - (m_new == -__builtin_inff() ? 0.f : m_new));
            l_run *= alpha;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int i = 0; i < 16; ++i) o[mt][i] *= alpha;
            m_run = m_new;
        }
        const float m_use = m_run == -__builtin_inff() ? 0.f : m_run;  // nothing visible yet
        float sum = 0.f;
#pragma unroll
        for (int T = 0; T < NT; ++T)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const float pv = __builtin_amdgcn_exp2f(fmaf(st[T][i], cs, -m_use));
                st[T][i] = pv;
                sum += pv;
            }
        l_run += sum;
        bf16x8 pb[NT][2];
#pragma unroll
        for (int T = 0; T < NT; ++T)
#pragma unroll
            for (int ss = 0; ss < 2; ++ss) pb[T][ss] = acc_to_operand(st[T], ss);
        __builtin_amdgcn_s_setprio(kPrioPV);
        // O^T += V^T P^T in groups of 16 keys; the V^T fragments of the next group are
        // requested before the MFMAs of the current one so that LDS latency hides behind them
        bf16x8 va[2][MT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) va[0][mt] = fo.frag_t(smem, k_off, mt, 0);
#pragma unroll
        for (int g = 0; g < 2 * NT; ++g) {
            if (g + 1 < 2 * NT) {
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
                    va[(g + 1) & 1][mt] = fo.frag_t(smem, k_off, mt, 16 * (g + 1));
            }
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) o[mt] = mfma32(va[g & 1][mt], pb[g >> 1][g & 1], o[mt]);
        }
    };
    // Tiles come in ascending key order, so those that need the bound (they straddle the
    // diagonal or the end of the sequence) are the last ones.  Mask-free tiles go two at a time
    // through a body whose LDS stage offsets are compile-time constants (fragment addresses are
    // then a precomputed register plus an immediate: no vector arithmetic per fetch); the rest
    // takes the masked body with a run-time stage.  Waves may leave the first loop at different
    // tiles; both loops run the same fetches and barriers.
    constexpr int kWaveKeys = 32 * NT;  // keys of a tile that a wave looks at, from j0 + 32 wk on
    auto needs_mask = [&](int j0) {
        return (p.causal && (j0 + 32 * wk + kWaveKeys - 1 > i0 + 32 * wq)) || (j0 + 32 * wk + kWaveKeys > p.n);
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
        tile(std::integral_constant<int, kTileBytes>{}, jb, std::false_type{});
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
        if (!(p.causal && (i0 + 32 * wq + 31 < j0 + 32 * wk))) tile((it & 1) * kTileBytes, j0, std::true_type{});
        wait_direct_loads();
        __syncthreads();
    }

    fwd_finish<D, SPLIT, 4 * kTileBytes>(p, smem, base, bh, i0 + 32 * wq, wq, wk, o, m_run, l_run);
}

// The same forward with the three parts of a tile's work taken from three tiles, so that the matrix instructions of one wave have vector
// instructions of the same wave between them: step t forms the scores of tile t + 1 and the product of tile t - 1 while it
// takes the exponentials of tile t.  For a wave that has a SIMD to itself (d = 256, whose 512 registers leave room for one) or shares
// it with one wave in step with it (SPLIT = 4: eight waves, 64 queries, tiles of 128 keys, each wave 32 of them); with two workgroups on
// a CU the plain body is as fast or faster.  K runs one step ahead of V: during step t the copies of K(t + 2) and V(t) arrive in the places of
// K(t) and V(t - 2).  What is left per step is instruction issue: a wave alone issues one about every 5 cycles, and taking away copies,
// exponentials or maxima one at a time shortens a step by 5 to 25 % each.
// us, before -> now: d = 256  h8 n4096 182 -> 148   b2 h16 n8192 causal 1596 -> 1217   h8 n1024 36 -> 28   h16 n2048 causal 96 -> 73
// (SPLIT = 4: see eight_waves)
template <int D, int SPLIT>
__device__ __forceinline__ void fwd_pipe(const FusedParams p, char* smem) {
    constexpr int NW = SPLIT == 4 ? 8 : 4;  // waves
    constexpr int BR = SPLIT == 1 ? 128 : 64, BC = SPLIT == 4 ? 128 : 64, KS = D / 16, MT = D / 32;
    constexpr int NT = SPLIT == 1 ? 2 : 1;  // 32-key parts of a tile per wave
    constexpr int kTileBytes = BC * D * 2;

    const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, l32 = lane & 31;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave index, uniform
    const int wq = SPLIT == 1 ? w : w & 1, wk = SPLIT == 1 ? 0 : w >> 1;
    const int q_blocks = (p.n + BR - 1) / BR;
    int bh, blk;
    decode_block_causal(blockIdx.x, q_blocks, p.batch * p.heads, p.resident, bh, blk);
    const int ib = p.causal ? q_blocks - 1 - blk : blk;  // causal: longest rows first
    const long base = (long)(bh / p.heads) * p.stride_b + (long)(bh % p.heads) * p.stride_h;
    const long ld = p.stride_n;
    const int i0 = ib * BR;

    int n_it, lp0 = 0;
    if (p.list_ptr) {
        const int32_t* lptr = p.list_ptr + (long)bh * p.list_stride;  // this (batch, head)'s mask
        const int lb = ib / (128 / BR);  // the lists are per 128 rows
        lp0 = lptr[lb];
        int entries = lptr[lb + 1] - lp0;
        if (p.causal) entries = causal_row_entries(p.list_idx, lp0, entries, lb);
        n_it = entries * (128 / BC);
    } else {
        const int k_end = p.causal ? min(p.n, i0 + BR) : p.n;
        n_it = (k_end + BC - 1) / BC;
    }
    auto tile_start = [&](int it) -> int { return tile_start_row<BC>(p.list_idx, lp0, 0, it); };

    // K and V tiles go straight from global memory into the LDS stage that was last read one
    // iteration ago; rows past n repeat the last row and are masked below.
    TileLoader<D, BC, NW> loader;
    loader.init(tid, ld);
    // [K stage 0][K stage 1][V stage 0][V stage 1]: every fetch of a fragment is a register plus an immediate of 16 bits
    auto fetch_k = [&](int j0, int stage) { loader.load(p.K + base, ld, j0, p.n, smem + stage * kTileBytes, tid); };
    auto fetch_v = [&](int j0, int stage) { loader.load(p.V + base, ld, j0, p.n, smem + (2 + stage) * kTileBytes, tid); };
    // the first tiles are requested before the resident Q rows, so that the latencies overlap; those come through the places of V
    auto start_of = [&](int t) { return t < n_it ? tile_start(t) : 0; };
    int j[3] = {start_of(0), start_of(1), start_of(2)};  // of tiles t, t + 1, t + 2
    if (n_it > 0) fetch_k(j[0], 0);
    if (n_it > 1) fetch_k(j[1], 1);

    const int q = i0 + 32 * wq + l32;
    FragOffsets<D> lane_offsets;
    lane_offsets.init(lane);
    bf16x8 qf[KS];
    load_queries<D, SPLIT, 0>(p, base, i0 + 32 * wq, smem + 2 * kTileBytes + w * (32 * D * 2), lane_offsets, lane, qf, [] {});

    f32x16 o[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[mt][i] = 0.f;
    float m_run = -__builtin_inff();  // running maximum of scale * log2(e) * s
    float l_run = 0.f;                // this lane's share of sum exp2(scaled s - m_run)

    // Scores are kept raw in the accumulators and scaled inside the exponential: with
    // cs = |scale| log2(e) > 0 the row maximum commutes with the scaling.  A negative scale is
    // moved into Q (sign flip of the resident fragments), a zero scale becomes a denormal-sized
    // positive one so that masked (-inf) scores stay -inf.
    const float cs = fmaxf(fabsf(p.scale) * kLog2e, 1.17549435e-38f);
    if (p.scale < 0.f) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            u32x4 v = __builtin_bit_cast(u32x4, qf[ks]);
            v ^= 0x80008000u;
            qf[ks] = __builtin_bit_cast(bf16x8, v);
        }
    }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) settle(qf[ks]);
    FragAddrs<D> fo;
    fo.init(lane_offsets);
    if constexpr (SPLIT > 1) fo.shift_rows(32 * wk);
    fo.shift_transposed(2 * kTileBytes);
    wait_direct_loads();
    __syncthreads();

    f32x16 st[NT];      // scores of the tile whose exponentials come next
    bf16x8 pb[NT][2];   // weights of the tile before it
    auto scores = [&](auto off, f32x16 (&s)[NT]) {
#pragma unroll
        for (int T = 0; T < NT; ++T)
#pragma unroll
            for (int i = 0; i < 16; ++i) s[T][i] = 0.f;
        // (fragments are requested a few products ahead and no further: all of them at once would not fit the registers)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            if (ks % 4 == 0) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int T = 0; T < NT; ++T) s[T] = mfma32(fo.frag(smem, off, 32 * T, ks), qf[ks], s[T]);
        }
        __builtin_amdgcn_sched_barrier(0);
        // (d = 256, 128 queries: 470 registers per lane; left to the compiler 512 and 60 bytes of scratch)
#pragma unroll
        for (int T = 0; T < NT; ++T) to_vector_registers(s[T]);
    };
    auto values = [&](auto off) {
#pragma unroll
        for (int g = 0; g < 2 * NT; ++g) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) o[mt] = mfma32(fo.frag_t(smem, off, mt, 16 * g), pb[g >> 1][g & 1], o[mt]);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    auto mask_scores = [&](int j0) {
        const int lim = (p.causal ? min(q, p.n - 1) : p.n - 1) - j0 - 32 * wk - 4 * h;
#pragma unroll
        for (int T = 0; T < NT; ++T)
#pragma unroll
            for (int i = 0; i < 16; ++i)
                st[T][i] = (32 * T + 8 * (i >> 2) + (i & 3) > lim) ? -__builtin_inff() : st[T][i];
    };
    constexpr float kSlack = 8.f;
    // whether some row's reference point has to move, seen from each lane's own scores; then m_run, l_run and `alpha`
    auto reference = [&](float& alpha) -> bool {
        float mxa = max3(st[0][0], st[0][1], st[0][2]), mxb = max3(st[NT - 1][3], st[NT - 1][4], st[NT - 1][5]);
        if constexpr (NT == 1) {
#pragma unroll
            for (int i = 6; i < 14; i += 4) {
                mxa = max3(mxa, st[0][i], st[0][i + 1]);
                mxb = max3(mxb, st[0][i + 2], st[0][i + 3]);
            }
            mxa = max3(mxa, st[0][14], st[0][15]);
        } else {
#pragma unroll
            for (int i = 3; i < 15; i += 2) mxa = max3(mxa, st[0][i], st[0][i + 1]);
            mxb = max3(mxb, st[1][0], st[1][1]);
#pragma unroll
            for (int i = 6; i < 16; i += 2) mxb = max3(mxb, st[1][i], st[1][i + 1]);
            mxb = max3(mxb, st[0][15], st[1][2]);
        }
        float mx = __builtin_elementwise_maximum(mxa, mxb);
        if (__builtin_amdgcn_ballot_w64(mx * cs > m_run + kSlack) == 0) return false;
        mx = __builtin_elementwise_maximum(mx, __shfl_xor(mx, 32, 64));
        const float cand = mx * cs;
        const float m_new = cand > m_run + kSlack ? cand : m_run;
        alpha = __builtin_amdgcn_exp2f(m_run - (m_new == -__builtin_inff() ? 0.f : m_new));
        l_run *= alpha;
        m_run = m_new;
        return true;
    };
    auto weights = [&]() {
        const float m_use = (m_run == -__builtin_inff()) ? 0.f : m_run;
        float sum[2] = {0.f, 0.f};
#pragma unroll
        for (int T = 0; T < NT; ++T)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const float pv = __builtin_amdgcn_exp2f(fmaf(st[T][i], cs, -m_use));
                st[T][i] = pv;
                sum[i & 1] += pv;
            }
        l_run += sum[0] + sum[1];
    };
    auto pack = [&]() {
#pragma unroll
        for (int T = 0; T < NT; ++T)
#pragma unroll
            for (int ss = 0; ss < 2; ++ss) pb[T][ss] = acc_to_operand(st[T], ss);
    };
    auto rescale = [&](float alpha) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) to_vector_registers(o[mt]);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int i = 0; i < 16; ++i) o[mt][i] *= alpha;
    };
    constexpr int kWaveKeys = 32 * NT;
    auto needs_mask = [&](int j0) {
        return (p.causal && (j0 + 32 * wk + kWaveKeys - 1 > i0 + 32 * wq)) || (j0 + 32 * wk + kWaveKeys > p.n);
    };
    auto visible = [&](int j0) { return !(p.causal && (i0 + 32 * wq + 31 < j0 + 32 * wk)); };
    if (n_it > 0) scores(std::integral_constant<int, 0>{}, st);
    __syncthreads();  // the first step overwrites what these scores came from
    bool prev = false;  // pb holds weights
    auto advance = [&](int t) {
        j[0] = j[1];
        j[1] = j[2];
        j[2] = start_of(t + 3);
    };
    constexpr int kInst = TileLoader<D, BC, NW>::kInst;
    // step t: exponentials of tile t, scores of tile t + 1, product of tile t - 1
    auto general = [&](int t) {
        const int j0 = j[0];
        const bool more = t + 1 < n_it;
        if (t + 2 < n_it) fetch_k(j[2], t & 1);
        fetch_v(j0, t & 1);
        float alpha = 1.f;
        f32x16 nx[NT];
        const bool vis = visible(j0);
        if (more) scores((~t & 1) * kTileBytes, nx);
        if (prev) values((~t & 1) * kTileBytes);
        if (vis) {
            if (needs_mask(j0)) mask_scores(j0);
            const bool grow = reference(alpha);
            weights();
            pack();
            if (grow) rescale(alpha);
        }
        prev = vis;
        if (more) {
#pragma unroll
            for (int T = 0; T < NT; ++T) st[T] = nx[T];
        }
        wait_direct_loads();
        __syncthreads();
        advance(t);
    };
    auto fast = [&](int t, auto stage) {
        constexpr int here = decltype(stage)::value * kTileBytes, there = kTileBytes - here;  // stages of tiles t, and t - 1 and t + 1
        static_assert(KS == 2 * MT && 2 * kInst == KS, "as many value as score products, and one copy, per slot");
        float alpha = 1.f;
        // a tile past the end: the first one again, into a place that is not read any more
        const int jk = t + 2 < n_it ? j[2] : 0;
        const __bf16* next_k = p.K + base + (unsigned long long)(unsigned)jk * (unsigned)ld;
        const __bf16* next_v = p.V + base + (unsigned long long)(unsigned)j[0] * (unsigned)ld;
        loader.hold(next_k);
        loader.hold(next_v);
        advance(t);
        bf16x8 fk[KS][NT], fv[KS][NT];
        constexpr int kAhead = 2;
        auto request = [&](auto i) {
#pragma unroll
            for (int T = 0; T < NT; ++T) {
                const int v = i * NT + T;
                fk[i][T] = fo.frag(smem, there, 32 * T, i);
                fv[i][T] = fo.frag_t(smem, there, v % MT, 16 * (v / MT));
            }
        };
        static_for<kAhead>(request);
        const bool grow = reference(alpha);
        const float m_use = (m_run == -__builtin_inff()) ? 0.f : m_run;
        f32x16 nx[NT];
#pragma unroll
        for (int T = 0; T < NT; ++T)
#pragma unroll
            for (int i = 0; i < 16; ++i) nx[T][i] = 0.f;
        float sum[2] = {0.f, 0.f};
        bf16x8 nb[NT][2];
        static_for<KS>([&](auto slot) {
            constexpr int sl = decltype(slot)::value;
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (sl + kAhead < KS) request(std::integral_constant<int, sl + kAhead>{});
#pragma unroll
            for (int T = 0; T < NT; ++T) nx[T] = mfma32(fk[sl][T], qf[sl], nx[T]);
            if constexpr (sl < kInst) loader.load_one(sl, next_k, smem + here);
            else loader.load_one(sl - kInst, next_v, smem + 2 * kTileBytes + here);
            constexpr int per = 16 * NT / KS;
#pragma unroll
            for (int e = 0; e < per; ++e) {
                const int x = sl * per + e, T = x / 16, i = x % 16;
                const float pv = __builtin_amdgcn_exp2f(fmaf(st[T][i], cs, -m_use));
                st[T][i] = pv;
                sum[x & 1] += pv;
                asm volatile("" : "+v"(st[T][i]));  // formed in this slot
            }
#pragma unroll
            for (int x = 0; x < 2 * NT; ++x)
                if ((sl + 1) * per >= 8 * (x + 1) && sl * per < 8 * (x + 1)) nb[x / 2][x % 2] = acc_to_operand(st[x / 2], x % 2);
#pragma unroll
            for (int T = 0; T < NT; ++T) {
                const int v = sl * NT + T, g = v / MT;
                o[v % MT] = mfma32(fv[sl][T], pb[g / 2][g % 2], o[v % MT]);
            }
        });
        __builtin_amdgcn_sched_barrier(0);
        l_run += sum[0] + sum[1];
#pragma unroll
        for (int T = 0; T < NT; ++T) {
            pb[T][0] = nb[T][0];
            pb[T][1] = nb[T][1];
            st[T] = nx[T];
        }
        if (grow) rescale(alpha);
        wait_direct_loads();
        __syncthreads();
    };
    int t = 0;
    // tile t takes the fast body: there is a next one, nothing of t is masked, and the tiles fetched meanwhile lie inside
    auto fast_ok = [&](int t) {
        return prev && t + 1 < n_it && !needs_mask(j[0]) && j[1] + BC <= p.n && (t + 2 >= n_it || j[2] + BC <= p.n);
    };
    while (t < n_it) {
        for (; t < n_it && !((t & 1) && fast_ok(t)); ++t) general(t);
        while (t < n_it && fast_ok(t)) {
            fast(t++, std::integral_constant<int, 1>{});
            if (!(t < n_it && fast_ok(t))) break;
            fast(t++, std::integral_constant<int, 0>{});
        }
    }
    if (prev) values((~n_it & 1) * kTileBytes);
    __syncthreads();  // (the end of the block uses the stages)

    fwd_finish<D, SPLIT, 4 * kTileBytes>(p, smem, base, bh, i0 + 32 * wq, wq, wk, o, m_run, l_run);
}

// Whether a launch of blocks of 64 queries takes eight waves (two query halves, four key parts of tiles of 128 keys, the pipelined
// body) instead of four.  Half the steps, each 1.2 to 1.3 times as long with two waves per SIMD from one workgroup, of which a CU
// holds one: it wins while there is at most one for each CU, unless a row is only a few steps long.  us, four waves -> eight:
//   d = 128  h8 n800 15.8 -> 15.9   h16 n1024 18.5 -> 16.9   h8 n2048 31.1 -> 25.8   h1 n8192 108 -> 79   h16 n2048 (beyond the line) 42 -> 48
//   d = 64   h8 n333 7.2 -> 8.1 and b2 h12 n600 causal 9.9 -> 10.4 (too short)   h8 n1024 13.3 -> 12.0   h4 n1500 18.4 -> 16.0
// Causal blocks differ in length, and a launch that holds all of them at once takes as long as its longest: there one and a half blocks per CU
// in turn are still faster, of long sequences two.  Not where the call has a form with a block mask, whose lists are shorter and in no such
// order (causal with half of the other blocks, d = 128 h14 n1500 19.1 -> 24.8, h4 n8192 66 -> 73), and whose bits have to be those of the
// call without one: the weight gradient alone.  us of all of it, causal:
//   d = 128  h16 n1500 70.4 -> 66.7   h3 n8192 219 -> 193   h4 n8192 267 -> 244   h30 n1024 (480 blocks, beyond) 65.6 -> 69.3
//   d = 64   h20 n1024 39.2 -> 37.4   h5 n4096 86 -> 79   h8 n4000 99.6 -> 95.9   h20 n1500 (480, beyond) 55.0 -> 56.5
inline bool eight_waves(const FusedParams& p, int blocks) {
    return p.n >= 768 && blocks <= (!p.causal || p.mask_form ? 256 : p.n < 2560 ? 384 : 512);
}

constexpr int fwd_per_cu(int d) { return d == 64 ? 4 : d == 128 ? 2 : 1; }

template <int D>
__global__ void __launch_bounds__(kThreads, fwd_per_cu(D)) fwd_kernel(FusedParams p) {
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    fwd_block<D, 1>(p, smem);
}

template <int D>
__global__ void __launch_bounds__(kThreads, fwd_per_cu(D)) fwd_split_kernel(FusedParams p) {
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    fwd_block<D, 2>(p, smem);
}

template <int D, int SPLIT>
__global__ void __launch_bounds__(SPLIT == 4 ? 2 * kThreads : kThreads, D <= 128 ? 2 : 1) fwd_pipe_kernel(FusedParams p) {
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    fwd_pipe<D, SPLIT>(p, smem);
}

template <int D>
static hipError_t launch_fwd(const FusedParams& p, const int32_t* csr_ptr, const int32_t* csr_idx,
                             hipStream_t stream) {
    const int heads = p.batch * p.heads;
    const bool split = few_blocks((p.n + 127) / 128 * heads, fwd_per_cu(D), p.causal && !p.mask_form);
    const int blocks = (split ? (p.n + 63) / 64 : (p.n + 127) / 128) * heads;
    const bool eight = D <= 128 && split && eight_waves(p, blocks);
    void (*fn)(FusedParams);
    if constexpr (D == 256) fn = split ? fwd_pipe_kernel<D, 2> : fwd_pipe_kernel<D, 1>;
    else fn = eight ? fwd_pipe_kernel<D, 4> : split ? fwd_split_kernel<D> : fwd_kernel<D>;
    const int lds = (eight ? 2 : 1) * 2 * (2 * 64 * D * 2);
    const hipError_t e = allow_lds(fn, lds);
    if (e != hipSuccess) return e;
    FusedParams pf = p;
    pf.list_ptr = csr_ptr;
    pf.list_idx = csr_idx;
    if (p.causal && !csr_ptr) pf.resident = causal_resident(blocks, eight ? 1 : fwd_per_cu(D));
    hipLaunchKernelGGL(fn, dim3((unsigned)blocks), dim3(eight ? 2 * kThreads : kThreads), lds, stream, pf);
    return hipGetLastError();
}

hipError_t launch_fwd_fused(int d, const FusedParams& p, const int32_t* csr_ptr, const int32_t* csr_idx,
                            hipStream_t stream) {
    switch (d) {
        case 64: return launch_fwd<64>(p, csr_ptr, csr_idx, stream);
        case 128: return launch_fwd<128>(p, csr_ptr, csr_idx, stream);
        case 256: return launch_fwd<256>(p, csr_ptr, csr_idx, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace attn
