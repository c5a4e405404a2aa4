// Large-d path (d in {512, 1024}; the kernels also take 256): the regime where a d x d working set no longer fits the
// per-CU LDS and register budget (the paper's small-cache case, M = o(d^2)).  It follows the
// four-phase small-cache algorithm of App. C: square tiles with the contraction loop split
// into chunks, and the n x n matrices f (here P) and p (here dS) written to memory between
// the phases:
//   scores kernel : per tile S^T = K Q^T with a k-loop over d-chunks, f = exp(S - LSE); then dP^T = V dO^T
//                   with a second k-loop and p = f o (q - v) (phases 1 to 3; one sweep over the tile
//                   because v = rowsum(dO o O) is precomputed) -> P, dS in HBM
//   gemm kernel   : dV = P^T dO, dK = scale dS^T Q, dQ = scale dS K as tiled products with the
//                   k-loop over n (phase 4 written for dQ/dK/dV instead of A_1^T p A_2)
// The forward uses the same kernels: exp(S) written to HBM with its sum per row and chunk of 64 keys, a combine step for LSE,
// and O = exp(S) V, its rows divided by the sum of the weights as written.
#include <type_traits>

#include "attn_common.hpp"
#include "attn_internal.hpp"
#include "attn_tiles.hpp"

namespace attn {

// ---------------------------------------------------------------------------------- 256 x 256 tiles
// The main loop of the kernels that give a CU one workgroup of eight waves with a 256 x 256 tile, a 128 x 64 block (4 x 2 accumulators) per wave.
// Against the 256 x 128 tiles of two workgroups of four waves it copies two thirds of the bytes per MFMA: 32 instead of 48 of the
// 64 bytes per cycle that the copy path of a CU moves.  Four stages of 32 columns (copies three steps ahead), and the fragments of a
// step's first products are read during the step before it, so that no wave waits for LDS behind a barrier.
// The copies of a step are issued one by one between its products: all of them at its top, every wave waits there for the copy path
// and the matrix pipes stand still (a step of the scores kernel took 2200 cycles for 1024 of products: the sum of both).
//   copy(k, stage, u)       issues copy u of the kCopies of k-step k
//   read_a(stage, ks, t), read_b(stage, ks, t)  a fragment of half ks of the step in that stage (stage, ks, t, u: constants)
// steps: a multiple of 4.  Every wave is past its last read of the stages when this returns.
constexpr int kWide = 256, kWideThreads = 512, kWideStage = kWide * 32 * 2, kWideLds = 8 * kWideStage;  // [A stages][B stages]
constexpr int kRowsStage = 2 * kWideStage, kMeetUnit = 12;  // wide_product_rows
__device__ __forceinline__ void meet() { asm volatile("s_barrier" ::: "memory"); }
template <int kCopies, typename Copy>
__device__ __forceinline__ void wide_begin(Copy copy) {
    static_for<3>([&](auto k) { static_for<kCopies>([&](auto u) { copy(decltype(k)::value, k, u); }); });
}
template <int kCopies, typename Copy, typename ReadA, typename ReadB>
__device__ __forceinline__ void wide_product(int steps, f32x16 (&c)[4][2], Copy copy, ReadA read_a, ReadB read_b) {
#pragma unroll
    for (int tm = 0; tm < 4; ++tm)
#pragma unroll
        for (int tn = 0; tn < 2; ++tn)
#pragma unroll
            for (int i = 0; i < 16; ++i) c[tm][tn][i] = 0.f;
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kCopies) : "memory");
    meet();
    // a product of 32 x 64 x 16 is a unit, eight to a step; the first operand is read three units ahead, the second half a step
    bf16x8 a[4], b[2][2];
    static_for<3>([&](auto t) { a[decltype(t)::value] = read_a(std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{}, t); });
    static_for<2>([&](auto t) { b[0][decltype(t)::value] = read_b(std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{}, t); });
    auto step = [&](int k, auto stage, auto copies, auto next) {
        constexpr int s = decltype(stage)::value;
        constexpr bool kCopy = decltype(copies)::value, kNext = decltype(next)::value;
        static_for<8>([&](auto unit) {
            constexpr int u = decltype(unit)::value, x = u / 4, tm = u % 4;
            if constexpr (tm == 0 && (x == 0 || kNext))
                static_for<2>([&](auto t) {
                    b[x ^ 1][decltype(t)::value] = read_b(std::integral_constant<int, (s + x) % 4>{}, std::integral_constant<int, x ^ 1>{}, t);
                });
            if constexpr (u + 3 < 8 || kNext)
                a[(tm + 3) % 4] = read_a(std::integral_constant<int, (s + (u + 3) / 8) % 4>{}, std::integral_constant<int, (u + 3) / 4 % 2>{},
                                         std::integral_constant<int, (tm + 3) % 4>{});
#pragma unroll
            for (int tn = 0; tn < 2; ++tn) c[tm][tn] = mfma32(b[x][tn], a[tm], c[tm][tn]);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (kCopy && u < kCopies) copy(k + 3, std::integral_constant<int, (s + 3) % 4>{}, unit);
        });
        if constexpr (kCopy) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kCopies) : "memory");  // step k + 2 has landed
        else wait_direct_loads();
        meet();
    };
    constexpr std::true_type yes{};
    constexpr std::false_type no{};
    int k = 0;
    for (; k + 4 < steps; k += 4) {
        step(k, std::integral_constant<int, 0>{}, yes, yes);
        step(k + 1, std::integral_constant<int, 1>{}, yes, yes);
        step(k + 2, std::integral_constant<int, 2>{}, yes, yes);
        step(k + 3, std::integral_constant<int, 3>{}, yes, yes);
    }
    step(k, std::integral_constant<int, 0>{}, yes, yes);
    step(k + 1, std::integral_constant<int, 1>{}, no, yes);
    step(k + 2, std::integral_constant<int, 2>{}, no, yes);
    step(k + 3, std::integral_constant<int, 3>{}, no, no);
}

// The same for operands that are read along their rows: two stages of 64 columns, so that a copy takes whole cache lines of 128 bytes
// (with 32 columns every line crossed the path from L2 twice).  A step is 16 units.  From unit 13 on nothing reads its stage any more: there the waves
// meet, the next stage has landed, and the copies for the step after it begin.
//   copy(k, stage, u)       issues copy u of the kCopies (8 or 9) of k-step k
//   read_a(stage, ks, t), read_b(stage, ks, t)  a fragment of quarter ks
// steps: even, at least 4, or 2 (TWO).  The copies of step 0 have been issued and waited for by each wave (not by all).
template <int kCopies, bool TWO, typename Copy, typename ReadA, typename ReadB>
__device__ __forceinline__ void wide_product_rows(int steps, f32x16 (&c)[4][2], Copy copy, ReadA read_a, ReadB read_b) {
#pragma unroll
    for (int tm = 0; tm < 4; ++tm)
#pragma unroll
        for (int tn = 0; tn < 2; ++tn)
#pragma unroll
            for (int i = 0; i < 16; ++i) c[tm][tn][i] = 0.f;
    meet();
    bf16x8 a[4], b[2][2];
    constexpr std::integral_constant<int, 0> zero{};
    static_for<3>([&](auto t) { a[decltype(t)::value] = read_a(zero, zero, t); });
    static_for<2>([&](auto t) { b[0][decltype(t)::value] = read_b(zero, zero, t); });
    // early: the copies of step k + 1 that are issued here (0 none, 1 all, 2 those that step k - 1 has not); late: step k + 2 exists
    auto step = [&](int k, auto stage, auto early, auto next, auto late) {
        constexpr int s = decltype(stage)::value, kEarly = decltype(early)::value;
        constexpr bool kNext = decltype(next)::value, kLate = decltype(late)::value;
        static_for<16>([&](auto unit) {
            constexpr int u = decltype(unit)::value, x = u / 4, tm = u % 4;
            if constexpr (x < 3 ? tm == 0 : u == kMeetUnit + 1 && kNext)  // (the next stage is not read before the waves have met)
                static_for<2>([&](auto t) {
                    b[(x + 1) & 1][decltype(t)::value] = read_b(std::integral_constant<int, x < 3 ? s : 1 - s>{}, std::integral_constant<int, (x + 1) % 4>{}, t);
                });
            if constexpr (u + 3 < 16 || kNext)
                a[(tm + 3) % 4] = read_a(std::integral_constant<int, u + 3 < 16 ? s : 1 - s>{}, std::integral_constant<int, (u + 3) / 4 % 4>{},
                                         std::integral_constant<int, (tm + 3) % 4>{});
#pragma unroll
            for (int tn = 0; tn < 2; ++tn) c[tm][tn] = mfma32(b[x & 1][tn], a[tm], c[tm][tn]);
            __builtin_amdgcn_sched_barrier(0);
            constexpr int first = kEarly == 1 ? 0 : 3, n = kEarly ? kCopies - first : 0;
            if constexpr (u < n) copy(k + 1, std::integral_constant<int, 1 - s>{}, std::integral_constant<int, first + u>{});
            if constexpr (u == kMeetUnit && kNext) {
                asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
            }
            if constexpr (u > kMeetUnit && kLate) copy(k + 2, stage, std::integral_constant<int, u - kMeetUnit - 1>{});
        });
    };
    constexpr std::integral_constant<int, 1> one{};
    constexpr std::integral_constant<int, 2> two{};
    constexpr std::true_type yes{};
    constexpr std::false_type no{};
    if constexpr (TWO) {
        step(0, zero, one, yes, no);
    } else {
        step(0, zero, one, yes, yes);
        step(1, one, two, yes, yes);
        for (int k = 2; k + 2 < steps; k += 2) {
            step(k, zero, two, yes, yes);
            step(k + 1, one, two, yes, yes);
        }
        step(steps - 2, zero, two, yes, no);
    }
    step(steps - 1, one, zero, no, no);
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Scores kernel.  Accumulator: lane <-> query, register <-> key.  Modes:
//   kProbs    exp2(s - e) of the scores s (times log2 e) written to the workspace in bf16, and e and the row sum per 64-key chunk (the
//             forward).  e is the chunk's largest score rounded up to a whole number, so what is written is at most 1 and no sweep over
//             the scores has to come first (it took 154 of 487 us at b1 h8 n4096 d512); the product kernel aligns the
//             chunks of a row: a whole number is an exact shift of the exponents.
//   kBackward P and dS.  The two products of a tile are formed one after the other - S^T over all of d, then dP^T
//             over all of d - so that the wave can hold its block of the one in progress.  Between the
//             passes P stays in registers, rounded to bf16 as it is stored (dS = P (dP - delta) uses that rounded P).
enum ScoreMode { kProbs = 1, kBackward = 2 };
// O is divided by the sum of what was written, rounded to bf16, not by l: a row that is one key then has that key's value, and the
// roundings of the other rows cancel in part (with l the error at d = 512 was up to 1.2 times that of rounding f).  A chunk's
// stat_m holds e and the ratio of the two sums, which is off one by 2^-9 at most: e + kRatio (ratio - 1).  The combine step leaves there by
// how many powers of two the product kernel lowers the chunk, as exponents of a pair of bf16, and a row's factor in stat_l of its first chunk.
constexpr float kRatio = 16.f;
// Tiles of 256 x 256: a wave has 128 queries x 64 keys, one chunk of the statistics.  P and dS leave a wave
// by itself, 32 rows x 128 bytes at a time through its part of the second stage, so that nothing but the products has a barrier and the first copies
// of the second product arrive during the exponentials.  LSE and delta come with the first copies: a load in between would wait for
// every copy and store in front of it.
// us at b1 h8 n4096 d512, tiles of 128 x 256 by two workgroups of four waves on a CU -> now: forward 206 -> 183, backward 390 -> 317; one tile alone (n = 243)
// 21 -> 13 and 34 -> 23.  What is left of the 317: the chip runs at its power limit (1.6 GHz against 2.4 for one tile alone, whose products
// keep the matrix pipe 85 % busy), and a tenth of a tile is its second exponential half with no products beside it.
// TWO: d = 128, two steps a product.
constexpr int kWideScoreLds = kWideLds + 2 * kWide * 4;
template <int MODE, bool TWO>
__global__ void __launch_bounds__(kWideThreads, 2) ld_scores_kernel(LargeDParams p) {
    constexpr int BK = 64;
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, l32 = lane & 31;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = w >> 2, wn = w & 3;  // queries 128 wm .., keys 64 wn ..
    const int nb = p.npad / kWide;
    const ScoreTile tile = score_tile(blockIdx.x, nb, p.batch * p.heads, p.causal != 0);
    // (uniform, but divided on the vector unit: everything formed from them would stay there)
    const int bh = __builtin_amdgcn_readfirstlane(tile.bh), qb = __builtin_amdgcn_readfirstlane(tile.qb), kb = __builtin_amdgcn_readfirstlane(tile.kb);
    // No workgroup ends here.  Without the branch the compiler forms the addresses of the whole kernel in front of the first product and keeps
    // them: 220 registers instead of 190 in the forward, 256 and 92 bytes of scratch instead of 252 in the backward.
    if (bh >= p.batch * p.heads) return;
    const int batch = __builtin_amdgcn_readfirstlane(bh / p.heads);
    const long base = (long)batch * p.stride_b + (long)(bh - batch * p.heads) * p.stride_h;
    const int k0 = kb * kWide, q0 = qb * kWide;
    const long ld = p.stride_n;

    // this lane's place in the first of the four copies of an operand's step; the next one is 64 rows further
    const int row0 = 8 * w + (lane >> 3);
    const unsigned col0 = (unsigned)((lane & 7) ^ swz<BK>(row0)) * 16u;
    const unsigned lds = __builtin_amdgcn_readfirstlane((unsigned)(size_t)(ATTN_LDS char*)smem);
    // What the loops need per lane is kept to four registers and formed again from them (opaque to the compiler, which would keep all of it:
    // in the second product, with the packed P of the first, there is no register to spare).
    int rq[BK / 16];
#pragma unroll
    for (int ks = 0; ks < BK / 16; ++ks) rq[ks] = tile_off<BK>(128 * wm + l32, 2 * ks + h);
    const int keys_from = (64 * wn - 128 * wm) * (BK * 2) + kWideLds / 2;  // of the key rows, from the place of the query rows
    auto read_a = [&](auto stage, auto half, auto tile) {
        return FragOffsets<BK>::read(smem, rq[decltype(half)::value], decltype(stage)::value * kRowsStage + 32 * decltype(tile)::value * (BK * 2));
    };
    auto read_b = [&](auto stage, auto half, auto tile) {
        int from = keys_from;
        asm volatile("" : "+s"(from));
        return FragOffsets<BK>::read(smem, rq[decltype(half)::value] + from, decltype(stage)::value * kRowsStage + 32 * decltype(tile)::value * (BK * 2));
    };
    auto copier = [&](const __bf16* head_q, const __bf16* head_k) {
        return [&, head_q, head_k](int step, auto stage, auto copy_index) {  // rows past n repeat the last row
            constexpr int u = decltype(copy_index)::value, at = decltype(stage)::value * kRowsStage + (u & 3) * 8192 + (u < 4 ? 0 : kWideLds / 2);
            const int first = min((u < 4 ? q0 : k0) + 64 * (u & 3), p.n - 1);
            const unsigned off = (unsigned)min(row0, p.n - 1 - first) * (unsigned)ld * 2u + col0;
            copy_to_lds<16, true>(lds + 1024u * w, at, off, TileLoader<kWide, 32, 8>::uniform((u < 4 ? head_q : head_k) + (long)first * ld + step * BK));
        };
    };
    const int steps = p.d / BK;
    f32x16 c[4][2];
    // 32 queries x 64 keys of this wave, from 32 tm on, on their way to a matrix in the workspace
    char* mine = smem + kRowsStage + 4096 * w;
    auto put = [&](int t, int g, u32x2 v) { *reinterpret_cast<u32x2*>(mine + tile_off<64>(l32, 4 * t + g) + 8 * h) = v; };
    auto store = [&](__bf16* M, int tm) {
        int row_lane = lane;  // formed here, not carried in registers through the products
        asm volatile("" : "+v"(row_lane));
        const int cc = row_lane & 7;
        wave_exchange();
#pragma unroll
        for (int r = 0; r < 32; r += 8) {
            const int row = r + (row_lane >> 3);
            const long off = ((long)bh * p.npad + q0 + 128 * wm + 32 * tm + row) * p.npad + k0 + 64 * wn + 8 * cc;
            *reinterpret_cast<u32x4*>(M + off) = *reinterpret_cast<const u32x4*>(mine + tile_off<64>(row, cc));
        }
        wave_exchange();
    };

    const float* lds_lse = reinterpret_cast<const float*>(smem + kWideLds) + 128 * wm + l32;
    if constexpr (MODE == kBackward) {  // rows past n repeat the last row
        const unsigned row = (unsigned)min(q0 + (tid & 255), p.n - 1);
        copy_to_lds<4, true>(lds + kWideLds + 256u * w, 0, 4u * row,
                             TileLoader<kWide, 32, 8>::uniform(reinterpret_cast<const __bf16*>((w < 4 ? p.LSE : p.delta) + (long)bh * p.n)));
    }
    const auto first = copier(p.Q + base, p.K + base);
    auto begin = [&](const auto& copy) { static_for<8>([&](auto u) { copy(0, std::integral_constant<int, 0>{}, u); }); };
    begin(first);
    wait_direct_loads();
    wide_product_rows<8, TWO>(steps, c, first, read_a, read_b);
    const float cs = p.scale * kLog2e;
    const bool need_mask = (p.causal && kb == qb) || (k0 + kWide > p.n);
    // the tile that straddles the diagonal or the end of the sequence takes a body of its own (decided per element, it was 17 instructions
    // for each of the scores)
    auto by_mask = [&](auto body) {
        if (need_mask) body(std::true_type{});
        else body(std::false_type{});
    };
    if constexpr (MODE == kProbs) {
        by_mask([&](auto masked) {
// The scaled score is rounded once, for the maximum and for its exponential, in both bodies: joined to the subtraction of e (which the
// compiler does where no mask stands between) a score had one rounding more or less by whether its tile touches the diagonal or the end.
#pragma clang fp contract(off)
#pragma unroll
            for (int tm = 0; tm < 4; ++tm) {
                const int q = q0 + 128 * wm + 32 * tm + l32;
                // key k0 + 64 wn + 32 t + 8 g + 4 h + r is visible iff 32 t + 8 g + r <= lim
                const int lim = (p.causal ? min(q, p.n - 1) : p.n - 1) - k0 - 64 * wn - 4 * h;
                float mx = -__builtin_inff();
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        float v = c[tm][t][i] * cs;
                        if constexpr (decltype(masked)::value) v = 32 * t + acc_row(i, 0) > lim ? -__builtin_inff() : v;
                        c[tm][t][i] = v;
                        mx = fmaxf(mx, v);
                    }
                mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
                const float e = mx == -__builtin_inff() ? 0.f : __builtin_ceilf(mx);
                float sum = 0.f, sum_r = 0.f;
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        float pv[4];
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            pv[r] = __builtin_amdgcn_exp2f(c[tm][t][4 * g + r] - e);
                            sum += pv[r];
                        }
                        u32x2 a;
                        a[0] = q < p.n ? pack_bf16(pv[0], pv[1]) : 0;
                        a[1] = q < p.n ? pack_bf16(pv[2], pv[3]) : 0;
#pragma unroll
                        for (int x = 0; x < 2; ++x) {
                            const unsigned pair = a[x];
                            sum_r += __builtin_bit_cast(float, pair << 16);
                            sum_r += __builtin_bit_cast(float, pair & 0xffff0000u);
                        }
                        put(t, g, a);
                    }
                sum += __shfl_xor(sum, 32, 64);
                sum_r += __shfl_xor(sum_r, 32, 64);
                if (q < p.n && h == 0) {
                    const long o = ((long)bh * (4 * nb) + k0 / 64 + wn) * p.n + q;  // [bh][chunk][query]
                    p.stat_m[o] = mx == -__builtin_inff() ? mx : sum > 0.f ? fmaf(sum_r / sum - 1.f, kRatio, e) : e;
                    p.stat_l[o] = sum;
                }
                store(p.P, tm);
            }
        });
        return;
    }
    const auto second = copier(p.dO + base, p.V + base);
    begin(second);
    uint32_t pk[4][2][8];  // P, rounded to bf16 as it is stored
    by_mask([&](auto masked) {
#pragma unroll
        for (int tm = 0; tm < 4; ++tm) {
            const int q = q0 + 128 * wm + 32 * tm + l32;
            const int lim = (p.causal ? min(q, p.n - 1) : p.n - 1) - k0 - 64 * wn - 4 * h;
            const float lse2 = q < p.n ? lds_lse[32 * tm] * kLog2e : __builtin_inff();
            const bool none = lse2 == -__builtin_inff();  // a fully masked row
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    float pv[4];
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        pv[r] = __builtin_amdgcn_exp2f(c[tm][t][4 * g + r] * cs - lse2);
                        if constexpr (decltype(masked)::value) pv[r] = 32 * t + 8 * g + r > lim ? 0.f : pv[r];
                    }
                    pk[tm][t][2 * g] = none ? 0 : pack_bf16(pv[0], pv[1]);
                    pk[tm][t][2 * g + 1] = none ? 0 : pack_bf16(pv[2], pv[3]);
                    put(t, g, u32x2{pk[tm][t][2 * g], pk[tm][t][2 * g + 1]});
                }
            if (tm == 0) wait_direct_loads();  // the copies, issued an epilogue's quarter ago; no store is in flight yet
            store(p.P, tm);
        }
    });
    wide_product_rows<8, TWO>(steps, c, second, read_a, read_b);
#pragma unroll
    for (int tm = 0; tm < 4; ++tm) {
        const int q = q0 + 128 * wm + 32 * tm + l32;
        const float dl = q < p.n ? lds_lse[kWide + 32 * tm] : 0.f;  // (P is 0 in rows past n)
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                float dv[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const uint32_t word = pk[tm][t][2 * g + (r >> 1)];
                    const float pv = __builtin_bit_cast(float, (r & 1) ? (word & 0xffff0000u) : (word << 16));
                    dv[r] = pv * (c[tm][t][4 * g + r] - dl);
                }
                put(t, g, u32x2{pack_bf16(dv[0], dv[1]), pack_bf16(dv[2], dv[3])});
            }
        store(p.dS, tm);
    }
}

// LSE from the per-chunk sums, and for the product kernel a row's factor and the shift of each of its chunks: the weights of a row are
// lowered to sum to at most 1, so that the product is finite wherever the row of O is.
// A workgroup takes 16 rows; 16 threads per row each fold every 16th chunk into a running (e, sum) pair, and the 16 pairs of a row are folded through LDS (one thread per row alone spent its time
// waiting for one load after the other).  Statistics are [bh][chunk][query]: threads that stand for consecutive
// queries read consecutive floats.
constexpr int kCombineRows = 16, kCombineParts = kThreads / kCombineRows;
__global__ void __launch_bounds__(kThreads) ld_lse_combine_kernel(LargeDParams p) {
    __shared__ float part_m[kCombineParts][kCombineRows], part_l[kCombineParts][kCombineRows], part_r[kCombineParts][kCombineRows];
    __shared__ float row_top[kCombineRows];
    const int rl = threadIdx.x % kCombineRows, g = threadIdx.x / kCombineRows;
    const long rows = (long)p.batch * p.heads * p.n;
    const long r = (long)blockIdx.x * kCombineRows + rl;
    const bool ok = r < rows;
    const int q = ok ? (int)(r % p.n) : 0;
    const int nb = p.npad / 128;
    const int chunks = ok ? 2 * (p.causal ? q / 128 + 1 : nb) : 0;
    const long pitch = p.n;
    const long head = ok ? (r / p.n) * (2 * nb) * pitch + q : 0;
    float M = -__builtin_inff(), L = 0.f, R = 0.f;  // R: the sum of the rounded values
    auto fold = [&](float m, float l, float r) {
        if (m == -__builtin_inff()) {  // nothing visible, or nothing but NaN, which leaves LSE alone and makes the row of O NaN
            R += r;
            return;
        }
        const float top = fmaxf(M, m), old = __builtin_amdgcn_exp2f(M - top), now = __builtin_amdgcn_exp2f(m - top);  // (exp2(-inf) = 0 at the start)
        L = L * old + l * now;
        R = R * old + r * now;
        M = top;
    };
    for (int c = g; c < chunks; c += kCombineParts) {
        const float mc = p.stat_m[head + c * pitch], lc = p.stat_l[head + c * pitch], e = rintf(mc);
        fold(e, lc, mc == -__builtin_inff() ? lc : fmaf(lc, (mc - e) * (1.f / kRatio), lc));
    }
    part_m[g][rl] = M;
    part_l[g][rl] = L;
    part_r[g][rl] = R;
    __syncthreads();
    if (g == 0 && ok) {
        for (int k = 1; k < kCombineParts; ++k) fold(part_m[k][rl], part_l[k][rl], part_r[k][rl]);
        p.LSEout[r] = L > 0.f ? (M + __builtin_amdgcn_logf(L)) * kLn2 : -__builtin_inff();
        const int up = L > 0.f ? max(__builtin_amdgcn_frexp_expf(R), 0) : 0;  // R <= 2^up
        p.stat_l[head] = L > 0.f ? __builtin_amdgcn_ldexpf(1.f, up) / R : 0.f;
        row_top[rl] = M + (float)up;
    }
    __syncthreads();
    // every chunk that the product kernel reads: whole blocks of 256 keys
    const int read = ok ? 4 * (p.causal ? q / 256 + 1 : nb / 2) : 0;
    const float top = row_top[rl];
    for (int c = g; c < read; c += kCombineParts) {
        float* e = p.stat_m + head + c * pitch;
        const float by = c < chunks ? top - rintf(*e) : 0.f;
        *e = __builtin_bit_cast(float, (unsigned)fminf(fmaxf(by, 0.f), 255.f) * 0x00800080u);
    }
}

// C[m][n] = alpha * sum_k A(m, k) B(k, n): 128 x 128 output tile per workgroup, k-loop over the
// sequence.  A is one of the n x n matrices in the workspace (row pitch npad): read as stored
// ([m][k], A_KMAJOR = false: dQ = dS K, O = P V) or transposed ([k][m], A_KMAJOR = true:
// dV = P^T dO, dK = dS^T Q).  B is an [n, d] tensor, k along its rows.  Under the causal rule
// the k-range of a tile shrinks to the blocks the scores kernel wrote.
struct GemmArgs {
    const __bf16* A;  // workspace matrix, [bh][npad][npad]
    const __bf16* B;  // [b, h, n, d] tensor
    __bf16* C;        // [b, h, n, d] tensor
    float alpha;
};

// Output tile of the product kernel: 256 rows x 128 columns per workgroup, a 128 x 64 block (4 x 2
// accumulators) per wave: six fragments from LDS feed eight MFMAs, and a k-step of 32 moves 24 KB
// from global memory for 64 MFMAs.  (With 128 x 128 tiles the copies alone, at the 64 B/clk that
// the vector memory path delivers per CU, took as long as the MFMAs.)
constexpr int kGemmBK = 32, kGemmM = 256;
constexpr int gemm_stage(bool rows) { return (kGemmM + 128) * kGemmBK * 2 + (rows ? kGemmM * 4 : 0); }  // (ROWS: and a shift per row)
// ROWS: A holds exp2(s - e) of the forward.  The chunks of a row are aligned on the way into the product, by a saturating subtraction of
// exponents on pairs of bf16 (two vector instructions per MFMA), and a row of C is multiplied by its factor.  The shifts come with the
// operands, 1 KB per k-step: a load in the step, whose wait would drain the copies in flight, made the forward of scores of
// standard deviation 4 slower than two sweeps were.  us of the forward for scores of standard deviation 1 / 4 / 8, two sweeps with P =
// exp(S - LSE), one sweep with shifts loaded where a tile needs any, and now:
//   d = 512   h8 n4096         487 / 496 / 495   372 / 438 / 436   373 / 378 / 379
//             h8 n4096 causal  296 / 302 / 301   233 / 324 / 324   233 / 235 / 236      h2 n700 causal 58 / - / 59   49 / - / 63   47 / - / 47
//   d = 1024  h8 n2000 causal  177 / - / 180     131 / - / 168     131 / - / 132
template <bool A_KMAJOR, bool ROWS>
__device__ __forceinline__ void gemm_tile(const LargeDParams& p, const GemmArgs& g, char* smem, int bh, int mb, int nb) {
    static_assert(!(A_KMAJOR && ROWS), "the rows of A are the rows of C");
    constexpr int BK = kGemmBK, TM = kGemmM;
    constexpr int kTileA = TM * BK * 2, kTileB = 128 * BK * 2, kStage = gemm_stage(ROWS);
    const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, l32 = lane & 31;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave index, uniform
    const int wm = w >> 1, wn = w & 1;
    const int m0 = mb * TM, n0 = nb * 128;
    const int batch = __builtin_amdgcn_readfirstlane(bh / p.heads);
    const long base = (long)batch * p.stride_b + (long)(bh - batch * p.heads) * p.stride_h;
    const __bf16* gA = g.A + (long)bh * p.npad * p.npad;  // npad x npad, zero beyond n
    const __bf16* gB = g.B + base;
    int k_begin = 0, k_end = p.npad;
    if (p.causal) {
        if (A_KMAJOR) k_begin = m0;   // queries at or after this key block
        else k_end = m0 + TM;         // keys at or before this query block
    }

    f32x16 c[4][2];
#pragma unroll
    for (int tm = 0; tm < 4; ++tm)
#pragma unroll
        for (int tn = 0; tn < 2; ++tn)
#pragma unroll
            for (int i = 0; i < 16; ++i) c[tm][tn][i] = 0.f;
    // Operand tiles go straight from global memory into the LDS stage that was last read one
    // step ago.  Rows of B past n repeat the last row; they meet columns (rows, if A is read
    // transposed) of A that are zero.  Lane offsets of the copies and of the fragment reads are
    // computed once; the k-loop runs three steps per iteration so that the stage offsets are
    // immediates.
    TileLoader<TM, BK> copy_at;   // A read transposed: BK rows of TM columns
    TileLoader<BK, TM> copy_a;    // A as stored: TM rows of BK columns
    TileLoader<128, BK> copy_b;
    if (A_KMAJOR) copy_at.init(tid, p.npad);
    else copy_a.init(tid, p.npad);
    copy_b.init(tid, p.stride_n);
    const unsigned row_off = (unsigned)min(m0 + tid, p.n - 1) * 4u;  // the shift of this lane's row
    auto fetch = [&](int k, int stage) {
        char* at = smem + stage * kStage;
        if (A_KMAJOR) copy_at.load(gA + m0 + (long)k * p.npad, at);
        else copy_a.load(gA + k + (long)m0 * p.npad, at);
        copy_b.load(gB + n0, p.stride_n, k, p.n, at + kTileA, tid);
        if constexpr (ROWS) {  // rows past n repeat the last row
            const float* shifts = p.stat_m + ((long)bh * (p.npad / 64) + k / 64) * p.n;
            const unsigned dst = __builtin_amdgcn_readfirstlane((unsigned)(size_t)(ATTN_LDS char*)at) + 256u * w;
            copy_to_lds<4, false>(dst, kTileA + kTileB, row_off, shifts);
        }
    };
    // A read transposed: one register pair per 32-row tile t.  A as stored: one register per k-step, the 16-byte
    // chunk 2 ks + h of this lane's row (the 32-row tiles are immediates apart); B is then fetched with its k index
    // in the same natural order.  (Reading A in 8-byte halves to match the other order cost 44 % LDS bank conflicts.)
    int ra[4][2], rc[BK / 16], rb[2][2];
    {
        FragOffsets<TM> fa;
        FragOffsets<128> fb;
        fa.init(lane);
        fb.init(lane);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            ra[t][0] = fa.tr(4 * wm + t, 0);
            ra[t][1] = fa.tr(4 * wm + t, 1);
        }
        // A as stored: whole 16-byte chunks of this lane's row (k in natural order), chunk 2 ks + h
#pragma unroll
        for (int ks = 0; ks < BK / 16; ++ks) rc[ks] = tile_off<BK>(128 * wm + l32, 2 * ks + h);
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int half = 0; half < 2; ++half)
                rb[t][half] = (A_KMAJOR ? fb.tr(2 * wn + t, half) : FragOffsets<128>::tr_natural(lane, 2 * wn + t, half)) + kTileA;
    }
    // Three stages: the copies of step k + 2 are issued while step k is multiplied, so two steps' worth of bytes
    // (48 KB per workgroup) are in flight; with two stages the product kernels waited for memory at every step.
    constexpr int kCopiesPerFetch = (kTileA + kTileB) / (1024 * 4) + (ROWS ? 1 : 0);  // per wave
    fetch(k_begin, 0);
    if (k_begin + BK < k_end) {
        fetch(k_begin + BK, 1);
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kCopiesPerFetch) : "memory");
    } else {
        wait_direct_loads();
    }
    __syncthreads();
    auto step = [&](int k, auto stage_index) {
        constexpr int si = decltype(stage_index)::value, so = si * kStage;
        const bool more = k + 2 * BK < k_end;
        if (more) fetch(k + 2 * BK, (si + 2) % 3);
        unsigned lower[4];  // of a pair of weights, per 32-row tile
        if constexpr (ROWS) {
#pragma unroll
            for (int t = 0; t < 4; ++t)
                lower[t] = *reinterpret_cast<const unsigned*>(smem + so + kTileA + kTileB + (128 * wm + 32 * t + l32) * 4);
        }
#pragma unroll
        for (int ks = 0; ks < BK / 16; ++ks) {
            bf16x8 a[4], b[2];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                if (A_KMAJOR) {
                    a[t] = FragOffsets<TM>::read_t(smem, ra[t][0], ra[t][1], 16 * ks, so);
                } else {
                    a[t] = FragOffsets<BK>::read(smem, rc[ks], so + 32 * t * (BK * 2));
                }
            }
            if constexpr (ROWS) {
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
                    u32x4 v = __builtin_bit_cast(u32x4, a[t]);
#pragma unroll
                    for (int x = 0; x < 4; ++x) {
                        const unsigned pair = v[x], by = lower[t];  // (a bit cast of a vector's element takes element 0)
                        v[x] = __builtin_bit_cast(unsigned, __builtin_elementwise_sub_sat(__builtin_bit_cast(u16x2, pair), __builtin_bit_cast(u16x2, by)));
                    }
                    a[t] = __builtin_bit_cast(bf16x8, v);
                }
            }
#pragma unroll
            for (int t = 0; t < 2; ++t)
                b[t] = A_KMAJOR ? FragOffsets<128>::read_t(smem, rb[t][0], rb[t][1], 16 * ks, so)
                                : FragOffsets<128>::read_t_natural(smem, rb[t][0], rb[t][1], 16 * ks, so);
#pragma unroll
            for (int tm = 0; tm < 4; ++tm)
#pragma unroll
                for (int tn = 0; tn < 2; ++tn) c[tm][tn] = mfma32(b[tn], a[tm], c[tm][tn]);
        }
        // step k + 1 must have landed; the copies just issued may stay in flight
        if (more) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kCopiesPerFetch) : "memory");
        else wait_direct_loads();
        __syncthreads();
    };
    int k = k_begin;
    for (; k + 3 * BK <= k_end; k += 3 * BK) {
        step(k, std::integral_constant<int, 0>{});
        step(k + BK, std::integral_constant<int, 1>{});
        step(k + 2 * BK, std::integral_constant<int, 2>{});
    }
    if (k < k_end) {
        step(k, std::integral_constant<int, 0>{});
        if (k + BK < k_end) step(k + BK, std::integral_constant<int, 1>{});
    }
    // accumulator: lane <-> output row, register <-> output column (a wave's own rows and columns: nothing to wait for but its own writes)
    typedef RowStage<64> Rows;
    char* mine = smem + w * Rows::kBytes;
    float factor[4];  // (all of them in front of the stores, behind which a load would wait)
#pragma unroll
    for (int tm = 0; tm < 4; ++tm) {
        const int row = m0 + 128 * wm + 32 * tm + l32;
        factor[tm] = g.alpha;
        if constexpr (ROWS) factor[tm] = row < p.n ? p.stat_l[(long)bh * (p.npad / 64) * p.n + row] : 0.f;
    }
#pragma unroll
    for (int tm = 0; tm < 4; ++tm) {
        const int row0 = m0 + 128 * wm + 32 * tm;
        const float f = factor[tm];
        const bool none = ROWS && f == 0.f;  // a row with no finite sum
#pragma unroll
        for (int tn = 0; tn < 2; ++tn)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float v[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = none ? 0.f : c[tm][tn][4 * q + e] * f;
                Rows::put(mine, 4 * tn + q, u32x2{pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])}, lane);
            }
        if (n0 + 64 * wn < p.d) Rows::store(mine, g.C + base + (long)row0 * p.stride_n + n0 + 64 * wn, p.stride_n, p.n - row0, lane);
    }
}

// C[m][n] = alpha * sum_k A(m, k) B(k, n) as in ld_gemm_kernel, tiles of 256 x 256.
template <bool A_KMAJOR, bool ROWS>
__device__ __forceinline__ void gemm_wide_tile(const LargeDParams& p, const GemmArgs& g, char* smem, int bh, int mb, int nb) {
    static_assert(!(A_KMAJOR && ROWS), "the rows of A are the rows of C");
    constexpr int BK = A_KMAJOR ? 32 : 64, kStage = kWide * BK * 2;  // columns of a step
    const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, l32 = lane & 31;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = w >> 2, wn = w & 3;  // rows 128 wm .., columns 64 wn ..
    const int m0 = mb * kWide, n0 = nb * kWide;
    const int batch = __builtin_amdgcn_readfirstlane(bh / p.heads);
    const long base = (long)batch * p.stride_b + (long)(bh - batch * p.heads) * p.stride_h;
    const __bf16* gA = g.A + (long)bh * p.npad * p.npad;  // npad x npad, zero beyond n
    const __bf16* gB = g.B + base + n0;
    int k_begin = 0, k_end = p.npad;
    if (p.causal) {
        if (A_KMAJOR) k_begin = m0;   // queries at or after this key block
        else k_end = m0 + kWide;      // keys at or before this query block
    }
    // This lane's place in the first copy of an operand's step; the next one is 16 rows of 256 columns further (A read transposed, and
    // B), or 64 rows of 64 (A as stored).  Rows of B past n repeat the last row.
    constexpr int kCopiesA = BK / 16;
    const int row_t = 2 * w + (lane >> 5), row_a = 8 * w + (lane >> 3);
    const unsigned col_t = (unsigned)((lane & 31) ^ swz<kWide>(row_t)) * 16u, col_a = (unsigned)((lane & 7) ^ swz<64>(row_a)) * 16u;
    const unsigned off_a = A_KMAJOR ? (unsigned)row_t * (unsigned)p.npad * 2u + col_t : (unsigned)row_a * (unsigned)p.npad * 2u + col_a;
    const unsigned lds = __builtin_amdgcn_readfirstlane((unsigned)(size_t)(ATTN_LDS char*)smem);
    const unsigned row_off = (unsigned)min(m0 + tid, p.n - 1) * 4u;  // ROWS: the shift of this lane's row (waves 4 to 7: not read)
    auto copy = [&](int step, auto stage, auto copy_index) {
        constexpr int s = decltype(stage)::value, u = decltype(copy_index)::value;
        const int k = k_begin + step * BK;
        typedef TileLoader<kWide, BK, 8> Loader;
        if constexpr (u < kCopiesA) {
            const __bf16* first = A_KMAJOR ? gA + m0 + (long)(k + 16 * u) * p.npad : gA + k + (long)(m0 + 64 * u) * p.npad;
            copy_to_lds<16, true>(lds + 1024u * w, s * kStage + 8192 * u, off_a, Loader::uniform(first));
        } else if constexpr (u < 2 * kCopiesA) {
            constexpr int v = u - kCopiesA;
            const int first = min(k + 16 * v, p.n - 1);
            const unsigned off = (unsigned)min(row_t, p.n - 1 - first) * (unsigned)p.stride_n * 2u + col_t;
            copy_to_lds<16, true>(lds + 1024u * w, kWideLds / 2 + s * kStage + 8192 * v, off, Loader::uniform(gB + (long)first * p.stride_n));
        } else {  // ROWS: rows past n repeat the last row
            const float* shifts = p.stat_m + ((long)bh * (p.npad / 64) + k / 64) * p.n;
            copy_to_lds<4, true>(lds + 256u * w, kWideLds + s * 2048, row_off, Loader::uniform(reinterpret_cast<const __bf16*>(shifts)));
        }
    };
    int ra[4][2], rc[BK / 16], rb[2][2];
    {
        FragOffsets<kWide> f;
        f.init(lane);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            ra[t][0] = f.tr(4 * wm + t, 0);
            ra[t][1] = f.tr(4 * wm + t, 1);
        }
#pragma unroll
        for (int ks = 0; ks < BK / 16; ++ks) rc[ks] = tile_off<BK>(128 * wm + l32, 2 * ks + h);
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int half = 0; half < 2; ++half)
                rb[t][half] = (A_KMAJOR ? f.tr(2 * wn + t, half) : FragOffsets<kWide>::tr_natural(lane, 2 * wn + t, half)) + kWideLds / 2;
    }
    const int r_lower = kWideLds + (128 * wm + l32) * 4;
    auto read_b = [&](auto stage, auto half, auto tile) {
        constexpr int so = decltype(stage)::value * kStage, ks = decltype(half)::value, t = decltype(tile)::value;
        return A_KMAJOR ? FragOffsets<kWide>::read_t(smem, rb[t][0], rb[t][1], 16 * ks, so)
                        : FragOffsets<kWide>::read_t_natural(smem, rb[t][0], rb[t][1], 16 * ks, so);
    };
    auto read_a = [&](auto stage, auto half, auto tile) {
        constexpr int so = decltype(stage)::value * kStage, ks = decltype(half)::value, t = decltype(tile)::value;
        if constexpr (A_KMAJOR) return FragOffsets<kWide>::read_t(smem, ra[t][0], ra[t][1], 16 * ks, so);
        bf16x8 a = FragOffsets<BK>::read(smem, rc[ks], so + 32 * t * (BK * 2));
        if constexpr (ROWS) {
            typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
            const unsigned by = *reinterpret_cast<const unsigned*>(smem + r_lower + decltype(stage)::value * 2048 + 128 * t);
            u32x4 v = __builtin_bit_cast(u32x4, a);
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                const unsigned pair = v[x];
                v[x] = __builtin_bit_cast(unsigned, __builtin_elementwise_sub_sat(__builtin_bit_cast(u16x2, pair), __builtin_bit_cast(u16x2, by)));
            }
            a = __builtin_bit_cast(bf16x8, v);
        }
        return a;
    };
    f32x16 c[4][2];
    const int steps = (k_end - k_begin) / BK;
    if constexpr (A_KMAJOR) {
        wide_begin<4>(copy);
        wide_product<4>(steps, c, copy, read_a, read_b);
    } else {
        constexpr int kCopies = 8 + (ROWS ? 1 : 0);
        static_for<kCopies>([&](auto u) { copy(0, std::integral_constant<int, 0>{}, u); });
        wait_direct_loads();
        wide_product_rows<kCopies, false>(steps, c, copy, read_a, read_b);
    }
    // accumulator: lane <-> output row, register <-> output column
    typedef RowStage<64> Rows;
    char* mine = smem + w * Rows::kBytes;
    float factor[4];  // (all of them in front of the stores, behind which a load would wait)
#pragma unroll
    for (int tm = 0; tm < 4; ++tm) {
        const int row = m0 + 128 * wm + 32 * tm + l32;
        factor[tm] = g.alpha;
        if constexpr (ROWS) factor[tm] = row < p.n ? p.stat_l[(long)bh * (p.npad / 64) * p.n + row] : 0.f;
    }
#pragma unroll
    for (int tm = 0; tm < 4; ++tm) {
        const int row0 = m0 + 128 * wm + 32 * tm;
        const float f = factor[tm];
        const bool none = ROWS && f == 0.f;  // a row with no finite sum
#pragma unroll
        for (int tn = 0; tn < 2; ++tn)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float v[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = none ? 0.f : c[tm][tn][4 * q + e] * f;
                Rows::put(mine, 4 * tn + q, u32x2{pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])}, lane);
            }
        if (n0 + 64 * wn < p.d) Rows::store(mine, g.C + base + (long)row0 * p.stride_n + n0 + 64 * wn, p.stride_n, p.n - row0, lane);
    }
}

struct GradArgs {
    GemmArgs g[3];  // forward: one
};
__device__ __forceinline__ ProductTile find_tile(const LargeDParams& p, int count, int mbs, int nbs) {
    ProductTile t = product_tile(blockIdx.x, count, mbs, nbs, p.batch * p.heads, p.causal != 0);
    t.which = __builtin_amdgcn_readfirstlane(t.which);  // (see ld_scores_kernel)
    t.bh = __builtin_amdgcn_readfirstlane(t.bh);
    t.mb = __builtin_amdgcn_readfirstlane(t.mb);
    t.nb = __builtin_amdgcn_readfirstlane(t.nb);
    return t;
}
template <bool BACKWARD>
__global__ void __launch_bounds__(kThreads, 2) ld_gemm_kernel(LargeDParams p, GradArgs g) {
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    const ProductTile t = find_tile(p, BACKWARD ? 3 : 1, p.npad / kGemmM, (p.d + 127) / 128);
    if constexpr (!BACKWARD) gemm_tile<false, true>(p, g.g[0], smem, t.bh, t.mb, t.nb);
    else if (t.which < 2) gemm_tile<true, false>(p, g.g[t.which], smem, t.bh, t.mb, t.nb);
    else gemm_tile<false, false>(p, g.g[2], smem, t.bh, t.mb, t.nb);
}
template <bool BACKWARD>
__global__ void __launch_bounds__(kWideThreads, 2) ld_gemm_wide_kernel(LargeDParams p, GradArgs g) {
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    const ProductTile t = find_tile(p, BACKWARD ? 3 : 1, p.npad / kWide, p.d / kWide);
    if constexpr (!BACKWARD) gemm_wide_tile<false, true>(p, g.g[0], smem, t.bh, t.mb, t.nb);
    else if (t.which < 2) gemm_wide_tile<true, false>(p, g.g[t.which], smem, t.bh, t.mb, t.nb);
    else gemm_wide_tile<false, false>(p, g.g[2], smem, t.bh, t.mb, t.nb);
}

static hipError_t set_lds(const void* fn, int bytes) {
    return hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
}

constexpr int gemm_lds(bool rows) { return 3 * gemm_stage(rows); }  // three stages of an A and a B tile (72 or 75 KB: two workgroups per CU)
// Whether `tiles` product tiles of 256 x 256 fill the chip: with one for every other CU they are faster than 256 x 128, of which a CU holds
// two; under the causal rule, whose tiles differ in length, they have to be more than the CUs, and longer than one row block (backward).  us of the
// forward / backward, tiles of 256 x 128 -> 256 x 256:
//   full    d = 512  h8 n4096 346 / 716 -> 313 / 672   h8 n1000 46 / 62 -> 49 / 59   h1 n4096 98 / 102 -> 107 / 114   h16 n128 28 / 36 -> 29 / 37
//   causal, forward (tiles)    d = 512  h8 n2040 (128, below) 0.95 as fast   h28 n1780 (392) 1.05   h16 n4090 (512) 1.12   d = 1024  h8 n4090 (512) 1.10
//   causal, backward (tiles)   d = 256  h8 n2040 (192, below) 82 -> 85   h22 n3060 (792) 440 -> 419
//     d = 512  h4 n2550 (240, below) 100 -> 100   h2 n3060 (144, below) 86 -> 95   h12 n1270 (360) 88 -> 85   h8 n2550 (480) 166 -> 156   h133 n250 (798, one block) 97 -> 102
//     d = 1024  h2 n2040 (192, below) 87 -> 91   h10 n1000 (480) 104 -> 98   h4 n2040 (384) 111 -> 105   h6 n3060 (864) 321 -> 313
inline bool wide_products(const LargeDParams& p, unsigned tiles, bool backward) {
    if (p.d < kWide) return false;
    if (!p.causal) return tiles > 128;
    return backward ? tiles > 320 && p.npad > kWide : tiles > 256;
}
template <bool BACKWARD>
static void run_gemm(const LargeDParams& p, const GradArgs& g, hipStream_t stream) {
    const unsigned count = BACKWARD ? 3 : 1, bh = (unsigned)(p.batch * p.heads), wide = count * (unsigned)(p.d / kWide) * (unsigned)(p.npad / kWide) * bh;
    if (wide_products(p, wide, BACKWARD)) {
        hipLaunchKernelGGL(ld_gemm_wide_kernel<BACKWARD>, dim3(wide), dim3(kWideThreads), kWideLds + (BACKWARD ? 0 : 4096), stream, p, g);
        return;
    }
    hipLaunchKernelGGL(ld_gemm_kernel<BACKWARD>, dim3(count * (unsigned)((p.d + 127) / 128) * (unsigned)(p.npad / kGemmM) * bh), dim3(kThreads),
                       gemm_lds(!BACKWARD), stream, p, g);
}

// LDS sizes of the large-d kernels on the current device (set on every call: cheap, and per device).
hipError_t configure_larged() {
    hipError_t e = set_lds(reinterpret_cast<const void*>(ld_scores_kernel<kProbs, false>), kWideScoreLds);
    if (e == hipSuccess) e = set_lds(reinterpret_cast<const void*>(ld_scores_kernel<kBackward, false>), kWideScoreLds);
    if (e == hipSuccess) e = set_lds(reinterpret_cast<const void*>(ld_scores_kernel<kBackward, true>), kWideScoreLds);
    if (e == hipSuccess) e = set_lds(reinterpret_cast<const void*>(ld_gemm_kernel<true>), gemm_lds(false));
    if (e == hipSuccess) e = set_lds(reinterpret_cast<const void*>(ld_gemm_kernel<false>), gemm_lds(true));
    if (e == hipSuccess) e = set_lds(reinterpret_cast<const void*>(ld_gemm_wide_kernel<true>), kWideLds);
    if (e == hipSuccess) e = set_lds(reinterpret_cast<const void*>(ld_gemm_wide_kernel<false>), kWideLds + 4096);
    return e;
}

hipError_t launch_larged(bool backward, const LargeDParams& p, hipStream_t stream) {
    const hipError_t ce = configure_larged();
    if (ce != hipSuccess) return ce;
    const unsigned bh = (unsigned)(p.batch * p.heads);
    const dim3 tiles((unsigned)score_tiles(p.npad / kWide, p.causal != 0) * bh), threads(kWideThreads);
    if (!backward) {  // (d = 512 and 1024)
        hipLaunchKernelGGL((ld_scores_kernel<kProbs, false>), tiles, threads, kWideScoreLds, stream, p);
        const long rows = (long)bh * p.n;
        hipLaunchKernelGGL(ld_lse_combine_kernel, dim3((unsigned)((rows + kCombineRows - 1) / kCombineRows)), dim3(kThreads), 0, stream, p);
        run_gemm<false>(p, GradArgs{{{p.P, p.V, p.Oout, 1.f}}}, stream);
    } else {
        hipLaunchKernelGGL((p.d == 128 ? ld_scores_kernel<kBackward, true> : ld_scores_kernel<kBackward, false>), tiles, threads, kWideScoreLds, stream, p);
        run_gemm<true>(p, GradArgs{{{p.P, p.dO, p.dV, 1.f}, {p.dS, p.Q, p.dK, p.scale}, {p.dS, p.K, p.dQ, p.scale}}}, stream);
    }
    return hipGetLastError();
}

}  // namespace attn
