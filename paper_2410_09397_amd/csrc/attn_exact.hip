// Attention in fp32 arithmetic on the matrix cores, for what the bf16 tile kernels do not take: fp32 tensors of any
// d <= 128, bf16 tensors of any d <= 256 (multiples of 8), and block masks of any edge that is a multiple of 16.
// Nothing is rounded below fp32 on the way:
//   fp32 tensors  every product is v_mfma_f32_16x16x4_f32 (an fp32 multiply-add chain)
//   bf16 tensors  S = Q K^T and dP = dO V^T have bf16 operands, whose products are exact in fp32
//                 (v_mfma_f32_16x16x32_bf16); f and p stay fp32: each is written as the sum of three bf16 numbers
//                 (8 significant bits each, together the 24 of an fp32 number) and the second products run once
//                 per part
// Formulas: A, l, f, O, q, p of App. B.4 with the scale, mask and log-sum-exp readings.
//
// A workgroup owns 16 XG rows (queries for O and dQ, keys for dK and dV); its four waves take the 16- or 32-row
// steps of the other sequence in turn, so that short sequences still fill the chip, and their partial results are
// summed through LDS in a fixed order.  (The row-per-wave FMA kernels of attn_generic.hip read both operands from memory
// for every multiply-add: 1 TFLOP/s at best.  Forward and backward together, before and now: fp32 b1 h1 n256 d64
// 347 -> 24 us, b2 h6 n777 d80 causal 4.25 -> 0.135 ms; bf16 b1 h8 n1500 d96 causal 11.6 -> 0.090 ms.)  No operand passes through LDS: the first products read both operands as
// rows, which is how they lie in memory, and for the second products a lane loads 2 or 4 adjacent columns of each
// of its rows and the output columns come out permuted accordingly (put right at the store).
#include "attn_common.hpp"
#include "attn_internal.hpp"

namespace attn {

namespace {

constexpr int kWaves = 4;

typedef float f32x4_u __attribute__((ext_vector_type(4), aligned(4)));
typedef float f32x2_u __attribute__((ext_vector_type(2), aligned(4)));

template <bool BF>
struct Kind {
    typedef float T;
    typedef f32x4 Row;                          // one lane's share of a 64-byte piece of 16 rows
    static constexpr int kChunk = 16, kG = 1;   // columns per piece; 16-row groups per step
};
template <>
struct Kind<true> {
    typedef __bf16 T;
    typedef bf16x8 Row;
    static constexpr int kChunk = 32, kG = 2;
};

__device__ __forceinline__ f32x4 mma_rows(f32x4 a, f32x4 b, f32x4 c) {
#pragma unroll
    for (int e = 0; e < 4; ++e) c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], b[e], c, 0, 0, 0);
    return c;
}
__device__ __forceinline__ f32x4 mma_rows(bf16x8 a, bf16x8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// Lane l of a wave: r16 = l % 16, h4 = l / 16.
// Row operand: 16 rows, lane <-> row r16, columns chunk * s + (16 bytes at 16 h4) of piece s.  Columns at or past d
// read as zero (only the last 32 of the padded width DP can be).
template <bool BF, bool QUAD, int DP>
struct RowLoader {
    typedef typename Kind<BF>::Row Row;
    typedef typename Kind<BF>::T T;
    static constexpr int kNS = DP / Kind<BF>::kChunk;
    // off: byte offset of the row plus 16 h4
    static __device__ __forceinline__ void load(const char* base, unsigned off, int h4, int d, Row (&out)[kNS]) {
#pragma unroll
        for (int s = 0; s < kNS; ++s) {
            constexpr int kPer = 16 / sizeof(T);
            const int col = Kind<BF>::kChunk * s + kPer * h4;
            if (Kind<BF>::kChunk * (s + 1) <= DP - 32) {
                if constexpr (BF) out[s] = *reinterpret_cast<const bf16x8*>(base + off + 64 * s);
                else out[s] = *reinterpret_cast<const f32x4_u*>(base + off + 64 * s);
            } else if constexpr (BF) {
                const bool ok = col < d;
                const bf16x8 v = *reinterpret_cast<const bf16x8*>(base + (ok ? off + 64 * s : off - 16 * h4));
                const bf16x8 zero = {0, 0, 0, 0, 0, 0, 0, 0};
                out[s] = ok ? v : zero;
            } else if constexpr (QUAD) {
                const bool ok = col < d;
                const f32x4 v = *reinterpret_cast<const f32x4_u*>(base + (ok ? off + 64 * s : off - 16 * h4));
                const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
                out[s] = ok ? v : zero;
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const bool ok = col + e < d;
                    const float v = *reinterpret_cast<const float*>(base + (ok ? off + 64 * s + 4 * e : off - 16 * h4));
                    out[s][e] = ok ? v : 0.f;
                }
            }
        }
    }
};

// Column operand of the second products: for each of the 4 kG rows 16 g + 4 h4 + i of a step the lane loads 4 adjacent
// columns 64 B + 4 r16 of every 64-column group B and, if DP has an odd number of 32-column halves, 2 adjacent columns of
// the last one.  Used as A operand, column b of the lane's 4 (2) gives the 16 output rows m <-> column 64 B + 4 m + b.
template <bool BF, bool QUAD, int DP>
struct ColLoader {
    static constexpr int kN4 = DP / 64, kN2 = (DP % 64) / 32, kRows = 4 * Kind<BF>::kG;
    typedef typename Kind<BF>::T T;
    u32x4 f4[BF ? 1 : (kN4 ? kN4 : 1)][kRows];
    u32x2 h4v[kN4 ? kN4 : 1][kRows];  // bf16: four columns; fp32: unused
    u32x2 f2[BF ? 1 : (kN2 ? kN2 : 1)][kRows];
    uint32_t h2[kN2 ? kN2 : 1][kRows];
    // off[r]: byte offset of row r (no lane part)
    __device__ __forceinline__ void load(const char* base, const unsigned (&off)[kRows], int r16, int d) {
#pragma unroll
        for (int B = 0; B < kN4; ++B) {
            const bool edge = 64 * (B + 1) > DP - 32;
            const int col = 64 * B + 4 * r16;
            const bool ok = !edge || col < d;
#pragma unroll
            for (int r = 0; r < kRows; ++r) {
                if constexpr (BF) {
                    const u32x2 v = *reinterpret_cast<const u32x2*>(base + off[r] + (ok ? 2 * col : 0));
                    h4v[B][r] = v;
                    if (edge && !ok) h4v[B][r] = u32x2{0, 0};
                } else if (QUAD || !edge) {
                    const f32x4 v = *reinterpret_cast<const f32x4_u*>(base + off[r] + (ok ? 4 * col : 0));
                    f4[B][r] = __builtin_bit_cast(u32x4, v);
                    if (edge && !ok) f4[B][r] = u32x4{0, 0, 0, 0};
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const bool oke = col + e < d;
                        const uint32_t v = *reinterpret_cast<const uint32_t*>(base + off[r] + (oke ? 4 * (col + e) : 0));
                        f4[B][r][e] = oke ? v : 0u;
                    }
                }
            }
        }
        if constexpr (kN2 != 0) {
            const int col = 64 * kN4 + 2 * r16;
            const bool ok = col < d;
#pragma unroll
            for (int r = 0; r < kRows; ++r) {
                if constexpr (BF) {
                    const uint32_t v = *reinterpret_cast<const uint32_t*>(base + off[r] + (ok ? 2 * col : 0));
                    h2[0][r] = ok ? v : 0u;
                } else if (QUAD) {
                    const f32x2 v = *reinterpret_cast<const f32x2_u*>(base + off[r] + (ok ? 4 * col : 0));
                    f2[0][r] = ok ? __builtin_bit_cast(u32x2, v) : u32x2{0, 0};
                } else {
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        const bool oke = col + e < d;
                        const uint32_t v = *reinterpret_cast<const uint32_t*>(base + off[r] + (oke ? 4 * (col + e) : 0));
                        f2[0][r][e] = oke ? v : 0u;
                    }
                }
            }
        }
    }
    // the word of row r, 64-group B that holds 16-bit column b (bf16)
    __device__ __forceinline__ bf16x8 block16(int nb) const {
        u32x4 w;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            uint32_t lo, hi;
            int b;
            if (nb < 4 * kN4) {
                b = nb & 3;
                lo = h4v[nb >> 2][2 * j][b >> 1];
                hi = h4v[nb >> 2][2 * j + 1][b >> 1];
            } else {
                b = nb & 1;
                lo = h2[0][2 * j];
                hi = h2[0][2 * j + 1];
            }
            w[j] = __builtin_amdgcn_perm(hi, lo, (b & 1) ? 0x07060302u : 0x05040100u);
        }
        return __builtin_bit_cast(bf16x8, w);
    }
    __device__ __forceinline__ float elem32(int nb, int r) const {
        return __builtin_bit_cast(float, nb < 4 * kN4 ? f4[nb >> 2][r][nb & 3] : f2[0][r][nb & 1]);
    }
};

// A 4 kG x 16 block of f or p as the B operand of the second products.
template <bool BF>
struct Weights;
template <>
struct Weights<false> {
    f32x4 w;
    __device__ __forceinline__ void set(const f32x4 (&v)[1]) { w = v[0]; }
};
template <>
struct Weights<true> {
    bf16x8 part[3];  // v = part[0] + part[1] + part[2], exactly
    __device__ __forceinline__ void set(const f32x4 (&v)[2]) {
        u32x4 w[3];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            float a = v[j >> 1][2 * (j & 1)], b = v[j >> 1][2 * (j & 1) + 1];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                w[k][j] = pack_bf16(a, b);
                a -= __builtin_bit_cast(float, w[k][j] << 16);
                b -= __builtin_bit_cast(float, w[k][j] & 0xffff0000u);
            }
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) part[k] = __builtin_bit_cast(bf16x8, w[k]);
    }
};

// acc[x][nb] += columns^T weights[x] for XG groups of 16 owned rows: every column fragment feeds XG products
template <bool BF, bool QUAD, int DP, int XG>
__device__ __forceinline__ void accumulate(f32x4 (&acc)[XG][DP / 16], const ColLoader<BF, QUAD, DP>& cols, const Weights<BF> (&w)[XG]) {
#pragma unroll
    for (int nb = 0; nb < DP / 16; ++nb) {
        if constexpr (BF) {
            const bf16x8 a = cols.block16(nb);
#pragma unroll
            for (int k = 2; k >= 0; --k)
#pragma unroll
                for (int x = 0; x < XG; ++x) acc[x][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, w[x].part[k], acc[x][nb], 0, 0, 0);
        } else {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float a = cols.elem32(nb, r);
#pragma unroll
                for (int x = 0; x < XG; ++x) acc[x][nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, w[x].w[r], acc[x][nb], 0, 0, 0);
            }
        }
    }
}

// The 16-row groups of the other sequence that a workgroup visits: dense (group g starts at row 16 g) or the kept blocks
// of a block list (edge a multiple of 16), trimmed at group granularity by the causal rule.
struct Groups {
    const int32_t* idx;
    int first, per, block, count, n;
    __device__ __forceinline__ int start(int g) const {  // n (nothing there) past the end
        if (g >= count) return n;
        const int f = first + g;
        if (!idx) return 16 * f;
        return idx[f / per] * block + (f % per) * 16;
    }
};
// rows_after: the owned rows are keys and see queries at or after them; else queries that see keys up to them
__device__ __forceinline__ Groups make_groups(const GenericParams& p, int bh, bool rows_after, int r0, int r_last) {
    Groups g;
    g.n = p.n;
    g.block = p.block;
    const int32_t* ptr = rows_after ? p.csc_ptr : p.csr_ptr;
    if (!ptr) {
        g.idx = nullptr;
        g.per = 1;
        const int all = (p.n + 15) / 16;
        g.first = p.causal && rows_after ? r0 / 16 : 0;
        g.count = (p.causal && !rows_after ? min(all, r_last / 16 + 1) : all) - g.first;
        return g;
    }
    ptr += (long)bh * p.mask_stride;
    g.idx = rows_after ? p.csc_idx : p.csr_idx;
    g.per = p.block / 16;
    int e0 = ptr[r0 / p.block], e1 = ptr[r0 / p.block + 1];
    int skip = 0;
    if (p.causal) {
        if (rows_after) {
            while (e0 < e1 && (g.idx[e0] + 1) * p.block <= r0) ++e0;
            if (e0 < e1 && g.idx[e0] * p.block <= r0) skip = (r0 - g.idx[e0] * p.block) / 16;
        } else {
            while (e0 < e1 && g.idx[e1 - 1] * p.block > r_last) --e1;
        }
    }
    g.first = e0 * g.per + skip;
    g.count = (e1 - e0) * g.per - skip;
    return g;
}

// Sum of the four waves' accumulators (x-th group, row r16: 4 columns at a time) and the store.  `factor(w, row)` scales
// the part of wave w.  red: [kWaves][16 XG][DP + 4] floats.
template <bool BF, bool QUAD, int DP, int XG, typename F>
__device__ __forceinline__ void combine_store(const f32x4 (&acc)[XG][DP / 16], float* red, int w, int lane, char* out, unsigned ldb,
                                              int row0, int n, int d, F factor) {
    constexpr int kPitch = DP + 4;
    typedef typename Kind<BF>::T T;
    const int r16 = lane & 15, h4 = lane >> 4;
#pragma unroll
    for (int x = 0; x < XG; ++x) {
        float* row = red + (w * 16 * XG + 16 * x + r16) * kPitch;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
#pragma unroll
            for (int B = 0; B < DP / 64; ++B)
                *reinterpret_cast<f32x4*>(row + 64 * B + 16 * h4 + 4 * i) =
                    f32x4{acc[x][4 * B][i], acc[x][4 * B + 1][i], acc[x][4 * B + 2][i], acc[x][4 * B + 3][i]};
            if constexpr (DP % 64 != 0)
                *reinterpret_cast<f32x2*>(row + 64 * (DP / 64) + 8 * h4 + 2 * i) =
                    f32x2{acc[x][DP / 16 - 2][i], acc[x][DP / 16 - 1][i]};
        }
    }
    __syncthreads();
    constexpr int kQuads = DP / 4;
    for (int t = w * 64 + lane; t < 16 * XG * kQuads; t += kWaves * 64) {
        const int r = t / kQuads, c = (t % kQuads) * 4;
        f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < kWaves; ++k) {
            const f32x4 v = *reinterpret_cast<const f32x4*>(red + (k * 16 * XG + r) * kPitch + c);
            const float f = factor(k, r);
#pragma unroll
            for (int e = 0; e < 4; ++e) s[e] = fmaf(v[e], f, s[e]);
        }
        if (row0 + r >= n || c >= d) continue;
        char* o = out + (size_t)(row0 + r) * ldb + c * sizeof(T);
        if constexpr (BF) {
            *reinterpret_cast<u32x2*>(o) = u32x2{pack_bf16(s[0], s[1]), pack_bf16(s[2], s[3])};
        } else if constexpr (QUAD) {
            *reinterpret_cast<f32x4_u*>(o) = s;
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (c + e < d) reinterpret_cast<float*>(o)[e] = s[e];
        }
    }
}

template <typename T>
__device__ __forceinline__ const char* head_base(const void* ptr, long base) {
    return reinterpret_cast<const char*>(static_cast<const T*>(ptr) + base);
}

// s * scale * log2(e) - m with the constant in two parts (its rounding alone would shift every f of a row by
// |s| 2^-24 relative)
__device__ __forceinline__ float scaled(float s, float hi, float lo, float m) { return fmaf(s, lo, fmaf(s, hi, -m)); }

template <bool BF, bool QUAD, int DP, int XG>
__global__ void __launch_bounds__(kWaves * 64, 2) exact_fwd_kernel(GenericParams p) {
    typedef Kind<BF> KD;
    typedef typename KD::T T;
    typedef RowLoader<BF, QUAD, DP> Rows;
    typedef ColLoader<BF, QUAD, DP> Cols;
    constexpr int G = KD::kG, NS = Rows::kNS;
    extern __shared__ __attribute__((aligned(16))) float red[];
    __shared__ float st_m[kWaves][16 * XG], st_l[kWaves][16 * XG];
    const int tid = threadIdx.x, lane = tid & 63, r16 = lane & 15, h4 = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int blocks = (p.n + 16 * XG - 1) / (16 * XG);
    int bh, blk;
    decode_block(blockIdx.x, blocks, p.batch * p.heads, bh, blk);
    if (p.causal) blk = blocks - 1 - blk;  // longest rows first
    const int i0 = blk * 16 * XG;
    const long base = (long)(bh / p.heads) * p.stride_b + (long)(bh % p.heads) * p.stride_h;
    const unsigned ldb = (unsigned)p.stride_n * sizeof(T);
    const char *Q = head_base<T>(p.Q, base), *K = head_base<T>(p.K, base), *V = head_base<T>(p.V, base);
    const Groups groups = make_groups(p, bh, false, i0, min(p.n, i0 + 16 * XG) - 1);

    typename KD::Row qf[XG][NS];
    int lim[XG];
#pragma unroll
    for (int x = 0; x < XG; ++x) {
        const int q = i0 + 16 * x + r16;
        Rows::load(Q, (unsigned)min(q, p.n - 1) * ldb + 16 * h4, h4, p.d, qf[x]);
        lim[x] = p.causal ? min(q + 1, p.n) : p.n;
    }
    // a negative scale moves into Q, a zero one becomes a tiny positive one (masked scores must stay -inf)
    float chi = p.c_hi, clo = p.c_lo;
    if (p.scale < 0.f) {
        chi = -chi;
        clo = -clo;
#pragma unroll
        for (int x = 0; x < XG; ++x)
#pragma unroll
            for (int s = 0; s < NS; ++s) qf[x][s] = -qf[x][s];
    }
    chi = fmaxf(chi, 1.17549435e-38f);
    const int lim_all = p.causal ? min(i0 + 1, p.n) : p.n;  // rows below it are visible to every query here

    f32x4 acc[XG][DP / 16];
    float m_run[XG], l_run[XG];
#pragma unroll
    for (int x = 0; x < XG; ++x) {
        m_run[x] = -__builtin_inff();
        l_run[x] = 0.f;
#pragma unroll
        for (int nb = 0; nb < DP / 16; ++nb) acc[x][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    for (int g0 = w * G; g0 < groups.count; g0 += kWaves * G) {
        typename KD::Row kf[G][NS];
        Cols vc;
        int kb[G];
        unsigned off[4 * G];
        bool full = true;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            kb[g] = groups.start(g0 + g);
            full = full && kb[g] + 16 <= lim_all;
            Rows::load(K, (unsigned)min(kb[g] + r16, p.n - 1) * ldb + 16 * h4, h4, p.d, kf[g]);
#pragma unroll
            for (int i = 0; i < 4; ++i) off[4 * g + i] = (unsigned)min(kb[g] + 4 * h4 + i, p.n - 1) * ldb;
        }
        vc.load(V, off, r16, p.d);
        f32x4 st[XG][G];
#pragma unroll
        for (int x = 0; x < XG; ++x)
#pragma unroll
            for (int g = 0; g < G; ++g) st[x][g] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int x = 0; x < XG; ++x) st[x][g] = mma_rows(kf[g][s], qf[x][s], st[x][g]);
        Weights<BF> wt[XG];
#pragma unroll
        for (int x = 0; x < XG; ++x) {
            if (!full) {
#pragma unroll
                for (int g = 0; g < G; ++g)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        st[x][g][i] = kb[g] + 4 * h4 + i < lim[x] ? st[x][g][i] : -__builtin_inff();
            }
            float mx = st[x][0][0];
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int i = 0; i < 4; ++i) mx = __builtin_elementwise_maximum(mx, st[x][g][i]);
            mx = __builtin_elementwise_maximum(mx, __shfl_xor(mx, 16, 64));
            mx = __builtin_elementwise_maximum(mx, __shfl_xor(mx, 32, 64));
            // the reference point of the exponentials follows the row maximum with a slack of 2^8 (see the tile kernels)
            const float cand = mx * chi;
            const bool grow = cand > m_run[x] + 8.f;
            const float m_new = grow ? cand : m_run[x];
            const float m_use = m_new == -__builtin_inff() ? 0.f : m_new;
            if (__builtin_amdgcn_ballot_w64(grow) != 0) {
                const float alpha = __builtin_amdgcn_exp2f(m_run[x] - m_use);
                l_run[x] *= alpha;
#pragma unroll
                for (int nb = 0; nb < DP / 16; ++nb) acc[x][nb] *= alpha;
            }
            m_run[x] = m_new;
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    float v = __builtin_amdgcn_exp2f(scaled(st[x][g][i], chi, clo, m_use));
                    // (with a two-part constant -inf - (-inf) can appear at a masked score)
                    if (!full) v = kb[g] + 4 * h4 + i < lim[x] ? v : 0.f;
                    st[x][g][i] = v;
                    l_run[x] += v;
                }
            wt[x].set(st[x]);
        }
        accumulate<BF, QUAD, DP, XG>(acc, vc, wt);
    }
    // the waves' partial rows: a common reference point per row, then O = sum of parts / l
#pragma unroll
    for (int x = 0; x < XG; ++x) {
        float l = l_run[x];
        l += __shfl_xor(l, 16, 64);
        l += __shfl_xor(l, 32, 64);
        if (h4 == 0) {
            st_m[w][16 * x + r16] = m_run[x];
            st_l[w][16 * x + r16] = l;
        }
    }
    __syncthreads();
    if (tid < 16 * XG) {
        float M = -__builtin_inff(), L = 0.f;
#pragma unroll
        for (int k = 0; k < kWaves; ++k) M = fmaxf(M, st_m[k][tid]);
        const float M_use = M == -__builtin_inff() ? 0.f : M;
        float f[kWaves];
#pragma unroll
        for (int k = 0; k < kWaves; ++k) {
            f[k] = __builtin_amdgcn_exp2f(st_m[k][tid] - M_use);
            L = fmaf(st_l[k][tid], f[k], L);
        }
        const float inv = L > 0.f ? 1.f / L : 0.f;
#pragma unroll
        for (int k = 0; k < kWaves; ++k) st_l[k][tid] = f[k] * inv;
        if (i0 + tid < p.n)
            p.LSE_out[(long)bh * p.n + i0 + tid] =
                L > 0.f ? fmaf(M, kLn2, fmaf(M, -1.90465421e-9f, __builtin_amdgcn_logf(L) * kLn2)) : -__builtin_inff();  // (ln 2 in two parts)
    }
    // (combine_store has a barrier between its two halves)
    combine_store<BF, QUAD, DP, XG>(acc, red, w, lane, const_cast<char*>(head_base<T>(p.O, base)), ldb, i0, p.n, p.d,
                                    [&](int k, int r) { return st_l[k][r]; });
}

// log2 form of a row's LSE in two parts; a row with nothing visible (LSE = -inf) gives f = 0
struct Lse2 {
    float hi, lo;
    __device__ __forceinline__ void set(float lse) {
        constexpr float kLog2eLo = 1.92596299e-8f;  // log2(e) - (float)log2(e)
        hi = lse * kLog2e;
        lo = fmaf(lse, kLog2e, -hi) + lse * kLog2eLo;
        if (lse == -__builtin_inff()) {
            hi = __builtin_inff();
            lo = 0.f;
        }
    }
};

__device__ __forceinline__ float dot_pair(f32x4 a, f32x4 b, float c) {
#pragma unroll
    for (int e = 0; e < 4; ++e) c = fmaf(a[e], b[e], c);
    return c;
}
__device__ __forceinline__ float dot_pair(bf16x8 a, bf16x8 b, float c) {
#pragma unroll
    for (int e = 0; e < 8; ++e) c = fmaf((float)a[e], (float)b[e], c);
    return c;
}

// dQ of 16 XG queries
template <bool BF, bool QUAD, int DP, int XG>
__device__ __forceinline__ void exact_dq(const GenericParams& p, float* red, int bh, int blk) {
    typedef Kind<BF> KD;
    typedef typename KD::T T;
    typedef RowLoader<BF, QUAD, DP> Rows;
    typedef ColLoader<BF, QUAD, DP> Cols;
    constexpr int G = KD::kG, NS = Rows::kNS;
    const int tid = threadIdx.x, lane = tid & 63, r16 = lane & 15, h4 = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i0 = blk * 16 * XG;
    const long base = (long)(bh / p.heads) * p.stride_b + (long)(bh % p.heads) * p.stride_h;
    const unsigned ldb = (unsigned)p.stride_n * sizeof(T);
    const char *Q = head_base<T>(p.Q, base), *K = head_base<T>(p.K, base), *V = head_base<T>(p.V, base);
    const char *dO = head_base<T>(p.dO, base), *O = head_base<T>(p.O_in, base);
    const Groups groups = make_groups(p, bh, false, i0, min(p.n, i0 + 16 * XG) - 1);

    typename KD::Row qf[XG][NS], gf[XG][NS];
    int lim[XG];
    Lse2 lse[XG];
    float delta[XG];
#pragma unroll
    for (int x = 0; x < XG; ++x) {
        const int q = i0 + 16 * x + r16, qc = min(q, p.n - 1);
        const unsigned o = (unsigned)qc * ldb + 16 * h4;
        typename KD::Row of[NS];
        Rows::load(O, o, h4, p.d, of);
        Rows::load(dO, o, h4, p.d, gf[x]);
        Rows::load(Q, o, h4, p.d, qf[x]);
        lim[x] = p.causal ? min(q + 1, p.n) : p.n;
        lse[x].set(p.LSE_in[(long)bh * p.n + qc]);
        float s = 0.f;
#pragma unroll
        for (int k = 0; k < NS; ++k) s = dot_pair(of[k], gf[x][k], s);
        s += __shfl_xor(s, 16, 64);
        s += __shfl_xor(s, 32, 64);
        delta[x] = s;
    }
    const int lim_all = p.causal ? min(i0 + 1, p.n) : p.n;

    f32x4 acc[XG][DP / 16];
#pragma unroll
    for (int x = 0; x < XG; ++x)
#pragma unroll
        for (int nb = 0; nb < DP / 16; ++nb) acc[x][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int g0 = w * G; g0 < groups.count; g0 += kWaves * G) {
        typename KD::Row kf[G][NS], vf[G][NS];
        Cols kc;
        int kb[G];
        unsigned off[4 * G];
        bool full = true;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            kb[g] = groups.start(g0 + g);
            full = full && kb[g] + 16 <= lim_all;
            const unsigned o = (unsigned)min(kb[g] + r16, p.n - 1) * ldb + 16 * h4;
            Rows::load(K, o, h4, p.d, kf[g]);
            Rows::load(V, o, h4, p.d, vf[g]);
#pragma unroll
            for (int i = 0; i < 4; ++i) off[4 * g + i] = (unsigned)min(kb[g] + 4 * h4 + i, p.n - 1) * ldb;
        }
        kc.load(K, off, r16, p.d);
        f32x4 st[XG][G], dp[XG][G];
#pragma unroll
        for (int x = 0; x < XG; ++x)
#pragma unroll
            for (int g = 0; g < G; ++g) st[x][g] = dp[x][g] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int x = 0; x < XG; ++x) {
                    st[x][g] = mma_rows(kf[g][s], qf[x][s], st[x][g]);
                    dp[x][g] = mma_rows(vf[g][s], gf[x][s], dp[x][g]);
                }
        Weights<BF> wt[XG];
#pragma unroll
        for (int x = 0; x < XG; ++x) {
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    float f = __builtin_amdgcn_exp2f(scaled(st[x][g][i], p.c_hi, p.c_lo, lse[x].hi) - lse[x].lo);
                    if (!full) f = kb[g] + 4 * h4 + i < lim[x] ? f : 0.f;
                    dp[x][g][i] = f * (dp[x][g][i] - delta[x]);
                }
            wt[x].set(dp[x]);
        }
        accumulate<BF, QUAD, DP, XG>(acc, kc, wt);
    }
    const float scale = p.scale;
    combine_store<BF, QUAD, DP, XG>(acc, red, w, lane, const_cast<char*>(head_base<T>(p.dQ, base)), ldb, i0, p.n, p.d,
                                    [&](int, int) { return scale; });
}

// dK, dV of 16 XG keys.  v = rowsum(dO o O) of the streamed queries is formed here again from rows that are loaded
// anyway (dO) and one more (O), so that both halves of the backward run in one launch with nothing between them.
template <bool BF, bool QUAD, int DP, int XG>
__device__ __forceinline__ void exact_dkdv(const GenericParams& p, float* red, int bh, int blk) {
    typedef Kind<BF> KD;
    typedef typename KD::T T;
    typedef RowLoader<BF, QUAD, DP> Rows;
    typedef ColLoader<BF, QUAD, DP> Cols;
    constexpr int G = KD::kG, NS = Rows::kNS;
    const int tid = threadIdx.x, lane = tid & 63, r16 = lane & 15, h4 = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j0 = blk * 16 * XG;
    const long base = (long)(bh / p.heads) * p.stride_b + (long)(bh % p.heads) * p.stride_h;
    const unsigned ldb = (unsigned)p.stride_n * sizeof(T);
    const char *Q = head_base<T>(p.Q, base), *K = head_base<T>(p.K, base), *V = head_base<T>(p.V, base);
    const char *dO = head_base<T>(p.dO, base), *O = head_base<T>(p.O_in, base);
    const float* lse_row = p.LSE_in + (long)bh * p.n;
    const Groups groups = make_groups(p, bh, true, j0, min(p.n, j0 + 16 * XG) - 1);

    typename KD::Row kf[XG][NS], vf[XG][NS];
#pragma unroll
    for (int x = 0; x < XG; ++x) {
        const unsigned o = (unsigned)min(j0 + 16 * x + r16, p.n - 1) * ldb + 16 * h4;
        Rows::load(K, o, h4, p.d, kf[x]);
        Rows::load(V, o, h4, p.d, vf[x]);
    }
    f32x4 dk[XG][DP / 16], dv[XG][DP / 16];
#pragma unroll
    for (int x = 0; x < XG; ++x)
#pragma unroll
        for (int nb = 0; nb < DP / 16; ++nb) dk[x][nb] = dv[x][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int g0 = w * G; g0 < groups.count; g0 += kWaves * G) {
        int qb[G];
        unsigned off[4 * G];
        bool full = true;
        f32x4 st[XG][G], dp[XG][G];
#pragma unroll
        for (int x = 0; x < XG; ++x)
#pragma unroll
            for (int g = 0; g < G; ++g) st[x][g] = dp[x][g] = f32x4{0.f, 0.f, 0.f, 0.f};
        float delta[G];
        Lse2 lse[G][4];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            qb[g] = groups.start(g0 + g);
            full = full && qb[g] + 16 <= p.n && (!p.causal || qb[g] >= j0 + 16 * XG - 1);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int r = qb[g] + 4 * h4 + i;
                off[4 * g + i] = (unsigned)min(r, p.n - 1) * ldb;
                lse[g][i].set(lse_row[min(r, p.n - 1)]);
            }
            const unsigned o = (unsigned)min(qb[g] + r16, p.n - 1) * ldb + 16 * h4;
            typename KD::Row qf[NS], gf[NS], of[NS];
            Rows::load(Q, o, h4, p.d, qf);
            Rows::load(dO, o, h4, p.d, gf);
            Rows::load(O, o, h4, p.d, of);
            float s = 0.f;
#pragma unroll
            for (int k = 0; k < NS; ++k) {
                s = dot_pair(of[k], gf[k], s);
#pragma unroll
                for (int x = 0; x < XG; ++x) {
                    st[x][g] = mma_rows(qf[k], kf[x][k], st[x][g]);
                    dp[x][g] = mma_rows(gf[k], vf[x][k], dp[x][g]);
                }
            }
            s += __shfl_xor(s, 16, 64);
            s += __shfl_xor(s, 32, 64);
            delta[g] = s;  // of row r16
        }
        Weights<BF> wp[XG], wd[XG];
        f32x4 dl[G];
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int i = 0; i < 4; ++i) dl[g][i] = __shfl(delta[g], 4 * h4 + i, 64);
#pragma unroll
        for (int x = 0; x < XG; ++x) {
            const int key = j0 + 16 * x + r16;
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    float f = __builtin_amdgcn_exp2f(scaled(st[x][g][i], p.c_hi, p.c_lo, lse[g][i].hi) - lse[g][i].lo);
                    if (!full) {
                        const int q = qb[g] + 4 * h4 + i;
                        f = q < p.n && (!p.causal || q >= key) ? f : 0.f;
                    }
                    st[x][g][i] = f;
                    dp[x][g][i] = f * (dp[x][g][i] - dl[g][i]);
                }
            wp[x].set(st[x]);
            wd[x].set(dp[x]);
        }
        {
            Cols gc;
            gc.load(dO, off, r16, p.d);
            accumulate<BF, QUAD, DP, XG>(dv, gc, wp);
        }
        {
            Cols qc;
            qc.load(Q, off, r16, p.d);
            accumulate<BF, QUAD, DP, XG>(dk, qc, wd);
        }
    }
    const float scale = p.scale;
    combine_store<BF, QUAD, DP, XG>(dv, red, w, lane, const_cast<char*>(head_base<T>(p.dV, base)), ldb, j0, p.n, p.d,
                                    [&](int, int) { return 1.f; });
    __syncthreads();  // red is free again
    combine_store<BF, QUAD, DP, XG>(dk, red, w, lane, const_cast<char*>(head_base<T>(p.dK, base)), ldb, j0, p.n, p.d,
                                    [&](int, int) { return scale; });
}

// One launch for the whole backward: even tiles are query blocks (dQ), odd ones key blocks (dK, dV), the longest of
// both first under the causal rule.
template <bool BF, bool QUAD, int DP, int XG>
__global__ void __launch_bounds__(kWaves * 64, 1) exact_bwd_kernel(GenericParams p) {
    extern __shared__ __attribute__((aligned(16))) float red[];
    const int blocks = (p.n + 16 * XG - 1) / (16 * XG);
    int bh, t;
    decode_block(blockIdx.x, 2 * blocks, p.batch * p.heads, bh, t);
    const int blk = t >> 1;
    if (t & 1) exact_dkdv<BF, QUAD, DP, XG>(p, red, bh, blk);
    else exact_dq<BF, QUAD, DP, XG>(p, red, bh, p.causal ? blocks - 1 - blk : blk);
}

template <bool BF, bool QUAD, int DP, int XG>
hipError_t run_exact(const GenericParams& p, bool backward, hipStream_t stream) {
    constexpr int lds = kWaves * 16 * XG * (DP + 4) * (int)sizeof(float);
    const int blocks = (p.n + 16 * XG - 1) / (16 * XG);
    const void* fn = backward ? reinterpret_cast<const void*>(exact_bwd_kernel<BF, QUAD, DP, XG>)
                              : reinterpret_cast<const void*>(exact_fwd_kernel<BF, QUAD, DP, XG>);
    if (lds > 60 * 1024) {
        const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e != hipSuccess) return e;
    }
    const dim3 grid((unsigned)(blocks * p.batch * p.heads * (backward ? 2 : 1)));
    if (backward)
        hipLaunchKernelGGL((exact_bwd_kernel<BF, QUAD, DP, XG>), grid, dim3(kWaves * 64), lds, stream, p);
    else
        hipLaunchKernelGGL((exact_fwd_kernel<BF, QUAD, DP, XG>), grid, dim3(kWaves * 64), lds, stream, p);
    return hipGetLastError();
}

template <bool BF, bool QUAD>
hipError_t run_width(const GenericParams& p, bool backward, hipStream_t stream) {
    const int w = (p.d + 31) / 32;  // the width is the next multiple of 32: the loads bound columns in the last 32 only
    if (w <= 1) return run_exact<BF, QUAD, 32, 1>(p, backward, stream);
    if (w <= 2) return run_exact<BF, QUAD, 64, 1>(p, backward, stream);
    if (w <= 3) return run_exact<BF, QUAD, 96, 1>(p, backward, stream);
    if (w <= 4) return run_exact<BF, QUAD, 128, 1>(p, backward, stream);
    if constexpr (BF) {
        if (w <= 5) return run_exact<BF, QUAD, 160, 1>(p, backward, stream);
        if (w <= 6) return run_exact<BF, QUAD, 192, 1>(p, backward, stream);
        if (w <= 7) return run_exact<BF, QUAD, 224, 1>(p, backward, stream);
        if (w <= 8) return run_exact<BF, QUAD, 256, 1>(p, backward, stream);
    }
    return hipErrorInvalidValue;
}

}  // namespace

// What is left to the FMA kernels: head dimensions whose accumulators and resident rows do not fit 512 registers per
// lane here, block edges that cut through a 16-row group, and heads of 4 GB and more.
bool exact_takes(bool is_bf16, const GenericParams& p) {
    if (p.d > (is_bf16 ? 256 : 128)) return false;
    if (p.csr_ptr && p.block % 16 != 0) return false;
    // 32-bit byte offsets within one head
    return (double)p.n * (double)p.stride_n * (is_bf16 ? 2.0 : 4.0) < 4.0e9;
}

hipError_t launch_exact(bool is_bf16, bool backward, const GenericParams& p, hipStream_t stream) {
    if (is_bf16) return run_width<true, true>(p, backward, stream);
    return p.d % 4 == 0 ? run_width<false, true>(p, backward, stream) : run_width<false, false>(p, backward, stream);
}

}  // namespace attn
