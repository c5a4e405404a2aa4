// Attention for short sequences and for fp32 arithmetic on the matrix cores.
//
// A workgroup owns 16 XG rows (queries for O and dQ, keys for dK and dV).  Its four or eight waves take the 16- or 32-row
// steps of the other sequence in turn, so that short sequences still fill the chip, and their partial results are
// summed through LDS in a fixed order.  Each wave stages its own steps in LDS (global_load_lds, whole rows, swizzled) and
// waits for its own copies only: there is no barrier before the final sum.  Both uses of a staged tensor, as rows in
// the first products and as columns in the second, read the one copy.
//
// Kinds of arithmetic:
//   kF32   fp32 tensors of any d <= 128: every product is v_mfma_f32_16x16x4_f32 (an fp32 multiply-add chain)
//   kBf3   bf16 tensors of any d <= 256, nothing rounded below fp32 on the way: S = Q K^T and dP = dO V^T have bf16
//          operands, whose products are exact in fp32 (v_mfma_f32_16x16x32_bf16); f and p stay fp32, each written as
//          the sum of three bf16 numbers (8 significant bits each, together the 24 of an fp32 number), and the
//          second products run once per part
// Formulas: A, l, f, O, q, p of App. B.4 with the scale, mask and log-sum-exp readings.
//
// Forward + backward, each timed by itself with calls back to back, against the row-per-wave FMA kernels as they were when these
// were written (1 TFLOP/s: both operands of every multiply-add came from memory): fp32 b1 h1 n256 d64 347 -> 25 us for the step,
// b2 h6 n777 d80 causal 1416 + 2173 -> 20 + 58 us, bf16 b1 h8 n1500 d96 causal 4050 + 5550 -> 18 + 41 us.  What bounds them now:
// fp32 the matrix pipe, busy for 57 % of the CUs' cycles in the long backward and 46 % in the forward; bf16 the vector
// instructions that split f and p (6 to 9 per matrix instruction, which is busy for 19 to 30 %) and the latency of a step;
// the shortest calls, launches.  Reading the row operands straight from global memory in MFMA order, without LDS, costs
// one L1 access per lane (64 per KB instead of 16) and measured 135 and 90 us on the last two.
#include "attn_rows.hpp"

namespace attn {

namespace {

enum Kind { kF32 = 0, kBf3 = 3 };

typedef float f32x4_u __attribute__((ext_vector_type(4), aligned(4)));

template <int KIND>
struct Traits {  // bf16
    typedef __bf16 T;
    typedef bf16x8 Row;                            // one lane's share of a 64-byte piece of 16 rows
    static constexpr int kChunk = 32, kG = 2;      // columns per piece; 16-row groups per step
};
template <>
struct Traits<kF32> {
    typedef float T;
    typedef f32x4 Row;
    static constexpr int kChunk = 16, kG = 1;
};

__device__ __forceinline__ f32x4 mma_rows(f32x4 a, f32x4 b, f32x4 c) {
#pragma unroll
    for (int e = 0; e < 4; ++e) c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], b[e], c, 0, 0, 0);
    return c;
}
__device__ __forceinline__ f32x4 mma_rows(bf16x8 a, bf16x8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ const char* uniform_ptr(const char* p) {
    const unsigned long long a = reinterpret_cast<unsigned long long>(p);
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)a), hi = __builtin_amdgcn_readfirstlane((unsigned)(a >> 32));
    return reinterpret_cast<const char*>(((unsigned long long)hi << 32) | lo);
}

// ------------------------------------------------------------------------------ staged steps
// Lane l of a wave: r16 = l % 16, h4 = l / 16.
//
// One tensor of one step in LDS: 16 kG rows of DP columns (P bytes), 16-byte chunks XOR-swizzled by row so that 8 lanes
// that read one chunk column of 8 rows, and 16 lanes that read 2 chunks of 4 rows, hit every bank at most once.
template <int P>
__device__ __forceinline__ constexpr int stage_swz(int r) {
    constexpr int g = P / 64;  // a row is g quarters of the 64 banks
    if (g % 2 == 1) return (r >> 2) & 3;
    if (g % 4 == 2) return (((r >> 1) & 1) << 1) | ((r >> 2) & 1);
    return ((r & 3) << 2) | ((r >> 2) & 3);
}

// Copies one tensor's step into LDS, one instruction per KB: the lane at LDS position (row, chunk) fetches the chunk
// that the swizzle puts there.  Rows at or past n repeat the last row; columns at or past d (only the last 32 of the
// padded width can be) repeat columns of the same row: the zeros of the owned rows cancel them in the first products, and in
// the second they only reach output columns that are not stored.  QUAD: rows are whole 16-byte pieces; else 4 bytes
// at a time.
template <int KIND, bool QUAD, int DP>
struct StageLoader {
    static constexpr int kEs = sizeof(typename Traits<KIND>::T), G = Traits<KIND>::kG;
    static constexpr int P = DP * kEs, kGroupBytes = 16 * P, kBytes = kGroupBytes * G;
    static constexpr int kPiece = QUAD ? 1024 : 256, kLane = QUAD ? 16 : 4;
    static constexpr int kInst = kGroupBytes / kPiece;  // per 16-row group
    static constexpr int kCopies = kInst * G;           // per step
    unsigned voff[kInst];
    static __device__ __forceinline__ void where(int u, int lane, int d, int& row, unsigned& col_bytes) {
        const int b = u * kPiece + lane * kLane;  // byte position inside the group
        row = b / P;
        const int c = (((b % P) >> 4) ^ stage_swz<P>(row)) * 16 + (b & 15);
        col_bytes = c < d * kEs ? c : 0;
    }
    __device__ __forceinline__ void init(int lane, unsigned ldb, int d) {
#pragma unroll
        for (int u = 0; u < kInst; ++u) {
            int row;
            unsigned cb;
            where(u, lane, d, row, cb);
            voff[u] = (unsigned)row * ldb + cb;
        }
    }
    // start[g]: first row of group g (n: nothing there, the last row is repeated); lds: byte address of the stage
    __device__ __forceinline__ void load(const char* base, const int (&start)[G], int n, unsigned ldb, int d, unsigned lds, int lane) const {
#pragma unroll
        for (int g = 0; g < G; ++g) {
            // the counter of outstanding copies holds 63: whole rows in 16-byte pieces stay below it by the size of LDS
            if constexpr (!QUAD) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(62 - kInst) : "memory");
            const unsigned dst = __builtin_amdgcn_readfirstlane(lds) + g * kGroupBytes;
            if (start[g] + 16 <= n) {
                const char* first = uniform_ptr(base + (size_t)start[g] * ldb);
#pragma unroll
                for (int u = 0; u < kInst; ++u) copy_to_lds<kLane>(dst, u * kPiece, voff[u], first, u == 0);
            } else {
                const char* first = uniform_ptr(base);
                int l = lane;
                asm volatile("" : "+v"(l));  // positions are formed here, not kept in registers for this rare case
#pragma unroll
                for (int u = 0; u < kInst; ++u) {
                    int row;
                    unsigned cb;
                    where(u, l, d, row, cb);
                    copy_to_lds<kLane>(dst, u * kPiece, (unsigned)min(start[g] + row, n - 1) * ldb + cb, first, u == 0);
                }
            }
        }
    }
};

// Waits until at most N of this wave's copies are outstanding (they complete in order; no other vector memory
// instruction is in flight in the loops that use this).
template <int N>
__device__ __forceinline__ void wait_copies() {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N < 63 ? N : 63) : "memory");
}
// This wave's LDS reads have returned: what they read may be overwritten.
__device__ __forceinline__ void wait_reads() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// Reads of a staged step at byte `imm` of the wave's part of LDS.
//   row      operand of the first products: lane <-> row r16 of group g, 16 bytes at 16 h4 of the 64-byte piece s
//   block16  column operand of 16 output columns nb, bf16: transposing reads; element t <-> row 16 (t / 4) + 4 h4 + t % 4
//   block4   fp32: columns 64 B + 4 r16 .. + 3 of row 4 h4 + i, i.e. four operands; used as A operand number b, output row m
//            <-> column 64 B + 4 m + b
//   block2   fp32, the last 32 columns of an odd width: columns 2 r16, 2 r16 + 1
//   block1   fp32, the first 16 of these 32 where d needs no more: column r16
// NARROW (fp32, widths that are not whole 64s, where output columns come four to an operand): columns from DP - 16 on lie past d, and
// their pieces are left out of the first products and of the output columns of the second.  Kernels of their own: tested in
// the loop, d = 96 lost 3.6 %, and bf16, which would save one block of the second products, as much as it gained.  us, forward / backward:
// b2 h6 n777 d80 causal 21.3 / 68.8 -> 19.9 / 61.0, b2 h3 n1000 d16 15.5 / 37.4 -> 11.9 / 26.2, h2 n1000 d77 26.1 / 44.0 -> 24.2 / 39.5
template <int KIND, int DP, bool NARROW>
struct StageReader {
    static constexpr int P = DP * (int)sizeof(typename Traits<KIND>::T), kGroupBytes = 16 * P, kN4 = DP / 64;
    typedef typename Traits<KIND>::Row Row;
    int rb[4], cb[KIND == kF32 ? 4 : 8], c2[KIND == kF32 ? 4 : 1];
    __device__ __forceinline__ void init(int lane, int wave_off) {
        const int r16 = lane & 15, h4 = lane >> 4;
#pragma unroll
        for (int q = 0; q < 4; ++q) rb[q] = wave_off + r16 * P + (((4 * q + h4) ^ stage_swz<P>(r16)) << 4);
        if constexpr (KIND == kF32) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int row = 4 * h4 + i;
                cb[i] = wave_off + row * P + ((r16 ^ stage_swz<P>(row)) << 4);
                const int piece = NARROW ? r16 >> 2 : r16 >> 1, in = NARROW ? 4 * (r16 & 3) : 8 * (r16 & 1);
                c2[i] = wave_off + row * P + 256 * kN4 + ((piece ^ stage_swz<P>(row)) << 4) + in;
            }
        } else {
            const int row = 4 * h4 + (r16 >> 2);
#pragma unroll
            for (int q = 0; q < 8; ++q)
                cb[q] = wave_off + row * P + (((2 * q + ((r16 >> 1) & 1)) ^ stage_swz<P>(row)) << 4) + 8 * (r16 & 1);
        }
    }
    __device__ __forceinline__ Row row(const char* smem, int imm, int g, int s) const {
        return *reinterpret_cast<const Row*>(smem + rb[s & 3] + (imm + 256 * (s >> 2) + g * kGroupBytes));
    }
    __device__ __forceinline__ bf16x8 block16(const char* smem, int imm, int nb) const {
        const char* a = smem + cb[nb & 7] + (imm + 256 * (nb >> 3));
        const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((i16x4 ATTN_LDS*)a);
        const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((i16x4 ATTN_LDS*)(a + kGroupBytes));
        typedef short i16x8 __attribute__((ext_vector_type(8)));
        const i16x8 r = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        return __builtin_bit_cast(bf16x8, r);
    }
    __device__ __forceinline__ f32x4 block4(const char* smem, int imm, int B, int i) const {
        return *reinterpret_cast<const f32x4*>(smem + cb[i] + (imm + 256 * B));
    }
    __device__ __forceinline__ f32x2 block2(const char* smem, int imm, int i) const {
        return *reinterpret_cast<const f32x2*>(smem + c2[i] + imm);
    }
    __device__ __forceinline__ float block1(const char* smem, int imm, int i) const {
        return *reinterpret_cast<const float*>(smem + c2[i] + imm);
    }
};

// An owned row (lane <-> row r16) straight from memory in MFMA order, zero at and past column d.  row: its first byte.
template <int KIND, bool QUAD, int DP>
__device__ __forceinline__ void load_owned(const char* row, int h4, int d, typename Traits<KIND>::Row (&out)[DP / Traits<KIND>::kChunk]) {
    typedef typename Traits<KIND>::T T;
    constexpr int kPer = 16 / sizeof(T);
#pragma unroll
    for (int s = 0; s < DP / Traits<KIND>::kChunk; ++s) {
        const int col = Traits<KIND>::kChunk * s + kPer * h4;
        if constexpr (KIND != kF32) {
            const bf16x8 v = *reinterpret_cast<const bf16x8*>(row + (col < d ? 2 * col : 0));
            const bf16x8 zero = {0, 0, 0, 0, 0, 0, 0, 0};
            out[s] = col < d ? v : zero;
        } else if constexpr (QUAD) {
            const f32x4 v = *reinterpret_cast<const f32x4_u*>(row + (col < d ? 4 * col : 0));
            const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
            out[s] = col < d ? v : zero;
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float v = *reinterpret_cast<const float*>(row + (col + e < d ? 4 * (col + e) : 0));
                out[s][e] = col + e < d ? v : 0.f;
            }
        }
    }
}

// ------------------------------------------------------------------------------ second products
// A 16 kG x 16 block of f or p (lane <-> owned row) as the B operand of the second products.
template <int KIND>
struct Weights {
    bf16x8 part[KIND];  // kBf3: v = part[0] + part[1] + part[2], exactly
    __device__ __forceinline__ void set(const f32x4 (&v)[2]) {
        u32x4 w[KIND];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            float a = v[j >> 1][2 * (j & 1)], b = v[j >> 1][2 * (j & 1) + 1];
#pragma unroll
            for (int k = 0; k < KIND; ++k) {
                w[k][j] = pack_bf16(a, b);
                a -= __builtin_bit_cast(float, w[k][j] << 16);
                b -= __builtin_bit_cast(float, w[k][j] & 0xffff0000u);
            }
        }
#pragma unroll
        for (int k = 0; k < KIND; ++k) part[k] = __builtin_bit_cast(bf16x8, w[k]);
    }
};
template <>
struct Weights<kF32> {
    f32x4 w;
    __device__ __forceinline__ void set(const f32x4 (&v)[1]) { w = v[0]; }
};

// acc[x][nb] += columns^T weights[x]: every column operand read from LDS feeds XG products (per part)
template <int KIND, int DP, int XG, bool NARROW>
__device__ __forceinline__ void accumulate(f32x4 (&acc)[XG][DP / 16], const StageReader<KIND, DP, NARROW>& rd, const char* smem, int imm,
                                           const Weights<KIND> (&w)[XG]) {
    if constexpr (KIND != kF32) {
#pragma unroll
        for (int nb = 0; nb < DP / 16; ++nb) {
            const bf16x8 a = rd.block16(smem, imm, nb);
#pragma unroll
            for (int k = KIND - 1; k >= 0; --k)
#pragma unroll
                for (int x = 0; x < XG; ++x) acc[x][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, w[x].part[k], acc[x][nb], 0, 0, 0);
        }
    } else {
#pragma unroll
        for (int B = 0; B < DP / 64; ++B)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const f32x4 a = rd.block4(smem, imm, B, i);
#pragma unroll
                for (int b = 0; b < 4; ++b)
#pragma unroll
                    for (int x = 0; x < XG; ++x)
                        acc[x][4 * B + b] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[b], w[x].w[i], acc[x][4 * B + b], 0, 0, 0);
            }
        if constexpr (DP % 64 != 0) {
            if constexpr (NARROW) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float a = rd.block1(smem, imm, i);
#pragma unroll
                    for (int x = 0; x < XG; ++x)
                        acc[x][DP / 16 - 2] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, w[x].w[i], acc[x][DP / 16 - 2], 0, 0, 0);
                }
                return;
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const f32x2 a = rd.block2(smem, imm, i);
#pragma unroll
                for (int b = 0; b < 2; ++b)
#pragma unroll
                    for (int x = 0; x < XG; ++x)
                        acc[x][DP / 16 - 2 + b] =
                            __builtin_amdgcn_mfma_f32_16x16x4f32(a[b], w[x].w[i], acc[x][DP / 16 - 2 + b], 0, 0, 0);
            }
        }
    }
}

// ------------------------------------------------------------------------------ which steps
// The 16-row groups of the other sequence that a workgroup visits: dense (group g starts at row 16 g) or the kept blocks
// of a block list (edge a multiple of 16), trimmed at group granularity by the causal rule.
struct Groups {
    const int32_t* idx;
    int first, per, block, count, n;
    __device__ __forceinline__ int start(int g) const {  // n (nothing there) past the end
        if (g >= count) return n;
        const int f = first + g;
        if (!idx) return 16 * f;
        // through the constant address space: a scalar load (the lists are never written by these kernels)
        typedef const int32_t __attribute__((address_space(4))) * const_i32_ptr;
        return ((const_i32_ptr)(unsigned long long)idx)[__builtin_amdgcn_readfirstlane(f / per)] * block + (f % per) * 16;
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

// ------------------------------------------------------------------------------ sum over the waves
// `factor(w, row)` scales the part of wave w.  red: [NW][16 XG][DP + 4] floats, over the stages.
// Returns whether this thread met a sum that is not finite.
template <int KIND, bool QUAD, int DP, int XG, int NW, bool NARROW, typename F>
__device__ __forceinline__ bool combine_store(const f32x4 (&acc)[XG][DP / 16], float* red, int w, int lane, char* out, unsigned ldb,
                                              int row0, int n, int d, F factor) {
    constexpr int kPitch = DP + 4;
    typedef typename Traits<KIND>::T T;
    const int r16 = lane & 15, h4 = lane >> 4;
    __syncthreads();  // every wave is past its last step (or past the previous sum)
#pragma unroll
    for (int x = 0; x < XG; ++x) {
        float* row = red + (w * 16 * XG + 16 * x + r16) * kPitch;
        if constexpr (KIND != kF32) {
#pragma unroll
            for (int nb = 0; nb < DP / 16; ++nb) *reinterpret_cast<f32x4*>(row + 16 * nb + 4 * h4) = acc[x][nb];
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
#pragma unroll
                for (int B = 0; B < DP / 64; ++B)
                    *reinterpret_cast<f32x4*>(row + 64 * B + 16 * h4 + 4 * i) =
                        f32x4{acc[x][4 * B][i], acc[x][4 * B + 1][i], acc[x][4 * B + 2][i], acc[x][4 * B + 3][i]};
                if constexpr (DP % 64 != 0) {
                    if constexpr (NARROW) row[64 * (DP / 64) + 4 * h4 + i] = acc[x][DP / 16 - 2][i];
                    else *reinterpret_cast<f32x2*>(row + 64 * (DP / 64) + 8 * h4 + 2 * i) = f32x2{acc[x][DP / 16 - 2][i], acc[x][DP / 16 - 1][i]};
                }
            }
        }
    }
    __syncthreads();
    constexpr int kQuads = DP / 4;
    float bad = 0.f;  // 0 x finite stays 0
    for (int t = w * 64 + lane; t < 16 * XG * kQuads; t += NW * 64) {
        const int r = t / kQuads, c = (t % kQuads) * 4;
        f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < NW; ++k) {
            const f32x4 v = *reinterpret_cast<const f32x4*>(red + (k * 16 * XG + r) * kPitch + c);
            const float f = factor(k, r);
#pragma unroll
            for (int e = 0; e < 4; ++e) s[e] = fmaf(v[e], f, s[e]);
        }
        if (row0 + r >= n || c >= d) continue;
#pragma unroll
        for (int e = 0; e < 4; ++e) bad = fmaf(s[e], 0.f, bad);
        char* o = out + (size_t)(row0 + r) * ldb + c * sizeof(T);
        if constexpr (KIND != kF32) {
            *reinterpret_cast<u32x2*>(o) = u32x2{pack_bf16(s[0], s[1]), pack_bf16(s[2], s[3])};
        } else if constexpr (QUAD) {
            *reinterpret_cast<f32x4_u*>(o) = s;
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (c + e < d) reinterpret_cast<float*>(o)[e] = s[e];
        }
    }
    return !(bad == 0.f);
}

// The rows of a workgroup once more, one per wave, where a result is not finite (the barrier is passed by every wave
// either way).  In a matrix product an infinity or a NaN reaches results that must not depend on it: a weight of zero at an
// invisible row of the step, a zero column of the padded width and the three bf16 parts of a weight all meet it.  The redone
// rows have what the definition gives.  One test per result; a test of the staged steps doubled the accumulators' registers.
template <int XG, int NW, typename F>
__device__ __forceinline__ void redo_rows(bool bad, int w, int row0, int n, F row) {
    if (!__syncthreads_or(bad)) return;
    // the kernel's argument is read again here: held in scalar registers for this rare part, it made them spill
    unsigned long long args = (unsigned long long)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(args));
    const GenericParams& p = *reinterpret_cast<const GenericParams*>(args);
#pragma unroll 1
    for (int r = row0 + w; r < min(n, row0 + 16 * XG); r += NW) row(p, r);
}

template <typename T>
__device__ __forceinline__ const char* head_base(const void* ptr, long base) {
    return reinterpret_cast<const char*>(static_cast<const T*>(ptr) + base);
}

// s * scale * log2(e) - m with the constant in two parts (its rounding alone would shift every f of a row by
// |s| 2^-24 relative)
__device__ __forceinline__ float scaled(float s, float hi, float lo, float m) { return fmaf(s, lo, fmaf(s, hi, -m)); }

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

// Owned 16-row groups per workgroup: bf16 operands of 16 x 32 feed one 16-cycle MFMA each, which is twice the LDS rate,
// so there each feeds two; fp32 operands feed 32 cycles per 256 bytes.
template <int KIND, int DP>
constexpr int kOwned = KIND != kF32 && DP <= 128 ? 2 : 1;
// Whether the key owners can form v = rowsum(dO o O) of the streamed queries themselves (then the backward is one launch):
// where the stages of Q, dO and O fit LDS together.  Which of the two a call takes: own_rows.
template <int DP>
constexpr bool kCanOwnDelta = DP <= 192;

// One step's stage of a wave: K, V forward; Q, dO, O (or v) and LSE backward.
template <int KIND, bool QUAD, int DP, bool OWN>
__host__ __device__ constexpr int stage_lds(bool backward) {
    typedef StageLoader<KIND, QUAD, DP> L;
    return L::kBytes * (backward && OWN ? 3 : 2) + (backward ? 512 : 0);
}
// Whether a workgroup can have eight waves (their stages fit LDS) instead of four; which it has is decided at launch.
template <int KIND, bool QUAD, int DP, bool OWN>
__host__ __device__ constexpr bool eight_waves(bool backward) {
    if (backward && KIND != kF32 && DP == 128) return false;  // (256 registers per lane and accumulators beside them)
    return 8 * stage_lds<KIND, QUAD, DP, OWN>(backward) <= 156 * 1024;
}

// Which (batch, head), block and role (0: queries, 1: keys) a workgroup has.  Dense lists of equal length: all of one
// head on one XCD.  Under the causal rule a block's work grows with its distance from one end, and which workgroups share
// a CU decides the run time: workgroup L lands on CU L mod 256 while there is room, so ranks (longest first over all heads)
// are laid out in rounds of 256, every second one reversed, and each CU gets a long, a short, a long ... one.  (In
// head order some CUs had twice the average work.)  Time in head order over time in this order, the causal half of the shapes
// below: forward 0.9 to 1.65, backward 0.82 to 1.66, on average 1.0 up to 256 workgroups, 1.1 to 1.5 up to 2048; beyond 4096 0.96 to 1.06:
// there the order no longer matters, and it needs no upper line.
__device__ __forceinline__ void balanced_block(int linear, int blocks, int bh_total, int roles, int causal, int& bh, int& rank, int& role) {
    const int per = bh_total * roles;
    if (!causal) {
        decode_block(linear, blocks * roles, bh_total, bh, rank);
        role = rank % roles;
        rank /= roles;
        return;
    }
    const int round = linear >> 8, in = linear & 255;
    int r = linear;
    if ((round & 1) && (round + 1) * 256 <= blocks * per) r = round * 256 + (31 - (in >> 3)) * 8 + (in & 7);
    rank = r / per;
    const int rest = r % per;
    bh = rest / roles;
    role = rest % roles;
}

// ------------------------------------------------------------------------------------ forward
// fp32, 32 columns: as many waves as the registers of the loop alone allow (64 instead of 68, which the redone rows would take: 7 %
// of the time of 32768 heads of 4 rows)
template <int KIND, bool QUAD, int DP, int XG, int NW, bool NARROW>
__global__ void __launch_bounds__(NW * 64, KIND == kF32 && DP == 32 ? (QUAD ? 8 : 7) : 2) stream_fwd_kernel(GenericParams p) {
    typedef Traits<KIND> TR;
    typedef typename TR::T T;
    typedef StageLoader<KIND, QUAD, DP> Loader;
    constexpr int G = TR::kG, NS = DP / TR::kChunk, kV = Loader::kBytes;
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    __shared__ float st_m[NW][16 * XG], st_l[NW][16 * XG];
    const int tid = threadIdx.x, lane = tid & 63, r16 = lane & 15, h4 = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int blocks = (p.n + 16 * XG - 1) / (16 * XG);
    int bh, blk, role;
    balanced_block(blockIdx.x, blocks, p.batch * p.heads, 1, p.causal, bh, blk, role);
    if (p.causal) blk = blocks - 1 - blk;  // longest rows first
    const int i0 = blk * 16 * XG;
    const long base = (long)(bh / p.heads) * p.stride_b + (long)(bh % p.heads) * p.stride_h;
    const unsigned ldb = (unsigned)p.stride_n * sizeof(T);
    const char *Q = head_base<T>(p.Q, base), *K = head_base<T>(p.K, base), *V = head_base<T>(p.V, base);
    const Groups groups = make_groups(p, bh, false, i0, min(p.n, i0 + 16 * XG) - 1);

    constexpr int C = Loader::kCopies;
    const int wave_off = w * stage_lds<KIND, QUAD, DP, false>(false);
    const unsigned lds = (unsigned)(size_t)(ATTN_LDS char*)smem + wave_off;
    Loader ld;
    ld.init(lane, ldb, p.d);
    StageReader<KIND, DP, NARROW> rd;
    rd.init(lane, wave_off);
    int kb[G], kb_next[G];
    auto next_step = [&](int g0) {
#pragma unroll
        for (int g = 0; g < G; ++g) kb_next[g] = groups.start(g0 + g);
    };

    // The place of K is free as soon as the first products have read it, that of V after the second ones: the copies of
    // the next step go out there, each with the other half of a step to arrive in.  The first step is requested in front
    // of the owned rows, so that the latencies overlap.
    if (w * G < groups.count) {
        next_step(w * G);
        ld.load(K, kb_next, p.n, ldb, p.d, lds, lane);
        ld.load(V, kb_next, p.n, ldb, p.d, lds + kV, lane);
    }

    typename TR::Row qf[XG][NS];
    int lim[XG];
#pragma unroll
    for (int x = 0; x < XG; ++x) {
        const int q = i0 + 16 * x + r16;
        load_owned<KIND, QUAD, DP>(Q + (size_t)min(q, p.n - 1) * ldb, h4, p.d, qf[x]);
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
#pragma unroll
    for (int x = 0; x < XG; ++x)
#pragma unroll
        for (int s = 0; s < NS; ++s) settle(qf[x][s]);
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
    for (int g0 = w * G; g0 < groups.count; g0 += NW * G) {
        const bool more = g0 + NW * G < groups.count;
        bool full = true;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            kb[g] = kb_next[g];
            full = full && kb[g] + 16 <= lim_all;
        }
        wait_copies<C>();  // K is there; V, requested after it, may be on its way
        f32x4 st[XG][G];
#pragma unroll
        for (int x = 0; x < XG; ++x)
#pragma unroll
            for (int g = 0; g < G; ++g) st[x][g] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < NS - NARROW; ++s)
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const typename TR::Row kf = rd.row(smem, 0, g, s);
#pragma unroll
                for (int x = 0; x < XG; ++x) st[x][g] = mma_rows(kf, qf[x][s], st[x][g]);
            }
        wait_reads();
        // the scores are taken out of the matrix pipe before the branch: read behind it, the compiler (ROCm 7.2) left out the
        // wait that an MFMA result needs on the path around the copies
#pragma unroll
        for (int x = 0; x < XG; ++x)
#pragma unroll
            for (int g = 0; g < G; ++g) asm volatile("" : "+v"(st[x][g]));
        if (more) {
            next_step(g0 + NW * G);
            ld.load(K, kb_next, p.n, ldb, p.d, lds, lane);
        }
        Weights<KIND> wt[XG];
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
            // The reference point of the exponentials follows the row maximum with a slack of 2^8 (see the tile kernels).
            // Whether it has to move is seen from each lane's own scores; the maximum over the lanes of a row is formed
            // only then (two cross-lane reads, some 250 cycles).
            if (__builtin_amdgcn_ballot_w64(mx * chi > m_run[x] + 8.f) != 0) {
                mx = __builtin_elementwise_maximum(mx, __shfl_xor(mx, 16, 64));
                mx = __builtin_elementwise_maximum(mx, __shfl_xor(mx, 32, 64));
                const float cand = mx * chi;
                const float m_new = cand > m_run[x] + 8.f ? cand : m_run[x];
                const float alpha = __builtin_amdgcn_exp2f(m_run[x] - (m_new == -__builtin_inff() ? 0.f : m_new));
                l_run[x] *= alpha;
#pragma unroll
                for (int nb = 0; nb < DP / 16; ++nb) acc[x][nb] *= alpha;
                m_run[x] = m_new;
            }
            const float m_use = m_run[x] == -__builtin_inff() ? 0.f : m_run[x];  // nothing visible yet
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
        if (more) wait_copies<C>();
        else wait_copies<0>();
        accumulate(acc, rd, smem, kV, wt);
        if (more) {
            wait_reads();
            ld.load(V, kb_next, p.n, ldb, p.d, lds + kV, lane);
        }
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
        for (int k = 0; k < NW; ++k) M = fmaxf(M, st_m[k][tid]);
        const float M_use = M == -__builtin_inff() ? 0.f : M;
        float f[NW];
#pragma unroll
        for (int k = 0; k < NW; ++k) {
            f[k] = __builtin_amdgcn_exp2f(st_m[k][tid] - M_use);
            L = fmaf(st_l[k][tid], f[k], L);
        }
        const float inv = L > 0.f ? 1.f / L : 0.f;
#pragma unroll
        for (int k = 0; k < NW; ++k) st_l[k][tid] = f[k] * inv;
        if (i0 + tid < p.n)
            p.LSE_out[(long)bh * p.n + i0 + tid] =
                L > 0.f ? fmaf(M, kLn2, fmaf(M, -1.90465421e-9f, __builtin_amdgcn_logf(L) * kLn2)) : -__builtin_inff();  // (ln 2 in two parts)
    }
    const bool bad = combine_store<KIND, QUAD, DP, XG, NW, NARROW>(acc, reinterpret_cast<float*>(smem), w, lane, const_cast<char*>(head_base<T>(p.O, base)),
                                                       ldb, i0, p.n, p.d, [&](int k, int r) { return st_l[k][r]; });
    redo_rows<XG, NW>(bad, w, i0, p.n, [&](const GenericParams& p, int i) {
        row_forward<T, row_words<T>(DP)>(p, bh, i, lane, reinterpret_cast<float*>(smem) + w * DP);
    });
}

// ----------------------------------------------------------------------------------- backward
// dQ of 16 XG queries
template <int KIND, bool QUAD, int DP, int XG, int NW, bool NARROW, bool OWN>
__device__ __forceinline__ void stream_dq(const GenericParams& p, char* smem, int bh, int blk) {
    typedef Traits<KIND> TR;
    typedef typename TR::T T;
    typedef StageLoader<KIND, QUAD, DP> Loader;
    constexpr int G = TR::kG, NS = DP / TR::kChunk, kV = Loader::kBytes;
    const int tid = threadIdx.x, lane = tid & 63, r16 = lane & 15, h4 = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i0 = blk * 16 * XG;
    const long base = (long)(bh / p.heads) * p.stride_b + (long)(bh % p.heads) * p.stride_h;
    const unsigned ldb = (unsigned)p.stride_n * sizeof(T);
    const char *Q = head_base<T>(p.Q, base), *K = head_base<T>(p.K, base), *V = head_base<T>(p.V, base);
    const char *dO = head_base<T>(p.dO, base), *O = head_base<T>(p.O_in, base);
    const Groups groups = make_groups(p, bh, false, i0, min(p.n, i0 + 16 * XG) - 1);

    constexpr int C = Loader::kCopies;
    const int wave_off = w * stage_lds<KIND, QUAD, DP, OWN>(true);
    const unsigned lds = (unsigned)(size_t)(ATTN_LDS char*)smem + wave_off;
    Loader ld;
    ld.init(lane, ldb, p.d);
    StageReader<KIND, DP, NARROW> rd;
    rd.init(lane, wave_off);
    int kb[G], kb_next[G];
    auto next_step = [&](int g0) {
#pragma unroll
        for (int g = 0; g < G; ++g) kb_next[g] = groups.start(g0 + g);
    };

    if (w * G < groups.count) {
        next_step(w * G);
        ld.load(V, kb_next, p.n, ldb, p.d, lds + kV, lane);
        ld.load(K, kb_next, p.n, ldb, p.d, lds, lane);
    }

    typename TR::Row qf[XG][NS], gf[XG][NS];
    int lim[XG];
    Lse2 lse[XG];
    float delta[XG];
#pragma unroll
    for (int x = 0; x < XG; ++x) {
        const int q = i0 + 16 * x + r16, qc = min(q, p.n - 1);
        typename TR::Row of[NS];
        load_owned<KIND, QUAD, DP>(O + (size_t)qc * ldb, h4, p.d, of);
        load_owned<KIND, QUAD, DP>(dO + (size_t)qc * ldb, h4, p.d, gf[x]);
        load_owned<KIND, QUAD, DP>(Q + (size_t)qc * ldb, h4, p.d, qf[x]);
        lim[x] = p.causal ? min(q + 1, p.n) : p.n;
        lse[x].set(p.LSE_in[(long)bh * p.n + qc]);
        float s = 0.f;
#pragma unroll
        for (int k = 0; k < NS; ++k) s = dot_pair(of[k], gf[x][k], s);
        s += __shfl_xor(s, 16, 64);
        s += __shfl_xor(s, 32, 64);
        delta[x] = s;
#pragma unroll
        for (int k = 0; k < NS; ++k) {
            settle(qf[x][k]);
            settle(gf[x][k]);
        }
        settle(lse[x].hi);
    }
    const int lim_all = p.causal ? min(i0 + 1, p.n) : p.n;

    f32x4 acc[XG][DP / 16];
#pragma unroll
    for (int x = 0; x < XG; ++x)
#pragma unroll
        for (int nb = 0; nb < DP / 16; ++nb) acc[x][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int g0 = w * G; g0 < groups.count; g0 += NW * G) {
        const bool more = g0 + NW * G < groups.count;
        bool full = true;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            kb[g] = kb_next[g];
            full = full && kb[g] + 16 <= lim_all;
        }
        f32x4 st[XG][G], dp[XG][G];
#pragma unroll
        for (int x = 0; x < XG; ++x)
#pragma unroll
            for (int g = 0; g < G; ++g) st[x][g] = dp[x][g] = f32x4{0.f, 0.f, 0.f, 0.f};
        wait_copies<C>();  // V is there; K, requested after it, may be on its way
#pragma unroll
        for (int s = 0; s < NS - NARROW; ++s)
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const typename TR::Row vf = rd.row(smem, kV, g, s);
#pragma unroll
                for (int x = 0; x < XG; ++x) dp[x][g] = mma_rows(vf, gf[x][s], dp[x][g]);
            }
        wait_copies<0>();
#pragma unroll
        for (int s = 0; s < NS - NARROW; ++s)
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const typename TR::Row kf = rd.row(smem, 0, g, s);
#pragma unroll
                for (int x = 0; x < XG; ++x) st[x][g] = mma_rows(kf, qf[x][s], st[x][g]);
            }
        wait_reads();
        // the scores are taken out of the matrix pipe before the branch: read behind it, the compiler (ROCm 7.2) left out the
        // wait that an MFMA result needs on the path around the copies
#pragma unroll
        for (int x = 0; x < XG; ++x)
#pragma unroll
            for (int g = 0; g < G; ++g) asm volatile("" : "+v"(st[x][g]));
        if (more) {
            next_step(g0 + NW * G);
            ld.load(V, kb_next, p.n, ldb, p.d, lds + kV, lane);
        }
        Weights<KIND> wt[XG];
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
        accumulate(acc, rd, smem, 0, wt);
        if (more) {
            wait_reads();
            ld.load(K, kb_next, p.n, ldb, p.d, lds, lane);
        }
    }
    const float scale = p.scale;
    const bool bad = combine_store<KIND, QUAD, DP, XG, NW, NARROW>(acc, reinterpret_cast<float*>(smem), w, lane, const_cast<char*>(head_base<T>(p.dQ, base)),
                                                       ldb, i0, p.n, p.d, [&](int, int) { return scale; });
    redo_rows<XG, NW>(bad, w, i0, p.n, [&](const GenericParams& p, int i) {
        float* rows = reinterpret_cast<float*>(smem) + w * 2 * DP;
        row_dq<T, row_words<T>(DP)>(p, bh, i, lane, row_delta<T>(p, bh, i, lane), rows, rows + DP);
    });
}

// dK, dV of 16 XG keys.  With OWN the row sums v of the streamed queries are formed here again (fp32: from the
// fragments at hand; bf16: the diagonal of dO O^T), so that both halves of the backward run in one launch with nothing
// between them.
template <int KIND, bool QUAD, int DP, int XG, int NW, bool NARROW, bool OWN>
__device__ __forceinline__ void stream_dkdv(const GenericParams& p, char* smem, int bh, int blk) {
    typedef Traits<KIND> TR;
    typedef typename TR::T T;
    typedef StageLoader<KIND, QUAD, DP> Loader;
    constexpr int G = TR::kG, NS = DP / TR::kChunk, kG_ = Loader::kBytes, kO = 2 * Loader::kBytes;
    constexpr int kRows = stage_lds<KIND, QUAD, DP, OWN>(true) - 512;  // LSE (and v) of the step's queries
    const int tid = threadIdx.x, lane = tid & 63, r16 = lane & 15, h4 = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j0 = blk * 16 * XG;
    const long base = (long)(bh / p.heads) * p.stride_b + (long)(bh % p.heads) * p.stride_h;
    const unsigned ldb = (unsigned)p.stride_n * sizeof(T);
    const char *Q = head_base<T>(p.Q, base), *K = head_base<T>(p.K, base), *V = head_base<T>(p.V, base);
    const char *dO = head_base<T>(p.dO, base), *O = head_base<T>(p.O_in, base);
    const char* lse_row = uniform_ptr(reinterpret_cast<const char*>(p.LSE_in + (long)bh * p.n));
    const char* delta_row = uniform_ptr(reinterpret_cast<const char*>(p.delta + (long)bh * p.n));
    const Groups groups = make_groups(p, bh, true, j0, min(p.n, j0 + 16 * XG) - 1);

    constexpr int C = Loader::kCopies;
    const int wave_off = w * stage_lds<KIND, QUAD, DP, OWN>(true);
    const unsigned lds = (unsigned)(size_t)(ATTN_LDS char*)smem + wave_off;
    Loader ld;
    ld.init(lane, ldb, p.d);
    StageReader<KIND, DP, NARROW> rd;
    rd.init(lane, wave_off);
    int qb[G], qb_next[G];
    auto next_step = [&](int g0) {
#pragma unroll
        for (int g = 0; g < G; ++g) qb_next[g] = groups.start(g0 + g);
    };
    // O of the next step (or v) and LSE, one float per query
    auto fetch_rows = [&]() {
        int first = qb_next[0];
        if constexpr (G == 2) first += (lane & 16) ? qb_next[1] - qb_next[0] : 0;
        const int r = first + r16;
        const unsigned off = (unsigned)min(r, p.n - 1) * 4u;
        if constexpr (OWN) ld.load(O, qb_next, p.n, ldb, p.d, lds + kO, lane);
        else copy_to_lds<4, true>(__builtin_amdgcn_readfirstlane(lds), kRows + 256, off, delta_row);
        copy_to_lds<4, true>(__builtin_amdgcn_readfirstlane(lds), kRows, off, lse_row);
    };

    if (w * G < groups.count) {
        next_step(w * G);
        fetch_rows();
        ld.load(dO, qb_next, p.n, ldb, p.d, lds + kG_, lane);
        ld.load(Q, qb_next, p.n, ldb, p.d, lds, lane);
    }

    typename TR::Row kf[XG][NS], vf[XG][NS];
#pragma unroll
    for (int x = 0; x < XG; ++x) {
        const size_t o = (size_t)min(j0 + 16 * x + r16, p.n - 1) * ldb;
        load_owned<KIND, QUAD, DP>(K + o, h4, p.d, kf[x]);
        load_owned<KIND, QUAD, DP>(V + o, h4, p.d, vf[x]);
#pragma unroll
        for (int k = 0; k < NS; ++k) {
            settle(kf[x][k]);
            settle(vf[x][k]);
        }
    }
    f32x4 dk[XG][DP / 16], dv[XG][DP / 16];
#pragma unroll
    for (int x = 0; x < XG; ++x)
#pragma unroll
        for (int nb = 0; nb < DP / 16; ++nb) dk[x][nb] = dv[x][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int g0 = w * G; g0 < groups.count; g0 += NW * G) {
        const bool more = g0 + NW * G < groups.count;
        bool full = true;
        f32x4 st[XG][G], dp[XG][G];
#pragma unroll
        for (int x = 0; x < XG; ++x)
#pragma unroll
            for (int g = 0; g < G; ++g) st[x][g] = dp[x][g] = f32x4{0.f, 0.f, 0.f, 0.f};
        float lse[G][4], dl[G][4];
        wait_copies<C>();  // O, LSE and dO are there; Q, requested after them, may be on its way
#pragma unroll
        for (int g = 0; g < G; ++g) {
            qb[g] = qb_next[g];
            full = full && qb[g] + 16 <= p.n && (!p.causal || qb[g] >= j0 + 16 * XG - 1);
            const f32x4 l4 = *reinterpret_cast<const f32x4*>(smem + wave_off + kRows + 64 * g + 16 * h4);
            f32x4 d4;
            if constexpr (!OWN) d4 = *reinterpret_cast<const f32x4*>(smem + wave_off + kRows + 256 + 64 * g + 16 * h4);
            f32x4 diag = {0.f, 0.f, 0.f, 0.f};
            float dot = 0.f;
#pragma unroll
            for (int s = 0; s < NS - NARROW; ++s) {
                const typename TR::Row gr = rd.row(smem, kG_, g, s);
#pragma unroll
                for (int x = 0; x < XG; ++x) dp[x][g] = mma_rows(gr, vf[x][s], dp[x][g]);
                if constexpr (OWN) {
                    typename TR::Row orow = rd.row(smem, kO, g, s);
                    constexpr int kPer = 16 / sizeof(T);
                    if (TR::kChunk * (s + 1) > DP - 32 && p.d < DP) {
#pragma unroll
                        for (int e = 0; e < kPer; ++e)
                            if (TR::kChunk * s + kPer * h4 + e >= p.d) orow[e] = (T)0.f;
                    }
                    if constexpr (KIND == kF32) dot = dot_pair(orow, gr, dot);
                    else diag = mma_rows(orow, gr, diag);
                }
            }
            if constexpr (OWN && KIND == kF32) {
                dot += __shfl_xor(dot, 16, 64);
                dot += __shfl_xor(dot, 32, 64);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                lse[g][i] = l4[i];
                // row 4 h4 + i: its sum is in every lane with that r16 (fp32), or on the diagonal (bf16)
                if constexpr (!OWN) dl[g][i] = d4[i];
                else if constexpr (KIND == kF32) dl[g][i] = __shfl(dot, 4 * h4 + i, 64);
                else dl[g][i] = __shfl(diag[i], 20 * h4 + i, 64);
            }
        }
        wait_copies<0>();
#pragma unroll
        for (int s = 0; s < NS - NARROW; ++s)
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const typename TR::Row qr = rd.row(smem, 0, g, s);
#pragma unroll
                for (int x = 0; x < XG; ++x) st[x][g] = mma_rows(qr, kf[x][s], st[x][g]);
            }
        wait_reads();
        // the scores are taken out of the matrix pipe before the branch: read behind it, the compiler (ROCm 7.2) left out the
        // wait that an MFMA result needs on the path around the copies
#pragma unroll
        for (int x = 0; x < XG; ++x)
#pragma unroll
            for (int g = 0; g < G; ++g) asm volatile("" : "+v"(st[x][g]));
        if (more) {
            next_step(g0 + NW * G);
            fetch_rows();
        }
        Weights<KIND> wp[XG], wd[XG];
        Lse2 l2[G][4];
        float lse_min = lse[0][0];
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                l2[g][i].set(lse[g][i]);
                lse_min = fminf(lse_min, lse[g][i]);
            }
        // a query that saw nothing, or nothing but NaN, takes no part whatever its scores and its v are
        full = full && __builtin_amdgcn_ballot_w64(lse_min == -__builtin_inff()) == 0;
#pragma unroll
        for (int x = 0; x < XG; ++x) {
            const int key = j0 + 16 * x + r16;
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    st[x][g][i] = __builtin_amdgcn_exp2f(scaled(st[x][g][i], p.c_hi, p.c_lo, l2[g][i].hi) - l2[g][i].lo);
                    dp[x][g][i] -= dl[g][i];
                }
            if (!full) {  // (one branch for the block: one per value, and the compiler moves the comparisons in front of it)
#pragma unroll
                for (int g = 0; g < G; ++g)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int q = qb[g] + 4 * h4 + i;
                        const bool on = q < p.n && (!p.causal || q >= key) && lse[g][i] != -__builtin_inff();
                        st[x][g][i] = on ? st[x][g][i] : 0.f;
                        dp[x][g][i] = on ? dp[x][g][i] : 0.f;
                    }
            }
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int i = 0; i < 4; ++i) dp[x][g][i] *= st[x][g][i];
            wp[x].set(st[x]);
            wd[x].set(dp[x]);
        }
        accumulate(dv, rd, smem, kG_, wp);
        if (more) {
            wait_reads();
            ld.load(dO, qb_next, p.n, ldb, p.d, lds + kG_, lane);
        }
        accumulate(dk, rd, smem, 0, wd);
        if (more) {
            wait_reads();
            ld.load(Q, qb_next, p.n, ldb, p.d, lds, lane);
        }
    }
    const float scale = p.scale;
    const bool bad_v = combine_store<KIND, QUAD, DP, XG, NW, NARROW>(dv, reinterpret_cast<float*>(smem), w, lane,
                                                         const_cast<char*>(head_base<T>(p.dV, base)), ldb, j0, p.n, p.d, [&](int, int) { return 1.f; });
    const bool bad_k = combine_store<KIND, QUAD, DP, XG, NW, NARROW>(dk, reinterpret_cast<float*>(smem), w, lane,
                                                         const_cast<char*>(head_base<T>(p.dK, base)), ldb, j0, p.n, p.d, [&](int, int) { return scale; });
    redo_rows<XG, NW>(bad_v || bad_k, w, j0, p.n, [&](const GenericParams& p, int j) {
        float* rows = reinterpret_cast<float*>(smem) + w * 2 * DP;
        row_dkdv<T, row_words<T>(DP), kCanOwnDelta<DP>>(p, bh, j, lane, rows, rows + DP);
    });
}

// One launch for dQ, dK and dV: query blocks and key blocks side by side.
template <int KIND, bool QUAD, int DP, int XG, int NW, bool NARROW, bool OWN>
__global__ void __launch_bounds__(NW * 64, NW == 8 || DP <= 96 ? 2 : 1) stream_bwd_kernel(GenericParams p) {
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    const int blocks = (p.n + 16 * XG - 1) / (16 * XG);
    int bh, blk, role;
    balanced_block(blockIdx.x, blocks, p.batch * p.heads, 2, p.causal, bh, blk, role);
    if (role) stream_dkdv<KIND, QUAD, DP, XG, NW, NARROW, OWN>(p, smem, bh, blk);
    else stream_dq<KIND, QUAD, DP, XG, NW, NARROW, OWN>(p, smem, bh, p.causal ? blocks - 1 - blk : blk);
}

// v = rowsum(dO o O), 16 rows per wave, in front of a backward whose key owners read it (own_rows): the sums of stream_dkdv in the
// same order, so the same bits.  Reads O and dO once; a launch of its own costs 2 to 3 us.
template <int KIND, bool QUAD, int DP>
__global__ void __launch_bounds__(kThreads) stream_rows_kernel(GenericParams p) {
    typedef Traits<KIND> TR;
    typedef typename TR::T T;
    constexpr int NS = DP / TR::kChunk;
    const int lane = threadIdx.x & 63, r16 = lane & 15, h4 = lane >> 4;
    const unsigned rows = (unsigned)p.batch * p.heads * p.n, row = (blockIdx.x * (kThreads / 64) + threadIdx.x / 64) * 16 + r16;
    const unsigned in = min(row, rows - 1), bh = in / p.n;  // rows past the end repeat the last one
    const long first = (long)(bh / p.heads) * p.stride_b + (long)(bh % p.heads) * p.stride_h + (long)(in % p.n) * p.stride_n;
    typename TR::Row of[NS], gf[NS];
    load_owned<KIND, QUAD, DP>(head_base<T>(p.O_in, first), h4, p.d, of);
    load_owned<KIND, QUAD, DP>(head_base<T>(p.dO, first), h4, p.d, gf);
    float v = 0.f;
    if constexpr (KIND == kF32) {
#pragma unroll
        for (int s = 0; s < NS; ++s) v = dot_pair(of[s], gf[s], v);
        v += __shfl_xor(v, 16, 64);
        v += __shfl_xor(v, 32, 64);
    } else {
        f32x4 diag = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < NS; ++s) diag = mma_rows(of[s], gf[s], diag);
        v = (r16 & 2) ? ((r16 & 1) ? diag[3] : diag[2]) : ((r16 & 1) ? diag[1] : diag[0]);
    }
    if (row < rows && h4 == (KIND == kF32 ? 0 : r16 >> 2)) p.delta[row] = v;
}

template <int KIND, bool QUAD, int DP, int NW, bool BACKWARD, bool NARROW, bool OWN>
hipError_t launch_waves(const GenericParams& p, dim3 grid, hipStream_t stream) {
    constexpr int XG = kOwned<KIND, DP>;
    constexpr int stages = NW * stage_lds<KIND, QUAD, DP, OWN>(BACKWARD), red = NW * 16 * XG * (DP + 4) * (int)sizeof(float);
    constexpr int lds = stages > red ? stages : red;
    auto kernel = [] {
        if constexpr (BACKWARD) return stream_bwd_kernel<KIND, QUAD, DP, XG, NW, NARROW, OWN>;
        else return stream_fwd_kernel<KIND, QUAD, DP, XG, NW, NARROW>;
    }();
    if constexpr (lds > 60 * 1024) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e != hipSuccess) return e;
    }
    if constexpr (BACKWARD && !OWN) {
        const long rows = (long)p.batch * p.heads * p.n;  // (below 2^28: stream_takes)
        hipLaunchKernelGGL((stream_rows_kernel<KIND, QUAD, DP>), dim3((unsigned)((rows + kThreads / 4 - 1) / (kThreads / 4))), dim3(kThreads), 0, stream, p);
    }
    hipLaunchKernelGGL(kernel, grid, dim3(NW * 64), lds, stream, p);
    return hipGetLastError();
}

// Whether the key owners form the row sums themselves or read those of stream_rows_kernel.  Read, a step copies two tensors instead of
// three and a third of its LDS reads go; in fp32 a third or a fourth workgroup fits a CU's LDS as well (beyond d = 96: eight waves instead of four), in
// bf16 the registers hold the number at two.  The price is the launch in front, 2 to 3 us with the host's share.  So the line is one of work, pairs times
// padded columns, and narrow fp32 heads with at most one workgroup per CU gain nothing.  The sums have the same bits either way, so a masked call, whose
// lists the host does not know, keeps its one launch; but not where the wave count goes with it: fp32 beyond d = 96 goes by the pairs of the call without a
// mask, whose bits it has to have.  us of the backward, one launch -> two:
//   fp32  d32 h32 n1100 201 -> 185   d64 h8 n1100 causal 62 -> 52   d77 h6 n700 82 -> 66   d80 h12 n777 causal 60.8 -> 58   d80 h9 n900 causal 60.5 -> 59.4
//         of 2e8 to 3.2e8 causal, 31 calls: 1.02 to 1.19 times as fast (d40 h6 n1100 42.6 -> 41.3, d96 h20 n500 59 -> 53); full, 27 calls: 1.0 to 1.22, but with
//         3850 to 4030 rows, two full rounds of eight waves either way, 0.96 to 0.99 (d77 h6 n672 54.5 -> 56.8)
//         d128 h16 n1024 429 -> 308, h13 n300 46 -> 41   (below the lines) d64 h3 n900 causal 24.3 -> 27.7, d128 h8 n390 causal 31.3 -> 30.7
//         masked, share of the other blocks kept: d128 h16 n1024 0.05 93 -> 66, 0.3 205 -> 146, h4 n1024 0.3 68 -> 56, 0.15 55 -> 50, the diagonal alone 26.5 -> 29.0
//   bf16  d56 h8 n1100 49 -> 44   d96 h8 n1100 60 -> 53, h2 n1300 23.9 -> 23.6   d120 h8 n1100 110 -> 91   d192 h8 n1100 168 -> 125
//         of 3e8 to 4.3e8 up to d = 96, 29 calls: 0.99 to 1.1, but d96 b2 h15 n475 causal 27.6 -> 28.9
//         (below) d96 h20 n512 causal 21.9 -> 22.4   d120 h13 n300 causal 18.7 -> 18.9   d160 h5 n512 causal 17.6 -> 18.1
inline bool own_rows(bool f32, int width, const GenericParams& p) {
    const double rows = (double)p.batch * p.heads * p.n, work = rows * p.n * width * (p.causal ? 0.5 : 1.0);
    if (f32 && width > 96) return work < 1e8;
    if (p.csr_ptr) return true;
    if (f32) return work < 2e8 || rows <= 16 * 128;  // (128 blocks of 16 queries and as many of keys)
    return work < (width > 96 ? 2e8 : 3e8);
}

// A wave's step is a chain of copies, LDS reads, products and exponentials, so two waves per SIMD are wanted and short
// chains: eight waves per workgroup while there are at most two workgroups per CU, four beyond, where two or more
// workgroups on a CU fill each other's prologue and final sum.  Time with eight over time with four, 324 shapes of n = 200 to
// 2000, 2 to 64 heads, d = 32 to 192, both types, causal and full: up to 256 workgroups 0.69 to 1.0, 257 to 512 0.81 to 1.38 (either
// can win, by how full the second round is), 513 to 768 0.96 to 1.59, beyond 0.96 to 1.96.  Two and three stages per wave hid
// no more than one.
template <int KIND, bool QUAD, int DP, bool BACKWARD, bool NARROW, bool OWN>
hipError_t run_waves(const GenericParams& p, hipStream_t stream) {
    constexpr int rows = 16 * kOwned<KIND, DP>;
    const dim3 grid((unsigned)((p.n + rows - 1) / rows * p.batch * p.heads * (BACKWARD ? 2 : 1)));
    if constexpr (eight_waves<KIND, QUAD, DP, OWN>(BACKWARD))
        if (grid.x <= 512) return launch_waves<KIND, QUAD, DP, 8, BACKWARD, NARROW, OWN>(p, grid, stream);
    return launch_waves<KIND, QUAD, DP, 4, BACKWARD, NARROW, OWN>(p, grid, stream);
}
template <int KIND, bool QUAD, int DP, bool NARROW>
hipError_t run_direction(const GenericParams& p, bool backward, hipStream_t stream) {
    if (!backward) return run_waves<KIND, QUAD, DP, false, NARROW, false>(p, stream);
    if constexpr (kCanOwnDelta<DP>)
        if (own_rows(KIND == kF32, DP, p)) return run_waves<KIND, QUAD, DP, true, NARROW, true>(p, stream);
    return run_waves<KIND, QUAD, DP, true, NARROW, false>(p, stream);
}
template <int KIND, bool QUAD, int DP>
hipError_t run_stream(const GenericParams& p, bool backward, hipStream_t stream) {
    if constexpr (KIND == kF32 && DP % 64 != 0)
        if (p.d <= DP - 16) return run_direction<KIND, QUAD, DP, true>(p, backward, stream);
    return run_direction<KIND, QUAD, DP, false>(p, backward, stream);
}

template <int KIND, bool QUAD>
hipError_t run_width(const GenericParams& p, bool backward, hipStream_t stream) {
    switch ((p.d + 31) / 32) {  // the next multiple of 32: the loads bound columns in the last 32 only
        case 1: return run_stream<KIND, QUAD, 32>(p, backward, stream);
        case 2: return run_stream<KIND, QUAD, 64>(p, backward, stream);
        case 3: return run_stream<KIND, QUAD, 96>(p, backward, stream);
        case 4: return run_stream<KIND, QUAD, 128>(p, backward, stream);
        default: break;
    }
    if constexpr (KIND != kF32) {
        switch ((p.d + 31) / 32) {
            case 5: return run_stream<KIND, QUAD, 160>(p, backward, stream);
            case 6: return run_stream<KIND, QUAD, 192>(p, backward, stream);
            case 7: return run_stream<KIND, QUAD, 224>(p, backward, stream);
            case 8: return run_stream<KIND, QUAD, 256>(p, backward, stream);
            default: break;
        }
    }
    return hipErrorInvalidValue;
}

}  // namespace

// Sequences of a few rows in many heads: a block of 16 or 32 rows costs what it costs with one row in it, and there is one
// for every head; a row per wave costs by the row.  The line lies where the blocks are more than the CUs hold at a time, and at
// the rows below which the row kernels win, measured over 64 to 32768 heads.  us, forward / backward, matrix cores -> rows:
//   fp32 d16    n1 h32768 57 / 180 -> 22 / 47     n2 h4096 11 / 26 -> 11 / 21     n3 h32768 (beyond the line) 58 / 184 -> 65 / 123
//   fp32 d64    n2 h4096 17 / 50 -> 12 / 28       n5 h4096 (beyond) 18 / 54 -> 31 / 71     n1 h512 (beyond) 11 / 14 -> 11 / 19
//   fp32 d128   n1 h4096 37 / 216 -> 12 / 28      n6 h4096 backward 218 -> 133, forward (beyond) 39 -> 66
//   bf16 d32    n2 h32768 91 / 372 -> 42 / 88     n4 h32768 92 / 375 -> 86 / 191   n8 h4096 (beyond) 15 / 46 -> 25 / 49
//   bf16 d192   n6 h4096 80 / 246 -> 50 / 111     n8 h32768 (beyond) 643 / 2028 -> 722 / 1653
static bool few_rows(bool is_bf16, bool backward, const GenericParams& p) {
    const int rows = is_bf16 ? (p.d > 128 || (backward && p.d > 64) ? 6 : 4) : (backward && p.d > 96 ? 6 : 2);
    const long width = (p.d + 31) / 32 * 32;
    return p.n <= rows && (long)p.batch * p.heads * width >= (is_bf16 ? 65536 : 98304);
}

// What is left to the FMA kernels: head dimensions whose accumulators, owned rows and stages do not fit a CU here,
// block edges that cut through the rows a workgroup owns, heads of 4 GB and more (32-bit byte offsets), few rows in many
// heads, and more blocks than a launch of 2^32 threads has.
bool stream_takes(bool is_bf16, bool backward, const GenericParams& p) {
    if (p.d > (is_bf16 ? 256 : 128)) return false;
    const int owned = is_bf16 && p.d <= 128 ? 32 : 16;
    if (p.csr_ptr && p.block % owned != 0) return false;
    if (few_rows(is_bf16, backward, p)) return false;
    if ((double)p.batch * p.heads * (((long)p.n + owned - 1) / owned) * (backward ? 2 : 1) * 256.0 >= 4294967296.0) return false;
    return (double)p.n * (double)p.stride_n * (is_bf16 ? 2.0 : 4.0) < 4.0e9;
}

hipError_t launch_stream(bool is_bf16, bool backward, const GenericParams& p, hipStream_t stream) {
    if (is_bf16) return run_width<kBf3, true>(p, backward, stream);
    // fp32 tensors may start on any 4 bytes: 16-byte copies only where every row does start on 16 (bf16 calls are checked
    // for that where they enter)
    uintptr_t all = 0;
    for (const void* t : {p.Q, p.K, p.V, (const void*)p.O, p.O_in, p.dO, (const void*)p.dQ, (const void*)p.dK, (const void*)p.dV})
        all |= reinterpret_cast<uintptr_t>(t);
    const bool quad = (all & 15) == 0 && (p.d | p.stride_n | p.stride_h | p.stride_b) % 4 == 0;
    return quad ? run_width<kF32, true>(p, backward, stream) : run_width<kF32, false>(p, backward, stream);
}

}  // namespace attn
