// Attention row by row in fp32 multiply-adds: one wavefront owns one row; lanes split the other sequence for the score-like
// quantities and the columns for the outputs.  The FMA kernels run on it, and the matrix-core kernels of the same
// arithmetic redo rows with it whose result is not finite.
//
// us, forward / backward, with 4- or 2-byte loads and one row in flight at a time -> 16-byte loads in the sums over columns and
// several rows in flight in those over rows: fp32 b1 h4 n300 d200 causal 455 / 937 -> 75 / 190, bf16 b1 h4 n512 d512 with 40 % of
// 64-blocks 1457 / 3364 -> 174 / 430.  As redone rows of the matrix-core kernels (which have fewer waves for them): bf16 b1 h8
// n512 d192 with one infinite key element per head 2170 / 4936 -> 318 / 613, all NaN 686 / 1564 -> 108 / 103 (the row kernels
// alone, as they were: 1519 / 2427 and 667 / 311).
#pragma once
#include "attn_common.hpp"
#include "attn_internal.hpp"

namespace attn {

template <typename T> __device__ __forceinline__ float ldf(const T* p) { return (float)*p; }
template <typename T> __device__ __forceinline__ void stf(T* p, float v) { *p = (T)v; }

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, 64);
    return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) v = fmaxf(v, __shfl_xor(v, m, 64));
    return v;
}

// 16 bytes of a row.  fp32 rows start on any 4 bytes; bf16 rows start on 16 and are whole pieces (the host checks both).
template <typename T> struct Piece;
template <> struct Piece<float> { typedef float V __attribute__((ext_vector_type(4), aligned(4))); };
template <> struct Piece<__bf16> { typedef bf16x8 V; };

// Sums over a row of d, in the order of its columns.  A lane reads a row of its own, so every load instruction is 64 L1
// accesses whatever its width, and these bound the row functions: 16 bytes at a time.
//   dot_row    a . b,  a in LDS
//   dot_rows2  a . b and c . b, the row b read once
template <typename T>
__device__ __forceinline__ float dot_row(const float* a_lds, const T* b, int d) {
    constexpr int P = 16 / (int)sizeof(T);
    float s = 0.f;
    int k = 0;
#pragma unroll 1
    for (; k + P <= d; k += P) {
        const typename Piece<T>::V v = *reinterpret_cast<const typename Piece<T>::V*>(b + k);
#pragma unroll
        for (int e = 0; e < P; ++e) s = fmaf(a_lds[k + e], (float)v[e], s);
    }
    for (; k < d; ++k) s = fmaf(a_lds[k], ldf(b + k), s);
    return s;
}
template <typename T>
__device__ __forceinline__ void dot_rows2(const float* a_lds, const T* c, const T* b, int d, float& ab, float& cb) {
    constexpr int P = 16 / (int)sizeof(T);
    ab = cb = 0.f;
    int k = 0;
#pragma unroll 1
    for (; k + P <= d; k += P) {
        const typename Piece<T>::V v = *reinterpret_cast<const typename Piece<T>::V*>(b + k);
        const typename Piece<T>::V u = *reinterpret_cast<const typename Piece<T>::V*>(c + k);
#pragma unroll
        for (int e = 0; e < P; ++e) {
            ab = fmaf(a_lds[k + e], (float)v[e], ab);
            cb = fmaf((float)u[e], (float)v[e], cb);
        }
    }
    for (; k < d; ++k) {
        ab = fmaf(a_lds[k], ldf(b + k), ab);
        cb = fmaf(ldf(c + k), ldf(b + k), cb);
    }
}

// N weighted sums over the same rows j, in order:  acc[s][column] += sum_j weight[s] of lane j * row[s]_j[column].  A lane has
// the columns of the 4-byte words lane + 64 u of a row (fp32: one column each, bf16: two), u < WORDS.  Several rows are
// requested at a time: one by one, each waits out a load (300 cycles and more, and a redone row has its SIMD nearly to itself).
// Words past the row's end read its last one and are not stored.
template <typename T, int WORDS, int N>
struct WeightedRows {
    static constexpr int kPer = 4 / (int)sizeof(T), kRows = WORDS <= 2 ? 8 / N : WORDS <= 4 ? 4 : 2;
    float acc[N][WORDS][kPer];
    unsigned word[WORDS];
    __device__ __forceinline__ WeightedRows(int lane, int d) {
#pragma unroll
        for (int u = 0; u < WORDS; ++u) word[u] = (unsigned)min(lane + 64 * u, d / kPer - 1);
#pragma unroll
        for (int s = 0; s < N; ++s)
#pragma unroll
            for (int u = 0; u < WORDS; ++u)
#pragma unroll
                for (int e = 0; e < kPer; ++e) acc[s][u][e] = 0.f;
    }
    template <int R>
    __device__ __forceinline__ void some(const float (&weight)[N], const T* const (&row)[N], long ld, int j) {
        // the address of a row is the same for all lanes: kept in scalar registers, with one vector register per word
        typedef const uint32_t __attribute__((address_space(1))) * global_ptr;
        uint32_t v[N][R][WORDS];
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int s = 0; s < N; ++s) {
                const unsigned long long a = reinterpret_cast<unsigned long long>(row[s] + (j + r) * ld);
                const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)a), hi = __builtin_amdgcn_readfirstlane((unsigned)(a >> 32));
                const global_ptr first = (global_ptr)(((unsigned long long)hi << 32) | lo);
#pragma unroll
                for (int u = 0; u < WORDS; ++u) v[s][r][u] = first[word[u]];
            }
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int s = 0; s < N; ++s) {
                const float w = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, weight[s]), j + r));
#pragma unroll
                for (int u = 0; u < WORDS; ++u) {
                    if constexpr (kPer == 1) {
                        acc[s][u][0] = fmaf(w, __builtin_bit_cast(float, v[s][r][u]), acc[s][u][0]);
                    } else {
                        acc[s][u][0] = fmaf(w, __builtin_bit_cast(float, v[s][r][u] << 16), acc[s][u][0]);
                        acc[s][u][1] = fmaf(w, __builtin_bit_cast(float, v[s][r][u] & 0xffff0000u), acc[s][u][1]);
                    }
                }
            }
    }
    // rows first .. last - 1 of a chunk of 64 at row[s]; false when every sum is NaN, which no further row changes
    __device__ __forceinline__ bool add(const float (&weight)[N], const T* const (&row)[N], long ld, int first, int last) {
        int j = first;
#pragma unroll 1
        for (; j + kRows <= last; j += kRows) some<kRows>(weight, row, ld, j);
#pragma unroll 1
        for (; j < last; ++j) some<1>(weight, row, ld, j);
        bool number = false;
#pragma unroll
        for (int s = 0; s < N; ++s)
#pragma unroll
            for (int u = 0; u < WORDS; ++u)
#pragma unroll
                for (int e = 0; e < kPer; ++e) number = number || acc[s][u][e] == acc[s][u][e];
        return __builtin_amdgcn_ballot_w64(number) != 0;
    }
    __device__ __forceinline__ void store(int s, T* row, int lane, int d, float factor) const {
#pragma unroll
        for (int u = 0; u < WORDS; ++u) {
            const int k = (lane + 64 * u) * kPer;
            if (k < d) {
#pragma unroll
                for (int e = 0; e < kPer; ++e) stf(row + k + e, acc[s][u][e] * factor);
            }
        }
    }
};
// words per lane for rows of up to d columns
template <typename T>
__host__ __device__ constexpr int row_words(int d) { return (d * (int)sizeof(T) + 255) / 256; }

// Visible range of the other index for row r: ranges are whole blocks of the list (or one
// range 0..n when dense), clipped by the causal rule.  `row_is_query` picks the rule's side.
struct Ranges {
    const int32_t *ptr, *idx;
    int block, n, causal;
    __device__ __forceinline__ int count(int r) const { return ptr ? ptr[r / block + 1] - ptr[r / block] : 1; }
    __device__ __forceinline__ void get(int r, int a, bool row_is_query, int& lo, int& hi) const {
        lo = 0;
        hi = n;
        if (ptr) {
            const int b = idx[ptr[r / block] + a];
            lo = b * block;
            hi = min(n, lo + block);
        }
        if (causal) {
            if (row_is_query) hi = min(hi, r + 1);  // keys j <= i
            else lo = max(lo, r);                   // queries i >= j
        }
    }
};

// What this wave wrote to LDS can be read by all its lanes.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// WORDS: 4-byte words of a row per lane, row_words(d) or more.  qs, gs, ks, vs: d floats of LDS of this wave.
// O_i and LSE_i
template <typename T, int WORDS>
__device__ __forceinline__ void row_forward(const GenericParams& p, int bh, int i, int lane, float* qs) {
    const long base = (long)(bh / p.heads) * p.stride_b + (long)(bh % p.heads) * p.stride_h;
    const T *Q = (const T*)p.Q + base, *K = (const T*)p.K + base, *V = (const T*)p.V + base;
    T* O = (T*)p.O + base;
    for (int k = lane; k < p.d; k += 64) qs[k] = ldf(Q + (long)i * p.stride_n + k);
    wave_sync();
    const Ranges rg{p.csr_ptr ? p.csr_ptr + (long)bh * p.mask_stride : nullptr, p.csr_idx, p.block, p.n, p.causal};
    const int nr = rg.count(i);
    float m = -__builtin_inff();
    for (int a = 0; a < nr; ++a) {
        int lo, hi;
        rg.get(i, a, true, lo, hi);
        for (int j = lo + lane; j < hi; j += 64) m = fmaxf(m, p.scale * dot_row(qs, K + (long)j * p.stride_n, p.d));
    }
    m = wave_max(m);
    WeightedRows<T, WORDS, 1> sum(lane, p.d);
    float l = 0.f;
    bool more = true;
    if (m != -__builtin_inff()) {
        for (int a = 0; a < nr && more; ++a) {
            int lo, hi;
            rg.get(i, a, true, lo, hi);
            for (int j0 = lo; j0 < hi && more; j0 += 64) {
                const int j = j0 + lane;
                float e = 0.f;
                if (j < hi) e = expf(p.scale * dot_row(qs, K + (long)j * p.stride_n, p.d) - m);
                l += e;
                more = sum.add({e}, {V + (long)j0 * p.stride_n}, p.stride_n, 0, min(64, hi - j0)) || __builtin_amdgcn_ballot_w64(l != l) == 0;
            }
        }
        l = wave_sum(l);
    }
    const float inv = l > 0.f ? 1.f / l : 0.f;
    sum.store(0, O + (long)i * p.stride_n, lane, p.d, inv);
    if (lane == 0) p.LSE_out[(long)bh * p.n + i] = l > 0.f ? m + logf(l) : -__builtin_inff();
}

// v_i = dO_i . O_i
template <typename T>
__device__ __forceinline__ float row_delta(const GenericParams& p, int bh, int i, int lane) {
    const long off = (long)(bh / p.heads) * p.stride_b + (long)(bh % p.heads) * p.stride_h + (long)i * p.stride_n;
    float s = 0.f;
    for (int k = lane; k < p.d; k += 64) s = fmaf(ldf((const T*)p.O_in + off + k), ldf((const T*)p.dO + off + k), s);
    return wave_sum(s);
}

// dQ_i = scale sum_j p_ij K_j
template <typename T, int WORDS>
__device__ __forceinline__ void row_dq(const GenericParams& p, int bh, int i, int lane, float v, float* qs, float* gs) {
    const long base = (long)(bh / p.heads) * p.stride_b + (long)(bh % p.heads) * p.stride_h;
    const T *Q = (const T*)p.Q + base, *K = (const T*)p.K + base, *V = (const T*)p.V + base, *G = (const T*)p.dO + base;
    for (int k = lane; k < p.d; k += 64) {
        qs[k] = ldf(Q + (long)i * p.stride_n + k);
        gs[k] = ldf(G + (long)i * p.stride_n + k);
    }
    wave_sync();
    const float lse = p.LSE_in[(long)bh * p.n + i];
    const Ranges rg{p.csr_ptr ? p.csr_ptr + (long)bh * p.mask_stride : nullptr, p.csr_idx, p.block, p.n, p.causal};
    const int nr = rg.count(i);
    WeightedRows<T, WORDS, 1> sum(lane, p.d);
    bool more = true;
    if (lse != -__builtin_inff()) {
        for (int a = 0; a < nr && more; ++a) {
            int lo, hi;
            rg.get(i, a, true, lo, hi);
            for (int j0 = lo; j0 < hi && more; j0 += 64) {
                const int j = j0 + lane;
                float pp = 0.f;
                if (j < hi) {
                    const float f = expf(p.scale * dot_row(qs, K + (long)j * p.stride_n, p.d) - lse);
                    pp = f * (dot_row(gs, V + (long)j * p.stride_n, p.d) - v);
                }
                more = sum.add({pp}, {K + (long)j0 * p.stride_n}, p.stride_n, 0, min(64, hi - j0));
            }
        }
    }
    sum.store(0, (T*)p.dQ + base + (long)i * p.stride_n, lane, p.d, p.scale);
}

// dK_j = scale sum_i p_ij Q_i, dV_j = sum_i f_ij dO_i; OWN_V: v_i is formed here, else read from p.delta
template <typename T, int WORDS, bool OWN_V>
__device__ __forceinline__ void row_dkdv(const GenericParams& p, int bh, int j, int lane, float* ks, float* vs) {
    const long base = (long)(bh / p.heads) * p.stride_b + (long)(bh % p.heads) * p.stride_h;
    const T *Q = (const T*)p.Q + base, *K = (const T*)p.K + base, *V = (const T*)p.V + base, *G = (const T*)p.dO + base;
    const float* lse = p.LSE_in + (long)bh * p.n;
    for (int k = lane; k < p.d; k += 64) {
        ks[k] = ldf(K + (long)j * p.stride_n + k);
        vs[k] = ldf(V + (long)j * p.stride_n + k);
    }
    wave_sync();
    const Ranges rg{p.csc_ptr ? p.csc_ptr + (long)bh * p.mask_stride : nullptr, p.csc_idx, p.block, p.n, p.causal};
    const int nr = rg.count(j);
    WeightedRows<T, WORDS, 2> sum(lane, p.d);
    bool more = true;
    for (int a = 0; a < nr && more; ++a) {
        int lo, hi;
        rg.get(j, a, false, lo, hi);
        // chunks start on multiples of 64 so that dense and block-list runs sum in the same order
        for (int i0 = lo & ~63; i0 < hi && more; i0 += 64) {
            const int i = i0 + lane;
            float f = 0.f, pp = 0.f;
            if (i >= lo && i < hi && lse[i] != -__builtin_inff()) {
                f = expf(p.scale * dot_row(ks, Q + (long)i * p.stride_n, p.d) - lse[i]);
                float q, v;
                if constexpr (OWN_V) {
                    dot_rows2(vs, (const T*)p.O_in + base + (long)i * p.stride_n, G + (long)i * p.stride_n, p.d, q, v);
                } else {
                    q = dot_row(vs, G + (long)i * p.stride_n, p.d);
                    v = p.delta[(long)bh * p.n + i];
                }
                pp = f * (q - v);
            }
            more = sum.add({f, pp}, {G + (long)i0 * p.stride_n, Q + (long)i0 * p.stride_n}, p.stride_n, max(0, lo - i0), min(64, hi - i0));
        }
    }
    sum.store(0, (T*)p.dV + base + (long)j * p.stride_n, lane, p.d, 1.f);
    sum.store(1, (T*)p.dK + base + (long)j * p.stride_n, lane, p.d, p.scale);
}

}  // namespace attn
