// Attention row by row in fp32 multiply-adds: one wavefront owns one row; lanes split the other sequence for the score-like
// quantities and the columns for the outputs.  The FMA kernels run on it, and the matrix-core kernels of the same
// arithmetic redo rows with it whose result is not finite.
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

template <typename T>
__device__ __forceinline__ float dot_row(const float* a_lds, const T* b, int d) {
    float s = 0.f;
    for (int k = 0; k < d; ++k) s = fmaf(a_lds[k], ldf(b + k), s);
    return s;
}

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

// COLS: output columns per lane, d <= 64 COLS.  qs, gs, ks, vs: d floats of LDS of this wave.
// O_i and LSE_i
template <typename T, int COLS>
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
    float acc[COLS];
#pragma unroll
    for (int u = 0; u < COLS; ++u) acc[u] = 0.f;
    float l = 0.f;
    if (m != -__builtin_inff()) {
        for (int a = 0; a < nr; ++a) {
            int lo, hi;
            rg.get(i, a, true, lo, hi);
            for (int j0 = lo; j0 < hi; j0 += 64) {
                const int j = j0 + lane;
                float e = 0.f;
                if (j < hi) e = expf(p.scale * dot_row(qs, K + (long)j * p.stride_n, p.d) - m);
                l += e;
                const int cnt = min(64, hi - j0);
                for (int jj = 0; jj < cnt; ++jj) {
                    const float ej = __shfl(e, jj, 64);
#pragma unroll
                    for (int u = 0; u < COLS; ++u) {
                        const int k = lane + 64 * u;
                        if (k < p.d) acc[u] = fmaf(ej, ldf(V + (long)(j0 + jj) * p.stride_n + k), acc[u]);
                    }
                }
            }
        }
        l = wave_sum(l);
    }
    const float inv = l > 0.f ? 1.f / l : 0.f;
#pragma unroll
    for (int u = 0; u < COLS; ++u) {
        const int k = lane + 64 * u;
        if (k < p.d) stf(O + (long)i * p.stride_n + k, acc[u] * inv);
    }
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
template <typename T, int COLS>
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
    float acc[COLS];
#pragma unroll
    for (int u = 0; u < COLS; ++u) acc[u] = 0.f;
    if (lse != -__builtin_inff()) {
        for (int a = 0; a < nr; ++a) {
            int lo, hi;
            rg.get(i, a, true, lo, hi);
            for (int j0 = lo; j0 < hi; j0 += 64) {
                const int j = j0 + lane;
                float pp = 0.f;
                if (j < hi) {
                    const float f = expf(p.scale * dot_row(qs, K + (long)j * p.stride_n, p.d) - lse);
                    pp = f * (dot_row(gs, V + (long)j * p.stride_n, p.d) - v);
                }
                const int cnt = min(64, hi - j0);
                for (int jj = 0; jj < cnt; ++jj) {
                    const float pj = __shfl(pp, jj, 64);
#pragma unroll
                    for (int u = 0; u < COLS; ++u) {
                        const int k = lane + 64 * u;
                        if (k < p.d) acc[u] = fmaf(pj, ldf(K + (long)(j0 + jj) * p.stride_n + k), acc[u]);
                    }
                }
            }
        }
    }
#pragma unroll
    for (int u = 0; u < COLS; ++u) {
        const int k = lane + 64 * u;
        if (k < p.d) stf((T*)p.dQ + base + (long)i * p.stride_n + k, acc[u] * p.scale);
    }
}

// dK_j = scale sum_i p_ij Q_i, dV_j = sum_i f_ij dO_i; delta(i): v_i, asked for by the lane that needs it
template <typename T, int COLS, typename F>
__device__ __forceinline__ void row_dkdv(const GenericParams& p, int bh, int j, int lane, F delta, float* ks, float* vs) {
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
    float ak[COLS], av[COLS];
#pragma unroll
    for (int u = 0; u < COLS; ++u) { ak[u] = 0.f; av[u] = 0.f; }
    for (int a = 0; a < nr; ++a) {
        int lo, hi;
        rg.get(j, a, false, lo, hi);
        // chunks start on multiples of 64 so that dense and block-list runs sum in the same order
        for (int i0 = lo & ~63; i0 < hi; i0 += 64) {
            const int i = i0 + lane;
            float f = 0.f, pp = 0.f;
            if (i >= lo && i < hi && lse[i] != -__builtin_inff()) {
                f = expf(p.scale * dot_row(ks, Q + (long)i * p.stride_n, p.d) - lse[i]);
                pp = f * (dot_row(vs, G + (long)i * p.stride_n, p.d) - delta(i));
            }
            const int cnt = min(64, hi - i0);
            for (int ii = 0; ii < cnt; ++ii) {
                const float fi = __shfl(f, ii, 64), pi = __shfl(pp, ii, 64);
#pragma unroll
                for (int u = 0; u < COLS; ++u) {
                    const int k = lane + 64 * u;
                    if (k < p.d) {
                        av[u] = fmaf(fi, ldf(G + (long)(i0 + ii) * p.stride_n + k), av[u]);
                        ak[u] = fmaf(pi, ldf(Q + (long)(i0 + ii) * p.stride_n + k), ak[u]);
                    }
                }
            }
        }
    }
#pragma unroll
    for (int u = 0; u < COLS; ++u) {
        const int k = lane + 64 * u;
        if (k < p.d) {
            stf((T*)p.dK + base + (long)j * p.stride_n + k, ak[u] * p.scale);
            stf((T*)p.dV + base + (long)j * p.stride_n + k, av[u]);
        }
    }
}

}  // namespace attn
