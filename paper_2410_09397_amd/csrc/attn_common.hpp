// Shared device helpers for the gfx950 attention kernels: vector types, the LDS tile
// layout, MFMA operand fetches and bf16 packing.  HIP device code only.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

namespace attn {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

#define ATTN_LDS __attribute__((address_space(3)))

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr int kThreads = 256;  // four 64-lane wavefronts per workgroup, one per SIMD

// f(std::integral_constant<int, 0>{}), ... , N - 1: for register arrays indexed by what is uniform but not known to the compiler
template <int N, int I = 0, typename F>
__device__ __forceinline__ void static_for(F f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<N, I + 1>(f);
    }
}

// ---------------------------------------------------------------------------------------
// 32x32x16 bf16 MFMA.  Operand layout (lane l, h = l / 32):
//   A (32 x 16): row l % 32, k = 8h .. 8h+7        B (16 x 32): column l % 32, k = 8h .. 8h+7
//   C (32 x 32): column l % 32, register i <-> row 8 (i / 4) + 4h + i % 4
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// Results of matrix products that vector instructions read next, moved to ordinary registers here where the compiler keeps them in accumulator
// registers.  (No wait states: the compiler adds those itself, also behind branches.)
__device__ __forceinline__ void to_vector_registers(f32x16& v) { asm volatile("" : "+v"(v)); }

// Row of accumulator register i for a lane in half h.
__device__ __forceinline__ int acc_row(int i, int h) { return 8 * (i >> 2) + 4 * h + (i & 3); }

// Two fp32 -> packed bf16 pair, round to nearest even (one v_cvt_pk_bf16_f32).
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
    f32x2 v = {lo, hi};
    bf16x2 r = __builtin_convertvector(v, bf16x2);
    return __builtin_bit_cast(uint32_t, r);
}

// Registers 8s .. 8s+7 of an accumulator as one bf16 B operand.  Its k index (h, t) then
// stands for accumulator row 16s + 8 (t / 4) + 4h + t % 4, which load_frag_t() mirrors.
__device__ __forceinline__ bf16x8 acc_to_operand(const f32x16& c, int s) {
    u32x4 r;
    r[0] = pack_bf16(c[8 * s + 0], c[8 * s + 1]);
    r[1] = pack_bf16(c[8 * s + 2], c[8 * s + 3]);
    r[2] = pack_bf16(c[8 * s + 4], c[8 * s + 5]);
    r[3] = pack_bf16(c[8 * s + 6], c[8 * s + 7]);
    return __builtin_bit_cast(bf16x8, r);
}

__device__ __forceinline__ float max3(float a, float b, float c) {
    return __builtin_elementwise_maximum(a, __builtin_elementwise_maximum(b, c));
}

// ---------------------------------------------------------------------------------------
// LDS tile: R rows of D bf16, row-major, no padding, 16-byte chunks XOR-swizzled by row so
// that both fetch patterns below spread over all 64 banks:
//   - row-major fetch: 16 lanes read the same chunk column of 16 consecutive rows,
//   - transposed fetch: 32 lanes read 4 consecutive rows x 4 consecutive chunks.
// ---------------------------------------------------------------------------------------
template <int D>
__device__ __forceinline__ int swz(int row) {
    if constexpr (D >= 128)
        return ((row & 3) << 2) | ((row >> 2) & 3);
    else if constexpr (D == 64)
        return (((row >> 1) & 1) << 2) | ((row >> 2) & 3);
    else  // D == 32: four chunks per row, only the row-major fetch is used
        return (row >> 2) & 3;
}

// Byte offset of 16-byte chunk c (8 elements) of a tile row.
template <int D>
__device__ __forceinline__ int tile_off(int row, int c) {
    return row * (D * 2) + ((c ^ swz<D>(row)) << 4);
}

// A (or B) operand whose k index runs along the tile's contiguous dimension:
// lane l holds row row0 + l % 32, elements 16 ks + 8h .. +7.
template <int D>
__device__ __forceinline__ bf16x8 load_frag(const char* tile, int row0, int ks, int lane) {
    const int row = row0 + (lane & 31);
    return *reinterpret_cast<const bf16x8*>(tile + tile_off<D>(row, 2 * ks + (lane >> 5)));
}

// A operand whose k index runs along the tile's rows (the tile is read transposed):
// lane l holds column col0 + l % 32 and, for t = 0..7, row row16 + 8 (t / 4) + 4h + t % 4.
// Two ds_read_b64_tr_b16: within each group of 16 lanes, lane s supplies the address of
// row + s / 4, columns 4 (s % 4) .. +3, and receives column s of the four rows.
template <int D>
__device__ __forceinline__ bf16x8 load_frag_t(const char* tile, int col0, int row16, int lane) {
    const int s = lane & 15;
    const int row = row16 + 4 * (lane >> 5) + (s >> 2);
    const int col = col0 + 16 * ((lane >> 4) & 1) + 4 * (s & 3);
    const int off0 = tile_off<D>(row, col >> 3) + ((col & 4) << 1);
    const int off1 = tile_off<D>(row + 8, col >> 3) + ((col & 4) << 1);
    i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((i16x4 ATTN_LDS*)(tile + off0));
    i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((i16x4 ATTN_LDS*)(tile + off1));
    typedef short i16x8 __attribute__((ext_vector_type(8)));
    i16x8 r = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, r);
}

// The same two fetches with the lane-dependent part of the address hoisted out of the hot
// loop.  The swizzle is an XOR on the chunk field (bits 4..7 of the byte offset), tiles start on
// 256-byte boundaries and rows that are a multiple of 16 apart share their swizzle term, so
//   offset(ks)  = (tile + rm0) ^ (ks << 5)            + row0 * row_bytes      (load_frag)
//   offset(mt)  = (tile + tr0) ^ (mt << 6) [^ 32 for the rows + 8 half] + ...  (load_frag_t)
// i.e. one per-lane base per tile, one XOR per fetch and a compile-time immediate.
template <int D>
struct FragOffsets {
    int rm0, tr0;
    __device__ __forceinline__ void init(int lane) {
        rm0 = tile_off<D>(lane & 31, lane >> 5);
        const int s = lane & 15;
        const int col = 16 * ((lane >> 4) & 1) + 4 * (s & 3);
        tr0 = tile_off<D>(4 * (lane >> 5) + (s >> 2), col >> 3) + ((col & 4) << 1);
    }
    // tile_off: byte offset of the tile inside `lds` (multiple of 256); rows row0 + l % 32 with
    // row0 a multiple of 16
    __device__ __forceinline__ bf16x8 frag(const char* lds, int tile_off_bytes, int row0, int ks) const {
        const int a = (tile_off_bytes + rm0) ^ (ks << 5);
        return *reinterpret_cast<const bf16x8*>(lds + a + row0 * (D * 2));
    }
    // columns 32 mt + l % 32; rows row16 + 8 (t / 4) + 4h + t % 4 with row16 a multiple of 16
    __device__ __forceinline__ bf16x8 frag_t(const char* lds, int tile_off_bytes, int mt, int row16) const {
        const int a = (tile_off_bytes + tr0) ^ (mt << 6);
        return read_t(lds, a, a ^ 32, row16);
    }
    // Per-fetch address registers for loops whose tile offsets are compile-time constants: with
    //   rm(ks)       = rm0 ^ (ks << 5)              (+ any multiple of 256)
    //   tr(mt, half) = tr0 ^ (mt << 6) ^ (half << 5)
    // kept in registers, a fetch is a register plus an immediate and needs no vector arithmetic.
    __device__ __forceinline__ int rm(int ks) const { return rm0 ^ (ks << 5); }
    __device__ __forceinline__ int tr(int mt, int half) const { return tr0 ^ (mt << 6) ^ (half << 5); }
    static __device__ __forceinline__ bf16x8 read(const char* lds, int rm_ks, int imm) {
        return *reinterpret_cast<const bf16x8*>(lds + rm_ks + imm);
    }
    // imm: tile offset + row16 * row bytes
    static __device__ __forceinline__ bf16x8 read_t(const char* lds, int tr_lo, int tr_hi, int row16, int imm = 0) {
        i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((i16x4 ATTN_LDS*)(lds + tr_lo + (imm + row16 * (D * 2))));
        i16x4 hi =
            __builtin_amdgcn_ds_read_tr16_b64_v4i16((i16x4 ATTN_LDS*)(lds + tr_hi + (imm + (row16 + 8) * (D * 2))));
        typedef short i16x8 __attribute__((ext_vector_type(8)));
        i16x8 r = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        return __builtin_bit_cast(bf16x8, r);
    }
    // The transposed fetch with the k index in natural order: element t of lane half h <-> row row16 + 8h + t, which
    // pairs with an operand that is read row-major as whole 16-byte chunks.  tr_natural(lane, mt, half) is the
    // address register (half 1 = rows + 4: one step of the row swizzle, 16 bytes), read_t_natural the fetch.
    static __device__ __forceinline__ int tr_natural(int lane, int mt, int half) {
        const int s = lane & 15;
        const int col = 16 * ((lane >> 4) & 1) + 4 * (s & 3);
        const int base = tile_off<D>(8 * (lane >> 5) + (s >> 2), col >> 3) + ((col & 4) << 1);
        return base ^ (mt << 6) ^ (half << 4);
    }
    static __device__ __forceinline__ bf16x8 read_t_natural(const char* lds, int tr_lo, int tr_hi, int row16, int imm = 0) {
        i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((i16x4 ATTN_LDS*)(lds + tr_lo + (imm + row16 * (D * 2))));
        i16x4 hi =
            __builtin_amdgcn_ds_read_tr16_b64_v4i16((i16x4 ATTN_LDS*)(lds + tr_hi + (imm + (row16 + 4) * (D * 2))));
        typedef short i16x8 __attribute__((ext_vector_type(8)));
        i16x8 r = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        return __builtin_bit_cast(bf16x8, r);
    }
};

// The address registers of all fragments of a [rows x D] tile (static indices only).  The swizzle stays within 16 chunks
// (256 bytes), so fragments 256 bytes apart share a register.
template <int D>
struct FragAddrs {
    static constexpr int kRm = D / 16 < 8 ? D / 16 : 8, kTr = D / 32 < 4 ? D / 32 : 4;
    int rmk[kRm];
    int trk[kTr][2];
    __device__ __forceinline__ void init(const FragOffsets<D>& fo) {
#pragma unroll
        for (int ks = 0; ks < kRm; ++ks) rmk[ks] = fo.rm(ks);
#pragma unroll
        for (int mt = 0; mt < kTr; ++mt) {
            trk[mt][0] = fo.tr(mt, 0);
            trk[mt][1] = fo.tr(mt, 1);
        }
    }
    // all fetches `rows` (a multiple of 16) further down the tile
    __device__ __forceinline__ void shift_rows(int rows) {
#pragma unroll
        for (int ks = 0; ks < kRm; ++ks) rmk[ks] += rows * (D * 2);
        shift_transposed(rows * (D * 2));
    }
    // the transposed fetches `bytes` (a multiple of 256) further on
    __device__ __forceinline__ void shift_transposed(int bytes) {
#pragma unroll
        for (int mt = 0; mt < kTr; ++mt) {
            trk[mt][0] += bytes;
            trk[mt][1] += bytes;
        }
    }
    __device__ __forceinline__ bf16x8 frag(const char* lds, int tile_off_bytes, int row0, int ks) const {
        return FragOffsets<D>::read(lds, rmk[ks % kRm], tile_off_bytes + row0 * (D * 2) + 256 * (ks / kRm));
    }
    __device__ __forceinline__ bf16x8 frag_t(const char* lds, int tile_off_bytes, int mt, int row16) const {
        return FragOffsets<D>::read_t(lds, trk[mt % kTr][0], trk[mt % kTr][1], row16, tile_off_bytes + 256 * (mt / kTr));
    }
};

// Operand whose k index runs along the tile's contiguous dimension, but with the k order of
// load_frag_t (element t of half h <-> column 16 ks + 8 (t / 4) + 4h + t % 4), for products
// whose other operand is read transposed.
template <int D>
__device__ __forceinline__ bf16x8 load_frag_perm(const char* tile, int row0, int ks, int lane) {
    const int row = row0 + (lane & 31), h = lane >> 5;
    const u32x2 lo = *reinterpret_cast<const u32x2*>(tile + tile_off<D>(row, 2 * ks) + 8 * h);
    const u32x2 hi = *reinterpret_cast<const u32x2*>(tile + tile_off<D>(row, 2 * ks + 1) + 8 * h);
    u32x4 r = {lo[0], lo[1], hi[0], hi[1]};
    return __builtin_bit_cast(bf16x8, r);
}

// One copy instruction: BYTES (4 or 16) per lane from global memory to LDS at dst + imm + BYTES lane; off: byte offset of the lane
// from the uniform address base.  Inline assembly hides from the compiler what it would otherwise put in between: one wait state
// from the write of M0 to the copy, and five from a vector instruction that has written base (readfirstlane, or a scalar
// register restored from a lane) to the copy.  The hardware checks neither.  FIRST: base may just have been formed.
template <int BYTES, bool FIRST>
__device__ __forceinline__ void copy_to_lds(unsigned dst, int imm, unsigned off, const void* base) {
    static_assert(BYTES == 16 || BYTES == 4, "widths of the instruction");
    constexpr int kWait = FIRST ? 3 : 0;  // s_nop n is n + 1 states
    if constexpr (BYTES == 16)
        asm volatile("s_add_u32 m0, %0, %1\n\ts_nop %4\n\tglobal_load_lds_dwordx4 %2, %3"
                     :
                     : "s"(dst), "i"(imm), "v"(off), "s"(base), "n"(kWait)
                     : "memory", "m0", "scc");
    else
        asm volatile("s_add_u32 m0, %0, %1\n\ts_nop %4\n\tglobal_load_lds_dword %2, %3"
                     :
                     : "s"(dst), "i"(imm), "v"(off), "s"(base), "n"(kWait)
                     : "memory", "m0", "scc");
}
template <int BYTES>
__device__ __forceinline__ void copy_to_lds(unsigned dst, int imm, unsigned off, const void* base, bool first) {  // (first: known after inlining)
    if (first) copy_to_lds<BYTES, true>(dst, imm, off, base);
    else copy_to_lds<BYTES, false>(dst, imm, off, base);
}

// Asynchronous copy of a [ROWS x D] bf16 tile from global memory straight into a swizzled LDS
// tile (global_load_lds_dwordx4: no staging registers).  One instruction moves 1 KB per wave and
// lands lane l's 16 bytes at LDS base + 16 l, so the lane that owns LDS position (row, chunk p)
// fetches global chunk p ^ swz(row): the swizzle is applied on the global side.  Rows at or
// beyond rows_valid re-read the last valid row (finite values that the callers mask out).
// The copy is complete for the issuing wave after wait_direct_loads().
template <int D, int ROWS, int NW = 4>  // NW: waves of the workgroup (all of them take part)
__device__ __forceinline__ void load_tile_direct(const __bf16* base, long ld, int row_begin, int rows_valid,
                                                 char* tile, int tid) {
    constexpr int kRowsPerInst = 1024 / (D * 2);
    constexpr int kInst = ROWS / (NW * kRowsPerInst);
    static_assert(ROWS % (NW * kRowsPerInst) == 0, "tile must split evenly over the workgroup's waves");
    const int lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
#pragma unroll
    for (int u = 0; u < kInst; ++u) {
        const int row = (u * NW + w) * kRowsPerInst + lane / (D / 8);
        const int c = (lane % (D / 8)) ^ swz<D>(row);
        const int grow = min(row_begin + row, rows_valid - 1);
        // Issued as inline assembly on purpose: for the builtin the compiler cannot tell which LDS
        // bytes a copy in flight will write and drains all of them (s_waitcnt vmcnt(0)) before the
        // next transposing LDS read, i.e. in the middle of the iteration.  Here the wait is ours:
        // wait_direct_loads() right before the barrier that publishes the stage.
        const unsigned dst = __builtin_amdgcn_readfirstlane((unsigned)(size_t)(ATTN_LDS char*)(tile + (u * NW + w) * 1024));
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
                     :
                     : "s"(dst), "v"(base + (long)grow * ld + c * 8)
                     : "memory", "m0");
    }
}
__device__ __forceinline__ void wait_direct_loads() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// The same copy for the tiles of a streaming loop, with everything that does not change from
// tile to tile taken out of the loop: each lane keeps the byte offset of its 16 bytes relative to
// the tile's first row (one register per copy instruction), the tile's first row is a scalar
// base address, and a copy is one instruction with no vector arithmetic in front of it.
// (Address arithmetic per copy - a 64-bit multiply-add, a clamp, the swizzle - is as expensive
// on the vector unit as the MFMA it feeds.)  Tiles that reach past rows_valid take the
// clamping path of load_tile_direct.  Offsets are 32-bit: ROWS * ld * 2 must stay below 2^32.
template <int D, int ROWS, int NW = 4>
struct TileLoader {
    static constexpr int kRowsPerInst = 1024 / (D * 2);
    static constexpr int kInst = ROWS / (NW * kRowsPerInst);
    static_assert(ROWS % (NW * kRowsPerInst) == 0, "tile must split evenly over the workgroup's waves");
    // whether the tile's address may come from vector registers: at d = 256 the scalar ones do not hold it in every kernel (the
    // CPU tests look for a copy without its waits in the assembly of every kernel)
    static constexpr bool kFormed = D == 256;
    unsigned voff[kInst];
    unsigned lds0;  // byte offset of this wave's first 1 KB piece inside a tile
    __device__ __forceinline__ void init(int tid, long ld) {
        const int lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
#pragma unroll
        for (int u = 0; u < kInst; ++u) {
            const int row = (u * NW + w) * kRowsPerInst + lane / (D / 8);
            const int c = (lane % (D / 8)) ^ swz<D>(row);
            voff[u] = (unsigned)row * (unsigned)ld * 2u + (unsigned)c * 16u;
        }
        lds0 = (unsigned)w * 1024u;
    }
    // The scalar base of the copy instructions: the address is uniform, but the compiler has to
    // be told so where it cannot prove it (it then hands the assembler a vector register pair).
    static __device__ __forceinline__ const __bf16* uniform(const __bf16* ptr) {
        const unsigned long long a = reinterpret_cast<unsigned long long>(ptr);
        const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)a);
        const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(a >> 32));
        return reinterpret_cast<const __bf16*>(((unsigned long long)hi << 32) | lo);
    }
    // first_row: address of the tile's first row (uniform); all ROWS rows must exist
    __device__ __forceinline__ void load(const __bf16* first_row_in, char* tile) const {
        const __bf16* first_row = uniform(first_row_in);
        const unsigned t0 =
            __builtin_amdgcn_readfirstlane((unsigned)(size_t)(ATTN_LDS char*)tile) + lds0;
#pragma unroll
        for (int u = 0; u < kInst; ++u) copy_to_lds<16>(t0, u * NW * 1024, voff[u], first_row, kFormed && u == 0);
    }
    // Copy instruction u of load() on its own, for callers that spread the copies over their MFMAs.  Their address has been through
    // hold(): formed from vector registers for each copy it would need the wait of a first copy every time.
    static __device__ __forceinline__ void hold(const __bf16*& first_row) {
        first_row = uniform(first_row);
        asm volatile("" : "+s"(first_row));
    }
    __device__ __forceinline__ void load_one(int u, const __bf16* first_row_in, char* tile) const {
        const __bf16* first_row = uniform(first_row_in);
        const unsigned t0 =
            __builtin_amdgcn_readfirstlane((unsigned)(size_t)(ATTN_LDS char*)tile) + lds0;
        copy_to_lds<16>(t0, u * NW * 1024, voff[u], first_row, kFormed && u == 0);
    }
    // any tile: clamps rows at rows_valid - 1 when the tile reaches past the end
    __device__ __forceinline__ void load(const __bf16* base, long ld, int row_begin, int rows_valid, char* tile,
                                         int tid) const {
        if (row_begin + ROWS <= rows_valid)
            load(base + (long)row_begin * ld, tile);
        else
            load_tile_direct<D, ROWS, NW>(base, ld, row_begin, rows_valid, tile, tid);
    }
};

// Between writes to LDS and reads of the same bytes by other lanes of the wave.  The hardware takes the LDS operations of a wave in order; the compiler is
// told here that lanes meet (by addresses alone, which differ per lane, it could move a read in front of a write).  No instruction.
__device__ __forceinline__ void wave_exchange() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A wave's result of 32 rows x W columns of bf16 on its way to memory through LDS: accumulators hold four consecutive columns of a
// row per lane, and stored as they are every instruction writes 8 bytes to each of 32 rows.  From here it leaves in whole rows,
// 16 bytes per lane.  (Rows 2 W + 16 bytes apart: 16 lanes that write one column group together touch every bank once.)
template <int W>
struct RowStage {
    static constexpr int kPitch = 2 * W + 16, kBytes = 32 * kPitch, kLanes = W / 8;  // lanes per row
    // columns 8 g + 4 h .. +3 of row l % 32
    static __device__ __forceinline__ void put(char* at, int g, u32x2 v, int lane) {
        *reinterpret_cast<u32x2*>(at + (lane & 31) * kPitch + 16 * g + 8 * (lane >> 5)) = v;
    }
    // rows 0 .. min(32, rows) - 1 to dst, ld elements apart, by `waves` waves of which this is number `wave`
    template <int ROWS = 32, int WAVES = 1>
    static __device__ __forceinline__ void store(const char* at, __bf16* dst, long ld, int rows, int lane, int wave = 0) {
        constexpr int kRows = 64 * WAVES / kLanes;
        const int c = lane % kLanes;
        if constexpr (WAVES == 1) wave_exchange();  // (several waves: behind their barrier)
#pragma unroll
        for (int r = 0; r < ROWS; r += kRows) {
            const int row = r + (64 * wave + lane) / kLanes;
            if (row < rows && (kRows <= ROWS || row < ROWS))
                *reinterpret_cast<u32x4*>(dst + (long)row * ld + 8 * c) = *reinterpret_cast<const u32x4*>(at + row * kPitch + 16 * c);
        }
        if constexpr (WAVES == 1) wave_exchange();  // (the next rows may come through the same place)
    }
};

// Marks a register value as used here.  Ordinary global loads issued before the streaming loop
// must be complete before it starts: otherwise the compiler's own wait for them lands inside the
// loop and, vmcnt being one in-order counter, also drains the tile copies in flight.
template <typename T>
__device__ __forceinline__ void settle(const T& v) {
    asm volatile("" : : "v"(v));
}

// Workgroup barrier that orders LDS traffic only: it waits for this wave's LDS operations but
// not for global loads still in flight (__syncthreads would also drain those).
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Start row of streamed tile `it` of a workgroup: dense tiles follow one another from t0;
// under a block mask, entry it / sub of the block list picks a 128-row block and it % sub the
// tile inside it.  The list read is forced onto the scalar unit (all values are uniform).
template <int TILE>
__device__ __forceinline__ int tile_start_row(const int32_t* list_idx, int lp0, int t0, int it) {
    constexpr int kSub = 128 / TILE;
    // the result is uniform and is made a scalar here: every address derived from it (tile copies, row
    // statistics) is then scalar arithmetic, not vector instructions that would compete with the MFMAs
    if (list_idx) {
        const int e = __builtin_amdgcn_readfirstlane(lp0 + it / kSub);
        // read through the constant address space: a scalar load (the lists are never written by these kernels),
        // which neither occupies a vector register nor waits behind the tile copies and atomics in flight
        typedef const int32_t __attribute__((address_space(4))) * const_i32_ptr;
        const const_i32_ptr cidx = (const_i32_ptr)(unsigned long long)list_idx;
        return cidx[e] * 128 + (it % kSub) * TILE;
    }
    return __builtin_amdgcn_readfirstlane((t0 + it) * TILE);
}

// Block lists under the causal rule.  The row list of query block b (ascending key blocks) only
// needs the entries <= b, the column list of key block b (ascending query blocks) only the entries
// >= b: everything else is invisible, and a tile that is not in the list is neither copied nor
// waited for.  All values are uniform (scalar loads).
__device__ __forceinline__ int causal_row_entries(const int32_t* idx, int first, int count, int b) {
    while (count > 0 && idx[first + count - 1] > b) --count;
    return count;
}
__device__ __forceinline__ int causal_col_skip(const int32_t* idx, int first, int count, int b) {
    int skip = 0;
    while (skip < count && idx[first + skip] < b) ++skip;
    return skip;
}

// Head and tile decoding shared by the kernels.  Workgroups are handed to the 8 XCDs round
// robin by linear id, so ids congruent mod 8 share an L2: all tiles of one (batch, head) are
// given to one XCD when the head count allows it.
__device__ __forceinline__ void decode_block(int linear, int tiles, int bh_total, int& bh, int& tile) {
    if ((bh_total & 7) == 0) {
        const int xcd = linear & 7, slot = linear >> 3;
        bh = (slot / tiles) * 8 + xcd;
        tile = slot % tiles;
    } else {
        bh = linear / tiles;
        tile = linear % tiles;
    }
}

// The same for a causal launch whose tiles differ in length: `rank` 0 is the longest tile of a head.  `resident` > 0: ranks
// run over all heads of an XCD together, longest first, and the first `resident` rounds of 32 (the workgroups that
// share the XCD's 32 CUs from the start) go back and forth, so that each CU gets a long, a short, a long ... one.
// `resident` == 0: head after head.
__device__ __forceinline__ void decode_block_causal(int linear, int tiles, int bh_total, int resident, int& bh, int& rank) {
    if (resident == 0) {
        decode_block(linear, tiles, bh_total, bh, rank);
        return;
    }
    const bool by_xcd = (bh_total & 7) == 0;
    const int xcds = by_xcd ? 8 : 1, cus = by_xcd ? 32 : 256;
    const int xcd = linear & (xcds - 1), heads = bh_total / xcds;
    int slot = linear / xcds;
    const int round = slot / cus;
    if ((round & 1) && round < resident) {  // (a last round that is not full starts with its shortest as well)
        const int first = round * cus, last = min(first + cus, tiles * heads) - 1;
        slot = first + last - slot;
    }
    rank = slot / heads;
    bh = (slot % heads) * xcds + xcd;
}

// `resident` for a causal launch of `grid` workgroups of which per_cu fit a CU.  In head order a CU got the same tile index of
// two heads (the two longest, say) while the launch is small, and the last head's long tiles started late when it is a
// few rounds long.  Over all heads, longest first (us, forward / dQ / dK dV): d = 64 b4 h16 n2048 70 / 83 / 97 -> 49 / 63 /
// 87; d = 128 b2 h16 n1024 28 / 35 / 34 -> 27 / 34 / 29, n4096 178 / 229 / 263 -> 140 / 186 / 261; d = 256 b3 h5 n3000
// 219 / 260 / 221 -> 134 / 157 / 184.  From eight rounds on head order is kept: the tail is short then, and an XCD that
// works on one head at a time finds more in its L2 (d = 128 b2 h32 n8192: forward the same, dK dV 1982 against 2056 us).
inline int causal_resident(int grid, int per_cu) { return grid < 8 * 256 * per_cu ? per_cu : 0; }

// Whether a launch of `blocks` blocks of 128 queries, per_cu of which fit a CU, leaves so much of the chip idle that blocks of 64
// queries, with the two key halves of a tile on two waves, are faster: with one block on a CU a SIMD has one wave, which waits out
// every latency of its chain.  The line lies where the smaller blocks still fit the chip twice per CU (once at d = 256).  Under the
// causal rule half of their tiles do not exist, and twice as many are still faster, but not under a block mask, whose lists the
// host does not know: a call that could have been made with a mask gets the line of the masked one, so that a causal call and
// the same call through a lower-triangular mask have the same bits.  `half_exist`: causal, and there is no such call (the weight
// gradient).  us, forward / dQ, 128 -> 64 queries, 16 heads:
//   d = 128, full     n1024 26 / 32 -> 20 / 23    n2048 50 / 62 -> 47 / 57    n3072 (beyond the line) 88 / 117 -> 110 / 130
//   d = 128, causal   n1024 26 / 31 -> 19 / 22    n2048 47 / 58 -> 38 / 42    n4096 105 / 131 -> 91 / 110
//   d = 64, full      n2048 36 / 41 -> 33 / 35    n3072 (beyond) 62 / 75 -> 64 / 69    n4096 (beyond) 95 / 113 -> 102 / 131
//   d = 256, full     n1024 53 / 64 -> 39 / 43    n1536 (beyond) 76 / 92 -> 100 / 107
//   d = 256, causal   n2048 96 / 113 -> 77 / 84   n3072 (beyond) 140 / 164 -> 166 / 175
// (the forward of d = 256 before it was pipelined; since then, full, n1024 42 -> 30, n1536 (beyond) 59 -> 78; causal, n2048 74 -> 62, but
// a full call of that size lies on the same side of the line, n3072 (beyond) 105 -> 126)
// and calls on both sides of the line with the rule against 128 queries always (us, forward / backward with dK dV, 16 heads; a
// mask keeps the diagonal and the stated share of the other blocks):
//   d = 64, causal    n1024 19 / 39 -> 15 / 32    n2048 34 / 72 -> 26 / 57
//   d = 64, mask 10 % n2048 14 / 35 -> 13 / 33    40 % and causal n2048 17 / 43 -> 15 / 41
//   d = 128, mask 10 % n1024 13 / 35 -> 11 / 31   n2048 19 / 52 -> 18 / 51    40 % and causal n2048 23 / 65 -> 20 / 63
//   d = 256, mask 10 % n600 26 / 57 -> 19 / 47    n1024 26 / 63 -> 20 / 53    40 % and causal n1024 38 / 80 -> 28 / 65
inline bool few_blocks(int blocks, int per_cu, bool half_exist) {
    return (long)blocks * (half_exist ? 1 : 2) <= 256 * (per_cu < 2 ? per_cu : 2);
}

// Kernel arguments common to the fused kernels.  Strides are in elements.
struct FusedParams {
    const __bf16 *Q, *K, *V, *O, *dO;
    __bf16 *Oout, *dQ, *dK, *dV;
    const float* LSE;    // [batch*heads, n] natural-log sums (backward input)
    float* LSEout;       // forward output
    float* delta;        // [batch*heads, n] rowsum(dO o O), workspace
    long stride_b, stride_h, stride_n;
    int batch, heads, n;
    float scale;
    int causal;
    // block-sparse lists (nullptr = dense): ptr/idx give, per 128-row block of the resident
    // operand, the 128-row blocks of the streamed operand that are visible, ascending.
    const int32_t *list_ptr, *list_idx;
    // under a block mask, optionally: the 128-row blocks of the resident operand in the order the
    // workgroups take them (longest list first), nullptr = ascending
    const int32_t* order;
    // masks per (batch, head): entries between the list_ptr (order) arrays of consecutive pairs; 0 = one shared mask
    int list_stride, order_stride;
    int resident;  // causal, no mask: see decode_block_causal
    bool mask_form;  // the entry point has a form with a block mask: see few_blocks
    bool may_join;   // backward: the caller did not ask for two launches
};

}  // namespace attn
