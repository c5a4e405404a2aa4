// Which tile a workgroup of the large-d kernels has: index arithmetic and nothing of the device, so that the CPU tests run it as well.
#pragma once
#include <math.h>

#if defined(__HIPCC__)
#define ATTN_HD __host__ __device__ __forceinline__
#else
#define ATTN_HD inline
#endif

namespace attn {

// Consecutive workgroups go to the 8 XCDs in turn.  The tile of a workgroup, so that each XCD gets a contiguous run of the tiles (runs that differ by
// one at most): neighbours share their operands in the XCD's L2.  us of the call, such runs only for multiples of 8 -> always: causal, whose visible tiles
// often are none, d = 512 h7 n2600 forward 105 -> 99, backward 168 -> 163; d = 128 in four phases h7 n3000 (546 tiles) 114 -> 109; d = 1024 h7 n1571
// 79 -> 75, 133 -> 128; full d = 512 h5 n1571 68 -> 63, 100 -> 86; d = 1024 h6 n3824 418 -> 390, 901 -> 871.
ATTN_HD int xcd_run(int block, int total) {
    const int xcd = block & 7, each = total >> 3, more = total & 7;
    return xcd * each + (xcd < more ? xcd : more) + (block >> 3);
}

// Score tiles of 256 queries x 256 keys, nb by nb of them for each of bhs (batch, head) pairs.  Under the causal rule only the tiles on and below the
// diagonal are launched.  With all of them launched and the others ending at once, the others still had their share of the chip: a workgroup takes
// nearly all the LDS of a CU, workgroups start in order, and one that will end at once waits for a CU while those behind it could have started.  us
// of the call, causal, all launched -> those: d = 512 h7 n1571 (196 of 343 tiles) forward 77 -> 63, backward 140 -> 115; h6 n3824 200 -> 163,
// 324 -> 285; d = 1024 h7 n1571 111 -> 88, 195 -> 154; where all start at once or fill the chip many times over the same (h12 n1000, h8 n4096).
ATTN_HD int score_tiles(int nb, bool causal) { return causal ? nb * (nb + 1) / 2 : nb * nb; }
struct ScoreTile {
    int bh, qb, kb;
};
// Regions of 4 x 4 tiles (full calls: where the count allows) read the fewest rows.
ATTN_HD ScoreTile score_tile(int block, int nb, int bhs, bool causal) {
    const int per_head = score_tiles(nb, causal), total = per_head * bhs;
    const int t = xcd_run(block, total);
    ScoreTile s;
    s.bh = t / per_head;
    const int tile = t - s.bh * per_head;
    if (causal) {
        // 8 R R + 2 R tiles in front of the rows 4 R .. 4 R + 3: R regions of 16 and one of 10 on the diagonal for each four rows
        int R = (int)((sqrtf(1.f + 8.f * (float)tile) - 1.f) * 0.125f);
        if (8 * R * R + 2 * R > tile) --R;
        else if (8 * (R + 1) * (R + 1) + 2 * (R + 1) <= tile) ++R;
        int in = tile - (8 * R * R + 2 * R);
        const int rows = nb - 4 * R < 4 ? nb - 4 * R : 4, beside = 4 * R * rows;
        if (in < beside) {
            const int region = in / (4 * rows);
            in -= region * 4 * rows;
            s.qb = 4 * R + in / 4;
            s.kb = 4 * region + in % 4;
        } else {
            in -= beside;
            const int row = in >= 6 ? 3 : in >= 3 ? 2 : in >= 1 ? 1 : 0;
            s.qb = 4 * R + row;
            s.kb = 4 * R + in - row * (row + 1) / 2;
        }
    } else if ((nb & 3) == 0) {
        const int region = tile / 16, in = tile % 16, regions = nb / 4;
        s.qb = (region / regions) * 4 + in / 4;
        s.kb = (region % regions) * 4 + in % 4;
    } else {
        s.qb = tile / nb;
        s.kb = tile % nb;
    }
    return s;
}

// The product tiles of a launch of `count` products (forward: O; backward: dV = P^T dO, dK = dS^T Q, dQ = dS K, whose tiles together fill what a launch
// for each of the three leaves idle), mbs row blocks by nbs column blocks for each (batch, head).
struct ProductTile {
    int which, bh, mb, nb;
};
// The column tiles of a row block read the same rows of P or dS, so they follow one another on one XCD.  Under the causal rule row blocks differ
// in length: longest first, the row blocks to the XCDs in turn (the last count * mbs * bhs % 8 of them, the shortest, tile by tile).  Dealt out tile
// by tile where the (batch, head) pairs are no multiple of 8, every XCD read all of P.  us of the call, causal, tile by tile -> row block by row block:
// d = 512 h9 n1571 forward 68 -> 66, backward 145 -> 104; h6 n3824 163 -> 154, 285 -> 265; d = 1024 h4 n4096 220 -> 188, 388 -> 375; h5 n1571 74 -> 71, 120 -> 111
ATTN_HD ProductTile product_tile(int block, int count, int mbs, int nbs, int bhs, bool causal) {
    ProductTile t;
    int s = block;
    if (causal) {
        const int units = count * mbs * bhs, in_turn = (units & ~7) * nbs;
        int unit;
        if (s < in_turn) {
            const int xcd = s & 7;
            s >>= 3;
            unit = (s / nbs) * 8 + xcd;
        } else {
            s -= in_turn;
            unit = (units & ~7) + s / nbs;
        }
        t.nb = s % nbs;
        t.bh = unit % bhs;
        unit /= bhs;
        t.which = unit % count;
        const int rank = unit / count;
        t.mb = count == 3 && t.which < 2 ? rank : mbs - 1 - rank;  // keys from the first block on, queries from the last
    } else {
        const int total = count * mbs * nbs * bhs;
        if ((total & 7) == 0) s = (s >> 3) + (s & 7) * (total >> 3);
        t.nb = s % nbs;
        s /= nbs;
        t.mb = s % mbs;
        s /= mbs;
        t.which = s % count;
        t.bh = s / count;
    }
    return t;
}

}  // namespace attn
