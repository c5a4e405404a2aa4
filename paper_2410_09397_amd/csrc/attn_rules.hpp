// Rules that choose a kernel of the fused backward by the size of the call: nothing of the device, so that the CPU tests run them as well.
#pragma once

namespace attn {

// Whether a short call runs in one launch alone (bwd_short_kernel): every key block forms the row sums of the queries it sees again and keeps
// them in LDS, instead of a launch in front that forms each once (3 to 4 us, and 2 us of the host).  The price grows with the rows and with
// the blocks that share a CU, so the line lies at 256 rows (d = 64: 448) and one block per CU; under the causal rule, where a key block sees half of the
// rows, at d = 64 at three, without it there at two up to 200 rows.  Not under a block mask, whose order of blocks needs the launch in front anyway.  us of the backward, two launches -> one:
//   full     d64 h33 n200 (264 blocks) 11.9 -> 11.0, h62 n200 (496) 13.8 -> 13.4, h80 n200 (640, beyond) 13.8 -> 14.0, h47 n256 (376, beyond) 12.6 -> 13.4
//            h2 n300 12.0 -> 9.5, h17 n448 (238 blocks) 12.6 -> 11.7, h38 n320 (380, beyond) 14.0 -> 15.5, h45 n448 (630, beyond) 22.0 -> 25.8
//   causal   d64 h8 n333 11.4 -> 10.2, h50 n320 (500 blocks) 13.0 -> 12.0, h63 n384 (756) 16.8 -> 16.8, h110 n320 (1100, beyond) 21.7 -> 21.8
//   d128 h16 n256 12.6 -> 12.0, h31 n256 causal 14.8 -> 14.3, h37 n256 (296 blocks, beyond) 17.8 -> 26.7   d256 b4 h16 n66 16.7 -> 12.7, b2 h23 n97 causal 17.8 -> 14.2
constexpr int kOwnRows = 448;
inline bool own_rows(bool causal, int n, int d, long grid, bool masked) {
    if (masked || n > (d == 64 ? kOwnRows : 256)) return false;
    return grid <= (d != 64 ? 256 : causal ? 768 : n <= 200 ? 512 : 256);
}

// Whether blocks of 64 queries and of 64 keys get eight waves instead of four (two groups that take a block's tiles in turn and add up at
// the end; all the LDS of a CU at d = 128).  A block of four waves that has a CU to itself waits out every latency of its chain (1.3 us a
// tile at d = 128); two of them on a CU take 2 us for a tile each, and eight waves as long for two tiles of one block.  So the line lies where every block has
// a CU; under the causal rule, whose blocks differ in length, at one and a half.  Not for a few tiles, which the end of the block
// costs more.  The rule does not look at the mask (see few_blocks) nor at whether one launch or two are made: the sums of a block keep their order.
// `mask_form`: dQ and dK / dV share the chip; else (the weight gradient) dQ is alone.  us of the backward, four waves -> eight:
//   full     d128 h11 n700 24.0 -> 21.6   h4 n2048 48.9 -> 41.6   h1 n8000 163 -> 127   h10 n1024 (beyond) 32 -> 44   d64 h4 n1500 27.3 -> 22.0
//   causal   d128 h16 n700 21.9 -> 21.0   h2 n4000 72.5 -> 61.9   h14 n1024 (beyond) 29.2 -> 30.0   d64 h12 n1000 20.3 -> 18.6   h24 n600 (beyond) 16.0 -> 17.4
//   weight gradient   full d128 h16 n1024 54.8 -> 52.8, h5 n2412 85 -> 77, d64 h12 n1500 (beyond) 56 -> 64   causal d64 h16 n1200 44.6 -> 41.8, d128 h2 n9251 275 -> 237
// dQ alone under the causal rule, where no masked call with shorter lists loses by it (see eight_waves): more blocks than CUs only if the short ones among
// them leave room for the rest, so the line moves with the length, from one block for each CU to two:
//   weight gradient, causal   d64 h60 n300 (300 blocks, beyond) 28.7 -> 30.3, h61 n336 (366, beyond) 31.1 -> 33.6   d128 h41 n500 (328, beyond) 49.5 -> 52.7
//            d64 h26 n700 (286) 1.04 as fast, h34 n700 (374, beyond) 0.98   d128 h20 n1024 (320) 1.04, h23 n1024 (368, beyond) 0.95, h18 n1280 (360) 1.03
//   causal   d64 h20 n1500 54.9 -> 53.9, h6 n5000 118 -> 107, h30 n1024 (beyond) 44.8 -> 45.3   d128 h16 n1900 85.6 -> 82.3, h4 n8192 268 -> 243, h22 n1900 (660 blocks, beyond) 98 -> 105
inline bool eight_waves_bwd(bool causal, bool mask_form, int n, int bh) {
    const long blocks = (long)((n + 63) / 64) * bh * (mask_form ? 2 : 1);
    if (n <= 256) return false;
    if (!causal) return blocks <= 256;
    return blocks <= (mask_form ? 384 : n < 640 ? 256 : n < 1200 ? 320 : n < 1500 ? 384 : 512);
}

}  // namespace attn
