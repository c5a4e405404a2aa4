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

}  // namespace attn
