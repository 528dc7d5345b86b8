// Tile arithmetic shared by the host's launch rules and the GEMM kernels; plain
// C++, so that the rules can be checked on the CPU.
#pragma once

// Tiles of one XCD's contiguous share when 8 XCDs with `workgroups` each walk
// the `total` tiles of a grouped product: rounded up to a multiple of 4, so that
// most bands of row tiles (kRasterBand) stay on one XCD, unless that would take
// its workgroups one more round.  The tiles of few experts often fill less than
// one: 48 tiles of 32 K steps each, shares of 8 walked by 6 workgroups per XCD
// in two rounds, 66 us; shares of 6 in one, 40.
constexpr int xcd_share(int total, int workgroups) {
    const int n = (total + 7) >> 3, up = (n + 3) & ~3;
    return (up + workgroups - 1) / workgroups == (n + workgroups - 1) / workgroups ? up : n;
}
