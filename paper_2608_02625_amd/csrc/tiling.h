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

// Tile of a GEMM launch and its variant (see the list in gemm.hip).
struct GemmTile {
    int bm, bn, variant;
};

// Tiles of a dense product with M x N outputs of K products each.  The ping-pong
// 256x256 tile is the best per output, but one is a CU's whole work for a while:
// what decides is which part of the area of its rounds over the 256 CUs the
// product covers.  Below that, tiles of a quarter and a sixteenth of the size,
// as many as two (or three) workgroups per CU hold at once.  A shorter K needs
// fuller rounds, since a tile's start and epilogue weigh more.  Times below are
// us with the launch, big tiles against the best of the small ones.
struct BigTiles {
    long long rounds;
    double fill;
};
constexpr long long tiles_of(long long M, long long N, int bm, int bn) {
    return (M + bm - 1) / bm * ((N + bn - 1) / bn);
}
constexpr BigTiles big_tiles(long long M, long long N) {
    const long long rounds = (tiles_of(M, N, 256, 256) + 255) / 256;
    return {rounds, (double)M * (double)N / (65536. * 256. * (double)rounds)};
}

// Residual products (O, dense down).  Whole tiles, one round, K 1024: 16384 x
// 1024 52 / 47; K 1536: 8192 x 1536 (fill .75) 50 / 51, 16384 x 1536 (.75 of
// two) 102 / 101; K 2048: 6144 x 2048 (.75) 59 / 60, 8192 x 2048 73 / 79, 10240
// x 2048 (.62 of two) 112 / 94.  From two full rounds on an epilogue overlaps
// the next tile: K 1024: 32768 x 1024 95 / 112, 24576 x 1024 (.75) 85 / 83; K
// 768: 40960 x 768 (.94) 83 / 87; K 512: 65536 x 512 72 / 76.
// Partly filled tiles (rows or columns not a multiple of 256) check every
// element in their epilogue, 15 to 25 us at the end of the launch: 8100 x 2048
// x 2048 97 / 80 (8192: 73 / 79), 16300 163 / 168, 12200 (.74 of two) 134 / 122,
// 32768 x 1152 x 1152 (.75 of three) 154 / 127, 4000 x 4096 x 4096 138 / 148.
// Small tiles, K 2048: 512 rows (256 tiles of 64x64) 15.2 on 64x64 with five
// stages, 21.0 on 128x64; 1263 rows (640) 28.2 on 64x64 with three stages, 30.2
// on 64x128; 2048 rows (1024) 30.6 on 128x128, 35.3 on 64x128.
constexpr GemmTile resid_tile(long long M, long long N, long long K) {
    const BigTiles b = big_tiles(M, N);
    const bool whole = M % 256 == 0 && N % 256 == 0;
    const bool big = !whole      ? K * b.rounds >= 3072 && b.fill >= 0.82
                     : K >= 1280 ? b.fill >= 0.75
                                 : K >= 512 && b.rounds >= 2 && b.fill >= 0.82;
    if (big) return {256, 256, 11};
    const long long n = tiles_of(M, N, 64, 64);
    if (n <= 512) return {64, 64, 3};
    if (n <= 768) return {64, 64, 4};
    return {128, 128, 3};
}

// QKV (M = features, N = tokens).  K 2048, 3072 features: 4096 tokens (fill .75)
// 59 / 59, 6144 (.56 of two) 105 / 89, 10240 (.94) 122 / 151; K 1536, 2560: 5120
// (.78) 48 / 58, 4096 (.62) 44 / 44, 8192 (.62 of two) 88 / 76; K 1024, 3072:
// 4096 (.75) 38 / 35, 4200 (.77) 39 / 43, 8192 (.75 of two) 69 / 64, 32768 213 /
// 255; K 768, 2304: 6144 (.84) 35 / 37, 16384 (.75 of three) 87 / 77; K 512,
// 1536: 10240 (.94) 30 / 30, 16384 (.75 of two) 49 / 41, 32768 76 / 80; K 384,
// 1152: 65536 102 / 100; K 256, 768: 32768 (.75 of two) 40 / 32, 65536 56 / 58;
// K 128, 512: 65536 41 / 37.  Small tiles, K 2048: 512 tokens (192 tiles of
// 128x64) 21.6, on 128x128 26.8; 1263 (480) 28.8 / 28.4; 2048 (768) 43.1 / 38.8.
// With 4096-long rows 128x128 is ahead sooner: 512 tokens (384 tiles of 128x64)
// 52.0 / 45.5.
constexpr GemmTile qkv_tile(long long M, long long N, long long K) {
    const double least = K >= 1536 ? 0.72 : K >= 1024 ? 0.76 : K >= 768 ? 0.83 : 0.92;
    if (K >= 512 && big_tiles(M, N).fill >= least) return {256, 256, 11};
    return tiles_of(M, N, 128, 64) <= (K < 4096 ? 512 : 256) ? GemmTile{128, 64, 3} : GemmTile{128, 128, 4};
}

// Gate/up of the dense FFN: M rows, N interleaved gate and up columns.  Half the
// stores per product, so big tiles are ahead sooner, in a single round (no
// second one nearly empty) from half of it on.  K 4096, 22016 columns: 512 rows
// (fill .67) 81 / 102, 256 (.34) 77 / 79; K 2176, 8704: 1024 (.53) 46 / 52, 2048
// (.53 of two) 92 / 83, 4096 (.71 of three) 145 / 155; K 1024, 8192: 1024 (.5)
// 25 / 23, 4200 (.68 of three) 74 / 76, 32768 435 / 552; K 512, 4096: 4096 22 /
// 24, 6144 (.75 of two) 31 / 33, 5120 (.61 of two) 30 / 28; K 256, 2048: 6144
// (.75) 14.6 / 14.0, 20480 (.83 of three) 30 / 32, 32768 41 / 47; K 128, 2048:
// 8192 13.7 / 14.7, 65536 63 / 70. Small tiles, 64x128 / 128x128: while one per
// CU is enough the smaller ones, K 1024: 256 rows (256 tiles of 64x128) 10.9 /
// 13.6, 320 (320) 15.9 / 13.9; K 2048, 11264 columns: 128 rows (176) 15.3 /
// 20.8, 256 (352) 22.7 / 21.9; K 4096, 22016: 64 rows (172) 44.0 / 46.6, 128
// (344) 65 / 52.
constexpr GemmTile gate_up_tile(long long M, long long N, long long K) {
    const BigTiles b = big_tiles(M, N);
    if (b.fill >= (K < 512 ? 0.8 : K >= 1024 && b.rounds == 1 ? 0.51 : 0.67)) return {256, 256, 11};
    return tiles_of(M, N, 64, 128) <= 256 ? GemmTile{64, 128, 3} : GemmTile{128, 128, 3};
}

// Expert products of `groups` experts (shared ones among them) of ffn hidden
// features: what counts is the rows that an expert gets on average.  gate/up +
// down in us, d 2048, 64x128 / 128x128 / 256x256 tiles.  65 groups of 1024: 12
// rows each 174 / 207 / 237; 64 rows 201 / 198 / 218; 96 rows 201 / 199 / 219;
// 112 rows - / 210 / 243; 128 rows, two inputs, 254 / 226 / 238 and - / 251 /
// 250; 158 rows - / 279 / 248.  96 of 768: 64 rows 187 / 196 / 210; 107 rows 233
// / 217 / 224; 128 rows 286 / 254 / 237. An expert with more rows than a tile
// takes its weights twice: with many groups that costs more than the finer split
// gains.  128 of 768: 48 rows 225 / 230 / 231; 64 rows 277 / 255 / 251; 96 rows
// 317 / 274 / 261.  161 of 1024: 38 rows 372 / 382 / 401; 51 rows 423 / 406 /
// 426; 77 rows 496 / 435 / 438.  257 of 1536, d 4096: 47 rows - / 1866 / 1851;
// 64 rows 2228 / 1953 / 1902.  The line between them, in gate/up tiles of 128
// columns, lies between the 1152 of 96 groups of 768 and the 1536 of 128.
constexpr GemmTile expert_tile(long long groups, long long ffn, double rows) {
    const bool few = groups * ((2 * ffn + 127) / 128) <= 1280;
    if (rows <= 40 || (few && rows <= 72)) return {64, 128, 3};
    if (rows <= (few ? 120 : 48)) return {128, 128, 3};
    return {256, 256, 11};
}
