// sizes.hpp -- transform lengths n the library is compiled for (one object per size):
// 2^a 3^b (b <= 1; 384, 768 and 1536 make padding to B_3 reach n = 256, 512 and 1024),
// 5 * 2^a and 7 * 2^a.
// The build script reads this list.
#pragma once
#define GS_SIZE_LIST(X) X(8) X(12) X(16) X(20) X(24) X(28) X(32) X(40) X(48) X(56) X(64) X(80) X(96) X(112) X(128) X(160) X(192) X(224) X(256) X(320) X(384) X(512) X(640) X(768) X(1024) X(1536) X(2048)
#define GS_MAX_N_3D 1024

// Grid of the fused pass: persistent (rounds of co-resident blocks looping over pencil
// groups, the per-thread stage twiddles kept in registers across groups) for 3D cubic grids of
// n = 256 and, without the dipolar factor (whose registers on top cost occupancy), 384, 512, 640 and
// 768; one block per pencil group elsewhere, where the twiddles held across
// groups cost occupancy.  Whole evaluations, one block per group -> persistent: 256^3 651 ->
// 620, 384^3 2766 -> 2665, 512^3 5874 -> 5809 us, 640^3 16.4 -> 15.5, 768^3 25.6 -> 25.4 ms, but 160^3 200 -> 203, 320^3 1610 ->
// 1682, dipolar 384^3 2693 -> 2910, dipolar 128^3 87.2 -> 88.6 us, 1024^3 57.2 -> 58.2 ms; 96^3, 128^3 and 192^3 equal.
constexpr bool gs_fused_persistent(int d, int n, bool dipolar) {
    return d == 3 && (n == 256 || ((n == 384 || n == 512 || n == 640 || n == 768) && !dipolar));
}
// The same on grids whose axes differ, by the length n of the fused axis: always, never, or where
// the pass's array X2 (a slab's planes) is larger than the 256 MB cache (with the energy's sums,
// whose kernel gives up one wave of three for the loop, from 190 MB).  Whole evaluations (z
// first), one block per group -> persistent:
//   plain: 128x256x512 648 -> 634, 512x256x128 698 -> 661, 384x256x320 1570 -> 1470, 256x192x320 637
//   -> 612, 128x256x192 243 -> 238; 192x128x160 156 -> 158 (energy 170 -> 166); but 224x320x192 (28
//   values per thread) 658 -> 759 us
//   dipolar, 192 and 256: 192x128x160 164 -> 159, 192x256x128 261 -> 250, 256x128x192 257 -> 251,
//   256x192x320 668 -> 630, 256x256x512 1513 -> 1430 us; 384 and 512 equal
//   dipolar, 128: the loop takes the kernel from four waves per SIMD to two, which costs as long as
//   the cache serves it: 128x96x96 (X2 38 MB) 60.3 -> 62.3, 128x96x160 85.1 -> 89.4, 128x256x192
//   (202 MB) 247.5 -> 252.8, 128x256x224 (236 MB) 312 -> 317, and gains beyond: 128x256x320 (336 MB)
//   421 -> 420, 128x384x256 506 -> 492, 128x512x256 670 -> 655; with the energy 128x160x256 (168 MB)
//   230.8 -> 233.6, 128x256x192 (202 MB) 272.3 -> 269.6, 128x256x224 340 -> 333, 128x256x320 459 ->
//   442 us.
enum class Loop { never, always, beyond_cache };
constexpr Loop gs_fused_loop_g(int d, int n, bool dipolar) {
    if (d != 3) return Loop::never;
    if (n == 128) return dipolar ? Loop::beyond_cache : Loop::always;
    return n == 192 || n == 256 || ((n == 384 || n == 512) && !dipolar) ? Loop::always : Loop::never;
}
constexpr bool gs_fused_persistent_g(int d, int n, bool dipolar, bool energy, double x2_bytes) {
    const Loop r = gs_fused_loop_g(d, n, dipolar);
    return r == Loop::always || (r == Loop::beyond_cache && x2_bytes > (energy ? 190e6 : 256e6));
}

// Lengths for which the cubic passes are also compiled in tile-shape variants (more or fewer
// rows or pencils per block; the same bits) that the plan autotuner chooses among.
constexpr bool gs_tile_variants(int n) { return n >= 128; }
