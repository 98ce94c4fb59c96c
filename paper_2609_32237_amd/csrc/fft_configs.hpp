// fft_configs.hpp -- per-size kernel shapes and the instantiation dispatcher.
//
// Shapes (points per thread P, transforms per workgroup C, radix sequence,
// exchange mode, twiddle mode, persistence) are chosen for gfx950: wave64,
// 160 KiB LDS per CU, 512 VGPRs per SIMD lane.  Rows keep one transform per
// 64-1024 threads; columns keep a strip of C adjacent columns so each row
// access is a C-element segment.  The paper's M6 schedules (Section VI:
// 16-8-8-8 for 8192 and 16-16-8-8 for 16384, 16 values per thread) were
// shaped by a 32 KiB threadgroup buffer; these use larger radices because the
// LDS is five times larger.
//
// Each size lists its variants.  row_shape, kRowMatched and column_shape name
// the one that a call takes (the migration pass and the rows with the binary16
// exchange take index 0 of theirs).  Every variant computes the same
// transform, and the tests force each of them.
#pragma once

#include "fft_kernel.hpp"

namespace mi355fft {

template <int N>
struct Configs;

// Each list's defaults are given per storage (FP32, FP16) for the plain
// transform and for the matched-filter (SAR) kernels (storage of the
// intermediate): FP16 storage moves half the bytes per point, so its kernels
// are limited by arithmetic issue and prefer the higher-occupancy split
// exchange; the matched-filter kernels hold two transforms' worth of state and
// prefer the shapes that do not spill.  The TWMODE 0 variants are kept as
// regression cases for the table-read twiddle path.
//                 N     P  C  COLS   XCHG        TW PERSIST radices
// Short transforms serve as the column passes of four-step transforms longer
// than 16384 points (many columns per workgroup, one or two exchanges).
template <>
struct Configs<64> {
    using Rows = KList<KCfg<64, 16, 16, false, XCHG_SPLIT, 1, false, Radices<16, 4>>>;
    using Cols = KList<KCfg<64, 16, 64, true, XCHG_SPLIT, 1, false, Radices<16, 4>>>;
    using Rcmc = Rows;
    using RowsHalf = Rows;
    static constexpr int kRowDefault[2] = {0, 0};
    static constexpr int kRowMatched[2] = {0, 0};
};
template <>
struct Configs<128> {
    using Rows = KList<KCfg<128, 16, 16, false, XCHG_SPLIT, 1, false, Radices<16, 8>>>;
    using Cols = KList<KCfg<128, 16, 32, true, XCHG_SPLIT, 1, false, Radices<16, 8>>>;
    using Rcmc = Rows;
    using RowsHalf = Rows;
    static constexpr int kRowDefault[2] = {0, 0};
    static constexpr int kRowMatched[2] = {0, 0};
};
template <>
struct Configs<256> {
    using Rows = KList<KCfg<256, 16, 16, false, XCHG_SPLIT, 1, false, Radices<16, 16>>>;
    using Cols = KList<KCfg<256, 16, 16, true, XCHG_SPLIT, 1, false, Radices<16, 16>>,
                       KCfg<256, 16, 32, true, XCHG_SPLIT, 1, false, Radices<16, 16>>>;
    using Rcmc = Rows;
    using RowsHalf = Rows;
    static constexpr int kRowDefault[2] = {0, 0};
    static constexpr int kRowMatched[2] = {0, 0};
};
template <>
struct Configs<512> {
    using Rows = KList<KCfg<512, 16, 8, false, XCHG_SPLIT, 1, false, Radices<16, 16, 2>>>;
    // 32 points per thread in two stages: one exchange instead of two (the
    // four-step passes of 2^25 points 106 + 104 against 112 + 106 us)
    using Cols = KList<KCfg<512, 32, 16, true, XCHG_SPLIT, 1, false, Radices<32, 16>>,
                       KCfg<512, 32, 32, true, XCHG_SPLIT, 1, false, Radices<32, 16>>>;
    using Rcmc = Rows;
    using RowsHalf = Rows;
    static constexpr int kRowDefault[2] = {0, 0};
    static constexpr int kRowMatched[2] = {0, 0};
};
template <>
struct Configs<1024> {
    using Rows = KList<KCfg<1024, 16, 4, false, XCHG_SPLIT, 1, false, Radices<16, 16, 4>>,
                       KCfg<1024, 16, 4, false, XCHG_FULL, 1, false, Radices<16, 16, 4>>,
                       KCfg<1024, 16, 4, false, XCHG_FULL, 1, true, Radices<16, 16, 4>>,
                       KCfg<1024, 16, 4, false, XCHG_FULL, 0, false, Radices<16, 16, 4>>,
                       KCfg<1024, 16, 1, false, XCHG_FULL, 1, false, Radices<16, 16, 4>>,
                       // every exchange across the lanes of one wave, no LDS:
                       // four transforms (waves) or one per workgroup
                       KCfg<1024, 16, 4, false, XCHG_LANE, 1, false, Radices<16, 16, 4>>,
                       KCfg<1024, 16, 1, false, XCHG_LANE, 1, false, Radices<16, 16, 4>>>;
    // two stages, one exchange; 8 or 16 columns (64-byte pieces or whole lines in FP32)
    using Cols = KList<KCfg<1024, 32, 8, true, XCHG_SPLIT, 1, false, Radices<32, 32>>,
                       KCfg<1024, 32, 16, true, XCHG_SPLIT, 1, false, Radices<32, 32>>,
                       KCfg<1024, 16, 8, true, XCHG_FULL, 0, false, Radices<16, 16, 4>>,
                       // the second stage's 992 factors from LDS: FP32 SAR images, in whose
                       // two transforms a computed factor's rounding counts twice (error
                       // against FP64 over 1024 columns 3.77e-7, with computed factors
                       // 3.98e-7; 24.6 / 24.0 us)
                       KCfg<1024, 32, 8, true, XCHG_SPLIT, 3, false, Radices<32, 32>>,
                       KCfg<1024, 32, 16, true, XCHG_SPLIT, 3, false, Radices<32, 32>>>;
    // 8 range bins per strip: 229 against 256 us for 16 (which held one
    // Doppler bin per thread, too few for the column gather) on a 1024 x 16384
    // range-Doppler chain
    using Rcmc = KList<KCfg<1024, 16, 8, false, XCHG_SPLIT, 1, false, Radices<16, 16, 4>>,
                       KCfg<1024, 16, 4, false, XCHG_SPLIT, 1, false, Radices<16, 16, 4>>>;
    using RowsHalf = KList<KCfg<1024, 16, 4, false, XCHG_HALF, 1, false, Radices<16, 16, 4>>>;
    // (plain rows go by their batch, row_shape)
    // matched: one transform, one wave, per workgroup against four of each, SAR
    // 1024 x 1024 25.2 / 27.0 us, 4096 x 1024 50.2 / 51.2, range-Doppler 31.8 /
    // 32.8 and 74.8 / 76.7
    static constexpr int kRowDefault[2] = {1, 0};
    static constexpr int kRowMatched[2] = {4, 4};
};
template <>
struct Configs<2048> {
    using Rows = KList<KCfg<2048, 16, 2, false, XCHG_SPLIT, 1, false, Radices<16, 16, 8>>,
                       KCfg<2048, 16, 2, false, XCHG_FULL, 1, false, Radices<16, 16, 8>>,
                       KCfg<2048, 16, 2, false, XCHG_FULL, 1, true, Radices<16, 16, 8>>,
                       KCfg<2048, 16, 2, false, XCHG_FULL, 0, false, Radices<16, 16, 8>>,
                       KCfg<2048, 16, 1, false, XCHG_FULL, 1, false, Radices<16, 16, 8>>>;
    using Cols = KList<KCfg<2048, 16, 4, true, XCHG_SPLIT, 1, false, Radices<16, 16, 8>>,
                       KCfg<2048, 16, 8, true, XCHG_SPLIT, 1, false, Radices<16, 16, 8>>,
                       KCfg<2048, 16, 4, true, XCHG_FULL, 0, false, Radices<16, 16, 8>>,
                       // 64 points per thread: one exchange, whole lines with 16 columns
                       KCfg<2048, 64, 8, true, XCHG_SPLIT, 1, false, Radices<64, 32>>,
                       KCfg<2048, 64, 16, true, XCHG_SPLIT, 1, false, Radices<64, 32>>>;
    // 32 points per thread: 228 against 241 us (16 points, 8 range bins) and
    // 247 us (16 points, 4 range bins) for a 2048 x 8192 range-Doppler chain
    // with FP32 intermediates, 199 against 197 and 212 us with FP16
    using Rcmc = KList<KCfg<2048, 32, 8, false, XCHG_SPLIT, 1, false, Radices<16, 16, 8>>,
                       KCfg<2048, 16, 8, false, XCHG_SPLIT, 1, false, Radices<16, 16, 8>>>;
    using RowsHalf = KList<KCfg<2048, 16, 2, false, XCHG_HALF, 1, false, Radices<16, 16, 8>>>;
    // FP32: one transform per workgroup against two (88.7 / 91.2 us for 2^25
    // points, 25.6 / 25.9 for 2^23; FP16 50.8 / 51.7, but 16.2 / 14.4 for 2^23
    // and 187 / 183 for 2^27), matched too (SAR 4096 x 2048 81.6 / 84.1 us,
    // FP16 75.2 / 73.9; range-Doppler 111.5 / 114.3, FP16 98.2 / 97.6)
    static constexpr int kRowDefault[2] = {4, 0};
    static constexpr int kRowMatched[2] = {4, 0};
};
template <>
struct Configs<4096> {
    // measured in the hardware's block order: the hint cost about 2% on this
    // shape and gained 2-5% on the others (the default is now index 8, below)
    using Rows = KList<KCfg<4096, 16, 1, false, XCHG_FULL, 1, false, Radices<16, 16, 16>, false>,
                       KCfg<4096, 16, 1, false, XCHG_SPLIT, 1, false, Radices<16, 16, 16>>,
                       KCfg<4096, 16, 1, false, XCHG_FULL, 1, true, Radices<16, 16, 16>>,
                       KCfg<4096, 16, 1, false, XCHG_SPLIT, 1, true, Radices<16, 16, 16>>,
                       KCfg<4096, 16, 1, false, XCHG_FULL, 0, false, Radices<16, 16, 16>>,
                       KCfg<4096, 16, 1, false, XCHG_SPLIT, 0, false, Radices<16, 16, 16>>,
                       // every factor from the per-stage tables
                       KCfg<4096, 16, 1, false, XCHG_FULL, 2, false, Radices<16, 16, 16>, false>,
                       KCfg<4096, 16, 1, false, XCHG_SPLIT, 2, false, Radices<16, 16, 16>>,
                       // the complex exchange with streaming row stores
                       KCfg<4096, 16, 1, false, XCHG_FULL, 1, false, Radices<16, 16, 16>, true>,
                       // the second stage's 240 factors from LDS (twiddle mode 3)
                       KCfg<4096, 16, 1, false, XCHG_SPLIT, 3, false, Radices<16, 16, 16>>>;
    using Cols = KList<KCfg<4096, 32, 4, true, XCHG_SPLIT, 1, false, Radices<16, 16, 16>>,
                       KCfg<4096, 32, 4, true, XCHG_SPLIT, 0, false, Radices<16, 16, 16>>,
                       // (the second stage's factors from LDS: error against FP64
                       // 1.35e-7, with computed factors 1.51e-7)
                       KCfg<4096, 16, 4, true, XCHG_SPLIT, 3, false, Radices<16, 16, 16>>,
                       KCfg<4096, 32, 8, true, XCHG_SPLIT, 1, false, Radices<16, 16, 16>>,
                       KCfg<4096, 32, 8, true, XCHG_SPLIT, 2, false, Radices<16, 16, 16>>,
                       // two radix-64 stages, 64 points per thread: one exchange per
                       // transform instead of two, and fewer VALU instructions per
                       // point (87 against 93 for the matched pass)
                       KCfg<4096, 64, 8, true, XCHG_SPLIT, 1, false, Radices<64, 64>>,
                       KCfg<4096, 64, 4, true, XCHG_SPLIT, 1, false, Radices<64, 64>>>;
    // 8-column strips measured fastest for both column passes: 64-byte row
    // pieces against 32 (plain 82 vs 117 us, matched 88 vs 100 us per 4096^2
    // with 32 points per thread).  Radix 64, 8 columns, 30 interleaved
    // flushed samples per 4096^2 workload: plain 75.2 against 78.8 us (FP32)
    // and 53.8 against 55.0 (FP16); SAR chain 143.1 against 157.1 us (FP32
    // intermediate) and 131.3 against 135.7 (FP16).
    using Rcmc = KList<KCfg<4096, 32, 8, false, XCHG_SPLIT, 1, false, Radices<16, 16, 16>>,
                       KCfg<4096, 16, 4, false, XCHG_SPLIT, 1, false, Radices<16, 16, 16>>,
                       KCfg<4096, 32, 8, false, XCHG_SPLIT, 2, false, Radices<16, 16, 16>>>;
    using RowsHalf = KList<KCfg<4096, 16, 1, false, XCHG_HALF, 1, false, Radices<16, 16, 16>>>;
    // FP32 rows: with the rows' XCD groups, streaming stores win back to back
    // (6,108-6,171 against 6,015-6,027 GB/s, same process; flushed 6,120
    // against 6,298, where a call without them leaves its write-back for later)
    // FP16 rows: the second stage's factors from LDS, 27.8 against 29.9 us for
    // 2^24 points, 49.2 / 53.4 for 2^25 (smaller batches: row_shape)
    // matched rows: the same, SAR chain 145.0 against 148.0 us (FP16 123.0 /
    // 124.2), range-Doppler chain 200.6-201.1 / 199.9-200.7 (FP16 178.3 / 182.8)
    // matched columns (the SAR azimuth pass): bound by the 64-byte pieces of
    // the image rows (128 MiB strided reads alone take 34 us, writes 24 us);
    // the 4-column strips' 32-byte pieces cost more.  Image after image, on
    // inputs that no cache holds, an FP32 chain takes 146 us with 8 columns
    // and 152 with 4 (FP16 124 and 132); a single chain after a flush, where
    // the intermediate is still in the Infinity Cache, 141 and 135.
    static constexpr int kRowDefault[2] = {8, 9};
    static constexpr int kRowMatched[2] = {9, 9};
};
template <>
struct Configs<8192> {
    using Rows = KList<KCfg<8192, 16, 1, false, XCHG_SPLIT, 1, false, Radices<16, 16, 16, 2>>,
                       KCfg<8192, 32, 1, false, XCHG_FULL, 1, false, Radices<32, 16, 16>>,
                       KCfg<8192, 16, 1, false, XCHG_SPLIT, 1, true, Radices<16, 16, 16, 2>>,
                       KCfg<8192, 16, 1, false, XCHG_FULL, 0, false, Radices<16, 16, 16, 2>>,
                       KCfg<8192, 32, 1, false, XCHG_SPLIT, 1, false, Radices<32, 16, 16>>,
                       KCfg<8192, 32, 1, false, XCHG_SPLIT, 2, false, Radices<32, 16, 16>>,
                       KCfg<8192, 16, 1, false, XCHG_SPLIT, 2, false, Radices<16, 16, 16, 2>>,
                       // the second stage's 240 factors from LDS (twiddle mode 3)
                       KCfg<8192, 16, 1, false, XCHG_SPLIT, 3, false, Radices<16, 16, 16, 2>>,
                       // three stages with the second one's 480 factors from LDS
                       KCfg<8192, 32, 1, false, XCHG_SPLIT, 3, false, Radices<32, 16, 16>>>;
    // three stages, the second one's 240 factors from LDS (error against FP64
    // 1.43e-7 in FP32, with squared powers in the layers 1.61e-7; 4096 columns
    // in place 219 / 227 us); 4 columns hold a CU (64 or 32 points per
    // thread), 2 columns half
    using Cols = KList<KCfg<8192, 64, 4, true, XCHG_SPLIT, 3, false, Radices<16, 16, 32>>,
                       KCfg<8192, 32, 4, true, XCHG_SPLIT, 3, false, Radices<16, 16, 32>>,
                       KCfg<8192, 32, 2, true, XCHG_SPLIT, 3, false, Radices<16, 16, 32>>,
                       KCfg<8192, 32, 2, true, XCHG_SPLIT, 0, false, Radices<16, 16, 16, 2>>>;
    using Rcmc = KList<KCfg<8192, 32, 4, false, XCHG_SPLIT, 1, false, Radices<16, 16, 16, 2>>,
                       KCfg<8192, 16, 2, false, XCHG_SPLIT, 1, false, Radices<16, 16, 16, 2>>>;
    // binary16 exchange: three stages 5.5 TB/s, four stages 4.8
    using RowsHalf = KList<KCfg<8192, 32, 1, false, XCHG_HALF, 1, false, Radices<32, 16, 16>>,
                           KCfg<8192, 16, 1, false, XCHG_HALF, 1, false, Radices<16, 16, 16, 2>>>;
    // FP16: 32 points per thread in three stages, 5.7 vs 4.9 TB/s.  FP32:
    // the second stage's factors from LDS, 5,740 against 5,607 GB/s flushed
    // and 5,700-5,731 against 5,318-5,604 back to back (same box, one run)
    static constexpr int kRowDefault[2] = {7, 4};
    // matched: three stages too (SAR 1024 x 8192 79.2 against 83.7 us and, with
    // an FP16 intermediate, 69.1 / 74.0; 2048 x 8192 155 / 154 and 132.5 /
    // 138.3; range-Doppler 102.9 / 110.3 and 90.6 / 95.1)
    static constexpr int kRowMatched[2] = {4, 4};
};
template <>
struct Configs<16384> {
    using Rows = KList<KCfg<16384, 16, 1, false, XCHG_SPLIT, 1, false, Radices<16, 16, 16, 4>>,
                       KCfg<16384, 32, 1, false, XCHG_SPLIT, 1, false, Radices<16, 16, 16, 4>>,
                       KCfg<16384, 32, 1, false, XCHG_SPLIT, 1, true, Radices<16, 16, 16, 4>>,
                       KCfg<16384, 32, 1, false, XCHG_SPLIT, 0, false, Radices<16, 16, 16, 4>>,
                       KCfg<16384, 32, 1, false, XCHG_SPLIT, 1, false, Radices<32, 16, 32>>,
                       KCfg<16384, 32, 1, false, XCHG_SPLIT, 2, false, Radices<32, 16, 32>>,
                       // the second stage's 240 factors from LDS (twiddle mode 3)
                       KCfg<16384, 16, 1, false, XCHG_SPLIT, 3, false, Radices<16, 16, 16, 4>>,
                       // three stages with the second one's 480 factors from LDS
                       KCfg<16384, 32, 1, false, XCHG_SPLIT, 3, false, Radices<32, 16, 32>>>;
    using Cols = KList<KCfg<16384, 32, 2, true, XCHG_SPLIT, 1, false, Radices<32, 16, 32>>,
                       KCfg<16384, 32, 1, true, XCHG_SPLIT, 1, false, Radices<32, 16, 32>>,
                       KCfg<16384, 32, 1, true, XCHG_SPLIT, 0, false, Radices<16, 16, 16, 4>>>;
    // three stages (32 x 16 x 32) against four: one exchange and one twiddle
    // pass fewer; measured 5.5 vs 5.3 TB/s (FP32) and 4.9 vs 3.8 TB/s (FP16).
    // FP32: four stages with the second stage's factors from LDS beat both,
    // 5,800-5,816 against 5,660-5,693 GB/s flushed and 5,637-5,828 against
    // 5,128-5,722 back to back (two boxes, same process each)
    static constexpr int kRowDefault[2] = {6, 4};
    using Rcmc = KList<KCfg<16384, 32, 2, false, XCHG_SPLIT, 1, false, Radices<16, 16, 16, 4>>,
                       KCfg<16384, 16, 1, false, XCHG_SPLIT, 1, false, Radices<16, 16, 16, 4>>>;
    // binary16 exchange: three stages fastest (4.8 TB/s), then 32 points per
    // thread in four stages (4.3), then 16 (4.0)
    using RowsHalf = KList<KCfg<16384, 32, 1, false, XCHG_HALF, 1, false, Radices<32, 16, 32>>,
                           KCfg<16384, 32, 1, false, XCHG_HALF, 1, false, Radices<16, 16, 16, 4>>,
                           KCfg<16384, 16, 1, false, XCHG_HALF, 1, false, Radices<16, 16, 16, 4>>>;
    static constexpr int kRowMatched[2] = {4, 4};
};

// The row shape of a plain transform (index into Rows) by its storage and
// batch.  Times in us, back to back on inputs that no cache holds.
//   1024   one wave, one transform per workgroup (no barrier waits) against
//          four of each: FP32 6.5 / 7.4 for 1500 transforms, 8.7 / 8.9 for
//          2500, but 12.8 / 11.8 for 4096, 25.9 / 25.4 for 8192, 57.9 / 56.6 for
//          20000 (87.0 / 89.2 for 32768, 351 / 347 for 131072); FP16 5.7 / 6.2
//          for 2048, 7.9 / 8.2 for 4096, 11.4 / 9.5 for 5000, 15.8 / 14.1 for
//          8192, 21.9 / 22.5 for 12288, 48.4 / 50.4 for 32768
//   2048   FP16, up to 511: one transform per workgroup instead of two (64
//          transforms, one flushed call, 7.3 against 8.1 us)
//   4096   FP16, up to 2048: every factor computed, 5.3 against 5.6 for 300
//          transforms (filling the LDS table is not repaid), 6.2 / 6.6 for 512,
//          8.2 / 8.5 for 800, level from 1024 to 2048, 29.9 / 27.8 for 4096
//   8192   FP32, up to 2^25 points: three stages of 32 points per thread, 26.1
//          against 28.5 for 1024 transforms, 93.5 / 96.1 for 4096 (7.1 / 7.0
//          for one); beyond, memory-bound, the higher occupancy wins (8192
//          transforms 182.3 / 183.4).  Both shapes read the second stage's
//          factors from LDS: error against FP64 1.40e-7 and 1.41e-7, where
//          squared powers gave 1.59e-7.
//   16384  FP32, up to 127, half of the CUs: the same (10.0 against 11.1 for
//          one transform, 12.7 / 13.3 for 100, but 14.3 / 14.1 for 128, 20.6 /
//          18.9 for 256, 31.0 / 29.7 for 512, 59.3 / 54.2 for 1024; error
//          1.49e-7 and 1.50e-7, with squared powers 1.69e-7)
template <int N>
constexpr int row_shape(int half, long long batch) {
    if (N == 1024) return half ? (batch <= 4096 || batch >= 12288 ? 4 : 0) : (batch <= 3072 ? 4 : 1);
    if (N == 2048 && half && batch <= 511) return 4;
    if (N == 4096 && half && batch <= 2048) return 1;
    if (N == 8192 && !half && batch <= 4096) return 8;
    if (N == 16384 && !half && batch <= 127) return 7;
    return Configs<N>::kRowDefault[half];
}

// The column shape of a pass over `columns` columns in all (every problem of
// the grid counted), `row` of them side by side, by what the pass does:
//   plain    the transform (and the last pass of the split forms);
//   twiddled the four-step epilogues (at most 32 points per thread);
//   scaled   the range-Doppler chain's azimuth pass, written transposed;
//   matched  the SAR azimuth pass (two transforms).
// half: FP16 storage on either side.  Wider strips read and write longer
// pieces of each row (whole 128-byte lines at 16 FP32 columns) and pay once
// there are strips enough for the 256 CUs; with fewer columns narrow strips
// keep more CUs busy.  Times in us, narrower against wider shape, on inputs
// that no cache holds:
//   256   both passes of 2^16 points (16 / 32 columns a strip): 16384 columns
//         29.7 / 30.8, 32768 52.5 / 53.2 (FP16 34.4 / 33.1), 65536 100.4 /
//         97.0 (FP16 63.7 / 59.4)
//   512   both passes of 2^18 points (16 / 32): 16384 columns 54.6 / 54.8 (FP16
//         36.6 / 38.1), 32768 97.7 / 98.1 (FP16 68.3 / 64.3), 49664 145.6 /
//         151.6 (FP16 96.7 / 99.2), 65536 206.8 / 198.6 (FP16 125.3 / 122.7)
//   1024  (8 / 16) 3000 columns 15.4 / 14.9, 4096 18.1 / 15.0 but 4100 17.5 /
//         20.4, 6000 25.1 / 26.3 (FP16 18.0 / 16.6), 8192 39.0 / 29.2, 16384
//         82.9 / 70.5 (FP16 50.2 / 41.4); SAR over 4096 columns 42.0 / 43.8,
//         8192 79.4 / 76.6 (FP16 69.3 / 69.2), 16384 163 / 152 (135 / 131);
//         range-Doppler over 8192 104.0 / 102.8 (FP16 90.7 / 90.2)
//   2048  (4 and 8 columns of 16 points per thread, 8 and 16 of 64) 1000
//         columns 13.8, 14.7, 15.9, 21.1; 2048 24.4, 18.4, 19.3, 23.2; 4096
//         65.5, 44.2, 39.3, 28.7 (FP16 29.3, 24.8, 24.0, 21.4); 8192 145, 104,
//         83.9, 58.4 (FP16 82.3, 68.2, 51.7, 48.3); 16384 358, 235, 179, 158
//         (FP16 191, 166, 106, 87.8); SAR over 1024 31.9, 35.9, 39.2, 44.8;
//         4096 93.4, 77.6, 73.8, 78.9 (FP16 86.5, 73.3, 67.8, 71.5); 8192 208,
//         164, 155, 159; range-Doppler over 2048 61.4, 62.3, 64.5, 68.4; 4096
//         102.8, 101.0, 103.0, 107.4 (FP16 98.5, 95.7, 95.4, 96.5); 8192 216,
//         209, 208, 213 (FP16 176, 175, 177, 184)
//         The second pass of 2^22 points, FP32, in rows of 2048 columns: 8
//         columns of 16 points against 16 of 64, whole transforms: 3 of them
//         89.7 / 99.9, 8 236 / 248, 16 463 / 463, 32 904 / 892
//   4096  (4 columns with 1024 threads / 8 of 64 points) 250 columns 20.0 /
//         25.5, 1000 22.8 / 24.7, 1025 30.9 / 30.5, 1536 48.9 / 33.6; SAR over
//         1024 columns 49.0 / 55.5, over 2048 95.1 / 80.6; range-Doppler (4 / 8
//         columns of 64 points) over 1024 74.7 / 80.1, over 4096 201 / 209 (FP16
//         182 / 182)
//   8192  in place (2 / 4): 100 columns 23.2 / 25.6, 512 33.3 / 40.2 (256
//         strips of 2), 700 50.6 / 38.9, 1000 56.1 / 41.4 (43.5 with 64
//         points), 4096 290 / 237 (214); SAR over 1024 98.6 / 92.8 (93.0; FP16
//         94.2 / 85.9, 90.1), 2048 235 / 197 (178); range-Doppler over 4096 630
//         / 649, over 2048 244 / 245, FP16 216 / 210
//   16384 in place (1 / 2): 100 columns 42.7 / 45.8, 200 47.8 / 46.4, 1000 208 /
//         116; SAR over 1024 265 / 199, range-Doppler 284 / 274
enum { COLS_PLAIN, COLS_TWIDDLED, COLS_SCALED, COLS_MATCHED };
template <int N>
constexpr int column_shape(int use, int half, long long columns, long long row) {
    if (N == 256) return columns >= 32768 ? 1 : 0;
    if (N == 512) return columns >= (half ? 32768 : 65536) ? 1 : 0;
    if (N == 1024) return (use == COLS_MATCHED && !half ? 3 : 0) + (columns >= 8192 ? 1 : 0);
    if (N == 2048) {
        if (columns < 2048 || (use == COLS_SCALED && columns < 4096)) return 0;
        if (columns < 4096 || use == COLS_TWIDDLED) return 1;
        if (use == COLS_PLAIN) return !half && row < 4096 && columns < 32768 ? 1 : 4;
        return use == COLS_MATCHED || half || columns >= 8192 ? 3 : 1;
    }
    if (N == 4096) {
        if (use == COLS_SCALED) return 6;
        return columns <= 1024 ? 2 : 5;
    }
    if (N == 8192) {
        if (use == COLS_SCALED) return half ? 1 : 2;
        if (use == COLS_PLAIN && columns <= 512) return 2;
        return half || (use == COLS_PLAIN && columns <= 1024) ? 1 : 0;
    }
    if (N == 16384) return use == COLS_PLAIN && columns < 256 ? 1 : 0;
    return 0;
}

template <class L>
struct KListSize;
template <class... Ks>
struct KListSize<KList<Ks...>> {
    static constexpr int value = sizeof...(Ks);
};

// The four-step epilogues hold at most 32 points per thread and run on columns
// of at most 2048 points: the leading shapes of each list that fit (the
// shapes a plan may force for its twiddled passes).
constexpr int kMaxTwiddledN = 2048;
template <int N, class... Ks>
constexpr int twiddled_shapes(KList<Ks...>) {
    constexpr int points[] = {Ks::P...};
    int k = 0;
    while (N <= kMaxTwiddledN && k < (int)sizeof...(Ks) && points[k] <= 32) ++k;
    return k;
}
// column_shape stays among them on both sides of every power of two
template <int N>
constexpr bool twiddled_shapes_fit() {
    if (N > kMaxTwiddledN) return true;
    const int most = twiddled_shapes<N>(typename Configs<N>::Cols{});
    for (int half = 0; half < 2; ++half)
        for (int l = 0; l <= 40; ++l)
            for (int d = -1; d <= 1; ++d)
                for (long long row : {(1LL << l) + d, 64LL})
                    if (column_shape<N>(COLS_TWIDDLED, half, (1LL << l) + d, row) >= most) return false;
    return true;
}

// Calls f(K{}) for the idx-th entry of the list.
template <class F, class K, class... Ks>
hipError_t with_variant(int idx, KList<K, Ks...>, F &&f) {
    if (idx == 0) return f(K{});
    if constexpr (sizeof...(Ks) > 0) {
        return with_variant(idx - 1, KList<Ks...>{}, f);
    } else {
        return hipErrorInvalidValue;
    }
}

// Supported (layout, storage, direction, epilogue) combinations:
//   plain FFT:  rows or columns, input storage == output storage, either direction;
//   matched:    forward, multiply by conj(spec) (spec carries 1/N), inverse:
//               rows read FP32 and write FP32 or FP16 (range compression);
//               columns read FP32 or FP16 and write FP32 (azimuth compression);
//   scaled:     columns, forward, input storage == output storage (the azimuth
//               FFT of the full range-Doppler chain);
//   twiddled:   columns of at most 2048 points, either direction, input
//               storage == output storage, written as rows (first pass of a
//               four-step transform), or written in place with the factor
//               keyed by the second grid axis (middle pass of a three-pass
//               transform); matched with such factors at 128 points;
//   RCMC:       the Rcmc list (row-mapped, several transforms per workgroup),
//               inverse, read FP32 or FP16, write FP32 columns (migration
//               correction, azimuth filter and azimuth inverse FFT).
template <class K>
hipError_t dispatch_cfg_full(int in_st, int out_st, int inv, int epi, const void *in, void *out, const float2 *tw,
                             const float2 *spec, const KArgs &a, hipStream_t s) {
    if (epi == EPI_NONE) {
        if (in_st != out_st) return hipErrorInvalidValue;
        if (in_st == 0)
            return inv ? launch_one<K, 0, 0, true, EPI_NONE>(in, out, tw, spec, a, s)
                       : launch_one<K, 0, 0, false, EPI_NONE>(in, out, tw, spec, a, s);
        return inv ? launch_one<K, 1, 1, true, EPI_NONE>(in, out, tw, spec, a, s)
                   : launch_one<K, 1, 1, false, EPI_NONE>(in, out, tw, spec, a, s);
    }
    if (epi == EPI_SCALE) {
        if constexpr (K::COLS && !K::PERSIST) {
            if (inv || in_st != out_st) return hipErrorInvalidValue;
            return in_st == 0 ? launch_one<K, 0, 0, false, EPI_SCALE>(in, out, tw, spec, a, s)
                              : launch_one<K, 1, 1, false, EPI_SCALE>(in, out, tw, spec, a, s);
        } else {
            return hipErrorInvalidValue;
        }
    }
    if (epi == EPI_TWIDDLE) {
        if constexpr (K::COLS && !K::PERSIST && K::P <= 32 && K::N <= kMaxTwiddledN) {
            if (in_st != out_st) return hipErrorInvalidValue;
            if (in_st == 0)
                return inv ? launch_one<K, 0, 0, true, EPI_TWIDDLE>(in, out, tw, spec, a, s)
                           : launch_one<K, 0, 0, false, EPI_TWIDDLE>(in, out, tw, spec, a, s);
            return inv ? launch_one<K, 1, 1, true, EPI_TWIDDLE>(in, out, tw, spec, a, s)
                       : launch_one<K, 1, 1, false, EPI_TWIDDLE>(in, out, tw, spec, a, s);
        } else {
            return hipErrorInvalidValue;
        }
    }
    if (epi == EPI_TWIDDLE_Y) {
        if constexpr (K::COLS && !K::PERSIST && K::P <= 32 && K::N <= kMaxTwiddledN) {
            if (in_st != out_st) return hipErrorInvalidValue;
            if (in_st == 0)
                return inv ? launch_one<K, 0, 0, true, EPI_TWIDDLE_Y>(in, out, tw, spec, a, s)
                           : launch_one<K, 0, 0, false, EPI_TWIDDLE_Y>(in, out, tw, spec, a, s);
            return inv ? launch_one<K, 1, 1, true, EPI_TWIDDLE_Y>(in, out, tw, spec, a, s)
                       : launch_one<K, 1, 1, false, EPI_TWIDDLE_Y>(in, out, tw, spec, a, s);
        } else {
            return hipErrorInvalidValue;
        }
    }
    if (epi == EPI_MATCHED_Y) {
        if constexpr (K::COLS && !K::PERSIST && K::N == 128) {  // the split azimuth pass: 16384 = 128 x 128
            if (inv || in_st != 0 || out_st != 0) return hipErrorInvalidValue;
            return launch_one<K, 0, 0, false, EPI_MATCHED_Y>(in, out, tw, spec, a, s);
        } else {
            return hipErrorInvalidValue;
        }
    }
    if (epi == EPI_RCMC) return hipErrorInvalidValue;  // only through dispatch_rcmc
    if (epi != EPI_MATCHED || inv) return hipErrorInvalidValue;
    if constexpr (!K::COLS) {
        if (in_st != 0) return hipErrorInvalidValue;
        return out_st == 0 ? launch_one<K, 0, 0, false, EPI_MATCHED>(in, out, tw, spec, a, s)
                           : launch_one<K, 0, 1, false, EPI_MATCHED>(in, out, tw, spec, a, s);
    } else {
        if (out_st != 0) return hipErrorInvalidValue;
        return in_st == 0 ? launch_one<K, 0, 0, false, EPI_MATCHED>(in, out, tw, spec, a, s)
                          : launch_one<K, 1, 0, false, EPI_MATCHED>(in, out, tw, spec, a, s);
    }
}

template <class K>
hipError_t dispatch_cfg(int in_st, int out_st, int inv, int epi, const void *in, void *out, const float2 *tw,
                        const float2 *spec, const KArgs &a, hipStream_t s) {
    if constexpr (K::XCHG == XCHG_LANE) {
        // the cross-lane exchange: plain row transforms, either storage
        if (epi != EPI_NONE || in_st != out_st) return hipErrorInvalidValue;
        if (in_st == 0)
            return inv ? launch_one<K, 0, 0, true, EPI_NONE>(in, out, tw, spec, a, s)
                       : launch_one<K, 0, 0, false, EPI_NONE>(in, out, tw, spec, a, s);
        return inv ? launch_one<K, 1, 1, true, EPI_NONE>(in, out, tw, spec, a, s)
                   : launch_one<K, 1, 1, false, EPI_NONE>(in, out, tw, spec, a, s);
    } else if constexpr (K::XCHG == XCHG_HALF) {
        // the binary16 exchange: FP16 storage, plain transforms only
        if (epi != EPI_NONE || in_st != 1 || out_st != 1) return hipErrorInvalidValue;
        return inv ? launch_one<K, 1, 1, true, EPI_NONE>(in, out, tw, spec, a, s)
                   : launch_one<K, 1, 1, false, EPI_NONE>(in, out, tw, spec, a, s);
    } else {
        return dispatch_cfg_full<K>(in_st, out_st, inv, epi, in, out, tw, spec, a, s);
    }
}

template <class K>
hipError_t dispatch_rcmc(int in_st, int out_st, int inv, const void *in, void *out, const float2 *tw,
                         const float2 *spec, const KArgs &a, hipStream_t s) {
    if (!inv || out_st != 0) return hipErrorInvalidValue;
    return in_st == 0 ? launch_one<K, 0, 0, true, EPI_RCMC>(in, out, tw, spec, a, s)
                      : launch_one<K, 1, 0, true, EPI_RCMC>(in, out, tw, spec, a, s);
}

template <int N>
hipError_t dispatch(int variant, int layout, int in_st, int out_st, int inv, int epi, const void *in, void *out,
                    const float2 *tw, const float2 *spec, const KArgs &a, hipStream_t s) {
    auto f = [&](auto k) { return dispatch_cfg<decltype(k)>(in_st, out_st, inv, epi, in, out, tw, spec, a, s); };
    if (layout == LAYOUT_ROWS_HALF) {
        if constexpr (N >= 1024) {
            return with_variant(variant >= 0 ? variant : 0, typename Configs<N>::RowsHalf{}, f);
        } else {
            return hipErrorInvalidValue;
        }
    }
    if (layout == LAYOUT_RCMC) {
        if constexpr (N >= 1024) {
            if (epi != EPI_RCMC) return hipErrorInvalidValue;
            auto g = [&](auto k) { return dispatch_rcmc<decltype(k)>(in_st, out_st, inv, in, out, tw, spec, a, s); };
            return with_variant(variant >= 0 ? variant : 0, typename Configs<N>::Rcmc{}, g);
        } else {
            return hipErrorInvalidValue;
        }
    }
    const int half = (in_st | out_st) != 0;  // any FP16 storage involved
    if (layout == LAYOUT_ROWS) {
        const int v = variant >= 0         ? variant
                      : epi == EPI_MATCHED ? Configs<N>::kRowMatched[half]
                                           : row_shape<N>(half, a.batch);
        return with_variant(v, typename Configs<N>::Rows{}, f);
    }
    using Cols = typename Configs<N>::Cols;
    static_assert(twiddled_shapes_fit<N>(), "the four-step epilogues hold at most 32 points per thread");
    const long long columns = a.batch * (a.outer > 1 ? a.outer : 1) * (a.outer2 > 1 ? a.outer2 : 1);
    const int use = epi == EPI_NONE      ? COLS_PLAIN
                    : epi == EPI_SCALE   ? COLS_SCALED
                    : epi == EPI_MATCHED ? COLS_MATCHED
                                         : COLS_TWIDDLED;
    const int v = variant >= 0 ? variant : column_shape<N>(use, half, columns, a.batch);
    return with_variant(v, Cols{}, f);
}

template <int N>
int variant_count(int layout) {
    return layout == LAYOUT_ROWS            ? KListSize<typename Configs<N>::Rows>::value
           : layout == LAYOUT_COLS          ? KListSize<typename Configs<N>::Cols>::value
           : layout == LAYOUT_COLS_TWIDDLED ? twiddled_shapes<N>(typename Configs<N>::Cols{})
           : layout == LAYOUT_RCMC          ? KListSize<typename Configs<N>::Rcmc>::value
                                            : KListSize<typename Configs<N>::RowsHalf>::value;
}

}  // namespace mi355fft
