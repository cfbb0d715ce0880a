// ns_size_plans.hpp -- line plans of the passes of every other grid size up to 512
// (FP32) and of the FP64 fields.
//
// The kernels are those of ns_fast.hpp; a size's x-forward pass is one kernel with
// the stage operation as an argument (OP_ANY) instead of one kernel per stage, so
// that a size costs nine kernels.  Each SizePlan names the plans (threads a line,
// inverse radices, forward radices) of the x, y, z and adjoint z passes and the
// lines per block of the two z passes.
//
// How a plan was chosen: of all radix lists and thread counts that fit a tile of 128-byte
// rows in 512 threads (y passes: 1024), the one of least estimated time,
// instructions of a thread (butterflies, twiddles, LDS exchanges, idle butterflies
// included) times wavefronts per line over 1 - 1/(occupancy) with registers of about
// 70 + 11.5 EPT (x of FP32), 90 + 24 EPT (x of FP64), 36 + 5 w EPT (y) and 40 + 13 w EPT (z), w = 1 (FP32) or 2 (FP64);
// up to N = 80, where a launch does not fill the chip, the one with the fewest
// instructions a thread.  z passes keep a line inside one wavefront (4, 8, 16, 32
// or 64 threads), and the lines per block divide N^2.  The x plans were then timed
// against up to five others, the two cheapest estimates in each of five ranges of threads
// a line (to 64 threads in FP32, 128 in FP64; EPT at most 12 and 10), PS-RK2 random and
// RK4 steps and the gradient, and replaced where the steps were 1.5% faster or more: the x
// passes of FP32 want more threads a line and 5 to 10 registers a transform than the
// estimate gave (their x-forward kernel holds operands for every stage).  From N = 48 on the
// y and z plans were timed against three others and replaced where their pass was 4% faster.  Random steps, us:
// 100^3 10 10 over 12 to 5 4 5 over 25 131 -> 114, 150^3 3 5 10 over 16 to 6 5 5
// over 32 approx 285 -> 244, 288^3 2 12 12 over 24 to 6 6 8 over 48 1690 -> 1530, 500^3
// 5 10 10 over 28 to 10 5 10 over 50 13.4 -> 10.3 ms; FP64 384^3 8 6 8 to 6 8 8 over 64 6.40 ->
// 6.07 ms; y passes, us: 400^3 4 10 10 over 40 to 32 threads 16 5 5 956 -> 706, FP64 360^3 10 4
// 9 over 48 to 10 6 6 over 60 1299 -> 953; z passes: 200^3 5 4 10 over 32 to 8 5 5 over 16 92 ->
// 72, FP64 240^3 8 5 6 to 3 4 4 5 over 64 276 -> 217.
//
// Against the size-generic passes these sizes ran before (LDS Stockham stages over a
// runtime plan: an LDS round trip and two barriers a radix, index divisions, shift
// factors evaluated per point): five approx steps at 150^3 FP32 4.71 -> 1.24 ms, two
// RK4 steps at 128^3 FP64 1.70 -> 0.68 ms, ten exact steps at 32^3 FP64 2.43 -> 1.00 ms.
#pragma once

#include "ns_fast.hpp"

namespace ns {

template <typename T, int N>
struct SizePlan;
template <> struct SizePlan<float, 16> {
  using X = LinePlan<16, 4, Radices<4, 4>, Radices<4, 4>>;
  using Y = LinePlan<16, 4, Radices<4, 4>, Radices<4, 4>>;
  using Z = LinePlan<16, 8, Radices<4, 4>, Radices<4, 4>>;
  using ZA = LinePlan<16, 8, Radices<4, 4>, Radices<4, 4>>;
  static constexpr int PZ = 32, PZA = 32;
};
template <> struct SizePlan<float, 18> {
  using X = LinePlan<18, 6, Radices<6, 3>, Radices<3, 6>>;
  using Y = LinePlan<18, 8, Radices<6, 3>, Radices<3, 6>>;
  using Z = LinePlan<18, 16, Radices<6, 3>, Radices<3, 6>>;
  using ZA = LinePlan<18, 16, Radices<6, 3>, Radices<3, 6>>;
  static constexpr int PZ = 4, PZA = 4;
};
template <> struct SizePlan<float, 20> {
  using X = LinePlan<20, 5, Radices<5, 4>, Radices<4, 5>>;
  using Y = LinePlan<20, 8, Radices<5, 4>, Radices<4, 5>>;
  using Z = LinePlan<20, 8, Radices<5, 4>, Radices<4, 5>>;
  using ZA = LinePlan<20, 8, Radices<5, 4>, Radices<4, 5>>;
  static constexpr int PZ = 16, PZA = 16;
};
template <> struct SizePlan<float, 24> {
  using X = LinePlan<24, 16, Radices<4, 2, 3>, Radices<3, 2, 4>>;
  using Y = LinePlan<24, 8, Radices<6, 4>, Radices<4, 6>>;
  using Z = LinePlan<24, 16, Radices<4, 2, 3>, Radices<3, 2, 4>>;
  using ZA = LinePlan<24, 16, Radices<4, 2, 3>, Radices<3, 2, 4>>;
  static constexpr int PZ = 16, PZA = 16;
};
template <> struct SizePlan<float, 30> {
  using X = LinePlan<30, 15, Radices<5, 2, 3>, Radices<3, 2, 5>>;
  using Y = LinePlan<30, 8, Radices<6, 5>, Radices<5, 6>>;
  using Z = LinePlan<30, 16, Radices<5, 2, 3>, Radices<3, 2, 5>>;
  using ZA = LinePlan<30, 16, Radices<5, 2, 3>, Radices<3, 2, 5>>;
  static constexpr int PZ = 4, PZA = 4;
};
template <> struct SizePlan<float, 32> {
  using X = LinePlan<32, 16, Radices<4, 2, 4>, Radices<4, 2, 4>>;
  using Y = LinePlan<32, 16, Radices<4, 2, 4>, Radices<4, 2, 4>>;
  using Z = LinePlan<32, 16, Radices<4, 2, 4>, Radices<4, 2, 4>>;
  using ZA = LinePlan<32, 16, Radices<4, 2, 4>, Radices<4, 2, 4>>;
  static constexpr int PZ = 16, PZA = 16;
};
template <> struct SizePlan<float, 36> {
  using X = LinePlan<36, 12, Radices<3, 3, 4>, Radices<4, 3, 3>>;
  using Y = LinePlan<36, 12, Radices<4, 3, 3>, Radices<3, 3, 4>>;
  using Z = LinePlan<36, 16, Radices<4, 3, 3>, Radices<3, 3, 4>>;
  using ZA = LinePlan<36, 16, Radices<4, 3, 3>, Radices<3, 3, 4>>;
  static constexpr int PZ = 16, PZA = 16;
};
template <> struct SizePlan<float, 40> {
  using X = LinePlan<40, 20, Radices<4, 2, 5>, Radices<5, 2, 4>>;
  using Y = LinePlan<40, 20, Radices<5, 2, 4>, Radices<4, 2, 5>>;
  using Z = LinePlan<40, 32, Radices<5, 2, 4>, Radices<4, 2, 5>>;
  using ZA = LinePlan<40, 32, Radices<5, 2, 4>, Radices<4, 2, 5>>;
  static constexpr int PZ = 8, PZA = 8;
};
template <> struct SizePlan<float, 48> {
  using X = LinePlan<48, 16, Radices<4, 3, 4>, Radices<4, 3, 4>>;
  using Y = LinePlan<48, 16, Radices<4, 3, 4>, Radices<4, 3, 4>>;
  using Z = LinePlan<48, 16, Radices<4, 3, 4>, Radices<4, 3, 4>>;
  using ZA = LinePlan<48, 16, Radices<4, 3, 4>, Radices<4, 3, 4>>;
  static constexpr int PZ = 16, PZA = 16;
};
template <> struct SizePlan<float, 50> {
  using X = LinePlan<50, 28, Radices<5, 2, 5>, Radices<5, 2, 5>>;
  using Y = LinePlan<50, 28, Radices<5, 2, 5>, Radices<5, 2, 5>>;
  using Z = LinePlan<50, 32, Radices<5, 2, 5>, Radices<5, 2, 5>>;
  using ZA = LinePlan<50, 32, Radices<5, 2, 5>, Radices<5, 2, 5>>;
  static constexpr int PZ = 4, PZA = 4;
};
template <> struct SizePlan<float, 54> {
  using X = LinePlan<54, 18, Radices<6, 3, 3>, Radices<3, 3, 6>>;
  using Y = LinePlan<54, 20, Radices<6, 3, 3>, Radices<3, 3, 6>>;
  using Z = LinePlan<54, 32, Radices<3, 2, 3, 3>, Radices<3, 3, 2, 3>>;
  using ZA = LinePlan<54, 32, Radices<6, 3, 3>, Radices<3, 3, 6>>;
  static constexpr int PZ = 2, PZA = 4;
};
template <> struct SizePlan<float, 60> {
  using X = LinePlan<60, 20, Radices<5, 3, 4>, Radices<4, 3, 5>>;
  using Y = LinePlan<60, 20, Radices<5, 3, 4>, Radices<4, 3, 5>>;
  using Z = LinePlan<60, 32, Radices<5, 3, 4>, Radices<4, 3, 5>>;
  using ZA = LinePlan<60, 32, Radices<5, 3, 4>, Radices<4, 3, 5>>;
  static constexpr int PZ = 8, PZA = 8;
};
template <> struct SizePlan<float, 72> {
  using X = LinePlan<72, 36, Radices<4, 2, 3, 3>, Radices<3, 3, 2, 4>>;
  using Y = LinePlan<72, 24, Radices<6, 3, 4>, Radices<4, 3, 6>>;
  using Z = LinePlan<72, 32, Radices<6, 3, 4>, Radices<4, 3, 6>>;
  using ZA = LinePlan<72, 64, Radices<4, 2, 3, 3>, Radices<3, 3, 2, 4>>;
  static constexpr int PZ = 2, PZA = 4;
};
template <> struct SizePlan<float, 80> {
  using X = LinePlan<80, 20, Radices<5, 4, 4>, Radices<4, 4, 5>>;
  using Y = LinePlan<80, 20, Radices<5, 4, 4>, Radices<4, 4, 5>>;
  using Z = LinePlan<80, 32, Radices<5, 4, 4>, Radices<4, 4, 5>>;
  using ZA = LinePlan<80, 32, Radices<5, 4, 4>, Radices<4, 4, 5>>;
  static constexpr int PZ = 8, PZA = 8;
};
template <> struct SizePlan<float, 90> {
  using X = LinePlan<90, 30, Radices<6, 3, 5>, Radices<5, 3, 6>>;
  using Y = LinePlan<90, 12, Radices<10, 9>, Radices<9, 10>>;
  using Z = LinePlan<90, 16, Radices<10, 9>, Radices<9, 10>>;
  using ZA = LinePlan<90, 16, Radices<10, 9>, Radices<9, 10>>;
  static constexpr int PZ = 4, PZA = 4;
};
template <> struct SizePlan<float, 96> {
  using X = LinePlan<96, 48, Radices<4, 2, 3, 4>, Radices<4, 3, 2, 4>>;
  using Y = LinePlan<96, 12, Radices<12, 8>, Radices<8, 12>>;
  using Z = LinePlan<96, 16, Radices<8, 2, 6>, Radices<6, 2, 8>>;
  using ZA = LinePlan<96, 16, Radices<8, 2, 6>, Radices<6, 2, 8>>;
  static constexpr int PZ = 16, PZA = 16;
};
template <> struct SizePlan<float, 100> {
  using X = LinePlan<100, 25, Radices<5, 4, 5>, Radices<5, 4, 5>>;
  using Y = LinePlan<100, 12, Radices<10, 10>, Radices<10, 10>>;
  using Z = LinePlan<100, 32, Radices<5, 4, 5>, Radices<5, 4, 5>>;
  using ZA = LinePlan<100, 16, Radices<10, 10>, Radices<10, 10>>;
  static constexpr int PZ = 2, PZA = 16;
};
template <> struct SizePlan<float, 108> {
  using X = LinePlan<108, 32, Radices<3, 6, 6>, Radices<6, 6, 3>>;
  using Y = LinePlan<108, 12, Radices<12, 9>, Radices<9, 12>>;
  using Z = LinePlan<108, 16, Radices<3, 4, 9>, Radices<9, 4, 3>>;
  using ZA = LinePlan<108, 16, Radices<3, 4, 9>, Radices<9, 4, 3>>;
  static constexpr int PZ = 16, PZA = 16;
};
template <> struct SizePlan<float, 120> {
  using X = LinePlan<120, 12, Radices<10, 12>, Radices<12, 10>>;
  using Y = LinePlan<120, 12, Radices<12, 10>, Radices<10, 12>>;
  using Z = LinePlan<120, 32, Radices<6, 4, 5>, Radices<5, 4, 6>>;
  using ZA = LinePlan<120, 32, Radices<6, 4, 5>, Radices<5, 4, 6>>;
  static constexpr int PZ = 2, PZA = 8;
};
template <> struct SizePlan<float, 150> {
  using X = LinePlan<150, 32, Radices<6, 5, 5>, Radices<5, 5, 6>>;
  using Y = LinePlan<150, 16, Radices<3, 5, 10>, Radices<10, 5, 3>>;
  using Z = LinePlan<150, 32, Radices<6, 5, 5>, Radices<5, 5, 6>>;
  using ZA = LinePlan<150, 32, Radices<6, 5, 5>, Radices<5, 5, 6>>;
  static constexpr int PZ = 4, PZA = 4;
};
template <> struct SizePlan<float, 162> {
  using X = LinePlan<162, 54, Radices<6, 3, 3, 3>, Radices<3, 3, 3, 6>>;
  using Y = LinePlan<162, 20, Radices<2, 9, 9>, Radices<9, 9, 2>>;
  using Z = LinePlan<162, 32, Radices<9, 3, 6>, Radices<6, 3, 9>>;
  using ZA = LinePlan<162, 32, Radices<3, 3, 3, 6>, Radices<6, 3, 3, 3>>;
  static constexpr int PZ = 4, PZA = 4;
};
template <> struct SizePlan<float, 180> {
  using X = LinePlan<180, 36, Radices<6, 5, 6>, Radices<6, 5, 6>>;
  using Y = LinePlan<180, 20, Radices<2, 9, 10>, Radices<10, 9, 2>>;
  using Z = LinePlan<180, 32, Radices<5, 6, 6>, Radices<6, 6, 5>>;
  using ZA = LinePlan<180, 32, Radices<5, 6, 6>, Radices<6, 6, 5>>;
  static constexpr int PZ = 8, PZA = 8;
};
template <> struct SizePlan<float, 200> {
  using X = LinePlan<200, 50, Radices<5, 2, 4, 5>, Radices<5, 4, 2, 5>>;
  using Y = LinePlan<200, 20, Radices<2, 10, 10>, Radices<10, 10, 2>>;
  using Z = LinePlan<200, 16, Radices<8, 5, 5>, Radices<5, 5, 8>>;
  using ZA = LinePlan<200, 32, Radices<5, 4, 10>, Radices<10, 4, 5>>;
  static constexpr int PZ = 4, PZA = 8;
};
template <> struct SizePlan<float, 250> {
  using X = LinePlan<250, 50, Radices<2, 5, 5, 5>, Radices<5, 5, 5, 2>>;
  using Y = LinePlan<250, 28, Radices<5, 5, 10>, Radices<10, 5, 5>>;
  using Z = LinePlan<250, 64, Radices<5, 2, 5, 5>, Radices<5, 5, 2, 5>>;
  using ZA = LinePlan<250, 32, Radices<5, 5, 10>, Radices<10, 5, 5>>;
  static constexpr int PZ = 2, PZA = 4;
};
template <> struct SizePlan<float, 288> {
  using X = LinePlan<288, 48, Radices<6, 6, 8>, Radices<8, 6, 6>>;
  using Y = LinePlan<288, 24, Radices<2, 12, 12>, Radices<12, 12, 2>>;
  using Z = LinePlan<288, 64, Radices<8, 6, 6>, Radices<6, 6, 8>>;
  using ZA = LinePlan<288, 64, Radices<8, 6, 6>, Radices<6, 6, 8>>;
  static constexpr int PZ = 4, PZA = 4;
};
template <> struct SizePlan<float, 300> {
  using X = LinePlan<300, 60, Radices<2, 5, 5, 6>, Radices<6, 5, 5, 2>>;
  using Y = LinePlan<300, 32, Radices<3, 10, 10>, Radices<10, 10, 3>>;
  using Z = LinePlan<300, 64, Radices<2, 5, 5, 6>, Radices<6, 5, 5, 2>>;
  using ZA = LinePlan<300, 64, Radices<2, 5, 5, 6>, Radices<6, 5, 5, 2>>;
  static constexpr int PZ = 4, PZA = 4;
};
template <> struct SizePlan<float, 320> {
  using X = LinePlan<320, 40, Radices<10, 4, 8>, Radices<8, 4, 10>>;
  using Y = LinePlan<320, 40, Radices<10, 4, 8>, Radices<8, 4, 10>>;
  using Z = LinePlan<320, 64, Radices<8, 5, 8>, Radices<8, 5, 8>>;
  using ZA = LinePlan<320, 64, Radices<8, 5, 8>, Radices<8, 5, 8>>;
  static constexpr int PZ = 4, PZA = 4;
};
template <> struct SizePlan<float, 400> {
  using X = LinePlan<400, 40, Radices<10, 10, 4>, Radices<4, 10, 10>>;
  using Y = LinePlan<400, 32, Radices<16, 5, 5>, Radices<5, 5, 16>>;
  using Z = LinePlan<400, 32, Radices<16, 5, 5>, Radices<5, 5, 16>>;
  using ZA = LinePlan<400, 64, Radices<10, 4, 10>, Radices<10, 4, 10>>;
  static constexpr int PZ = 2, PZA = 4;
};
template <> struct SizePlan<float, 432> {
  using X = LinePlan<432, 54, Radices<3, 4, 4, 9>, Radices<9, 4, 4, 3>>;
  using Y = LinePlan<432, 32, Radices<16, 3, 3, 3>, Radices<3, 3, 3, 16>>;
  using Z = LinePlan<432, 64, Radices<3, 4, 4, 9>, Radices<9, 4, 4, 3>>;
  using ZA = LinePlan<432, 64, Radices<3, 4, 4, 9>, Radices<9, 4, 4, 3>>;
  static constexpr int PZ = 4, PZA = 4;
};
template <> struct SizePlan<float, 450> {
  using X = LinePlan<450, 45, Radices<3, 5, 10, 3>, Radices<3, 10, 5, 3>>;
  using Y = LinePlan<450, 45, Radices<3, 5, 10, 3>, Radices<3, 10, 5, 3>>;
  using Z = LinePlan<450, 64, Radices<5, 9, 10>, Radices<10, 9, 5>>;
  using ZA = LinePlan<450, 64, Radices<5, 9, 10>, Radices<10, 9, 5>>;
  static constexpr int PZ = 4, PZA = 4;
};
template <> struct SizePlan<float, 480> {
  using X = LinePlan<480, 32, Radices<4, 3, 5, 8>, Radices<8, 5, 3, 4>>;
  using Y = LinePlan<480, 48, Radices<4, 10, 12>, Radices<12, 10, 4>>;
  using Z = LinePlan<480, 64, Radices<5, 4, 8, 3>, Radices<3, 8, 4, 5>>;
  using ZA = LinePlan<480, 64, Radices<10, 4, 4, 3>, Radices<3, 4, 4, 10>>;
  static constexpr int PZ = 2, PZA = 4;
};
template <> struct SizePlan<float, 486> {
  using X = LinePlan<486, 64, Radices<3, 9, 2, 9>, Radices<9, 2, 9, 3>>;
  using Y = LinePlan<486, 56, Radices<6, 9, 9>, Radices<9, 9, 6>>;
  using Z = LinePlan<486, 64, Radices<3, 2, 9, 9>, Radices<9, 9, 2, 3>>;
  using ZA = LinePlan<486, 64, Radices<3, 2, 9, 9>, Radices<9, 9, 2, 3>>;
  static constexpr int PZ = 4, PZA = 4;
};
template <> struct SizePlan<float, 500> {
  using X = LinePlan<500, 50, Radices<10, 5, 10>, Radices<10, 5, 10>>;
  using Y = LinePlan<500, 52, Radices<5, 10, 10>, Radices<10, 10, 5>>;
  using Z = LinePlan<500, 64, Radices<5, 10, 10>, Radices<10, 10, 5>>;
  using ZA = LinePlan<500, 64, Radices<5, 10, 10>, Radices<10, 10, 5>>;
  static constexpr int PZ = 4, PZA = 4;
};
template <> struct SizePlan<double, 16> {
  using X = LinePlanD<16, 8, Radices<4, 2, 2>, Radices<2, 2, 4>>;
  using Y = LinePlanD<16, 8, Radices<4, 4>, Radices<4, 4>>;
  using Z = LinePlanD<16, 8, Radices<4, 4>, Radices<4, 4>>;
  using ZA = LinePlanD<16, 8, Radices<4, 4>, Radices<4, 4>>;
  static constexpr int PZ = 32, PZA = 32;
};
template <> struct SizePlan<double, 18> {
  using X = LinePlanD<18, 6, Radices<6, 3>, Radices<3, 6>>;
  using Y = LinePlanD<18, 8, Radices<6, 3>, Radices<3, 6>>;
  using Z = LinePlanD<18, 16, Radices<6, 3>, Radices<3, 6>>;
  using ZA = LinePlanD<18, 16, Radices<6, 3>, Radices<3, 6>>;
  static constexpr int PZ = 4, PZA = 4;
};
template <> struct SizePlan<double, 20> {
  using X = LinePlanD<20, 8, Radices<4, 5>, Radices<5, 4>>;
  using Y = LinePlanD<20, 8, Radices<5, 4>, Radices<4, 5>>;
  using Z = LinePlanD<20, 8, Radices<5, 4>, Radices<4, 5>>;
  using ZA = LinePlanD<20, 8, Radices<5, 4>, Radices<4, 5>>;
  static constexpr int PZ = 16, PZA = 16;
};
template <> struct SizePlan<double, 24> {
  using X = LinePlanD<24, 12, Radices<4, 2, 3>, Radices<3, 2, 4>>;
  using Y = LinePlanD<24, 8, Radices<6, 4>, Radices<4, 6>>;
  using Z = LinePlanD<24, 8, Radices<6, 4>, Radices<4, 6>>;
  using ZA = LinePlanD<24, 8, Radices<6, 4>, Radices<4, 6>>;
  static constexpr int PZ = 32, PZA = 32;
};
template <> struct SizePlan<double, 30> {
  using X = LinePlanD<30, 15, Radices<5, 2, 3>, Radices<3, 2, 5>>;
  using Y = LinePlanD<30, 8, Radices<6, 5>, Radices<5, 6>>;
  using Z = LinePlanD<30, 16, Radices<5, 2, 3>, Radices<3, 2, 5>>;
  using ZA = LinePlanD<30, 16, Radices<5, 2, 3>, Radices<3, 2, 5>>;
  static constexpr int PZ = 4, PZA = 4;
};
template <> struct SizePlan<double, 32> {
  using X = LinePlanD<32, 16, Radices<4, 2, 4>, Radices<4, 2, 4>>;
  using Y = LinePlanD<32, 16, Radices<4, 2, 4>, Radices<4, 2, 4>>;
  using Z = LinePlanD<32, 16, Radices<4, 2, 4>, Radices<4, 2, 4>>;
  using ZA = LinePlanD<32, 16, Radices<4, 2, 4>, Radices<4, 2, 4>>;
  static constexpr int PZ = 16, PZA = 16;
};
template <> struct SizePlan<double, 36> {
  using X = LinePlanD<36, 12, Radices<3, 3, 4>, Radices<4, 3, 3>>;
  using Y = LinePlanD<36, 16, Radices<4, 3, 3>, Radices<3, 3, 4>>;
  using Z = LinePlanD<36, 16, Radices<4, 3, 3>, Radices<3, 3, 4>>;
  using ZA = LinePlanD<36, 16, Radices<4, 3, 3>, Radices<3, 3, 4>>;
  static constexpr int PZ = 16, PZA = 16;
};
template <> struct SizePlan<double, 40> {
  using X = LinePlanD<40, 24, Radices<5, 2, 4>, Radices<4, 2, 5>>;
  using Y = LinePlanD<40, 24, Radices<5, 2, 4>, Radices<4, 2, 5>>;
  using Z = LinePlanD<40, 32, Radices<5, 2, 4>, Radices<4, 2, 5>>;
  using ZA = LinePlanD<40, 32, Radices<5, 2, 4>, Radices<4, 2, 5>>;
  static constexpr int PZ = 8, PZA = 8;
};
template <> struct SizePlan<double, 48> {
  using X = LinePlanD<48, 16, Radices<4, 3, 4>, Radices<4, 3, 4>>;
  using Y = LinePlanD<48, 16, Radices<4, 3, 4>, Radices<4, 3, 4>>;
  using Z = LinePlanD<48, 16, Radices<4, 3, 4>, Radices<4, 3, 4>>;
  using ZA = LinePlanD<48, 16, Radices<4, 3, 4>, Radices<4, 3, 4>>;
  static constexpr int PZ = 16, PZA = 16;
};
template <> struct SizePlan<double, 50> {
  using X = LinePlanD<50, 25, Radices<5, 2, 5>, Radices<5, 2, 5>>;
  using Y = LinePlanD<50, 32, Radices<5, 2, 5>, Radices<5, 2, 5>>;
  using Z = LinePlanD<50, 32, Radices<5, 2, 5>, Radices<5, 2, 5>>;
  using ZA = LinePlanD<50, 32, Radices<5, 2, 5>, Radices<5, 2, 5>>;
  static constexpr int PZ = 4, PZA = 4;
};
template <> struct SizePlan<double, 54> {
  using X = LinePlanD<54, 24, Radices<6, 3, 3>, Radices<3, 3, 6>>;
  using Y = LinePlanD<54, 24, Radices<6, 3, 3>, Radices<3, 3, 6>>;
  using Z = LinePlanD<54, 32, Radices<3, 2, 3, 3>, Radices<3, 3, 2, 3>>;
  using ZA = LinePlanD<54, 32, Radices<6, 3, 3>, Radices<3, 3, 6>>;
  static constexpr int PZ = 2, PZA = 4;
};
template <> struct SizePlan<double, 60> {
  using X = LinePlanD<60, 24, Radices<5, 3, 4>, Radices<4, 3, 5>>;
  using Y = LinePlanD<60, 24, Radices<5, 3, 4>, Radices<4, 3, 5>>;
  using Z = LinePlanD<60, 32, Radices<5, 3, 4>, Radices<4, 3, 5>>;
  using ZA = LinePlanD<60, 32, Radices<5, 3, 4>, Radices<4, 3, 5>>;
  static constexpr int PZ = 8, PZA = 8;
};
template <> struct SizePlan<double, 64> {
  using X = LinePlanD<64, 16, Radices<4, 4, 4>, Radices<4, 4, 4>>;
  using Y = LinePlanD<64, 16, Radices<4, 4, 4>, Radices<4, 4, 4>>;
  using Z = LinePlanD<64, 16, Radices<4, 4, 4>, Radices<4, 4, 4>>;
  using ZA = LinePlanD<64, 16, Radices<4, 4, 4>, Radices<4, 4, 4>>;
  static constexpr int PZ = 16, PZA = 16;
};
template <> struct SizePlan<double, 72> {
  using X = LinePlanD<72, 36, Radices<4, 2, 3, 3>, Radices<3, 3, 2, 4>>;
  using Y = LinePlanD<72, 24, Radices<6, 3, 4>, Radices<4, 3, 6>>;
  using Z = LinePlanD<72, 32, Radices<6, 3, 4>, Radices<4, 3, 6>>;
  using ZA = LinePlanD<72, 32, Radices<6, 3, 4>, Radices<4, 3, 6>>;
  static constexpr int PZ = 8, PZA = 8;
};
template <> struct SizePlan<double, 80> {
  using X = LinePlanD<80, 24, Radices<5, 4, 4>, Radices<4, 4, 5>>;
  using Y = LinePlanD<80, 24, Radices<5, 4, 4>, Radices<4, 4, 5>>;
  using Z = LinePlanD<80, 32, Radices<4, 4, 5>, Radices<5, 4, 4>>;
  using ZA = LinePlanD<80, 32, Radices<5, 4, 4>, Radices<4, 4, 5>>;
  static constexpr int PZ = 2, PZA = 8;
};
template <> struct SizePlan<double, 90> {
  using X = LinePlanD<90, 32, Radices<6, 3, 5>, Radices<5, 3, 6>>;
  using Y = LinePlanD<90, 16, Radices<10, 9>, Radices<9, 10>>;
  using Z = LinePlanD<90, 32, Radices<5, 3, 3, 2>, Radices<2, 3, 3, 5>>;
  using ZA = LinePlanD<90, 16, Radices<10, 9>, Radices<9, 10>>;
  static constexpr int PZ = 4, PZA = 4;
};
template <> struct SizePlan<double, 96> {
  using X = LinePlanD<96, 24, Radices<4, 4, 6>, Radices<6, 4, 4>>;
  using Y = LinePlanD<96, 24, Radices<6, 4, 4>, Radices<4, 4, 6>>;
  using Z = LinePlanD<96, 32, Radices<4, 2, 3, 4>, Radices<4, 3, 2, 4>>;
  using ZA = LinePlanD<96, 16, Radices<8, 2, 6>, Radices<6, 2, 8>>;
  static constexpr int PZ = 2, PZA = 16;
};
template <> struct SizePlan<double, 100> {
  using X = LinePlanD<100, 32, Radices<5, 4, 5>, Radices<5, 4, 5>>;
  using Y = LinePlanD<100, 25, Radices<5, 4, 5>, Radices<5, 4, 5>>;
  using Z = LinePlanD<100, 32, Radices<5, 4, 5>, Radices<5, 4, 5>>;
  using ZA = LinePlanD<100, 32, Radices<5, 4, 5>, Radices<5, 4, 5>>;
  static constexpr int PZ = 8, PZA = 8;
};
template <> struct SizePlan<double, 108> {
  using X = LinePlanD<108, 24, Radices<6, 3, 6>, Radices<6, 3, 6>>;
  using Y = LinePlanD<108, 16, Radices<9, 4, 3>, Radices<3, 4, 9>>;
  using Z = LinePlanD<108, 16, Radices<9, 4, 3>, Radices<3, 4, 9>>;
  using ZA = LinePlanD<108, 16, Radices<9, 4, 3>, Radices<3, 4, 9>>;
  static constexpr int PZ = 4, PZA = 16;
};
template <> struct SizePlan<double, 120> {
  using X = LinePlanD<120, 30, Radices<5, 4, 6>, Radices<6, 4, 5>>;
  using Y = LinePlanD<120, 32, Radices<6, 4, 5>, Radices<5, 4, 6>>;
  using Z = LinePlanD<120, 32, Radices<6, 4, 5>, Radices<5, 4, 6>>;
  using ZA = LinePlanD<120, 16, Radices<10, 4, 3>, Radices<3, 4, 10>>;
  static constexpr int PZ = 8, PZA = 16;
};
template <> struct SizePlan<double, 128> {
  using X = LinePlanD<128, 32, Radices<4, 2, 4, 4>, Radices<4, 4, 2, 4>>;
  using Y = LinePlanD<128, 16, Radices<8, 4, 4>, Radices<4, 4, 8>>;
  using Z = LinePlanD<128, 16, Radices<8, 4, 4>, Radices<4, 4, 8>>;
  using ZA = LinePlanD<128, 32, Radices<4, 2, 4, 4>, Radices<4, 4, 2, 4>>;
  static constexpr int PZ = 16, PZA = 8;
};
template <> struct SizePlan<double, 144> {
  using X = LinePlanD<144, 24, Radices<6, 2, 2, 6>, Radices<6, 2, 2, 6>>;
  using Y = LinePlanD<144, 24, Radices<4, 6, 6>, Radices<6, 6, 4>>;
  using Z = LinePlanD<144, 32, Radices<4, 6, 6>, Radices<6, 6, 4>>;
  using ZA = LinePlanD<144, 64, Radices<4, 3, 3, 4>, Radices<4, 3, 3, 4>>;
  static constexpr int PZ = 8, PZA = 4;
};
template <> struct SizePlan<double, 150> {
  using X = LinePlanD<150, 30, Radices<5, 5, 6>, Radices<6, 5, 5>>;
  using Y = LinePlanD<150, 32, Radices<6, 5, 5>, Radices<5, 5, 6>>;
  using Z = LinePlanD<150, 32, Radices<6, 5, 5>, Radices<5, 5, 6>>;
  using ZA = LinePlanD<150, 32, Radices<6, 5, 5>, Radices<5, 5, 6>>;
  static constexpr int PZ = 4, PZA = 4;
};
template <> struct SizePlan<double, 160> {
  using X = LinePlanD<160, 40, Radices<5, 2, 4, 4>, Radices<4, 4, 2, 5>>;
  using Y = LinePlanD<160, 32, Radices<8, 5, 4>, Radices<4, 5, 8>>;
  using Z = LinePlanD<160, 32, Radices<4, 5, 8>, Radices<8, 5, 4>>;
  using ZA = LinePlanD<160, 32, Radices<8, 5, 4>, Radices<4, 5, 8>>;
  static constexpr int PZ = 2, PZA = 8;
};
template <> struct SizePlan<double, 162> {
  using X = LinePlanD<162, 27, Radices<6, 3, 3, 3>, Radices<3, 3, 3, 6>>;
  using Y = LinePlanD<162, 27, Radices<9, 3, 6>, Radices<6, 3, 9>>;
  using Z = LinePlanD<162, 32, Radices<6, 3, 3, 3>, Radices<3, 3, 3, 6>>;
  using ZA = LinePlanD<162, 32, Radices<9, 3, 6>, Radices<6, 3, 9>>;
  static constexpr int PZ = 4, PZA = 4;
};
template <> struct SizePlan<double, 180> {
  using X = LinePlanD<180, 36, Radices<6, 6, 5>, Radices<5, 6, 6>>;
  using Y = LinePlanD<180, 40, Radices<6, 5, 6>, Radices<6, 5, 6>>;
  using Z = LinePlanD<180, 64, Radices<5, 3, 3, 4>, Radices<4, 3, 3, 5>>;
  using ZA = LinePlanD<180, 64, Radices<5, 3, 3, 4>, Radices<4, 3, 3, 5>>;
  static constexpr int PZ = 4, PZA = 4;
};
template <> struct SizePlan<double, 192> {
  using X = LinePlanD<192, 64, Radices<4, 3, 4, 4>, Radices<4, 4, 3, 4>>;
  using Y = LinePlanD<192, 24, Radices<3, 8, 8>, Radices<8, 8, 3>>;
  using Z = LinePlanD<192, 32, Radices<8, 6, 4>, Radices<4, 6, 8>>;
  using ZA = LinePlanD<192, 64, Radices<4, 3, 4, 4>, Radices<4, 4, 3, 4>>;
  static constexpr int PZ = 8, PZA = 4;
};
template <> struct SizePlan<double, 200> {
  using X = LinePlanD<200, 56, Radices<5, 2, 4, 5>, Radices<5, 4, 2, 5>>;
  using Y = LinePlanD<200, 40, Radices<8, 5, 5>, Radices<5, 5, 8>>;
  using Z = LinePlanD<200, 64, Radices<5, 2, 4, 5>, Radices<5, 4, 2, 5>>;
  using ZA = LinePlanD<200, 64, Radices<5, 2, 4, 5>, Radices<5, 4, 2, 5>>;
  static constexpr int PZ = 4, PZA = 4;
};
template <> struct SizePlan<double, 216> {
  using X = LinePlanD<216, 40, Radices<6, 6, 6>, Radices<6, 6, 6>>;
  using Y = LinePlanD<216, 18, Radices<12, 3, 6>, Radices<6, 3, 12>>;
  using Z = LinePlanD<216, 32, Radices<9, 8, 3>, Radices<3, 8, 9>>;
  using ZA = LinePlanD<216, 32, Radices<9, 8, 3>, Radices<3, 8, 9>>;
  static constexpr int PZ = 2, PZA = 8;
};
template <> struct SizePlan<double, 240> {
  using X = LinePlanD<240, 64, Radices<3, 4, 4, 5>, Radices<5, 4, 4, 3>>;
  using Y = LinePlanD<240, 32, Radices<10, 8, 3>, Radices<3, 8, 10>>;
  using Z = LinePlanD<240, 64, Radices<3, 4, 4, 5>, Radices<5, 4, 4, 3>>;
  using ZA = LinePlanD<240, 32, Radices<10, 8, 3>, Radices<3, 8, 10>>;
  static constexpr int PZ = 2, PZA = 8;
};
template <> struct SizePlan<double, 250> {
  using X = LinePlanD<250, 50, Radices<5, 5, 10>, Radices<10, 5, 5>>;
  using Y = LinePlanD<250, 32, Radices<10, 5, 5>, Radices<5, 5, 10>>;
  using Z = LinePlanD<250, 64, Radices<5, 2, 5, 5>, Radices<5, 5, 2, 5>>;
  using ZA = LinePlanD<250, 64, Radices<5, 2, 5, 5>, Radices<5, 5, 2, 5>>;
  static constexpr int PZ = 4, PZA = 4;
};
template <> struct SizePlan<double, 256> {
  using X = LinePlanD<256, 64, Radices<4, 4, 4, 4>, Radices<4, 4, 4, 4>>;
  using Y = LinePlanD<256, 32, Radices<8, 4, 8>, Radices<8, 4, 8>>;
  using Z = LinePlanD<256, 32, Radices<8, 4, 8>, Radices<8, 4, 8>>;
  using ZA = LinePlanD<256, 64, Radices<4, 4, 4, 4>, Radices<4, 4, 4, 4>>;
  static constexpr int PZ = 8, PZA = 4;
};
template <> struct SizePlan<double, 270> {
  using X = LinePlanD<270, 56, Radices<6, 3, 5, 3>, Radices<3, 5, 3, 6>>;
  using Y = LinePlanD<270, 32, Radices<10, 3, 9>, Radices<9, 3, 10>>;
  using Z = LinePlanD<270, 32, Radices<10, 3, 9>, Radices<9, 3, 10>>;
  using ZA = LinePlanD<270, 32, Radices<10, 3, 9>, Radices<9, 3, 10>>;
  static constexpr int PZ = 4, PZA = 4;
};
template <> struct SizePlan<double, 288> {
  using X = LinePlanD<288, 48, Radices<6, 6, 8>, Radices<8, 6, 6>>;
  using Y = LinePlanD<288, 24, Radices<12, 2, 12>, Radices<12, 2, 12>>;
  using Z = LinePlanD<288, 64, Radices<8, 6, 6>, Radices<6, 6, 8>>;
  using ZA = LinePlanD<288, 64, Radices<8, 6, 6>, Radices<6, 6, 8>>;
  static constexpr int PZ = 4, PZA = 4;
};
template <> struct SizePlan<double, 300> {
  using X = LinePlanD<300, 64, Radices<6, 5, 5, 2>, Radices<2, 5, 5, 6>>;
  using Y = LinePlanD<300, 64, Radices<6, 5, 5, 2>, Radices<2, 5, 5, 6>>;
  using Z = LinePlanD<300, 64, Radices<6, 5, 5, 2>, Radices<2, 5, 5, 6>>;
  using ZA = LinePlanD<300, 64, Radices<10, 5, 6>, Radices<6, 5, 10>>;
  static constexpr int PZ = 4, PZA = 4;
};
template <> struct SizePlan<double, 320> {
  using X = LinePlanD<320, 80, Radices<4, 4, 4, 5>, Radices<5, 4, 4, 4>>;
  using Y = LinePlanD<320, 80, Radices<5, 4, 4, 4>, Radices<4, 4, 4, 5>>;
  using Z = LinePlanD<320, 64, Radices<8, 5, 8>, Radices<8, 5, 8>>;
  using ZA = LinePlanD<320, 64, Radices<8, 5, 8>, Radices<8, 5, 8>>;
  static constexpr int PZ = 4, PZA = 4;
};
template <> struct SizePlan<double, 324> {
  using X = LinePlanD<324, 56, Radices<6, 3, 3, 6>, Radices<6, 3, 3, 6>>;
  using Y = LinePlanD<324, 56, Radices<9, 6, 6>, Radices<6, 6, 9>>;
  using Z = LinePlanD<324, 64, Radices<6, 3, 3, 6>, Radices<6, 3, 3, 6>>;
  using ZA = LinePlanD<324, 64, Radices<9, 6, 6>, Radices<6, 6, 9>>;
  static constexpr int PZ = 4, PZA = 4;
};
template <> struct SizePlan<double, 360> {
  using X = LinePlanD<360, 72, Radices<6, 5, 2, 6>, Radices<6, 2, 5, 6>>;
  using Y = LinePlanD<360, 60, Radices<10, 6, 6>, Radices<6, 6, 10>>;
  using Z = LinePlanD<360, 64, Radices<6, 6, 10>, Radices<10, 6, 6>>;
  using ZA = LinePlanD<360, 64, Radices<10, 6, 6>, Radices<6, 6, 10>>;
  static constexpr int PZ = 2, PZA = 4;
};
template <> struct SizePlan<double, 384> {
  using X = LinePlanD<384, 64, Radices<6, 8, 8>, Radices<8, 8, 6>>;
  using Y = LinePlanD<384, 64, Radices<8, 6, 8>, Radices<8, 6, 8>>;
  using Z = LinePlanD<384, 64, Radices<8, 6, 8>, Radices<8, 6, 8>>;
  using ZA = LinePlanD<384, 64, Radices<8, 6, 8>, Radices<8, 6, 8>>;
  static constexpr int PZ = 4, PZA = 4;
};
template <> struct SizePlan<double, 400> {
  using X = LinePlanD<400, 56, Radices<10, 4, 10>, Radices<10, 4, 10>>;
  using Y = LinePlanD<400, 50, Radices<10, 4, 10>, Radices<10, 4, 10>>;
  using Z = LinePlanD<400, 64, Radices<10, 4, 10>, Radices<10, 4, 10>>;
  using ZA = LinePlanD<400, 64, Radices<10, 4, 10>, Radices<10, 4, 10>>;
  static constexpr int PZ = 4, PZA = 4;
};
template <> struct SizePlan<double, 432> {
  using X = LinePlanD<432, 72, Radices<6, 6, 2, 6>, Radices<6, 2, 6, 6>>;
  using Y = LinePlanD<432, 56, Radices<9, 4, 4, 3>, Radices<3, 4, 4, 9>>;
  using Z = LinePlanD<432, 64, Radices<3, 4, 4, 9>, Radices<9, 4, 4, 3>>;
  using ZA = LinePlanD<432, 64, Radices<12, 4, 9>, Radices<9, 4, 12>>;
  static constexpr int PZ = 2, PZA = 4;
};
template <> struct SizePlan<double, 450> {
  using X = LinePlanD<450, 90, Radices<6, 5, 5, 3>, Radices<3, 5, 5, 6>>;
  using Y = LinePlanD<450, 56, Radices<10, 9, 5>, Radices<5, 9, 10>>;
  using Z = LinePlanD<450, 64, Radices<5, 9, 10>, Radices<10, 9, 5>>;
  using ZA = LinePlanD<450, 64, Radices<10, 9, 5>, Radices<5, 9, 10>>;
  static constexpr int PZ = 2, PZA = 4;
};
template <> struct SizePlan<double, 480> {
  using X = LinePlanD<480, 64, Radices<10, 4, 4, 3>, Radices<3, 4, 4, 10>>;
  using Y = LinePlanD<480, 64, Radices<10, 4, 4, 3>, Radices<3, 4, 4, 10>>;
  using Z = LinePlanD<480, 64, Radices<12, 4, 10>, Radices<10, 4, 12>>;
  using ZA = LinePlanD<480, 64, Radices<12, 4, 10>, Radices<10, 4, 12>>;
  static constexpr int PZ = 4, PZA = 4;
};
template <> struct SizePlan<double, 486> {
  using X = LinePlanD<486, 64, Radices<9, 2, 3, 9>, Radices<9, 3, 2, 9>>;
  using Y = LinePlanD<486, 64, Radices<9, 2, 3, 9>, Radices<9, 3, 2, 9>>;
  using Z = LinePlanD<486, 64, Radices<6, 9, 9>, Radices<9, 9, 6>>;
  using ZA = LinePlanD<486, 64, Radices<6, 9, 9>, Radices<9, 9, 6>>;
  static constexpr int PZ = 4, PZA = 4;
};
template <> struct SizePlan<double, 500> {
  using X = LinePlanD<500, 56, Radices<10, 5, 10>, Radices<10, 5, 10>>;
  using Y = LinePlanD<500, 56, Radices<10, 5, 10>, Radices<10, 5, 10>>;
  using Z = LinePlanD<500, 64, Radices<10, 5, 10>, Radices<10, 5, 10>>;
  using ZA = LinePlanD<500, 64, Radices<10, 5, 10>, Radices<10, 5, 10>>;
  static constexpr int PZ = 2, PZA = 4;
};
template <> struct SizePlan<double, 512> {
  using X = LinePlanD<512, 64, Radices<8, 8, 8>, Radices<8, 8, 8>>;
  using Y = LinePlanD<512, 64, Radices<8, 8, 8>, Radices<8, 8, 8>>;
  using Z = LinePlanD<512, 64, Radices<8, 8, 8>, Radices<8, 8, 8>>;
  using ZA = LinePlanD<512, 64, Radices<8, 8, 8>, Radices<8, 8, 8>>;
  static constexpr int PZ = 4, PZA = 4;
};

}  // namespace ns

// X(type, size) for every plan above
#define NS_FOR_EACH_SIZE(X) \
  X(float, 16) \
  X(float, 18) \
  X(float, 20) \
  X(float, 24) \
  X(float, 30) \
  X(float, 32) \
  X(float, 36) \
  X(float, 40) \
  X(float, 48) \
  X(float, 50) \
  X(float, 54) \
  X(float, 60) \
  X(float, 72) \
  X(float, 80) \
  X(float, 90) \
  X(float, 96) \
  X(float, 100) \
  X(float, 108) \
  X(float, 120) \
  X(float, 150) \
  X(float, 162) \
  X(float, 180) \
  X(float, 200) \
  X(float, 250) \
  X(float, 288) \
  X(float, 300) \
  X(float, 320) \
  X(float, 400) \
  X(float, 432) \
  X(float, 450) \
  X(float, 480) \
  X(float, 486) \
  X(float, 500) \
  X(double, 16) \
  X(double, 18) \
  X(double, 20) \
  X(double, 24) \
  X(double, 30) \
  X(double, 32) \
  X(double, 36) \
  X(double, 40) \
  X(double, 48) \
  X(double, 50) \
  X(double, 54) \
  X(double, 60) \
  X(double, 64) \
  X(double, 72) \
  X(double, 80) \
  X(double, 90) \
  X(double, 96) \
  X(double, 100) \
  X(double, 108) \
  X(double, 120) \
  X(double, 128) \
  X(double, 144) \
  X(double, 150) \
  X(double, 160) \
  X(double, 162) \
  X(double, 180) \
  X(double, 192) \
  X(double, 200) \
  X(double, 216) \
  X(double, 240) \
  X(double, 250) \
  X(double, 256) \
  X(double, 270) \
  X(double, 288) \
  X(double, 300) \
  X(double, 320) \
  X(double, 324) \
  X(double, 360) \
  X(double, 384) \
  X(double, 400) \
  X(double, 432) \
  X(double, 450) \
  X(double, 480) \
  X(double, 486) \
  X(double, 500) \
  X(double, 512)
