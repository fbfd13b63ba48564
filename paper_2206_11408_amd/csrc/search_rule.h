// Which instance a search launch takes, and on how many workgroups (host
// arithmetic only; the instances are in search_kernel.h).
#pragma once

#include <cstdint>

namespace finger {

// Query waves per CU that the registers of a wide-pass instance leave (two
// waves per SIMD; three for 132 to 256 dimensions, four in plain search).
constexpr int wide_waves_per_cu(bool plain, int g, int t4) {
  return g == 32 && t4 == 2 ? (plain ? 16 : 12) : 8;
}

// Wide or narrow passes of exact distances for vectors longer than 128 (g
// lanes to a vector, t4 float4 a lane).  nq queries on `waves` query waves.
//
// A wide pass makes fewer dependent trips to memory and leaves fewer resident
// waves.  While every query has a wave at once anyway, the trips are what
// counts: 1,000 queries, ef 16 / 100, wide against narrow: 256 dimensions bf16
// 1.48 / 1.22 times as fast, 512 bf16 1.23 / 1.11, 960 fp8 1.25 / 1.17, 2,048
// plain 1.02 / 1.06.  Past that a second, mostly empty round of waves costs
// more than the trips save (narrow against wide at 2,500 queries: 300 f32
// 1.32 / 1.46, 480 bf16 1.17 / 1.38, 960 bf16 1.21 / 1.31, 1,028 bf16 1.29 /
// 1.35; at 3,500: 192 bf16 1.17 / 1.28).  From about 9,000 queries on there
// are rounds enough for the partial one not to matter, and the wide passes
// of 132 to 256 dimensions in FINGER mode and of 516 to 1,024 win again
// (10,000 queries: 256 bf16 1.23 / 1.02, 960 fp8 1.17 / 0.98, 960 plain 0.97 /
// 1.07); the other shapes' do not.
//
// `mixed`: queries of different ef from a queue.  There is no round of waves to
// fill, and of the shapes that win again with many queries 132 to 256
// dimensions win at every size (256 dimensions, ef 12 to 101, 3,500 to 7,000
// queries: 1.08 to 1.15; 132: 1.02 to 1.05), 516 to 1,024 up to 12 queries a CU
// (2,500 and 3,000 queries: 516 1.02 to 1.11, 768 1.02 to 1.15, 1,024 1.06 to
// 1.30; beyond, 516 dimensions lose down to 0.77).
constexpr bool wide_passes(bool plain, int g, int t4, int64_t nq, int64_t waves, int cus, bool mixed = false) {
  if (g == 8) return false;
  if (nq <= (int64_t)wide_waves_per_cu(plain, g, t4) * cus || waves <= (int64_t)8 * cus) return true;
  const bool again = g == 64 ? t4 == 4 : t4 == 2 && !plain;
  return again && (mixed ? g == 32 || nq <= (int64_t)12 * cus : nq >= (int64_t)36 * cus);
}

// Workgroups of a static launch (query i belongs to workgroup i mod blocks).
// Each serves nq / blocks queries, so workgroups that wait for a resident one
// to end add a round of as many queries again: with several queries to a
// workgroup the grid is what is resident.  Wide instances of three and two
// waves a SIMD on the default grid of up to 16 a CU, 20,000 queries, ef 100:
// 256 dimensions bf16 1.33 times as fast with it, 960 1.21, 1,028 1.29.
constexpr int resident_blocks(int blocks, int64_t nq, int64_t per_cu, int cus) {
  return blocks < nq && per_cu > 0 && per_cu * cus < blocks ? (int)(per_cu * cus) : blocks;
}

}  // namespace finger
