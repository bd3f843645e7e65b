// Configurations of the batched form's grouped LU, per precision and order
// bucket: the panel width and the loop of the trailing update (feast::GROUP_*).
// Written by `python -m paper_1404_1768_amd.autotune` from factorisation
// timings of every candidate on AMD Radeon Graphics (gfx950:sramecc+:xnack-); entries are looked up with the order
// n* that splits a batch's LU work in half.
#pragma once
#include <cstdint>

namespace feast_tune {

struct Entry {
  int64_t lo, hi;  // bucket: lo <= n* < hi
  int prec;        // FEAST_FP64 or FEAST_MIXED
  int nb;          // panel width, 64 or 128
  int update;      // feast::GROUP_PLAIN or GROUP_UPDATE_M3
};

inline constexpr Entry kBatch[] = {
    {64, 384, 0, 128, 1},  // ms: nb128_u1 4.08, nb128_u2 4.07, nb64_u1 4.15, nb64_u2 4.14
    {64, 384, 1, 128, 1},  // ms: nb128_u1 3.31, nb128_u2 3.30, nb64_u1 3.34, nb64_u2 3.31
    {384, 768, 0, 128, 1},  // ms: nb128_u1 14.38, nb128_u2 14.21, nb64_u1 14.97, nb64_u2 14.46
    {384, 768, 1, 128, 1},  // ms: nb128_u1 9.29, nb128_u2 9.01, nb64_u1 9.58, nb64_u2 9.25
    {768, 1536, 0, 128, 1},  // ms: nb128_u1 50.31, nb128_u2 47.81, nb64_u1 51.73, nb64_u2 48.50
    {768, 1536, 1, 128, 1},  // ms: nb128_u1 30.44, nb128_u2 28.35, nb64_u1 31.41, nb64_u2 29.26
    {1536, 3072, 0, 128, 1},  // ms: nb128_u1 191.80, nb128_u2 174.56, nb64_u1 196.84, nb64_u2 177.69
    {1536, 3072, 1, 128, 1},  // ms: nb128_u1 106.74, nb128_u2 96.19, nb64_u1 113.96, nb64_u2 101.59
    {3072, 16385, 0, 128, 1},  // ms: nb128_u1 156.37, nb128_u2 142.67, nb64_u1 162.92, nb64_u2 145.81
    {3072, 16385, 1, 128, 1},  // ms: nb128_u1 89.54, nb128_u2 80.22, nb64_u1 94.46, nb64_u2 83.95
};

}  // namespace feast_tune
