// The tile rules of the grouped GEMMs as a C library for test_tile_rule.py.
#include "tile_rule.hpp"

extern "C" {
int fwd_tile(int cus, int N, int K, long groups, long rows_hint, long rows2, int epilogue) {
  return moe::fwd_tile({cus, N, K, groups, rows_hint, rows2}, (moe::FwdEpilogue)epilogue);
}
int bwd_rows_tile(int cus, long groups, long rows_hint, long max_rows, int N, int K) {
  return moe::bwd_rows_tile(cus, groups, rows_hint, max_rows, N, K);
}
void wgrad_order(int i, int tm, int tn, int f32, int* mn) {
  const moe::TileMN o = moe::wgrad_order(i, tm, tn, f32);
  mn[0] = o.m;
  mn[1] = o.n;
}
int band_m(int bm) { return moe::band_m(bm); }
int wgrad_on_ring(long rows_hint, long pitch) { return moe::wgrad_on_ring(rows_hint, pitch); }
}
