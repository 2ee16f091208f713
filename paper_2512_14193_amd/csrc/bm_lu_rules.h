// Host rules of the LU: how a panel runs, the workgroups it needs resident, and from
// these how many problems are factored together and on how many of a server's lanes
// small requests run.  (No HIP here: the tests compile it with a host compiler.)
#pragma once

#include <stddef.h>

#define LU_NB 64                  // LU panel width
#define PANEL_PMAX 256            // max workgroups of a panel launch
#define SNT 448                   // threads of an exchanging panel's workgroup: one chain + SNB bulk wavefronts
#define SNB 6
// LDS requested by every panel launch: more than 160 KB minus any GEMM workgroup's
// share, so that no workgroup of the concurrent trailing update lands on a CU that
// runs a panel workgroup (the chain would lose issue slots), nor another panel's
#define PANEL_LDS_ALLOC ((size_t)LU_NB * (128 + 1) * 16)  // exchanging
#define SPN_LDS_ALLOC ((size_t)120 * 1024)                // streaming

// How the panel of R rows and jb columns runs: kind of kernel (panel_fn_of), its
// workgroups, and the exchange words it uses (slots_refill).  The streaming panel
// holds (rows per thread) x (columns per workgroup) values in a thread's registers.
// Per 64-column panel (us, alone on the device; threads x rows per thread x columns
// per workgroup):
//   rows      streaming                            exchanging (64 or 128 rows/workgroup)
//     64       47 (64x1x8)                          135
//    512       60 (256x2x4), 65 (512x1x4)           130
//   1024       72 (512x2x4), 77 (x8), 76 (256x4x4)  130
//   2048       94 (512x4x4), 108 (x2), 125 (1024x2x4)  131 to 155
//   2688      119 (448x6x4)                         150
//   3136      306 (448x8x4, spilled)                151
//   4032      167 (512x8x4), 200 (448x9x2)          152
// A thread of 512 or fewer holds 256 registers, which six rows of four columns fill with
// the next column's multipliers on their way.  Beyond 2688 rows they cannot be on their
// way, or a workgroup holds two columns, and reading the earlier columns becomes the
// chain: the exchanging panel (128 rows per workgroup) takes over.
struct lu_shape {
  int kind, wgs, threads, fill_h;
  long fill_n;
  size_t lds;
};
#define PANEL_KINDS 6
#define PANEL_STREAM_MAX_R 2688

// The orders and batches taken: counted by workgroups of 64 rows, 128 beyond 2048,
// whatever the panel's own are (lu_panel_wgs: the count that residency needs).
static inline int lu_order_units(int n) { return (n > 2048) ? (n + 127) / 128 : (n + 63) / 64; }

static inline bool panel_shape(int R, int jb, int ncu, lu_shape *o) {
  const int pmax = (ncu < PANEL_PMAX) ? ncu : PANEL_PMAX;
  if (R < 1 || lu_order_units(R) > pmax) return false;
  if (R <= PANEL_STREAM_MAX_R) {
    static const int cw[PANEL_KINDS - 1] = {8, 4, 4, 4, 4}, nt[PANEL_KINDS - 1] = {64, 256, 512, 512, 448};
    int k = (R <= LU_NB) ? 0 : 1;
    while (k > 0 && R > (256 << k)) ++k;
    o->kind = k;
    o->wgs = (jb + cw[k] - 1) / cw[k];
    o->threads = nt[k] + 64;
    o->lds = SPN_LDS_ALLOC;
    o->fill_n = (long)jb * R;
    o->fill_h = jb;
  } else {
    const int P = (R + 127) / 128;
    o->kind = PANEL_KINDS - 1;
    o->wgs = P;
    o->threads = SNT;
    o->lds = PANEL_LDS_ALLOC;
    o->fill_n = (long)jb * ((long)P * (jb + 1) + jb);
    o->fill_h = jb * P;
  }
  return true;
}

// Workgroups of the widest panel of an LU of order n (0: the order is not taken).  All
// of a panel's workgroups wait for each other, so they must run at the same time.
static inline int lu_panel_wgs(int n, int ncu) {
  int most = 0;
  for (int R = n; R > 0; R -= LU_NB) {
    lu_shape s;
    if (!panel_shape(R, (R < LU_NB) ? R : LU_NB, ncu, &s)) return 0;
    if (s.wgs > most) most = s.wgs;
  }
  return most;
}

// Of `count` problems of order n, how many are factored in shared launches: what the
// device holds at once.  0: refused.
static inline int lu_batch_fit(int n, int count, int ncu) {
  const int wgs = lu_panel_wgs(n, ncu);
  if (wgs == 0 || (long)count * lu_order_units(n) > ncu) return 0;
  const int fit = ncu / wgs;
  return (fit < 1) ? 1 : (fit < count) ? fit : count;
}

// A server's lanes: the configurations taken, and of `lanes` lanes those that small
// requests (N <= cmax) use, so that the panels of all of them stay within half of the
// CUs; and the requests of order n that one of these lanes may factor together.
static inline bool srv_lanes_ok(int lanes, int cmax, int ncu) {
  return lanes == 1 || (cmax <= 2048 && lanes * ((cmax + 63) / 64) <= ncu / 2);
}
static inline int srv_small_lanes(int lanes, int cmax, int ncu) {
  const int wgs = lu_panel_wgs(cmax, ncu), fit = (wgs > 0) ? ncu / 2 / wgs : 1;
  return (fit < 1) ? 1 : (fit < lanes) ? fit : lanes;
}
static inline int srv_batch_limit(int n, int batch_max, int small_lanes, int ncu) {
  const int wgs = lu_panel_wgs(n, ncu), fit = (wgs > 0) ? ncu / 2 / small_lanes / wgs : 1;
  const int b = (batch_max < fit) ? batch_max : fit;
  return (b < 1) ? 1 : b;
}
