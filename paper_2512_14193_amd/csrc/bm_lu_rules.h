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

// ---------------------------------------------------------------------------
// The segments of the product beside the panels (bm_getrf_schur_run)
// ---------------------------------------------------------------------------
#define SP_MAXSEG 10

struct sp_seg {
  int b0, b1, ks;  // blocks [b0, b1), k split into ks slices
};

// k-slices of a product of `tiles` tiles on `slots` workgroups: enough to fill
// them in one round, at most 16, each at least 256 deep (the three-multiplication
// form), and the partials within the workspace
static inline int sp_ksplit(int tiles, int slots, int k, size_t w_cap) {
  int ks = (tiles <= slots) ? slots / tiles : 1;
  const int kmax = (k / 256 > 1) ? k / 256 : 1;
  if (ks > kmax) ks = kmax;
  if (ks > 16) ks = 16;
  while (ks > 1 && (size_t)ks * tiles * 64 * 64 > w_cap) --ks;
  return ks < 1 ? 1 : ks;
}

static inline double sp_time(int tiles, int ks, int slots, int k, double per_k) {
  int kc = (k + ks - 1) / ks;
  kc = (kc + 15) / 16 * 16;
  const int rounds = (tiles * ks + slots - 1) / slots;
  return rounds * per_k * kc + (ks > 1 ? 0.006 : 0.0);
}

// per_k1, per_k2: ms per unit of k of a round of tiles, one workgroup per CU and two
// (block 0, whole device).  Returns 1 when, with a panel of the chain taking beta ms, the
// planned product has at most SP_MAXSEG segments and ends before the chain of panels (the
// overlap pays), else 0 (then the product is better formed in full first).
static inline int sp_plan_at(double beta, double per_k1, double per_k2, int n, int k, int ncu, int gs, size_t w_cap,
                             sp_seg *seg, int *nseg_out) {
  const int B = (n + LU_NB - 1) / LU_NB, tb = B;  // blocks; row tiles of a block
  const double margin = 0.03;
  int nseg = 0;
  const int ks0 = sp_ksplit(tb, 2 * ncu, k, w_cap);
  const double t0 = sp_time(tb, ks0, 2 * ncu, k, per_k2);
  seg[nseg++] = {0, 1, ks0};
  double E = t0;
  int f = 1;
  while (f < B) {
    if (nseg == SP_MAXSEG) return 0;
    const double limit = t0 + beta * f - margin, least = tb * per_k1 * k / gs;  // least: ms a block, all slots busy
    int best = 1, bks = sp_ksplit(tb, gs, k, w_cap);
    double bt = sp_time(tb, bks, gs, k, per_k1);
    for (int b = 2; b <= B - f && E + b * least <= limit + 1e-6; ++b) {
      const int ks = sp_ksplit(tb * b, gs, k, w_cap);
      const double t = sp_time(tb * b, ks, gs, k, per_k1), fin = E + t;
      int a = (int)((fin - t0) / beta);
      if (a > f - 1) a = f - 1;
      if (a < 0) a = 0;
      const double step = 0.012 + 8.0 * n * (64.0 * b) * 64.0 / 25e9;
      if (fin + a * step <= limit) {
        best = b;
        bks = ks;
        bt = t;
      }
    }
    // a segment that would leave a single block, which alone would need a catch-up
    // step for every panel before it, takes the rest
    if (B - f - best == 1 && nseg >= 2) {
      best = B - f;
      bks = sp_ksplit(tb * best, gs, k, w_cap);
      bt = sp_time(tb * best, bks, gs, k, per_k1);
    }
    seg[nseg++] = {f, f + best, bks};
    E += bt;
    f += best;
  }
  *nseg_out = nseg;
  return (E <= t0 + beta * B - margin) ? 1 : 0;
}

// The plan for the shortest panel time that needs few segments.  A panel with the
// launches to the next one takes 0.09 to 0.12 ms, but each segment's catch-up steps slow
// the chain in ways the model leaves out, so a plan of many segments loses what it gains
// (n = 1728: 9 segments 3.41 ms, 14 segments 4.30, 7 segments 3.74, product first 4.23;
// n = 2048: 9 segments 4.72, 13 segments 5.45, 24 segments 7.35, product first 5.20).
// First with the product an eighth slower than it runs alone, which leaves it room beside
// the updates (n = 1728: 3.25 ms, planned at its own rate 3.50), then, where that finds
// none, at its own rate and with the panels of more than 2048 rows in mind, 0.12 to 0.15 ms
// and the launches (product first -> beside the panels: n = 2176 5.77 -> 5.18 ms,
// 2240 6.00 -> 5.81, 2368 6.88 -> 6.41, 2432 7.12 -> 6.78; from about 2460 on no plan is
// found).  Every factorisation plans anew: a plan is given up at its eleventh segment and
// a segment's widths are tried up to the bound, 1 to 3 us on the host in all (with every
// plan and width tried to the end 12 us at n = 2048 and 110 at 4096).
static inline int sp_plan(int n, int k, int ncu, int gs, size_t w_cap, sp_seg *seg, int *nseg_out) {
  for (int i = 0; i <= 4; ++i)
    if (sp_plan_at(0.09 + 0.015 * i, 0.49 / 4096, 0.84 / 4096, n, k, ncu, gs, w_cap, seg, nseg_out)) return 1;
  for (int i = 0; i <= 7; ++i)
    if (sp_plan_at(0.09 + 0.015 * i, 0.43 / 4096, 0.74 / 4096, n, k, ncu, gs, w_cap, seg, nseg_out)) return 1;
  return 0;
}
