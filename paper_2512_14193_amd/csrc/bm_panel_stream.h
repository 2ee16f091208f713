// Panel factorisation by column streaming (included by bm_getrf.hip, which defines
// the exchange words and wave reductions used here).
//
// Workgroup g holds columns [g CW, (g + 1) CW) of the panel over all R rows, in
// registers (RPT rows per thread), so the search for a pivot, the exchange and the
// multipliers of a column never leave the workgroup: one barrier per column.  A
// finished column of multipliers goes to the exchange buffer as it is produced, and
// the workgroups of the later columns apply it as it arrives, one column behind the
// chain; only the first pivot search of a workgroup waits for another workgroup (a
// store and a load through memory, once per CW columns instead of twice per column).
//
// Rows are not moved.  A row keeps its register slot (slot r holds row j + r of the
// panel as it came); an extra wavefront of each workgroup, the clerk, follows the
// interchanges in LDS, which gives ties their order (smallest position first) and the
// rows their places at the end, keeps the rows of U and publishes the pivots.  A row
// that has been a pivot is final right of the diagonal: its entries move to LDS (s_u)
// and the row is marked (gone[]) for the search; the update runs over all rows with no
// test, and what it leaves in such a row is not used.
//
// What bounds a column is the length of its chain of dependent instructions, each a
// few cycles, so the search compares the high words of |Re| + |Im| only (an integer
// maximum).  Where two rows share the largest high word, or the largest is zero (values
// below 2^-1042), infinite or NaN, the column takes the exact search instead.  Measured
// per column: 0.65 us at 64 rows to 1.25 us at 2048 and 1.7 at 2688 (2.05 to 2.3 us with
// an exchange of candidates between workgroups of 64 or 128 rows), a hand-off between
// workgroups 0.5 to 1 us.
//
// Exchange words, each 16 bytes, written once with agent scope over the empty
// pattern and polled by the readers:
//   slots[c R + r]       multiplier of row slot r for column c
//   slots[SLOT_HDR + c]  {row slot of the pivot, zero-pivot flag, 0, 0}
#pragma once

// workgroup barrier for LDS traffic only (global stores stay in flight)
__device__ inline void spn_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// lane I of each row of 16 lanes, in every lane of the row
template <int I>
__device__ inline double row_bcast_f64(double v) {
  const long w = (long)__double_as_longlong(v);
  return __longlong_as_double(__builtin_amdgcn_update_dpp(0l, w, 0x150 + I, 0xf, 0xf, true));
}
// (every lane of these patterns has a source, so the move folds into the maximum)
template <int CTRL>
__device__ inline int dpp_max_i32(int v) {
  return max(v, __builtin_amdgcn_mov_dpp(v, CTRL, 0xf, 0xf, true));
}
// maximum over aligned groups of W = 2, 4, 8 or 16 lanes, and over the wavefront
template <int W>
__device__ inline int group_max_i32(int v) {
  if constexpr (W >= 2) v = dpp_max_i32<0xB1>(v);    // quad_perm [1,0,3,2]
  if constexpr (W >= 4) v = dpp_max_i32<0x4E>(v);    // quad_perm [2,3,0,1]
  if constexpr (W >= 8) v = dpp_max_i32<0x141>(v);   // row_half_mirror
  if constexpr (W >= 16) v = dpp_max_i32<0x140>(v);  // row_mirror
  return v;
}
__device__ inline int smax_i32(int a, int b) {
  int r;
  asm("s_max_i32 %0, %1, %2" : "=s"(r) : "s"(a), "s"(b) : "scc");
  return r;
}
__device__ inline int wave_max_i32(int v) {
  v = group_max_i32<16>(v);
  return smax_i32(smax_i32(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)),
                  smax_i32(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
}

// (i: a constant once the loop around it is unrolled)
__device__ __forceinline__ double row_bcast_at(double v, int i) {
  switch (i) {
    case 0: return row_bcast_f64<0>(v);
    case 1: return row_bcast_f64<1>(v);
    case 2: return row_bcast_f64<2>(v);
    case 3: return row_bcast_f64<3>(v);
    case 4: return row_bcast_f64<4>(v);
    case 5: return row_bcast_f64<5>(v);
    case 6: return row_bcast_f64<6>(v);
    case 7: return row_bcast_f64<7>(v);
    case 8: return row_bcast_f64<8>(v);
    case 9: return row_bcast_f64<9>(v);
    case 10: return row_bcast_f64<10>(v);
    case 11: return row_bcast_f64<11>(v);
    case 12: return row_bcast_f64<12>(v);
    case 13: return row_bcast_f64<13>(v);
    case 14: return row_bcast_f64<14>(v);
    default: return row_bcast_f64<15>(v);
  }
}

template <int NT, int RPT, int CW, class T, bool BAT>
__global__ __launch_bounds__(NT + 64) void panel_stream_kernel(int N, T *A, long lda, int j, int jb_, int G,
                                                               int32_t *ipiv, int32_t *dev_err, cplx *slots,
                                                               cplx *next_slots, long fill_n, int fill_h, int32_t *swp,
                                                               bm_lu_batch bb) {
  if constexpr (BAT) {
    const int b = blockIdx.y;
    A = (T *)bb.A[b];
    ipiv = bb.ipiv[b];
    dev_err = bb.err[b];
    slots = bb.cur[b];
    next_slots = bb.nxt[b];
    swp = bb.swp[b];
  }
  constexpr int NW = NT / 64;  // wavefronts that hold rows; wavefront NW is the clerk
  constexpr int NWP = (NW > 8) ? 16 : (NW > 4) ? 8 : NW;  // lanes that compare their candidates
  static_assert(CW <= 16 && (CW & (CW - 1)) == 0 && NW <= 16, "a pivot row lies in a row of 16 lanes");
  // only the last panel of a matrix (at most 64 rows) can have fewer than 64 columns
  constexpr bool FULL = NT * RPT > LU_NB;
  const int jb = FULL ? LU_NB : jb_;
  __shared__ st_v2 s_u[LU_NB][CW];        // U of these columns, by pivot
  __shared__ int4 s_h[2][NW];             // candidate of each wavefront: high word, row slot, how many have it,
  __shared__ st_v2 s_row[2][NW][CW + 1];  // its columns (and its first entry's reciprocal)
  __shared__ double s_hv[NW];
  __shared__ unsigned short s_pos[NT * RPT];  // position of each row slot
  __shared__ unsigned short s_at[LU_NB];      // row slot at each of the panel's first positions
  __shared__ int s_pick;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wave_of_lane = min(lane & (NWP - 1), NW - 1);
  const int g = (int)blockIdx.x, c0 = g * CW, R = N - j;
  const int nst = (FULL || c0 < jb) ? c0 : jb;  // columns of the earlier workgroups
  const __amdgpu_buffer_rsrc_t rs = rec_rsrc(slots);
  bool ok = true;
  auto expired = [&](unsigned long long &t0) __attribute__((always_inline)) {
    if (!ok) return true;
    if (t0 == 0) t0 = wall_clock64();
    if (!wait_expired(t0)) return false;
    atomicOr(dev_err, 1);
    ok = false;
    return true;
  };
  // The header of column t, the same address in every lane.  The lanes of one load can
  // see a word at different times, before and after it is written, so the compiler must
  // not take the loaded value for uniform (it would test any lane where every lane is
  // meant, and poll on without loading again): the offset is opaque to it.
  int zero_off;
  asm("v_mov_b32 %0, 0" : "=v"(zero_off));
  auto header = [&](int t) __attribute__((always_inline)) {
    return __builtin_amdgcn_raw_buffer_load_b128(rs, zero_off, (SLOT_HDR + t) * (int)sizeof(cplx), BM_CPOL_SC1);
  };
  // The winner of an own column among the wavefronts' candidates (buffer sb); false:
  // the exact search decides.
  struct pick {
    int ww, slot;
    bool fast;
  };
  auto winner = [&](int sb) __attribute__((always_inline)) {
    const int4 h = s_h[sb][wave_of_lane];
    const int hm = __builtin_amdgcn_readfirstlane(group_max_i32<NWP>(h.x));
    const unsigned mk = (unsigned)(__ballot(h.x == hm) & ((1ull << NW) - 1));
    pick o;
    o.ww = __ffs((int)mk) - 1;
    o.slot = __builtin_amdgcn_readlane(h.y, o.ww);
    const int nw = __builtin_amdgcn_readlane(h.z, o.ww);
    o.fast = ((mk & (mk - 1)) | (unsigned)(nw ^ 1) | ((unsigned)hm - 1u >= 0x7fefffffu ? 1u : 0u)) == 0;
    return o;
  };

  if (wave == NW) {
    // The clerk.  The row at position c of the panel takes the pivot row's position (every
    // lane alike).  The LDS reads of a step are used in the next one, when they have long
    // arrived.  (Positions >= jb hold their own row until it is a pivot, so s_at covers the
    // first jb positions only.)
    if (lane < LU_NB) s_at[lane] = (unsigned short)lane;
    int tk_c = -1, tk_slot = 0, tk_p = 0, tk_row = 0, mypiv = 0;
    auto track_end = [&]() __attribute__((always_inline)) {
      if (tk_c >= 0) {
        s_pos[tk_row] = (unsigned short)tk_p;
        s_pos[tk_slot] = (unsigned short)tk_c;
        if (tk_p < jb) s_at[tk_p] = (unsigned short)tk_row;
        s_at[tk_c] = (unsigned short)tk_slot;
        mypiv = (lane == tk_c) ? tk_p : mypiv;
        tk_c = -1;
      }
    };
    auto track = [&](int c, int slot) __attribute__((always_inline)) {
      track_end();
      tk_c = c;
      tk_slot = slot;
      tk_p = s_pos[slot];
      tk_row = s_at[c];
    };
    spn_barrier();  // (the rows' positions are written)
    if (g > 0) spn_barrier();  // (the rows' trial step)
    for (int t = 0; t < nst; ++t) {
      bm_v4i hw = header(t);
      unsigned long long t0 = 0;
      while (__any(rec_empty(hw)) && !expired(t0)) hw = header(t);
      const int slot = __builtin_amdgcn_readfirstlane(hw[0]);
      if (slot >= 0) track(t, slot);
      spn_barrier();
    }
#pragma unroll 1
    for (int q = 0; q < CW; ++q) {
      const int c = c0 + q, sb = q & 1;
      if (!FULL && c >= jb) break;
      spn_barrier();
      pick o = winner(sb);
      int zero = 0;
      if (!o.fast) {
        track_end();
        if (lane == 0) s_pick = 0x7fffffff;
        spn_barrier();
        zero = (wave_max_f64(s_hv[wave_of_lane]) > 0.0) ? 0 : 1;
        spn_barrier();
        o.slot = __builtin_amdgcn_readfirstlane(min(s_pick & 0xffff, NT * RPT - 1));
        o.ww = 0;
        spn_barrier();
      }
      if (lane == 0) {
        const bm_v4i hd = {o.slot, zero, 0, 0};
        __builtin_amdgcn_raw_buffer_store_b128(hd, rs, (SLOT_HDR + c) * (int)sizeof(cplx), 0, BM_CPOL_SC1);
      }
      if (lane < CW - q) s_u[c][q + lane] = s_row[sb][o.ww][lane];
      track(c, o.slot);
    }
    // the interchanges of the later columns, as they are decided; workgroup 0 also
    // records all of them (pivots, zero pivots, net permutation)
    int done = (c0 + CW < jb) ? c0 + CW : jb;
    unsigned long long t0 = 0, zeros = 0;
    while (done < jb || g == 0) {
      bm_v4i h = {0, 0, 0, 0};
      if (lane < jb) h = rec_load(rs, SLOT_HDR + lane);
      const unsigned long long em = __ballot(lane < jb && rec_empty(h));
      zeros = __ballot(lane < jb && h[0] >= 0 && h[1] != 0);
      const bool late = em != 0 && expired(t0);
      const int avail = (em && !late) ? (int)__ffsll((long long)em) - 1 : jb;
      for (; done < avail; ++done) {
        const int slot = __builtin_amdgcn_readlane(h[0], done);
        if (slot >= 0) track(done, slot);
      }
      if (done >= jb && (!em || late)) break;
      __builtin_amdgcn_s_sleep(2);
    }
    track_end();
    spn_barrier();
    if (g == 0) {
      // net permutation of the panel's interchanges on rows >= j: pairs (dst, src).  A
      // row that has left the first jb positions for good was one of theirs.
      const int at = (lane < jb) ? s_at[lane] : lane, ps = (lane < jb) ? s_pos[lane] : 0;
      const bool m1 = at != lane, m2 = ps >= jb;
      const unsigned long long b1 = __ballot(m1), b2 = __ballot(m2);
      const int n1 = __popcll(b1);
      const unsigned long long below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
      if (m1) {
        const int k = __popcll(b1 & below);
        swp[1 + 2 * k] = j + lane;
        swp[2 + 2 * k] = j + at;
      }
      if (m2) {
        const int k = n1 + __popcll(b2 & below);
        swp[1 + 2 * k] = j + ps;
        swp[2 + 2 * k] = j + lane;
      }
      if (lane == 0) swp[0] = n1 + __popcll(b2);
      if (lane < jb) ipiv[j + lane] = j + mypiv;
      if (lane == 0 && zeros && dev_err[1] == 0) dev_err[1] = j + (int)__ffsll((long long)zeros);
    }
    return;
  }

  st_v2 a[RPT][CW];
  int gone[RPT], off[RPT];  // sign bit: no candidate; byte offset of the row's exchange word in a column
  auto load = [&]() __attribute__((always_inline)) {
    int jc = j + c0;
    asm volatile("" : "+s"(jc));  // (the addresses are formed here, not held in registers from before)
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
      const int r = k * NT + tid;
      gone[k] = (r < R) ? 0 : (int)0x80000000;
#pragma unroll
      for (int q = 0; q < CW; ++q)
        a[k][q] = ld_z(A, (long)(j + ((r < R) ? r : 0)) + (long)((FULL || c0 + q < jb) ? jc + q : j) * lda);
    }
  };
#pragma unroll
  for (int k = 0; k < RPT; ++k) {
    const int r = k * NT + tid;
    s_pos[r] = (unsigned short)r;
    off[k] = 16 * ((r < R) ? r : R - 1);
  }
  spn_barrier();
  // a pivot row leaves the search (with_row(k) in the thread that holds it)
  auto retire = [&](unsigned slot, auto &&with_row) __attribute__((always_inline)) {
    if (slot % NT >> 6 == wave) {
#pragma unroll
      for (int k = 0; k < RPT; ++k)
        if (slot / NT == k && lane == (slot & 63)) {
          gone[k] = (int)0x80000000;
          with_row(k);
        }
    }
  };
  // column i less l times the pivot row (which every row of 16 lanes of `u` holds), into column i - s
  auto update = [&](int i, int s, const st_v2(&l)[RPT], st_v2 u) __attribute__((always_inline)) {
    const double ux = row_bcast_at(u.x, i), uy = row_bcast_at(u.y, i);
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
      const double x = fma(l[k].y, uy, fma(-l[k].x, ux, a[k][i].x));
      const double y = fma(-l[k].y, ux, fma(-l[k].x, uy, a[k][i].y));
      a[k][i - s] = st_v2{x, y};
    }
  };
  auto word = [&](int o, int t) __attribute__((always_inline)) {
    return __builtin_amdgcn_raw_buffer_load_b128(rs, o, t * R * (int)sizeof(cplx), BM_CPOL_SC1);
  };

  // Pass 0 is a trial step of the own-column loop on made-up rows, which writes nothing
  // anybody reads: it brings the loop's code into the instruction cache while the first
  // workgroup works (measured: 0.6 to 1.2 us per workgroup of the chain otherwise).
#pragma unroll 1
  for (int pass = (g == 0) ? 1 : 0; pass < 2; ++pass) {
    if (pass == 0) {
#pragma unroll
      for (int k = 0; k < RPT; ++k) {
        gone[k] = 0;
#pragma unroll
        for (int q = 0; q < CW; ++q) a[k][q] = st_v2{(k == 0 && tid == 0) ? 4.0 : 1.0, 0.0};
      }
    } else {
      load();
      // columns of the earlier workgroups, as they arrive
      bm_v4i hw, lw[RPT];
      auto fetch = [&](int t) __attribute__((always_inline)) {
        hw = header(t);
#pragma unroll
        for (int k = 0; k < RPT; ++k) lw[k] = word(off[k], t);
      };
      if (nst > 0) fetch(0);
#pragma unroll 1
      for (int t = 0; t < nst; ++t) {
        unsigned long long t0 = 0;
        for (;;) {
          bool need = rec_empty(hw);
#pragma unroll
          for (int k = 0; k < RPT; ++k) need = need || rec_empty(lw[k]);
          if (!__any(need) || expired(t0)) break;
          if (rec_empty(hw)) hw = header(t);
#pragma unroll
          for (int k = 0; k < RPT; ++k)
            if (rec_empty(lw[k])) lw[k] = word(off[k], t);
        }
        const int slot = __builtin_amdgcn_readfirstlane(hw[0]);  // (-1 after an expired wait: no row)
        st_v2 l[RPT];
#pragma unroll
        for (int k = 0; k < RPT; ++k) l[k] = to_v2(rec_value(lw[k]));
        if (t + 1 < nst) fetch(t + 1);
        // the pivot row's entries of these columns, from the thread that holds the row
        if (slot >= 0)
          retire(slot, [&](int k) __attribute__((always_inline)) {
#pragma unroll
            for (int q = 0; q < CW; ++q) s_u[t][q] = a[k][q];
          });
        spn_barrier();
        const st_v2 u = s_u[t][lane & (CW - 1)];
#pragma unroll
        for (int q = 0; q < CW; ++q) update(q, 0, l, u);
      }
      // every load has arrived: no wait for one inside the loop, which would wait for the
      // stores of the multipliers as well (vmcnt(0), the other counters left alone)
      __builtin_amdgcn_s_waitcnt(0x0F70);
    }
    // The workgroup's own columns.  One loop body for all of them (straight-line code
    // for each would run cold): the update shifts the columns left, so that the current
    // one is always a[.][0].
#pragma unroll 1
    for (int q = 0; q < CW; ++q) {
      const int c = c0 + q, sb = q & 1, left = CW - q;  // columns left, this one included
      if (!FULL && c >= jb) break;
      // the wavefront's largest high word and the rows that have it
      int hk[RPT], hi = (int)0x80000000;
#pragma unroll
      for (int k = 0; k < RPT; ++k) {
        hk[k] = __double2hiint(fabs(a[k][0].x) + fabs(a[k][0].y)) | gone[k];
        hi = max(hi, hk[k]);
      }
      // (with one row per thread the reciprocal is taken beside the search)
      cplx ip = cmk(0, 0);
      if (RPT == 1) {
        ip = pivot_recip(cmk(a[0][0].x, a[0][0].y));
        asm volatile("" : "+v"(ip.x), "+v"(ip.y));
      }
      const int him = wave_max_i32(hi);
      int nh = 0;
#pragma unroll
      for (int k = 0; k < RPT; ++k) nh += __popcll(__ballot(hk[k] == him));
#pragma unroll
      for (int k = 0; k < RPT; ++k)
        if (hk[k] == him) {
          s_h[sb][wave] = make_int4(him, k * NT + tid, nh, 0);
#pragma unroll
          for (int i = 0; i < CW; ++i) s_row[sb][wave][i] = a[k][i];
          if (RPT == 1) s_row[sb][wave][CW] = st_v2{ip.x, ip.y};
        }
      spn_barrier();
      pick o = winner(sb);
      bool zero = false;
      if (!o.fast && pass > 0) {
        // the exact search: largest value that compares, then smallest position (by the
        // clerk's table).  A column of NaNs keeps the row at its position.
        double v = -1.0;
#pragma unroll
        for (int k = 0; k < RPT; ++k) {
          const double w = fabs(a[k][0].x) + fabs(a[k][0].y);
          if (gone[k] >= 0 && w > v) v = w;
        }
        v = wave_max_f64(v);
        if (lane == 0) s_hv[wave] = v;
        spn_barrier();
        const double vm = wave_max_f64(s_hv[wave_of_lane]);
        int best = 0x7fffffff;
#pragma unroll
        for (int k = 0; k < RPT; ++k) {
          const double w = fabs(a[k][0].x) + fabs(a[k][0].y);
          const int ps = s_pos[k * NT + tid];
          if ((vm < 0.0) ? ps == c : (gone[k] >= 0 && w == vm)) best = min(best, (ps << 16) | (k * NT + tid));
        }
        if (best != 0x7fffffff) atomicMin(&s_pick, best);
        spn_barrier();
        o.slot = __builtin_amdgcn_readfirstlane(min(s_pick & 0xffff, NT * RPT - 1));
        o.ww = 0;
        zero = !(vm > 0.0);
#pragma unroll
        for (int k = 0; k < RPT; ++k)
          if (k * NT + tid == o.slot) {
#pragma unroll
            for (int i = 0; i < CW; ++i) s_row[sb][0][i] = a[k][i];
            if (RPT == 1) s_row[sb][0][CW] = st_v2{ip.x, ip.y};
          }
        spn_barrier();
      }
      const st_v2 u = s_row[sb][o.ww][lane & (CW - 1)];
      if (RPT == 1) {
        const st_v2 ipv = s_row[sb][o.ww][CW];
        ip = cmk(ipv.x, ipv.y);
      } else {
        const st_v2 u0 = s_row[sb][o.ww][0];
        ip = pivot_recip(cmk(u0.x, u0.y));
      }
      if (zero) ip = cmk(0, 0);
      st_v2 l[RPT];
#pragma unroll
      for (int k = 0; k < RPT; ++k) l[k] = to_v2(cmul(cmk(a[k][0].x, a[k][0].y), ip));
      if (pass > 0) {
#pragma unroll
        for (int k = 0; k < RPT; ++k) {
          bm_v4i z;
          z[0] = __double2loint(l[k].x);
          z[1] = __double2hiint(l[k].x);
          z[2] = __double2loint(l[k].y);
          z[3] = __double2hiint(l[k].y);
          // (rows past R: beside the words in use)
          __builtin_amdgcn_raw_buffer_store_b128(z, rs, 16 * (k * NT + tid) + ((k * NT + tid < R) ? 0 : 16 * LU_NB * R),
                                                 c * R * (int)sizeof(cplx), BM_CPOL_SC1);
        }
      }
      // (columns past the last one hold nothing any more)
      constexpr int H1 = (CW >= 8) ? CW / 4 : CW / 2, H2 = CW / 2;
#pragma unroll
      for (int i = 1; i < H1; ++i) update(i, 1, l, u);
      if (left > H1) {
#pragma unroll
        for (int i = (H1 > 1 ? H1 : 1); i < (H2 > H1 ? H2 : CW); ++i) update(i, 1, l, u);
      }
      if (H2 > H1 && left > H2) {
#pragma unroll
        for (int i = H2; i < CW; ++i) update(i, 1, l, u);
      }
      retire(o.slot, [](int) {});
      if (pass == 0) break;
    }
  }

  // refill the words the next panel uses in the other buffer with the empty pattern:
  // the workgroups before the last share it, which have done their columns
  const int nfill = (G > 1) ? G - 1 : 1;
  if (g < nfill) slots_refill(next_slots, fill_n, fill_h, g * NT + tid, nfill * NT);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this thread's multipliers have reached memory
  spn_barrier();                                    // the clerk has every position

  // entries right of the diagonal of a pivot row are in LDS, the multipliers in the
  // exchange buffer, where this thread wrote them
#pragma unroll
  for (int k = 0; k < RPT; ++k) {
    const int r = k * NT + tid;
    if (r < R) {
      bm_v4i z[CW];
#pragma unroll
      for (int q = 0; q < CW; ++q) z[q] = word(off[k], (FULL || c0 + q < jb) ? c0 + q : 0);
      const int ps = s_pos[r];
#pragma unroll
      for (int q = 0; q < CW; ++q)
        if (FULL || c0 + q < jb) {
          const bool up = ps <= c0 + q;
          const st_v2 u = s_u[up ? ps : 0][q], m = to_v2(rec_value(z[q]));
          st_z(A, (long)(j + ps) + (long)(j + c0 + q) * lda, st_v2{up ? u.x : m.x, up ? u.y : m.y});
        }
    }
  }
}
