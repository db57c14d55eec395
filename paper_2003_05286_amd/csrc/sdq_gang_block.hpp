// sdq_gang_block.hpp -- the blocked QR of the gang kernels, included by
// sdq_gang.hip.
//
// The pivoted QR of a gang pays one exchange between its workgroups per
// column, 8 us at n = 256 and 19 us at n = 1024.  The stabilized chains and the
// middle matrices do not need pivoting in every step (see sdq_block.hpp: sort
// by norm, test, repeat), so the members exchange once per 16-column panel:
// the member that holds it factors the panel with four to sixteen waves (each
// holds every fourth .. sixteenth row tile; the dot products of a step meet in
// LDS, one workgroup barrier per column), publishes reflectors and triangular
// factor through coherent stores and one flag, and every member applies them to
// its own columns on MFMA.
//
// Bound by the chain of panels: 28 k cycles to factor and publish one at n =
// 256 (16.7 k in its 16 steps, 9 k storing), 20 k for the next owner to apply
// it.  Against a pivot per column: sweeps 237 -> 92 ms at n = 256 (64 chains)
// and 459 -> 158 at n = 1024, pairs 161 -> 34 and 129 -> 14.
//
// Published per panel p, in the gang's scratch: the reflectors (su on the
// diagonal, zero above) as row-major 16-column rows and once more in the
// operand order of V X, Tw [16][16], su[16] and R's diagonal [16].

// (4 and 2 give the same errors from n = 144 on, and fewer blocks repeat the sort)
constexpr double kGangSortedGrowth = 4.0;
constexpr int kApplyTiles = 5;  // row tiles per wave of a panel application, at most

// The exchange area of a panel application or of a triangular solve: six
// 16 x 16 slots behind the slab where they fit, else the four of L.xbuf.
__host__ __device__ constexpr bool slots_in_slab(const GangGeom& g) { return g.w * g.ldr + 6 * 256 <= kGangSlab; }
// That area and kApplyTiles hold for every size: nct column tiles of a member
// share the waves, and a wave's tiles and the slots (four for one or two
// column tiles, else one each) follow.
constexpr bool gang_blocks_fit() {
  for (int nt = kMaxNT + 1; nt <= kGangMaxN / 16; ++nt) {
    const GangGeom g = gang_geom(nt);
    if (g.G == 0) return false;
    for (int nct = 1; nct <= g.w / 16; ++nct) {
      const int ks = kWaves / nct, slots = nct <= 2 ? 4 : nct;
      if (ks * kApplyTiles < nt && nct == g.w / 16) return false;
      if (slots > (slots_in_slab(g) ? 6 : 4)) return false;
    }
  }
  return true;
}
static_assert(gang_blocks_fit(), "a panel application's tiles and exchange slots");

struct GPanel {
  double* v1;
  double* v2;
  double* tw;
  double* meta;
};
__device__ __forceinline__ GPanel panel_at(const GC& c, int p) {
  const int64_t np = c.geo.npad;
  GPanel a;
  a.v1 = sc_V(c) + p * np * 16;
  a.v2 = sc_V2(c) + p * np * 16;
  a.tw = sc_tw(c) + (int64_t)p * 256;
  a.meta = sc_meta(c) + (int64_t)p * 32;
  return a;
}

// coherent 8-byte load at a wave-uniform base plus a 32-bit lane offset
// (doubles): see ld_coh_col
__device__ __forceinline__ __amdgpu_buffer_rsrc_t uniform_rsrc(const double* p, int doubles) {
  const unsigned long long a = (unsigned long long)p;
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)a);
  const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(a >> 32));
  return __builtin_amdgcn_make_buffer_rsrc((void*)(((unsigned long long)hi << 32) | lo), (short)0, doubles * 8,
                                           0x00020000);
}
template <bool COH>
__device__ __forceinline__ double ld_buf(__amdgpu_buffer_rsrc_t rs, int lane_off, int off) {
  return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rs, lane_off * 8, off * 8, COH ? 16 : 0));
}

__device__ __forceinline__ Lane gang_lane(const GC& c) {
  Lane ln;
  int t = c.t;
  asm volatile("" : "+v"(t));
  ln.t = t;
  ln.w = __builtin_amdgcn_readfirstlane(t >> 6);
  ln.l = t & 63;
  ln.g = ln.l >> 4;
  ln.cl = ln.l & 15;
  return ln;
}

// The 16 steps of a panel over 4 NW4 waves of one workgroup; wave v holds the
// row tiles v, v + 4 NW4, ... counted from the diagonal one (wave 0's first).
// As panel_qr, but a step's dot products and row J go through LDS, and the
// last wave leaves the products v_J^T v_c (c < J) and the scalar c_J in L.gram
// for the triangular factor (in registers it would not fit beside the rows).
template <int RT, int NW4>
__device__ __forceinline__ void gang_panel_steps(const Lane& ln, double (&b)[RT][4], double& hs_l) {
  const int v = ln.w;
  hs_l = 0.0;
  static_for<16>([&](auto jc) {
    constexpr int J = decltype(jc)::value, R0 = J >> 2, G0 = J & 3;
    double p = 0.0;
    if (v == 0) {
      dot_head<J, RT>(p, b);
    } else if constexpr (RT == 4) {
      dot_tiles<J>(p, b[0], b[1], b[2], b[3]);
    } else {
#pragma unroll
      for (int t = 0; t < RT; ++t) dot_tiles<J>(p, b[t]);
    }
    const double ws = sum_col(p);
    double* pr = L.pred + (J & 1) * (17 * 16);
    if (ln.g == 0) pr[v * 16 + ln.cl] = ws;
    if (v == 0 && ln.g == G0) pr[256 + ln.cl] = b[0][R0];
    __syncthreads();
    double a = pr[ln.g * 16 + ln.cl];
#pragma unroll
    for (int i = 1; i < NW4; ++i) a += pr[(ln.g + 4 * i) * 16 + ln.cl];
    const double ajc = pr[256 + ln.cl];
    const double dot = sum_col(a);
    const double s = bcast_col<J>(dot), alpha = bcast_col<J>(ajc);
    const double q = fma(alpha, alpha, s);
    const double r0 = __builtin_amdgcn_rsq(q);
    double h = q * r0;
    const double hr = 0.5 * r0;
    h = fma(h, fma(-hr, h, 0.5), h);
    h = fma(fma(-h, h, q), hr, h);
    const double hs = copysign(h, alpha);
    const double su = alpha + hs;
    const double c = rcp_mid(0.5 * fma(su, su, s));
    const double d = fma(su, ajc, dot);
    const double cd = -c * d;
    const double f = __hiloint2double(ln.cl > J ? __double2hiint(cd) : 0, __double2loint(cd));
    if (v == 0) {
      axpy_head<J, RT>(b, su, f);
      static_for<(RT > 2 ? RT - 2 : 0) / 2>([&](auto tc) {
        constexpr int t = 2 + 2 * decltype(tc)::value;
        axpy_tiles<J>(b[t], b[t + 1], f);
      });
    } else {
      if constexpr (RT % 2 == 1) axpy_tiles<J>(b[0], f);
      static_for<RT / 2>([&](auto tc) {
        constexpr int t = RT % 2 + 2 * decltype(tc)::value;
        axpy_tiles<J>(b[t], b[t + 1], f);
      });
    }
    hs_l = ln.cl == J ? hs : hs_l;
    if (v == 4 * NW4 - 1 && ln.g == 0) L.gram[J * 16 + ln.cl] = ln.cl == J ? c : d;
  });
}

// The panel whose steps left the range of a double's squares, from the slab,
// which still holds its columns (panel_careful; wave 0 alone).  The triangular
// factor in the half of L.pred that the last step does not use: another wave
// may still be reading its own half and writing L.gram.
__device__ __attribute__((noinline)) void gang_panel_careful(const GC& c, int p) {
  const Lane ln = gang_lane(c);
  const int rows = c.geo.npad - 16 * p, ldr = c.geo.ldr;
  double* col = L.S + (16 * p - c.c0) * ldr + 16 * p;
  const CarefulDiag cd = panel_careful<false>(col, L.pred, rows, ldr);
  const double su = cd.su_l, beta = cd.beta_l;
  const GPanel g = panel_at(c, p);
  if (ln.g == 0) {
    st_coh(g.meta + ln.cl, su);
    st_coh(g.meta + 16 + ln.cl, beta);
  }
#pragma unroll 1
  for (int i = ln.g; i < rows; i += 4) {
    const double x = col[ln.cl * ldr + i], v = i > ln.cl ? x : (i == ln.cl ? su : 0.0);
    const int rt = p + (i >> 4), row = i & 15;
    st_coh(g.v1 + rt * 256 + row * 16 + ln.cl, v);
    st_coh(g.v2 + rt * 256 + (ln.cl >> 2) * 64 + (ln.cl & 3) * 16 + row, v);
    if (i < 16) {
      st_coh(g.tw + ln.cl * 16 + i, L.pred[ln.cl * 16 + i]);
      if (i > ln.cl) col[ln.cl * ldr + i] = 0.0;
    }
  }
}

// Factor panel p (in this member's slab) and write it to the gang's scratch;
// the slab keeps R's diagonal tile.  Every wave of the workgroup calls it.
// Not inlined: the inline assembly's operands must not be spilled, and the
// callers keep much alive.
template <int RT, int NW4>
__device__ __attribute__((noinline)) void gang_panel(const GC& c, int p) {
  const Lane ln = gang_lane(c);
  constexpr int NW = 4 * NW4;
  const int nrt = c.geo.npad / 16, cnt = nrt - p, ldr = c.geo.ldr;
  __syncthreads();  // L.pred is free
  if (ln.w >= NW) {
#pragma unroll 1
    for (int j = 0; j < 16; ++j) __syncthreads();
    return;
  }
  double* col = L.S + (16 * p - c.c0 + ln.cl) * ldr + 16 * p;
  double b[RT][4], hs_l;
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    const int rt = ln.w + NW * t;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const double x = col[16 * min(rt, cnt - 1) + ln.g + 4 * r];
      b[t][r] = rt < cnt ? x : 0.0;
    }
  }
  gang_panel_steps<RT, NW4>(ln, b, hs_l);
  if (!plain_panel(hs_l)) {  // the same numbers in every wave
    if (ln.w == 0) gang_panel_careful(c, p);
    __builtin_amdgcn_s_waitcnt(0);
    return;
  }
  const GPanel g = panel_at(c, p);
  if (ln.w == 0) {
    double al = 0.0;
#pragma unroll
    for (int r = 0; r < 4; ++r) al = ln.g + 4 * r == ln.cl ? b[0][r] : al;
    const double su = sum_col(al) + hs_l;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = ln.g + 4 * r;
      col[row] = row < ln.cl ? b[0][r] : (row == ln.cl ? -hs_l : 0.0);
      b[0][r] = row > ln.cl ? b[0][r] : (row == ln.cl ? su : 0.0);
    }
    if (ln.g == 0) {
      st_coh(g.meta + ln.cl, su);
      st_coh(g.meta + 16 + ln.cl, -hs_l);
    }
  }
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    const int rt = p + ln.w + NW * t;
    if (rt < nrt) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = ln.g + 4 * r;
        st_coh(g.v1 + rt * 256 + row * 16 + ln.cl, b[t][r]);
        st_coh(g.v2 + rt * 256 + (ln.cl >> 2) * 64 + (ln.cl & 3) * 16 + row, b[t][r]);
      }
    }
  }
  if (ln.w == NW - 1) {
    double T[16];
    static_for<16>([&](auto jc) {
      constexpr int J = decltype(jc)::value;
      const double d = L.gram[J * 16 + ln.cl];
      const double c = bcast_col<J>(d);
      const double ts = tri_dot<J>(d, T);
      T[J] = ln.cl == J ? c : -c * ts;
    });
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (ln.g == q) {
#pragma unroll
        for (int e = 0; e < 4; ++e) st_coh(g.tw + ln.cl * 16 + 4 * q + e, T[4 * q + e]);
      }
  }
  __builtin_amdgcn_s_waitcnt(0);  // at the coherence point before the flag
}

// Wait until panel number seq (counted over the launch) is published; false
// when the gang is broken (as wait_keys).
__device__ void wait_panel(GC& c, unsigned seq) {
  if (c.t == 0) {
    int good = 1;
    const unsigned long long t0 = wall_clock64();
    for (;;) {
      if (!c.ok) break;
      if (__hip_atomic_load(gmem(&c.bar[8]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= seq) break;
      if (__hip_atomic_load(gmem(&c.bar[1]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u) {
        good = 0;
        break;
      }
      if (wall_clock64() - t0 > kSpinTicks) {
        __hip_atomic_exchange(gmem(&c.bar[1]), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        good = 0;
        break;
      }
    }
    L.ok = good;
  }
  __syncthreads();
  c.ok = c.ok && L.ok != 0;
  __syncthreads();
}

// C <- Q_p^T C (QT) or Q_p C for the member's column tiles from ct_lo on.
// The 16 waves split into ks per column tile; each takes every ks-th row tile
// from p on, reads its share of the reflectors at once, and keeps to these
// tiles of the slab in both products, so that only the 16 x 16 products
// X = V^T C meet: ks parts are summed in a fixed order over up to four LDS
// slots per column tile, a barrier per round.  Ends with a barrier.  Some 20 k
// cycles at n = 256, 4 k of them in each product (four waves a SIMD); with the
// second product's operands loaded before the sums, and tiles beyond the
// panel's too, it took 25 k.
template <bool QT, bool COH>
__device__ __attribute__((noinline)) void gang_apply(const GC& c, int p, int ct_lo) {
  const Lane ln = gang_lane(c);
  const int nrt = c.geo.npad / 16, cnt = nrt - p, ldr = c.geo.ldr;
  const int nct_all = min(c.geo.w / 16, nrt - c.c0 / 16);  // column tiles inside the matrix
  const int nct = nct_all - ct_lo;
  if (nct <= 0) return;  // the same for the whole workgroup
  const int ks = kWaves / nct, sl = nct == 1 ? 4 : (nct == 2 ? 2 : 1);
  const int rounds = (ks + sl - 1) / sl;
  const int cti = ln.w / ks, part = ln.w - cti * ks;
  const bool on = cti < nct;
  const GPanel g = panel_at(c, p);
  const __amdgpu_buffer_rsrc_t r1 = uniform_rsrc(g.v1, nrt * 256), r2 = uniform_rsrc(g.v2, nrt * 256),
                               rt_ = uniform_rsrc(g.tw, 256);
  double* xb = slots_in_slab(c.geo) ? L.S + c.geo.w * ldr : L.xbuf;
  double* col = L.S + (16 * (ct_lo + min(cti, nct - 1)) + ln.cl) * ldr + 16 * p + ln.g;
  double tv[4], a[kApplyTiles][4];
  d4 x = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int i = 0; i < kApplyTiles; ++i)
    if (part + ks * i < cnt) {
#pragma unroll
      for (int r = 0; r < 4; ++r) a[i][r] = ld_buf<COH>(r1, ln.g * 16 + ln.cl + (p + part + ks * i) * 256, r * 64);
    }
#pragma unroll
  for (int r = 0; r < 4; ++r)
    tv[r] = ld_buf<COH>(rt_, QT ? (ln.g + 4 * r) * 16 + ln.cl : ln.cl * 16 + ln.g + 4 * r, 0);
  // X = V^T C, a tile's operand of the second product loaded behind its first
  // (a barrier waits for every load: issued after this loop they would all be
  // waited for in the first round of sums)
#pragma unroll
  for (int i = 0; i < kApplyTiles; ++i) {
    const int k = part + ks * i;
    if (k < cnt) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if (on) x = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i][r], col[16 * k + 4 * r], x, 0, 0, 0);
        a[i][r] = ld_buf<COH>(r2, ln.l + (p + k) * 256, r * 64);
      }
    }
  }
  double* slot = xb + ((on ? cti : 0) * sl + part % sl) * 256 + ln.l;
  for (int rd = 0; rd < rounds; ++rd) {
    if (on && part / sl == rd) {
#pragma unroll
      for (int r = 0; r < 4; ++r) slot[64 * r] = rd == 0 ? x[r] : slot[64 * r] + x[r];
    }
    __syncthreads();
  }
  if (on) {
    const int used = min(sl, ks);
    const double* xs = xb + cti * sl * 256 + ln.l;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      double s = xs[64 * r];
      for (int u = 1; u < used; ++u) s += xs[u * 256 + 64 * r];
      x[r] = s;
    }
    d4 x2 = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int r = 0; r < 4; ++r) x2 = __builtin_amdgcn_mfma_f64_16x16x4f64(tv[r], x[r], x2, 0, 0, 0);
#pragma unroll
    for (int r = 0; r < 4; ++r) x2[r] = -x2[r];
#pragma unroll
    for (int i = 0; i < kApplyTiles; ++i) {
      const int k = part + ks * i;
      if (k < cnt) {
        d4 acc = d4{col[16 * k], col[16 * k + 4], col[16 * k + 8], col[16 * k + 12]};
#pragma unroll
        for (int r = 0; r < 4; ++r) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i][r], x2[r], acc, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) col[16 * k + 4 * r] = acc[r];
      }
    }
  }
  __syncthreads();
}

// C <- Q_p^T C as gang_apply, one reflector at a time (see panel_steps): each
// reflector's products with the columns are summed over the waves of a column
// tile through LDS, one barrier a reflector.
__device__ __attribute__((noinline)) void gang_apply_steps(const GC& c, int p, int ct_lo) {
  const Lane ln = gang_lane(c);
  const int nrt = c.geo.npad / 16, cnt = nrt - p, ldr = c.geo.ldr;
  const int nct = min(c.geo.w / 16, nrt - c.c0 / 16) - ct_lo;
  if (nct <= 0) return;  // the same for the whole workgroup
  const int ks = kWaves / nct, cti = ln.w / ks, part = ln.w - cti * ks;
  const bool on = cti < nct;
  const GPanel g = panel_at(c, p);
  const __amdgpu_buffer_rsrc_t r1 = uniform_rsrc(g.v1, nrt * 256), rt_ = uniform_rsrc(g.tw, 256);
  double* col = L.S + (16 * (ct_lo + min(cti, nct - 1)) + ln.cl) * ldr + 16 * p + ln.g;
  double a[kApplyTiles][4], x[kApplyTiles][4];
  const double cd = ld_buf<true>(rt_, ln.cl * 16 + ln.cl, 0);
#pragma unroll
  for (int i = 0; i < kApplyTiles; ++i) {
    const int k = min(part + ks * i, cnt - 1);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      a[i][r] = ld_buf<true>(r1, ln.g * 16 + ln.cl + (p + k) * 256, r * 64);
      x[i][r] = col[16 * k + 4 * r];
    }
  }
#pragma unroll
  for (int i = 0; i < kApplyTiles; ++i)
    if (!(on && part + ks * i < cnt)) {
#pragma unroll
      for (int r = 0; r < 4; ++r) a[i][r] = x[i][r] = 0.0;
    }
  rows_landed<kApplyTiles>(x);
  static_for<16>([&](auto jc) {
    constexpr int J = decltype(jc)::value;
    double* pr = L.xbuf + (J & 1) * 256;
    const double q = sum_col(dot_rows<J>(a, x));
    if (ln.g == 0) pr[ln.w * 16 + ln.cl] = q;
    __syncthreads();
    double s = 0.0;
    for (int u = ln.g; u < ks; u += 4) s += pr[(min(cti, nct - 1) * ks + u) * 16 + ln.cl];
    const double f = -bcast_col<J>(cd) * sum_col(s);
    axpy_rows<J>(x, a, f);
  });
#pragma unroll
  for (int i = 0; i < kApplyTiles; ++i)
    if (on && part + ks * i < cnt) {
#pragma unroll
      for (int r = 0; r < 4; ++r) col[16 * (part + ks * i) + 4 * r] = x[i][r];
    }
  __syncthreads();
}

// Unit vectors in the padding columns of the slab (inside npad).
__device__ void slab_pad_unit(const GC& c) {
  const int np = c.geo.npad, n = c.n;
  for (int idx = c.t; idx < np * c.geo.w; idx += kGangThreads) {
    const int cc = idx / np, i = idx - cc * np, gc = c.c0 + cc;
    if (gc >= n && gc < np) L.S[cc * c.geo.ldr + i] = i == gc ? 1.0 : 0.0;
  }
  __syncthreads();
}

// The slab's matrix = Q R, columns as they stand: panels in the gang's
// scratch, diag R in L.beta, R (column-major, npad x npad, zero below the
// diagonal) in sc_R, visible to the gang.  Returns whether |R_ic| cs_c <=
// growth |R_ii| cs_i everywhere (cs: L.tau; NaN fails; test = false: always).
// A panel is published into scratch that the factorization before it used too,
// so every member has to be done with that one (bsolve_gang, bform_gang read
// its panels and R) before the first panel here is written.  The sort that
// precedes a tested factorization exchanges columns after that; without it the
// members meet here: a gang takes the middle matrices of many items in a row,
// and nothing else holds a member back that has finished its own columns first.
__device__ bool bqr_gang(GC& c_io, bool test) {
  GC c = c_io;
  const int nrt = c.geo.npad / 16, np = c.geo.npad, n = c.n, ldr = c.geo.ldr;
  if (!test) gang_sync(c);
  slab_pad_unit(c);
#pragma unroll 1
  for (int p = 0; p < nrt; ++p) {
    const int owner = 16 * p / c.geo.w, cnt = nrt - p;
    const unsigned seq = ++c.pseq;
    if (c.g == owner) {
      if (cnt <= 4) gang_panel<1, 1>(c, p);
      else if (cnt <= 8) gang_panel<2, 1>(c, p);
      else if (cnt <= 16) gang_panel<4, 1>(c, p);
      else if (cnt <= 32) gang_panel<4, 2>(c, p);
      else gang_panel<4, 4>(c, p);
      __syncthreads();
      if (c.t == 0) __hip_atomic_store(gmem(&c.bar[8]), seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else {
      wait_panel(c, seq);
    }
    if (c.t < 16) {
      const GPanel g = panel_at(c, p);
      L.beta[16 * p + c.t] = __longlong_as_double((long long)ld_coh_u64(g.meta + 16 + c.t));
    }
    // column tiles right of the panel
    const int ct_lo = max(0, p + 1 - c.c0 / 16);
    if (test && p < kStepPanels) gang_apply_steps(c, p, ct_lo);
    else gang_apply<true, true>(c, p, ct_lo);
  }
  __syncthreads();
  int bad = 0;
  {
    double* R = sc_R(c);
    for (int idx = c.t; idx < np * c.geo.w; idx += kGangThreads) {
      const int cc = idx / np, i = idx - cc * np, gc = c.c0 + cc;
      if (gc >= np) continue;
      const double x = i <= gc ? L.S[cc * ldr + i] : 0.0;
      if (test && i < gc && gc < n && !(fabs(x) * L.tau[gc] <= kGangSortedGrowth * fabs(L.beta[i]) * L.tau[i])) bad = 1;
      gmem(R)[(int64_t)gc * np + i] = x;
    }
  }
  if (test && __any(bad) && c.l == 0)
    __hip_atomic_fetch_add(gmem(&c.bar[9]), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  gang_sync(c);
  bool fine = true;
  if (test) {
    if (c.t == 0) L.vote = __hip_atomic_load(gmem(&c.bar[9]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    const unsigned v = L.vote;
    fine = v == c.votes || !c.ok;
    c.votes = v;
    __syncthreads();
  }
  c_io = c;
  return fine;
}

// The slab's columns <- Q (slab), where the slab holds unit vectors or columns
// that vanish below their own panel (so that panels right of a column tile
// leave it alone).
__device__ void bform_gang(const GC& c) {
  const int nrt = c.geo.npad / 16;
#pragma unroll 1
  for (int p = min(nrt - 1, (c.c0 + c.geo.w) / 16 - 1); p >= 0; --p)
    gang_apply<false, false>(c, p, max(0, p - c.c0 / 16));
}

// Column tile w of row tile p: z = R_pp^{-1} y, to the slab and, negated, to
// exchange slot w.
__device__ __attribute__((noinline)) void gang_tri_solve(const GC& c, int p, double* xb) {
  const Lane ln = gang_lane(c);
  const int np = c.geo.npad, ldr = c.geo.ldr;
  const auto* dg = gmem(sc_R(c)) + (int64_t)16 * p * np + 16 * p;
  double rr[16][4];
#pragma unroll
  for (int j = 0; j < 16; ++j)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (4 * r <= j) rr[j][r] = dg[(int64_t)j * np + ln.g + 4 * r];
  const double ri = 1.0 / L.beta[16 * p + ln.cl];
  double* col = L.S + (16 * ln.w + ln.cl) * ldr + 16 * p + ln.g;
  double z[4] = {col[0], col[4], col[8], col[12]};
  static_for<16>([&](auto jc) {
    constexpr int J = 15 - decltype(jc)::value, R0 = J >> 2, G0 = J & 3;
    const double zj = bcast_row<G0>(z[R0]) * bcast_col<J>(ri);
#pragma unroll
    for (int r = 0; r <= R0; ++r) {
      if (r < R0) z[r] = fma(-rr[J][r], zj, z[r]);
      else z[r] = ln.g < G0 ? fma(-rr[J][r], zj, z[r]) : (ln.g == G0 ? zj : z[r]);
    }
  });
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    col[4 * r] = z[r];
    xb[ln.w * 256 + 64 * r + ln.l] = -z[r];
  }
}

// slab <- R^{-1} Q^T slab for the last bqr_gang.  The back substitution goes
// from the last row tile up: one wave per column tile solves the diagonal tile
// (z to the slab and, negated, to the exchange slots), then all waves take the
// tile out of the rows above on MFMA.
__device__ void bsolve_gang(const GC& c) {
  const int nrt = c.geo.npad / 16, np = c.geo.npad, ldr = c.geo.ldr;
#pragma unroll 1
  for (int p = 0; p < nrt; ++p) gang_apply<true, false>(c, p, 0);
  const int nct = min(c.geo.w / 16, nrt - c.c0 / 16);
  if (nct <= 0) return;
  double* xb = slots_in_slab(c.geo) ? L.S + c.geo.w * ldr : L.xbuf;
  const int ks = kWaves / nct;
#pragma unroll 1
  for (int p = nrt - 1; p >= 0; --p) {
    const Lane ln = gang_lane(c);
    const double* R = sc_R(c) + (int64_t)16 * p * np;  // columns 16 p ..
    if (ln.w < nct) gang_tri_solve(c, p, xb);
    __syncthreads();
    const int cti = ln.w / ks, part = ln.w - cti * ks;
    if (cti < nct) {
      double z[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) z[r] = xb[cti * 256 + 64 * r + ln.l];
      double* col = L.S + (16 * cti + ln.cl) * ldr + ln.g;
      for (int rt = part; rt < p; rt += ks) {
        double a[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) a[r] = gmem(R)[(int64_t)(ln.g + 4 * r) * np + 16 * rt + ln.cl];
        d4 acc = d4{col[16 * rt], col[16 * rt + 4], col[16 * rt + 8], col[16 * rt + 12]};
#pragma unroll
        for (int r = 0; r < 4; ++r) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[r], z[r], acc, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) col[16 * rt + 4 * r] = acc[r];
      }
    }
    __syncthreads();
  }
}

// Sort the slab's columns by descending key (own columns' keys and scales in
// L.vn1 / L.vn2): the columns move between the members through the scratch.
// On return L.piv[i] = the original column at place i (composed with the
// earlier passes' when pass > 0), L.tau[i] = the scale at place i.
__device__ void sort_gang(GC& c, int pass) {
  const int n = c.n, np = c.geo.npad, ldr = c.geo.ldr;
  double* keys = sc_keys(c);
  double* scales = keys + np;
  for (int cc = c.t; cc < c.geo.w; cc += kGangThreads) {
    const int gc = c.c0 + cc;
    if (gc < n) {
      gmem(keys)[gc] = L.vn1[cc];
      gmem(scales)[gc] = L.vn2[cc];
    }
  }
  gang_sync(c);
  for (int i = c.t; i < np; i += kGangThreads) L.tau[i] = i < n ? gmem(keys)[i] : -1.0;
  __syncthreads();
  static_assert(kGangMaxN <= kGangThreads, "one column per thread");
  int rank = c.t, from = 0;
  double sc = 1.0;
  if (c.t < n) {
    const double k = L.tau[c.t];
    int before = 0;
#pragma unroll 8
    for (int i = 0; i < n; ++i) {
      const double ki = L.tau[i];
      before += (ki > k || (ki == k && i < c.t)) ? 1 : 0;
    }
    rank = before;
    sc = gmem(scales)[c.t];
    from = pass == 0 ? c.t : (int)L.piv[c.t];
  }
  __syncthreads();
  if (c.t < np) {
    L.tau[rank] = sc;
    L.piv[rank] = c.t < n ? from : c.t;
    // place of every column, for the exchange (L.beta is free)
    L.beta[c.t] = (double)rank;
  }
  __syncthreads();
  double* X = sc_G(c, 0);
  for (int idx = c.t; idx < np * c.geo.w; idx += kGangThreads) {
    const int cc = idx / np, i = idx - cc * np, gc = c.c0 + cc;
    if (gc < n) gmem(X)[(int64_t)((int)L.beta[gc]) * np + i] = L.S[cc * ldr + i];
  }
  gang_sync(c);
  slab_for_each<false>(c, [&](int i, int gc) { return gmem(X)[(int64_t)gc * np + i]; }, SetOrZero{});
}

// T's rows in the order L.piv, times L.tau, into the slab
__device__ void fill_sorted_t(GC& c, const double* Tg) {
  const int n = c.n;
  slab_fill_rows(c, [&](int i, int gc) {
    int row = L.piv[i];
    row = row < 0 ? 0 : (row >= n ? n - 1 : row);
    return gmem(Tg)[(int64_t)row * n + gc] * L.tau[i];
  });
}

// Stabilization of one block, as stabilize_sorted: the slab holds the block's
// product with U (D in L.beta), T in HBM (Tg, own columns, row-major); on
// return the slab holds the new U, Tg the new T and L.beta D.  False, the same
// for every member, where the growth test fails in every pass.
__device__ bool stabilize_gang(GC& c, double* Tg) {
  const int n = c.n, np = c.geo.npad, ldr = c.geo.ldr;
  // unit-size columns, their norms and scales
  for (int cc = c.w; cc < c.geo.w; cc += kWaves) {
    const int gc = c.c0 + cc;
    if (gc >= n) continue;
    double* col = L.S + cc * ldr;
    double am = 0.0;
    for (int i = c.l; i < n; i += 64) am = fmax(am, fabs(col[i]));
    am = wave_max(am);
    const double sc = pow2_scale(am), usc = pow2_unscale(am);
    double ss = 0.0;
    for (int i = c.l; i < n; i += 64) {
      const double x = col[i] * sc;
      col[i] = x;
      ss = fma(x, x, ss);
    }
    ss = wave_sum(ss);
    if (c.l == 0) {
      const double scale = fabs(L.beta[gc]) * usc;
      const double key = sqrt(ss) * scale;
      L.vn1[cc] = key >= 0.0 ? key : 0.0;  // NaN -> 0
      L.vn2[cc] = scale;
    }
  }
  __syncthreads();
  bool sorted = false;
  for (int pass = 0; pass < kSortPasses; ++pass) {
    sort_gang(c, pass);
    sorted = bqr_gang(c, true);
    if (sorted || pass == kSortPasses - 1) break;
    // the next keys: the revealed D, raised where a column outgrows a row
    for (int cc = c.w; cc < c.geo.w; cc += kWaves) {
      const int gc = c.c0 + cc;
      if (gc >= n) continue;
      const double scale = L.tau[gc], own = fabs(L.beta[gc]) * scale;
      double lift = 0.0;
      for (int i = c.l; i < gc; i += 64) {
        const double y = fabs(L.S[cc * ldr + i]) * scale;
        if (y > kGangSortedGrowth * fabs(L.beta[i]) * L.tau[i]) lift = fmax(lift, y);
      }
      lift = wave_max(lift);
      if (c.l == 0) {
        const double d = fmax(own, lift);
        L.vn1[cc] = d >= 0.0 ? d : 0.0;
        L.vn2[cc] = scale;
      }
    }
    __syncthreads();
    // the scaled columns themselves, as the sort left them
    const double* X = sc_G(c, 0);
    slab_for_each<false>(c, [&](int i, int gc) { return gmem(X)[(int64_t)gc * np + i]; }, SetOrZero{});
  }
  if (!sorted) return false;
  for (int i = c.t; i < n; i += kGangThreads) L.beta[i] = fabs(L.beta[i]) * L.tau[i];
  __syncthreads();
  fill_sorted_t(c, Tg);
  slab_gemm(c, AColMajor{sc_R(c), np}, One{}, [&](int row) { return row < n ? 1.0 / L.beta[row] : 0.0; });
  slab_store_rowmajor(c, Tg);
  slab_identity(c);
  bform_gang(c);
  return true;
}
