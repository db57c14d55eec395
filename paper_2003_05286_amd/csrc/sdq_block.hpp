// sdq_block.hpp -- blocked Householder QR of a register matrix (one 16-column
// tile per wave), included by sdq_device.hpp: the factorization of the
// stabilized sweeps after their first block, and the solves of the middle
// matrices.
//
// Why blocked.  A pivoted QR (cpqr) settles one column per step: a pivot
// search over all waves, a barrier, the reflector and the norm downdate of
// every column, about 3 200 cycles a step at n = 64.  Inside a sweep the
// matrix to be factorized is graded by D already, and sorting its columns by
// norm once gives a factorization as accurate as pivoting, provided R's rows
// stay below a small multiple of its diagonal (tested after each; see
// kSortedGrowth).  Without a pivot search the QR is a sequence of
// 16-column panels: the wave holding a panel factors it by itself, with no
// barrier inside, and the other waves apply it as a compact WY block
// reflector on MFMA (the first ones reflector by reflector: panel_steps).
//
// Bound by the panel's wave: it issues one instruction every 4.7 cycles
// whatever they depend on, 350 / 490 / 660 cycles a step at 16 / 64 / 112
// rows; two chains share a CU up to n = 64, so that one's panels run beside
// the other's products.  Sweeps with pivoting in every step -> with this: one
// chain of n = 16 0.21 -> 0.11 ms, 96 of n = 49 1.49 -> 1.14, 512 of n = 64
// 12.4 -> 7.5, 24 of n = 121 7.1 -> 4.6.
//
// LDS: panel q (columns 16q .. 16q+15) in S.R at q NP 16, one 16 x 16 tile
// per row tile: R on and above the diagonal, the reflectors below it (their
// diagonal in S.tau); S.tw: the 16 x 16 triangular factors Tw,
// Q_q = I - V Tw V^T.  Within a tile, entry (i, c) is at 16 i + (c ^ i): both
// operand orders (V^T and V) then read 64 different banks per instruction,
// without padding (at 8 tiles the panels fill 128 of the 160 KB).
#pragma once

constexpr int kTile = 256;
constexpr int kStepPanels = 2;  // panels of a graded block applied by panel_steps
__device__ __forceinline__ int tile_idx(int i, int c) { return 16 * i + (c ^ i); }

// Above kMaxNT tiles (SM::RG) LDS holds the panels from their diagonal tile
// down only; R's tiles above go to the workgroup's device memory (S.rg).
template <int NT, class SM>
__device__ __forceinline__ int panel_off(int p) {
  return SM::RG ? (p * NT - p * (p - 1) / 2) * kTile : (p * NT + p) * kTile;
}
// (through a buffer resource with the tile in the scalar offset: no 64-bit
// address per tile is kept in vector registers)
template <class SM>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rg_rsrc(const SM& S, int bytes) {
  const unsigned long long a = (unsigned long long)S.rg;
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)a);
  const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(a >> 32));
  return __builtin_amdgcn_make_buffer_rsrc((void*)(((unsigned long long)hi << 32) | lo), (short)0, bytes, 0x00020000);
}
typedef unsigned u2 __attribute__((ext_vector_type(2)));
template <int NT, class SM>
__device__ __forceinline__ double upper_ld(const SM& S, int p, int rt, int idx) {
  if constexpr (SM::RG)
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rg_rsrc(S, NT * NT * kTile * 8), idx * 8,
                                                                          (p * NT + rt) * kTile * 8, 0));
  else return S.R[(p * NT + rt) * kTile + idx];
}
template <int NT, class SM>
__device__ __forceinline__ void upper_st(SM& S, int p, int rt, int idx, double v) {
  if constexpr (SM::RG)
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, v), rg_rsrc(S, NT * NT * kTile * 8), idx * 8,
                                          (p * NT + rt) * kTile * 8, 0);
  else S.R[(p * NT + rt) * kTile + idx] = v;
}

// lane J of each 16-lane row to all lanes of the row (one instruction for
// the 64-bit value)
template <int J>
__device__ __forceinline__ double bcast_col(double v) {
  return __longlong_as_double(
      __builtin_amdgcn_mov_dpp((long long)__double_as_longlong(v), 0x150 + J, 0xf, 0xf, true));
}
// 16-lane row G0 to all four rows
template <int G0>
__device__ __forceinline__ double bcast_row(double v) {
  const unsigned lo = __double2loint(v), hi = __double2hiint(v);
  const auto a = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
  const auto b = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
  const unsigned l1 = a[G0 & 1], h1 = b[G0 & 1];
  const auto c = __builtin_amdgcn_permlane32_swap(l1, l1, false, false);
  const auto d = __builtin_amdgcn_permlane32_swap(h1, h1, false, false);
  return __hiloint2double((int)d[G0 >> 1], (int)c[G0 >> 1]);
}

// Multiply-adds whose first factor is lane J of the lane's 16-lane row: the
// broadcast is part of the instruction (v_fmac_f64 with DPP row_newbcast),
// which the compiler does not form from a move and an fma.  The compiler does
// not look into inline assembly for the wait states these need, so they are
// here: two between a vector instruction that writes a register and a DPP
// read of it (each group begins with s_nop 1; one whose result a lane exchange
// reads next ends with it too); where row_mask leaves rows out, two as well
// before it for its destination, and one after it before that is read.
#define SDQ_FD(D, A, B, J, M) "v_fmac_f64_dpp " D ", " A ", " B " row_newbcast:" J " row_mask:" M " bank_mask:0xf\n"
#define SDQ_DOT(X) SDQ_FD("%[p]", "%[" #X "]", "%[" #X "]", "%[J]", "0xf")
#define SDQ_DOTM(X) SDQ_FD("%[p]", "%[" #X "]", "%[" #X "]", "%[J]", "%[M]") "s_nop 0\n"
#define SDQ_DOT4(X) SDQ_DOT(X##0) SDQ_DOT(X##1) SDQ_DOT(X##2) SDQ_DOT(X##3)
#define SDQ_IN4(X, V) [X##0] "v"(V[0]), [X##1] "v"(V[1]), [X##2] "v"(V[2]), [X##3] "v"(V[3])
#define SDQ_IO4(X, V) [X##0] "+v"(V[0]), [X##1] "+v"(V[1]), [X##2] "+v"(V[2]), [X##3] "+v"(V[3])

// p += sum of x[J] x over the entries below row J of the first min(RT, 4)
// tiles.  Row J = 4 R0 + G0 of the diagonal tile is in register R0 of the
// 16-lane row G0: of that register only the rows after G0 count (mask M, none
// for G0 = 3), of the later registers all.
template <int J, int RT, int NT>
__device__ __forceinline__ void dot_head(double& p, const double (&t)[NT][4]) {
  constexpr int R0 = J >> 2, M = (0xe << (J & 3)) & 0xf;
#define SDQ_DOT_CASE(DIAG, MORE, ...) \
  asm("s_nop 1\n" DIAG MORE "s_nop 1" : [p] "+v"(p) : [J] "n"(J), [M] "n"(M), SDQ_IN4(a, t[0]) __VA_ARGS__);
#define SDQ_DOT_CASES(MORE, ...)                                                                             \
  if constexpr (R0 == 0 && M) SDQ_DOT_CASE(SDQ_DOTM(a0) SDQ_DOT(a1) SDQ_DOT(a2) SDQ_DOT(a3), MORE, __VA_ARGS__) \
  else if constexpr (R0 == 0) SDQ_DOT_CASE(SDQ_DOT(a1) SDQ_DOT(a2) SDQ_DOT(a3), MORE, __VA_ARGS__)           \
  else if constexpr (R0 == 1 && M) SDQ_DOT_CASE(SDQ_DOTM(a1) SDQ_DOT(a2) SDQ_DOT(a3), MORE, __VA_ARGS__)     \
  else if constexpr (R0 == 1) SDQ_DOT_CASE(SDQ_DOT(a2) SDQ_DOT(a3), MORE, __VA_ARGS__)                       \
  else if constexpr (R0 == 2 && M) SDQ_DOT_CASE(SDQ_DOTM(a2) SDQ_DOT(a3), MORE, __VA_ARGS__)                 \
  else if constexpr (R0 == 2) SDQ_DOT_CASE(SDQ_DOT(a3), MORE, __VA_ARGS__)                                   \
  else if constexpr (M) SDQ_DOT_CASE(SDQ_DOTM(a3), MORE, __VA_ARGS__)                                        \
  else if constexpr (RT > 1) SDQ_DOT_CASE("", MORE, __VA_ARGS__)
  if constexpr (RT == 1) {
    SDQ_DOT_CASES("", )
  } else if constexpr (RT == 2) {
    SDQ_DOT_CASES(SDQ_DOT4(b), , SDQ_IN4(b, t[1]))
  } else if constexpr (RT == 3) {
    SDQ_DOT_CASES(SDQ_DOT4(b) SDQ_DOT4(c), , SDQ_IN4(b, t[1]), SDQ_IN4(c, t[2]))
  } else {
    SDQ_DOT_CASES(SDQ_DOT4(b) SDQ_DOT4(c) SDQ_DOT4(d), , SDQ_IN4(b, t[1]), SDQ_IN4(c, t[2]), SDQ_IN4(d, t[3]))
  }
#undef SDQ_DOT_CASES
#undef SDQ_DOT_CASE
}
// p += sum of x[J] x over whole tiles
template <int J>
__device__ __forceinline__ void dot_tiles(double& p, const double (&t0)[4]) {
  asm("s_nop 1\n" SDQ_DOT4(a) "s_nop 1" : [p] "+v"(p) : [J] "n"(J), SDQ_IN4(a, t0));
}
template <int J>
__device__ __forceinline__ void dot_tiles(double& p, const double (&t0)[4], const double (&t1)[4],
                                          const double (&t2)[4], const double (&t3)[4]) {
  asm("s_nop 1\n" SDQ_DOT4(a) SDQ_DOT4(b) SDQ_DOT4(c) SDQ_DOT4(d) "s_nop 1"
      : [p] "+v"(p)
      : [J] "n"(J), SDQ_IN4(a, t0), SDQ_IN4(b, t1), SDQ_IN4(c, t2), SDQ_IN4(d, t3));
}

// x += x[J] f below row J, row J itself += s f (s the same in every lane); the
// first one or two tiles.  SDQ_AXM: the rows of register R0 after G0; SDQ_AXS:
// row J, two instructions or more later.
#define SDQ_AX(X) SDQ_FD("%[" #X "]", "%[" #X "]", "%[f]", "%[J]", "0xf")
#define SDQ_AXM(X) SDQ_FD("%[" #X "]", "%[" #X "]", "%[f]", "%[J]", "%[M]")
#define SDQ_AXS(X) SDQ_FD("%[" #X "]", "%[s]", "%[f]", "%[J]", "%[M0]")
#define SDQ_AX4(X) SDQ_AX(X##0) SDQ_AX(X##1) SDQ_AX(X##2) SDQ_AX(X##3)
template <int J, int RT, int NT>
__device__ __forceinline__ void axpy_head(double (&t)[NT][4], double s, double f) {
  constexpr int R0 = J >> 2, G0 = J & 3, M = (0xe << G0) & 0xf, M0 = 1 << G0;
#define SDQ_AX_CASE(BODY, ...)                      \
  asm("s_nop 1\n" BODY                              \
      : SDQ_IO4(a, t[0]) __VA_ARGS__                \
      : [s] "v"(s), [f] "v"(f), [J] "n"(J), [M] "n"(M), [M0] "n"(M0));
  if constexpr (RT == 1) {
    if constexpr (R0 == 0 && M) SDQ_AX_CASE(SDQ_AXM(a0) SDQ_AX(a1) SDQ_AX(a2) SDQ_AXS(a0) SDQ_AX(a3), )
    else if constexpr (R0 == 0) SDQ_AX_CASE(SDQ_AXS(a0) SDQ_AX(a1) SDQ_AX(a2) SDQ_AX(a3), )
    else if constexpr (R0 == 1 && M) SDQ_AX_CASE(SDQ_AXM(a1) SDQ_AX(a2) SDQ_AX(a3) SDQ_AXS(a1) "s_nop 0", )
    else if constexpr (R0 == 1) SDQ_AX_CASE(SDQ_AXS(a1) SDQ_AX(a2) SDQ_AX(a3), )
    else if constexpr (R0 == 2 && M) SDQ_AX_CASE(SDQ_AXM(a2) SDQ_AX(a3) "s_nop 0\n" SDQ_AXS(a2) "s_nop 0", )
    else if constexpr (R0 == 2) SDQ_AX_CASE(SDQ_AXS(a2) SDQ_AX(a3), )
    else if constexpr (M) SDQ_AX_CASE(SDQ_AXM(a3) "s_nop 1\n" SDQ_AXS(a3) "s_nop 0", )
    else SDQ_AX_CASE(SDQ_AXS(a3) "s_nop 0", )
  } else {
#define SDQ_AX_CASES(R, DIAG)                                                                                      \
  if constexpr (R0 == R) {                                                                                         \
    if constexpr (M != 0)                                                                                          \
      SDQ_AX_CASE(SDQ_AXM(a##R) DIAG SDQ_AX(b0) SDQ_AX(b1) SDQ_AXS(a##R) SDQ_AX(b2) SDQ_AX(b3), , SDQ_IO4(b, t[1])) \
    else                                                                                                           \
      SDQ_AX_CASE(SDQ_AXS(a##R) DIAG SDQ_AX4(b), , SDQ_IO4(b, t[1]))                                               \
  }
    SDQ_AX_CASES(0, SDQ_AX(a1) SDQ_AX(a2) SDQ_AX(a3))
    SDQ_AX_CASES(1, SDQ_AX(a2) SDQ_AX(a3))
    SDQ_AX_CASES(2, SDQ_AX(a3))
    SDQ_AX_CASES(3, )
#undef SDQ_AX_CASES
  }
#undef SDQ_AX_CASE
}
template <int J>
__device__ __forceinline__ void axpy_tiles(double (&t0)[4], double f) {
  asm("s_nop 1\n" SDQ_AX4(a) : SDQ_IO4(a, t0) : [f] "v"(f), [J] "n"(J));
}
template <int J>
__device__ __forceinline__ void axpy_tiles(double (&t0)[4], double (&t1)[4], double f) {
  asm("s_nop 1\n" SDQ_AX4(a) SDQ_AX4(b) : SDQ_IO4(a, t0), SDQ_IO4(b, t1) : [f] "v"(f), [J] "n"(J));
}

// p += sum of a[J] x over one or two tiles and x += a[J] f, for another
// matrix's rows x; a lane exchange may follow dot_with after dot_done only
#define SDQ_DW(X, Y) SDQ_FD("%[p]", "%[" #X "]", "%[" #Y "]", "%[J]", "0xf")
#define SDQ_AW(X, Y) SDQ_FD("%[" #Y "]", "%[" #X "]", "%[f]", "%[J]", "0xf")
#define SDQ_W4(OP, A, X) OP(A##0, X##0) OP(A##1, X##1) OP(A##2, X##2) OP(A##3, X##3)
template <int J>
__device__ __forceinline__ void dot_with(double& p, const double (&a)[4], const double (&x)[4]) {
  asm("s_nop 1\n" SDQ_W4(SDQ_DW, a, x) : [p] "+v"(p) : [J] "n"(J), SDQ_IN4(a, a), SDQ_IN4(x, x));
}
template <int J>
__device__ __forceinline__ void dot_with(double& p, const double (&a)[4], const double (&x)[4], const double (&b)[4],
                                         const double (&y)[4]) {
  asm("s_nop 1\n" SDQ_W4(SDQ_DW, a, x) SDQ_W4(SDQ_DW, b, y)
      : [p] "+v"(p)
      : [J] "n"(J), SDQ_IN4(a, a), SDQ_IN4(x, x), SDQ_IN4(b, b), SDQ_IN4(y, y));
}
__device__ __forceinline__ void dot_done(double& p) { asm("s_nop 1" : "+v"(p)); }
template <int J>
__device__ __forceinline__ void axpy_with(double (&x)[4], const double (&a)[4], double f) {
  asm("s_nop 1\n" SDQ_W4(SDQ_AW, a, x) : SDQ_IO4(x, x) : [J] "n"(J), SDQ_IN4(a, a), [f] "v"(f));
}
template <int J>
__device__ __forceinline__ void axpy_with(double (&x)[4], const double (&a)[4], double (&y)[4], const double (&b)[4],
                                          double f) {
  asm("s_nop 1\n" SDQ_W4(SDQ_AW, a, x) SDQ_W4(SDQ_AW, b, y)
      : SDQ_IO4(x, x), SDQ_IO4(y, y)
      : [J] "n"(J), SDQ_IN4(a, a), SDQ_IN4(b, b), [f] "v"(f));
}
// the same over NT tiles, and the rows' last write two wait states before a
// matrix instruction may read them
template <int J, int NT>
__device__ __forceinline__ double dot_rows(const double (&a)[NT][4], const double (&x)[NT][4]) {
  double p = 0.0;
  static_for<NT / 2>([&](auto tc) {
    constexpr int t = 2 * decltype(tc)::value;
    dot_with<J>(p, a[t], x[t], a[t + 1], x[t + 1]);
  });
  if constexpr (NT % 2 == 1) dot_with<J>(p, a[NT - 1], x[NT - 1]);
  dot_done(p);
  return p;
}
template <int J, int NT>
__device__ __forceinline__ void axpy_rows(double (&x)[NT][4], const double (&a)[NT][4], double f) {
  static_for<NT / 2>([&](auto tc) {
    constexpr int t = 2 * decltype(tc)::value;
    axpy_with<J>(x[t], a[t], x[t + 1], a[t + 1], f);
  });
  if constexpr (NT % 2 == 1) axpy_with<J>(x[NT - 1], a[NT - 1], f);
}
template <int NT>
__device__ __forceinline__ void rows_done(double (&x)[NT][4]) {
#pragma unroll
  for (int t = 0; t < NT; ++t) asm volatile("" : SDQ_IO4(a, x[t]));
  asm volatile("s_nop 1");
#pragma unroll
  for (int t = 0; t < NT; ++t) asm volatile("" : SDQ_IO4(a, x[t]));
}
// rows that matrix instructions may have written just before: let them land
// before inline assembly reads them (18 wait states)
template <int RT, int NT>
__device__ __forceinline__ void rows_landed(double (&b)[NT][4]) {
#pragma unroll
  for (int t = 0; t < RT; ++t) asm volatile("" : SDQ_IO4(a, b[t]));
  asm volatile("s_nop 15\ns_nop 7");
#pragma unroll
  for (int t = 0; t < RT; ++t) asm volatile("" : SDQ_IO4(a, b[t]));
}

// sum_{c < J} d[c] T[c]: d from lane c of the row, T[c] the lane's own
#define SDQ_TD(C) SDQ_FD("%[p]", "%[d]", "%[t" #C "]", #C, "0xf")
#define SDQ_TD1 SDQ_TD(0)
#define SDQ_TD2 SDQ_TD1 SDQ_TD(1)
#define SDQ_TD3 SDQ_TD2 SDQ_TD(2)
#define SDQ_TD4 SDQ_TD3 SDQ_TD(3)
#define SDQ_TD5 SDQ_TD4 SDQ_TD(4)
#define SDQ_TD6 SDQ_TD5 SDQ_TD(5)
#define SDQ_TD7 SDQ_TD6 SDQ_TD(6)
#define SDQ_TD8 SDQ_TD7 SDQ_TD(7)
#define SDQ_TD9 SDQ_TD8 SDQ_TD(8)
#define SDQ_TD10 SDQ_TD9 SDQ_TD(9)
#define SDQ_TD11 SDQ_TD10 SDQ_TD(10)
#define SDQ_TD12 SDQ_TD11 SDQ_TD(11)
#define SDQ_TD13 SDQ_TD12 SDQ_TD(12)
#define SDQ_TD14 SDQ_TD13 SDQ_TD(13)
#define SDQ_TD15 SDQ_TD14 SDQ_TD(14)
#define SDQ_TI(C) [t##C] "v"(T[C])
#define SDQ_TI4 SDQ_TI(0), SDQ_TI(1), SDQ_TI(2), SDQ_TI(3)
#define SDQ_TI8 SDQ_TI4, SDQ_TI(4), SDQ_TI(5), SDQ_TI(6), SDQ_TI(7)
#define SDQ_TI12 SDQ_TI8, SDQ_TI(8), SDQ_TI(9), SDQ_TI(10), SDQ_TI(11)
#define SDQ_TRI(J_, ...) \
  if constexpr (J == J_) asm("s_nop 1\n" SDQ_TD##J_ : [p] "+v"(p) : [d] "v"(d), __VA_ARGS__);
template <int J>
__device__ __forceinline__ double tri_dot(double d, const double (&T)[16]) {
  double p = 0.0;
  SDQ_TRI(1, SDQ_TI(0))
  SDQ_TRI(2, SDQ_TI(0), SDQ_TI(1))
  SDQ_TRI(3, SDQ_TI(0), SDQ_TI(1), SDQ_TI(2))
  SDQ_TRI(4, SDQ_TI4)
  SDQ_TRI(5, SDQ_TI4, SDQ_TI(4))
  SDQ_TRI(6, SDQ_TI4, SDQ_TI(4), SDQ_TI(5))
  SDQ_TRI(7, SDQ_TI4, SDQ_TI(4), SDQ_TI(5), SDQ_TI(6))
  SDQ_TRI(8, SDQ_TI8)
  SDQ_TRI(9, SDQ_TI8, SDQ_TI(8))
  SDQ_TRI(10, SDQ_TI8, SDQ_TI(8), SDQ_TI(9))
  SDQ_TRI(11, SDQ_TI8, SDQ_TI(8), SDQ_TI(9), SDQ_TI(10))
  SDQ_TRI(12, SDQ_TI12)
  SDQ_TRI(13, SDQ_TI12, SDQ_TI(12))
  SDQ_TRI(14, SDQ_TI12, SDQ_TI(12), SDQ_TI(13))
  SDQ_TRI(15, SDQ_TI12, SDQ_TI(12), SDQ_TI(13), SDQ_TI(14))
  return p;
}

// Sum of p over the four lanes of a column, and the value that x has in row
// G0 of them, both to all four: one transposing exchange of the two instead
// of a reduction and a broadcast.
__device__ __forceinline__ void sum_and_pick(double p, double x, bool in_g0, double& sum, double& pick) {
  const double m = in_g0 ? x : 0.0;
  const auto a = __builtin_amdgcn_permlane16_swap(__double2loint(p), __double2loint(m), false, false);
  const auto b = __builtin_amdgcn_permlane16_swap(__double2hiint(p), __double2hiint(m), false, false);
  // even rows: two rows' p; odd rows: two rows' m
  const double v = __hiloint2double((int)b[0], (int)a[0]) + __hiloint2double((int)b[1], (int)a[1]);
  const double w = pl32_pair_sum(v);
  const auto c = __builtin_amdgcn_permlane16_swap(__double2loint(w), __double2loint(w), false, false);
  const auto d = __builtin_amdgcn_permlane16_swap(__double2hiint(w), __double2hiint(w), false, false);
  sum = __hiloint2double((int)d[0], (int)c[0]);
  pick = __hiloint2double((int)d[1], (int)c[1]);
}

// Householder QR of one 16-column panel by the wave that holds it, rows in
// b[0 .. RT) (row 0 of b[0] is the panel's first diagonal row; tiles past
// the matrix are zero).  The reflector of column J is kept unscaled,
// v_J = (su at row J; column J below it), H = I - c v v^T with
// h = ||x||, su = alpha + sign(alpha) h, c = 2 / v^T v (of the rounded v: from
// h it would leave H further from orthogonal), and always reflects (a column
// with nothing below row J changes sign), so that only a column of zeros, or
// one whose squares leave the range of a double, is a special case: the caller
// looks at beta (plain_panel) and takes panel_careful for those.
// On return b holds R above the diagonal, the reflectors below
// it and alpha on it; su_l, beta_l the reflector's and R's diagonal entry of
// the lane's column; T row cl of the triangular factor.  Columns from `live`
// on are unit vectors (padding): of a one-tile matrix, groups of four such steps
// are left out, with T zero there and R's diagonal one (a chain of two sites
// took 1.3 times as long as with pivoting otherwise; at eight tiles the
// branches spill a thousand registers).
// Bound: one wave issues an instruction about every five cycles whatever its
// dependences are, so the step is written for few instructions (82 at 64
// rows): straight-line code, no LDS access, no barrier; the dot products of
// column J with all columns give its norm and the Gram entries of the
// triangular factor too.
template <int RT, int NT>
__device__ __forceinline__ void panel_qr(const Lane& L, const int live, double (&b)[NT][4], double (&T)[16],
                                         double& su_l, double& beta_l) {
  rows_landed<RT>(b);
  double hs_l = -1.0;
  auto step = [&](auto jc) {
    constexpr int J = decltype(jc)::value, R0 = J >> 2, G0 = J & 3;
    double p = 0.0;
    dot_head<J, RT>(p, b);
    static_for<(RT > 4 ? RT - 4 : 0) / 4>([&](auto tc) {
      constexpr int t = 4 + 4 * decltype(tc)::value;
      dot_tiles<J>(p, b[t], b[t + 1], b[t + 2], b[t + 3]);
    });
    static_for<RT % 4 * (RT > 4)>([&](auto tc) { dot_tiles<J>(p, b[RT / 4 * 4 + decltype(tc)::value]); });
    double dot, ajc;
    sum_and_pick(p, b[0][R0], L.g == G0, dot, ajc);  // x_J^T a_c below row J; row J
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
    const double d = fma(su, ajc, dot);  // v_J^T a_c
    const double cd = -c * d;
    // columns up to J stay as they are (the low word alone is a denormal)
    const double f = __hiloint2double(L.cl > J ? __double2hiint(cd) : 0, __double2loint(cd));
    axpy_head<J, RT>(b, su, f);
    static_for<(RT > 2 ? RT - 2 : 0) / 2>([&](auto tc) {
      constexpr int t = 2 + 2 * decltype(tc)::value;
      axpy_tiles<J>(b[t], b[t + 1], f);
    });
    if constexpr (RT > 2 && RT % 2 == 1) axpy_tiles<J>(b[RT - 1], f);
    hs_l = L.cl == J ? hs : hs_l;
    // column J of the triangular factor: c on the diagonal, -c T V^T v_J above
    // (the sum is zero in the rows from J on)
    const double ts = tri_dot<J>(d, T);
    T[J] = L.cl == J ? c : -c * ts;
  };
  static_for<4>([&](auto gc) {
    constexpr int J0 = 4 * decltype(gc)::value;
    if (NT > 1 || J0 < live) {
      static_for<4>([&](auto jc) { step(std::integral_constant<int, J0 + decltype(jc)::value>{}); });
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q) T[J0 + q] = 0.0;
    }
  });
  // beta = -hs, su = alpha + hs, alpha on the diagonal
  beta_l = -hs_l;
  double al = 0.0;
#pragma unroll
  for (int r = 0; r < 4; ++r) al = L.g + 4 * r == L.cl ? b[0][r] : al;
  su_l = sum_col(al) + hs_l;
}

// Whether panel_qr's squares stayed inside the range: every ||x|| of the panel
// (|beta_l|) between these powers of two, zero and NaN not among them.
// (Entries below 2^-537 do not count beside 2^-300; a reflector's
// products with columns of any other panel stay normal too.)
__device__ __forceinline__ bool plain_panel(double beta_l) {
  const double h = fabs(beta_l);
  return __all(h >= 0x1p-300 && h <= 0x1p300);
}

// one wave's LDS accesses before it, by all lanes, before those after it
__device__ __forceinline__ void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// The same panel, in LDS, for columns of any size, by one wave: before a
// column becomes a reflector it is scaled to unit size by a power of two (the
// reflector stays so; R's entry is scaled back), and a column of zeros reflects
// its first entry: v = e_J, c = 2, so that every column's reflector reflects.
// Entry (i, c), 0 <= i < rows, at x: in panel layout, or (ld > 0) at c ld + i;
// R with its diagonal on return.  tw: the triangular factor, a tile or (ld > 0)
// row-major; su_l: the diagonal of the lane's reflector.
// Reached by middle matrices that are singular or far from one in size (and by
// NaN); a row at a time, as slow as that is.
struct CarefulDiag {
  double su_l, beta_l;
};
template <bool TILES>
__device__ __forceinline__ CarefulDiag panel_careful(double* x, double* tw, int rows, int ld) {
  const Lane L = lane_id_per_item();
  auto at = [&](int i, int c) -> double& {
    return TILES ? x[kTile * (i >> 4) + tile_idx(i & 15, c)] : x[c * ld + i];
  };
  auto tri = [&](int i, int c) -> double& { return tw[TILES ? tile_idx(i, c) : 16 * i + c]; };
  CarefulDiag out = {0.0, 0.0};
  wave_fence();
#pragma unroll 1
  for (int J = 0; J < 16; ++J) {
    double mx = 0.0;
#pragma unroll 1
    for (int i = J + L.l; i < rows; i += 64) mx = fmax(mx, fabs(at(i, J)));
#pragma unroll 1
    for (int m = 32; m >= 1; m >>= 1) mx = fmax(mx, __shfl_xor(mx, m));
    const int e = mx > 0.0 && isfinite(mx) ? ilogb(mx) : 0;
#pragma unroll 1
    for (int i = J + L.l; i < rows; i += 64) at(i, J) = ldexp(at(i, J), -e);
    wave_fence();
    double p = 0.0;
#pragma unroll 1
    for (int i = L.g; i < rows; i += 4)
      if (i > J) p = fma(at(i, J), at(i, L.cl), p);
    const double dot = sum_col(p), ajc = at(J, L.cl);
    const double s = __shfl(dot, J), alpha = __shfl(ajc, J);
    const double hs = copysign(sqrt(fma(alpha, alpha, s)), alpha);
    const double su = hs == 0.0 ? 1.0 : alpha + hs;
    const double c = hs == 0.0 ? 2.0 : 2.0 / fma(su, su, s);
    const double d = fma(su, ajc, dot), f = -c * d;
    wave_fence();  // row J is read
    if (L.cl > J) {
#pragma unroll 1
      for (int i = L.g; i < rows; i += 4)
        if (i > J) at(i, L.cl) = fma(at(i, J), f, at(i, L.cl));
      if (L.g == 0) at(J, L.cl) = fma(su, f, ajc);
    }
    if (L.cl == J) out = CarefulDiag{su, -ldexp(hs, e)};
    double ts = 0.0;
#pragma unroll 1
    for (int i = 0; i < J; ++i) ts = fma(__shfl(d, i), tri(L.cl, i), ts);
    if (L.g == 0) tri(L.cl, J) = L.cl == J ? c : (L.cl < J ? -c * ts : 0.0);
    wave_fence();
  }
  if (L.g == 0) at(L.cl, L.cl) = out.beta_l;
  wave_fence();
  return out;
}

// C <- Q_p^T C (QT) or Q_p C for one column tile, rows in b[0 .. cnt) from
// row tile p on (cnt = NT - p, wave-uniform): X = V^T C, X <- Tw' X,
// C <- C - V X on MFMA.  vp: the panel at its first diagonal row.  The
// operands of a row tile are read one tile ahead.
template <int NT, bool QT>
__device__ __forceinline__ void panel_apply(double (&b)[NT][4], const int cnt, const double* vp, const double* tw,
                                            const double* su) {
  const Lane L = lane_id_per_item();
  const double vd = su[L.cl];
  d4 x = d4{0.0, 0.0, 0.0, 0.0}, x2 = x;
  double a[4], an[4], tv[4];
  int pt[4], pn[4];  // (row g + 4r, reflector cl) and (row cl, reflector g + 4r) of a tile
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    pt[r] = tile_idx(L.g + 4 * r, L.cl);
    pn[r] = tile_idx(L.cl, L.g + 4 * r);
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const double v = vp[pt[r]];
    const int row = L.g + 4 * r;
    a[r] = row > L.cl ? v : (row == L.cl ? vd : 0.0);
    tv[r] = QT ? tw[pt[r]] : tw[pn[r]];
  }
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    if (t + 1 < NT) {
      const int tn = t + 1 < cnt ? t + 1 : cnt - 1;
#pragma unroll
      for (int r = 0; r < 4; ++r) an[r] = vp[kTile * tn + pt[r]];
    }
    if (t < cnt) {
#pragma unroll
      for (int r = 0; r < 4; ++r) x = __builtin_amdgcn_mfma_f64_16x16x4f64(a[r], b[t][r], x, 0, 0, 0);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) a[r] = an[r];
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const double v = vp[pn[r]];
    const int refl = L.g + 4 * r;
    a[r] = L.cl > refl ? v : (L.cl == refl ? vd : 0.0);
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) x2 = __builtin_amdgcn_mfma_f64_16x16x4f64(tv[r], x[r], x2, 0, 0, 0);
#pragma unroll
  for (int r = 0; r < 4; ++r) x2[r] = -x2[r];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    if (t + 1 < NT) {
      const int tn = t + 1 < cnt ? t + 1 : cnt - 1;
#pragma unroll
      for (int r = 0; r < 4; ++r) an[r] = vp[kTile * tn + pn[r]];
    }
    if (t < cnt) {
      d4 acc = d4{b[t][0], b[t][1], b[t][2], b[t][3]};
#pragma unroll
      for (int r = 0; r < 4; ++r) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[r], x2[r], acc, 0, 0, 0);
#pragma unroll
      for (int r = 0; r < 4; ++r) b[t][r] = acc[r];
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) a[r] = an[r];
  }
}

// C <- Q_p^T C as panel_apply, one reflector at a time on the vector units: a
// column that is nearly in the span of the reflectors before shrinks on the
// way, and with it what a reflector adds to its error, while the block
// reflector's coefficients all carry the error of the column as it came.  The
// columns of a product of slices shrink most in the first panels
// (kStepPanels; with none the errors are 1.2 to 1.5 times those of pivoting,
// more than two change nothing).  A step takes some 50 instructions at 64 rows;
// 512 chains of n = 64 take 1 % longer with it.
template <int NT>
__device__ __forceinline__ void panel_steps(double (&b)[NT][4], const int cnt, const double* vp, const double* tw,
                                            const double* su) {
  const Lane L = lane_id_per_item();
  const double vd = su[L.cl], cd = tw[tile_idx(L.cl, L.cl)];
  double a[NT][4];  // row g + 4 r of a tile, reflector cl
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = L.g + 4 * r;
      const double v = vp[kTile * min(t, cnt - 1) + tile_idx(row, L.cl)];
      a[t][r] = t >= cnt ? 0.0 : (t > 0 || row > L.cl ? v : (row == L.cl ? vd : 0.0));
    }
  rows_landed<NT>(b);
  static_for<16>([&](auto jc) {
    constexpr int J = decltype(jc)::value;
    const double f = -bcast_col<J>(cd) * sum_col(dot_rows<J>(a, b));
    axpy_rows<J>(b, a, f);
  });
  rows_done(b);
}

// row tiles one up (the first becomes the last) / one down
template <int NT>
__device__ __forceinline__ void rotate_up(double (&b)[NT][4]) {
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const double x = b[0][r];
#pragma unroll
    for (int t = 0; t + 1 < NT; ++t) b[t][r] = b[t + 1][r];
    b[NT - 1][r] = x;
  }
}
template <int NT>
__device__ __forceinline__ void rotate_down(double (&b)[NT][4]) {
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const double x = b[NT - 1][r];
#pragma unroll
    for (int t = NT - 1; t > 0; --t) b[t][r] = b[t - 1][r];
    b[0][r] = x;
  }
}

// Factor the panel of this wave (row tiles rotated so that b[0] is the
// diagonal one) and store it: panel and R above it, Tw, the reflectors'
// diagonal (S.tau) and diag R.
template <int NT, class SM>
__device__ __forceinline__ void panel_factor(SM& S, double (&b)[NT][4], const int p, const int n) {
  const Lane L = lane_id_per_item();
  double T[16], su_l, beta_l;
  const int cnt = NT - p, live = n - 16 * p;
  double* vp = S.R + panel_off<NT, SM>(p);
  // R above the panel goes out first; its registers are zero rows from here on.
  // The panel's rows go to their place as they are, for panel_careful.
#pragma unroll
  for (int t = 0; t < NT; ++t)
    if (t >= cnt) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        upper_st<NT>(S, p, t - cnt, tile_idx(L.g + 4 * r, L.cl), b[t][r]);
        b[t][r] = 0.0;
      }
    } else {
#pragma unroll
      for (int r = 0; r < 4; ++r) vp[kTile * t + tile_idx(L.g + 4 * r, L.cl)] = b[t][r];
    }
  if constexpr (NT >= 4) {
    // the lower half of the panels have at most half the rows
    if (cnt <= NT / 2) panel_qr<NT / 2, NT>(L, live, b, T, su_l, beta_l);
    else panel_qr<NT, NT>(L, live, b, T, su_l, beta_l);
  } else {
    panel_qr<NT, NT>(L, live, b, T, su_l, beta_l);
  }
  double* tw = S.tw + p * kTile;
  if (plain_panel(beta_l)) {
    const Lane L = lane_id_per_item();
#pragma unroll
    for (int r = 0; r < 4; ++r) b[0][r] = L.g + 4 * r == L.cl ? beta_l : b[0][r];
#pragma unroll
    for (int t = 0; t < NT; ++t)
      if (t < cnt) {
#pragma unroll
        for (int r = 0; r < 4; ++r) vp[kTile * t + tile_idx(L.g + 4 * r, L.cl)] = b[t][r];
      }
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (L.g == q) {
#pragma unroll
        for (int c = 0; c < 4; ++c) tw[tile_idx(L.cl, 4 * q + c)] = T[4 * q + c];
      }
  } else {
    const CarefulDiag cd = panel_careful<true>(vp, tw, 16 * cnt, 0);
    su_l = cd.su_l;
    beta_l = cd.beta_l;
  }
  if (L.g == 0) {
    S.tau[16 * p + L.cl] = su_l;
    S.red_diag[16 * p + L.cl] = beta_l;
  }
}

// the padding columns as unit vectors
template <int NT>
__device__ __forceinline__ void pad_unit(const Lane& L, const int n, double (&b)[NT][4]) {
  const int col = 16 * L.w + L.cl;
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) b[t][r] = col < n ? b[t][r] : (16 * t + L.g + 4 * r == col ? 1.0 : 0.0);
}

// W = Q R for the register matrix W as its columns stand (padding columns:
// unit vectors), Q and R left in LDS in panels; diag R in S.red_diag.  With
// YN > 0 the same Q^T is applied to the register matrix Y, whose rows are in
// place again afterwards.  The first STEPS panels are applied by panel_steps:
// kStepPanels of a graded block, all of them where the solution is the result.
// Starts with a barrier after which S.R is free to write; ends with one.
template <int NT, int YN, int STEPS, class SM>
__device__ __forceinline__ void block_qr(const Lane& L, const int n, SM& S, double (&b)[NT][4], double (*Y)[4]) {
  __syncthreads();
#pragma unroll 1
  for (int p = 0; p < NT; ++p) {
    if (L.w == p) panel_factor<NT>(S, b, p, n);
    __syncthreads();
    const double* vp = S.R + panel_off<NT, SM>(p);
    const double* tw = S.tw + p * kTile;
    if (L.w > p) {
      if (p < STEPS) panel_steps<NT>(b, NT - p, vp, tw, S.tau + 16 * p);
      else panel_apply<NT, true>(b, NT - p, vp, tw, S.tau + 16 * p);
      rotate_up<NT>(b);
    }
    if constexpr (YN > 0) {
      double(&y)[NT][4] = *reinterpret_cast<double(*)[NT][4]>(Y);
      if (p < STEPS) panel_steps<NT>(y, NT - p, vp, tw, S.tau + 16 * p);
      else panel_apply<NT, true>(y, NT - p, vp, tw, S.tau + 16 * p);
      rotate_up<NT>(y);
    }
  }
}

// This wave's column tile of Q from the panels: Q_0 ... Q_w applied to the
// tile of the identity.
template <int NT, class SM>
__device__ __forceinline__ void block_form(const Lane& L, const SM& S, double (&b)[NT][4]) {
  const int w = L.w;
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) b[t][r] = t == 0 && L.g + 4 * r == L.cl ? 1.0 : 0.0;
#pragma unroll 1
  for (int p = w; p >= 0; --p) {
    const Lane L = lane_id_per_item();
    panel_apply<NT, false>(b, NT - p, S.R + panel_off<NT, SM>(p), S.tw + p * kTile,
                           S.tau + 16 * p);
    if (p > 0) rotate_down<NT>(b);
  }
}

// Y <- R^{-1} Y with R in panels: from the last row tile up, the triangular
// solve of the diagonal tile in this wave's registers, then the tile's
// contribution to the rows above on MFMA.  No barrier.
template <int NT, class SM>
__device__ __forceinline__ void block_back_subst(const Lane& L, const SM& S, double (&y)[NT][4]) {
#pragma unroll 1
  for (int p = NT - 1; p >= 0; --p) {
    const Lane L = lane_id_per_item();
    rotate_down<NT>(y);  // y[0]: row tile p, y[1 ..]: row tiles 0 .. p - 1 at y[NT - p ..]
    const double* pp = S.R + p * (NT * kTile);
    const double* dg = pp + p * kTile;
    const double ri = 1.0 / dg[tile_idx(L.cl, L.cl)];
    double z[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) z[r] = y[0][r];
    static_for<16>([&](auto jc) {
      constexpr int J = 15 - decltype(jc)::value, R0 = J >> 2, G0 = J & 3;
      const double zj = bcast_row<G0>(z[R0]) * bcast_col<J>(ri);
#pragma unroll
      for (int r = 0; r <= R0; ++r) {
        const double rr = dg[tile_idx(L.g + 4 * r, J)];
        if (r < R0) z[r] = fma(-rr, zj, z[r]);
        else z[r] = L.g < G0 ? fma(-rr, zj, z[r]) : (L.g == G0 ? zj : z[r]);
      }
    });
#pragma unroll
    for (int r = 0; r < 4; ++r) y[0][r] = z[r];
    // rows above: y_i -= R_ip z
#pragma unroll
    for (int t = 1; t < NT; ++t) {
      const int rt = t - (NT - p);  // row tile of y[t], t >= NT - p
      if (rt >= 0) {
        const double* a = pp + kTile * rt;
        d4 acc = d4{y[t][0], y[t][1], y[t][2], y[t][3]};
#pragma unroll
        for (int r = 0; r < 4; ++r) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[tile_idx(L.cl, L.g + 4 * r)], -z[r], acc, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) y[t][r] = acc[r];
      }
    }
  }
}
