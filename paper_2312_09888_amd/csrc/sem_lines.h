// Line-exchange kernels for Q, the counts and the gradient (part of
// sem_kernels.hip; every order, FP64 and FP32).
//
// A workgroup of TH threads takes E elements (P = N + 1).  Every thread plays
// two roles: it owns the nodes t, t + TH, ... of the block, consecutive in
// memory, so that loads and stores touch whole cache lines; and it
// differentiates lines t, t + TH, ... of the 3 P^2 lines per element (r-, s-
// and t-lines together).  LDS holds every line's P values side by side: an
// owner writes its node's value to the three lines through the node, the
// line's thread replaces the values by their derivative in place (even-odd
// form, all outputs of a line), the owner reads its three derivatives back.
// A location belongs to one owner and one line thread, so a pass takes two
// barriers, and an owner writes the next field's value where it has just
// read.
//
// Bound: HBM (8 values per node for Q), with the vector ALU close behind:
// some 24 multiply-adds per node and field in the even-odd form, as many
// instructions again for the chain rule and the exchange.  The forms this
// replaced were bound by what they did beside that: a register pencil of two
// halves per element left 28 of 128 lanes idle at N = 9, held five nodes'
// geometry per thread (187 registers, two waves per SIMD) and applied D along
// r in the plain form; the node-per-thread tile of FP64 N = 8, 9 read D and
// three lines from LDS per node (LDS bound).
template <int N, int E_, int TH_, int PI_, int NF_>
struct LineCfg {
  static constexpr int P = N + 1, NP = P * P * P, LN = 3 * P * P;
  static constexpr int E = E_, TH = TH_;
  static constexpr int PI = PI_;                           // LDS pitch of a line
  static constexpr int NF = NF_;                           // fields per pass, 1 or 3
  static constexpr int NL = E * LN, NN = E * NP;
  static constexpr int R = (NN + TH - 1) / TH;             // nodes per thread
  static constexpr int SZ = NL * PI;                       // LDS values of a field
  static constexpr int NW = TH / 64;
  static_assert(TH % 64 == 0 && TH <= 1024 && PI >= P, "whole waves, whole lines");
  // Every thread owns a node in round r whatever the number of elements (the
  // last workgroup may have fewer than E).
  static constexpr bool full(int r) { return (r + 1) * TH <= NP; }
};

// Workgroup shapes {elements, threads, pitch, fields per pass}, from a sweep
// of Q alone (16,384 to 2^21 elements).  Two rules came out of it.  Threads:
// so many that two owner rounds (three at N = 8) nearly fill, whatever the
// lines do (line rounds leave whole waves idle, which cost nothing, while a
// third or fourth round costs registers): FP64 N = 9 took 27.6 ps per point
// with 384 threads and 18.0 with 512, N = 8 22.8 with 384 and 15.9 with 256;
// small elements keep one or two waves (a barrier of one wave is free).
// Pitch: the one that spreads a wave's lines over the banks (odd, or 4 or 20
// modulo 64 words for wide accesses): FP32 N = 7 10.4 with 8 and 7.0 with 9.
// Three fields per pass halve the barriers where LDS allows it without losing
// a wave (FP64 N = 4 17.6 against 14.1), one where it does not (FP64 N = 8
// 16.5 against 17.9).  ps per point of Q alone at 16,384 elements and more,
// this form against the fastest of the replaced ones, on one box: FP32 N =
// 2..9 9.8 / 7.2 / 8.1 / 8.5 / 8.1 / 7.3 / 7.9 / 13.1 against 10.3 / 7.5 / 9.5
// / 10.9 / 13.9 / 9.3 / 13.9 / 21.6; FP64 14.8 / 13.1 / 14.1 / 14.9 / 15.2 /
// 14.3 / 16.5 / 17.8 against 21.7 / 13.6 / 22.9 / 22.4 / 27.8 / 12.4 / 42.1 /
// 39.4 (6.4 and 12.8 are the bytes at 5 TB/s).  N = 1 has no lines in LDS
// (pair_deriv); its shapes are whole waves.  N = 7 FP64 had a form of its own,
// four waves on swizzled tiles fetched by direct loads, 2 to 5 % faster for Q
// alone of 65,536 elements: LineQ gives Q alone a shape of its own; with the
// counts this form is the faster one (the Q phase of the 65,536-element
// snapshot 0.555 before, 0.527 ms with the packed slots).
constexpr int kLineCfg64[kMaxOrder + 1][4] = {
    {0, 0, 0, 0},   {8, 64, 2, 3},  {9, 256, 3, 3},  {1, 64, 6, 3},  {1, 128, 5, 3},
    {1, 256, 6, 3}, {1, 128, 7, 3},  {1, 256, 10, 1}, {1, 256, 9, 1}, {1, 512, 10, 1}};
constexpr int kLineCfg32[kMaxOrder + 1][4] = {
    {0, 0, 0, 0},  {16, 64, 2, 3}, {9, 256, 3, 3}, {1, 64, 4, 3},  {2, 128, 5, 3},
    {1, 64, 7, 1}, {1, 128, 7, 3},  {1, 256, 9, 3}, {1, 256, 9, 3}, {1, 512, 10, 1}};
constexpr int line_cfg(int n, bool f64, int k) {
  return f64 ? kLineCfg64[n][k] : kLineCfg32[n][k];
}
template <int N, typename T>
using LineOf = LineCfg<N, line_cfg(N, sizeof(T) == 8, 0), line_cfg(N, sizeof(T) == 8, 1),
                       line_cfg(N, sizeof(T) == 8, 2), line_cfg(N, sizeof(T) == 8, 3)>;

// Shape of Q alone where another one than the counting kernel's, the gradient's
// and the batch's is faster; FAR: its eight fields exceed the shared 256 MiB
// cache (kLineNear).  Beyond it more bytes in flight a wave win, within it the
// shorter chain: a thread a node and all fields in one pass at order 7 in FP64
// (512 elements 6.6 us, 7.5 with the table's shape; 8,192: 57.7 and 59.0; 65,536:
// 489 and 475).  Order 3 in FP32: 524,288 elements 253 us with two elements a wave,
// 260 with one; 8,192: 9.1 and 8.1.  Order 2: 1,242,756 elements 280 us with nine
// elements a wave, 347 with the table's shape; 155,344: 42.0 and 39.9.
template <int N, typename T, bool FAR>
struct LineQ {
  using Shape = LineOf<N, T>;
};
template <>
struct LineQ<7, double, false> {
  using Shape = LineCfg<7, 1, 512, 10, 3>;
};
template <>
struct LineQ<3, float, true> {
  using Shape = LineCfg<3, 2, 64, 4, 3>;
};
template <>
struct LineQ<2, float, true> {
  using Shape = LineCfg<2, 9, 64, 3, 1>;
};
constexpr int64_t kLineNear = int64_t(256) << 20;

// Waves per SIMD to hold (launch bound): FP64 N = 6..9 sit a few registers
// around the limits of three and four waves; elsewhere the compiler's choice.
template <int N, typename T, class C>
constexpr int line_waves() {
  return sizeof(T) == 4 || N < 6 ? 1 : N == 6 || N == 8 ? 3 : C::NF == 3 ? 6 : 4;
}

// LDS values of `fields` fields' lines (order 1 needs none).
template <int N, class C>
constexpr int line_tile(int fields) { return N == 1 ? 1 : fields * C::SZ; }

// Offsets of an owner's nodes in their three lines.
template <class C>
struct LineOwner {
  int a[C::R][3];
  __device__ __forceinline__ explicit LineOwner(int t) {
    constexpr int P = C::P;
#pragma unroll
    for (int r = 0; r < C::R; ++r) {
      const int o = t + r * C::TH;
      const int el = C::E == 1 ? 0 : o / C::NP, n = o - el * C::NP;
      const int i = n % P, j = (n / P) % P, k = n / (P * P);
      const int base = el * C::LN;
      a[r][0] = (base + j + P * k) * C::PI + i;
      a[r][1] = (base + P * P + i + P * k) * C::PI + j;
      a[r][2] = (base + 2 * P * P + i + P * j) * C::PI + k;
    }
  }
};

// Value of the lane whose number differs in bit X (0, 1 or 2) only: quad_perm
// [1,0,3,2], [2,3,0,1]; [3,2,1,0] of the half row mirrored.
template <int X, typename T>
__device__ __forceinline__ T lane_across(T v) {
  if constexpr (X == 0) return dpp_move<0xb1>(v);
  else if constexpr (X == 1) return dpp_move<0x4e>(v);
  else return dpp_move<0x1b>(dpp_move<0x141>(v));
}

// Order 1: an element is eight neighbouring lanes and a line two of them, so
// the derivatives need no exchange: (f_1 - f_0) D_11 at both ends.  Q of
// 4,194,304 elements in FP32: 363 us with pencils, 395 through LDS, 185 so.
template <int X, class C, typename K, typename T>
__device__ __forceinline__ T pair_deriv(T v, K d11, int t) {
  const K own = (K)v, other = (K)lane_across<X>(v);
  return (T)(d11 * (((t >> X) & 1) ? own - other : other - own));
}

// F fields through the exchange: values at the owner's nodes in f, reference
// derivatives (r, s, t) there in g.  nn nodes and nl lines exist.
template <int N, class C, int F, typename T>
__device__ __forceinline__ void line_pass(const T (*f)[C::R], const LineOwner<C>& own,
                                          const coef_t<N, T>* __restrict__ d, T* tile, int t,
                                          int nn, int nl, T (*g)[C::R][3]) {
  constexpr int P = C::P, TASKS = F * C::NL;
  if constexpr (N == 1) {
    const coef_t<N, T> d11 = coef(d, 3);
#pragma unroll
    for (int c = 0; c < F; ++c)
#pragma unroll
      for (int r = 0; r < C::R; ++r) {
        g[c][r][0] = pair_deriv<0, C>(f[c][r], d11, t);
        g[c][r][1] = pair_deriv<1, C>(f[c][r], d11, t);
        g[c][r][2] = pair_deriv<2, C>(f[c][r], d11, t);
      }
    return;
  }
#pragma unroll
  for (int c = 0; c < F; ++c)
#pragma unroll
    for (int r = 0; r < C::R; ++r)
      if (C::full(r) || t + r * C::TH < nn) {
#pragma unroll
        for (int x = 0; x < 3; ++x) tile[c * C::SZ + own.a[r][x]] = f[c][r];
      }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < (TASKS + C::TH - 1) / C::TH; ++q) {
    const int task = t + q * C::TH;
    bool live = (q + 1) * C::TH <= TASKS || task < TASKS;
    if constexpr (C::E > 1) live = live && (F == 1 ? task : task % C::NL) < nl;
    if (live) {
      T* line = tile + task * C::PI;
      T v[P], out[P];
#pragma unroll
      for (int m = 0; m < P; ++m) v[m] = line[m];
      line_deriv_all<P>(d, v, out);
#pragma unroll
      for (int m = 0; m < P; ++m) line[m] = out[m];
    }
  }
  __syncthreads();
#pragma unroll
  for (int c = 0; c < F; ++c)
#pragma unroll
    for (int r = 0; r < C::R; ++r)
      if (C::full(r) || t + r * C::TH < nn) {
#pragma unroll
        for (int x = 0; x < 3; ++x) g[c][r][x] = tile[c * C::SZ + own.a[r][x]];
      }
}

// Three fields, C::NF at a time.
template <int N, class C, typename T>
__device__ __forceinline__ void line_pass3(const T (&f)[3][C::R], const LineOwner<C>& own,
                                           const coef_t<N, T>* __restrict__ d, T* tile, int t,
                                           int nn, int nl, T (&g)[3][C::R][3]) {
#pragma unroll
  for (int c = 0; c < 3; c += C::NF)
    line_pass<N, C, C::NF>(f + c, own, d, tile, t, nn, nl, g + c);
}

template <class C, typename T>
__device__ __forceinline__ void line_load(const T* __restrict__ src, int t, int nn,
                                          T (&f)[C::R]) {
#pragma unroll
  for (int r = 0; r < C::R; ++r)
    if (C::full(r) || t + r * C::TH < nn) f[r] = src[t + r * C::TH];
}

// Where a thread owns nodes of several elements, or another shape takes over
// with the size, a node's sums are written out in multiply-adds: which products
// the compiler contracts depends on the code around them, and an element's
// values must not depend on where in the list it stands.  (Elsewhere its choice
// is as fast or faster: FP64 N = 8, 9 3 %, N = 2 5 %.)
template <int N, typename T>
constexpr bool kLineFixed = sizeof(T) == 4 ? N <= 4 : N == 7;
template <bool FIXED, typename T>
__device__ __forceinline__ T cross2(T a, T b, T c, T d) {   // a b - c d
  if constexpr (FIXED) return fma(a, b, -(c * d));
  else return a * b - c * d;
}
template <bool FIXED, typename T>
__device__ __forceinline__ T dot3(T a0, T b0, T a1, T b1, T a2, T b2) {
  if constexpr (FIXED) return fma(a2, b2, fma(a0, b0, a1 * b1));
  else return a0 * b0 + a1 * b1 + a2 * b2;
}

// 1 / det J: FP32 the hardware reciprocal (1 ulp), FP64 the refined one.
__device__ __forceinline__ float line_recip(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ double line_recip(double x) { return recip_refined(x); }

// J^-1 at the owner's nodes from the coordinates; false if det J is not
// positive at one of them.
template <int N, class C, typename T>
__device__ __forceinline__ bool line_geometry(const T (&f)[3][C::R], const LineOwner<C>& own,
                                              const coef_t<N, T>* __restrict__ d, T* tile, int t,
                                              int nn, int nl, InvJac<T> (&kk)[C::R]) {
  T g[3][C::R][3];
  line_pass3<N, C>(f, own, d, tile, t, nn, nl, g);
  bool ok = true;
#pragma unroll
  for (int r = 0; r < C::R; ++r) {
    InvJac<T>& K = kk[r];
    const T xr = g[0][r][0], xs = g[0][r][1], xt = g[0][r][2];
    const T yr = g[1][r][0], ys = g[1][r][1], yt = g[1][r][2];
    const T zr = g[2][r][0], zs = g[2][r][1], zt = g[2][r][2];
    constexpr bool FX = kLineFixed<N, T>;
    const T c0 = cross2<FX>(ys, zt, yt, zs), c1 = cross2<FX>(yt, zr, yr, zt);
    const T c2 = cross2<FX>(yr, zs, ys, zr);
    const T det = dot3<FX>(xr, c0, xs, c1, xt, c2);
    const T inv = line_recip(det);
    K.rx = c0 * inv;
    K.ry = cross2<FX>(xt, zs, xs, zt) * inv;
    K.rz = cross2<FX>(xs, yt, xt, ys) * inv;
    K.sx = c1 * inv;
    K.sy = cross2<FX>(xr, zt, xt, zr) * inv;
    K.sz = cross2<FX>(xt, yr, xr, yt) * inv;
    K.tx = c2 * inv;
    K.ty = cross2<FX>(xs, zr, xr, zs) * inv;
    K.tz = cross2<FX>(xr, ys, xs, yr) * inv;
    if (C::full(r) || t + r * C::TH < nn) ok = ok && det > T(0);
  }
  return ok;
}

// ---------------------------------------------------------------------------
// counting from node values held by their owners
// ---------------------------------------------------------------------------
//
// The bits (value > c) of 64 consecutive nodes are one ballot; the ballots of
// a block's nodes, written to LDS in node order, are a bit string in which a
// row of P nodes is P consecutive bits.  A wave takes one (isovalue, element),
// up to order 4 several of them, and a lane a row of N cells: the four rows of
// bits around it give by bit operations the cells whose corners differ, and
// only those (a few per cent) look their case up.  Against a word per node holding four isovalues' bits
// and eight reads per cell whatever its case, the counts cost about half the
// instructions.

constexpr int kBitGroup = 4;     // isovalues per round
template <class C>
struct LineBits {
  static constexpr int W = (C::NN + 63) / 64;      // ballots per isovalue
  uint64_t bits[kBitGroup][W + 1];                 // one word past the last row's
};

// P bits from bit b on.
__device__ __forceinline__ uint32_t bit_row(const uint32_t* bits, int b) {
  const uint32_t* w = bits + (b >> 5);
  return __builtin_amdgcn_alignbit(w[1], w[0], b & 31);
}

// Lanes that count one element at one isovalue: the rows of cells, rounded up
// to what one DPP reduction adds up (a lane, a quad, a row of 16, the wave).
// Extraction at four isovalues, FP32: 155,344 order-2 elements 216 us with a
// wave for each count, 168 so; 524,288 order-1 elements 560 and 399.
constexpr int count_lanes_of(int n) {
  return n == 1 ? 1 : n == 2 ? 4 : n <= 4 ? 16 : 64;
}

// Triangles + (active cells << 16) of one element at one isovalue, summed
// over G lanes into the last of them (lane: the lane's number among them);
// bits: the isovalue's bit string, bit0: the element's first node.  dump: the
// element's cells' cases (optional).  Every lane of the wave must be active;
// lanes without an element pass live = false.
template <int N, int G = 64>
__device__ __forceinline__ uint32_t count_rows(const uint32_t* bits, int bit0, int lane,
                                               const uint8_t* tab, uint8_t* dump = nullptr,
                                               bool live = true) {
  constexpr int P = N + 1;
  uint32_t sum = 0;
#pragma unroll
  for (int q = 0; q < (N * N + G - 1) / G; ++q) {
    const int row = lane + G * q;
    if (live && row < N * N) {
      const int j = row % N, k = row / N;
      const int b = bit0 + (j + P * k) * P;
      const uint32_t r0 = bit_row(bits, b), r1 = bit_row(bits, b + P);
      const uint32_t r2 = bit_row(bits, b + P * P), r3 = bit_row(bits, b + P * P + P);
      uint32_t any = r0 | r1 | r2 | r3, all = r0 & r1 & r2 & r3;
      any |= any >> 1;
      all &= all >> 1;
      uint32_t act = any & ~all & ((1u << N) - 1);
      sum += (uint32_t)__builtin_popcount(act) << 16;
      if (dump) {
        for (int i = 0; i < N; ++i)
          dump[row * N + i] = (uint8_t)(((r0 >> i) & 3) | (((r1 >> i) & 3) << 2) |
                                        (((r2 >> i) & 3) << 4) | (((r3 >> i) & 3) << 6));
      }
      while (act) {
        const int i = __builtin_ctz(act);
        act &= act - 1;
        sum += tab[((r0 >> i) & 3) | (((r1 >> i) & 3) << 2) | (((r2 >> i) & 3) << 4) |
                   (((r3 >> i) & 3) << 6)];
      }
    }
  }
  if constexpr (G == 1) return sum;
  else if constexpr (G == 4) return quad_sum(sum);
  else if constexpr (G == 16) return row_sum16(sum);
  else return wave_sum_to63(sum);
}

// Counts of the block's elements e .. e + ne - 1 at every isovalue from the
// owners' values qv (NaN as -inf, or NaN: both compare below).  tab: the 256
// triangle counts in LDS, published by the caller or by the first barrier.
template <int N, class C, typename T>
__device__ __forceinline__ void line_count(const T (&qv)[C::R], int64_t e, int t, int ne, int nn,
                                           const CountSink<T>& sink, LineBits<C>& sb,
                                           const uint8_t* tab) {
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
  for (int g = 0; g < sink.n_iso; g += kBitGroup) {
    const int m = sink.n_iso - g < kBitGroup ? sink.n_iso - g : kBitGroup;
    if (g > 0) __syncthreads();   // every wave is done with the previous bits
#pragma unroll
    for (int s = 0; s < kBitGroup; ++s) {
      if (s < m) {
        const T c = sink.iso.v[g + s];
#pragma unroll
        for (int r = 0; r < C::R; ++r) {
          const uint64_t b = __ballot((C::full(r) || t + r * C::TH < nn) && qv[r] > c);
          const int w = wave + r * C::NW;
          if (lane == 0 && w < LineBits<C>::W) sb.bits[s][w] = b;
        }
      }
    }
    __syncthreads();
    constexpr int G = count_lanes_of(N), W = 64 / G;   // lanes a count, counts a wave
    for (int p0 = wave * W; p0 < m * ne; p0 += C::NW * W) {
      const int p = W == 1 ? p0 : p0 + lane / G;
      const bool live = W == 1 || p < m * ne;
      const int s = !live ? 0 : C::E == 1 ? p : p / ne, el = C::E == 1 || !live ? 0 : p - s * ne;
      const uint32_t sum = count_rows<N, G>(reinterpret_cast<const uint32_t*>(sb.bits[s]),
                                            el * C::NP, lane % G, tab, nullptr, live);
      if (live && lane % G == G - 1)
        sink.cnt[(int64_t)(g + s) * sink.n_elem + e + el] = (int)sum;
    }
  }
}

// ---------------------------------------------------------------------------
// Q, |omega|, ranges and counts
// ---------------------------------------------------------------------------

template <int N, typename T, bool COUNT, class C>
__device__ __forceinline__ void qcrit_lines_elem(
    int64_t e, int t, int ne, const coef_t<N, T>* __restrict__ dmat, const T* __restrict__ x,
    const T* __restrict__ y, const T* __restrict__ z, const T* __restrict__ u,
    const T* __restrict__ v, const T* __restrict__ w, T* __restrict__ q, T* __restrict__ om,
    T* __restrict__ qmm, int32_t* __restrict__ status, const CountSink<T>* sink = nullptr) {
  constexpr int NP = C::NP, R = C::R, NW = C::NW;
  __shared__ __align__(16) T tile[line_tile<N, C>(C::NF)];
  __shared__ T red[2 * NW];
  __shared__ uint32_t s_tab[COUNT ? 64 : 1];
  const int64_t base = e * NP;
  const int nn = C::E == 1 ? C::NN : ne * NP, nl = C::E == 1 ? C::NL : ne * C::LN;
  const LineOwner<C> own(t);
  T fx[3][R], fu[3][R];
  line_load<C>(x + base, t, nn, fx[0]);
  line_load<C>(y + base, t, nn, fx[1]);
  line_load<C>(z + base, t, nn, fx[2]);
  line_load<C>(u + base, t, nn, fu[0]);
  line_load<C>(v + base, t, nn, fu[1]);
  line_load<C>(w + base, t, nn, fu[2]);
  uint32_t tab4 = 0;
  if (COUNT && t < 64) tab4 = reinterpret_cast<const uint32_t*>(sink->ntri)[t];
  InvJac<T> kk[R];
  const bool ok = line_geometry<N, C>(fx, own, dmat, tile, t, nn, nl, kk);
  T qv[R], ov[R];
  if constexpr (kLineFixed<N, T>) {
    // rows of the velocity gradient, folded into Q and |omega|^2 as they come
    T a01[R], a02[R], a12[R];
    auto row = [&](int c, const T (&g)[R][3]) {
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const InvJac<T>& K = kk[r];
        const T a0 = dot3<true>(g[r][0], K.rx, g[r][1], K.sx, g[r][2], K.tx);
        const T a1 = dot3<true>(g[r][0], K.ry, g[r][1], K.sy, g[r][2], K.ty);
        const T a2 = dot3<true>(g[r][0], K.rz, g[r][1], K.sz, g[r][2], K.tz);
        if (c == 0) {
          qv[r] = a0;
          a01[r] = a1;
          a02[r] = a2;
        } else if (c == 1) {
          qv[r] = fma(T(2), a01[r] * a0, fma(qv[r], qv[r], a1 * a1));
          ov[r] = a0 - a01[r];
          a12[r] = a2;
        } else {
          qv[r] = T(-0.5) * fma(T(2), fma(a02[r], a0, a12[r] * a1), fma(a2, a2, qv[r]));
          const T w1 = a1 - a12[r], w2 = a02[r] - a0;
          ov[r] = vort_root(fma(w2, w2, fma(ov[r], ov[r], w1 * w1)));
        }
      }
    };
    T g[C::NF][R][3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      if (c % C::NF == 0) line_pass<N, C, C::NF>(fu + c, own, dmat, tile, t, nn, nl, g);
      row(c, g[c % C::NF]);
    }
  } else if constexpr (C::NF == 3) {
    T g[3][R][3];
    line_pass3<N, C>(fu, own, dmat, tile, t, nn, nl, g);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const InvJac<T>& K = kk[r];
      T a[3][3];
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        a[c][0] = g[c][r][0] * K.rx + g[c][r][1] * K.sx + g[c][r][2] * K.tx;
        a[c][1] = g[c][r][0] * K.ry + g[c][r][1] * K.sy + g[c][r][2] * K.ty;
        a[c][2] = g[c][r][0] * K.rz + g[c][r][1] * K.sz + g[c][r][2] * K.tz;
      }
      qv[r] = T(-0.5) * (a[0][0] * a[0][0] + a[1][1] * a[1][1] + T(2) * (a[0][1] * a[1][0]) +
                         a[2][2] * a[2][2] + T(2) * (a[0][2] * a[2][0] + a[1][2] * a[2][1]));
      const T w1 = a[2][1] - a[1][2], w2 = a[0][2] - a[2][0], w3 = a[1][0] - a[0][1];
      ov[r] = vort_root(w3 * w3 + w1 * w1 + w2 * w2);
    }
  } else {
    // rows of the velocity gradient folded into Q and |omega|^2 as they come
    T a01[R], a02[R], a12[R], g[1][R][3];
    line_pass<N, C, 1>(fu, own, dmat, tile, t, nn, nl, g);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const InvJac<T>& K = kk[r];
      const T fr = g[0][r][0], fs = g[0][r][1], ft = g[0][r][2];
      const T a00 = fr * K.rx + fs * K.sx + ft * K.tx;
      a01[r] = fr * K.ry + fs * K.sy + ft * K.ty;
      a02[r] = fr * K.rz + fs * K.sz + ft * K.tz;
      qv[r] = a00 * a00;
    }
    line_pass<N, C, 1>(fu + 1, own, dmat, tile, t, nn, nl, g);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const InvJac<T>& K = kk[r];
      const T fr = g[0][r][0], fs = g[0][r][1], ft = g[0][r][2];
      const T a10 = fr * K.rx + fs * K.sx + ft * K.tx;
      const T a11 = fr * K.ry + fs * K.sy + ft * K.ty;
      a12[r] = fr * K.rz + fs * K.sz + ft * K.tz;
      qv[r] = qv[r] + a11 * a11 + T(2) * (a01[r] * a10);
      const T w3 = a10 - a01[r];
      ov[r] = w3 * w3;
    }
    line_pass<N, C, 1>(fu + 2, own, dmat, tile, t, nn, nl, g);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const InvJac<T>& K = kk[r];
      const T fr = g[0][r][0], fs = g[0][r][1], ft = g[0][r][2];
      const T a20 = fr * K.rx + fs * K.sx + ft * K.tx;
      const T a21 = fr * K.ry + fs * K.sy + ft * K.ty;
      const T a22 = fr * K.rz + fs * K.sz + ft * K.tz;
      qv[r] = T(-0.5) * (qv[r] + a22 * a22 + T(2) * (a02[r] * a20 + a12[r] * a21));
      const T w1 = a21 - a12[r], w2 = a02[r] - a20;
      ov[r] = vort_root(ov[r] + w1 * w1 + w2 * w2);
    }
  }
  T mn = pos_inf<T>(), mx = neg_inf<T>();
#pragma unroll
  for (int r = 0; r < R; ++r) {
    if (C::full(r) || t + r * C::TH < nn) {
      const int64_t o = base + t + r * C::TH;
      if (q) q[o] = qv[r];
      if (om) om[o] = ov[r];
      qv[r] = qv[r] != qv[r] ? neg_inf<T>() : qv[r];
      mn = qv[r] < mn ? qv[r] : mn;
      mx = qv[r] > mx ? qv[r] : mx;
    }
  }
  // an inverted element (rare) is flagged by its own lanes: no block vote
  if (!ok && status) atomicOr(status, SEM_FLAG_BAD_JACOBIAN);
  if (COUNT && t < 64) s_tab[t] = tab4;
  if constexpr (C::E == 1) {
    wave_minmax(mn, mx);
    if ((t & 63) == 63) {
      red[t >> 6] = mn;
      red[NW + (t >> 6)] = mx;
    }
    __syncthreads();
    if (qmm && t == 0) {
      mn = red[0];
      mx = red[NW];
#pragma unroll
      for (int i = 1; i < NW; ++i) {
        mn = fmin(mn, red[i]);
        mx = fmax(mx, red[NW + i]);
      }
      qmm[2 * e] = mn;
      qmm[2 * e + 1] = mx;
    }
  } else if constexpr (N == 1) {
    // ranges over an element's eight lanes
#pragma unroll
    for (int r = 0; r < R; ++r) {
      T a = qv[r], b = qv[r];
      a = fmin(a, lane_across<0>(a));
      b = fmax(b, lane_across<0>(b));
      a = fmin(a, lane_across<1>(a));
      b = fmax(b, lane_across<1>(b));
      a = fmin(a, lane_across<2>(a));
      b = fmax(b, lane_across<2>(b));
      const int o = t + r * C::TH;
      if (qmm && (t & 7) == 0 && o < nn) {
        qmm[2 * (e + o / 8)] = a;
        qmm[2 * (e + o / 8) + 1] = b;
      }
    }
  } else {
    // ranges: the values through LDS, a wave per element
    __syncthreads();   // every derivative of the last pass is read
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (C::full(r) || t + r * C::TH < nn) tile[t + r * C::TH] = qv[r];
    __syncthreads();
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
    for (int el = wave; qmm && el < ne; el += NW) {
      T a = pos_inf<T>(), b = neg_inf<T>();
      for (int n = lane; n < NP; n += 64) {
        const T c = tile[el * NP + n];
        a = c < a ? c : a;
        b = c > b ? c : b;
      }
      wave_minmax(a, b);
      if (lane == 63) {
        qmm[2 * (e + el)] = a;
        qmm[2 * (e + el) + 1] = b;
      }
    }
  }
  if constexpr (COUNT) {
    clear_active(sink->active, sink->n_iso);
    __shared__ LineBits<C> sb;
    line_count<N, C>(qv, e, t, ne, nn, *sink, sb, reinterpret_cast<const uint8_t*>(s_tab));
  }
}

template <int N, typename T, class C>
__global__ void __launch_bounds__((C::TH), (line_waves<N, T, C>()))
qcrit_lines(const coef_t<N, T>* __restrict__ dmat, const T* __restrict__ x,
            const T* __restrict__ y, const T* __restrict__ z, const T* __restrict__ u,
            const T* __restrict__ v, const T* __restrict__ w, T* __restrict__ q,
            T* __restrict__ om, T* __restrict__ qmm, int32_t* __restrict__ status,
            int64_t e_begin, int64_t n_elem) {
  const int64_t e0 = e_begin + (int64_t)blockIdx.x * C::E;
  const int ne = n_elem - e0 < C::E ? (int)(n_elem - e0) : C::E;
  qcrit_lines_elem<N, T, false, C>(e0, threadIdx.x, ne, dmat, x, y, z, u, v, w, q, om, qmm, status);
}

// Q, |omega|, range and the per-(isovalue, element) counts in one pass.
template <int N, typename T, class C>
__global__ void __launch_bounds__((C::TH), (line_waves<N, T, C>()))
qcount_lines(const coef_t<N, T>* __restrict__ dmat, const T* __restrict__ x,
             const T* __restrict__ y, const T* __restrict__ z, const T* __restrict__ u,
             const T* __restrict__ v, const T* __restrict__ w, T* __restrict__ q,
             T* __restrict__ om, T* __restrict__ qmm, int32_t* __restrict__ status,
             int64_t e_begin, CountSink<T> sink) {
  const int64_t e0 = e_begin + (int64_t)blockIdx.x * C::E;
  const int ne = sink.n_elem - e0 < C::E ? (int)(sink.n_elem - e0) : C::E;
  qcrit_lines_elem<N, T, true, C>(e0, threadIdx.x, ne, dmat, x, y, z, u, v, w, q, om, qmm, status,
                               &sink);
}

// Physical gradient of f.
template <int N, typename T, class C>
__global__ void __launch_bounds__((C::TH), (line_waves<N, T, C>()))
derivs_lines(const coef_t<N, T>* __restrict__ dmat, const T* __restrict__ x,
             const T* __restrict__ y, const T* __restrict__ z, const T* __restrict__ f,
             T* __restrict__ gx, T* __restrict__ gy, T* __restrict__ gz,
             int32_t* __restrict__ status, int64_t e_begin, int64_t n_elem) {
  constexpr int R = C::R;
  __shared__ __align__(16) T tile[line_tile<N, C>(C::NF)];
  const int t = threadIdx.x;
  const int64_t e0 = e_begin + (int64_t)blockIdx.x * C::E, base = e0 * C::NP;
  const int ne = C::E == 1 || n_elem - e0 >= C::E ? C::E : (int)(n_elem - e0);
  const int nn = C::E == 1 ? C::NN : ne * C::NP, nl = C::E == 1 ? C::NL : ne * C::LN;
  const LineOwner<C> own(t);
  T fx[3][R], ff[1][R], g[1][R][3];
  line_load<C>(x + base, t, nn, fx[0]);
  line_load<C>(y + base, t, nn, fx[1]);
  line_load<C>(z + base, t, nn, fx[2]);
  line_load<C>(f + base, t, nn, ff[0]);
  InvJac<T> kk[R];
  const bool ok = line_geometry<N, C>(fx, own, dmat, tile, t, nn, nl, kk);
  line_pass<N, C, 1>(ff, own, dmat, tile, t, nn, nl, g);
#pragma unroll
  for (int r = 0; r < R; ++r) {
    if (C::full(r) || t + r * C::TH < nn) {
      const InvJac<T>& K = kk[r];
      const int64_t o = base + t + r * C::TH;
      constexpr bool FX = kLineFixed<N, T>;
      gx[o] = dot3<FX>(g[0][r][0], K.rx, g[0][r][1], K.sx, g[0][r][2], K.tx);
      gy[o] = dot3<FX>(g[0][r][0], K.ry, g[0][r][1], K.sy, g[0][r][2], K.ty);
      gz[o] = dot3<FX>(g[0][r][0], K.rz, g[0][r][1], K.sz, g[0][r][2], K.tz);
    }
  }
  if (!ok && status) atomicOr(status, SEM_FLAG_BAD_JACOBIAN);
}
