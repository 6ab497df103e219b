// Register-resident 2D FFT engine for gfx950 (wave64).
//
// A P x P complex field is spread over NT = P * TPR threads of a workgroup,
// TPR = P / E threads per line, E elements per thread.  Thread t owns line
// l = t / TPR and lane-in-line q (the TPR lanes of a line are adjacent lanes
// of one wavefront).  For TPR <= 4, q = t % TPR.  For TPR = 8 the lanes of
// the upper half are relabelled, q = p ^ 3 for p = t % 8 >= 4 (lanes
// 4, 5, 6, 7 hold q = 7, 6, 5, 4), so that the distance-4 partner of every
// lane, q ^ 4, is the lane 7 - p: one row_half_mirror move instead of a quad
// permute and a mirror.  The partners at distance 2 and 1 stay p ^ 2, p ^ 1.
//
//   "strided"  layout: element index  x = q + TPR * n,        n = 0..E-1
//   "blocked"  layout: element index  k + E * bitrev(q),      k = 0..E-1
//
// A forward line transform takes strided data to blocked spectra: an E-point
// FFT in registers on the stride-TPR subsequence, a twiddle w_P^{q k}, then a
// TPR-point DFT across the lanes (radix-2 decimation in frequency through
// lane shuffles, which leaves the output blocks in bit-reversed lane order).
// The inverse line transform runs the same steps backwards.  Both are
// unnormalized: inv(fwd(x)) = P x.
//
// 2D: rows (index x, line = y) and columns (index y, line = kx).  The field
// moves between row and column ownership through an LDS transpose, one real
// component at a time (both at once where the kernel has the LDS for two
// planes), through a padded P x P buffer per component.
//
//   row real (strided in x) --fwd rows--> row spectra (blocked in kx)
//     --T1--> column real (strided in y) --fwd cols--> column spectra
//   and back with the inverse transforms and T2.
#pragma once
#include <hip/hip_runtime.h>

#include <utility>

namespace qb {

// ------------------------------------------------------------------ constexpr trig
// Taylor series after reduction to [-pi/4, pi/4]; used only for the compile-time
// twiddles of the in-register transforms.
constexpr double kPi = 3.14159265358979323846264338327950288;

constexpr double cx_sin_small(double x) {
  double term = x, sum = x;
  for (int k = 1; k < 14; ++k) {
    term *= -x * x / ((2.0 * k) * (2.0 * k + 1.0));
    sum += term;
  }
  return sum;
}
constexpr double cx_cos_small(double x) {
  double term = 1.0, sum = 1.0;
  for (int k = 1; k < 14; ++k) {
    term *= -x * x / ((2.0 * k - 1.0) * (2.0 * k));
    sum += term;
  }
  return sum;
}
// cos / sin of 2 pi a / b for integers 0 <= a < b, b a power of two.
constexpr double cx_cos_frac(int a, int b) {
  // octant reduction: angle = 2 pi a / b = (pi/4) * (8a/b)
  const int a8 = a * 8;
  const int oct = a8 / b;               // 0..7
  const double r = (double)(a8 - oct * b) / b * (kPi / 4.0);  // [0, pi/4)
  switch (oct) {
    case 0: return cx_cos_small(r);
    case 1: return cx_sin_small(kPi / 4.0 - r);
    case 2: return -cx_sin_small(r);
    case 3: return -cx_cos_small(kPi / 4.0 - r);
    case 4: return -cx_cos_small(r);
    case 5: return -cx_sin_small(kPi / 4.0 - r);
    case 6: return cx_sin_small(r);
    default: return cx_cos_small(kPi / 4.0 - r);
  }
}
constexpr double cx_sin_frac(int a, int b) {
  const int a8 = a * 8;
  const int oct = a8 / b;
  const double r = (double)(a8 - oct * b) / b * (kPi / 4.0);
  switch (oct) {
    case 0: return cx_sin_small(r);
    case 1: return cx_cos_small(kPi / 4.0 - r);
    case 2: return cx_cos_small(r);
    case 3: return cx_sin_small(kPi / 4.0 - r);
    case 4: return -cx_sin_small(r);
    case 5: return -cx_cos_small(kPi / 4.0 - r);
    case 6: return -cx_cos_small(r);
    default: return -cx_sin_small(kPi / 4.0 - r);
  }
}

template <int A, int B>
struct Tw {
  static constexpr double c = cx_cos_frac(A, B);
  static constexpr double s = cx_sin_frac(A, B);
};

constexpr int ilog2(int n) { return n <= 1 ? 0 : 1 + ilog2(n / 2); }
constexpr int bitrev_c(int v, int bits) {
  int r = 0;
  for (int i = 0; i < bits; ++i) r |= ((v >> i) & 1) << (bits - 1 - i);
  return r;
}
__host__ __device__ inline int bitrev_rt(int v, int bits) {
  int r = 0;
  for (int i = 0; i < bits; ++i) r |= ((v >> i) & 1) << (bits - 1 - i);
  return r;
}

template <typename T>
__device__ __forceinline__ void cmul(T ar, T ai, T br, T bi, T& cr, T& ci) {
  const T r = ar * br - ai * bi;
  ci = ar * bi + ai * br;
  cr = r;
}

// ------------------------------------------------------------------ in-register FFT
// y[k] = sum_n x[O + S n] exp(DIR * 2 pi i n k / E), natural order in and out.
template <typename T, int E, int DIR>
struct RegFft {
  template <int S, int O, int IN_N>
  static __device__ __forceinline__ void run(const T (&xr)[IN_N], const T (&xi)[IN_N], T (&yr)[E],
                                             T (&yi)[E]) {
    if constexpr (E == 1) {
      yr[0] = xr[O];
      yi[0] = xi[O];
    } else {
      constexpr int H = E / 2;
      T er[H], ei[H], orr[H], oi[H];
      RegFft<T, H, DIR>::template run<2 * S, O, IN_N>(xr, xi, er, ei);
      RegFft<T, H, DIR>::template run<2 * S, O + S, IN_N>(xr, xi, orr, oi);
      butterflies(er, ei, orr, oi, yr, yi, std::make_integer_sequence<int, H>{});
    }
  }

  template <int H, int... K>
  static __device__ __forceinline__ void butterflies(const T (&er)[H], const T (&ei)[H], const T (&orr)[H],
                                                     const T (&oi)[H], T (&yr)[E], T (&yi)[E],
                                                     std::integer_sequence<int, K...>) {
    (bfly<H, K>(er, ei, orr, oi, yr, yi), ...);
  }

  template <int H, int K>
  static __device__ __forceinline__ void bfly(const T (&er)[H], const T (&ei)[H], const T (&orr)[H],
                                              const T (&oi)[H], T (&yr)[E], T (&yi)[E]) {
    T tr, ti;
    if constexpr (K == 0) {
      tr = orr[K];
      ti = oi[K];
    } else if constexpr (4 * K == E) {
      // w = exp(DIR * i pi / 2) = DIR * i
      if constexpr (DIR < 0) {
        tr = oi[K];
        ti = -orr[K];
      } else {
        tr = -oi[K];
        ti = orr[K];
      }
    } else {
      constexpr T c = (T)Tw<K, E>::c;
      constexpr T s = (T)(DIR * Tw<K, E>::s);
      tr = orr[K] * c - oi[K] * s;
      ti = orr[K] * s + oi[K] * c;
    }
    yr[K] = er[K] + tr;
    yi[K] = ei[K] + ti;
    yr[K + H] = er[K] - tr;
    yi[K + H] = ei[K] - ti;
  }
};

template <typename T, int E, int DIR>
__device__ __forceinline__ void reg_fft(T (&zr)[E], T (&zi)[E]) {
  T yr[E], yi[E];
  RegFft<T, E, DIR>::template run<1, 0, E>(zr, zi, yr, yi);
#pragma unroll
  for (int k = 0; k < E; ++k) {
    zr[k] = yr[k];
    zi[k] = yi[k];
  }
}

// ------------------------------------------------------------------ lane shuffles
// Value of lane (lane ^ MASK) for MASK in {1, 2}, by a DPP quad_perm move,
// and for MASK = 7 the value of lane 7 - i in each group of 8 lanes
// (row_half_mirror): the distance-4 partner under the TPR = 8 lane labels.
template <int MASK>
__device__ __forceinline__ int xor_lane_i32(int v) {
  if constexpr (MASK == 1) {
    return __builtin_amdgcn_mov_dpp(v, 0xB1, 0xF, 0xF, false);  // quad_perm [1,0,3,2]
  } else if constexpr (MASK == 2) {
    return __builtin_amdgcn_mov_dpp(v, 0x4E, 0xF, 0xF, false);  // quad_perm [2,3,0,1]
  } else {
    static_assert(MASK == 7, "lane mask must be 1, 2 or 7");
    return __builtin_amdgcn_mov_dpp(v, 0x141, 0xF, 0xF, false);  // row_half_mirror
  }
}

template <int MASK>
__device__ __forceinline__ float xor_lane(float v) {
  return __int_as_float(xor_lane_i32<MASK>(__float_as_int(v)));
}

template <int MASK>
__device__ __forceinline__ double xor_lane(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = xor_lane_i32<MASK>((int)(b & 0xffffffffll));
  const int hi = xor_lane_i32<MASK>((int)(b >> 32));
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// z += s z(partner lane) for every element.  In float32 one instruction per
// element (the DPP read is the first source of a v_fmac), written as asm in
// blocks of eight: the compiler leaves the move and the multiply-add apart.  A
// DPP read needs two wait states after the VALU write of its register, which
// nothing outside the asm block guarantees; inside a block every instruction
// reads a register of its own.
#define QB_FMAC_DPP8(CTRL)                                                                              \
  asm("s_nop 1\n\t"                                                                                     \
      "v_fmac_f32_dpp %0, %0, %8 " CTRL " row_mask:0xf bank_mask:0xf\n\t"                               \
      "v_fmac_f32_dpp %1, %1, %8 " CTRL " row_mask:0xf bank_mask:0xf\n\t"                               \
      "v_fmac_f32_dpp %2, %2, %8 " CTRL " row_mask:0xf bank_mask:0xf\n\t"                               \
      "v_fmac_f32_dpp %3, %3, %8 " CTRL " row_mask:0xf bank_mask:0xf\n\t"                               \
      "v_fmac_f32_dpp %4, %4, %8 " CTRL " row_mask:0xf bank_mask:0xf\n\t"                               \
      "v_fmac_f32_dpp %5, %5, %8 " CTRL " row_mask:0xf bank_mask:0xf\n\t"                               \
      "v_fmac_f32_dpp %6, %6, %8 " CTRL " row_mask:0xf bank_mask:0xf\n\t"                               \
      "v_fmac_f32_dpp %7, %7, %8 " CTRL " row_mask:0xf bank_mask:0xf"                                    \
      : "+v"(z[b]), "+v"(z[b + 1]), "+v"(z[b + 2]), "+v"(z[b + 3]), "+v"(z[b + 4]), "+v"(z[b + 5]),     \
        "+v"(z[b + 6]), "+v"(z[b + 7])                                                                   \
      : "v"(s))
template <int MASK, int E>
__device__ __forceinline__ void add_lanes(float (&z)[E], float s) {
  static_assert(E % 8 == 0, "blocks of eight");
#pragma unroll
  for (int b = 0; b < E; b += 8) {
    if constexpr (MASK == 1)
      QB_FMAC_DPP8("quad_perm:[1,0,3,2]");
    else if constexpr (MASK == 2)
      QB_FMAC_DPP8("quad_perm:[2,3,0,1]");
    else
      QB_FMAC_DPP8("row_half_mirror");
  }
}
#undef QB_FMAC_DPP8
template <int MASK, int E>
__device__ __forceinline__ void add_lanes(double (&z)[E], double s) {
#pragma unroll
  for (int k = 0; k < E; ++k) z[k] = fma(xor_lane<MASK>(z[k]), s, z[k]);
}

// ------------------------------------------------------------------ engine
// Whether the spectra carry the lane signs of lanes_fwd; the host's table of
// -k (negk, for k_grad_pre) has to agree.
template <typename T>
constexpr bool signed_spectra(int P) {
  return !(sizeof(T) == 4 && P == 128);
}

template <typename T, int P_, int E_, bool XB_ = false>
struct Fft2 {
  static constexpr int P = P_;
  static constexpr int E = E_;
  static constexpr int TPR = P / E;
  static constexpr int NT = P * TPR;
  static constexpr int LB = ilog2(TPR);
  // LDS transpose layout: row kx holds y at y + off(kx), rows LD apart, with
  // off(kx) = (BW / TPR) * (kx / E), BW the number of elements per 128-byte
  // bank cycle, LD = P + TPR.  Every transpose access of a wavefront then
  // falls into distinct banks, and each thread's E accesses differ by
  // compile-time constants (one address register per direction).
  static constexpr int BW = 128 / (int)sizeof(T);
  static constexpr int LD = P + TPR;
  static constexpr int PLANE = P * LD + (TPR - 1) * (BW / TPR);  // one real plane of the transpose buffer
  // With XB the real and imaginary planes move together through two buffers.
  static constexpr bool XB = XB_;
  static constexpr int LDS_SCALARS = (XB ? 2 : 1) * PLANE;
  static_assert(TPR >= 1 && TPR <= 8 && (TPR & (TPR - 1)) == 0, "TPR must be 1, 2, 4 or 8");
  static_assert(E * TPR == P, "E * TPR must equal P");
  static_assert(P % BW == 0, "P must be a multiple of the bank width");

  static constexpr bool SIGNED = signed_spectra<T>(P);

  int t, line, q, bq;
  T* lds;          // transpose buffer, LDS_SCALARS scalars
  const T* tw;     // LDS: (cos, sin)(2 pi q k / P) at [q][k], q < TPR, k < E, row stride TWS
  // padded row stride of the twiddle table: the TPR rows start in different banks
  static constexpr int TWS = 2 * E + 2;
  static constexpr int TW_SCALARS = TPR * TWS;

  // logical lane q of physical lane p (an involution, see the header)
  static __host__ __device__ constexpr int lane_label(int p) { return TPR == 8 ? p ^ (3 * (p >> 2)) : p; }

  __device__ __forceinline__ void init(T* lds_buf, const T* twi) {
    t = threadIdx.x;
    line = t / TPR;
    q = lane_label(t % TPR);
    bq = bitrev_rt(q, LB);
    lds = lds_buf;
    tw = twi;
  }
  __device__ __forceinline__ int sx(int n) const { return q + TPR * n; }     // strided index
  __device__ __forceinline__ int bk(int k) const { return k + E * bq; }      // blocked index
  // LDS position of (kx row inside the buffer, y) without the bank offset
  __device__ __forceinline__ int addr(int kxl, int y) const { return kxl * LD + y; }
  // bank offset of a kx row: spreads the TPR row groups kx / E over the banks
  __device__ __forceinline__ int off_of(int kx) const { return (BW / TPR) * (kx / E); }

  // w_P^{q k} multiply, sign SG (-1 forward, +1 inverse), k = 1..E-1
  template <int SG>
  __device__ __forceinline__ void twiddle(T (&zr)[E], T (&zi)[E]) const {
    // The table is constant, so the compiler would keep all E twiddles in
    // registers across the whole kernel; an opaque base index makes it load
    // them where they are used instead.
    int base = q * TWS;
    __asm__ volatile("" : "+v"(base));
#pragma unroll
    for (int k = 1; k < E; ++k) {
      const T* w = tw + base + 2 * k;
      const T c = w[0], s = SG < 0 ? -w[1] : w[1];
      const T r = zr[k] * c - zi[k] * s;
      zi[k] = zr[k] * s + zi[k] * c;
      zr[k] = r;
    }
  }

  // Twiddle of the H = 4 lane stage as (re, im): -w_8^r, r = q mod 4, on the
  // upper lanes (conjugated for the inverse), 1 on the lower ones.
  template <int SG>
  __device__ __forceinline__ void w8(T& wr, T& wi) const {
    const T c = (T)0.70710678118654752440;
    const int r = q & 3;
    const T cr = r == 0 ? (T)1 : (r == 1 ? c : (r == 2 ? (T)0 : -c));
    const T sr = r == 0 ? (T)0 : (r == 2 ? (T)1 : c);
    wr = (q & 4) ? -cr : (T)1;
    wi = (q & 4) ? (SG < 0 ? sr : -sr) : (T)0;
  }

  // Cross-lane DFT of size TPR for every k (forward: decimation in frequency,
  // natural lane order in, bit-reversed out): stage H = TPR/2 .. 1 adds the
  // partner lane q ^ H, then the upper lanes take the twiddle w_{2H}^{q mod H}.
  // A stage is z + s z_partner with s = +1 on lower and -1 on upper lanes:
  // one fused multiply-add whose partner operand is a DPP read (in float32 a
  // single instruction, 4.3 clocks; a separate move took 4.3 and the add 2.7),
  // which leaves the upper lanes with the sign reversed.  The twiddles of the
  // H = 4 stage and the rotation of lane 3 after the H = 2 stage take that
  // sign up; what is left after the last stage is a factor
  //   sigma(q) = (-1)^(number of ones in q mod 4)
  // on the spectrum, which lanes_inv expects and undoes.  Every spectrum the
  // kernels keep carries it: in two dimensions the entry (kx, ky) has the sign
  // sigma(lane of kx) sigma(lane of ky).  Tables and phases multiply through;
  // only a step that mixes k with another frequency has to look (k_grad_pre).
  __device__ __forceinline__ void lanes_fwd(T (&zr)[E], T (&zi)[E]) const {
    if constexpr (TPR == 8) {
      const T sg = (q & 4) ? (T)-1 : (T)1;
      T wr, wi;
      w8<-1>(wr, wi);
      add_lanes<7>(zr, sg);
      add_lanes<7>(zi, sg);
#pragma unroll
      for (int k = 0; k < E; ++k) cmul(zr[k], zi[k], wr, wi, zr[k], zi[k]);
    }
    if constexpr (TPR >= 4) {
      const T sg = (q & 2) ? (T)-1 : (T)1;
      const bool rot = (q & 3) == 3;
      add_lanes<2>(zr, sg);
      add_lanes<2>(zi, sg);
#pragma unroll
      for (int k = 0; k < E; ++k) {
        const T dr = zr[k], di = zi[k];
        zr[k] = rot ? di : dr;       // d (-i) = (d_i, -d_r)
        zi[k] = rot ? -dr : di;
      }
    }
    if constexpr (TPR >= 2) {
      const T sg = (q & 1) ? (T)-1 : (T)1;
      add_lanes<1>(zr, sg);
      add_lanes<1>(zi, sg);
    }
  }
  // exact reverse of lanes_fwd (unnormalized: times TPR)
  __device__ __forceinline__ void lanes_inv(T (&zr)[E], T (&zi)[E]) const {
    if constexpr (TPR >= 2) {
      const T sg = (q & 1) ? (T)1 : (T)-1;
      add_lanes<1>(zr, sg);
      add_lanes<1>(zi, sg);
    }
    if constexpr (TPR >= 4) {
      const T sg = (q & 2) ? (T)1 : (T)-1;
      const bool rot = (q & 3) == 3;
#pragma unroll
      for (int k = 0; k < E; ++k) {
        // z i = (-z_i, z_r) on lane 3
        const T dr = zr[k], di = zi[k];
        zr[k] = rot ? -di : dr;
        zi[k] = rot ? dr : di;
      }
      add_lanes<2>(zr, sg);
      add_lanes<2>(zi, sg);
    }
    if constexpr (TPR == 8) {
      const T sg = (q & 4) ? (T)1 : (T)-1;
      T wr, wi;
      w8<+1>(wr, wi);
#pragma unroll
      for (int k = 0; k < E; ++k) cmul(zr[k], zi[k], wr, wi, zr[k], zi[k]);
      add_lanes<7>(zr, sg);
      add_lanes<7>(zi, sg);
    }
  }

  // twiddle w_8^r, r = 0..3, of the H = 4 lane stage (conjugated for the
  // inverse), as (re, im)
  template <int SG>
  __device__ __forceinline__ void w8_true(int r, T& wr, T& wi) const {
    const T c = (T)0.70710678118654752440;
    wr = r == 0 ? (T)1 : (r == 1 ? c : (r == 2 ? (T)0 : -c));
    const T s = r == 0 ? (T)0 : (r == 2 ? (T)1 : c);
    wi = SG < 0 ? -s : s;
  }

  // The lane stages with the upper lanes' sign in the multiply-add (a move and
  // an FMA per value) and no sign left on the spectrum.
  // Cross-lane DFT of size TPR for every k.  Forward (decimation in
  // frequency, natural lane order in, bit-reversed out):
  //   stage H = TPR/2 .. 1: lower lane z + o, upper lane (o - z) w_{2H}^{q mod H}
  // The H = 2 stage twiddle is w_4 = -i (lanes with q mod 4 = 3), applied as a
  // component swap; the H = 4 stage (TPR = 8) multiplies the upper lanes by
  // w_8^{q mod 4}.
  __device__ __forceinline__ void lanes_fwd_true(T (&zr)[E], T (&zi)[E]) const {
    if constexpr (TPR == 8) {
      const T sg = (q & 4) ? (T)-1 : (T)1;
      T wr, wi;
      w8_true<-1>((q & 4) ? (q & 3) : 0, wr, wi);
#pragma unroll
      for (int k = 0; k < E; ++k) {
        const T orr = xor_lane<7>(zr[k]), oi = xor_lane<7>(zi[k]);
        const T dr = sg * zr[k] + orr, di = sg * zi[k] + oi;
        zr[k] = dr * wr - di * wi;
        zi[k] = dr * wi + di * wr;
      }
    }
    if constexpr (TPR >= 4) {
      const T sg = (q & 2) ? (T)-1 : (T)1;
      const bool rot = (q & 3) == 3;
#pragma unroll
      for (int k = 0; k < E; ++k) {
        const T orr = xor_lane<2>(zr[k]), oi = xor_lane<2>(zi[k]);
        const T dr = sg * zr[k] + orr, di = sg * zi[k] + oi;
        zr[k] = rot ? di : dr;       // (d) * (-i) = (d_i, -d_r)
        zi[k] = rot ? -dr : di;
      }
    }
    if constexpr (TPR >= 2) {
      const T sg = (q & 1) ? (T)-1 : (T)1;
#pragma unroll
      for (int k = 0; k < E; ++k) {
        const T orr = xor_lane<1>(zr[k]), oi = xor_lane<1>(zi[k]);
        zr[k] = sg * zr[k] + orr;
        zi[k] = sg * zi[k] + oi;
      }
    }
  }
  // exact reverse of lanes_fwd_true (unnormalized: times TPR)
  __device__ __forceinline__ void lanes_inv_true(T (&zr)[E], T (&zi)[E]) const {
    if constexpr (TPR >= 2) {
      const T sg = (q & 1) ? (T)-1 : (T)1;
#pragma unroll
      for (int k = 0; k < E; ++k) {
        const T orr = xor_lane<1>(zr[k]), oi = xor_lane<1>(zi[k]);
        zr[k] = sg * zr[k] + orr;
        zi[k] = sg * zi[k] + oi;
      }
    }
    if constexpr (TPR >= 4) {
      const T sg = (q & 2) ? (T)-1 : (T)1;
      const bool rot = (q & 3) == 3;
#pragma unroll
      for (int k = 0; k < E; ++k) {
        // undo the -i of lanes q mod 4 = 3: multiply by +i = (-z_i, z_r)
        const T ar = rot ? -zi[k] : zr[k];
        const T ai = rot ? zr[k] : zi[k];
        const T orr = xor_lane<2>(ar), oi = xor_lane<2>(ai);
        zr[k] = sg * ar + orr;
        zi[k] = sg * ai + oi;
      }
    }
    if constexpr (TPR == 8) {
      const T sg = (q & 4) ? (T)-1 : (T)1;
      T wr, wi;
      w8_true<+1>((q & 4) ? (q & 3) : 0, wr, wi);
#pragma unroll
      for (int k = 0; k < E; ++k) {
        const T ar = zr[k] * wr - zi[k] * wi, ai = zr[k] * wi + zi[k] * wr;
        const T orr = xor_lane<7>(ar), oi = xor_lane<7>(ai);
        zr[k] = sg * ar + orr;
        zi[k] = sg * ai + oi;
      }
    }
  }

  // forward: strided -> blocked, exp(-2 pi i ...)
  __device__ __forceinline__ void fwd_line(T (&zr)[E], T (&zi)[E]) const {
    reg_fft<T, E, -1>(zr, zi);
    if constexpr (TPR > 1) {
      twiddle<-1>(zr, zi);
      if constexpr (SIGNED)
        lanes_fwd(zr, zi);
      else
        lanes_fwd_true(zr, zi);
    }
  }

  // inverse: blocked -> strided, exp(+2 pi i ...), unnormalized
  __device__ __forceinline__ void inv_line(T (&zr)[E], T (&zi)[E]) const {
    if constexpr (TPR > 1) {
      if constexpr (SIGNED)
        lanes_inv(zr, zi);
      else
        lanes_inv_true(zr, zi);
      twiddle<+1>(zr, zi);
    }
    reg_fft<T, E, +1>(zr, zi);
  }

  // T1: row spectra (blocked in kx, line = y) -> column real (strided in y, line = kx)
  // T2: column real -> row spectra, back along the same addresses.
  // A thread writes in T1 where it last read in T2 and the other way round, so
  // a transpose that follows its opposite (OWN) finds the addresses it
  // writes free: one barrier, between the writes and the reads, with two
  // planes, three with one.  Otherwise a leading barrier waits for the reads
  // of the transpose before.
  template <bool OWN>
  __device__ __forceinline__ void t_rows_to_cols(T (&zr)[E], T (&zi)[E]) const {
    auto wr = [&](T* p, const T (&z)[E]) {
#pragma unroll
      for (int k = 0; k < E; ++k) p[addr(bk(k), line) + off_of(bk(k))] = z[k];
    };
    auto rd = [&](const T* p, T (&z)[E]) {
#pragma unroll
      for (int n = 0; n < E; ++n) z[n] = p[addr(line, sx(n)) + off_of(line)];
    };
    move<OWN>(zr, zi, wr, rd);
  }
  template <bool OWN>
  __device__ __forceinline__ void t_cols_to_rows(T (&zr)[E], T (&zi)[E]) const {
    auto wr = [&](T* p, const T (&z)[E]) {
#pragma unroll
      for (int n = 0; n < E; ++n) p[addr(line, sx(n)) + off_of(line)] = z[n];
    };
    auto rd = [&](const T* p, T (&z)[E]) {
#pragma unroll
      for (int k = 0; k < E; ++k) z[k] = p[addr(bk(k), line) + off_of(bk(k))];
    };
    move<OWN>(zr, zi, wr, rd);
  }
  template <bool OWN, typename W, typename R>
  __device__ __forceinline__ void move(T (&zr)[E], T (&zi)[E], W wr, R rd) const {
    if constexpr (!OWN) __syncthreads();
    if constexpr (XB) {
      wr(lds, zr);
      wr(lds + PLANE, zi);
      __syncthreads();
      rd(lds, zr);
      rd(lds + PLANE, zi);
    } else {
      wr(lds, zr);
      __syncthreads();
      rd(lds, zr);
      __syncthreads();
      wr(lds, zi);
      __syncthreads();
      rd(lds, zi);
    }
  }

  // full 2D: row real -> column spectra (OWN: the last transform was an inv2;
  // FREE: the next one may be another fwd2 with OWN, so the transpose ends
  // with a barrier)
  template <bool OWN = false, bool FREE = false>
  __device__ __forceinline__ void fwd2(T (&zr)[E], T (&zi)[E]) const {
    fwd_line(zr, zi);
    t_rows_to_cols<OWN>(zr, zi);
    if constexpr (FREE) __syncthreads();
    fwd_line(zr, zi);
  }
  // full 2D: column spectra -> row real (OWN: the last transform was a fwd2;
  // FREE: the next one may be another inv2 with OWN)
  template <bool OWN = false, bool FREE = false>
  __device__ __forceinline__ void inv2(T (&zr)[E], T (&zi)[E]) const {
    inv_line(zr, zi);
    t_cols_to_rows<OWN>(zr, zi);
    if constexpr (FREE) __syncthreads();
    inv_line(zr, zi);
  }
};

}  // namespace qb
