// Device code of the float32 fringe search (Eq. 5 with the Eq. 4 rate term,
// Sec. 5.1) and the helpers it shares with the other kernels: compile-time
// twiddles, in-register DFTs (dense, and pruned to a compile-time set of
// non-zero inputs), the segment sums of Eq. 3, the SBD pass and the MBD peak.
// Included by frbx_kernels.hip and, for kernels specialised to an IF lattice
// at run time, compiled by hipRTC (which provides the HIP device environment
// itself: no runtime or standard headers then).
#pragma once

#ifndef __HIPCC_RTC__
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "frbx_internal.h"
#endif

namespace frbx {

// ---------------------------------------------------------------- helpers
// A compile-time loop index (value usable in constant expressions).
template <int I>
struct Index {
  static constexpr int value = I;
};

template <int I, int N, typename F>
__device__ __forceinline__ void static_for(F &&f) {
  if constexpr (I < N) {
    f(Index<I>{});
    static_for<I + 1, N>(f);
  }
}

constexpr int ilog2(int n) { return n <= 1 ? 0 : 1 + ilog2(n >> 1); }

constexpr int bitrev(int i, int bits) {
  int r = 0;
  for (int b = 0; b < bits; ++b) r |= ((i >> b) & 1) << (bits - 1 - b);
  return r;
}

// Compile-time sine/cosine of (pi/2) * x, x in [0, 1), by Taylor series in
// double; used only for the fixed twiddles of the in-register DFTs.
constexpr double kHalfPi = 1.57079632679489661923;
constexpr double taylor_sin(double t) {
  double term = t, sum = t;
  for (int i = 1; i < 18; ++i) {
    term *= -t * t / ((2.0 * i) * (2.0 * i + 1.0));
    sum += term;
  }
  return sum;
}
constexpr double taylor_cos(double t) {
  double term = 1.0, sum = 1.0;
  for (int i = 1; i < 18; ++i) {
    term *= -t * t / ((2.0 * i - 1.0) * (2.0 * i));
    sum += term;
  }
  return sum;
}
// exp(-2 pi i k / n) = (c, s): quadrant reduction on the integers first.
constexpr double tw_re(int k, int n) {
  k = ((k % n) + n) % n;
  const int q = (4 * k) / n;
  const double t = kHalfPi * double(4 * k - q * n) / double(n);
  const double c = taylor_cos(t), s = taylor_sin(t);
  return q == 0 ? c : q == 1 ? -s : q == 2 ? -c : s;
}
constexpr double tw_im(int k, int n) {
  k = ((k % n) + n) % n;
  const int q = (4 * k) / n;
  const double t = kHalfPi * double(4 * k - q * n) / double(n);
  const double c = taylor_cos(t), s = taylor_sin(t);
  const double sn = q == 0 ? s : q == 1 ? c : q == 2 ? -s : -c;  // sin(2 pi k / n)
  return -sn;
}

__device__ __forceinline__ float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
  return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

// a * exp(-2 pi i K / N) with the twiddle known at compile time.
template <int K, int N>
__device__ __forceinline__ float2 twmul(float2 a) {
  constexpr int k = ((K % N) + N) % N;
  if constexpr (k == 0) {
    return a;
  } else if constexpr (4 * k == N) {
    return make_float2(a.y, -a.x);
  } else if constexpr (2 * k == N) {
    return make_float2(-a.x, -a.y);
  } else if constexpr (4 * k == 3 * N) {
    return make_float2(-a.y, a.x);
  } else {
    constexpr float c = static_cast<float>(tw_re(k, N));
    constexpr float s = static_cast<float>(tw_im(k, N));
    return make_float2(a.x * c - a.y * s, a.x * s + a.y * c);
  }
}

// In-register forward DFT of NP points, X[k] = sum_i x[i] exp(-2 pi i ik/NP):
// radix-2 decimation in frequency, natural order in and out.
template <int NP>
__device__ __forceinline__ void dft(float2 (&x)[NP]) {
  constexpr int L = ilog2(NP);
  static_for<0, L>([&](auto st) {
    constexpr int span = NP >> (decltype(st)::value + 1);
    static_for<0, NP / 2>([&](auto bi) {
      constexpr int b = decltype(bi)::value;
      constexpr int grp = b / span, pos = b % span;
      constexpr int i0 = grp * 2 * span + pos, i1 = i0 + span;
      const float2 a = x[i0], c = x[i1];
      x[i0] = cadd(a, c);
      x[i1] = twmul<pos * (NP / (2 * span)), NP>(csub(a, c));
    });
  });
  float2 y[NP];
  static_for<0, NP>([&](auto i) {
    constexpr int ii = decltype(i)::value;
    y[bitrev(ii, L)] = x[ii];
  });
  static_for<0, NP>([&](auto i) { x[decltype(i)::value] = y[decltype(i)::value]; });
}

// Inputs of the radix-2 decimation-in-frequency DFT below that can be non-
// zero before stage `stage`, given those of the input (bit i: x[i]): a
// butterfly's two outputs are zero exactly when both its inputs are.
constexpr unsigned dft_stage_mask(int np, unsigned mask, int stage) {
  for (int st = 0; st < stage; ++st) {
    const int span = np >> (st + 1);
    unsigned out = 0u;
    for (int b = 0; b < np / 2; ++b) {
      const int grp = b / span, pos = b % span;
      const int i0 = grp * 2 * span + pos, i1 = i0 + span;
      if (((mask >> i0) | (mask >> i1)) & 1u) out |= (1u << i0) | (1u << i1);
    }
    mask = out;
  }
  return mask;
}

// dft<NP> for an input that is zero outside the compile-time set MASK (bit
// i: x[i] may be non-zero; the others must hold +0): butterflies with two
// zero inputs are skipped and those with one skip the addition.  The
// results equal dft<NP>'s (adding an exact zero changes nothing but, at
// most, the sign of a zero).
template <int NP, unsigned MASK>
__device__ __forceinline__ void dft_masked(float2 (&x)[NP]) {
  constexpr int L = ilog2(NP);
  static_for<0, L>([&](auto st) {
    constexpr int stage = decltype(st)::value;
    constexpr unsigned nz = dft_stage_mask(NP, MASK, stage);
    constexpr int span = NP >> (stage + 1);
    static_for<0, NP / 2>([&](auto bi) {
      constexpr int b = decltype(bi)::value;
      constexpr int grp = b / span, pos = b % span;
      constexpr int i0 = grp * 2 * span + pos, i1 = i0 + span;
      constexpr bool z0 = !((nz >> i0) & 1u), z1 = !((nz >> i1) & 1u);
      constexpr int tk = pos * (NP / (2 * span));
      if constexpr (z0 && z1) {
        // both zero: so are both outputs
      } else if constexpr (z1) {
        x[i1] = twmul<tk, NP>(x[i0]);
      } else if constexpr (z0) {
        // x[i0] holds an exact +0: 0 - c, as in dft<NP>, keeps the product
        // and its rounding the same as the dense transform's (the compiler
        // may not fold it into a negation)
        const float2 c = x[i1];
        x[i1] = twmul<tk, NP>(csub(x[i0], c));
        x[i0] = c;
      } else {
        const float2 a = x[i0], c = x[i1];
        x[i0] = cadd(a, c);
        x[i1] = twmul<tk, NP>(csub(a, c));
      }
    });
  });
  float2 y[NP];
  static_for<0, NP>([&](auto i) {
    constexpr int ii = decltype(i)::value;
    y[bitrev(ii, L)] = x[ii];
  });
  static_for<0, NP>([&](auto i) { x[decltype(i)::value] = y[decltype(i)::value]; });
}

// Make the LDS writes of this wave visible to its other lanes before they
// read, and keep the compiler from moving LDS accesses across the point.
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Size split of an F-point transform into (A in-register points of pass 1)
// x (B lanes of pass 1).
template <int F> struct Split;
template <> struct Split<8> { static constexpr int A = 4, B = 2; };
template <> struct Split<16> { static constexpr int A = 4, B = 4; };
template <> struct Split<32> { static constexpr int A = 8, B = 4; };
template <> struct Split<64> { static constexpr int A = 8, B = 8; };
template <> struct Split<128> { static constexpr int A = 16, B = 8; };
template <> struct Split<256> { static constexpr int A = 16, B = 16; };

// BLK threads search one segment: a work-group of kBlock, or one wave (four
// segments to a work-group).
template <int J, int M, int BLK = kBlock>
struct FringeShape {
  static constexpr int JA = Split<J>::A, JB = Split<J>::B;
  static constexpr int MA = Split<M>::A, MB = Split<M>::B;
  static constexpr int G = MA > MB ? MA : MB;    // lanes per MBD column group
  static constexpr int COLS = BLK / G;           // columns per round
  static constexpr int SG = MA * MB + 16;        // float2 per group scratch
};

// LDS plan (float2 units): X tile [N+1][J+1] (rows of IFs, the last kept
// zero), or [max(N+1, MB)][J+1] in the compact form (rows of lattice
// positions, those without an IF kept zero), a scratch area shared by the
// SBD transpose and the MBD transposes, and the PJ-point SBD twiddle table.
// The host sizes the launch with the larger plan (CL = true), once per
// segment of the work-group.
template <int J, int M, bool CL = true, int BLK = kBlock>
__host__ __device__ inline void fringe_lds_plan(int n_if, int sbd_pad, int &x_off, int &s_off,
                                                int &t_off, int &total) {
  using S = FringeShape<J, M, BLK>;
  const int xs = J + 1;
  const int x_rows = CL && S::MB > n_if + 1 ? S::MB : n_if + 1;
  const int x_sz = x_rows * xs;
  const int t_sz = n_if * S::JA * (S::JB + 1);
  const int m_sz = S::COLS * S::SG;
  const int s_sz = t_sz > m_sz ? t_sz : m_sz;
  x_off = 0;
  s_off = x_sz;
  t_off = x_sz + s_sz;
  total = t_off + sbd_pad * J;
}


// ------------------------------------------------------- shared fringe steps
// Which segment a work-group handles.  Work-groups are dealt to the 8 XCDs
// round-robin; in sweeps over the XCDs each gets a run of kXcdRun consecutive
// ones, so that overlapping segments share an L2.  Which XCD takes which run
// of a sweep varies from sweep to sweep: the windows of a DM trial cost more
// the longer they are, and a trial of about 256 segments would otherwise give
// one XCD the longest of every trial.  Fewer than kXcdSweeps sweeps do not even
// that out and go one by one (1265 segments of 16 IFs x 256 channels: 3.86 ms
// in runs, 3.3 ms one by one).
constexpr int kXcdRun = 32, kXcdSweeps = 16;
// A work-group that takes `per` segments takes consecutive ones (slot w).
__device__ __forceinline__ void block_segment(const FringeArgs &a, bool dump, int &dl, int &seg, int per = 1,
                                              int w = 0) {
  if (dump) {
    dl = a.dump_dl;
    seg = a.dump_seg;
    return;
  }
  const int nb = gridDim.x;
  const int bx = blockIdx.x;
  const int i = bx >> 3;
  const int sweeps = nb / (8 * kXcdRun), sweep = i / kXcdRun;
  const int turn = int(unsigned(sweep) * 0x9E3779B1u >> 29);   // (any spread-out sequence of 0 to 7)
  const int run = sweeps >= kXcdSweeps && sweep < sweeps ? (sweep * 8 + ((bx + turn) & 7)) * kXcdRun + i % kXcdRun : bx;
  const int lb = run * per + w;
  dl = lb / a.seg_total;
  seg = lb - dl * a.seg_total;
}

// Segment sum of Eq. 3 with the Eq. 4 rate rotation about the window centre
// for rate bin r: y[i1] = sum_u ph[r][n1][u] W[k0 + u][n1][JB i1 + i2], with
// the j = 0 point excluded from the fit (Sec. 2.3).
template <int JA, int JB>
__device__ __forceinline__ void segment_sum(float2 (&y)[JA], const float2 *wd, const float2 *rph,
                                            int r, int N, int J, int l, int R, bool act, int n1,
                                            int i2s) {
  static_for<0, JA>([&](auto i) { y[decltype(i)::value] = make_float2(0.f, 0.f); });
  if (!act) return;
  const int NJ = N * J;
  const float2 *src = wd + n1 * J + i2s;
  const float2 *ph = rph + (r * N + n1) * l;
  // (the rate test inside the AP loop: with it outside, the compiler issues
  // the loads of an AP one at a time, each waited for)
  for (int u = 0; u < l; ++u) {
    if (R > 1) {
      const float2 p = ph[u];
      static_for<0, JA>([&](auto i) {
        constexpr int ii = decltype(i)::value;
        const float2 v = src[int64_t(u) * NJ + JB * ii];
        y[ii] = cadd(y[ii], cmul(v, p));
      });
    } else {
      static_for<0, JA>([&](auto i) {
        constexpr int ii = decltype(i)::value;
        y[ii] = cadd(y[ii], src[int64_t(u) * NJ + JB * ii]);
      });
    }
  }
  if (i2s == 0) y[0] = make_float2(0.f, 0.f);
}

// SBD pass 1 of tile c: x[i1] = y[i1] w_{P JA}^{i1 c}; JA-point DFT over i1;
// twiddle w_PJ^{i2 (c + P k1)}; store transposed T[n][k1][i2].
__device__ __forceinline__ float2 load_vis(const void *p, int64_t i, bool f16) {
  if (f16) {
    const _Float16 *h = static_cast<const _Float16 *>(p) + 2 * i;
    return make_float2(float(h[0]), float(h[1]));
  }
  return static_cast<const float2 *>(p)[i];
}

// The same segment sum gathered straight from the input of baseline b at DM
// trial d: W[k][c] = cal[c] V[c][k + dk[d][c]] (zero past the last AP),
// formed and accumulated in the same order as the dedispersed path.
template <int JA, int JB>
__device__ __forceinline__ void segment_sum_direct(float2 (&y)[JA], const FringeArgs &a, int b, int d,
                                                   int64_t k0, const float2 *rph, int r, int N, int J,
                                                   int l, int R, bool act, int n1, int i2s) {
  static_for<0, JA>([&](auto i) { y[decltype(i)::value] = make_float2(0.f, 0.f); });
  if (!act) return;
  const int NJ = N * J;
  const float2 *ph = rph + (r * N + n1) * l;
  static_for<0, JA>([&](auto i) {
    constexpr int ii = decltype(i)::value;
    const int c = n1 * J + JB * ii + i2s;
    const float2 cal = a.cal[int64_t(b) * NJ + c];
    const int64_t row = (int64_t(b) * NJ + c) * a.vis_stride;
    const int64_t f0 = k0 + a.dk[int64_t(d) * NJ + c];
    for (int u = 0; u < l; ++u) {
      const int64_t f = f0 + u;
      const float2 v = f < a.vis_frames ? load_vis(a.vis, row + f, a.vis_f16 != 0) : make_float2(0.f, 0.f);
      const float2 w = cmul(v, cal);
      y[ii] = R > 1 ? cadd(y[ii], cmul(w, ph[u])) : cadd(y[ii], w);
    }
  });
  if (i2s == 0) y[0] = make_float2(0.f, 0.f);
}

template <int JA, int JB>
__device__ __forceinline__ void sbd_pass1(const float2 (&y)[JA], const float2 *pre,
                                          const float2 *TW, float2 *Sc, int c, int P, int PJ,
                                          bool act, int n1, int i2s) {
  if (!act) return;
  float2 x[JA];
  static_for<0, JA>([&](auto i) {
    constexpr int ii = decltype(i)::value;
    x[ii] = cmul(y[ii], pre[c * JA + ii]);
  });
  dft<JA>(x);
  static_for<0, JA>([&](auto k) {
    constexpr int kk = decltype(k)::value;
    const float2 w = TW[(i2s * (c + P * kk)) & (PJ - 1)];
    Sc[(n1 * JA + kk) * (JB + 1) + i2s] = cmul(x[kk], w);
  });
}

// Peak of one MBD column after the last MBD pass: lane k1 holds
// z[k2] = G(s', k1 + MA k2) for SBD bin s' = c + P col.  The key of a cell
// is |G|^2 with its 4 lowest mantissa bits replaced by (15 - k2), so one
// unsigned max keeps the value (to 2^-19 relative) and the lowest MBD bin
// among equal values; the running best keeps the lowest packed index.
template <int M, int MA, int MB, bool DUMP>
__device__ __forceinline__ void mbd_column_peak(const float2 (&z)[MB], int r, int c, int col, int k1,
                                                int P, int PJ, float *dump, float &best_v,
                                                int32_t &best_i) {
  // shifted bins: s = (s' + PJ/2) mod PJ, m = k1 + MA ((k2 + MB/2) mod MB)
  const int sp = c + P * col;
  const int s = (sp + (PJ >> 1)) & (PJ - 1);
  const int32_t base = (r * PJ + s) * M + k1;
  unsigned kmax = 0u;
  static_for<0, MB / 2>([&](auto kk) {
    constexpr int ka = 2 * decltype(kk)::value, kb = ka + 1;
    constexpr int k2a = (ka + MB / 2) & (MB - 1), k2b = (kb + MB / 2) & (MB - 1);
    const float va = z[k2a].x * z[k2a].x + z[k2a].y * z[k2a].y;
    const float vb = z[k2b].x * z[k2b].x + z[k2b].y * z[k2b].y;
    const unsigned ua = (__float_as_uint(va) & 0xFFFFFFF0u) | unsigned(15 - ka);
    const unsigned ub = (__float_as_uint(vb) & 0xFFFFFFF0u) | unsigned(15 - kb);
    kmax = max(kmax, max(ua, ub));
    if constexpr (DUMP) {
      dump[base + MA * ka] = va;
      dump[base + MA * kb] = vb;
    }
  });
  const float cv = __uint_as_float(kmax & 0xFFFFFFF0u);
  const int ck = 15 - int(kmax & 15u);
  const int32_t ci = base + MA * ck;
  if (cv > best_v || (cv == best_v && ci < best_i)) {
    best_v = cv;
    best_i = ci;
  }
}

// Largest |G|^2 of one MBD column into blk, as float bits: |G|^2 >= 0
// orders like its bits, and a cell that is not a number outranks every
// number (its bits are above those of +inf).
template <int MB>
__device__ __forceinline__ void mbd_column_max(const float2 (&z)[MB], unsigned &blk) {
  unsigned m = blk;
  static_for<0, MB / 2>([&](auto kk) {
    constexpr int ka = 2 * decltype(kk)::value, kb = ka + 1;
    const float va = z[ka].x * z[ka].x + z[ka].y * z[ka].y;
    const float vb = z[kb].x * z[kb].x + z[kb].y * z[kb].y;
    m = max(m, max(__float_as_uint(va), __float_as_uint(vb)));
  });
  blk = m;
}

// ---------------------------------------------- candidates of a screened search
// The quads (four SBD bins of a sub-grid) of a segment that its screening
// records leave standing: first the one with the largest screened |G|, then,
// once that one's own |G| is known, every other that could exceed it.
struct Candidates {
  const unsigned char *rec;   // the segment's R records
  int R, units, per_c;        // per_c = J / 16 units per sub-grid
  __device__ __forceinline__ float2 bounds(int r) const {
    return *reinterpret_cast<const float2 *>(rec + int64_t(r) * screen_rec_bytes(units));
  }
  // the four quads of unit u at rate r
  __device__ __forceinline__ unsigned quads(int r, int u) const {
    return reinterpret_cast<const unsigned *>(rec + int64_t(r) * screen_rec_bytes(units) + 8)[u];
  }
  // the quad with the largest screened |G| as (rate * P + sub-grid, quad of
  // the sub-grid); rc = -1 when no record knows one.  Every wave of the
  // work-group finds the same (R and units are at most 64).
  __device__ __forceinline__ void first(int lane, int P, int &rc, int &qd) const {
    float top = -1.0f;
    int r = lane;
    if (lane < R) {
      const float2 ab = bounds(lane);
      if (ab.y < __builtin_inff()) top = ab.x;
    }
    for (int off = 32; off > 0; off >>= 1) {
      const float ot = __shfl_xor(top, off, 64);
      const int orr = __shfl_xor(r, off, 64);
      if (ot > top || (ot == top && orr < r)) {
        top = ot;
        r = orr;
      }
    }
    rc = -1;
    qd = 0;
    if (!(top > 0.0f)) return;
    const unsigned w = lane < units ? quads(r, lane) : 0u;
    int g = -1;
    for (int k = 3; k >= 0; --k)
      if (((w >> (8 * k)) & 255u) == 1u) g = k;
    const unsigned long long is_top = __ballot(g >= 0);
    if (!is_top) return;
    const int u = __ffsll(is_top) - 1;
    rc = r * P + u / per_c;
    qd = 4 * (u - (u / per_c) * per_c) + __shfl(g, u, 64);
  }
  // f(rc, unit of the sub-grid, quads of the unit as 4 bits) for every unit
  // with a quad whose |G| can reach `amp` (< 0: any), units t, t + n, ...
  template <typename F>
  __device__ __forceinline__ void each(int t, int n, int P, float amp, F &&f) const {
    for (int i = t; i < R * units; i += n) {
      const int r = i / units, u = i - (i / units) * units;
      const unsigned w = quads(r, u);
      if (w == 0u) continue;
      const float2 ab = bounds(r);
      const bool known = ab.y < __builtin_inff();
      unsigned bits = 0u;
      for (int k = 0; k < 4; ++k) {
        const unsigned v = (w >> (8 * k)) & 255u;
        if (v != 0u && (!known || ab.x - float(v - 1) * ab.y >= amp * 0.99999f)) bits |= 1u << k;
      }
      if (bits) f(r * P + u / per_c, u - (u / per_c) * per_c, bits);
    }
  }
  // the units of `each` as bit masks cand[rc] of the work-group's threads
  // (cleared before)
  __device__ __forceinline__ void mark(int t, int n, int P, float amp, unsigned *cand) const {
    each(t, n, P, amp, [&](int rc, int u, unsigned) { atomicOr(&cand[rc], 1u << u); });
  }
};

// CL (compact lattice): every IF sits at a lattice position below MB once
// the positions are shifted by a common offset (which changes only the phase
// of G, not |G|).  The first MBD pass then has one non-zero input per lane
// and reduces to the identity: X holds one row per position, and each lane
// of the second pass reads the MB rows of its column directly, twiddles them
// and transforms; the first pass and its LDS transpose drop out.
// LIST: one work-group per entry of a.seg_list instead of per segment of the
// tile (re-evaluation of selected segments).
// ROWS (general form): the rows i1 of the first MBD pass that hold an IF
// (bit i1 for lattice positions MB i1 + i2), 0 for all; the pass then
// reads and transforms only those rows (a kernel specialised to the IF
// lattice when the search starts; the same sums).
// CAND (M = 256): only the candidate units of the segment's screening
// records are transformed, for the segments that find_kernel leaves (every
// unit a candidate, or many).  The result is the full search's: the sub-grid
// with the largest |G|^2 (all bits; then the lowest), its cells keyed; with
// fewer than 8 (rate, sub-grid) pairs the keys alone decide.
// BLK = 64: one wave per segment, for shapes whose SBD pass has at most 64
// lanes' work (N x JB): in a work-group of 256 most threads would wait at its
// barriers, while four independent waves need none.
template <int J, int M, bool DUMP, bool CL, bool LIST, unsigned ROWS, bool CAND, int BLK>
__device__ __forceinline__ void fringe_segment(const FringeArgs &a, int dl, int seg, int lb, int ld, int slot,
                                               float2 *lds_all, float *red_v, int32_t *red_i) {
  using S = FringeShape<J, M, BLK>;
  constexpr int JA = S::JA, JB = S::JB, MA = S::MA, MB = S::MB, G = S::G, COLS = S::COLS;
  constexpr unsigned RMASK = ROWS ? ROWS : (MA >= 32 ? ~0u : (1u << MA) - 1u);
  constexpr int NW = BLK / 64;              // waves per segment

  const int N = a.n_if, R = a.n_rate, P = a.sbd_pad;
  const int PJ = P * J;
  const int NJ = N * J;
  // (a work-group's own thread index is not masked: that cost the M = 128 kernels
  // 14 to 45 registers and with them a wave per SIMD, 6.0 against 4.5 ms for
  // 86272 segments of 9 IFs x 128 channels, 2 rates, 0.28 against 0.25 ms for
  // 2384 of 5 IFs x 32 channels, 4 rates)
  const int t = BLK == kBlock ? int(threadIdx.x) : int(threadIdx.x % BLK);
  auto sync = [&]() {
    if constexpr (BLK == kBlock) __syncthreads();
    else wave_lds_sync();
  };
  int wi = 0;
  while (wi + 1 < a.n_win && a.win_off[wi + 1] <= seg) ++wi;
  const int l = a.win_len[wi];
  const int q = seg - a.win_off[wi];
  const int64_t k0 = a.win_k0[wi] + int64_t(q) * a.win_hop[wi];
  const float2 *wd = LIST ? nullptr : a.w + int64_t(dl) * a.w_dm_stride + k0 * NJ;
  const float2 *rph = a.rate_ph + a.rate_off[wi];

  int x_off, s_off, t_off, total;
  fringe_lds_plan<J, M, CL, BLK>(N, P, x_off, s_off, t_off, total);
  // (the candidate masks, R P words, follow the plan)
  float2 *const lds = lds_all + slot * (total + (CAND ? (R * P + 1) / 2 : 0));
  float2 *X = lds + x_off;
  float2 *Sc = lds + s_off;
  float2 *TW = lds + t_off;
  constexpr int XS = J + 1;

  for (int i = t; i < PJ; i += BLK) TW[i] = a.tw_sbd[i];
  if constexpr (CL) {
    // rows of lattice positions without an IF stay zero
    for (int i = t; i < MB * XS; i += BLK) X[i] = make_float2(0.f, 0.f);
  } else {
    // the zero row read for empty lattice points
    for (int i = t; i < XS; i += BLK) X[N * XS + i] = make_float2(0.f, 0.f);
  }

  // ---- per-lane constants of the MBD transform
  const int grp = t / G, gl = t - grp * G;
  const bool m_p1 = gl < MB;  // pass-1 lane: lattice residue i2 = gl
  const bool m_p2 = gl < MA;  // pass-2 lane: output residue k1 = gl
  constexpr int NT = CL ? MB : MA;
  float2 twm[NT];   // general: w_M^(i2 k1) for k1 < MA; compact: w_M^(i2 k1) for i2 < MB
  int rowoff[CL ? 1 : MA];
  if constexpr (CL) {
    if (m_p2) {
      static_for<0, MB>([&](auto i) {
        constexpr int ii = decltype(i)::value;
        twm[ii] = a.tw_mbd[(gl * ii) & (M - 1)];
      });
    }
  } else if (m_p1) {
    static_for<0, MA>([&](auto k) {
      constexpr int kk = decltype(k)::value;
      twm[kk] = a.tw_mbd[(gl * kk) & (M - 1)];
      if constexpr ((RMASK >> kk) & 1u) rowoff[kk] = a.mbd_row[MB * kk + gl] * XS;
    });
  }
  float2 *Sg = Sc + grp * S::SG;

  // ---- per-lane roles of the SBD transform
  const bool s_p1 = t < N * JB;
  const int n1 = t / JB, i2s = t - (t / JB) * JB;

  float best_v = -1.0f;
  int32_t best_i = 0x7fffffff;
  float2 y[JA];

  auto sums = [&](int r) {
    if constexpr (LIST)
      segment_sum_direct<JA, JB>(y, a, lb, ld, k0, rph, r, N, J, l, R, s_p1, n1, i2s);
    else
      segment_sum<JA, JB>(y, wd, rph, r, N, J, l, R, s_p1, n1, i2s);
  };
  // SBD transform of sub-grid c -> X
  auto sbd = [&](int c) {
    sync();
    sbd_pass1<JA, JB>(y, a.pre_sbd, TW, Sc, c, P, PJ, s_p1, n1, i2s);
    sync();
    // SBD pass 2: JB-point DFT over i2 -> X[n][a = k1 + JA k2], the SBD
    // bin s' = c + P a of the standard (unshifted) transform.
    for (int v = t; v < N * JA; v += BLK) {
      const int n2 = v / JA, k1 = v - (v / JA) * JA;
      float2 z[JB];
      static_for<0, JB>([&](auto i) {
        constexpr int ii = decltype(i)::value;
        z[ii] = Sc[(n2 * JA + k1) * (JB + 1) + ii];
      });
      dft<JB>(z);
      const int xrow = CL ? a.mbd_pos[n2] : n2;
      static_for<0, JB>([&](auto k) {
        constexpr int kk = decltype(k)::value;
        X[xrow * XS + k1 + JA * kk] = z[kk];
      });
    }
    sync();
  };
  // MBD transform of every SBD column of sub-grid c (rate r); FIND: the
  // cells' keys and the running (value, packed index) of the lane, else
  // only the largest |G|^2 (float bits) into blk
  // (FIND 2: keys and maximum, and only columns [from, to))
  auto mbd = [&](int r, int c, auto find_tag, unsigned &blk, int from = 0, int to = J) {
    constexpr int FIND = decltype(find_tag)::value;
    auto column = [&](const float2 (&z)[MB], int col) {
      if constexpr (FIND != 0)
        mbd_column_peak<M, MA, MB, DUMP>(z, r, c, col, gl, P, PJ, a.dump, best_v, best_i);
      if constexpr (FIND != 1)
        mbd_column_max<MB>(z, blk);
    };
    const int a_lo = FIND == 2 ? from : 0, a_hi = FIND == 2 ? to : J;
    if constexpr (CL) {
      // compact lattice: z[i2] = X(position i2) w_M^(i2 k1), MB-point DFT
      for (int a0 = a_lo; a0 < a_hi; a0 += COLS) {
        const int col = a0 + grp;
        if (col < J && m_p2) {
          float2 z[MB];
          z[0] = X[col];
          static_for<1, MB>([&](auto i) {
            constexpr int ii = decltype(i)::value;
            z[ii] = cmul(X[ii * XS + col], twm[ii]);
          });
          dft<MB>(z);
          column(z, col);
        }
      }
    } else {
      // MBD over the IF lattice, one column a of this SBD tile per group.
      // Unrolled by 4: the columns' LDS offsets become immediates.
#pragma unroll (CAND ? 1 : 4)
      for (int a0 = a_lo; a0 < a_hi; a0 += COLS) {
        const int col = a0 + grp;
        if (col < J) {
          if (m_p1) {
            float2 x[MA];
            static_for<0, MA>([&](auto i) {
              constexpr int ii = decltype(i)::value;
              if constexpr ((RMASK >> ii) & 1u) x[ii] = X[rowoff[ii] + col];
              else x[ii] = make_float2(0.f, 0.f);
            });
            dft_masked<MA, RMASK>(x);
            static_for<0, MA>([&](auto k) {
              constexpr int kk = decltype(k)::value;
              // w_M^(i2 k1) is 1 at k1 = 0
              Sg[kk * MB + (gl ^ (kk & (MB - 1)))] = kk == 0 ? x[0] : cmul(x[kk], twm[kk]);
            });
          }
          wave_lds_sync();
          if (m_p2) {
            float2 z[MB];
            static_for<0, MB>([&](auto i) {
              constexpr int ii = decltype(i)::value;
              z[ii] = Sg[gl * MB + (ii ^ (gl & (MB - 1)))];
            });
            dft<MB>(z);
            column(z, col);
          }
          wave_lds_sync();
        }
      }
    }
  };

  // ---- the search.  DUMP and LIST key every cell as they go, and so does
  // every search with fewer than 8 (rate, sub-grid) pairs, where searching
  // one of them again would cost more than keying saves.  Otherwise the
  // scan keeps per lane only the largest |G|^2 (float bits) over each
  // (rate, sub-grid) and the first (rate, sub-grid) holding the lane's
  // maximum; the one holding the block's maximum is searched again with
  // keys to find its cell.  A cell that is not a number then makes the
  // segment's power NaN (index -1).
  constexpr bool SCAN = !DUMP && !LIST;
  const bool scan = SCAN && R * P >= 8;
  if constexpr (CAND) {
    static_assert(M == 256 && 16 % COLS == 0, "a unit is 16 columns");
    unsigned *cand = reinterpret_cast<unsigned *>(lds + total);   // [R P] after the plan
    const Candidates cs{a.screen + (int64_t(dl) * a.seg_total + seg) * R * screen_rec_bytes(a.screen_units), R,
                        a.screen_units, J / 16};
    for (int i = t; i < R * P; i += BLK) cand[i] = 0u;
    unsigned top = 0u;           // largest |G|^2 (bits) so far and its (rate, sub-grid)
    int top_rc = 0x7fffffff, cur_r = -1;
    float run_v = -1.0f;         // the lane's keyed peak over what counts so far
    int32_t run_i = 0x7fffffff;
    int rc0, sb0;
    cs.first(t & 63, P, rc0, sb0);
    sb0 >>= 2;   // the quad's unit
    for (int it = rc0 >= 0 ? -1 : 0; it < R * P; ++it) {
      if (it == 0) {   // what the first unit leaves
        sync();   // cand is cleared
        cs.mark(t, BLK, P, rc0 >= 0 ? sqrtf(__uint_as_float(top)) : -1.0f, cand);
        sync();
      }
      const int rc = it < 0 ? rc0 : it;
      // (the first unit's sub-grid: again with the first only if others are left)
      const unsigned mask = it < 0 ? 1u << sb0 : cand[rc] == 1u << sb0 && rc == rc0 ? 0u : cand[rc];
      if (!mask) continue;
      const int r = rc / P, c = rc - (rc / P) * P;
      if (r != cur_r) {
        sums(r);
        cur_r = r;
      }
      sbd(c);
      unsigned blk = 0u;
      best_v = -1.0f;
      best_i = 0x7fffffff;
      for (unsigned m = mask; m; m &= m - 1) {
        const int a0 = 16 * (__ffs(int(m)) - 1);
        mbd(r, c, Index<2>{}, blk, a0, a0 + 16);
      }
      for (int off = 32; off > 0; off >>= 1) blk = max(blk, unsigned(__shfl_xor(int(blk), off, 64)));
      if ((t & 63) == 0) red_v[t >> 6] = __uint_as_float(blk);
      sync();
      for (int w = 0; w < NW; ++w) blk = max(blk, __float_as_uint(red_v[w]));
      // (the next sbd's first barrier ends the reads of red_v)
      const bool better = blk > top || (blk == top && rc < top_rc);
      if (scan && better && rc != top_rc) {
        run_v = best_v;
        run_i = best_i;
      } else if (!scan || rc == top_rc) {
        if (best_v > run_v || (best_v == run_v && best_i < run_i)) {
          run_v = best_v;
          run_i = best_i;
        }
      }
      if (better) {
        top = blk;
        top_rc = rc;
      }
    }
    if (scan && top > 0x7F800000u) {   // a cell that is not a number (non-finite input)
      if (t == 0) {
        const int64_t o = int64_t(dl) * a.seg_total + seg;
        a.power[o] = __builtin_nanf("");
        a.pidx[o] = -1;
      }
      return;
    }
    best_v = run_v;
    best_i = run_i;
    sync();   // the reads of red_v are done
  } else {
    unsigned scan_v = 0u;
    int scan_rc = 0;
    for (int r = 0; r < R; ++r) {
      sums(r);
      for (int c = 0; c < P; ++c) {
        sbd(c);
        unsigned blk = 0u;
        if (!scan) {
          mbd(r, c, Index<1>{}, blk);
        } else {
          mbd(r, c, Index<0>{}, blk);
          if (blk > scan_v) {
            scan_v = blk;
            scan_rc = r * P + c;
          }
        }
      }
    }
    if (scan) {
      // block maximum and its (rate, sub-grid): larger value, then lower
      // (rate, sub-grid)
      for (int off = 32; off > 0; off >>= 1) {
        const unsigned ov = __shfl_xor(scan_v, off, 64);
        const int orc = __shfl_xor(scan_rc, off, 64);
        if (ov > scan_v || (ov == scan_v && orc < scan_rc)) {
          scan_v = ov;
          scan_rc = orc;
        }
      }
      if ((t & 63) == 0) {
        red_v[t >> 6] = __uint_as_float(scan_v);
        red_i[t >> 6] = scan_rc;
      }
      sync();
      unsigned vmax = __float_as_uint(red_v[0]);
      int rc = red_i[0];
      for (int w = 1; w < NW; ++w) {
        const unsigned v = __float_as_uint(red_v[w]);
        if (v > vmax || (v == vmax && red_i[w] < rc)) {
          vmax = v;
          rc = red_i[w];
        }
      }
      if (vmax > 0x7F800000u) {   // a cell that is not a number (non-finite input)
        if (t == 0) {
          const int64_t o = int64_t(dl) * a.seg_total + seg;
          a.power[o] = __builtin_nanf("");
          a.pidx[o] = -1;
        }
        return;
      }
      const int r = rc / P, c = rc - (rc / P) * P;
      sums(r);
      sbd(c);   // its first barrier also ends the reads of red_* above
      unsigned unused = 0u;
      mbd(r, c, Index<1>{}, unused);
    }
  }

  // ---- block reduction: larger |G|^2 wins, ties -> lower packed index
  for (int off = 32; off > 0; off >>= 1) {
    const float ov = __shfl_xor(best_v, off, 64);
    const int32_t oi = __shfl_xor(best_i, off, 64);
    if (ov > best_v || (ov == best_v && oi < best_i)) {
      best_v = ov;
      best_i = oi;
    }
  }
  if ((t & 63) == 0) {
    red_v[t >> 6] = best_v;
    red_i[t >> 6] = best_i;
  }
  sync();
  if (t == 0 && !DUMP) {
    float bv = red_v[0];
    int32_t bi = red_i[0];
    for (int w = 1; w < NW; ++w) {
      if (red_v[w] > bv || (red_v[w] == bv && red_i[w] < bi)) {
        bv = red_v[w];
        bi = red_i[w];
      }
    }
    const int64_t o = int64_t(dl) * a.seg_total + seg;
    a.power[o] = bv >= 0.0f ? sqrtf(bv) : __builtin_nanf("");
    a.pidx[o] = bv >= 0.0f ? bi : -1;
  }
}

// One work-group per segment of the tile (BLK = 64: per four segments); LIST:
// per entry of a.seg_list; CAND: over the segments of a.left_list.
template <int J, int M, bool DUMP, bool CL, bool LIST = false, unsigned ROWS = 0u, bool CAND = false, int BLK = kBlock>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(J <= 64 && !DUMP && !LIST ? 3 : 1)))
void fringe_kernel(FringeArgs a) {
  static_assert(BLK == kBlock || (BLK == 64 && !DUMP && !LIST && !CAND), "one wave per segment: plain searches");
  constexpr int PER = kBlock / BLK;         // segments per work-group
  extern __shared__ float2 lds_all[];
  __shared__ float red_v[kBlock / 64];
  __shared__ int32_t red_i[kBlock / 64];
  const int slot = PER > 1 ? __builtin_amdgcn_readfirstlane(int(threadIdx.x) / BLK) : 0;
  if constexpr (CAND) {
    const int n = a.left_n ? *a.left_n : a.n_dt * a.seg_total;
    for (int64_t i = blockIdx.x; i < n; i += gridDim.x) {
      const int at = a.left_n ? a.left_list[i] : int(i);
      fringe_segment<J, M, DUMP, CL, LIST, ROWS, CAND, BLK>(a, at / a.seg_total, at % a.seg_total, 0, 0, slot, lds_all,
                                                            red_v, red_i);
      __syncthreads();
    }
  } else {
    int dl, seg, lb = 0, ld = 0;
    if constexpr (LIST) {
      lb = a.seg_list[3 * blockIdx.x];
      ld = a.seg_list[3 * blockIdx.x + 1];
      seg = a.seg_list[3 * blockIdx.x + 2];
      dl = lb * a.n_dm + ld;   // cube row
    } else {
      // spread runs of consecutive segments over the 8 XCDs so that
      // overlapping segments share an L2
      block_segment(a, DUMP, dl, seg, PER, slot);
      if (PER > 1 && dl >= a.n_dt) return;   // (no barriers follow)
    }
    fringe_segment<J, M, DUMP, CL, LIST, ROWS, CAND, BLK>(a, dl, seg, lb, ld, slot, lds_all, red_v + slot * (BLK / 64),
                                                          red_i + slot * (BLK / 64));
  }
}

// ---------------------------------------------------- candidates of a segment
// The screened float32 search (M = 256) of a segment by one wave: each
// candidate quad by itself, in fringe_kernel's arithmetic.  Of the SBD
// transform's J bins a quad needs four, which share one output of its second
// pass: the first pass runs for every IF and stores its four outputs, the
// second keeps one bin of each, and the MBD pass takes the four columns at
// once, 16 lanes each.  A work-group per segment spent most of its time at the
// barriers of two or three such candidates, of 16 bins each; a wave needs none,
// and twelve segments are in flight on a CU.  What bounds it now is the latency
// of a wave's own chain (records, spectra, two LDS transposes).  41184 segments
// of 32 IFs x 64 channels, 8 rates: 1.76 -> 0.97 ms; 163840 of 8 IFs x 32
// channels, one rate: 1.35 -> 0.69 ms.
// Segments about which the records know nothing, or with so many candidates
// that the whole transform is cheaper, go to a.left_list.
constexpr int kFindScratch(int n_if, int jb, bool compact) {
  const int t = n_if * 4 * (jb + 1), m = compact ? 0 : 4 * (256 + 16);
  return t > m ? t : m;
}
constexpr int kFindStride(int n_if, int jb, bool compact, int masks) {   // float2 per wave
  return kFindScratch(n_if, jb, compact) + (compact ? 16 : n_if + 1) * 5 + masks;
}

// The cells keep fringe_kernel's last bits: the values of a transform are
// formed before one is chosen (left to itself the compiler moves additions
// into the branches), and the twiddles of the first JA / 4 outputs add their
// products in the order in which it adds them there.  Nothing but the compiler
// fixes that order: tests/test_gpu_screen_bits.py fails where another one
// chooses differently.
template <int NP>
__device__ __forceinline__ void formed(float2 (&x)[NP]) {
#pragma unroll
  for (int i = 0; i < NP; ++i) asm volatile("" : "+v"(x[i].x), "+v"(x[i].y));
}

template <int J, bool CL, unsigned ROWS = 0u>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(3)))
void find_kernel(FringeArgs a) {
  constexpr int M = 256, MA = 16, MB = 16, G = 16;
  constexpr int JA = Split<J>::A, JB = Split<J>::B;
  constexpr unsigned RMASK = ROWS ? ROWS : 0xFFFFu;
  extern __shared__ float2 lds_all[];
  const int N = a.n_if, R = a.n_rate, P = a.sbd_pad, PJ = P * J, NJ = N * J;
  const int t = threadIdx.x & 63, slot = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
  int dl, seg;
  block_segment(a, false, dl, seg, kBlock / 64, slot);
  if (dl >= a.n_dt) return;
  const int64_t at = int64_t(dl) * a.seg_total + seg;
  float2 *const Sc = lds_all + slot * kFindStride(N, JB, CL, R * P);
  float2 *const X = Sc + kFindScratch(N, JB, CL);   // [row][5], columns 0-3
  unsigned long long *const quads = reinterpret_cast<unsigned long long *>(X + (CL ? 16 : N + 1) * 5);   // [R P]

  // ---- candidates: leave the segment to fringe_kernel if nothing is known
  const Candidates cs{a.screen + at * R * screen_rec_bytes(a.screen_units), R, a.screen_units, J / 16};
  int rc0, qd0;
  cs.first(t, P, rc0, qd0);
  const bool unknown = __any(t < R && !(cs.bounds(t < R ? t : 0).y < __builtin_inff()));
  auto leave = [&]() {
    if (t == 0) a.left_list[atomicAdd(a.left_n, 1)] = int(at);
  };
  if (rc0 < 0 || unknown) {
    leave();
    return;
  }
  int wi = 0;
  while (wi + 1 < a.n_win && a.win_off[wi + 1] <= seg) ++wi;
  const int l = a.win_len[wi];
  const int64_t k0 = a.win_k0[wi] + int64_t(seg - a.win_off[wi]) * a.win_hop[wi];
  const float2 *wd = a.w + int64_t(dl) * a.w_dm_stride + k0 * NJ;
  const float2 *rph = a.rate_ph + a.rate_off[wi];

  for (int i = t; i < R * P; i += 64) quads[i] = 0ull;
  for (int i = t; i < (CL ? 16 : N + 1) * 5; i += 64) X[i] = make_float2(0.f, 0.f);   // rows without an IF stay zero
  const int grp = t / G, gl = t - grp * G;
  float2 twm[16];
  int rowoff[CL ? 1 : MA];
  if constexpr (CL) {
    static_for<0, MB>([&](auto i) { twm[decltype(i)::value] = a.tw_mbd[(gl * decltype(i)::value) & (M - 1)]; });
  } else {
    static_for<0, MA>([&](auto k) {
      constexpr int kk = decltype(k)::value;
      twm[kk] = a.tw_mbd[(gl * kk) & (M - 1)];
      if constexpr ((RMASK >> kk) & 1u) rowoff[kk] = a.mbd_row[MB * kk + gl] * 5;
    });
  }
  float2 *const Sg = Sc + grp * (MA * MB + 16);

  const bool scan = R * P >= 8;   // (as in fringe_kernel)
  unsigned top = 0u;              // largest |G|^2 (bits) so far and its (rate, sub-grid)
  int top_rc = 0x7fffffff;
  float run_v = -1.0f, best_v;    // the lane's keyed peak over what counts so far, and of this sub-grid
  int32_t run_i = 0x7fffffff, best_i;

  for (int it = -1; it < R * P; ++it) {
    if (it == 0) {   // what the first quad leaves
      wave_lds_sync();
      int n_q = 0;
      cs.each(t, 64, P, sqrtf(__uint_as_float(top)), [&](int rc, int u, unsigned bits) {
        atomicOr(&quads[rc], (unsigned long long)bits << (4 * u));
        n_q += __popc(bits);
      });
      for (int off = 32; off > 0; off >>= 1) n_q += __shfl_xor(n_q, off, 64);
      const int all = R * P * (J / 4);
      if (n_q > max(all / 6, min(all / 2, 16))) {
        leave();
        return;
      }
      wave_lds_sync();
    }
    const int rc = it < 0 ? rc0 : it;
    // (the first quad's sub-grid: again with the first only if others are left)
    unsigned long long mask = it < 0 ? 1ull << qd0 : quads[rc];
    if (it >= 0 && rc == rc0 && mask == 1ull << qd0) mask = 0ull;
    mask = (unsigned long long)unsigned(__builtin_amdgcn_readfirstlane(int(mask >> 32))) << 32 |
           unsigned(__builtin_amdgcn_readfirstlane(int(mask)));
    if (!mask) continue;
    const int r = rc / P, c = rc - (rc / P) * P;
    unsigned blk = 0u;
    best_v = -1.0f;
    best_i = 0x7fffffff;
    for (; mask; mask &= mask - 1) {
      const int qd = __ffsll(mask) - 1, a0 = 4 * qd;
      const int kb = a0 & (JA - 1), k2 = a0 / JA;   // bins a0 .. a0 + 3 = kb .. kb + 3 of the first pass, k2 of the second
      wave_lds_sync();
      for (int v = t; v < N * JB; v += 64) {
        const int n1 = v / JB, i2 = v - (v / JB) * JB;
        float2 x[JA];
        segment_sum<JA, JB>(x, wd, rph, r, N, J, l, R, true, n1, i2);
        static_for<0, JA>([&](auto i) {
          constexpr int ii = decltype(i)::value;
          x[ii] = cmul(x[ii], a.pre_sbd[c * JA + ii]);
        });
        dft<JA>(x);
        formed(x);
        static_for<0, JA / 4>([&](auto b) {
          constexpr int k0b = 4 * decltype(b)::value;
          if (kb == k0b) {
            static_for<0, 4>([&](auto i) {
              constexpr int kk = k0b + decltype(i)::value;
              const float2 w = a.tw_sbd[(i2 * (c + P * kk)) & (PJ - 1)];
              const float2 y = cmul(x[kk], w);
              Sc[(n1 * 4 + decltype(i)::value) * (JB + 1) + i2] =
                  kk < JA / 4 ? make_float2(y.x, fmaf(x[kk].x, w.y, x[kk].y * w.x)) : y;
            });
          }
        });
      }
      wave_lds_sync();
      for (int v = t; v < N * 4; v += 64) {
        const int n2 = v >> 2, i = v & 3;
        float2 z[JB];
        static_for<0, JB>([&](auto q) { z[decltype(q)::value] = Sc[(n2 * 4 + i) * (JB + 1) + decltype(q)::value]; });
        dft<JB>(z);
        formed(z);
        const int xrow = CL ? a.mbd_pos[n2] : n2;
        static_for<0, JB>([&](auto q) {
          if (k2 == decltype(q)::value) X[xrow * 5 + i] = z[decltype(q)::value];
        });
      }
      wave_lds_sync();
      float2 z[MB];
      if constexpr (CL) {
        z[0] = X[grp];
        static_for<1, MB>([&](auto i) {
          constexpr int ii = decltype(i)::value;
          z[ii] = cmul(X[ii * 5 + grp], twm[ii]);
        });
      } else {
        float2 x[MA];
        static_for<0, MA>([&](auto i) {
          constexpr int ii = decltype(i)::value;
          if constexpr ((RMASK >> ii) & 1u) x[ii] = X[rowoff[ii] + grp];
          else x[ii] = make_float2(0.f, 0.f);
        });
        dft_masked<MA, RMASK>(x);
        static_for<0, MA>([&](auto k) {
          constexpr int kk = decltype(k)::value;
          // w_M^(i2 k1) is 1 at k1 = 0
          Sg[kk * MB + (gl ^ (kk & (MB - 1)))] = kk == 0 ? x[0] : cmul(x[kk], twm[kk]);
        });
        wave_lds_sync();
        static_for<0, MB>([&](auto i) {
          constexpr int ii = decltype(i)::value;
          z[ii] = Sg[gl * MB + (ii ^ (gl & (MB - 1)))];
        });
      }
      dft<MB>(z);
      mbd_column_peak<M, MA, MB, false>(z, r, c, a0 + grp, gl, P, PJ, nullptr, best_v, best_i);
      mbd_column_max<MB>(z, blk);
    }
    for (int off = 32; off > 0; off >>= 1) blk = max(blk, unsigned(__shfl_xor(int(blk), off, 64)));
    const bool better = blk > top || (blk == top && rc < top_rc);
    if (scan && better && rc != top_rc) {
      run_v = best_v;
      run_i = best_i;
    } else if (!scan || rc == top_rc) {
      if (best_v > run_v || (best_v == run_v && best_i < run_i)) {
        run_v = best_v;
        run_i = best_i;
      }
    }
    if (better) {
      top = blk;
      top_rc = rc;
    }
  }
  for (int off = 32; off > 0; off >>= 1) {
    const float ov = __shfl_xor(run_v, off, 64);
    const int32_t oi = __shfl_xor(run_i, off, 64);
    if (ov > run_v || (ov == run_v && oi < run_i)) {
      run_v = ov;
      run_i = oi;
    }
  }
  if (t == 0) {
    a.power[at] = run_v >= 0.0f ? sqrtf(run_v) : __builtin_nanf("");
    a.pidx[at] = run_v >= 0.0f ? run_i : -1;
  }
}

}  // namespace frbx
