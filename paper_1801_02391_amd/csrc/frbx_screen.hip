// Screening pass of the fringe search (Eq. 5 with the Eq. 4 rate term,
// Sec. 5.1) on the gfx950 matrix cores.
//
// The search keeps one number per segment, the largest |G| over (rate, SBD,
// MBD), so all but a few cells are needed only to know that they are smaller.
// screen_kernel evaluates every cell in float16 (float32 accumulation) and
// reports, per segment and rate, the units (16 SBD bins of one sub-grid x
// all MBD bins) whose largest |G| lies within twice a rigorous error bound
// of the rate's largest; the search's own kernel then evaluates those units,
// in its own arithmetic, and nothing else.  Since the bound covers every
// rounding of this pass, the unit that holds the search's maximum is always
// among them and the search's result is what it is without this pass, bit
// for bit.
//
// Both transforms are real-embedded complex GEMMs chained in registers:
//   SBD  X[n][s] = sum_j y[n][j] w_PJ^(j s): A = the segment sums (rows n, K =
//        (j, re/im)), B = the constant DFT matrix of 16 SBD bins;
//   MBD  G[s][m] = sum_n X[n][s] w_M^(q_n m): A = X (rows s, K = (n, re/im)),
//        B = the constant lattice matrix of 16 MBD bins.
// The accumulator of v_mfma_f32_16x16x32_f16 holds, per lane, one column
// (s) and four rows (n); rounded to float16 these are exactly a lane's K
// elements of the next product's A operand (row s), so X never leaves the
// registers.  With A = [re, im] against B = [cos, sin] the product is the
// real part, and with A' = [im, -re] against the same B the imaginary part:
// one constant matrix serves both.
//
// One wave takes one (segment, rate): it forms the segment sums in registers
// in the A layout, and streams both constant matrices from LDS, where one
// work-group of eight waves per CU keeps them for the whole launch; waves
// never wait for each other.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "frbx_fringe.h"
#include "frbx_internal.h"

namespace frbx {
namespace {

typedef _Float16 h8_t __attribute__((ext_vector_type(8)));
typedef _Float16 h2_t __attribute__((ext_vector_type(2)));
typedef float f4_t __attribute__((ext_vector_type(4)));
typedef unsigned u4_t __attribute__((ext_vector_type(4)));

constexpr int kScreenBlock = 64 * kScreenWaves;

// The A operands of the real and the imaginary part from four complex
// values: [re, im] and [im, -re].
__device__ __forceinline__ void embed(const float (&re)[4], const float (&im)[4], h8_t &a, h8_t &b) {
  const h2_t r0 = {_Float16(re[0]), _Float16(re[1])}, r1 = {_Float16(re[2]), _Float16(re[3])};
  const h2_t i0 = {_Float16(im[0]), _Float16(im[1])}, i1 = {_Float16(im[2]), _Float16(im[3])};
  const u4_t x = {__builtin_bit_cast(unsigned, r0), __builtin_bit_cast(unsigned, r1),
                  __builtin_bit_cast(unsigned, i0), __builtin_bit_cast(unsigned, i1)};
  const u4_t y = {x[2], x[3], x[0] ^ 0x80008000u, x[1] ^ 0x80008000u};
  a = __builtin_bit_cast(h8_t, x);
  b = __builtin_bit_cast(h8_t, y);
}

// Largest value of the wave, in every lane (v >= 0).
__device__ __forceinline__ float wave_max(float v) {
  auto step = [&](auto ctrl) {
    constexpr int c = decltype(ctrl)::value;
    v = fmaxf(v, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), c, 0xf, 0xf, true)));
  };
  step(Index<0xb1>{});    // quad_perm 1 0 3 2
  step(Index<0x4e>{});    // quad_perm 2 3 0 1
  step(Index<0x141>{});   // row_half_mirror
  step(Index<0x140>{});   // row_mirror
  step(Index<0x142>{});   // row_bcast15
  step(Index<0x143>{});   // row_bcast31
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}

// HALF: the MBD product on half of its columns.  Rows n hold the IFs of even
// lattice position in chunk 0 and of odd position in chunk 1; with a and b
// their sums for bin m < M / 2, G(m) = a + b and G(m + M/2) = a - b, and only
// the larger counts: max |a +- b|^2 = |a|^2 + |b|^2 + 2 |Re a conj(b)|.
// The SBD product does the same over even and odd channels: with e and o
// their sums for bin s' < PJ / 2, X(s') = e + o, X(s' + PJ/2) = e - o.
template <int J, int NK, bool HALF>
__global__ __launch_bounds__(kScreenBlock) __attribute__((amdgpu_waves_per_eu(2)))
void screen_kernel(ScreenArgs a) {
  constexpr int KP = J / 32;               // pairs of SBD K chunks (16 even + 16 odd channels)
  constexpr int NSB = J / 16, NH = NSB / 2;
  constexpr int MT = HALF ? 8 : 16;        // MBD column tiles
  constexpr int UP = 2;                    // unit pairs per pass over the MBD matrix
  extern __shared__ h8_t lds_h[];
  h8_t *const Fm = lds_h;                  // [MT][NK][64]
  h8_t *const Fs = lds_h + MT * NK * 64;   // [units / 2][2 KP][64]
  const int N = a.n_if, R = a.n_rate, NJ = N * J, units = a.units;
  {
    const h8_t *gm = static_cast<const h8_t *>(a.f_mbd), *gs = static_cast<const h8_t *>(a.f_sbd);
    for (int i = threadIdx.x; i < MT * NK * 64; i += kScreenBlock) Fm[i] = gm[i];
    for (int i = threadIdx.x; i < units * KP * 64; i += kScreenBlock) Fs[i] = gs[i];
  }
  __syncthreads();
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, row = lane & 15, g = lane >> 4;
  // the IF of this lane's rows (absent rows read the first IF's data and are cleared)
  int rif[NK];
  static_for<0, NK>([&](auto i) { rif[decltype(i)::value] = a.row_if[16 * decltype(i)::value + row]; });
  // Tasks (segment, rate), rate fastest.  Work-groups are dealt to the 8
  // XCDs round-robin: XCD x takes a contiguous eighth of the tasks, so that
  // the waves in flight on it read the same few segments from its L2.
  const int nb = gridDim.x;
  const bool split = (nb & 7) == 0;
  const int xcd = split ? blockIdx.x & 7 : 0, n_x = split ? 8 : 1;
  const int slot = split ? blockIdx.x >> 3 : blockIdx.x;
  const int stride = (nb / n_x) * kScreenWaves;
  const int lo = int(int64_t(a.n_task) * xcd / n_x), hi = int(int64_t(a.n_task) * (xcd + 1) / n_x);

  for (int task = lo + slot * kScreenWaves + wave; task < hi; task += stride) {
    const int sg = task / R, r = task - sg * R;
    const int dl = sg / a.seg_total, seg = sg - dl * a.seg_total;
    int wi = 0;
    while (wi + 1 < a.n_win && a.win_off[wi + 1] <= seg) ++wi;
    const int l = a.win_len[wi];
    const int64_t k0 = a.win_k0[wi] + int64_t(seg - a.win_off[wi]) * a.win_hop[wi];
    const float2 *wd = a.w + int64_t(dl) * a.w_dm_stride + k0 * NJ;
    const float2 *ph = a.rate_ph + a.rate_off[wi] + int64_t(r) * N * l;

    // ---- segment sums (Eq. 3 with the Eq. 4 rotation): lane (row, g) holds
    // row 16 nt + row, channels 32 kp + 8 h + 2 g + {0, 1}, h < 4:
    // y[nt][kp][4 h + {0, 1}] even, {2, 3} odd channel
    float y[NK][KP][16];
    static_for<0, NK * KP * 16>([&](auto i) {
      constexpr int k = decltype(i)::value;
      y[k / (KP * 16)][(k / 16) % KP][k % 16] = 0.f;
    });
    int off[NK], pho[NK];
    static_for<0, NK>([&](auto i) {
      constexpr int nt = decltype(i)::value;
      const int n = max(rif[nt], 0);
      off[nt] = n * J + 2 * g;
      pho[nt] = n * l;
    });
    for (int u = 0; u < l; ++u) {
      const float2 *src = wd + int64_t(u) * NJ;
      float4 v[NK][KP][4];
      float2 p[NK];
      static_for<0, NK>([&](auto i) {
        constexpr int nt = decltype(i)::value;
        p[nt] = ph[pho[nt] + u];
        static_for<0, KP * 4>([&](auto kk) {
          constexpr int k = decltype(kk)::value;
          v[nt][k / 4][k % 4] = *reinterpret_cast<const float4 *>(src + off[nt] + 8 * k);
        });
      });
      static_for<0, NK>([&](auto i) {
        constexpr int nt = decltype(i)::value;
        static_for<0, KP * 4>([&](auto kk) {
          constexpr int k = decltype(kk)::value;
          const float4 x = v[nt][k / 4][k % 4];
          float *o = &y[nt][k / 4][4 * (k % 4)];
          o[0] = fmaf(x.x, p[nt].x, fmaf(-x.y, p[nt].y, o[0]));
          o[1] = fmaf(x.x, p[nt].y, fmaf(x.y, p[nt].x, o[1]));
          o[2] = fmaf(x.z, p[nt].x, fmaf(-x.w, p[nt].y, o[2]));
          o[3] = fmaf(x.z, p[nt].y, fmaf(x.w, p[nt].x, o[3]));
        });
      });
    }
    static_for<0, NK>([&](auto i) {
      constexpr int nt = decltype(i)::value;
      if (g == 0) y[nt][0][0] = y[nt][0][1] = 0.f;   // the j = 0 point is not fitted
      if (rif[nt] < 0) {
        static_for<0, KP * 16>([&](auto kk) {
          constexpr int k = decltype(kk)::value;
          y[nt][k / 16][k % 16] = 0.f;
        });
      }
    });
    // bounds from above: row_max on sum_j |y[n][j]| (so on |X[n]|) of every
    // IF, s1 on sum |y|, by Cauchy-Schwarz over each lane's 8 KP values; a
    // NaN or infinite component leaves s1 not finite
    float s1 = 0.f, row_max = 0.f;
    static_for<0, NK>([&](auto i) {
      constexpr int nt = decltype(i)::value;
      float e2 = 0.f;
      static_for<0, KP * 16>([&](auto kk) {
        constexpr int k = decltype(kk)::value;
        e2 = fmaf(y[nt][k / 16][k % 16], y[nt][k / 16][k % 16], e2);
      });
      float t = sqrtf(e2 * float(8 * KP));
      t += __shfl_xor(t, 16, 64);
      t += __shfl_xor(t, 32, 64);
      row_max = fmaxf(row_max, t);
      s1 += t;
    });
    for (int o = 8; o > 0; o >>= 1) {
      s1 += __shfl_xor(s1, o, 64);
      row_max = fmaxf(row_max, __shfl_xor(row_max, o, 64));
    }
    unsigned char *rec = a.rec + int64_t(task) * screen_rec_bytes(units);
    // outside this range |G|^2 could leave the float32 range
    if (!(s1 < 1e15f) || !(s1 > 1e-12f)) {
      if (lane == 0) *reinterpret_cast<float2 *>(rec) = make_float2(0.f, __builtin_inff());
      if (lane < units) rec[8 + lane] = 1;
      continue;
    }
    // power-of-two scale with row_max * scale < 2^15
    const int e = int(__float_as_uint(row_max * 1.0001f) >> 23) - 127;
    const float sc = __uint_as_float(unsigned(127 + 14 - e) << 23);

    // A operands: chunk 2 kp holds the even channels, 2 kp + 1 the odd ones
    h8_t ya[NK][2 * KP], yb[NK][2 * KP];
    static_for<0, NK * 2 * KP>([&](auto i) {
      constexpr int nt = decltype(i)::value / (2 * KP), kc = decltype(i)::value % (2 * KP);
      float re[4], im[4];
      static_for<0, 4>([&](auto q) {
        constexpr int h = decltype(q)::value;
        re[h] = y[nt][kc / 2][4 * h + 2 * (kc % 2)] * sc;
        im[h] = y[nt][kc / 2][4 * h + 2 * (kc % 2) + 1] * sc;
      });
      embed(re, im, ya[nt][kc], yb[nt][kc]);
    });

    float mine = 0.f;   // largest |G|^2 of unit `lane`
    float x2 = 0.f;     // largest sum of |X|^2 over this lane's IFs
    for (int p0 = 0; p0 < units / 2; p0 += UP) {
      // SBD of UP unit pairs -> A operands of the MBD product
      h8_t xa[2 * UP][NK], xb[2 * UP][NK];
      static_for<0, UP>([&](auto pi) {
        constexpr int p = decltype(pi)::value;
        h8_t b[2 * KP];
        static_for<0, 2 * KP>([&](auto kk) {
          constexpr int kc = decltype(kk)::value;
          b[kc] = Fs[((p0 + p) * 2 * KP + kc) * 64 + lane];
        });
        float z2[2] = {0.f, 0.f};
        static_for<0, NK>([&](auto i) {
          constexpr int nt = decltype(i)::value;
          f4_t er = {0.f, 0.f, 0.f, 0.f}, ei = er, dr = er, di = er;
          static_for<0, KP>([&](auto kk) {
            constexpr int k = 2 * decltype(kk)::value;
            er = __builtin_amdgcn_mfma_f32_16x16x32_f16(ya[nt][k], b[k], er, 0, 0, 0);
            ei = __builtin_amdgcn_mfma_f32_16x16x32_f16(yb[nt][k], b[k], ei, 0, 0, 0);
            dr = __builtin_amdgcn_mfma_f32_16x16x32_f16(ya[nt][k + 1], b[k + 1], dr, 0, 0, 0);
            di = __builtin_amdgcn_mfma_f32_16x16x32_f16(yb[nt][k + 1], b[k + 1], di, 0, 0, 0);
          });
          float re[2][4], im[2][4];
          static_for<0, 4>([&](auto q) {
            constexpr int k = decltype(q)::value;
            re[0][k] = er[k] + dr[k];
            im[0][k] = ei[k] + di[k];
            re[1][k] = er[k] - dr[k];
            im[1][k] = ei[k] - di[k];
          });
          static_for<0, 2>([&](auto hh) {
            constexpr int h = decltype(hh)::value;
            embed(re[h], im[h], xa[2 * p + h][nt], xb[2 * p + h][nt]);
            const u4_t w = __builtin_bit_cast(u4_t, xa[2 * p + h][nt]);
            static_for<0, 4>([&](auto q) {
              const h2_t c = __builtin_bit_cast(h2_t, w[decltype(q)::value]);
              z2[h] = __builtin_amdgcn_fdot2(c, c, z2[h], false);
            });
          });
        });
        x2 = fmaxf(x2, fmaxf(z2[0], z2[1]));
      });
      // MBD of the units, 16 columns at a time
      float mx[2 * UP];
      static_for<0, 2 * UP>([&](auto ui) { mx[decltype(ui)::value] = 0.f; });
#pragma unroll 2
      for (int ct = 0; ct < MT; ++ct) {
        h8_t b[NK];
        static_for<0, NK>([&](auto i) { b[decltype(i)::value] = Fm[(ct * NK + decltype(i)::value) * 64 + lane]; });
        static_for<0, 2 * UP>([&](auto ui) {
          constexpr int u = decltype(ui)::value;
          const f4_t zero = {0.f, 0.f, 0.f, 0.f};
          f4_t gr = __builtin_amdgcn_mfma_f32_16x16x32_f16(xa[u][0], b[0], zero, 0, 0, 0);
          f4_t gi = __builtin_amdgcn_mfma_f32_16x16x32_f16(xb[u][0], b[0], zero, 0, 0, 0);
          float v[4];
          if constexpr (HALF) {
            const f4_t hr = __builtin_amdgcn_mfma_f32_16x16x32_f16(xa[u][1], b[1], zero, 0, 0, 0);
            const f4_t hi_ = __builtin_amdgcn_mfma_f32_16x16x32_f16(xb[u][1], b[1], zero, 0, 0, 0);
            static_for<0, 4>([&](auto q) {
              constexpr int k = decltype(q)::value;
              const float t = fmaf(hi_[k], hi_[k], fmaf(hr[k], hr[k], fmaf(gi[k], gi[k], gr[k] * gr[k])));
              const float d = fmaf(gi[k], hi_[k], gr[k] * hr[k]);
              v[k] = fmaf(2.f, fabsf(d), t);
            });
          } else {
            static_for<1, NK>([&](auto i) {
              constexpr int nt = decltype(i)::value;
              gr = __builtin_amdgcn_mfma_f32_16x16x32_f16(xa[u][nt], b[nt], gr, 0, 0, 0);
              gi = __builtin_amdgcn_mfma_f32_16x16x32_f16(xb[u][nt], b[nt], gi, 0, 0, 0);
            });
            static_for<0, 4>([&](auto q) {
              constexpr int k = decltype(q)::value;
              v[k] = fmaf(gr[k], gr[k], gi[k] * gi[k]);
            });
          }
          mx[u] = fmaxf(fmaxf(mx[u], v[0]), v[1]);
          mx[u] = fmaxf(fmaxf(mx[u], v[2]), v[3]);
        });
      }
      // pair p is units sb and sb + NH of sub-grid c
      static_for<0, 2 * UP>([&](auto ui) {
        constexpr int u = decltype(ui)::value;
        const int p = p0 + u / 2;
        const int id = (p / NH) * NSB + p % NH + (u % 2) * NH;
        const float m = wave_max(mx[u]);
        mine = lane == id ? m : mine;
      });
    }
    // |screened G - G| <= eps_y sum |y| + eps_x sqrt(N) max_s |X(s)|_2 + ...
    x2 = fmaxf(x2, __shfl_xor(x2, 1, 64));
    x2 = fmaxf(x2, __shfl_xor(x2, 2, 64));
    x2 = fmaxf(x2, __shfl_xor(x2, 4, 64));
    x2 = fmaxf(x2, __shfl_xor(x2, 8, 64));
    x2 += __shfl_xor(x2, 16, 64);
    x2 += __shfl_xor(x2, 32, 64);
    const float bound = a.eps_y * s1 * sc + a.eps_x * sqrtf(x2 * float(N)) + a.abs_scaled + a.abs_plain * sc;
    // the record: A, B and per unit its distance below A in steps of B / 127
    const float A = sqrtf(wave_max(mine));
    if (lane == 0) *reinterpret_cast<float2 *>(rec) = make_float2(A / sc, bound / sc);
    if (lane < units) {
      const float d = (A - sqrtf(mine)) * (127.f / bound);
      rec[8 + lane] = d <= 254.f ? (unsigned char)(1 + int(d)) : (unsigned char)0;
    }
  }
}

constexpr size_t kScreenLdsMax = 150 * 1024;

size_t screen_lds(int n_chan, int n_if, bool half, int units) {
  return size_t((half ? 8 : 16) * (n_if <= 16 ? 1 : 2) + units * (n_chan / 32)) * 64 * sizeof(h8_t);
}

// f(kernel) for the instantiation of a shape
template <typename F>
hipError_t with_kernel(int n_chan, int n_if, bool half, F &&f) {
  const bool two = n_if > 16;
  switch (n_chan) {
    case 32: return half ? f(&screen_kernel<32, 2, true>) : two ? f(&screen_kernel<32, 2, false>) : f(&screen_kernel<32, 1, false>);
    case 64: return half ? f(&screen_kernel<64, 2, true>) : two ? f(&screen_kernel<64, 2, false>) : f(&screen_kernel<64, 1, false>);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

bool screen_supported(int n_chan, int n_mbd, int n_if, int sbd_pad) {
  if (n_mbd != 256 || n_if < 1 || n_if > 32) return false;
  if (n_chan != 32 && n_chan != 64) return false;
  const int units = sbd_pad * n_chan / 16;
  return units >= 4 && units <= kScreenUnitsMax && screen_lds(n_chan, n_if, false, units) <= kScreenLdsMax;
}

hipError_t screen_blocks(int n_chan, int n_if, bool half, int sbd_pad, int device, int *blocks) {
  const size_t lds = screen_lds(n_chan, n_if, half, sbd_pad * n_chan / 16);
  (void)hipGetLastError();
  return with_kernel(n_chan, n_if, half, [&](auto kern) -> hipError_t {
    const void *fn = reinterpret_cast<const void *>(kern);
    // (the largest any shape needs: the attribute belongs to the function, not to this context)
    hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, int(kScreenLdsMax));
    if (e != hipSuccess) return e;
    int per_cu = 0, cus = 0;
    if ((e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, kScreenBlock, lds)) != hipSuccess) return e;
    if ((e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device)) != hipSuccess) return e;
    *blocks = std::max(1, per_cu) * std::max(1, cus);
    return hipSuccess;
  });
}

hipError_t launch_screen(int n_chan, const ScreenArgs &a, int blocks, hipStream_t s) {
  if (a.n_task <= 0) return hipSuccess;
  if (a.units < 4 || a.units % 4 || a.units > kScreenUnitsMax || a.n_if < 1 || a.n_if > 32 || blocks < 1 || !a.rec ||
      !a.f_sbd || !a.f_mbd || (a.half && a.n_if <= 16))
    return hipErrorInvalidValue;
  const size_t lds = screen_lds(n_chan, a.n_if, a.half != 0, a.units);
  if (lds > kScreenLdsMax) return hipErrorInvalidValue;
  const int need = (a.n_task + kScreenWaves - 1) / kScreenWaves;
  (void)hipGetLastError();
  return with_kernel(n_chan, a.n_if, a.half != 0, [&](auto kern) -> hipError_t {
    hipLaunchKernelGGL(kern, dim3(std::min(blocks, need)), dim3(kScreenBlock), lds, s, a);
    return hipGetLastError();
  });
}

}  // namespace frbx
