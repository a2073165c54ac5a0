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
// registers.  A = [re, im] against B = [cos, sin] is the real part of the
// product, against [-sin, cos] the imaginary one.
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
typedef float f4_t __attribute__((ext_vector_type(4)));

constexpr int kScreenBlock = 64 * kScreenWaves;

// A operand [re, im] of four complex values.
__device__ __forceinline__ h8_t pack(const float (&re)[4], const float (&im)[4]) {
  return h8_t{_Float16(re[0]), _Float16(re[1]), _Float16(re[2]), _Float16(re[3]),
              _Float16(im[0]), _Float16(im[1]), _Float16(im[2]), _Float16(im[3])};
}

// Largest value of the wave, in every lane (v >= 0: its bits order like it).
__device__ __forceinline__ float wave_max(float v) {
  unsigned m = __float_as_uint(v);
  auto step = [&](auto ctrl) {
    constexpr int c = decltype(ctrl)::value;
    m = max(m, unsigned(__builtin_amdgcn_update_dpp(0, int(m), c, 0xf, 0xf, true)));
  };
  step(Index<0xb1>{});    // quad_perm 1 0 3 2
  step(Index<0x4e>{});    // quad_perm 2 3 0 1
  step(Index<0x141>{});   // row_half_mirror
  step(Index<0x140>{});   // row_mirror
  step(Index<0x142>{});   // row_bcast15
  step(Index<0x143>{});   // row_bcast31
  return __uint_as_float(unsigned(__builtin_amdgcn_readlane(int(m), 63)));
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
  h8_t *const Fm = lds_h;                      // [MT][NK][re, im][64]
  h8_t *const Fs = lds_h + MT * NK * 2 * 64;   // [units / 2][2 KP][re, im][64]
  __shared__ int next;                         // tasks taken by the work-group
  const int N = a.n_if, R = a.n_rate, NJ = N * J, units = a.units;
  {
    const h8_t *gm = static_cast<const h8_t *>(a.f_mbd), *gs = static_cast<const h8_t *>(a.f_sbd);
    for (int i = threadIdx.x; i < MT * NK * 2 * 64; i += kScreenBlock) Fm[i] = gm[i];
    for (int i = threadIdx.x; i < units * KP * 2 * 64; i += kScreenBlock) Fs[i] = gs[i];
    if (threadIdx.x == 0) next = 0;
  }
  __syncthreads();
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

  for (;;) {
    // the work-group's next task: waves on one SIMD do not advance evenly (the
    // older one issues first), so none has tasks of its own
    int k = 0;
    if (lane == 0) k = atomicAdd(&next, 1);
    k = __builtin_amdgcn_readfirstlane(k);
    const int64_t at = lo + int64_t(k / kScreenWaves) * stride + slot * kScreenWaves + k % kScreenWaves;
    if (at >= hi) break;
    const int task = int(at);
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
    int off[NK], pho[NK];
    static_for<0, NK>([&](auto i) {
      constexpr int nt = decltype(i)::value;
      const int n = max(rif[nt], 0);
      off[nt] = n * J + 2 * g;
      pho[nt] = n * l;
    });
    auto add_ap = [&](int u, auto first_tag) {
      constexpr bool FIRST = decltype(first_tag)::value != 0;
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
          o[0] = fmaf(x.x, p[nt].x, FIRST ? -x.y * p[nt].y : fmaf(-x.y, p[nt].y, o[0]));
          o[1] = fmaf(x.x, p[nt].y, FIRST ? x.y * p[nt].x : fmaf(x.y, p[nt].x, o[1]));
          o[2] = fmaf(x.z, p[nt].x, FIRST ? -x.w * p[nt].y : fmaf(-x.w, p[nt].y, o[2]));
          o[3] = fmaf(x.z, p[nt].y, FIRST ? x.w * p[nt].x : fmaf(x.w, p[nt].x, o[3]));
        });
      });
    };
    add_ap(0, Index<1>{});
    for (int u = 1; u < l; ++u) add_ap(u, Index<0>{});
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
    h8_t ya[NK][2 * KP];
    static_for<0, NK * 2 * KP>([&](auto i) {
      constexpr int nt = decltype(i)::value / (2 * KP), kc = decltype(i)::value % (2 * KP);
      float re[4], im[4];
      static_for<0, 4>([&](auto q) {
        constexpr int h = decltype(q)::value;
        re[h] = y[nt][kc / 2][4 * h + 2 * (kc % 2)] * sc;
        im[h] = y[nt][kc / 2][4 * h + 2 * (kc % 2) + 1] * sc;
      });
      ya[nt][kc] = pack(re, im);
    });

    float mine = 0.f;   // largest |G|^2 of unit `lane`
    float x2 = 0.f;     // largest sum of |X|^2 over this lane's IFs
    for (int p0 = 0; p0 < units / 2; p0 += UP) {
      // SBD of UP unit pairs -> A operands of the MBD product
      h8_t xa[2 * UP][NK];
      static_for<0, UP>([&](auto pi) {
        constexpr int p = decltype(pi)::value;
        h8_t b[2 * KP][2];
        static_for<0, 4 * KP>([&](auto kk) {
          constexpr int k = decltype(kk)::value;
          b[k / 2][k % 2] = Fs[((p0 + p) * 4 * KP + k) * 64 + lane];
        });
        float z2[2] = {0.f, 0.f};
        static_for<0, NK>([&](auto i) {
          constexpr int nt = decltype(i)::value;
          f4_t er = {0.f, 0.f, 0.f, 0.f}, ei = er, dr = er, di = er;
          static_for<0, KP>([&](auto kk) {
            constexpr int k = 2 * decltype(kk)::value;
            er = __builtin_amdgcn_mfma_f32_16x16x32_f16(ya[nt][k], b[k][0], er, 0, 0, 0);
            ei = __builtin_amdgcn_mfma_f32_16x16x32_f16(ya[nt][k], b[k][1], ei, 0, 0, 0);
            dr = __builtin_amdgcn_mfma_f32_16x16x32_f16(ya[nt][k + 1], b[k + 1][0], dr, 0, 0, 0);
            di = __builtin_amdgcn_mfma_f32_16x16x32_f16(ya[nt][k + 1], b[k + 1][1], di, 0, 0, 0);
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
            xa[2 * p + h][nt] = pack(re[h], im[h]);
            static_for<0, 4>([&](auto q) {
              constexpr int k = decltype(q)::value;
              z2[h] = fmaf(re[h][k], re[h][k], fmaf(im[h][k], im[h][k], z2[h]));
            });
          });
        });
        x2 = fmaxf(x2, fmaxf(z2[0], z2[1]));
      });
      // MBD of the units, 16 columns at a time: the products of a step (one
      // unit, 16 columns) are issued among the powers of the step before
      float mx[2 * UP];
      static_for<0, 2 * UP>([&](auto ui) { mx[decltype(ui)::value] = 0.f; });
      f4_t acc[2][4];   // HALF: re, im of a, re, im of b; else re, im
      auto product = [&](auto ui, const h8_t (&b)[NK][2], f4_t (&o)[4]) {
        constexpr int u = decltype(ui)::value;
        const f4_t zero = {0.f, 0.f, 0.f, 0.f};
        o[0] = __builtin_amdgcn_mfma_f32_16x16x32_f16(xa[u][0], b[0][0], zero, 0, 0, 0);
        o[1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(xa[u][0], b[0][1], zero, 0, 0, 0);
        if constexpr (HALF) {
          o[2] = __builtin_amdgcn_mfma_f32_16x16x32_f16(xa[u][1], b[1][0], zero, 0, 0, 0);
          o[3] = __builtin_amdgcn_mfma_f32_16x16x32_f16(xa[u][1], b[1][1], zero, 0, 0, 0);
        } else {
          static_for<1, NK>([&](auto i) {
            constexpr int nt = decltype(i)::value;
            o[0] = __builtin_amdgcn_mfma_f32_16x16x32_f16(xa[u][nt], b[nt][0], o[0], 0, 0, 0);
            o[1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(xa[u][nt], b[nt][1], o[1], 0, 0, 0);
          });
        }
      };
      auto powers = [&](const f4_t (&o)[4], float &m) {
        float v[4];
        static_for<0, 4>([&](auto q) {
          constexpr int k = decltype(q)::value;
          v[k] = fmaf(o[1][k], o[1][k], o[0][k] * o[0][k]);
          if constexpr (HALF) {
            v[k] = fmaf(o[3][k], o[3][k], fmaf(o[2][k], o[2][k], v[k]));
            v[k] = fmaf(2.f, fabsf(fmaf(o[1][k], o[3][k], o[0][k] * o[2][k])), v[k]);
          }
        });
        m = fmaxf(fmaxf(m, v[0]), v[1]);
        m = fmaxf(fmaxf(m, v[2]), v[3]);
      };
      h8_t b[NK][2], bn[NK][2];
      auto operand = [&](int ct, h8_t (&o)[NK][2]) {
        static_for<0, 2 * NK>([&](auto i) {
          constexpr int k = decltype(i)::value;
          o[k / 2][k % 2] = Fm[(ct * 2 * NK + k) * 64 + lane];
        });
      };
      operand(0, b);
      product(Index<0>{}, b, acc[0]);
#pragma unroll 1
      for (int ct = 0; ct < MT; ++ct) {
        const int cn = ct + 1 < MT ? ct + 1 : 0;
        operand(cn, bn);
        static_for<0, 2 * UP>([&](auto ui) {
          constexpr int u = decltype(ui)::value, un = (u + 1) % (2 * UP);
          product(Index<un>{}, un == 0 ? bn : b, acc[(u + 1) & 1]);
          powers(acc[u & 1], mx[u]);
          static_for<0, (HALF ? 4 : 2 * NK)>([&](auto) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                            // one MFMA,
            __builtin_amdgcn_sched_group_barrier(0x002, HALF ? 8 : NK == 2 ? 3 : 5, 0);   // its share of the powers
          });
        });
        static_for<0, 2 * NK>([&](auto i) {
          constexpr int k = decltype(i)::value;
          b[k / 2][k % 2] = bn[k / 2][k % 2];
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
  return size_t((half ? 8 : 16) * (n_if <= 16 ? 1 : 2) + units * (n_chan / 32)) * 2 * 64 * sizeof(h8_t);
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
