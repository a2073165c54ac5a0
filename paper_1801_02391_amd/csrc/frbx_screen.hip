// Screening pass of the fringe search (Eq. 5 with the Eq. 4 rate term,
// Sec. 5.1) on the gfx950 matrix cores.
//
// The search keeps one number per segment, the largest |G| over (rate, SBD,
// MBD), so all but a few cells are needed only to know that they are smaller.
// screen_kernel evaluates every cell in float16 (float32 accumulation) and
// reports, per segment and rate, the quads (4 SBD bins of one sub-grid x all
// MBD bins; from 128 channels on units of 16 bins) whose largest |G| lies
// within twice a rigorous error bound of the rate's largest; the search's own
// kernel then evaluates those, in its own arithmetic, and nothing else.  Since
// the bound covers every rounding of this pass, the cell that is the search's
// maximum is always among them and the search's result is what it is without
// this pass, bit for bit.
//
// Bound by vector issue: 41184 segments of 32 IFs x 64 channels with 8 rates
// take 4.8 ms (evaluating every cell in float32 took 14.0).  A task issues 7030
// vector instructions, 592 of them matrix products (0.65 PFLOP/s): at four
// cycles each 88 % of the SIMDs' cycles at 2.07 GHz, the matrix pipes busy in
// 30 %.  With 128 channels 67 % and 18 % (0.40 PFLOP/s, 420 bytes of scratch
// per lane, 8.7 ms for 22824 segments).
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
// work-group of eight waves per CU keeps them for the whole launch.
//
// Where the sums are large (64 channels or more, at least four rates) the
// eight waves take consecutive tasks, mostly the rates of one segment, and
// read its spectra from an LDS ring that they fill together, direct from
// memory, while they are still at the tasks before: every rate for itself
// fetched each spectrum again (45 GB a launch at 32 IFs x 128 channels, where
// the sums then took half the pass).  Elsewhere waves never wait for each
// other.
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
template <int C>
__device__ __forceinline__ unsigned dpp_max(unsigned m) {
  return max(m, unsigned(__builtin_amdgcn_update_dpp(0, int(m), C, 0xf, 0xf, true)));
}
// largest (as bits) of the 16 lanes of a row, in all of them
__device__ __forceinline__ unsigned row_max16(float v) {
  unsigned m = dpp_max<0xb1>(__float_as_uint(v));   // quad_perm 1 0 3 2
  m = dpp_max<0x4e>(m);                             // quad_perm 2 3 0 1
  m = dpp_max<0x141>(m);                            // row_half_mirror
  return dpp_max<0x140>(m);                         // row_mirror
}
__device__ __forceinline__ float wave_max(float v) {
  unsigned m = row_max16(v);
  m = dpp_max<0x142>(m);   // row_bcast15
  m = dpp_max<0x143>(m);   // row_bcast31
  return __uint_as_float(unsigned(__builtin_amdgcn_readlane(int(m), 63)));
}

// SBD: with j = RX i + p (RX = J / 16 residues p of 16 channels i each) and
// the bins s' = s0 + 16 P k of one sub-grid (s0 = c + P column, k < RX),
// X(s') = sum_p w_RX^(p k) E_p(s0), E_p = sum_i y[RX i + p] w_PJ^(j s0): one
// product of K = (16 i, re/im) per residue and an RX-point DFT in registers
// give all RX units of the sub-grid.
// HALF: the MBD product on half of its columns.  Rows n hold the IFs of even
// lattice position in chunk 0 and of odd position in chunk 1; with a and b
// their sums for bin m < M / 2, G(m) = a + b and G(m + M/2) = a - b, and only
// the larger counts: max |a +- b|^2 = |a|^2 + |b|^2 + 2 |Re a conj(b)|.
// Otherwise the columns may be a coarser grid of the MBD axis (a.tiles x 16
// bins), whose largest |G| bounds the full grid's (a.gamma).
// RING: the spectra come through the LDS ring.  With 256 channels the ring's
// room comes from the SBD matrix: E_p = w_PJ^(p s0) sum_i y[RX i + p]
// w_PJ^(RX i s0) with one matrix per sub-grid and the factor applied in
// float32.
constexpr int kRing = 3;   // slabs

// What one slab of the ring holds: NTS x 16 operand rows of CH chunks of two
// channels (NP slabs to an AP), then every wave's rate phasors of the AP's
// rows.  The chunks of a row are stored in XOR order so that the 16 rows a
// read touches lie in different banks.
template <int J, int NK>
struct Slab {
  static constexpr int NP = (J == 128 && NK == 2) || J == 256 ? 2 : 1;
  static constexpr int NTS = J == 128 ? 1 : NK;               // 16-row tiles
  static constexpr int HS = J == 256 ? 2 : 4;                 // h of a lane's channels
  static constexpr int CH = HS * 4 * (J / 16) / 2;            // 16-byte chunks per row
  static constexpr int BYTES = NTS * 16 * CH * 16;
  static constexpr int LOADS = BYTES / 1024 / kScreenWaves;   // per wave, 1 KiB each
  static constexpr int STRIDE = BYTES + kScreenWaves * 256;
};

// 64 lanes x 16 (4) bytes from each lane's address to LDS offset `lds` + 16
// (4) lane, without passing through registers; completion counts in vmcnt.
__device__ __forceinline__ void load_lds16(const void *src, unsigned lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds), "v"(src) : "memory", "m0");
}
__device__ __forceinline__ void load_lds4(const void *src, unsigned lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off" ::"s"(lds), "v"(src) : "memory", "m0");
}

// A position in the sequence of slabs of the work-group's blocks of eight
// tasks: block, segment, AP and part.
struct SlabCursor {
  int block, sg, last_sg, u, l, part;
  const float2 *wd, *ph;   // the segment's spectra and its window's phasors
};

template <int J, int NK, bool HALF, bool RING>
__global__ __launch_bounds__(kScreenBlock) __attribute__((amdgpu_waves_per_eu(2)))
void screen_kernel(ScreenArgs a) {
  constexpr int RX = J / 16;
  constexpr int CG = RX >= 4 ? 1 : 4 / RX;   // sub-grids per pass over the MBD matrix
  constexpr int U = CG * RX;                 // units per pass
  constexpr bool TWIDDLE = RING && J == 256;
  constexpr int NF = TWIDDLE ? 1 : RX;       // SBD matrices per sub-grid
  extern __shared__ h8_t lds_h[];
  const int N = a.n_if, R = a.n_rate, NJ = N * J, units = a.units, P = units / RX;
  const int MT = HALF ? 8 : a.tiles;
  char *const ring = reinterpret_cast<char *>(lds_h);   // first: its offsets stay within 64 KiB
  h8_t *const Fm = lds_h + (RING ? kRing * Slab<J, NK>::STRIDE / 16 : 0);   // [MT][NK][re, im][64]
  h8_t *const Fs = Fm + MT * NK * 2 * 64;                                   // [P][NF][re, im][64]
  float2 *const TW = reinterpret_cast<float2 *>(Fs + P * NF * 2 * 64);      // TWIDDLE: [P J]
  __shared__ int next;                                  // tasks taken by the work-group
  {
    const h8_t *gm = static_cast<const h8_t *>(a.f_mbd), *gs = static_cast<const h8_t *>(a.f_sbd);
    for (int i = threadIdx.x; i < MT * NK * 2 * 64; i += kScreenBlock) Fm[i] = gm[i];
    for (int i = threadIdx.x; i < P * NF * 2 * 64; i += kScreenBlock)
      Fs[i] = gs[i / (NF * 128) * (RX * 128) + i % (NF * 128)];
    if constexpr (TWIDDLE)
      for (int i = threadIdx.x; i < P * J; i += kScreenBlock) TW[i] = a.tw_sbd[i];
    if (threadIdx.x == 0) next = 0;
  }
  __syncthreads();
  const int lane = threadIdx.x & 63, row = lane & 15, g = lane >> 4;
  // the IF of this lane's rows (absent rows read the first IF's data and are cleared)
  int rif[NK];
  static_for<0, NK>([&](auto i) { rif[decltype(i)::value] = a.row_if[16 * decltype(i)::value + row]; });
  // Tasks (segment, rate), rate fastest, dealt out in sweeps over the grid.
  // Work-groups go to the 8 XCDs round-robin: those of one XCD take
  // consecutive tasks of a sweep, so that the waves in flight on it read the
  // same few segments from its L2.
  const int nb = gridDim.x;
  const int slot = (nb & 7) == 0 ? (blockIdx.x & 7) * (nb >> 3) + (blockIdx.x >> 3) : blockIdx.x;

  // window and address of a segment
  auto segment = [&](int sg, int &l, const float2 *&wd, const float2 *&ph) {
    const int dl = sg / a.seg_total, seg = sg - dl * a.seg_total;
    int wi = 0;
    while (wi + 1 < a.n_win && a.win_off[wi + 1] <= seg) ++wi;
    l = a.win_len[wi];
    const int64_t k0 = a.win_k0[wi] + int64_t(seg - a.win_off[wi]) * a.win_hop[wi];
    wd = a.w + int64_t(dl) * a.w_dm_stride + k0 * NJ;
    ph = a.rate_ph + a.rate_off[wi];
  };

  // ---- the ring: slab n of the sequence lies in slot n % kRing; slab n + 2
  // is asked for when every wave has finished with slab n - 1
  using SL = Slab<J, NK>;
  const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
  const int n_block = (a.n_task + kScreenWaves - 1) / kScreenWaves;
  const unsigned ring_at = unsigned(reinterpret_cast<uintptr_t>(
      (__attribute__((address_space(3))) char *)ring));
  unsigned goff[SL::NP][RING && SL::LOADS > 0 ? SL::LOADS : 1];   // this lane's elements of a part, from the AP's start
  unsigned poff = 0;                                              // and of the phasors: row, and re or im
  if constexpr (RING) {
    static_for<0, SL::NP * SL::LOADS>([&](auto i) {
      constexpr int part = decltype(i)::value / SL::LOADS, q = decltype(i)::value % SL::LOADS;
      const int pos = (wave * SL::LOADS + q) * 64 + lane;
      const int rw = pos / SL::CH, c = (pos % SL::CH) ^ (rw & 15);
      const int rt = SL::NTS < NK ? part * 16 + rw : rw;
      const int n = max(a.row_if[rt], 0), j0 = SL::HS < 4 ? part * SL::CH * 2 : 0;
      goff[part][q] = unsigned(n * J + j0 + 2 * c);
    });
    const int prow = lane / 2 < 16 * NK ? max(a.row_if[lane / 2], 0) : 0;
    poff = unsigned(prow);
  }
  auto open_block = [&](SlabCursor &c) {
    const int t0 = c.block * kScreenWaves;
    c.sg = t0 / R;
    c.last_sg = min(t0 + kScreenWaves - 1, a.n_task - 1) / R;
    c.u = c.part = 0;
    segment(c.sg, c.l, c.wd, c.ph);
  };
  // to the next slab; false at the end of the block
  auto advance = [&](SlabCursor &c) -> bool {
    if (++c.part < SL::NP) return true;
    c.part = 0;
    if (++c.u < c.l) return true;
    c.u = 0;
    if (++c.sg > c.last_sg) return false;
    segment(c.sg, c.l, c.wd, c.ph);
    return true;
  };
  auto fetch = [&](const SlabCursor &c, int at) {
    const unsigned dst = ring_at + unsigned(at) * SL::STRIDE;
    const float2 *ap = c.wd + int64_t(c.u) * NJ;
    static_for<0, (RING ? SL::LOADS : 0)>([&](auto i) {
      constexpr int q = decltype(i)::value;
      unsigned o = goff[0][q];
      if constexpr (SL::NP > 1) o = c.part ? goff[1][q] : o;
      load_lds16(ap + o, dst + unsigned(wave * SL::LOADS + q) * 1024u);
    });
    // the phasors of this wave's rate (of any rate where the segment is not its own)
    const int task = min(c.block * kScreenWaves + wave, a.n_task - 1), rr = task % R;
    const float *pv = reinterpret_cast<const float *>(c.ph + (int64_t(rr) * N + poff) * c.l + c.u) + (lane & 1);
    load_lds4(pv, dst + SL::BYTES + unsigned(wave) * 256u);
  };
  SlabCursor ld{}, use{};      // next slab to fetch, next to use
  int ld_at = 0, use_at = 0;   // their slots
  bool more = false;           // ld is valid
  auto fetch_next = [&]() {
    if (!more) return;
    fetch(ld, ld_at);
    ld_at = ld_at + 1 == kRing ? 0 : ld_at + 1;
    if (!advance(ld)) {
      ld.block += nb;
      more = ld.block < n_block;
      if (more) open_block(ld);
    }
  };
  if constexpr (RING) {
    ld.block = use.block = slot;
    more = slot < n_block;
    if (more) open_block(ld);
    fetch_next();
    fetch_next();
  }

  for (;;) {
    int task;
    bool live = true;   // (RING: the last block may have fewer tasks than waves)
    if constexpr (RING) {
      if (use.block >= n_block) break;
      task = use.block * kScreenWaves + wave;
      live = task < a.n_task;
    } else {
      // the work-group's next task: waves on one SIMD do not advance evenly (the
      // older one issues first), so none has tasks of its own
      int k = 0;
      if (lane == 0) k = atomicAdd(&next, 1);
      k = __builtin_amdgcn_readfirstlane(k);
      const int64_t at = (int64_t(k / kScreenWaves) * nb + slot) * kScreenWaves + k % kScreenWaves;
      if (at >= a.n_task) break;
      task = int(at);
    }
    const int sg = task / R, r = task - sg * R;
    int l = 1;
    const float2 *wd, *ph;
    if constexpr (!RING) {
      segment(sg, l, wd, ph);
      ph += int64_t(r) * N * l;
    }

    // ---- segment sums (Eq. 3 with the Eq. 4 rotation): lane (row, g) holds
    // row 16 nt + row, channels RX (4 h + g) + p, h < 4: y[nt][p][2 h + re/im]
    float y[NK][RX][8];
    // largest component of any of them after any AP, the j = 0 point's apart:
    // what the float32 rounding of the sums scales with (far above the sums
    // themselves where the APs of a window cancel)
    float sum_max = 0.f, sum_max0 = 0.f;
    auto grow = [](float &m, float re, float im) { m = fmaxf(fmaxf(m, fabsf(re)), fabsf(im)); };
    if constexpr (RING) {
      static_for<0, NK * RX * 8>([&](auto kk) {
        constexpr int q = decltype(kk)::value;
        y[q / (RX * 8)][(q / 8) % RX][q % 8] = 0.f;
      });
      open_block(use);
      for (bool in_block = true; in_block;) {
        // this wave's loads of the slab are done (one newer slab may be on its
        // way) and its reads of the slab before; then everyone's
        if (more) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(SL::LOADS + 1) : "memory");
        else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        fetch_next();
        if (use.sg == sg && live) {
          l = use.l;
          const char *sl = ring + use_at * SL::STRIDE;
          const float2 *pw = reinterpret_cast<const float2 *>(sl + SL::BYTES + wave * 256);
          const float4 *rows = reinterpret_cast<const float4 *>(sl);
          int rw = row, gr = g;
          // (RX >= 8: the addresses are formed anew, not kept in registers from slab to slab)
          if constexpr (RX >= 8) asm volatile("" : "+v"(rw), "+v"(gr));
          auto part = [&](auto pt) {
            constexpr int PT = decltype(pt)::value;
            static_for<0, SL::NTS>([&](auto ti) {
              constexpr int tl = decltype(ti)::value, nt = SL::NTS < NK ? PT : tl;
              const float2 w = pw[16 * nt + rw];
              static_for<0, SL::HS * RX / 2>([&](auto kk) {
                constexpr int hl = decltype(kk)::value / (RX / 2), pp = decltype(kk)::value % (RX / 2);
                constexpr int h = (SL::HS < 4 ? SL::HS * PT : 0) + hl;
                const float4 x = rows[(16 * tl + rw) * SL::CH + (((4 * hl + gr) * (RX / 2) + pp) ^ rw)];
                float *o = &y[nt][2 * pp][2 * h], *o2 = &y[nt][2 * pp + 1][2 * h];
                o[0] = fmaf(x.x, w.x, fmaf(-x.y, w.y, o[0]));
                o[1] = fmaf(x.x, w.y, fmaf(x.y, w.x, o[1]));
                o2[0] = fmaf(x.z, w.x, fmaf(-x.w, w.y, o2[0]));
                o2[1] = fmaf(x.z, w.y, fmaf(x.w, w.x, o2[1]));
                grow(pp == 0 && h == 0 ? sum_max0 : sum_max, o[0], o[1]);
                grow(sum_max, o2[0], o2[1]);
              });
            });
          };
          if constexpr (SL::NP == 1) {
            part(Index<0>{});
          } else {
            if (use.part == 0) part(Index<0>{});
            else part(Index<1>{});
          }
        }
        use_at = use_at + 1 == kRing ? 0 : use_at + 1;
        in_block = advance(use);
      }
      use.block += nb;
      if (!live) continue;
    }
    if constexpr (!RING) {
    int off[NK], pho[NK];
    static_for<0, NK>([&](auto i) {
      constexpr int nt = decltype(i)::value;
      const int n = max(rif[nt], 0);
      off[nt] = n * J + RX * g;
      pho[nt] = n * l;
    });
    // loads of two channels at a time (one with RX = 1), 16 in flight: several
    // APs together where one AP has fewer, parts of an AP where it has more
    constexpr int PP = RX > 1 ? RX / 2 : 1;               // loads per (row, h)
    constexpr int NL = NK * 4 * PP, UA = NL < 16 ? 16 / NL : 1, NB = NL < 16 ? NL : 16;
    auto add_aps = [&](int u0, auto first_tag) {
      constexpr bool FIRST = decltype(first_tag)::value != 0;
      const float2 *src[UA];
      float2 p[UA][NK];
      static_for<0, UA>([&](auto ai) {
        constexpr int ua = decltype(ai)::value;
        const int u = min(u0 + ua, l - 1);   // past the segment: its last AP with weight 0
        src[ua] = wd + int64_t(u) * NJ;
        static_for<0, NK>([&](auto i) {
          constexpr int nt = decltype(i)::value;
          p[ua][nt] = ph[pho[nt] + u];
          if (ua > 0 && u0 + ua >= l) p[ua][nt] = make_float2(0.f, 0.f);
        });
      });
      static_for<0, NL / NB>([&](auto bi) {
        float4 v[UA][NB];
        static_for<0, UA * NB>([&](auto kk) {
          constexpr int ua = decltype(kk)::value / NB, q = decltype(bi)::value * NB + decltype(kk)::value % NB;
          constexpr int nt = q / (4 * PP), h = (q / PP) % 4, pp = q % PP;
          const float2 *at2 = src[ua] + off[nt] + 4 * RX * h + 2 * pp;
          if constexpr (RX > 1) {
            v[ua][q % NB] = *reinterpret_cast<const float4 *>(at2);
          } else {
            const float2 z = *at2;
            v[ua][q % NB] = make_float4(z.x, z.y, 0.f, 0.f);
          }
        });
        if constexpr (NL > NB) __builtin_amdgcn_sched_barrier(0);
        static_for<0, UA * NB>([&](auto kk) {
          constexpr int ua = decltype(kk)::value / NB, q = decltype(bi)::value * NB + decltype(kk)::value % NB;
          constexpr int nt = q / (4 * PP), h = (q / PP) % 4, pp = q % PP;
          constexpr bool SET = FIRST && ua == 0;
          const float4 x = v[ua][q % NB];
          const float2 w = p[ua][nt];
          float *o = &y[nt][2 * pp < RX ? 2 * pp : 0][2 * h];
          o[0] = fmaf(x.x, w.x, SET ? -x.y * w.y : fmaf(-x.y, w.y, o[0]));
          o[1] = fmaf(x.x, w.y, SET ? x.y * w.x : fmaf(x.y, w.x, o[1]));
          grow(pp == 0 && h == 0 ? sum_max0 : sum_max, o[0], o[1]);
          if constexpr (RX > 1) {
            float *o2 = &y[nt][2 * pp + 1 < RX ? 2 * pp + 1 : 0][2 * h];
            o2[0] = fmaf(x.z, w.x, SET ? -x.w * w.y : fmaf(-x.w, w.y, o2[0]));
            o2[1] = fmaf(x.z, w.y, SET ? x.w * w.x : fmaf(x.w, w.x, o2[1]));
            grow(sum_max, o2[0], o2[1]);
          }
        });
      });
    };
    add_aps(0, Index<1>{});
    for (int u = UA; u < l; u += UA) add_aps(u, Index<0>{});
    }
    static_for<0, NK>([&](auto i) {
      constexpr int nt = decltype(i)::value;
      if (g == 0) y[nt][0][0] = y[nt][0][1] = 0.f;   // the j = 0 point is not fitted
      if (rif[nt] < 0) {
        static_for<0, RX * 8>([&](auto kk) {
          constexpr int q = decltype(kk)::value;
          y[nt][q / 8][q % 8] = 0.f;
        });
      }
    });
    // bounds from above: row_max on sum_j |y[n][j]| (so on |X[n]|) of every
    // IF, s1 on sum |y|, by Cauchy-Schwarz over each lane's 4 RX values; a
    // NaN or infinite component leaves s1 not finite
    float s1 = 0.f, row_max = 0.f;
    static_for<0, NK>([&](auto i) {
      constexpr int nt = decltype(i)::value;
      float e2 = 0.f;
      static_for<0, RX * 8>([&](auto kk) {
        constexpr int q = decltype(kk)::value;
        e2 = fmaf(y[nt][q / 8][q % 8], y[nt][q / 8][q % 8], e2);
      });
      float t = sqrtf(e2 * float(4 * RX));
      t += __shfl_xor(t, 16, 64);
      t += __shfl_xor(t, 32, 64);
      row_max = fmaxf(row_max, t);
      s1 += t;
    });
    // the rounding of the sums, in units of eps_y: a.eps_sum l for every
    // channel's largest partial sum (screen_bounds)
    sum_max = g == 0 ? sum_max : fmaxf(sum_max, sum_max0);
    if (NK == 1 && rif[0] < 0) sum_max = 0.f;
    sum_max += __shfl_xor(sum_max, 16, 64);
    sum_max += __shfl_xor(sum_max, 32, 64);
    float s1p = fmaf(a.eps_sum * float(l), sum_max, s1);
    for (int o = 8; o > 0; o >>= 1) {
      s1 += __shfl_xor(s1, o, 64);
      s1p += __shfl_xor(s1p, o, 64);
      row_max = fmaxf(row_max, __shfl_xor(row_max, o, 64));
    }
    unsigned char *rec = a.rec + int64_t(task) * screen_rec_bytes(units);
    // outside this range |G|^2 could leave the float32 range
    if (!(s1p < 1e15f) || !(s1 > 1e-12f)) {
      if (lane == 0) *reinterpret_cast<float2 *>(rec) = make_float2(0.f, __builtin_inff());
      if (lane < units) reinterpret_cast<unsigned *>(rec + 8)[lane] = 0x01010101u;
      continue;
    }
    // power-of-two scale with row_max * scale < 2^15
    const int e = int(__float_as_uint(row_max * 1.0001f) >> 23) - 127;
    const float sc = __uint_as_float(unsigned(127 + 14 - e) << 23);

    // A operands, one chunk per residue
    h8_t ya[NK][RX];
    static_for<0, NK * RX>([&](auto i) {
      constexpr int nt = decltype(i)::value / RX, p = decltype(i)::value % RX;
      float re[4], im[4];
      static_for<0, 4>([&](auto q) {
        constexpr int h = decltype(q)::value;
        re[h] = y[nt][p][2 * h] * sc;
        im[h] = y[nt][p][2 * h + 1] * sc;
      });
      ya[nt][p] = pack(re, im);
    });

    // QUADS: largest |G|^2 (bits) of quad g of the units 16 k + row; else of
    // unit `lane`, for its four quads
    constexpr bool QUADS = RX <= 4;
    unsigned keep[QUADS ? 4 : 1] = {};
    float x2 = 0.f;     // largest sum of |X|^2 over this lane's IFs
    h8_t b[NK][2], bn[NK][2];   // MBD operands of a tile (tile 0 here and after every pass) and the next
    auto operand = [&](int ct, h8_t (&o)[NK][2]) {
      static_for<0, 2 * NK>([&](auto i) {
        constexpr int q = decltype(i)::value;
        o[q / 2][q % 2] = Fm[(ct * 2 * NK + q) * 64 + lane];
      });
    };
    operand(0, b);
    for (int c0 = 0; c0 * RX < units; c0 += CG) {
      // of the two waves of a SIMD the older issues first; the one that is ahead
      // steps back, so that both reach the ring's barrier together
      if constexpr (RING) {
        if (c0 == 0) __builtin_amdgcn_s_setprio(3);
        else if (c0 == 1) __builtin_amdgcn_s_setprio(2);
        else if (c0 == 2) __builtin_amdgcn_s_setprio(1);
        else __builtin_amdgcn_s_setprio(0);
      }
      // SBD of CG sub-grids -> A operands of the MBD product
      h8_t xa[U][NK];
      static_for<0, CG>([&](auto ci) {
        constexpr int cc = decltype(ci)::value;
        float z2[RX];
        static_for<0, NK>([&](auto i) {
          constexpr int nt = decltype(i)::value;
          f4_t er[RX], ei[RX];
          const h8_t *const fs = Fs + (c0 + cc) * NF * 2 * 64 + lane;
          h8_t bs[2][2] = {{fs[0], fs[64]}};
          const int s0 = c0 + cc + P * row;
          static_for<0, RX>([&](auto pi) {
            constexpr int p = decltype(pi)::value, q = TWIDDLE ? 0 : p & 1;
            const f4_t zero = {0.f, 0.f, 0.f, 0.f};
            if constexpr (p + 1 < NF) {
              bs[(p + 1) & 1][0] = fs[(p + 1) * 128];
              bs[(p + 1) & 1][1] = fs[(p + 1) * 128 + 64];
            }
            er[p] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ya[nt][p], bs[q][0], zero, 0, 0, 0);
            ei[p] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ya[nt][p], bs[q][1], zero, 0, 0, 0);
            if constexpr (TWIDDLE && p > 0) {
              const float2 w = TW[(p * s0) & (P * J - 1)];
              static_for<0, 4>([&](auto hh) {
                constexpr int h = decltype(hh)::value;
                const float2 z = cmul(make_float2(er[p][h], ei[p][h]), w);
                er[p][h] = z.x;
                ei[p][h] = z.y;
              });
            }
            // (keeps the operands of later residues out of the registers)
            if constexpr (RX >= 8) __builtin_amdgcn_sched_barrier(0);
          });
          // RX-point DFT over the residues, for each of the lane's four IFs
          float2 x[4][RX];
          static_for<0, 4>([&](auto q) {
            constexpr int h = decltype(q)::value;
            static_for<0, RX>([&](auto pi) { x[h][decltype(pi)::value] = make_float2(er[decltype(pi)::value][h], ei[decltype(pi)::value][h]); });
            dft<RX>(x[h]);
          });
          static_for<0, RX>([&](auto ki) {
            constexpr int kx = decltype(ki)::value;
            const float re[4] = {x[0][kx].x, x[1][kx].x, x[2][kx].x, x[3][kx].x};
            const float im[4] = {x[0][kx].y, x[1][kx].y, x[2][kx].y, x[3][kx].y};
            xa[cc * RX + kx][nt] = pack(re, im);
            float z = nt == 0 ? 0.f : z2[kx];
            static_for<0, 4>([&](auto q) {
              constexpr int h = decltype(q)::value;
              z = fmaf(re[h], re[h], fmaf(im[h], im[h], z));
            });
            z2[kx] = z;
          });
          // (one row tile's products and DFTs at a time: both together do not fit the registers)
          if constexpr (RX >= 8) __builtin_amdgcn_sched_barrier(0);
        });
        static_for<0, RX>([&](auto ki) { x2 = fmaxf(x2, z2[decltype(ki)::value]); });
      });
      // MBD of the units, 16 columns at a time: the products of a step (one
      // unit, 16 columns) are issued among the powers of the step before
      float mx[U];
      static_for<0, U>([&](auto ui) { mx[decltype(ui)::value] = 0.f; });
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
          constexpr int h = decltype(q)::value;
          v[h] = fmaf(o[1][h], o[1][h], o[0][h] * o[0][h]);
          if constexpr (HALF) {
            v[h] = fmaf(o[3][h], o[3][h], fmaf(o[2][h], o[2][h], v[h]));
            v[h] = fmaf(2.f, fabsf(fmaf(o[1][h], o[3][h], o[0][h] * o[2][h])), v[h]);
          }
        });
        m = fmaxf(fmaxf(m, v[0]), v[1]);
        m = fmaxf(fmaxf(m, v[2]), v[3]);
      };
      product(Index<0>{}, b, acc[0]);
#pragma unroll 1
      for (int ct = 0; ct < MT; ++ct) {
        operand(ct + 1 < MT ? ct + 1 : 0, bn);
        static_for<0, U>([&](auto ui) {
          constexpr int u = decltype(ui)::value, un = (u + 1) % U;
          product(Index<un>{}, un == 0 ? bn : b, acc[(u + 1) & 1]);
          powers(acc[u & 1], mx[u]);
          static_for<0, (HALF ? 4 : 2 * NK)>([&](auto) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                            // one MFMA,
            __builtin_amdgcn_sched_group_barrier(0x002, HALF ? 8 : NK == 2 ? 3 : 5, 0);   // its share of the powers
          });
        });
        static_for<0, 2 * NK>([&](auto i) {
          constexpr int q = decltype(i)::value;
          b[q / 2][q % 2] = bn[q / 2][q % 2];
        });
      }
      if constexpr (QUADS) {
        // a lane's powers are of the quad g of the unit; U divides 16
        unsigned part = 0u;
        static_for<0, U>([&](auto ui) {
          constexpr int u = decltype(ui)::value;
          const unsigned m = row_max16(mx[u]);
          part = row == ((c0 * RX + u) & 15) ? m : part;
        });
        static_for<0, 4>([&](auto k) {
          if ((c0 * RX) >> 4 == decltype(k)::value) keep[decltype(k)::value] = max(keep[decltype(k)::value], part);
        });
      } else {
        static_for<0, U>([&](auto ui) {
          constexpr int u = decltype(ui)::value;
          const unsigned m = __float_as_uint(wave_max(mx[u]));
          keep[0] = lane == c0 * RX + u ? m : keep[0];
        });
      }
    }
    // |screened G - G| <= eps_y (sum |y| + rounding of the sums) + eps_x sqrt(N) max_s |X(s)|_2 + ...
    x2 = fmaxf(x2, __shfl_xor(x2, 1, 64));
    x2 = fmaxf(x2, __shfl_xor(x2, 2, 64));
    x2 = fmaxf(x2, __shfl_xor(x2, 4, 64));
    x2 = fmaxf(x2, __shfl_xor(x2, 8, 64));
    x2 += __shfl_xor(x2, 16, 64);
    x2 += __shfl_xor(x2, 32, 64);
    const float bound = a.eps_y * s1p * sc + a.eps_x * sqrtf(x2 * float(N)) + a.abs_scaled + a.abs_plain * sc;
    // the record: a quad with screened maximum u has |G| <= gamma (u + bound);
    // it counts where that reaches A - bound, below the segment's largest |G|
    unsigned most = keep[0];
    if constexpr (QUADS) most = max(max(keep[0], keep[1]), max(keep[2], keep[3]));
    const float A = sqrtf(wave_max(__uint_as_float(most)));
    const float width = A + bound - (A - bound) / a.gamma;
    if (lane == 0) *reinterpret_cast<float2 *>(rec) = make_float2(a.gamma * (A + bound) / sc, a.gamma * width / (254.f * sc));
    auto mark = [&](unsigned v) {
      const float d = (A - sqrtf(__uint_as_float(v))) * (254.f / width);
      return d <= 254.f ? 1u + unsigned(d) : 0u;
    };
    if constexpr (QUADS) {
      static_for<0, 4>([&](auto k) {
        constexpr int kk = decltype(k)::value;
        if (16 * kk + row < units) rec[8 + 4 * (16 * kk + row) + g] = (unsigned char)mark(keep[kk]);
      });
    } else {
      if (lane < units) reinterpret_cast<unsigned *>(rec + 8)[lane] = mark(keep[0]) * 0x01010101u;
    }
  }
}

constexpr size_t kScreenLdsMax = 156 * 1024;

// The ring form: 64 channels or more and at least four rates.
bool screen_ring(int n_chan, int n_rate) { return n_chan >= 64 && n_rate >= 4; }

size_t screen_lds(int n_chan, int n_if, int n_rate, bool half, int tiles, int units) {
  const int nk = n_if <= 16 ? 1 : 2;
  size_t ring = 0, sbd = size_t(units);
  size_t tw = 0;
  if (screen_ring(n_chan, n_rate)) {
    ring = kRing * (n_chan == 64 ? (nk == 1 ? Slab<64, 1>::STRIDE : Slab<64, 2>::STRIDE)
                    : n_chan == 128 ? (nk == 1 ? Slab<128, 1>::STRIDE : Slab<128, 2>::STRIDE)
                                    : Slab<256, 1>::STRIDE);
    if (n_chan == 256) {
      sbd = size_t(units) / 16;
      tw = size_t(units) * 16 * sizeof(float2);
    }
  }
  return ring + (size_t(half ? 8 : tiles) * nk + sbd) * 2 * 64 * sizeof(h8_t) + tw;
}

// f(kernel) for the instantiation of a shape
template <int J, bool RING, typename F>
hipError_t with_kernel_j(int n_if, bool half, F &&f) {
  if (n_if <= 16) return f(&screen_kernel<J, 1, false, RING>);
  if constexpr (J <= 128) return half ? f(&screen_kernel<J, 2, true, RING>) : f(&screen_kernel<J, 2, false, RING>);
  return hipErrorInvalidValue;
}

template <typename F>
hipError_t with_kernel(int n_chan, int n_if, int n_rate, bool half, F &&f) {
  const bool ring = screen_ring(n_chan, n_rate);
  switch (n_chan) {
    case 16: return with_kernel_j<16, false>(n_if, half, f);
    case 32: return with_kernel_j<32, false>(n_if, half, f);
    case 64: return ring ? with_kernel_j<64, true>(n_if, half, f) : with_kernel_j<64, false>(n_if, half, f);
    case 128: return ring ? with_kernel_j<128, true>(n_if, half, f) : with_kernel_j<128, false>(n_if, half, f);
    case 256: return ring ? with_kernel_j<256, true>(n_if, half, f) : with_kernel_j<256, false>(n_if, half, f);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

bool screen_supported(int n_chan, int n_mbd, int n_if, int n_rate, bool half, int tiles, int sbd_pad) {
  if (n_mbd != 256 || n_if < 1 || n_if > (n_chan == 256 ? 16 : 32)) return false;
  if (n_chan != 16 && n_chan != 32 && n_chan != 64 && n_chan != 128 && n_chan != 256) return false;
  const int units = sbd_pad * n_chan / 16;
  return units >= 4 && units <= kScreenUnitsMax && screen_lds(n_chan, n_if, n_rate, half, tiles, units) <= kScreenLdsMax;
}

hipError_t screen_blocks(int n_chan, int n_if, int n_rate, bool half, int tiles, int sbd_pad, int device, int *blocks) {
  const size_t lds = screen_lds(n_chan, n_if, n_rate, half, tiles, sbd_pad * n_chan / 16);
  (void)hipGetLastError();
  return with_kernel(n_chan, n_if, n_rate, half, [&](auto kern) -> hipError_t {
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
      !a.f_sbd || !a.f_mbd || !a.tw_sbd || a.n_rate < 1 || (a.half && a.n_if <= 16) ||
      a.tiles < 1 || a.tiles > 16 || !(a.gamma >= 1.f))
    return hipErrorInvalidValue;
  const size_t lds = screen_lds(n_chan, a.n_if, a.n_rate, a.half != 0, a.tiles, a.units);
  if (lds > kScreenLdsMax) return hipErrorInvalidValue;
  const int need = (a.n_task + kScreenWaves - 1) / kScreenWaves;
  (void)hipGetLastError();
  return with_kernel(n_chan, a.n_if, a.n_rate, a.half != 0, [&](auto kern) -> hipError_t {
    hipLaunchKernelGGL(kern, dim3(std::min(blocks, need)), dim3(kScreenBlock), lds, s, a);
    return hipGetLastError();
  });
}

}  // namespace frbx
