// int_cells_kernel.hip -- QUASAR reconstruction for INT-b groups on gfx950,
// the binned form: each weight is placed once among the code thresholds of
// all candidates, and every candidate's moments come from per-group cell sums.
//
// Algorithm 1 (Sec. 4.1.2) needs, for every clip factor f_k, the weighted
// moments sum h q, sum h q^2 and sum h q w of the RTN codes q = q_k(u)
// (Eq. rtn) of the group's normalised positions u.  Each q_k is a
// non-decreasing step function of u:
//   q_k(u) = q0 + #{b in 1..NB : u >= T(k, b)},
// with q0 = 0 and NB = qmax for asymmetric groups, q0 = -Q and NB = 2Q for
// symmetric ones, and T(k, b) the least fp32 u whose code under clip k is at
// least q0 + b.  The host finds every T(k, b) exactly, for the kernels' own fp32
// code recipe, from one fp64 quotient and its neighbours, and sorts the
// distinct ones, t_0 < ... < t_{M-1}.  The cell of u is #{i : t_i <= u} in
// [0, M]; all K codes of a weight are fixed by its cell.  With
// P_b = sum of h over the weights with u >= T(k, b) (a suffix sum over cells)
// and PW_b the same sum of h w, and n = q - q0:
//   sum h n = sum_b P_b,   sum h n^2 = sum_b (2b - 1) P_b,   sum h n w = sum_b PW_b.
// So the per-weight work no longer grows with the number of clips: one
// bucket lookup and two LDS additions per weight replace K code evaluations
// and 3K moment updates.
//
// Per weight: u; its bucket among 512 slices of [-1, 1] (the host table gives
// the cell at the bucket's lower edge and the one threshold inside it; grids
// whose thresholds lie closer take 256 slices and up to three compares), its
// cell, then h and h w added into the group's cell as exact int64 values
// (LDS atomics).  A group's lanes are spread over the wavefront (8 apart), so
// members of one group that hit the same cell do not serialise the atomic.
// Per group: suffix sums over the cells, in place and in integers (each of
// the L lanes takes a chunk into registers; the chunk totals are combined
// across lanes with DPP and permlane swaps), then each lane assembles the
// moments of the clips it owns from NB suffix sums each and solves and scores
// them exactly as the direct form does (int_common.h).
//
// What bounds it: on the Llama-3.1-8B layer set (INT2 g64, 12 clips, EMA, 14.4
// bytes per weight) a launch moves 5.0 TB/s, about a plain copy's rate, with
// the VALU busy 72% and the LDS 60% of the time (SQ_ACTIVE_INST_VALU and
// SQ_LDS_IDX_ACTIVE over the compute units' cycles).  Measured steps, all
// on that set: fp64 suffix sums, rounded cell by cell in two passes over the
// LDS, and binning and atomics as two loops: 688 us; in integers, one pass in
// registers, one loop, one compare per weight: 643; the fit's tests once per
// group instead of once per clip: 635; h and h w swapped in odd cells: 634; the staged
// stores non-temporal: 624 (Qwen3-0.6B set, INT3 with 8 clips: 48.9, 42.0, 41.8,
// 41.2, 39.9).
// Forms.  Both sums in a cell (16 bytes) keep four workgroups on a compute
// unit up to 8 cells a lane and three at 9 and 10 (46.5 KB of LDS).  At 12 and
// more they would leave two: the SPLIT form takes h and then h w through
// 8-byte cells (each weight's cell is kept, one byte), and keeps four.  INT3
// g128 with 15 clips (91 cells), the Llama set: 709 us; both sums at once 1018;
// the direct kernel 1172.  At g64 SPLIT meets the 128 VGPRs of four wavefronts
// and spills 1 with the EMA on fp32 W, 2 to 10 with the AdamW step; from
// int_split_least's sizes on it is still 2 to 19% faster than the direct kernel there
// (INT3, 9 and 10 clips, fp32 W, AdamW).  A form with 8 weights per
// lane (half the groups per wavefront, so half the LDS) took 750 us there,
// and 59 against 45 us on the Qwen3-0.6B set (INT3, 8 clips): its per-group
// work is spread over twice the wavefronts.
// The emitted codes are recomputed from u with the fp32 recipe, so they are
// bit-identical to the direct form's.
#include <type_traits>

#include "device_common.h"
#include "int_common.h"
#include "quasar_internal.h"

namespace quasar {
namespace {

constexpr int N = kIntN;

// Lanes of one group: spread over the wavefront (member j of a group 8 lanes
// from member j - 1), so that LDS atomics from members of one group that hit
// the same address do not serialise.
constexpr bool kSpread = true;

typedef unsigned long long u64;

// x of the lane that DPP control CTRL names (0 where it names none)
template <int CTRL>
__device__ __forceinline__ u64 dpp_u64(u64 x) {
  return ((u64)dpp_u32<CTRL>((uint32_t)(x >> 32)) << 32) | dpp_u32<CTRL>((uint32_t)x);
}

// The value x of the lane in the paired row (ROWS = 16: rows 0 <-> 1, 2 <-> 3)
// or half (ROWS = 32), at the same position, for a lane in an even row (the
// lower half) when `low` is set: the swap leaves the even rows' values in its
// first result and the odd rows' in its second.
template <int ROWS>
__device__ __forceinline__ u64 paired(u64 x, bool low) {
  uint32_t alo, blo, ahi, bhi;
  swap_rows<ROWS>((uint32_t)x, alo, blo);
  swap_rows<ROWS>((uint32_t)(x >> 32), ahi, bhi);
  return low ? ((u64)bhi << 32) | blo : ((u64)ahi << 32) | alo;
}

// Exclusive suffix sum over the members of a group: member j gets the sum of
// the values of members j+1 .. L-1 (integers: exact).  Members 2i and 2i+1
// share a row of 16 (8 lanes apart), so member j's suffix is its row partner's
// value (j even) plus the totals of the later rows, exchanged between rows and
// halves without LDS.
template <int L>
__device__ __forceinline__ u64 members_excl_suffix(u64 x, int j) {
  static_assert(kSpread, "members 8 lanes apart");
  const u64 nb = dpp_u64<kDppRor8>(x);  // member j ^ 1
  u64 e = (j & 1) ? 0ull : nb;
  const u64 r = x + nb;                 // this row's two members
  const int row = j >> 1;               // the group's rows in order
  const u64 t = paired<16>(r, (row & 1) == 0);
  if constexpr (L == 4) {
    e += row == 0 ? t : 0ull;
  } else {
    const u64 o = paired<32>(r + t, row < 2);  // the other half's four members
    e += ((row & 1) ? 0ull : t) + (row < 2 ? o : 0ull);
  }
  return e;
}

// x * scale rounded to an integer (ties to even), as int64, for
// |x * scale| < 2^51: x * scale + 1.5 2^52 (one fma, one rounding) lies in
// [2^52, 2^53), where its bit pattern is that of 1.5 2^52 plus the integer,
// and the low word of 1.5 2^52 is zero.
constexpr double kMagic = 6755399441055744.0;  // 1.5 * 2^52
constexpr uint32_t kMagicHi = 0x43380000u;
__device__ __forceinline__ u64 scaled_to_i64(double x, double scale) {
  const u64 b = (u64)__double_as_longlong(__builtin_fma(x, scale, kMagic));
  return ((u64)((uint32_t)(b >> 32) - kMagicHi) << 32) | (uint32_t)b;
}
// ... and back, correctly rounded: the high word exactly times 2^32 plus the
// low word, one rounding
__device__ __forceinline__ double i64_to_double(u64 n) {
  return __builtin_fma((double)(int32_t)(uint32_t)(n >> 32), 4294967296.0, (double)(uint32_t)n);
}
__device__ __forceinline__ double u64_to_double(u64 n) {
  return __builtin_fma((double)(uint32_t)(n >> 32), 4294967296.0, (double)(uint32_t)n);
}

// SPLIT: a cell holds one int64, and the two sums are taken one after the
// other in the same LDS (h, then h w); otherwise a cell holds both.
template <bool W_BF16, int EMA, int BITS, int G, bool SYM, bool SPLIT>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4))) void int_cells_kernel(IntParams p) {
  constexpr int L = G / N;     // lanes per group
  constexpr int GPW = 64 / L;  // groups per wavefront
  constexpr int QMAX = SYM ? (1 << (BITS - 1)) - 1 : (1 << BITS) - 1;
  constexpr int NB = SYM ? 2 * QMAX : QMAX;  // code steps per clip
  constexpr int OWN = kMaxClips / L;         // clips a lane may own
  constexpr int CELL = SPLIT ? 8 : 16;       // bytes
  static_assert(2 * kThreads == kIntBuckets && kThreads == kCellBuckets && kThreads == kMaxClips * kCellSteps, "table entries per thread");
  static_assert((size_t)int_stage_bytes<kSpread, G>() == int_cells_stage_bytes(G), "the launch sizes the stage");

  extern __shared__ __align__(16) u64 s_hist[];  // [wave][group slot][cell]{h, h w}, or the store stage
  // one compare: 512 entries {threshold, cell offset}; more: 256 entries
  // {cell offset, three thresholds}
  __shared__ __align__(16) uint4 s_bucket[kThreads];
  __shared__ __align__(16) uint8_t s_tp[kMaxClips * kCellSteps];
  __shared__ float s_alpha[kMaxClips], s_clip[kMaxClips];
  __shared__ float s_win[kThreads / 64][GPW][4];

  using M = Members<L, kSpread>;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = wave_index();
  const int j = M::member(lane), slot = M::slot(lane);
  const int K = p.n_clips;
  const int cmax = p.cells.cmax;

  // Byte offset of cell c's sum of h in its group.  With both sums in a cell,
  // odd cells hold h w first: the atomics on h then use all LDS banks and not
  // the even pairs only (and those on h w, 8 bytes to the other side, as well).
  auto h_offset = [&](int c) { return SPLIT ? (uint32_t)c * 8u : (uint32_t)c * 16u + (uint32_t)(c & 1) * 8u; };
  {  // the tables, read from the kernel-argument segment with per-lane indices
    const IntCells& cl = kernarg_params<IntParams>()->cells;
    if (cmax == 1) {
      const int c0 = cl.base[2 * tid], c1 = cl.base[2 * tid + 1];
      s_bucket[tid] = make_uint4(as_u32(cl.thr[c0]), h_offset(c0) | h_offset(c0 + 1) << 16, as_u32(cl.thr[c1]),
                                 h_offset(c1) | h_offset(c1 + 1) << 16);
    } else {
      const int c = cl.base[tid];
      s_bucket[tid] = make_uint4((uint32_t)c, as_u32(cl.thr[c]), as_u32(cl.thr[c + 1]), as_u32(cl.thr[c + 2]));
    }
    s_tp[tid] = (&cl.tp[0][0])[tid];
  }
  if (tid < kMaxClips) {
    s_alpha[tid] = p.alpha[tid];
    s_clip[tid] = p.clip[tid];
  }
  __syncthreads();

  int64_t blk = blockIdx.x;
  const IntMatrix mtx = int_matrix(p, blk);
  const int64_t wave_g0 = (blk * (kThreads / 64) + wave) * GPW;
  int64_t gid = wave_g0 + slot;
  const bool active = gid < mtx.n_groups;
  if (!active) gid = mtx.n_groups - 1;  // recompute the last group; nothing is stored
  const int64_t e0 = gid * G + (int64_t)j * N;

  // this wavefront's LDS: its groups' cells, before that the stage of the
  // EMA's store, and after them the stage of the exact path and of r's store
  const int cpl = p.cells.cpl;
  const int wave_bytes = (int)int_cells_wave_bytes(G, SPLIT, cpl);
  u64* const s_wave = s_hist + wave * (wave_bytes / 8);
  const WaveImage im = int_image<L>(s_wave, wave_g0, mtx.n_groups, slot, j, lane, p.store);

  WRegs<W_BF16> wr;
  float v[N];
  int_load<W_BF16, EMA, kSpread, G>(p, mtx, im, e0, wr, v);
  const IntRange rg = int_range<L, SYM, W_BF16, kSpread>(wr);

  // ---- this group's cells: lane j owns cells [j cpl, (j + 1) cpl) -----------
  // Groups are int_cells_stride(L, cpl) cells apart, an odd number, so that the
  // same cell of the wavefront's groups falls in different LDS banks.
  const int stride = int_cells_stride(L, cpl);
  u64* const hist = s_wave + slot * (stride * (CELL / 8));
  // clear the wavefront's whole area, 16 bytes per lane and step
  auto clear = [&]() {
    const int n16 = (GPW * stride * CELL + 15) / 16;
    uint4* z = reinterpret_cast<uint4*>(s_wave);
#pragma unroll 1
    for (int i = lane; i < n16; i += 64) z[i] = make_uint4(0u, 0u, 0u, 0u);
  };
  clear();

  // ---- h and h w of every weight into its cell, as exact integers --------------
  // h and h w are scaled by powers of two that bring the group's largest |h|
  // and |h| max|w| below 2^B, B = 51, rounded to integers and added as int64:
  // every cell sum is exact (below 2^58), whatever the order of the atomics,
  // and so is every sum over cells; a clip's moments are rounded once each to
  // fp64.  Clips whose codes agree on the whole group get bit-identical
  // moments, so their scores tie exactly and the lowest index wins, as in the
  // exact definition.  A term loses at most 2^-52 of the largest one; the fit
  // below checks what that can do to it.
  constexpr int B = 51;
  float hmax = 0.0f;
#pragma unroll
  for (int i = 0; i < N; i++) hmax = fmaxf(hmax, v[i]);
  hmax = M::max(hmax);
  const float wabs = SYM ? rg.mx : fmaxf(fabsf(rg.mn), fabsf(rg.mx));
  // 2^eh > hmax and 2^ew > max |w| (frexp exponents)
  const int eh = __builtin_amdgcn_frexp_expf(hmax), ew = __builtin_amdgcn_frexp_expf(wabs);
  const double sh = __builtin_amdgcn_ldexp(1.0, B - eh), shw = __builtin_amdgcn_ldexp(1.0, B - eh - ew);
  double Svww = 0.0;
  wave_lds_fence();  // the cells are clear

  auto add = [&](u64* c, u64 x) {
    __hip_atomic_fetch_add(c, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
  };
  // the cell at byte offset `off` of this group
  auto cell_at = [&](uint32_t off) { return reinterpret_cast<u64*>(reinterpret_cast<char*>(hist) + off); };

  // The cell of a weight: its bucket's first cell plus up to cmax compares
  // (IntCells).  Thresholds outside u's bucket lie on the far side of u and
  // the table's padding is NaN, so the compares never pass the last threshold.
  // Four weights at a time, and their bucket entries are read while the four
  // before them are added into their cells.  SPLIT: only h is added, and the
  // cells' offsets (one byte each, in units of 8) are kept for h w.
  uint32_t cells[SPLIT ? N / 4 : 1];
  auto fill = [&](auto cmax_tag) {
    constexpr int C = decltype(cmax_tag)::value;
    float w[4], u[4];
    typename std::conditional<C == 1, uint2, uint4>::type e[4];
    auto fetch = [&](int i0) {
#pragma unroll
      for (int t = 0; t < 4; t++) {
        w[t] = wr.get(i0 + t);
        u[t] = int_u<SYM>(w[t], rg);
        if constexpr (C == 1)
          e[t] = reinterpret_cast<const uint2*>(s_bucket)[cell_bucket512(u[t], p.cells.shift)];
        else
          e[t] = s_bucket[cell_bucket(u[t])];
      }
    };
    fetch(0);
#pragma unroll
    for (int i0 = 0; i0 < N; i0 += 4) {
      uint32_t off[4];
      float x[4];
#pragma unroll
      for (int t = 0; t < 4; t++) {
        if constexpr (C == 1) {
          off[t] = __builtin_amdgcn_ubfe(e[t].y, u[t] >= as_f32(e[t].x) ? 16u : 0u, 16u);
        } else {
          uint32_t c = e[t].x + (u[t] >= as_f32(e[t].y) ? 1u : 0u) + (u[t] >= as_f32(e[t].z) ? 1u : 0u);
          if constexpr (C > 2) c += (u[t] >= as_f32(e[t].w) ? 1u : 0u);
          off[t] = h_offset((int)c);
        }
        x[t] = w[t];
      }
      if (i0 + 4 < N) fetch(i0 + 4);
#pragma unroll
      for (int t = 0; t < 4; t++) {
        // opaque: the conversions are the same in every copy of this loop, and
        // would otherwise be made for all N weights before the branch on cmax
        float vi = v[i0 + t];
        asm volatile("" : "+v"(vi));
        const double V = (double)vi;
        add(cell_at(off[t]), scaled_to_i64(V, sh));
        if constexpr (!SPLIT) {
          const double Wd = (double)x[t];
          const double VW = V * Wd;
          Svww = __builtin_fma(VW, Wd, Svww);
          add(cell_at(off[t] ^ 8u), scaled_to_i64(VW, shw));
        }
      }
      if constexpr (SPLIT) {
        static_assert(CELL == 8, "offsets in units of 8 fit a byte each");
        cells[i0 / 4] = (off[0] >> 3) | (off[1] << 5) | (off[2] << 13) | (off[3] << 21);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  if (cmax == 1)
    fill(std::integral_constant<int, 1>{});
  else if (cmax == 2)
    fill(std::integral_constant<int, 2>{});
  else
    fill(std::integral_constant<int, 3>{});
  wave_lds_fence();

  // A weight among merged thresholds (rare) lies in the unsafe cell, where the
  // cell does not fix every clip's code: its group takes the exact path below
  // unless its saliency is 0 (h >= 0, so the cell's sum of h is 0 exactly when
  // every weight in it has h = 0, and those weights add nothing to any moment).
  const int ucell = p.cells.unsafe_cell;
  const bool group_unsafe = ucell >= 0 && *cell_at(h_offset(ucell)) != 0;
  wave_lds_fence();  // read before the sums are taken in place

  // ---- suffix sums over the cells, in place and in integers: the lane's
  // cells are read into registers (a compile-time count, the host rounds cpl
  // up to it; the cells past the last threshold are zero), summed from the
  // top down, and the total of the members above this one added.  The suffix
  // sums are written h first in every cell.
  auto suffix = [&](auto cpl_tag) {
    constexpr int C = decltype(cpl_tag)::value;
    if constexpr (SPLIT) {
      u64* mc = hist + j * C;
      u64 t[C];
#pragma unroll
      for (int c = 0; c < C; c++) t[c] = mc[c];
#pragma unroll
      for (int c = C - 2; c >= 0; c--) t[c] += t[c + 1];
      const u64 x = members_excl_suffix<L>(t[0], j);
#pragma unroll
      for (int c = 0; c < C; c++) mc[c] = t[c] + x;
    } else {
      ulonglong2* mc = reinterpret_cast<ulonglong2*>(hist) + j * C;
      ulonglong2 t[C];
#pragma unroll
      for (int c = 0; c < C; c++) {  // C is even, so c's parity is the cell's
        t[c] = mc[c];
        if (c & 1) t[c] = make_ulonglong2(t[c].y, t[c].x);
      }
#pragma unroll
      for (int c = C - 2; c >= 0; c--) {
        t[c].x += t[c + 1].x;
        t[c].y += t[c + 1].y;
      }
      const u64 xh = members_excl_suffix<L>(t[0].x, j), xw = members_excl_suffix<L>(t[0].y, j);
#pragma unroll
      for (int c = 0; c < C; c++) mc[c] = make_ulonglong2(t[c].x + xh, t[c].y + xw);
    }
  };
  auto suffix_sums = [&]() {
    if constexpr (SPLIT) {
      if (cpl <= 12)
        suffix(std::integral_constant<int, 12>{});
      else if (cpl == 14)
        suffix(std::integral_constant<int, 14>{});
      else
        suffix(std::integral_constant<int, 16>{});
    } else {
      if (cpl == 2)
        suffix(std::integral_constant<int, 2>{});
      else if (cpl == 4)
        suffix(std::integral_constant<int, 4>{});
      else if (cpl == 6)
        suffix(std::integral_constant<int, 6>{});
      else if (cpl == 8)
        suffix(std::integral_constant<int, 8>{});
      else
        suffix(std::integral_constant<int, 10>{});
    }
    wave_lds_fence();
  };
  suffix_sums();

  // ---- the clips this lane owns, k = j + L t: moments from NB suffix sums, in
  // integers.  From the highest step down, R is the sum of the P_b so far and
  // S the sum of the R: sum_b b P_b, so sum_b (2b - 1) P_b = 2 S - R.  P_b <=
  // 2^58, so 7 steps keep S below 2^63; with 14 or 15 steps the upper ones are
  // summed on their own: sum_{b > 8} b P_b = S_hi + 8 R_hi.
  double A0[OWN], A1[OWN], A2[OWN];
  auto steps = [&](int k, auto&& f) {  // f(b, cell) for b = NB .. 1
    const uint4 tw4 = *reinterpret_cast<const uint4*>(s_tp + k * kCellSteps);
    const uint32_t tw[4] = {tw4.x, tw4.y, tw4.z, tw4.w};
#pragma unroll
    for (int b = NB; b >= 1; b--) f(b, (int)((tw[(b - 1) >> 2] >> (8 * ((b - 1) & 3))) & 0xffu));
  };
  u64 tot_h, tot_w;  // the whole group's sums: cell 0's suffix
#pragma unroll
  for (int t = 0; t < OWN; t++) {
    A0[t] = A1[t] = A2[t] = 0.0;
    const int k = j + L * t;
    if (k < K) {
      u64 R = 0, S = 0, Q = 0, Rhi = 0, Shi = 0;
      steps(k, [&](int b, int c) {
        if constexpr (SPLIT) {
          R += hist[c];
        } else {
          const ulonglong2 s = reinterpret_cast<const ulonglong2*>(hist)[c];
          R += s.x;
          Q += s.y;
        }
        S += R;
        if (b == 9) {
          Rhi = R;
          Shi = S;
          R = S = 0;
        }
      });
      A0[t] = u64_to_double(R);
      A1[t] = __builtin_fma(2.0, u64_to_double(S), -A0[t]);
      if constexpr (NB > 8) {
        const double rh = u64_to_double(Rhi);
        A1[t] += __builtin_fma(2.0, u64_to_double(Shi), 15.0 * rh);
        A0[t] += rh;
      }
      A2[t] = i64_to_double(Q);
    }
  }
  tot_h = hist[0];
  if constexpr (!SPLIT) {
    tot_w = hist[1];
  } else {
    // h w through the same cells
    wave_lds_fence();
    clear();
    wave_lds_fence();
#pragma unroll
    for (int i = 0; i < N; i++) {
      const double V = (double)v[i], Wd = (double)wr.get(i);
      const double VW = V * Wd;
      Svww = __builtin_fma(VW, Wd, Svww);
      add(hist + ((cells[i / 4] >> (8 * (i & 3))) & 0xffu), scaled_to_i64(VW, shw));
      if (i % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    }
    wave_lds_fence();
    suffix_sums();
#pragma unroll
    for (int t = 0; t < OWN; t++) {
      const int k = j + L * t;
      if (k < K) {
        u64 Q = 0;
        steps(k, [&](int, int c) { Q += hist[c]; });
        A2[t] = i64_to_double(Q);
      }
    }
    tot_w = hist[0];
  }

  // back from the integer scale (exact: powers of two)
  const double rsh = __builtin_amdgcn_ldexp(1.0, eh - B), rshw = __builtin_amdgcn_ldexp(1.0, eh + ew - B);
  IntMoments mo;
  mo.Sv = u64_to_double(tot_h) * rsh;
  mo.Svw = i64_to_double(tot_w) * rshw;
  mo.Svww = M::sum(Svww);
  mo.thr = 1e-12 * mo.Sv * mo.Sv * (double)QMAX * (double)QMAX;
  mo.rSv = rcp_f64(mo.Sv);
  // each term of sum h and of sum h w is off by at most half a unit of its
  // fixed point; the moments and the fit's products carry fp64 roundings
  mo.qh = 0.5 * (double)G * rsh;
  mo.qhw = 0.5 * (double)G * rshw;
  mo.rel = 0x1p-47;
  mo.wabs = (double)wabs;
  int_fit_bounds<QMAX>(mo);
#pragma unroll
  for (int t = 0; t < OWN; t++) {
    A0[t] *= rsh;
    A1[t] *= rsh;
    A2[t] *= rshw;
    if constexpr (SYM) {  // q = n - Q
      A1[t] = __builtin_fma((double)QMAX * (double)QMAX, mo.Sv, __builtin_fma(-2.0 * (double)QMAX, A0[t], A1[t]));
      A2[t] = __builtin_fma(-(double)QMAX, mo.Svw, A2[t]);
    }
  }

  // Selection.  With fp32 (s, z) the candidate's score is that of its exact
  // fit up to the fp32 rounding of (s, z), a relative 1e-12 or so; the exact
  // fit's score is C - num^2 / (Sv D) (asymmetric: num = Sv A2 - A0 Svw,
  // D = Sv A1 - A0^2; symmetric: C - A2^2 / A1), with C the same for every
  // clip.  So each lane ranks its clips by num^2 / D (cross-multiplied, ties
  // to the lowest index), fits and scores only its best one, and the group's
  // argmin runs over keys made from D / num^2.
  // Groups with a clip whose fit degenerates (no saliency, all of it on one
  // code), and deployed precisions other than fp32, score every clip
  // (int_fit_score).  A group with a clip whose fit the moments cannot fix
  // accurately enough (int_fit_ill), or with a weight among merged
  // thresholds, evaluates every clip straight from its weights
  // (int_exact_wave).
  //
  // The tests that find such groups cost more per clip than the ranking.  So
  // the ranking only keeps the least D and |num| of its clips, and one bound
  // per group over all possible codes (A0 <= Q Sv, A1 <= Q^2 Sv) tells
  // whether any clip could fail a test; the tests run, clip by clip, only for
  // the groups it cannot clear (about one in a thousand).
  IntBest best = int_best_init();
  bool full = p.param_dtype != 0;
  bool ill = group_unsafe;
  int bk = -1;
  double bn = 0.0, bd = 1.0, b0 = 0.0, b1 = 0.0, b2 = 0.0;
  if (!full && !group_unsafe) {
    constexpr double Q = (double)QMAX;
    double dmin = 1e300, nmin = 1e300;
    // unrolled: the clips' fp64 chains interleave
#pragma unroll
    for (int t = 0; t < OWN; t++) {
      const int k = j + L * t;
      if (k < K) {
        const double D = SYM ? A1[t] : __builtin_fma(mo.Sv, A1[t], -(A0[t] * A0[t]));
        const double num = SYM ? A2[t] : __builtin_fma(mo.Sv, A2[t], -(A0[t] * mo.Svw));
        dmin = min_key(dmin, D);
        nmin = min_key(nmin, fabs(num));
        const double n2 = num * num;
        if (t == 0 || n2 * bd > bn * D) {
          bk = k;
          bn = n2;
          bd = D;
          b0 = A0[t];
          b1 = A1[t];
          b2 = A2[t];
        }
      }
    }
    // int_fit_ill's error bounds at their largest (symmetric: its rel A1 is
    // far below kFitTol A1, the factor 2 covers it)
    const double eD = SYM ? 2.0 * mo.qh * Q * Q : __builtin_fma(2.0 * mo.rel * Q * Q, mo.Sv * mo.Sv, mo.eD0);
    const double eN = SYM ? (mo.qhw + mo.rel * mo.wabs * mo.Sv) * Q : __builtin_fma(mo.eN1 * Q, mo.Sv, mo.eN0);
    const bool clear = (eD <= kFitTol * dmin) & (eN <= kFitTol * nmin) & (SYM || dmin - eD > mo.thr);
    if (M::max(clear ? 0.0f : 1.0f) > 0.0f) {
      bool degenerate = false;
#pragma unroll
      for (int t = 0; t < OWN; t++) {
        if (j + L * t < K) {
          ill |= int_fit_ill<SYM, QMAX>(mo, A0[t], A1[t], A2[t]);
          degenerate |= SYM ? (A1[t] == 0.0) : (mo.Sv == 0.0 || mo.Sv * A1[t] - A0[t] * A0[t] <= mo.thr);
        }
      }
      ill = M::max(ill ? 1.0f : 0.0f) > 0.0f;
      full = M::max(degenerate ? 1.0f : 0.0f) > 0.0f;
    }
  }
  if (!ill) {
    if (full) {
#pragma unroll
      for (int t = 0; t < OWN; t++) {
        const int k = j + L * t;
        if (k < K) int_fit_score<SYM, QMAX>(p, k, s_clip[k], rg, mo, A0[t], A1[t], A2[t], best);
      }
      ill = M::max(best.ill ? 1.0f : 0.0f) > 0.0f;
    } else if (bk >= 0) {
      int_fit_score<SYM, QMAX>(p, bk, s_clip[bk], rg, mo, b0, b1, b2, best);
      // rank by D / num^2 (num = 0: the worst fit, kept finite)
      best.key = make_key(fmin(bd * rcp_f64(bn), 1e300), bk);
    }
  }
  {
    // The wavefront's cell areas are no longer needed: they stage the
    // flagged groups.  A member lane reads its saliencies again: v' when this
    // kernel stored it, written by another lane of this wavefront, which the
    // workgroup-scope fences make visible (the workgroup's waves share the
    // compute unit's vector cache).
    auto load_h = [&](float (&hv)[N]) {
      if constexpr (EMA != 0) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
      }
      load16<false>(mtx.v, e0, hv);
#pragma unroll
      for (int i = 0; i < N; i++) hv[i] = weight_of(hv[i], p.weighting);
    };
    int_exact_wave<L, SYM, QMAX, kSpread, W_BF16>(p, wr, load_h, rg, s_alpha, s_clip, lane,
                                                  ill && active && !rg.constant, reinterpret_cast<float*>(s_wave),
                                                  best);
  }

  int_finish<W_BF16, EMA, BITS, G, SYM, kSpread>(p, mtx, wr, rg, mo.Sv, best, s_alpha, s_win[wave][slot], j, gid, im,
                                         active);
}

template <bool W_BF16, int EMA, int BITS, int G, bool SPLIT>
hipError_t launch_s(const IntParams& p, hipStream_t s) {
  constexpr int64_t groups_per_block = int_units_per_block(G);
  const int64_t blocks =
      p.batch.n > 1 ? p.batch.total_blocks : (p.n_groups + groups_per_block - 1) / groups_per_block;
  const size_t lds = int_cells_lds_bytes(G, SPLIT, p.cells.cpl);
  const dim3 grid((unsigned)blocks), block(kThreads);
  if (p.symmetric) {
    if constexpr (EMA <= 2) {
      hipLaunchKernelGGL((int_cells_kernel<W_BF16, EMA, BITS, G, true, SPLIT>), grid, block, lds, s, p);
      return hipGetLastError();
    } else {
      return hipErrorInvalidValue;
    }
  }
  hipLaunchKernelGGL((int_cells_kernel<W_BF16, EMA, BITS, G, false, SPLIT>), grid, block, lds, s, p);
  return hipGetLastError();
}

// INT2: at most 3 thresholds a clip, the tie ones merged into two, 35 cells
static_assert(3 * kMaxClips - (kMaxClips - 2) + 1 <= 4 * int_cells_most(false), "INT2 grids take both sums at once");

template <bool W_BF16, int EMA, int BITS, int G>
hipError_t launch_g(const IntParams& p, hipStream_t s) {
  if constexpr (BITS > 2) {  // INT2 grids fit without
    if (p.cells.split) return launch_s<W_BF16, EMA, BITS, G, true>(p, s);
  }
  return launch_s<W_BF16, EMA, BITS, G, false>(p, s);
}

template <bool W_BF16, int EMA, int BITS>
hipError_t launch_b(const IntParams& p, int group, hipStream_t s) {
  return group == 64 ? launch_g<W_BF16, EMA, BITS, 64>(p, s) : launch_g<W_BF16, EMA, BITS, 128>(p, s);
}

template <bool W_BF16, int EMA>
hipError_t launch_e(const IntParams& p, int bits, int group, hipStream_t s) {
  switch (bits) {
    case 2: return launch_b<W_BF16, EMA, 2>(p, group, s);
    case 3: return launch_b<W_BF16, EMA, 3>(p, group, s);
    default: return launch_b<W_BF16, EMA, 4>(p, group, s);
  }
}

template <bool W_BF16>
hipError_t launch_w(const IntParams& p, int bits, int group, int ema_mode, hipStream_t s) {
  switch (ema_mode) {
    case 1: return launch_e<W_BF16, 1>(p, bits, group, s);
    case 2: return launch_e<W_BF16, 2>(p, bits, group, s);
    case 3: return launch_e<W_BF16, 3>(p, bits, group, s);
    case 4: return launch_e<W_BF16, 4>(p, bits, group, s);
    case 5: return launch_e<W_BF16, 5>(p, bits, group, s);
    case 6: return launch_e<W_BF16, 6>(p, bits, group, s);
    default: return launch_e<W_BF16, 0>(p, bits, group, s);
  }
}

}  // namespace

hipError_t launch_int_cells(const IntParams& p, int bits, int group, bool w_bf16, int ema_mode, hipStream_t s) {
  return w_bf16 ? launch_w<true>(p, bits, group, ema_mode, s) : launch_w<false>(p, bits, group, ema_mode, s);
}

}  // namespace quasar
