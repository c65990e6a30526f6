// rubin_kernel.hip -- QUASAR for the Rubin INT3 lookup-table format on gfx950
// (App. B, Eq. rubin-fit).
//
// A block is 8 rows x 64 columns (512 weights) with 3-bit indices and an
// 8-entry E4M3 codebook.  For every clip factor f the indices are the INT3
// codes of the range [c - f rho, c + f rho] (the same fp32 recipe as the
// affine kernel: u = fma(w, 1/rho, -c/rho), q = clamp(rint(fma(u, alpha_f, 3.5)))),
// each codebook entry is the saliency-weighted mean of the weights with that
// index rounded to E4M3, and the candidate is scored with Eq. fisher-obj; the
// lowest score is emitted.
//
// Every code is a non-decreasing function of u, so the codes a weight gets
// under all K clips are fixed by how many of the 7K per-clip thresholds
// T(k, b) = min{u : q_k(u) >= b + 1} lie at or below u.  That count -- the
// weight's cell, 0 .. 7K -- is what the kernel bins by, once per block (the
// host adds boundaries that are no threshold, splitting the cells that hold
// most of a block: the lanes of one LDS atomic that meet on a cell
// serialise, and no code changes inside a cell either way), and
// for clip k the weights with code b are exactly the cells in a fixed range
// [tpos(k, b), tpos(k, b + 1)).  The per-clip work then reads two prefix sums
// per codebook entry instead of re-binning 512 weights.  The thresholds are
// exact fp32 values found on the host.  A weight finds its cell either from
// a table over 256 equal slices of u plus at most three compares (BK, the
// bucket form, with the clips' tie thresholds just below u = 0 merged into
// one; a block with a weight between them sums its code-3 and code-4 entries
// directly) or by descending an implicit binary search tree over all of them
// (node n's children at 2n and 2n + 1; any clip grid).
//
// The cell sums of h and h w are kept as integers.  Each value is scaled by a
// power of two fixed per block (from the block's largest h and |w|), to x
// with |x| < 2^51, and split into hi = rint(x - 1) and lo = trunc((x - hi)
// 2^21), in [2^20, 3 2^20]: x = hi + lo 2^-21 whenever x is a
// multiple of 2^-21, else lo falls short by less than one unit.  Three 64-bit
// LDS atomics per weight add the high limbs of h and of h w and both low
// limbs, packed into the halves of one word (the sums of a half over a block
// stay below 2^31, so no carry crosses).  Integer addition is exact and
// order-independent, so the sums -- and everything computed from them -- are
// deterministic.  A codebook entry's sums are differences of two prefix sums,
// exact when every scaled value of the block is a multiple of 2^-21 (for h:
// when no saliency lies below 2^-49 of the block's largest) and within 2^-12
// units otherwise.  An entry whose h sum is below 2^18 units (about 2^-33 of
// the block's largest h) is recomputed directly in fp64, so every other
// entry's h sum is within 2^-30 relative; so is one whose weights all have a
// saliency that the fixed point lost to 0 (found from a per-cell flag, set by a
// weight with h > 0 whose value is 0).
//
// Work decomposition: one wavefront per block, lane l holding row l/8 of the
// block and its 8 consecutive columns 8 (l % 8) .. 8 (l % 8) + 7.  The
// per-clip phase runs 8 clips at a time, lane (k, b) = (l / 8, l % 8) owning
// codebook entry b of clip k.
//
// What bounds it: on the Llama-3.1-8B layer set (15 clips, EMA, 14.4 bytes per
// weight) 711 us, 4.4 TB/s, with the LDS busy 78% of the time (24 atomics per
// wavefront at random cells, 16 cycles each: about 400 of its 750 cycles) and
// the VALU 77%.  754 us before the limbs were split with
// three fmas (six instructions before), the argmin taken once over all clips,
// the tie and lost-saliency tests made by one unsigned minimum each, and the
// codes emitted as bytes that permute the codebook (no LDS lookup per weight),
// 718 before whole lines of W and g were loaded non-temporally.
#include <type_traits>

#include "device_common.h"
#include "quasar_internal.h"

namespace quasar {
namespace {

constexpr int NE = 8;          // weights per lane
constexpr int kWaves = kThreads / 64;
constexpr int kCells = kRubinThresholds;  // cell ids 0 .. (boundaries) <= 127 < 128
constexpr int kHiBits = 51;    // |scaled value| < 2^51: its nearest integer is the high limb
constexpr int kLoBits = 21;    // the low limb counts units of 2^-21
constexpr double kMagic = 6755399441055744.0;  // 1.5 * 2^52: x + kMagic rounds x to an integer
constexpr uint32_t kMagicHi = 0x43380000u;     // ... its bit pattern's high word

// E4M3 byte of x (nearest even, |x| clamped to 448 first: the conversion
// gives NaN above 464), +0 for a zero result.
__device__ __forceinline__ uint32_t e4m3_byte(float x) {
  x = fminf(fmaxf(x, -448.0f), 448.0f);
  uint32_t e = (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(x, 0.0f, 0, false) & 0xffu;
  return e == 0x80u ? 0u : e;
}
__device__ __forceinline__ float e4m3_value(uint32_t e) { return __builtin_amdgcn_cvt_f32_fp8((int)e, 0); }

// x = a s (s a power of two, |x| < 2^51; the product is exact) as hi + lo
// 2^-21 with hi = rint(x - 1) and lo = trunc((x - hi) 2^21), x - hi in
// [1/2, 3/2], so lo lies in [2^20, 3 2^20].  t = fma(a, s, 1.5 2^52 - 1) lands
// where the fp64 spacing is 1: it is 1.5 2^52 + hi, whose bit pattern minus
// that of 1.5 2^52 (low word zero) is hi as a two's-complement integer.
// -hi 2^21 is one exact fma of t, and (x - hi) 2^21 one fma more, rounded once
// at a spacing of 2^-31.  s21 = s 2^21.  The constants sit in registers (an
// instruction reads one scalar operand, and s is the other).
struct LimbConsts {
  double m1, c21, m21;  // 1.5 2^52 - 1, -2^21, 1.5 2^73
  __device__ __forceinline__ LimbConsts() : m1(kMagic - 1.0), c21(-0x1p21), m21(kMagic * 0x1p21) {
    asm volatile("" : "+v"(m1), "+v"(c21), "+v"(m21));
  }
};
__device__ __forceinline__ void split_limbs(double a, double s, double s21, const LimbConsts& k, int64_t& hi,
                                            uint32_t& lo) {
  const double t = __builtin_fma(a, s, k.m1);
  const uint64_t b = (uint64_t)__double_as_longlong(t);
  hi = (int64_t)(((uint64_t)((uint32_t)(b >> 32) - kMagicHi) << 32) | (uint32_t)b);
  lo = (uint32_t)__builtin_fma(a, s21, __builtin_fma(t, k.c21, k.m21));  // truncates toward zero
}
static_assert(kLoBits == 21, "split_limbs scales the remainder by 2^21");
// the sum of n values from the sums of their high and low limbs (the high
// sums stay below 2^60 in magnitude)
__device__ __forceinline__ double join_limbs(int64_t hi, uint32_t lo) {
  return __builtin_fma((double)lo, 0x1p-21, (double)hi);
}

typedef long long ll2 __attribute__((ext_vector_type(2)));

// cells 2 l and 2 l + 1 of a cell row as one 16-byte LDS access
__device__ __forceinline__ ll2* cell_pair(int64_t* row, int l) { return reinterpret_cast<ll2*>(row + 2 * l); }

// x of the lane SHIFT places lower in the same row of 16 lanes, 0 for the
// first SHIFT lanes of a row (row_shr with bound_ctrl)
template <int SHIFT>
__device__ __forceinline__ int64_t row_shr64(int64_t x) {
  const uint64_t u = (uint64_t)x;
  const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)u, 0x110 + SHIFT, 0xf, 0xf, true);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(u >> 32), 0x110 + SHIFT, 0xf, 0xf, true);
  return (int64_t)(((uint64_t)hi << 32) | lo);
}


// BK: the bucket form of the cells (RubinParams::buckets), else the tree form.
template <bool W_BF16, int EMA, bool BK>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(5))) void rubin_reconstruct_kernel(RubinParams p) {
  static_assert(kThreads == kCellBuckets, "one bucket entry per thread");
  // per cell, one row each (so that lanes on different cells spread over the
  // banks): the high limbs of h and of h w in scaled units, both low limbs
  // (h in the lower half), and a flag for an h > 0 lost to the fixed point;
  // then their exclusive prefix sums.  Rows of kCells + 2 entries keep every
  // row 16-byte aligned for the 128-bit accesses of the scan.  One copy of
  // the cells per wavefront (a second copy for the odd lanes, which halves the
  // atomics that meet on one address, measured slower once it set the
  // occupancy)
  __shared__ __align__(16) int64_t s_limb[kWaves][4][kCells + 2];
  __shared__ float s_thr[BK ? 1 : kCells];        // tree form: thresholds in search-tree order
  __shared__ uint4 s_bucket[BK ? kCellBuckets : 1];  // bucket form: first cell, next three thresholds
  __shared__ uint8_t s_tpos[kMaxClips][9];        // cell range of code b under clip k
  __shared__ __align__(8) uint8_t s_lut[kWaves][8];  // the winner's codebook, E4M3 bytes
  __shared__ float s_alpha[kMaxClips], s_clip[kMaxClips];

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = wave_index();
  const int K = p.n_clips;
  if (tid < kMaxClips) {
    s_alpha[tid] = p.alpha[tid];
    s_clip[tid] = p.clip[tid];
  }
  if constexpr (BK) {  // read from the kernel-argument segment with per-lane indices
    const RubinParams* kp = kernarg_params<RubinParams>();
    const int c = kp->base[tid];
    s_bucket[tid] = make_uint4((uint32_t)c, as_u32(kp->thr[c]), as_u32(kp->thr[c + 1]), as_u32(kp->thr[c + 2]));
  } else {
    if (tid < kCells) s_thr[tid] = p.thr[tid];
  }
  if (tid < kMaxClips * 9) (&s_tpos[0][0])[tid] = (&p.tpos[0][0])[tid];
  __syncthreads();

  // this workgroup's matrix (see int_kernel.hip)
  int64_t blk = blockIdx.x;
  struct {
    const void* W;
    float* v;
    const void* g;
    uint8_t* codes;
    uint8_t* lut;
    void* r;
    uint8_t* best_clip;
    float* err;
    int64_t n_blocks, cols, blocks_per_row;
  } mtx = {p.W, p.v, p.g, p.codes, p.lut, p.r, p.best_clip, p.err, p.n_blocks, p.cols, p.blocks_per_row};
  if (p.batch.n > 1) {
    const MatrixSlot& ms = batch_slot<RubinParams>(blk);
    mtx = {ms.W, ms.v, ms.g, ms.codes, static_cast<uint8_t*>(ms.scales), ms.r, ms.best_clip, ms.err, ms.n_units,
         ms.cols, ms.blocks_per_row};
  }
  int64_t bid = blk * kWaves + wave;
  const bool active = bid < mtx.n_blocks;  // uniform per wavefront
  if (!active) return;                   // no block-wide barrier follows
  const int64_t rb = bid / mtx.blocks_per_row, cb = bid - rb * mtx.blocks_per_row;
  const int64_t e0 = (rb * 8 + (lane >> 3)) * mtx.cols + cb * 64 + (lane & 7) * NE;

  // ---- load (each byte once), optional fused EMA, weighting ------------------
  float w[NE], v[NE];
  // bf16 W and g: 8 lanes' 16 bytes are one row of the block, a whole line, so
  // they pass by the caches (with r's stores, Llama set: 718 -> 711 us)
  if constexpr (W_BF16) {
    const uint4 t = ld128_nt(reinterpret_cast<const uint16_t*>(mtx.W) + e0);
    const uint32_t d[4] = {t.x, t.y, t.z, t.w};
#pragma unroll
    for (int k = 0; k < 4; k++) {
      w[2 * k] = as_f32(d[k] << 16);
      w[2 * k + 1] = as_f32(d[k] & 0xffff0000u);
    }
  } else {
    const float* wp = reinterpret_cast<const float*>(mtx.W) + e0;
    const uint4 a = ld128(wp), b = ld128(wp + 4);
    w[0] = as_f32(a.x); w[1] = as_f32(a.y); w[2] = as_f32(a.z); w[3] = as_f32(a.w);
    w[4] = as_f32(b.x); w[5] = as_f32(b.y); w[6] = as_f32(b.z); w[7] = as_f32(b.w);
  }
  {
    const uint4 a = ld128(mtx.v + e0), b = ld128(mtx.v + e0 + 4);
    v[0] = as_f32(a.x); v[1] = as_f32(a.y); v[2] = as_f32(a.z); v[3] = as_f32(a.w);
    v[4] = as_f32(b.x); v[5] = as_f32(b.y); v[6] = as_f32(b.z); v[7] = as_f32(b.w);
  }
  if constexpr (EMA != 0) {
    float g[NE];
    if constexpr (EMA == 1) {
      const uint4 t = ld128_nt(reinterpret_cast<const uint16_t*>(mtx.g) + e0);
      const uint32_t d[4] = {t.x, t.y, t.z, t.w};
#pragma unroll
      for (int k = 0; k < 4; k++) {
        g[2 * k] = as_f32(d[k] << 16);
        g[2 * k + 1] = as_f32(d[k] & 0xffff0000u);
      }
    } else {
      const float* gp = reinterpret_cast<const float*>(mtx.g) + e0;
      const uint4 a = ld128(gp), b = ld128(gp + 4);
      g[0] = as_f32(a.x); g[1] = as_f32(a.y); g[2] = as_f32(a.z); g[3] = as_f32(a.w);
      g[4] = as_f32(b.x); g[5] = as_f32(b.y); g[6] = as_f32(b.z); g[7] = as_f32(b.w);
    }
#pragma unroll
    for (int i = 0; i < NE; i++) {
      const float t = g[i] * g[i];
      const float u = p.omb2 * t;
      v[i] = __builtin_fmaf(p.beta2, v[i], u);
    }
    st128(mtx.v + e0, make_uint4(as_u32(v[0]), as_u32(v[1]), as_u32(v[2]), as_u32(v[3])));
    st128(mtx.v + e0 + 4, make_uint4(as_u32(v[4]), as_u32(v[5]), as_u32(v[6]), as_u32(v[7])));
  }
  if (p.weighting != 0) {
#pragma unroll
    for (int i = 0; i < NE; i++) v[i] = weight_of(v[i], p.weighting);
  }

  // ---- block range, clip-independent moments, fixed-point scales --------------
  float mn = w[0], mx = w[0], hm = v[0];
#pragma unroll
  for (int i = 1; i < NE; i++) {
    mn = fminf(mn, w[i]);
    mx = fmaxf(mx, w[i]);
    hm = fmaxf(hm, v[i]);
  }
  mn = rows_min(run_min<16>(mn));
  mx = rows_max(run_max<16>(mx));
  double H[NE], HW[NE];
  double sww = 0.0;
#pragma unroll
  for (int i = 0; i < NE; i++) {
    H[i] = (double)v[i];
    HW[i] = H[i] * (double)w[i];  // exact: 24 x 24 significant bits
    sww = __builtin_fma(HW[i], (double)w[i], sww);
  }
  sww = rows_sum(run_sum<16>(sww));

  const bool constant = (mx == mn);
  double sh = 0.0;  // sum h, for a constant block's error only
  if (constant) {   // uniform
#pragma unroll
    for (int i = 0; i < NE; i++) sh += H[i];
    sh = rows_sum(run_sum<16>(sh));
  }
  const float c = 0.5f * (mx + mn);
  const float rho = 0.5f * (mx - mn);
  // a constant block's positions give code 0 under any clip
  const float rrho = constant ? 0.0f : 1.0f / rho;
  const float nc = constant ? -0x1p60f : -(c * rrho);
  float u[NE];
#pragma unroll
  for (int i = 0; i < NE; i++) u[i] = __builtin_fmaf(w[i], rrho, nc);

  uint8_t* const lut = s_lut[wave];
  double best_key = __longlong_as_double(0x7ff0000000000000ll);  // +inf

  if (!constant) {  // uniform
    // h < 2^eh and |h w| < 2^(eh + ew): the scaled values stay below 2^51,
    // and the limb sums of 512 of them below 2^60
    hm = rows_max(run_max<16>(hm));
    int eh, ew;
    (void)__builtin_frexpf(hm, &eh);
    (void)__builtin_frexpf(fmaxf(fabsf(mn), fabsf(mx)), &ew);
    const int sh_exp = kHiBits - eh, sw_exp = kHiBits - eh - ew;

    // ---- cells: clear, then add every weight's limbs into its cell ------------
    int64_t(*limb)[kCells + 2] = s_limb[wave];
#pragma unroll
    for (int j = 0; j < 4; j++) *cell_pair(limb[j], lane) = ll2{0, 0};
    wave_lds_fence();
    // the cell of every weight: the number of thresholds <= u
    int pos[NE];
    bool unsafe = false;
    if constexpr (BK) {
      // the bucket's first cell plus cmax compares (thresholds outside u's
      // bucket lie on the far side of u; the padding is NaN), four bucket
      // reads in flight at a time
      auto bin = [&](auto cmax_tag) {
        constexpr int C = decltype(cmax_tag)::value;
#pragma unroll
        for (int i0 = 0; i0 < NE; i0 += 4) {
          uint4 e[4];
#pragma unroll
          for (int t = 0; t < 4; t++) e[t] = s_bucket[cell_bucket(u[i0 + t])];
#pragma unroll
          for (int t = 0; t < 4; t++) {
            const float x = u[i0 + t];
            int c = (int)e[t].x + (x >= as_f32(e[t].y) ? 1 : 0);
            if constexpr (C > 1) c += (x >= as_f32(e[t].z) ? 1 : 0);
            if constexpr (C > 2) c += (x >= as_f32(e[t].w) ? 1 : 0);
            pos[i0 + t] = c;
          }
        }
      };
      if (p.cmax == 1)
        bin(std::integral_constant<int, 1>{});
      else if (p.cmax == 2)
        bin(std::integral_constant<int, 2>{});
      else
        bin(std::integral_constant<int, 3>{});
      // a weight in [unsafe_lo, unsafe_hi] (both negative floats, whose bit
      // patterns grow downwards; both +inf: none): the least of the
      // differences, as unsigned integers, is at most the span's
      const uint32_t top = as_u32(p.unsafe_hi);
      uint32_t near = 0xffffffffu;
#pragma unroll
      for (int i = 0; i < NE; i++) near = min(near, as_u32(u[i]) - top);
      unsafe = near <= as_u32(p.unsafe_lo) - top;
    } else {
      // descend the implicit search tree (node n has children 2n, 2n + 1; the
      // leaves 128 .. 255 are the counts), one level for all 8 weights at a
      // time so that their reads overlap
      int node[NE];
#pragma unroll
      for (int i = 0; i < NE; i++) node[i] = 1;
#pragma unroll
      for (int d = 0; d < 7; d++) {
#pragma unroll
        for (int i = 0; i < NE; i++) node[i] = 2 * node[i] + (s_thr[node[i]] <= u[i] ? 1 : 0);
      }
#pragma unroll
      for (int i = 0; i < NE; i++) pos[i] = node[i] - kCells;
    }
    // a weight between tie thresholds: the block's code-3 and code-4 entries
    // are summed directly below
    const bool block_unsafe = __ballot(unsafe) != 0;  // uniform
    const double s_h = __builtin_ldexp(1.0, sh_exp), s_hw = __builtin_ldexp(1.0, sw_exp);
    const double s_h21 = __builtin_ldexp(1.0, sh_exp + kLoBits), s_hw21 = __builtin_ldexp(1.0, sw_exp + kLoBits);
    const LimbConsts lc;
#pragma unroll
    for (int i = 0; i < NE; i++) {
      int64_t xh, xw;
      uint32_t lh, lw;
      split_limbs(H[i], s_h, s_h21, lc, xh, lh);
      split_limbs(HW[i], s_hw, s_hw21, lc, xw, lw);
      atomicAdd(reinterpret_cast<unsigned long long*>(&limb[0][pos[i]]), (unsigned long long)xh);
      atomicAdd(reinterpret_cast<unsigned long long*>(&limb[1][pos[i]]), (unsigned long long)xw);
      atomicAdd(reinterpret_cast<unsigned long long*>(&limb[2][pos[i]]), ((unsigned long long)lw << 32) | lh);
    }
    // a saliency in (0, 2^-21 units) is 0 in the limbs (rare): its cell is flagged
    const uint32_t lim = as_u32(__builtin_ldexpf(1.0f, -kLoBits - sh_exp));
    uint32_t least = 0xffffffffu;  // the least h > 0, as its bit pattern minus 1 (h = 0 wraps to the largest)
#pragma unroll
    for (int i = 0; i < NE; i++) least = min(least, as_u32(v[i]) - 1u);
    const bool block_lost = __ballot(lim != 0u && least < lim - 1u) != 0;  // uniform
    if (block_lost) {
#pragma unroll
      for (int i = 0; i < NE; i++)
        if (as_u32(v[i]) - 1u < lim - 1u) limb[3][pos[i]] = 1;
    }
    wave_lds_fence();

    // ---- exclusive prefix sums over the cells: lane 16 j + c takes cells
    // 8 c .. 8 c + 7 of limb j and sums them in order, and the lane totals are
    // scanned across the lane's row of 16 (one row per limb).  Integer
    // addition: exact. -------------------------------------------------------
    {
      static_assert(kCells == 4 * 16 * 8 / 4, "16 lanes x 8 cells cover one limb");
      const int j = lane >> 4, c = lane & 15;
      ll2* seg = reinterpret_cast<ll2*>(&limb[j][8 * c]);
      ll2 a[4];
#pragma unroll
      for (int t = 0; t < 4; t++) a[t] = seg[t];
      int64_t in[8];  // inclusive sums within the segment
      in[0] = a[0].x;
#pragma unroll
      for (int t = 1; t < 8; t++) in[t] = in[t - 1] + ((t & 1) ? a[t >> 1].y : a[t >> 1].x);
      int64_t x = in[7];
      x += row_shr64<1>(x);
      x += row_shr64<2>(x);
      x += row_shr64<4>(x);
      x += row_shr64<8>(x);
      const int64_t e = x - in[7];  // the cells before the segment
      seg[0] = ll2{e, e + in[0]};
#pragma unroll
      for (int t = 1; t < 4; t++) seg[t] = ll2{e + in[2 * t - 1], e + in[2 * t]};
      if (c == 15) limb[j][kCells] = x;
    }
    wave_lds_fence();

    // ---- clips, 8 at a time: lane (kk, b) owns codebook entry b of clip k0+kk --
    // the lane keeps the better of its clips, and the clips meet once at the end
    const int kk = lane >> 3, b = lane & 7;
    uint32_t best_e = 0;
    for (int k0 = 0; k0 < K; k0 += 8) {
      const int k = k0 + kk;
      const bool live = k < K;
      const int kc = live ? k : 0;
      const int t0 = s_tpos[kc][b], t1 = s_tpos[kc][b + 1];
      const int64_t cnt = block_lost ? limb[3][t1] - limb[3][t0] : 0;
      const uint64_t lo = (uint64_t)(limb[2][t1] - limb[2][t0]);  // no borrow crosses: both halves grow
      const double hbu = join_limbs(limb[0][t1] - limb[0][t0], (uint32_t)lo);
      double hb = __builtin_ldexp(hbu, -sh_exp);
      double hwb = __builtin_ldexp(join_limbs(limb[1][t1] - limb[1][t0], (uint32_t)(lo >> 32)), -sw_exp);
      // entries with a saliency sum below 2^18 units (where the limbs' 2^-12
      // units could exceed 2^-30 of it) or lost to the fixed point, and in a
      // block with weights between tie thresholds the entries of codes 3 and
      // 4: fp64 sums straight from the weights
      const bool coarse = hbu < 0x1p18 && (hbu > 0.0 || cnt > 0);
      uint64_t need = __ballot(live && (coarse || (block_unsafe && (b == 3 || b == 4))));
      while (need) {  // uniform; rare (h spanning over 2^33 in a block, or a weight at the tie)
        const int L = __builtin_ctzll(need);
        need &= need - 1;
        const int kL = k0 + (L >> 3), bL = L & 7;
        const float al = uniform_f32(s_alpha[kL]);
        double sa = 0.0, sb = 0.0;
#pragma unroll
        for (int i = 0; i < NE; i++) {
          const float q = __builtin_amdgcn_fmed3f(__builtin_rintf(__builtin_fmaf(u[i], al, 3.5f)), 0.0f, 7.0f);
          if ((int)q == bL) {
            sa += H[i];
            sb += HW[i];
          }
        }
        sa = rows_sum(run_sum<16>(sa));
        sb = rows_sum(run_sum<16>(sb));
        if (lane == L) {
          hb = sa;
          hwb = sb;
        }
      }
      // Eq. rubin-fit: the loss-aware mean, in E4M3; an index with no saliency
      // mass keeps the E4M3 value of its grid level
      float meanf;
      if (hb > 0.0) {
        meanf = (float)div_f64(hwb, hb, rcp_f64(hb));
      } else {
        const float f = s_clip[kc];
        const float fr = f * rho;
        meanf = __builtin_fmaf((float)b, (2.0f * fr) / 7.0f, c - fr);
      }
      const uint32_t e = e4m3_byte(meanf);
      const double cv = (double)e4m3_value(e);
      // score: sum_b (C_b^2 H_b - 2 C_b HW_b) + sum h w^2, over the 8 lanes of the clip
      const double score = sww + run_sum<8>(cv * (cv * hb - 2.0 * hwb));
      const double key = live ? make_key(score, k) : __longlong_as_double(0x7ff0000000000000ll);
      if (key < best_key) {
        best_key = key;
        best_e = e;
      }
    }
    // the 8 lanes of a clip hold one key (bit-identical sums): the two clips
    // of a row meet with one mirror step, then the rows combine
    const double kmin = rows_min_f64(min_key(best_key, dpp_f64<kDppMirror>(best_key)));
    if (best_key == kmin) lut[b] = (uint8_t)best_e;  // the 8 lanes of the winning clip
    best_key = kmin;
  } else if (lane < 8) {  // constant block: every code 0, every entry E4M3(w)
    lut[lane] = (uint8_t)e4m3_byte(mn);
  }
  wave_lds_fence();

  // ---- emit ------------------------------------------------------------------
  const uint2 book = *reinterpret_cast<const uint2*>(lut);
  const int kstar = constant ? 0 : key_index(best_key);
  float err;
  if (constant) {
    const double d = (double)e4m3_value(book.x & 0xffu) - (double)mn;
    err = (float)(sh * d * d);
  } else {
    err = (float)__longlong_as_double(__double_as_longlong(best_key) & ~15ll);
  }
  // the codes as bytes (v_cvt_pk_u8_f32 rounds to nearest even and takes
  // negative values to 0); a byte permute of the codebook by four codes gives
  // their four entries
  const float alpha = s_alpha[kstar];
  uint32_t q4[2] = {0u, 0u};
#pragma unroll
  for (int i = 0; i < NE; i++)
    q4[i >> 2] = __builtin_amdgcn_cvt_pk_u8_f32(fminf(__builtin_fmaf(u[i], alpha, 3.5f), 7.0f), i & 3, q4[i >> 2]);
  float r[NE];
#pragma unroll
  for (int t = 0; t < 2; t++) {
    const int e = (int)__builtin_amdgcn_perm(book.y, book.x, q4[t]);
    const auto r01 = __builtin_amdgcn_cvt_pk_f32_fp8(e, false), r23 = __builtin_amdgcn_cvt_pk_f32_fp8(e, true);
    r[4 * t] = r01[0]; r[4 * t + 1] = r01[1];
    r[4 * t + 2] = r23[0]; r[4 * t + 3] = r23[1];
  }
  // 3-bit stream: a dot product with 1, 8, 64 packs three codes, the fourth
  // byte joins at bit 9
  uint32_t bits = 0;
#pragma unroll
  for (int t = 0; t < 2; t++) {
    const uint32_t b12 = __builtin_amdgcn_udot4(q4[t], 0x00400801u, 0u, false) | ((q4[t] >> 24) << 9);
    bits |= b12 << (12 * t);
  }
  // 24 bits per lane at byte offset 3 lane of the block's 192-byte stream:
  // lanes 4i .. 4i + 3 hold its dwords 3i .. 3i + 2, which lanes 4i, 4i + 1 and
  // 4i + 2 store whole, each with its upper neighbour's bits (row_shl:1:
  // lane l reads lane l + 1 of its row of 16; lane 4i + 3 stores nothing)
  {
    const uint32_t up = dpp_u32<0x101>(bits);
    const int part = lane & 3;
    if (part < 3) {
      const uint32_t d = (bits >> (8 * part)) | (up << (24 - 8 * part));
      *reinterpret_cast<uint32_t*>(mtx.codes + bid * 192 + (lane >> 2) * 12 + part * 4) = d;
    }
  }
  if (mtx.r) {
    if constexpr (W_BF16) {
      // r is what is read next: plain stores until the set is far larger than
      // the last-level cache (one matrix, bf16 g, the pass and a reader of r:
      // 2^25 weights 151 us with non-temporal stores, 144 without, the pass
      // alone the same; Llama set, the pass alone 725 and 731)
      const uint4 x = make_uint4(pack_bf16x2(r[0], r[1]), pack_bf16x2(r[2], r[3]), pack_bf16x2(r[4], r[5]),
                                 pack_bf16x2(r[6], r[7]));
      uint16_t* const dst = reinterpret_cast<uint16_t*>(mtx.r) + e0;
      if (p.stream_r)
        st128_nt(dst, x);
      else
        st128(dst, x);
    } else {
      float* rp = reinterpret_cast<float*>(mtx.r) + e0;
      st128(rp, make_uint4(as_u32(r[0]), as_u32(r[1]), as_u32(r[2]), as_u32(r[3])));
      st128(rp + 4, make_uint4(as_u32(r[4]), as_u32(r[5]), as_u32(r[6]), as_u32(r[7])));
    }
  }
  if (lane == 0) {
    *reinterpret_cast<uint2*>(mtx.lut + bid * 8) = book;
    if (mtx.best_clip) mtx.best_clip[bid] = (uint8_t)kstar;
    if (mtx.err) mtx.err[bid] = err;
  }
}

template <bool W_BF16, bool BK>
hipError_t launch_b(const RubinParams& p, int ema_mode, hipStream_t s) {
  const int64_t blocks = p.batch.n > 1 ? p.batch.total_blocks : (p.n_blocks + kWaves - 1) / kWaves;
  const dim3 grid((unsigned)blocks), block(kThreads);
  switch (ema_mode) {
    case 1: hipLaunchKernelGGL((rubin_reconstruct_kernel<W_BF16, 1, BK>), grid, block, 0, s, p); break;
    case 2: hipLaunchKernelGGL((rubin_reconstruct_kernel<W_BF16, 2, BK>), grid, block, 0, s, p); break;
    default: hipLaunchKernelGGL((rubin_reconstruct_kernel<W_BF16, 0, BK>), grid, block, 0, s, p); break;
  }
  return hipGetLastError();
}

template <bool W_BF16>
hipError_t launch_e(const RubinParams& p, int ema_mode, hipStream_t s) {
  return p.buckets ? launch_b<W_BF16, true>(p, ema_mode, s) : launch_b<W_BF16, false>(p, ema_mode, s);
}

}  // namespace

hipError_t launch_rubin(const RubinParams& p, bool w_bf16, int ema_mode, hipStream_t s) {
  return w_bf16 ? launch_e<true>(p, ema_mode, s) : launch_e<false>(p, ema_mode, s);
}

}  // namespace quasar
