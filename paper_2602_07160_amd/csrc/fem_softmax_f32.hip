// fp32 causal softmax-prior FEM read on the fp32 matrix instructions.
//
// For fp32 inputs the read must be accurate to ~1e-4, which bf16 operands
// cannot give; this path evaluates, per (b, h, t, j),
//   F = (1/beta_j) log sum_{i<=t} p_t(i) e^{beta_j v_ij},  p_t = softmax(q_t . k_i / sqrt d)
// (free-energy read, Sec. 2.3, softmax prior, Sec. 1) with every operand,
// product and sum in fp32 (v_mfma_f32_32x32x2_f32):
//
//   S^T = K Q^T,  P = 2^(s log2e/sqrt d - m_t),  E = 2^(beta log2e v - c_j),
//   O^T += E^T P^T,  l_t = sum_i P,  F = (log2(O / l) + c_j) / (beta_j log2 e),
//
// with m_t a running row maximum and c_j a running column maximum, both raised
// lazily.  The exponents carry no bias: near the maxima they are small, so
// their rounding stays at 2^-24 of the term.  An output whose weighted mean
// of E fell below kLow may have lost terms to underflow; it, and one whose
// mean passed kHigh or is NaN, is recomputed from its own keys by a joint
// log-sum-exp per (t, j).
//
// Bound by the fp32 matrix rate (64 cycles per 32x32x2 product, 155 TFLOP/s
// as measured on a large product).  One workgroup takes 32 query rows; its
// four waves split the 32-key tiles (wave w: tiles w, w + 4, ...) and meet in
// LDS at the end, so a short context still has T / 32 workgroups of four
// independent chains and a long one wastes only half a 32 x 32 tile per
// block on the causal mask.  The tile loop uses no LDS and no barrier: the
// contraction order is free, so lane (n, hl) of S^T takes dims 8g + 4hl + 0..3
// of key n in one 16-byte load (four products), lane (j, hl) of E^T loads V
// of its channel (a 128-byte row segment per half wave) and tilts it in
// place, and P feeds the second product straight from S^T's accumulator.
// The next tile's K loads are issued after the last product that reads the
// current ones and its V loads after O's, one tile ahead of their use.
// B4 H12 T1024 d64: 3950 us with one workgroup per query row on the vector
// units, 77 us here (83 TFLOP/s; 112 at B2 H24 T4096, where a workgroup's
// start and end weigh less); B1 H1 T128 d32: 28 and 5.7 us.  Other widths at
// T1024: B4 H12 d32 3810 and 40, d50 3890 and 107; B2 H12 d96 2310
// and 93, d128 2370 and 86; B1 H12 d130 1350 and 146, d200 1415 and 174, d256
// 1495 and 117 (a width that is no multiple of four loads K one dword at a
// time).  Error against float64 at these shapes 2e-7 to 3e-7 of the 2-norm
// (5e-7 to 1.2e-6 before).

#include "fem_device.h"
#include "fem_internal.h"

#include <type_traits>

namespace fem {
namespace {

constexpr int kMaxD = 256;
constexpr int kRows = 32;       // query rows per workgroup, keys per tile
constexpr int kWaves = 4;
constexpr float kRowLag = 8.f;
constexpr float kColLag = 16.f;
// Smallest trusted O / l.  A term that P or E flushed to zero was below 2^-126
// times 2^kColLag, so 2^24 keys lose less than 2^-86, 2^-24 of 2^-62.
constexpr float kLow = 0x1p-60f;
// Largest trusted O / l.  It stays near 2^kColLag as long as the exponents do;
// only where the rounding of c_j itself (2^-24 of |beta v|) is of that size,
// from |beta v| of about 2^30 on, can E pass it, up to infinity.
constexpr float kHigh = 0x1p60f;

// How the widths meet: d == D; d a multiple of 4 below D; any d below D.
constexpr int kFull = 0, kVec4 = 1, kAny = 2;

__device__ __forceinline__ f32x16 mfma32(float a, float b, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

// Accumulator row of register i in lane half hl.
__device__ __forceinline__ int acc_row(int i, int hl) { return 8 * (i >> 2) + 4 * hl + (i & 3); }

// base and bytes are wave-uniform; read from the first lane, they sit in SGPRs
// also where the compiler formed them on the vector unit.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buf(const float* base, unsigned bytes) {
  const uint64_t b = reinterpret_cast<uint64_t>(base);
  const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((unsigned)(b >> 32));
  const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((unsigned)b);
  return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<float*>(((uint64_t)hi << 32) | lo),
                                           (short)0, __builtin_amdgcn_readfirstlane((int)bytes),
                                           0x00020000);
}
__device__ __forceinline__ float load1(__amdgpu_buffer_rsrc_t r, unsigned off) {
  return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, 0));
}

template <int D>
struct F32Smem {
  static constexpr int OROW = D + 1;
  float o[kWaves][kRows * OROW];  // each wave's O [query][channel] at the common shifts
  float m[kWaves][kRows], l[kWaves][kRows];
  __align__(16) float f[kWaves][D];  // column factors to the common shift
  float c[kWaves][D], bl[D];         // column shifts; beta log2 e
  __align__(16) int redo[kWaves];      // per wave: has outputs to recompute
};

// How the epilogue and the recomputation share out a block's outputs: thread
// tid has channel j0 + tid % kLanes of each group of kLanes channels, and rows
// p * kStep + tid / kLanes, p < kPasses.
template <int D>
struct Share {
  static constexpr int kLanes = D < 64 ? D : 64;
  static constexpr int kStep = kWaves * 64 / kLanes;
  static constexpr int kPasses = kRows / kStep;
  static constexpr int kGroups = D / kLanes;
  static_assert(kGroups * kPasses <= 32, "one flag word per thread");
};

// x with -inf and +inf replaced by the type's largest values.
__device__ __forceinline__ float finite(float x) {
  return __builtin_amdgcn_fmed3f(x, -3.4028235e38f, 3.4028235e38f);
}

// (M, S) of a log2-sum-exp2 M + log2(S), and N further terms.  M may be any
// value: a term of -inf adds nothing, +inf gives +inf and NaN stays in S.
template <int N>  // a power of two
__device__ __forceinline__ void lse_add(float& M, float& S, const float (&x)[N]) {
  float mx = M;
#pragma unroll
  for (int u = 0; u < N; ++u) mx = fmaxf(mx, x[u]);
  const float at = finite(mx);
  float e[N];
#pragma unroll
  for (int u = 0; u < N; ++u) e[u] = exp2_hw(x[u] - at);
#pragma unroll
  for (int w = N / 2; w > 0; w >>= 1) {
#pragma unroll
    for (int u = 0; u < w; ++u) e[u] += e[u + w];
  }
  S = fmaf(S, exp2_hw(M - at), e[0]);
  M = mx;
}

// The flagged outputs of one block (bit group * kPasses + p of `low`: this
// thread's row of pass p) from their own keys: F = (LSE_i(s_i + beta v_i) - LSE_i(s_i)) / beta, each
// log-sum-exp with its own maximum, i.e. without shared shifts.  Per round the
// four waves form the scores of four key tiles on the matrix instructions,
// leave them in LDS, and each thread then takes them through the sums of its
// channels and rows that have a flagged output, eight keys at a time with V
// read once for all its rows.  Dims at or past d are zero in both operands (in
// the block's first pass K holds the next row's there).
// Bound by the exponentials.  Every output flagged (us a call; then a wave
// taking one row and eight channels at a time, which formed the row's scores
// anew for each; then the first kernel, one workgroup a row): B4 H12 T1024 d64
// 213, 3085 and 3980; B2 H12 T1024 d128 384, 9370 and 2440; B1 H12 T1024 d256
// 714, 32100 and 1580.  The first one is ahead (by up to 1.9) where few blocks
// leave the chip idle: B1 H16 T96 d100 52, 2200 and 29, B1 H8 T256 d128 100, 2670
// and 88, B1 H1 T1024 d128 343, 9330 and 243.
template <int D, int FORM, class Rows, class Load4>
__device__ __forceinline__ void recompute(F32Smem<D>& sm, Rows&& rows, Load4&& load4,
                                          const float* __restrict__ Qh,
                                          const float* __restrict__ Kh,
                                          const float* __restrict__ Vh, float* __restrict__ Oh,
                                          int T, int d, int qb, unsigned low, float scale2) {
  using Sh = Share<D>;
  constexpr int NP = Sh::kPasses, NG = Sh::kGroups, KU = 8, SROW = kWaves * kRows + 4;
  static_assert(kRows * SROW * sizeof(float) <= sizeof(sm.o), "the scores take O's place");
  float* sc = &sm.o[0][0];  // [query][key of the round]
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));  // nothing of this is formed, and held, before the tile loop
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 31, hl = lane >> 5, q0 = qb * kRows;
  const __amdgpu_buffer_rsrc_t rq = rows(Qh, q0, 0);
  const auto frag = [&](__amdgpu_buffer_rsrc_t r, int g) {
    f32x4 x = load4(r, g);
    if constexpr (FORM != kFull) {
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (8 * g + 4 * hl + u >= d) x[u] = 0.f;
    }
    return x;
  };
  const int r0 = tid / Sh::kLanes;
  int ch[NG];
  float bl[NG], M[NG][NP], S[NG][NP], m = -INFINITY, l = 0.f;
  unsigned rowsof = 0;  // bits as in low: some lane of this wave has a flagged output
#pragma unroll
  for (int group = 0; group < NG; ++group) {
    const int j = group * Sh::kLanes + tid % Sh::kLanes;
    ch[group] = min(j, d - 1);
    bl[group] = sm.bl[j];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      const int bit = group * NP + p;
      rowsof |= __any((low >> bit) & 1u) ? 1u << bit : 0u;
      M[group][p] = -INFINITY;
      S[group][p] = 0.f;
    }
  }
  for (int kb0 = 0; kb0 <= qb; kb0 += kWaves) {
    const int kb = kb0 + wave, k0 = kb0 * kRows;
    if (kb <= qb) {
      const __amdgpu_buffer_rsrc_t rk = rows(Kh, kb * kRows, 0);
      f32x16 s = {};
#pragma unroll 4
      for (int g = 0; g < D / 8; ++g) {
        const f32x4 a = frag(rk, g), b = frag(rq, g);
#pragma unroll
        for (int u = 0; u < 4; ++u) s = mfma32(a[u], b[u], s);
      }
      float x[16];
#pragma unroll
      for (int i = 0; i < 16; ++i)
        x[i] = kb * kRows + acc_row(i, hl) > q0 + n ? -INFINITY : s[i] * scale2;
      lse_add(m, l, x);
#pragma unroll
      for (int g = 0; g < 4; ++g)
        *reinterpret_cast<f32x4*>(sc + n * SROW + wave * kRows + 8 * g + 4 * hl) =
            f32x4{x[4 * g], x[4 * g + 1], x[4 * g + 2], x[4 * g + 3]};
    }
    __syncthreads();
    const int nk = min(kWaves, qb + 1 - kb0) * kRows;
    // last: the round of the diagonal tile (keys after a row stay out, whatever V holds)
    const auto walk = [&](const auto group, const auto last) __attribute__((always_inline)) {
      constexpr int G = decltype(group)::value;
      const float* vj = Vh + ch[G];
      const auto load_v = [&](int kk, float (&v)[KU]) {
#pragma unroll
        for (int u = 0; u < KU; ++u) v[u] = vj[(size_t)min(k0 + kk + u, T - 1) * d];
      };
      float v[KU], vn[KU];
      load_v(0, v);
      for (int kk = 0; kk < nk; kk += KU) {
        load_v(kk + KU, vn);
        f32x4 sr[NP][KU / 4];  // every row's scores first: one wait
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
          for (int w = 0; w < KU / 4; ++w)
            sr[p][w] = *reinterpret_cast<const f32x4*>(sc + (p * Sh::kStep + r0) * SROW + kk + 4 * w);
#pragma unroll
        for (int p0 = 0; p0 < NP; p0 += 2) {  // rows in pairs: two independent chains
          if (!((rowsof >> (G * NP + p0)) & 3u)) continue;
#pragma unroll
          for (int p = p0; p < p0 + 2; ++p) {
            const int lim = q0 + p * Sh::kStep + r0 - (k0 + kk);
            float x[KU];
#pragma unroll
            for (int u = 0; u < KU; ++u) {
              x[u] = fmaf(v[u], bl[G], sr[p][u >> 2][u & 3]);
              if (decltype(last)::value && u > lim) x[u] = -INFINITY;
            }
            lse_add(M[G][p], S[G][p], x);
          }
        }
#pragma unroll
        for (int u = 0; u < KU; ++u) v[u] = vn[u];
      }
    };
    const auto walk_group = [&](const auto group) __attribute__((always_inline)) {
      if (!((rowsof >> (decltype(group)::value * NP)) & ((1u << NP) - 1u))) return;
      if (kb0 + kWaves > qb) walk(group, std::true_type());
      else walk(group, std::false_type());
    };
    walk_group(std::integral_constant<int, 0>());
    if constexpr (NG > 1) walk_group(std::integral_constant<int, 1>());
    if constexpr (NG > 2) {
      walk_group(std::integral_constant<int, 2>());
      walk_group(std::integral_constant<int, 3>());
    }
    __syncthreads();  // the scores are read before the next round's
  }
  // the scores' log-sum-exp: lane halves, then the waves' parts
  {
    const float m1 = other_half(m), l1 = other_half(l), mx = fmaxf(m, m1), at = finite(mx);
    l = l * exp2_hw(m - at) + l1 * exp2_hw(m1 - at);
    if (hl == 0) {
      sm.m[wave][n] = mx;
      sm.l[wave][n] = l;
    }
  }
  __syncthreads();
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    const int r = p * Sh::kStep + r0;
    float mr = sm.m[0][r];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) mr = fmaxf(mr, sm.m[w][r]);
    const float at = finite(mr);
    float lr = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) lr += sm.l[w][r] * exp2_hw(sm.m[w][r] - at);
#pragma unroll
    for (int group = 0; group < NG; ++group)
      if ((low >> (group * NP + p)) & 1u)
        Oh[(size_t)(q0 + r) * d + ch[group]] =
            ((M[group][p] - mr) + (log2_hw(S[group][p]) - log2_hw(lr))) / bl[group];
  }
  __syncthreads();  // the tables are read before the next block's
}

template <int D, int FORM>
__global__ __launch_bounds__(kWaves * 64, D <= 32 ? 3 : D <= 128 ? 2 : 1) void softmax_f32_kernel(
    const float* __restrict__ Q, const float* __restrict__ K, const float* __restrict__ V,
    const float* __restrict__ beta, float* __restrict__ out, int H, int T, int d_arg, int nqb) {
  constexpr int NCB = D / 32;       // 32-channel blocks
  constexpr int NG = D / 8;         // groups of 8 dims: one 16-byte load, four products
  // D <= 64: a whole tile of K and of V sits in registers, loaded one tile
  // ahead.  Wider: K in chunks of 32 dims and V in blocks of 32 channels, two
  // of each, loaded one chunk or block ahead.
  constexpr bool AHEAD = D <= 64;
  constexpr int KC = D < 64 ? NG : D == 64 ? 8 : 4, NC = NG / KC;
  constexpr int NVB = AHEAD ? NCB : 2;
  __shared__ F32Smem<D> sm;
  const int d = FORM == kFull ? D : d_arg;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 31, hl = lane >> 5;
  const int bh = blockIdx.x, h = bh % H;
  const size_t base = (size_t)bh * T * d;
  const float* Qh = Q + base;
  const float* Kh = K + base;
  const float* Vh = V + base;
  float* Oh = out + base;
  const float scale2 = kLog2e / sqrtf((float)d);

  // Rows t0 + r0 .. t0 + 31 of a [T, d] matrix as a buffer resource: one 32-bit
  // lane offset serves every load, and rows at or past T read zero.
  const auto rows = [&](const float* x, int t0, int r0) {
    const int end = min(kRows, T - t0);
    // (a select, not max: min and max together become one vector instruction)
    return buf(x + (size_t)(t0 + r0) * d, (unsigned)(end > r0 ? end - r0 : 0) * (unsigned)d * 4u);
  };
  // dims 8g + 4hl + 0..3 of row n of a tile.  Dims at or past d read whatever
  // follows (the query holds zeros there).
  const unsigned koff = (unsigned)(n * d + 4 * hl) * 4u;
  const auto load4 = [&](__amdgpu_buffer_rsrc_t r, int g) {
    f32x4 x;
    if constexpr (FORM == kAny) {
#pragma unroll
      for (int u = 0; u < 4; ++u) x[u] = load1(r, koff + (8 * g + u) * 4u);
    } else {
      x = __builtin_bit_cast(
          f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)(koff + 32u * g), 0, 0));
    }
    return x;
  };
  // this lane's tilt channels cb * 32 + n, clamped into range (their outputs
  // are not stored)
  int ch[NCB];
  float bl[NCB];
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb) {
    ch[cb] = FORM == kFull ? cb * 32 + n : min(cb * 32 + n, d - 1);
    bl[cb] = beta[h * d + ch[cb]] * kLog2e;
  }

  // (the grid's second dimension is limited, so very long contexts loop)
  for (int yb = blockIdx.y; yb < nqb; yb += gridDim.y) {
    const int qb = nqb - 1 - yb;  // longest causal extent first
    const int q0 = qb * kRows, tq = q0 + n;
    f32x4 qf[NG];
    {
      const __amdgpu_buffer_rsrc_t rq = rows(Qh, q0, 0);
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        qf[g] = load4(rq, g);
        if constexpr (FORM != kFull) {
#pragma unroll
          for (int u = 0; u < 4; ++u)
            if (8 * g + 4 * hl + u >= d) qf[g][u] = 0.f;
        }
      }
    }
    // V of this lane's channel cb * 32 + n, keys acc_row(i, hl) of tile t0.  The
    // row steps beyond the immediate offset's 4 KiB (steps of 8 for a runtime
    // d) are resources of their own, so that every load's bounds check sees its
    // whole offset (a scalar offset is not part of that check).  vrow, the
    // lane's first row, passes through every tile unseen: as a loop invariant
    // its sums with the steps would each take a register, and spill.
    unsigned vrow = (unsigned)(4 * hl * d + (FORM == kFull ? n : 0)) * 4u;
    const auto load_v = [&](int t0, int cb, f32x16& x) {
      constexpr int GR = FORM != kFull ? 1 : D == 32 ? 4 : D == 64 ? 2 : 1;  // steps a resource
      const unsigned off = vrow + (unsigned)(FORM == kFull ? cb * 32 : ch[cb]) * 4u;
#pragma unroll
      for (int g = 0; g < 4; g += GR) {
        const __amdgpu_buffer_rsrc_t r = rows(Vh, t0, 8 * g);
#pragma unroll
        for (int i = 0; i < 4 * GR; ++i)
          x[4 * g + i] = load1(r, off + (unsigned)((8 * (i >> 2) + (i & 3)) * d) * 4u);
      }
    };

    f32x16 acc[NCB], vx[NVB];
    f32x4 kf[AHEAD ? 1 : 2][KC];
    const auto load_kc = [&](__amdgpu_buffer_rsrc_t r, int c) {  // chunk c of a tile's K
#pragma unroll
      for (int g = 0; g < KC; ++g) kf[AHEAD ? 0 : c & 1][g] = load4(r, c * KC + g);
    };
    float cj[NCB], m = -INFINITY, l = 0.f;
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
      acc[cb] = f32x16{};
      cj[cb] = -INFINITY;
    }
    // K before V, as in the tile loop, and without a branch around them (a wave
    // without a tile loads the last one and drops it): the loop's first wait is
    // shared by every way into it, and would otherwise be for V too.
    {
      const int kf0 = min(wave, qb) * kRows;
      load_kc(rows(Kh, kf0, 0), 0);
      __builtin_amdgcn_sched_barrier(0);
      if (AHEAD) {
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) load_v(kf0, cb, vx[cb]);
      }
    }
    // One tile; last: the diagonal one, with the causal mask and, where T ends
    // inside it, keys that stay out of the column maxima and give E = 0.
    const auto tile = [&](const int kb, const auto last) __attribute__((always_inline)) {
      const int k0 = kb * kRows;
      const int kn = min(kb + kWaves, qb) * kRows;  // (past the end: loaded, not used)
      asm("" : "+v"(vrow));
      // resources of the loads below: K of this tile's later chunks and of the
      // next tile
      const __amdgpu_buffer_rsrc_t rk = rows(Kh, k0, 0), rkn = rows(Kh, kn, 0);
      // ---- tilt of block cb: column maximum, lazily raised shift, E in place
      // of V; the shift's factor is owed to the accumulator
      float owed[NCB];
      const auto tilt = [&](int cb) {
        f32x16& x = vx[cb % NVB];
        if (last) {
#pragma unroll
          for (int i = 0; i < 16; ++i)
            if (k0 + acc_row(i, hl) >= T) x[i] = -INFINITY;
        }
        float mx = x[0];
#pragma unroll
        for (int i = 1; i < 16; ++i) mx = fmaxf(mx, x[i]);
        mx = fmaxf(mx, other_half(mx)) * bl[cb];
        const float cn = mx > cj[cb] + kColLag ? mx : cj[cb];
        owed[cb] = cn == cj[cb] ? 1.f : exp2_hw(cj[cb] - cn);
        cj[cb] = cn;
#pragma unroll
        for (int i = 0; i < 16; ++i) x[i] = exp2_hw(fmaf(x[i], bl[cb], -cn));
      };
      const auto pay = [&](int cb) {  // the rows of O^T are channels: row r's factor is in lane r
        if (kb != wave && __any(owed[cb] != 1.f)) {
#pragma unroll
          for (int i = 0; i < 16; ++i) acc[cb][i] *= __shfl(owed[cb], acc_row(i, hl));
        }
      };
      f32x16 s = {};
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        if (c + 1 < NC) load_kc(rk, c + 1);
        else if (!AHEAD) load_v(k0, 0, vx[0]);
#pragma unroll
        for (int g = 0; g < KC; ++g)
#pragma unroll
          for (int u = 0; u < 4; ++u)
            s = mfma32(kf[AHEAD ? 0 : c & 1][g][u], qf[c * KC + g][u], s);
        if (!AHEAD) __builtin_amdgcn_sched_barrier(0);
      }
      if (AHEAD) {
        // the tilt's vector work between the second half of S's products (the
        // first half covers the latency of V's loads)
        __builtin_amdgcn_sched_group_barrier(0x008, 2 * KC, 0);
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) tilt(cb);
#pragma unroll
        for (int i = 0; i < 2 * KC; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // one MFMA
          __builtin_amdgcn_sched_group_barrier(0x402, 10, 0);  // vector and transcendental
        }
        load_kc(rkn, 0);
      }
      // ---- row maximum and probabilities
      if (last) {
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (k0 + acc_row(i, hl) > tq) s[i] = -INFINITY;
      }
      float mx = s[0];
#pragma unroll
      for (int i = 1; i < 16; ++i) mx = fmaxf(mx, s[i]);
      mx = fmaxf(mx, other_half(mx)) * scale2;
      if (__any(mx > m + kRowLag)) {
        const float mn = mx > m + kRowLag ? mx : m;
        const float f = mn == m ? 1.f : exp2_hw(m - mn);
        m = mn;
        l *= f;
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
          for (int i = 0; i < 16; ++i) acc[cb][i] *= f;
      }
      float ls = 0.f;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        s[i] = exp2_hw(fmaf(s[i], scale2, -m));
        ls += s[i];
      }
      l += ls;
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) {
        if (!AHEAD) {
          if (cb + 1 < NCB) load_v(k0, cb + 1, vx[(cb + 1) % NVB]);
          else load_kc(rkn, 0);
          tilt(cb);
        }
        pay(cb);
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[cb] = mfma32(vx[cb % NVB][i], s[i], acc[cb]);
        if (AHEAD) {
          load_v(kn, cb, vx[cb]);
          // exponentials, products and loads in turn (left alone, the loads
          // come in one burst after the products: B2 H24 T4096 945 and 921 us)
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x402, 6, 1);
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 1);
            __builtin_amdgcn_sched_group_barrier(0x020, 1, 1);
          }
        } else __builtin_amdgcn_sched_barrier(0);
      }
    };
    if constexpr (AHEAD) {
      int kb = wave;
      for (; kb < qb; kb += kWaves) tile(kb, std::false_type());
      if (kb == qb) tile(kb, std::true_type());
    } else {  // (a second copy of the wide tile costs it registers)
      for (int kb = wave; kb <= qb; kb += kWaves) tile(kb, kb == qb);
    }
    l += other_half(l);

    // ---- the four waves meet at common shifts M (row) and C (column); a wave
    // that had no tile has shifts of -inf, i.e. factors of zero.  (The thread
    // index anew: what the rest derives from it is not held through the tile
    // loop.)
    int et = tid;
    asm volatile("" : "+v"(et));
    const int en = et & 31, eh = (et >> 5) & 1;
    if (eh == 0) {
      sm.m[wave][en] = m;
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) {
        sm.c[wave][cb * 32 + en] = cj[cb];
        if (wave == 0) sm.bl[cb * 32 + en] = bl[cb];
      }
    }
    __syncthreads();
    // sm.f: each wave's column factors
    for (int j = et; j < D; j += kWaves * 64) {
      float c[kWaves];
#pragma unroll
      for (int w = 0; w < kWaves; ++w) c[w] = sm.c[w][j];
      const float C = fmaxf(fmaxf(c[0], c[1]), fmaxf(c[2], c[3]));
#pragma unroll
      for (int w = 0; w < kWaves; ++w) sm.f[w][j] = exp2_hw(c[w] - C);
    }
    const float M = fmaxf(fmaxf(sm.m[0][en], sm.m[1][en]), fmaxf(sm.m[2][en], sm.m[3][en]));
    const float fr = exp2_hw(m - M);
    if (eh == 0) sm.l[wave][en] = l * fr;
    __syncthreads();
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int j = cb * 32 + 8 * g + 4 * eh;
        const f32x4 fc = *reinterpret_cast<const f32x4*>(&sm.f[wave][j]);
#pragma unroll
        for (int u = 0; u < 4; ++u)
          sm.o[wave][en * sm.OROW + j + u] = acc[cb][4 * g + u] * fr * fc[u];
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    __syncthreads();
    // ---- epilogue, channel fastest; the LDS reads of all of a thread's rows
    // are independent
    using Sh = Share<D>;
    unsigned low = 0;  // outputs to recompute: bit group * kPasses + p
#pragma unroll
    for (int group = 0; group < Sh::kGroups; ++group) {
      const int j = group * Sh::kLanes + et % Sh::kLanes;
      const bool on = j < d;
      const float C = fmaxf(fmaxf(sm.c[0][j], sm.c[1][j]), fmaxf(sm.c[2][j], sm.c[3][j]));
      const float ib = 1.f / sm.bl[j];
      unsigned lg = 0;
#pragma unroll
      for (int p = 0; p < Sh::kPasses; ++p) {
        const int r = p * Sh::kStep + et / Sh::kLanes, t = q0 + r;
        const float L = (sm.l[0][r] + sm.l[1][r]) + (sm.l[2][r] + sm.l[3][r]);
        const int at = r * sm.OROW + j;
        const float mean = ((sm.o[0][at] + sm.o[1][at]) + (sm.o[2][at] + sm.o[3][at])) / L;
        const bool live = on && t < T;
        if (live) Oh[(size_t)t * d + j] = (log2_hw(mean) + C) * ib;
        lg |= live && !(mean >= kLow && mean <= kHigh) ? 1u << p : 0u;
      }
      low |= lg << (group * Sh::kPasses);
    }
    const bool redo = __any(low != 0);
    if (lane == 0) sm.redo[wave] = redo;
    __syncthreads();  // (also: the tables are read before the next block's)
    if ((sm.redo[0] | sm.redo[1]) | (sm.redo[2] | sm.redo[3]))  // rare
      recompute<D, FORM>(sm, rows, load4, Qh, Kh, Vh, Oh, T, d, qb, low, scale2);
  }
}

// Short contexts: one workgroup per query row, since a 32 x 32 tile then holds
// few live entries and one wave walks its whole chain of products (see
// takes_rows).  Sixteen lanes form a score (a row of K in 64-byte segments); then
// a thread has one channel and every so manieth eight of the row's keys, and the
// key groups meet in LDS.  With m the row's largest score and M the largest
// fma(beta v, s - m) so far a term is 2^((beta v - M) + (s - m)), both parts near
// zero where the term counts; where M is so large that its own rounding matters
// it is 2^(x - M) with x rounded like M.  Bound by latency: T1, T16 and T64 of one
// (b, h) at d256 5.2, 5.7 and 8.9 us a call (19.3, 22.5 and 26.1 in tiles), at d130
// 4.9, 5.3 and 7.8 (26.0, 29.9 and 36.0).  Error against float64 2e-8 to 1e-7.
constexpr int kRowKeys = 512;  // longest context
constexpr int kScoreLanes = 16;

template <int NT>
__global__ __launch_bounds__(NT) void softmax_f32_rows_kernel(
    const float* __restrict__ Q, const float* __restrict__ K, const float* __restrict__ V,
    const float* __restrict__ beta, float* __restrict__ out, int H, int T, int d, int lanes_log2) {
  constexpr int NU = kMaxD / kScoreLanes, KU = 8;
  constexpr float kBig = 0x1p20f;
  __shared__ float sc[kRowKeys + KU];
  __shared__ float pm[NT], ps[NT];
  const int tid = threadIdx.x, lane = tid & 63;
  const int bh = blockIdx.x, h = bh % H, t = T - 1 - (int)blockIdx.y, n = t + 1;
  const size_t base = (size_t)bh * T * d;
  const float* Kh = K + base;
  const int j = tid & ((1 << lanes_log2) - 1), grp = tid >> lanes_log2, ngrp = NT >> lanes_log2;
  const float* vj = V + base + min(j, d - 1);
  const float bl = beta[h * d + min(j, d - 1)] * kLog2e;
  const auto load_v = [&](int i0, float (&v)[KU]) {  // (0 past the row: its score is -inf)
#pragma unroll
    for (int u = 0; u < KU; ++u) v[u] = i0 + u < n ? vj[(size_t)(i0 + u) * d] : 0.f;
  };
  float v[KU];
  load_v(grp * KU, v);
  {
    const int c0 = tid % kScoreLanes;
    float qr[NU];
#pragma unroll
    for (int u = 0; u < NU; ++u)
      qr[u] = c0 + u * kScoreLanes < d ? Q[base + (size_t)t * d + c0 + u * kScoreLanes] : 0.f;
    const float scale2 = kLog2e / sqrtf((float)d);
    for (int i = tid / kScoreLanes; i < n; i += NT / kScoreLanes) {
      float dot = 0.f;
#pragma unroll
      for (int u = 0; u < NU; ++u) {
        const int c = c0 + u * kScoreLanes;
        if (u * kScoreLanes < d) dot = fmaf(qr[u], c < d ? Kh[(size_t)i * d + c] : 0.f, dot);
      }
#pragma unroll
      for (int x = kScoreLanes / 2; x > 0; x >>= 1) dot += __shfl_xor(dot, x);
      if (c0 == 0) sc[i] = dot * scale2;
    }
  }
  if (tid < KU) sc[n + tid] = -INFINITY;
  __syncthreads();
  // the prior's normaliser, by every wave
  float m = -INFINITY, l = 0.f;
  for (int i = lane; i < n; i += 64) m = fmaxf(m, sc[i]);
  m = finite(wave_max(m));
  for (int i = lane; i < n; i += 64) l += exp2_hw(sc[i] - m);
  l = wave_sum(l);
  float M = -INFINITY, S = 0.f;
  for (int i0 = grp * KU; i0 < n; i0 += ngrp * KU) {
    float vn[KU], st[KU], x[KU];
    load_v(i0 + ngrp * KU, vn);
    float mx = M;
#pragma unroll
    for (int u = 0; u < KU; ++u) {
      st[u] = sc[i0 + u] - m;
      x[u] = fmaf(v[u], bl, st[u]);
      mx = fmaxf(mx, x[u]);
    }
    const float at = finite(mx);
    const bool big = fabsf(at) >= kBig;
    float e = 0.f;
#pragma unroll
    for (int u = 0; u < KU; ++u)
      e += exp2_hw(big ? x[u] - at : fmaf(v[u], bl, -at) + st[u]);
    S = fmaf(S, exp2_hw(M - at), e);
    M = mx;
#pragma unroll
    for (int u = 0; u < KU; ++u) v[u] = vn[u];
  }
  pm[tid] = M;
  ps[tid] = S;
  __syncthreads();
  if (grp == 0 && j < d) {
    const int live = min(ngrp, (n + KU - 1) / KU);  // groups that had keys
    for (int g = 1; g < live; ++g) M = fmaxf(M, pm[(g << lanes_log2) + j]);
    const float at = finite(M);
    S = 0.f;
    for (int g = 0; g < live; ++g)
      S = fmaf(ps[(g << lanes_log2) + j], exp2_hw(pm[(g << lanes_log2) + j] - at), S);
    out[base + (size_t)t * d + j] = (M + (log2_hw(S) - log2_hw(l))) / bl;
  }
}

template <int D, int FORM>
hipError_t launch(const float* Q, const float* K, const float* V, const float* beta, float* out,
                  int nbh, int H, int T, int d, hipStream_t stream) {
  const int nqb = (T - 1) / kRows + 1;
  const dim3 grid((unsigned)nbh, (unsigned)min(nqb, 65535)), block(kWaves * 64);
  hipLaunchKernelGGL((softmax_f32_kernel<D, FORM>), grid, block, 0, stream, Q, K, V, beta, out, H,
                     T, d, nqb);
  return hipGetLastError();
}

// One workgroup per row, or per 32 rows?  By the rows (nbh T), the work (nbh T T)
// and T.  Measured (us a call, rows and tiles; 1, 8, 32 and 128 (b, h)) at:
//   d = 7: 8 of T48 6.4 and 6.7, 32 of T32 7.1 and 6.9, 200 of T8 5.0 and 6.4,
//     256 of T16 8.4 and 6.6;
//   d = 32: 1 of T32 5.4 and 5.6, 32 5.5 and 6.0, 32 of T48 6.8 and 5.8, 200 of
//     T8 5.0 and 6.1, 128 of T16 8.1 and 5.5;
//   d = 50: 8 of T128 10.7 and 12.2, 32 of T64 10.8 and 11.8, of T96 15.9 and
//     12.0, 128 of T16 8.4 and 10.1, of T32 14.2 and 11.9;
//   d = 64: 1 of T192 9.6 and 10.5, of T256 11.4 and 10.5, 8 of T96 7.5 and 8.4,
//     of T128 10.8 and 8.5, 32 of T48 7.8 and 8.4, 128 of T8 5.2 and 7.0, of T16
//     8.3 and 7.6;
//   d = 100: 8 of T128 14.7 and 15.1, 32 of T64 13.4 and 15.3, of T96 21.1 and
//     15.2, 128 of T16 9.3 and 13.3, of T32 17.2 and 15.3;
//   d = 128: 1 of T256 16.3 and 17.7, 8 of T96 9.1 and 13.2, of T128 15.1 and
//     13.1, 32 of T48 8.3 and 13.0, of T64 13.5 and 13.1, 128 of T16 9.2 and 11.2;
//   d = 130: 1 of T512 40 and 79, 32 of T96 29 and 37, of T128 47 and 39, 128 of
//     T48 36 and 37; d = 200: 32 of T96 33 and 36, 128 of T48 40 and 41;
//   d = 256: 1 of T256 26 and 37, 8 of T128 21 and 27, 32 of T64 20 and 27, of T96
//     34 and 27, 128 of T32 24 and 27, of T48 42 and 27.
bool takes_rows(int nbh, int T, int d) {
  struct Most {
    int rows, work, T;
  };
  constexpr Most kMost[4][2] = {{{2048, 32768, 32}, {2048, 18432, 48}},       // d = 32; narrower
                                {{1536, 73728, 192}, {2048, 131072, 512}},   // d = 64; 33 .. 63
                                {{2048, 73728, 256}, {2048, 131072, 512}},   // d = 128; 65 .. 127
                                {{4096, 131072, 512}, {6144, 294912, 512}}}; // d = 256; 129 .. 255
  const int w = d <= 32 ? 0 : d <= 64 ? 1 : d <= 128 ? 2 : 3;
  const Most m = kMost[w][d == 32 << w ? 0 : 1];
  return T <= m.T && (int64_t)nbh * T <= m.rows && (int64_t)nbh * T * T <= m.work;
}

template <int NT>
hipError_t launch_rows(const float* Q, const float* K, const float* V, const float* beta, float* out,
                       int nbh, int H, int T, int d, int lanes_log2, hipStream_t stream) {
  hipLaunchKernelGGL(softmax_f32_rows_kernel<NT>, dim3((unsigned)nbh, (unsigned)T), dim3(NT), 0,
                     stream, Q, K, V, beta, out, H, T, d, lanes_log2);
  return hipGetLastError();
}

// As many threads as have keys (eight each) or form the scores in two rounds, up
// to 256; 512 where the rows leave most of the chip idle: 8 (b, h) of T96 d64 7.5
// us a call and 9.2 with 256, of T128 11.6 and 10.8.
hipError_t launch_rows(const float* Q, const float* K, const float* V, const float* beta, float* out,
                       int nbh, int H, int T, int d, hipStream_t stream) {
  int lanes_log2 = 3;  // a power of two of lanes covers the channels
  while ((1 << lanes_log2) < d) ++lanes_log2;
  const int threads = max((T + 7) / 8 << lanes_log2, 8 * T);
  const auto go = [&](auto f) { return f(Q, K, V, beta, out, nbh, H, T, d, lanes_log2, stream); };
  if (threads <= 64) return go(launch_rows<64>);
  if (threads <= 128) return go(launch_rows<128>);
  if (d <= 32 || threads <= 256 || nbh * T > 768) return go(launch_rows<256>);
  return go(launch_rows<512>);
}

}  // namespace

hipError_t launch_softmax_f32(const float* Q, const float* K, const float* V, const float* beta,
                              float* out, int B, int H, int T, int d, hipStream_t stream) {
  if (d < 1 || d > kMaxD) return hipErrorInvalidValue;
  const int D = d <= 32 ? 32 : d <= 64 ? 64 : d <= 128 ? 128 : 256;
  const int form = d == D ? kFull : d % 4 == 0 ? kVec4 : kAny;
  if (takes_rows(B * H, T, d)) return launch_rows(Q, K, V, beta, out, B * H, H, T, d, stream);
  const auto go = [&](auto f) { return f(Q, K, V, beta, out, B * H, H, T, d, stream); };
#define FEM_F32_FORM(W)                                  \
  if (D == W) {                                          \
    if (form == kFull) return go(launch<W, kFull>);      \
    if (form == kVec4) return go(launch<W, kVec4>);      \
    return go(launch<W, kAny>);                          \
  }
  FEM_F32_FORM(32)
  FEM_F32_FORM(64)
  FEM_F32_FORM(128)
  FEM_F32_FORM(256)
#undef FEM_F32_FORM
  return hipErrorInvalidValue;
}

}  // namespace fem
