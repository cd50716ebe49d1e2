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
// units, 79 us here (82 TFLOP/s; 113 at B2 H24 T4096, where a workgroup's
// start and end weigh less); B1 H1 T128 d32: 28 and 5.7 us.  Error against
// float64 at these shapes 2e-7 to 3e-7 of the 2-norm (5e-7 to 1.2e-6 before).

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
constexpr int kBatch = 8;         // channels recomputed per pass of the exact path

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

// Streaming log2-sum-exp2 accumulator: value = m + log2(s), for
// terms of any kind: a term of -inf adds
// nothing, +inf gives +inf, and NaN stays in s whatever m is.
struct LseAny {
  float m = -INFINITY;
  float s = 0.f;
  __device__ __forceinline__ void add(float w) {
    if (w > m) {
      s = s * exp2_hw(m - w) + 1.f;
      m = w;
    } else if (w != -INFINITY) {
      s += w == m ? 1.f : exp2_hw(w - m);
    }
  }
  // Combine across the 64 lanes of a wave; every lane gets the total.
  __device__ __forceinline__ float wave_total() const {
    float M = wave_max(m);
    float part = s == 0.f ? 0.f : m == M ? s : s * exp2_hw(m - M);
    float S = wave_sum(part);
    return M + log2_hw(S);
  }
};

// Exact fp32 read of channels ch[0..nb) of row t by one wave: per channel the
// joint log-sum-exp of (score + tilt) over the keys i <= t, minus that of
// the scores.  Lane c < nb returns channel ch[c]'s value.
__device__ float exact_row_f32(const float* __restrict__ Qh, const float* __restrict__ Kh,
                               const float* __restrict__ Vh, int t, int d, const int (&ch)[kBatch],
                               const float (&bl)[kBatch], int nb, float scale2) {
  const int lane = threadIdx.x & 63;
  LseAny den, num[kBatch];
  const float* qr = Qh + (size_t)t * d;
  for (int i = lane; i <= t; i += 64) {
    const float* kr = Kh + (size_t)i * d;
    float dot = 0.f;
    for (int c = 0; c < d; ++c) dot = fmaf(qr[c], kr[c], dot);
    const float s = dot * scale2;
    den.add(s);
#pragma unroll
    for (int c = 0; c < kBatch; ++c)
      if (c < nb) num[c].add(fmaf(Vh[(size_t)i * d + ch[c]], bl[c], s));
  }
  const float l = den.wave_total();
  float mine = 0.f;
#pragma unroll
  for (int c = 0; c < kBatch; ++c) {
    if (c < nb) {
      const float o = (num[c].wave_total() - l) / bl[c];
      if (lane == c) mine = o;
    }
  }
  return mine;
}

template <int D>
struct F32Smem {
  static constexpr int OROW = D + 1;
  float o[kWaves][kRows * OROW];  // each wave's O [query][channel] at the common shifts
  float m[kWaves][kRows], l[kWaves][kRows];
  __align__(16) float f[kWaves][D];  // column factors to the common shift
  float c[kWaves][D], bl[D];         // column shifts; beta log2 e
};

template <int D, int FORM>
__global__ __launch_bounds__(kWaves * 64, D <= 128 ? 2 : 1) void softmax_f32_kernel(
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
    return buf(x + (size_t)(t0 + r0) * d,
               (unsigned)max(min(kRows, T - t0) - r0, 0) * (unsigned)d * 4u);
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
    // row steps of 8 are resources of their own, so that every load's bounds
    // check sees its whole offset (a scalar offset is not part of that check).
    // The lane offset is formed anew for every block: kept for all of them,
    // the wide forms spill it (d = 128 256 bytes a lane, 212 so).
    const auto load_v = [&](int t0, int cb, f32x16& x) {
      unsigned off = (unsigned)(4 * hl * d + ch[cb]) * 4u;
      asm volatile("" : "+v"(off));
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const __amdgpu_buffer_rsrc_t r = rows(Vh, t0, 8 * g);
#pragma unroll
        for (int u = 0; u < 4; ++u) x[4 * g + u] = load1(r, off + (unsigned)(u * d) * 4u);
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
    if (wave <= qb) {
      load_kc(rows(Kh, wave * kRows, 0), 0);
      if (AHEAD) {
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) load_v(wave * kRows, cb, vx[cb]);
      }
    }
    // One tile; last: the diagonal one, with the causal mask and, where T ends
    // inside it, keys that stay out of the column maxima and give E = 0.
    const auto tile = [&](const int kb, const auto last) __attribute__((always_inline)) {
      const int k0 = kb * kRows;
      const int kn = min(kb + kWaves, qb) * kRows;  // (past the end: loaded, not used)
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
        if (AHEAD) load_v(kn, cb, vx[cb]);
        else __builtin_amdgcn_sched_barrier(0);
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
    // that had no tile has shifts of -inf, i.e. factors of zero
    if (hl == 0) {
      sm.m[wave][n] = m;
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) {
        sm.c[wave][cb * 32 + n] = cj[cb];
        if (wave == 0) sm.bl[cb * 32 + n] = bl[cb];
      }
    }
    __syncthreads();
    // sm.f: each wave's column factors
    for (int j = tid; j < D; j += kWaves * 64) {
      float c[kWaves];
#pragma unroll
      for (int w = 0; w < kWaves; ++w) c[w] = sm.c[w][j];
      const float C = fmaxf(fmaxf(c[0], c[1]), fmaxf(c[2], c[3]));
#pragma unroll
      for (int w = 0; w < kWaves; ++w) sm.f[w][j] = exp2_hw(c[w] - C);
    }
    const float M = fmaxf(fmaxf(sm.m[0][n], sm.m[1][n]), fmaxf(sm.m[2][n], sm.m[3][n]));
    const float fr = exp2_hw(m - M);
    if (hl == 0) sm.l[wave][n] = l * fr;
    __syncthreads();
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int j = cb * 32 + 8 * g + 4 * hl;
        const f32x4 fc = *reinterpret_cast<const f32x4*>(&sm.f[wave][j]);
#pragma unroll
        for (int u = 0; u < 4; ++u)
          sm.o[wave][n * sm.OROW + j + u] = acc[cb][4 * g + u] * fr * fc[u];
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    __syncthreads();
    // ---- epilogue, channel fastest: a thread keeps one channel (of each
    // group of LPR) and takes every RPI-th row; the LDS reads of all its rows
    // are independent
    constexpr int LPR = D < 64 ? D : 64, RPI = kWaves * 64 / LPR;  // lanes a row, rows a pass
#pragma unroll
    for (int j0 = 0; j0 < D; j0 += LPR) {
      const int j = j0 + tid % LPR;
      const bool on = j < d;
      const float C = fmaxf(fmaxf(sm.c[0][j], sm.c[1][j]), fmaxf(sm.c[2][j], sm.c[3][j]));
      const float ib = 1.f / sm.bl[j];
      unsigned low = 0;  // bit p: this thread's row of pass p
#pragma unroll
      for (int p = 0; p < kRows / RPI; ++p) {
        const int r = p * RPI + tid / LPR, t = q0 + r;
        const float L = (sm.l[0][r] + sm.l[1][r]) + (sm.l[2][r] + sm.l[3][r]);
        const int at = r * sm.OROW + j;
        const float mean = ((sm.o[0][at] + sm.o[1][at]) + (sm.o[2][at] + sm.o[3][at])) / L;
        const bool live = on && t < T;
        if (live) Oh[(size_t)t * d + j] = (log2_hw(mean) + C) * ib;
        low |= live && !(mean >= kLow && mean <= kHigh) ? 1u << p : 0u;
      }
      // rare: a mean that lost range (or is NaN), recomputed exactly, one row
      // at a time by the whole wave
      while (true) {
        const uint64_t who = __ballot(low != 0);
        if (who == 0) break;
        const int src = __builtin_ctzll(who);
        const int p = __builtin_ctz(__builtin_amdgcn_readlane(low, src));
        const int r = p * RPI + (wave * 64 + src) / LPR;
        // the row's flagged channels: lanes of the same row
        const bool same = (tid / LPR) == (wave * 64 + src) / LPR && ((low >> p) & 1u);
        uint64_t todo = __ballot(same);
        if (same) low &= ~(1u << p);
        while (todo != 0) {
          int chs[kBatch];
          float bls[kBatch];
          int nb = 0, mych = 0;
#pragma unroll
          for (int c = 0; c < kBatch; ++c) {
            chs[c] = 0;
            bls[c] = 1.f;
            if (todo == 0) continue;
            const int ln = __builtin_ctzll(todo);
            todo &= todo - 1;
            chs[c] = j0 + (wave * 64 + ln) % LPR;
            bls[c] = sm.bl[chs[c]];
            nb = c + 1;
            if (lane == c) mych = chs[c];
          }
          const float x = exact_row_f32(Qh, Kh, Vh, q0 + r, d, chs, bls, nb, scale2);
          asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // after the stores above
          if (lane < nb) Oh[(size_t)(q0 + r) * d + mych] = x;
        }
      }
    }
    __syncthreads();  // the tables are read before the next block's
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

}  // namespace

hipError_t launch_softmax_f32(const float* Q, const float* K, const float* V, const float* beta,
                              float* out, int B, int H, int T, int d, hipStream_t stream) {
  if (d < 1 || d > kMaxD) return hipErrorInvalidValue;
  const int D = d <= 32 ? 32 : d <= 64 ? 64 : d <= 128 ? 128 : 256;
  const int form = d == D ? kFull : d % 4 == 0 ? kVec4 : kAny;
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
