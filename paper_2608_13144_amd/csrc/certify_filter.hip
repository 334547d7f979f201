// Certification through a float16 filter: the exact float64 logits of only
// the classes that can matter.
//
// The margin needs the two largest logits of a row and the tight radius the
// least (s_y - s_j) / ||W_y - W_j||; which classes those are, float16 matrix
// instructions (32 times the float64 rate) tell within a rigorous error E:
//   |s'_c - s_c| <= E_c = E_0 + gamma |b_c|, E_0 = k ||w||_max ||z|| + eta terms
// (k = 2u + u^2 + gamma (1 + u)^2, u = 2^-11; for a bf16 store, exact in
// float16, k = u + gamma (1 + u); gamma covers four times the float32
// accumulation, whose order the matrix core does not specify).  E is E_c for
// the classes that can matter: |b_c| <= |b|_max, and, as b_c = s_c - w_c . z
// and such a class's s_c is about as large as the row's top two, |b_c| is less
// than three times M + E_0 + ||w||_max ||z||, M = max(|s'_(1)|, |s'_(2)|); so a
// class that a bias of -1e9 masks does not widen it.
//   pass 1  the two largest s' of every row;
//   pass 2  the classes with s'_c >= s'_(2) - 2E.  Two classes have s >= s'_(2)
//           - E, so every class of the true top two, ties included, is listed;
//   exact   float64 sums of the listed classes: label, margin, radius;
//   tight   pass 3 lists the classes with (s_y - s'_j - E) <= rho ||W_y - W_j||,
//           rho the exact ratio of the second class, which bounds the minimum
//           from above, and their exact ratios give the minimum.  (Those that
//           matter have s_j >= s_y - 2 rho ||w||_max, so |b_j| is at most
//           |s_y| + 2 rho ||w||_max + ||w||_max ||z||.)
// The numbers that leave are float64 sums as before, of the same values.  Rows
// that list too many classes (crowded or repeated head rows), lie outside the
// float16 range or are not finite are left to the float64 kernel.
//
// What bounds it: the passes read each row once (registers) and the head's
// image from LDS; the float64 kernel formed all C logits at half of 78.6
// TFLOP/s.  At N = 1M, d = 256, C = 200: 2.54 -> 0.70 ms (the candidates alone
// are 1 GiB, 0.2 ms at 5.2 TB/s), tight 3.13 -> 1.22 ms; at N = 65,536 with a
// bfloat16 store 173 -> 58 us.  What is left is the latency of the exact sums'
// loads (a row again and two to three head rows of it).
//
// A wave holds 32 rows as B operands for all of d (64 rows a wave halve the
// head's LDS reads but leave two waves per SIMD to hide the latency of the
// exact sums: 0.82 against 0.70 ms); four waves share the 32-class tiles of the
// head, stored in operand order (lane l of k-step ks reads 16 bytes at 16 l),
// copied through registers one tile ahead.  Rows are columns of the 32x32 output, so a lane sees 16 classes of
// its own row per tile and keeps the running top two without any exchange.
#include <limits.h>

#include <type_traits>

#include "lc_certify.hpp"

namespace lc {

typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kCfThreads = 256;
constexpr int kCfWaves = kCfThreads / kWave;
constexpr int kCfTile = 32;   // classes per tile
constexpr int kCfList = 8;    // listed classes per lane (two lanes share a row)

// Head image in operand order, norms rounded up (infinite past the float16
// range) and the bias, padded to whole tiles (-inf: never listed).
struct HeadImage {
  u32x4* w16;   // [tiles][d / 16][64]
  float* wn;    // [tiles * 32]
  float* bias;  // [tiles * 32]
  float* dist;  // [C][stride] row distances in float32 for pass 3, or null
  int stride;   // C rounded up to 4
};

// The image takes at most half of the float64 copy's room (C > 32); the
// float32 distances get the rest where it holds them (without them pass 3
// reads the float64 table: a load per class instead of one per four, each
// touching 64 lines).
inline HeadImage head_layout(void* ws, int32_t C, int32_t d) {
  const int64_t pad = (C + kCfTile - 1) / kCfTile * kCfTile;
  unsigned char* p = static_cast<unsigned char*>(ws);
  HeadImage h;
  h.w16 = reinterpret_cast<u32x4*>(p);
  h.wn = reinterpret_cast<float*>(p + pad * d * 2);
  h.bias = h.wn + pad;
  h.stride = (C + 3) / 4 * 4;
  const int64_t used = pad * d * 2 + pad * 8, room = static_cast<int64_t>(C) * d * 8;
  h.dist = used + static_cast<int64_t>(C) * h.stride * 4 <= room ? h.bias + pad : nullptr;
  return h;
}

__global__ __launch_bounds__(kCfThreads) void dist32_kernel(const double* __restrict__ row_dist, int C, HeadImage h) {
  const int64_t t = static_cast<int64_t>(blockIdx.x) * kCfThreads + threadIdx.x;
  if (t >= static_cast<int64_t>(C) * h.stride) return;
  const int64_t y = t / h.stride, j = t % h.stride;
  h.dist[t] = j < C ? static_cast<float>(row_dist[y * C + j]) : 0.0f;
}

// One wave per class row.
__global__ __launch_bounds__(kCfThreads) void head_image_kernel(const float* __restrict__ W, const float* __restrict__ b,
                                                                int C, int d, int pad, HeadImage h) {
  const int lane = lane_id();
  const int c = static_cast<int>(blockIdx.x) * kCfWaves + static_cast<int>(threadIdx.x) / kWave;
  if (c >= pad) return;
  double s = 0.0;
  for (int ch = lane; ch < d / 8; ch += kWave) {  // 16-byte chunks of the image row
    float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (c < C) {
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = W[static_cast<int64_t>(c) * d + ch * 8 + j];
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) s = __builtin_fma(static_cast<double>(v[j]), static_cast<double>(v[j]), s);
    const int64_t at = (static_cast<int64_t>(c / kCfTile) * (d / 16) + ch / 2) * kWave + (ch & 1) * 32 + c % kCfTile;
    h.w16[at] = pack_f16x8(v);
  }
  s = wave_sum(s);
  if (lane == 0) {
    h.wn[c] = s < kF16Range2 ? static_cast<float>(__builtin_sqrt(s) * (1.0 + 1e-6)) : __builtin_inff();
    h.bias[c] = c < C ? (b ? b[c] : 0.0f) : -__builtin_inff();
  }
}

__device__ __forceinline__ f32x16 mfma_logits(u32x4 w, u32x4 z, f32x16 acc) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, w), __builtin_bit_cast(f16x8, z), acc, 0, 0,
                                                0);
}

// Class of accumulator i of a lane in half h, within its tile.
__device__ __forceinline__ int tile_class(int i, int h) { return 8 * (i >> 2) + 4 * h + (i & 3); }

// The same sum in every lane of a 16-lane group up to the order of the last
// two additions; lane 0's is the one used.
__device__ __forceinline__ double sum16(double v) {
  v += dpp_f64<kDppQuadXor1>(v);
  v += dpp_f64<kDppQuadXor2>(v);
  v += dpp_f64<kDppRowRor4>(v);
  v += dpp_f64<kDppRowRor8>(v);
  return v;
}

constexpr int kCfRowsW = 32;                  // rows per wave
constexpr int kCfRows = kCfWaves * kCfRowsW;  // rows per workgroup

template <bool BF16_STORE, bool TIGHT, int KS>
__global__ __launch_bounds__(kCfThreads, KS <= 16 ? 3 : 2) void certify_filter_kernel(
    const float* __restrict__ z, int64_t N, int d, const float* __restrict__ W, const float* __restrict__ b, int C,
    double sigma, const HeadImage head, const double* __restrict__ row_dist, int32_t* __restrict__ label_out,
    float* __restrict__ r_out, float* __restrict__ margin_out, float* __restrict__ norm2_out) {
  __shared__ __attribute__((aligned(16))) u32x4 wt[2][KS * kWave];
  __shared__ uint16_t list[kCfWaves][kWave][kCfList];
  __shared__ int count[kCfWaves][kWave];
  __shared__ float red[2][kCfWaves];
  __shared__ double s_top[TIGHT ? kCfWaves : 1][kCfRowsW];
  __shared__ double s_rho[TIGHT ? kCfWaves : 1][kCfRowsW];
  __shared__ int s_lab[TIGHT ? kCfWaves : 1][kCfRowsW];

  const int lane = lane_id();
  const int wave = uniform(static_cast<int>(threadIdx.x) / kWave);
  const int c32 = lane & 31, h = lane >> 5;
  const int nk = d / 16;
  const int tiles = (C + kCfTile - 1) / kCfTile;
  const int64_t row0 = static_cast<int64_t>(blockIdx.x) * kCfRows + wave * kCfRowsW;

  // head maxima
  float wmax = 0.0f, bmax = 0.0f;
  for (int c = static_cast<int>(threadIdx.x); c < C; c += kCfThreads) {
    wmax = __builtin_fmaxf(wmax, head.wn[c]);
    bmax = __builtin_fmaxf(bmax, __builtin_fabsf(head.bias[c]));
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    wmax = __builtin_fmaxf(wmax, __shfl_xor(wmax, o, kWave));
    bmax = __builtin_fmaxf(bmax, __shfl_xor(bmax, o, kWave));
  }
  if (lane == 0) {
    red[0][wave] = wmax;
    red[1][wave] = bmax;
  }

  // The lane's row as B operand: row row0 + c32, k = 16 ks + 8 h + j (stored
  // values); its squared norm the first time.
  u32x4 zb[KS];
  double nrm = 0.0;
  auto load_operands = [&](auto first) {
    const int64_t e = row0 + c32;
    const float* row = z + (e < N ? e : N - 1) * d;
    double s = 0.0;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      zb[ks] = u32x4{0u, 0u, 0u, 0u};
      if (ks < nk) {
        const f32x4 x0 = *reinterpret_cast<const f32x4*>(row + 16 * ks + 8 * h);
        const f32x4 x1 = *reinterpret_cast<const f32x4*>(row + 16 * ks + 8 * h + 4);
        float v[8] = {x0[0], x0[1], x0[2], x0[3], x1[0], x1[1], x1[2], x1[3]};
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          if constexpr (BF16_STORE) v[j] = bf16_round_f32(v[j]);
          if constexpr (decltype(first)::value)
            s = __builtin_fma(static_cast<double>(v[j]), static_cast<double>(v[j]), s);
        }
        zb[ks] = pack_f16x8(v);
      }
    }
    if constexpr (decltype(first)::value) {
      nrm = s + __shfl_xor(s, 32, kWave);
      if (norm2_out && h == 0 && e < N) norm2_out[e] = static_cast<float>(nrm);
    }
  };
  load_operands(std::true_type{});

  // One tile of the head through registers into LDS: thread t carries chunks
  // t, t + 256, ... of nk * 64.
  constexpr int kIters = KS * kWave / kCfThreads;
  u32x4 carry[kIters];
  auto fetch = [&](int t) {
#pragma unroll
    for (int j = 0; j < kIters; ++j) {
      const int i = j * kCfThreads + static_cast<int>(threadIdx.x);
      if (i < nk * kWave) carry[j] = head.w16[static_cast<int64_t>(t) * nk * kWave + i];
    }
  };
  auto put = [&](int buf) {
#pragma unroll
    for (int j = 0; j < kIters; ++j) {
      const int i = j * kCfThreads + static_cast<int>(threadIdx.x);
      if (i < nk * kWave) wt[buf][i] = carry[j];
    }
  };
  // Logits of one tile, started at the bias.
  auto logits = [&](int t, int buf) {
    f32x16 acc;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const f32x4 bv = *reinterpret_cast<const f32x4*>(head.bias + t * kCfTile + 8 * j + 4 * h);
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[4 * j + i] = bv[i];
    }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      if (ks < nk) acc = mfma_logits(wt[buf][ks * kWave + lane], zb[ks], acc);
    return acc;
  };
  // Every tile in order: the next one is fetched while this one is formed.
  // (A buffer is written after a barrier that follows its last readers.)
  auto sweep = [&](auto&& each) {
    __syncthreads();
    fetch(0);
    put(0);
    for (int t = 0; t < tiles; ++t) {
      if (t + 1 < tiles) fetch(t + 1);
      __syncthreads();
      each(t, logits(t, t & 1));
      if (t + 1 < tiles) put((t + 1) & 1);
    }
  };

  // pass 1: the two largest filtered logits of the row
  float v1 = -__builtin_inff(), v2 = -__builtin_inff();
  sweep([&](int, const f32x16& acc) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      v2 = __builtin_amdgcn_fmed3f(v1, v2, acc[i]);
      v1 = __builtin_fmaxf(v1, acc[i]);
    }
  });
  wmax = bmax = 0.0f;
#pragma unroll
  for (int w = 0; w < kCfWaves; ++w) {
    wmax = __builtin_fmaxf(wmax, red[0][w]);
    bmax = __builtin_fmaxf(bmax, red[1][w]);
  }
  // E_0 (returns ||w||_max ||z||), and E where |b_c| <= bound
  auto row_error = [&](double& e0) {
    constexpr double u = 1.0 / 2048.0, eta = 1.0 / 16384.0;
    const double gam = 4.0 * (d + 2.0) / 16777216.0;
    const double k = BF16_STORE ? u + gam * (1.0 + u) : 2.0 * u + u * u + gam * (1.0 + u) * (1.0 + u);
    const double wm = static_cast<double>(wmax);
    const double zn = __builtin_sqrt(nrm);
    e0 = (k * wm * zn + eta * (1.0 + u) * (1.0 + gam) * __builtin_sqrt(static_cast<double>(d)) * (wm + zn) +
          (1.0 + gam) * d * eta * eta) *
             (1.0 + 1e-6) +
         kFilterAbsSlack;
    return wm * zn;
  };
  auto with_bias = [&](double e0, double bound) {
    const double gam = 4.0 * (d + 2.0) / 16777216.0;
    return e0 + gam * __builtin_fmin(static_cast<double>(bmax), bound) * (1.0 + 1e-6);
  };
  double err;
  float cut;
  {
    const float o1 = __shfl_xor(v1, 32, kWave), o2 = __shfl_xor(v2, 32, kWave);
    v2 = __builtin_fmaxf(__builtin_fminf(v1, o1), __builtin_fmaxf(v2, o2));
    v1 = __builtin_fmaxf(v1, o1);
    double e0;
    const double wz = row_error(e0);
    const double top = static_cast<double>(__builtin_fmaxf(__builtin_fabsf(v1), __builtin_fabsf(v2)));
    err = with_bias(e0, 3.0 * (top + e0 + wz));
    if (!(nrm < kF16Range2)) err = __builtin_inf();  // also a NaN row
    cut = f32_round_down(static_cast<double>(v2) - 2.0 * err);
  }

  // pass 2: the classes that reach the cut
  int n = 0;
  // appends the classes of the zero bits of `sign` (bit 15 - i = accumulator i)
  auto push = [&](int t, uint32_t sign, int skip) {
    uint32_t m = ~sign & 0xffffu;
    while (__ballot(m != 0u) != 0ull) {
      if (m != 0u) {
        const int bit = 31 - __builtin_clz(m);
        m &= ~(1u << bit);
        const int c = t * kCfTile + tile_class(15 - bit, h);
        if (c < C && c != skip) {
          if (n < kCfList) list[wave][lane][n] = static_cast<uint16_t>(c);
          ++n;
        }
      }
    }
  };
  sweep([&](int t, const f32x16& acc) {
    uint32_t sign = 0u;
#pragma unroll
    for (int i = 0; i < 16; ++i)
      sign = __builtin_amdgcn_alignbit(sign, __builtin_bit_cast(uint32_t, acc[i] - cut), 31);
    push(t, sign, -1);
  });
  // The lists are the wave's own.  A row whose error is infinite is left to
  // the float64 kernel whatever it lists.
  auto publish = [&]() {
    count[wave][lane] = err < __builtin_inf() ? n : kCfList + 1;
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
    __builtin_amdgcn_wave_barrier();
  };
  publish();

  // exact logits: 16 lanes per row
  const int l16 = lane & 15, grp = lane >> 4;
  constexpr int kZ = (KS + 3) / 4;  // float4 of a row per lane
  auto load_row = [&](int rr, f32x4(&zv)[kZ]) {
    const int64_t e = row0 + rr;
    const float* row = z + (e < N ? e : N - 1) * d;
#pragma unroll
    for (int j = 0; j < kZ; ++j) {
      zv[j] = f32x4{0.f, 0.f, 0.f, 0.f};
      const int k = 4 * l16 + 64 * j;
      if (k < d) zv[j] = *reinterpret_cast<const f32x4*>(row + k);
      if constexpr (BF16_STORE) {
#pragma unroll
        for (int i = 0; i < 4; ++i) zv[j][i] = bf16_round_f32(zv[j][i]);
      }
    }
  };
  auto load_head = [&](int c, f32x4(&wv)[kZ]) {
    const float* w = W + static_cast<int64_t>(c) * d;
#pragma unroll
    for (int j = 0; j < kZ; ++j) {
      wv[j] = f32x4{0.f, 0.f, 0.f, 0.f};
      const int k = 4 * l16 + 64 * j;
      if (k < d) wv[j] = *reinterpret_cast<const f32x4*>(w + k);
    }
  };
  auto exact_logit = [&](int c, const f32x4(&wv)[kZ], const f32x4(&zv)[kZ]) {
    double s0 = 0.0, s1 = 0.0;
#pragma unroll
    for (int j = 0; j < kZ; ++j) {
      s0 = __builtin_fma(static_cast<double>(zv[j][0]), static_cast<double>(wv[j][0]), s0);
      s1 = __builtin_fma(static_cast<double>(zv[j][1]), static_cast<double>(wv[j][1]), s1);
      s0 = __builtin_fma(static_cast<double>(zv[j][2]), static_cast<double>(wv[j][2]), s0);
      s1 = __builtin_fma(static_cast<double>(zv[j][3]), static_cast<double>(wv[j][3]), s1);
    }
    return sum16(s0 + s1) + (b ? static_cast<double>(b[c]) : 0.0);
  };
  // Every row of the wave, four at a time: `begin(rr)` its state,
  // `take(state, logit, class)` for each listed class, `end(state, rr, ok)`.
  // A row is settled when both of its lanes' lists hold what was listed, at
  // least `least` classes, and it is not marked left.  Bound by the latency of
  // the row and head loads: two classes at once, the next row on its way.
  auto each_row = [&](int least, auto&& left, auto&& begin, auto&& take, auto&& end) {
    constexpr int kSteps = kCfRowsW / 4;
    f32x4 next[kZ];
    load_row(grp, next);
    for (int it = 0; it < kSteps; ++it) {
      const int rr = it * 4 + grp;
      const int n0 = count[wave][rr], n1 = count[wave][rr + 32];
      const bool ok = !left(rr) && n0 <= kCfList && n1 <= kCfList && n0 + n1 >= least;
      const int total = ok ? n0 + n1 : 0;
      auto st = begin(rr);
      f32x4 zv[kZ];
#pragma unroll
      for (int j = 0; j < kZ; ++j) zv[j] = next[j];
      for (int j = 0; j == 0 || __ballot(j < total) != 0ull; j += 2) {
        // every lane takes part; past a row's list: class 0, not looked at
        f32x4 wv[2][kZ];
        int c[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const int i = j + u;
          c[u] = i < total ? static_cast<int>(i < n0 ? list[wave][rr][i] : list[wave][rr + 32][i - n0]) : 0;
          load_head(c[u], wv[u]);
        }
        if (j == 0 && it + 1 < kSteps) load_row((it + 1) * 4 + grp, next);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const double sv = exact_logit(c[u], wv[u], zv);
          if (j + u < total) take(st, sv, c[u]);
        }
      }
      end(st, rr, ok);
    }
  };
  struct Top2 {
    double v1, v2;
    int i1, i2;
  };
  each_row(
      2, [](int) { return false; },
      [](int) { return Top2{-__builtin_inf(), -__builtin_inf(), INT_MAX, INT_MAX}; },
      [](Top2& t, double sv, int c) {
        if (sv > t.v1 || (sv == t.v1 && c < t.i1)) {
          t.v2 = t.v1;
          t.i2 = t.i1;
          t.v1 = sv;
          t.i1 = c;
        } else if (sv > t.v2 || (sv == t.v2 && c < t.i2)) {
          t.v2 = sv;
          t.i2 = c;
        }
      },
      [&](const Top2& t, int rr, bool ok) {
        const int64_t e = row0 + rr;
        if (l16 != 0) return;
        const double m = t.v1 - t.v2;
        if (e < N) {
          label_out[e] = ok ? t.i1 : kCertPending;
          if (ok) {
            if constexpr (!TIGHT) r_out[e] = f32_round_down(m / (sigma * kSqrt2));  // toward zero (r >= 0)
            if (margin_out) margin_out[e] = static_cast<float>(m);
          }
        }
        if constexpr (TIGHT) {
          const double den = ok ? row_dist[static_cast<int64_t>(t.i1) * C + t.i2] : 0.0;
          s_top[wave][rr] = t.v1;
          s_rho[wave][rr] = den > 0.0 ? m / den : __builtin_inf();
          s_lab[wave][rr] = ok ? t.i1 : -1;
        }
      });

  // tight radius: the classes whose ratio may go below the second class's.
  // sy - s' - E <= rho dist, as rho dist + s' >= sy - E in float32 with 1e-6
  // of every magnitude to spare.
  if constexpr (TIGHT) {
    __builtin_amdgcn_s_waitcnt(0xC07F);
    __builtin_amdgcn_wave_barrier();
    load_operands(std::false_type{});  // again: kept, they would take the exact sums' registers
    const int lab = s_lab[wave][c32];
    const double sy = s_top[wave][c32];
    const float rho = static_cast<float>(s_rho[wave][c32] * (1.0 + 1e-6));
    double e0;
    const double wz = row_error(e0);
    const double bound = __builtin_fabs(sy) + 2.0 * s_rho[wave][c32] * static_cast<double>(wmax) + wz;
    const double big = __builtin_fabs(sy) + wz + __builtin_fmin(static_cast<double>(bmax), bound);
    const float low = f32_round_down(sy - with_bias(e0, bound) - 1e-6 * big);
    const int64_t y = lab < 0 ? 0 : lab;
    n = 0;
    sweep([&](int t, const f32x16& acc) {
      uint32_t sign = 0u;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int c = t * kCfTile + tile_class(4 * j, h);
        f32x4 dist;
        if (head.dist) {
          // past C: the next row's values or the table behind it, against -inf logits
          dist = *reinterpret_cast<const f32x4*>(head.dist + y * head.stride + c);
        } else {
#pragma unroll
          for (int i = 0; i < 4; ++i) dist[i] = static_cast<float>(row_dist[y * C + (c + i < C ? c + i : C - 1)]);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float v = __builtin_fmaf(rho, dist[i], acc[4 * j + i]);
          sign = __builtin_amdgcn_alignbit(sign, __builtin_bit_cast(uint32_t, v - low), 31);
        }
      }
      push(t, lab < 0 ? 0xffffu : sign, lab);
    });
    publish();
    struct Least {
      double best, sy;
      int y;
    };
    each_row(
        0, [&](int rr) { return s_lab[wave][rr] < 0; },
        [&](int rr) { return Least{__builtin_inf(), s_top[wave][rr], s_lab[wave][rr]}; },
        [&](Least& t, double sv, int c) {
          const double den = row_dist[static_cast<int64_t>(t.y) * C + c];
          if (den > 0.0) {
            const double q = (t.sy - sv) / den;
            t.best = q < t.best ? q : t.best;
          }
        },
        [&](const Least& t, int rr, bool ok) {
          const int64_t e = row0 + rr;
          if (l16 != 0 || e >= N) return;
          if (ok) {
            r_out[e] = f32_round_down(t.best);  // toward zero (r >= 0)
          } else {
            label_out[e] = kCertPending;
          }
        });
  }
}

template <bool BF16_STORE, bool TIGHT, int KS>
hipError_t launch_filter(const float* z, int64_t N, int d, const float* W, const float* b, int C, double sigma,
                         const HeadImage& head, const double* row_dist, int32_t* label_out, float* r_out,
                         float* margin_out, float* norm2_out, hipStream_t s) {
  hipLaunchKernelGGL((certify_filter_kernel<BF16_STORE, TIGHT, KS>),
                     dim3(static_cast<unsigned>((N + kCfRows - 1) / kCfRows)), dim3(kCfThreads), 0, s, z, N, d, W, b, C, sigma, head, row_dist, label_out, r_out, margin_out,
                     norm2_out);
  return hipGetLastError();
}

template <bool BF16_STORE, bool TIGHT>
hipError_t launch_filter_d(const float* z, int64_t N, int d, const float* W, const float* b, int C, double sigma,
                           const HeadImage& head, const double* row_dist, int32_t* label_out, float* r_out,
                           float* margin_out, float* norm2_out, hipStream_t s) {
#define LC_CF(KS) \
  launch_filter<BF16_STORE, TIGHT, KS>(z, N, d, W, b, C, sigma, head, row_dist, label_out, r_out, margin_out, norm2_out, s)
  if (d <= 64) return LC_CF(4);
  if (d <= 128) return LC_CF(8);
  if (d <= 256) return LC_CF(16);
  return LC_CF(32);
#undef LC_CF
}

// The filter adds two launches and several dependent passes, so it pays by the
// matrix work it saves.  Measured over d = 64 .. 512, C = 40 .. 200, N = 4,096 ..
// 65,536 (float64 against filter): at N C d = 8.4e8 52.8 and 35.7 us (d = 64, C
// = 200), 56.7 and 40.6 (128, 100), 62.4 and 54.6 (256, 200), 66.9 and 67.9
// (512, 100); at half of that 34.2 and 32.8, 35.5 and 40.5, 38.8 and 46.4; at
// four times it 167 and 64, 253 and 93.  Where every row lists too many classes
// (200 near copies of one head row, N = 262,144, d = 256) the filter is spent
// for nothing: 654 and 823 us, tight 900 and 1,159.  Up to 32 classes (one tile, most of
// it padding for ten) the float64 kernel is near the memory time.
bool certify_filter_takes(int64_t N, int32_t d, int32_t C) {
  return d <= 512 && C > 32 && C <= 65536 && N < (1ll << 37) &&
         static_cast<double>(N) * static_cast<double>(C) * static_cast<double>(d) >= 8.0e8;
}

hipError_t certify_filter_run(const float* z, int64_t N, int32_t d, const float* W, const float* b, int32_t C,
                              double sigma, bool bf16, bool tight, const double* row_dist, int32_t* label_out,
                              float* r_out, float* margin_out, float* norm2_out, void* head_ws, hipStream_t s) {
  const HeadImage head = head_layout(head_ws, C, d);
  const int pad = (C + kCfTile - 1) / kCfTile * kCfTile;
  hipLaunchKernelGGL(head_image_kernel, dim3(static_cast<unsigned>(pad / kCfWaves)), dim3(kCfThreads), 0, s, W, b, C, d,
                     pad, head);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (tight && head.dist) {
    const int64_t cells = static_cast<int64_t>(C) * head.stride;
    hipLaunchKernelGGL(dist32_kernel, dim3(static_cast<unsigned>((cells + kCfThreads - 1) / kCfThreads)),
                       dim3(kCfThreads), 0, s, row_dist, C, head);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
#define LC_CF(B, T) \
  launch_filter_d<B, T>(z, N, d, W, b, C, sigma, head, row_dist, label_out, r_out, margin_out, norm2_out, s)
  if (bf16) return tight ? LC_CF(true, true) : LC_CF(true, false);
  return tight ? LC_CF(false, true) : LC_CF(false, false);
#undef LC_CF
}

}  // namespace lc
