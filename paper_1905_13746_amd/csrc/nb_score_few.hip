// Naive Bayes scoring of short rows by a few classes (three to seven), on the
// vector ALUs (paper, section 4: the class with the highest posterior wins).
//
// A file of at most 128 bytes is a few operations per class, and what bounds the
// call is what a file costs beside them.  The matrix-core kernel (nb_score_tile.hip)
// reduces each of its files over 16 lanes, whatever the class count: 0.055 ns per
// file, above the 0.022-0.05 ns that HBM takes for the row and its outputs.  Here
// each lane owns ONE file: all lanes of a wave step through the same feature at the
// same time, so the table value of (feature, class) is the same for the whole wave
// and comes from LDS as a broadcast read, and the decision is a loop over the
// lane's own sums.  Feature bytes are staged per wave through LDS: a coalesced load
// of 64 files x 64 bytes, then each lane reads its own file's 64 bytes.
//
// Sums are two-level: the features of 64 bytes accumulate into an inner partial that
// is added to the running total, in the order of the features alone.
#include <algorithm>

#include "nb_device.hpp"
#include "nb_internal.hpp"

namespace nb {
namespace {

constexpr int kWaves = 4;
constexpr int kThreads = 64 * kWaves;
constexpr int kStepBytes = 64;      // bytes of each file per sub-step
constexpr int kRowBytes = 128;      // bytes of the longest row
constexpr int kRowPad = 16;         // LDS row padding (bank spread)
constexpr int kXRow = kStepBytes + kRowPad;

struct ScoreFewArgs {
  const uint8_t* x;
  int64_t ld_bytes;
  int64_t n;
  int64_t total_bytes;
  const float* rows32;       // [P+1][Fp] class-major scoring rows
  const uint16_t* rows16;    // same, BF16
  const float* row_bias;     // [P+1]
  int32_t* labels;
  float* log_post;
  float* scores;
  int32_t F, Fp, C, wt;
  int32_t ns;                // rows used: C, or C + 1 with the aux row (index C)
};

__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// NS: sums per file, >= a.ns (the C class-centred rows, whose differences are the
// posteriors', plus the aux row that restores the raw scores; extra sums see zero
// rows).
template <int XT, int NS, bool BIN>
__global__ __launch_bounds__(kThreads) void score_few_kernel(ScoreFewArgs a) {
  constexpr int EB = (XT == NB_X_I32) ? 4 : 1;
  constexpr int KS = kStepBytes / EB;          // features per sub-step
  constexpr int kFeatures = kRowBytes / EB;
  static_assert(NS % 4 == 0, "float4 table reads");
  __shared__ __attribute__((aligned(16))) float tbl[kFeatures * NS];
  __shared__ __attribute__((aligned(16))) uint8_t xs[kWaves][64 * kXRow];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int C = a.C;
  const int64_t ld = a.ld_bytes;
  // the table, feature-major
  for (int i = threadIdx.x; i < kFeatures * NS; i += kThreads) {
    const int s = i / kFeatures, f = i % kFeatures;
    const int64_t src = (int64_t)s * a.Fp + f;      // Fp >= 1024: zeros past the last feature
    tbl[f * NS + s] = (s >= a.ns) ? 0.0f : (a.wt == NB_W_BF16) ? dev::bf16_to_f32(a.rows16[src]) : a.rows32[src];
  }
  float bias[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) bias[s] = s < a.ns ? a.row_bias[s] : 0.0f;
  __syncthreads();

  const int64_t ntile = (a.n + kThreads - 1) / kThreads;
  for (int64_t tile = blockIdx.x; tile < ntile; tile += gridDim.x) {
    const int64_t row0 = tile * kThreads + wave * 64;     // this wave's 64 files
    float acc[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) acc[s] = 0.0f;

    for (int ks = 0; ks < a.F; ks += KS) {
      // stage 64 files x 64 bytes: piece p = lane + 64 t -> (row p/4, 16-byte column p%4);
      // one wave-uniform buffer resource per sub-step, per-lane 32-bit offsets
      const int64_t wbase = row0 * ld + (int64_t)ks * EB;
      const auto rsrc = dev::make_rsrc(a.x + wbase, a.total_bytes - wbase);
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int p = lane + 64 * t;
        const int r = p >> 2, c16 = p & 3;
        const int64_t row = row0 + r;
        dev::u32x4 v = {0u, 0u, 0u, 0u};
        if (row < a.n) {
          const int64_t rel = (int64_t)r * ld + 16 * c16;
          if (wbase + rel + 16 <= a.total_bytes) {
            v = dev::buffer_load16(rsrc, (uint32_t)rel);
          } else {
            v = dev::load16_guarded(a.x + wbase + rel, a.total_bytes - (wbase + rel));
          }
        }
        *reinterpret_cast<dev::u32x4*>(&xs[wave][r * kXRow + 16 * c16]) = v;
      }
      wave_lds_sync();
      dev::u32x4 mine[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) mine[q] = *reinterpret_cast<const dev::u32x4*>(&xs[wave][lane * kXRow + 16 * q]);
      wave_lds_sync();
      // FP8 bytes past the last feature may encode NaN: clear them
      const int nvalid = min(KS, a.F - ks);
      if (XT == NB_X_FP8 && nvalid < KS) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int d = 0; d < 4; ++d) {
            const int b0 = 16 * q + 4 * d;
            const int nb = min(4, max(0, nvalid - b0));
            mine[q][d] &= (nb >= 4) ? ~0u : ((1u << (8 * nb)) - 1u);
          }
      }
      float inner[NS];
#pragma unroll
      for (int s = 0; s < NS; ++s) inner[s] = 0.0f;
      const float* tb = tbl + ks * NS;
#pragma unroll
      for (int e = 0; e < KS; ++e) {
        float g;
        if (XT == NB_X_I32) {
          g = (float)(int32_t)mine[e >> 2][e & 3];
        } else if (XT == NB_X_U8) {
          g = (float)((mine[e >> 4][(e >> 2) & 3] >> (8 * (e & 3))) & 0xFFu);
        } else {
          const uint32_t w = mine[e >> 4][(e >> 2) & 3];
          g = ((e & 2) ? __builtin_amdgcn_cvt_pk_f32_fp8(w, true) : __builtin_amdgcn_cvt_pk_f32_fp8(w, false))[e & 1];
        }
        // presence: a clamp to [0, 1] for integer counts (folds into the
        // conversion), a compare for FP8 values
        if (BIN) g = (XT == NB_X_FP8) ? (g > 0.0f ? 1.0f : 0.0f) : __builtin_amdgcn_fmed3f(g, 0.0f, 1.0f);
        const float* te = tb + e * NS;
#pragma unroll
        for (int s4 = 0; s4 < NS; s4 += 4) {
          const float4 w4 = *reinterpret_cast<const float4*>(te + s4);
          inner[s4 + 0] = fmaf(g, w4.x, inner[s4 + 0]);
          inner[s4 + 1] = fmaf(g, w4.y, inner[s4 + 1]);
          inner[s4 + 2] = fmaf(g, w4.z, inner[s4 + 2]);
          inner[s4 + 3] = fmaf(g, w4.w, inner[s4 + 3]);
        }
      }
#pragma unroll
      for (int s = 0; s < NS; ++s) acc[s] += inner[s];
    }

    // epilogue: one file per lane
    const int64_t row = row0 + lane;
    if (row < a.n) {
      float sc[NS];
#pragma unroll
      for (int s = 0; s < NS; ++s) sc[s] = acc[s] + bias[s];
      float m = -INFINITY;
      int best = 0;
#pragma unroll
      for (int s = 0; s < NS; ++s)
        if (s < C && sc[s] > m) {
          m = sc[s];
          best = s;
        }
      float z = 0.0f;
#pragma unroll
      for (int s = 0; s < NS; ++s)
        if (s < C) z += __expf(sc[s] - m);
      const float lse = m + __logf(z);
      if (a.labels) a.labels[row] = best;
      if (a.log_post) {
#pragma unroll
        for (int s = 0; s < NS; ++s)
          if (s < C) a.log_post[row * C + s] = sc[s] - lse;
      }
      if (a.scores) {
        float aux = 0.0f;
#pragma unroll
        for (int s = 0; s < NS; ++s)
          if (s == C) aux = sc[s];
#pragma unroll
        for (int s = 0; s < NS; ++s)
          if (s < C) a.scores[row * C + s] = sc[s] + aux;
      }
    }
  }
}

using KernelFn = void (*)(ScoreFewArgs);

template <int XT>
KernelFn pick_few(int ns, bool bin) {
  if (ns <= 4) return bin ? score_few_kernel<XT, 4, true> : score_few_kernel<XT, 4, false>;
  return bin ? score_few_kernel<XT, 8, true> : score_few_kernel<XT, 8, false>;
}

}  // namespace

// Whether these kernels serve a call: where they were the faster ones for some n and
// hardly the slower ones for any (the choice must not depend on n: nor may the order
// of a file's sums).  1,000,000 files, us here and on the matrix cores: bytes, 3
// classes, F = 4 22 and 54, F = 64 30 and 55, F = 128 54 and 55 (300,000: 16 and 20),
// F = 192 76 and 72; 5 classes, F = 64 49 and 55, F = 128 77 and 57; 7 classes, F = 16
// 53 and 55; int32, 7 classes, F = 8 47 and 57, F = 32 73 and 59.
bool score_few(const nb_model* m, int32_t xtype) {
  const int C = m->n_classes, bytes = m->n_features * elem_bytes(xtype);
  return C <= 4 ? bytes <= kRowBytes : bytes <= 64 && C <= (xtype == NB_X_I32 ? 7 : 5);
}

int launch_score_few(const nb_model* m, const nb_layout& L, const void* x, int32_t xtype, int64_t n, int64_t ld,
                     int32_t wtype, int32_t* labels, float* log_post, float* scores, hipStream_t s) {
  const int ns = m->n_classes + (scores ? 1 : 0);
  const bool bin = m->kind == NB_BERNOULLI;
  const KernelFn fn = xtype == NB_X_U8    ? pick_few<NB_X_U8>(ns, bin)
                      : xtype == NB_X_I32 ? pick_few<NB_X_I32>(ns, bin)
                                          : pick_few<NB_X_FP8>(ns, bin);
  const int eb = elem_bytes(xtype);
  const uint8_t* base = static_cast<const uint8_t*>(m->dev);
  ScoreFewArgs a;
  a.x = static_cast<const uint8_t*>(x);
  a.ld_bytes = ld * eb;
  a.n = n;
  a.total_bytes = ((n - 1) * ld + m->n_features) * (int64_t)eb;
  a.rows32 = reinterpret_cast<const float*>(base + L.off_form_f32);
  a.rows16 = reinterpret_cast<const uint16_t*>(base + L.off_form_bf16);
  a.row_bias = reinterpret_cast<const float*>(base + L.off_form_bias);
  a.labels = labels;
  a.log_post = log_post;
  a.scores = scores;
  a.F = m->n_features;
  a.Fp = L.padded_features;
  a.C = m->n_classes;
  a.wt = wtype;
  a.ns = ns;
  const int64_t ntile = (n + kThreads - 1) / kThreads;
  const int64_t cap = (int64_t)resident_per_cu(reinterpret_cast<const void*>(fn), kThreads, 0) * device_cu_count();
  const unsigned grid = (unsigned)std::max<int64_t>(1, std::min(ntile, cap));
  hipLaunchKernelGGL(fn, dim3(grid), dim3(kThreads), 0, s, a);
  NB_HIP_CHECK(hipGetLastError());
  return NB_OK;
}

}  // namespace nb
