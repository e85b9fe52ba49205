// Naive Bayes scoring of 16 classes with a BF16 table, labels and log
// posteriors, on the matrix cores: the benchmark's precision configuration.
// The general kernel (nb_score_tile.hip) serves every other class count (but for
// short rows of a few classes, nb_score_few.hip), the FP32 table and raw scores; here
// the whole table stays in LDS, which keeps the
// wave's load stream free of table slices and barriers: 360 against 368-376 us
// for 500,000 FP8 files at F = 4096, 191 against 196-200 us for 800,000 byte
// files at F = 1000.
//
// s~[file, class] = sum_f g(x_f) W~[class, f] is a skinny GEMM (M = files, N =
// classes, K = features).  Feature bytes (uint8 counts or FP8-e4m3) convert
// exactly to BF16; products accumulate in FP32 (v_mfma_f32_16x16x32_bf16).
// The K order inside a tile is free (the same permutation on A and B leaves
// the sum unchanged), so each lane takes 16 contiguous feature bytes of its
// file per 64-feature window (lane group q = lane / 16 takes bytes 16q .. 16q +
// 15) and feeds two MFMAs with them; the matching B fragment is 8 contiguous
// BF16 entries of one class row.  After the K loop the 16x16 accumulator tiles
// (lane l holds rows 4*(l/16)..+3 of column l%16) are reduced across the 16
// lanes of each column group for the max / log-sum-exp epilogue; labels take
// the lowest class index among maxima.
#include <algorithm>
#include <type_traits>

#include "nb_internal.hpp"
#include "nb_mfma.hpp"

namespace nb {
namespace {

constexpr int kWindow = 64;                 // features per window (one 16-byte load per lane)

struct ScoreMArgs {
  const uint8_t* x;
  int64_t ld_bytes;
  int64_t n;
  int64_t total_bytes;
  const uint16_t* rows16;   // [16][Fp] class-major BF16 rows
  const float* row_bias;    // [16]
  int32_t* labels;
  float* log_post;
  int32_t F, Fp;
  int64_t nfast;            // leading wave tiles with every row and load in bounds
};

// One column tile (16 score rows) and Fp <= 4096.  A wave tile is 16 files; a group is 512 features.  Each group's loads
// read 512 contiguous bytes of each of the 16 files (a wave instruction
// covers 2 files x 512 bytes, eight instructions per group) instead of the
// A-operand layout's 16 files x 64 bytes, and the wave transposes them
// through a private 8 KB LDS stage into the operand layout.  The run length
// per file is what counts on HBM: with the same stage scheme, 128 contiguous
// bytes per file (32 files per tile) held the kernel at 69% of peak, 256
// bytes gave the same, 512 bytes 78%, whatever the waves per CU (8 or 16) or
// the groups in flight (2 to 5); 1024 bytes leave room for only two waves
// per CU.  LDS holds the whole BF16 table (16 rows x Fp, no padding: the
// 16-byte granules of row r are XOR-swizzled by r, so the 16 rows read by
// one B fragment fall in distinct banks) plus the four waves' stages; granule
// p of file r of a stage sits at p ^ (r & 15) (p ^ ((r >> 1) & 7) for
// 128-byte groups), which keeps both the line-shaped writes and the
// operand-shaped reads free of bank conflicts.  Loads run kStageDepth - 1
// groups ahead in registers, across tile boundaries.
constexpr int kStageWaves = 4;
constexpr int kStageThreads = 64 * kStageWaves;
constexpr int kStageMT = 1;                       // 16-file MFMA tiles per wave tile
constexpr int kStageFiles = 16 * kStageMT;        // files per wave tile
constexpr int kStageGB = 512;                     // features (bytes) per file per group
constexpr int kStageWin = kStageGB / kWindow;     // 64-feature windows per group
constexpr int kStageNG = kStageGB / 16;           // 16-byte granules per file per group
constexpr int kStageFPI = 1024 / kStageGB;        // files per wave load instruction
constexpr int kStageLoads = kStageFiles / kStageFPI;   // 16-byte loads per lane per group
constexpr int kStageBytes = kStageFiles * kStageGB;
static_assert(kStageGB >= 128 && kStageGB <= 1024 && kStageFiles % kStageFPI == 0, "stage shape");
constexpr int kStageDepth = 3;
// Destination of outputs the caller did not request, of the lanes that hold no
// label and of absent rows: the epilogue stores unconditionally so that the number of
// memory operations in flight stays known at compile time.
__device__ int32_t g_stage_sink_label[64];
__device__ float g_stage_sink_post[64 * 16];

template <int XT, bool BIN>
__global__ __launch_bounds__(kStageThreads) void scoreM_stage_kernel(ScoreMArgs a) {
  extern __shared__ __attribute__((aligned(16))) dev::u32x4 lds4[];
  dev::u32x4* tbl = lds4;                                    // [16][Fp / 8] granules, swizzled
  const int gpr = a.Fp / 8;                                  // granules per table row
  for (int i = threadIdx.x; i < 16 * gpr; i += kStageThreads) {
    const int r = i / gpr, g = i - r * gpr;
    tbl[r * gpr + (g ^ r)] = *reinterpret_cast<const dev::u32x4*>(a.rows16 + (int64_t)r * a.Fp + 8 * g);
  }
  __syncthreads();

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  dev::u32x4* stg = lds4 + 16 * gpr + wave * (kStageBytes / 16);
  const int col = lane & 15, q = lane >> 4;
  const int64_t ld = a.ld_bytes;
  const int64_t wave_id = (int64_t)blockIdx.x * kStageWaves + wave;
  const int64_t nwaves = (int64_t)gridDim.x * kStageWaves;
  const int ngroups = (a.F + kStageGB - 1) / kStageGB;
  const float bias = a.row_bias[col];
  // load lane layout: instruction j covers files kStageFPI j + lane / kStageNG,
  // granule lane % kStageNG
  const int lr = lane / kStageNG, lp = lane % kStageNG;
  uint32_t rel[kStageLoads];
#pragma unroll
  for (int j = 0; j < kStageLoads; ++j) rel[j] = (uint32_t)((kStageFPI * j + lr) * ld) + 16 * lp;
  int wpos[kStageLoads];
#pragma unroll
  for (int j = 0; j < kStageLoads; ++j) wpos[j] = stage_granule<kStageNG>(kStageFPI * j + lr, lp);
  // operand lane layout: tile mt, window u -> file 16 mt + col, granule 4 u + q
  int rpos[kStageMT][kStageWin];
#pragma unroll
  for (int mt = 0; mt < kStageMT; ++mt)
#pragma unroll
    for (int u = 0; u < kStageWin; ++u) rpos[mt][u] = stage_granule<kStageNG>(16 * mt + col, 4 * u + q);

  f32x4 acc[kStageMT][1];
  auto zero_acc = [&]() {
#pragma unroll
    for (int mt = 0; mt < kStageMT; ++mt) acc[mt][0] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  };
  // transpose one group through the stage and multiply it into acc
  auto compute_group = [&](int g, const dev::u32x4 (&src)[kStageLoads]) {
    // the previous group's operand reads are done before the stage is
    // rewritten: LDS operations of a wave complete in order
#pragma unroll
    for (int j = 0; j < kStageLoads; ++j) stg[wpos[j]] = src[j];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int u = 0; u < kStageWin; ++u) {
      const int f0 = g * kStageGB + u * kWindow;         // first feature of the window
      dev::u32x4 av[kStageMT][2];
#pragma unroll
      for (int mt = 0; mt < kStageMT; ++mt) {
        dev::u32x4 xv = stg[rpos[mt][u]];
        if (XT == NB_X_FP8 && f0 + 16 * q + 16 > a.F) {   // NaN encodings past the last feature
          const int nv = max(0, a.F - (f0 + 16 * q));
#pragma unroll
          for (int d = 0; d < 4; ++d) {
            const int nb = min(4, max(0, nv - 4 * d));
            xv[d] &= (nb >= 4) ? ~0u : ((1u << (8 * nb)) - 1u);
          }
        }
        float g16[16];
        to_bf16<XT, BIN>(xv, av[mt][0], av[mt][1], g16);
      }
      const int G = (f0 + 16 * q) / 8;                    // table granule of this lane's k-group
      const dev::u32x4 b0 = tbl[col * gpr + (G ^ col)];
      const dev::u32x4 b1 = tbl[col * gpr + ((G + 1) ^ col)];
#pragma unroll
      for (int mt = 0; mt < kStageMT; ++mt) {
        acc[mt][0] = mfma(av[mt][0], b0, acc[mt][0]);
        acc[mt][0] = mfma(av[mt][1], b1, acc[mt][0]);
      }
    }
  };
  // Epilogue of a tile, 16 classes in the 16 columns (lane: files 4 q + i of
  // class col): max and lowest arg-max over the 16 lanes of a file, log-sum-exp.
  // A file whose sums are all NaN (an FP8 NaN among its features) compares with
  // nothing and keeps label 0.  FULL: every row is present and every store is
  // issued (to a sink when the output was not requested).
  const bool want_lab = a.labels != nullptr, want_lp = a.log_post != nullptr;
  auto finish = [&](int64_t row0, auto full) {
    constexpr bool FULL = decltype(full)::value;
#pragma unroll
    for (int mt = 0; mt < kStageMT; ++mt) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int64_t row = row0 + 16 * mt + 4 * q + i;
        const float sv = acc[mt][0][i] + bias;
        float m = sv;
        int best = col;
#pragma unroll
        for (int sh = 1; sh < 16; sh <<= 1) {
          const float om = __shfl_xor(m, sh);
          const int ob = __shfl_xor(best, sh);
          if (om > m || (om == m && ob < best)) {
            m = om;
            best = ob;
          }
        }
        float z = __expf(sv - m);
#pragma unroll
        for (int sh = 1; sh < 16; sh <<= 1) z += __shfl_xor(z, sh);
        const float lse = m + __logf(z);
        const bool present = FULL || row < a.n;
        int32_t* pl = (want_lab && present && col == 0) ? a.labels + row : g_stage_sink_label + lane;
        float* pp = (want_lp && present) ? a.log_post + row * 16 + col : g_stage_sink_post + lane;
        *pl = best;
        *pp = sv - lse;
      }
    }
  };

  // ---- full tiles [0, a.nfast): one pipelined stream of (tile, group)
  // units; loads run kStageDepth - 1 units ahead and cross tile boundaries.
  // The prefetch past the last unit re-reads the last unit (an L2 hit).
  const int my_tiles = (a.nfast > wave_id) ? (int)((a.nfast - wave_id + nwaves - 1) / nwaves) : 0;
  const int units = my_tiles * ngroups;
  auto issue = [&](int k, dev::u32x4 (&dst)[kStageLoads]) {
    k = min(k, units - 1);
    const int it = k / ngroups, g = k - it * ngroups;
    const int64_t wbase = (wave_id + (int64_t)it * nwaves) * kStageFiles * ld + (int64_t)g * kStageGB;
    const auto rsrc = dev::make_rsrc(a.x + wbase, a.total_bytes - wbase);
#pragma unroll
    for (int j = 0; j < kStageLoads; ++j) dst[j] = dev::buffer_load16(rsrc, rel[j]);
    __builtin_amdgcn_sched_barrier(0);
  };
  int cg = 0, ct = 0;
  auto consume = [&](const dev::u32x4 (&src)[kStageLoads]) {
    compute_group(cg, src);
    if (++cg == ngroups) {
      finish((wave_id + (int64_t)ct * nwaves) * kStageFiles, std::true_type{});
      zero_acc();
      cg = 0;
      ++ct;
    }
  };
  zero_acc();
  if (units > 0) {
    // kStageDepth register buffers in rotation: unit k + kStageDepth - 1 is
    // issued just before unit k is consumed
    dev::u32x4 buf[kStageDepth][kStageLoads];
#pragma unroll
    for (int d = 0; d < kStageDepth - 1; ++d) issue(d, buf[d]);
    bool done = false;
    for (int k = 0; !done; k += kStageDepth) {
#pragma unroll
      for (int d = 0; d < kStageDepth; ++d) {
        if (!done) {
          issue(k + d + kStageDepth - 1, buf[(d + kStageDepth - 1) % kStageDepth]);
          consume(buf[d]);
          if (k + d + 1 >= units) done = true;
        }
      }
    }
  }

  // ---- remaining tiles: guarded loads, partial rows
  const int64_t nwtile = (a.n + kStageFiles - 1) / kStageFiles;
  for (int64_t wt = a.nfast + wave_id; wt < nwtile; wt += nwaves) {
    const int64_t row0 = wt * kStageFiles;
    zero_acc();
    for (int g = 0; g < ngroups; ++g) {
      dev::u32x4 v[kStageLoads];
      const int64_t wbase = row0 * ld + (int64_t)g * kStageGB;
#pragma unroll
      for (int j = 0; j < kStageLoads; ++j) {
        v[j] = dev::u32x4{0u, 0u, 0u, 0u};
        const int64_t off = wbase + rel[j];
        if (row0 + kStageFPI * j + lr < a.n) v[j] = dev::load16_guarded(a.x + off, a.total_bytes - off);
      }
      compute_group(g, v);
    }
    finish(row0, std::false_type{});
  }
}

int max_lds_per_block() {
  static int v = 0;
  if (v == 0) {
    int dev = 0, b = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&b, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) == hipSuccess && b > 0)
      v = b;
    else
      v = 64 * 1024;
  }
  return v;
}

}  // namespace

// Whether the staged kernel serves a call: 16 classes on the BF16 table, no raw
// scores, and a table that fits LDS beside the stages.
bool score16_staged(const nb_model* m, const nb_layout& L, int32_t wtype, const float* scores) {
  const size_t lds = (size_t)16 * L.padded_features * sizeof(uint16_t) + (size_t)kStageWaves * kStageBytes;
  return wtype == NB_W_BF16 && m->n_classes == 16 && !scores && lds <= (size_t)max_lds_per_block();
}

int launch_score16_staged(const nb_model* m, const nb_layout& L, const void* x, int32_t xtype, int64_t n, int64_t ld,
                          int32_t* labels, float* log_post, hipStream_t s) {
  const bool bin = m->kind == NB_BERNOULLI;
  const uint8_t* base = static_cast<const uint8_t*>(m->dev);
  ScoreMArgs a;
  a.x = static_cast<const uint8_t*>(x);
  a.ld_bytes = ld;
  a.n = n;
  a.total_bytes = (n - 1) * ld + m->n_features;
  a.rows16 = reinterpret_cast<const uint16_t*>(base + L.off_form_bf16);
  a.row_bias = reinterpret_cast<const float*>(base + L.off_form_bias);
  a.labels = labels;
  a.log_post = log_post;
  a.F = m->n_features;
  a.Fp = L.padded_features;
  // leading tiles whose rows all exist and whose group loads stay in the buffer
  const int64_t span = (int64_t)((a.F + kStageGB - 1) / kStageGB) * kStageGB;
  const int64_t full = n / kStageFiles;
  const int64_t rmax = (a.total_bytes >= span) ? (a.total_bytes - span) / a.ld_bytes : -1;
  a.nfast = std::max<int64_t>(0, std::min(full, (rmax + 1) / kStageFiles));
  const size_t lds = (size_t)16 * L.padded_features * sizeof(uint16_t) + (size_t)kStageWaves * kStageBytes;
  const void* sf = (xtype == NB_X_U8) ? (bin ? reinterpret_cast<const void*>(scoreM_stage_kernel<NB_X_U8, true>)
                                              : reinterpret_cast<const void*>(scoreM_stage_kernel<NB_X_U8, false>))
                                      : (bin ? reinterpret_cast<const void*>(scoreM_stage_kernel<NB_X_FP8, true>)
                                              : reinterpret_cast<const void*>(scoreM_stage_kernel<NB_X_FP8, false>));
  NB_HIP_CHECK(hipFuncSetAttribute(sf, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  const int64_t nwtile = (n + kStageFiles - 1) / kStageFiles;
  const int64_t want = (nwtile + kStageWaves - 1) / kStageWaves;
  const int64_t cap = (int64_t)resident_per_cu(sf, kStageThreads, lds) * device_cu_count();
  const unsigned grid = (unsigned)std::max<int64_t>(1, std::min(want, cap));
  void* args[] = {&a};
  NB_HIP_CHECK(hipLaunchKernel(sf, dim3(grid), dim3(kStageThreads), args, lds, s));
  NB_HIP_CHECK(hipGetLastError());
  return NB_OK;
}

}  // namespace nb
