// Naive Bayes scoring for more than two classes on the matrix cores (paper,
// section 4: the class with the highest posterior wins; here C >= 3, e.g. malware
// families), with the FP32 or the BF16 table (short rows of a few classes run in
// nb_score_few.hip, 16 classes on the BF16 table without raw scores in
// nb_score_mfma.hip).
//
// s[file, class] = sum_f g(x_f) W[class, f] is a skinny GEMM (M = files, N =
// classes, K = features).  Byte counts and FP8-e4m3 values are exact in BF16.
// A BF16 table feeds v_mfma_f32_16x16x32_bf16 directly; an FP32 table entry
// (24 significant bits) is the exact sum of three BF16 numbers (its leading 8
// bits, the next 8 and the last 8), so three products with FP32 accumulation
// give what an FP32 multiply-add gives: every product is exact and the sums
// round in FP32.  The vector ALUs need C + 1 operations per feature byte, which
// held 16 classes at 0.85 TB/s of features; three MFMAs per 16 classes cost a
// quarter of the matrix cores' time at the rate HBM delivers the bytes.  int32
// features go through v_mfma_f32_16x16x4_f32 (FP32 products and sums, a third of
// the matrix cores' time at that rate), four of them per 16-byte load.
//
// What bounds it is HBM and, with the FP32 table, the waits that two waves per SIMD
// leave open.  Counters of 4,000,000 files of 16 classes, F = 4096 (5.4 TB/s, HBM
// traffic 1.001 x): vector ALUs busy 44% of the cycles, LDS 36% without a bank
// conflict, matrix cores 22%; a wave waits for 29% of its time, for 7% on LDS.  16 files
// share each table read; 32 files per unit halve the LDS traffic but leave one wave
// per SIMD the registers, and measured slower (415 against 345 us).  A wave's unit is 16
// files x KB bytes, loaded as KB contiguous bytes of each file (512 where the
// table leaves room: 256-byte runs took 415 us for the same files), one unit
// ahead in registers, and transposed through the wave's private LDS stage, SS
// bytes at a time, into the operand layout.  The table of a slice's features
// is split into its BF16 parts while it is staged in LDS, two slices deep: a
// workgroup walks the slices with PT units of files per wave, so a slice is
// staged once per 16 PT files of each of its waves.  A table of at most two
// slices stays in LDS and the waves run without barriers.
//
// Measured (us; byte features but for the last three), beside the other design
// tried for each: one file per lane on the vector ALUs for the FP32 table and int32
// features, matrix cores on 64-byte loads without a stage for the BF16 table.
//                                                     other   this
//   FP32, 16 classes, F = 4096, 400,003 files         1,718    354  (4.6 TB/s)
//   the same with raw scores                          1,980    362
//   FP32, 20 classes, F = 2000, 300,000 files           905    204
//   FP32, 7 classes, F = 1000, 600,000 files            347    152
//   FP32, 16 classes, F = 1000, 2,000 files             128     13
//   BF16, 40 classes, F = 1000, 400,001 files, scores   214    127
//   BF16, 100 classes, F = 2000, 150,000 files          354    154
//   int32, 7 classes, F = 2964, 67,476 files, scores    645    230
//   int32, 16 classes, F = 1792, 111,607 files          484    180
//   int32, 24 classes, F = 1000, 100,000 files          887    158
//
// Sums: the products of 128 consecutive features (16 int32 ones) go to fresh
// accumulators (leading parts and lower parts apart), whose sum is added to the
// file's running totals: a term passes through few roundings, and the order depends on
// the feature index alone.  Sixteen classes on the BF16 table are the exception
// (ROW): where the kernel of nb_score_mfma.hip takes the calls without raw scores,
// the ones with them sum as it does, in one accumulator per row and with its order of
// the log-sum-exp, so that what is asked for beside them changes no label and no log
// posterior.
#include <algorithm>
#include <type_traits>

#include "nb_internal.hpp"
#include "nb_mfma.hpp"

namespace nb {
namespace {

constexpr int kWindow = 64;      // bytes of a file per 16-byte load of the operand layout
constexpr int kFlush = 128;      // byte features per fresh accumulator

// Waves per SIMD that a kernel's registers have to leave room for: the kernels of
// short rows live by occupancy (two of a workgroup's waves per SIMD otherwise).
constexpr int tile_waves(int NT, int KB, int NW, bool AUX) { return NT == 1 && KB <= 256 ? (AUX ? 3 : 4) : NW / 4; }

struct ScoreTileArgs {
  const uint8_t* x;
  int64_t ld_bytes;
  int64_t n;
  int64_t total_bytes;
  const void* rows;         // [P+1][Fp] class-major rows, FP32 (three parts) or BF16 (one)
  const float* row_bias;    // [P+1]
  int32_t* labels;
  float* log_post;
  float* scores;
  int32_t F, Fp, C, ns;     // ns: rows used (C, or C + 1 with the aux row)
  int64_t nfast;            // leading files whose loads (whole slices) stay in the buffer
  int64_t wide_tiles;       // workgroup tiles of PT units per wave; single-unit tiles follow
};

// A lane value whose uses the compiler must not move out of the enclosing
// loop: the addresses derived from it are computed where they are used instead
// of being held in registers across the whole kernel.
__device__ __forceinline__ int here(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

// The value of the lane N places on in its row of 16 (a vector ALU operand
// modifier: no LDS traffic).
template <int N>
__device__ __forceinline__ float ror16(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x120 + N, 0xf, 0xf, true));
}
template <int N>
__device__ __forceinline__ int ror16(int v) {
  return __builtin_amdgcn_update_dpp(0, v, 0x120 + N, 0xf, 0xf, true);
}

// The four lanes' sum, then eight's, then sixteen's: the order of a butterfly over
// lane distances 1, 2, 4 and 8 (equal within the lanes already summed, so mirrored
// lanes stand for the exchanged ones).
__device__ __forceinline__ float butterfly16(float v) {
  v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xf, 0xf, true));    // lanes 1 0 3 2
  v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x4E, 0xf, 0xf, true));    // lanes 2 3 0 1
  v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x141, 0xf, 0xf, true));   // half row mirror
  v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x140, 0xf, 0xf, true));   // row mirror
  return v;
}

template <int N>
__device__ __forceinline__ void argmax_step(float& m, int& best) {
  const float om = ror16<N>(m);
  const int ob = ror16<N>(best);
  const bool take = om > m || (om == m && ob < best);
  m = take ? om : m;
  best = take ? ob : best;
}

// NT: 16-class column tiles.  NP: BF16 parts of a table entry (3: FP32 table,
// 1: BF16 table; int32 features: entries are staged in FP32 from either).  MT:
// 16-file tiles of a unit.  PT: units per wave of a wide workgroup tile (even:
// the two load buffers alternate), or 1: no wide tiles.  KB: bytes per file of a slice.  SS: bytes per
// file of the stage.  NW: waves.  AUX: the raw scores' aux row, which would need a column
// tile of its own, is contracted on the vector ALUs (one FMA per byte, a
// quarter of a lane's operations) from the FP32 values at hand.  ROW: one
// accumulator per row.
template <int XT, int NT, int NP, bool BIN, int MT, int PT, int KB, int SS, int NW, bool AUX, bool ROW>
__global__ __launch_bounds__(64 * NW, tile_waves(NT, KB, NW, AUX)) void score_tile_kernel(ScoreTileArgs a) {
  constexpr bool I32 = XT == NB_X_I32;
  constexpr int EB = I32 ? 4 : 1;           // bytes per feature
  constexpr int KS = KB / EB;               // features per slice
  constexpr int WF = kWindow / EB;          // features per window
  static_assert(!ROW || (NP == 1 && !I32), "one accumulator");
  static_assert((PT == 1 || PT % 2 == 0) && SS % kFlush == 0 && KB % SS == 0 && 1024 % KB == 0, "tile shape");
  constexpr int kThreads = 64 * NW;
  constexpr int GF = 16 * MT;               // files per unit
  constexpr int NG = SS / 16;               // granules per file of the stage
  constexpr int FPI = 1024 / SS;            // files per wave load instruction
  constexpr int NLS = GF / FPI;             // loads per lane per stage
  constexpr int NL = KB / SS * NLS;         // loads per lane per unit
  constexpr int TE = I32 ? 4 : 8;           // table entries per granule: FP32 or BF16
  constexpr int GPR = KS / TE;              // table granules per row of a slice
  constexpr int kPart = 16 * NT * GPR;      // granules of one part of a slice
  constexpr int NPS = I32 ? 1 : NP;         // parts staged
  constexpr int kSlice = NPS * kPart;
  constexpr int kAcc = NPS == 3 ? 2 : 1;     // accumulators: leading parts, lower parts
  constexpr int TG = (kPart + kThreads - 1) / kThreads;   // table granules staged per thread
  constexpr bool kWhole = kPart % kThreads == 0;           // else the last ones are absent
  // [2][NPS][16 NT][GPR], the stages, AUX: [2][KS] floats
  extern __shared__ __attribute__((aligned(16))) dev::u32x4 lds4[];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  dev::u32x4* const stg = lds4 + 2 * kSlice + wave * (GF * NG);
  float* const auxt = reinterpret_cast<float*>(lds4 + 2 * kSlice + NW * (GF * NG));
  const int col = lane & 15, q = lane >> 4;
  const int lr = lane / NG, lp = lane % NG;
  const int64_t ld = a.ld_bytes;
  const int nsl = (a.F + KS - 1) / KS, row_bytes = a.F * EB;
  const bool resident = nsl <= 2;

  // ---- table slices
  const auto trsrc = dev::make_rsrc(a.rows, (int64_t)a.ns * a.Fp * (NP == 3 ? 4 : 2));   // rows >= ns read as zero
  constexpr int SE = NP == 3 ? 4 : 2;       // bytes of a source entry
  constexpr int TV = (TE * SE + 15) / 16;   // loads per granule (16 bytes; 8 for four BF16 entries)
  constexpr int TA = AUX ? (KS + kThreads - 1) / kThreads : 1;
  const auto arsrc = dev::make_rsrc(static_cast<const uint8_t*>(a.rows) + (int64_t)a.C * a.Fp * (NP == 3 ? 4 : 2),
                                    AUX ? (int64_t)a.Fp * (NP == 3 ? 4 : 2) : 0);
  float ta[TA];
  auto load_table = [&](int s, dev::u32x4 (&t)[TG][TV]) {
    if constexpr (AUX) {
#pragma unroll
      for (int i = 0; i < TA; ++i) {
        const int f = s * KS + (int)threadIdx.x + i * kThreads;
        ta[i] = NP == 3 ? __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(arsrc, 4 * f, 0, 0))
                        : dev::bf16_to_f32((uint16_t)__builtin_amdgcn_raw_buffer_load_b16(arsrc, 2 * f, 0, 0));
      }
    }
    const int tid = here(threadIdx.x);
#pragma unroll
    for (int i = 0; i < TG; ++i) {
      const int g = kWhole ? tid + i * kThreads : min(tid + i * kThreads, kPart - 1), r = g / GPR, p = g % GPR;
      const uint32_t e = (uint32_t)(r * a.Fp + s * KS + TE * p);
#pragma unroll
      for (int v = 0; v < TV; ++v) {
        if constexpr (TE * SE == 8) {
          const auto w = __builtin_amdgcn_raw_buffer_load_b64(trsrc, (int)(e * SE), 0, 0);
          t[i][v] = dev::u32x4{(uint32_t)w[0], (uint32_t)w[1], 0u, 0u};
        } else {
          const auto w = __builtin_amdgcn_raw_buffer_load_b128(trsrc, (int)(e * SE + 16 * v), 0, 0);
          t[i][v] = dev::u32x4{(uint32_t)w[0], (uint32_t)w[1], (uint32_t)w[2], (uint32_t)w[3]};
        }
      }
    }
  };
  auto write_table = [&](int buffer, const dev::u32x4 (&t)[TG][TV]) {
    if constexpr (AUX) {
#pragma unroll
      for (int i = 0; i < TA; ++i)
        if (KS % kThreads == 0 || (int)threadIdx.x + i * kThreads < KS)
          auxt[buffer * KS + threadIdx.x + i * kThreads] = ta[i];
    }
    dev::u32x4* const dst = lds4 + buffer * kSlice;
    const int tid = here(threadIdx.x);
#pragma unroll
    for (int i = 0; i < TG; ++i) {
      // (absent granules repeat the last one)
      const int g = kWhole ? tid + i * kThreads : min(tid + i * kThreads, kPart - 1), r = g / GPR, p = g % GPR;
      const int at = r * GPR + (p ^ (r & 15));
      if constexpr (I32 && NP == 1) {       // BF16 entries widened: exact
        dst[at] = dev::u32x4{t[i][0][0] << 16, t[i][0][0] & 0xFFFF0000u, t[i][0][1] << 16, t[i][0][1] & 0xFFFF0000u};
      } else if constexpr (NPS == 1) {
        dst[at] = t[i][0];
      } else {
        // leading 8 significant bits, the next 8, the rest (at most 8): each
        // subtraction is exact, and so is their sum
        dev::u32x4 hi, mid, lo;
#pragma unroll
        for (int d = 0; d < 4; ++d) {
          float h[2], m[2], l[2];
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            const int k = 2 * d + e;
            const float w = __uint_as_float(t[i][k / 4 % TV][k % 4]);
            h[e] = __uint_as_float(__float_as_uint(w) & 0xFFFF0000u);
            const float r1 = w - h[e];
            m[e] = __uint_as_float(__float_as_uint(r1) & 0xFFFF0000u);
            l[e] = r1 - m[e];
          }
          hi[d] = pack_bf16(h[0], h[1]);
          mid[d] = pack_bf16(m[0], m[1]);
          lo[d] = pack_bf16(l[0], l[1]);
        }
        dst[at] = hi;
        dst[kPart + at] = mid;
        dst[2 * kPart + at] = lo;
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  // Lane parts of the LDS addresses: what differs between the windows, tiles
  // and parts of a unit beyond these is a constant offset.  Writes: load j of a
  // unit covers files FPI j + lr, and 16 / FPI loads 16 files.  Operand reads:
  // window u of file col sits at lane part u % kRW.  Table reads: granule 8 u +
  // 2 q + h of row col at lane part (u % 2, h).
  constexpr int kRW = NG >= 16 ? 4 : 2;
  constexpr int kBlock = I32 ? kWindow : kFlush;   // bytes per fresh accumulator (16 int32 features)
  int wpos[16 / FPI], rpos[kRW], tpos[2][2], tpos4[4];
#pragma unroll
  for (int j = 0; j < 16 / FPI; ++j) wpos[j] = stage_granule<NG>(FPI * j + lr, lp);
#pragma unroll
  for (int w = 0; w < kRW; ++w) rpos[w] = stage_granule<NG>(col, 4 * w + q);
#pragma unroll
  for (int w = 0; w < 2; ++w)
#pragma unroll
    for (int h = 0; h < 2; ++h) tpos[w][h] = col * GPR + ((8 * w + 2 * q + h) ^ col);
#pragma unroll
  for (int w = 0; w < 4; ++w) tpos4[w] = col * GPR + ((4 * w + q) ^ col);    // int32: granule 4 u + q
  float bias[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) bias[nt] = (16 * nt + col < a.ns) ? a.row_bias[16 * nt + col] : 0.0f;

  auto zero = [&](f32x4 (&tot)[MT][NT]) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) tot[mt][nt] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  };

  // Transpose one unit of slice s (its table in `buffer`) through the stage and
  // add its products to tot.
  auto compute = [&](int s, int buffer, const dev::u32x4 (&src)[NL], f32x4 (&tot)[MT][NT], float (&taux)[MT]) {
    const dev::u32x4* const tb = lds4 + buffer * kSlice;
    dev::u32x4 xv[MT];
    auto read_window = [&](int u) {
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
        xv[mt] = (stg + rpos[u % kRW])[(16 * mt) * NG + u % (SS / kWindow) / kRW * 4 * kRW];
    };
#pragma unroll
    for (int b = 0; b < KB / kBlock; ++b) {
      // the last slice of a row: what holds no features is left out, by halves
      // (a branch at every sum made full slices 3% slower; with the aux row's
      // registers it is the cheaper form: 378 against 394 us)
      constexpr int kSkip = AUX || KB == kBlock ? 1 : KB / kBlock / 2;
      if (b > 0 && b % kSkip == 0 && s * KB + b * kBlock >= row_bytes) break;
      if (b % (SS / kBlock) == 0) {
        // the operand reads of what the stage held are done before it is
        // rewritten: LDS operations of a wave complete in order
#pragma unroll
        for (int j = 0; j < NLS; ++j)
          (stg + wpos[j % (16 / FPI)])[j / (16 / FPI) * 16 * NG] = src[b / (SS / kBlock) * NLS + j];
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        read_window(b * (kBlock / kWindow));
      }
      f32x4 acc[kAcc][MT][NT];
#pragma unroll
      for (int h = 0; h < kAcc; ++h) zero(acc[h]);
      if constexpr (ROW) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) acc[0][mt][nt] = tot[mt][nt];
      }
      float aacc[MT] = {};
#pragma unroll
      for (int w = 0; w < kBlock / kWindow; ++w) {
        // the table reads of a window are in flight while its bytes are
        // converted; the scheduler must not gather several windows' reads
        // (there are no registers for them)
        const int u = b * (kBlock / kWindow) + w;
        auto add_aux = [&](int mt, int e0, const float (&g)[16], int n) {
          const float4* const wa = reinterpret_cast<const float4*>(auxt + buffer * KS + e0);
#pragma unroll
          for (int d = 0; d < 4; ++d) {
            if (4 * d >= n) continue;
            const float4 w4 = wa[d];
            aacc[mt] = fmaf(g[4 * d], w4.x, aacc[mt]);
            aacc[mt] = fmaf(g[4 * d + 1], w4.y, aacc[mt]);
            aacc[mt] = fmaf(g[4 * d + 2], w4.z, aacc[mt]);
            aacc[mt] = fmaf(g[4 * d + 3], w4.w, aacc[mt]);
          }
          // summed here: left alone, the compiler moves every window's sums
          // to the end of the unit and spills their operands
          asm volatile("" : "+v"(aacc[mt]));
        };
        if constexpr (I32) {
          // four values per lane and window, one FP32 MFMA for each
          dev::u32x4 bv[NT];
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) bv[nt] = (tb + tpos4[u % 4])[16 * nt * GPR + u / 4 * 16];
          float g[MT][16];
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              g[mt][e] = (float)(int32_t)xv[mt][e];
              if (BIN) g[mt][e] = __builtin_amdgcn_fmed3f(g[mt][e], 0.0f, 1.0f);
            }
            if constexpr (AUX) add_aux(mt, u * WF + 4 * q, g[mt], 4);
          }
          if ((u + 1) % (SS / kWindow) != 0) read_window(u + 1);
#pragma unroll
          for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
              for (int mt = 0; mt < MT; ++mt)
                acc[0][mt][nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(g[mt][e], __uint_as_float(bv[nt][e]),
                                                                      acc[0][mt][nt], 0, 0, 0);
        } else {
          // column tiles in groups whose operands the registers hold beside the sums
          // (16 tiles at two waves per SIMD)
          constexpr int kGroup = NT > 8 && PT == 1 ? 4 : NT;
          dev::u32x4 av[MT][2];
#pragma unroll
          for (int n0 = 0; n0 < NT; n0 += kGroup) {
            dev::u32x4 bv[kGroup][2][NP];
#pragma unroll
            for (int nt = 0; nt < kGroup; ++nt)
#pragma unroll
              for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int part = 0; part < NP; ++part)
                  bv[nt][h][part] = (tb + tpos[u % 2][h])[part * kPart + 16 * (n0 + nt) * GPR + u / 2 * 16];
            if (n0 == 0) {
#pragma unroll
              for (int mt = 0; mt < MT; ++mt) {
                const int f0 = s * KS + u * kWindow + 16 * q;
                if (XT == NB_X_FP8 && f0 + 16 > a.F) {   // NaN encodings past the last feature
                  const int nv = max(0, a.F - f0);
#pragma unroll
                  for (int d = 0; d < 4; ++d) {
                    const int nb = min(4, max(0, nv - 4 * d));
                    xv[mt][d] &= (nb >= 4) ? ~0u : ((1u << (8 * nb)) - 1u);
                  }
                }
                float g[16];
                to_bf16<XT, BIN>(xv[mt], av[mt][0], av[mt][1], g);
                if constexpr (AUX) add_aux(mt, u * kWindow + 16 * q, g, 16);
              }
              if ((u + 1) % (SS / kWindow) != 0) read_window(u + 1);
            }
#pragma unroll
            for (int nt = 0; nt < kGroup; ++nt)
#pragma unroll
              for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int part = 0; part < NP; ++part)
#pragma unroll
                  for (int mt = 0; mt < MT; ++mt) {
                    f32x4& c = acc[part == 0 ? 0 : kAcc - 1][mt][n0 + nt];
                    c = mfma(av[mt][h], bv[nt][h][part], c);
                  }
            if (n0 + kGroup < NT) __builtin_amdgcn_sched_barrier(0);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (AUX) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) taux[mt] += aacc[mt];
      }
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          if constexpr (ROW) tot[mt][nt] = acc[0][mt][nt];
          else tot[mt][nt] += kAcc == 2 ? acc[0][mt][nt] + acc[kAcc - 1][mt][nt] : acc[0][mt][nt];
        }
    }
  };

  // Outputs of the unit that starts at file row0.  A lane holds files 4 q + i
  // of each 16-file tile for class 16 nt + col.  Every store is issued; those
  // of absent files, classes and outputs are out of their descriptor's range.
  const float abias = AUX ? a.row_bias[a.C] : 0.0f;
  auto finish = [&](int64_t row0, const f32x4 (&tot)[MT][NT], float (&taux)[MT]) {
    const int64_t left = a.n - row0;
    const auto rl = dev::make_rsrc(a.labels + row0, a.labels ? left * 4 : 0);
    const auto rp = dev::make_rsrc(a.log_post + row0 * a.C, a.log_post ? left * a.C * 4 : 0);
    const auto rs = dev::make_rsrc(a.scores + row0 * a.C, a.scores ? left * a.C * 4 : 0);
    const int col = here(lane & 15), q = here(lane >> 4);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      // AUX: lane (col, q) holds file col's sum over the q-th 16 bytes of every window
      float file_aux = 0.0f;
      if constexpr (AUX) {
        file_aux = taux[mt] + __shfl_xor(taux[mt], 16);
        file_aux += __shfl_xor(file_aux, 32);
        file_aux += abias;
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int r = 16 * mt + 4 * q + i;
        float sv[NT];
        float m = -INFINITY;
        int best = 1 << 30;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          const int c = 16 * nt + col;
          sv[nt] = tot[mt][nt][i] + bias[nt];
          const bool take = c < a.C && sv[nt] > m;
          m = take ? sv[nt] : m;
          best = take ? c : best;
        }
        argmax_step<8>(m, best);
        argmax_step<4>(m, best);
        argmax_step<2>(m, best);
        argmax_step<1>(m, best);
        float z = 0.0f;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) z += (16 * nt + col < a.C) ? __expf(sv[nt] - m) : 0.0f;
        if constexpr (ROW) {
          z = butterfly16(z);
        } else {
          z += ror16<8>(z);
          z += ror16<4>(z);
          z += ror16<2>(z);
          z += ror16<1>(z);
        }
        const float lse = m + __logf(z);
        best = best < a.C ? best : 0;      // no sum compares (NaN features)
        __builtin_amdgcn_raw_buffer_store_b32((uint32_t)best, rl, (int)(col == 0 ? 4u * r : dev::kNoAccess), 0, 0);
        float aux = 0.0f;       // the raw-score offset sits in column C
        if constexpr (AUX) {
          aux = __shfl(file_aux, 4 * q + i);
        } else if (a.ns > a.C) {
          float mine = 0.0f;
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) mine = (16 * nt + col == a.C) ? sv[nt] : mine;
          aux = __shfl(mine, (lane & ~15) | (a.C & 15));
        }
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          const int c = 16 * nt + col;
          const uint32_t off = c < a.C ? (uint32_t)(r * a.C + c) * 4u : dev::kNoAccess;
          __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(sv[nt] - lse), rp, (int)off, 0, 0);
          if (AUX || a.ns > a.C)
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(sv[nt] + aux), rs, (int)off, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };

  const uint32_t voff = (uint32_t)(lr * ld) + 16u * lp;
  auto issue = [&](int64_t row0, int s, dev::u32x4 (&dst)[NL]) {
    const int64_t base = row0 * ld + (int64_t)s * KB;
    const auto rsrc = dev::make_rsrc(a.x + base, a.total_bytes - base);
#pragma unroll
    for (int j = 0; j < NL; ++j) {
      // bytes past the last feature belong to the next row, whose own loads fetch them
      const bool live = s * KB + j / NLS * SS + 16 * lp < row_bytes;
      dst[j] = dev::buffer_load16(
          rsrc, live ? voff + (uint32_t)(FPI * (j % NLS)) * (uint32_t)ld + j / NLS * SS : dev::kNoAccess);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  dev::u32x4 tg[TG][TV];
  load_table(0, tg);
  write_table(0, tg);
  if (resident && nsl > 1) {
    load_table(1, tg);
    write_table(1, tg);
  }
  __syncthreads();
  int cur = 0;              // buffer of the current slice (a resident table: slice s sits in buffer s)
  dev::u32x4 buf[2][NL];

  // One slice: the next slice's table (slice 0 after the last, for the next
  // tile) is loaded before the slice's units and written to the other buffer,
  // which the barrier before this slice freed, after them.
  auto begin_slice = [&](int sn) {
    if (!resident) load_table(sn, tg);
  };
  auto end_slice = [&](int sn) {
    if (resident) {
      cur = sn;
    } else {
      cur ^= 1;
      write_table(cur, tg);
      __syncthreads();
    }
  };

  // ---- wide tiles: PT units per wave and slice, every load in bounds; unit p
  // of wave w starts at file ((tile PT + p) NW + w) GF
  if constexpr (PT > 1) {
    auto wide_row = [&](int64_t tile, int p) { return ((tile * PT + p) * NW + wave) * GF; };
    if ((int64_t)blockIdx.x < a.wide_tiles) issue(wide_row(blockIdx.x, 0), 0, buf[0]);
    for (int64_t tile = blockIdx.x; tile < a.wide_tiles; tile += gridDim.x) {
      f32x4 tot[PT][MT][NT];
      float taux[PT][MT] = {};
#pragma unroll
      for (int p = 0; p < PT; ++p) zero(tot[p]);
      const int64_t next = tile + gridDim.x < a.wide_tiles ? tile + gridDim.x : tile;   // after the last: a re-read
      for (int s = 0; s < nsl; ++s) {
        const int sn = s + 1 < nsl ? s + 1 : 0;
        begin_slice(sn);
#pragma unroll
        for (int p = 0; p < PT; ++p) {
          if (p + 1 < PT) issue(wide_row(tile, p + 1), s, buf[(p + 1) & 1]);
          else issue(wide_row(sn ? tile : next, 0), sn, buf[0]);
          compute(s, cur, buf[p & 1], tot[p], taux[p]);
        }
        end_slice(sn);
      }
#pragma unroll
      for (int p = 0; p < PT; ++p) finish(wide_row(tile, p), tot[p], taux[p]);
    }
  }

  // ---- the remaining files, one unit per wave and tile; units that reach the
  // buffer's end take guarded loads
  const int64_t done = a.wide_tiles * PT * NW * GF;
  const int64_t per_tile = (int64_t)NW * GF;
  for (int64_t tile = blockIdx.x; done + tile * per_tile < a.n; tile += gridDim.x) {
    const int64_t row0 = done + tile * per_tile + wave * GF;
    const bool fast = row0 + GF <= a.nfast;
    auto fetch = [&](int s, dev::u32x4 (&dst)[NL]) {
      if (fast) {
        issue(row0, s, dst);
      } else {
#pragma unroll
        for (int j = 0; j < NL; ++j) {
          const int64_t row = row0 + FPI * (j % NLS) + lr, off = row * ld + (int64_t)s * KB + j / NLS * SS + 16 * lp;
          dst[j] = dev::u32x4{0u, 0u, 0u, 0u};
          if (row < a.n) dst[j] = dev::load16_guarded(a.x + off, a.total_bytes - off);
        }
      }
    };
    f32x4 tot[MT][NT];
    float taux[MT] = {};
    zero(tot);
    fetch(0, buf[0]);
    for (int s = 0; s < nsl; s += 2) {
      const int s1 = s + 1 < nsl ? s + 1 : 0, s2 = s + 2 < nsl ? s + 2 : 0;
      begin_slice(s1);
      if (s1) fetch(s1, buf[1]);
      compute(s, cur, buf[0], tot, taux);
      end_slice(s1);
      if (!s1) break;
      begin_slice(s2);
      if (s2) fetch(s2, buf[0]);
      compute(s1, cur, buf[1], tot, taux);
      end_slice(s2);
    }
    finish(row0, tot, taux);
  }
}

using KernelFn = void (*)(ScoreTileArgs);

struct TileKernel {
  KernelFn fn = nullptr;
  int slice = 0, files = 0, units = 0, waves = 0;   // KB, 16 MT, PT, NW
  size_t lds = 0;
  bool aux = false;
};

template <int XT, int NT, int NP, bool BIN, int MT, int PT, int KB, int SS, int NW, bool AUX = false, bool ROW = false>
TileKernel tile_kernel() {
  TileKernel k;
  k.fn = score_tile_kernel<XT, NT, NP, BIN, MT, PT, KB, SS, NW, AUX, ROW>;
  k.slice = KB;
  k.files = 16 * MT;
  k.units = PT;
  k.waves = NW;
  const bool i32 = XT == NB_X_I32;      // FP32 entries, KB / 4 of them
  k.lds = (size_t)2 * (i32 ? 1 : NP) * 16 * NT * KB * (i32 ? 1 : 2) + (size_t)NW * 16 * MT * SS +
          (AUX ? 8 * (i32 ? KB / 4 : KB) : 0);
  k.aux = AUX;
  return k;
}

// Short rows (at most 256 features, 128 for int32: two slices of a quarter of the
// size) run in workgroups of four waves with a table small enough for four of them
// per CU.  A file is then a chain of one or two loads and an epilogue, and with one
// workgroup of eight waves per CU, as long rows have it, the chain's latency was all
// the time: 300,000 files of 7 classes 35 us at any F up to 256, now 20 (F = 64) to 26
// (F = 256); 1,000,000 int32 files of 16 classes, F = 16, 118 -> 57.  Sums are the
// same.

// int32 features: at most 32 score rows, either table.
template <int NP, bool BIN>
TileKernel pick_tile_i32(int nt, bool aux, bool narrow) {
  if (narrow) {
    if (nt == 1 && aux) return tile_kernel<NB_X_I32, 1, NP, BIN, 1, 2, 256, 256, 4, true>();
    if (nt == 1) return tile_kernel<NB_X_I32, 1, NP, BIN, 1, 2, 256, 256, 4>();
    if (nt == 2) return tile_kernel<NB_X_I32, 2, NP, BIN, 1, 2, 256, 256, 8>();
  }
  if (nt == 1 && aux) return tile_kernel<NB_X_I32, 1, NP, BIN, 1, 2, 1024, 256, 8, true>();
  if (nt == 1) return tile_kernel<NB_X_I32, 1, NP, BIN, 1, 2, 1024, 256, 8>();
  if (nt == 2) return tile_kernel<NB_X_I32, 2, NP, BIN, 1, 2, 1024, 256, 8>();
  return {};
}

// The slice is as long as two slices of the table and the waves' stages fit
// the 160 KB of LDS.
//
// 129 to 256 score rows: the sums of two units take the registers of a wave per SIMD,
// so a call of more files than such waves hold (small: one unit each) takes one unit
// per wave and two waves per SIMD (200 classes, F = 1000, 30,000 files: 94 -> 38 us;
// 10,000 FP8 files at F = 4096 84 against 122).
template <int XT, bool BIN>
TileKernel pick_tile(int nt, bool f32, bool aux, bool four, bool row, bool narrow, bool small) {
  if (narrow && nt == 1) {
    if (f32 && aux) return tile_kernel<XT, 1, 3, BIN, 1, 2, 128, 128, 4, true>();
    if (f32) return tile_kernel<XT, 1, 3, BIN, 1, 2, 128, 128, 4>();
    if (!aux) return tile_kernel<XT, 1, 1, BIN, 1, 2, 128, 128, 4>();
  }
  if (f32) {
    if (nt == 1 && aux)
      return four ? tile_kernel<XT, 1, 3, BIN, 1, 4, 512, 128, 8, true>()
                  : tile_kernel<XT, 1, 3, BIN, 1, 2, 512, 128, 8, true>();
    if (nt == 1) return tile_kernel<XT, 1, 3, BIN, 1, 2, 512, 256, 8>();
    if (nt == 2)
      return four ? tile_kernel<XT, 2, 3, BIN, 1, 4, 256, 256, 8>() : tile_kernel<XT, 2, 3, BIN, 1, 2, 256, 256, 8>();
    return {};
  }
  if (nt == 1 && aux)
    return row ? tile_kernel<XT, 1, 1, BIN, 1, 2, 512, 512, 4, true, true>()
               : tile_kernel<XT, 1, 1, BIN, 1, 2, 512, 512, 4, true>();
  switch (nt) {
    case 1: return tile_kernel<XT, 1, 1, BIN, 1, 2, 512, 256, 4>();
    case 2: return tile_kernel<XT, 2, 1, BIN, 1, 2, 512, 512, 8>();
    case 3: return tile_kernel<XT, 3, 1, BIN, 1, 2, 512, 512, 8>();
    case 4: return tile_kernel<XT, 4, 1, BIN, 1, 2, 256, 256, 8>();
    case 8: return tile_kernel<XT, 8, 1, BIN, 1, 2, 256, 128, 8>();
    case 16:
      return small ? tile_kernel<XT, 16, 1, BIN, 1, 2, 128, 128, 4>() : tile_kernel<XT, 16, 1, BIN, 1, 1, 128, 128, 8>();
    default: return {};
  }
}

// column tiles rounded up to a compiled count (extra columns are zero rows)
int round_nt(int nt) { return nt <= 4 ? nt : nt <= 8 ? 8 : nt <= 16 ? 16 : 0; }

}  // namespace

// Entry from nb_score for C >= 3 (arguments validated by the caller: at most 32
// rows for the FP32 table and int32 features, 256 for byte features on BF16).
int launch_score_tile(const nb_model* m, const nb_layout& L, const void* x, int32_t xtype, int64_t n, int64_t ld,
                      int32_t wtype, int32_t* labels, float* log_post, float* scores, hipStream_t s) {
  const int C = m->n_classes;
  const int ns = C + (scores ? 1 : 0);
  const bool f32 = wtype == NB_W_F32, bin = m->kind == NB_BERNOULLI;
  const bool aux = scores && C == 16;      // 16 classes fill the tile: the aux row would need a second one
  const int nt = aux ? 1 : round_nt((ns + 15) / 16);
  // Four units per wave and slice for the FP32 table of 16 classes with raw scores
  // and of 17 to 32 score rows, from 1,025 features (its slices, which do not stay in
  // LDS, are then staged half as often) and from four units for every workgroup: 16
  // classes, raw scores, F = 4096, 400,003 files 379 us with two, 362 with four; 90,000
  // files 100 us, where four leave only single-unit tiles, 116; a resident table, F =
  // 700, 189 against 193.  Two elsewhere: one column tile without the aux row differs
  // less (16 classes, F = 2000, 400,000 files 211 us with two, 204 with four; 3
  // classes, F = 4096, 200,000 files 191 and 195), and so do 17 to 32 rows of 513 to
  // 1,024 features, whose slices are half as long (20 classes, 300,000 files, F =
  // 1000: 119 and 112; 31 classes, 1,000,000 files, F = 800: 307 both).  Sums are the
  // same.
  const int64_t per_round = (int64_t)128 * device_cu_count();
  const bool four = f32 && m->n_features > 1024 && n >= 4 * per_round;
  const bool narrow = m->n_features <= (xtype == NB_X_I32 ? 128 : 256);
  const bool small = n <= (int64_t)64 * device_cu_count();
  const bool row = xtype != NB_X_I32 && score16_staged(m, L, wtype, nullptr);
  TileKernel k;
  if (xtype == NB_X_I32) {
    if (f32) k = bin ? pick_tile_i32<3, true>(nt, aux, narrow) : pick_tile_i32<3, false>(nt, aux, narrow);
    else k = bin ? pick_tile_i32<1, true>(nt, aux, narrow) : pick_tile_i32<1, false>(nt, aux, narrow);
  } else if (xtype == NB_X_U8) {
    k = bin ? pick_tile<NB_X_U8, true>(nt, f32, aux, four, row, narrow, small) : pick_tile<NB_X_U8, false>(nt, f32, aux, four, row, narrow, small);
  } else {
    k = bin ? pick_tile<NB_X_FP8, true>(nt, f32, aux, four, row, narrow, small) : pick_tile<NB_X_FP8, false>(nt, f32, aux, four, row, narrow, small);
  }
  if (!k.fn) return fail(NB_EINVAL, "too many score columns for the table type");
  const uint8_t* base = static_cast<const uint8_t*>(m->dev);
  ScoreTileArgs a;
  a.x = static_cast<const uint8_t*>(x);
  const int eb = elem_bytes(xtype);
  a.ld_bytes = ld * eb;
  a.n = n;
  a.total_bytes = ((n - 1) * ld + m->n_features) * eb;
  a.rows = base + (f32 ? L.off_form_f32 : L.off_form_bf16);
  a.row_bias = reinterpret_cast<const float*>(base + L.off_form_bias);
  a.labels = labels;
  a.log_post = log_post;
  a.scores = scores;
  a.F = m->n_features;
  a.Fp = L.padded_features;
  a.C = C;
  a.ns = aux ? C : ns;
  // files whose slices all lie inside the buffer
  const int64_t span = ((int64_t)a.F * eb + k.slice - 1) / k.slice * k.slice;
  a.nfast = a.total_bytes >= span ? std::min(n, (a.total_bytes - span) / a.ld_bytes + 1) : 0;
  const void* fn = reinterpret_cast<const void*>(k.fn);
  NB_HIP_CHECK(hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)k.lds));
  const int64_t cap = (int64_t)resident_per_cu(fn, 64 * k.waves, k.lds) * device_cu_count();
  // Whole rounds of wide tiles; what is left goes to single-unit tiles when
  // these need fewer units per workgroup than another round of wide ones.
  const int64_t per_tile = (int64_t)k.files * k.waves;           // files of a single-unit tile
  const int64_t tiles = (n + per_tile - 1) / per_tile;
  const int64_t wide_fit = a.nfast / (per_tile * k.units);       // wide tiles with every load in bounds
  const int64_t rounds = tiles / (cap * k.units);
  const int64_t rest = tiles - rounds * cap * k.units;
  a.wide_tiles =
      k.units == 1 ? 0 : std::min(wide_fit, rest > cap * (k.units - 1) ? (rounds + 1) * cap : rounds * cap);
  const int64_t want = std::max(a.wide_tiles, tiles - a.wide_tiles * k.units);
  const unsigned grid = (unsigned)std::max<int64_t>(1, std::min(want, cap));
  hipLaunchKernelGGL(k.fn, dim3(grid), dim3(64 * k.waves), k.lds, s, a);
  NB_HIP_CHECK(hipGetLastError());
  return NB_OK;
}

}  // namespace nb
