// Projections of large batches on the matrix cores (gfx950 MFMA): steps of
// kWideMinBatch to 64 sequences over layers of more than a few MB (wide_pays).
//
// The kernels of mfma_proj.hip give a grid row of blocks 16 sequences, so a
// step of 64 streamed every weight four times. Here a block computes all
// sequences of its rows and the weights are read once. What a block loads is
// then its weights (HBM) and the activation operand of its k-tiles (L2), 4 bytes
// per input and sequence, which at 64 sequences is two to ten times its
// weights; both wait in one queue. So
//   * the loop runs over the k-tiles, and every operand tile meets all stripes
//     of the block (up to NS at a time, their sums in registers) while it is
//     in registers: the operand crosses the load path once per NS stripes;
//   * the 8 waves of a block split the k-tiles, so no two waves of a block
//     load the same data, nothing is staged and the loop has no barrier; the
//     waves' sums meet once, in LDS;
//   * 8 waves per CU leave a lane 256 registers: the sums of NS stripes and
//     NBUF tiles of weights and operand in flight;
//   * the QKV, O and down projections split the k-tiles over ks blocks, each
//     with ks times the stripes and 1 / ks of the operand, and store their
//     sums as parts. The attention adds the QKV parts as it reads q, k and v;
//     a small kernel adds those of the O projection (with the residual,
//     RMSNorm2's factor and the gate/up operand) and one those of the down
//     projection (with the residual and the rounding of y). Handing the parts
//     over inside the launch, through coherent stores and a ticket as
//     mfma_proj.hip does, cost 9 us at 64 sequences, a launch about 4.
// Operand layout: [k-tile][16-sequence tile][level][lane][8] bf16, the rows of
// a matrix instruction are 16 sequences, and the two levels of the split are
// two instructions into the same sums.
// The QKV operand (x * gamma1, exact in two levels) and 1/rms(x) are prepared
// once by a small kernel (3.5 us with its boundary): built by every block, as
// the 16-sequence kernel does, the conversion alone is 6.7 us of vector work per
// CU at 64 sequences, and its registers crowd the sums (QKV 22.5 us from the
// prepared operand, 26.9-30.9 us built in place).
// MI355X, kernel us, the 16-sequence kernels -> these: Phi-3 at 64 sequences QKV
// 49.0 -> 22.5, O 24.9 -> 10.2, gate/up 75.9 -> 29.9, down 43.6 -> 18.7 (layer
// 468 -> 372); Llama3-8B at 32 sequences 29.9 -> 15.3, 16.3 -> 10.4, 88.0 ->
// 43.2, 48.5 -> 25.7. Gate/up at 64 sequences of Phi-3 (30 us, 1.2 MB a block, 40
// GB/s per CU): with the weights pointed at one tile 16 us, with the operand at
// one tile 21 (timing only), so the two streams' times add up for the most
// part. By counters 302 MB go through L2 (63 % hits, 600 cycles a request on
// average, about 10 KB in flight per CU), the matrix cores are busy 17 % and the
// vector units 11 % of the cycles: it waits for loads, but neither for HBM (107 MB)
// nor at the rate at which CUs read shared data alone (80-100 GB/s). Two or three
// tiles in flight, rotated operand chunks and 32-bit offsets made no difference.
#include "common.h"
#include "kernels.h"

#include <math.h>

namespace fasttps {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int kWW = 8;            // waves per block
constexpr int kWT = kWW * kWave;  // threads per block
constexpr int kWGrid = 256;       // blocks (one per CU)
constexpr size_t kRedBytes = 144 * 1024;  // LDS for the waves' sums

template <int N>
struct IntTag {
  static constexpr int value = N;
};

__device__ __forceinline__ bf16x8 as_bf16x8(v4u v) { return __builtin_bit_cast(bf16x8, v); }

// floats of one wave's sums of a stripe: 16 columns of NSEQ sequences, padded
// so that columns start 4 banks apart
template <int NBT>
constexpr int red_col() { return 16 * NBT + 4; }
template <int NBT>
constexpr int red_stripe() { return kWW * 16 * red_col<NBT>(); }
// stripes whose sums share LDS before one epilogue
template <int NBT, int NS>
constexpr int red_stripes() {
  constexpr int cap = (int)(kRedBytes / (red_stripe<NBT>() * sizeof(float)));
  return NS < cap ? NS : cap;
}

enum class WMode { kPart, kQkv, kGateUp };

template <WMode MODE, int NBT, int NS, int NBUF>
__global__ __launch_bounds__(kWT) __attribute__((amdgpu_waves_per_eu(2, 2))) void mfma_wide_kernel(MfmaArgs a) {
  constexpr int NSEQ = 16 * NBT;
  constexpr int NOUT = NSEQ * 16;  // (sequence, column) slots of a stripe
  constexpr int RCOL = red_col<NBT>();
  extern __shared__ __attribute__((aligned(16))) float red[];  // [stripe][wave][16][RCOL]

  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int G = gridDim.x, blk = blockIdx.x;
  const int ks = a.ks;
  const int rg = blk / ks, kq = blk - rg * ks;  // row group and part of the k-tiles
  const int NGr = G / ks;
  const int nstr = (a.ns - 1 - rg) / NGr + 1;  // stripes rg, rg + NGr, ... (>= 1)
  const int kbeg = kq * a.ktq, kend = min(kbeg + a.ktq, a.kt);
  // the wave's k-tiles: the part's, dealt in 8 runs that differ by one at most
  const int kn = max(kend - kbeg, 0);
  const int t0 = kbeg + kn * wave / kWW;
  const int nt = kbeg + kn * (wave + 1) / kWW - t0;
  const int R = a.rh;
  const int n16 = lane & 15, kg = lane >> 4;
  const int nb = a.batch;
  constexpr bool gate_up = MODE == WMode::kGateUp;

  // this lane's chunk of a weight tile and of an operand tile (rows past the
  // stripe and sequences past the batch repeat the last one; their results
  // are dropped)
  const unsigned wl = (unsigned)(kg * R + min(n16, R - 1));
  const unsigned al = (unsigned)(n16 + 16 * kg);
  const unsigned al_last = (unsigned)(min(n16, nb - 1 - 16 * (NBT - 1)) + 16 * kg);
  const v4u* W = reinterpret_cast<const v4u*>(a.w);
  const v4u* A = reinterpret_cast<const v4u*>(a.a_in);

  // N stripes from the block's stripe i0 on
  auto pass = [&](int i0, auto n_tag) {
    constexpr int N = decltype(n_tag)::value;
    f4 acc[N][NBT];
#pragma unroll
    for (int s = 0; s < N; ++s)
#pragma unroll
      for (int bt = 0; bt < NBT; ++bt) acc[s][bt] = f4{0.f, 0.f, 0.f, 0.f};
    v4u wr[NBUF][N], ar[NBUF][NBT][2];
    auto load = [&](int r, int t) {
#pragma unroll
      for (int s = 0; s < N; ++s) wr[r][s] = ld_stream(W + ((size_t)(rg + (i0 + s) * NGr) * a.kt + t) * 4 * R + wl);
#pragma unroll
      for (int bt = 0; bt < NBT; ++bt)
#pragma unroll
        for (int lvl = 0; lvl < 2; ++lvl)
          ar[r][bt][lvl] = (A + ((size_t)t * a.nbtc + 2 * bt + lvl) * kWave)[bt == NBT - 1 ? al_last : al];
      __builtin_amdgcn_sched_barrier(0);
    };
    auto consume = [&](int r) {
#pragma unroll
      for (int bt = 0; bt < NBT; ++bt)
#pragma unroll
        for (int lvl = 0; lvl < 2; ++lvl)
#pragma unroll
          for (int s = 0; s < N; ++s)
            acc[s][bt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(ar[r][bt][lvl]), as_bf16x8(wr[r][s]),
                                                                 acc[s][bt], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    };
    if (nt > 0) {
#pragma unroll
      for (int r = 0; r < NBUF; ++r) load(r, t0 + min(r, nt - 1));
      int i = 0;
      for (; i + 2 * NBUF <= nt; i += NBUF)
#pragma unroll
        for (int r = 0; r < NBUF; ++r) {
          consume(r);
          load(r, t0 + i + r + NBUF);
        }
      const int m = nt - i;  // tiles left, fewer than 2 NBUF; the first NBUF of them are in flight
#pragma unroll
      for (int r = 0; r < NBUF; ++r)
        if (r < m) {
          consume(r);
          if (r + NBUF < m) load(r, t0 + i + r + NBUF);
        }
#pragma unroll
      for (int r = 0; r + 1 < NBUF; ++r)
        if (r + NBUF < m) consume(r);
    }
    // ---- the waves' sums meet, CH stripes at a time --------------------------
    constexpr int CH = red_stripes<NBT, N>();
#pragma unroll
    for (int c0 = 0; c0 < N; c0 += CH) {
      const int nc = N - c0 < CH ? N - c0 : CH;
#pragma unroll
      for (int c = 0; c < CH; ++c)
        if (c0 + c < N) {
          // lane l holds sequences 4 (l / 16) .. + 3 of each 16-sequence tile
          float* rw = red + ((size_t)c * kWW + wave) * 16 * RCOL + n16 * RCOL + 4 * kg;
#pragma unroll
          for (int bt = 0; bt < NBT; ++bt) *reinterpret_cast<f4*>(rw + 16 * bt) = acc[c0 + c][bt];
        }
      __syncthreads();
      // the sum of column n of sequence b over the waves
      auto col = [&](int c, int b, int n) {
        const float* rc = red + (size_t)c * red_stripe<NBT>() + n * RCOL + b;
        float v = 0.f;
#pragma unroll
        for (int w = 0; w < kWW; ++w) v += rc[(size_t)w * 16 * RCOL];
        return v;
      };
      if constexpr (gate_up) {
        // units of a stripe: gate columns [0, R / 2), up columns [R / 2, R);
        // lanes n = 0..7 of a sequence hold its units
        constexpr int UG = (CH * NSEQ * 8 + kWT - 1) / kWT;
#pragma unroll
        for (int i = 0; i < UG; ++i) {
          const int q = tid + i * kWT, c = min(q / (NSEQ * 8), nc - 1), b = q / 8 % NSEQ, n = q % 8;
          const int u = R / 2 * (rg + (i0 + c0 + c) * NGr) + n;
          const bool ok = q < nc * NSEQ * 8 && b < nb && n < R / 2 && u < a.rows;
          const float inv = a.inv_in[min(b, nb - 1)];
          const float gt = inv * col(c, b, n), up = inv * col(c, b, min(n + R / 2, 15));
          const float av = gt / (1.0f + expf(-gt)) * up;
          const uint32_t hi = f32_to_bf16(av), lo = f32_to_bf16(av - __uint_as_float(hi << 16));
          // even lanes store the pair's hi levels, odd lanes its lo levels
          // (units come in pairs: K and R / 2 are even)
          const uint32_t mine = hi | (lo << 16);
          const uint32_t other = (uint32_t)__builtin_amdgcn_mov_dpp((int)mine, kDppQuadXor1, 0xF, 0xF, false);
          const uint32_t pair = n % 2 ? (other >> 16) | (mine & 0xFFFF0000u) : (mine & 0xFFFFu) | (other << 16);
          if (ok) {
            a.out[(size_t)b * a.rows + u] = av;
            *reinterpret_cast<uint32_t*>(a.a_out + wide_operand_offset(b, u & ~1, a.a_out_nbtc) +
                                         (n % 2 ? kWave * 8 : 0)) = pair;
          }
        }
      } else {
        constexpr int U = (CH * NOUT + kWT - 1) / kWT;
#pragma unroll
        for (int i = 0; i < U; ++i) {
          const int q = tid + i * kWT, c = min(q / NOUT, nc - 1), b = q / 16 % NSEQ, n = q % 16;
          const int row = R * (rg + (i0 + c0 + c) * NGr) + n;
          float v = col(c, b, n);
          if (MODE == WMode::kQkv) v *= a.inv_in[min(b, nb - 1)];
          if (q < nc * NOUT && b < nb && n < R && row < a.rows)
            a.out[((size_t)kq * a.part_seqs + b) * a.rows + row] = v;
        }
      }
      if (c0 + CH < N || a.passes > 1) __syncthreads();
    }
  };
  // the block's stripes in a.passes passes of NS or NS - 1
  int i0 = 0;
  for (int p = 0; p < a.passes; ++p) {
    const int n = nstr / a.passes + (p < nstr % a.passes ? 1 : 0);
    if (n == NS) {
      pass(i0, IntTag<NS>{});
    } else {
      if constexpr (NS > 1) pass(i0, IntTag<NS - 1>{});
    }
    i0 += n;
  }
}

// The QKV operand x * gamma1 in its two exact levels, and 1/rms(x), one block
// per sequence.
constexpr int kPrepThreads = 256;
__global__ __launch_bounds__(kPrepThreads) void wide_prep_kernel(const uint16_t* __restrict__ x,
                                                                 const uint16_t* __restrict__ gamma, int din,
                                                                 float eps, int nbtc, uint16_t* __restrict__ op,
                                                                 float* __restrict__ inv) {
  __shared__ float red[kPrepThreads / kWave];
  const int b = blockIdx.x;
  const v4u* xr = reinterpret_cast<const v4u*>(x + (size_t)b * din);
  float ss = 0.f;
  for (int c = threadIdx.x; c < din / 8; c += kPrepThreads) {
    float xf[8], g[8];
    unpack8(xr[c], xf);
    unpack8(reinterpret_cast<const v4u*>(gamma)[c], g);
    uint32_t h[8], l[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      // a product of two bf16 numbers has at most 16 significant bits: its
      // truncation and the remainder are both bf16 numbers
      const float v = xf[e] * g[e];
      h[e] = __float_as_uint(v) & 0xFFFF0000u;
      l[e] = __float_as_uint(v - __uint_as_float(h[e]));
      ss = fmaf(xf[e], xf[e], ss);
    }
    v4u* dst = reinterpret_cast<v4u*>(op + wide_operand_offset(b, 8 * c, nbtc));
    dst[0] = v4u{(h[0] >> 16) | h[1], (h[2] >> 16) | h[3], (h[4] >> 16) | h[5], (h[6] >> 16) | h[7]};
    dst[kWave] = v4u{(l[0] >> 16) | (l[1] & 0xFFFF0000u), (l[2] >> 16) | (l[3] & 0xFFFF0000u),
                     (l[4] >> 16) | (l[5] & 0xFFFF0000u), (l[6] >> 16) | (l[7] & 0xFFFF0000u)};
  }
  ss = block_sum(ss, red);
  if (threadIdx.x == 0) inv[b] = 1.0f / sqrtf(ss / (float)din + eps);
}

// h1 = x + the parts of W_o o, the gate/up operand h1 * gamma2 in two levels
// and RMSNorm2's factor; one block per sequence, eight elements per thread
// (one round trip).
__global__ __launch_bounds__(1024) void wide_oproj_sum_kernel(const float* __restrict__ part, int parts, int batch,
                                                              const uint16_t* __restrict__ x,
                                                              const uint16_t* __restrict__ gamma, int D, float eps,
                                                              float* __restrict__ h1_out, uint16_t* __restrict__ op,
                                                              int nbtc, float* __restrict__ inv) {
  __shared__ float red[1024 / kWave];
  const int b = blockIdx.x, c = threadIdx.x;
  const bool ok = c < D / 8;
  float ss = 0.f;
  if (ok) {
    float h[8], g[8];
    unpack8(reinterpret_cast<const v4u*>(x + (size_t)b * D)[c], h);
    unpack8(reinterpret_cast<const v4u*>(gamma)[c], g);
    f4 p[kWideMaxParts][2];
#pragma unroll
    for (int j = 0; j < kWideMaxParts; ++j) {
      const f4* pr = reinterpret_cast<const f4*>(part + ((size_t)min(j, parts - 1) * batch + b) * D) + 2 * c;
      p[j][0] = pr[0];
      p[j][1] = pr[1];
    }
    uint32_t hi[8], lo[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      float v = 0.f;
#pragma unroll
      for (int j = 0; j < kWideMaxParts; ++j) v += j < parts ? p[j][e / 4][e % 4] : 0.f;
      h[e] += v;
      ss = fmaf(h[e], h[e], ss);
      const float hg = h[e] * g[e];
      hi[e] = f32_to_bf16(hg);
      lo[e] = f32_to_bf16(hg - __uint_as_float(hi[e] << 16));
    }
    f4* ho = reinterpret_cast<f4*>(h1_out + (size_t)b * D) + 2 * c;
    ho[0] = f4{h[0], h[1], h[2], h[3]};
    ho[1] = f4{h[4], h[5], h[6], h[7]};
    v4u* dst = reinterpret_cast<v4u*>(op + wide_operand_offset(b, 8 * c, nbtc));
    dst[0] = v4u{hi[0] | (hi[1] << 16), hi[2] | (hi[3] << 16), hi[4] | (hi[5] << 16), hi[6] | (hi[7] << 16)};
    dst[kWave] = v4u{lo[0] | (lo[1] << 16), lo[2] | (lo[3] << 16), lo[4] | (lo[5] << 16), lo[6] | (lo[7] << 16)};
  }
  ss = block_sum(ss, red);
  if (threadIdx.x == 0) inv[b] = 1.0f / sqrtf(ss / (float)D + eps);
}

// y = bf16(h1 + the parts of W_down a), four elements per thread
__global__ __launch_bounds__(256) void wide_down_sum_kernel(const float* __restrict__ part, int parts, int n4,
                                                            const float* __restrict__ h1, uint16_t* __restrict__ y) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= n4) return;
  const f4 h = reinterpret_cast<const f4*>(h1)[i];
  f4 p[kWideMaxParts];
#pragma unroll
  for (int j = 0; j < kWideMaxParts; ++j) p[j] = reinterpret_cast<const f4*>(part)[(size_t)min(j, parts - 1) * n4 + i];
  uint32_t o[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    float v = 0.f;
#pragma unroll
    for (int j = 0; j < kWideMaxParts; ++j) v += j < parts ? p[j][e] : 0.f;
    o[e] = f32_to_bf16(h[e] + v);
  }
  reinterpret_cast<uint2*>(y)[i] = make_uint2(o[0] | (o[1] << 16), o[2] | (o[3] << 16));
}

// the test hook's view of q|k|v, one block row per sequence
__global__ __launch_bounds__(256) void wide_pair_sum_kernel(const float* __restrict__ src, size_t part,
                                                            const int* __restrict__ split, int rows,
                                                            float* __restrict__ dst) {
  const int c = blockIdx.x * 256 + threadIdx.x, b = blockIdx.y;
  if (c >= rows) return;
  const size_t i = (size_t)b * rows + c;
  dst[i] = split[b] ? src[i] + src[part + i] : src[i];
}

// stripes whose sums a lane holds at once (6 beyond 32 sequences; with four
// sequence tiles the compiler then spills 2 to 8 of the 256 registers, 12 to 36
// bytes a lane: Phi-3's QKV at 64 sequences)
constexpr int ns_max(int nbt) { return nbt <= 2 ? 8 : 6; }

struct WideGeom {
  int nbt, ks, ngr, ktq, nstr_max, passes, ns;
};
WideGeom wide_geom(WMode mode, int ns, int kt, int rh, int batch) {
  WideGeom g;
  g.nbt = (batch + 15) / 16;
  const int nstr0 = (ns + kWGrid - 1) / kWGrid;  // stripes per block, whole rows
  // Parts: the QKV projection has kWideQkvParts, the O and down projections
  // as many as bring the operand KB of a k-tile (2 nbt, spread over ks
  // blocks' stripes) to the weight KB (ks nstr0 rh / 16): on MI355X at 64
  // Phi-3 sequences O took 15.4 us and down 34.7 us in one part (sums stored
  // by the block itself), 10.2 and 18.7 us in four
  int ks = mode == WMode::kQkv ? kWideQkvParts : 1;
  if (mode == WMode::kPart)
    while (ks < kWideMaxParts && 2 * g.nbt * 16 > ks * nstr0 * rh && kt >= 2 * ks * kWW) ks *= 2;
  if (mode == WMode::kPart)
    while (ks > 1 && (ks - 1) * ((kt + ks - 1) / ks) >= kt) ks /= 2;
  g.ks = ks;
  g.ngr = ns < kWGrid / ks ? ns : kWGrid / ks;
  g.ktq = (kt + ks - 1) / ks;
  g.nstr_max = (ns + g.ngr - 1) / g.ngr;
  g.passes = (g.nstr_max + ns_max(g.nbt) - 1) / ns_max(g.nbt);
  g.ns = (g.nstr_max + g.passes - 1) / g.passes;
  return g;
}

template <WMode MODE, int NBT, int NS>
hipError_t launch_ns(const MfmaArgs& a, int ngr, hipStream_t s, KernelEvents ev) {
  // tiles in flight: what 256 registers hold beside the sums
  constexpr int NBUF = 4 * NS * NBT + 12 * (NS + 2 * NBT) <= 160 ? 3 : 2;
  const size_t lds = (size_t)red_stripes<NBT, NS>() * red_stripe<NBT>() * sizeof(float);
  return ext_launch(mfma_wide_kernel<MODE, NBT, NS, NBUF>, dim3(ngr * a.ks), dim3(kWT), lds, s, ev, a);
}

template <WMode MODE, int NBT>
hipError_t launch_nbt(const MfmaArgs& a, const WideGeom& g, hipStream_t s, KernelEvents ev) {
  switch (g.ns) {
    case 1: return launch_ns<MODE, NBT, 1>(a, g.ngr, s, ev);
    case 2: return launch_ns<MODE, NBT, 2>(a, g.ngr, s, ev);
    case 3: return launch_ns<MODE, NBT, 3>(a, g.ngr, s, ev);
    case 4: return launch_ns<MODE, NBT, 4>(a, g.ngr, s, ev);
    case 5: return launch_ns<MODE, NBT, 5>(a, g.ngr, s, ev);
    case 6: return launch_ns<MODE, NBT, 6>(a, g.ngr, s, ev);
    default: break;
  }
  if constexpr (ns_max(NBT) > 6) {
    switch (g.ns) {
      case 7: return launch_ns<MODE, NBT, 7>(a, g.ngr, s, ev);
      case 8: return launch_ns<MODE, NBT, 8>(a, g.ngr, s, ev);
      default: break;
    }
  }
  return hipErrorInvalidValue;
}

template <WMode MODE>
hipError_t launch_mode(const MfmaArgs& a_in, hipStream_t s, KernelEvents ev) {
  MfmaArgs a = a_in;
  if (a.batch < kWideMinBatch || a.batch > 64 || a.ns < 1 || a.kt < 1 || a.din % 8 != 0) return hipErrorInvalidValue;
  if (a.rh < 2 || a.rh > 16 || a.rh % 4 != 0 || a.nbtc < 2 * ((a.batch + 15) / 16)) return hipErrorInvalidValue;
  const WideGeom g = wide_geom(MODE, a.ns, a.kt, a.rh, a.batch);
  a.ks = g.ks;
  a.ktq = g.ktq;
  a.passes = g.passes;
  switch (g.nbt) {
    case 2: return launch_nbt<MODE, 2>(a, g, s, ev);
    case 3: return launch_nbt<MODE, 3>(a, g, s, ev);
    case 4: return launch_nbt<MODE, 4>(a, g, s, ev);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

size_t wide_part_floats(int ns, int kt, int rh, int rows, int batch) {
  size_t most = 0;
  for (int b = kWideMinBatch; b <= batch; ++b) {
    const size_t f = (size_t)wide_geom(WMode::kPart, ns, kt, rh, b).ks * b * rows;
    if (f > most) most = f;
  }
  return most;
}

hipError_t launch_wide_qkv(const MfmaArgs& a_in, uint16_t* op, float* inv, hipStream_t s, KernelEvents ev,
                           KernelEvents ev2) {
  MfmaArgs a = a_in;
  if (a.part_seqs < a.batch) return hipErrorInvalidValue;
  const hipError_t e = ext_launch(wide_prep_kernel, dim3(a.batch), dim3(kPrepThreads), 0, s, ev, a.x_bf16, a.gamma,
                                  a.din, a.eps, a.nbtc, op, inv);
  if (e != hipSuccess) return e;
  a.a_in = op;
  a.inv_in = inv;
  return launch_mode<WMode::kQkv>(a, s, ev2);
}

hipError_t launch_wide_oproj(const MfmaArgs& a_in, float* inv, hipStream_t s, KernelEvents ev, KernelEvents ev2) {
  MfmaArgs a = a_in;
  const int parts = wide_geom(WMode::kPart, a.ns, a.kt, a.rh, a.batch).ks;
  if (!a.kpart || a.kpart_cap < (size_t)parts * a.batch * a.rows || a.rows > 8192) return hipErrorInvalidValue;
  a.out = a.kpart;
  a.part_seqs = a.batch;
  const hipError_t e = launch_mode<WMode::kPart>(a, s, ev);
  if (e != hipSuccess) return e;
  const int threads = (a.rows / 8 + kWave - 1) / kWave * kWave;
  return ext_launch(wide_oproj_sum_kernel, dim3(a.batch), dim3(threads), 0, s, ev2, (const float*)a.kpart, parts,
                    a.batch, a.x_bf16, a.gamma, a.rows, a.eps, a_in.out, a.a_out, a.a_out_nbtc, inv);
}

hipError_t launch_wide_gate_up(const MfmaArgs& a, hipStream_t s, KernelEvents ev) {
  return launch_mode<WMode::kGateUp>(a, s, ev);
}

hipError_t launch_wide_down(const MfmaArgs& a_in, hipStream_t s, KernelEvents ev, KernelEvents ev2) {
  MfmaArgs a = a_in;
  const int parts = wide_geom(WMode::kPart, a.ns, a.kt, a.rh, a.batch).ks;
  if (!a.kpart || a.kpart_cap < (size_t)parts * a.batch * a.rows) return hipErrorInvalidValue;
  a.out = a.kpart;
  a.part_seqs = a.batch;
  const hipError_t e = launch_mode<WMode::kPart>(a, s, ev);
  if (e != hipSuccess) return e;
  const int n4 = a.batch * a.rows / 4;
  return ext_launch(wide_down_sum_kernel, dim3((n4 + 255) / 256), dim3(256), 0, s, ev2, (const float*)a.kpart, parts,
                    n4, a.res_f32, a.out_bf16);
}

hipError_t launch_wide_qkv_sum(const float* parts, size_t part, const int* split, int rows, int batch, float* dst,
                               hipStream_t s) {
  return ext_launch(wide_pair_sum_kernel, dim3((rows + 255) / 256, batch), dim3(256), 0, s, KernelEvents{}, parts, part,
                    split, rows, dst);
}

}  // namespace fasttps
