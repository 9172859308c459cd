// Split-KV decode attention on the matrix cores (gfx950): groups of query heads,
// and long batches over 8-bit caches (attention_on_mfma).
//
// The vector kernel (attn_body.h) spends per cached element one FMA per query
// head for the scores, one for the output, and the decoding of 8-bit codes.
// For groups of four that is as much issue time as the HBM stream takes, and
// its accumulators (4 heads x d / 4 per lane) leave room for one tile in
// flight. Here both products run on v_mfma_f32_16x16x32_bf16, still in 32-bit
// precision: a cached element is a bf16 number (8-bit codes convert exactly),
// q and the softmax weights are fp32 numbers cut into three bf16 levels
// (hi + mid + lo = the number, 24 significand bits), every product of a level
// and an element is exact, and the sums are fp32. The 16 rows (columns) of an
// instruction hold level * 4 + head, so the levels cost no extra instruction.
//
// A wave takes 32 positions at a time:
//   * scores: S = K q^T, two instructions rows x d / 32 steps; lane l loads the
//     16-byte chunk l / 16 (+ 4 per step) of position l % 16, which is the
//     operand as it is. The result of lane l is level * 4 + head = l % 16 at
//     positions 4 (l / 16) .. + 3; two DPP moves add the levels, so every lane
//     holds head l % 4 at 8 positions;
//   * softmax: reference maximum per head, the same in the whole wave, moved
//     lazily (as in the vector kernel) when some lane's score passes it;
//   * output: O += P V with P as the first operand: lane l already holds the
//     weights of row l % 16 at its 8 positions, and takes its level of them.
//     V comes as whole rows (lane l: chunk l % 16 of its 8 positions, four full
//     rows per load instruction), and one byte permute per pair of positions
//     turns the lane's 8 x 8 block, so instruction m of 8 yields the elements
//     8 (l % 16) + m. No lane exchange, no LDS, no barrier in the loop.
// A tile's K registers are refilled as soon as its scores are done, its V
// registers after its output, so one tile and a half is in flight per wave.
// MI355X, attention us, vector kernel -> this one: groups of four, d = 128, 1 x
// 8191 entries 13.0 -> 7.9, 4 x 32768 102 -> 81.4 (6.6 TB/s), 32 ragged sequences
// over an INT8 cache 96.6 -> 52.2 (5.4 TB/s). K by plain loads: with the
// non-temporal policy 71 instead of 63 us, by 16 instead of 8 bytes a lane 63 -> 57 us
// (INT8); V non-temporal: 84 us, plain 94 (4 x 32768).
// Non-finite cache entries: the mid and lo levels' contributions are dropped
// where they are not finite (0 * inf), the hi level alone then carries the
// infinity, as in the vector kernel's products. A score of -inf has weight 0
// beside a finite one of its wave (in the vector kernel the first score of a
// lane must be finite, else the head is NaN).
#include "attn_body.h"

namespace fasttps {

namespace {

using attn::kThreads;
using attn::merge_factor;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef attn::v2u v2u;

constexpr int kPos = 32;                            // positions per wave and tile
constexpr int kTileM = kAttnMfmaTile;               // positions per block and tile
static_assert(kTileM == kPos * (kThreads / kWave), "four waves of 32 positions");
constexpr int kLevels = 3;

template <int D, int G, int KVF>
struct alignas(16) MfmaSmem {
  float q[G][D];
  alignas(16) uint8_t knew[D * attn::kv_bytes<KVF>()];  // the new entry as stored
  alignas(16) uint8_t vnew[D * attn::kv_bytes<KVF>()];
  float o[kThreads / kWave][kLevels][G][D];  // the waves' o, per level
  float m[kThreads / kWave + 1][G];          // the waves' reference maxima; then the new entry's scores
  float l[kThreads / kWave][G];
};

// eight cache elements as loaded
template <int KVF>
using Chunk8 = typename std::conditional<KVF == kKvBf16, v4u, v2u>::type;

__device__ __forceinline__ bf16x8 as_bf16x8(v4u v) { return __builtin_bit_cast(bf16x8, v); }
__device__ __forceinline__ uint32_t top_halves(float lo, float hi) {
  return __builtin_amdgcn_perm(__float_as_uint(hi), __float_as_uint(lo), 0x07060302u);
}

// as bf16 (exact for every code)
template <int KVF>
__device__ __forceinline__ v4u to_bf16(v4u c) { return c; }
template <int KVF>
__device__ __forceinline__ v4u to_bf16(v2u c) {
  static_assert(KVF != kKvBf16, "8-bit codes");
  if constexpr (KVF == kKvFp8) {
    return v4u{__builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(c.x, 1.0f, false)),
               __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(c.x, 1.0f, true)),
               __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(c.y, 1.0f, false)),
               __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(c.y, 1.0f, true))};
  } else {
    float f[8];
    attn::decode_chunk<KVF>(c, f);
    return v4u{top_halves(f[0], f[1]), top_halves(f[2], f[3]), top_halves(f[4], f[5]), top_halves(f[6], f[7])};
  }
}

// The top half of a lane's level of x: level 0 keeps x (m1 = m2 = 0), level 1
// subtracts the truncation of x to bf16 (m1 = 0xFFFF0000), level 2 then that
// of the rest too (m2 = 0xFFFF0000). Truncations are exact numbers of 8
// significant bits, so the three levels add up to x.
__device__ __forceinline__ float level_of(float x, uint32_t m1, uint32_t m2) {
  const float r = x - __uint_as_float(__float_as_uint(x) & m1);
  return r - __uint_as_float(__float_as_uint(r) & m2);
}

// The sum over the lanes of a 16-lane row that share lane % 4, the same bits in
// all of them: by 8 first, then by 4, both steps add the same two numbers in
// every lane. (The level lanes cut one weight into its levels, so they must
// hold one weight; row_stride4_sum adds in another order in each lane.)
__device__ __forceinline__ float level_sum(float v) {
  v += dpp_mov<kDppRowRor8>(v);
  return v + dpp_mov<kDppRowRor4>(v);
}

__device__ __forceinline__ float finite_or_zero(float v) { return fabsf(v) < INFINITY ? v : 0.f; }

template <int D, int G, int KVF, bool PARTS>
__device__ __forceinline__ void attn_mfma_body(const AttnArgs& a, float kscale, float vscale) {
  using IO = attn::GlobalIO<PARTS>;
  using Smem = MfmaSmem<D, G, KVF>;
  using Body = attn::AttnBody<D, G, 1, false, KVF, IO, false, Smem>;
  using Chunk = Chunk8<KVF>;
  constexpr int NCH = D / 8;      // chunks of 8 elements per row
  constexpr int NS = D / 32;      // steps of the scores
  __shared__ Smem sm;
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  Body body(a, IO{}, sm, tid, blockIdx.x, blockIdx.y, a.order.p[blockIdx.z], true);
  const int P = body.P;
  body.own_new = (P / kTileM) % a.nsplit == body.s;  // the split whose tile holds slot P
  body.load_prologue();
  __builtin_amdgcn_sched_barrier(0);  // keep the prologue loads ahead of the tiles

  const int n = lane & 15, grp = lane >> 4;  // operand row (column), k group
  const int head = n & 3, level = n >> 2;
  const uint32_t m1 = level >= 1 ? 0xFFFF0000u : 0u, m2 = level >= 2 ? 0xFFFF0000u : 0u;
  const char* Kc = reinterpret_cast<const char*>(body.Kc);
  const char* Vc = reinterpret_cast<const char*>(body.Vc);
  constexpr int ROWB = D * attn::kv_bytes<KVF>();  // bytes of a cached row
  constexpr int CHB = sizeof(Chunk);
  const unsigned vch = (n < NCH ? n : NCH - 1) * CHB;  // lanes past the row repeat its last chunk

  // this wave's tiles: positions t0 .. t0 + 31, t0 + stride, ... below P. Rows
  // past the last cached entry repeat it (masked below)
  const int stride = a.nsplit * kTileM;
  int t0 = body.s * kTileM + wave * kPos;
  Chunk kr[2][NS], vr[8];
  // position k (of 8) of this lane's group within a tile
  auto pos_of = [&](int k) { return 16 * (k / 4) + 4 * grp + k % 4; };
  // byte offsets of this lane's rows within a tile: they change only when a
  // tile reaches past the last cached entry (rows past it repeat it), so the
  // loads of the others take no vector arithmetic (uniform base, lane offset)
  unsigned koff[2], voff[8];
  auto set_rows = [&](int last) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
      koff[h] = (unsigned)(min(16 * h + n, last) * ROWB) + 16u * grp;
#pragma unroll
    for (int k = 0; k < 8; ++k) voff[k] = (unsigned)(min(pos_of(k), last) * ROWB) + vch;
  };
  auto load_k = [&](int t) {
    const char* base = Kc + (size_t)t * ROWB;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if constexpr (KVF == kKvBf16) {
#pragma unroll
        for (int st = 0; st < NS; ++st) kr[h][st] = *reinterpret_cast<const Chunk*>(base + 64 * st + koff[h]);
      } else {
        // 16 bytes serve two steps, so that a load takes 64 bytes of a row
#pragma unroll
        for (int st = 0; st + 1 < NS; st += 2) {
          const v4u c = *reinterpret_cast<const v4u*>(base + 32 * st + koff[h]);
          kr[h][st] = Chunk{c.x, c.y};
          kr[h][st + 1] = Chunk{c.z, c.w};
        }
        if constexpr (NS % 2)
          kr[h][NS - 1] = *reinterpret_cast<const Chunk*>(base + 32 * (NS - 1) + (koff[h] - 8u * grp));
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  auto load_v = [&](int t) {
    const char* base = Vc + (size_t)t * ROWB;
#pragma unroll
    for (int k = 0; k < 8; ++k) vr[k] = ld_stream(reinterpret_cast<const Chunk*>(base + voff[k]));
    __builtin_amdgcn_sched_barrier(0);
  };
  // the first tile, unconditionally (a wave without one reads the last cached
  // entry, and slot 0 of an empty cache, and uses neither), so that the count
  // of loads behind the prologue's is known
  const int tp = min(t0, body.last);
  set_rows(body.last - tp);
  load_k(tp);
  load_v(tp);
  body.prologue(kscale, vscale);

  // this lane's column of q: its level of head n % 4 (zero past the group and
  // in the fourth level, which only pads)
  v4u qr[NS];
  // the first of the eight elements lane group grp holds in step st
  auto q_dim = [&](int st) {
    return KVF != kKvBf16 && st < NS / 2 * 2 ? 64 * (st / 2) + 16 * grp + 8 * (st % 2) : 32 * st + 8 * grp;
  };
#pragma unroll
  for (int st = 0; st < NS; ++st) {
    float f[8];
#pragma unroll
    for (int e = 0; e < 8; ++e)
      f[e] = head < G && level < kLevels ? level_of(sm.q[head < G ? head : 0][q_dim(st) + e], m1, m2) : 0.f;
    qr[st] = v4u{top_halves(f[0], f[1]), top_halves(f[2], f[3]), top_halves(f[4], f[5]), top_halves(f[6], f[7])};
  }
  // an 8-bit cache's K scale folds into the softmax scale
  const float scale = KVF == kKvBf16 ? a.scale : a.scale * kscale;

  float m = -INFINITY, l = 0.f;  // head n % 4: the wave's reference, this lane's share of the sum
  f4 o[8];                       // rows 4 grp + i: level grp, head i; column n: elements 8 n + mm
#pragma unroll
  for (int mm = 0; mm < 8; ++mm) o[mm] = f4{0.f, 0.f, 0.f, 0.f};

  // LAST: the wave's last tile, the only one that may reach past P (masked) and
  // the one that refills nothing
  auto tile = [&](int t, auto last_tag) {
    constexpr bool LAST = decltype(last_tag)::value;
    f4 s2[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      s2[h] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int st = 0; st < NS; ++st)
        s2[h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(to_bf16<KVF>(kr[h][st])), as_bf16x8(qr[st]), s2[h],
                                                        0, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (!LAST) {
      if (t + stride + kPos > P) set_rows(body.last - (t + stride));  // (uniform; the last refill)
      load_k(t + stride);
    }
    float sc[8], tot = 0.f, mx = -INFINITY;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      sc[k] = level_sum(s2[k / 4][k % 4]) * scale;
      tot += sc[k];
    }
    if (__any(!(fabsf(tot) < INFINITY))) {
      // some score is not finite: the lower levels' shares count only where
      // they are (rare; checked on the sum, one comparison for eight)
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const float v = s2[k / 4][k % 4];
        sc[k] = level_sum(level > 0 ? finite_or_zero(v) : v) * scale;
      }
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      if (LAST) sc[k] = t + pos_of(k) < P ? sc[k] : -INFINITY;
      mx = fmaxf(mx, sc[k]);
    }
    if (__any(mx > m + attn::kLazyRescale)) {
      // the heads whose scores pass their reference by more than the bound
      // move it to the wave's largest score; the others keep theirs
      mx = row_stride4_max(mx);
      mx = fmaxf(mx, __shfl_xor(mx, 16));
      mx = fmaxf(mx, __shfl_xor(mx, 32));
      const float mn = mx > m + attn::kLazyRescale ? mx : m;
      const float cf = merge_factor(m, mn);
      m = mn;
      l *= cf;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float ci = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(cf), i));
#pragma unroll
        for (int mm = 0; mm < 8; ++mm) o[mm][i] *= ci;
      }
    }
    float pl[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      float p = __expf(sc[k] - m);
      if (LAST) p = t + pos_of(k) < P ? p : 0.f;
      l += p;
      pl[k] = level_of(p, m1, m2);
    }
    const bf16x8 pa = as_bf16x8(v4u{top_halves(pl[0], pl[1]), top_halves(pl[2], pl[3]), top_halves(pl[4], pl[5]),
                                    top_halves(pl[6], pl[7])});
    v4u vv[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      vv[k] = to_bf16<KVF>(vr[k]);
      // a masked position's weight is zero, but the row it repeats may hold an infinity
      if (LAST) vv[k] = t + pos_of(k) < P ? vv[k] : v4u{0u, 0u, 0u, 0u};
    }
#pragma unroll
    for (int mm = 0; mm < 8; ++mm) {
      const uint32_t sel = mm % 2 ? 0x07060302u : 0x05040100u;
      v4u b;
#pragma unroll
      for (int r = 0; r < 4; ++r) b[r] = __builtin_amdgcn_perm(vv[2 * r + 1][mm / 2], vv[2 * r][mm / 2], sel);
      o[mm] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pa, as_bf16x8(b), o[mm], 0, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (!LAST) load_v(t + stride);
  };
  if (t0 < P) {
    for (; t0 + stride < P; t0 += stride) tile(t0, BoolTag<false>{});
    tile(t0, BoolTag<true>{});
  }

  // ---- merge: the waves' states and the new entry ------------------------------
  l += __shfl_xor(l, 16);
  l += __shfl_xor(l, 32);
  if (lane < G) {
    sm.m[wave][lane] = m;
    sm.l[wave][lane] = l;
  }
  if (grp < kLevels && n < NCH) {
#pragma unroll
    for (int i = 0; i < G; ++i) {
      f4* dst = reinterpret_cast<f4*>(&sm.o[wave][grp][i][8 * n]);
      dst[0] = f4{o[0][i], o[1][i], o[2][i], o[3][i]};
      dst[1] = f4{o[4][i], o[5][i], o[6][i], o[7][i]};
    }
  }
  // element e of the new entry's row in LDS (its rounded value)
  auto new_elem = [&](const uint8_t* row, int e) {
    if constexpr (KVF == kKvBf16) {
      return bf16_to_f32(reinterpret_cast<const uint16_t*>(row)[e]);
    } else {
      float f[4];
      attn::decode_word<KVF>(reinterpret_cast<const uint32_t*>(row)[e / 4], f);
      return e % 4 == 0 ? f[0] : e % 4 == 1 ? f[1] : e % 4 == 2 ? f[2] : f[3];
    }
  };
  // the new entry N_p (Eq. 1 slot): its score for head `wave`, by that wave
  float snew = -INFINITY;
  if (body.own_new && wave < G) {
    float t = 0.f;
    for (int e = lane; e < D; e += kWave) t = fmaf(sm.q[wave][e], new_elem(sm.knew, e), t);
    snew = wave_sum(t) * scale;
  }
  if (wave < G && lane == 0) sm.m[kThreads / kWave][wave] = snew;
  body.write_dbg();
  __syncthreads();
  for (int i = tid; i < G * D; i += kThreads) {
    const int h = i / D, e = i % D;
    float M = sm.m[kThreads / kWave][h];
#pragma unroll
    for (int w = 0; w < kThreads / kWave; ++w) M = fmaxf(M, sm.m[w][h]);
    const float fn = merge_factor(sm.m[kThreads / kWave][h], M);
    float L = fn, O = body.own_new ? fn * new_elem(sm.vnew, e) : 0.f;
#pragma unroll
    for (int w = 0; w < kThreads / kWave; ++w) {
      const float f = merge_factor(sm.m[w][h], M);
      L = fmaf(sm.l[w][h], f, L);
      const float ow = sm.o[w][0][h][e] + (finite_or_zero(sm.o[w][1][h][e]) + finite_or_zero(sm.o[w][2][h][e]));
      O = fmaf(ow, f, O);
    }
    const float ov = KVF == kKvBf16 ? O : O * vscale;  // an 8-bit cache's V scale
    if (a.direct) {
      attn::put_direct(a, body.b, body.g * G + h, e, D, ov, L);
      continue;
    }
    float* pr = body.io.rec(a, body.b, body.g * G + h, body.s, D);
    body.io.part(pr + kPartLead + e, ov);
    if (e == 0) {
      body.io.part(pr, M);
      body.io.part(pr + 1, L);
    }
  }
}

template <int D, int G, bool PARTS>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 8))) void attn_mfma_kernel(AttnArgs a) {
  attn_mfma_body<D, G, kKvBf16, PARTS>(a, 1.f, 1.f);
}
// 8-bit cache: the KV head's two scales come from the argument block
template <int D, int G, int KVF, bool PARTS>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 8))) void attn_mfma_kv8_kernel(
    AttnArgs a, KvScales sc) {
  attn_mfma_body<D, G, KVF, PARTS>(a, sc.k[blockIdx.y], sc.v[blockIdx.y]);
}

template <int D, int G, bool PARTS>
hipError_t launch_p(const AttnArgs& a, const KvScales* sc, hipStream_t s, KernelEvents ev) {
  const dim3 grid(a.nsplit, a.n_kv_heads, a.batch);
  switch (a.kv_format) {
    case kKvBf16:
      if constexpr (G >= 2) return ext_launch(attn_mfma_kernel<D, G, PARTS>, grid, dim3(kThreads), 0, s, ev, a);
      return hipErrorInvalidValue;
    case kKvFp8:
      return ext_launch(attn_mfma_kv8_kernel<D, G, kKvFp8, PARTS>, grid, dim3(kThreads), 0, s, ev, a, *sc);
    case kKvInt8:
      return ext_launch(attn_mfma_kv8_kernel<D, G, kKvInt8, PARTS>, grid, dim3(kThreads), 0, s, ev, a, *sc);
    default: return hipErrorInvalidValue;
  }
}

template <int D, int G>
hipError_t launch_g(const AttnArgs& a, const KvScales* sc, hipStream_t s, KernelEvents ev) {
  return a.qkv_part ? launch_p<D, G, true>(a, sc, s, ev) : launch_p<D, G, false>(a, sc, s, ev);
}

template <int D>
hipError_t launch_d(const AttnArgs& a, const KvScales* sc, hipStream_t s, KernelEvents ev) {
  switch (a.n_heads / a.n_kv_heads) {
    case 1:
      if constexpr (D > 64) return launch_g<D, 1>(a, sc, s, ev);
      return hipErrorInvalidValue;
    case 2: return launch_g<D, 2>(a, sc, s, ev);
    case 4: return launch_g<D, 4>(a, sc, s, ev);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

// Which steps run here; the line lies where the layer steps cross on MI355X
// (this kernel against the vector kernel, us a layer step; D the hidden size):
//   groups of four, every cache: D 4096, d 128, 8 x 4096 entries 61.1 against
//     69.3 (bf16), 56.1 against 59.8 (FP8); 1 x 8000 43.1 against 45.4
//   groups of two, bf16, d 96 and 128: d 128, 8 x 4096 83.6 against 86.7; 1 x
//     8000 50.0 against 52.7; D 1536, 16 KV heads, d 96, 1 x 16 26.7 against 26.9
//   groups of two, bf16, d 64: this kernel's prologue (the levels of q) costs
//     0.5 us more, which shorter loops do not win back; except between 65 and
//     128 positions, which are one tile here and two there (no combine launch).
//     D 1536, 8 and 16 KV heads: 1 x 200 23.8 against 23.3 and 25.2 against 24.7, 1 x
//     700 24.1 against 24.6 and 26.1 against 27.1; 4 x 64 30.7 against 30.0, 4 x 128
//     30.7 against 32.5; 4 x 200 (6400 rows) 33.2 against 32.6, 16 KV heads 8 x 500
//     (64000) 36.5 against 35.9, 16 x 500 (128000) 38.7 against 40.2
//   8-bit caches in smaller groups: from two sequences with 2^18 cached rows
//     up (about 512 positions per block), and not one head at d = 64 (half of
//     a load's lanes repeat): groups of two, d 128, 32 ragged 94.2 against
//     113.9; one head, d 96, 16 x 4096 109 against 114, 4 x 1000 40.7 against
//     39.9; d 64, 4 ragged INT8 44.8 against 41.9; at one sequence from 57 /
//     55 down to 40 / 34
//   groups of two at d 64 over 8-bit caches: from about 1090 positions per block
//     up. FP8 / INT8, 16 KV heads, D 2048, 8 x 4000 entries 48.2 / 49.8 against 47.9 /
//     48.2, 4 of 500-16000 (546k rows) 49.5 / 51.4 against 52.4 / 52.3; 32 KV heads, D
//     4096, 8 x 2100 96.6 / 97.8 against 95.1 / 95.7, 64 x 300 157.4 / 159.6 against
//     159.3 / 160.2, 8 x 4000 105.6 / 107.2 against 110.9 / 111.2
//   one head over a bf16 cache: never (d 96, 8 x 4096 99.9 against 96.1)
bool attention_on_mfma(const AttnShape& t) {
  // the accuracy study (bf16 caches only) keeps the vector kernel, which rounds
  // its weights; an 8-bit step ignores the switch
  if (t.p_bf16 && t.kv_format == kKvBf16) return false;
  if (t.group == 4) return true;
  if (t.kv_format == kKvBf16) {
    if (t.group != 2 || t.head_dim > 64) return t.group == 2;
    if (t.batch == 1) return t.max_pos > 2 * kAttnMfmaTile;
    return t.cached_rows > (1L << 16) || (t.max_pos > kAttnMfmaTile / 2 && t.max_pos <= kAttnMfmaTile);
  }
  if (t.batch < 2 || t.cached_rows < (1L << 18)) return false;
  if (t.head_dim > 64) return true;
  return t.group == 2 && t.cached_rows >= (17L << 15);
}

hipError_t launch_attention_mfma(const AttnArgs& a, const KvScales* sc, hipStream_t s, KernelEvents ev) {
  if (a.nsplit < 1 || a.nsplit > a.nsplit_cap) return hipErrorInvalidValue;
  if (a.p_bf16 && a.kv_format == kKvBf16) return hipErrorInvalidValue;
  if (a.kv_format != kKvBf16 && (!sc || a.n_kv_heads > kMaxKvHeads)) return hipErrorInvalidValue;
  switch (a.head_dim) {
    case 64: return launch_d<64>(a, sc, s, ev);
    case 96: return launch_d<96>(a, sc, s, ev);
    case 128: return launch_d<128>(a, sc, s, ev);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace fasttps
