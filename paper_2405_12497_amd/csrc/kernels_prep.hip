// Per-pair quantisation (Sec. 3.3.1) for codes of 5 to 16 words and B_q <= 4.
//
// The kernel is bound by vector issue: per coordinate a residual, its extrema
// and square, a random uniform, a rounding and a store. What keeps that short:
//   - a wave takes up to 8 consecutive pairs, nearly always of one query: the
//     query's coordinates and norm are read and summed once, the next pair's
//     centroid is in flight while this one computes, and the pairs' FP64
//     scalars are evaluated together, one pair per lane;
//   - SplitMix64's first half is shared by a pair's lanes. The generator's
//     state differs between the draws of a pair only in its low 12 bits, so
//     the sum with the golden-ratio increment has two possible upper parts
//     (with and without a carry), the first xor-shift and the high word's
//     product with the first multiplier are uniform, and a draw starts with one
//     xor and one 32 x 64 bit product instead of a 64-bit add, shift, xor and
//     a 64 x 64 bit product;
//   - quantised values stay in FP32 until they are stored, two per conversion.
// 1.28 M pairs at D = 768 take 800 us; a wave per pair with the whole generator
// per draw took 1250 us.
#include "rbq_internal.hpp"
#include "rbq_prep.hpp"
#include "wave_select.hpp"

// old with lane `lane` (uniform) set to the uniform value v.
__device__ int amdgcn_writelane(int v, int lane, int old) __asm("llvm.amdgcn.writelane.i32");

namespace rbq {
namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / kWave;
constexpr int kMaxPairs = 8;   // consecutive pairs per wave, at most

constexpr uint64_t kGolden = 0x9E3779B97F4A7C15ull, kMul1 = 0xBF58476D1CE4E5B9ull, kMul2 = 0x94D049BB133111EBull;
constexpr uint64_t kLow = 0xFFFull;   // state bits that differ between a pair's draws

// What a pair's draws share of SplitMix64, without or with a carry out of the
// low 12 bits of state + kGolden: the xor-shifted sum is (lo ^ l) for a draw's
// low bits l in the low word and a uniform high word, whose product with the
// low word of kMul1 is hp.
struct DrawBase {
  uint32_t lo, hp;
};
__device__ __forceinline__ DrawBase draw_base(uint64_t x) {   // x: the sum with its low 12 bits zero
  const uint64_t y = x ^ (x >> 30);
  DrawBase b;
  b.lo = (uint32_t)y;
  b.hp = (uint32_t)(y >> 32) * (uint32_t)kMul1;
  return b;
}

// The two 24-bit fields (bits 40..63 and 16..39 of the output) of the draw with
// low bits l.
__device__ __forceinline__ void draw_fields(uint32_t blo, uint32_t bhp, uint32_t l, uint32_t& f0, uint32_t& f1) {
  const uint32_t y = blo ^ l;
  uint64_t z = (uint64_t)y * (uint32_t)kMul1 + ((uint64_t)bhp << 32);
  z += (uint64_t)(y * (uint32_t)(kMul1 >> 32)) << 32;
  z = (z ^ (z >> 27)) * kMul2;
  const uint32_t hi = (uint32_t)(z >> 32);
  f0 = hi >> 8;                                                          // z ^ (z >> 31) leaves bits 33.. as they are
  f1 = (__builtin_amdgcn_alignbit(hi, (uint32_t)z, 16) ^ (hi >> 15)) & 0xFFFFFFu;
}

// Output formats: bit planes of every pair (popcount scan); the fragment
// scan's FP8 rows, and planes of the bootstrap pairs; plain int8 rows and
// planes of every pair (parity export).
enum { kPlanesOnly = 0, kFragments = 1, kPlain = 2 };

// W: words per code (exact). MIX: some draw of a pair has lanes with and
// without the carry (the host knows from the seed and W).
template <int W, int FMT, bool MIX>
__global__ __launch_bounds__(kThreads) void k_prep_wide(SearchDev s, int kPairs) {
  constexpr int T2 = (W + 1) / 2;   // draws per lane
  const int lane = lane_id();
  const int64_t npairs = s.nq * s.nprobe;
  // one query's pairs are consecutive: a contiguous run of blocks per XCD
  // reads the query's rotated vector into one L2
  const int64_t blk = xcd_block(blockIdx.x, gridDim.x);
  const int64_t g0 = uniform_i64((blk * kWaves + (threadIdx.x >> 6)) * kPairs);
  if (g0 >= npairs) return;
  // lane j < kPairs (a power of two): pair g0 + j's query, list (-1: past the query's nprobe) and
  // whether its bit planes are wanted
  const int64_t gl = min(g0 + (lane & (kPairs - 1)), npairs - 1);
  const int32_t ql = (int32_t)(gl / s.nprobe);
  const int32_t rl = (int32_t)(gl - (int64_t)ql * s.nprobe);
  const int32_t pr = s.probe[gl];
  const int32_t npq = s.nprobe_q ? s.nprobe_q[ql] : s.nprobe;
  const bool in = lane < kPairs && g0 + lane < npairs;
  const int32_t listl = in && rl < min(max(npq, 1), s.nprobe) ? pr : -1;
  uint64_t want_planes = ~0ull;
  if (FMT == kFragments) want_planes = __ballot(s.pair_choff[gl + ql] < s.q_p0[ql]);
  // draw t's low bits on this lane, and where they carry
  uint32_t low[T2];
  uint64_t carry[T2];
#pragma unroll
  for (int t = 0; t < T2; ++t) {
    const uint32_t v = (uint32_t)((s.seed & kLow) ^ (uint64_t)(t * kWave + lane)) + (uint32_t)(kGolden & kLow);
    low[t] = v & (uint32_t)kLow;
    carry[t] = __ballot(v > (uint32_t)kLow);
  }
  const uint64_t seed_hi = s.seed & ~kLow;
  const float fqmax = (float)s.qmax;
  const float q8_scale = frag_scale(lane);
  const uint32_t q8_at = (uint32_t)(FMT == kFragments ? frag_pos(lane) : lane);
  float x[W], c[W], cn[W];
  float qn = 0.f;
  int curq = -1;
  float o_min = 0.f, o_range = 0.f, o_b = 0.f;   // lane j: pair j's results
  int o_sq = 0;
  auto row_of = [&](int list, float (&v)[W]) {
    const char* p = reinterpret_cast<const char*>(s.crot + (int64_t)list * (W * kWave));
#pragma unroll
    for (int t = 0; t < W; ++t) v[t] = *reinterpret_cast<const float*>(p + 4u * (uint32_t)(t * kWave + lane));
  };
  const uint64_t act = __ballot(listl >= 0);
  int j = act ? (int)__builtin_ctzll(act) : kPairs;
  if (j < kPairs) row_of(__builtin_amdgcn_readlane(listl, j), c);
  while (j < kPairs) {
    const uint64_t rest = act & (~0ull << (j + 1));
    const int jn = rest ? (int)__builtin_ctzll(rest) : kPairs;
    const int list = __builtin_amdgcn_readlane(listl, j);
    const int64_t q = __builtin_amdgcn_readlane(ql, j);
    const int64_t g = g0 + j;
    if ((int)q != curq) {
      const char* p = reinterpret_cast<const char*>(s.qrot + q * (W * kWave));
#pragma unroll
      for (int t = 0; t < W; ++t) x[t] = *reinterpret_cast<const float*>(p + 4u * (uint32_t)(t * kWave + lane));
      float qq = 0.f;
#pragma unroll
      for (int t = 0; t < W; ++t) qq = fmaf(x[t], x[t], qq);
      qn = sqrtf(wave_sum(qq));
      curq = (int)q;
    }
    if (jn < kPairs) row_of(__builtin_amdgcn_readlane(listl, jn), cn);
    float rv[W];
    float ss = 0.f;
#pragma unroll
    for (int t = 0; t < W; ++t) rv[t] = x[t] - c[t];
    float rmin = rv[0], rmax = rv[0];
#pragma unroll
    for (int t = 0; t < W; ++t) {
      rmin = fminf(rmin, rv[t]);
      rmax = fmaxf(rmax, rv[t]);
      ss = fmaf(rv[t], rv[t], ss);
    }
    float b = uniform_f32(sqrtf(wave_sum(ss)));
    b = pair_norm(s, q, list, b, qn);
    rmin = wave_min(rmin);
    rmax = wave_max(rmax);
    const float range = rmax - rmin;
    const float scale = (b > 0.f) && (range > 0.f) ? fqmax / range : 0.f;
    // the pair's shared part of the generator, without and with a carry
    const uint64_t xs = ((seed_hi ^ (((uint64_t)(s.qid_base + q) << 40) + ((uint64_t)(uint32_t)list << 12))) & ~kLow) +
                        (kGolden & ~kLow);
    const DrawBase d0 = draw_base(xs), d1 = draw_base(xs + (kLow + 1));
    float qf[W];
    float sum = 0.f;
#pragma unroll
    for (int t = 0; t < T2; ++t) {
      uint32_t blo, bhp, f0, f1;
      if constexpr (MIX) {
        const bool cy = (carry[t] >> lane) & 1;
        blo = cy ? d1.lo : d0.lo;
        bhp = cy ? d1.hp : d0.hp;
      } else {
        blo = carry[t] ? d1.lo : d0.lo;
        bhp = carry[t] ? d1.hp : d0.hp;
      }
      draw_fields(blo, bhp, low[t], f0, f1);
      qf[2 * t] = round_even_word(rv[2 * t], rmin, scale, f0, fqmax);
      sum += qf[2 * t];
      if (2 * t + 1 < W) {
        qf[2 * t + 1] = round_odd_word(rv[2 * t + 1], rmin, scale, f1, fqmax);
        sum += qf[2 * t + 1];
      }
    }
    const int sq = wave_sum_i((int)sum);
    if constexpr (FMT == kFragments) {
      int8_t* q8 = s.qu8 + g * (W * kWave);
#pragma unroll
      for (int t = 0; t < T2; ++t) {
        const bool two = 2 * t + 1 < W;
        const int v = __builtin_amdgcn_cvt_pk_fp8_f32(qf[2 * t] * q8_scale, two ? qf[two ? 2 * t + 1 : 0] * q8_scale : 0.f,
                                                      0, false);
        q8[(uint32_t)(2 * t * kWave) + q8_at] = (int8_t)v;
        if (two) q8[(uint32_t)((2 * t + 1) * kWave) + q8_at] = (int8_t)(v >> 8);
      }
    } else if constexpr (FMT == kPlain) {
      int8_t* q8 = s.qu8 + g * (W * kWave);
#pragma unroll
      for (int t = 0; t < W; ++t) q8[(uint32_t)(t * kWave) + q8_at] = (int8_t)((int)qf[t] - s.qoff);
    }
    if (FMT != kFragments || ((want_planes >> j) & 1)) {
      // lane k < 4 W ends with plane word k (plane k / W, word k % W)
      int wlo = 0, whi = 0;
#pragma unroll
      for (int t = 0; t < W; ++t) {
        const int qi = (int)qf[t];
#pragma unroll
        for (int jb = 0; jb < 4; ++jb) {
          const uint64_t w = __ballot((qi >> jb) & 1);
          wlo = amdgcn_writelane((int)(uint32_t)w, jb * W + t, wlo);
          whi = amdgcn_writelane((int)(uint32_t)(w >> 32), jb * W + t, whi);
        }
      }
      if (lane < 4 * W) s.planes[g * (4 * W) + lane] = ((uint64_t)(uint32_t)whi << 32) | (uint32_t)wlo;
    }
    if (s.metric != 0) pair_ip_term(s, g, q, list);
    o_min = lane == j ? rmin : o_min;
    o_range = lane == j ? range : o_range;
    o_b = lane == j ? b : o_b;
    o_sq = lane == j ? sq : o_sq;
#pragma unroll
    for (int t = 0; t < W; ++t) c[t] = cn[t];
    j = jn;
  }
  if (in) s.pairs[g0 + lane] = listl >= 0 ? pair_record(s, o_min, o_range, o_b, o_sq, listl) : empty_record();
}

template <int W>
void launch_w(const SearchDev& s, dim3 grid, int per, bool mix, hipStream_t st) {
  auto run = [&](auto fmt) {
    constexpr int FMT = decltype(fmt)::value;
    if (mix)
      hipLaunchKernelGGL((k_prep_wide<W, FMT, true>), grid, dim3(kThreads), 0, st, s, per);
    else
      hipLaunchKernelGGL((k_prep_wide<W, FMT, false>), grid, dim3(kThreads), 0, st, s, per);
  };
  if (s.frag)
    run(IntC<kFragments>{});
  else if (s.qu8)
    run(IntC<kPlain>{});
  else
    run(IntC<kPlanesOnly>{});
}

}  // namespace

bool launch_prep_wide(const SearchDev& s, hipStream_t st) {
  if (s.npl != 4 || s.W < 5 || s.W > 16) return false;
  const int64_t npairs = s.nq * s.nprobe;
  // The draws of word pair t have low bits (seed ^ (64 t + lane)) mod 2^12: an
  // aligned run of 64, which carries as a whole unless it holds the boundary
  // 2^12 - (kGolden mod 2^12).
  const uint32_t edge = (uint32_t)((kLow + 1 - (kGolden & kLow)) >> 6);
  bool mix = false;
  for (int t = 0; t < (s.W + 1) / 2; ++t) mix = mix || (((uint32_t)(s.seed & kLow) >> 6) ^ (uint32_t)t) == edge;
  // as many pairs per wave as leave 8192 waves (8 per SIMD): 2048 pairs at
  // D = 960 take 9 us a pair per wave and 20 us eight
  int per = 1;
  while (per < kMaxPairs && npairs >= (int64_t)2 * per * 8192) per *= 2;
  const dim3 grid((unsigned)((npairs + per * kWaves - 1) / (per * kWaves)));
  switch (s.W) {
    case 5: launch_w<5>(s, grid, per, mix, st); break;
    case 6: launch_w<6>(s, grid, per, mix, st); break;
    case 7: launch_w<7>(s, grid, per, mix, st); break;
    case 8: launch_w<8>(s, grid, per, mix, st); break;
    case 9: launch_w<9>(s, grid, per, mix, st); break;
    case 10: launch_w<10>(s, grid, per, mix, st); break;
    case 11: launch_w<11>(s, grid, per, mix, st); break;
    case 12: launch_w<12>(s, grid, per, mix, st); break;
    case 13: launch_w<13>(s, grid, per, mix, st); break;
    case 14: launch_w<14>(s, grid, per, mix, st); break;
    case 15: launch_w<15>(s, grid, per, mix, st); break;
    default: launch_w<16>(s, grid, per, mix, st); break;
  }
  return true;
}

}  // namespace rbq
