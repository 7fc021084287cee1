// Batched scan for B_q <= 4 and codes up to 16 words: the integer <x_b, q_u>
// of Sec. 3.3.2 for 32 codes x 32 quantised queries at a time on
// v_mfma_scale_f32_32x32x64_f8f6f4, codes as FP4 and queries as FP6.
//
// Why this form. The contraction itself is cheap (a 32 x 32 block at D = 768
// takes 12 matrix instructions of 32 cycles); what the scan spends its time on
// is the vector work beside it: turning code bits into operand values, the
// estimator and bound of every output, and writing the candidates. So
//   - a 32-wide block: each expanded code serves 32 queries (a 16 x 16 block
//     of v_mfma_i32_16x16x64_i8 expands every code twice as often);
//   - FP4 codes: E2M1 holds 0.5, 1 and 2 as a single bit, so one AND per eight
//     code bits leaves bit n of a nibble in place as a value (the fourth bit
//     takes a shift: its own place is the sign);
//   - FP6 queries: E2M3 holds q / 2, q / 4 and q / 8 for q <= 15 exactly, which
//     makes every product q / 4; the block scale 2^2 returns q, and the FP32 sum
//     of integers below 2^24 is <x_b, q_u> exactly. FP6 x FP4 runs at 32 cycles
//     per instruction, FP8 x FP4 at 64 and int8 at 64 per 64 dimensions, and
//     the queries' fragments take 6 W registers instead of 8 W;
//   - a lane owns one query (the output's column), so the query's constants
//     sit in registers; the 32 codes' factors come from LDS by broadcast reads;
// Per 32 x 32 block at W = 12 that is 290 vector instructions where four
// 16 x 16 int8 blocks took about 680.
// Bound by their issue and by the candidates' stores: 10,000 queries x 128 lists of
// 2 M codes at D = 768 take 1115 us (2343 on 16 x 16 int8 blocks), 256 x 8 lists at
// D = 960 72 us (90).
#include "rbq_internal.hpp"
#include "rbq_runtime.hpp"
#include "scan_code.hpp"
#include "wave_select.hpp"

namespace rbq {
namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / kWave;
constexpr int kMaxFragW = 16;   // code words whose query fragments fit in registers

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef unsigned u32x6 __attribute__((ext_vector_type(6)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x32 __attribute__((ext_vector_type(32)));

// Operand layouts of v_mfma_scale_f32_32x32x64_f8f6f4 with FP4 A and FP6 B, as
// measured on gfx950: lane l holds row (column) l % 32 and, in element e < 32,
// k = 32 (l / 32) + e; output register i of lane l is row 8 (i / 4) + 4 (l / 32)
// + i % 4 of column l % 32. A K step takes 32 code bits w per lane (a half word);
// element e = 8 m + n carries dimension 4 n + m of the half: nibble n of code
// dword w & (0x11111111 << m) (m = 3: (w >> 1) & 0x44444444) is that dimension's
// bit worth 0.5, 1, 2 or 2, and byte 8 m + n of the query's half word holds the
// dimension's q_u times 0.5, 0.25, 0.125 or 0.125 (frag_pos, frag_scale: FP8 in
// memory).

// Wait states between the last product of a block and the first read of its
// result. The compiler's own distance after a scaled product of mixed formats
// has been too short on gfx950; the accumulator passes through the wait.
__device__ __forceinline__ void result_wait(f32x16& acc) {
  asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7" : "+v"(acc));
}

// 32 FP8 values in memory order -> the FP6 fragment (every value is exact in
// FP8, FP16 and FP6).
__device__ __forceinline__ u32x6 fp6_fragment(const i32x4& lo, const i32x4& hi) {
  f16x32 h;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int v = i < 4 ? lo[i & 3] : hi[i & 3];
    const f16x2 a = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(v, 1.0f, false);
    const f16x2 b = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(v, 1.0f, true);
    h[4 * i] = a[0];
    h[4 * i + 1] = a[1];
    h[4 * i + 2] = b[0];
    h[4 * i + 3] = b[1];
  }
  return __builtin_amdgcn_cvt_scalef32_pk32_fp6_f16(h, 1.0f);
}

// LDS of one wave: the block's 32 code factors {G, H, popcount, code term}, and
// for the candidates of a block the bounds of its 32 x 32 outputs
// ([register / 4][lane][register % 4]).
struct WaveLds {
  float4 fac[32];
  float4 low[4][kWave];
};

// What a lane holds of its query (column): the estimator's constants, the
// threshold tau - pt, where its candidates go, and the outputs that may become
// candidates: all 16, or none where the column is not scanned (past the unit's
// pairs, or a chunk the bootstrap has scanned). Its segment then belongs to
// another column or to the bootstrap, so no value of a bound may let it store.
struct Column {
  float a1, a2, a0, coefh, pt, thr;
  uint32_t live;   // 0xFFFF or 0
  Cand* seg;
};

// A block of 32 codes as a lane loads it: lane group g takes both halves of
// code words 2 p + g (one 8-byte load each; the two halves are the K steps 2 p
// and 2 p + 1), and of an odd last word its half; the code's scan factors and
// inner-product term.
template <int WS>
struct Block {
  uint2 w[WS / 2 > 0 ? WS / 2 : 1];
  uint32_t last;
  float2 sf;
  float fi;
};

// Next-unit hook of frag_unit: called once, early in the unit.
struct NoHook {
  __device__ __forceinline__ void operator()() const {}
};

// One unit on one wave: codes [start, start + n) of a list against the 32
// queries whose fragments are fq. Candidates (bound without the pair term <=
// thr) are appended to each column's segment in code order; returns how many
// this lane's column has.
// The next block's loads are issued before this block's products and waited for
// before its candidates are stored: stores and loads share one in-order
// counter, so a load waited for after them would wait for their completion too.
template <bool DEBUG, int WS, class Hook>
__device__ __forceinline__ int frag_unit(const SearchDev& s, int64_t start, int n, const Column& c, const u32x6 (&fq)[WS],
                                         WaveLds& L, Hook hook, const PairRec* rec, int32_t* dbg_ip, int32_t* dbg_pc,
                                         float* dbg_est, float* dbg_dist, float* dbg_lb, int64_t dbg_base) {
  const int lane = lane_id();
  const int col = lane & 31, grp = lane >> 5;
  constexpr int NP = WS / 2;
  // wave-uniform bases (the unit's first 64-code row, its first factors) and
  // 32-bit byte offsets: position x = o0 + r of unit code r has word w at
  // ((x >> 6) W + w) 64 + (x & 63)
  const int o0 = (int)(start & 63);
  const char* cbase = reinterpret_cast<const char*>(s.codes) + (size_t)(start >> 6) * WS * 512;
  const char* cbase4 = cbase + 4096;   // words 8..: within the loads' immediate offsets
  const char* sbase = reinterpret_cast<const char*>(s.sfac + start);
  const char* fbase = s.metric != 0 ? reinterpret_cast<const char*>(s.fip + start) : nullptr;
  // codes past the end load the last one; their outputs are dropped
  auto load = [&](int rb, Block<WS>& k) {
    const uint32_t r = (uint32_t)min(rb + col, n - 1);
    const uint32_t x = (uint32_t)o0 + r;
    const uint32_t wb = 8u * ((x >> 6) * (uint32_t)WS * 64u + (x & 63u));
    const uint32_t wg = wb + 512u * (uint32_t)grp;
#pragma unroll
    for (int p = 0; p < NP; ++p)
      k.w[p] = *reinterpret_cast<const uint2*>((p < 4 ? cbase : cbase4) + (wg + 1024u * (uint32_t)(p & 3)));
    if constexpr (WS % 2 == 1)
      k.last = *reinterpret_cast<const uint32_t*>((WS > 8 ? cbase4 : cbase) +
                                                  (wb + 512u * (uint32_t)((WS - 1) & 7) + 4u * (uint32_t)grp));
    k.sf = *reinterpret_cast<const float2*>(sbase + 8u * r);
    if (fbase != nullptr) k.fi = *reinterpret_cast<const float*>(fbase + 4u * r);
  };
  int count = 0;
  auto block = [&](int rb, const Block<WS>& k, Block<WS>& next) {
    if (rb + 32 < n) load(rb + 32, next);
    f32x16 acc;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.f;
    int pcp = 0;
    auto step = [&](uint32_t w, int t) {
      pcp += __popc(w);
      const i32x8 a = {(int)(w & 0x11111111u), (int)(w & 0x22222222u), (int)(w & 0x44444444u),
                       (int)((w >> 1) & 0x44444444u), 0, 0, 0, 0};
      const i32x8 b = {(int)fq[t][0], (int)fq[t][1], (int)fq[t][2], (int)fq[t][3], (int)fq[t][4], (int)fq[t][5], 0, 0};
      // formats: A FP4 (4), B FP6 E2M3 (2); E8M0 scales 2^0 and 2^2
      acc = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, acc, 4, 2, 0, 127, 0, 129);
    };
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      step(k.w[p].x, 2 * p);
      step(k.w[p].y, 2 * p + 1);
    }
    if constexpr (WS % 2 == 1) step(k.last, WS - 1);
    // the two lane groups hold the two halves of the code's bits
    const auto sw = __builtin_amdgcn_permlane32_swap((uint32_t)pcp, (uint32_t)pcp, false, false);
    const int pc = (int)(sw[0] + sw[1]);
    if (grp == 0) {
      const float ct = fbase != nullptr ? -k.fi : code_term_l2(k.sf);
      L.fac[col] = make_float4(k.sf.x, k.sf.y, (float)pc, ct);
    }
    wave_lds_sync();
    const int left = n - rb;   // codes of the block that exist, if below 32
    // bounds without the pair term (as est_y / est_dl on the integer product);
    // pass: bit 15 - i is the test of output i (an ordered compare, so that a NaN
    // bound or threshold fails as in the other scans; the sign of thr - bound, which
    // a NaN may pass, is 1% faster: 1087 to 1105 us of 10,000 queries x 128 lists at
    // D = 768, compared 1106 to 1136). The factors are read two outputs ahead:
    // left alone, the compiler reads each right before its use to save registers
    // and waits 16 times.
    float low[16];
    uint32_t pass = 0;
    float4 fc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i) fc[0][i] = L.fac[4 * grp + i];
    result_wait(acc);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      if ((i & 1) == 0 && i < 14) {
#pragma unroll
        for (int e = 0; e < 2; ++e) fc[((i >> 1) + 1) & 1][e] = L.fac[8 * ((i + 2) >> 2) + 4 * grp + ((i + 2) & 3) + e];
        asm volatile("" ::: "memory");
      }
      const float4 f = fc[(i >> 1) & 1][i & 1];
      const float y = fmaf(c.a1, acc[i], fmaf(c.a2, f.z, c.a0));
      const float d0 = fmaf(f.x, y, f.w);
      low[i] = fmaf(c.coefh, f.y, d0);
      if constexpr (DEBUG) {
        const int code = 8 * (i >> 2) + 4 * grp + (i & 3);
        if (col == 0 && code < left) {
          const int64_t o = start + rb + code - dbg_base;
          dbg_ip[o] = (int)acc[i];
          dbg_pc[o] = (int)f.z;
          dbg_est[o] = estimate_est(*rec, s.fac[start + rb + code].y, (int)acc[i], (int)f.z);
          dbg_dist[o] = d0 + c.pt;
          dbg_lb[o] = low[i] + c.pt;
        }
      } else {
        pass = pass + pass + (low[i] <= c.thr ? 1u : 0u);
      }
    }
    if constexpr (!DEBUG) {
      uint32_t mask = pass & c.live;   // bit 15 - i: output i is a candidate
      if (left < 32) {   // the last block: codes past the end
        const uint32_t v = ~(0xFFFFFFFFu >> left) << (4 * grp);   // this lane's codes: its nibbles from bit 31 down
        mask &= ((v >> 16) & 0xF000u) | ((v >> 12) & 0x0F00u) | ((v >> 8) & 0x00F0u) | ((v >> 4) & 0x000Fu);
      }
#pragma unroll
      for (int p = 0; p < NP; ++p) {
        keep_loaded(next.w[p].x);
        keep_loaded(next.w[p].y);
      }
      if constexpr (WS % 2 == 1) keep_loaded(next.last);
      keep_loaded(next.sf.x);
      keep_loaded(next.fi);
      if (__ballot(mask != 0u) != 0ull) {
        // the column's 32 codes in order, first code at bit 31: this lane's
        // groups of four between its partner's
        uint32_t sp = (mask | (mask << 8)) & 0x00FF00FFu;
        sp = (sp | (sp << 4)) & 0x0F0F0F0Fu;
        const auto pr = __builtin_amdgcn_permlane32_swap(sp, sp, false, false);
        const uint32_t all = ((uint32_t)pr[0] << 4) | (uint32_t)pr[1];
#pragma unroll
        for (int j = 0; j < 4; ++j) L.low[j][lane] = make_float4(low[4 * j], low[4 * j + 1], low[4 * j + 2], low[4 * j + 3]);
        wave_lds_sync();
        // each lane's passing outputs one after the other (a few per lane)
        uint32_t m = mask << 16;
        while (__ballot(m != 0u) != 0ull) {
          if (m != 0u) {
            const int i = __clz((int)m);
            m &= ~(0x80000000u >> i);
            const int code = 8 * (i >> 2) + 4 * grp + (i & 3);
            Cand cd;
            cd.pos = (int32_t)start + rb + code;
            cd.lb = reinterpret_cast<const float*>(&L.low[i >> 2][lane])[i & 3] + c.pt;
            c.seg[count + __popc(all & ~(0xFFFFFFFFu >> code))] = cd;
          }
        }
        count += __popc(all);
      }
    }
    wave_lds_sync();   // the next block's values overwrite these
  };
  Block<WS> A, B;
  load(0, A);
  B = A;
  hook();
  for (int rb = 0; rb < n; rb += 64) {
    block(rb, A, B);
    if (rb + 32 < n) block(rb + 32, B, A);
  }
  return count;
}

template <int WS>
__device__ __forceinline__ void load_fragments(const int8_t* row, int grp, u32x6 (&fq)[WS]) {
  // K step t: half t % 2 of word t - t % 2 + grp; of an odd last word half grp
#pragma unroll
  for (int t = 0; t < WS; ++t) {
    const i32x4* p = reinterpret_cast<const i32x4*>(
        row + (t == WS - 1 && WS % 2 == 1 ? 64 * t + 32 * grp : 64 * (t - t % 2 + grp) + 32 * (t % 2)));
    fq[t] = fp6_fragment(p[0], p[1]);
  }
}

// Work units (MfUnit: list chunk x group of 32 pairs, ordered by list, then
// chunk, then group) are cut into kScanSlices contiguous slices; a workgroup
// starts on the slice of its XCD (workgroups go to the XCDs in turn), so the
// groups of one chunk run on one XCD and share its L2, then moves on to the
// other slices.
struct Slices {
  int64_t total;
  int64_t lo, size, own;   // current slice: first unit, units, units given to its waves
  unsigned long long* ctr;
  int x0, j;
  // The slice's first units belong to the waves that start on it, one each; the
  // rest are claimed from its counter. A counter is only added to where it can
  // have units left (4096 waves that each tried all eight took 100 us on their
  // addresses).
  __device__ __forceinline__ void open(const SearchDev& s) {
    const int x = (x0 + j) % kScanSlices;
    lo = total * x / kScanSlices;
    size = total * (x + 1) / kScanSlices - lo;
    own = (int64_t)kWaves * ((gridDim.x + kScanSlices - 1 - x) / kScanSlices);
    ctr = s.counters + kScanSliceCtr + kScanSliceStride * x;
  }
  __device__ __forceinline__ uint32_t issue() const {   // a claim's ticket, in lane 0
    uint32_t t = 0;
    if (lane_id() == 0) t = (uint32_t)atomicAdd(ctr, 1ull);
    return t;
  }
  // The unit of a ticket, or (slice exhausted) of a claim on the next slice
  // that has one; -1: no unit is left.
  __device__ __forceinline__ int64_t take(const SearchDev& s, int64_t at) {
    for (;;) {
      if (at < size) return lo + at;
      for (;;) {
        if (++j >= kScanSlices) return -1;
        open(s);
        const uint32_t seen = (uint32_t)__hip_atomic_load(ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (own + uniform_i32((int)seen) < size) break;
      }
      at = own + uniform_i32((int)issue());
    }
  }
};

template <int WS>
__global__ __launch_bounds__(kThreads, WS <= 6 ? 4 : WS <= 12 && WS != 11 ? 3 : 2) void k_scan_frag(SearchDev s) {
  __shared__ WaveLds lds[kWaves];
  WaveLds& L = lds[threadIdx.x / kWave];
  const int lane = lane_id(), col = lane & 31, grp = lane >> 5;
  Slices sl;
  sl.total = uniform_i64(s.mf_unit_off[s.nlist]);
  sl.x0 = (int)(blockIdx.x % kScanSlices);
  sl.j = 0;
  sl.open(s);
  int64_t at = uniform_i64((int64_t)kWaves * (blockIdx.x / kScanSlices) + threadIdx.x / kWave);
  int64_t u = sl.take(s, at);
  while (u >= 0) {
    const MfUnit un = s.mf_units[u];
    const int64_t start = uniform_i32(un.start);
    const int n = uniform_i32(un.n), slot = uniform_i32(un.slot), cr = uniform_i32(un.chunk_rows);
    const int ch = cr >> 5, nrow = (cr & 31) + 1;
    const MfRow row = s.mf_rows[slot + min(col, nrow - 1)];
    const bool live = col < nrow && ch >= row.first;
    // the next unit's claim travels while this one runs, unless the slice is
    // about to end (a wave that holds a unit it has not begun delays the end)
    const int64_t here = u - sl.lo;
    const bool ahead = here + 2 * sl.own < sl.size;
    uint32_t ticket = 0;
    int64_t nu = -2;
    if (ahead) ticket = sl.issue();
    if (__ballot(live) != 0ull) {   // else every pair scanned this chunk in the bootstrap
      u32x6 fq[WS];
      load_fragments<WS>(s.qu8 + (int64_t)row.g * (64 * WS), grp, fq);
      Column c;
      c.a1 = row.a1;
      c.a2 = row.a2;
      c.a0 = row.a0;
      c.coefh = row.coefh;
      c.pt = row.pt;
      c.thr = row.thr;
      c.live = live ? 0xFFFFu : 0u;
      c.seg = s.seg + row.seg + (int64_t)ch * s.chunk;
      const int count = frag_unit<false, WS>(s, start, n, c, fq, L, [&]() {
        if (ahead) nu = sl.take(s, sl.own + uniform_i32((int)ticket));
      }, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, 0);
      if (live && grp == 0) s.seg_count[row.count + ch] = count;
    }
    if (nu == -2) {
      if (!ahead) {
        if (sl.own < sl.size) ticket = sl.issue();
        else ticket = 0;   // nothing to claim on this slice: take() moves on
      }
      nu = sl.take(s, sl.own + uniform_i32((int)ticket));
    }
    u = nu;
  }
}

// Debug: one caller-given quantised query (column 0) against a whole list, one
// wave per chunk, through the unit code the search runs.
template <int WS>
__global__ __launch_bounds__(kWave) void k_debug_frag(SearchDev s, const PairRec* recp, const int8_t* qu8, int32_t list,
                                                      int32_t* ip, int32_t* pc, float* est, float* dist, float* lb) {
  __shared__ WaveLds L;
  const float hwk = s.eps0 / sqrtf((float)(s.dp - 1));
  const PairTerms t = s.metric != 0 ? pair_terms_ip(*recp, hwk, s.pair_pt[0]) : pair_terms(*recp, hwk);
  const int64_t lbeg = uniform_i32(s.list_off[list]), lend = uniform_i32(s.list_off[list + 1]);
  const int64_t start = lbeg + (int64_t)blockIdx.x * s.chunk;
  const int64_t end = lend < start + s.chunk ? lend : start + s.chunk;
  if (start >= end) return;
  u32x6 fq[WS];
  load_fragments<WS>(qu8, lane_id() >> 5, fq);
  Column c;
  c.a1 = t.a1;
  c.a2 = t.a2;
  c.a0 = t.a0;
  c.coefh = t.coefh;
  c.pt = t.pt;
  c.thr = -__builtin_inff();
  c.live = 0u;
  c.seg = nullptr;
  (void)frag_unit<true, WS>(s, start, (int)(end - start), c, fq, L, NoHook{}, recp, ip, pc, est, dist, lb, lbeg);
}

template <bool DBG>
const void* frag_kernel(int W) {
#define RBQ_FR(WS_) \
  case WS_: return DBG ? (const void*)k_debug_frag<WS_> : (const void*)k_scan_frag<WS_>
  switch (W) {
    RBQ_FR(1);
    RBQ_FR(2);
    RBQ_FR(3);
    RBQ_FR(4);
    RBQ_FR(5);
    RBQ_FR(6);
    RBQ_FR(7);
    RBQ_FR(8);
    RBQ_FR(9);
    RBQ_FR(10);
    RBQ_FR(11);
    RBQ_FR(12);
    RBQ_FR(13);
    RBQ_FR(14);
    RBQ_FR(15);
    RBQ_FR(16);
    default: return nullptr;
  }
#undef RBQ_FR
}

}  // namespace

bool scan_frag_available(int W, int npl) { return npl == 4 && W >= 1 && W <= kMaxFragW; }

int scan_frag_blocks_per_cu(int W) {
  int v = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&v, frag_kernel<false>(W), kThreads, 0) != hipSuccess || v < 1) v = 1;
  return v;
}

hipError_t launch_scan_frag(const SearchDev& s, int grid, hipStream_t st) {
  void* args[] = {(void*)&s};
  return hipLaunchKernel(frag_kernel<false>(s.W), dim3(grid), dim3(kThreads), args, 0, st);
}

hipError_t launch_debug_frag(const SearchDev& s, const PairRec* rec, const int8_t* qu8, int32_t list, int nchunks,
                             int32_t* ip, int32_t* pc, float* est, float* dist, float* lb, hipStream_t st) {
  void* args[] = {(void*)&s,  (void*)&rec, (void*)&qu8,  (void*)&list, (void*)&ip,
                  (void*)&pc, (void*)&est, (void*)&dist, (void*)&lb};
  return hipLaunchKernel(frag_kernel<true>(s.W), dim3(nchunks), dim3(kWave), args, 0, st);
}

}  // namespace rbq
