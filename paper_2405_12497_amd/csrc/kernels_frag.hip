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
//     sit in registers; the 32 codes' factors come from LDS by broadcast reads.
// Per 32 x 32 block at W = 12 that is about 270 vector instructions where four
// 16 x 16 int8 blocks took about 680.
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
// + i % 4 of column l % 32. Element e = 8 m + n of lane group g carries
// dimension 64 t + 32 g + 4 n + m of code word t: nibble n of code dword
// w & (0x11111111 << m) (m = 3: (w >> 1) & 0x44444444) is that dimension's bit
// worth 0.5, 1, 2 or 2, and byte 8 m + n of the query row holds the dimension's
// q_u times 0.5, 0.25, 0.125 or 0.125 (frag_pos, frag_scale: FP8 in memory).

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

// LDS of one wave: the block's 32 code factors {G, H, popcount, code term} and
// the bounds of its 32 x 32 outputs ([register / 4][lane][register % 4]).
struct WaveLds {
  float4 fac[32];
  float4 low[4][kWave];
};

// What a lane holds of its query (column): the estimator's constants, the
// threshold tau - pt (-inf where the column is not scanned: no bound passes),
// and where its candidates go.
struct Column {
  float a1, a2, a0, coefh, pt, thr;
  Cand* seg;
};

// One unit on one wave: codes [start, start + n) of a list against the 32
// queries whose fragments are fq. Candidates (bound without the pair term <=
// thr) are appended to each column's segment in code order; returns how many
// this lane's column has.
template <bool DEBUG, int WS>
__device__ int frag_unit(const SearchDev& s, int64_t start, int n, const Column& c, const u32x6 (&fq)[WS], WaveLds& L,
                         const PairRec* rec, int32_t* dbg_ip, int32_t* dbg_pc, float* dbg_est, float* dbg_dist,
                         float* dbg_lb, int64_t dbg_base) {
  const int lane = lane_id();
  const int col = lane & 31, grp = lane >> 5;
  // wave-uniform bases (the unit's first 64-code row, its first factors) and
  // 32-bit byte offsets: position x = o0 + r of unit code r has word w at
  // ((x >> 6) W + w) 64 + (x & 63)
  const int o0 = (int)(start & 63);
  const char* cbase = reinterpret_cast<const char*>(s.codes) + (size_t)(start >> 6) * WS * 512;
  const char* sbase = reinterpret_cast<const char*>(s.sfac + start);
  const char* fbase = s.metric != 0 ? reinterpret_cast<const char*>(s.fip + start) : nullptr;
  uint32_t cw[WS];
  float2 sf;
  float fi = 0.f;
  // this lane's half of every word of its code (past the end: the last code,
  // whose outputs are dropped), its factors and inner-product term
  auto load = [&](int rb) {
    const uint32_t r = (uint32_t)min(rb + col, n - 1);
    const uint32_t x = (uint32_t)o0 + r;
    const uint32_t wb = 8u * ((x >> 6) * (uint32_t)WS * 64u + (x & 63u)) + 4u * (uint32_t)grp;
#pragma unroll
    for (int t = 0; t < WS; ++t) cw[t] = *reinterpret_cast<const uint32_t*>(cbase + (wb + 512u * (uint32_t)t));
    sf = *reinterpret_cast<const float2*>(sbase + 8u * r);
    if (fbase != nullptr) fi = *reinterpret_cast<const float*>(fbase + 4u * r);
  };
  int count = 0;
  load(0);
  for (int rb = 0; rb < n; rb += 32) {
    f32x16 acc;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.f;
    int pcp = 0;
#pragma unroll
    for (int t = 0; t < WS; ++t) {
      const uint32_t w = cw[t];
      pcp += __popc(w);
      const i32x8 a = {(int)(w & 0x11111111u), (int)(w & 0x22222222u), (int)(w & 0x44444444u),
                       (int)((w >> 1) & 0x44444444u), 0, 0, 0, 0};
      const i32x8 b = {(int)fq[t][0], (int)fq[t][1], (int)fq[t][2], (int)fq[t][3], (int)fq[t][4], (int)fq[t][5], 0, 0};
      // formats: A FP4 (4), B FP6 E2M3 (2); E8M0 scales 2^0 and 2^2
      acc = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, acc, 4, 2, 0, 127, 0, 129);
    }
    // the two lane groups hold the two halves of the code's bits
    const auto sw = __builtin_amdgcn_permlane32_swap((uint32_t)pcp, (uint32_t)pcp, false, false);
    const int pc = (int)(sw[0] + sw[1]);
    if (grp == 0) {
      const float ct = fbase != nullptr ? -fi : code_term_l2(sf);
      L.fac[col] = make_float4(sf.x, sf.y, (float)pc, ct);
    }
    wave_lds_sync();
    if (rb + 32 < n) load(rb + 32);   // in flight during this block's products and outputs
    result_wait(acc);
    // bounds without the pair term (as est_y / est_dl on the integer product);
    // fails: bit 15 - i is the sign of thr - bound of output i (two cheap
    // instructions without a lane mask between them). A NaN bound may count as
    // passing: the rerank drops it.
    // The factors are read four outputs ahead: left alone, the compiler reads
    // each right before its use to save registers and waits 16 times.
    float low[16];
    uint32_t fails = 0;
    float4 fc[2][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) fc[0][i] = L.fac[4 * grp + i];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      if ((i & 3) == 0 && i < 12) {
#pragma unroll
        for (int e = 0; e < 4; ++e) fc[(i >> 2) + 1 & 1][e] = L.fac[8 * (i >> 2) + 8 + 4 * grp + e];
        asm volatile("" ::: "memory");
      }
      const float4 f = fc[(i >> 2) & 1][i & 3];
      const float y = fmaf(c.a1, acc[i], fmaf(c.a2, f.z, c.a0));
      const float d0 = fmaf(f.x, y, f.w);
      low[i] = fmaf(c.coefh, f.y, d0);
      if constexpr (DEBUG) {
        const int r = rb + 8 * (i >> 2) + 4 * grp + (i & 3);
        if (col == 0 && r < n) {
          const int64_t o = start + r - dbg_base;
          dbg_ip[o] = (int)acc[i];
          dbg_pc[o] = (int)f.z;
          dbg_est[o] = estimate_est(*rec, s.fac[start + r].y, (int)acc[i], (int)f.z);
          dbg_dist[o] = d0 + c.pt;
          dbg_lb[o] = low[i] + c.pt;
        }
      } else {
        fails = __builtin_amdgcn_alignbit(fails, __float_as_uint(c.thr - low[i]), 31);
      }
    }
    if constexpr (!DEBUG) {
      const uint32_t mask = ~fails & 0xFFFFu;
      if (__ballot(mask != 0u) != 0ull) {
        // the column's 32 codes in order, first code at bit 31: this lane's
        // groups of four between its partner's
        uint32_t sp = (mask | (mask << 8)) & 0x00FF00FFu;
        sp = (sp | (sp << 4)) & 0x0F0F0F0Fu;
        const auto pr = __builtin_amdgcn_permlane32_swap(sp, sp, false, false);
        const int left = n - rb;   // codes of the block that exist
        const uint32_t all = (((uint32_t)pr[0] << 4) | (uint32_t)pr[1]) & (left < 32 ? ~(0xFFFFFFFFu >> left) : ~0u);
        // each lane's passing outputs one after the other (a few per lane)
#pragma unroll
        for (int j = 0; j < 4; ++j) L.low[j][lane] = make_float4(low[4 * j], low[4 * j + 1], low[4 * j + 2], low[4 * j + 3]);
        wave_lds_sync();
        uint32_t m = mask << 16;
        while (__ballot(m != 0u) != 0ull) {
          if (m != 0u) {
            const int i = __clz((int)m);
            m &= ~(0x80000000u >> i);
            const int code = 8 * (i >> 2) + 4 * grp + (i & 3);
            Cand cd;
            cd.pos = (int32_t)start + rb + code;
            cd.lb = reinterpret_cast<const float*>(&L.low[i >> 2][lane])[i & 3] + c.pt;
            if (code < left) c.seg[count + __popc(all & ~(0xFFFFFFFFu >> code))] = cd;
          }
        }
        count += __popc(all);
      }
    }
    wave_lds_sync();   // the next block's factors overwrite these
  }
  return count;
}

// The list holding unit u: the largest l < n with off[l] <= u, by a 64-way
// search (three rounds of loads for 16,384 lists).
__device__ __forceinline__ int wave_find_list(const int64_t* __restrict__ off, int n, int64_t u) {
  int lo = 0, hi = n;   // off[lo] <= u, and the list is in [lo, hi)
  const int lane = lane_id();
  while (hi - lo > 1) {
    const int step = (hi - lo + kWave - 1) / kWave;
    const int idx = lo + lane * step;
    const bool ok = idx < hi && off[min(idx, n - 1)] <= u;
    const uint64_t m = __ballot(ok);
    const int j = 63 - __clzll((long long)m);   // lane 0 always holds (off[lo] <= u)
    lo = uniform_i32(lo + j * step);
    hi = min(hi, lo + step);
  }
  return lo;
}

template <int WS>
__device__ __forceinline__ void load_fragments(const int8_t* row, int grp, u32x6 (&fq)[WS]) {
#pragma unroll
  for (int t = 0; t < WS; ++t) {
    const i32x4* p = reinterpret_cast<const i32x4*>(row + 64 * t + 32 * grp);
    fq[t] = fp6_fragment(p[0], p[1]);
  }
}

// Work units are (list, chunk of the list's codes, group of 32 pairs), ordered
// by list, then chunk, then group, cut into kScanSlices contiguous slices; a
// workgroup starts on the slice of its XCD (workgroups go to the XCDs in
// turn), so the groups of one chunk run on one XCD and share its L2, then
// moves on to the other slices. Each wave claims its units by itself.
template <int WS>
__global__ __launch_bounds__(kThreads, WS <= 6 ? 4 : WS <= 12 ? 3 : 2) void k_scan_frag(SearchDev s) {
  __shared__ WaveLds lds[kWaves];
  WaveLds& L = lds[threadIdx.x / kWave];
  const int lane = lane_id(), col = lane & 31, grp = lane >> 5;
  const int64_t total = uniform_i64(s.mf_unit_off[s.nlist]);
  const int x0 = (int)(blockIdx.x % kScanSlices);
  for (int j = 0; j < kScanSlices; ++j) {
    const int x = (x0 + j) % kScanSlices;
    const int64_t lo = total * x / kScanSlices;
    const int64_t size = total * (x + 1) / kScanSlices - lo;
    // The slice's first units belong to the waves that start on it, one each; the
    // rest are claimed from its counter. A counter is only added to where it can
    // have units left (4096 waves that each tried all eight took 100 us on their
    // addresses).
    const int64_t own = (int64_t)kWaves * ((gridDim.x + kScanSlices - 1 - x) / kScanSlices);
    unsigned long long* ctr = s.counters + kScanSliceCtr + kScanSliceStride * x;
    int64_t next = -1;
    if (j == 0) {
      next = (int64_t)kWaves * (blockIdx.x / kScanSlices) + threadIdx.x / kWave;
    } else {
      const unsigned long long seen = __hip_atomic_load(ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (own + uniform_i64((int64_t)seen) >= size) continue;
    }
    for (;;) {
      if (next < 0) {
        if (own >= size) break;
        unsigned long long cl = 0;
        if (lane == 0) cl = atomicAdd(ctr, 1ull);
        next = own + uniform_i64((int64_t)cl);   // lane 0's claim (every lane is active)
      }
      if (next >= size) break;
      const int64_t u = lo + uniform_i64(next);
      next = -1;
      const int list = wave_find_list(s.mf_unit_off, s.nlist, u);
      const int local = (int)uniform_i64(u - s.mf_unit_off[list]);
      const int64_t p0 = uniform_i64(s.mf_pair_off[list]);
      const int cnt = (int)(uniform_i64(s.mf_pair_off[list + 1]) - p0);
      const int ngroups = (cnt + 31) / 32;
      const int ch = local / ngroups;
      const int gi = local - ch * ngroups;
      const int64_t lbeg = uniform_i32(s.list_off[list]), lend = uniform_i32(s.list_off[list + 1]);
      const int64_t start = lbeg + (int64_t)ch * s.chunk;
      const int n = (int)(min(lend, start + s.chunk) - start);
      const MfRow row = s.mf_rows[p0 + min(32 * gi + col, cnt - 1)];
      const bool live = 32 * gi + col < cnt && ch >= row.first;
      if (__ballot(live) == 0ull) continue;   // every pair scanned this chunk in the bootstrap
      u32x6 fq[WS];
      load_fragments<WS>(s.qu8 + (int64_t)row.g * (64 * WS), grp, fq);
      Column c;
      c.a1 = row.a1;
      c.a2 = row.a2;
      c.a0 = row.a0;
      c.coefh = row.coefh;
      c.pt = row.pt;
      c.thr = live && row.thr == row.thr ? row.thr : -__builtin_inff();
      c.seg = s.seg + row.seg + (int64_t)ch * s.chunk;
      const int count = frag_unit<false, WS>(s, start, n, c, fq, L, nullptr, nullptr, nullptr, nullptr, nullptr,
                                             nullptr, 0);
      if (live && grp == 0) s.seg_count[row.count + ch] = count;
    }
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
  c.seg = nullptr;
  (void)frag_unit<true, WS>(s, start, (int)(end - start), c, fq, L, recp, ip, pc, est, dist, lb, lbeg);
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
