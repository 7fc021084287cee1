// Batched scan in block form, for B_q > 4 and for codes above 16 words
// (kernels_frag.hip takes the rest), and the grouping of pairs by list for both:
// the integer <x_b, q_u> of Sec. 3.3.2 for all (query, code) pairs of one IVF list
// at once, as an int8 matrix product on the MFMA units:
//   IP[pairs x codes] = Qu[pairs x D] (B_q bits, less 128 for 8) * Xb[D x codes] (0/1).
// The paper evaluates the same batched contraction with 4-bit look-up tables
// in SIMD registers; on CDNA4 the contraction maps onto v_mfma_i32_16x16x64_i8.
//
// Grouping. The (query, list) pairs of the main phase are bucketed by list.
// A work unit is (list, chunk of the list's codes, group of 16 pairs): the 16
// quantised queries are staged in LDS once and every 64-code block of the
// chunk is multiplied against them; each wave owns 16 codes of the block,
// expands their bits to bytes in registers and issues one MFMA per 64
// dimensions. Candidates (lb <= tau) are compacted per pair in code order, so
// the segments are identical to those of the popcount scan.
#include <algorithm>
#include <type_traits>

#include "rbq_internal.hpp"
#include "rbq_runtime.hpp"
#include "scan_code.hpp"

namespace rbq {
namespace {

constexpr int kThreads = 256;
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

struct RowInfo {
  PairTerms t;        // the pair's estimator constants (pair_terms / pair_terms_ip)
  float thr;          // tau - pt, what the bound without the pair term is tested against
  int32_t valid;      // 1 when this row's chunk belongs to the scanned phase
  int64_t seg_base;   // first segment slot of (pair, chunk)
  int64_t count_slot; // seg_count index of (pair, chunk)
};

// 4 bits -> 4 bytes of 0/1: the nibble's bits land on bits 0, 8, 16, 24.
__device__ __forceinline__ int nib_to_bytes(uint32_t nib) { return (int)((nib * 0x00204081u) & 0x01010101u); }
__device__ __forceinline__ uint32_t nib_to_bytes_u(uint32_t nib) { return (nib * 0x00204081u) & 0x01010101u; }

// FP8 (E4M3, OCP: bias 7) encodings of the integers 0..15, all exact: the
// query operand of the FP8 x FP4 contraction (B_q <= 4).
__constant__ uint8_t kFp8Int[16] = {0x00, 0x38, 0x40, 0x44, 0x48, 0x4A, 0x4C, 0x4E,
                                    0x50, 0x51, 0x52, 0x53, 0x54, 0x55, 0x56, 0x57};

// 8 code bits -> 8 FP4 (E2M1) values 0 or 1.0 (0b0010) in one dword. The
// nibbles come out in the order of dimensions 0, 4, 1, 5, 2, 6, 3, 7 of the
// byte.
__device__ __forceinline__ int bits_to_fp4x8(uint32_t x) {
  const uint32_t lo = (uint32_t)nib_to_bytes_u(x & 15u), hi = (uint32_t)nib_to_bytes_u((x >> 4) & 15u);
  return (int)((lo | (hi << 4)) << 1);
}

// Operand layouts of v_mfma_scale_f32_16x16x128_f8f6f4 (FP8 A, FP4 B), as
// measured on gfx950: lane group g of the B operand holds the 32 values
// k = 32 g .. 32 g + 31 (nibble e is k = 32 g + e), while lane group g of the
// A operand holds k = 16 g .. 16 g + 15 in bytes 0..15 and k = 64 + 16 g ..
// 64 + 16 g + 15 in bytes 16..31. The B side carries the code bits of
// dimensions 128 t + 32 g .. +31 in the nibble order of bits_to_fp4x8, so the
// query byte at A position x (0..127 within a 128-dimension block) must be the
// dimension that B's k(x) holds: k(x) = 16 (x / 32) + x % 32 for x % 32 < 16,
// else 64 + 16 (x / 32) + x % 32 - 16. A group of 8 consecutive positions
// maps to the 8 dimensions starting at k(x) rounded down to 8, in the nibble order.
// Wait states between the last scaled FP8 x FP4 MFMA of a code block and the
// first read of its result. The compiler's own distance for this mixed-format
// instruction (about 12) returned wrong sums on gfx950 once nothing else sat
// between the product and the read. The accumulator passes through the wait
// (in the accumulation registers the product wrote), so the product comes
// before it and every read of the result after it.
__device__ __forceinline__ void f4_result_wait(f32x4& acc) {
  asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7\n\ts_nop 7" : "+a"(acc));
}

__device__ __forceinline__ int f4_src_dim(int d) {
  const int x = d & 127, g = x >> 5, e = x & 31;
  return (d & ~127) + (e < 16 ? 16 * g + e : 64 + 16 * g + (e - 16));
}

// One (list, chunk, RG x 16-row group) unit. rows[], rg_live[] and A must be
// in LDS already. Each wave takes 16 codes of every 64-code block, expands
// their bits once per code word and multiplies them against the RG row groups
// (one MFMA each; row groups without a live row are skipped), then writes the
// candidates of valid rows into their segments and their counts.
// F4: the query rows in LDS are FP8 codes placed by f4_src_dim and in the
// nibble order of bits_to_fp4x8, each row padded to a multiple of 128
// dimensions, and every v_mfma_scale_f32_16x16x128_f8f6f4 takes 128 dimensions
// (two code words) of 16 codes against 16 query rows; FP32 accumulation of
// integer products below 16 over at most 4096 dimensions is exact, so the
// inner products are those of the int8 contraction bit for bit.
template <bool DEBUG, bool F4, int WS, int RG>
__device__ void mfma_unit(const SearchDev& s, int64_t start, int64_t end, const RowInfo* rows,
                          const int32_t* rg_live, const int8_t* A, uint16_t (*masks)[4], int32_t* rowcnt,
                          int32_t* dbg_ip, int32_t* dbg_pc, float* dbg_est, float* dbg_dist,
                          float* dbg_lb, int64_t dbg_base, const PairRec* rec) {
  const int wave = threadIdx.x >> 6, lane = lane_id();
  const int col = lane & 15, grp = lane >> 4;
  const int dp = s.dp, W = s.W;
  const int dpa = F4 ? (dp + 127) / 128 * 128 : dp;
  bool hl[RG];
#pragma unroll
  for (int h = 0; h < RG; ++h) hl[h] = uniform_i32(rg_live[h]) != 0;
  for (int64_t blk = start; blk < end; blk += 64) {
    const bool pvalid = blk + wave * 16 + col < end;
    // lanes past the end read the block's first code (in bounds) and are masked
    const int64_t p = pvalid ? blk + wave * 16 + col : blk;
    const uint32_t keep = pvalid ? 0xFFFFu : 0u;
    i32x4 acc[RG];
#pragma unroll
    for (int h = 0; h < RG; ++h) acc[h] = i32x4{0, 0, 0, 0};
    int pcp = 0;
    if constexpr (F4) {
      // lane group grp: dimensions 128 t2 + 32 grp .. +31, half (grp & 1) of
      // word 2 t2 + (grp >> 1); four words' reads are issued before their products
      const uint32_t keep32 = pvalid ? 0xFFFFFFFFu : 0u;
      const uint32_t* c32 = reinterpret_cast<const uint32_t*>(s.codes);
      f32x4 accf[RG];
#pragma unroll
      for (int h = 0; h < RG; ++h) accf[h] = f32x4{0.f, 0.f, 0.f, 0.f};
      auto step = [&](uint32_t bits, int t2) {
        pcp += __popc(bits);
        i32x8 b = {bits_to_fp4x8(bits & 0xFFu), bits_to_fp4x8((bits >> 8) & 0xFFu),
                   bits_to_fp4x8((bits >> 16) & 0xFFu), bits_to_fp4x8(bits >> 24), 0, 0, 0, 0};
#pragma unroll
        for (int h = 0; h < RG; ++h) {
          if (!hl[h]) continue;
          const i32x8 a = *reinterpret_cast<const i32x8*>(A + (size_t)(16 * h + col) * dpa + t2 * 128 + grp * 32);
          // formats: A FP8 E4M3 (0), B FP4 E2M1 (4); E8M0 scales 127 = 2^0
          accf[h] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a, b, accf[h], 0, 4, 0, 127, 0, 127);
        }
      };
      auto load = [&](int t2) -> uint32_t {
        const int w = 2 * t2 + (grp >> 1);
        const uint32_t v = c32[2 * code_word_index(p, min(w, W - 1), W) + (grp & 1)];
        return w < W ? v & keep32 : 0u;
      };
      const int T2 = (W + 1) / 2;
      for (int t0 = 0; t0 < T2; t0 += 4) {
        uint32_t bw[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) bw[j] = load(min(t0 + j, T2 - 1));
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (t0 + j < T2) step(bw[j], t0 + j);
      }
#pragma unroll
      for (int h = 0; h < RG; ++h) {
        f4_result_wait(accf[h]);
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[h][i] = (int)accf[h][i];
      }
    } else {
      // the lane's 16-bit slice (dimensions 64 t + 16 grp .. +15) of each code
      // word; every word read is issued before the first product
      const uint16_t* c16 = reinterpret_cast<const uint16_t*>(s.codes);
      auto step = [&](uint32_t bits, int t) {
        bits &= keep;
        pcp += __popc(bits);
        i32x4 b;
        b[0] = nib_to_bytes(bits & 15u);
        b[1] = nib_to_bytes((bits >> 4) & 15u);
        b[2] = nib_to_bytes((bits >> 8) & 15u);
        b[3] = nib_to_bytes((bits >> 12) & 15u);
#pragma unroll
        for (int h = 0; h < RG; ++h) {
          if (!hl[h]) continue;
          // A fragment: row 16 h + col, dimensions 64 t + 16 grp .. +15
          const i32x4 a = *reinterpret_cast<const i32x4*>(A + (size_t)(16 * h + col) * dp + t * 64 + grp * 16);
          acc[h] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, b, acc[h], 0, 0, 0);
        }
      };
      if constexpr (WS > 0) {
        uint32_t bw[WS];
#pragma unroll
        for (int t = 0; t < WS; ++t) bw[t] = c16[4 * code_word_index(p, t, WS) + grp];
#pragma unroll
        for (int t = 0; t < WS; ++t) step(bw[t], t);
      } else {
        for (int t0 = 0; t0 < W; t0 += 4) {
          uint32_t bw[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) bw[j] = c16[4 * code_word_index(p, min(t0 + j, W - 1), W) + grp];
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (t0 + j < W) step(bw[j], t0 + j);
        }
      }
    }
    // popcount of the code: the four lane groups hold its four 16-bit slices
    int pc = pcp + __shfl_xor(pcp, 16, kWave);
    pc += __shfl_xor(pc, 32, kWave);
    const float2 sf = s.sfac[p];
    const float ct = s.metric != 0 ? -s.fip[p] : code_term_l2(sf);
    // acc[h][i] + qoff * pc = IP of row 16 h + 4 grp + i with code `col` (the
    // int8 operand holds q_u - qoff, so that B_q = 8 values fit)
    bool pass[RG][4];
    float lbv[RG][4];
#pragma unroll
    for (int h = 0; h < RG; ++h) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        pass[h][i] = false;
        lbv[h][i] = __builtin_inff();
        if (!hl[h]) continue;
        const int row = 16 * h + 4 * grp + i;
        const RowInfo& ri = rows[row];
        float d0, l0;
        const int ipv = acc[h][i] + s.qoff * pc;
        est_dl(ri.t, sf, ct, est_y(ri.t, ipv, pc), d0, l0);
        const bool live = pvalid && ri.valid;
        const float lb = live ? l0 + ri.t.pt : __builtin_inff();
        if (DEBUG && row == 0 && live) {
          const int64_t o = p - dbg_base;
          dbg_ip[o] = ipv;
          dbg_pc[o] = pc;
          dbg_est[o] = estimate_est(*rec, s.fac[p].y, ipv, pc);
          dbg_dist[o] = d0 + ri.t.pt;
          dbg_lb[o] = lb;
        }
        pass[h][i] = live && l0 <= ri.thr;   // the bound test without the pair term
        lbv[h][i] = lb;
      }
    }
    if (DEBUG) continue;
    // per-row 16-bit masks of this wave's codes
#pragma unroll
    for (int h = 0; h < RG; ++h) {
      if (!hl[h]) continue;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint64_t m = __ballot(pass[h][i]);
        if (lane < 4) masks[16 * h + 4 * lane + i][wave] = (uint16_t)((m >> (16 * lane)) & 0xFFFFu);
      }
    }
    __syncthreads();
#pragma unroll
    for (int h = 0; h < RG; ++h) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (!pass[h][i]) continue;
        const int row = 16 * h + 4 * grp + i;
        uint64_t m64 = 0;
#pragma unroll
        for (int w = 0; w < 4; ++w) m64 |= (uint64_t)masks[row][w] << (16 * w);
        const int bit = wave * 16 + col;
        const int before = __popcll(m64 & ((1ull << bit) - 1ull));
        Cand cd;
        cd.pos = (int32_t)p;
        cd.lb = lbv[h][i];
        s.seg[rows[row].seg_base + rowcnt[row] + before] = cd;
      }
    }
    __syncthreads();
    if (threadIdx.x < 16 * RG && rg_live[threadIdx.x >> 4]) {
      const int row = threadIdx.x;
      uint64_t m64 = 0;
      for (int w = 0; w < 4; ++w) m64 |= (uint64_t)masks[row][w] << (16 * w);
      rowcnt[row] += __popcll(m64);
    }
    __syncthreads();
  }
}

__device__ __forceinline__ int64_t ub64(const int64_t* a, int64_t n, int64_t v) {
  int64_t lo = 0, hi = n;
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if (a[mid] <= v) lo = mid + 1; else hi = mid;
  }
  return lo;
}

// ---------------------------------------------------------------- grouping
// The main-phase pairs bucketed by list: a pair's slot is its list's first slot
// plus its rank in the list (any order), and slot records (MfRow) hold all that
// a scan unit needs of the pair, so that a unit reads one contiguous run.
// k_group_count counts pairs per list and ranks them: blocks of 16,384 pairs
// rank theirs with LDS counters (nlist <= 24,576 of them fit), then each block
// takes its share of every list with one device atomic per list it met. One
// atomic per pair on the lists' counters instead, and another per pair to
// scatter, took 220 us for 1.28 M pairs on 4096 lists; counting and ranking
// take 13 us, the offsets 8 us, the records 48 us. Up to 16,384 pairs are one
// block, which also computes the offsets.
constexpr int kGrpThreads = 1024, kGrpPer = 16;

// Exclusive scans of the lists' pair counts and unit counts by one block of
// kGrpThreads threads (tiles of kOffPer consecutive lists per thread; wave
// scans, then the 16 wave totals), and the work counters reset. count(l): the
// pairs of list l.
constexpr int kOffPer = 4;

template <class Count>
__device__ __forceinline__ void group_offsets(const SearchDev& s, Count count) {
  __shared__ int32_t wp[kGrpThreads / kWave], wu[kGrpThreads / kWave];
  const int t = threadIdx.x, lane = lane_id(), wave = t >> 6;
  if (t == 0) s.counters[2] = 0;
  if (t < kScanSlices) s.counters[kScanSliceCtr + kScanSliceStride * t] = 0;
  const int rows = 16 * s.mf_rg;
  int64_t carry_p = 0, carry_u = 0;
  for (int base = 0; base < s.nlist; base += kGrpThreads * kOffPer) {
    const int l0 = base + t * kOffPer;
    int c[kOffPer], u[kOffPer], lo[kOffPer + 1];
#pragma unroll
    for (int i = 0; i <= kOffPer; ++i) lo[i] = s.list_off[min(l0 + i, s.nlist)];
#pragma unroll
    for (int i = 0; i < kOffPer; ++i) c[i] = count(min(l0 + i, s.nlist - 1));
    // a tile's sums fit 32 bits: at most 2^31 pairs in all, and units of at
    // least one pair and one code each
    int sp = 0, su = 0;
#pragma unroll
    for (int i = 0; i < kOffPer; ++i) {
      c[i] = l0 + i < s.nlist ? c[i] : 0;
      u[i] = c[i] > 0 ? ((lo[i + 1] - lo[i] + s.chunk - 1) / s.chunk) * ((c[i] + rows - 1) / rows) : 0;
      sp += c[i];
      su += u[i];
    }
    int ip = sp, iu = su;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const int yp = __shfl_up(ip, o, kWave), yu = __shfl_up(iu, o, kWave);
      ip += lane >= o ? yp : 0;
      iu += lane >= o ? yu : 0;
    }
    if (lane == kWave - 1) {
      wp[wave] = ip;
      wu[wave] = iu;
    }
    __syncthreads();
    int64_t bp = carry_p + ip - sp, bu = carry_u + iu - su;
    for (int w = 0; w < kGrpThreads / kWave; ++w) {
      bp += w < wave ? wp[w] : 0;
      bu += w < wave ? wu[w] : 0;
      carry_p += wp[w];
      carry_u += wu[w];
    }
#pragma unroll
    for (int i = 0; i < kOffPer; ++i) {
      if (l0 + i < s.nlist) {
        s.mf_pair_off[l0 + i] = bp;
        s.mf_unit_off[l0 + i] = bu;
      }
      bp += c[i];
      bu += u[i];
    }
    __syncthreads();   // the next tile's totals overwrite these
  }
  if (t == 0) {
    s.mf_pair_off[s.nlist] = carry_p;
    s.mf_unit_off[s.nlist] = carry_u;
  }
}

__global__ __launch_bounds__(kGrpThreads) void k_group_offsets(SearchDev s) {
  group_offsets(s, [&](int l) { return s.mf_cnt[l]; });
}

__global__ __launch_bounds__(kGrpThreads) void k_group_count(SearchDev s) {
  extern __shared__ int32_t hist[];
  const int64_t np = s.nq * s.nprobe;
  const int64_t g0 = (int64_t)blockIdx.x * (kGrpThreads * kGrpPer) + threadIdx.x;
  for (int l = threadIdx.x; l < s.nlist; l += kGrpThreads) hist[l] = 0;
  int list[kGrpPer], rank[kGrpPer];
  // four pairs per thread at a time: clamped reads, all in flight together,
  // then the tests
  const int64_t left = np - (int64_t)blockIdx.x * (kGrpThreads * kGrpPer);   // pairs from this block on
#pragma unroll
  for (int i0 = 0; i0 < kGrpPer; i0 += 4) {
#pragma unroll
    for (int i = i0; i < i0 + 4; ++i) list[i] = -1;
    if ((int64_t)i0 * kGrpThreads >= left) continue;   // uniform
    int c0[4], c1[4], p0[4], l[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int64_t gc = min(g0 + (int64_t)(i0 + e) * kGrpThreads, np - 1);
      const int64_t q = gc / s.nprobe;
      const int64_t o = gc + q;   // choff row stride is nprobe + 1
      c0[e] = s.pair_choff[o];
      c1[e] = s.pair_choff[o + 1];
      p0[e] = s.q_p0[q];
      l[e] = s.probe[gc];
    }
    // a main-phase chunk remains: chunks before q_p0 were scanned by phase 0
    // (a rank past the query's nprobe has no chunk)
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (g0 + (int64_t)(i0 + e) * kGrpThreads < np && c1[e] > c0[e] && c1[e] > p0[e]) list[i0 + e] = l[e];
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kGrpPer; ++i) rank[i] = list[i] >= 0 ? atomicAdd(&hist[list[i]], 1) : -1;
  __syncthreads();
  if (gridDim.x == 1) {   // the block has seen every pair: ranks are final, and the counts are here
    group_offsets(s, [&](int l) { return hist[l]; });
#pragma unroll
    for (int i = 0; i < kGrpPer; ++i) {
      const int64_t g = g0 + (int64_t)i * kGrpThreads;
      if (g < np) s.mf_pairs[g] = rank[i];
    }
    return;
  }
  for (int l = threadIdx.x; l < s.nlist; l += kGrpThreads) {
    const int c = hist[l];
    if (c > 0) hist[l] = atomicAdd(&s.mf_cnt[l], c);
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kGrpPer; ++i) {
    const int64_t g = g0 + (int64_t)i * kGrpThreads;
    if (g < np) s.mf_pairs[g] = list[i] >= 0 ? hist[list[i]] + rank[i] : -1;
  }
}

// The fragment scan's units, a thread per unit: its list by binary search over
// the lists' unit offsets.
__device__ __forceinline__ void group_units(const SearchDev& s, int block, int nblocks) {
  const int64_t total = s.mf_unit_off[s.nlist];
  for (int64_t u = (int64_t)block * blockDim.x + threadIdx.x; u < total; u += (int64_t)nblocks * blockDim.x) {
    const int list = (int)(ub64(s.mf_unit_off, s.nlist + 1, u) - 1);
    const int local = (int)(u - s.mf_unit_off[list]);
    const int64_t p0 = s.mf_pair_off[list];
    const int cnt = (int)(s.mf_pair_off[list + 1] - p0);
    const int groups = (cnt + 31) / 32;
    const int c = local / groups, gi = local - c * groups;
    const int beg = s.list_off[list], len = s.list_off[list + 1] - beg;
    MfUnit un;
    un.start = beg + c * s.chunk;
    un.n = min(s.chunk, len - c * s.chunk);
    un.slot = (int32_t)p0 + 32 * gi;
    un.chunk_rows = (c << 5) | (min(cnt - 32 * gi, 32) - 1);
    s.mf_units[u] = un;
  }
}

// Every main-phase pair's record to its slot (after tau is known); the first
// unit_blocks blocks write the units.
__global__ __launch_bounds__(256) void k_group_scatter(SearchDev s, int unit_blocks) {
  if ((int)blockIdx.x < unit_blocks) {
    group_units(s, blockIdx.x, unit_blocks);
    return;
  }
  const int64_t g = (int64_t)(blockIdx.x - unit_blocks) * blockDim.x + threadIdx.x;
  if (g >= s.nq * s.nprobe) return;
  const int rank = s.mf_pairs[g];
  if (rank < 0) return;
  const int64_t q = g / s.nprobe;
  const PairRec rec = s.pairs[g];
  const float hwk = s.eps0 / sqrtf((float)(s.dp - 1));
  const int c0 = s.pair_choff[g + q];
  MfRow row;
  const PairTerms t = s.metric != 0 ? pair_terms_ip(rec, hwk, s.pair_pt[g]) : pair_terms(rec, hwk);
  row.a1 = t.a1;
  row.a2 = t.a2;
  row.a0 = t.a0;
  row.coefh = t.coefh;
  row.pt = t.pt;
  row.thr = s.tau[q] - t.pt;
  row.first = max(0, s.q_p0[q] - c0);
  row.g = (int32_t)g;
  row.seg = s.off_seg[q] + s.pair_codeoff[g + q];
  row.count = s.off_ch[q] + c0;
  s.mf_rows[s.mf_pair_off[rec.list] + rank] = row;
}

// ---------------------------------------------------------------- persistent MFMA scan
// FP8 row of the F4 path from 8 int8 query values (0..15) at a time: byte m
// of each group of 8 holds dimension pi(m) of the group, pi = 0, 4, 1, 5, 2, 6, 3, 7.
__device__ __forceinline__ uint64_t fp8_group(uint64_t v) {
  uint64_t out = 0;
#pragma unroll
  for (int m = 0; m < 8; ++m) {
    const int src = (m & 1) ? 4 + (m >> 1) : (m >> 1);
    out |= (uint64_t)kFp8Int[(v >> (8 * src)) & 15u] << (8 * m);
  }
  return out;
}

template <bool F4, int WS, int RG>
__global__ __launch_bounds__(kThreads) void k_scan_mfma(SearchDev s) {
  constexpr int R = 16 * RG;
  extern __shared__ __attribute__((aligned(16))) int8_t A[];   // R x dpa
  __shared__ RowInfo rows[R];
  __shared__ uint16_t masks[R][4];
  __shared__ int32_t rowcnt[R];
  __shared__ int32_t rg_live[RG];
  __shared__ int64_t sh_u;
  const int64_t total = uniform_i64(s.mf_unit_off[s.nlist]);
  const int dpa = F4 ? (s.dp + 127) / 128 * 128 : s.dp;
  for (;;) {
    if (threadIdx.x == 0) {
      sh_u = (int64_t)atomicAdd(&s.counters[2], 1ull);
#pragma unroll
      for (int h = 0; h < RG; ++h) rg_live[h] = 0;
    }
    __syncthreads();
    const int64_t u = uniform_i64(sh_u);
    __syncthreads();
    if (u >= total) break;
    const int list = uniform_i32((int)(ub64(s.mf_unit_off, s.nlist + 1, u) - 1));
    const int64_t local = uniform_i64(u - s.mf_unit_off[list]);
    const int cnt = uniform_i32((int)(s.mf_pair_off[list + 1] - s.mf_pair_off[list]));
    const int ngroups = (cnt + R - 1) / R;
    const int c = (int)(local / ngroups);
    const int gi = (int)(local - (int64_t)c * ngroups);
    const int64_t lbeg = uniform_i64(s.list_off[list]), lend = uniform_i64(s.list_off[list + 1]);
    const int64_t start = lbeg + (int64_t)c * s.chunk;
    const int64_t end = lend < start + s.chunk ? lend : start + s.chunk;
    if (threadIdx.x < R) {
      const int i = threadIdx.x;
      RowInfo ri;
      ri.valid = 0;
      ri.thr = -__builtin_inff();
      ri.seg_base = 0;
      ri.count_slot = -1;
      ri.t.a1 = ri.t.a2 = ri.t.a0 = ri.t.pt = ri.t.coefh = 0.f;
      if (R * gi + i < cnt) {
        const MfRow r = s.mf_rows[s.mf_pair_off[list] + R * gi + i];
        ri.t.a1 = r.a1;
        ri.t.a2 = r.a2;
        ri.t.a0 = r.a0;
        ri.t.pt = r.pt;
        ri.t.coefh = r.coefh;
        if (c >= r.first) {
          ri.valid = 1;
          ri.thr = r.thr;
          ri.seg_base = r.seg + (int64_t)c * s.chunk;
          ri.count_slot = r.count + c;
          rg_live[i >> 4] = 1;
        }
      }
      rows[i] = ri;
      rowcnt[i] = 0;
    }
    // stage the R quantised queries (zero rows for missing pairs)
    if constexpr (F4) {   // FP8, rows padded to a multiple of 128 dimensions
      for (int idx = threadIdx.x * 8; idx < R * dpa; idx += kThreads * 8) {
        const int i = idx / dpa, d = idx - i * dpa;
        uint64_t v = 0;
        const int src = f4_src_dim(d);
        if (R * gi + i < cnt && src < s.dp) {
          const int64_t g = s.mf_rows[s.mf_pair_off[list] + R * gi + i].g;
          v = fp8_group(*reinterpret_cast<const uint64_t*>(s.qu8 + g * s.dp + src));
        }
        *reinterpret_cast<uint64_t*>(A + idx) = v;
      }
    } else {
      for (int idx = threadIdx.x * 16; idx < R * s.dp; idx += kThreads * 16) {
        const int i = idx / s.dp, d = idx - i * s.dp;
        i32x4 v = {0, 0, 0, 0};
        if (R * gi + i < cnt) {
          const int64_t g = s.mf_rows[s.mf_pair_off[list] + R * gi + i].g;
          v = *reinterpret_cast<const i32x4*>(s.qu8 + g * s.dp + d);
        }
        *reinterpret_cast<i32x4*>(A + idx) = v;
      }
    }
    __syncthreads();
    mfma_unit<false, F4, WS, RG>(s, start, end, rows, rg_live, A, masks, rowcnt, nullptr, nullptr, nullptr,
                                 nullptr, nullptr, 0, nullptr);
    if (threadIdx.x < R && rows[threadIdx.x].valid) s.seg_count[rows[threadIdx.x].count_slot] = rowcnt[threadIdx.x];
    __syncthreads();
  }
}

// Debug: one caller-given quantised query (row 0) against a whole list, with
// the kernel instantiation the search uses for this code width.
template <bool F4, int WS, int RG>
__global__ __launch_bounds__(kThreads) void k_debug_mfma(SearchDev s, const PairRec* recp,
                                                         const int8_t* qu8, int32_t list, int32_t* ip,
                                                         int32_t* pc, float* est, float* dist,
                                                         float* lb) {
  constexpr int R = 16 * RG;
  extern __shared__ __attribute__((aligned(16))) int8_t A[];
  __shared__ RowInfo rows[R];
  __shared__ uint16_t masks[R][4];
  __shared__ int32_t rowcnt[R];
  __shared__ int32_t rg_live[RG];
  const float hwk = s.eps0 / sqrtf((float)(s.dp - 1));
  const int dpa = F4 ? (s.dp + 127) / 128 * 128 : s.dp;
  if (threadIdx.x < R) {
    RowInfo ri;
    ri.valid = threadIdx.x == 0;
    ri.thr = __builtin_inff();
    ri.seg_base = 0;
    ri.count_slot = -1;
    ri.t = s.metric != 0 ? pair_terms_ip(*recp, hwk, s.pair_pt[0]) : pair_terms(*recp, hwk);
    rows[threadIdx.x] = ri;
    rowcnt[threadIdx.x] = 0;
  }
  if (threadIdx.x < RG) rg_live[threadIdx.x] = threadIdx.x == 0;
  if constexpr (F4) {
    for (int idx = threadIdx.x * 8; idx < R * dpa; idx += kThreads * 8)
      *reinterpret_cast<uint64_t*>(A + idx) =
          idx < dpa && f4_src_dim(idx) < s.dp ? fp8_group(*reinterpret_cast<const uint64_t*>(qu8 + f4_src_dim(idx))) : 0ull;
  } else {
    for (int idx = threadIdx.x; idx < R * s.dp; idx += kThreads) A[idx] = idx < s.dp ? qu8[idx] : (int8_t)0;
  }
  __syncthreads();
  const int64_t lbeg = uniform_i64(s.list_off[list]), lend = uniform_i64(s.list_off[list + 1]);
  const int64_t start = lbeg + (int64_t)blockIdx.x * s.chunk;
  const int64_t end = lend < start + s.chunk ? lend : start + s.chunk;
  if (start >= end) return;
  mfma_unit<true, F4, WS, RG>(s, start, end, rows, rg_live, A, masks, rowcnt, ip, pc, est, dist, lb, lbeg, recp);
}

// Clears counters (a kernel rather than a memset, so that the sequence can be
// captured in a graph).
__global__ void k_zero_u32(uint32_t* __restrict__ p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0u;
}

__global__ void k_fill_i32(int32_t* __restrict__ p, int64_t n, int32_t v) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// Block-form kernels per (code width, row groups): W words of 64 bits,
// compile-time for the common widths of the int8 contraction (every word read
// is then issued before the first product) and a runtime width otherwise; RG
// groups of 16 query rows per unit. The FP8 x FP4 contraction reaches the
// block form only above the fragment scan's 16 words.
template <bool F4, bool DBG>
const void* kernel_for(int W, int rg) {
#define RBQ_MF(WS_, RG_) (DBG ? (const void*)k_debug_mfma<F4, WS_, RG_> : (const void*)k_scan_mfma<F4, WS_, RG_>)
  if constexpr (!F4) {
    if (rg == 4 && W == 12) return RBQ_MF(12, 4);
    if (rg == 2) {
      switch (W) {
        case 12: return RBQ_MF(12, 2);
        case 15: return RBQ_MF(15, 2);
        case 16: return RBQ_MF(16, 2);
        default: break;
      }
    }
    if (rg == 1) {
      switch (W) {
        case 1: return RBQ_MF(1, 1);
        case 2: return RBQ_MF(2, 1);
        case 3: return RBQ_MF(3, 1);
        case 4: return RBQ_MF(4, 1);
        case 8: return RBQ_MF(8, 1);
        case 12: return RBQ_MF(12, 1);
        case 15: return RBQ_MF(15, 1);
        case 16: return RBQ_MF(16, 1);
        default: break;
      }
    }
  }
  if (rg == 4) return RBQ_MF(0, 4);
  if (rg == 2) return RBQ_MF(0, 2);
  return RBQ_MF(0, 1);
#undef RBQ_MF
}

template <bool DBG>
const void* block_kernel(bool f4, int W, int rg) {
  return f4 ? kernel_for<true, DBG>(W, rg) : kernel_for<false, DBG>(W, rg);
}

int row_bytes(bool f4, int dp) { return f4 ? (dp + 127) / 128 * 128 : dp; }

// LDS for the query tile: at most what a block may hold beyond the kernel's
// static arrays (8 KiB reserved for them).
size_t lds_budget() {
  static size_t lim = 0;
  if (!lim) {
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) == hipSuccess && v > 16384)
      lim = (size_t)v - 8192;
    else
      lim = 56 * 1024;
  }
  return lim;
}

void allow_lds(const void* f, size_t bytes) {
  (void)hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

}  // namespace

int mfma_row_groups(int dp, bool f4, int npl, int want) {
  if (scan_frag_available(dp / 64, npl)) return 2;
  const size_t rb = (size_t)row_bytes(f4, dp);
  // default one group: with more, every wave re-reads RG query tiles from LDS
  // per 64 codes, and LDS bandwidth, not the MFMA rate, sets the pace
  int rg = want == 1 || want == 2 || want == 4 ? want : 1;
  while (rg > 1 && (size_t)16 * rg * rb > lds_budget()) rg >>= 1;
  return rg;
}

int scan_mfma_blocks_per_cu(int dp, bool f4, int rg, int npl) {
  if (scan_frag_available(dp / 64, npl)) return scan_frag_blocks_per_cu(dp / 64);
  const void* f = block_kernel<false>(f4, dp / 64, rg);
  const size_t bytes = (size_t)16 * rg * row_bytes(f4, dp);
  allow_lds(f, bytes);
  int v = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&v, f, kThreads, bytes) != hipSuccess || v < 1) v = 1;
  return v;
}

hipError_t launch_fill_i32(int32_t* p, int64_t n, int32_t v, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_i32, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, p, n, v);
  return hipGetLastError();
}

hipError_t launch_zero_u32(void* p, int64_t nwords, hipStream_t st) {
  if (nwords <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_zero_u32, dim3((unsigned)((nwords + 255) / 256)), dim3(256), 0, st, (uint32_t*)p, nwords);
  return hipGetLastError();
}

hipError_t launch_group_mfma(const SearchDev& s, hipStream_t st) {
  const int64_t np = s.nq * s.nprobe;
  const size_t shm = (size_t)s.nlist * sizeof(int32_t);   // at most 96 KiB (kMaxNlist)
  if (shm > 32768) allow_lds((const void*)k_group_count, shm);
  const unsigned blocks = (unsigned)((np + kGrpThreads * kGrpPer - 1) / (kGrpThreads * kGrpPer));
  hipLaunchKernelGGL(k_group_count, dim3(blocks), dim3(kGrpThreads), shm, st, s);
  if (blocks > 1) hipLaunchKernelGGL(k_group_offsets, dim3(1), dim3(kGrpThreads), 0, st, s);
  const int ub = s.frag ? (int)std::min<int64_t>(128, (np + 255) / 256) : 0;
  hipLaunchKernelGGL(k_group_scatter, dim3((unsigned)(ub + (np + 255) / 256)), dim3(256), 0, st, s, ub);
  return hipGetLastError();
}

hipError_t launch_scan_mfma(const SearchDev& s, int phase, int grid, hipStream_t st) {
  (void)phase;
  if (s.frag) return launch_scan_frag(s, grid, st);
  const bool f4 = s.mfma_f4 != 0;
  const void* f = block_kernel<false>(f4, s.W, s.mf_rg);
  const size_t bytes = (size_t)16 * s.mf_rg * row_bytes(f4, s.dp);
  allow_lds(f, bytes);
  void* args[] = {(void*)&s};
  return hipLaunchKernel(f, dim3(grid), dim3(kThreads), args, bytes, st);
}

hipError_t launch_debug_mfma(const SearchDev& s, const PairRec* rec, const int8_t* qu8,
                             int32_t list, int nchunks, int32_t* ip, int32_t* pc, float* est,
                             float* dist, float* lb, hipStream_t st) {
  if (nchunks <= 0) return hipSuccess;
  if (s.frag) return launch_debug_frag(s, rec, qu8, list, nchunks, ip, pc, est, dist, lb, st);
  const bool f4 = s.mfma_f4 != 0;
  const void* f = block_kernel<true>(f4, s.W, s.mf_rg);
  const size_t bytes = (size_t)16 * s.mf_rg * row_bytes(f4, s.dp);
  allow_lds(f, bytes);
  void* args[] = {(void*)&s, (void*)&rec, (void*)&qu8, (void*)&list, (void*)&ip, (void*)&pc,
                  (void*)&est, (void*)&dist, (void*)&lb};
  return hipLaunchKernel(f, dim3(nchunks), dim3(kThreads), args, bytes, st);
}

}  // namespace rbq
