// Per-replica fairness and served-experience metrics (Sec. 5 definitions: service
// provided for requests and interactions, served users, delayed users, aborted
// interactions and wasted tokens) plus Jain's index of the charged service.
// Integer accumulation only (atomics on integers are order-independent, so the
// result is deterministic); Jain's sums are exact 128-bit before the fp64 division.
// Each replica's total charged service is also summed exactly (the low and high 32-bit
// halves of every admitted cost in two 64-bit counters): at 2^62 or more the call
// reports an overflow, and below that no per-user sum can wrap.
#include <algorithm>

#include "fs_device.h"
#include "fs_launch.h"

namespace fs {
namespace {

enum : int {
  C_ADMITTED, C_THROTTLED, C_INTERACTIONS, C_FULL, C_ABORTED, C_WASTED,
  C_COST_LO,  // sum of the low 32 bits of the admitted costs
  C_COST_HI,  // sum of their high bits (costs are below 2^62)
  C_NUM = 8
};
enum : uint32_t { U_HAS = 1, U_FULL = 2, U_DELAYED = 4 };
enum : uint32_t { I_SERVED = 1, I_UNSERVED = 2 };

size_t up(size_t x) { return (x + 255) / 256 * 256; }

struct MLayout {
  size_t charged, uflags, iflags, counters, total;
};

MLayout mlayout(const fs_trace *t) {
  MLayout L;
  size_t ru = size_t(t->n_replicas) * size_t(t->n_users);
  size_t n = size_t(t->rep_off_h[t->n_replicas]);
  size_t o = 0;
  L.charged = o; o += up(ru * 8);
  L.uflags = o; o += up(ru * 4);
  L.iflags = o; o += up((n > 0 ? n : 1) * 4);
  L.counters = o; o += up(size_t(t->n_replicas) * C_NUM * 8);
  L.total = o;
  return L;
}

struct MArgs {
  DevTrace t;
  const int64_t *cost;
  const int8_t *status;
  const int32_t *admit_step;
  const int64_t *max_gap;
  int64_t tau;
  int32_t D;
  unsigned long long *charged;
  uint32_t *uflags, *iflags;
  unsigned long long *counters;
  fs_metrics m;
  int32_t *err;
  int32_t chunk;               // consecutive records a work-group takes
  unsigned long long *part;    // [R][parts][8] partial sums of the finish pass
  int32_t parts;               // work-groups a replica's users are summed by (1: in the finish pass)
};

__global__ void k_m_zero(MArgs a, int64_t RU, int64_t N) {
  const int64_t stride = int64_t(gridDim.x) * blockDim.x;
  for (int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; i < RU; i += stride) {
    a.charged[i] = 0;
    a.uflags[i] = 0;
  }
  if (a.t.call)  // (only later calls add interaction flags)
    for (int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; i < N; i += stride)
      a.iflags[i] = 0;
  for (int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; i < int64_t(a.t.R) * C_NUM;
       i += stride)
    a.counters[i] = 0;
}

__device__ inline bool first_call(const DevTrace &t, int64_t g) { return !t.call || t.call[g] == 0; }

// An interaction's flags: its later calls OR theirs into iflags[first call]; the first
// call's own flag comes from its status where it is read, which spares one atomic per
// interaction.
__device__ inline uint32_t own_iflag(int8_t st) { return st == 0 ? I_SERVED : I_UNSERVED; }

// The flags that the later calls of the interaction starting at g added (none, and
// the array is not cleared, when every record is a single-call interaction).
__device__ inline uint32_t later_iflags(const MArgs &a, int64_t g) {
  return a.t.call ? a.iflags[g] : 0u;
}

// admit_step - ts / tau > D.  For ts >= 0 the quotient is a floor, so this holds iff
// ts < (admit_step - D) * tau, which needs no division while the product fits.
__device__ inline bool is_delayed(int32_t astep, int64_t ts, int64_t tau, int32_t D) {
  if (ts >= 0 && tau <= (int64_t(1) << 30)) return ts < (int64_t(astep) - D) * tau;
  return int64_t(astep) - ts / tau > D;
}

__device__ inline unsigned long long wave_sum(unsigned long long v) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) {
    unsigned long long o = (unsigned long long)__shfl_xor((long long)v, m, 64);
    v += o;
  }
  return v;
}
// An admitted cost as charged service: in [0, 2^62), else a range error (not added).
__device__ inline bool cost_ok(int64_t c) { return c >= 0 && c < kValueLimit; }

// Replicas whose users fit in LDS: a work-group takes a chunk of consecutive records and,
// for each replica segment among them, sums the charged service and ORs the user
// flags in LDS tables indexed by user, then adds each touched user's values to global
// memory once.  Per-replica counts are reduced over the work-group.
constexpr int kChunk = 8192;      // at most
constexpr int kChunkLeast = 1024;
constexpr int kLdsUsers = 4096;  // beyond, the hash tables below (at 4,096 users the indexed ones take
                                 // 146 us against 304 for 1M requests, 426 against 486 for 10M)

// Sums three per-thread counts over the work-group (NW waves) and adds them to the
// replica's counters c0, c1, c2 (c < 0: unused).
// (c0b >= 0: x0's total also goes to counter c0b)
template <int NW = 4>
__device__ inline void block_count3(uint32_t x0, uint32_t x1, uint32_t x2,
                                    unsigned long long *cr, int c0, int c1, int c2,
                                    unsigned long long (*s_red)[NW], int c0b = -1) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const unsigned long long packed =
      uint64_t(x0) | (uint64_t(x1) << 21) | (uint64_t(x2) << 42);  // each at most a chunk's records
  const unsigned long long tw = wave_sum(packed);
  if (lane == 0) s_red[0][wave] = tw;
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long t = 0;
    for (int w = 0; w < NW; ++w) t += s_red[0][w];
    const unsigned long long m = (uint64_t(1) << 21) - 1;
    if (c0 >= 0 && (t & m)) atomicAdd(cr + c0, t & m);
    if (c0b >= 0 && (t & m)) atomicAdd(cr + c0b, t & m);
    if (c1 >= 0 && ((t >> 21) & m)) atomicAdd(cr + c1, (t >> 21) & m);
    if (c2 >= 0 && ((t >> 42) & m)) atomicAdd(cr + c2, (t >> 42) & m);
  }
}

// Adds the work-group's sums of the admitted costs' low and high halves to the
// replica's counters (each block sum is below 2^48: a chunk has fewer than 2^16 records).
template <int NW = 4>
__device__ inline void block_cost2(unsigned long long lo, unsigned long long hi,
                                   unsigned long long *cr, unsigned long long (*s_red)[NW]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const unsigned long long tl = wave_sum(lo), th = wave_sum(hi);
  if (lane == 0) {
    s_red[0][wave] = tl;
    s_red[1][wave] = th;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long l = 0, h = 0;
    for (int w = 0; w < NW; ++w) {
      l += s_red[0][w];
      h += s_red[1][w];
    }
    if (l) atomicAdd(cr + C_COST_LO, l);
    if (h) atomicAdd(cr + C_COST_HI, h);
  }
}

// Pass 1, LDS tables (U <= kLdsUsers): dynamic LDS of U * 12 bytes.
constexpr int kRecBatch = 4;  // records per thread whose loads are issued together
__global__ void __launch_bounds__(256) k_m_records_lds(MArgs a) {
  extern __shared__ unsigned long long s_dyn[];
  __shared__ unsigned long long s_red[2][4];
  const DevTrace &t = a.t;
  unsigned long long *const s_chg = s_dyn;
  uint32_t *const s_uf = reinterpret_cast<uint32_t *>(s_dyn + t.U);
  const int64_t c0 = blockIdx.x * int64_t(a.chunk);
  const int64_t c1 = c0 + a.chunk < t.N ? c0 + a.chunk : t.N;
  int32_t r = replica_of(t.rep_off, t.R, c0);
  int32_t code = 0;
  for (int64_t s0 = c0; s0 < c1; s0 = t.rep_off[r + 1], ++r) {
    while (t.rep_off[r + 1] <= s0) ++r;  // (empty replicas)
    const int64_t base = t.rep_off[r];
    const int64_t s1 = t.rep_off[r + 1] < c1 ? t.rep_off[r + 1] : c1;
    for (int32_t k = threadIdx.x; k < t.U; k += 256) {
      s_chg[k] = 0;
      s_uf[k] = 0;
    }
    __syncthreads();
    uint32_t n_adm = 0, n_thr = 0, n_int = 0;
    unsigned long long c_lo = 0, c_hi = 0;
    for (int64_t g0 = s0 + threadIdx.x; g0 < s1; g0 += kRecBatch * 256) {
      int32_t uk[kRecBatch], ap[kRecBatch], cl[kRecBatch], hd[kRecBatch], as[kRecBatch];
      int8_t st[kRecBatch];
      int64_t ts[kRecBatch], cs[kRecBatch];
#pragma unroll
      for (int j = 0; j < kRecBatch; ++j) {
        const int64_t g = g0 + j * 256;
        const bool v = g < s1;
        uk[j] = v ? t.user[g] : 0;
        ap[j] = v ? t.app[g] : 0;
        cl[j] = (v && t.call) ? t.call[g] : 0;
        hd[j] = (v && t.call) ? t.head[g] : 0;
        st[j] = v ? a.status[g] : int8_t(-1);
        as[j] = v ? a.admit_step[g] : 0;
        ts[j] = v ? t.ts[g] : 0;
        cs[j] = v ? a.cost[g] : 0;
      }
#pragma unroll
      for (int j = 0; j < kRecBatch; ++j) {
        const int64_t g = g0 + j * 256;
        if (g >= s1) continue;
        const int64_t i = g - base;
        const int32_t k = uk[j];
        bool ok = k >= 0 && k < t.U && ap[j] >= 0 && ap[j] < t.A;
        const bool fc = cl[j] == 0;
        int64_t h = i;
        if (ok && !fc) {
          h = hd[j];
          ok = h >= 0 && h < i;
        }
        if (!ok) {
          code = int32_t(FS_E_RANGE);
          continue;
        }
        const bool served = st[j] == 0;
        uint32_t uf = U_HAS;
        if (served && is_delayed(as[j], ts[j], a.tau, a.D)) uf |= U_DELAYED;
        // without interaction links a served request is a fully served interaction (the
        // interaction pass is not run)
        if (served && !t.call) uf |= U_FULL;
        if (!fc) atomicOr(a.iflags + base + h, own_iflag(st[j]));
        if (served && !cost_ok(cs[j])) {
          code = int32_t(FS_E_RANGE);
        } else if (served && cs[j]) {
          atomicAdd(&s_chg[k], (unsigned long long)cs[j]);
          c_lo += uint64_t(cs[j]) & 0xffffffffull;
          c_hi += uint64_t(cs[j]) >> 32;
        }
        atomicOr(&s_uf[k], uf);
        n_adm += served ? 1u : 0u;
        n_thr += st[j] > 0 ? 1u : 0u;
        n_int += fc ? 1u : 0u;
      }
    }
    __syncthreads();
    unsigned long long *const chg = a.charged + int64_t(r) * t.U;
    uint32_t *const ufg = a.uflags + int64_t(r) * t.U;
    for (int32_t k = threadIdx.x; k < t.U; k += 256) {
      const uint32_t f = s_uf[k];
      if (!f) continue;
      const unsigned long long c = s_chg[k];
      if (c) atomicAdd(chg + k, c);
      if ((ufg[k] & f) != f) atomicOr(ufg + k, f);
    }
    block_count3(n_adm, n_thr, n_int, a.counters + int64_t(r) * C_NUM, C_ADMITTED, C_THROTTLED,
                 C_INTERACTIONS, s_red, t.call ? -1 : int(C_FULL));
    __syncthreads();
    block_cost2(c_lo, c_hi, a.counters + int64_t(r) * C_NUM, s_red);
    __syncthreads();
  }
  if (code) raise_err(a.err, code);
}

// Pass 2, LDS tables (U <= kLdsUsers).
__global__ void __launch_bounds__(256) k_m_interactions_lds(MArgs a) {
  extern __shared__ unsigned long long s_dyn[];
  __shared__ unsigned long long s_red[2][4];
  const DevTrace &t = a.t;
  uint8_t *const s_full = reinterpret_cast<uint8_t *>(s_dyn);
  const int64_t c0 = blockIdx.x * int64_t(a.chunk);
  const int64_t c1 = c0 + a.chunk < t.N ? c0 + a.chunk : t.N;
  int32_t r = replica_of(t.rep_off, t.R, c0);
  for (int64_t s0 = c0; s0 < c1; s0 = t.rep_off[r + 1], ++r) {
    while (t.rep_off[r + 1] <= s0) ++r;
    const int64_t s1 = t.rep_off[r + 1] < c1 ? t.rep_off[r + 1] : c1;
    for (int32_t k = threadIdx.x; k < t.U; k += 256) s_full[k] = 0;
    __syncthreads();
    uint32_t n_full = 0, n_ab = 0;
    for (int64_t g = s0 + threadIdx.x; g < s1; g += 256) {
      if (!first_call(t, g)) continue;
      const int32_t k = t.user[g];
      if (k < 0 || k >= t.U) continue;
      const uint32_t f = later_iflags(a, g) | own_iflag(a.status[g]);
      const bool full = !(f & I_UNSERVED);
      if (full) s_full[k] = 1;  // (the same value from every writer)
      n_full += full ? 1u : 0u;
      n_ab += ((f & I_SERVED) && (f & I_UNSERVED)) ? 1u : 0u;
    }
    __syncthreads();
    uint32_t *const ufg = a.uflags + int64_t(r) * t.U;
    for (int32_t k = threadIdx.x; k < t.U; k += 256)
      if (s_full[k] && !(ufg[k] & U_FULL)) atomicOr(ufg + k, uint32_t(U_FULL));
    block_count3(n_full, n_ab, 0, a.counters + int64_t(r) * C_NUM, C_FULL, C_ABORTED, -1, s_red);
    __syncthreads();
  }
}

// More users than an LDS table holds: a work-group's chunk goes through an LDS hash table
// keyed by (replica, user), so that each user it meets reaches global memory once (a
// heavy user of one replica is in most chunks, thousands of times in each), and the
// per-replica counts are reduced over the work-group.  One replica's counters and its
// heaviest user are single addresses: with one atomic a wave on them the two passes over
// 10M requests of 100,000 users took 7.7 and 1.9 ms, the atomics of 156,000 waves on one
// line at 6-10 ns each.  What is left is bound by the atomics of the tables' entries, about
// 15 G/s over the chip, so a work-group takes as many records as its table of 8,192 users
// holds, one work-group a CU: 1.2M entries over those 10M requests, where chunks of 8,192
// records make 1.9M.
constexpr int kHashThreads = 1024;
constexpr int kHashWaves = kHashThreads / 64;
constexpr int kHashBits = 13;
constexpr int kHashSlots = 1 << kHashBits;
constexpr int kHashChunk = 40960;  // records of a work-group, at most
static_assert(kChunk < (1 << 16) && kHashChunk < (1 << 16), "packed counts and the block sums of the costs");
constexpr int kHashProbes = 8;
constexpr uint32_t kHashEmpty = 0xffffffffu;  // (a key is below R * U <= 2^31)

struct HashLds {
  unsigned long long sum[kHashSlots];
  uint32_t key[kHashSlots], flag[kHashSlots];
  unsigned long long red[2][kHashWaves];
};

__device__ inline uint32_t hash_slot(uint32_t key) { return (key * 2654435761u) >> (32 - kHashBits); }

// Replicas of few requests: with the counts reduced over the work-group segment after segment,
// its barriers (and idle waves) take longer than the records, so there each wave takes
// segments of its own and adds their counts itself.  20,000 replicas of 50 requests: 1,163 us by
// the work-group, 663 by waves; 2,000 of 500: 202 and 167; 1,000 of 1,000: 148 and 148; 64 of
// 1,000: 88 and 100; 500 of 2,000: 133 and 170.
constexpr int kWaveSegment = 512;  // requests a replica on average, below which waves take them (and
                                   // no replica has four times as many)

// Adds three per-thread counts and the costs' halves, summed over the wave, to the counters.
__device__ inline void wave_counts(uint32_t x0, uint32_t x1, uint32_t x2, unsigned long long *cr, int c0,
                                   int c1, int c2, int c0b, unsigned long long lo, unsigned long long hi) {
  const unsigned long long t =
      wave_sum(uint64_t(x0) | (uint64_t(x1) << 21) | (uint64_t(x2) << 42));  // (at most a chunk's records)
  const unsigned long long tl = wave_sum(lo), th = wave_sum(hi);
  if ((threadIdx.x & 63) != 0) return;
  const unsigned long long m = (uint64_t(1) << 21) - 1;
  if (t & m) atomicAdd(cr + c0, t & m);
  if (c0b >= 0 && (t & m)) atomicAdd(cr + c0b, t & m);
  if ((t >> 21) & m) atomicAdd(cr + c1, (t >> 21) & m);
  if (c2 >= 0 && ((t >> 42) & m)) atomicAdd(cr + c2, (t >> 42) & m);
  if (tl) atomicAdd(cr + C_COST_LO, tl);
  if (th) atomicAdd(cr + C_COST_HI, th);
}

// The replica segments of a work-group's chunk [c0, c1): take(r, s0, s1) for each, by the whole
// work-group one after the other, or (WAVES) by each wave for every kHashWaves-th.
template <bool WAVES, class F>
__device__ __forceinline__ void for_segments(const DevTrace &t, int64_t c0, int64_t c1, F take) {
  int32_t r = replica_of(t.rep_off, t.R, c0);
  if (WAVES) {
    for (r += threadIdx.x >> 6; r < t.R && t.rep_off[r] < c1; r += kHashWaves) {
      const int64_t b = t.rep_off[r], e = t.rep_off[r + 1];
      if (e > c0 && e > b) take(r, b > c0 ? b : c0, e < c1 ? e : c1);
    }
    return;
  }
  for (int64_t s0 = c0; s0 < c1; s0 = t.rep_off[r + 1], ++r) {
    while (t.rep_off[r + 1] <= s0) ++r;  // (empty replicas)
    take(r, s0, t.rep_off[r + 1] < c1 ? t.rep_off[r + 1] : c1);
  }
}

template <bool WAVES>
__global__ void __launch_bounds__(kHashThreads) k_m_records_hash(MArgs a) {
  extern __shared__ __align__(16) unsigned char m_smem[];
  HashLds &sm = *reinterpret_cast<HashLds *>(m_smem);
  const DevTrace &t = a.t;
  for (int k = threadIdx.x; k < kHashSlots; k += kHashThreads) {
    sm.sum[k] = 0;
    sm.key[k] = kHashEmpty;
    sm.flag[k] = 0;
  }
  __syncthreads();
  const int64_t c0 = blockIdx.x * int64_t(a.chunk);
  const int64_t c1 = c0 + a.chunk < t.N ? c0 + a.chunk : t.N;
  constexpr int kT = WAVES ? 64 : kHashThreads;  // threads a segment is taken by
  const int tid = WAVES ? threadIdx.x & 63 : threadIdx.x;
  int32_t code = 0;
  for_segments<WAVES>(t, c0, c1, [&](int32_t r, int64_t s0, int64_t s1) {
    const int64_t base = t.rep_off[r];
    uint32_t n_adm = 0, n_thr = 0, n_int = 0;
    unsigned long long c_lo = 0, c_hi = 0;
    for (int64_t g0 = s0 + tid; g0 < s1; g0 += kRecBatch * kT) {
      int32_t uk[kRecBatch], ap[kRecBatch], cl[kRecBatch], hd[kRecBatch], as[kRecBatch];
      int8_t st[kRecBatch];
      int64_t ts[kRecBatch], cs[kRecBatch];
#pragma unroll
      for (int j = 0; j < kRecBatch; ++j) {
        const int64_t g = g0 + j * kT;
        const bool v = g < s1;
        uk[j] = v ? t.user[g] : 0;
        ap[j] = v ? t.app[g] : 0;
        cl[j] = (v && t.call) ? t.call[g] : 0;
        hd[j] = (v && t.call) ? t.head[g] : 0;
        st[j] = v ? a.status[g] : int8_t(-1);
        as[j] = v ? a.admit_step[g] : 0;
        ts[j] = v ? t.ts[g] : 0;
        cs[j] = v ? a.cost[g] : 0;
      }
#pragma unroll
      for (int j = 0; j < kRecBatch; ++j) {
        const int64_t g = g0 + j * kT;
        if (g >= s1) continue;
        const int64_t i = g - base;
        bool ok = uk[j] >= 0 && uk[j] < t.U && ap[j] >= 0 && ap[j] < t.A;
        const bool fc = cl[j] == 0;
        int64_t h = i;
        if (ok && !fc) {
          h = hd[j];
          ok = h >= 0 && h < i;
        }
        if (!ok) {
          code = int32_t(FS_E_RANGE);
          continue;
        }
        const bool served = st[j] == 0;
        uint32_t uf = U_HAS;
        if (served && is_delayed(as[j], ts[j], a.tau, a.D)) uf |= U_DELAYED;
        if (served && !t.call) uf |= U_FULL;
        if (!fc) atomicOr(a.iflags + base + h, own_iflag(st[j]));
        unsigned long long c = 0;
        if (served && !cost_ok(cs[j])) {
          code = int32_t(FS_E_RANGE);
        } else if (served) {
          c = (unsigned long long)cs[j];
          c_lo += c & 0xffffffffull;
          c_hi += c >> 32;
        }
        n_adm += served ? 1u : 0u;
        n_thr += st[j] > 0 ? 1u : 0u;
        n_int += fc ? 1u : 0u;
        const uint32_t key = uint32_t(int64_t(r) * t.U + uk[j]);
        uint32_t s = hash_slot(key);
        int p = 0;
        for (; p < kHashProbes; ++p, s = (s + 1) & (kHashSlots - 1)) {
          uint32_t k = sm.key[s];
          if (k == kHashEmpty) k = atomicCAS(&sm.key[s], kHashEmpty, key);
          if (k == kHashEmpty || k == key) break;
        }
        if (p < kHashProbes) {
          if (c) atomicAdd(&sm.sum[s], c);
          if ((sm.flag[s] & uf) != uf) atomicOr(&sm.flag[s], uf);
        } else {  // (the table is full around the slot)
          if (c) atomicAdd(a.charged + key, c);
          if ((a.uflags[key] & uf) != uf) atomicOr(a.uflags + key, uf);
        }
      }
    }
    unsigned long long *const cr = a.counters + int64_t(r) * C_NUM;
    if (WAVES) {
      wave_counts(n_adm, n_thr, n_int, cr, C_ADMITTED, C_THROTTLED, C_INTERACTIONS, t.call ? -1 : int(C_FULL),
                  c_lo, c_hi);
      return;
    }
    block_count3<kHashWaves>(n_adm, n_thr, n_int, cr, C_ADMITTED, C_THROTTLED, C_INTERACTIONS, sm.red,
                             t.call ? -1 : int(C_FULL));
    __syncthreads();
    block_cost2<kHashWaves>(c_lo, c_hi, cr, sm.red);
    __syncthreads();
  });
  __syncthreads();
  for (int k = threadIdx.x; k < kHashSlots; k += kHashThreads) {
    const uint32_t key = sm.key[k];
    if (key == kHashEmpty) continue;
    const uint32_t f = sm.flag[k];
    if (sm.sum[k]) atomicAdd(a.charged + key, sm.sum[k]);
    if ((a.uflags[key] & f) != f) atomicOr(a.uflags + key, f);
  }
  if (code) raise_err(a.err, code);
}

// Pass 2 with many users: a fully served interaction sets its user's flag once per
// work-group (a direct-mapped table of the users already seen) and only when the flag is
// not yet visible.
template <bool WAVES>
__global__ void __launch_bounds__(kHashThreads) k_m_interactions_hash(MArgs a) {
  __shared__ uint32_t s_seen[kHashSlots];
  __shared__ unsigned long long s_red[2][kHashWaves];
  const DevTrace &t = a.t;
  for (int k = threadIdx.x; k < kHashSlots; k += kHashThreads) s_seen[k] = kHashEmpty;
  __syncthreads();
  const int64_t c0 = blockIdx.x * int64_t(a.chunk);
  const int64_t c1 = c0 + a.chunk < t.N ? c0 + a.chunk : t.N;
  constexpr int kT = WAVES ? 64 : kHashThreads;
  const int tid = WAVES ? threadIdx.x & 63 : threadIdx.x;
  for_segments<WAVES>(t, c0, c1, [&](int32_t r, int64_t s0, int64_t s1) {
    uint32_t n_full = 0, n_ab = 0;
    for (int64_t g0 = s0 + tid; g0 < s1; g0 += kRecBatch * kT) {
      int32_t uk[kRecBatch];
      uint32_t f[kRecBatch];
      bool ok[kRecBatch];
#pragma unroll
      for (int j = 0; j < kRecBatch; ++j) {
        const int64_t g = g0 + j * kT;
        ok[j] = g < s1 && first_call(t, g);
        uk[j] = g < s1 ? t.user[g] : -1;
        f[j] = g < s1 ? (later_iflags(a, g) | own_iflag(a.status[g])) : 0u;
      }
#pragma unroll
      for (int j = 0; j < kRecBatch; ++j) {
        if (!ok[j] || uk[j] < 0 || uk[j] >= t.U) continue;
        const bool full = !(f[j] & I_UNSERVED);
        n_full += full ? 1u : 0u;
        n_ab += ((f[j] & I_SERVED) && (f[j] & I_UNSERVED)) ? 1u : 0u;
        if (!full) continue;
        const uint32_t key = uint32_t(int64_t(r) * t.U + uk[j]);
        const uint32_t s = hash_slot(key);
        // (the exchange lets one of the user's lanes go on, and again after another user)
        if (s_seen[s] == key || atomicExch(&s_seen[s], key) == key) continue;
        if (!(a.uflags[key] & U_FULL))  // (a stale value only costs an atomic)
          atomicOr(a.uflags + key, uint32_t(U_FULL));
      }
    }
    unsigned long long *const cr = a.counters + int64_t(r) * C_NUM;
    if (WAVES) {
      wave_counts(n_full, n_ab, 0, cr, C_FULL, C_ABORTED, -1, -1, 0, 0);
      return;
    }
    block_count3<kHashWaves>(n_full, n_ab, 0, cr, C_FULL, C_ABORTED, -1, s_red);
    __syncthreads();
  });
}

// Pass 3: per admitted record of an aborted interaction -- wasted tokens.  Chunked like
// the LDS passes; a replica segment without aborted interactions (every replica under
// the paper's policy) is skipped without reading its records.
__global__ void __launch_bounds__(256) k_m_wasted(MArgs a) {
  __shared__ unsigned long long s_red[1][4];
  const DevTrace &t = a.t;
  const int64_t c0 = blockIdx.x * int64_t(a.chunk);
  const int64_t c1 = c0 + a.chunk < t.N ? c0 + a.chunk : t.N;
  int32_t r = replica_of(t.rep_off, t.R, c0);
  for (int64_t s0 = c0; s0 < c1; s0 = t.rep_off[r + 1], ++r) {
    while (t.rep_off[r + 1] <= s0) ++r;
    const int64_t base = t.rep_off[r];
    const int64_t s1 = t.rep_off[r + 1] < c1 ? t.rep_off[r + 1] : c1;
    unsigned long long *const cr = a.counters + int64_t(r) * C_NUM;
    if (cr[C_ABORTED] == 0) continue;  // (uniform over the work-group)
    unsigned long long w = 0;
    for (int64_t g = s0 + threadIdx.x; g < s1; g += 256) {
      if (a.status[g] != 0) continue;
      const int64_t i = g - base;
      const int64_t h = first_call(t, g) ? i : t.head[g];
      if (h < 0 || h > i) continue;
      const uint32_t f =
          later_iflags(a, base + h) | (h == i ? I_SERVED : own_iflag(a.status[base + h]));
      if ((f & I_SERVED) && (f & I_UNSERVED)) w += (unsigned long long)tokens_of(t, g);
    }
    const unsigned long long tw = wave_sum(w);
    if ((threadIdx.x & 63) == 0) s_red[0][threadIdx.x >> 6] = tw;
    __syncthreads();
    if (threadIdx.x == 0) {
      const unsigned long long tot = s_red[0][0] + s_red[0][1] + s_red[0][2] + s_red[0][3];
      if (tot) atomicAdd(cr + C_WASTED, tot);
    }
    __syncthreads();
  }
}

struct U128 {
  unsigned long long lo, hi;
};
__device__ inline U128 add128(U128 a, U128 b) {
  U128 c;
  c.lo = a.lo + b.lo;
  c.hi = a.hi + b.hi + (c.lo < a.lo ? 1ull : 0ull);
  return c;
}
__device__ inline double to_double(U128 v) {
  return double(v.hi) * 18446744073709551616.0 + double(v.lo);
}

// The sums over a replica's users that pass 4 needs, of the thread's share of [k0, k1).
struct UserSums {
  U128 s1 = {0, 0}, s2 = {0, 0};
  unsigned long long cnt[3] = {0, 0, 0};  // users with a request, fully served, delayed
};
__device__ inline UserSums user_sums(const MArgs &a, int32_t r, uint32_t k0, uint32_t k1) {
  UserSums u;
  for (uint32_t k = k0 + threadIdx.x; k < k1; k += blockDim.x) {  // (k1 may be 2^31 - 1)
    const int64_t uk = int64_t(r) * a.t.U + k;
    const uint32_t f = a.uflags[uk];
    const unsigned long long x = a.charged[uk];
    if (!(f & U_HAS)) continue;
    u.cnt[0] += 1;
    u.cnt[1] += (f & U_FULL) ? 1 : 0;
    u.cnt[2] += (f & U_DELAYED) ? 1 : 0;
    u.s1 = add128(u.s1, U128{x, 0});
    const U128 sq{x * x, __umul64hi(x, x)};
    u.s2 = add128(u.s2, sq);
  }
  return u;
}
struct SumsLds {
  U128 s1[256], s2[256];
  unsigned long long cnt[256][3];
};
// The work-group's total (256 threads), left in entry 0.
__device__ inline void block_sums(const UserSums &u, SumsLds &sm) {
  sm.s1[threadIdx.x] = u.s1;
  sm.s2[threadIdx.x] = u.s2;
  for (int c = 0; c < 3; ++c) sm.cnt[threadIdx.x][c] = u.cnt[c];
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) {
      sm.s1[threadIdx.x] = add128(sm.s1[threadIdx.x], sm.s1[threadIdx.x + w]);
      sm.s2[threadIdx.x] = add128(sm.s2[threadIdx.x], sm.s2[threadIdx.x + w]);
      for (int c = 0; c < 3; ++c) sm.cnt[threadIdx.x][c] += sm.cnt[threadIdx.x + w][c];
    }
    __syncthreads();
  }
}

// The users of a replica in a.parts work-groups (many users of few replicas: one work-group
// over 100,000 users took 230 us), each one's sums to its row.
__global__ void __launch_bounds__(256) k_m_user_parts(MArgs a) {
  __shared__ SumsLds sm;
  const int32_t r = blockIdx.x / a.parts, p = blockIdx.x % a.parts;
  const uint32_t U = a.t.U, per = (U + a.parts - 1) / a.parts;  // (k0 + per is below 2^31 + 512)
  const uint32_t k0 = p * per, k1 = k0 + per < U ? k0 + per : U;
  block_sums(user_sums(a, r, k0, k1), sm);
  if (threadIdx.x == 0) {
    unsigned long long *const o = a.part + int64_t(blockIdx.x) * 8;
    o[0] = sm.s1[0].lo;
    o[1] = sm.s1[0].hi;
    o[2] = sm.s2[0].lo;
    o[3] = sm.s2[0].hi;
    for (int c = 0; c < 3; ++c) o[4 + c] = sm.cnt[0][c];
  }
}

// Pass 4: one block per replica -- Jain's index and the percentages.
__global__ void __launch_bounds__(256) k_m_finish(MArgs a) {
  const int32_t r = blockIdx.x;
  __shared__ SumsLds sm;
  UserSums u;
  if (a.parts == 1) {
    u = user_sums(a, r, 0, a.t.U);
  } else if (int(threadIdx.x) < a.parts) {
    const unsigned long long *const o = a.part + (int64_t(r) * a.parts + threadIdx.x) * 8;
    u.s1 = U128{o[0], o[1]};
    u.s2 = U128{o[2], o[3]};
    for (int c = 0; c < 3; ++c) u.cnt[c] = o[4 + c];
  }
  block_sums(u, sm);
  if (threadIdx.x == 0) {
    const unsigned long long *C = a.counters + r * C_NUM;
    const int64_t n = a.t.rep_off[r + 1] - a.t.rep_off[r];
    U128 S1 = sm.s1[0], S2 = sm.s2[0];
    const unsigned long long nu = sm.cnt[0][0];
    // the exact total charged service: hi * 2^32 + lo
    const unsigned long long lo = C[C_COST_LO], hi = C[C_COST_HI];
    if ((hi >> 30) != 0 || ((hi << 32) + lo) < (hi << 32) ||
        (hi << 32) + lo >= (unsigned long long)kValueLimit)
      raise_err(a.err, FS_E_OVERFLOW);
    double jain = 1.0;
    if (S2.lo != 0 || S2.hi != 0) {
      double d1 = to_double(S1);
      jain = (d1 * d1) / (double(nu) * to_double(S2));
    }
    auto pct = [](unsigned long long x, unsigned long long y) {
      return y == 0 ? 0.0 : 100.0 * double(x) / double(y);
    };
    a.m.jain[r] = jain;
    a.m.max_gap_tokens[r] = double(a.max_gap[r]) / 65536.0;
    a.m.svc_req_pct[r] = pct(C[C_ADMITTED], (unsigned long long)n);
    a.m.svc_int_pct[r] = pct(C[C_FULL], C[C_INTERACTIONS]);
    a.m.served_users_pct[r] = pct(sm.cnt[0][1], nu);
    a.m.delayed_users_pct[r] = pct(sm.cnt[0][2], nu);
    a.m.throttled[r] = int64_t(C[C_THROTTLED]);
    a.m.aborted_midway[r] = int64_t(C[C_ABORTED]);
    a.m.wasted_tokens[r] = int64_t(C[C_WASTED]);
  }
}

int grid_for(int64_t n, int threads) {
  int64_t b = (n + threads - 1) / threads;
  if (b < 1) b = 1;
  if (b > 65536) b = 65536;
  return int(b);
}

}  // namespace

size_t metrics_workspace_bytes(const fs_trace *t) { return mlayout(t).total; }

hipError_t launch_metrics(const fs_trace *t, const int64_t *cost, const fs_outputs *out,
                          const fs_engine *eng, int32_t delay_steps, fs_metrics *m, void *ws,
                          hipStream_t s) {
  MLayout L = mlayout(t);
  char *w = static_cast<char *>(ws);
  MArgs a;
  a.t = dev_trace(t);
  a.cost = cost;
  a.status = out->status;
  a.admit_step = out->admit_step;
  a.max_gap = out->max_gap;
  a.tau = eng->step_us;
  a.D = delay_steps;
  a.charged = reinterpret_cast<unsigned long long *>(w + L.charged);
  a.uflags = reinterpret_cast<uint32_t *>(w + L.uflags);
  a.iflags = reinterpret_cast<uint32_t *>(w + L.iflags);
  a.counters = reinterpret_cast<unsigned long long *>(w + L.counters);
  a.m = *m;
  a.err = out->err;
  const int64_t RU = int64_t(t->n_replicas) * t->n_users;
  const int64_t N = a.t.N;
  hipLaunchKernelGGL(k_m_zero, dim3(grid_for(RU > N ? RU : N, 256)), dim3(256), 0, s, a, RU, N);
  // The finish pass in parts of at least 2,048 users, up to 256 a replica and about 1,024
  // work-groups, when the rows fit where the interaction flags were (not read any more).
  a.part = reinterpret_cast<unsigned long long *>(a.iflags);
  a.parts = 1;
  {
    int64_t parts = std::min<int64_t>(t->n_users / 2048, 256);
    parts = std::min<int64_t>(parts, std::max<int64_t>(1024 / t->n_replicas, 1));
    if (parts > 1 && size_t(t->n_replicas) * size_t(parts) * 64 <= size_t(N) * 4) a.parts = int32_t(parts);
  }
  // Chunks of kChunk records, less when they would leave the chip idle (four a CU), but at
  // most 256 of one replica: its counters are one line that every chunk of it adds to.  One
  // replica of 1M requests in 1,024, 512, 256 and 128 chunks: 173, 115, 108 and 149 us with
  // 1,024 users, 242, 167, 146 and 170 us with 4,096; 64 replicas of 20,000 requests in 1,280,
  // 640, 320 and 192 chunks: 71, 84, 107 and 162 us.
  int64_t most_n = 0;
  for (int32_t r = 0; r < t->n_replicas; ++r)
    most_n = std::max<int64_t>(most_n, t->rep_off_h[r + 1] - t->rep_off_h[r]);
  // (The wasted-token pass adds one value a chunk: four chunks a CU.)
  auto chunk_of = [](int64_t per) {
    return int32_t(std::min<int64_t>(kChunk, (std::max<int64_t>(per, kChunkLeast) + 255) / 256 * 256));
  };
  const int32_t wasted_chunk = chunk_of(N / 1024);
  a.chunk = chunk_of(std::max<int64_t>(N / 1024, most_n / 256));
  if (N > 0) {
    const int64_t chunks = (N + a.chunk - 1) / a.chunk;
    if (t->n_users <= kLdsUsers) {
      hipLaunchKernelGGL(k_m_records_lds, dim3(chunks), dim3(256), size_t(t->n_users) * 12, s, a);
      if (t->call)  // (without links the records pass counts the fully served interactions)
        hipLaunchKernelGGL(k_m_interactions_lds, dim3(chunks), dim3(256), size_t(t->n_users), s, a);
    } else {
      const bool waves = N / t->n_replicas < kWaveSegment && most_n < 4 * kWaveSegment;
      const auto records = waves ? k_m_records_hash<true> : k_m_records_hash<false>;
      const auto interactions = waves ? k_m_interactions_hash<true> : k_m_interactions_hash<false>;
      (void)hipFuncSetAttribute(reinterpret_cast<const void *>(records),
                                hipFuncAttributeMaxDynamicSharedMemorySize, int(sizeof(HashLds)));
      // a whole number of work-groups a CU, each of at most kHashChunk records
      const int64_t rounds = (N + int64_t(kHashChunk) * 256 - 1) / (int64_t(kHashChunk) * 256);
      const int64_t per = (N + rounds * 256 - 1) / (rounds * 256);
      a.chunk = int32_t(std::max<int64_t>((per + 255) / 256 * 256, 2048));
      const int64_t groups = (N + a.chunk - 1) / a.chunk;
      hipLaunchKernelGGL(records, dim3(groups), dim3(kHashThreads), sizeof(HashLds), s, a);
      if (t->call)
        hipLaunchKernelGGL(interactions, dim3(groups), dim3(kHashThreads), 0, s, a);
    }
    a.chunk = wasted_chunk;
    hipLaunchKernelGGL(k_m_wasted, dim3((N + wasted_chunk - 1) / wasted_chunk), dim3(256), 0, s, a);
  }
  if (a.parts > 1)
    hipLaunchKernelGGL(k_m_user_parts, dim3(t->n_replicas * a.parts), dim3(256), 0, s, a);
  hipLaunchKernelGGL(k_m_finish, dim3(t->n_replicas), dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace fs
