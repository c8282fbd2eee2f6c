// WSC scheduler steps for the paper's policy under the token-budget step engine: the
// pool pass, one wavefront per trace replica, one queued call per lane.
//
// The decisions of a step are a merge.  A user's queued calls are served in a fixed
// order (its ready later calls by record, then its first calls by record), and the
// counter a call is chosen by is the user's counter plus the costs of the user's calls
// ahead of it, which does not depend on the order in which other users are served.  So
// every queued call has a key (tier, counter before it, user, position) that stays the
// same while the calls ahead of it are admitted, and a step admits the queued calls in
// the order of their keys while its budget lasts.  A lane keeps one call with its key;
// a step's admissions are: each lane's rank and the tokens ranked before it (one pass
// over the occupied lanes), the lanes whose tokens before are below the budget, and
// their outputs, all lane-parallel.  Admitted lanes just fall free: no other key moves.
//
// What ends a batch early (the rest of the step follows in another batch): a call whose
// next call has already arrived (that one becomes ready at the charged counter), and a
// user's last pooled call while more of its first calls wait in the spill list.
//
// Per-user state (a slot: the counter after the user's pooled calls, their number, the
// spill list) and the counters of the window's users are in LDS, read and updated by the
// lanes of the user's calls.  First calls beyond the pool's room go to the user's segment of
// the state buffer and come back 16 at a time.
//
// What bounds it: the latency of one wave's dependent instructions (about 8 clocks each; no
// memory or matrix unit is near its rate), so the work per step is what is kept small.  One
// call per lane replaced one user per lane with sequential admissions (about 1,300 clocks
// each: an argmin, the chosen user's next call and its new key in a dependent chain), which
// remains in fs_sched_onchip.hip for the policy flags, the literal engine, the replicas that
// outgrow the pool (more than 64 users and ready calls at once) and deep queues of chained calls
// (kDeep).  Kernel and set-up, before and after: one replica of 300,000 requests, 100,000 users
// and 17 admissions a step 204 -> 59 ms; 1,024 replicas of 20,000 requests without interactions
// 12.8 -> 8.9 ms; 64 replicas of 100,000 requests, 12 traces, 74-79 -> 55-81 ms (median 75.6 ->
// 58.6; the longest are those with a deep replica).
#pragma once
#include "fs_sched_common.h"

namespace fs {
namespace sched {
namespace {

constexpr int64_t kPackLimit = int64_t(1) << 40;  // costs that fit a packed request
constexpr uint64_t kTokMask = (uint64_t(1) << 24) - 1;
// Whether a call fits a packed request, (cost << 24) | tokens (its three lengths, each below
// 2^24, may sum to more); one that does not is taken by the global-memory pass.
__device__ __forceinline__ bool fits_packed(int64_t cst, int32_t tok) {
  return ((uint64_t(cst) / uint64_t(kPackLimit)) | (uint32_t(tok) >> 24)) == 0;  // (cst >= 0)
}
// window flags
constexpr int32_t kFirst = 1;        // first call of its interaction
constexpr int32_t kReasonShift = 1;  // bits 1-2: raw throttle reason (0 within limits)
constexpr int32_t kHeadBlk = 8;      // later call whose interaction's first call was throttled
constexpr int32_t kPrevAdm = 16;     // later call whose previous call has been admitted
constexpr int32_t kBig = 32;         // does not fit a packed request
constexpr int32_t kPrevDrop = 64;    // later call whose previous call was dropped

// A queued request on chip: record, its next call (-1: none), (cost << 24) | tokens.
struct __align__(16) Ent {
  int32_t rec, succ;
  uint32_t lo, hi;
};

__device__ inline Ent mk_ent(int32_t rec, int32_t sc, uint32_t lo, uint32_t hi) {
  Ent e;
  e.rec = rec;
  e.succ = sc;
  e.lo = lo;
  e.hi = hi;
  return e;
}

__device__ inline int32_t ff1(uint64_t m) { return __ffsll((long long)m) - 1; }

// A field of the kernel's argument block, loaded with a scalar load where it is used
// instead of being held in a scalar register for the whole kernel.  The block is the
// kernel's only argument, at the start of the kernarg segment.
template <class T>
__device__ __forceinline__ T arg_at(uint32_t off) {
  __asm__ volatile("" : "+s"(off));
  const __attribute__((address_space(4))) char *k =
      (const __attribute__((address_space(4))) char *)__builtin_amdgcn_kernarg_segment_ptr();
  return *(const __attribute__((address_space(4))) T *)(k + off);
}
#define KARG(f) arg_at<decltype(SchedArgs{}.f)>(uint32_t(offsetof(SchedArgs, f)))

#define STATE(T, field) reinterpret_cast<T *>(KARG(state) + KARG(L.field))

// Lane masks: the lanes where p holds (no detour over an integer), whether this lane is in
// a mask, the lanes of a mask below this one, and a nonempty mask's first lane.
__device__ __forceinline__ uint64_t bal(bool p) { return __builtin_amdgcn_ballot_w64(p); }
__device__ __forceinline__ bool in_mask(uint64_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }
__device__ __forceinline__ int32_t below(uint64_t m) {
  return int32_t(__builtin_amdgcn_mbcnt_hi(uint32_t(m >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(m), 0)));
}
__device__ __forceinline__ int first_of(uint64_t m) { return __builtin_ctzll(m); }
// a < b for wave-uniform values less than 2^62 apart, in scalar registers (there is no
// scalar 64-bit order comparison, and a vector one would move the values it selects).
__device__ __forceinline__ bool less_s(int64_t a, int64_t b) {
  int32_t h = int32_t(uint64_t(a - b) >> 32);
  __asm__ volatile("" : "+s"(h));
  return h < 0;
}

// floor(ts / tau), at most INT32_MAX, for ts >= 0: the product with the reciprocal is off by
// less than one below 2^32, so one correction either way makes it exact.
__device__ __forceinline__ int32_t step_of(int64_t ts, int64_t tau, double tau_inv) {
  const double f = double(ts) * tau_inv;
  int64_t q = f < 4294967296.0 ? int64_t(uint32_t(f)) : int64_t(1) << 32;
  const int64_t d = ts - q * tau;
  q += (q >> 32) ? 0 : (d < 0 ? -1 : (d >= tau ? 1 : 0));
  return q < INT32_MAX ? int32_t(q) : INT32_MAX;
}

constexpr uint32_t kPTier1 = 0x80000000u;  // a first call, in the key's high word
constexpr int kAheadBits = 6;              // position among the user's pooled calls
// Calls the pool takes without looking at whose they are, and a user's share beyond that.  More
// room makes more evictions where queues are long, less makes more refills.  In ms, with 28 and
// 6 / 20 and 4 / 44 and 6 / 28 and 2 / 28 and 12: one replica of 100,000 users 59.2 / 62.4 /
// 57.7 / 61.5 / 58.2; 64 replicas (three traces) 59.1 / 59.7 / 59.1 / 60.7 / 59.2; 64 with long
// queues and no interactions 12.1 / 12.3 / 13.3 / 14.5 / 14.3; one of 2,000 users with a long queue
// 68.9 / 68.4 / 72.9 / 71.8 / 72.2.
constexpr int kPoolRoom = 28, kPoolShare = 6;
// A pool of more than kNearMin calls is ranked below the key of rank kNearRank while at least
// kNearLeast calls are: a ranking costs about 55 clocks a call and a step admits a handful.  In
// ms, with 20, 8, 16 / always all / 12, 4, 8 / 32, 8, 28 / 20, 2, 16: 64 replicas (three traces)
// 59.1 / 62.5 / 60.3 / 60.8 / 59.0, the same in 12 slices 8.70 / 9.33 / 8.80 / 8.93 / 8.66, one
// replica of 100,000 users 59.2 / 57.5 / 61.3 / 58.4 / 61.1.
constexpr int kNearMin = 20, kNearLeast = 8, kNearRank = 16;

// A queue that the slot pass serves faster is handed over to it: kDeep spilled calls or more and
// fewer than kSlow / kSlowDen admissions a batch over the last kRateBatches, or kVeryDeep and
// fewer than kSlowVery / kSlowDen (chains whose next calls have arrived end most batches after one
// or two calls, and each batch is ranked anew).  The slot pass takes about 2,300 clocks an
// admission; the pool 2,150 at 2.1 admissions a batch, 2,300 to 2,430 at 1.8, and from 1,024
// spilled calls on 2,370 to 2,540 at 2.0 to 2.2 and up to 2,790 at 1.8.  In ms, slot pass alone /
// pool alone / this rule: 64 replicas of 20,000 requests at 0.8 of the capacity 16.0 / 21.1 /
// 16.9, at 0.6 and never throttled 73.2 / 86.6 / 74.4; 64 of 100,000 without limits 92.2 / 121.7 /
// 97.4 and with equal weights 96.7 / 121.6 / 100.5; with limits, 12 traces, 75-80 / 77-88 / 75-83
// and 16 of another kind 74-79 / 52-90 / 52-82.  A rate of 2 from 64 calls on (or a look every 128
// batches) also hands over queues that the pool serves faster (65 -> 74), as does kVeryDeep at
// 1,024 (65 -> 68); a rate of 5/3 leaves some that it serves slower (82.4 for 78.8), as does
// kDeep at 256 (16.8 -> 17.1).
constexpr int kDeep = 64, kVeryDeep = 1536, kSlow = 9, kSlowVery = 11, kSlowDen = 5, kRateBatches = 512;
constexpr int32_t kOutDeep = 3;  // rs->overflow of a replica handed over for its queue

// A slot's record: the counter after the user's pooled calls; the number of pooled calls, of
// the ready ones among them (kRdyOne each) and the user's window lane plus one (kWinOne
// each), all at most 64; the number of spilled calls (as many as the replica has records).
struct __align__(16) SlotRec {
  uint32_t plo, phi, num, spilled;
};
constexpr uint32_t kNumMask = 0xffu, kRdyOne = 0x100u, kWinOne = 0x1000000u;
__device__ __forceinline__ uint32_t ready_of(uint32_t num) { return (num / kRdyOne) & kNumMask; }

constexpr int kOutStage = 192;  // admissions kept until the next window (then written together)

// Byte offsets of the pool pass's LDS (the cache, counters and tables follow).
// Entry 64 of an array takes the stores of lanes that have none to make.
struct PoolLds {
  static constexpr int stage = 0;                // [65] two 16-byte words: calls placed
  static constexpr int adm = stage + 65 * 32;     // [kOutStage + 1] admitted records and steps
  static constexpr int slot = adm + (kOutStage + 2) * 8;  // [65] SlotRec
  static constexpr int win = slot + 65 * 16;     // [65] a window user: counter (8), slot or -1 (4)
  static constexpr int uc = win + 65 * 16;       // [65] u64 the user's counter
  static constexpr int xu = uc + 66 * 8;         // [65] i32 user of the slot, -1 free
  static constexpr int sph = xu + 66 * 4;        // [64] u32 first spilled call's place
  static constexpr int seg = sph + 64 * 4;       // [64] u32 the user's segment
  static constexpr int cap = seg + 64 * 4;       // [64] u32 its places
  static constexpr int freex = cap + 64 * 4;     // [65] i32 free slots (a stack)
  static constexpr int end = (freex + 66 * 4 + 15) / 16 * 16;
};
// Entries of the request-state table past the cache's M: states of records it no longer holds.
constexpr int kStAdm = 0, kStNone = 1, kStBlk = 2, kStPad = 16;

// Ranks of the pooled calls in the order of (key, user, position) and the tokens ranked
// before each, as rank << 26 | tokens (the pool's tokens sum to less than 2^26).  p: the
// order as one word, all ones in a lane without a ranked call.  The calls are lanes
// [0, top) of sh, sl (their words) and sa (their tokens | 1 << 26), taken eight at a time
// by lane reads: new calls take the lowest free lanes, so the pool's own lanes serve.  A
// ranking takes about 300 clocks and 44 to 58 more a call (635 for 8.9 calls on average over 1,024
// replicas without interactions, 965 for 11.5 over 64 with).
__device__ __forceinline__ uint32_t pool_rank(uint64_t p, uint32_t sh, uint32_t sl, uint32_t sa, int32_t top) {
  uint32_t acc = 0;
#pragma unroll
  for (int b = 0; b < 8; ++b) {
    if (8 * b >= top) break;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int j = 8 * b + i;
      const uint64_t pj = (uint64_t(rdlu(sh, j)) << 32) | rdlu(sl, j);
      const uint32_t aj = rdlu(sa, j);
      acc += pj < p ? aj : 0u;
    }
  }
  return acc;
}

// The same for keys too far apart for one word, or more tokens: rank and tokens apart.
__device__ __forceinline__ void pool_rank_wide(uint64_t k, uint32_t ua, uint32_t tok, uint64_t occ,
                                               uint32_t &rank, uint32_t &pre) {
  uint32_t n = 0, acc = 0;
  for (uint64_t m = occ; m; m &= m - 1) {
    const int j = ff1(m);
    const uint64_t kj = uint64_t(rdl64(int64_t(k), j));
    const uint32_t uj = rdlu(ua, j), tj = rdlu(tok, j);
    const bool lt = kj < k || (kj == k && uj < ua);
    n += lt ? 1u : 0u;
    acc += lt ? tj : 0u;
  }
  rank = n;
  pre = acc;
}

// Runs replica blockIdx.x until a.n_steps are done or its queue is drained, or hands it
// over (rs->overflow, at a point before an arrival) when it outgrows the pool.  resumed: it
// comes back within the launch (rs->s_end is where the call ends).
template <bool LINKS>
__device__ __forceinline__ void pool_replica(const SchedArgs &a, char *smem, bool resumed) {
  const int32_t r = blockIdx.x;
  const int lane = threadIdx.x;
  const uint64_t lt = (uint64_t(1) << lane) - 1;
  const int32_t M = a.oc.p_cache, tab = a.oc.p_tab;
  const bool ulds = a.oc.p_users != 0;
  const int32_t U = a.t.U;
  const int ubits = U > 1 ? 32 - __builtin_clz(uint32_t(U - 1)) : 0;
  const int ksh = ubits + kAheadBits;  // shift of the counter in the one-word order
  const bool want_coa = a.counter_on_arrival != nullptr;
  const bool want_seq = a.admit_seq != nullptr || a.counter_after != nullptr;
  uint4 *const s_stage = reinterpret_cast<uint4 *>(smem + PoolLds::stage);
  uint2 *const s_adm = reinterpret_cast<uint2 *>(smem + PoolLds::adm);
  SlotRec *const s_slot = reinterpret_cast<SlotRec *>(smem + PoolLds::slot);
  uint4 *const s_win = reinterpret_cast<uint4 *>(smem + PoolLds::win);
  unsigned long long *const s_uc = reinterpret_cast<unsigned long long *>(smem + PoolLds::uc);
  int32_t *const s_xu = reinterpret_cast<int32_t *>(smem + PoolLds::xu);
  uint32_t *const s_sph = reinterpret_cast<uint32_t *>(smem + PoolLds::sph);
  uint32_t *const s_seg = reinterpret_cast<uint32_t *>(smem + PoolLds::seg);
  uint32_t *const s_cap = reinterpret_cast<uint32_t *>(smem + PoolLds::cap);
  int32_t *const s_free = reinterpret_cast<int32_t *>(smem + PoolLds::freex);
  Ent *const cache = reinterpret_cast<Ent *>(smem + PoolLds::end);         // [M]
  int64_t *const u_lds = reinterpret_cast<int64_t *>(cache + M);           // [U]
  uint8_t *const u_rep = reinterpret_cast<uint8_t *>(u_lds + (ulds ? U : 0));  // [tab]
  uint8_t *const st8 = u_rep + tab;                                        // [M + kStPad]

  const int64_t base = a.t.rep_off[r];
  const int32_t n = int32_t(a.t.rep_off[r + 1] - base);
  RepState *const rs = reinterpret_cast<RepState *>(a.state + a.L.reps) + r;
  int64_t *const u_all = reinterpret_cast<int64_t *>(a.state + a.L.u_all) + int64_t(r) * U;

  // ---- scalar state of the replica
  int32_t s = int32_t(uni64(rs->s)), nxt = int32_t(uni64(rs->nxt));
  int32_t low = int32_t(uni64(rs->low)), seq = int32_t(uni64(rs->seq));
  int64_t debt = uni64(rs->debt), backlog = uni64(rs->backlog), gap = uni64(rs->gap);
  int64_t last_exit_u = uni64(rs->last_exit_u);
  int32_t last_exit = uni(rs->last_exit);
  const int64_t s_end = resumed ? uni64(rs->s_end) : a.n_steps < 0 ? INT64_MAX : int64_t(s) + a.n_steps;
  const int64_t C = a.cap, theta = a.theta < -1 ? -1 : a.theta;  // (-1: always overloaded)
  const double tau_inv = 1.0 / double(a.tau);
  // stopped inside a step (only the global-memory kernel resumes that), or too many records
  // for 32-bit byte offsets
  if (uni(rs->mid) || n >= (1 << 29)) {
    if (lane == 0) {
      rs->overflow = 1;
      rs->s_end = s_end;
    }
    return;
  }
  if (ulds)
    for (int32_t k = lane; k < U; k += 64) u_lds[k] = u_all[k];
  s_xu[lane] = -1;
  s_free[lane] = lane;
  if (lane < 3) st8[M + lane] = lane == kStAdm ? 1 : lane == kStBlk ? 2 : 0;
  __syncthreads();

  auto set_u = [&](int32_t k, int64_t v) {
    if (ulds)
      ((__attribute__((address_space(3))) int64_t *)u_lds)[k] = v;
    else
      ((__attribute__((address_space(1))) int64_t *)u_all)[k] = v;
  };

  // ---- the pool: one queued call per lane
  uint32_t kh = 0xffffffffu, kl = 0xffffffffu;  // key: first call << 63 | counter before it
  uint32_t ua = 0xffffffffu;                    // user << 6 | position among its pooled calls
  int32_t qx = 0, q_rec = 0, q_succ = -1;       // slot, record, next call
  uint32_t q_lo = 0, q_hi = 0;                  // cost << 24 | tokens
  uint64_t occ = 0;                             // occupied lanes
  uint32_t rank = 0, pre = 0;                   // place in the order, tokens ranked before
  bool dirty = false;                           // calls were added: rank, pre to be taken again
  uint64_t nearm = 0, far = ~uint64_t(0);       // the calls ranked, the key they stay below
  int32_t nX = 0;                               // backlogged users (slots)
  int32_t n_adm = 0;                            // admissions staged in s_adm
  int32_t sp_total = 0;                         // spilled calls
  int64_t minX = 0;
  int32_t code = 0;
  bool overflow = false;

  // ---- window of upcoming records, one per lane
  int32_t wbase = nxt - 64, cache_lo = nxt;  // (no window yet)
  const int32_t cache_from = nxt;
  int32_t w_step = INT32_MAX, w_user = -1, w_why = 0, w_head = -1, w_prev = -1, w_succ = -1;
  int32_t w_pst = 0, w_hst = 0;  // the previous and first calls' entries in st8
  uint32_t w_lo = 0, w_hi = 0, w_tsum = 0;  // w_tsum: tokens of the window up to the lane
  uint64_t w_first = 0, w_over = 0, w_big = 0, w_old = 0;  // masks of window lanes: first
  // calls, those over a limit, those that do not fit a packed request, later calls whose
  // previous call is older than the cache and was undecided when the window was loaded
  int32_t w_rep = lane;  // the lane that stands for the window lanes of this user
  uint64_t w_gm = 0;     // the window lanes of this lane's user
  int32_t w_ps = -1;     // the last one before this lane
  int32_t o_st = 0;
  int64_t o_coa = 0;
  struct RawRec {
    int64_t ts, cst;
    int32_t usr, call, hd, pv, li, lo, ls, why, sc;
  };
  RawRec pf{0, 0, -1, 0, -1, -1, 0, 0, 0, 0, -1};
  int32_t pf_at = -1;  // the window base pf was loaded for

  // Data of an arrived record read from the inputs (when it is no longer cached).
  auto load_rec = [&](int32_t i, int32_t &sc, uint32_t &lo, uint32_t &hi) {
    const int64_t g = base + i;
    const int32_t *len_sys = KARG(t.len_sys);
    const int32_t tok = KARG(t.len_in)[g] + KARG(t.len_out)[g] + (len_sys ? len_sys[g] : 0);
    const uint64_t pk = (uint64_t(KARG(cost)[g]) << 24) | uint32_t(tok);
    sc = LINKS ? uni(STATE(const int32_t, succ)[g]) : -1;
    lo = uint32_t(uni(int32_t(uint32_t(pk))));
    hi = uint32_t(uni(int32_t(uint32_t(pk >> 32))));
  };
  auto fetch_rec = [&](int32_t i, int32_t &sc, uint32_t &lo, uint32_t &hi) {
    if (i >= cache_lo) {
      const Ent e = cache[i & (M - 1)];
      sc = uni(e.succ);
      lo = uint32_t(uni(int32_t(e.lo)));
      hi = uint32_t(uni(int32_t(e.hi)));
    } else {
      load_rec(i, sc, lo, hi);
    }
  };

  // The staged admissions' fates, statuses and steps.
  auto flush_admitted = [&]() {
    char *const o_fate = reinterpret_cast<char *>(STATE(int8_t, fate) + base);
    char *const o_status = reinterpret_cast<char *>(KARG(status) + base);
    char *const o_step = reinterpret_cast<char *>(KARG(admit_step) + base);
    for (int32_t i = lane; i < n_adm; i += 64) {
      const uint2 e = s_adm[i];
      o_fate[e.x] = 0;
      o_status[e.x] = 0;
      *reinterpret_cast<int32_t *>(o_step + (e.x << 2)) = int32_t(e.y);
    }
    n_adm = 0;
  };
  // Throttled arrivals and the counters on arrival of the records before nxt.
  auto flush_window = [&](int32_t wb) {
    const int32_t done = nxt - wb;
    int64_t *const coa = KARG(counter_on_arrival);
    if (lane < done) {
      const int64_t g = base + wb + lane;
      if (o_st > 0) {
        int32_t *const as = KARG(admit_seq);
        int64_t *const ca = KARG(counter_after);
        STATE(int8_t, fate)[g] = int8_t(o_st);
        KARG(status)[g] = int8_t(o_st);
        KARG(admit_step)[g] = -1;
        if (as) as[g] = -1;
        if (ca) ca[g] = -1;
      }
      if (coa) coa[g] = o_coa;
    }
    o_st = 0;
  };

  // The lane standing for each window user and the lanes of the same user, through a table
  // indexed by the user's low bits (a user that lost its entry to another sends the window
  // to the matching bit by bit), then the slots of the users that are backlogged.
  auto match_window = [&](int32_t &xr, int32_t &xuser) {
    const bool wv = w_user >= 0;
    const uint64_t wvm = bal(wv);
    const int32_t hw = w_user & (tab - 1);
    if (wv) u_rep[hw] = uint8_t(lane);
    wave_fence();
    xuser = s_xu[lane];
    const int32_t rr = wv ? int32_t(u_rep[hw]) & 63 : lane;
    const int32_t rx = int32_t(u_rep[xuser & (tab - 1)]) & 63;
    const int32_t rr_user = __builtin_amdgcn_ds_bpermute(rr << 2, w_user);
    const int32_t rx_user = __builtin_amdgcn_ds_bpermute(rx << 2, w_user);
    uint64_t g = wvm;
    xr = -1;
    if (!bal(wv && rr_user != w_user)) {
#pragma unroll
      for (int b = 0; b < 6; ++b) {
        const uint64_t W = bal(((rr >> b) & 1) != 0);
        g &= ((rr >> b) & 1) ? W : ~W;
      }
      w_rep = rr;
      if (xuser >= 0 && rx_user == xuser) xr = rx;
    } else {
      for (int b = 0; b < ubits; ++b) {
        const bool wb = (uint32_t(w_user) >> b) & 1u;
        const uint64_t W = bal(wb);
        g &= wb ? W : ~W;
      }
      w_rep = wv ? __ffsll((long long)g) - 1 : lane;
      for (uint64_t m = bal(xuser >= 0); m; m &= m - 1) {
        const int j = ff1(m);
        const uint64_t f = bal(w_user == rdl(xuser, j));
        if (lane == j && f) xr = ff1(f);
      }
    }
    w_gm = wv ? g : 0;
    w_ps = (w_gm & lt) ? 63 - __clzll((long long)(w_gm & lt)) : -1;
  };

  // The window that starts at old (if any) is done: its throttled arrivals and the admissions
  // since are written after the new window's dependent loads (before them when those read
  // fates), so that no wait for a load also waits for these stores.
  auto load_window = [&](int32_t old) {
    wave_fence();
    const int32_t i = wbase + lane;
    struct {
      const int64_t *ts;
      const int32_t *user, *call, *head, *prev, *len_in, *len_sys, *len_out;
    } T = {KARG(t.ts),   KARG(t.user),   KARG(t.call),    KARG(t.head),
           KARG(t.prev), KARG(t.len_in), KARG(t.len_sys), KARG(t.len_out)};
    const int64_t *const costp = KARG(cost);
    const uint8_t *const reason = KARG(reason);
    const int64_t tau = KARG(tau);
    char *const st = KARG(state);
    const size_t o_succ = KARG(L.succ), o_fate = KARG(L.fate);
    // record ii's fields, raw (no arithmetic on a loaded value, so that nothing waits);
    // lanes past the last record read the last record, absent arrays a stand-in
    auto fetch = [&](int32_t ii, RawRec &f) {
      const int64_t g = base + (ii < n ? ii : n - 1);
      f.call = LINKS ? T.call[g] : 0;
      f.usr = T.user[g];
      f.ts = T.ts[g];
      f.hd = LINKS ? T.head[g] : ii;
      f.pv = LINKS ? T.prev[g] : -1;
      f.li = T.len_in[g];
      f.lo = T.len_out[g];
      f.ls = (T.len_sys ? T.len_sys : T.len_in)[g];
      f.cst = costp[g];
      f.why = (reason ? reason : reinterpret_cast<const uint8_t *>(T.len_in))[g];
      f.sc = LINKS ? reinterpret_cast<const int32_t *>(st + o_succ)[g] : -1;
    };
    if (pf_at != wbase) fetch(i, pf);  // (the first window of the call)
    const RawRec c = pf;
    const bool in = i < n;
    int64_t c_u = ulds ? u_lds[c.usr] : ld_fresh(u_all + c.usr);
    const int32_t lo_ = wbase + 64 - M;
    cache_lo = lo_ > cache_from ? lo_ : cache_from;
    int8_t pf_fate = -1, hf_fate = -1;
    const bool aged = LINKS && in && c.call > 0 && (c.pv < cache_lo || c.hd < cache_lo);
    const bool early = LINKS && bal(aged) != 0;
    if (early) {
      if (old >= cache_from) flush_window(old);
      flush_admitted();
    }
    if (aged) {
      const int8_t *const fate = reinterpret_cast<const int8_t *>(st + o_fate) + base;
      pf_fate = ld_fresh(fate + c.pv);
      hf_fate = ld_fresh(fate + c.hd);
    }
    const int32_t tok = c.li + c.lo + (T.len_sys ? c.ls : 0);
    const int32_t why = reason ? c.why : 0;
    w_step = in ? step_of(c.ts, tau, tau_inv) : INT32_MAX;
    w_user = in ? c.usr : -1;
    w_why = why;
    w_head = in ? c.hd : -1;
    w_prev = in ? c.pv : -1;
    w_succ = in ? c.sc : -1;
    const uint64_t pk = (uint64_t(c.cst) << 24) | uint32_t(tok);
    w_lo = uint32_t(pk);
    w_hi = uint32_t(pk >> 32);
    w_tsum = wave_incl_scan32(in ? uint32_t(tok) : 0u);
    const bool first = c.call == 0;
    w_first = bal(in && first);
    w_over = bal(in && first && why != 0);
    w_big = bal(in && !fits_packed(c.cst, tok));
    if (LINKS) {
      const bool later = in && !first;
      w_pst = M + kStNone;
      w_hst = M + kStNone;
      if (later) {
        w_pst = c.pv >= cache_lo ? (c.pv & (M - 1)) : M + (pf_fate == 0 ? kStAdm : kStNone);
        w_hst = c.hd >= cache_lo ? (c.hd & (M - 1))
                                 : M + ((hf_fate == 1 || hf_fate == 2) ? kStBlk : kStNone);
      }
      w_old = bal(later && c.pv < cache_lo && pf_fate != 0);
      if (in) st8[i & (M - 1)] = 0;  // undecided
    }
    if (in) cache[i & (M - 1)] = mk_ent(i, c.sc, w_lo, w_hi);
    int32_t xr, xuser;
    match_window(xr, xuser);  // (while the counters are on their way)
    // every loaded value is in its register from here on: no later wait on HBM
    __asm__ volatile("" ::"v"(w_step), "v"(w_user), "v"(w_why), "v"(w_head), "v"(w_prev),
                     "v"(w_succ), "v"(w_lo), "v"(w_hi), "v"(c_u));
    if (!early) {
      if (old >= cache_from) flush_window(old);
      flush_admitted();
    }
    // the next window's records, into the registers this window's just left
    pf_at = wbase + 64;
    fetch(pf_at + lane, pf);
    s_win[lane] = make_uint4(uint32_t(uint64_t(c_u)), uint32_t(uint64_t(c_u) >> 32), 0xffffffffu, 0u);
    wave_fence();
    if (xuser >= 0) {
      s_slot[lane].num = (s_slot[lane].num & (kWinOne - 1)) | uint32_t(xr + 1) * kWinOne;
      if (xr >= 0) s_win[xr].z = uint32_t(lane);
    }
    wave_fence();
  };

  // Ranks of the pooled calls.  With more than kNearMin of them, those from key `far` on are
  // left out (nearm: the calls ranked) while at least a few are below it: a step admits a
  // handful, and `far` is set from a ranking of all to the key of rank kNearRank.
  auto take_ranks = [&]() {
    const uint32_t tok = q_lo & uint32_t(kTokMask);
    const uint64_t key = (uint64_t(kh) << 32) | kl;
    nearm = occ;
    const bool many = LINKS && __popcll(occ) > kNearMin;  // (without interactions queues stay small)
    if (many) {
      const uint64_t nm = occ & bal(key < far);
      if (__popcll(nm) >= kNearLeast) nearm = nm;
    }
    // the order as one word: first call << 63 | counter - least << ksh | user << 6 | position
    const uint64_t rel = (key & ~(uint64_t(kPTier1) << 32)) - uint64_t(minX);
    const bool wide = (nearm & bal((rel >> (63 - ksh)) != 0)) != 0;
    if (FS_RARE(wide || backlog >= (int64_t(1) << 26))) {
      pool_rank_wide(key, ua, tok, nearm, rank, pre);
    } else {
      const bool nr = in_mask(nearm);
      const uint64_t q = (rel << ksh) | (uint64_t(kh & kPTier1) << 32) | ua;
      const uint64_t p = nr ? q : ~uint64_t(0);
      uint32_t sh = uint32_t(p >> 32), sl = uint32_t(p), sa = nr ? tok | (1u << 26) : 0u;
      int32_t top = 64 - __builtin_clzll(nearm);
      if (LINKS && nearm != occ) {
        // the calls ranked packed into the lowest lanes, the others (which count for nothing)
        // above them
        const int32_t nn = __popcll(nearm);
        const int32_t to = (nr ? below(nearm) : nn + below(~nearm)) << 2;
        sh = uint32_t(__builtin_amdgcn_ds_permute(to, int(sh)));
        sl = uint32_t(__builtin_amdgcn_ds_permute(to, int(sl)));
        sa = uint32_t(__builtin_amdgcn_ds_permute(to, int(sa)));
        top = nn;
      }
      const uint32_t rp = pool_rank(p, sh, sl, sa, top);
      rank = rp >> 26;
      pre = rp & ((1u << 26) - 1);
    }
    if (many) {
      if (nearm == occ) {
        const int l = first_of(occ & bal(rank == uint32_t(kNearRank)));
        far = (uint64_t(rdlu(kh, l)) << 32) | rdlu(kl, l);
      } else {
        rank = in_mask(nearm) ? rank : 0x7fffffffu;
        pre = in_mask(nearm) ? pre : 0xffffffffu;
      }
    }
    dirty = false;
  };
  // Lane l was just added to calls whose ranks are known: its rank, and theirs after it (two
  // ballots and two lane reads, against a ranking of all of them).
  auto rank_one = [&](int l) {
    const uint64_t key = (uint64_t(kh) << 32) | kl;
    const uint64_t kj = uint64_t(rdl64(int64_t(key), l));
    const uint32_t uj = rdlu(ua, l), tok = q_lo & uint32_t(kTokMask), tj = rdlu(tok, l);
    if (kj >= far) {  // not among the ranked
      if (lane == l) {
        rank = 0x7fffffffu;
        pre = 0xffffffffu;
      }
      return;
    }
    const uint64_t gm = nearm & bal(key > kj || (key == kj && ua > uj));
    const uint32_t c = uint32_t(__popcll(nearm & ~gm));
    const uint32_t pj = gm ? rdlu(pre, first_of(gm & bal(rank == c)))
                           : (c ? rdlu(pre + tok, first_of(nearm & bal(rank == c - 1))) : 0u);
    const bool gt = in_mask(gm);
    rank = lane == l ? c : (gt ? rank + 1 : rank);
    pre = lane == l ? pj : (gt ? pre + tj : pre);
    nearm |= uint64_t(1) << l;
  };
  // A free pool lane takes call (rec, sc, lo, hi) of slot x with key k at position ah.
  auto place = [&](int32_t x, int32_t user, uint64_t k, int32_t ah, int32_t rec, int32_t sc,
                   uint32_t lo, uint32_t hi) -> int {
    const int l = first_of(~occ);
    occ |= uint64_t(1) << l;
    if (lane == l) {
      kh = uint32_t(k >> 32);
      kl = uint32_t(k);
      ua = (uint32_t(user) << kAheadBits) | uint32_t(ah);
      qx = x;
      q_rec = rec;
      q_succ = sc;
      q_lo = lo;
      q_hi = hi;
    }
    return l;
  };
  // First call rec joins the end of slot x's pooled calls.
  auto append = [&](int32_t x, int32_t user, int32_t rec, int32_t sc, uint32_t lo, uint32_t hi) {
    wave_fence();
    const SlotRec e = s_slot[x];
    const uint64_t pe = uint64_t(uni64(int64_t((uint64_t(e.phi) << 32) | e.plo)));
    const uint32_t num = uint32_t(uni(int32_t(e.num)));
    place(x, user, pe | (uint64_t(1) << 63), int32_t(num & kNumMask), rec, sc, lo, hi);
    const uint64_t v = pe + (((uint64_t(hi) << 32) | lo) >> 24);
    if (lane == 0) {
      s_slot[x].plo = uint32_t(v);
      s_slot[x].phi = uint32_t(v >> 32);
      s_slot[x].num = num + 1;
    }
    wave_fence();
    dirty = true;
  };
  // Slot x gains the ready later call rec (a free lane exists): it goes between the user's
  // ready calls by record; the user's calls after it move behind by its cost.
  auto ready_insert = [&](int32_t x, int32_t rec, int32_t sc, uint32_t lo, uint32_t hi) {
    wave_fence();
    const uint64_t cst = ((uint64_t(hi) << 32) | lo) >> 24;
    const SlotRec e = s_slot[x];
    const int32_t user = uni(s_xu[x]);
    const uint32_t num = uint32_t(uni(int32_t(e.num)));
    const uint64_t pe = uint64_t(uni64(int64_t((uint64_t(e.phi) << 32) | e.plo)));
    const bool aft = ((occ >> lane) & 1) && qx == x && ((kh & kPTier1) || q_rec > rec);
    const uint64_t am = bal(aft);
    const int32_t ah = int32_t(num & kNumMask) - __popcll(am);
    uint64_t k = pe;
    if (am) {
      const int l = ff1(bal(aft && int32_t(ua & 63u) == ah));
      k = (uint64_t(rdlu(kh, l) & ~kPTier1) << 32) | rdlu(kl, l);
      if (aft) {
        const uint64_t v = ((uint64_t(kh) << 32) | kl) + cst;
        kh = uint32_t(v >> 32);
        kl = uint32_t(v);
        ++ua;
      }
    }
    const uint64_t v = pe + cst;
    if (lane == 0) {
      s_slot[x].plo = uint32_t(v);
      s_slot[x].phi = uint32_t(v >> 32);
      s_slot[x].num = num + 1 + kRdyOne;
    }
    wave_fence();
    const bool all = nearm == occ;
    const int l = place(x, user, k, ah, rec, sc, lo, hi);
    if (am || dirty || !LINKS) {
      dirty = true;
    } else {
      if (all) far = ~uint64_t(0);
      rank_one(l);
    }
  };
  // The spill list of a user: its first calls beyond the pool, in order, in the user's
  // segment of the state buffer (a place per request of the user, used as a ring).  Its
  // segment and places, read when the list of a slot without one starts.
  auto seg_of = [&](int32_t user, bool has, int32_t x, uint32_t &sb, uint32_t &cap, uint32_t &head) {
    if (has) {
      sb = s_seg[x];
      cap = s_cap[x];
      head = s_sph[x];
    } else {
      const uint32_t *const ss = STATE(const uint32_t, seg_start) + int64_t(r) * U + user;
      sb = ss[0];
      cap = ss[1] - sb;
      head = 0;
      s_seg[x] = sb;
      s_cap[x] = cap;
      s_sph[x] = 0;
    }
  };
  auto place_of = [&](uint32_t at, uint32_t cap) -> uint32_t { return at >= cap ? at - cap : at; };
  auto spill_append = [&](int32_t x, int32_t user, int32_t rec, int32_t sc, uint32_t lo, uint32_t hi) {
    wave_fence();
    const uint32_t e = uint32_t(uni(int32_t(s_slot[x].spilled)));
    if (lane == 0) {
      uint32_t sb, cap, head;
      seg_of(user, e != 0, x, sb, cap, head);
      STATE(Ent, seg_pk)[int64_t(sb) + place_of(head + e, cap)] = mk_ent(rec, sc, lo, hi);
      s_slot[x].spilled = e + 1;
    }
    wave_fence();
    ++sp_total;
  };
  // Up to 16 calls of slot x's spill list come back to the pool, in order: one load.
  auto spill_refill = [&](int32_t x) {
    wave_fence();
    const SlotRec e = s_slot[x];
    const uint32_t spilled = uint32_t(uni(int32_t(e.spilled))), num = uint32_t(uni(int32_t(e.num)));
    const uint32_t sb = s_seg[x], cap = s_cap[x], head = s_sph[x];
    const int32_t user = uni(s_xu[x]);
    uint32_t m = spilled;
    if (m > 16) m = 16;
    if (__popcll(occ) > kPoolRoom && m > uint32_t(kPoolShare)) m = kPoolShare;
    if (m > uint32_t(64 - __popcll(occ))) m = uint32_t(64 - __popcll(occ));
    if (m == 0) return;
    const bool mine = uint32_t(lane) < m;
    Ent v = mk_ent(-1, -1, 0, 0);
    if (mine) v = STATE(Ent, seg_pk)[int64_t(sb) + place_of(head + uint32_t(lane), cap)];
    // the counter before each: the costs of those before it, over the first 16 lanes
    const uint64_t cst = ((uint64_t(v.hi) << 32) | v.lo) >> 24;
    uint64_t sum = cst;
#pragma unroll
    for (int d = 1; d < 16; d <<= 1) {
      const int src = (lane >= d ? lane - d : lane) << 2;
      const uint32_t lo = uint32_t(__builtin_amdgcn_ds_bpermute(src, int(uint32_t(sum))));
      const uint32_t hi = uint32_t(__builtin_amdgcn_ds_bpermute(src, int(uint32_t(sum >> 32))));
      sum += lane >= d ? (uint64_t(hi) << 32) | lo : 0;
    }
    const uint64_t pe = (uint64_t(e.phi) << 32) | e.plo;
    const uint64_t k = pe + sum - cst;
    if (mine) {
      s_stage[2 * lane] = make_uint4(uint32_t(k >> 32) | kPTier1, uint32_t(k),
                                     (uint32_t(user) << kAheadBits) | ((num & kNumMask) + uint32_t(lane)),
                                     uint32_t(x));
      s_stage[2 * lane + 1] = make_uint4(uint32_t(v.rec), uint32_t(v.succ), v.lo, v.hi);
    }
    wave_fence();
    const int32_t fi = below(~occ);
    const uint64_t tm = bal(fi < int32_t(m)) & ~occ;
    if (in_mask(tm)) {
      const uint4 ea = s_stage[2 * fi], eb = s_stage[2 * fi + 1];
      kh = ea.x;
      kl = ea.y;
      ua = ea.z;
      qx = int32_t(ea.w);
      q_rec = int32_t(eb.x);
      q_succ = int32_t(eb.y);
      q_lo = eb.z;
      q_hi = eb.w;
    }
    occ |= tm;
    if (uint32_t(lane) == m - 1) {
      const uint64_t v1 = pe + sum;
      s_slot[x] = SlotRec{uint32_t(v1), uint32_t(v1 >> 32), num + m, spilled - m};
      s_sph[x] = place_of(head + m, cap);
    }
    wave_fence();
    sp_total -= int32_t(m);
    dirty = true;
  };
  // The last pooled first call of every user with two or more pooled calls goes to the
  // front of its user's spill list.  Returns the number of lanes freed.
  auto evict = [&]() -> int32_t {
    wave_fence();
    const bool oc = (occ >> lane) & 1;
    const int32_t ah = int32_t(ua & 63u);
    const SlotRec e = s_slot[oc ? qx : 64];
    const bool ev = oc && (kh & kPTier1) && ah > 0 && ah == int32_t(e.num & kNumMask) - 1;
    const uint64_t em = bal(ev);
    if (!em) return 0;
    if (ev) {
      uint32_t sb, cap, head;
      seg_of(int32_t(ua >> kAheadBits), e.spilled != 0, qx, sb, cap, head);
      head = head ? head - 1 : cap - 1;
      STATE(Ent, seg_pk)[int64_t(sb) + head] = mk_ent(q_rec, q_succ, q_lo, q_hi);
      s_sph[qx] = head;
      s_slot[qx] = SlotRec{kl, kh & ~kPTier1, e.num - 1, e.spilled + 1};
      kh = kl = ua = 0xffffffffu;
    }
    wave_fence();
    occ &= ~em;
    sp_total += __popcll(em);
    dirty = true;
    return __popcll(em);
  };

  // The arrivals in window lanes [j0, j1) (all of the current step), in stream order.
  // The overload test of each needs the tokens queued before it: the queue only grows
  // during the arrivals, so the first that finds it above the threshold is found from a
  // prefix sum taken as if none were throttled, and every later one finds it above too.
  // Returns false, having changed nothing, when the pool has no room for them all.
  auto arrive = [&](int32_t j0, int32_t j1) -> bool {
    const uint64_t inbm = (~uint64_t(0) << j0) & (~uint64_t(0) >> (64 - j1));
    const bool inb = in_mask(inbm);
    const uint32_t tok = w_lo & uint32_t(kTokMask);
    const uint64_t cst = ((uint64_t(w_hi) << 32) | w_lo) >> 24;
    const uint4 we = s_win[w_rep];
    uint8_t ps = 0, hs = 0;
    if (LINKS) {
      ps = st8[w_pst];
      hs = st8[w_hst];
    }
    const int64_t u0 = int64_t((uint64_t(we.y) << 32) | we.x);
    int32_t x = int32_t(we.z);  // the user's slot, -1 outside Q
    uint64_t padm = LINKS ? bal(ps == 1) & inbm : 0;
    const uint64_t hblk = LINKS ? bal(hs == 2) & inbm : 0;
    if (LINKS && FS_RARE((w_old & inbm) != 0)) {
      flush_admitted();
      const int8_t *const fate = STATE(const int8_t, fate) + base;
      bool pa = false;
      if (in_mask(w_old & inbm)) pa = ld_fresh(fate + w_prev) == 0;
      padm |= bal(pa);
    }
    uint32_t total = rdlu(w_tsum, j1 - 1) - (j0 > 0 ? rdlu(w_tsum, j0 - 1) : 0u);
    uint64_t blk = hblk, bfm = 0;  // throttled arrivals, the first calls among them
    if ((w_over & inbm) != 0 && less_s(theta, backlog + int64_t(total))) {
      const uint32_t c0 = in_mask(inbm & ~hblk) ? tok : 0u;
      const uint32_t excl = wave_incl_scan32(c0) - c0;
      const int64_t thr = theta - backlog;  // overloaded at a lane iff excl > thr
      const uint32_t th32 = thr >= int64_t(INT32_MAX) ? 0x7fffffffu : uint32_t(thr);
      // first calls throttled: over a limit while the system is overloaded
      bfm = w_over & inbm & (thr < 0 ? ~uint64_t(0) : bal(excl > th32));
      blk |= bfm;
      if (LINKS && bfm) {  // later calls of an interaction throttled in this batch
        const int32_t hl = w_head - wbase;
        const bool hin = hl >= j0 && hl < j1;
        const int src = __builtin_amdgcn_ds_bpermute((hin ? hl : lane) << 2, in_mask(bfm) ? 1 : 0);
        blk |= bal(hin && src != 0) & inbm & ~w_first;
      }
    }
    const uint64_t ub = inbm & ~blk;
    const uint64_t F = ub & w_first, rdym = LINKS ? ub & padm : 0;
    const int32_t need = __popcll(F | rdym), held = __popcll(occ);
    // room: a lane for every new call, a slot for every new user
    if (FS_RARE(__popcll(ub) > 64 - nX || need > 64 - held || (ub & w_big) != 0)) return false;
    if (blk) {
      if (in_mask(blk)) o_st = in_mask(bfm) ? w_why : 3;
      if (LINKS && in_mask(blk)) st8[(wbase + lane) & (M - 1)] = 2;
      total = wave_sum32(in_mask(ub) ? tok : 0u);
    }
    backlog += int64_t(total);
    // a user outside Q is lifted to the least counter in Q; with Q empty, to the last
    // exit's counter, until the first call that joins sets the least counter
    int64_t lift = minX;
    if (nX == 0) {
      const int64_t l0 = last_exit >= 0 ? last_exit_u : 0;
      lift = l0;
      if (ub) {
        const int f = first_of(ub);
        const int64_t uf = rdl64(u0, f);
        minX = less_s(l0, uf) ? uf : l0;
        lift = in_mask(~uint64_t(0) << f) ? minX : l0;
      }
    }
    const int64_t lifted = u0 > lift ? u0 : lift;
    if (want_coa) {  // (an optional output)
      const int64_t us = int64_t(s_uc[x >= 0 ? x : 0]);
      if (inb) o_coa = x >= 0 ? us : lifted;
    }
    const uint64_t same = w_gm & inbm;
    if (blk) {
      // users that stay outside Q (all of their arrivals throttled): the lifted counter
      const bool ou = in_mask(blk) && x < 0 && (same & ub) == 0 && (same >> lane) == 1;
      if (ou && lifted != u0) {
        set_u(w_user, lifted);
        s_win[w_rep].x = uint32_t(uint64_t(lifted));
        s_win[w_rep].y = uint32_t(uint64_t(lifted) >> 32);
      }
      if (!ub) return true;
    }
    // does some user have two arrivals here?  (their calls are then chained below)
    const bool dup = (bal(w_ps >= j0) & inbm) != 0;
    // users joining Q, one each at their first unthrottled arrival
    uint64_t jm = bal(x < 0) & ub;
    if (dup) jm &= bal((same & ub & lt) == 0);
    if (jm) {
      const bool jl = in_mask(jm);
      const int32_t xs = s_free[63 - nX - (jl ? below(jm) : 0)];
      nX += __popcll(jm);
      const int32_t xd = jl ? xs : 64;
      s_xu[xd] = w_user;
      s_slot[xd] = SlotRec{uint32_t(uint64_t(lifted)), uint32_t(uint64_t(lifted) >> 32),
                           uint32_t(w_rep + 1) * kWinOne, 0u};
      s_win[jl ? w_rep : 64].z = uint32_t(xs);
      if (want_coa) s_uc[xd] = uint64_t(lifted);
      x = jl ? xs : x;
      if (dup) {
        wave_fence();
        x = int32_t(s_win[w_rep].z);
      }
    }
    x = in_mask(ub) ? x : 64;
    wave_fence();
    const SlotRec e = s_slot[x];
    const uint64_t pe = (uint64_t(e.phi) << 32) | e.plo;
    const int32_t cn = int32_t(e.num & kNumMask);
    // ready later calls go before the user's first calls: at the end of its pooled calls
    // when none of those is a first call, else one at a time below
    uint64_t slow = 0;
    if (LINKS && rdym) {
      slow = bal(int32_t(ready_of(e.num)) != cn);
      if (dup) slow |= bal((same & F & lt) != 0);
      slow &= rdym;
    }
    uint64_t app = (F | rdym) & ~slow;  // calls appended to their users' pooled calls
    // a user's first calls stay together in order: behind spilled ones, or beyond the
    // share of the pool a user may hold while it is filling up, a call is spilled
    if (FS_RARE(sp_total > 0 || held + need > kPoolRoom)) {
      const int32_t most = held + need <= kPoolRoom ? kPoolRoom : kPoolShare;
      const uint64_t sp = F & bal(e.spilled != 0 || cn + __popcll(same & F & lt) >= most);
      if (sp) {
        app &= ~sp;
        const uint64_t sm = same & sp;
        if (in_mask(sp)) {
          uint32_t sb, cap, head;
          seg_of(w_user, e.spilled != 0, x, sb, cap, head);
          const uint32_t i = uint32_t(__popcll(sm & lt)), c = e.spilled;
          STATE(Ent, seg_pk)[int64_t(sb) + place_of(head + c + i, cap)] = mk_ent(wbase + lane, w_succ, w_lo, w_hi);
          if ((sm >> lane) == 1) s_slot[x].spilled = c + i + 1;
        }
        wave_fence();
        sp_total += __popcll(sp);
      }
    }
    const bool isA = in_mask(app), isR = LINKS && in_mask(rdym);
    uint64_t k = pe;  // the counter before this call: after the user's earlier ones
    uint32_t num = e.num;
    uint64_t last = app;
    if (dup) {
      const uint64_t sa = same & app;
      const int32_t t = isA ? __popcll(sa & lt) : 0;
      const int p = t > 0 ? 63 - __clzll((long long)(sa & lt)) : lane;
      for (int32_t q = 1; bal(t >= q); ++q) {
        const uint64_t v = k + cst;
        const uint32_t lo = uint32_t(__builtin_amdgcn_ds_bpermute(p << 2, int(uint32_t(v))));
        const uint32_t hi = uint32_t(__builtin_amdgcn_ds_bpermute(p << 2, int(uint32_t(v >> 32))));
        k = t == q ? (uint64_t(hi) << 32) | lo : k;
      }
      num += uint32_t(t);
      if (LINKS) num += kRdyOne * uint32_t(__popcll(sa & rdym & lt));
      last &= bal((sa >> lane) == 1);
    }
    const uint64_t k1 = k + cst;
    {  // the user's record after its last call appended here (the spill field stays)
      SlotRec *const d = s_slot + (in_mask(last) ? x : 64);
      d->plo = uint32_t(k1);
      d->phi = uint32_t(k1 >> 32);
      d->num = num + 1 + (isR ? kRdyOne : 0u);
    }
    // the new calls take the lowest free lanes
    if (app) {
      const int32_t i = isA ? below(app) : 64;
      s_stage[2 * i] = make_uint4(uint32_t(k >> 32) | (isR ? 0u : kPTier1), uint32_t(k),
                                  (uint32_t(w_user) << kAheadBits) | (num & kNumMask), uint32_t(x));
      s_stage[2 * i + 1] = make_uint4(uint32_t(wbase + lane), uint32_t(w_succ), w_lo, w_hi);
      wave_fence();
      const int32_t fi = below(~occ);
      const uint64_t tm = bal(fi < __popcll(app)) & ~occ;
      const bool tk = in_mask(tm);
      const uint4 ea = s_stage[2 * fi], eb = s_stage[2 * fi + 1];
      kh = tk ? ea.x : kh;
      kl = tk ? ea.y : kl;
      ua = tk ? ea.z : ua;
      qx = tk ? int32_t(ea.w) : qx;
      q_rec = tk ? int32_t(eb.x) : q_rec;
      if (LINKS) q_succ = tk ? int32_t(eb.y) : q_succ;
      q_lo = tk ? eb.z : q_lo;
      q_hi = tk ? eb.w : q_hi;
      occ |= tm;
      dirty = true;
    }
    if (LINKS)
      for (; FS_RARE(slow != 0); slow &= slow - 1) {
        const int l = first_of(slow);
        ready_insert(rdl(x, l), wbase + l, rdl(w_succ, l), rdlu(w_lo, l), rdlu(w_hi, l));
      }
    return true;
  };

  // ---- rebuild the queue left by a previous call: arrived records still undecided
  for (int32_t b0 = low; b0 < nxt && !overflow; b0 += 64) {
    const int8_t *const fate = STATE(const int8_t, fate) + base;
    const int32_t i = b0 + lane;
    const bool q = i < nxt && ld_fresh(fate + i) == -1;
    uint64_t m = bal(q);
    if (!m) continue;
    // the queued records' fields, lane-parallel
    const int64_t g = base + (q ? i : b0);
    const int32_t *const len_sys = KARG(t.len_sys);
    const int32_t *const callp = KARG(t.call);
    const int32_t ku = KARG(t.user)[g];
    const int32_t tok = KARG(t.len_in)[g] + KARG(t.len_out)[g] + (len_sys ? len_sys[g] : 0);
    const int64_t cst = KARG(cost)[g];
    const int32_t call = LINKS ? callp[g] : 0;
    const int32_t pv = LINKS ? KARG(t.prev)[g] : -1;
    const int32_t scv = LINKS ? STATE(const int32_t, succ)[g] : -1;
    const int64_t uv = ulds ? u_lds[ku] : ld_fresh(u_all + ku);
    const bool padm = q && call > 0 && ld_fresh(fate + (pv >= 0 ? pv : 0)) == 0;
    const uint64_t pk = (uint64_t(cst) << 24) | uint32_t(tok);
    const uint64_t bigm = bal(q && !fits_packed(cst, tok));
    const uint64_t padmm = bal(padm), laterm = bal(call > 0);
    if (bigm) overflow = true;
    while (m && !overflow) {
      const int l = ff1(m);
      m &= m - 1;
      const int32_t rec = b0 + l, k = rdl(ku, l), sc = rdl(scv, l);
      const uint32_t lo = rdlu(uint32_t(pk), l), hi = rdlu(uint32_t(pk >> 32), l);
      wave_fence();
      const int32_t xuser = s_xu[lane];
      const uint64_t fm = bal(xuser == k);
      int32_t x = ff1(fm);
      if (!fm) {
        if (nX == 64) {
          overflow = true;
          break;
        }
        x = uni(s_free[63 - nX]);
        const int64_t uk = rdl64(uv, l);
        if (lane == 0) {
          s_xu[x] = k;
          s_slot[x] = SlotRec{uint32_t(uint64_t(uk)), uint32_t(uint64_t(uk) >> 32), 0u, 0u};
          s_uc[x] = uint64_t(uk);
        }
        wave_fence();
        ++nX;
      }
      if ((laterm >> l) & 1) {
        if (!((padmm >> l) & 1)) continue;  // waits for its previous call
        if (!~occ && !evict()) {
          overflow = true;
          break;
        }
        ready_insert(x, rec, sc, lo, hi);
      } else {
        // (room is made first: the user's own last call may be one that goes)
        const bool room = ~occ != 0 || evict() != 0;
        const SlotRec e = s_slot[x];
        const int32_t cn = uni(int32_t(e.num & kNumMask));
        const bool many = cn >= (__popcll(occ) < kPoolRoom ? kPoolRoom : kPoolShare);
        if (uni(int32_t(e.spilled)) != 0 || many) {
          spill_append(x, k, rec, sc, lo, hi);
        } else if (room) {
          append(x, k, rec, sc, lo, hi);
        } else {
          overflow = true;
          break;
        }
      }
    }
  }
  if (overflow) {  // nothing in the state buffer has changed yet
    if (lane == 0) {
      rs->overflow = 1;
      rs->mid = 0;
      rs->s_end = s_end;
    }
    return;
  }

  // Least and largest counter of the backlogged users (their calls at position 0).
  auto head_range = [&](int64_t &mn, int64_t &mx) {
    const bool hd = ((occ >> lane) & 1) && (ua & 63u) == 0;
    const uint32_t vh = kh & ~kPTier1;
    uint32_t hv = hd ? vh : 0xffffffffu, hx = hd ? vh : 0u;
    wave_minmax32v(hv, hx);
    const uint32_t mnh = uint32_t(uni(int32_t(hv))), mxh = uint32_t(uni(int32_t(hx)));
    uint32_t lv = hd && vh == mnh ? kl : 0xffffffffu, lx = hd && vh == mxh ? kl : 0u;
    wave_minmax32v(lv, lx);
    mn = int64_t((uint64_t(mnh) << 32) | uint32_t(uni(int32_t(lv))));
    mx = int64_t((uint64_t(mxh) << 32) | uint32_t(uni(int32_t(lx))));
  };
  if (nX > 0) {
    int64_t mx;
    head_range(minX, mx);
    dirty = true;
  }

  // ---- steps.  One loop: a pass takes the arrivals of step s in the window, then a batch
  // of its admissions, then ends the step; it starts over for the next window, for fewer
  // arrivals at a time, or for another batch of the step.  (One loop, so that the values
  // it carries have one place and are not copied between loops.)
  int64_t budget = 0;
  // batches that ended early since the last look at their rate (the others end a step each),
  // the step and the admissions then
  int32_t cuts = 0, s_look = s, seq_look = seq;
  bool deep = false;
  bool admit = false;  // the step's arrivals are done
  bool moved = false;  // the step has admitted
  int32_t lim = 64;    // arrivals taken at once
  while (true) {
    if (!admit) {
      if (nxt - wbase == 64 && nxt < n) {
        const int32_t old = wbase;
        wbase = nxt;
        load_window(old);
        const int32_t batches = cuts + (s - s_look);
        if (LINKS && batches >= kRateBatches) {
          // (the slot pass rebuilds the queue first: not for fewer steps than queued calls)
          deep = sp_total >= kDeep && s_end - s >= int64_t(sp_total) &&
                 int64_t(seq - seq_look) * kSlowDen < int64_t(batches) * (sp_total < kVeryDeep ? kSlow : kSlowVery);
          if (deep) {
            overflow = true;
            break;
          }
          cuts = 0;
          s_look = s;
          seq_look = seq;
        }
      }
      if (int64_t(s) >= s_end) break;
      const int j = nxt - wbase;
      if (nX == 0) {
        if (nxt == n) break;
        // nothing queued: the steps before the next arrival only pay back debt
        int32_t target = rdl(w_step, j);
        if (int64_t(target) > s_end) target = int32_t(s_end);
        if (target > s) {
          const int64_t k = target - s;
          if (debt < 0)
            debt = (k >= (int64_t(1) << 22) ? k >= (-debt + C - 1) / C : debt + k * C >= 0) ? 0 : debt + k * C;
          s = target;
          if (int64_t(s) >= s_end) break;
        }
      }
      if (FS_RARE(s == INT32_MAX)) {
        code = FS_E_OVERFLOW;
        break;
      }
      // monitoring stream: arrivals of step s in stream order
      if (nxt < n) {
        const uint64_t after = bal(w_step > s) & (~uint64_t(0) << j);
        const int32_t je = after ? first_of(after) : 64;
        if (je > j) {
          const int32_t j1 = je - j > lim ? j + lim : je;
          if (!arrive(j, j1)) {
            // no room: calls that are not next go to the spill lists, then fewer at a time
            if (evict() == 0) {
              if (j1 - j == 1) {
                overflow = true;  // (nothing of this arrival has happened)
                break;
              }
              lim = (j1 - j) >> 1;
            }
            continue;
          }
          lim = 64;
          nxt = wbase + j1;
          if (j1 < je || (j1 == 64 && nxt < n)) continue;
        }
      }
      budget = C + debt;
      admit = true;
      moved = false;
    }

    // execution stream: admit in key order while the step has budget
    if (occ && less_s(0, budget)) {
      const bool oc = in_mask(occ);
      const uint32_t tok = q_lo & uint32_t(kTokMask);
      const SlotRec e = s_slot[oc ? qx : 64];
      moved = true;
      if (dirty || (LINKS && !nearm)) take_ranks();
      const uint32_t bud = (budget >> 32) ? 0xffffffffu : uint32_t(budget);
      // (of the ranked calls: `pre` of the others starts at all ones and falls with every batch)
      uint64_t fm = bal(pre < bud) & (LINKS ? nearm : occ);
      if (LINKS && FS_RARE(fm == nearm && nearm != occ)) {  // all ranked calls fit: rank all
        far = 0;
        take_ranks();
        fm = bal(pre < bud) & nearm;
      }
      const int32_t ah = int32_t(ua & 63u), cn = int32_t(e.num & kNumMask);
      const uint64_t tailm = bal(ah == cn - 1);
      int cl = -1;
      if (LINKS || sp_total > 0) {
        // a call whose next call has arrived, or a user's last pooled call before spilled
        // ones, ends the batch
        uint64_t cutm = LINKS ? bal(uint32_t(q_succ) < uint32_t(nxt)) : 0;
        if (sp_total > 0) cutm |= tailm & bal(e.spilled != 0);
        cutm &= fm;
        if (cutm) {
          const uint32_t rc = wave_min32(in_mask(cutm) ? rank : 0xffffffffu);
          fm &= bal(rank <= rc);
          cl = first_of(cutm & bal(rank == rc));
        }
      }
      if (FS_RARE(!fm)) {
        code = FS_E_STATE;
        break;
      }
      const bool fin = in_mask(fm);
      const uint32_t m = uint32_t(__popcll(fm));
      const uint64_t unew = ((uint64_t(kh & ~kPTier1) << 32) | kl) + (((uint64_t(q_hi) << 32) | q_lo) >> 24);
      if (FS_RARE((bal(uint32_t(unew >> 32) >= uint32_t(uint64_t(kValueLimit) >> 32)) & fm) != 0)) {
        code = FS_E_OVERFLOW;
        break;
      }
      const int lastl = first_of(bal(rank == m - 1) & fm);  // the last admitted
      const uint32_t used = rdlu(pre + tok, lastl);
      s_adm[fin ? n_adm + below(fm) : kOutStage] = make_uint2(uint32_t(q_rec), uint32_t(s));
      n_adm += int32_t(m);
      if (FS_RARE(n_adm > kOutStage - 64)) flush_admitted();
      if (fin && (LINKS || want_seq || want_coa)) {
        if (LINKS) st8[q_rec >= cache_lo ? (q_rec & (M - 1)) : M + kStPad - 1] = 1;
        if (want_seq) {  // (optional outputs)
          int32_t *const as = KARG(admit_seq);
          int64_t *const ca = KARG(counter_after);
          if (as) as[base + q_rec] = seq + int32_t(rank);
          if (ca) ca[base + q_rec] = int64_t(unew);
        }
        if (want_coa)  // (the user's counter for its next arrivals, whatever else is asked for)
          __hip_atomic_fetch_max(s_uc + qx, (unsigned long long)unew, __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_WORKGROUP);
      }
      budget -= int64_t(used);
      backlog -= int64_t(used);
      seq += int32_t(m);
      // users that leave Q: their last pooled call is admitted, none is spilled or ready
      uint64_t lm = fm & tailm;
      if (cl >= 0) lm &= ~(uint64_t(1) << cl);
      // the admitted calls of users that stay leave their counts and positions
      if (lm != fm) {
        if (fin)
          __hip_atomic_fetch_add(&s_slot[qx].num, 0u - 1u - ((kh & kPTier1) ? 0u : kRdyOne), __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_WORKGROUP);
        wave_fence();
        const int32_t c_new = int32_t(s_slot[oc ? qx : 64].num & kNumMask);
        ua = in_mask(occ & ~fm) ? ua - uint32_t(cn - c_new) : ua;
      }
      if (lm) {
        // counters back to u; the last one in order is the last exit
        int ll = lastl;
        if (!((lm >> lastl) & 1)) {
          const uint32_t rl = wave_max32(in_mask(lm) ? rank : 0u);
          ll = first_of(lm & bal(rank == rl));
        }
        last_exit = int32_t(rdlu(ua, ll) >> kAheadBits);
        last_exit_u = rdl64(int64_t(unew), ll);
        const bool lv = in_mask(lm);
        const uint32_t w = e.num / kWinOne;
        uint4 *const we = s_win + (lv && w ? w - 1 : 64);
        we->x = uint32_t(unew);
        we->y = uint32_t(unew >> 32);
        we->z = 0xffffffffu;
        if (lv) set_u(int32_t(ua >> kAheadBits), int64_t(unew));
        s_xu[lv ? qx : 64] = -1;
        s_free[lv ? 64 - nX + below(lm) : 64] = qx;
        nX -= __popcll(lm);
      }
      rank -= m;
      pre -= used;
      kh = fin ? 0xffffffffu : kh;
      kl = fin ? 0xffffffffu : kl;
      ua = fin ? 0xffffffffu : ua;
      occ &= ~fm;
      if (LINKS) nearm &= ~fm;
      wave_fence();
      if (cl >= 0) {
        const int32_t c_x = rdl(qx, cl), c_sc = rdl(q_succ, cl);
        if (LINKS && uint32_t(c_sc) < uint32_t(nxt)) {
          int32_t s2;
          uint32_t lo2, hi2;
          fetch_rec(c_sc, s2, lo2, hi2);
          ready_insert(c_x, c_sc, s2, lo2, hi2);
        }
        if (LINKS) ++cuts;
        if (sp_total > 0 && uni(int32_t(s_slot[c_x].num & kNumMask)) == 0) spill_refill(c_x);
        continue;
      }
    }
    admit = false;
    debt = less_s(budget, 0) ? budget : 0;
    if (occ) {  // the gap sample, and the least counter for the next arrivals
      int64_t mx;
      if (moved) {
        // the first in order holds the least counter, if no ready call is queued; without
        // an admission the least counter is as it was
        if (!dirty && (!LINKS || nearm) && (!LINKS || !(occ & bal(!(kh & kPTier1))))) {
          const int l = first_of(occ & bal(rank == 0));
          minX = int64_t((uint64_t(rdlu(kh, l) & ~kPTier1) << 32) | rdlu(kl, l));
        } else {
          head_range(minX, mx);
        }
      }
      const uint64_t d = ((uint64_t(kh & ~kPTier1) << 32) | kl) - uint64_t(minX);
      if (occ & bal((ua & 63u) == 0) & bal(d > uint64_t(gap))) {
        int64_t mn;
        head_range(mn, mx);
        gap = mx - mn;
      }
    }
    ++s;
  }

  if (code) raise_err(a.err, code);
  if (wbase >= cache_from) flush_window(wbase);
  flush_admitted();

  // ---- save: counters of queued users back to u; the queue itself is rebuilt from
  // the records that have arrived and are still undecided
  if (((occ >> lane) & 1) && (ua & 63u) == 0)
    set_u(int32_t(ua >> kAheadBits), int64_t((uint64_t(kh & ~kPTier1) << 32) | kl));
  wave_fence();
  __syncthreads();
  if (ulds)
    for (int32_t k = lane; k < U; k += 64) u_all[k] = u_lds[k];
  // lowest record index that may still be queued
  {
    const int8_t *const fate = STATE(const int8_t, fate) + base;
    while (low < nxt) {
      const int32_t i = low + lane;
      const bool q = i < nxt && ld_fresh(fate + i) == -1;
      const uint64_t m = bal(q);
      if (m) {
        low += ff1(m);
        break;
      }
      low += 64;
    }
    if (low > nxt) low = nxt;
  }
  const bool drained = nxt == n && nX == 0;
  if (lane == 0) {
    rs->s = s;
    rs->nxt = nxt;
    rs->debt = debt;
    rs->backlog = backlog;
    rs->seq = seq;
    rs->gap = gap;
    rs->last_exit_u = last_exit_u;
    rs->low = low;
    rs->last_exit = last_exit;
    rs->done = drained ? 1 : 0;
    rs->overflow = deep ? kOutDeep : overflow ? 1 : 0;
    rs->mid = 0;
    rs->mid_budget = 0;
    rs->s_end = s_end;
    if (!overflow) {
      KARG(steps)[r] = s;
      KARG(decisions)[r] = seq;
      KARG(max_gap)[r] = gap;
    }
  }
  wave_fence();
  if (!overflow) {
    int64_t *const counter = KARG(counter) + int64_t(r) * U;
    for (int32_t k = lane; k < U; k += 64) counter[k] = ulds ? u_lds[k] : ld_fresh(u_all + k);
  }
}

}  // namespace
}  // namespace sched
}  // namespace fs
