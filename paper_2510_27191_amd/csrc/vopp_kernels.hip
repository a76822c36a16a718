// vopp_kernels.hip -- HIP kernels of one VOPP planning step for gfx950.
//
// One iteration of Alg. 1 is a short, fixed sequence of phases:
//
//   forward     one thread per episode runs every level of the vectorized
//               forward search (Alg. 2) with its state in registers: draw the
//               action from the softmax of the belief's preferences (Eq. 6),
//               call G, count the visit and reward into the action node
//               (AppendActions), and find or insert the child belief
//               (belief, action, observation) (AppendBeliefs).  Once an
//               episode creates a belief it is alone: the rest of its path is
//               a run of single-visit records, written without any look-up
//               (see vopp_device.hpp).
//   claim       long rows (|A| > kMaxA) only: first visits of action nodes, and
//               the leaves that became full.
//   accumulate  folds the trace of visits into the full beliefs (LDS-aggregated
//               atomics) and lists the beliefs that became full.
//   backup      Alg. 3 over every belief: the runs first, each walked bottom-up
//               by one thread (dev_chain), then one phase per depth over the
//               full beliefs of that depth; leaves take their mean heuristic,
//               internal beliefs update their preference row with
//               Q = C/N + gamma W and V = L_eta Psi, and each belief hands V*N_b
//               to its parent action's W (in a register inside a run, else a
//               64-bit add).  The root runs in double precision.
//
// All cross-episode sums (rewards, heuristics, V*N_b) are 64-bit fixed-point
// integer atomics, so the results do not depend on thread order; which episode
// creates a belief that several reach depends on the order of insertions, the
// tree and every value in it do not.
//
// Every phase is a __device__ function of (plan view, block index within the
// phase, block count of the phase).  The single-plan path launches one kernel
// per phase (for rows of up to kMaxA actions three per iteration: the search,
// the trace together with the runs, the full beliefs together with the root);
// the batched path launches k_batch, whose blocks each run one phase of one
// instance of a batch (BatchItem), so one launch advances every instance of
// the batch by one phase.
#include <hip/hip_ext.h>

#include <algorithm>
#include <climits>
#include <type_traits>

#include "vopp_device.hpp"
#include "vopp_launch.hpp"

namespace vopp {

// ---------------------------------------------------------------------------
// Open-addressing table of 16-byte slots, load <= 1/2.  Finds or inserts key;
// the inserting thread writes key | stamp.  Returns the slot, or ~0u if the
// table has no free slot left (an internal error, reported by the plan).
//
// A key hashes to a bucket of 4 slots (64 bytes), which the probe reads with
// one round of loads and scans in registers; a full bucket continues into the
// next.  Within a bucket the key visits the slots in a rotated order that is a
// function of the key, so every thread that looks for one key meets the same
// first empty slot (linear probing over a fixed per-key sequence: one
// compare-and-swap there decides the insert), while different keys spread
// their inserts over the bucket.  A wavefront waits for its slowest lane, so
// reading whole buckets and deciding in registers keeps most wavefronts at one
// read and at most one compare-and-swap per lane (a compare-and-swap is about
// twice as slow as a read).  Buckets of 8 slots cost twice the loads and scan.
// Keys and belief ids written by earlier kernels are visible to the plain
// loads; a key being inserted by this kernel may read as empty, and then the
// compare-and-swap returns it.
// ---------------------------------------------------------------------------
constexpr uint32_t kBucket = 4;

struct Bucket {
  uint4 v[kBucket];
  uint32_t base, rot;
};
__device__ __forceinline__ void bucket_load(const TreeView& t, Bucket& b) {
  const uint4* ln = reinterpret_cast<const uint4*>(&t.h_slot[b.base]);
#pragma unroll
  for (int j = 0; j < (int)kBucket; ++j) b.v[j] = ln[j];
}
// The first bucket of a key's probe sequence and the key's slot order in it.
__device__ __forceinline__ void bucket_read(const TreeView& t, unsigned long long key,
                                            Bucket& b) {
  const unsigned long long hk = mix64(key);
  b.base = (uint32_t)hk & t.h_mask & ~(kBucket - 1);
  b.rot = (uint32_t)(hk >> 40) & (kBucket - 1);
  bucket_load(t, b);
}
// A lane per episode: of the calling lanes with `in` set, those whose keys are
// equal have one leader; returns its number (the caller's own for a lane that
// leads or has `in` unset).  Where thousands of episodes share a few new beliefs,
// each lane's atomic on a belief's table slot or record takes its turn at one
// address; the leader's serves the lanes behind it (at most kAlone keys that one
// lane only has are looked at).  A plan of 60,000 episodes over 6 beliefs of two
// levels took 1,499 us without, 748 with; 65,536 over 30 beliefs of four levels
// 1,480 and 655.
constexpr int kAlone = 8;
__device__ __forceinline__ int lead_lane(bool in, unsigned long long key) {
  const int lane = threadIdx.x & 63;
  int lead = lane, alone = 0;
  while (alone < kAlone) {
    const unsigned long long m = __ballot(in);
    if (m == 0ull) break;
    const int l = __ffsll((long long)m) - 1;
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)key, l);
    const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(key >> 32), l);
    const bool same = in && (uint32_t)key == lo && (uint32_t)(key >> 32) == hi;
    if (same) {
      lead = l;
      in = false;
    }
    if (__popcll(__ballot(same)) == 1) ++alone;
  }
  return lead;
}
// crowd (uniform): levels below it are those at which lanes of the wavefront may
// have the same key (lead_lane); level: the caller's.  won:
// inserted by this call.  fresh: the stamp found is `stamp` (for a key
// found, not inserted: another episode of this launch inserted it, and id is
// not known yet); id: else the belief's id.  b: the key's first bucket, read.
__device__ __forceinline__ uint32_t probe(const TreeView& t, Bucket& b, unsigned long long key,
                                          unsigned long long stamp, int crowd, int level,
                                          bool& won, bool& fresh, int& id) {
  const uint32_t lines = (t.h_mask + 1) / kBucket;
  for (uint32_t n = 0; n <= 2 * lines; ++n) {
    // The first slot in the key's order that holds the key or is empty.
    uint32_t best = kBucket;
    int at = -1;
    bool empty = false;
    int rid = -1;
    unsigned long long seen = kEmptyKey;
#pragma unroll
    for (int j = 0; j < (int)kBucket; ++j) {
      const unsigned long long cur = ((unsigned long long)b.v[j].y << 32) | b.v[j].x;
      const uint32_t pos = ((uint32_t)j - b.rot) & (kBucket - 1);
      if ((cur == kEmptyKey || (cur & ~kStampMask) == key) && pos < best) {
        best = pos;
        at = j;
        empty = cur == kEmptyKey;
        seen = cur;
        rid = (int)b.v[j].z;
      }
    }
    if (at < 0) {                               // the bucket is full: next bucket
      b.base = (b.base + kBucket) & t.h_mask;
      bucket_load(t, b);
      continue;
    }
    const uint32_t slot = b.base + (uint32_t)at;
    if (empty) {
      int lead = (int)(threadIdx.x & 63);
      if (crowd) lead = lead_lane(level < crowd, key);
      const bool behind = lead != (int)(threadIdx.x & 63);
      if (!behind) seen = atomicCAS(&t.h_slot[slot].key, kEmptyKey, key | stamp);
      if (crowd && __any(behind)) {             // what the leader found there, or put
        const uint32_t lo = __shfl((uint32_t)seen, lead, 64);
        const uint32_t hi = __shfl((uint32_t)(seen >> 32), lead, 64);
        if (behind) {
          seen = ((unsigned long long)hi << 32) | lo;
          if (seen == kEmptyKey) seen = key | stamp;
        }
      }
      if (seen == kEmptyKey) {
        won = true;
        fresh = true;
        id = -1;
        return slot;
      }
      if ((seen & ~kStampMask) != key) {        // another key took it: the next slot
        atomicAdd(&t.counters[4], 1ull);
#pragma unroll
        for (int j = 0; j < (int)kBucket; ++j) {
          if (j == at) {
            b.v[j].x = (uint32_t)seen;
            b.v[j].y = (uint32_t)(seen >> 32);
          }
        }
        continue;
      }
      rid = -1;                                 // inserted by this launch
    }
    won = false;
    fresh = (seen & kStampMask) == stamp;
    id = fresh ? -1 : rid;
    return slot;
  }
  won = false;
  fresh = false;
  id = -1;
  return ~0u;
}

// Table key of the child of belief id under `low`, its action and observation
// (the observation takes the low ob bits, the action the next 26 - ob).
__device__ __forceinline__ unsigned long long belief_key(int id, uint32_t low) {
  return ((unsigned long long)(uint32_t)id << kKeyLowBits) | low;
}
__device__ __forceinline__ uint32_t key_low(int a, int obs, int ob) {
  return ((uint32_t)a << ob) | (uint32_t)obs;
}

// ---------------------------------------------------------------------------
// Shared memory of every phase (one static allocation per kernel).
// ---------------------------------------------------------------------------

// Block-level pre-aggregation.  Shallow tree levels funnel many episodes into
// few nodes (every episode of an iteration passes through one of the |A| root
// action nodes), so same-address global atomics would serialise.  Each block
// first combines its contributions per key in an LDS hash table and then
// issues one global atomic per distinct key.  Integer adds are
// order-independent, so results stay bit-identical.
constexpr int kAggSlots = 2 * kBlock;      // at most kBlock keys per block

struct AggTable {
  unsigned long long key[kAggSlots];
  unsigned long long a[kAggSlots];
  unsigned long long b[kAggSlots];
};

struct Smem {
  AggTable agg;
  unsigned long long wave[kBlock / 64];
  alignas(16) float psi0[kMaxA];   // the initial row
  float e0[kMaxA];                 // and its weights (RowBase)
  unsigned int n[2];
};

// Obstacle centres the forward search stages in LDS.
constexpr int kDiskLds = 64;

// What the forward search reads at every level, staged once per block.
struct SearchSmem {
  alignas(16) float psi0[kMaxA];   // the initial row
  alignas(16) float gauss[4096];   // the navigation model's noise table
  double psi0_cdf[kMaxA];          // running sums of the draws at new beliefs
  double root_cdf[kMaxA];          // and at the root
  float disks[2 * kDiskLds];       // obstacle centres, if there are no more than this
  unsigned long long wave[kBlock / 64];
};

__device__ __forceinline__ void agg_clear(AggTable& T) {
  for (int i = threadIdx.x; i < kAggSlots; i += kBlock) {
    T.key[i] = kEmptyKey;
    T.a[i] = 0ull;
    T.b[i] = 0ull;
  }
}

__device__ __forceinline__ int agg_slot(AggTable& T, unsigned long long key) {
  uint32_t h = (uint32_t)((key * 0x9E3779B97F4A7C15ull) >> 55);   // 9 bits
  while (true) {
    const unsigned long long prev = atomicCAS(&T.key[h], kEmptyKey, key);
    if (prev == kEmptyKey || prev == key) return (int)h;
    h = (h + 1) & (kAggSlots - 1);
  }
}

__device__ __forceinline__ unsigned long long wave_sum(unsigned long long v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

__device__ __forceinline__ unsigned long long wave_incl_scan(unsigned long long v) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    unsigned long long n = __shfl_up(v, off, 64);
    if (lane >= off) v += n;
  }
  return v;
}

// Sum over the block; red holds kBlock / 64 words of LDS.  Called by every
// thread of the block (it contains barriers); thread 0 gets the total.
__device__ __forceinline__ unsigned long long block_sum(unsigned long long v,
                                                        unsigned long long* red) {
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  unsigned long long t = 0;
  if (threadIdx.x == 0)
    for (int i = 0; i < kBlock / 64; ++i) t += red[i];
  __syncthreads();
  return t;
}

// ---------------------------------------------------------------------------
// Phase: set-up of a plan.  Clears the belief table (sized for one belief per
// episode and iteration, so it is small beside the tree), the counts and the
// root.
// ---------------------------------------------------------------------------
// LDS of the set-up of a plan with more than kMaxA actions (the root's draw
// table is built by the block).
struct SetupSmem {
  double buf[kBlock];
  double red[kBlock / 64];
  double bc;
  unsigned long long part[kBlock];
};
__device__ double block_max64(double v, double* red);
__device__ double block_ordered_sum(const double* x, int A, double m, double eta, double* cdf,
                                    double* buf, double* bc);

__device__ void dev_setup(const PlanView& P, int blk, int nblk, SetupSmem* ss) {
  const TreeView& T = P.t;
  const size_t hcap = (size_t)T.h_mask + 1;
  const size_t tid = (size_t)blk * kBlock + threadIdx.x;
  const size_t stride = (size_t)nblk * kBlock;
  if (!P.carry) {                               // else the re-rooting wrote it
    uint4* hs = reinterpret_cast<uint4*>(T.h_slot);
    const uint4 ones = make_uint4(~0u, ~0u, ~0u, ~0u);
    for (size_t i = tid; i < hcap; i += stride) hs[i] = ones;
  }
  // No episode of this plan has ended: zero run words, two at a time (the list
  // of full beliefs starts past an odd one).
  const size_t run_words = ((size_t)P.K * (size_t)P.n_p + 1) / 2;
  for (size_t i = tid; i < run_words; i += stride) reinterpret_cast<uint32_t*>(T.run)[i] = 0u;
  // Root action-node sums; with a kept root, stripe 0 of N and C starts from
  // its record (written below by block 0).
  for (size_t i = tid; i < (size_t)3 * T.ra * kStripes; i += stride)
    if (!(P.carry && i % kStripes == 0 && i < (size_t)2 * T.ra * kStripes)) T.root_acc[i] = 0ull;
  if (blk == 0) {
    if (!P.carry) {                             // a fresh root: every field of belief 0
      for (int i = threadIdx.x; i < T.ra; i += kBlock) {
        rec_psi(T, 0)[i] = 0.0f;
        rec_n(T, 0)[i] = 0;
        rec_c(T, 0)[i] = 0ull;
        rec_w(T, 0)[i] = 0ull;
      }
      for (int i = threadIdx.x; i < T.bw; i += kBlock) rec_bits(T, 0)[i] = 0u;
      if (threadIdx.x == 0) T.node[0].V = 0.0f;
    }
    for (int i = threadIdx.x; i <= kMaxDepth; i += kBlock) T.full_cnt[i] = 0u;
    __syncthreads();
    const int j = threadIdx.x;
    for (int i = j; i < kStatRows * kStripes; i += kBlock) T.stats[i] = 0ull;
    if (j == 0) {
      T.gate[0] = (unsigned long long)wall_clock64();   // start of the plan
      T.gate[1] = 0ull;
      T.gate[2] = 0ull;
    }
    for (int a = j; a < T.ra; a += kBlock) {
      // Initial preferences ln pi0 / eta: the root keeps them in double
      // precision, every other belief starts from their f32 rounding.
      const double v = a < P.m.nA ? P.m.logpi0[a] / P.eta64 : 0.0;
      T.psi0[a] = (float)v;
      if (a < P.m.nA) {
        if (P.carry) {                          // the kept root's own row and sums
          // (long rows: the kept belief's columns count where its bitmap says)
          const bool v = T.ra <= kMaxA || ((rec_bits(T, 0)[a >> 5] >> (a & 31)) & 1u);
          T.psi_root[a] = (double)rec_psi(T, 0)[a];
          T.root_acc[((size_t)0 * T.ra + a) * kStripes] =
              v ? (unsigned long long)(long long)rec_n(T, 0)[a] : 0ull;
          T.root_acc[((size_t)1 * T.ra + a) * kStripes] = v ? rec_c(T, 0)[a] : 0ull;
        } else {
          rec_psi(T, 0)[a] = (float)v;
          T.psi_root[a] = v;
        }
      } else if (P.carry) {
        T.root_acc[((size_t)0 * T.ra + a) * kStripes] = 0ull;
        T.root_acc[((size_t)1 * T.ra + a) * kStripes] = 0ull;
      }
    }
    __syncthreads();
    if (T.ra > kMaxA) {                         // long rows: the block builds the table
      double mloc = -INFINITY;
      for (int a = j; a < P.m.nA; a += kBlock) mloc = fmax(mloc, T.psi_root[a]);
      const double m = block_max64(mloc, ss->red);
      block_ordered_sum(T.psi_root, P.m.nA, m, P.eta64, T.root_cdf, ss->buf, &ss->bc);
      // The initial row's running sums: eta * psi0 = ln pi0.
      double m0 = -INFINITY;
      for (int a = j; a < P.m.nA; a += kBlock) m0 = fmax(m0, P.m.logpi0[a]);
      m0 = block_max64(m0, ss->red);
      block_ordered_sum(P.m.logpi0, P.m.nA, m0, 1.0, T.psi0_cdf64, ss->buf, &ss->bc);
    }
    if (j == 0) {
      if (T.ra <= kMaxA) {
        root_cdf(T.psi_root, P.m.nA, P.eta64, T.root_cdf);
        // The initial row ln pi0 / eta in double precision: its running sums
        // serve the draws at beliefs created in the current iteration.
        double m = P.m.logpi0[0] / P.eta64;
        for (int a = 1; a < P.m.nA; ++a) m = fmax(m, P.m.logpi0[a] / P.eta64);
        double run = 0.0;
        for (int a = 0; a < P.m.nA; ++a) {
          run = run + exp(P.eta64 * (P.m.logpi0[a] / P.eta64 - m));
          T.psi0_cdf64[a] = run;
        }
      }
      T.info[0] = BeliefInfo{0, P.carry ? T.info[0].Nb : 0, kEmptyKey};
      T.node[0].link = kLinkFull;
      T.v_root[0] = P.carry ? (double)T.node[0].V : 0.0;
      T.counters[1] = 0ull;
      T.counters[4] = 0ull;
    }
  }
}

// ---------------------------------------------------------------------------
// Phase: the forward search of iteration k over D levels (Alg. 2).
// ---------------------------------------------------------------------------

// An episode's state.
struct Episode {
  int s;                      // tabular, or navigation (x, y)
  float x, y;
};

// The rows of a belief that becomes full: what its single visit left there
// (link, r, psi: its record).  own: its parent and key, for a belief inside a
// run (a run's first belief has them already).  fresh: created in this
// iteration.  Only the episode that set kLinkClaim calls, and no other reads
// these rows before the next launch.
__device__ __forceinline__ void make_full(const PlanView& P, const float* psi0s, int id,
                                          uint32_t link, float r, float psi,
                                          unsigned long long own, bool fresh) {
  const TreeView& T = P.t;
  const int ra = T.ra;
  const int a = (link & kLinkAct) ? (int)((link & kLinkKey) >> P.m.obs_bits) : -1;
  float* prow = rec_psi(T, id);
  int* nrow = rec_n(T, id);
  ulonglong2* cq = reinterpret_cast<ulonglong2*>(rec_c(T, id));
  ulonglong2* wq = reinterpret_cast<ulonglong2*>(rec_w(T, id));
  const ulonglong2 z2 = make_ulonglong2(0ull, 0ull);
  const unsigned long long fx = to_fix(r, P.fix_scale);
  for (int j = 0; j < ra; j += 4) {
    float4 q = *reinterpret_cast<const float4*>(psi0s + j);
    if (a == j) q.x = psi;
    if (a == j + 1) q.y = psi;
    if (a == j + 2) q.z = psi;
    if (a == j + 3) q.w = psi;
    *reinterpret_cast<float4*>(prow + j) = q;
    *reinterpret_cast<int4*>(nrow + j) =
        make_int4(a == j, a == j + 1, a == j + 2, a == j + 3);
    cq[j / 2] = make_ulonglong2(a == j ? fx : 0ull, a == j + 1 ? fx : 0ull);
    cq[j / 2 + 1] = make_ulonglong2(a == j + 2 ? fx : 0ull, a == j + 3 ? fx : 0ull);
    wq[j / 2] = z2;
    wq[j / 2 + 1] = z2;
  }
  // A leaf that this iteration created: its creator's arrival counts.
  const bool leaf = fresh && a < 0;
  if (!(link & kLinkHead)) T.info[id] = BeliefInfo{leaf ? 1 : 0, 1, own};
  else if (leaf) atomicAdd(&T.info[id].leaf_cnt, 1);
  if (a < 0) T.node[id].u.leaf_h = leaf ? fx : 0ull;
}

// Whether the caller is the first to reach the single-visit belief id besides
// its creator (link: its record's flags as read; a full or claimed one: no).
__device__ __forceinline__ bool claim(const TreeView& T, int id, uint32_t link,
                                      uint32_t more = 0u) {
  if (id == 0 || (link & (kLinkFull | kLinkClaim))) return false;
  return !(atomicOr(&T.node[id].link, kLinkClaim | more) & kLinkClaim);
}
// claim() by a lane per episode.
__device__ __forceinline__ bool claim_lanes(const TreeView& T, int id, uint32_t link,
                                            bool crowd, uint32_t more = 0u) {
  const bool want = id != 0 && !(link & (kLinkFull | kLinkClaim));
  const int lead = lead_lane(want && crowd, (unsigned long long)(uint32_t)id);
  return want && lead == (int)(threadIdx.x & 63) && claim(T, id, link, more);
}

// Stores and loads that pass the caches of this XCD: what an episode's run
// leaves for the episodes of the same launch that reach its first belief.
__device__ __forceinline__ void store_seen(BeliefNode* p, uint32_t v, uint32_t link, uint32_t r,
                                           uint32_t psi) {
  unsigned long long* q = reinterpret_cast<unsigned long long*>(p);
  __hip_atomic_store(q, ((unsigned long long)link << 32) | v, __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
  __hip_atomic_store(q + 1, ((unsigned long long)psi << 32) | r, __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void store_seen(BeliefInfo* p, unsigned long long own) {
  unsigned long long* q = reinterpret_cast<unsigned long long*>(p);
  __hip_atomic_store(q, 1ull << 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // {0, 1}
  __hip_atomic_store(q + 1, own, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint4 load_seen(const BeliefNode* p) {
  const unsigned long long* q = reinterpret_cast<const unsigned long long*>(p);
  const unsigned long long a =
      __hip_atomic_load(q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const unsigned long long b =
      __hip_atomic_load(q + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return make_uint4((uint32_t)a, (uint32_t)(a >> 32), (uint32_t)b, (uint32_t)(b >> 32));
}
// Whether the run of an episode of this launch (its word as read) has come so
// far that its belief at level d is written.
__device__ __forceinline__ bool run_has(uint32_t run, int d) {
  return (run & kRunOpen) ? (int)(run & kRunMask) > d : run != 0u;
}

// Whether a wait of this launch that has taken `turns` turns is given up: it
// reached its bound, or another wait of the plan has.
__device__ __forceinline__ bool wait_over(const PlanView& P, uint32_t turns) {
  if (turns > P.wait_turns) return true;
  return (turns & 1023u) == 0u &&
         (__hip_atomic_load(&P.t.counters[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) &
          kErrWait);
}
// Every store of this wavefront so far has reached the point all XCDs see.
__device__ __forceinline__ void stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// The leaf of a plan of one level that the calling episode created, found in
// slot h; the slot's id is read by later launches only.
__device__ __forceinline__ void make_leaf(const TreeView& T, uint32_t h, int id,
                                          unsigned long long own) {
  T.h_slot[h].id = id;
  BeliefNode nb;
  nb.V = 0.0f;
  nb.link = kLinkFull | kLinkBare;
  nb.u.leaf_h = 0ull;
  T.node[id] = nb;
  T.info[id] = BeliefInfo{0, 0, own};
}
// The trace word of a leaf that needs no look: its id, or ~(table slot).
__device__ __forceinline__ unsigned long long leaf_word(int id) {
  return id < 0 ? kTraceSlot | (uint32_t)~id : (unsigned long long)(uint32_t)id;
}

// Runs episode ep from e to its end.  ONE: a plan of one level (one_level).
//
// Two episodes of one launch may reach the same new belief.  The one that
// inserted its key owns it and never waits: it goes on along its run, and
// once the belief's record is written it publishes the belief's id in the table
// slot (one level later, when the record's store has long arrived).  The other
// looks at the slot once per turn of its loop until the id is there, then goes on
// from the belief like any visitor.  If it draws the owner's own action and
// observation it follows the owner's run, each belief of it once the owner's run
// word (TreeView::run) says that it is written; the owner says so one level
// later, when the record's store has arrived.  (To the end of the owner's run, as
// it was before, the followers of few beliefs waited once per level: 3 x 8
// levels of 16,384 episodes over 511 beliefs took 484 us, now 408, and 65,536
// of nav2d over one cell 760, now 690.)  Owners run already and wait for
// nothing, and a turn of the loop moves every other lane of the wavefront on as
// well, so every wait ends.
// (P.wait_turns bounds them all the same, for a tree that something else wrote
// to: the episode then ends where it waits and the plan reports an error.)
//
// Bound by dependent accesses while the episode visits beliefs of the
// tree (node and row, table line, compare-and-swap: 2 to 3 levels of them),
// then by the arithmetic of its run (Philox, draw, G; one 16-byte store per
// level, no atomics).  Before beliefs of a single visit had records of their
// own, every level probed the table, wrote 128 bytes or more per belief and
// counted its visit with two atomics: 57 us a launch instead of 36 for 65,536
// episodes of nav2d to depth 10, 202 instead of 142 for sparse4096.
constexpr int kPolls = 4;
template <int AM, bool NAV, bool TRACE, bool ONE>
__device__ void search(const PlanView& P, int k, int D, int ep, const Episode& e0,
                       const SearchSmem& L, const DiskCache& dc, unsigned long long& g,
                       unsigned long long& nt) {
  const float* psi0s = L.psi0;
  const TreeView& T = P.t;
  const int t0 = first_step(P, k);            // level step of level 0
  const int first_new = 1 + t0 * P.n_p;       // ids created in this iteration
  const int A = NAV ? 4 : P.m.nA, ob = P.m.obs_bits;
  const size_t n_p = (size_t)P.n_p;
  const unsigned long long stamp = (unsigned long long)(k - 1) << kStampShift;
  int s = e0.s, id = 0, d = 0;
  float x = e0.x, y = e0.y;
  // The running sums of the initial row in registers for short rows, so that
  // a draw at a belief created in this iteration issues no memory access.
  constexpr int kCdfRegs = AM <= 8 ? AM : 1;
  double cdf0[kCdfRegs];
#pragma unroll
  for (int j = 0; j < kCdfRegs; ++j) cdf0[j] = (AM <= 8 && j < A) ? L.psi0_cdf[j] : 0.0;
  // Inputs of the next level, read ahead of the previous level's writes: a
  // wait for a load also waits for every memory operation issued before it.
  U4 w = draw(P, (uint32_t)ep, kTagStep, 0u, (uint32_t)k);
  NavNoise z{0.0f, 0.0f, 0.0f, 0.0f};
  if (NAV) z = nav_noise(L.gauss, w);
  float row[AM];
  uint32_t link = 0;          // the record of the belief it visits (root: 0)
  float nr = 0.0f, npsi = 0.0f;
  unsigned long long own = 0; // its parent and key, if it was reached by a run
  // Reads the record of belief id, and its row if it has one of its own (a
  // single-visit belief's row is the initial one but for one entry).
  auto arrive = [&](bool want_row) {
    const bool is_new = id >= first_new;
    want_row = want_row && !is_new;
    uint4 q;
    if (is_new) q = load_seen(&T.node[id]);
    else q = *reinterpret_cast<const uint4*>(&T.node[id]);
    if (want_row) load_row<AM>(rec_psi(T, id), A, row);
    link = q.y;
    nr = __uint_as_float(q.z);
    npsi = __uint_as_float(q.w);
    if (want_row && !(link & kLinkFull)) {
      const int a1 = (link & kLinkAct) ? (int)((link & kLinkKey) >> ob) : -1;
#pragma unroll
      for (int j = 0; j < AM; ++j)
        if (j < A) row[j] = j == a1 ? npsi : psi0s[j];
    }
  };
#pragma unroll
  for (int j = 0; j < AM; ++j) row[j] = 0.0f;
  bool tail = false;          // it stands on a belief of its own
  uint32_t head = 0;          // kLinkHead at the first of its run
  int tl = 0;                 // levels that visited existing beliefs
  uint32_t slot = 0;          // of its first belief, or of the one it waits for
  int id_head = 0;
  int to_publish = 0;         // 1: the first belief's record is to be written, 2: is
                              // written, the slot's id is not
  int waits = 0;              // 1: for the id in the slot, 2: for the record of
                              // the belief id, in the run of its creator
  bool alive = true;
  // The draw at a belief created in this iteration.
  auto draw_new = [&](uint32_t x0) {
    if constexpr (AM <= 8) return draw_cdf64_regs<AM>(cdf0, A, x0);
    else return draw_cdf64(L.psi0_cdf, A, x0);
  };
  // G under the drawn action a (or the forced one, then a is that).
  auto step = [&](int& a, float& r, int& obs, bool& term) {
    if (TRACE) {
      const size_t di = (size_t)(t0 + d - P.carry_steps) * n_p + ep;
      T.dbg_act[di] = (short)a;               // the kernel's own decision
      if (T.dbg_force) {
        const short f = T.dbg_force[di];
        if (f >= 0 && f < A) a = f;
      }
    }
    if constexpr (!NAV) {
      int sn;
      tabular_step(P.m, s, a, w, sn, obs, r);
      s = sn;
    } else {
      float nx, ny;
      nav_step_z(P.m, dc, P.m.nav.n_disks <= kDiskLds ? L.disks : P.m.disks, x, y, a, z, nx, ny,
                 obs, r, term);
      x = nx;
      y = ny;
    }
    ++g;
    if (TRACE) T.dbg_obs[(size_t)(t0 + d - P.carry_steps) * n_p + ep] = obs;
  };
  // The next level's random block and noise.
  auto next_block = [&]() {
    w = draw(P, (uint32_t)ep, kTagStep, (uint32_t)(d + 1), (uint32_t)k);
    if (NAV) z = nav_noise(L.gauss, w);
  };
  // A level on its own run: the whole action node and the link to the next
  // belief.
  auto run_level = [&](int a) {
    float r;
    int obs;
    bool term = false;
    step(a, r, obs, term);
    if (!head) {                      // the records above this one are written
      stores_done();
      __hip_atomic_store(&T.run[(size_t)(k - 1) * n_p + ep], (unsigned short)(kRunOpen | d),
                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    const uint32_t ln = key_low(a, obs, ob) | kLinkAct | (term ? 0u : kLinkChild) | head;
    store_seen(&T.node[id], 0u, ln, __float_as_uint(r), __float_as_uint(psi0s[a]));
    next_block();
    alive = !term;
    if (alive) {
      id += P.n_p;
      head = 0;
      ++d;
    }
  };
  // One level at a belief of the tree.
  auto level = [&]() {
    // Eq. (6): the root's running sums (double precision), those of the
    // initial row for a belief created in this iteration, else the row.
    int a;
    bool tie = false;
    if (id == 0) {
      a = draw_cdf64(L.root_cdf, A, w.x);
      tie = (k > 1 || P.carry) && near_tie64(L.root_cdf, A, w.x, a);
    } else if (id >= first_new) {
      a = draw_new(w.x);
    } else {
      a = draw_row32<AM>(row, A, P.eta, w.x, tie);
    }
    nt += tie ? 1u : 0u;
    float r;
    int obs;
    bool term = false;
    step(a, r, obs, term);
    const uint32_t low = key_low(a, obs, ob);
    // A belief of the tree.
    const int b = id;
    const uint32_t blink = link;
    const bool by_run = (blink & kLinkChild) && (blink & kLinkKey) == low;
    const bool look = !term && !by_run;
    const unsigned long long bk = belief_key(b, low);
    Bucket line;
    if (look) bucket_read(T, bk, line);
    const bool first = P.crowd ? claim_lanes(T, b, blink, d <= P.crowd) : claim(T, b, blink);
    next_block();
    const float b_r = nr, b_psi = npsi;
    const unsigned long long b_own = own;
    bool won = false;
    uint32_t h = 0;
    if (term) {
      alive = false;                          // FilterTerminals
      tl = d + 1;
    } else if (by_run) {                      // where its creator went
      id = b + P.n_p;
      own = bk;
      if (b >= first_new) waits = 2;
    } else {
      // AppendBeliefs: find or insert (b, a, o).
      bool fresh = false;
      int old = -1;
      h = probe(T, line, bk, stamp, P.crowd, d, won, fresh, old);
      if (h == ~0u) {                         // table full: stop and report
        atomicOr((unsigned int*)&T.counters[1], kErrTable);
        alive = false;
        tl = d + 1;
      } else if (ONE && won) {
        id = 1 + t0 * P.n_p + ep;
        tl = 1;
        make_leaf(T, h, id, bk);
      } else if (won) {
        tail = true;
        head = kLinkHead;
        tl = d + 1;
        id = 1 + (t0 + d) * P.n_p + ep;
        id_head = id;
        slot = h;
        to_publish = 1;
      } else if (ONE && fresh) {
        id = ~(int)h;
      } else if (fresh) {
        slot = h;
        waits = 1;
      } else {
        id = old;
      }
    }
    if (!ONE && alive && !tail && !waits) arrive(d + 1 < D);
    // Writes of level d: the visit and reward of (b, a) (AppendActions) go
    // to the row if it may be written in this launch, else to the trace.
    unsigned long long tk = kEmptyKey;
    if (d >= kDirectLevel && (blink & kLinkFull)) {
      atomicAdd(&rec_n(T, b)[a], 1);
      const unsigned long long fx = to_fix(r, P.fix_scale);
      if (fx) atomicAdd(&rec_c(T, b)[a], fx);
    } else {
      tk = ((unsigned long long)(uint32_t)b << kActBits) | (uint32_t)a |
           (first ? kTraceClaim : 0ull);
    }
    T.tr_key[(size_t)d * n_p + ep] = tk;
    T.tr_val[(size_t)d * n_p + ep] = r;
    if (first) make_full(P, psi0s, b, blink, b_r, b_psi, b_own, b >= first_new);
    if (!ONE && won) store_seen(&T.info[id], bk);
    if (alive) ++d;
  };
  // The end of the episode: its leaf, its run word.
  auto finish = [&]() {
    if (TRACE && !alive) {
      for (int q = d + 1; q < D; ++q) {
        const size_t di = (size_t)(t0 + q - P.carry_steps) * n_p + ep;
        T.dbg_act[di] = (short)-1;
        T.dbg_obs[di] = -1;
      }
    }
    uint32_t run;
    if (!alive) {                               // d: the level it ended at
      run = (uint32_t)tl | (tail ? (uint32_t)(d - tl + 1) << kRunLenShift : 0u);
    } else {
      float hv = 0.0f;                          // ValueHeuristic of the leaf state
      if constexpr (!NAV) {
        if (P.m.H) hv = P.m.H[s];
      } else {
        hv = nav_heuristic(P.m.nav, x, y);
      }
      const unsigned long long fx = to_fix(hv, P.fix_scale);
      if (tail) {
        store_seen(&T.node[id], __float_as_uint(from_fix(fx, P.fix_inv)), head,
                   __float_as_uint(hv), 0u);
        run = (uint32_t)tl | (uint32_t)(D - tl + 1) << kRunLenShift;
      } else {
        run = (uint32_t)D;
        const bool first = ONE ? false : P.crowd ? claim_lanes(T, id, link, d <= P.crowd) : claim(T, id, link);
        if (ONE) {
          run |= kRunLeaf | (uint32_t)tl << kRunLenShift;
          T.tr_key[(size_t)D * n_p + ep] = leaf_word(id);
          T.tr_val[(size_t)D * n_p + ep] = hv;
        } else if (D >= kDirectLevel && (link & kLinkFull)) {
          atomicAdd(&T.info[id].leaf_cnt, 1);
          if (fx) atomicAdd(&T.node[id].u.leaf_h, fx);
        } else {
          run |= kRunLeaf;
          T.tr_key[(size_t)D * n_p + ep] =
              (unsigned long long)(uint32_t)id | (first ? kTraceClaim : 0ull);
          T.tr_val[(size_t)D * n_p + ep] = hv;
        }
        if (first) make_full(P, psi0s, id, link, nr, npsi, own, id >= first_new);
      }
    }
    if (!ONE) stores_done();
    if (to_publish)
      __hip_atomic_store(&T.h_slot[slot].id, id_head, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    to_publish = 0;
    __hip_atomic_store(&T.run[(size_t)(k - 1) * n_p + ep], (unsigned short)run, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
  };
  // The loop ends for the whole wavefront at once, so that a lane that has ended
  // has published its run before any lane of the wavefront waits again.
  bool done = false;
  uint32_t turns = 0;         // of the wavefront, with a lane that waits
  do {
    if (__any(waits) && wait_over(P, ++turns)) {
      if (waits) {            // levels 0 .. d - 1 are in the trace
        atomicOr((unsigned int*)&T.counters[1], kErrWait);
        waits = 0;
        alive = false;
        tl = d;
      }
    }
    if (to_publish == 2) {
      stores_done();
      __hip_atomic_store(&T.h_slot[slot].id, id_head, __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
      to_publish = 0;
    }
    // Once every lane left is on its own run, a loop of just that (about 1,300
    // cycles a level against 4,700 through the branches above).
    if (__all(done || (tail && !to_publish))) {
      if (!done) {
        while (alive && d < D) {
          const int a = draw_new(w.x);
          run_level(a);
        }
      }
    }
    if (!done) {
      // A turn costs the wavefront its slowest lane (4 us with a visited
      // belief in it), so a lane that waits looks up to kPolls times (0.3 us
      // each) before it lets the turn go by, and goes on in the same turn.  With
      // one look, and the own runs' levels in level()'s branches, a launch
      // took 31 us instead of 22 (2,048 episodes of nav2d) and 44 instead of
      // 36 (65,536).
      for (int tries = 0; tries < kPolls && __any(waits); ++tries) {
        if (waits == 1) {
          const int got = __hip_atomic_load(&T.h_slot[slot].id, __ATOMIC_RELAXED,
                                            __HIP_MEMORY_SCOPE_AGENT);
          if (got >= 0) {
            id = got;
            waits = -1;
          }
        } else if (waits == 2) {
          const int owner = (id - 1) % P.n_p;
          const uint32_t run = __hip_atomic_load(&T.run[(size_t)(k - 1) * n_p + owner],
                                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          if (run_has(run, d)) waits = -1;
        }
        if (__all(waits <= 0)) break;
      }
      if (waits < 0) {
        waits = 0;
        arrive(d < D);
      }
      if (!waits) {
        if (!tail && alive && d < D) level();
        if (tail && alive && d < D) {
          run_level(draw_new(w.x));
          if (to_publish) to_publish = 2;
        } else if (!waits && !(alive && d < D)) {
          finish();
          done = true;
        }
      }
    }
  } while (__ballot(!done));
}

// The block's particle steps and near ties (both in one word: a block makes
// fewer than 2^32 of each).
__device__ __forceinline__ void tally(const TreeView& T, int blk, unsigned long long g,
                                      unsigned long long nt, unsigned long long* red) {
  g = block_sum(g | (nt << 32), red);
  if (threadIdx.x == 0 && (g & 0xffffffffull))
    atomicAdd(&T.stats[blk % kStripes], g & 0xffffffffull);
  if (threadIdx.x == 0 && (g >> 32))
    atomicAdd(&T.stats[kStatNear * kStripes + blk % kStripes], g >> 32);
}

// The initial row in LDS (every thread of the block calls).
__device__ __forceinline__ void stage_psi0(const TreeView& T, float* psi0s) {
  for (int i = threadIdx.x; i < T.ra; i += kBlock) psi0s[i] = T.psi0[i];
  __syncthreads();
}
// The search's tables: a level of a run then reads no global memory in the
// navigation model, and the root's draw (a serial scan of the running sums)
// none in any.
template <bool NAV>
__device__ __forceinline__ void stage_search(const PlanView& P, SearchSmem& L) {
  const int j = threadIdx.x;
  if constexpr (NAV) {
    const float4* src = reinterpret_cast<const float4*>(P.m.gauss);
    float4* dst = reinterpret_cast<float4*>(L.gauss);
#pragma unroll
    for (int i = 0; i < 1024 / kBlock; ++i) dst[i * kBlock + j] = src[i * kBlock + j];
    if (j < 2 * min(P.m.nav.n_disks, kDiskLds)) L.disks[j] = P.m.disks[j];
  }
  if (j < P.m.nA) {
    L.psi0_cdf[j] = P.t.psi0_cdf64[j];
    L.root_cdf[j] = P.t.root_cdf[j];
  }
  stage_psi0(P.t, L.psi0);
}

// Alg. 1: the episode starts at the root with a state drawn from the belief
// particles.
__device__ __forceinline__ Episode at_root(const PlanView& P, int k, int ep, bool report) {
  Episode e{0, 0.0f, 0.0f};
  const U4 w = draw(P, (uint32_t)ep, kTagRoot, 0, (uint32_t)k);
  const uint32_t idx = __umulhi(w.x, (uint32_t)P.e.n_belief);
  if (P.m.kind == kTabular) {
    e.s = ((const int*)P.e.belief)[idx];
    if ((unsigned)e.s >= (unsigned)P.m.nS) {   // caller's particle out of range
      if (report) atomicOr((unsigned int*)&P.t.counters[1], kErrState);
      e.s = 0;
    }
  } else {
    const float* bf = (const float*)P.e.belief;
    e.x = bf[idx];
    e.y = bf[P.e.n_belief + idx];
  }
  return e;
}

// All episodes from the root, one thread each.
template <int AM, bool NAV, bool TRACE, bool ONE>
__device__ void dev_forward(const PlanView& P, int k, int D, int blk, SearchSmem& L) {
  stage_search<NAV>(P, L);
  // dev_full of this iteration starts from nothing.
  if (blk == 0 && threadIdx.x == 0) P.t.counters[2] = P.t.counters[3] = 0ull;
  const int ep = blk * kBlock + threadIdx.x;
  unsigned long long g = 0, nt = 0;
  const DiskCache dc = NAV ? load_disks(P.m) : DiskCache{};
  if (ep < P.n_p) {
    const Episode e = at_root(P, k, ep, true);
    search<AM, NAV, TRACE, ONE>(P, k, D, ep, e, L, dc, g, nt);
  }
  tally(P.t, blk, g, nt, L.wave);
}

// ---------------------------------------------------------------------------
// Phase: fold the trace of iteration k (D levels) into the rows.
// Aggregation keys: (id << (kActBits + 1)) | (a << 1) for action nodes,
// (id << (kActBits + 1)) | 1 for leaves.
// ---------------------------------------------------------------------------

// Stripe q (0: N, 1: C, 2: W) of root action a for the calling block.
__device__ __forceinline__ unsigned long long* root_stripe(const TreeView& T, int q, int a) {
  // Long rows spread the root's visits over many actions: no striping there.
  const int stripe = T.ra > kMaxA ? 0 : (int)(blockIdx.x % kStripes);
  return T.root_acc + ((size_t)q * T.ra + a) * kStripes + stripe;
}

// The trace word of episode ep at `lvl` (D: its leaf), or kEmptyKey.
__device__ __forceinline__ unsigned long long trace_word(const PlanView& P, int k, int D,
                                                         int lvl, int ep) {
  const uint32_t run = P.t.run[(size_t)(k - 1) * (size_t)P.n_p + ep];
  const bool has = lvl < D ? lvl < (int)(run & kRunMask) : (run & kRunLeaf) != 0;
  return has ? P.t.tr_key[(size_t)lvl * (size_t)P.n_p + ep] : kEmptyKey;
}

// The parent and key of belief id (link: its record's) once its run is
// complete: inside a run, the belief before it.
__device__ __forceinline__ unsigned long long own_of(const TreeView& t, int id, uint32_t link,
                                                     int n_p) {
  if (link & (kLinkHead | kLinkClaim | kLinkFull)) return t.info[id].own;
  const int par = id - n_p;
  return ((unsigned long long)(uint32_t)par << kKeyLowBits) | (t.node[par].link & kLinkKey);
}
// The action of a single-visit belief's one node, or -1.
__device__ __forceinline__ int one_action(uint32_t link, int ob) {
  return (link & kLinkAct) ? (int)((link & kLinkKey) >> ob) : -1;
}
// A long-row belief that becomes full (make_full), by one lane: its action node
// (the other columns are cleared by their first visit) and the rest but Psi and the
// bitmap.
__device__ __forceinline__ void make_full_node(const PlanView& P, int id, uint32_t link, float r,
                                               unsigned long long own, bool fresh) {
  const TreeView& T = P.t;
  const int a = one_action(link, P.m.obs_bits);
  const unsigned long long fx = to_fix(r, P.fix_scale);
  if (a >= 0) {
    rec_n(T, id)[a] = 1;
    rec_c(T, id)[a] = fx;
    rec_w(T, id)[a] = 0ull;
  }
  const bool leaf = fresh && a < 0;
  if (!(link & kLinkHead)) T.info[id] = BeliefInfo{leaf ? 1 : 0, 1, own};
  else if (leaf) atomicAdd(&T.info[id].leaf_cnt, 1);
  if (a < 0) T.node[id].u.leaf_h = leaf ? fx : 0ull;
}
// Quad i of a long row, with psi as the row's entry a (a < 0: none).
__device__ __forceinline__ float4 with_entry(float4 v, int i, int a, float psi) {
  if (a >> 2 == i) {
    if ((a & 3) == 0) v.x = psi;
    if ((a & 3) == 1) v.y = psi;
    if ((a & 3) == 2) v.z = psi;
    if ((a & 3) == 3) v.w = psi;
  }
  return v;
}
// The bitmap of such a belief, by W lanes.
template <int W>
__device__ __forceinline__ void store_bits(const TreeView& T, int id, int a, int lane) {
  uint32_t* bits = rec_bits(T, id);
  for (int i = lane; i < T.bw; i += W) bits[i] = a >> 5 == i ? 1u << (a & 31) : 0u;
}

// Long rows.  The first visit of each (b, a) in the trace of an iteration sets bit
// a of b's bitmap and clears N[a], C[a] and W[a] (the root keeps its sums
// elsewhere).  A leaf's visits come as its table slot or its id: here the first
// one besides its creator's makes it full, and the word becomes the id.  (In the
// search an episode would wait for a new leaf's creator, read the leaf's
// record and set its flag, one after the other, only to end there; and once the
// policy leans to one action, most episodes set one flag.  Four iterations to
// depth 2, 16,384 episodes: 364 us that way, 335 this way with 65 actions, 1,058
// and 1,029 with 3,000.)  All of it before the accumulate pass adds the visits.
// Blocks 0 .. claim_visit_blocks - 1 take the visits of (b, a), the others the
// leaves, claim_leaves episodes a wavefront: the wavefront writes the rows of
// the leaves it makes full, so there are few to each, unless they stay bare.
__host__ __device__ inline int claim_visit_blocks(int n_p, int D) {
  const long long b = ((long long)D * n_p + kBlock - 1) / kBlock;
  return (int)(b < (1 << 16) ? b : 1 << 16);
}
__host__ __device__ inline int claim_leaves(const PlanView& P, int D) {
  return D == P.depth ? 64 : 8;
}
__global__ __launch_bounds__(kBlock) void k_claim_wide(PlanView P, int k, int D) {
  if (budget_spent(P, k)) return;
  const TreeView& T = P.t;
  const int first_new = 1 + first_step(P, k) * P.n_p;
  const int lane = threadIdx.x & 63;
  const int visit_blocks = claim_visit_blocks(P.n_p, D);
  if ((int)blockIdx.x < visit_blocks) {
    const long long n = (long long)D * P.n_p;
    for (long long i = (long long)blockIdx.x * kBlock + threadIdx.x; i < n;
         i += (long long)visit_blocks * kBlock) {
      const int lvl = (int)(i / P.n_p);
      const unsigned long long tk = trace_word(P, k, D, lvl, (int)(i - (long long)lvl * P.n_p));
      if (tk == kEmptyKey) continue;
      const unsigned long long body = tk & ~kTraceClaim;
      const int id = (int)(body >> kActBits);
      if (id == 0) continue;
      const int a = (int)(body & kActMask);
      const uint32_t bit = 1u << (a & 31);
      if (!(atomicOr(&rec_bits(T, id)[a >> 5], bit) & bit)) {
        rec_n(T, id)[a] = 0;
        rec_c(T, id)[a] = 0ull;
        rec_w(T, id)[a] = 0ull;
      }
    }
    return;
  }
  const int per = claim_leaves(P, D);
  const int ep =
      (((int)blockIdx.x - visit_blocks) * (kBlock / 64) + (int)(threadIdx.x >> 6)) * per + lane;
  unsigned long long tk = kEmptyKey;
  if (lane < per && ep < P.n_p) tk = trace_word(P, k, D, D, ep);
  int id = 0;
  uint4 q = make_uint4(0u, 0u, 0u, 0u);
  if (tk != kEmptyKey) {
    id = (tk & kTraceSlot) ? max(T.h_slot[tk & ~kTraceSlot].id, 0) : (int)tk;
    q = *reinterpret_cast<const uint4*>(&T.node[id]);
  }
  // (a leaf at the plan's full depth never draws an action: it needs no row)
  const bool bare = D == P.depth && !(q.y & kLinkAct);
  const bool first = claim_lanes(T, id, q.y, true, bare ? kLinkBare : 0u);
  if (first || (tk != kEmptyKey && (tk & kTraceSlot)))
    T.tr_key[(size_t)D * (size_t)P.n_p + ep] =
        (unsigned long long)(uint32_t)id | (first ? kTraceClaim : 0ull);
  if (first)
    make_full_node(P, id, q.y, __uint_as_float(q.z), own_of(T, id, q.y, P.n_p), id >= first_new);
  const unsigned long long all = __ballot(first && !bare);
  if (!all) return;                             // uniform
  const int a = one_action(q.y, P.m.obs_bits);
  const auto each = [&](auto f) {
    for (unsigned long long m = all; m; m &= m - 1) {
      const int src = __ffsll((long long)m) - 1;
      f((int)__builtin_amdgcn_readlane(id, src), (int)__builtin_amdgcn_readlane(a, src),
        __uint_as_float(__builtin_amdgcn_readlane(q.w, src)));
    }
  };
  // A lane reads N quads of the initial row, then stores them to one belief after
  // the other, so no load waits behind a store.
  constexpr int N = 8;
  const int nq = T.ra / 4;
  for (int i0 = lane; i0 < (nq + 63) / 64 * 64; i0 += 64 * N) {   // uniform
    float4 v[N];
#pragma unroll
    for (int u = 0; u < N; ++u) {
      v[u] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      if (i0 + 64 * u < nq) v[u] = reinterpret_cast<const float4*>(T.psi0)[i0 + 64 * u];
    }
    each([&](int b, int ba, float psi) {
      float4* p = reinterpret_cast<float4*>(rec_psi(T, b));
#pragma unroll
      for (int u = 0; u < N; ++u)
        if (i0 + 64 * u < nq) p[i0 + 64 * u] = with_entry(v[u], i0 + 64 * u, ba, psi);
    });
  }
  each([&](int b, int ba, float) { store_bits<64>(T, b, ba, lane); });
}

__device__ void dev_accum(const PlanView& P, int k, int D, int blk, int nblk, Smem& sm) {
  const TreeView& T = P.t;
  AggTable& G = sm.agg;
  const int per = (P.n_p + kBlock - 1) / kBlock;   // chunks of kBlock items per level
  for (int c = blk; c < (D + 1) * per; c += nblk) {
    const int lvl = c / per;
    const int ep = (c - lvl * per) * kBlock + threadIdx.x;
    unsigned long long tk = kEmptyKey;
    if (ep < P.n_p) tk = trace_word(P, k, D, lvl, ep);
    const bool has = tk != kEmptyKey;
    const bool leaf = lvl == D;
    if (!__syncthreads_or(has)) continue;          // uniform
    // Beliefs that became full join the list of their depth, lvl.
    const bool claimed = has && (tk & kTraceClaim);
    const unsigned long long cm = __ballot(claimed);
    const int wv = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) sm.wave[wv] = (unsigned long long)__popcll(cm);
    const unsigned long long body = tk & ~kTraceClaim;
    int id = (int)(leaf ? body : body >> kActBits);
    if (leaf && has && (body & kTraceSlot))        // (a plan of one level)
      id = max(T.h_slot[body & ~kTraceSlot].id, 0);
    float v = 0.0f;
    if (has) v = T.tr_val[(size_t)lvl * (size_t)P.n_p + ep];
    agg_clear(G);
    __syncthreads();
    if (threadIdx.x == 0) {
      unsigned int n = 0;
      for (int i = 0; i < kBlock / 64; ++i) n += (unsigned int)sm.wave[i];
      sm.n[0] = n ? atomicAdd(&T.full_cnt[lvl], n) : 0u;
      sm.n[1] = n;
    }
    if (has) {
      const unsigned long long key = ((unsigned long long)(uint32_t)id << (kActBits + 1)) |
                                     (leaf ? 1ull : ((body & kActMask) << 1));
      const int sl = agg_slot(G, key);
      atomicAdd(&G.a[sl], 1ull);
      const unsigned long long fx = to_fix(v, P.fix_scale);
      if (fx) atomicAdd(&G.b[sl], fx);
    }
    __syncthreads();
    if (sm.n[1]) {
      if (claimed) {
        unsigned int at = sm.n[0] + (unsigned int)__popcll(cm & ((1ull << (threadIdx.x & 63)) - 1));
        for (int i = 0; i < wv; ++i) at += (unsigned int)sm.wave[i];
        T.full[full_first(P, lvl) + at] = id;
        // (atomic: its own children may become full in this launch, too)
        atomicOr(&T.node[id].link, kLinkFull);
        // (the sweep of long rows does not use it: 10 us a launch there)
        const int up = T.ra <= kMaxA ? (int)(T.info[id].own >> kKeyLowBits) : 0;
        if (up && !(T.node[up].link & kLinkInner)) atomicOr(&T.node[up].link, kLinkInner);
      }
    }
    for (int j = threadIdx.x; j < kAggSlots; j += kBlock) {
      const unsigned long long k2 = G.key[j];
      if (k2 == kEmptyKey) continue;
      const int rid = (int)(k2 >> (kActBits + 1));
      if (k2 & 1ull) {
        atomicAdd(&T.info[rid].leaf_cnt, (int)G.a[j]);
        if (G.b[j]) atomicAdd(&T.node[rid].u.leaf_h, G.b[j]);
      } else if (rid == 0) {
        const int a = (int)((k2 >> 1) & kActMask);
        atomicAdd(root_stripe(T, 0, a), G.a[j]);
        if (G.b[j]) atomicAdd(root_stripe(T, 1, a), G.b[j]);
      } else {
        const int a = (int)((k2 >> 1) & kActMask);
        atomicAdd(&rec_n(T, rid)[a], (int)G.a[j]);
        if (G.b[j]) atomicAdd(&rec_c(T, rid)[a], G.b[j]);
      }
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// Backup (Alg. 3).
// ---------------------------------------------------------------------------

// Adds f to the W accumulator of action `target & kActMask` of belief
// target >> kActBits.
__device__ __forceinline__ void push_one(const TreeView& T, unsigned long long target,
                                         unsigned long long f) {
  const int b = (int)(target >> kActBits), a = (int)(target & kActMask);
  if (b == 0) atomicAdd(root_stripe(T, 2, a), f);
  else atomicAdd(&rec_w(T, b)[a], f);
}

// Pushes of a block into action nodes that it shares: combined in LDS first
// (every thread of the block calls; f = 0: nothing to push).
__device__ __forceinline__ void push_shared(const TreeView& T, AggTable& G,
                                            unsigned long long target, unsigned long long f) {
  if (!__syncthreads_or(f != 0ull)) return;   // uniform: nothing to push
  agg_clear(G);
  __syncthreads();
  if (f) atomicAdd(&G.a[agg_slot(G, target)], f);
  __syncthreads();
  for (int j = threadIdx.x; j < kAggSlots; j += kBlock)
    if (G.key[j] != kEmptyKey && G.a[j]) push_one(T, G.key[j], G.a[j]);
  __syncthreads();
}

// Beliefs of this depth or deeper mostly have distinct parents and push
// directly; shallower ones share a few parents.
constexpr int kPushDirectDepth = 3;

__device__ __forceinline__ unsigned long long push_value(const PlanView& P, float V, int N) {
  return N > 0 ? to_fix(V * (float)N, P.fix_scale) : 0ull;
}
// The action node a belief hangs under, from BeliefInfo::own.
__device__ __forceinline__ unsigned long long parent_of(unsigned long long own, int ob) {
  return ((own >> kKeyLowBits) << kActBits) | ((own & kLinkKey) >> ob);
}

// The full beliefs of one depth: those of a kept subtree (packed at the front
// of the ids), then the list.
struct FullSet {
  int n_kept, n, kept0;
  const int* ids;
};
__device__ __forceinline__ FullSet full_set(const PlanView& P, int dep) {
  FullSet s;
  s.n_kept = P.carry ? P.t.carry_rng[2 * dep + 1] : 0;
  s.kept0 = P.carry ? 1 + P.t.carry_rng[2 * dep] * P.n_p : 0;
  s.n = s.n_kept + (int)P.t.full_cnt[dep];
  s.ids = P.t.full + full_first(P, dep);
  return s;
}
__device__ __forceinline__ int full_id(const FullSet& s, int i) {
  return i < s.n_kept ? s.kept0 + i : s.ids[i - s.n_kept];
}

// Value and visits of full leaf b, read as q and in: with visits in this
// iteration, their mean heuristic and count.
__device__ __forceinline__ void leaf_value(const PlanView& P, int b, const uint4& q,
                                           const BeliefInfo& in, float& V, int& N) {
  const TreeView& T = P.t;
  V = __uint_as_float(q.x);
  N = in.Nb;
  if (in.leaf_cnt > 0) {
    const unsigned long long hs = ((unsigned long long)q.w << 32) | q.z;
    V = from_fix(hs, P.fix_inv) / (float)in.leaf_cnt;
    N = in.leaf_cnt;
    T.node[b].V = V;
    T.info[b].Nb = N;
    T.info[b].leaf_cnt = 0;
    if (hs) T.node[b].u.leaf_h = 0ull;
  }
}

// Full leaves of this iteration take count and mean heuristic; every full
// belief of depth D pushes V*N_b to its parent action.  Beliefs base ..
// base + kBlock - 1 of the set; every thread of the block calls.
__device__ __forceinline__ void full_leaves(const PlanView& P, const FullSet& S, int dep, int base,
                                            Smem& sm) {
  const TreeView& T = P.t;
  const int i = base + threadIdx.x;
  unsigned long long target = 0, f = 0;
  if (i < S.n) {
    // Every field is read before the first store: on CDNA a wait for a
    // load also waits for the stores issued before it.
    const int b = full_id(S, i);
    const uint4 nq = *reinterpret_cast<const uint4*>(&T.node[b]);
    const BeliefInfo in = T.info[b];
    float V;
    int N;
    leaf_value(P, b, nq, in, V, N);
    target = parent_of(in.own, P.m.obs_bits);
    f = push_value(P, V, N);
  }
  if (dep >= kPushDirectDepth) {
    if (f) push_one(T, target, f);
  } else {
    push_shared(T, sm.agg, target, f);
  }
}
__device__ void dev_backup_leaf(const PlanView& P, int dep, int k, int blk, int nblk, Smem& sm) {
  const FullSet S = full_set(P, dep);
  unsigned long long n = 0;
  for (int base = blk * kBlock; base < S.n; base += nblk * kBlock) {
    full_leaves(P, S, dep, base, sm);
    n += min(kBlock, S.n - base);
  }
  if (n && counts_tree(P, k) && threadIdx.x == 0)
    atomicAdd(&stat_bank(P, k)[kStripes + blk % kStripes], n);
}

// The leaves of one item of a plan of one level: run_chunks blocks of runs, one
// unless there are more than kFullCap of them; returns how many.  Every thread
// of the block calls.
__device__ __forceinline__ int run_chunks(const PlanView& P, int k) {
  constexpr int all = kBlock * kFullCap;
  return (k * P.n_p + all - 1) / all;
}
__device__ __forceinline__ int run_items(const PlanView& P, int k) {
  const int per = kBlock * run_chunks(P, k);
  return (k * P.n_p + per - 1) / per;
}
__device__ __forceinline__ int run_leaves(const PlanView& P, int k, int item, Smem& sm) {
  const TreeView& T = P.t;
  const int chunks = run_chunks(P, k);
  int n = 0;
  for (int c = item * chunks; c < (item + 1) * chunks; ++c) {
    const int i = c * kBlock + (int)threadIdx.x;
    bool has = false;
    unsigned long long target = 0, f = 0;
    if (i < k * P.n_p) {
      // All reads at once; of no belief, if the run word says that there is none.
      const int kk = i / P.n_p;
      const int id = 1 + first_step(P, kk + 1) * P.n_p + (i - kk * P.n_p);
      const uint32_t run = T.run[i];
      const uint4 q = *reinterpret_cast<const uint4*>(&T.node[id]);
      const BeliefInfo in = T.info[id];
      has = ((run >> kRunLenShift) & kRunMask) != 0u;
      if (has) {
        float V;
        int N;
        leaf_value(P, id, q, in, V, N);
        target = parent_of(in.own, P.m.obs_bits);
        f = push_value(P, V, N);
      }
    }
    const int m = __syncthreads_count(has);
    if (m) push_shared(T, sm.agg, target, f);   // uniform
    n += m;
  }
  return n;
}

// Iterations of one level over long rows: every run is one leaf, which pushes into
// the root.  A thread each, in the leaf sweep's launch: a launch of the walk for
// them was 9 to 12 us more an iteration of plans of depth 1 (111 to 3,000
// actions).
__device__ void dev_leaf_runs(const PlanView& P, int k, int blk, int nblk, Smem& sm) {
  const TreeView& T = P.t;
  const bool all_full = one_level(P);
  unsigned long long n = 0;
  const long long all = (long long)k * P.n_p;
  for (long long i = (long long)blk * kBlock + threadIdx.x; i < all; i += (long long)nblk * kBlock) {
    const int kk = (int)(i / P.n_p) + 1, ep = (int)(i % P.n_p);
    const int id = 1 + first_step(P, kk) * P.n_p + ep;
    // All reads at once; of no belief, if the run word says that there is none.
    const uint32_t run = T.run[i];
    const uint4 q = *reinterpret_cast<const uint4*>(&T.node[id]);
    const BeliefInfo in = T.info[id];
    if (!((run >> kRunLenShift) & kRunMask)) continue;
    float V = __uint_as_float(q.x);
    int N = 1;
    if (all_full) leaf_value(P, id, q, in, V, N);
    else if (q.y & (kLinkFull | kLinkClaim)) continue;
    const unsigned long long f = push_value(P, V, N);
    if (f) push_one(T, parent_of(in.own, P.m.obs_bits), f);
    ++n;
  }
  n = block_sum(n, sm.wave);
  if (n && counts_tree(P, k) && threadIdx.x == 0)
    atomicAdd(&stat_bank(P, k)[kStripes + blk % kStripes], n);
}

// L_eta Psi of a row whose entry is psi0s[j] but for entry a (a < 0: none),
// in the order of the level sweep's sums.  flat: psi0s is one value (the
// uniform reference policy): one exponential serves the whole row, since the
// weight of the largest entry is exp(0) = 1.  Otherwise, for rows of more than
// 8 actions, the entries' weights against the row's largest are kept in LDS (B)
// and serve every row whose largest entry that still is; the loops stay loops,
// since 64 exponentials written out spilled 724 bytes a thread (a walk of 5
// levels of 40 actions under a prior: a launch took 32 us, now 21).
struct RowBase {
  float m0, m1;              // the largest entry, and the largest besides entry top
  int top;                   // the first of that value
  const float* e0;           // exp(eta (psi0s[j] - m0))
};
template <int AM>
__device__ __forceinline__ float one_row_value(const float (&p0)[AM <= 8 ? AM : 1],
                                               const float* psi0s, int A, int a, float pa,
                                               float eta, bool flat, const RowBase& B) {
  auto at = [&](int j) { return j == a ? pa : (AM <= 8 ? p0[AM <= 8 ? j : 0] : psi0s[j]); };
  float m, se = 0.0f;
  if (flat) {
    const float p = p0[0];
    if (a < 0) pa = p;
    m = A == 1 ? pa : fmaxf(pa, p);
    const float e = expf(eta * (fminf(pa, p) - m));
    const float ep = p == m ? 1.0f : e, ea = pa == m ? 1.0f : e;
#pragma unroll
    for (int j = 0; j < AM; ++j)
      if (j < A) se = se + (j == a ? ea : ep);
  } else if constexpr (AM > 8) {
    m = a < 0 ? B.m0 : fmaxf(a == B.top ? B.m1 : B.m0, pa);
    if (m == B.m0) {
      const float ea = expf(eta * (pa - m));
#pragma unroll 4
      for (int j = 0; j < A; ++j) se = se + (j == a ? ea : B.e0[j]);
    } else {
#pragma unroll 1
      for (int j = 0; j < A; ++j) se = se + expf(eta * (at(j) - m));
    }
  } else {
    m = at(0);
#pragma unroll
    for (int j = 1; j < AM; ++j)
      if (j < A) m = fmaxf(m, at(j));
#pragma unroll
    for (int j = 0; j < AM; ++j)
      if (j < A) se = se + expf(eta * (at(j) - m));
  }
  return m + logf(se) / eta;
}

// The single-visit beliefs: one thread walks the run of one (iteration,
// episode) from its last belief up to the first one or to a full one, holding
// the value that goes up in a register (N = 1 all along), and pushes it into
// the full belief (or the root) above.  Its records are 16 bytes each, read
// and written by consecutive lanes at consecutive addresses, one level at a
// time and kChainAhead levels ahead; the parent of a single-visit belief is
// visited by nothing else in this phase, so there is nothing to wait for.
constexpr int kChainAhead = 4;

template <int AM>
__device__ void dev_chain(const PlanView& P, int k, int blk, int nblk, Smem& sm) {
  const TreeView& T = P.t;
  const int A = P.m.nA, ob = P.m.obs_bits, D = depth_at(P, k);
  const float gamma = P.m.gamma, eta = P.eta;
  stage_psi0(T, sm.psi0);
  constexpr int kRegs = AM <= 8 ? AM : 1;
  float p0[kRegs];
#pragma unroll
  for (int j = 0; j < kRegs; ++j) p0[j] = sm.psi0[j < A ? j : 0];
  bool flat = true;
  for (int j = 1; j < A; ++j) flat = flat && sm.psi0[j] == sm.psi0[0];
  RowBase B{0.0f, 0.0f, 0, sm.e0};
  if constexpr (AM > 8) {
    if (!flat) {                                // uniform
      B.m0 = -INFINITY;
      for (int j = 0; j < A; ++j)
        if (sm.psi0[j] > B.m0) {
          B.m0 = sm.psi0[j];
          B.top = j;
        }
      B.m1 = -INFINITY;
      for (int j = 0; j < A; ++j)
        if (j != B.top) B.m1 = fmaxf(B.m1, sm.psi0[j]);
      if ((int)threadIdx.x < A) sm.e0[threadIdx.x] = expf(eta * (sm.psi0[threadIdx.x] - B.m0));
      __syncthreads();
    }
  }
  const float v0 = one_row_value<AM>(p0, sm.psi0, A, -1, 0.0f, eta, flat, B);
  const int per = (P.n_p + kBlock - 1) / kBlock;
  unsigned long long visits = 0, inner = 0, leaves = 0;
  for (int c = blk; c < k * per; c += nblk) {
    const int kk = c / per + 1;
    const int ep = (c - (kk - 1) * per) * kBlock + threadIdx.x;
    uint32_t run = 0;
    if (ep < P.n_p) run = T.run[(size_t)(kk - 1) * (size_t)P.n_p + ep];
    const int len = (int)((run >> kRunLenShift) & kRunMask);
    const int top = (int)(run & kRunMask) - 1;          // level of its first belief
    unsigned long long target = 0, f = 0;
    int above = D;                                      // depth of what it pushes into
    if (len > 0) {
      const int last = top + len - 1;
      const int id_top = 1 + (first_step(P, kk) + top) * P.n_p + ep;
      bool open = true, first = true;
      float V = 0.0f;
      for (int l0 = last; l0 >= top && open; l0 -= kChainAhead) {
        uint4 q[kChainAhead];
#pragma unroll
        for (int j = 0; j < kChainAhead; ++j) {
          const int l = max(l0 - j, top);
          q[j] = *reinterpret_cast<const uint4*>(&T.node[id_top + (l - top) * P.n_p]);
        }
#pragma unroll
        for (int j = 0; j < kChainAhead; ++j) {
          const int l = l0 - j;
          if (l < top || !open) continue;
          const uint32_t link = q[j].y;
          const int id = id_top + (l - top) * P.n_p;
          const int a = (int)((link & kLinkKey) >> ob);
          if (link & (kLinkFull | kLinkClaim)) {
            // (a run whose last belief is full pushes from the depth sweep)
            if (!first) {
              target = ((unsigned long long)(uint32_t)id << kActBits) | (uint32_t)a;
              f = push_value(P, V, 1);
            }
            above = l + 1;
            open = false;
            continue;
          }
          if (l + 1 == D) ++leaves;
          else ++visits;
          if (link & kLinkAct) {
            // V_curr = L_eta Psi before the update: the stored value, or the
            // initial row's at the first backup.
            const float vc = kk == k ? v0 : __uint_as_float(q[j].x);
            const float r = fix_round(__uint_as_float(q[j].z), P.fix_scale, P.fix_inv);
            const float w = first ? 0.0f : fix_round(V, P.fix_scale, P.fix_inv);
            const float pa = (__uint_as_float(q[j].w) - vc) + (r + gamma * w);
            V = one_row_value<AM>(p0, sm.psi0, A, a, pa, eta, flat, B);
            *reinterpret_cast<uint4*>(&T.node[id]) =
                make_uint4(__float_as_uint(V), link, q[j].z, __float_as_uint(pa));
            ++inner;
          } else {
            V = __uint_as_float(q[j].x);
          }
          first = false;
        }
      }
      if (open) {
        target = parent_of(T.info[id_top].own, ob);
        f = push_value(P, V, 1);
        above = top;
      }
    }
    if (f && above + 1 >= kPushDirectDepth) push_one(T, target, f);
    push_shared(T, sm.agg, target, above + 1 < kPushDirectDepth ? f : 0ull);
  }
  // The sweeps' work over the plan, then the tree statistics.
  const unsigned long long vi = block_sum(visits | (inner << 32), sm.wave);
  const unsigned long long lf = block_sum(leaves, sm.wave);
  if (threadIdx.x == 0) {
    const unsigned long long v = vi & 0xffffffffull, in = vi >> 32;
    unsigned long long* sw = T.stats + (size_t)kStatSweep * kStripes + blk % kStripes;
    if (v) atomicAdd(sw, v);
    if (in) atomicAdd(sw + kStripes, in);
    if (in) atomicAdd(sw + 2 * kStripes, in);
    if (counts_tree(P, k)) {
      unsigned long long* bank = stat_bank(P, k);
      if (in) atomicAdd(&bank[blk % kStripes], in);
      if (v + lf) atomicAdd(&bank[kStripes + blk % kStripes], v + lf);
    }
  }
}

// The trace and the runs in one launch: the two touch nothing in common (the
// walk goes by kLinkClaim, which the search has set), so half of the blocks
// take one and half the other.
__host__ __device__ inline int fold_split(int nblk) { return nblk < 2 ? 0 : (nblk + 1) / 2; }
template <int AM>
__device__ void dev_fold(const PlanView& P, int k, int blk, int nblk, Smem& sm) {
  const int half = fold_split(nblk);
  if (half == 0) {
    dev_accum(P, k, depth_at(P, k), 0, 1, sm);
    dev_chain<AM>(P, k, 0, 1, sm);
  } else if (blk < half) {
    dev_chain<AM>(P, k, blk, half, sm);
  } else {
    dev_accum(P, k, depth_at(P, k), blk - half, nblk - half, sm);
  }
}

// An accumulator that other blocks of the same launch add to, once their adds
// are known to be done (the line may be stale in this XCD's cache).
__device__ __forceinline__ unsigned long long read_shared(const unsigned long long* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

struct SweepCount {
  unsigned long long beliefs, internal, nodes;
};

// Lanes that share a full belief in the sweep below, a quad of its row each.
template <int AM>
constexpr int kRowLanes = AM / 4;

// Full beliefs of depth dep >= 1, base .. base + kBlock / kRowLanes - 1 of the
// set, AM >= |A|.  wait() returns once the deeper depths' adds to W are done;
// every thread of the block calls it, after its other loads are on their way.
// pushed() tells the next depth that this item's adds have arrived; the row's
// stores come after it and take their time beside the next depth's work (10 us
// of 45 for the 89,700 beliefs at depth 2 of nav2d).  V and N_b are kept
// only by the last iteration's sweep, for the caller: a belief with an
// action node computes both anew in every iteration.
//
// Bound by latency and by the requests of rows at random ids, so a row is read
// in 16-byte pieces by as many lanes as it has quads: with a thread per row, a
// row of 40 actions took 24 us a depth, nearly all of it one thread's
// arithmetic.  The exponentials are the lane's own four; every
// lane adds up the row's in action order, so the sums round as before.  Only
// a belief with a full child (kLinkInner) is added to in this launch and
// reads W past the caches after the wait (about 23 G requests/s); the others,
// all but 281 of the 89,700 at depth 2 of nav2d, read it with the rest of the
// row.
template <int AM, typename Wait, typename Done>
__device__ __forceinline__ void full_level(const PlanView& P, const FullSet& S, int dep, int k,
                                           int base, Smem& sm, SweepCount& cnt, Wait wait,
                                           Done pushed) {
  constexpr int kLanes = kRowLanes<AM>;
  const TreeView& T = P.t;
  const int A = P.m.nA;
  const float gamma = P.m.gamma, eta = P.eta, inv = P.fix_inv;
  const int g = (int)threadIdx.x & (kLanes - 1), j0 = 4 * g;
  const int i = base + (int)threadIdx.x / kLanes;
  const bool have = i < S.n;
  const int b = have ? full_id(S, i) : 0;
  const bool mine = have && j0 < A;
  float* prow = rec_psi(T, b) + j0;
  unsigned long long* wrow = rec_w(T, b) + j0;
  BeliefInfo in{0, 0, 0ull};
  float V = 0.0f;
  bool inner = false;
  int n[4] = {0, 0, 0, 0};
  float psi[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  unsigned long long cf[4] = {0, 0, 0, 0}, wf[4] = {0, 0, 0, 0};
  // Two rounds of loads, both before the belief's first store (a wait for a
  // load also waits for the stores issued before it): the parent, value and
  // visit counts, then the rest of the row of a belief with an action node.
  if (have) {
    in = T.info[b];
    const uint2 q = *reinterpret_cast<const uint2*>(&T.node[b]);
    V = __uint_as_float(q.x);
    inner = i < S.n_kept || (q.y & kLinkInner) != 0u;
    if (mine) {
      const int4 c = *reinterpret_cast<const int4*>(rec_n(T, b) + j0);
      n[0] = c.x; n[1] = c.y; n[2] = c.z; n[3] = c.w;
    }
  }
  int N = in.Nb;
  bool vis[4];
  int nsum = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    vis[j] = j0 + j < A && n[j] > 0;
    nsum += vis[j] ? n[j] : 0;
  }
#pragma unroll
  for (int off = kLanes / 2; off > 0; off >>= 1) nsum += __shfl_xor(nsum, off, 64);
  const bool any = nsum > 0;
  if (any && mine) {
    const float4 q = *reinterpret_cast<const float4*>(prow);
    psi[0] = q.x; psi[1] = q.y; psi[2] = q.z; psi[3] = q.w;
    const ulonglong2* c2 = reinterpret_cast<const ulonglong2*>(rec_c(T, b) + j0);
    const ulonglong2 c01 = c2[0], c23 = c2[1];
    cf[0] = c01.x; cf[1] = c01.y; cf[2] = c23.x; cf[3] = c23.y;
    if (!inner) {
      const ulonglong2* w2 = reinterpret_cast<const ulonglong2*>(wrow);
      const ulonglong2 w01 = w2[0], w23 = w2[1];
      wf[0] = w01.x; wf[1] = w01.y; wf[2] = w23.x; wf[3] = w23.y;
    }
  }
  // Sum over the row in action order, in every lane of the row.
  auto row_sum = [&](const float (&e)[4]) {
    float se = 0.0f;
    if constexpr (kLanes == 1) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (j < A) se = se + e[j];
    } else {
      const int l0 = ((int)threadIdx.x & 63) - g;
      for (int q = 0; 4 * q < A; ++q) {
        float x[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) x[j] = __shfl(e[j], l0 + q, 64);
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (4 * q + j < A) se = se + x[j];
      }
    }
    return se;
  };
  // L_eta of the row.
  auto row_value = [&]() {
    float m = -INFINITY;
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (j0 + j < A) m = fmaxf(m, psi[j]);
#pragma unroll
    for (int off = kLanes / 2; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
    float e[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) e[j] = j0 + j < A ? expf(eta * (psi[j] - m)) : 0.0f;
    return m + logf(row_sum(e)) / eta;
  };
  wait();
  unsigned long long target = 0, f = 0;
  if (any) {
    if (inner) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (vis[j]) wf[j] = read_shared(wrow + j);
    }
    // V_curr = L_eta Psi (Eq. 3) before the update.
    const float vc = row_value();
    // Q = C/N + gamma W with W = sum_children V N_b / N; Psi <- Psi - V_curr + Q.
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (vis[j]) {
        const float c = from_fix(cf[j], inv);
        const float w = from_fix(wf[j], inv);
        const float fn = (float)n[j];
        const float q = c / fn + gamma * (w / fn);
        psi[j] = (psi[j] - vc) + q;
        ++cnt.nodes;
      }
    }
    // V = L_eta Psi after the update; N_b = sum_a N(b, a).
    V = row_value();
    N = nsum;
  }
  if (have && g == 0) {
    target = parent_of(in.own, P.m.obs_bits);
    f = push_value(P, V, N);
    ++cnt.beliefs;
    if (any) ++cnt.internal;
  }
  if (dep >= kPushDirectDepth) {
    if (f) push_one(T, target, f);
  } else {
    push_shared(T, sm.agg, target, f);
  }
  pushed();
  if (any && mine) {
    *reinterpret_cast<float4*>(prow) = make_float4(psi[0], psi[1], psi[2], psi[3]);
    // W is rebuilt by the children's pushes of the next iteration.
    ulonglong2* w2 = reinterpret_cast<ulonglong2*>(wrow);
    if ((vis[0] && wf[0]) || (vis[1] && wf[1])) w2[0] = make_ulonglong2(0ull, 0ull);
    if ((vis[2] && wf[2]) || (vis[3] && wf[3])) w2[1] = make_ulonglong2(0ull, 0ull);
    if (g == 0 && counts_tree(P, k)) {
      T.node[b].V = V;
      T.info[b].Nb = N;
    }
  }
}

template <int AM, typename Wait>
__device__ void dev_backup_root(const PlanView& P, int k, Smem& sm, Wait wait);

// The full beliefs of every depth and the root, in one launch.  Blocks take
// items (a block's beliefs of one depth; the root last) from a counter, deepest
// depth first; an item waits until every item of the deeper depths is done,
// with everything but W already read.  Items are taken in that order by blocks
// that run, so whatever the residency the lowest unfinished item waits for
// nothing.  Only the W accumulators pass from one depth to the next: they are
// added to and read past the caches, so an item needs no cache write-back or
// invalidation, only its own adds to have arrived.  Most depths hold no full
// belief: they cost nothing here and about 4.4 us each as a launch of their
// own (nav2d, depth 10: nine of them and the root's, in every iteration).
template <int AM, bool ONE>
__device__ void dev_full(const PlanView& P, int k, int blk, Smem& sm) {
  const TreeView& T = P.t;
  const int D = depth_at(P, k);
  const int lane = threadIdx.x & 63;
  const FullSet leaves = full_set(P, D);
  const int n_set = (leaves.n + kBlock - 1) / kBlock;
  // (a plan of one level: its own leaves by the run words, after the kept ones)
  const int n_leaf = n_set + (ONE ? run_items(P, k) : 0);
  // Lane l: the first item of depth D - 1 - l; lane D - 1: the root's.
  const int my_dep = D - 1 - lane;
  int n = 0;
  constexpr int per = kBlock / kRowLanes<AM>;     // beliefs of a level's item
  if (my_dep >= 1) n = (full_set(P, my_dep).n + per - 1) / per;
  int start = n_leaf + (int)wave_incl_scan((unsigned long long)n) - n;
  if (my_dep < 0) start = INT_MAX;
  SweepCount cnt{0, 0, 0};
  unsigned long long leaf_cnt = 0;
  for (;;) {
    if (threadIdx.x == 0) sm.n[0] = (unsigned int)atomicAdd(&T.counters[2], 1ull);
    __syncthreads();
    const int item = (int)sm.n[0];
    const int l = __popcll(__ballot(start <= item)) - 1;
    const int first = l < 0 ? 0 : __shfl(start, l, 64);
    const int dep = D - 1 - l;                    // D: the leaves
    if (dep == 0 && item > first) break;          // past the root: uniform
    auto wait = [&]() {
      if (threadIdx.x == 0 && first > 0) {
        uint32_t turns = 0;
        while (read_shared(&T.counters[3]) < (unsigned long long)first) {
          if (wait_over(P, ++turns)) {            // ends every wait of this launch
            atomicOr((unsigned int*)&T.counters[1], kErrWait);
            atomicAdd(&T.counters[3], 1ull << 32);
          } else {
            __builtin_amdgcn_s_sleep(1);
          }
        }
      }
      __syncthreads();
    };
    if (dep == 0) {
      dev_backup_root<AM>(P, k, sm, wait);
      break;
    }
    auto pushed = [&]() {
      stores_done();                              // this wavefront's adds
      __syncthreads();
      if (threadIdx.x == 0) atomicAdd(&T.counters[3], 1ull);
    };
    if (dep == D) {
      if (!ONE || item < n_set) {
        full_leaves(P, leaves, D, item * kBlock, sm);
        leaf_cnt += min(kBlock, leaves.n - item * kBlock);
      } else {
        leaf_cnt += run_leaves(P, k, item - n_set, sm);
      }
      pushed();
    } else if constexpr (!ONE) {
      full_level<AM>(P, full_set(P, dep), dep, k, (item - first) * per, sm, cnt, wait, pushed);
    }
  }
  __syncthreads();
  // The sweep's work over the plan (every iteration), then the tree
  // statistics (the last iteration).  A block visits fewer than 2^32 beliefs.
  const unsigned long long vi = block_sum(cnt.beliefs | (cnt.internal << 32), sm.wave);
  const unsigned long long nd = block_sum(cnt.nodes, sm.wave);
  if (threadIdx.x == 0) {
    unsigned long long* sw = T.stats + (size_t)kStatSweep * kStripes + blk % kStripes;
    if (vi & 0xffffffffull) atomicAdd(sw, vi & 0xffffffffull);
    if (vi >> 32) atomicAdd(sw + kStripes, vi >> 32);
    if (nd) atomicAdd(sw + 2 * kStripes, nd);
    if (counts_tree(P, k)) {
      unsigned long long* bank = stat_bank(P, k);
      const unsigned long long nb = (vi & 0xffffffffull) + leaf_cnt;
      if (nd) atomicAdd(&bank[blk % kStripes], nd);
      if (nb) atomicAdd(&bank[kStripes + blk % kStripes], nb);
    }
  }
}

// Anytime plan (Alg. 1 loops while the budget lasts), run by the first
// wavefront of the root backup: this iteration's backups are done; the next
// one runs only if time is left and K is not reached.  The decision goes to
// the later phases (gate) and to the host, which stops enqueueing.
__device__ __forceinline__ void root_gate(const PlanView& P, int k, int lane) {
  if (!P.timed) return;
  unsigned long long* next = stat_bank(P, k + 1);
  next[lane] = 0ull;
  next[kStripes + lane] = 0ull;
  if (lane == 0) {
    const unsigned long long now = (unsigned long long)wall_clock64();
    const unsigned long long stop =
        (k >= P.K || now - P.t.gate[0] >= P.budget_ticks) ? 1ull : 0ull;
    P.t.gate[1] = stop ? (unsigned long long)k : 0ull;
    P.t.gate[2] = (unsigned long long)k;
    __hip_atomic_store(P.gate_host, (unsigned long long)k | (stop << 32), __ATOMIC_RELEASE,
                       __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

// ---------------------------------------------------------------------------
// Sweeps for long action rows (|A| > kMaxA): one wavefront per belief; lane l
// holds the quads l, l + 64, ... of the row.
// ---------------------------------------------------------------------------
__device__ __forceinline__ double wave_max64(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off, 64));
  return v;
}

__device__ __forceinline__ float wave_maxf(float v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = fmaxf(v, __shfl_xor(v, off, 64));
  return v;
}
__device__ __forceinline__ float wave_sumf(float v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// Level sweep of the internal beliefs of depth dep-1 >= 1 (Alg. 3, Eq. 3, 5)
// over long rows, one wavefront per belief.  Lane l holds the quads l,
// l + 64, ... of the row (QPL of them; the padding past |A| and quads past the
// row masked off) in registers for the whole update, so a belief costs one
// batch of loads for Psi, N and its metadata, one batch of C and W loads per
// four quads of the lane, and the stores at the end: no load waits behind a
// store of the same belief.
template <int QPL>
__device__ void dev_backup_level_wide(const PlanView& P, int dep, int k, int blk, int nblk,
                                      Smem& sm) {
  static_assert(QPL % 4 == 0 && 4 * QPL <= 64, "quads per lane");
  const TreeView& T = P.t;
  const FullSet S = full_set(P, dep - 1);
  const int A = P.m.nA;
  const int nq = T.ra / 4;
  const float gamma = P.m.gamma, eta = P.eta, inv = P.fix_inv;
  const int lane = threadIdx.x & 63;
  const int waves = kBlock / 64;
  unsigned long long nodes = 0, beliefs = 0;  // tree statistics (lane 0 counts)
  unsigned long long internal = 0;            // beliefs with an action node
  {
    for (int i = blk * waves + (int)(threadIdx.x >> 6); i < S.n; i += nblk * waves) {
      // b is uniform: addresses are a scalar base plus 32-bit lane offsets.
      const int b = __builtin_amdgcn_readfirstlane(full_id(S, i));
      const float4* p4 = reinterpret_cast<const float4*>(rec_psi(T, b));
      const uint32_t* bits = rec_bits(T, b);
      const int* nrow = rec_n(T, b);
      const unsigned long long* crow = rec_c(T, b);
      unsigned long long* wrow = rec_w(T, b);
      // Psi and the visited flags (the bitmap's nibble of each quad).
      float pf[4 * QPL];
      uint32_t vb[QPL];
#pragma unroll
      for (int i = 0; i < QPL; ++i) {
        const int q = lane + 64 * i;
        float4 v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        uint32_t w = 0u;
        if (q < nq) {
          v = p4[q];
          w = bits[q >> 3];
        }
        pf[4 * i] = v.x; pf[4 * i + 1] = v.y; pf[4 * i + 2] = v.z; pf[4 * i + 3] = v.w;
        vb[i] = w;
      }
      // Read after the row: these uniform values are moved to scalar
      // registers at once, which waits for them.
      const float V0 = T.node[b].V;
      const int N0 = T.info[b].Nb;
      const unsigned long long own = T.info[b].own;
#pragma unroll
      for (int i = 0; i < QPL; ++i) vb[i] = (vb[i] >> (4 * ((lane + 64 * i) & 7))) & 15u;
      bool vis = false;                         // padding is never visited
#pragma unroll
      for (int i = 0; i < QPL; ++i) vis = vis || vb[i] != 0u;
      float V;
      int N;
      const bool upd = __any(vis);
      unsigned long long clear = 0ull;          // W entries to clear (bit per action)
      uint32_t changed = 0u;                    // quads of Psi to store
      if (upd) {
        // V_curr = L_eta Psi (Eq. 3) before the update.
        float m = -INFINITY;
#pragma unroll
        for (int i = 0; i < 4 * QPL; ++i)
          if (4 * (lane + 64 * (i >> 2)) + (i & 3) < A) m = fmaxf(m, pf[i]);
        m = wave_maxf(m);
        float se = 0.0f;
#pragma unroll
        for (int i = 0; i < 4 * QPL; ++i)
          if (4 * (lane + 64 * (i >> 2)) + (i & 3) < A) se = se + expf(eta * (pf[i] - m));
        const float vc = m + logf(wave_sumf(se)) / eta;
        // Psi <- Psi - V_curr + Q, Q = C/N + gamma W/N (Eq. 5), for visited
        // actions.  An unvisited action reads the belief's info instead (read
        // above), so the loads issue without branches.
        const int* spare_n = &T.info[b].Nb;
        const unsigned long long* spare_l = &T.info[b].own;
        int nsum = 0, nn = 0;
#pragma unroll
        for (int i0 = 0; i0 < QPL; i0 += 4) {
          unsigned long long cf[16], wf[16];
          int nf[16];
#pragma unroll
          for (int t = 0; t < 16; ++t) {
            const int i = 4 * i0 + t;
            const int j = 4 * (lane + 64 * (i >> 2)) + (i & 3);
            const bool v = (vb[i >> 2] >> (i & 3)) & 1u;
            nf[t] = *(v ? nrow + j : spare_n);
            cf[t] = *(v ? crow + j : spare_l);
            wf[t] = *(v ? wrow + j : spare_l);
          }
#pragma unroll
          for (int t = 0; t < 16; ++t) {
            asm volatile("" : "+v"(nf[t]));
            asm volatile("" : "+v"(cf[t]));
            asm volatile("" : "+v"(wf[t]));
          }
#pragma unroll
          for (int t = 0; t < 16; ++t) {
            const int i = 4 * i0 + t;
            if (((vb[i >> 2] >> (i & 3)) & 1u) && nf[t] > 0) {
              const float cv = from_fix(cf[t], inv);
              const float w = from_fix(wf[t], inv);
              const float fn = (float)nf[t];
              pf[i] = (pf[i] - vc) + (cv / fn + gamma * (w / fn));
              nsum += nf[t];
              ++nn;
              changed |= 1u << (i >> 2);
              if (wf[t]) clear |= 1ull << i;
            }
          }
        }
        // V = L_eta Psi after the update; N_b = sum_a N(b, a).
        float m2 = -INFINITY;
#pragma unroll
        for (int i = 0; i < 4 * QPL; ++i)
          if (4 * (lane + 64 * (i >> 2)) + (i & 3) < A) m2 = fmaxf(m2, pf[i]);
        m2 = wave_maxf(m2);
        float se2 = 0.0f;
#pragma unroll
        for (int i = 0; i < 4 * QPL; ++i)
          if (4 * (lane + 64 * (i >> 2)) + (i & 3) < A) se2 = se2 + expf(eta * (pf[i] - m2));
        V = m2 + logf(wave_sumf(se2)) / eta;
        N = (int)wave_sum((unsigned long long)nsum);
        nodes += wave_sum((unsigned long long)nn);
        ++internal;
      } else {
        V = V0;
        N = N0;
      }
      if (lane == 0) {
        ++beliefs;
        const unsigned long long f = push_value(P, V, N);
        if (f) push_one(T, parent_of(own, P.m.obs_bits), f);
      }
      // The record's stores come last, so that nothing above waits for them.
      if (upd) {
        T.node[b].V = V;                        // the same value in every lane
        T.info[b].Nb = N;
        float4* pw4 = reinterpret_cast<float4*>(rec_psi(T, b));
#pragma unroll
        for (int i = 0; i < QPL; ++i)
          if ((changed >> i) & 1u)
            pw4[lane + 64 * i] = make_float4(pf[4 * i], pf[4 * i + 1], pf[4 * i + 2], pf[4 * i + 3]);
#pragma unroll
        for (int i = 0; i < 4 * QPL; ++i)
          if ((clear >> i) & 1ull) wrow[4 * (lane + 64 * (i >> 2)) + (i & 3)] = 0ull;
      }
    }
  }
  if (lane == 0) {
    unsigned long long* sw = T.stats + (size_t)kStatSweep * kStripes + blk % kStripes;
    if (beliefs) atomicAdd(sw, beliefs);
    if (internal) atomicAdd(sw + kStripes, internal);
    if (nodes) atomicAdd(sw + 2 * kStripes, nodes);
    if (counts_tree(P, k)) {
      unsigned long long* bank = stat_bank(P, k);
      if (nodes) atomicAdd(&bank[blk % kStripes], nodes);
      if (beliefs) atomicAdd(&bank[kStripes + blk % kStripes], beliefs);
    }
  }
}

// The single-visit beliefs of long rows (dev_chain), one wavefront per run,
// kWideRuns runs of one iteration per wavefront: the lanes hold the initial row
// in registers and evaluate L_eta of it with one entry replaced, in the order
// of the level sweep, so no row is read or written.  The records of the runs
// are read by the lanes together, kChainAhead levels at a time.
constexpr int kWideRuns = 16;

template <int QPL>
__device__ __forceinline__ float wave_row_value(const float (&p0)[4 * QPL], int A, int a, float pa,
                                                float eta, int lane) {
  float m = -INFINITY;
#pragma unroll
  for (int i = 0; i < 4 * QPL; ++i) {
    const int j = 4 * (lane + 64 * (i >> 2)) + (i & 3);
    if (j < A) m = fmaxf(m, j == a ? pa : p0[i]);
  }
  m = wave_maxf(m);
  float se = 0.0f;
#pragma unroll
  for (int i = 0; i < 4 * QPL; ++i) {
    const int j = 4 * (lane + 64 * (i >> 2)) + (i & 3);
    if (j < A) se = se + expf(eta * ((j == a ? pa : p0[i]) - m));
  }
  return m + logf(wave_sumf(se)) / eta;
}

template <int QPL>
__device__ void dev_chain_wide(const PlanView& P, int k, int blk, int nblk) {
  const TreeView& T = P.t;
  const int A = P.m.nA, ob = P.m.obs_bits, D = depth_at(P, k);
  const int nq = T.ra / 4;
  const float gamma = P.m.gamma, eta = P.eta;
  const int lane = threadIdx.x & 63;
  const int waves = kBlock / 64;
  float p0[4 * QPL];
#pragma unroll
  for (int i = 0; i < QPL; ++i) {
    float4 v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (lane + 64 * i < nq) v = reinterpret_cast<const float4*>(T.psi0)[lane + 64 * i];
    p0[4 * i] = v.x; p0[4 * i + 1] = v.y; p0[4 * i + 2] = v.z; p0[4 * i + 3] = v.w;
  }
  const float v0 = wave_row_value<QPL>(p0, A, -1, 0.0f, eta, lane);
  unsigned long long visits = 0, inner = 0, leaves = 0;
  const int per = (P.n_p + kWideRuns - 1) / kWideRuns;
  for (int c = blk * waves + (int)(threadIdx.x >> 6); c < k * per; c += nblk * waves) {
    const int kk = c / per + 1;
    const int ep = (c - (kk - 1) * per) * kWideRuns + lane;
    uint32_t run = 0;
    if (lane < kWideRuns && ep < P.n_p) run = T.run[(size_t)(kk - 1) * (size_t)P.n_p + ep];
    const int my_len = (int)((run >> kRunLenShift) & kRunMask);
    const int my_top = (int)(run & kRunMask) - 1;
    const int my_id = 1 + (first_step(P, kk) + my_top) * P.n_p + ep;   // its first belief
    uint4 q[kChainAhead];
#pragma unroll
    for (int j = 0; j < kChainAhead; ++j)
      q[j] = my_len > 0 ? *reinterpret_cast<const uint4*>(
                              &T.node[my_id + max(my_len - 1 - j, 0) * P.n_p])
                        : make_uint4(0u, 0u, 0u, 0u);
    // A run that is a leaf only needs no row: a lane each, all at once.
    const bool leaf_only = my_len == 1 && !(q[0].y & kLinkAct);
    const bool push = leaf_only && !(q[0].y & (kLinkFull | kLinkClaim));
    if (push) {
      const unsigned long long f = push_value(P, __uint_as_float(q[0].x), 1);
      if (f) push_one(T, parent_of(T.info[my_id].own, ob), f);
    }
    const unsigned long long n_push = (unsigned long long)__popcll(__ballot(push));
    // (every run of iteration kk that is one leaf is at the depth of its leaves)
    if (depth_at(P, kk) == D) leaves += n_push;
    else visits += n_push;
    unsigned long long todo = __ballot(my_len > 0 && !leaf_only);
    while (todo) {
      const int src = __ffsll((long long)todo) - 1;
      todo &= todo - 1;
      const int len = __builtin_amdgcn_readfirstlane(__shfl(my_len, src, 64));
      const int top = __builtin_amdgcn_readfirstlane(__shfl(my_top, src, 64));
      const int id_top = __builtin_amdgcn_readfirstlane(__shfl(my_id, src, 64));
      unsigned long long target = 0, f = 0;
      bool open = true, first = true;
      float V = 0.0f;
      for (int i0 = len - 1; i0 >= 0 && open; i0 -= kChainAhead) {
#pragma unroll
        for (int j = 0; j < kChainAhead; ++j) {
          const int i = i0 - j;
          if (i < 0 || !open) continue;
          const int id = id_top + i * P.n_p;
          uint4 n;
          if (i0 == len - 1) {
            n = make_uint4(__shfl(q[j].x, src, 64), __shfl(q[j].y, src, 64),
                           __shfl(q[j].z, src, 64), __shfl(q[j].w, src, 64));
          } else {
            n = *reinterpret_cast<const uint4*>(&T.node[id]);
          }
          const uint32_t link = __builtin_amdgcn_readfirstlane(n.y);
          const int a = (int)((link & kLinkKey) >> ob);
          if (link & (kLinkFull | kLinkClaim)) {
            if (!first) {
              target = ((unsigned long long)(uint32_t)id << kActBits) | (uint32_t)a;
              f = push_value(P, V, 1);
            }
            open = false;
            continue;
          }
          if (top + i + 1 == D) ++leaves;
          else ++visits;
          if (link & kLinkAct) {
            const float vc = kk == k ? v0 : __uint_as_float(n.x);
            const float r = fix_round(__uint_as_float(n.z), P.fix_scale, P.fix_inv);
            const float w = first ? 0.0f : fix_round(V, P.fix_scale, P.fix_inv);
            const float pa = (__uint_as_float(n.w) - vc) + (r + gamma * w);
            V = wave_row_value<QPL>(p0, A, a, pa, eta, lane);
            if (lane == 0)
              *reinterpret_cast<uint4*>(&T.node[id]) =
                  make_uint4(__float_as_uint(V), link, n.z, __float_as_uint(pa));
            ++inner;
          } else {
            V = __uint_as_float(n.x);
          }
          first = false;
        }
      }
      if (open && lane == 0) {
        target = parent_of(T.info[id_top].own, ob);
        f = push_value(P, V, 1);
      }
      if (f && lane == 0) push_one(T, target, f);
    }
  }
  if (lane == 0) {
    unsigned long long* sw = T.stats + (size_t)kStatSweep * kStripes + blk % kStripes;
    if (visits) atomicAdd(sw, visits);
    if (inner) atomicAdd(sw + kStripes, inner);
    if (inner) atomicAdd(sw + 2 * kStripes, inner);
    if (counts_tree(P, k)) {
      unsigned long long* bank = stat_bank(P, k);
      if (inner) atomicAdd(&bank[blk % kStripes], inner);
      if (visits + leaves) atomicAdd(&bank[kStripes + blk % kStripes], visits + leaves);
    }
  }
}

__device__ double block_max64(double v, double* red) {
  v = wave_max64(v);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double r = red[0];
  for (int i = 1; i < kBlock / 64; ++i) r = fmax(r, red[i]);
  __syncthreads();
  return r;
}

// Running sums over a = 0 .. A-1 of exp(eta (x_a - m)), by a block scan over
// chunks of kBlock actions (wavefront scans, then the wavefront totals); with
// cdf set they are stored.  Every thread calls; all get the total.  The scan
// adds in a tree order rather than the serial one: the sums differ from the
// serial definition's by a few units in the last place (about 1e-15
// relative), far below the margin at which a root draw counts as a near tie.
__device__ double block_ordered_sum(const double* x, int A, double m, double eta, double* cdf,
                                    double* buf, double* bc) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  double carry = 0.0;
  for (int base = 0; base < A; base += kBlock) {
    const int j = base + (int)threadIdx.x;
    double v = j < A ? exp(eta * (x[j] - m)) : 0.0;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const double o = __shfl_up(v, off, 64);
      if (lane >= off) v += o;
    }
    if (lane == 63) buf[wv] = v;
    __syncthreads();
    double before = carry;
    for (int w = 0; w < wv; ++w) before += buf[w];
    double total = carry;
    for (int w = 0; w < kBlock / 64; ++w) total += buf[w];
    if (cdf && j < A) cdf[j] = before + v;
    carry = total;
    __syncthreads();
  }
  (void)bc;
  return carry;
}

// Running sums, in the order of block_ordered_sum, of exp(eta (x - m)) for a
// row whose entry j = i*kBlock + threadIdx.x is x[i] of the calling thread
// (held in registers); with cdf set they are stored.  Every thread calls;
// all get the total.
template <int PER>
__device__ double block_ordered_sum_regs(const double (&x)[PER], int A, double m, double eta,
                                         double* cdf, double* buf) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  double carry = 0.0;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int base = i * kBlock;
    if (base >= A) break;                       // uniform
    const int j = base + (int)threadIdx.x;
    double v = j < A ? exp(eta * (x[i] - m)) : 0.0;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const double o = __shfl_up(v, off, 64);
      if (lane >= off) v += o;
    }
    if (lane == 63) buf[wv] = v;
    __syncthreads();
    double before = carry;
    for (int w = 0; w < wv; ++w) before += buf[w];
    double total = carry;
    for (int w = 0; w < kBlock / 64; ++w) total += buf[w];
    if (cdf && j < A) cdf[j] = before + v;
    carry = total;
    __syncthreads();
  }
  return carry;
}

// The root row (|A| > kMaxA) in double precision, by one block.  Thread t
// holds actions t, t + kBlock, ... of the row and of the root's sums (one
// stripe for long rows) in registers: one batch of loads, the update and its
// sums (in the order of block_ordered_sum), then the stores, so that no load
// waits behind a store.
__device__ void dev_backup_root_wide(const PlanView& P, int k, double* buf) {
  constexpr int PER = kMaxAWide / kBlock;
  const TreeView& T = P.t;
  const int A = P.m.nA;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const double eta = P.eta64;
  __shared__ double red[kBlock / 64];
  __shared__ unsigned long long cnt[2];
  if (wv == 0) root_gate(P, k, lane);
  if (threadIdx.x == 0) { cnt[0] = 0ull; cnt[1] = 0ull; }
  double* psi = T.psi_root;
  double pv[PER];
  int nv[PER];
  unsigned long long cv[PER], wv64[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int j = i * kBlock + (int)threadIdx.x;
    pv[i] = -INFINITY;
    nv[i] = 0;
    cv[i] = 0ull;
    wv64[i] = 0ull;
    if (j < A) {
      pv[i] = psi[j];
      nv[i] = (int)T.root_acc[((size_t)0 * T.ra + j) * kStripes];
      cv[i] = T.root_acc[((size_t)1 * T.ra + j) * kStripes];
      wv64[i] = T.root_acc[((size_t)2 * T.ra + j) * kStripes];
    }
  }
  double mloc = -INFINITY;
  unsigned long long nodes = 0, nsum = 0;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    mloc = fmax(mloc, pv[i]);
    nodes += nv[i] > 0 ? 1ull : 0ull;
    nsum += (unsigned long long)(nv[i] > 0 ? nv[i] : 0);
  }
  nodes = wave_sum(nodes);
  nsum = wave_sum(nsum);
  __syncthreads();                              // cnt cleared
  if (lane == 0) {
    atomicAdd(&cnt[0], nodes);
    atomicAdd(&cnt[1], nsum);
  }
  const double m = block_max64(mloc, red);
  const bool any = cnt[0] != 0ull;              // uniform: an action node exists
  double vc = 0.0, mm = 0.0, run = 0.0;
  if (any) {
    // V_curr = L_eta Psi before the update (Eq. 3).
    vc = m + log(block_ordered_sum_regs<PER>(pv, A, m, eta, nullptr, buf)) / eta;
    // Psi <- Psi - V_curr + Q for the actions with an action node (Eq. 5).
    double m2 = -INFINITY;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      if (nv[i] > 0) {
        const double c = (double)(long long)cv[i] * P.fix_inv64;
        const double w = (double)(long long)wv64[i] * P.fix_inv64;
        pv[i] = (pv[i] - vc) + (c / (double)nv[i] + P.m.gamma64 * (w / (double)nv[i]));
      }
      m2 = fmax(m2, pv[i]);
    }
    mm = block_max64(m2, red);
    // V = L_eta Psi after the update, and the running sums of the root draw.
    run = block_ordered_sum_regs<PER>(pv, A, mm, eta, T.root_cdf, buf);
  }
  // The root record's columns (N, C, W) and the updated row; W's stripe is
  // cleared for the next iteration.
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int j = i * kBlock + (int)threadIdx.x;
    if (j < A) {
      rec_n(T, 0)[j] = nv[i];
      rec_c(T, 0)[j] = cv[i];
      rec_w(T, 0)[j] = wv64[i];
      T.root_acc[((size_t)2 * T.ra + j) * kStripes] = 0ull;
      if (any && nv[i] > 0) psi[j] = pv[i];
    }
  }
  if (any && threadIdx.x == 0) {
    const double v = mm + log(run) / eta;
    T.v_root[0] = v;
    T.node[0].V = (float)v;
    T.info[0].Nb = (int)cnt[1];
    if (counts_tree(P, k)) atomicAdd(&stat_bank(P, k)[0], cnt[0]);
  }
}

// The root row in double precision, updated in place, by one block (rows of up
// to kMaxA actions).  Sixteen lanes sum the 64 stripes of one of the 3|A| sums
// (N, C, W of each action); lane j of the first wavefront then owns action j:
// it evaluates that action's exponentials, and every lane adds them up in
// action order (the order of the serial definition, so every sum rounds
// exactly as it would there).

// Lane j's value in every lane (j uniform).
__device__ __forceinline__ double lane_value(double x, int j) {
  const unsigned long long v = (unsigned long long)__double_as_longlong(x);
  const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)v, j);
  const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(v >> 32), j);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
// Sum of x over lanes 0..A-1 in lane order; upto: the sum up to this lane.
__device__ __forceinline__ double ordered_sum(double x, int A, double& upto) {
  const int lane = threadIdx.x & 63;
  double s = 0.0;
  for (int j = 0; j < A; ++j) {
    s = s + lane_value(x, j);
    if (lane == j) upto = s;
  }
  return s;
}

template <int AM, typename Wait>
__device__ void dev_backup_root(const PlanView& P, int k, Smem& sm, Wait wait) {
  const TreeView& T = P.t;
  const int A = P.m.nA;
  double p_me = -INFINITY;
  if ((int)threadIdx.x < A) p_me = T.psi_root[threadIdx.x];
  static_assert(3 * kMaxA <= kAggSlots && kStripes == 64, "sums fit the table");
  unsigned long long* sums = sm.agg.a;          // [3][A]
  // Sums first .. first + n - 1 of them; every load is issued before the first
  // is waited for (40 actions, one after the other: 8 us of the root's 13).
  auto stripes = [&](auto rounds, int first, int n, auto read) {
    constexpr int R = decltype(rounds)::value;
    unsigned long long v[R][4];
#pragma unroll
    for (int x = 0; x < R; ++x) {
      const int r = x * (kBlock / 16) + (int)threadIdx.x / 16;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        v[x][i] = 0;
        if (r < n) {
          const int q = (first + r) / A, a = first + r - q * A;
          v[x][i] = read(T.root_acc + ((size_t)q * T.ra + a) * kStripes + (threadIdx.x & 15) + 16 * i);
        }
      }
    }
#pragma unroll
    for (int x = 0; x < R; ++x) {
      const int r = x * (kBlock / 16) + (int)threadIdx.x / 16;
      unsigned long long t = (v[x][0] + v[x][1]) + (v[x][2] + v[x][3]);
#pragma unroll
      for (int off = 8; off > 0; off >>= 1) t += __shfl_xor(t, off, 16);
      if (r < n && (threadIdx.x & 15) == 0) sums[first + r] = t;
    }
  };
  constexpr int kPer = kBlock / 16;             // sums of one round
  // N and C were added to in earlier launches, W in this one.
  stripes(std::integral_constant<int, (2 * AM + kPer - 1) / kPer>{}, 0, 2 * A,
          [](const unsigned long long* p) { return *p; });
  wait();
  stripes(std::integral_constant<int, (AM + kPer - 1) / kPer>{}, 2 * A, A,
          [](const unsigned long long* p) { return read_shared(p); });
  __syncthreads();
  for (int r = threadIdx.x; r < A * kStripes; r += kBlock)
    T.root_acc[(size_t)2 * T.ra * kStripes + r] = 0ull;
  if (threadIdx.x >= 64) return;
  const int lane = threadIdx.x;
  root_gate(P, k, lane);
  const bool act = lane < A;
  const long long n_me = act ? (long long)sums[lane] : 0;
  const long long c_me = act ? (long long)sums[A + lane] : 0;
  const long long w_me = act ? (long long)sums[2 * A + lane] : 0;
  double* psi = T.psi_root;
  const double eta = P.eta64;
  if (act) {                                  // belief 0 keeps the totals
    rec_n(T, 0)[lane] = (int)n_me;
    rec_c(T, 0)[lane] = (unsigned long long)c_me;
  }
  const int nodes = __popcll(__ballot(act && n_me > 0));
  if (counts_tree(P, k) && lane == 0) atomicAdd(&stat_bank(P, k)[0], (unsigned long long)nodes);
  if (nodes == 0) return;
  // V_curr = L_eta Psi before the update (Eq. 3).
  const double m = wave_max64(p_me);
  double upto = 0.0;
  const double vc = m + log(ordered_sum(act ? exp(eta * (p_me - m)) : 0.0, A, upto)) / eta;
  // Psi <- Psi - V_curr + Q for the actions with an action node (Eq. 5).
  double p_new = p_me;
  if (act && n_me > 0) {
    const double c = (double)c_me * P.fix_inv64;
    const double w = (double)w_me * P.fix_inv64;
    const double q = c / (double)n_me + P.m.gamma64 * (w / (double)n_me);
    p_new = (p_me - vc) + q;
    psi[lane] = p_new;
  }
  // V = L_eta Psi after the update, and the running sums of the root draw.
  const double m2 = wave_max64(act ? p_new : -INFINITY);
  const double run = ordered_sum(act ? exp(eta * (p_new - m2)) : 0.0, A, upto);
  if (act) T.root_cdf[lane] = upto;
  const long long nsum = (long long)wave_sum((unsigned long long)n_me);
  if (lane != 0) return;
  const double v = m2 + log(run) / eta;
  T.v_root[0] = v;
  T.node[0].V = (float)v;
  T.info[0].Nb = (int)nsum;
}

// Alg. 1: argmax of the root preferences (lowest index on ties) and the
// result record.  Run by the block's first wavefront (64 lanes, one per stripe).
__device__ void dev_select(const PlanView& P) {
  static_assert(kStripes == 64, "one lane per stripe");
  if (threadIdx.x >= 64) return;
  const TreeView& T = P.t;
  const int lane = threadIdx.x;
  const int k_last = P.timed ? (int)T.gate[2] : P.K;   // iterations that ran
  const unsigned long long* bank = stat_bank(P, k_last);
  const unsigned long long steps = wave_sum(T.stats[lane]);
  const unsigned long long nodes = wave_sum(bank[lane]);
  const unsigned long long nb = 1 + wave_sum(bank[kStripes + lane]);
  const unsigned long long near = wave_sum(T.stats[kStatNear * kStripes + lane]);
  const unsigned long long sw_v = wave_sum(T.stats[kStatSweep * kStripes + lane]);
  const unsigned long long sw_i = wave_sum(T.stats[(kStatSweep + 1) * kStripes + lane]);
  const unsigned long long sw_n = wave_sum(T.stats[(kStatSweep + 2) * kStripes + lane]);
  const int A = P.m.nA;
  double* out = P.out;
  // Argmax with the lowest index on ties: each lane scans actions lane,
  // lane + 64, ..., then the wavefront keeps the larger value, or the lower
  // index of equal values.
  int best = lane < A ? lane : 0;
  double bv = T.psi_root[best];
  for (int j = lane; j < A; j += 64) {
    const double v = T.psi_root[j];
    out[1 + j] = v;
    if (v > bv) { bv = v; best = j; }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const double ov = __shfl_xor(bv, off, 64);
    const int ob = __shfl_xor(best, off, 64);
    if (ov > bv || (ov == bv && ob < best)) { bv = ov; best = ob; }
  }
  if (lane != 0) return;
  out[0] = (double)best;
  out[A + 1] = T.v_root[0];
  out[A + 2] = (double)steps;
  out[A + 3] = (double)nb;
  out[A + 4] = (double)nodes;
  out[A + 5] = (double)T.counters[1];
  out[A + 6] = (double)near;
  out[A + 7] = (double)sw_v;
  out[A + 8] = (double)sw_i;
  out[A + 9] = (double)sw_n;
  // The allocation-free entry point's result holds |A| + 10 values.
  if (!P.short_out) out[A + 10] = (double)T.counters[4];
}

// ---------------------------------------------------------------------------
// Served episodes: one step of the true environment, then the sequential
// importance resampling belief update tau(b, a, o) (Alg. 1, belief update).
// Likelihoods are exact integers, so every side draws the same particles:
//   tabular: thr_o - thr_{o-1} of the observation row Z(s', a, .);
//   navigation: the number of 12-bit noise indices per axis whose observation
//   falls in the observed grid cell (the cell is monotone in the index, so two
//   binary searches over the 4096-entry table count them), multiplied.
// Resampling is multinomial: a 64-bit Philox word u per new particle picks
// the particle whose inclusive weight sum first exceeds (u * total) >> 64.
// ---------------------------------------------------------------------------
__device__ void dev_env(const PlanView& P, int t) {
  if (threadIdx.x != 0) return;
  const int a = (int)P.out[0];                 // the action the last plan chose
  const U4 w = philox(0u, kTagEnv << 24, 0u, (uint32_t)t, P.f.env_seed_lo, P.f.env_seed_hi);
  int* env = P.f.env;
  int obs;
  float r;
  bool term = false;
  if (P.m.kind == kTabular) {
    int sn;
    tabular_step(P.m, env[0], a, w, sn, obs, r);
    env[0] = sn;
  } else {
    float nx, ny;
    nav_step(P.m, __int_as_float(env[0]), __int_as_float(env[1]), a, w, nx, ny, obs, r,
             term);
    env[0] = __float_as_int(nx);
    env[1] = __float_as_int(ny);
  }
  env[2] = obs;
  env[3] = a;
  env[4] = __float_as_int(r);
  env[5] = term ? 1 : 0;
}

// Number of table indices j whose observation nx + sd*G[j] falls in cell kx.
__device__ __forceinline__ unsigned nav_cell_count(const ModelView& m, float nx, float sd,
                                                   int kx) {
  // first j with cell(j) >= kx, and first j with cell(j) > kx
  int lo = 0, hi = 4096;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (nav_axis(m.nav, nx + sd * m.gauss[mid]) >= kx) hi = mid; else lo = mid + 1;
  }
  const int first = lo;
  hi = 4096;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (nav_axis(m.nav, nx + sd * m.gauss[mid]) > kx) hi = mid; else lo = mid + 1;
  }
  return (unsigned)(lo - first);
}

// Propagates particle i and returns its integer weight.
__device__ __forceinline__ unsigned long long pf_weight(const PlanView& P, int t, int i) {
  const int M = P.f.M;
  const int a = P.f.env[3], o = P.f.env[2];
  const U4 x = philox((uint32_t)i, kTagPF << 24, 0u, (uint32_t)t, P.seed_lo, P.seed_hi);
  if (P.m.kind == kTabular) {
    const int s = ((const int*)P.f.part)[i];
    const int sn = tabular_next(P.m, s, a, x.y);
    ((int*)P.f.prop)[i] = sn;
    const uint32_t* zr =
        row_leaves(P.m.thrZ + ((size_t)sn * P.m.nA + a) * P.m.rZ.stride, P.m.rZ);
    return (unsigned long long)(zr[o] - (o > 0 ? zr[o - 1] : 0u));
  }
  const float* pf = (const float*)P.f.part;
  float nx, ny;
  nav_move(P.m, pf[i], pf[M + i], a, x.y, nx, ny);
  float* q = (float*)P.f.prop;
  q[i] = nx;
  q[M + i] = ny;
  const float sd = nav_obs_sd(P.m.nav, nx);
  const int kn = P.m.nav.key_n;
  return (unsigned long long)nav_cell_count(P.m, nx, sd, o / kn) *
         (unsigned long long)nav_cell_count(P.m, ny, sd, o % kn);
}

// Inclusive scan over the block; *total: its sum.  red holds kBlock / 64 words
// of LDS; every thread of the block calls.
__device__ __forceinline__ unsigned long long block_incl_scan(unsigned long long v,
                                                              unsigned long long* red,
                                                              unsigned long long* total) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const unsigned long long incl = wave_incl_scan(v);
  if (lane == 63) red[wid] = incl;
  __syncthreads();
  unsigned long long off = 0, tot = 0;
#pragma unroll
  for (int q = 0; q < kBlock / 64; ++q) {
    if (q < wid) off += red[q];
    tot += red[q];
  }
  __syncthreads();
  *total = tot;
  return off + incl;
}

// The particles are cut into at most kPfSegs segments (pf_segment(M) each); w
// holds the weights' inclusive sums within a segment, so a segment's total is
// its last word.  Each block of the resampling adds up the totals for
// itself: at 65,536 particles 256 loads and a scan in LDS, where a launch of one
// block that scanned all the weights took 63 us of the update's 111.
__device__ void dev_pf_weight(const PlanView& P, int t, int blk, unsigned long long* red) {
  const int M = P.f.M, seg = pf_segment(M);
  unsigned long long carry = 0;
  for (int base = blk * seg; base < min(M, (blk + 1) * seg); base += kBlock) {
    const int i = base + threadIdx.x;
    unsigned long long tot;
    const unsigned long long incl =
        block_incl_scan(i < M ? pf_weight(P, t, i) : 0ull, red, &tot);
    if (i < M) P.f.w[i] = carry + incl;
    carry += tot;
  }
}

// pre: kPfSegs + kBlock / 64 words of LDS.
__device__ void dev_pf_resample(const PlanView& P, int t, int blk, unsigned long long* pre) {
  const int j = blk * kBlock + threadIdx.x;
  const int M = P.f.M, seg = pf_segment(M), n_seg = pf_segments(M);
  constexpr int kPer = kPfSegs / kBlock;
  unsigned long long v[kPer], mine = 0, total;
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const int g = (int)threadIdx.x * kPer + q;
    v[q] = g < n_seg ? P.f.w[min((g + 1) * seg, M) - 1] : 0ull;
    mine += v[q];
  }
  unsigned long long run = block_incl_scan(mine, pre + kPfSegs, &total) - mine;
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    run += v[q];
    pre[(int)threadIdx.x * kPer + q] = run;
  }
  __syncthreads();
  if (j == 0) *reinterpret_cast<unsigned long long*>(P.f.env + 6) = total;
  if (j >= M) return;
  int src = j;                                   // zero total: keep propagation
  if (total > 0ull) {
    const U4 y = philox((uint32_t)j, kTagResample << 24, 0u, (uint32_t)t, P.seed_lo,
                        P.seed_hi);
    const unsigned long long u = ((unsigned long long)y.x << 32) | y.y;
    unsigned long long target = __umul64hi(u, total);
    // First i whose running sum is > target: its segment, then its place.
    int lo = 0, hi = n_seg - 1;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (pre[mid] > target) hi = mid; else lo = mid + 1;
    }
    if (lo > 0) target -= pre[lo - 1];
    hi = min((lo + 1) * seg, M) - 1;
    lo *= seg;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (P.f.w[mid] > target) hi = mid; else lo = mid + 1;
    }
    src = lo;
  }
  if (P.m.kind == kTabular) {
    ((int*)P.f.part)[j] = ((const int*)P.f.prop)[src];
  } else {
    const float* q = (const float*)P.f.prop;
    float* pf = (float*)P.f.part;
    pf[j] = q[src];
    pf[M + j] = q[M + src];
  }
}

// ---------------------------------------------------------------------------
// Forward search for long action rows (|A| > kMaxA, tabular models): one
// half wavefront per episode.  The episode's state is the same in every lane
// of the half; the lanes share the softmax draw (lane l owns the quads l,
// l + 32, ... of the row), the record initialisation, and lane 0 of the half
// does the episode's table probe and its scalar writes.  The draw of Eq. (6)
// takes single-precision weights exp(eta (psi_j - max)), sums each quad of
// four in double precision and keeps it rounded once to single precision (in
// LDS), and finds the first running sum above t = u * total by an inclusive
// double-precision scan over the half per chunk of 128 actions.  Every
// running sum is then within 2^-24 of itself (relative) of the sum of the
// single-precision weights, and a row whose entries are all equal gives
// floor(u |A|) exactly.
// ---------------------------------------------------------------------------
__device__ __forceinline__ float long_row_weight(float v, float m, float eta) {
  return expf(eta * (v - m));
}

// Long-row episodes run on half a wavefront (kHalf = 32 lanes), so that a
// wavefront carries two independent episodes: each is a chain of dependent
// reads, and two chains per wavefront hide twice as much of their latency.
// The helpers below reduce, scan and vote within the caller's half (lane is
// the lane within the half).
constexpr int kHalf = 32;

__device__ __forceinline__ float half_maxf(float v) {
#pragma unroll
  for (int off = kHalf / 2; off > 0; off >>= 1) v = fmaxf(v, __shfl_xor(v, off, kHalf));
  return v;
}
// Sum and inclusive scan over the half in double precision, in a fixed
// order (the same for every call).
__device__ __forceinline__ double half_sum64(double v) {
#pragma unroll
  for (int off = kHalf / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, kHalf);
  return v;
}
__device__ __forceinline__ double half_incl_scan64(double v, int lane) {
#pragma unroll
  for (int off = 1; off < kHalf; off <<= 1) {
    const double n = __shfl_up(v, off, kHalf);
    if (lane >= off) v += n;
  }
  return v;
}
// Votes of the caller's half, bit l for lane l of the half.
__device__ __forceinline__ uint32_t half_ballot(bool p) {
  return (uint32_t)(__ballot(p) >> (threadIdx.x & kHalf));
}

// The long-row draw from the double-precision running sums of a row's softmax
// weights (A <= 4096): the first a with t < cdf[a], t = u * cdf[A - 1].  Lane
// l reads the end of run l of ceil(A / 32) actions; the half then reads the
// chosen run (at most 128 entries, four per lane, in order).  Two rounds of
// loads.
__device__ int draw_long_cdf(const double* __restrict__ cdf, int A, uint32_t x0, int lane) {
  const int step = (A + kHalf - 1) / kHalf;
  const double tot = cdf[A - 1];
  const int e = min((lane + 1) * step, A) - 1;
  const bool run_ok = lane * step < A;
  const double end = run_ok ? cdf[e] : 0.0;
  const double t = (double)(x0 >> 8) * (1.0 / 16777216.0) * tot;
  const uint32_t hit = half_ballot(run_ok && t < end);
  if (!hit) return A - 1;
  const int r = __ffs(hit) - 1;
  const int lo = r * step, hi = min(lo + step, A);
  double v[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int j = lo + u * kHalf + lane;
    v[u] = j < hi ? cdf[j] : 0.0;
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int j = lo + u * kHalf + lane;
    const uint32_t h2 = half_ballot(j < hi && t < v[u]);
    if (h2) return lo + u * kHalf + (__ffs(h2) - 1);
  }
  return A - 1;
}

constexpr int kLongChunks = kMaxAWide / (4 * kHalf);   // chunks of 128 actions

// qs: this half's LDS area of kLongChunks * kHalf quad sums (single-precision
// bits).  Entry a1 of the row (a1 < 0: none) is p1 instead.  near: t lies within
// kTieRel * total of a boundary next to it (rows
// whose entries are all equal never count).
__device__ int draw_long_row(const float* __restrict__ row, int a1, float p1, int A, float eta,
                             uint32_t x0, int lane, uint32_t* qs, bool& near) {
  // Lane l of the half holds the quads l, l + 32, ... (the row is padded to
  // a multiple of 4; padding is masked off).  Each weight is evaluated once:
  // the lane keeps its quad sum of every chunk (in LDS, for registers), the
  // half scans those once the total is known, and only the chosen quad is
  // evaluated again.
  const float4* r4 = reinterpret_cast<const float4*>(row);
  auto read = [&](int q) {
    return with_entry(r4[q], q, a1, p1);
  };
  const int nq = (A + 3) / 4;
  const int nc = (nq + kHalf - 1) / kHalf;
  float m = -INFINITY, mn = INFINITY;
#pragma unroll 4
  for (int q = lane; q < nq; q += kHalf) {
    const float4 v = read(q);
    const int j = 4 * q;
    m = fmaxf(m, v.x);
    mn = fminf(mn, v.x);
    if (j + 1 < A) { m = fmaxf(m, v.y); mn = fminf(mn, v.y); }
    if (j + 2 < A) { m = fmaxf(m, v.z); mn = fminf(mn, v.z); }
    if (j + 3 < A) { m = fmaxf(m, v.w); mn = fminf(mn, v.w); }
  }
  m = half_maxf(m);
  const bool flat = -half_maxf(-mn) == m;
  auto quad = [&](int q, float (&w)[4]) {
    const float4 v = read(q);
    const int j = 4 * q;
    w[0] = long_row_weight(v.x, m, eta);
    w[1] = j + 1 < A ? long_row_weight(v.y, m, eta) : 0.0f;
    w[2] = j + 2 < A ? long_row_weight(v.z, m, eta) : 0.0f;
    w[3] = j + 3 < A ? long_row_weight(v.w, m, eta) : 0.0f;
  };
  double tot = 0.0;
  for (int c = 0; c < nc; ++c) {
    const int q = c * kHalf + lane;
    float sq = 0.0f;
    if (q < nq) {
      float w[4];
      quad(q, w);
      sq = (float)((((double)w[0] + (double)w[1]) + (double)w[2]) + (double)w[3]);
    }
    qs[c * kHalf + lane] = __float_as_uint(sq);
    tot += (double)sq;
  }
  tot = half_sum64(tot);
  const double t = (double)(x0 >> 8) * (1.0 / 16777216.0) * tot;
  double base = 0.0;
  for (int c = 0; c < nc; ++c) {
    const double sq = (double)__uint_as_float(qs[c * kHalf + lane]);
    const double incl = half_incl_scan64(sq, lane) + base;
    const uint32_t hit = half_ballot(c * kHalf + lane < nq && t < incl);
    if (hit) {
      const int src = __ffs(hit) - 1;
      int pick = 3;                             // within the chosen quad
      int tie = 0;
      if (lane == src) {
        float w[4];
        quad(c * kHalf + lane, w);
        double run = incl - sq, below = run;
        for (int u = 0; u < 4; ++u) {
          below = run;
          run += (double)w[u];
          if (t < run) { pick = u; break; }
        }
        if (pick == 3) run = incl;              // the quad's rounded sum bounds it
        const int a = 4 * (c * kHalf + lane) + pick;
        const double lim = kTieRel * tot;
        tie = !flat && ((a > 0 && t - below <= lim) || (a < A - 1 && run - t <= lim));
      }
      near = __shfl(tie, src, kHalf) != 0;
      return 4 * (c * kHalf + src) + __shfl(pick, src, kHalf);
    }
    base = __shfl(incl, kHalf - 1, kHalf);
  }
  near = false;
  return A - 1;
}

// search() on half a wavefront: the episode's state is the same in every lane.
template <bool ONE>
__device__ void search_wide(const PlanView& P, int k, int D, int ep, const Episode& e0,
                            uint32_t* qs, unsigned long long& g, unsigned long long& nt) {
  const TreeView& T = P.t;
  const int lane = threadIdx.x & (kHalf - 1);
  const int t0 = first_step(P, k);
  const int first_new = 1 + t0 * P.n_p;
  const int A = P.m.nA, ob = P.m.obs_bits;
  const size_t n_p = (size_t)P.n_p;
  const unsigned long long stamp = (unsigned long long)(k - 1) << kStampShift;
  int s = e0.s, d = 0;
  int id = 0;                 // < 0: of a leaf known by its table slot ~id
  uint32_t link = 0;
  float nr = 0.0f, npsi = 0.0f;
  auto arrive = [&]() {
    uint4 q;
    if (id >= first_new) q = load_seen(&T.node[id]);
    else q = *reinterpret_cast<const uint4*>(&T.node[id]);
    link = q.y;
    nr = __uint_as_float(q.z);
    npsi = __uint_as_float(q.w);
  };
  bool tail = false;
  uint32_t head = 0;
  int tl = 0;                 // (1 also for the creator of a leaf of a plan of one level)
  uint32_t slot = 0;
  int id_head = 0, to_publish = 0, waits = 0;
  bool alive = true;
  // One level of the search.
  auto level = [&]() {
    const U4 w = draw(P, (uint32_t)ep, kTagStep, (uint32_t)d, (uint32_t)k);
    bool tie = false;
    int a;
    if (id == 0) {
      a = draw_long_cdf(T.root_cdf, A, w.x, lane);
      tie = (k > 1 || P.carry) && near_tie64(T.root_cdf, A, w.x, a);
    } else if (id >= first_new) {
      a = draw_long_cdf(T.psi0_cdf64, A, w.x, lane);
    } else {
      const bool full = (link & kLinkFull) != 0;
      const int a1 = !full && (link & kLinkAct) ? (int)((link & kLinkKey) >> ob) : -1;
      a = draw_long_row(full ? rec_psi(T, id) : T.psi0, a1, npsi, A, P.eta, w.x, lane, qs, tie);
    }
    nt += tie ? 1u : 0u;
    const int drawn = a;
    const size_t di = (size_t)(t0 + d - P.carry_steps) * n_p + ep;
    if (T.dbg_force) {
      const short f = T.dbg_force[di];
      if (f >= 0 && f < A) a = f;
    }
    int sn, obs;
    float r;
    tabular_step(P.m, s, a, w, sn, obs, r);
    s = sn;
    ++g;
    if (T.dbg_act && lane == 0) {
      T.dbg_act[di] = (short)drawn;
      T.dbg_obs[di] = obs;
    }
    const uint32_t low = key_low(a, obs, ob);
    if (tail) {
      if (!head) stores_done();               // the records above this one
      if (lane == 0 && !head)
        __hip_atomic_store(&T.run[(size_t)(k - 1) * n_p + ep], (unsigned short)(kRunOpen | d),
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (lane == 0)
        store_seen(&T.node[id], 0u, low | kLinkAct | kLinkChild | head, __float_as_uint(r),
                   __float_as_uint(T.psi0[a]));
      if (to_publish) to_publish = 2;
      id += P.n_p;
      head = 0;
      ++d;
      return;
    }
    const int b = id;
    const uint32_t blink = link;
    const float b_r = nr, b_psi = npsi;
    const unsigned long long bk = belief_key(b, low);
    int first = 0;
    if (lane == 0) first = claim(T, b, blink);
    int won = 0, fresh = 0, old = -1;
    uint32_t h = 0;
    const bool to_leaf = d + 1 == D;            // k_claim_wide sees to it
    if ((blink & kLinkChild) && (blink & kLinkKey) == low) {
      id = b + P.n_p;
      if (b >= first_new && !to_leaf) waits = 2;
    } else {
      // AppendBeliefs by lane 0 of the half; the outcome goes to the half.
      if (lane == 0) {
        Bucket line;
        bucket_read(T, bk, line);
        bool bw = false, bf = false;
        h = probe(T, line, bk, stamp, 0, 0, bw, bf, old);
        won = bw;
        fresh = bf;
      }
      h = __shfl(h, 0, kHalf);
      won = __shfl(won, 0, kHalf);
      fresh = __shfl(fresh, 0, kHalf);
      old = __shfl(old, 0, kHalf);
      if (h == ~0u) {
        if (lane == 0) atomicOr((unsigned int*)&T.counters[1], kErrTable);
        alive = false;
        tl = d + 1;
      } else if (ONE && won) {
        id = 1 + t0 * P.n_p + ep;
        tl = 1;
        if (lane == 0) make_leaf(T, h, id, bk);
      } else if (won) {
        tail = true;
        head = kLinkHead;
        tl = d + 1;
        id = 1 + (t0 + d) * P.n_p + ep;
        id_head = id;
        slot = h;
        to_publish = 1;
      } else if (fresh && to_leaf) {
        id = ~(int)h;
      } else if (fresh) {
        slot = h;
        waits = 1;
      } else {
        id = old;
      }
    }
    if (alive && !tail && !waits && !to_leaf) arrive();
    first = __shfl(first, 0, kHalf);
    if (lane == 0) {
      // Every visit goes to the trace: the first visit of (b, a) clears its
      // columns in the claim pass, before any count is added.
      T.tr_key[(size_t)d * n_p + ep] = ((unsigned long long)(uint32_t)b << kActBits) |
                                       (uint32_t)a | (first ? kTraceClaim : 0ull);
      T.tr_val[(size_t)d * n_p + ep] = r;
      if (won && tail) store_seen(&T.info[id], bk);
    }
    if (first) {
      if (lane == 0) {
        unsigned long long own = 0;             // (a run's first belief has it already)
        if (!(blink & kLinkHead))
          own = belief_key(b - P.n_p, load_seen(&T.node[b - P.n_p]).y & kLinkKey);
        make_full_node(P, b, blink, b_r, own, b >= first_new);
      }
      const int a1 = one_action(blink, ob);
      float4* q = reinterpret_cast<float4*>(rec_psi(T, b));
      const float4* p0 = reinterpret_cast<const float4*>(T.psi0);
      for (int i = lane; i < T.ra / 4; i += kHalf) q[i] = with_entry(p0[i], i, a1, b_psi);
      store_bits<kHalf>(T, b, a1, lane);
    }
    if (alive) ++d;
  };
  // The end of the episode: its leaf, its run word.
  auto finish = [&]() {
    uint32_t run = (uint32_t)tl;
    if (alive) {
      const float hv = P.m.H ? P.m.H[s] : 0.0f;
      const unsigned long long fx = to_fix(hv, P.fix_scale);
      if (tail) {
        if (lane == 0)
          store_seen(&T.node[id], __float_as_uint(from_fix(fx, P.fix_inv)), head,
                     __float_as_uint(hv), 0u);
        run = (uint32_t)tl | (uint32_t)(D - tl + 1) << kRunLenShift;
      } else {
        run = (uint32_t)D | kRunLeaf | (uint32_t)tl << kRunLenShift;
        if (lane == 0) {
          T.tr_key[(size_t)D * n_p + ep] = leaf_word(id);
          T.tr_val[(size_t)D * n_p + ep] = hv;
        }
      }
    }
    if (tail) stores_done();                    // (nobody waits for another's word)
    if (lane == 0) {
      if (to_publish)
        __hip_atomic_store(&T.h_slot[slot].id, id_head, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(&T.run[(size_t)(k - 1) * n_p + ep], (unsigned short)run, __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
    }
    to_publish = 0;
  };
  // The loop ends for the whole wavefront at once, so that a lane that has ended
  // has published its run before any lane of the wavefront waits again.
  bool done = false;
  uint32_t turns = 0;         // of the wavefront, with a half that waits
  do {
    if (__any(waits) && wait_over(P, ++turns)) {
      if (waits) {            // levels 0 .. d - 1 are in the trace
        if (lane == 0) atomicOr((unsigned int*)&T.counters[1], kErrWait);
        waits = 0;
        alive = false;
        tl = d;
      }
    }
    if (to_publish == 2) {
      stores_done();
      if (lane == 0)
        __hip_atomic_store(&T.h_slot[slot].id, id_head, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
      to_publish = 0;
    }
    if (!done) {
      if (waits) {                                // every lane of the half reads the same
        if (waits == 1) {
          const int got = __shfl(__hip_atomic_load(&T.h_slot[slot].id, __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_AGENT), 0, kHalf);
          if (got >= 0) {
            id = got;
            waits = 0;
          }
        } else {
          const int owner = (id - 1) % P.n_p;
          const uint32_t run = (uint32_t)__shfl(
              (int)__hip_atomic_load(&T.run[(size_t)(k - 1) * n_p + owner], __ATOMIC_RELAXED,
                                     __HIP_MEMORY_SCOPE_AGENT), 0, kHalf);
          if (run_has(run, d)) waits = 0;
        }
        if (!waits) arrive();
        else if (__all(waits)) __builtin_amdgcn_s_sleep(1);
      } else if (alive && d < D) {
        level();
      } else {
        finish();
        done = true;
      }
    }
  } while (__ballot(!done));
}

// Four wavefronts per SIMD (128 registers, a few spilled): each episode is a
// chain of dependent reads, so residency is what hides them.
template <bool ONE>
__global__ __launch_bounds__(kBlock, 4) void k_forward_wide(PlanView P, int k, int D) {
  __shared__ unsigned long long red[kBlock / 64];
  __shared__ uint32_t qsum[kBlock / kHalf][kLongChunks * kHalf];
  if (budget_spent(P, k)) return;
  const int lane = threadIdx.x & (kHalf - 1);
  const int ep = blockIdx.x * (kBlock / kHalf) + (threadIdx.x / kHalf);   // uniform per half
  unsigned long long g = 0, nt = 0;
  if (ep < P.n_p) {
    const Episode e = at_root(P, k, ep, lane == 0);
    search_wide<ONE>(P, k, D, ep, e, qsum[threadIdx.x / kHalf], g, nt);
  }
  tally(P.t, blockIdx.x, lane == 0 ? g : 0ull, lane == 0 ? nt : 0ull, red);
}

__global__ void k_env(PlanView P, int t) { dev_env(P, t); }
__global__ __launch_bounds__(kBlock) void k_pf_weight(PlanView P, int t) {
  __shared__ unsigned long long red[kBlock / 64];
  dev_pf_weight(P, t, blockIdx.x, red);
}
__global__ __launch_bounds__(kBlock) void k_pf_resample(PlanView P, int t) {
  __shared__ unsigned long long pre[kPfSegs + kBlock / 64];
  dev_pf_resample(P, t, blockIdx.x, pre);
}
__global__ __launch_bounds__(kBlock) void k_setup(PlanView P) {
  __shared__ SetupSmem ss;
  dev_setup(P, blockIdx.x, gridDim.x, &ss);
}
// The phases of one iteration return at once when a time budget ran out
// at the end of an earlier iteration.
template <int AM, bool NAV, bool TRACE, bool ONE>
__global__ __launch_bounds__(kBlock) void k_forward(PlanView P, int k, int D) {
  __shared__ SearchSmem L;
  if (budget_spent(P, k)) return;
  dev_forward<AM, NAV, TRACE, ONE>(P, k, D, blockIdx.x, L);
}
__global__ __launch_bounds__(kBlock) void k_accum(PlanView P, int k, int D) {
  __shared__ Smem sm;
  if (budget_spent(P, k)) return;
  dev_accum(P, k, D, blockIdx.x, gridDim.x, sm);
}
template <int AM>
__global__ __launch_bounds__(kBlock) void k_fold(PlanView P, int k) {
  __shared__ Smem sm;
  if (budget_spent(P, k)) return;
  dev_fold<AM>(P, k, blockIdx.x, gridDim.x, sm);
}
template <int QPL>
__global__ __launch_bounds__(kBlock) void k_chain_wide(PlanView P, int k) {
  if (budget_spent(P, k)) return;
  dev_chain_wide<QPL>(P, k, blockIdx.x, gridDim.x);
}
__global__ __launch_bounds__(kBlock) void k_backup_leaf(PlanView P, int dep, int k) {
  __shared__ Smem sm;
  if (budget_spent(P, k)) return;
  dev_backup_leaf(P, dep, k, blockIdx.x, gridDim.x, sm);
  if (dep == 1) dev_leaf_runs(P, k, blockIdx.x, gridDim.x, sm);
}
template <int AM>
__global__ __launch_bounds__(kBlock) void k_full(PlanView P, int k) {
  __shared__ Smem sm;
  if (budget_spent(P, k)) return;
  dev_full<AM, false>(P, k, blockIdx.x, sm);
}
template <int AM>
__global__ __launch_bounds__(kBlock) void k_full_one(PlanView P, int k) {
  __shared__ Smem sm;
  if (budget_spent(P, k)) return;
  dev_full<AM, true>(P, k, blockIdx.x, sm);
}
template <int QPL>
__global__ __launch_bounds__(kBlock) void k_backup_level_wide(PlanView P, int dep, int k) {
  __shared__ Smem sm;
  if (budget_spent(P, k)) return;
  dev_backup_level_wide<QPL>(P, dep, k, blockIdx.x, gridDim.x, sm);
}
__global__ __launch_bounds__(kBlock) void k_backup_root_wide(PlanView P, int k) {
  __shared__ double buf[kBlock];
  if (budget_spent(P, k)) return;
  dev_backup_root_wide(P, k, buf);
}
__global__ void k_select(PlanView P) { dev_select(P); }

// ---------------------------------------------------------------------------
// Batched kernel: block -> (instance, phase) through the item list, sorted by
// first block.  AMAX bounds the padded action count of the batch.
// ---------------------------------------------------------------------------
// A block runs one phase at a time.
union BatchSmem {
  Smem sm;
  SearchSmem search;
};

// The phases whose code depends on the row length, for AM >= |A|.
template <int AM>
__device__ __forceinline__ void run_rows(const PlanView& P, const BatchItem& it, int blk,
                                         BatchSmem& bs) {
  Smem& sm = bs.sm;
  SearchSmem& L = bs.search;
  const int k = it.a0;
  switch (it.kind) {
    case kPhaseForward:
      if (AM == 4 && P.m.kind == kNav) dev_forward<AM, true, false, false>(P, k, depth_at(P, k), blk, L);
      else dev_forward<AM, false, false, false>(P, k, depth_at(P, k), blk, L);
      break;
    case kPhaseFold: dev_fold<AM>(P, k, blk, it.nblk, sm); break;
    case kPhaseFull: dev_full<AM, false>(P, k, blk, sm); break;
    default: break;
  }
}
// One phase item of one instance, as block blk of its nblk (LDS in sm).
template <int AMAX>
__device__ __forceinline__ void run_item(const PlanView& P, const BatchItem& it, int blk,
                                         BatchSmem& bs) {
  Smem& sm = bs.sm;
  const int Apad = P.m.Apad;
  switch (it.kind) {
    case kPhaseSetup: dev_setup(P, blk, it.nblk, nullptr); break;   // |A| <= 16
    case kPhaseSelect: dev_select(P); break;
    case kPhaseEnv: dev_env(P, it.a0); break;
    case kPhasePFWeight: dev_pf_weight(P, it.a0, blk, sm.wave); break;
    case kPhasePFResample:
      static_assert(sizeof(AggTable) >= (kPfSegs + kBlock / 64) * sizeof(unsigned long long),
                    "the segment sums fit the table");
      dev_pf_resample(P, it.a0, blk, reinterpret_cast<unsigned long long*>(&sm.agg));
      break;
    default:
      if (Apad <= 4) {
        run_rows<4>(P, it, blk, bs);
      } else if constexpr (AMAX >= 8) {
        if (Apad <= 8) run_rows<8>(P, it, blk, bs);
        else if constexpr (AMAX >= 16) run_rows<16>(P, it, blk, bs);
      }
      break;
  }
}

template <int AMAX>
__global__ __launch_bounds__(kBlock) void k_batch(const PlanView* __restrict__ views,
                                                  const BatchItem* __restrict__ items,
                                                  int n_items) {
  __shared__ BatchSmem sm;
  const int g = blockIdx.x;
  int lo = 0, hi = n_items - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (items[mid].blk0 <= g) lo = mid; else hi = mid - 1;
  }
  const BatchItem it = items[lo];
  const int blk = g - it.blk0;
  if (blk >= it.nblk) return;          // uniform per block
  run_item<AMAX>(views[it.inst], it, blk, sm);
}

// The persistent batched launch.  Every block loops: take a tile (one block's
// share) of some instance's current phase from the queue, run it, and report
// it finished; the last finisher of a phase moves its instance to the next
// phase.  Taking a tile is one atomic add on the instance's word, whose old
// value names the phase and the tile together, so a block never runs a tile
// of a phase that has not started.  Memory order: each finisher releases its
// block's writes (agent scope) before it counts; the last finisher publishes
// the next phase with a release; a taker acquires after the add.  A block
// that finds no tile sleeps briefly and looks again; it returns once every
// instance is past its last phase.
//
// The queue drains whatever the residency.  A tile may wait for another tile of
// its phase, but only for work that a running block has already taken and that
// waits for nothing itself: an episode of a forward tile waits for the creator of
// a belief, which inserted it and so runs, and creators never wait (search()); a
// tile of the full beliefs waits for items of lower numbers, which are taken in
// that order (dev_full()).  Tiles that ran in another order than they are taken,
// creators that wait, or items given out ahead of time would break that.
__global__ void k_persist_reset(PersistView V) {
  const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x);
  if (i < V.n) {
    V.word[i] = 0ull;
    V.done[i] = 0u;
  }
  if (i == 0) *V.finished = 0u;
}

template <int AMAX>
__global__ __launch_bounds__(kBlock) void k_batch_persistent(const PlanView* __restrict__ views,
                                                             PersistView V) {
  __shared__ BatchSmem sm;
  __shared__ int take[3];
  int cur = (int)(blockIdx.x % (unsigned)V.n);
  for (;;) {
    if (threadIdx.x < 64) {
      // Wavefront 0 looks for a tile: its lanes read 64 instances' words at
      // once (this block's last instance first, then the others in turn), and
      // the instances with a tile left are tried in that order, one atomic
      // add each, until one yields a tile.
      const int lane = (int)threadIdx.x;
      int inst = -1, ph = 0, tile = 0;
      for (int base = 0; base < V.n && inst < 0; base += 64) {
        const int q = base + lane;
        int i = 0;
        bool avail = false;
        if (q < V.n) {
          i = cur + q < V.n ? cur + q : cur + q - V.n;
          const int np = V.ph_off[i + 1] - V.ph_off[i];
          const unsigned long long w =
              __hip_atomic_load(&V.word[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          const int g = (int)(w >> 32);
          avail = g < np && (unsigned)w < (unsigned)V.phases[V.ph_off[i] + g].nblk;
        }
        unsigned long long m = __ballot(avail);
        while (m && inst < 0) {
          const int src = __ffsll((long long)m) - 1;
          m &= m - 1;
          int got = 0, g2 = 0, t2 = 0;
          if (lane == src) {
            const unsigned long long o = atomicAdd(&V.word[i], 1ull);
            g2 = (int)(o >> 32);
            t2 = (int)(unsigned)o;
            const int np = V.ph_off[i + 1] - V.ph_off[i];
            got = g2 < np && (unsigned)t2 < (unsigned)V.phases[V.ph_off[i] + g2].nblk;
          }
          if (__shfl(got, src, 64)) {
            inst = __shfl(i, src, 64);
            ph = __shfl(g2, src, 64);
            tile = __shfl(t2, src, 64);
          }
        }
      }
      if (lane == 0) {
        if (inst >= 0) {
          __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        } else if (__hip_atomic_load(V.finished, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >=
                   (unsigned)V.n) {
          inst = -2;
        }
        take[0] = inst;
        take[1] = ph;
        take[2] = tile;
      }
    }
    __syncthreads();
    const int inst = take[0], ph = take[1], tile = take[2];
    __syncthreads();
    if (inst == -2) return;
    if (inst == -1) {
      __builtin_amdgcn_s_sleep(8);
      continue;
    }
    cur = inst;
    const BatchItem it = V.phases[V.ph_off[inst] + ph];
    if (it.kind == kPhaseForward) {
      // A forward tile runs several of the phase's blocks of episodes
      // (blk0 of them in all, nblk tiles).
      for (int sub = tile; sub < it.blk0; sub += it.nblk) {
        run_item<AMAX>(views[inst], it, sub, sm);
        __syncthreads();
      }
    } else {
      run_item<AMAX>(views[inst], it, tile, sm);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
      const unsigned d = atomicAdd(&V.done[inst], 1u) + 1u;
      if (d == (unsigned)it.nblk) {
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        __hip_atomic_store(&V.done[inst], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const int np = V.ph_off[inst + 1] - V.ph_off[inst];
        __hip_atomic_exchange(&V.word[inst], (unsigned long long)(ph + 1) << 32,
                              __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
        if (ph + 1 == np) atomicAdd(V.finished, 1u);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Launchers (host side).
// ---------------------------------------------------------------------------
static inline int blocks_for(long long n) { return (int)((n + kBlock - 1) / kBlock); }

// (By what is cleared, in units of 16 bytes: the table, the root's striped sums,
// the run words.  By the table alone, which is short where episodes are few, one
// block cleared 1.5 MB of root sums for 390 episodes over 954 actions, 53 us.)
int setup_blocks(const PlanView& P) {
  const long long work = (long long)P.t.h_mask + 1 + 3ll * P.t.ra * kStripes / 2 +
                         (long long)P.K * P.n_p / 8;
  long long g = (work + kBlock * 8 - 1) / (kBlock * 8);
  return (int)std::max(1ll, std::min(g, 1024ll));
}

int forward_blocks(const PlanView& P) { return blocks_for(P.n_p); }

int accum_blocks(const PlanView& P, int D, int cap) {
  const long long g = (long long)blocks_for(P.n_p) * (D + 1);
  return (int)std::max(1ll, std::min(g, (long long)cap));
}

LaunchTiming& launch_timing() {
  static thread_local LaunchTiming t;
  return t;
}

// A plan kernel's launch, timed by its own dispatch when a profiling bracket
// is open on this thread (launch_timing).
template <typename... KArgs, typename... Args>
static void plan_launch(void (*kernel)(KArgs...), dim3 g, dim3 b, uint32_t shm, hipStream_t s,
                        Args... args) {
  LaunchTiming& t = launch_timing();
  if (t.stop) {
    hipExtLaunchKernelGGL(kernel, g, b, shm, s, t.start, t.stop, 0u, args...);
    t.start = nullptr;
    t.used = true;
  } else {
    hipLaunchKernelGGL(kernel, g, b, shm, s, args...);
  }
}

hipError_t launch_setup(const PlanView& P, hipStream_t s) {
  plan_launch(k_setup, dim3(setup_blocks(P)), dim3(kBlock), 0, s, P);
  return hipGetLastError();
}
// Calls F<AM>'s launch for the smallest AM that holds the rows.
#define VOPP_BY_ROW(F, g, b, s, ...)                                            \
  do {                                                                         \
    const int Ap_ = P.m.Apad;                                                  \
    if (Ap_ <= 4) plan_launch(F<4>, g, b, 0, s, __VA_ARGS__);                  \
    else if (Ap_ <= 8) plan_launch(F<8>, g, b, 0, s, __VA_ARGS__);             \
    else if (Ap_ <= 16) plan_launch(F<16>, g, b, 0, s, __VA_ARGS__);           \
    else if (Ap_ <= 32) plan_launch(F<32>, g, b, 0, s, __VA_ARGS__);           \
    else plan_launch(F<kMaxA>, g, b, 0, s, __VA_ARGS__);                       \
  } while (0)
// The same for long rows, by quads per lane: rows of up to 1024, 2048, 3072,
// 4096 actions.
#define VOPP_BY_LONG_ROW(F, g, b, s, ...)                                       \
  do {                                                                         \
    const int qpl_ = (P.m.Apad / 4 + 63) / 64;                                 \
    if (qpl_ <= 4) plan_launch(F<4>, g, b, 0, s, __VA_ARGS__);                 \
    else if (qpl_ <= 8) plan_launch(F<8>, g, b, 0, s, __VA_ARGS__);            \
    else if (qpl_ <= 12) plan_launch(F<12>, g, b, 0, s, __VA_ARGS__);          \
    else plan_launch(F<16>, g, b, 0, s, __VA_ARGS__);                          \
  } while (0)

static dim3 wide_grid(const PlanView& P) {
  return dim3((P.n_p + kBlock / kHalf - 1) / (kBlock / kHalf));
}
template <bool TRACE, bool ONE>
static void launch_forward_rows(const PlanView& P, int k, int D, hipStream_t s) {
  const dim3 g(forward_blocks(P)), b(kBlock);
  const int Ap = P.m.Apad;
  if (P.m.kind == kNav) plan_launch(k_forward<4, true, TRACE, ONE>, g, b, 0, s, P, k, D);
  else if (Ap <= 4) plan_launch(k_forward<4, false, TRACE, ONE>, g, b, 0, s, P, k, D);
  else if (Ap <= 8) plan_launch(k_forward<8, false, TRACE, ONE>, g, b, 0, s, P, k, D);
  else if (Ap <= 16) plan_launch(k_forward<16, false, TRACE, ONE>, g, b, 0, s, P, k, D);
  else if (Ap <= 32) plan_launch(k_forward<32, false, TRACE, ONE>, g, b, 0, s, P, k, D);
  else plan_launch(k_forward<kMaxA, false, TRACE, ONE>, g, b, 0, s, P, k, D);
}
template <bool ONE>
static void launch_forward_of(const PlanView& P, int k, hipStream_t s) {
  const int D = depth_at(P, k);
  if (P.m.Apad > kMaxA) plan_launch(k_forward_wide<ONE>, wide_grid(P), dim3(kBlock), 0, s, P, k, D);
  else if (P.t.dbg_act) launch_forward_rows<true, ONE>(P, k, D, s);
  else launch_forward_rows<false, ONE>(P, k, D, s);
}
hipError_t launch_forward(const PlanView& P, int k, hipStream_t s) {
  if (one_level(P)) launch_forward_of<true>(P, k, s);
  else launch_forward_of<false>(P, k, s);
  return hipGetLastError();
}
hipError_t launch_accum(const PlanView& P, int k, int grid, hipStream_t s) {
  const int D = depth_at(P, k);
  if (!one_level(P)) {
    const int leaves = kBlock / 64 * claim_leaves(P, D);   // episodes a block
    plan_launch(k_claim_wide, dim3(claim_visit_blocks(P.n_p, D) + (P.n_p + leaves - 1) / leaves),
                dim3(kBlock), 0, s, P, k, D);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  plan_launch(k_accum, dim3(grid), dim3(kBlock), 0, s, P, k, D);
  return hipGetLastError();
}
hipError_t launch_fold(const PlanView& P, int k, int grid, hipStream_t s) {
  const dim3 g(grid), b(kBlock);
  if (one_level(P)) plan_launch(k_accum, g, b, 0, s, P, k, depth_at(P, k));   // no runs to walk
  else VOPP_BY_ROW(k_fold, g, b, s, P, k);
  return hipGetLastError();
}
hipError_t launch_chain(const PlanView& P, int k, int grid, hipStream_t s) {
  const dim3 g(grid), b(kBlock);
  VOPP_BY_LONG_ROW(k_chain_wide, g, b, s, P, k);
  return hipGetLastError();
}
hipError_t launch_backup_leaf(const PlanView& P, int dep, int k, int grid, hipStream_t s) {
  plan_launch(k_backup_leaf, dim3(grid), dim3(kBlock), 0, s, P, dep, k);
  return hipGetLastError();
}
hipError_t launch_full(const PlanView& P, int k, int grid, hipStream_t s) {
  const dim3 g(grid), b(kBlock);
  if (one_level(P)) VOPP_BY_ROW(k_full_one, g, b, s, P, k);
  else VOPP_BY_ROW(k_full, g, b, s, P, k);
  return hipGetLastError();
}
hipError_t launch_backup_level(const PlanView& P, int dep, int k, int grid, hipStream_t s) {
  const dim3 g(grid), b(kBlock);
  VOPP_BY_LONG_ROW(k_backup_level_wide, g, b, s, P, dep, k);
  return hipGetLastError();
}
hipError_t launch_backup_root(const PlanView& P, int k, hipStream_t s) {
  plan_launch(k_backup_root_wide, dim3(1), dim3(kBlock), 0, s, P, k);
  return hipGetLastError();
}
hipError_t launch_select(const PlanView& P, hipStream_t s) {
  plan_launch(k_select, dim3(1), dim3(64), 0, s, P);
  return hipGetLastError();
}
hipError_t launch_env(const PlanView& P, int t, hipStream_t s) {
  hipLaunchKernelGGL(k_env, dim3(1), dim3(64), 0, s, P, t);
  return hipGetLastError();
}
hipError_t launch_pf_weight(const PlanView& P, int t, hipStream_t s) {
  hipLaunchKernelGGL(k_pf_weight, dim3(pf_segments(P.f.M)), dim3(kBlock), 0, s, P, t);
  return hipGetLastError();
}
hipError_t launch_pf_resample(const PlanView& P, int t, hipStream_t s) {
  hipLaunchKernelGGL(k_pf_resample, dim3(blocks_for(P.f.M)), dim3(kBlock), 0, s, P, t);
  return hipGetLastError();
}
// Whether a belief of a finished plan has a row of its own.
__device__ __forceinline__ bool has_row(const TreeView& t, uint32_t link) {
  return (link & kLinkFull) && !((t.ra > kMaxA || t.one) && (link & kLinkBare));
}
// Action and N, C of the action node of a belief without.
struct OneNode {
  int a, n;                  // a = -1: none
  unsigned long long c;
  float psi;
};
__device__ __forceinline__ OneNode one_node(const BeliefNode& b, int ob, float scale) {
  OneNode o{-1, 0, 0ull, 0.0f};
  if (b.link & kLinkAct) {
    o.a = (int)((b.link & kLinkKey) >> ob);
    o.n = 1;
    o.c = to_fix(b.u.one.r, scale);
    o.psi = b.u.one.psi;
  }
  return o;
}

// The tree dump: belief ids[i]'s fields packed at out + i * dump_bytes(ra)
// (layout in vopp_device.hpp), one thread per belief.
__global__ __launch_bounds__(kBlock) void k_gather(TreeView t, int n_p, int ob, float scale,
                                                   const int* ids, int n, unsigned char* out) {
  const int ra = t.ra;
  const size_t db = (size_t)dump_bytes(ra);
  for (long long i = (long long)blockIdx.x * kBlock + threadIdx.x; i < n;
       i += (long long)gridDim.x * kBlock) {
    const int id = ids[i];
    const BeliefNode b = t.node[id];
    const bool full = has_row(t, b.link);
    const OneNode one = one_node(b, ob, scale);
    unsigned char* o = out + (size_t)i * db;
    float* po = reinterpret_cast<float*>(o);
    int* no = reinterpret_cast<int*>(o + dump_n_off(ra));
    unsigned long long* co = reinterpret_cast<unsigned long long*>(o + dump_c_off(ra));
    for (int j = 0; j < ra; ++j) {
      po[j] = full ? rec_psi(t, id)[j] : j == one.a ? one.psi : t.psi0[j];
      no[j] = full ? rec_n(t, id)[j] : j == one.a ? one.n : 0;
      co[j] = full ? rec_c(t, id)[j] : j == one.a ? one.c : 0ull;
    }
    const unsigned long long own = id == 0 ? kEmptyKey : own_of(t, id, b.link, n_p);
    unsigned char* tl = o + dump_tail_off(ra);
    *reinterpret_cast<float*>(tl) = b.V;
    *reinterpret_cast<int*>(tl + 4) = (b.link & kLinkFull) ? t.info[id].Nb : 1;
    *reinterpret_cast<int*>(tl + 8) = (int)(own & ((1ull << ob) - 1));
    *reinterpret_cast<int*>(tl + 12) = 0;
    *reinterpret_cast<unsigned long long*>(tl + 16) =
        id == 0 ? kEmptyKey : parent_of(own, ob);
    uint32_t* bo = reinterpret_cast<uint32_t*>(o + dump_bits_off(ra));
    for (int j = 0; j < t.bw; ++j)
      bo[j] = full ? rec_bits(t, id)[j] : one.a >> 5 == j ? 1u << (one.a & 31) : 0u;
  }
}
hipError_t launch_gather(const TreeView& t, int n_p, int ob, float scale, const int* ids, int n,
                         unsigned char* out, hipStream_t s) {
  const int g = (int)std::max(1ll, std::min(((long long)n + kBlock - 1) / kBlock, 4096ll));
  hipLaunchKernelGGL(k_gather, dim3(g), dim3(kBlock), 0, s, t, n_p, ob, scale, ids, n, out);
  return hipGetLastError();
}
// ---------------------------------------------------------------------------
// Tree re-rooting between real steps (the outer loop of Alg. 1): the belief
// reached from the root by the executed action and the perceived observation
// becomes the root of the next plan; its descendants keep their records
// (statistics) and move one level up.  The passes run depth by depth, so a
// belief's parent is always done before it.
// ---------------------------------------------------------------------------

// Slot of `key` (any stamp) in a table no kernel is inserting into, or ~0u.
// An insert takes the first empty-or-matching slot of the key's bucket in the
// key's rotated order and moves to the next bucket only when it is full,
// and slots are never emptied during a plan, so the first such slot decides.
__device__ uint32_t find_slot(const TreeView& t, unsigned long long key) {
  const unsigned long long hk = mix64(key);
  uint32_t base = (uint32_t)hk & t.h_mask & ~(kBucket - 1);
  const uint32_t rot = (uint32_t)(hk >> 40) & (kBucket - 1);
  const uint32_t lines = (t.h_mask + 1) / kBucket;
  for (uint32_t n = 0; n < lines; ++n) {
    uint32_t best = kBucket;
    int at = -1;
    bool empty = false;
    for (int j = 0; j < (int)kBucket; ++j) {
      const unsigned long long cur = t.h_slot[base + j].key;
      const uint32_t pos = ((uint32_t)j - rot) & (kBucket - 1);
      if ((cur == kEmptyKey || (cur & ~kStampMask) == key) && pos < best) {
        best = pos;
        at = j;
        empty = cur == kEmptyKey;
      }
    }
    if (at >= 0) return empty ? ~0u : base + (uint32_t)at;
    base = (base + kBucket) & t.h_mask;
  }
  return ~0u;
}

__global__ void k_reroot_find(TreeView t, int a, int obs, int ob, int* out) {
  if (threadIdx.x != 0) return;
  const uint32_t h = find_slot(t, belief_key(0, key_low(a, obs, ob)));
  out[0] = h == ~0u ? -1 : t.h_slot[h].id;
}

// Source belief of position i of the launch's level steps, or -1.
__device__ __forceinline__ int reroot_record(const RerootView& V, long long i) {
  const RerootStep st = V.steps[i / V.src_n_p];
  const int ep = (int)(i % V.src_n_p);
  bool there;
  if (st.iter < 0) {                          // a kept subtree's step: packed
    there = ep < st.n;
  } else {
    const uint32_t run = V.src.run[(size_t)st.iter * (size_t)V.src_n_p + ep];
    const int top = (int)(run & kRunMask) - 1;
    there = st.level >= top && st.level < top + (int)((run >> kRunLenShift) & kRunMask);
  }
  return there ? (int)(1 + (size_t)st.step * (size_t)V.src_n_p + (size_t)ep) : -1;
}

// Mark pass: kept[r] for the beliefs of one source depth, with counts of the
// kept beliefs and of their action nodes (and, at depth 1, the root's visits).
__global__ __launch_bounds__(kBlock) void k_reroot_mark(RerootView V) {
  const long long i = (long long)blockIdx.x * kBlock + threadIdx.x;
  unsigned long long nb = 0, nn = 0, nv = 0;
  if (i < (long long)V.n_steps * V.src_n_p) {
    const int r = reroot_record(V, i);
    if (r > 0) {
      bool keep;
      if (V.src_depth == 1) {
        keep = r == V.root_rec;
      } else {
        keep = V.kept[own_of(V.src, r, V.src.node[r].link, V.src_n_p) >> kKeyLowBits] != 0;
      }
      if (keep) {
        V.kept[r] = 1;
        nb = 1;
        const uint32_t link = V.src.node[r].link;
        const int* n = rec_n(V.src, r);
        const uint32_t* bits = rec_bits(V.src, r);
        const bool wide = V.src.ra > kMaxA;   // long rows: columns valid per bitmap
        const bool full = has_row(V.src, link);
        if (!full) nn = nv = (link & kLinkAct) ? 1ull : 0ull;
        for (int j = 0; full && j < V.A; ++j) {
          const int c = (!wide || ((bits[j >> 5] >> (j & 31)) & 1u)) ? n[j] : 0;
          nn += c > 0 ? 1ull : 0ull;
          nv += (unsigned long long)(c > 0 ? c : 0);
        }
      }
    }
  }
  nb = wave_sum(nb);
  nn = wave_sum(nn);
  nv = wave_sum(nv);
  if ((threadIdx.x & 63) == 0 && nb) {
    atomicAdd(&V.cnt[V.src_depth], nb);
    atomicAdd(&V.cnt[kRerootCnt + V.src_depth], nn);
    if (V.src_depth == 1) atomicAdd(&V.cnt[2 * kRerootCnt + 1], nv);
  }
}

// Copy pass: each kept belief of one source depth gets the next position of
// its new depth's level steps (the root: record 0), its record is copied with
// the fixed-point sums rescaled, and it is inserted in the destination table
// under its new parent's slot id.
__global__ __launch_bounds__(kBlock) void k_reroot_copy(RerootView V) {
  const long long i = (long long)blockIdx.x * kBlock + threadIdx.x;
  if (i >= (long long)V.n_steps * V.src_n_p) return;
  const int r = reroot_record(V, i);
  if (r <= 0 || !V.kept[r]) return;
  const int d_new = V.src_depth - 1;
  int nr = 0;
  if (d_new > 0) {
    const unsigned long long q = atomicAdd(&V.cnt[3 * kRerootCnt + d_new], 1ull);
    const long long t = (long long)V.first_step + (long long)(q / (unsigned long long)V.dst_n_p);
    nr = (int)(1 + t * V.dst_n_p + (long long)(q % (unsigned long long)V.dst_n_p));
  }
  V.new_id[r] = nr;
  const BeliefNode b = V.src.node[r];
  const bool full = has_row(V.src, b.link);
  const OneNode one = one_node(b, V.obs_bits, V.src_scale);
  const int ra = V.src.ra;
  const bool wide = ra > kMaxA;             // long rows: columns valid per bitmap
  for (int j = 0; j < V.src.bw; ++j)
    rec_bits(V.dst, nr)[j] =
        full ? rec_bits(V.src, r)[j] : one.a >> 5 == j ? 1u << (one.a & 31) : 0u;
  unsigned long long* c = rec_c(V.dst, nr);
  unsigned long long* w = rec_w(V.dst, nr);
  for (int j = 0; j < ra; ++j) {
    rec_psi(V.dst, nr)[j] = full ? rec_psi(V.src, r)[j] : j == one.a ? one.psi : V.src.psi0[j];
    if (wide && !((rec_bits(V.dst, nr)[j >> 5] >> (j & 31)) & 1u)) continue;
    rec_n(V.dst, nr)[j] = full ? rec_n(V.src, r)[j] : j == one.a ? one.n : 0;
    unsigned long long cj = full ? rec_c(V.src, r)[j] : j == one.a ? one.c : 0ull;
    if (V.rescale != 1.0 && cj)
      cj = (unsigned long long)llrint((double)(long long)cj * V.rescale);
    c[j] = cj;
    w[j] = 0ull;
  }
  BeliefNode nb;
  nb.V = b.V;
  nb.link = kLinkFull;
  nb.u.leaf_h = 0ull;
  V.dst.node[nr] = nb;
  const int Nb = (b.link & kLinkFull) ? V.src.info[r].Nb : 1;
  if (d_new == 0) {
    V.dst.info[nr] = BeliefInfo{0, Nb, kEmptyKey};
    return;
  }
  const unsigned long long own = own_of(V.src, r, b.link, V.src_n_p);
  const int np = V.new_id[(int)(own >> kKeyLowBits)];
  const unsigned long long key = belief_key(np, (uint32_t)(own & kLinkKey));
  V.dst.info[nr] = BeliefInfo{0, Nb, key};
  bool won = false, fresh = false;
  int id = -1;
  Bucket line;
  bucket_read(V.dst, key, line);
  const uint32_t h = probe(V.dst, line, key, kCarryStamp, 0, 0, won, fresh, id);
  if (h == ~0u || !won) {
    atomicOr((unsigned int*)&V.cnt[4 * kRerootCnt], 1u);
    return;
  }
  V.dst.h_slot[h].id = nr;
}

__global__ __launch_bounds__(kBlock) void k_fill16(uint4* p, size_t n, uint4 v) {
  for (size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x; i < n;
       i += (size_t)gridDim.x * kBlock)
    p[i] = v;
}

hipError_t launch_reroot_find(const TreeView& t, int a, int obs, int ob, int* out,
                              hipStream_t s) {
  hipLaunchKernelGGL(k_reroot_find, dim3(1), dim3(64), 0, s, t, a, obs, ob, out);
  return hipGetLastError();
}
static int reroot_blocks(const RerootView& V) {
  return (int)std::max(1ll, ((long long)V.n_steps * V.src_n_p + kBlock - 1) / kBlock);
}
hipError_t launch_reroot_mark(const RerootView& V, hipStream_t s) {
  if (V.n_steps <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_reroot_mark, dim3(reroot_blocks(V)), dim3(kBlock), 0, s, V);
  return hipGetLastError();
}
hipError_t launch_reroot_copy(const RerootView& V, hipStream_t s) {
  if (V.n_steps <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_reroot_copy, dim3(reroot_blocks(V)), dim3(kBlock), 0, s, V);
  return hipGetLastError();
}
hipError_t launch_fill16(void* p, size_t n, uint4 v, hipStream_t s) {
  if (n == 0) return hipSuccess;
  const int g = (int)std::min<size_t>((n + kBlock - 1) / kBlock, 8192);
  hipLaunchKernelGGL(k_fill16, dim3(g), dim3(kBlock), 0, s, reinterpret_cast<uint4*>(p), n, v);
  return hipGetLastError();
}

hipError_t launch_persistent(const PlanView* views, const PersistView& V, int n_blocks,
                             int amax, hipStream_t s) {
  hipLaunchKernelGGL(k_persist_reset, dim3((V.n + kBlock - 1) / kBlock), dim3(kBlock), 0, s, V);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const dim3 g(n_blocks), b(kBlock);
  if (amax <= 4) hipLaunchKernelGGL(k_batch_persistent<4>, g, b, 0, s, views, V);
  else if (amax <= 8) hipLaunchKernelGGL(k_batch_persistent<8>, g, b, 0, s, views, V);
  else hipLaunchKernelGGL(k_batch_persistent<16>, g, b, 0, s, views, V);
  return hipGetLastError();
}

int persistent_blocks_per_cu(int amax) {
  const void* f = amax <= 4 ? (const void*)k_batch_persistent<4>
                 : amax <= 8 ? (const void*)k_batch_persistent<8>
                             : (const void*)k_batch_persistent<16>;
  int n = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, f, kBlock, 0) != hipSuccess || n < 1)
    n = 1;
  return n;
}

hipError_t launch_batch(const PlanView* views, const BatchItem* items, int n_items,
                        int n_blocks, int amax, hipStream_t s) {
  if (n_blocks <= 0) return hipSuccess;
  const dim3 g(n_blocks), b(kBlock);
  if (amax <= 4) hipLaunchKernelGGL(k_batch<4>, g, b, 0, s, views, items, n_items);
  else if (amax <= 8) hipLaunchKernelGGL(k_batch<8>, g, b, 0, s, views, items, n_items);
  else hipLaunchKernelGGL(k_batch<16>, g, b, 0, s, views, items, n_items);
  return hipGetLastError();
}

}  // namespace vopp
