// Integer stage of the rasteriser on gfx950: compaction of the binned entries,
// the sort of their float32 depths (LSD radix, or by counting where they are
// few), and the tiles' lists -- for every tile the entries that touch it, in
// depth order -- with their [start, end) ranges.  The (tile, entry) pairs are never sorted: a wavefront takes 64
// depth-ordered entries and a patch of 8 x 8 tiles, and ballots of the columns
// and rows that the entries cover give each tile its entries, so a pair costs
// one write.  Which entries touch a patch is found by testing them all where
// that is cheap; otherwise each entry is emitted once per patch it touches
// (about a twelfth of the pairs) and these items are radix sorted by patch.
//
// Every kernel reads its element count from device memory and takes a grid
// sized by a host-side upper bound, so the stage needs no host round trip
// (and can be captured) when the pair capacity is fixed.
#include "internal.h"
#include "pairs.h"

namespace sixdgs {
namespace {

constexpr int kItems = 8;                     // items per thread
constexpr int kChunk = kBlock * kItems;       // items per workgroup (2048)
constexpr int kWaves = kBlock / 64;

__device__ __forceinline__ uint32_t load_count(const uint32_t* ptr, uint32_t fixed, uint32_t cap) {
  uint32_t c = ptr ? *ptr : fixed;
  return c < cap ? c : cap;
}

// Inclusive scan over a 64-lane wavefront.
__device__ __forceinline__ uint32_t wave_scan_incl(uint32_t x) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    uint32_t y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  return x;
}

// Exclusive scan of one value per thread over the workgroup of WAVES wavefronts;
// returns the exclusive prefix and the workgroup total.
template <int WAVES = kWaves>
__device__ __forceinline__ uint32_t block_scan_excl(uint32_t x, uint32_t& total) {
  __shared__ uint32_t s_w[WAVES];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  uint32_t inc = wave_scan_incl(x);
  if (lane == 63) s_w[wv] = inc;
  __syncthreads();
  uint32_t before = 0;
  total = 0;
#pragma unroll
  for (int w = 0; w < WAVES; w++) {
    const uint32_t s = s_w[w];
    before += (w < wv) ? s : 0u;
    total += s;
  }
  __syncthreads();
  return before + inc - x;
}

// ------------------------------------------------------------ radix sort
// The depth order's passes (the item sort's are further below): one kernel
// per pass, where each workgroup takes the next 2,048 items (4,096 from
// kLargeSort entries on) in ticket order, ranks them stably by digit in LDS, and
// finds where its items of each digit go by looking back over the per-digit
// counts that earlier workgroups publish (a status word per digit: aggregate of
// that workgroup alone, or inclusive prefix through it).  The global digit offsets come from a
// histogram of every pass taken before the first pass, so each pass reads and
// writes the data once.  Tickets make a workgroup wait only on workgroups that
// are already running; the wait is bounded and reports a timeout in the error
// word instead of spinning forever.
constexpr int kRItems = 16;
constexpr int kRItemsSmall = 8;           // short sorts: 2048 items per workgroup, 2x the workgroups
constexpr int64_t kLargeSort = 1 << 20;    // from this many entries the depth sort uses kRItems
constexpr int64_t kLargePairs = 1 << 27;   // from this pair capacity on the items' sort uses kRItems
// Items per thread of the item sort's workgroups (and items per emission
// block: kBlock times this); a dozen pairs are an item.  By the capacity, which
// sizes the fixed mode's grids whatever the scene: larger blocks then leave half
// as many workgroups to find nothing to do.  The stage with 8 and with 16: one
// 1600x900 view of 500k (17M pairs) at a capacity of 26M 185 and 197 us, 134M
// 197 and 195, 537M 277 and 223; 8 1080p views of 1M (49M) at 74M 444 and 456,
// 134M 464 and 455; 8 uneven views of 500k (74M) at 111M 554 and 563; 16 (146M)
// at 219M 988 and 953.
inline int sort_items(int64_t pcap) { return pcap >= kLargePairs ? kRItems : kRItemsSmall; }
constexpr uint32_t kStAgg = 1u << 30;
constexpr uint32_t kStIncl = 2u << 30;
constexpr uint32_t kStVal = kStAgg - 1u;
constexpr int kMaxSpin = 1 << 20;

// The global digit histograms are kept as kGhCopies copies that workgroups
// add into by workgroup index: every workgroup adds its counts of every digit
// at its end, and atomics on one word serialise (about 17 ns apart on MI355X:
// 800 workgroups adding into 128 words took 16 us, 14 of them waiting), so
// the copies cut each word's queue; readers sum the copies.
constexpr int kGhCopies = 16;
constexpr int kGhStride = kMaxPasses * 256;  // words from one copy to the next

__device__ __forceinline__ uint32_t* ghist_copy(uint32_t* ghist, int64_t blk) {
  return ghist + (blk % kGhCopies) * kGhStride;
}
// Total count of digit d in the histogram at g (one pass's row of copy 0).
__device__ __forceinline__ uint32_t ghist_total(const uint32_t* g, int d) {
  uint32_t s = 0;
#pragma unroll
  for (int c = 0; c < kGhCopies; c++) s += g[c * kGhStride + d];
  return s;
}

// Up to this many entries the depth sort counts, for each, the entries before
// it (k_rank).  The four radix passes take 26 us of 476 entries and 31 of 9,300:
// each waits for the one before and for earlier workgroups' counts.  Counting
// takes 5 and 15, but n^2 / 64 comparisons: all of 15,000 entries binned, the
// stage takes 73 us with it and 84 with the passes, all of 20,000, 85 and 85
// (half of 30,000, 72 and 83, but half is not promised).
constexpr int64_t kRankEntries = 20480;
// Entries that a wavefront of it compares 256 with: more wavefronts for the
// fewest, fewer atomic adds to each place for more (9,300 entries: 34 us with
// segments of 16, 20 of 32, 15 of 64).
inline uint32_t rank_segment(int64_t E) { return E <= 2048 ? 16u : 64u; }
inline bool rank_entries(int64_t E) { return E <= kRankEntries; }

// Radix state of one sort: global digit histograms, tickets and look-back
// status words, laid out in one buffer.
struct RadixState {
  uint32_t* ghist;        // [kGhCopies][kMaxPasses][256]
  uint32_t* tickets;      // [kMaxPasses] passes, then [2] scans (padded to 256 words)
  uint32_t* status;       // [kMaxPasses][nblk][256]: look-back words (depth sort), chunk tables (item sort)
  uint64_t* scan_status;  // [2][nscan] look-back words of the two scans over entries
  int64_t nblk, nscan;
  int64_t nplace;         // words after the scans' for the places of a short depth sort
  int items;              // items per thread of the passes
  __host__ __device__ int64_t words() const {
    return (int64_t)kMaxPasses * 256 * (nblk + 1 + kGhCopies) + 4 * nscan + nplace;
  }
};

inline int64_t radix_blocks(int64_t bound, int items) {
  const int64_t chunk = (int64_t)kBlock * items;
  return (bound + chunk - 1) / chunk;
}

// extra: words between the tickets and the status words.
RadixState radix_state(uint32_t* base, int64_t bound, int items, bool with_scans, int64_t extra = 0) {
  RadixState r;
  r.items = items;
  r.nblk = radix_blocks(bound, items);
  r.nscan = with_scans ? (bound + kChunk - 1) / kChunk : 0;
  r.nplace = with_scans && rank_entries(bound) ? (bound + 3) / 4 * 4 : 0;
  r.ghist = base;
  r.tickets = base + kGhCopies * kGhStride;
  r.status = base + (kGhCopies + 1) * kGhStride + extra;
  r.scan_status = reinterpret_cast<uint64_t*>(r.status + (int64_t)kMaxPasses * r.nblk * 256);
  return r;
}

// Pass layout of a key with `bits` significant bits: ceil(bits / 8) passes of
// equal digit width (fewer buckets per pass when the key is short).
struct RadixPlan {
  int npass, dbits;
};
RadixPlan radix_plan(int bits) {
  RadixPlan p;
  p.npass = (bits + 7) / 8;
  if (p.npass < 1) p.npass = 1;
  p.dbits = (bits + p.npass - 1) / p.npass;
  if (p.dbits < 1) p.dbits = 1;
  return p;
}

__device__ __forceinline__ uint32_t st_load(const uint32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_store(uint32_t* p, uint32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Exclusive prefix over earlier workgroups from their 64-bit look-back words
// (flag in the high half, a 32-bit sum in the low half); bounded wait.
constexpr uint64_t kSc64Agg = 1ull << 32;
constexpr uint64_t kSc64Incl = 2ull << 32;

__device__ __forceinline__ uint64_t st_load64(const uint64_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_store64(uint64_t* p, uint64_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Exclusive prefix over workgroups [0, blk) from their look-back words at
// status[j * stride] (an aggregate of workgroup j alone, or an inclusive
// prefix through it).  A window of predecessors is read per round trip and
// summed nearest first until an inclusive word; a word not yet published is
// waited on, boundedly (a timeout sets *err and gives up).
constexpr int kLookWin = 4;

__device__ __forceinline__ bool lb_incl(uint32_t s) { return (s & kStIncl) != 0; }
__device__ __forceinline__ uint32_t lb_val(uint32_t s) { return s & kStVal; }
__device__ __forceinline__ uint32_t lb_load(const uint32_t* p) { return st_load(p); }
__device__ __forceinline__ bool lb_incl(uint64_t s) { return (s & kSc64Incl) != 0; }
__device__ __forceinline__ uint32_t lb_val(uint64_t s) { return (uint32_t)s; }
__device__ __forceinline__ uint64_t lb_load(const uint64_t* p) { return st_load64(p); }

template <class W>
__device__ uint32_t look_back(const W* status, int64_t stride, int64_t blk, uint32_t* err) {
  uint32_t excl = 0;
  for (int64_t j = blk - 1; j >= 0; j -= kLookWin) {
    W s[kLookWin];
#pragma unroll
    for (int k = 0; k < kLookWin; k++) s[k] = (j - k >= 0) ? lb_load(status + (j - k) * stride) : W(0);
#pragma unroll
    for (int k = 0; k < kLookWin; k++) {
      if (j - k < 0) return excl;  // not reached: the first workgroup publishes an inclusive word
      W v = s[k];
      for (int spin = 0; !v && spin < kMaxSpin; spin++) {
        __builtin_amdgcn_s_sleep(1);
        v = lb_load(status + (j - k) * stride);
      }
      if (!v) {
        atomicOr(err, 1u);
        return excl;
      }
      excl += lb_val(v);
      if (lb_incl(v)) return excl;
    }
  }
  return excl;
}

constexpr int kPsum = 16, kPsumStride = 16;  // 64-bit words of one sum, a cache line apart

// A workgroup's total of x (each wavefront's saturated), added to *sum.
template <int WAVES>
__device__ __forceinline__ void block_add(uint32_t x, uint64_t* sum) {
  __shared__ uint32_t s_w[WAVES];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x = __builtin_elementwise_add_sat(x, (uint32_t)__shfl_xor((int)x, o, 64));
  if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = x;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint64_t all = 0;
#pragma unroll
    for (int w = 0; w < WAVES; w++) all += s_w[w];
    if (all) atomicAdd(reinterpret_cast<unsigned long long*>(sum), (unsigned long long)all);
  }
}

// Single-pass exclusive scan of f(i) over i < count, handing (i, prefix,
// value) to g.  Workgroups take 2048 items each in ticket order (8192 from
// kLargeSort items on, where taking the tickets, 17 ns apart, bounded it: 8M
// entries 101 -> 61 us) and chain their prefixes through look-back words; the workgroup holding the last item
// writes the total.  With HIST, g.key(i) of every item with a non-zero value
// also enters the digit histograms of a 4-pass, 8-bit radix sort.
template <class F, class G, bool FLAGS, bool HIST, int THREADS>
__global__ void __launch_bounds__(THREADS) k_scan1(F f, G g, const uint32_t* count_ptr, uint32_t fixed, uint32_t cap,
                                                  uint32_t* ticket, uint64_t* status, uint32_t* total_out,
                                                  uint32_t* ghist, uint64_t* psum, HostCount host, uint32_t* err) {
  __shared__ uint32_t s_blk, s_pre;
  __shared__ uint32_t s_h[HIST ? kMaxPasses : 1][256];
  constexpr int kChunkT = THREADS * kItems;
  const int t = threadIdx.x;
  if (t == 0) s_blk = atomicAdd(ticket, 1u);
  if (HIST && t < 256) {
#pragma unroll
    for (int p = 0; p < kMaxPasses; p++) s_h[p][t] = 0;
  }
  __syncthreads();
  const int64_t blk = s_blk;
  const uint32_t count = load_count(count_ptr, fixed, cap);
  const int64_t start = blk * kChunkT;
  if (start >= count) {  // uniform
    if (blk == 0 && t == 0 && total_out) {
      *total_out = 0u;
      publish(host, 0u);
    }
    return;
  }
  const int64_t base = start + (int64_t)t * kItems;
  uint32_t v[kItems];
  uint32_t sum = 0;
#pragma unroll
  for (int k = 0; k < kItems; k++) {
    v[k] = (base + k < count) ? f(base + k) : 0u;
    sum += v[k];
  }
  uint32_t key[FLAGS ? kItems : 1];
  if constexpr (FLAGS) {
    sum = 0;
#pragma unroll
    for (int k = 0; k < kItems; k++) sum = __builtin_elementwise_add_sat(sum, v[k]);
    block_add<THREADS / 64>(sum, &psum[blk % kPsum * kPsumStride]);
    sum = 0;
#pragma unroll
    for (int k = 0; k < kItems; k++) {
      key[k] = v[k] ? g.key(base + k) : 0u;
      v[k] = v[k] ? 1u : 0u;
      sum += v[k];
    }
  }
  uint32_t total;
  uint32_t pre = block_scan_excl<THREADS / 64>(sum, total);
  uint64_t* my = status + blk;
  if (t == 0) st_store64(my, (blk == 0 ? kSc64Incl : kSc64Agg) | total);
  if constexpr (HIST) {
    // (before the wait on earlier workgroups.)  The lanes whose upper digits
    // equal the first's add as one: depths share them, and same-address
    // shared-memory atomics serialise
#pragma unroll
    for (int k = 0; k < kItems; k++) {
      if (v[k]) {
        const bool leader = __lane_id() == (unsigned)(__ffsll((unsigned long long)__ballot(1)) - 1);
#pragma unroll
        for (int p = 0; p < kMaxPasses; p++) {
          const uint32_t d = (key[k] >> (8 * p)) & 255u;
          if (p < 2) {
            atomicAdd(&s_h[p][d], 1u);
          } else {
            const uint32_t d0 = __builtin_amdgcn_readfirstlane(d);
            const uint64_t same = __ballot(d == d0);
            if (d != d0)
              atomicAdd(&s_h[p][d], 1u);
            else if (leader)
              atomicAdd(&s_h[p][d0], (uint32_t)__popcll(same));
          }
        }
      }
    }
  }
  if (t == 0) {
    uint32_t excl = 0;
    if (blk > 0) {
      excl = look_back(status, 1, blk, err);
      st_store64(my, kSc64Incl | (uint32_t)(excl + total));
    }
    s_pre = excl;
    if (start + kChunkT >= count && total_out) {
      *total_out = excl + total;
      publish(host, excl + total);
    }
  }
  __syncthreads();
  pre += s_pre;
#pragma unroll
  for (int k = 0; k < kItems; k++) {
    if constexpr (FLAGS) {
      if (v[k]) g.put(base + k, pre, key[k]);
    } else {
      if (base + k < count) g(base + k, pre, v[k]);
    }
    pre += v[k];
  }
  if constexpr (HIST) {  // (every wavefront's adds are in: the barrier above)
    uint32_t* gh = ghist_copy(ghist, blk);
#pragma unroll
    for (int p = 0; p < kMaxPasses; p++)
      if (t < 256 && s_h[p][t]) atomicAdd(&gh[p * 256 + t], s_h[p][t]);
  }
}

template <bool FLAGS, bool HIST, class F, class G>
void scan1(F f, G g, const uint32_t* count_ptr, uint32_t fixed, uint32_t cap, int64_t bound, uint32_t* ticket,
           uint64_t* status, uint32_t* total_out, uint32_t* ghist, uint64_t* psum, HostCount host, uint32_t* err, hipStream_t st) {
  auto launch = [&](auto kernel, int threads) {
    const int64_t chunk = (int64_t)threads * kItems;
    const int64_t nb = std::max<int64_t>((bound + chunk - 1) / chunk, 1);  // one workgroup writes a zero total
    hipLaunchKernelGGL(kernel, dim3((unsigned)nb), dim3(threads), 0, st, f, g, count_ptr, fixed, cap, ticket, status,
                       total_out, ghist, psum, host, err);
  };
  if (bound >= kLargeSort)
    launch(k_scan1<F, G, FLAGS, HIST, 1024>, 1024);
  else
    launch(k_scan1<F, G, FLAGS, HIST, kBlock>, kBlock);
}

// Up to four word ranges a preparation kernel zeroes.
struct ZeroList {
  uint32_t* p[4];
  int64_t n[4];
};

// Zeroes the first zero_words words of a radix state, the regions of z and
// the tile ranges; when given the depth-sorted entries, records for every
// emission block the sorted entry whose pairs contain the block's first pair
// (normally the item-offset scan records them; this is for pair buffers that
// were regrown after it).
__global__ void __launch_bounds__(kBlock) k_stage_prep(RadixState rs, int64_t zero_words, ZeroList z,
                                                       uint2* __restrict__ ranges, int64_t nranges,
                                                       const uint32_t* __restrict__ counters,
                                                       const uint32_t* __restrict__ total,
                                                       const uint32_t* __restrict__ poff, uint32_t pcap,
                                                       uint32_t* __restrict__ blk_start, int64_t nblk_start,
                                                       uint32_t chunk) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i < zero_words / 4) reinterpret_cast<uint4*>(rs.ghist)[i] = make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
  for (int k = 0; k < 4; k++)
    if (z.p[k] && i < z.n[k]) z.p[k][i] = 0u;
  if (ranges && i < nranges) ranges[i] = make_uint2(0xFFFFFFFFu, 0u);  // a patch without items
  if (blk_start && i < (int64_t)counters[0] && counters[1] <= pcap) {
    const uint32_t o = poff[i];
    const uint32_t end = i + 1 < (int64_t)counters[0] ? poff[i + 1] : *total;
    for (uint32_t b = (o + chunk - 1) / chunk; (int64_t)b * chunk < end && b < nblk_start; b++)
      blk_start[b] = (uint32_t)i;
  }
}

// One stable pass over the digit at `shift` (width dbits) of keys[0, count).
template <int ITEMS>
__global__ void __launch_bounds__(kBlock) k_onesweep(const uint32_t* __restrict__ kin,
                                                     const uint32_t* __restrict__ vin, uint32_t* __restrict__ kout,
                                                     uint32_t* __restrict__ vout, const uint32_t* count_ptr,
                                                     uint32_t cap, int shift, int dbits,
                                                     const uint32_t* __restrict__ ghist, uint32_t* ticket,
                                                     uint32_t* status, uint32_t* err) {
  constexpr int kChunkI = kBlock * ITEMS;
  constexpr int kWaveItems = kChunkI / kWaves;
  __shared__ uint32_t s_key[kChunkI];
  __shared__ uint32_t s_val[kChunkI];
  __shared__ uint32_t s_wc[kWaves][256];  // per-wave digit counts, then exclusive prefixes over waves
  __shared__ uint32_t s_lex[256];         // exclusive digit offsets inside the workgroup
  __shared__ uint32_t s_gb[256];          // output position of LDS slot 0 of each digit
  __shared__ uint32_t s_blk;
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  if (t == 0) s_blk = atomicAdd(ticket, 1u);
#pragma unroll
  for (int w = 0; w < kWaves; w++) s_wc[w][t] = 0;
  __syncthreads();
  const int64_t blk = s_blk;
  const uint32_t count = load_count(count_ptr, cap, cap);
  const int64_t base = blk * kChunkI;
  if (base >= count) return;  // uniform; no later workgroup has items, so none waits on this one
  const uint32_t mask = (1u << dbits) - 1u;
  const bool own = (uint32_t)t <= mask;
  const uint32_t gh = own ? ghist_total(ghist, t) : 0u;  // issued early: used after the look-back
  const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  const int64_t wbase = base + (int64_t)wv * kWaveItems;  // each wavefront ranks consecutive items
  uint32_t key[ITEMS], val[ITEMS], loc[ITEMS];
#pragma unroll
  for (int r = 0; r < ITEMS; r++) {
    const int64_t i = wbase + r * 64 + lane;
    key[r] = i < count ? kin[i] : 0u;
    val[r] = i < count ? vin[i] : 0u;
  }
  // every key has the same digit in this pass (e.g. the exponent byte of
  // depths within one octave): the stable order is the input order, so the
  // pass is a copy (decided while the loads are in flight)
  if (__syncthreads_or(own && gh == count)) {
#pragma unroll
    for (int r = 0; r < ITEMS; r++) {
      const int64_t i = wbase + r * 64 + lane;
      if (i < count) {
        kout[i] = key[r];
        vout[i] = val[r];
      }
    }
    return;
  }
#pragma unroll
  for (int r = 0; r < ITEMS; r++) {
    const bool valid = wbase + r * 64 + lane < count;
    const uint32_t d = (key[r] >> shift) & mask;
    uint64_t m = __ballot(valid);
    for (int b = 0; b < dbits; b++) {
      const bool bit = (d >> b) & 1u;
      const uint64_t bb = __ballot(bit);
      m &= bit ? bb : ~bb;
    }
    const uint32_t rank = __popcll(m & lt);
    // every lane of a digit group reads the running count before its first lane moves it on
    const uint32_t pre = s_wc[wv][d];
    if (valid && rank == 0) s_wc[wv][d] = pre + (uint32_t)__popcll(m);
    loc[r] = valid ? ((pre + rank) << 8 | d) : 0xFFFFFFFFu;
  }
  __syncthreads();
  uint32_t tot = 0;
#pragma unroll
  for (int w = 0; w < kWaves; w++) {
    const uint32_t c = s_wc[w][t];
    s_wc[w][t] = tot;
    tot += c;
  }
  uint32_t* my = status + blk * 256 + t;
  if (own) st_store(my, (blk == 0 ? kStIncl : kStAgg) | tot);
  uint32_t total;
  const uint32_t lex = block_scan_excl(tot, total);
  s_lex[t] = lex;
  __syncthreads();
#pragma unroll
  for (int r = 0; r < ITEMS; r++) {
    if (loc[r] != 0xFFFFFFFFu) {
      const uint32_t d = loc[r] & 255u;
      const uint32_t pos = s_lex[d] + s_wc[wv][d] + (loc[r] >> 8);
      if (pos < (uint32_t)kChunkI) {  // always true; guards LDS against inconsistent counts
        s_key[pos] = key[r];
        s_val[pos] = val[r];
      }
    }
  }
  // exclusive prefix of this digit over the earlier workgroups
  uint32_t excl = 0;
  if (own && blk > 0) {
    excl = look_back(status + t, 256, blk, err);
    st_store(my, kStIncl | (excl + tot));
  }
  const uint32_t gex = block_scan_excl(gh, total);
  s_gb[t] = gex + excl - lex;  // modular: adding an LDS slot of this digit lands in range
  __syncthreads();
  const int64_t left = (int64_t)count - base;
  const int nvalid = left < kChunkI ? (int)left : kChunkI;
#pragma unroll
  for (int r = 0; r < ITEMS; r++) {
    const int k = r * kBlock + t;
    if (k < nvalid) {
      const uint32_t kk = s_key[k];
      const uint32_t o = s_gb[(kk >> shift) & mask] + (uint32_t)k;
      if (o < count) {  // always true for a consistent histogram; guards the buffers
        kout[o] = kk;
        vout[o] = s_val[k];
      }
    }
  }
}

// ---------------------------------------------------- reduce-then-scan passes
// The item sort's passes in three launches with no chain between workgroups
// (the wait on earlier workgroups' counts dominated the one-kernel passes at
// a few thousand workgroups, and the emission counts the first pass's chunks
// for free):
// each chunk's digit counts (2,048 or 4,096 items, sort_items; k_digit_count;
// for the first pass the emission writes them), one scan per digit over the
// chunks, offset by the
// counts of the smaller digits (k_digit_scan), and the stable scatter
// (k_digit_scatter), where chunk b's items of digit d start at the scanned
// table entry (d, b).  The tables are [digit][chunk]; chunks past the item
// count are read as zero.

// Stable ranks of the workgroup's items by digit, each wavefront over its
// consecutive items (ballot matching): loc[r] = (rank in the wavefront << 8) |
// digit, or ~0 past the count; on return wc[w][d] holds the count of digit d in
// the wavefronts before w, and the return value is the workgroup's count of
// digit threadIdx.x.
template <int ITEMS>
__device__ __forceinline__ uint32_t rank_chunk(uint32_t (*wc)[256], const uint32_t (&key)[ITEMS], int64_t wbase,
                                               uint32_t count, int shift, int dbits, uint32_t (&loc)[ITEMS]) {
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const uint32_t mask = (1u << dbits) - 1u;
  const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
#pragma unroll
  for (int r = 0; r < ITEMS; r++) {
    const bool valid = wbase + r * 64 + lane < count;
    const uint32_t d = (key[r] >> shift) & mask;
    uint64_t m = __ballot(valid);
    for (int b = 0; b < dbits; b++) {
      const bool bit = (d >> b) & 1u;
      const uint64_t bb = __ballot(bit);
      m &= bit ? bb : ~bb;
    }
    const uint32_t rank = __popcll(m & lt);
    // every lane of a digit group reads the running count before its first lane moves it on
    const uint32_t pre = wc[wv][d];
    if (valid && rank == 0) wc[wv][d] = pre + (uint32_t)__popcll(m);
    loc[r] = valid ? ((pre + rank) << 8 | d) : 0xFFFFFFFFu;
  }
  __syncthreads();
  uint32_t tot = 0;
#pragma unroll
  for (int w = 0; w < kWaves; w++) {
    const uint32_t c = wc[w][t];
    wc[w][t] = tot;
    tot += c;
  }
  return tot;
}

template <int ITEMS>
__global__ void __launch_bounds__(kBlock) k_digit_count(const uint32_t* __restrict__ kin, const uint32_t* count_ptr,
                                                        uint32_t cap, int shift, int dbits,
                                                        uint32_t* __restrict__ table, int64_t nblk) {
  constexpr int kChunkI = kBlock * ITEMS;
  __shared__ uint32_t s_wc[kWaves][256];
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int64_t blk = blockIdx.x;
  const uint32_t count = load_count(count_ptr, cap, cap);
  const int64_t base = blk * kChunkI;
  if (base >= count) return;  // uniform
#pragma unroll
  for (int w = 0; w < kWaves; w++) s_wc[w][t] = 0;
  __syncthreads();
  const int64_t wbase = base + (int64_t)wv * (kChunkI / kWaves);
  uint32_t key[ITEMS], loc[ITEMS];
#pragma unroll
  for (int r = 0; r < ITEMS; r++) {
    const int64_t i = wbase + r * 64 + lane;
    key[r] = i < count ? kin[i] : 0u;
  }
  const uint32_t tot = rank_chunk<ITEMS>(s_wc, key, wbase, count, shift, dbits, loc);
  if ((uint32_t)t < (1u << dbits)) table[(int64_t)t * nblk + blk] = tot;
}

// One workgroup per digit d: table[d][b] <- (items of digits < d) + (items of
// digit d in chunks < b), over the chunks that hold items.
__global__ void __launch_bounds__(kBlock) k_digit_scan(uint32_t* __restrict__ table, int64_t nblk,
                                                       const uint32_t* count_ptr, uint32_t cap, int chunk_items,
                                                       const uint32_t* __restrict__ ghist) {
  const int d = blockIdx.x, t = threadIdx.x;
  const uint32_t count = load_count(count_ptr, cap, cap);
  const int64_t used = ((int64_t)count + chunk_items - 1) / chunk_items;
  uint32_t dbase;  // items of the digits below d: the total of this scan
  block_scan_excl((uint32_t)t < (uint32_t)d ? ghist_total(ghist, t) : 0u, dbase);
  uint32_t* row = table + (int64_t)d * nblk;
  const int64_t per = (used + kBlock - 1) / kBlock;
  const int64_t b0 = min<int64_t>((int64_t)t * per, used), b1 = min<int64_t>(b0 + per, used);
  uint32_t sum = 0;
  for (int64_t b = b0; b < b1; b++) sum += row[b];
  uint32_t all;
  uint32_t pre = dbase + block_scan_excl(sum, all);
  for (int64_t b = b0; b < b1; b++) {
    const uint32_t c = row[b];
    row[b] = pre;
    pre += c;
  }
}

template <int ITEMS>
__global__ void __launch_bounds__(kBlock) k_digit_scatter(const uint32_t* __restrict__ kin,
                                                          const uint32_t* __restrict__ vin, uint32_t* __restrict__ kout,
                                                          uint32_t* __restrict__ vout, const uint32_t* count_ptr,
                                                          uint32_t cap, int shift, int dbits,
                                                          const uint32_t* __restrict__ table, int64_t nblk) {
  constexpr int kChunkI = kBlock * ITEMS;
  __shared__ uint32_t s_key[kChunkI];
  __shared__ uint32_t s_val[kChunkI];
  __shared__ uint32_t s_wc[kWaves][256];
  __shared__ uint32_t s_lex[256];
  __shared__ uint32_t s_gb[256];
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int64_t blk = blockIdx.x;
  const uint32_t count = load_count(count_ptr, cap, cap);
  const int64_t base = blk * kChunkI;
  if (base >= count) return;  // uniform
  const uint32_t mask = (1u << dbits) - 1u;
  const bool own = (uint32_t)t <= mask;
  const uint32_t gstart = own ? table[(int64_t)t * nblk + blk] : 0u;  // issued early
#pragma unroll
  for (int w = 0; w < kWaves; w++) s_wc[w][t] = 0;
  __syncthreads();
  const int64_t wbase = base + (int64_t)wv * (kChunkI / kWaves);
  uint32_t key[ITEMS], val[ITEMS], loc[ITEMS];
#pragma unroll
  for (int r = 0; r < ITEMS; r++) {
    const int64_t i = wbase + r * 64 + lane;
    key[r] = i < count ? kin[i] : 0u;
    val[r] = i < count ? vin[i] : 0u;
  }
  const uint32_t tot = rank_chunk<ITEMS>(s_wc, key, wbase, count, shift, dbits, loc);
  uint32_t total;
  const uint32_t lex = block_scan_excl(tot, total);
  s_lex[t] = lex;
  s_gb[t] = gstart - lex;  // modular: adding an LDS slot of this digit lands in range
  __syncthreads();
#pragma unroll
  for (int r = 0; r < ITEMS; r++) {
    if (loc[r] != 0xFFFFFFFFu) {
      const uint32_t d = loc[r] & 255u;
      const uint32_t pos = s_lex[d] + s_wc[wv][d] + (loc[r] >> 8);
      if (pos < (uint32_t)kChunkI) {  // always true; guards LDS against inconsistent counts
        s_key[pos] = key[r];
        s_val[pos] = val[r];
      }
    }
  }
  __syncthreads();
  const int64_t left = (int64_t)count - base;
  const int nvalid = left < kChunkI ? (int)left : kChunkI;
#pragma unroll
  for (int r = 0; r < ITEMS; r++) {
    const int k = r * kBlock + t;
    if (k < nvalid) {
      const uint32_t kk = s_key[k];
      const uint32_t o = s_gb[(kk >> shift) & mask] + (uint32_t)k;
      if (o < count) {  // always true for consistent tables; guards the buffers
        kout[o] = kk;
        vout[o] = s_val[k];
      }
    }
  }
}

// Sorts (keys, vals) of length *count_ptr (<= bound) over plan.npass digits
// whose histograms are already in rs.ghist; returns which buffer of the
// ping-pong pair holds the result.
int radix_sort(uint32_t* keys[2], uint32_t* vals[2], const uint32_t* count_ptr, int64_t bound, RadixPlan plan,
               const RadixState& rs, uint32_t* err, hipStream_t st) {
  const int64_t nb = rs.nblk;
  int cur = 0;
  if (nb == 0) return cur;
  for (int p = 0; p < plan.npass; p++) {
    auto k = rs.items == kRItems ? k_onesweep<kRItems> : k_onesweep<kRItemsSmall>;
    hipLaunchKernelGGL(k, dim3((unsigned)nb), dim3(kBlock), 0, st, keys[cur], vals[cur], keys[cur ^ 1],
                       vals[cur ^ 1], count_ptr, (uint32_t)bound, p * plan.dbits, plan.dbits, rs.ghist + p * 256,
                       rs.tickets + p, rs.status + (int64_t)p * rs.nblk * 256, err);
    cur ^= 1;
  }
  return cur;
}

// ------------------------------------------------------------ the stage
struct TileCount {
  const uint32_t* tiles;
  __device__ uint32_t operator()(int64_t i) const { return tiles[i]; }
};
struct CompactDepth {
  const float* depth;
  uint32_t* dkey;
  uint32_t* dval;
  // depths of binned entries exceed z_near > 0, so their bit patterns order as the values
  __device__ uint32_t key(int64_t i) const { return __float_as_uint(depth[i]); }
  __device__ void put(int64_t i, uint32_t pre, uint32_t key) const {
    dkey[pre] = key;
    dval[pre] = (uint32_t)i;
  }
};
// The tile rectangle of a sorted entry: x first | y first << 16, and x last | y
// last << 16, with y counted on from one view to the next by 2,048 (a view has
// at most 2,048 tiles each way, so each half is a non-negative int16 and one
// packed subtraction compares both); an empty one is in no patch.
__device__ __forceinline__ uint2 entry_rect(const ViewTable& vt, const Rec* rec, uint32_t e) {
  const uint32_t view = e / (uint32_t)vt.n;
  const ViewDesc& vd = vt.v[view];
  const float4 ra = rec[e].a, rb = rec[e].b;
  int x0, y0, x1, y1;
  tile_rect(ra.x, ra.y, rb.z, rb.w, vt.tile_shift_x, vt.tile_shift_y, vd.ntx, vd.nty, x0, y0, x1, y1);
  if (x1 <= x0 || y1 <= y0) return make_uint2(2047u, 0u);  // x last 0: before the first
  const uint32_t base = view << 27;
  return make_uint2((uint32_t)(x0 | y0 << 16) + base, (uint32_t)((x1 - 1) | (y1 - 1) << 16) + base);
}
static_assert(kMaxViews <= 16, "a rectangle's y halves hold 16 views of 2,048 tile rows");

// A short depth sort by counting: entry i's place is the number of entries j
// before it in (key, j) order.  A wavefront compares 256 entries with a segment
// of them and adds its counts to the entries' places (zero before).
__global__ void __launch_bounds__(kBlock) k_rank(const uint32_t* __restrict__ key,
                                                 const uint32_t* __restrict__ counters, uint32_t segment,
                                                 uint32_t* __restrict__ place) {
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t n = counters[0];
  const uint32_t i0 = (blockIdx.x * kWaves + wv) * 256, j0 = blockIdx.y * segment;
  if (i0 >= n || j0 >= n) return;
  // keys below ~0 (a caller's depth may be any bit pattern), so that one more is
  // still a key; ~0 past the last entry, before which everything is
  const uint32_t kj = j0 + lane < n ? min(key[j0 + lane], ~1u) : ~0u;
  uint32_t k[4], c[4] = {0, 0, 0, 0};
#pragma unroll
  for (int r = 0; r < 4; r++) {
    const uint32_t i = i0 + 64 * r + lane;
    k[r] = i < n ? min(key[i], ~1u) : 0u;
  }
  if (j0 >= i0 && j0 < i0 + 256) {  // the segment is in the wavefront's own 256: equal keys before i count
    const int own = (int)(j0 - i0) >> 6, off = (int)(j0 - i0) & 63;
    uint32_t ties = 0;
    for (int j = 0; j < (int)segment; j++)
      ties += (uint32_t)__builtin_amdgcn_readlane(kj, j) == (own == 0 ? k[0] : own == 1 ? k[1] : own == 2 ? k[2] : k[3]) && off + j < lane ? 1u : 0u;
#pragma unroll
    for (int r = 0; r < 4; r++) c[r] = r == own ? ties : 0u;
  }
#pragma unroll
  for (int r = 0; r < 4; r++) k[r] += j0 < i0 + 64 * r ? 1u : 0u;  // all before i: equal ones count
  for (int j = 0; j < (int)segment; j += 8)  // (segments are 16 or 64)
#pragma unroll
    for (int u = 0; u < 8; u++) {
      const uint32_t q = (uint32_t)__builtin_amdgcn_readlane(kj, j + u);
#pragma unroll
      for (int r = 0; r < 4; r++) c[r] += q < k[r] ? 1u : 0u;
    }
#pragma unroll
  for (int r = 0; r < 4; r++)
    if (i0 + 64 * r + lane < n && c[r]) atomicAdd(&place[i0 + 64 * r + lane], c[r]);
}

// All sorted entries' rectangles, and the pair count from its partial sums.
// place: nullptr, or where each entry of the compacted list goes (then dsorted
// is written as well).
__global__ void __launch_bounds__(kBlock) k_rects(ViewTable vt, const Rec* __restrict__ rec,
                                                  const uint32_t* __restrict__ dval,
                                                  const uint32_t* __restrict__ place, uint32_t* __restrict__ dsorted,
                                                  const uint64_t* __restrict__ psum, HostCount host,
                                                  uint32_t* __restrict__ counters,
                                                  uint32_t* __restrict__ rect0, uint32_t* __restrict__ rect1) {
  const uint32_t i = blockIdx.x * kBlock + threadIdx.x;
  if (blockIdx.x == 0 && threadIdx.x < 64) {
    uint64_t sum = threadIdx.x < kPsum ? psum[threadIdx.x * kPsumStride] : 0u;
#pragma unroll
    for (int o = kPsum / 2; o > 0; o >>= 1) sum += (uint64_t)__shfl_xor((unsigned long long)sum, o, 64);
    if (threadIdx.x == 0) {
      const uint32_t s = pair_total(sum);
      counters[1] = s;
      counters[7] = 0u;
      publish(host, s);
    }
  }
  if (i >= counters[0]) return;
  const uint32_t e = dval[i];
  const uint2 r = entry_rect(vt, rec, e);
  uint32_t at = i;
  if (place) {
    at = place[i];
    if (at >= counters[0]) return;  // never; guards the buffers
    dsorted[at] = e;
  }
  rect0[at] = r.x;
  rect1[at] = r.y;
}

// The patches that a sorted entry's rectangle touches.
struct PatchCount {
  const uint32_t* rect0;
  const uint32_t* rect1;
  __device__ uint32_t operator()(int64_t i) const {
    const uint32_t r0 = rect0[i], r1 = rect1[i];
    const int w = (int)((r1 >> 3) & 255u) - (int)((r0 >> 3) & 255u) + 1;
    const int h = (int)((r1 >> 19) & 255u) - (int)((r0 >> 19) & 255u) + 1;
    return w > 0 && h > 0 ? (uint32_t)(w * h) : 0u;
  }
};
struct CountVal {
  const uint32_t* c;
  __device__ uint32_t operator()(int64_t i) const { return c[i]; }
};
struct StoreRange {
  uint2* ranges;
  uint32_t pcap;
  __device__ void operator()(int64_t i, uint32_t pre, uint32_t n) const {
    const PairRange r = pair_range(pre, n, pcap);
    ranges[i] = make_uint2(r.first, r.end);
  }
};
// The item offset of each depth-sorted entry, and for every emission block
// that starts inside the entry's items, the entry.
struct StoreOffset {
  uint32_t* poff;
  uint32_t* blk_start;
  int64_t nblk_start;
  int64_t chunk;  // items per emission block
  __device__ void operator()(int64_t i, uint32_t pre, uint32_t n) const {
    poff[i] = pre;
    for (int64_t b = ((int64_t)pre + chunk - 1) / chunk; b * chunk < (int64_t)pre + n && b < nblk_start; b++)
      blk_start[b] = (uint32_t)i;
  }
};

// whether the call's pairs did not fit (no list is written then)
__device__ __forceinline__ bool overflowed(const uint32_t* counters, uint32_t pcap) {
  return max(counters[1], counters[7]) > pcap;
}

// Load-balanced emission of the (patch, entry) items: workgroup b writes items
// [chunk b, chunk (b + 1)) in depth order.  It walks the depth-sorted entries
// from the one holding its first item, 256 entries per step; each thread finds
// the entry of an item by binary search over the entries' item offsets in LDS
// and the item's patch from its index in the entry's rectangle of patches
// (row-major, the order the count came from), so consecutive threads write
// consecutive items whatever the entries' sizes.  The digit histograms of every
// pass of the sort are accumulated on the way.  An item's key: the patch's id,
// and above its 20 bits the tiles of the patch that the entry covers (x first,
// x last, y first, y last, 3 bits each).
constexpr uint32_t kPatchMask = (1u << 20) - 1u;

__global__ void __launch_bounds__(kBlock) k_emit(ViewTable vt, const uint32_t* __restrict__ rect0,
                                                 const uint32_t* __restrict__ rect1,
                                                 const uint32_t* __restrict__ dval, const uint32_t* __restrict__ poff,
                                                 const uint32_t* __restrict__ blk_start,
                                                 uint32_t* __restrict__ counters, uint32_t pcap, int npass, int dbits,
                                                 uint32_t* __restrict__ ghist, uint32_t* __restrict__ pkey,
                                                 uint32_t* __restrict__ pval, uint32_t* __restrict__ table0,
                                                 uint32_t chunk) {
  __shared__ uint32_t s_o[kBlock + 1];  // item offset of each entry of the step; [kBlock]: the next step's
  __shared__ uint32_t s_e[kBlock];      // entry id
  __shared__ uint32_t s_r0[kBlock], s_r1[kBlock];  // its rectangle
  __shared__ uint32_t s_h[kMaxPasses][256];
  const int t = threadIdx.x;
  // blk_start holds an entry for every workgroup of the grid: read with the
  // counts, not after them
  uint32_t ib = blk_start[blockIdx.x];
  const uint32_t nb = counters[0];
  const uint32_t S = counters[7];
  if (overflowed(counters, pcap)) {
    if (blockIdx.x == 0 && t == 0) counters[2] = 1u;
    return;
  }
  const int64_t p0 = (int64_t)blockIdx.x * chunk;
  if (p0 >= S) return;  // uniform
  const uint32_t p1 = (uint32_t)min<int64_t>(p0 + chunk, (int64_t)S);
  const uint32_t mask = (1u << dbits) - 1u;
#pragma unroll
  for (int p = 0; p < kMaxPasses; p++) s_h[p][t] = 0;
  for (;;) {
    const uint32_t i = ib + t;
    if (i < nb) {
      const uint32_t o = poff[i];
      s_o[t] = o;
      // an entry whose items start past this block is never chosen by the
      // search below: its rectangle is not read
      if (o < p1) {
        s_e[t] = dval[i];
        s_r0[t] = rect0[i];
        s_r1[t] = rect1[i];
      }
    } else {
      s_o[t] = S;  // past the last entry: never chosen by the search below
    }
    if (t == 0) s_o[kBlock] = (uint64_t)ib + kBlock < nb ? poff[ib + kBlock] : S;
    __syncthreads();
    const uint32_t lo = max((uint32_t)p0, s_o[0]);
    const uint32_t hi = min(p1, s_o[kBlock]);
    for (uint32_t q = lo + t; q < hi; q += kBlock) {
      int j = 0;  // last entry of the step whose items start at or before q
#pragma unroll
      for (int step = kBlock / 2; step > 0; step >>= 1)
        if (s_o[j + step] <= q) j += step;
      const uint32_t local = q - s_o[j];
      const uint32_t r0 = s_r0[j], r1 = s_r1[j];
      const uint32_t px0 = (r0 >> 3) & 255u, px1 = (r1 >> 3) & 255u, py0 = (r0 >> 19) & 255u, py1 = (r1 >> 19) & 255u;
      const uint32_t w = px1 - px0 + 1;
      const uint32_t ty = local / w, px = px0 + (local - ty * w), py = py0 + ty;
      const uint32_t tiles = (px == px0 ? r0 & 7u : 0u) | (px == px1 ? r1 & 7u : 7u) << 3 |
                             (py == py0 ? (r0 >> 16) & 7u : 0u) << 6 | (py == py1 ? (r1 >> 16) & 7u : 7u) << 9;
      const ViewDesc& vd = vt.v[r0 >> 27];
      const uint32_t key = tiles << 20 | (vd.patch_base + py * ((vd.ntx + 7) >> 3) + px);
      pkey[q] = key;
      pval[q] = s_e[j];
      // Lanes whose digit equals the first active lane's add as one: same-address
      // shared-memory atomics from one wavefront serialise.
      const uint64_t act = __ballot(1);
      const bool leader = __lane_id() == (unsigned)(__ffsll((unsigned long long)act) - 1);
      for (int p = 0; p < npass; p++) {
        const uint32_t d = (key >> (p * dbits)) & mask;
        const uint32_t d0 = __builtin_amdgcn_readfirstlane(d);
        const uint64_t same = __ballot(d == d0);
        if (d != d0)
          atomicAdd(&s_h[p][d], 1u);
        else if (leader)
          atomicAdd(&s_h[p][d0], (uint32_t)__popcll(same));
      }
    }
    const bool done = s_o[kBlock] >= p1;
    __syncthreads();
    if (done) break;
    ib += kBlock;
  }
  uint32_t* gh = ghist_copy(ghist, blockIdx.x);
  for (int p = 0; p < npass; p++)
    if (s_h[p][t]) atomicAdd(&gh[p * 256 + t], s_h[p][t]);
  // this chunk's counts of the first pass's digits (the chunk is the pass's)
  if ((uint32_t)t <= mask) table0[(int64_t)t * gridDim.x + blockIdx.x] = s_h[0][t];
}

// Order in which the compositing kernels take the tiles: longest lists first
// (buckets of log2 of the pair count, heaviest bucket first), so the tiles
// whose per-pixel walks are longest start before the light ones and the
// kernels' tails shrink (LPT scheduling); the order inside a bucket is
// arbitrary.  k_list_scan counts the buckets, into kOrderCopies copies by
// patch; workgroups of the kernel that writes the lists then take
// kOrderTiles tiles each, reserve their places inside each bucket with one
// device atomic per bucket and write the order beside the others' lists.
constexpr int kOrderBuckets = 33;
constexpr int kOrderU = 4;                                  // tiles per thread
constexpr uint32_t kOrderTiles = kBlock * kOrderU;
constexpr int kOrderCopies = 16;
constexpr int kOrderStateWords = 64 * (kOrderCopies + 1);   // bucket counts, then bucket cursors

__host__ __device__ inline uint32_t order_wgs(uint32_t total_tiles) { return (total_tiles + kOrderTiles - 1) / kOrderTiles; }

// the bucket of a tile with c pairs (heaviest first: 0 holds 2^31 pairs and
// more, the last the empty tiles)
__device__ __forceinline__ int order_bucket(uint32_t c) { return kOrderBuckets - 1 - (c ? 32 - __clz(c) : 0); }

// A wavefront's lane l holds a counter of bucket l.  Per lane with b >= 0, adds
// one to bucket b's; returns what it was before for the first lane of a bucket,
// one more for the next ...  In registers, since a wavefront's tiles share a few
// buckets and shared-memory atomics on one word serialise (7,744 tiles took a
// workgroup 11 us that way).
__device__ __forceinline__ uint32_t bucket_add(uint32_t& n, int b) {
  const int lane = (int)__lane_id();
  uint32_t place = 0;
  for (uint64_t todo = __ballot(b >= 0); todo;) {
    const int b0 = __builtin_amdgcn_readlane(b, __ffsll((unsigned long long)todo) - 1);
    const uint64_t same = __ballot(b == b0);
    const uint32_t at = __builtin_amdgcn_mbcnt_hi((uint32_t)(same >> 32), __builtin_amdgcn_mbcnt_lo(
                                                                              (uint32_t)same, __builtin_amdgcn_readlane(n, b0)));
    place = b == b0 ? at : place;
    n += lane == b0 ? (uint32_t)__popcll(same) : 0u;
    todo &= ~same;
  }
  return place;
}

// Zeroes the gradient-accumulator row of entry i if it is binned (a tile
// count above zero).  Taken in entry order, consecutive threads write
// consecutive rows (the binned entries in depth order would scatter them),
// and the unbinned ones cost a 4-byte read.
__device__ __forceinline__ void zero_g2d_entry(int64_t i, const uint32_t* __restrict__ tiles, int64_t E,
                                               float* __restrict__ g2d) {
  if (i < E && tiles[i] > 0) {
    float* p = g2d + i * kG2D;
#pragma unroll
    for (int k = 0; k < kG2D; k++) p[k] = 0.f;
  }
}

// The order of tiles [wg * kOrderTiles, ...), by one workgroup.
__device__ __forceinline__ void order_tiles(const uint2* __restrict__ ranges, uint32_t total_tiles, uint32_t wg,
                                            uint32_t* __restrict__ state, uint32_t* __restrict__ order) {
  __shared__ uint32_t s_n[64];  // the workgroup's count per bucket, then its first place
  const uint32_t t = threadIdx.x, lane = t & 63;
  if (t < 64) s_n[t] = 0;
  __syncthreads();
  const uint32_t k0 = wg * kOrderTiles + t;
  int b[kOrderU];
#pragma unroll
  for (int u = 0; u < kOrderU; u++) {
    const uint32_t k = k0 + u * kBlock;
    const uint2 r = k < total_tiles ? ranges[k] : make_uint2(0u, 0u);
    b[u] = k < total_tiles ? order_bucket(r.y - r.x) : -1;
  }
  uint32_t n = 0;
#pragma unroll
  for (int u = 0; u < kOrderU; u++) bucket_add(n, b[u]);
  uint32_t at = n ? atomicAdd(&s_n[lane], n) : 0u;  // the wavefront's part
  __syncthreads();
  if (t < 64) {
    uint32_t c = 0;
#pragma unroll
    for (int k = 0; k < kOrderCopies; k++) c += state[64 * k + lane];
    const uint32_t off = wave_scan_incl(c) - c;  // first place of each bucket
    if (s_n[lane]) s_n[lane] = off + atomicAdd(&state[64 * kOrderCopies + lane], s_n[lane]);
  }
  __syncthreads();
  at += s_n[lane];
#pragma unroll
  for (int u = 0; u < kOrderU; u++) {
    const uint32_t pos = bucket_add(at, b[u]);
    if (b[u] >= 0 && pos < total_tiles) order[pos] = k0 + u * kBlock;
  }
}

// ----------------------------------------------------- the lists of the tiles
// A wavefront takes 64 depth-ordered entries that touch a patch.  Per entry, 8
// column and 8 row bits say which of the patch's 8 x 8 tiles it covers; the
// ballots of the bits are, per column and row, the entries that cover it; and
// the entries of a tile are those of its column and its row.  A first kernel
// counts them (lane t holds tile t's) into one row of a table per chunk of
// entries and patch; k_list_scan turns a patch's rows into exclusive prefixes and
// its tiles' totals; the scan of the totals over the tiles gives the ranges;
// the second kernel's lanes then know where their entries go, in each tile a
// dozen neighbours or so at a time.  Radix sorting the pairs (8 bytes) by tile
// moved each five times, 124 vector instructions per 64 and pass, and bound the
// stage by memory: 16 views of 500k Gaussians, 144M pairs, 3,235 us for the
// whole stage then and 953 now (283 of them the writes, 2.0 TB/s: runs of
// 50 bytes); one 1408x1408 view of 175k, 4.9M pairs, 181 and 106; one 800x800
// view of 300k, 3.4M pairs, 158 and 113.
__device__ __forceinline__ uint32_t readlane(uint32_t v, int l) { return __builtin_amdgcn_readlane(v, l); }
// lane q of (lo, hi) = m (a vector instruction may read a scalar register that
// another wrote two wait states later)
__device__ __forceinline__ void put_lane(uint32_t& lo, uint32_t& hi, uint64_t m, int q) {
  asm("s_nop 1\n\tv_writelane_b32 %0, %2, %4\n\tv_writelane_b32 %1, %3, %4"
      : "+v"(lo), "+v"(hi)
      : "s"((uint32_t)m), "s"((uint32_t)(m >> 32)), "n"(q));
}
// Has a loaded value waited for here: where it is next used, the wait would
// also be for the stores in between (one counter holds both).
__device__ __forceinline__ void arrived(uint32_t& v) { asm volatile("" : "+v"(v)); }

typedef short Short2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ Short2 as_short2(uint32_t v) { return __builtin_bit_cast(Short2, v); }
__device__ __forceinline__ uint32_t as_uint(Short2 v) { return __builtin_bit_cast(uint32_t, v); }

// the columns and rows x0 .. x1, y0 .. y1 of a patch as 8 + 8 bits
__device__ __forceinline__ uint32_t patch_bits(uint32_t x0, uint32_t x1, uint32_t y0, uint32_t y1) {
  return ((2u << x1) - (1u << x0)) | ((2u << y1) - (1u << y0)) << 8;
}

// Up to 64 entries of a patch, in order by lane (bits 0: none): lane t gets the
// mask of those that cover the patch's tile t.
__device__ __forceinline__ uint2 tile_masks(uint32_t bits) {
  const int lane = (int)__lane_id();
  uint32_t lo = 0, hi = 0;
#pragma unroll
  for (int q = 0; q < 16; q++) put_lane(lo, hi, __ballot((bits >> q) & 1u), q);
  const int x = lane & 7, y = 8 + (lane >> 3);
  return make_uint2(__shfl(lo, x, 64) & __shfl(lo, y, 64), __shfl(hi, x, 64) & __shfl(hi, y, 64));
}
__device__ __forceinline__ uint32_t popc(uint2 m) { return (uint32_t)(__popc(m.x) + __popc(m.y)); }

// Writes e of the lanes in a tile's mask to out[at ...].
__device__ __forceinline__ void write_tile(uint64_t m, uint32_t e, uint32_t at, uint32_t* __restrict__ out) {
  const uint32_t to = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, at));
  if (__builtin_amdgcn_inverse_ballot_w64(m))
    *reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(out) + (uint64_t)(uint32_t)(4 * to)) = e;
}

// The same for two rows of tiles, with the writes: lane t's n, t < 16, moves on by
// the entries of the t-th of these tiles, and entry e of the lane goes to
// out[n ...] of those it covers.  False if the output were exceeded (never for
// consistent counts).
__device__ __forceinline__ bool write_rows(uint32_t bits, uint32_t e, int row0, uint32_t& n, uint32_t pcap,
                                           uint32_t* __restrict__ out) {
  const int lane = (int)__lane_id();
  uint64_t col[8];
  uint32_t lo = 0, hi = 0;
#pragma unroll
  for (int x = 0; x < 8; x++) {
    col[x] = __ballot((bits >> x) & 1u);
    put_lane(lo, hi, col[x], x);
  }
  const uint32_t rbits = bits >> (8 + row0);
#pragma unroll
  for (int r = 0; r < 2; r++) put_lane(lo, hi, __ballot((rbits >> r) & 1u), 8 + r);
  const int x = lane & 7, y = 8 + ((lane >> 3) & 1);
  const uint32_t cnt = popc(make_uint2(__shfl(lo, x, 64) & __shfl(lo, y, 64), __shfl(hi, x, 64) & __shfl(hi, y, 64)));
  if (__ballot((uint64_t)n + cnt > pcap)) return false;
#pragma unroll 1
  for (int r = 0; r < 2; r++) {
    const uint64_t row = (uint64_t)readlane(hi, 8 + r) << 32 | readlane(lo, 8 + r);
    if (row == 0) continue;
#pragma unroll
    for (int c = 0; c < 8; c++) write_tile(col[c] & row, e, readlane(n, 8 * r + c), out);
  }
  n += cnt;
  return true;
}

// the view of a patch (every lane calls)
__device__ __forceinline__ int patch_view(const ViewTable& vt, uint32_t patch) {
  const int l = (int)__lane_id();
  return __popcll(__ballot(l < vt.nview && (uint32_t)vt.v[min(l, kMaxViews - 1)].patch_base <= patch)) - 1;
}

// the global id of tile l of patch (px, py) of a view, or -1 past the view's edge
__device__ __forceinline__ int patch_tile(const ViewDesc& vd, int px, int py, int l) {
  const int x = px * 8 + (l & 7), y = py * 8 + (l >> 3);
  return x < vd.ntx && y < vd.nty ? vd.tile_base + y * vd.ntx + x : -1;
}
__device__ __forceinline__ int patch_tile(const ViewTable& vt, uint32_t patch, int l) {
  const ViewDesc& vd = vt.v[patch_view(vt, patch)];
  const int npx = (vd.ntx + 7) >> 3, local = (int)patch - vd.patch_base, py = local / npx;
  return patch_tile(vd, local - py * npx, py, l);
}

// Lists from the items sorted by patch, kListItems per wavefront.  Every (chunk,
// patch) that occurs has table row chunk + patch: both only grow along the
// items, so no two share one and a patch's are adjacent.  The first kernel also
// writes each patch's range of the items (into `ranges`, where k_list_scan
// reads it before the tiles' ranges go there).
constexpr int kListSteps = 4;
constexpr uint32_t kListItems = 64 * kListSteps;
constexpr int kListWG = 8192;  // workgroups at most: each takes further chunks

// Which unit of work a workgroup takes: consecutive ones run on different XCDs,
// so each XCD takes a run of the units (neighbours, which complete each other's
// cache lines).  Loops while the id is below 8 * ceil(units / 8); may return
// an id past the last.
__device__ __forceinline__ uint32_t xcd_unit(uint32_t b, uint32_t units) { return (b & 7u) * ((units + 7u) / 8u) + (b >> 3); }

// The patch_bits of an item's key.
__device__ __forceinline__ uint32_t item_bits(uint32_t key) {
  const uint32_t r = key >> 20;
  return patch_bits(r & 7, (r >> 3) & 7, (r >> 6) & 7, r >> 9);
}

__global__ void __launch_bounds__(kBlock) k_item_counts(const uint32_t* __restrict__ key,
                                                        const uint32_t* __restrict__ counters, uint32_t pcap,
                                                        uint32_t* __restrict__ table, uint2* __restrict__ ranges) {
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (overflowed(counters, pcap)) return;
  const uint32_t S = counters[7];
  const uint32_t nchunk = (S + kListItems - 1) / kListItems;
  for (uint32_t c = blockIdx.x * kWaves + wv; c < nchunk; c += gridDim.x * kWaves) {
    const uint32_t i0 = c * kListItems, i1 = min(i0 + kListItems, S);
    uint32_t n = 0, patch = i0 > 0 ? key[i0 - 1] & kPatchMask : ~0u;  // goes on from the chunk before
    bool first = true;
    uint32_t k = i0 + lane < i1 ? key[i0 + lane] : ~0u;
    for (uint32_t i = i0; i < i1; i += 64) {
      const uint32_t in = i + 64 + lane;
      const uint32_t kn = in < i1 ? key[in] : ~0u;
      const uint32_t id = k & kPatchMask;
      uint64_t todo = __ballot(i + lane < i1);
      while (todo) {
        const int f = __ffsll((unsigned long long)todo) - 1;
        const uint32_t p = readlane(id, f);
        if (first || p != patch) {
          if (!first) table[(uint64_t)(c + patch) * 64 + lane] = n;
          if (p != patch && lane == 0) {  // patch ends and p starts here
            if (patch != ~0u) ranges[patch].y = i + f;
            ranges[p].x = i + f;
          }
          n = 0;
          patch = p;
          first = false;
        }
        todo &= ~__ballot(id == p);
        n += popc(tile_masks(id == p ? item_bits(k) : 0u));
      }
      k = kn;
    }
    table[(uint64_t)(c + patch) * 64 + lane] = n;
    if (i1 == S && lane == 0) ranges[patch].y = S;
  }
}

// A tile's entries of the whole chunk are written one step after the other: step
// by step over the 64 tiles, the half-written cache lines of all wavefronts did
// not fit the L2 caches (144M pairs, 4.5M lines: 11.4M line write-backs and
// 342 us, now 4.9M and 283 us; chunks of 512 items 310 us).
__global__ void __launch_bounds__(kBlock) k_item_lists(ViewTable vt, const uint32_t* __restrict__ key,
                                                       const uint32_t* __restrict__ val,
                                                       const uint32_t* __restrict__ counters, uint32_t pcap,
                                                       const uint32_t* __restrict__ table,
                                                       const uint2* __restrict__ ranges, uint32_t* __restrict__ out,
                                                       uint32_t* __restrict__ order_state,
                                                       uint32_t* __restrict__ order) {
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // the first workgroups order the tiles
  const uint32_t first_wg = order_wgs((uint32_t)vt.total_tiles);
  if (blockIdx.x < first_wg) {
    order_tiles(ranges, (uint32_t)vt.total_tiles, blockIdx.x, order_state, order);
    return;
  }
  if (overflowed(counters, pcap)) return;
  const uint32_t S = counters[7];
  const uint32_t nchunk = (S + kListItems - 1) / kListItems;
  const uint32_t units = (nchunk + kWaves - 1) / kWaves;
  for (uint32_t b = blockIdx.x - first_wg; b < (units + 7) / 8 * 8; b += gridDim.x - first_wg) {
    const uint32_t u = xcd_unit(b, units);
    const uint32_t c = u * kWaves + wv;
    if (u >= units || c >= nchunk) continue;
    const uint32_t i0 = c * kListItems + lane;
    uint32_t k[kListSteps], e[kListSteps];
#pragma unroll
    for (int s = 0; s < kListSteps; s++) {
      const bool in = i0 + 64 * s < S;
      k[s] = in ? key[i0 + 64 * s] : ~0u;
      e[s] = in ? val[i0 + 64 * s] : 0u;
    }
    const uint32_t plast = key[min(c * kListItems + kListItems, S) - 1] & kPatchMask;
    for (uint32_t p = readlane(k[0], 0) & kPatchMask;;) {
      const int tile = patch_tile(vt, p, lane);
      uint32_t n = table[(uint64_t)(c + p) * 64 + lane] + (tile >= 0 ? ranges[tile].x : 0u);
      uint2 m[kListSteps];
      uint32_t cnt = 0;
#pragma unroll
      for (int s = 0; s < kListSteps; s++) {
        const bool mine = (k[s] & kPatchMask) == p;
        m[s] = make_uint2(0u, 0u);
        if (__ballot(mine)) m[s] = tile_masks(mine ? item_bits(k[s]) : 0u);
        cnt += popc(m[s]);
      }
      if (__ballot((uint64_t)n + cnt > pcap)) return;  // never for consistent counts; guards the buffer
#pragma unroll
      for (int s = 0; s < kListSteps; s++) arrived(e[s]);
      arrived(n);
      for (uint64_t todo = __ballot(cnt > 0); todo; todo &= todo - 1) {
        const int t = __ffsll((unsigned long long)todo) - 1;
        uint32_t at = readlane(n, t);
#pragma unroll
        for (int s = 0; s < kListSteps; s++) {
          const uint64_t mt = (uint64_t)readlane(m[s].y, t) << 32 | readlane(m[s].x, t);
          write_tile(mt, e[s], at, out);
          at += (uint32_t)__popcll(mt);
        }
      }
      if (p == plast) break;
      // the next patch among the chunk's items
      uint32_t next = ~0u;
#pragma unroll
      for (int s = kListSteps - 1; s >= 0; s--) {
        const uint64_t after = __ballot((k[s] & kPatchMask) > p && i0 + 64 * s < S);
        if (after) next = readlane(k[s], __ffsll((unsigned long long)after) - 1) & kPatchMask;
      }
      if (next == ~0u) break;
      p = next;
    }
  }
}

// Lists straight from the depth-sorted entries: a workgroup tests a chunk of
// them (STEPS x 64 per wavefront) against one patch and collects those that
// touch it in LDS.  To count, each wavefront takes every fourth 64 of them; to
// write, each takes all of them for two of the patch's rows of tiles (the
// writes of one tile follow each other, and a wavefront's walk over a full
// chunk is a quarter as long).  Row patch * chunks + chunk of the table.
template <bool WRITE, int STEPS>
__global__ void __launch_bounds__(kBlock) k_entry_lists(ViewTable vt, const uint32_t* __restrict__ rect0,
                                                        const uint32_t* __restrict__ rect1,
                                                        const uint32_t* __restrict__ dval,
                                                        uint32_t* __restrict__ counters, uint32_t pcap,
                                                        uint32_t* __restrict__ table,
                                                        const uint2* __restrict__ ranges, uint32_t* __restrict__ out,
                                                        uint32_t* __restrict__ order_state,
                                                        uint32_t* __restrict__ order) {
  constexpr uint32_t kEntries = kBlock * STEPS;
  __shared__ uint32_t s_bits[kEntries], s_e[WRITE ? kEntries : 1], s_n[kWaves][64];
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  uint32_t u = blockIdx.x;
  if (WRITE) {  // the first workgroups order the tiles
    const uint32_t wgs = order_wgs((uint32_t)vt.total_tiles);
    if (u < wgs) {
      order_tiles(ranges, (uint32_t)vt.total_tiles, u, order_state, order);
      return;
    }
    u -= wgs;
  }
  if (overflowed(counters, pcap)) {
    if (!WRITE && blockIdx.x == 0 && threadIdx.x == 0) counters[2] = 1u;
    return;
  }
  const uint32_t nb = counters[0];
  const uint32_t nchunk = (nb + kEntries - 1) / kEntries;
  const uint32_t units = nchunk * (uint32_t)vt.total_patches;
  if (u >= units) return;
  const uint32_t patch = u / nchunk, c = u - patch * nchunk;
  const uint32_t view = (uint32_t)patch_view(vt, patch);
  const ViewDesc& vd = vt.v[view];
  const int npx = (vd.ntx + 7) >> 3, local = (int)patch - vd.patch_base, py = local / npx, px = local - py * npx;
  uint32_t* row = table + ((uint64_t)patch * nchunk + c) * 64;
  const Short2 patch_first = {(short)(8 * px), (short)(8 * py + 2048 * (int)view)};
  const Short2 patch_last = {(short)(8 * px + 7), (short)(8 * py + 7 + 2048 * (int)view)};
  const uint32_t i0 = c * kEntries + wv * (64 * STEPS) + lane;
  uint32_t a[STEPS], b[STEPS], e[STEPS];
#pragma unroll
  for (int s = 0; s < STEPS; s++) {
    const uint32_t i = i0 + 64 * s;
    a[s] = i < nb ? rect0[i] : 0x7FFF7FFFu;  // (starts behind every patch)
    b[s] = i < nb ? rect1[i] : 0u;
    e[s] = WRITE && i < nb ? dval[i] : 0u;
  }
  uint32_t n = 0;
  if (WRITE) {
    const int t = 16 * wv + (lane & 15);  // lanes 0 .. 15: the wavefront's two rows of tiles
    const int tile = patch_tile(vd, px, py, t);
    n = row[t] + (tile >= 0 ? ranges[tile].x : 0u);
  }
  uint64_t m[STEPS];
  uint32_t mine = 0;
#pragma unroll
  for (int s = 0; s < STEPS; s++) {
    // to the rectangle's first tile from the patch's last, and to the patch's
    // first from its last; the entry touches the patch if no half is negative
    const Short2 d0 = patch_last - as_short2(a[s]), d1 = as_short2(b[s]) - patch_first;
    const bool hit = ((as_uint(d0) | as_uint(d1)) & 0x80008000u) == 0;
    const uint32_t f = as_uint(__builtin_elementwise_min(d0, Short2{7, 7}));
    const uint32_t l = as_uint(__builtin_elementwise_min(d1, Short2{7, 7}));
    const uint32_t xb = (2u << (l & 7u)) - (128u >> (f & 7u)), yb = (2u << ((l >> 16) & 7u)) - (128u >> ((f >> 16) & 7u));
    a[s] = hit ? xb | yb << 8 : 0u;
    m[s] = __ballot(hit);
    mine += (uint32_t)__popcll(m[s]);
  }
  if (lane == 0) s_n[wv][0] = mine;
  __syncthreads();
  uint32_t nh = 0, at = 0;
#pragma unroll
  for (int w = 0; w < kWaves; w++) {
    at += w < wv ? s_n[w][0] : 0u;
    nh += s_n[w][0];
  }
#pragma unroll
  for (int s = 0; s < STEPS; s++) {
    if (a[s]) {
      const uint32_t k = __builtin_amdgcn_mbcnt_hi((uint32_t)(m[s] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m[s], at));
      s_bits[k] = a[s];
      if (WRITE) s_e[k] = e[s];
    }
    at += (uint32_t)__popcll(m[s]);
  }
  __syncthreads();
  if constexpr (WRITE) {
    arrived(n);
    for (uint32_t k = 0; k < nh; k += 64) {
      const bool in = k + lane < nh;
      if (!write_rows(in ? s_bits[k + lane] : 0u, in ? s_e[k + lane] : 0u, 2 * wv, n, pcap, out)) return;
    }
  } else {
    for (uint32_t k = 64 * wv; k < nh; k += kBlock)
      n += popc(tile_masks(k + lane < nh ? s_bits[k + lane] : 0u));
    s_n[wv][lane] = n;
    __syncthreads();
    if (wv == 0) row[lane] = s_n[0][lane] + s_n[1][lane] + s_n[2][lane] + s_n[3][lane];
  }
}

// One workgroup per patch: the rows of its chunks become exclusive prefixes,
// and their sums the tiles' pair counts.  chunk: that of k_entry_lists, or 0
// for k_item_lists.  Also counts the tiles' buckets of the order.  Workgroups past the patches zero the screen-space gradient
// accumulators of the binned entries (when g2d is given) for the backward that
// may follow.
constexpr int kScanThreads = 1024;
__global__ void __launch_bounds__(kScanThreads) k_list_scan(ViewTable vt, const uint2* __restrict__ ranges,
                                                            const uint32_t* __restrict__ counters, uint32_t pcap,
                                                            uint32_t chunk, uint32_t* __restrict__ table,
                                                            uint32_t* __restrict__ tile_count,
                                                            uint32_t* __restrict__ order_state,
                                                            const uint32_t* __restrict__ tiles, int64_t E,
                                                            float* __restrict__ g2d) {
  constexpr int kW = kScanThreads / 64;
  __shared__ uint32_t s_n[kW][64];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const uint32_t patch = blockIdx.x;
  if (patch >= (uint32_t)vt.total_patches) {
    zero_g2d_entry((int64_t)(patch - vt.total_patches) * kScanThreads + threadIdx.x, tiles, E, g2d);
    return;
  }
  uint32_t c0 = 0, c1 = 0;  // the patch's rows
  uint64_t row0 = patch;    // of chunk 0
  if (!overflowed(counters, pcap)) {
    if (chunk) {
      c1 = (counters[0] + chunk - 1) / chunk;
      row0 = (uint64_t)patch * c1;
    } else {
      const uint2 r = ranges[patch];  // (UINT_MAX, 0) for a patch without items
      if (r.x < r.y) {
        c0 = r.x / kListItems;
        c1 = (r.y - 1) / kListItems + 1;
      }
    }
  }
  const uint32_t per = (c1 - c0 + kW - 1) / kW;
  const uint32_t b = min(c0 + wv * per, c1), e = min(b + per, c1);
  uint32_t* row = table + row0 * 64 + lane;
  uint32_t sum = 0;
#pragma unroll 8
  for (uint32_t c = b; c < e; c++) sum += row[(uint64_t)c * 64];
  s_n[wv][lane] = sum;
  __syncthreads();
  uint32_t pre = 0, total = 0;
#pragma unroll
  for (int w = 0; w < kW; w++) {
    const uint32_t v = s_n[w][lane];
    pre += w < wv ? v : 0u;
    total += v;
  }
#pragma unroll 8
  for (uint32_t c = b; c < e; c++) {
    const uint32_t v = row[(uint64_t)c * 64];
    row[(uint64_t)c * 64] = pre;
    pre += v;
  }
  if (wv == 0) {
    const int tile = patch_tile(vt, patch, lane);
    if (tile >= 0) tile_count[tile] = total;
    uint32_t n = 0;
    bucket_add(n, tile >= 0 ? order_bucket(total) : -1);
    if (n) atomicAdd(&order_state[patch % kOrderCopies * 64 + lane], n);
  }
}

__global__ void __launch_bounds__(kBlock) k_zero_g2d(const uint32_t* __restrict__ tiles, int64_t E,
                                                     float* __restrict__ g2d) {
  zero_g2d_entry((int64_t)blockIdx.x * kBlock + threadIdx.x, tiles, E, g2d);
}

__global__ void __launch_bounds__(kBlock) k_import(const float* __restrict__ u, const float* __restrict__ v,
                                                   const float* __restrict__ ex, const float* __restrict__ ey,
                                                   const float* __restrict__ depth,
                                                   const int32_t* __restrict__ alive, ViewTable vt,
                                                   Rec* __restrict__ rec, uint32_t* __restrict__ tiles) {
  const int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  const int64_t E = vt.n * vt.nview;
  if (e >= E) return;
  uint32_t count = 0;
  if (alive[e]) {
    const ViewDesc& vd = vt.v[e / vt.n];
    int x0, y0, x1, y1;
    tile_rect(u[e], v[e], ex[e], ey[e], vt.tile_shift_x, vt.tile_shift_y, vd.ntx, vd.nty, x0, y0, x1, y1);
    count = (uint32_t)((x1 - x0) * (y1 - y0));
    Rec r;
    r.a = make_float4(u[e], v[e], 0.f, 0.f);
    r.b = make_float4(0.f, 0.f, ex[e], ey[e]);
    r.c = make_float4(0.f, 0.f, 0.f, depth[e]);
    rec[e] = r;
  }
  tiles[e] = count;
}

}  // namespace

namespace {
RadixState depth_state(const SortBuffers& b) {
  // short sorts take small workgroups (more of them in flight); long ones the pairs' size
  return radix_state(b.rstate_depth, b.E, b.E >= kLargeSort ? kRItems : kRItemsSmall, true);
}
}  // namespace

// Whether a workgroup per patch and chunk tests every sorted entry
// (k_entry_lists) or the entries are sorted by patch first (k_item_lists), which
// takes five launches more, but no time per patch.  The stage's time: 300k
// Gaussians in one 800x800 view, 14M tests, 130 us testing and 159 sorting; 500k
// in one 1600x900 view, 50M tests, 220 and 196.
namespace {
inline bool test_entries(int64_t E, int64_t patches) { return E * patches <= (1ll << 25); }
inline bool tests_entries(const SortBuffers& b) { return test_entries(b.E, b.total_patches); }
// Entries per workgroup of the tests: 1,024 collect more of a patch's entries
// at once, 256 make enough workgroups of a small call (1.5M tests: the same;
// 4M: 82 us with 1,024 and 91 with 256).
inline uint32_t entry_chunk(int64_t E, int64_t patches) { return kBlock * (E * patches <= (1ll << 20) ? 1u : 4u); }

// the tile scan's look-back words stand between the tickets and the tables
inline int64_t tile_scan_words(int64_t total_tiles) { return 2 * ((total_tiles + kChunk - 1) / kChunk + 1); }
inline int64_t pair_zero_words(int64_t total_tiles) {
  return ((kGhCopies + 1) * kGhStride + tile_scan_words(total_tiles) + 3) / 4 * 4;
}
RadixState pair_state(const SortBuffers& b, int64_t bound, int items) {
  return radix_state(b.rstate_pairs, bound, items, false,
                     pair_zero_words(b.total_tiles) - (kGhCopies + 1) * kGhStride);
}
}  // namespace

bool sorts_items(const SortBuffers& b) { return !tests_entries(b); }

// One preparation for the whole stage: the depth sort's state, the pair
// sort's histograms, the tile ranges, the tile order's counts and the
// backward work-item count.
BinPrep bin_prep(const SortBuffers& b) {
  const RadixState rs = depth_state(b);
  BinPrep bp{{b.rstate_depth, b.order_state, b.n_items, b.rstate_pairs},
             {rs.words(), (int64_t)kOrderStateWords, 1, pair_zero_words(b.total_tiles)},
             b.ranges,
             b.total_tiles,
             0};
  bp.threads = bp.nranges;
  for (int k = 0; k < 4; k++) bp.threads = std::max(bp.threads, bp.n[k]);
  return bp;
}

void launch_bin_count(SortBuffers& b, const ViewTable& vt, bool prepped, hipStream_t st) {
  const uint32_t E = (uint32_t)b.E;
  const RadixState rs = depth_state(b);
  const RadixPlan plan{4, 8};
  if (!prepped) {
    const ZeroList z{{b.order_state, b.n_items, b.rstate_pairs, nullptr},
                     {(int64_t)kOrderStateWords, 1, pair_zero_words(b.total_tiles), 0}};
    int64_t prep = rs.words() / 4;
    for (int k = 0; k < 3; k++) prep = std::max(prep, z.n[k]);
    prep = std::max(prep, b.total_tiles);
    hipLaunchKernelGGL(k_stage_prep, dim3((unsigned)((prep + kBlock - 1) / kBlock)), dim3(kBlock), 0, st, rs,
                       rs.words(), z, b.ranges, b.total_tiles, (const uint32_t*)b.counters,
                       (const uint32_t*)nullptr, (const uint32_t*)nullptr, 0u, (uint32_t*)nullptr, (int64_t)0, 0u);
  }
  // compaction of the binned entries with their depth keys, and for the passes the keys' digit histograms
  uint64_t* psum = reinterpret_cast<uint64_t*>(rs.tickets + 256);
  const TileCount tc{b.tiles};
  const CompactDepth cd{b.depth, b.dkey[0], b.dval[0]};
  uint32_t* ticket = rs.tickets + kMaxPasses;
  uint32_t* place = nullptr;
  // depth order (stable: equal depths keep entry order)
  if (rank_entries(b.E)) {
    place = reinterpret_cast<uint32_t*>(rs.scan_status + 2 * rs.nscan);
    scan1<true, false>(tc, cd, nullptr, E, E, b.E, ticket, rs.scan_status, &b.counters[0], (uint32_t*)nullptr, psum,
                       HostCount{}, &b.counters[3], st);
    const uint32_t segment = rank_segment(b.E);
    if (E)
      hipLaunchKernelGGL(k_rank, dim3((E + kBlock * 4 - 1) / (kBlock * 4), (E + segment - 1) / segment), dim3(kBlock),
                         0, st, (const uint32_t*)b.dkey[0], (const uint32_t*)b.counters, segment, place);
    b.dsorted = 1;
  } else {
    scan1<true, true>(tc, cd, nullptr, E, E, b.E, ticket, rs.scan_status, &b.counters[0], rs.ghist, psum,
                      HostCount{}, &b.counters[3], st);
    b.dsorted = radix_sort(b.dkey, b.dval, &b.counters[0], b.E, plan, rs, &b.counters[3], st);
  }
  hipLaunchKernelGGL(k_rects, dim3(std::max(1u, (E + kBlock - 1) / kBlock)), dim3(kBlock), 0, st, vt, b.rec,
                     (const uint32_t*)b.dval[place ? 0 : b.dsorted], (const uint32_t*)place, b.dval[1],
                     (const uint64_t*)psum, b.host_pairs, b.counters, b.dkey[0], b.dkey[1]);
  // item offsets in depth order
  if (!tests_entries(b))
    scan1<false, false>(PatchCount{b.dkey[0], b.dkey[1]},
                 StoreOffset{b.poff, b.blk_start, b.nblk_start, (int64_t)kBlock * sort_items(b.pcap)},
                 &b.counters[0], 0u, E, b.E, rs.tickets + kMaxPasses + 1, rs.scan_status + rs.nscan, &b.counters[7],
                 (uint32_t*)nullptr, (uint64_t*)nullptr, b.host_items, &b.counters[3], st);
}

void launch_bin_emit(SortBuffers& b, const ViewTable& vt, int64_t items_hint, bool regrown, hipStream_t st) {
  const bool direct = tests_entries(b);
  const int64_t bound = direct ? 0 : items_hint < b.pcap ? items_hint : b.pcap;
  const int items = sort_items(b.pcap);
  const uint32_t chunk = (uint32_t)(kBlock * items), cap = (uint32_t)b.pcap;
  const RadixState rs = pair_state(b, bound, items);
  uint32_t* count = &b.counters[7];
  if (regrown) {
    // the passes write every table entry they read: only the histograms, the
    // tickets and the tile scan's state start from zero
    const int64_t zero_words = pair_zero_words(b.total_tiles);
    const ZeroList z{{nullptr, nullptr, nullptr, nullptr}, {0, 0, 0, 0}};
    const int64_t prep = std::max<int64_t>(zero_words / 4, direct ? 0 : b.E);
    hipLaunchKernelGGL(k_stage_prep, dim3((unsigned)((prep + kBlock - 1) / kBlock)), dim3(kBlock), 0, st, rs,
                       zero_words, z, (uint2*)nullptr, (int64_t)0, (const uint32_t*)b.counters, (const uint32_t*)count,
                       (const uint32_t*)b.poff, cap, direct ? nullptr : b.blk_start, rs.nblk, chunk);
  }
  const uint32_t* const rect0 = b.dkey[0];
  const uint32_t* const rect1 = b.dkey[1];
  const uint32_t* const dval = b.dval[b.dsorted];
  uint32_t* const table = rs.status;
  const uint32_t T = (uint32_t)b.total_tiles;
  // the scan of the tiles' counts, which stand in the tile order's place
  auto ranges_of = [&](uint32_t list_chunk) {
    const unsigned gz = b.g2d ? (unsigned)((b.E + kScanThreads - 1) / kScanThreads) : 0u;
    hipLaunchKernelGGL(k_list_scan, dim3((unsigned)b.total_patches + gz), dim3(kScanThreads), 0, st, vt,
                       (const uint2*)b.ranges, (const uint32_t*)b.counters, cap, list_chunk, table, b.tile_order,
                       b.order_state, (const uint32_t*)b.tiles, b.E, b.g2d);
    scan1<false, false>(CountVal{b.tile_order}, StoreRange{b.ranges, cap}, nullptr, T, T, T, rs.tickets,
                 reinterpret_cast<uint64_t*>(rs.tickets + kGhStride), (uint32_t*)nullptr, (uint32_t*)nullptr,
                 (uint64_t*)nullptr, HostCount{}, &b.counters[3], st);
  };
  const unsigned ow = order_wgs(T);
  int cur = 0;
  if (direct) {
    const uint32_t lc = entry_chunk(b.E, b.total_patches);
    const int64_t units = (b.E + lc - 1) / lc * b.total_patches;
    if (units)
      hipLaunchKernelGGL((lc == kBlock ? k_entry_lists<false, 1> : k_entry_lists<false, 4>), dim3((unsigned)units),
                         dim3(kBlock), 0, st, vt, rect0, rect1, dval, b.counters, cap, table, (const uint2*)b.ranges,
                         b.pval[0], b.order_state, b.tile_order);
    ranges_of(lc);
    if (units + ow)
      hipLaunchKernelGGL((lc == kBlock ? k_entry_lists<true, 1> : k_entry_lists<true, 4>), dim3((unsigned)units + ow),
                         dim3(kBlock), 0, st, vt, rect0, rect1, dval, b.counters, cap, table, (const uint2*)b.ranges,
                         b.pval[0], b.order_state, b.tile_order);
  } else {
    // the items, with every pass's digit histogram and the first pass's per-chunk
    // counts; then the passes, each a scan of the chunk counts and a scatter
    // (the chunk counts of later passes taken from their input)
    int bits = 1;
    while ((1ll << bits) < b.total_patches) bits++;
    const RadixPlan plan = radix_plan(bits);
    const uint32_t bound32 = (uint32_t)bound;
    const int64_t nb = rs.nblk;
    if (nb) {
      hipLaunchKernelGGL(k_emit, dim3((unsigned)nb), dim3(kBlock), 0, st, vt, rect0, rect1, dval, b.poff, b.blk_start,
                         b.counters, cap, plan.npass, plan.dbits, rs.ghist, b.pkey[0], b.pval[0], rs.status, chunk);
      for (int p = 0; p < plan.npass; p++) {
        uint32_t* tp = rs.status + (int64_t)p * nb * 256;
        const int shift = p * plan.dbits;
        if (p > 0)
          hipLaunchKernelGGL(items == kRItems ? k_digit_count<kRItems> : k_digit_count<kRItemsSmall>,
                             dim3((unsigned)nb), dim3(kBlock), 0, st, b.pkey[cur], count, bound32, shift, plan.dbits,
                             tp, nb);
        hipLaunchKernelGGL(k_digit_scan, dim3(1u << plan.dbits), dim3(kBlock), 0, st, tp, nb, count, bound32,
                           (int)chunk, (const uint32_t*)(rs.ghist + p * 256));
        hipLaunchKernelGGL(items == kRItems ? k_digit_scatter<kRItems> : k_digit_scatter<kRItemsSmall>,
                           dim3((unsigned)nb), dim3(kBlock), 0, st, b.pkey[cur], b.pval[cur], b.pkey[cur ^ 1],
                           b.pval[cur ^ 1], count, bound32, shift, plan.dbits, (const uint32_t*)tp, nb);
        cur ^= 1;
      }
    }
    const int64_t units = (bound + kListItems * kWaves - 1) / (kListItems * kWaves);
    const unsigned grid = (unsigned)std::min<int64_t>((units + 7) / 8 * 8, kListWG);
    const uint32_t* const k = b.pkey[cur];
    const uint32_t* const v = b.pval[cur];
    if (units)
      hipLaunchKernelGGL(k_item_counts, dim3(grid), dim3(kBlock), 0, st, k, (const uint32_t*)b.counters, cap, table,
                         b.ranges);
    ranges_of(0);
    if (grid + ow)
      hipLaunchKernelGGL(k_item_lists, dim3(grid + ow), dim3(kBlock), 0, st, vt, k, v, (const uint32_t*)b.counters, cap,
                         (const uint32_t*)table, (const uint2*)b.ranges, b.pval[cur ^ 1], b.order_state, b.tile_order);
    cur ^= 1;
  }
  b.psorted = cur;
}

int64_t chunk_scan_words(int64_t n) { return 2 + 2 * ((n + kChunk - 1) / kChunk + 1); }

namespace {
struct CountOffset {
  uint32_t* off;
  __device__ void operator()(int64_t i, uint32_t pre, uint32_t) const { off[i] = pre; }
};
__global__ void __launch_bounds__(kBlock) k_zero_words(uint32_t* __restrict__ p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i < n) p[i] = 0u;
}
}  // namespace

void launch_count_scan(const uint32_t* cnt, int64_t n, uint32_t* off, uint32_t* total, HostCount host, uint32_t* state,
                       uint32_t* err, hipStream_t st) {
  const int64_t words = chunk_scan_words(n);
  hipLaunchKernelGGL(k_zero_words, dim3((unsigned)((words + kBlock - 1) / kBlock)), dim3(kBlock), 0, st, state, words);
  const uint32_t N = (uint32_t)n;
  scan1<false, false>(CountVal{cnt}, CountOffset{off}, nullptr, N, N, n, state, reinterpret_cast<uint64_t*>(state + 2), total,
               (uint32_t*)nullptr, (uint64_t*)nullptr, host, err, st);
}

int64_t sort_state_words(int64_t bound, bool pairs) {
  // the pair state sized for the smaller blocks, whichever sort_items picks
  return radix_state(nullptr, bound, kRItemsSmall, !pairs).words();
}
// The table's rows take the place of the passes' tables: those of sorted items
// (besides one a patch) are half as many words, those of tested entries may be
// more (then there are no passes).
int64_t list_state_words(int64_t E, int64_t total_tiles, int64_t total_patches, int64_t pcap) {
  const int64_t tables = (int64_t)kMaxPasses * 256 * radix_blocks(pcap, kRItemsSmall);
  const int64_t rows = test_entries(E, total_patches)
                           ? total_patches * ((E + entry_chunk(E, total_patches) - 1) / entry_chunk(E, total_patches))
                           : 0;
  return tile_scan_words(total_tiles) + 4 + 64 * (total_patches + 2) + std::max<int64_t>(64 * rows - tables, 0);
}
int64_t sort_block_starts(int64_t pcap) { return radix_blocks(pcap, kRItemsSmall) + 1; }
int64_t order_state_words() { return kOrderStateWords; }

void launch_zero_g2d(const SortBuffers& b, float* g2d, hipStream_t st) {
  const unsigned g = (unsigned)((b.E + kBlock - 1) / kBlock);
  if (g) hipLaunchKernelGGL(k_zero_g2d, dim3(g), dim3(kBlock), 0, st, (const uint32_t*)b.tiles, b.E, g2d);
}

void launch_import_records(const float* u, const float* v, const float* ex, const float* ey, const float* depth,
                           const int32_t* alive, const ViewTable& vt, Rec* rec, uint32_t* tiles, hipStream_t st) {
  const int64_t E = vt.n * vt.nview;
  const unsigned g = (unsigned)((E + kBlock - 1) / kBlock);
  if (g) hipLaunchKernelGGL(k_import, dim3(g), dim3(kBlock), 0, st, u, v, ex, ey, depth, alive, vt, rec, tiles);
}

}  // namespace sixdgs
