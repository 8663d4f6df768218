// kvc_global_select: the budget-th largest composite score of each sequence's
// pool {I[l,k]} and the per-layer lengths N_l it induces (Section 3.3: global
// pool, B_total, N_l).
//
// Radix select on the order-preserving integer image of the fp32 scores, three
// digits of 11/11/10 bits from the top: each pass histograms the candidates
// that match the prefix found so far, a one-workgroup step picks the digit
// that holds the wanted rank.  A last sweep counts, per layer, the entries
// above the threshold and those equal to it; ties are granted in ascending
// layer order until the budget is met (within a layer the tied entries are the
// ranks right after the ones above the threshold, so each layer keeps a prefix).
//
// The digit search after a histogram pass and the final bookkeeping run in the
// last workgroup of the sequence to finish (each workgroup takes a ticket once its
// atomic updates are complete; the one that draws the last ticket reads the totals
// with device-scope atomic loads), so a call is five launches instead of eleven.
//
// Inside kvc_compress the rows of the pool are known to be sorted (the composite of sorted
// scores is sorted, in floating point too), the scratch is clear (the rank kernel does that on the
// way where the workspace has room for it beside its own) and the scores are still to be aggregated
// over the heads: launch_composite_select then needs three launches.  The first pass aggregates, stores and histograms, and the last workgroup of the
// third pass finds the counts of a row by searching it instead of sweeping all rows.  Composite
// and selection of 32 layers x 777 tokens: 34 -> 30 us; at 131072 tokens the pass as a
// whole is within the noise of the separate launches.
//
// A "layer" here is a row of the pool: a layer, or a (layer, head) pair in the
// unstructured variant.  With a per-row floor f the first f ranks of every row
// are kept unconditionally and stay out of the histograms; the budget that is
// searched for is what remains after them.
#include <algorithm>
#include <mutex>

#include "kvc_internal.h"

namespace kvc {

namespace {

// Scratch of kvc_global_select_static: the histograms, counters, tickets and
// per-sequence state that kvc_global_select takes from the caller's workspace.
// One copy per GPU, held until the process ends.  In host code the array's name
// is only a stand-in for the symbol; its device address is looked up once per
// device (static_scratch) and that pointer is what kernels receive.
static __device__ __align__(256) unsigned char scratch[KVC_SELECT_STATIC_BYTES];

constexpr int SEL_BINS = 2048;
constexpr int SEL_THREADS = 256;
constexpr int SEL_PER_BLOCK = SEL_THREADS * 8;   // fewest elements of a row per workgroup

struct SelState {
  uint32_t prefix;       // bits of the threshold key fixed so far
  uint32_t bad;          // set when a histogram did not add up (see find_digit)
  uint64_t remaining;    // rank still to descend inside the prefix bucket (1-based)
  uint64_t expect;       // candidates the next histogram pass must count: the pool, then
                         // the population of the bucket chosen by the pass before
};

struct BudgetTable { int64_t b[KVC_MAX_BATCH]; };

// What the first pass on cleared scratch and the last pass over sorted rows need besides.
struct SelectExtra {
  int rows;
  float* tau;
  int32_t* lengths;
  int64_t* offsets;
  BudgetTable budget;
};

__device__ __forceinline__ void digit_of(int pass, uint32_t key, uint32_t* digit, uint32_t* hi) {
  // pass 0: bits 31..21, pass 1: bits 20..10, pass 2: bits 9..0
  if (pass == 0) { *digit = key >> 21; *hi = 0; }
  else if (pass == 1) { *digit = (key >> 10) & 2047u; *hi = key >> 21; }
  else { *digit = key & 1023u; *hi = key >> 10; }
}

// Scratch and state of a stage call; budget.b[] already excludes the floor entries.
__global__ void select_init(uint32_t* words, int count, SelState* state, BudgetTable budget, SeqTable seq,
                            int rows, int floor_rank) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) words[i] = 0;
  if (i < seq.batch) {
    const int n = seq.cu[i + 1] - seq.cu[i];
    state[i].prefix = 0;
    state[i].bad = 0;
    state[i].remaining = (uint64_t)budget.b[i];
    state[i].expect = (uint64_t)rows * (uint64_t)max(n - floor_rank, 0);   // entries that compete
  }
}

__global__ void select_clear(uint32_t* words, int count) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) words[i] = 0;
}

__device__ __forceinline__ uint32_t load_agent(const uint32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Ticket of a workgroup that has finished its part for sequence b: true for the
// one that drew the last of `expected` tickets.
//
// INVARIANT: inside one kernel, workgroups hand data to the last one through
// device-scope atomic read-modify-writes ONLY (histogram bins, row counts).  Those
// are performed at the device's coherence point and are complete once the issuing
// wave's vector-memory counter has drained; so the release side is that wait, not a
// device-scope release fence (whose write-back of the whole L2 cost 150 us per
// launch here, 2048 workgroups each paying it).  The last workgroup reads the totals
// with device-scope atomic loads.  A plain store would NOT be visible to the last
// workgroup this way: anything else a kernel produces (state[], lengths, offsets) is
// written by the last workgroup itself and read by a later kernel.  This relies on
// returned-less atomics counting in vmcnt and being performed in L2, which holds on
// gfx950; find_digit checks that every histogram adds up to the population it must
// cover, so a violation cannot pass silently (tau becomes NaN).
// Tickets are drawn in two levels (groups of SEL_GROUP workgroups, then the groups
// of a sequence), each counter on a cache line of its own: two thousand
// workgroups drawing from one address took 30 us per launch.
constexpr int SEL_GROUP = 64;
constexpr int SEL_TICKET_WORDS = 32;   // one 128-byte line per counter

// tickets: [4 kernels][batch][groups + 1][SEL_TICKET_WORDS]; slot `groups` is the second level
__device__ __forceinline__ bool last_workgroup(uint32_t* tickets, int kernel_id, int batch, int b) {
  __shared__ uint32_t is_last;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  wait_vmcnt<0>();                             // my atomics have been performed
  __syncthreads();
  if (threadIdx.x == 0) {
    const uint32_t nblocks = gridDim.x * gridDim.y;
    const uint32_t groups = (nblocks + SEL_GROUP - 1) / SEL_GROUP;
    const uint32_t flat = blockIdx.y * gridDim.x + blockIdx.x, g = flat / SEL_GROUP;
    const uint32_t in_group = min((uint32_t)SEL_GROUP, nblocks - g * SEL_GROUP);
    uint32_t* base = tickets + ((size_t)(kernel_id * batch + b) * (groups + 1)) * SEL_TICKET_WORDS;
    uint32_t last = atomicAdd(base + (size_t)g * SEL_TICKET_WORDS, 1u) == in_group - 1;
    if (last) last = atomicAdd(base + (size_t)groups * SEL_TICKET_WORDS, 1u) == groups - 1;
    is_last = last;
  }
  __syncthreads();
  const bool last = is_last != 0;
  if (last) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  return last;
}

// Inclusive prefix sum over the SEL_THREADS threads of a workgroup; *total = sum of all.
__device__ __forceinline__ uint64_t block_scan_incl(uint64_t v, uint64_t* total) {
  __shared__ uint64_t wave_tot[SEL_THREADS / 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint64_t incl = v;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const uint64_t o = __shfl_up(incl, off);
    if (lane >= off) incl += o;
  }
  __syncthreads();                              // the previous call's readers are done
  if (lane == 63) wave_tot[wave] = incl;
  __syncthreads();
  uint64_t add = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < SEL_THREADS / 64; ++w) {
    const uint64_t x = wave_tot[w];
    if (w < wave) add += x;
    tot += x;
  }
  *total = tot;
  return incl + add;
}

// One workgroup: picks the digit whose bucket holds the wanted rank, walking from
// the largest digit down.  Thread t owns bins [bins - (t+1)*per, bins - t*per) in
// descending order; a prefix sum over the threads names the owner of the rank.
// FRESH (pass 0 on state[b] that is all zero): looks for rank `budget` among `pool` entries; otherwise
// goes on from state[b].  *found (LDS): the threshold bits fixed so far.
template <bool FRESH>
__device__ __forceinline__ void find_digit(int pass, int b, const uint32_t* __restrict__ hist,
                                           SelState* state, uint64_t budget, uint64_t pool,
                                           uint32_t* found) {
  const uint64_t want = FRESH ? budget : state[b].remaining;    // uniform
  if (want == 0) return;                       // budget 0: nothing to find
  const uint64_t expect = FRESH ? pool : state[b].expect;       // uniform; read before anyone updates it
  const uint32_t prefix = state[b].prefix;
  const uint32_t* gh = hist + ((size_t)b * 3 + pass) * SEL_BINS;
  const int bins = pass == 2 ? 1024 : SEL_BINS;
  const int per = bins / SEL_THREADS;          // 8 or 4 bins per thread
  const int t = threadIdx.x;
  uint32_t c[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) c[j] = j < per ? load_agent(&gh[bins - 1 - (t * per + j)]) : 0u;
  uint64_t mine = 0;
#pragma unroll
  for (int j = 0; j < 8; ++j) mine += c[j];
  uint64_t total;
  const uint64_t incl = block_scan_incl(mine, &total);
  uint64_t run = incl - mine;
  // every candidate of this pass must have been counted (see last_workgroup)
  if (t == 0 && total != expect) state[b].bad = 1;
  // the thread whose range holds the rank; a rank past the pool ends in the last bin
  if (run < want && (want <= incl || t == SEL_THREADS - 1)) {
    uint32_t digit = 0, population = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      if (j < per) {
        const int bin = bins - 1 - (t * per + j);
        digit = (uint32_t)bin;
        population = c[j];
        if (run + c[j] >= want) break;
        run += c[j];
      }
    }
    const uint32_t shift = pass == 0 ? 21u : (pass == 1 ? 10u : 0u);
    state[b].prefix = prefix | digit << shift;
    state[b].remaining = want - run;           // rank inside the chosen bucket
    state[b].expect = population;              // what the next pass must count
    *found = prefix | digit << shift;
  }
}

// Adds an element's digit to the workgroup's histogram.  Rows are usually sorted, so the 64
// elements of a wave step mostly share one digit: then one lane adds the whole count instead
// of 64 atomics on one address.
__device__ __forceinline__ void hist_add(uint32_t* lh, bool ok, uint32_t digit) {
  const uint64_t all = __ballot(ok);
  if (all == 0) return;                                // wave-uniform
  const int leader = __ffsll((unsigned long long)all) - 1;
  const uint32_t d0 = __builtin_amdgcn_readlane(digit, leader);
  const uint64_t same = __ballot(ok && digit == d0);
  if (same == all) {
    if ((int)(threadIdx.x & 63) == leader) atomicAdd(&lh[d0], (uint32_t)__popcll(all));
  } else if (ok) {
    atomicAdd(&lh[digit], 1u);
  }
}

// Lengths and offsets of sequence b from its per-row counts, by one workgroup.
// The retained total of a sequence is its budget (known on the host), so the first
// offset of every sequence comes from the table.  Ties at the threshold go to the
// rows in ascending order until the budget is met: row l takes
// min(eq_l, max(0, ties - sum of eq over the rows before it)).  count_at(l, i): entries of row l
// above (i = 0) and equal to (i = 1) the threshold, whose key is tau_key.
template <typename COUNT>
__device__ __forceinline__ void finalize_sequence(int b, const SeqTable& seq, int layers,
                                                  int floor_rank, const BudgetTable& budget,
                                                  uint32_t tau_key, const SelState* state,
                                                  const COUNT& count_at, float* tau,
                                                  int32_t* lengths, int64_t* offsets) {
  int64_t off = 0;       // rows retained by the sequences before mine
  for (int p = 0; p < b; ++p) {
    const int n_p = seq.cu[p + 1] - seq.cu[p];
    off += budget.b[p] + (int64_t)layers * (floor_rank < n_p ? floor_rank : n_p);
  }
  const int64_t want = budget.b[b];
  const int n_b = seq.cu[b + 1] - seq.cu[b];
  const int64_t kept_first = floor_rank < n_b ? floor_rank : n_b;   // the floor entries
  const int t = threadIdx.x;
  if (tau && t == 0) {
    // stored through the integer image: the library is compiled under the assumption
    // that no NaN occurs, which a floating-point select of a NaN need not survive
    const uint32_t bits = want > 0 ? __float_as_uint(ordered_to_float(tau_key)) : 0x7f800000u;
    reinterpret_cast<uint32_t*>(tau)[b] = state[b].bad ? 0x7fc00000u : bits;
  }
  uint64_t above_mine = 0;
  if (want > 0)
    for (int l = t; l < layers; l += SEL_THREADS) above_mine += count_at(l, 0);
  uint64_t above;
  block_scan_incl(above_mine, &above);
  const int64_t ties = want - (int64_t)above;
  uint64_t eq_before = 0, len_before = 0;      // carried over the chunks of SEL_THREADS rows
  for (int l0 = 0; l0 < layers; l0 += SEL_THREADS) {
    const int l = l0 + t;
    const bool live = l < layers;
    uint64_t gt = 0, eq = 0;
    if (live && want > 0) {
      gt = count_at(l, 0);
      eq = count_at(l, 1);
    }
    uint64_t eq_chunk, len_chunk;
    const uint64_t eq_excl = eq_before + block_scan_incl(eq, &eq_chunk) - eq;
    int64_t take = ties - (int64_t)eq_excl;
    take = take < 0 ? 0 : (take > (int64_t)eq ? (int64_t)eq : take);
    const uint64_t len = live ? uint64_t(kept_first) + gt + uint64_t(take) : 0;
    const uint64_t len_excl = len_before + block_scan_incl(len, &len_chunk) - len;
    if (live) {
      lengths[b * layers + l] = (int32_t)len;
      offsets[b * layers + l] = off + (int64_t)len_excl;
    }
    eq_before += eq_chunk;
    len_before += len_chunk;
  }
  if (b == seq.batch - 1 && t == 0) offsets[seq.batch * layers] = off + (int64_t)len_before;
}

// Entries [first, n) of a descending row that lie above (x) and at (y) the threshold: both
// borders are searched by the `lanes` (a power of two) adjacent lanes of a group together, each
// step cutting the stretch by lanes + 1.  Every lane of the group gets the result.
__device__ __forceinline__ uint2 count_sorted(const float* row, int first, int n, uint32_t tau_key,
                                              int lanes, bool live) {
  const int lane = threadIdx.x & 63, j = lane & (lanes - 1);
  const uint64_t group = (lanes == 64 ? ~0ull : (1ull << lanes) - 1) << (lane - j);
  int lo[2], hi[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) { lo[s] = live ? first : 0; hi[s] = live ? n : 0; }
  while (__any(lo[0] < hi[0] || lo[1] < hi[1])) {
    int probe[2];
    float x[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      // (inside [lo, hi) for every lane while the stretch is not empty)
      probe[s] = lo[s] + (int)((uint64_t)(uint32_t)(hi[s] - lo[s]) * (j + 1) / (lanes + 1));
      x[s] = lo[s] < hi[s] ? row[probe[s]] : 0.f;
    }
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const uint32_t key = float_to_ordered(x[s]);
      const bool before = lo[s] < hi[s] && (s == 0 ? key > tau_key : key >= tau_key);
      const int c = __popcll(__ballot(before) & group);    // probes before the border
      const int below = __shfl(probe[s], (lane - j) + max(c - 1, 0));
      const int above = __shfl(probe[s], (lane - j) + min(c, lanes - 1));
      if (lo[s] < hi[s]) {
        if (c < lanes) hi[s] = above;
        if (c > 0) lo[s] = below + 1;
      }
    }
  }
  return make_uint2(lo[0] - first, lo[1] - lo[0]);
}

// grid: (token blocks, rows, batch).  SORTED (last pass, at most SEL_THREADS rows): every row is
// descending, and the last workgroup of a sequence finds its counts, lengths and offsets.
// FRESH: pass 0 on cleared state.
template <bool SORTED, bool FRESH>
__device__ __forceinline__ void select_hist_body(
    const float* __restrict__ I, const SeqTable& seq, int total, int pass, int floor_rank, int per_block,
    SelState* state, uint32_t* __restrict__ hist /* [batch][3][SEL_BINS] */, uint32_t* __restrict__ tickets,
    const SelectExtra* extra) {
  __shared__ __attribute__((aligned(8))) uint32_t lh[SEL_BINS];
  __shared__ uint32_t found;
  const int b = blockIdx.z;
  const int tok0 = seq.cu[b], n = seq.cu[b + 1] - tok0;
  const int begin = max((int)blockIdx.x * per_block, floor_rank);   // ranks below the floor do not compete
  const bool active = begin < n && begin < (int)(blockIdx.x + 1) * per_block;   // uniform in the workgroup
  if (active) {
    const int end = min(n, (int)(blockIdx.x + 1) * per_block);
    for (int i = threadIdx.x; i < SEL_BINS; i += SEL_THREADS) lh[i] = 0;
    __syncthreads();
    const uint32_t want_hi = pass == 0 ? 0u : (pass == 1 ? state[b].prefix >> 21 : state[b].prefix >> 10);
    const float* row = I + (size_t)blockIdx.y * total + tok0;
    for (int i0 = begin; i0 < end; i0 += SEL_THREADS * 4) {   // four loads in flight per thread
      float x[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int i = i0 + e * SEL_THREADS + (int)threadIdx.x;
        x[e] = row[i < end ? i : end - 1];              // clamped; dropped below
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int i = i0 + e * SEL_THREADS + (int)threadIdx.x;
        uint32_t digit, hi;
        digit_of(pass, float_to_ordered(x[e]), &digit, &hi);
        hist_add(lh, i < end && hi == want_hi, digit);
      }
    }
    __syncthreads();
    uint32_t* gh = hist + ((size_t)b * 3 + pass) * SEL_BINS;
    for (int i = threadIdx.x; i < SEL_BINS; i += SEL_THREADS)
      if (lh[i]) atomicAdd(&gh[i], lh[i]);
  }
  // every workgroup of the sequence takes a ticket, the idle ones included
  if (!last_workgroup(tickets, pass, seq.batch, b)) return;
  if constexpr (FRESH)
    find_digit<true>(pass, b, hist, state, (uint64_t)extra->budget.b[b],
                     (uint64_t)extra->rows * (uint64_t)max(n - floor_rank, 0), &found);
  else
    find_digit<false>(pass, b, hist, state, 0, 0, &found);
  if constexpr (SORTED) {
    const BudgetTable& budget = extra->budget;
    const int rows = extra->rows;
    __syncthreads();                                       // found
    const uint32_t tau_key = budget.b[b] > 0 ? found : 0u;
    uint2* rc = reinterpret_cast<uint2*>(lh);              // counts of a row (the histogram is flushed)
    int lanes = 64;
    while (lanes * rows > SEL_THREADS) lanes /= 2;         // at least 1: rows <= SEL_THREADS
    const int r = (int)threadIdx.x / lanes;
    if (budget.b[b] > 0) {                                 // uniform
      const uint2 c = count_sorted(I + (size_t)min(r, rows - 1) * total + tok0, min(floor_rank, n), n,
                                   tau_key, lanes, r < rows);
      if (r < rows && ((int)threadIdx.x & (lanes - 1)) == 0) rc[r] = c;
    }
    __syncthreads();
    finalize_sequence(b, seq, rows, floor_rank, budget, tau_key, state,
                      [&](int l, int i) -> uint64_t { return i ? rc[l].y : rc[l].x; }, extra->tau, extra->lengths, extra->offsets);
  }
}

// The plain pass keeps its argument block, with the grid's size that the system puts behind it, within
// one cache line: the size is first asked for behind a barrier of every workgroup, and from the
// next line three launches over 64 sequences took 60 us for 55.
__global__ __launch_bounds__(SEL_THREADS) void select_hist(
    const float* __restrict__ I, SeqTable seq, int total, int pass, int floor_rank, int per_block, SelState* state,
    uint32_t* __restrict__ hist, uint32_t* __restrict__ tickets) {
  select_hist_body<false, false>(I, seq, total, pass, floor_rank, per_block, state, hist, tickets, nullptr);
}
template <bool SORTED, bool FRESH>
__global__ __launch_bounds__(SEL_THREADS) void select_hist_with(
    const float* __restrict__ I, SeqTable seq, int total, int pass, int floor_rank, int per_block, SelState* state,
    uint32_t* __restrict__ hist, uint32_t* __restrict__ tickets, SelectExtra extra) {
  select_hist_body<SORTED, FRESH>(I, seq, total, pass, floor_rank, per_block, state, hist, tickets, &extra);
}

// The composite (mean or maximum over the heads of the rank-aligned scores) and the first
// histogram pass over it.  grid: (rank blocks, layers, batch); the heads are joined in ascending
// order as in kvc_composite.  HKV heads known at compile time: VEC consecutive ranks per thread, all
// loads of a thread in flight together.  HKV = 0, any number: CH_RANKS ranks of CH_HEADS heads in
// flight.  One at a time made a chain of the heads: 32 layers of 4096 ranks took 35 us with 12 heads
// and 80 with 32 (the composite and the histogram as two launches 17 and 23); with 4 ranks 16 and
// 26, with 8 12 and 15; 64 heads, 8 layers of 16384, 36 and 20 (two launches 30).
constexpr int CH_RANKS = 8, CH_HEADS = 4;
template <int HKV, int VEC>
__global__ __launch_bounds__(SEL_THREADS) void composite_hist(
    const float* __restrict__ sorted, SeqTable seq, int hkv_arg, int total, int head_max,
    int floor_rank, int per_block, float* __restrict__ I, SelState* state,
    uint32_t* __restrict__ hist, uint32_t* __restrict__ tickets, BudgetTable budget) {
  __shared__ uint32_t lh[SEL_BINS];
  __shared__ uint32_t found;
  const int hkv = HKV ? HKV : hkv_arg;
  const int b = blockIdx.z, l = blockIdx.y;
  const int tok0 = seq.cu[b], n = seq.cu[b + 1] - tok0;
  const int begin = (int)blockIdx.x * per_block;
  if (begin < n) {                                       // uniform in the workgroup
    const int end = min(n, begin + per_block);
    for (int i = threadIdx.x; i < SEL_BINS; i += SEL_THREADS) lh[i] = 0;
    __syncthreads();
    const float* p0 = sorted + (size_t)l * hkv * total + tok0;
    float* out = I + (size_t)l * total + tok0;
    if constexpr (HKV > 0) {
      typedef float vec_t __attribute__((ext_vector_type(VEC)));
      for (int i0 = begin; i0 < end; i0 += SEL_THREADS * VEC) {
        const int i = i0 + (int)threadIdx.x * VEC;
        const bool live = i < end;                       // VEC > 1: n is a multiple of VEC (host-checked)
        const float* p = p0 + (live ? i : begin);
        vec_t x[HKV];
#pragma unroll
        for (int h = 0; h < HKV; ++h) x[h] = __builtin_nontemporal_load(reinterpret_cast<const vec_t*>(p + (size_t)h * total));
        vec_t acc = x[0];
#pragma unroll
        for (int h = 1; h < HKV; ++h) {
          if (head_max) {
#pragma unroll
            for (int j = 0; j < VEC; ++j) acc[j] = fmaxf(acc[j], x[h][j]);
          } else {
            acc += x[h];
          }
        }
        if (!head_max) acc = acc / float(hkv);
        if (live) *reinterpret_cast<vec_t*>(out + i) = acc;
#pragma unroll
        for (int j = 0; j < VEC; ++j) hist_add(lh, live && i + j >= floor_rank, float_to_ordered(acc[j]) >> 21);
      }
    } else {
      for (int i0 = begin; i0 < end; i0 += SEL_THREADS * CH_RANKS) {
        const float* p[CH_RANKS];
        float acc[CH_RANKS];
#pragma unroll
        for (int e = 0; e < CH_RANKS; ++e) {
          p[e] = p0 + min(i0 + e * SEL_THREADS + (int)threadIdx.x, end - 1);   // clamped; dropped below
          acc[e] = *p[e];
        }
        int h = 1;
        for (; h + CH_HEADS <= hkv; h += CH_HEADS) {     // (no branch among the loads, or they go out one by one)
          float x[CH_HEADS][CH_RANKS];
#pragma unroll
          for (int j = 0; j < CH_HEADS; ++j)
#pragma unroll
            for (int e = 0; e < CH_RANKS; ++e) x[j][e] = p[e][(size_t)(h + j) * total];
#pragma unroll
          for (int j = 0; j < CH_HEADS; ++j)
#pragma unroll
            for (int e = 0; e < CH_RANKS; ++e) acc[e] = head_max ? fmaxf(acc[e], x[j][e]) : acc[e] + x[j][e];
        }
        for (; h < hkv; ++h) {
          float x[CH_RANKS];
#pragma unroll
          for (int e = 0; e < CH_RANKS; ++e) x[e] = p[e][(size_t)h * total];
#pragma unroll
          for (int e = 0; e < CH_RANKS; ++e) acc[e] = head_max ? fmaxf(acc[e], x[e]) : acc[e] + x[e];
        }
#pragma unroll
        for (int e = 0; e < CH_RANKS; ++e) {
          const int i = i0 + e * SEL_THREADS + (int)threadIdx.x;
          if (!head_max) acc[e] = acc[e] / float(hkv);
          if (i < end) out[i] = acc[e];
          hist_add(lh, i < end && i >= floor_rank, float_to_ordered(acc[e]) >> 21);
        }
      }
    }
    __syncthreads();
    uint32_t* gh = hist + (size_t)b * 3 * SEL_BINS;
    for (int i = threadIdx.x; i < SEL_BINS; i += SEL_THREADS)
      if (lh[i]) atomicAdd(&gh[i], lh[i]);
  }
  if (last_workgroup(tickets, 0, seq.batch, b))
    find_digit<true>(0, b, hist, state, (uint64_t)budget.b[b],
               (uint64_t)gridDim.y * (uint64_t)max(n - floor_rank, 0), &found);
}

// grid: (token blocks, layers, batch): counts[b][l] = {#(I > tau), #(I == tau)}; the
// last workgroup of a sequence then writes its lengths and offsets.
__global__ __launch_bounds__(SEL_THREADS) void select_count(
    const float* __restrict__ I, SeqTable seq, int total, int layers, int floor_rank, int per_block,
    BudgetTable budget, const SelState* __restrict__ state, uint32_t* __restrict__ counts,
    uint32_t* __restrict__ tickets, float* tau, int32_t* lengths, int64_t* offsets) {
  __shared__ uint32_t sh[2];
  const int b = blockIdx.z;
  const int tok0 = seq.cu[b], n = seq.cu[b + 1] - tok0;
  const int begin = max((int)blockIdx.x * per_block, floor_rank);
  const bool active = begin < n && begin < (int)(blockIdx.x + 1) * per_block;   // uniform in the workgroup
  if (active) {
    const int end = min(n, (int)(blockIdx.x + 1) * per_block);
    if (threadIdx.x < 2) sh[threadIdx.x] = 0;
    __syncthreads();
    const uint32_t tau_key = state[b].prefix;
    const float* row = I + (size_t)blockIdx.y * total + tok0;
    uint32_t gt = 0, eq = 0;
    for (int i = begin + threadIdx.x; i < end; i += SEL_THREADS) {
      const uint32_t key = float_to_ordered(row[i]);
      gt += key > tau_key;
      eq += key == tau_key;
    }
    for (int off = 32; off >= 1; off >>= 1) { gt += __shfl_xor(gt, off); eq += __shfl_xor(eq, off); }
    if ((threadIdx.x & 63) == 0) { atomicAdd(&sh[0], gt); atomicAdd(&sh[1], eq); }
    __syncthreads();
    if (threadIdx.x < 2 && sh[threadIdx.x])
      atomicAdd(&counts[((size_t)b * layers + blockIdx.y) * 2 + threadIdx.x], sh[threadIdx.x]);
  }
  if (last_workgroup(tickets, 3, seq.batch, b))
    finalize_sequence(b, seq, layers, floor_rank, budget, state[b].prefix, state,
                      [&](int l, int i) -> uint64_t { return load_agent(&counts[((size_t)b * layers + l) * 2 + i]); },
                      tau, lengths, offsets);
}

// Batches whose sequences are all empty launch nothing else.  grid: (batch)
__global__ __launch_bounds__(SEL_THREADS) void select_finalize(
    SeqTable seq, int layers, int floor_rank, BudgetTable budget,
    const SelState* __restrict__ state, const uint32_t* __restrict__ counts, float* tau,
    int32_t* lengths, int64_t* offsets) {
  const int b = blockIdx.x;
  finalize_sequence(b, seq, layers, floor_rank, budget, state[b].prefix, state,
                    [&](int l, int i) -> uint64_t { return counts[((size_t)b * layers + l) * 2 + i]; },
                    tau, lengths, offsets);
}

// Elements of a row per workgroup: every workgroup clears and flushes a 2048-bin
// histogram, so big pools (many rows) get longer stretches per workgroup, about
// 4096 workgroups per sequence at most.
inline int select_per_block(const Problem& pb) {
  int per = SEL_PER_BLOCK;
  while (per < (1 << 20) && ((pb.max_seqlen + per - 1) / per) * int64_t(pb.sel_rows) > 4096) per *= 2;
  return per;
}

struct SelectLayout { size_t off_hist, off_counts, off_tickets, off_state, total; int words; };

SelectLayout select_layout(const Problem& pb) {
  SelectLayout L{};
  size_t cur = 0;
  const size_t hist_words = size_t(pb.batch) * 3 * SEL_BINS;
  const size_t count_words = size_t(pb.batch) * pb.sel_rows * 2;
  L.off_hist = cur;   cur += hist_words * 4;
  L.off_counts = cur; cur += align_up(count_words * 4);
  // 3 passes + the count sweep, each with one counter line per group of workgroups + 1
  // (sized for the shortest stretch per workgroup, so that the size never shrinks when
  // max_seqlen grows: callers may size the workspace with an upper bound)
  const size_t sel_blocks = size_t((pb.max_seqlen + SEL_PER_BLOCK - 1) / SEL_PER_BLOCK) * pb.sel_rows;
  const size_t sel_groups = (sel_blocks + SEL_GROUP - 1) / SEL_GROUP;
  L.off_tickets = cur; cur += align_up(4 * size_t(pb.batch) * (sel_groups + 1) * SEL_TICKET_WORDS * 4);
  L.off_state = cur;  cur += align_up(size_t(pb.batch) * sizeof(SelState));
  L.words = int(cur / 4);                     // all of it starts from zero
  L.total = cur;
  return L;
}

}  // namespace

size_t select_workspace_bytes(const Problem& pb) { return select_layout(pb).total; }
int select_clear_words(const Problem& pb) { return select_layout(pb).words; }

// Device address of this GPU's copy of `scratch` (looked up on the first call on
// each device, with that device current).
kvc_status select_static_scratch(void** ptr) {
  constexpr int MAX_DEVICES = 64;
  static std::mutex mu;
  static void* per_device[MAX_DEVICES] = {};
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
  if (dev < 0 || dev >= MAX_DEVICES) {
    set_error("device ordinal %d outside [0, %d)", dev, MAX_DEVICES);
    return KVC_ERR_UNSUPPORTED;
  }
  std::lock_guard<std::mutex> lock(mu);
  if (!per_device[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return hip_fail(e, "hipGetSymbolAddress(scratch)");
    if (!p) { set_error("hipGetSymbolAddress(scratch) returned NULL"); return KVC_ERR_HIP; }
    per_device[dev] = p;
  }
  *ptr = per_device[dev];
  return KVC_OK;
}

// What is left to compete for after the floor entries.
static BudgetTable open_budgets(const Problem& pb, const int64_t* budget) {
  BudgetTable bt{};
  for (int b = 0; b < pb.batch; ++b) {
    const int64_t n_b = pb.seq.cu[b + 1] - pb.seq.cu[b];
    bt.b[b] = budget[b] - int64_t(pb.sel_rows) * (pb.min_per_layer < n_b ? pb.min_per_layer : n_b);
  }
  return bt;
}

// Passes [first_pass, 3) and the counts.  fresh: the scratch is all zero (otherwise select_init has
// set the state, or a first pass has).
static kvc_status select_passes(const Problem& pb, const float* I, const BudgetTable& bt, int first_pass,
                                bool fresh, bool sorted, float* tau, int32_t* lengths, int64_t* offsets, char* w,
                                hipStream_t stream) {
  const SelectLayout L = select_layout(pb);
  uint32_t* hist = reinterpret_cast<uint32_t*>(w + L.off_hist);
  uint32_t* counts = reinterpret_cast<uint32_t*>(w + L.off_counts);
  uint32_t* tickets = reinterpret_cast<uint32_t*>(w + L.off_tickets);
  SelState* state = reinterpret_cast<SelState*>(w + L.off_state);
  const int total = int(pb.total), rows = pb.sel_rows, floor_rank = pb.min_per_layer;
  const int per_block = select_per_block(pb);
  dim3 grid((unsigned)((pb.max_seqlen + per_block - 1) / per_block), rows, pb.batch);
  // more rows than threads (unstructured pools) keep the counting sweep: one workgroup
  // searching them one row per thread and round would take longer than the sweep's launch
  const bool search = sorted && rows <= SEL_THREADS;
  const SelectExtra extra{rows, tau, lengths, offsets, bt};
  for (int pass = first_pass; pass < 3; ++pass) {
    if (pass == 2 && search)
      KVC_LAUNCH("select_hist", stream, select_hist_with<true, false><<<grid, SEL_THREADS, 0, stream>>>(
          I, pb.seq, total, pass, floor_rank, per_block, state, hist, tickets, extra));
    else if (pass == 0 && fresh)
      KVC_LAUNCH("select_hist", stream, select_hist_with<false, true><<<grid, SEL_THREADS, 0, stream>>>(
          I, pb.seq, total, pass, floor_rank, per_block, state, hist, tickets, extra));
    else
      KVC_LAUNCH("select_hist", stream, select_hist<<<grid, SEL_THREADS, 0, stream>>>(
          I, pb.seq, total, pass, floor_rank, per_block, state, hist, tickets));
  }
  if (!search)
    KVC_LAUNCH("select_count", stream, select_count<<<grid, SEL_THREADS, 0, stream>>>(
        I, pb.seq, total, rows, floor_rank, per_block, bt, state, counts, tickets, tau, lengths, offsets));
  return KVC_OK;
}

kvc_status launch_select_clear(const Problem& pb, void* ws, hipStream_t stream) {
  const int words = select_clear_words(pb);
  KVC_LAUNCH("select_clear", stream, select_clear<<<(words + 255) / 256, 256, 0, stream>>>(
      static_cast<uint32_t*>(ws), words));
  return KVC_OK;
}

kvc_status launch_global_select(const Problem& pb, const float* I, const int64_t* budget,
                                float* tau, int32_t* lengths, int64_t* offsets, void* ws,
                                hipStream_t stream) {
  const SelectLayout L = select_layout(pb);
  char* w = static_cast<char*>(ws);
  const BudgetTable bt = open_budgets(pb, budget);
  const int words = int(L.off_state / 4);
  KVC_LAUNCH("select_init", stream, select_init<<<(std::max(words, pb.batch) + 255) / 256, 256, 0, stream>>>(
      reinterpret_cast<uint32_t*>(w), words, reinterpret_cast<SelState*>(w + L.off_state), bt, pb.seq, pb.sel_rows,
      pb.min_per_layer));
  if (pb.max_seqlen > 0) return select_passes(pb, I, bt, 0, false, false, tau, lengths, offsets, w, stream);
  KVC_LAUNCH("select_finalize", stream, select_finalize<<<pb.batch, SEL_THREADS, 0, stream>>>(
      pb.seq, pb.sel_rows, pb.min_per_layer, bt, reinterpret_cast<SelState*>(w + L.off_state),
      reinterpret_cast<uint32_t*>(w + L.off_counts), tau, lengths, offsets));
  return KVC_OK;
}

kvc_status launch_composite_select(const Problem& pb, const float* S_sorted, float* I,
                                   const int64_t* budget, float* tau, int32_t* lengths,
                                   int64_t* offsets, void* ws, hipStream_t stream) {
  const SelectLayout L = select_layout(pb);
  char* w = static_cast<char*>(ws);
  const BudgetTable bt = open_budgets(pb, budget);
  if (pb.unstructured)   // the pool is the rank-aligned per-head scores themselves
    return select_passes(pb, S_sorted, bt, 0, true, true, tau, lengths, offsets, w, stream);
  const int total = int(pb.total), head_max = pb.agg_head == KVC_AGG_MAX;
  const int per_block = select_per_block(pb);
  dim3 grid((unsigned)((pb.max_seqlen + per_block - 1) / per_block), pb.layers, pb.batch);
  // four ranks per thread need 16-byte aligned sequences in every layer
  bool vec4 = (reinterpret_cast<uintptr_t>(S_sorted) | reinterpret_cast<uintptr_t>(I)) % 16 == 0;
  for (int b = 0; b <= pb.batch; ++b) vec4 = vec4 && pb.seq.cu[b] % 4 == 0;
#define KVC_COMPOSITE_HIST(HKV, VEC)                                                              \
  KVC_LAUNCH("composite_hist", stream, composite_hist<HKV, VEC><<<grid, SEL_THREADS, 0, stream>>>( \
      S_sorted, pb.seq, pb.hkv, total, head_max, pb.min_per_layer, per_block, I,                   \
      reinterpret_cast<SelState*>(w + L.off_state), reinterpret_cast<uint32_t*>(w + L.off_hist),   \
      reinterpret_cast<uint32_t*>(w + L.off_tickets), bt))
  if (pb.hkv == 8 && vec4) KVC_COMPOSITE_HIST(8, 4);
  else if (pb.hkv == 8) KVC_COMPOSITE_HIST(8, 1);
  else if (pb.hkv == 4 && vec4) KVC_COMPOSITE_HIST(4, 4);
  else if (pb.hkv == 4) KVC_COMPOSITE_HIST(4, 1);
  else KVC_COMPOSITE_HIST(0, 1);
#undef KVC_COMPOSITE_HIST
  return select_passes(pb, I, bt, 1, false, true, tau, lengths, offsets, w, stream);
}

}  // namespace kvc
