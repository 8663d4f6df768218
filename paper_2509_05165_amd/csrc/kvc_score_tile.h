// Matrix-core kernels of kvc_score for every shape the query-stationary kernels do not
// take: bf16 and float32, any head size, any window.  Included by kvc_score.hip only.
//
// The roles are the reverse of the query-stationary kernels: a workgroup (4 waves) keeps
// TILE_KEYS keys of one KV head in registers and streams the head's query rows
// through LDS, 64 rows at a time, one tile ahead.  All query rows of a key then pass
// through one wave, so the window and the group need not divide anything: the statistics
// of a row over the keys of a wave, and the aggregate over the rows of a key, never leave
// the wave (four waves' statistics of a row meet in LDS).  K is read from memory once per
// pass, whatever the number of query rows; the query rows of a head are small and come
// out of the cache.
//
// Both types use the same operand layout, 16-byte pieces: of a row's pieces, lane l of a
// 32x32 operand holds piece 2 ks + l / 32 of row l % 32 in step ks.  For bf16 that is
// the operand of one v_mfma_f32_32x32x16_bf16; for float32 the four elements of the piece
// feed four v_mfma_f32_32x32x2_f32 (any order of the products is as good as another, as
// long as both operands agree).  float32 products and sums stay float32 throughout.
//
// LDS tile: row r at slot r * SP (SP slots of 16 bytes, a power of two, so that a direct global->LDS
// load brings whole rows), its piece p at slot p ^ f(r) of the row, so that the reads of 16 consecutive
// rows cover all banks.  Rows that don't fill their k-steps (head sizes of 72, 192, ...) end in copies of their
// last piece, which meet zeros of the keys; slots past the k-steps (80, 96, ...) are never read.  Clearing the tiles
// instead cost every workgroup up to 64 KB of LDS writes and a barrier: score stage in us, cleared / now, 28 layers of
// 16/8 heads, M = 14, heads of 192 5662 tokens 236.9 / 209.0, of 104 10662 tokens 222.1 / 209.1, float32 heads of 48
// 3000 tokens 120.5 / 114.7.
#pragma once

namespace kvc {
namespace {

constexpr int TL_THREADS = 256;
constexpr int TL_ROWS = 64;          // query rows per LDS tile

struct TileArgs {
  int batch, group, window, total, pieces;
  int hkv, row_split;                // STATS: the row tiles of a head are dealt to row_split workgroups
  int head_rows;                     // EMIT: window rounded up to 8 (rows of a head in tile order)
  uint32_t head_magic;               // EMIT: ceil(2^32 / head_rows)
  int causal, group_max;
  int linear;                        // rows in tile order follow one another in memory
  float c2;
  size_t rows_all, rows_layer;       // query rows of the launch, of a layer: batch * Hq * window
  size_t out_layer_stride;
};

// 16-byte slots of a row in LDS: a power of two, so that a load instruction brings whole rows.
constexpr int tile_slots(int ksteps) { return ksteps <= 4 ? 8 : ksteps <= 8 ? 16 : 2 * ksteps; }

// Per kernel: waves per SIMD, 32-key blocks per wave, tiles of query rows in LDS, k-steps by which the
// fragments run ahead of their products.  Score stage in us, 200 task tokens x 8192 tokens x 32 layers of
// 32 heads of 128 / 14k tokens in heads of 64: the emit pass with 3 and 4 waves and two key blocks
// takes 373 / 65, with 2 and 3 waves 424 / 72, with three key blocks and 2 waves 402, with four 435.  A third
// tile lets the emit pass read across the tile border; the statistics pass gains nothing from it (461 / 92
// with two and with three).  Heads of 80 have no room for it beside four waves: 263 us against 273 (3 waves,
// three tiles) and 277 before at M = 200, 16 layers of 2 x 4096 tokens.
//
// The fragments run ahead only as far as the registers of these waves reach without spills.  A
// float32 step is eight products of 64 cycles, so two steps are plenty; for bf16 heads of 128 two (and for
// the mean of heads of 64), of 80 one.  With four steps (five at heads of 80) the max pooling forms of heads of 128 and float32 heads of 32 and 64 spilled
// 4 to 6 registers, and mean pooling had a wave less.  Score stage in us, 16 layers of 32/8 heads, 2 x 1365..4096 tokens (float32
// 2 x 341..1024), further ahead / now: mean of heads of 128 M = 8 77.8 / 71.5, M = 50 of 28 layers of 28/4 heads 192 / 177,
// of 80 146 / 141; of float32 64 M = 100 329 / 322; max of heads of 128 M = 8 73.9 / 70.9.
constexpr int tile_waves(int ks) { return ks > 16 ? 1 : ks > 8 ? 2 : ks > 5 ? 3 : 4; }
constexpr int tile_least(int ks) { return ks <= 4 ? 1 : ks <= 5 ? 9 : ks <= 6 ? 11 : ks <= 8 ? 9 : ks + 1; }   // pieces of a row
constexpr int tile_kb(int ks) { return ks > 16 ? 1 : 2; }
constexpr int tile_ring(int ks, bool emit) { return emit && ks <= 8 && ks != 5 ? 3 : 2; }
constexpr int tile_ahead(int ks, bool emit, bool mean, bool f32) {
  if (emit && (f32 || ks == 8 || (ks == 4 && mean))) return 2;
  return emit && ks == 5 ? 1 : ks % 4 == 0 ? 4 : ks;      // (divides ks)
}

// As lds_dma16_s, 4 bytes per lane.
__device__ __forceinline__ void lds_dma4_s(const void* sbase, uint32_t voff, uint32_t lds_base) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" ::"s"(lds_base), "v"(voff), "s"(sbase)
               : "memory");
}

__device__ __forceinline__ uint4 load16(const __attribute__((address_space(1))) char* base, uint32_t off) {
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  const u32x4 v = *reinterpret_cast<const __attribute__((address_space(1))) u32x4*>(base + off);
  return make_uint4(v.x, v.y, v.z, v.w);
}

// One k-step (16 bytes of every row of both operands) of a 32x32 tile.
template <typename T>
__device__ __forceinline__ f32x16 tile_mma(uint4 rows, uint4 cols, f32x16 acc) {
  if constexpr (sizeof(T) == 2) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(rows), as_bf16x8(cols), acc, 0, 0, 0);
  } else {
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(rows.x), __uint_as_float(cols.x), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(rows.y), __uint_as_float(cols.y), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(rows.z), __uint_as_float(cols.z), acc, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(rows.w), __uint_as_float(cols.w), acc, 0, 0, 0);
  }
}

// KS: k-steps (pairs of 16-byte pieces) a row is padded to; KB: 32-key blocks per wave.
// grid: ((sequence, chunk) pairs, Hkv * row_split, layers)
//
// STATS: keys on the rows of the matrix tile, so a lane owns one query row: maximum and
// sum of 2^(t - max) over the wave's keys, then over the workgroup's, to part_m / part_s.
// EMIT: queries on the rows, a lane owns one key.  In tile order every query head is
// padded to a multiple of 8 rows, so each group of four accumulator registers (8 rows) belongs to
// one head; the padding rows are copies of the last one (the mean leaves them out).
//
// What bounds it is the vector port and the issue of one wave (fragment reads, products, the vector work
// on their result, one after the other), so a wave issues little else: the tile loads start from scalar
// addresses and keep their lane offsets, the log-sum-exps of a tile come the same way, masks stay
// out of the common path, the buffers of the ring are constants, and the statistics of four tiles
// are joined by all threads at once.  With an address computed per lane and load the address code
// was half of what a wave issued in the emit pass.  Score stage, 200 task tokens, 32 heads of 128 and 8192
// tokens x 32 layers, statistics + emit in us: 493 + 449 then, 461 + 373 now (0.98 PFLOP/s over both);
// heads of 64 in a ragged batch of 14k tokens 97 + 77, 92 + 65.  Measured and left: the keys of the next
// chunk prefetched into registers while a workgroup walks over chunks (543 + 436), fixed wave priorities (537 +
// 436), two accumulator sets and one wave less (5 % slower at heads of 64).
template <typename T, int KS, bool EMIT, bool TASK_MAX>
__global__ __launch_bounds__(TL_THREADS, tile_waves(KS)) void score_tile(
    PtrTable q_tab, PtrTable k_tab, SeqTable seq, TileArgs a, float* __restrict__ part_m,
    float* __restrict__ part_s, const float* __restrict__ lse2, float* __restrict__ out) {
  constexpr int SP = tile_slots(KS);            // 16-byte slots per row in LDS
  constexpr int RPD = 64 / SP;                  // rows that one load instruction brings
  constexpr int DMA = TL_ROWS / RPD / 4;        // load instructions per wave and tile
  constexpr int KB = tile_kb(KS), KEYS = 4 * 32 * KB;
  constexpr int RING = tile_ring(KS, EMIT);
  constexpr int AHEAD = tile_ahead(KS, EMIT, !TASK_MAX, sizeof(T) == 4);
  // EMIT, float32: the log-sum-exps carry what rounding took from them, too
  constexpr bool REST = EMIT && sizeof(T) == 4;
  __shared__ __attribute__((aligned(1024))) uint4 qtile[RING][TL_ROWS * SP];
  constexpr int GROUP = KS == 5 ? 2 : 4;        // STATS: tiles whose statistics are joined at a time
  __shared__ float2 stat[EMIT ? 1 : 2 * GROUP][4][EMIT ? 1 : TL_ROWS];
  // EMIT: the log-sum-exps of a tile's rows
  __shared__ __attribute__((aligned(256))) float lses[EMIT ? RING : 1][EMIT ? TL_ROWS : 4];
  __shared__ __attribute__((aligned(256))) float rests[REST ? RING : 1][REST ? TL_ROWS : 4];

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int col = lane & 31, half = lane >> 5;
  const int P = a.pieces;
  const int R = EMIT ? a.group * a.head_rows : a.group * a.window;
  const int all_tiles = (R + TL_ROWS - 1) / TL_ROWS;

  const int layer = blockIdx.z;
  const int h = blockIdx.y / a.row_split, split = blockIdx.y - h * a.row_split;
  int b = 0, chunk = blockIdx.x;
  for (; b < a.batch - 1; ++b) {
    const int nc = (seq.cu[b + 1] - seq.cu[b] + KEYS - 1) / KEYS;
    if (chunk < nc) break;
    chunk -= nc;
  }
  const int tok0 = seq.cu[b], n = seq.cu[b + 1] - tok0;
  if (chunk * KEYS >= n) return;
  const int t_begin = EMIT ? 0 : (int)((uint32_t)all_tiles * (uint32_t)split / (uint32_t)a.row_split);
  const int t_end = EMIT ? all_tiles : (int)((uint32_t)all_tiles * (uint32_t)(split + 1) / (uint32_t)a.row_split);
  if (t_begin >= t_end) return;
  // first query row of the (sequence, KV head) in its layer, among the rows of the launch
  const size_t head_row = ((size_t)b * a.hkv + h) * (uint32_t)(a.group * a.window);
  const size_t qrow0 = (size_t)layer * a.rows_layer + head_row;
  const uint4* q_head = static_cast<const uint4*>(q_tab.p[layer]) + head_row * P;

  // ---- query tiles to LDS ----
  // Load j of a tile (j = 4 i + wave) brings the RPD rows from j RPD on, in tile order; they lie in one
  // group of 8, hence in one query head, and follow one another in memory.  The row they start from is
  // scalar, and a lane's offset from it is the same for every tile unless the head ends before the
  // group does (then its last row is read again).
  const int rr = lane / SP, slot = lane % SP;
  const uint32_t qtile_lds = (uint32_t)(size_t)(__attribute__((address_space(3))) uint4*)(&qtile[0][0]);
  const uint32_t lses_lds = (uint32_t)(size_t)(__attribute__((address_space(3))) float*)(&lses[0][0]);
  const uint32_t rests_lds = (uint32_t)(size_t)(__attribute__((address_space(3))) float*)(&rests[0][0]);
  auto lane_slot = [&](int i) {         // what the k-steps read in the lane's slot: piece of a padded row
    const int swz = KS == 4 ? (wave * 4 + (rr >> 1)) & 7 : ((i * 4 * RPD) & 15) ^ ((wave * RPD + rr) & 15);
    return slot ^ swz;
  };
  auto lane_piece = [&](int i) { return min(lane_slot(i), P - 1); };    // (past the row its last one: they meet zeros)
  const uint32_t qoff = (uint32_t)((wave * RPD + rr) * P + lane_piece(0)) * 16u;
  // query row (among the head's group * window) behind row `pr` in tile order, and how many of its head follow
  auto source_row = [&](uint32_t pr, int& behind) -> int {
    if (!EMIT) {
      const int row = min((int)pr, R - 1);
      behind = R - 1 - row;
      return row;
    }
    uint32_t g = __umulhi(pr, a.head_magic);           // exact or one too large
    if (g * (uint32_t)a.head_rows > pr) --g;
    int m = (int)(pr - g * (uint32_t)a.head_rows);
    if ((int)g >= a.group) { g = (uint32_t)a.group - 1; m = 0; }
    m = min(m, a.window - 1);
    behind = a.window - 1 - m;
    return (int)g * a.window + m;
  };
  auto scalar64 = [](uint64_t x) {
    return ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(x >> 32)) << 32) |
           (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)x);
  };
  int ahead_t = t_begin, ahead_buf = 0;   // the next tile to be asked for, and its buffer
  auto issue_tile = [&]() {
    const int t = ahead_t;
    if (EMIT && wave == (t & 3)) {      // a row per lane
      int behind;
      const uint32_t off = (uint32_t)source_row((uint32_t)(t * TL_ROWS + lane), behind) * 4u;
      lds_dma4_s(reinterpret_cast<const void*>(scalar64(reinterpret_cast<uint64_t>(lse2 + qrow0))), off,
                 __builtin_amdgcn_readfirstlane(lses_lds + ahead_buf * (TL_ROWS * 4)));
      if (REST)
        lds_dma4_s(reinterpret_cast<const void*>(scalar64(reinterpret_cast<uint64_t>(lse2 + a.rows_all + qrow0))), off,
                   __builtin_amdgcn_readfirstlane(rests_lds + ahead_buf * (TL_ROWS * 4)));
    }
    const uint32_t dst = qtile_lds + (uint32_t)ahead_buf * (TL_ROWS * SP * 16) + wave * 1024;
    const uint64_t tile = reinterpret_cast<uint64_t>(q_head) + (uint64_t)(uint32_t)t * (uint32_t)(TL_ROWS * 16 * P);
    if (a.linear && (t + 1) * TL_ROWS <= R) {
#pragma unroll
      for (int i = 0; i < DMA; ++i) {
        const uint64_t base = scalar64(tile + (uint32_t)(i * 4 * RPD * 16) * (uint32_t)P);
        const uint32_t off = RPD >= 4 ? qoff : (uint32_t)((wave * RPD + rr) * P + lane_piece(i)) * 16u;
        if (SP == 2 * KS || lane_slot(i) < 2 * KS)
          lds_dma16_s<false>(reinterpret_cast<const void*>(base), off, __builtin_amdgcn_readfirstlane(dst + i * 4096));
      }
    } else {
      // (opaque: the products of the offsets are not worth registers across the tile loop)
      int rrow = rr;
      asm volatile("" : "+v"(rrow));
#pragma unroll
      for (int i = 0; i < DMA; ++i) {
        const uint32_t pr = (uint32_t)__builtin_amdgcn_readfirstlane(t * TL_ROWS + (4 * i + wave) * RPD);
        int behind;
        const int row = source_row(pr, behind);
        const uint64_t base = scalar64(reinterpret_cast<uint64_t>(q_head) + (uint64_t)(uint32_t)row * (uint32_t)(P * 16));
        const uint32_t off = (uint32_t)(min(rrow, behind) * P + lane_piece(i)) * 16u;
        if (SP == 2 * KS || lane_slot(i) < 2 * KS)
          lds_dma16_s<false>(reinterpret_cast<const void*>(base), off, __builtin_amdgcn_readfirstlane(dst + i * 4096));
      }
    }
    ahead_buf = ahead_buf + 1 == RING ? 0 : ahead_buf + 1;
    ++ahead_t;
  };

  for (int i = 0; i < RING - 1; ++i)
    if (ahead_t < t_end) issue_tile();
  // ---- keys: registers for the whole kernel ----
  uint4 kf[KB][KS];
  {
    // scalar address of the wave's first key (or of the last one there is), keys behind it
    const int row = min(chunk * KEYS + wave * 32 * KB, n - 1), behind = n - 1 - row;
    // (rebuilt as a global-memory pointer: through the integers the compiler would lose that)
    typedef const __attribute__((address_space(1))) char* global_ptr;
    const global_ptr base = (global_ptr)scalar64(reinterpret_cast<uint64_t>(k_tab.p[layer]) +
        (((uint64_t)(uint32_t)h * (uint32_t)a.total + (uint32_t)(tok0 + row)) * (uint32_t)(P * 16)));
    // (a row piece by piece: with the two rows of a lane in turn the parts of a 128-byte line are asked for too
    // far apart, 75 -> 94 us for 66k tokens in heads of 104)
    auto load_keys = [&](auto full) {
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) {
        const uint32_t off = (uint32_t)(min(kb * 32 + col, behind) * P) * 16u + half * 16u;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          kf[kb][ks] = make_uint4(0, 0, 0, 0);
          if (decltype(full)::value || 2 * ks + 1 < tile_least(KS) || 2 * ks + half < P)
            kf[kb][ks] = load16(base, off + ks * 32);
        }
      }
    };
    // Rows that don't fill their k-steps: pieces past the row are zero (times a copy of the last piece, which the
    // queries have there, a key of minus infinity would make the logit NaN).  Full rows have a path without the
    // branches between the loads, which cost them up to 11 % (heads of 64, M = 6, 32 layers of 16788 tokens); where
    // only the last piece may be past the row one masked load is the faster form (heads of 80, M = 14, 28 layers of
    // 16/8 heads, 10662 tokens, 157.8 us against 170.5 with two paths).
    if ((KS != 5 && KS != 6) && P == 2 * KS) load_keys(std::true_type{});
    else load_keys(std::false_type{});
  }
  const int subs = a.head_rows >> 3;                              // EMIT: groups of 8 rows per query head
  const float inv_window = 1.f / float(a.window);
  // STATS: up to GROUP tiles wait in LDS for the four waves' statistics of a row to be joined, a row per
  // thread; their rows start at st_row of part_m / part_s
  size_t st_row = 0;
  int st_tiles = 0, st_rows = 0, st_group = 0;
  auto store_stats = [&]() {
    if ((int)threadIdx.x < st_rows) {
      float2 x[4];
#pragma unroll
      for (int w = 0; w < 4; ++w) x[w] = stat[st_group * GROUP + wave][w][lane];
      const float mm = fmaxf(fmaxf(x[0].x, x[1].x), fmaxf(x[2].x, x[3].x));
      float ss = 0.f;
#pragma unroll
      for (int w = 0; w < 4; ++w) ss += x[w].y * fast_exp2(x[w].x - mm);
      part_m[st_row + threadIdx.x] = mm;
      part_s[st_row + threadIdx.x] = ss;
    }
    st_tiles = st_rows = 0;
    st_group ^= 1;
  };

  // fragments of block `blk` of the tile in buffer `buf`
  const int swz = KS == 4 ? (col >> 1) & 7 : col & 15;
  const int fbase = col * SP * 16 + ((half ^ swz) << 4);
  auto frag = [&](int buf, int blk, int ks) {
    int at = fbase;
    // (opaque where registers are short: no address per k-step is kept)
    if (REST || (EMIT && KS == 5)) asm volatile("" : "+v"(at));
    const unsigned char* p = reinterpret_cast<const unsigned char*>(&qtile[buf][blk * 32 * SP]);
    return *reinterpret_cast<const uint4*>(p + (at ^ (32 * ks)));
  };
  uint4 qf[AHEAD];
  const int wkey0 = chunk * KEYS + wave * 32 * KB;           // first key of the wave
  const bool active = wkey0 < n;                              // wave-uniform, like the next two
  const bool ragged = wkey0 + 32 * KB > n;
  const bool masked = a.causal && wkey0 + 32 * KB - 1 > n - a.window;
  int sub = 0, heads = a.group;       // EMIT: groups of 8 rows done of the current head; heads left
  float tacc[KB], gacc[KB];           // EMIT: current head's aggregate, group's
#pragma unroll
  for (int kb = 0; kb < KB; ++kb) { tacc[kb] = TASK_MAX ? NEG_BIG : 0.f; gacc[kb] = 0.f; }
  auto finish_head = [&]() {
    // (rows behind the last head are copies of rows before them)
    if (heads > 0) {
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) {
        const float tv = cross_half<TASK_MAX>(tacc[kb]);
        const float sv = TASK_MAX ? fast_exp2(tv) : tv * inv_window;
        gacc[kb] = a.group_max ? fmaxf(gacc[kb], sv) : gacc[kb] + sv;
        tacc[kb] = TASK_MAX ? NEG_BIG : 0.f;
      }
      --heads;
    }
    sub = 0;
  };
  auto tile = [&](const int t, auto buffer) __attribute__((always_inline)) {
    const int buf = buffer;
    // this tile (RING 3: and the next, which the fragments run into) is complete, and every wave is done
    // with the tile before, whose buffer the next load takes
    wait_loads();
    wait_lds();
    __syncthreads();
    if (!EMIT && st_tiles == GROUP) store_stats();
    if (ahead_t < t_end) issue_tile();
    const int next_buf = buf + 1 == RING ? 0 : buf + 1;
    if (!active) {                      // a wave without keys only keeps the others company
      if (!EMIT) {
        stat[st_group * GROUP + st_tiles][wave][lane] = make_float2(NEG_BIG, 0.f);
        if (st_tiles++ == 0) st_row = (size_t)chunk * a.rows_all + qrow0 + t * TL_ROWS;
        st_rows += min(R - t * TL_ROWS, TL_ROWS);
      }
      return;
    }
    if (RING == 2 || t == t_begin) {
#pragma unroll
      for (int ks = 0; ks < AHEAD; ++ks) qf[ks] = frag(buf, 0, ks);
    }
#pragma unroll
    for (int blk = 0; blk < 2; ++blk) {
      f32x16 acc[KB];
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[kb][r] = 0.f;
      float4 nl[4];                     // EMIT: lse2 of the lane's rows
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
          acc[kb] = EMIT ? tile_mma<T>(qf[ks % AHEAD], kf[kb][ks], acc[kb])
                         : tile_mma<T>(kf[kb][ks], qf[ks % AHEAD], acc[kb]);
        // (behind the last tile they are read and not used)
        if (ks + AHEAD < KS) qf[ks % AHEAD] = frag(buf, blk, ks + AHEAD);
        else if (blk == 0) qf[ks % AHEAD] = frag(buf, 1, ks + AHEAD - KS);
        else if (RING > 2) qf[ks % AHEAD] = frag(next_buf, 0, ks + AHEAD - KS);
        if (EMIT && ks == KS / 2) {
#pragma unroll
          for (int i = 0; i < 4; ++i)
            nl[i] = *reinterpret_cast<const float4*>(&lses[buf][blk * 32 + 8 * i + 4 * half]);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (!EMIT) {
        if (ragged) {                     // keys past the sequence drop out
          int mine = wkey0 + 4 * half;    // (opaque, or 32 key positions are formed outside the branch)
          asm volatile("" : "+v"(mine));
#pragma unroll
          for (int kb = 0; kb < KB; ++kb)
#pragma unroll
            for (int r = 0; r < 16; ++r)
              if (mine + kb * 32 + acc_row(r, 0) >= n) acc[kb][r] = -__builtin_inff();
        }
        if (masked) {                     // task token m sees keys up to n - window + m
          const int seen = n - a.window + (t * TL_ROWS + blk * 32 + col) % a.window;
          int mine = wkey0 + 4 * half;
          asm volatile("" : "+v"(mine));
#pragma unroll
          for (int kb = 0; kb < KB; ++kb)
#pragma unroll
            for (int r = 0; r < 16; ++r)
              if (mine + kb * 32 + acc_row(r, 0) > seen) acc[kb][r] = -__builtin_inff();
        }
        float amax = acc[0][0];
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
          for (int r = 0; r < 16; ++r) amax = fmaxf(amax, acc[kb][r]);
        // (no key seen: the maximum stays finite and every 2^(-inf) below is 0)
        const float mx = fmaxf(cross_half<true>(amax) * a.c2, NEG_BIG);
        float s = 0.f;
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
          for (int r = 0; r < 16; ++r) s += fast_exp2(fmaf(acc[kb][r], a.c2, -mx));
        s = cross_half<false>(s);
        if (half == 0) stat[st_group * GROUP + st_tiles][wave][blk * 32 + col] = make_float2(mx, s);
      } else {
        // registers 4 i .. 4 i + 3 hold rows 8 i + 4 half .. + 3 of the block
        if (masked) {                     // on its own, so that the common case has no mask to look at
          int m8 = sub;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int seen = n - a.window + 8 * m8 + 4 * half;     // last key that the first of the four sees
#pragma unroll
            for (int kb = 0; kb < KB; ++kb)
#pragma unroll
              for (int r = 0; r < 4; ++r)
                // (a row behind the window is a copy of its last one, which sees every key)
                if (wkey0 + kb * 32 + col > min(seen + r, n - 1)) acc[kb][4 * i + r] = -__builtin_inff();
            if (++m8 == subs) m8 = 0;
          }
        }
        // whole: all rows lie in the window (or don't matter, being copies: the maximum), and the mean looks at
        // none of them.  Mean pooling, score stage in us, each row looked at / not: 16 layers of 32/8 heads, 2 x 1365..4096
        // tokens, heads of 128 M = 200 357 / 341, of 80 M = 100 163 / 157; float32 heads of 32, 2 x 341..1024, M = 100 125.8 / 123.4.
        auto fold = [&](int i, auto whole) {
          float4 rest = make_float4(0.f, 0.f, 0.f, 0.f);
          if (REST) rest = *reinterpret_cast<const float4*>(&rests[buf][blk * 32 + 8 * i + 4 * half]);
          const int rows = decltype(whole)::value ? 4 : a.window - 8 * sub - 4 * half;
#pragma unroll
          for (int kb = 0; kb < KB; ++kb) {
            float x0 = fmaf(acc[kb][4 * i], a.c2, -nl[i].x), x1 = fmaf(acc[kb][4 * i + 1], a.c2, -nl[i].y);
            float x2 = fmaf(acc[kb][4 * i + 2], a.c2, -nl[i].z), x3 = fmaf(acc[kb][4 * i + 3], a.c2, -nl[i].w);
            if (REST) { x0 -= rest.x; x1 -= rest.y; x2 -= rest.z; x3 -= rest.w; }
            if (TASK_MAX) {
              tacc[kb] = fmaxf(fmaxf(tacc[kb], x0), x1);
              tacc[kb] = fmaxf(fmaxf(tacc[kb], x2), x3);
            } else {
              tacc[kb] += ((rows > 0 ? fast_exp2(x0) : 0.f) + (rows > 1 ? fast_exp2(x1) : 0.f)) +
                          ((rows > 2 ? fast_exp2(x2) : 0.f) + (rows > 3 ? fast_exp2(x3) : 0.f));
            }
          }
          ++sub;
        };
        if (TASK_MAX ? sub + 4 <= subs : 8 * sub + 32 <= a.window) {   // the block ends within the query head
#pragma unroll
          for (int i = 0; i < 4; ++i) fold(i, std::true_type{});
          if (sub == subs) finish_head();
        } else {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            fold(i, std::integral_constant<bool, TASK_MAX>{});
            if (sub == subs) finish_head();
          }
        }
      }
    }
    if (!EMIT) {
      if (st_tiles++ == 0) st_row = (size_t)chunk * a.rows_all + qrow0 + t * TL_ROWS;
      st_rows += min(R - t * TL_ROWS, TL_ROWS);
    }
  };
  if constexpr (KS <= 8) {            // the buffers of the ring are constants of the addresses
    for (int t = t_begin; t < t_end; t += RING) {
      tile(t, std::integral_constant<int, 0>{});
      if (t + 1 < t_end) tile(t + 1, std::integral_constant<int, 1>{});
      if (RING == 3 && t + 2 < t_end) tile(t + 2, std::integral_constant<int, RING - 1>{});
    }
  } else {
    int buf = 0;
    for (int t = t_begin; t < t_end; ++t) {
      tile(t, buf);
      buf = buf + 1 == RING ? 0 : buf + 1;
    }
  }
  if constexpr (EMIT) {
    float* out_head = out + (size_t)layer * a.out_layer_stride + (size_t)h * a.total + tok0;
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
      const int key = wkey0 + kb * 32 + col;
      if (half == 0 && key < n) out_head[key] = gacc[kb];
    }
  }
  if constexpr (!EMIT) {
    wait_memory();
    __syncthreads();
    store_stats();
  }
}

// k-steps a row of `pieces` 16-byte pieces is padded to: head sizes 64, 80, 96, 128 and 256 in
// bf16 and 32, 64, 128 and 256 in float32 need no padding.
inline int tile_ksteps(int dtype, int pieces) {
  const int ks = (pieces + 1) / 2;
  if (dtype == KVC_BF16) return ks <= 4 ? 4 : ks <= 5 ? 5 : ks <= 6 ? 6 : ks <= 8 ? 8 : 16;
  return ks <= 4 ? 4 : ks <= 8 ? 8 : ks <= 16 ? 16 : 32;
}
// keys per workgroup of the statistics pass
constexpr int tile_keys(int ksteps) { return 128 * tile_kb(ksteps); }

}  // namespace
}  // namespace kvc
