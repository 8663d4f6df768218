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
// LDS tile: row r at slot r * PS (PS = 2 KS + 1 slots of 16 bytes: an odd stride, so that the
// reads of 16 consecutive rows cover all banks).  The direct global->LDS loads write
// consecutive slots; 64 rows of PS slots are exactly PS wave instructions.
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
  float c2;
  size_t rows_all;                   // query rows of the launch: layers * batch * Hq * window
  size_t out_layer_stride;
};

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
// one head; the padding rows carry lse = +1e30 and contribute nothing.
//
// What bounds it is latency inside a wave (fragment reads, products, the vector work on their
// result, one after the other) and the vector port, so registers are held to what four waves per
// SIMD (rows of up to 160 bytes), three (256) or two (512) leave, masks stay out of the common
// path and the tile loads take 32-bit offsets from a scalar base.  The emit pass also waits for
// what it has only just asked for: the compiler cannot see that wait_memory covers the key
// fragments and puts its own vmcnt(0) in front of the first product of every tile, behind the loads
// of the next one, and load_nl negates what it loads at once; the tile loads run ahead in the
// statistics pass only.  200 task tokens, 32 heads of 128 and 8192 tokens x 32 layers, both passes:
// 1126 us with two waves and the mask looked at per element, 1062 with three, 989 without the
// mask, 972 now (0.88 PFLOP/s); heads of 64 in a ragged batch of 14k tokens 206, 202, 187, 186.  A
// form with two accumulator sets and prefetched fragments, one wave less, took 1075 and 262.
template <typename T, int KS, int KB, bool EMIT, bool TASK_MAX>
__global__ __launch_bounds__(TL_THREADS, KS > 16 ? 1 : KS > 8 ? 2 : KS > 5 ? 3 : 4) void score_tile(
    PtrTable q_tab, PtrTable k_tab, SeqTable seq, TileArgs a, float* __restrict__ part_m,
    float* __restrict__ part_s, const float* __restrict__ lse2, float* __restrict__ out) {
  constexpr int PS = 2 * KS + 1;
  constexpr int KEYS = 4 * 32 * KB;
  constexpr int DMA = (PS + 3) / 4;             // load instructions per wave and tile, at most
  __shared__ __attribute__((aligned(16))) uint4 qtile[2][TL_ROWS * PS];
  __shared__ float2 stat[EMIT ? 1 : 2][4][EMIT ? 1 : TL_ROWS];
  // EMIT: minus the log-sum-exps of a tile's rows; float32 keeps what rounding took from them, too
  constexpr bool REST = EMIT && sizeof(T) == 4;
  // An opaque copy of the lane keeps what a tile load's offsets are made of out of the live set:
  // otherwise the emit forms whose registers are used up spill it (2 to 15 registers), and every
  // reload waits for the loads before it between two loads of a tile.  Score stage, 16 layers of
  // 4096 tokens, 32/8 heads, in us without / with: bf16 d = 80 79 / 71, 128 (M = 200) 252 / 245,
  // 256 207 / 189, float32 d = 64 327 / 298, 128 613 / 577.  The forms with registers to spare
  // gain nothing (bf16 d = 64 54.0 / 54.2) or lose (bf16 d = 96, 4 layers of 3 x 699 tokens, 53.1 /
  // 54.9; float32 d = 256 1344 / 1369).
  constexpr bool OPAQUE = EMIT && (sizeof(T) == 4 ? KS < 32 : KS == 5 || KS >= 8);
  __shared__ __attribute__((aligned(16))) float nls[EMIT ? 2 : 1][EMIT ? TL_ROWS : 4];
  __shared__ __attribute__((aligned(16))) float rests[REST ? 2 : 1][REST ? TL_ROWS : 4];

  const int layer = blockIdx.z;
  int b = 0, chunk = blockIdx.x;
  for (; b < a.batch - 1; ++b) {
    const int nc = (seq.cu[b + 1] - seq.cu[b] + KEYS - 1) / KEYS;
    if (chunk < nc) break;
    chunk -= nc;
  }
  const int tok0 = seq.cu[b], n = seq.cu[b + 1] - tok0;
  if (chunk * KEYS >= n) return;
  const int h = blockIdx.y / a.row_split, split = blockIdx.y - h * a.row_split;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int col = lane & 31, half = lane >> 5;
  const int wkey0 = chunk * KEYS + wave * 32 * KB;       // first key of the wave
  const int P = a.pieces;
  const uint4* q_head = static_cast<const uint4*>(q_tab.p[layer]) +
                        ((size_t)b * a.hkv + h) * a.group * a.window * P;
  const uint4* k_head = static_cast<const uint4*>(k_tab.p[layer]) + ((size_t)h * a.total + tok0) * P;
  // first query row of this (layer, sequence, KV head) among the rows of the launch
  const size_t qrow0 = (((size_t)layer * a.batch + b) * a.hkv + h) * a.group * a.window;
  const int R = EMIT ? a.group * a.head_rows : a.group * a.window;
  const int all_tiles = (R + TL_ROWS - 1) / TL_ROWS;
  const int t_begin = EMIT ? 0 : (int)((int64_t)all_tiles * split / a.row_split);
  const int t_end = EMIT ? all_tiles : (int)((int64_t)all_tiles * (split + 1) / a.row_split);
  if (t_begin >= t_end) return;

  // query row (among the head's group * window) that row `pr` in tile order stands for, and
  // whether it is a real one; never falling with pr
  auto source_row = [&](int pr, bool& real) -> int {
    if (!EMIT) { real = pr < R; return min(pr, R - 1); }
    uint32_t g = __umulhi((uint32_t)pr, a.head_magic);   // exact or one too large
    if (g * (uint32_t)a.head_rows > (uint32_t)pr) --g;
    const int m = pr - (int)g * a.head_rows;
    real = (int)g < a.group && m < a.window;
    return (int)g < a.group ? (int)g * a.window + min(m, a.window - 1) : a.group * a.window - 1;
  };
  const uint32_t qtile_lds = (uint32_t)(size_t)(__attribute__((address_space(3))) uint4*)(&qtile[0][0]);
  auto issue_tile = [&](int t) {
    const uint32_t dst = __builtin_amdgcn_readfirstlane(qtile_lds + (uint32_t)(t & 1) * (TL_ROWS * PS * 16));
    // scalar base: the first row of the tile; the others follow within 64 rows of it
    bool real;
    int ln = lane;
    if (OPAQUE) asm volatile("" : "+v"(ln));
    const int first = __builtin_amdgcn_readfirstlane(source_row(t * TL_ROWS, real));
    const uint64_t addr = reinterpret_cast<uint64_t>(q_head) + (uint64_t)(uint32_t)first * (uint32_t)(P * 16);
    const uint64_t base = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(addr >> 32)) << 32) |
                          (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)addr);
#pragma unroll
    for (int i = 0; i < DMA; ++i) {
      const int j = i * 4 + wave;                        // wave-uniform
      if (j < PS) {
        const int slot = j * 64 + ln;
        const int r = slot / PS, piece = min(slot - r * PS, P - 1);
        const uint32_t off = (uint32_t)((source_row(t * TL_ROWS + r, real) - first) * P + piece) * 16u;
        lds_dma16_s<false>(reinterpret_cast<const void*>(base), off, dst + j * 1024);
      }
    }
  };
  // EMIT: minus the log-sum-exp of row `lane` of tile t (and minus the rest of it)
  // (the sign and the padding rows where the loads are used: here they would wait for them at once)
  auto load_nl = [&](int t, float& rest) -> float {
    bool real;
    const int r = source_row(t * TL_ROWS + lane, real);
    rest = REST ? lse2[a.rows_all + qrow0 + r] : 0.f;
    return lse2[qrow0 + r];
  };
  auto store_nl = [&](int t, float lse, float rest) {
    bool real;
    source_row(t * TL_ROWS + lane, real);
    nls[t & 1][lane] = real ? -lse : NEG_BIG;
    if (REST) rests[t & 1][lane] = -rest;
  };

  issue_tile(t_begin);
  // ---- keys: registers for the whole kernel; pieces past the row are zero ----
  uint4 kf[KB][KS];
#pragma unroll
  for (int kb = 0; kb < KB; ++kb) {
    const uint4* krow = k_head + (size_t)min(wkey0 + kb * 32 + col, n - 1) * P;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const int piece = 2 * ks + half;
      kf[kb][ks] = piece < P ? krow[piece] : make_uint4(0, 0, 0, 0);
    }
  }
  float next_nl = 0.f, next_rest = 0.f;
  if (EMIT && wave == 0) {
    next_nl = load_nl(t_begin, next_rest);
    store_nl(t_begin, next_nl, next_rest);
  }

  const bool active = wkey0 < n;                                  // wave-uniform, like the next two
  const bool ragged = wkey0 + 32 * KB > n;
  const bool masked = a.causal && wkey0 + 32 * KB - 1 > n - a.window;
  const int subs = a.head_rows >> 3;                              // EMIT: groups of 8 rows per query head
  int sub = 0;                                                    // EMIT: of them, done of the current head
  float tacc[KB], gacc[KB];                                       // EMIT: current head's aggregate, group's
#pragma unroll
  for (int kb = 0; kb < KB; ++kb) { tacc[kb] = TASK_MAX ? NEG_BIG : 0.f; gacc[kb] = 0.f; }
  const float inv_window = 1.f / float(a.window);
  auto finish_head = [&]() {
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
      const float tv = cross_half<TASK_MAX>(tacc[kb]);
      const float sv = TASK_MAX ? fast_exp2(tv) : tv * inv_window;
      gacc[kb] = a.group_max ? fmaxf(gacc[kb], sv) : gacc[kb] + sv;
      tacc[kb] = TASK_MAX ? NEG_BIG : 0.f;
    }
    sub = 0;
  };
  // STATS: one wave joins the four waves' statistics of tile t (a row per lane)
  auto store_stats = [&](int t) {
    const int row = t * TL_ROWS + lane;
    if (wave != (t & 3) || row >= R) return;
    float2 x[4];
#pragma unroll
    for (int w = 0; w < 4; ++w) x[w] = stat[t & 1][w][lane];
    const float mm = fmaxf(fmaxf(x[0].x, x[1].x), fmaxf(x[2].x, x[3].x));
    float ss = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) ss += x[w].y * fast_exp2(x[w].x - mm);
    part_m[(size_t)chunk * a.rows_all + qrow0 + row] = mm;
    part_s[(size_t)chunk * a.rows_all + qrow0 + row] = ss;
  };

  for (int t = t_begin; t < t_end; ++t) {
    wait_loads();
    wait_lds();
    __syncthreads();                      // tile t is complete; every wave is done with tile t-1
    if (!EMIT && t > t_begin) store_stats(t - 1);
    if (t + 1 < t_end) {
      issue_tile(t + 1);
      if (EMIT && wave == 0) next_nl = load_nl(t + 1, next_rest);
    }
#pragma unroll
    for (int blk = 0; blk < 2; ++blk) {
      if (EMIT && !active) break;
      f32x16 acc[KB];
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[kb][r] = 0.f;
      // EMIT: -lse2 of the lane's rows, read from LDS before the products so that it is there after them
      float4 nl[4];
      if (EMIT) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          nl[i] = *reinterpret_cast<const float4*>(&nls[t & 1][blk * 32 + 8 * i + 4 * half]);
      }
      const uint4* qrow = &qtile[t & 1][(blk * 32 + col) * PS + half];
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const uint4 qf = qrow[2 * ks];
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
          acc[kb] = EMIT ? tile_mma<T>(qf, kf[kb][ks], acc[kb]) : tile_mma<T>(kf[kb][ks], qf, acc[kb]);
      }
      if constexpr (!EMIT) {
        if (ragged) {                     // keys past the sequence drop out
#pragma unroll
          for (int kb = 0; kb < KB; ++kb)
#pragma unroll
            for (int r = 0; r < 16; ++r)
              if (wkey0 + kb * 32 + acc_row(r, half) >= n) acc[kb][r] = -__builtin_inff();
        }
        if (masked) {                     // task token m sees keys up to n - window + m
          const int seen = n - a.window + (t * TL_ROWS + blk * 32 + col) % a.window;
#pragma unroll
          for (int kb = 0; kb < KB; ++kb)
#pragma unroll
            for (int r = 0; r < 16; ++r)
              if (wkey0 + kb * 32 + acc_row(r, half) > seen) acc[kb][r] = -__builtin_inff();
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
        if (half == 0) stat[t & 1][wave][blk * 32 + col] = make_float2(mx, s);
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
                if (wkey0 + kb * 32 + col > seen + r) acc[kb][4 * i + r] = -__builtin_inff();
            if (++m8 == subs) m8 = 0;
          }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          float4 rest = make_float4(0.f, 0.f, 0.f, 0.f);
          if (REST) rest = *reinterpret_cast<const float4*>(&rests[t & 1][blk * 32 + 8 * i + 4 * half]);
#pragma unroll
          for (int kb = 0; kb < KB; ++kb) {
            float x0 = fmaf(acc[kb][4 * i], a.c2, nl[i].x), x1 = fmaf(acc[kb][4 * i + 1], a.c2, nl[i].y);
            float x2 = fmaf(acc[kb][4 * i + 2], a.c2, nl[i].z), x3 = fmaf(acc[kb][4 * i + 3], a.c2, nl[i].w);
            if (REST) { x0 += rest.x; x1 += rest.y; x2 += rest.z; x3 += rest.w; }
            if (TASK_MAX) {
              tacc[kb] = fmaxf(fmaxf(tacc[kb], x0), x1);
              tacc[kb] = fmaxf(fmaxf(tacc[kb], x2), x3);
            } else {
              tacc[kb] += (fast_exp2(x0) + fast_exp2(x1)) + (fast_exp2(x2) + fast_exp2(x3));
            }
          }
          if (++sub == subs) finish_head();
        }
      }
    }
    if (EMIT && wave == 0 && t + 1 < t_end) store_nl(t + 1, next_nl, next_rest);
  }
  if constexpr (!EMIT) {
    wait_memory();
    __syncthreads();
    store_stats(t_end - 1);
  } else {
    float* out_head = out + (size_t)layer * a.out_layer_stride + (size_t)h * a.total + tok0;
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
      const int key = wkey0 + kb * 32 + col;
      if (half == 0 && key < n) out_head[key] = gacc[kb];
    }
  }
}

// k-steps a row of `pieces` 16-byte pieces is padded to: head sizes 64, 80, 96, 128 and 256 in
// bf16 and 32, 64, 128 and 256 in float32 need no padding.
inline int tile_ksteps(int dtype, int pieces) {
  const int ks = (pieces + 1) / 2;
  if (dtype == KVC_BF16) return ks <= 4 ? 4 : ks <= 5 ? 5 : ks <= 6 ? 6 : ks <= 8 ? 8 : 16;
  return ks <= 4 ? 4 : ks <= 8 ? 8 : ks <= 16 ? 16 : 32;
}
// keys per workgroup: two 32-key blocks per wave; one where a row takes 128 registers
constexpr int tile_keys(int ksteps) { return ksteps > 16 ? 128 : 256; }

}  // namespace
}  // namespace kvc
