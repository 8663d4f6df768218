// Max-pooling emit pass of kvc_score for the shapes of kvc_score_mfma.h, key-stationary: a workgroup keeps
// 256 keys of a KV head in registers and all query rows of the head pass through it.
// Included by kvc_score.hip only.
//
// The roles, the ring of query tiles and its loads are those of kvc_score_tile.h.  K is read once
// whatever the number of rows, a wave has the whole aggregate over task tokens and group of its keys in
// registers (no partials, no joining of waves), and no wave works on rows that don't exist.  Every
// rounding is that of the query-stationary emit pass: the accumulators of a 32-row block start from
// -(lse2[row] - lse2[first row])/c2 (score_merge wrote these start values), maximum, one FMA per
// block, one exponential per query head; heads are summed in row chunks of 256 rows, in order, and the
// row chunks in order.  A row chunk that score_merge found too spread out (EMIT_SPREAD_LIMIT) takes the
// exact form: zero start, one FMA per element.
#pragma once

namespace kvc {
namespace {

constexpr int EK_KB = 2;                       // 32-key blocks of a wave
static_assert(EK_KEYS == 4 * 32 * EK_KB, "a block of keys per wave");
constexpr int EK_RING = 3;
constexpr int EK_TILE = TL_ROWS * MF_D * 2;    // bytes of a tile of query rows

struct EmitKeysArgs {
  int batch, hkv, group, window, total, row_chunks;
  float c2;
  int causal, group_max;
  size_t rows_layer, rows_all;                 // query rows of a layer (batch * Hq * window), of the launch
  int chunk_shift;                             // MERGES: log2 of the keys of a statistics chunk
  size_t out_layer_stride;
};

// grid: ((sequence, chunk) pairs, Hkv, layers)
//
// MERGES: heads of one row chunk, statistics of a few chunks: a workgroup merges them for its rows
// itself (as score_merge_few, bit for bit), and start, lse2 and far are not used.
template <bool MERGES>
__global__ __launch_bounds__(TL_THREADS, 3) void score_emit_keys(
    PtrTable q_tab, PtrTable k_tab, SeqTable seq, EmitKeysArgs a, const float* __restrict__ part_m,
    const float* __restrict__ part_s, const float* __restrict__ start, const float* __restrict__ lse2,
    const uint32_t* __restrict__ far, float* __restrict__ out) {
  constexpr int ROWBUF = MERGES ? MF_RCHUNK / TL_ROWS : EK_RING;    // tiles whose start values are in LDS
  __shared__ __attribute__((aligned(1024))) unsigned char qtile[EK_RING][EK_TILE];
  __shared__ __attribute__((aligned(256))) float starts[ROWBUF][TL_ROWS], lses[ROWBUF][TL_ROWS];

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int col = lane & 31, half = lane >> 5;
  const int layer = blockIdx.z, h = blockIdx.y;
  int b = 0, chunk = blockIdx.x;
  for (; b < a.batch - 1; ++b) {
    const int nc = (seq.cu[b + 1] - seq.cu[b] + EK_KEYS - 1) / EK_KEYS;
    if (chunk < nc) break;
    chunk -= nc;
  }
  const int tok0 = seq.cu[b], n = seq.cu[b + 1] - tok0;
  if (chunk * EK_KEYS >= n) return;
  const int R = a.group * a.window, blocks = R / 32, tiles = (blocks + 1) / 2;
  const size_t head_row = ((size_t)b * a.hkv + h) * (uint32_t)R;
  const size_t qrow0 = (size_t)layer * a.rows_layer + head_row;
  auto scalar64 = [](uint64_t x) {
    return ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(x >> 32)) << 32) |
           (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)x);
  };

  // ---- query tiles to LDS: load j = 4 i + wave brings rows 4 j .. + 3, piece p of row r at slot p ^ (r & 15) ----
  const uint64_t q_head = scalar64(reinterpret_cast<uint64_t>(q_tab.p[layer]) + head_row * (MF_D * 2));
  const uint32_t qtile_lds = (uint32_t)(size_t)(__attribute__((address_space(3))) unsigned char*)(&qtile[0][0]);
  const uint32_t starts_lds = (uint32_t)(size_t)(__attribute__((address_space(3))) float*)(&starts[0][0]);
  const uint32_t lses_lds = (uint32_t)(size_t)(__attribute__((address_space(3))) float*)(&lses[0][0]);
  const int drow = wave * 4 + (lane >> 4);
  const uint32_t qoff = (uint32_t)(drow * MF_D * 2 + (((lane & 15) ^ (drow & 15)) << 4));
  int ahead_t = 0, ahead_buf = 0;       // the next tile to be asked for, and its buffer
  auto issue_tile = [&]() {
    const int t = ahead_t;
    if (!MERGES && wave == (t & 3)) {   // a row per lane
      const uint32_t off = (uint32_t)min(t * TL_ROWS + lane, R - 1) * 4u;
      lds_dma4_s(reinterpret_cast<const void*>(scalar64(reinterpret_cast<uint64_t>(start + qrow0))), off,
                 __builtin_amdgcn_readfirstlane(starts_lds + ahead_buf * (TL_ROWS * 4)));
      lds_dma4_s(reinterpret_cast<const void*>(scalar64(reinterpret_cast<uint64_t>(lse2 + qrow0))), off,
                 __builtin_amdgcn_readfirstlane(lses_lds + ahead_buf * (TL_ROWS * 4)));
    }
    const uint32_t dst = qtile_lds + (uint32_t)ahead_buf * EK_TILE + wave * 1024;
    const uint64_t tile = q_head + (uint64_t)(uint32_t)t * EK_TILE;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (i < 2 || 2 * t + 1 < blocks)  // (the last tile may have one block)
        lds_dma16_s<false>(reinterpret_cast<const void*>(scalar64(tile + i * 4096)), qoff,
                           __builtin_amdgcn_readfirstlane(dst + i * 4096));
    ahead_buf = ahead_buf + 1 == EK_RING ? 0 : ahead_buf + 1;
    ++ahead_t;
  };
  for (int i = 0; i < EK_RING - 1; ++i)
    if (ahead_t < tiles) issue_tile();

  // ---- keys: registers for the whole kernel ----
  const int wkey0 = chunk * EK_KEYS + wave * 32 * EK_KB;       // first key of the wave
  uint4 kf[EK_KB][8];
  {
    // scalar address of the wave's first key (or of the last one there is), keys behind it
    const int row = min(wkey0, n - 1), behind = n - 1 - row;
    typedef const __attribute__((address_space(1))) char* global_ptr;
    const global_ptr base = (global_ptr)scalar64(reinterpret_cast<uint64_t>(k_tab.p[layer]) +
        ((uint64_t)(uint32_t)h * (uint32_t)a.total + (uint32_t)(tok0 + row)) * (MF_D * 2));
#pragma unroll
    for (int kb = 0; kb < EK_KB; ++kb) {
      const uint32_t off = (uint32_t)min(kb * 32 + col, behind) * (MF_D * 2) + half * 16;
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) kf[kb][ks] = load16(base, off + ks * 32);
    }
  }
  // row chunks that take the exact form
  uint32_t exact_chunks = 0;
  if constexpr (MERGES) {
    const int row = threadIdx.x;
    float lse = 0.f, rest;
    if (row < R) lse = merge_few(part_m, part_s, qrow0 + row, a.rows_all, (n + (1 << a.chunk_shift) - 1) >> a.chunk_shift, rest);
    const float diff = __shfl(lse, lane & 32) - lse;   // (-lse2) - (-lse2 of the first row of the block)
    starts[0][row] = diff * (1.f / a.c2);
    lses[0][row] = lse;
    exact_chunks = __syncthreads_or(row < R && fabsf(diff) > EMIT_SPREAD_LIMIT) ? 1u : 0u;
  }
  for (int rc = MERGES ? a.row_chunks : 0; rc < a.row_chunks; ++rc)
    exact_chunks |= (far[(((size_t)layer * a.batch + b) * a.hkv + h) * a.row_chunks + rc] & 1u) << rc;
  exact_chunks = __builtin_amdgcn_readfirstlane(exact_chunks);

  const int bpg = a.window / 32;                               // blocks per query head
  const int unit = bpg > 8 ? bpg : 8;                          // blocks whose heads are summed on their own
  int head_left = bpg, unit_left = unit;                       // blocks left of the query head, of those
  const bool masked = a.causal && wkey0 + 32 * EK_KB - 1 > n - a.window;
  const float c2 = a.c2;
  float head[EK_KB], sum[EK_KB], total[EK_KB];                 // of the query head, the row chunk, the group
#pragma unroll
  for (int kb = 0; kb < EK_KB; ++kb) { head[kb] = NEG_BIG; sum[kb] = total[kb] = 0.f; }
  float pair[EK_KB] = {0.f, 0.f};                              // bpg = 1: value of an even block

  const int fbase = col * 256 + ((half ^ (col & 15)) << 4);
  auto frag = [&](int buf, int blk, int ks) {
    int at = fbase;                     // (opaque: no address per k-step is kept, registers are short)
    asm volatile("" : "+v"(at));
    return *reinterpret_cast<const uint4*>(&qtile[buf][blk * 8192 + (at ^ (32 * ks))]);
  };
  uint4 qf[4];                          // fragments run four k-steps ahead of their products
  f32x16 sv;                            // start values of the next block
  auto load_starts = [&](int rows, int blk) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float4 v = *reinterpret_cast<const float4*>(&starts[rows][blk * 32 + 8 * i + 4 * half]);
      sv[4 * i] = v.x; sv[4 * i + 1] = v.y; sv[4 * i + 2] = v.z; sv[4 * i + 3] = v.w;
    }
  };

  auto tile = [&](const int t, auto buffer) __attribute__((always_inline)) {
    constexpr int buf = decltype(buffer)::value, next_buf = buf + 1 == EK_RING ? 0 : buf + 1;
    // (behind the last tile its values are read again and not used)
    const int rows = MERGES ? t : buf, next_rows = MERGES ? min(t + 1, ROWBUF - 1) : next_buf;
    // this tile and the next, which the fragments run into, are complete, and every wave is done with the
    // tile before, whose buffer the next load takes
    wait_loads();
    wait_lds();
    __syncthreads();
    if (ahead_t < tiles) issue_tile();
    if (t == 0) {
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) qf[ks] = frag(buf, 0, ks);
      load_starts(rows, 0);
    }
#pragma unroll
    for (int blk = 0; blk < 2; ++blk) {
      const int block = 2 * t + blk;
      if (blk == 1 && block >= blocks) break;
      const bool exact = exact_chunks >> (block >> 3) & 1;
      f32x16 acc[EK_KB];
      const float base = -lses[rows][blk * 32];
      if (exact) {
        asm volatile("");               // (a branch, not 16 selects)
#pragma unroll
        for (int r = 0; r < 16; ++r) sv[r] = 0.f;
      }
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) {
#pragma unroll
        for (int kb = 0; kb < EK_KB; ++kb)
          acc[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(qf[ks & 3]), as_bf16x8(kf[kb][ks]),
                                                            ks == 0 ? sv : acc[kb], 0, 0, 0);
        // (behind the last block they are read and not used)
        if (ks < 4) qf[ks] = frag(buf, blk, ks + 4);
        else if (blk == 0) qf[ks & 3] = frag(buf, 1, ks - 4);
        else qf[ks & 3] = frag(next_buf, 0, ks - 4);
        if (ks == 1) load_starts(blk ? next_rows : rows, blk ^ 1);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (masked) {                     // task token m sees keys up to n - window + m
        const int seen = n - a.window + (block * 32) % a.window + 4 * half;
#pragma unroll
        for (int kb = 0; kb < EK_KB; ++kb)
#pragma unroll
          for (int r = 0; r < 16; ++r)
            if (wkey0 + kb * 32 + col > seen + acc_row(r, 0)) acc[kb][r] = NEG_BIG;
      }
      float v[EK_KB];
      if (exact) {
#pragma unroll
        for (int kb = 0; kb < EK_KB; ++kb) v[kb] = NEG_BIG;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float4 l = *reinterpret_cast<const float4*>(&lses[rows][blk * 32 + 8 * i + 4 * half]);
#pragma unroll
          for (int kb = 0; kb < EK_KB; ++kb) {
            v[kb] = fmaxf(fmaxf(v[kb], fmaf(acc[kb][4 * i], c2, -l.x)), fmaf(acc[kb][4 * i + 1], c2, -l.y));
            v[kb] = fmaxf(fmaxf(v[kb], fmaf(acc[kb][4 * i + 2], c2, -l.z)), fmaf(acc[kb][4 * i + 3], c2, -l.w));
          }
        }
      } else {
#pragma unroll
        for (int kb = 0; kb < EK_KB; ++kb) {
          v[kb] = fmaxf(acc[kb][0], acc[kb][1]);
#pragma unroll
          for (int r = 2; r < 16; r += 2) v[kb] = fmaxf(fmaxf(v[kb], acc[kb][r]), acc[kb][r + 1]);
          v[kb] = fmaf(v[kb], c2, base);
        }
      }
      // (the two half-waves are joined at the end of a head only: rounding is monotone)
      if (bpg == 1) {
#pragma unroll
        for (int kb = 0; kb < EK_KB; ++kb) {
          const float s = fast_exp2(cross_half<true>(v[kb]));
          if (blk == 0) pair[kb] = s;
          if (blk == 1 || block + 1 == blocks) {
            const float other = blk == 1 ? s : 0.f;
            const float part = a.group_max ? fmaxf(pair[kb], other) : pair[kb] + other;
            sum[kb] = a.group_max ? fmaxf(sum[kb], part) : sum[kb] + part;
          }
        }
      } else {
#pragma unroll
        for (int kb = 0; kb < EK_KB; ++kb) head[kb] = fmaxf(head[kb], v[kb]);
        if (--head_left == 0) {
          head_left = bpg;
#pragma unroll
          for (int kb = 0; kb < EK_KB; ++kb) {
            const float s = fast_exp2(cross_half<true>(head[kb]));
            sum[kb] = a.group_max ? fmaxf(sum[kb], s) : sum[kb] + s;
            head[kb] = NEG_BIG;
          }
        }
      }
      if (--unit_left == 0 || block + 1 == blocks) {
        unit_left = unit;
#pragma unroll
        for (int kb = 0; kb < EK_KB; ++kb) {
          total[kb] = a.group_max ? fmaxf(total[kb], sum[kb]) : total[kb] + sum[kb];
          sum[kb] = 0.f;
        }
      }
    }
  };
  for (int t = 0; t < tiles; t += EK_RING) {
    tile(t, std::integral_constant<int, 0>{});
    if (t + 1 < tiles) tile(t + 1, std::integral_constant<int, 1>{});
    if (t + 2 < tiles) tile(t + 2, std::integral_constant<int, 2>{});
  }
  const int key = wkey0 + half * 32 + col;
  if (key < n)
    out[(size_t)layer * a.out_layer_stride + (size_t)h * a.total + tok0 + key] = half ? total[1] : total[0];
}

}  // namespace
}  // namespace kvc
