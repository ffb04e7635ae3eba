// Per-task segmented kernels: LoRA shrink (a4), LoRA expand (the standalone
// vfm_lora_apply), and the per-task linear heads (a12).
//
// Rows are in plan order, so every task owns one contiguous segment of rows
// (and of requests).  Work is split into VFM_ROW_TILE-row tiles that never
// cross a task boundary (the plan's rtile_off), so a skewed task mix (a Zipf
// head task holding a third of the rows) still spreads over many blocks, and
// each block reads exactly one task's factors.  The task's A / B / head
// weights are gathered through the per-task pointer tables, so attaching or
// removing a task is a pointer update (paper Section 4.1 task extensions;
// Table 1 attach_adapter / remove_adapter).
//
// bf16: v_mfma_f32_16x16x32_bf16 with operands read straight from global
// memory (16-byte per-lane loads); the adapter factor feeds the MFMA A slot,
// the activation rows the B slot, so each lane ends with 4 consecutive
// output columns of one row.  fp32: the fp32 MFMA for the shrink, plain dot
// products elsewhere.
#include <algorithm>

#include "vfm_internal.h"

namespace {

__device__ __forceinline__ f32x4 mfma16(const bf16x8& a, const bf16x8& b, const f32x4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// Locate the task and row range of segmented tile `bid`.
__device__ inline void tile_rows(const Plan& pl, int bid, int& t, int& r0, int& r1) {
  t = upper_index(pl.rtile_off, pl.n_tasks + 1, bid);
  r0 = pl.seg_row[t] + (bid - pl.rtile_off[t]) * VFM_ROW_TILE;
  r1 = min(r0 + VFM_ROW_TILE, pl.seg_row[t + 1]);
}

// ---------------------------------------------------------------------------
// shrink: U[m, ucol + j] = s_t * X[m, :] . A_t[j, :]   (j < rpad, zero past r_t)
// ---------------------------------------------------------------------------
typedef const void __attribute__((address_space(1)))* gptr_t;
typedef void __attribute__((address_space(3)))* lptr_t;
__device__ __attribute__((aligned(16))) bf16 g_seg_zero[8];  // zero-initialised at load

// The task owning tile `tile` of the tiling that cuts each task's rows into
// ceil(rows_t / ROWS) tiles, in task order, and the tile's first row; one
// wave counts the tiles (each lane a contiguous run of tasks, then a prefix
// over the lanes) and the lane holding the tile finds it.  Returns false
// (block-uniform) past the last tile.  sl: 2 ints of LDS.
template <int ROWS>
__device__ inline bool rows_tile_task(const Plan& pl, int tile, int* sl, int* t_out, int* r0_out) {
  if (threadIdx.x < 64) {
    const int lane = threadIdx.x, n = pl.n_tasks;
    if (lane == 0) sl[0] = -1;
    const int per = (n + 63) / 64;
    const int t0 = min(lane * per, n), t1 = min(t0 + per, n);
    int cnt = 0;
    for (int t = t0; t < t1; ++t) cnt += (pl.seg_row[t + 1] - pl.seg_row[t] + ROWS - 1) / ROWS;
    int incl = cnt;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int v = __shfl_up(incl, o, 64);
      if (lane >= o) incl += v;
    }
    int off = incl - cnt;
    if (tile >= off && tile < incl) {
      for (int t = t0; t < t1; ++t) {
        const int nt = (pl.seg_row[t + 1] - pl.seg_row[t] + ROWS - 1) / ROWS;
        if (tile < off + nt) {
          sl[0] = t;
          sl[1] = pl.seg_row[t] + (tile - off) * ROWS;
          break;
        }
        off += nt;
      }
    }
  }
  __syncthreads();
  *t_out = sl[0];
  *r0_out = sl[1];
  return *t_out >= 0;
}

template <int NP, int NSUB, int NWV>
__global__ __launch_bounds__(64 * NWV) void shrink_bf16_kernel(Plan pl, ShrinkArgs a) {
  // One block per tile of 16 * NWV rows of one task (the plan's 64-row tiles
  // with 4 waves; 96-row tiles with 6 when the batch has more 64-row tiles
  // than CUs, so one round of blocks covers it); wave w owns 16 rows and
  // every projection of the group, so each row is read once for all of
  // them.  Each 64-column chunk of the task's A rows (shared by the waves)
  // and of the tile's activation rows goes through an LDS ring of NST stages
  // fed by global_load_lds: every wave-wide load moves 8 whole 128-byte rows,
  // and NST - 1 chunks are in flight while one is consumed.  A rows past the
  // rank come from a zero page; only the NSUB 16-row sub-tiles that the
  // largest rank reaches are computed.  LDS rows are 128 B with chunk
  // swizzle kc ^ ((row >> 1) & 7); a stage holds AR A rows, then the tile's
  // rows, then padding to whole block passes.  A row's sums are the same
  // MFMAs in the same order for either tile size.
  static_assert(NWV == 4 || NWV == 6, "the swizzle repeats every block pass for an even wave count");
  constexpr int ROWS = 16 * NWV;                // activation rows per block
  constexpr int AR = NP * NSUB * 16;            // A rows the MFMAs read per chunk
  constexpr int PR = 8 * NWV;                   // LDS rows one block pass of 16-byte loads fills
  constexpr int SR = (AR + ROWS + PR - 1) / PR * PR;   // LDS rows per stage
  constexpr int NST = 4;
  constexpr int ND = SR / PR;                   // 16-byte pieces per thread and chunk
  static_assert(NWV != 4 || ROWS == VFM_ROW_TILE, "the plan's row tiles");
  // one LDS object (the task slot sits past the ring): with a second one the
  // compiler would wait for the ring's DMA before every fragment read
  __shared__ __attribute__((aligned(16))) bf16 As[NST][SR * 64 + 8];
  int* const sl = reinterpret_cast<int*>(&As[NST - 1][SR * 64]);
  const int tile = blockIdx.x;
  int t, r0;
  if (NWV == 4) {
    t = block_tile_task(pl, tile, sl);
    r0 = pl.seg_row[t] + (tile - pl.rtile_off[t]) * VFM_ROW_TILE;
  } else if (!rows_tile_task<ROWS>(pl, tile, sl, &t, &r0)) {
    return;                                     // block-uniform: past the last tile
  }
  const int r1 = min(r0 + ROWS, pl.seg_row[t + 1]);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int rank = min(a.rank[t], NSUB * 16) & ~7;
  const float sc = a.scale[t];
  const bf16* X = (const bf16*)a.X;
  bf16* U = (bf16*)a.U;
  const int m = r0 + wave * 16 + (lane & 15);
  f32x4 acc[NP][NSUB];
#pragma unroll
  for (int pp = 0; pp < NP; ++pp)
#pragma unroll
    for (int s2 = 0; s2 < NSUB; ++s2) acc[pp][s2] = f32x4{0.f, 0.f, 0.f, 0.f};
  if (rank > 0) {   // block-uniform
    const bf16* src0[ND];
    const int prow0 = wave * 8 + (lane >> 3);
    const int kcl = (lane & 7) ^ ((prow0 >> 1) & 7);   // same for prow0 + PR i
#pragma unroll
    for (int i = 0; i < ND; ++i) {
      const int row = prow0 + i * PR;
      if (row < AR) {                                   // row = (pp*NSUB + s2)*16 + j
        const int pp = row / (NSUB * 16), j = row % (NSUB * 16);
        const bf16* At = (const bf16*)a.A[pp][t];         // NULL: a projection the task leaves bare
        src0[i] = j < rank && At != nullptr ? At + (int64_t)j * a.K + kcl * 8 : nullptr;
      } else if (row < AR + ROWS) {                     // rows past the tile's end re-read its last row
        src0[i] = X + (int64_t)min(r0 + row - AR, r1 - 1) * a.ldx + kcl * 8;
      } else {
        src0[i] = nullptr;                              // padding rows (never read)
      }
    }
    const int nc = a.K / 64;
    // every chunk index past the end re-reads the last chunk, so each step
    // issues the same ND loads and one wait count holds throughout
    auto issue = [&](int c, int st) {
      const int cc = min(c, nc - 1);
#pragma unroll
      for (int i = 0; i < ND; ++i) {
        const bf16* src = src0[i] ? src0[i] + cc * 64 : g_seg_zero;
        __builtin_amdgcn_global_load_lds((gptr_t)src, (lptr_t)(&As[st][(i * NWV + wave) * 512]), 16, 0, 0);
      }
    };
#pragma unroll
    for (int i = 0; i < NST - 1; ++i) issue(i, i);
    for (int c0 = 0; c0 < nc; c0 += NST) {
#pragma unroll
      for (int j = 0; j < NST; ++j) {
        const int c = c0 + j;
        if (c >= nc) break;
        // chunk c landed once at most (NST - 2) later groups are outstanding
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NST - 2) * ND) : "memory");
        __builtin_amdgcn_s_barrier();     // every wave's part is in LDS; stage (c-1) is free
        issue(c + NST - 1, (j + NST - 1) % NST);
        const bf16* Ab = As[j];
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
          const int kc = kk * 4 + (lane >> 4);
          const int xr = AR + wave * 16 + (lane & 15);
          const bf16x8 xf = *reinterpret_cast<const bf16x8*>(Ab + xr * 64 + ((kc ^ ((xr >> 1) & 7)) * 8));
#pragma unroll
          for (int pp = 0; pp < NP; ++pp)
#pragma unroll
            for (int s2 = 0; s2 < NSUB; ++s2) {
              const int r = (pp * NSUB + s2) * 16 + (lane & 15);
              const bf16x8 af = *reinterpret_cast<const bf16x8*>(Ab + r * 64 + ((kc ^ ((r >> 1) & 7)) * 8));
              acc[pp][s2] = mfma16(af, xf, acc[pp][s2]);
            }
        }
      }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // nothing lands after the block ends
  }
  if (m < r1) {
#pragma unroll
    for (int pp = 0; pp < NP; ++pp)
#pragma unroll
      for (int s2 = 0; s2 < NSUB; ++s2) {
        bf16x4 o;
#pragma unroll
        for (int i = 0; i < 4; ++i) o[i] = (bf16)(acc[pp][s2][i] * sc);
        *reinterpret_cast<bf16x4*>(U + (int64_t)m * a.ldu + a.ucol[pp] + s2 * 16 + 4 * (lane >> 4)) = o;
      }
    // the slot's columns past the computed sub-tiles (past every task's rank)
    for (int pp = 0; pp < NP; ++pp)
      for (int s2 = NSUB; s2 < a.rpad / 16; ++s2)
        *reinterpret_cast<bf16x4*>(U + (int64_t)m * a.ldu + a.ucol[pp] + s2 * 16 + 4 * (lane >> 4)) = bf16x4{};
  }
}

// fp32 shrink: one block per (16-row group of a segmented tile, projection),
// v_mfma_f32_16x16x4_f32 with the task's A rows in the A slot and the 16
// activation rows in the B slot; the 4 waves each take a quarter of K and
// their sums are added in wave order, so the chain over K is a quarter as
// long (latency bound: 1024 rows of width 256, 14.3 us with one thread per
// (row, column) over all of K, 5.4 us so).  A lane's 16-byte load holds 4
// consecutive k; MFMA e takes component e of both operands.
template <int NSUB>
__global__ __launch_bounds__(256) void shrink_f32_kernel(Plan pl, ShrinkArgs a) {
  __shared__ int tslot;
  __shared__ f32x4 red[4][NSUB][64];
  const int tile = blockIdx.x >> 2, grp = blockIdx.x & 3, p = blockIdx.y;
  const int t = block_tile_task(pl, tile, &tslot);
  const int r0 = pl.seg_row[t] + (tile - pl.rtile_off[t]) * VFM_ROW_TILE + grp * 16;
  const int r1 = min(pl.seg_row[t] + (tile - pl.rtile_off[t] + 1) * VFM_ROW_TILE, pl.seg_row[t + 1]);
  if (r0 >= r1) return;                               // block-uniform
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, g = lane >> 4;
  const int m = r0 + (lane & 15);
  // a NULL factor: a projection the task leaves bare
  const int rank = a.A[p][t] != nullptr ? min(a.rank[t], NSUB * 16) & ~7 : 0;
  f32x4 acc[NSUB];
#pragma unroll
  for (int s = 0; s < NSUB; ++s) acc[s] = f32x4{0.f, 0.f, 0.f, 0.f};
  if (rank > 0) {
    const int kq = a.K / 4, ko = wave * kq + 4 * g;   // K is a multiple of 64
    const float* xr = (const float*)a.X + (int64_t)min(m, r1 - 1) * a.ldx + ko;
    const float* ar[NSUB];
#pragma unroll
    for (int s = 0; s < NSUB; ++s)
      ar[s] = (const float*)a.A[p][t] + (int64_t)min(s * 16 + (lane & 15), rank - 1) * a.K + ko;
    // (not unrolled by the compiler, whatever it is told: a step waits for its own loads)
    for (int k = 0; k < kq; k += 16) {
      const f32x4 xv = *reinterpret_cast<const f32x4*>(xr + k);
#pragma unroll
      for (int s = 0; s < NSUB; ++s) {
        f32x4 av = *reinterpret_cast<const f32x4*>(ar[s] + k);
        if (s * 16 + (lane & 15) >= rank) av = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[s] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[e], xv[e], acc[s], 0, 0, 0);
      }
    }
  }
#pragma unroll
  for (int s = 0; s < NSUB; ++s) red[wave][s][lane] = acc[s];
  __syncthreads();
  const float sc = a.scale[t];
  // one sub-tile per wave; the slot's columns past the computed ones are zeros
  if (m < r1 && wave < a.rpad / 16) {
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if (wave < NSUB) v = (((red[0][wave][lane] + red[1][wave][lane]) + red[2][wave][lane]) + red[3][wave][lane]) * sc;
    *reinterpret_cast<f32x4*>((float*)a.U + (int64_t)m * a.ldu + a.ucol[p] + wave * 16 + 4 * g) = v;
  }
}

// ---------------------------------------------------------------------------
// expand: Y[m, n] += U[m, ucol + :r] . B_t[n, :r]     (fp32 Y)
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void expand_bf16_kernel(Plan pl, ExpandArgs a) {
  int t, r0, r1;
  tile_rows(pl, blockIdx.x, t, r0, r1);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int rank = min(a.rank[t], a.max_rank) & ~7;
  const int wr0 = r0 + wave * 16;
  const bf16* Bt = (const bf16*)a.B[t];
  if (rank <= 0 || wr0 >= r1 || Bt == nullptr) return;
  const int n0 = blockIdx.y * 64;
  const bf16* U = (const bf16*)a.U;
  f32x4 acc[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) acc[s] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int m = wr0 + (lane & 15);
  for (int kk = 0; kk < rank; kk += 32) {
    const int kof = kk + 8 * (lane >> 4);
    bf16x8 xf = {};
    if (m < r1 && kof < rank) xf = *reinterpret_cast<const bf16x8*>(U + (int64_t)m * a.ldu + a.ucol + kof);
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int n = n0 + s * 16 + (lane & 15);
      bf16x8 wf = {};
      if (n < a.N && kof < rank) wf = *reinterpret_cast<const bf16x8*>(Bt + (int64_t)n * rank + kof);
      acc[s] = mfma16(wf, xf, acc[s]);
    }
  }
  if (m >= r1) return;
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const int n = n0 + s * 16 + 4 * (lane >> 4);
    if (n >= a.N) continue;
    float4* dst = reinterpret_cast<float4*>(a.Y + (int64_t)m * a.ldy + n);
    float4 o = *dst;
    o.x += acc[s][0]; o.y += acc[s][1]; o.z += acc[s][2]; o.w += acc[s][3];
    *dst = o;
  }
}

__global__ __launch_bounds__(256) void expand_f32_kernel(Plan pl, ExpandArgs a) {
  int t, r0, r1;
  tile_rows(pl, blockIdx.x, t, r0, r1);
  const int rank = min(a.rank[t], a.max_rank) & ~7;
  const float* Bt = (const float*)a.B[t];
  if (rank <= 0 || Bt == nullptr) return;
  const int n0 = blockIdx.y * 64;
  const float* U = (const float*)a.U;
  for (int e = threadIdx.x; e < (r1 - r0) * 64; e += 256) {
    const int m = r0 + e / 64, n = n0 + e % 64;
    if (n >= a.N) continue;
    float s = 0.f;
    for (int j = 0; j < rank; ++j) s += U[(int64_t)m * a.ldu + a.ucol + j] * Bt[(int64_t)n * rank + j];
    a.Y[(int64_t)m * a.ldy + n] += s;
  }
}

// ---------------------------------------------------------------------------
// heads: out[out_off[order[p]] + n] = pooled[p] . W_t[n] + b_t[n]
//
// HID: the MLP heads' first layer, hid[p, n] = act(pooled[p] . W1_t[n] +
// b1_t[n]) for tasks with an MLP head; otherwise the output layer, out =
// in[p] . W_t[n] + b_t[n] with `in` the pooled row (linear head) or the
// hidden row (MLP head).
//
// Bound by the tasks' weights, each read once, and by the latency of the
// chain over K.  One block per (task, 16 outputs): its 8 waves split K and
// add their sums in wave order through LDS, so a wave's chain is K / 8 and
// the chip holds outputs / 16 times 8 waves per task (256 requests of 71
// tasks, 256 outputs of K = 4096: 1136 blocks; 214.8 us with a wave walking
// the whole K for 16 outputs, 36.9 us = 4.1 TB/s of weights so).  Up to
// HEAD_NG groups of 16 requests share a pass over the weights (2 instead of
// 4: 10 us more, the task of 55 requests then reads its weights twice).  A
// request's sums depend on K alone, never on the other requests.
// ---------------------------------------------------------------------------
constexpr int HEAD_WAVES = 8;
constexpr int HEAD_NG = 4;

// acc[j] = the wave's share of K (32-column steps k0 .. k1) of 16 outputs
// times the 16 requests of group j
template <int NG>
__device__ __forceinline__ void head_dots(const bf16* wrow, const bf16* const (&xrow)[HEAD_NG], int k0, int k1,
                                          f32x4 (&acc)[HEAD_NG]) {
  constexpr int U = NG <= 2 ? 8 : 4;                    // steps whose loads are in flight together
  int k = k0;
  for (; k + 32 * U <= k1; k += 32 * U) {
    bf16x8 wf[U], xf[U][NG];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      wf[u] = *reinterpret_cast<const bf16x8*>(wrow + k + 32 * u);
#pragma unroll
      for (int j = 0; j < NG; ++j) xf[u][j] = *reinterpret_cast<const bf16x8*>(xrow[j] + k + 32 * u);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int j = 0; j < NG; ++j) acc[j] = mfma16(wf[u], xf[u][j], acc[j]);
  }
  for (; k < k1; k += 32) {
    const bf16x8 wf = *reinterpret_cast<const bf16x8*>(wrow + k);
#pragma unroll
    for (int j = 0; j < NG; ++j)
      acc[j] = mfma16(wf, *reinterpret_cast<const bf16x8*>(xrow[j] + k), acc[j]);
  }
}

// BYREQ: the table has more tasks than the batch has requests.  A block is
// then found by plan position, and a task's blocks are those of its first
// request, so the grid grows with the batch and not with the table: pooling
// and head of one request among 8192 tasks of 1000 outputs 316 us with a block
// per task and 16 outputs, 18.8 us so (among 16 tasks: 17.5).
template <bool HID, bool BYREQ>
__global__ __launch_bounds__(64 * HEAD_WAVES) void heads_bf16_kernel(Plan pl, const bf16* __restrict__ pooled,
                                                                    int d, vfm_head_table h, int nchunk,
                                                                    bf16* __restrict__ hid,
                                                                    float* __restrict__ out) {
  __shared__ f32x4 red[HEAD_WAVES][HEAD_NG][64];
  // a task's blocks follow each other, in task order: the tasks of skewed
  // mixes that own most requests (the first ids under a Zipf law) start first
  const int i = blockIdx.x / nchunk, chunk = blockIdx.x % nchunk;
  const int t = BYREQ ? pl.task[i] : i;
  if (BYREQ && i > 0 && pl.task[i - 1] == t) return;   // block-uniform: not the task's first request
  // every table entry is requested before the first is used
  const int p0 = pl.seg_req[t], p1 = pl.seg_req[t + 1];
  const void* const w1 = h.W1 != nullptr ? h.W1[t] : nullptr;
  const void* const w0 = HID ? nullptr : h.W[t];
  const int no = HID ? h.hidden : h.n_out[t];
  const bf16* bt = HID ? (h.b1 ? (const bf16*)h.b1[t] : nullptr) : (h.b ? (const bf16*)h.b[t] : nullptr);
  const bool mlp = w1 != nullptr;
  if (p0 == p1 || chunk * 16 >= no || (HID && !mlp)) return;   // block-uniform
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const bf16* Wt = (const bf16*)(HID ? w1 : w0);
  const bool from_hid = !HID && mlp;
  const int K = from_hid ? h.hidden : d;              // a multiple of 64
  const bf16* in = from_hid ? hid : pooled;
  const int k0 = wave * (K / 32) / HEAD_WAVES * 32, k1 = (wave + 1) * (K / 32) / HEAD_WAVES * 32;
  for (int n0 = chunk * 16; n0 < no; n0 += nchunk * 16)
  for (int pb = p0; pb < p1; pb += 16 * HEAD_NG) {
    const bf16* wrow = Wt + (int64_t)min(n0 + (lane & 15), no - 1) * K + 8 * (lane >> 4);
    const bf16* xrow[HEAD_NG];
    f32x4 acc[HEAD_NG];
#pragma unroll
    for (int j = 0; j < HEAD_NG; ++j) {
      xrow[j] = in + (int64_t)min(pb + 16 * j + (lane & 15), p1 - 1) * K + 8 * (lane >> 4);
      acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    const int ng = min((p1 - pb + 15) / 16, HEAD_NG);   // block-uniform
    // where this wave's group goes, read ahead of the products
    const int p = pb + 16 * (wave % HEAD_NG) + (lane & 15), nb = n0 + 4 * (lane >> 4);
    const int req = HID ? 0 : pl.order[min(p, p1 - 1)];
    const int o0 = HID ? 0 : pl.out_off[req], o1 = HID ? 0 : pl.out_off[req + 1];
    if (ng == 1) head_dots<1>(wrow, xrow, k0, k1, acc);
    else if (ng == 2) head_dots<2>(wrow, xrow, k0, k1, acc);
    else head_dots<HEAD_NG>(wrow, xrow, k0, k1, acc);
#pragma unroll
    for (int j = 0; j < HEAD_NG; ++j)
      if (j < ng) red[wave][j][lane] = acc[j];
    __syncthreads();
    if (wave < ng && p < p1) {                         // wave j finishes group j
      f32x4 v = red[0][wave][lane];
#pragma unroll
      for (int w = 1; w < HEAD_WAVES; ++w) {
        const f32x4 u = red[w][wave][lane];
        v[0] += u[0]; v[1] += u[1]; v[2] += u[2]; v[3] += u[3];
      }
      const int lim = HID ? no : min(no, o1 - o0);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (nb + i >= lim) break;
        const float y = v[i] + (bt ? (float)bt[nb + i] : 0.f);
        if (HID) hid[(int64_t)p * h.hidden + nb + i] = (bf16)(h.act == VFM_ACT_RELU ? fmaxf(y, 0.f) : gelu_fast(y));
        else out[o0 + nb + i] = y;
      }
    }
    __syncthreads();                                   // red is reused by the next groups
  }
}

// fp32: 16 lanes per (request, output), each lane every 16th group of 4
// columns, so a block has 16 dots in flight (one thread per dot walked K
// alone: 40.1 us for 16 requests of 10 outputs, 6.0 us so).
template <bool HID>
__global__ __launch_bounds__(256) void heads_f32_kernel(Plan pl, const float* __restrict__ pooled,
                                                        int d, vfm_head_table h, float* __restrict__ hid,
                                                        float* __restrict__ out) {
  const int t = blockIdx.x;
  const bool mlp = h.W1 != nullptr && h.W1[t] != nullptr;
  if (HID && !mlp) return;
  const int n_out = HID ? h.hidden : h.n_out[t];
  const int n0 = blockIdx.y * 64;
  const int p0 = pl.seg_req[t], p1 = pl.seg_req[t + 1];
  if (p0 == p1 || n0 >= n_out) return;
  const float* Wt = (const float*)(HID ? h.W1[t] : h.W[t]);
  const float* bt = HID ? (h.b1 ? (const float*)h.b1[t] : nullptr) : (h.b ? (const float*)h.b[t] : nullptr);
  const bool from_hid = !HID && mlp;
  const int K = from_hid ? h.hidden : d;              // a multiple of 64
  const float* in = from_hid ? hid : pooled;
  const int sub = threadIdx.x & 15, nc = min(64, n_out - n0);
  const int total = (p1 - p0) * nc;
  for (int e0 = 0; e0 < total; e0 += 16) {
    const int e = min(e0 + (int)(threadIdx.x >> 4), total - 1);   // the last ones again past the end
    const int p = p0 + e / nc, n = n0 + e % nc;
    const float* x = in + (int64_t)p * K + 4 * sub;
    const float* w = Wt + (int64_t)n * K + 4 * sub;
    float s = 0.f;
#pragma unroll 4
    for (int k = 0; k < K; k += 64) {
      const float4 xv = *reinterpret_cast<const float4*>(x + k), wv = *reinterpret_cast<const float4*>(w + k);
      s = fmaf(xv.x, wv.x, s);
      s = fmaf(xv.y, wv.y, s);
      s = fmaf(xv.z, wv.z, s);
      s = fmaf(xv.w, wv.w, s);
    }
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) s += __shfl_xor(s, o, 64);
    if (sub != 0 || e0 + (int)(threadIdx.x >> 4) >= total) continue;
    s += bt ? bt[n] : 0.f;
    if (HID) {
      hid[(int64_t)p * h.hidden + n] =
          h.act == VFM_ACT_RELU ? fmaxf(s, 0.f) : 0.5f * s * (1.f + erff(s * 0.70710678118654752440f));
    } else {
      const int req = pl.order[p];
      if (n < min(n_out, pl.out_off[req + 1] - pl.out_off[req])) out[pl.out_off[req] + n] = s;
    }
  }
}

// ---------------------------------------------------------------------------
// Greedy token selection: one block per request (original order), each
// thread scans a strided share of the request's outputs, then the wave and
// the block reduce (value, index) pairs.
// ---------------------------------------------------------------------------
__device__ inline bool greedy_better(float v, int i, float bv, int bi) {
  if (i < 0) return false;
  if (bi < 0) return true;
  return v > bv || (v == bv && i < bi);
}

__global__ __launch_bounds__(256) void greedy_kernel(Plan pl, const float* __restrict__ out,
                                                     int32_t* __restrict__ ids) {
  __shared__ float sv[4];
  __shared__ int si[4];
  const int i = blockIdx.x;
  const int o0 = pl.out_off[i], n = pl.out_off[i + 1] - o0;
  float bv = 0.f;
  int bi = -1;
  for (int j = threadIdx.x; j < n; j += 256) {
    const float v = out[o0 + j];
    if (v == v && greedy_better(v, j, bv, bi)) { bv = v; bi = j; }
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    const float ov = __shfl_xor(bv, off, 64);
    const int oi = __shfl_xor(bi, off, 64);
    if (greedy_better(ov, oi, bv, bi)) { bv = ov; bi = oi; }
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) { sv[wave] = bv; si[wave] = bi; }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 4; ++w)
      if (greedy_better(sv[w], si[w], bv, bi)) { bv = sv[w]; bi = si[w]; }
    ids[i] = bi;
  }
}

}  // namespace

hipError_t launch_lora_shrink(int dtype, const Plan& pl, const ShrinkArgs& a, hipStream_t s) {
  if (pl.n_rtiles == 0 || a.n_proj == 0) return hipSuccess;
  if (dtype == VFM_BF16) {
    // the plan's 64-row tiles while one round of blocks holds them, else
    // 96-row tiles (a bound on their count; blocks past the last one leave)
    const bool big = pl.n_rtiles > 256;
    const dim3 grid(big ? (pl.T + 95) / 96 + std::min(pl.n_tasks, pl.n_req) : pl.n_rtiles);
    // sub-tiles the table's ranks need: 1 (rank <= 16), 2 (<= 32) or 4
    const int ns = a.nsub <= 1 ? 1 : (a.nsub == 2 ? 2 : 4);
#define SHR(NP_, NS_)                                                                              \
  do {                                                                                             \
    if (big) hipLaunchKernelGGL((shrink_bf16_kernel<NP_, NS_, 6>), grid, dim3(384), 0, s, pl, a); \
    else hipLaunchKernelGGL((shrink_bf16_kernel<NP_, NS_, 4>), grid, dim3(256), 0, s, pl, a);     \
  } while (0)
#define SHR_NP(NS_) do { if (a.n_proj == 1) SHR(1, NS_); else if (a.n_proj == 2) SHR(2, NS_); else SHR(3, NS_); } while (0)
    if (ns == 1) SHR_NP(1);
    else if (ns == 2) SHR_NP(2);
    else SHR_NP(4);
#undef SHR_NP
#undef SHR
  } else {
    dim3 grid(4 * pl.n_rtiles, a.n_proj);
    if (a.nsub <= 1) hipLaunchKernelGGL(shrink_f32_kernel<1>, grid, dim3(256), 0, s, pl, a);
    else if (a.nsub == 2) hipLaunchKernelGGL(shrink_f32_kernel<2>, grid, dim3(256), 0, s, pl, a);
    else hipLaunchKernelGGL(shrink_f32_kernel<4>, grid, dim3(256), 0, s, pl, a);
  }
  return hipGetLastError();
}

hipError_t launch_lora_expand(int dtype, const Plan& pl, const ExpandArgs& a, hipStream_t s) {
  if (pl.n_rtiles == 0) return hipSuccess;
  dim3 grid(pl.n_rtiles, (a.N + 63) / 64);
  if (dtype == VFM_BF16) hipLaunchKernelGGL(expand_bf16_kernel, grid, dim3(256), 0, s, pl, a);
  else hipLaunchKernelGGL(expand_f32_kernel, grid, dim3(256), 0, s, pl, a);
  return hipGetLastError();
}

// The pooled rows sit at the start of the head workspace; the MLP heads'
// hidden rows follow at the next 256-byte boundary ([n_req, hidden]).
hipError_t launch_heads(int dtype, const Plan& pl, const void* pooled, int d,
                        const vfm_head_table& h, float* out, hipStream_t s) {
  const size_t es = dtype == VFM_BF16 ? 2 : 4;
  char* hid = (char*)pooled + (((size_t)pl.n_req * d * es + 255) & ~(size_t)255);
  // blocks per task: one per 16 outputs, fewer (each then takes several
  // chunks) only where tasks x chunks would outgrow a grid
  const bool byreq = pl.n_req < h.n_tasks;
  const int nt = byreq ? pl.n_req : h.n_tasks;
  auto chunks = [&](int n) { return std::max(1, std::min((n + 15) / 16, (1 << 22) / nt)); };
  const int nh = chunks(h.hidden), no = chunks(h.max_out);
#define HEADS_BF16(HID_, BY_, N_)                                                                        \
  hipLaunchKernelGGL((heads_bf16_kernel<HID_, BY_>), dim3(nt * N_), dim3(64 * HEAD_WAVES), 0, s, pl, \
                     (const bf16*)pooled, d, h, N_, (bf16*)hid, out)
  if (h.W1 && h.hidden > 0) {
    if (dtype == VFM_BF16) { if (byreq) HEADS_BF16(true, true, nh); else HEADS_BF16(true, false, nh); }
    else
      hipLaunchKernelGGL((heads_f32_kernel<true>), dim3(h.n_tasks, (h.hidden + 63) / 64), dim3(256), 0, s, pl,
                         (const float*)pooled, d, h, (float*)hid, out);
  }
  if (h.max_out == 0) return hipGetLastError();
  if (dtype == VFM_BF16) { if (byreq) HEADS_BF16(false, true, no); else HEADS_BF16(false, false, no); }
  else
    hipLaunchKernelGGL((heads_f32_kernel<false>), dim3(h.n_tasks, (h.max_out + 63) / 64), dim3(256), 0, s, pl,
                       (const float*)pooled, d, h, (float*)hid, out);
#undef HEADS_BF16
  return hipGetLastError();
}

hipError_t launch_greedy(const Plan& pl, const float* out, int32_t* ids, hipStream_t s) {
  hipLaunchKernelGGL(greedy_kernel, dim3(pl.n_req), dim3(256), 0, s, pl, out, ids);
  return hipGetLastError();
}
