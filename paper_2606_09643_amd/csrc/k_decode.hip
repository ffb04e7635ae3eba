// Shared projections for small batches (decode: one token per request).
//
// With a few hundred rows every weight element is used by few rows, so the
// shared projections stream the weights from HBM, and the per-task LoRA work
// is a gather of each task's factors for the handful of rows it owns
// (Section 4.2 adapter handling, applied per task on the shared batch).
// Three kernels per projection group replace the large-tile GEMM:
//
//   gemm_skinny    Z[s, m, n] = sum over K range s of X[m, k] W[n, k]:
//                  row x column tiles, LDS rings fed by global_load_lds,
//                  K split so the grid covers the chip (or, with enough
//                  rows, every split walked by one block).
//                  Partials stay per split (fp32, no atomics), so results
//                  do not depend on scheduling.
//   shrink_split   P[c, m, slot + j] = sum over K chunk c of X[m, k] A_t[j, k]:
//                  one block per (task row tile, K chunk), so a task's A
//                  factors are read once, by many blocks at a time; up to 64
//                  rows in blocks of the GEMM's launch.
//   finalize       per row: U = bf16(s_t * sum_c P) rebuilt in LDS, then
//                  y = sum of the slices + U B_t^T + bias and the activation
//                  or residual epilogue, streamed one thread per 4 outputs
//                  (B_t rows read straight from the task's factor: the
//                  per-task adapter gather).
#include <algorithm>

#include "vfm_internal.h"

namespace {

typedef const void __attribute__((address_space(1)))* gptr_t;
typedef void __attribute__((address_space(3)))* lptr_t;

__device__ __forceinline__ f32x4 mfma16(const bf16x8& a, const bf16x8& b, const f32x4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
// 128-byte LDS rows: logical 16-byte chunk kc of row r sits at chunk
// kc ^ ((r >> 1) & 7), which spreads the 16-row fragment reads over all banks.
__device__ __forceinline__ int swz(int row, int kc) { return kc ^ ((row >> 1) & 7); }

constexpr int SBK = 64;

// ---------------------------------------------------------------------------
// Split-K segmented shrink: one wave's NG groups of 16 rows from row m0 (rows
// below r1 are the tile's) of task t, NP projections from pp0 on, columns of K
// chunk c; A rows feed the MFMA A slot, X rows the B slot.  The groups share
// the A rows of a step and go through K together: a wave's time is its chain of
// loads (a tile's 16-row groups one after the other in the GEMM's launch: one
// 64-row prompt, ranks 16 / 64, of a 4096-wide layer 184.2 / 294.3 us, together
// 166.8 / 212.0; 1024-wide 118.5 / 188.9, 95.3 / 136.9).
// ---------------------------------------------------------------------------
template <int NP, int NSUB, int NG>
__device__ __forceinline__ void shrink_split_rows(const Plan& pl, const ShrinkSplitArgs& a, int t, int m0, int r1,
                                                  int c, int pp0, int lane) {
  const int rank = min(a.rank[t], NSUB * 16);
  const int m = m0 + (lane & 15);
  const int k0 = c * a.kchunk, k1 = min(k0 + a.kchunk, a.K);
  f32x4 acc[NG][NP][NSUB];
#pragma unroll
  for (int g = 0; g < NG; ++g)
#pragma unroll
    for (int pp = 0; pp < NP; ++pp)
#pragma unroll
      for (int s = 0; s < NSUB; ++s) acc[g][pp][s] = f32x4{0.f, 0.f, 0.f, 0.f};
  if (rank > 0 && m0 < r1) {
    const bf16* xrow[NG];
#pragma unroll
    for (int g = 0; g < NG; ++g)
      xrow[g] = (const bf16*)a.X + (int64_t)min(m + 16 * g, r1 - 1) * a.ldx + 8 * (lane >> 4);
    // told that the factors lie in global memory: with a projection known only
    // at run time the compiler loses track of it and loads them flat
    typedef const bf16 __attribute__((address_space(1)))* growp;
    typedef const bf16x8 __attribute__((address_space(1)))* gfragp;
    growp arow[NP][NSUB];
    bool on[NP][NSUB];
#pragma unroll
    for (int pp = 0; pp < NP; ++pp) {
      const growp At = (growp)((const void* const __attribute__((address_space(1)))*)a.A[pp0 + pp])[t];
      // NULL: a projection the task leaves bare (its rows read X and count as zeros)
      const bool bare = At == nullptr;
      const growp A0 = bare ? (growp)a.X : At;
#pragma unroll
      for (int s = 0; s < NSUB; ++s) {
        on[pp][s] = s * 16 + (lane & 15) < rank && !bare;
        arow[pp][s] = A0 + (bare ? 0 : (int64_t)min(s * 16 + (lane & 15), rank - 1) * a.K) + 8 * (lane >> 4);
      }
    }
    // (not unrolled by the compiler, whatever it is told: a step waits for its own loads)
    for (int k = k0; k < k1; k += 32) {
      bf16x8 xf[NG];
#pragma unroll
      for (int g = 0; g < NG; ++g) xf[g] = *reinterpret_cast<const bf16x8*>(xrow[g] + k);
#pragma unroll
      for (int pp = 0; pp < NP; ++pp)
#pragma unroll
        for (int s = 0; s < NSUB; ++s) {
          bf16x8 af = *(gfragp)(arow[pp][s] + k);
          if (!on[pp][s]) af = bf16x8{};
#pragma unroll
          for (int g = 0; g < NG; ++g) acc[g][pp][s] = mfma16(af, xf[g], acc[g][pp][s]);
        }
    }
  }
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    if (m + 16 * g >= r1) continue;
    float* P = a.P + ((int64_t)c * pl.T + m + 16 * g) * a.ldp;
#pragma unroll
    for (int pp = 0; pp < NP; ++pp)
#pragma unroll
      for (int s = 0; s < NSUB; ++s)
        *reinterpret_cast<float4*>(P + a.ucol[pp0 + pp] + s * 16 + 4 * (lane >> 4)) =
            make_float4(acc[g][pp][s][0], acc[g][pp][s][1], acc[g][pp][s][2], acc[g][pp][s][3]);
  }
}

// A launch of its own: block (row tile, K chunk), wave w takes rows 16 w ..
template <int NP, int NSUB>
__global__ __launch_bounds__(256) void shrink_split_kernel(Plan pl, ShrinkSplitArgs a) {
  __shared__ int s_task;
  const int tile = blockIdx.x;
  const int t = block_tile_task(pl, tile, &s_task);
  const int r0 = pl.seg_row[t] + (tile - pl.rtile_off[t]) * VFM_ROW_TILE;
  const int r1 = min(r0 + VFM_ROW_TILE, pl.seg_row[t + 1]);
  shrink_split_rows<NP, NSUB, 1>(pl, a, t, r0 + (threadIdx.x >> 6) * 16, r1, blockIdx.y, 0, threadIdx.x & 63);
}

// Part of the split GEMM's launch: wave item (row tile, projection, K chunk).
__device__ __forceinline__ void shrink_split_item(const Plan& pl, const ShrinkSplitArgs& a, int item, int lane) {
  const int c = item % a.kchunks, pp = item / a.kchunks % a.n_proj, tile = item / a.kchunks / a.n_proj;
  if (tile >= pl.n_rtiles) return;             // wave-uniform
  // the tile's task, the last one whose tiles start at or before it: a search in
  // 64 parts, one round of loads up to 64 tasks, two up to 4096 (one decode row
  // of a 2048-wide layer, 128 / 1024 / 8192 tasks: 69 / 78 / 157 us with a scan
  // of the table, 64 tasks a round, 69 / 70 / 70 so)
  int t = 0;
  for (int len = pl.n_tasks; len > 1;) {
    const int part = (len + 63) / 64;
    const bool before = lane * part < len && pl.rtile_off[t + min(lane * part, len - 1)] <= tile;
    const int k = (int)__builtin_popcountll(__ballot(before)) - 1;   // part 0 always is: rtile_off[t] <= tile
    t += k * part;
    len = min(part, len - k * part);
  }
  const int r0 = pl.seg_row[t] + (tile - pl.rtile_off[t]) * VFM_ROW_TILE;
  const int r1 = min(r0 + VFM_ROW_TILE, pl.seg_row[t + 1]);
  if (r1 - r0 <= 16) {
    if (a.nsub <= 1) shrink_split_rows<1, 1, 1>(pl, a, t, r0, r1, c, pp, lane);
    else if (a.nsub == 2) shrink_split_rows<1, 2, 1>(pl, a, t, r0, r1, c, pp, lane);
    else shrink_split_rows<1, 4, 1>(pl, a, t, r0, r1, c, pp, lane);
  } else {
    if (a.nsub <= 1) shrink_split_rows<1, 1, 4>(pl, a, t, r0, r1, c, pp, lane);
    else if (a.nsub == 2) shrink_split_rows<1, 2, 4>(pl, a, t, r0, r1, c, pp, lane);
    else shrink_split_rows<1, 4, 4>(pl, a, t, r0, r1, c, pp, lane);
  }
}

// ---------------------------------------------------------------------------
// Split-K GEMM, BM rows x BN = 64 * NWN columns per block, 4 x NWN waves of
// BM / 4 x 64.
//
// Every weight element is used by the few hundred rows of one tile only, so
// the weight stream comes from HBM at full latency while the activation
// columns are L2 hits.  Half of the waves load activation stages (XST - 1
// steps ahead, XST LDS stages), the other half weight stages (WST - 1 steps
// ahead, WST LDS stages): a wave's loads complete in issue order, so
// keeping the two streams in different waves lets the short-latency
// activation loads be waited on without waiting for the weight loads
// behind them.  All waves take part in the MFMA work.
//
// BM is 64, 128 or 256, the smallest that holds the batch (256-row tiles
// beyond): a tile's rows past the batch cost their LDS fill and their MFMAs
// like real ones, and a 256-row tile of one row spends more on them than on
// the weights.  One row of the 7B decoder, QKV / O / gate+up / down: 27.4 /
// 12.3 / 47.2 / 28.0 us with 256-row tiles, 18.7 / 8.9 / 29.6 / 20.8 with 64
// (5.4 / 3.8 / 6.1 / 4.3 TB/s of weights); deeper weight rings in the LDS that
// this frees (6 or 8 stages) gained nothing, deeper activation rings a little
// (37 rows, down: 23.5 -> 21.0 us with 4 activation and 3 weight stages).  The
// K steps and their order are
// the same for every BM, and so are a row's sums.
// ---------------------------------------------------------------------------
template <int N>
__device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N < 64, "vmcnt field");
  // vmcnt(N) (bits 3:0 and 15:14), lgkmcnt / expcnt not waited
  __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}
// wait until at most `newer` steps (MAX at most) of R loads each are outstanding
template <int R, int MAX>
__device__ __forceinline__ void wait_newer(int newer) {
  if constexpr (MAX == 0) {
    wait_vm<0>();
  } else {
    if (newer >= MAX) wait_vm<MAX * R>();
    else wait_newer<R, MAX - 1>(newer);
  }
}

//
// WALK: a block walks every split of its tile, adding each split's sums to a
// total (the finalize's order), and writes one slice.  With enough rows the
// row tiles alone give every CU a block, and the splits' partials, written and
// read back, are what is left to save.
template <int BM, int NWN, int XST, int WST, bool SHRINK, bool WALK>
__global__ __launch_bounds__(256 * NWN) void gemm_skinny_kernel(SkinnyArgs a) {
  // loader waves: half for each operand, except 192 columns (12 waves), whose
  // activation rows need a power-of-two share (8 activation, 4 weight)
  constexpr int BN = 64 * NWN, FM = BM / 64, NW = 4 * NWN, XW = NWN == 3 ? 8 : NW / 2, WW = NW - XW;
  constexpr int SA = BM * SBK, SB = BN * SBK;
  constexpr int XR = BM / (8 * XW), WR = BN / (8 * WW);    // 1 KB rounds per stage and loader wave
  static_assert(XR * 8 * XW == BM && WR * 8 * WW == BN, "loader rounds");
  static_assert(XST >= 2 && WST >= 2, "stages");
  __shared__ __attribute__((aligned(16))) bf16 smem[XST * SA + WST * SB];
  // wave index in an SGPR, so the loader roles below are scalar branches
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave & 3, wn = wave >> 2;
  if constexpr (SHRINK) {
    // the first nsh blocks (a multiple of 8) run the split shrink of the same X
    if ((int)blockIdx.x < a.nsh) {
      if (blockIdx.y == 0) shrink_split_item(a.pl, a.sh, blockIdx.x * NW + wave, lane);
      return;
    }
  }
  const int nsh = SHRINK ? a.nsh : 0;
  const int ntn = (a.N + BN - 1) / BN;
  // consecutive blocks land on one XCD (the dispatcher deals block ids out
  // to the 8 XCDs in turn), so the blocks of one K split share that XCD's
  // L2 copy of the split's activation columns; the grid is padded to a
  // multiple of 8 and the padding blocks leave at once
  const int bx = (blockIdx.x & 7) * ((gridDim.x - nsh) >> 3) + ((blockIdx.x - nsh) >> 3);
  // WALK: the row tiles of a column tile follow each other (one XCD's L2 then
  // serves the weights to all but the first)
  const int ntm = WALK ? (a.M + BM - 1) / BM : 1;
  if (bx >= ntn * (WALK ? ntm : a.nsplit)) return;
  const int tn = WALK ? bx / ntm : bx % ntn, split = WALK ? 0 : bx / ntn;
  const int m0 = (WALK ? bx % ntm : (int)blockIdx.y) * BM, n0 = tn * BN;
  const int nkt = a.K / SBK;
  const int kt0 = WALK ? 0 : (int)((int64_t)split * nkt / a.nsplit);
  const int kt1 = WALK ? nkt : (int)((int64_t)(split + 1) * nkt / a.nsplit);
  const int nk = kt1 - kt0;

  // loader rows: wave lw of its operand fills rows lw * 8 + (lane >> 3) +
  // 8 * (loader waves) * i; the swizzle is applied on the global side, so
  // lane l writes chunk (l & 7) of its row (the chunk permutation is the
  // same for every round because 4 * loader waves is a multiple of 8)
  const bool xload = wave < XW;
  const int lw = xload ? wave : wave - XW;
  const int row0 = lw * 8 + (lane >> 3);
  const int kc0 = (lane & 7) ^ ((row0 >> 1) & 7);
  constexpr int MR = XR > WR ? XR : WR;
  const bf16* src[MR];
  if (xload) {
#pragma unroll
    for (int i = 0; i < XR; ++i)
      src[i] = (const bf16*)a.X + (int64_t)min(m0 + row0 + i * 8 * XW, a.M - 1) * a.ldx + kt0 * SBK + kc0 * 8;
  } else {
#pragma unroll
    for (int i = 0; i < WR; ++i) {
      const int n = min(n0 + row0 + i * 8 * WW, a.N - 1);
      const bool hi = a.W2 != nullptr && n >= a.n_half;
      src[i] = (const bf16*)(hi ? a.W2 : a.W) + (int64_t)(hi ? n - a.n_half : n) * a.K + kt0 * SBK + kc0 * 8;
    }
  }
  bf16* const Xs = smem;
  bf16* const Ws = smem + XST * SA;
  auto issue_x = [&](int j, int slot) {   // step j of the block's K range
#pragma unroll
    for (int i = 0; i < XR; ++i)
      __builtin_amdgcn_global_load_lds((gptr_t)(src[i] + j * SBK),
                                       (lptr_t)(Xs + slot * SA + (i * XW + lw) * 512), 16, 0, 0);
  };
  // the weights are read once per forward: nontemporal (cache policy 2, nt)
  auto issue_w = [&](int j, int slot) {
#pragma unroll
    for (int i = 0; i < WR; ++i)
      __builtin_amdgcn_global_load_lds((gptr_t)(src[i] + j * SBK),
                                       (lptr_t)(Ws + slot * SB + (i * WW + lw) * 512), 16, 0, 2);
  };

  f32x4 acc[FM][4];
#pragma unroll
  for (int mi = 0; mi < FM; ++mi)
#pragma unroll
    for (int ni = 0; ni < 4; ++ni) acc[mi][ni] = f32x4{0.f, 0.f, 0.f, 0.f};
  f32x4 tot[WALK ? FM : 1][WALK ? 4 : 1];
  int sp = 1, next = WALK ? nkt / a.nsplit : 0;   // the split after the current one, and where it starts
  bool first = true;
  if (nk > 0) {
    if (xload) {
#pragma unroll
      for (int j = 0; j < XST - 1; ++j)
        if (j < nk) issue_x(j, j);
    } else {
#pragma unroll
      for (int j = 0; j < WST - 1; ++j)
        if (j < nk) issue_w(j, j);
    }
    int xs = 0, ws = 0;                           // stages of step j
    for (int j = 0; j < nk; ++j) {
      // this wave's loads of step j have landed, up to XST - 2 (WST - 2) newer
      // steps are in flight
      if (xload) wait_newer<XR, XST - 2>(min(nk - 1 - j, XST - 2));
      else wait_newer<WR, WST - 2>(min(nk - 1 - j, WST - 2));
      __builtin_amdgcn_s_barrier();
      // every wave is past step j - 1, whose X stage and W stage are free
      if (xload) {
        if (j + XST - 1 < nk) issue_x(j + XST - 1, xs == 0 ? XST - 1 : xs - 1);
      } else {
        if (j + WST - 1 < nk) issue_w(j + WST - 1, ws == 0 ? WST - 1 : ws - 1);
      }
      const bf16* As = Xs + xs * SA;
      const bf16* Bs = Ws + ws * SB;
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
        const int kc = kk * 4 + (lane >> 4);
        bf16x8 wf[4], xf[FM];
#pragma unroll
        for (int ni = 0; ni < 4; ++ni) {
          const int r = wn * 64 + ni * 16 + (lane & 15);
          wf[ni] = *reinterpret_cast<const bf16x8*>(Bs + r * SBK + swz(r, kc) * 8);
        }
#pragma unroll
        for (int mi = 0; mi < FM; ++mi) {
          const int r = wm * 16 * FM + mi * 16 + (lane & 15);
          xf[mi] = *reinterpret_cast<const bf16x8*>(As + r * SBK + swz(r, kc) * 8);
        }
#pragma unroll
        for (int mi = 0; mi < FM; ++mi)
#pragma unroll
          for (int ni = 0; ni < 4; ++ni) acc[mi][ni] = mfma16(wf[ni], xf[mi], acc[mi][ni]);
      }
      xs = xs == XST - 1 ? 0 : xs + 1;
      ws = ws == WST - 1 ? 0 : ws + 1;
      if constexpr (WALK) {
        if (j + 1 == next) {                        // block-uniform: the end of a split
#pragma unroll
          for (int mi = 0; mi < FM; ++mi)
#pragma unroll
            for (int ni = 0; ni < 4; ++ni) {
              tot[mi][ni] = first ? acc[mi][ni] : tot[mi][ni] + acc[mi][ni];
              acc[mi][ni] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
          first = false;
          ++sp;
          next = (int)((int64_t)sp * nkt / a.nsplit);
        }
      }
    }
  }
  // lane holds D[n = 4 * (lane >> 4) + i][m = lane & 15] of each 16 x 16 block
  float* Zs = a.Z + (int64_t)split * a.M * a.N;
#pragma unroll
  for (int mi = 0; mi < FM; ++mi) {
    const int m = m0 + wm * 16 * FM + mi * 16 + (lane & 15);
    if (m >= a.M) continue;
#pragma unroll
    for (int ni = 0; ni < 4; ++ni) {
      const int n = n0 + wn * 64 + ni * 16 + 4 * (lane >> 4);
      if (n >= a.N) continue;
      f32x4 v = acc[mi][ni];
      if constexpr (WALK) v = tot[mi][ni];
      *reinterpret_cast<float4*>(Zs + (int64_t)m * a.N + n) = make_float4(v[0], v[1], v[2], v[3]);
    }
  }
}

// ---------------------------------------------------------------------------
// Finalize: sum of the partial slices (fixed order) + the row's LoRA
// difference (fin_lora_delta, from the split shrink's partials) + bias +
// epilogue.  Block (column range, row): the row's U is rebuilt once in LDS,
// then each thread takes 4 output columns; every load is independent of the
// others, so the kernel streams the partials.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void finalize_kernel(FinalizeArgs a) {
  __shared__ float Us[3 * VFM_MAX_RANK], red[256];
  __shared__ __attribute__((aligned(16))) float cols[4][256];
  __shared__ float rcs[64], rsn[64];          // the row's rotary angles (head_dim / 2 <= 64)
  // Block b takes (column block, row) number (b % 8) * per + b / 8, rows
  // fastest: consecutive blocks of one XCD (one L2) take consecutive rows of
  // one column block, so a task's B rows, read again for its next rows, come
  // from that XCD's L2 instead of beyond it.
  const int ncb = (a.N / 4 + 255) / 256;
  const int per = gridDim.x / 8;
  const int lid = (blockIdx.x % 8) * per + blockIdx.x / 8;
  if (lid >= ncb * a.M) return;               // block-uniform
  const int m = lid % a.M, cb = lid / a.M;
  int t = 0, r = 0;
  FinB bp = {};
  if (a.lora.enabled) {                       // block-uniform
    t = a.lora.row_task[m];
    bp = fin_lora_bptrs(a.lora, t);
    r = fin_lora_u(a.lora, m, Us, red);
  }
  if (a.rope.on) {                            // block-uniform: the row's angles, as launch_rope
    const int half = a.rope.head_dim >> 1;
    if (threadIdx.x < half) {
      const float inv = exp2f(-(2.0f * (float)threadIdx.x / (float)a.rope.head_dim) * a.rope.log2_theta);
      float sn, cs;
      sincosf((float)a.rope.pl.pos[m] * inv, &sn, &cs);
      rcs[threadIdx.x] = cs;
      rsn[threadIdx.x] = sn;
    }
    __syncthreads();
  }
  const int n = (cb * 256 + threadIdx.x) * 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), first = cb * 1024 + wave * 256;
  if (first >= a.N) return;                   // wave-uniform; lanes past N leave after the LoRA sums
  const bool swiglu = a.epi == EPI_SWIGLU;
  const int nz = swiglu ? 2 * a.N : a.N;   // columns of Z
  const int64_t zs = (int64_t)a.M * nz;
  const float* z = a.Z + (int64_t)m * nz + min(n, a.N - 4);
  float4 v = sum_slices(z, zs, a.nslices), u = make_float4(0.f, 0.f, 0.f, 0.f);
  if (swiglu) u = sum_slices(z + a.N, zs, a.nslices);
  if (a.lora.enabled) {
    add4(v, fin_lora_wave(a.lora, bp, r, swiglu ? 0 : -1, first, a.N, Us, cols[wave]));
    if (swiglu) add4(u, fin_lora_wave(a.lora, bp, r, 1, first, a.N, Us, cols[wave]));
  }
  if (n >= a.N) return;
  if (a.bias && !swiglu) {
    const bf16x4 bv = *reinterpret_cast<const bf16x4*>((const bf16*)a.bias + n);
    v.x += (float)bv[0]; v.y += (float)bv[1]; v.z += (float)bv[2]; v.w += (float)bv[3];
  }
  if (a.epi == EPI_RESID) {
    float4* xo = reinterpret_cast<float4*>((float*)a.out + (int64_t)m * a.ldo + n);
    float4 xv = *xo;
    add4(xv, v);
    *xo = xv;
    return;
  }
  if (a.rope.on && n < 2 * a.rope.d) {        // q and k columns (whole waves: d % 256 == 0)
    // rotate-half: column i of a head pairs with column i + head_dim / 2,
    // held head_dim / 8 lanes away (4 columns per lane)
    const int dh = a.rope.head_dim, half = dh >> 1;
    const int cin = n % dh;
    float4 pv;
    pv.x = __shfl_xor(v.x, dh / 8, 64);
    pv.y = __shfl_xor(v.y, dh / 8, 64);
    pv.z = __shfl_xor(v.z, dh / 8, 64);
    pv.w = __shfl_xor(v.w, dh / 8, 64);
    const bool second = cin >= half;
    const int i0 = second ? cin - half : cin;
    float x4[4] = {v.x, v.y, v.z, v.w};
    const float p4[4] = {pv.x, pv.y, pv.z, pv.w};
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const float cs = rcs[i0 + c], sn = rsn[i0 + c];
      x4[c] = second ? p4[c] * sn + x4[c] * cs : x4[c] * cs - p4[c] * sn;
    }
    v = make_float4(x4[0], x4[1], x4[2], x4[3]);
  }
  const float g4[4] = {v.x, v.y, v.z, v.w};
  const float u4[4] = {u.x, u.y, u.z, u.w};
  bf16x4 o;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    float y = g4[c];
    if (swiglu) y = silu_fast(y) * u4[c];
    else if (a.epi == EPI_GELU) y = gelu_fast(y);
    o[c] = (bf16)y;
  }
  *reinterpret_cast<bf16x4*>((bf16*)a.out + (int64_t)m * a.ldo + n) = o;
  if (a.rope.on && a.rope.kc != nullptr && n >= a.rope.d) {   // the row's k (rotated) and v to its slot
    const int dd = a.rope.d, dh = a.rope.head_dim;
    const bool isv = n >= 2 * dd;
    const int cc = isv ? n - 2 * dd : n - dd;
    const int hh = cc / dh;
    const int64_t slot = kv_slot(a.rope.pl, a.rope.kp, a.rope.pl.row_req[m], a.rope.pl.pos[m]);
    bf16* dst = (isv ? a.rope.vc : a.rope.kc) + ((int64_t)hh * a.rope.kv_slots + slot) * dh + (cc - hh * dh);
    *reinterpret_cast<bf16x4*>(dst) = o;
  }
}

// Column-tile width and K split of the small-batch GEMM for an N x K
// weight: for each tile width (128, 192, 256 columns) K is split until one
// row tile fills the chip once (one block per CU), at most 6 ways for wide
// weights (N >= 8192) so the fp32 partials stay below the weight bytes; the
// width whose blocks each stream the fewest weight bytes wins (the 7B
// gate/up weight: 230 blocks of 192 columns instead of 172 of 256).  The
// split depends on the weight shape only, never on the batch, so a row's
// result does not depend on the other rows.
void skinny_shape(int N, int K, int* bn, int* nsplit) {
  const int nkt = K / SBK;
  const bool wide = N >= 8192;
  const int cap = wide ? 6 : 16;
  // the tile width whose one round of blocks streams the fewest weight
  // steps per block (rounds x width x K steps of a split); ties go to fewer
  // splits (fewer partial bytes)
  long best = -1;
  for (const int b : {128, 192, 256}) {
    const int tiles = (N + b - 1) / b;
    const int ns = std::max(1, std::min(std::min(256 / tiles, cap), nkt));
    const long rounds = ((long)tiles * ns + 255) / 256;
    const long cost = rounds * b * ((nkt + ns - 1) / ns);
    if (best < 0 || cost < best || (cost == best && ns < *nsplit)) {
      best = cost;
      *bn = b;
      *nsplit = ns;
    }
  }
}

// The walking launch's tile for an M-row batch, or bm 0 for the split launch:
// the faster one by an estimate (us) fitted on 200 to 1000 rows of the 7B
// decoder's weights.  A block's K step takes what its waves need from barrier
// to barrier, whatever the depth of the rings; one block per CU runs at a
// time.  The split launch also writes and reads back nsplit - 1 more slices of
// 4 M N bytes.  Layers of other widths, 257 / 400 / 640 / 1000 rows, split against
// the rule: 1024 wide 155.9 / 173.0 / 232.3 / 311.4 -> 114.2 / 118.8 / 135.6 /
// 157.4 us (its other projections direct), 2048 wide 217 / 254 / 346 / 493 -> 186 /
// 213 / 261 / 319, 8192 wide 1307 / 1426 / 2110 / 2904 -> 1197 / 1326 / 1855 / 2631;
// none of 28 (1024 to 8192 wide, decoders and encoders) is slower.  333 rows:
// QKV 65.0 -> 55.9 us as 128 x 192, gate+up 105.2 ->
// 71.4 as 192 x 192, the finalizes 36.2 / 42.4 -> 28.6 / 35.0; O and down stay
// split (33.3, 66.4 against 44.1, 108.4).  1000 rows: QKV 135.8 -> 94.9, gate+up
// 210.2 -> 178.1, O 65.7 -> 49.6, down 131.6 -> 119.0.
struct Walk { int bm, bn; };
Walk skinny_walk(int M, int N, int K, int split_bn, int nsplit) {
  Walk best = {0, 0};
  // one row tile of the split launch: its weights are read once, and the walk
  // was slower (130 / 192 / 256 rows of 7B decode 302 / 345 / 393 us a layer
  // walked, 291 / 338 / 387 split)
  if (M <= 256 || nsplit < 2) return best;
  const double nkt = K / SBK;
  const double step = split_bn == 128 ? 1.2 : split_bn == 192 ? 1.55 : 1.9;
  const int blocks = (N + split_bn - 1) / split_bn * nsplit * ((M + 255) / 256);
  double cost = (blocks + 255) / 256 * (nkt / nsplit * step + 7.0) + (nsplit - 1) * 4e-6 * M * N / 6.6;
  constexpr struct { int bm, bn; double step; } cand[4] = {
      {128, 128, 0.62}, {128, 192, 0.78}, {192, 192, 1.0}, {256, 192, 1.32}};
  for (const auto& c : cand) {
    const int tiles = (N + c.bn - 1) / c.bn * ((M + c.bm - 1) / c.bm);
    const double t = (tiles + 255) / 256 * (nkt * c.step + 6.0);
    if (t < cost) { cost = t; best = {c.bm, c.bn}; }
  }
  return best;
}

}  // namespace

int skinny_splits(int N, int K) {
  int bn, ns;
  skinny_shape(N, K, &bn, &ns);
  return ns;
}

hipError_t launch_gemm_skinny(const SkinnyArgs& a0, hipStream_t s) {
  if (a0.M == 0) return hipSuccess;
  SkinnyArgs a = a0;
  int bn;
  skinny_shape(a.N, a.K, &bn, &a.nsplit);
  // up to 64 rows: 128-column blocks of 80 KB of LDS, two per CU, whatever
  // the width the split was chosen for (the split alone fixes the sums), and
  // the shrink's blocks beside them: one 7B decode row, shrink + GEMM of QKV /
  // O / gate+up / down 23.6 / 13.5 / 34.7 / 25.5 us in launches of their own,
  // 19.5 / 9.8 / 32.8 / 20.2 us together.  At 100 rows (60 tasks) the shrink's
  // blocks hold up the GEMM's by what their launch costs: kept apart there.
  const int bm = a.M <= 64 ? 64 : a.M <= 128 ? 128 : 256;
  if (bm == 64) bn = 128;
  const int ntn = (a.N + bn - 1) / bn;
  a.nsh = a.sh.n_proj > 0 ? ((a.pl.n_rtiles * a.sh.kchunks * a.sh.n_proj + 7) / 8 + 7) & ~7 : 0;
  if (a.nsh > 0 && bm != 64) return hipErrorInvalidValue;
  dim3 grid(((ntn * a.nsplit + 7) & ~7) + a.nsh, (a.M + bm - 1) / bm);
  const Walk wk = skinny_walk(a.M, a.N, a.K, bn, a.nsplit);
  if (wk.bm > 0) {
    const int tiles = (a.N + wk.bn - 1) / wk.bn * ((a.M + wk.bm - 1) / wk.bm);
    const dim3 g((tiles + 7) & ~7);
    if (wk.bm == 256) hipLaunchKernelGGL((gemm_skinny_kernel<256, 3, 2, 4, false, true>), g, dim3(768), 0, s, a);
    else if (wk.bm == 192) hipLaunchKernelGGL((gemm_skinny_kernel<192, 3, 3, 3, false, true>), g, dim3(768), 0, s, a);
    else if (wk.bn == 192) hipLaunchKernelGGL((gemm_skinny_kernel<128, 3, 4, 4, false, true>), g, dim3(768), 0, s, a);
    else hipLaunchKernelGGL((gemm_skinny_kernel<128, 2, 4, 4, false, true>), g, dim3(512), 0, s, a);
    return hipGetLastError();
  }
#define VFM_SK(BM_)                                                                                           \
  do {                                                                                                        \
    if (bn == 128) hipLaunchKernelGGL((gemm_skinny_kernel<BM_, 2, BM_ == 256 ? 3 : 4, 4, false, false>), grid, dim3(512), 0, s, a); \
    else if (bn == 192) hipLaunchKernelGGL((gemm_skinny_kernel<BM_, 3, BM_ == 256 ? 2 : 4, 4, false, false>), grid, dim3(768), 0, s, a); \
    else hipLaunchKernelGGL((gemm_skinny_kernel<BM_, 4, 2, 3, false, false>), grid, dim3(1024), 0, s, a);        \
  } while (0)
  if (bm == 64) hipLaunchKernelGGL((gemm_skinny_kernel<64, 2, 4, 3, true, false>), grid, dim3(512), 0, s, a);
  else if (bm == 128) VFM_SK(128);
  else VFM_SK(256);
#undef VFM_SK
  return hipGetLastError();
}

int skinny_slices(int M, int N, int K) {
  int bn, ns;
  skinny_shape(N, K, &bn, &ns);
  return skinny_walk(M, N, K, bn, ns).bm > 0 ? 1 : ns;
}

// K chunks of the split shrink: fixed 256-column chunks (the last one
// ragged), independent of the batch for the same reason as the GEMM split.
int shrink_chunks(int K) { return (K + SHRINK_CHUNK - 1) / SHRINK_CHUNK; }

hipError_t launch_shrink_split(const Plan& pl, const ShrinkSplitArgs& a0, hipStream_t s) {
  if (pl.n_rtiles == 0 || a0.n_proj == 0) return hipSuccess;
  const ShrinkSplitArgs& a = a0;
  dim3 grid(pl.n_rtiles, a.kchunks);
#define VFM_SS(NP_, NS_) hipLaunchKernelGGL((shrink_split_kernel<NP_, NS_>), grid, dim3(256), 0, s, pl, a)
  // only the sub-tiles the table's largest rank reaches: 1 (rank <= 16), 2 (<= 32) or 4
#define VFM_SS_NP(NS_) do { if (a.n_proj == 1) VFM_SS(1, NS_); else if (a.n_proj == 2) VFM_SS(2, NS_); else VFM_SS(3, NS_); } while (0)
  if (a.nsub <= 1) VFM_SS_NP(1);
  else if (a.nsub == 2) VFM_SS_NP(2);
  else VFM_SS_NP(4);
#undef VFM_SS_NP
#undef VFM_SS
  return hipGetLastError();
}

hipError_t launch_finalize(const FinalizeArgs& a, hipStream_t s) {
  if (a.M == 0 || a.N == 0) return hipSuccess;
  const int ncb = (a.N / 4 + 255) / 256;
  hipLaunchKernelGGL(finalize_kernel, dim3(((int64_t)ncb * a.M + 7) / 8 * 8), dim3(256), 0, s, a);
  return hipGetLastError();
}
