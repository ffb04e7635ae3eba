// Shared projections (a3, a7, a9, a10): ONE GEMM over every row of the mixed
// batch, C[m, n] = sum_k X[m, k] W[n, k], with the per-task LoRA expand fused
// in as extra MFMA steps and the bias / activation / residual fused into the
// epilogue.
//
// The paper batches all requests through the shared backbone and then adds
// each adapter's difference on its own requests (Section 4.2, adapter
// handling; Fig. 5 (c)).  Here the difference is not a second pass over the
// output: rows are sorted by task, so a tile's rows form runs of one task
// each, and after the K loop the tile runs more MFMA steps whose operands are
// U (the per-row shrink output s_t x A_t^T) and B_t (the task's expand factor,
// read straight from its device pointer), each run meeting its own factor.
// The sum is exactly x W^T + s_t (x A_t^T) B_t^T per row.
//
// bf16 path (gfx950): v_mfma_f32_16x16x32_bf16 on LDS tiles fed by
// global_load_lds (gemm_tile.inc): 256-row tiles of 8 waves, or 64- and
// 128-row ones of 4 where those cannot fill the chip, with an XOR swizzle so
// that the 16-byte fragment reads are bank-conflict free.  The weight tile
// feeds the MFMA A slot and the activation tile the B slot, so each lane ends
// up with 4 consecutive output columns of one row.  Their offsets inside an
// operand are 32-bit: operands of 2^31 elements or more take a
// register-staged kernel (gemm_bf16_kernel).
//
// fp32 path: fp32 MFMA with small tiles and K split over a block's waves
// (gemm_f32_kernel), the same epilogues.
#include <algorithm>
#include <type_traits>

#include "vfm_internal.h"

namespace {

constexpr int BM = 128, BN = 128, BK = 64;

// LDS chunk swizzle of a [rows][64 bf16] tile (128-byte rows, eight 16-byte
// chunks): logical chunk kc of row r lives at physical chunk kc ^ ((r >> 1) & 7).
// Measured on gfx950 with the LDS bank-conflict counter: zero conflicts for
// the ds_read_b128 fragment reads of both the 16x16 and the 32x32 MFMA
// operand layouts (rows r..r+15 at one logical chunk).
__device__ __forceinline__ int swz_bits(int row) { return (row >> 1) & 7; }
__device__ __forceinline__ int swz(int row, int kc) { return kc ^ swz_bits(row); }

__device__ __forceinline__ float gelu_erf(float v) {
  return 0.5f * v * (1.f + erff(v * 0.70710678118654752440f));
}
__device__ __forceinline__ float silu_exact(float v) { return v / (1.f + expf(-v)); }  // fp32 outputs

__device__ __forceinline__ f32x4 mfma16(const bf16x8& a, const bf16x8& b, const f32x4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

typedef const void __attribute__((address_space(1)))* gptr_t;
typedef void __attribute__((address_space(3)))* lptr_t;

// Per-task LoRA expand for one wave's FM x FN fragment grid, a task at a time,
// each task's sums going to its own rows only.  wrow0 / wcol0: the wave's
// first row / first B-tile row.
template <int FM, int FN, bool SWIGLU>
__device__ __forceinline__ void lora_expand_frags(const GemmArgs& a, int m0, int BMrows, int wrow0,
                                                  int n0, int wcol0, int lane,
                                                  f32x4 (&acc)[FM][FN]) {
  const GemmLora& L = a.lora;
  const bf16* U = (const bf16*)L.U;
  const int mlast = min(m0 + BMrows, a.M) - 1;
  const int t0 = L.row_task[m0], t1 = L.row_task[mlast];
  for (int t = t0; t <= t1; ++t) {
    const int r = min(L.rank[t], L.max_rank) & ~7;
    if (r <= 0) continue;
    const int s0 = L.seg_row[t], s1 = L.seg_row[t + 1];
    if (s0 >= s1 || s1 <= wrow0 || s0 >= wrow0 + FM * 16) continue;   // no rows here
    for (int kk = 0; kk < r; kk += 32) {
      const int kof = kk + 8 * (lane >> 4);
      const bool kin = kof < r;
      bf16x8 xf[FM];
#pragma unroll
      for (int mi = 0; mi < FM; ++mi) xf[mi] = bf16x8{};
#pragma unroll
      for (int ni = 0; ni < FN; ++ni) {
        int slot, nrow, nlim;
        if (SWIGLU) {
          const int sub = wcol0 / 16 + ni;
          slot = sub & 1;
          const int jb = n0 + (sub >> 1) * 16;
          if (jb >= a.N) continue;
          nrow = jb + (lane & 15);
          nlim = a.N;
        } else {
          const int nb = n0 + wcol0 + ni * 16;
          if (nb >= a.N) continue;
          slot = nb / L.slot_width;
          nrow = nb - slot * L.slot_width + (lane & 15);
          nlim = L.slot_width;
        }
        if (L.B[slot] == nullptr || L.B[slot][t] == nullptr) continue;   // no adapters, or none of this task
        // a pointer from the table: read as global memory, not through flat addressing
        typedef const bf16 __attribute__((address_space(1)))* growp;
        const growp Bt = (growp)L.B[slot][t];
        bf16x8 wf = {};
        if (kin && nrow < nlim) wf = *(const bf16x8 __attribute__((address_space(1)))*)(Bt + (int64_t)nrow * r + kof);
#pragma unroll
        for (int mi = 0; mi < FM; ++mi) {
          const int m = wrow0 + mi * 16 + (lane & 15);
          const bool own = m >= s0 && m < s1;
          bf16x8 x = {};
          if (own && m < a.M) x = *reinterpret_cast<const bf16x8*>(U + (int64_t)m * L.ldu + L.ucol[slot] + kof);
          const f32x4 v = mfma16(wf, x, acc[mi][ni]);
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[mi][ni][e] = own ? v[e] : acc[mi][ni][e];
        }
      }
    }
  }
}

// The backbone sums of one wave's fragment grid, operands read straight from
// global memory: the K steps of the tile kernels in their order.
template <int FM, int FN, bool SWIGLU>
__device__ __forceinline__ void backbone_frags(const GemmArgs& a, int wrow0, int n0, int wcol0, int lane,
                                               f32x4 (&acc)[FM][FN]) {
#pragma unroll
  for (int mi = 0; mi < FM; ++mi)
#pragma unroll
    for (int ni = 0; ni < FN; ++ni) acc[mi][ni] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int x = lane & 15;
#pragma unroll 1
  for (int k = 8 * (lane >> 4); k < a.K; k += 32) {
    bf16x8 wf[FN], xf[FM];
#pragma unroll
    for (int ni = 0; ni < FN; ++ni) {
      const int sub = wcol0 / 16 + ni;               // SwiGLU: gate and up rows alternate by 16
      const int row = SWIGLU ? n0 + (sub >> 1) * 16 + x : n0 + wcol0 + ni * 16 + x;
      const bf16* W = (const bf16*)(SWIGLU && (sub & 1) ? a.W2 : a.W);
      wf[ni] = *reinterpret_cast<const bf16x8*>(W + (int64_t)min(row, a.N - 1) * a.K + k);
    }
#pragma unroll
    for (int mi = 0; mi < FM; ++mi)
      xf[mi] = *reinterpret_cast<const bf16x8*>((const bf16*)a.X + (int64_t)min(wrow0 + mi * 16 + x, a.M - 1) * a.ldx + k);
#pragma unroll
    for (int mi = 0; mi < FM; ++mi)
#pragma unroll
      for (int ni = 0; ni < FN; ++ni) acc[mi][ni] = mfma16(wf[ni], xf[mi], acc[mi][ni]);
  }
}

// Epilogue for one wave's FM x FN fragment grid; lane holds 4 consecutive
// output columns of one row per fragment.  Bias is read once per column
// group and the residual loads of a row group are issued together, so the
// global-memory latency is paid FM times, not FM x FN times.
template <int EPI, bool SWIGLU, int FM, int FN>
__device__ __forceinline__ void epilogue_frags(const GemmArgs& a, int wrow0, int n0, int wcol0,
                                               int lane, const f32x4 (&acc)[FM][FN]) {
  if (SWIGLU) {
#pragma unroll
    for (int mi = 0; mi < FM; ++mi) {
      const int m = wrow0 + mi * 16 + (lane & 15);
      if (m >= a.M) continue;
#pragma unroll
      for (int ni = 0; ni < FN; ni += 2) {
        const int sub = wcol0 / 16 + ni;
        const int j = n0 + (sub >> 1) * 16 + 4 * (lane >> 4);
        if (j >= a.N) continue;
        bf16x4 o;
#pragma unroll
        for (int r = 0; r < 4; ++r) o[r] = (bf16)(silu_fast(acc[mi][ni][r]) * acc[mi][ni + 1][r]);
        *reinterpret_cast<bf16x4*>((bf16*)a.out + (int64_t)m * a.ldo + j) = o;
      }
    }
    return;
  }
  const bf16* bias = (const bf16*)a.bias;
  f32x4 bv[FN];
#pragma unroll
  for (int ni = 0; ni < FN; ++ni) {
    bv[ni] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int n = n0 + wcol0 + ni * 16 + 4 * (lane >> 4);
    if (bias && n < a.N) {
      const bf16x4 bb = *reinterpret_cast<const bf16x4*>(bias + n);
#pragma unroll
      for (int r = 0; r < 4; ++r) bv[ni][r] = (float)bb[r];
    }
  }
#pragma unroll
  for (int mi = 0; mi < FM; ++mi) {
    const int m = wrow0 + mi * 16 + (lane & 15);
    if (m >= a.M) continue;
    if (EPI == EPI_RESID) {
      float* row = (float*)a.out + (int64_t)m * a.ldo;
      float4 old[FN];
#pragma unroll
      for (int ni = 0; ni < FN; ++ni) {
        const int n = n0 + wcol0 + ni * 16 + 4 * (lane >> 4);
        old[ni] = n < a.N ? *reinterpret_cast<const float4*>(row + n) : make_float4(0.f, 0.f, 0.f, 0.f);
      }
#pragma unroll
      for (int ni = 0; ni < FN; ++ni) {
        const int n = n0 + wcol0 + ni * 16 + 4 * (lane >> 4);
        if (n >= a.N) continue;
        float4 o = old[ni];
        o.x += acc[mi][ni][0] + bv[ni][0];
        o.y += acc[mi][ni][1] + bv[ni][1];
        o.z += acc[mi][ni][2] + bv[ni][2];
        o.w += acc[mi][ni][3] + bv[ni][3];
        *reinterpret_cast<float4*>(row + n) = o;
      }
    } else {
      bf16* row = (bf16*)a.out + (int64_t)m * a.ldo;
#pragma unroll
      for (int ni = 0; ni < FN; ++ni) {
        const int n = n0 + wcol0 + ni * 16 + 4 * (lane >> 4);
        if (n >= a.N) continue;
        bf16x4 o;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float v = acc[mi][ni][r] + bv[ni][r];
          o[r] = (bf16)(EPI == EPI_GELU ? gelu_fast(v) : v);
        }
        *reinterpret_cast<bf16x4*>(row + n) = o;
      }
    }
  }
}

// Epilogue of the large-M kernel through LDS.  The MFMA fragments leave each
// lane with 4 consecutive columns of 16 different rows, so direct stores are
// 16 row pieces of 32 B (bf16) or 64 B (fp32) per instruction.  Here the
// finished values (bias, activation applied) go into the idle operand LDS as
// a row-major tile first, and the block then writes whole rows, 16 B per lane
// with consecutive lanes on consecutive addresses.  16-byte chunk q of tile
// row r sits at chunk q ^ (r & S), S + 1 the largest power of two (at most 8)
// dividing the row's chunk count, which spreads the fragment writes of
// consecutive rows over distinct banks.  The fp32 residual tile (4 B per
// value) is done in two halves of rows.
template <int QR>
__device__ __forceinline__ int lds_chunk(int r, int q) {
  constexpr int LOW = QR & -QR, S = (LOW < 8 ? LOW : 8) - 1;
  return q ^ (r & S);
}

template <int EPI, bool SWIGLU, int BMT, int BNT, int WM, int NST, int FM, int FN>
__device__ __forceinline__ void epilogue_lds(const GemmArgs& a, char* lds, int m0, int n0, int wm, int wn,
                                             int lane, int tid, const f32x4 (&acc)[FM][FN], const float4* old) {
  constexpr int NTH = 128 * WM, TM = BMT / WM, TN = BNT / 2;
  constexpr int NC = SWIGLU ? BNT / 2 : BNT;        // output columns of the tile
  const int g = lane >> 4;
  __syncthreads();                                  // every wave is done with the operand stages
  if (EPI != EPI_RESID) {
    constexpr int QR = NC / 8;                      // 16-byte chunks per row (bf16)
    static_assert(QR % 4 == 0, "row chunks");
    static_assert(BMT * NC * 2 <= NST * (BMT + BNT) * BK * 2, "tile fits the operand LDS");
    bf16* T = reinterpret_cast<bf16*>(lds);
    if (SWIGLU) {
#pragma unroll
      for (int mi = 0; mi < FM; ++mi) {
        const int r = wm * TM + mi * 16 + (lane & 15);
#pragma unroll
        for (int ni = 0; ni < FN; ni += 2) {
          const int sub = wn * TN / 16 + ni;
          const int j = (sub >> 1) * 16 + 4 * g;     // tile column of the lane's 4 values
          bf16x4 o;
#pragma unroll
          for (int e = 0; e < 4; ++e) o[e] = (bf16)(silu_fast(acc[mi][ni][e]) * acc[mi][ni + 1][e]);
          *reinterpret_cast<bf16x4*>(T + r * NC + lds_chunk<QR>(r, j >> 3) * 8 + (j & 4)) = o;
        }
      }
    } else {
      const bf16* bias = (const bf16*)a.bias;
      f32x4 bv[FN];
#pragma unroll
      for (int ni = 0; ni < FN; ++ni) {
        bv[ni] = f32x4{0.f, 0.f, 0.f, 0.f};
        const int j = wn * TN + ni * 16 + 4 * g;
        if (bias && n0 + j < a.N) {
          const bf16x4 bb = *reinterpret_cast<const bf16x4*>(bias + n0 + j);
#pragma unroll
          for (int e = 0; e < 4; ++e) bv[ni][e] = (float)bb[e];
        }
      }
#pragma unroll
      for (int mi = 0; mi < FM; ++mi) {
        const int r = wm * TM + mi * 16 + (lane & 15);
        bf16* row = T + r * NC + (g & 1) * 4;
#pragma unroll
        for (int ni = 0; ni < FN; ++ni) {
          const int q = (wn * TN + ni * 16) / 8 + (g >> 1);   // 16-byte chunk of the lane's 4 values
          bf16x4 o;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float v = acc[mi][ni][e] + bv[ni][e];
            o[e] = (bf16)(EPI == EPI_GELU ? gelu_fast(v) : v);
          }
          *reinterpret_cast<bf16x4*>(row + lds_chunk<QR>(r, q) * 8) = o;
        }
      }
    }
    __syncthreads();
    bf16* out = (bf16*)a.out;
    if (EPI == EPI_STORE && !SWIGLU && a.rope.on && n0 < 2 * a.rope.d) {   // block-uniform
      // Rotary embedding of the q / k columns on the staged rows (the tile
      // holds whole heads): a thread takes 8 columns i .. i + 7 of a head's
      // first half and their partners i + head_dim / 2, rotates both in
      // fp32 and stores both.  The angle pos * theta^(-2i / head_dim), in
      // revolutions reduced to [0, 1), feeds the hardware sine and cosine.
      const int hc = a.rope.head_dim / 8;            // 16-byte chunks per head
      const int hh = hc / 2;
      const float l2t = a.rope.log2_theta, inv_hd = 2.0f / (float)a.rope.head_dim;
#pragma unroll 2
      for (int e = tid; e < BMT * (QR / 2); e += NTH) {
        const int r = e / (QR / 2), qq = e % (QR / 2);
        const int q1 = (qq / hh) * hc + qq % hh, q2 = q1 + hh;
        const int m = m0 + r;
        const bf16x8 v1 = *reinterpret_cast<const bf16x8*>(T + r * NC + lds_chunk<QR>(r, q1) * 8);
        const bf16x8 v2 = *reinterpret_cast<const bf16x8*>(T + r * NC + lds_chunk<QR>(r, q2) * 8);
        if (m >= a.M) continue;
        const float pf = (float)a.rope.pos[m];
        const int i0 = (qq % hh) * 8;                // frequency index of the first column
        bf16x8 o1, o2;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const float x = pf * (exp2f(-(float)(i0 + j) * inv_hd * l2t) * 0.15915494309189535f);
          const float fr = x - floorf(x);
          const float cs = __builtin_amdgcn_cosf(fr), sn = __builtin_amdgcn_sinf(fr);
          const float x1 = (float)v1[j], x2 = (float)v2[j];
          o1[j] = (bf16)(x1 * cs - x2 * sn);
          o2[j] = (bf16)(x2 * cs + x1 * sn);
        }
        bf16* orow = out + (int64_t)m * a.ldo + n0;
        *reinterpret_cast<bf16x8*>(orow + q1 * 8) = o1;
        *reinterpret_cast<bf16x8*>(orow + q2 * 8) = o2;
      }
      return;
    }
#pragma unroll 4
    for (int e = tid; e < BMT * QR; e += NTH) {
      const int r = e / QR, q = e % QR;
      const int m = m0 + r, n = n0 + q * 8;
      const bf16x8 v = *reinterpret_cast<const bf16x8*>(T + r * NC + lds_chunk<QR>(r, q) * 8);
      if (m < a.M && n < a.N) *reinterpret_cast<bf16x8*>(out + (int64_t)m * a.ldo + n) = v;
    }
    return;
  }
  // fp32 residual: x[m, n] += acc + bias, rows of each half staged as fp32
  constexpr int HR = BMT / 2;                       // rows per half
  constexpr int QR = NC / 4;                        // 16-byte chunks per row (fp32)
  static_assert(QR % 4 == 0, "row chunks");
  static_assert(HR * NC * 4 <= NST * (BMT + BNT) * BK * 2, "half tile fits the operand LDS");
  float* T = reinterpret_cast<float*>(lds);
  const bf16* bias = (const bf16*)a.bias;
  float* x = (float*)a.out;
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    if (wm / (WM / 2) == half) {                    // these waves own the half's rows
#pragma unroll
      for (int ni = 0; ni < FN; ++ni) {
        const int j = wn * TN + ni * 16 + 4 * g;
        float bv[4] = {0.f, 0.f, 0.f, 0.f};
        if (bias && n0 + j < a.N) {
          const bf16x4 bb = *reinterpret_cast<const bf16x4*>(bias + n0 + j);
#pragma unroll
          for (int e = 0; e < 4; ++e) bv[e] = (float)bb[e];
        }
#pragma unroll
        for (int mi = 0; mi < FM; ++mi) {
          const int r = wm % (WM / 2) * TM + mi * 16 + (lane & 15);   // row within the half
          const float4 o = make_float4(acc[mi][ni][0] + bv[0], acc[mi][ni][1] + bv[1],
                                       acc[mi][ni][2] + bv[2], acc[mi][ni][3] + bv[3]);
          *reinterpret_cast<float4*>(T + r * NC + lds_chunk<QR>(r, j >> 2) * 4) = o;
        }
      }
    }
    __syncthreads();
    constexpr int UNROLL = WM == 2 ? HR * QR / NTH : 4;   // `old` is indexed by constants
#pragma unroll UNROLL
    for (int e = tid; e < HR * QR; e += NTH) {
      const int r = e / QR, q = e % QR;
      const int m = m0 + half * HR + r, n = n0 + q * 4;
      if (m < a.M && n < a.N) {
        const float4 v = *reinterpret_cast<const float4*>(T + r * NC + lds_chunk<QR>(r, q) * 4);
        float4* dst = reinterpret_cast<float4*>(x + (int64_t)m * a.ldo + n);
        float4 o;
        if constexpr (WM == 2) o = old[(half * HR * QR + e - tid) / NTH];
        else o = *dst;
        o.x += v.x; o.y += v.y; o.z += v.z; o.w += v.w;
        *dst = o;
      }
    }
    if (half == 0) __syncthreads();                 // the second half reuses the buffer
  }
}

// ---------------------------------------------------------------------------
// Large-M bf16 GEMM: BMT x BNT x 64 block tile (256 rows, 128 / 192 / 256
// columns), 8 waves (4 along M x 2 along N) of (BMT/4) x (BNT/2), operands
// streamed global -> LDS with global_load_lds_dwordx4 (no staging registers),
// two LDS stages (up to 128 KB), and an XCD-aware tile order: consecutive
// block ids land on different XCDs (each with its own L2), so block b takes
// logical tile (b % 8) * per + b / 8 and logical tiles run in groups of LGM
// row-tiles sweeping all column tiles, keeping each XCD's X rows and W
// columns resident in its L2.  The launcher picks the tile shape per GEMM
// so that the last round of tiles fills the 256 CUs as far as possible.
//
// The per-task LoRA expand runs as extra 64-wide K steps of the same
// pipeline: for the tasks t with rows in the tile, the A tile holds the
// shrink outputs U[m, slot cols] of t's rows (rows of other tasks zero) and
// the B tile holds B_t[n, :r_t] (zero past the rank); with ranks <= 16 up to
// four tasks share a step, each in its own 16 columns (SwiGLU: two, 16 gate
// and 16 up columns each).  The MFMA loop cannot tell these steps from the
// backbone's.
// ---------------------------------------------------------------------------
constexpr int LGM = 4;


// wait until at most `later` steps of ND loads each are outstanding (MAX at
// most), and for this wave's LDS accesses
template <int ND, int MAX>
__device__ __forceinline__ void wait_steps(int later) {
  static_assert(ND * MAX < 64, "vmcnt field");
  if constexpr (MAX == 0) {
    __builtin_amdgcn_s_waitcnt(0x0070);
  } else {
    // vmcnt(MAX ND) (bits 3:0 and 15:14), lgkmcnt(0)
    if (later >= MAX) __builtin_amdgcn_s_waitcnt(0x0070 | (MAX * ND & 15) | ((MAX * ND >> 4) << 14));
    else wait_steps<ND, MAX - 1>(later);
  }
}

template <int EPI, bool SWIGLU, int BMT, int BNT, bool PACK>
__global__ __launch_bounds__(512, 1) void gemm_bf16_large_kernel(GemmArgs a) {
  constexpr int WM = 4, NST = 2;
#include "gemm_tile.inc"
}

// The same tile for products with too few 256-row tiles to fill the chip: 4
// waves, 64 x 64 outputs with 4 LDS stages (64 KB, 2 blocks per CU) or 128 x
// 64 with 2 (48 KB, 3 blocks per CU).  A 256-row tile is fed at ~25 bytes per
// clock and CU and idles the matrix units through its first loads and its
// stores; small tiles move more operand bytes per output but cover more CUs
// and overlap one block's stores with another's K loop.  1518 x 1024 outputs
// (48 tiles of 256 x 128): 24.7 -> 12.2 us at K = 1024, 49.0 -> 22.3 at K =
// 2816; 4728 x 768 at K = 3072: 55.4 -> 40.5.  More stages for 128 x 64 (3: 2
// blocks per CU), fewer for 64 x 64, and 64 x 128 or 128 x 128 tiles were
// slower or equal.  K steps and their order are those of the large tiles.
template <int EPI, bool SWIGLU, int BMT, int BNT, bool PACK>
__global__ __launch_bounds__(256, 2) void gemm_bf16_mid_kernel(GemmArgs a) {
  constexpr int WM = 2, NST = BMT == 64 ? 4 : 2;
#include "gemm_tile.inc"
}

// ---------------------------------------------------------------------------
// bf16 GEMM with 64-bit offsets (operands of 2^31 elements or more): 128x128x64,
// 4 waves of 64x64, register-staged LDS double buffer.
// ---------------------------------------------------------------------------
template <int EPI, bool SWIGLU>
__global__ __launch_bounds__(256, 2) void gemm_bf16_kernel(GemmArgs a) {
  __shared__ __attribute__((aligned(16))) bf16 As[2][BM * BK];
  __shared__ __attribute__((aligned(16))) bf16 Bs[2][BN * BK];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  constexpr int NT = SWIGLU ? BN / 2 : BN;  // output columns per block
  const int n_tiles_n = (a.N + NT - 1) / NT;
  const int tn = blockIdx.x % n_tiles_n, tm = blockIdx.x / n_tiles_n;
  const int m0 = tm * BM, n0 = tn * NT;
  const bf16* X = (const bf16*)a.X;
  const bf16* W = (const bf16*)a.W;
  const bf16* W2 = (const bf16*)a.W2;

  const bf16* xsrc[4];
  const bf16* wsrc[4];
  int lds_off[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int c = tid + 256 * i, row = c >> 3, kc = c & 7;
    const int m = min(m0 + row, a.M - 1);
    xsrc[i] = X + (int64_t)m * a.ldx + kc * 8;
    const bf16* wb = W;
    int wrow;
    if (SWIGLU) {
      const int sub = row >> 4;
      wb = (sub & 1) ? W2 : W;
      wrow = min(n0 + (sub >> 1) * 16 + (row & 15), a.N - 1);
    } else {
      wrow = min(n0 + row, a.N - 1);
    }
    wsrc[i] = wb + (int64_t)wrow * a.K + kc * 8;
    lds_off[i] = row * BK + swz(row, kc) * 8;
  }

  bf16x8 xr[4], wr[4];
  f32x4 acc[4][4];
#pragma unroll
  for (int mi = 0; mi < 4; ++mi)
#pragma unroll
    for (int ni = 0; ni < 4; ++ni) acc[mi][ni] = f32x4{0.f, 0.f, 0.f, 0.f};

  const int nk = a.K / BK;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    xr[i] = *reinterpret_cast<const bf16x8*>(xsrc[i]);
    wr[i] = *reinterpret_cast<const bf16x8*>(wsrc[i]);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    *reinterpret_cast<bf16x8*>(&As[0][lds_off[i]]) = xr[i];
    *reinterpret_cast<bf16x8*>(&Bs[0][lds_off[i]]) = wr[i];
  }
  __syncthreads();

  for (int kt = 0; kt < nk; ++kt) {
    const int st = kt & 1;
    if (kt + 1 < nk) {
      const int k0 = (kt + 1) * BK;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        xr[i] = *reinterpret_cast<const bf16x8*>(xsrc[i] + k0);
        wr[i] = *reinterpret_cast<const bf16x8*>(wsrc[i] + k0);
      }
    }
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      const int kc = kk * 4 + (lane >> 4);
      bf16x8 wf[4], xf[4];
#pragma unroll
      for (int ni = 0; ni < 4; ++ni) {
        const int r = wn * 64 + ni * 16 + (lane & 15);
        wf[ni] = *reinterpret_cast<const bf16x8*>(&Bs[st][r * BK + swz(r, kc) * 8]);
      }
#pragma unroll
      for (int mi = 0; mi < 4; ++mi) {
        const int r = wm * 64 + mi * 16 + (lane & 15);
        xf[mi] = *reinterpret_cast<const bf16x8*>(&As[st][r * BK + swz(r, kc) * 8]);
      }
#pragma unroll
      for (int mi = 0; mi < 4; ++mi)
#pragma unroll
        for (int ni = 0; ni < 4; ++ni) acc[mi][ni] = mfma16(wf[ni], xf[mi], acc[mi][ni]);
    }
    if (kt + 1 < nk) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        *reinterpret_cast<bf16x8*>(&As[st ^ 1][lds_off[i]]) = xr[i];
        *reinterpret_cast<bf16x8*>(&Bs[st ^ 1][lds_off[i]]) = wr[i];
      }
    }
    __syncthreads();
  }

  const int wrow0 = m0 + wm * 64;
  if (a.lora.enabled)
    lora_expand_frags<4, 4, SWIGLU>(a, m0, BM, wrow0, n0, wn * 64, lane, acc);
  epilogue_frags<EPI, SWIGLU, 4, 4>(a, wrow0, n0, wn * 64, lane, acc);
}

// ---------------------------------------------------------------------------
// fp32: v_mfma_f32_16x16x4_f32 (fp32 products and sums), (16 FM) x (16 FN)
// outputs per block, the block's 4 waves each taking a quarter of K and
// adding their sums in wave order through LDS.
//
// The fp32 batches are small (1024 rows of a 256-wide encoder: 0.13 - 0.54
// GFLOP a product), so the kernel is bound by the latency of its chain over
// K, not by the matrix units: small tiles and the K split give every CU
// blocks and shorten the chain fourfold, and operands go from global memory
// (L2) straight into registers with no barrier.  A lane's 16-byte load holds
// 4 consecutive k of one row; MFMA j of a 16-column step takes component j of
// both operands, i.e. the columns {4 g + j}, which only reorders the sum.
// 64x64 FMA tiles with two barriers per 16 columns took 39.5 / 18.9 / 23.2 /
// 63.2 us for that encoder's QKV / O / up / down, this kernel 14.0 / 5.5 /
// 14.0 / 11.5 us (60 TFLOP/s at 4096 rows).  A row's sums depend on K alone: the tile shape, chosen by the
// number of blocks, does not change them.
// ---------------------------------------------------------------------------
__device__ __forceinline__ f32x4 mfma_f32(float a, float b, const f32x4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// s_t (x A_t^T) B_t^T of row m, columns nrow .. nrow + 3 of one LoRA slot
__device__ __forceinline__ f32x4 lora_f32(const GemmLora& L, int slot, int m, int nrow) {
  f32x4 s = {0.f, 0.f, 0.f, 0.f};
  const int t = L.row_task[m];
  const int r = min(L.rank[t], L.max_rank) & ~7;
  if (r <= 0 || L.B[slot] == nullptr || L.B[slot][t] == nullptr) return s;
  // a pointer from the table: read as global memory, not through flat addressing
  typedef const float __attribute__((address_space(1)))* growp;
  typedef const f32x4 __attribute__((address_space(1)))* gvecp;
  const growp Bt = (growp)L.B[slot][t] + (int64_t)nrow * r;
  const float* u = (const float*)L.U + (int64_t)m * L.ldu + L.ucol[slot];
  for (int q = 0; q < r; q += 4) {
    const f32x4 uv = *reinterpret_cast<const f32x4*>(u + q);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const f32x4 bv = *(gvecp)(Bt + (int64_t)c * r + q);
#pragma unroll
      for (int e = 0; e < 4; ++e) s[c] = fmaf(uv[e], bv[e], s[c]);
    }
  }
  return s;
}

template <int EPI, bool SWIGLU, int FM, int FN>
__global__ __launch_bounds__(256) void gemm_f32_kernel(GemmArgs a) {
  constexpr int NWT = SWIGLU ? 2 : 1, NF = FM * FN;
  static_assert(NF % 4 == 0, "each wave finishes NF / 4 fragments");
  __shared__ f32x4 red[4][NWT][NF][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int ntn = (a.N + 16 * FN - 1) / (16 * FN);
  const int m0 = blockIdx.x / ntn * (16 * FM), n0 = blockIdx.x % ntn * (16 * FN);
  const int kq = a.K / 4, ko = wave * kq + 4 * (lane >> 4);      // K is a multiple of 64
  const float* xp[FM];
  const float* wp[NWT][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
    xp[i] = (const float*)a.X + (int64_t)min(m0 + 16 * i + (lane & 15), a.M - 1) * a.ldx + ko;
#pragma unroll
  for (int i = 0; i < FN; ++i) {
    const int64_t o = (int64_t)min(n0 + 16 * i + (lane & 15), a.N - 1) * a.K + ko;
    wp[0][i] = (const float*)a.W + o;
    if (SWIGLU) wp[NWT - 1][i] = (const float*)a.W2 + o;
  }
  f32x4 acc[NWT][FM][FN];
#pragma unroll
  for (int w = 0; w < NWT; ++w)
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j) acc[w][i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  f32x4 xv[2][FM], wv[2][NWT][FN];
  auto load = [&](int s, int k) {
#pragma unroll
    for (int i = 0; i < FM; ++i) xv[s][i] = *reinterpret_cast<const f32x4*>(xp[i] + k);
#pragma unroll
    for (int w = 0; w < NWT; ++w)
#pragma unroll
      for (int j = 0; j < FN; ++j) wv[s][w][j] = *reinterpret_cast<const f32x4*>(wp[w][j] + k);
  };
  auto step = [&](int s) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int w = 0; w < NWT; ++w)
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
          for (int j = 0; j < FN; ++j) acc[w][i][j] = mfma_f32(wv[s][w][j][e], xv[s][i][e], acc[w][i][j]);
  };
  load(0, 0);
  for (int k = 0; k < kq; k += 32) {                  // two 16-column steps, the next one's loads in flight
    if (k + 16 < kq) load(1, k + 16);
    step(0);
    if (k + 32 < kq) load(0, k + 32);
    if (k + 16 < kq) step(1);
  }
#pragma unroll
  for (int w = 0; w < NWT; ++w)
#pragma unroll
    for (int f = 0; f < NF; ++f) red[wave][w][f][lane] = acc[w][f / FN][f % FN];
  __syncthreads();
  const GemmLora& L = a.lora;
#pragma unroll
  for (int q = 0; q < NF / 4; ++q) {
    const int f = wave + 4 * q;
    const int m = m0 + 16 * (f / FN) + (lane & 15), n = n0 + 16 * (f % FN) + 4 * (lane >> 4);
    if (m >= a.M || n >= a.N) continue;
    f32x4 v[NWT];
#pragma unroll
    for (int w = 0; w < NWT; ++w) v[w] = ((red[0][w][f][lane] + red[1][w][f][lane]) + red[2][w][f][lane]) + red[3][w][f][lane];
    if (L.enabled) {
      const int slot = SWIGLU ? 0 : n / L.slot_width;
      v[0] += lora_f32(L, slot, m, SWIGLU ? n : n - slot * L.slot_width);
      if (SWIGLU) v[NWT - 1] += lora_f32(L, 1, m, n);
    }
    if (a.bias && !SWIGLU) v[0] += *reinterpret_cast<const f32x4*>((const float*)a.bias + n);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (SWIGLU) v[0][e] = silu_exact(v[0][e]) * v[NWT - 1][e];
      else if (EPI == EPI_GELU) v[0][e] = gelu_erf(v[0][e]);
    }
    f32x4* dst = reinterpret_cast<f32x4*>((float*)a.out + (int64_t)m * a.ldo + n);
    *dst = EPI == EPI_RESID ? *dst + v[0] : v[0];
  }
}

// 64x64 tiles where they give every CU a block, and a short K every CU two (one
// block's stores then overlap another's K loop), else 32x32.  4096 rows x 256
// columns of K = 1024: 27.5 us against 36.0 with 32x32 tiles; 1024 rows, 64
// such blocks: 11.5 us with 32x32.  Encoder layers, 32x32 against 64x64 at
// widths 512 / 1024: 512 rows 119.1 / 276.2 against 119.1 / 270.2 us, 4096 rows
// 515.8 / 1658 against 460.8 / 1381.  At width 256, products of K = 256 with 256
// to 511 such blocks: 1024 / 2048 / 4096 rows 92.0 / 122.2 / 191.3 us a layer
// with 64x64, 88.7 / 117.9 / 188.7 with 32x32.  SwiGLU's second weight takes the
// accumulators of the larger tile, so it stays at 32x32.
template <int EPI, bool SW>
void launch_f32(const GemmArgs& a, hipStream_t s) {
  auto blocks = [&](int b) { return (a.M + b - 1) / b * ((a.N + b - 1) / b); };
  if constexpr (!SW) {
    if (blocks(64) >= (a.K < 512 ? 512 : 256)) {
      hipLaunchKernelGGL((gemm_f32_kernel<EPI, SW, 4, 4>), dim3(blocks(64)), dim3(256), 0, s, a);
      return;
    }
  }
  hipLaunchKernelGGL((gemm_f32_kernel<EPI, SW, 2, 2>), dim3(blocks(32)), dim3(256), 0, s, a);
}

// Tile shapes of the large GEMM for an M x N product.  A launch of R tiles
// costs its rounds of 256 concurrent tiles (one per CU) times the bytes a
// tile moves per K step (BMT + BNT rows of 128 B; the loop is bound by that
// stream).  The candidates are the shapes whose column tiles do not straddle
// a LoRA slot.  Besides one launch of the cheapest shape, the rows may be
// split: whole 256-row tiles of one shape in full rounds, then the remaining
// rows with narrower tiles, so the last, partly filled round costs less.
// Every shape runs the same K steps in the same order, so a row's outputs do
// not depend on which launch or tile shape computes it.
struct LargeShape { int bm, bn; };
constexpr LargeShape kLargeShapes[3] = {{256, 256}, {256, 192}, {256, 128}};
inline bool shape_ok(const LargeShape& c, bool sw, int lora_slot_width, int rope_hd) {
  return !(lora_slot_width > 0 && !sw && lora_slot_width % c.bn) && !(rope_hd > 0 && c.bn % rope_hd);
}
inline double launch_cost(int rows, int N, bool sw, const LargeShape& c) {
  if (rows <= 0) return 0.0;
  const int nt = sw ? c.bn / 2 : c.bn;
  const long tiles = (long)((rows + c.bm - 1) / c.bm) * ((N + nt - 1) / nt);
  const long rounds = (tiles + 255) / 256;
  return (double)rounds * (c.bm + c.bn) * (sw ? 2.0 * nt / c.bn : 1.0);
}
struct LargePlan { LargeShape main, tail; int m1; };   // rows [0, m1) main, [m1, M) tail
inline LargePlan large_plan(int M, int N, bool sw, int lora_slot_width, int rope_hd) {
  LargePlan best = {{0, 0}, {0, 0}, M};
  double best_cost = 0.0;
  for (const LargeShape& c : kLargeShapes) {
    if (!shape_ok(c, sw, lora_slot_width, rope_hd)) continue;
    const double cost = launch_cost(M, N, sw, c);
    if (best.main.bm == 0 || cost < best_cost * 0.97) { best = {c, {0, 0}, M}; best_cost = cost; }
  }
  if (best.main.bm == 0) return best;
  const double single = best_cost;
  const LargeShape mc = best.main;
  const int nt = sw ? mc.bn / 2 : mc.bn;
  const int ntn = (N + nt - 1) / nt, mt = (M + mc.bm - 1) / mc.bm;
  // A last round under a quarter full already runs well below a full
  // round's time (its few tiles do not share L2 and HBM bandwidth): no split
  // (measured: the 7B QKV's 32-tile last round is cheaper than a 256 x 128
  // tail launch).  Otherwise a split must beat the single launch by 1.5%.
  const int last = (int)(((long)mt * ntn) % 256);
  if (last == 0 || last < 64) return best;
  const int full = (int)(((long)mt * ntn) / 256 * 256 / ntn);   // row tiles filling whole rounds
  for (int r1 = full; r1 >= 1 && r1 >= full - 2; --r1) {
    const int m1 = r1 * mc.bm;
    if (m1 >= M) continue;
    for (const LargeShape& t : kLargeShapes) {
      if (!shape_ok(t, sw, lora_slot_width, rope_hd)) continue;
      const double cost = launch_cost(m1, N, sw, mc) + launch_cost(M - m1, N, sw, t);
      if (cost < single * 0.985 && cost < best_cost) { best = {mc, t, m1}; best_cost = cost; }
    }
  }
  return best;
}

// Estimated time (us) of the plan above and of one launch of bm x 64 mid
// tiles.  A tile's K step costs its (bm + bn) operand rows of 128 B at the 47
// GB/s each CU is fed with (2.7 ns a row); to that a 256-row tile adds its
// first loads and its stores, 7 us per 128 columns, in every round, while the
// mid tiles share a CU and overlap theirs but once.  Fitted on products of
// 1182 to 8700 rows, 768 to 4224 columns and K = 768 to 3072.
inline double large_time(const LargePlan& p, int M, int N, int K, bool sw) {
  auto one = [&](int rows, const LargeShape& c) {
    if (rows <= 0) return 0.0;
    const int nt = sw ? c.bn / 2 : c.bn;
    const long tiles = (long)((rows + c.bm - 1) / c.bm) * ((N + nt - 1) / nt);
    return (tiles + 255) / 256 * (K / BK * (c.bm + c.bn) * 0.0027 + 7.0 * c.bn / 128);
  };
  return one(p.m1, p.main) + one(M - p.m1, p.tail);
}
inline double mid_time(int M, int N, int K, bool sw, int bm) {
  const int nt = sw ? 32 : 64;
  const double per_cu = (double)((M + bm - 1) / bm) * ((N + nt - 1) / nt) / 256.0;
  return (per_cu < 1.0 ? 1.0 : per_cu) * (K / BK) * (bm + 64) * 0.0024 + 4.0;
}

template <int EPI, bool SW, int BMT, int BNT>
void launch_large(const GemmArgs& a, hipStream_t s) {
  const int nt = SW ? BNT / 2 : BNT;
  const int ntiles = ((a.m_hi - a.m_lo + BMT - 1) / BMT) * ((a.N + nt - 1) / nt);
  const int grid = (ntiles + 7) / 8 * 8;
  // ranks <= 16 share LoRA steps (up to four runs per step)
  if (a.lora.enabled && a.lora.max_rank <= 16)
    hipLaunchKernelGGL((gemm_bf16_large_kernel<EPI, SW, BMT, BNT, true>), dim3(grid), dim3(512), 0, s, a);
  else
    hipLaunchKernelGGL((gemm_bf16_large_kernel<EPI, SW, BMT, BNT, false>), dim3(grid), dim3(512), 0, s, a);
}
template <int EPI, bool SW>
void launch_large_shape(const GemmArgs& a, const LargeShape& sh, hipStream_t s) {
  if (sh.bn == 256) launch_large<EPI, SW, 256, 256>(a, s);
  else if (sh.bn == 192) launch_large<EPI, SW, 256, 192>(a, s);
  else launch_large<EPI, SW, 256, 128>(a, s);
}

template <int EPI, bool SW, int BMT>
void launch_mid(const GemmArgs& a, hipStream_t s) {
  const int nt = SW ? 32 : 64;
  const int ntiles = ((a.M + BMT - 1) / BMT) * ((a.N + nt - 1) / nt);
  const int grid = (ntiles + 7) / 8 * 8;
  if (a.lora.enabled && a.lora.max_rank <= 16)
    hipLaunchKernelGGL((gemm_bf16_mid_kernel<EPI, SW, BMT, 64, true>), dim3(grid), dim3(256), 0, s, a);
  else
    hipLaunchKernelGGL((gemm_bf16_mid_kernel<EPI, SW, BMT, 64, false>), dim3(grid), dim3(256), 0, s, a);
}

template <int EPI, bool SW>
hipError_t launch_one(int dtype, const GemmArgs& a0, hipStream_t s) {
  if (dtype != VFM_BF16) {
    if (a0.rope.on) return hipErrorInvalidValue;
    launch_f32<EPI, SW>(a0, s);
    return hipGetLastError();
  }
  // 32-bit element offsets inside a tile
  const bool fits32 = (int64_t)a0.M * a0.ldx < ((int64_t)1 << 31) && (int64_t)a0.N * a0.K < ((int64_t)1 << 31);
  const int slot = a0.lora.enabled && !SW ? a0.lora.slot_width : 0;
  // the fused rotary embedding needs whole heads in a tile
  const int rope_hd = a0.rope.on ? a0.rope.head_dim : 0;
  const LargePlan pl = large_plan(a0.M, a0.N, SW, slot, rope_hd);
  const bool large_ok = fits32 && pl.main.bm > 0 && a0.M >= 1024;
  const bool mid_ok = fits32 && slot % 64 == 0 && (rope_hd == 0 || rope_hd == 64);
  const double t64 = mid_time(a0.M, a0.N, a0.K, SW, 64), t128 = mid_time(a0.M, a0.N, a0.K, SW, 128);
  if (mid_ok && (!large_ok || std::min(t64, t128) < large_time(pl, a0.M, a0.N, a0.K, SW))) {
    GemmArgs a = a0;
    a.m_lo = 0;
    a.m_hi = a.M;
    if (t64 <= t128) launch_mid<EPI, SW, 64>(a, s);
    else launch_mid<EPI, SW, 128>(a, s);
  } else if (large_ok) {
    GemmArgs a = a0;
    a.m_lo = 0;
    a.m_hi = pl.m1;
    launch_large_shape<EPI, SW>(a, pl.main, s);
    if (pl.m1 < a0.M) {
      a.m_lo = pl.m1;
      a.m_hi = a0.M;
      launch_large_shape<EPI, SW>(a, pl.tail, s);
    }
  } else if (a0.rope.on) {
    return hipErrorInvalidValue;   // only the tile kernels apply the rotary embedding
  } else {
    const GemmArgs& a = a0;
    const int nt = SW ? BN / 2 : BN;
    const int grid = ((a.M + BM - 1) / BM) * ((a.N + nt - 1) / nt);
    hipLaunchKernelGGL((gemm_bf16_kernel<EPI, SW>), dim3(grid), dim3(256), 0, s, a);
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_gemm(int dtype, const GemmArgs& a, hipStream_t s) {
  if (a.M == 0) return hipSuccess;
  switch (a.epi) {
    case EPI_STORE: return launch_one<EPI_STORE, false>(dtype, a, s);
    case EPI_GELU: return launch_one<EPI_GELU, false>(dtype, a, s);
    case EPI_RESID: return launch_one<EPI_RESID, false>(dtype, a, s);
    case EPI_SWIGLU: return launch_one<EPI_STORE, true>(dtype, a, s);
  }
  return hipErrorInvalidValue;
}
