// fp32 MFMA GEMM for gfx950 (v_mfma_f32_32x32x2_f32): C = A . B, A row-major
// [M, K], B row-major [K, N] or given by its transpose [N, K].
//
// 128x128 or 64x64 output tile per workgroup, four waves (2 x 2) of 64x64 or
// 32x32.  K advances in 32-wide tiles through NS = 2 LDS stages that buffer
// loads write directly (four hold a CU to two workgroups: 1000 x 600 in 8 shards
// of 128 27.9 us against 26.4, 1961 x 1776 x 2176 143 against 136); the pipeline is that of the bf16 tile kernel (one barrier
// per K tile, before its last step, after which the stage is refilled and the
// next tile's first fragments are read).  A #sum runs in one accumulator over
// all K or as one fp32 partial per K range.
//
// The MFMA takes one float per lane, k = lane / 32.  A lane of half h reads
// the 16 bytes k = 8 s + 4 h .. + 3 of its row at once, and element e of both
// operands feeds MFMA e, which so contracts k = 8 s + e and 8 s + 4 + e: one
// LDS read per four MFMAs, where the order inside the 8 k does not matter.
//
// Bound by the matrix cores (157 TFLOP/s): 64 cycles per MFMA against 16 bytes
// of LDS reads per lane and four MFMAs.  Against one 32x32 accumulator a wave
// over a single register-staged LDS buffer (the staged kernel below, which used
// to run every size): 1800 x 2056 x 2048 204 -> 126 us (74 -> 120 TFLOP/s),
// 4096^3 at 144 TFLOP/s.
#include "kernels.h"
#include "lds_dma.h"

namespace partir {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int BK = 32, NT = 256, KK = BK / 8, NS = 2;
constexpr uint32_t OOB = 0x80000000u;          // offset that reads as zero

// K-contiguous tile: 128-byte rows of eight 16-byte chunks, chunk c of row r
// at position c ^ swz(r).  A fragment read takes one chunk of 32 rows in the
// low lanes and the next chunk of the same rows in the high lanes.  Rows of
// one parity share their banks: bits 1 and 2 send four of them to different
// chunk pairs, bit 3 the next four to the other chunk of the pair, so neither
// 8 rows x 2 chunks nor 16 rows x 1 chunk meet on a bank.
__device__ __forceinline__ int swz(int r) { return (r & 6) | ((r >> 3) & 1); }
// [k][n] tile: rows of 4 BN bytes, chunk c of k row r at c ^ kn_swz(r): the
// rows 8 s + e and 8 s + 4 + e that one read takes 128 bytes of fall on
// different halves of the banks.
__device__ __forceinline__ int kn_swz(int r) { return 8 * ((r >> 2) & 1); }

template <int BT, int BKN>
__device__ __forceinline__ void gemm_f32_body(const GemmF32Params& p) {
  constexpr int WT = BT / 2, NB = WT / 32;         // a wave's part of the tile, in 32-wide blocks
  constexpr int OP = BT * BK * 4, STAGE = 2 * OP;
  constexpr int LO = BT / 32;                      // wave loads (1 KiB) per wave, operand and K tile
  constexpr int LPS = 2 * LO;
  __shared__ __attribute__((aligned(1024))) char smem[NS * STAGE];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int h = lane >> 5, l32 = lane & 31;

  // XCD x (workgroups go round-robin to the 8 XCDs) takes a contiguous run of
  // the tile order, four tile rows at a time
  const int ntiles = p.tiles_m * p.tiles_n;
  int bid;
  {
    const int x = blockIdx.x & 7, q = gridDim.x >> 3, r = gridDim.x & 7;
    bid = x * q + min(x, r) + (int)(blockIdx.x >> 3);
  }
  const int split = bid / ntiles;
  const int tix = bid - split * ntiles;
  const int gidx = tix / (4 * p.tiles_n), first_m = gidx * 4;
  const int gm = min(p.tiles_m - first_m, 4);
  const int rr = tix - gidx * 4 * p.tiles_n;
  const int tn = rr / gm, tm = first_m + rr - tn * gm;
  const int row0 = tm * BT, col0 = tn * BT;
  const int rows = min(BT, p.M - row0), cols = min(BT, p.N - col0);
  const int k_begin = p.nsplit > 1 ? split * p.ks : 0;
  const int k_end = p.nsplit > 1 ? min(p.K, k_begin + p.ks) : p.K;
  const int nk = (k_end - k_begin + BK - 1) / BK;

  // K-contiguous operand: load j of wave w fills tile rows 32 j + 8 w .. +7,
  // lane L taking row +L/8 and LDS chunk L%8 = global chunk (L%8) ^ swz(row);
  // one descriptor per 32 rows bounds the valid rows (rows past it read
  // zero).  B as [K, N]: load j of wave w fills R = 256 / BT k rows at
  // R (4 j + w); a descriptor per K tile bounds the rows at the end of K and
  // the last one at the last column.
  __amdgpu_buffer_rsrc_t ra[LO], rb[LO];
#pragma unroll
  for (int j = 0; j < LO; ++j) {
    ra[j] = make_rsrc(p.A + (int64_t)(row0 + 32 * j) * p.lda, (uint32_t)(min(max(rows - 32 * j, 0), 32) * p.lda * 4));
    if (!BKN)
      rb[j] = make_rsrc(p.B + (int64_t)(col0 + 32 * j) * p.ldb, (uint32_t)(min(max(cols - 32 * j, 0), 32) * p.ldb * 4));
  }
  const int lrow = 8 * wave + (lane >> 3);
  const int lchunk = (lane & 7) ^ swz(lrow);
  const uint32_t a_voff = (uint32_t)(lrow * p.lda * 4 + lchunk * 16);
  const uint32_t b_voff = (uint32_t)(lrow * p.ldb * 4 + lchunk * 16);
  uint32_t b_kn[LO];
  if (BKN) {
    constexpr int R = 256 / BT;
#pragma unroll
    for (int j = 0; j < LO; ++j) {
      const int r = R * (4 * j + wave) + lane / (BT / 4);
      b_kn[j] = (uint32_t)(r * p.ldb * 4 + (((lane % (BT / 4)) ^ kn_swz(r)) << 4));
    }
  }
  const uint32_t b_cut = (uint32_t)(p.ldb - (p.N - col0)) * 4;   // what the last k row lacks of a whole leading dim
  // the loads of K tile kt into stage st (past the end of K: zeros)
  struct LoadSet {
    __amdgpu_buffer_rsrc_t rb;   // B as [K, N]
    char* lds;
    uint32_t so, va, vb;
  };
  auto prep = [&](int kt, int st) -> LoadSet {
    LoadSet L;
    const int kb = k_begin + kt * BK;
    const uint32_t kmask = (kb + lchunk * 4 < k_end) ? 0u : OOB;
    L.lds = smem + st * STAGE + wave * 1024;
    L.so = (uint32_t)kb * 4;
    L.va = a_voff | kmask;
    L.vb = b_voff | kmask;
    if (BKN) {
      const uint32_t kvalid = (uint32_t)min(max(k_end - kb, 0), BK);
      L.rb = make_rsrc(p.B + (int64_t)kb * p.ldb + col0, kvalid * (uint32_t)p.ldb * 4 - (kvalid ? b_cut : 0u));
    }
    return L;
  };
  auto issue = [&](const LoadSet& L, int q) {
    if (q < LO)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(ra[q], (lds_void*)(L.lds + q * 4096), 16, L.va, L.so, 0, 0);
    else if (BKN)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(L.rb, (lds_void*)(L.lds + OP + (q - LO) * 4096), 16, b_kn[q - LO], 0, 0, 0);
    else
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rb[q - LO], (lds_void*)(L.lds + OP + (q - LO) * 4096), 16, L.vb, L.so, 0, 0);
  };
  // fragments of step s (k = 8 s .. + 7) of the tile in stage st
  auto ldfrag = [&](int st, int s, f32x4* a, f32x4* b) {
    const char* pa = smem + st * STAGE;
    const char* pb = pa + OP;
    const int ko = ((2 * s + h) ^ swz(l32)) << 4;
#pragma unroll
    for (int i = 0; i < NB; ++i) a[i] = lds_read<f32x4>(pa + (wm * WT + 32 * i + l32) * (BK * 4) + ko);
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      if constexpr (BKN) {
        const int k = 8 * s + 4 * h, n = wn * WT + 32 * j + l32;
        const char* q = pb + k * (BT * 4) + ((((n >> 2) ^ kn_swz(k)) << 4) | ((n & 3) << 2));
#pragma unroll
        for (int e = 0; e < 4; ++e) b[j][e] = lds_read<float>(q + e * (BT * 4));   // k .. k + 3 share kn_swz
      } else {
        b[j] = lds_read<f32x4>(pb + (wn * WT + 32 * j + l32) * (BK * 4) + ko);
      }
    }
  };
  f32x16 acc[NB][NB];
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;
  // the 4 NB^2 MFMAs of a step; `after(i)` follows MFMA i
  auto mma = [&](const f32x4* a, const f32x4* b, auto after) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) {
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i][e], b[j][e], acc[i][j], 0, 0, 0);
          after((e * NB + i) * NB + j);
        }
  };

  f32x4 fa[2][NB], fb[2][NB];
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const LoadSet L = prep(s, s);
#pragma unroll
    for (int q = 0; q < LPS; ++q) issue(L, q);
  }
  WAIT_VMCNT(LPS * (NS - 1));
  asm volatile("s_barrier" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
  ldfrag(0, 0, fa[0], fb[0]);
  int st = 0;
  for (int kt = 0; kt < nk; ++kt) {
#pragma unroll
    for (int s = 0; s < KK - 1; ++s) {
      ldfrag(st, s + 1, fa[(s + 1) & 1], fb[(s + 1) & 1]);
      mma(fa[s & 1], fb[s & 1], [](int) {});
    }
    const LoadSet L = prep(kt + NS, st);
    st = (st + 1 == NS) ? 0 : st + 1;
    __builtin_amdgcn_sched_barrier(0);
    WAIT_LGKMCNT(0);                // every read of this stage done,
    WAIT_VMCNT(LPS * (NS - 2));     // this wave's loads of tile kt + 1 landed
    asm volatile("s_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    // One load after each MFMA: a wave that issues its loads in a row waits
    // for the address unit with its matrix core idle (4096^3: 980 us in a
    // row, 955 spread out).
    mma(fa[(KK - 1) & 1], fb[(KK - 1) & 1], [&](int i) {
      if (i < LPS) issue(L, i);
      if (i == 0) ldfrag(st, 0, fa[0], fb[0]);
      if (i <= LPS) __builtin_amdgcn_sched_barrier(0);
    });
  }
  WAIT_VMCNT(0);   // no LDS write is in flight at exit

  // lane holds C[m = 8 (v / 4) + 4 h + v % 4][n = lane % 32] of each 32x32
  // block: 128-byte runs of two rows per store
  float* out = p.C + (p.epi == EPI_PARTIAL ? split * p.part_stride : 0);
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const int nl = wn * WT + 32 * j + l32;
      if (nl >= cols) continue;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int ml = wm * WT + 32 * i + 8 * (v >> 2) + 4 * h + (v & 3);
        if (ml < rows) out[(int64_t)(row0 + ml) * p.ldc + col0 + nl] = acc[i][j][v];
      }
    }
}

template <int BT, int BKN>
__global__ __launch_bounds__(NT, 2) void gemm_f32_kernel(GemmF32Params p) { gemm_f32_body<BT, BKN>(p); }

// Any leading dimension (64-bit addresses; the kernel above bounds its loads
// by 32-bit byte ranges), and a short K on many workgroups (the planner says
// where the line lies): 64x64 tiles, K in steps of 16 through one LDS buffer,
// register-staged.
constexpr int LT = 64, LBK = 16, PAD = 4;
__global__ __launch_bounds__(NT) void gemm_f32_staged_kernel(GemmF32Params p) {
  __shared__ float As[LBK][LT + PAD];
  __shared__ float Bs[LBK][LT + PAD];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int ntiles = p.tiles_m * p.tiles_n;
  const int split = blockIdx.x / ntiles;
  const int t = blockIdx.x - split * ntiles;
  const int tm = t / p.tiles_n, tn = t - tm * p.tiles_n;
  const int row0 = tm * LT, col0 = tn * LT;
  const int rows = min(LT, p.M - row0), cols = min(LT, p.N - col0);
  const int k_begin = p.nsplit > 1 ? split * p.ks : 0;
  const int k_end = p.nsplit > 1 ? min(p.K, k_begin + p.ks) : p.K;

  f32x16 acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
  // loader coordinates: A tile [64 m][16 k] as 256 float4 along k
  const int am = tid >> 2, ak = (tid & 3) * 4;
  for (int kb = k_begin; kb < k_end; kb += LBK) {
    {
      f32x4 v = {0.f, 0.f, 0.f, 0.f};
      if (am < rows && kb + ak < k_end) v = *(const f32x4*)(p.A + (int64_t)(row0 + am) * p.lda + kb + ak);
#pragma unroll
      for (int e = 0; e < 4; ++e) As[ak + e][am] = v[e];
    }
    if (p.b_nk) {  // B^T [N, K]: same pattern as A
      f32x4 v = {0.f, 0.f, 0.f, 0.f};
      if (am < cols && kb + ak < k_end) v = *(const f32x4*)(p.B + (int64_t)(col0 + am) * p.ldb + kb + ak);
#pragma unroll
      for (int e = 0; e < 4; ++e) Bs[ak + e][am] = v[e];
    } else {       // B [K, N]: 16 rows of 64 along n
      const int bk = tid >> 4, bn = (tid & 15) * 4;
      f32x4 v = {0.f, 0.f, 0.f, 0.f};
      if (bn < cols && kb + bk < k_end) v = *(const f32x4*)(p.B + (int64_t)(kb + bk) * p.ldb + col0 + bn);
      *(f32x4*)&Bs[bk][bn] = v;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < LBK; kk += 2) {
      const float a = As[kk + (lane >> 5)][wm * 32 + (lane & 31)];
      const float b = Bs[kk + (lane >> 5)][wn * 32 + (lane & 31)];
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, acc, 0, 0, 0);
    }
    __syncthreads();
  }
  const int nl = wn * 32 + (lane & 31);
  if (nl >= cols) return;
  float* out = p.C + (p.epi == EPI_PARTIAL ? split * p.part_stride : 0);
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int ml = wm * 32 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
    if (ml < rows) out[(int64_t)(row0 + ml) * p.ldc + col0 + nl] = acc[v];
  }
}

template <int BT>
void launch(const GemmF32Params& p, dim3 grid, hipStream_t s) {
  if (p.b_nk) hipLaunchKernelGGL((gemm_f32_kernel<BT, 0>), grid, dim3(NT), 0, s, p);
  else hipLaunchKernelGGL((gemm_f32_kernel<BT, 1>), grid, dim3(NT), 0, s, p);
}

constexpr int64_t kMaxLd = (int64_t)1 << 24;   // 32 rows (or k rows) within a 2^31-byte range

}  // namespace

int gemm_f32_tile() { return LT; }

hipError_t launch_gemm_f32(const GemmF32Params& p, hipStream_t s) {
  const int64_t nwg = (int64_t)p.tiles_m * p.tiles_n * p.nsplit;
  if (nwg <= 0 || nwg >= ((int64_t)1 << 31)) return hipErrorInvalidValue;
  const dim3 grid((unsigned)nwg);
  if (p.staged ? p.tile != LT : (p.lda > kMaxLd || p.ldb > kMaxLd)) return hipErrorInvalidValue;
  if (p.staged) {
    hipLaunchKernelGGL(gemm_f32_staged_kernel, grid, dim3(NT), 0, s, p);
  } else if (p.tile == 128) {
    launch<128>(p, grid, s);
  } else if (p.tile == 64) {
    launch<64>(p, grid, s);
  } else {
    return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace partir
