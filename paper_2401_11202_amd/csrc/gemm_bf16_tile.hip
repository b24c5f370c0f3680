// bf16 MFMA GEMM for gfx950 in 128x128 and 64x64 output tiles: the products
// whose 256x256 tiles (gemm_bf16.hip) would leave most of the chip idle.
//
// Same contract, operand layouts and #tile / #sum semantics as gemm_bf16.hip:
// C = A . B^T, A K-contiguous or stored [K, M], B K-contiguous or stored
// [K, N], the epilogues of GemmEpi, device-local arrays.  The same MFMA
// (16x16x32, K ascending in steps of 32) forms every sum, so an output element
// whose K range is not split has the same bits whichever tile computed it.
//
// 2 x WN waves own equal parts of the tile.  K advances in 64-wide tiles
// through NS LDS stages filled by direct-to-LDS buffer loads; one barrier per
// K tile, in its middle:
//   step 0   MFMAs of k 0..31,  fragments of k 32..63 read meanwhile
//   wait     tile kt+1 landed (the younger loads stay in flight), barrier
//   refill   this stage with tile kt+NS (every wave has read all of it)
//   step 1   MFMAs of k 32..63, first fragments of tile kt+1 read meanwhile
// so between NS - 1 and NS tiles are in flight.
//
// The 128-wide tile has two forms.  A grid of at most one workgroup a CU is
// bound by the latency of this chain and by the bytes in flight: four stages
// (128 KiB) and eight waves, so that a SIMD has a second wave to run while one
// waits for its fragments (2048^3 24.4 us with four waves, 21.7 with eight;
// 200 x 16384 x 4096 39.4 and 36.0).  A larger grid runs two workgroups of
// four waves a CU on two stages each (4096^3 119 us; with eight waves 122,
// their smaller wave tiles read more LDS).  Per K tile (2048 x 2048 x 8192,
// one workgroup a CU) the MFMAs alone take 0.29 us, with the fragment reads
// 0.40, with the loads 0.52: the waits for loads and fragments bound it, not a
// unit at its rate (200 x 16384 x 4096, counters: matrix cores busy 0.32 of
// cycles, LDS reads 0.25, HBM 3.5 TB/s), and the 256-wide tile with fewer of
// them per MFMA is better on whole waves (4096^3: 95 us).  Before / after
// this kernel (launch time, us): 2048^3 44 -> 22, 200 x 16384 x 4096 57 -> 36,
// 200 x 4096 x 16384 108 -> 42 (4 K parts), 512 x 1024 x 256 13 -> 7 (64-wide).
#include <type_traits>

#include "kernels.h"
#include "device_math.h"
#include "lds_dma.h"

namespace partir {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef short i16x4 __attribute__((ext_vector_type(4)));

constexpr int BK = 64;
constexpr uint32_t OOB = 0x80000000u;          // offset that reads as zero

template <typename T>
__device__ __forceinline__ T pick3(int g, T a, T b, T c) { return g == 0 ? a : (g == 1 ? b : c); }

template <int BM, int BN, int WN, int NS, int AMN, int BMN, int PARTS>
__device__ __forceinline__ void tile_body(const GemmParams& p, const GemmParts* t) {
  static_assert(!(PARTS && (AMN || BMN)), "device-local arrays are K-contiguous");
  constexpr int NW = 2 * WN;                       // waves, 2 x WN
  constexpr int WTM = BM / 2, WTN = BN / WN;       // a wave's part of the tile
  constexpr int MI = WTM / 16, NJ = WTN / 16;
  constexpr int OPA = BM * BK * 2, OPB = BN * BK * 2, STAGE = OPA + OPB;
  constexpr int LA = BM / (8 * NW), LB = BN / (8 * NW);        // wave loads (1 KiB) per wave per K tile
  constexpr int LPS = LA + LB;
  // epilogue staging: 16 rows of the wave's columns, fp32, padded
  constexpr int CP = WTN + 4;
  constexpr int CW = 16 * CP * 4;
  static_assert(NW * 2 * CW <= NS * STAGE, "epilogue staging fits the K stages");
  __shared__ __attribute__((aligned(1024))) char smem[NS * STAGE];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;

  // ---- which tile -----------------------------------------------------------
  // XCD x (workgroups go round-robin to the 8 XCDs) takes a contiguous run of
  // the tile order, so neighbouring tiles share that XCD's L2.
  const int ntiles = p.tiles_m * p.tiles_n;
  int bid;
  {
    const int x = blockIdx.x & 7, q = gridDim.x >> 3, r = gridDim.x & 7;
    bid = x * q + min(x, r) + (int)(blockIdx.x >> 3);
  }
  const int split = bid / ntiles;
  const int tix = bid - split * ntiles;
  const int per_group = p.group_m * p.tiles_n;
  const int gidx = tix / per_group;
  const int first_m = gidx * p.group_m;
  const int gm = min(p.tiles_m - first_m, p.group_m);
  const int rr = tix - gidx * per_group;
  const int tm = first_m + rr % gm;
  const int tn = rr / gm;
  const int row0 = tm * BM;
  const int rows = min(BM, p.M - row0);
  const int grp = tn / p.tpn;
  const int col0 = (tn - grp * p.tpn) * BN;
  const int cols = min(BN, p.N - col0);
  const int k_begin = p.nsplit > 1 ? split * p.ks : 0;
  const int k_end = p.nsplit > 1 ? min(p.K, k_begin + p.ks) : p.K;
  const int nk = (k_end - k_begin + BK - 1) / BK;

  // ---- global -> LDS loads ----------------------------------------------------
  // K-contiguous operand: load j of wave w fills tile rows 8 (NW j + w) .. +7;
  // lane L takes row +L/8 and LDS chunk L%8 = global chunk (L%8) ^ gemm_swz(row).
  // One descriptor per 64 rows bounds the valid rows (rows past it read zero).
  // MN-major operand: load j of wave w fills R = 512 / W k rows at R (NW j + w);
  // a descriptor per K tile bounds the k rows at the end of K and the last one
  // at the operand's last column.
  const uint16_t* Bg = pick3(grp, p.B[0], p.B[1], p.B[2]);
  __amdgpu_buffer_rsrc_t ra[BM / 64], rb[BN / 64];
  auto b_ptr = [&](int r0, int kp) -> const uint16_t* {
    if (PARTS && t->b_nrows) {
      const int gb = grp * t->b_gstride;
      const int n = col0 + (r0 < cols ? r0 : 0);    // rows past the end: any part, size 0 below
      const int nb = n / t->b_nrows;
      return t->b[gb + nb * t->b_nk + kp] + (int64_t)(n - nb * t->b_nrows) * p.ldb;
    }
    return Bg + (int64_t)(col0 + r0) * p.ldb;
  };
  auto b_desc = [&](int kp) {
#pragma unroll
    for (int j = 0; j < BN / 64; ++j)
      rb[j] = make_rsrc(b_ptr(64 * j, kp), (uint32_t)(min(max(cols - 64 * j, 0), 64) * p.ldb * 2));
  };
  if (!AMN) {
#pragma unroll
    for (int j = 0; j < BM / 64; ++j) {
      const uint16_t* a = p.A + (int64_t)(row0 + 64 * j) * p.lda;
      if (PARTS && t->a_rows) {
        const int r = row0 + (64 * j < rows ? 64 * j : 0);
        const int ab = r / t->a_rows;
        a = t->a[ab] + (int64_t)(r - ab * t->a_rows) * p.lda;
      }
      ra[j] = make_rsrc(a, (uint32_t)(min(max(rows - 64 * j, 0), 64) * p.lda * 2));
    }
  }
  if (!BMN) b_desc(0);
  // the all_gather of B along K: the part that holds K tile kt (a K tile never
  // spans two, and they come in order)
  int b_kpart = 0, b_k0 = 0;
  auto b_advance = [&](int kt) {
    if (PARTS && t->b_nrows) {
      const int kb = k_begin + kt * BK;
      while (kb >= b_k0 + t->b_kcols && b_kpart + 1 < t->b_nk) {
        ++b_kpart;
        b_k0 += t->b_kcols;
        b_desc(b_kpart);
      }
    }
  };
  const int lrow = 8 * wave + (lane >> 3);
  const int lchunk = (lane & 7) ^ gemm_swz(lrow);
  constexpr int RL = 8 * NW, LPB = 64 / RL;   // rows per load of all waves, loads per 64 rows
  uint32_t a_voff[LPB], b_voff[LPB];
#pragma unroll
  for (int e = 0; e < LPB; ++e) {
    a_voff[e] = (uint32_t)((lrow + RL * e) * p.lda * 2 + lchunk * 16);
    b_voff[e] = (uint32_t)((lrow + RL * e) * p.ldb * 2 + lchunk * 16);
  }
  uint32_t a_mv[LA], b_mv[LB];
  if (AMN) {
    constexpr int R = 512 / BM;
    const int r0 = R * wave + lane / (BM / 8);
#pragma unroll
    for (int j = 0; j < LA; ++j)
      a_mv[j] = (uint32_t)((NW * R * j + r0) * p.lda * 2 + (((lane % (BM / 8)) ^ gemm_mn_swz<BM>(r0)) << 4));
  }
  if (BMN) {
    constexpr int R = 512 / BN;
    const int r0 = R * wave + lane / (BN / 8);
#pragma unroll
    for (int j = 0; j < LB; ++j)
      b_mv[j] = (uint32_t)((NW * R * j + r0) * p.ldb * 2 + (((lane % (BN / 8)) ^ gemm_mn_swz<BN>(r0)) << 4));
  }
  // what the last k row of an MN-major operand lacks of a whole leading dim
  const uint32_t a_cut = (uint32_t)(p.lda - (p.M - row0)) * 2, b_cut = (uint32_t)(p.ldb - (p.N - col0)) * 2;
  // K tile kt into stage `st` (past the end of K: zeros, so the number of
  // loads in flight never depends on kt)
  auto gload = [&](int kt, int st) {
    const int kb = k_begin + kt * BK;
    char* la = smem + st * STAGE + wave * 1024;
    char* lb = la + OPA;
    const uint32_t kmask = (kb + lchunk * 8 < k_end) ? 0u : OOB;
    const uint32_t so = (uint32_t)kb * 2;
    const uint32_t kvalid = (uint32_t)min(max(k_end - kb, 0), BK);
    if constexpr (AMN) {
      const uint32_t bytes = kvalid * (uint32_t)p.lda * 2 - (kvalid ? a_cut : 0u);
      const __amdgpu_buffer_rsrc_t r = make_rsrc(p.A + (int64_t)kb * p.lda + row0, bytes);
#pragma unroll
      for (int j = 0; j < LA; ++j)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void*)(la + j * NW * 1024), 16, a_mv[j], 0, 0, 0);
    } else {
#pragma unroll
      for (int j = 0; j < LA; ++j)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(ra[j / LPB], (lds_void*)(la + j * NW * 1024), 16, a_voff[j % LPB] | kmask, so, 0, 0);
    }
    if constexpr (BMN) {
      const uint32_t bytes = kvalid * (uint32_t)p.ldb * 2 - (kvalid ? b_cut : 0u);
      const __amdgpu_buffer_rsrc_t r = make_rsrc(Bg + (int64_t)kb * p.ldb + col0, bytes);
#pragma unroll
      for (int j = 0; j < LB; ++j)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void*)(lb + j * NW * 1024), 16, b_mv[j], 0, 0, 0);
    } else {
      const uint32_t so_b = PARTS ? (uint32_t)(kb - b_k0) * 2 : so;
#pragma unroll
      for (int j = 0; j < LB; ++j)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rb[j / LPB], (lds_void*)(lb + j * NW * 1024), 16, b_voff[j % LPB] | kmask, so_b, 0, 0);
    }
  };

  // ---- MFMA operand reads (fragment layouts as in gemm_bf16.hip) --------------
  const int g16 = lane >> 4, j16 = lane & 15;
  const int fsw = gemm_swz(j16);
  const int mn_row = 8 * g16 + (j16 >> 2);
  const int mn_col = 4 * (j16 & 3);
  auto mn_frag = [&](const char* op, auto width, int ks, int bc) -> bf16x8 {
    constexpr int W = decltype(width)::value;
    const int col = bc + mn_col;
    const char* pl = op + (32 * ks + mn_row) * (2 * W) + (((col >> 3) ^ gemm_mn_swz<W>(mn_row)) << 4) + ((col & 4) << 1);
    const i16x4 lo = lds_read_tr16(pl);
    const i16x4 hi = lds_read_tr16(pl + 4 * 2 * W);
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };
  auto ldfrag = [&](int st, int ks, bf16x8* a, bf16x8* b) {
    const char* pa = smem + st * STAGE;
    const char* pb = pa + OPA;
    const int ko = ((4 * ks + g16) ^ fsw) << 4;
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      if constexpr (AMN) a[i] = mn_frag(pa, std::integral_constant<int, BM>{}, ks, wm * WTM + i * 16);
      else a[i] = lds_read<bf16x8>(pa + (wm * WTM + i * 16 + j16) * (BK * 2) + ko);
    }
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      if constexpr (BMN) b[j] = mn_frag(pb, std::integral_constant<int, BN>{}, ks, wn * WTN + j * 16);
      else b[j] = lds_read<bf16x8>(pb + (wn * WTN + j * 16 + j16) * (BK * 2) + ko);
    }
  };
  f32x4 acc[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  auto mma = [&](const bf16x8* a, const bf16x8* b) {
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[j], a[i], acc[i][j], 0, 0, 0);
  };
  auto barrier = [] {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };

  // instruction order of a step: the next fragments' reads (and the refill's
  // loads) spread over its MFMAs, the reads two per MFMA from the start
  constexpr int NRD = MI * (AMN ? 2 : 1) + NJ * (BMN ? 2 : 1);
#define SGB(mask, n) __builtin_amdgcn_sched_group_barrier(mask, n, 0)   // MFMA 0x8, VMEM 0x20, DS read 0x100
#define SLOTS(loads)                                                     \
  _Pragma("unroll") for (int sl = 0; sl < MI * NJ; ++sl) {               \
    SGB(0x8, 1);                                                         \
    if (2 * sl < NRD) SGB(0x100, 2);                                     \
    if ((loads) && sl < LPS) SGB(0x20, 1);                               \
  }
  bf16x8 fa0[MI], fb0[NJ], fa1[MI], fb1[NJ];
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    b_advance(s);
    gload(s, s);
  }
  WAIT_VMCNT(LPS * (NS - 1));
  barrier();
  ldfrag(0, 0, fa0, fb0);
  int st = 0;
  for (int kt = 0; kt < nk; ++kt) {
    b_advance(kt + NS);
    ldfrag(st, 1, fa1, fb1);
    mma(fa0, fb0);
    SLOTS(false);
    __builtin_amdgcn_sched_barrier(0);
    WAIT_LGKMCNT(0);
    WAIT_VMCNT(LPS * (NS - 2));
    barrier();
    gload(kt + NS, st);
    st = (st + 1 == NS) ? 0 : st + 1;
    ldfrag(st, 0, fa0, fb0);
    mma(fa1, fb1);
    SLOTS(true);
  }
#undef SLOTS
#undef SGB
  WAIT_VMCNT(0);
  WAIT_LGKMCNT(0);
  barrier();   // every load landed, every read done: the stages are free

  // ---- epilogue ----------------------------------------------------------------
  // A lane holds 4 consecutive columns of one row per 16x16 block.  Each wave
  // passes its rows 16 at a time through its own piece of LDS (no workgroup
  // barrier) and stores them as whole row runs of its columns.
  const float* bias = pick3(grp, p.bias[0], p.bias[1], p.bias[2]);
  void* Cg = pick3(grp, p.C[0], p.C[1], p.C[2]);
  const int epi = p.epi, act = p.act;
  const int wr0 = wm * WTM, wc0 = wn * WTN;
  float* cs = (float*)(smem + wave * 2 * CW);
  auto wave_sync = [] {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  if (bias) {
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int nl = wc0 + j * 16 + 4 * g16;
      if (nl < cols) {
        const f32x4 bv = *(const f32x4*)(bias + col0 + nl);
#pragma unroll
        for (int i = 0; i < MI; ++i) acc[i][j] += bv;
      }
    }
  }
  // fp32 rows: 4 columns per lane, bf16 rows: 8 per lane
  auto put = [&](int i, bool apply_act) {
    float* c = cs + (i & 1) * (CW / 4);
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      f32x4 v = acc[i][j];
      if (apply_act) {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = gelu_erf(v[e]);
      }
      *(f32x4*)(c + j16 * CP + j * 16 + 4 * g16) = v;
    }
    wave_sync();
    return c;
  };
  auto store_bf16 = [&](uint16_t* out, bool apply_act, bool parted) {
    constexpr int LR = WTN / 8, RPP = 64 / LR;   // lanes per row, rows per pass
    const int cr = lane / LR, cc = (lane % LR) * 8;
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      const float* c = put(i, apply_act);
      uint16_t* ob = out + (int64_t)(row0 + wr0 + i * 16) * p.ldc;
      if (PARTS && parted) {   // the 16 rows share a part (c_rows % 16 == 0): one scalar table read
        const int r = row0 + wr0 + i * 16, cb = min(r, p.M - 1) / t->c_rows;
        ob = (uint16_t*)t->c[cb] + (int64_t)(r - cb * t->c_rows) * p.ldc;
      }
#pragma unroll
      for (int r0 = 0; r0 < 16; r0 += RPP) {
        const f32x4 lo = *(const f32x4*)(c + (r0 + cr) * CP + cc), hi = *(const f32x4*)(c + (r0 + cr) * CP + cc + 4);
        const int rl = wr0 + i * 16 + r0 + cr, cl = wc0 + cc;
        if (rl >= rows || cl >= cols) continue;
        const bf16x8 o = {(__bf16)lo[0], (__bf16)lo[1], (__bf16)lo[2], (__bf16)lo[3],
                          (__bf16)hi[0], (__bf16)hi[1], (__bf16)hi[2], (__bf16)hi[3]};
        uint16_t* dst = ob + (int64_t)(r0 + cr) * p.ldc + col0 + cl;
        const i32x4 v = __builtin_bit_cast(i32x4, o);
        if (cl + 8 <= cols) *(i32x4*)dst = v;
        else *(int2*)dst = make_int2(v[0], v[1]);   // a 4-column tail (cols % 8 == 4)
      }
      wave_sync();
    }
  };
  if (epi == EPI_BF16 || epi == EPI_BF16_SAVE) {
    if (epi == EPI_BF16_SAVE) store_bf16((uint16_t*)p.aux, false, false);
    store_bf16((uint16_t*)Cg, act != 0, PARTS && t->c_rows);
    return;
  }
  constexpr int LR = WTN / 4, RPP = 64 / LR, NP = 16 / RPP;
  const int cr = lane / LR, cc = (lane % LR) * 4;
  float* out = epi == EPI_PARTIAL ? p.partial + split * p.part_stride : (float*)Cg;
  const int64_t ldo = epi == EPI_PARTIAL ? p.part_ld : p.ldc;
  const bool parted = PARTS && epi != EPI_PARTIAL && t->c_rows;
  // start of the 16 rows of block i (which share a part: one scalar table read)
  auto rows_of = [&](int i) -> float* {
    const int r = row0 + wr0 + i * 16;
    if (parted) {
      const int cb = min(r, p.M - 1) / t->c_rows;
      return (float*)t->c[cb] + (int64_t)(r - cb * t->c_rows) * ldo;
    }
    return out + (int64_t)r * ldo;
  };
  // a residual (which may alias C: each element is read, then written, by
  // the same lane) is read before the rows are staged: one round trip
  f32x4 rv[MI][NP];
  if (epi == EPI_RESID_F32) {
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      const float* src = parted ? rows_of(i) : p.resid + (int64_t)(row0 + wr0 + i * 16) * p.ldr;
      const int64_t lds = parted ? ldo : p.ldr;
#pragma unroll
      for (int k = 0; k < NP; ++k) {
        const int rl = wr0 + i * 16 + k * RPP + cr;
        rv[i][k] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        if (rl < rows && wc0 + cc < cols)
          rv[i][k] = *(const f32x4*)(src + (k * RPP + cr) * lds + col0 + wc0 + cc);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    const float* c = put(i, act != 0);
    float* dst = rows_of(i) + col0 + wc0 + cc;
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      const int rl = wr0 + i * 16 + k * RPP + cr;
      f32x4 v = *(const f32x4*)(c + (k * RPP + cr) * CP + cc);
      if (rl >= rows || wc0 + cc >= cols) continue;
      if (epi == EPI_RESID_F32) v = rv[i][k] + v;
      *(f32x4*)(dst + (k * RPP + cr) * ldo) = v;
    }
    wave_sync();
  }
}

// waves per SIMD by LDS
constexpr int waves_per_simd(int bm, int bn, int wn, int ns) {
  return 160 * 1024 / (ns * (bm + bn) * BK * 2) * 2 * wn / 4;
}

template <int BM, int BN, int WN, int NS, int AMN, int BMN>
__global__ __launch_bounds__(128 * WN, waves_per_simd(BM, BN, WN, NS)) void gemm_bf16_tile_kernel(GemmParams p) {
  tile_body<BM, BN, WN, NS, AMN, BMN, 0>(p, nullptr);
}

template <int BM, int BN, int WN, int NS>
__global__ __launch_bounds__(128 * WN, waves_per_simd(BM, BN, WN, NS))
void gemm_bf16_tile_parts_kernel(GemmParams p, GemmParts t) {
  tile_body<BM, BN, WN, NS, 0, 0, 1>(p, &t);
}

template <int BM, int BN, int WN, int NS>
hipError_t launch(const GemmParams& p, const GemmParts* t, hipStream_t s) {
  const dim3 grid((unsigned)((int64_t)p.tiles_m * p.tiles_n * p.nsplit)), block(128 * WN);
  if (t) hipLaunchKernelGGL((gemm_bf16_tile_parts_kernel<BM, BN, WN, NS>), grid, block, 0, s, p, *t);
  else if (p.a_mn && p.b_mn) hipLaunchKernelGGL((gemm_bf16_tile_kernel<BM, BN, WN, NS, 1, 1>), grid, block, 0, s, p);
  else if (p.b_mn) hipLaunchKernelGGL((gemm_bf16_tile_kernel<BM, BN, WN, NS, 0, 1>), grid, block, 0, s, p);
  else if (!p.a_mn) hipLaunchKernelGGL((gemm_bf16_tile_kernel<BM, BN, WN, NS, 0, 0>), grid, block, 0, s, p);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace

hipError_t launch_gemm_bf16_tile(const GemmParams& p, const GemmParts* t, hipStream_t s) {
  const int64_t nwg = (int64_t)p.tiles_m * p.tiles_n * p.nsplit;
  if (nwg <= 0 || nwg >= ((int64_t)1 << 31) || p.tail_parts > 1) return hipErrorInvalidValue;
  if (t && (p.nsplit != 1 || p.a_mn || p.b_mn || (t->a_rows && t->a_rows % 64) || (t->c_rows && t->c_rows % 16) ||
            (t->b_nrows && (t->b_nrows % 64 || t->b_kcols % 64 || t->b_nk < 1 || t->b_gstride < 0 ||
                            (p.ngroups > 1 && t->b_gstride == 0) ||
                            (int64_t)(p.ngroups - 1) * t->b_gstride +
                                    (int64_t)((p.N + t->b_nrows - 1) / t->b_nrows) * t->b_nk > kMaxParts))))
    return hipErrorInvalidValue;
  if (p.tile == 128) return nwg > 256 ? launch<128, 128, 2, 2>(p, t, s) : launch<128, 128, 4, 4>(p, t, s);
  if (p.tile == 64) return launch<64, 64, 2, 4>(p, t, s);
  return hipErrorInvalidValue;
}

}  // namespace partir
