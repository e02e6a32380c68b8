// Projections of the probe's decoder layer: C = A W^T with A [M][K] and the
// weight W [N][K] both K-contiguous, fused epilogues (residual adds, SwiGLU).
//
// bf16 path: fp16 activations A, bf16 weights, v_mfma_f32_16x16x32_f16 with
// fp32 accumulation.  A workgroup computes a BM x BN tile with WGM x WGN waves
// (each a (BM/WGM) x (BN/WGN) sub-tile) and consumes K in steps of BK (32 or
// 64: one or two MFMAs deep).  Each step's A and W tiles are loaded straight
// into LDS, S - 1 steps ahead of use, through an S-stage ring (one barrier per
// step; S = 2 is plain double buffering: the loads of step k + 1 are issued
// right after the barrier of step k and waited for before the next); weights stay bf16 in LDS and are converted exactly to fp16 (|w| in
// [2^-14, 65504]) as a wave reads its fragments.  A row of a stage tile is BK
// values = PPR 16-byte pieces; piece kp of row r sits at
//   r * PPR + (kp ^ ((r >> 1) & (PPR - 1)))
// which leaves the 16-byte fragment reads of 16 consecutive rows free of LDS
// bank conflicts for both PPR = 4 and 8 (the LDS bank-conflict counter reads 0;
// a shift of 2 for PPR = 4 measured conflicts on half the LDS cycles).
// SwiGLU: the BN weight rows of a tile alternate 16 gate rows and the 16
// matching up rows, so every lane holds gate and up of the same outputs.
// Split-K (PART, small M: the product then streams the weights with too few
// workgroups to keep enough loads in flight): blockIdx.y takes a slice of the
// K steps and writes its fp32 partial tile; gemm_reduce4 sums the slices in a
// fixed order and applies the epilogue.
// Weights come either as the caller's bf16 matrices (WBF16, converted per
// fragment) or as an fp16 image of them made once for the frozen head (no
// conversion: the same values, so the same results bit for bit).
// Tile order: workgroups are dealt to the XCDs round-robin (launch index mod
// the XCD count).  The launch index is re-mapped so that each XCD takes a
// contiguous run of a grouped tile order (group_m row tiles, then the next
// column tile): the workgroups that share an XCD's L2 at one time then cover a
// compact block of group_m row tiles by (CUs per XCD / group_m) column tiles,
// instead of every row tile of one column tile, and fetch far fewer operand
// bytes from beyond the L2 (27B-shaped gate/up on 8192 rows: 15% faster).
// K order: on the STREAM tiles each column tile starts its slice at another step and
// wraps round.  A product of few rows streams the weights, and workgroups in step
// all read the same K columns, whose lines lie a row (a multiple of 8 KB) apart
// and so crowd onto few memory channels; started apart they spread (128 rows,
// SwiGLU 24576 x 4096 in 128 x 96 tiles: 48.1 -> 42.5 us; 90 rows 46.7 -> 40.1).
// Products of many rows keep the common order, in which neighbours share operand
// lines in the L2.  Column tiles need not divide N: a last tile re-reads the
// last 32 columns in place of those past N and does not store them.
#include "common.h"
#include "kernels.h"

namespace sp {
namespace {

__device__ __forceinline__ float silu(float g) { return g / (1.0f + __expf(-g)); }

// Tile (m_tile, n_tile) of launch index L among nwg tiles (see the tile order above).
__device__ __forceinline__ void tile_of(int L, int nwg, int mtiles, int ntiles, int n_xcd, int group_m,
                                        int& m_tile, int& n_tile) {
  const int x = L % n_xcd, r = L / n_xcd;
  const int q = nwg / n_xcd, rem = nwg % n_xcd;
  const int t = (x < rem ? x * (q + 1) : rem * (q + 1) + (x - rem) * q) + r;
  const int per_group = group_m * ntiles;
  const int g = t / per_group, in = t - g * per_group;
  const int gm = min(group_m, mtiles - g * group_m);  // the last group may hold fewer row tiles
  m_tile = g * group_m + in % gm;
  n_tile = in / gm;
}

// STREAM: the tiles of few rows, with the K order by column tile and ragged columns.
template <int BM, int BN, int WGM, int WGN, int S, int BK, bool STREAM, int EPI, bool PART, bool WBF16>
__global__ __launch_bounds__(64 * WGM * WGN) void gemm_lds(const GemmParams p) {
  constexpr int NW = WGM * WGN, WM = BM / WGM, WN = BN / WGN, MT = WM / 16, NT = WN / 16;
  constexpr int PPR = BK / 8;                        // 16-byte pieces per tile row
  constexpr int RPI = 64 / PPR;                      // tile rows per 64-piece load
  constexpr int SWS = 1;                             // swizzle: kp ^ ((r >> SWS) & (PPR - 1))
  constexpr int NIA = BM / RPI, NI = NIA + BN / RPI;  // 64-piece loads per step
  constexpr int IPW = (NI + NW - 1) / NW;            // loads per wave per step
  constexpr int STAGE = (BM + BN) * PPR;             // pieces per stage
  static_assert(!STREAM || BN % 32 == 0, "ragged columns come 32 at a time");
  // SwiGLU on one row tile (the streaming tiles): the weights are read once, so
  // their loads are non-temporal and leave the activations in the L2 (16 rows,
  // 24576 x 4096: 37.3 -> 33.6 us; 128 rows: 42.5 -> 41.8; with K split it measured slower)
  constexpr bool WNT = STREAM && EPI == kEpiSwiglu && !PART && BM <= 128;
  static_assert(BK == 32 || BK == 64, "step depth");
  static_assert(WM % 16 == 0 && WN % 16 == 0, "wave tile");
  static_assert(S >= 2 && (S - 2) * IPW < 64, "stages");
  static_assert(EPI != kEpiSwiglu || WN % 32 == 0, "SwiGLU pairs 16 gate and 16 up columns");
  __shared__ u32x4 lds[S * STAGE];

  const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, la = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  __builtin_assume(wave >= 0 && wave < NW);
  const int wm = wave / WGN, wn = wave % WGN;

  const int mtiles = (p.M + BM - 1) / BM, ntiles = (p.N + BN - 1) / BN;
  int m_tile, n_tile;
  tile_of(blockIdx.x, gridDim.x, mtiles, ntiles, p.n_xcd, p.group_m, m_tile, n_tile);
  const int m0 = m_tile * BM, n0 = n_tile * BN;

  // This wave's loads: slots j*NW + wave (mod NI; a wave count that does not
  // divide NI re-issues a few slots with the same bytes).  Per slot: the
  // RPI-row block's base pointer (uniform), its place in the stage and the
  // lane's byte offset (fixed; each K step adds 2 BK bytes to the base).
  const char* gbase[IPW];
  int lds_piece[IPW];
  uint32_t lane_off[IPW];
  const int row_in = lane / PPR, kslot = lane % PPR;
#pragma unroll
  for (int j = 0; j < IPW; ++j) {
    const int sl = (j * NW + wave) % NI;
    const int blk = sl < NIA ? sl : sl - NIA;            // RPI-row block of the A or W tile
    const int kp = kslot ^ (((blk * RPI + row_in) >> SWS) & (PPR - 1));
    if (sl < NIA) {
      const int g = min(m0 + blk * RPI + row_in, p.M - 1);  // rows past M re-read row M-1; never stored
      gbase[j] = (const char*)p.a;
      lane_off[j] = (uint32_t)(g * p.lda * 2 + kp * 16);
      lds_piece[j] = blk * 64;
    } else {
      int src, row;
      const int r = blk * RPI, n = STREAM ? min(n0 + (r & ~31), p.N - 32) + (r & 31) : n0 + r;
      if (EPI == kEpiSwiglu) {  // an RPI-row block lies inside one 16-row gate or up group
        src = (n >> 4) & 1;
        row = 16 * (n >> 5) + (n & 15) + row_in;
      } else {  // b_split0/1 are multiples of 32
        src = n < p.b_split0 ? 0 : (n < p.b_split1 ? 1 : 2);
        row = n - (src == 0 ? 0 : (src == 1 ? p.b_split0 : p.b_split1)) + row_in;
      }
      gbase[j] = (const char*)(src == 0 ? p.b[0] : (src == 1 ? p.b[1] : p.b[2]));
      lane_off[j] = (uint32_t)(row * p.ldb * 2 + kp * 16);
      lds_piece[j] = BM * PPR + blk * 64;
    }
  }
  const int KT = p.K / BK;
  const int kb = (int)(((int64_t)KT * blockIdx.y) / gridDim.y);       // this slice's K steps
  const int ke = (int)(((int64_t)KT * (blockIdx.y + 1)) / gridDim.y);
  const int k_off = STREAM ? n_tile % (ke - kb) : 0;  // where in the slice this tile starts
  auto issue = [&](int kt, int stg) __attribute__((always_inline)) {
    if (STREAM) {
      kt += k_off;
      if (kt >= ke) kt -= ke - kb;
    }
#pragma unroll
    for (int j = 0; j < IPW; ++j) {
      const char* src = gbase[j] + kt * 2 * BK;
      u32x4* dst = &lds[stg * STAGE + lds_piece[j]];
      if (WNT && (j * NW + wave) % NI >= NIA) ld16_to_lds<true>(src, lane_off[j], dst);
      else ld16_to_lds<false>(src, lane_off[j], dst);
    }
  };

  f32x4 acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  // Steps past the last re-load the last one (into a stage no later step
  // reads), so every step issues the same loads and one vmcnt value fits all.
#pragma unroll
  for (int st = 0; st < S - 1; ++st) issue(min(kb + st, ke - 1), st);
  int stg = 0;
  for (int kt = kb; kt < ke; ++kt) {
    wait_vmcnt<(S - 2) * IPW>();  // this wave's loads of step kt have landed
    lds_barrier();                // everyone's have; everyone is done with step kt - 1
    issue(min(kt + S - 1, ke - 1), stg == 0 ? S - 1 : stg - 1);
    const u32x4* As = lds + stg * STAGE;
    const u32x4* Bs = As + BM * PPR;
#pragma unroll
    for (int ks = 0; ks < BK / 32; ++ks) {
      // piece 4 ks + la of rows 16x + li (the row's swizzle depends on li only)
      const int pc = (4 * ks + la) ^ ((li >> SWS) & (PPR - 1));
      f16x8 af[MT], bfr[NT];
#pragma unroll
      for (int i = 0; i < MT; ++i) af[i] = __builtin_bit_cast(f16x8, As[(wm * WM + 16 * i + li) * PPR + pc]);
#pragma unroll
      for (int j = 0; j < NT; ++j)
        bfr[j] = __builtin_bit_cast(f16x8, WBF16 ? bf16x8_to_f16x8(Bs[(wn * WN + 16 * j + li) * PPR + pc])
                                                 : Bs[(wn * WN + 16 * j + li) * PPR + pc]);
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = mfma16x16x32(af[i], bfr[j], acc[i][j]);
    }
    if constexpr (BK == 64 && !WBF16) {
      // Instruction order of the step: the first half-step's fragment reads,
      // then the second half-step's reads one by one between the first
      // half-step's products, then the remaining products.  Left to itself the
      // compiler issued the second reads only after every product of the first
      // half, so each step waited out an LDS round trip with the matrix cores
      // idle (27B-shaped gate/up 2.30 -> 2.23 ms, o and down 2-3% faster).
      constexpr int NF = MT + NT, NM = MT * NT;
      __builtin_amdgcn_sched_group_barrier(0x100, NF, 0);  // 0x100: LDS reads
#pragma unroll
      for (int f = 0; f < NF; ++f) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // 0x008: MFMA
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      }
      __builtin_amdgcn_sched_group_barrier(0x008, 2 * NM - NF, 0);
    }
    stg = stg == S - 1 ? 0 : stg + 1;
  }
  wait_vmcnt<0>();

  // Lane holds C[16i + 4la + r][16j + li] of the wave tile.
  bool oor = false;  // an fp16 SwiGLU output out of fp16's range
  const int cols = STREAM ? p.N - n0 - wn * WN : WN;  // columns from the wave's first to the last
#pragma unroll
  for (int i = 0; i < MT; ++i) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = m0 + wm * WM + 16 * i + 4 * la + r;
      if (m >= p.M) continue;
      if (PART) {
        float* prow = p.part + ((int64_t)blockIdx.y * p.M + m) * p.N + n0 + wn * WN + li;
#pragma unroll
        for (int j = 0; j < NT; ++j)
          if (16 * j < cols) prow[16 * j] = acc[i][j][r];
      } else if (EPI == kEpiSwiglu) {
#pragma unroll
        for (int j = 0; j < NT; j += 2) {
          if (16 * j >= cols) continue;
          const int pair = (wn * WN + 16 * j) >> 5;
          const int n = n_tile * (BN / 2) + 16 * pair + li;
          const float gt = acc[i][j][r], up = acc[i][j + 1][r];
          const float v = silu(gt) * up;
          oor |= !(fabsf(v) <= 65504.0f);
          ((f16*)p.c)[(int64_t)m * p.ldc + n] = (f16)v;
        }
      } else {
#pragma unroll
        for (int j = 0; j < NT; ++j) {
          if (16 * j >= cols) continue;
          const int n = n0 + wn * WN + 16 * j + li;
          float v = acc[i][j][r];
          if (EPI == kEpiResidRow)
            v += (float)((const bf16*)p.r)[(int64_t)(m % p.r_mod) * p.r_ld + n];
          else if (EPI == kEpiResidF32)
            v += ((const float*)p.r)[(int64_t)m * p.r_ld + n];
          else if (EPI == kEpiRowScale)
            v *= ((const float*)p.r)[m];
          ((float*)p.c)[(int64_t)m * p.ldc + n] = v;
        }
      }
    }
  }
  if (EPI == kEpiSwiglu && !PART && __any(oor) && lane == 0 && p.status) atomicOr(p.status, kStatusRange);
}

// ---------------------------------------------------------------- few rows
// C = A W^T on at most 16 rows (or few 16-row tiles of small matrices, one per
// blockIdx.y): bound by the read of the weights, so the kernel is a reader of W
// with matrix-core products.  One workgroup takes 16 weight rows (SwiGLU: 16
// gate rows and the 16 matching up rows) over the whole of K; its NW
// waves take contiguous slices of K, load their A and W fragments straight into
// registers (16 bytes per lane; no wave shares a fragment with another, so LDS
// would only add a copy) U steps of 32 ahead, and the partial tiles are summed in
// wave order through LDS.  Every output column then has NW waves of loads in
// flight, without partial sums in memory or a second launch.
// Measured, fp16 weights, against one wave per 16 columns through an LDS ring: 5
// rows, 4096 x 4096 13.0 -> 10.2 us, 4096 x 12288 30.6 -> 21.5 us (4.7 TB/s, launch
// included), 2560 x 9728 22.7 -> 16.6 us.  What is left over the read is the A
// fragments, which every workgroup fetches from its L2 (1 row takes 2-3 us less
// than 8), so wide SwiGLU and more rows are faster on the streaming tiles (see
// stream_choice).  Several row tiles: 20 rows of 512 x 768 10.0 us as four 32 x 128
// tiles, 5.6 us here.
// PK = 2 (at most 8 rows): a 16-row A fragment would be half repeats, so one load
// brings two steps of the 8 rows (lanes li 0-7 the even step, 8-15 the odd one)
// and the odd step's product takes the fragment rotated by 8 rows; rows 8-15 of
// the product are never stored.
__device__ __forceinline__ u32x4 rotate_8_rows(u32x4 v) {  // lane li of each 16 takes lane (li + 8) % 16
  u32x4 o;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    o[i] = (unsigned)__builtin_amdgcn_update_dpp(0, (int)v[i], 0x128, 0xf, 0xf, false);  // row_ror:8
  return o;
}

template <int NW, int U, int PK, int EPI, bool WBF16>
__global__ __launch_bounds__(64 * NW) void gemm_rows(const GemmParams p) {
  static_assert((PK == 1 || PK == 2) && U % PK == 0, "packed steps");
  constexpr int NT = EPI == kEpiSwiglu ? 2 : 1;  // 16-row weight tiles
  constexpr int RP = 16 / PK;                    // rows of A held per step
  __shared__ f32x4 red[NW][NT][64];
  const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, la = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int KT = p.K / 32, KP = (KT + 1) / 2;  // steps of 32; pairs of steps (whole 128-byte lines of W)
  const int kb = 2 * (KP * wave / NW), ke = min(KT, 2 * (KP * (wave + 1) / NW));

  const int m0 = 16 * blockIdx.y;
  // rows past M read row M - 1 again; never stored
  const uint16_t* ap = (const uint16_t*)p.a + (int64_t)min(m0 + li % RP, p.M - 1) * p.lda + 8 * la;
  const uint16_t* wp[NT];
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    const int n = 16 * blockIdx.x;  // a 16-column tile lies inside one block of weight rows
    const int src = EPI == kEpiSwiglu ? j : n < p.b_split0 ? 0 : (n < p.b_split1 ? 1 : 2);
    const int row = n - (EPI == kEpiSwiglu || src == 0 ? 0 : (src == 1 ? p.b_split0 : p.b_split1));
    const void* b = src == 0 ? p.b[0] : (src == 1 ? p.b[1] : p.b[2]);
    wp[j] = (const uint16_t*)b + (int64_t)(row + li) * p.ldb + 8 * la;
  }

  f32x4 acc[NT];
#pragma unroll
  for (int j = 0; j < NT; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};

  struct Frag { u32x4 a[U / PK], w[U][NT]; };
  Frag f0, f1;
  auto load = [&](Frag& f, int k) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int kk = 32 * min(k + u, ke - 1);  // steps past the slice re-read its last one, unused
#pragma unroll
      for (int j = 0; j < NT; ++j) f.w[u][j] = ld16v(wp[j] + kk);
    }
#pragma unroll
    for (int u = 0; u < U / PK; ++u) f.a[u] = ld16v(ap + 32 * min(k + PK * u + li / RP, ke - 1));
  };
  auto mul = [&](const Frag& f, int k) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (k + u >= ke) break;
      const f16x8 a = __builtin_bit_cast(f16x8, u % PK == 0 ? f.a[u / PK] : rotate_8_rows(f.a[u / PK]));
#pragma unroll
      for (int j = 0; j < NT; ++j)
        acc[j] = mfma16x16x32(a, __builtin_bit_cast(f16x8, WBF16 ? bf16x8_to_f16x8(f.w[u][j]) : f.w[u][j]), acc[j]);
    }
  };
  if (kb < ke) {
    load(f0, kb);
    for (int k = kb; k < ke; k += 2 * U) {
      if (k + U < ke) load(f1, k + U);
      mul(f0, k);
      if (k + 2 * U < ke) load(f0, k + 2 * U);
      if (k + U < ke) mul(f1, k + U);
    }
  }

#pragma unroll
  for (int j = 0; j < NT; ++j) red[wave][j][lane] = acc[j];
  __syncthreads();
  if (wave > 0) return;
  // lane holds C[m0 + 4la + r][16 blockIdx.x + li]
  f32x4 v[NT];
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    v[j] = acc[j];
    for (int w = 1; w < NW; ++w) v[j] += red[w][j][lane];
  }
  bool oor = false;
  const int n = 16 * blockIdx.x + li;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int m = m0 + 4 * la + r;
    if (m >= p.M) continue;
    if (EPI == kEpiSwiglu) {
      const float s = silu(v[0][r]) * v[NT - 1][r];
      oor |= !(fabsf(s) <= 65504.0f);
      ((f16*)p.c)[(int64_t)m * p.ldc + n] = (f16)s;
    } else {
      float x = v[0][r];
      if (EPI == kEpiResidRow)
        x += (float)((const bf16*)p.r)[(int64_t)(m % p.r_mod) * p.r_ld + n];
      else if (EPI == kEpiResidF32)
        x += ((const float*)p.r)[(int64_t)m * p.r_ld + n];
      else if (EPI == kEpiRowScale)
        x *= ((const float*)p.r)[m];
      ((float*)p.c)[(int64_t)m * p.ldc + n] = x;
    }
  }
  if (EPI == kEpiSwiglu && __any(oor) && lane == 0 && p.status) atomicOr(p.status, kStatusRange);
}

template <int NW, int U, int PK, int EPI>
hipError_t launch_rows(const GemmParams& p, hipStream_t s) {
  constexpr int cols = EPI == kEpiSwiglu ? 32 : 16;
  if (p.M < 1 || (PK == 2 && p.M > 8) || p.K % 32 || p.N % cols) return hipErrorInvalidValue;
  if (EPI != kEpiSwiglu && (p.b_split0 % 16 || p.b_split1 % 16)) return hipErrorInvalidValue;
  const dim3 block(64 * NW), grid(p.N / cols, (p.M + 15) / 16);
  if (p.b_f16) hipLaunchKernelGGL((gemm_rows<NW, U, PK, EPI, false>), grid, block, 0, s, p);
  else hipLaunchKernelGGL((gemm_rows<NW, U, PK, EPI, true>), grid, block, 0, s, p);
  return hipGetLastError();
}

// Up to 8 rows: packed A fragments.  The wave counts and depths are the fastest
// measured of 2-16 waves, 4 or 8 steps and one or two weight tiles.
template <int EPI>
hipError_t launch_rows_any(const GemmParams& p, hipStream_t s) {
  if constexpr (EPI == kEpiSwiglu) return p.M <= 8 ? launch_rows<4, 4, 2, EPI>(p, s) : launch_rows<4, 4, 1, EPI>(p, s);
  else return p.M <= 8 ? launch_rows<4, 8, 2, EPI>(p, s) : launch_rows<8, 4, 1, EPI>(p, s);
}

hipError_t launch_gemm_rows(Epilogue epi, const GemmParams& p, hipStream_t s) {
  switch (epi) {
    case kEpiStore: return launch_rows_any<kEpiStore>(p, s);
    case kEpiResidRow: return launch_rows_any<kEpiResidRow>(p, s);
    case kEpiResidF32: return launch_rows_any<kEpiResidF32>(p, s);
    case kEpiRowScale: return launch_rows_any<kEpiRowScale>(p, s);
    case kEpiSwiglu: return launch_rows_any<kEpiSwiglu>(p, s);
  }
  return hipErrorInvalidValue;
}

// ---------------------------------------------------------------- fp32 path
// C = A W^T in fp32 throughout (fp32 matrix-core products, whose A and B fragments
// are one value per lane).  One workgroup takes 16 MT rows by 16 outputs (SwiGLU: 16
// gate and the 16 matching up rows of W) over the whole of K, its NW waves
// contiguous slices of K, summed in wave order through LDS, as gemm_rows does.
// Lane (li, la) loads four consecutive k of row li (16 bytes) and element e feeds
// product e: the four lanes of a product then hold k = 16 j + 4 la + e of step j, the
// same k in A and W.  The small fp32 heads are bound by latency: a thread per
// output walking K took 35-124 us a product on 16 rows (256 to 1024 deep), this
// 3-5 us.
template <int MT, int NW, int EPI>
__global__ __launch_bounds__(64 * NW) void gemm_f32(const GemmParams p) {
  constexpr int NT = EPI == kEpiSwiglu ? 2 : 1, U = 4;
  __shared__ f32x4 red[NW][MT * NT][64];
  const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, la = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n_out = EPI == kEpiSwiglu ? p.N / 2 : p.N;
  const int n0 = 16 * blockIdx.x;
  const int64_t m_first = (int64_t)16 * MT * (blockIdx.y + (int64_t)gridDim.y * blockIdx.z);
  if (m_first >= p.M) return;  // the grid's last layer may be partial
  const int m0 = (int)m_first;
  const int KT = (p.K + 15) / 16, kb = KT * wave / NW, ke = KT * (wave + 1) / NW;

  const float* ap[MT];
  const float* wp[NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)  // rows past M and outputs past n_out re-read the last; never stored
    ap[i] = (const float*)p.a + (int64_t)min(m0 + 16 * i + li, p.M - 1) * p.lda;
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    const int n = min(n0 + li, n_out - 1);
    const int src = EPI == kEpiSwiglu ? j : n < p.b_split0 ? 0 : (n < p.b_split1 ? 1 : 2);
    const int row = n - (EPI == kEpiSwiglu || src == 0 ? 0 : (src == 1 ? p.b_split0 : p.b_split1));
    const void* b = src == 0 ? p.b[0] : (src == 1 ? p.b[1] : p.b[2]);
    wp[j] = (const float*)b + (int64_t)row * p.ldb;
  }

  f32x4 acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int k0 = kb; k0 < ke; k0 += U) {
    f32x4 a[U][MT], w[U][NT];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = 16 * (k0 + u) + 4 * la;
      const bool in = k0 + u < ke && k < p.K;  // K % 4 == 0: a lane's four k are all in or all out
      const int kk = in ? k : 0;
#pragma unroll
      for (int j = 0; j < NT; ++j) {
        w[u][j] = *reinterpret_cast<const f32x4*>(wp[j] + kk);
        if (!in) w[u][j] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        a[u][i] = *reinterpret_cast<const f32x4*>(ap[i] + kk);
        if (!in) a[u][i] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
          for (int j = 0; j < NT; ++j) acc[i][j] = mfma16x16x4_f32(a[u][i][e], w[u][j][e], acc[i][j]);
  }
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) red[wave][i * NT + j][lane] = acc[i][j];
  __syncthreads();

  // lane holds C[m0 + 16i + 4la + r][n0 + li]; wave w finishes row tiles w, w + NW, ...
  const int n = n0 + li;
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    if (i % NW != wave || n >= n_out) continue;
    f32x4 v[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      v[j] = red[0][i * NT + j][lane];
      for (int w = 1; w < NW; ++w) v[j] += red[w][i * NT + j][lane];
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = m0 + 16 * i + 4 * la + r;
      if (m >= p.M) continue;
      float x = v[0][r];
      if (EPI == kEpiSwiglu) x = x / (1.0f + expf(-x)) * v[NT - 1][r];
      if (EPI == kEpiResidRow) x += ((const float*)p.r)[(int64_t)(m % p.r_mod) * p.r_ld + n];
      if (EPI == kEpiResidF32) x += ((const float*)p.r)[(int64_t)m * p.r_ld + n];
      if (EPI == kEpiRowScale) x *= ((const float*)p.r)[m];
      ((float*)p.c)[(int64_t)m * p.ldc + n] = x;
    }
  }
}

// Four row tiles per workgroup (each weight fragment then serves 64 rows) where
// that still leaves a workgroup per compute unit, else one.  Row tiles past the
// 65535 of the grid's y go to further layers in z.
template <int EPI>
hipError_t launch_f32(const GemmParams& p, hipStream_t s) {
  if (p.K % 4 || p.lda % 4 || p.ldb % 4) return hipErrorInvalidValue;
  const int n_out = EPI == kEpiSwiglu ? p.N / 2 : p.N, cols = (n_out + 15) / 16;
  const int cus = p.n_cus > 0 ? p.n_cus : 256;
  const bool four = p.M > 16 && (int64_t)cols * (((int64_t)p.M + 63) / 64) >= cus;
  const int64_t tiles = ((int64_t)p.M + (four ? 63 : 15)) / (four ? 64 : 16);
  const dim3 grid(cols, (unsigned)std::min<int64_t>(tiles, 65535), (unsigned)((tiles + 65534) / 65535)), block(512);
  if (four) hipLaunchKernelGGL((gemm_f32<4, 8, EPI>), grid, block, 0, s, p);
  else hipLaunchKernelGGL((gemm_f32<1, 8, EPI>), grid, block, 0, s, p);
  return hipGetLastError();
}

// Sum of the split-K slices and the epilogue, four consecutive outputs per thread
// (16-byte partial loads) and one output row per blockIdx.y.  SwiGLU: output o of
// tile o / (bn/2) has its gate column 32 ((o % (bn/2)) / 16) + o % 16 in the tile's
// interleaved columns and its up column 16 later.
template <int EPI>
__global__ __launch_bounds__(256) void gemm_reduce4(const GemmParams p, int ksplit, int bn) {
  const int n_out = EPI == kEpiSwiglu ? p.N / 2 : p.N;
  const int m = blockIdx.y, o = 4 * (blockIdx.x * 256 + threadIdx.x);
  if (o >= n_out) return;
  const int64_t slice = (int64_t)p.M * p.N;
  const float* src = p.part + (int64_t)m * p.N;
  if (EPI == kEpiSwiglu) {
    const int w = o % (bn / 2);  // o % 4 == 0: the four outputs share one 16-column group
    const int g = (o / (bn / 2)) * bn + 32 * (w / 16) + w % 16;
    float4 gt = make_float4(0.f, 0.f, 0.f, 0.f), up = gt;
    for (int k = 0; k < ksplit; ++k) {
      const float4 a = *reinterpret_cast<const float4*>(src + k * slice + g);
      const float4 u = *reinterpret_cast<const float4*>(src + k * slice + g + 16);
      gt.x += a.x; gt.y += a.y; gt.z += a.z; gt.w += a.w;
      up.x += u.x; up.y += u.y; up.z += u.z; up.w += u.w;
    }
    const float v[4] = {silu(gt.x) * up.x, silu(gt.y) * up.y, silu(gt.z) * up.z, silu(gt.w) * up.w};
    f16x4 h;
    bool oor = false;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      h[e] = (f16)v[e];
      oor |= !(fabsf(v[e]) <= 65504.0f);
    }
    *reinterpret_cast<f16x4*>((f16*)p.c + (int64_t)m * p.ldc + o) = h;
    if (oor && p.status) atomicOr(p.status, kStatusRange);
    return;
  }
  float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int k = 0; k < ksplit; ++k) {
    const float4 a = *reinterpret_cast<const float4*>(src + k * slice + o);
    v.x += a.x; v.y += a.y; v.z += a.z; v.w += a.w;
  }
  if (EPI == kEpiResidRow) {
    const bf16* rr = (const bf16*)p.r + (int64_t)(m % p.r_mod) * p.r_ld + o;
    v.x += (float)rr[0]; v.y += (float)rr[1]; v.z += (float)rr[2]; v.w += (float)rr[3];
  }
  if (EPI == kEpiResidF32) {
    const float4 r = *reinterpret_cast<const float4*>((const float*)p.r + (int64_t)m * p.r_ld + o);
    v.x += r.x; v.y += r.y; v.z += r.z; v.w += r.w;
  }
  if (EPI == kEpiRowScale) {
    const float sc = ((const float*)p.r)[m];
    v.x *= sc; v.y *= sc; v.z *= sc; v.w *= sc;
  }
  *reinterpret_cast<float4*>((float*)p.c + (int64_t)m * p.ldc + o) = v;
}

// The same sums with the row's RMSNorm (or two in a row) after them: one workgroup
// per row, one thread per four values (CH chunks of blockDim of them), so that a
// row's slices are all requested at once and the row stays in registers between
// the sum and the norm.  Bound by launch and load latency: one launch less than
// gemm_reduce4 and rmsnorm_rows (128 rows of 4096, four slices: 9.6 us for the
// two, 6.0 us here).
template <int EPI, int CH>
__global__ __launch_bounds__(1024) void gemm_reduce_norm(const GemmParams p, int ksplit) {
  __shared__ float red[2][16];
  const int m = blockIdx.x, d = p.N, T = blockDim.x, tid = threadIdx.x;
  const int64_t slice = (int64_t)p.M * d;
  const float* src = p.part + (int64_t)m * d;
  f32x4 v[CH], g[CH];
  auto load_gain = [&](const void* gain) __attribute__((always_inline)) {
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const int i = 4 * (tid + T * c);
      if (i < d) {
        const bf16x4 h = *reinterpret_cast<const bf16x4*>((const bf16*)gain + i);
        g[c] = f32x4{(float)h[0], (float)h[1], (float)h[2], (float)h[3]};
      }
    }
  };
  auto row_sum = [&](float x, float* r) __attribute__((always_inline)) {
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
    if ((tid & 63) == 0) r[tid >> 6] = x;
    __syncthreads();
    float s = r[0];
    for (int w = 1; w < T / 64; ++w) s += r[w];
    return s;
  };
  f32x4 res[CH];
#pragma unroll
  for (int c = 0; c < CH; ++c) {
    const int i = 4 * (tid + T * c);
    v[c] = res[c] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (i >= d) continue;
    if (EPI == kEpiResidRow) {
      const bf16x4 r = *reinterpret_cast<const bf16x4*>((const bf16*)p.r + (int64_t)(m % p.r_mod) * p.r_ld + i);
      res[c] = f32x4{(float)r[0], (float)r[1], (float)r[2], (float)r[3]};
    }
    if (EPI == kEpiResidF32) res[c] = *reinterpret_cast<const f32x4*>((const float*)p.r + (int64_t)m * p.r_ld + i);
  }
  load_gain(p.norm_gain);
  for (int k0 = 0; k0 < ksplit; k0 += 4) {
    f32x4 t[4][CH];
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int c = 0; c < CH; ++c)
        if (k0 + q < ksplit && 4 * (tid + T * c) < d)
          t[q][c] = *reinterpret_cast<const f32x4*>(src + (k0 + q) * slice + 4 * (tid + T * c));
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int c = 0; c < CH; ++c)
        if (k0 + q < ksplit && 4 * (tid + T * c) < d) v[c] += t[q][c];
  }
  float ss = 0.f;
#pragma unroll
  for (int c = 0; c < CH; ++c) {
    const int i = 4 * (tid + T * c);
    if (i >= d) continue;
    v[c] += res[c];
    *reinterpret_cast<f32x4*>((float*)p.c + (int64_t)m * p.ldc + i) = v[c];
#pragma unroll
    for (int e = 0; e < 4; ++e) ss += v[c][e] * v[c][e];
  }
  float inv = 1.0f / sqrtf(row_sum(ss, red[0]) / (float)d + p.norm_eps);
  for (int pass = 0; pass < (p.norm_gain2 ? 2 : 1); ++pass) {
    float ss2 = 0.f;
    if (pass) load_gain(p.norm_gain2);
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      if (4 * (tid + T * c) >= d) continue;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        v[c][e] = v[c][e] * inv * g[c][e];
        ss2 += v[c][e] * v[c][e];
      }
    }
    if (p.norm_gain2 && pass == 0) inv = 1.0f / sqrtf(row_sum(ss2, red[1]) / (float)d + p.norm_eps);
  }
  bool oor = false;
#pragma unroll
  for (int c = 0; c < CH; ++c) {
    const int i = 4 * (tid + T * c);
    if (i >= d) continue;
    f16x4 h;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      h[e] = (f16)v[c][e];
      oor |= !(fabsf(v[c][e]) <= 65504.0f);
    }
    *reinterpret_cast<f16x4*>((f16*)p.norm_out + (int64_t)m * p.norm_ld + i) = h;
  }
  if (__any(oor) && (tid & 63) == 0 && p.status) atomicOr(p.status, kStatusRange);
}

template <int EPI>
hipError_t launch_reduce_norm(const GemmParams& p, int ksplit, hipStream_t s) {
  const int ch = (p.N + 4095) / 4096, t = (p.N / 4 + ch - 1) / ch;
  const dim3 grid(p.M), block((t + 63) / 64 * 64);
  if (ch == 1) hipLaunchKernelGGL((gemm_reduce_norm<EPI, 1>), grid, block, 0, s, p, ksplit);
  else hipLaunchKernelGGL((gemm_reduce_norm<EPI, 2>), grid, block, 0, s, p, ksplit);
  return hipGetLastError();
}

// What launch_gemm asks of a tile; the kernels of the rest are not built.
enum : int { kGate = 1, kGateSplit = 2, kPlain = 4, kPlainSplit = 8 };  // SwiGLU, the other epilogues; with K split

template <int BM, int BN, int WGM, int WGN, int S, int BK, int USE, bool ST, bool PART, bool WB>
hipError_t launch_tile_k(Epilogue epi, const GemmParams& p, dim3 grid, hipStream_t s) {
  const dim3 block(64 * WGM * WGN);
  if (epi == kEpiSwiglu) {
    if constexpr ((USE & (PART ? kGateSplit : kGate)) != 0) {
      static_assert((BN / WGN) % 32 == 0, "a wave holds whole pairs of gate and up columns");
      hipLaunchKernelGGL((gemm_lds<BM, BN, WGM, WGN, S, BK, ST, kEpiSwiglu, PART, WB>), grid, block, 0, s, p);
      return hipGetLastError();
    }
  } else if constexpr ((USE & (PART ? kPlainSplit : kPlain)) != 0) {
    if constexpr (PART) {  // the reduction applies the epilogue
      hipLaunchKernelGGL((gemm_lds<BM, BN, WGM, WGN, S, BK, ST, kEpiStore, PART, WB>), grid, block, 0, s, p);
    } else {
      switch (epi) {
        case kEpiStore: hipLaunchKernelGGL((gemm_lds<BM, BN, WGM, WGN, S, BK, ST, kEpiStore, PART, WB>), grid, block, 0, s, p); break;
        case kEpiResidRow: hipLaunchKernelGGL((gemm_lds<BM, BN, WGM, WGN, S, BK, ST, kEpiResidRow, PART, WB>), grid, block, 0, s, p); break;
        case kEpiResidF32: hipLaunchKernelGGL((gemm_lds<BM, BN, WGM, WGN, S, BK, ST, kEpiResidF32, PART, WB>), grid, block, 0, s, p); break;
        case kEpiRowScale: hipLaunchKernelGGL((gemm_lds<BM, BN, WGM, WGN, S, BK, ST, kEpiRowScale, PART, WB>), grid, block, 0, s, p); break;
        case kEpiSwiglu: break;
      }
    }
    return hipGetLastError();
  }
  return hipErrorInvalidValue;
}

hipError_t launch_gemm_reduce(Epilogue epi, const GemmParams& p, int ksplit, int bn, hipStream_t s);

// K split ksplit ways (ksplit > 1: fp32 partials in p.part, then the reduction).
// BM_WAVES x BN_WAVES: the waves of a workgroup for weights as stored.  Each wave
// converts the columns it holds, so where WGN is 1 all WGM waves of a tile would convert
// all of its columns: 192 rows of 34816 x 5120 in 256 x 160 tiles took 491 us in 8 x 1
// waves and 109 in 2 x 5 (fp16 image, 8 x 1: 112); 128 x 160, 128 rows of 24576 x 4096, 80.6 and
// 58.2; 64 x 160, 58.7 and 46.0 on 33 rows; 128 x 96, 52.1 and 47.3.  The fp16 image is as
// fast or faster in the first layout.  Every output is the same sum in either.
template <int BM, int BN, int WGM, int WGN, int S, int BK, int USE, bool ST = false, int BM_WAVES = WGM, int BN_WAVES = WGN>
hipError_t launch_tile(Epilogue epi, const GemmParams& p, int ksplit, hipStream_t s) {
  if (p.K % BK || p.K / BK < ksplit) return hipErrorInvalidValue;  // slices of whole steps, maybe uneven
  const dim3 grid(((p.M + BM - 1) / BM) * ((p.N + BN - 1) / BN), ksplit);
  hipError_t e;
  if (ksplit > 1)
    e = p.b_f16 ? launch_tile_k<BM, BN, WGM, WGN, S, BK, USE, ST, true, false>(epi, p, grid, s)
                : launch_tile_k<BM, BN, BM_WAVES, BN_WAVES, S, BK, USE, ST, true, true>(epi, p, grid, s);
  else
    e = p.b_f16 ? launch_tile_k<BM, BN, WGM, WGN, S, BK, USE, ST, false, false>(epi, p, grid, s)
                : launch_tile_k<BM, BN, BM_WAVES, BN_WAVES, S, BK, USE, ST, false, true>(epi, p, grid, s);
  if (e != hipSuccess || ksplit == 1) return e;
  return launch_gemm_reduce(epi, p, ksplit, BN, s);
}

// Tile shapes (BM, BN, waves along M, waves along N, K-step depth); the stage
// counts are in launch_tile_index.  The residual epilogues (o, down) prefer
// 256 x 128 tiles with 64-deep steps, which at 2048-8192 rows take half the
// time of 128 x 64.  Index 9 is the 32 x 128 tile of the 17-32-row products.
// Index 10 is 256 x 256 with 64-deep steps, double-buffered (two 64 KB stages):
// 64-deep steps halve the barriers per unit of K and load whole 128-byte rows
// per step (32-deep steps load half rows, and with them half cache lines), and
// more stages measured no faster (SwiGLU, fp16 weights, 8192 x 34816 x 5120:
// 2.35 ms against 2.59 ms for 256 x 256 in 32-deep steps; 2048 x 24576 x 4096:
// 0.335 ms against 0.368 ms).  Index 11 is 256 x 160 in three 52 KB stages, for
// residual products whose 256 x 256 or 256 x 128 grids end in a partial round
// (8192 x 5120: 1024 tiles, four whole rounds); index 12 is 256 x 192 with
// 64-deep steps, double-buffered, for SwiGLU grids of one round (512 x 24576 x
// 4096: 119 us against 124 us in 32-deep steps).  Index 13 is 256 x 160 for SwiGLU
// grids that it puts in fewer rounds (256 x 34816 x 5120: 113 us, one round of 218,
// against 140; 512 x 19456 x 2560: 56 against 71).  From there (kStreamTiles) on the
// tiles are STREAM ones; those after it serve products of at most 256 rows (see
// stream_choice), with as many 64-deep stages as fit in LDS.
struct TileShape { int bm, bn, wgm, wgn, bk; };
constexpr int kNumTiles = 28, kStreamTiles = 13, kRaggedWide = 13;
constexpr TileShape kTiles[kNumTiles] = {
    {256, 256, 2, 4, 32}, {256, 192, 4, 2, 32}, {256, 128, 4, 2, 64}, {128, 64, 4, 2, 64},
    {64, 64, 2, 2, 64},   {32, 64, 1, 2, 64},   {16, 32, 1, 1, 64},  {16, 16, 1, 1, 64},
    {16, 32, 1, 1, 32},   {32, 128, 1, 4, 64},  {256, 256, 4, 2, 64}, {256, 160, 4, 2, 64},
    {256, 192, 4, 2, 64}, {256, 160, 8, 1, 64},
    {16, 64, 1, 4, 64},   {16, 96, 1, 3, 64},   {16, 160, 1, 5, 64},  {32, 96, 2, 1, 64},  {32, 160, 1, 5, 64},
    {64, 64, 2, 2, 64},   {64, 96, 4, 1, 64},   {64, 128, 2, 4, 64},  {64, 160, 4, 1, 64}, {128, 96, 4, 1, 64},
    {128, 128, 2, 4, 64}, {128, 160, 4, 1, 64}, {32, 128, 1, 4, 64},  {128, 64, 4, 2, 64}};
constexpr int kOrderSwiglu[9] = {0, 1, 2, 3, 4, 5, 6, 7, 8};
constexpr int kOrderResid[9] = {2, 1, 0, 3, 4, 5, 6, 7, 8};

bool tile_ok(const GemmParams& p, Epilogue epi, const TileShape& t) {
  const int unit = &t >= &kTiles[kStreamTiles] ? 32 : t.bn;  // ragged columns
  if (p.N % unit || p.K % t.bk) return false;
  if (epi == kEpiSwiglu) return (t.bn / t.wgn) % 32 == 0;
  return p.b_split0 % unit == 0 && p.b_split1 % unit == 0;
}

hipError_t launch_tile_index(int c, Epilogue epi, const GemmParams& p, int ksplit, hipStream_t s) {
  switch (c) {
    case 0: return launch_tile<256, 256, 2, 4, 3, 32, kPlain | kGate>(epi, p, ksplit, s);
    case 1: return launch_tile<256, 192, 4, 2, 3, 32, kPlain | kGate>(epi, p, ksplit, s);
    case 2: return launch_tile<256, 128, 4, 2, 3, 64, kPlain | kPlainSplit | kGate>(epi, p, ksplit, s);
    case 3: return launch_tile<128, 64, 4, 2, 6, 64, kPlain | kPlainSplit | kGate>(epi, p, ksplit, s);
    case 4: return launch_tile<64, 64, 2, 2, 8, 64, kPlain | kGate>(epi, p, ksplit, s);
    case 5: return launch_tile<32, 64, 1, 2, 8, 64, kPlain | kGate>(epi, p, ksplit, s);
    case 6: return launch_tile<16, 32, 1, 1, 8, 64, kPlain | kGate>(epi, p, ksplit, s);
    case 7: return launch_tile<16, 16, 1, 1, 8, 64, kPlain>(epi, p, ksplit, s);
    case 8: return launch_tile<16, 32, 1, 1, 8, 32, kPlain | kGate>(epi, p, ksplit, s);
    case 9: return launch_tile<32, 128, 1, 4, 6, 64, kPlain | kPlainSplit | kGate | kGateSplit>(epi, p, ksplit, s);
    case 10: return launch_tile<256, 256, 4, 2, 2, 64, kPlain | kPlainSplit | kGate>(epi, p, ksplit, s);
    case 11: return launch_tile<256, 160, 4, 2, 3, 64, kPlain>(epi, p, ksplit, s);
    case 12: return launch_tile<256, 192, 4, 2, 2, 64, kGate>(epi, p, ksplit, s);
    case 13: return launch_tile<256, 160, 8, 1, 3, 64, kGate, true, 2, 5>(epi, p, ksplit, s);
    case 14: return launch_tile<16, 64, 1, 4, 14, 64, kPlain | kPlainSplit, true>(epi, p, ksplit, s);
    case 15: return launch_tile<16, 96, 1, 3, 10, 64, kGate, true>(epi, p, ksplit, s);
    case 16: return launch_tile<16, 160, 1, 5, 7, 64, kGate, true>(epi, p, ksplit, s);
    case 17: return launch_tile<32, 96, 2, 1, 8, 64, kGate, true, 1, 3>(epi, p, ksplit, s);
    case 18: return launch_tile<32, 160, 1, 5, 6, 64, kPlain | kPlainSplit | kGate, true>(epi, p, ksplit, s);
    case 19: return launch_tile<64, 64, 2, 2, 8, 64, kPlain | kPlainSplit, true>(epi, p, ksplit, s);
    case 20: return launch_tile<64, 96, 4, 1, 7, 64, kPlain | kPlainSplit | kGate, true, 1, 3>(epi, p, ksplit, s);
    case 21: return launch_tile<64, 128, 2, 4, 6, 64, kPlain | kPlainSplit, true>(epi, p, ksplit, s);
    case 22: return launch_tile<64, 160, 4, 1, 5, 64, kPlain | kPlainSplit | kGate, true, 2, 5>(epi, p, ksplit, s);
    case 23: return launch_tile<128, 96, 4, 1, 5, 64, kPlain | kPlainSplit | kGate, true, 2, 3>(epi, p, ksplit, s);
    case 24: return launch_tile<128, 128, 2, 4, 5, 64, kPlain | kPlainSplit, true>(epi, p, ksplit, s);
    case 25: return launch_tile<128, 160, 4, 1, 4, 64, kPlain | kPlainSplit | kGate, true, 2, 5>(epi, p, ksplit, s);
    case 26: return launch_tile<32, 128, 1, 4, 6, 64, kPlain | kPlainSplit, true>(epi, p, ksplit, s);
    case 27: return launch_tile<128, 64, 4, 2, 6, 64, kPlain | kPlainSplit, true>(epi, p, ksplit, s);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_gemm_reduce(Epilogue epi, const GemmParams& p, int ksplit, int bn, hipStream_t s) {
  const int n_out = epi == kEpiSwiglu ? p.N / 2 : p.N;
  auto aligned = [](const void* q, uintptr_t to) { return ((uintptr_t)q & (to - 1)) == 0; };
  // every row of a split product is 4 or more values wide and aligned to them
  if (n_out % 4 || p.N % 4 || p.ldc % 4 || !aligned(p.part, 16) || p.M > 65535 ||
      (epi == kEpiSwiglu ? !aligned(p.c, 8) || bn % 32 : !aligned(p.c, 16)) ||
      (epi == kEpiResidRow && (p.r_ld % 4 || !aligned(p.r, 8))) || (epi == kEpiResidF32 && (p.r_ld % 4 || !aligned(p.r, 16))))
    return hipErrorInvalidValue;
  // the norm that follows, where one is asked for (rows of up to 8192 values)
  if ((epi == kEpiResidRow || epi == kEpiResidF32) && p.norm_gain && p.norm_done && p.N <= 8192 && p.norm_ld % 4 == 0 &&
      aligned(p.norm_out, 8) && aligned(p.norm_gain, 8) && aligned(p.norm_gain2, 8)) {
    *p.norm_done = true;
    return epi == kEpiResidRow ? launch_reduce_norm<kEpiResidRow>(p, ksplit, s) : launch_reduce_norm<kEpiResidF32>(p, ksplit, s);
  }
  const dim3 g4((unsigned)((n_out / 4 + 255) / 256), (unsigned)p.M);
  switch (epi) {
    case kEpiStore: hipLaunchKernelGGL(gemm_reduce4<kEpiStore>, g4, dim3(256), 0, s, p, ksplit, bn); break;
    case kEpiResidRow: hipLaunchKernelGGL(gemm_reduce4<kEpiResidRow>, g4, dim3(256), 0, s, p, ksplit, bn); break;
    case kEpiResidF32: hipLaunchKernelGGL(gemm_reduce4<kEpiResidF32>, g4, dim3(256), 0, s, p, ksplit, bn); break;
    case kEpiRowScale: hipLaunchKernelGGL(gemm_reduce4<kEpiRowScale>, g4, dim3(256), 0, s, p, ksplit, bn); break;
    case kEpiSwiglu: hipLaunchKernelGGL(gemm_reduce4<kEpiSwiglu>, g4, dim3(256), 0, s, p, ksplit, bn); break;
  }
  return hipGetLastError();
}

}  // namespace

// The columns [n1, N) of a product as a product of their own (same rows and
// K): weights, output and residual offset by n1 columns.  SwiGLU counts n1 in
// gate and up rows together (n1 / 2 output columns); other epilogues need a
// single weight block.
static GemmParams columns_from(const GemmParams& p, Epilogue epi, int n1) {
  GemmParams q = p;
  q.N = p.N - n1;
  if (epi == kEpiSwiglu) {
    const int oc = n1 / 2;
    q.b[0] = (const uint16_t*)p.b[0] + (int64_t)oc * p.ldb;
    q.b[1] = (const uint16_t*)p.b[1] + (int64_t)oc * p.ldb;
    q.b[2] = q.b[1];
    q.c = (f16*)p.c + oc;
    return q;
  }
  for (int i = 0; i < 3; ++i) q.b[i] = (const uint16_t*)p.b[0] + (int64_t)n1 * p.ldb;
  q.b_split0 = q.b_split1 = q.N;
  q.c = (float*)p.c + n1;
  if (epi == kEpiResidRow) q.r = (const uint16_t*)p.r + n1;
  if (epi == kEpiResidF32) q.r = (const float*)p.r + n1;
  return q;
}

// A grid of 256 x 256 tiles that takes more than one round and ends in a
// partial one: its whole rounds as 256 x 256 tiles over the first columns (all
// row tiles of each), the remaining columns as 256 x 128 tiles (rate: their
// throughput relative to 256 x 256) in a second launch.  Returns the number of
// 256-wide column tiles of the first launch when that prices cheaper than
// `other` (rounds x tile area / rate of the single-launch choice), else 0.
static int whole_round_columns(const GemmParams& p, int cus, double other, double rate2) {
  const int mt = (p.M + 255) / 256, nt = p.N / 256;
  const long t10 = (long)mt * nt, whole = (t10 / cus) * cus;
  if (p.N % 256 || t10 <= cus || whole == t10 || whole % mt) return 0;
  const int na = (int)(whole / mt);
  const long tail2 = (long)mt * (nt - na) * 2;
  // (and the second launch: about 4 us, in the unit of the others)
  const double cost = (double)(whole / cus) * 65536.0 + (double)((tail2 + cus - 1) / cus) * 32768.0 / rate2 + 1e7 / p.K;
  return cost < other ? na : 0;
}

// Products of at most 256 rows stream the weights: one round of workgroups, each
// with as many 64-deep stages in flight as its LDS holds, is the shape that
// reads them fastest, and a second round or a half-empty one costs as much as a
// whole one.  SwiGLU (up to 128 rows) takes the column width that covers
// N in the fewest columns per compute unit; the other epilogues the width and
// the number of K slices with the least
//   width x steps + rows x steps / 2 + 0.16 x partial sums per compute unit
// (+ 200, about 0.7 us, past four slices: the reduction's second round of loads),
// steps being a slice's: weights, activations (from the L2) and the reduction, in
// the proportions of the times measured at 64 and 128 rows.  Measured, fp16
// weights, before -> now, 128 rows: SwiGLU 24576 x 4096 60.8 -> 41.8 us, 34816 x 5120
// 127.9 -> 77.8, 19456 x 2560 39.3 -> 32.3, 5120 x 17408 73.6 -> 44.2 (eight slices),
// 4096 x 12288 33.4 -> 30.8, 6144 x 4096 27.0 -> 20.2; 64 rows: 55.4 -> 34.5, 129.4 ->
// 70.0, 37.1 -> 25.7, 58.3 -> 40.0, 27.3 -> 26.8, 23.1 -> 17.3; 16 rows: SwiGLU 42.6 ->
// 33.6, 97.9 -> 65.1, 29.3 -> 21.5; 256 rows: 4096 x 4096 26.2 -> 22.4, 4096 x 12288
// 52.4 -> 43.0, 2560 x 9728 42.1 -> 28.8.  Returns the tile, or -1 where no choice fills
// half the compute units (narrow heads: the smaller tiles below).  A slice has at least
// six steps (128 rows of 3072 x 2048 in eight of four: 13.9 us, in four 12.5).
static int stream_choice(Epilogue epi, const GemmParams& p, int cus, int* ksplit) {
  static constexpr int kBy16[] = {14}, kBy32[] = {26, 18}, kBy64[] = {19, 20, 21, 22}, kBy128[] = {27, 23, 24, 25};
  static constexpr int kGate16[] = {15, 16}, kGate32[] = {17, 18}, kGate64[] = {20, 22}, kGate128[] = {23, 25};
  const bool gate = epi == kEpiSwiglu;
  const int* cand = p.M <= 16 ? (gate ? kGate16 : kBy16) : p.M <= 32 ? (gate ? kGate32 : kBy32)
                    : p.M <= 64 ? (gate ? kGate64 : kBy64) : (gate ? kGate128 : kBy128);
  const int n = gate ? 2 : p.M <= 16 ? 1 : p.M <= 32 ? 2 : 4;
  int best = -1;
  double best_cost = 0.0;
  for (int i = 0; i < n; ++i) {
    const TileShape& t = kTiles[cand[i]];
    if (!tile_ok(p, epi, t)) continue;
    const long tiles = (long)((p.M + t.bm - 1) / t.bm) * ((p.N + t.bn - 1) / t.bn);
    const int KT = p.K / t.bk;
    for (int ks = 1; ks <= (gate ? 1 : 8); ++ks) {
      if (ks > 1 && (tiles * ks > cus || KT < 6 * ks || !p.part ||
                     (size_t)ks * p.M * p.N * sizeof(float) > p.part_bytes))
        break;
      if (2 * tiles * ks < cus) continue;
      const double rounds = (double)((tiles * ks + cus - 1) / cus);
      const double steps = rounds * ((KT + ks - 1) / ks);
      const double cost = steps * (t.bn + 0.5 * t.bm) + (ks > 1 ? 0.16 * ks * p.M * p.N / cus : 0.0) + (ks > 4 ? 200.0 : 0.0);
      if (best < 0 || cost < best_cost) { best = cand[i]; best_cost = cost; *ksplit = ks; }
    }
  }
  return best;
}

// Price of a plan for at most 256 rows, in us: a tile's steps per round of workgroups,
// the weights' bytes and a constant, fitted per tile to every plan of 4680 products (4
// to 256 rows of 180 matrices, weights as stored and as the fp16 image) with a spread
// of 9 percent; the reduction of a split by slices and partial sums; gemm_rows (tile
// kRows) by depth and workgroups per compute unit.  One price for both kinds of weights:
// the plan, and with it the order of every sum, must not depend on the kind.
// The shapes of the streaming tiles (stream_choice) follow the heads they were tuned on;
// against the plans of any number of rows this decides.  Without it 269 of those
// products were over a tenth slower than on the latter (128 rows of 3072 x 1024: 11.4 us
// against 6.6), now 10, by up to a fifth.  Negative: not priced.
constexpr int kRows = -1;
constexpr double kNormLaunch = 1.5;  // what a norm of its own costs over one in a split's reduction
struct PlanCost { double step, mb, fixed; };
constexpr PlanCost kTileCost[kNumTiles] = {
    {}, {}, {0.752, 0.035, 3.98}, {0.313, 0.067, 4.27}, {0.216, 0.087, 3.99}, {0.205, 0.071, 4.23},
    {0.178, 0.200, 3.45}, {0.135, 0.200, 3.15}, {}, {0.222, 0.125, 3.55}, {1.536, 0.081, 5.57}, {}, {}, {},
    {0.126, 0.103, 4.76}, {0.205, 0.086, 4.63}, {0.362, 0.079, 4.24}, {0.255, 0.072, 4.74}, {0.394, 0.070, 4.24},
    {0.197, 0.091, 4.32}, {0.319, 0.062, 4.55}, {0.371, 0.064, 4.13}, {0.489, 0.052, 4.34}, {0.475, 0.036, 4.79},
    {0.502, 0.042, 4.49}, {0.666, 0.021, 4.92}, {0.291, 0.081, 3.89}, {0.319, 0.076, 4.31}};

static double plan_price(Epilogue epi, const GemmParams& p, int cus, int tile, int ks) {
  const bool gate = epi == kEpiSwiglu;
  const double mb = 2e-6 * p.N * p.K, norm = p.norm_done ? kNormLaunch : 0.0;
  if (tile == kRows) {
    const long wgs = (long)(p.N / (gate ? 32 : 16)) * ((p.M + 15) / 16);
    const double depth = p.K / 1024.0 * (double)((wgs + cus - 1) / cus);
    if (gate) return p.M <= 8 ? 2.02 * depth + 0.061 * mb + 2.3 : 2.65 * depth + 0.043 * mb + 2.2;
    return norm + (p.M <= 8 ? 1.10 * depth + 0.056 * mb + 2.6 : 1.63 * depth + 0.028 * mb + 2.7);
  }
  const PlanCost& c = kTileCost[tile];
  if (c.step == 0.0) return -1.0;
  const TileShape& t = kTiles[tile];
  const long wgs = (long)((p.M + t.bm - 1) / t.bm) * ((p.N + t.bn - 1) / t.bn) * ks;
  const int steps = (p.K / t.bk + ks - 1) / ks;
  const double rounds = (double)((wgs + cus - 1) / cus);
  double us = c.step * steps * rounds + c.mb * mb + c.fixed;
  // one-wave tiles, several to a compute unit: a wave's chain of steps, or the weights'
  // bytes, read again by each row tile (partly from the L2)
  if (t.wgm * t.wgn == 1)
    us = std::max(c.step * steps, c.mb * mb * std::max(1.0, 0.4 * ((p.M + t.bm - 1) / t.bm))) + c.fixed;
  // streaming tiles that leave compute units idle have fewer loads in flight (64 rows of
  // 16384 x 3072, 171 workgroups: 28.3 us against 22.1 for 256 of 64 x 64)
  if (gate && tile >= kStreamTiles && p.M > 32 && wgs < cus) us *= 1.0 + 0.3 * (1.0 - (double)wgs / cus);
  const double part_mb = 4e-6 * ks * p.M * p.N;
  if (ks > 1) return us + (gate ? 0.90 + 0.31 * ks + 0.63 * part_mb : 0.93 + 0.28 * ks + 0.41 * part_mb);
  // unsplit, the epilogue reads the residuals one by one
  const double outs = (double)t.bm * t.bn / (64 * t.wgm * t.wgn) * rounds;
  return us + norm + (gate || epi == kEpiStore ? 0.0 : 0.04 * outs);
}

// A plan: the tile, its K slices, and (first > 0) the leading 256-column tiles that go to
// tile 10 in a launch before it.
struct TilePlan { int tile, ksplit, first; };

// The plan on the tiles that serve any number of rows.
static TilePlan tile_plan(Epilogue epi, const GemmParams& p, int cus) {
  auto fits = [&](int ks) { return p.part && (size_t)ks * p.M * p.N * sizeof(float) <= p.part_bytes; };
  // 17..32 rows (where a streaming tile is not the cheaper plan): a 32-row by 128-column tile
  // with four waves, and K split so that the grid has enough workgroups in
  // flight (each slice at least 8 steps of 64).  (Up to 16 rows the one-wave
  // 16-row tiles below measured faster.)
  if (p.M > 16 && p.M <= 32 && tile_ok(p, epi, kTiles[9])) {
    const int tiles = p.N / 128, KT = p.K / 64;
    int ks = 1;
    while (ks < 16 && tiles * ks * 2 <= 4 * cus && KT / (ks * 2) >= 8 && fits(ks * 2)) ks *= 2;
    return {9, ks, 0};
  }
  // K of 4096 or more with a few hundred rows (o and down on 129-1024 rows):
  // 256 x 128 tiles with K split re-read the activations and weights half as
  // often as 128 x 64 tiles at the same workgroup count.  As many slices (2-4, on more
  // than 256 rows and K of 8192 up to 6,
  // of whole 64-deep steps, not necessarily equal) as keep the grid within one
  // round (1024 x 2560 x 9728, 80 tiles: 76 us in three slices against 94 us in
  // two; 1024 x 2560 x 4096: 41 us against 47; 512 x 4096 x 4096, 64 tiles: 38
  // us in four against 41 us for 256 tiles of 128 x 64; 512 x 4096 x 12288: 77
  // us in four against 111 us in two; 512 x 2560 x 9728, 40 tiles: 40.5 us in six
  // against 46.4 in four).
  if (epi != kEpiSwiglu && p.M > 128 && p.M <= 1024 && p.K >= 4096 && tile_ok(p, epi, kTiles[2])) {
    const long tiles = (long)((p.M + 255) / 256) * (p.N / 128);
    const int ks = (int)std::min<long>(p.M > 256 && p.K >= 8192 ? 6 : 4, std::max<long>(2, cus / tiles));
    if (p.K % 64 == 0 && p.K / 64 >= 8 * ks && fits(ks)) return {2, ks, 0};
  }
  // 33..256 rows of the other epilogues (QKV on more than 128 rows, K under 4096 there,
  // and where a streaming tile is not the cheaper plan): 128 x 64 tiles with K split
  // until the grid has a workgroup per compute unit (o on 256 rows of the 27B shape:
  // 58 us against 71 for 256 x 128).
  if (epi != kEpiSwiglu && p.M > 32 && p.M <= 256 && tile_ok(p, epi, kTiles[3]) && p.part) {
    const long tiles = (long)((p.M + 127) / 128) * (p.N / 64);
    int ks = 2;
    while (ks < 8 && tiles * ks < cus) ks *= 2;
    if (p.K / 64 / ks >= 8 && fits(ks)) return {3, ks, 0};
  }
  // The wide tiles, priced by the rounds of workgroups the grid takes on the
  // compute units (a last partial round costs a whole one) times the tile's
  // work over its measured relative rate (2048-8192 rows, fp16 weights).
  auto cheapest = [&](const int* cand, const double* rate, int n) {
    int best = -1;
    double best_cost = 0.0;
    for (int i = 0; i < n; ++i) {
      const TileShape& t = kTiles[cand[i]];
      if (!tile_ok(p, epi, t)) continue;
      const long tiles = (long)((p.M + t.bm - 1) / t.bm) * ((p.N + t.bn - 1) / t.bn);
      if (cand[i] == kRaggedWide && 2 * tiles < cus) continue;
      const double cost = (double)((tiles + cus - 1) / cus) * t.bm * t.bn / rate[i];
      if (best < 0 || cost < best_cost) { best = cand[i]; best_cost = cost; }
    }
    return best;
  };
  // SwiGLU (gate/up) on more than 256 rows, and on 128-256 rows when 256 x 128
  // tiles would fill at least half the compute units (fewer wide tiles would
  // leave most of them idle; the order below then takes smaller ones).  At
  // 1024 x 19456 x 2560 this takes 256 x 128 (608 tiles, 0.140 ms) over
  // 256 x 256 (304 tiles: two rounds, the second nearly empty, 0.154 ms); at
  // 256 x 34816 x 5120 (last-row-only rows of the 27B shape) 256 x 160 in one round
  // of 218 tiles (112 us) over 136 of 256 x 256 (140 us).  Not 256 x 160 where its
  // grid leaves half the compute units idle, on widths that no other wide tile
  // divides (896 x 704 x 3072: 50 us, 27 in 64 x 64).
  const long tiles2 = (long)((p.M + 255) / 256) * (p.N / 128);
  if (epi == kEpiSwiglu && (p.M > 256 || (p.M >= 128 && 2 * tiles2 >= cus))) {
    static const int cand[5] = {10, 0, 2, 12, 13};
    static const double rate[5] = {1.0, 0.91, 0.87, 0.855, 0.78};
    const int best = cheapest(cand, rate, 5);
    // (1024 x 19456 x 2560: 124 us against 137 us for 608 tiles of 256 x 128
    // and 149 us for 304 of 256 x 256)
    if (best >= 0 && tile_ok(p, epi, kTiles[10])) {
      const TileShape& tb = kTiles[best];
      const long tb_tiles = (long)((p.M + tb.bm - 1) / tb.bm) * ((p.N + tb.bn - 1) / tb.bn);
      const int bi = best == 10 ? 0 : best == 0 ? 1 : best == 2 ? 2 : best == 12 ? 3 : 4;
      const int na = whole_round_columns(p, cus, (double)((tb_tiles + cus - 1) / cus) * tb.bm * tb.bn / rate[bi], 0.87);
      if (na > 0) return {2, 1, na};
    }
    if (best >= 0) return {best, 1, 0};
  }
  // Residual products on more than 1024 rows whose 256 x 128 grid fills the
  // compute units: 8192 x 5120 takes 256 x 160 (four whole rounds; o 0.408 ms,
  // down 1.39 ms) over 256 x 256 (three rounds, the last half empty; 0.413,
  // 1.40) and 256 x 128 (five rounds; 0.428, 1.43).
  // Long K on more than 1024 rows whose 256 x 256 grid fills at most half the
  // compute units: those tiles with K split in two (2048 x 4096 x 12288, down:
  // 201 us against 218 us for 256 tiles of 256 x 128; with K = 4096, o, the
  // split measured slower).
  if (epi != kEpiSwiglu && p.M > 1024 && p.K >= 8192 && tile_ok(p, epi, kTiles[10]) &&
      2 * (long)((p.M + 255) / 256) * (p.N / 256) <= cus && p.K % 128 == 0 && fits(2))
    return {10, 2, 0};
  // The mixed plan above applies here too (single weight block): 8192 x 5120
  // as two rounds of 256 x 256 over 4096 columns and one of 256 x 128 over the
  // last 1024 (down 1.22 ms, o 0.369 ms, against 1.34 and 0.389 for 256 x 160).
  if (epi != kEpiSwiglu && p.M > 1024 && tile_ok(p, epi, kTiles[2]) &&
      (long)((p.M + 255) / 256) * (p.N / 128) >= cus) {
    static const int cand[3] = {10, 11, 2};
    static const double rate[3] = {1.0, 0.84, 0.80};
    const int best = cheapest(cand, rate, 3);
    if (best >= 0 && tile_ok(p, epi, kTiles[10]) && p.b_split0 >= p.N) {
      const TileShape& tb = kTiles[best];
      const long tb_tiles = (long)((p.M + tb.bm - 1) / tb.bm) * ((p.N + tb.bn - 1) / tb.bn);
      const int bi = best == 10 ? 0 : best == 11 ? 1 : 2;
      const int na = whole_round_columns(p, cus, (double)((tb_tiles + cus - 1) / cus) * tb.bm * tb.bn / rate[bi], 0.80);
      if (na > 0) return {2, 1, na};
    }
    if (best >= 0) return {best, 1, 0};
  }
  // First tile (in preference order) that gives at least one workgroup per
  // compute unit, else the valid tile with the most workgroups.
  const int* order = epi == kEpiSwiglu ? kOrderSwiglu : kOrderResid;
  int best = -1;
  long best_tiles = -1;
  for (int i = 0; i < 9; ++i) {
    const int c = order[i];
    if (!tile_ok(p, epi, kTiles[c])) continue;
    const long tiles = (long)((p.M + kTiles[c].bm - 1) / kTiles[c].bm) * (p.N / kTiles[c].bn);
    if (tiles >= cus) { best = c; break; }
    if (tiles > best_tiles) { best_tiles = tiles; best = c; }
  }
  return {best, 1, 0};
}

hipError_t launch_gemm(DType dt, Epilogue epi, const GemmParams& p0, hipStream_t s) {
  if (p0.M <= 0) return hipSuccess;
  if (dt == kF32) {
    switch (epi) {
      case kEpiStore: return launch_f32<kEpiStore>(p0, s);
      case kEpiResidRow: return launch_f32<kEpiResidRow>(p0, s);
      case kEpiResidF32: return launch_f32<kEpiResidF32>(p0, s);
      case kEpiRowScale: return launch_f32<kEpiRowScale>(p0, s);
      case kEpiSwiglu: return launch_f32<kEpiSwiglu>(p0, s);
    }
    return hipErrorInvalidValue;
  }
  if (p0.K % 32 || p0.lda % 8 || p0.ldb % 8) return hipErrorInvalidValue;
  GemmParams p = p0;
  const int cus = p.n_cus > 0 ? p.n_cus : 256;
  if (p.n_xcd < 1) p.n_xcd = 1;
  // group of row tiles: the XCD's compute units then cover about a square of
  // tiles (8 row tiles by 4 column tiles with 32 compute units per XCD)
  if (p.group_m < 1) p.group_m = 8;
  const TilePlan tp = tile_plan(epi, p, cus);
  // Up to 256 rows, the streaming tiles or gemm_rows instead, unless the plan above
  // prices clearly cheaper (3%).  The streaming tiles serve SwiGLU up to 128 rows; up to 16 rows, the other
  // epilogues: long K of matrices wider than gemm_rows takes (5120 x 17408: 37 us
  // against 44 for the one-wave tiles; 6144 x 4096 stays there, 12.9 us against 15.7),
  // and from 13 rows and K = 9216 those it would take (16 rows: 2560 x 9728 21.7 -> 17.5
  // us, 4096 x 12288 27.2 -> 24.8; at 9 rows 18.4 -> 17.2 and 23.7 -> 24.6; 13 rows of 4096 x
  // 8192: 17.6 against 18.7).  17-128 rows, unless
  // gemm_rows covers them with a workgroup per compute unit.  129-256 rows: K
  // of 4096 or more, not the QKV product (7168 x 5120: 37.7 us on the plan above, 39.0).
  const int rows_cols = epi == kEpiSwiglu ? 32 : 16;
  const bool rows_fit = (int64_t)(p.N / rows_cols) * ((p.M + 15) / 16) <= cus;
  const bool stream = epi == kEpiSwiglu ? p.M <= 128 && !(p.M > 16 && rows_fit)
                      : p.M <= 16       ? (rows_fit ? p.M > 12 && p.K >= 9216 : p.K >= 8192)
                      : p.M <= 128      ? !rows_fit
                                        : p.M <= 256 && p.K >= 4096 && epi != kEpiStore;
  auto dearer = [&](int tile, int ks) {  // than the plan above
    if (tp.first) return false;
    const double mine = plan_price(epi, p, cus, tile, ks), other = tp.tile < 0 ? -1.0 : plan_price(epi, p, cus, tp.tile, tp.ksplit);
    return mine >= 0.0 && other >= 0.0 && other < 0.97 * mine;
  };
  if (stream) {
    int ks = 1;
    const int t = stream_choice(epi, p, cus, &ks);
    if (t >= 0) {
      if (dearer(t, ks)) return launch_tile_index(tp.tile, epi, p, tp.ksplit, s);
      return launch_tile_index(t, epi, p, ks, s);
    }
  }
  // gemm_rows: at most one workgroup per compute unit (16 rows of matrices up to
  // 4096 wide, more rows of narrower ones), and the SwiGLU of up to 16 rows that the
  // streaming tiles leave.  Wider
  // products on few rows keep the one-wave tiles: their tiles do not divide
  // evenly over the compute units either way, and one wave each balances better
  // (5 rows: 6144 x 4096 12.5 us against 13.5).  Long K of narrow matrices leaves most
  // compute units idle here and is split over workgroups by its price (32 rows of 1024 x
  // 4096: 9.9 us here, 10.3 in eight slices; 512 x 8192 16.7 and 10.8; 1024 x 28672
  // 52.2 and 24.5).
  if (((epi == kEpiSwiglu && p.M <= 16) || rows_fit) && p.N % rows_cols == 0 &&
      (epi == kEpiSwiglu || (p.b_split0 % 16 == 0 && p.b_split1 % 16 == 0)) && !dearer(kRows, 1))
    return launch_gemm_rows(epi, p, s);
  if (tp.first) {
    GemmParams q = p;
    q.N = 256 * tp.first;
    if (epi != kEpiSwiglu) q.b_split0 = q.b_split1 = q.N;
    const hipError_t e = launch_tile_index(10, epi, q, 1, s);
    return e != hipSuccess ? e : launch_tile_index(tp.tile, epi, columns_from(p, epi, q.N), 1, s);
  }
  return launch_tile_index(tp.tile, epi, p, tp.ksplit, s);
}

}  // namespace sp
