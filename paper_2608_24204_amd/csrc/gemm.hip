// Prefill projections: C[M, N] = A[M, K] x W[N, K]^T with fused epilogues.
//
// A holds activations (one row per prompt position), W the bf16 weights in their
// [out, in] layout, so both operands are contiguous along K, which is the layout
// the gfx950 matrix cores consume (8 consecutive K values per lane).
//
// MFMA kernels.  A arrives as NT bf16 planes whose sum is the fp32 activation
// (see ActBuf); the weights are exact bf16, so the kernels accumulate the NT
// products A_p W^T with v_mfma_f32_16x16x32_bf16 and the result carries the
// activation's precision, not bf16's.  Operands are staged through LDS in 32-deep K
// steps (64-byte rows with the 16-byte chunks XOR-swizzled by row, so that neither
// the stores nor the fragment reads hit the same bank twice); tiles are dealt to the
// 8 XCDs in contiguous ranges (workgroups are dispatched round-robin over XCDs), so
// the blocks resident on one XCD share tiles through that XCD's L2.  Three variants:
// tiles of bf16 weights (k_gemm_dma), tiles of 8-bit weights (k_gemm_q8), and few rows
// (k_gemm_rows, either weights; k_gemm_skinny where K is no multiple of 128).
//
// Vector kernel: plain fp32 64x64 tiles, for fp32 weights / fp32 activations.
#include "common.h"
#include "kernels.h"

#include <algorithm>
#include <type_traits>

namespace wici {

// ------------------------------------------------------------------ epilogue
// The value of the lane's neighbour across bit 0 of the lane index: in a matrix-core
// result tile lane l holds column l % 16, so this is the SwiGLU partner (gate 2i,
// up 2i + 1).  A DPP quad permutation [1, 0, 3, 2] (a register move, where a
// shuffle goes through the LDS permute unit).
__device__ __forceinline__ float pair_swap(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xF, 0xF, false));
}

template <int EPI>
__device__ __forceinline__ void epi_out(float* C, int ldc, const ActBuf& H, int ldh, int M,
                                        int N, int m, int n, float v, float other) {
  if (m >= M || n >= N) return;
  if (EPI == GEMV_STORE) C[(size_t)m * ldc + n] = v;
  else if (EPI == GEMV_RESID) C[(size_t)m * ldc + n] += v;
  else if (EPI == GEMV_SWIGLU) {
    if (!(n & 1)) store_act(H, (size_t)m * ldh + (n >> 1), silu(v) * other);
  }
}

// --------------------------------------------------------------------- MFMA
constexpr int kLDK = 32;  // LDS row (bf16 elements): 64 bytes, four 16-byte chunks

// LDS position (bf16 elements) of 16-byte chunk `chunk` of tile row `row`: the chunk
// index is XOR-ed with bits 2-3 of the row.  Sixteen lanes that store together
// (4 consecutive rows x 4 chunks, as loaded from global memory) then cover four
// disjoint 64-byte bank ranges, and sixteen lanes that read a fragment (16 rows,
// one chunk) cover all 64 banks once: neither access conflicts.
__device__ __forceinline__ int lds_swz(int row) { return (row >> 2) & 3; }
__device__ __forceinline__ int lds_chunk(int row, int chunk) {
  return row * kLDK + 8 * (chunk ^ lds_swz(row));
}

// --------------------------------------------------------- MFMA, direct to LDS
// bf16 weights: a K step's tiles go from global memory straight into LDS (buffer
// loads to LDS: each lane's 16 bytes land at its wavefront's LDS base + 16 x lane,
// so the row swizzle is applied by choosing which chunk each lane fetches) through
// a ring of STG stages, with no registers held for them and no register-to-LDS
// copy.  The waits are explicit (a step's loads counted down, then a bare barrier): a
// __syncthreads would wait for every load in flight.  One lane offset serves all
// loads of an operand: the row ranges differ in their buffer descriptors (scalar
// registers), whose bounds return zeros for rows past M or N (their outputs are
// dropped).
//
// Shape: WMW x WNW wavefronts, each 16 TMW x 16 TNW outputs.
//
// Schedule: the activation fragments are read GI row tiles at a time, one group
// ahead of the products that use them, and the next step's weight fragments and
// first group behind the step's last products: after its last fragment read of a
// step a wavefront waits for the next stage and the barrier, refills the stage just
// read, and then multiplies the last group while the next step's fragments arrive.
// So no product waits for an LDS read issued just before it.  K is walked in pairs
// of steps (two register sets in turn).
//
// The products are formed as W A^T: a lane then holds four consecutive columns of
// one row and stores 16 bytes (fp32).  For SwiGLU the weight rows of a tile are
// dealt so that a lane's four tiles are sixteen consecutive columns, i.e. eight
// outputs, 16 bytes per term plane.
// A lane's results of one output row m: columns 4 fc + r of each 16-column tile from n0
// on, or (SwiGLU) 16 fc + 4 (j % 4) + r of the 64 of four tiles.  vec: the rows of C are
// aligned to four values.
template <int EPI, int TNW>
__device__ __forceinline__ void store_rows(const floatx4_t (&acc)[TNW], float* C, int ldc,
                                           const ActBuf& H, int ldh, int N, int m, int n0, int fc,
                                           bool vec) {
  if constexpr (EPI == GEMV_SWIGLU) {
#pragma unroll
    for (int j = 0; j < TNW; j += 4) {
      const int n = n0 + j * 16 + fc * 16;
      float o[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const floatx4_t& c = acc[j + e / 2];
        o[e] = silu(c[2 * (e & 1)]) * c[2 * (e & 1) + 1];
      }
      if (n + 16 <= N && ldh % 8 == 0) {
        store_act8(H, (size_t)m * ldh + n / 2, o);
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (n + 2 * e + 1 < N) store_act(H, (size_t)m * ldh + n / 2 + e, o[e]);
      }
    }
  } else {
#pragma unroll
    for (int j = 0; j < TNW; ++j) {
      const int n = n0 + j * 16 + fc * 4;
      float* p = C + (size_t)m * ldc + n;
      if (vec && n + 4 <= N) {
        floatx4_t v = acc[j];
        if (EPI == GEMV_RESID) v = *reinterpret_cast<const floatx4_t*>(p) + v;
        *reinterpret_cast<floatx4_t*>(p) = v;
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (n + r < N) p[r] = EPI == GEMV_RESID ? p[r] + acc[j][r] : acc[j][r];
      }
    }
  }
}

__device__ __forceinline__ void dma16(const bf16_t* g, bf16_t* lds_wave) {
  __builtin_amdgcn_global_load_lds(g, (__attribute__((address_space(3))) void*)lds_wave, 16, 0, 0);
}
// 4 bytes a lane
__device__ __forceinline__ void dma4(const void* g, bf16_t* lds_wave) {
  __builtin_amdgcn_global_load_lds(g, (__attribute__((address_space(3))) void*)lds_wave, 4, 0, 0);
}
// s_waitcnt with vmcnt <= VM, lgkmcnt 0, expcnt unconstrained (gfx9 encoding)
template <int VM>
__device__ __forceinline__ void wait_vm_lgkm() {
  static_assert(VM >= 0 && VM < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((VM & 15) | ((VM >> 4) << 14) | (7 << 4));
}

template <int NT, int EPI, int WMW, int WNW, int TMW, int TNW, int STG, int GI, bool NMAJ>
__global__ __launch_bounds__(64 * WMW * WNW) __attribute__((amdgpu_waves_per_eu(2))) void
k_gemm_dma(const bf16_t* __restrict__ A, size_t a_plane, int lda, const bf16_t* __restrict__ W,
           int M, int N, int K, int ks, float* __restrict__ C, size_t c_split, int ldc, ActBuf H,
           int ldh) {
  constexpr int NW = WMW * WNW, BM = 16 * TMW * WMW, BN = 16 * TNW * WNW;
  constexpr int PAP = BM * 4 / (64 * NW);       // 16-byte units per lane: a plane of A,
  constexpr int PA = NT * PAP;                  // all of A,
  constexpr int PB = BN * 4 / (64 * NW);        // and W, per stage
  constexpr int PER = PA + PB, STAGE = (NT * BM + BN) * kLDK;
  constexpr int GP = TMW / GI, G = NT * GP;     // groups per plane and step
  constexpr bool DEAL = EPI == GEMV_SWIGLU;
  static_assert(BM * 4 % (64 * NW) == 0 && BN * 4 % (64 * NW) == 0, "whole units per lane");
  static_assert(TMW % GI == 0 && G % 2 == 0, "an even number of groups");
  static_assert(!DEAL || TNW % 4 == 0, "sixteen consecutive columns per lane");
  static_assert(STG >= 2 && STG <= 3 && 2 * PER < 64, "stage ring");
  extern __shared__ __attribute__((aligned(16))) bf16_t smem[];

  const int n_mt = (M + BM - 1) / BM, n_nt = (N + BN - 1) / BN;
  int m0, n0;
  if (NMAJ) {
    // each XCD owns a contiguous range of weight column tiles for every row tile,
    // the row tiles of one column tile on consecutive workgroups (so the blocks
    // resident on an XCD share weight tiles through its L2)
    const int nper = (n_nt + 7) / 8, loc = blockIdx.x / 8;
    const int nt_i = (blockIdx.x % 8) * nper + loc / n_mt;
    if (nt_i >= n_nt || loc >= nper * n_mt) return;
    m0 = (loc % n_mt) * BM;
    n0 = nt_i * BN;
  } else {
    const int T = n_mt * n_nt, per_xcd = (T + 7) / 8;
    const int t = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
    if (t >= T) return;
    m0 = (t / n_nt) * BM;
    n0 = (t % n_nt) * BN;
  }
  const int kbeg = blockIdx.y * ks;
  C += blockIdx.y * c_split;

  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int wm = wave / WNW, wn = wave % WNW;

  // LDS chunk of a weight row: as lds_swz, or for dealt rows (a fragment's sixteen
  // lanes read rows 16 (l / 4) + l % 4 of 64) by the row's bits 4-5, so that they
  // cover all 64 banks once either way
  auto w_swz = [](int row) { return DEAL ? (row >> 4) & 3 : lds_swz(row); };
  // this lane's unit of a load of 16 NW rows: row r0 of them (4 lanes a row); the
  // weight rows' swizzle depends on the row range when dealt, the offset with it
  const int r0 = wave * 16 + (lane >> 2);
  const int offA = (int)(((size_t)r0 * lda + ((lane & 3) ^ lds_swz(r0)) * 8) * 2);
  const int offW = (int)(((size_t)r0 * K + ((lane & 3) ^ w_swz(r0)) * 8) * 2);
  static_assert(!DEAL || (NW * 16) % 64 == 0, "the swizzle is the same in every row range");
  auto issue = [&](int stage, int kt) {
    bf16_t* sb = smem + stage * STAGE;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const bool isA = i < PA;
      const int rr = (isA ? i % PAP : i - PA) * NW * 16;  // first row of the range
      const int ld = isA ? lda : K, cnt = min((isA ? M - m0 : N - n0) - rr, NW * 16);
      const bf16_t* base = isA ? A + (i / PAP) * a_plane + (size_t)(m0 + rr) * lda + kbeg
                               : W + (size_t)(n0 + rr) * K + kbeg;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          rsrc(base, cnt > 0 ? ((size_t)(cnt - 1) * ld + ks) * 2 : 0),
          (__attribute__((address_space(3))) void*)(sb + (i * NW + wave) * 512), 16,
          isA ? offA : offW, kt * (kBK * 2), 0, 0);
    }
  };

  floatx4_t acc[TMW][TNW];
#pragma unroll
  for (int i = 0; i < TMW; ++i)
#pragma unroll
    for (int j = 0; j < TNW; ++j) acc[i][j] = floatx4_t{0.f, 0.f, 0.f, 0.f};
  const int fr = lane & 15, fc = lane >> 4;
  // weight row of the wavefront's range that lane fr of tile j multiplies
  auto w_row = [&](int j) {
    return wn * 16 * TNW + (DEAL ? (j / 4) * 64 + (fr >> 2) * 16 + (j % 4) * 4 + (fr & 3) : j * 16 + fr);
  };
  auto readW = [&](const bf16_t* sb, bf16x8_t (&b)[TNW]) {
#pragma unroll
    for (int j = 0; j < TNW; ++j) {
      const int row = w_row(j);
      b[j] = *reinterpret_cast<const bf16x8_t*>(sb + (NT * BM + row) * kLDK + 8 * (fc ^ w_swz(row)));
    }
  };
  auto readA = [&](const bf16_t* sb, int g, bf16x8_t (&a)[GI]) {
#pragma unroll
    for (int i = 0; i < GI; ++i)
      a[i] = *reinterpret_cast<const bf16x8_t*>(
          sb + lds_chunk((g / GP) * BM + wm * 16 * TMW + (g % GP * GI + i) * 16 + fr, fc));
  };
  auto mult = [&](int g, const bf16x8_t (&a)[GI], const bf16x8_t (&b)[TNW]) {
#pragma unroll
    for (int i = 0; i < GI; ++i)
#pragma unroll
      for (int j = 0; j < TNW; ++j) {
        floatx4_t& c = acc[g % GP * GI + i][j];
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[j], a[i], c, 0, 0, 0);
      }
  };
  // wait for a stage: `later` stages were issued after it
  auto wait_stage = [&](int later) {
    if (later >= 2) wait_vm_lgkm<2 * PER>();
    else if (later == 1) wait_vm_lgkm<PER>();
    else wait_vm_lgkm<0>();
  };
  const int KT = ks / kBK;  // even
#pragma unroll
  for (int s = 0; s < STG; ++s)
    if (s < KT) issue(s, s);
  wait_stage(min(STG, KT) - 1);
  __builtin_amdgcn_s_barrier();
  bf16x8_t b0[TNW], b1[TNW], a0[GI], a1[GI];
  readW(smem, b0);
  readA(smem, 0, a0);
  // one K step on the weight fragments b; leaves the next step's in bn (after the
  // last step: whatever the stage holds, unused)
  auto step = [&](int kt, const bf16x8_t (&b)[TNW], bf16x8_t (&bn)[TNW]) {
    const bf16_t* sb = smem + (kt % STG) * STAGE;
#pragma unroll
    for (int g = 0; g < G - 1; ++g) {
      if (g & 1) readA(sb, g + 1, a0);
      else readA(sb, g + 1, a1);
      __builtin_amdgcn_sched_barrier(0);  // the reads stay ahead of the products
      if (g & 1) mult(g, a1, b);
      else mult(g, a0, b);
      __builtin_amdgcn_sched_barrier(0);
    }
    wait_stage(min(STG - 2, KT - 2 - kt));
    __builtin_amdgcn_s_barrier();
    if (kt + STG < KT) issue(kt % STG, kt + STG);
    const bf16_t* sn = smem + ((kt + 1) % STG) * STAGE;
    readW(sn, bn);
    readA(sn, 0, a0);
    __builtin_amdgcn_sched_barrier(0);
    mult(G - 1, a1, b);
    __builtin_amdgcn_sched_barrier(0);
  };
  for (int kt = 0; kt < KT; kt += 2) {
    step(kt, b0, b1);
    step(kt + 1, b1, b0);
  }

  const bool vec = N % 4 == 0 && ldc % 4 == 0;
#pragma unroll
  for (int i = 0; i < TMW; ++i) {
    const int m = m0 + wm * 16 * TMW + i * 16 + fr;
    if (m < M) store_rows<EPI, TNW>(acc[i], C, ldc, H, ldh, N, m, n0 + wn * 16 * TNW, fc, vec);
  }
}

typedef unsigned u32x2_t __attribute__((ext_vector_type(2)));
// 8 codes (q + 128) as 8 bf16 values q, exact: with its top bit flipped a code byte
// is q in two's complement, which one instruction converts to fp32 (byte select and
// sign extension included); the upper halves of two of those are the bf16 pair.
__device__ __forceinline__ bf16x8_t q8_frag(u32x2_t c) {
  unsigned o[4];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int w = (int)(c[h] ^ 0x80808080u);
    const float f0 = (float)(int8_t)w, f1 = (float)(int8_t)(w >> 8);
    const float f2 = (float)(int8_t)(w >> 16), f3 = (float)(w >> 24);
    o[2 * h] = __builtin_amdgcn_perm(__float_as_uint(f1), __float_as_uint(f0), 0x07060302u);
    o[2 * h + 1] = __builtin_amdgcn_perm(__float_as_uint(f3), __float_as_uint(f2), 0x07060302u);
  }
  return __builtin_bit_cast(bf16x8_t, make_uint4(o[0], o[1], o[2], o[3]));
}

// ------------------------------------------------------------- MFMA, Q8 weights
// The same product, schedule and epilogue for 8-bit weights, 128 x 128 tiles of four
// 64 x 64 wavefronts.  A 32-deep step is one quantisation block: its products (all
// terms) are summed in a fresh accumulator and added times the column's block scale,
// so the codes go through the matrix cores as exact bf16 integers.  The step is bound
// by the vector ALU (64 scale FMAs a wavefront and the code conversion) beside the
// matrix cores, so what matters is that the two overlap: a row tile's FMAs stand
// behind the next one's products, and the codes of the step after are converted once
// per workgroup, 16 per thread, on their way from registers into LDS (converted by
// each wavefront that reads them they cost twice that).  Scales go through LDS as
// fp32, a pair of steps at a time.  Every load is unconditional (past the last step the
// last one's again), so the compiler's own waits count exactly.
template <int NT, int EPI>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_gemm_q8(
    const bf16_t* __restrict__ A, size_t a_plane, int lda, const uint8_t* __restrict__ W,
    const unsigned short* __restrict__ S, int M, int N, int K, int ks, float* __restrict__ C,
    size_t c_split, int ldc, ActBuf H, int ldh) {
  constexpr int BM = 128, BN = 128, NW = 4, TMW = 4, TNW = 4, STG = 2;
  constexpr int PAP = 2, PA = NT * PAP;         // 16-byte units per lane: a plane of A, all of A
  constexpr int ASTAGE = NT * BM * kLDK, WSTAGE = BN * kLDK;
  constexpr bool DEAL = EPI == GEMV_SWIGLU;
  extern __shared__ __attribute__((aligned(16))) bf16_t smem[];
  bf16_t* Ws = smem + STG * ASTAGE;                        // [2][BN][kLDK]
  float* Sc = reinterpret_cast<float*>(Ws + 2 * WSTAGE);   // [2 pairs][2 steps][BN]

  const int n_mt = (M + BM - 1) / BM, n_nt = (N + BN - 1) / BN;
  const int T = n_mt * n_nt, per_xcd = (T + 7) / 8;
  const int t = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
  if (t >= T) return;
  const int m0 = (t / n_nt) * BM, n0 = (t % n_nt) * BN;
  const int kbeg = blockIdx.y * ks;
  C += blockIdx.y * c_split;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int wm = wave >> 1, wn = wave & 1, fr = lane & 15, fc = lane >> 4;
  const int KT = ks / kBK;  // even

  auto w_swz = [](int row) { return DEAL ? (row >> 4) & 3 : lds_swz(row); };
  const int r0 = wave * 16 + (lane >> 2);
  const int offA = (int)(((size_t)r0 * lda + ((lane & 3) ^ lds_swz(r0)) * 8) * 2);
  auto issue = [&](int stage, int kt) {
    bf16_t* sb = smem + stage * ASTAGE;
#pragma unroll
    for (int i = 0; i < PA; ++i) {
      const int rr = (i % PAP) * NW * 16, cnt = min(M - m0 - rr, NW * 16);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          rsrc(A + (i / PAP) * a_plane + (size_t)(m0 + rr) * lda + kbeg,
               cnt > 0 ? ((size_t)(cnt - 1) * lda + ks) * 2 : 0),
          (__attribute__((address_space(3))) void*)(sb + (i * NW + wave) * 512), 16, offA,
          kt * (kBK * 2), 0, 0);
    }
  };
  // this thread's half row of codes (16) per step, and its scale per pair of steps
  const int wr = tid >> 1, wh = tid & 1, wrow = min(n0 + wr, N - 1);
  const uint8_t* wsrc = W + (size_t)wrow * K + kbeg + wh * 16;
  const unsigned short* ssrc = S + (size_t)wrow * (K / 32) + kbeg / 32 + wh;
  typedef unsigned u32x4_v __attribute__((ext_vector_type(4)));
  auto wload = [&](int kt) {
    return *reinterpret_cast<const u32x4_v*>(wsrc + (size_t)min(kt, KT - 1) * kBK);
  };
  auto sload = [&](int pair) { return ssrc[2 * min(pair, KT / 2 - 1)]; };
  auto wstore = [&](int buf, u32x4_v v) {
    bf16_t* row = Ws + buf * WSTAGE + wr * kLDK;
    *reinterpret_cast<bf16x8_t*>(row + 8 * ((2 * wh) ^ w_swz(wr))) = q8_frag(u32x2_t{v.x, v.y});
    *reinterpret_cast<bf16x8_t*>(row + 8 * ((2 * wh + 1) ^ w_swz(wr))) = q8_frag(u32x2_t{v.z, v.w});
  };
  auto sstore = [&](int buf, unsigned short v) {
    Sc[(buf * 2 + wh) * BN + wr] = (float)__builtin_bit_cast(_Float16, v);
  };

  floatx4_t acc[TMW][TNW];
#pragma unroll
  for (int i = 0; i < TMW; ++i)
#pragma unroll
    for (int j = 0; j < TNW; ++j) acc[i][j] = floatx4_t{0.f, 0.f, 0.f, 0.f};
  auto readW = [&](int buf, bf16x8_t (&b)[TNW]) {
#pragma unroll
    for (int j = 0; j < TNW; ++j) {
      const int row = wn * 64 + (DEAL ? (fr >> 2) * 16 + j * 4 + (fr & 3) : j * 16 + fr);
      b[j] = *reinterpret_cast<const bf16x8_t*>(Ws + buf * WSTAGE + row * kLDK + 8 * (fc ^ w_swz(row)));
    }
  };
  auto readS = [&](int pairbuf, int h, floatx4_t (&d)[TNW]) {  // columns of this lane's results
#pragma unroll
    for (int j = 0; j < TNW; ++j)
      d[j] = *reinterpret_cast<const floatx4_t*>(
          Sc + (pairbuf * 2 + h) * BN + wn * 64 + (DEAL ? fc * 16 + j * 4 : j * 16 + fc * 4));
  };
  auto readA = [&](int stage, int i, bf16x8_t (&a)[NT]) {
#pragma unroll
    for (int p = 0; p < NT; ++p)
      a[p] = *reinterpret_cast<const bf16x8_t*>(smem + stage * ASTAGE +
                                                lds_chunk(p * BM + wm * 64 + i * 16 + fr, fc));
  };
  auto mult = [&](const bf16x8_t (&a)[NT], const bf16x8_t (&b)[TNW], floatx4_t (&q)[TNW]) {
#pragma unroll
    for (int p = 0; p < NT; ++p)
#pragma unroll
      for (int j = 0; j < TNW; ++j)
        q[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
            b[j], a[p], p ? q[j] : floatx4_t{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
  };
  auto fold = [&](int i, const floatx4_t (&q)[TNW], const floatx4_t (&d)[TNW]) {
#pragma unroll
    for (int j = 0; j < TNW; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[i][j][r] += q[j][r] * d[j][r];
  };

  issue(0, 0);
  u32x4_v rw = wload(0);
  unsigned short rs = sload(0);
  wstore(0, rw);
  sstore(0, rs);
  rw = wload(1);
  rs = sload(1);
  issue(1, 1);
  wait_vm_lgkm<0>();
  __builtin_amdgcn_s_barrier();
  bf16x8_t b0[TNW], b1[TNW], a0[NT], a1[NT];
  floatx4_t d[TNW], q0[TNW], q1[TNW];
  readW(0, b0);
  readA(0, 0, a0);
  auto step = [&](int kt, auto odd_t, const bf16x8_t (&b)[TNW], bf16x8_t (&bn)[TNW]) {
    constexpr int ODD = decltype(odd_t)::value;
    const int pb = (kt >> 1) & 1;
    readS(pb, ODD, d);
    // the next step's codes (and, once a pair, the next pair's scales) into LDS; the
    // ones after that requested
    wstore(1 - ODD, rw);
    if (ODD) sstore(1 - pb, rs);
    rw = wload(kt + 2);
    if (ODD) rs = sload((kt >> 1) + 2);
    readA(ODD, 1, a1);
    __builtin_amdgcn_sched_barrier(0);
    mult(a0, b, q0);
    readA(ODD, 2, a0);
    mult(a1, b, q1);
    fold(0, q0, d);
    __builtin_amdgcn_sched_barrier(0);
    readA(ODD, 3, a1);
    mult(a0, b, q0);
    fold(1, q1, d);
    __builtin_amdgcn_sched_barrier(0);
    // the next stage of A has landed (this step's code and scale loads may be in
    // flight), every wavefront has read this one and written the next codes
    wait_vm_lgkm<1 + ODD>();
    __builtin_amdgcn_s_barrier();
    issue(ODD, min(kt + 2, KT - 1));
    readW(1 - ODD, bn);
    readA(1 - ODD, 0, a0);
    __builtin_amdgcn_sched_barrier(0);
    mult(a1, b, q1);
    fold(2, q0, d);
    fold(3, q1, d);
    __builtin_amdgcn_sched_barrier(0);
  };
  for (int kt = 0; kt < KT; kt += 2) {
    step(kt, std::integral_constant<int, 0>{}, b0, b1);
    step(kt + 1, std::integral_constant<int, 1>{}, b1, b0);
  }
  wait_vm_lgkm<0>();  // the last refills

  const bool vec = N % 4 == 0 && ldc % 4 == 0;
#pragma unroll
  for (int i = 0; i < TMW; ++i) {
    const int m = m0 + wm * 64 + i * 16 + fr;
    if (m < M) store_rows<EPI, TNW>(acc[i], C, ldc, H, ldh, N, m, n0 + wn * 64, fc, vec);
  }
}

// ------------------------------------------------------------ skinny (M <= 32)
// For a handful of rows (a batched decode step: one row per sequence) the product
// is bound by streaming W, like the decode GEMV, not by the matrix cores.  A
// workgroup owns 16 TN columns (weight rows) and all M (<= 16 TM) rows; its four
// wavefronts split K and add their partial tiles through LDS at the end.  A
// wavefront loads its weight fragments straight from memory into the operand
// registers of v_mfma_f32_16x16x32_bf16 (lane l: row n0 + 16 j + l % 16, eight
// consecutive K at 8 (l / 16)), two K steps per batch, double-buffered, every
// load unconditional (rows clamped; rows of A past M are clamped too and their
// outputs dropped), so a batch's wait leaves the next batch in flight.  The
// activation fragments (NT bf16 planes, TM row tiles) come from L2.
template <int NT, int TM, int TN>
struct SkinnyBatch {
  static constexpr int D = 2;  // K steps per batch
  bf16x8_t w[D][TN];
  bf16x8_t a[D][NT][TM];
};

template <int NT, int TM, int TN, int EPI>
__global__ __launch_bounds__(256) void k_gemm_skinny(const bf16_t* __restrict__ A,
                                                     size_t a_plane, int lda,
                                                     const bf16_t* __restrict__ W, int M, int N,
                                                     int K, float* __restrict__ C, int ldc,
                                                     ActBuf H, int ldh) {
  using Bt = SkinnyBatch<NT, TM, TN>;
  constexpr int D = Bt::D;
  __shared__ floatx4_t red[4][TM][TN][64];
  const int n0 = blockIdx.x * 16 * TN;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int fr = lane & 15, fk = (lane >> 4) * 8;
  const int KT = K / kBK;
  const int kt0 = wave * KT / 4, kt1 = (wave + 1) * KT / 4, nst = kt1 - kt0;
  const int nb = (nst + D - 1) / D;  // batches of this wavefront
  const bf16_t* wrow[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j) wrow[j] = W + (size_t)min(n0 + j * 16 + fr, N - 1) * K + fk;
  const bf16_t* arow[TM];
#pragma unroll
  for (int i = 0; i < TM; ++i) arow[i] = A + (size_t)min(i * 16 + fr, M - 1) * lda + fk;

  auto issue = [&](Bt& buf, int b) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      const int k = min(kt0 + b * D + d, KT - 1) * kBK;
#pragma unroll
      for (int j = 0; j < TN; ++j)
        buf.w[d][j] = __builtin_nontemporal_load(reinterpret_cast<const bf16x8_t*>(wrow[j] + k));
#pragma unroll
      for (int p = 0; p < NT; ++p)
#pragma unroll
        for (int i = 0; i < TM; ++i)
          buf.a[d][p][i] = *reinterpret_cast<const bf16x8_t*>(arow[i] + p * a_plane + k);
    }
  };
  floatx4_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = floatx4_t{0.f, 0.f, 0.f, 0.f};
  auto compute = [&](const Bt& buf, int b) {
#pragma unroll
    for (int d = 0; d < D; ++d)
      if (b * D + d < nst) {
#pragma unroll
        for (int p = 0; p < NT; ++p)
#pragma unroll
          for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(buf.a[d][p][i], buf.w[d][j],
                                                                  acc[i][j], 0, 0, 0);
      }
  };
  Bt b0, b1;
  issue(b0, 0);
  int b = 0;
  for (; b + 2 < nb; b += 2) {
    issue(b1, b + 1);
    compute(b0, b);
    issue(b0, b + 2);
    compute(b1, b + 1);
  }
  if (b + 1 < nb) {
    issue(b1, b + 1);
    compute(b0, b);
    compute(b1, b + 1);
  } else if (b < nb) {
    compute(b0, b);
  }

  // sum the four K ranges, then the epilogue (lane: rows 16 i + 4 (l / 16) + r,
  // column l % 16 of tile j)
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) red[wave][i][j][lane] = acc[i][j];
  __syncthreads();
  for (int t = wave; t < TM * TN; t += 4) {
    const int i = t / TN, j = t % TN;
    floatx4_t v = red[0][i][j][lane];
#pragma unroll
    for (int w = 1; w < 4; ++w) {
      const floatx4_t u = red[w][i][j][lane];
      v[0] += u[0]; v[1] += u[1]; v[2] += u[2]; v[3] += u[3];
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = i * 16 + (lane >> 4) * 4 + r, n = n0 + j * 16 + (lane & 15);
      const float o = EPI == GEMV_SWIGLU ? pair_swap(v[r]) : 0.f;
      epi_out<EPI>(C, ldc, H, ldh, M, N, m, n, v[r], o);
    }
  }
}

// ------------------------------------------------- few rows, staged through LDS
// The same product for up to 16 TM rows, K a multiple of 128: bound by streaming
// W.  A workgroup owns 64 WN weight rows (16 WN per wavefront) and all rows of A,
// and walks its K range in KC-deep slices through a ring of STG LDS stages, the
// weight slice and the activation slice (NT planes x 16 TM rows) fetched by
// global_load_lds_dwordx4 in whole 128-byte lines.  (Fragment-shaped loads
// straight into registers touch sixteen rows per instruction, 64 bytes each, and
// stream no faster than ~4.9 TB/s.)  The 16-byte chunks of a row are
// XOR-swizzled by the row's low bits, so a fragment read (sixteen rows, one
// chunk) covers all 64 banks once.
//
// Q8 weights: the slice holds the codes as they are (half the bytes); each
// fragment belongs to one wavefront, which converts its eight codes per lane to
// exact bf16 integers on the way into the matrix cores, sums a 32-deep block's
// NT products in a fresh accumulator and adds it times the block's scale (the
// lane's column).  A slice's scales go through LDS with its stage (in registers
// the compiler waited for every load in flight before each slice).
//
// Products with few weight rows are split along K over grid slots.  With c_split
// each split writes its own output, c_split elements after the one before, and the
// next kernel adds them (prompts: nothing depends on where a workgroup runs).
// Without it they are summed in the launch: the splits
// of a tile occupy workgroup indices of one residue mod 8, so they run on
// one XCD (dispatch deals workgroups to the XCDs in turn) and exchange their
// partials through its L2, as the decode attention merge does: each split
// stores its accumulators, waits for the L2 to acknowledge them, records its
// XCD and takes a ticket from the tile's counter; the last one drops its CU's
// L1, adds the partials in split order (so the sum does not depend on timing),
// applies the epilogue and resets the counter.  A split that ran elsewhere
// sets *fault.

// LDS chunk (16 bytes) of a row's chunk c, for rows of CH chunks: rows of 256 bytes
// all start at bank 0, rows of 128 bytes alternate between two halves.
template <int CH>
__device__ __forceinline__ int rows_swz(int row, int c) {
  return CH == 16 ? c ^ (row & 15) : c ^ ((row >> 1) & 7);
}

// Two LDS dwords, as a plain vector load: a load through a struct (uint2) or a bit
// cast carries no type information, and the compiler then waits for every
// direct-to-LDS load in flight first (s_waitcnt vmcnt(0), which empties the ring).
__device__ __forceinline__ u32x2_t lds_b64(const bf16_t* p) {
  const u32x2_t v = *reinterpret_cast<const u32x2_t*>(p);
  return v;
}

template <int NT, int TM, int WN, int KC, int STG, int EPI, bool Q8>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_gemm_rows(const bf16_t* __restrict__ A, size_t a_plane,
                                                   int lda, const void* __restrict__ Wv, int M,
                                                   int N, int K, int nsplit, int ks,
                                                   float* __restrict__ C, size_t c_split, int ldc,
                                                   ActBuf H, int ldh, floatx4_t* __restrict__ part,
                                                   int* __restrict__ sync,
                                                   int* __restrict__ fault, int drill,
                                                   const unsigned short* __restrict__ S) {
  constexpr int BN = 64 * WN;
  constexpr int CHA = KC / 8;                      // 16-byte chunks per activation row
  constexpr int CHW = Q8 ? KC / 16 : KC / 8;       // and per weight row
  constexpr int WUNITS = BN * CHW;                 // weight units (16 bytes) per slice
  // activation units per slice, whole instructions (the last units may be padding)
  constexpr int XUNITS = (NT * 16 * TM * CHA + 255) / 256 * 256;
  constexpr int PL = (WUNITS + XUNITS) / 256;      // units per lane per slice
  constexpr int SUNITS = Q8 ? 64 : 0;              // Q8: 256 dwords of block scales
  constexpr int STAGE = (WUNITS + XUNITS + SUNITS) * 8;  // bf16 elements per stage
  constexpr int VM = PL + (Q8 ? 1 : 0);            // vector-memory operations per slice
  static_assert(kRowsKC % KC == 0 && (CHA == 8 || CHA == 16) && (CHW == 8 || CHW == 16), "slices");
  static_assert(!Q8 || (KC == 128 && WN <= 2), "four block scales per row and slice");
  static_assert(STG >= 2 && STG <= 4, "stage ring of 2-4");
  // 32-deep steps whose fragments are read together, as the registers allow
  constexpr auto group = [](int n) { return n * (NT * TM + WN) * 4 + TM * WN * 4 <= 192; };
  constexpr int SG = Q8 ? (NT * TM <= 6 ? 4 : 2)
                     : group(KC / kBK) ? KC / kBK : group(2) ? 2 : 1;
  // Up to 32 rows of bf16 weights a slice's products are summed by themselves and added to
  // the earlier slices' sums while the next slice is read.  One fp32 sum over a whole K range
  // put the keys and values of prompts of up to 16 rows 40% further from 64 bits than
  // k_gemm_skinny's four over a quarter each (8B, three terms, 4.9e-7 against 3.6e-7; so
  // 1.7e-7), and gate/up's results up to 32.  Times are the same up to 16 rows; at 17 to 32,
  // where slices are 64 deep, three-term products take up to 4% more (8B QKV 13.4 -> 14.0 us,
  // LM head 185 -> 189), gate/up of two terms 41.2 as before.  (From 33 rows the tiles' sums
  // were no shorter, and it would cost 3 to 7%.)
  constexpr bool BLK = !Q8 && TM <= 2;
  extern __shared__ __attribute__((aligned(16))) bf16_t smem[];

  const int T = (N + BN - 1) / BN;
  const int loc = blockIdx.x / 8;
  const int t = blockIdx.x % 8 + 8 * (loc / nsplit), split = loc % nsplit;
  if (t >= T) return;
  const int n0 = t * BN, kbeg = split * ks;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;

  // unit u = (i * 4 + wave) * 64 + lane of a stage: weight row u / CHW for u <
  // WUNITS, else activation plane / row; its LDS chunk holds the row's global
  // chunk of the same swizzle (an involution)
  const char* src[PL];
  constexpr int WI = WUNITS / 256;                 // weight units of a lane come first
  static_assert(WUNITS % 256 == 0, "a lane's unit i is weights or activations for every lane");
#pragma unroll
  for (int i = 0; i < PL; ++i) {
    const int u = (i * 4 + wave) * 64 + lane;
    if (i < WI) {
      const int r = u / CHW, c = rows_swz<CHW>(r, u % CHW);
      src[i] = static_cast<const char*>(Wv) +
               ((size_t)min(n0 + r, N - 1) * K + kbeg) * (Q8 ? 1 : 2) + c * 16;
    } else {
      const int v = u - WUNITS, p = min(v / (16 * TM * CHA), NT - 1), r = (v / CHA) % (16 * TM);
      const int c = rows_swz<CHA>(r, v % CHA);
      src[i] = reinterpret_cast<const char*>(A + p * a_plane + (size_t)min(r, M - 1) * lda + kbeg) +
               c * 16;
    }
  }
  const int fr = lane & 15, g = lane >> 4;
  // Q8: lane tid fetches dword tid % 2 of weight row tid / 2's scales (four halves
  // per slice); past the tile's rows the last row's again
  const unsigned short* ssrc = nullptr;
  if constexpr (Q8)
    ssrc = S + (size_t)min(n0 + min(tid >> 1, BN - 1), N - 1) * (K / 32) + kbeg / 32 + 2 * (tid & 1);
  // Each workgroup starts its walk at its own slice and wraps around: in lockstep
  // every workgroup would read the same K offset of rows 8 KB apart, which
  // crowds a few HBM channels.  Offsets of 7 slices between the workgroups of
  // an XCD and 4 between XCDs measured best (a bare stream of the 8B gate/up
  // weights: 5.2 -> 6.0 TB/s; offsets of 1 slice: 4.2).
  const int KT = ks / KC;
  const int rot = ((blockIdx.x / 8) * 7 + (blockIdx.x % 8) * 4) % KT;
  auto issue = [&](int stage, int kt) {
    bf16_t* sb = smem + stage * STAGE;
    const int kk = kt + rot < KT ? kt + rot : kt + rot - KT;
#pragma unroll
    for (int i = 0; i < PL; ++i)
      dma16(reinterpret_cast<const bf16_t*>(src[i] + (size_t)kk * KC * (Q8 && i < WI ? 1 : 2)),
            sb + (i * 4 + wave) * 512);
    if constexpr (Q8) dma4(ssrc + kk * (KC / 32), sb + (WUNITS + XUNITS) * 8 + wave * 128);
  };

  floatx4_t acc[TM][WN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < WN; ++j) acc[i][j] = floatx4_t{0.f, 0.f, 0.f, 0.f};
  floatx4_t blk[TM][WN];  // BLK: the last slice's sums, not yet in acc
  auto fold = [&]() {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < WN; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[i][j][r] += blk[i][j][r];
  };
  if constexpr (BLK) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < WN; ++j) blk[i][j] = floatx4_t{0.f, 0.f, 0.f, 0.f};
  }
  auto compute = [&](int stage) {
    const bf16_t* sb = smem + stage * STAGE;
    const bf16_t* xb = sb + WUNITS * 8;
    if constexpr (BLK) fold();
    u32x2_t sc[WN];
    if constexpr (Q8) {
#pragma unroll
      for (int j = 0; j < WN; ++j)
        sc[j] = lds_b64(sb + (WUNITS + XUNITS) * 8 + ((wave * WN + j) * 16 + fr) * 4);
    }
    // the slice's 32-deep steps in groups of SG: a group's fragment reads are issued
    // together, and its products are independent chains
#pragma unroll
    for (int s0 = 0; s0 < KC / kBK; s0 += SG) {
      u32x2_t wq[SG][WN];
      bf16x8_t wf[SG][WN], xf[SG][TM][NT];
#pragma unroll
      for (int u = 0; u < SG; ++u) {
        const int st = s0 + u;
#pragma unroll
        for (int j = 0; j < WN; ++j) {
          const int wr = (wave * WN + j) * 16 + fr;
          if constexpr (Q8)  // 8 codes: half of chunk 2 st + g / 2
            wq[u][j] = lds_b64(sb + (wr * CHW + rows_swz<CHW>(wr, 2 * st + (g >> 1))) * 8 +
                               4 * (g & 1));
          else
            wf[u][j] = *reinterpret_cast<const bf16x8_t*>(
                sb + (wr * CHW + rows_swz<CHW>(wr, 4 * st + g)) * 8);
        }
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int p = 0; p < NT; ++p) {
            const int xr = i * 16 + fr;
            xf[u][i][p] = *reinterpret_cast<const bf16x8_t*>(
                xb + ((p * 16 * TM + xr) * CHA + rows_swz<CHA>(xr, 4 * st + g)) * 8);
          }
      }
      // the group's reads stay ahead of its products (the compiler otherwise deals them out
      // two or three at a time with a wait for each: 8B gate/up at 128 rows 94 -> 86 us)
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < SG; ++u) {
        if constexpr (Q8) {
#pragma unroll
          for (int j = 0; j < WN; ++j) wf[u][j] = q8_frag(wq[u][j]);
        }
      }
      floatx4_t q[SG][TM][WN];
      if constexpr (Q8) {
#pragma unroll
        for (int p = 0; p < NT; ++p)
#pragma unroll
          for (int u = 0; u < SG; ++u)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
              for (int j = 0; j < WN; ++j)
                q[u][i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                    xf[u][i][p], wf[u][j], p ? q[u][i][j] : floatx4_t{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
#pragma unroll
        for (int u = 0; u < SG; ++u)
#pragma unroll
          for (int j = 0; j < WN; ++j) {
            const int st = s0 + u;
            const unsigned w = st < 2 ? sc[j].x : sc[j].y;
            const float d =
                (float)__builtin_bit_cast(_Float16, (unsigned short)(st & 1 ? w >> 16 : w & 0xffffu));
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
              for (int r = 0; r < 4; ++r) acc[i][j][r] += q[u][i][j][r] * d;
          }
      } else {
#pragma unroll
        for (int u = 0; u < SG; ++u)
#pragma unroll
          for (int p = 0; p < NT; ++p)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
              for (int j = 0; j < WN; ++j) {
                floatx4_t& c = BLK ? blk[i][j] : acc[i][j];
                c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                    xf[u][i][p], wf[u][j],
                    BLK && s0 + u + p == 0 ? floatx4_t{0.f, 0.f, 0.f, 0.f} : c, 0, 0, 0);
              }
      }
    }
  };
#pragma unroll
  for (int s = 0; s < STG - 1; ++s)
    if (s < KT) issue(s, s);
  for (int kt = 0; kt < KT; ++kt) {
    const int ahead = min(STG - 2, KT - 1 - kt);  // later slices already issued
    if (ahead >= 2) wait_vm_lgkm<2 * VM>();
    else if (ahead == 1) wait_vm_lgkm<VM>();
    else wait_vm_lgkm<0>();
    __builtin_amdgcn_s_barrier();
    if (kt + STG - 1 < KT) issue((kt + STG - 1) % STG, kt + STG - 1);
    compute(kt % STG);
  }
  if constexpr (BLK) fold();

  auto out_row = [&](int i, int r) { return i * 16 + 4 * g + r; };
  auto out_col = [&](int j) { return n0 + (wave * WN + j) * 16 + fr; };
  // The residual rows are requested at once (clamped into C), in the split that adds
  // them: read where they are added, each value waited out a round trip of its own
  // (8B O at 64 rows 18.6 -> 15.9 us, down 40.3 -> 37.3 with the reads above; more than
  // 96 rows leave no registers for them).
  constexpr bool PRE = EPI == GEMV_RESID && TM <= 6;
  float old[TM][WN][4];
  auto load_old = [&]() {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < WN; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          old[i][j][r] = C[(size_t)min(out_row(i, r), M - 1) * ldc + min(out_col(j), N - 1)];
  };
  if (PRE && nsplit == 1) load_old();
  if (EPI == GEMV_STORE && c_split) {
    C += split * c_split;
  } else if (nsplit > 1) {
    __shared__ int s_last;
    constexpr int FR = TM * WN;  // accumulator tiles of a wavefront
    floatx4_t* slab = part + ((size_t)(t * nsplit + split) * 4 + wave) * FR * 64;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < WN; ++j) slab[(i * WN + j) * 64 + lane] = acc[i][j];
    const int me = xcc_id();
    int* line = sync + (size_t)t * kRowsSyncLine;
    if (tid == 0) line[32 + split] = me;
    // this thread's stores have reached the L2 (the empty asm keeps the compiler
    // from moving memory operations across the wait)
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0);
    asm volatile("" ::: "memory");
    __syncthreads();
    if (tid == 0) {
      const int old = __hip_atomic_fetch_add(line, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      s_last = old == nsplit - 1;
      if (old == nsplit - 1)  // reset for the next launch
        __hip_atomic_exchange(line, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    __syncthreads();
    if (!s_last) return;
    // drop this CU's L1 (it may hold lines of the partials from before their
    // stores); the loads below also bypass it (sc0)
    asm volatile("buffer_inv sc0" ::: "memory");
    const __amdgpu_buffer_rsrc_t rp =
        rsrc(part + (size_t)t * nsplit * 4 * FR * 64, (size_t)nsplit * 4 * FR * 64 * 16);
    const __amdgpu_buffer_rsrc_t rs = rsrc(line, kRowsSyncLine * 4);
    if (wave == 0 && lane < nsplit) {
      const int xo = __builtin_amdgcn_raw_buffer_load_b32(rs, (32 + lane) * 4, 0, 1);
      if (xo != me || drill) *fault = 1;
    }
    if (PRE) load_old();
    floatx4_t sum[TM][WN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < WN; ++j) sum[i][j] = floatx4_t{0.f, 0.f, 0.f, 0.f};
    // the partials of SU splits are in flight together (past the last split the last
    // one's again, not added)
    constexpr int SU = FR <= 2 ? 8 : FR <= 4 ? 4 : 2;
    for (int s0 = 0; s0 < nsplit; s0 += SU) {
      u32x4_t v[SU][TM][WN];
#pragma unroll
      for (int u = 0; u < SU; ++u)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < WN; ++j)
            v[u][i][j] = load_l2(rp, (int)((((size_t)min(s0 + u, nsplit - 1) * 4 + wave) * FR +
                                            i * WN + j) * 64 + lane) * 16);
#pragma unroll
      for (int u = 0; u < SU; ++u)
        if (s0 + u < nsplit) {
#pragma unroll
          for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < WN; ++j) {
              sum[i][j][0] += __uint_as_float(v[u][i][j].x);
              sum[i][j][1] += __uint_as_float(v[u][i][j].y);
              sum[i][j][2] += __uint_as_float(v[u][i][j].z);
              sum[i][j][3] += __uint_as_float(v[u][i][j].w);
            }
        }
    }
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < WN; ++j) acc[i][j] = sum[i][j];
  }
  // epilogue
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < WN; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = out_row(i, r), n = out_col(j);
        const float v = acc[i][j][r];
        if (PRE) {
          if (m < M && n < N) C[(size_t)m * ldc + n] = old[i][j][r] + v;
        } else {
          const float o = EPI == GEMV_SWIGLU ? pair_swap(v) : 0.f;
          epi_out<EPI>(C, ldc, H, ldh, M, N, m, n, v, o);
        }
      }
}

// ------------------------------------------------------------------- vector fp32
template <typename WT, int EPI>
__global__ __launch_bounds__(256) void k_gemm_f32(const float* __restrict__ A, int lda,
                                                  const WT* __restrict__ W, int M, int N, int K,
                                                  float* __restrict__ C, int ldc, ActBuf H,
                                                  int ldh, const unsigned short* __restrict__ S) {
  constexpr int BM = 64, BN = 64, BK = 16;
  __shared__ float As[BK][BM + 4];
  __shared__ float Ws[BK][BN + 4];
  const int tid = threadIdx.x, ty = tid >> 4, tx = tid & 15;
  const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;
  const int lr = tid >> 2, lk = (tid & 3) * 4;
  float acc[4][4] = {};
  for (int k0 = 0; k0 < K; k0 += BK) {
    const int am = m0 + lr, wn = n0 + lr;
    float4 a = am < M ? *reinterpret_cast<const float4*>(A + (size_t)am * lda + k0 + lk)
                      : make_float4(0, 0, 0, 0);
    float w[4];
    if (wn < N) {
      if constexpr (sizeof(WT) == 1) {  // Q8: (code - 128) * block scale
        const float d = (float)__builtin_bit_cast(_Float16, S[(size_t)wn * (K / 32) + (k0 + lk) / 32]);
#pragma unroll
        for (int e = 0; e < 4; ++e) w[e] = ((float)W[(size_t)wn * K + k0 + lk + e] - 128.f) * d;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) w[e] = Elem<WT>::load(W + (size_t)wn * K + k0 + lk + e);
      }
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) w[e] = 0.f;
    }
    __syncthreads();
    As[lk + 0][lr] = a.x; As[lk + 1][lr] = a.y; As[lk + 2][lr] = a.z; As[lk + 3][lr] = a.w;
#pragma unroll
    for (int e = 0; e < 4; ++e) Ws[lk + e][lr] = w[e];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < BK; ++k) {
      float av[4], wv[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) { av[i] = As[k][ty * 4 + i]; wv[i] = Ws[k][tx * 4 + i]; }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] += av[i] * wv[j];
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int m = m0 + ty * 4 + i, n = n0 + tx * 4 + j;
      epi_out<EPI>(C, ldc, H, ldh, M, N, m, n, acc[i][j], (j & 1) ? 0.f : acc[i][j | 1]);
    }
}

// ------------------------------------------------------------------- launchers
template <int NT, int EPI>
static hipError_t gemm_q8_launch(const ActBuf& A, int lda, const void* W, int M, int N, int K,
                                 float* C, int ldc, const ActBuf& H, int ldh, hipStream_t st,
                                 int nsplit = 1, size_t c_split = 0) {
  if (K % (2 * kBK * nsplit)) return hipErrorInvalidValue;  // K ranges of whole pairs of steps
  const int tiles = ((M + 127) / 128) * ((N + 127) / 128);
  const size_t lds = (2 * NT * 128 + 2 * 128) * kLDK * sizeof(bf16_t) + 4 * 128 * sizeof(float);
  const unsigned short* S = reinterpret_cast<const unsigned short*>(
      static_cast<const char*>(W) + q8_scale_offset(N, K));
  auto fn = &k_gemm_q8<NT, EPI>;
  if (lds > 65536)
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(fn),
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  hipLaunchKernelGGL(fn, dim3((tiles + 7) / 8 * 8, nsplit), dim3(256), lds, st, A.planes,
                     A.plane_stride, lda, static_cast<const uint8_t*>(W), S, M, N, K, K / nsplit, C,
                     c_split, ldc, H, ldh);
  return hipGetLastError();
}

template <int NT, int EPI, int WMW, int WNW, int TMW, int TNW, int STG, int GI, bool NMAJ>
static hipError_t gemm_dma_launch(const ActBuf& A, int lda, const void* W, int M, int N, int K,
                                  float* C, int ldc, const ActBuf& H, int ldh, hipStream_t st,
                                  int nsplit = 1, size_t c_split = 0) {
  constexpr int BM = 16 * TMW * WMW, BN = 16 * TNW * WNW;
  if (K % (2 * kBK * nsplit)) return hipErrorInvalidValue;  // K ranges of whole pairs of steps
  const int n_mt = (M + BM - 1) / BM, n_nt = (N + BN - 1) / BN;
  const int grid = NMAJ ? 8 * ((n_nt + 7) / 8) * n_mt : (n_mt * n_nt + 7) / 8 * 8;
  const size_t lds = (size_t)STG * (NT * BM + BN) * kLDK * sizeof(bf16_t);
  auto fn = &k_gemm_dma<NT, EPI, WMW, WNW, TMW, TNW, STG, GI, NMAJ>;
  if (lds > 65536)
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(fn),
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  hipLaunchKernelGGL(fn, dim3(grid, nsplit), dim3(64 * WMW * WNW), lds, st, A.planes,
                     A.plane_stride, lda, static_cast<const bf16_t*>(W), M, N, K, K / nsplit, C,
                     c_split, ldc, H, ldh);
  return hipGetLastError();
}

// (SwiGLU of three terms on 128 x 256 takes all 256 registers and spills 3, one of which
// is read back every second step; 128 x 128, which spills none, takes 627 us against 616
// at 1024 rows of 8B gate/up, 1254 against 1164 at 2048, 3217 against 2942 on 32B.)
template <int NT, int EPI>
static hipError_t gemm_dma_pick(const ActBuf& A, int lda, const void* W, int M, int N, int K,
                                float* C, int ldc, const ActBuf& H, int ldh, hipStream_t st,
                                int nsplit = 1, size_t c_split = 0) {
  switch (tile_shape(NT, M, N, K, nsplit, EPI == GEMV_SWIGLU)) {
    case TILE_128x256:
      return gemm_dma_launch<NT, EPI, 2, 2, 4, 8, 2, 1, true>(A, lda, W, M, N, K, C, ldc, H, ldh,
                                                              st, nsplit, c_split);
    case TILE_128x128:
      return gemm_dma_launch<NT, EPI, 2, 2, 4, 4, 2, 2, false>(A, lda, W, M, N, K, C, ldc, H, ldh,
                                                               st, nsplit, c_split);
    default:
      // (SwiGLU's dealt columns need four tiles a wavefront: 2 x 2 of 32 x 64)
      if constexpr (EPI == GEMV_SWIGLU)
        return gemm_dma_launch<NT, EPI, 2, 2, 2, 4, 3, NT % 2 ? 1 : 2, true>(
            A, lda, W, M, N, K, C, ldc, H, ldh, st, nsplit, c_split);
      else
        return gemm_dma_launch<NT, EPI, 1, 4, 4, 2, 3, 2, true>(A, lda, W, M, N, K, C, ldc, H, ldh,
                                                                st, nsplit, c_split);
  }
}

template <int EPI, bool Q8>
static hipError_t gemm_mfma(const ActBuf& A, int lda, const void* W, int M, int N, int K,
                            float* C, int ldc, const ActBuf& H, int ldh, hipStream_t st) {
  if (!Q8) {
    switch (A.nt) {
      case 1: return gemm_dma_pick<1, EPI>(A, lda, W, M, N, K, C, ldc, H, ldh, st);
      case 2: return gemm_dma_pick<2, EPI>(A, lda, W, M, N, K, C, ldc, H, ldh, st);
      case 3: return gemm_dma_pick<3, EPI>(A, lda, W, M, N, K, C, ldc, H, ldh, st);
      default: return hipErrorInvalidValue;
    }
  }
  switch (A.nt) {
    case 1: return gemm_q8_launch<1, EPI>(A, lda, W, M, N, K, C, ldc, H, ldh, st);
    case 2: return gemm_q8_launch<2, EPI>(A, lda, W, M, N, K, C, ldc, H, ldh, st);
    case 3: return gemm_q8_launch<3, EPI>(A, lda, W, M, N, K, C, ldc, H, ldh, st);
    default: return hipErrorInvalidValue;
  }
}

template <int NT, int TM, int TN, int EPI>
static hipError_t gemm_skinny_launch(const ActBuf& A, int lda, const void* W, int M, int N, int K,
                                     float* C, int ldc, const ActBuf& H, int ldh, hipStream_t st) {
  const int grid = (N + 16 * TN - 1) / (16 * TN);
  hipLaunchKernelGGL((k_gemm_skinny<NT, TM, TN, EPI>), dim3(grid), dim3(256), 0, st, A.planes,
                     A.plane_stride, lda, static_cast<const bf16_t*>(W), M, N, K, C, ldc, H, ldh);
  return hipGetLastError();
}

// Columns per workgroup: as many as still leave >= 512 workgroups (2 per CU).
template <int NT, int TM, int EPI>
static hipError_t gemm_skinny_tn(const ActBuf& A, int lda, const void* W, int M, int N, int K,
                                 float* C, int ldc, const ActBuf& H, int ldh, hipStream_t st) {
  if (N >= 64 * 512)
    return gemm_skinny_launch<NT, TM, 4, EPI>(A, lda, W, M, N, K, C, ldc, H, ldh, st);
  if (N >= 32 * 512)
    return gemm_skinny_launch<NT, TM, 2, EPI>(A, lda, W, M, N, K, C, ldc, H, ldh, st);
  return gemm_skinny_launch<NT, TM, 1, EPI>(A, lda, W, M, N, K, C, ldc, H, ldh, st);
}

template <int EPI>
static hipError_t gemm_skinny(const ActBuf& A, int lda, const void* W, int M, int N, int K,
                              float* C, int ldc, const ActBuf& H, int ldh, hipStream_t st) {
#define WICI_SKT(NT_)                                                                         \
  return M <= 16 ? gemm_skinny_tn<NT_, 1, EPI>(A, lda, W, M, N, K, C, ldc, H, ldh, st)        \
                 : gemm_skinny_tn<NT_, 2, EPI>(A, lda, W, M, N, K, C, ldc, H, ldh, st)
  switch (A.nt) {
    case 1: WICI_SKT(1);
    case 2: WICI_SKT(2);
    case 3: WICI_SKT(3);
    default: return hipErrorInvalidValue;
  }
#undef WICI_SKT
}

template <int NT, int TM, int WN, int KC, int STG, int EPI, bool Q8>
static hipError_t gemm_rows_launch(const ActBuf& A, int lda, const void* W, int M, int N, int K,
                                   int nsplit, float* C, size_t c_split, int ldc, const ActBuf& H,
                                   int ldh, float* part, int* sync, int* fault, hipStream_t st,
                                   int drill = 0) {
  const int T = (N + 64 * WN - 1) / (64 * WN);
  const int grid = 8 * ((T + 7) / 8) * nsplit;
  const size_t lds =
      (size_t)STG * (64 * WN * (Q8 ? 1 : 2) * KC + (NT * 16 * TM * 2 * KC + 4095) / 4096 * 4096 +
                     (Q8 ? 1024 : 0));
  const unsigned short* S =
      Q8 ? reinterpret_cast<const unsigned short*>(static_cast<const char*>(W) +
                                                   q8_scale_offset(N, K))
         : nullptr;
  auto fn = &k_gemm_rows<NT, TM, WN, KC, STG, EPI, Q8>;
  if (lds >= 65536)
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(fn),
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  hipLaunchKernelGGL(fn, dim3(grid), dim3(256), lds, st, A.planes, A.plane_stride, lda, W, M, N, K,
                     nsplit, K / nsplit, C, c_split, ldc, H, ldh,
                     reinterpret_cast<floatx4_t*>(part), sync, fault, drill, S);
  return hipGetLastError();
}

template <typename WT, int EPI>
static hipError_t gemm_f32(const ActBuf& A, int lda, const WT* W, int M, int N, int K, float* C,
                           int ldc, const ActBuf& H, int ldh, hipStream_t st) {
  dim3 grid((N + 63) / 64, (M + 63) / 64);
  const unsigned short* S =
      sizeof(WT) == 1 ? reinterpret_cast<const unsigned short*>(
                            reinterpret_cast<const char*>(W) + q8_scale_offset(N, K))
                      : nullptr;
  hipLaunchKernelGGL((k_gemm_f32<WT, EPI>), grid, dim3(256), 0, st, A.f32, lda, W, M, N, K, C,
                     ldc, H, ldh, S);
  return hipGetLastError();
}

// The launch shapes of the few-rows kernel: TM 16-row tiles, 64 WN weight rows per
// workgroup, KC-deep slices in STG stages.
template <int TM_, int WN_, int KC_, int STG_>
struct RowsShape {
  static constexpr int TM = TM_, WN = WN_, KC = KC_, STG = STG_;
};

template <int NT, int EPI, bool Q8>
static hipError_t gemm_rows(const RowsPlan& p, const ActBuf& A, int lda, const void* W, int M,
                            int N, int K, float* C, size_t c_split, int ldc, const ActBuf& H,
                            int ldh, float* part, int* sync, int* fault, hipStream_t st,
                            bool drill) {
  auto go = [&](auto shape) {
    using R = decltype(shape);
    return gemm_rows_launch<NT, R::TM, R::WN, R::KC, R::STG, EPI, Q8>(
        A, lda, W, M, N, K, p.nsplit, C, c_split, ldc, H, ldh, part, sync, fault, st, drill);
  };
  // Slices are 128 deep up to 32 rows and 64 from 33 on (48 rows: gate/up 60.5 us at
  // 128), the stages as many as leave two workgroups per CU, or one with wide slices.
  const bool wide = p.wn == 2;
  if constexpr (Q8) {
    switch (p.tm) {
      case 1: return go(RowsShape<1, 1, 128, 4>{});
      case 2: return wide ? go(RowsShape<2, 2, 128, 3>{}) : go(RowsShape<2, 1, 128, 3>{});
      case 3: return go(RowsShape<3, 1, 128, 2>{});
      default: return wide ? go(RowsShape<4, 2, 128, NT <= 2 ? 3 : 2>{}) : go(RowsShape<4, 1, 128, 2>{});
    }
  } else {
    switch (p.tm) {
      case 1: return wide ? go(RowsShape<1, 2, 128, 3>{}) : go(RowsShape<1, 1, 128, 3>{});
      case 2: return wide ? go(RowsShape<2, 2, 64, 4>{}) : go(RowsShape<2, 1, 128, 3>{});
      case 3: return wide ? go(RowsShape<3, 2, 64, 3>{}) : go(RowsShape<3, 1, 64, 3>{});
      case 4: return wide ? go(RowsShape<4, 2, 64, 3>{}) : go(RowsShape<4, 1, 64, 3>{});
      case 6: return go(RowsShape<6, 2, 64, 3>{});
      default: return go(RowsShape<8, 2, 64, 2>{});
    }
  }
}

template <int NT, int EPI>
static hipError_t gemm_rows_wt(int wt, const RowsPlan& p, const ActBuf& A, int lda, const void* W,
                               int M, int N, int K, float* C, size_t c_split, int ldc,
                               const ActBuf& H, int ldh, float* part, int* sync, int* fault,
                               hipStream_t st, bool drill) {
  return wt == W_Q8 ? gemm_rows<NT, EPI, true>(p, A, lda, W, M, N, K, C, c_split, ldc, H, ldh, part,
                                               sync, fault, st, drill)
                    : gemm_rows<NT, EPI, false>(p, A, lda, W, M, N, K, C, c_split, ldc, H, ldh,
                                                part, sync, fault, st, drill);
}

template <int NT>
static hipError_t gemm_split_nt(int wt, const ActBuf& A, int lda, const void* W, int M, int N,
                                int K, int nsplit, float* P, size_t p_split, hipStream_t st) {
  const ActBuf none{};
  if (gemm_rows_best(wt, NT, M, N, K, nsplit)) {
    const RowsPlan p = rows_plan(wt, GEMV_STORE, M, N, K, kAddedOutside, nsplit);
    return p.nsplit == nsplit
               ? gemm_rows_wt<NT, GEMV_STORE>(wt, p, A, lda, W, M, N, K, P, p_split, N, none, 0,
                                              nullptr, nullptr, nullptr, st, false)
               : hipErrorInvalidValue;
  }
  if (M <= 32 || K % (2 * kBK * nsplit)) return hipErrorInvalidValue;
  if (wt == W_Q8)
    return gemm_q8_launch<NT, GEMV_STORE>(A, lda, W, M, N, K, P, N, none, 0, st, nsplit, p_split);
  return gemm_dma_pick<NT, GEMV_STORE>(A, lda, W, M, N, K, P, N, none, 0, st, nsplit, p_split);
}

hipError_t launch_gemm_split(int wt, const ActBuf& A, int lda, const void* W, int M, int N, int K,
                             int nsplit, float* P, size_t p_split, hipStream_t st) {
  if (nsplit < 1 || (wt != W_BF16 && wt != W_Q8)) return hipErrorInvalidValue;
  switch (A.nt) {
    case 1: return gemm_split_nt<1>(wt, A, lda, W, M, N, K, nsplit, P, p_split, st);
    case 2: return gemm_split_nt<2>(wt, A, lda, W, M, N, K, nsplit, P, p_split, st);
    case 3: return gemm_split_nt<3>(wt, A, lda, W, M, N, K, nsplit, P, p_split, st);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_gemm_rows(int wt, int epi, const ActBuf& A, int lda, const void* W, int M,
                            int N, int K, float* C, int ldc, const ActBuf& H, int ldh,
                            float* part, size_t part_floats, int* sync, int* fault,
                            hipStream_t st, bool drill) {
  if (!gemm_rows_takes(wt, A.nt, M, K))
    return launch_gemm(wt, epi, A, lda, W, M, N, K, C, ldc, H, ldh, st);
  const bool merge = part && sync && fault;
  const RowsPlan p = rows_plan(wt, epi, M, N, K, part_floats, merge ? 16 : 1);
#define WICI_RW(NT_, E)                                                                          \
  return gemm_rows_wt<NT_, E>(wt, p, A, lda, W, M, N, K, C, 0, ldc, H, ldh, part, sync, fault, st, \
                              drill)
#define WICI_RW_NT(E)            \
  switch (A.nt) {                \
    case 1: WICI_RW(1, E);       \
    case 2: WICI_RW(2, E);       \
    default: WICI_RW(3, E);      \
  }
  switch (epi) {
    case GEMV_STORE: WICI_RW_NT(GEMV_STORE)
    case GEMV_RESID: WICI_RW_NT(GEMV_RESID)
    case GEMV_SWIGLU: WICI_RW_NT(GEMV_SWIGLU)
    default: return hipErrorInvalidValue;
  }
#undef WICI_RW_NT
#undef WICI_RW
}

hipError_t launch_gemm(int wt, int epi, const ActBuf& A, int lda, const void* W, int M, int N,
                       int K, float* C, int ldc, const ActBuf& H, int ldh, hipStream_t st) {
  if (K % kBK) return hipErrorInvalidValue;
#define WICI_EPI(CALL)                                      \
  switch (epi) {                                            \
    case GEMV_STORE: return CALL(GEMV_STORE);               \
    case GEMV_RESID: return CALL(GEMV_RESID);               \
    case GEMV_SWIGLU: return CALL(GEMV_SWIGLU);             \
    default: return hipErrorInvalidValue;                   \
  }
  if (A.nt == 0) {
#define WICI_F32(E) gemm_f32<WT_, E>(A, lda, static_cast<const WT_*>(W), M, N, K, C, ldc, H, ldh, st)
    if (wt == W_BF16) { using WT_ = bf16_t; WICI_EPI(WICI_F32) }
    if (wt == W_F32) { using WT_ = float; WICI_EPI(WICI_F32) }
    if (wt == W_Q8) { using WT_ = uint8_t; WICI_EPI(WICI_F32) }
#undef WICI_F32
    return hipErrorInvalidValue;
  }
#define WICI_SK(E) gemm_skinny<E>(A, lda, W, M, N, K, C, ldc, H, ldh, st)
  if (wt == W_BF16 && M <= 32) { WICI_EPI(WICI_SK) }
#undef WICI_SK
#define WICI_MF(E) gemm_mfma<E, Q8_>(A, lda, W, M, N, K, C, ldc, H, ldh, st)
  if (wt == W_BF16) { constexpr bool Q8_ = false; WICI_EPI(WICI_MF) }
  if (wt == W_Q8) { constexpr bool Q8_ = true; WICI_EPI(WICI_MF) }
#undef WICI_MF
#undef WICI_EPI
  return hipErrorInvalidValue;
}

}  // namespace wici
