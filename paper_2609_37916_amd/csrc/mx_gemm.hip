// Block-scaled minifloat matmul on the gfx950 MX matrix cores.
//
// The paper's ScaledMatMul path (Section VI, quantized inference) multiplies
// block-scaled minifloats -- FP8 / FP6 / FP4 grids -- and checks the result
// bit for bit against an F32 reference.  The element formats are the OCP MX
// ones (E4M3, E5M2, E2M3, E3M2, E2M1, 32 elements per E8M0 scale), which is
// exactly what v_mfma_scale_f32_32x32x64_f8f6f4 consumes: the matrix core
// applies the two blocks' scales itself, so codes and scales go from memory to
// the instruction untouched and the products are exact; only the fp32
// accumulation rounds.
//
//   y[m, n] = sum_k X(m, k) W(n, k),  X(m, k) = xs[m][k/32] * code_x[m][k], likewise W
//
// Storage (one row per m or n, K along the row): FP8 one byte per code, FP6
// four codes per three bytes (little-endian bit stream), FP4 two per byte
// (lower k in the low nibble); scales [rows][K/32] bytes.
//
// Design (three tiles, chosen by the number of tiles a call has, see
// launch_mx_typed: 256 x 128 and 128 x 128 with eight waves in a 4 x 2 grid,
// 64 x 64 with four):
//  * A stage is 128 k: the rows' 128 / 96 / 64 bytes (FP8 / FP6 / FP4) go
//    global -> LDS by DMA into a 128-byte row pitch with the 16-byte chunks
//    XOR-swizzled by (row / 2) mod 8; the rows' four scale bytes per stage go
//    by a dword DMA.  256 x 128: three stages (150 KB, one block per CU), so two
//    stages are in flight while one is multiplied, which is what hides the
//    memory latency -- with two 128 x 128 stages per block and two blocks per
//    CU only one stage per block was in flight and every stage waited for it.
//    The tall tile keeps the tile count at or below the CU count at the
//    benchmark shape (71 x 3 tiles for M = 18048, N = 384), so no CU runs a
//    second tile after the others have finished.
//  * Calls with few such tiles are bound by what one CU can load: 1 x 4096 x 4096
//    ran 32 blocks of 48 KB stages.  128 x 128 has four stages (136 KB, one block
//    per CU), 64 x 64 four (68 KB, two blocks per CU); eight 64 x 64 stages or 64 x
//    128 tiles measured slower (e4m3 60 x 2048 x 4096: 12.8 and 16.1 us against
//    11.7; 1000 x 4096 x 4096: 58.3 and 52.7 against 52.0).
//  * Operand layout of the instruction (lane l: row l % 32, half h = l / 32),
//    checked on the GPU against the oracle: FP6 / FP4 lanes hold the 32 codes
//    of block h contiguously; FP8 lanes hold bytes 16h .. 16h+15 of block 0 in
//    their first four registers and of block 1 in the last four.  Lane half h
//    supplies the scale of block h (byte 0 of the scale register).
//  * The weight rows are the instruction's A operand, the activation rows its
//    B operand, so each lane ends up with one output row and four consecutive
//    output columns per register quad: 16-byte stores.
#include "common.hpp"
#include "kernels.hpp"

namespace rlx {
namespace {

constexpr int kMxStageK = 128;     // k per stage
constexpr int kMxPitch = 128;      // LDS bytes per staged row

// LDS of a stage: the rows, then one 256-byte scale DMA per wave: x rows, then
// w rows, then (the waves left over) copies that are never read, so every wave
// issues as many loads per stage.
__host__ __device__ constexpr int mx_stage_bytes(int BM, int BN, int NW) { return (BM + BN) * kMxPitch + NW * 256; }

__host__ __device__ constexpr int mx_bits(int fmt) { return fmt <= 1 ? 8 : (fmt <= 3 ? 6 : 4); }

__device__ __forceinline__ int mx_swz(int row, int chunk) { return chunk ^ ((row >> 1) & 7); }

typedef int mx_v8i __attribute__((ext_vector_type(8)));

// The instruction operand of one lane: row r of a staged operand, MFMA step s
// (0 or 1) of the stage, lane half h.
template <int FMT>
__device__ __forceinline__ mx_v8i mx_fragment(const uint8_t* rows, int r, int s, int h) {
  const uint8_t* base = rows + r * kMxPitch;
  auto chunk = [&](int c) { return *reinterpret_cast<const uint4*>(base + mx_swz(r, c) * 16); };
  mx_v8i v;
  if constexpr (mx_bits(FMT) == 8) {
    const uint4 a = chunk(4 * s + h), b = chunk(4 * s + 2 + h);
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
    v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
  } else if constexpr (mx_bits(FMT) == 6) {
    // block 2s + h is bytes 24(2s + h) .. +23: chunks (3s, 3s+1) from byte 0
    // for h = 0, chunks (3s+1, 3s+2) from byte 8 for h = 1
    const uint4 a = chunk(3 * s + h), b = chunk(3 * s + 1 + h);
    v[0] = h ? a.z : a.x; v[1] = h ? a.w : a.y; v[2] = h ? b.x : a.z;
    v[3] = h ? b.y : a.w; v[4] = h ? b.z : b.x; v[5] = h ? b.w : b.y;
    v[6] = 0; v[7] = 0;
  } else {
    const uint4 a = chunk(2 * s + h);
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
    v[4] = 0; v[5] = 0; v[6] = 0; v[7] = 0;
  }
  return v;
}

// WMW x WNW waves of BM/WMW x BN/WNW outputs, S stages in the ring.
template <int BM, int BN, int WMW, int WNW, int S, int FX, int FW>
__global__ __launch_bounds__(WMW * WNW * 64) void mx_gemm_kernel(MxGemmParams p) {
  constexpr int NW = WMW * WNW, WM = BM / WMW, WN = BN / WNW, TM = WM / 32, TN = WN / 32;
  constexpr int kOpBytes = (BM + BN) * kMxPitch, kStageBytes = mx_stage_bytes(BM, BN, NW);
  constexpr int kOutPitch = BN + 4;  // floats per LDS row of the output tile (16-byte aligned, rows 4 banks apart)
  // per wave per stage: rows * 128 B / (waves * 1 KB) chunk DMAs + 1 scale DMA
  constexpr int CL = kOpBytes / (NW * 1024), LPS = CL + 1;
  static_assert((BM + BN) / 64 <= NW && kOpBytes % (NW * 1024) == 0 && (S - 2) * LPS < 64, "DMA layout");
  static_assert(BM * kOutPitch * 4 <= S * kStageBytes && S * kStageBytes <= 160 * 1024, "output tile in the stage ring");
  __shared__ __attribute__((aligned(1024))) uint8_t smem[S * kStageBytes];
  const int M = p.M, N = p.N, K = p.K;
  const int n_tiles = N / BN;
  const int live = n_tiles * ((M + BM - 1) / BM);
  const int bid = blockIdx.x;
  if (bid >= live) return;
  // XCD-aware order: workgroups go round-robin over the 8 XCDs; XCD x takes a
  // contiguous run of tiles (row-major over (row tile, column tile))
  const int q8 = live >> 3, r8 = live & 7, xcd = bid & 7;
  const int tile = xcd * q8 + min(xcd, r8) + (bid >> 3);
  const int m0 = (tile / n_tiles) * BM, n0 = (tile % n_tiles) * BN;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WNW, wn = wave % WNW, l32 = lane & 31, h = lane >> 5;
  const int KT = K / kMxStageK;
  constexpr int RBX = kMxStageK * mx_bits(FX) / 8, RBW = kMxStageK * mx_bits(FW) / 8;  // bytes per stage row
  const size_t pitch_x = (size_t)K * mx_bits(FX) / 8, pitch_w = (size_t)K * mx_bits(FW) / 8;
  const int sb_row = K / 32;  // scale bytes per row

  // Chunk DMA: instruction i of wave w fills staged rows 8(w + NW i) .. +7; lane
  // lands at row (lane >> 3), physical chunk (lane & 7).  Chunks past the
  // format's row bytes are never read; their lanes fetch chunk 0 again.
  const uint8_t* src[CL];
  int step_bytes[CL];
#pragma unroll
  for (int i = 0; i < CL; ++i) {
    const int row = (wave + NW * i) * 8 + (lane >> 3);
    const int c = mx_swz(row, lane & 7);
    if (row < BM) {
      const int m = min(m0 + row, M - 1);
      src[i] = reinterpret_cast<const uint8_t*>(p.x) + (size_t)m * pitch_x + (c * 16 < RBX ? c * 16 : 0);
      step_bytes[i] = RBX;
    } else {
      src[i] = reinterpret_cast<const uint8_t*>(p.w) + (size_t)(n0 + row - BM) * pitch_w + (c * 16 < RBW ? c * 16 : 0);
      step_bytes[i] = RBW;
    }
  }
  // Scale DMA, one dword per row and stage: the first BM/64 waves x rows 64w ..
  // 64w+63, the next BN/64 w rows likewise, the others w rows again (unread)
  const uint8_t* ssrc;
  {
    constexpr int XW = BM / 64, WW = BN / 64;
    const int row = (wave < XW ? wave : (wave - XW) % WW) * 64 + lane;
    ssrc = wave < XW ? p.x_scales + (size_t)min(m0 + row, M - 1) * sb_row
                     : p.w_scales + (size_t)(n0 + row) * sb_row;
  }
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)smem;
  auto issue = [&](int kt, int buf) {
    const uint32_t sbase = lds0 + buf * kStageBytes;
#pragma unroll
    for (int i = 0; i < CL; ++i)
      lds_dma16(src[i] + (size_t)kt * step_bytes[i],
                __builtin_amdgcn_readfirstlane(sbase + (wave + NW * i) * 8 * kMxPitch));
    lds_dma4(ssrc + kt * 4, __builtin_amdgcn_readfirstlane(sbase + kOpBytes + wave * 256));
  };

  typedef float f32x16 __attribute__((ext_vector_type(16)));
  f32x16 acc[TM][TN];
#pragma unroll
  for (int a = 0; a < TM; ++a)
#pragma unroll
    for (int b = 0; b < TN; ++b)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.0f;

  // Stages kt .. kt + S - 2 are in flight when stage kt's wait begins; stage
  // kt + S - 1 is issued after the barrier that follows it, into the buffer of
  // stage kt - 1, which every wave has finished multiplying by then.
  issue(0, 0);
#pragma unroll
  for (int st = 1; st < S - 1; ++st)
    if (st < KT) issue(st, st);
  for (int kt = 0; kt < KT; ++kt) {
    const int buf = kt % S;
    if (kt + S - 2 < KT)
      wait_vmcnt<LPS * (S - 2)>();  // stage kt landed; the S - 2 after it in flight
    else
      wait_stage<LPS, S - 3>(KT - 1 - kt);
    __syncthreads();
    if (kt + S - 1 < KT) issue(kt + S - 1, (kt + S - 1) % S);
    const uint8_t* xs = smem + buf * kStageBytes;
    const uint8_t* ws = xs + BM * kMxPitch;
    const uint32_t* sx = reinterpret_cast<const uint32_t*>(xs + kOpBytes);  // [BM] x rows, then [BN] w rows
    const uint32_t* sw = sx + BM;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      mx_v8i xf[TM], wf[TN];
      int xsc[TM], wsc[TN];
#pragma unroll
      for (int t = 0; t < (TM > TN ? TM : TN); ++t) {
        if (t < TM) {
          const int rx = wm * WM + t * 32 + l32;
          xf[t] = mx_fragment<FX>(xs, rx, s, h);
          xsc[t] = (int)((sx[rx] >> (8 * (2 * s + h))) & 0xFF);
        }
        if (t < TN) {
          const int rw = wn * WN + t * 32 + l32;
          wf[t] = mx_fragment<FW>(ws, rw, s, h);
          wsc[t] = (int)((sw[rw] >> (8 * (2 * s + h))) & 0xFF);
        }
      }
#pragma unroll
      for (int tm = 0; tm < TM; ++tm)
#pragma unroll
        for (int tn = 0; tn < TN; ++tn)
          acc[tm][tn] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(wf[tn], xf[tm], acc[tm][tn], FW, FX, 0,
                                                                         wsc[tn], 0, xsc[tm]);
    }
  }

  // Epilogue through LDS (the stage ring is free once every wave is past the
  // loop): lane holds output row wm*WM + tm*32 + l32 of the tile and, per
  // register quad i, columns wn*WN + tn*32 + 8i + 4h .. +3.  The tile goes to
  // LDS row-major, then every wave stores whole rows: written from the
  // instruction layout, each store touched 32 rows with 32 bytes apiece.
  float* out_lds = reinterpret_cast<float*>(smem);
  __syncthreads();
#pragma unroll
  for (int tm = 0; tm < TM; ++tm)
#pragma unroll
    for (int tn = 0; tn < TN; ++tn)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int r = wm * WM + tm * 32 + l32, c = wn * WN + tn * 32 + 8 * i + 4 * h;
        *reinterpret_cast<float4*>(out_lds + r * kOutPitch + c) =
            make_float4(acc[tm][tn][4 * i], acc[tm][tn][4 * i + 1], acc[tm][tn][4 * i + 2], acc[tm][tn][4 * i + 3]);
      }
  __syncthreads();
  constexpr int kRowThreads = BN / 4;                   // float4 per row
  constexpr int kRowsPerPass = NW * 64 / kRowThreads;   // rows stored per pass
  const int rr = tid / kRowThreads, c4 = (tid % kRowThreads) * 4;
#pragma unroll 4
  for (int r = rr; r < BM; r += kRowsPerPass) {
    const int m = m0 + r;
    if (m < M)
      *reinterpret_cast<float4*>(p.y + (size_t)m * N + n0 + c4) = *reinterpret_cast<const float4*>(out_lds + r * kOutPitch + c4);
  }
}

template <int BM, int BN, int WMW, int WNW, int S, int FX, int FW>
hipError_t launch_mx_tile(const MxGemmParams& p, hipStream_t s) {
  const dim3 grid((p.N / BN) * ((p.M + BM - 1) / BM)), block(WMW * WNW * 64);
  RLX_LOG_LAUNCH("mx_gemm_kernel", grid, block, 0, "tile=%dx%d stages=%d formats=%d,%d M=%d N=%d K=%d", BM, BN, S, FX, FW,
                 p.M, p.N, p.K);
  hipLaunchKernelGGL((mx_gemm_kernel<BM, BN, WMW, WNW, S, FX, FW>), grid, block, 0, s, p);
  return hipGetLastError();
}

template <int FX, int FW>
hipError_t launch_mx_typed(const MxGemmParams& p, hipStream_t s) {
  // Smaller tiles use more CUs and start with less to load; larger ones stream fewer
  // bytes per product.  64 x 64 run two blocks per CU, so up to 512 of them are
  // one pass over the chip; 128 x 128 one block, 256 of them.  Measured (us,
  // 256x128 / 128x128 / 64x64 tiles, e4m3, M x N x K):
  //   1 x 4096 x 4096     30.5 / 19.9 / 11.6   (64 64x64 tiles)
  //   200 x 4096 x 1024   11.4 / 8.4 / 5.6     (256)
  //   4096 x 512 x 4096   35.3 / 28.0 / 22.8   (512)
  //   1100 x 2048 x 1024  12.7 / 9.8 / 10.8    (576; 144 128x128 tiles)
  //   1000 x 4096 x 4096  39.1 / 35.9 / 52.0   (1024; 256)
  //   2300 x 2048 x 1024  14.9 / 17.5 / 15.4   (1152; 288)
  //   4000 x 4096 x 4096  96.2 / 127.0 / 190.2 (4032; 1024)
  // (e2m1 alike.)  A row's products are added in the same order in all three.
  const auto tiles = [&](int bm, int bn) { return (long)((p.M + bm - 1) / bm) * (p.N / bn); };
  if (tiles(64, 64) <= 512) return launch_mx_tile<64, 64, 2, 2, 4, FX, FW>(p, s);
  if (tiles(128, 128) <= 256) return launch_mx_tile<128, 128, 4, 2, 4, FX, FW>(p, s);
  return launch_mx_tile<256, 128, 4, 2, 3, FX, FW>(p, s);
}

template <int FX>
hipError_t launch_mx_w(const MxGemmParams& p, hipStream_t s) {
  switch (p.fw) {
    case 0: return launch_mx_typed<FX, 0>(p, s);
    case 1: return launch_mx_typed<FX, 1>(p, s);
    case 2: return launch_mx_typed<FX, 2>(p, s);
    case 3: return launch_mx_typed<FX, 3>(p, s);
    case 4: return launch_mx_typed<FX, 4>(p, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace

bool mx_gemm_supported(int M, int N, int K) { return M >= 0 && N > 0 && K > 0 && N % 128 == 0 && K % 128 == 0; }

hipError_t launch_mx_gemm(const MxGemmParams& p, hipStream_t s) {
  if (!mx_gemm_supported(p.M, p.N, p.K) || p.fx < 0 || p.fx > 4 || p.fw < 0 || p.fw > 4) return hipErrorInvalidValue;
  if (p.M == 0) return hipSuccess;
  switch (p.fx) {
    case 0: return launch_mx_w<0>(p, s);
    case 1: return launch_mx_w<1>(p, s);
    case 2: return launch_mx_w<2>(p, s);
    case 3: return launch_mx_w<3>(p, s);
    case 4: return launch_mx_w<4>(p, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace rlx
