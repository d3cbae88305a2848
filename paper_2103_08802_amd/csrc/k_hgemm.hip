// Halo GEMM kernel for the large wide 3x3 convolutions without a BN prologue (forward of activated
// inputs, data gradient) of the parareal VGG sub-networks and the paper's coarse blocks (Table vgg,
// Sec. 4.2.1): bf16 v_mfma_f32_32x32x16_bf16 with fp32 accumulation.
//
// What bounds these layers is feeding the matrix cores: a 128 x 128 tile that stages its input rows
// once per filter tap moves 15.6 KB from L2 per MFLOP, writes them to LDS through registers and reads
// 64 x 64 wave tiles back at the LDS's full rate.  Here a workgroup of four waves owns 256 output
// pixels x TN output channels, and per 64-channel chunk its input pixels plus the one-pixel halo are
// staged ONCE for all nine taps (4.5 to 5.1 KB per MFLOP): every tap reads its fragments from the same LDS
// rows at a shifted row, padding taps from a row of zeros.  The filter rows of a tap (TN x 64
// channels) are double-buffered.  All staging is by 16-byte global-to-LDS loads (no registers, no
// vector instructions); such a load writes its wave's 64 chunks contiguously, so bank conflicts are
// avoided by choice of the global chunk each lane fetches: row r of 128 bytes keeps channel chunk c in
// slot c ^ (r & 7).  Waves of 128 x 64 (TN = 128) read 6 KB of LDS per 8 MFMAs; two workgroups share a
// CU (LDS, 256 registers), so one computes while the other waits for its chunk.
//
// The 256 output pixels are consecutive pixels of the flattened (image, row, column) index for maps up to
// HG_FLATW columns wide (halo: W + 1 pixels on both sides); wider maps, whose rows would make that halo
// larger than the tile, take 16 x 16 pixel patches (halo rows 18 x 18).
//
// Measured (VGG layers at 224 px, batch 128, one stream; gemm_conv_kernel before): 128-column tiles, forward
// 740 -> 1050 TFLOP/s, data gradient 766 -> 1070; 64-column tiles 393 -> 615 and 446 -> 745.  A library
// product of 8192 x 8192 matrices runs at 1116 on the same card; the 64-column tiles are held by LDS
// reads (their 64 x 64 wave tiles need the full rate, 128 bytes a clock).
//
// K runs channel chunk outer, tap inner, 16 channels per MFMA: the order of gemm_conv_kernel, so the
// two kernels' results are bit-identical; the fp32 tile goes through the same epilogue in two 128-pixel
// halves (its BN partial rows, of the same pixels in flat tiles and of a patch's half in others).
#include "device_common.h"
#include "pnn_internal.h"
#include "conv_epilogue.h"

#include <type_traits>

#pragma clang diagnostic ignored "-Winline-asm"   // m0 is a reserved register: clobbering it is what is meant

namespace pnn {

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int HM = HG_BM;                         // output pixels per workgroup
constexpr int HROW = 128;                         // LDS bytes of a row: 64 channels
constexpr int HA_ROWS = HG_AROWS;                 // input rows staged, at most (a multiple of 8)

// 64 lanes' 16 bytes each (base + voff per lane) into LDS bytes [lds, lds + 1024) in lane order.  A load to LDS
// needs one wait state after the scalar write of m0 that names its LDS address (the compiler adds it between
// instructions of its own, not inside an asm block).
__device__ __forceinline__ void load_lds16(uint32_t lds, const void* base, uint32_t voff) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(voff), "s"(base)
               : "memory", "m0");
}
// the wave's own global-to-LDS loads have landed; then every wave's have
__device__ __forceinline__ void lds_ready() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

}  // namespace

// Problems: 3x3, stride 1, pad 1, output grid = input grid, Cg % 64 == 0, ncol % TN == 0, bf16, no
// prologue; W <= HG_FLATW, or P and Q multiples of 16 (hgemm_ok)
template <int MODE, int TN>
__global__ __launch_bounds__(256, 2) void hgemm_conv_kernel(const ConvLaunch L) {
  using T = uint16_t;
  constexpr int VE = 8;
  constexpr int MI = TN == 128 ? 4 : 2;           // 32-row MFMA blocks per wave (two 32-column blocks)
  constexpr int NBI = TN / 32;                    // filter loads per wave and tap (8 rows each)
  constexpr int NAI = (HA_ROWS + 31) / 32;               // input loads per wave and chunk, at most
  constexpr int A_BYTES = (HA_ROWS + 1) * HROW;   // staged rows and the row of zeros
  constexpr int B_BYTES = TN * HROW;              // one filter buffer
  constexpr int LDA = TN + 4;
  constexpr int EPI_BYTES = 128 * LDA * 4 + 8 * TN * 4;   // staged half tile; BN constants; pivot
  constexpr int SMEM = A_BYTES + 2 * B_BYTES > EPI_BYTES ? A_BYTES + 2 * B_BYTES : EPI_BYTES;
  static_assert(2 * SMEM <= 160 * 1024, "two workgroups per CU");
  __shared__ __attribute__((aligned(1024))) unsigned char smem[SMEM];

  const int gi = find_group(L);
  const ConvProb& P = L.p[gi];
  const int local = blockIdx.x - P.tile_begin;
  // Workgroups go to the eight XCDs round-robin by blockIdx.  The column tiles of a row tile read the
  // same input rows, and neighbouring row tiles share their halo: each XCD takes a contiguous run of
  // row tiles, the column tiles of one after the other.
  const int tr = (P.tiles_m + 1) / 2;             // 256-pixel row tiles
  const int per = tr / 8;
  int tm, tn;
  if (local < 8 * per * P.tiles_n) {
    const int q = local >> 3;
    tm = (local & 7) * per + q / P.tiles_n;
    tn = q % P.tiles_n;
  } else {
    const int l2 = local - 8 * per * P.tiles_n;
    tm = 8 * per + l2 / P.tiles_n;
    tn = l2 % P.tiles_n;
  }
  const int n0 = tn * TN;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int r32 = lane & 31, kh = lane >> 5;
  const int wr = TN == 128 ? wave >> 1 : wave, wc = TN == 128 ? wave & 1 : 0;
  const bool patch = P.Q > HG_FLATW;
  const int W = P.Q, H = P.P, PQ = H * W;

  // the tile's first pixel (flat) or patch origin
  const int m0 = tm * HM;
  int img = 0, py = 0, px = 0;
  if (patch) {
    const int pw = W >> 4, pp = pw * (H >> 4);
    img = tm / pp;
    const int rem = tm - img * pp;
    py = rem / pw * 16;
    px = (rem - rem / pw * pw) * 16;
  }

  // input loads: load j of the wave fills rows 8 (wave + 4 j) .. + 7; the lane's row and channel chunk
  const int lrow = lane >> 3, lch = (lane & 7) ^ lrow;
  const int R = patch ? 18 * 18 : HM + 2 * W + 2;
  uint32_t aoff[NAI];
#pragma unroll
  for (int j = 0; j < NAI; ++j) {
    const int r = 8 * (wave + 4 * j) + lrow;
    long pix;
    if (patch) {
      const int y = r / 18, x = r - 18 * y;       // (rows past the halo: clamped like its padding)
      const int ih = min(max(py - 1 + y, 0), H - 1), iw = min(max(px - 1 + x, 0), W - 1);
      pix = (long)img * PQ + ih * W + iw;
    } else {
      pix = min(max((long)m0 - W - 1 + r, 0L), (long)P.M - 1);
    }
    aoff[j] = (uint32_t)((pix * P.Cg + 8 * lch) * 2);
  }
  const uint32_t lds0 = (uint32_t)(size_t)(__attribute__((address_space(3))) unsigned char*)smem;
  const uint32_t boff = (uint32_t)(((long)(n0 + 8 * wave + lrow) * P.K + 8 * lch) * 2);
  const uint32_t bstep = (uint32_t)(32L * P.K * 2);   // 32 filter rows on
  const int nai = (R + 31 - 8 * wave) / 32;           // the wave's loads of a chunk: rows below R (and up to 7 more)

  // the lane's fragment rows: LDS row of the output pixel itself and the taps inside the image
  int arow[MI];
  unsigned amask[MI];
  const int RS = patch ? 18 : W;
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    const int lm = wr * (32 * MI) + 32 * i + r32;
    int p, q;
    bool v = true;
    if (patch) {
      p = py + (lm >> 4);
      q = px + (lm & 15);
      arow[i] = ((lm >> 4) + 1) * 18 + (lm & 15) + 1;
    } else {
      const int m = m0 + lm;
      v = m < P.M;
      const int mm = v ? m : 0;
      const int n = div_l2(mm, PQ, P.pq_log2);
      const int rem = mm - n * PQ;
      p = div_l2(rem, W, P.q_log2);
      q = rem - p * W;
      arow[i] = lm + W + 1;
    }
    unsigned mk = 0;
#pragma unroll
    for (int t = 0; t < 9; ++t) {
      const int dr = MODE == MODE_FWD ? t / 3 - 1 : 1 - t / 3;
      const int dq = MODE == MODE_FWD ? t % 3 - 1 : 1 - t % 3;
      mk |= (v && (unsigned)(p + dr) < (unsigned)H && (unsigned)(q + dq) < (unsigned)W) ? 1u << t : 0u;
    }
    amask[i] = mk;
  }
  uint32_t bfr[4];                                    // byte offset of the lane's filter fragments, by 16-channel step
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) bfr[kk] = (wc * 64 + r32) * HROW + ((32 * kk + 16 * kh) ^ ((r32 & 7) << 4));

  f32x16 acc[MI][2];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  const char* in = (const char*)P.in;
  const char* wm = (const char*)P.wmat;
  const int nchunk = P.Cg / 64;
  auto load_a = [&](int cb) {
#pragma unroll
    for (int j = 0; j < NAI; ++j)
      if (j < nai) load_lds16(lds0 + (wave + 4 * j) * 1024, in + cb * HROW, aoff[j]);
  };
  auto load_b = [&](int cb, int tap, int buf) {
    const char* base = wm + ((long)tap * P.Cg + cb * 64) * 2;
#pragma unroll
    for (int j = 0; j < NBI; ++j)
      load_lds16(lds0 + A_BYTES + buf * B_BYTES + (wave + 4 * j) * 1024, base, boff + j * bstep);
  };

  if (tid < HROW / 4) *(float*)(smem + HA_ROWS * HROW + 4 * tid) = 0.f;
  load_b(0, 0, 0);
  int buf = 0;
  for (int cb = 0; cb < nchunk; ++cb) {
    load_a(cb);
#pragma unroll 1
    for (int tap = 0; tap < 9; ++tap) {
      lds_ready();
      // the buffer read by the step before is free: every wave is past it
      if (tap < 8) load_b(cb, tap + 1, buf ^ 1);
      else if (cb + 1 < nchunk) load_b(cb + 1, 0, buf ^ 1);
      const int dr = MODE == MODE_FWD ? tap / 3 - 1 : 1 - tap / 3;
      const int dq = MODE == MODE_FWD ? tap % 3 - 1 : 1 - tap % 3;
      const int shift = dr * RS + dq;
      uint32_t ab[MI], ax[MI];
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        const int rr = arow[i] + shift;
        ab[i] = ((amask[i] >> tap) & 1u) ? rr * HROW : HA_ROWS * HROW;
        ax[i] = ((rr & 7) << 4) ^ (16 * kh);
      }
      const unsigned char* bb = smem + A_BYTES + buf * B_BYTES;
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        bf16x8 a[MI], b[2];
#pragma unroll
        for (int i = 0; i < MI; ++i) a[i] = *(const bf16x8*)(smem + (ab[i] + ((32 * kk) ^ ax[i])));
#pragma unroll
        for (int j = 0; j < 2; ++j) b[j] = *(const bf16x8*)(bb + bfr[kk] + 32 * j * HROW);
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
      }
      buf ^= 1;
    }
    lds_ready();                                      // every wave is past the chunk: its rows may be overwritten
  }

  // epilogue: the 128-pixel halves one after the other through the staged fp32 tile
  float* accs = (float*)smem;
  float* bn_s = accs + 128 * LDA;
  float* piv = bn_s + 7 * TN;
  const bool bnmask = MODE == MODE_BWD && (P.flags & (EPI_BN_MASK | EPI_BN_APPLY));
  constexpr int ncc = TN / VE, rpp = 256 / ncc, NCH = 128 / rpp;
  const int cc0 = (tid % ncc) * VE;
  const void* pf = (MODE == MODE_FWD) ? P.res
                   : ((P.flags & EPI_STORE_F32) ? nullptr : (bnmask ? P.zsrc : P.res));
  const void* pf2 = (MODE == MODE_FWD) ? P.ext : ((P.flags & EPI_BN_APPLY) ? P.res : nullptr);
  if (bnmask && tid < TN) {
    const int col = n0 + tid;
#pragma unroll
    for (int k = 0; k < 4; ++k) bn_s[k * TN + tid] = P.bnst[k * P.ncol + col];
    if (P.flags & EPI_BN_APPLY) {
#pragma unroll
      for (int k = 0; k < 3; ++k) bn_s[(4 + k) * TN + tid] = P.coef[k * P.ncol + col];
    }
  }
#pragma unroll 1
  for (int h = 0; h < 2; ++h) {
    const int tmh = 2 * tm + h;                       // the half's BN partial row
    if (tmh * 128 >= P.M) break;
    // row r of the half -> output pixel
    auto rowm = [&](int r) {
      return patch ? (img * H + py + 8 * h + (r >> 4)) * W + px + (r & 15) : tmh * 128 + r;
    };
    uint4 pre[NCH], pre2[NCH];
#pragma unroll
    for (int k = 0; k < NCH; ++k) {
      const int m = rowm(tid / ncc + k * rpp);
      const long o = (long)m * P.ncol + n0 + cc0;
      pre[k] = (pf != nullptr && m < P.M) ? *(const uint4*)((const T*)pf + o) : make_uint4(0, 0, 0, 0);
      pre2[k] = (pf2 != nullptr && m < P.M) ? *(const uint4*)((const T*)pf2 + o) : make_uint4(0, 0, 0, 0);
    }
    if (h > 0) __syncthreads();                       // the first half's tile has been read
    if ((wr * 32 * MI) / 128 == h) {
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int e = 0; e < 16; ++e)
            accs[((wr * 32 * MI) % 128 + 32 * i + 8 * (e >> 2) + 4 * kh + (e & 3)) * LDA + wc * 64 + 32 * j + r32] =
                acc[i][j][e];
    }
    __syncthreads();
    conv_epilogue<T, MODE, 128, TN, LDA, TN>(P, accs, piv, bn_s, tmh, n0, pre, pre2, rowm);
  }
}

int launch_hgemm(const ConvLaunch& L, int tiles, int mode, int tn, hipStream_t s) {
  if (tn == 64) {
    if (mode == MODE_FWD)
      hipLaunchKernelGGL((hgemm_conv_kernel<MODE_FWD, 64>), dim3(tiles), dim3(256), 0, s, L);
    else
      hipLaunchKernelGGL((hgemm_conv_kernel<MODE_BWD, 64>), dim3(tiles), dim3(256), 0, s, L);
  } else {
    if (mode == MODE_FWD)
      hipLaunchKernelGGL((hgemm_conv_kernel<MODE_FWD, 128>), dim3(tiles), dim3(256), 0, s, L);
    else
      hipLaunchKernelGGL((hgemm_conv_kernel<MODE_BWD, 128>), dim3(tiles), dim3(256), 0, s, L);
  }
  return (int)hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// Short halo GEMM: the same convolution (and its data gradient) where 256-pixel tiles would leave CUs idle.
// 128 pixels x 64 output channels per workgroup, four waves of 32 x 64; maps of at most SG_FLATW columns.
//
// Such a launch is one workgroup per CU and runs at that workgroup's latency: gemm_conv_kernel's 128 x 128 tiles
// (half of the CUs at 8 x 8 pixels x 256 channels, batch 128) wait for their loads and a barrier in each of
// the 9 Cg / 64 steps, and its forward forms the BN prologue once per tap.  Here the filter rows run two steps
// ahead in three buffers, and the next chunk's input rows arrive during the current chunk's taps, one
// 16-byte load per lane and step, so no step waits for a load issued in the one before.  A BN prologue is
// applied in place, once per chunk: a wave activates the rows that it loaded itself two steps earlier.
//
// K runs as in gemm_conv_kernel (chunk outer, tap inner): the convolution's results are bit-identical to its
// unsplit ones.  The BN partial rows formed with them are not: a thread of a 64-column tile adds every 32nd row of it,
// of a 128-column tile every 16th.
// Measured (the paper's coarse blocks, batch 128, 9.7 GFLOP a launch; gemm_conv_kernel before): 256 channels at
// 8 x 8 pixels, 256 workgroups, forward 50.0 -> 28.2 us, data gradient 39.8 -> 23.5; 128 channels at 16 x 16, 512
// workgroups, 32.9 -> 22.2 and 26.4 -> 18.1 us (343 to 534 TFLOP/s).
// ------------------------------------------------------------------------------------------------
template <int MODE>
__global__ __launch_bounds__(256, 2) void sgemm_conv_kernel(const ConvLaunch L) {
  using T = uint16_t;
  constexpr int VE = 8, TN = 64, BM = 128;
  constexpr int A_BYTES = SG_AROWS * HROW;            // one input buffer
  constexpr int B_BYTES = TN * HROW;                  // one filter buffer
  constexpr int ZERO = 2 * A_BYTES;                   // the row of zeros
  constexpr int B0 = ZERO + HROW;
  constexpr int LDA = TN + 4;
  constexpr int SMEM = B0 + 3 * B_BYTES;
  static_assert(BM * LDA * 4 + 8 * TN * 4 <= SMEM, "the epilogue's tile, BN constants and pivot");
  static_assert(2 * (SMEM + CONV_PRO_MAXC * 8) <= 160 * 1024, "two workgroups per CU");
  static_assert(SG_AROWS % 8 == 0 && (SG_AROWS / 8 + 3) / 4 <= 7, "a wave's pieces are activated by tap 8");
  __shared__ __attribute__((aligned(1024))) unsigned char smem[SMEM];
  __shared__ __attribute__((aligned(16))) float2 pro_s[CONV_PRO_MAXC];

  const int gi = find_group(L);
  const ConvProb& P = L.p[gi];
  const int local = blockIdx.x - P.tile_begin;
  // the column tiles of a row tile on one XCD, as in hgemm_conv_kernel
  const int per = P.tiles_m / 8;
  int tm, tn;
  if (local < 8 * per * P.tiles_n) {
    const int q = local >> 3;
    tm = (local & 7) * per + q / P.tiles_n;
    tn = q % P.tiles_n;
  } else {
    const int l2 = local - 8 * per * P.tiles_n;
    tm = 8 * per + l2 / P.tiles_n;
    tn = l2 % P.tiles_n;
  }
  const int n0 = tn * TN, m0 = tm * BM;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int r32 = lane & 31, kh = lane >> 5;
  const int W = P.Q, H = P.P, PQ = H * W;
  const bool prologue = MODE == MODE_FWD && P.pro != nullptr;

  // input loads: piece j of the wave fills rows 8 (wave + 4 j) .. + 7 (pixels clamped to the tensor: a clamped
  // row is no tap's, its output pixel being outside or at the image's edge)
  const int lrow = lane >> 3, lch = (lane & 7) ^ lrow;
  const int R = BM + 2 * W + 2;
  const int nai = (R + 31 - 8 * wave) / 32;
  const uint32_t lds0 = (uint32_t)(size_t)(__attribute__((address_space(3))) unsigned char*)smem;
  const uint32_t boff = (uint32_t)(((long)(n0 + 8 * wave + lrow) * P.K + 8 * lch) * 2);
  const uint32_t bstep = (uint32_t)(32L * P.K * 2);
  const char* in = (const char*)P.in;
  const char* wm = (const char*)P.wmat;
  const int nchunk = P.Cg / 64, total = 9 * nchunk;
  auto load_a = [&](int cb, int j) {
    const long pix = min(max((long)m0 - W - 1 + 8 * (wave + 4 * j) + lrow, 0L), (long)P.M - 1);
    load_lds16(lds0 + (cb & 1) * A_BYTES + (wave + 4 * j) * 1024, in + cb * HROW, (uint32_t)((pix * P.Cg + 8 * lch) * 2));
  };
  auto load_b = [&](int cb, int tap, int buf) {
    const char* base = wm + ((long)tap * P.Cg + cb * 64) * 2;
#pragma unroll
    for (int j = 0; j < TN / 32; ++j)
      load_lds16(lds0 + B0 + buf * B_BYTES + (wave + 4 * j) * 1024, base, boff + j * bstep);
  };
  // piece j of chunk cb, loaded by this lane: ReLU(x scale + shift) of its 8 channels
  auto activate = [&](int cb, int j) {
    uint4* at = (uint4*)(smem + (cb & 1) * A_BYTES + (wave + 4 * j) * 1024 + 16 * lane);
    Chunk<T> v;
    unpack_chunk<T>(*at, v);
    const float2* ps = pro_s + cb * 64 + 8 * lch;
    float f[VE];
#pragma unroll
    for (int e = 0; e < VE; ++e) f[e] = fmaxf(fmaf(v.v[e], ps[e].x, ps[e].y), 0.0f);
    uint4 w;
    store_chunk<T>(&w, 0, f);
    *at = w;
  };

  // the lane's fragment row: LDS row of the output pixel itself and the taps inside the image
  const int lm = wave * 32 + r32, arow = lm + W + 1;
  unsigned amask = 0;
  {
    const int m = m0 + lm;
    const bool v = m < P.M;
    const int mm = v ? m : 0;
    const int rem = mm - div_l2(mm, PQ, P.pq_log2) * PQ;
    const int p = div_l2(rem, W, P.q_log2);
    const int q = rem - p * W;
#pragma unroll
    for (int t = 0; t < 9; ++t) {
      const int dr = MODE == MODE_FWD ? t / 3 - 1 : 1 - t / 3;
      const int dq = MODE == MODE_FWD ? t % 3 - 1 : 1 - t % 3;
      amask |= (v && (unsigned)(p + dr) < (unsigned)H && (unsigned)(q + dq) < (unsigned)W) ? 1u << t : 0u;
    }
  }
  uint32_t bfr[4];
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) bfr[kk] = B0 + r32 * HROW + ((32 * kk + 16 * kh) ^ ((r32 & 7) << 4));

  f32x16 acc[2];
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[j][e] = 0.f;

  if (tid < HROW / 4) *(float*)(smem + ZERO + 4 * tid) = 0.f;
  if (prologue)
    for (int c = tid; c < P.Cg; c += 256) pro_s[c] = make_float2(P.pro[c], P.pro[P.Cg + c]);
  for (int j = 0; j < nai; ++j) load_a(0, j);
  load_b(0, 0, 0);
  load_b(0, 1, 1);
  if (prologue) {
    // all but the second filter tap has landed; the constants are in LDS
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt vmcnt(2) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    for (int j = 0; j < nai; ++j) activate(0, j);
  }
  int buf = 0, s = 0;
  bool piece = false;                                 // an input piece was issued in the step before
  for (int cb = 0; cb < nchunk; ++cb) {
    const bool more = cb + 1 < nchunk;
#pragma unroll 1
    for (int tap = 0; tap < 9; ++tap, ++s) {
      // Issued since this step's filter rows (two steps ago, after that step's input piece): the step before's
      // piece and the next step's filter rows.  All else has landed, in every wave, and every wave is past the
      // step before, whose filter buffer (and, at tap 0, input buffer) is free.
      __builtin_amdgcn_sched_barrier(0);
      if (s + 1 >= total) asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
      else if (piece) asm volatile("s_waitcnt vmcnt(3) lgkmcnt(0)\n\ts_barrier" ::: "memory");
      else asm volatile("s_waitcnt vmcnt(2) lgkmcnt(0)\n\ts_barrier" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
      piece = more && tap < nai;
      if (piece) load_a(cb + 1, tap);
      const int b2 = buf == 0 ? 2 : buf - 1;          // (buf + 2) % 3
      if (tap < 7) load_b(cb, tap + 2, b2);
      else if (more) load_b(cb + 1, tap - 7, b2);
      if (prologue && more && tap >= 2 && tap - 2 < nai) activate(cb + 1, tap - 2);
      const int dr = MODE == MODE_FWD ? tap / 3 - 1 : 1 - tap / 3;
      const int dq = MODE == MODE_FWD ? tap % 3 - 1 : 1 - tap % 3;
      const int rr = arow + dr * W + dq;
      const uint32_t ab = ((amask >> tap) & 1u) ? (cb & 1) * A_BYTES + rr * HROW : ZERO;
      const uint32_t ax = ((rr & 7) << 4) ^ (16 * kh);
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        const bf16x8 a = *(const bf16x8*)(smem + (ab + ((32 * kk) ^ ax)));
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const bf16x8 b = *(const bf16x8*)(smem + buf * B_BYTES + bfr[kk] + 32 * j * HROW);
          acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc[j], 0, 0, 0);
        }
      }
      buf = buf == 2 ? 0 : buf + 1;
    }
  }
  lds_ready();                                        // every wave is past its last fragments

  float* accs = (float*)smem;
  float* bn_s = accs + BM * LDA;
  float* piv = bn_s + 7 * TN;
  const bool bnmask = MODE == MODE_BWD && (P.flags & (EPI_BN_MASK | EPI_BN_APPLY));
  constexpr int ncc = TN / VE, rpp = 256 / ncc, NCH = BM / rpp;
  const int cc0 = (tid % ncc) * VE;
  const void* pf = (MODE == MODE_FWD) ? P.res
                   : ((P.flags & EPI_STORE_F32) ? nullptr : (bnmask ? P.zsrc : P.res));
  const void* pf2 = (MODE == MODE_FWD) ? P.ext : ((P.flags & EPI_BN_APPLY) ? P.res : nullptr);
  if (bnmask && tid < TN) {
    const int col = n0 + tid;
#pragma unroll
    for (int k = 0; k < 4; ++k) bn_s[k * TN + tid] = P.bnst[k * P.ncol + col];
    if (P.flags & EPI_BN_APPLY) {
#pragma unroll
      for (int k = 0; k < 3; ++k) bn_s[(4 + k) * TN + tid] = P.coef[k * P.ncol + col];
    }
  }
  uint4 pre[NCH], pre2[NCH];
#pragma unroll
  for (int k = 0; k < NCH; ++k) {
    const int m = m0 + tid / ncc + k * rpp;
    const long o = (long)m * P.ncol + n0 + cc0;
    pre[k] = (pf != nullptr && m < P.M) ? *(const uint4*)((const T*)pf + o) : make_uint4(0, 0, 0, 0);
    pre2[k] = (pf2 != nullptr && m < P.M) ? *(const uint4*)((const T*)pf2 + o) : make_uint4(0, 0, 0, 0);
  }
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int e = 0; e < 16; ++e)
      accs[(wave * 32 + 8 * (e >> 2) + 4 * kh + (e & 3)) * LDA + 32 * j + r32] = acc[j][e];
  __syncthreads();
  conv_epilogue<T, MODE, BM, TN, LDA, TN>(P, accs, piv, bn_s, tm, n0, pre, pre2);
}

int launch_sgemm(const ConvLaunch& L, int tiles, int mode, hipStream_t s) {
  if (mode == MODE_FWD)
    hipLaunchKernelGGL((sgemm_conv_kernel<MODE_FWD>), dim3(tiles), dim3(256), 0, s, L);
  else
    hipLaunchKernelGGL((sgemm_conv_kernel<MODE_BWD>), dim3(tiles), dim3(256), 0, s, L);
  return (int)hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// Weight gradient of a large wide 3x3 / stride 1 / pad 1 bf16 convolution without a BN prologue:
// dW[co][(r, s, c)] = sum over pixels of g[pixel][co] in[pixel + (r - 1, s - 1)][c], TC output channels x TK
// input channels x the three taps of one filter row per workgroup, split over the pixels.
//
// wgrad_gemm_kernel stages one tap's operands per workgroup through registers (15.6 KB from L2 per MFLOP
// at 128 x 128).  Here the gradient rows and the input rows
// are staged once for three taps (7.8 KB per MFLOP at 128 x 64) by global-to-LDS loads, three stages in flight, and a
// gradient fragment read from LDS serves three MFMA columns.
//
// Pixels run over rows padded by one column, u = row (W + 1) + x with x = W a pad of zeros, so that the input
// pixel of tap s is u + s - 1 with no test at the image's sides: the pads multiply to zero, and one pad
// serves the right side of its row and the left side of the next.  Pads, rows outside the image (r = 0, 2)
// and pixels past the end are loaded from a line of zeros.  A pad's zero gradient meets the input pixels on both
// sides of it, and an infinity there would make a tap NaN that it does not belong to: a workgroup whose sums
// hold a NaN forms them again with those input pixels cleared too (clearing them in every pass would put vector
// instructions between the LDS reads and the MFMAs).
//
// Stages of 64 pixels, pixel-major; fragments by the transposed LDS read, which takes 32 bytes from each of
// four consecutive rows per 16 lanes, two such groups eight rows apart at a time: the 32-byte pieces of a
// row are permuted by the row's index (wg2_swz) so that these eight fall on distinct banks.
//
// Measured (as above; wgrad_gemm_kernel before): 128 x 64 tiles 547 (its 128 x 128 tiles; 240 at 128 x 64) ->
// 888 TFLOP/s, 64 x 64 tiles 279 -> 645, held by LDS reads.
// ------------------------------------------------------------------------------------------------
namespace {

__device__ __attribute__((aligned(256))) const uint4 hg_zeros[16] = {};

typedef short wv4s16 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) wv4s16 lds_wv4s16;

// 64 lanes' 16 bytes each (per-lane addresses) into LDS bytes [lds, lds + 1024) in lane order (wait state: above)
__device__ __forceinline__ void load_lds16(uint32_t lds, const void* addr) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds), "v"(addr)
               : "memory", "m0");
}

// XOR of the 16-byte slot of row r (an even number: pairs stay together)
template <int W>
__device__ __forceinline__ int wg2_swz(int r) {
  return W == 128 ? 2 * ((r & 3) | ((r >> 1) & 4)) : 2 * (((r >> 1) & 1) | ((r >> 2) & 2));
}

constexpr int WG2_PX = 64;                        // pixels per stage
// staging of a W-channel operand: ROWS rows of 2 W bytes, whole 1 KB loads
template <int W, int ROWS>
struct Wg2Op {
  static constexpr int RB = 2 * W;                // bytes per row
  static constexpr int RPL = 1024 / RB;           // rows per load
  static constexpr int NL = (ROWS + RPL - 1) / RPL;   // loads per stage
  static constexpr int NW = (NL + 3) / 4;         // loads per wave, at most
  static constexpr int BYTES = NL * 1024;
};

}  // namespace

template <int TC, int TK>
__global__ __launch_bounds__(256, 2) void wgrad_row_kernel(const WgradLaunch L) {
  using OG = Wg2Op<TC, WG2_PX>;
  using OA = Wg2Op<TK, WG2_PX + 2>;
  constexpr int NI = TC / 32, NJ = TK / 32;       // 16-channel MFMA blocks per wave
  constexpr int STG = OG::BYTES + OA::BYTES;
  constexpr int NST = 3;
  constexpr int AHEAD = OG::NL / 4 + OA::NL / 4;  // loads of one stage that every wave issues
  static_assert(OG::NL % 4 == 0 && OA::NL % 4 == 1, "the first wave loads the input's last rows");
  __shared__ __attribute__((aligned(1024))) unsigned char smem[NST * STG];
  const int gi = find_group(L);
  const WgradProb& P = L.p[gi];
  const int local = blockIdx.x - P.tile_begin;
  // the tiles of a split (same pixels) on one XCD, as in wgrad_gemm_kernel
  const int tcn = P.Co / TC, tkn = P.Cg / TK;
  const int NT = 3 * tcn * tkn;
  const int S8 = P.splits & ~7;
  int t, split;
  if (local < S8 * NT) {
    const int q = local >> 3;
    split = (local & 7) + 8 * (q / NT);
    t = q % NT;
  } else {
    const int l2 = local - S8 * NT;
    split = S8 + l2 / NT;
    t = l2 % NT;
  }
  const int fr = t % 3, tt = t / 3;               // filter row
  const int co0 = tt / tkn * TC, c0 = tt % tkn * TK;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int r16 = lane & 15, grp = lane >> 4;
  const int wr = wave >> 1, wc = wave & 1;
  const int W1 = P.Q + 1, H = P.P;
  const int U = P.B * H * W1;
  const int u0 = split * P.mchunk;
  const int u1 = min(U, u0 + P.mchunk);
  const int nst = (u1 - u0 + WG2_PX - 1) / WG2_PX;

  // the rows this lane loads: (padded) pixel u -> row index and column, advanced by a stage at a time
  struct Row {
    int u, row, x, p;                             // p: row within the image
  };
  auto make_row = [&](int u) {
    Row r;
    r.u = u;
    const int uc = max(u, 0);
    r.row = uc / W1;
    r.x = uc - r.row * W1;
    r.p = r.row % H;
    return r;
  };
  const int sx = WG2_PX % W1, sr = WG2_PX / W1, sp = sr % H;
  auto advance = [&](Row& r) {
    const bool neg = r.u < 0;                     // (u = -1: the next is 63, from pixel 0's place less one)
    int x = r.x + sx - (neg ? 1 : 0), row = r.row + sr, p = r.p + sp;
    if (x < 0) { x += W1; --row; --p; if (p < 0) p += H; }
    if (x >= W1) { x -= W1; ++row; ++p; }
    if (p >= H) p -= H;
    r.u += WG2_PX;
    r.x = x;
    r.row = row;
    r.p = p;
  };
  Row rg[OG::NW], ra[OA::NW];
  uint32_t cg_[OG::NW], ca_[OA::NW];              // byte offset of the lane's chunk within the tile's channels
  auto first_rows = [&]() {
#pragma unroll
    for (int j = 0; j < OG::NW; ++j) {
      const int r = OG::RPL * (wave + 4 * j) + lane / (64 / OG::RPL);
      rg[j] = make_row(u0 + r);
      cg_[j] = 16 * ((lane % (64 / OG::RPL)) ^ wg2_swz<TC>(r)) + 2 * co0;
    }
#pragma unroll
    for (int j = 0; j < OA::NW; ++j) {
      const int r = OA::RPL * (wave + 4 * j) + lane / (64 / OA::RPL);
      ra[j] = make_row(u0 - 1 + r);
      ca_[j] = 16 * ((lane % (64 / OA::RPL)) ^ wg2_swz<TK>(r)) + 2 * c0;
    }
  };
  const uint32_t lds0 = (uint32_t)(size_t)(__attribute__((address_space(3))) unsigned char*)smem;
  const char* const gbase = (const char*)P.g;
  const char* const abase = (const char*)P.in;
  const char* const zero = (const char*)hg_zeros;
  const int Wd = P.Q;
  auto issue = [&](int st) {
    const uint32_t b = lds0 + st * STG;
#pragma unroll
    for (int j = 0; j < OG::NW; ++j) {
      const Row& r = rg[j];
      const bool ok = r.u < u1 && r.x < Wd;
      const char* a = ok ? gbase + ((long)(r.row * Wd + r.x) * P.Co * 2 + cg_[j]) : zero;
      load_lds16(b + (wave + 4 * j) * 1024, a);
      advance(rg[j]);
    }
#pragma unroll
    for (int j = 0; j < OA::NW; ++j) {
      if (j < OA::NL / 4 || wave == 0) {
        const Row& r = ra[j];
        const int ih = r.p + fr - 1;
        const bool ok = r.u >= 0 && r.u < U && r.x < Wd && (unsigned)ih < (unsigned)H;
        const char* a = ok ? abase + ((long)((r.row + fr - 1) * Wd + r.x) * P.Cg * 2 + ca_[j]) : zero;
        load_lds16(b + OG::BYTES + (wave + 4 * j) * 1024, a);
      }
      advance(ra[j]);
    }
  };

  // the lane's byte offsets for the transposed reads: lane group grp takes pixels 8 grp + (r16 / 4) (and + 4),
  // channels 4 (r16 % 4) of a 16-channel block; block i of the wave at offset ^ (32 i)
  const int bch = (r16 & 3) >> 1, bby = 8 * (r16 & 1);
  const int row_g = 8 * grp + (r16 >> 2);
  const uint32_t off_g = row_g * OG::RB + 16 * (((wr * (TC / 2)) / 8 + bch) ^ wg2_swz<TC>(row_g)) + bby;
  uint32_t off_a[3][2];
#pragma unroll
  for (int s = 0; s < 3; ++s)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int r = row_g + s + 4 * h;
      off_a[s][h] = OG::BYTES + r * OA::RB + 16 * (((wc * (TK / 2)) / 8 + bch) ^ wg2_swz<TK>(r)) + bby;
    }
  auto frag = [&](uint32_t lo, uint32_t hi) {
    const wv4s16 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_wv4s16*)(uintptr_t)lo);
    const wv4s16 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_wv4s16*)(uintptr_t)hi);
    const uint2 l2 = __builtin_bit_cast(uint2, a), h2 = __builtin_bit_cast(uint2, b);
    return make_uint4(l2.x, l2.y, h2.x, h2.y);
  };

  f32x4 acc[3][NI][NJ];
  // the workgroup's sums (CLEAR: the side taps' input pixels that a pad meets are cleared)
  auto sums = [&](auto clear) {
    constexpr bool CLEAR = decltype(clear)::value;
#pragma unroll
    for (int s = 0; s < 3; ++s)
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[s][i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    first_rows();
    issue(0);
    issue(1);
    int st = 0;
#pragma unroll 1
    for (int n = 0; n < nst; ++n) {
      // this stage has landed (the next one's loads may be in flight) and every wave is past the stage before
      // it, whose buffer the stage after the next takes
      __builtin_amdgcn_sched_barrier(0);
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(AHEAD) : "memory");
      __builtin_amdgcn_sched_barrier(0);
      issue(st == 0 ? 2 : st - 1);                // (past the end: zeros, or input rows that no gradient row meets)
      const uint32_t b = lds0 + st * STG;
#pragma unroll
      for (int sub = 0; sub < WG2_PX / 32; ++sub) {
        Frag<uint16_t> a[NI], f[3][NJ];
#pragma unroll
        for (int i = 0; i < NI; ++i) {
          const uint32_t o = b + (off_g ^ (32 * i)) + sub * 32 * OG::RB;
          a[i].from_raw(frag(o, o + 4 * OG::RB));
        }
        uint32_t keep[4] = {~0u, ~0u, ~0u, ~0u};  // the lane's eight pixels, two to a word
        if constexpr (CLEAR) {
#pragma unroll
          for (int e = 0; e < 8; ++e)
            if ((u0 + n * WG2_PX + sub * 32 + 8 * grp + e) % W1 == Wd) keep[e / 2] &= e % 2 ? 0xffffu : 0xffff0000u;
        }
#pragma unroll
        for (int s = 0; s < 3; ++s)
#pragma unroll
          for (int j = 0; j < NJ; ++j) {
            uint4 v = frag(b + (off_a[s][0] ^ (32 * j)) + sub * 32 * OA::RB,
                           b + (off_a[s][1] ^ (32 * j)) + sub * 32 * OA::RB);
            if (CLEAR && s != 1) v = make_uint4(v.x & keep[0], v.y & keep[1], v.z & keep[2], v.w & keep[3]);
            f[s][j].from_raw(v);
          }
#pragma unroll
        for (int s = 0; s < 3; ++s)
#pragma unroll
          for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j) mma(a[i], f[s][j], acc[s][i][j]);
      }
      st = st == NST - 1 ? 0 : st + 1;
    }
    // loads past the end are still in flight: they must land before the workgroup's LDS is used again or given back
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  };
  sums(std::false_type{});
  bool nan = false;
#pragma unroll
  for (int s = 0; s < 3; ++s)
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) nan = nan || acc[s][i][j][e] != acc[s][i][j][e];
  int* flags = (int*)smem;
  const int any = __any(nan);
  __syncthreads();                                // every wave is past its last fragments, and its loads have landed
  if (lane == 0) flags[wave] = any;
  __syncthreads();
  const bool again = (flags[0] | flags[1] | flags[2] | flags[3]) != 0;
  if (again) {
    __syncthreads();                              // (the flags have been read)
    sums(std::true_type{});
  }

  // the partial tile: lane (r16, grp) holds rows 4 grp + e of each 16 x 16 block
#pragma unroll
  for (int s = 0; s < 3; ++s)
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int co = co0 + wr * (TC / 2) + 16 * i + 4 * grp + e;
          const int k = (3 * fr + s) * P.Cg + c0 + wc * (TK / 2) + 16 * j + r16;
          P.part[((long)split * P.Co + co) * P.K + k] = acc[s][i][j][e];
        }
}

int launch_wgrad_row(const WgradLaunch& L, int tiles, int tc, int tk, hipStream_t s) {
  if (tc == 128 && tk == 64)
    hipLaunchKernelGGL((wgrad_row_kernel<128, 64>), dim3(tiles), dim3(256), 0, s, L);
  else if (tc == 64 && tk == 128)
    hipLaunchKernelGGL((wgrad_row_kernel<64, 128>), dim3(tiles), dim3(256), 0, s, L);
  else if (tc == 64 && tk == 64)
    hipLaunchKernelGGL((wgrad_row_kernel<64, 64>), dim3(tiles), dim3(256), 0, s, L);
  else
    return (int)hipErrorInvalidValue;
  return (int)hipGetLastError();
}

}  // namespace pnn
