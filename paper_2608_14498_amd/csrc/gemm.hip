// GEMMs of the backbone: C[M,N] (epi)= A[M,K] . B[N,K]^T with fp32 accumulation.
// A is row-major activations, B is nn.Linear weights [out, in] given as up to three row
// segments (q/k/v or gate/up projections without a concatenated copy).
//
// 16-bit (v_mfma_f32_32x32x16_bf16 / _f16): a 256x256 C tile per workgroup of 8 waves (4x2, each
// 64x128, two waves per SIMD), K in 64-deep slabs, fp32 accumulators in registers.
//   * A/B slabs are staged through LDS, double buffered (2 x 64 KiB), each row of 8
//     16-byte chunks XOR-swizzled so that any 8 (32-bank) or 16 (64-bank) consecutive
//     rows read by one MFMA operand fetch hit distinct banks: no LDS bank conflicts.
//   * Main kernel: the load unit copies the next slab straight into the idle LDS buffer
//     (buffer_load ... lds), issued at the top of the current slab and interleaved with
//     its MFMAs; the tile barrier sits before the last k-step so the next slab's first
//     fragments are read under that step's MFMAs.  A register-staged variant (global ->
//     VGPR -> LDS) serves operands that do not fit one 2 GiB buffer window.
//   * The MFMAs take the B fragment as first operand, so each lane ends with 4
//     consecutive columns of one output row: 8-byte bf16 / 16-byte fp32 stores.
//   * Tiles are visited in groups of 8 tile-rows and the block index is remapped so each
//     XCD walks a contiguous range of tiles (its L2 holds the shared A/B slabs).
//   * Epilogues: bf16 store, fp32 store, fp32 accumulate (residual), fused SwiGLU (each
//     wave's 128 B rows are 64 gate + the matching 64 up rows, so gate and up of one
//     output feature land in the same lane), and fp32 split-K partials.
//
// fp32: 32x32 tiles of v_mfma_f32_32x32x2 (exact fp32 products) for the fp32 model.
#include "gemm_common.h"

#include <stdlib.h>

namespace rp {

constexpr int GB_M = 256, GB_N = 256;

// Transposed B (BSeg::trans): the slab is staged as stored, [64 k][256 n] with 32
// 16-byte chunks per k row, and physical chunk = logical chunk ^ swzt(k).  One
// transposed fragment read covers 4 consecutive k rows x 4 consecutive chunks per half
// wave; the XOR gives those 16 (row, chunk) pairs distinct bank groups with 32 or with
// 64 banks (bits 1-2 and bits 2-3 of the chunk index both differ across the 4 rows).
__device__ __forceinline__ int swzt(int k) { return (k & 3) * 5; }

// Per-lane element offsets (within a transposed slab) of the B fragments j = 0..NJ-1 at
// k-step 0; k-step ks adds ks*16 rows and the second read 4 rows (same swizzle: k % 4 is
// unchanged).  Lane l = 16g + p addresses k row 8(g/2) + p/4 at column
// n0 + 16(g%2) + 4(p%4), so that ds_read_b64_tr_b16 hands it k = 8(l/32) + 0..3 (then
// + 4..7 from the second read) of column n0 + l%32: the MFMA operand layout, the same k
// order as the A fragment.
template <int NJ>
__device__ __forceinline__ void bt_offsets(int lane, int n_wave, int (&off)[NJ]) {
  const int g = lane >> 4, p = lane & 15;
  const int kr = 8 * (g >> 1) + (p >> 2);
  const int nb = n_wave + 16 * (g & 1) + 4 * (p & 3);
#pragma unroll
  for (int j = 0; j < NJ; ++j) off[j] = kr * GB_N + ((((nb >> 3) + 4 * j) ^ swzt(kr)) << 3) + (nb & 7);
}

// B fragment from a transposed LDS slab at element offset off (see bt_offsets).
template <typename T16>
__device__ __forceinline__ typename Half16<T16>::V8 bt_frag(const void* slab, int off) {
  const T16* p = reinterpret_cast<const T16*>(slab) + off;
  const v4i16_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_t*)p);
  const v4i16_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_t*)(p + 4 * GB_N));
  const uint2 l = __builtin_bit_cast(uint2, lo), h = __builtin_bit_cast(uint2, hi);
  return Half16<T16>::as_v8(make_uint4(l.x, l.y, h.x, h.y));
}

// Epilogue of the bf16 kernels.  The MFMAs take the B fragment as their first operand,
// so a lane holds rows of C^T: acc[i][j][e] = C(row i*32 + fr, col j*32 + 8(e/4) + 4 fk
// + e%4) of the wave tile, i.e. four consecutive columns of one row per e/4.
template <int EPI, typename T16, int MI, int NJ, int TM, int TN>
__device__ __forceinline__ void gemm_epilogue(const GemmArgs& g, f32x16_t (&acc)[MI][NJ], int tm, int tn, int wm,
                                              int wn, int fr, int fk) {
  const int mb = tm * GB_M + wm * TM + fr;
  if (EPI == EPI_SWIGLU) {  // gate in acc[i][j], up in acc[i][j + 2]
    const bool vec = (g.ldc & 3) == 0 && ((uintptr_t)g.C & 7) == 0;
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      const int m = mb + i * 32;
      if (m >= g.M) continue;
      T16* row = (T16*)g.C + (int64_t)m * g.ldc;
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          float v[4];
#pragma unroll
          for (int t = 0; t < 4; ++t) v[t] = silu_mul(acc[i][j][4 * q + t], acc[i][j + 2][4 * q + t]);
          store4h(row, tn * 128 + wn * 64 + j * 32 + 8 * q + 4 * fk, g.N, v, vec);
        }
    }
    return;
  }
  bool vec;
  if (EPI == -1)
    vec = (g.N & 3) == 0 && ((uintptr_t)g.partials & 15) == 0;
  else if (EPI == EPI_STORE)
    vec = (g.ldc & 3) == 0 && ((uintptr_t)g.C & 7) == 0;
  else
    vec = (g.ldc & 3) == 0 && ((uintptr_t)g.C & 15) == 0;
  const int nb = tn * GB_N + wn * TN + 4 * fk;
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    const int m = mb + i * 32;
    if (m >= g.M) continue;
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int n0 = nb + j * 32 + 8 * q;
        const float v[4] = {acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
        if (EPI == -1)
          store4<false>(g.partials + ((int64_t)blockIdx.y * g.M + m) * g.N, n0, g.N, v, vec);
        else if (EPI == EPI_STORE)
          store4h((T16*)g.C + (int64_t)m * g.ldc, n0, g.N, v, vec);
        else if (EPI == EPI_STORE_F32)
          store4<false>((float*)g.C + (int64_t)m * g.ldc, n0, g.N, v, vec);
        else
          store4<true>((float*)g.C + (int64_t)m * g.ldc, n0, g.N, v, vec);
      }
  }
}

// Online log-sum-exp epilogue of the lm_head (EPI_LSE): each wave reduces every row of
// its 64 x 128 block over the block's in-range columns to (max, sum 2^(x log2e - max))
// in log2 units, the two lanes of a row (column halves fk = 0, 1) merged by a shuffle;
// the lane holding column ids[m] writes the target logit.  Column block p = tn*2 + wn.
template <int MI, int NJ, int TM, int TN>
__device__ __forceinline__ void gemm_epilogue_lse(const GemmArgs& g, f32x16_t (&acc)[MI][NJ], int tm, int tn, int wm,
                                                  int wn, int fr, int fk) {
  static_assert(TN == 128, "two 128-column blocks per 256-column tile");
  constexpr float kL2e = 1.4426950408889634f;
  const int c0 = tn * GB_N + wn * TN + 4 * fk;
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    const int m = tm * GB_M + wm * TM + i * 32 + fr;
    const int mc = min(m, g.M - 1);
    const int id = min(max(g.lse.ids[mc], 0), g.n_all - 1) - g.n_off;
    float mx = -INFINITY;
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e)
        if (c0 + j * 32 + 8 * (e >> 2) + (e & 3) < g.N) mx = fmaxf(mx, acc[i][j][e]);
    mx = fmaxf(mx, __shfl_xor(mx, 32, kWave));
    const float ms = mx * kL2e;
    float sum = 0.f;
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int col = c0 + j * 32 + 8 * (e >> 2) + (e & 3);
        if (col < g.N) sum += exp2f(fmaf(acc[i][j][e], kL2e, -ms));
        if (col == id && m < g.M) g.lse.tgt[m] = acc[i][j][e];
      }
    sum += __shfl_xor(sum, 32, kWave);
    if (fk == 0 && m < g.M)
      *reinterpret_cast<float2*>(g.lse.lse + ((int64_t)m * g.n_part + g.n_off / 128 + tn * 2 + wn) * 2) =
          make_float2(ms, sum);
  }
}

int32_t lse_parts(int32_t N) { return ((N + GB_N - 1) / GB_N) * 2; }

// Epilogue through LDS for the 8-wave kernels (wave tile 64 x 128).  After the main
// loop the LDS is free: each wave stages its sub-tile in a private 16 KiB region and
// writes it back as whole row segments (256 B of bf16 or 512 B of fp32 per row), one
// 16-byte access per lane, instead of 4 columns x 32 rows per store instruction.
// Staging layout: row-major, 8-byte (bf16) or 16-byte (fp32) chunks XOR-swizzled with
// the row so that the 32 rows written by one instruction fall in distinct banks.
template <int EPI, typename T16, int MI, int NJ, int TM, int TN>
__device__ __forceinline__ void gemm_epilogue_lds(const GemmArgs& g, f32x16_t (&acc)[MI][NJ], uint8_t* stage,
                                                  int tm, int tn, int wm, int wn, int lane) {
  static_assert((MI == 2 || MI == 4) && NJ == 4 && TM == 32 * MI && TN == 128, "wave tile 64x128 or 128x128");
  const int fr = lane & 31, fk = lane >> 5;
  const int mw = tm * GB_M + wm * TM;  // first row of the wave tile
  if (EPI == EPI_SWIGLU || EPI == EPI_STORE) {
    // bf16 output: SwiGLU gives 64 features per row (rows of 128 B), plain 128 (256 B)
    constexpr int W8 = EPI == EPI_SWIGLU ? 16 : 32;  // 8-byte chunks per staged row
    constexpr int XM = W8 - 1;
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      const int r = i * 32 + fr;
#pragma unroll
      for (int j = 0; j < (EPI == EPI_SWIGLU ? 2 : NJ); ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          float v[4];
#pragma unroll
          for (int t = 0; t < 4; ++t)
            v[t] = EPI == EPI_SWIGLU ? silu_mul(acc[i][j][4 * q + t], acc[i][j + 2][4 * q + t]) : acc[i][j][4 * q + t];
          const int c8 = j * 8 + 2 * q + fk;
          *reinterpret_cast<uint2*>(stage + r * (W8 * 8) + ((c8 ^ (r & XM)) << 3)) =
              make_uint2(Half16<T16>::pack2(v[0], v[1]), Half16<T16>::pack2(v[2], v[3]));
        }
    }
    constexpr int LPR = W8 / 2;  // lanes per row (16 bytes each)
    constexpr int RPI = 64 / LPR;  // rows per instruction
    const int ncol0 = EPI == EPI_SWIGLU ? tn * 128 + wn * 64 : tn * GB_N + wn * TN;
    const bool vec = (g.ldc & 7) == 0 && ((uintptr_t)g.C & 15) == 0;
    const int k = lane % LPR;
#pragma unroll
    for (int s = 0; s < TM / RPI; ++s) {
      const int r = s * RPI + lane / LPR;
      uint4 v = *reinterpret_cast<const uint4*>(stage + r * (W8 * 8) + ((k ^ ((r & XM) >> 1)) << 4));
      if (r & 1) {  // the two 8-byte halves were stored swapped
        const uint32_t x = v.x, y = v.y;
        v.x = v.z;
        v.y = v.w;
        v.z = x;
        v.w = y;
      }
      const int m = mw + r, n = ncol0 + k * 8;
      if (m >= g.M) continue;
      T16* dst = (T16*)g.C + (int64_t)m * g.ldc + n;
      if (vec && n + 7 < g.N) {
        st_out16<true>((void*)dst, v);
      } else {
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (n + e < g.N) reinterpret_cast<uint16_t*>(dst)[e] = (uint16_t)(w[e >> 1] >> (16 * (e & 1)));
      }
    }
    return;
  }
  // fp32 outputs (store, residual accumulate, split-K partials): two passes of 32 rows,
  // staged rows of 128 floats (32 chunks of 16 bytes)
  const F32Out out = f32_out<EPI>(g);
  const int ncol0 = tn * GB_N + wn * TN;
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    if (i > 0) __builtin_amdgcn_s_waitcnt(0xc07f);  // previous pass's LDS reads are done (lgkmcnt(0))
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int c16 = j * 8 + 2 * q + fk;
        *reinterpret_cast<float4*>(stage + fr * 512 + ((c16 ^ (fr & 15)) << 4)) =
            make_float4(acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
      }
    store_rows<EPI, T16, 2>(g, out, stage, mw + i * 32, ncol0, lane, 0);
  }
}

// ------------------------------------------------------------------------------------
// bf16 MFMA GEMM
// ------------------------------------------------------------------------------------
template <int EPI, typename T16, int WGM, bool BT = false>
__global__ __launch_bounds__(WGM * 2 * 64) void k_gemm_bf16(GemmArgs g) {
  typedef typename Half16<T16>::V8 V8;
  constexpr int NT = WGM * 2 * 64;
  constexpr int TM = GB_M / WGM, TN = GB_N / 2;
  constexpr int MI = TM / 32, NJ = TN / 32;
  constexpr int LOADS = (GB_M * 8) / NT;  // 16-byte chunks per matrix per thread: 8 or 4
  constexpr int MM = MI * NJ;              // MFMAs per k-step
  __shared__ uint4 As[2][GB_M * 8];
  __shared__ uint4 Bs[2][GB_N * 8];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  int tm, tn;
  tile_coords(xcd_remap(blockIdx.x, gridDim.x), g.tiles_m, g.tiles_n, &tm, &tn);
  const int m0 = tm * GB_M;
  const int kbeg = blockIdx.y * g.k_chunk;
  const int kend = min(g.K, kbeg + g.k_chunk);
  const int KT = (kend - kbeg) / GB_K;

  const int lc = tid & 7, lr = tid >> 3;
  const T16* Ab = (const T16*)g.A + kbeg + lc * 8;
  // logical B row staged in local B row r of this tile
  auto b_logical = [&](int r) -> int {
    if (EPI == EPI_SWIGLU) {  // per 128-row half: 64 gate rows then the matching 64 up rows
      const int w = r >> 7, c = r & 127;
      const int f = min(tn * 128 + w * 64 + (c & 63), g.N - 1) + g.n_off;
      return (c >= 64 ? g.B.n1 : 0) + f;
    }
    return min(tn * GB_N + r, g.N - 1) + g.n_off;
  };
  uint4 ra0, ra1, ra2, ra3, ra4, ra5, ra6, ra7, rb0, rb1, rb2, rb3, rb4, rb5, rb6, rb7;
#define G_LDA(i_, kt_)                                                                                    \
  if (i_ < LOADS) {                                                                                       \
    const int r_ = lr + (NT / 8) * i_;                                                                    \
    ra##i_ = *reinterpret_cast<const uint4*>(Ab + (int64_t)min(m0 + r_, g.M - 1) * g.lda + (kt_) * GB_K); \
  }
#define G_LDB(i_, kt_)                                                                                 \
  if (i_ < LOADS) {                                                                                    \
    if (BT) {                                                                                          \
      const int kr_ = (tid >> 5) + (NT / 32) * i_;                                                     \
      rb##i_ = *reinterpret_cast<const uint4*>((const T16*)g.B.b0 +                                    \
                                               (int64_t)(kbeg + (kt_) * GB_K + kr_) * g.ldb +          \
                                               min(tn * GB_N + (tid & 31) * 8, g.N - 8) + g.n_off);   \
    } else {                                                                                           \
      const int r_ = lr + (NT / 8) * i_;                                                               \
      rb##i_ = *reinterpret_cast<const uint4*>(brow<T16>(g.B, b_logical(r_), g.ldb) + kbeg + lc * 8 + \
                                               (kt_) * GB_K);                                          \
    }                                                                                                  \
  }
#define G_STA(i_, buf_)                                    \
  if (i_ < LOADS) {                                        \
    const int r_ = lr + (NT / 8) * i_;                     \
    As[(buf_)][r_ * 8 + (lc ^ swz(r_))] = ra##i_;          \
  }
#define G_STB(i_, buf_)                                             \
  if (i_ < LOADS) {                                                 \
    if (BT) {                                                       \
      const int kr_ = (tid >> 5) + (NT / 32) * i_;                  \
      Bs[(buf_)][kr_ * 32 + ((tid & 31) ^ swzt(kr_))] = rb##i_;     \
    } else {                                                        \
      const int r_ = lr + (NT / 8) * i_;                            \
      Bs[(buf_)][r_ * 8 + (lc ^ swz(r_))] = rb##i_;                 \
    }                                                               \
  }
#define G_LOAD_A(kt_) G_LDA(0, kt_) G_LDA(1, kt_) G_LDA(2, kt_) G_LDA(3, kt_) G_LDA(4, kt_) G_LDA(5, kt_) G_LDA(6, kt_) G_LDA(7, kt_)
#define G_LOAD_B(kt_) G_LDB(0, kt_) G_LDB(1, kt_) G_LDB(2, kt_) G_LDB(3, kt_) G_LDB(4, kt_) G_LDB(5, kt_) G_LDB(6, kt_) G_LDB(7, kt_)
#define G_STORE_A(b_) G_STA(0, b_) G_STA(1, b_) G_STA(2, b_) G_STA(3, b_) G_STA(4, b_) G_STA(5, b_) G_STA(6, b_) G_STA(7, b_)
#define G_STORE_B(b_) G_STB(0, b_) G_STB(1, b_) G_STB(2, b_) G_STB(3, b_) G_STB(4, b_) G_STB(5, b_) G_STB(6, b_) G_STB(7, b_)
#define G_FRAGS(AF, BF, ks_)                                                   \
  _Pragma("unroll") for (int i = 0; i < MI; ++i) {                             \
    const int r_ = wm * TM + i * 32 + fr;                                      \
    AF[i] = Half16<T16>::as_v8(As[buf][r_ * 8 + (((ks_) * 2 + fk) ^ swz(r_))]); \
  }                                                                            \
  _Pragma("unroll") for (int j = 0; j < NJ; ++j) {                             \
    if (BT) {                                                                  \
      BF[j] = bt_frag<T16>(&Bs[buf][0], btoff[j] + (ks_) * 16 * GB_N);         \
    } else {                                                                   \
      const int r_ = wn * TN + j * 32 + fr;                                    \
      BF[j] = Half16<T16>::as_v8(Bs[buf][r_ * 8 + (((ks_) * 2 + fk) ^ swz(r_))]); \
    }                                                                          \
  }
#define G_MMA(AF, BF)                                                           \
  _Pragma("unroll") for (int i = 0; i < MI; ++i)                                \
  _Pragma("unroll") for (int j = 0; j < NJ; ++j)                                \
    acc[i][j] = Half16<T16>::mma(BF[j], AF[i], acc[i][j]);
// spread n_other_ instructions of class mask_ evenly over the MM MFMAs of this region
#define G_INTERLEAVE(mask_, n_other_)                                           \
  _Pragma("unroll") for (int q = 0; q < (n_other_); ++q) {                      \
    __builtin_amdgcn_sched_group_barrier(0x008, MM / (n_other_), 0);            \
    __builtin_amdgcn_sched_group_barrier((mask_), 1, 0);                        \
  }

  f32x16_t acc[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  if (KT > 0) {
    G_LOAD_A(0);
    G_LOAD_B(0);
    G_STORE_A(0);
    G_STORE_B(0);
  }
  __syncthreads();

  const int fr = lane & 31, fk = lane >> 5;
  int btoff[NJ];
  if (BT) bt_offsets<NJ>(lane, wn * TN, btoff);
  for (int kt = 0; kt < KT; ++kt) {
    const int buf = kt & 1;
    const int ktn = kt + 1 < KT ? kt + 1 : kt;  // the last tile re-loads itself into the idle buffer
    V8 af0[MI], bf0[NJ], af1[MI], bf1[NJ];
    G_FRAGS(af0, bf0, 0);
    G_FRAGS(af1, bf1, 1);
    __builtin_amdgcn_sched_barrier(0);
    G_MMA(af0, bf0);
    G_LOAD_A(ktn);
    G_INTERLEAVE(0x020, LOADS);
    __builtin_amdgcn_sched_barrier(0);
    G_FRAGS(af0, bf0, 2);
    __builtin_amdgcn_sched_barrier(0);
    G_MMA(af1, bf1);
    G_LOAD_B(ktn);
    G_INTERLEAVE(0x020, LOADS);
    __builtin_amdgcn_sched_barrier(0);
    G_FRAGS(af1, bf1, 3);
    __builtin_amdgcn_sched_barrier(0);
    // buffer buf^1 was last read before the previous barrier, so it can be refilled now
    G_MMA(af0, bf0);
    G_STORE_A(buf ^ 1);
    G_INTERLEAVE(0x200, LOADS);
    __builtin_amdgcn_sched_barrier(0);
    G_MMA(af1, bf1);
    G_STORE_B(buf ^ 1);
    G_INTERLEAVE(0x200, LOADS);
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();
  }
#undef G_LDA
#undef G_LDB
#undef G_STA
#undef G_STB
#undef G_LOAD_A
#undef G_LOAD_B
#undef G_STORE_A
#undef G_STORE_B
#undef G_FRAGS
#undef G_MMA
#undef G_INTERLEAVE

  if (EPI == EPI_ROPE) {  // staged through the (now idle) slab buffers: 16 KiB per wave
    __syncthreads();
    uint8_t* stage = (uint8_t*)(wave < 4 ? &As[0][0] : &Bs[0][0]) + (wave & 3) * 16384;
    gemm_epilogue_lds<EPI, T16, MI, NJ, TM, TN>(g, acc, stage, tm, tn, wm, wn, lane);
  } else if (EPI == EPI_LSE) {
    gemm_epilogue_lse<MI, NJ, TM, TN>(g, acc, tm, tn, wm, wn, fr, fk);
  } else {
    gemm_epilogue<EPI, T16, MI, NJ, TM, TN>(g, acc, tm, tn, wm, wn, fr, fk);
  }
}

// ------------------------------------------------------------------------------------
// bf16 MFMA GEMM fed by direct global->LDS loads (global_load_lds_dwordx4).
// Same tile, wave layout, swizzle and epilogues as k_gemm_bf16, but the coming slabs are
// copied straight into idle LDS buffers by the load unit, with no VGPRs or LDS store
// instructions spent on staging.  One load instruction writes 64 consecutive 16-byte
// LDS chunks (8 rows of one slab); the swizzle is applied by choosing which global
// chunk each lane fetches.  The 8-wave form keeps three B slabs and two A slabs in LDS
// (5 x 32 KiB, all of the CU's 160 KiB): B copies are issued during the second k-step of
// the slab two before theirs, A copies right after the barrier one slab ahead, so each
// slab barrier waits only for the A copies issued one slab earlier (with two stages of
// both, for all of them: the matrix cores were busy 68-69% of the cycles and the prefix
// GEMMs took 4-6% longer; with the B copies issued beside the A copies after the
// barrier, 1-1.5% longer).  Three A stages instead gain as
// much time, but the early A copies cost the gate/up GEMM 23% more L2 misses (its B
// panels are shared by twice as many concurrent tiles as its A panels).  The 4-wave
// form keeps two of each.  The buffers are separate arrays and the k loop is unrolled
// over their rotation (6 slabs, or 2), so every LDS access names its buffer at compile
// time.
// ------------------------------------------------------------------------------------
template <int EPI, typename T16, int WGM, bool BT = false>
__global__ __launch_bounds__(WGM * 128) __attribute__((amdgpu_waves_per_eu(WGM == 2 ? 1 : 2, WGM == 2 ? 1 : 2)))
void k_gemm_bf16_dma(GemmArgs g) {
#if defined(__HIP_DEVICE_COMPILE__)  // buffer resources exist only in the device pass
  constexpr int NT = WGM * 2 * 64;
  constexpr int TM = GB_M / WGM, TN = GB_N / 2;
  constexpr int MI = TM / 32, NJ = TN / 32;
  constexpr int LOADS = (GB_M * 8) / NT;  // load instructions per matrix per wave: 4 (8 waves) or 8
  constexpr int MM = MI * NJ;
  constexpr int NREAD = MI + (BT ? 2 : 1) * NJ;  // LDS fragment reads per k-step
  typedef __attribute__((address_space(3))) void lds_void;
  typedef typename Half16<T16>::V8 V8;
  // native vector element type: each fragment read is one 16-byte LDS load in the IR
  typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
  __shared__ u32x4_t As0[GB_M * 8], As1[GB_M * 8];
  __shared__ u32x4_t Bs0[GB_N * 8], Bs1[GB_N * 8], Bs2[GB_N * 8];

  // 128x128 wave tiles hold 256 accumulator registers, which must live in the AGPR file.
  // An empty asm statement that names an AGPR keeps the compiler from assuming that the
  // kernel uses none (it would then put MFMA results in VGPRs and spill).
  if (WGM == 2) asm volatile("" ::: "a0");
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  int tm, tn;
  tile_coords(xcd_remap(blockIdx.x, gridDim.x), g.tiles_m, g.tiles_n, &tm, &tn);
  const int m0 = tm * GB_M;
  const int kbeg = blockIdx.y * g.k_chunk;
  const int kend = min(g.K, kbeg + g.k_chunk);
  const int KT = (kend - kbeg) / GB_K;

  // Load instruction i of this wave fills LDS rows wave*8*LOADS + 8i .. +8; lane l writes
  // physical chunk l%8 of row +l/8, which holds logical chunk (l%8) ^ swz(row).  Sources
  // are byte offsets into the buffer resource of A or of the B segment that holds the
  // instruction's 8 rows (the host checked that every block lies in one segment of less
  // than 4 GiB); the slab offset is uniform.
  const __amdgpu_buffer_rsrc_t rsA = __builtin_amdgcn_make_buffer_rsrc((void*)g.A, 0, -1, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsB0 = __builtin_amdgcn_make_buffer_rsrc((void*)g.B.b0, 0, -1, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsB1 = __builtin_amdgcn_make_buffer_rsrc((void*)g.B.b1, 0, -1, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsB2 = __builtin_amdgcn_make_buffer_rsrc((void*)g.B.b2, 0, -1, 0x00020000);
  auto b_logical = [&](int r) -> int {
    if (EPI == EPI_SWIGLU) {  // per 128-row half: 64 gate rows then the matching 64 up rows
      const int w = r >> 7, cc = r & 127;
      return (cc >= 64 ? g.B.n1 : 0) + min(tn * 128 + w * 64 + (cc & 63), g.N - 1) + g.n_off;
    }
    return min(tn * GB_N + r, g.N - 1) + g.n_off;
  };
  uint32_t aoff[LOADS], boff[LOADS];
  __amdgpu_buffer_rsrc_t rsB[LOADS];
#pragma unroll
  for (int i = 0; i < LOADS; ++i) {
    const int r0 = wave * 8 * LOADS + 8 * i;  // first row of the block (wave-uniform)
    const int r = r0 + (lane >> 3);
    const int c = (lane & 7) ^ swz(r);
    aoff[i] = 2u * ((uint32_t)min(m0 + r, g.M - 1) * (uint32_t)g.lda + (uint32_t)(kbeg + c * 8));
    if (BT) {
      // the same 64 LDS chunks hold k rows 2(wave*LOADS + i) and +1 of the transposed slab;
      // columns past N (N % 8 == 0) re-read the last chunk, and their results are dropped
      const int kr = 2 * (wave * LOADS + i) + (lane >> 5);
      const int cb = (lane & 31) ^ swzt(kr);
      rsB[i] = rsB0;
      boff[i] = 2u * ((uint32_t)(kbeg + kr) * (uint32_t)g.ldb + (uint32_t)(min(tn * GB_N + cb * 8, g.N - 8) + g.n_off));
    } else {
      const int br0 = b_logical(r0);
      const int seg = br0 < g.B.n1 ? 0 : br0 < g.B.n2 ? 1 : 2;
      rsB[i] = seg == 0 ? rsB0 : seg == 1 ? rsB1 : rsB2;
      const int sbeg = seg == 0 ? 0 : seg == 1 ? g.B.n1 : g.B.n2;
      boff[i] = 2u * ((uint32_t)(b_logical(r) - sbeg) * (uint32_t)g.ldb + (uint32_t)(kbeg + c * 8));
    }
  }
  // byte step of B per slab: 64 elements along a row, or 64 rows of the transposed layout
  const uint32_t bstep = BT ? (uint32_t)GB_K * 2u * (uint32_t)g.ldb : (uint32_t)GB_K * 2u;
#define D_LOAD(DA, DB, kt_)                                                                            \
  _Pragma("unroll") for (int i = 0; i < LOADS; ++i) {                                                 \
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsA, (lds_void*)(DA + (wave * LOADS + i) * 64), 16, aoff[i], \
                                             (kt_) * (GB_K * 2), 0, 0);                                \
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsB[i], (lds_void*)(DB + (wave * LOADS + i) * 64), 16, boff[i], \
                                             (int)((uint32_t)(kt_) * bstep), 0, 0);                   \
  }
#define D_LOADA(DA, kt_)                                                                               \
  _Pragma("unroll") for (int i = 0; i < LOADS; ++i)                                                   \
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsA, (lds_void*)(DA + (wave * LOADS + i) * 64), 16, aoff[i], \
                                             (kt_) * (GB_K * 2), 0, 0);
#define D_LOADB(DB, kt_)                                                                               \
  _Pragma("unroll") for (int i = 0; i < LOADS; ++i)                                                   \
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsB[i], (lds_void*)(DB + (wave * LOADS + i) * 64), 16, boff[i], \
                                             (int)((uint32_t)(kt_) * bstep), 0, 0);
#define D_FRAGS(AF, BF, SA, SB, ks_)                                          \
  _Pragma("unroll") for (int i = 0; i < MI; ++i) {                            \
    const int r_ = wm * TM + i * 32 + fr;                                     \
    AF[i] = __builtin_bit_cast(V8, SA[r_ * 8 + (((ks_) * 2 + fk) ^ swz(r_))]); \
  }                                                                           \
  _Pragma("unroll") for (int j = 0; j < NJ; ++j) {                            \
    if (BT) {                                                                 \
      BF[j] = bt_frag<T16>(SB, btoff[j] + (ks_) * 16 * GB_N);                 \
    } else {                                                                  \
      const int r_ = wn * TN + j * 32 + fr;                                   \
      BF[j] = __builtin_bit_cast(V8, SB[r_ * 8 + (((ks_) * 2 + fk) ^ swz(r_))]); \
    }                                                                         \
  }
#define D_MMA(AF, BF)                                                         \
  _Pragma("unroll") for (int i = 0; i < MI; ++i)                              \
  _Pragma("unroll") for (int j = 0; j < NJ; ++j)                              \
    acc[i][j] = Half16<T16>::mma(BF[j], AF[i], acc[i][j]);
  // One 64-deep slab read from (SA, SB); slab kt_+1 is already streaming into (DA, DB).
  // The barrier sits before the last k-step: every wave's copies of slab kt_+1 have
  // landed and every wave has finished reading (SA, SB), so the fragments of k-step 0 of
  // the next slab are read (from DA, DB) under the MFMAs of k-step 3, and the copies of
  // the coming slabs go into (SA, SB) right there.  Issued straight after the barrier,
  // copies have at least a whole slab of MFMA time to land and each CU keeps L2 misses in
  // flight without a gap (the misses' fabric bandwidth, not the MFMAs, bounds the large
  // GEMMs).  D_TILE (4 waves, two stages of A and B) issues slab kt_+2 and waits for
  // every copy.  D_TILE3 (8 waves) issues B of slab kt_+2 into PB (the B buffer slab
  // kt_-1 used, free since the last barrier) under the MFMAs of k-step 1, and A of slab
  // kt_+2 after the barrier; at the barrier only those B copies may still be in flight.
  // Within a k-step each MFMA is followed by one fragment read of the next k-step and
  // then by one copy, so neither the reads nor the copies bunch up in front of the MFMAs
  // (reads grouped ahead of the k-step's MFMAs: the prefix GEMMs took 2% longer).
#define D_REGION(n_mem_, mem_mask_)                                                        \
  _Pragma("unroll") for (int q = 0; q < MM; ++q) {                                         \
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                                     \
    if (q < NREAD) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);                      \
    if (q < (n_mem_)) __builtin_amdgcn_sched_group_barrier((mem_mask_), 1, 0);             \
  }
#define D_TILE(SA, SB, DA, DB, kt_)                                           \
  {                                                                           \
    D_FRAGS(af1, bf1, SA, SB, 1);                                             \
    D_MMA(af0, bf0);                                                          \
    D_REGION(0, 0x000);                                                       \
    __builtin_amdgcn_sched_barrier(0);                                        \
    D_FRAGS(af0, bf0, SA, SB, 2);                                             \
    D_MMA(af1, bf1);                                                          \
    D_REGION(0, 0x000);                                                       \
    __builtin_amdgcn_sched_barrier(0);                                        \
    D_FRAGS(af1, bf1, SA, SB, 3);                                             \
    D_MMA(af0, bf0);                                                          \
    D_REGION(0, 0x000);                                                       \
    __builtin_amdgcn_sched_barrier(0);                                        \
    /* every copy of this wave has landed before any wave passes: the next */ \
    /* slab is read from rows other waves copied (a plain __syncthreads()  */ \
    /* did not always wait for the LDS-DMA copies)                         */ \
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory"); \
    D_FRAGS(af0, bf0, DA, DB, 0);                                             \
    D_MMA(af1, bf1);                                                          \
    D_LOAD(SA, SB, min((kt_) + 2, KT - 1));                                   \
    D_REGION(2 * LOADS, 0x010);                                               \
    __builtin_amdgcn_sched_barrier(0);                                        \
  }
#define D_TILE3(SA, SB, DA, DB, PB, kt_)                                      \
  {                                                                           \
    D_FRAGS(af1, bf1, SA, SB, 1);                                             \
    D_MMA(af0, bf0);                                                          \
    D_REGION(0, 0x000);                                                       \
    __builtin_amdgcn_sched_barrier(0);                                        \
    D_FRAGS(af0, bf0, SA, SB, 2);                                             \
    D_MMA(af1, bf1);                                                          \
    D_LOADB(PB, min((kt_) + 2, KT - 1));                                      \
    D_REGION(LOADS, 0x010);                                                   \
    __builtin_amdgcn_sched_barrier(0);                                        \
    D_FRAGS(af1, bf1, SA, SB, 3);                                             \
    D_MMA(af0, bf0);                                                          \
    D_REGION(0, 0x000);                                                       \
    __builtin_amdgcn_sched_barrier(0);                                        \
    /* this wave's copies of slab kt_+1 (B issued during slab kt_-1, A after */ \
    /* the last barrier) have landed; the B copies of kt_+2 may not have     */ \
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(LOADS) : "memory"); \
    D_FRAGS(af0, bf0, DA, DB, 0);                                             \
    D_MMA(af1, bf1);                                                          \
    D_LOADA(SA, min((kt_) + 2, KT - 1));                                      \
    D_REGION(LOADS, 0x010);                                                   \
    __builtin_amdgcn_sched_barrier(0);                                        \
  }

  f32x16_t acc[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  const int fr = lane & 31, fk = lane >> 5;
  int btoff[NJ];
  if (BT) bt_offsets<NJ>(lane, wn * TN, btoff);
  V8 af0[MI], bf0[NJ], af1[MI], bf1[NJ];
  if (WGM == 2) {
    if (KT > 0) {
      D_LOAD(As0, Bs0, 0);
      asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
      D_FRAGS(af0, bf0, As0, Bs0, 0);
      D_LOAD(As1, Bs1, min(1, KT - 1));  // beyond the last slab: a harmless re-load into an idle buffer
      int kt = 0;
      for (; kt + 2 <= KT; kt += 2) {
        D_TILE(As0, Bs0, As1, Bs1, kt);
        D_TILE(As1, Bs1, As0, Bs0, kt + 1);
      }
      if (kt < KT) D_TILE(As0, Bs0, As1, Bs1, kt);
    }
  } else if (KT > 0) {
    // slab s lives in As[s % 2] and Bs[s % 3]; B of slab 2 goes out during slab 0, A of
    // slab 1 after the first fragment reads; past the last slab the copies re-load it
    // into a buffer no later slab reads
    D_LOADB(Bs0, 0);
    D_LOADA(As0, 0);
    D_LOADB(Bs1, min(1, KT - 1));
    asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
    D_FRAGS(af0, bf0, As0, Bs0, 0);
    D_LOADA(As1, min(1, KT - 1));
    int kt = 0;
    for (; kt + 6 <= KT; kt += 6) {
      D_TILE3(As0, Bs0, As1, Bs1, Bs2, kt);
      D_TILE3(As1, Bs1, As0, Bs2, Bs0, kt + 1);
      D_TILE3(As0, Bs2, As1, Bs0, Bs1, kt + 2);
      D_TILE3(As1, Bs0, As0, Bs1, Bs2, kt + 3);
      D_TILE3(As0, Bs1, As1, Bs2, Bs0, kt + 4);
      D_TILE3(As1, Bs2, As0, Bs0, Bs1, kt + 5);
    }
    if (kt < KT) D_TILE3(As0, Bs0, As1, Bs1, Bs2, kt);
    if (kt + 1 < KT) D_TILE3(As1, Bs1, As0, Bs2, Bs0, kt + 1);
    if (kt + 2 < KT) D_TILE3(As0, Bs2, As1, Bs0, Bs1, kt + 2);
    if (kt + 3 < KT) D_TILE3(As1, Bs0, As0, Bs1, Bs2, kt + 3);
    if (kt + 4 < KT) D_TILE3(As0, Bs1, As1, Bs2, Bs0, kt + 4);
  }
#undef D_LOAD
#undef D_LOADA
#undef D_LOADB
#undef D_FRAGS
#undef D_MMA
#undef D_TILE
#undef D_TILE3
#undef D_REGION
  // no copy into LDS is still in flight past here (the last slabs' re-loads included)
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
  if (EPI == EPI_LSE) {
    gemm_epilogue_lse<MI, NJ, TM, TN>(g, acc, tm, tn, wm, wn, lane & 31, lane >> 5);
    return;
  }
  uint8_t* stage = WGM == 2 ? (uint8_t*)(wave == 0 ? As0 : wave == 1 ? As1 : wave == 2 ? Bs0 : Bs1)
                            : (uint8_t*)(wave < 2 ? As0 : wave < 4 ? As1 : wave < 6 ? Bs0 : Bs1) + (wave & 1) * 16384;
  gemm_epilogue_lds<EPI, T16, MI, NJ, TM, TN>(g, acc, stage, tm, tn, wm, wn, lane);
#endif
}

// ------------------------------------------------------------------------------------
// fp32 MFMA GEMM (v_mfma_f32_32x32x2: exact fp32 products, fp32 accumulation).
// A 32x32 tile per workgroup; its four waves take a quarter of K each and their sums are
// added in LDS, so that also the few hundred rows of a small fp32 model fill the chip.  Wave
// fragments come straight from global memory: lane l holds row l % 32 and the four k of half
// l / 32 of every 8 (the same k for A and B), one 16-byte load for four MFMAs, 32 k (a
// 128-byte line per row) loaded ahead.  Bound by load latency at these sizes: 1024 x 256 x
// 688 takes 12 us (launch and timing events included), where 64x64 tiles of VALU products
// through LDS took 144; 1024 x 1376 x 256 21 us, from 43.
// ------------------------------------------------------------------------------------
constexpr int GF_M = 32, GF_N = 32, GF_K = 16;

template <int EPI, bool BT = false>
__global__ __launch_bounds__(256) void k_gemm_f32(GemmArgs g) {
  __shared__ float4 red[4][GF_M * GF_N / 4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int tm, tn;
  tile_coords(xcd_remap(blockIdx.x, gridDim.x), g.tiles_m, g.tiles_n, &tm, &tn);
  const int kbeg = blockIdx.y * g.k_chunk;
  const int nch = (min(g.K, kbeg + g.k_chunk) - kbeg) / 8;  // chunks of 8 k (K % 8 == 0)
  const int per = (nch + 3) / 4, c0 = min(wave * per, nch), c1 = min(c0 + per, nch);
  const int fr = lane & 31, fk = lane >> 5;
  const int n = min(tn * GF_N + fr, g.N - 1);
  const float* Ap = (const float*)g.A + (int64_t)min(tm * GF_M + fr, g.M - 1) * g.lda + kbeg + 4 * fk;
  const float* Bp = BT ? (const float*)g.B.b0 + (int64_t)(kbeg + 4 * fk) * g.ldb + n
                       : brow<float>(g.B, n, g.ldb) + kbeg + 4 * fk;
  auto load = [&](int c, float4 (&a)[4], float4 (&b)[4]) {  // chunks c .. c+3; zeros past the wave's range
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      a[u] = b[u] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (c + u < c1) {
        const int k = (c + u) * 8;
        a[u] = *reinterpret_cast<const float4*>(Ap + k);
        if (BT) {
          const float* p = Bp + (int64_t)k * g.ldb;
          b[u] = make_float4(p[0], p[g.ldb], p[2 * (int64_t)g.ldb], p[3 * (int64_t)g.ldb]);
        } else {
          b[u] = *reinterpret_cast<const float4*>(Bp + k);
        }
      }
    }
  };
  f32x16_t acc;
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[e] = 0.f;
  auto mma = [&](const float4 (&a)[4], const float4 (&b)[4]) {  // B first: four columns of a row per lane
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(b[u].x, a[u].x, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(b[u].y, a[u].y, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(b[u].z, a[u].z, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(b[u].w, a[u].w, acc, 0, 0, 0);
    }
  };
  float4 a0[4], b0[4], a1[4], b1[4];
  load(c0, a0, b0);
  for (int c = c0; c < c1; c += 8) {
    load(c + 4, a1, b1);
    mma(a0, b0);
    load(c + 8, a0, b0);
    mma(a1, b1);
  }
  // acc[e] = C(row fr, column 8 (e/4) + 4 fk + e%4); 16-byte chunk q of row r at q ^ (r & 7)
#pragma unroll
  for (int q = 0; q < 4; ++q)
    red[wave][fr * 8 + ((2 * q + fk) ^ (fr & 7))] = make_float4(acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]);
  __syncthreads();
  const int r = tid >> 3, q = tid & 7, m = tm * GF_M + r;
  if (m >= g.M) return;
  float v[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const float4 x = red[w][r * 8 + (q ^ (r & 7))];
    v[0] += x.x;
    v[1] += x.y;
    v[2] += x.z;
    v[3] += x.w;
  }
  const F32Out out = f32_out<EPI>(g);
  store4<EPI == EPI_ADD_F32>(out.p + (int64_t)m * out.ld, tn * GF_N + 4 * q, g.N, v, out.vec);
}

// ------------------------------------------------------------------------------------
// split-K reduction + epilogue (fixed summation order: deterministic)
// ------------------------------------------------------------------------------------
template <int EPI, typename T>
__global__ __launch_bounds__(256) void k_splitk_reduce(const float* __restrict__ part, int splitk, int M,
                                                       int N, void* C, int ldc) {
  const int64_t total = (int64_t)M * N;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < total;
       i += (int64_t)gridDim.x * blockDim.x) {
    float v = 0.f;
    for (int z = 0; z < splitk; ++z) v += part[z * total + i];
    const int64_t m = i / N, n = i - m * N;
    if (EPI == EPI_STORE) {
      stf((T*)C + m * ldc + n, v);
    } else if (EPI == EPI_STORE_F32) {
      ((float*)C)[m * ldc + n] = v;
    } else {
      ((float*)C)[m * ldc + n] += v;
    }
  }
}

size_t gemm_partial_floats(int32_t M, int32_t N, int32_t splitk) {
  return splitk > 1 ? (size_t)splitk * M * N : 0;
}

// The LDS-DMA kernel addresses A and each B segment through its own buffer resource with
// 32-bit byte offsets, and picks the B segment per load instruction (8 consecutive tile
// rows).  Usable when A and every used B segment span less than 4 GiB and no 8-row block
// straddles a segment boundary: boundaries at multiples of 8 rows (q/k/v), or the fused
// SwiGLU layout, whose 64-row gate and up runs never mix within a block.  b_rows is the
// number of logical B rows (N, or n1 + N for the fused SwiGLU layout).
static bool dma_setup(const GemmArgs& g, int64_t b_rows, bool swiglu) {
  constexpr uint64_t kLim = 0xFFFFFF00ull;
  if (g.M <= 0 || g.K <= 0) return false;
  const uint64_t a_ext = ((uint64_t)(g.M - 1) * (uint64_t)g.lda + (uint64_t)g.K) * 2u;
  if (a_ext > kLim) return false;
  if (g.B.trans)  // one stored [K][N] matrix; the slab step is a signed 32-bit offset
    return ((uint64_t)(g.K - 1) * (uint64_t)g.ldb + (uint64_t)g.N) * 2u <= 0x7FFFFF00ull;
  const int64_t start[3] = {0, g.B.n1, g.B.n2};
  const int64_t end[3] = {g.B.n1, g.B.n2, b_rows};
  for (int k = 0; k < 3; ++k) {
    const int64_t rows = std::min(end[k], b_rows) - start[k];
    if (rows <= 0) continue;
    if (((uint64_t)(rows - 1) * (uint64_t)g.ldb + (uint64_t)g.K) * 2u > kLim) return false;
    if (!swiglu && k > 0 && start[k] % 8 != 0) return false;
  }
  return true;
}

static int gemm_waves() {
  static const int w = [] {
    const char* e = getenv("RP_GEMM_WAVES");
    return e && atoi(e) == 4 ? 4 : 8;
  }();
  return w;
}

// bf16 GEMMs run 8 waves per workgroup (two per SIMD, 64x128 per wave); operands are
// streamed by the LDS-DMA kernel unless they span more than its 2 GiB buffer window.
template <int EPI, typename T16, bool BT = false>
static void launch_half(hipStream_t s, GemmArgs& g, dim3 grid, int64_t b_rows, bool allow_dma = true) {
  if (allow_dma && dma_setup(g, b_rows, EPI == EPI_SWIGLU)) {
    if (!BT && gemm_waves() == 4)  // (the 4-wave tile has no registers left for transposed reads)
      k_gemm_bf16_dma<EPI, T16, 2, false><<<grid, 256, 0, s>>>(g);
    else
      k_gemm_bf16_dma<EPI, T16, 4, BT><<<grid, 512, 0, s>>>(g);
  }
  else
    k_gemm_bf16<EPI, T16, 4, BT><<<grid, 512, 0, s>>>(g);
}

// ------------------------------------------------------------------------------------
// Skinny GEMM: at most 64 rows of A (a decode batch, the last rows of a prefix), 16-bit.
// Such a product reads each weight once and is bound by HBM bandwidth, so the weights
// are streamed, not tiled for reuse.  A workgroup of SW waves owns 32*SW adjacent
// columns (32 per wave) and one K split, and walks the split's 64-deep k slabs through a
// 2-stage LDS ring filled by direct global->LDS loads: per stage one A slab (the few
// rows, copied once and shared by the waves; rows past M repeat row M-1 and their
// results are dropped) and each wave's 32 B rows (8 lanes read a whole 128-byte row
// segment).  Per slab t: wait for this wave's copies of slab t, barrier (every wave's
// copies of t have landed and every wave is done with the stage that takes t+1), issue
// the copies of t+1, then the MFMAs of t.  At 64 rows a workgroup holds 48 KiB of LDS,
// so three fit on a CU and a launch of up to 768 workgroups runs in one round (a 3-stage
// ring, 72 KiB, fitted two: the 592 workgroups of a 7B decode gate/up projection ran in
// two rounds, and the decode step took 1.5% longer).  Past the end the copies re-read
// the last slab into the idle stage.  The MFMA takes the B fragment first and each
// fragment has the k order of the tiled kernels, so every output is the MFMA chain it is
// there (the same bits).  A transposed B ([K][N] storage) is staged k-row-major and read
// with ds_read_b64_tr_b16 into the same fragments.  Output fp32 [split][M][ldo]
// (partials), or C itself (stored or accumulated) for one split.
// ------------------------------------------------------------------------------------
struct SkinnyArgs {
  int M, N, K;
  const void* A;
  int lda;
  BSeg B;
  int ldb;
  float* out;
  int ldo;
  int64_t plane;  // elements between splits of out
  int k_chunk;
  int add;        // accumulate into out (one split)
  ArgmaxPart* arg;  // one split, out may be NULL: each wave's per-row (max, lowest column of it), [M][ceil(N/32)]
};

template <typename T16, int RF, bool BT, int SW>
__global__ __launch_bounds__(SW * 64) void k_gemm_skinny(SkinnyArgs g) {
#if defined(__HIP_DEVICE_COMPILE__)
  typedef __attribute__((address_space(3))) void lds_void;
  typedef typename Half16<T16>::V8 V8;
  typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
  constexpr int ACH = RF * 32 * 8;   // A chunks per stage: RF*32 rows x 8 chunks of 16 bytes
  constexpr int BCH = 32 * 8;        // B chunks per wave per stage: 32 columns x 64 k
  constexpr int AL = ACH / 64 / SW;  // A copy instructions per wave per stage
  constexpr int BL = BCH / 64;       // B copy instructions per wave per stage
  static_assert(AL >= 1 && ACH % (64 * SW) == 0, "A stage split over the waves");
  __shared__ u32x4_t As0[ACH], As1[ACH];
  __shared__ u32x4_t Bs0[SW * BCH], Bs1[SW * BCH];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int fr = lane & 31, fk = lane >> 5;
  const int nw0 = (blockIdx.x * SW + wave) * 32;  // first column of this wave
  const int kbeg = blockIdx.y * g.k_chunk;
  const int nst = (min(g.K, kbeg + g.k_chunk) - kbeg) / 64;  // >= 1 (the host sizes the splits)

  // copy sources: byte offsets into A's buffer resource and into that of the B segment
  // holding the instruction's rows (the host checked that they fit 32 bits)
  const __amdgpu_buffer_rsrc_t rsA = __builtin_amdgcn_make_buffer_rsrc((void*)g.A, 0, -1, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsB0 = __builtin_amdgcn_make_buffer_rsrc((void*)g.B.b0, 0, -1, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsB1 = __builtin_amdgcn_make_buffer_rsrc((void*)g.B.b1, 0, -1, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsB2 = __builtin_amdgcn_make_buffer_rsrc((void*)g.B.b2, 0, -1, 0x00020000);
  uint32_t aoff[AL], boff[BL];
  __amdgpu_buffer_rsrc_t rsB[BL];
#pragma unroll
  for (int i = 0; i < AL; ++i) {
    const int q = (wave * AL + i) * 64 + lane, row = q / 8, lc = (q % 8) ^ swz(row);
    aoff[i] = 2u * ((uint32_t)min(row, g.M - 1) * (uint32_t)g.lda + (uint32_t)(kbeg + lc * 8));
  }
#pragma unroll
  for (int i = 0; i < BL; ++i) {
    const int q = i * 64 + lane;
    if (BT) {  // k row q/4 of the slab, 4 chunks of 8 columns; columns past N re-read the last chunk
      const int kr = q / 4, lc = q % 4;
      rsB[i] = rsB0;
      boff[i] = 2u * ((uint32_t)(kbeg + kr) * (uint32_t)g.ldb + (uint32_t)min(nw0 + lc * 8, g.N - 8));
    } else {  // column row q/8 (clamped to the last column), 8 rows per instruction
      const int row = q / 8, lc = (q % 8) ^ swz(row);
      const int r0 = min(nw0 + i * 8, g.N - 1), r = min(nw0 + row, g.N - 1);
      const int seg = r0 < g.B.n1 ? 0 : r0 < g.B.n2 ? 1 : 2;
      rsB[i] = seg == 0 ? rsB0 : seg == 1 ? rsB1 : rsB2;
      const int sbeg = seg == 0 ? 0 : seg == 1 ? g.B.n1 : g.B.n2;
      boff[i] = 2u * ((uint32_t)(r - sbeg) * (uint32_t)g.ldb + (uint32_t)(kbeg + lc * 8));
    }
  }
  const uint32_t bstep = BT ? 64u * 2u * (uint32_t)g.ldb : 64u * 2u;
  // transposed fragment reads: lane 16 gq + p addresses k row 8 (gq/2) + p/4 (+4 for the
  // second read) at column 16 (gq%2) + 4 (p%4) of this wave's 32 columns
  int btk = 0, btc = 0;
  if (BT) {
    const int gq = lane >> 4, p = lane & 15;
    btk = 8 * (gq >> 1) + (p >> 2);
    btc = 16 * (gq & 1) + 4 * (p & 3);
  }

  f32x16_t acc[RF];
#pragma unroll
  for (int rf = 0; rf < RF; ++rf)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[rf][e] = 0.f;

  auto load = [&](u32x4_t* Ad, u32x4_t* Bd, int t) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < AL; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsA, (lds_void*)(Ad + (wave * AL + i) * 64), 16,
                                               aoff[i] + (uint32_t)t * 128u, 0, 0, 0);
#pragma unroll
    for (int i = 0; i < BL; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsB[i], (lds_void*)(Bd + wave * BCH + i * 64), 16,
                                               boff[i] + (uint32_t)t * bstep, 0, 0, 0);
  };
  auto slab = [&](const u32x4_t* Ac, const u32x4_t* Bc) __attribute__((always_inline)) {
    const u32x4_t* Bw = Bc + wave * BCH;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      V8 bf;
      if (BT) {
        const T16* base = reinterpret_cast<const T16*>(Bw);
        const int kr = ks * 16 + btk;
        const v4i16_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_t*)(base + kr * 32 + btc));
        const v4i16_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_t*)(base + (kr + 4) * 32 + btc));
        const uint2 l2 = __builtin_bit_cast(uint2, lo), h2 = __builtin_bit_cast(uint2, hi);
        bf = Half16<T16>::as_v8(make_uint4(l2.x, l2.y, h2.x, h2.y));
      } else {
        bf = __builtin_bit_cast(V8, Bw[fr * 8 + ((ks * 2 + fk) ^ swz(fr))]);
      }
#pragma unroll
      for (int rf = 0; rf < RF; ++rf) {
        const int row = rf * 32 + fr;
        const V8 af = __builtin_bit_cast(V8, Ac[row * 8 + ((ks * 2 + fk) ^ swz(row))]);
        acc[rf] = Half16<T16>::mma(bf, af, acc[rf]);
      }
    }
  };
  // Wait for this wave's copies of the slab about to be read and for its LDS reads, then
  // the barrier.  The asm also keeps the compiler from moving LDS accesses across the
  // barrier.
#define SK_STEP(AC_, BC_, AN_, BN_, tt_)                                                \
  {                                                                                     \
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");          \
    load(AN_, BN_, min((tt_) + 1, nst - 1));                                            \
    if ((tt_) < nst) slab(AC_, BC_);                                                    \
  }
  load(As0, Bs0, 0);
  for (int t = 0; t < nst; t += 2) {
    SK_STEP(As0, Bs0, As1, Bs1, t);
    SK_STEP(As1, Bs1, As0, Bs0, t + 1);
  }
#undef SK_STEP
  __builtin_amdgcn_s_waitcnt(0);  // no copy into LDS outlives the wave

  // acc[rf][e] = C(row rf*32 + fr, column nw0 + 8 (e/4) + 4 fk + e%4)
  if (g.arg) {  // argmax of each row over this wave's 32 columns; NaN never wins, ties go low
#pragma unroll
    for (int rf = 0; rf < RF; ++rf) {
      float best = -INFINITY;
      int bi = 0x7fffffff;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int n = nw0 + 8 * (e >> 2) + 4 * fk + (e & 3);
        const float v = acc[rf][e];
        if (n < g.N && (v > best || (v == best && n < bi))) {
          best = v;
          bi = n;
        }
      }
      const float vo = __shfl_xor(best, 32, 64);
      const int io = __shfl_xor(bi, 32, 64);
      if (vo > best || (vo == best && io < bi)) {
        best = vo;
        bi = io;
      }
      const int m = rf * 32 + fr;
      // row-major candidates: row m's are contiguous for the reduction
      if (fk == 0 && m < g.M && nw0 < g.N)
        g.arg[(int64_t)m * ((g.N + 31) / 32) + blockIdx.x * SW + wave] = ArgmaxPart{best, bi};
    }
    if (!g.out) return;
  }
  float* outp = g.out + (int64_t)blockIdx.y * g.plane;
  const bool vec = (g.ldo & 3) == 0 && ((uintptr_t)g.out & 15) == 0 && (g.plane & 3) == 0;
#pragma unroll
  for (int rf = 0; rf < RF; ++rf) {
    const int m = rf * 32 + fr;
    if (m >= g.M) continue;
    float* row = outp + (int64_t)m * g.ldo;
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      const float v[4] = {acc[rf][4 * q4], acc[rf][4 * q4 + 1], acc[rf][4 * q4 + 2], acc[rf][4 * q4 + 3]};
      const int n = nw0 + 8 * q4 + 4 * fk;
      if (g.add)
        store4<true>(row, n, g.N, v, vec);
      else
        store4<false>(row, n, g.N, v, vec);
    }
  }
#endif
}

// Waves per workgroup of the skinny GEMM (32 columns each; they share the A slabs).
// Four measured best at every decode shape: the shared A slab costs less per weight
// byte, and the LDS (48 KiB a workgroup at 64 rows) still holds three workgroups per CU.
constexpr int kSkinnyWaves = 4;

#ifndef RP_SKINNY_BLOCKS
#define RP_SKINNY_BLOCKS 512
#endif
int32_t gemm_skinny_splitk(int32_t M, int32_t N, int32_t K) {
  if (M > 64 || K % 64) return 1;
  const int cols = 32 * kSkinnyWaves;
  const int tiles = (N + cols - 1) / cols;
  const int s = (RP_SKINNY_BLOCKS + tiles - 1) / tiles;   // about two workgroups per CU
  const int cap = std::max(1, std::min(16, K / 64 / 4));  // at least 4 slabs per split
  return std::max(1, std::min(s, cap));
}

// Operands the skinny kernel takes (16-bit, as launch_gemm validated them).
static bool skinny_setup(const GemmArgs& g, Epi epi, bool split) {
  if (g.M > 64 || g.K % 64 || (g.lda & 7) || ((uintptr_t)g.A & 15)) return false;
  if (((uint64_t)(g.M - 1) * (uint64_t)g.lda + (uint64_t)g.K) * 2u > 0xFFFFFF00ull) return false;
  if (!(epi == EPI_PARTIALS || ((epi == EPI_STORE_F32 || epi == EPI_ADD_F32) && !split) || split)) return false;
  if (epi == EPI_SWIGLU || epi == EPI_LSE || epi == EPI_ROPE) return false;
  if (g.B.trans)
    return !((g.N & 7) || (g.ldb & 7) || ((uintptr_t)g.B.b0 & 15)) &&
           ((uint64_t)(g.K - 1) * (uint64_t)g.ldb + (uint64_t)g.N) * 2u <= 0x7FFFFF00ull;
  const int64_t start[3] = {0, g.B.n1, g.B.n2};
  const int64_t end[3] = {g.B.n1, g.B.n2, g.N};
  for (int k = 0; k < 3; ++k) {
    const int64_t rows = std::min<int64_t>(end[k], g.N) - start[k];
    if (rows <= 0) continue;
    if (k > 0 && start[k] % 8 != 0) return false;
    if (((uint64_t)(rows - 1) * (uint64_t)g.ldb + (uint64_t)g.K) * 2u > 0xFFFFFF00ull) return false;
  }
  return true;
}

template <typename T16, bool BT, int SW>
static void launch_skinny_w(hipStream_t s, const SkinnyArgs& a, dim3 grid) {
  if (a.M <= 32)
    k_gemm_skinny<T16, 1, BT, SW><<<grid, SW * 64, 0, s>>>(a);
  else
    k_gemm_skinny<T16, 2, BT, SW><<<grid, SW * 64, 0, s>>>(a);
}

template <typename T16>
static void launch_skinny(hipStream_t s, const GemmArgs& g, int splitk, float* out, int ldo, int64_t plane,
                          bool add, ArgmaxPart* arg = nullptr) {
  SkinnyArgs a;
  a.M = g.M;
  a.N = g.N;
  a.K = g.K;
  a.A = g.A;
  a.lda = g.lda;
  a.B = g.B;
  a.ldb = g.ldb;
  a.out = out;
  a.ldo = ldo;
  a.plane = plane;
  a.k_chunk = g.k_chunk;
  a.add = add ? 1 : 0;
  a.arg = arg;
  constexpr int SW = kSkinnyWaves;
  const dim3 grid((g.N + 32 * SW - 1) / (32 * SW), splitk);
  if (g.B.trans)
    launch_skinny_w<T16, true, SW>(s, a, grid);
  else
    launch_skinny_w<T16, false, SW>(s, a, grid);
}

int32_t gemm_effective_splitk(rp_dtype dt, int32_t K, int32_t splitk) {
  const int bk = dt != RP_F32 ? GB_K : GF_K;
  const int kblocks = (K + bk - 1) / bk;
  if (splitk < 1) splitk = 1;
  if (splitk > kblocks) splitk = kblocks;
  const int k_chunk = ((kblocks + splitk - 1) / splitk) * bk;
  return (K + k_chunk - 1) / k_chunk;
}

// A launch of 256x256 tiles pays for a whole round of 256 however few tiles the last one
// holds.  Where that is dear, the 256x256 kernel takes the rows or the columns that fill its
// rounds and the flexible tiles the rest, as a second launch (every output keeps its bits).
// us, whole / cut: 7B down projection of 14229 rows (784 tiles, 3.06 rounds) 1800 / 1539,
// gate/up of 1024 rows (592, 2.3) 258 / 241, lm_head of 1024 rows (2376, 9.3) 1017 / 992;
// 32B down projection of 10000 rows 2600 / 2210.
// A tail of rows reads all of B a second time.  Where B is far more than the Infinity Cache's
// 256 MB and that read is all of the tail's cost, it takes 7% more than at 5 TB/s (lm_head of 130
// rows: 234 us for 218): else the fused lm_head of 880 and 926 rows was cut after 768, 977 and 1004
// us a call, cut by columns 926 and 926 (whole: 942 and 950).  A gate/up projection of 271 MB is
// cut by rows: two layers of 2570 rows 2437 us a call, by columns 2493.
static bool cut_last_round(GemmArgs* g, GemmArgs* tail, int epi, int c_bytes) {
  const int nt = epi == EPI_SWIGLU ? 128 : GB_N;  // output columns of a tile
  const int64_t tm = (g->M + GB_M - 1) / GB_M, tn = (g->N + nt - 1) / nt;
  const int64_t full = tm * tn / 256 * 256;
  const bool big_b = 2. * g->K * g->N * (epi == EPI_SWIGLU ? 2. : 1.) > 512e6;
  double best = gemm_cost_256(*g, epi, 1) * 0.97;  // below 3% the second launch is not worth it
  GemmArgs head_best, tail_best;
  bool found = false;
  for (int rows = 0; rows < 2; ++rows) {
    const int64_t keep = full / (rows ? tn : tm);  // tile rows (columns) of the head
    if (keep < 1 || keep >= (rows ? tm : tn)) continue;
    GemmArgs h = *g, t = *g;
    if (rows) {
      const int64_t m = keep * GB_M;
      h.M = (int)m;
      t.M = g->M - (int)m;
      t.A = (const char*)g->A + m * g->lda * 2;
      if (epi == EPI_LSE) {
        t.lse.ids += m;
        t.lse.lse += m * g->n_part * 2;
        t.lse.tgt += m;
      } else if (epi == EPI_ROPE) {
        t.rope.q = (char*)g->rope.q + m * g->rope.hq * 2;
        t.rope.k = (char*)g->rope.k + m * g->rope.hkv * 2;
        t.rope.v = (char*)g->rope.v + m * g->rope.hkv * 2;
        t.rope.cs = g->rope.cs + m * (g->rope.D / 2);
      } else {
        t.C = (char*)g->C + m * g->ldc * c_bytes;
      }
    } else {
      const int64_t n = keep * nt;
      h.N = (int)n;
      t.N = g->N - (int)n;
      t.n_off = (int)n;
      if (epi != EPI_LSE && epi != EPI_ROPE) t.C = (char*)g->C + n * c_bytes;
    }
    const double cost_tail = std::max(gemm_cost_flex(t, epi, 1), rows && big_b ? 1.07 * gemm_hbm_floor(t, epi, 1) : 0.);
    const double cost = gemm_cost_256(h, epi, 1) + cost_tail + 3000.;
    if (cost < best) {
      best = cost;
      head_best = h;
      tail_best = t;
      found = true;
    }
  }
  if (found) {
    *g = head_best;
    *tail = tail_best;
  }
  return found;
}

// The fused SwiGLU with K summed as split-K partials would be: at most 64 rows, two or three
// chunks (what k_gemm_flex has the registers for).
bool gemm_swiglu_chunks(rp_dtype dt, int32_t M, int32_t N, int32_t K, int32_t splitk) {
  return dt != RP_F32 && M <= 64 && K % GB_K == 0 && gemm_effective_splitk(dt, K, splitk) <= 3 &&
         (uint64_t)N * K * 2u <= 0xFFFFFF00ull;
}

// The kernels of one GEMM: g (and tail, the launch that follows where the last round is cut).
struct GemmChoice {
  GemmForm form;
  GemmArgs g, tail;
  int splitk;
  bool split;      // partials (summed by the caller, or by the reduction)
  int epi;         // epilogue of the kernel (-1: partials)
  int64_t b_rows;  // logical rows of B
};
static GemmChoice gemm_choose(rp_dtype dt, Epi epi, int splitk, GemmArgs g) {
  const bool half = dt != RP_F32;
  GemmChoice c;
  if (splitk < 1) splitk = 1;
  const int bk = half ? GB_K : GF_K;
  const int kblocks = (g.K + bk - 1) / bk;
  if (splitk > kblocks) splitk = kblocks;
  g.k_chunk = ((kblocks + splitk - 1) / splitk) * bk;
  splitk = (g.K + g.k_chunk - 1) / g.k_chunk;
  if (epi == EPI_SWIGLU && splitk > 1) {  // the chunks are summed in the kernel
    g.k_sum = g.k_chunk;
    g.k_chunk = g.K;
    splitk = 1;
  }
  c.splitk = splitk;
  // EPI_PARTIALS: the partials epilogue even for one split, and no reduction here
  c.split = splitk > 1 || epi == EPI_PARTIALS;
  c.b_rows = epi == EPI_SWIGLU ? (int64_t)g.B.n1 + g.N : g.N;
  c.epi = c.split ? -1 : (int)epi;
  c.g = g;
  c.form = kGemmF32;
  if (!half) return c;
  const bool flex_ok = (epi != EPI_STORE || c.split) && dma_setup(g, c.b_rows, epi == EPI_SWIGLU);
  if (g.k_sum) {
    c.form = flex_ok ? kGemmFlex : kGemmNone;
    return c;
  }
  const bool flex = flex_ok && gemm_cost_flex(g, c.epi, splitk) < 0.9 * gemm_cost_256(g, c.epi, splitk);
  // Up to 64 rows the skinny kernel streams the weights with three workgroups of two stages
  // per CU; where its launch is less than one such workgroup per CU, the flexible tile's deeper
  // ring reads faster (same bits).  Of 48 rows, 7B shapes, us (with timing events), skinny /
  // flexible: q/k/v in 3 splits (108 workgroups) 21 / 16, down in 8 (224) 44 / 36; a decode
  // step's 504 and 448 workgroups: 15 / 19 and 36 / 38.
  if (skinny_setup(g, epi, c.split) && !(flex && (int64_t)((g.N + 127) / 128) * splitk <= 256)) {
    c.form = kGemmSkinny;
  } else if (flex) {
    c.form = kGemmFlex;
  } else {
    const bool cut = flex_ok && !c.split && cut_last_round(&c.g, &c.tail, epi, epi == EPI_SWIGLU ? 2 : 4);
    c.form = !cut ? kGemm256 : c.tail.M < g.M ? kGemmCutRows : kGemmCutCols;
  }
  return c;
}

GemmForm gemm_form(rp_dtype dt, int32_t M, int32_t N, int32_t K, bool trans, Epi epi, int32_t splitk, int32_t* tile) {
  GemmArgs g{};
  g.M = M;
  g.N = N;
  g.K = K;
  g.lda = K;
  g.B = BSeg{nullptr, nullptr, nullptr, N, epi == EPI_SWIGLU ? 2 * N : N, trans};
  g.ldb = trans ? N : K;
  g.ldc = N;
  g.n_part = lse_parts(N);
  g.n_all = N;
  const GemmChoice c = gemm_choose(dt, epi, splitk, g);
  *tile = c.form == kGemmFlex ? gemm_flex_tile(c.g, c.epi, c.splitk)
          : c.form == kGemmCutRows || c.form == kGemmCutCols ? gemm_flex_tile(c.tail, c.epi, 1) : 0;
  return c.form;
}

hipError_t launch_gemm(hipStream_t s, rp_dtype dt, int32_t M, int32_t N, int32_t K, const void* A,
                       int32_t lda, const BSeg& B, int32_t ldb, void* C, int32_t ldc, Epi epi,
                       int32_t splitk, float* partials, const LseOut* lse, const RopeOut* rope) {
  if (M <= 0 || N <= 0) return hipSuccess;
  const bool half = dt != RP_F32;
  if (epi == EPI_ROPE &&
      (!half || splitk > 1 || B.trans || !rope || (rope->D != 64 && rope->D != 128) ||
       N != rope->hq + 2 * rope->hkv || (rope->hq % rope->D) || (rope->hkv % rope->D) || ((uintptr_t)rope->cs & 15) ||
       (((uintptr_t)rope->q | (uintptr_t)rope->k | (uintptr_t)rope->v) & 7)))
    return hipErrorInvalidValue;
  if (epi == EPI_SWIGLU && (!half || (splitk > 1 && !gemm_swiglu_chunks(dt, M, N, K, splitk)))) return hipErrorInvalidValue;
  if (epi == EPI_LSE && (!half || splitk > 1 || !lse)) return hipErrorInvalidValue;
  if (epi == EPI_PARTIALS && !partials) return hipErrorInvalidValue;
  // a transposed B serves the row-parallel projections: residual or split-K epilogue
  if (B.trans && ((epi != EPI_ADD_F32 && epi != EPI_PARTIALS && splitk <= 1) || ldb < N ||
                  (half && ((N & 7) || (ldb & 7) || ((uintptr_t)B.b0 & 15)))))
    return hipErrorInvalidValue;
  GemmArgs g;
  g.M = M;
  g.N = N;
  g.K = K;
  g.A = A;
  g.lda = lda;
  g.B = B;
  g.ldb = ldb;
  g.C = C;
  g.ldc = ldc;
  g.partials = partials;
  g.lse = lse ? *lse : LseOut{nullptr, nullptr, nullptr};
  g.rope = rope ? *rope : RopeOut{};
  g.n_part = lse_parts(N);
  g.n_all = N;
  GemmChoice c = gemm_choose(dt, epi, splitk, g);
  if (c.form == kGemmNone) return hipErrorInvalidValue;
  g = c.g;
  splitk = c.splitk;
  const bool split = c.split;
  if (c.form == kGemmSkinny) {
    // split: partials (summed by the caller, or by the reduction below); else C itself
    with_half16(dt, [&](auto tag_) {
      using H = decltype(tag_);
      if (split)
        launch_skinny<H>(s, g, splitk, partials, N, (int64_t)M * N, false);
      else
        launch_skinny<H>(s, g, 1, (float*)C, ldc, 0, epi == EPI_ADD_F32);
    });
  } else if (c.form == kGemmFlex) {
    const hipError_t em = launch_flex_gemm(s, dt, c.epi, g, splitk);
    if (em != hipSuccess) return em;
  } else if (half) {
    const int64_t b_rows = c.b_rows;
    g.tiles_m = (g.M + GB_M - 1) / GB_M;
    g.tiles_n = epi == EPI_SWIGLU ? (g.N + 127) / 128 : (g.N + GB_N - 1) / GB_N;
    dim3 grid(g.tiles_m * g.tiles_n, splitk);
    with_half16(dt, [&](auto tag_) {
      using H = decltype(tag_);
      if (B.trans && split)
        launch_half<-1, H, true>(s, g, grid, b_rows);
      else if (B.trans)
        launch_half<EPI_ADD_F32, H, true>(s, g, grid, b_rows);
      else if (split)
        launch_half<-1, H>(s, g, grid, b_rows);
      else if (epi == EPI_STORE)
        launch_half<EPI_STORE, H>(s, g, grid, b_rows);
      else if (epi == EPI_STORE_F32)
        launch_half<EPI_STORE_F32, H>(s, g, grid, b_rows);
      else if (epi == EPI_SWIGLU)
        launch_half<EPI_SWIGLU, H>(s, g, grid, b_rows);
      else if (epi == EPI_LSE)
        launch_half<EPI_LSE, H>(s, g, grid, b_rows);
      else if (epi == EPI_ROPE)
        launch_half<EPI_ROPE, H>(s, g, grid, b_rows);
      else
        launch_half<EPI_ADD_F32, H>(s, g, grid, b_rows);
    });
    if (c.form != kGemm256) {
      const hipError_t em = launch_flex_gemm(s, dt, epi, c.tail, 1);
      if (em != hipSuccess) return em;
    }
  } else {
    g.tiles_m = (M + GF_M - 1) / GF_M;
    g.tiles_n = (N + GF_N - 1) / GF_N;
    dim3 grid(g.tiles_m * g.tiles_n, splitk);
    if (B.trans && split)
      k_gemm_f32<-1, true><<<grid, 256, 0, s>>>(g);
    else if (B.trans)
      k_gemm_f32<EPI_ADD_F32, true><<<grid, 256, 0, s>>>(g);
    else if (split)
      k_gemm_f32<-1><<<grid, 256, 0, s>>>(g);
    else if (epi == EPI_ADD_F32)
      k_gemm_f32<EPI_ADD_F32><<<grid, 256, 0, s>>>(g);
    else
      k_gemm_f32<EPI_STORE_F32><<<grid, 256, 0, s>>>(g);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || !split || epi == EPI_PARTIALS) return e;
  const int64_t total = (int64_t)M * N;
  const int blocks = (int)std::min<int64_t>((total + 255) / 256, 4096);
  if (epi == EPI_STORE && dt == RP_BF16)
    k_splitk_reduce<EPI_STORE, bf16_t><<<blocks, 256, 0, s>>>(partials, splitk, M, N, C, ldc);
  else if (epi == EPI_STORE && dt == RP_F16)
    k_splitk_reduce<EPI_STORE, f16_t><<<blocks, 256, 0, s>>>(partials, splitk, M, N, C, ldc);
  else if (epi == EPI_STORE || epi == EPI_STORE_F32)
    k_splitk_reduce<EPI_STORE_F32, float><<<blocks, 256, 0, s>>>(partials, splitk, M, N, C, ldc);
  else
    k_splitk_reduce<EPI_ADD_F32, float><<<blocks, 256, 0, s>>>(partials, splitk, M, N, C, ldc);
  return hipGetLastError();
}

// C = A . B^T reduced to each row's argmax (the lowest column of the row's maximum; NaN
// never wins; -1 for a row with no candidate), C stored only if the caller wants it: the
// skinny kernel writes each wave's per-row candidate and k_argmax_parts picks among them in
// column order (64 x 152064: 4 us, where reading the stored logits back took 16).
bool gemm_argmax_supported(rp_dtype dt, int32_t M, int32_t N, int32_t K, int32_t lda, int32_t ldb) {
  if (dt == RP_F32 || M < 1 || N < 1 || M > 64 || K % 64) return false;
  if (gemm_skinny_splitk(M, N, K) != 1 || gemm_effective_splitk(dt, K, gemm_skinny_splitk(M, N, K)) != 1) return false;
  GemmArgs g;
  g.M = M;
  g.N = N;
  g.K = K;
  g.A = nullptr;
  g.lda = lda;
  g.B = BSeg{nullptr, nullptr, nullptr, N, N};
  g.ldb = ldb;
  return skinny_setup(g, EPI_STORE_F32, false);
}

size_t gemm_argmax_parts(int32_t M, int32_t N) { return (size_t)M * ((N + 31) / 32); }

__global__ __launch_bounds__(256) void k_argmax_parts(const ArgmaxPart* __restrict__ part, int nparts, int M,
                                                      int32_t* __restrict__ out) {
  const int m = blockIdx.x;
  float best = -INFINITY;
  int bi = 0x7fffffff;
  auto merge = [&](const ArgmaxPart& p) {
    if (p.v > best || (p.v == best && p.i < bi)) {
      best = p.v;
      bi = p.i;
    }
  };
  // row m's candidates are contiguous: eight coalesced loads in flight per thread (the
  // merge is order-independent: a total order on (value, -index), NaN never wins)
  const ArgmaxPart* row = part + (int64_t)m * nparts;
  int t = threadIdx.x;
  for (; t + 7 * 256 < nparts; t += 8 * 256) {
    ArgmaxPart p[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) p[u] = row[t + u * 256];
#pragma unroll
    for (int u = 0; u < 8; ++u) merge(p[u]);
  }
  for (; t < nparts; t += 256) merge(row[t]);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const float vb = __shfl_xor(best, o, kWave);
    const int ib = __shfl_xor(bi, o, kWave);
    if (vb > best || (vb == best && ib < bi)) {
      best = vb;
      bi = ib;
    }
  }
  __shared__ float sv[4];
  __shared__ int si[4];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (lane == 0) {
    sv[w] = best;
    si[w] = bi;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int k = 1; k < 4; ++k)
      if (sv[k] > best || (sv[k] == best && si[k] < bi)) {
        best = sv[k];
        bi = si[k];
      }
    out[m] = bi == 0x7fffffff ? -1 : bi;
  }
}

hipError_t launch_gemm_argmax(hipStream_t s, rp_dtype dt, int32_t M, int32_t N, int32_t K, const void* A,
                              int32_t lda, const BSeg& B, int32_t ldb, float* C, ArgmaxPart* parts, int32_t* out) {
  if (!gemm_argmax_supported(dt, M, N, K, lda, ldb) || B.trans || ((uintptr_t)A & 15) || ((uintptr_t)B.b0 & 15) ||
      !parts || !out)
    return hipErrorInvalidValue;
  GemmArgs g;
  g.M = M;
  g.N = N;
  g.K = K;
  g.A = A;
  g.lda = lda;
  g.B = B;
  g.ldb = ldb;
  g.k_chunk = K;
  with_half16(dt, [&](auto tag_) {
    using H = decltype(tag_);
    launch_skinny<H>(s, g, 1, C, N, 0, false, parts);
  });
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  k_argmax_parts<<<M, 256, 0, s>>>(parts, (N + 31) / 32, M, out);
  return hipGetLastError();
}

// Timing-harness hook: plain bf16 store epilogue; variant 0 forces the register-staged
// kernel, any other value the LDS-DMA kernel.
hipError_t launch_gemm_variant(hipStream_t s, int variant, int32_t M, int32_t N, int32_t K, const void* A,
                               const void* B, void* C) {
  GemmArgs g;
  g.M = M;
  g.N = N;
  g.K = K;
  g.A = A;
  g.lda = K;
  g.B = BSeg{B, B, B, N, N};
  g.ldb = K;
  g.C = C;
  g.ldc = N;
  g.partials = nullptr;
  g.k_chunk = K;
  g.tiles_m = (M + GB_M - 1) / GB_M;
  g.tiles_n = (N + GB_N - 1) / GB_N;
  dim3 grid(g.tiles_m * g.tiles_n, 1);
  launch_half<EPI_STORE, bf16_t>(s, g, grid, N, variant != 0);
  return hipGetLastError();
}

}  // namespace rp
