// 16-bit MFMA GEMM over tiles of 32 RF rows by 32 SW columns: the launches whose 256x256
// tiles would leave much of the chip idle or would mostly compute padding (short prompts,
// responses, decode batches).
#include "gemm_common.h"

#include <algorithm>

namespace rp {

// Transposed B slabs are staged as stored, [64 k][128 n], 16 chunks of 16 bytes per k row
// (one row spans all 64 banks): a transposed fragment read covers 4 k rows x 4 chunks per
// half wave, which this XOR gives distinct banks.
__device__ __forceinline__ int swzx(int k) { return (k & 3) << 2; }

template <int N>
__device__ __forceinline__ void wait_vm_barrier() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

// SW waves side by side, each 32 RF rows by 32 columns; 64-deep k slabs of A and B are copied
// straight into an NS-stage LDS ring (buffer_load ... lds, rows XOR-swizzled as in the
// 256x256 kernel) up to NS - 1 slabs ahead.  MFMA shape, operand order and k order are those
// of the other 16-bit kernels, so every output is the same MFMA chain: the same bits
// whichever tile computes it.  Bound by the copies (see flex_pick): with the MFMAs and the
// fragment reads taken out the kernel takes 98-100% of its time, without the copies half.
// CK (SwiGLU only): K is summed in two or three chunks of k_sum, added in order as
// launch_splitk_swiglu adds that many split-K partials, so a decode step's gate/up projection
// keeps the bits of its split form without writing the partials.  (Four chunks, added as
// (0 + 1) + (2 + 3), need a third set of accumulators: at 160 rows 179 us, 121 split.)
template <int EPI, typename T16, int RF, int SW, int NS, bool BT = false, bool CK = false>
__global__ __launch_bounds__(SW * 64) void k_gemm_flex(GemmArgs g) {
#if defined(__HIP_DEVICE_COMPILE__)
  typedef __attribute__((address_space(3))) void lds_void;
  typedef typename Half16<T16>::V8 V8;
  typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
  constexpr int MT = 32 * RF, NT = 32 * SW;     // tile
  constexpr int AI = 4 * RF;                    // copy instructions (8 rows each) of an A slab
  constexpr int LA = (AI + SW - 1) / SW, LB = 4, L = LA + LB;  // per wave (A: the last may repeat)
  constexpr int SC = (MT + NT) * 8;             // 16-byte chunks of a stage: A rows, then B rows
  constexpr int NREAD = RF + (BT ? 2 : 1);      // LDS reads per k-step
  constexpr uint32_t kOob = 0xFFFFFFF0u;        // past every resource's extent: nothing is fetched
  static_assert(NS >= 2 && NS <= 6 && (NS - 1) * L <= 63, "ring");
  static_assert(SW == 4 || (!BT && EPI == (SW == 2 ? -1 : (int)EPI_SWIGLU)), "128-column tiles");
  __shared__ u32x4_t S0[SC], S1[SC];
  __shared__ u32x4_t S2[NS > 2 ? SC : 1], S3[NS > 3 ? SC : 1], S4[NS > 4 ? SC : 1], S5[NS > 5 ? SC : 1];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int tm, tn;
  tile_coords(xcd_remap(blockIdx.x, gridDim.x), g.tiles_m, g.tiles_n, &tm, &tn);
  const int m0 = tm * MT;
  const int kbeg = blockIdx.y * g.k_chunk;
  const int KT = (min(g.K, kbeg + g.k_chunk) - kbeg) / GB_K;
  static_assert(!CK || EPI == EPI_SWIGLU, "chunked sums");

  const __amdgpu_buffer_rsrc_t rsA = __builtin_amdgcn_make_buffer_rsrc((void*)g.A, 0, (int)0xFFFFFF00u, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsB0 = __builtin_amdgcn_make_buffer_rsrc((void*)g.B.b0, 0, (int)0xFFFFFF00u, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsB1 = __builtin_amdgcn_make_buffer_rsrc((void*)g.B.b1, 0, (int)0xFFFFFF00u, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsB2 = __builtin_amdgcn_make_buffer_rsrc((void*)g.B.b2, 0, (int)0xFFFFFF00u, 0x00020000);
  auto b_logical = [&](int r) -> int {
    if (EPI == EPI_SWIGLU)  // a wave's 32 rows: 16 gate rows, then the matching 16 up rows
      return ((r & 16) ? g.B.n1 : 0) + min((tn * SW + (r >> 5)) * 16 + (r & 15), g.N - 1) + g.n_off;
    return min(tn * NT + r, g.N - 1) + g.n_off;
  };
  uint32_t aoff[LA], boff[LB];
  int ablk[LA];  // 8-row block each A copy fills
  __amdgpu_buffer_rsrc_t rsB[LB];
#pragma unroll
  for (int i = 0; i < LA; ++i) {
    ablk[i] = min(wave * LA + i, AI - 1);
    const int r = ablk[i] * 8 + (lane >> 3);
    const int c = (lane & 7) ^ swz(r);
    aoff[i] = 2u * ((uint32_t)min(m0 + r, g.M - 1) * (uint32_t)g.lda + (uint32_t)(kbeg + c * 8));
  }
#pragma unroll
  for (int i = 0; i < LB; ++i) {
    if (BT) {  // 64 chunks = 4 k rows; columns past N (N % 8 == 0) re-read the last chunk
      const int kr = 4 * (wave * LB + i) + (lane >> 4);
      const int cb = (lane & 15) ^ swzx(kr);
      rsB[i] = rsB0;
      boff[i] = 2u * ((uint32_t)(kbeg + kr) * (uint32_t)g.ldb + (uint32_t)(min(tn * NT + cb * 8, g.N - 8) + g.n_off));
    } else {
      const int r0 = (wave * LB + i) * 8, r = r0 + (lane >> 3);
      const int c = (lane & 7) ^ swz(r);
      const int br0 = b_logical(r0);
      const int seg = br0 < g.B.n1 ? 0 : br0 < g.B.n2 ? 1 : 2;
      rsB[i] = seg == 0 ? rsB0 : seg == 1 ? rsB1 : rsB2;
      const int sbeg = seg == 0 ? 0 : seg == 1 ? g.B.n1 : g.B.n2;
      boff[i] = 2u * ((uint32_t)(b_logical(r) - sbeg) * (uint32_t)g.ldb + (uint32_t)(kbeg + c * 8));
    }
  }
  const uint32_t bstep = BT ? (uint32_t)GB_K * 2u * (uint32_t)g.ldb : (uint32_t)GB_K * 2u;
  // Copies of slab t_ into stage D_; past the last slab the offsets are out of range, so
  // nothing is fetched and the count of outstanding copies stays the same.
#define X_LOAD(D_, t_)                                                                                   \
  {                                                                                                      \
    const uint32_t oob_ = (t_) < KT ? 0u : kOob;                                                         \
    const int so_ = (t_) < KT ? (t_) : 0;                                                                \
    _Pragma("unroll") for (int i = 0; i < LA; ++i) __builtin_amdgcn_raw_ptr_buffer_load_lds(             \
        rsA, (lds_void*)(D_ + ablk[i] * 64), 16, aoff[i] | oob_, so_ * (GB_K * 2), 0, 0);                \
    _Pragma("unroll") for (int i = 0; i < LB; ++i) __builtin_amdgcn_raw_ptr_buffer_load_lds(             \
        rsB[i], (lds_void*)(D_ + MT * 8 + (wave * LB + i) * 64), 16, boff[i] | oob_,                     \
        (int)((uint32_t)so_ * bstep), 0, 0);                                                             \
  }
#define X_FRAGS(AF, BF, S_, ks_)                                                                  \
  if (BT) {                                                                                       \
    const T16* p_ = reinterpret_cast<const T16*>(S_ + MT * 8) + btoff + (ks_) * 16 * NT;          \
    const v4i16_t lo_ = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_t*)p_);                \
    const v4i16_t hi_ = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_t*)(p_ + 4 * NT));     \
    const uint2 l2_ = __builtin_bit_cast(uint2, lo_), h2_ = __builtin_bit_cast(uint2, hi_);       \
    BF = Half16<T16>::as_v8(make_uint4(l2_.x, l2_.y, h2_.x, h2_.y));                              \
  } else {                                                                                        \
    BF = __builtin_bit_cast(V8, S_[bfr[ks_]]);                                                    \
  }                                                                                               \
  _Pragma("unroll") for (int i = 0; i < RF; ++i) AF[i] = __builtin_bit_cast(V8, S_[afr[ks_] + i * 256]);
#define X_MMA(AF, BF) \
  _Pragma("unroll") for (int i = 0; i < RF; ++i) acc[i] = Half16<T16>::mma(BF, AF[i], acc[i]);
#define X_REGION(n_mem_)                                                                          \
  _Pragma("unroll") for (int q = 0; q < RF; ++q) {                                                \
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                                            \
    if (q * 2 < NREAD) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);                         \
    if ((n_mem_) > 0) __builtin_amdgcn_sched_group_barrier(0x010, ((n_mem_) + RF - 1) / RF, 0);   \
  }
  // One slab read from S_ (next slab in N_): each k-step's fragments are read under the
  // previous k-step's MFMAs.  The barrier before the last k-step says that this slab has
  // been read by every wave and that every wave's copies of the next one have landed; the
  // copies of slab t + NS then go into S_.
#define X_SLAB(S_, N_, t_)                             \
  {                                                    \
    X_FRAGS(af1, bf1, S_, 1);                          \
    X_MMA(af0, bf0);                                   \
    X_REGION(0);                                       \
    __builtin_amdgcn_sched_barrier(0);                 \
    X_FRAGS(af0, bf0, S_, 2);                          \
    X_MMA(af1, bf1);                                   \
    X_REGION(0);                                       \
    __builtin_amdgcn_sched_barrier(0);                 \
    X_FRAGS(af1, bf1, S_, 3);                          \
    X_MMA(af0, bf0);                                   \
    X_REGION(0);                                       \
    __builtin_amdgcn_sched_barrier(0);                 \
    wait_vm_barrier<(NS - 2) * L>();                   \
    X_FRAGS(af0, bf0, N_, 0);                          \
    X_MMA(af1, bf1);                                   \
    X_LOAD(S_, (t_) + NS);                             \
    X_REGION(L);                                       \
    __builtin_amdgcn_sched_barrier(0);                 \
    if (CK && (t_) + 1 == fold_at && fold_at < KT) fold(); \
  }

  f32x16_t acc[RF];
#pragma unroll
  for (int i = 0; i < RF; ++i)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[i][e] = 0.f;
  f32x16_t done[CK ? RF : 1];  // the sum of the chunks that are done
  bool first = true;
  int fold_at = CK ? g.k_sum / GB_K : 0;  // slab count at the running chunk's end
  auto fold = [&]() __attribute__((always_inline)) {
    if constexpr (CK) {
#pragma unroll
      for (int i = 0; i < RF; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          done[i][e] = first ? acc[i][e] : done[i][e] + acc[i][e];
          acc[i][e] = 0.f;
        }
      first = false;
      fold_at += g.k_sum / GB_K;
    }
  };
  const int fr = lane & 31, fk = lane >> 5;
  int afr[4], bfr[4];  // chunk of fragment 0 at each k-step (32 rows on, the swizzle repeats)
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
    afr[ks] = fr * 8 + ((ks * 2 + fk) ^ swz(fr));
    bfr[ks] = (MT + wave * 32 + fr) * 8 + ((ks * 2 + fk) ^ swz(fr));
  }
  int btoff = 0;
  if (BT) {
    const int gq = lane >> 4, p = lane & 15;
    const int kr = 8 * (gq >> 1) + (p >> 2);
    const int nb = wave * 32 + 16 * (gq & 1) + 4 * (p & 3);
    btoff = kr * NT + (((nb >> 3) ^ swzx(kr)) << 3) + (nb & 7);
  }
  V8 af0[RF], af1[RF], bf0, bf1;
  if (KT > 0) {
    X_LOAD(S0, 0);
    X_LOAD(S1, 1);
    if constexpr (NS > 2) X_LOAD(S2, 2);
    if constexpr (NS > 3) X_LOAD(S3, 3);
    if constexpr (NS > 4) X_LOAD(S4, 4);
    if constexpr (NS > 5) X_LOAD(S5, 5);
    wait_vm_barrier<(NS - 1) * L>();
    X_FRAGS(af0, bf0, S0, 0);
    // The loop is unrolled over the ring, each stage an array of its own, and has no exit
    // inside: so the compiler's own waits for the copies are exact.
    int kt = 0;
    for (; kt + NS <= KT; kt += NS) {
      X_SLAB(S0, S1, kt);
      if constexpr (NS == 2) X_SLAB(S1, S0, kt + 1);
      if constexpr (NS > 2) X_SLAB(S1, S2, kt + 1);
      if constexpr (NS == 3) X_SLAB(S2, S0, kt + 2);
      if constexpr (NS > 3) X_SLAB(S2, S3, kt + 2);
      if constexpr (NS == 4) X_SLAB(S3, S0, kt + 3);
      if constexpr (NS > 4) X_SLAB(S3, S4, kt + 3);
      if constexpr (NS == 5) X_SLAB(S4, S0, kt + 4);
      if constexpr (NS > 5) X_SLAB(S4, S5, kt + 4);
      if constexpr (NS == 6) X_SLAB(S5, S0, kt + 5);
    }
    if (kt < KT) X_SLAB(S0, S1, kt);
    if constexpr (NS > 2)
      if (kt + 1 < KT) X_SLAB(S1, S2, kt + 1);
    if constexpr (NS > 3)
      if (kt + 2 < KT) X_SLAB(S2, S3, kt + 2);
    if constexpr (NS > 4)
      if (kt + 3 < KT) X_SLAB(S3, S4, kt + 3);
    if constexpr (NS > 5)
      if (kt + 4 < KT) X_SLAB(S4, S5, kt + 4);
  }
#undef X_LOAD
#undef X_FRAGS
#undef X_MMA
#undef X_REGION
#undef X_SLAB
  if constexpr (CK) {  // the last chunk is still in acc
#pragma unroll
    for (int i = 0; i < RF; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][e] = done[i][e] + acc[i][e];
  }
  wait_vm_barrier<0>();  // no copy into LDS is in flight, every wave has read its fragments

  // ---- epilogue through LDS: fp32 rows staged in the idle stages (blocks of 32 rows of NT
  // columns, 16-byte chunk c of row r at c ^ (r & CX)), then written back as whole row
  // segments; PB blocks at a time ----
  constexpr int BPS = (RF + SW) / SW;             // blocks per stage
  constexpr int PB = BPS * NS < RF ? BPS * NS : RF;
  constexpr int RC = EPI == EPI_SWIGLU ? NT / 8 : NT / 4;  // 16-byte chunks per staged row that are used
  constexpr int CX = SW == 4 ? 15 : (EPI == EPI_SWIGLU ? 3 : 7);  // keeps a chunk inside its row
  static_assert((RC & CX) == 0 || RC % (CX + 1) == 0, "swizzle stays in the row");
  auto block = [&](int b) -> uint8_t* {
    const int s = b / BPS;
    u32x4_t* p = s == 0 ? S0 : S1;
    if constexpr (NS > 2) p = s == 2 ? S2 : p;
    if constexpr (NS > 3) p = s == 3 ? S3 : p;
    if constexpr (NS > 4) p = s == 4 ? S4 : p;
    if constexpr (NS > 5) p = s == 5 ? S5 : p;
    return (uint8_t*)p + (b % BPS) * (SW * 4096);
  };
#pragma unroll
  for (int p0 = 0; p0 < RF; p0 += PB) {
    const int nb = RF - p0 < PB ? RF - p0 : PB;
    if (p0 > 0) __syncthreads();  // the previous blocks have been written back
#pragma unroll
    for (int i = 0; i < PB; ++i) {
      if (i >= nb) continue;
      uint8_t* st = block(i) + fr * (NT * 4);
      if (EPI == EPI_SWIGLU) {  // gate of a feature in acc[..][e], up in acc[..][e + 8]
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          float v[4];
#pragma unroll
          for (int t = 0; t < 4; ++t) v[t] = silu_mul(acc[p0 + i][4 * q + t], acc[p0 + i][8 + 4 * q + t]);
          *reinterpret_cast<float4*>(st + (((wave * 4 + 2 * q + fk) ^ (fr & CX)) << 4)) =
              make_float4(v[0], v[1], v[2], v[3]);
        }
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q)
          *reinterpret_cast<float4*>(st + (((wave * 8 + 2 * q + fk) ^ (fr & CX)) << 4)) = make_float4(
              acc[p0 + i][4 * q], acc[p0 + i][4 * q + 1], acc[p0 + i][4 * q + 2], acc[p0 + i][4 * q + 3]);
      }
    }
    __syncthreads();
    const int mp = m0 + p0 * 32;  // first row of this pass
    if constexpr (EPI == EPI_LSE) {
      // two threads per row, each over its half of every 8 columns in the order (and with
      // the arithmetic) of the 256x256 kernel: the same partials bit for bit
      constexpr float kL2e = 1.4426950408889634f;
      for (int u = tid; u < nb * 64; u += SW * 64) {
        const int row = u >> 1, hf = u & 1, m = mp + row;
        const uint8_t* st = block(row >> 5) + (row & 31) * 512;
        const int c0 = tn * NT + 4 * hf;
        const int id = min(max(g.lse.ids[min(m, g.M - 1)], 0), g.n_all - 1) - g.n_off;
        float mx = -INFINITY;
#pragma unroll 4
        for (int q = 0; q < 16; ++q) {
          const float4 v = *reinterpret_cast<const float4*>(st + (((2 * q + hf) ^ (row & 15)) << 4));
          const float x[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (c0 + 8 * q + e < g.N) mx = fmaxf(mx, x[e]);
        }
        mx = fmaxf(mx, __shfl_xor(mx, 1, kWave));
        const float ms = mx * kL2e;
        float sum = 0.f;
#pragma unroll 4
        for (int q = 0; q < 16; ++q) {
          const float4 v = *reinterpret_cast<const float4*>(st + (((2 * q + hf) ^ (row & 15)) << 4));
          const float x[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int col = c0 + 8 * q + e;
            if (col < g.N) sum += exp2f(fmaf(x[e], kL2e, -ms));
            if (col == id && m < g.M) g.lse.tgt[m] = x[e];
          }
        }
        sum += __shfl_xor(sum, 1, kWave);
        if (hf == 0 && m < g.M)
          *reinterpret_cast<float2*>(g.lse.lse + ((int64_t)m * g.n_part + g.n_off / 128 + tn) * 2) = make_float2(ms, sum);
      }
    } else if constexpr (EPI == EPI_SWIGLU) {
      const bool vec = (g.ldc & 3) == 0 && ((uintptr_t)g.C & 7) == 0;
#pragma unroll 4
      for (int u = tid; u < nb * 32 * RC; u += SW * 64) {  // 4 features (8 bytes) per thread
        const int r = u / RC, k = u % RC, m = mp + r;
        const float4 v =
            *reinterpret_cast<const float4*>(block(r >> 5) + (r & 31) * (NT * 4) + ((k ^ (r & CX)) << 4));
        const float x[4] = {v.x, v.y, v.z, v.w};
        if (m < g.M) store4h((T16*)g.C + (int64_t)m * g.ldc, tn * (NT / 2) + 4 * k, g.N, x, vec);
      }
    } else if constexpr (SW == 4) {
      const F32Out out = f32_out<EPI>(g);
      for (int h = wave; h < 2 * nb; h += SW)  // 16-row units, spread over the waves
        store_rows<EPI, T16, 1>(g, out, block(h >> 1), mp + (h >> 1) * 32, tn * NT, lane, h & 1);
    } else {
      const F32Out out = f32_out<EPI>(g);
#pragma unroll 4
      for (int u = tid; u < nb * 32 * RC; u += SW * 64) {
        const int r = u / RC, k = u % RC, m = mp + r;
        const float4 v =
            *reinterpret_cast<const float4*>(block(r >> 5) + (r & 31) * (NT * 4) + ((k ^ (r & CX)) << 4));
        const float x[4] = {v.x, v.y, v.z, v.w};
        if (m < g.M) store4<EPI == EPI_ADD_F32>(out.p + (int64_t)m * out.ld, tn * NT + 4 * k, g.N, x, out.vec);
      }
    }
  }
#endif
}

// Which tile.  A compute unit keeps about 64 KB of copies in flight, whatever the number of
// stages, and a slab that comes from HBM is 1.0-1.5 us away: it fills its slabs at 55-65 GB/s
// (a probe with the copies alone, 128x128 tiles: 58 GB/s a unit with 112 and with 256 units
// busy, one to three slabs ahead; 97 when the operands sit in the Infinity Cache, 125 in
// L2).  So a tile costs its slabs' bytes at that rate, 66 ns for 32 rows of A or of B (some
// 15% more when all units copy), plus a fill and an epilogue that grow with the tile; a launch
// takes as many rounds of 256 tiles, the last one by what it holds; and no launch is faster
// than its weights and outputs at 5 TB/s.  The 256x256 kernel moves the fewest bytes per
// product (1.2-1.45 us a slab, 12 us a tile) and wins when its rounds are full; a tenth of
// margin keeps it where the model cannot tell.  Measured, 7B shapes, us, 256x256 / the tile
// picked here: down projection of 470 rows 342 / 116 (64 rows by 128), of 800 340 / 142
// (128 by 128), of 1641 345 / 249 (256 by 128), of 2500 360 / 340 (160 by 128, two workgroups
// a unit); gate/up of 48 rows 80 / 52 (64 by 160: 237 tiles, one round), of 130 rows 88 / 64
// (160 by 160), of 470 163 / 142 and of 800 255 / 218 (160 by 128, two a unit); q/k/v of 470
// rows 80 / 40; lm_head of 130 rows 252 / 234, of 300 485 / 425; q/k/v of a decode step of 160
// rows in 14 splits 22 / 20.  At 1024 rows the gate/up (258 against 288) and at 600 the
// lm_head (652 / 770) stay there.
// Partials of few rows take 64 by 64 where 128 columns give too few workgroups: 48 rows, with
// timing events, 128 / 64 columns: down in 4 splits (112 / 224 workgroups) 47 / 37, q/k/v in 3
// 17 / 13, o 15 / 13.
struct FlexTile {
  int RF, SW, NS;
};
constexpr FlexTile kFlexTiles[] = {{2, 4, 6}, {4, 4, 5}, {5, 4, 4}, {5, 4, 2}, {8, 4, 3}, {2, 5, 5},
                                   {4, 5, 4}, {5, 5, 4}, {2, 2, 6}};

static int flex_cols(const GemmArgs& g, int epi, int SW) {
  return epi == EPI_SWIGLU ? (g.N + 16 * SW - 1) / (16 * SW)
                           : epi == EPI_LSE ? (g.N + 255) / 256 * 2 : (g.N + 32 * SW - 1) / (32 * SW);
}

// Time in ns that HBM takes for B and the output, which no tile avoids.
double gemm_hbm_floor(const GemmArgs& g, int epi, int splitk) {
  const double out = (double)g.M * g.N;
  const double bytes = 2. * g.K * g.N * (epi == EPI_SWIGLU ? 2. : 1.) +
                       (epi == -1 ? 5. * splitk * out : epi == EPI_SWIGLU || epi == EPI_ROPE ? 2. * out : epi == EPI_LSE ? 0. : 4. * out);
  return bytes / 5000.;
}

double gemm_cost_256(const GemmArgs& g, int epi, int splitk) {
  const int64_t tiles = (int64_t)((g.M + 255) / 256) * (epi == EPI_SWIGLU ? (g.N + 127) / 128 : (g.N + 255) / 256) * splitk;
  const double kt = g.k_chunk / GB_K, full = (double)(tiles / 256), rem = (double)(tiles % 256);
  const double t = full * (kt * 1426. + 12000.) + (rem > 0 ? kt * (1170. + rem) + 12000. : 0.);
  return std::max(t, gemm_hbm_floor(g, epi, splitk));
}

static int flex_pick(const GemmArgs& g, int epi, int splitk, double* best) {
  const double kt = g.k_chunk / GB_K, floor = gemm_hbm_floor(g, epi, splitk);
  int pick = 0;
  double least = 1e30;
  for (int i = 0; i < (int)(sizeof kFlexTiles / sizeof kFlexTiles[0]); ++i) {
    const FlexTile& f = kFlexTiles[i];
    if (f.SW == 5 && epi != EPI_SWIGLU) continue;
    if (f.SW == 2 && (epi != -1 || g.B.trans)) continue;
    if (g.k_sum && f.RF > 2) continue;
    const int64_t tiles = (int64_t)((g.M + 32 * f.RF - 1) / (32 * f.RF)) * flex_cols(g, epi, f.SW) * splitk;
    const double full = (double)(tiles / 256), rem = (double)(tiles % 256);
    double t;
    if (f.NS == 2) {
      // two workgroups a unit: pays where most units have both; beyond a few rounds they drift
      // apart and the launch ends evenly
      if (tiles <= 256) continue;
      const double rounds = tiles < 2048 ? 2. * (double)((tiles + 511) / 512) : tiles / 256. + 0.1;
      t = rounds * (kt * 580. + 4300.);
    } else {
      double slab = 66. * (f.RF + f.SW), tile = 2000. + 215. * f.RF * f.SW;
      if (f.SW == 5) slab = std::max(slab, 170. * f.RF);  // five waves on four SIMDs: the MFMAs of two
      t = full * (kt * slab * 1.05 + tile) + (rem > 0 ? kt * slab * (0.9 + 0.15 * rem / 256.) + tile : 0.);
    }
    if (t < least) {
      least = t;
      pick = i;
    }
  }
  *best = std::max(least, floor);
  return pick;
}

double gemm_cost_flex(const GemmArgs& g, int epi, int splitk) {
  double c;
  flex_pick(g, epi, splitk, &c);
  return c;
}

template <typename T16, int RF, int SW, int NS>
static void launch_flex_t(hipStream_t s, int epi, GemmArgs g, int splitk) {
  g.tiles_m = (g.M + 32 * RF - 1) / (32 * RF);
  g.tiles_n = flex_cols(g, epi, SW);
  const dim3 grid(g.tiles_m * g.tiles_n, splitk);
  if constexpr (SW == 2) {
    k_gemm_flex<-1, T16, RF, SW, NS><<<grid, SW * 64, 0, s>>>(g);
    return;
  }
  if constexpr (RF == 2 && SW != 2)
    if (g.k_sum) {
      k_gemm_flex<EPI_SWIGLU, T16, RF, SW, NS, false, true><<<grid, SW * 64, 0, s>>>(g);
      return;
    }
  if constexpr (SW == 5) {
    k_gemm_flex<EPI_SWIGLU, T16, RF, SW, NS><<<grid, SW * 64, 0, s>>>(g);
  } else if constexpr (SW == 4) {
    if (g.B.trans && epi == -1)
      k_gemm_flex<-1, T16, RF, SW, NS, true><<<grid, SW * 64, 0, s>>>(g);
    else if (g.B.trans)
      k_gemm_flex<EPI_ADD_F32, T16, RF, SW, NS, true><<<grid, SW * 64, 0, s>>>(g);
    else if (epi == -1)
      k_gemm_flex<-1, T16, RF, SW, NS><<<grid, SW * 64, 0, s>>>(g);
    else if (epi == EPI_STORE_F32)
      k_gemm_flex<EPI_STORE_F32, T16, RF, SW, NS><<<grid, SW * 64, 0, s>>>(g);
    else if (epi == EPI_SWIGLU)
      k_gemm_flex<EPI_SWIGLU, T16, RF, SW, NS><<<grid, SW * 64, 0, s>>>(g);
    else if (epi == EPI_LSE)
      k_gemm_flex<EPI_LSE, T16, RF, SW, NS><<<grid, SW * 64, 0, s>>>(g);
    else if (epi == EPI_ROPE)
      k_gemm_flex<EPI_ROPE, T16, RF, SW, NS><<<grid, SW * 64, 0, s>>>(g);
    else
      k_gemm_flex<EPI_ADD_F32, T16, RF, SW, NS><<<grid, SW * 64, 0, s>>>(g);
  }
}

int gemm_flex_tile(const GemmArgs& g, int epi, int splitk) {
  double cost;
  const FlexTile& f = kFlexTiles[flex_pick(g, epi, splitk, &cost)];
  return 100 * f.RF + 10 * f.SW + f.NS;
}

hipError_t launch_flex_gemm(hipStream_t s, rp_dtype dt, int epi, const GemmArgs& g, int splitk) {
  double cost;
  const int pick = flex_pick(g, epi, splitk, &cost);
  with_half16(dt, [&](auto tag_) {
    using H = decltype(tag_);
    switch (pick) {
      case 0: launch_flex_t<H, 2, 4, 6>(s, epi, g, splitk); break;
      case 1: launch_flex_t<H, 4, 4, 5>(s, epi, g, splitk); break;
      case 2: launch_flex_t<H, 5, 4, 4>(s, epi, g, splitk); break;
      case 3: launch_flex_t<H, 5, 4, 2>(s, epi, g, splitk); break;
      case 4: launch_flex_t<H, 8, 4, 3>(s, epi, g, splitk); break;
      case 5: launch_flex_t<H, 2, 5, 5>(s, epi, g, splitk); break;
      case 6: launch_flex_t<H, 4, 5, 4>(s, epi, g, splitk); break;
      case 7: launch_flex_t<H, 5, 5, 4>(s, epi, g, splitk); break;
      default: launch_flex_t<H, 2, 2, 6>(s, epi, g, splitk); break;
    }
  });
  return hipGetLastError();
}

}  // namespace rp
