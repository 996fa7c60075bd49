// What the GEMM kernels share: arguments, tile order, LDS swizzle, epilogue stores.
#pragma once

#include "device_common.h"
#include "rp_internal.h"

namespace rp {

constexpr int GB_K = 64;  // k slab of the 16-bit kernels

struct GemmArgs {
  int M, N, K;
  const void* A;
  int lda;
  BSeg B;
  int ldb;
  void* C;
  int ldc;
  int tiles_m, tiles_n;
  int k_chunk;       // K range per split (multiple of the k slab)
  float* partials;   // split-K: [splitk][M][N] fp32
  LseOut lse;        // EPI_LSE outputs
  int n_part;        // EPI_LSE column blocks per row
  RopeOut rope;      // EPI_ROPE outputs
  int n_off = 0;     // first logical column: a launch may take columns n_off .. n_off + N - 1 of B
  int n_all = 0;     // EPI_LSE: columns of the whole product
  int k_sum = 0;     // EPI_SWIGLU, at most 64 rows: K summed in chunks of k_sum (0: one chain)
};

template <typename T>
__device__ __forceinline__ const T* brow(const BSeg& b, int n, int ldb) {
  if (n < b.n1) return (const T*)b.b0 + (int64_t)n * ldb;
  if (n < b.n2) return (const T*)b.b1 + (int64_t)(n - b.n1) * ldb;
  return (const T*)b.b2 + (int64_t)(n - b.n2) * ldb;
}

__device__ __forceinline__ void tile_coords(int t, int tiles_m, int tiles_n, int* tm, int* tn) {
  constexpr int G = 8;
  const int per_group = G * tiles_n;
  const int group = t / per_group;
  const int first_m = group * G;
  const int gsize = min(tiles_m - first_m, G);
  const int in = t - group * per_group;
  *tm = first_m + in % gsize;
  *tn = in / gsize;
}

// Physical 16-byte chunk of logical chunk c in LDS row r is c ^ swz(r).
__device__ __forceinline__ int swz(int r) { return (r & 7) ^ ((r >> 3) & 1); }

__device__ __forceinline__ float silu_mul(float g, float u) { return g / (1.0f + expf(-g)) * u; }

// Four consecutive outputs n0..n0+3 of one row: one 8-byte (bf16) or 16-byte (fp32)
// access when the row is aligned for it and the four columns are all inside [0, N).
template <typename T16>
__device__ __forceinline__ void store4h(T16* row, int n0, int N, const float (&v)[4], bool vec) {
  if (vec && n0 + 3 < N) {
    *reinterpret_cast<uint2*>(row + n0) =
        make_uint2(Half16<T16>::pack2(v[0], v[1]), Half16<T16>::pack2(v[2], v[3]));
  } else {
#pragma unroll
    for (int t = 0; t < 4; ++t)
      if (n0 + t < N) stf(row + n0 + t, v[t]);
  }
}
template <bool ADD>
__device__ __forceinline__ void store4(float* row, int n0, int N, const float (&v)[4], bool vec) {
  if (vec && n0 + 3 < N) {
    float4* p = reinterpret_cast<float4*>(row + n0);
    float4 o = ADD ? *p : make_float4(0.f, 0.f, 0.f, 0.f);
    o.x += v[0];
    o.y += v[1];
    o.z += v[2];
    o.w += v[3];
    *p = o;
  } else {
#pragma unroll
    for (int t = 0; t < 4; ++t)
      if (n0 + t < N) row[n0 + t] = ADD ? row[n0 + t] + v[t] : v[t];
  }
}

#ifndef RP_GEMM_NT_STORE
#define RP_GEMM_NT_STORE 1
#endif
// 16-byte global store of the epilogue.  Outputs that no later step of the kernel reads
// (16-bit stores, fp32 stores) are written non-temporally, so that they do not evict the
// A/B slab lines the other workgroups of the XCD are still reading from L2; residual and
// split-K outputs, re-read soon, are stored normally.
template <bool NT>
__device__ __forceinline__ void st_out16(void* p, uint4 v) {
  if (NT && RP_GEMM_NT_STORE) {
    typedef uint32_t u4_t __attribute__((ext_vector_type(4)));
    u4_t w = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(w, reinterpret_cast<u4_t*>(p));
  } else {
    *reinterpret_cast<uint4*>(p) = v;
  }
}
template <bool NT>
__device__ __forceinline__ void st_out16(float* p, float4 v) {
  st_out16<NT>((void*)p, make_uint4(__float_as_uint(v.x), __float_as_uint(v.y), __float_as_uint(v.z), __float_as_uint(v.w)));
}


// Destination of a GEMM's fp32 rows: C, or this split's plane of the partials (EPI -1).
struct F32Out {
  float* p;
  int64_t ld;
  bool vec;  // rows start 16-byte aligned
};
template <int EPI>
__device__ __forceinline__ F32Out f32_out(const GemmArgs& g) {
  if (EPI == -1)
    return F32Out{g.partials + (int64_t)blockIdx.y * g.M * g.N, g.N, (g.N & 3) == 0 && ((uintptr_t)g.partials & 15) == 0};
  return F32Out{(float*)g.C, g.ldc, (g.ldc & 3) == 0 && ((uintptr_t)g.C & 15) == 0};
}

// Write back a staged block of fp32 rows: row r of `stage` (512 bytes, 128 columns from
// ncol0; 16-byte chunk c of it at c ^ (r & 15)) is output row m0 + r.  One wave takes the
// 16 * NB rows 16 * hb0 ..; 32 lanes hold one row, so every access is a whole row segment.
template <int EPI, typename T16, int NB>
__device__ __forceinline__ void store_rows(const GemmArgs& g, const F32Out& out, const uint8_t* stage, int m0,
                                           int ncol0, int lane, int hb0) {
  const int k = lane & 31;
  if (EPI == EPI_ROPE) {
    // q/k/v projection: the lane's 4 columns lie in one head (D divides 128), their
    // rotate-half partners D/2 columns away in the same staged row
    const RopeOut& ro = g.rope;
    const int half = ro.D >> 1;
    const int c = ncol0 + 4 * k + g.n_off;
    if (c - g.n_off < g.N) {
      const int seg = c < ro.hq ? 0 : c < ro.hq + ro.hkv ? 1 : 2;
      const int cc = seg == 0 ? c : seg == 1 ? c - ro.hq : c - ro.hq - ro.hkv;  // column in its segment
      const int64_t ld = seg == 0 ? ro.hq : ro.hkv;
      T16* dst0 = (T16*)(seg == 0 ? ro.q : seg == 1 ? ro.k : ro.v) + cc;
      const T16* bias = (const T16*)(seg == 0 ? ro.bq : seg == 1 ? ro.bk : ro.bv);
      const bool second = (cc & half) != 0;
      const int pair = cc & (half - 1);
      const int kp = k ^ (half >> 2);
      float bo[4] = {0.f, 0.f, 0.f, 0.f}, bp[4] = {0.f, 0.f, 0.f, 0.f};
      if (bias) {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          bo[t] = ldf(bias + cc + t);
          bp[t] = ldf(bias + (cc ^ half) + t);
        }
      }
#pragma unroll 4
      for (int sr = 0; sr < 8 * NB; ++sr) {
        const int r = 2 * (8 * hb0 + sr) + (lane >> 5);
        const int m = m0 + r;
        if (m >= g.M) continue;
        const float4 v = *reinterpret_cast<const float4*>(stage + r * 512 + ((k ^ (r & 15)) << 4));
        const float4 w = *reinterpret_cast<const float4*>(stage + r * 512 + ((kp ^ (r & 15)) << 4));
        const float x[4] = {v.x + bo[0], v.y + bo[1], v.z + bo[2], v.w + bo[3]};
        const float xp[4] = {w.x + bp[0], w.y + bp[1], w.z + bp[2], w.w + bp[3]};
        float y[4];
        if (seg == 2) {
#pragma unroll
          for (int t = 0; t < 4; ++t) y[t] = x[t];
        } else {
          const float4* tp = reinterpret_cast<const float4*>(ro.cs + (int64_t)m * half + pair);
          const float4 t0 = tp[0], t1 = tp[1];
          const float co[4] = {t0.x, t0.z, t1.x, t1.z}, si[4] = {t0.y, t0.w, t1.y, t1.w};
          float unused;
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            if (second)
              rope_rotate(xp[t], x[t], co[t], si[t], &unused, &y[t]);
            else
              rope_rotate(x[t], xp[t], co[t], si[t], &y[t], &unused);
          }
        }
        store4(dst0 + m * ld, y);
      }
    }
    return;
  }
  if (out.vec && ncol0 + 128 <= g.N) {
    // every column is in range: read the staged rows, then (residual) the matching rows of
    // C at once, then add and store; rows past M are clamped for the read and skipped for
    // the store; batches of 8 rows keep the staged values and C within the register budget
#pragma unroll
    for (int hb = 0; hb < NB; ++hb) {
      float4 v[8], c[8];
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        const int r = 2 * ((hb0 + hb) * 8 + s) + (lane >> 5);
        v[s] = *reinterpret_cast<const float4*>(stage + r * 512 + ((k ^ (r & 15)) << 4));
      }
      if (EPI == EPI_ADD_F32) {
#pragma unroll
        for (int s = 0; s < 8; ++s) {
          const int m = min(m0 + 2 * ((hb0 + hb) * 8 + s) + (lane >> 5), g.M - 1);
          c[s] = *reinterpret_cast<const float4*>(out.p + (int64_t)m * out.ld + ncol0 + k * 4);
        }
      }
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        const int m = m0 + 2 * ((hb0 + hb) * 8 + s) + (lane >> 5);
        float4 o = v[s];
        if (EPI == EPI_ADD_F32) {
          o.x += c[s].x;
          o.y += c[s].y;
          o.z += c[s].z;
          o.w += c[s].w;
        }
        if (m < g.M) st_out16<EPI == EPI_STORE_F32>(out.p + (int64_t)m * out.ld + ncol0 + k * 4, o);
      }
    }
    return;
  }
#pragma unroll
  for (int s = 0; s < 8 * NB; ++s) {
    const int r = 2 * (8 * hb0 + s) + (lane >> 5);
    const float4 v = *reinterpret_cast<const float4*>(stage + r * 512 + ((k ^ (r & 15)) << 4));
    const int m = m0 + r, n = ncol0 + k * 4;
    if (m >= g.M) continue;
    float* dst = out.p + (int64_t)m * out.ld + n;
    if (out.vec && n + 3 < g.N) {
      float4 o = v;
      if (EPI == EPI_ADD_F32) {
        const float4 c = *reinterpret_cast<const float4*>(dst);
        o.x += c.x;
        o.y += c.y;
        o.z += c.z;
        o.w += c.w;
      }
      st_out16<EPI == EPI_STORE_F32>(dst, o);
    } else {
      const float w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (n + e < g.N) dst[e] = EPI == EPI_ADD_F32 ? dst[e] + w[e] : w[e];
    }
  }
}

// GEMM over small tiles (gemm_flex.hip): the cost in ns of the best tile (and of the
// 256x256 kernel), by which the dispatch picks; the time that HBM takes for B and the output; the
// best tile as 100 RF + 10 SW + NS.
double gemm_hbm_floor(const GemmArgs& g, int epi, int splitk);
int gemm_flex_tile(const GemmArgs& g, int epi, int splitk);
double gemm_cost_256(const GemmArgs& g, int epi, int splitk);
double gemm_cost_flex(const GemmArgs& g, int epi, int splitk);
hipError_t launch_flex_gemm(hipStream_t s, rp_dtype dt, int epi, const GemmArgs& g, int splitk);

}  // namespace rp
