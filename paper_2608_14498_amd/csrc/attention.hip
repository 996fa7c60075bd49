// Attention kernels.
//
// One kernel serves both passes.  For sequence b the key space is the
// concatenation of segment 0 (the prefix KV rows, positions 0..n0-1; empty in the
// prefix pass) and segment 1 (the rows of the queries themselves, positions
// n0..), so a key's index in that space IS its position and the causal rule is
// "key index <= query position" everywhere: the prefix pass is causal attention
// over the prompt, the suffix pass sees every prefix key plus the causal block of
// its own response.
//
// bf16 (MFMA): a workgroup owns 4 waves x QW x 32 queries of one q head.  Each
// 64-key tile is staged in LDS (K row-major, V transposed); the wave computes
// S^T = K Q^T with v_mfma_f32_32x32x16_bf16 so that every lane holds the scores of
// ONE query (its softmax row statistics stay in-lane), then O^T += V^T P^T reusing
// the score registers, converted to bf16, directly as the B operand.  K/V tile loads
// for tile t+1 are in flight while tile t is computed (double-buffered LDS).
//
// fp32: the same tiles on the fp32 matrix cores, keys split over the waves of a workgroup.
//
// decode: split-KV over 1024-key chunks, all q heads of a kv head per wave,
// then a merge over chunks.
#include "device_common.h"
#include "rp_internal.h"

#include <math.h>

#include <type_traits>

namespace rp {

struct QBlock {
  int b, r_begin, r_end;  // rows of this block: P per query of sequence b, from its first query on
};

// Linear q-block index -> (sequence, block); blocks of a sequence are visited
// last-first (the longest causal rows start first).  P rows per query.
__device__ __forceinline__ QBlock find_qblock(const SeqTable& st, int qbl, int BQ, int P) {
  for (int b = 0; b < st.n; ++b) {
    const int nr = (st.q_cu[b + 1] - st.q_cu[b]) * P;
    const int nb = (nr + BQ - 1) / BQ;
    if (qbl < nb) {
      const int qb = nb - 1 - qbl;
      QBlock r;
      r.b = b;
      r.r_begin = qb * BQ;
      r.r_end = min(nr, r.r_begin + BQ);
      return r;
    }
    qbl -= nb;
  }
  QBlock r;
  r.b = -1;
  r.r_begin = r.r_end = 0;
  return r;
}

// ------------------------------------------------------------------------------------
// bf16 / fp16 MFMA flash attention
//
// K and V tiles are staged row-major in LDS ([key][Dh], 16-byte chunks, per-operand XOR
// swizzle) by direct global->LDS loads (buffer_load ... lds): one load instruction fills
// 64 consecutive chunks, and the swizzle is applied by choosing which global chunk each
// lane fetches.  The two LDS buffers are separate arrays and the tile loop is unrolled
// by two, so every LDS access names its buffer at compile time and the compiler waits
// on exactly the loads that filled it.  Each key segment of the sequence is one buffer
// resource whose extent ends at the segment's last row: rows past the end read as
// zeros (keys that the causal mask removes, with zero values), so no index is clamped.
//
// S^T = K Q^T reads K fragments with ds_read_b128.  The V^T operand of O^T += V^T P^T
// is read with ds_read_b64_tr_b16: within a 16-lane group, lane i receives column i%4
// of the 8-byte chunks addressed by lanes i/4, i/4+4, i/4+8, i/4+12, so lane p
// addressing V[k0 + p/4][d0 + 4(p%4)] hands lane i the four keys k0..k0+3 of head
// dimension d0+i -- the MFMA operand, with no transposed copy of V.
//
// LONG (queries over a long first key segment: the suffix pass, the last rows of a prefix):
//  - the rows of a block are (query, q head of one kv head) pairs, so that 48 responses'
//    tokens of a 7-head group are 336 rows in 3 blocks, not 7 blocks of 48;
//  - the sequence's keys are cut into attn_chunks() chunks with a softmax of their own, merged
//    in order by fa_merge_weights.  A workgroup takes one chunk and leaves its partial to
//    k_attn_split_merge, or all of them, merged in registers (attn_long_plan).  Both give the
//    same bits, so the launch may choose by the whole batch.
// A layer's attention, 7B shapes, us with timing events, before / now: 48 queries over 1501
// keys 36 / 23, the last rows of 1200, 2048 and 3001 keys (fp16) 63 / 24, both bound by a few
// key tiles in a row and two launches; 4 x 256 over 4096 99 / 99, 16 responses of 64 .. 1000
// over 4096 and 8190 keys 692 / 692 (890 TFLOP/s).  Waves without a row compute all the same:
// a branch round them cost the full blocks 2 to 5%.
// ------------------------------------------------------------------------------------
// Block -> (q block, q head), XCD-aware.  Workgroup i runs on XCD i % 8, which has its
// own L2, so the q heads that share a kv head (one GQA group, reading the same K/V
// tiles) are kept on one XCD: with Hkv dividing 8, each group gets 8/Hkv XCDs that take
// its (q block, head) items in turn; with Hkv a multiple of 8, XCD x gets the groups
// g = x mod 8.  Items run q-block-major, longest q blocks first.  Other head counts use
// the plain order.  Returns the grid size; blocks past the work map to q blocks
// beyond the last (find_qblock reports none).
struct FaMap {
  int mode, G, X;  // mode 0: plain, 1: 8/Hkv XCDs per group, 2: Hkv/8 groups per XCD
};
__host__ __device__ inline FaMap fa_map(int Hq, int Hkv) {
  FaMap m;
  m.G = Hq / Hkv;
  if (8 % Hkv == 0) {
    m.mode = 1;
    m.X = 8 / Hkv;
  } else if (Hkv % 8 == 0) {
    m.mode = 2;
    m.X = Hkv / 8;
  } else {
    m.mode = 0;
    m.X = 1;
  }
  return m;
}
inline int fa_grid(const FaMap& m, int nqb, int Hq) {
  if (m.mode == 1) return 8 * ((nqb * m.G + m.X - 1) / m.X);
  return nqb * Hq;
}
__device__ __forceinline__ void fa_block(const FaMap& m, int bid, int Hq, int* qbl, int* h) {
  const int x = bid & 7, r = bid >> 3;
  if (m.mode == 1) {
    const int i = r * m.X + x % m.X;
    *qbl = i / m.G;
    *h = (x / m.X) * m.G + i % m.G;
  } else if (m.mode == 2) {
    const int per = m.X * m.G;  // items of one q block on one XCD
    const int rem = r % per;
    *qbl = r / per;
    *h = ((rem / m.G) * 8 + x) * m.G + rem % m.G;
  } else {
    *qbl = bid / Hq;
    *h = bid % Hq;
  }
}

constexpr float kMaskVal = -1e30f;
constexpr float kLazy = 8.f;  // log2 headroom of the lazily updated softmax max
typedef __attribute__((address_space(3))) void lds_void_t;
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

// LDS chunk swizzles (16-byte chunks of a K or V row).  K rows are read 16 bytes per lane
// (row = key), so consecutive keys take distinct chunks.  V rows are read with
// ds_read_b64_tr_b16: in each 32-lane half, lane bits 0,1,4 pick the column within a
// 32-column block and bits 2,3 the key within a group of four; XOR-ing the key's low two
// bits into chunk bits 2,3 (D = 128: a row spans all 64 banks) or 1,2 (D = 64: two rows
// do, the key's bit 0 picking the half) makes the 32 lanes of a half hit 64 distinct
// banks.  (Chunk bits 1,2 at D = 128 left one bank bit fixed: half the banks, and the
// LDS bank-conflict counter at 14% of the prefix kernel's cycles.)
template <int D>
__device__ __forceinline__ int kswz(int key) { return D == 128 ? (key & 15) : (key & 7); }
template <int D>
__device__ __forceinline__ int vswz(int key) { return D == 128 ? (key & 3) << 2 : (key & 3) << 1; }

__device__ __forceinline__ void fa_merge_weights(float& M, float& L, float m, float l, float* wa, float* wb) {
  const float mn = fmaxf(M, m);
  *wa = __builtin_amdgcn_exp2f(M - mn);
  *wb = __builtin_amdgcn_exp2f(m - mn);
  L = fmaf(l, *wb, L * *wa);
  M = mn;
}

// kDense: a row per (query, head), one pass over the keys.  kLong: packed rows, one chunk of keys
// a workgroup (of those that have several).  kLongFold: packed rows, all chunks, merged here.
enum AttnForm { kDense, kLong, kLongFold };
template <typename T16, int D, int QW, int KT, int NW, AttnForm FORM>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(QW == 1 ? 2 : 1, QW == 1 ? 2 : 1)))
void k_attn_bf16(SeqTable st, AttnArgs a) {
#if defined(__HIP_DEVICE_COMPILE__)  // buffer resources exist only in the device pass
  typedef Half16<T16> H;
  typedef typename H::V8 V8;
  constexpr bool LONG = FORM != kDense, FOLD = FORM == kLongFold;
  constexpr int BQ = NW * 32 * QW;
  constexpr int CH = D / 8;               // 16-byte chunks per K/V row
  constexpr int KSTEPS = D / 16;          // MFMA k-steps of S^T (over Dh)
  constexpr int DB = D / 32;              // 32-row blocks of O^T
  constexpr int KB = KT / 32;             // 32-key blocks per tile
  constexpr int LOADS = (KT * CH) / (NW * 64);  // load instructions per wave per matrix
  static_assert(LOADS >= 1 && (KT * CH) % (NW * 64) == 0 && 64 % CH == 0, "tile loader");
  __shared__ u32x4_t Ks0[KT * CH], Ks1[KT * CH], Vs0[KT * CH], Vs1[KT * CH];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int h, qbl;
  const int G = a.Hq / a.Hkv, P = LONG ? G : 1;  // P rows per query; LONG: h is the kv head
  fa_block(fa_map(LONG ? a.Hkv : a.Hq, a.Hkv), blockIdx.x, LONG ? a.Hkv : a.Hq, &qbl, &h);
  QBlock qb = find_qblock(st, qbl, BQ, P);
  if (qb.b < 0) return;
  // Block-uniform values, moved to scalar registers (the sequence table is indexed
  // dynamically, which the compiler cannot prove uniform).
  const int b = __builtin_amdgcn_readfirstlane(qb.b);
  qb.r_begin = __builtin_amdgcn_readfirstlane(qb.r_begin);
  qb.r_end = __builtin_amdgcn_readfirstlane(qb.r_end);
  const int g = LONG ? h : h / G;
  const int krow0 = __builtin_amdgcn_readfirstlane(st.k_beg(b));
  const int n0 = __builtin_amdgcn_readfirstlane(st.pos0(b));
  const int qrow0 = __builtin_amdgcn_readfirstlane(st.q_cu[b]);
  const int nq = __builtin_amdgcn_readfirstlane(st.q_cu[b + 1]) - qrow0;
  const int qpos_first = n0 + qb.r_begin / P;
  const int qpos_last = n0 + (qb.r_end - 1) / P;
  // Key tiles: the first P0 tiles hold the n0 first-segment keys (the last of them may be
  // partial: its rows past n0 read as zeros and are masked), the rest the segment-1 keys
  // n0 .. qpos_last this block needs, from position n0 on.  No tile mixes the segments,
  // so each tile's copies name one buffer resource.  Tile t's first key position is
  // kpos0(t).
  const int P0 = (n0 + KT - 1) / KT;
  auto kpos0 = [&](int t) { return t < P0 ? t * KT : n0 + (t - P0) * KT; };
  // Tiles t_begin .. t_end-1 of this block.  LONG: chunk c of nch is the first-segment tiles
  // P0 c / nch .. P0 (c + 1) / nch (at least one each: a chunk is 256 keys or more), the last
  // chunk also the segment-1 tiles (the causal keys): it is the longest and runs at
  // blockIdx.y 0.
  int t_begin = 0, t_end = P0 + (qpos_last - n0 + KT) / KT, chunk = 0;
  const int nch = LONG ? attn_chunks(n0, nq, a.Hq, a.Hkv, a.most_chunks) : 1;
  const bool split = FORM == kLong && nch > 1;
  if (FORM == kLong && (int)blockIdx.y >= nch) return;
  auto chunk_end = [&](int c) { return c + 1 < nch ? P0 * (c + 1) / nch : t_end; };
  if (split) {
    chunk = nch - 1 - (int)blockIdx.y;
    t_begin = P0 * chunk / nch;
    t_end = chunk_end(chunk);
  }
  int fold_at = !FOLD || nch == 1 ? -1 : chunk_end(0);  // tile count at which a chunk is done

  // Key segments as buffer resources: segment 0 = the n0 prefix rows, segment 1 = the
  // nq rows of the queries; key kv of segment s is at byte (kv - start_s) * row_bytes.
  // The host guarantees those offsets, past-the-end tile rows included, fit 32 bits.
  const int64_t kv_ld = (int64_t)a.Hkv * D;
  const uint32_t row_bytes = (uint32_t)kv_ld * sizeof(T16);
  const uint32_t ext0 = n0 > 0 ? (uint32_t)(n0 - 1) * row_bytes + D * sizeof(T16) : 0u;
  const uint32_t ext1 = (uint32_t)(nq - 1) * row_bytes + D * sizeof(T16);
  const int64_t e0 = (int64_t)krow0 * kv_ld + (int64_t)g * D, e1 = (int64_t)qrow0 * kv_ld + (int64_t)g * D;
  // (64-bit products are formed in vector registers: uniform_ptr returns them to scalar
  // registers, where a buffer resource must live.)
  const __amdgpu_buffer_rsrc_t rsK0 =
      __builtin_amdgcn_make_buffer_rsrc(uniform_ptr((void*)((const T16*)a.k0 + e0)), 0, (int)ext0, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsV0 =
      __builtin_amdgcn_make_buffer_rsrc(uniform_ptr((void*)((const T16*)a.v0 + e0)), 0, (int)ext0, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsK1 =
      __builtin_amdgcn_make_buffer_rsrc(uniform_ptr((void*)((const T16*)a.k1 + e1)), 0, (int)ext1, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsV1 =
      __builtin_amdgcn_make_buffer_rsrc(uniform_ptr((void*)((const T16*)a.v1 + e1)), 0, (int)ext1, 0x00020000);

  // Load instruction j of this wave fills LDS chunks (wave*LOADS + j)*64 + lane, i.e.
  // tile key (wave*LOADS + j)*64/CH + lane/CH, physical chunk lane%CH, which holds
  // logical chunk (lane%CH) ^ swizzle(key).
  uint32_t koff[LOADS], voff[LOADS];
#pragma unroll
  for (int j = 0; j < LOADS; ++j) {
    const int slot = (wave * LOADS + j) * 64 + lane, key = slot / CH, cp = slot % CH;
    koff[j] = (uint32_t)key * row_bytes + (uint32_t)((cp ^ kswz<D>(key)) * 16);
    voff[j] = (uint32_t)key * row_bytes + (uint32_t)((cp ^ vswz<D>(key)) * 16);
  }
#define FA_DMA(RS_, OFF_, DST_, j_) \
  __builtin_amdgcn_raw_ptr_buffer_load_lds(RS_, (lds_void_t*)((DST_) + (wave * LOADS + (j_)) * 64), 16, OFF_, 0, 0, 0)
#define FA_LOAD_SEG(RK_, RV_, KD_, VD_, so_)            \
  _Pragma("unroll") for (int j = 0; j < LOADS; ++j) {   \
    FA_DMA(RK_, koff[j] + (so_), KD_, j);               \
    FA_DMA(RV_, voff[j] + (so_), VD_, j);               \
  }
  // Each (uniform) branch names its buffer resources (a selected resource would be formed
  // in vector registers); all offsets go in the range-checked vector offset (the scalar
  // offset is not range-checked).  Both branches issue the same copies, so the compiler
  // counts the outstanding ones exactly.
#define FA_LOAD(KD_, VD_, t_)                                                         \
  {                                                                                   \
    const int tt_ = __builtin_amdgcn_readfirstlane(t_);  /* uniform: scalar branch */ \
    if (tt_ < P0) {                                                                   \
      FA_LOAD_SEG(rsK0, rsV0, KD_, VD_, (uint32_t)(tt_ * KT) * row_bytes);            \
    } else {                                                                          \
      FA_LOAD_SEG(rsK1, rsV1, KD_, VD_, (uint32_t)((tt_ - P0) * KT) * row_bytes);     \
    }                                                                                 \
  }

  // ---- queries of this lane: column (lane & 31) of each 32-query block ----
  const int fr = lane & 31, fk = lane >> 5;
  V8 qf[QW][KSTEPS];
  int qpos[QW];
#pragma unroll
  for (int qi = 0; qi < QW; ++qi) {
    const int r_raw = qb.r_begin + (wave * QW + qi) * 32 + fr;
    const int r = min(r_raw, qb.r_end - 1), q = r / P;
    qpos[qi] = n0 + r_raw / P;
    const T16* qp = (const T16*)a.q + (int64_t)(qrow0 + q) * a.q_ld + (h * P + r - q * P) * D + fk * 8;
#pragma unroll
    for (int ks = 0; ks < KSTEPS; ++ks) qf[qi][ks] = H::as_v8(*reinterpret_cast<const uint4*>(qp + ks * 16));
  }

  f32x16_t o[QW][DB];
  float m_run[QW], l_run[QW];
#pragma unroll
  for (int qi = 0; qi < QW; ++qi) {
    m_run[qi] = kMaskVal;
    l_run[qi] = 0.f;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int e = 0; e < 16; ++e) o[qi][db][e] = 0.f;
  }
  // FOLD: the merged chunks so far
  f32x16_t ot[FOLD ? QW : 1][FOLD ? DB : 1];
  float m_tot[QW], l_tot[QW];
  if constexpr (FOLD) {
#pragma unroll
    for (int qi = 0; qi < QW; ++qi) {
      m_tot[qi] = kMaskVal;
      l_tot[qi] = 0.f;
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int e = 0; e < 16; ++e) ot[qi][db][e] = 0.f;
    }
  }
  auto fold = [&]() __attribute__((always_inline)) {
    if constexpr (FOLD) {
#pragma unroll
      for (int qi = 0; qi < QW; ++qi) {
        float wa, wb;
        fa_merge_weights(m_tot[qi], l_tot[qi], m_run[qi], l_run[qi] + __shfl_xor(l_run[qi], 32, kWave), &wa, &wb);
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
          for (int e = 0; e < 16; ++e) {
            ot[qi][db][e] = fmaf(o[qi][db][e], wb, ot[qi][db][e] * wa);
            o[qi][db][e] = 0.f;
          }
        m_run[qi] = kMaskVal;
        l_run[qi] = 0.f;
      }
      fold_at = chunk_end(++chunk);
    }
  };
  const float c2 = a.scale * 1.4426950408889634f;  // scores in log2 units
  // V^T fragment addressing (see header): 16-lane group -> d0, lane p = lane % 16
  const int tr_p = lane & 15;
  const int tr_key = fk * 4 + (tr_p >> 2);                     // + kb*32 + hh*16 (+8 for the second read)
  const int tr_col = ((lane & 16) ? 16 : 0) + 4 * (tr_p & 3);  // + db*32

  // One key tile computed from (Kc, Vc).
  auto compute = [&](const u32x4_t* Kc, const u32x4_t* Vc, int t) __attribute__((always_inline)) {
    // ---- S^T = K Q^T: s[qi][kb][e] = score(key t*KT + kb*32 + 8(e/4) + 4 fk + e%4, query fr) ----
    f32x16_t s[QW][KB];
#pragma unroll
    for (int ks = 0; ks < KSTEPS; ++ks) {
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) {
        const int key = kb * 32 + fr;
        const V8 kf = __builtin_bit_cast(V8, Kc[key * CH + ((ks * 2 + fk) ^ kswz<D>(key))]);
#pragma unroll
        for (int qi = 0; qi < QW; ++qi)
          s[qi][kb] = H::mma(kf, qf[qi][ks], ks == 0 ? f32x16_t{} : s[qi][kb]);
      }
    }

    // ---- mask (diagonal tiles only), online softmax per lane = per query ----
    // Scores stay raw until the exponent: p = 2^(s*c2 - m) with m in log2 units.  The
    // running max m is raised only when some lane's tile max exceeds it by more than
    // kLazy (wave-uniform test), so p <= 2^kLazy and the O^T rescale is skipped on most
    // tiles; numerator and denominator share the same m, so the result is unchanged.
    // masked: first-segment keys past n0 (the last first-segment tile only) and causal
    // keys past the query (segment-1 tiles that reach past the block's first query)
    const bool seg0 = t < P0;
    const bool need_mask = seg0 ? (t * KT + KT > n0) : (kpos0(t) + KT - 1 > qpos_first);
#pragma unroll
    for (int qi = 0; qi < QW; ++qi) {
      if (need_mask) {
        const int lim = (seg0 ? n0 - 1 : qpos[qi]) - kpos0(t) - 4 * fk;  // last visible offset - 4 fk
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
          for (int e = 0; e < 16; ++e)
            if (kb * 32 + 8 * (e >> 2) + (e & 3) > lim) s[qi][kb][e] = kMaskVal;
      }
      float mx = kMaskVal;
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int e = 0; e < 16; ++e) mx = fmaxf(mx, s[qi][kb][e]);
      mx = fmaxf(mx, __shfl_xor(mx, 32, kWave)) * c2;
      if (__any(mx > m_run[qi] + kLazy)) {
        const float m_new = fmaxf(m_run[qi], mx);
        const float alpha = __builtin_amdgcn_exp2f(m_run[qi] - m_new);
        m_run[qi] = m_new;
        l_run[qi] *= alpha;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
          for (int e = 0; e < 16; ++e) o[qi][db][e] *= alpha;
      }
      const float nm = -m_run[qi];
      float ls = 0.f;
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const float p = __builtin_amdgcn_exp2f(fmaf(s[qi][kb][e], c2, nm));
          s[qi][kb][e] = p;
          ls += p;
        }
      l_run[qi] += ls;
    }

    // ---- O^T += V^T P^T over the sixteen-key steps (kb, hh) ----
    const T16* vbase = reinterpret_cast<const T16*>(Vc);
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
#pragma unroll
      for (int hh = 0; hh < 2; ++hh) {
        V8 pf[QW];
#pragma unroll
        for (int qi = 0; qi < QW; ++qi) {
          const f32x16_t& sv = s[qi][kb];
          pf[qi] = H::as_v8(make_uint4(H::pack2(sv[hh * 8 + 0], sv[hh * 8 + 1]), H::pack2(sv[hh * 8 + 2], sv[hh * 8 + 3]),
                                       H::pack2(sv[hh * 8 + 4], sv[hh * 8 + 5]), H::pack2(sv[hh * 8 + 6], sv[hh * 8 + 7])));
        }
        const int ka = kb * 32 + hh * 16 + tr_key, kc = ka + 8;
#pragma unroll
        for (int db = 0; db < DB; ++db) {
          const int col = db * 32 + tr_col;
          const int ca = ((col >> 3) ^ vswz<D>(ka)) * 8 + (col & 7);
          const int cc = ((col >> 3) ^ vswz<D>(kc)) * 8 + (col & 7);
          const v4i16_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_t*)(vbase + ka * D + ca));
          const v4i16_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_t*)(vbase + kc * D + cc));
          const uint2 l2 = __builtin_bit_cast(uint2, lo), h2 = __builtin_bit_cast(uint2, hi);
          const V8 vf = H::as_v8(make_uint4(l2.x, l2.y, h2.x, h2.y));
#pragma unroll
          for (int qi = 0; qi < QW; ++qi) o[qi][db] = H::mma(vf, pf[qi], o[qi][db]);
        }
      }
    }
  };

  // Loads of tile t+1 into (Kn, Vn) are issued first and land while tile t is computed
  // from (Kc, Vc); the closing barrier (which waits for this wave's loads) makes them
  // visible to every wave.  (A third buffer with two tiles in flight and explicit
  // per-tile waits measured slower: 5.47 against 4.96 ms per layer at 2 x 16384 keys.)
  auto tile = [&](const u32x4_t* Kc, const u32x4_t* Vc, u32x4_t* Kn, u32x4_t* Vn, int t) __attribute__((always_inline)) {
    if (t + 1 < t_end) FA_LOAD(Kn, Vn, t + 1);
    compute(Kc, Vc, t);
    if (FOLD && t + 1 == fold_at) fold();
    __syncthreads();
  };
  FA_LOAD(Ks0, Vs0, t_begin);
  __syncthreads();
  int t = t_begin;
  for (; t + 2 <= t_end; t += 2) {
    tile(Ks0, Vs0, Ks1, Vs1, t);
    tile(Ks1, Vs1, Ks0, Vs0, t + 1);
  }
  if (t < t_end) tile(Ks0, Vs0, Ks1, Vs1, t);
#undef FA_DMA
#undef FA_LOAD_SEG
#undef FA_LOAD

  // ---- normalise and store: o[qi][db][e] = O^T(dh = db*32 + 8(e/4) + 4 fk + e%4, query fr) ----
  if (split) {  // partial of one chunk: (max in log2 units, sum, unnormalised o)
#pragma unroll
    for (int qi = 0; qi < QW; ++qi) {
      const int r = qb.r_begin + (wave * QW + qi) * 32 + fr, q = r / P;
      const float l = l_run[qi] + __shfl_xor(l_run[qi], 32, kWave);
      if (r >= qb.r_end) continue;
      float* pp = a.part + ((int64_t)(qrow0 + q) * a.Hq + h * P + r - q * P) * attn_part_record(gridDim.y, D);
      if (fk == 0) *reinterpret_cast<float2*>(pp + gridDim.y * D + 2 * chunk) = make_float2(m_run[qi], l);
      pp += chunk * D;
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int e4 = 0; e4 < 4; ++e4)
          *reinterpret_cast<float4*>(pp + db * 32 + 8 * e4 + 4 * fk) =
              make_float4(o[qi][db][4 * e4], o[qi][db][4 * e4 + 1], o[qi][db][4 * e4 + 2], o[qi][db][4 * e4 + 3]);
    }
    return;
  }
#pragma unroll
  for (int qi = 0; qi < QW; ++qi) {
    const int r = qb.r_begin + (wave * QW + qi) * 32 + fr, q = r / P;
    float l = l_run[qi] + __shfl_xor(l_run[qi], 32, kWave);
    if constexpr (FOLD) {
      if (nch > 1) l = l_tot[qi];  // (the last chunk was folded at t_end)
    }
    if (r >= qb.r_end) continue;
    const float inv = 1.0f / l;
    T16* op = (T16*)a.o + (int64_t)(qrow0 + q) * a.Hq * D + (h * P + r - q * P) * D;
#pragma unroll
    for (int db = 0; db < DB; ++db) {
      f32x16_t v = o[qi][db];
      if constexpr (FOLD) {
        if (nch > 1) v = ot[qi][db];
      }
#pragma unroll
      for (int e4 = 0; e4 < 4; ++e4) {
        const int dh = db * 32 + 8 * e4 + 4 * fk;
        uint2 w;
        w.x = H::pack2(v[4 * e4] * inv, v[4 * e4 + 1] * inv);
        w.y = H::pack2(v[4 * e4 + 2] * inv, v[4 * e4 + 3] * inv);
        *reinterpret_cast<uint2*>(op + dh) = w;
      }
    }
  }
#endif
}

// ------------------------------------------------------------------------------------
// fp32 attention on the fp32 matrix cores (v_mfma_f32_32x32x2: exact fp32 products).
// A workgroup owns 32 queries of one head; its NW waves take the 32-key tiles in turn and
// their (max, sum, o) are combined in LDS, so that also the few hundred queries of a small
// fp32 model fill the chip.  Per tile S^T = K Q^T (lane l holds query l % 32 and the head
// dimensions 8 j + 4 (l / 32) + 0..3, the same for K and Q: 16-byte loads straight from
// global memory), then O^T += V^T P^T with the scores as they are: score register e belongs
// to keys 8 (e/4) + e%4 (+ 4 in the upper half wave), which is the k pair of MFMA e.  The V
// values of a tile and the K rows of the wave's next one are in flight under the score
// MFMAs.  Bound by load latency at these sizes (2 x 512 queries, 4 heads of 64, launch and
// timing events included: 23 us a layer, where one thread per query walked the keys in 685;
// 2 x 64 queries over 512 + 64 keys: 24, from 784).  A split by tile index alone: a sequence's result does not depend on the batch.
// ------------------------------------------------------------------------------------
template <int D, int NW>
__global__ __launch_bounds__(NW * 64) void k_attn_f32(SeqTable st, AttnArgs a) {
  constexpr int BQ = 32, KT = 32, NC = D / 8, DB = D / 32;
  __shared__ float4 part[NW][DB * 4][64];  // unnormalised o of each wave: [quad][lane]
  __shared__ float2 ml[NW][64];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int fr = lane & 31, fk = lane >> 5;
  const int h = blockIdx.x % a.Hq;
  QBlock qb = find_qblock(st, blockIdx.x / a.Hq, BQ, 1);
  if (qb.b < 0) return;
  const int b = __builtin_amdgcn_readfirstlane(qb.b);
  qb.r_begin = __builtin_amdgcn_readfirstlane(qb.r_begin);
  qb.r_end = __builtin_amdgcn_readfirstlane(qb.r_end);
  const int g = h / (a.Hq / a.Hkv);
  const int n0 = __builtin_amdgcn_readfirstlane(st.pos0(b));
  const int qrow0 = __builtin_amdgcn_readfirstlane(st.q_cu[b]);
  const int krow0 = __builtin_amdgcn_readfirstlane(st.k_beg(b));
  const int qrow_raw = qrow0 + qb.r_begin + fr, qrow = min(qrow_raw, qrow0 + qb.r_end - 1);
  const int qi = qrow - qrow0;                     // this lane's query among its sequence's
  const int nk1 = qb.r_end;                        // segment-1 keys this block needs
  const int P0 = (n0 + KT - 1) / KT;               // no tile mixes the key segments
  const int ntiles = P0 + (nk1 + KT - 1) / KT;
  const int64_t kv_ld = (int64_t)a.Hkv * D;

  float4 q[NC];
  const float* qp = (const float*)a.q + (int64_t)qrow * a.q_ld + h * D + 4 * fk;
#pragma unroll
  for (int j = 0; j < NC; ++j) q[j] = *reinterpret_cast<const float4*>(qp + 8 * j);

  // first key row of tile t and the number of its keys that exist (rows past them re-read
  // the last one; their scores are masked)
  auto tile_rows = [&](int t, const float** k, const float** v, int* cnt) {
    const bool s0 = t < P0;
    const int first = s0 ? t * KT : (t - P0) * KT;
    const int64_t off = (int64_t)((s0 ? krow0 : qrow0) + first) * kv_ld + (int64_t)g * D;
    *k = (const float*)(s0 ? a.k0 : a.k1) + off;
    *v = (const float*)(s0 ? a.v0 : a.v1) + off;
    *cnt = min(KT, (s0 ? n0 : nk1) - first);
  };
  float4 kf[NC];
  auto load_k = [&](int t) {
    const float *k, *v;
    int cnt;
    tile_rows(t, &k, &v, &cnt);
    const float* kp = k + (int64_t)min(fr, cnt - 1) * kv_ld + 4 * fk;
#pragma unroll
    for (int j = 0; j < NC; ++j) kf[j] = *reinterpret_cast<const float4*>(kp + 8 * j);
  };
  f32x16_t o[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int e = 0; e < 16; ++e) o[db][e] = 0.f;
  // Lowest number, not -inf: a tile whose scores are all -inf must leave the weights numbers, and
  // its wave a sum of 0, where other waves hold the other keys.
  float m = -3.4028235e38f, l = 0.f;
  if (wave < ntiles) load_k(wave);
  for (int t = wave; t < ntiles; t += NW) {
    const float *kb, *vb;
    int cnt;
    tile_rows(t, &kb, &vb, &cnt);
    float vf[DB][16];
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const float* vp = vb + (int64_t)min(8 * (e >> 2) + 4 * fk + (e & 3), cnt - 1) * kv_ld + fr;
#pragma unroll
      for (int db = 0; db < DB; ++db) vf[db][e] = vp[db * 32];
    }
    f32x16_t s;
#pragma unroll
    for (int e = 0; e < 16; ++e) s[e] = 0.f;
#pragma unroll
    for (int j = 0; j < NC; ++j) {
      s = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[j].x, q[j].x, s, 0, 0, 0);
      s = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[j].y, q[j].y, s, 0, 0, 0);
      s = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[j].z, q[j].z, s, 0, 0, 0);
      s = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[j].w, q[j].w, s, 0, 0, 0);
    }
    if (t + NW < ntiles) load_k(t + NW);
    // s[e] = score(key 8 (e/4) + 4 fk + e%4 of the tile, query fr); last visible key of the tile:
    const int lim = (t < P0 ? cnt - 1 : min(cnt - 1, qi - (t - P0) * KT)) - 4 * fk;
    float mx = -INFINITY;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      s[e] = 8 * (e >> 2) + (e & 3) <= lim ? s[e] * a.scale : -INFINITY;
      mx = fmaxf(mx, s[e]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 32, kWave));
    const float mn = fmaxf(m, mx);  // every query sees a key of every tile its block visits
    const float alpha = expf(m - mn);
    m = mn;
    l *= alpha;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int e = 0; e < 16; ++e) o[db][e] *= alpha;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      s[e] = 8 * (e >> 2) + (e & 3) <= lim ? expf(s[e] - mn) : 0.f;
      l += s[e];
    }
    // A masked key's weight is 0, and 0 * inf would leak a non-finite value of a later token
    // into an earlier query: the causal tile of such values is added key by key instead.
    bool odd = false;
    if (t >= P0) {
#pragma unroll
      for (int e = 0; e < 16; ++e)
#pragma unroll
        for (int db = 0; db < DB; ++db) odd |= !(fabsf(vf[db][e]) <= 3.4028235e38f);
      odd = __any(odd);
    }
    if (!odd) {
#pragma unroll
      for (int e = 0; e < 16; ++e)
#pragma unroll
        for (int db = 0; db < DB; ++db) o[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(vf[db][e], s[e], o[db], 0, 0, 0);
    } else {
#pragma unroll
      for (int e = 0; e < 16; ++e)
        for (int f = 0; f < 2; ++f) {  // key 8 (e/4) + 4 f + e%4: its weight sits in half f
          const int key = 8 * (e >> 2) + 4 * f + (e & 3);
          const float pk = __shfl(s[e], fr + 32 * f, kWave);
          const bool seen = key - 4 * fk <= lim;
          const float* vp = vb + (int64_t)min(key, cnt - 1) * kv_ld;
#pragma unroll
          for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int c = 0; c < 16; ++c)
              if (seen) o[db][c] = fmaf(pk, vp[db * 32 + 8 * (c >> 2) + 4 * fk + (c & 3)], o[db][c]);
        }
    }
  }
  // ---- combine the waves: o[db][e] = O^T(dim db*32 + 8 (e/4) + 4 fk + e%4, query fr) ----
  l += __shfl_xor(l, 32, kWave);
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int c = 0; c < 4; ++c)
      part[wave][db * 4 + c][lane] = make_float4(o[db][4 * c], o[db][4 * c + 1], o[db][4 * c + 2], o[db][4 * c + 3]);
  ml[wave][lane] = make_float2(m, l);
  __syncthreads();
  float M = -INFINITY, L = 0.f, f[NW];
#pragma unroll
  for (int w = 0; w < NW; ++w) M = fmaxf(M, ml[w][lane].x);
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    f[w] = w < ntiles ? expf(ml[w][lane].x - M) : 0.f;
    L += ml[w][lane].y * f[w];
  }
  const float inv = 1.0f / L;
  if (qrow_raw >= qrow0 + qb.r_end) return;
  float* op = (float*)a.o + (int64_t)qrow * a.Hq * D + h * D + 4 * fk;
  for (int c = wave; c < DB * 4; c += NW) {
    float v[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      if (w >= ntiles) continue;
      const float4 x = part[w][c][lane];
      v[0] = fmaf(x.x, f[w], v[0]);
      v[1] = fmaf(x.y, f[w], v[1]);
      v[2] = fmaf(x.z, f[w], v[2]);
      v[3] = fmaf(x.w, f[w], v[3]);
    }
    *reinterpret_cast<float4*>(op + (c >> 2) * 32 + 8 * (c & 3)) =
        make_float4(v[0] * inv, v[1] * inv, v[2] * inv, v[3] * inv);
  }
}

// Merge of chunk partials: one wave per (query row, q head), lane i holding head dimensions
// i*D/64 ..; rows of sequences of one chunk were written by the attention kernel.  The o of
// chunk c of (row, head) is at (row*Hq + head) * attn_part_record(S, D) + c*D, its (max in log2
// units, sum) at S*D + 2c there.  The chunks are merged in order, as the attention kernel does
// when it takes them all.
template <typename T16, int D>
__global__ __launch_bounds__(256) void k_attn_split_merge(SeqTable st, const float* __restrict__ part, int S, int Hq,
                                                          int Hkv, int most, int64_t items, T16* __restrict__ o) {
  typedef Half16<T16> H;
  constexpr int PER = D / 64;
  const int64_t item = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (item >= items) return;
  const int lane = threadIdx.x & 63;
  const int b = seq_of_row(st, (int)(item / Hq));
  const int nch = attn_chunks(st.pos0(b), st.q_cu[b + 1] - st.q_cu[b], Hq, Hkv, most);
  if (nch == 1) return;
  const float* p = part + item * attn_part_record(S, D);
  const float* ml = p + S * D;
  float v[kAttnMaxSplits][PER], m[kAttnMaxSplits], l[kAttnMaxSplits];
#pragma unroll
  for (int c = 0; c < kAttnMaxSplits; ++c) {  // every load in flight at once
    const int cc = min(c, nch - 1);
    m[c] = ml[2 * cc];
    l[c] = ml[2 * cc + 1];
#pragma unroll
    for (int e = 0; e < PER; ++e) v[c][e] = p[cc * D + lane * PER + e];
  }
  float M = kMaskVal, L = 0.f, acc[PER];
#pragma unroll
  for (int e = 0; e < PER; ++e) acc[e] = 0.f;
#pragma unroll
  for (int c = 0; c < kAttnMaxSplits; ++c) {
    if (c >= nch) break;
    float wa, wb;
    fa_merge_weights(M, L, m[c], l[c], &wa, &wb);
#pragma unroll
    for (int e = 0; e < PER; ++e) acc[e] = fmaf(v[c][e], wb, acc[e] * wa);
  }
  const float inv = 1.0f / L;
  T16* op = o + item * D + lane * PER;
  if constexpr (PER == 2) {
    *reinterpret_cast<uint32_t*>(op) = H::pack2(acc[0] * inv, acc[1] * inv);
  } else {
    // rounded to fp32 first, as the attention kernel's packed conversion does (a product and
    // its conversion to fp16 otherwise become one instruction with one rounding)
    float r = acc[0] * inv;
    asm("" : "+v"(r));
    stf(op, r);
  }
}

size_t attn_partial_floats(int64_t R, int32_t Hq, int32_t D, int32_t max_splits) {
  return max_splits > 1 ? (size_t)R * Hq * attn_part_record(max_splits, D) : 0;
}

int count_qblocks(const SeqTable& st, int BQ, int P = 1) {
  int n = 0;
  for (int b = 0; b < st.n; ++b) n += ((st.q_cu[b + 1] - st.q_cu[b]) * P + BQ - 1) / BQ;
  return n;
}

// Long sequences: 8 waves (256 rows) share each K/V tile, halving the tile loads per query;
// shorter ones keep 4 waves, whose smaller blocks balance better.  Each wave sees the same rows
// and key tiles in the same order either way (same results).
static bool attn_wide(const SeqTable& st) {
  int max_q = 0;
  for (int b = 0; b < st.n; ++b) max_q = std::max(max_q, st.q_cu[b + 1] - st.q_cu[b]);
  return max_q >= 8192;
}

// Rounds that x times as many equal workgroups take as the CUs hold two of: a last round of one
// workgroup a CU takes little over half of a full one, and after a few rounds the workgroups have
// drifted apart and end evenly.
static double attn_rounds(double x) {
  const double full = floor(x + 1e-6), rem = x - full;
  if (rem < 1e-6) return full;
  const double last = rem <= 0.5 ? 0.5 + 0.3 * rem : std::min(1., 0.65 + 0.37 * rem);
  return full + rem + (last - rem) * (full <= 1. ? 1. : 1.5 / full);
}

// Chunks on workgroups of their own (S slots, then a merge), or all chunks of a block in one?
// Cut, the last round of workgroups is shorter and few blocks reach more CUs; whole, nothing is
// written and a block's tiles follow each other.  Both give the same bits, so the whole batch
// decides: two workgroups a CU (one of 8 waves), 32 ns a key and round of them (19.5 with
// D = 64), 4 us a workgroup, the partials' bytes at 6 TB/s (some of them move under the tiles),
// 4 us for the merge.  Over 1124 batches (1 to 3500 blocks, 512 to 32768 keys, 6 to 40 heads) the
// choice costs 0.6% over the better form on average, 29% at most, where "cut below 512 blocks"
// cost 5.7% and 136%.  us, whole / cut: 8 responses of 700 tokens over 16384 keys, 12 heads (528
// blocks) 881 / 654, of 1000 969 / 898; 64 of 128 over 1024 keys, 6 heads (384 blocks) 56 / 102;
// 128 of 40 over 4096, 28 heads (1536 blocks) 482 / 695; 48 tokens over 1501, 28 heads 36 / 23.
AttnLongPlan attn_long_plan(const SeqTable& st, const AttnArgs& a, int32_t total_q) {
  AttnLongPlan p;
  p.wide = attn_wide(st);
  const int BQ = p.wide ? 256 : 128, P = a.Hq / a.Hkv;
  p.grid = fa_grid(fa_map(a.Hkv, a.Hkv), count_qblocks(st, BQ, P), a.Hkv);
  p.chunks = 1;
  const double slots = p.wide ? 256. : 512., key = a.D == 128 ? 0.032 : 0.0195, start = 4.;
  double whole = 0., cut = 0., bytes = 0.;                  // us of all workgroups
  double longest_whole = start, longest_cut = start;        // and of the longest one
  for (int b = 0; b < st.n; ++b) {
    const int n0 = st.pos0(b), nq = st.q_cu[b + 1] - st.q_cu[b];
    if (nq <= 0) continue;
    const int c = attn_chunks(n0, nq, a.Hq, a.Hkv, a.most_chunks);
    p.chunks = std::max(p.chunks, c);
    const double blocks = (double)(((int64_t)nq * P + BQ - 1) / BQ) * a.Hkv, work = key * (n0 + 0.5 * nq);
    whole += blocks * (work + start);
    cut += blocks * (work + start * c);
    longest_whole = std::max(longest_whole, work + start);
    longest_cut = std::max(longest_cut, work / c + start);
    if (c > 1) bytes += (double)nq * a.Hq * c * (a.D + 2) * 4.;
  }
  const bool fit = a.part && (int64_t)attn_partial_floats(total_q, a.Hq, a.D, p.chunks) <= a.part_floats;
  p.fold = p.chunks > 1 && (!fit || attn_rounds(whole / longest_whole / slots) * longest_whole <=
                                        attn_rounds(cut / longest_cut / slots) * longest_cut + bytes / 6e6 + 4.);
  p.S = p.fold ? 1 : p.chunks;
  return p;
}

// Timing-harness hook: forced tile shape (0: 32 queries/wave x 64-key tiles,
// 1: 64 queries/wave x 32-key tiles).
hipError_t launch_attention_variant(hipStream_t s, int variant, const SeqTable& st, const AttnArgs& a) {
  const FaMap m = fa_map(a.Hq, a.Hkv);
  if (variant == 0)
    k_attn_bf16<bf16_t, 128, 1, 64, 4, kDense><<<fa_grid(m, count_qblocks(st, 128), a.Hq), 256, 0, s>>>(st, a);
  else
    k_attn_bf16<bf16_t, 128, 2, 32, 4, kDense><<<fa_grid(m, count_qblocks(st, 256), a.Hq), 256, 0, s>>>(st, a);
  return hipGetLastError();
}

hipError_t launch_attention(hipStream_t s, rp_dtype dt, const SeqTable& st, const AttnArgs& a, int32_t total_q) {
  if (total_q <= 0) return hipSuccess;
  if (dt != RP_F32) {
    // The 16-bit kernel addresses a sequence's keys with 32-bit byte offsets.
    for (int b = 0; b < st.n; ++b) {
      const int64_t keys = (int64_t)st.pos0(b) + (st.q_cu[b + 1] - st.q_cu[b]);
      if ((keys + 64) * a.Hkv * a.D * 2 > (int64_t)UINT32_MAX) return hipErrorInvalidValue;
    }
    hipError_t e = hipSuccess;
    with_half16(dt, [&](auto tag_) {
      using H = decltype(tag_);
      if (a.long_keys) {
        const AttnLongPlan lp = attn_long_plan(st, a, total_q);
        const bool wide = lp.wide, fold = lp.fold;
        const int S = lp.S;
        const dim3 g(lp.grid, S);
        auto run = [&](auto d_, auto nw_) {
          constexpr int D = decltype(d_)::value, NW = decltype(nw_)::value;
          if (fold)
            k_attn_bf16<H, D, 1, 64, NW, kLongFold><<<g, NW * 64, 0, s>>>(st, a);
          else
            k_attn_bf16<H, D, 1, 64, NW, kLong><<<g, NW * 64, 0, s>>>(st, a);
        };
        typedef std::integral_constant<int, 4> N4;
        typedef std::integral_constant<int, 8> N8;
        if (a.D == 128) {
          typedef std::integral_constant<int, 128> D128;
          wide ? run(D128{}, N8{}) : run(D128{}, N4{});
        } else {
          typedef std::integral_constant<int, 64> D64;
          wide ? run(D64{}, N8{}) : run(D64{}, N4{});
        }
        if (S > 1 && (e = hipGetLastError()) == hipSuccess) {
          const int64_t items = (int64_t)total_q * a.Hq;
          const int mgrid = (int)((items + 3) / 4);
          if (a.D == 128)
            k_attn_split_merge<H, 128><<<mgrid, 256, 0, s>>>(st, a.part, S, a.Hq, a.Hkv, a.most_chunks, items, (H*)a.o);
          else
            k_attn_split_merge<H, 64><<<mgrid, 256, 0, s>>>(st, a.part, S, a.Hq, a.Hkv, a.most_chunks, items, (H*)a.o);
        }
        return;
      }
      const bool wide = attn_wide(st);
      const int grid = fa_grid(fa_map(a.Hq, a.Hkv), count_qblocks(st, wide ? 256 : 128), a.Hq);
      if (a.D == 128) {
        if (wide)
          k_attn_bf16<H, 128, 1, 64, 8, kDense><<<grid, 512, 0, s>>>(st, a);
        else
          k_attn_bf16<H, 128, 1, 64, 4, kDense><<<grid, 256, 0, s>>>(st, a);
      } else {
        if (wide)
          k_attn_bf16<H, 64, 1, 64, 8, kDense><<<grid, 512, 0, s>>>(st, a);
        else
          k_attn_bf16<H, 64, 1, 64, 4, kDense><<<grid, 256, 0, s>>>(st, a);
      }
    });
    if (e != hipSuccess) return e;
  } else {
    const int nqb = count_qblocks(st, 32);
    if (a.D == 128)  // the fragments of 128 dimensions need the registers of one wave per SIMD
      k_attn_f32<128, 4><<<nqb * a.Hq, 256, 0, s>>>(st, a);
    else
      k_attn_f32<64, 8><<<nqb * a.Hq, 512, 0, s>>>(st, a);
  }
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------
// Decode attention: split-KV partials + merge.
//
// A decode step reads every cached key and value once and does ~7 flop per byte for a
// 7-head GQA group, so it is bound by HBM bandwidth.  Each wave owns one 1024-key chunk
// of one (sequence, kv head) and streams it with no block barrier: LPK lanes hold one
// key row (8 head dims each, one 16-byte load), KPW keys per pass, and an R-deep ring of
// K/V loads stays in flight (16 KB per wave at 16-bit) while earlier passes are scored.
// All G q heads of the group read the same loaded row.  Each group of LPK lanes keeps an
// online softmax per head (log2 domain, running max raised only when a score exceeds it
// by more than 2^8, so the rescale branch is rarely taken); the groups are merged with
// lane shuffles and the wave writes (max, sum, o[D]) per head for the merge kernel.
// Partial layout (both kernels and the merge): o of (item = b * Hq + q head, chunk c) at
// part[(item * nchunks + c) * D], whole 128-byte lines written by one wave, then the
// (max, sum) pairs at part[B * Hq * nchunks * D + (item * nchunks + c) * 2].
// ------------------------------------------------------------------------------------
constexpr int DC_KEYS = 1024;  // keys per chunk (one wave)
constexpr int DC_MAXG = 8;    // q heads per kv head (validated on the host)

// Output of a decode attention: PER head dimensions of o, times 1 / l, stored as T.  The forms
// that a batch size picks give one sequence the same bits, so the conversion is fixed here and
// not the compiler's choice: one dimension a lane (D = 64) in fp16 is a product and conversion
// with a single rounding, pairs are rounded to fp32 first.
template <typename T>
__device__ __forceinline__ uint32_t scaled16(float x, float s) {
  if constexpr (std::is_same<T, f16_t>::value) {
    uint32_t r;
    asm("v_fma_mixlo_f16 %0, %1, %2, 0" : "=v"(r) : "v"(x), "v"(s));
    return r & 0xffffu;
  } else {
    return (uint32_t)f2bf(x * s);
  }
}
template <typename T, int PER>
__device__ __forceinline__ void store_scaled(T* p, const float (&o)[PER], float s) {
  if constexpr (sizeof(T) == 4) {
#pragma unroll
    for (int e = 0; e < PER; ++e) p[e] = o[e] * s;
  } else if constexpr (PER == 1) {
    *reinterpret_cast<uint16_t*>(p) = (uint16_t)scaled16<T>(o[0], s);
  } else {
    *reinterpret_cast<uint32_t*>(p) = Half16<T>::pack2(o[0] * s, o[1] * s);
  }
}

template <typename T, int D>
__global__ __launch_bounds__(256) void k_decode_attn_part(const T* __restrict__ q, int q_ld,
                                                          const T* __restrict__ ck, const T* __restrict__ cv,
                                                          const int32_t* __restrict__ kv_len, int cap,
                                                          int max_pos, int B, int Hq, int Hkv, float scale,
                                                          int nchunks, float* __restrict__ part) {
  constexpr int LPK = D / 8;                  // lanes per key row
  constexpr int KPW = kWave / LPK;            // keys per pass
  constexpr int NPASS = DC_KEYS / KPW;        // passes per chunk
  constexpr int R = sizeof(T) == 4 ? 4 : 8;   // passes in flight
  static_assert(NPASS % R == 0, "ring");
  const int lane = threadIdx.x & 63;
  const int wid = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int c = wid % nchunks, bg = wid / nchunks;
  if (bg >= B * Hkv) return;
  const int g = bg % Hkv, b = bg / Hkv;
  const int G = Hq / Hkv;
  const int n = min(max(kv_len[b], 0), min(cap, max_pos) - 1);  // new token slot; keys 0..n
  const int k_begin = c * DC_KEYS;
  const int nkeys = min(DC_KEYS, n + 1 - k_begin);
  const int64_t rec = (int64_t)(b * Hq + g * G) * nchunks + c;
  float* out = part + rec * D;                                  // o records
  float* oml = part + (int64_t)B * Hq * nchunks * D + rec * 2;  // (max, sum)
  const int64_t head_stride = (int64_t)nchunks * D, ml_stride = (int64_t)nchunks * 2;
  if (nkeys <= 0) {
    if (lane < G) {
      oml[lane * ml_stride] = -INFINITY;
      oml[lane * ml_stride + 1] = 0.f;
    }
    return;
  }
  const int sub = lane % LPK, kk = lane / LPK;
  const float c2 = scale * 1.4426950408889634f;  // scores in log2 units
  float qr[DC_MAXG][8];
#pragma unroll
  for (int h = 0; h < DC_MAXG; ++h) {
    if (h < G) {
      float t[8];
      const T* qp = q + (int64_t)b * q_ld + (g * G + h) * D + sub * 8;
#pragma unroll
      for (int e = 0; e < 8; ++e) t[e] = ldf(qp + e);
#pragma unroll
      for (int e = 0; e < 8; ++e) qr[h][e] = t[e] * c2;
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) qr[h][e] = 0.f;
    }
  }
  const int64_t row_ld = (int64_t)Hkv * D;
  const T* kb = ck + ((int64_t)b * cap + k_begin) * row_ld + g * D + sub * 8;
  const T* vb = cv + ((int64_t)b * cap + k_begin) * row_ld + g * D + sub * 8;
  // rows past the chunk's last key re-read that key (in bounds) and are masked
  auto row = [&](int p) -> int64_t { return (int64_t)min(p * KPW + kk, nkeys - 1) * row_ld; };
  typename Raw8<T>::type kr[R], vr[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    kr[r] = ld_raw8(kb + row(r));
    vr[r] = ld_raw8(vb + row(r));
  }
  float m[DC_MAXG], l[DC_MAXG], o[DC_MAXG][8];
#pragma unroll
  for (int h = 0; h < DC_MAXG; ++h) {
    m[h] = -1e30f;
    l[h] = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) o[h][e] = 0.f;
  }
  const int npass = (nkeys + KPW - 1) / KPW;
  for (int p0 = 0; p0 < npass; p0 += R) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int p = p0 + r;
      if (p < npass) {
        float kv[8];
        unpack8(kr[r], kv);
        if (p + R < NPASS) kr[r] = ld_raw8(kb + row(p + R));
        const bool valid = p * KPW + kk < nkeys;
        float sc[DC_MAXG];
        bool raise = false;
#pragma unroll
        for (int h = 0; h < DC_MAXG; ++h) {
          if (h < G) {
            float a = 0.f;
#pragma unroll
            for (int e = 0; e < 8; ++e) a = fmaf(qr[h][e], kv[e], a);
            a = LPK == 16 ? row16_sum(a) : oct8_sum(a);
            sc[h] = valid ? a : -1e30f;
            raise |= sc[h] > m[h] + 8.f;
          }
        }
        if (__any(raise)) {
#pragma unroll
          for (int h = 0; h < DC_MAXG; ++h) {
            if (h < G) {
              const float mn = fmaxf(m[h], sc[h]);
              const float al = __builtin_amdgcn_exp2f(m[h] - mn);
              m[h] = mn;
              l[h] *= al;
#pragma unroll
              for (int e = 0; e < 8; ++e) o[h][e] *= al;
            }
          }
        }
        float vv[8];
        unpack8(vr[r], vv);
        if (p + R < NPASS) vr[r] = ld_raw8(vb + row(p + R));
#pragma unroll
        for (int h = 0; h < DC_MAXG; ++h) {
          if (h < G) {
            const float pk = __builtin_amdgcn_exp2f(sc[h] - m[h]);
            l[h] += pk;
#pragma unroll
            for (int e = 0; e < 8; ++e) o[h][e] = fmaf(pk, vv[e], o[h][e]);
          }
        }
      }
    }
  }
  // merge the KPW key groups of the wave, then write (max in natural-log units, sum, o)
#pragma unroll
  for (int h = 0; h < DC_MAXG; ++h) {
    if (h < G) {
      float M = m[h];
#pragma unroll
      for (int off = LPK; off < kWave; off <<= 1) M = fmaxf(M, __shfl_xor(M, off, kWave));
      const float f = __builtin_amdgcn_exp2f(m[h] - M);
      float L = l[h] * f;
#pragma unroll
      for (int off = LPK; off < kWave; off <<= 1) L += __shfl_xor(L, off, kWave);
      float ov[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        float a = o[h][e] * f;
#pragma unroll
        for (int off = LPK; off < kWave; off <<= 1) a += __shfl_xor(a, off, kWave);
        ov[e] = a;
      }
      float* oh = out + h * head_stride;
      if (lane == 0) {
        oml[h * ml_stride] = M * 0.6931471805599453f;
        oml[h * ml_stride + 1] = L;
      }
      if (kk == 0) {
#pragma unroll
        for (int e = 0; e < 8; ++e) oh[sub * 8 + e] = ov[e];
      }
    }
  }
}

// 16-bit models: the same split-KV chunks on the matrix cores.  One wave owns one chunk
// of one (sequence, kv head); the G q heads of the group are the query columns of the
// prefix kernel's tile (S^T = K Q^T with v_mfma_f32_32x32x16, the scores reused as the
// B operand of O^T += V^T P^T, V^T read with ds_read_b64_tr_b16; columns >= G are
// zero and ignored).  32-key K and V tiles stream into a 3-stage per-wave LDS ring by
// direct global->LDS loads through a buffer resource whose extent ends at the
// sequence's last key, so rows past it read as zeros; the wave needs no barrier: the
// compiler waits on the loads that filled a stage before reading it, and a stage is
// refilled only after the MFMAs that consumed it.  A workgroup holds DC_WAVES waves, the
// consecutive chunks of one group; at the end they combine their (max, sum, o) through
// LDS and the group writes one partial record, so the partials written and merged are a
// DC_WAVES-th of one record per chunk.
constexpr int DC_WAVES = 3;
__host__ __device__ inline int decode_groups(int nchunks) { return (nchunks + DC_WAVES - 1) / DC_WAVES; }
// DEEP: a launch whose chunks are no more than the compute units runs one wave per chunk
// with a 5-stage ring instead (four tiles ahead: a lone wave with two is bound by the latency
// of HBM, 1.1 us a tile).  The chunks' records then go to `part` and `sums`, and
// k_decode_chunk_merge combines them as the workgroups and the merge do here, operation for
// operation: the same bits.  One sequence of 4000 keys, 4 kv heads of 128: 42 -> 32 us a layer
// (launches and timing events included).
constexpr int DC_DEEP = 5;  // four tiles ahead: 64 copies, about what a wave can have outstanding
template <typename T16, int D, bool DEEP>
__global__ __launch_bounds__(64 * (DEEP ? 1 : DC_WAVES)) void k_decode_attn_mfma(const T16* __restrict__ q, int q_ld,
                                                                    const T16* __restrict__ ck, const T16* __restrict__ cv,
                                                                    const int32_t* __restrict__ kv_len, int cap,
                                                                    int max_pos, int B, int Hq, int Hkv, float scale,
                                                                    int nchunks, float* __restrict__ part,
                                                                    float4* __restrict__ sums, T16* __restrict__ out) {
#if defined(__HIP_DEVICE_COMPILE__)
  typedef Half16<T16> H;
  typedef typename H::V8 V8;
  constexpr int KT = 32;                 // keys per tile
  constexpr int NT = DC_KEYS / KT;       // tiles per chunk
  constexpr int CH = D / 8;              // 16-byte chunks per row
  constexpr int KSTEPS = D / 16;
  constexpr int DB = D / 32;
  constexpr int LOADS = (KT * CH) / 64;  // load instructions per matrix per tile
  static_assert(NT % 3 == 0 || NT > 3, "ring");
  constexpr int PSL = KT * CH * 4 / 64;  // floats per lane in one K stage
  static_assert(DB * 16 <= 2 * PSL && PSL >= 2, "merge data fits the wave's K stages");
  constexpr int NW = DEEP ? 1 : DC_WAVES;
  constexpr int SH = DEEP ? 1 : KT * CH, SD = DEEP ? 2 * KT * CH : 1;
  __shared__ u32x4_t Ksa[NW][SH], Ksb[NW][SH], Ksc[NW][SH];
  __shared__ u32x4_t Vsa[NW][SH], Vsb[NW][SH], Vsc[NW][SH];
  __shared__ u32x4_t R0[SD], R1[SD], R2[SD], R3[SD], R4[SD];  // K tile, then V tile
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  u32x4_t *Ks0 = Ksa[wave], *Ks1 = Ksb[wave], *Ks2 = Ksc[wave];
  u32x4_t *Vs0 = Vsa[wave], *Vs1 = Vsb[wave], *Vs2 = Vsc[wave];
  // kv head fastest: the Hkv workgroups that read the same cache rows (each its own
  // 2*D-byte slice of a row) are dispatched together, so each row is fetched while open
  const int nrec = DEEP ? nchunks : decode_groups(nchunks);
  const int g = blockIdx.x % Hkv, bgr = blockIdx.x / Hkv;
  const int grp = bgr % nrec, b = bgr / nrec;
  const int c = grp * NW + wave;
  const int G = Hq / Hkv;
  // query columns: lane column fr is q head g*G + fr (zero beyond G); issued first, so they
  // are in flight while kv_len is read and are covered by the wait for the first tile
  const int fr = lane & 31, fk = lane >> 5;
  V8 qf[KSTEPS];
#pragma unroll
  for (int ks = 0; ks < KSTEPS; ++ks) {
    uint4 v = make_uint4(0u, 0u, 0u, 0u);
    if (fr < G) v = *reinterpret_cast<const uint4*>(q + (int64_t)b * q_ld + (g * G + fr) * D + ks * 16 + fk * 8);
    qf[ks] = H::as_v8(v);
  }
  const int n = min(max(kv_len[b], 0), min(cap, max_pos) - 1);  // keys 0..n
  const int k_begin = c * DC_KEYS;
  const int nkeys = c < nchunks ? min(DC_KEYS, n + 1 - k_begin) : 0;
  f32x16_t o[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int e = 0; e < 16; ++e) o[db][e] = 0.f;
  float m_run = kMaskVal, l_run = 0.f;
  if (nkeys > 0) {  // (uniform) this wave's chunk holds keys
  const int ntiles = (nkeys + KT - 1) / KT;
  // keys of this chunk as a buffer resource: rows k_begin .. n of (b, g); byte offsets
  // key * row_bytes fit 32 bits (cap * Hkv * D * 2 bytes is checked on the host)
  const uint32_t row_bytes = (uint32_t)Hkv * D * sizeof(T16);
  const uint32_t ext = (uint32_t)(nkeys - 1) * row_bytes + D * sizeof(T16);
  const int64_t e0 = ((int64_t)b * cap + k_begin) * Hkv * D + (int64_t)g * D;
  const __amdgpu_buffer_rsrc_t rsK =
      __builtin_amdgcn_make_buffer_rsrc(uniform_ptr((void*)(ck + e0)), 0, (int)ext, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsV =
      __builtin_amdgcn_make_buffer_rsrc(uniform_ptr((void*)(cv + e0)), 0, (int)ext, 0x00020000);
  uint32_t koff[LOADS], voff[LOADS];
#pragma unroll
  for (int j = 0; j < LOADS; ++j) {
    const int slot = j * 64 + lane, key = slot / CH, cp = slot % CH;
    koff[j] = (uint32_t)key * row_bytes + (uint32_t)((cp ^ kswz<D>(key)) * 16);
    voff[j] = (uint32_t)key * row_bytes + (uint32_t)((cp ^ vswz<D>(key)) * 16);
  }
#define DM_LOAD(KD_, VD_, t_)                                                                                \
  _Pragma("unroll") for (int j = 0; j < LOADS; ++j) {                                                       \
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsK, (lds_void_t*)((KD_) + j * 64), 16, koff[j] + (uint32_t)(t_) * KT * row_bytes, 0, 0, 0); \
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsV, (lds_void_t*)((VD_) + j * 64), 16, voff[j] + (uint32_t)(t_) * KT * row_bytes, 0, 0, 0); \
  }
  const float c2 = scale * 1.4426950408889634f;
  const int tr_p = lane & 15;
  const int tr_key = fk * 4 + (tr_p >> 2);
  const int tr_col = ((lane & 16) ? 16 : 0) + 4 * (tr_p & 3);

  auto tile = [&](const u32x4_t* Kc, const u32x4_t* Vc, int t) __attribute__((always_inline)) {
    f32x16_t sc;
#pragma unroll
    for (int ks = 0; ks < KSTEPS; ++ks) {
      const V8 kf = __builtin_bit_cast(V8, Kc[fr * CH + ((ks * 2 + fk) ^ kswz<D>(fr))]);
      sc = H::mma(kf, qf[ks], ks == 0 ? f32x16_t{} : sc);
    }
    // sc[e] = score(key t*KT + 8(e/4) + 4 fk + e%4, head fr)
    const int lim = nkeys - 1 - t * KT - 4 * fk;
    if (t * KT + KT > nkeys) {
#pragma unroll
      for (int e = 0; e < 16; ++e)
        if (8 * (e >> 2) + (e & 3) > lim) sc[e] = kMaskVal;
    }
    float mx = kMaskVal;
#pragma unroll
    for (int e = 0; e < 16; ++e) mx = fmaxf(mx, sc[e]);
    mx = fmaxf(mx, __shfl_xor(mx, 32, kWave)) * c2;
    if (__any(mx > m_run + kLazy)) {
      const float m_new = fmaxf(m_run, mx);
      const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
      m_run = m_new;
      l_run *= alpha;
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int e = 0; e < 16; ++e) o[db][e] *= alpha;
    }
    const float nm = -m_run;
    float ls = 0.f;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const float pv = __builtin_amdgcn_exp2f(fmaf(sc[e], c2, nm));
      sc[e] = pv;
      ls += pv;
    }
    l_run += ls;
    const T16* vbase = reinterpret_cast<const T16*>(Vc);
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) {
      const V8 pf = H::as_v8(make_uint4(H::pack2(sc[hh * 8 + 0], sc[hh * 8 + 1]), H::pack2(sc[hh * 8 + 2], sc[hh * 8 + 3]),
                                        H::pack2(sc[hh * 8 + 4], sc[hh * 8 + 5]), H::pack2(sc[hh * 8 + 6], sc[hh * 8 + 7])));
      const int ka = hh * 16 + tr_key, kc = ka + 8;
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        const int col = db * 32 + tr_col;
        const int ca = ((col >> 3) ^ vswz<D>(ka)) * 8 + (col & 7);
        const int cc = ((col >> 3) ^ vswz<D>(kc)) * 8 + (col & 7);
        const v4i16_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_t*)(vbase + ka * D + ca));
        const v4i16_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_t*)(vbase + kc * D + cc));
        const uint2 l2 = __builtin_bit_cast(uint2, lo), h2 = __builtin_bit_cast(uint2, hi);
        o[db] = H::mma(H::as_v8(make_uint4(l2.x, l2.y, h2.x, h2.y)), pf, o[db]);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  // Tile t reads stage t % 3; after it, the stage is refilled with tile t + 3 (rows past
  // the chunk's last key read as zeros and are never used).  The prologue and the steady
  // loop issue every load unconditionally (a short chunk re-reads its last tile), so the
  // compiler counts exactly which loads a stage waits for and the later ones stay in
  // flight; only the last few tiles (no loop) take branches.
  // Tile 0 runs before the loop: its wait for stage 0 also covers the query loads issued
  // ahead of the copies, so no register load is pending when the loop starts (a loop
  // whose loads fill only LDS but which reads registers still loading from before it
  // makes the compiler drain every load, these copies included, ahead of the loop).
  if constexpr (DEEP) {
    // every copy is issued, also past the chunk's tiles (out of range: nothing is fetched), so
    // the compiler counts them exactly; tile 0 runs before the loop as below
#define DD_LOAD(R_, t_) DM_LOAD(R_, (R_) + KT * CH, t_)
#define DD_STEP(R_, u_)                                  \
  if (t + (u_) < ntiles) tile(R_, R_ + KT * CH, t + (u_)); \
  DD_LOAD(R_, t + (u_) + DC_DEEP);
    DD_LOAD(R0, 0);
    DD_LOAD(R1, 1);
    DD_LOAD(R2, 2);
    DD_LOAD(R3, 3);
    DD_LOAD(R4, 4);
    tile(R0, R0 + KT * CH, 0);
    DD_LOAD(R0, DC_DEEP);
    for (int t = 1; t < ntiles; t += DC_DEEP) {
      DD_STEP(R1, 0);
      DD_STEP(R2, 1);
      DD_STEP(R3, 2);
      DD_STEP(R4, 3);
      DD_STEP(R0, 4);
    }
#undef DD_LOAD
#undef DD_STEP
  } else {
  DM_LOAD(Ks0, Vs0, 0);
  DM_LOAD(Ks1, Vs1, min(1, ntiles - 1));
  DM_LOAD(Ks2, Vs2, min(2, ntiles - 1));
  tile(Ks0, Vs0, 0);
  DM_LOAD(Ks0, Vs0, min(3, ntiles - 1));
  int t = 1;  // tiles t, t+1, t+2 in (or on their way to) stages 1, 2, 0
  for (; t + 6 <= ntiles; t += 3) {
    tile(Ks1, Vs1, t);
    DM_LOAD(Ks1, Vs1, t + 3);
    tile(Ks2, Vs2, t + 1);
    DM_LOAD(Ks2, Vs2, t + 4);
    tile(Ks0, Vs0, t + 2);
    DM_LOAD(Ks0, Vs0, t + 5);
  }
  const int r = ntiles - t;  // 0 .. 5 tiles left
  if (r > 0) tile(Ks1, Vs1, t);
  if (r > 3) { DM_LOAD(Ks1, Vs1, t + 3); }
  if (r > 1) tile(Ks2, Vs2, t + 1);
  if (r > 4) { DM_LOAD(Ks2, Vs2, t + 4); }
  if (r > 2) tile(Ks0, Vs0, t + 2);
  if (r > 3) tile(Ks1, Vs1, t + 3);
  if (r > 4) tile(Ks2, Vs2, t + 4);
  }
#undef DM_LOAD
  __builtin_amdgcn_s_waitcnt(0);  // this wave's copies have landed: its stages are free
  }
  if constexpr (DEEP) {  // this chunk's record
    const float lo = __shfl_xor(l_run, 32, kWave);
    if (fr < G) {
      const int64_t rec = (int64_t)(b * Hq + g * G + fr) * nchunks + c;
      if (fk == 0) sums[rec] = make_float4(m_run, l_run, lo, 0.f);  // (kMaskVal, 0, 0) without keys
      if (nkeys > 0) {
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
          for (int e4 = 0; e4 < 4; ++e4)
            *reinterpret_cast<float4*>(part + rec * D + db * 32 + 8 * e4 + 4 * fk) =
                make_float4(o[db][4 * e4], o[db][4 * e4 + 1], o[db][4 * e4 + 2], o[db][4 * e4 + 3]);
      }
    }
    return;
  }
  // ---- combine the group's chunks: waves 1.. leave o in their own first two K stages and
  // (max, sum) in the third (lane-major, conflict-free); wave 0 rescales them to the
  // common max and adds ----
  // o[db][e] = O^T(dim db*32 + 8(e/4) + 4 fk + e%4, head fr), unnormalised; m in log2 units
  if (wave > 0) {
    float* mine0 = reinterpret_cast<float*>(Ks0);
    float* mine1 = reinterpret_cast<float*>(Ks1);
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int i = db * 16 + e;
        (i < PSL ? mine0 : mine1)[(i % PSL) * 64 + lane] = o[db][e];
      }
    reinterpret_cast<float*>(Ks2)[lane] = m_run;
    reinterpret_cast<float*>(Ks2)[64 + lane] = l_run;
  }
  __syncthreads();
  if (wave != 0) return;
  if (nkeys <= 0) {  // the group's first chunk is past the last key: so are the others
    if (lane < G) {
      const int64_t rec = (int64_t)(b * Hq + g * G + lane) * nrec + grp;
      *reinterpret_cast<float2*>(part + (int64_t)B * Hq * nrec * D + rec * 2) = make_float2(-INFINITY, 0.f);
    }
    return;
  }
  float mw[DC_WAVES], M = m_run;
  mw[0] = m_run;
#pragma unroll
  for (int w = 1; w < DC_WAVES; ++w) {
    mw[w] = reinterpret_cast<const float*>(Ksc[w])[lane];
    M = fmaxf(M, mw[w]);
  }
  const float f0 = __builtin_amdgcn_exp2f(m_run - M);
  float lsum = l_run * f0;
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int e = 0; e < 16; ++e) o[db][e] *= f0;
#pragma unroll
  for (int w = 1; w < DC_WAVES; ++w) {
    const float* t0 = reinterpret_cast<const float*>(Ksa[w]);
    const float* t1 = reinterpret_cast<const float*>(Ksb[w]);
    const float fw = __builtin_amdgcn_exp2f(mw[w] - M);  // 0 for an empty chunk (max kMaskVal)
    lsum = fmaf(reinterpret_cast<const float*>(Ksc[w])[64 + lane], fw, lsum);
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int i = db * 16 + e;
        o[db][e] = fmaf((i < PSL ? t0 : t1)[(i % PSL) * 64 + lane], fw, o[db][e]);
      }
  }
  const float l = lsum + __shfl_xor(lsum, 32, kWave);
  if (nrec == 1) {  // the sequence's only record: the result itself, as the merge would form it
    if (fr < G) {
      const float inv = 1.0f / l;
      T16* oh = out + (int64_t)(b * Hq + g * G + fr) * D;
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int e4 = 0; e4 < 4; ++e4) {
          float v[4];  // (+ 0: the merge adds its one record to 0)
#pragma unroll
          for (int t = 0; t < 4; ++t) v[t] = o[db][4 * e4 + t] + 0.f;
          uint2 w;
          if constexpr (D == 64) {
            w.x = scaled16<T16>(v[0], inv) | scaled16<T16>(v[1], inv) << 16;
            w.y = scaled16<T16>(v[2], inv) | scaled16<T16>(v[3], inv) << 16;
          } else {
            w.x = H::pack2(v[0] * inv, v[1] * inv);
            w.y = H::pack2(v[2] * inv, v[3] * inv);
          }
          *reinterpret_cast<uint2*>(oh + db * 32 + 8 * e4 + 4 * fk) = w;
        }
    }
    return;
  }
  if (fr < G) {
    const int64_t rec = (int64_t)(b * Hq + g * G + fr) * nrec + grp;
    float* oh = part + rec * D;
    if (fk == 0)
      *reinterpret_cast<float2*>(part + (int64_t)B * Hq * nrec * D + rec * 2) =
          make_float2(M * 0.6931471805599453f, l);
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int e4 = 0; e4 < 4; ++e4) {
        const int dh = db * 32 + 8 * e4 + 4 * fk;
        *reinterpret_cast<float4*>(oh + dh) =
            make_float4(o[db][4 * e4], o[db][4 * e4 + 1], o[db][4 * e4 + 2], o[db][4 * e4 + 3]);
      }
  }
#endif
}

// Merge of the DEEP kernel's chunk records, one wave per (sequence, q head): lane r combines
// the sums of chunks 3 r .. 3 r + 2 as wave 0 of a workgroup does above (each half wave's sum
// apart, then added), the groups are merged as in k_decode_attn_merge, and each lane forms its
// D/64 dimensions of every group's o on the way.  At most 64 groups.
template <typename T, int D>
__global__ __launch_bounds__(256) void k_decode_chunk_merge(const float* __restrict__ part,
                                                            const float4* __restrict__ sums, int nchunks, int items,
                                                            T* __restrict__ o) {
  constexpr int PER = D / 64;
  static_assert(DC_WAVES == 3, "groups of three chunks");
  const int item = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (item >= items) return;
  const int nrec = decode_groups(nchunks);
  const float4 none = make_float4(kMaskVal, 0.f, 0.f, 0.f);
  float4 s[3];
#pragma unroll
  for (int w = 0; w < 3; ++w) {
    const int c = lane * 3 + w;
    s[w] = c < nchunks ? sums[(int64_t)item * nchunks + c] : none;
  }
  float M3 = s[0].x;
#pragma unroll
  for (int w = 1; w < 3; ++w) M3 = fmaxf(M3, s[w].x);
  float f[3];
#pragma unroll
  for (int w = 0; w < 3; ++w) f[w] = __builtin_amdgcn_exp2f(s[w].x - M3);
  float l0 = s[0].y * f[0], l1 = s[0].z * f[0];
#pragma unroll
  for (int w = 1; w < 3; ++w) {
    l0 = fmaf(s[w].y, f[w], l0);
    l1 = fmaf(s[w].z, f[w], l1);
  }
  const bool has = lane < nrec && s[0].x > kMaskVal;  // chunks with keys come first
  const float mc = has ? M3 * 0.6931471805599453f : -INFINITY;
  const float M = wave_max(mc);
  const float wt = has ? expf(mc - M) : 0.f;
  const float L = wave_sum(has ? wt * (l0 + l1) : 0.f);
  const int nv = __popcll(__ballot(has));
  float acc[PER];
#pragma unroll
  for (int e = 0; e < PER; ++e) acc[e] = 0.f;
  for (int r = 0; r < nv; ++r) {
    const float wr = __shfl(wt, r, kWave);
    const float* oc = part + ((int64_t)item * nchunks + 3 * r) * D + lane * PER;
    float og[PER];
#pragma unroll
    for (int w = 0; w < 3; ++w) {
      const float fw = __shfl(f[w], r, kWave);
      const bool in = __shfl(s[w].x, r, kWave) > kMaskVal;
#pragma unroll
      for (int e = 0; e < PER; ++e) {
        const float x = in ? oc[w * D + e] : 0.f;
        og[e] = w == 0 ? x * fw : fmaf(x, fw, og[e]);
      }
    }
#pragma unroll
    for (int e = 0; e < PER; ++e) acc[e] = fmaf(wr, og[e], acc[e]);
  }
  const float inv = 1.0f / L;
  store_scaled(o + (int64_t)item * D + lane * PER, acc, inv);
}

// Merge of the decode chunks: one wave per (sequence, q head).  Lane c holds chunk c's
// (max, sum) (chunks with keys come first; the rest have max -inf and stale o, never
// read), the wave reduces them, and each lane then sums its D/64 head dimensions over the
// chunks with every chunk's weight taken from its lane, all loads independent.
template <typename T, int D>
__global__ __launch_bounds__(256) void k_decode_attn_merge(const float* __restrict__ part, int nchunks, int items,
                                                           T* __restrict__ o) {
  constexpr int PER = D / 64;
  const int item = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (item >= items) return;
  const float* p = part + (int64_t)item * nchunks * D;                                    // o records
  const float* pml = part + (int64_t)items * nchunks * D + (int64_t)item * nchunks * 2;  // (max, sum)
  float M = -INFINITY;
  for (int c = lane; c < nchunks; c += 64) M = fmaxf(M, pml[2 * c]);
  M = wave_max(M);
  float L = 0.f, acc[PER];
#pragma unroll
  for (int e = 0; e < PER; ++e) acc[e] = 0.f;
  for (int c0 = 0; c0 < nchunks; c0 += 64) {
    const int c = c0 + lane;
    const float mc = c < nchunks ? pml[2 * c] : -INFINITY;
    const bool has = mc > -INFINITY;
    const float w = has ? expf(mc - M) : 0.f;
    L += has ? w * pml[2 * c + 1] : 0.f;
    const int nv = __popcll(__ballot(has));  // chunks with keys: a prefix of c0 ..
#pragma unroll 4
    for (int j = 0; j < nv; ++j) {
      const float wj = __shfl(w, j, kWave);
      const float* oc = p + (int64_t)(c0 + j) * D + lane * PER;
#pragma unroll
      for (int e = 0; e < PER; ++e) acc[e] = fmaf(wj, oc[e], acc[e]);
    }
  }
  L = wave_sum(L);
  const float inv = 1.0f / L;
  store_scaled(o + (int64_t)item * D + lane * PER, acc, inv);
}

size_t decode_attn_partial_floats(int32_t B, int32_t Hq, int32_t D, int32_t cap) {
  const int nchunks = (cap + DC_KEYS - 1) / DC_KEYS;
  return (size_t)B * Hq * nchunks * (D + 2);
}

// One wave per chunk where each can have a compute unit to itself (and the records fit).  Up to
// three chunks are one record of the three-wave form, which writes the result itself: without the
// merge it is faster, unless three full chunks of rows of 1 KB and more share a CU.  us with
// launches and timing events, a wave per chunk / three waves: 998 keys, 2 kv heads of 128, 64
// sequences 33 / 27; 2046 keys 34 / 30; 3070 keys 33 / 30, but 33 / 43 with 4 kv heads.
bool decode_attn_deep(int32_t B, int32_t Hq, int32_t Hkv, int32_t D, int32_t cap, int64_t sums_floats) {
  const int nchunks = (cap + DC_KEYS - 1) / DC_KEYS;
  return (nchunks > 3 || (nchunks == 3 && Hkv * D >= 512)) && (int64_t)B * Hkv * nchunks <= 256 &&
         decode_groups(nchunks) <= 64 && (int64_t)B * Hq * nchunks * 4 <= sums_floats;
}

hipError_t launch_decode_attention(hipStream_t s, rp_dtype dt, const void* q, int32_t q_ld,
                                   const void* cache_k, const void* cache_v, const int32_t* kv_len,
                                   int32_t cap, int32_t max_pos, int32_t B, int32_t Hq, int32_t Hkv,
                                   int32_t D, float scale, float* partials, float* sums, int64_t sums_floats, void* o) {
  const int nchunks = (cap + DC_KEYS - 1) / DC_KEYS;
  if (dt == RP_F32) {
    const int grid = (B * Hkv * nchunks + 3) / 4;  // one wave per chunk, 4 waves per workgroup
    if (D == 128)
      k_decode_attn_part<float, 128><<<grid, 256, 0, s>>>((const float*)q, q_ld, (const float*)cache_k,
                                                          (const float*)cache_v, kv_len, cap, max_pos, B, Hq, Hkv,
                                                          scale, nchunks, partials);
    else
      k_decode_attn_part<float, 64><<<grid, 256, 0, s>>>((const float*)q, q_ld, (const float*)cache_k,
                                                         (const float*)cache_v, kv_len, cap, max_pos, B, Hq, Hkv,
                                                         scale, nchunks, partials);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (D == 128)
      k_decode_attn_merge<float, 128><<<(B * Hq + 3) / 4, 256, 0, s>>>(partials, nchunks, B * Hq, (float*)o);
    else
      k_decode_attn_merge<float, 64><<<(B * Hq + 3) / 4, 256, 0, s>>>(partials, nchunks, B * Hq, (float*)o);
    return hipGetLastError();
  }
  // the 16-bit kernel addresses a sequence's cache rows with 32-bit byte offsets
  if ((int64_t)cap * Hkv * D * 2 > (int64_t)INT32_MAX) return hipErrorInvalidValue;
  const int nrec = decode_groups(nchunks);
  const bool deep = decode_attn_deep(B, Hq, Hkv, D, cap, sums_floats) && sums && !((uintptr_t)sums & 15);
  const int grid = B * Hkv * (deep ? nchunks : nrec), mgrid = (B * Hq + 3) / 4;
  with_half16(dt, [&](auto tag_) {
    using H = decltype(tag_);
    auto run = [&](auto d_) {
      constexpr int DD = decltype(d_)::value;
      if (deep) {
        k_decode_attn_mfma<H, DD, true><<<grid, 64, 0, s>>>((const H*)q, q_ld, (const H*)cache_k, (const H*)cache_v,
                                                            kv_len, cap, max_pos, B, Hq, Hkv, scale, nchunks, partials,
                                                            (float4*)sums, (H*)o);
        k_decode_chunk_merge<H, DD><<<mgrid, 256, 0, s>>>(partials, (const float4*)sums, nchunks, B * Hq, (H*)o);
        return;
      }
      k_decode_attn_mfma<H, DD, false><<<grid, 64 * DC_WAVES, 0, s>>>((const H*)q, q_ld, (const H*)cache_k,
                                                                      (const H*)cache_v, kv_len, cap, max_pos, B, Hq,
                                                                      Hkv, scale, nchunks, partials, nullptr, (H*)o);
      if (nrec > 1) k_decode_attn_merge<H, DD><<<mgrid, 256, 0, s>>>(partials, nrec, B * Hq, (H*)o);
    };
    if (D == 128)
      run(std::integral_constant<int, 128>());
    else
      run(std::integral_constant<int, 64>());
  });
  return hipGetLastError();
}

}  // namespace rp
