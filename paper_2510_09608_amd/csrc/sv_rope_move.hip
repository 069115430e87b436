// Bandwidth-bound row movers: storing new K/V (K rotated at its assigned
// position), rotating fresh Q/K in place, and the compaction gather that moves
// every surviving K/V row of every layer to its new slot while re-rotating K by
// the position shift (Sec. 2.1: states are reused, positions stay contiguous).
//
// All three share one thread layout.  A row of head_dim elements is split into
// a low and a high half; the rotary pairing is (i, i + head_dim/2), so a thread
// that owns 16 bytes of the low half and the matching 16 bytes of the high half
// holds complete pairs.  Rows are 128-512 bytes, a wavefront therefore covers
// 4-16 whole rows with two fully coalesced 16-byte accesses per lane.

#include <hip/hip_bf16.h>

#include "sv_internal.h"

namespace sv {
namespace {

template <typename T>
struct Vec16;
template <>
struct Vec16<float> {
  static constexpr int N = 4;
  float4 raw;
  __device__ float get(int e) const { return ((const float*)&raw)[e]; }
  __device__ void set(int e, float x) { ((float*)&raw)[e] = x; }
};
template <>
struct Vec16<__hip_bfloat16> {
  static constexpr int N = 8;
  uint4 raw;
  __device__ float get(int e) const {
    const uint32_t w = ((const uint32_t*)&raw)[e >> 1];
    return __uint_as_float((e & 1) ? (w & 0xffff0000u) : (w << 16));
  }
  __device__ void set(int e, float x) {  // round to nearest even
    uint32_t u = __float_as_uint(x);
    u += 0x7fffu + ((u >> 16) & 1u);
    uint32_t& w = ((uint32_t*)&raw)[e >> 1];
    w = (e & 1) ? ((w & 0x0000ffffu) | (u & 0xffff0000u)) : ((w & 0xffff0000u) | (u >> 16));
  }
};

template <typename T, int D>
struct RowGeom {
  static constexpr int EPV = 16 / (int)sizeof(T);  // elements per 16-byte vector
  static constexpr int TPR = (D / 2) / EPV;        // threads per row
  static constexpr int ROWS = 256 / TPR;           // rows per 256-thread block
};

// cos/sin of angle for a rotation by pos * inv_freq; double for fp32 data (the
// fp32 workload is held to 1e-5), float for bf16 data.
template <typename T>
__device__ __forceinline__ void rot_cs(double angle, float& c, float& s) {
  if constexpr (sizeof(T) == 4) {
    double sd, cd;
    sincos(angle, &sd, &cd);
    c = (float)cd;
    s = (float)sd;
  } else {
    sincosf((float)angle, &s, &c);
  }
}

__device__ __forceinline__ int pos_of_freq(const int4& p, int i, int rope_mode, int s0, int s01) {
  if (rope_mode != SV_ROPE_3D) return p.x;
  return i < s0 ? p.x : (i < s01 ? p.y : p.z);
}

template <typename T, int D>
__device__ __forceinline__ void rotate_pair_vec(Vec16<T>& lo, Vec16<T>& hi, const int4 p, int i0, int rope_mode,
                                                int s0, int s01, const double* __restrict__ inv_freq) {
  double f[Vec16<T>::N];   // all frequencies first: loaded one by one between the sincos evaluations, each is a round trip
#pragma unroll
  for (int e = 0; e < Vec16<T>::N; ++e) f[e] = inv_freq[i0 + e];
#pragma unroll
  for (int e = 0; e < Vec16<T>::N; ++e) {
    const int i = i0 + e;
    float c, s;
    rot_cs<T>((double)pos_of_freq(p, i, rope_mode, s0, s01) * f[e], c, s);
    const float a = lo.get(e), b = hi.get(e);
    lo.set(e, a * c - b * s);
    hi.set(e, b * c + a * s);
  }
}

// ---------------------------------------------------------------------------------
// Store n new tokens of one layer: cache[K|V][h][slot0 + j] = (rotated K | V)[j][h].
// bx: block of ROWS tokens, h: kv head, which: 0 = K, 1 = V.
// ---------------------------------------------------------------------------------
template <typename T, int D>
__device__ __forceinline__ void append_rows(int bx, int h, int which, const T* __restrict__ k_in,
                                            const T* __restrict__ v_in, T* __restrict__ k_cache, T* __restrict__ v_cache,
                                            const int4* __restrict__ pos4, const double* __restrict__ inv_freq,
                                            int64_t slot0, int n, int n_kv_heads, size_t head_stride_elems,
                                            int rope_mode, int s0, int s01, const float2* __restrict__ cs_tab = nullptr) {
  using G = RowGeom<T, D>;
  const int j = bx * G::ROWS + threadIdx.x / G::TPR;
  if (j >= n) return;
  const int t = threadIdx.x % G::TPR;
  const T* src = (which == 0 ? k_in : v_in) + ((size_t)j * n_kv_heads + h) * D;
  T* dst = (which == 0 ? k_cache : v_cache) + (size_t)h * head_stride_elems + (size_t)(slot0 + j) * D;
  Vec16<T> lo, hi;
  // The (uniform) choice of where cos/sin come from is made BEFORE the row's loads, so that on the table's path the
  // row and its cos/sin go out together: with the choice behind the row's loads the compiler waited for the row
  // before it issued the table's loads, two memory round trips for a kernel that is little else.
  if (which == 0 && cs_tab != nullptr) {   // (a table is only ever given with a rotary mode)
    // cos/sin of the run's tokens were tabulated when it was registered: [token][pair]
    const float2* cs = cs_tab + (size_t)j * (D / 2) + t * G::EPV;
    lo.raw = *(const decltype(lo.raw)*)(src + t * G::EPV);
    hi.raw = *(const decltype(hi.raw)*)(src + D / 2 + t * G::EPV);
    float2 r[Vec16<T>::N];
#pragma unroll
    for (int e = 0; e < Vec16<T>::N; ++e) r[e] = cs[e];
#pragma unroll
    for (int e = 0; e < Vec16<T>::N; ++e) {
      const float a = lo.get(e), b = hi.get(e);
      lo.set(e, a * r[e].x - b * r[e].y);
      hi.set(e, b * r[e].x + a * r[e].y);
    }
  } else {
    lo.raw = *(const decltype(lo.raw)*)(src + t * G::EPV);
    hi.raw = *(const decltype(hi.raw)*)(src + D / 2 + t * G::EPV);
    if (which == 0 && rope_mode != SV_ROPE_NONE)
      rotate_pair_vec<T, D>(lo, hi, pos4[slot0 + j], t * G::EPV, rope_mode, s0, s01, inv_freq);
  }
  *(decltype(lo.raw)*)(dst + t * G::EPV) = lo.raw;
  *(decltype(hi.raw)*)(dst + D / 2 + t * G::EPV) = hi.raw;
}

// ---------------------------------------------------------------------------------
// Rotate rows of x [n][n_heads][D] in place at the positions of slots slot0 + j.
// bx: block of ROWS (token, head) rows.
// ---------------------------------------------------------------------------------
template <typename T, int D>
__device__ __forceinline__ void rope_rows(int bx, T* __restrict__ x, const int4* __restrict__ pos4,
                                          const double* __restrict__ inv_freq, int64_t slot0, int n, int n_heads,
                                          int rope_mode, int s0, int s01, const float2* __restrict__ cs_tab = nullptr) {
  using G = RowGeom<T, D>;
  const int64_t row = (int64_t)bx * G::ROWS + threadIdx.x / G::TPR;
  if (row >= (int64_t)n * n_heads) return;
  const int t = threadIdx.x % G::TPR;
  const int j = (int)(row / n_heads);
  T* p = x + row * D;
  Vec16<T> lo, hi;
  if (cs_tab != nullptr) {   // cos/sin of the run's tokens, tabulated when it was registered: [token][pair]
    const float2* cs = cs_tab + (size_t)j * (D / 2) + t * G::EPV;   // (the row and its cos/sin go out together)
    lo.raw = *(const decltype(lo.raw)*)(p + t * G::EPV);
    hi.raw = *(const decltype(hi.raw)*)(p + D / 2 + t * G::EPV);
    float2 r[Vec16<T>::N];
#pragma unroll
    for (int e = 0; e < Vec16<T>::N; ++e) r[e] = cs[e];
#pragma unroll
    for (int e = 0; e < Vec16<T>::N; ++e) {
      const float a = lo.get(e), b = hi.get(e);
      lo.set(e, a * r[e].x - b * r[e].y);
      hi.set(e, b * r[e].x + a * r[e].y);
    }
  } else {
    lo.raw = *(const decltype(lo.raw)*)(p + t * G::EPV);
    hi.raw = *(const decltype(hi.raw)*)(p + D / 2 + t * G::EPV);
    rotate_pair_vec<T, D>(lo, hi, pos4[slot0 + j], t * G::EPV, rope_mode, s0, s01, inv_freq);
  }
  *(decltype(lo.raw)*)(p + t * G::EPV) = lo.raw;
  *(decltype(hi.raw)*)(p + D / 2 + t * G::EPV) = hi.raw;
}

// The same as a launch of its own: a head per thread, rows as they lie (fp32 up to 600 workgroups or with one head, see rope_apply_t).
// grid: ceil(n * n_heads / ROWS)
template <typename T, int D>
__global__ __launch_bounds__(256) void k_rope_rows_flat(T* __restrict__ x, const int4* __restrict__ pos4,
                                                        const double* __restrict__ inv_freq, int64_t slot0, int n,
                                                        int n_heads, int rope_mode, int s0, int s01,
                                                        const float2* __restrict__ cs_tab) {
  rope_rows<T, D>(blockIdx.x, x, pos4, inv_freq, slot0, n, n_heads, rope_mode, s0, s01, cs_tab);
}

// A thread takes its place of HG heads of a token: position, cos/sin and what is divided are worked out once for them, below the
// rows' loads.  With a head per thread, and the token from a 64-bit division, the launch was bound by
// that: 5376 tokens of 28 heads (77 MB) 17.2 us, with 4 heads 13.0 (5.9 TB/s).
// grid: ceil(n / ROWS) * ceil(n_heads / HG), the heads' shares side by side.  cs_tab: of the run that starts at slot0, or NULL.
template <typename T, int D, int HG>
__global__ __launch_bounds__(256) void k_rope_rows(T* __restrict__ x, const int4* __restrict__ pos4,
                                                   const double* __restrict__ inv_freq, int64_t slot0, int n,
                                                   int n_heads, int rope_mode, int s0, int s01,
                                                   const float2* __restrict__ cs_tab) {
  using G = RowGeom<T, D>;
  constexpr int E = Vec16<T>::N;
  const uint32_t shares = (uint32_t)(n_heads + HG - 1) / HG, tokens = blockIdx.x / shares, share = blockIdx.x - tokens * shares;
  const int j = tokens * G::ROWS + threadIdx.x / G::TPR, t = threadIdx.x % G::TPR;
  if (j >= n) return;
  T* const p = x + ((size_t)j * n_heads + HG * share) * D + t * G::EPV;
  const int heads = min(HG, n_heads - (int)(HG * share));
  Vec16<T> lo[HG], hi[HG];
#pragma unroll
  for (int h = 0; h < HG; ++h) {
    const T* const row = p + min(h, heads - 1) * D;
    lo[h].raw = *(const decltype(lo[h].raw)*)row;
    hi[h].raw = *(const decltype(hi[h].raw)*)(row + D / 2);
  }
  float2 r[E];
  if (cs_tab != nullptr) {   // cos/sin of the run's tokens, tabulated when it was registered: [token][pair]
    const float2* cs = cs_tab + (size_t)j * (D / 2) + t * G::EPV;
#pragma unroll
    for (int e = 0; e < E; ++e) r[e] = cs[e];
  } else {
    const int4 pos = pos4[slot0 + j];
    double f[E];
#pragma unroll
    for (int e = 0; e < E; ++e) f[e] = inv_freq[t * G::EPV + e];
#pragma unroll
    for (int e = 0; e < E; ++e) rot_cs<T>((double)pos_of_freq(pos, t * G::EPV + e, rope_mode, s0, s01) * f[e], r[e].x, r[e].y);
  }
#pragma unroll
  for (int h = 0; h < HG; ++h) {
    if (h >= heads) break;
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const float a = lo[h].get(e), b = hi[h].get(e);
      lo[h].set(e, a * r[e].x - b * r[e].y);
      hi[h].set(e, b * r[e].x + a * r[e].y);
    }
    *(decltype(lo[h].raw)*)(p + h * D) = lo[h].raw;
    *(decltype(hi[h].raw)*)(p + h * D + D / 2) = hi[h].raw;
  }
}

// Everything that stores a run of new tokens of one layer in a row-major cache, in ONE launch: workgroup ids [0, nb_k)
// rotate and store K rows, [nb_k, 2 nb_k) store V rows, the rest rotate Q rows in place.
template <typename T, int D>
__global__ __launch_bounds__(256) void k_store_tokens(T* __restrict__ q, const T* __restrict__ k_in, const T* __restrict__ v_in,
                                                      T* __restrict__ k_cache, T* __restrict__ v_cache,
                                                      const int4* __restrict__ pos4, const double* __restrict__ inv_freq,
                                                      int64_t slot0, int n, int n_q_heads, int n_kv_heads,
                                                      size_t head_stride_elems, int rope_mode, int s0, int s01, int nb_k,
                                                      const float2* __restrict__ cs_tab) {
  const int gx_k = nb_k / n_kv_heads;
  int b = blockIdx.x;
  if (b < 2 * nb_k) {
    const int which = b >= nb_k;
    if (which) b -= nb_k;
    append_rows<T, D>(b % gx_k, b / gx_k, which, k_in, v_in, k_cache, v_cache, pos4, inv_freq, slot0, n, n_kv_heads,
                      head_stride_elems, rope_mode, s0, s01, cs_tab);
    return;
  }
  rope_rows<T, D>(b - 2 * nb_k, q, pos4, inv_freq, slot0, n, n_q_heads, rope_mode, s0, s01, cs_tab);
}

// ---------------------------------------------------------------------------------
// Storing V of new tokens into the blocked V^T layout (see sv_internal.h): rows [slot0, slot0 + n) of one kv head
// that fall into the group of 32 slots [32 grp, 32 grp + 32) are staged row-major in LDS, then every thread
// collects two pieces of 8 keys x one head dim (a block row) and writes each as 16 bytes, or element by element
// where a piece is only partly new (its other keys belong to older tokens).  Consecutive lanes write
// consecutive rows of a block: 1 KB contiguous per store instruction.
// Slots past the end of a stream inside its last block hold zeros or old values, never NaN patterns (the store is
// cleared at create time): the attention kernels multiply them by probabilities of exactly zero.
// ---------------------------------------------------------------------------------
constexpr int VG = 32;                     // slots per workgroup of the V^T store (4 blocks)
template <int D>
constexpr int VT_SROW = D * 2 + 16;        // bytes per staged row in LDS

template <int D>
__device__ __forceinline__ void append_v_t_group(char* sT, int grp, int hk, const __hip_bfloat16* __restrict__ v_in,
                                                 __hip_bfloat16* __restrict__ v_cache, int64_t slot0, int n,
                                                 int n_kv_heads, size_t head_stride_elems) {
  const int tid = threadIdx.x;
  const int64_t key0 = (int64_t)grp * VG;
  constexpr int NP = VG * D / 8 / 256, CPR = D / 8;   // 16-byte pieces per thread, per row
  // the loads of a thread are unconditional (a slot of the group outside the run reads the run's nearest row and
  // stages zeros) and issued together: guarded, the compiler waited for the first before it issued the second
  uint4 vin[NP];
#pragma unroll
  for (int i = 0; i < NP; ++i) {
    const int cid = tid + 256 * i, key = cid / CPR, c16 = cid % CPR;
    const int64_t kc = min(max(key0 + key, slot0), slot0 + n - 1);
    vin[i] = *(const uint4*)(v_in + ((size_t)(kc - slot0) * n_kv_heads + hk) * D + c16 * 8);
  }
#pragma unroll
  for (int i = 0; i < NP; ++i) {
    const int cid = tid + 256 * i, key = cid / CPR, c16 = cid % CPR;
    const int64_t kk = key0 + key;
    const bool in_run = (kk >= slot0) & (kk < slot0 + n);
    *(uint4*)(sT + key * VT_SROW<D> + c16 * 16) = in_run ? vin[i] : make_uint4(0, 0, 0, 0);
  }
  __syncthreads();
  unsigned short* head_base = (unsigned short*)v_cache + (size_t)hk * head_stride_elems;
#pragma unroll
  for (int i = 0; i < NP; ++i) {
    const int piece = tid + 256 * i, p = piece / D, d = piece % D;   // block p of the group, head dim d
    unsigned short e[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) e[j] = *(const unsigned short*)(sT + (8 * p + j) * VT_SROW<D> + d * 2);
    const int64_t k8 = key0 + 8 * p;
    unsigned short* dst = head_base + vt_elem<D>(k8, d);
    if (k8 >= slot0 && k8 + 8 <= slot0 + n) {
      uint4 w;
      w.x = e[0] | ((uint32_t)e[1] << 16), w.y = e[2] | ((uint32_t)e[3] << 16);
      w.z = e[4] | ((uint32_t)e[5] << 16), w.w = e[6] | ((uint32_t)e[7] << 16);
      *(uint4*)dst = w;
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (k8 + j >= slot0 && k8 + j < slot0 + n) dst[j] = e[j];
    }
  }
}

// ---------------------------------------------------------------------------------
// Everything that stores a run of new tokens of one layer in a blocked-V^T cache, in ONE launch: K rows (rotated
// at their positions), V into its V^T blocks, and, when q is given, the rotation of the tokens' Q rows in place (the
// chunk prefill's prologue).  The three jobs are independent; workgroup ids [0, nb_k) do the first,
// [nb_k, nb_k + nb_q) the second, the rest the third.
// ---------------------------------------------------------------------------------
// All 14 dwords of its arguments reach the wavefront in SGPRs at launch, so no scalar fetch precedes the loads of a
// kernel that is little more than one memory round trip: the V plane follows the K plane of the layer, the job
// boundaries follow from n, slot0 and the head counts, and cos/sin come from the run's table only (cs_tab NULL: no
// rotary embedding, rows are copied; a cache with a rotary mode always has the table for a run this kernel is given).
// shape: bit 1 = rotate q, bits 8-15 kv heads, bits 16-31 query heads.
template <int D>
__global__ __launch_bounds__(256) void k_store_tokens_vt(
    __hip_bfloat16* __restrict__ q, const __hip_bfloat16* __restrict__ k_in, const __hip_bfloat16* __restrict__ v_in,
    __hip_bfloat16* __restrict__ k_cache, const float2* __restrict__ cs_tab, int slot0, int n, uint32_t head_stride_elems,
    uint32_t shape) {
  __shared__ __attribute__((aligned(16))) char sT[VG * VT_SROW<D>];
  using T = __hip_bfloat16;
  using G = RowGeom<T, D>;
  const int n_kv_heads = (shape >> 8) & 255, n_q_heads = (int)(shape >> 16);
  __hip_bfloat16* const v_cache = k_cache + (size_t)n_kv_heads * head_stride_elems;   // K and V planes of a layer are adjacent
  const int gx_k = (n + G::ROWS - 1) / G::ROWS, nb_k = gx_k * n_kv_heads;
  const int nb_q = (shape & 2) ? (n * n_q_heads + G::ROWS - 1) / G::ROWS : 0;
  const int blk0 = slot0 / VG, n_blk = (slot0 + n - 1) / VG - blk0 + 1;   // groups of 32 slots
  int b = blockIdx.x;
  if (b >= nb_k + nb_q) {
    b -= nb_k + nb_q;
    append_v_t_group<D>(sT, blk0 + b % n_blk, b / n_blk, v_in, v_cache, slot0, n, n_kv_heads, head_stride_elems);
    return;
  }
  // a K row into the cache, or a Q row in place: the row and its token's cos/sin go out together, one round trip
  const bool is_k = b < nb_k;
  const int t = threadIdx.x % G::TPR;
  int j;
  const T* src;
  T* dst;
  if (is_k) {
    const int h = b / gx_k;
    j = (b % gx_k) * G::ROWS + threadIdx.x / G::TPR;
    if (j >= n) return;
    src = k_in + ((size_t)j * n_kv_heads + h) * D;
    dst = k_cache + (size_t)h * head_stride_elems + (size_t)(slot0 + j) * D;
  } else {
    const int64_t row = (int64_t)(b - nb_k) * G::ROWS + threadIdx.x / G::TPR;
    if (row >= (int64_t)n * n_q_heads) return;
    j = (int)(row / n_q_heads);
    dst = q + row * D;
    src = dst;
  }
  Vec16<T> lo, hi;
  lo.raw = *(const decltype(lo.raw)*)(src + t * G::EPV);
  hi.raw = *(const decltype(hi.raw)*)(src + D / 2 + t * G::EPV);
  if (cs_tab != nullptr) {   // [token of the run][pair]
    const float2* cs = cs_tab + (size_t)j * (D / 2) + t * G::EPV;
    float2 r[Vec16<T>::N];
#pragma unroll
    for (int e = 0; e < Vec16<T>::N; ++e) r[e] = cs[e];
#pragma unroll
    for (int e = 0; e < Vec16<T>::N; ++e) {
      const float a = lo.get(e), bb = hi.get(e);
      lo.set(e, a * r[e].x - bb * r[e].y);
      hi.set(e, bb * r[e].x + a * r[e].y);
    }
  }
  *(decltype(lo.raw)*)(dst + t * G::EPV) = lo.raw;
  *(decltype(hi.raw)*)(dst + D / 2 + t * G::EPV) = hi.raw;
}

// The same three jobs with cos/sin evaluated from the tokens' positions: runs that have no table (longer than the
// cache's max_q_tokens).
template <int D>
__global__ __launch_bounds__(256) void k_store_tokens_vt_pos(
    __hip_bfloat16* __restrict__ q, const __hip_bfloat16* __restrict__ k_in, const __hip_bfloat16* __restrict__ v_in,
    __hip_bfloat16* __restrict__ k_cache, __hip_bfloat16* __restrict__ v_cache, const int4* __restrict__ pos4,
    const double* __restrict__ inv_freq, int64_t slot0, int n, int n_q_heads, int n_kv_heads, size_t head_stride_elems,
    int rope_mode, int s0, int s01, int gx_k, int nb_k, int nb_q, int blk0, int n_blk,
    const float2* __restrict__ cs_tab) {
  __shared__ __attribute__((aligned(16))) char sT[VG * VT_SROW<D>];
  using T = __hip_bfloat16;
  int b = blockIdx.x;
  if (b < nb_k) {
    append_rows<T, D>(b % gx_k, b / gx_k, 0, k_in, v_in, k_cache, v_cache, pos4, inv_freq, slot0, n, n_kv_heads,
                         head_stride_elems, rope_mode, s0, s01, cs_tab);
    return;
  }
  b -= nb_k;
  if (b < nb_q) {
    rope_rows<T, D>(b, q, pos4, inv_freq, slot0, n, n_q_heads, rope_mode, s0, s01, cs_tab);
    return;
  }
  b -= nb_q;
  append_v_t_group<D>(sT, blk0 + b % n_blk, b / n_blk, v_in, v_cache, slot0, n, n_kv_heads, head_stride_elems);
}

// ---------------------------------------------------------------------------------
// Compaction gather over all layers: new[l][K|V][h][j] = old[l][K|V][h][src[j]],
// K re-rotated by row turn[j] - 1 of dtab where turn[j] != 0.  old and new are the two halves of the
// ping-pong store, so no row is overwritten before it is read.
// Token groups (ROWS tokens) below x0 are not moved: the caller knows that the new half holds them already (tokens
// that two evictions in a row left in place, unshifted: the sink text at the front of a stream in steady state).
// Bound by memory.  A table row belongs to a shift, not to a token, so a workgroup's 32 tokens mostly share one 512-byte row
// out of L1 (with a row per token the table was twice the K row it turned: 28 layers at 4.5k tokens 90.7 -> 84 us).
// grid: (ceil(n_new / ROWS) - x0, n_kv_heads, 2 * n_layers)
// ---------------------------------------------------------------------------------
template <typename T, int D>
__global__ __launch_bounds__(256) void k_compact(const T* __restrict__ old_base, T* __restrict__ new_base,
                                                 const int32_t* __restrict__ src, const int32_t* __restrict__ turn,
                                                 const float2* __restrict__ dtab, int n_new,
                                                 size_t head_stride_elems, size_t tensor_stride_elems, int rotate,
                                                 int v_blocked, int x0) {
  using G = RowGeom<T, D>;
  const int bx = (int)blockIdx.x + x0;   // token group; the groups below x0 stay where they are
  const int h = blockIdx.y;
  const int which = blockIdx.z & 1;   // z = 2 * layer + which, tensors are laid out in that order
  const size_t plane = (size_t)blockIdx.z * tensor_stride_elems + (size_t)h * head_stride_elems;
  typedef __attribute__((__vector_size__(4 * sizeof(unsigned)))) unsigned u32x4;
  if constexpr (sizeof(T) == 2) {
    if (which == 1 && v_blocked) {
      // V in the blocked V^T layout.  The workgroup moves the same tokens as a workgroup of K rows (32 at head_dim
      // 128, 64 at 64): 512 block rows of 16 bytes, two per thread (block p, head dim d), consecutive lanes on
      // consecutive rows.  A new block whose 8 tokens were consecutive in the old cache and started at a multiple of
      // 8 is a copy of an old block, contiguous on both sides (the rule when runs of 8 k tokens leave).  Consecutive but
      // off by some tokens (the rule behind a run of any other length) it is two old block rows, shifted together in
      // registers; only blocks across the end of a run, one per run, gather their elements one by one.  (The source
      // index is the same for the 64 lanes of a wavefront: scalar loads and scalar branches.)
      // Bound by memory; 28 layers of 4 kv heads at about 4.5k retained tokens, runs that are no multiple of 8:
      // 170 us with all those blocks gathered -> 91, what runs of 8 k tokens take.
      static_assert(G::ROWS / 8 * D == 512, "K rows and V^T blocks share the grid");
      const unsigned short* so = (const unsigned short*)old_base + plane;
      unsigned short* sn = (unsigned short*)new_base + plane;
      u32x4 w[2], w_next[2];
      int off[2];
      bool live[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int p = __builtin_amdgcn_readfirstlane((threadIdx.x + 256 * i) / D), d = threadIdx.x % D;
        const int jc = bx * G::ROWS + 8 * p;
        live[i] = jc < n_new;   // a block wholly past the end: nothing to move
        off[i] = 0;
        if (!live[i]) continue;
        const int sa = src[jc];
        if (jc + 7 < n_new && src[jc + 7] == sa + 7) {
          off[i] = sa & 7;
          if (off[i] == 0) {
            w[i] = __builtin_nontemporal_load((const u32x4*)(so + vt_elem<D>(sa, d)));
          } else {   // (each old block row is read twice: kept in the caches)
            w[i] = *(const u32x4*)(so + vt_elem<D>(sa - off[i], d));
            w_next[i] = *(const u32x4*)(so + vt_elem<D>(sa - off[i] + 8, d));
          }
        } else {
          unsigned short e[8];
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            e[j] = 0;
            if (jc + j < n_new) e[j] = so[vt_elem<D>(src[jc + j], d)];
          }
          w[i][0] = e[0] | ((uint32_t)e[1] << 16), w[i][1] = e[2] | ((uint32_t)e[3] << 16);
          w[i][2] = e[4] | ((uint32_t)e[5] << 16), w[i][3] = e[6] | ((uint32_t)e[7] << 16);
        }
      }
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int p = __builtin_amdgcn_readfirstlane((threadIdx.x + 256 * i) / D), d = threadIdx.x % D;
        if (!live[i]) continue;
        if (off[i] != 0) {
          uint32_t y[8] = {w[i][0], w[i][1], w[i][2], w[i][3], w_next[i][0], w_next[i][1], w_next[i][2], w_next[i][3]};
          if (off[i] & 4) {
#pragma unroll
            for (int k = 0; k < 6; ++k) y[k] = y[k + 2];
          }
          if (off[i] & 2) {
#pragma unroll
            for (int k = 0; k < 5; ++k) y[k] = y[k + 1];
          }
          if (off[i] & 1) {
#pragma unroll
            for (int k = 0; k < 4; ++k) y[k] = __builtin_amdgcn_alignbit(y[k + 1], y[k], 16);
          }
          w[i] = u32x4{y[0], y[1], y[2], y[3]};
        }
        *(u32x4*)(sn + vt_elem<D>((int64_t)bx * G::ROWS + 8 * p, d)) = w[i];
      }
      return;
    }
  }
  const int j = bx * G::ROWS + threadIdx.x / G::TPR;
  if (j >= n_new) return;
  const int t = threadIdx.x % G::TPR;
  const T* s = old_base + plane + (size_t)src[j] * D;
  const int row = which == 0 && rotate ? turn[j] : 0;
  T* d = new_base + plane + (size_t)j * D;
  Vec16<T> lo, hi;
  // the old buffer is read once and dead afterwards: non-temporal loads (16 bytes as a native vector); measured
  // 92.8 -> 90 us for 28 layers at 5.1k retained tokens, non-temporal stores on top of that: no change
  static_assert(sizeof(lo.raw) == sizeof(u32x4), "16-byte vectors");
  {
    const u32x4 a = __builtin_nontemporal_load((const u32x4*)(s + t * G::EPV));
    const u32x4 b = __builtin_nontemporal_load((const u32x4*)(s + D / 2 + t * G::EPV));
    __builtin_memcpy(&lo.raw, &a, 16);
    __builtin_memcpy(&hi.raw, &b, 16);
  }
  if (which == 0 && row != 0) {
    const float2* cs = dtab + (size_t)(row - 1) * (D / 2) + t * G::EPV;
#pragma unroll
    for (int e = 0; e < Vec16<T>::N; ++e) {
      const float2 r = cs[e];
      const float a = lo.get(e), b = hi.get(e);
      lo.set(e, a * r.x - b * r.y);
      hi.set(e, b * r.x + a * r.y);
    }
  }
  *(decltype(lo.raw)*)(d + t * G::EPV) = lo.raw;
  *(decltype(hi.raw)*)(d + D / 2 + t * G::EPV) = hi.raw;
}

// The run's cos/sin table, written when the run was registered; NULL where there is none (a run longer than max_q_tokens,
// an eviction since, other slots than the last run's).
const float2* run_table(const sv_cache* c, int stream, int64_t slot0, int n) {
  const StreamState& st = c->st[stream];
  if (!st.cs_tab_valid || st.pending_slot0 != slot0 || st.pending_n != n) return nullptr;
  return c->run_cs(stream);
}

template <typename T, int D>
hipError_t store_tokens_t(const sv_cache* c, int stream, int layer, int64_t slot0, int n, void* q, const void* k, const void* v,
                          hipStream_t s) {
  using G = RowGeom<T, D>;
  const int cur = c->st[stream].cur, Hq = c->cfg.n_q_heads, Hkv = c->cfg.n_kv_heads;
  const size_t off = (size_t)stream * (size_t)c->cfg.capacity_tokens;
  const int s0 = c->cfg.mrope_sections[0], s01 = s0 + c->cfg.mrope_sections[1];
  const int nb_k = (n + G::ROWS - 1) / G::ROWS * Hkv;
  const int nb_q = q && c->cfg.rope_mode != SV_ROPE_NONE ? (int)(((int64_t)n * Hq + G::ROWS - 1) / G::ROWS) : 0;
  hipLaunchKernelGGL((k_store_tokens<T, D>), dim3(2 * nb_k + nb_q), dim3(256), 0, s, (T*)q, (const T*)k, (const T*)v,
                     (T*)c->kv_ptr(stream, cur, layer, 0), (T*)c->kv_ptr(stream, cur, layer, 1),
                     c->meta[cur].pos4 + off, c->inv_freq, slot0, n, Hq, Hkv, c->head_stride / sizeof(T),
                     c->cfg.rope_mode, s0, s01, nb_k, run_table(c, stream, slot0, n));
  return hipGetLastError();
}

template <typename T, int D>
hipError_t rope_apply_t(const sv_cache* c, int stream, int64_t slot0, int n, void* q, void* k, hipStream_t s) {
  using G = RowGeom<T, D>;
  const int cur = c->st[stream].cur;
  const size_t off = (size_t)stream * (size_t)c->cfg.capacity_tokens;
  const int s0 = c->cfg.mrope_sections[0], s01 = s0 + c->cfg.mrope_sections[1];
  void* ptrs[2] = {q, k};
  const int heads[2] = {c->cfg.n_q_heads, c->cfg.n_kv_heads};
  for (int a = 0; a < 2; ++a) {
    if (!ptrs[a]) continue;
    const int h = heads[a];
    auto launch = [&](auto kernel, int64_t workgroups) {
      hipLaunchKernelGGL(kernel, dim3((unsigned)workgroups), dim3(256), 0, s, (T*)ptrs[a], c->meta[cur].pos4 + off, c->inv_freq, slot0, n,
                         h, c->cfg.rope_mode, s0, s01, run_table(c, stream, slot0, n));
    };
    const int64_t blocks = (n + G::ROWS - 1) / G::ROWS, full = (int64_t)n * h / G::ROWS;
    // The more heads per thread that leave some 400 workgroups (us, 1, 2 and 4 heads: 2000 x 28 8.2, 7.75 and 7.5, 5000 x 8 6.3, 6.25 and
    // 6.6, 3000 x 12 6.1, 6.0 and 6.1, 700 x 28 4.4, 4.2 and 4.2), but with at most a quarter of a token's places empty, whose threads
    // load a row that is there again (1, 2 and 4 heads: 131000 tokens of one head of 128 15.1, 15.3 and 16.7, 95000 of two of
    // 64 11.0, 8.7 and 9.3, 26000 of five of 128 14.1, 12.3 and 14.6, 29000 of three 10.7, 9.8 and 8.0, 22000 of six 14.6, 11.3 and 11.5).
    // fp32 with one head each: rows as they lie are the faster way (28 heads of 128, 126 tokens 3.20 and 3.32, 255 3.85 and 3.98; bf16 is
    // 1 % slower so).
    if (full >= 1600 && 3 * ((h + 3) / 4) <= h) launch(k_rope_rows<T, D, 4>, blocks * ((h + 3) / 4));
    else if (full >= 600 && h >= 2) launch(k_rope_rows<T, D, 2>, blocks * ((h + 1) / 2));
    else if constexpr (sizeof(T) == 4) launch(k_rope_rows_flat<T, D>, ((int64_t)n * h + G::ROWS - 1) / G::ROWS);
    else launch(k_rope_rows<T, D, 1>, blocks * h);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <typename T, int D>
hipError_t compact_t(const sv_cache* c, int stream, int64_t n_new, int64_t n_still, hipStream_t s) {
  using G = RowGeom<T, D>;
  const int cur = c->st[stream].cur;
  const size_t off = (size_t)stream * (size_t)c->cfg.capacity_tokens;
  const int rotate = c->cfg.rope_mode != SV_ROPE_NONE;
  float2* dtab = c->dtab + off * (D / 2);   // rows of the tokens with a shift, written by the eviction scan
  const int groups = (int)((n_new + G::ROWS - 1) / G::ROWS), x0 = (int)std::min<int64_t>(n_still / G::ROWS, groups);
  if (x0 == groups) return hipSuccess;
  dim3 grid((unsigned)(groups - x0), c->cfg.n_kv_heads, 2 * c->cfg.n_layers);
  hipLaunchKernelGGL((k_compact<T, D>), grid, dim3(256), 0, s, (const T*)c->kv_ptr(stream, cur, 0, 0),
                     (T*)c->kv_ptr(stream, cur ^ 1, 0, 0), c->src + off, c->turn + off, dtab, (int)n_new,
                     c->head_stride / sizeof(T), c->tensor_stride / sizeof(T), rotate, c->v_blocked ? 1 : 0, x0);
  return hipGetLastError();
}

}  // namespace

#define SV_DISPATCH(fn, ...)                                                                   \
  do {                                                                                         \
    if (c->cfg.dtype == SV_DTYPE_F32) {                                                        \
      return c->cfg.head_dim == 64 ? fn<float, 64>(__VA_ARGS__) : fn<float, 128>(__VA_ARGS__); \
    }                                                                                          \
    return c->cfg.head_dim == 64 ? fn<__hip_bfloat16, 64>(__VA_ARGS__)                         \
                                 : fn<__hip_bfloat16, 128>(__VA_ARGS__);                       \
  } while (0)

hipError_t launch_rope_apply(const sv_cache* c, int stream, int64_t slot0, int n, void* q, void* k,
                             hipStream_t s) {
  SV_DISPATCH(rope_apply_t, c, stream, slot0, n, q, k, s);
}

hipError_t launch_compact(const sv_cache* c, int stream, int64_t n_new, int64_t n_still, hipStream_t s) {
  SV_DISPATCH(compact_t, c, stream, n_new, n_still, s);
}

template <int D>
static hipError_t store_tokens_vt(const sv_cache* c, int stream, int layer, int64_t slot0, int n, void* q, const void* k,
                                  const void* v, hipStream_t s) {
  using G = RowGeom<__hip_bfloat16, D>;
  const int Hq = c->cfg.n_q_heads, Hkv = c->cfg.n_kv_heads, cur = c->st[stream].cur;
  const int gx_k = (n + G::ROWS - 1) / G::ROWS, nb_k = gx_k * Hkv;
  const bool rot_q = q && c->cfg.rope_mode != SV_ROPE_NONE;
  const int nb_q = rot_q ? (int)(((int64_t)n * Hq + G::ROWS - 1) / G::ROWS) : 0;
  const int blk0 = (int)(slot0 / VG), n_blk = (int)((slot0 + n - 1) / VG) - blk0 + 1;   // groups of 32 slots
  // what the kernel's packed arguments can carry, and the layout it relies on (V plane right behind the K plane)
  if (Hkv > 255 || Hq > 65535 || c->head_stride / 2 > 0xffffffffull || (int64_t)n * Hq > 0x7fffffff ||
      c->kv_ptr(stream, cur, layer, 1) != c->kv_ptr(stream, cur, layer, 0) + (size_t)Hkv * c->head_stride)
    return hipErrorInvalidValue;
  const float2* cs_tab = nullptr;
  if (c->cfg.rope_mode != SV_ROPE_NONE) {   // the run's cos/sin table, written when the run was registered
    cs_tab = run_table(c, stream, slot0, n);
    if (!cs_tab) {   // positions and sincos
      const size_t off = (size_t)stream * (size_t)c->cfg.capacity_tokens;
      hipLaunchKernelGGL(k_store_tokens_vt_pos<D>, dim3(nb_k + nb_q + n_blk * Hkv), dim3(256), 0, s, (__hip_bfloat16*)q,
                         (const __hip_bfloat16*)k, (const __hip_bfloat16*)v,
                         (__hip_bfloat16*)c->kv_ptr(stream, cur, layer, 0), (__hip_bfloat16*)c->kv_ptr(stream, cur, layer, 1),
                         c->meta[cur].pos4 + off, c->inv_freq, slot0, n, Hq, Hkv, c->head_stride / 2, c->cfg.rope_mode,
                         c->cfg.mrope_sections[0], c->cfg.mrope_sections[0] + c->cfg.mrope_sections[1], gx_k, nb_k, nb_q,
                         blk0, n_blk, (const float2*)nullptr);
      return hipGetLastError();
    }
  }
  const uint32_t shape = (uint32_t)rot_q << 1 | (uint32_t)Hkv << 8 | (uint32_t)Hq << 16;
  hipLaunchKernelGGL(k_store_tokens_vt<D>, dim3(nb_k + nb_q + n_blk * Hkv), dim3(256), 0, s, (__hip_bfloat16*)q,
                     (const __hip_bfloat16*)k, (const __hip_bfloat16*)v, (__hip_bfloat16*)c->kv_ptr(stream, cur, layer, 0),
                     cs_tab, (int)slot0, n, (uint32_t)(c->head_stride / 2), shape);
  return hipGetLastError();
}

hipError_t launch_store_tokens(const sv_cache* c, int stream, int layer, int64_t slot0, int n, void* q, const void* k,
                               const void* v, hipStream_t s) {
  if (c->v_blocked)
    return c->cfg.head_dim == 64 ? store_tokens_vt<64>(c, stream, layer, slot0, n, q, k, v, s)
                                 : store_tokens_vt<128>(c, stream, layer, slot0, n, q, k, v, s);
  SV_DISPATCH(store_tokens_t, c, stream, layer, slot0, n, q, k, v, s);
}

}  // namespace sv
