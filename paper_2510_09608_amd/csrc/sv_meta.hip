// Integer side of the path: registering new tokens, and the eviction scan that
// turns the three budgets of Sec. 2.1 into a gather list plus new contiguous
// positions (Sec. 2.1, "Contiguous RoPE").  Everything here is exact integer work.

#include <algorithm>

#include "sv_internal.h"

namespace sv {
namespace {

// cos/sin of a rotary angle, as the row movers compute them: angle in double, for bf16 data sincosf of its float value
__device__ __forceinline__ float2 angle_cs(int p, double freq, int f32_data) {
  const double ang = (double)p * freq;
  float2 cs;
  if (f32_data) {
    double sd, cd;
    sincos(ang, &sd, &cd);
    cs = make_float2((float)cd, (float)sd);
  } else {
    sincosf((float)ang, &cs.y, &cs.x);
  }
  return cs;
}
// metadata of token j of a run that begins at `slot0`; next: the scalar position counter before the run
__device__ __forceinline__ void write_token(const MetaPtrs& m, int64_t slot0, int j, int next, int type, int64_t gid, int64_t rank,
                                            int rope3d, int blk, int gT, int gH, int gW) {
  const int64_t slot = slot0 + j;
  m.gid[slot] = gid;
  m.rank[slot] = rank;
  m.type[slot] = (uint8_t)type;
  if (rope3d && blk >= 0) {
    const int lt = j / (gH * gW), lh = (j / gW) % gH, lw = j % gW;
    m.blk[slot] = blk;
    m.local4[slot] = make_short4((short)lt, (short)lh, (short)lw, (short)max(gT, max(gH, gW)));
    m.pos4[slot] = make_int4(next + lt, next + lh, next + lw, next);
  } else {
    const int p = rope3d ? next + j : (int)slot;
    m.blk[slot] = -1;
    m.local4[slot] = make_short4(0, 0, 0, 1);
    m.pos4[slot] = make_int4(p, p, p, p);
  }
}
// the position that pair i of token j of the run turns by
__device__ __forceinline__ int angle_pos(int64_t slot0, int j, int i, int next, int rope3d, int blk, int gH, int gW, int s0, int s01) {
  if (!rope3d) return (int)(slot0 + j);   // 1-D: position == slot
  if (blk < 0) return next + j;
  const int lt = j / (gH * gW), lh = (j / gW) % gH, lw = j % gW;
  return next + (i < s0 ? lt : (i < s01 ? lh : lw));
}

// ---------------------------------------------------------------------------------
// New tokens: slot, arrival id, rank within type, block coordinates and position.
// The scalar position counter lives in device memory as a two-entry ping-pong
// (read next_in, write next_out) so that no thread can read a value another
// block has already advanced.
// ---------------------------------------------------------------------------------
__global__ void k_meta_append(MetaPtrs m, const int32_t* __restrict__ next_in, int32_t* __restrict__ next_out,
                              int64_t slot0, int n, int64_t gid0, int64_t rank_text0, int64_t rank_vis0,
                              int type_uniform, TypeMask mask, int rope3d, int blk, int gT, int gH, int gW,
                              const double* __restrict__ inv_freq, int half, int s0, int s01, int f32_data, int32_t* __restrict__ n_dev,
                              float2* __restrict__ cs_tab, int ahead) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  const int next = *next_in - ahead;   // text tokens that were registered ahead are taken back
  if (cs_tab != nullptr && j < n * half) {
    // cos/sin of every new token's rotary angles (thread = one token, one frequency)
    const int tok = j / half, i = j % half;
    cs_tab[j] = angle_cs(angle_pos(slot0, tok, i, next, rope3d, blk, gH, gW, s0, s01), inv_freq[i], f32_data);
  }
  if (j == 0) {
    int adv;
    if (!rope3d) adv = (int)(slot0 + n) - next;  // 1-D: position == slot
    else if (blk >= 0) adv = max(gT, max(gH, gW));
    else adv = n;
    *next_out = next + adv;
    *n_dev = (int32_t)(slot0 + n);   // the device's own token count (cross-checked by sv_cache_retained)
  }
  if (j >= n) return;
  int type;
  int64_t rank;
  if (type_uniform >= 0) {
    type = type_uniform;
    rank = (type == SV_TEXT ? rank_text0 : rank_vis0) + j;
  } else {
    type = (mask.w[j >> 5] >> (j & 31)) & 1;
    int vis_before = 0;
    for (int w = 0; w < (j >> 5); ++w) vis_before += __popc(mask.w[w]);
    vis_before += __popc(mask.w[j >> 5] & ((1u << (j & 31)) - 1u));
    rank = type == SV_VISION ? rank_vis0 + vis_before : rank_text0 + (j - vis_before);
  }
  write_token(m, slot0, j, next, type, gid0 + j, rank, rope3d, blk, gT, gH, gW);
}

// ---------------------------------------------------------------------------------
// The next n_ahead text tokens of each of several streams (decode steps of a batch): what k_meta_append writes for a run of them,
// one workgroup of one wavefront per stream and token, so that a step of 16 streams costs one launch and not 16 in a row (2.1 us
// and a gap each: 0.7 of the 3.4 ms that a second of 16 ragged streams took at 4 layers).  What a decoded token's registration
// writes (arrival id, rank, position, rotary cos/sin) follows from the stream's counts alone, so kAhead steps share one launch: the
// steps behind the first find their token registered unless the stream was appended to or evicted in between, which starts from
// the tokens that are really there.  A token's cos/sin have a row by slot: a captured step may hold no registration, and when it
// is replayed later steps have registered other tokens.  A launch in every step, back to back with the attention, took 5.1 us: 16 ragged
// streams, 4 layers, 16 tokens 2714 -> 2657 us; one stream, 28 layers, 256 vision and 16 text tokens layer by layer 3811 -> 3770.
// ---------------------------------------------------------------------------------
struct TokenRow {
  int64_t gid, rank;   // arrival id, rank among the stream's text tokens
  int32_t slot;
  int32_t stream;      // stream << 2 | live half << 1 | live entry of the position ping-pong
};
constexpr int kMaxTokenRows = 64;
struct TokenTable {
  TokenRow r[kMaxTokenRows];
};
__global__ __launch_bounds__(64) void k_meta_tokens(MetaPtrs m0, MetaPtrs m1, int32_t* __restrict__ next_pos,
                                                    float2* __restrict__ slot_cs, const double* __restrict__ inv_freq,
                                                    int32_t* __restrict__ n_dev, int64_t capacity, int half, int rope3d,
                                                    int rope_none, int f32_data, TokenTable tab) {
  const TokenRow r = tab.r[blockIdx.x];
  const int sid = r.stream >> 2, parity = r.stream & 1, lane = threadIdx.x, j = blockIdx.y, n_ahead = gridDim.y;
  const int next = next_pos[2 * sid + parity];
  const int p = (rope3d ? next : r.slot) + j;   // 1-D: position == slot
  const int64_t at = (int64_t)sid * capacity + r.slot + j;
  if (lane < half) slot_cs[at * half + lane] = rope_none ? make_float2(1.f, 0.f) : angle_cs(p, inv_freq[lane], f32_data);
  if (lane == 0) {
    const bool second = (r.stream & 2) != 0;
    (second ? m1.gid : m0.gid)[at] = r.gid + j;
    (second ? m1.rank : m0.rank)[at] = r.rank + j;
    (second ? m1.type : m0.type)[at] = (uint8_t)SV_TEXT;
    (second ? m1.blk : m0.blk)[at] = -1;
    (second ? m1.local4 : m0.local4)[at] = make_short4(0, 0, 0, 1);
    (second ? m1.pos4 : m0.pos4)[at] = make_int4(p, p, p, p);
    if (j == n_ahead - 1) {
      next_pos[2 * sid + (parity ^ 1)] = p + 1;
      n_dev[sid] = r.slot + n_ahead;   // the device's own token count
    }
  }
}

// ---------------------------------------------------------------------------------
// Eviction scan, several workgroups per stream.
//
// keep(i)  : text  -> rank < n_sink or rank >= text_lo     (sink + recent text)
//            vision-> rank >= vis_lo                         (recent vision)
// dst(i)   : exclusive prefix count of keep
// base'(i) : exclusive prefix sum over kept tokens of the position advance, where a
//            text token advances by 1 and a vision block advances by its extent at
//            its last retained token.  With every token its own block of extent 1
//            (1-D mode) base' equals dst.
// Survivors' metadata is written compacted to `out`; src[dst] = i is the gather
// list for the K/V move.  Re-rotation: the shift base - base' of a token, one scalar even in 3-D mode because t, h and w
// shift together, turns pair i by -(shift * inv_freq[i]).  The survivors of a wavefront nearly always share one shift, so
// every distinct shift of a wavefront gets one row dtab[r][pair] = (cos, -sin) of shift * inv_freq[pair] (so that the mover
// applies the formula of a forward rotation), r being the slot of the first token that has it, and
// turn[dst] = r + 1, or 0 for a token that keeps its position.
//
// Workgroup w owns the tokens [w * span, (w + 1) * span), span = passes x 256, one token per thread and pass.
//   1. It counts its kept tokens and their advances (within a wavefront: ballot + popcount, and a scan by DPP adds whose
//      last lane is the sum and which step 3 uses again) and
//      publishes the two totals as 64-bit words {value, launch tag} with relaxed device-scope atomic stores.
//   2. It reads the words of all workgroups before it (by other wavefronts than the one that published, where it can: loads
//      of a wavefront return behind the acknowledgement of its stores), again and again until each carries this
//      launch's tag (a word is its own ready flag: a 64-bit access is single-copy atomic and a word is written once
//      per launch; the writers wait for nothing and are dispatched earlier), and sums them: the carry.
//      The tag lives in device memory behind the words: a launch uses the stored value + 1 (never 0), and the last
//      workgroup, which ends only after every other one has published, i.e. read the tag, stores the new value and
//      zeroes the words of the workgroups this launch did not have; so a word left over from an earlier launch
//      carries the tag before this one or none, and nothing depends on host state (a captured launch can be replayed).
//   3. It adds the carry and the wavefronts before and writes the survivors' metadata.
//   4. It writes the table rows: the 64 sincos of a shift at once (lane = rotary pair, angle in double).
// Bound by its chain of latencies: tokens in, totals across, survivors out (a microsecond each).  With shuffles through LDS
// for the sums and the scan (each step a round trip of 100 cycles) and a 512-byte table row per token, 64 of them one after
// the other, it took 11 to 13 us at 5 to 18 thousand tokens and 7 at 60; this way 5.3 to 6.2 and 3.2.
// At most kScanMaxWG workgroups: longer caches take several passes per workgroup.
//
// Registration.  A second's eviction is followed by the registration of its vision and of its text tokens, which needs nothing
// from it but the position counter.  Where the caller knows them (sv_stream_step), `n_reg` more workgroups without tokens of their
// own, behind the others, wait for the totals as those do and write what k_meta_append would have, in two launches (the smallest
// second, fp32, 1 layer, 16 + 4 tokens, where every launch is 3 to 4 us of the host: 42.9 -> 38.9 us).  An instantiation of its own
// (R: one Registration, or nothing): in a plain eviction's it cost 34 spilled SGPRs.
// ---------------------------------------------------------------------------------
constexpr int kScanThreads = 256;
constexpr int kScanWaves = kScanThreads / 64;
constexpr int kScanPollLimit = 1 << 16;

struct ScanTok {
  int type, blk, old_base, type_n, blk_n;
  int64_t rank, gid, rank_n;
  short4 loc;
};

// inclusive sum over the lanes of a wavefront: rows of 16, then the rows' last lanes onto the rows behind
__device__ __forceinline__ int wave_scan(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);   // row_shr:1
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);   // row_shr:2
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);   // row_shr:4
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);   // row_shr:8
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1 and 3
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2 and 3
  return x;
}

struct Registration {
  int n_reg;
  NewRuns runs;
  int rope3d, s0, s01;
  float2* cs_tab;
};

template <typename... R>
__global__ __launch_bounds__(kScanThreads) void k_evict_scan(MetaPtrs in, MetaPtrs out, int32_t* __restrict__ src,
                                                             int32_t* __restrict__ turn, float2* __restrict__ dtab,
                                                             const double* __restrict__ inv_freq, int half,
                                                             int f32_data, int32_t* __restrict__ next_out,
                                                             int32_t* __restrict__ n_out, int n_old, int64_t n_sink,
                                                             int64_t text_lo, int64_t vis_lo, int passes,
                                                             unsigned long long* agg, R... reg) {
  constexpr bool REG = sizeof...(R) > 0;
  __shared__ int2 sh_pass[kScanWaves], sh_all[kScanWaves], sh_carry[kScanWaves];   // {kept tokens, advance}
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int w = blockIdx.x, span = passes * kScanThreads;
  const int first = w * span;
  const uint32_t tag_old = (uint32_t)agg[2 * kScanWords];   // written by the launch before this one
  const double my_freq = dtab != nullptr && lane < half ? inv_freq[lane] : 0.0;
  bool registers = false;
  if constexpr (REG) registers = w >= (int)gridDim.x - (reg, ...).n_reg;

  // The token and its successor (the look-ahead for "last of its block").  Indices are clamped instead of guarded
  // and the rule below is written without short-circuits, so that every load is unconditional and all nine go out
  // together: guarded, the compiler sinks each load into the branch that uses it, one memory round trip after another.
  auto load_tok = [&](int i) {
    ScanTok t;
    const int ic = min(i, n_old - 1), in_ = min(i + 1, n_old - 1);
    t.type = in.type[ic];
    t.rank = in.rank[ic];
    t.blk = in.blk[ic];
    t.gid = in.gid[ic];
    t.loc = in.local4[ic];
    t.old_base = in.pos4[ic].w;
    t.type_n = in.type[in_];
    t.rank_n = in.rank[in_];
    t.blk_n = in.blk[in_];
    return t;
  };
  auto kept = [&](int type, int64_t rank) {
    const bool text_ok = (rank < n_sink) | (rank >= text_lo), vis_ok = rank >= vis_lo;
    return type == SV_TEXT ? text_ok : vis_ok;
  };
  auto eval = [&](const ScanTok& t, int i, bool& keep, int& adv) {
    keep = (i < n_old) & kept(t.type, t.rank);
    // last retained token of its vision block?  (a token without a block, blk < 0, is its own block)
    const bool next_stays = (t.blk >= 0) & (t.blk_n == t.blk) & (i + 1 < n_old) & kept(t.type_n, t.rank_n);
    const int adv_vis = next_stays ? 0 : (int)t.loc.w;
    adv = keep ? (t.type == SV_TEXT ? 1 : adv_vis) : 0;
  };

  // ---- 1. totals of this workgroup's tokens; pass 0 stays in registers for step 3
  const ScanTok t0 = load_tok(first + tid);
  bool keep0;
  int adv0;
  eval(t0, first + tid, keep0, adv0);
  const unsigned long long bal0 = __ballot(keep0);
  const int incl0 = wave_scan(adv0);
  int2 all = make_int2(__popcll(bal0), __builtin_amdgcn_readlane(incl0, 63));
  if (lane == 0) sh_pass[wave] = all;
  if (passes > 1) {
    int more = 0;
    for (int p = 1; p < passes; ++p) {
      const int i = first + p * kScanThreads + tid;
      bool keep;
      int adv;
      eval(load_tok(i), i, keep, adv);
      all.x += __popcll(__ballot(keep));
      more += adv;
    }
    all.y += __builtin_amdgcn_readlane(wave_scan(more), 63);
  }
  if (lane == 0) sh_all[wave] = all;
  uint32_t tag = tag_old + 1u == 0u ? 1u : tag_old + 1u;
  asm volatile("" : "+s"(tag));   // every wavefront has the old tag before the workgroup publishes
  __syncthreads();
  const unsigned long long tag_hi = (unsigned long long)tag << 32;
  if (tid == kScanThreads - 1) {
    int tc = 0, ta = 0;
#pragma unroll
    for (int k = 0; k < kScanWaves; ++k) tc += sh_all[k].x, ta += sh_all[k].y;
    __hip_atomic_store(agg + 2 * w, tag_hi | (uint32_t)tc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(agg + 2 * w + 1, tag_hi | (uint32_t)ta, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  // ---- 2. carry: totals of all workgroups before this one
  {
    int cc = 0, ca = 0;
    bool lost = false;
    for (int b0 = 64 * wave; b0 < w; b0 += kScanThreads) {
      const int b = min(b0 + lane, w - 1);
      unsigned long long wc, wa;
      int it = 0;
      bool miss;
#pragma clang loop unroll(disable)
      do {
        if (it > 8) __builtin_amdgcn_s_sleep(1);
        wc = __hip_atomic_load(agg + 2 * b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        wa = __hip_atomic_load(agg + 2 * b + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        miss = __ballot((((uint32_t)(wc >> 32) ^ tag) | ((uint32_t)(wa >> 32) ^ tag)) != 0) != 0;
      } while (miss && ++it < kScanPollLimit);
      lost = lost || miss;
      if (b0 + lane < w) cc += (int)(uint32_t)wc, ca += (int)(uint32_t)wa;
    }
    if (64 * wave < w) {
      cc = __builtin_amdgcn_readlane(wave_scan(cc), 63), ca = __builtin_amdgcn_readlane(wave_scan(ca), 63);
      // a word that never showed its tag (the limit is far beyond any launch's length): this workgroup writes
      // nothing, and the failure shows in the device's own token count, which sv_cache_retained checks against the host's
      if (lost) cc = INT32_MIN / 8;
    }
    if (lane == 0) sh_carry[wave] = make_int2(cc, ca);
  }
  __syncthreads();
  int run_cnt = 0, run_adv = 0;
#pragma unroll
  for (int k = 0; k < kScanWaves; ++k) run_cnt += sh_carry[k].x, run_adv += sh_carry[k].y;
  if (run_cnt < 0) {
    if (tid == 0) *n_out = -1;
    return;
  }

  // ---- 3. and 4. own tokens on top of the carry, survivors out, table rows
  for (int p = 0; p < passes && !registers; ++p) {
    const int i = first + p * kScanThreads + tid;
    ScanTok t = t0;
    bool keep = keep0;
    int adv = adv0, incl = incl0;
    unsigned long long bal = bal0;
    if (p > 0) {
      t = load_tok(i);
      eval(t, i, keep, adv);
      bal = __ballot(keep), incl = wave_scan(adv);
      __syncthreads();   // the totals of the pass before have been read
      if (lane == 63) sh_pass[wave] = make_int2(__popcll(bal), incl);
      __syncthreads();
    }
    int seg_cnt = run_cnt, seg_adv = run_adv;
#pragma unroll
    for (int k = 0; k < kScanWaves; ++k) {
      const int2 x = sh_pass[k];
      if (k < wave) seg_cnt += x.x, seg_adv += x.y;
      run_cnt += x.x, run_adv += x.y;
    }
    const int d = seg_cnt + __popcll(bal & ((1ull << lane) - 1ull));
    const int nb = seg_adv + (incl - adv);
    const int shift = t.old_base - nb;
    if (keep) {
      out.gid[d] = t.gid;
      out.rank[d] = t.rank;
      out.type[d] = (uint8_t)t.type;
      out.blk[d] = t.blk;
      out.local4[d] = t.loc;
      out.pos4[d] = make_int4(nb + t.loc.x, nb + t.loc.y, nb + t.loc.z, nb);
      src[d] = i;
    }
    int row = 0;
    if (dtab != nullptr) {
      unsigned long long m = __ballot(keep && shift != 0);
      while (m) {   // uniform over the wavefront: one distinct shift each time
        const int l = __ffsll((long long)m) - 1;
        const int sq = __builtin_amdgcn_readlane(shift, l), dd = __builtin_amdgcn_readlane(d, l);
        const bool same = keep && shift == sq;
        m &= ~__ballot(same);
        if (same) row = dd + 1;
        if (lane < half) {
          float2 cs;
          const double ang = (double)sq * my_freq;
          if (f32_data) {
            double sd, cd;
            sincos(ang, &sd, &cd);
            cs = make_float2((float)cd, (float)-sd);
          } else {
            // bf16 rows: float accuracy is ample, and the double-precision sincos with its large-argument reduction
            // costs microseconds per call; the angle is reduced to [-pi, pi] in double first (error ~1e-13)
            const double turns = rint(ang * 0.15915494309189535);
            const float r = (float)fma(turns, -6.283185307179586, ang);
            float sf, cf;
            sincosf(r, &sf, &cf);
            cs = make_float2(cf, -sf);
          }
          dtab[(size_t)dd * half + lane] = cs;
        }
      }
    }
    if (keep) turn[d] = row;
  }
  int new_cnt = 0, new_adv = 0;   // registered tokens, and what they move the scalar position counter by
  if constexpr (REG) {
    const Registration& g = (reg, ...);
    const NewRuns& runs = g.runs;
    const int adv_vis = g.rope3d && runs.blk >= 0 ? max(runs.gT, max(runs.gH, runs.gW)) : runs.n_vision;
    new_cnt = runs.n_vision + runs.n_text, new_adv = adv_vis + runs.n_text;
    if (registers) {   // the position counter is the sum of all advances
      const int next_text = run_adv + adv_vis;
      const int64_t slot_text = (int64_t)runs.n_kept + runs.n_vision;
      const int at = (w - ((int)gridDim.x - g.n_reg)) * kScanThreads + tid, step = g.n_reg * kScanThreads;
      auto cs_of = [&](int j, int i) {
        const bool vis = j < runs.n_vision;
        const int p = vis ? angle_pos(runs.n_kept, j, i, run_adv, g.rope3d, runs.blk, runs.gH, runs.gW, g.s0, g.s01)
                          : angle_pos(slot_text, j - runs.n_vision, i, next_text, g.rope3d, -1, 1, 1, g.s0, g.s01);
        return angle_cs(p, inv_freq[i], f32_data);
      };
      for (int j = at; j < new_cnt; j += step) {
        if (j < runs.n_vision)
          write_token(out, runs.n_kept, j, run_adv, SV_VISION, runs.gid0 + j, runs.rank_vis0 + j, g.rope3d, runs.blk, runs.gT, runs.gH,
                      runs.gW);
        else
          write_token(out, slot_text, j - runs.n_vision, next_text, SV_TEXT, runs.gid0 + j, runs.rank_text0 + (j - runs.n_vision),
                      g.rope3d, -1, 1, 1, 1);
      }
      if (dtab != nullptr)
        for (int x = at; x < new_cnt * half; x += step) g.cs_tab[x] = cs_of(x / half, x % half);
    }
  }
  if (w == (int)gridDim.x - 1) {
    if (tid == 0) {
      *next_out = run_adv + new_adv;
      *n_out = run_cnt + new_cnt;
      agg[2 * kScanWords] = tag;
    }
    for (int b = (int)gridDim.x + tid; b < kScanWords; b += kScanThreads) agg[2 * b] = 0ull, agg[2 * b + 1] = 0ull;
  }
}

}  // namespace

hipError_t launch_meta_append(const sv_cache* c, int stream, int next_parity, int64_t slot0, int n,
                              int64_t gid0, int64_t rank_text0, int64_t rank_vis0, int type_uniform,
                              const TypeMask* mask, int blk, int gT, int gH, int gW, bool with_cs_tab, hipStream_t s) {
  const size_t off = (size_t)stream * (size_t)c->cfg.capacity_tokens;
  MetaPtrs m = c->meta[c->st[stream].cur];
  m.gid += off, m.rank += off, m.pos4 += off, m.local4 += off, m.blk += off, m.type += off;
  TypeMask mk = {};
  if (mask) mk = *mask;
  const int half = c->cfg.head_dim / 2;
  const int threads = 256, blocks = ((with_cs_tab ? n * half : n) + threads - 1) / threads;
  const int32_t* nin = c->next_pos + 2 * stream + next_parity;
  int32_t* nout = c->next_pos + 2 * stream + (next_parity ^ 1);
  hipLaunchKernelGGL(k_meta_append, dim3(blocks), dim3(threads), 0, s, m, nin, nout, slot0, n, gid0, rank_text0,
                     rank_vis0, type_uniform, mk, c->cfg.rope_mode == SV_ROPE_3D ? 1 : 0, blk, gT, gH, gW,
                     c->inv_freq, half,
                     c->cfg.mrope_sections[0], c->cfg.mrope_sections[0] + c->cfg.mrope_sections[1],
                     c->cfg.dtype == SV_DTYPE_F32 ? 1 : 0, c->n_dev + stream,
                     with_cs_tab ? c->cs_tab + (size_t)stream * c->cs_rows * half : nullptr, c->st[stream].ahead);
  return hipGetLastError();
}

hipError_t launch_meta_tokens(const sv_cache* c, const int32_t* streams, int n_list, int n_ahead, hipStream_t s) {
  for (int r0 = 0; r0 < n_list; r0 += kMaxTokenRows) {
    const int nr = std::min(kMaxTokenRows, n_list - r0);
    TokenTable tab;
    for (int b = 0; b < nr; ++b) {
      const int sid = streams[r0 + b];
      const StreamState& st = c->st[sid];
      tab.r[b] = {st.next_gid, st.n_text, (int32_t)st.len, sid << 2 | st.cur << 1 | st.next_parity};
    }
    hipLaunchKernelGGL(k_meta_tokens, dim3(nr, n_ahead), dim3(64), 0, s, c->meta[0], c->meta[1], c->next_pos, c->dtab,
                       c->inv_freq, c->n_dev, c->cfg.capacity_tokens, c->cfg.head_dim / 2,
                       c->cfg.rope_mode == SV_ROPE_3D ? 1 : 0, c->cfg.rope_mode == SV_ROPE_NONE ? 1 : 0,
                       c->cfg.dtype == SV_DTYPE_F32 ? 1 : 0, tab);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_evict_scan(const sv_cache* c, int stream, int next_parity, int64_t n_old, int64_t n_sink,
                             int64_t text_lo, int64_t vis_lo, const NewRuns* runs, hipStream_t s) {
  const size_t off = (size_t)stream * (size_t)c->cfg.capacity_tokens;
  const int cur = c->st[stream].cur;
  MetaPtrs in = c->meta[cur], out = c->meta[cur ^ 1];
  in.gid += off, in.rank += off, in.pos4 += off, in.local4 += off, in.blk += off, in.type += off;
  out.gid += off, out.rank += off, out.pos4 += off, out.local4 += off, out.blk += off, out.type += off;
  const int half = c->cfg.head_dim / 2;
  const int tiles = (int)((n_old + kScanThreads - 1) / kScanThreads);
  // two cos/sin per thread of the registering workgroups
  const int n_reg = runs ? std::max(1, std::min(kScanMaxReg, ((runs->n_vision + runs->n_text) * half + 2 * kScanThreads - 1) / (2 * kScanThreads))) : 0;
  const int passes = (tiles + kScanMaxWG - 1) / kScanMaxWG;
  const int wgs = (tiles + passes - 1) / passes;
  unsigned long long* agg = c->scan_agg + (size_t)stream * 2 * (kScanWords + 1);
  auto launch = [&](auto kernel, auto... reg) {
    hipLaunchKernelGGL(kernel, dim3(wgs + n_reg), dim3(kScanThreads), 0, s, in, out, c->src + off, c->turn + off,
                       c->cfg.rope_mode != SV_ROPE_NONE ? c->dtab + off * half : nullptr, c->inv_freq, half,
                       c->cfg.dtype == SV_DTYPE_F32 ? 1 : 0, c->next_pos + 2 * stream + (next_parity ^ 1), c->n_dev + stream, (int)n_old,
                       n_sink, text_lo, vis_lo, passes, agg, reg...);
  };
  if (runs)
    launch(k_evict_scan<Registration>,
           Registration{n_reg, *runs, c->cfg.rope_mode == SV_ROPE_3D ? 1 : 0, c->cfg.mrope_sections[0],
                        c->cfg.mrope_sections[0] + c->cfg.mrope_sections[1], c->cs_tab + (size_t)stream * c->cs_rows * half});
  else
    launch(k_evict_scan<>);
  return hipGetLastError();
}

}  // namespace sv
