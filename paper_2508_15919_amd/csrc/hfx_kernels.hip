// Device code of libhfxattn for gfx950 (MI355X): one persistent kernel that drains the
// cost-ordered work items of a scheduled step -- decode ranges (HBM-bound streaming of KV
// pages: the token-generation phase of HFX Section 2.1) and prefill tiles (dense bf16 MFMA
// contraction with a causal mask: its prompt phase) -- plus the split merge, the page gather
// hook, the KV append and the page copy.  Wavefronts are 64 lanes wide; every tiling below is
// written for that.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cstring>
#include <mutex>

#include "hfx_desc.h"
#include "hfx_launch.h"

namespace hfx {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

#define NEG_INF (-__builtin_inff())

struct KArgs {
  const char* desc;      // device descriptor blob (read-only here; the control words go through `ctrl`)
  const __bf16* q;       // [T][Hq][D]
  const __bf16* pool;    // [pages][Hkv][2][16*D]
  float* ws;             // split partials
  __bf16* out;           // [T][Hq][D]
};

template <int D>
struct Smem {
  // prefill: a ring of stage slots of 32 keys (two pages) each: the two pages' K blocks, then their V blocks
  static constexpr int kBlockBytes = HFX_PAGE * D * 2;
  static constexpr int kStageBytes = 4 * kBlockBytes;
  static constexpr int kStages = 4;
  // decode: per-wavefront partial rows [4][16][D + 4] floats (same memory; an item is one or the other)
  static constexpr int kPartStride = D + 4;
  static constexpr int kPartBytes = 4 * 16 * kPartStride * 4;
  static constexpr int kBytes = kStages * kStageBytes > kPartBytes ? kStages * kStageBytes : kPartBytes;
};

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ bf16x8 ld16(const __bf16* p) { return *reinterpret_cast<const bf16x8*>(p); }

// `x` where keep, -inf elsewhere, as a select on the bit pattern: the scores of masked keys may be
// NaN (unused slots hold anything), and the file is compiled with -fno-honor-nans, under which a
// floating-point select of a NaN is not defined.
__device__ __forceinline__ float keep_or_neg_inf(float x, bool keep) {
  const unsigned u = keep ? __builtin_bit_cast(unsigned, x) : 0xff800000u;
  return __builtin_bit_cast(float, u);
}

// Exchange between lane n and lane n ^ 32 with the swap instruction gfx950 has for it (the upper half
// of one register against the lower half of another); a shuffle would go through LDS and put
// its latency, and a wait for every LDS read in flight, into the softmax of every stage.
// swap32(x): {x of the lower-half lane of the pair, x of its upper-half lane}, in both lanes.
// The copies in and out are hidden from the optimizer, which otherwise folds the swap of a value
// with itself, and whatever combines its two results, into the value.
struct Pair32 {
  float lo, hi;
};
__device__ __forceinline__ Pair32 swap32(float x) {
  const unsigned u = __builtin_bit_cast(unsigned, x);
  unsigned u2 = u;
  asm volatile("" : "+v"(u2));
  const auto r = __builtin_amdgcn_permlane32_swap(u, u2, false, false);
  unsigned a = r[0], b = r[1];
  asm volatile("" : "+v"(a), "+v"(b));
  Pair32 p;
  p.lo = __builtin_bit_cast(float, a);
  p.hi = __builtin_bit_cast(float, b);
  return p;
}
__device__ __forceinline__ float max_xor32(float x) {
  const Pair32 p = swap32(x);
  return fmaxf(p.lo, p.hi);
}
__device__ __forceinline__ float sum_xor32(float x) {
  const Pair32 p = swap32(x);
  return p.lo + p.hi;
}

// zero the elements e >= nv of an 8-element bf16 vector (nv may be <= 0 or >= 8)
__device__ __forceinline__ bf16x8 keep_first(bf16x8 v, int nv) {
  const unsigned bits = (1u << min(max(nv, 0), 8)) - 1u;
  u32x4 u = __builtin_bit_cast(u32x4, v);
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const int lo = (int)(bits << (31 - 2 * w)) >> 31, hi = (int)(bits << (30 - 2 * w)) >> 31;   // all ones where kept
    u[w] &= __builtin_amdgcn_perm((unsigned)hi, (unsigned)lo, 0x05040100u);
  }
  return __builtin_bit_cast(bf16x8, u);
}

// ----------------------------------------------------------------------------------------------
// Split merge (runs as its own small launch after the persistent kernel, so the partials are
// ordered by the kernel boundary and no fences or arrival counters are needed).  One workgroup
// per merge unit combines a few rows of a group's partials (m, l, acc):
//   m* = max m_s,  l* = sum l_s 2^(m_s - m*),  out = sum acc_s 2^(m_s - m*) / l*
// (m is kept in the base-2 domain throughout), rounds to bf16 and stores.  A thread owns one
// float4 column of a row; for groups with many splits 8 threads share the splits of that column
// (one row per workgroup) so that all loads are in flight together, for groups with at most 8
// splits one thread takes them all (8 rows per workgroup).
// ----------------------------------------------------------------------------------------------
// The body of the merge for a group whose threads see at most N splits each.
template <int D, int N>
__device__ __forceinline__ void merge_rows(const HfxUnit& un, const HfxGroup& gr, const float* __restrict__ ws, const float* __restrict__ ml,
                                           int Hq, int G, __bf16* __restrict__ out, float* s_max, float* s_l,
                                           f32x4 (*s_acc)[D / 4]) {
  constexpr int C4 = D / 4;                       // float4 columns of a row
  const int tid = threadIdx.x;
  const int col = tid % C4, q = tid / C4;
  const bool wide = N == 8 && gr.nsplit > 8;      // only the first 8 thread rows are used below
  const int SL = wide ? 8 : 1;                    // threads sharing one row's splits
  const int sl = wide ? q : 0;
  const int row = wide ? un.chunk : un.chunk * 8 + q;
  const bool row_ok = q < 8 && row < gr.rows_per_split;
  const int rows = gr.rows_per_split, ns = gr.nsplit, base = gr.base_row;
  // All loads are issued without lane predicates (a thread without a split in a slot, or outside
  // the group's rows, reads a neighbour's partial and gives it weight 0): under per-lane
  // conditions the compiler waits for each slot's loads before it asks for the next.
  const int row_c = row < rows ? row : rows - 1;
  float mv[N], lv[N];
  f32x4 av[N];
  bool ok[N];
#pragma unroll
  for (int i = 0; i < N; ++i) {                   // the planner never makes more than 64 splits
    const int s = sl + i * SL;
    ok[i] = row_ok && s < ns;
    const long pr = (long)base + (long)(s < ns ? s : ns - 1) * rows + row_c;
    const float2 t = *reinterpret_cast<const float2*>(ml + pr * 2);
    mv[i] = t.x;
    lv[i] = t.y;
    av[i] = *reinterpret_cast<const f32x4*>(ws + pr * D + col * 4);
  }
  float mloc = NEG_INF;
#pragma unroll
  for (int i = 0; i < N; ++i) mloc = fmaxf(mloc, ok[i] ? mv[i] : NEG_INF);
  float mm = mloc;
  if (wide) {
    if (col == 0) s_max[q] = mloc;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 8; ++i) mm = fmaxf(mm, s_max[i]);
  }
  float ll = 0.f;
  f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const float w = ok[i] ? fast_exp2(mv[i] - mm) : 0.f;
    ll += lv[i] * w;
    o += av[i] * w;
  }
  if (wide) {
    s_acc[q][col] = o;
    if (col == 0) s_l[q] = ll;
    __syncthreads();
    if (q != 0) return;
#pragma unroll
    for (int i = 1; i < 8; ++i) {
      o += s_acc[i][col];
      ll += s_l[i];
    }
  }
  if (!row_ok) return;
  long orow;
  if (gr.type == HFX_ITEM_DECODE) {
    orow = (long)gr.q_start * Hq + gr.h0 * G + row;
  } else {
    const int w = row / HFX_WAVE_ROWS, nn = row % HFX_WAVE_ROWS;
    const int head = gr.h0 + w % gr.hn;
    const int qrow = gr.row0 + (w / gr.hn) * HFX_WAVE_ROWS + nn;
    if (qrow >= gr.q_len) return;
    orow = ((long)gr.q_start + qrow) * Hq + head;
  }
  const float inv = 1.0f / ll;
  bf16x4 ob;
#pragma unroll
  for (int e = 0; e < 4; ++e) ob[e] = (__bf16)(o[e] * inv);
  *reinterpret_cast<bf16x4*>(out + orow * D + col * 4) = ob;
}

template <int D>
__global__ __launch_bounds__(HFX_WG_THREADS) void merge_kernel(const HfxUnit* __restrict__ units,
                                                               const HfxGroup* __restrict__ groups,
                                                               const float* __restrict__ ws,
                                                               const float* __restrict__ ml, int Hq, int G,
                                                               __bf16* __restrict__ out) {
  constexpr int Q = HFX_WG_THREADS / (D / 4);     // threads per column: 8 (D = 128) or 16 (D = 64)
  __shared__ float s_max[Q];
  __shared__ float s_l[Q];
  __shared__ f32x4 s_acc[Q][D / 4];
  // Everything the launch can know on the host comes in as an argument: unit -> group -> partials
  // is the whole chain of dependent loads, and the (m, l) pairs and the accumulator rows of all
  // splits are asked for together.  One copy of the body per number of slots, so that a group of
  // two splits does not pay for eight.  (A unit record that carried a copy of its group saved one
  // trip, about a microsecond, and cost the host ten to write and upload.)
  const HfxUnit un = units[blockIdx.x];
  const HfxGroup gr = groups[un.group];
  const int ns = gr.nsplit;
  if (ns <= 2) merge_rows<D, 2>(un, gr, ws, ml, Hq, G, out, s_max, s_l, s_acc);
  else if (ns <= 4) merge_rows<D, 4>(un, gr, ws, ml, Hq, G, out, s_max, s_l, s_acc);
  else merge_rows<D, 8>(un, gr, ws, ml, Hq, G, out, s_max, s_l, s_acc);
}

// ----------------------------------------------------------------------------------------------
// Decode item.  One wavefront per kv-head (hn of them), the other 4/hn wavefronts of the
// workgroup interleave over page pairs.  Per pair (32 tokens) and kv-head a wavefront issues
// 16 coalesced 16-byte loads per lane and 16 MFMA 16x16x32:
//   S^T[token][head] = K[token][:] . Q[head][:]      (A = K rows, B = Q^T)
//   O^T[d][head]    += V^T[d][token] . P^T[token][head]   (A = V^T rows, B = P^T)
// The two 16-token score tiles take their rows from the page pair such that, in the MFMA
// result layout, each lane ends up holding 8 consecutive tokens of one page -- exactly the
// 16 bytes of a dimension-major V row that the second contraction needs, with no shuffles.
// ----------------------------------------------------------------------------------------------
// Work-queue tickets of a workgroup.  It holds the item it is processing and the item after it
// (whose record is therefore known while the current item runs, so that a prefill item can
// request the first tiles of its successor before it ends).  The ticket after those is asked
// for by thread 0 shortly before the current item ends, published through LDS ahead of a
// barrier the item crosses anyway, and taken at the hand-over.  Asking late matters: a
// workgroup that asks at the start of a long item reserves work it will not touch for a long
// time, and in a step with about three items per workgroup that left half the chip idle while
// the other half worked through its reservations.  The first two tickets of a workgroup are its
// index plus 0 and 1 grids (the queue is in descending cost, so this deals the largest items
// out evenly, and a workgroup starts without a round trip to a counter).  Where that deals all items, no counter
// is touched: atomics on one address from all over the chip take about 14 ns each, one after the other, and 256 workgroups that
// ask for a ticket and report their end spend 7 us on them (4 decodes of 100 to 2000 tokens 13.7 us, 12.7 without; a prompt of 777
// tokens 17.5 and 16.7; 300 rows behind 3000 on 64-wide heads 25.7 and 23.5; 512 workgroups of one short decode piece each 21.2
// and 12.2).
constexpr int kDealtTickets = 2;
struct Tickets {
  int cur, nxt;
  int parity;
  bool queue;        // there may be items behind the next one
  bool own;          // ... and among them some for this die (first wavefront)
  const int* order;  // queue position -> item, if the queue does not hold the items in their order
};

// The dealt tickets of a step whose queue is in descending cost.  Workgroups b and b + 256 share a CU, so
// dealt straight the largest item meets the 256th largest on one CU, the smallest two of the round
// meet on another, and the second round gives the workgroups with the largest items one more.  Here the
// first round runs up and then down the queue -- with fewer items than workgroups, the CUs that stay with
// one workgroup get the largest -- and the second runs down, both within the positions that are equal
// modulo the number of classes.  (2500 tokens on 32/8 heads 66 -> 57 us, 4096 tokens 134 -> 126 us; nothing on queues of
// many items.)
// `mode` is set by the launch: the grid is HFX_PLAN_WGS (1), or more than half of that, one item each (2).
__device__ __forceinline__ void deal_balanced(Tickets& t, int mode, int n_items) {
  constexpr int kHalf = HFX_PLAN_WGS / 2, kLow = HFX_QUEUE_CLASSES - 1;
  const int b = (int)blockIdx.x;
  if (mode == 1) {
    if (b >= kHalf) t.cur = kHalf + (((HFX_PLAN_WGS - 1 - b) & ~kLow) | (b & kLow));
    t.nxt = HFX_PLAN_WGS + (((HFX_PLAN_WGS - 1 - t.cur) & ~kLow) | (b & kLow));
  } else {
    const int paired = n_items - kHalf;           // CUs with two workgroups
    if (b >= kHalf) t.cur = n_items - 1 - (b - kHalf);
    else t.cur = b < paired ? kHalf - paired + b : b - paired;
  }
}

// Queue positions past the dealt ones, up to die_items, fall into HFX_QUEUE_CLASSES classes, position p into class
// p % HFX_QUEUE_CLASSES, each with a counter of its own; those behind are shared.  A workgroup asks the counter of the class of its index and, once that class
// is empty, the shared one.  Workgroups are placed on the chip's dies round-robin by index, so a class is served by the workgroups of
// one die, and the planner puts items that read the same keys into one class: they then share
// that die's L2.  The shared end of the queue, the smallest items, is what lets the dies end together.  Without die_items all positions are shared.
//
// What bounds the counters: atomics and atomic loads on one line from all over the chip are served one after the other, 14 ns
// each.  With all counters on one line, and every workgroup whose class was empty reading the eight of them one by one to find work elsewhere, the end
// of a step with classes took 40 to 90 us, whatever the step (17 short prompts of each of six tasks 87 us from one queue and 185 with classes);
// with a line each, and one load for all eight, still 4 to 6 us, which the shared end does not cost (31 short prompts on 8/1 heads 46 us and 40).
// A workgroup that knows the queue to be empty asks no more, and workgroups report their end by class.  The prefill-heavy mixed step, which has classes,
// took 858 us before and 818 after.
//
// Thread 0 asks for one more ticket; the reply, an offset from the dealt tickets or from the shared positions, goes to
// tickets_publish.  The other lanes keep what `pending` held: a select on it would
// wait for the reply, and with it for everything in flight, wherever the compiler places it.
__device__ __forceinline__ void tickets_reserve(const Tickets& t, int& pending, int* ctrl) {
  if (!t.queue) return;
  int word = t.own ? HFX_CTRL_TICKETS((int)blockIdx.x & (HFX_QUEUE_CLASSES - 1)) : HFX_CTRL_SHARED;
  asm volatile("" : "+s"(word));      // (the address is formed here and not kept in vector registers)
  if (threadIdx.x == 0) pending = atomicAdd(ctrl + word, 1);
}
// The first wavefront turns the reply into an item and thread 0 puts it into LDS (two slots alternate, so one barrier per hand-over is
// enough).
__device__ __forceinline__ void tickets_publish(Tickets& t, int pending, int* s_tk, int* ctrl, const HfxHeader* H) {
  if (!t.queue || uniform((int)threadIdx.x >> 6) != 0) return;
  const int dealt = kDealtTickets * (int)gridDim.x, die_items = (int)H->die_items, shared = max(dealt, die_items);
  int pos = uniform(pending);
  if (t.own) {
    pos = dealt + pos * HFX_QUEUE_CLASSES + ((int)blockIdx.x & (HFX_QUEUE_CLASSES - 1));
    if (pos >= die_items) {
      t.own = false;
      int word = HFX_CTRL_SHARED, reply = 0;
      asm volatile("" : "+s"(word));
      if (threadIdx.x == 0) reply = atomicAdd(ctrl + word, 1);
      pos = shared + uniform(reply);
    }
  } else {
    pos += shared;
  }
  if (t.order && pos < H->n_items) pos = t.order[pos];
  if (threadIdx.x == 0) s_tk[t.parity] = pos;
}
// ... after a workgroup barrier that follows tickets_publish.  Counters only grow: once a ticket is past the end, so are all later ones.
__device__ __forceinline__ void tickets_take(Tickets& t, int* s_tk, int n_items) {
  t.cur = t.nxt;
  t.nxt = 0x7fffffff;
  if (t.queue) t.nxt = uniform(s_tk[t.parity]);
  t.queue = t.nxt < n_items;
  t.parity ^= 1;
}

template <int D>
struct PairRegs {
  bf16x8 ka[D / 32], kb[D / 32], v[D / 16];
};

template <int D>
__device__ __forceinline__ void decode_load(PairRegs<D>& r, const __bf16* pool, int pg0, int pg1, int Hkv, int g,
                                            int k_sel, int k_off, int v_sel, int v_off) {
  constexpr long kBlock = 16 * D;
  const __bf16* kp = pool + (((long)(k_sel ? pg1 : pg0) * Hkv + g) * 2) * kBlock + k_off;
  const __bf16* vp = pool + (((long)(v_sel ? pg1 : pg0) * Hkv + g) * 2 + 1) * kBlock + v_off;
#pragma unroll
  for (int kk = 0; kk < D / 32; ++kk) {   // 32 dimensions = two 16-dimension groups of 256 elements each
    r.ka[kk] = ld16(kp + kk * 512);
    r.kb[kk] = ld16(kp + kk * 512 + 4 * 16);
  }
#pragma unroll
  for (int b = 0; b < D / 16; ++b) r.v[b] = ld16(vp + b * 256);
}

template <int D>
__device__ __forceinline__ void decode_compute(PairRegs<D>& r, const bf16x8* qf, f32x4* o, float& m, float& l,
                                               float sl2, int nv) {
  f32x4 sa = {0.f, 0.f, 0.f, 0.f}, sb = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int kk = 0; kk < D / 32; ++kk) {
    sa = __builtin_amdgcn_mfma_f32_16x16x32_bf16(r.ka[kk], qf[kk], sa, 0, 0, 0);
    sb = __builtin_amdgcn_mfma_f32_16x16x32_bf16(r.kb[kk], qf[kk], sb, 0, 0, 0);
  }
  float s[8];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    s[e] = sa[e] * sl2;
    s[4 + e] = sb[e] * sl2;
  }
  if (nv < 8) {
#pragma unroll
    for (int e = 0; e < 8; ++e) s[e] = keep_or_neg_inf(s[e], e < nv);
  }
  float mx = fmaxf(fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3])), fmaxf(fmaxf(s[4], s[5]), fmaxf(s[6], s[7])));
  mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
  mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
  const float mn = fmaxf(m, mx);
  const float alpha = fast_exp2(m - mn);
  float ps = 0.f;
  bf16x8 pb;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const float p = fast_exp2(s[e] - mn);
    ps += p;
    pb[e] = (__bf16)p;
  }
  l = l * alpha + ps;
  m = mn;
#pragma unroll
  for (int b = 0; b < D / 16; ++b) {
    o[b] *= alpha;
    const bf16x8 vv = (nv < 8) ? keep_first(r.v[b], nv) : r.v[b];
    o[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vv, pb, o[b], 0, 0, 0);
  }
}

// What a wavefront derives from a decode item: its kv-head, its share of the page pairs, and the
// pages of its first two pairs.
struct DecodeWave {
  int g;          // kv-head
  int step;       // pages between two pairs of this wavefront
  int pp, pe;     // next page (pair-aligned) and end of the item's page range
  int tend;       // tokens of the context that the item may see (end of its range or of the context)
  int bt0, last_page;
  int a0, a1, b0, b1;   // page ids of the pair at pp and of the one after it
};

__device__ __forceinline__ int decode_page(const int* __restrict__ bt, const DecodeWave& d, int i) {
  return bt[d.bt0 + (i < d.last_page ? i : d.last_page)];
}

__device__ __forceinline__ DecodeWave decode_wave(const int* __restrict__ bt, const HfxItem& it, int wave) {
  DecodeWave d;
  const int HW = it.hn, sh = HW >> 1;      // 1, 2 or 4, and its logarithm
  d.g = it.h0 + (wave & (HW - 1));
  d.step = 8 >> sh;
  d.pp = it.kb + 2 * (wave >> sh);
  d.pe = it.ke;
  d.tend = min(it.ke * HFX_PAGE, it.rq.ctx_len);
  d.bt0 = it.rq.bt_start;
  d.last_page = it.rq.n_pages - 1;
  d.a0 = decode_page(bt, d, d.pp);
  d.a1 = decode_page(bt, d, d.pp + 1);
  d.b0 = decode_page(bt, d, d.pp + d.step);
  d.b1 = decode_page(bt, d, d.pp + d.step + 1);
  return d;
}

// Runs the decode item t.cur and carries on for as long as the workgroup's next item is a decode
// item too: the first KV pair of the next item is requested before the current item's partial
// results are combined and stored, so the KV stream of a workgroup does not stop between items.
// Returns with t.cur at the first item it did not process.
template <int D>
__device__ void decode_run(const KArgs& a, const HfxHeader* H, const HfxItem* __restrict__ items, int n_items,
                           Tickets& t, int* s_tk, int* ctrl, char* smem) {
  const int tid = threadIdx.x;
  int lane = tid & 63;
  asm volatile("" : "+v"(lane));     // what follows from it is formed per run, not kept in registers through prefill runs
  const int wave = uniform(tid >> 6);
  const int Hq = H->num_q_heads, Hkv = H->num_kv_heads;
  const int G = Hq / Hkv;
  const int n = lane & 15, j = lane >> 4;
  const float sl2 = H->softmax_scale * 1.4426950408889634f;
  const int* bt = reinterpret_cast<const int*>(a.desc + H->off_bt);
  // K rows of the two score tiles: row rho of tile A is (page rho>>3, token ((rho>>2)&1)*8 + (rho&3)),
  // tile B the same + 4 tokens.  V: lane group j reads tokens (j&1)*8.. of page j>>1 for row d = 16b + n.
  const int k_sel = n >> 3;
  const int k_off = (j >> 1) * 256 + (((n >> 2) & 1) * 8 + (n & 3)) * 16 + (j & 1) * 8;
  const int v_sel = j >> 1;
  const int v_off = n * 16 + (j & 1) * 8;
  const int tok_lane = (j >> 1) * 16 + (j & 1) * 8;   // first of this lane's 8 tokens inside the pair

  HfxItem it = items[t.cur];
  DecodeWave d = decode_wave(bt, it, wave);
  PairRegs<D> r0, r1;
  if (d.pp < d.pe) decode_load<D>(r0, a.pool, d.a0, d.a1, Hkv, d.g, k_sel, k_off, v_sel, v_off);
  bf16x8 qf[D / 32];
  auto q_load = [&](const HfxItem& item, int g) {
    const int hh = n < G ? n : G - 1;
    const __bf16* qrow = a.q + ((long)item.rq.q_start * Hq + g * G + hh) * D + j * 8;
#pragma unroll
    for (int kk = 0; kk < D / 32; ++kk) {
      bf16x8 tq = ld16(qrow + kk * 32);
      qf[kk] = keep_first(tq, n < G ? 8 : 0);
    }
  };
  q_load(it, d.g);

  for (;;) {
    // the record of the next item and, if it is a decode item, this wavefront's share of it
    const HfxItem nx = items[t.nxt < n_items ? t.nxt : t.cur];
    const bool carry_on = t.nxt < n_items && nx.type == HFX_ITEM_DECODE;
    const DecodeWave dn = decode_wave(bt, nx, wave);

    f32x4 o[D / 16];
#pragma unroll
    for (int b = 0; b < D / 16; ++b) o[b] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m = NEG_INF, l = 0.f;
    const int step = d.step, pe = d.pe, tend = d.tend, g = d.g;
    int pp = d.pp;
    int a0 = d.a0, a1 = d.a1, b0 = d.b0, b1 = d.b1;
    bool reserved = false;
    int pending = 0;
    // page ids are fetched one pair ahead of the KV loads that need them
    while (pp < pe) {
      if (!reserved && pp + 4 * step >= pe) {   // a few pairs before the end (thread 0 sits in the first wavefront, which always has pairs)
        tickets_reserve(t, pending, ctrl);
        reserved = true;
      }
      if (pp + step < pe) decode_load<D>(r1, a.pool, b0, b1, Hkv, g, k_sel, k_off, v_sel, v_off);
      if (pp + 2 * step < pe) {
        a0 = decode_page(bt, d, pp + 2 * step);
        a1 = decode_page(bt, d, pp + 2 * step + 1);
      }
      {
        const int nv = tend - (pp * HFX_PAGE + tok_lane);
        if ((pp + 2) * HFX_PAGE <= tend) decode_compute<D>(r0, qf, o, m, l, sl2, 8);
        else decode_compute<D>(r0, qf, o, m, l, sl2, nv);
      }
      pp += step;
      if (pp >= pe) break;
      if (pp + step < pe) decode_load<D>(r0, a.pool, a0, a1, Hkv, g, k_sel, k_off, v_sel, v_off);
      if (pp + 2 * step < pe) {
        b0 = decode_page(bt, d, pp + 2 * step);
        b1 = decode_page(bt, d, pp + 2 * step + 1);
      }
      {
        const int nv = tend - (pp * HFX_PAGE + tok_lane);
        if ((pp + 2) * HFX_PAGE <= tend) decode_compute<D>(r1, qf, o, m, l, sl2, 8);
        else decode_compute<D>(r1, qf, o, m, l, sl2, nv);
      }
      pp += step;
    }
    // The reply to the ticket request has come back in front of the last pairs' loads (returns
    // are in order), so publishing it here waits for nothing; after the requests below it would
    // wait for them.  The barriers of the epilogue stand between this write and its readers.
    tickets_publish(t, pending, s_tk, ctrl, H);
    // both register sets and the Q operand are free now: start on the next item
    if (carry_on) {
      if (dn.pp < dn.pe) decode_load<D>(r0, a.pool, dn.a0, dn.a1, Hkv, dn.g, k_sel, k_off, v_sel, v_off);
      q_load(nx, dn.g);
    }
    l += __shfl_xor(l, 16, 64);
    l += __shfl_xor(l, 32, 64);

    // wavefront partial -> LDS: part[wave][head n][D + 4]; o[b][v] is dimension 16b + 4j + v
    constexpr int PS = Smem<D>::kPartStride;
    float* part = reinterpret_cast<float*>(smem);
    if (n < G) {
      float* dst = part + ((wave * 16 + n) * PS);
#pragma unroll
      for (int b = 0; b < D / 16; ++b) *reinterpret_cast<f32x4*>(dst + b * 16 + 4 * j) = o[b];
      if (j == 0) {
        dst[D] = m;
        dst[D + 1] = l;
      }
    }
    __syncthreads();

    // combine the TW token partitions of each head; row = hwi * G + hh
    const int HW = it.hn, TW = 4 >> (HW >> 1);
    const int rows = HW * G;
    float* ws_acc = a.ws;
    float* ws_ml = reinterpret_cast<float*>(reinterpret_cast<char*>(a.ws) + H->ws_off_ml);
    constexpr int C4 = D / 4;
    for (int idx = tid; idx < rows * C4; idx += HFX_WG_THREADS) {
      const int row = idx / C4, d4 = (idx % C4) * 4;
      const int hwi = row / G, hh = row % G;
      float mm = NEG_INF;
      for (int tt = 0; tt < TW; ++tt) mm = fmaxf(mm, part[((tt * HW + hwi) * 16 + hh) * PS + D]);
      float ll = 0.f;
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
      for (int tt = 0; tt < TW; ++tt) {
        const float* src = part + ((tt * HW + hwi) * 16 + hh) * PS;
        const float wgt = fast_exp2(src[D] - mm);
        ll += src[D + 1] * wgt;
        acc += *reinterpret_cast<const f32x4*>(src + d4) * wgt;
      }
      if (it.group < 0) {
        const float inv = 1.0f / ll;
        bf16x4 ob;
#pragma unroll
        for (int e = 0; e < 4; ++e) ob[e] = (__bf16)(acc[e] * inv);
        *reinterpret_cast<bf16x4*>(a.out + ((long)it.rq.q_start * Hq + it.h0 * G + row) * D + d4) = ob;
      } else {
        const long pr = (long)it.slot_row + row;
        *reinterpret_cast<f32x4*>(ws_acc + pr * D + d4) = acc;
        if (d4 == 0) {
          ws_ml[pr * 2] = mm;
          ws_ml[pr * 2 + 1] = ll;
        }
      }
    }
    __syncthreads();                  // frees the LDS partials; the ticket was published before the one above
    tickets_take(t, s_tk, n_items);
    if (!carry_on) break;
    it = nx;
    d = dn;
  }
}

// s_waitcnt vmcnt(N) alone (gfx9 encoding: vmcnt in bits 3:0 and 15:14, the other counters left at their maxima)
#define HFX_WAIT_VMCNT(N) __builtin_amdgcn_s_waitcnt(((N) & 15) | (((N) >> 4) << 14) | (7 << 4) | (15 << 8))

// ----------------------------------------------------------------------------------------------
// Prefill item.  Four wavefronts, each owning 32 chunk rows of one q-head; all four share the
// kv-head.  Both contractions take their streamed operand from LDS:
//   S^T[key][row]  = K[key][:] . Q[row][:]        A = K rows out of the ring, B = Q^T in registers;
//   O^T[d][row]   += V^T[d][key] . P^T[key][row]  A = V^T rows out of the ring (a dimension-major
//                                                 V block is the operand layout), B = P^T from the
//                                                 score registers.
// Each lane owns one query row (a column of S^T and O^T), so the running sum and rescale
// are lane-local up to one exchange with lane ^ 32.  The K rows of a score tile are taken in the
// order that leaves every lane with 8 consecutive keys of one page per 16-key MFMA step.
//
// Keys arrive in stages of 32 (two pages' K and V blocks, 16 KB at D = 128) in a ring of four stage
// slots, filled by direct-to-LDS loads about four stages ahead of their use: they take no registers and no
// vector instructions (54 bytes per clock and CU out of the L2, measured; a stage pair needs 32 KB in
// about 2240 clocks).
//
// What bounds it: the matrix cores, at the clock the chip's power leaves them.  Every matrix instruction of the
// stage loop is followed by one LDS read of a fragment and one sixteenth of the softmax (an exponential, and every other time the
// sum and rounding of a pair), so that vector unit, LDS and matrix cores are asked for at an even rate whichever
// phases the two wavefronts of a SIMD are in; and the common stage pairs run in a loop of their own, without conditions,
// scalar loads or bursts of copies.  Clocks a pair of stages in that loop, waits at its synchronisation points included, of which the
// matrix instructions are 1024: 1573 for a wavefront that has its SIMD to itself, 1980 and 2510 for the older and the younger of two
// in a 4096-row chunk behind 61440 tokens, so that the matrix cores are busy 2 * 1024 of 2243 clocks there, 91 %.  The loop is 0.91 of the
// workgroups' time in that step and 0.82 to 0.87 where tiles are shorter.  With the whole softmax behind the score instructions and one loop for
// all stages the clocks were 2350, 2450 and 3050.  Times of the two loops, both in turn on one card: 4 prompt chunks of 2048 rows behind up to 12288
// earlier tokens beside 32 decodes (0.96 TFLOP) 879 and 841 us; a 4096-row chunk behind 61440 tokens and 16 decodes 1020 and 943; a single prompt of 777
// tokens 18.2 and 15.7.  (With listed copies and the counters on lines of their own 797 to 837, 938 to 970 and 14.8 to 15.4 by the card.)
// A value fragment takes the registers of the key fragment used up before it, and the other way round.
// Tried with it: the synchronisation point behind the second value instruction instead of in front of the first (-1.5 to +1.5 %); a ring
// of eight stages where a workgroup has its CU to itself (slower: nobody waits for a copy with four).
// ----------------------------------------------------------------------------------------------

// One stage slot: [page 0 K][page 1 K][page 0 V][page 1 V], a block of 32 D bytes each, and
// wavefront w copies block w, 1 KB (64 lanes of 16 bytes) per instruction.  An instruction puts lane
// l's 16 bytes at 16 l, so the order inside a 1 KB chunk is chosen by the address each lane reads from:
//   keys  : two 16-dimension groups of 16 slots x 32 bytes; LDS order (group, half, slot), so that
//           the 16 lanes that the LDS serves together (16 slots, same half) hit 16 bank groups;
//   values: 32 dimension rows of two 16-byte halves; the halves of rows 8-15 and 24-31 change places,
//           so that 16 rows read at the same half hit 16 bank groups instead of colliding in pairs.
__device__ __forceinline__ unsigned copy_lane_offset(int wave, int lane) {
  if (wave < 2) return (unsigned)((lane >> 5) * 512 + (lane & 15) * 32 + ((lane >> 4) & 1) * 16);
  return (unsigned)((lane >> 1) * 32 + ((lane & 1) ^ ((lane >> 4) & 1)) * 16);
}

// Direct-to-LDS copy of one kilobyte, number `piece` of a block: base (scalar) + voff (lane) in memory, lds + 16 * lane in LDS.  The
// instruction has no destination register; the compiler does not know of the load, so its own
// vector-memory waits only become stricter by it, and the ring's waits are the explicit ones below.  The LDS
// address travels in m0: the compiler reserves that register but merges its own settings of it where it sees no
// other write between them, so the write is declared.  (Its warning that a clobber does not save a
// reserved register is switched off: nothing lives in m0 across a statement.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void piece_copy(const char* base, unsigned voff, unsigned lds, int piece) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 offset:%3"
               :: "v"(voff), "s"(base), "s"(lds), "n"(piece * 1024) : "memory", "m0");
}
// Numbers `piece` and piece + 1.
__device__ __forceinline__ void two_pieces_copy(const char* base, unsigned voff, unsigned lds, int piece) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 offset:%3\n\tglobal_load_lds_dwordx4 %0, %1 offset:%4"
               :: "v"(voff), "s"(base), "s"(lds), "n"(piece * 1024), "n"(piece * 1024 + 1024) : "memory", "m0");
}
#pragma clang diagnostic pop

// A whole block.
template <int D>
__device__ __forceinline__ void block_copy(const char* base, unsigned voff, unsigned lds) {
#pragma unroll
  for (int piece = 0; piece < D / 32; piece += 2) two_pieces_copy(base, voff, lds, piece);
}

// Workgroup barrier of the ring: this wavefront's LDS reads are done.  The compiler may move loads across
// the barrier builtin, which claims no memory effect, so the empty asm on both sides holds them.
__device__ __forceinline__ void ring_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Per-wavefront state of a prefill item that lives across stages.
template <int D>
struct PrefillWave {
  f32x16 o[D / 32];        // O^T accumulators per 32-dimension block
  bf16x8 qf[D / 16];       // Q^T operand fragments
  float m, l;              // reference exponent (base-2 domain) and running sum
};

#define HFX_M_NONE (-3.402823466e38f)   // reference exponent before the first stage: lower than any score

// Weights of 16 scores against reference exponent m, and their sum (fp32, four partial sums; plain
// adds, because the two-element dot-product instruction does not issue while a matrix instruction
// executes).
__device__ __forceinline__ float weights(const f32x16& s, float sl2, float m, bf16x8* pb) {
  float ps[4];
#pragma unroll
  for (int v = 0; v < 16; v += 2) {
    const float p0 = fast_exp2(__builtin_fmaf(s[v], sl2, -m));
    const float p1 = fast_exp2(__builtin_fmaf(s[v + 1], sl2, -m));
    if (v < 8) ps[v >> 1] = p0 + p1;
    else ps[(v >> 1) & 3] += p0 + p1;
    pb[v >> 3][v & 7] = (__bf16)p0;
    pb[v >> 3][(v & 7) + 1] = (__bf16)p1;
  }
  return (ps[0] + ps[1]) + (ps[2] + ps[3]);
}

// Masks the scores of keys that this lane's row must not see (those past `pos`): s[v] is key
// key0 + (v>>3)*16 + (v&7)   (key0 already includes the lane's 8j).  The visible ones are the first few
// of the 16, so one bit mask says which; selects on compares would hold 16 condition masks at once.  Masked
// scores may be NaN (unused slots hold anything), hence integer operations.
__device__ __forceinline__ void mask_scores(f32x16& s, int pos, int key0) {
  const int d = pos - key0;
  const int visible = min(max(d + 1, 0), 8) + min(max(d - 15, 0), 8);
  const int bits = (1 << visible) - 1;
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const unsigned keep = (unsigned)((int)((unsigned)bits << (31 - v)) >> 31);     // all ones where visible
    const float x = s[v];            // (a bit cast of the vector element itself would read element 0)
    s[v] = __builtin_bit_cast(float, (__builtin_bit_cast(unsigned, x) & keep) | (0xff800000u & ~keep));
  }
}

// Maximum over the 32 scores of this lane's row (16 here, 16 in lane ^ 32), in the base-2 domain.
__device__ __forceinline__ float row_max(const f32x16& s, float sl2) {
  float mx = fmaxf(s[0], s[1]);
#pragma unroll
  for (int v = 2; v < 16; v += 2) mx = fmaxf(fmaxf(mx, s[v]), s[v + 1]);   // v_max3_f32
  return max_xor32(mx) * sl2;
}

// m is the reference exponent of an item's running sums: the maximum of its first stage to begin
// with.  A stage's weights are taken against the m at hand; only when some lane's 16 weights sum to
// more than 2^8 -- its maximum has grown well over m -- is m raised to the maximum, O and l rescaled,
// and the weights taken again.  So the common stage needs neither the maximum nor the exchange
// between the lanes of a row, and no weight exceeds 2^8.
template <int D>
__device__ __forceinline__ void settle_weights(PrefillWave<D>& w, const f32x16& s, bf16x8* pb, float sum, float sl2) {
  if (__builtin_expect(__any(sum > 256.0f), 0)) {
    const float mx = fmaxf(w.m, row_max(s, sl2));
    const float alpha = fast_exp2(w.m - mx);
    w.l *= alpha;
#pragma unroll
    for (int b = 0; b < D / 32; ++b) w.o[b] *= alpha;
    w.m = mx;
    sum = weights(s, sl2, w.m, pb);
  }
  w.l += sum;
}

// Scores of an item's first stage: S^T = K . Q^T out of K fragments in registers; the accumulators are cleared between the
// instructions.
template <int D>
__device__ __forceinline__ f32x16 first_scores(PrefillWave<D>& w, const bf16x8* kf) {
  f32x16 s;
#pragma unroll
  for (int v = 0; v < 16; ++v) s[v] = 0.f;
#pragma unroll
  for (int kk = 0; kk < D / 16; ++kk) {
    s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[kk], w.qf[kk], s, 0, 0, 0);
#pragma unroll
    for (int v = 0; v < 8; ++v) {
      float zero = 0.f;
      asm volatile("" : "+v"(zero));
      w.o[kk / 2][kk % 2 * 8 + v] = zero;
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  return s;
}

template <int D>
__device__ __forceinline__ void read_keys(bf16x8* kf, const char* slot, int k_lane) {
#pragma unroll
  for (int kk = 0; kk < D / 16; ++kk) kf[kk] = *reinterpret_cast<const bf16x8*>(slot + kk * 512 + k_lane);
}

// Which scores have their weights formed behind which matrix instruction: number i of the value phase takes scores
// [values[i], values[i + 1]) of the next stage, number i of the score phase [scores[i], scores[i + 1]) of the present one.
// The first value instruction takes none, because the scores of the next stage come out of the matrix instruction just before it,
// and the last score instruction none, so that the sum of the weights is known by the end of its phase.
template <int D>
struct Share;
template <>
struct Share<128> {
  static constexpr int values[9] = {0, 0, 1, 2, 3, 5, 6, 7, 8}, scores[9] = {8, 9, 10, 11, 13, 14, 15, 16, 16};
};
template <>
struct Share<64> {
  static constexpr int values[5] = {0, 2, 4, 6, 8}, scores[5] = {8, 10, 12, 14, 16};
};

// The weights of a stage on their way.  A pair is summed and rounded one portion after its exponentials, so that nothing
// waits for an exponential just issued.  The empty asm statements hold the results where they are formed: left to itself
// the compiler puts the sums and roundings of all portions behind the last one.
struct Weighing {
  float p[16], ps[4];
  unsigned pw[8];            // rounded pairs

  __device__ __forceinline__ void finish(int i) {
    const float t = p[2 * i] + p[2 * i + 1];
    if (i < 4) ps[i] = t;
    else ps[i & 3] += t;
    const bf16x2 r = {(__bf16)p[2 * i], (__bf16)p[2 * i + 1]};
    pw[i] = __builtin_bit_cast(unsigned, r);
    asm volatile("" : "+v"(pw[i]), "+v"(ps[i & 3]));
  }
  // weights of scores [e0, e1), and the pairs that were completed in [before, e0)
  __device__ __forceinline__ void portion(int before, int e0, int e1, const f32x16& s, float sl2, float m) {
#pragma unroll
    for (int e = 0; e < 16; ++e)
      if (e >= e0 && e < e1) {
        p[e] = fast_exp2(__builtin_fmaf(s[e], sl2, -m));
        asm volatile("" : "+v"(p[e]));
      }
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (2 * i + 1 >= before && 2 * i + 1 < e0) finish(i);
  }
  __device__ __forceinline__ bf16x8 fragment(int sp) const {
    return __builtin_bit_cast(bf16x8, u32x4{pw[4 * sp], pw[4 * sp + 1], pw[4 * sp + 2], pw[4 * sp + 3]});
  }
  __device__ __forceinline__ float sum() const { return (ps[0] + ps[1]) + (ps[2] + ps[3]); }
};

template <int D>
__device__ __forceinline__ bf16x8 value_fragment(const char* slot, int i, int v_lane) {
  constexpr int B = D / 32;
  return *reinterpret_cast<const bf16x8*>(slot + (2 + i / B) * Smem<D>::kBlockBytes + (i % B) * 1024 + v_lane);
}

// First phase of a stage: scores of the next stage out of its key fragments, the second half of the weights of the
// present one (scores cur) between them; the value fragments of the present stage take the place of each key
// fragment as it is used up.
template <int D>
__device__ __forceinline__ f32x16 scores_phase(const PrefillWave<D>& w, bf16x8* frag, const f32x16& cur, Weighing& wt, float sl2,
                                               const char* v_slot, int v_lane) {
  constexpr int S = D / 16;
  f32x16 acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
#pragma unroll
  for (int i = 0; i < S; ++i) {
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag[i], w.qf[i], acc, 0, 0, 0);
    frag[i] = value_fragment<D>(v_slot, i, v_lane);
    wt.portion(i == 0 ? Share<D>::values[S - 1] : Share<D>::scores[i - 1], Share<D>::scores[i], Share<D>::scores[i + 1], cur, sl2, w.m);
    __builtin_amdgcn_sched_barrier(0);
  }
  wt.portion(Share<D>::scores[S - 1], 16, 16, cur, sl2, w.m);
  return acc;
}

struct NoCopy {
  __device__ __forceinline__ void operator()(int) const {}
};

// Second phase: weighted values of the present stage, the first half of the weights of the next one (scores next) between
// them, and the key fragments of the stage after next in the place of the value fragments.  copy(i) issues what is to be
// copied behind instruction i.
template <int D, class Copy>
__device__ __forceinline__ void values_phase(PrefillWave<D>& w, bf16x8* frag, const bf16x8* pb, const f32x16& next, Weighing& wt,
                                             float sl2, const char* k_slot, int k_lane, Copy copy) {
  constexpr int B = D / 32, S = 2 * B;
#pragma unroll
  for (int i = 0; i < S; ++i) {
    w.o[i % B] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag[i], pb[i / B], w.o[i % B], 0, 0, 0);
    frag[i] = *reinterpret_cast<const bf16x8*>(k_slot + i * 512 + k_lane);
    copy(i);
    wt.portion(i == 0 ? 0 : Share<D>::values[i - 1], Share<D>::values[i], Share<D>::values[i + 1], next, sl2, w.m);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// What a wavefront derives from a prefill item: its q-head and rows, and the key ranges that
// decide whether a stage is worked on and whether it needs masks.
struct WaveRows {
  int head, row0;             // q-head and first chunk row
  int wave_kend, wave_pmin;
};

__device__ __forceinline__ WaveRows wave_rows(const HfxItem& it, int wave) {
  WaveRows r;
  // hn is 1, 2 or 4 (a division would take the vector unit, and with it all that follows from its result)
  r.head = it.h0 + (wave & (it.hn - 1));
  r.row0 = it.row0 + (wave >> (it.hn >> 1)) * HFX_WAVE_ROWS;
  const int p = it.rq.ctx_len - it.rq.q_len;
  r.wave_kend = r.row0 < it.rq.q_len ? min(it.ke, p + min(r.row0 + HFX_WAVE_ROWS, it.rq.q_len)) : 0;   // keys >= this: nothing to do
  r.wave_pmin = p + r.row0;                                                            // keys <= this are visible to every row
  return r;
}

// Q^T operand fragments of this lane's row (rows past the chunk read the last row and are never stored)
template <int D>
__device__ __forceinline__ void q_load(bf16x8* qf, const __bf16* q, int row0, int last, int Hq, int n, int j) {
  const __bf16* qp = q + (long)min(row0 + n, last) * Hq * D + j * 8;
#pragma unroll
  for (int kk = 0; kk < D / 16; ++kk) qf[kk] = ld16(qp + kk * 16);
}

// Result of a finished item: normalised bf16 rows, or (m, l, acc) partial rows when the item is one split of a group.
// A lane holds 4-dimension pieces of its own row, so stored straight from the registers every
// instruction would touch 32 rows with 16 bytes each, and the write path takes one request per
// (instruction, line).  The bf16 rows therefore go through `stage` (2 KB of LDS owned by this
// wavefront, 32 dimensions of its 32 rows at a time) and leave in 64-byte pieces, 16 rows per
// instruction.  The 16-byte units of a row are permuted by the row number, and the two 8-byte halves of a unit
// change places in rows 16-31, so that writes and reads spread over all LDS banks.
template <int D>
__device__ __forceinline__ void prefill_store(const KArgs& a, const HfxHeader* H, const HfxItem& it, const WaveRows& r,
                                              const PrefillWave<D>& w, int Hq, int wave, int lane, char* stage) {
  // o[b][v] is dimension 32b + (v>>2)*8 + 4j + (v&3) of chunk row row0 + (lane & 31)
  const float lsum = sum_xor32(w.l);
  // The lane's parts of the destination addresses are formed here, per call: left visible, the
  // compiler hoists them out of the item loop, runs out of registers and parks them in scratch
  // memory, and the reload at every hand-over waits for every load the stage ring has in flight.
  asm volatile("" : "+v"(lane));
  const int n = lane & 31, j = lane >> 5;
  if (it.group < 0) {
    const float inv = 1.0f / lsum;
    const int row0 = r.row0;
    const int rr = lane >> 2, u = lane & 3;      // read-back: row rr + 16i, 16-byte unit u
    __bf16* dst = a.out + (((long)it.rq.q_start + row0 + rr) * Hq + r.head) * D + u * 8;
    char* wr = stage + n * 64 + (j ^ (n >> 4)) * 8;
    const char* rd = stage + rr * 64 + ((u ^ ((rr >> 2) & 3)) * 16);
    // LDS serves a wavefront's accesses in order, so the next 32 dimensions are written while the lines of these are on
    // their way back
    u32x4 line[D / 32][2];
#pragma unroll
    for (int b = 0; b < D / 32; ++b) {
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        bf16x4 ob;
#pragma unroll
        for (int e = 0; e < 4; ++e) ob[e] = (__bf16)(w.o[b][q4 * 4 + e] * inv);
        *reinterpret_cast<bf16x4*>(wr + ((q4 ^ ((n >> 2) & 3)) * 16)) = ob;
      }
#pragma unroll
      for (int i = 0; i < 2; ++i) line[b][i] = *reinterpret_cast<const u32x4*>(rd + i * 1024);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
      if (row0 + rr + 16 * i < it.rq.q_len) {
#pragma unroll
        for (int b = 0; b < D / 32; ++b) {
          const u32x4 t = line[b][i];
          *reinterpret_cast<u32x4*>(dst + (long)i * 16 * Hq * D + b * 32) = i == 1 ? u32x4{t[2], t[3], t[0], t[1]} : t;
        }
      }
  } else {
    float* ws_acc = a.ws;
    float* ws_ml = reinterpret_cast<float*>(reinterpret_cast<char*>(a.ws) + H->ws_off_ml);
    const long pr = (long)it.slot_row + wave * HFX_WAVE_ROWS + n;
    float* dst = ws_acc + pr * D + 4 * j;
#pragma unroll
    for (int b = 0; b < D / 32; ++b)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        f32x4 t = {w.o[b][q4 * 4], w.o[b][q4 * 4 + 1], w.o[b][q4 * 4 + 2], w.o[b][q4 * 4 + 3]};
        *reinterpret_cast<f32x4*>(dst + b * 32 + q4 * 8) = t;
      }
    if (j == 0) {
      ws_ml[pr * 2] = w.m;
      ws_ml[pr * 2 + 1] = lsum;
    }
  }
}

// The workgroup's stream of stage copies: the stages of the current item and then those of the next
// item, if that is a prefill item too (the item after next has no ticket yet).  Which block a copy takes is read from a list in LDS,
// one a wavefront, whose entries run on from item to item, so that a copy is the same few instructions wherever it is issued: no scalar loads of page
// ids (which the next wait for an LDS read would wait for as well), and whole pairs run up to the end of an item.  With page ids of the
// present item alone in LDS, and only of long ones, a prompt of 777 tokens took 15.9 us instead of 15.1, 14 steps of one to five prompts 1.017
// times as long on average, 21 of short prompts 1.016 times.  Wave-uniform.
struct CopyStream {
  int count;          // stages copied so far, over all items of the run
  int listed;         // stages whose blocks are in the list, likewise
  int left;           // stages of the item being listed that are still to be asked for
  int bt;             // stored block-table entry of the next of them: the page that this wavefront copies
  int last;           // block-table entry of the request's last page
  int head;           // kv-head of the item being listed
  int asked;          // stages whose page ids are on their way, to be listed next ...
  int asked_head;     // ... and their kv-head
  int in_next;        // the item being listed is the next one, not the current one
  int limit;          // stages that could be copied at the last synchronisation point without overwriting one still to be read
};
constexpr int kListed = 128;      // entries of a wavefront's list; up to 64 are asked for when that many are free

__device__ __forceinline__ int item_stages(const HfxItem& it) { return (int)((unsigned)(it.ke - it.kb + HFX_STAGE_KEYS - 1) / HFX_STAGE_KEYS); }

// What the loop over an item's stages needs to know of the item after it: how to copy its stages and where its Q rows are.
// (Its whole record kept in scalar registers through that loop, and everything that can be derived from it formed
// ahead of it, cost 67 registers' worth of spills and about 150 instructions an item.)
struct NextItem {
  int left, bt, last, head;   // as in CopyStream
  int q_row0, q_last;         // first chunk row of this wavefront, last of the chunk
  const __bf16* q;            // row 0 of the chunk, this wavefront's head
};

// Stages that an item must have left for whole pairs to be looked for.  (2, 3 or 4 instead: 22 steps of short prompts 0.996 to 0.997 times as fast,
// 38 others the same within 0.1 %.)
constexpr int kPairsFrom = 6;

// Runs the prefill item t.cur and, for as long as the workgroup's next item is a prefill item as
// well, carries straight on into it: the stage ring does not drain between items, only the
// per-row state (Q, O, m, l) is swapped.  Returns with t.cur at the first item it did not process.
//
// A wavefront's work on stage s, in two phases:
//   first  : scores of stage s + 1 (matrix cores, K fragments in registers) between the second half of the softmax
//            of stage s (vector unit) and the reads of its value fragments;
//   second : weighted values of stage s between the first half of the softmax of stage s + 1 and the reads of the key
//            fragments of stage s + 2.
// Two stages make a step of the loop, so that the scores change places without being moved, and there
// is one synchronisation point per step, between the phases of its first stage g: the keys up to stage
// g + 3 and the values up to stage g + 2 have landed, every wavefront has taken the fragments of keys up to
// g + 1 and values up to g, and their slots are copied into next.  (One point per stage: 1.75 M cycles instead
// of 1.67 M.)
template <int D>
__device__ void prefill_run(const KArgs& a, const HfxHeader* H, const HfxItem* __restrict__ items, int n_items,
                            Tickets& t, int* s_tk, int* ctrl, char* smem, char* o_stage, int* s_ids) {
  constexpr int SK = HFX_STAGE_KEYS;
  constexpr int RING = Smem<D>::kStages;
  const int tid = threadIdx.x;
  int lane = tid & 63;
  asm volatile("" : "+v"(lane));     // what follows from it is formed per run, not kept in registers through decode runs
  const int wave = uniform(tid >> 6);
  const int Hq = H->num_q_heads, Hkv = H->num_kv_heads;
  const int G = Hq / Hkv;
  const int n = lane & 31, j = lane >> 5;
  char* stage = o_stage + wave * 2048;
  const float sl2 = H->softmax_scale * 1.4426950408889634f;
  const int* __restrict__ bt = reinterpret_cast<const int*>(a.desc + H->off_bt);
  // row of this lane's key inside the stage's 32 keys
  const int krow = (n >> 4) * 16 + ((n >> 2) & 1) * 8 + ((n >> 3) & 1) * 4 + (n & 3);
  const int k_lane = (krow >> 4) * Smem<D>::kBlockBytes + j * 256 + (krow & 15) * 16;
  const int v_lane = (n * 2 + (j ^ ((n >> 3) & 1))) * 16;   // V^T rows 32b + n, keys 8j.. of a page
  const unsigned voff = copy_lane_offset(wave, lane);
  const unsigned lds_ring = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)smem + wave * Smem<D>::kBlockBytes;
  const char* pool = reinterpret_cast<const char*>(a.pool) + (wave >> 1) * Smem<D>::kBlockBytes;
  const int key_wave = 1 - (wave >> 1);   // 1: this wavefront copies keys, which are read a stage before the values

  HfxItem it = items[t.cur];
  CopyStream cs;
  const unsigned inv_g = 0xffffffffu / (unsigned)G + 1u;      // h / G by a multiplication (0 for G = 1)
  auto q_rows = [&](const HfxItem& item, const WaveRows& r) { return a.q + ((long)item.rq.q_start * Hq + r.head) * D; };
  auto next_item = [&](const HfxItem& item) {
    const WaveRows r = wave_rows(item, wave);
    const int g = G == 1 ? item.h0 : (int)__umulhi((unsigned)item.h0, inv_g);
    NextItem x;
    x.left = item_stages(item);
    x.bt = item.rq.bt_start + (int)((unsigned)item.kb / HFX_PAGE) + (wave & 1);
    x.last = item.rq.bt_start + item.rq.n_pages - 1;
    x.head = g;
    x.q_row0 = r.row0;
    x.q_last = item.rq.q_len - 1;
    x.q = q_rows(item, r);
    return x;
  };
  const HfxItem item1 = items[t.nxt < n_items ? t.nxt : t.cur];
  NextItem nx = next_item(item1);
  bool next_ok = t.nxt < n_items && item1.type == HFX_ITEM_PREFILL;
  int* const list = s_ids + wave * kListed;
  int page_ids = 0;                    // of the stages asked for, one a lane
  auto list_start = [&](const NextItem& item) {
    cs.left = item.left;
    cs.bt = item.bt;
    cs.last = item.last;
    cs.head = item.head;
  };
  // asks for page ids if there is room for them; the item after the current one follows it as soon as it is known
  auto list_ask = [&]() {
    if (cs.left <= 0 && !cs.in_next && next_ok) {
      cs.in_next = 1;
      list_start(nx);
    }
    if (cs.left > 0 && cs.asked == 0 && cs.listed - cs.count <= kListed - 64) {
      page_ids = bt[min(cs.bt + 2 * lane, cs.last)];
      cs.asked = min(cs.left, 64);
      cs.asked_head = cs.head;
      cs.left -= cs.asked;
      cs.bt += 2 * 64;
    }
  };
  // ... and lists them, behind a wait for all loads.  (Entries past the item's last stage are overwritten by the next item's.)
  auto list_write = [&]() {
    if (cs.asked > 0) {
      list[(cs.listed + lane) & (kListed - 1)] = page_ids * Hkv + cs.asked_head;
      cs.listed += cs.asked;
      cs.asked = 0;
    }
  };
  // waits until the list reaches `limit`, as far as the items to come are known
  auto list_until = [&](int limit) {
    while (cs.listed < limit) {
      list_ask();
      if (cs.asked == 0) break;
      HFX_WAIT_VMCNT(0);
      list_write();
    }
  };
  auto block_base = [&](int entry) { return pool + (unsigned long)(unsigned)entry * (2 * Smem<D>::kBlockBytes); };
  auto slot_lds = [&](int stage_no) { return lds_ring + (stage_no & (RING - 1)) * Smem<D>::kStageBytes; };   // slots are handed out round-robin over the whole run
  // the list from the next stage to be copied on, an entry a lane
  auto list_read = [&]() { return list[(cs.count + lane) & (kListed - 1)]; };
  // copies the next n stages, all in a row, by what list_read gave
  auto copy_stages = [&](int n, int entries) {
#pragma unroll 1
    for (int i = 0; i < n; ++i) {
      block_copy<D>(block_base(__builtin_amdgcn_readlane(entries, i)), voff, slot_lds(cs.count));
      ++cs.count;
    }
  };
  cs.count = 0;
  cs.listed = 0;
  cs.asked = 0;
  cs.in_next = 0;

  // The stage in which the next ticket is asked for and published (the workgroup waits for the reply there:
  // a reply in flight through the stage loop would make the compiler wait for it, and with it for every copy
  // in flight, wherever it touches the register).  Short items ask at the hand-over, where the reply comes
  // back with Q, and have no such stage.
  int n_st, publish_st;
  auto set_ticket_points = [&]() {
    n_st = item_stages(it);
    publish_st = n_st > 6 ? n_st - 3 : -(1 << 30);
  };
  set_ticket_points();
  int pending = 0;
  if (n_st <= 6) tickets_reserve(t, pending, ctrl);

  PrefillWave<D> w;
  WaveRows wr = wave_rows(it, wave);
  q_load<D>(w.qf, q_rows(it, wr), wr.row0, it.rq.q_len - 1, Hq, n, j);
  int g_st = 0;      // stages multiplied so far, over all items of the run: the ring position
  // The first copies of the run do not wait for a list: their page ids are scalar loads.  Block-table entries are read a little past the last page of a
  // request, up to the seventh entry behind it; those entries name the last page again.
  static_assert(HFX_BT_PAD >= 7, "entries behind a request's last page that the copy stream may read");
  {
    const NextItem first = next_item(it);
    list_start(first);
    cs.limit = RING - 1 + key_wave;
    const int n0 = min(n_st, cs.limit);
    int page[RING];
#pragma unroll
    for (int i = 0; i < RING; ++i) page[i] = bt[cs.bt + 2 * i];
#pragma unroll
    for (int i = 0; i < RING; ++i)
      if (i < n0) block_copy<D>(block_base(page[i] * Hkv + cs.head), voff, slot_lds(i));
    cs.count = cs.listed = n0;
    cs.left -= n0;
    cs.bt += 2 * n0;
    list_ask();
  }
  if (n_st <= 6) tickets_publish(t, pending, s_tk, ctrl, H);

  // Synchronisation point of the ring: what has been copied so far has landed and everyone's fragment reads
  // so far are done, so that copies may go on up to `limit`; returns how many that are.  The next ticket is asked
  // for and published here, and the list goes on.  The entries are read ahead of the waits (one prompt of 777 tokens 15.1 us, read one by one behind them 15.2;
  // 42 chunks of 4 rows behind 5321 on 64-wide 8/8 heads 87.0 and 88.9).
  auto sync_point = [&](int limit, int& entries) {
    entries = list_read();
    if (g_st == publish_st || g_st + 1 == publish_st) {
      int reply = 0;
      tickets_reserve(t, reply, ctrl);
      tickets_publish(t, reply, s_tk, ctrl, H);
    }
    HFX_WAIT_VMCNT(0);
    ring_barrier();
    if (cs.asked > 0 || cs.listed < limit) {
      list_write();
      list_until(limit);
      entries = list_read();
    }
    list_ask();
    cs.limit = limit;
    return min(limit, cs.listed) - cs.count;
  };
  for (;;) {
    w.l = 0.f;
    const int wave_end = wr.wave_kend, unmasked_upto = wr.wave_pmin, ctx_len = it.rq.ctx_len;
    const int end_st = g_st + n_st - 1;      // the item's last stage
    publish_st += g_st;
    int kt = it.kb;
    auto mask_stage = [&](f32x16& s, int key0) {     // keys past this lane's row's horizon (rows past the chunk: its last row's)
      mask_scores(s, min(wr.wave_pmin + n, ctx_len - 1), key0 + j * 8);
    };
    bf16x8 frag[D / 16];     // key fragments of the next stage, then value fragments of the present one
    f32x16 s0, s1;
    Weighing wt;
    // the first stage: its scores, their maximum as the reference exponent, and the first half of its weights
    int entries;
    const int due = sync_point(g_st + RING - 1 + key_wave, entries);
    read_keys<D>(frag, smem + (g_st & (RING - 1)) * Smem<D>::kStageBytes, k_lane);
    copy_stages(due, entries);
    s0 = first_scores<D>(w, frag);
    read_keys<D>(frag, smem + ((g_st + 1) & (RING - 1)) * Smem<D>::kStageBytes, k_lane);
    if (kt + SK - 1 > unmasked_upto) mask_stage(s0, kt);
    w.m = fmaxf(HFX_M_NONE, row_max(s0, sl2));
    wt.portion(0, 0, 4, s0, sl2, w.m);
    wt.portion(0, 4, 8, s0, sl2, w.m);
    wt.portion(4, Share<D>::values[D / 16 - 1], Share<D>::values[D / 16 - 1], s0, sl2, w.m);
    auto slot = [&](int st) { return smem + (st & (RING - 1)) * Smem<D>::kStageBytes; };
    auto mask_values = [&](bf16x8* vf) {   // unused V slots may hold anything
#pragma unroll
      for (int i = 0; i < D / 16; ++i) vf[i] = keep_first(vf[i], ctx_len - (kt + i / (D / 32) * 16 + j * 8));
    };
    // One stage: `cur` holds its scores, `next` receives those of the stage after it.  Every other stage
    // synchronises between its two phases.
    auto stage_step = [&](f32x16& cur, f32x16& next, bool sync) {
      const bool busy = kt < wave_end;
      bf16x8 pb[2];
      __builtin_amdgcn_sched_barrier(0);
      if (busy) {
        next = scores_phase<D>(w, frag, cur, wt, sl2, slot(g_st), v_lane);
        pb[0] = wt.fragment(0);
        pb[1] = wt.fragment(1);
        settle_weights<D>(w, cur, pb, wt.sum(), sl2);
      }
      if (sync) {
        int ahead;
        const int n_due = sync_point(g_st + RING + 1 + key_wave, ahead);
        copy_stages(n_due, ahead);
      }
      if (busy) {
        if (kt + 2 * SK - 1 > unmasked_upto) mask_stage(next, kt + SK);
        __builtin_amdgcn_sched_barrier(0);
        values_phase<D>(w, frag, pb, next, wt, sl2, slot(g_st + 2), k_lane, NoCopy());
      }
      ++g_st;
      kt += SK;
    };
    for (;;) {
      // Pairs of stages that every row of the wavefront sees whole, with the short form of the synchronisation point: the common
      // case, without any other condition.  The copies are issued one behind each of the matrix instructions that follow that point: in a
      // burst in front of them they hold up the wavefront (a 4096-row chunk behind 61440 tokens 970 us, 950 so), and spread over
      // twice as many they land later, which chunks of few rows wait for (42 of 4 rows behind 5321 on 8/8 heads of 64 97.5 and 92.6,
      // 97 of one row behind 12208 on 24/8 heads 1294 and 1251; 90.7 and 1182 with one burst and the loop before).
      // Where heads are 64 wide, a wavefront without rows copies in a loop of its own.  In chunks of few rows, where one wavefront of an item has all of them, the
      // others' copies are what the item waits for: by way of the general form 30 chunks of 2 rows behind 2100 to 4100 on 8/8 heads take 49.4 us and 48.0 so, 46 behind
      // 1100 to 2200 36.8 and 35.0, 42 of 4 behind 5321 87.0 and 85.4; prompts are the same within 1 %.  (128 wide, with twice the work a stage: 16 of 2 rows
      // behind 700 to 1250 19.6 and 20.0, others the same.)
      if (D == 64 && wave_end == 0 && end_st - g_st >= kPairsFrom && cs.asked == 0 && cs.count == g_st + RING - 1 + key_wave) {
        int stages = min(cs.listed - cs.count - (cs.left > 0 ? 2 : 0), (publish_st > g_st ? min(publish_st - 1, end_st - 1) : end_st - 1) - g_st + 1) & ~1;
        kt += max(stages, 0) * SK;
#pragma unroll 1
        for (; stages > 0; stages -= 2) {
          const int entries = list_read();
          HFX_WAIT_VMCNT(0);
          ring_barrier();
          copy_stages(2, entries);
          g_st += 2;
        }
      }
      int pairs = 0;
      if (end_st - g_st >= kPairsFrom && wave_end > 0 && kt + 3 * SK - 1 <= unmasked_upto && cs.asked == 0 && cs.count == g_st + RING - 1 + key_wave)
        pairs = uniform(min(min((int)((unsigned)(unmasked_upto - kt - 3 * SK + 1) / (2 * SK)) + 1, (cs.listed - cs.count - (cs.left > 0 ? 2 : 0)) >> 1),
                            ((publish_st > g_st ? min(publish_st - 1, end_st - 1) : end_st - 1) - g_st + 1) >> 1));
      if (pairs > 0) {
        kt += pairs * (2 * SK);
#pragma unroll 1
        do {
          __builtin_amdgcn_sched_barrier(0);
          s1 = scores_phase<D>(w, frag, s0, wt, sl2, slot(g_st), v_lane);
          const int id0 = list[cs.count & (kListed - 1)], id1 = list[(cs.count + 1) & (kListed - 1)];
          bf16x8 pb[2] = {wt.fragment(0), wt.fragment(1)};
          settle_weights<D>(w, s0, pb, wt.sum(), sl2);
          HFX_WAIT_VMCNT(0);
          ring_barrier();
          const char* base0 = block_base(uniform(id0));
          const char* base1 = block_base(uniform(id1));
          const unsigned lds0 = slot_lds(cs.count), lds1 = slot_lds(cs.count + 1);
          __builtin_amdgcn_sched_barrier(0);
          values_phase<D>(w, frag, pb, s1, wt, sl2, slot(g_st + 2), k_lane, [&](int i) {
            if (i < D / 32) piece_copy(base0, voff, lds0, i);
            else piece_copy(base1, voff, lds1, i - D / 32);
          });
          s0 = scores_phase<D>(w, frag, s1, wt, sl2, slot(g_st + 1), v_lane);
          pb[0] = wt.fragment(0);
          pb[1] = wt.fragment(1);
          settle_weights<D>(w, s1, pb, wt.sum(), sl2);
          __builtin_amdgcn_sched_barrier(0);
          values_phase<D>(w, frag, pb, s0, wt, sl2, slot(g_st + 3), k_lane, NoCopy());
          g_st += 2;
          cs.count += 2;
        } while (--pairs > 0);
      }
      if (g_st == end_st) break;
      stage_step(s0, s1, true);
      if (g_st == end_st) {
        s0 = s1;
        break;
      }
      stage_step(s1, s0, false);
    }
    // the item's last stage: Q is not needed any more, and the next item's is asked for
    if (next_ok) q_load<D>(w.qf, nx.q, nx.q_row0, nx.q_last, Hq, n, j);
    if (kt < wave_end) {
      bf16x8 pb[2];
#pragma unroll
      for (int i = 0; i < D / 16; ++i) frag[i] = value_fragment<D>(slot(g_st), i, v_lane);
      wt.portion(Share<D>::values[D / 16 - 1], 8, 12, s0, sl2, w.m);
      wt.portion(8, 12, 16, s0, sl2, w.m);
      wt.portion(12, 16, 16, s0, sl2, w.m);
      pb[0] = wt.fragment(0);
      pb[1] = wt.fragment(1);
      settle_weights<D>(w, s0, pb, wt.sum(), sl2);
      if (kt + SK > ctx_len) mask_values(frag);
#pragma unroll
      for (int i = 0; i < D / 16; ++i)
        w.o[i % (D / 32)] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag[i], pb[i / (D / 32)], w.o[i % (D / 32)], 0, 0, 0);
    }
    ++g_st;
    // hand-over: the item is finished; its successor's first stages are in the ring or on their way.  The records of the
    // successor and of the item after that are asked for ahead of the store; a workgroup's last item waits for none.
    tickets_take(t, s_tk, n_items);
    if (!next_ok) {
      prefill_store<D>(a, H, it, wr, w, Hq, wave, lane, stage);
      break;
    }
    const HfxItem item_c = items[t.cur];
    const HfxItem item_n = items[t.nxt < n_items ? t.nxt : t.cur];
    if (!cs.in_next) list_start(nx);
    cs.in_next = 0;
    nx = next_item(item_n);
    next_ok = t.nxt < n_items && item_n.type == HFX_ITEM_PREFILL;
    list_ask();
    prefill_store<D>(a, H, it, wr, w, Hq, wave, lane, stage);
    it = item_c;
    wr = wave_rows(it, wave);
    set_ticket_points();
    pending = 0;
    if (n_st <= 6) tickets_reserve(t, pending, ctrl);
    // Q is needed by the next MFMA; waiting for it in so many words also tells the compiler that
    // nothing is in flight when the stage loop is re-entered
    if (n_st <= 6) tickets_publish(t, pending, s_tk, ctrl, H);
    HFX_WAIT_VMCNT(0);
    list_write();
    // the list went no further than the last item, or less far than its first stages: these are waited for
    if (cs.count < g_st + min(n_st, 2)) {
      list_until(cs.limit);
      copy_stages(min(cs.limit, cs.listed) - cs.count, list_read());
      HFX_WAIT_VMCNT(0);
    }
  }
  __syncthreads();     // every wavefront is done with the ring before the LDS is used for anything else
}

// ----------------------------------------------------------------------------------------------
// The persistent kernel: workgroups pull items in descending modelled cost until the queue is
// empty.  A workgroup always knows its next item (see Tickets).  The queue counters live in the
// descriptor; the last workgroup to leave a launch that uses them restores them to zero so the descriptor can serve the
// next one.
// ----------------------------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(HFX_WG_THREADS, 2) void mixed_attention_kernel(
    const HfxHeader hdr, const char* __restrict__ desc, int* __restrict__ ctrl, const __bf16* __restrict__ q,
    const __bf16* __restrict__ pool, float* __restrict__ ws, __bf16* __restrict__ out) {
  // The descriptor's header travels as a kernel argument (the host has it anyway), which takes one
  // dependent load off the start of every workgroup.
  // The descriptor tables are read-only and distinct from everything written here, which lets
  // the compiler fetch them with scalar loads that do not queue behind the KV stream
  KArgs a;
  a.desc = desc;
  a.q = q;
  a.pool = pool;
  a.ws = ws;
  a.out = out;
  __shared__ __attribute__((aligned(1024))) char smem[Smem<D>::kBytes];
  __shared__ int s_tk[2];
  // result rows on their way out (prefill_store)
  __shared__ __attribute__((aligned(128))) char s_ostage[4 * 2048];
  __shared__ int s_ids[4 * kListed];     // blocks of stages to come (prefill_run)
  const HfxHeader* H = &hdr;
  const HfxItem* items = reinterpret_cast<const HfxItem*>(a.desc + H->off_items);
  const int n_items = H->n_items;
  Tickets t;
  t.cur = (int)blockIdx.x;
  t.nxt = (int)(blockIdx.x + gridDim.x);
  if (hdr.deal_balanced) deal_balanced(t, (int)hdr.deal_balanced, n_items);
  t.order = nullptr;
  if (H->off_queue) {
    t.order = reinterpret_cast<const int*>(a.desc + H->off_queue);
    if (t.cur < n_items) t.cur = t.order[t.cur];
    if (t.nxt < n_items) t.nxt = t.order[t.nxt];
  }
  t.own = (int)H->die_items > kDealtTickets * (int)gridDim.x;
  t.parity = 0;
  t.queue = n_items > kDealtTickets * (int)gridDim.x;
  while (t.cur < n_items) {
    if (items[t.cur].type == HFX_ITEM_DECODE) {
      decode_run<D>(a, H, items, n_items, t, s_tk, &ctrl[0], smem);
    } else {
      prefill_run<D>(a, H, items, n_items, t, s_tk, &ctrl[0], smem, s_ostage, s_ids);
    }
  }
  // the ticket fetched last is never used; it must have reached the counter before this
  // workgroup reports itself finished, or it could land after the reset below
  HFX_WAIT_VMCNT(0);
  asm volatile("" ::: "memory");
  if (n_items > kDealtTickets * (int)gridDim.x && threadIdx.x == 0) {
    // the workgroups of a class count themselves, and its last one the classes
    const int cls = (int)blockIdx.x & (HFX_QUEUE_CLASSES - 1);
    if (atomicAdd(ctrl + HFX_CTRL_DONE(cls), 1) == ((int)gridDim.x - cls + HFX_QUEUE_CLASSES - 1) / HFX_QUEUE_CLASSES - 1 &&
        atomicAdd(ctrl + HFX_CTRL_DONE(HFX_QUEUE_CLASSES), 1) == min((int)gridDim.x, HFX_QUEUE_CLASSES) - 1) {
      for (int c = 0; c < HFX_QUEUE_CLASSES; ++c) {
        atomicExch(ctrl + HFX_CTRL_TICKETS(c), 0);
        atomicExch(ctrl + HFX_CTRL_DONE(c), 0);
      }
      atomicExch(ctrl + HFX_CTRL_SHARED, 0);
      atomicExch(ctrl + HFX_CTRL_DONE(HFX_QUEUE_CLASSES), 0);
    }
  }
}

// Upload of a staging buffer that the GPU can read (pinned host memory): 8-byte words, four of a thread in flight.  Loads of
// system scope, so that no cache of the GPU answers with what the buffer held before.  Bound: the host link.
// An engine uploads the next step's descriptor while the present step's attention runs.  Two workgroups of that kernel with 128-wide heads take
// 2 * 248 of a SIMD's 512 registers (247 a lane, handed out eight at a time), so this one takes no more than 16: with 18 it
// found no place until the first workgroups of the launch ended.  And a CU answers its loads in order, so that one which
// hosts a workgroup of this kernel waits for the host link with all it has: few of them, going round a loop, 2 KB a wavefront.
// Steps of 384 and 1152 short requests (0.94 and 2.96 MB), us a step, uploaded beside the launch before and, second, ahead of the launch
// on the same stream: by a copy engine 315.3 and 339.4, 1063 and 1116; one workgroup for each 8 KB with 18 registers 324.0 and 329.8,
// 1105 and 1110, with 16 registers 320.2 and 328.5, 1091 and 1108; 128 workgroups 320.5 and 328.6, 1080 and 1107; 32 315.3 and 328.3,
// 1063 and 1107; 12 315.8 and 329.8, 1064 and 1110.
constexpr unsigned kUploadWgs = 32;
__device__ __forceinline__ void upload_words(const char* __restrict__ src, char* __restrict__ dst, unsigned words, unsigned workgroup, unsigned workgroups) {
  const int word = (threadIdx.x >> 6) * 256 + (threadIdx.x & 63);       // and 64, 128, 192 further on: one address for all four
  for (unsigned first = workgroup * 1024; first < words; first += workgroups * 1024) {
    const int left = (int)min(words - first, 1024u) - word;
    const uint64_t* from = reinterpret_cast<const uint64_t*>(src) + first + word;
    uint64_t* to = reinterpret_cast<uint64_t*>(dst) + first + word;
    uint64_t v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (64 * j < left) v[j] = __hip_atomic_load(from + 64 * j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (64 * j < left) to[64 * j] = v[j];
  }
}
__global__ __launch_bounds__(256) void upload_kernel(const char* __restrict__ src, char* __restrict__ dst, unsigned words) {
  upload_words(src, dst, words, blockIdx.x, gridDim.x);
}

// ---------------------------------------------------------------------------------------
// Page copy: pool pages named by (src, dst) id pairs move between two pools of the same
// geometry (or inside one).  The device half of handing a request's KV blocks from the
// instance that prefilled it to the instance that decodes it (HFX Section 3.3.1,
// disaggregated mode; Section 3.4).  16-byte units, of which a page has 256, 512 or a multiple of
// 1024 (1, 2 or a multiple of 4 kv-heads); a workgroup moves 16 KB with all of its
// loads in flight before the first store.  The page of a 4 KB piece is the same for the whole workgroup, so that its id
// is one scalar load and nothing is divided per thread.
// Stream: the pages are not read again, nor do they find a place in the last-level cache.
// Bound: memory.  In pieces of 64 KB a die, copies past the caches are 2 to 3 % faster than in pieces of 16 KB: 134 MB each way 58.2 us a call and
// 59.6, 268 MB 109.3 and 113.3; runs of 8 to 32 workgroups are like 4, smaller copies the same either way.
// N: pairs that come with the arguments; 0: they are in device memory.  An upload kernel ahead of this one costs 5 us of a short copy, for a
// list that fits the arguments of a launch.  Of a longer list the arguments hold the first N, and workgroups ahead of those that copy upload the rest
// for a second launch meanwhile.
// ---------------------------------------------------------------------------------------
constexpr int kFewPairs = 60, kMostPairs = 496;      // the latter fill the 4 KB that the arguments of a launch may take
struct ListRest {
  const char* from;
  char* to;
  unsigned words, workgroups;     // the first `workgroups` of the launch upload: a multiple of 8
};
template <int N>
struct PagePairs {
  int2 id[N];
};
template <>
struct PagePairs<kMostPairs> {
  int2 id[kMostPairs];
  ListRest rest;
};
static_assert(sizeof(PagePairs<kMostPairs>) + 32 <= 4096, "with the kernel's other arguments");
template <>
struct PagePairs<0> {
  const int2* id;
};
template <bool Stream, int N>
__global__ __launch_bounds__(256) void copy_pages_kernel(const PagePairs<N> pairs, long n_pairs, unsigned units_per_page,
                                                         const u32x4* __restrict__ src, u32x4* __restrict__ dst) {
  constexpr unsigned kPiece = 256, kPieces = 4;
  const bool whole = units_per_page >= kPieces * kPiece;        // the workgroup stays inside a page
  const unsigned per_page = whole ? units_per_page / (kPieces * kPiece) : 1;
  // Workgroups go to the dies by their index modulo 8: of 32 in a row a die takes four that follow each other, 64 KB.
  constexpr unsigned kDies = HFX_QUEUE_CLASSES, kRun = 4;
  unsigned index = blockIdx.x, count = gridDim.x;
  if constexpr (N == kMostPairs) {
    if (index < pairs.rest.workgroups) {
      upload_words(pairs.rest.from, pairs.rest.to, pairs.rest.words, index, pairs.rest.workgroups);
      return;
    }
    index -= pairs.rest.workgroups;
    count -= pairs.rest.workgroups;
  }
  if (index < count / (kDies * kRun) * (kDies * kRun))
    index = index / (kDies * kRun) * (kDies * kRun) + index % kDies * kRun + index / kDies % kRun;
  const unsigned page = index / per_page, part = index - page * per_page;
  u32x4 v[kPieces];
  long to[kPieces];
#pragma unroll
  for (unsigned j = 0; j < kPieces; ++j) {
    const unsigned unit = part * (kPieces * kPiece) + j * kPiece;
    const unsigned skip = whole ? 0 : unit / units_per_page;     // small pages: this piece's, from the workgroup's first
    const long pr = whole ? (long)page : (long)page * (kPieces * kPiece / units_per_page) + skip;
    to[j] = -1;
    if (pr < n_pairs) {
      const int2 id = pairs.id[pr];
      const unsigned off = unit - skip * units_per_page + threadIdx.x;
      const u32x4* from = src + (long)id.x * units_per_page + off;
      v[j] = Stream ? __builtin_nontemporal_load(from) : *from;
      to[j] = (long)id.y * units_per_page + off;
    }
  }
#pragma unroll
  for (unsigned j = 0; j < kPieces; ++j)
    if (to[j] >= 0) __builtin_nontemporal_store(v[j], dst + to[j]);
}

// Page gather: a workgroup of 2 D threads takes one (page, kv-head) at a time.  A thread moves one 16-byte
// piece of keys, taken in the order of the destination rows (a row of D elements leaves whole; four rows are
// 128 contiguous bytes of the source block), and one of values, which are dimension-major in the
// pool and turn round in LDS: a piece is 8 slots of one dimension there and 8 dimensions of one
// slot on the way out.  Rows in LDS are 16 bytes longer than the data, which spreads the 2-byte
// writes of one piece and the 16-byte reads of one row over the banks.  Bound: memory, 4 D Hkv bytes a
// token each way.  (12345 tokens of 8 kv-heads, 101 MB: 16.4 us a call on the same buffers, which stay in the 256 MB
// last-level cache, 6.1 TB/s; 20.9 us, 4.8 TB/s, rotating over eight sets of buffers, from HBM.  One thread per element with
// 64-bit divisions took 44.7 us on the same buffers.)
template <int D>
__global__ __launch_bounds__(2 * D) void gather_kv_kernel(const char* __restrict__ desc, const uint16_t* __restrict__ pool,
                                                          int request, uint16_t* __restrict__ k_out,
                                                          uint16_t* __restrict__ v_out) {
  constexpr int LD = D + 8;                       // LDS row stride in elements
  __shared__ __attribute__((aligned(16))) uint16_t sv[2][HFX_PAGE * LD];
  const HfxHeader* H = reinterpret_cast<const HfxHeader*>(desc);
  const HfxReq rq = reinterpret_cast<const HfxReq*>(desc + H->off_req)[request];
  const int* bt = reinterpret_cast<const int*>(desc + H->off_bt) + rq.bt_start;
  const int Hkv = H->num_kv_heads, tid = threadIdx.x;
  const int slot = tid / (D / 8), piece = tid % (D / 8);          // destination row and 16-byte piece of it
  const int d = tid >> 1, s0 = (tid & 1) * 8;                     // source row of the values and half of it
  const long units = (long)rq.n_pages * Hkv;
  int buf = 0;
  for (long u = blockIdx.x; u < units; u += gridDim.x, buf ^= 1) {
    const int page = (int)(u / Hkv), g = (int)(u - (long)page * Hkv);
    const uint16_t* kblk = pool + (((long)bt[page] * Hkv + g) * 2) * (16L * D);
    const u32x4 kv = *reinterpret_cast<const u32x4*>(kblk + ((piece >> 1) * HFX_PAGE + slot) * 16 + (piece & 1) * 8);
    const u32x4 vv = *reinterpret_cast<const u32x4*>(kblk + 16 * D + tid * 8);
    uint16_t* row = sv[buf];
#pragma unroll
    for (int e = 0; e < 8; ++e) row[(s0 + e) * LD + d] = (uint16_t)(vv[e >> 1] >> (16 * (e & 1)));
    __syncthreads();           // the only one: the next unit is written to the other buffer
    const long t = (long)page * HFX_PAGE + slot;
    if (t < rq.ctx_len) {
      const long to = (t * Hkv + g) * D + piece * 8;
      __builtin_nontemporal_store(kv, reinterpret_cast<u32x4*>(k_out + to));
      __builtin_nontemporal_store(*reinterpret_cast<const u32x4*>(row + slot * LD + piece * 8), reinterpret_cast<u32x4*>(v_out + to));
    }
  }
}

// The same for buffers that are not 16-byte aligned: one thread per (token, kv-head, dimension).
__global__ void gather_kv_unaligned_kernel(const char* desc, const uint16_t* pool, int request, uint16_t* k_out,
                                           uint16_t* v_out) {
  const HfxHeader* H = reinterpret_cast<const HfxHeader*>(desc);
  const HfxReq rq = reinterpret_cast<const HfxReq*>(desc + H->off_req)[request];
  const int* bt = reinterpret_cast<const int*>(desc + H->off_bt) + rq.bt_start;
  const int Hkv = H->num_kv_heads, D = H->head_dim;
  const long total = (long)rq.ctx_len * Hkv * D;
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (long)gridDim.x * blockDim.x) {
    const int d = (int)(i % D);
    const int g = (int)((i / D) % Hkv);
    const long t = i / ((long)D * Hkv);
    const long pg = bt[t / HFX_PAGE];
    const int slot = (int)(t % HFX_PAGE);
    const long blk = ((pg * Hkv + g) * 2) * (16L * D);
    k_out[i] = pool[blk + ((long)(d / 16) * HFX_PAGE + slot) * 16 + d % 16];
    v_out[i] = pool[blk + 16L * D + (long)d * HFX_PAGE + slot];
  }
}

// KV append: one workgroup of 2 D threads per (run, kv-head), a run being the new tokens of one request that
// fall into one page (at most 16 consecutive slots).  A thread takes one 16-byte piece of a token's key
// row and one of its value row, both loads at once.  Keys go straight to the pool's block order (four
// slots are 128 contiguous bytes there); values are dimension-major in the pool and turn round in LDS, so that
// a row of the block (one dimension) gets its run of slots as one contiguous piece -- stored token by token,
// it took one 2-byte request per (token, dimension), which was most of the launch.  Bound: memory, 4 D bytes a
// token and head each way.  (8224 tokens of long chunks, 8 kv-heads, 67 MB: 11.3 us a call on the same buffers, in the
// last-level cache, 6.0 TB/s, 12.7 with 4-byte loads in a loop and both halves through LDS; 17.1 us, 3.9 TB/s, rotating over
// ten sets of buffers, from HBM.  36940 tokens of short prompts, 303 MB: 68.7 us, 4.4 TB/s, and 72.4.)
template <int D>
__global__ __launch_bounds__(2 * D) void append_kv_kernel(const HfxRun* __restrict__ runs, int n_runs, unsigned die_row_log2,
                                                          const uint16_t* __restrict__ k_new,
                                                          const uint16_t* __restrict__ v_new,
                                                          uint16_t* __restrict__ pool) {
  constexpr int LD = D + 8;                       // LDS row stride in elements
  __shared__ __attribute__((aligned(16))) uint16_t sv[HFX_PAGE * LD];
  // Workgroups go to the dies by their index modulo 8: of 8 << die_row_log2 in a row a die takes 1 << die_row_log2 that follow each other.
  const unsigned heads = gridDim.x, all = heads * (unsigned)n_runs, row = (1u << die_row_log2) - 1, group = 8 * row + 7;
  unsigned block = (blockIdx.z * gridDim.y + blockIdx.y) * heads + blockIdx.x;
  if (block >= all) return;
  if (block < (all & ~group)) block = (block & ~group) | (block & 7) << die_row_log2 | (block >> 3 & row);
  const int index = (int)(block / heads);
  const HfxRun run = runs[index];
  const int Hkv = (int)heads, g = (int)(block - (unsigned)index * heads), tid = threadIdx.x;
  uint16_t* kblk = pool + (((long)run.page * Hkv + g) * 2) * (16L * D);
  const int tok = tid / (D / 8), piece = tid % (D / 8);
  if (tok < run.n) {
    const long src = ((long)(run.row0 + tok) * Hkv + g) * D + piece * 8;
    const u32x4 kv = *reinterpret_cast<const u32x4*>(k_new + src);
    const u32x4 vv = *reinterpret_cast<const u32x4*>(v_new + src);
    // K block [D/16][16 slots][16]
    *reinterpret_cast<u32x4*>(kblk + ((piece >> 1) * HFX_PAGE + run.slot0 + tok) * 16 + (piece & 1) * 8) = kv;
    *reinterpret_cast<u32x4*>(sv + (run.slot0 + tok) * LD + piece * 8) = vv;
  }
  __syncthreads();
  // V block [D][16 slots]: this thread has 8 slots of dimension tid / 2; slots outside the run hold what was in
  // LDS and are not stored
  const int d = tid >> 1, s0 = (tid & 1) * 8;
  uint16_t* dst = kblk + 16L * D + tid * 8;
  const int lo = run.slot0 - s0, hi = lo + run.n;     // the run, relative to the thread's slots
  if (lo >= 8 || hi <= 0) return;
  uint16_t x[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) x[e] = sv[(s0 + e) * LD + d];
  if (lo <= 0 && hi >= 8) {
    u32x4 v;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = (uint32_t)x[2 * e] | ((uint32_t)x[2 * e + 1] << 16);
    *reinterpret_cast<u32x4*>(dst) = v;
  } else {
    // part of them: two at a time where both belong to the run
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const int a = 2 * w, b = 2 * w + 1;
      const bool in_a = a >= lo && a < hi, in_b = b >= lo && b < hi;
      if (in_a && in_b) *reinterpret_cast<uint32_t*>(dst + a) = (uint32_t)x[a] | ((uint32_t)x[b] << 16);
      else if (in_a) dst[a] = x[a];
      else if (in_b) dst[b] = x[b];
    }
  }
}

// ------------------------------------------------------------------ static workspace
// Split partials for callers that cannot allocate device memory: a fixed array inside the code
// object, one copy per GPU, held until the process ends.  In host code the array's name is only a
// handle for hipGetSymbolAddress; the device address it yields (per device) is what launches get.
static __device__ __align__(256) unsigned char scratch[HFX_STATIC_WS_BYTES];

hipError_t static_workspace(void** ptr) {
  static std::mutex mu;
  static void* addr[HFX_MAX_DEVICES];
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= HFX_MAX_DEVICES) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    addr[dev] = p;
  }
  *ptr = addr[dev];
  return hipSuccess;
}

// ------------------------------------------------------------------ host-side launch helpers
// Launches a kernel without dynamic LDS and answers for this launch alone.  (hipGetLastError() names the last error of any
// earlier call of the thread: with one that the caller had not read yet, work was enqueued and HFX_ERR_DEVICE returned.)  The error
// of a launch that fails is read here, because the caller learns of it; an older one stays the caller's to read.
template <typename... P, typename... A>
static hipError_t launch(void (*kernel)(P...), dim3 grid, unsigned threads, hipStream_t stream, const A&... args) {
  static_assert(sizeof...(P) == sizeof...(A), "one value for each parameter");
  auto call = [&](P... values) {
    void* address[] = {(void*)&values...};
    return hipLaunchKernel(reinterpret_cast<const void*>(kernel), grid, dim3(threads), address, 0, stream);
  };
  const hipError_t e = call(args...);
  if (e != hipSuccess) (void)hipGetLastError();
  return e;
}

hipError_t max_resident_workgroups(int head_dim, int* per_cu) {
  if (head_dim == 128)
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(per_cu, mixed_attention_kernel<128>, HFX_WG_THREADS, 0);
  return hipOccupancyMaxActiveBlocksPerMultiprocessor(per_cu, mixed_attention_kernel<64>, HFX_WG_THREADS, 0);
}

hipError_t launch_mixed_attention(const HfxHeader& h, int grid, void* desc, const void* q, const void* pool, void* ws,
                                  void* out, hipStream_t stream) {
  const int head_dim = h.head_dim, n_units = h.n_units;
  HfxHeader hk = h;          // as the kernel gets it: how the first tickets are dealt also depends on the grid
  if (grid != HFX_PLAN_WGS) hk.die_items = 0;      // every class needs its workgroups
  if (h.deal_balanced)
    hk.deal_balanced = grid == HFX_PLAN_WGS ? 1u : grid > HFX_PLAN_WGS / 2 && grid == h.n_items ? 2u : 0u;
  const char* d = static_cast<const char*>(desc);
  int* ctrl = reinterpret_cast<int*>(static_cast<char*>(desc) + h.off_ctrl);
  const __bf16* qp = static_cast<const __bf16*>(q);
  const __bf16* pp = static_cast<const __bf16*>(pool);
  float* wp = static_cast<float*>(ws);
  __bf16* op = static_cast<__bf16*>(out);
  hipError_t e = launch(head_dim == 128 ? mixed_attention_kernel<128> : mixed_attention_kernel<64>, dim3(grid), HFX_WG_THREADS, stream, hk, d, ctrl, qp,
                        pp, wp, op);
  if (e == hipSuccess && n_units > 0) {
    const HfxUnit* units = reinterpret_cast<const HfxUnit*>(d + h.off_units);
    const HfxGroup* groups = reinterpret_cast<const HfxGroup*>(d + h.off_groups);
    const float* ml = reinterpret_cast<const float*>(static_cast<const char*>(ws) + h.ws_off_ml);
    const int Hq = h.num_q_heads, G = h.num_q_heads / h.num_kv_heads;
    e = launch(head_dim == 128 ? merge_kernel<128> : merge_kernel<64>, dim3(n_units), HFX_WG_THREADS, stream, units, groups, wp, ml, Hq, G, op);
  }
  return e;
}

// Whether a kernel on `stream` may copy `bytes` from host to device by itself: from pinned memory that the GPU sees under the same
// address to memory of the stream's own GPU, which is the current one, both whole inside one allocation.  (A query of
// any other address succeeds and tells of no memory; it leaves no error behind.)
static bool kernel_may_upload(const void* host, const void* device, size_t bytes, hipStream_t stream) {
  if (((reinterpret_cast<uintptr_t>(host) | reinterpret_cast<uintptr_t>(device) | bytes) & 7u) != 0 || bytes >> 34 != 0) return false;    // 2^31 words
  struct Memory {
    unsigned type = hipMemoryTypeUnregistered;
    int gpu = -1;
    void* on_gpu = nullptr;
    char* start = nullptr;
    size_t size = 0;
  } from, to;
  auto query = [](const void* p, Memory* m) {
    hipPointer_attribute which[] = {HIP_POINTER_ATTRIBUTE_MEMORY_TYPE, HIP_POINTER_ATTRIBUTE_DEVICE_ORDINAL, HIP_POINTER_ATTRIBUTE_DEVICE_POINTER,
                                    HIP_POINTER_ATTRIBUTE_RANGE_START_ADDR, HIP_POINTER_ATTRIBUTE_RANGE_SIZE};
    void* answer[] = {&m->type, &m->gpu, &m->on_gpu, &m->start, &m->size};
    return hipDrvPointerGetAttributes(5, which, answer, const_cast<void*>(p)) == hipSuccess;
  };
  auto whole = [&](const void* p, const Memory& m) {
    const char* at = static_cast<const char*>(p);
    return at >= m.start && (size_t)(at - m.start) <= m.size && m.size - (size_t)(at - m.start) >= bytes;
  };
  if (!query(host, &from) || from.type != hipMemoryTypeHost || from.on_gpu != host || !whole(host, from)) return false;
  if (!query(device, &to) || to.type != hipMemoryTypeDevice || !whole(device, to)) return false;
  int current = -1;
  if (hipGetDevice(&current) != hipSuccess || current != to.gpu) return false;
  // the handles that name a stream of the current GPU without being one: asked for the GPU of these, the runtime follows them
  if (stream == nullptr || stream == hipStreamLegacy || stream == hipStreamPerThread) return true;
  hipDevice_t streams = -1;
  return hipStreamGetDevice(stream, &streams) == hipSuccess && streams == to.gpu;
}

// Pinned memory is read by a kernel: the runtime gives a megabyte to a copy engine, and the next kernel on the same stream started 10 to
// 20 us after that engine's end; a few kilobytes it copies with a kernel too.  What that gives and costs is said at upload_kernel.
hipError_t upload(const void* host, void* device, size_t bytes, hipStream_t stream) {
  if (bytes == 0) return hipSuccess;
  if (!kernel_may_upload(host, device, bytes, stream)) return hipMemcpyAsync(device, host, bytes, hipMemcpyHostToDevice, stream);
  const unsigned n = (unsigned)(bytes / 8);
  return launch(upload_kernel, dim3(std::min((n + 1023u) / 1024u, kUploadWgs)), 256, stream, static_cast<const char*>(host), static_cast<char*>(device), n);
}

// Copies of at most a quarter of the last-level cache leave their source in it, where it may still be from the writing of those pages (41 MB
// each way, three sets of buffers in turn: 21.1 us, 25.1 streaming; 134 MB 61.2 and 60.2; all with the list uploaded ahead).  With a division by the
// page size for each 16 bytes the kernel took 26.8 and 61.2.  (Where two sets of 134 MB alternate, half of the source is still in the cache and the
// line could lie higher: 49.4 us instead of 59.5.)
constexpr long kCopyStreamBytes = 64l << 20;
template <int N>
static hipError_t launch_copy_pages(const PagePairs<N>& pairs, long n_pairs, unsigned units_per_page, bool past_cache, unsigned others, const void* src,
                                    void* dst, hipStream_t stream) {
  const long blocks = (n_pairs * units_per_page + 1023) / 1024 + others;
  if (blocks > 0x7fffffffL) return hipErrorInvalidValue;
  return launch(past_cache ? copy_pages_kernel<true, N> : copy_pages_kernel<false, N>, dim3((unsigned)blocks), 256, stream, pairs,
                n_pairs, units_per_page, static_cast<const u32x4*>(src), static_cast<u32x4*>(dst));
}

// Whether launches on `stream` are being recorded.  The stream of the null handle cannot be.
static bool may_be_captured(hipStream_t stream) {
  if (stream == nullptr || stream == hipStreamLegacy) return false;
  hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
  return hipStreamIsCapturing(stream, &status) != hipSuccess || status != hipStreamCaptureStatusNone;
}

// The list goes with the launch where an upload kernel would carry it; the host hands over all of the argument block, so there are
// two sizes.  A recorded launch reads the staging buffer when it is replayed, and goes on doing so.  Copies of pages of 8 kv-heads of 128,
// called in a row: 2 to 50 pages 13.1 us uploaded, 11.1 with 60 in the arguments, 11.8 with 496; 188 pages 13.7 and 12.1; 494 pages 17.5 and 14.5.
// Longer lists, uploaded ahead of the copy and, second, beside the first 496 pages: 563 pages 18.8 and 17.9, 688 21.0 and 19.6, 1250 39.1 and 37.9,
// 4096 109.0 and 108.0; 4063 of 32 KB 27.9 and 26.2.
hipError_t copy_pages(const void* host, void* device, long n_pairs, unsigned units_per_page, const void* src, void* dst, hipStream_t stream) {
  const size_t bytes = sizeof(int2) * (size_t)n_pairs;
  const bool past_cache = n_pairs * units_per_page * 16 > kCopyStreamBytes;
  const PagePairs<0> all = {static_cast<const int2*>(device)};
  if (!kernel_may_upload(host, device, bytes, stream) || may_be_captured(stream)) {
    const hipError_t e = upload(host, device, bytes, stream);
    return e != hipSuccess ? e : launch_copy_pages(all, n_pairs, units_per_page, past_cache, 0, src, dst, stream);
  }
  if (n_pairs <= kFewPairs) {
    PagePairs<kFewPairs> few;
    std::memcpy(few.id, host, bytes);
    return launch_copy_pages(few, n_pairs, units_per_page, past_cache, 0, src, dst, stream);
  }
  const long n = std::min<long>(n_pairs, kMostPairs), left = n_pairs - n;
  PagePairs<kMostPairs> most;
  std::memcpy(most.id, host, sizeof(int2) * (size_t)n);
  const unsigned words = (unsigned)left, workgroups = std::min((words + 8191u) / 8192u * 8u, kUploadWgs);
  most.rest = {static_cast<const char*>(host) + 8 * n, static_cast<char*>(device) + 8 * n, words, workgroups};
  const hipError_t e = launch_copy_pages(most, n, units_per_page, past_cache, workgroups, src, dst, stream);
  return e != hipSuccess || left == 0 ? e : launch_copy_pages(PagePairs<0>{all.id + n}, left, units_per_page, past_cache, 0, src, dst, stream);
}

// Far more than are resident (8 to a CU), so that only very long requests go round the loop.
static const long kGatherMaxWgs = 8192;

hipError_t launch_gather_kv(const HfxHeader& h, int n_tokens, const void* desc, const void* pool, int request,
                            void* k_out, void* v_out, hipStream_t stream) {
  const char* ds = static_cast<const char*>(desc);
  const uint16_t* src = static_cast<const uint16_t*>(pool);
  uint16_t* ko = static_cast<uint16_t*>(k_out);
  uint16_t* vo = static_cast<uint16_t*>(v_out);
  // the pieces need 16-byte alignment, which the entry point does not ask of its callers
  if (((reinterpret_cast<uintptr_t>(pool) | reinterpret_cast<uintptr_t>(k_out) | reinterpret_cast<uintptr_t>(v_out)) & 15u) == 0) {
    const long units = (long)((n_tokens + HFX_PAGE - 1) / HFX_PAGE) * h.num_kv_heads;      // (page, kv-head) pairs
    const unsigned grid = (unsigned)std::min<long>(std::max<long>(units, 1), kGatherMaxWgs);
    return launch(h.head_dim == 128 ? gather_kv_kernel<128> : gather_kv_kernel<64>, dim3(grid), 2u * (unsigned)h.head_dim, stream, ds, src, request, ko, vo);
  }
  const long blocks = ((long)n_tokens * h.num_kv_heads * h.head_dim + 255) / 256;
  return launch(gather_kv_unaligned_kernel, dim3((unsigned)std::min<long>(std::max<long>(blocks, 1), 4096)), 256, stream, ds, src, request, ko, vo);
}

hipError_t launch_append_kv(const HfxHeader& h, const void* desc, const void* k_new, const void* v_new, void* pool,
                            hipStream_t stream) {
  if (h.n_runs <= 0) return hipSuccess;
  const HfxRun* runs = reinterpret_cast<const HfxRun*>(static_cast<const char*>(desc) + h.off_runs);
  // the heads of a run follow each other, so that what runs at the same time reads whole token rows (11.4 us on 8224
  // tokens, 11.7 with the runs of a head in a row); the runs fill the two slower dimensions, the first of
  // which holds at most 65535
  const unsigned per_z = (unsigned)std::min(h.n_runs, 32768);
  const dim3 grid((unsigned)h.num_kv_heads, per_z, ((unsigned)h.n_runs + per_z - 1) / per_z);
  // Pieces of 16 blocks a die where the pages go past the cache, of 4 otherwise.  One block, 4 and 16, us a call: 90000 tokens of 8 kv-heads 145.3, 140.8 and
  // 132.2, 36000 58.5, 57.0 and 54.7, 12000 18.2, 18.3 and 18.5, 8224 of long chunks beside 32 decodes 12.5, 12.5 and 13.1.
  const unsigned die_row_log2 = (long)h.n_runs * h.num_kv_heads * h.head_dim * (4 * HFX_PAGE) > kCopyStreamBytes ? 4u : 2u;
  return launch(h.head_dim == 128 ? append_kv_kernel<128> : append_kv_kernel<64>, grid, 2u * (unsigned)h.head_dim, stream, runs, h.n_runs, die_row_log2,
                static_cast<const uint16_t*>(k_new), static_cast<const uint16_t*>(v_new), static_cast<uint16_t*>(pool));
}

}  // namespace hfx
