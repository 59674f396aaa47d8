// Causal attention for many query rows (prefix prefill and candidate scoring), bf16, gfx950 MFMA.
//
// A work item is up to 64 consecutive positions of one sequence, one KV head and up to four of
// its query heads.  The workgroup has 8 waves: wave w owns head 4 * hg + w % 4 of the group and
// positions 32 (w / 4) .. + 31 of the item, which are its MFMA columns.  Two waves per SIMD let
// one wave's softmax run under the other's MFMAs, and the LDS only reaches its full read rate
// with eight waves per CU.
// One or two heads past a multiple of four take several items of a sequence to a workgroup (REST).
// Where that gives fewer workgroups than the chip has compute units, two waves share the 32
// columns of a head (prefill_attention_split_kernel), or four that score and four that add take two heads' (prefill_attention_pair_kernel): they
// score different key blocks and add different
// coordinates of the result, so that a row's sum runs over its keys in the same order as with one wave
// and has the same bits whatever else is in the launch (300 positions of the 8B shape after 1024 / 4096
// keys: 38 -> 19 / 108 -> 45 us).
// Keys are streamed page by page (64 keys) through LDS and shared by the waves: first the
// shared-prefix pages that are visible to the block, then (scoring) the sequence's own suffix
// pages.  Pages are stored in MFMA fragment order, so a page is copied to LDS as it is (by
// loads that write LDS directly, one to two steps ahead) and an operand is one
// conflict-free 16-byte read per lane.  Each item sees all keys of its rows, so
// it normalises and writes bf16 itself.  Operand mapping and the softmax scheme are those of
// the decode kernel (transposed scores, lazy base-2 reference maximum); the addition is the
// causal mask, applied only to blocks that reach past the first position of the item.
#include "kernels_mfma.h"

#include <algorithm>
#include <type_traits>

namespace mc {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) uint32_t v4u;
typedef __attribute__((ext_vector_type(2))) uint32_t v2u;

__device__ inline f32x16 mfma32p(v4u a, v4u b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                 __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
__device__ inline uint32_t pack2p_bf16(float a, float b) {
  typedef __attribute__((ext_vector_type(2))) float f32x2;
  typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
}

constexpr int PPG = 64;                       // keys per page

template <int HD> struct PTile {
  static constexpr int K_ELEMS = PPG * HD, V_ELEMS = PPG * HD, PAGE_ELEMS = K_ELEMS + V_ELEMS;
  static constexpr int NF = HD / 16;          // 1 KB fragments per 32-key block (K and V alike)
  static constexpr int CPT = PPG * HD / 8 / 512;            // 16-byte loads per thread and K (or V) page
};

// LDS of the two kernels
template <int HD> struct PWhole {              // pages of K and V together, three steps of one page
  static constexpr int STEPS = 3, LPS = 2 * PTile<HD>::CPT;   // LPS: loads into LDS per wave and step
  static constexpr int LDS_BYTES = STEPS * PTile<HD>::PAGE_ELEMS * 2;
};
template <int HD> struct PSplit {              // two waves per head: a step is two blocks, one page
  static constexpr int KS = 2, HEADS = 8 / KS;
  static constexpr int SLOTS = 3;                            // steps of K, and of V, held in LDS
  static constexpr int LPH = PTile<HD>::CPT;                 // loads into LDS per wave and step of K (of V)
  static constexpr int NDT = HD / 32 / KS;                   // 32-coordinate tiles of the result per wave
  static constexpr int K_BYTES = SLOTS * PTile<HD>::K_ELEMS * 2;
  // K slots, V slots, the probabilities of eight blocks, their sums and references, flags
  static constexpr int LDS_BYTES = 2 * K_BYTES + 8 * (2048 + 256 + 256) + 64;
};

constexpr int kPrefillMaxPids = 1024;
typedef __attribute__((address_space(3))) int lds_int;

// All but the newest N vector memory operations of this wave have landed, loads into LDS among them,
// (ALL_LDS: and its LDS reads and writes), then the workgroup's barrier.  (__syncthreads() would wait
// for every load in flight.)
template <int N, bool ALL_LDS = false>
__device__ inline void wait_barrier_p() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (ALL_LDS ? 0x0070 : 0x0F70));
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// The pages that positions up to last_pos see, in order: prefix keys [0, nA), then the own suffix's
// [0, nB) at absolute positions prefix_len + j.
struct PPages {
  int nA, nB, nPA, n, prefix_len;
  const int32_t *table;
  __device__ inline PPages(const PrefillAttnArgs &a, int tab, int last_pos) {
    prefix_len = a.prefix_len;
    nA = min(a.prefix_len, last_pos + 1);
    nB = (tab >= 0 && last_pos >= a.prefix_len) ? last_pos - a.prefix_len + 1 : 0;
    nPA = (nA + PPG - 1) / PPG;
    n = nPA + (nB + PPG - 1) / PPG;
    table = n > nPA ? a.page_table + (size_t)tab * a.table_stride : nullptr;
  }
  // ids of pages p0 .. p0 + 63, one per lane (0 past the end)
  __device__ inline int ids(int p0) const {
    const int p = p0 + (int)(threadIdx.x & 63);
    return p < nPA ? p : p < n ? table[p - nPA] : 0;
  }
  // 32-key block blk of page pi: the position of its key 0; returns how many of its keys exist
  __device__ inline int block(int pi, int blk, int &abs0) const {
    const bool in_a = pi < nPA;
    abs0 = (in_a ? pi * PPG : prefix_len + (pi - nPA) * PPG) + 32 * blk;
    return min(32, (in_a ? min(PPG, nA - pi * PPG) : min(PPG, nB - (pi - nPA) * PPG)) - 32 * blk);
  }
};

// Pages go from global memory straight into LDS (lane i of a wave-wide 16-byte load lands at
// the wave's base + 16 i: the page is copied as it is).  The same number of loads is issued whether or
// not the page exists (one past the end has a range of no bytes: nothing is fetched), so the waits can
// count.  They are buffer loads because the compiler counts those; after a global (flat) load
// into LDS it waits for everything in flight before the next use of any load.
__device__ inline __amdgpu_buffer_rsrc_t page_range(const bf16_t *page, bool exists, int hd) {
  return __builtin_amdgcn_make_buffer_rsrc((void *)page, 0, exists ? PPG * hd * (int)sizeof(bf16_t) : 0, 0x00020000);
}
// piece i of PTile<HD>::CPT; dst: this wave's part of the page's place in LDS
__device__ inline void load_piece(__amdgpu_buffer_rsrc_t r, bf16_t *dst, int i) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void *)(dst + 4096 * i), 16, threadIdx.x * 16, 8192 * i, 0, 0);
}

// Scores of keys that do not exist (from n_valid on) or lie after the lane's query position go to
// -infinity.  abs0: position of the block's key 0; key of register r: 8 (r / 4) + 4 h + r % 4.
__device__ inline void mask_scores(f32x16 &s, int n_valid, int abs0, int pos_start, int my_pos, int h) {
  if (n_valid < 32 || abs0 + 31 > pos_start) {
    const int lim = min(n_valid, my_pos - abs0 + 1);      // keys [0, lim) are visible
#pragma unroll
    for (int r = 0; r < 16; ++r)
      if (8 * (r >> 2) + 4 * h + (r & 3) >= lim) s[r] = -INFINITY;
  }
}

// Probabilities against the reference m as it stands (see the decode kernel: any reference gives the
// same normalised result, it only has to keep the numbers in range) and the lane's sum of them.
__device__ inline float block_probs(const f32x16 &s, float scale2, float m, f32x16 &p) {
  float rs = 0.f;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    p[r] = __builtin_amdgcn_exp2f(fmaf(s[r], scale2, -m));
    rs += p[r];
  }
  return rs;
}
// Only if a lane's sum leaves the range - a score far above the reference, or no reference yet (m =
// -inf yields inf or NaN) - the reference moves to the block's maximum and the accumulators are
// rescaled; the common case spends no instruction on maxima.
__device__ inline bool leaves_range(float rs) { return __any(!(rs <= kSoftmaxSumLimit)); }
__device__ inline float moved_reference(const f32x16 &s, float scale2, float m) {
  float mx = max16f(s);
  mx = fmaxf(mx, other_half(mx));
  return fmaxf(m, mx * scale2);                 // stays -inf for a column that has seen no key
}
__device__ inline float rescale_factor(float m, float m_new) {
  return (m_new == -INFINITY) ? 1.0f : __builtin_amdgcn_exp2f(m - m_new);
}
// a column with no visible key so far: 0 as reference, all its p are 0
__device__ inline float usable_reference(float m) { return (m == -INFINITY) ? 0.f : m; }
__device__ inline void pack_probs(const f32x16 &p, v4u (&pb)[2]) {
  pb[0] = v4u{pack2p_bf16(p[0], p[1]), pack2p_bf16(p[2], p[3]), pack2p_bf16(p[4], p[5]), pack2p_bf16(p[6], p[7])};
  pb[1] = v4u{pack2p_bf16(p[8], p[9]), pack2p_bf16(p[10], p[11]), pack2p_bf16(p[12], p[13]), pack2p_bf16(p[14], p[15])};
}

// coordinates 32 dt .. + 31 of this lane's row
template <int HD>
__device__ inline void store_tile(const PrefillAttnArgs &a, int row, int head, int dt, int h, const f32x16 &o, float inv) {
  bf16_t *out = (bf16_t *)a.out;
  const int Hq = a.n_q_heads;
#pragma unroll
  for (int r4 = 0; r4 < 4; ++r4) {
    const int d = dt * 32 + 8 * r4 + 4 * h;
    const size_t at = a.out_tiled ? tiled_offset(row, head * HD + d, Hq * HD) : ((size_t)row * Hq + head) * HD + d;
    v2u pk = {pack2p_bf16(o[4 * r4] * inv, o[4 * r4 + 1] * inv), pack2p_bf16(o[4 * r4 + 2] * inv, o[4 * r4 + 3] * inv)};
    *(v2u *)(out + at) = pk;
  }
}

// TILED_ZERO: block b takes eight 32-row tiles, marks the rows that the items cover (a thread per item: one round trip) and
// writes zeros to the others, where a fill of the whole output takes 5 us (300 rows of 4096) to 11 us
// (8192 rows).  The split kernel has such blocks behind those of its items, and they run beside them.  In the
// whole-item kernel the added code moved the loop's registers and its place (two sequences of 831 rows after 1940 keys,
// heads of 64: 57 -> 61 us), so there something is launched ahead of it: the same for an output that outgrows the L2s (8 x 1024
// rows of 4096: 600 -> 592 us for the call), a fill of the whole for a smaller one, whose lines the stores then find in L2
// (5 sequences of 350 to 700 rows: 63.8 us by the fill, 66.2 by the uncovered rows alone).
__device__ inline void zero_uncovered_rows(const PrefillAttnArgs &a, int b, int K) {
  __shared__ uint32_t cover[8];
  const int tid = threadIdx.x, row0 = 256 * b;
  if (tid < 8) cover[tid] = 0;
  __syncthreads();
  for (int i = tid; i < a.n_items; i += 512) {
    const int4 item = a.items[i];
    const int from = max(item.x, row0), to = min(item.x + item.y, row0 + 256);         // rows [from, to) of this block's
    for (int r = from; r < to; r = (r | 31) + 1) {
      const uint32_t upto = to > (r | 31) ? ~0u : (1u << (to & 31)) - 1;
      atomicOr(&cover[(r - row0) >> 5], upto & (~0u << (r & 31)));
    }
  }
  __syncthreads();
  for (int t = 0; t < 8 && row0 + 32 * t < a.rows; ++t) {
    const uint32_t bare = __builtin_amdgcn_readfirstlane(~cover[t]);
    if (bare == 0) continue;
    for (int k = 8 * tid; k < K; k += 8 * 512)
      for (uint32_t left = bare; left; left &= left - 1)
        *(v4u *)((bf16_t *)a.out + tiled_offset(row0 + 32 * t + __builtin_ctz(left), k, K)) = v4u{0, 0, 0, 0};
  }
}

__global__ __launch_bounds__(512) void zero_uncovered_rows_kernel(PrefillAttnArgs a) {
  zero_uncovered_rows(a, blockIdx.x, a.n_q_heads * a.head_dim);
}

__global__ __launch_bounds__(256) void zero_rows_kernel(v4u *out, size_t pieces) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i < pieces) out[i] = v4u{0, 0, 0, 0};
}
constexpr size_t kL2Bytes = 32u << 20;         // of the eight XCDs together

// Waves per SIMD: two at head_dim 128 (190 registers); at head_dim 64 (125 registers, 52 KB of LDS) two workgroups
// share a compute unit.  (With an upper bound of two there the second stays out: 8 x 1024 rows after 4096
// keys, 32 / 8 heads of 64, 339 -> 390 us.)
//
// REST: the heads past a multiple of four, one or two of them, would leave six or four of the eight waves idle, so their
// workgroup takes four or two neighbouring items, where those have the same keys.  Each of these items has a workgroup of its own in the grid
// (the lists are on the device), at its end and the first of each four or two before the others; those whose item an earlier one takes end at once.
// (In the items' order, workgroups that stay and others in turn, the dispatcher deals all that stay to the same quarter or half of the units.)
template <int HD, bool REST>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, HD == 64 ? 4 : 2)))
void prefill_attention_kernel(PrefillAttnArgs a) {
  using TL = PTile<HD>;
  using SP = PWhole<HD>;
  extern __shared__ __attribute__((aligned(16))) unsigned char plds_raw[];
  bf16_t *lds = (bf16_t *)plds_raw;
  lds_int *pids = (lds_int *)(plds_raw + SP::LDS_BYTES);
  const int tid = threadIdx.x, lane = tid & 63, col = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int Hq = a.n_q_heads, Hkv = a.n_kv_heads, G = Hq / Hkv, HG = (G + 3) / 4;

  int id = blockIdx.x;
  // KV heads first: with eight of them an XCD (workgroups are dealt to the eight in turn) meets one
  // head's keys and values only
  const int kvh = id % Hkv; id /= Hkv;
  int hg, n_near = 1, slot = 0;                 // items that the workgroup may take, this one's place among them
  const int rest = G & 3, two = rest >> 1;        // REST: one head or two (two = 0, 1) past a multiple of four
  if (REST && id >= a.n_items * (G >> 2)) {
    hg = G >> 2;
    n_near = 4 >> two;
    id -= a.n_items * hg;
    const int groups = (a.n_items + n_near - 1) >> (2 - two);
    slot = (id >= groups) + (id >= 2 * groups) + (id >= 3 * groups);
    id = ((id - slot * groups) << (2 - two)) + slot;
    if (id >= a.n_items) return;
  } else {
    hg = id % (REST ? G / 4 : HG);
    id /= REST ? G / 4 : HG;
  }
  // head within the group, half of the item's rows, the wave's item
  int hw = wave % 4, half = wave >> 2;
  const int4 first = a.items[id];              // row_start, n_rows (<= 64), pos_start, table row
  int4 item = first;
  const int tab = first.w;
  int last_pos = first.z + first.y - 1;        // of the whole workgroup: pages every wave helps to stage
  bool has_item = true;
  if (n_near > 1) {
    const int n_left = min(n_near - slot, a.n_items - id);
    const int before = a.items[max(id - 1, 0)].w;
    int4 near[4];                                // one round trip for all
#pragma unroll
    for (int i = 1; i < 4; ++i) near[i] = a.items[min(id + i, a.n_items - 1)];
    if (slot > 0 && before == tab) return;       // an earlier one has this item
    int n = 1;
#pragma unroll
    for (int i = 1; i < 4; ++i)
      if (n == i && i < n_left && near[i].w == tab) {
        last_pos = max(last_pos, near[i].z + near[i].y - 1);
        n = i + 1;
      }
    hw = wave & two;
    half = wave >> two & 1;
    const int which = wave >> (1 + two);
    has_item = which < n;
#pragma unroll
    for (int i = 1; i < 4; ++i)
      if (has_item && which == i) item = near[i];
  }
  const int n_rows = item.y;
  const int row_start = item.x + 32 * half;     // this wave's rows and their first position
  const int pos_start = item.z + 32 * half;
  const int my_rows = min(32, n_rows - 32 * half);
  const int g = 4 * hg + hw;
  const bool wave_active = g < G && my_rows > 0 && has_item;   // uniform per wave
  const int head = kvh * G + (g < G ? g : 0);
  const bool col_valid = col < my_rows;
  const int my_pos = pos_start + (col_valid ? col : 0);
  const int my_last = pos_start + my_rows - 1;     // last position of this wave's rows

  // visible keys: prefix [0, nA), then own suffix [0, nB) at absolute positions prefix_len + j.  (PPages says the
  // same; with it here 8 x 1024 rows after 4096 keys took 597 instead of 586 us.)
  const int nA = min(a.prefix_len, last_pos + 1);
  const int nB = (tab >= 0 && last_pos >= a.prefix_len) ? last_pos - a.prefix_len + 1 : 0;
  const int nPA = (nA + PPG - 1) / PPG, nPB = (nB + PPG - 1) / PPG, n_pages = nPA + nPB;
  const int32_t *table = (nPB > 0) ? a.page_table + (size_t)tab * a.table_stride : nullptr;
  const bool pids_in_lds = nPB <= kPrefillMaxPids;
  if (nPB > 0 && pids_in_lds) {
    for (int i = tid; i < nPB; i += 512) pids[i] = table[i];
    __syncthreads();
  }

  v4u qf[HD / 16];
  {
    // a wave without rows reads the item's first row (its result is never stored)
    const int qr = wave_active ? row_start + (col_valid ? col : 0) : item.x;
    const bf16_t *qrow = (const bf16_t *)a.q + ((size_t)qr * Hq + head) * HD + 8 * h;
#pragma unroll
    for (int c = 0; c < HD / 16; ++c) qf[c] = *(const v4u *)(qrow + 16 * c);
  }
  const float scale2 = 1.4426950408889634f / sqrtf((float)HD);
  f32x16 o[HD / 32];
#pragma unroll
  for (int dt = 0; dt < HD / 32; ++dt)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[dt][r] = 0.f;
  float m = -INFINITY, l = 0.f;

  const size_t page_stride = (size_t)Hkv * PPG * HD, head_off = (size_t)kvh * PPG * HD;
  const bf16_t *kA = (const bf16_t *)a.k_prefix, *vA = (const bf16_t *)a.v_prefix;
  const bf16_t *kB = (const bf16_t *)a.k_suffix, *vB = (const bf16_t *)a.v_suffix;
  // pages arrive SP::STEPS - 1 ahead of the one in use (see load_piece)
  auto page_of = [&](int pi) __attribute__((always_inline)) -> int {
    if (pi >= n_pages) return 0;
    if (pi < nPA) return pi;
    if (pids_in_lds) return __builtin_amdgcn_readfirstlane(pids[pi - nPA]);
    return __builtin_amdgcn_readfirstlane(table[pi - nPA]);
  };
  auto issue = [&](int pi, int page, int buf) __attribute__((always_inline)) {
    const bool in_a = pi < nPA;
    const size_t at = (size_t)page * page_stride + head_off;
    const __amdgpu_buffer_rsrc_t kr = page_range((in_a ? kA : kB) + at, pi < n_pages, HD);
    const __amdgpu_buffer_rsrc_t vr = page_range((in_a ? vA : vB) + at, pi < n_pages, HD);
    bf16_t *kt = lds + buf * TL::PAGE_ELEMS + wave * 512, *vt = kt + TL::K_ELEMS;   // buf: of a page
#pragma unroll
    for (int i = 0; i < TL::CPT; ++i) {
      load_piece(kr, kt, i);
      load_piece(vr, vt, i);
    }
  };
  // one 32-key block whose key 0 sits at absolute position abs0; n_valid keys exist
  auto process = [&](int buf, int blk, int n_valid, int abs0) __attribute__((always_inline)) {
    const bf16_t *kt = lds + buf * TL::PAGE_ELEMS, *vt = kt + TL::K_ELEMS;
    const bf16_t *kblk = kt + (blk * TL::NF * 64 + lane) * 8, *vblk = vt + (blk * TL::NF * 64 + lane) * 8;
    // all key fragments are asked for before the first MFMA, a value fragment after each: they
    // arrive under the score MFMAs and the softmax
    v4u kf[TL::NF], vf[TL::NF];
#pragma unroll
    for (int c = 0; c < TL::NF; ++c) kf[c] = *(const v4u *)(kblk + c * 512);
    __builtin_amdgcn_sched_barrier(0);
    f32x16 s;
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
    for (int c = 0; c < TL::NF; ++c) {
      s = mfma32p(kf[c], qf[c], s);
      vf[c] = *(const v4u *)(vblk + c * 512);
      __builtin_amdgcn_sched_barrier(0);
    }
    mask_scores(s, n_valid, abs0, pos_start, my_pos, h);
    f32x16 p;
    float rs = block_probs(s, scale2, m, p);
    if (leaves_range(rs)) {
      const float m_new = moved_reference(s, scale2, m), corr = rescale_factor(m, m_new);
      l *= corr;
      m = m_new;
#pragma unroll
      for (int dt = 0; dt < HD / 32; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[dt][r] *= corr;
      rs = block_probs(s, scale2, usable_reference(m), p);
    }
    rs += other_half(rs);
    l += rs;
    v4u pb[2];
    pack_probs(p, pb);
#pragma unroll
    for (int dt = 0; dt < HD / 32; ++dt)
#pragma unroll
      for (int sl = 0; sl < 2; ++sl) o[dt] = mfma32p(vf[dt * 2 + sl], pb[sl], o[dt]);
  };
  auto consume = [&](int pi, int buf, int blk) __attribute__((always_inline)) {
    const bool in_a = pi < nPA;
    const int abs_page = in_a ? pi * PPG : a.prefix_len + (pi - nPA) * PPG;
    const int keys_here = in_a ? min(PPG, nA - pi * PPG) : min(PPG, nB - (pi - nPA) * PPG);
    const int nv = min(32, keys_here - 32 * blk);
    if (nv > 0 && abs_page + 32 * blk <= my_last) process(buf, blk, nv, abs_page + 32 * blk);   // else all masked
  };

  int next_page = page_of(0);
  auto issue_next = [&](int pi, int buf) __attribute__((always_inline)) {
    issue(pi, next_page, buf);
    next_page = page_of(pi + 1);
  };
#pragma unroll
  for (int st = 0; st + 1 < SP::STEPS; ++st) issue_next(st, st);
  int buf = 0;
  // The loop's place among the 32-byte lines of the instruction fetch is fixed here (by s_nop, passed once): left to
  // the code before it, the same loop took 586 or 599 us at 8 x 1024 rows after 4096 keys, and at head_dim 64
  // 76 or 78 us at 2 x 607 rows after 3418.
  asm volatile(".p2align 5\n.fill %0, 4, 0xbf800000" ::"i"(HD == 128 ? 3 : 0));
  for (int pi = 0; pi < n_pages; ++pi) {
    // page pi has landed once at most the loads of the later ones that were issued are outstanding;
    // past the barrier that holds for every wave, and page pi - 1 is no longer read
    wait_barrier_p<(SP::STEPS - 2) * SP::LPS>();
    issue_next(pi + SP::STEPS - 1, buf >= 1 ? buf - 1 : SP::STEPS - 1);
    if (wave_active) {
      consume(pi, buf, 0);
      consume(pi, buf, 1);
    }
    buf = buf == SP::STEPS - 1 ? 0 : buf + 1;
  }
  wait_barrier_p<0>();                         // no load into LDS outlives the loop

  if (wave_active && col_valid) {
    const float inv = 1.0f / l;                  // l > 0: every row sees at least its own key
#pragma unroll
    for (int dt = 0; dt < HD / 32; ++dt) store_tile<HD>(a, row_start + col, head, dt, h, o[dt], inv);
  }
}

// The same with two waves for the 32 columns of a head: a workgroup has one half of an item's rows and
// four heads, and a step is a page, two blocks of 32 keys.  In a step wave kg of a head scores block kg and leaves
// its probabilities and their sums in LDS, all against the reference that stood when the step began;
// past a barrier every wave adds both blocks, in order, to the result coordinates it owns.  The first step
// waits for block 0's maximum instead; where a block's sums leave the range later, which is seldom, the blocks
// are done again one by one, the reference moving in between.  So a row's additions and references are those
// of one wave that walks all keys.  (States of separate key groups merged at the end are faster for few rows, but then a row's
// last bits change with the number of groups, that is with the launch.)
// A wave's chain bounds it: scores, exponentials, the probabilities' way through
// LDS, value products, two barriers, and what scalar work stands between.  Fragments are read half a step ahead of
// their use: K of the next step beside the value products, V under the scores; K's and V's slots are refilled at the
// barrier behind that, which
// gives a load 2 SLOTS - 1 half steps to land.
template <int HD>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
void prefill_attention_split_kernel(PrefillAttnArgs a, int n_main) {
  if ((int)blockIdx.x >= n_main) return zero_uncovered_rows(a, (int)blockIdx.x - n_main, a.n_q_heads * HD);
  using TL = PTile<HD>;
  using SP = PSplit<HD>;
  constexpr int NF = TL::NF, NDT = SP::NDT, KS = SP::KS;
  extern __shared__ __attribute__((aligned(16))) unsigned char plds_raw[];
  bf16_t *k_lds = (bf16_t *)plds_raw, *v_lds = (bf16_t *)(plds_raw + SP::K_BYTES);
  v4u *probs = (v4u *)(plds_raw + 2 * SP::K_BYTES);             // [8 waves][2][64]
  float *sums = (float *)(probs + 8 * 128), *refs = sums + 8 * 64;   // [8 waves][64]
  int *state = (int *)(refs + 8 * 64), *moved = state + 8;      // per wave: 0 no visible key, 1 scored, 2 out of range
  const int tid = threadIdx.x, lane = tid & 63, col = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int Hq = a.n_q_heads, Hkv = a.n_kv_heads, G = Hq / Hkv, HG = (G + SP::HEADS - 1) / SP::HEADS;

  int id = blockIdx.x;
  const int kvh = id % Hkv; id /= Hkv;
  const int hg = id % HG; id /= HG;
  // head, block of a step, half of the item's rows (waves of one kg on different SIMDs)
  const int hw = wave % SP::HEADS, kg = wave / SP::HEADS, half = id & 1;
  const int4 item = a.items[id >> 1];
  const int row_start = item.x + 32 * half, pos_start = item.z + 32 * half, my_rows = min(32, item.y - 32 * half);
  if (my_rows <= 0) return;                     // the whole workgroup: the item has no second half
  const int g = SP::HEADS * hg + hw;
  const bool active = g < G;                    // uniform per head
  const int head = kvh * G + (active ? g : 0);
  const bool col_valid = col < my_rows;
  const int my_pos = pos_start + (col_valid ? col : 0), my_last = pos_start + my_rows - 1;
  const PPages pages(a, item.w, my_last);

  v4u qf[NF];
  {
    const bf16_t *qrow = (const bf16_t *)a.q + ((size_t)(row_start + (col_valid ? col : 0)) * Hq + head) * HD + 8 * h;
#pragma unroll
    for (int c = 0; c < NF; ++c) qf[c] = *(const v4u *)(qrow + 16 * c);
  }
  const float scale2 = 1.4426950408889634f / sqrtf((float)HD);
  // this wave's coordinate tiles: NDT * kg .. + NDT - 1
  f32x16 o[NDT];
#pragma unroll
  for (int x = 0; x < NDT; ++x)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[x][r] = 0.f;
  float m = -INFINITY, l = 0.f;

  // K of a step, then, half a step later, V of the same step.  A wave's scalar work stands between the barrier and
  // its products, so there is little of it: page ids come out of a register of 64, addresses by one multiplication.
  const uint32_t page_bytes = (uint32_t)Hkv * PPG * HD * 2;
  const size_t head_off = (size_t)kvh * PPG * HD * 2;
  const char *kA = (const char *)a.k_prefix + head_off, *vA = (const char *)a.v_prefix + head_off;
  const char *kB = (const char *)a.k_suffix + head_off, *vB = (const char *)a.v_suffix + head_off;
  int ids = pages.ids(0), ids_next = pages.ids(64);
  uint64_t off;
  auto issue_k = [&](int pi, int slot) __attribute__((always_inline)) {          // a step is a page
    if ((pi & 63) == 0 && pi > 0) {
      ids = ids_next;
      ids_next = pages.ids(pi + 64);
    }
    off = (uint64_t)(uint32_t)__builtin_amdgcn_readlane(ids, pi & 63) * page_bytes;
    const __amdgpu_buffer_rsrc_t kr = page_range((const bf16_t *)((pi < pages.nPA ? kA : kB) + off), pi < pages.n, HD);
#pragma unroll
    for (int c = 0; c < TL::CPT; ++c) load_piece(kr, k_lds + slot * TL::K_ELEMS + wave * 512, c);
  };
  auto issue_v = [&](int pi, int slot) __attribute__((always_inline)) {
    const __amdgpu_buffer_rsrc_t vr = page_range((const bf16_t *)((pi < pages.nPA ? vA : vB) + off), pi < pages.n, HD);
#pragma unroll
    for (int c = 0; c < TL::CPT; ++c) load_piece(vr, v_lds + slot * TL::V_ELEMS + wave * 512, c);
  };
#pragma unroll
  for (int st = 0; st < SP::SLOTS; ++st) {
    issue_k(st, st);
    issue_v(st, st);
  }

  auto wave_of = [&](int i) __attribute__((always_inline)) { return i * SP::HEADS + hw; };   // of this head, block i
  v4u *my_probs = probs + wave * 128 + lane;
  // this wave's probabilities and their sums to LDS
  auto leave_probs = [&](const f32x16 &p, float rs) __attribute__((always_inline)) {
    v4u pb[2];
    pack_probs(p, pb);
    my_probs[0] = pb[0];
    my_probs[64] = pb[1];
    sums[wave * 64 + lane] = rs + other_half(rs);
  };
  v4u kf[NF], vf[KS][NDT][2], pb[KS][2];
  float rs[KS];
  auto read_k = [&](int slot) __attribute__((always_inline)) {
    const bf16_t *kblk = k_lds + slot * TL::K_ELEMS + (kg * NF * 64 + lane) * 8;
#pragma unroll
    for (int c = 0; c < NF; ++c) kf[c] = *(const v4u *)(kblk + c * 512);
  };
  auto read_v = [&](int slot) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < KS; ++i) {
      const bf16_t *vblk = v_lds + slot * TL::V_ELEMS + (i * NF * 64 + lane) * 8;
#pragma unroll
      for (int x = 0; x < NDT; ++x)
#pragma unroll
        for (int sl = 0; sl < 2; ++sl) vf[i][x][sl] = *(const v4u *)(vblk + ((NDT * kg + x) * 2 + sl) * 512);
    }
  };
  auto read_probs = [&](int i) __attribute__((always_inline)) {
    rs[i] = sums[wave_of(i) * 64 + lane];
    pb[i][0] = probs[wave_of(i) * 128 + lane];
    pb[i][1] = probs[wave_of(i) * 128 + 64 + lane];
  };
  auto add_block = [&](int i) __attribute__((always_inline)) {
    l += rs[i];
#pragma unroll
    for (int x = 0; x < NDT; ++x)
#pragma unroll
      for (int sl = 0; sl < 2; ++sl) o[x] = mfma32p(vf[i][x][sl], pb[i][sl], o[x]);
  };
  // the loads issued after those that a barrier waits for: 2 SLOTS - 2 half steps
  constexpr int kAhead = (2 * SP::SLOTS - 2) * SP::LPH;
  const int n_steps = pages.n;
  // steps whose keys all exist and lie before every row, in the prefix
  const int n_plain = min(pages.nA, pos_start + 1) / (32 * KS);
  wait_barrier_p<kAhead + SP::LPH>();           // K of step 0
  read_k(0);
  int slot = 0;
  for (int st = 0; st < n_steps; ++st) {
    // V of this step is there; its K is in registers, the last step's probabilities are no longer read
    wait_barrier_p<kAhead, true>();
    issue_k(st + SP::SLOTS, slot);
    read_v(slot);
    __builtin_amdgcn_sched_barrier(0);
    const bool plain = st < n_plain;
    int abs0 = 0, nv = 32;
    bool live = active;                         // uniform; else all masked
    if (!plain) {
      nv = pages.block(st, kg, abs0);
      live = active && nv > 0 && abs0 <= my_last;
    }
    f32x16 s;
    int found = 0;
    if (live) {
#pragma unroll
      for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
      for (int c = 0; c < NF; ++c) s = mfma32p(kf[c], qf[c], s);
      if (!plain) mask_scores(s, nv, abs0, pos_start, my_pos, h);
    }
    if (st == 0) {
      // the first reference is block 0's maximum, as any block finds it that comes first
      if (kg == 0 && live) refs[wave * 64 + lane] = moved_reference(s, scale2, m);
      wait_barrier_p<63, true>();
      m = refs[wave_of(0) * 64 + lane];
    }
    if (live) {
      f32x16 p;
      const float sum = block_probs(s, scale2, m, p);
      found = leaves_range(sum) ? 2 : 1;
      leave_probs(p, sum);
    }
    if (lane == 0) state[wave] = found;
    // K of the next step is there, and the heads' probabilities; V of this one is in registers
    wait_barrier_p<kAhead, true>();
    const int states = state[lane & 7];
#pragma unroll
    for (int i = 0; i < KS; ++i) read_probs(i);
    slot = slot == SP::SLOTS - 1 ? 0 : slot + 1;
    read_k(slot);
    __builtin_amdgcn_sched_barrier(0);
    issue_v(st + SP::SLOTS, slot >= 1 ? slot - 1 : SP::SLOTS - 1);
    const unsigned int lives = (unsigned int)__ballot(states != 0);     // bit w: wave w's block
    if (!__any(states == 2)) {
      if (plain) {
        if (active)
#pragma unroll
          for (int i = 0; i < KS; ++i) add_block(i);
      } else {
#pragma unroll
        for (int i = 0; i < KS; ++i)
          if ((lives >> wave_of(i)) & 1) add_block(i);
      }
    } else {
      // block by block, the whole workgroup together
#pragma unroll
      for (int i = 0; i < KS; ++i) {
        if (kg == i && live) {
          f32x16 p;
          float sum = block_probs(s, scale2, m, p);
          const bool move = leaves_range(sum);
          if (move) {
            const float m_new = moved_reference(s, scale2, m);
            refs[wave * 64 + lane] = m_new;
            sum = block_probs(s, scale2, usable_reference(m_new), p);
          }
          leave_probs(p, sum);
          if (lane == 0) moved[wave] = move;
        }
        wait_barrier_p<63, true>();
        if ((lives >> wave_of(i)) & 1) {
          if (__builtin_amdgcn_readfirstlane(moved[wave_of(i)])) {
            const float m_new = refs[wave_of(i) * 64 + lane], corr = rescale_factor(m, m_new);
            l *= corr;
            m = m_new;
#pragma unroll
            for (int x = 0; x < NDT; ++x)
#pragma unroll
              for (int r = 0; r < 16; ++r) o[x][r] *= corr;
          }
          read_probs(i);
          add_block(i);
        }
      }
    }
  }
  wait_barrier_p<0>();                          // no load into LDS outlives the loop

  if (active && col_valid) {
    const float inv = 1.0f / l;
#pragma unroll
    for (int x = 0; x < NDT; ++x) store_tile<HD>(a, row_start + col, head, NDT * kg + x, h, o[x], inv);
  }
}

// The same with the work of 32 columns split by kind, for few workgroups: a workgroup has two heads, and a step is four
// blocks of 32 keys.  Four waves score, each one block for both heads, and leave probabilities and sums in LDS; beside them
// four waves add the step before, each 32 coordinates for both heads (head_dim 64: of one head).  A scoring and an adding
// wave share a SIMD, so value products run under exponentials, and there is one barrier per step.  A block's keys are read by one wave
// only, and so is a tile of its values, so both go from memory to registers and LDS holds the probabilities alone.  References
// move as in the kernel above: all four blocks are scored against the one that stood when the step began, and where
// a sum leaves the range the scoring waves do the step again block by block while the adding waves wait.  So the bits are the same, too.
// Bound by a scoring wave's chain, 2300 cycles per step at head_dim 128 (8B heads, 300 rows after 4096 keys, by the cycle counter): eight
// loads to ask for 400 (32 KB of keys and 32 of values per step at 64 bytes per cycle: 1024 in all), products and exponentials of the
// first head 700 to 950, exponentials of the second 700 (a wave alone on the vector unit issues an instruction every 6 to
// 12 cycles), barrier and flags 300.  Two scoring waves per SIMD, the next step's products under this one's exponentials, keys
// by LDS, and loads spread among the exponentials were measured and are no faster.
// us, one wave kind doing all four blocks' work in turn (two barriers, keys and values by LDS) -> this: 8B heads, 300 rows after 256 /
// 1024 / 4096 keys 13.5 -> 12.1 / 21.7 -> 19.0 / 52.6 -> 45.4, heads of 64 after 1024 / 4096 17.6 -> 13.0 / 44.0 -> 30.5.
template <int HD> struct PPair {
  static constexpr int NF = HD / 16, KB = 4, HEADS = 2;         // blocks per step, heads per workgroup
  static constexpr int ADD_HEADS = HD == 128 ? 2 : 1;           // heads per adding wave
  // probabilities of eight (block, head) pairs, twice; their sums, twice; references; flags
  static constexpr int PROBS = 0, SUMS = 2 * 8 * 2048, REFS = SUMS + 2 * 8 * 256, FLAGS = REFS + 8 * 256, LDS_BYTES = FLAGS + 128;
};

template <int HD>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, HD == 64 ? 4 : 2)))
void prefill_attention_pair_kernel(PrefillAttnArgs a, int n_main) {
  if ((int)blockIdx.x >= n_main) return zero_uncovered_rows(a, (int)blockIdx.x - n_main, a.n_q_heads * HD);
  using SP = PPair<HD>;
  constexpr int NF = SP::NF, KB = SP::KB, NH = SP::HEADS;
  extern __shared__ __attribute__((aligned(16))) unsigned char plds_raw[];
  v4u *probs = (v4u *)(plds_raw + SP::PROBS);                   // [2][8][2][64]
  float *sums = (float *)(plds_raw + SP::SUMS), *refs = (float *)(plds_raw + SP::REFS);   // [2][8][64], [8][64]
  int *state = (int *)(plds_raw + SP::FLAGS), *moved = state + 16;   // [2][8]: 0 no visible key, 1 scored, 2 out of range; [8]
  const int tid = threadIdx.x, lane = tid & 63, col = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), kg = wave & 3;
  const int Hq = a.n_q_heads, Hkv = a.n_kv_heads, G = Hq / Hkv, HG = (G + NH - 1) / NH;

  int id = blockIdx.x;
  const int kvh = id % Hkv; id /= Hkv;
  const int hg = id % HG; id /= HG;
  // Several sequences: second halves of the items last.  Items of up to 32 rows have none, and workgroups that end at once in turn with others
  // leave the dispatcher half of the units (32 sequences of 20 rows after 3000 keys, 8 / 8 heads of 128: 52 -> 29 us).  One sequence, whose
  // items are full: in turn (1000 rows of the 8B heads after 256 keys 30, 34 apart).
  const bool apart = a.page_table != nullptr;
  const int half = apart ? id >= a.n_items : id & 1;
  const int4 item = a.items[apart ? id - (half ? a.n_items : 0) : id >> 1];
  const int row_start = item.x + 32 * half, pos_start = item.z + 32 * half, my_rows = min(32, item.y - 32 * half);
  if (my_rows <= 0) return;                     // the whole workgroup: the item has no second half
  const bool both = NH * hg + 1 < G;            // the second head exists
  const int head0 = kvh * G + NH * hg;
  const bool col_valid = col < my_rows;
  const int my_pos = pos_start + (col_valid ? col : 0), my_last = pos_start + my_rows - 1;
  const PPages pages(a, item.w, my_last);
  const float scale2 = 1.4426950408889634f / sqrtf((float)HD);
  const uint32_t page_bytes = (uint32_t)Hkv * PPG * HD * 2;
  const size_t head_off = (size_t)kvh * PPG * HD * 2;
  int ids = pages.ids(0), ids_next = pages.ids(64);
  const int n_steps = (pages.n + 1) / 2;
  // steps whose keys all exist and lie before every row, in the prefix
  const int n_plain = min(pages.nA, pos_start + 1) / (32 * KB);

  if (wave < 4) {
    // ---- scores: block kg of every step, for both heads
    v4u qf[NH][NF], kf[2][NF];
#pragma unroll
    for (int x = 0; x < NH; ++x) {
      const bf16_t *qrow = (const bf16_t *)a.q + ((size_t)(row_start + (col_valid ? col : 0)) * Hq + head0 + (both ? x : 0)) * HD + 8 * h;
#pragma unroll
      for (int c = 0; c < NF; ++c) qf[x][c] = *(const v4u *)(qrow + 16 * c);
    }
    const char *kA = (const char *)a.k_prefix + head_off + (kg & 1) * NF * 1024 + lane * 16;
    const char *kB = (const char *)a.k_suffix + head_off + (kg & 1) * NF * 1024 + lane * 16;
    auto load_k = [&](int step, v4u (&f)[NF]) __attribute__((always_inline)) {
      const int p0 = 2 * step, pi = p0 + (kg >> 1);
      if ((p0 & 63) == 0 && p0 > 0) {
        ids = ids_next;
        ids_next = pages.ids(p0 + 64);
      }
      // a page past the end: the first one again, never used
      const uint64_t off = (uint64_t)(uint32_t)(pi < pages.n ? __builtin_amdgcn_readlane(ids, pi & 63) : 0) * page_bytes;
      const char *k = (pi < pages.nPA || pi >= pages.n ? kA : kB) + off;
#pragma unroll
      for (int c = 0; c < NF; ++c) f[c] = *(const v4u *)(k + c * 1024);
    };
    load_k(0, kf[0]);
    float m[NH] = {-INFINITY, -INFINITY};
    auto leave_probs = [&](int buf, int x, const f32x16 &p, float rs) __attribute__((always_inline)) {
      v4u pb[2];
      pack_probs(p, pb);
      v4u *mine = probs + (buf * 8 + kg * NH + x) * 128 + lane;
      mine[0] = pb[0];
      mine[64] = pb[1];
      sums[(buf * 8 + kg * NH + x) * 64 + lane] = rs + other_half(rs);
    };
    auto score = [&](const v4u (&f)[NF], int x, f32x16 &s) __attribute__((always_inline)) {
#pragma unroll
      for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
      for (int c = 0; c < NF; ++c) s = mfma32p(f[c], qf[x][c], s);
    };
    auto step = [&](int st, auto parity) __attribute__((always_inline)) {
      constexpr int U = decltype(parity)::value;
      const bool plain = st < n_plain;
      f32x16 s[NH];
      int found[NH] = {0, 0};
      load_k(st + 1, kf[U ^ 1]);
      __builtin_amdgcn_sched_barrier(0);
      if (plain && both && st > 0) {
        score(kf[U], 0, s[0]);
        __builtin_amdgcn_sched_barrier(0);
        score(kf[U], 1, s[1]);
        float sum[NH];
        f32x16 p;
        sum[0] = block_probs(s[0], scale2, m[0], p);
        leave_probs(U, 0, p, sum[0]);
        __builtin_amdgcn_sched_barrier(0);
        sum[1] = block_probs(s[1], scale2, m[1], p);
        leave_probs(U, 1, p, sum[1]);
#pragma unroll
        for (int x = 0; x < NH; ++x) found[x] = leaves_range(sum[x]) ? 2 : 1;
      } else {
        int abs0 = 0, nv = 32;
        bool live = true;
        if (!plain) {
          const int pi = 2 * st + (kg >> 1);
          nv = pages.block(pi, kg & 1, abs0);
          live = pi < pages.n && nv > 0 && abs0 <= my_last;
        }
        if (live) {
#pragma unroll
          for (int x = 0; x < NH; ++x) {
            score(kf[U], x, s[x]);
            if (!plain) mask_scores(s[x], nv, abs0, pos_start, my_pos, h);
          }
        }
        if (st == 0) {
          // the first reference is block 0's maximum, as any block finds it that comes first
          if (kg == 0)
#pragma unroll
            for (int x = 0; x < NH; ++x) refs[x * 64 + lane] = moved_reference(s[x], scale2, m[x]);
          wait_barrier_p<63, true>();
#pragma unroll
          for (int x = 0; x < NH; ++x) m[x] = refs[x * 64 + lane];
        }
        if (live) {
#pragma unroll
          for (int x = 0; x < NH; ++x) {
            if (x == 1 && !both) break;
            f32x16 p;
            const float sum = block_probs(s[x], scale2, m[x], p);
            found[x] = leaves_range(sum) ? 2 : 1;
            leave_probs(U, x, p, sum);
          }
        }
      }
      if (lane < NH) state[U * 8 + kg * NH + lane] = lane ? found[1] : found[0];
      wait_barrier_p<63, true>();
      if (__any(state[U * 8 + (lane & 7)] == 2)) {
        // block by block, the whole workgroup together
#pragma unroll 1
        for (int i = 0; i < KB; ++i) {
          if (kg == i) {
#pragma unroll
            for (int x = 0; x < NH; ++x) {
              if (!found[x]) continue;
              f32x16 p;
              float sum = block_probs(s[x], scale2, m[x], p);
              const bool move = leaves_range(sum);
              if (move) {
                const float m_new = moved_reference(s[x], scale2, m[x]);
                refs[(i * NH + x) * 64 + lane] = m_new;
                sum = block_probs(s[x], scale2, usable_reference(m_new), p);
              }
              leave_probs(U, x, p, sum);
              if (lane == 0) moved[i * NH + x] = move;
            }
          }
          wait_barrier_p<63, true>();
#pragma unroll
          for (int x = 0; x < NH; ++x)
            if (__builtin_amdgcn_readfirstlane(state[U * 8 + i * NH + x]) && __builtin_amdgcn_readfirstlane(moved[i * NH + x]))
              m[x] = refs[(i * NH + x) * 64 + lane];
        }
      }
    };
    for (int st = 0; st < n_steps; st += 2) {
      step(st, std::integral_constant<int, 0>{});
      if (st + 1 < n_steps) step(st + 1, std::integral_constant<int, 1>{});
    }
    return;
  }

  // ---- sums: 32 coordinates of both heads (head_dim 64: of one head)
  constexpr int AH = SP::ADD_HEADS;
  const int dt = AH == 2 ? kg : kg & 1, x0 = AH == 2 ? 0 : kg >> 1;
  const char *vA = (const char *)a.v_prefix + head_off + dt * 2048 + lane * 16;
  const char *vB = (const char *)a.v_suffix + head_off + dt * 2048 + lane * 16;
  v4u vf[2][KB][2];
  auto load_v = [&](int step, v4u (&f)[KB][2]) __attribute__((always_inline)) {
    const int p0 = 2 * step;
    if ((p0 & 63) == 0 && p0 > 0) {
      ids = ids_next;
      ids_next = pages.ids(p0 + 64);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int pi = p0 + i;
      const uint64_t off = (uint64_t)(uint32_t)(pi < pages.n ? __builtin_amdgcn_readlane(ids, pi & 63) : 0) * page_bytes;
      const char *v = (pi < pages.nPA || pi >= pages.n ? vA : vB) + off;
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int sl = 0; sl < 2; ++sl) f[2 * i + b][sl] = *(const v4u *)(v + (b * NF + sl) * 1024);
    }
  };
  load_v(0, vf[0]);
  load_v(1, vf[1]);
  f32x16 o[AH];
  float m[AH], l[AH];
#pragma unroll
  for (int x = 0; x < AH; ++x) {
    l[x] = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) o[x][r] = 0.f;
  }
  auto add_block = [&](int buf, int i, int x, const v4u (&f)[2]) __attribute__((always_inline)) {
    const int at = buf * 8 + i * NH + x0 + x;
    const v4u p0 = probs[at * 128 + lane], p1 = probs[at * 128 + 64 + lane];
    l[x] += sums[at * 64 + lane];
    o[x] = mfma32p(f[0], p0, o[x]);
    o[x] = mfma32p(f[1], p1, o[x]);
  };
  unsigned int lives = 0;                       // of the step to be added; 0: nothing is left of it
  auto add_step = [&](auto parity) __attribute__((always_inline)) {
    constexpr int U = decltype(parity)::value;
    v4u pb[KB][AH][2];
    float rs[KB][AH];
#pragma unroll
    for (int i = 0; i < KB; ++i)
#pragma unroll
      for (int x = 0; x < AH; ++x) {
        const int at = U * 8 + i * NH + x0 + x;
        pb[i][x][0] = probs[at * 128 + lane];
        pb[i][x][1] = probs[at * 128 + 64 + lane];
      }
#pragma unroll
    for (int i = 0; i < KB; ++i)
#pragma unroll
      for (int x = 0; x < AH; ++x) rs[i][x] = sums[(U * 8 + i * NH + x0 + x) * 64 + lane];
    __builtin_amdgcn_sched_barrier(0);
    if (lives == 0xFFu) {
#pragma unroll
      for (int i = 0; i < KB; ++i)
#pragma unroll
        for (int sl = 0; sl < 2; ++sl)
#pragma unroll
          for (int x = 0; x < AH; ++x) o[x] = mfma32p(vf[U][i][sl], pb[i][x][sl], o[x]);
#pragma unroll
      for (int i = 0; i < KB; ++i)
#pragma unroll
        for (int x = 0; x < AH; ++x) l[x] += rs[i][x];
    } else {
#pragma unroll
      for (int i = 0; i < KB; ++i)
#pragma unroll
        for (int x = 0; x < AH; ++x)
          if ((lives >> (i * NH + x0 + x)) & 1) {
            l[x] += rs[i][x];
#pragma unroll
            for (int sl = 0; sl < 2; ++sl) o[x] = mfma32p(vf[U][i][sl], pb[i][x][sl], o[x]);
          }
    }
  };
  auto step = [&](int st, auto parity) __attribute__((always_inline)) {
    constexpr int U = decltype(parity)::value;
    if (st > 0) {
      add_step(std::integral_constant<int, U ^ 1>{});
      load_v(st + 1, vf[U ^ 1]);
    } else {
      wait_barrier_p<63, true>();
#pragma unroll
      for (int x = 0; x < AH; ++x) m[x] = refs[(x0 + x) * 64 + lane];
    }
    wait_barrier_p<63, true>();
    const int states = state[U * 8 + (lane & 7)];
    lives = (unsigned int)__ballot(states != 0) & 0xFFu;
    if (__any(states == 2)) {
#pragma unroll
      for (int i = 0; i < KB; ++i) {
        wait_barrier_p<63, true>();
#pragma unroll
        for (int x = 0; x < AH; ++x) {
          const int e = i * NH + x0 + x;
          if (!((lives >> e) & 1)) continue;
          if (__builtin_amdgcn_readfirstlane(moved[e])) {
            const float m_new = refs[e * 64 + lane], corr = rescale_factor(m[x], m_new);
            l[x] *= corr;
            m[x] = m_new;
#pragma unroll
            for (int r = 0; r < 16; ++r) o[x][r] *= corr;
          }
          add_block(U, i, x, vf[U][i]);
        }
      }
      lives = 0;
    }
  };
  for (int st = 0; st < n_steps; st += 2) {
    step(st, std::integral_constant<int, 0>{});
    if (st + 1 < n_steps) step(st + 1, std::integral_constant<int, 1>{});
  }
  if (n_steps & 1) add_step(std::integral_constant<int, 0>{});
  else add_step(std::integral_constant<int, 1>{});
  if (col_valid) {
#pragma unroll
    for (int x = 0; x < AH; ++x) {
      if (x0 + x == 1 && !both) break;
      store_tile<HD>(a, row_start + col, head0 + x0 + x, dt, h, o[x], 1.0f / l[x]);
    }
  }
}

bool prefill_attention_mfma_supported(int page_tokens, int head_dim, int Hq, int Hkv) {
  return page_tokens == PPG && (head_dim == 64 || head_dim == 128) && Hq % Hkv == 0;
}

enum { PREFILL_WHOLE, PREFILL_SPLIT, PREFILL_PAIR };

// Whole items: do the heads past a multiple of four go by several items to a workgroup?  Measured at 257 to 3200 workgroups of whole items, sequences of
// 20 to 300 rows after 64 to 8192 keys, 1, 2, 5 and 6 heads per KV head; the time with a workgroup per item / this one's:
// sequences of several items 1.1 to 2.1 (40 / 8 heads of 128, 8 x 1024 rows after 4096 keys 978 / 771 us, 5 x 200 after 1000 68 / 40; 8 / 8 heads, 8 x 1024 after 4096
// 482 / 163), but not in one round of workgroups, where nothing is won (160 workgroups, 5 x 200 rows after 1000 keys 34 / 37 us), nor where even the
// neighbours all found leave as many rounds (40 / 8 heads, 8 x 256: 320 of 512, 0.94 to 1.00).
// Sequences of one item: five and six heads 1.0 to 1.5, as the full workgroups go first; one and two heads, whose waves spread over more SIMDs, 1.1 to 1.4
// from 1000 keys on, but 0.83 to 1.1 up to 300, and items of up to 32 rows 0.88 to 1.0.
// One head of 64, whose workgroups go two to a unit: 0.89 to 1.00 up to 512 workgroups, 1.1 to 1.7 above.
constexpr long kComputeUnits = 256;
constexpr int kRestShortKeys = 1000;
static bool rest_heads(const PrefillAttnArgs &a) {
  const int G = a.n_q_heads / a.n_kv_heads;
  if (G % 4 != 1 && G % 4 != 2) return false;
  const int near = 4 / (G % 4), stride = a.page_table ? a.table_stride : near;         // a sequence's pages: its items at most
  const long whole = (long)a.n_kv_heads * a.n_items * ((G + 3) / 4), least = (long)a.n_kv_heads * ((long)a.n_items * (G / 4) + (a.n_items + near - 1) / near);
  auto rounds = [](long groups) { return (groups + kComputeUnits - 1) / kComputeUnits; };
  if (whole <= (a.head_dim == 64 && G == 1 ? 2 : 1) * kComputeUnits) return false;
  if (G < 4 && stride == 1) return a.prefix_len >= kRestShortKeys;
  return stride < near || rounds(least) < rounds(whole);
}

// workgroups of a form
template <int HD>
static long prefill_grid(const PrefillAttnArgs &a, int form) {
  const int heads = form == PREFILL_PAIR ? PPair<HD>::HEADS : 4, G = a.n_q_heads / a.n_kv_heads;
  if (form == PREFILL_WHOLE && rest_heads(a)) {
    const int near = 4 / (G % 4);
    return (long)a.n_kv_heads * (a.n_items * (G / 4) + (a.n_items + near - 1) / near * near);
  }
  return (long)a.n_items * (form == PREFILL_WHOLE ? 1 : 2) * a.n_kv_heads * ((G + heads - 1) / heads);
}

// A workgroup is a chain over all keys of its rows, so as long as one round of workgroups (a compute
// unit holds one) leaves units idle, more of them with shorter steps are faster.  All forms give the same bits.  A second round
// of the pair form, whose step is the shortest for its work, gains against whole items at any length for one sequence, which all its workgroups walk
// together, and behind a long prefix for several; against two waves per head, which have half of its workgroups, behind a longer one, as its workgroups' fixed
// part counts twice.  Measured at 257 to 512 workgroups of it, one sequence of 300 to 1500 rows after 64 to 8192 keys, 2 to 100 sequences of 20 to 320
// rows after 64 to 8192, 1 to 8 heads per KV head; the other form's time / this one's:
// one sequence: whole items 1.3 to 1.6; two waves per head, head_dim 64, 0.97 (400 rows after 64 keys), 1.03 from 500 after 64 on, 1.2 after 8192; 128, up to four
// heads 0.98 (600 after 64), 1.02 to 1.08 from 800 after 64 on, five to eight heads 0.90 to 1.02 up to 1024 keys, 1.00 to 1.07 after 2048;
// several: whole items 0.7 to 0.9 up to 300 keys, 1.0 to 1.2 at 1000, 1.13 to 1.7 at 2047; two waves per head, head_dim 64, 0.8 to 0.9 up to 300 keys, 1.01 to 1.07 at
// 2047, 1.1 at 3000; 128 0.7 to 0.9 up to 1000, 0.91 to 0.97 at 2047, 0.96 to 1.04 at 3000 (items of up to 32 rows, half of whose workgroups end at once, 1.8).
template <int HD>
static int prefill_form(const PrefillAttnArgs &a) {
  const long pairs = prefill_grid<HD>(a, PREFILL_PAIR);
  const bool split = prefill_grid<HD>(a, PREFILL_SPLIT) <= kComputeUnits;
  if (pairs <= kComputeUnits) return PREFILL_PAIR;
  if (pairs <= 2 * kComputeUnits) {
    int least;                                  // keys from which the second round is faster
    if (a.page_table) least = split && HD == 128 ? 3072 : 2048;
    else least = !split ? 0 : HD == 64 ? 512 : a.n_q_heads / a.n_kv_heads <= 4 ? 768 : 2048;
    if (a.prefix_len >= least) return PREFILL_PAIR;
  }
  return split ? PREFILL_SPLIT : PREFILL_WHOLE;
}

template <int HD>
static int launch_prefill_hd(hipStream_t st, const PrefillAttnArgs &a) {
  const int form = prefill_form<HD>(a);
  const unsigned n_main = (unsigned)prefill_grid<HD>(a, form), n_zero = a.out_tiled == TILED_ZERO ? (a.rows + 255) / 256 : 0;
  if (form == PREFILL_PAIR) {
    MC_TRY(raise_dynamic_lds_limit((const void *)prefill_attention_pair_kernel<HD>, PPair<HD>::LDS_BYTES));
    prefill_attention_pair_kernel<HD><<<n_main + n_zero, 512, PPair<HD>::LDS_BYTES, st>>>(a, (int)n_main);
  } else if (form == PREFILL_SPLIT) {
    MC_TRY(raise_dynamic_lds_limit((const void *)prefill_attention_split_kernel<HD>, PSplit<HD>::LDS_BYTES));
    prefill_attention_split_kernel<HD><<<n_main + n_zero, 512, PSplit<HD>::LDS_BYTES, st>>>(a, (int)n_main);
  } else {
    const int lds = PWhole<HD>::LDS_BYTES + kPrefillMaxPids * (int)sizeof(int);
    const auto kernel = rest_heads(a) ? prefill_attention_kernel<HD, true> : prefill_attention_kernel<HD, false>;
    MC_TRY(raise_dynamic_lds_limit((const void *)kernel, lds));
    const size_t pieces = (size_t)padded_rows(a.rows) * a.n_q_heads * HD / 8;
    if (n_zero && pieces * 16 <= kL2Bytes) zero_rows_kernel<<<(unsigned)((pieces + 255) / 256), 256, 0, st>>>((v4u *)a.out, pieces);
    else if (n_zero) zero_uncovered_rows_kernel<<<n_zero, 512, 0, st>>>(a);
    kernel<<<n_main, 512, lds, st>>>(a);
  }
  MC_HIP(hipGetLastError());
  return MC_OK;
}

int launch_attention_prefill_mfma(hipStream_t st, const PrefillAttnArgs &a) {
  if (a.n_items <= 0) return MC_OK;
  if (!prefill_attention_mfma_supported(a.page_tokens, a.head_dim, a.n_q_heads, a.n_kv_heads))
    MC_FAIL(MC_ERR_UNSUPPORTED, "prefill attention: shape not covered");
  return a.head_dim == 128 ? launch_prefill_hd<128>(st, a) : launch_prefill_hd<64>(st, a);
}

void prefill_attention_plan(const PrefillAttnArgs &a, int32_t out[2]) {
  const int form = a.head_dim == 128 ? prefill_form<128>(a) : prefill_form<64>(a);
  out[0] = form == PREFILL_WHOLE && rest_heads(a) ? 3 : form;
  out[1] = (int32_t)(a.head_dim == 128 ? prefill_grid<128>(a, form) : prefill_grid<64>(a, form));
}

}  // namespace mc
