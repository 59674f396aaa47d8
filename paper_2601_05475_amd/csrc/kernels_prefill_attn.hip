// Causal attention for many query rows (prefix prefill and candidate scoring), bf16, gfx950 MFMA.
//
// A work item is up to 64 consecutive positions of one sequence, one KV head and up to four of
// its query heads.  The workgroup has 8 waves: wave w owns head 4 * hg + w % 4 of the group and
// positions 32 (w / 4) .. + 31 of the item, which are its MFMA columns.  Two waves per SIMD let
// one wave's softmax run under the other's MFMAs, and the LDS only reaches its full read rate
// with eight waves per CU.
// Where that gives fewer workgroups than the chip has compute units, the waves split the keys as
// well: with 2 (4) key groups a workgroup has one half of the item's rows and 4 (2) heads, every
// group takes every second (fourth) 32-key block, and the groups' states of the same columns are
// merged in LDS at the end (300 positions after 4096 keys of the 8B shape: 106 -> 45 us).
// Keys are streamed page by page (64 keys) through LDS and shared by the waves: first the
// shared-prefix pages that are visible to the block, then (scoring) the sequence's own suffix
// pages.  Pages are stored in MFMA fragment order, so a page is copied to LDS as it is (by
// loads that write LDS directly, one or two steps ahead) and an operand is one
// conflict-free 16-byte read per lane.  Each item sees all keys of its rows, so
// it normalises and writes bf16 itself.  Operand mapping and the softmax scheme are those of
// the decode kernel (transposed scores, lazy base-2 reference maximum); the addition is the
// causal mask, applied only to blocks that reach past the first position of the item.
#include "kernels_mfma.h"

#include <algorithm>

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

// KS = key groups of a workgroup (see the head of the file): pages staged per step, steps held in
// LDS, query heads and 32-row halves of an item per workgroup.
template <int HD, int KS> struct PSplit {
  static constexpr int PP = KS == 4 ? 2 : 1;
  static constexpr int STEPS = KS == 4 && HD == 128 ? 2 : 3;
  static constexpr int HEADS = KS == 4 ? 2 : 4, HALVES = KS == 1 ? 2 : 1;
  static constexpr int LPS = 2 * PTile<HD>::CPT * PP;       // loads into LDS per wave and step
  static constexpr int LDS_BYTES = STEPS * PP * PTile<HD>::PAGE_ELEMS * 2;
  // the states that the key groups 1 .. KS - 1 hand over at the end use the page buffers
  static_assert((KS - 1) * (8 / KS) * 64 * (HD / 2 + 2) * 4 <= LDS_BYTES, "states fit the page buffers");
};

constexpr int kPrefillMaxPids = 1024;

// All but the newest N vector memory operations of this wave have landed, loads into LDS among them,
// then the workgroup's barrier.  (__syncthreads() would wait for every load in flight.)
template <int N>
__device__ inline void wait_barrier_p() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0F70);    // vmcnt <= N; the other counters free
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

template <int HD, int KS>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
void prefill_attention_kernel(PrefillAttnArgs a) {
  using TL = PTile<HD>;
  using SP = PSplit<HD, KS>;
  extern __shared__ __attribute__((aligned(16))) unsigned char plds_raw[];
  bf16_t *lds = (bf16_t *)plds_raw;
  typedef __attribute__((address_space(3))) int lds_int;
  lds_int *pids = (lds_int *)(plds_raw + SP::LDS_BYTES);
  const int tid = threadIdx.x, lane = tid & 63, col = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int Hq = a.n_q_heads, Hkv = a.n_kv_heads, G = Hq / Hkv, HG = (G + SP::HEADS - 1) / SP::HEADS;

  int id = blockIdx.x;
  // KV heads first: with eight of them an XCD (workgroups are dealt to the eight in turn) meets one
  // head's keys and values only
  const int kvh = id % Hkv; id /= Hkv;
  const int hg = id % HG; id /= HG;
  // head within the group, half of the item's rows, key group
  const int hw = wave % SP::HEADS, half = KS == 1 ? wave >> 2 : (id & 1), kg = KS == 1 ? 0 : wave / SP::HEADS;
  if (KS > 1) id >>= 1;
  const int4 item = a.items[id];               // row_start, n_rows (<= 64), pos_start, table row
  const int n_rows = item.y, tab = item.w;
  const int row_start = item.x + 32 * half;     // this wave's rows and their first position
  const int pos_start = item.z + 32 * half;
  const int my_rows = min(32, n_rows - 32 * half);
  if (KS > 1 && my_rows <= 0) return;           // the whole workgroup: the item has no second half
  const int g = SP::HEADS * hg + hw;
  const bool wave_active = g < G && my_rows > 0;   // uniform per wave
  const int head = kvh * G + (g < G ? g : 0);
  const bool col_valid = col < my_rows;
  const int my_pos = pos_start + (col_valid ? col : 0);
  const int my_last = pos_start + my_rows - 1;     // last position of this wave's rows

  // visible keys: prefix [0, nA), then own suffix [0, nB) at absolute positions prefix_len + j
  const int last_pos = KS == 1 ? item.z + n_rows - 1 : my_last;   // of the workgroup: pages every wave helps to stage
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
  // Pages go from global memory straight into LDS (lane i of a wave-wide 16-byte load lands at
  // the wave's base + 16 i: the page is copied as it is), SP::STEPS - 1 steps of SP::PP pages ahead
  // of the one in use.  The same number of loads is issued whether or not the page exists (a page past
  // the end has a range of no bytes: nothing is fetched), so the wait before the barrier can
  // count: all but the newest page's loads have landed.  They are buffer loads because the compiler
  // counts those; after a global (flat) load into LDS it waits for everything in flight before the
  // next use of any load.
  auto page_of = [&](int pi) __attribute__((always_inline)) -> int {
    if (pi >= n_pages) return 0;
    if (pi < nPA) return pi;
    if (pids_in_lds) return __builtin_amdgcn_readfirstlane(pids[pi - nPA]);
    return __builtin_amdgcn_readfirstlane(table[pi - nPA]);
  };
  auto issue = [&](int pi, int page, int buf) __attribute__((always_inline)) {
    const bool in_a = pi < nPA;
    const size_t at = (size_t)page * page_stride + head_off;
    const int bytes = pi < n_pages ? PPG * HD * (int)sizeof(bf16_t) : 0;
    const __amdgpu_buffer_rsrc_t kr = __builtin_amdgcn_make_buffer_rsrc((void *)((in_a ? kA : kB) + at), 0, bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t vr = __builtin_amdgcn_make_buffer_rsrc((void *)((in_a ? vA : vB) + at), 0, bytes, 0x00020000);
    bf16_t *kt = lds + buf * TL::PAGE_ELEMS + wave * 512, *vt = kt + TL::K_ELEMS;   // buf: of a page
#pragma unroll
    for (int i = 0; i < TL::CPT; ++i) {
      __builtin_amdgcn_raw_ptr_buffer_load_lds(kr, (__attribute__((address_space(3))) void *)(kt + 4096 * i), 16, tid * 16, 8192 * i, 0, 0);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(vr, (__attribute__((address_space(3))) void *)(vt + 4096 * i), 16, tid * 16, 8192 * i, 0, 0);
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
    // key of register r: 8 (r / 4) + 4 h + r % 4; it is masked if it does not exist or lies
    // after this lane's query position
    if (n_valid < 32 || abs0 + 31 > pos_start) {
      const int lim = min(n_valid, my_pos - abs0 + 1);      // keys [0, lim) are visible
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (8 * (r >> 2) + 4 * h + (r & 3) >= lim) s[r] = -INFINITY;
    }
    // Probabilities against the reference m as it stands (see the decode kernel: any reference
    // gives the same normalised result, it only has to keep the numbers in range).  Only if a
    // lane's sum leaves the range - a score far above the reference, or no reference yet (m =
    // -inf yields inf or NaN) - the block's maximum is taken, the reference moved and the
    // accumulators rescaled; the common case spends no instruction on maxima.
    f32x16 p;
    float rs = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      p[r] = __builtin_amdgcn_exp2f(fmaf(s[r], scale2, -m));
      rs += p[r];
    }
    if (__any(!(rs <= kSoftmaxSumLimit))) {
      float mx = max16f(s);
      mx = fmaxf(mx, other_half(mx));
      const float m_new = fmaxf(m, mx * scale2);    // stays -inf for a column that has seen no key
      const float corr = (m_new == -INFINITY) ? 1.0f : __builtin_amdgcn_exp2f(m - m_new);
      l *= corr;
      m = m_new;
#pragma unroll
      for (int dt = 0; dt < HD / 32; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[dt][r] *= corr;
      // a column with no visible key so far: 0 as reference, all its p are 0
      const float mref = (m == -INFINITY) ? 0.f : m;
      rs = 0.f;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        p[r] = __builtin_amdgcn_exp2f(fmaf(s[r], scale2, -mref));
        rs += p[r];
      }
    }
    rs += other_half(rs);
    l += rs;
    v4u pb[2];
    pb[0] = v4u{pack2p_bf16(p[0], p[1]), pack2p_bf16(p[2], p[3]), pack2p_bf16(p[4], p[5]), pack2p_bf16(p[6], p[7])};
    pb[1] = v4u{pack2p_bf16(p[8], p[9]), pack2p_bf16(p[10], p[11]), pack2p_bf16(p[12], p[13]), pack2p_bf16(p[14], p[15])};
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

  int next_page[SP::PP];
  auto issue_step = [&](int step, int slot) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < SP::PP; ++i) {
      issue(step * SP::PP + i, next_page[i], slot * SP::PP + i);
      next_page[i] = page_of((step + 1) * SP::PP + i);
    }
  };
#pragma unroll
  for (int i = 0; i < SP::PP; ++i) next_page[i] = page_of(i);
#pragma unroll
  for (int st = 0; st + 1 < SP::STEPS; ++st) issue_step(st, st);
  const int n_steps = (n_pages + SP::PP - 1) / SP::PP;
  int slot = 0;
  for (int st = 0; st < n_steps; ++st) {
    // the pages of this step have landed once at most the loads of the later ones that were issued
    // are outstanding; past the barrier that holds for every wave, and the last step's pages are no
    // longer read
    wait_barrier_p<(SP::STEPS - 2) * SP::LPS>();
    issue_step(st + SP::STEPS - 1, slot >= 1 ? slot - 1 : SP::STEPS - 1);
    if (wave_active) {
      if (KS == 1) {
        consume(st, slot, 0);
        consume(st, slot, 1);
      } else {
        const int pi = st * SP::PP + (kg >> 1) % SP::PP;
        if (pi < n_pages) consume(pi, slot * SP::PP + (kg >> 1) % SP::PP, kg & 1);
      }
    }
    slot = slot == SP::STEPS - 1 ? 0 : slot + 1;
  }
  wait_barrier_p<0>();                         // no load into LDS outlives the loop

  if (KS > 1) {
    // the key groups' states of the same columns meet in LDS: group 0 merges the others' into its own
    constexpr int WPG = 8 / KS, REGS = HD / 2;  // waves per key group; accumulator registers of a lane
    float *so = (float *)plds_raw;              // [KS - 1][WPG][REGS + 2][64]
    if (kg > 0) {
      float *dst = so + ((kg - 1) * WPG + hw) * (REGS + 2) * 64 + lane;
#pragma unroll
      for (int dt = 0; dt < HD / 32; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) dst[(dt * 16 + r) * 64] = o[dt][r];
      dst[REGS * 64] = m;
      dst[(REGS + 1) * 64] = l;
    }
    __syncthreads();
    if (kg > 0) return;
    const float *src = so + hw * (REGS + 2) * 64 + lane;
    float M = m;
#pragma unroll
    for (int k = 0; k < KS - 1; ++k) M = fmaxf(M, src[(k * WPG * (REGS + 2) + REGS) * 64]);
    // a group that saw no key of the column has m = -inf and no weight
    const float f0 = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - M);
    l *= f0;
#pragma unroll
    for (int dt = 0; dt < HD / 32; ++dt)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[dt][r] *= f0;
#pragma unroll 1
    for (int k = 0; k < KS - 1; ++k) {
      const float *ks = src + k * WPG * (REGS + 2) * 64;
      const float mk = ks[REGS * 64], fk = mk == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mk - M);
      l += fk * ks[(REGS + 1) * 64];
#pragma unroll
      for (int dt = 0; dt < HD / 32; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[dt][r] += fk * ks[(dt * 16 + r) * 64];
    }
  }
  if (wave_active && col_valid) {
    const float inv = 1.0f / l;                  // l > 0: every row sees at least its own key
    bf16_t *out = (bf16_t *)a.out;
    const int row = row_start + col;
#pragma unroll
    for (int dt = 0; dt < HD / 32; ++dt)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        const int d = dt * 32 + 8 * r4 + 4 * h;
        const size_t at = a.out_tiled ? tiled_offset(row, head * HD + d, Hq * HD)
                                      : ((size_t)row * Hq + head) * HD + d;
        v2u pk = {pack2p_bf16(o[dt][4 * r4] * inv, o[dt][4 * r4 + 1] * inv),
                  pack2p_bf16(o[dt][4 * r4 + 2] * inv, o[dt][4 * r4 + 3] * inv)};
        *(v2u *)(out + at) = pk;
      }
  }
}

bool prefill_attention_mfma_supported(int page_tokens, int head_dim, int Hq, int Hkv) {
  return page_tokens == PPG && (head_dim == 64 || head_dim == 128) && Hq % Hkv == 0;
}

template <int HD, int KS>
static long prefill_grid(const PrefillAttnArgs &a) {
  using SP = PSplit<HD, KS>;
  const int G = a.n_q_heads / a.n_kv_heads;
  return (long)a.n_items * (2 / SP::HALVES) * a.n_kv_heads * ((G + SP::HEADS - 1) / SP::HEADS);
}

template <int HD, int KS>
static int launch_prefill_t(hipStream_t st, const PrefillAttnArgs &a) {
  using SP = PSplit<HD, KS>;
  const int lds = SP::LDS_BYTES + kPrefillMaxPids * (int)sizeof(int);
  MC_TRY(raise_dynamic_lds_limit((const void *)prefill_attention_kernel<HD, KS>, lds));
  prefill_attention_kernel<HD, KS><<<(unsigned)prefill_grid<HD, KS>(a), 512, lds, st>>>(a);
  MC_HIP(hipGetLastError());
  return MC_OK;
}

template <int HD>
static int launch_prefill_hd(hipStream_t st, const PrefillAttnArgs &a) {
  // A workgroup is a chain over all keys of its rows, so as long as one round of workgroups (a
  // compute unit holds one) leaves units idle, more of them with fewer columns each are faster; a
  // second round costs what the split gains.  8B heads, one sequence after 4096 keys, us with 1 / 2 /
  // 4 key groups: 65 rows 100 / 60 / 43, 300 rows 106 / 64 / 45, 512 rows (256 workgroups with four
  // groups) 112 / 68 / 53, 800 rows 119 / 76 / 92, 1024 rows (256 with two) 125 / 86 / 100; four
  // sequences of 400 rows 123 / 133 / 171.
  // Up to 2560 shared keys the split saves 10 - 30 us a layer, and there the order of additions of one
  // group is kept: the ids that a session samples and the ranks that it gives follow the last bits of
  // its prefill.
  constexpr long kComputeUnits = 256;
  constexpr int kShortChain = 2560;
  if (a.prefix_len <= kShortChain) return launch_prefill_t<HD, 1>(st, a);
  if (prefill_grid<HD, 4>(a) <= kComputeUnits) return launch_prefill_t<HD, 4>(st, a);
  if (prefill_grid<HD, 2>(a) <= kComputeUnits) return launch_prefill_t<HD, 2>(st, a);
  return launch_prefill_t<HD, 1>(st, a);
}

int launch_attention_prefill_mfma(hipStream_t st, const PrefillAttnArgs &a) {
  if (a.n_items <= 0) return MC_OK;
  if (!prefill_attention_mfma_supported(a.page_tokens, a.head_dim, a.n_q_heads, a.n_kv_heads))
    MC_FAIL(MC_ERR_UNSUPPORTED, "prefill attention: shape not covered");
  return a.head_dim == 128 ? launch_prefill_hd<128>(st, a) : launch_prefill_hd<64>(st, a);
}

}  // namespace mc
