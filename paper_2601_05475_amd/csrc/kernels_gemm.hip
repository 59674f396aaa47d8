// Many-row bf16 GEMM on tiled operands (gfx950, v_mfma_f32_32x32x16_bf16):
//   out[m][n] = sum_k a[m][k] w[n][k]                 (fp32, row-major), or
//   out_t[m][n] = silu(a . wg[n]) * (a . wu[n])        (bf16, tiled; the SwiGLU form).
//
// A workgroup of 4 waves owns 256 rows of a and 128 rows of w (64 of wg and of wu in the SwiGLU
// form); a wave keeps 8 accumulator tiles of 32 x 32 (its own 64 rows of a x all 128 rows of w).  Few
// tiles take other shapes, a wave then mostly owning 32 rows of a: 64, 96, 128, 192 or 256 rows of a (2 to 6 waves) and 128, 64
// or 32 rows of w, or 320 and 384 rows (10 and 12 waves) and 64 of wg and of wu (see plain_form and swiglu_form);
// an output's sum runs over K in the same order in all of them, so they give the same bits.
// Two workgroups share a CU (two waves per SIMD, 232 registers each): they run out of step, so
// the barrier, prologue and epilogue of one are covered by the matrix work of the other.
// The two operands reach the matrix cores by different roads, which splits the traffic between
// LDS and the vector memory path instead of loading one of them with everything:
//   * w is shared by the four waves: one 64-deep unit (4 blocks of 4 KB, already in MFMA operand
//     order, so they are copied to LDS as they are and read back conflict-free) per step, in one of
//     four LDS stages (with operands two units ahead; the narrow tiles run four ahead).  Buffer loads
//     that write LDS directly bring unit u + 3 while unit u is multiplied; the one barrier per unit waits for those of unit u + 2 only (a counted wait), so
//     the first fragments of unit u + 1 are read before the barrier that ends unit u and no wave
//     starts a unit waiting for LDS.
//   * a rows belong to one wave only, and the tiled layout holds them in operand order: a wave
//     loads its fragments straight from memory into the registers the MFMAs read (1 KB per wave
//     and fragment, fully coalesced), two units ahead, refilling each fragment's registers as soon
//     as the chunk that used them has been issued.
// A wave's loads return in the order in which they were issued, so the wait for the oldest a fragment
// is also a wait for every weight load before it: both kinds run two units ahead, or the shorter
// distance would rule.  (With w through registers, one unit ahead, a unit took the latency of an
// HBM load however little there was to multiply: 300 x 4096 x 14336 181 -> 135 us, 1024 rows
// 190 -> 170 us; at 8192 rows, where L2 serves most loads, 750 -> 731 us.)
// The loads into LDS are buffer loads because the compiler counts those: after a global (flat) load
// into LDS it waits for everything in flight before the next use of any load.
// Per 16-deep chunk a wave reads 4 fragments from LDS, loads 2 from memory and issues 8 MFMAs.
// What bounds the smaller tiles is the compute unit's load path: it takes loads in the order in which they were
// issued, HBM's latency among them, about 32 to 50 KB in flight, which is 60 to 80 GB/s for the mix of weights from
// HBM and activations from L2 (110 to 130 GB/s where L2 has everything).  A unit of a tile of RT x CT blocks costs
// 4 KB (RT + CT) of that, whatever there is to multiply: taking the MFMAs, the barriers or the LDS look-ahead out
// changes nothing, nor do operands four or eight units ahead, so the rules below look for few operand bytes
// per compute unit, not for deep pipelines; asking for the weights of four units at once (B) does help.
// At 8192 rows the part is at its power limit (the matrix pipes are 81 % busy at a lowered clock),
// and variants that differ in barrier scope or fragment look-ahead land on the same rate.
//
// Workgroup numbering follows the hardware's round-robin deal of workgroups to the 8 XCDs: the
// ids that land on one XCD walk a compact patch of output tiles (8 row tiles deep), so that XCD's
// L2 serves each operand tile to several workgroups and HBM sees it about once per patch
// row/column.
#include "kernels_mfma.h"

#include <algorithm>
#include <type_traits>

namespace mc {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) uint32_t v4u;

__device__ inline f32x16 mfma32g(v4u a, v4u b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                 __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
__device__ inline float silu_g(float g) { return g / (1.0f + expf(-g)); }
__device__ inline uint32_t pack2g_bf16(float a, float b) {
  typedef __attribute__((ext_vector_type(2))) float f32x2;
  typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
}

constexpr int kPatchRows = 8;     // output-tile patch walked by one XCD: 8 row tiles deep

// tile (tm, tn) of workgroup `id`; false if the id is padding
__device__ inline bool gemm_tile_of(int id, int tiles_m, int tiles_n, int &tm, int &tn) {
  const int total = tiles_m * tiles_n;
  const int per_xcd = (total + 7) >> 3;
  const int L = (id & 7) * per_xcd + (id >> 3);
  if ((id >> 3) >= per_xcd || L >= total) return false;
  const int band = L / (kPatchRows * tiles_n);              // band of kPatchRows row tiles
  const int rows_here = min(kPatchRows, tiles_m - band * kPatchRows);
  const int in_band = L - band * kPatchRows * tiles_n;
  tn = in_band / rows_here;
  tm = band * kPatchRows + in_band % rows_here;
  return true;
}

// What a workgroup does with its 256 x 128 sums: store them (fp32), the SwiGLU product of two
// weight matrices (bf16, tiled), the fused QKV epilogue (rope_store_quad), or out += sums.
enum { GEMM_STORE = 0, GEMM_SWIGLU = 1, GEMM_ROPE = 2, GEMM_ACCUM = 3 };
// row stride (floats) of a wave's 32 x 128 parking area in the GEMM_ROPE epilogue: 128 + 4, so
// that the 16-byte writes of eight lanes (eight rows) fall into different banks
constexpr int kParkStride = 132;

// All but the newest N vector memory operations of this wave have landed, loads into LDS among them,
// then the workgroup's barrier.  (__syncthreads() would wait for every load in flight.)
template <int N>
__device__ inline void wait_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0F70);    // vmcnt <= N; the other counters free
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// The two ways of a wave's 32 x 32 TN sums, parked in LDS, to queries, keys and values.
// Quad by quad, any head_dim and page: consecutive lanes take consecutive quads of one row.
template <int TN>
__device__ inline void rope_store_quads(const RopeOut &ro, int M, int m0, int n0, const float *park, int lane) {
  constexpr int kBatch = 4;                  // quads per lane whose loads go out together
#pragma unroll 1
  for (int it0 = 0; it0 < 32 * TN * 8 / 64; it0 += kBatch) {
    float4 s[kBatch];
    RopeQuad rq[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int e = (it0 + u) * 64 + lane, row = e / (TN * 8), quad = e % (TN * 8);
      s[u] = *(const float4 *)(park + row * kParkStride + 4 * quad);
      rq[u] = rope_load_quad(ro, min(m0 + row, M - 1), n0 + 4 * quad);
    }
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int e = (it0 + u) * 64 + lane, row = e / (TN * 8), quad = e % (TN * 8);
      if (m0 + row < M) rope_store_quad(ro, m0 + row, n0 + 4 * quad, s[u], rq[u]);
    }
  }
}

// In pieces of 16 bytes, 32 columns (half of them a head's first coordinates, half their partners, or 32 coordinates of
// a value head) at a time: a lane rotates eight pairs of one row and stores two pieces; for the keys the lanes of a store are
// 32 rows, which is a fragment of the page, and a value piece is eight rows of one coordinate, as a fragment has
// them.  By quads a key took 4-byte stores 16 bytes apart and a value 2-byte stores 64 bytes apart, and the
// launch waited for the workgroups that had those: 1000 x 6144 x 4096 75 -> 67 us in a search depth (the plain product
// 57), with the angle table's launch 2048 rows 136 -> 122, 4096 203 -> 186, 8192 375 -> 359.
// Needs whole 32-column blocks inside a head, fragment-order pages and aligned bases.
__device__ inline bool rope_pieces_ok(const RopeOut &ro) {
  return kv_fragment_layout(ro.pg, ro.hd) && (((uintptr_t)ro.q_out | (uintptr_t)ro.k_pages | (uintptr_t)ro.v_pages) & 15) == 0;
}
struct RopeRow {
  int pos, off, page;
};
__device__ inline RopeRow rope_row(const RopeOut &ro, int M, int m) {
  m = min(m, M - 1);
  return RopeRow{ro.row_pos[m], ro.row_off[m], ro.row_page[m]};
}
__device__ inline void rope_store_pieces(const RopeOut &ro, int M, int m0, int n0, int blocks, const RopeRow &mine, const float *park, int lane) {
  const int hd = ro.hd, half = hd >> 1, j = lane & 31, h = lane >> 5;
  const size_t pelems = (size_t)ro.Hkv * hd * ro.pg;
  const int off = mine.off, page = mine.page, rows = min(32, M - m0);
  // The rows fill consecutive slots, of one page between two slots that are multiples of 16: then 16 slots that the values'
  // pieces span have one page.  (The session's passes; a caller's slots may be any.)
  const int off0 = __builtin_amdgcn_readfirstlane(off), before = __shfl_up(page, 1, 32);
  const bool in_line = j >= rows || (off == (off0 + j) % ro.pg && (j == 0 || off % 16 == 0 || page == before));
  const bool regular = __all(in_line);
  // Queries are rows of memory: a store's lanes share a row as far as the columns of one head at hand go (4 blocks of a
  // 128-wide head: eight lanes, whole lines).
  const int span = hd % (32 * blocks) == 0 ? blocks : 32 * blocks % hd == 0 ? hd / 32 : 1;
#pragma unroll 1
  for (int x = 0; x < blocks; ++x) {
    const int n = n0 + 32 * x, head = n / hd;
    if (head < ro.Hq + ro.Hkv) {
      const bool query = head < ro.Hq;
      const int per_row = query ? 2 * span : 1, x0 = query ? x - x % span : x;              // lanes of a row; first block at hand
      const int row = query ? (x - x0) * (64 / per_row) + lane / per_row : j, g = query ? lane % per_row : h;
      const int i = ((n0 + 32 * x0) % hd >> 1) + 8 * g;                                        // this lane's pairs: i .. i + 7
      const int p = query ? __shfl(mine.pos, row) : mine.pos;
      const float4 *src = (const float4 *)(park + 32 * x0 + row * kParkStride + 16 * g);
      const double2 *tp = ro.table + (size_t)p * half + i;
      v4u lo, hi;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float4 s = src[e];
        const double2 t0 = tp[2 * e], t1 = tp[2 * e + 1];
        const double lo0 = s.x, hi0 = s.y, lo1 = s.z, hi1 = s.w;
        lo[e] = (uint32_t)f32_to_bf16((float)(lo0 * t0.x - hi0 * t0.y)) | ((uint32_t)f32_to_bf16((float)(lo1 * t1.x - hi1 * t1.y)) << 16);
        hi[e] = (uint32_t)f32_to_bf16((float)(hi0 * t0.x + lo0 * t0.y)) | ((uint32_t)f32_to_bf16((float)(hi1 * t1.x + lo1 * t1.y)) << 16);
      }
      if (row < rows) {
        bf16_t *dst = query ? (bf16_t *)ro.q_out + ((size_t)(m0 + row) * ro.Hq + head) * hd
                            : (bf16_t *)ro.k_pages + (size_t)page * pelems + (size_t)(head - ro.Hq) * ro.pg * hd;
        *(v4u *)(dst + (query ? i : k_elem_offset(off, i, ro.pg, hd))) = lo;
        *(v4u *)(dst + (query ? i + half : k_elem_offset(off, i + half, ro.pg, hd))) = hi;
      }
      continue;
    }
    const int jp = n % hd;
    const float *blk = park + 32 * x;
    bf16_t *vh = (bf16_t *)ro.v_pages + (size_t)(head - ro.Hq - ro.Hkv) * ro.pg * hd;
    if (regular) {
      // lane: coordinate jp + j; slots 16 g + 4 h + {0..3, 8..11} of the 16-slot groups that the rows reach into
      for (int r0 = -(off0 & 15); r0 < rows; r0 += 16) {
        const int pg_of = __shfl(page, max(0, r0)), slot = (off0 + r0) % ro.pg;
        bf16_t *dst = vh + (size_t)pg_of * pelems + v_elem_offset(slot + 4 * h, jp + j, ro.pg, hd);
        const int ra = r0 + 4 * h, rb = ra + 8;
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = blk[min(max((e < 4 ? ra : rb - 4) + e, 0), 31) * kParkStride + j];
        if (ra >= 0 && rb + 3 < rows) {
          v4u w;
#pragma unroll
          for (int e = 0; e < 4; ++e) w[e] = (uint32_t)f32_to_bf16(v[2 * e]) | ((uint32_t)f32_to_bf16(v[2 * e + 1]) << 16);
          *(v4u *)dst = w;
        } else {
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const int r = (e < 4 ? ra : rb - 4) + e;
            if (r >= 0 && r < rows) dst[e] = f32_to_bf16(v[e]);
          }
        }
      }
    } else {
      for (int c = h; c < 32; c += 2)
        if (j < rows) (vh + (size_t)page * pelems)[v_elem_offset(off, jp + c, ro.pg, hd)] = f32_to_bf16(blk[j * kParkStride + c]);
    }
  }
}

// 1 KB pieces that a wave brings of a unit of `blocks` weight blocks, which divide over as many of the waves as they can
constexpr int weight_pieces(int blocks, int waves) {
  int per = (4 * blocks + waves - 1) / waves;
  while (4 * blocks % per) ++per;
  return per;
}

// TM: 32-row tiles of a per wave; TN: 32-row tiles of each weight matrix per workgroup; D: units by which
// the operands run ahead; WV: waves; NT: w's lines are read by this workgroup only and need not stay in L2; B: 0, or the
// units (a multiple of D) whose weights are asked for at once, at the start of the B units before them, where otherwise every unit
// asks for one.  A wave's loads return in order, so an activation fragment that L2 has waits for every weight load
// from HBM before it; in bursts that wait comes once per B units.  Gains where the compute units' load path is full: 500 x
// 4096 x 14336 by 128 x 64 86 -> 77 us, 640 x 2048 x 8192 49 -> 43 (see plain_form); eight units at once are no better, and
// the SwiGLU form loses (300 x 14336 x 4096 by 320 rows 75 -> 88).
template <int MODE, int TM, int TN, int D, int WV, bool NT, int B>
__global__ __launch_bounds__(64 * WV) __attribute__((amdgpu_waves_per_eu(WV > 8 ? 3 : 2, WV > 8 ? 3 : 2)))
void gemm256_kernel(int M, int Mw, int N, int K, int tiles_m, int tiles_n, const bf16_t *__restrict__ a,
                    const bf16_t *__restrict__ w, const bf16_t *__restrict__ w2,
                    float *__restrict__ out, bf16_t *__restrict__ out_t, RopeOut ro) {
  constexpr bool SWIGLU = MODE == GEMM_SWIGLU;
  constexpr int NW = SWIGLU ? 2 : 1;       // weight matrices
  constexpr int WT = NW * TN;              // weight tiles of one wave
  constexpr int AB = WV * TM;              // 32-row tiles of a per workgroup
  constexpr int WB = TN;                   // blocks of each weight matrix per unit (workgroup)
  constexpr int NBW = NW * WB;             // weight blocks of 256 chunks per unit
  constexpr int PW = weight_pieces(NBW, WV), LW = 4 * NBW / PW;    // 1 KB pieces of w per unit and wave, waves that bring them
  constexpr bool kEven = 4 % WV == 0;      // a load's waves bring neighbouring pieces of a block that is known here
  constexpr int S = B ? 2 * B : D + 2;     // LDS stages of one unit each
  extern __shared__ __attribute__((aligned(16))) unsigned char gemm_lds[];
  v4u *lds = (v4u *)gemm_lds;              // [S][NBW][256], then 1 KB where waves that bring no weights let their empty loads land
  const int tid = threadIdx.x, lane = tid & 63, j = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave;
  int tm, tn;
  if (!gemm_tile_of(blockIdx.x, tiles_m, tiles_n, tm, tn)) return;
  const int U = K >> 6;
  const int mt0 = tm * AB, nt0 = tn * WB;  // first 32-row tile of a / of each weight matrix
  const int m_tiles = (M + 31) >> 5;

  // Weight staging in pieces of 1 KB (a chunk of a block), w's blocks first, then w2's.  With more waves than the
  // pieces divide over, the last waves' loads have an empty range: they fetch nothing and keep the load counts alike.
  const int w_bytes = LW == WV || wave < LW ? WB * U * 4096 : 0;
  const __amdgpu_buffer_rsrc_t wsrc =
      __builtin_amdgcn_make_buffer_rsrc((void *)(w + (size_t)nt0 * U * 2048), 0, w_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t w2src =
      SWIGLU ? __builtin_amdgcn_make_buffer_rsrc((void *)(w2 + (size_t)nt0 * U * 2048), 0, w_bytes, 0x00020000) : wsrc;
  const uint32_t w_off = (kEven ? tid : lane) * 16u;
  // the rows of a come straight from memory in operand order: a chunk of a tile is 1 KB, 16 bytes per lane
  const char *asrc[TM];
#pragma unroll
  for (int y = 0; y < TM; ++y)
    asrc[y] = (const char *)(a + (size_t)min(mt0 + TM * wm + y, m_tiles - 1) * U * 2048);
  const uint32_t a_off = lane * 16u;

  f32x16 acc[WT][TM];
#pragma unroll
  for (int x = 0; x < WT; ++x)
#pragma unroll
    for (int y = 0; y < TM; ++y)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[x][y][r] = 0.f;

  // Loads past the last unit re-read the last unit (in bounds, never used), so that every
  // iteration issues the same loads and the load counters stay exact.
  auto load_w = [&](int u, int stage) __attribute__((always_inline)) {
    const uint32_t at = (uint32_t)min(u, U - 1) * 4096u;
#pragma unroll
    for (int i = 0; i < PW; ++i) {
      constexpr int kPer = kEven ? 4 / WV : 1;
      const int b = kEven ? i / kPer : (wave * PW + i) >> 2, c0 = kEven ? WV * (i % kPer) : (wave * PW + i) & 3;
      v4u *dst = lds + (LW == WV || wave < LW ? stage * NBW * 256 + b * 256 + c0 * 64 + (kEven ? wave * 64 : 0) : S * NBW * 256);
      const uint32_t from = LW == WV || wave < LW ? at + (uint32_t)((b < WB ? b : b - WB) * U) * 4096u + (uint32_t)c0 * 1024u : 0u;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(b < WB ? wsrc : w2src, (__attribute__((address_space(3))) void *)dst,
                                               16, w_off, from, 0, NT ? 2 : 0);
    }
  };
  v4u fa[D][4][TM];
  auto load_a = [&](int slot, int u, int c) __attribute__((always_inline)) {
    const uint32_t at = a_off + (uint32_t)min(u, U - 1) * 4096u + (uint32_t)c * 1024u;
#pragma unroll
    for (int y = 0; y < TM; ++y) fa[slot][c][y] = *(const v4u *)(asrc[y] + at);
  };
  auto read_w = [&](v4u (&fw)[WT], int stage, int c) __attribute__((always_inline)) {
    const v4u *cw = lds + stage * NBW * 256 + lane + c * 64;
#pragma unroll
    for (int x = 0; x < TN; ++x) {
      fw[x] = cw[x * 256];
      if (SWIGLU) fw[TN + x] = cw[(WB + x) * 256];
    }
  };
  auto multiply = [&](const v4u (&fa_)[TM], const v4u (&fw)[WT]) __attribute__((always_inline)) {
#pragma unroll
    for (int y = 0; y < TM; ++y)
#pragma unroll
      for (int x = 0; x < WT; ++x) acc[x][y] = mfma32g(fw[x], fa_[y], acc[x][y]);
  };

  v4u fw[2][WT];
#pragma unroll
  for (int d = 0; d < (B ? B : D + 1); ++d) load_w(d, d);
#pragma unroll
  for (int d = 0; d < D; ++d)
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      load_a(d, d, c);
      __builtin_amdgcn_sched_barrier(0);
    }
  wait_barrier<0>();
  read_w(fw[0], 0, 0);
  // Unit u sits in stage u % S.  The stage that takes unit u + D + 1 was last read during unit u - 1,
  // which every wave left before the barrier that ended it.  At the barrier that ends unit u
  // everything older than the fragments of a for unit u + 1 has landed: the weights of unit u + 2,
  // issued just before them, among it.
  // In bursts: the stages that take units u + B .. u + 2 B - 1, u a multiple of B, were last read in the B units before u, and the
  // burst has to have landed at the barrier that ends unit u + B - 2, the loads of a since then not.
  int cur = 0;
  auto unit = [&](int u, int slot, int b) __attribute__((always_inline)) {
    const int nxt = cur == S - 1 ? 0 : cur + 1;
    if (B == 0) load_w(u + D + 1, cur == 0 ? S - 1 : cur - 1);
    else if (b == 0)
#pragma unroll
      for (int i = 0; i < B; ++i) load_w(u + B + i, (cur + B + i) % S);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      if (c < 3) read_w(fw[(c + 1) & 1], cur, c + 1);
      else read_w(fw[0], nxt, 0);
      multiply(fa[slot][c], fw[c & 1]);
      load_a(slot, u + D, c);
      constexpr int kPairs = TM * WT < WT ? TM * WT : WT;
#pragma unroll
      for (int i = 0; i < kPairs; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);    // one LDS read
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);    // one MFMA
      }
      __builtin_amdgcn_sched_group_barrier(0x008, TM * WT - kPairs, 0);
      __builtin_amdgcn_sched_group_barrier(0x020, TM, 0);     // the loads of a
      __builtin_amdgcn_sched_barrier(0);
    }
    if (B == 0) wait_barrier<4 * TM + (D - 1) * (PW + 4 * TM)>();
    else if (b == B - 2) wait_barrier<B ? (B - 1) * 4 * TM : 0>();
    else wait_barrier<63>();
    cur = nxt;
  };
  int u = 0;
  constexpr int kGroup = B ? B : D;
  do {                                     // U is a multiple of kGroup
#pragma unroll
    for (int d = 0; d < kGroup; ++d) unit(u + d, d % D, d);
    u += kGroup;
  } while (u < U);
  wait_barrier<0>();                         // no load into LDS outlives the loop

  // weight rows are the A operand: a lane holds column m = j of the tile and, per register quad,
  // four consecutive n
  if (MODE == GEMM_ROPE) {
    // The rotation epilogue is long; it runs as a rolled loop over what the wave first parks in its own
    // slice of LDS (free after the last barrier above).
    float *park = (float *)gemm_lds + wave * (32 * kParkStride);
    const bool pieces = rope_pieces_ok(ro);
    RopeRow mine[TM];
#pragma unroll
    for (int y = 0; y < TM; ++y) mine[y] = rope_row(ro, M, 32 * (mt0 + TM * wm + y) + j);
#pragma unroll
    for (int y = 0; y < TM; ++y) {
      const int m0 = 32 * (mt0 + TM * wm + y);
#pragma unroll
      for (int x = 0; x < TN; ++x)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
          const f32x16 &g = acc[x][y];
          *(float4 *)(park + j * kParkStride + 32 * x + 8 * r4 + 4 * h) =
              make_float4(g[4 * r4], g[4 * r4 + 1], g[4 * r4 + 2], g[4 * r4 + 3]);
        }
      if (m0 >= M) continue;
      if (pieces) rope_store_pieces(ro, M, m0, 32 * nt0, TN, mine[y], park, lane);
      else rope_store_quads<TN>(ro, M, m0, 32 * nt0, park, lane);
    }
    return;
  }
#pragma unroll
  for (int y = 0; y < TM; ++y) {
    const int m = 32 * (mt0 + TM * wm + y) + j;
    if (m >= (SWIGLU ? Mw : M)) continue;                  // Mw > M: the padding rows too, as zeros
#pragma unroll
    for (int x = 0; x < TN; ++x)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        const int n = 32 * (nt0 + x) + 8 * r4 + 4 * h;
        const f32x16 &g = acc[x][y];
        if (SWIGLU) {
          const f32x16 &uu = acc[TN + x][y];
          uint2 pk;
          pk.x = pack2g_bf16(silu_g(g[4 * r4]) * uu[4 * r4], silu_g(g[4 * r4 + 1]) * uu[4 * r4 + 1]);
          pk.y = pack2g_bf16(silu_g(g[4 * r4 + 2]) * uu[4 * r4 + 2], silu_g(g[4 * r4 + 3]) * uu[4 * r4 + 3]);
          if (m >= M) pk = make_uint2(0u, 0u);
          *(uint2 *)(out_t + tiled_offset(m, n, N)) = pk;
        } else if (MODE == GEMM_ACCUM) {
          float4 *p = (float4 *)(out + (size_t)m * N + n);
          const float4 old = *p;
          *p = make_float4(old.x + g[4 * r4], old.y + g[4 * r4 + 1], old.z + g[4 * r4 + 2], old.w + g[4 * r4 + 3]);
        } else {
          *(float4 *)(out + (size_t)m * N + n) =
              make_float4(g[4 * r4], g[4 * r4 + 1], g[4 * r4 + 2], g[4 * r4 + 3]);
        }
      }
  }
}

// Matrix-core rate with nothing else going on: every wave keeps 8 accumulator tiles and issues
// MFMAs on operands it loaded once.  What this reaches with realistic operand values is the
// practical ceiling of any GEMM on the part (the clock follows the power drawn, which depends on
// the data: all-zero operands run markedly faster).
__global__ __launch_bounds__(256) void mfma_probe_kernel(const v4u *__restrict__ operands,
                                                         float *__restrict__ out, int iters) {
  const size_t t = (size_t)blockIdx.x * 256 + threadIdx.x;
  v4u a[2], b[4];
#pragma unroll
  for (int i = 0; i < 2; ++i) a[i] = operands[t * 6 + i];
#pragma unroll
  for (int i = 0; i < 4; ++i) b[i] = operands[t * 6 + 2 + i];
  f32x16 acc[8];
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;
  for (int it = 0; it < iters; ++it) {
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
      for (int y = 0; y < 2; ++y) acc[x * 2 + y] = mfma32g(b[x], a[y], acc[x * 2 + y]);
  }
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) s += acc[i][r];
  out[t] = s;
}

int launch_mfma_probe(hipStream_t st, const void *operands, float *out, int n_workgroups, int iters) {
  mfma_probe_kernel<<<n_workgroups, 256, 0, st>>>((const v4u *)operands, out, iters);
  MC_HIP(hipGetLastError());
  return MC_OK;
}

bool gemm256_supported(int M, int N, int K, bool swiglu) {
  (void)swiglu;
  return M >= 1 && K >= 256 && K % 256 == 0 && N % 128 == 0;      // whole groups of four 64-deep units
}

// Plain products: rows per workgroup (64: two waves, 128: four, 256: four with two row tiles each) and weight tiles per
// workgroup.  The first form of the list with which one round (a workgroup to each of the 256 compute units) covers
// the product, else the 256 x 128 tile, which moves the fewest operand bytes per flop; up to 128 rows at least not its
// empty half.  A workgroup is a serial chain over K whose pace is set by its loads, so the list goes by the
// operand bytes per unit: 64 x 32, 128 x 32, 64 x 64, 128 x 64, 128 x 128.  But for one place: 128 x 32 takes five blocks of 4 KB and
// comes before 64 x 64, which takes four.  That gains where 64 x 64 has fewer workgroups (2048 x 8192, 300 rows) and costs
// where it has as many (4096 x 14336, 200 rows).  us, N x K = 4096 x 14336: 100 rows 43 / 62 / 61 / 78 / 115 (256 x 128: 130), 200 rows
// 78 / 60 / 52 / 72 / 105, 256 rows 78 / 64 / 64 / 79 / 125, 300 rows - / 96 / 95 / 67 / 96 (128), 512 rows - / 119 / 122 / 80 / 115
// (150), 1024 rows - / 240 / - / 168 / 126 (158), 1500 rows 327 / 227 / 205 (162) by 128 x 32 / 64 / 128; 4096 x 4096: 100
// rows 15 / 21 / 20 / 25 / 35; 2048 x 8192: 100 rows 25 / 36 / 36 / 45 / 66, 256 rows 26 / 36 / 36 / 45 / 65, 300 rows 43 / 31 / 37 / 39 /
// 56; 6144 x 4096: 100 rows 25 / 21 / 20 / 26 / 36; 5120 x 27648: 100 rows 157 / 125 / 122 / 159, 160 rows 64 x 64 101, 128 x 64 161.
// Over a long K three waves (96 x 64) take the place of 128 x 64 where that is at least 4/3 of the workgroups and still one round: the
// load of a unit that has four row tiles sets the pace of all.  us, 128 x 64 and 96 x 64: 4096 x 14336 (192 and 256 workgroups), 300 rows
// 69 / 67, 330 rows 75 / 71, 384 rows 81 / 75; 4096 x 12288, 300 rows 59 / 58, 384 rows 69 / 64; 5120 x 27648 (160 and 240), 211 rows
// 144 / 126, 256 rows 159 / 133; 3072 x 16384 (144 and 192), 384 rows 87 / 80; 2048 x 12288 (160 and 224), 600 rows 61 / 54.  With fewer
// more it is slower: 2048 x 12288, 576 rows (160 and 192) 57 / 61, 641 rows (192 and 224) 55 / 61; 3072 x 16384, 448 rows (192 and 240)
// 78 / 78; 4096 x 14336, 288 rows (192 both) 66 / 75.  So it is over a short K (2048 x 8192, 768 rows 35 / 36; 4096 x 4096, 384 rows
// 20 / 21); between 8192 and 12288 nothing was measured.
// Weights in bursts (see the kernel): 128 x 64 from K = 2048 on where the row tiles are full to seven eighths and the last one by half, and from K = 4096 on
// two more forms ahead of 128 x 128, 192 x 64 and, up to K = 5120 and where the last row tile is full to three quarters, 256 x 64.  Unit by unit a last row tile
// of few rows leaves the load path to the others; a burst takes it whatever is in it.  us, weights from HBM (each call another matrix).
// 128 x 64 unit by unit / in bursts: 4096 x 14336, 450 rows 81 / 75, 512 rows 86 / 77, 400 rows (the last tile 16) 74 / 77; 2048 x 8192, 640 rows 49 / 43, 1000 rows
// 51 / 47, 800 rows (32) 42.2 / 43.4, 900 rows (4) 43.3 / 44.5; 2048 x 2048, 1000 rows 17.1 / 16.6; 3072 x 2048, 500 rows 16.4 / 15.2.
// 128 x 128 / 192 x 64: 4096 x 14336, 640 rows 125 / 106, 700 rows 108 / 105; 2048 x 8192, 1100 rows 69 / 59, 1300 rows 59.7 / 60.4; 5120 x 5120, 500 rows 50 / 42;
// 5120 x 27648, 576 rows 229 / 212; 7168 x 5120, 384 rows 52 / 43; K = 2048, 4096 columns 600 rows 18 / 20.
// 128 x 128 / 256 x 64: 6144 x 4096, 450 rows 40 / 37; 7168 x 5120, 512 rows 53 / 48, 400 rows (the last tile 144) 44 / 45; 4096 x 4096, 1024 rows 43 / 41, 900 rows (132)
// 38 / 40; 5120 x 5120, 768 rows 52 / 48, 700 rows (188) 46 / 47; over a long K 4096 x 8192, 1024 rows 76 / 78, 900 rows 67 / 72, 2048 x 8192, 2000 rows 75 / 78, 4096 x 14336,
// 1000 rows 130 / 126, 900 rows 114 / 136, 5120 x 27648, 768 rows 247 / 261.  Between K = 5120 and 8192 nothing was measured.
struct GemmForm { int waves, tm, tn; bool burst = false; };
constexpr long kComputeUnits = 256;
static GemmForm plain_form(int M, int N, int K) {
  for (const GemmForm f : {GemmForm{2, 1, 1}, GemmForm{4, 1, 1}, GemmForm{2, 1, 2}, GemmForm{4, 1, 2}, GemmForm{6, 1, 2, true}, GemmForm{4, 2, 2, true},
                           GemmForm{4, 1, 4}}) {
    const int rows = 32 * f.waves * f.tm;
    const long row_tiles = (M + rows - 1) / rows;
    if (row_tiles * (N / 32) / f.tn > kComputeUnits) continue;
    const long last = M - (row_tiles - 1) * rows;              // rows of the last row tile
    if (f.burst && (K < 4096 || (f.tm == 2 && (K > 5120 || 4 * last < 3 * rows)))) continue;
    if (f.waves == 4 && f.tm == 1 && f.tn == 2) {
      const long by_96 = (M + 95) / 96;
      if (K >= 12288 && 3 * by_96 >= 4 * row_tiles && by_96 * (N / 64) <= kComputeUnits) return GemmForm{3, 1, 2};
      return GemmForm{4, 1, 2, K >= 2048 && 8L * M > 7L * rows * row_tiles && 2 * last >= rows};
    }
    return f;
  }
  return GemmForm{4, M <= 128 ? 1 : 2, 4};
}

// The SwiGLU form has two weight matrices and a wide output: 128 x (32 + 32) or 128 x (64 + 64) where one round covers the
// product.  Otherwise tiles of 256 rows, two workgroups to a compute unit, or of 320 or 384 rows (a wave per row tile), one
// to a unit: whichever takes least by the rounds that it needs, in hundredths of a microsecond per 64-deep unit as measured.
// A round of 512 workgroups of 256 rows takes 152, of up to 256 (one to a unit) 92, one of 256 workgroups of 320 or 384 rows
// 122 or 125.  us, N x K = 14336 x 4096, 256 / 320 / 384 rows per workgroup: 300 rows 97 / 78 / 81, 330 and 384 rows 99 / 96 and more /
// 80, 512 rows 103 / 120 / 120, 640 rows 147 / 145 / 154, 900 rows 195 / 208 / -; 27648 x 5120: 300 rows 228 / 182 / 195, 384 rows 238 / - /
// 190, 640 rows 355 / 340 / 374, 900 rows 428 / 506; 8192 x 2048: 640 rows 49 / 41 / 45, 300 rows 32 / 37 / 37.
// (Smaller forms, us: 14336 x 4096, 128 rows 77 / 49 / 62 by 256 rows, 128 x (64 + 64), 128 x (32 + 32); 256 rows 59 / 76 / 100.)
static GemmForm swiglu_form(int M, int N) {
  const long row_tiles = (M + 127) / 128, groups = N / 64;
  if (row_tiles * groups * 2 <= kComputeUnits) return GemmForm{4, 1, 1};
  if (row_tiles * groups <= kComputeUnits || M <= 128) return GemmForm{4, 1, 2};
  const long wide = (M + 255) / 256 * groups, rest = wide % (2 * kComputeUnits);
  GemmForm best{4, 2, 2};
  long least = wide / (2 * kComputeUnits) * 152 + (rest == 0 ? 0 : rest <= kComputeUnits ? 92 : 152);
  for (const int waves : {10, 12}) {
    const long count = (M + 32 * waves - 1) / (32 * waves) * groups;
    const long cost = (count + kComputeUnits - 1) / kComputeUnits * (waves == 10 ? 122 : 125);
    // a tenth less, as few rounds say little (2100 x 8192 x 2048: 137 us by 256 rows, 145 by 384)
    if (cost < (best.waves == 4 ? least * 9 / 10 : least)) {
      least = cost;
      best = GemmForm{waves, 1, 2};
    }
  }
  return best;
}

void gemm256_plan(int M, int N, int K, bool swiglu, int32_t *out3) {
  const GemmForm f = swiglu ? swiglu_form(M, N) : plain_form(M, N, K);
  out3[0] = 32 * f.waves * f.tm;
  out3[1] = 32 * f.tn;
  out3[2] = (M + out3[0] - 1) / out3[0] * (N / out3[1]);
}

template <int MODE, int TM, int TN, int D, int WV, bool NT = false, int B = 0>
static int launch_gemm256_t(hipStream_t st, int M, int Mw, int N, int K, const bf16_t *a, const bf16_t *w,
                            const bf16_t *w2, float *out, bf16_t *out_t, const RopeOut &ro) {
  const int tiles_m = (M + 32 * WV * TM - 1) / (32 * WV * TM), tiles_n = N / (32 * TN);
  const int per_xcd = (tiles_m * tiles_n + 7) / 8;
  // the stages of the unit's weight blocks and a place for empty loads; the parking areas of the rotation epilogue may need more
  constexpr int NBW = TN * (MODE == GEMM_SWIGLU ? 2 : 1);
  const int lds = std::max<int>((B ? 2 * B : D + 2) * NBW * 4096 + (weight_pieces(NBW, WV) * WV > 4 * NBW ? 1024 : 0),
                                MODE == GEMM_ROPE ? WV * 32 * kParkStride * (int)sizeof(float) : 0);
  MC_TRY(raise_dynamic_lds_limit((const void *)gemm256_kernel<MODE, TM, TN, D, WV, NT, B>, lds));
  gemm256_kernel<MODE, TM, TN, D, WV, NT, B><<<8 * per_xcd, 64 * WV, lds, st>>>(M, Mw, N, K, tiles_m, tiles_n, a, w, w2, out, out_t, ro);
  MC_HIP(hipGetLastError());
  return MC_OK;
}

int launch_gemm256(hipStream_t st, int M, int N, int K, const void *a, const void *w,
                   const void *w2, float *out, void *out_t, const RopeOut *rope, int accumulate, bool zero_pad) {
  const bool swiglu = w2 != nullptr;
  const int Mw = zero_pad ? padded_rows(M) : M;
  if (!gemm256_supported(M, N, K, swiglu)) MC_FAIL(MC_ERR_UNSUPPORTED, "GEMM: M=%d N=%d K=%d not covered", M, N, K);
  if ((swiglu && (rope || accumulate)) || (rope && accumulate))
    MC_FAIL(MC_ERR_INVALID, "GEMM: one output form at a time");
  if (rope && (rope->hd % 4 || N != (rope->Hq + 2 * rope->Hkv) * rope->hd))
    MC_FAIL(MC_ERR_INVALID, "fused QKV output: N = (Hq + 2 Hkv) hd, hd %% 4 == 0");
  const bf16_t *A = (const bf16_t *)a, *W = (const bf16_t *)w, *W2 = (const bf16_t *)w2;
  bf16_t *OT = (bf16_t *)out_t;
  const GemmForm f = swiglu ? swiglu_form(M, N) : plain_form(M, N, K);
  auto run = [&](auto mode) -> int {
    constexpr int MODE = decltype(mode)::value;
    const RopeOut ro = rope ? *rope : RopeOut{};
    if constexpr (MODE == GEMM_SWIGLU) {
      if (f.tm == 2) return launch_gemm256_t<MODE, 2, 2, 2, 4>(st, M, Mw, N, K, A, W, W2, out, OT, ro);
      if (f.waves == 10) return launch_gemm256_t<MODE, 1, 2, 2, 10>(st, M, Mw, N, K, A, W, W2, out, OT, ro);
      if (f.waves == 12) return launch_gemm256_t<MODE, 1, 2, 2, 12>(st, M, Mw, N, K, A, W, W2, out, OT, ro);
      // one row tile: every weight is read once (14336 x 4096, 100 rows: 49.4 -> 45.7 us)
      if (f.tn == 2 && M <= 128) return launch_gemm256_t<MODE, 1, 2, 2, 4, true>(st, M, Mw, N, K, A, W, W2, out, OT, ro);
      if (f.tn == 2) return launch_gemm256_t<MODE, 1, 2, 2, 4>(st, M, Mw, N, K, A, W, W2, out, OT, ro);
      return launch_gemm256_t<MODE, 1, 1, 2, 4>(st, M, Mw, N, K, A, W, W2, out, OT, ro);
    } else {
      if (f.tm == 2 && f.tn == 4) return launch_gemm256_t<MODE, 2, 4, 2, 4>(st, M, Mw, N, K, A, W, W2, out, OT, ro);
      if (f.tm == 2) return launch_gemm256_t<MODE, 2, 2, 2, 4, false, 4>(st, M, Mw, N, K, A, W, W2, out, OT, ro);
      if (f.waves == 6) return launch_gemm256_t<MODE, 1, 2, 4, 6, false, 4>(st, M, Mw, N, K, A, W, W2, out, OT, ro);
      if (f.waves == 3) return launch_gemm256_t<MODE, 1, 2, 4, 3>(st, M, Mw, N, K, A, W, W2, out, OT, ro);
      if (f.tn == 4) return launch_gemm256_t<MODE, 1, 4, 2, 4>(st, M, Mw, N, K, A, W, W2, out, OT, ro);
      if (f.waves == 2 && f.tn == 2) return launch_gemm256_t<MODE, 1, 2, 4, 2>(st, M, Mw, N, K, A, W, W2, out, OT, ro);
      if (f.waves == 2) return launch_gemm256_t<MODE, 1, 1, 4, 2>(st, M, Mw, N, K, A, W, W2, out, OT, ro);
      if (f.tn == 2 && f.burst) return launch_gemm256_t<MODE, 1, 2, 4, 4, false, 4>(st, M, Mw, N, K, A, W, W2, out, OT, ro);
      if (f.tn == 2) return launch_gemm256_t<MODE, 1, 2, 4, 4>(st, M, Mw, N, K, A, W, W2, out, OT, ro);
      return launch_gemm256_t<MODE, 1, 1, 4, 4>(st, M, Mw, N, K, A, W, W2, out, OT, ro);
    }
  };
  if (swiglu) return run(std::integral_constant<int, GEMM_SWIGLU>{});
  if (rope) return run(std::integral_constant<int, GEMM_ROPE>{});
  if (accumulate) return run(std::integral_constant<int, GEMM_ACCUM>{});
  return run(std::integral_constant<int, GEMM_STORE>{});
}

}  // namespace mc
