// Many-row bf16 GEMM on tiled operands (gfx950, v_mfma_f32_32x32x16_bf16):
//   out[m][n] = sum_k a[m][k] w[n][k]                 (fp32, row-major), or
//   out_t[m][n] = silu(a . wg[n]) * (a . wu[n])        (bf16, tiled; the SwiGLU form).
//
// A workgroup of 4 waves owns 256 (few tiles: 128) rows of a and 128 rows of w (64 of wg and of wu in
// the SwiGLU form); a wave keeps 8 (4) accumulator tiles of 32 x 32 (its own 64 (32) rows of a x all
// 128 rows of w).
// Two workgroups share a CU (two waves per SIMD, 215 registers each): they run out of step, so
// the barrier, prologue and epilogue of one are covered by the matrix work of the other.
// The two operands reach the matrix cores by different roads, which splits the traffic between
// LDS and the vector memory path instead of loading one of them with everything:
//   * w is shared by the four waves: one 64-deep unit (4 blocks of 4 KB, already in MFMA operand
//     order, so they are copied to LDS as they are and read back conflict-free) per step, in one of
//     four LDS stages.  Buffer loads that write LDS directly bring unit u + 3 while unit u is
//     multiplied; the one barrier per unit waits for those of unit u + 2 only (a counted wait), so
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

// TM: 32-row tiles of a per wave, 2 or 1 (256 or 128 rows of a per workgroup).  gridDim.y > 1: the
// workgroups of split y take units [y, y + 1) * units_per_split of K and store their sums to
// out + y * M * N.
template <int MODE, int TM>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
void gemm256_kernel(int M, int N, int K, int units_per_split, int tiles_m, int tiles_n, const bf16_t *__restrict__ a,
                    const bf16_t *__restrict__ w, const bf16_t *__restrict__ w2,
                    float *__restrict__ out, bf16_t *__restrict__ out_t, RopeOut ro) {
  constexpr bool SWIGLU = MODE == GEMM_SWIGLU;
  constexpr int NW = SWIGLU ? 2 : 1;       // weight matrices
  constexpr int TN = SWIGLU ? 2 : 4;       // 32-row tiles of each weight matrix per wave
  constexpr int WT = NW * TN;              // weight tiles of one wave (4)
  constexpr int AB = 4 * TM;               // 32-row tiles of a per workgroup
  constexpr int WB = TN;                   // blocks of each weight matrix per unit (workgroup)
  constexpr int NBW = NW * WB;             // 4 weight blocks of 256 chunks per unit
  extern __shared__ __attribute__((aligned(16))) unsigned char gemm_lds[];
  v4u *lds = (v4u *)gemm_lds;              // [4 stages][NBW][256]
  const int tid = threadIdx.x, lane = tid & 63, j = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave;
  int tm, tn;
  if (!gemm_tile_of(blockIdx.x, tiles_m, tiles_n, tm, tn)) return;
  const int KU = K >> 6, u_first = blockIdx.y * units_per_split, U = min(units_per_split, KU - u_first);
  if (MODE == GEMM_STORE) out += (size_t)blockIdx.y * M * N;
  const int mt0 = tm * AB, nt0 = tn * WB;  // first 32-row tile of a / of each weight matrix
  const int m_tiles = (M + 31) >> 5;

  // weight staging: thread t brings chunk t of every block of the unit, w's blocks first, then w2's
  const __amdgpu_buffer_rsrc_t wsrc =
      __builtin_amdgcn_make_buffer_rsrc((void *)(w + (size_t)nt0 * KU * 2048), 0, WB * KU * 4096, 0x00020000);
  const __amdgpu_buffer_rsrc_t w2src =
      SWIGLU ? __builtin_amdgcn_make_buffer_rsrc((void *)(w2 + (size_t)nt0 * KU * 2048), 0, WB * KU * 4096, 0x00020000) : wsrc;
  const uint32_t s_off = tid * 16u;
  // the rows of a come straight from memory in operand order: a chunk of a tile is 1 KB, 16 bytes per lane
  const char *asrc[TM];
#pragma unroll
  for (int y = 0; y < TM; ++y)
    asrc[y] = (const char *)(a + ((size_t)min(mt0 + TM * wm + y, m_tiles - 1) * KU + u_first) * 2048);
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
    const uint32_t at = (uint32_t)(u_first + min(u, U - 1)) * 4096u;
    v4u *dst = lds + stage * NBW * 256 + wave * 64;
#pragma unroll
    for (int i = 0; i < NBW; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(i < WB ? wsrc : w2src, (__attribute__((address_space(3))) void *)(dst + i * 256),
                                               16, s_off, at + (uint32_t)((i < WB ? i : i - WB) * KU) * 4096u, 0, 0);
  };
  v4u fa[2][4][TM];
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
  for (int d = 0; d < 3; ++d) load_w(d, d);
#pragma unroll
  for (int d = 0; d < 2; ++d)
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      load_a(d, d, c);
      __builtin_amdgcn_sched_barrier(0);
    }
  wait_barrier<0>();
  read_w(fw[0], 0, 0);
  // Stage (u + 3) % 4 was last read during unit u - 1, which every wave left before the barrier that
  // ended it.  At the barrier that ends unit u everything older than the fragments of a for unit
  // u + 1 has landed: the weights of unit u + 2, issued at the top of unit u - 1, before them.
  auto unit = [&](int u, int slot) __attribute__((always_inline)) {
    const int cur = u & 3, nxt = (u + 1) & 3;
    load_w(u + 3, (u + 3) & 3);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      if (c < 3) read_w(fw[(c + 1) & 1], cur, c + 1);
      else read_w(fw[0], nxt, 0);
      multiply(fa[slot][c], fw[c & 1]);
      load_a(slot, u + 2, c);
#pragma unroll
      for (int i = 0; i < WT; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);    // one LDS read
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);    // one MFMA
      }
      __builtin_amdgcn_sched_group_barrier(0x008, TM * WT - WT, 0);
      __builtin_amdgcn_sched_group_barrier(0x020, TM, 0);     // the loads of a
      __builtin_amdgcn_sched_barrier(0);
    }
    wait_barrier<8 * TM + NBW>();            // a of units u + 1 and u + 2, w of unit u + 3 may be in flight
  };
  int u = 0;
  do {                                     // U is even and at least 2
    unit(u, 0);
    unit(u + 1, 1);
    u += 2;
  } while (u < U);
  wait_barrier<0>();                         // no load into LDS outlives the loop

  // weight rows are the A operand: a lane holds column m = j of the tile and, per register quad,
  // four consecutive n
  if (MODE == GEMM_ROPE) {
    // The rotation epilogue is long; it runs as a rolled loop over quads that the wave first
    // parks in its own slice of LDS (free after the last barrier above).  The loop hands
    // consecutive lanes consecutive quads of one row, so table reads and query stores coalesce.
    float *park = (float *)gemm_lds + wave * (32 * kParkStride);
    const int n_wave = 32 * nt0;
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
      constexpr int kBatch = 4;        // quads per lane whose loads go out together
#pragma unroll 1
      for (int it0 = 0; it0 < 32 * TN * 8 / 64; it0 += kBatch) {
        float4 s[kBatch];
        RopeQuad rq[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
          const int e = (it0 + u) * 64 + lane, row = e / (TN * 8), quad = e % (TN * 8);
          s[u] = *(const float4 *)(park + row * kParkStride + 4 * quad);
          rq[u] = rope_load_quad(ro, min(m0 + row, M - 1), n_wave + 4 * quad);
        }
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
          const int e = (it0 + u) * 64 + lane, row = e / (TN * 8), quad = e % (TN * 8);
          if (m0 + row < M) rope_store_quad(ro, m0 + row, n_wave + 4 * quad, s[u], rq[u]);
        }
      }
    }
    return;
  }
#pragma unroll
  for (int y = 0; y < TM; ++y) {
    const int m = 32 * (mt0 + TM * wm + y) + j;
    if (m >= M) continue;
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

// =====================================================================================
// The same products for a few hundred rows.  One 256 x 128 tile per workgroup leaves most of the
// chip idle there (300 x 4096 x 14336: 64 workgroups for 256 compute units, each a serial chain of
// 224 units), and a split of K over workgroups needs a place for partial sums.  Here the tile is 64
// rows of a x 32 WT rows of w and K is split over the eight WAVES of a workgroup: wave s takes units
// s, s + 8, ... with the whole tile in its accumulators, streams both operands from memory straight
// into MFMA operand registers (the tiled layout is the operand order; 1 KB per load, a chunk's
// registers are refilled for the wave's next unit right after the MFMAs that read them) and meets the
// other seven in LDS at the end.  No barrier and no LDS in the loop; complete sums in a fixed order,
// so every epilogue of the large kernel works on them and results do not depend on scheduling.
// What bounds it: a workgroup pulls its 64 + 32 WT operand rows through one compute unit's L1 at
// 60-70 GB/s (100 when few workgroups run); neither two units in flight per wave nor other K orders
// nor leaving the MFMAs out changed that.  300 x 4096 x 14336: 135 -> 82 us (181 with the weights
// through registers), 128 x 4096 x 14336: 128 -> 46 us, 300 x 6144 x 4096: 44 -> 26 us.
// =====================================================================================
constexpr int kSlices = 8;                 // waves per workgroup, one K slice each

template <int MODE, int WT>
__global__ __launch_bounds__(64 * kSlices) __attribute__((amdgpu_waves_per_eu(2, 2)))
void gemm_kslice_kernel(int M, int N, int K, int tiles_m, int tiles_n, const bf16_t *__restrict__ a,
                        const bf16_t *__restrict__ w, const bf16_t *__restrict__ w2,
                        float *__restrict__ out, bf16_t *__restrict__ out_t, RopeOut ro) {
  constexpr bool SWIGLU = MODE == GEMM_SWIGLU;
  constexpr int NW = SWIGLU ? 2 : 1;       // weight matrices
  constexpr int TN = WT / NW;              // 32-row tiles of each weight matrix
  constexpr int TM = 2;                    // 32-row tiles of a
  extern __shared__ __attribute__((aligned(16))) unsigned char gemm_lds[];
  float4 *red = (float4 *)gemm_lds;        // [kSlices][WT][4 quads][64 slots]
  const int tid = threadIdx.x, lane = tid & 63, j = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // consecutive ids of one XCD walk the row tiles of one weight tile first: its L2 hands the
  // weights to all of them
  const int total = tiles_m * tiles_n, per_xcd = (total + 7) >> 3;
  const int L = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= per_xcd || L >= total) return;
  const int tm = L % tiles_m, tn = L / tiles_m;
  const int U = K >> 6, mt0 = tm * TM, nt0 = tn * TN, m_tiles = (M + 31) >> 5;

  const char *src[TM + WT];
#pragma unroll
  for (int y = 0; y < TM; ++y) src[y] = (const char *)(a + (size_t)min(mt0 + y, m_tiles - 1) * U * 2048);
#pragma unroll
  for (int x = 0; x < WT; ++x)
    src[TM + x] = (const char *)(x < TN ? w + (size_t)(nt0 + x) * U * 2048 : w2 + (size_t)(nt0 + x - TN) * U * 2048);
  const uint32_t lane_off = lane * 16u;

  f32x16 acc[WT][TM];
#pragma unroll
  for (int x = 0; x < WT; ++x)
#pragma unroll
    for (int y = 0; y < TM; ++y)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[x][y][r] = 0.f;

  v4u f[4][TM + WT];
  auto load = [&](int u, int c) __attribute__((always_inline)) {
    const uint32_t at = lane_off + (uint32_t)u * 4096u + (uint32_t)c * 1024u;
#pragma unroll
    for (int i = 0; i < TM + WT; ++i) f[c][i] = *(const v4u *)(src[i] + at);
  };
  auto multiply = [&](int c) __attribute__((always_inline)) {
#pragma unroll
    for (int y = 0; y < TM; ++y)
#pragma unroll
      for (int x = 0; x < WT; ++x) acc[x][y] = mfma32g(f[c][TM + x], f[c][y], acc[x][y]);
  };
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    load(min(wave, U - 1), c);
    __builtin_amdgcn_sched_barrier(0);         // in the order of the loop, whose waits then leave the later loads in flight
  }
  int u = wave;
  for (; u + kSlices < U; u += kSlices)
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      multiply(c);
      load(u + kSlices, c);
      __builtin_amdgcn_sched_barrier(0);
    }
  if (u < U)                                   // (a short K leaves the last waves without a unit)
#pragma unroll
    for (int c = 0; c < 4; ++c) multiply(c);

  // A lane holds column j of a row tile and, per register quad, four consecutive n.  Quad (x, r4)
  // of lane (j, h) sits in slot 2 j + h, rotated by twice the quad's number: the 32 quads of one
  // row then fall into different banks, and so do the quads of a wave that walks rows.
#pragma unroll
  for (int y = 0; y < TM; ++y) {
    const int m0 = 32 * (mt0 + y);
    if (m0 >= M) break;                                  // uniform
    if (y) __syncthreads();                              // the first half has been read
#pragma unroll
    for (int x = 0; x < WT; ++x)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        const f32x16 &g = acc[x][y];
        red[((wave * WT + x) * 4 + r4) * 64 + ((2 * j + h + 2 * (4 * x + r4)) & 63)] =
            make_float4(g[4 * r4], g[4 * r4 + 1], g[4 * r4 + 2], g[4 * r4 + 3]);
      }
    __syncthreads();
    auto sum = [&](int x, int r4, int row, int hh) __attribute__((always_inline)) {
      const float4 *p = red + (x * 4 + r4) * 64 + ((2 * row + hh + 2 * (4 * x + r4)) & 63);
      float4 t = p[0];
#pragma unroll
      for (int s = 1; s < kSlices; ++s) {
        const float4 v = p[s * WT * 256];
        t.x += v.x; t.y += v.y; t.z += v.z; t.w += v.w;
      }
      return t;
    };
    if (SWIGLU) {
      // tiled output: 32 rows x 16 bytes of one chunk are neighbours, so lanes walk the rows
      for (int e = tid; e < TN * 256; e += 64 * kSlices) {
        const int x = e >> 8, r4 = (e >> 6) & 3, hh = e & 1, row = (e >> 1) & 31;
        const int m = m0 + row, n = 32 * (nt0 + x) + 8 * r4 + 4 * hh;
        const float4 g = sum(x, r4, row, hh), v = sum(TN + x, r4, row, hh);
        if (m < M) {
          uint2 pk;
          pk.x = pack2g_bf16(silu_g(g.x) * v.x, silu_g(g.y) * v.y);
          pk.y = pack2g_bf16(silu_g(g.z) * v.z, silu_g(g.w) * v.w);
          *(uint2 *)(out_t + tiled_offset(m, n, N)) = pk;
        }
      }
    } else {
      // row-major output: consecutive lanes take consecutive quads of one row
      for (int e = tid; e < WT * 256; e += 64 * kSlices) {
        const int row = e / (8 * WT), q = e % (8 * WT);
        const int m = m0 + row, n = 32 * nt0 + 4 * q;
        const float4 t = sum(q >> 3, (q >> 1) & 3, row, q & 1);
        if (m >= M) continue;
        if (MODE == GEMM_ROPE) {
          rope_store_quad(ro, m, n, t, rope_load_quad(ro, m, n));
        } else {
          float4 *p = (float4 *)(out + (size_t)m * N + n);
          if (MODE == GEMM_ACCUM) {
            const float4 old = *p;
            *p = make_float4(old.x + t.x, old.y + t.y, old.z + t.z, old.w + t.w);
          } else {
            *p = t;
          }
        }
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
  return M >= 1 && K >= 128 && K % 128 == 0 && N % 128 == 0;      // whole pairs of 64-deep units
}

constexpr int kComputeUnits = 256;

// Weight tiles per workgroup of the K-slice kernel, or 0 where the large tiles are better: the fewest
// with which one round of workgroups (a compute unit holds one) covers the product.  More rounds
// repeat its start and its reduction, and the large tiles move fewer operand bytes.
// Large tiles / 4 / 2 / 1 weight tiles, us, at the largest row counts that take each and past them:
// 4096 x 14336 (N x K): 128 rows 128 / 91 / 62 / 46, 256 rows 133 / 80 / 55 / 73, 512 rows 125 / 85 /
// 117 / 159, 768 rows 130 / 160 / 178 / 278; SwiGLU 8192 x 2048: 128 rows 21 / 19 / 24.
static int kslice_tiles(int M, int N, bool swiglu) {
  const long row_tiles = (M + 63) / 64;
  for (int wt = swiglu ? 2 : 1; wt <= 4; wt *= 2)
    if (row_tiles * (N / 32) * (swiglu ? 2 : 1) / wt <= kComputeUnits) return wt;
  return 0;
}

// 128 instead of 256 rows of a per workgroup: where the chip holds all of those tiles at once, one to
// a compute unit (1024 x 4096 x 14336: 170 -> 132 us; 1024 x 6144 x 4096, 384 tiles: 54 -> 68 us), or
// the row count would leave half of a large tile empty (128 rows of SwiGLU 14336 x 4096: 62 -> 49 us).
static bool gemm_half_rows(int M, int N, bool swiglu) {
  return M <= 128 || (long)((M + 127) / 128) * (N / (swiglu ? 64 : 128)) <= kComputeUnits;
}

template <int MODE, int TM>
static int launch_gemm256_t(hipStream_t st, int M, int N, int K, int n_splits, const bf16_t *a, const bf16_t *w,
                            const bf16_t *w2, float *out, bf16_t *out_t, const RopeOut &ro) {
  const int tiles_m = (M + 128 * TM - 1) / (128 * TM), tiles_n = N / (MODE == GEMM_SWIGLU ? 64 : 128);
  const int per_xcd = (tiles_m * tiles_n + 7) / 8;
  const int units = K / 64, per_split = (units / 2 + n_splits - 1) / n_splits * 2;      // whole pairs of units
  // four stages of 4 weight blocks; the parking areas of the rotation epilogue need a little more
  const int lds = std::max<int>(4 * 4 * 4096, MODE == GEMM_ROPE ? 4 * 32 * kParkStride * (int)sizeof(float) : 0);
  MC_TRY(raise_dynamic_lds_limit((const void *)gemm256_kernel<MODE, TM>, lds));
  gemm256_kernel<MODE, TM><<<dim3(8 * per_xcd, n_splits), 256, lds, st>>>(M, N, K, per_split, tiles_m, tiles_n, a, w, w2, out, out_t, ro);
  MC_HIP(hipGetLastError());
  return MC_OK;
}

template <int MODE, int WT>
static int launch_kslice_t(hipStream_t st, int M, int N, int K, const bf16_t *a, const bf16_t *w, const bf16_t *w2,
                           float *out, bf16_t *out_t, const RopeOut &ro) {
  const int tiles_m = (M + 63) / 64, tiles_n = N / 32 * (MODE == GEMM_SWIGLU ? 2 : 1) / WT;
  const int per_xcd = (tiles_m * tiles_n + 7) / 8, lds = kSlices * WT * 4096;
  MC_TRY(raise_dynamic_lds_limit((const void *)gemm_kslice_kernel<MODE, WT>, lds));
  gemm_kslice_kernel<MODE, WT><<<8 * per_xcd, 64 * kSlices, lds, st>>>(M, N, K, tiles_m, tiles_n, a, w, w2, out, out_t, ro);
  MC_HIP(hipGetLastError());
  return MC_OK;
}

int launch_gemm256(hipStream_t st, int M, int N, int K, const void *a, const void *w,
                   const void *w2, float *out, void *out_t, const RopeOut *rope, int accumulate) {
  const bool swiglu = w2 != nullptr;
  if (!gemm256_supported(M, N, K, swiglu)) MC_FAIL(MC_ERR_UNSUPPORTED, "GEMM: M=%d N=%d K=%d not covered", M, N, K);
  if ((swiglu && (rope || accumulate)) || (rope && accumulate))
    MC_FAIL(MC_ERR_INVALID, "GEMM: one output form at a time");
  if (rope && (rope->hd % 4 || N != (rope->Hq + 2 * rope->Hkv) * rope->hd))
    MC_FAIL(MC_ERR_INVALID, "fused QKV output: N = (Hq + 2 Hkv) hd, hd %% 4 == 0");
  const bf16_t *A = (const bf16_t *)a, *W = (const bf16_t *)w, *W2 = (const bf16_t *)w2;
  bf16_t *OT = (bf16_t *)out_t;
  const int wt = kslice_tiles(M, N, swiglu);
  auto run = [&](auto mode) -> int {
    constexpr int MODE = decltype(mode)::value;
    const RopeOut ro = rope ? *rope : RopeOut{};
    if (wt == 4) return launch_kslice_t<MODE, 4>(st, M, N, K, A, W, W2, out, OT, ro);
    if (wt == 2) return launch_kslice_t<MODE, 2>(st, M, N, K, A, W, W2, out, OT, ro);
    if constexpr (MODE != GEMM_SWIGLU)
      if (wt == 1) return launch_kslice_t<MODE, 1>(st, M, N, K, A, W, W2, out, OT, ro);
    return gemm_half_rows(M, N, swiglu) ? launch_gemm256_t<MODE, 1>(st, M, N, K, 1, A, W, W2, out, OT, ro)
                                        : launch_gemm256_t<MODE, 2>(st, M, N, K, 1, A, W, W2, out, OT, ro);
  };
  if (swiglu) return run(std::integral_constant<int, GEMM_SWIGLU>{});
  if (rope) return run(std::integral_constant<int, GEMM_ROPE>{});
  if (accumulate) return run(std::integral_constant<int, GEMM_ACCUM>{});
  return run(std::integral_constant<int, GEMM_STORE>{});
}

}  // namespace mc
