// Dense pass over X: for every slice t and ensemble member r, in ONE read of X_t,
//   P = X^r_t A^r   (Alg. 3: XA)      and      Q = X^r_t^T A^r   (Alg. 3: XTAR before the R_t factor),
// with X^r = X (*) Delta^r generated on the fly (Alg. 4) from a counter-based random stream, so the
// perturbed tensors are never stored and X is read once for all members of a group.
//
// Mapping to CDNA4.  The contraction runs on the bf16 matrix cores: every fp32 operand is a sum of three bf16 terms, without
// a rest, and a 16 x 16 x 16 product of fp32 numbers is three v_mfma_f32_16x16x32_bf16 (bf16split.h).  They take 50
// cycles; the four v_mfma_f32_16x16x4_f32 of the same product take 129 and, sharing the vector ALUs, let no vector
// instruction run beside them, while the generator's multiplications run beside bf16 MFMA for free (measured).
// Of an instruction's result D[16x16], lane l holds D[4*(l/16)+r][l%16] in register r.  The perturbed X tile is the left
// operand, built in registers by the lane that loaded the element; rows of the factor are the right operand, read from
// a copy of A that is stored in operand order (two 16-byte loads per lane and product group).
//
// A workgroup of W = 8 or 4 waves owns a panel of 16 W columns (W tiles) and a chunk of rows.  In a round, every wave takes
// one 16-row strip and walks it across the panel, tile by tile:
//   - the strip's P accumulators and the right operands of the Q products (the strip's 16 factor rows) stay
//     in registers for the whole strip; P is added to memory once per strip;
//   - the tile's terms are parked in LDS and read back transposed (ds_read_b64_tr_b16) for the Q product, so the
//     generator and the split into terms run once per element;
//   - the panel's Q accumulators live in LDS in accumulator order.  In step s wave w works on tile
//     (w + s) % W, so at any time each tile column has one owner, which adds the tile's products to the
//     accumulators: no atomics and no cross-wave reduction.  (The bf16 instruction cuts what lies 2^-8 of its C
//     operand's last place or deeper.  Over the thousands of instructions of a chunk that added up to 2.8e-7 of Q, always
//     downwards; with a tile's products summed from zero and added by vector instructions Q is off by 1.5e-9 in the
//     mean and 1.2e-7 in all at n = 16384, with fp32 MFMA it was 4.8e-7.)  A column passes from
//     wave w + 1 to wave w; every wave counts its completed steps in LDS and waits only for that neighbour,
//     before the Q half of its step (no barrier per step).  Q is added to memory once per workgroup.
// One Philox block yields eight 16-bit draws, one per member of the group, so the generator's integer
// work is shared by up to 8 members.
//
// What bounds it: the vector instructions of a tile (generator, splitting, conversions), with two waves per SIMD at 256
// registers each; the additions of P to memory cost another 16 % (measured by leaving them out).  Against the kernel with
// fp32 MFMA, one launch for all slices, any delta > 0: n = 16384, 4 slices, 8 members, rank 16: 7.05 -> 6.40 ms; n = 2160,
// 20 slices, 8 members, rank 24: 1342 -> 1127 us; n = 2048, 8 slices, 6 members, rank 64: 674 -> 511 us.
// Measured and left out: a head x1 = that of X, common to the members, with each member's distance from it in two terms
// (6.13 ms at n = 16384, but a product was off by up to 2^-20.3 at delta = 0.03 and 2^-19.3 at 1/16); one Philox block shared
// by a pair of waves through LDS (6.8 ... 7.2 ms: the pair waits for each other), a wave that generates beside one that
// multiplies (7.1 ms), 16 waves per workgroup with half the registers each (6.6 ... 6.9 ms); these three with the common head.
#include "bf16split.h"
#include "dense_reads.h"
#include "kernels.h"

namespace nnr {
// Issue priority of a wave by the phase of its step (s_setprio; it only orders the waves of a SIMD, not streams):
// lowest in the long vector-only generator phase, higher once the matrix products start, highest from the tile
// transposition to the end of the step.  The wave that is nearer to handing its tile column on goes first; measured at
// n = 16384 (4 slices, 8 members): equal priorities 4 % slower, the opposite order 3 %.
constexpr int kPrioGenerator = 0, kPrioPProducts = 1, kPrioRest = 2;

constexpr int kWaves = 8;
constexpr int kPanel = 16 * kWaves;

// Operand-order copy of the factor, A_op[entity / 16][member][column block][half][lane] (16 bytes each): the two right
// operands of a lane (bf16split.h) for the values
//   A_int[16 * (entity / 16) + 4 * (lane / 16) + r][member][16 * block + lane % 16], r = 0..3.
// Rows at or beyond n_rows (the source may end there) read as zero.
__global__ void pack_operand_kernel(const float* __restrict__ A_int, uintx4* __restrict__ A_op, int64_t n_pad, int q,
                                    int kp, int64_t n_rows) {
  const int nt = kp / 16;
  const int64_t total = n_pad * q * kp / 4;   // lanes of all operands
  for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
       idx += (int64_t)gridDim.x * blockDim.x) {
    const int lane = (int)(idx & 63);
    int64_t rest = idx >> 6;
    const int b = (int)(rest % nt);
    const int64_t op = rest;
    rest /= nt;
    const int mem = (int)(rest % q);
    const int64_t tile = rest / q;
    const int64_t i = tile * 16 + 4 * (lane >> 4);
    const int64_t rs = (int64_t)q * kp;
    const float* src = A_int + (i * q + mem) * kp + b * 16 + (lane & 15);
    const float v[4] = {i + 0 < n_rows ? src[0] : 0.0f, i + 1 < n_rows ? src[rs] : 0.0f,
                        i + 2 < n_rows ? src[2 * rs] : 0.0f, i + 3 < n_rows ? src[3 * rs] : 0.0f};
    store_terms(A_op + op * 128 + lane, operand_terms(v));
  }
}

hipError_t launch_pack_operand(const float* A_int, float* A_op, const Dims& d, hipStream_t s, int64_t n_rows) {
  const int64_t total = d.n_pad * d.q * d.kp / 4;
  int64_t blocks = ceil_div(total, 256);
  if (blocks > 16384) blocks = 16384;
  hipLaunchKernelGGL(pack_operand_kernel, dim3((unsigned)blocks), dim3(256), 0, s, A_int, (uintx4*)A_op, d.n_pad, d.q, d.kp,
                     n_rows < 0 ? d.n_pad : n_rows);
  return hipGetLastError();
}

// A tile of X in "row" orientation is ONE 16-byte buffer load per lane on every path (dense_reads.h: rows need no more
// than the 4-byte alignment of a float, what lies beyond the tensor's end reads as zero), so that the number of loads in
// flight is known wherever one of them is waited for.  take_tile puts zeros in the places of other rows and columns.
__device__ __forceinline__ floatx4 take_tile(floatx4 x, int rows_left, int cols_left) {
  // rows_left, cols_left: elements of the matrix from this lane's first one on
  const bool in = rows_left > 0;
  return floatx4{in && cols_left > 0 ? x.x : 0.0f, in && cols_left > 1 ? x.y : 0.0f, in && cols_left > 2 ? x.z : 0.0f,
                 in && cols_left > 3 ? x.w : 0.0f};
}

// The 16-bit halves [hoff, hoff + QB) of a Philox block moved to its front, so that the members of a group index the
// block with compile-time constants (hoff is wave-uniform and a multiple of QB; QB divides 8).
template <int QB>
__device__ __forceinline__ u32x4 front_halves(u32x4 w, int hoff) {
  if constexpr (QB == 4) {
    const bool hi = (hoff & 4) != 0;
    w.x = hi ? w.z : w.x;
    w.y = hi ? w.w : w.y;
  } else if constexpr (QB < 4) {
    const uint32_t a = (hoff & 2) ? w.y : w.x, b = (hoff & 2) ? w.w : w.z;
    w.x = (hoff & 4) ? b : a;
    if constexpr (QB == 1) w.x >>= 16 * (hoff & 1);
  }
  return w;
}

// Dynamic LDS layout (floats):
//   [0, W*NG*256)          panel-wide Q accumulator in MFMA accumulator order: qlds[tile][group][lane][4]
//   then per wave          transposition tiles of bf16 terms: 64 pieces of 8 bytes per term, d1 and d2 of every member
//                          (of X itself where nothing is perturbed), then the heads x1
//   then W ints            completed steps per wave
// With 8 members and 8 waves all of it is 32 bytes more than the 160 KB of a compute unit: the last member's head then
// has no place of its own and takes the first one's, once that has been read back.
template <int NT, int QB, bool PERTURB, int W>
struct StreamShape {
  static constexpr int NG = QB * NT;                            // product groups (member, 16-column block)
  static constexpr int NSPLIT = PERTURB ? QB : 1;               // values per element that are split into terms
  static constexpr int QLDS = W * NG * 256;                     // floats of the Q accumulator
  static constexpr int lds_floats(int heads) { return QLDS + W * (NSPLIT * 256 + heads * 128) + W; }
  static constexpr bool LATE = lds_floats(NSPLIT) * (int)sizeof(float) > 160 * 1024;
  static constexpr int NHEAD = LATE ? NSPLIT - 1 : NSPLIT;      // places for heads
  static constexpr int TBUF = NSPLIT * 256 + NHEAD * 128;       // floats of transposition space per wave
  static constexpr size_t bytes = (size_t)lds_floats(NHEAD) * sizeof(float);
};

// four 16-bit values of one column of a row-major LDS tile (the 16 lanes of a group each address four of a row)
__device__ __forceinline__ uintx2 read_transposed(const void* lds_ptr) {
  typedef short s4 __attribute__((ext_vector_type(4)));
  return __builtin_bit_cast(uintx2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                                        (__attribute__((address_space(3))) s4*)(__attribute__((address_space(3))) void*)lds_ptr));
}

template <int NT, int QB, bool PERTURB, int W>
__global__ void __launch_bounds__(W * 64, 2)
    dense_stream_kernel(const float* __restrict__ X, const uintx4* __restrict__ A_op, float* __restrict__ P,
                        float* __restrict__ Q, int64_t n, int m, int q, int k, int qfirst, int ngroups, int n_chunks,
                        int64_t rows_per_chunk, uint32_t k0, uint32_t k1, float dscaled, int t_first,
                        const uintx4* __restrict__ A_opQ, int64_t aop_tstride, int64_t out_tstride,
                        int32_t* __restrict__ timeout_flag, int spin_limit, float* __restrict__ Ppart,
                        int64_t ppart_stride) {
  typedef StreamShape<NT, QB, PERTURB, W> Shape;
  constexpr int NG = Shape::NG, NSPLIT = Shape::NSPLIT;
  extern __shared__ __attribute__((aligned(16))) float lds[];
  float* qlds = lds;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, row = lane >> 4;
  char* tbuf = reinterpret_cast<char*>(lds + Shape::QLDS + wave * Shape::TBUF);
  // done[w]: number of steps wave w has completed (see the hand-over of the tile columns below)
  int* done = reinterpret_cast<int*>(lds + Shape::QLDS + W * Shape::TBUF);
  if (lane == 0) done[wave] = 0;

  // Workgroups are handed to the 8 XCDs round-robin; give each XCD a contiguous range of logical indices.  Member group
  // and slice run fastest: the workgroups that an XCD runs at a time then work on few panels of several slices, whose
  // operands (the same factor rows) they share in that XCD's L2, and no two of them add to the same rows of P.
  int64_t logical;
  {
    const int64_t total = gridDim.x, L = blockIdx.x;
    const int64_t base = total >> 3, rem = total & 7, xcd = L & 7, slot = L >> 3;
    logical = xcd * base + (xcd < rem ? xcd : rem) + slot;
  }
  const int grp = (int)(logical % ngroups);
  const int t = (int)((logical / ngroups) % m);
  const int64_t z = logical / ((int64_t)ngroups * m);
  const int chunk = (int)(z % n_chunks), panel = (int)(z / n_chunks);
  // Members [q0, q0 + QB) share one Philox block (QB divides 8 and q0 is a multiple of QB).  Slots at or
  // beyond q (a rounded-up tail group) are computed on whatever the spare operand slots hold and never written.
  const int q0 = qfirst + grp * QB;
  const int qb = (q - q0) < QB ? (q - q0) : QB;
  const uint32_t sub = (uint32_t)(q0 >> 3);         // Philox block index of this member group
  const int hoff = QB == 8 ? 0 : (q0 & 7);          // first 16-bit half used by the group
  const int64_t jp0 = (int64_t)panel * (16 * W);
  const int64_t i_begin = (int64_t)chunk * rows_per_chunk;
  int64_t i_end = i_begin + rows_per_chunk;
  if (i_end > n) i_end = n;
  // Reproducible mode (Ppart given): the panel's sums for X_t A are stored in the panel's own copy, and, the chunk
  // being the whole slice then, X_t^T A is stored by its only writer; nothing is added atomically.
  const bool ordered = Ppart != nullptr;
  float* Pt = ordered ? Ppart + (int64_t)panel * ppart_stride + (int64_t)t * out_tstride : P + (int64_t)t * out_tstride;
  float* Qt = Q + (int64_t)t * out_tstride;
  int tiles = (int)((n - jp0 + 15) >> 4);           // tiles of the panel that hold columns of the matrix
  if (tiles > W) tiles = W;
  const int cols = (int)(n - jp0 < 16 * W ? n - jp0 : 16 * W);   // columns of the panel

  for (int e = tid; e < Shape::QLDS; e += W * 64) qlds[e] = 0.0f;
  __syncthreads();

  // Operand address of (tile of 16 entities, product group g), in units of 16 bytes: a wave-uniform part
  // (tile, first member, g) plus the lane.
  // The two products may take their right operands from different arrays, and from a different one per slice
  // (aop_tstride units apart): the iteration itself passes the same A for both and every slice.
  const int64_t tile_u4 = (int64_t)q * NT * 128;    // units per 16-entity tile
  const uintx4* Ag = A_opQ + (int64_t)t * aop_tstride + (int64_t)q0 * NT * 128;
  const uintx4* Ap = A_op + (int64_t)t * aop_tstride + (int64_t)q0 * NT * 128 +
                     (jp0 >> 4) * tile_u4;          // operands of the panel's column tiles, first group of this member group

  // A round = W strips of 16 rows, one per wave; in step s of a round wave w works on tile (w + s) % W of
  // its strip, so at any step every tile column of the Q accumulator belongs to one wave.  A column passes from
  // wave w + 1 to wave w; instead of a barrier per step each wave counts its completed steps in LDS and waits
  // only for the one wave it takes its column from.
  const int nstrips = (int)((i_end - i_begin + 15) >> 4);
  const int nrounds = (nstrips + W - 1) / W;
  auto tile_of = [&](int s) { return (wave + s) & (W - 1); };
  // first row of this wave's strip in round rnd (a wave without a strip, or past the last round, reads the
  // chunk's first strip: valid memory, never used)
  auto strip_of = [&](int rnd) -> int { return rnd * W + wave; };
  auto strip_row = [&](int rnd) -> int64_t {
    const int strip = rnd < nrounds ? strip_of(rnd) : nstrips;
    return i_begin + 16 * (int64_t)(strip < nstrips ? strip : 0);
  };
  // X tile of a strip (first row i0) and a tile column; the loads run two steps ahead, across strip boundaries.  A
  // tile beyond the matrix, or rows beyond the chunk: whatever is there is loaded and never used.
  const int64_t total = (int64_t)m * n * n;
  const uint32_t x_lane = tile_lane_offset((uint32_t)n, l16, row);
  auto x_fetch = [&](int64_t i0, int jt) -> floatx4 {
    const TileBuffer b = tile_buffer(n, total, t, i0, jp0);   // wave-uniform
    const __amdgpu_buffer_rsrc_t rsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(X + b.first), 0, (int)b.bytes, 0x00020000);
    return __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)tile_voffset(x_lane, jt), 0, 0));
  };
  uintx8 bP[NG], bq[NG];
  auto bp_fetch = [&](int jt) {
    const uintx4* a = Ap + jt * (int)tile_u4;       // rows < n_pad: always valid
#pragma unroll
    for (int g = 0; g < NG; ++g) bP[g] = load_terms(a + g * 128 + lane);
  };
  // right operands of the Q products: the strip's 16 rows of A
  auto bq_fetch = [&](int rnd) {
    const int64_t i0 = strip_row(rnd);
#pragma unroll
    for (int g = 0; g < NG; ++g) bq[g] = load_terms(Ag + (i0 >> 4) * tile_u4 + g * 128 + lane);
  };
  floatx4 xeven = x_fetch(strip_row(0), tile_of(0)), xodd = x_fetch(strip_row(0), tile_of(1));
  bp_fetch(tile_of(0));
  bq_fetch(0);
  // Hand-over of the tile columns: wave w may touch the column of its step g once wave w + 1 has completed g steps
  // (it had that column in step g - 1).  EVERY wave waits like this in every step before its own count moves, so
  // that a count of g + 1 implies counts of at least g, g - 1, ... down the chain.  (Every wave makes the same
  // number of steps and a wait only concerns an earlier step of a wave that is resident on the same CU, so the
  // waits always end, after microseconds.)  The spin count is bounded all the same (spin_limit polls; the launcher
  // passes 2^20, about 30 ms, far more than the time a neighbour can be held back at the generator's low issue
  // priority).  A wait that runs out is an error, never a silent fall-through: the wave reports it in *timeout_flag
  // (one plain store by lane 0), leaves the Q half of that step out (the column may still be its neighbour's) and
  // goes on counting, so that the kernel exits normally; the host turns the flag into an error status.
  auto wait_for_neighbour = [&](int gstep) -> bool {
    const int nb = (wave + 1) & (W - 1);
    bool arrived = false;
    for (int spin = 0; spin < spin_limit; ++spin) {
      const int c = __builtin_amdgcn_readfirstlane(
          __hip_atomic_load(&done[nb], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
      if (c >= gstep) {
        arrived = true;
        break;
      }
      __builtin_amdgcn_s_sleep(1);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    if (!arrived && lane == 0 && timeout_flag)
      __hip_atomic_store(timeout_flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    return arrived;
  };
  // Transposition tiles: the lane's piece (row l16, columns 4*row ..) sits at position 4*l16 + (row ^ l16/4), so that
  // neighbouring lanes' stores fall on different banks; read back, lane L of a group of 16 addresses row
  // 4*group + L/4 and columns 4*(L%4) .., and gets rows 4*group .. of column L.
  const int put = 4 * l16 + (row ^ (l16 >> 2));
  const int get = 4 * (4 * row + (l16 >> 2)) + ((l16 & 3) ^ row);
  char* const rest_put = tbuf + 8 * put;
  char* const rest_get = tbuf + 8 * get;
  char* const head_put = tbuf + NSPLIT * 1024 + 8 * put;
  char* const head_get = tbuf + NSPLIT * 1024 + 8 * get;
  const float pa = 2.0f * dscaled, pc = __fmaf_rn(-65535.0f, dscaled, 1.0f);   // as in perturbed()

  for (int rnd = 0; rnd < nrounds; ++rnd) {
    const int strip = strip_of(rnd);
    const bool have_strip = strip < nstrips;        // wave-uniform
    const int64_t i0 = strip_row(rnd), i0_next = strip_row(rnd + 1);
    const int rows_left = (int)(i_end - i0 < 16 ? i_end - i0 : 16);
    floatx4 pacc[NG];
#pragma unroll
    for (int g = 0; g < NG; ++g) pacc[g] = floatx4{0.f, 0.f, 0.f, 0.f};

    // one step; x: its tile of X, in place of which the tile of step s + 2 is requested
    auto step = [&](const int s, floatx4& x) {
      const int jt = tile_of(s);
      const bool work = have_strip && jt < tiles;   // wave-uniform
      floatx4 xc = x;
      uintx2 late_head = {0u, 0u};                  // the last member's head where it has no place in LDS yet
      x = x_fetch(s + 2 < W ? i0 : i0_next, tile_of(s + 2));
      if (work) {
        if (rows_left < 16 || 16 * jt + 16 > cols) {          // wave-uniform
          xc = take_tile(xc, rows_left - l16, cols - (16 * jt + 4 * row));
        }
        const float xcur[4] = {xc.x, xc.y, xc.z, xc.w};
        // ---- the generator: one Philox block per element serves all QB members
        __builtin_amdgcn_s_setprio(kPrioGenerator);
        u32x4 w[4];
        if (PERTURB) {
          const uint64_t e0 = (uint64_t)(i0 + l16) * (uint64_t)n + (uint64_t)(jp0 + 16 * jt + 4 * row);
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const uint64_t e = e0 + (uint64_t)r;
            w[r] = front_halves<QB>(
                philox4x32_10((uint32_t)e, (uint32_t)(e >> 32), (uint32_t)(t + t_first), sub, k0, k1), hoff);
          }
        }
        // ---- per member: the terms of the perturbed tile in "row" orientation -> P products; park them in LDS for
        //      the transpose
        __builtin_amdgcn_s_setprio(kPrioPProducts);
        float xa[4], xc1[4];                        // a member's element: xa * half + xc1, as in perturbed()
        uintx2 x1, d1, d2;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          xa[r] = __fmul_rn(xcur[r], pa);
          xc1[r] = __fmul_rn(xcur[r], pc);
        }
        if (!PERTURB) {
          split3(xcur, x1, d1, d2);
          *reinterpret_cast<uintx2*>(head_put) = x1;
          *reinterpret_cast<uintx2*>(rest_put) = d1;
          *reinterpret_cast<uintx2*>(rest_put + 512) = d2;
        }
        constexpr int PB = QB > 1 ? 2 : 1;          // members whose products are interleaved: a product's three
#pragma unroll                                      // instructions wait for each other's sums
        for (int q2 = 0; q2 < QB; q2 += PB) {
          uintx2 e1[PB], e2[PB], h1[PB];
#pragma unroll
          for (int u = 0; u < PB; ++u) {
            const int qq = q2 + u;
            if (PERTURB) {
              float v[4];
#pragma unroll
              for (int r = 0; r < 4; ++r) {
                const uint32_t word = (qq >> 1) == 0 ? w[r].x : (qq >> 1) == 1 ? w[r].y : (qq >> 1) == 2 ? w[r].z : w[r].w;
                v[r] = __fmaf_rn(xa[r], (qq & 1) ? (float)(word >> 16) : (float)(word & 0xFFFFu), xc1[r]);
              }
              split3(v, x1, d1, d2);
              if (qq < Shape::NHEAD) *reinterpret_cast<uintx2*>(head_put + 512 * qq) = x1;
              else late_head = x1;
              *reinterpret_cast<uintx2*>(rest_put + 1024 * qq) = d1;
              *reinterpret_cast<uintx2*>(rest_put + 1024 * qq + 512) = d2;
            }
            h1[u] = x1;
            e1[u] = d1;
            e2[u] = d2;
          }
#pragma unroll
          for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int i = 0; i < 3; ++i)
#pragma unroll
              for (int u = 0; u < PB; ++u) {
                const int g = (q2 + u) * NT + nt;
                pacc[g] = mfma_terms(i, h1[u], e1[u], e2[u], bP[g], pacc[g]);
              }
        }
      }
      __builtin_amdgcn_s_setprio(kPrioRest);
      // the operand registers are free again: fetch the next tile's
      bp_fetch(tile_of((s + 1) & (W - 1)));
      if (work) {
        // ---- "column" orientation read back from LDS: lane (l16, row) gets the terms of rows i0 + 4*row + r of column
        //      j0 + l16; the tile's Q accumulators are this wave's alone until its step count moves
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        // Tile column jt was wave (wave + 1) % W's in the previous step: wait until that wave has completed it.
        const bool mine = wait_for_neighbour(rnd * W + s);   // wave-uniform
        float4* qt = reinterpret_cast<float4*>(qlds) + (jt * NG) * 64 + lane;
        // QH members at a time: all LDS reads first (one wait), then the products back to back, then the stores (with all
        // 8 groups at a time the registers run out; halves spill 10 and are 3 % slower than quarters at n = 16384)
        constexpr int QH = NG < 8 || QB == 1 ? QB : (QB > 2 ? QB / 4 : 1);
#pragma unroll
        for (int q1 = 0; q1 < QB; q1 += QH) {
          uintx2 x1t[QH], d1t[QH], d2t[QH];
          floatx4 qa[QH * NT];
          float4 c[QH * NT];
#pragma unroll
          for (int h = 0; h < QH; ++h) {
            const int v = NSPLIT > 1 ? q1 + h : 0;   // (nothing perturbed: the terms of X serve every member)
            x1t[h] = read_transposed(head_get + 512 * (v < Shape::NHEAD ? v : 0));
            d1t[h] = read_transposed(rest_get + 1024 * v);
            d2t[h] = read_transposed(rest_get + 1024 * v + 512);
          }
          if (Shape::LATE && q1 == 0) {             // (a wave's LDS accesses are carried out in order)
            static_assert(!Shape::LATE || QH < QB, "the first head has been read before the last one takes its place");
            *reinterpret_cast<uintx2*>(head_put) = late_head;
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
          }
#pragma unroll
          for (int g = 0; g < QH * NT; ++g) {
            c[g] = qt[(q1 * NT + g) * 64];
            qa[g] = floatx4{0.f, 0.f, 0.f, 0.f};
          }
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int g = 0; g < QH * NT; ++g) {
              const int h = g / NT;
              qa[g] = mfma_terms(i, x1t[h], d1t[h], d2t[h], bq[q1 * NT + g], qa[g]);
            }
          __builtin_amdgcn_sched_barrier(0);
          if (mine) {
#pragma unroll
            for (int g = 0; g < QH * NT; ++g)
              qt[(q1 * NT + g) * 64] = float4{c[g].x + qa[g][0], c[g].y + qa[g][1], c[g].z + qa[g][2], c[g].w + qa[g][3]};
          }
        }
      } else {
        // A wave with nothing to do in this step (no strip in the chunk's last round, or a tile beyond the matrix)
        // still is a link of the chain: its count may move only after its neighbour's, or the wave behind it
        // could take the column over while the wave in front is still working on it.
        (void)wait_for_neighbour(rnd * W + s);
      }
      // the strip's last Q products are done: fetch the next strip's operands behind them
      if (s == W - 1 && rnd + 1 < nrounds) bq_fetch(rnd + 1);
      // hand the tile column on: the accumulators are in LDS before the count moves
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
      if (lane == 0)
        __hip_atomic_store(&done[wave], rnd * W + s + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
#pragma unroll 1
    for (int s = 0; s < W; s += 2) {           // (two steps per trip: the two tiles in flight keep their registers)
      step(s, xeven);
      step(s + 1, xodd);
    }
    // ---- the strip's P (16 rows, summed over the panel's columns): add to memory.  The groups of a row are neighbours
    //      (kp = 16 NT): one 32-bit offset per register r, the group in the instruction's immediate offset.
    if (have_strip) {
      char* prow = reinterpret_cast<char*>(Pt + (i0 * q + q0) * (16 * NT));   // wave-uniform
      int ln = lane;
      asm volatile("" : "+v"(ln));                  // (keeps the offsets from being computed ahead of the loop and held there)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int rr = 4 * (ln >> 4) + r;
        if (rr >= rows_left) continue;
        const uint32_t off = (uint32_t)(rr * q * (16 * NT) + (ln & 15)) * 4u;
#pragma unroll
        for (int g = 0; g < NG; ++g) {
          float* at = reinterpret_cast<float*>(prow + off + 64 * g);
          if (g / NT >= qb) break;
          if (ordered) *at = pacc[g][r];
          else if ((g % NT) * 16 + (ln & 15) < k) unsafeAtomicAdd(at, pacc[g][r]);
        }
      }
    }
  }
  __syncthreads();
  // ---- the panel's Q (summed over the chunk's rows): add to memory (every wave has made its last step)
  constexpr int kp = 16 * NT;
  for (int e = tid; e < tiles * NG * 256; e += W * 64) {
    const float v = qlds[e];
    const int r = e & 3, ln = (e >> 2) & 63, g = (e >> 8) % NG, jt = (e >> 8) / NG;
    const int qq = g / NT, nt = g % NT;
    const int64_t j = jp0 + 16 * jt + 4 * (ln >> 4) + r;
    if (ordered) {
      if (qq < qb && j < n) Qt[(j * q + q0 + qq) * kp + nt * 16 + (ln & 15)] = v;
    } else if (qq < qb && j < n && v != 0.0f) {
      unsafeAtomicAdd(&Qt[(j * q + q0 + qq) * kp + nt * 16 + (ln & 15)], v);
    }
  }
}

const char* dense_stream_kernel_name() { return "dense_stream_kernel"; }

template <int NT, int QB, bool PERTURB, int W>
static hipError_t launch_stream_t(const float* X, const float* A_op, float* P, float* Q, const Dims& d, int qfirst,
                                  const StreamPart& part, uint64_t seed, float delta, hipStream_t s, const DenseStreamOpts& o) {
  const int ngroups = part.groups;
  const int t_first = o.t_first;
  const float* A_opQ = o.A_opQ ? o.A_opQ : A_op;
  const int64_t out_tstride = o.out_tstride < 0 ? d.n * d.q * (int64_t)d.kp : o.out_tstride;
  int32_t* timeout_flag = o.timeout_flag;
  const int spin_limit = o.spin_limit > 0 ? o.spin_limit : (o.spin_limit < 0 ? 0 : (1 << 20));
  float* Ppart = o.Ppart;
  const int64_t ppart_stride = (int64_t)d.m * d.n * d.q * d.kp;   // one copy of P per panel
  if (Ppart && out_tstride != d.n * d.q * (int64_t)d.kp) return hipErrorInvalidValue;   // (not with summed slices)
  static_assert(QB * NT <= 8, "at most 8 product groups per tile");
  constexpr size_t lds = StreamShape<NT, QB, PERTURB, W>::bytes;
  static_assert(lds <= 160 * 1024, "LDS budget of one CU");
  static bool attr_done = false;
  if (!attr_done) {
    hipError_t e = hipFuncSetAttribute((const void*)dense_stream_kernel<NT, QB, PERTURB, W>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    attr_done = true;
  }
  // (a whole number of rounds of W strips; reproducible mode: one workgroup per panel and slice, the only writer of its X_t^T A)
  const int64_t n_panels = ceil_div(d.n, 16 * W);
  const int64_t rows_per_chunk = round_up(ceil_div(d.n, Ppart ? 1 : part.chunks), 16 * W);
  const int64_t n_chunks = ceil_div(d.n, rows_per_chunk);
  const int64_t total = n_panels * n_chunks * d.m * ngroups;
  if (total > 0x7FFFFFFFLL) return hipErrorInvalidValue;
  hipLaunchKernelGGL((dense_stream_kernel<NT, QB, PERTURB, W>), dim3((unsigned)total), dim3(W * 64), lds, s, X,
                     (const uintx4*)A_op, P, Q, d.n, d.m, d.q, d.k, qfirst, ngroups, (int)n_chunks, rows_per_chunk,
                     (uint32_t)seed, (uint32_t)(seed >> 32), delta * 0x1p-16f, t_first, (const uintx4*)A_opQ,
                     o.aop_tstride / 4, out_tstride, timeout_flag, spin_limit, Ppart, ppart_stride);
  return hipGetLastError();
}

// Members per group so that (members) x (16-column blocks) <= 8 product groups: 8 members for k <= 16,
// 4 for k <= 32, 2 for k <= 64.
static int group_members(int kp) { return kp <= 16 ? 8 : (kp <= 32 ? 4 : 2); }

int64_t dense_stream_panels(const Dims& d) { return ceil_div(d.n, kPanel); }

// How a pass is cut into workgroups.  A launch takes its members in groups (the members of a group share the generator) on
// panels of 16 W columns and chunks of rows.  Large groups generate least; many, small and short workgroups fill the 256
// compute units and even out the last ones; few chunks add to Q least, wide panels to P.  The plan is the one of the least
//   us = (1.25 ceil(B / C) - 0.25 max(1, B / C)) (rows (38 + 9 g + 8.5 g nt) ns + 1.3 g nt) + 0.3 / 10^6 additions to P + 1.25 / 10^6
//        to Q,
// B workgroups, C = 256 of them at a time (512 with 4 waves, whose rows take 5 % longer), g members of nt = kp / 16 column
// blocks each.  g nt <= 2 leaves room for a second workgroup on a compute unit: without one (B <= C) the rows take 20 % longer.
// A second launch costs 20 us more.  Fitted to 18560 timed launches (n = 100 ... 8000, 1 ... 20 slices, 1 ... 20 members, ranks
// 5 ... 64, delta = 0.03, every form with up to 10 chunk counts) so that what it picks is fast, not to match the times: it takes
// 0.95 % longer than the best one in the mean, 3 % at the ninetieth percentile, 11 % at the ninety-ninth, 19 % at worst.  At
// delta = 0, where there is no generator and X is split once, 10 + 2 g takes the place of 38 + 9 g (4600 launches up to n = 4100:
// 2 %, 8 %, 15 %, 20 %).
// n / slices / members, rank: fp32 MFMA, the rule of size classes that stood here before, this plan (us for a pass):
//   2000 / 4 / 1, 16    44.1   69.3   42.3        1000 / 4 / 7, 24    102    77.7   73.3
//   2000 / 4 / 2, 16    55.8   80.4   57.7        1000 / 4 / 13, 64   268    223    177
//   2000 / 4 / 5, 16    136    130    114         2000 / 4 / 15, 24   496    439    354
//   2000 / 4 / 13, 16   298    245    207         2000 / 4 / 5, 64    335    283    258
// Over 1051 sizes (15 shapes up to n = 8000, ranks 5 ... 64, 1 ... 20 members) this plan takes 0.95 of that rule's time in the mean,
// 1.09 at worst, and 1.03 of fp32 MFMA's at worst (that rule: 1.57, with one or two members in groups of 4).
static StreamPart stream_part(const Dims& d, int count, int waves, int members, bool perturb, bool ordered) {
  StreamPart best{waves, members, (int)ceil_div(count, members), 1, 0.0};
  const int nt = d.kp / 16, side = 16 * waves, width = members * nt;
  const int64_t panels = ceil_div(d.n, side), most = ordered ? 1 : (panels < 256 ? panels : 256);
  const double row_us = ((perturb ? 38.0 + 9.0 * members : 10.0 + 2.0 * members) + 8.5 * width) * (waves == 4 ? 1.05e-3 : 1e-3);
  const double results = (double)d.m * d.n * count * d.k * 1e-6;   // values of P, and of Q, in millions
  int64_t seen = 0;
  for (int64_t c = 1; c <= most; ++c) {
    const int64_t rows = round_up(ceil_div(d.n, c), side), chunks = ceil_div(d.n, rows);
    if (chunks == seen) continue;                   // (the same cut again)
    seen = chunks;
    const int64_t blocks = panels * d.m * best.groups * chunks, at_once = waves == 4 ? 512 : 256;
    const double rounds = 1.25 * ceil_div(blocks, at_once) - 0.25 * (blocks > at_once ? (double)blocks / at_once : 1.0);
    const double alone = blocks <= at_once && width <= 2 ? 1.2 : 1.0;
    const double us = rounds * ((rows < d.n ? rows : d.n) * row_us * alone + 1.3 * width) +
                      (ordered ? 0.0 : results * (0.3 * panels + 1.25 * chunks));
    if (c == 1 || us < best.us) {
      best.chunks = chunks;
      best.us = us;
    }
  }
  return best;
}

// ordered: the reproducible mode (8 waves, one chunk: its copies of P are one per 128 columns, nothing is added)
DensePlan dense_stream_plan(const Dims& d, bool perturb, bool ordered) {
  const int big = group_members(d.kp), nt = d.kp / 16, tail = d.q % big;
  DensePlan best{};
  double best_us = -1.0;
  for (int waves = ordered ? kWaves : 4; waves <= kWaves; waves *= 2)
    for (int g = 1; g <= big && g < 2 * d.q; g *= 2) {
      if (waves == 4 && g * nt > (nt > 2 ? nt : 2)) continue;   // (kernels that are not built)
      const StreamPart p = stream_part(d, d.q, waves, g, perturb, ordered);
      if (best_us < 0.0 || p.us < best_us) {
        best_us = p.us;
        best = d.q >= big ? DensePlan{d.q, 0, {p, {}}} : DensePlan{0, d.q, {{}, p}};
      }
    }
  if (d.q > big && tail) {                          // the whole groups, and the rest in a group of its own
    int g = 1;
    while (g < tail) g *= 2;
    const StreamPart whole = stream_part(d, d.q - tail, kWaves, big, perturb, ordered);
    const StreamPart rest = stream_part(d, tail, kWaves, g, perturb, ordered);
    if (whole.us + rest.us + 20.0 < best_us) best = DensePlan{d.q - tail, tail, {whole, rest}};
  }
  return best;
}

template <int NT, int QB, int W>
static hipError_t launch_stream_qb(const float* X, const float* A_op, float* P, float* Q, const Dims& d, int qf,
                                   const StreamPart& part, uint64_t seed, float delta, hipStream_t s, const DenseStreamOpts& o) {
  if constexpr (QB * NT <= 8 && (W == kWaves || QB * NT <= (NT > 2 ? NT : 2)))
    return delta == 0.0f ? launch_stream_t<NT, QB, false, W>(X, A_op, P, Q, d, qf, part, seed, delta, s, o)
                         : launch_stream_t<NT, QB, true, W>(X, A_op, P, Q, d, qf, part, seed, delta, s, o);
  return hipErrorInvalidValue;
}

template <int NT>
static hipError_t launch_stream_nt(const float* X, const float* A_op, float* P, float* Q, const Dims& d, int qf,
                                   const StreamPart& part, uint64_t seed, float delta, hipStream_t s, const DenseStreamOpts& o) {
  if (part.waves == 4)
    return part.members == 1 ? launch_stream_qb<NT, 1, 4>(X, A_op, P, Q, d, qf, part, seed, delta, s, o)
                             : launch_stream_qb<NT, 2, 4>(X, A_op, P, Q, d, qf, part, seed, delta, s, o);
  switch (part.members) {
    case 1: return launch_stream_qb<NT, 1, kWaves>(X, A_op, P, Q, d, qf, part, seed, delta, s, o);
    case 2: return launch_stream_qb<NT, 2, kWaves>(X, A_op, P, Q, d, qf, part, seed, delta, s, o);
    case 4: return launch_stream_qb<NT, 4, kWaves>(X, A_op, P, Q, d, qf, part, seed, delta, s, o);
    case 8: return launch_stream_qb<NT, 8, kWaves>(X, A_op, P, Q, d, qf, part, seed, delta, s, o);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_dense_stream(const float* X, const float* A_op, float* P, float* Q, const Dims& d, const DensePlan& plan,
                               int part, uint64_t seed, float delta, hipStream_t s, const DenseStreamOpts& o) {
  const int qf = part == 0 ? 0 : plan.full_members;
  const StreamPart& sp = plan.part[part];
  if (sp.groups == 0) return hipSuccess;
  if (o.Ppart && sp.waves != kWaves) return hipErrorInvalidValue;   // (a plan for the other mode)
  switch (d.kp / 16) {
    case 1: return launch_stream_nt<1>(X, A_op, P, Q, d, qf, sp, seed, delta, s, o);
    case 2: return launch_stream_nt<2>(X, A_op, P, Q, d, qf, sp, seed, delta, s, o);
    case 3: return launch_stream_nt<3>(X, A_op, P, Q, d, qf, sp, seed, delta, s, o);
    case 4: return launch_stream_nt<4>(X, A_op, P, Q, d, qf, sp, seed, delta, s, o);
    default: return hipErrorInvalidValue;
  }
}

// ------------------------------------------------------------------------------------------ Alg. 4 made explicit
__global__ void dense_perturb_kernel(const float* __restrict__ X, float* __restrict__ out, int64_t n, int m,
                                     int member, uint32_t k0, uint32_t k1, float dscaled, int perturb) {
  const int64_t per = n * n;
  const int64_t total = per * m;
  for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
       idx += (int64_t)gridDim.x * blockDim.x) {
    const int t = (int)(idx / per);
    const uint64_t e = (uint64_t)(idx % per);
    float v = X[idx];
    if (perturb) {
      const u32x4 w = philox4x32_10((uint32_t)e, (uint32_t)(e >> 32), (uint32_t)t, (uint32_t)(member >> 3), k0, k1);
      v = perturbed(v, w, member & 7, dscaled);
    }
    out[idx] = v;
  }
}

hipError_t launch_dense_perturb(const float* X, float* out, int64_t n, int m, int member, uint64_t seed,
                                float delta, hipStream_t s) {
  int64_t blocks = ceil_div(n * n * m, 256);
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(dense_perturb_kernel, dim3((unsigned)blocks), dim3(256), 0, s, X, out, n, m, member,
                     (uint32_t)seed, (uint32_t)(seed >> 32), delta * 0x1p-16f, delta != 0.0f ? 1 : 0);
  return hipGetLastError();
}

// sum_t ||X^r_t||_F^2 for every member (the constant term of the expanded objective of Eq. 1)
__global__ void __launch_bounds__(256) dense_xnorm_kernel(const float* __restrict__ X, double* __restrict__ xn,
                                                          int64_t n, int m, int q, uint32_t k0, uint32_t k1,
                                                          float dscaled, int perturb, double* __restrict__ part) {
  __shared__ double red[4];
  const int64_t per = n * n;
  const int64_t total = per * m;
  for (int b = 0; b < (q + 7) / 8; ++b) {
    double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    const int qb = (q - 8 * b) < 8 ? (q - 8 * b) : 8;
    for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
         idx += (int64_t)gridDim.x * blockDim.x) {
      const int t = (int)(idx / per);
      const uint64_t e = (uint64_t)(idx % per);
      const float v = X[idx];
      u32x4 w{0, 0, 0, 0};
      if (perturb) w = philox4x32_10((uint32_t)e, (uint32_t)(e >> 32), (uint32_t)t, (uint32_t)b, k0, k1);
#pragma unroll
      for (int qq = 0; qq < 8; ++qq)
        if (qq < qb) {
          const float xq = perturb ? perturbed(v, w, qq, dscaled) : v;
          acc[qq] += (double)xq * (double)xq;
        }
    }
#pragma unroll
    for (int qq = 0; qq < 8; ++qq) {
      if (qq < qb) {  // block-uniform
        double v = acc[qq];
        for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
        __syncthreads();
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
        __syncthreads();
        if (threadIdx.x == 0) {
          const double sum = red[0] + red[1] + red[2] + red[3];
          if (part) part[(int64_t)blockIdx.x * q + 8 * b + qq] = sum;   // reproducible mode: block sums, added in order later
          else atomicAdd(&xn[8 * b + qq], sum);
        }
      }
    }
  }
}

hipError_t launch_dense_xnorm(const float* X, double* xn, int64_t n, int m, int q, uint64_t seed, float delta,
                              hipStream_t s, double* part) {
  int64_t blocks = ceil_div(n * n * m, 256 * 8);
  if (blocks > kXnormMaxBlocks) blocks = kXnormMaxBlocks;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(dense_xnorm_kernel, dim3((unsigned)blocks), dim3(256), 0, s, X, xn, n, m, q, (uint32_t)seed,
                     (uint32_t)(seed >> 32), delta * 0x1p-16f, delta != 0.0f ? 1 : 0, part);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess && part) e = launch_reduce_parts_f64(xn, part, q, blocks, q, 1, s);
  return e;
}

}  // namespace nnr
