// Work-tile functions of the compute actors' behaviours (gfx950).
//
// Each function processes one work tile of one message with a 256-thread
// workgroup (4 wave64s) and returns after its stores are issued; the caller
// synchronises the workgroup and accounts for the tile.
//
// Floating point: this file is compiled with -ffp-contract=off and the
// pragma below, so no multiply-add is fused and every operation is one
// IEEE round-to-nearest operation in the type written, in the order
// written -- the escape-time counts must match the CPU oracle bit for bit.
#pragma once
#pragma clang fp contract(off)

#include "caf_internal.h"

namespace cafgpu {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

__device__ inline uint32_t lane_id() { return threadIdx.x & 63u; }

// Global-memory (address space 1) views of the pointers a message carries.
// Accesses through them are global_* instructions, counted by the vector
// memory counter only; through generic pointers they would be flat_*
// instructions, which also count against the LDS counter, so every wait for
// an LDS read would also wait for the outstanding global prefetch.
#define CAF_GLOBAL __attribute__((address_space(1)))
template <typename T>
__device__ __forceinline__ CAF_GLOBAL T* global_ptr(T* p) {
  return (CAF_GLOBAL T*)p;
}
// LDS (address space 3) views, for the same reason: the matrix tiles are
// called from several kernels, and through a generic pointer their LDS
// accesses would be flat_* instructions too.
#define CAF_LDS __attribute__((address_space(3)))
typedef CAF_LDS uint8_t lds_u8;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4a2 __attribute__((ext_vector_type(4), aligned(2)));
// A 16-byte global load, returned as V (float4 or uint4).
template <typename V, typename T>
__device__ __forceinline__ V load_global(const CAF_GLOBAL T* p) {
  static_assert(sizeof(V) == 16, "16-byte loads");
  const u32x4 r = *reinterpret_cast<const CAF_GLOBAL u32x4*>(p);
  return __builtin_bit_cast(V, r);
}
__device__ inline uint32_t wave_id() { return threadIdx.x >> 6; }

// Reply data is stored past the L2 (a system-scope store writes through), so
// a completion needs no writeback of the L2: it waits for the workgroup's
// stores and writes its record.  A release fence writes back every dirty line
// of the XCD's L2, whoever wrote it, and holds up its other workgroups
// meanwhile; with replies left in the L2 each finished message paid one.
template <typename T>
__device__ __forceinline__ void store_reply(CAF_GLOBAL T* p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
template <typename T>
__device__ __forceinline__ void store_reply(T* p, T v) {
  store_reply(global_ptr(p), v);
}
// Waits until this wave's stores have reached memory.
__device__ __forceinline__ void wait_stores() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// ---------------------------------------------------------------------------
// Mandelbrot escape time (the paper's Mandelbrot workloads, Sec. 7.4 and
// Sec. 7.5; the recurrence is the textbook set definition, z_0 = 0,
// z <- z^2 + c, count = first k with |z_k|^2 > 4, else max_iter).
//
// A message covers global rows [row0, row0 + rows) of a width-wide image and
// replies uint16 counts, row-major [rows][width].  Its pixels are cut into
// 4 x 16 blocks (lane -> row lane/16, column lane%16: each row segment is a
// contiguous 32-byte store), numbered in groups of P blocks -- 8 x 32 pixels
// in float, 8 x 16 in double -- that a wave iterates together, and a work
// tile is tcfg/64 consecutive blocks.  A compact group holds pixels of
// similar escape times, so fewer of a wave's lanes idle while its slowest
// pixel finishes than in a 4 x 64 row of blocks.  The waves of the
// workgroup take groups of the tile from an LDS counter, so a slow group
// does not hold the others.  Every lane iterates its own pixels; the wave
// leaves the loop as soon as the ballot of lanes that have not escaped is
// empty -- the early exit is wave-uniform and no lane's count moves past
// its escape.
// ---------------------------------------------------------------------------
// Escape counts of P pixels per lane, interleaved, so each wave carries P
// independent dependency chains.  gfx950 issues two plain fp32 VALU
// instructions per SIMD in one quad cycle when two waves have one ready, so
// the loop is written to keep the vector units fed and the scalar unit (one
// per compute unit, shared by its four SIMDs) idle:
//  * a pixel that escapes is frozen by making its zr a quiet NaN: |z|^2 is
//    then NaN, which never passes the > 4 test again, and lanes outside the
//    tile start frozen (cr = NaN).  The per-iteration test therefore needs
//    no live-lane masking: it is one compare of the largest of the P
//    magnitudes against 4 -- the maximum ignores NaN operands and returns
//    one of the others exactly, so the test is exactly "some live pixel
//    escapes" -- and one branch on its result;
//  * the iteration limit is checked once per block of kEscapeUnroll
//    iterations; an escape seen at an iteration >= max_iter (the last block
//    may run past it) leaves the count at max_iter;
//  * counts, freezing and the check for a finished wave are selects on the
//    rare branch, which ends the loop at the end of the current block once
//    every pixel of the wave has escaped.
// Each iteration is the recurrence's 3 multiplies and 5 adds/subtracts per
// pixel, in the order the oracle takes them, and each pixel's test is
// decided by its own |z|^2 > 4.  valid[p] = false marks a lane's pixel p as
// outside the tile.
constexpr uint32_t kEscapeUnroll = 4;

// The larger of two magnitudes (v_max): IEEE maxNum, so a NaN operand (a
// frozen pixel) yields the other operand, and otherwise one of the two
// operands exactly.
__device__ __forceinline__ float max_of(float a, float b) { return __builtin_fmaxf(a, b); }
__device__ __forceinline__ double max_of(double a, double b) { return __builtin_fmax(a, b); }
template <typename T>
__device__ __forceinline__ T quiet_nan() {
  if constexpr (sizeof(T) == 4) return __builtin_nanf("");
  else return __builtin_nan("");
}

template <typename T, int P>
__device__ __forceinline__ void escape_count(const T (&cr_in)[P], const T (&ci_in)[P],
                                             const bool (&valid)[P], uint32_t max_iter,
                                             uint32_t (&n)[P]) {
  const uint32_t lim = __builtin_amdgcn_readfirstlane(max_iter);
  const T nan = quiet_nan<T>();
  T zr[P], zi[P], cr[P], ci[P];
  uint32_t left = 0;  // this lane's pixels still iterating
#pragma unroll
  for (int p = 0; p < P; ++p) {
    n[p] = lim;
    cr[p] = valid[p] ? cr_in[p] : nan;
    ci[p] = ci_in[p];
    zr[p] = T(0);
    zi[p] = T(0);
    left += valid[p] ? 1u : 0u;
  }
  if (lim == 0 || __builtin_amdgcn_ballot_w64(left != 0) == 0) return;
  uint32_t stop = lim;  // lowered on the rare branch once the wave is done
  for (uint32_t it = 0; it < stop; it += kEscapeUnroll) {
#pragma unroll
    for (uint32_t u = 0; u < kEscapeUnroll; ++u) {
      T m[P];
#pragma unroll
      for (int p = 0; p < P; ++p) {
        const T r2 = zr[p] * zr[p];
        const T i2 = zi[p] * zi[p];
        m[p] = r2 + i2;
        const T t = zr[p] * zi[p];
        const T tt = t + t;
        zi[p] = tt + ci[p];
        const T d = r2 - i2;
        zr[p] = d + cr[p];
      }
      T mx = m[0];
#pragma unroll
      for (int p = 1; p < P; ++p) mx = max_of(mx, m[p]);
      if (__builtin_expect(__builtin_amdgcn_ballot_w64(mx > T(4)) != 0, 0)) {
        asm volatile("" ::: "memory");
        const uint32_t k = it + u;
        const uint32_t kk = k < lim ? k : lim;
#pragma unroll
        for (int p = 0; p < P; ++p) {
          const bool e = m[p] > T(4);
          n[p] = e ? kk : n[p];
          zr[p] = e ? nan : zr[p];
          left -= e ? 1u : 0u;
        }
        if (__builtin_amdgcn_ballot_w64(left != 0) == 0) stop = 0;
      }
    }
  }
}

// Tiles tile .. tile + count - 1 of one message: their blocks form one
// range that the four waves share, so a claimed run of small tiles keeps
// every wave busy while the tiles stay small enough to even out the end of
// a batch.
//
// Issue priority: a SIMD issues from its oldest ready wave first, and the
// drain's workgroups live as long as the launch, so the waves of the
// workgroups dispatched last get only the leftover issue slots and their
// runs take several times longer than the others'.  Runs claimed early in a
// batch then finish last, on a nearly idle chip.  A wave therefore raises
// its priority as its run ages (after kPrioStepTicks of the 100 MHz wall
// clock, then twice and four times that) and drops back when the run ends,
// so runs finish closer to the order they were claimed in.
constexpr uint64_t kPrioStepTicks = 10000;  // 100 us

template <typename T>
__device__ void mandel_tile(const Desc& d, uint32_t tile, uint32_t count, uint32_t* lds_ctr) {
  // pixels per lane: four in float (the loop dual-issues), two in double
  constexpr int P = sizeof(T) == 4 ? 4 : 2;
  T re_min, im_min, step_re, step_im;
  if constexpr (sizeof(T) == 8) {
    re_min = d.p.m64.re_min;
    im_min = d.p.m64.im_min;
    step_re = d.p.m64.step_re;
    step_im = d.p.m64.step_im;
  } else {
    re_min = d.p.m32.re_min;  // rounded to float once by the host
    im_min = d.p.m32.im_min;
    step_re = d.p.m32.step_re;
    step_im = d.p.m32.step_im;
  }
  const uint32_t width = d.p.m64.width, row0 = d.p.m64.row0, rows = d.p.m64.rows;
  const uint32_t max_iter = d.p.m64.max_iter;
  const auto out = global_ptr(reinterpret_cast<uint16_t*>(d.out));
  // colour reply (a transformation fused at spawn): palette[min(n, len - 1)]
  const bool rgba = (d.flags & DF_RGBA) != 0;
  const auto pal = global_ptr(reinterpret_cast<const uint32_t*>(d.in0));
  const uint32_t pal_last = d.numel - 1u;
  const auto out32 = global_ptr(reinterpret_cast<uint32_t*>(d.out));
  constexpr uint32_t GC = sizeof(T) == 8 ? 1u : 2u;  // a group's block columns
  static_assert(GC == mandel_group_cols(sizeof(T) == 8) && GC * kMandelGroupRows == P,
                "a wave's group is P blocks");
  const uint32_t bw = (width + kMandelBlockW - 1) / kMandelBlockW;
  const uint32_t gw = (bw + GC - 1) / GC;  // groups across
  const uint32_t nb = mandel_blocks(width, rows, sizeof(T) == 8);
  const uint32_t bpt = d.tcfg / 64;
  const uint32_t b0 = tile * bpt;
  const uint32_t b1 = min(nb, b0 + bpt * count);
  const uint32_t lane = lane_id();
  if (threadIdx.x == 0) *lds_ctr = 0;
  __syncthreads();
  // A wave takes a group of P blocks at a time, one pixel of each per lane.
  const uint64_t run_t0 = wall_clock64();
  for (;;) {
    {
      const uint64_t age = wall_clock64() - run_t0;
      if (age > 4 * kPrioStepTicks) __builtin_amdgcn_s_setprio(3);
      else if (age > 2 * kPrioStepTicks) __builtin_amdgcn_s_setprio(2);
      else if (age > kPrioStepTicks) __builtin_amdgcn_s_setprio(1);
    }
    uint32_t b = 0;
    if (lane == 0) b = atomicAdd(lds_ctr, (uint32_t)P);
    b = __builtin_amdgcn_readfirstlane(b) + b0;
    if (b >= b1) break;
    uint32_t y[P], x[P], n[P];
    bool v[P];
    T cr[P], ci[P];
#pragma unroll
    for (int k = 0; k < P; ++k) {
      const uint32_t bk = b + k;
      const uint32_t q = bk / P, r = bk % P;  // group, block within it
      const uint32_t qy = q / gw, qx = q - qy * gw;
      const uint32_t by = qy * kMandelGroupRows + r / GC, bx = qx * GC + r % GC;
      y[k] = by * kMandelBlockH + lane / kMandelBlockW;
      x[k] = bx * kMandelBlockW + lane % kMandelBlockW;
      v[k] = bk < b1 && y[k] < rows && x[k] < width;
      T gx = (T)x[k];
      T xm = gx * step_re;
      cr[k] = re_min + xm;
      T gy = (T)(row0 + y[k]);
      T ym = gy * step_im;
      ci[k] = im_min + ym;
    }
    escape_count<T, P>(cr, ci, v, max_iter, n);
#pragma unroll
    for (int k = 0; k < P; ++k) {
      if (!v[k]) continue;
      const uint64_t at = (uint64_t)y[k] * width + x[k];
      if (rgba) store_reply(out32 + at, (uint32_t)pal[min(n[k], pal_last)]);
      else store_reply(out + at, (uint16_t)n[k]);
    }
  }
  __builtin_amdgcn_s_setprio(0);
}

// ---------------------------------------------------------------------------
// Dense product C = A * B of flat row-major n x n matrices (Sec. 4.6, the
// matrix_multiply actor: two input arrays, the output array last), on the
// matrix cores with fp32 accumulation.  A work tile is a TE x TE block of C
// (TE = 64 or 128); its four waves each own a (TE/2) x (TE/2) quarter made
// of 32 x 32 MFMA blocks.  K advances in LDS-staged slices; rows, columns
// and k beyond n are zero-filled on load and masked on store, so any n
// works.
//
// MFMA operand layout used (32 x 32 output blocks): lane l supplies A row
// l % 32 and B column l % 32; the k index a lane supplies is the same
// function of (l / 32, element) for A and B, so the product sums every k
// exactly once.  Output register r of lane l holds row
// 8*(r/4) + 4*(l/32) + r%4, column l % 32.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void tile_coords(uint32_t tile, uint32_t n, uint32_t te,
                                            uint32_t& tm, uint32_t& tn) {
  const uint32_t tpr = (n + te - 1) / te;
  tm = tile / tpr;
  tn = tile - tm * tpr;
}

template <int TE>
__device__ __forceinline__ void store_c(CAF_GLOBAL float* C, uint32_t n, uint32_t row_base,
                                        uint32_t col_base, const floatx16& acc) {
  const uint32_t lane = lane_id();
  const uint32_t col = col_base + (lane & 31);
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const uint32_t row = row_base + 8 * (r / 4) + 4 * (lane >> 5) + (r & 3);
    if (row < n && col < n) store_reply(C + ((uint64_t)row * n + col), acc[r]);
  }
}

// fp32 inputs, on the bf16 matrix cores.  Each operand element is split into
// three bf16 terms, a = a1 + a2 + a3: a1 = bf16(a), a2 = bf16(a - a1),
// a3 = a - a1 - a2, which is exact (3 x 8 significant bits and the signs hold
// fp32's 24; the split is Dekker's idea with bf16 parts, as in Henry, Tang
// and Heinecke, "Leveraging the bfloat16 Artificial Intelligence Datatype For
// Higher-Precision Computations", ARITH 2019).  A product is then nine terms,
// each exact in fp32.  a1 b1 has an accumulator of its own and seven more
// share a second one, whose roundings are 2^-8 as large; a3 b3, at most
// 2^-36 |a b|, is left out: less than those roundings.  Eight 32x32x16 bf16
// instructions (32 cycles each) replace eight 32x32x2 fp32 ones (64 cycles).
//
// Errors against float64, in 2^-24 of the sum of |a b|, root mean square,
// fp32 instructions / this: entries U(-1, 1) 0.40 / 0.11 at n = 512, U(0, 1)
// 5.1 / 1.9, magnitudes spread over 2^-20 .. 2^20 0.95 / 0.83 at n = 33 and
// 1.9 / 1.4 at 512; sums of one term (a diagonal factor) 0.42 / 0.42, at most
// 0.500 / 0.506 of the last place.  Up to n = 32 the bf16 instruction's own
// sum of 16 products could be the larger (magnitudes over 2^-10 .. 2^10, n = 4:
// 0.39 / 0.58), and those products are one block: they take the fp32
// instructions.
// Products in a batch, 256 of n = 512: 815 us with the fp32 instructions,
// 650 us (106 TFLOP/s); 4,096 of 64 .. 512 3455 -> 2800.  The clock drops to
// 1.7 GHz under the matrix instructions, which are under way in half of its
// cycles in that mix (an eighth of the 1.3 PFLOP/s that large bf16 products
// reach would be 163 TFLOP/s); the rest is the slices' barriers and operand
// reads, 3.5 times the operands' bytes from beyond the L2.
//
// The split is exact only while no term underflows, and a value near the top
// of the range rounds to infinity.  So a 32 x 32 block of C is redone with
// the fp32 instructions (gemm_f32_direct) if an output in it is not finite,
// or if its operands hold numbers so small that bits may have been lost
// (F32Note) and one of its outputs is so small that these bits could show.
// Infinities, NaNs, tiny and huge inputs come out as those instructions give
// them; a softmax or a Gaussian kernel matrix, which holds tiny numbers next
// to ordinary ones, is not redone (128 products of n = 512: 400 us as for
// U(-1, 1) entries, 1490 us when every 128-tile with a product of entries
// below 2^-100 was redone, 480 with fp32 instructions only).  Where every
// output is about as small as fp32 holds, below 2^-122, the whole product is:
// 930 us, 485 with fp32 instructions only.
// What is noted does not depend on the tile edge, nor does any sum: the same
// product has the same bits whatever the load chose.
//
// Layout.  K advances in slices of 16 (TE = 128) or 2 x 16 (TE = 64), which
// two waves load as A and two as B, 16 elements per thread.  LDS holds, per
// 16 deep sub-slice, the three terms of A as [row][k] and of B as
// [column][k], rows of 32 bytes padded to 48 (16-byte reads of 8 consecutive
// rows touch distinct banks); two terms of consecutive k are packed by one
// conversion, which also transposes B.  Registers hold the next two slices,
// so a load has two slices of matrix work to arrive in.
//
// Any n > 32 and any alignment of floats: 16-byte loads, from addresses
// clamped into the matrix, put right in the last slice of a tile where n is
// no multiple of the slice depth and at the matrix's edges (512 products of
// n = 17 .. 500: 1316 us with element loads and fp32 instructions, 489).
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// One 32 x 32 block of C by one wave with the fp32 matrix instructions,
// operands straight from memory: products of n <= 32 and the blocks described
// above.  16 k at a time, the lower half of the wave the first eight of them
// and the upper half the others, loaded one step ahead.
__device__ __noinline__ void gemm_f32_direct(const float* A, const float* B, float* C, uint32_t n,
                                             uint32_t row0, uint32_t col0) {
  const auto Ag = global_ptr(A);
  const auto Bg = global_ptr(B);
  const uint32_t lane = lane_id(), kl = (lane >> 5) * 8;
  const uint32_t row = min(row0 + (lane & 31), n - 1u), col = min(col0 + (lane & 31), n - 1u);
  const auto Ar = Ag + row * n + kl;
  const auto Bc = Bg + kl * n + col;
  floatx16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  const uint32_t whole = n / 16;  // steps of 16 k inside the matrix
  f32x4u a[2], an[2];
  float b[8], bn[8];
  auto load = [&](uint32_t k0) {
    an[0] = *reinterpret_cast<const CAF_GLOBAL f32x4u*>(Ar + k0);
    an[1] = *reinterpret_cast<const CAF_GLOBAL f32x4u*>(Ar + k0 + 4);
#pragma unroll
    for (uint32_t q = 0; q < 8; ++q) bn[q] = Bc[(k0 + q) * n];
  };
  auto multiply = [&]() {
#pragma unroll
    for (uint32_t q = 0; q < 8; ++q)
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[q >> 2][q & 3], b[q], acc, 0, 0, 0);
  };
  if (whole) load(0);
  for (uint32_t s = 0; s < whole; ++s) {
#pragma unroll
    for (int q = 0; q < 2; ++q) a[q] = an[q];
#pragma unroll
    for (int q = 0; q < 8; ++q) b[q] = bn[q];
    if (s + 1 < whole) load((s + 1) * 16);
    multiply();
  }
  if (n % 16) {
#pragma unroll
    for (uint32_t q = 0; q < 8; ++q) {
      const uint32_t k = whole * 16 + kl + q, kc = min(k, n - 1u);
      a[q >> 2][q & 3] = k < n ? Ag[row * n + kc] : 0.f;
      b[q] = k < n ? Bg[kc * n + col] : 0.f;
    }
    multiply();
  }
  store_c<32>(global_ptr(C), n, row0, col0, acc);
}

// Where the split may lose bits (biased exponents): an element below 2^-110
// has bits below the smallest bf16 number, 2^-133, and a product below 2^-100
// may have some below the smallest fp32 one.
constexpr uint32_t kSplitMinExp = 127 - 110;
constexpr uint32_t kSplitMinExpSum = 2 * 127 - 100;

// What a tile notes of its operands, per 64 rows of A and 64 columns of B:
// the smallest exponent of a non-zero element (255: all are zero), and 255
// minus the largest.
struct F32Note {
  uint32_t a[2][2], b[2][2];
};
constexpr uint32_t kF32NoteBytes = 3 * sizeof(F32Note);

constexpr uint32_t kF32BufBytes = 36864;

// The part of a tile stream that one wave runs: the waves that load A and
// those that load B differ in how they split and store a slice, and each has
// its own copy of the loop, so that a step is one basic block in which the
// split's vector instructions are scheduled between the matrix instructions
// (a 32-cycle matrix instruction leaves seven vector issue slots; the split
// takes five of them).
template <int TE, int NBUF, bool kA>
__device__ __forceinline__ void gemm_f32_stream(const float* __restrict__ A,
                                                const float* __restrict__ B,
                                                float* __restrict__ C, uint32_t n, uint32_t tile0,
                                                uint32_t count, lds_u8* lds,
                                                CAF_LDS F32Note* s_note) {
  constexpr uint32_t WB = TE / 64;           // 32 x 32 blocks per wave and dimension
  constexpr uint32_t SUB = 128 / TE;         // 16 deep sub-slices per slice
  constexpr uint32_t KS = 16 * SUB;          // k per slice
  constexpr uint32_t ROW = 48;               // bytes of an LDS row
  constexpr uint32_t PLANE = TE * ROW;       // one term of one operand, one sub-slice
  constexpr uint32_t OPND = 3 * PLANE;       // its three terms
  constexpr uint32_t BUF = SUB * 2 * OPND;   // bytes of an LDS buffer
  static_assert(BUF == kF32BufBytes, "slice buffer");
  const auto Cg = global_ptr(C);
  const auto src = reinterpret_cast<const CAF_GLOBAL uint8_t*>(global_ptr(kA ? A : B));
  const uint32_t t = threadIdx.x, lane = lane_id(), w = wave_id();
  const uint32_t wm = w >> 1, wn = w & 1;
  const uint32_t tt = t & 127u;

  floatx16 acc[WB][WB], low[WB][WB];  // a1 b1, and the other eight terms
  auto zero_acc = [&]() {
#pragma unroll
    for (uint32_t i = 0; i < WB; ++i)
#pragma unroll
      for (uint32_t j = 0; j < WB; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = low[i][j][r] = 0.f;
  };
  zero_acc();

  const uint32_t nk = (n + KS - 1) / KS;  // slices per tile: two or more, n > 32
  const uint32_t steps = count * nk;
  // What a thread loads of a slice.  A: four rows TE / 4 apart, 4 k each (the
  // lanes of a row side by side).  B: a block of 4 k x 4 columns.
  const uint32_t a_row = tt / (4 * SUB), a_k = (tt % (4 * SUB)) * 4;
  const uint32_t b_k = (tt & 3u) * 4 + (tt / TE) * 16, b_col = ((tt % TE) >> 2) * 4;
  // Element offsets of its four 16-byte loads, clamped to the matrix's last
  // four elements: a load past the end of a row reads the next row's first
  // elements, one past the matrix its last ones.  fix() and edge() put right
  // what lies beyond n.
  const uint32_t last4 = n * n - 4u;
  const uint32_t stride = kA ? (TE / 4) * n : n;  // between the four loads
  const uint32_t kstep = kA ? KS : KS * n;        // between slices
  struct Slice {
    f32x4u v[4];
  };
  uint32_t ltile = tile0, lk = 0, loff;  // the slice to load next
  auto seek = [&]() {
    uint32_t tm, tn;
    tile_coords(ltile, n, TE, tm, tn);
    loff = kA ? (tm * TE + a_row) * n + a_k : b_k * n + tn * TE + b_col;
  };
  seek();
  auto load = [&](Slice& s) {
#pragma unroll
    for (uint32_t q = 0; q < 4; ++q) {
      const uint32_t off = min(loff + q * stride, last4) * 4u;
      s.v[q] = *reinterpret_cast<const CAF_GLOBAL f32x4u*>(src + off);
    }
  };
  auto load_next = [&](uint32_t step) {  // advances to slice `step` (at most one further)
    if (step >= steps) return;
    if (++lk == nk) {
      lk = 0;
      ++ltile;
      seek();
    } else {
      loff += kstep;
    }
  };
  // elements d .. 3 of v moved to the front, zeros behind (d >= 4: all zeros)
  auto shift = [](f32x4u v, uint32_t d) {
    f32x4u r;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float x = d == 0 ? v[e] : 0.f;
#pragma unroll
      for (int f = e + 1; f < 4; ++f) x = d == (uint32_t)(f - e) ? v[f] : x;
      r[e] = x;
    }
    return r;
  };
  // The last slice of a tile where n is no multiple of KS: loads that were
  // clamped are moved back into place, and k beyond n is zero in A and in B
  // (in both: the other operand's leftovers may be infinite).
  auto fix = [&](Slice& s, uint32_t tm, uint32_t tn) {
    const uint32_t k0 = (nk - 1) * KS;
    const uint32_t off = kA ? (tm * TE + a_row) * n + k0 + a_k : (k0 + b_k) * n + tn * TE + b_col;
#pragma unroll
    for (uint32_t q = 0; q < 4; ++q) {
      const uint32_t o = off + q * stride;
      const uint32_t d = o - min(o, last4);
      s.v[q] = shift(s.v[q], d);
      if constexpr (kA) {
#pragma unroll
        for (uint32_t e = 0; e < 4; ++e)
          if (k0 + a_k + e >= n) s.v[q][e] = 0.f;
      } else {
        if (k0 + b_k + q >= n) s.v[q] = f32x4u{0.f, 0.f, 0.f, 0.f};
      }
    }
  };
  // Rows of A and columns of B outside the matrix, in tiles at its edge, are
  // zero: they neither feed an output nor are noted.
  auto edge = [&](Slice& s, uint32_t tm, uint32_t tn) {
#pragma unroll
    for (uint32_t q = 0; q < 4; ++q) {
      if constexpr (kA) {
        if (tm * TE + a_row + q * (TE / 4) >= n) s.v[q] = f32x4u{0.f, 0.f, 0.f, 0.f};
      } else {
#pragma unroll
        for (uint32_t e = 0; e < 4; ++e)
          if (tn * TE + b_col + e >= n) s.v[q][e] = 0.f;
      }
    }
  };
  // Smallest non-zero and largest magnitude of this thread's elements of the
  // tile, as bits << 1, the former less one.  A: per 64 rows.
  constexpr int NOTES = kA ? (int)WB : 1;
  uint32_t vmin[NOTES], vmax[NOTES];
  auto clear_note = [&]() {
#pragma unroll
    for (int q = 0; q < NOTES; ++q) {
      vmin[q] = 0xFFFFFFFFu;
      vmax[q] = 0;
    }
  };
  clear_note();
  // two consecutive k of one row or column -> a packed pair of each term
  auto split = [&](float x, float y, int half, uint32_t (&p)[3]) {
    const uint32_t mx = __builtin_bit_cast(uint32_t, x) << 1, my = __builtin_bit_cast(uint32_t, y) << 1;
    vmin[half] = min(vmin[half], min(mx - 1u, my - 1u));
    vmax[half] = max(vmax[half], max(mx, my));
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const f32x2 xy = {x, y};
      const uint32_t h = __builtin_bit_cast(uint32_t, __builtin_convertvector(xy, bf16x2));
      p[q] = h;
      if (q < 2) {
        x = x - __builtin_bit_cast(float, h << 16);
        y = y - __builtin_bit_cast(float, h & 0xFFFF0000u);
      }
    }
  };
  const uint32_t dst0 = kA ? (a_k >> 4) * (2 * OPND) + a_row * ROW + (a_k & 15u) * 2
                           : (b_k >> 4) * (2 * OPND) + OPND + b_col * ROW + (b_k & 15u) * 2;
  auto lstore = [&](const Slice& s, lds_u8* buf) {
    lds_u8* dst = buf + dst0;
#pragma unroll
    for (uint32_t q = 0; q < 4; ++q) {  // row q of A, column q of B
      uint32_t lo[3], hi[3];
      const int half = kA ? (int)(q * WB / 4) : 0;
      split(kA ? s.v[q][0] : s.v[0][q], kA ? s.v[q][1] : s.v[1][q], half, lo);
      split(kA ? s.v[q][2] : s.v[2][q], kA ? s.v[q][3] : s.v[3][q], half, hi);
#pragma unroll
      for (uint32_t p = 0; p < 3; ++p)
        *reinterpret_cast<CAF_LDS u32x2*>(dst + p * PLANE + q * (kA ? TE / 4 : 1) * ROW) =
            u32x2{lo[p], hi[p]};
    }
  };
  auto note = [&](uint32_t tseq) {  // the tile's last slice is in LDS
    typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
#pragma unroll
    for (int q = 0; q < NOTES; ++q) {
      uint32_t v = vmin[q] >> 24 | (255u - (vmax[q] >> 24)) << 16;
#pragma unroll
      for (int off = 32; off > 0; off >>= 1)
        v = __builtin_bit_cast(
            uint32_t, __builtin_elementwise_min(
                          __builtin_bit_cast(u16x2, v),
                          __builtin_bit_cast(u16x2, (uint32_t)__shfl_xor((int)v, off))));
      if (lane == 0) {
        CAF_LDS uint32_t* to = kA ? s_note[tseq % 3].a[q] : s_note[tseq % 3].b[tt / 64 * WB / 2];
        __hip_atomic_fetch_min(to, v & 0xFFFFu, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        __hip_atomic_fetch_min(to + 1, v >> 16, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
    }
    clear_note();
  };
  auto mfma_slice = [&](const lds_u8* buf) {
#pragma unroll
    for (uint32_t sub = 0; sub < SUB; ++sub) {
      const lds_u8* As = buf + sub * (2 * OPND) + (lane >> 5) * 16;
      const lds_u8* Bs = As + OPND;
      bf16x8 a[3][WB], b[WB];
#pragma unroll
      for (uint32_t p = 0; p < 3; ++p)
#pragma unroll
        for (uint32_t i = 0; i < WB; ++i)
          a[p][i] = __builtin_bit_cast(
              bf16x8, *reinterpret_cast<const CAF_LDS u32x4*>(
                          As + p * PLANE + (wm * (TE / 2) + i * 32 + (lane & 31)) * ROW));
#pragma unroll
      for (int pb = 2; pb >= 0; --pb) {
#pragma unroll
        for (uint32_t j = 0; j < WB; ++j)
          b[j] = __builtin_bit_cast(
              bf16x8, *reinterpret_cast<const CAF_LDS u32x4*>(
                          Bs + pb * PLANE + (wn * (TE / 2) + j * 32 + (lane & 31)) * ROW));
#pragma unroll
        for (int pa = pb == 2 ? 1 : 2; pa >= 0; --pa)  // all but a3 b3
#pragma unroll
          for (uint32_t i = 0; i < WB; ++i)
#pragma unroll
            for (uint32_t j = 0; j < WB; ++j) {
              floatx16& to = pa + pb ? low[i][j] : acc[i][j];
              to = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[pa][i], b[j], to, 0, 0, 0);
            }
      }
    }
  };
  // Stores the tile; has the 32 x 32 blocks redone for which the split does
  // not hold.
  auto finish_tile = [&](uint32_t tm, uint32_t tn, uint32_t tseq) {
    const CAF_LDS F32Note& nt = s_note[tseq % 3];
    const uint32_t ha = TE == 128 ? wm : 0u, hb = TE == 128 ? wn : 0u;
    const uint32_t ea = __builtin_amdgcn_readfirstlane(nt.a[ha][0]),
                   eb = __builtin_amdgcn_readfirstlane(nt.b[hb][0]);
    // an operand of zeros only (255) is exact
    const bool lossy = ea != 255u && eb != 255u &&
                       (ea < kSplitMinExp || eb < kSplitMinExp || ea + eb < kSplitMinExpSum);
    const uint32_t r0 = tm * TE + wm * (TE / 2), c0 = tn * TE + wn * (TE / 2);
    uint32_t redo = 0;  // bit per block
#pragma unroll
    for (uint32_t i = 0; i < WB; ++i)
#pragma unroll
      for (uint32_t j = 0; j < WB; ++j) {
        float any[2] = {0.f, 0.f};  // NaN if an output is not finite
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          acc[i][j][r] += low[i][j][r];
          any[r & 1] = __builtin_fmaf(acc[i][j][r], 0.f, any[r & 1]);
        }
        if (__builtin_amdgcn_ballot_w64(!(any[0] + any[1] == 0.f))) redo |= 1u << (i * WB + j);
      }
    if (__builtin_expect(lossy, 0)) {
      // What the split may have lost of an output, per k: 2^-134 of the other
      // operand's largest for small elements, and 2^-146.  It is nothing next
      // to the rounding of a sum, 2^-24 of its magnitude per k, where the
      // output alone is 2^24 times as large.
      auto largest = [](uint32_t inv) {  // 2^(exponent + 1) of the biased one, finite
        return __builtin_bit_cast(float, min(255u - inv + 1u, 254u) << 23);
      };
      const float ma = largest(__builtin_amdgcn_readfirstlane(nt.a[ha][1])),
                  mb = largest(__builtin_amdgcn_readfirstlane(nt.b[hb][1]));
      const float lost = 0x1p-110f * ((ea < kSplitMinExp ? mb : 0.f) +
                                      (eb < kSplitMinExp ? ma : 0.f)) + 0x1p-122f;
#pragma unroll
      for (uint32_t i = 0; i < WB; ++i)
#pragma unroll
        for (uint32_t j = 0; j < WB; ++j) {
          bool small = false;
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const uint32_t row = r0 + i * 32 + 8 * (r / 4) + 4 * (lane >> 5) + (r & 3);
            small |= row < n && __builtin_fabsf(acc[i][j][r]) < lost;
          }
          if (__builtin_amdgcn_ballot_w64(small && c0 + j * 32 + (lane & 31) < n))
            redo |= 1u << (i * WB + j);
        }
    }
#pragma unroll
    for (uint32_t i = 0; i < WB; ++i)
#pragma unroll
      for (uint32_t j = 0; j < WB; ++j)
        if (!(redo >> (i * WB + j) & 1u))
          store_c<TE>(Cg, n, r0 + i * 32, c0 + j * 32, acc[i][j]);
    while (__builtin_expect(redo != 0, 0)) {
      const uint32_t q = __builtin_ctz(redo);
      redo &= redo - 1u;
      const uint32_t rq = r0 + q / WB * 32, cq = c0 + q % WB * 32;
      if (rq < n && cq < n) gemm_f32_direct(A, B, C, n, rq, cq);
    }
    zero_acc();
    if (t < sizeof(F32Note) / 4)
      reinterpret_cast<CAF_LDS uint32_t*>(s_note + (tseq + 2) % 3)[t] = 255u;
  };

  Slice s0, s1;
  const bool ragged = n % KS != 0;
  // the slice that goes to LDS next: its position and its tile
  uint32_t sk = 0, sseq = 0, stm, stn;
  tile_coords(tile0, n, TE, stm, stn);
  load(s0);
  load_next(1);
  load(s1);
  load_next(2);
  auto put_right = [&](Slice& s, uint32_t k) {  // slice k of tile (stm, stn)
    if (ragged && k == nk - 1) fix(s, stm, stn);
    if ((kA ? stm : stn) * TE + TE > n) edge(s, stm, stn);
  };
  put_right(s0, 0);
  lstore(s0, lds);
  __syncthreads();
  uint32_t ctm = stm, ctn = stn, ck = 0, cseq = 0;  // the slice computed
  // Computes slice s from LDS, loads slice s + 2 into `in` and puts slice
  // s + 1, `out`, into LDS.  Past the end it loads and stores the last slice
  // again, into a buffer nobody reads.
  auto step = [&](uint32_t s, Slice& in, Slice& out) {
    const bool more = s + 1 < steps;
    if (more && ++sk == nk) {
      sk = 0;
      ++sseq;
      tile_coords(tile0 + sseq, n, TE, stm, stn);
    }
    if (more) put_right(out, sk);
    load(in);
    load_next(s + 3);
    __builtin_amdgcn_sched_barrier(0);
    mfma_slice(lds + (NBUF == 2 ? (s & 1u) * BUF : 0u));
    if constexpr (NBUF == 1) __syncthreads();  // every wave has read the buffer
    lstore(out, lds + (NBUF == 2 ? ((s + 1) & 1u) * BUF : 0u));
    if constexpr (NBUF == 2) {
      // matrix instructions with the split between them
      __builtin_amdgcn_sched_group_barrier(0x100, 4 * WB, 0);  // fragments first
#pragma unroll
      for (uint32_t q = 0; q < 8 * SUB * WB * WB; ++q) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, 5, 0);
        __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    if (sk == nk - 1 && more) note(sseq);
    if (ck == nk - 1) {
      finish_tile(ctm, ctn, cseq);
      ++cseq;
      ck = 0;
    } else {
      ++ck;
    }
    ctm = stm;
    ctn = stn;
    __syncthreads();
  };
  for (uint32_t s = 0; s < steps; s += 2) {
    step(s, s0, s1);
    if (s + 1 < steps) step(s + 1, s1, s0);
  }
}

// NBUF: LDS buffers (2, or 1 where the kernel variant has half the LDS).
// One call computes `count` consecutive output tiles (row-major tile order)
// of one product, as one stream of slices.  smem: NBUF x 36 KB and the notes.
template <int TE, int NBUF = 2>
__device__ __forceinline__ void gemm_f32_tile(const float* __restrict__ A,
                                              const float* __restrict__ B,
                                              float* __restrict__ C, uint32_t n, uint32_t tile0,
                                              uint32_t count, lds_u8* smem) {
  // three tiles' notes in turn, so that one is cleared while the next is in use
  CAF_LDS F32Note* s_note = reinterpret_cast<CAF_LDS F32Note*>(smem + NBUF * kF32BufBytes);
  const uint32_t t = threadIdx.x, w = __builtin_amdgcn_readfirstlane(wave_id());
  if (n <= 32) {  // one block
    if (w == 0) gemm_f32_direct(A, B, C, n, 0, 0);
    __syncthreads();
    return;
  }
  if (t < kF32NoteBytes / 4) reinterpret_cast<CAF_LDS uint32_t*>(s_note)[t] = 255u;
  __syncthreads();
  if (w < 2) gemm_f32_stream<TE, NBUF, true>(A, B, C, n, tile0, count, smem, s_note);
  else gemm_f32_stream<TE, NBUF, false>(A, B, C, n, tile0, count, smem, s_note);
}

// bfloat16 inputs: v_mfma_f32_32x32x16_bf16, k slices of kBf16SliceK.  Both operands
// are kept k-contiguous in LDS ([row][k] for A, [column][k] for B, rows
// padded by 16 bytes) so each lane reads its 8 k values with one 16-byte
// LDS load.  B is transposed on the way in: a thread loads a 4 (k) x 8 (n)
// block as four 16-byte rows and regroups it in registers with byte
// permutes into eight 8-byte columns.  smem: 2 x 2 x TE x (kBf16SliceK + 8)
// bf16.  One call computes `count` consecutive output tiles (row-major tile
// order) of one product.
// k per LDS slice of the bf16 tile: long enough that a slice's matrix-core
// work covers the next slice's global loads (64); a kernel variant that keeps
// more workgroups per compute unit uses 32, which halves the tile's LDS.
constexpr int kBf16SliceK = 64;

template <int TE, int BK = kBf16SliceK>
__device__ __forceinline__ void gemm_bf16_tile(const uint16_t* __restrict__ A, const uint16_t* __restrict__ B,
                               float* __restrict__ C, uint32_t n, uint32_t tile0,
                               uint32_t count, lds_u8* smem8) {
  typedef CAF_LDS uint16_t lds_u16;
  lds_u16* smem = reinterpret_cast<lds_u16*>(smem8);
  constexpr int LD = BK + 8;
  constexpr int WB = TE / 64;
  constexpr int QA = TE * BK / 8 / kThreads;  // 16-byte A chunks per thread
  constexpr int SLICE = 2 * TE * LD;          // bf16 per LDS buffer
  const auto Ag = reinterpret_cast<const CAF_GLOBAL uint8_t*>(global_ptr(A));
  const auto Bg = reinterpret_cast<const CAF_GLOBAL uint8_t*>(global_ptr(B));
  const auto Cg = global_ptr(C);
  const uint32_t t = threadIdx.x, lane = lane_id(), w = wave_id();
  const uint32_t wm = w >> 1, wn = w & 1;
  if (n < 3) {  // fewer than eight elements: no 16-byte loads
    if (t < n * n) {
      auto f = [](uint16_t h) { return __builtin_bit_cast(float, (uint32_t)h << 16); };
      const uint32_t r = t / n, c = t % n;
      float x = f(A[r * n]) * f(B[c]);  // exact
      if (n == 2) x = __builtin_fmaf(f(A[r * n + 1]), f(B[n + c]), x);
      store_reply(Cg + t, x);
    }
    __syncthreads();
    return;
  }
  floatx16 acc[WB][WB];
  auto zero_acc = [&]() {
#pragma unroll
    for (int i = 0; i < WB; ++i)
#pragma unroll
      for (int j = 0; j < WB; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  };
  auto store_tile = [&](uint32_t tm, uint32_t tn) {
#pragma unroll
    for (int i = 0; i < WB; ++i)
#pragma unroll
      for (int j = 0; j < WB; ++j)
        store_c<TE>(Cg, n, tm * TE + wm * (TE / 2) + i * 32, tn * TE + wn * (TE / 2) + j * 32,
                    acc[i][j]);
  };
  auto mfma_slice = [&](const lds_u16* As, const lds_u16* Bs) {
#pragma unroll
    for (int ks = 0; ks < BK; ks += 16) {
      const uint32_t kc = ks + 8 * (lane >> 5);
      bf16x8 a[WB], b[WB];
#pragma unroll
      for (int i = 0; i < WB; ++i)
        a[i] = __builtin_bit_cast(
            bf16x8, *reinterpret_cast<const CAF_LDS u32x4*>(
                        As + (wm * (TE / 2) + i * 32 + (lane & 31)) * LD + kc));
#pragma unroll
      for (int j = 0; j < WB; ++j)
        b[j] = __builtin_bit_cast(
            bf16x8, *reinterpret_cast<const CAF_LDS u32x4*>(
                        Bs + (wn * (TE / 2) + j * 32 + (lane & 31)) * LD + kc));
#pragma unroll
      for (int i = 0; i < WB; ++i)
#pragma unroll
        for (int j = 0; j < WB; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
    }
  };
  zero_acc();

  // The tiles of the range run as one stream of 64-deep slices: while the
  // matrix cores work on one slice, the next one (possibly the first of
  // the next tile) is already being loaded, so a tile's first loads and
  // its output stores overlap its neighbours' work.
  //
  // Every load is 16 bytes, at any alignment of elements (products of
  // n % 8 != 0 were loaded element by element: 1,024 of n = 500 6.4 ms, now
  // as n = 512's), and issued unconditionally from an address inside the
  // matrix, so the registers it fills have a single definition and the
  // compiler need not wait for the prefetch before the current slice's
  // matrix instructions.  A load past the end of a row reads the next row's
  // first elements, one past the matrix its last eight.  Rows of A and
  // columns of B outside the matrix only feed rows / columns of C that are
  // not stored; k beyond n is put right in lstore(), in a tile's last slice.
  // With TE = 64 only half the threads own a B block; the others load a
  // block and skip its store.
  constexpr int NB4 = (BK / 4) * (TE / 8);  // 4 (k) x 8 (n) blocks of B per slice
  static_assert(NB4 <= kThreads, "one B block per thread at most");
  const uint32_t kb = t % (BK / 4), nb = (t / (BK / 4)) % (TE / 8);  // k-block fastest
  const bool has_b = NB4 == kThreads || t < (uint32_t)NB4;
  uint32_t kca[QA];
#pragma unroll
  for (int q = 0; q < QA; ++q) kca[q] = ((t + kThreads * q) % (BK / 8)) * 8;
  const uint32_t last8 = n * n - 8u;
  uint32_t ao[QA], bo;  // element offsets of this thread's loads at k = 0
  auto sources = [&](uint32_t tm, uint32_t tn) {
#pragma unroll
    for (int q = 0; q < QA; ++q)
      ao[q] = (tm * TE + (t + kThreads * q) / (BK / 8)) * n + kca[q];
    bo = kb * 4 * n + tn * TE + nb * 8;
  };
  auto load8 = [&](const CAF_GLOBAL uint8_t* base, uint32_t o) {
    return __builtin_bit_cast(
        uint4, (u32x4)*reinterpret_cast<const CAF_GLOBAL u32x4a2*>(base + min(o, last8) * 2u));
  };
  uint4 ra[QA], rb[4];
  auto gload = [&](uint32_t k0) {
#pragma unroll
    for (int q = 0; q < QA; ++q) ra[q] = load8(Ag, ao[q] + k0);
#pragma unroll
    for (int r = 0; r < 4; ++r) rb[r] = load8(Bg, bo + (k0 + r) * n);
  };
  // elements d .. 7 moved to the front (the load was clamped by d)
  auto moved = [](uint4 v, uint32_t d) {
    const unsigned __int128 x = __builtin_bit_cast(unsigned __int128, v);
    return __builtin_bit_cast(uint4, d < 8 ? x >> (16 * d) : (unsigned __int128)0);
  };
  // the first m elements kept
  auto first = [](uint4 v, uint32_t m) {
    const unsigned __int128 x = __builtin_bit_cast(unsigned __int128, v);
    return __builtin_bit_cast(uint4, m < 8 ? x & (((unsigned __int128)1 << (16 * m)) - 1) : x);
  };
  // the slice's place in its tile's sources (ao, bo) is still that of the
  // slice stored: a tile's last slice is stored before its successor loads
  auto fix = [&](uint32_t k0) {
#pragma unroll
    for (int q = 0; q < QA; ++q) {
      const uint32_t o = ao[q] + k0, k = k0 + kca[q];
      ra[q] = first(moved(ra[q], o - min(o, last8)), k < n ? n - k : 0u);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const uint32_t o = bo + (k0 + r) * n;
      rb[r] = k0 + kb * 4 + r < n ? moved(rb[r], o - min(o, last8)) : make_uint4(0, 0, 0, 0);
    }
  };
  auto lstore = [&](lds_u16* buf, uint32_t k0, bool checked) {
    if (checked) fix(k0);
    lds_u16* As = buf;
    lds_u16* Bs = buf + TE * LD;
#pragma unroll
    for (int q = 0; q < QA; ++q) {
      const uint32_t idx = t + kThreads * q;
      *reinterpret_cast<CAF_LDS u32x4*>(As + (idx / (BK / 8)) * LD + kca[q]) =
          __builtin_bit_cast(u32x4, ra[q]);
    }
    if (has_b) {
      // column c of the block: k pairs (2m, 2m+1) from rows 2m and 2m+1,
      // low halves for even c, high halves for odd c
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        uint32_t col[2];
#pragma unroll
        for (int m = 0; m < 2; ++m) {
          const uint4 lo = rb[2 * m], hi = rb[2 * m + 1];
          const uint32_t wl = (c >> 1) == 0 ? lo.x : (c >> 1) == 1 ? lo.y : (c >> 1) == 2 ? lo.z : lo.w;
          const uint32_t wh = (c >> 1) == 0 ? hi.x : (c >> 1) == 1 ? hi.y : (c >> 1) == 2 ? hi.z : hi.w;
          col[m] = __builtin_amdgcn_perm(wh, wl, (c & 1) ? 0x07060302u : 0x05040100u);
        }
        *reinterpret_cast<CAF_LDS u32x2*>(Bs + (nb * 8 + c) * LD + kb * 4) = u32x2{col[0], col[1]};
      }
    }
  };
  const uint32_t nk = (n + BK - 1) / BK;   // slices per tile
  const uint32_t last = nk - 1;            // the only slice that can be partial
  const bool ragged = (n % BK) != 0;
  const uint32_t steps = count * nk;
  uint32_t tile = tile0, k = 0, tm, tn;
  tile_coords(tile, n, TE, tm, tn);
  sources(tm, tn);
  gload(0);
  lstore(smem, 0, ragged && last == 0);
  __syncthreads();
  uint32_t cur = 0;
  // Step s computes slice k of `tile` from LDS buffer `cur` and prefetches
  // step s + 1.  The last step is peeled off so that every iteration
  // issues its prefetch unconditionally.
  for (uint32_t s = 0; s + 1 < steps; ++s) {
    const bool tile_ends = k == last;
    const uint32_t otm = tm, otn = tn;
    const uint32_t k1 = tile_ends ? 0u : k + 1;
    if (tile_ends) {
      tile_coords(tile + 1, n, TE, tm, tn);
      sources(tm, tn);
    }
    const bool chk = ragged && k1 == last;
    gload(k1 * BK);
    // keep the prefetch ahead of the matrix instructions (the scheduler
    // would otherwise sink the loads to shorten their registers' lives)
    __builtin_amdgcn_sched_barrier(0);
    const lds_u16* buf = smem + cur * SLICE;
    mfma_slice(buf, buf + TE * LD);
    if (tile_ends) {
      store_tile(otm, otn);
      zero_acc();
      ++tile;
    }
    lstore(smem + (cur ^ 1u) * SLICE, k1 * BK, chk);
    __syncthreads();
    cur ^= 1u;
    k = k1;
  }
  {
    const lds_u16* buf = smem + cur * SLICE;
    mfma_slice(buf, buf + TE * LD);
    store_tile(tm, tn);
  }
}

// Wide bf16 tiles: 128 x 256 blocks of C (each wave 64 x 128, 2 x 4 MFMA
// blocks), for products with n % 32 == 0 and 16-byte aligned operands.  A
// wider block reads a quarter fewer operand bytes per flop than two 128 x 128
// tiles; a batch of mixed products is bound by those reads from beyond L2
// (each tile re-reads the A and B panels it shares with its neighbours).
// The drain's variant with two workgroups per compute unit has them, as a call
// beside the other matrix tiles.
//
// Operands go from global memory straight into a three-stage LDS ring
// (global_load_lds_dwordx4: 16 bytes per lane, laid out lane by lane per wave
// instruction), 32-deep k slices of 24 KB, so two slices are in flight while
// the third is multiplied and no registers stage them.  Rows are XOR-swizzled
// in 16-byte chunks: A (row-major, 64-byte rows) by (row / 2) % 4, B
// (row-major k x n, 512-byte rows) by 2 * (k % 4), so the fragment reads of
// a wave spread over the LDS banks.  A fragments (8 consecutive k of one
// row) are 16-byte LDS reads; B fragments (8 consecutive k of one column)
// come from the transposing read ds_read_b64_tr_b16: across 16 lanes that
// each address four consecutive bf16 of a row, lane j receives element j % 4
// of the rows addressed by lanes j / 4, j / 4 + 4, j / 4 + 8 and j / 4 + 12
// -- so lanes addressing B[k + r / 4][n0 + 4 (r % 4)] (r = 0..15) hand lane j
// the column B[k .. k + 3][n0 + j].  Two such reads give a lane its 8 k.
//
// The direct loads are waited for explicitly (vmcnt), then a barrier without
// a memory fence makes every wave's data visible.  The fragment reads are
// issued from inline assembly that waits for them itself (lgkmcnt): issued
// as builtins, the compiler would wait for every direct load in flight
// before them, as it cannot tell that they read another stage.  Output
// stores share the vmcnt counter with the loads, so after a tile's stores
// the next slice is waited for with vmcnt(0).
//
// Tile t of a product covers row block t / ceil(n / 256) and column block
// t % ceil(n / 256).  smem: 72 KB.
constexpr uint32_t kWideStages = 3;
constexpr uint32_t kWideSmemBytes = kWideStages * (128 * 32 + 32 * 256) * 2;

// s_waitcnt limiting only vmcnt (expcnt 7 and lgkmcnt 15 impose no wait)
#define CAF_WAIT_VMCNT(N) \
  __builtin_amdgcn_s_waitcnt(((N) & 15) | (((N) >> 4) << 14) | (7 << 4) | (15 << 8))

// Workgroup barrier without the memory fence of __syncthreads, fenced
// against compiler reordering of the LDS accesses around it.
__device__ __forceinline__ void barrier_no_fence() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

__device__ __forceinline__ void gemm_bf16_tile_wide(const uint16_t* __restrict__ A,
                                                    const uint16_t* __restrict__ B,
                                                    float* __restrict__ C, uint32_t n,
                                                    uint32_t tile0, uint32_t count, lds_u8* lds) {
  constexpr uint32_t TM = 128, TN = 256, BK = 32, WM = 2, WN = 4, NS = kWideStages;
  constexpr uint32_t A_BYTES = TM * BK * 2, B_BYTES = BK * TN * 2, STAGE = A_BYTES + B_BYTES;
  constexpr uint32_t LOADS = (A_BYTES + B_BYTES) / 16 / kThreads;  // direct loads per thread and slice
  const auto Ag = global_ptr(A);
  const auto Bg = global_ptr(B);
  const auto Cg = global_ptr(C);
  const uint32_t t = threadIdx.x, lane = lane_id(), w = wave_id();
  const uint32_t wm = w >> 1, wn = w & 1;
  const uint32_t lds0 = (uint32_t)(uintptr_t)lds;
  floatx16 acc[WM][WN];
  auto zero_acc = [&]() {
#pragma unroll
    for (uint32_t i = 0; i < WM; ++i)
#pragma unroll
      for (uint32_t j = 0; j < WN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  };
  zero_acc();
  const uint32_t nk = n / BK, tpr = (n + TN - 1) / TN;
  const uint32_t steps = count * nk;
  auto coords = [&](uint32_t tl, uint32_t& tm, uint32_t& tn) {
    tm = tl / tpr;
    tn = tl - tm * tpr;
  };
  // Direct loads of slice s into stage s % NS.  Rows beyond n read the last
  // row and columns beyond n the first ones: they only feed rows and
  // columns of C that are not stored.
  auto issue = [&](uint32_t s) {
    const uint32_t k0 = (s % nk) * BK;
    uint32_t tm, tn;
    coords(tile0 + s / nk, tm, tn);
    lds_u8* st = lds + (s % NS) * STAGE;
#pragma unroll
    for (uint32_t q = 0; q < A_BYTES / 16 / kThreads; ++q) {
      const uint32_t idx = q * kThreads + t;  // 16-byte chunk of the stage's A
      const uint32_t row = idx >> 2, c = (idx & 3) ^ ((row >> 1) & 3);
      const uint32_t grow = min(tm * TM + row, n - 1u);
      __builtin_amdgcn_global_load_lds(
          (const CAF_GLOBAL void*)(Ag + (uint64_t)grow * n + k0 + c * 8),
          (__attribute__((address_space(3))) void*)(st + (q * kThreads + w * 64) * 16), 16, 0, 0);
    }
#pragma unroll
    for (uint32_t q = 0; q < B_BYTES / 16 / kThreads; ++q) {
      const uint32_t idx = q * kThreads + t;  // 16-byte chunk of the stage's B
      const uint32_t krow = idx >> 5, c = (idx & 31) ^ ((krow & 3) << 1);
      uint32_t gcol = tn * TN + c * 8;
      if (gcol >= n) gcol = 0;
      __builtin_amdgcn_global_load_lds(
          (const CAF_GLOBAL void*)(Bg + (uint64_t)(k0 + krow) * n + gcol),
          (__attribute__((address_space(3))) void*)(st + A_BYTES + (q * kThreads + w * 64) * 16), 16,
          0, 0);
    }
  };
  auto compute = [&](uint32_t s) {
    const uint32_t st = lds0 + (s % NS) * STAGE, sb = st + A_BYTES;
    const uint32_t g = lane >> 4, j = lane & 15;
#pragma unroll
    for (uint32_t ks = 0; ks < BK; ks += 16) {
      uint32_t aad[WM], bad[WN][2];
#pragma unroll
      for (uint32_t i = 0; i < WM; ++i) {
        const uint32_t row = wm * 64 + i * 32 + (lane & 31);
        const uint32_t kc = (ks >> 3) + (lane >> 5);
        aad[i] = st + row * (BK * 2) + (kc ^ ((row >> 1) & 3)) * 16;
      }
#pragma unroll
      for (uint32_t jb = 0; jb < WN; ++jb) {
        const uint32_t n0 = wn * 128 + jb * 32 + (g & 1) * 16;
        const uint32_t kq = ks + (g >> 1) * 8;
#pragma unroll
        for (uint32_t h = 0; h < 2; ++h) {
          const uint32_t krow = kq + h * 4 + (j >> 2);
          const uint32_t e = n0 + 4 * (j & 3);  // first column this lane addresses
          bad[jb][h] = sb + krow * (TN * 2) + ((e >> 3) ^ ((krow & 3) << 1)) * 16 + (e & 7) * 2;
        }
      }
      u32x4 a0, a1;
      u32x2 b[WN][2];
      asm volatile(
          "ds_read_b128 %0, %10\n\t"
          "ds_read_b128 %1, %11\n\t"
          "ds_read_b64_tr_b16 %2, %12\n\t"
          "ds_read_b64_tr_b16 %3, %13\n\t"
          "ds_read_b64_tr_b16 %4, %14\n\t"
          "ds_read_b64_tr_b16 %5, %15\n\t"
          "ds_read_b64_tr_b16 %6, %16\n\t"
          "ds_read_b64_tr_b16 %7, %17\n\t"
          "ds_read_b64_tr_b16 %8, %18\n\t"
          "ds_read_b64_tr_b16 %9, %19\n\t"
          "s_waitcnt lgkmcnt(0)"
          : "=&v"(a0), "=&v"(a1), "=&v"(b[0][0]), "=&v"(b[0][1]), "=&v"(b[1][0]), "=&v"(b[1][1]),
            "=&v"(b[2][0]), "=&v"(b[2][1]), "=&v"(b[3][0]), "=&v"(b[3][1])
          : "v"(aad[0]), "v"(aad[1]), "v"(bad[0][0]), "v"(bad[0][1]), "v"(bad[1][0]),
            "v"(bad[1][1]), "v"(bad[2][0]), "v"(bad[2][1]), "v"(bad[3][0]), "v"(bad[3][1]));
      bf16x8 af[WM], bf[WN];
      af[0] = __builtin_bit_cast(bf16x8, a0);
      af[1] = __builtin_bit_cast(bf16x8, a1);
#pragma unroll
      for (uint32_t jb = 0; jb < WN; ++jb) {
        struct {
          u32x2 lo, hi;
        } pr = {b[jb][0], b[jb][1]};
        bf[jb] = __builtin_bit_cast(bf16x8, pr);
      }
#pragma unroll
      for (uint32_t i = 0; i < WM; ++i)
#pragma unroll
        for (uint32_t jb = 0; jb < WN; ++jb)
          acc[i][jb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i], bf[jb], acc[i][jb], 0, 0, 0);
    }
  };
  for (uint32_t s = 0; s < NS - 1 && s < steps; ++s) issue(s);
  bool stores_pending = false;
  for (uint32_t s = 0; s < steps; ++s) {
    // this thread's loads of slice s: the slice issued after it (if any) may
    // stay in flight, unless output stores were issued since
    if (stores_pending || s + 1 == steps) CAF_WAIT_VMCNT(0);
    else CAF_WAIT_VMCNT(LOADS);
    stores_pending = false;
    barrier_no_fence();  // every wave's slice s is in LDS, slice s - 1 is read
    if (s + NS - 1 < steps) issue(s + NS - 1);
    compute(s);
    if (s % nk == nk - 1) {
      uint32_t tm, tn;
      coords(tile0 + s / nk, tm, tn);
#pragma unroll
      for (uint32_t i = 0; i < WM; ++i)
#pragma unroll
        for (uint32_t jb = 0; jb < WN; ++jb)
          store_c<128>(Cg, n, tm * TM + wm * 64 + i * 32, tn * TN + wn * 128 + jb * 32, acc[i][jb]);
      zero_acc();
      stores_pending = true;
    }
  }
}


// ---------------------------------------------------------------------------
// Support behaviours (pipeline stages and ping-pong).
// ---------------------------------------------------------------------------
// A 16-byte write-through store (see store_reply) at byte `off` of the buffer
// `r`: bits 0 and 4 of the cache policy are sc0 and sc1.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t reply_buffer(void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(p, 0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ void store_reply16(__amdgpu_buffer_rsrc_t r, uint32_t off, u32x4 v) {
  __builtin_amdgcn_raw_buffer_store_b128(v, r, (int)off, 0, 17);
}

// Elements [base, base + len) of y = tanh(x), len <= 2^20.  HBM-bound: 16-byte
// loads and stores, two of each in flight per thread (8192 x 4100 through
// this and the row sums: 583 -> 284 us, 127 with the tiles now chosen).
__device__ __forceinline__ void tanh_range(const float* __restrict__ x, float* __restrict__ y,
                                           uint64_t base, uint32_t len) {
  const auto xg = global_ptr(x + base);
  const auto yb = reply_buffer(y + base, len * 4u);
  constexpr uint32_t U = 2, STEP = kThreads * 4;
  const uint32_t whole = len / (U * STEP) * (U * STEP);
  for (uint32_t e0 = threadIdx.x * 4; e0 < whole; e0 += U * STEP) {
    f32x4u v[U];
#pragma unroll
    for (uint32_t u = 0; u < U; ++u)
      v[u] = *reinterpret_cast<const CAF_GLOBAL f32x4u*>(xg + e0 + u * STEP);
#pragma unroll
    for (uint32_t u = 0; u < U; ++u) {
      f32x4u r;
#pragma unroll
      for (int c = 0; c < 4; ++c) r[c] = tanhf(v[u][c]);
      store_reply16(yb, (e0 + u * STEP) * 4u, __builtin_bit_cast(u32x4, r));
    }
  }
  for (uint32_t e = whole + threadIdx.x; e < len; e += kThreads)
    store_reply(global_ptr(y + base) + e, tanhf(xg[e]));
}

// Row sums of the `rows` rows of `cols` columns at x (far fewer than 2^32: a
// work tile's); kTanh: of the elements' tanh.  HBM-bound: 16-byte loads, R of them in flight per lane.  A
// row belongs to as many lanes (a power of two) as have a vector of it, so
// that short rows leave none idle (a chain's 128 x 128 matrix: 80 us as two
// passes, one row at a time; 52 in one pass, a row per wave); a lane sums its
// vectors in four chains, then the row's lanes meet in a tree.
template <bool kTanh, uint32_t R>
__device__ __forceinline__ void rowsum_rows(const float* __restrict__ x, float* __restrict__ y,
                                            uint32_t rows, uint32_t cols) {
  const uint32_t lane = lane_id();
  const auto xg = global_ptr(x);
  auto f = [](float v) { return kTanh ? tanhf(v) : v; };
  uint32_t per = 64;  // lanes per row
  while (per > 4 && per * 2 >= cols) per /= 2;
  const uint32_t l = lane & (per - 1u), step = 64 / per, whole = cols & ~3u;
  for (uint32_t rw = wave_id() * (R * step); rw < rows; rw += 4 * R * step) {
    const uint32_t r = rw + lane / per;  // this lane's rows: r, r + step, ...
    f32x4u s[R];
#pragma unroll
    for (uint32_t k = 0; k < R; ++k) s[k] = f32x4u{0.f, 0.f, 0.f, 0.f};
    for (uint32_t c = l * 4; c < whole; c += per * 4) {
      f32x4u v[R];
#pragma unroll
      for (uint32_t k = 0; k < R; ++k) {  // rows past the last: the last again
        const uint64_t row = min(r + k * step, rows - 1u);
        v[k] = *reinterpret_cast<const CAF_GLOBAL f32x4u*>(xg + row * cols + c);
      }
#pragma unroll
      for (uint32_t k = 0; k < R; ++k)
#pragma unroll
        for (int e = 0; e < 4; ++e) s[k][e] += f(v[k][e]);
    }
#pragma unroll
    for (uint32_t k = 0; k < R; ++k) {
      const uint64_t row = min(r + k * step, rows - 1u);
      float t = (s[k][0] + s[k][1]) + (s[k][2] + s[k][3]);
      if (l < (cols & 3u)) t += f(xg[row * cols + whole + l]);
      for (uint32_t off = per / 2; off > 0; off >>= 1) t += __shfl_xor(t, (int)off);
      if (l == 0 && r + k * step < rows) store_reply(y + r + k * step, t);
    }
  }
}

// The row actor with four vectors in flight, as calls: the full variants have
// the registers, but not in their drain loop.  The light variant inlines the
// same with one: a call in it costs its escape-time tiles 7%.
template <bool kTanh>
__device__ __noinline__ void rowsum_rows_call(const float* x, float* y, uint32_t rows,
                                              uint32_t cols) {
  rowsum_rows<kTanh, 4>(x, y, rows, cols);
}
template <bool kFull, bool kTanh>
__device__ __forceinline__ void rowsum_range(const float* x, float* y, uint32_t rows,
                                             uint32_t cols) {
  if constexpr (kFull) rowsum_rows_call<kTanh>(x, y, rows, cols);
  else rowsum_rows<kTanh, 1>(x, y, rows, cols);
}

__device__ __forceinline__ void tanh_tile(const Desc& d, uint32_t tile, uint32_t count) {
  const uint64_t ne = (uint64_t)d.p.s.rows * d.p.s.cols;
  const uint32_t te = tanh_tile_elems(d);
  const uint64_t base = (uint64_t)tile * te, end = base + (uint64_t)count * te;
  for (uint64_t b = base; b < end && b < ne; b += te)
    tanh_range(reinterpret_cast<const float*>(d.in0), reinterpret_cast<float*>(d.out), b,
               (uint32_t)min((uint64_t)te, ne - b));
}

template <bool kFull>
__device__ __forceinline__ void rowsum_tile(const Desc& d, uint32_t tile, uint32_t count) {
  const uint32_t tr = rowsum_tile_rows(d), r0 = tile * tr, cols = d.p.s.cols;
  const uint32_t rows = (uint32_t)min((uint64_t)count * tr, (uint64_t)(d.p.s.rows - r0));
  rowsum_range<kFull, false>(reinterpret_cast<const float*>(d.in0) + (uint64_t)r0 * cols,
                             reinterpret_cast<float*>(d.out) + r0, rows, cols);
}

__device__ void echo_tile(const Desc& d, uint8_t* inline_out) {
  const uint32_t n = d.numel;
  int32_t* dst = (d.flags & DF_INLINE_OUT) ? reinterpret_cast<int32_t*>(inline_out)
                                           : reinterpret_cast<int32_t*>(d.out);
  if (d.flags & DF_INLINE_IN) {
    // at most four values travel in the parameter block
    uint32_t w[4];
    __builtin_memcpy(w, d.p.raw, sizeof w);
    const uint32_t i = threadIdx.x;
    if (i < n)
      store_reply(dst + i, (int32_t)(i == 0 ? w[0] : i == 1 ? w[1] : i == 2 ? w[2] : w[3]));
    return;
  }
  const int32_t* src = reinterpret_cast<const int32_t*>(d.in0);
  for (uint32_t i = threadIdx.x; i < n; i += kThreads) store_reply(dst + i, src[i]);
}

}  // namespace cafgpu
