// Tile kernels of the tiled Householder QR and the persistent scheduler that
// runs them, for gfx950 (CDNA4).
//
// The six kernels of Algorithm 2 (GEQRT, UNMQR, TSQRT, TSMQR, TTQRT, TTMQR)
// work on b x b tiles in double precision with an inner blocking of 16:
// a panel of 16 columns is factored column by column (Householder
// reflectors, norms reduced across 16-lane groups), its compact-WY factor T
// (16 x 16, upper triangular) is formed, and the block reflector
// I - V T V^T is applied to the rest of the tile(s) with FP64 MFMA
// (v_mfma_f64_16x16x4f64).  The update kernels apply the 16-column panels of
// a finished factorization one after another with the V panels staged
// through LDS.
//
// Work split inside a workgroup (512 threads, 8 waves, one workgroup per CU
// so two waves share each SIMD): every wave owns a strip of 16 matrix
// columns and keeps the strip (b x 16 doubles) in registers as b/16 MFMA
// accumulators, so the reduction V^T C over the rows and the update
// C -= V W stay inside the wave; the waves only share the V panel and T in
// LDS.  An update task covers 128 columns (8 strips).  The column loop of
// the panel kernels runs on waves 0-3 (16 columns x 16 lanes).
//
// Register layout of an FP64 accumulator block (16 rows x 16 columns): lane
// l, element r holds MFMA row (l / 16) + 4 r, column l % 16.  Matrix rows
// are assigned to MFMA rows so that element r of lane l is matrix row
// 2 g + (r & 1) + 8 (r >> 1), g = l / 16: the four lane groups of a column
// cover its 16 rows as two contiguous 64-byte halves, each lane moving its
// rows with two 16-byte accesses (arow, roff).  The same permutation is
// applied to the reflector index of W = V^T C.
//
// V panels and T blocks go from memory straight into LDS (load_to_lds), the
// panel column-major: its operands in V^T C are then 16-byte LDS reads, the
// loads hold no registers, and no wave waits to copy them.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <type_traits>

#include "task.hpp"

namespace hqr {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef double d2 __attribute__((ext_vector_type(2)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f2 __attribute__((ext_vector_type(2)));

// Element type E of a factorization: double (FP64 MFMA) or float (FP32
// MFMA).  V4<E> is one MFMA accumulator block per lane, V2<E> a pair.
template <typename E> struct VecOf;
template <> struct VecOf<double> { typedef d4 v4; typedef d2 v2; };
template <> struct VecOf<float> { typedef f4 v4; typedef f2 v2; };
template <typename E> using V4 = typename VecOf<E>::v4;
template <typename E> using V2 = typename VecOf<E>::v2;

constexpr int IB = 16;      // inner blocking (columns per panel)
// LDS column stride of a staged panel (column-major): 16-byte aligned, and 16
// columns shift the banks by 4 words each, so that the 16-byte reads of one
// row pair (or quad) in 16 columns use every bank once.
template <typename E, int NB> constexpr int LDC = NB + 16 / (int)sizeof(E);
constexpr int LDZ = IB + 2; // LDS row stride of the products v_i^T v_j (16-byte aligned rows)
constexpr int NT = 512;     // threads per workgroup (8 waves, 2 per SIMD)

enum Kind { K_UNM = 0, K_TS = 1, K_TT = 2 };

__device__ __forceinline__ d4 mfma(double a, double b, d4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f4 mfma(float a, float b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// BF16 operands with FP32 accumulation (precision HQR_PREC_BF16): each
// operand is the float rounded to the nearest bfloat16 (ties to even); the
// product of two bfloat16 values is exact in FP32, where the matrix core
// accumulates.  One v_mfma_f32_16x16x16_bf16 takes four consecutive values
// of the reduction index per lane (lane l: index 4 (l / 16) + j, j < 4), the
// same four a lane feeds into four 16x16x4 FP32 products, so it replaces a
// group of four of them with the operands packed.
typedef short s4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ short bf16_bits(float x) {
  const uint32_t u = __builtin_bit_cast(uint32_t, x);
  return (short)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
}
__device__ __forceinline__ s4 bf16x4(float a, float b, float c, float d) {
  s4 r;
  r.x = bf16_bits(a);
  r.y = bf16_bits(b);
  r.z = bf16_bits(c);
  r.w = bf16_bits(d);
  return r;
}
__device__ __forceinline__ s4 bf16x4(const f4& v) { return bf16x4(v.x, v.y, v.z, v.w); }
__device__ __forceinline__ f4 mfma_bf(s4 a, s4 b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}

// Scalars of one Householder step from its head alpha and the squared norm
// ss > 0 of its tail: n = sqrt(alpha^2 + ss), 1 / (2 n) and 1 / (|alpha| + n).
// The hardware estimates (v_rsq, v_rcp) are refined to the working precision;
// the arguments are positive normal numbers, so no range scaling is needed.
//   g ~ n and h ~ 1 / (2 n) take one step together (Goldschmidt, FP64 2^-24
//   -> 2^-47), g one from its residual q - g^2, then h one with the new g;
//   the reciprocal starts from the first estimate of n, so that its latency
//   hides behind the refinement, and takes Newton steps r <- r + r (1 - d r)
//   with the refined d = |alpha| + n (two from 2^-23 in FP64, one in FP32).
template <typename E>
struct HouseScalars {
  E n, hn, rd;  // n, 1 / (2 n), 1 / (|alpha| + n)
};
__device__ __forceinline__ HouseScalars<double> house_scalars(double alpha, double ss) {
  const double q = fma(alpha, alpha, ss);
  const double y = __builtin_amdgcn_rsq(q);
  double g = q * y, h = 0.5 * y;
  double rd = __builtin_amdgcn_rcp(__builtin_fabs(alpha) + g);
  double r = fma(-g, h, 0.5);
  g = fma(g, r, g);
  h = fma(h, r, h);
  g = fma(fma(-g, g, q), h, g);
  r = fma(-g, h, 0.5);
  h = fma(h, r, h);
  const double dn = __builtin_fabs(alpha) + g;
  rd = fma(rd, fma(-dn, rd, 1.0), rd);
  rd = fma(rd, fma(-dn, rd, 1.0), rd);
  return {g, h, rd};
}
__device__ __forceinline__ HouseScalars<float> house_scalars(float alpha, float ss) {
  const float q = fmaf(alpha, alpha, ss);
  const float y = __builtin_amdgcn_rsqf(q);
  float g = q * y, h = 0.5f * y;
  float rd = __builtin_amdgcn_rcpf(__builtin_fabsf(alpha) + g);
  const float r = fmaf(-g, h, 0.5f);
  g = fmaf(g, r, g);
  h = fmaf(h, r, h);
  g = fmaf(fmaf(-g, g, q), h, g);
  const float dn = __builtin_fabsf(alpha) + g;
  rd = fmaf(rd, fmaf(-dn, rd, 1.0f), rd);
  return {g, h, rd};
}
// x with its sign bit flipped when `a`'s is set.
__device__ __forceinline__ double flip_sign(double x, double a) {
  const uint64_t u = __builtin_bit_cast(uint64_t, a) & (1ull << 63);
  return __builtin_bit_cast(double, __builtin_bit_cast(uint64_t, x) ^ u);
}
__device__ __forceinline__ float flip_sign(float x, float a) {
  const uint32_t u = __builtin_bit_cast(uint32_t, a) & (1u << 31);
  return __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, x) ^ u);
}

// Global-memory accessors for tile data inside the persistent launch.
//
// Tiles written by one workgroup are read by workgroups on other XCDs,
// whose L2 caches are not coherent with each other.  Agent-scope
// acquire/release fences would write back and invalidate a whole L2 at every
// task boundary; instead every tile access is a relaxed agent-scope access
// (coherent at device level on its own), and a task publishes its writes by
// waiting for its stores to complete before it bumps a dependency counter.
// The pointers are cast to the global address space: they reach the tile
// kernels through the task records, where the compiler would otherwise emit
// flat instructions (which also count against the LDS counter).
#ifndef HQR_GLOBAL_AS
#define HQR_GLOBAL_AS __attribute__((address_space(1)))
#endif
typedef HQR_GLOBAL_AS double gdouble;
typedef HQR_GLOBAL_AS float gfloat;

__device__ __forceinline__ double gload(const double* p) {
  return __hip_atomic_load((gdouble*)const_cast<double*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void gstore(double* p, double v) {
  __hip_atomic_store((gdouble*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float gload(const float* p) {
  return __hip_atomic_load((gfloat*)const_cast<float*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void gstore(float* p, float v) {
  __hip_atomic_store((gfloat*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ d2 gload2(const double* p) {
  d2 r;
  r.x = gload(p);
  r.y = gload(p + 1);
  return r;
}
__device__ __forceinline__ void gstore2(double* p, d2 v) {
  gstore(p, v.x);
  gstore(p + 1, v.y);
}

// Waits until this thread's global stores have completed.
__device__ __forceinline__ void stores_done() { __builtin_amdgcn_s_waitcnt(0); }

// 16-byte device-coherent accesses through a buffer resource: `base` is
// wave-uniform, `off` the element offset of this lane (< 2^28).
typedef unsigned int u4 __attribute__((ext_vector_type(4)));
constexpr int kCoherent = 16;  // cache policy bit: coherent at device scope
// FP64 tile loads and stores: device-coherent and non-temporal (a hint;
// with it the FP64 factorizations took 0.3-1% less time, the FP32 one 1.7%
// more, so float accesses keep the plain coherent policy).
constexpr int kTileAccess = kCoherent | 2;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const void* base) {
  // the base is wave-uniform by construction; say so, so that it lives in
  // scalar registers
  const uint64_t u = (uint64_t)base;
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)u);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(u >> 32));
  void* b = (void*)(((uint64_t)hi << 32) | lo);
  return __builtin_amdgcn_make_buffer_rsrc(b, 0, 0x7fffffff, 0x00020000);
}
typedef unsigned int u2 __attribute__((ext_vector_type(2)));

// Two consecutive elements at element offset `off` (16 bytes of double, 8
// of float) and four consecutive elements (two or one 16-byte accesses).
template <typename E>
__device__ __forceinline__ V2<E> bload2(__amdgpu_buffer_rsrc_t r, int off);
template <>
__device__ __forceinline__ d2 bload2<double>(__amdgpu_buffer_rsrc_t r, int off) {
  return __builtin_bit_cast(d2, __builtin_amdgcn_raw_buffer_load_b128(r, off * 8, 0, kTileAccess));
}
template <>
__device__ __forceinline__ f2 bload2<float>(__amdgpu_buffer_rsrc_t r, int off) {
  return __builtin_bit_cast(f2, __builtin_amdgcn_raw_buffer_load_b64(r, off * 4, 0, kCoherent));
}
__device__ __forceinline__ void bstore2(__amdgpu_buffer_rsrc_t r, int off, d2 v) {
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4, v), r, off * 8, 0, kTileAccess);
}
// One element at byte offset voff + soff (soff a wave-uniform constant),
// plain (non-coherent) load: for kernels that read what an earlier launch
// wrote.
template <typename E>
__device__ __forceinline__ E bload1(__amdgpu_buffer_rsrc_t r, int voff, int soff);
template <>
__device__ __forceinline__ double bload1<double>(__amdgpu_buffer_rsrc_t r, int voff, int soff) {
  return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
}
template <>
__device__ __forceinline__ float bload1<float>(__amdgpu_buffer_rsrc_t r, int voff, int soff) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
}
__device__ __forceinline__ f4 ld4(__amdgpu_buffer_rsrc_t r, int off) {
  return __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(r, off * 4, 0, kCoherent));
}
__device__ __forceinline__ void st4(__amdgpu_buffer_rsrc_t r, int off, f4 v) {
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4, v), r, off * 4, 0, kCoherent);
}

// One DPP step on a double: each lane receives the value of the lane picked
// by `ctrl` inside its row of 16 lanes.
template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const int lo = __builtin_amdgcn_mov_dpp((int)(uint32_t)u, CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(uint32_t)(u >> 32), CTRL, 0xf, 0xf, true);
  return __builtin_bit_cast(double, ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
}

// Reads lane `lane` (wave-uniform) of a double held in VGPRs.
__device__ __forceinline__ float readlane(float v, int lane) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
}
__device__ __forceinline__ double readlane(double v, int lane) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, lane);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), lane);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// The value that lane `lane` of the wave holds (any lane may ask for any).
__device__ __forceinline__ float lane_value(float v, int lane) {
  return __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(lane << 2, __builtin_bit_cast(int, v)));
}
__device__ __forceinline__ double lane_value(double v, int lane) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const int lo = __builtin_amdgcn_ds_bpermute(lane << 2, (int)(uint32_t)u);
  const int hi = __builtin_amdgcn_ds_bpermute(lane << 2, (int)(uint32_t)(u >> 32));
  return __builtin_bit_cast(double, ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
}

// Sums over the 16 lanes of a DPP row, returned in every lane of the row.
// Each step adds two partial sums in an order that does not depend on the
// lane (addition is commutative), so all 16 lanes hold bitwise the same sum.
// The two sums' steps are interleaved: each one's depend on each other, so
// the second fills the first one's latency.
template <typename E>
__device__ __forceinline__ void sum16x2(E& a, E& b) {
  E ta = dpp<0xB1>(a), tb = dpp<0xB1>(b);
  a += ta;
  b += tb;
  ta = dpp<0x4E>(a), tb = dpp<0x4E>(b);
  a += ta;
  b += tb;
  ta = dpp<0x124>(a), tb = dpp<0x124>(b);
  a += ta;
  b += tb;
  ta = dpp<0x128>(a), tb = dpp<0x128>(b);
  a += ta;
  b += tb;
}

// Workgroup barrier that orders LDS accesses only: global stores still in
// flight are not waited for (the data they carry is not read by another
// wave before a full barrier).
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

constexpr int kSlots = 4;  // staged panels in LDS

template <typename E, int NB>
struct Smem {
  // slots for staged V panels (column-major, stride LDC) and T blocks
  // (column-major, sq_at): the update tasks stage three panels ahead through
  // all four, the panel tasks one ahead through the first two.  In the panel
  // tasks' column loop V[0] hands the panel over and V[1] holds the published
  // columns.
  E V[kSlots][IB * LDC<E, NB>];
  E T[kSlots][IB * IB];
  // killer rows of a strip that the next panel updates (sq_at): one block per
  // wave of an update task; panel tasks: two per strip, by panel parity
  E C1[8][IB * IB];
  E C1r[2][IB * IB];  // the same for the row-split updates of one or two strips
  // panel tasks: each wave's part of W = V^T C of its strip, in the last two V
  // slots
  static_assert(2 * sizeof(E) * IB * LDC<E, NB> >= 8 * 64 * sizeof(V4<E>), "x does not fit in V slots 2-3");
  __device__ V4<E>* x() { return reinterpret_cast<V4<E>*>(V[2]); }
  E Z[IB * LDZ];     // products v_i^T v_j of the panel's reflectors (row j), for T
  E tau[IB];
  alignas(8) int wide[2];  // panel tasks: whether a panel has columns outside the range of raw products
  int task;  // index of the task taken by the workgroup (-1: launch aborted)
  int next;  // the following task index, taken ahead by finish_task (-2: none)
  int ok;    // 1 if the task's dependencies were met, 0 if the launch was aborted
};

// The scheduler's shared state and the tile kernels' staging buffers live in
// the launch's dynamic LDS.
extern __shared__ __attribute__((aligned(16))) double hqr_lds[];

template <typename E, int NB>
__device__ __forceinline__ Smem<E, NB>& smem() {
  // the base is read once: a function that is not inlined looks the offset of
  // dynamic LDS up in a table, which the compiler would otherwise repeat
  // inside the loops (a scalar load each time)
  typedef __attribute__((address_space(3))) char lchar;
  uint32_t b = (uint32_t)(uintptr_t)(lchar*)hqr_lds;
  __asm__("" : "+s"(b));
  return *reinterpret_cast<Smem<E, NB>*>((char*)(lchar*)(uintptr_t)b);
}

// Byte offset of an LDS object inside the workgroup's allocation.
__device__ __forceinline__ uint32_t lds_offset(const void* q) {
  typedef __attribute__((address_space(3))) const char lchar;
  return (uint32_t)(uintptr_t)(lchar*)q;
}

// A 16 x 16 block in LDS (T, C1) is column-major with each column's 16-byte
// units permuted by an exclusive or with bits of the column number, so that
// reading one unit of all 16 columns uses every bank once (unpermuted they
// share two or four banks: 900 cycles a panel, more than the products of T).
// sq_unit: the unit stored in place `u` of column c; sq_at: where element
// (i, c) is.
template <typename E>
__device__ __forceinline__ int sq_unit(int u, int c) {
  return sizeof(E) == 8 ? u ^ ((c >> 1) & 7) : u ^ ((c >> 2) & 3);
}
template <typename E>
__device__ __forceinline__ int sq_at(int i, int c) {
  constexpr int VW = 16 / (int)sizeof(E);
  return c * IB + VW * sq_unit<E>(i / VW, c) + i % VW;
}

// 16 bytes per lane from the buffer at byte offset `voff` straight into LDS
// at `lds` + 16 * lane (wave-uniform `lds`), device-coherent (without the
// non-temporal hint of the chunk's accesses: V and T are read by many
// workgroups, and with it UNM took 119 instead of 105 us); completion is
// counted in vmcnt (loads_left).  Issued as an instruction of its own: no
// register carries the data, and the compiler, which does not see the write,
// adds no wait in front of LDS reads of the other slot.  It does not see a
// vector memory instruction either, so the wait states that it would insert
// are part of the text: the resource words come from v_readfirstlane (rsrc),
// and such a read of a scalar register that a vector instruction wrote must be
// five wait states behind it (s_mov one, s_nop 3 four; the hardware does not
// check).  m0, read as the LDS address, needs one.  Naming m0 as overwritten
// keeps the compiler's own uses of it apart (it warns that it reserves m0).
__device__ __forceinline__ void load_to_lds(__amdgpu_buffer_rsrc_t r, int voff, uint32_t lds) {
  const uint32_t m = (uint32_t)__builtin_amdgcn_readfirstlane((int)lds);
  __asm__ __volatile__("s_mov_b32 m0, %0\n\ts_nop 3\n\tbuffer_load_dwordx4 %1, %2, 0 offen sc1 lds"
                       :
                       : "s"(m), "v"(voff), "s"(r)
                       : "memory", "m0");
}
// Waits until at most N of this wave's vector memory operations are left.
template <int N>
__device__ __forceinline__ void loads_left() {
  __asm__ __volatile__("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory");
}

// Waits for all of them with an instruction the compiler knows: it takes the
// loads it has issued itself for arrived.  For use ahead of a loop over panels
// that starts with data loaded in front of it: otherwise the compiler waits for
// that data at its first use in every iteration, not in the first alone, and
// so for whatever staging loads are in flight by then.
__device__ __forceinline__ void loads_done() { __builtin_amdgcn_s_waitcnt(0x0f70); }  // vmcnt(0)

// Lane coordinates.
struct Lane {
  int wave, g, q, pq;
  __device__ Lane() {
    const int t = threadIdx.x;
    wave = __builtin_amdgcn_readfirstlane(t >> 6);
    g = (t >> 4) & 3;
    q = t & 15;
    pq = 2 * (q & 3) + ((q >> 2) & 1) + 8 * (q >> 3);
  }
};

// Rows of a 16 x 16 block held in an MFMA accumulator.  Element r of lane
// (g, q) (g = lane / 16, q = lane % 16) holds column q and the matrix row
// arow + roff(r):
//     FP64: 2g + (r & 1) + 8 (r >> 1)   (rows 2g, 2g+1, 2g+8, 2g+9)
//     FP32: 4g + r
// FP32 accumulators hold MFMA row 4g + r, so its map is the identity.  The
// FP64 accumulator holds MFMA row g + 4r (measured on gfx950); matrix row x
// then sits at MFMA row pi^-1(x) with pi(g + 4r) = 2g + (r & 1) + 8 (r >> 1),
// and mrow is the row that lane q supplies as MFMA row q.  Either way the
// four lanes of a column cover its 16 rows as two contiguous 64-byte halves
// (FP64: two 16-byte accesses per lane) or one 64-byte run (FP32), so each
// access instruction writes whole segments (with four consecutive FP64 rows
// per lane the lanes of a column interleave at a 32-byte stride, which took
// twice as long to store), and the operands of V^T C are 16-byte LDS reads of
// the column-major panel.
template <typename E>
__device__ __forceinline__ int arow(const Lane& L) {  // row of element 0
  return sizeof(E) == 8 ? 2 * L.g : 4 * L.g;
}
template <typename E>
__device__ __forceinline__ int roff(int r) {  // row of element r minus that of element 0
  return sizeof(E) == 8 ? (r & 1) + 8 * (r >> 1) : r;
}
template <typename E>
__device__ __forceinline__ int mrow(const Lane& L) {
  return sizeof(E) == 8 ? L.pq : L.q;
}

// One column's four rows of a 16-row block in accumulator order: `off` is
// the element offset of the block's row 0 in that column.
template <typename E>
__device__ __forceinline__ V4<E> ldblk(__amdgpu_buffer_rsrc_t r, int off, const Lane& L);
template <>
__device__ __forceinline__ d4 ldblk<double>(__amdgpu_buffer_rsrc_t r, int off, const Lane& L) {
  const d2 x = bload2<double>(r, off + 2 * L.g);
  const d2 y = bload2<double>(r, off + 2 * L.g + 8);
  d4 v;
  v.x = x.x; v.y = x.y; v.z = y.x; v.w = y.y;
  return v;
}
template <>
__device__ __forceinline__ f4 ldblk<float>(__amdgpu_buffer_rsrc_t r, int off, const Lane& L) {
  return ld4(r, off + 4 * L.g);
}
__device__ __forceinline__ void stblk(__amdgpu_buffer_rsrc_t r, int off, const Lane& L, d4 v) {
  d2 x, y;
  x.x = v.x; x.y = v.y; y.x = v.z; y.y = v.w;
  bstore2(r, off + 2 * L.g, x);
  bstore2(r, off + 2 * L.g + 8, y);
}
__device__ __forceinline__ void stblk(__amdgpu_buffer_rsrc_t r, int off, const Lane& L, f4 v) {
  st4(r, off + 4 * L.g, v);
}

// Blocks 2b and 2b + 1 of a strip (32 rows from row 32b); `off` is the
// element offset of the strip's row 0 in the lane's column.
template <typename V>
__device__ __forceinline__ void ldpair(__amdgpu_buffer_rsrc_t rs, int off, int b, const Lane& L, V& lo, V& hi) {
  typedef decltype(lo.x + lo.x) E;
  lo = ldblk<E>(rs, off + 32 * b, L);
  hi = ldblk<E>(rs, off + 32 * b + 16, L);
}
template <typename V>
__device__ __forceinline__ void stpair(__amdgpu_buffer_rsrc_t rs, int off, int b, const Lane& L, const V& lo,
                                       const V& hi) {
  stblk(rs, off + 32 * b, L, lo);
  stblk(rs, off + 32 * b + 16, L, hi);
}

// ---------------------------------------------------------------------------
// Block-reflector application of one panel to one 16-column strip held by a
// wave.  `acc` holds rows 0..NB-1 of the strip of the matrix the reflectors
// act on below the identity part (C2 for TS/TT, C itself for UNM).  `c1` is
// the strip of the killer tile (rows 16p..16p+15) for TS/TT, or null.
//
//   W  = V_p^T acc (+ C1_p)      reduction over the active rows
//   W  = T_p^T W                  (T_p W when applying Q instead of Q^T)
//   C1_p -= W,   acc -= V_p W
//
// Active rows: UNM rows >= 16p (V unit lower triangular), TS all rows
// (V dense), TT rows < 16p + 16 (V upper triangular), in pairs of 16-row
// blocks (staging completes the pair that holds the diagonal block with
// zeros).
template <int KIND>
__device__ __forceinline__ bool pair_active(int b, int p) {
  return (KIND == K_UNM) ? (b >= (p >> 1)) : (KIND == K_TT ? b <= (p >> 1) : true);
}
// The block of the pair with the diagonal block that is all zeros (the one
// above it for UNM, the one below for TT).
template <int KIND>
__device__ __forceinline__ bool zero_block(int rb, int p) {
  return KIND != K_TS && (rb ^ 1) == p && (KIND == K_UNM) == ((p & 1) != 0);
}

// Staging of V panel p (columns 16p .. 16p+15 of tile `V`) and its T block
// into an LDS slot: wave w loads columns 2w and 2w+1 in pieces of up to 1 KB
// and an eighth of T.  Every wave issues OPS loads whatever the panel, so that
// loads_left can name those of one panel while later ones are in flight.  The
// pieces are issued one by one between the products of the panel before
// (`group` of the G pairs of row blocks).
template <typename E, int NB, int KIND>
struct Stage {
  __amdgpu_buffer_rsrc_t rv, rt;
  uint32_t lv, lt;
  int voff;
  bool on;
  static constexpr int CB = NB * (int)sizeof(E);        // bytes of a column
  static constexpr int PIECES = CB > 1024 ? CB / 1024 : 1;
  static constexpr int P = 2 * PIECES;
  static constexpr int OPS = P + 1;
  __device__ __forceinline__ Stage(const E* V, const E* Tblk, E* Vs, E* Ts, int panel, bool active, const Lane& L)
      : rv(rsrc(V)), rt(rsrc(Tblk)), lv(lds_offset(Vs) + 2 * L.wave * LDC<E, NB> * (int)sizeof(E)),
        lt(lds_offset(Ts) + 2 * L.wave * IB * (int)sizeof(E)), voff((16 * panel + 2 * L.wave) * CB + 16 * (threadIdx.x & 63)),
        on(active) {}
  __device__ __forceinline__ void piece(int i, const Lane& L) const {
    const int c = i / PIECES, h = i % PIECES, lane = threadIdx.x & 63;
    if (CB >= 1024 || 16 * lane < CB)
      load_to_lds(rv, voff + c * CB + 1024 * h, lv + c * LDC<E, NB> * (int)sizeof(E) + 1024 * h);
    if (i == 0) {
      constexpr int UC = IB * (int)sizeof(E) / 16;  // units per column of T: this wave's two columns
      if (lane < 2 * UC) {
        const int col = 2 * L.wave + lane / UC;
        load_to_lds(rt, 16 * (col * UC + sq_unit<E>(lane % UC, col)), lt);
      }
    }
  }
  template <int G>
  __device__ __forceinline__ void group(int b, const Lane& L) const {
    if (on) {
#pragma unroll
      for (int i = b * P / G; i < (b + 1) * P / G; ++i) piece(i, L);
    }
  }
  __device__ __forceinline__ void all(const Lane& L) const { group<1>(0, L); }
};

// Completes the staging of panel p once the wave's loads have arrived
// (loads_left): the pair of blocks that holds the diagonal block takes the
// structure of the kind in the wave's columns (UNM: unit diagonal, zeros
// above it; TT: zeros below it).  A workgroup barrier must follow.
template <typename E, int NB, int KIND>
__device__ __forceinline__ void stage_finish(E* Vs, int p) {
  if (KIND != K_TS) {
    const int col = threadIdx.x >> 5, r = threadIdx.x & 31;
    E* e = Vs + col * LDC<E, NB> + 32 * (p >> 1) + r;
    const int a = r - 16 * (p & 1);  // row minus the panel's first row
    if (KIND == K_UNM && a <= col) *e = (a == col) ? E(1) : E(0);
    if (KIND == K_TT && a > col) *e = E(0);
  }
}

// Killer rows of one panel (16 rows x 16 columns at `c1`, leading dimension
// NB) of the wave's strip straight into its LDS block.  They are loaded a
// panel ahead like V: an ordinary load would make the compiler wait, at its
// use, for every staging load issued after it.
template <typename E, int NB>
__device__ __forceinline__ void c1_start(const E* c1, E* dst) {
  constexpr int LPC = IB * (int)sizeof(E) / 16;  // lanes per column
  const int lane = threadIdx.x & 63;
  const __amdgpu_buffer_rsrc_t r = rsrc(c1);
  const uint32_t l = lds_offset(dst);
#pragma unroll
  for (int h = 0; h < LPC / 4; ++h) {
    const int c = h * (64 / LPC) + lane / LPC;
    load_to_lds(r, c * NB * (int)sizeof(E) + 16 * sq_unit<E>(lane % LPC, c), l + 1024 * h);
  }
}
__device__ __forceinline__ d4 c1_read(const double* c1, const Lane& L) {
  const d2 x = *reinterpret_cast<const d2*>(c1 + sq_at<double>(2 * L.g, L.q));
  const d2 y = *reinterpret_cast<const d2*>(c1 + sq_at<double>(2 * L.g + 8, L.q));
  return d4{x.x, x.y, y.x, y.y};
}
__device__ __forceinline__ f4 c1_read(const float* c1, const Lane& L) {
  return *reinterpret_cast<const f4*>(c1 + sq_at<float>(4 * L.g, L.q));
}
// vector memory operations per panel and wave after the staging loads of the
// next one: the C1 stores and the loads of the next C1
template <typename E, int KIND> constexpr int C1OPS = KIND == K_UNM ? 0 : (sizeof(E) == 8 ? 4 : 2);

// LDS operands of one pair of blocks: eight products.
template <typename E> struct PairOps;
template <> struct PairOps<double> {
  d4 l, h;
  __device__ __forceinline__ double lo(int r) const { return l[r]; }
  __device__ __forceinline__ double hi(int r) const { return h[r]; }
  template <int LD>
  __device__ __forceinline__ void load_w(const double* Vs, int b, const Lane& L) {  // V^T: column mrow, the lane's rows
    const double* a = Vs + L.pq * LD + 2 * L.g + 32 * b;
    const d2 x = *reinterpret_cast<const d2*>(a), y = *reinterpret_cast<const d2*>(a + 8);
    const d2 u = *reinterpret_cast<const d2*>(a + 16), v = *reinterpret_cast<const d2*>(a + 24);
    l = d4{x.x, x.y, y.x, y.y};
    h = d4{u.x, u.y, v.x, v.y};
  }
  template <int LD>
  __device__ __forceinline__ void load_c(const double* Vs, int b, const Lane& L) {  // V: row mrow, the lane's columns
    const double* a = Vs + 2 * L.g * LD + L.pq + 32 * b;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      l[r] = a[roff<double>(r) * LD];
      h[r] = a[roff<double>(r) * LD + 16];
    }
  }
};
template <> struct PairOps<float> {
  f4 l, h;
  __device__ __forceinline__ float lo(int r) const { return l[r]; }
  __device__ __forceinline__ float hi(int r) const { return h[r]; }
  template <int LD>
  __device__ __forceinline__ void load_w(const float* Vs, int b, const Lane& L) {
    const float* a = Vs + L.q * LD + 4 * L.g + 32 * b;
    l = *reinterpret_cast<const f4*>(a);
    h = *reinterpret_cast<const f4*>(a + 16);
  }
  template <int LD>
  __device__ __forceinline__ void load_c(const float* Vs, int b, const Lane& L) {
    const float* a = Vs + 4 * L.g * LD + L.q + 32 * b;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      l[r] = a[r * LD];
      h[r] = a[r * LD + 16];
    }
  }
};

// The same for one 16-row block rb: V^T (column mrow, the lane's rows) and V
// (row mrow, the lane's columns).
template <int LD>
__device__ __forceinline__ d4 block_w(const double* Vs, int rb, const Lane& L) {
  const double* a = Vs + L.pq * LD + 2 * L.g + 16 * rb;
  const d2 x = *reinterpret_cast<const d2*>(a), y = *reinterpret_cast<const d2*>(a + 8);
  return d4{x.x, x.y, y.x, y.y};
}
template <int LD>
__device__ __forceinline__ f4 block_w(const float* Vs, int rb, const Lane& L) {
  return *reinterpret_cast<const f4*>(Vs + L.q * LD + 4 * L.g + 16 * rb);
}
template <int LD, typename E>
__device__ __forceinline__ V4<E> block_c(const E* Vs, int rb, const Lane& L) {
  const E* a = Vs + arow<E>(L) * LD + mrow<E>(L) + 16 * rb;
  V4<E> v;
#pragma unroll
  for (int r = 0; r < 4; ++r) v[r] = a[roff<E>(r) * LD];
  return v;
}

// The products are issued one pair of blocks at a time (eight), with the LDS
// operands of the next pair loaded before them; scheduling barriers keep the
// compiler from hoisting all operand loads at once, which would not fit next
// to the accumulators, and from sinking a pair's loads behind the products
// they are to overlap with (an LDS latency for every eight products).
// Consecutive MFMAs never write the same accumulator.  Each pair has operands
// of its own, loaded whether or not the pair is active: handed on in one
// variable, or loaded under a condition, every pair copied 16 registers (158
// moves in a panel of UNM, 278 of TT).
//
// First part: V_p^T acc in two partial sums, without the zero block of the
// diagonal pair (6% of the products of a triangular tile; in the third part
// a form without it brought the copies back).  At nb = 256, inside a
// factorization: TT 114 us with copies and zero blocks, 103 without copies,
// 101 without either; UNM 118 with and 112 without both.
template <typename E, int NB, int KIND, bool BF>
__device__ __forceinline__ V4<E> panel_w(const V4<E> (&acc)[NB / 16], const E* __restrict__ Vs, int p, const Lane& L,
                                         const Stage<E, NB, KIND>* next = nullptr) {
  static_assert(!BF || sizeof(E) == 4, "BF16 products take float tiles");
  constexpr int NP = NB / 32, LD = LDC<E, NB>;
  V4<E> w0 = {E(0), E(0), E(0), E(0)}, w1 = w0;
  PairOps<E> first, o[NP];
  first.template load_w<LD>(Vs, KIND == K_UNM ? p >> 1 : 0, L);
#pragma unroll
  for (int b = 0; b < NP; ++b) {
    if (next) next->template group<NP>(b, L);
    if (pair_active<KIND>(b, p)) {
      if (KIND == K_UNM ? b == (p >> 1) : b == 0) {
        o[b] = first;
        __asm__ __volatile__("");  // (a branch, not selects in every pair)
      }
      __builtin_amdgcn_sched_barrier(0);
      if (b + 1 < NP) o[b + 1].template load_w<LD>(Vs, b + 1, L);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (BF) {
        w0 = mfma_bf(bf16x4(o[b].l), bf16x4(acc[2 * b]), w0);
        w1 = mfma_bf(bf16x4(o[b].h), bf16x4(acc[2 * b + 1]), w1);
      } else if constexpr (KIND != K_TS) {
        if (!zero_block<KIND>(2 * b, p)) {
          w0 = mfma(o[b].lo(0), acc[2 * b][0], w0);
          w1 = mfma(o[b].lo(1), acc[2 * b][1], w1);
          w0 = mfma(o[b].lo(2), acc[2 * b][2], w0);
          w1 = mfma(o[b].lo(3), acc[2 * b][3], w1);
        }
        if (!zero_block<KIND>(2 * b + 1, p)) {
          w0 = mfma(o[b].hi(0), acc[2 * b + 1][0], w0);
          w1 = mfma(o[b].hi(1), acc[2 * b + 1][1], w1);
          w0 = mfma(o[b].hi(2), acc[2 * b + 1][2], w0);
          w1 = mfma(o[b].hi(3), acc[2 * b + 1][3], w1);
        }
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          w0 = mfma(o[b].lo(r), acc[2 * b][r], w0);
          w1 = mfma(o[b].hi(r), acc[2 * b + 1][r], w1);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  return w0 + w1;
}

// Second part: T^T w (T w when not TRANS), in two chains of two products;
// its LDS operands are loaded before the first part, whose end it follows
// with nothing to hide their latency behind.
template <typename E, bool TRANS>
__device__ __forceinline__ V4<E> panel_t_load(const E* __restrict__ Ts, const Lane& L) {
  V4<E> t;
#pragma unroll
  for (int r = 0; r < 4; ++r)
    t[r] = TRANS ? Ts[sq_at<E>(arow<E>(L) + roff<E>(r), mrow<E>(L))] : Ts[sq_at<E>(mrow<E>(L), arow<E>(L) + roff<E>(r))];
  return t;
}
template <typename E, bool BF>
__device__ __forceinline__ V4<E> panel_t(const V4<E>& w, const V4<E>& t) {
  V4<E> x0 = {E(0), E(0), E(0), E(0)};
  if constexpr (BF) {
    return mfma_bf(bf16x4(t), bf16x4(w), x0);
  } else {
    V4<E> x1 = x0;
    x0 = mfma(t[0], w[0], x0);
    x1 = mfma(t[1], w[1], x1);
    x0 = mfma(t[2], w[2], x0);
    x1 = mfma(t[3], w[3], x1);
    return x0 + x1;
  }
}

// Third part: acc += V_p wn; `a` holds the operands of the first active pair
// (loaded ahead like those of T).
template <typename E, int NB, int KIND>
__device__ __forceinline__ PairOps<E> panel_add_load(const E* __restrict__ Vs, int p, const Lane& L) {
  PairOps<E> a;
  a.template load_c<LDC<E, NB>>(Vs, KIND == K_UNM ? p >> 1 : 0, L);
  return a;
}
template <typename E, int NB, int KIND, bool BF>
__device__ __forceinline__ void panel_add(V4<E> (&acc)[NB / 16], const E* __restrict__ Vs, PairOps<E> a,
                                          const V4<E>& wn, int p, const Lane& L) {
  constexpr int NP = NB / 32, LD = LDC<E, NB>;
  PairOps<E> o[NP];
#pragma unroll
  for (int b = 0; b < NP; ++b) {
    if (pair_active<KIND>(b, p)) {
      if (KIND == K_UNM ? b == (p >> 1) : b == 0) {
        o[b] = a;
        __asm__ __volatile__("");
      }
      __builtin_amdgcn_sched_barrier(0);
      if (b + 1 < NP) o[b + 1].template load_c<LD>(Vs, b + 1, L);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (BF) {
        const s4 wb = bf16x4(wn);
        acc[2 * b] = mfma_bf(bf16x4(o[b].l), wb, acc[2 * b]);
        acc[2 * b + 1] = mfma_bf(bf16x4(o[b].h), wb, acc[2 * b + 1]);
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          acc[2 * b] = mfma(o[b].lo(r), wn[r], acc[2 * b]);
          acc[2 * b + 1] = mfma(o[b].hi(r), wn[r], acc[2 * b + 1]);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

// Applies panel p (staged in Vs, Ts; the killer rows in c1s) while `next`, a
// later panel, is staged; c1 and c1n: the killer rows of this panel and of the
// next one (null: none).
template <typename E, int NB, int KIND, bool TRANS = true, bool BF = false>
__device__ __forceinline__ void apply_panel(V4<E> (&acc)[NB / 16], const E* __restrict__ Vs,
                                            const E* __restrict__ Ts, E* c1s, int p, E* c1, const E* c1n,
                                            const Lane& L, const Stage<E, NB, KIND>& next) {
  const V4<E> t = panel_t_load<E, TRANS>(Ts, L);
  V4<E> w = panel_w<E, NB, KIND, BF>(acc, Vs, p, L, &next);
  const PairOps<E> a = panel_add_load<E, NB, KIND>(Vs, p, L);
  V4<E> c1v = {E(0), E(0), E(0), E(0)};
  if (KIND != K_UNM) {
    // this panel's killer rows are older than the staging loads issued above
    if (next.on)
      loads_left<Stage<E, NB, KIND>::OPS>();
    else
      loads_left<0>();
    c1v = c1_read(c1s, L);
    w += c1v;
  }
  const V4<E> w2 = panel_t<E, BF>(w, t);
  if (KIND != K_UNM) {
    stblk(rsrc(c1), L.q * NB, L, c1v - w2);
    if (c1n) c1_start<E, NB>(c1n, c1s);
  }
  panel_add<E, NB, KIND, BF>(acc, Vs, a, -w2, p, L);
}

// ---------------------------------------------------------------------------
// Update task: a chunk of 64 or 128 columns of UNMQR / TSMQR / TTMQR, bounded
// by the FP64 matrix cores (TSMQR: 115 us of products per 128 columns at
// nb = 256).  With V staged through registers into a row-major panel a TSMQR
// took 152 us alone on every CU and 81 us in FP32, with the loads into LDS
// 147 and 73 us.  Inside a factorization (16384 x 8192, Greedy): UNMQR 113 ->
// 106 us, TTMQR 107 -> 102.  Loading only the rows of V that a triangular
// panel has made no difference.
//   V, T: the factored tile and its T (block column nb x 16).
//   C2: tile updated below the identity part (UNM: the tile itself).
//   C1: killer tile (TS/TT).
// TRANS applies Q^T (the panels in factorization order, T^T); otherwise Q
// (the panels in reverse order, T).  Only the first np panels are applied:
// the panels after them are identities (T = 0, the zero padding beyond the
// last matrix column of a ragged tile column).
template <typename E, int NB, int KIND, bool TRANS, bool BF = false>
__device__ __forceinline__ void run_update(Smem<E, NB>& sm, const E* V, const E* T, E* C1, E* C2,
                                           int64_t ld, int strips, int np = NB / IB) {
  const int NP = __builtin_amdgcn_readfirstlane(np);
  const Lane L;
  V4<E> acc[NB / 16];
  const int64_t coloff = (int64_t)(16 * L.wave) * ld;
  // Panel it + 3 is loaded while panel it is applied, into the slot that
  // panel it - 1 was read from (every wave finished that before the last
  // barrier).  Three panels ahead because a panel of the triangular kinds can
  // have a single pair of row blocks left, far less work than a load's latency,
  // and the copies do not wait for each other's round trips.
  auto pan = [&](int it) { return TRANS ? it : NP - 1 - it; };
  auto stage = [&](int it) {
    return Stage<E, NB, KIND>(V, T + pan(it) * 256, sm.V[it & 3], sm.T[it & 3], pan(it), it < NP, L);
  };
  constexpr int LOADS = NB / 16 * (sizeof(E) == 8 ? 2 : 1);  // of the chunk, per wave
  constexpr int S = Stage<E, NB, KIND>::OPS;
  E* c1 = KIND == K_UNM ? nullptr : C1 + coloff;
  const bool on = L.wave < strips;  // waves holding a strip of the chunk (uniform per wave)
  stage(0).all(L);
  if (KIND != K_UNM && on) c1_start<E, NB>(c1 + 16 * pan(0), sm.C1[L.wave]);
  stage(1).all(L);
  stage(2).all(L);
  // the chunk is loaded last: the first panel's products take its row
  // blocks in order as they arrive
  const __amdgpu_buffer_rsrc_t rc2 = rsrc(C2 + coloff);
#pragma unroll
  for (int b = 0; b < NB / 32; ++b)
    if (on) ldpair(rc2, L.q * (int)ld, b, L, acc[2 * b], acc[2 * b + 1]);
  // UNM waits for it before the loop (112 -> 106 us); TS and TT do not: their
  // killer rows have to be waited for in each panel anyway (with the wait in
  // front TT took 102.5 instead of 100.7 us, TS the same)
  if (KIND == K_UNM)
    loads_done();
  else if (on)
    loads_left<2 * S + LOADS>();
  else
    loads_left<2 * S>();
  stage_finish<E, NB, KIND>(sm.V[0], pan(0));
  lds_barrier();
#pragma unroll 1
  for (int it = 0; it < NP; ++it) {
    const int sl = it & 3, p = pan(it);
    // operations newer than the staging of panel it + 1 at its wait: the
    // staging of up to two later panels and (waves holding a strip) the C1
    // traffic of three panels
    if (on) {
      constexpr int C = 3 * C1OPS<E, KIND>;
      apply_panel<E, NB, KIND, TRANS, BF>(acc, sm.V[sl], sm.T[sl], sm.C1[L.wave], p, c1 + 16 * p,
                                          KIND != K_UNM && it + 1 < NP ? c1 + 16 * pan(it + 1) : nullptr, L,
                                          stage(it + 3));
      if (it + 3 < NP)
        loads_left<2 * S + C>();
      else if (it + 3 == NP)
        loads_left<S + C>();
      else
        loads_left<C>();
    } else {
      stage(it + 3).all(L);
      if (it + 3 < NP)
        loads_left<2 * S>();
      else if (it + 3 == NP)
        loads_left<S>();
      else
        loads_left<0>();
    }
    if (it + 1 < NP) stage_finish<E, NB, KIND>(sm.V[(it + 1) & 3], pan(it + 1));
    lds_barrier();
  }
#pragma unroll
  for (int b = 0; b < NB / 32; ++b)
    if (on) stpair(rc2, L.q * (int)ld, b, L, acc[2 * b], acc[2 * b + 1]);
}

// The same update for a chunk with at most S (1 or 2) live 16-column strips:
// a few right-hand sides, or the last columns of a ragged matrix.  One strip
// per wave would leave most waves idle, each panel's chain of products
// (row blocks, T, row blocks) running on one of them.  Here the row blocks of
// a strip are dealt to 8 / S waves: each forms its rows' part of W, all add
// the parts in the same order and form T^T W, and each updates its rows.
// Bounded by the latency of that chain (two barriers per panel); V is staged
// as in run_update.
template <typename E, int NB, int KIND, bool TRANS, bool BF, int S>
__device__ __forceinline__ void run_update_rows(Smem<E, NB>& sm, const E* V, const E* T, E* C1, E* C2, int strips,
                                                int np = NB / IB) {
  constexpr int RS = 8 / S, NBW = NB / 16 > RS ? NB / 16 / RS : 1, LD = LDC<E, NB>;
  constexpr int RING = S == 1 ? 2 : 1;  // killer-row blocks per strip
  constexpr int OPS = Stage<E, NB, KIND>::OPS;
  static_assert(sizeof(sm.C1) >= 8 * 64 * sizeof(V4<E>), "the parts of W do not fit in C1");
  const int NP = __builtin_amdgcn_readfirstlane(np);
  const Lane L;
  const int lane = threadIdx.x & 63;
  const int j = L.wave % S, rp = L.wave / S;  // strip and row part
  const bool on = j < strips;
  const bool keeps = KIND != K_UNM && on && rp == 0;  // loads and stores the strip's killer rows
  V4<E>* X = reinterpret_cast<V4<E>*>(sm.C1[0]);
  auto pan = [&](int it) { return TRANS ? it : NP - 1 - it; };
  auto stage = [&](int it) {
    return Stage<E, NB, KIND>(V, T + pan(it) * 256, sm.V[it & 3], sm.T[it & 3], pan(it), it < NP, L);
  };
  E* c1 = KIND == K_UNM ? nullptr : C1 + (int64_t)(16 * j) * NB;
  auto c1_block = [&](int it) { return sm.C1r[S == 1 ? (it & 1) : j]; };
  auto c1_load = [&](int it) {
    if (keeps && it < NP) c1_start<E, NB>(c1 + 16 * pan(it), c1_block(it));
  };
  const __amdgpu_buffer_rsrc_t rc2 = rsrc(C2 + (int64_t)(16 * j) * NB);
  V4<E> acc[NBW];
  stage(0).all(L);
  c1_load(0);
  if (RING > 1) c1_load(1);
  stage(1).all(L);
  stage(2).all(L);
#pragma unroll
  for (int i = 0; i < NBW; ++i)
    if (on && rp + RS * i < NB / 16) acc[i] = ldblk<E>(rc2, 16 * (rp + RS * i) + L.q * NB, L);
  loads_done();
  stage_finish<E, NB, KIND>(sm.V[0], pan(0));
  lds_barrier();
#pragma unroll 1
  for (int it = 0; it < NP; ++it) {
    const int p = pan(it);
    const E* Vs = sm.V[it & 3];
    auto active = [&](int rb) {
      return on && rb < NB / 16 && ((KIND == K_UNM) ? rb >= p : (KIND == K_TT ? rb <= p : true));
    };
    V4<E> w0 = {E(0), E(0), E(0), E(0)}, w1 = w0;
#pragma unroll
    for (int i = 0; i < NBW; ++i) {
      const int rb = rp + RS * i;
      if (active(rb)) {
        const V4<E> a = block_w<LD>(Vs, rb, L);
        if constexpr (BF) {
          w0 = mfma_bf(bf16x4(a), bf16x4(acc[i]), w0);
        } else {
          w0 = mfma(a[0], acc[i][0], w0);
          w1 = mfma(a[1], acc[i][1], w1);
          w0 = mfma(a[2], acc[i][2], w0);
          w1 = mfma(a[3], acc[i][3], w1);
        }
      }
    }
    if (on) X[L.wave * 64 + lane] = w0 + w1;
    // panel it + 1 and this panel's killer rows: everything older than the
    // staging of panel it + 2
    if (it + 2 < NP)
      loads_left<OPS>();
    else
      loads_left<0>();
    if (it + 1 < NP) stage_finish<E, NB, KIND>(sm.V[(it + 1) & 3], pan(it + 1));
    lds_barrier();
    V4<E> w = {E(0), E(0), E(0), E(0)}, c1v = w;
    if (on) {
      V4<E> part[RS];
#pragma unroll
      for (int r = 0; r < RS; ++r) part[r] = X[(j + S * r) * 64 + lane];
#pragma unroll
      for (int n = 1; n < RS; n *= 2)
#pragma unroll
        for (int r = 0; r + n < RS; r += 2 * n) part[r] += part[r + n];
      w = part[0];
      if (KIND != K_UNM) {
        c1v = c1_read(c1_block(it), L);
        w += c1v;
      }
    }
    const V4<E> t = panel_t_load<E, TRANS>(sm.T[it & 3], L);
    lds_barrier();  // the parts and the killer rows have been read
    c1_load(it + RING);
    stage(it + 3).all(L);  // the slot of panel it - 1
    if (on) {
      const V4<E> w2 = panel_t<E, BF>(w, t);
      if (keeps) stblk(rsrc(c1 + 16 * p), L.q * NB, L, c1v - w2);
      const V4<E> wn = -w2;
#pragma unroll
      for (int i = 0; i < NBW; ++i) {
        const int rb = rp + RS * i;
        if (active(rb)) {
          const V4<E> a = block_c<LD>(Vs, rb, L);
          if constexpr (BF) {
            acc[i] = mfma_bf(bf16x4(a), bf16x4(wn), acc[i]);
          } else {
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[i] = mfma(a[r], wn[r], acc[i]);
          }
        }
      }
    }
  }
#pragma unroll
  for (int i = 0; i < NBW; ++i)
    if (on && rp + RS * i < NB / 16) stblk(rc2, 16 * (rp + RS * i) + L.q * NB, L, acc[i]);
}

// Sum over 16 lanes, and over the two 16-lane rows of each half wave, returned
// in every one of those lanes.
template <typename E>
__device__ __forceinline__ E sum16(E v) {
  v += dpp<0xB1>(v);   // quad_perm [1,0,3,2]
  v += dpp<0x4E>(v);   // quad_perm [2,3,0,1]
  v += dpp<0x124>(v);  // row_ror:4
  v += dpp<0x128>(v);  // row_ror:8
  return v;
}
// The value held 16 (32) lanes away in the other row of the pair (half of the
// wave); `upper` says whether the calling lane is in the upper one.
__device__ __forceinline__ uint32_t other_row(uint32_t v, bool upper) {
  const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  return upper ? r[0] : r[1];
}
__device__ __forceinline__ uint32_t other_half(uint32_t v, bool upper) {
  const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return upper ? r[0] : r[1];
}
__device__ __forceinline__ double other_row(double v, bool upper) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  return __builtin_bit_cast(double, (uint64_t)other_row((uint32_t)u, upper) |
                                        ((uint64_t)other_row((uint32_t)(u >> 32), upper) << 32));
}
__device__ __forceinline__ float other_row(float v, bool upper) {
  return __builtin_bit_cast(float, other_row(__builtin_bit_cast(uint32_t, v), upper));
}
__device__ __forceinline__ double other_half(double v, bool upper) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  return __builtin_bit_cast(double, (uint64_t)other_half((uint32_t)u, upper) |
                                        ((uint64_t)other_half((uint32_t)(u >> 32), upper) << 32));
}
__device__ __forceinline__ float other_half(float v, bool upper) {
  return __builtin_bit_cast(float, other_half(__builtin_bit_cast(uint32_t, v), upper));
}

// The same update for a chunk with a single live column (one right-hand
// side).  The column and the killer's column stay in LDS for the whole task
// and the products are matrix-vector ones on the vector units, where the
// matrix cores would run 15 of 16 columns for nothing.  Per panel: thread
// (k, r) = (tid / 32, tid % 32) sums rows r + 32 m of v_k^T c, every wave
// forms T^T w from the 16 sums by itself, and the first NB / 64 waves update
// one row per thread: two barriers, no exchange of partial results but the
// 16 sums.  Bounded by that chain's latency.  V is staged as in run_update.
template <typename E, int NB, int KIND, bool TRANS>
__device__ __forceinline__ void run_update_vec(Smem<E, NB>& sm, const E* V, const E* T, E* C1, E* C2, int np) {
  constexpr int LD = LDC<E, NB>, OPS = Stage<E, NB, KIND>::OPS;
  static_assert(sizeof(sm.C1) >= (2 * NB + IB) * sizeof(E), "the columns do not fit in C1");
  const int NP = __builtin_amdgcn_readfirstlane(np);
  const Lane L;
  const int tid = threadIdx.x, k = tid >> 5, r = tid & 31;
  E* c = sm.C1[0];       // the updated column
  E* c1 = c + NB;        // the killer's column
  E* u = c1 + NB;        // the 16 sums of a panel
  auto pan = [&](int it) { return TRANS ? it : NP - 1 - it; };
  auto stage = [&](int it) {
    return Stage<E, NB, KIND>(V, T + pan(it) * 256, sm.V[it & 3], sm.T[it & 3], pan(it), it < NP, L);
  };
  E x = E(0), x1 = E(0);
  if (tid < NB) {
    x = gload(C2 + tid);
    if (KIND != K_UNM) x1 = gload(C1 + tid);
  }
  stage(0).all(L);
  stage(1).all(L);
  stage(2).all(L);
  if (tid < NB) {
    c[tid] = x;
    c1[tid] = x1;
  }
  loads_left<2 * OPS>();
  stage_finish<E, NB, KIND>(sm.V[0], pan(0));
  lds_barrier();
#pragma unroll 1
  for (int it = 0; it < NP; ++it) {
    const int p = pan(it);
    const E* Vs = sm.V[it & 3];
    const E* Ts = sm.T[it & 3];
    // rows by pairs of 16-row blocks, as staged (pair_active)
    E d0 = E(0), d1 = E(0);
#pragma unroll
    for (int m = 0; m < NB / 32; ++m) {
      if (pair_active<KIND>(m, p)) {
        const E t = Vs[k * LD + r + 32 * m] * c[r + 32 * m];
        if (m & 1) d1 += t; else d0 += t;
      }
    }
    E d = sum16(d0 + d1);
    d += other_row(d, (r & 16) != 0);
    if (KIND != K_UNM) d += c1[16 * p + k];
    if (r == 0) u[k] = d;
    lds_barrier();
    stage(it + 3).all(L);  // the slot of panel it - 1
    // T^T u (T u when not TRANS): lane (g, q) of every wave sums four terms of entry q
    E a = E(0);
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      const int i = 4 * L.g + n;
      a += (TRANS ? Ts[sq_at<E>(i, L.q)] : Ts[sq_at<E>(L.q, i)]) * u[i];
    }
    a += other_row(a, (L.g & 1) != 0);
    a += other_half(a, L.g >= 2);
    if (KIND != K_UNM && tid < 16) c1[16 * p + tid] -= a;
    if (L.wave < NB / 64) {
      const bool act = KIND == K_UNM ? tid >= 32 * (p >> 1) : (KIND == K_TT ? tid < 32 * (p >> 1) + 32 : true);
      E w[16];  // read while every lane is active: lane n holds entry n
#pragma unroll
      for (int n = 0; n < 16; ++n) w[n] = readlane(a, n);
      if (act) {
        E y0 = c[tid], y1 = E(0);
#pragma unroll
        for (int n = 0; n < 16; n += 2) {
          y0 -= Vs[n * LD + tid] * w[n];
          y1 -= Vs[(n + 1) * LD + tid] * w[n + 1];
        }
        c[tid] = y0 + y1;
      }
    }
    if (it + 3 < NP)
      loads_left<2 * OPS>();
    else if (it + 3 == NP)
      loads_left<OPS>();
    else
      loads_left<0>();
    if (it + 1 < NP) stage_finish<E, NB, KIND>(sm.V[(it + 1) & 3], pan(it + 1));
    lds_barrier();
  }
  if (tid < NB) {
    gstore(C2 + tid, c[tid]);
    if (KIND != K_UNM) gstore(C1 + tid, c1[tid]);
  }
}

// Chooses the form by the number of live strips: one or two by rows (see
// run_update_rows), more one per wave.  A chain of updates on one right-hand
// side (hqr_solve, 16384 x 512, nb = 256) took 1144 us with one strip per
// wave, 692 by rows; from three strips on four waves of the other form work,
// and the parts of W and the killer rows of four strips do not fit into LDS
// next to the V slots.
// A single column takes the vector form (BF16 products stay on the matrix
// cores): a task on one column 39 -> 17 us, the same solve 692 -> 420 us.
template <typename E, int NB, int KIND, bool TRANS, bool BF = false>
__device__ __forceinline__ void update_chunk(const E* V, const E* T, E* C1, E* C2, int cols, int np) {
  Smem<E, NB>& sm = smem<E, NB>();
  cols = __builtin_amdgcn_readfirstlane(cols);
  const int strips = (cols + 15) / 16;
  if (!BF && cols == 1)
    run_update_vec<E, NB, KIND, TRANS>(sm, V, T, C1, C2, np);
  else if (strips == 1)
    run_update_rows<E, NB, KIND, TRANS, BF, 1>(sm, V, T, C1, C2, strips, np);
  else if (strips == 2)
    run_update_rows<E, NB, KIND, TRANS, BF, 2>(sm, V, T, C1, C2, strips, np);
  else
    run_update<E, NB, KIND, TRANS, BF>(sm, V, T, C1, C2, NB, strips, np);
}

// ---------------------------------------------------------------------------
// Panel task: GEQRT (KIND = UNM: the tile factors itself), TSQRT (TS: the
// triangle R on top of the square tile A), TTQRT (TT: the triangle R on top
// of the triangle A).  `A` is the tile zeroed (or triangularised for GEQRT),
// `R` the killer tile (TS/TT).  T blocks go to `T`.
//
// Column j of panel p: head = the diagonal entry of the triangle on top
// (GEQRT: A(j,j); TS/TT: R(j,j)), tail = the entries of the column that the
// reflector zeroes (GEQRT: A(j+1:nb, j); TS: A(0:nb, j); TT: A(0:j+1, j)).
// With alpha = head and s = ||tail||: s = 0 gives tau = 0 (H = I);
// otherwise beta = -sign(alpha) sqrt(alpha^2 + s^2), tau = (beta - alpha)/beta,
// tail /= (alpha - beta), head = beta.
//
// The tile is processed in blocks of 64 columns (four 16-column panels),
// left-looking: a block first receives the task's earlier panels, then each
// of its panels is factored (panel_columns) and applied to the block's
// remaining strips (panel_block).

// Lane sets of the column loop as 64-bit masks in scalar registers: a wave
// holds four columns (groups of 16 lanes).  A condition made from such a mask
// needs no vector compare, and selects or short masked regions made from it
// no branch: a divergent `if` on a vector compare takes about 45 cycles.
__device__ __forceinline__ bool in_lanes(uint64_t mask) { return __builtin_amdgcn_inverse_ballot_w64(mask); }

// The column loop multiplies raw columns with each other.  With every nonzero
// column's largest magnitude inside [2^-B, 2^B] no product or scalar of it can
// overflow, and what underflows is far below the column's rounding: a norm is
// at least sqrt(smallest subnormal) = 2^-75 (FP32; FP64 2^-537) when its
// square is not zero, so reflector scales reach 2^75 (2^537), and sums have
// 2^8 terms.  FP32: products 2^88, factors 2^75 2^45 = 2^120; an underflow of
// 2^-150 per term 2^-67 after scaling, against 2^-64 of a column of 2^-40.
// FP64: 2^908, 2^992, 2^-530 against 2^-503.
// A factorization whose panels all are out of range takes 14-28% longer (4096 x
// 4096, nb = 256: FP32 6.3 -> 7.4 ms, FP64 10.4 -> 11.8; 2048 x 512, nb = 64:
// FP64 1.20 -> 1.54).
template <typename E> constexpr int kRawBits = sizeof(E) == 8 ? 450 : 40;

// True in the lanes of a column (16 lanes, NM rows each, and `rv`) that has a
// value other than zero and is not inside that range (infinities and NaN are
// outside).
template <typename E, int NM>
__device__ __forceinline__ bool outside_raw(const E (&x)[NM], E rv) {
  typedef typename std::conditional<sizeof(E) == 8, uint64_t, uint32_t>::type U;
  constexpr int MANT = sizeof(E) == 8 ? 20 : 23, BIAS = sizeof(E) == 8 ? 1023 : 127;
  constexpr uint32_t LO = (uint32_t)(BIAS - kRawBits<E>) << MANT, HI = (uint32_t)(BIAS + kRawBits<E>) << MANT;
  uint32_t top = 0, low = 0;  // largest high word without sign; low words
  auto take = [&](E v) {
    const U u = __builtin_bit_cast(U, v);
    const uint32_t h = (uint32_t)(u >> (8 * sizeof(E) - 32)) & 0x7fffffffu;
    top = top > h ? top : h;
    if (sizeof(E) == 8) low |= (uint32_t)u;
  };
#pragma unroll
  for (int m = 0; m < NM; ++m) take(x[m]);
  take(rv);
  if (low != 0 && top == 0) top = 1;
  auto row = [&](uint32_t o) { top = top > o ? top : o; };
  row((uint32_t)__builtin_amdgcn_mov_dpp((int)top, 0xB1, 0xf, 0xf, true));
  row((uint32_t)__builtin_amdgcn_mov_dpp((int)top, 0x4E, 0xf, 0xf, true));
  row((uint32_t)__builtin_amdgcn_mov_dpp((int)top, 0x124, 0xf, 0xf, true));
  row((uint32_t)__builtin_amdgcn_mov_dpp((int)top, 0x128, 0xf, 0xf, true));
  return top != 0 && (top < LO || top > HI);
}

// Factors panel p (columns c0 = 16p .. c0+15).  The 16 columns stay in
// registers during the column loop: thread (cc, q) = (tid / 16, tid % 16)
// holds column c0 + cc at the rows base + q + 16 m (base = c0 for GEQRT,
// 0 otherwise), so the reductions over rows are 16-lane DPP sums inside one
// wavefront.  The only data crossing groups is the column being factored,
// published through LDS (double buffered), which costs one workgroup
// barrier per column.
//
// Every group works on the raw column: after the barrier it reads the tail,
// forms the tail's squared norm and its product with the group's own column
// in one pass (both reductions interleaved), derives the reflector's scalars
// itself and updates its column; the next column is published at once.  The
// owner's norm, reflector scalars and scaling are therefore not a second
// serial stage in front of the others' product and update.  The loop body
// has no divergent branch.  Cycles per column (one workgroup alone, loads
// and stores of the panel included): TS at 256 / 128 / 64 rows 1918 / 1504 /
// 1236 with the two stages, 1462 / 1076 / 906 with one (whole tasks inside a
// 32768 x 2048 factorization, then and now: GEQRT 367 -> 361 us, TSQRT 424 ->
// 398, TTQRT 433 -> 401).
//
// Leaves V_p in sm.V[0] (with the structure of the kind), T_p in sm.T[0] and
// in `T`, and the factored columns in A (and R).
// The panel's columns are taken from sm.V[0] (column-major, stride LDC, left
// there by panel_block).
//
// Raw products first (SCALED = false); in the rare panel that has a column out
// of their range (kRawBits) nothing is stored and the result is 1: the panel
// is then taken again with scaled tails (panel_block).  The columns are looked
// over by waves 5 and 6 during the loop: done by waves 0-3, or with a branch
// in every column, it took 3% of a 512 x 256 factorization at nb = 64, and on
// wave 4, whose column of T takes almost as long as one of the loop, up to 10%;
// as it is 480 -> 482 us (4001 x 777, TTQRT at nb = 128: 1898 -> 1937; 48
// requests at nb = 256: 6025 -> 5935).
template <typename E, int NB, int KIND, int NS, bool SCALED>
__device__ __forceinline__ int panel_columns_ns(E* A, E* R, E* T, int p) {
  // NS row slots per thread are held: NB / 16, or half of that where it holds
  // the panel (panel_columns)
  constexpr int NM = NS;
  p = __builtin_amdgcn_readfirstlane(p);  // uniform: row-slot guards become scalar branches
  Smem<E, NB>& sm = smem<E, NB>();
  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool ct = w < 4;    // waves 0-3 hold the panel
  const int cc = tid >> 4;  // panel column of this thread (waves 0-3)
  const int q = tid & 15;   // its rows are base + q + 16 m
  const int c0 = 16 * p;
  const int base = (KIND == K_UNM) ? c0 : 0;
  // row slots that can hold rows of the panel (uniform): GEQRT rows < NB,
  // TT rows <= c0 + 15.  The other slots hold zeros; the column loop runs
  // over all slots (branch-free), only loads and stores skip them.
  const int nm = (KIND == K_UNM) ? NB / 16 - p : (KIND == K_TT ? p + 1 : NB / 16);
  E* Vs = sm.V[0];
  // published column, two buffers: NM rows per lane at a stride that spreads
  // the 16-byte accesses of a column's 16 lanes over all banks, then its
  // entries of the 16 rows that can hold the reflector's unit entry
  constexpr int VW = 16 / (int)sizeof(E);
  typedef E LV __attribute__((ext_vector_type(VW)));
  constexpr int VST = NM + (sizeof(E) == 8 ? 2 : (NM % 8 == 4 ? 8 : 4));
  constexpr int VBUF = 16 * VST + 16;
  static_assert(NM % 4 == 0 && 2 * VBUF <= IB * LDC<E, NB>, "published columns do not fit in V slot 1");
  E* Vb = sm.V[1];
  E* col = A + (int64_t)(c0 + cc) * NB;
  E x[NM];
  auto load = [&](int c) {  // rows of panel column c
    const int d = c0 + c - q;  // TT: rows below the diagonal hold the tile's own GEQRT reflectors
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      const bool act = m < nm && (KIND != K_TT || 16 * m <= d);
      x[m] = act ? sm.V[0][c * LDC<E, NB> + base + q + 16 * m] : E(0);
    }
  };
  // TS/TT: R(c0 + q, c0 + c) of the killer's diagonal block
  auto load_r = [&](int c) { return KIND != K_UNM && q <= c ? gload(R + (c0 + q) + (int64_t)(c0 + c) * NB) : E(0); };
  E rv = E(0);
  // T is formed column by column on lanes 0-15 of wave 4 while waves 0-3 run
  // the column loop, one row of T per lane: column k = jj - 1 once z(0:k, k)
  // and tau_k are visible (after the barrier of iteration jj).
  //   T(k,k) = tau_k,  T(i,k) = -tau_k sum_{i <= l < k} T(i,l) z(l,k)
  // Every product of the sum is formed, those with l >= k are exact zeros
  // (z(l,k) = 0, and row[l] = 0 until column l is formed); all 16 LDS reads
  // are issued together.
  E trow[16];
  const int ti = tid & 63;
  auto t_column = [&](int k) {
    const E tk = sm.tau[k];
    E z[16];
#pragma unroll
    for (int l = 0; l < 16; ++l) z[l] = sm.Z[k * LDZ + l];
    E a0 = E(0), a1 = E(0), a2 = E(0), a3 = E(0);
#pragma unroll
    for (int l = 0; l < 16; l += 4) {
      a0 += trow[l] * z[l];
      a1 += trow[l + 1] * z[l + 1];
      a2 += trow[l + 2] * z[l + 2];
      a3 += trow[l + 3] * z[l + 3];
    }
    const E acc = (a0 + a1) + (a2 + a3);
    const E val = (ti < k) ? -tk * acc : (ti == k ? tk : E(0));
#pragma unroll
    for (int l = 0; l < 16; ++l) trow[l] = (l == k) ? val : trow[l];
  };
  // lanes q == 0 of the wave's four columns
  constexpr uint64_t row0 = 0x0001000100010001ull;
  // publishes the wave's column of group g, column j of the panel: its tail
  // (the rows the reflector zeroes; the others, lanes `lo` of row slot 0, as
  // zeros) to the buffer of its parity, and its entries of the rows that can
  // hold the unit entry (entry j is the head)
  auto publish = [&](int j, int g, uint64_t lo) {
    E* vb = Vb + (j & 1) * VBUF;
    const E x0 = (KIND == K_UNM && in_lanes(lo)) ? E(0) : x[0];
    if (in_lanes(0xffffull << (16 * g))) {
      vb[16 * VST + q] = (KIND == K_UNM) ? x[0] : rv;
#pragma unroll
      for (int m = 0; m < NM; m += VW) {
        LV t;
#pragma unroll
        for (int h = 0; h < VW; ++h) t[h] = m + h == 0 ? x0 : x[m + h];
        *reinterpret_cast<LV*>(vb + q * VST + m) = t;
      }
    }
  };
  if (ct) rv = load_r(cc), load(cc);
  // own: the column's scale (of its stored tail) once it has been factored
  E own = E(1);
  if (ct) {
    sm.Z[q * LDZ + cc] = E(0);  // entries (i, j) with i >= j stay zero
    if (w == 0) publish(0, 0, row0);
    uint64_t rowj = row0;  // lanes q == jj
    uint64_t lo = row0;    // lanes q <= jj
    // all lanes, opaque: as a constant, a lane set like 0xffffffffffff0000 is
    // emitted as a 32-bit literal that the hardware extends with zeros
    uint64_t ones = ~0ull;
    __asm__("" : "+s"(ones));
    // The four columns of a wave are unrolled: the lane sets are constants
    // then, and waves whose columns are all beyond jj, or all factored, take
    // a path without selects.  All sixteen unrolled take tens of KB of code
    // per panel kind, and the panel tasks miss in the instruction cache that
    // a compute unit pair shares.
#pragma unroll 1
    for (int ow = 0; ow < 4; ++ow) {
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int jj = 4 * ow + g;
        const E* vb = Vb + (g & 1) * VBUF;
        E& tp = (KIND == K_UNM) ? x[0] : rv;  // the column's entry of row jj, in its lane q = jj
        const E xt = lane_value(tp, (tid & 48) + jj);
        lds_barrier();
        E v[NM];
#pragma unroll
        for (int m = 0; m < NM; m += VW) {
          const LV t = *reinterpret_cast<const LV*>(vb + q * VST + m);
#pragma unroll
          for (int h = 0; h < VW; ++h) v[m + h] = t[h];
        }
        const E alpha = vb[16 * VST + jj] + E(0);  // (-0 becomes +0: beta = -n then)
        // squared norm of the tail and its product with this column
        E s0 = v[0] * v[0], s1 = v[1] * v[1], s2 = v[2] * v[2], s3 = v[3] * v[3];
        E d0 = v[0] * x[0], d1 = v[1] * x[1], d2 = v[2] * x[2], d3 = v[3] * x[3];
#pragma unroll
        for (int m = 4; m < NM; m += 4) {
          s0 += v[m] * v[m];
          d0 += v[m] * x[m];
          s1 += v[m + 1] * v[m + 1];
          d1 += v[m + 1] * x[m + 1];
          s2 += v[m + 2] * v[m + 2];
          d2 += v[m + 2] * x[m + 2];
          s3 += v[m + 3] * v[m + 3];
          d3 += v[m + 3] * x[m + 3];
        }
        E ss = (s0 + s1) + (s2 + s3), d = (d0 + d1) + (d2 + d3);
        sum16x2(ss, d);
        // beta = -sign(alpha) n; tau = (beta - alpha) / beta = 1 + |alpha| / n;
        // scale = 1 / (alpha - beta) = sign(alpha) / (|alpha| + n);
        // a zero tail gives tau = 0, scale = 1, beta = alpha
        const bool nz = ss != E(0);
        const auto hs = house_scalars(alpha, ss);
        const E rn = hs.hn + hs.hn;
        const E scale = nz ? flip_sign(hs.rd, alpha) : E(1);
        E ts = nz ? flip_sign(rn, alpha) : E(0);  // tau * scale
        const E tau = nz ? fma(__builtin_elementwise_abs(alpha), rn, E(1)) : E(0);
        E t = fma(scale, d, xt);  // v^T x with v = [1; scale * tail]
        if (SCALED) {
          // the product with the scaled tail (at most 1), and no update by an
          // identity (an infinity times its zeros would not be zero)
          s0 = s1 = s2 = s3 = E(0);
#pragma unroll
          for (int m = 0; m < NM; m += 4) {
            s0 += (v[m] *= scale) * x[m];
            s1 += (v[m + 1] *= scale) * x[m + 1];
            s2 += (v[m + 2] *= scale) * x[m + 2];
            s3 += (v[m + 3] *= scale) * x[m + 3];
          }
          E e = (s0 + s1) + (s2 + s3);
          sum16x2(e, d);
          t = nz ? e + xt : E(0);
          ts = tau;
        }
        lo = (lo << 1) | row0;          // lanes q <= jj + 1
        if (w > ow) {
          const E f = ts * t;
#pragma unroll
          for (int m = 0; m < NM; ++m) x[m] -= f * v[m];
          tp = in_lanes(rowj) ? tp - tau * t : tp;
          if (g == 3 && w == ow + 1) publish(jj + 1, 0, lo);
        } else if (w == ow) {
          const uint64_t eq = 0xffffull << (16 * g), ab = g < 3 ? ones << (16 * ((g + 1) & 3)) : 0ull;
          if (g < 3) {
            const E f = in_lanes(ab) ? ts * t : E(0);
            const E tn = tp - tau * t;
            if (in_lanes(ab)) {
#pragma unroll
              for (int m = 0; m < NM; ++m) x[m] -= f * v[m];
            }
            tp = in_lanes(rowj & ab) ? tn : tp;
            publish(jj + 1, g + 1, lo);
          }
          tp = in_lanes(rowj & eq) ? (nz ? -flip_sign(hs.n, alpha) : alpha) : tp;
          if (g > 0 && in_lanes(rowj & ~(ab | eq))) sm.Z[jj * LDZ + cc] = own * t;  // v_cc^T v_jj
          own = in_lanes(eq) ? scale : own;
          if (in_lanes(rowj & eq)) sm.tau[jj] = tau;
        } else {
          if (in_lanes(rowj)) sm.Z[jj * LDZ + cc] = own * t;
        }
        rowj <<= 1;
      }
    }
    // the stored tails become reflector entries
#pragma unroll
    for (int m = 0; m < NM; ++m)
      if (!(KIND == K_UNM && m == 0)) x[m] *= own;
    if (KIND == K_UNM && q > cc) x[0] *= own;
  } else if (w == 4) {
#pragma unroll
    for (int l = 0; l < 16; ++l) trow[l] = E(0);
    lds_barrier();
#pragma unroll 1
    for (int jj = 1; jj < 16; ++jj) {
      lds_barrier();
      t_column(jj - 1);
    }
  } else if (!SCALED && w < 7) {
    // waves 5 and 6 look the columns over meanwhile, four at a time each (in
    // less time than a column of the loop takes)
    const int c = 8 * (w - 5) + ((tid >> 4) & 3);
    const E r0 = load_r(c), r1 = load_r(c + 4);
    lds_barrier();
    lds_barrier();
    load(c);
    bool out = outside_raw(x, r0);
    lds_barrier();
    lds_barrier();
    load(c + 4);
    out |= outside_raw(x, r1);
    sm.wide[w - 5] = __ballot(out) != 0;
#pragma unroll 1
    for (int jj = 4; jj < 16; ++jj) lds_barrier();
  } else {
#pragma unroll 1
    for (int jj = 0; jj < 16; ++jj) lds_barrier();
  }
  const int2 wide = *reinterpret_cast<const int2*>(sm.wide);
  lds_barrier();  // the published columns and sm.V[0] have been read by every wave
  if (!SCALED && __builtin_expect(__builtin_amdgcn_readfirstlane(wide.x | wide.y), 0)) return 1;
  // ---- the factored panel back to the tiles, and V_p into LDS
  // (the panel's number is made opaque so that the slots' conditions are formed
  // anew: kept from the loads above they would fill the scalar registers)
  int pe = p;
  __asm__("" : "+s"(pe));
  const int be = (KIND == K_UNM) ? 16 * pe : 0, de = 16 * pe + cc - q;
  const int ne = (KIND == K_UNM) ? NB / 16 - pe : (KIND == K_TT ? pe + 1 : NB / 16);
  E* cole = col + be + q;
  E* Ve = Vs + cc * LDC<E, NB> + be + q;
#pragma unroll
  for (int m = 0; m < NM; ++m) {
    if (ct && m < ne) {
      if (KIND != K_TT || 16 * m <= de) {
        gstore(cole + 16 * m, x[m]);
        E vv = x[m];
        if (KIND == K_UNM && m == 0 && q <= cc) vv = (q == cc) ? E(1) : E(0);  // unit diagonal, R above
        Ve[16 * m] = vv;
      } else {
        Ve[16 * m] = E(0);  // TT: zero below the diagonal of V
      }
    }
  }
  // the other half of the pair of blocks that holds the diagonal block
  if (KIND == K_UNM && ct && (p & 1)) Vs[cc * LDC<E, NB> + c0 - 16 + q] = E(0);
  if (KIND == K_TT && ct && !(p & 1)) Vs[cc * LDC<E, NB> + c0 + 16 + q] = E(0);
  if (KIND != K_UNM && ct && q <= cc) gstore(R + (c0 + q) + (int64_t)(c0 + cc) * NB, rv);
  // the last column of T, then T to LDS (for the strips) and to memory
  if (w == 4) {
    t_column(15);
    if (ti < 16) {
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        sm.T[0][sq_at<E>(ti, k)] = trow[k];
        gstore(T + p * 256 + ti + 16 * k, trow[k]);
      }
    }
  }
  // V_p and T_p in LDS are what the strips of the block need next; the columns just
  // stored are read back (block update) only after a full barrier
  lds_barrier();
  return 0;
}

// The column loop's cost follows the rows a panel can hold: GEQRT panel p
// has rows 16p .. NB-1 (NB/16 - p slots), TTQRT panel p rows 0 .. 16p+15
// (p + 1 slots); TSQRT always all NB/16.  GEQRT and TTQRT take half of the
// slots where these hold the panel, all otherwise.
template <typename E, int NB, int KIND, bool SCALED>
__device__ __forceinline__ int panel_columns(E* A, E* R, E* T, int p) {
  constexpr int NM = NB / 16;
  p = __builtin_amdgcn_readfirstlane(p);
  if constexpr (KIND != K_TS && NM > 4 && !SCALED) {
    const int nm = (KIND == K_UNM) ? NM - p : p + 1;
    if (nm <= NM / 2) return panel_columns_ns<E, NB, KIND, NM / 2, SCALED>(A, R, T, p);  // uniform
  }
  return panel_columns_ns<E, NB, KIND, NM, SCALED>(A, R, T, p);
}

// Row-split application of panel p inside a panel task: the strip of 16
// columns is shared by waves w and w + 4, wave half h = wave / 4 holding row
// blocks h NB/32 .. (h + 1) NB/32 - 1 of it in `acc`.  Each wave reduces its
// rows' part of W = V_p^T C, the two parts are exchanged through LDS and
// added in a fixed order (lower half + upper half, so both waves hold bitwise
// the same W), then each wave updates its own rows; the wave of the upper
// half (h = 0) also updates C1_p (TS/TT).  Every thread of the workgroup
// calls this (it contains a barrier); `on` says whether the wave holds a
// strip.  The killer rows are in LDS at c1s, or in c1v (c1s null).
template <typename E, int NB, int KIND, bool BF>
__device__ __forceinline__ void apply_panel_half(V4<E> (&acc)[NB / 32], const E* Vs, const E* Ts, int p, E* c1,
                                                 const E* c1s, V4<E> c1v, const Lane& L, int h, bool on) {
  constexpr int HRB = NB / 32, LD = LDC<E, NB>;
  Smem<E, NB>& sm = smem<E, NB>();
  const int lane = threadIdx.x & 63;
  auto active = [&](int rb) { return (KIND == K_UNM) ? rb >= p : (KIND == K_TT ? rb <= p : true); };
  if (on) {
    V4<E> w0 = {E(0), E(0), E(0), E(0)}, w1 = w0;
#pragma unroll
    for (int i = 0; i < HRB; ++i) {
      const int rb = h * HRB + i;
      if (active(rb)) {
        const V4<E> a = block_w<LD>(Vs, rb, L);
        if constexpr (BF) {
          if (i & 1)
            w1 = mfma_bf(bf16x4(a), bf16x4(acc[i]), w1);
          else
            w0 = mfma_bf(bf16x4(a), bf16x4(acc[i]), w0);
        } else {
          w0 = mfma(a[0], acc[i][0], w0);
          w1 = mfma(a[1], acc[i][1], w1);
          w0 = mfma(a[2], acc[i][2], w0);
          w1 = mfma(a[3], acc[i][3], w1);
        }
      }
    }
    sm.x()[L.wave * 64 + lane] = w0 + w1;
  }
  lds_barrier();
  if (on) {
    const V4<E> t = panel_t_load<E, true>(Ts, L);
    const V4<E> lo = sm.x()[(L.wave & 3) * 64 + lane], hi = sm.x()[((L.wave & 3) + 4) * 64 + lane];
    V4<E> w = lo + hi;
    if (KIND != K_UNM) {
      if (c1s) c1v = c1_read(c1s, L);
      w += c1v;
    }
    const V4<E> w2 = panel_t<E, BF>(w, t);
    if (KIND != K_UNM && h == 0) stblk(rsrc(c1), L.q * NB, L, c1v - w2);
    const V4<E> wn = -w2;
#pragma unroll
    for (int i = 0; i < HRB; ++i) {
      const int rb = h * HRB + i;
      if (active(rb)) {
        const V4<E> a = block_c<LD>(Vs, rb, L);
        if constexpr (BF) {
          acc[i] = mfma_bf(bf16x4(a), bf16x4(wn), acc[i]);
        } else {
#pragma unroll
          for (int r = 0; r < 4; ++r) acc[i] = mfma(a[r], wn[r], acc[i]);
        }
      }
    }
  }
}

// Block b of a panel task (columns 64b .. 64b+63) with its four strips kept
// in registers from start to end: strip 4b + w lives in waves w and w + 4
// (row halves).  The strips are loaded once, receive this task's earlier
// panels (left-looking), and then for each panel p of the block the strip of
// p is handed to the column loop through LDS (sm.V[0]) and the panel is
// applied to the block's later strips in registers; the factored columns
// reach memory through the column loop (GEQRT: the rows of a strip above its
// diagonal block, which the column loop does not cover, are stored at the
// hand-over).  No strip goes through memory between the panels of a block.
// When a panel is out of the range of raw products (panel_columns), the
// strips go to their place in the tile and the block is taken up again from
// that panel, `p0`, with scaled tails (SCALED), in a function of its own: nothing
// is held in registers across the call, and the common path's registers do not
// depend on it.
template <typename E, int NB, int KIND, bool BF>
__device__ __noinline__ void panel_block_scaled(E* A, E* R, E* T, int b, int p0);

template <typename E, int NB, int KIND, bool BF, bool SCALED>
__device__ __forceinline__ void panel_block(E* A, E* R, E* T, int b, int p0) {
  constexpr int HRB = NB / 32;
  b = __builtin_amdgcn_readfirstlane(b);
  Smem<E, NB>& sm = smem<E, NB>();
  const Lane L;
  const int w = L.wave & 3, h = L.wave >> 2;
  const int s = 4 * b + w;   // this wave's strip
  const int np = 4 * b;      // earlier panels of this task
  // row blocks held: TT rows up to the block's last diagonal block (below
  // them a TT victim holds its own GEQRT reflectors), otherwise all
  const int hi = (KIND == K_TT) ? 4 * b + 3 : NB / 16 - 1;
  const __amdgpu_buffer_rsrc_t rs = rsrc(A + (int64_t)(16 * s) * NB);
  E* c1s = KIND == K_UNM ? nullptr : R + (int64_t)(16 * s) * NB;  // killer's strip s
  const bool keeps = KIND != K_UNM && h == 0;  // loads and stores the strip's killer rows
  auto stage = [&](int p) {
    return Stage<E, NB, KIND>(A, T + p * 256, sm.V[p & 1], sm.T[p & 1], p, p < np, L);
  };
  auto c1_block = [&](int p) { return sm.C1[4 * (p & 1) + w]; };
  V4<E> c1v = {E(0), E(0), E(0), E(0)};
  V4<E> acc[HRB];
  if (!SCALED) {
    stage(0).all(L);
    if (keeps && np > 0) c1_start<E, NB>(c1s, c1_block(0));
  }
#pragma unroll
  for (int i = 0; i < HRB; ++i)
    if (h * HRB + i <= hi) acc[i] = ldblk<E>(rs, 16 * (h * HRB + i) + L.q * NB, L);
  if (!SCALED && np > 0) {
    loads_done();
    stage_finish<E, NB, KIND>(sm.V[0], 0);
    lds_barrier();
#pragma unroll 1
    for (int p = 0; p < np; ++p) {
      const int sl = p & 1;
      stage(p + 1).all(L);
      if (keeps && p + 1 < np) c1_start<E, NB>(c1s + 16 * (p + 1), c1_block(p + 1));
      apply_panel_half<E, NB, KIND, BF>(acc, sm.V[sl], sm.T[sl], p, c1s + 16 * p, c1_block(p), c1v, L, h, true);
      if (p + 1 < np) {
        // only this panel's C1 stores are newer
        if (keeps)
          loads_left<sizeof(E) == 8 ? 2 : 1>();
        else
          loads_left<0>();
        stage_finish<E, NB, KIND>(sm.V[sl ^ 1], p + 1);
      }
      lds_barrier();
    }
  }
#pragma unroll 1
  for (int p = SCALED ? __builtin_amdgcn_readfirstlane(p0) : np; p < np + 4; ++p) {
    // (loaded here, it arrives during the column loop)
    if (KIND != K_UNM && s > p) c1v = ldblk<E>(rsrc(c1s + 16 * p), L.q * NB, L);
    if (s == p) {
      E* H = sm.V[0] + L.q * LDC<E, NB>;
#pragma unroll
      for (int i = 0; i < HRB; ++i) {
        const int rb = h * HRB + i;
        if (rb <= hi) {
          const V4<E>& v = acc[i];
          if constexpr (sizeof(E) == 8) {
            *reinterpret_cast<V2<E>*>(H + 16 * rb + 2 * L.g) = V2<E>{v.x, v.y};
            *reinterpret_cast<V2<E>*>(H + 16 * rb + 2 * L.g + 8) = V2<E>{v.z, v.w};
          } else {
            *reinterpret_cast<V4<E>*>(H + 16 * rb + 4 * L.g) = v;
          }
          // GEQRT: rows above the diagonal block are final R entries
          if (KIND == K_UNM && rb < p) stblk(rs, 16 * rb + L.q * NB, L, v);
        }
      }
    }
    lds_barrier();
    if (__builtin_expect(panel_columns<E, NB, KIND, SCALED>(A, R, T, p), 0)) {
#pragma unroll
      for (int i = 0; i < HRB; ++i)
        if (s >= p && h * HRB + i <= hi) stblk(rs, 16 * (h * HRB + i) + L.q * NB, L, acc[i]);
      stores_done();
      __syncthreads();
      panel_block_scaled<E, NB, KIND, BF>(A, R, T, b, p);
      return;
    }
    if (p < np + 3)
      apply_panel_half<E, NB, KIND, BF>(acc, sm.V[0], sm.T[0], p, c1s + 16 * p, nullptr, c1v, L, h, s > p);
    lds_barrier();  // every wave is done with the V panel and T in LDS
  }
}

template <typename E, int NB, int KIND, bool BF>
__device__ __noinline__ void panel_block_scaled(E* A, E* R, E* T, int b, int p0) {
  panel_block<E, NB, KIND, BF, true>(A, R, T, b, p0);
}

// ---------------------------------------------------------------------------
// Scheduler steps.

// Waits until every lane's counter *c >= v (one counter per lane of the
// calling wave).  Returns false when the launch has been aborted: by this
// wait running past the spin limit (it then records the abort and what it
// was waiting for in ctrl[1..5]) or by another workgroup's abort.
// Every lane of the wave calls it; a lane with c == null or v == 0 has
// nothing to wait for.  The counters are polled in parallel instead of one
// after another.  Returns the same (uniform) result in every lane; on a
// time-out the lowest lane still waiting records its counter.
__device__ __forceinline__ bool wait_lanes(int32_t* c, uint32_t v, const LaunchArgs& a, int t) {
  bool done = (c == nullptr) || (v == 0);
  int64_t spins = 0;
  const int lane = threadIdx.x & 63;
  for (;;) {
    uint32_t seen = 0;
    if (!done) {
      seen = (uint32_t)__hip_atomic_load(c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      done = seen >= v;
    }
    const uint64_t pending = __ballot(!done);
    if (pending == 0) return true;
    ++spins;
    if (spins > a.spin_limit) {
      if (lane == __ffsll((unsigned long long)pending) - 1) {
        int32_t none = 0;
        if (__hip_atomic_compare_exchange_strong(&a.ctrl[1], &none, (int32_t)HQR_ERR_WATCHDOG, __ATOMIC_RELAXED,
                                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
          __hip_atomic_store(&a.ctrl[2], t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          __hip_atomic_store(&a.ctrl[3], (int32_t)(c - a.cnt), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          __hip_atomic_store(&a.ctrl[4], (int32_t)v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          __hip_atomic_store(&a.ctrl[5], (int32_t)seen, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
      }
      return false;
    }
    if ((spins & 63) == 0) {
      const int st = __builtin_amdgcn_readfirstlane(
          __hip_atomic_load(&a.ctrl[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
      if (st != 0) return false;
    }
    __builtin_amdgcn_s_sleep(2);
  }
}

__device__ __forceinline__ void trace(const LaunchArgs& a, int t, int phase) {
  if (a.trace && blockIdx.x < kTraceSlots) {
    __hip_atomic_store(&a.trace[2 * blockIdx.x], t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(&a.trace[2 * blockIdx.x + 1], phase, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

// Index of the XCD (accelerator complex die) running the wave.
__device__ __forceinline__ int xcc_id() {
  int x = 0;
  __asm__ __volatile__("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(x));
  return x & 0xf;
}

// Timeline record of task t: [0] picked, [1] inputs ready, [2] done (100 MHz
// real-time clock), [3] workgroup | XCD << 16.
__device__ __forceinline__ void stamp(const LaunchArgs& a, int t, int slot) {
  if (a.timeline && t >= 0) {
    a.timeline[4 * (int64_t)t + slot] = __builtin_amdgcn_s_memrealtime();
    if (slot == 0) a.timeline[4 * (int64_t)t + 3] = (uint64_t)blockIdx.x | ((uint64_t)xcc_id() << 16);
  }
}

__device__ __forceinline__ int32_t* counter(const LaunchArgs& a, int r, int c, int chunk) {
  return a.cnt + ((int64_t)r * a.cnt_cols + c) * a.chunks + chunk;
}

// The steps of one scheduler iteration are separate, non-inlined functions
// on purpose: each one holds the lane-divergent part of its step (the work
// of thread 0) together with the workgroup barrier that ends it, so the loop
// in the kernel contains only uniform control flow.  When these steps were
// inlined, the compiler moved thread 0's tail of an iteration out of the
// loop behind a divergent exit, and the other lanes re-ran the same task.

// Takes the next task index (uniform), or -1 when every task has been
// handed out or the launch was aborted.
template <typename E, int NB>
__device__ __noinline__ int take_task(const LaunchArgs& a) {
  Smem<E, NB>& sm = smem<E, NB>();
  if (threadIdx.x == 0) {
    int t = sm.next;
    sm.next = -2;
    // an aborted launch hands out no more tasks: every workgroup leaves at
    // its next pick, so the kernel ends soon after the first time-out
    if (__hip_atomic_load(&a.ctrl[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0)
      t = -1;
    else if (t == -2)
      t = __hip_atomic_fetch_add(&a.ctrl[0], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (t >= a.ntasks) t = -1;
    sm.task = t;
    trace(a, t, t < 0 ? TR_EXIT : TR_POPPED);
    stamp(a, t, 0);
  }
  __syncthreads();
  return __builtin_amdgcn_readfirstlane(sm.task);
}

// Dependency counters count 64-column sub-chunks of a tile.  A panel task
// works through its tile(s) block by block (64 columns each): it waits for
// block b's sub-chunk before touching block b and publishes it when the
// block is final, so a chain of panel tasks on one tile (a TS domain, a
// tree) advances one block behind its predecessor.  The last active
// sub-chunk is published only when the whole task is done, which is what
// the update tasks reading the factored tile wait for (task.pad & 0xff).
// An update task covers task.pad >> 8 sub-chunks starting at sub-chunk
// task.chunk.

// Thread 0 waits for the task's input versions (panel tasks: block 0);
// returns 1 (uniform) when they were reached, 0 when the launch was aborted.
template <typename E, int NB>
__device__ __noinline__ int wait_task(const LaunchArgs& a, int t, const DevTask& task) {
  Smem<E, NB>& sm = smem<E, NB>();
  if (threadIdx.x < 64) {
    // lane l waits for the l-th (counter, version) pair of the task
    const int l = threadIdx.x;
    const int op = task.op, i = task.row, piv = task.killer, k = task.k, j = task.j;
    int32_t* c = nullptr;
    uint32_t v = 0;
    if (a.B) {
      // apply launch: one counter per block of B
      if (op == UNMQR) {
        if (l == 0) c = counter(a, i, j, 0), v = task.v[1];
      } else {
        if (l == 0) c = counter(a, piv, j, 0), v = task.v[1];
        if (l == 1) c = counter(a, i, j, 0), v = task.v[2];
      }
    } else {
      const int c0 = task.chunk, cn = task.pad >> 8, cv = task.pad & 0xff;
      switch (op) {
        case GEQRT:
          if (l == 0) c = counter(a, i, k, 0), v = task.v[0];
          break;
        case TSQRT:
        case TTQRT:
          if (l == 0) c = counter(a, piv, k, 0), v = task.v[0];
          if (l == 1) c = counter(a, i, k, 0), v = task.v[1];
          break;
        case UNMQR:
          if (l == 0) c = counter(a, i, k, cv), v = task.v[0];
          if (l >= 1 && l <= cn) c = counter(a, i, j, c0 + l - 1), v = task.v[1];
          break;
        default:
          if (l == 0) c = counter(a, i, k, cv), v = task.v[0];
          if (l >= 1 && l <= cn) c = counter(a, piv, j, c0 + l - 1), v = task.v[1];
          if (l > cn && l <= 2 * cn) c = counter(a, i, j, c0 + l - cn - 1), v = task.v[2];
          break;
      }
    }
    const bool ok = wait_lanes(c, v, a, t);
    if (l == 0) {
      sm.ok = ok ? 1 : 0;
      trace(a, t, ok ? TR_READY : TR_ABORT);
      stamp(a, t, 1);
    }
  }
  __syncthreads();
  const int ok = __builtin_amdgcn_readfirstlane(sm.ok);
  // the producers' stores had completed when they bumped the counters, and
  // tile loads are device-coherent: no cache invalidation is needed
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  return ok;
}

// Panel tasks, inside the task: wait for block b (b >= 1) of the tile(s).
template <typename E, int NB>
__device__ __noinline__ int wait_block(const LaunchArgs& a, int t, const DevTask& task, int b) {
  Smem<E, NB>& sm = smem<E, NB>();
  __syncthreads();
  if (threadIdx.x < 64) {
    const int l = threadIdx.x;
    int32_t* c = nullptr;
    uint32_t v = 0;
    if (task.op == GEQRT) {
      if (l == 0) c = counter(a, task.row, task.k, b), v = task.v[0];
    } else {
      if (l == 0) c = counter(a, task.killer, task.k, b), v = task.v[0];
      if (l == 1) c = counter(a, task.row, task.k, b), v = task.v[1];
    }
    const bool ok = wait_lanes(c, v, a, t);
    if (l == 0) sm.ok = ok ? 1 : 0;
  }
  __syncthreads();
  const int ok = __builtin_amdgcn_readfirstlane(sm.ok);
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  return ok;
}

// Panel tasks, inside the task: block b of the tile(s) is final.
template <typename E, int NB>
__device__ __noinline__ void release_block(const LaunchArgs& a, const DevTask& task, int b) {
  stores_done();
  __syncthreads();
  if (threadIdx.x == 0) {
    __hip_atomic_fetch_add(counter(a, task.row, task.k, b), 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (task.op != GEQRT)
      __hip_atomic_fetch_add(counter(a, task.killer, task.k, b), 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// Publishes the task's tile writes and bumps the counters of the tiles it
// wrote (panel tasks: the last active block; the others went out with
// release_block).
template <typename E, int NB>
__device__ __noinline__ void finish_task(const LaunchArgs& a, int t, const DevTask& task) {
  // the next task index is taken while this task's stores drain
  int next = -2;
  if (threadIdx.x == 0) next = __hip_atomic_fetch_add(&a.ctrl[0], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  stores_done();
  __syncthreads();
  if (threadIdx.x == 0) {
    smem<E, NB>().next = next;
    trace(a, t, TR_DONE);
    stamp(a, t, 2);
    const int op = task.op, i = task.row, piv = task.killer, k = task.k, j = task.j;
    auto bump = [&](int32_t* c) { __hip_atomic_fetch_add(c, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
    if (a.B) {
      if (op != UNMQR) bump(counter(a, piv, j, 0));
      bump(counter(a, i, j, 0));
    } else {
      const int c0 = task.chunk, cn = task.pad >> 8;
      switch (op) {
        case GEQRT:
          bump(counter(a, i, k, task.chunk - 1));
          break;
        case TSQRT:
        case TTQRT:
          bump(counter(a, piv, k, task.chunk - 1));
          bump(counter(a, i, k, task.chunk - 1));
          break;
        case UNMQR:
          for (int c = c0; c < c0 + cn; ++c) bump(counter(a, i, j, c));
          break;
        default:
          for (int c = c0; c < c0 + cn; ++c) {
            bump(counter(a, piv, j, c));
            bump(counter(a, i, j, c));
          }
          break;
      }
    }
  }
}

// Tiles are stored contiguously (tile (r, c) at index c * mt + r, each one
// column-major with leading dimension nb), so a tile spans a few pages only.
template <typename E>
__device__ __forceinline__ E* tile_ptr(const LaunchArgs& a, int nb, int r, int c) {
  return (E*)a.A + ((int64_t)c * a.mt + r) * nb * nb;
}

template <typename E>
__device__ __forceinline__ E* t_block(void* T, const LaunchArgs& a, int nb, int r, int c) {
  return (E*)T + ((int64_t)r * a.nt + c) * nb * 16;
}

// One tile kernel per function (each gets its own register allocation).
// Panel tasks are on the critical path of the factorization: their waves
// run at raised priority.  The tile(s) are processed block by block (64
// columns) up to the last block holding matrix columns, left-looking: block
// b waits for the predecessor's block b,
// takes this task's earlier panels, is factored, and is published at once
// (except the last active block, published by finish_task).  Returns 0 when
// the launch was aborted while waiting.
template <typename E, int NB, int KIND, bool BF = false>
__device__ __noinline__ int panel_task(const LaunchArgs& a, int t, const DevTask& task) {
  E* T = t_block<E>((KIND == K_UNM) ? a.Tg : a.Tk, a, NB, task.row, task.k);
  E* A = tile_ptr<E>(a, NB, task.row, task.k);
  E* R = KIND == K_UNM ? nullptr : tile_ptr<E>(a, NB, task.killer, task.k);
  const int active = task.chunk;  // blocks holding matrix columns
  __builtin_amdgcn_s_setprio(2);
  for (int b = 0; b < NB / 64; ++b) {
    if (b >= active) {
      // blocks beyond the last matrix column (zero padding) are not factored:
      // their reflectors are the identity, T = 0 (what factoring the zero
      // columns would give), and the padding stays zero
      for (int e = threadIdx.x; e < (NB / 16 - 4 * b) * 256; e += NT) gstore(T + 4 * b * 256 + e, E(0));
      break;
    }
    if (b > 0 && !wait_block<E, NB>(a, t, task, b)) {
      __builtin_amdgcn_s_setprio(0);
      return 0;
    }
    panel_block<E, NB, KIND, BF, false>(A, R, T, b, 0);
    if (b + 1 < active) {
      release_block<E, NB>(a, task, b);
    } else {
      stores_done();
      __syncthreads();  // the next block reads the columns and T stored by this one
    }
  }
  __builtin_amdgcn_s_setprio(0);
  return 1;
}

// An update task covers one or two 64-column sub-chunks (one 16-column
// strip per wave; one sub-chunk at nb = 64 and at the ragged end of a tile).
template <typename E, int NB, int KIND, bool BF = false>
__device__ __noinline__ void update_task(const LaunchArgs& a, const DevTask& task) {
  void* T = (KIND == K_UNM) ? a.Tg : a.Tk;
  const int64_t colchunk = (int64_t)task.chunk * 64 * NB;
  const E* V = tile_ptr<E>(a, NB, task.row, task.k);
  const E* Tb = t_block<E>(T, a, NB, task.row, task.k);
  E* C1 = KIND == K_UNM ? nullptr : tile_ptr<E>(a, NB, task.killer, task.j) + colchunk;
  E* C2 = tile_ptr<E>(a, NB, task.row, task.j) + colchunk;
  // panels of the factored tile column that hold matrix columns: four per
  // 64-column block up to its last active block (task.pad & 0xff)
  const int np = 4 * ((task.pad & 0xff) + 1) < NB / IB ? 4 * ((task.pad & 0xff) + 1) : NB / IB;
  // columns of the chunk that belong to the matrix or to the right-hand sides;
  // the others are zero padding and stay zero
  const int64_t left = (task.j < a.nt ? a.N - (int64_t)task.j * NB : a.nrhs - (int64_t)(task.j - a.nt) * NB) - 64 * task.chunk;
  const int all = 64 * (task.pad >> 8);
  update_chunk<E, NB, KIND, true, BF>(V, Tb, C1, C2, left < all ? (int)left : all, np);
}

// Block of 64 columns of B (nb x 64, column-major) of tile row r.
template <typename E>
__device__ __forceinline__ E* b_block(const LaunchArgs& a, int nb, int r, int j) {
  return (E*)a.B + ((int64_t)j * a.mt + r) * nb * 64;
}

// The same transformation applied to a block of B (hqr_apply_qt/_q).
template <typename E, int NB, int KIND, bool TRANS>
__device__ __noinline__ void apply_task(const LaunchArgs& a, const DevTask& task) {
  void* T = (KIND == K_UNM) ? a.Tg : a.Tk;
  const int cols = a.nrhs - 64 * task.j;
  update_chunk<E, NB, KIND, TRANS>(tile_ptr<E>(a, NB, task.row, task.k), t_block<E>(T, a, NB, task.row, task.k),
                                   KIND == K_UNM ? nullptr : b_block<E>(a, NB, task.killer, task.j),
                                   b_block<E>(a, NB, task.row, task.j), cols < 64 ? cols : 64, NB / IB);
}

// Points the per-problem fields of `la` (tiles, T factors, counters, tile
// grid) at the problem of task t of a batched launch.
__device__ __forceinline__ void bind_problem(LaunchArgs& la, const LaunchArgs& a, int t) {
  const ProbDesc* d = a.probs + a.task_prob[t];
  char* w = (char*)a.ctrl;
  la.A = (double*)(w + d->tiles);
  la.Tg = (double*)(w + d->tg);
  la.Tk = (double*)(w + d->tk);
  la.cnt = (int32_t*)(w + d->cnt);
  la.mt = d->mt;
  la.nt = d->nt;
  la.cnt_cols = d->nt + d->nrt;
  la.N = d->N;
  la.nrhs = d->nrhs;
}

// Persistent scheduler.  Workgroups take task indices from a global cursor
// in dispatch order (a topological order of the task graph), wait until the
// dependency counters of the tiles the task touches reach the versions in
// the task record, run it, and bump the counters of the tiles it wrote.
// Every task a workgroup waits for was taken earlier by a running
// workgroup, so the wait always ends.  BATCH: the tasks of many independent
// problems share the cursor (each task names its problem).
template <typename E, int NB, bool BATCH, bool BF = false>
__global__ __launch_bounds__(NT, 1) void persistent_kernel(LaunchArgs args) {
  LaunchArgs la = args;
  if (threadIdx.x == 0) smem<E, NB>().next = -2;
  for (;;) {
    const int t = take_task<E, NB>(args);
    if (t < 0) break;
    const DevTask task = args.tasks[t];
    if (BATCH) bind_problem(la, args, t);
    const LaunchArgs& a = BATCH ? la : args;
    if (!wait_task<E, NB>(a, t, task)) break;
    int ok = 1;
    if (a.B) {
      if (a.trans) {
        switch (task.op) {
          case UNMQR: apply_task<E, NB, K_UNM, true>(a, task); break;
          case TSMQR: apply_task<E, NB, K_TS, true>(a, task); break;
          default: apply_task<E, NB, K_TT, true>(a, task); break;
        }
      } else {
        switch (task.op) {
          case UNMQR: apply_task<E, NB, K_UNM, false>(a, task); break;
          case TSMQR: apply_task<E, NB, K_TS, false>(a, task); break;
          default: apply_task<E, NB, K_TT, false>(a, task); break;
        }
      }
    } else {
      switch (task.op) {
        case GEQRT: ok = panel_task<E, NB, K_UNM, BF>(a, t, task); break;
        case TSQRT: ok = panel_task<E, NB, K_TS, BF>(a, t, task); break;
        case TTQRT: ok = panel_task<E, NB, K_TT, BF>(a, t, task); break;
        case UNMQR: update_task<E, NB, K_UNM, BF>(a, task); break;
        case TSMQR: update_task<E, NB, K_TS, BF>(a, task); break;
        default: update_task<E, NB, K_TT, BF>(a, task); break;
      }
    }
    if (!ok) break;  // aborted inside a panel task
    finish_task<E, NB>(a, t, task);
  }
}

// ---------------------------------------------------------------------------
// Small helpers.

__global__ void zero_i32_kernel(int32_t* p, int64_t n) {
  for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < n; x += (int64_t)gridDim.x * blockDim.x)
    p[x] = 0;
}

__global__ void init_ctrl_kernel(int32_t* ctrl, FactorSig sig, int32_t* cnt, int64_t ncnt) {
  const int64_t x0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (x0 < kCtrlWords) {
    const int w = (int)x0;
    ctrl[w] = (w >= kSigWord && w < kSigWord + kSigWords) ? sig.w[w - kSigWord] : 0;
  }
  for (int64_t x = x0; x < ncnt; x += (int64_t)gridDim.x * blockDim.x) cnt[x] = 0;
}

__global__ void check_sig_kernel(const int32_t* fctrl, FactorSig sig, int32_t* bctrl) {
  const int w = threadIdx.x;
  const bool bad = w < kSigWords && fctrl[kSigWord + w] != sig.w[w];
  if (__any(bad) && w == 0) bctrl[1] = HQR_ERR_FACTORS;
}

// Column-major M x N matrix (leading dimension lda) <-> blocks of NB rows
// x tw columns (block (i, j) at index j * mt + i, column-major inside with
// leading dimension NB; tw = NB for the tiles of A, 64 for the blocks of
// B).  `in` fills the blocks' first `cols` columns and zeroes the padding
// beyond M and N in them; `out` copies the M x N part back (cols = N).
// The matrix holds S elements, the blocks E elements (a float copy of a
// double matrix rounds each element to nearest).
//
// Bound by HBM.  A workgroup of 256 threads takes one block row's piece of
// kCopyCols columns at a time, a row per thread, so that the only index
// arithmetic per piece is scalar and a thread has that many independent loads in
// flight.  Against one element per thread, each with its own four 64-bit
// divisions: 607 -> 323 us per copy of a batch (48 problems of up to 16384 x
// 512, 0.71 GB each way plus padding), 120 -> 99 us on average for the copies
// of a 32768 x 2048 least squares, 860 -> 812 us for 131072 x 2048 (4.3 GB,
// 5.3 TB/s).
constexpr int kCopyCols = 8;

template <typename S, typename E, int NB>
__device__ __forceinline__ void copy_piece(S* A, int64_t lda, E* At, int64_t M, int64_t N, int tw, int mt,
                                           int64_t cols, uint32_t piece, int in) {
  constexpr int PASS = 256 / NB;  // columns per pass of the workgroup
  constexpr int K = kCopyCols / PASS;
  const uint32_t cg = piece / (uint32_t)mt;
  const int i = (int)(piece - cg * (uint32_t)mt);
  const int64_t c0 = (int64_t)cg * kCopyCols;  // tw is a multiple of kCopyCols: one block holds them all
  const int64_t j = tw == 64 ? c0 / 64 : c0 / NB;
  const int lr = threadIdx.x & (NB - 1), lc = threadIdx.x / NB;
  const int64_t row = (int64_t)i * NB + lr;
  E* t = At + ((j * mt + i) * tw + (c0 - j * tw) + lc) * NB + lr;
  S* g = A + row + (c0 + lc) * lda;
  if (in) {
    S v[K];
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = (row < M && c0 + lc + k * PASS < N) ? g[(int64_t)(k * PASS) * lda] : S(0);
#pragma unroll
    for (int k = 0; k < K; ++k)
      if (c0 + lc + k * PASS < cols) t[k * PASS * NB] = (E)v[k];
  } else {
    E v[K];
#pragma unroll
    for (int k = 0; k < K; ++k)
      if (c0 + lc + k * PASS < N) v[k] = t[k * PASS * NB];
#pragma unroll
    for (int k = 0; k < K; ++k)
      if (row < M && c0 + lc + k * PASS < N) g[(int64_t)(k * PASS) * lda] = (S)v[k];
  }
}

// (fits 32 bits: at 512 elements or more each, any matrix in memory)
__host__ __device__ inline int64_t copy_pieces(int mt, int64_t cols) { return (cols + kCopyCols - 1) / kCopyCols * mt; }

template <typename S, typename E, int NB>
__global__ __launch_bounds__(256) void tile_copy_kernel(S* A, int64_t lda, E* At, int64_t M, int64_t N, int tw, int mt,
                                                        int64_t cols, int in) {
  const uint32_t total = (uint32_t)copy_pieces(mt, cols);
  for (uint32_t x = blockIdx.x; x < total; x += gridDim.x) copy_piece<S, E, NB>(A, lda, At, M, N, tw, mt, cols, x, in);
}

// Batched copy: workgroup row blockIdx.y serves problem blockIdx.y, first
// its matrix (nt tile columns), then its right-hand sides (nrt tile columns
// appended to the same tile array).  Of those, columns past the last 64-column
// chunk with a live one are left as they are: no column's values reach
// another column, and none of them is copied out, kept with a factorization
// or looked at by a solve.
template <int NB>
__global__ __launch_bounds__(256) void copy_batched_kernel(const ProbDesc* descs, char* w, int in) {
  const ProbDesc* d = descs + blockIdx.y;
  double* At = (double*)(w + d->tiles);
  double* Bt = At + (int64_t)d->mt * d->nt * NB * NB;
  const int64_t ca = in ? (int64_t)d->nt * NB : d->N, cb = in ? ((int64_t)d->nrhs + 63) / 64 * 64 : d->nrhs;
  const uint32_t ta = (uint32_t)copy_pieces(d->mt, ca), tb = (uint32_t)copy_pieces(d->mt, cb);
  for (uint32_t x = blockIdx.x; x < ta + tb; x += gridDim.x) {
    if (x < ta)
      copy_piece<double, double, NB>(d->A, d->lda, At, d->M, d->N, NB, d->mt, ca, x, in);
    else
      copy_piece<double, double, NB>(d->B, d->ldb, Bt, d->M, d->nrhs, NB, d->mt, cb, x - ta, in);
  }
}

// ---------------------------------------------------------------------------
// Triangular solves with the leading N x N upper triangle R of factored tiles
// (tile (i, j) at (j mt + i) NB^2, column-major inside, leading dimension
// NB), y overwritten by the solution; arithmetic in FP64.  Row a of y is at
// y[(a / NB) rs + a % NB]: rs = NB for a contiguous vector, NB cw for a column
// of a matrix kept in tile-row blocks of cw columns.  A zero diagonal entry
// R_jj is recorded in ctrl (status HQR_ERR_SINGULAR, *info = max over such j of
// N - j; nword, when not null, receives N).
//
// Two forms.  trsv_solve: R x = y for one column in a workgroup of 256
// threads, for many columns or many problems at once, which fill the chip.
// trsv_chain: a workgroup per block of 64 unknowns, for up to 32 columns.
// In microseconds (NB = 256), trsv_solve against trsv_chain, launch included:
// 23 / 17 for N = 256, 52 / 30 for 512, 135 / 56 for 1024, 398 / 107 for 2048
// with one column; 52 / 40 for 512 and 403 / 160 for 2048 with 32.
//
// trsv_solve takes the unknowns 64 at a time from the bottom: wave 0
// holds the block's 64 x 64 triangle in registers, one equation per lane,
// and solves it lane by lane (reciprocals of the diagonal taken in
// parallel, each new unknown broadcast with a lane read); then every thread
// removes the block from one of the rows still to be solved at a time,
// with all 64 products' loads issued together.
template <int NB>
__device__ void trsv_solve(const double* R, int mt, int64_t N, double* y, int64_t rs, int32_t* ctrl, int32_t* info,
                           int32_t* nword) {
  __shared__ double xb[64];
  __shared__ double Rd[64 * 65];  // Rd[i * 65 + j] = R(k0 + i, k0 + j), zero outside the triangle
  const int t = threadIdx.x, lane = t & 63;
  const int64_t tsz = (int64_t)NB * NB;
  const int64_t nblk = (N + 63) / 64;
  for (int64_t bi = 0; bi < nblk; ++bi) {
    const int64_t blk = nblk - 1 - bi;
    const int64_t k0 = blk * 64;
    const int nv = (int)((N - k0) < 64 ? (N - k0) : 64);
    const int64_t kt = k0 / NB, ko = k0 - kt * NB;  // the 64 rows / columns lie in tile row / column kt
    const double* Rkk = R + (kt * mt + kt) * tsz + ko + ko * NB;
    {
      // the whole 64 x 64 square lies inside tile (kt, kt): every load is
      // issued before the first is used
      double rv[16];
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        const int e = t + 256 * k, i = e & 63, j = e >> 6;
        rv[k] = Rkk[i + (int64_t)j * NB];
      }
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        const int e = t + 256 * k, i = e & 63, j = e >> 6;
        Rd[i * 65 + j] = (i < nv && j < nv && i <= j) ? rv[k] : 0.0;
      }
    }
    double* yk = y + kt * rs + ko;  // y(k0)
    __syncthreads();
    if (t < 64) {
      // cf[s]: coefficient of unknown k0 + s in this lane's equation; a lane
      // beyond the nv unknowns solves 1 x = 0 and touches no other lane
      double cf[64];
#pragma unroll
      for (int s = 0; s < 64; ++s) cf[s] = Rd[lane * 65 + s];
      const bool in = lane < nv;
      const double dg = in ? Rd[lane * 66] : 1.0;
      if (in && dg == 0.0) {
        int32_t none = 0;
        __hip_atomic_compare_exchange_strong(&ctrl[1], &none, (int32_t)HQR_ERR_SINGULAR, __ATOMIC_RELAXED,
                                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_fetch_max(info, (int32_t)(N - (k0 + lane)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (nword) __hip_atomic_store(nword, (int32_t)N, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      const double rinv = 1.0 / dg;
      double v = in ? yk[lane] : 0.0;
#pragma unroll
      for (int st = 0; st < 64; ++st) {
        const int s = 63 - st;
        const double xs = readlane(v * rinv, s);
        // lanes whose unknown is still open take the product; solved lanes keep theirs
        const double u = v - cf[s] * xs;
        v = (lane == s) ? xs : (lane < s ? u : v);
      }
      xb[lane] = lane < nv ? v : 0.0;
      if (lane < nv) yk[lane] = v;
    }
    __syncthreads();
    // rows still open, those before the block (R(a, k0 + c), stride NB in c).
    // The 64 rows of a wave lie in one tile row (a wave's first row is a
    // multiple of 64), so the tile is addressed through a buffer resource with
    // one lane offset and a constant offset per column.  Only the bottom block
    // can hold fewer than 64 unknowns.
    for (int64_t a = t; a < k0; a += 256) {
      const int64_t at = a / NB, ao = a - at * NB;
      double acc[4] = {0.0, 0.0, 0.0, 0.0};
      const __amdgpu_buffer_rsrc_t rr = rsrc(R + (kt * mt + at) * tsz);  // tile (at, kt)
      const int vo = (int)((ao + ko * NB) * (int64_t)sizeof(double));
      constexpr int CS = NB * (int)sizeof(double);  // bytes from one column to the next
      if (nv == 64) {
        double r0[64];
#pragma unroll
        for (int c = 0; c < 64; ++c) r0[c] = bload1<double>(rr, vo, c * CS);
#pragma unroll
        for (int c = 0; c < 64; ++c) acc[c & 3] += r0[c] * xb[c];
      } else {
        for (int c = 0; c < nv; ++c) acc[c & 3] += bload1<double>(rr, vo, c * CS) * xb[c];
      }
      y[at * rs + ao] -= (acc[0] + acc[1]) + (acc[2] + acc[3]);
    }
    __syncthreads();
  }
}

// R x = y for column c of a matrix Y kept in tile-row blocks of cw columns
// (block (i, jb) at Y + (jb mt + i) NB cw, column-major with leading
// dimension NB): the tile columns of B appended to the factorization
// (cw = NB) or the blocks of B of the apply path (cw = 64).
template <int NB>
__device__ __forceinline__ void trsv_column(const double* R, double* Y, int cw, int mt, int64_t N, int c,
                                            int32_t* ctrl, int32_t* info, int32_t* nword) {
  double* y = Y + (int64_t)(c / cw) * mt * NB * cw + (int64_t)(c % cw) * NB;
  trsv_solve<NB>(R, mt, N, y, (int64_t)NB * cw, ctrl, info, nword);
}

// The solves with the blocks of 64 unknowns spread over workgroups (element
// type E; TRANS = 0: R x = y from the bottom, TRANS = 1: R^T x = y from the
// top): one workgroup per block and column, which keeps its block's diagonal
// triangle in registers, takes each earlier block's unknowns as soon as they
// are published, and publishes its own.  A single workgroup is held by what one
// compute unit can read (17 MB of R at N = 2048, 43 GB/s); here the chain of
// blocks is left, one hand-over (publish, poll, read the 64 unknowns) and one
// 64-step substitution each, about 3 us a block.  The sums are taken in the
// order of trsv_solve, so both forms give the same bits.
//
// Workgroups number themselves (ticket word) in the order of the solve, so a
// workgroup waits only for ones that run already, whatever order the hardware
// starts them in; each wait is bounded by the caller's spin limit, like those of
// the persistent launch.  Words of ctrl, zero at the start and zeroed again by
// the last workgroup: [kTrsvTicket], [kTrsvDone], and per column the number of
// published blocks ([kTrsvProgress + column], on a cache line of their own).
constexpr int kTrsvTicket = 16, kTrsvDone = 17, kTrsvProgress = 32;
constexpr int kTrsvCols = 32;
static_assert(kTrsvProgress + kTrsvCols <= kCtrlWords && kTrsvTicket >= kSigWord + kSigWords, "control words");

template <typename E, int NB, int TRANS>
__device__ __forceinline__ void trsv_chain(const E* R, double* Y, int cw, int mt, int64_t N, int ncols, int32_t* ctrl,
                                           int64_t spin_limit, bool record) {
  __shared__ int32_t ticket;
  __shared__ double part[2][4][64];
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (threadIdx.x == 0)
    ticket = __hip_atomic_fetch_add(&ctrl[kTrsvTicket], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  const int tk = __builtin_amdgcn_readfirstlane(ticket);
  const int nblk = (int)((N + 63) / 64);
  const int b = tk / ncols, col = tk - b * ncols;
  if (b >= nblk) return;  // not reached: the launch has one workgroup per block and column
  const int64_t tsz = (int64_t)NB * NB, rs = (int64_t)NB * cw;
  double* y = Y + (int64_t)(col / cw) * mt * rs + (int64_t)(col % cw) * NB;
  const int blk = TRANS ? b : nblk - 1 - b;
  const int64_t k0 = (int64_t)blk * 64;
  const int nv = (int)((N - k0) < 64 ? (N - k0) : 64);
  const int64_t at = k0 / NB, ao = k0 - at * NB;
  double* yk = y + at * rs + ao;
  const bool in = lane < nv;
  // wave 0: cf[s], the coefficient of unknown k0 + s in this lane's equation
  double cf[64], rinv = 1.0, v = 0.0;
  if (w == 0) {
    const __amdgpu_buffer_rsrc_t rk = rsrc(R + (at * mt + at) * tsz);
    const int base = (int)((ao + ao * NB) * (int64_t)sizeof(E));
    const int vo = base + lane * (TRANS ? NB : 1) * (int)sizeof(E);
#pragma unroll
    for (int s = 0; s < 64; ++s) {
      const double e = (double)bload1<E>(rk, vo, s * (TRANS ? 1 : NB) * (int)sizeof(E));
      cf[s] = (in && s < nv && (TRANS ? s <= lane : lane <= s)) ? e : 0.0;
    }
    const double dr = (double)bload1<E>(rk, base + lane * (NB + 1) * (int)sizeof(E), 0);
    const double dg = in ? dr : 1.0;
    if (record && in && dg == 0.0) {
      int32_t none = 0;
      __hip_atomic_compare_exchange_strong(&ctrl[1], &none, (int32_t)HQR_ERR_SINGULAR, __ATOMIC_RELAXED,
                                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_fetch_max(&ctrl[6], (int32_t)(N - (k0 + lane)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(&ctrl[7], (int32_t)N, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    rinv = 1.0 / dg;
    v = in ? yk[lane] : 0.0;
  }
  // earlier blocks: wave w takes the unknowns w, w + 4, ... of each; the next
  // block's coefficients are loaded before this one's unknowns are waited for
  E r[16];
  auto fetch = [&](int s) {
    const int64_t c0 = (int64_t)(TRANS ? s : nblk - 1 - s) * 64;
    const int64_t ct = c0 / NB, co = c0 - ct * NB;
    const __amdgpu_buffer_rsrc_t rr = rsrc(R + (TRANS ? at * mt + ct : ct * mt + at) * tsz);
    const int vo = (int)((TRANS ? co + w + (ao + lane) * NB : ao + lane + (co + w) * NB) * (int64_t)sizeof(E));
#pragma unroll
    for (int k = 0; k < 16; ++k) r[k] = bload1<E>(rr, vo, 4 * k * (TRANS ? 1 : NB) * (int)sizeof(E));
  };
  int32_t* progress = &ctrl[kTrsvProgress + col];
  int seen = 0;
  if (b > 0) fetch(0);
  for (int s = 0; s < b; ++s) {
    const int64_t c0 = (int64_t)(TRANS ? s : nblk - 1 - s) * 64;
    const int nc = (int)((N - c0) < 64 ? (N - c0) : 64);
    int64_t spins = 0;
    while (seen <= s) {  // (blocks known to be published are not asked for again)
      seen = __builtin_amdgcn_readfirstlane(
          __hip_atomic_load(progress, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
      if (seen > s) break;
      // past the limit, or another workgroup was: results are invalid, wait
      // for nothing more
      if (++spins > spin_limit) {
        int32_t none = 0;
        if (lane == 0)
          __hip_atomic_compare_exchange_strong(&ctrl[1], &none, (int32_t)HQR_ERR_WATCHDOG, __ATOMIC_RELAXED,
                                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        seen = nblk;
        break;
      }
      if ((spins & 63) == 0 && __builtin_amdgcn_readfirstlane(__hip_atomic_load(
                                   &ctrl[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) == HQR_ERR_WATCHDOG) {
        seen = nblk;
        break;
      }
      __builtin_amdgcn_s_sleep(1);
    }
    // published unknowns are read past the caches: no invalidation is needed
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    const int xi = w + 4 * (lane & 15);
    double x = 0.0;
    if (xi < nc)
      x = __hip_atomic_load(y + c0 / NB * rs + (c0 & (NB - 1)) + xi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    double acc = 0.0;
#pragma unroll
    for (int k = 0; k < 16; ++k) acc += (w + 4 * k < nc ? (double)r[k] : 0.0) * readlane(x, k);
    if (s + 1 < b) fetch(s + 1);
    part[s & 1][w][lane] = acc;
    lds_barrier();
    if (w == 0)
      v -= (part[s & 1][0][lane] + part[s & 1][1][lane]) + (part[s & 1][2][lane] + part[s & 1][3][lane]);
  }
  if (w == 0) {
    v = in ? v : 0.0;
#pragma unroll
    for (int st = 0; st < 64; ++st) {
      const int s = TRANS ? st : 63 - st;
      const double xs = readlane(v * rinv, s);
      const double u = v - cf[s] * xs;
      v = (lane == s) ? xs : ((TRANS ? lane > s : lane < s) ? u : v);
    }
    if (in) __hip_atomic_store(&yk[lane], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // the unknowns have reached the device's point of coherence before they
    // are counted
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (lane == 0) {
      if (b + 1 < nblk) {  // nobody waits for the last block
        __hip_atomic_store(progress, b + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        // arrived before this workgroup counts as done: on its way it could
        // land after the reset below and be taken for the next solve's
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      }
      const int total = nblk * ncols;
      if (__hip_atomic_fetch_add(&ctrl[kTrsvDone], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == total - 1) {
        // every workgroup has made its last read and its last write of these words
        for (int c = 0; c < ncols; ++c)
          __hip_atomic_store(&ctrl[kTrsvProgress + c], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&ctrl[kTrsvTicket], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&ctrl[kTrsvDone], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
  }
}

template <int NB>
__global__ __launch_bounds__(256) void trsv_chain_kernel(const double* R, double* Y, int cw, int mt, int64_t N,
                                                         int ncols, int32_t* ctrl, int64_t spin_limit) {
  trsv_chain<double, NB, 0>(R, Y, cw, mt, N, ncols, ctrl, spin_limit, true);
}

// One problem: workgroup x = right-hand-side column.  A zero diagonal entry
// sets ctrl[6] = max(N - j) and ctrl[7] = N.
template <int NB>
__global__ __launch_bounds__(256) void trsv_kernel(const double* R, double* Y, int cw, int mt, int64_t N,
                                                   int32_t* ctrl) {
  trsv_column<NB>(R, Y, cw, mt, N, blockIdx.x, ctrl, &ctrl[6], &ctrl[7]);
}

// Every problem of a batch in one launch: workgroup (x, q) solves
// right-hand-side column x of problem q (its B tile columns follow the
// matrix tiles).
template <int NB>
__global__ __launch_bounds__(256) void trsv_batched_kernel(const ProbDesc* descs, char* w, int32_t* ctrl,
                                                           int32_t* info) {
  const ProbDesc* d = descs + blockIdx.y;
  if ((int)blockIdx.x >= d->nrhs) return;
  const double* R = (const double*)(w + d->tiles);
  double* Y = (double*)(w + d->tiles) + (int64_t)d->mt * d->nt * NB * NB;
  trsv_column<NB>(R, Y, NB, d->mt, d->N, blockIdx.x, ctrl, info + blockIdx.y, nullptr);
}

// ---------------------------------------------------------------------------
// Iterative refinement of least squares (FP64 residuals, FP32 factors).

// f = b - r - A x (r may be null).  A: M x N column-major (lda).  Workgroup
// of 256 threads = 64 rows x 4 column groups (each group sums every fourth
// column, eight loads in flight), partial sums combined in a fixed order.
__global__ __launch_bounds__(256) void ir_residual_kernel(const double* A, int64_t lda, int64_t M, int64_t N,
                                                          const double* x, const double* b, const double* r,
                                                          double* f) {
  __shared__ double part[4][64];
  const int lr = threadIdx.x & 63, cg = threadIdx.x >> 6;
  const int64_t row = (int64_t)blockIdx.x * 64 + lr;
  double s = 0.0;
  if (row < M) {
#pragma unroll 8
    for (int64_t j = cg; j < N; j += 4) s += A[row + j * lda] * x[j];
  }
  part[cg][lr] = s;
  __syncthreads();
  if (cg == 0 && row < M)
    f[row] = b[row] - (r ? r[row] : 0.0) - ((part[0][lr] + part[1][lr]) + (part[2][lr] + part[3][lr]));
}

// g = -A^T r (SQ = 0), or g_j = sum_i A_ij^2 (SQ = 1, r unused).
// Workgroup per IR_ATR_COLS columns (so that a launch has several
// workgroups per compute unit); 256 threads stride over the rows, four rows
// in flight each; a fixed reduction tree per column.
constexpr int IR_ATR_COLS = 2;
template <int SQ>
__global__ __launch_bounds__(256) void ir_atr_kernel(const double* A, int64_t lda, int64_t M, int64_t N,
                                                     const double* r, double* g) {
  constexpr int C = IR_ATR_COLS;
  __shared__ double part[C][257];
  const int t = threadIdx.x;
  const int64_t c0 = (int64_t)blockIdx.x * C;
  const int nc = (int)((N - c0) < C ? (N - c0) : C);
  double s[C];
#pragma unroll
  for (int c = 0; c < C; ++c) s[c] = 0.0;
#pragma unroll 4
  for (int64_t i = t; i < M; i += 256) {
    const double ri = SQ ? 0.0 : r[i];
#pragma unroll
    for (int c = 0; c < C; ++c)
      if (c < nc) {
        const double aij = A[i + (c0 + c) * lda];
        s[c] += aij * (SQ ? aij : ri);
      }
  }
#pragma unroll
  for (int c = 0; c < C; ++c) part[c][t] = s[c];
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (t < w) {
#pragma unroll
      for (int c = 0; c < C; ++c) part[c][t] += part[c][t + w];
    }
    __syncthreads();
  }
  if (t < nc) g[c0 + t] = SQ ? part[t][0] : -part[t][0];
}

// Triangular solves of the refinement with the float tiles R of the FP32
// factorization, in FP64 arithmetic, y (contiguous) overwritten:
//   TRANS = 0: R x = y,  TRANS = 1: R^T x = y.
template <int NB, int TRANS>
__global__ __launch_bounds__(256) void ir_trsv_kernel(const float* R, int mt, int64_t N, double* y, int32_t* ctrl,
                                                      int64_t spin_limit) {
  trsv_chain<float, NB, TRANS>(R, y, 1, mt, N, 1, ctrl, spin_limit, false);
}

// y = d(0:N) - h;  then d(0:N) = h  (the two uses of h in one correction).
__global__ void ir_split_kernel(double* d, const double* h, double* y, int64_t N) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < N; i += (int64_t)gridDim.x * blockDim.x) {
    y[i] = d[i] - h[i];
    d[i] = h[i];
  }
}

// x += dx (N), r += dr (M).
__global__ void ir_update_kernel(double* x, const double* dx, int64_t N, double* r, const double* dr, int64_t M) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < M; i += (int64_t)gridDim.x * blockDim.x) {
    if (i < N) x[i] += dx[i];
    r[i] += dr[i];
  }
}

// out[k] = sum of squares of vector k (v[k], n[k] entries; a null vector
// gives 0), k < 4; one workgroup, fixed order.
struct Vec4Args {
  const double* v[4];
  int64_t n[4];
};
__global__ __launch_bounds__(256) void ir_norms_kernel(Vec4Args a, double* out) {
  __shared__ double part[4][256];
  const int t = threadIdx.x;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    double sk = 0.0;
    if (a.v[k])
      for (int64_t i = t; i < a.n[k]; i += 256) sk += a.v[k][i] * a.v[k][i];
    part[k][t] = sk;
  }
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (t < w) {
#pragma unroll
      for (int k = 0; k < 4; ++k) part[k][t] += part[k][t + w];
    }
    __syncthreads();
  }
  if (t < 4) out[t] = part[t][0];
}

// Records the last HIP failure for hqr_last_error().
static thread_local char g_last_error[256];

int record_hip(hipError_t e, const char* where) {
  if (e == hipSuccess) return 0;
  snprintf(g_last_error, sizeof(g_last_error), "%s: %s", where, hipGetErrorString(e));
  return HQR_ERR_HIP;
}

const char* last_error() { return g_last_error; }

void set_last_error(const char* msg) { snprintf(g_last_error, sizeof(g_last_error), "%s", msg); }

static int grid_for(int64_t n) {
  int64_t g = (n + 255) / 256;
  if (g > 65536) g = 65536;
  if (g < 1) g = 1;
  return (int)g;
}

int launch_ir_residual(const double* A, int64_t lda, int64_t M, int64_t N, const double* x, const double* b,
                       const double* r, double* f, void* stream) {
  hipLaunchKernelGGL(ir_residual_kernel, dim3((unsigned)((M + 63) / 64)), dim3(256), 0, (hipStream_t)stream, A, lda,
                     M, N, x, b, r, f);
  return record_hip(hipGetLastError(), "ir_residual_kernel launch");
}

int launch_ir_atr(const double* A, int64_t lda, int64_t M, int64_t N, const double* r, double* g, void* stream) {
  if (r)
    hipLaunchKernelGGL(ir_atr_kernel<0>, dim3((unsigned)((N + IR_ATR_COLS - 1) / IR_ATR_COLS)), dim3(256), 0,
                       (hipStream_t)stream, A, lda, M, N, r, g);
  else
    hipLaunchKernelGGL(ir_atr_kernel<1>, dim3((unsigned)((N + IR_ATR_COLS - 1) / IR_ATR_COLS)), dim3(256), 0,
                       (hipStream_t)stream, A, lda, M, N, r, g);
  return record_hip(hipGetLastError(), "ir_atr_kernel launch");
}

int launch_ir_trsv(const float* R, int nb, int mt, int64_t N, double* y, bool trans, int32_t* ctrl, int64_t spin_limit,
                   void* stream) {
  if (spin_limit <= 0) spin_limit = kDefaultSpinLimit;
  hipStream_t s = (hipStream_t)stream;
  const dim3 g((unsigned)((N + 63) / 64)), b(256);
#define HQR_IR_TRSV(NBV)                                                                     \
  if (trans)                                                                                 \
    hipLaunchKernelGGL((ir_trsv_kernel<NBV, 1>), g, b, 0, s, R, mt, N, y, ctrl, spin_limit); \
  else                                                                                       \
    hipLaunchKernelGGL((ir_trsv_kernel<NBV, 0>), g, b, 0, s, R, mt, N, y, ctrl, spin_limit);
  switch (nb) {
    case 64: HQR_IR_TRSV(64) break;
    case 128: HQR_IR_TRSV(128) break;
    default: HQR_IR_TRSV(256) break;
  }
#undef HQR_IR_TRSV
  return record_hip(hipGetLastError(), "ir_trsv_kernel launch");
}

int launch_ir_split(double* d, const double* h, double* y, int64_t N, void* stream) {
  hipLaunchKernelGGL(ir_split_kernel, dim3(grid_for(N)), dim3(256), 0, (hipStream_t)stream, d, h, y, N);
  return record_hip(hipGetLastError(), "ir_split_kernel launch");
}

int launch_ir_update(double* x, const double* dx, int64_t N, double* r, const double* dr, int64_t M, void* stream) {
  hipLaunchKernelGGL(ir_update_kernel, dim3(grid_for(M)), dim3(256), 0, (hipStream_t)stream, x, dx, N, r, dr, M);
  return record_hip(hipGetLastError(), "ir_update_kernel launch");
}

int launch_ir_norms(const double* const* v, const int64_t* n, double* out, void* stream) {
  Vec4Args a;
  for (int k = 0; k < 4; ++k) {
    a.v[k] = v[k];
    a.n[k] = n[k];
  }
  hipLaunchKernelGGL(ir_norms_kernel, dim3(1), dim3(256), 0, (hipStream_t)stream, a, out);
  return record_hip(hipGetLastError(), "ir_norms_kernel launch");
}

int launch_zero_i32(int32_t* p, int64_t n, void* stream) {
  if (n <= 0) return 0;
  hipLaunchKernelGGL(zero_i32_kernel, dim3(grid_for(n)), dim3(256), 0, (hipStream_t)stream, p, n);
  return record_hip(hipGetLastError(), "zero_i32_kernel launch");
}

int launch_init_ctrl(int32_t* ctrl, const FactorSig& sig, int32_t* cnt, int64_t ncnt, void* stream) {
  const int64_t n = ncnt > kCtrlWords ? ncnt : kCtrlWords;
  hipLaunchKernelGGL(init_ctrl_kernel, dim3(grid_for(n)), dim3(256), 0, (hipStream_t)stream, ctrl, sig, cnt, ncnt);
  return record_hip(hipGetLastError(), "init_ctrl_kernel launch");
}

int launch_check_sig(const int32_t* fctrl, const FactorSig& sig, int32_t* bctrl, void* stream) {
  hipLaunchKernelGGL(check_sig_kernel, dim3(1), dim3(64), 0, (hipStream_t)stream, fctrl, sig, bctrl);
  return record_hip(hipGetLastError(), "check_sig_kernel launch");
}

int launch_tile_copy(void* A, int a_f32, int64_t lda, void* At, int at_f32, int64_t M, int64_t N, int nb, int tw,
                     int mt, int nt, bool in, void* stream) {
  const int64_t cols = in ? (int64_t)nt * tw : N;
  if (cols <= 0 || mt <= 0) return 0;
  int64_t pieces = copy_pieces(mt, cols);
  if (pieces > 65536) pieces = 65536;
  const dim3 g((unsigned)pieces), b(256);
  hipStream_t s = (hipStream_t)stream;
  const int i = in ? 1 : 0;
#define HQR_TILE_COPY(S, E)                                                                                          \
  switch (nb) {                                                                                                      \
    case 64:                                                                                                         \
      hipLaunchKernelGGL((tile_copy_kernel<S, E, 64>), g, b, 0, s, (S*)A, lda, (E*)At, M, N, tw, mt, cols, i);       \
      break;                                                                                                         \
    case 128:                                                                                                        \
      hipLaunchKernelGGL((tile_copy_kernel<S, E, 128>), g, b, 0, s, (S*)A, lda, (E*)At, M, N, tw, mt, cols, i);      \
      break;                                                                                                         \
    default:                                                                                                         \
      hipLaunchKernelGGL((tile_copy_kernel<S, E, 256>), g, b, 0, s, (S*)A, lda, (E*)At, M, N, tw, mt, cols, i);      \
      break;                                                                                                         \
  }
  if (!a_f32 && !at_f32) {
    HQR_TILE_COPY(double, double)
  } else if (!a_f32 && at_f32) {
    HQR_TILE_COPY(double, float)
  } else if (a_f32 && at_f32) {
    HQR_TILE_COPY(float, float)
  } else {
    return HQR_ERR_INTERNAL;
  }
#undef HQR_TILE_COPY
  return record_hip(hipGetLastError(), "tile_copy_kernel launch");
}

int launch_tile_copy(double* A, int64_t lda, double* At, int64_t M, int64_t N, int nb, int tw, int mt, int nt,
                     bool in, void* stream) {
  return launch_tile_copy(A, 0, lda, At, 0, M, N, nb, tw, mt, nt, in, stream);
}

int launch_trsv(int nb, const double* R, double* Y, int cw, int32_t* ctrl, int64_t N, int mt, int nrhs,
                int64_t spin_limit, void* stream) {
  if (nrhs <= 0) return 0;
  if (spin_limit <= 0) spin_limit = kDefaultSpinLimit;
  hipStream_t s = (hipStream_t)stream;
  const int64_t nblk = (N + 63) / 64;
  // The spread form is the faster one wherever it can run; its line is the
  // number of control words, one per column, not where the times cross: at 33
  // columns the other form takes 52 us for N = 512 and 400 us for N = 2048,
  // this one at 32 columns 39 and 158.
  if (nrhs <= kTrsvCols) {
    const dim3 g((unsigned)(nblk * nrhs)), b(256);
    switch (nb) {
      case 64: hipLaunchKernelGGL(trsv_chain_kernel<64>, g, b, 0, s, R, Y, cw, mt, N, nrhs, ctrl, spin_limit); break;
      case 128: hipLaunchKernelGGL(trsv_chain_kernel<128>, g, b, 0, s, R, Y, cw, mt, N, nrhs, ctrl, spin_limit); break;
      default: hipLaunchKernelGGL(trsv_chain_kernel<256>, g, b, 0, s, R, Y, cw, mt, N, nrhs, ctrl, spin_limit); break;
    }
    return record_hip(hipGetLastError(), "trsv_chain_kernel launch");
  }
  switch (nb) {
    case 64: hipLaunchKernelGGL(trsv_kernel<64>, dim3(nrhs), dim3(256), 0, s, R, Y, cw, mt, N, ctrl); break;
    case 128: hipLaunchKernelGGL(trsv_kernel<128>, dim3(nrhs), dim3(256), 0, s, R, Y, cw, mt, N, ctrl); break;
    default: hipLaunchKernelGGL(trsv_kernel<256>, dim3(nrhs), dim3(256), 0, s, R, Y, cw, mt, N, ctrl); break;
  }
  return record_hip(hipGetLastError(), "trsv_kernel launch");
}

int launch_copy_batched(const ProbDesc* d, char* w, int count, int nb, bool in, int64_t max_elems, void* stream) {
  if (count <= 0) return 0;
  // workgroups per problem: one for every two pieces of the largest problem
  int64_t gx = (max_elems / nb / kCopyCols + 1) / 2;
  if (gx < 1) gx = 1;
  if (gx > 4096) gx = 4096;
  const dim3 g((unsigned)gx, count), b(256);
  hipStream_t s = (hipStream_t)stream;
  const int i = in ? 1 : 0;
  switch (nb) {
    case 64: hipLaunchKernelGGL(copy_batched_kernel<64>, g, b, 0, s, d, w, i); break;
    case 128: hipLaunchKernelGGL(copy_batched_kernel<128>, g, b, 0, s, d, w, i); break;
    default: hipLaunchKernelGGL(copy_batched_kernel<256>, g, b, 0, s, d, w, i); break;
  }
  return record_hip(hipGetLastError(), "copy_batched_kernel launch");
}

int launch_trsv_batched(int nb, const ProbDesc* d, char* w, int32_t* ctrl, int32_t* info, int count, int max_nrhs,
                        void* stream) {
  if (count <= 0 || max_nrhs <= 0) return 0;
  const dim3 grid(max_nrhs, count), block(256);
  hipStream_t s = (hipStream_t)stream;
  switch (nb) {
    case 64: hipLaunchKernelGGL(trsv_batched_kernel<64>, grid, block, 0, s, d, w, ctrl, info); break;
    case 128: hipLaunchKernelGGL(trsv_batched_kernel<128>, grid, block, 0, s, d, w, ctrl, info); break;
    default: hipLaunchKernelGGL(trsv_batched_kernel<256>, grid, block, 0, s, d, w, ctrl, info); break;
  }
  return record_hip(hipGetLastError(), "trsv_batched_kernel launch");
}

template <typename E, int NB>
static int occupancy_workers() {
  int dev = 0, cus = 0, per = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 1;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 1;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, persistent_kernel<E, NB, false>, NT, sizeof(Smem<E, NB>)) != hipSuccess ||
      per < 1)
    per = 1;
  return cus * per;
}

int default_workers(int nb, bool f32) {
  if (f32) {
    switch (nb) {
      case 64: return occupancy_workers<float, 64>();
      case 128: return occupancy_workers<float, 128>();
      default: return occupancy_workers<float, 256>();
    }
  }
  switch (nb) {
    case 64: return occupancy_workers<double, 64>();
    case 128: return occupancy_workers<double, 128>();
    default: return occupancy_workers<double, 256>();
  }
}

template <typename E, bool BF = false>
static int launch_persistent_t(int nb, const LaunchArgs& a, int workers, hipStream_t s) {
  const dim3 g(workers), b(NT);
  if (a.probs) {
    switch (nb) {
      case 64: hipLaunchKernelGGL((persistent_kernel<E, 64, true>), g, b, sizeof(Smem<E, 64>), s, a); break;
      case 128: hipLaunchKernelGGL((persistent_kernel<E, 128, true>), g, b, sizeof(Smem<E, 128>), s, a); break;
      case 256: hipLaunchKernelGGL((persistent_kernel<E, 256, true>), g, b, sizeof(Smem<E, 256>), s, a); break;
      default: return HQR_ERR_INTERNAL;
    }
  } else {
    switch (nb) {
      case 64: hipLaunchKernelGGL((persistent_kernel<E, 64, false, BF>), g, b, sizeof(Smem<E, 64>), s, a); break;
      case 128: hipLaunchKernelGGL((persistent_kernel<E, 128, false, BF>), g, b, sizeof(Smem<E, 128>), s, a); break;
      case 256: hipLaunchKernelGGL((persistent_kernel<E, 256, false, BF>), g, b, sizeof(Smem<E, 256>), s, a); break;
      default: return HQR_ERR_INTERNAL;
    }
  }
  return record_hip(hipGetLastError(), "persistent_kernel launch");
}

int launch_persistent(int nb, const LaunchArgs& a, int workers, void* stream, bool f32, bool bf16) {
  if (workers < 1) workers = 1;
  // the batched path runs in FP64 only; BF16 products take float tiles
  if (f32 && a.probs) return HQR_ERR_INTERNAL;
  if (bf16 && (!f32 || a.B)) return HQR_ERR_INTERNAL;
  if (bf16) return launch_persistent_t<float, true>(nb, a, workers, (hipStream_t)stream);
  return f32 ? launch_persistent_t<float>(nb, a, workers, (hipStream_t)stream)
             : launch_persistent_t<double>(nb, a, workers, (hipStream_t)stream);
}

}  // namespace hqr
