// kernels.hip -- gfx950 (CDNA4) device code of the sparse tile Cholesky.
//
// One persistent kernel executes every tile task of the factorization
// (Algorithm 1: SYRK/GEMM updates, POTRF, TRSM; Algorithm 3: partial
// accumulations and the GEADD tree) and of the triangular solves.  Workgroups
// of 256 threads (4 wave64) take tickets in the static order computed on the
// host and wait on a per-task counter of unfinished predecessors, the
// counterpart of the paper's progress table (Algorithm 2).
//
// Tile products use the FP64 matrix cores (v_mfma_f64_16x16x4f64) or, in the
// mixed mode, the FP32 ones (v_mfma_f32_16x16x4f32) on FP32 copies of the
// factor tiles.  Each wave owns a (T/2) x (T/2) quarter of the output tile.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>
#include <utility>

#include "launch.h"
#include "stiles_internal.h"

namespace stiles {

typedef double v4d __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int NT = 256;

// Global-memory accesses go through address-space-1 pointers, so that they
// are global (not flat) instructions: they then count only in vmcnt, and a
// wait for LDS data (lgkmcnt) never waits for a tile prefetch in flight.
#define GLOBAL __attribute__((address_space(1)))
#define INLINE __attribute__((always_inline))   // lambdas
template <typename E>
__device__ __forceinline__ GLOBAL E* gp(E* p) { return (GLOBAL E*)p; }
template <typename E>
__device__ __forceinline__ const GLOBAL E* gp(const E* p) { return (const GLOBAL E*)p; }

// Thread index for the task bodies, opaque to the compiler: the executor
// inlines every task body into its loop, and address arithmetic that depends
// only on the thread index would be moved out of the loop and kept in
// registers (then spilled) across all of them.
__device__ __forceinline__ int thread_id() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  __builtin_assume(t >= 0 && t < NT);
  return t;
}

// The pair (or slot) words of a task, read once: lane l of every wave holds
// word l (at most 64 words); word i is then taken with readlane into a scalar
// register, so the loop over the pairs issues no dependent metadata loads.
__device__ __forceinline__ int load_words(const int32_t* w, int n) {
  const int l = thread_id() & 63;
  return l < n ? gp(w)[l] : 0;
}
__device__ __forceinline__ int word(int v, int i) { return __builtin_amdgcn_readlane(v, i); }

// The eight words of a task, in scalar registers; pv: the first 64 words of
// its operand list (one per lane).  Both are static and are read before the
// task waits for its predecessors.
struct Task {
  int w[TASK_WORDS];
  int pv;
  __device__ __forceinline__ int operator[](int i) const { return w[i]; }
};

// Stores of task results are device-scope (sc1) stores: they are written
// through to the point of coherence of all XCDs, so once they have completed
// (s_waitcnt) they are visible to a task on any XCD that acquires after it.
// A task's release then needs no L2 write-back (buffer_wbl2), which costs
// about as much as several tile products.  Every global store of the task
// bodies must go through these.
__device__ __forceinline__ void st_dev(GLOBAL double* p, double v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_dev(GLOBAL float* p, float v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_dev(double* p, double v) { st_dev(gp(p), v); }
// The same for 16 bytes of a tile or vector block (an atomic store has at most 8): a buffer
// store, whose cache policy is an operand.  As inline asm the compiler would
// not count it, and a later wait for loads issued before it would wait for
// the store too.
typedef double v2d __attribute__((ext_vector_type(2)));
typedef unsigned v4u __attribute__((ext_vector_type(4)));
struct DevBlock {
  __amdgpu_buffer_rsrc_t rsrc;
  __device__ __forceinline__ DevBlock(double* block, int64_t bytes)
      : rsrc(__builtin_amdgcn_make_buffer_rsrc(block, 0, (int)bytes, 0x00020000)) {}
  // elements e and e + 1, e even
  __device__ __forceinline__ void store(int e, v2d v) const {
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, v), rsrc, 8 * e, 0, /* sc1 */ 16);
  }
  __device__ __forceinline__ void store(int e, v4d v) const {
    store(e, v2d{v[0], v[1]});
    store(e + 2, v2d{v[2], v[3]});
  }
  __device__ __forceinline__ void store(int e, double v) const {
    typedef unsigned v2u __attribute__((ext_vector_type(2)));
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(v2u, v), rsrc, 8 * e, 0, /* sc1 */ 16);
  }
};
template <int T>
struct DevTile : DevBlock {
  __device__ __forceinline__ explicit DevTile(double* tile) : DevBlock(tile, T * T * 8) {}
};

// ------------------------------------------------------------------ helpers

__device__ __forceinline__ int ld_relaxed(int32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_relaxed(int32_t* p, int32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void fence_acquire() { __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent"); }
__device__ __forceinline__ void fence_release() { __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent"); }

// ------------------------------------------------------- tile products (MFMA)
// 16 x 16 x 4 products: lane l holds A[l & 15][l >> 4], B[l >> 4][l & 15] and,
// in register r of the result, D[col(l, r)][l & 15].  The A operand is taken
// from Y (columns of C), the B operand from X (rows of C), so that the 16
// lanes of one row group touch neighbouring rows of a column-major tile.
template <typename E>
struct Mma;
template <>
struct Mma<double> {
  typedef v4d acc_t;
  static __device__ __forceinline__ v4d mfma(double a, double b, v4d c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int col(int lane, int r) { return (lane >> 4) + 4 * r; }   // result column
};
template <>
struct Mma<float> {
  typedef v4f acc_t;
  static __device__ __forceinline__ v4f mfma(float a, float b, v4f c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int col(int lane, int r) { return 4 * (lane >> 4) + r; }
};

// Whole-tile staging through registers: every thread moves its share of a
// T x T tile with 16-byte loads, so a tile arrives after one memory latency
// and the next pair can be in flight while the current one is multiplied.
template <int T, typename E>
struct TileStage {
  typedef E vec __attribute__((ext_vector_type(16 / sizeof(E))));
  static constexpr int EPV = 16 / sizeof(E);
  static constexpr int NV = T * T / NT / EPV;
  vec r[NV];
  __device__ __forceinline__ void load(const E* __restrict__ g) {
    const GLOBAL vec* v = (const GLOBAL vec*)g;
#pragma unroll
    for (int q = 0; q < NV; q++) r[q] = v[thread_id() + q * NT];
  }
  __device__ __forceinline__ void store(E* l) const {
    vec* v = reinterpret_cast<vec*>(l);
#pragma unroll
    for (int q = 0; q < NV; q++) v[thread_id() + q * NT] = r[q];
  }
};

// ------------------------------------------------------------ task bodies

struct Wait {
  ExecCtrl* ctrl;
  uint64_t limit;
  int32_t* flag;   // in LDS
};

// The calling workgroup waits until *cnt < bound (all predecessors, or all
// predecessors of one kind, have finished), then acquires.  Wave 0 polls.
// The wait is bounded: it gives up when another workgroup of the launch has
// given up (ctrl->abort) or when `limit` ticks of the 100 MHz wall clock pass
// without the counter falling; the first to give up sets ctrl->abort.  The
// result is the same for every thread (false: gave up).  The outcome goes
// through LDS (flag); the second barrier keeps a later wait from overwriting
// it before every wave has read it.
__device__ __forceinline__ bool wait_below(int32_t* cnt, int32_t bound, const Wait& wt) {
  if (thread_id() < 64) {
    int32_t ok = 1;
    if (__builtin_amdgcn_readfirstlane(ld_relaxed(cnt)) >= bound) {
      const uint64_t t0 = wall_clock64();
      for (;;) {
        __builtin_amdgcn_s_sleep(1);
        if (__builtin_amdgcn_readfirstlane(ld_relaxed(cnt)) < bound) break;
        if (__builtin_amdgcn_readfirstlane(ld_relaxed(&wt.ctrl->abort)) != 0) {
          ok = 0;
          break;
        }
        if (wall_clock64() - t0 > wt.limit) {
          st_relaxed(&wt.ctrl->abort, 1);
          ok = 0;
          break;
        }
      }
    }
    fence_acquire();
    if (thread_id() == 0) *wt.flag = ok;
  }
  __syncthreads();
  const bool ok = __builtin_amdgcn_readfirstlane(*wt.flag) != 0;
  __syncthreads();
  return ok;
}

// Waits until *a < ba (the answer 1) or, failing that, *b < bb (2); 0 if the
// launch is abandoned.
__device__ __forceinline__ int wait_first(int32_t* a, int32_t ba, int32_t* b, int32_t bb, const Wait& wt) {
  if (thread_id() < 64) {
    int32_t which = 0;
    const uint64_t t0 = wall_clock64();
    for (;;) {
      const int32_t va = ld_relaxed(a), vb = ld_relaxed(b);
      if (__builtin_amdgcn_readfirstlane(va) < ba) which = 1;
      else if (__builtin_amdgcn_readfirstlane(vb) < bb) which = 2;
      if (which != 0) break;
      if (__builtin_amdgcn_readfirstlane(ld_relaxed(&wt.ctrl->abort)) != 0) break;
      if (wall_clock64() - t0 > wt.limit) {
        st_relaxed(&wt.ctrl->abort, 1);
        break;
      }
      __builtin_amdgcn_s_sleep(1);
    }
    fence_acquire();
    if (thread_id() == 0) *wt.flag = which;
  }
  __syncthreads();
  const int which = __builtin_amdgcn_readfirstlane(*wt.flag);
  __syncthreads();
  return which;
}

// ---- operand ring of the update products
// Tile pairs stream through LDS in stages of KS columns of X and of Y (a
// column range of a column-major tile is contiguous), written by the memory
// system itself (global_load_lds: no staging registers and no LDS store
// instructions).  With NST slots the next NST - 2 stages have been issued
// when a stage's products begin, and one more follows during them; one
// barrier per stage, after its first step so that the matrix cores work
// meanwhile, says both that the next stage has arrived and that the slot of
// the previous one is free.  At T = 64 (four slots) it leaves the stage after
// the next in flight; at T = 32 (three, whole operand tiles) the next stage
// is the only one, and the barrier waits for it.  Tiles staged whole through registers gave the
// matrix cores nothing to do while a pair was stored to LDS and the next
// one's 16 loads went out; 512 workgroups of 12-product tasks on tiles in
// L2: FP64 49 -> 58 TFLOP/s, FP32 96 -> 105; on tiles in HBM both are bound by
// it (43 -> 44, 87 -> 89).
template <int T, typename E>
struct Ring {
  static constexpr int KS = T == 64 && sizeof(E) == 8 ? 16 : 32;   // columns per stage
  static constexpr int SPP = T / KS;                               // stages per tile pair
  static constexpr int HB = T * KS * (int)sizeof(E);               // bytes of one operand's stage
  static constexpr int NI = 2 * HB / 4096;                         // 1 KB transfers per wave and stage
  static constexpr int NST = T == 64 ? 4 : 3;                      // slots (64 KB; 48 KB at T = 32)
  static_assert(NST * 2 * HB <= 65536, "transfers address LDS below 64 KB, the ring starts at 0 (ExecLds)");
};

// 1 KB from base + voff (voff per lane) to LDS at lds + 16 lane.  No register
// is written, so nothing can be overwritten by a transfer in flight; it
// counts in vmcnt.  The LDS address goes in M0, which the compiler sets for
// this operand (it then knows what M0 holds; a write inside the statement
// would have to name a reserved register as clobbered); the wait state
// between that write and the transfer is in the statement.
__device__ __forceinline__ void lds_transfer(uint32_t lds, uint32_t voff, const char* base) {
  asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "{m0}"(lds), "v"(voff), "s"(base) : "memory");
}

// waits until at most `n` of this wave's newest transfers (n = 0, NI or 2 NI)
// are in flight, then for the other waves
template <int NI>
__device__ __forceinline__ void ring_barrier(int n) {
  if (n >= 2 * NI) asm volatile("s_waitcnt vmcnt(%0)" : : "n"(2 * NI) : "memory");
  else if (n >= NI) asm volatile("s_waitcnt vmcnt(%0)" : : "n"(NI) : "memory");
  else asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" : : : "memory");
}

// acc += sum over the np tile pairs of pv of X_p Y_p^T, this wave's quarter
// (rows r0, columns c0; none if !active), operands from `tiles`.  Block j of
// the quarter holds its rows 2 i + j (i = 0..15), block i its columns
// 2 j + i, so that a lane reads its operands for both blocks as one pair of
// neighbours: 16-byte LDS reads run at twice the rate of 8-byte ones, and
// the matrix cores of a lone workgroup wait for them (cycles per FP64 MFMA
// in a loop of reads and MFMAs: 69 against 81, without reads 64; two
// workgroups a CU 66 against 72).
template <int T, typename E>
__device__ __forceinline__ void ring_products(typename Mma<E>::acc_t (&acc)[T / 32][T / 32], const E* tiles, int pv,
                                              int np, E* ring, int r0, int c0, bool active) {
  typedef Ring<T, E> R;
  constexpr int NB = T / 32, NI = R::NI, NST = R::NST;
  const int tid = thread_id(), lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)ring + 1024 * wave;
  const uint32_t voff = 1024 * wave + 16 * lane;
  const int total = np * R::SPP;
  // transfer i of stage s into its slot
  const char *xb, *yb;
  uint32_t dst;
  auto stage = [&](int s, int slot) {
    const int p = s / R::SPP;
    const int64_t part = (int64_t)(s % R::SPP) * R::HB;
    xb = (const char*)(tiles + (int64_t)word(pv, 2 * p) * T * T) + part;
    yb = (const char*)(tiles + (int64_t)word(pv, 2 * p + 1) * T * T) + part;
    dst = lds0 + (uint32_t)slot * 2 * R::HB;
  };
  auto transfer = [&](int i) {
    const int c = 4096 * (i % (NI / 2));
    if (i < NI / 2) lds_transfer(dst + c, voff + c, xb);
    else lds_transfer(dst + R::HB + c, voff + c, yb);
  };
#pragma unroll
  for (int s = 0; s < NST - 1; s++)
    if (s < total) {
      stage(s, s);
#pragma unroll
      for (int i = 0; i < NI; i++) transfer(i);
    }
  ring_barrier<NI>((total < NST - 1 ? total : NST - 1) * NI - NI);
  int slot = 0, wslot = NST - 1;
  const int xo = r0 + NB * (lane & 15) + (lane >> 4) * T;
  const int yo = c0 + NB * (lane & 15) + (lane >> 4) * T + R::HB / (int)sizeof(E);
  typedef E vec __attribute__((ext_vector_type(NB)));
  constexpr int SLOT = 2 * R::HB / (int)sizeof(E);
  E a[NB], b[NB];
  {
    const vec y = *(const vec*)(ring + yo), x = *(const vec*)(ring + xo);
#pragma unroll
    for (int q = 0; q < NB; q++) {
      a[q] = y[q];
      b[q] = x[q];
    }
  }
#pragma unroll 1
  for (int s = 0; s < total; s++) {
    const E* cur = ring + slot * SLOT;
    slot = slot + 1 == NST ? 0 : slot + 1;
    const E* nxt = ring + slot * SLOT;
    const bool more = s + NST - 1 < total;
#pragma unroll
    for (int k = 0; k < R::KS; k += 4) {
      // the operands of the next step (at the end, of the next stage's first
      // one) are read from LDS while this step's MFMAs run
      E an[NB], bn[NB];
      const E* src = k + 4 < R::KS ? cur + (k + 4) * T : nxt;
      {
        const vec y = *(const vec*)(src + yo), x = *(const vec*)(src + xo);
#pragma unroll
        for (int q = 0; q < NB; q++) {
          an[q] = y[q];
          bn[q] = x[q];
        }
      }
      if (k >= 4 && more) {
#pragma unroll
        for (int i = (k / 4 - 1) * NI / (R::KS / 4 - 1); i < (k / 4) * NI / (R::KS / 4 - 1); i++) transfer(i);
      }
      __builtin_amdgcn_sched_barrier(0);
      if (active) {
#pragma unroll
        for (int i = 0; i < NB; i++)
#pragma unroll
          for (int j = 0; j < NB; j++) acc[i][j] = Mma<E>::mfma(a[i], b[j], acc[i][j]);
      }
      if (k == 0) {
        // early in the stage: the next one has arrived, and no wave still
        // reads the previous one, whose slot takes the next transfers
        const int last = s + NST - 2 < total ? s + NST - 2 : total - 1;
        if (s + 1 < total) ring_barrier<NI>((last - (s + 1)) * NI);
        if (more) stage(s + NST - 1, wslot);
        wslot = wslot + 1 == NST ? 0 : wslot + 1;
      }
#pragma unroll
      for (int q = 0; q < NB; q++) {
        a[q] = an[q];
        b[q] = bn[q];
      }
    }
  }
}

// UPD / PART: acc = sum_p X_p Y_p^T over a list of tile pairs (at most 32).
// mode 0: C_t -= acc (UPD), mode 1: P = acc (PART).  E = double on the factor
// tiles, float on their FP32 copies (mixed mode; the sum is then applied to
// the FP64 tile).
template <int T, typename E>
__device__ __forceinline__ void update_products(const ExecMat& M, const Task& w, int mode, const E* tiles, E* ring) {
  constexpr int TT = T * T, W = T / 2, NB = T / 32;
  const int tid = thread_id(), lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r0 = (wave >> 1) * W, c0 = (wave & 1) * W;
  const bool diag = (w[0] & TF_DIAG) != 0;
  const bool active = !(diag && c0 > r0);   // strictly upper quarter of a diagonal tile
  const bool accum = mode == 1 && (w[0] & TF_ACC) != 0;   // partial chain: P += sum
  double* const tile = mode == 0 ? M.tiles + (int64_t)w[1] * TT : M.part + (int64_t)w[4] * TT;
  const GLOBAL double* out = gp(tile);
  const DevTile<T> dev(tile);
  // this lane's elements: rows row0 + j, columns col(i, r)
  const int row0 = r0 + NB * (lane & 15);
  auto col = [&](int i, int r) { return c0 + NB * Mma<E>::col(lane, r) + i; };
  typedef double vec __attribute__((ext_vector_type(NB)));
  // the target's current value is needed only at the end: fetch it now
  vec cin[NB][4];
  if ((mode == 0 || accum) && active) {
#pragma unroll
    for (int i = 0; i < NB; i++)
#pragma unroll
      for (int r = 0; r < 4; r++) cin[i][r] = *(const GLOBAL vec*)(out + row0 + col(i, r) * T);
  }
  typename Mma<E>::acc_t acc[NB][NB];
#pragma unroll
  for (int i = 0; i < NB; i++)
#pragma unroll
    for (int j = 0; j < NB; j++) acc[i][j] = typename Mma<E>::acc_t{0, 0, 0, 0};
  ring_products<T, E>(acc, tiles, w.pv, w[3] - w[2], ring, r0, c0, active);
  if (!active && mode == 0) return;
#pragma unroll
  for (int i = 0; i < NB; i++)
#pragma unroll
    for (int r = 0; r < 4; r++) {
      vec v;
#pragma unroll
      for (int j = 0; j < NB; j++) {
        const double x = (double)acc[i][j][r];
        // above the diagonal the target keeps its value; an inactive
        // quarter's zeros keep a partial fully defined
        if (mode == 0) v[j] = !diag || row0 + j >= col(i, r) ? cin[i][r][j] - x : cin[i][r][j];
        else v[j] = accum && active ? cin[i][r][j] + x : x;
      }
      if constexpr (NB == 2) dev.store(row0 + col(i, r) * T, v2d{v[0], v[NB - 1]});
      else dev.store(row0 + col(i, r) * T, v[0]);
    }
}

template <int T>
__device__ __forceinline__ void task_update(const ExecMat& M, const Task& w, int mode, double* ring) {
  // FP32 products in mixed mode: the updates, and the partials of corner
  // tiles other than the arrow corner (separator rows under adaptable ND);
  // the arrow corner's partials too in the all-FP32 variant (mixed == 2)
  if (M.mixed && (mode == 0 || M.mixed == 2 || (w[0] & TF_ARROW) == 0))
    update_products<T, float>(M, w, mode, M.shadow, reinterpret_cast<float*>(ring));
  else
    update_products<T, double>(M, w, mode, M.tiles, ring);
}

// UPDB: a 2 x 2 block of update targets C_(r,c) -= sum_j L_(r,j) L_(c,j)^T,
// r in {ra, rb}, c in {k, k+1}, over a list of columns j.  Wave q owns
// target q: rows from operand X_(q & 1) = L_(ra|rb, j), columns from
// Y_(q >> 1) = L_(k|k+1, j), a whole T x T tile in its registers, so each
// operand tile is read once from memory for two products.  Per column j
// the four operand tiles go through LDS in two halves of T/2 k-columns
// (X halves in LX, Y halves in LY; a half of a column-major tile is
// contiguous); the next half is in flight in registers while the current
// one is multiplied.  The diagonal block (TF_DIAG: ra = k, rb = k+1) reads
// X_a = Y_k and X_b = Y_(k+1), stages only the Y halves, and its two
// diagonal targets compute their lower 16 x 16 blocks only.  E = double on
// the FP64 factor tiles, float on the FP32 copies in mixed mode (the
// product is then subtracted from the FP64 tile).
template <int T, typename E>
__device__ __forceinline__ void update_block(const ExecMat& M, const Task& w, const E* tiles, double* LXd, double* LYd) {
  typedef Mma<E> O;
  typedef typename O::acc_t acc_t;
  typedef E vec __attribute__((ext_vector_type(16 / sizeof(E))));
  constexpr int TT = T * T, H = T / 2, HE = T * H, NB = T / 16;
  constexpr int EPV = 16 / sizeof(E), NV = HE / NT / EPV;   // vectors per thread per half tile
  E* LX = reinterpret_cast<E*>(LXd);
  E* LY = reinterpret_cast<E*>(LYd);
  const int lane = thread_id() & 63;
  const int wave = __builtin_amdgcn_readfirstlane(thread_id() >> 6);
  const bool dg = (w[0] & TF_DIAG) != 0;
  const int nj = w[3];
  const int pv = w.pv;
  const int tgt = word(pv, wave);
  const bool active = tgt >= 0;
  const bool tdiag = dg && wave != 1;
  const int xs = wave & 1, ys = wave >> 1;
  // staged halves: the Y tiles (k, j), (k+1, j), then (non-diagonal block)
  // the X tiles (ra, j), (rb, j)
  const int nst = dg ? 2 : 4;
  vec st[4][NV];
  // an operand tile id of -1 (absent) is neither loaded nor used: the waves
  // whose X or Y it is skip that column
  auto stage_load = [&](int step) {
    const int j = step >> 1, h = step & 1;
#pragma unroll
    for (int q = 0; q < 4; q++) {
      // slot order in the list: xa, xb, yk, yk1
      const int id = q < nst ? word(pv, 4 + 4 * j + (q < 2 ? 2 + q : q - 2)) : -1;
      if (id >= 0) {
        const GLOBAL vec* g = (const GLOBAL vec*)(tiles + (int64_t)id * TT + h * HE);
#pragma unroll
        for (int v = 0; v < NV; v++) st[q][v] = g[thread_id() + v * NT];
      }
    }
  };
  auto stage_store = [&](int step) {
    const int j = step >> 1;
#pragma unroll
    for (int q = 0; q < 4; q++) {
      const int id = q < nst ? word(pv, 4 + 4 * j + (q < 2 ? 2 + q : q - 2)) : -1;
      if (id >= 0) {
        vec* l = reinterpret_cast<vec*>((q < 2 ? LY : LX) + (q & 1) * HE);
#pragma unroll
        for (int v = 0; v < NV; v++) l[thread_id() + v * NT] = st[q][v];
      }
    }
  };
  acc_t acc[NB][NB];
#pragma unroll
  for (int i = 0; i < NB; i++)
#pragma unroll
    for (int jj = 0; jj < NB; jj++) acc[i][jj] = acc_t{0, 0, 0, 0};
  const E* xl = (dg ? LY : LX) + xs * HE + (lane & 15) + (lane >> 4) * T;
  const E* yl = LY + ys * HE + (lane & 15) + (lane >> 4) * T;
  const int nsteps = 2 * nj;
  bool any = false;   // this wave's target received a product
  stage_load(0);
  for (int step = 0; step < nsteps; step++) {
    __syncthreads();
    stage_store(step);
    __syncthreads();
    if (step + 1 < nsteps) stage_load(step + 1);
    const int j = step >> 1;
    const bool use = active && word(pv, 4 + 4 * j + xs) >= 0 && word(pv, 4 + 4 * j + 2 + ys) >= 0;
    any |= use;
    if (use) {
#pragma unroll 2
      for (int k = 0; k < H; k += 4) {
        E a[NB], b[NB];
#pragma unroll
        for (int q = 0; q < NB; q++) {
          a[q] = yl[q * 16 + k * T];
          b[q] = xl[q * 16 + k * T];
        }
#pragma unroll
        for (int i = 0; i < NB; i++)
#pragma unroll
          for (int jj = 0; jj < NB; jj++)
            if (!tdiag || jj >= i) acc[i][jj] = O::mfma(a[i], b[jj], acc[i][jj]);
      }
    }
  }
  if (!any) return;
  GLOBAL double* out = gp(M.tiles + (int64_t)tgt * TT);
#pragma unroll
  for (int i = 0; i < NB; i++) {
    double cin[NB][4];
#pragma unroll
    for (int jj = 0; jj < NB; jj++)
#pragma unroll
      for (int r = 0; r < 4; r++) {
        const int row = 16 * jj + (lane & 15), col = 16 * i + O::col(lane, r);
        cin[jj][r] = (!tdiag || jj >= i) ? out[row + col * T] : 0.0;
      }
#pragma unroll
    for (int jj = 0; jj < NB; jj++)
#pragma unroll
      for (int r = 0; r < 4; r++) {
        const int row = 16 * jj + (lane & 15), col = 16 * i + O::col(lane, r);
        if (!tdiag || row >= col) st_dev(out + row + col * T, cin[jj][r] - (double)acc[i][jj][r]);
      }
  }
}

// The one task body that is a function: it needs nearly every register, and
// blocks are off by default.  M stays in global memory for it (a descriptor
// whose address is taken would live in scratch memory).
template <int T, int K>   // K: a copy for every kernel kind, not one compiled for all
__device__ __attribute__((noinline)) void task_update_block(const ExecMat* M, int w0, int nj, int pv, double* LX,
                                                            double* LY) {
  Task w;
  w.w[0] = __builtin_amdgcn_readfirstlane(w0);
  w.w[3] = __builtin_amdgcn_readfirstlane(nj);
  w.pv = pv;
  if (M->mixed) update_block<T, float>(*M, w, M->shadow, LX, LY);
  else update_block<T, double>(*M, w, M->tiles, LX, LY);
}

// TREE: P_c = P_a + P_b, or C_t -= P_a (+ P_b) at the root (Alg. 3 GEADD).
template <int T>
__device__ __forceinline__ void task_tree(const ExecMat& M, const Task& w) {
  constexpr int TT = T * T;
  typedef double d2 __attribute__((ext_vector_type(2)));
  const GLOBAL d2* pa = (const GLOBAL d2*)(M.part + (int64_t)w[2] * TT);
  const GLOBAL d2* pb = w[3] >= 0 ? (const GLOBAL d2*)(M.part + (int64_t)w[3] * TT) : nullptr;
  GLOBAL d2* dst = w[4] >= 0 ? (GLOBAL d2*)(M.part + (int64_t)w[4] * TT) : (GLOBAL d2*)(M.tiles + (int64_t)w[1] * TT);
  const bool apply = w[4] < 0;
#pragma unroll 4
  for (int e = thread_id(); e < TT / 2; e += NT) {
    const d2 s = pb ? pa[e] + pb[e] : pa[e];
    const d2 v = apply ? dst[e] - s : s;
    GLOBAL double* o = (GLOBAL double*)(dst + e);
    st_dev(o, v.x);
    st_dev(o + 1, v.y);
  }
}

// acc += rows r0 .. r0 + 15 of X Y^T: acc[i] covers columns 16 i + (lane >> 4)
// + 4 q of row r0 + (lane & 15); X, Y: whole tiles in LDS
template <int T>
__device__ __forceinline__ void mma_strip(v4d (&acc)[T / 16], const double* X, const double* Y, int r0, int lane) {
  constexpr int NB = T / 16;
  const double* xp = X + r0 + (lane & 15) + (lane >> 4) * T;
  const double* yp = Y + (lane & 15) + (lane >> 4) * T;
  double b = xp[0], a[NB];
#pragma unroll
  for (int i = 0; i < NB; i++) a[i] = yp[16 * i];
#pragma unroll
  for (int k = 0; k < T; k += 4) {
    double bn = 0.0, an[NB];
    if (k + 4 < T) {
      bn = xp[(k + 4) * T];
#pragma unroll
      for (int i = 0; i < NB; i++) an[i] = yp[16 * i + (k + 4) * T];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < NB; i++) acc[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b, acc[i], 0, 0, 0);
    if (k + 4 < T) {
      b = bn;
#pragma unroll
      for (int i = 0; i < NB; i++) a[i] = an[i];
    }
  }
}

// A diagonal tile into POTRF's buffer (leading dimension T + 17), with the
// identity blocks below it.
template <int T>
__device__ __forceinline__ void stage_diag(const double* C, double* S) {
  constexpr int LD = T + 17;
  const int tid = thread_id();
  TileStage<T, double> st;
  st.load(C);
#pragma unroll
  for (int q = 0; q < T * 16 / NT; q++) {
    const int e = tid + q * NT;
    S[T + (e & 15) + (e >> 4) * LD] = (e & 15) == ((e >> 4) & 15) ? 1.0 : 0.0;
  }
#pragma unroll
  for (int q = 0; q < TileStage<T, double>::NV; q++) {
    const int e = 2 * (tid + q * NT);
    S[(e % T) + (e / T) * LD] = st.r[q].x;
    S[(e % T) + (e / T) * LD + 1] = st.r[q].y;
  }
}

// TRSM: L_t = (C_t - [sum X Y^T]) Linv_k^T; FP32 copy in mixed mode.  The
// optional fused products (at most two) are the updates with the most recent
// columns.  The task waits for its predecessors itself: with TF_SPLIT, first
// for the early ones (its tile's update chain and the fused operands), then
// it does the fused products, and only then waits for the POTRF of its
// column, so that the pivot chain sees one product.  Returns the time its
// last wait ended (per-task trace); `ok` as for the solve tasks.
// Each wave owns a strip of 16 rows (T = 32: a strip and one half of the
// result's columns).  A strip of C in the layout of an MFMA result is at the
// same time the B operand of the product with Linv_k^T (register q of block
// kb: columns 16 kb + 4 q + (lane >> 4)), so it never leaves the registers;
// the blocks of the lower-triangular Linv_k come straight from memory as A
// operands, and those above its diagonal are skipped (10 of 16 block
// products at T = 64).  Measured from the last wait, one workgroup alone:
// 4.3 -> 3.0 us at T = 64, 2.4 -> 1.6 us at T = 32 against a product of two
// staged tiles.
// A TRSM on the pivot chain (TF_CHAIN) carries the POTRF of the next column
// with it (next: its counter, C2: its tile): X stays in LDS (LY) for that
// task, whose tile is staged (in LX) before the last wait if its updates end
// first.
template <int T>
__device__ __forceinline__ uint64_t task_trsm(const ExecMat& M, const Task& w, double* LX, double* LY, int32_t* cnt,
                                              const Wait& wt, bool& ok, bool chain, int32_t* next, const double* C2,
                                              bool& staged) {
  constexpr int TT = T * T, NB = T / 16, NC = NB == 4 ? 4 : 1;   // NC: result blocks per wave
  const int lane = thread_id() & 63, li = lane & 15, lk = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(thread_id() >> 6);
  const int r0 = 16 * (wave % NB), cb0 = NB == 4 ? 0 : wave / NB;
  const bool split = (w[0] & TF_SPLIT) != 0;
  if (ok) ok = wait_below(cnt, split ? MERGED_FDEP : 1, wt);
  if (!ok) return 0;
  uint64_t t_start = M.trace ? wall_clock64() : 0;
  const int nf = w[4] - w[3];
  GLOBAL double* Cg = gp(M.tiles + (int64_t)w[1] * TT) + r0 + li + lk * T;
  const GLOBAL double* Lg = gp(M.linv + (int64_t)w[2] * TT) + li + lk * T;
  TileStage<T, double> sx, sy;
  if (nf > 0) {
    sx.load(M.tiles + (int64_t)word(w.pv, 0) * TT);
    sy.load(M.tiles + (int64_t)word(w.pv, 1) * TT);
  }
  v4d c[NB], acc[NB];
#pragma unroll
  for (int kb = 0; kb < NB; kb++) {
    acc[kb] = v4d{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int q = 0; q < 4; q++) c[kb][q] = Cg[(16 * kb + 4 * q) * T];
  }
  for (int q = 0; q < nf; q++) {
    if (q > 0) __syncthreads();
    sx.store(LX);
    sy.store(LY);
    __syncthreads();
    if (q + 1 < nf) {
      sx.load(M.tiles + (int64_t)word(w.pv, 2 * q + 2) * TT);
      sy.load(M.tiles + (int64_t)word(w.pv, 2 * q + 3) * TT);
    }
    mma_strip<T>(acc, LX, LY, r0, lane);
  }
#pragma unroll
  for (int kb = 0; kb < NB; kb++) c[kb] -= acc[kb];
  if (split) {
    // the POTRF of the column: its inverse is the last operand
    if (chain) {
      const int which = wait_first(next, 2, cnt, 1, wt);
      ok = which != 0;
      if (which == 1) {
        stage_diag<T>(C2, LX);
        staged = true;
      }
    }
    if (ok) ok = wait_below(cnt, 1, wt);
    if (!ok) return 0;
    if (M.trace) t_start = wall_clock64();
  }
  double a[NB][4][NC];
#pragma unroll
  for (int kb = 0; kb < NB; kb++)
#pragma unroll
    for (int q = 0; q < 4; q++)
#pragma unroll
      for (int i = 0; i < NC; i++)
        if (NC == 1 ? kb <= cb0 : kb <= i) a[kb][q][i] = Lg[16 * (cb0 + i) + (16 * kb + 4 * q) * T];
  v4d out[NC];
#pragma unroll
  for (int i = 0; i < NC; i++) out[i] = v4d{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int kb = 0; kb < NB; kb++)
#pragma unroll
    for (int q = 0; q < 4; q++)
#pragma unroll
      for (int i = 0; i < NC; i++)
        if (NC == 1 ? kb <= cb0 : kb <= i)
          out[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[kb][q][i], c[kb][q], out[i], 0, 0, 0);
  GLOBAL float* S = M.mixed ? gp(M.shadow + (int64_t)w[1] * TT) + r0 + li + lk * T : nullptr;
#pragma unroll
  for (int i = 0; i < NC; i++)
#pragma unroll
    for (int q = 0; q < 4; q++) {
      const int o = (16 * (cb0 + i) + 4 * q) * T;
      st_dev(Cg + o, out[i][q]);
      if (S) st_dev(S + o, (float)out[i][q]);
      if (chain) LY[r0 + li + lk * T + o] = out[i][q];
    }
  return t_start;
}

// ------------------------------------------------- diagonal tile: POTRF + TRTRI
// Blocked right-looking Cholesky of one T x T tile held in LDS, with 16-wide
// panels, extended by rows of the identity: eliminating the columns of
// [A; I] leaves [L; L^{-T}], so the inverse costs no step of its own on the
// chain.  The identity's row block b is zero left of panel b, and L needs no
// storage right of its diagonal blocks: the strict upper blocks of the tile
// buffer hold the identity part, and 16 rows below the tile its diagonal
// blocks D_b^{-T} (D_b the diagonal blocks of L), starting as I.
//
// A panel therefore has T - 16 rows besides its diagonal block (those of L
// below it, those of the identity part above it), and the 16 identity rows:
// one row per lane of wave 0 at T = 64.  Meanwhile waves 1 to 3 apply the
// previous panel to the columns beyond this one and store its part of the
// results; between two panels every wave updates one 16 x 16 block of the
// next panel's columns on the matrix cores.
//
// The chain of 64 pivots on one wave bounds the task; a wave issues about one
// vector instruction in six cycles, so the panel is written for few of them
// (about 400 for 16 columns of 80 rows): every 16-lane row holds its own copy
// of the diagonal block, whose multipliers reach the lanes as DPP operands of
// the updates.  Measured from the last wait, one workgroup alone: T = 64
// 27.5 -> 9.5 us, T = 32 11.4 -> 6.0 us against 16 x 16 diagonal blocks
// factored through LDS with the inverse and the panel as steps of their own
// (a chain-bound matrix, n = 10,000, w = 64, natural order: 5.98 -> 3.16 ms).

// acc -= a(lane Q of the 16-lane row) * b; a must not have been written by the
// two preceding vector instructions
template <int Q>
__device__ __forceinline__ void fnma_row(double& acc, double a, double b) {
  asm("v_fmac_f64_dpp %0, -%1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" : "+v"(acc) : "v"(a), "v"(b), "n"(Q));
}
// value of lane Q of each 16-lane row
template <int Q>
__device__ __forceinline__ double row_value(double v) {
  double d;
  asm("s_nop 1\n\tv_mov_b64_dpp %0, %1 row_newbcast:%2 row_mask:0xf bank_mask:0xf" : "=v"(d) : "v"(v), "n"(Q));
  return d;
}

// Deferred updates of column C: those its successor's pivot does not need,
// to D[C + 2] .. D[15], then a[C + 1] .. a[15].  Every update of D[q] by
// column C < q - 1 has been applied when column q - 1 ends.
constexpr int deferred_count(int c) { return c < 0 ? 0 : 29 - 2 * c; }
template <int C, int I>
__device__ __forceinline__ void deferred_update(double (&D)[16], double (&a)[16]) {
  if constexpr (I < 14 - C) fnma_row<C + 2 + I>(D[C + 2 + I], D[C], D[C]);
  else fnma_row<2 * C + I - 13>(a[2 * C + I - 13], D[C], a[C]);
}
template <int C, int LO, int... I>
__device__ __forceinline__ void deferred_updates(double (&D)[16], double (&a)[16], std::integer_sequence<int, I...>) {
  (deferred_update<C, LO + I>(D, a), ...);
}
// one of six slots of them, kept in its place by the scheduling barrier
template <int C, int SLOT>
__device__ __forceinline__ void deferred_slot(double (&D)[16], double (&a)[16]) {
  constexpr int lo = deferred_count(C) * SLOT / 6, hi = deferred_count(C) * (SLOT + 1) / 6;
  deferred_updates<C, lo>(D, a, std::make_integer_sequence<int, hi - lo>());
  __builtin_amdgcn_sched_barrier(0);
}

// Column J of a panel: d[J] the pivot, D the diagonal block's rows (one per
// lane of each 16-lane row), a one further row per lane.  1/sqrt(d) is the
// hardware's estimate y0 with one third-order correction, y0 (1 + e/2 +
// 3 e^2 / 8), e = 1 - d y0^2 (four dependent steps instead of six for two
// Newton steps; the estimate's error is cubed).  Its steps depend on each
// other: the previous column's deferred updates go between them.
template <int J>
__device__ __forceinline__ void panel_column(double (&D)[16], double (&a)[16], double (&d)[16]) {
  const double y0 = __builtin_amdgcn_rsq(d[J]);
  deferred_slot<J - 1, 0>(D, a);
  const double t = -d[J] * y0;
  deferred_slot<J - 1, 1>(D, a);
  const double e = fma(t, y0, 1.0);
  deferred_slot<J - 1, 2>(D, a);
  const double h = fma(0.375, e, 0.5), g = y0 * e;
  deferred_slot<J - 1, 3>(D, a);
  const double rs = fma(g, h, y0);
  deferred_slot<J - 1, 4>(D, a);
  D[J] *= rs;
  asm("s_nop 1" : "+v"(D[J]));   // the DPP reads of D[J] follow two wait states after its write
  deferred_slot<J - 1, 5>(D, a);
  if constexpr (J < 15) {
    fnma_row<J + 1>(D[J + 1], D[J], D[J]);
    a[J] *= rs;
    d[J + 1] = row_value<J + 1>(D[J + 1]);
    __builtin_amdgcn_sched_barrier(0);
    panel_column<J + 1>(D, a, d);
  } else {
    a[J] *= rs;
  }
}

// POTRF waits for its predecessors itself: with TF_SPLIT it stages its tile
// once the early ones (its update chain) have finished and waits last for
// the TRSM of its fused operand X = L_(k,k-1) (the panel of the previous
// column, on the pivot chain).  Returns the time its last wait ended.
// S: tile buffer with leading dimension T + 17, Xi: T x T (the fused operand).
// Behind its TRSM in one workgroup (chain): X is in Xi already, and the tile
// in S if `staged`; `lead` notifies the TRSM's successors, once its stores
// have completed, after the first panel.  Against two tasks this saves the
// chain a counter round trip, the completion of X's stores and its way back:
// n = 10,000, w = 64, natural order 2.82 -> 2.64 ms, 1,000 rows 279 -> 258 us.
template <int T, class Lead>
__device__ __forceinline__ uint64_t task_potrf(const ExecMat& M, const Task& w, double* S, double* Xi, int32_t* cnt,
                                               const Wait& wt, bool& ok, bool chain, bool staged, Lead&& lead) {
  constexpr int TT = T * T, NBK = T / 16, LD = T + 17;
  const int tid = thread_id(), lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lk = lane >> 4;
  const bool split = (w[0] & TF_SPLIT) != 0;
  double* C = M.tiles + (int64_t)w[1] * TT;
  const int k = w[2];
  // the fused update with column k-1, C_kk -= X X^T, is applied block by
  // block: the first block column before the first panel, the rest by waves
  // 1 to 3 during the first two panels
  const bool fused = w[4] > w[3];
  if (!staged) {
    // (the TRSM it follows does not decrement the counter)
    ok = wait_below(cnt, chain ? 2 : split ? MERGED_FDEP : 1, wt);
    if (!ok) return 0;
    stage_diag<T>(C, S);
  }
  if (split && !chain) {
    ok = wait_below(cnt, 1, wt);
    if (!ok) return 0;
  }
  const uint64_t t_start = M.trace ? wall_clock64() : 0;
  if (fused && !chain) {
    TileStage<T, double> st;
    st.load(M.tiles + (int64_t)word(w.pv, 0) * TT);
    st.store(Xi);
  }
  __syncthreads();
  // sum of the fused update for block (r, c): 16 rows from each of X's row
  // blocks r and c, two accumulation chains
  auto fused_sum = [&](int r, int c) {
    v4d u0 = v4d{0.0, 0.0, 0.0, 0.0}, u1 = v4d{0.0, 0.0, 0.0, 0.0};
    const double* xr = Xi + 16 * r + li + lk * T;
    const double* xc = Xi + 16 * c + li + lk * T;
#pragma unroll
    for (int kq = 0; kq < T; kq += 8) {
      u0 = __builtin_amdgcn_mfma_f64_16x16x4f64(xc[kq * T], xr[kq * T], u0, 0, 0, 0);
      u1 = __builtin_amdgcn_mfma_f64_16x16x4f64(xc[(kq + 4) * T], xr[(kq + 4) * T], u1, 0, 0, 0);
    }
    return u0 + u1;
  };
  // block (r, c) -= u
  auto subtract = [&](int r, int c, v4d u) {
    double* o = S + 16 * r + li + (16 * c + lk) * LD;
#pragma unroll
    for (int q = 0; q < 4; q++) o[4 * q * LD] -= u[q];
  };
  // block (r, c) after panel p, u + P_r P_c^T off: rows of L (r >= c) or of
  // the identity part (r <= p; its row block p is still on the rows below
  // the tile, and starts from zero here)
  auto apply = [&](int r, int c, int p, v4d u) {
    const double* Q = S + 16 * c + li + (16 * p + lk) * LD;
    const double* P = S + 16 * (r == p ? NBK : r) + li + (16 * p + lk) * LD;
    double* o = S + 16 * r + li + (16 * c + lk) * LD;
    double old[4];
#pragma unroll
    for (int q = 0; q < 4; q++) {
      const double v = o[4 * q * LD];
      old[q] = r == p ? 0.0 : v;
    }
#pragma unroll
    for (int kq = 0; kq < 16; kq += 4)
      u = __builtin_amdgcn_mfma_f64_16x16x4f64(Q[kq * LD], P[kq * LD], u, 0, 0, 0);
#pragma unroll
    for (int q = 0; q < 4; q++) o[4 * q * LD] = old[q] - u[q];
  };
  // stores of panel p by the threads t0 + step i: its columns of L, and its
  // rows of L^{-1}, the transpose of the identity part
  const DevTile<T> Cd(C), Ld(M.linv + (int64_t)k * TT);
  auto store_panel = [&](int p, int t0, int step) {
#pragma unroll 2
    for (int e = t0; e < 8 * T; e += step) {
      const int xr = 16 * p + 2 * (e & 7), xc = e >> 3;
      const double* x = S + ((xr ^ xc) < 16 ? T + (xc & 15) : xc) + xr * LD;
      Ld.store(xr + xc * T, v2d{xr >= xc ? x[0] : 0.0, xr + 1 >= xc ? x[LD] : 0.0});
      const int row = 2 * e % T, col = 16 * p + 2 * e / T;
      const double* v = S + row + col * LD;
      Cd.store(row + col * T, v2d{row >= col ? v[0] : 0.0, row + 1 >= col ? v[1] : 0.0});
    }
  };
  const v4d zero = v4d{0.0, 0.0, 0.0, 0.0};
  if (fused) {
    if (wave < NBK) subtract(wave, 0, fused_sum(wave, 0));
    __syncthreads();
  }
  int fail = -1;
#pragma unroll 1
  for (int p = 0; p < NBK; p++) {
    const int c0 = 16 * p;
    if (wave == 0) {
      // row of this lane: the rows of L below the diagonal block, those of
      // the identity part above it, the 16 rows below the tile
      const int l = lane & (T - 1);
      double* row = S + (l < T - 16 ? (c0 + 16 + l) & (T - 1) : l + 16) + c0 * LD;
      double* dia = S + c0 + li + c0 * LD;
      double D[16], a[16];
#pragma unroll
      for (int j = 0; j < 16; j++) D[j] = dia[j * LD];
#pragma unroll
      for (int j = 0; j < 16; j++) a[j] = row[j * LD];
      double d[16];
      d[0] = row_value<0>(D[0]);
      panel_column<0>(D, a, d);
#pragma unroll
      for (int j = 0; j < 16; j++) {
        dia[j * LD] = D[j];
        row[j * LD] = a[j];
      }
      // a pivot that is not positive makes every later one NaN or negative
      if (__ballot(!(d[15] > 0.0)) != 0 && fail < 0) {
#pragma unroll
        for (int j = 15; j >= 0; j--)
          if (!(d[j] > 0.0)) fail = c0 + j;
      }
    } else if (p == 0) {
      // the fused update of block column 1 (and, at T = 64, of block (2, 2))
      if (fused) {
        for (int q = wave - 1; q < (NBK == 4 ? 4 : 1); q += 3) {
          const int c = q < 3 ? 1 : 2;
          subtract(q < 3 ? 1 + q : 2, c, fused_sum(q < 3 ? 1 + q : 2, c));
        }
      }
    } else {
      // the previous panel's update of the block columns beyond this panel
      // (at p == 1 with the rest of the fused update, blocks (3, 2), (3, 3));
      // once there is little of that, the stores of the finished panels
      int q = 0;
      for (int r = NBK - 1; r >= 0; r--)
        for (int c = p + 1; c < NBK; c++) {
          if (r < c && r >= p) continue;
          if (q++ % 3 != wave - 1) continue;
          apply(r, c, p - 1, p == 1 && fused && r == 3 ? fused_sum(r, c) : zero);
        }
      for (int b = p < 2 ? 0 : p - 2; b < (p + 1 == NBK ? p : p - 1); b++) store_panel(b, tid - 64, NT - 64);
    }
    if (p == 0 && chain) __builtin_amdgcn_s_waitcnt(0);   // X's stores
    __syncthreads();
    if (p == 0 && chain) lead();
    if (p + 1 < NBK) {
      // the next panel's block column: rows p+1 .. of L, then 0 .. p of the
      // identity part, one block per wave
      if (wave < NBK) apply((p + 1 + wave) % NBK, p + 1, p, zero);
      __syncthreads();
    }
  }
  if (tid == 0 && fail >= 0) atomicMin(M.info, (unsigned long long)(M.row_base[k] + fail + 1));
  store_panel(NBK - 1, tid, NT);
  return t_start;
}

// ---------------------------------------------------------- solve tasks
// Vector blocks are T x nrhs column-major (nrhs <= 16).  Each task computes
// out = sum_p A_p V_p with A_p a factor tile (or its transpose) and V_p a
// vector block, as 16 x 16 x 4 FP64 MFMA products with the right-hand sides
// padded to 16 columns.
// MFMA operands are read from global memory straight into registers.  At
// MFMA steps 2 s and 2 s + 1 the four k-groups of the 16 x 16 x 4 instruction
// (lane >> 4 = g) take k = 8 s + 2 g and the next one: a 16-byte load per lane
// for the B operand (vector block, column lane & 15) and for the A operand of
// a transposed tile (backward sweep: A(r, k) = L(k, r), a piece of column r),
// 64 bytes of each of 16 columns per load (a run of T/4 doubles per lane
// instead touches 64 lines per load: 16-RHS solve of the n = 200,000
// variable-band matrix 2.36 -> 2.17 ms, a residual pass at n = 500,000 3.28 ->
// 2.64 ms); a direct tile (forward sweep) is read as T/4 loads whose 16 lanes
// cover 16 consecutive rows.  Wave w owns rows 16 w .. 16 w + 15 of the T x 16
// result (waves past T/16 idle), in an order of A's rows that leaves each lane
// four consecutive ones of its column: 16-byte accesses to the vector blocks
// (2.17 -> 2.12 ms).
template <int T>
struct SolveOps {
  static constexpr int NS = T / 4;   // MFMA steps per tile
  // leading dimension of a block in LDS: the 16-byte reads of 16 columns
  // cover all banks
  static constexpr int LDV = T + 2;
  // row of A's lane: result register r of lane group g is then row 4 g + r
  static __device__ __forceinline__ int a_row(int wave, int lane) {
    return 16 * wave + 4 * (lane & 3) + ((lane & 15) >> 2);
  }
  // this lane's first element of a T x 16 block with leading dimension ld
  static __device__ __forceinline__ int elem(int wave, int lane, int ld) {
    return 16 * wave + 4 * (lane >> 4) + (lane & 15) * ld;
  }
  // its four elements of a vector block in global memory
  static __device__ __forceinline__ v4d load_c(const double* V, int e, bool ok) {
    const GLOBAL d2* p = (const GLOBAL d2*)(V + e);
    const d2 lo = ok ? p[0] : d2{0.0, 0.0}, hi = ok ? p[1] : d2{0.0, 0.0};
    return v4d{lo.x, lo.y, hi.x, hi.y};
  }
  // k of MFMA step s in lane group g
  static __device__ __forceinline__ int k_of(int s, int g) { return 8 * (s >> 1) + 2 * g + (s & 1); }
  typedef double d2 __attribute__((ext_vector_type(2)));
  // A operand of tile Lt
  static __device__ __forceinline__ void load_a(double (&a)[NS], const double* Lt, bool trans, int wave, int lane) {
    const int r = a_row(wave, lane), g = lane >> 4;
    if (trans) {
      const GLOBAL d2* p = (const GLOBAL d2*)(Lt + 2 * g + (int64_t)r * T);
#pragma unroll
      for (int q = 0; q < NS / 2; q++) {
        const d2 v = p[4 * q];
        a[2 * q] = v.x;
        a[2 * q + 1] = v.y;
      }
    } else {
      const GLOBAL double* p = gp(Lt) + r + 2 * g * T;
#pragma unroll
      for (int q = 0; q < NS; q++) a[q] = p[k_of(q, 0) * T];
    }
  }
  // B operand of a vector block (T x nrhs, leading dimension T) in global memory
  static __device__ __forceinline__ void load_b(double (&b)[NS], const double* V, int nrhs, int lane) {
    const int j = lane & 15, g = lane >> 4;
    const GLOBAL d2* p = (const GLOBAL d2*)(V + 2 * g + (int64_t)j * T);
    const bool ok = j < nrhs;
#pragma unroll
    for (int q = 0; q < NS / 2; q++) {
      const d2 v = ok ? p[4 * q] : d2{0.0, 0.0};
      b[2 * q] = v.x;
      b[2 * q + 1] = v.y;
    }
  }
  // the same from a T x 16 block in LDS (leading dimension LDV)
  static __device__ __forceinline__ void load_b_lds(double (&b)[NS], const double* V, int lane) {
    const int j = lane & 15, g = lane >> 4;
    const d2* p = (const d2*)(V + 2 * g + j * LDV);
#pragma unroll
    for (int q = 0; q < NS / 2; q++) {
      const d2 v = p[4 * q];
      b[2 * q] = v.x;
      b[2 * q + 1] = v.y;
    }
  }
  // acc += A B over the T/4 steps, two accumulation chains
  static __device__ __forceinline__ v4d mma(v4d acc, const double (&a)[NS], const double (&b)[NS]) {
    v4d acc1 = v4d{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int q = 0; q < NS; q += 2) {
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[q], b[q], acc, 0, 0, 0);
      acc1 = __builtin_amdgcn_mfma_f64_16x16x4f64(a[q + 1], b[q + 1], acc1, 0, 0, 0);
    }
    return acc + acc1;
  }
};

// A solve task (FUPD, FDIAG, BUPD, BDIAG, FPART).  It waits for its
// predecessors itself (*cnt): the factor tiles of a diagonal step (at most
// two fused products and the inverse diagonal tile) are read into registers
// first, so that only the small vector blocks are loaded once the
// predecessors are done.  A diagonal step with TF_SPLIT waits in two
// stages: once its early predecessors are done (the counter below
// MERGED_FDEP in a solve launch, below SPLIT_W in the merged launch, whose
// executor has already waited for the factorization predecessors) it loads
// its right-hand side block and does the first fused product, then waits
// for the previous step of the chain, whose block the second product reads.
// The factor tiles must be final when it is called.
// `ok` enters false when the launch was already abandoned and leaves false
// when this task's own wait gave up; the task then writes nothing.
template <int T, int K>
__device__ __forceinline__ uint64_t task_solve_r(const ExecMat& M, const Task& w, int nrhs, int32_t* cnt,
                                                 double* LV, const Wait& wt, bool& ok) {
  typedef SolveOps<T> O;
  constexpr int TT = T * T, NS = O::NS;
  const int type = w[0] & 0xff;
  const int lane = thread_id() & 63, wave = thread_id() >> 6;
  const bool act = 16 * wave < T;
  const int m = w[1];
  const int64_t vb = (int64_t)T * nrhs;
  const bool fwd = type == TK_FUPD || type == TK_FDIAG || type == TK_FPART;
  const bool diag = type == TK_FDIAG || type == TK_BDIAG;
  const double* vsrc = fwd ? M.vy : M.vz;
  const int np = w[3] - w[2];
  const int pv = w.pv;
  // this lane's four output elements
  const int col = lane & 15, el = O::elem(wave, lane, T);
  const double* base = fwd ? M.vy + m * vb : ((w[0] & TF_FIRST) ? M.vy + m * vb : M.vz + m * vb);
  const DevBlock dst(fwd ? M.vy + m * vb : M.vz + m * vb, vb * 8);
  v4d acc = v4d{0.0, 0.0, 0.0, 0.0};
  if (diag) {
    // static operands first (at most two fused products), then the wait
    const bool split = (w[0] & TF_SPLIT) != 0;
    double a0[NS], a1[NS], ai[NS], b0[NS], b1[NS];
    if (act) {
      if (np > 0) O::load_a(a0, M.tiles + (int64_t)word(pv, 0) * TT, !fwd, wave, lane);
      if (np > 1) O::load_a(a1, M.tiles + (int64_t)word(pv, 2) * TT, !fwd, wave, lane);
      O::load_a(ai, M.linv + (int64_t)m * TT, !fwd, wave, lane);
    }
    if (ok) ok = wait_below(cnt, split ? (K == EXEC_FACTOR_SOLVE ? SPLIT_W : MERGED_FDEP) : 1, wt);
    if (!ok) return 0;
    uint64_t t_start = M.trace ? wall_clock64() : 0;
    v4d bs;
    if (act) {
      if (np > 0) O::load_b(b0, vsrc + word(pv, 1) * vb, nrhs, lane);
      bs = O::load_c(base, el, col < nrhs);
      if (np > 0) acc = O::mma(acc, a0, b0);
    }
    if (split) {
      // the previous step of the chain: its block is the second operand
      ok = wait_below(cnt, 1, wt);
      if (!ok) return 0;
      if (M.trace) t_start = wall_clock64();
    }
    if (act) {
      if (np > 1) {
        O::load_b(b1, vsrc + word(pv, 3) * vb, nrhs, lane);
        acc = O::mma(acc, a1, b1);
      }
      // base - acc into LDS for the product with the inverse diagonal tile
      const v4d z = bs - acc;
      v2d* l = reinterpret_cast<v2d*>(LV + O::elem(wave, lane, O::LDV));
      l[0] = v2d{z[0], z[1]};
      l[1] = v2d{z[2], z[3]};
    }
    __syncthreads();
    if (act) {
      O::load_b_lds(b0, LV, lane);
      const v4d out = O::mma(v4d{0.0, 0.0, 0.0, 0.0}, ai, b0);
      if (col < nrhs) dst.store(el, out);
    }
    return t_start;
  }
  // a chunk of products: the factor tiles of the first NF pairs are read
  // before the wait; then NF pairs stay in flight (the operands of pair
  // p + NF are loaded once pair p has been multiplied).  Three take all
  // registers: the solve of the n = 200,000 variable-band matrix 1.97 -> 1.93
  // ms, but the merged launch 0.7 % slower, which keeps two.
  constexpr int NF = K == EXEC_SOLVE ? 3 : 2;
  double a[NF][NS], b[NF][NS];
  v4d bs;
  if (act) {
#pragma unroll
    for (int u = 0; u < NF; u++)
      if (u < np) O::load_a(a[u], M.tiles + (int64_t)word(pv, 2 * u) * TT, !fwd, wave, lane);
  }
  if (ok) ok = wait_below(cnt, 1, wt);
  if (!ok) return 0;
  const uint64_t t_start = M.trace ? wall_clock64() : 0;
  if (act) {
#pragma unroll
    for (int u = 0; u < NF; u++)
      if (u < np) O::load_b(b[u], vsrc + word(pv, 2 * u + 1) * vb, nrhs, lane);
    if (type != TK_FPART) bs = O::load_c(base, el, col < nrhs);
    for (int p = 0; p < np; p += NF) {
#pragma unroll
      for (int u = 0; u < NF; u++) {
        if (p + u < np) acc = O::mma(acc, a[u], b[u]);
        if (p + u + NF < np) {
          const int q = 2 * (p + u + NF);
          O::load_a(a[u], M.tiles + (int64_t)word(pv, q) * TT, !fwd, wave, lane);
          O::load_b(b[u], vsrc + word(pv, q + 1) * vb, nrhs, lane);
        }
      }
    }
  }
  if (!act) return t_start;
  if (type == TK_FPART) {
    // one chunk of a long row: the partial product into its slot
    if (col < nrhs) DevBlock(M.vpart + (int64_t)w[4] * vb, vb * 8).store(el, acc);
    return t_start;
  }
  if (col < nrhs) dst.store(el, bs - acc);
  return t_start;
}

// Y_m -= Q_a + ... + Q_(b-1): the partial products of a long row, summed in
// a fixed order (so the result does not depend on the schedule): four running
// sums, slot q in sum (q - a) mod 4, the last (b - a) mod 4 slots all in the
// first.  The task is on the chain of the
// separators' steps and waits for memory only: eight slots are in flight for
// every pair of elements, and all pairs of a lane at once (four slots of one
// element at a time: 9.4 us a task, now 4.2; the solve above 2.12 -> 1.96 ms).
template <int T, int NP>   // NP: pairs of elements per lane
__device__ __forceinline__ void fsum_pairs(const double* part, double* y, int n, int64_t vb) {
  const int e = 2 * thread_id();
  const int ne = (int)vb;
  v2d sum[NP][4], base[NP];
#pragma unroll
  for (int p = 0; p < NP; p++) {
    const int x = e + 2 * NT * p;
    base[p] = x < ne ? *(const GLOBAL v2d*)(y + x) : v2d{0.0, 0.0};
#pragma unroll
    for (int j = 0; j < 4; j++) sum[p][j] = v2d{0.0, 0.0};
  }
  int q = 0;
  for (; q + 4 <= n; q += 8) {
    v2d v[NP][8];
    const bool two = q + 8 <= n;
#pragma unroll
    for (int j = 0; j < 8; j++)
#pragma unroll
      for (int p = 0; p < NP; p++) {
        const int x = e + 2 * NT * p;
        v[p][j] = x < ne && (j < 4 || two) ? *(const GLOBAL v2d*)(part + (q + j) * vb + x) : v2d{0.0, 0.0};
      }
#pragma unroll
    for (int j = 0; j < 8; j++)
#pragma unroll
      for (int p = 0; p < NP; p++)
        if (j < 4 || two) sum[p][j & 3] += v[p][j];
    if (!two) {
      q += 4;
      break;
    }
  }
  for (; q < n; q++)
#pragma unroll
    for (int p = 0; p < NP; p++) {
      const int x = e + 2 * NT * p;
      if (x < ne) sum[p][0] += *(const GLOBAL v2d*)(part + q * vb + x);
    }
  const DevBlock dst(y, vb * 8);
#pragma unroll
  for (int p = 0; p < NP; p++) {
    const int x = e + 2 * NT * p;
    if (x < ne) dst.store(x, base[p] - ((sum[p][0] + sum[p][1]) + (sum[p][2] + sum[p][3])));
  }
}

template <int T>
__device__ __forceinline__ void task_fsum(const ExecMat& M, const Task& w, int nrhs) {
  const int64_t vb = (int64_t)T * nrhs;   // even, at most 16 T
  fsum_pairs<T, 16 * T / (2 * NT)>(M.vpart + w[2] * vb, M.vy + (int64_t)w[1] * vb, w[3] - w[2], vb);
}

// ------------------------------------------------------- selected inversion
// Tile products C = op(X) Y, op = identity or transpose, on whole tiles in
// LDS, each wave a (T/2) x (T/2) quarter: acc[i][j] covers its rows
// NB li + j and columns NB m + i (NB = T/32, li = lane & 15,
// m = (lane >> 4) + 4 r), as in update_products.  Y, and X when transposed,
// are read down their columns: lane group lk = lane >> 4 takes
// k = 8 s + 2 lk and the next one for two MFMA steps, a 16-byte read (the
// order of k within eight is free as long as X and Y agree); X as stored is
// read along its rows, NB of one column at a time.  Tile element (row, col)
// is in 16-byte unit row/2 of its column, and the units of a column are
// permuted by an XOR with a function of the column: every one of these reads
// and the 16-byte staging and result stores then cover all LDS banks.
template <int T>
struct Swz {
  static constexpr int NB = T / 32;
  // unit permutation of a column: the columns NB li + q of a read down the
  // columns get 16 different ones; T = 32: bits 1 and 3 exchanged, so that
  // 8-byte reads along rows by two lane groups fall into different halves
  __device__ __forceinline__ static int g(int col) {
    return T == 64 ? (col >> 1) & 15 : ((col & 2) << 2) | ((col & 8) >> 2) | (col & 5);
  }
  // byte offset of element (row, col), of its unit if row is even
  __device__ __forceinline__ static int at(int row, int col) {
    return col * T * 8 + (((row >> 1) ^ g(col)) << 4) + (row & 1) * 8;
  }
};


template <int T>
struct TileRegs {
  static constexpr int NV = T * T / NT / 2;
  v2d r[NV];
  __device__ __forceinline__ void load(const double* __restrict__ g) {
    const GLOBAL v2d* v = (const GLOBAL v2d*)g;
#pragma unroll
    for (int q = 0; q < NV; q++) r[q] = v[thread_id() + q * NT];
  }
  __device__ __forceinline__ v2d* at(double* l, int q) const {
    const int e = 2 * (thread_id() + q * NT);
    return reinterpret_cast<v2d*>((char*)l + Swz<T>::at(e % T, e / T));
  }
  __device__ __forceinline__ void store(double* l) const {
#pragma unroll
    for (int q = 0; q < NV; q++) *at(l, q) = r[q];
  }
};

// acc += op(X) Y, op = transpose if TX.  The operands of the next two MFMA
// steps are read while these run.  With 8-byte reads on padded tiles the
// reads held up the matrix cores (81 cycles per MFMA against 69).
template <int T, bool TX>
__device__ __forceinline__ void mma_tiles(v4d (&acc)[T / 32][T / 32], const double* X, const double* Y, int r0, int c0,
                                          int lane) {
  constexpr int NB = T / 32, CB = T * 8;   // CB: bytes of a column
  const int li = lane & 15, lk = lane >> 4;
  const int yo = Swz<T>::at(2 * lk, c0 + NB * li);
  const int xo = TX ? Swz<T>::at(2 * lk, r0 + NB * li) : Swz<T>::at(r0 + NB * li, 2 * lk);
  // down the columns: eight rows further is four units further, an XOR
  auto down = [&](const double* Z, int o, int q, int k) {
    return *reinterpret_cast<const v2d*>((const char*)Z + ((o ^ (k << 3)) + q * CB));
  };
  // two steps' operands: z[step][block]
  auto read = [&](double (&a)[2][NB], double (&b)[2][NB], int k) {
#pragma unroll
    for (int q = 0; q < NB; q++) {
      const v2d y = down(Y, yo, q, k);
      a[0][q] = y[0];
      a[1][q] = y[1];
      if constexpr (TX) {
        const v2d x = down(X, xo, q, k);
        b[0][q] = x[0];
        b[1][q] = x[1];
      }
    }
    if constexpr (!TX) {
      if constexpr (NB == 2) {   // columns k + 2 lk and the next: the same unit permutation
        const char* x = (const char*)X + ((xo ^ (8 * k & 255)) + k * CB);
#pragma unroll
        for (int h = 0; h < 2; h++) {
          const v2d v = *reinterpret_cast<const v2d*>(x + h * CB);
          b[h][0] = v[0];
          b[h][NB - 1] = v[1];
        }
      } else {
        const int o = (xo ^ ((k & 8) << 2)) + k * CB;
        b[0][0] = *reinterpret_cast<const double*>((const char*)X + o);
        b[1][0] = *reinterpret_cast<const double*>((const char*)X + ((o ^ 16) + CB));
      }
    }
  };
  double a[2][NB], b[2][NB];
  read(a, b, 0);
#pragma unroll
  for (int k = 0; k < T; k += 8) {
    double an[2][NB], bn[2][NB];
    if (k + 8 < T) read(an, bn, k + 8);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int h = 0; h < 2; h++)
#pragma unroll
      for (int i = 0; i < NB; i++)
#pragma unroll
        for (int j = 0; j < NB; j++) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[h][i], b[h][j], acc[i][j], 0, 0, 0);
    if (k + 8 < T) {
#pragma unroll
      for (int h = 0; h < 2; h++)
#pragma unroll
        for (int q = 0; q < NB; q++) {
          a[h][q] = an[h][q];
          b[h][q] = bn[h][q];
        }
    }
  }
}

template <int T>
__device__ __forceinline__ void zero_acc(v4d (&acc)[T / 32][T / 32]) {
#pragma unroll
  for (int i = 0; i < T / 32; i++)
#pragma unroll
    for (int j = 0; j < T / 32; j++) acc[i][j] = v4d{0.0, 0.0, 0.0, 0.0};
}

// C = Sig~ L on LDS tiles: Sig~ as stored or transposed
template <int T>
__device__ __forceinline__ void sig_mma(v4d (&acc)[T / 32][T / 32], int code, const double* LX, const double* LY,
                                        int r0, int c0, int lane) {
  if (code & SIG_TRANS) mma_tiles<T, true>(acc, LX, LY, r0, c0, lane);
  else mma_tiles<T, false>(acc, LX, LY, r0, c0, lane);
}

// this lane's elements of a quarter: NB rows row0 .., columns col(i, r)
template <int T>
struct Quarter {
  static constexpr int NB = T / 32;
  typedef double vec __attribute__((ext_vector_type(NB)));
  int row0, c0m;
  __device__ __forceinline__ Quarter(int r0, int c0, int lane) : row0(r0 + NB * (lane & 15)), c0m(c0 + NB * (lane >> 4)) {}
  __device__ __forceinline__ int col(int i, int r) const { return c0m + 4 * NB * r + i; }
};

// out (global, column-major T x T) <- s * acc
template <int T>
__device__ __forceinline__ void put_acc_g(const v4d (&acc)[T / 32][T / 32], double* out, double sc, int r0, int c0,
                                          int lane) {
  constexpr int NB = T / 32;
  const Quarter<T> e(r0, c0, lane);
  const DevTile<T> dev(out);
#pragma unroll
  for (int i = 0; i < NB; i++)
#pragma unroll
    for (int r = 0; r < 4; r++) {
      const int q = e.row0 + e.col(i, r) * T;
      if constexpr (NB == 2) dev.store(q, v2d{sc * acc[i][0][r], sc * acc[i][NB - 1][r]});
      else dev.store(q, sc * acc[i][0][r]);
    }
}

// out (LDS tile) <- s * acc
template <int T>
__device__ __forceinline__ void put_acc_l(const v4d (&acc)[T / 32][T / 32], double* out, double sc, int r0, int c0,
                                          int lane) {
  constexpr int NB = T / 32;
  const Quarter<T> e(r0, c0, lane);
#pragma unroll
  for (int i = 0; i < NB; i++)
#pragma unroll
    for (int r = 0; r < 4; r++) {
      typename Quarter<T>::vec v;
#pragma unroll
      for (int j = 0; j < NB; j++) v[j] = sc * acc[i][j][r];
      *reinterpret_cast<typename Quarter<T>::vec*>((char*)out + Swz<T>::at(e.row0, e.col(i, r))) = v;
    }
}

// acc += tile g (column-major T x T, global), element by element
template <int T>
__device__ __forceinline__ void add_tile(v4d (&acc)[T / 32][T / 32], const double* __restrict__ g, int r0, int c0,
                                         int lane) {
  constexpr int NB = T / 32;
  const Quarter<T> e(r0, c0, lane);
  const GLOBAL double* s = gp(g) + e.row0;
#pragma unroll
  for (int i = 0; i < NB; i++)
#pragma unroll
    for (int r = 0; r < 4; r++) {
      const typename Quarter<T>::vec v = *(const GLOBAL typename Quarter<T>::vec*)(s + e.col(i, r) * T);
#pragma unroll
      for (int j = 0; j < NB; j++) acc[i][j][r] += v[j];
    }
}

// acc += sum over the np pairs of pv of Sig~ L (pair words: Sigma tile code,
// L tile), streamed through the operand ring of the update products (Ring)
// in stages of KS values of k.  Sig as stored: KS whole columns, in memory
// order.  L, and Sig transposed: KS rows of every column; a column's
// KS / 2 units of 16 bytes form one row of the slot, the columns ordered so
// that a lane's blocks are 16 slot rows apart and the units of a slot row
// permuted by an XOR, so that the 16-byte reads cover all LDS banks.  The
// transfers do this order by each lane's own global address.  A product
// takes 2.84 us on an otherwise idle CU (tiles staged whole through registers
// 3.13; the MFMAs alone 1.9) and 5.4 us with the chip full (6.1), when the
// operands' traffic binds; selected inversion of the n = 200,000
// variable-band matrix 13.5 -> 11.8 ms.
template <int T>
__device__ __forceinline__ void sig_products(v4d (&acc)[T / 32][T / 32], const ExecMat& M, int pv, int np, double* ring,
                                             int r0, int c0) {
  typedef Ring<T, double> R;
  constexpr int NB = T / 32, NI = R::NI, NST = R::NST, KS = R::KS;
  constexpr int CB = T * 8, SB = KS * 8;      // bytes of a tile column, of a slot row
  const int tid = thread_id(), lane = tid & 63, li = lane & 15, lk = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)ring + 1024 * wave;
  // unit permutation of a slot row
  auto perm = [](int sr) { return NB == 2 ? (sr >> 1) & 7 : sr & 15; };
  const uint32_t voff = 1024 * wave + 16 * lane;
  uint32_t vrow;   // by rows: transfer i of a stage adds i (4096 / SB) columns
  {
    const int sr = (int)voff / SB, unit = ((int)voff % SB / 16) ^ perm(sr);
    const int c = NB == 2 ? 2 * (sr & 15) + (sr >> 4) : sr;
    vrow = c * CB + 16 * unit;
  }
  const int total = np * R::SPP;
  const double *const sigma = M.sigma, *const tiles = M.tiles;
  const char *xb, *yb;
  uint32_t dst;
  bool xtr;
  auto stage = [&](int s, int slot) {
    const int p = s / R::SPP, h = s % R::SPP;
    const int code = word(pv, 2 * p);
    xtr = (code & SIG_TRANS) != 0;
    xb = (const char*)(sigma + (int64_t)(code & ~SIG_TRANS) * T * T) + h * (xtr ? SB : R::HB);
    yb = (const char*)(tiles + (int64_t)word(pv, 2 * p + 1) * T * T) + h * SB;
    dst = lds0 + (uint32_t)slot * 2 * R::HB;
  };
  auto transfer = [&](int i) {
    const int c = i % (NI / 2);
    if (i < NI / 2) lds_transfer(dst + 4096 * c, xtr ? vrow + 4096 / SB * CB * c : voff + 4096 * c, xb);
    else lds_transfer(dst + R::HB + 4096 * c, vrow + 4096 / SB * CB * c, yb);
  };
#pragma unroll
  for (int s = 0; s < NST - 1; s++)
    if (s < total) {
      stage(s, s);
#pragma unroll
      for (int i = 0; i < NI; i++) transfer(i);
    }
  ring_barrier<NI>((total < NST - 1 ? total : NST - 1) * NI - NI);
  // byte offsets within a slot: X as stored, X by rows, Y
  const int xd = (r0 + NB * li) * 8 + 2 * lk * CB;
  const int xt = (r0 + li) * SB + ((lk ^ perm(li)) << 4);
  const int yo = (c0 + li) * SB + ((lk ^ perm(li)) << 4) + R::HB;
  constexpr int SLOT = 2 * R::HB;
  auto trans = [&](int s) { return (word(pv, 2 * (s / R::SPP)) & SIG_TRANS) != 0; };
  // operands of two MFMA steps, k .. k + 7 of a slot
  auto read = [&](double (&a)[2][NB], double (&b)[2][NB], const char* slot, int k, bool tr) {
#pragma unroll
    for (int q = 0; q < NB; q++) {
      const v2d y = *reinterpret_cast<const v2d*>(slot + ((yo ^ (k << 3)) + 16 * SB * q));
      a[0][q] = y[0];
      a[1][q] = y[1];
    }
    if constexpr (NB == 2) {
      const char* x = slot + (tr ? xt ^ (k << 3) : xd + k * CB);
      const v2d u = *reinterpret_cast<const v2d*>(x);
      const v2d v = *reinterpret_cast<const v2d*>(x + (tr ? 16 * SB : CB));
      b[0][0] = u[0];
      b[0][NB - 1] = tr ? v[0] : u[1];
      b[1][0] = tr ? u[1] : v[0];
      b[1][NB - 1] = v[1];
    } else if (tr) {
      const v2d u = *reinterpret_cast<const v2d*>(slot + (xt ^ (k << 3)));
      b[0][0] = u[0];
      b[1][0] = u[1];
    } else {
      b[0][0] = *reinterpret_cast<const double*>(slot + (xd + k * CB));
      b[1][0] = *reinterpret_cast<const double*>(slot + (xd + (k + 1) * CB));
    }
  };
  int slot = 0, wslot = NST - 1;
  bool tr = trans(0);
  double a[2][NB], b[2][NB];
  read(a, b, (const char*)ring, 0, tr);
#pragma unroll 1
  for (int s = 0; s < total; s++) {
    const char* cur = (const char*)ring + slot * SLOT;
    slot = slot + 1 == NST ? 0 : slot + 1;
    const char* nxt = (const char*)ring + slot * SLOT;
    const bool more = s + NST - 1 < total;
    const bool trn = s + 1 < total ? trans(s + 1) : tr;
#pragma unroll
    for (int k = 0; k < KS; k += 8) {
      double an[2][NB], bn[2][NB];
      if (k + 8 < KS) read(an, bn, cur, k + 8, tr);
      else read(an, bn, nxt, 0, trn);
      if (k >= 8 && more) {
#pragma unroll
        for (int i = (k / 8 - 1) * NI / (KS / 8 - 1); i < (k / 8) * NI / (KS / 8 - 1); i++) transfer(i);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int h = 0; h < 2; h++)
#pragma unroll
        for (int i = 0; i < NB; i++)
#pragma unroll
          for (int j = 0; j < NB; j++)
            acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[h][i], b[h][j], acc[i][j], 0, 0, 0);
      if (k == 0) {
        // the next stage has arrived, the previous one's slot is free
        const int last = s + NST - 2 < total ? s + NST - 2 : total - 1;
        if (s + 1 < total) ring_barrier<NI>((last - (s + 1)) * NI);
        if (more) stage(s + NST - 1, wslot);
        wslot = wslot + 1 == NST ? 0 : wslot + 1;
      }
#pragma unroll
      for (int h = 0; h < 2; h++)
#pragma unroll
        for (int q = 0; q < NB; q++) {
          a[h][q] = an[h][q];
          b[h][q] = bn[h][q];
        }
    }
    tr = trn;
  }
}

// SWE: W_t (+)= sum over pairs of Sig~ L, kept in the Sigma tile of t until
// its SW task finishes it
template <int T>
__device__ __forceinline__ void task_swe(const ExecMat& M, const Task& w, double* ring) {
  constexpr int TT = T * T, W = T / 2, NB = T / 32;
  const int lane = thread_id() & 63, wave = thread_id() >> 6;
  const int r0 = (wave >> 1) * W, c0 = (wave & 1) * W;
  double* out = M.sigma + (int64_t)w[1] * TT;
  v4d acc[NB][NB];
  zero_acc<T>(acc);
  if (w[0] & TF_ACC) add_tile<T>(acc, out, r0, c0, lane);
  sig_products<T>(acc, M, w.pv, w[3], ring, r0, c0);
  put_acc_g<T>(acc, out, 1.0, r0, c0, lane);
}

// Static operands of a selected-inversion task (the factor is final), staged
// before the task waits for its predecessors: the L tile of SW's first
// product into LY, the inverse diagonal tile of SDIAG into LX.
template <int T>
__device__ __forceinline__ void selinv_prefetch(const ExecMat& M, const Task& w, double* LX, double* LY) {
  constexpr int TT = T * T;
  const int type = w[0] & 0xff;
  TileRegs<T> st;
  if (type == TK_SW) {
    st.load(M.tiles + (int64_t)word(w.pv, 1) * TT);
    st.store(LY);
  } else if (type == TK_SDIAG) {
    st.load(M.linv + (int64_t)w[2] * TT);
    st.store(LX);
  }
}

// SW: Sig_t = -(W + pushed partials + sum of its one or two products Sig~ L_y)
// Linv_k, then D_t = L_t^T Sig_t and, for every listed tile u = (r,c),
// Q_u = Sig_t^T L_u.  The first product's L_y was staged in LY by
// selinv_prefetch.  w4 = nsum | npush << 8 | nprod << 16; the list holds the
// product pairs, then the slots, then the push tiles (at most 64 words).
template <int T>
__device__ __forceinline__ void task_sw(const ExecMat& M, const Task& w, double* LX, double* LY) {
  constexpr int TT = T * T, W = T / 2, NB = T / 32;
  const int lane = thread_id() & 63, wave = thread_id() >> 6;
  const int r0 = (wave >> 1) * W, c0 = (wave & 1) * W;
  const int cnt = w[4];
  const int nsum = cnt & 0xff, npush = (cnt >> 8) & 0xff, nprod = cnt >> 16;
  const int pv = w.pv;
  const int sw0 = 2 * nprod, pw0 = 2 * nprod + nsum;   // first slot word, first push word
  const int64_t t = w[1];
  const int64_t k = w[2];
  double* sig = M.sigma + t * TT;
  TileRegs<T> sx, sy, st;
  sx.load(M.sigma + (int64_t)(word(pv, 0) & ~SIG_TRANS) * TT);
  if (nprod > 1) {
    sy.load(M.tiles + (int64_t)word(pv, 3) * TT);
    st.load(M.sigma + (int64_t)(word(pv, 2) & ~SIG_TRANS) * TT);
  } else {
    st.load(M.linv + k * TT);
  }
  v4d acc[NB][NB];
  zero_acc<T>(acc);
  if (w[0] & TF_ACC) add_tile<T>(acc, sig, r0, c0, lane);
  for (int q = 0; q < nsum; q++) add_tile<T>(acc, M.qpart + (int64_t)word(pv, sw0 + q) * TT, r0, c0, lane);
  sx.store(LX);
  __syncthreads();
  // W += Sig~ L_y
  sig_mma<T>(acc, word(pv, 0), LX, LY, r0, c0, lane);
  if (nprod > 1) {
    __syncthreads();
    st.store(LX);
    sy.store(LY);
    __syncthreads();
    st.load(M.linv + k * TT);
    sig_mma<T>(acc, word(pv, 2), LX, LY, r0, c0, lane);
  }
  // Sig_t = -W Linv_k
  __syncthreads();
  put_acc_l<T>(acc, LX, 1.0, r0, c0, lane);
  st.store(LY);
  __syncthreads();
  st.load(M.tiles + t * TT);
  zero_acc<T>(acc);
  mma_tiles<T, false>(acc, LX, LY, r0, c0, lane);
  put_acc_g<T>(acc, sig, -1.0, r0, c0, lane);
  __syncthreads();
  put_acc_l<T>(acc, LX, -1.0, r0, c0, lane);   // LX = Sig_t
  st.store(LY);                                // LY = L_t
  __syncthreads();
  if (npush > 0) st.load(M.tiles + (int64_t)word(pv, pw0) * TT);
  // D_t = L_t^T Sig_t
  zero_acc<T>(acc);
  mma_tiles<T, true>(acc, LY, LX, r0, c0, lane);
  put_acc_g<T>(acc, M.dpart + t * TT, 1.0, r0, c0, lane);
  for (int q = 0; q < npush; q++) {
    const int64_t u = word(pv, pw0 + q);
    __syncthreads();
    st.store(LY);                              // LY = L_u
    __syncthreads();
    if (q + 1 < npush) st.load(M.tiles + (int64_t)word(pv, pw0 + q + 1) * TT);
    // Q_u = Sig_t^T L_u
    zero_acc<T>(acc);
    mma_tiles<T, true>(acc, LX, LY, r0, c0, lane);
    put_acc_g<T>(acc, M.qpart + u * TT, 1.0, r0, c0, lane);
  }
}

// SDIAG: Sig_kk = Linv_k^T (Linv_k - sum_r D_(r,k)), the D in list order
// (w4 = count, at most 64); the lower triangle is kept and mirrored, so the
// stored tile is symmetric.  Linv_k was staged in LX by selinv_prefetch.
template <int T>
__device__ __forceinline__ void task_sdiag(const ExecMat& M, const Task& w, double* LX, double* LY) {
  constexpr int TT = T * T, W = T / 2, NB = T / 32;
  typedef double d2 __attribute__((ext_vector_type(2)));
  const int lane = thread_id() & 63, wave = thread_id() >> 6;
  const int r0 = (wave >> 1) * W, c0 = (wave & 1) * W;
  const int nd = w[4];
  const int pv = w.pv;
  TileRegs<T> z;
#pragma unroll
  for (int v = 0; v < TileRegs<T>::NV; v++) z.r[v] = *z.at(LX, v);
  for (int q = 0; q < nd; q++) {
    const GLOBAL d2* dp = (const GLOBAL d2*)(M.dpart + (int64_t)word(pv, q) * TT);
#pragma unroll
    for (int v = 0; v < TileRegs<T>::NV; v++) z.r[v] -= dp[thread_id() + v * NT];
  }
  z.store(LY);
  __syncthreads();
  v4d acc[NB][NB];
  zero_acc<T>(acc);
  // Linv_k^T Z
  mma_tiles<T, true>(acc, LX, LY, r0, c0, lane);
  const DevTile<T> out(M.sigma + (int64_t)w[1] * TT);
  const Quarter<T> e(r0, c0, lane);
#pragma unroll
  for (int r = 0; r < 4; r++) {
    const int row = e.row0, col = e.col(0, r);   // NB x NB elements from here
    if constexpr (NB == 2) {
      // (above the diagonal: the mirrored element of a diagonal 2 x 2 block)
      const double up = row == col ? acc[0][NB - 1][r] : acc[NB - 1][0][r];
      if (row >= col) {
        out.store(row + col * T, v2d{acc[0][0][r], acc[0][NB - 1][r]});
        out.store(row + (col + 1) * T, v2d{up, acc[NB - 1][NB - 1][r]});
      }
      if (row > col) {
        out.store(col + row * T, v2d{acc[0][0][r], acc[NB - 1][0][r]});
        out.store(col + (row + 1) * T, v2d{acc[0][NB - 1][r], acc[NB - 1][NB - 1][r]});
      }
    } else if (row >= col) {
      out.store(row + col * T, acc[0][0][r]);
      out.store(col + row * T, acc[0][0][r]);
    }
  }
}

// TSUM: slot w1 = sum of the listed slots of dpart (c = 0) or qpart (c = 1),
// in list order; four running sums keep four loads in flight
template <int T>
__device__ __forceinline__ void task_tsum(const ExecMat& M, const Task& w) {
  constexpr int TT = T * T;
  typedef double d2 __attribute__((ext_vector_type(2)));
  double* base = w[4] == 1 ? M.qpart : M.dpart;
  const int32_t* lst = M.pairs + w[2];
  const int n = w[3];
  const DevTile<T> out(base + (int64_t)w[1] * TT);
  constexpr int NV = TT / 2 / NT;
  d2 s0[NV], s1[NV], s2[NV], s3[NV];
#pragma unroll
  for (int v = 0; v < NV; v++) s0[v] = s1[v] = s2[v] = s3[v] = d2{0.0, 0.0};
  auto slot = [&](int id) { return (const GLOBAL d2*)(base + (int64_t)id * TT); };
  for (int blk = 0; blk < n; blk += 64) {   // 64 slot words per load
    const int nb = n - blk < 64 ? n - blk : 64;
    const int pv = load_words(lst + blk, nb);
    int q = 0;
    for (; q + 4 <= nb; q += 4) {
      const GLOBAL d2* a = slot(word(pv, q));
      const GLOBAL d2* b = slot(word(pv, q + 1));
      const GLOBAL d2* c = slot(word(pv, q + 2));
      const GLOBAL d2* d = slot(word(pv, q + 3));
#pragma unroll
      for (int v = 0; v < NV; v++) {
        const int e = thread_id() + v * NT;
        s0[v] += a[e];
        s1[v] += b[e];
        s2[v] += c[e];
        s3[v] += d[e];
      }
    }
    for (; q < nb; q++) {
      const GLOBAL d2* a = slot(word(pv, q));
#pragma unroll
      for (int v = 0; v < NV; v++) s0[v] += a[thread_id() + v * NT];
    }
  }
#pragma unroll
  for (int v = 0; v < NV; v++) {
    const d2 t = (s0[v] + s1[v]) + (s2[v] + s3[v]);
    out.store(2 * (thread_id() + v * NT), t);
  }
}

// ---------------------------------------------------------------- executor

// first word and word count (at most 64 are read) of a task's operand list
__device__ __forceinline__ int operand_words(const ExecMat& M, const Task& w) {
  const int type = w[0] & 0xff;
  int off = 0, n = 0;
  if (type == TK_POTRF || type == TK_TRSM) {
    off = 2 * w[3];
    n = 2 * (w[4] - w[3]);
  } else if (type == TK_UPDB) {
    off = 2 * w[2];
    n = 4 + 4 * w[3];
  } else if (type == TK_SWE) {
    off = w[2];
    n = 2 * w[3];
  } else if (type == TK_SW) {
    off = w[3];
    n = 2 * (w[4] >> 16) + (w[4] & 0xff) + ((w[4] >> 8) & 0xff);
  } else if (type == TK_SDIAG) {
    off = w[3];
    n = w[4];
  } else if (type != TK_TREE && type != TK_FSUM && type != TK_TSUM) {
    off = 2 * w[2];
    n = 2 * (w[3] - w[2]);
  }
  return load_words(M.pairs + off, n);
}

// words of task lid and of its operand list
__device__ __forceinline__ void load_task(const ExecMat& M, int lid, Task& w) {
  const int wv = load_words(M.tasks + (int64_t)lid * TASK_WORDS, TASK_WORDS);
#pragma unroll
  for (int i = 0; i < TASK_WORDS; i++) w.w[i] = word(wv, i);
  w.pv = operand_words(M, w);
}

// One successor entry's decrement (Alg. 2 progress update).
__device__ __forceinline__ void notify_one(const ExecMat& M, int32_t sq) {
  int32_t dec = 1;
  if (sq & SUCC_FDEP) {   // an early predecessor of a two-stage wait
    dec = MERGED_FDEP;
    sq &= ~SUCC_FDEP;
  } else if (sq & SUCC_MID) {   // merged DAG: early solve predecessor of a diagonal step
    dec = SPLIT_W;
    sq &= ~SUCC_MID;
  }
  __hip_atomic_fetch_add(M.remaining + sq, -dec, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// per-task trace record
__device__ __forceinline__ void trace_task(const ExecMat& M, int lid, uint64_t claim, uint64_t start, int type,
                                           int ticket) {
  unsigned long long* tr = M.trace + 4 * (int64_t)lid;
  tr[0] = claim;
  tr[1] = start;
  tr[2] = wall_clock64();
  tr[3] = ((unsigned long long)blockIdx.x << 32) | ((unsigned)type << 24) | ((unsigned)ticket & 0xffffffu);
}

// LDS of the executor: factorization tasks use S (a tile; POTRF: leading
// dimension T + 17) and Xi (T x T) or, updates, the whole as a ring; solve
// tasks only a T x 16 block of Xi; selected-inversion tasks two tiles or the
// ring.  One object, so that the ring, whose transfers address LDS below
// 64 KB, starts at LDS address 0 whatever else the kernel keeps there.
template <int T, int KIND>
struct ExecLds {
  static constexpr bool SOLVE = KIND == EXEC_SOLVE;
  static constexpr int NS = SOLVE ? 2 : KIND == EXEC_SELINV ? T * T : T * (T + 17);
  static constexpr int NX = SOLVE ? SolveOps<T>::LDV * 16 : T * T;
  static constexpr int NR = SOLVE ? 0 : Ring<T, double>::NST * 2 * Ring<T, double>::HB / 8;
  double S[NS + NX > NR ? NS + NX : NR];
  int32_t ticket;   // the next task
  int32_t flag;     // the outcome of a wait
  int32_t last;     // the last workgroup to leave
};

// The task bodies are inlined into the executor: as functions they saved and
// restored their registers through scratch memory on every call (360 bytes a
// lane in the factorization kernel, 556 in the selected inversion).  With
// that, a task's static words read before its wait, its descriptor kept in
// scalar registers and the next ticket drawn while its stores complete, the
// part of an update task that does not depend on its product count fell from
// 8.4 to 4.7 us under full load, a panel TRSM from 6.7 to 4.4 us (with its
// strips), and the selected inversion of the n = 200,000 variable-band matrix
// from 20.4 to 13.5 ms.
// KIND selects the task set: factorization tasks (UPD, PART, TREE, POTRF,
// TRSM), triangular-solve tasks, or selected-inversion tasks; they are
// separate kernels so that each carries only its own code.
template <int T, int KIND>
__global__ __launch_bounds__(NT, T == 32 ? 3 : 2) void exec_kernel(const ExecMat* __restrict__ mats, const int32_t* __restrict__ order,
                                                  int32_t total, ExecCtrl* ctrl, int nrhs, uint64_t limit) {
  constexpr bool SOLVE = KIND == EXEC_SOLVE, SELINV = KIND == EXEC_SELINV, BOTH = KIND == EXEC_FACTOR_SOLVE;
  constexpr bool FACTOR = !SOLVE && !SELINV;
  typedef ExecLds<T, KIND> Lds;
  static_assert(offsetof(Lds, S) == 0, "transfers address LDS below 64 KB");
  __shared__ __attribute__((aligned(1024))) Lds lds;   // the kernel's only LDS object
  double* const S = lds.S;
  double* const Xi = S + Lds::NS;
  const Wait wt = {ctrl, limit, &lds.flag};
  // Control flow outside the task bodies is kept uniform across the
  // workgroup (values broadcast with readfirstlane, loops with uniform bounds
  // and predicated bodies): the compiler must never see a lane-divergent
  // region that straddles a barrier or the loop back-edge.
  if (threadIdx.x == 0) lds.ticket = atomicAdd(&ctrl->ticket, 1);
  __syncthreads();
  ExecMat M = mats[0];
  for (;;) {
    const int32_t t = __builtin_amdgcn_readfirstlane(lds.ticket);
    if (t >= total) break;
    int32_t mi = 0, lid = t;
    if (order) {
      mi = __builtin_amdgcn_readfirstlane(order[2 * t]);
      lid = __builtin_amdgcn_readfirstlane(order[2 * t + 1]);
      M = mats[mi];
    }
    Task w;
    load_task(M, lid, w);
    // the first successors, for the notification
    int32_t nsucc = w[6] - w[5];
    int succ0 = load_words(M.succ + w[5], nsucc);
    int32_t* cnt = M.remaining + lid;
    uint64_t t_claim = 0, t_start = 0;
    if (M.trace) t_claim = wall_clock64();
    const int type = w[0] & 0xff;
    // a TRSM of the pivot chain carries the next POTRF with it, whose own
    // ticket is void
    if (FACTOR && type == TK_POTRF && (w[0] & TF_CHAIN) != 0) {
      __syncthreads();
      if (threadIdx.x == 0) lds.ticket = atomicAdd(&ctrl->ticket, 1);
      __syncthreads();
      continue;
    }
    if constexpr (SELINV) selinv_prefetch<T>(M, w, S, Xi);
    // merged factorization + solve DAG: a solve task first waits for its
    // factorization predecessors only (the counter falls below MERGED_FDEP);
    // its factor tiles are final then
    bool ok = true;
    if constexpr (BOTH) {
      if (type >= TK_FUPD) ok = wait_below(cnt, MERGED_FDEP, wt);
    }
    // solve tasks other than FSUM wait for their predecessors themselves,
    // after reading their factor tiles; so do POTRF and TRSM (two-stage)
    const bool self_wait = ((SOLVE || BOTH) && type >= TK_FUPD && type != TK_FSUM) ||
                           (!SOLVE && !SELINV && (type == TK_POTRF || type == TK_TRSM));
    // wait until every predecessor has finished (Alg. 2 progress check);
    // wave 0 polls, then acquires for the workgroup (all its waves share
    // the CU's caches that the acquire invalidates)
    if (!self_wait && ok) ok = wait_below(cnt, 1, wt);
    if (M.trace) t_start = wall_clock64();
    // tasks on the pivot chain (diagonal factorization, panel solve, diagonal
    // solve steps) raise their waves' issue priority over the co-resident
    // update work of other workgroups on the same SIMDs
    const bool chain = SOLVE    ? (type == TK_FDIAG || type == TK_BDIAG)
                       : SELINV ? (type == TK_SW || type == TK_SDIAG)
                                : (type == TK_POTRF || type == TK_TRSM || type == TK_FDIAG || type == TK_BDIAG);
    if (chain) __builtin_amdgcn_s_setprio(3);
    if constexpr (SELINV) {
      if (!ok) {
      } else if (type == TK_SWE) task_swe<T>(M, w, S);
      else if (type == TK_SW) task_sw<T>(M, w, S, Xi);
      else if (type == TK_SDIAG) task_sdiag<T>(M, w, S, Xi);
      else task_tsum<T>(M, w);
    } else if constexpr (SOLVE) {
      if (type == TK_FSUM) {
        if (ok) task_fsum<T>(M, w, nrhs);
      } else {
        t_start = task_solve_r<T, KIND>(M, w, nrhs, cnt, Xi, wt, ok);
      }
    } else if (BOTH && type >= TK_FUPD) {
      if (type == TK_FSUM) {
        if (ok) task_fsum<T>(M, w, nrhs);
      } else {
        t_start = task_solve_r<T, KIND>(M, w, nrhs, cnt, Xi, wt, ok);
      }
    } else if (ok) {
      switch (type) {
        case TK_UPD: task_update<T>(M, w, 0, S); break;
        case TK_UPDB: task_update_block<T, KIND>(mats + mi, w[0], w[3], w.pv, S, Xi); break;
        case TK_PART: task_update<T>(M, w, 1, S); break;
        case TK_TREE: task_tree<T>(M, w); break;
        default: {
          // TRSM, POTRF, or both (the POTRF is the TRSM's first successor)
          const bool pair = (w[0] & TF_CHAIN) != 0;
          bool staged = false;
          uint64_t t_trsm = 0;
          Task w2 = w;
          int lid2 = lid, succ2 = succ0;
          if (type == TK_TRSM) {
            if (pair) {
              lid2 = word(succ0, 0) & ~(SUCC_FDEP | SUCC_MID);
              load_task(M, lid2, w2);
              succ2 = load_words(M.succ + w2[5], w2[6] - w2[5]);
            }
            t_start = t_trsm = task_trsm<T>(M, w, S, Xi, cnt, wt, ok, pair, M.remaining + lid2,
                                            M.tiles + (int64_t)w2[1] * (T * T), staged);
            if (!ok || !pair) break;
          }
          const int lid1 = lid, w5 = w[5], w7 = w[7], ns1 = nsucc, s1 = succ0;
          lid = lid2;
          w = w2;
          nsucc = w2[6] - w2[5];
          succ0 = succ2;
          cnt = M.remaining + lid2;
          // the TRSM's end, by the last wave (the first one has the panels)
          auto lead = [&]() INLINE {
            const int l = thread_id() - (NT - 64);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            if (l == 0) st_relaxed(M.remaining + lid1, w7);
            for (int32_t q0 = 0; q0 < ns1; q0 += 64) {
              const int32_t q = q0 + l;
              if (l >= 0 && q > 0 && q < ns1) notify_one(M, q0 == 0 ? s1 : gp(M.succ)[w5 + q]);
            }
            if (M.trace && l == 0) trace_task(M, lid1, t_claim, t_trsm, TK_TRSM, t);
          };
          t_start = task_potrf<T>(M, w, S, Xi, cnt, wt, ok, pair, staged, lead);
          break;
        }
      }
    }
    if (chain) __builtin_amdgcn_s_setprio(0);
    // the next ticket is drawn while this task's stores complete (the task
    // no longer waits for anything, so a ticket is never held by a workgroup
    // that waits for a later one)
    int32_t next = 0;
    if (threadIdx.x == 0) next = atomicAdd(&ctrl->ticket, 1);
    if (!ok) {
      // abandoned launch: the task is skipped and its matrix marked as timed
      // out (info 0, below every failing column); no successor is notified
      // and the counters are re-armed by the last workgroup to leave
      if (threadIdx.x == 0) {
        atomicMin(M.info, 0ull);
        lds.ticket = next;
      }
      __syncthreads();
      continue;
    }
    // every wave waits for its own stores (device-scope stores, coherent
    // once complete), then wave 0 notifies the successors (Alg. 2 progress
    // update); the workgroup-scope release only orders the notification
    // after the stores in the compiler
    __builtin_amdgcn_s_waitcnt(0);
    if (threadIdx.x == 0) lds.ticket = next;
    __syncthreads();
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    if (threadIdx.x == 0) st_relaxed(cnt, w[7]);   // re-arm for the next launch
    for (int32_t q0 = 0; q0 < nsucc; q0 += 64) {
      const int32_t q = q0 + (int32_t)threadIdx.x;
      if (threadIdx.x < 64 && q < nsucc) notify_one(M, q0 == 0 ? succ0 : gp(M.succ)[w[5] + q]);
    }
    if (M.trace && threadIdx.x == 0) trace_task(M, lid, t_claim, t_start, w[0] & 0xff, t);
  }
  // the last workgroup to leave re-arms the control block; after an abort it
  // also re-arms every progress counter of the launch (skipped tasks did not
  // re-arm theirs, and some were notified after being skipped).  Every
  // workgroup's notifications are complete before it counts itself out.
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if (threadIdx.x == 0) {
    fence_release();
    const int e = atomicAdd(&ctrl->exited, 1);
    lds.last = e == (int)gridDim.x - 1;
  }
  __syncthreads();
  if (__builtin_amdgcn_readfirstlane(lds.last)) {
    fence_acquire();
    if (__builtin_amdgcn_readfirstlane(ld_relaxed(&ctrl->abort)) != 0) {
      for (int32_t t = threadIdx.x; t < total; t += NT) {
        int32_t mi = 0, lid = t;
        if (order) {
          mi = order[2 * t];
          lid = order[2 * t + 1];
        }
        st_relaxed(mats[mi].remaining + lid, mats[mi].tasks[(int64_t)lid * TASK_WORDS + 7]);
      }
      __builtin_amdgcn_s_waitcnt(0);
      __syncthreads();
    }
    if (threadIdx.x == 0) {
      st_relaxed(&ctrl->abort, 0);
      ctrl->ticket = 0;
      ctrl->exited = 0;
    }
  }
}

hipError_t launch_exec(int T, int kind, const ExecMat* d_mats, const int32_t* d_order, int32_t total,
                       ExecCtrl* d_ctrl, int nrhs, int nwg, uint64_t wait_ticks, hipStream_t st) {
  if (total <= 0) return hipSuccess;
  if (nwg > total) nwg = total;
#define STILES_EXEC(TT, KK) \
  hipLaunchKernelGGL((exec_kernel<TT, KK>), dim3(nwg), dim3(NT), 0, st, d_mats, d_order, total, d_ctrl, nrhs, wait_ticks)
  if (T == 64) {
    if (kind == EXEC_SOLVE) STILES_EXEC(64, EXEC_SOLVE);
    else if (kind == EXEC_SELINV) STILES_EXEC(64, EXEC_SELINV);
    else if (kind == EXEC_FACTOR_SOLVE) STILES_EXEC(64, EXEC_FACTOR_SOLVE);
    else STILES_EXEC(64, EXEC_FACTOR);
  } else {
    if (kind == EXEC_SOLVE) STILES_EXEC(32, EXEC_SOLVE);
    else if (kind == EXEC_SELINV) STILES_EXEC(32, EXEC_SELINV);
    else if (kind == EXEC_FACTOR_SOLVE) STILES_EXEC(32, EXEC_FACTOR_SOLVE);
    else STILES_EXEC(32, EXEC_FACTOR);
  }
#undef STILES_EXEC
  return hipGetLastError();
}

// diagonal of Sigma (selected inversion) in the original ordering; NaN when
// the factorization failed.  One workgroup per tile row, one thread per row.
template <int T>
__global__ void selinv_diag_kernel(const double* __restrict__ sigma, const int32_t* __restrict__ trow_ptr,
                                   const int64_t* __restrict__ row_base, const int32_t* __restrict__ row_cnt,
                                   const int64_t* __restrict__ perm, int32_t ntr, const unsigned long long* info,
                                   double* __restrict__ out) {
  const int m = blockIdx.x, i = threadIdx.x;
  if (m >= ntr || i >= row_cnt[m]) return;
  const double v = sigma[(int64_t)(trow_ptr[m + 1] - 1) * T * T + i + i * T];
  out[perm[row_base[m] + i]] = *info != ~0ull ? __builtin_nan("") : v;
}

hipError_t launch_selinv_diag(int T, const double* sigma, const int32_t* trow_ptr, const int64_t* row_base,
                              const int32_t* row_cnt, const int64_t* perm, int32_t ntr,
                              const unsigned long long* info, double* out, hipStream_t st) {
  if (ntr <= 0) return hipSuccess;
  if (T == 64)
    hipLaunchKernelGGL((selinv_diag_kernel<64>), dim3(ntr), dim3(64), 0, st, sigma, trow_ptr, row_base, row_cnt, perm,
                       ntr, info, out);
  else
    hipLaunchKernelGGL((selinv_diag_kernel<32>), dim3(ntr), dim3(32), 0, st, sigma, trow_ptr, row_base, row_cnt, perm,
                       ntr, info, out);
  return hipGetLastError();
}

// ------------------------------------------------------------ value scatter

// column-major T x T tile out (and o2) from the row-major LDS buffer
// (leading dimension T + 1): two rows per 16-byte streaming store
template <int T>
__device__ __forceinline__ void store_tile_cm(const double* buf, double* out, double* o2) {
  typedef double d2 __attribute__((ext_vector_type(2)));
  constexpr int TT = T * T;
  GLOBAL d2* go = (GLOBAL d2*)out;
  GLOBAL d2* g2 = o2 ? (GLOBAL d2*)o2 : nullptr;
  for (int e2 = threadIdx.x; e2 < TT / 2; e2 += NT) {
    const int e = 2 * e2, c = e / T, r = e % T;
    const d2 v = d2{buf[r * (T + 1) + c], buf[(r + 1) * (T + 1) + c]};
    __builtin_nontemporal_store(v, go + e2);
    if (g2) __builtin_nontemporal_store(v, g2 + e2);
  }
}

// One T x T tile of the store from row-profile values: staged through LDS so
// that the reads follow the input rows and the stores the column-major tile.
// The first column and start offset of each of the tile's rows are read once
// into LDS, so every element costs one global load.
template <int T>
__device__ __forceinline__ void scatter_tile(const double* __restrict__ vals, const int64_t* __restrict__ in_rp,
                                             const int64_t* __restrict__ f, int m, int j,
                                             const int64_t* __restrict__ row_base,
                                             const int32_t* __restrict__ row_cnt, double* out, double* o2,
                                             double* buf) {
  constexpr int TT = T * T;
  __shared__ int64_t sf[T], sp[T];
  const int64_t rb = row_base[m], cb = row_base[j];
  const int rc = row_cnt[m], cc = row_cnt[j];
  if ((int)threadIdx.x < rc) {
    sf[threadIdx.x] = f[rb + threadIdx.x];
    sp[threadIdx.x] = in_rp[rb + threadIdx.x];
  }
  __syncthreads();
  // row-wise: consecutive threads read consecutive values; all of a
  // thread's loads are issued before any LDS store
  constexpr int NQ = TT / NT;
  double v[NQ];
#pragma unroll
  for (int q = 0; q < NQ; q++) {
    const int e = (int)threadIdx.x + q * NT;
    const int r = e / T, c = e % T;
    v[q] = (r >= rc && m == j && r == c) ? 1.0 : 0.0;   // padding row: unit diagonal
    if (r < rc) {
      const int64_t i = rb + r, g = cb + c;
      const int64_t fi = sf[r];
      if (c < cc && g <= i && g >= fi) v[q] = gp(vals)[sp[r] + (g - fi)];
    }
  }
#pragma unroll
  for (int q = 0; q < NQ; q++) {
    const int e = (int)threadIdx.x + q * NT;
    buf[(e / T) * (T + 1) + e % T] = v[q];
  }
  __syncthreads();
  store_tile_cm<T>(buf, out, o2);
}

template <int T>
__global__ __launch_bounds__(NT) void scatter_profile_kernel(const double* __restrict__ vals,
                                                             const int64_t* __restrict__ in_rp,
                                                             const int64_t* __restrict__ f,
                                                             const int32_t* __restrict__ trow,
                                                             const int32_t* __restrict__ tcol,
                                                             const int64_t* __restrict__ row_base,
                                                             const int32_t* __restrict__ row_cnt, double* tiles,
                                                             double* orig, unsigned long long* info) {
  constexpr int TT = T * T;
  __shared__ double buf[T * (T + 1)];
  const int64_t t = blockIdx.x;
  scatter_tile<T>(vals, in_rp, f, trow[t], tcol[t], row_base, row_cnt, tiles + t * TT, orig ? orig + t * TT : nullptr,
                  buf);
  if (t == 0 && threadIdx.x == 0) *info = ~0ull;
}

// Tile of P A P^T from row-profile values of the input ordering: element
// (r, c) of tile (m, j) is the input entry (perm[row], perm[col]), taken from
// the lower triangle (larger index as the row).  The gathers follow the tile
// rows; entries of reversed blocks are read transposed.
template <int T>
__device__ __forceinline__ void scatter_tile_perm(const double* __restrict__ vals, const int64_t* __restrict__ in_rp,
                                                  const int64_t* __restrict__ fin, const int64_t* __restrict__ perm,
                                                  int m, int j, const int64_t* __restrict__ row_base,
                                                  const int32_t* __restrict__ row_cnt, double* out, double* o2,
                                                  double* buf) {
  constexpr int TT = T * T;
  // per row and per column of the tile: input index, its first column and
  // its value offset (the larger input index of an entry names its row)
  __shared__ int64_t pr[T], pc[T], fr[T], fc[T], sr[T], sc[T];
  const int64_t rb = row_base[m], cb = row_base[j];
  const int rc = row_cnt[m], cc = row_cnt[j];
  if (threadIdx.x < T) {
    const int r = threadIdx.x;
    if (r < rc) {
      const int64_t o = perm[rb + r];
      pr[r] = o;
      fr[r] = fin[o];
      sr[r] = in_rp[o];
    }
  } else if (threadIdx.x < 2 * T) {
    const int c = threadIdx.x - T;
    if (c < cc) {
      const int64_t o = perm[cb + c];
      pc[c] = o;
      fc[c] = fin[o];
      sc[c] = in_rp[o];
    }
  }
  __syncthreads();
  // all of a thread's loads are issued before any LDS store (TT / NT of them
  // in flight per thread)
  constexpr int NQ = TT / NT;
  double v[NQ];
#pragma unroll
  for (int q = 0; q < NQ; q++) {
    const int e = (int)threadIdx.x + q * NT;
    const int r = e / T, c = e % T;
    v[q] = (r >= rc && m == j && r == c) ? 1.0 : 0.0;   // padding row: unit diagonal
    if (r < rc && c < cc && cb + c <= rb + r) {
      const int64_t oi = pr[r], oj = pc[c];
      const bool rowi = oi > oj;
      const int64_t lo = rowi ? oj : oi;
      const int64_t fh = rowi ? fr[r] : fc[c];
      const int64_t base = rowi ? sr[r] : sc[c];
      if (lo >= fh) v[q] = gp(vals)[base + (lo - fh)];
    }
  }
#pragma unroll
  for (int q = 0; q < NQ; q++) {
    const int e = (int)threadIdx.x + q * NT;
    buf[(e / T) * (T + 1) + e % T] = v[q];
  }
  __syncthreads();
  store_tile_cm<T>(buf, out, o2);
}

template <int T>
__global__ __launch_bounds__(NT) void scatter_perm_kernel(const double* __restrict__ vals,
                                                          const int64_t* __restrict__ in_rp,
                                                          const int64_t* __restrict__ fin,
                                                          const int64_t* __restrict__ perm,
                                                          const int32_t* __restrict__ trow,
                                                          const int32_t* __restrict__ tcol,
                                                          const int64_t* __restrict__ row_base,
                                                          const int32_t* __restrict__ row_cnt, double* tiles,
                                                          double* orig, unsigned long long* info) {
  constexpr int TT = T * T;
  __shared__ double buf[T * (T + 1)];
  const int64_t t = blockIdx.x;
  scatter_tile_perm<T>(vals, in_rp, fin, perm, trow[t], tcol[t], row_base, row_cnt, tiles + t * TT,
                       orig ? orig + t * TT : nullptr, buf);
  if (t == 0 && threadIdx.x == 0) *info = ~0ull;
}

hipError_t launch_scatter_perm(int T, const double* vals, const int64_t* in_rp, const int64_t* fin, const int64_t* perm,
                               const int32_t* trow, const int32_t* tcol, const int64_t* row_base,
                               const int32_t* row_cnt, int64_t ntiles, double* tiles, double* orig,
                               unsigned long long* info, hipStream_t st) {
  if (T == 64)
    hipLaunchKernelGGL(scatter_perm_kernel<64>, dim3((unsigned)ntiles), dim3(NT), 0, st, vals, in_rp, fin, perm, trow,
                       tcol, row_base, row_cnt, tiles, orig, info);
  else
    hipLaunchKernelGGL(scatter_perm_kernel<32>, dim3((unsigned)ntiles), dim3(NT), 0, st, vals, in_rp, fin, perm, trow,
                       tcol, row_base, row_cnt, tiles, orig, info);
  return hipGetLastError();
}

// every tile of every matrix of a batch: block b handles tile tmap[b].y of
// matrix tmap[b].x
template <int T>
__global__ __launch_bounds__(NT) void scatter_batch_kernel(const BatchDesc* __restrict__ desc,
                                                           const double* const* __restrict__ vals,
                                                           const int2* __restrict__ tmap) {
  constexpr int TT = T * T;
  __shared__ double buf[T * (T + 1)];
  const int2 mt = tmap[blockIdx.x];
  const BatchDesc& d = desc[mt.x];
  const int64_t t = mt.y;
  if (d.perm)
    scatter_tile_perm<T>(vals[mt.x], d.in_rp, d.f, d.perm, d.trow[t], d.tcol[t], d.row_base, d.row_cnt,
                         d.tiles + t * TT, d.orig ? d.orig + t * TT : nullptr, buf);
  else
    scatter_tile<T>(vals[mt.x], d.in_rp, d.f, d.trow[t], d.tcol[t], d.row_base, d.row_cnt, d.tiles + t * TT,
                    d.orig ? d.orig + t * TT : nullptr, buf);
  if (t == 0 && threadIdx.x == 0) *d.info = ~0ull;
}

hipError_t launch_scatter_batch(int T, const BatchDesc* desc, const double* const* vals, const int2* tmap,
                                int64_t total_tiles, hipStream_t st) {
  if (total_tiles <= 0) return hipSuccess;
  if (T == 64)
    hipLaunchKernelGGL(scatter_batch_kernel<64>, dim3((unsigned)total_tiles), dim3(NT), 0, st, desc, vals, tmap);
  else
    hipLaunchKernelGGL(scatter_batch_kernel<32>, dim3((unsigned)total_tiles), dim3(NT), 0, st, desc, vals, tmap);
  return hipGetLastError();
}

hipError_t launch_scatter_profile(int T, const double* vals, const int64_t* in_rp, const int64_t* f,
                                  const int32_t* trow, const int32_t* tcol, const int64_t* row_base,
                                  const int32_t* row_cnt, int64_t ntiles, double* tiles, double* orig,
                                  unsigned long long* info, hipStream_t st) {
  if (T == 64)
    hipLaunchKernelGGL(scatter_profile_kernel<64>, dim3((unsigned)ntiles), dim3(NT), 0, st, vals, in_rp, f, trow, tcol,
                       row_base, row_cnt, tiles, orig, info);
  else
    hipLaunchKernelGGL(scatter_profile_kernel<32>, dim3((unsigned)ntiles), dim3(NT), 0, st, vals, in_rp, f, trow, tcol,
                       row_base, row_cnt, tiles, orig, info);
  return hipGetLastError();
}

template <int T>
__global__ __launch_bounds__(NT) void fill_tiles_kernel(const int32_t* __restrict__ trow,
                                                        const int32_t* __restrict__ tcol,
                                                        const int32_t* __restrict__ row_cnt, double* tiles,
                                                        unsigned long long* info) {
  constexpr int TT = T * T;
  const int64_t t = blockIdx.x;
  const int m = trow[t], j = tcol[t], rc = row_cnt[m];
  double* out = tiles + t * TT;
  for (int e = threadIdx.x; e < TT; e += NT) {
    const int r = e % T, c = e / T;
    out[e] = (m == j && r == c && r >= rc) ? 1.0 : 0.0;
  }
  if (t == 0 && threadIdx.x == 0) *info = ~0ull;
}

__global__ void map_scatter_kernel(const double* __restrict__ vals, const int64_t* __restrict__ map, int64_t nnz,
                                   double* tiles, double* orig) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < nnz) {
    const int64_t o = map[e];
    tiles[o] = vals[e];
    if (orig) orig[o] = vals[e];
  }
}

hipError_t launch_scatter_map(int T, const double* vals, const int64_t* map, int64_t nnz, const int32_t* trow,
                              const int32_t* tcol, const int32_t* row_cnt, int64_t ntiles, double* tiles,
                              double* orig, unsigned long long* info, hipStream_t st) {
  if (T == 64) {
    hipLaunchKernelGGL(fill_tiles_kernel<64>, dim3((unsigned)ntiles), dim3(NT), 0, st, trow, tcol, row_cnt, tiles, info);
    if (orig)
      hipLaunchKernelGGL(fill_tiles_kernel<64>, dim3((unsigned)ntiles), dim3(NT), 0, st, trow, tcol, row_cnt, orig, info);
  } else {
    hipLaunchKernelGGL(fill_tiles_kernel<32>, dim3((unsigned)ntiles), dim3(NT), 0, st, trow, tcol, row_cnt, tiles, info);
    if (orig)
      hipLaunchKernelGGL(fill_tiles_kernel<32>, dim3((unsigned)ntiles), dim3(NT), 0, st, trow, tcol, row_cnt, orig, info);
  }
  if (nnz > 0)
    hipLaunchKernelGGL(map_scatter_kernel, dim3((unsigned)((nnz + NT - 1) / NT)), dim3(NT), 0, st, vals, map, nnz,
                       tiles, orig);
  return hipGetLastError();
}

template <int T>
__global__ __launch_bounds__(NT) void extract_kernel(const double* __restrict__ tiles, const int64_t* __restrict__ rp,
                                                     const int64_t* __restrict__ f, const int32_t* __restrict__ trow,
                                                     const int32_t* __restrict__ tcol,
                                                     const int64_t* __restrict__ row_base,
                                                     const int32_t* __restrict__ row_cnt, double* out) {
  constexpr int TT = T * T;
  const int64_t t = blockIdx.x;
  const int m = trow[t], j = tcol[t];
  const int64_t rb = row_base[m], cb = row_base[j];
  const int rc = row_cnt[m], cc = row_cnt[j];
  const double* src = tiles + t * TT;
  for (int e = threadIdx.x; e < TT; e += NT) {
    const int c = e / T, r = e % T;
    if (r >= rc || c >= cc) continue;
    const int64_t i = rb + r, g = cb + c;
    if (g <= i && g >= f[i]) out[rp[i] + (g - f[i])] = src[e];
  }
}

__global__ void zero_kernel(double* out, int64_t n) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x)
    out[e] = 0.0;
}

hipError_t launch_extract(int T, const double* tiles, const int64_t* rp, const int64_t* f, const int32_t* trow,
                          const int32_t* tcol, const int64_t* row_base, const int32_t* row_cnt, int64_t ntiles,
                          int64_t nnz, double* out, hipStream_t st) {
  // envelope entries outside the stored tiles (structural zeros of L) are zero
  if (nnz > 0)
    hipLaunchKernelGGL(zero_kernel, dim3((unsigned)std::min<int64_t>((nnz + NT - 1) / NT, 65536)), dim3(NT), 0, st, out,
                       nnz);
  if (T == 64)
    hipLaunchKernelGGL(extract_kernel<64>, dim3((unsigned)ntiles), dim3(NT), 0, st, tiles, rp, f, trow, tcol, row_base,
                       row_cnt, out);
  else
    hipLaunchKernelGGL(extract_kernel<32>, dim3((unsigned)ntiles), dim3(NT), 0, st, tiles, rp, f, trow, tcol, row_base,
                       row_cnt, out);
  return hipGetLastError();
}

// ------------------------------------------------------------------ logdet

// log-determinant: per tile row a fixed-shape wave reduction of log L_ii,
// then one block sums the tile-row partials (strided, then a binary tree).
// The single-matrix and batched launches share these two steps, so their
// results agree bit for bit.
template <int T>
__device__ __forceinline__ void logdet_row(const double* __restrict__ D, double* part_m, double* ws) {
  double v = threadIdx.x < T ? log(D[threadIdx.x * (T + 1)]) : 0.0;
  for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
  if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    double s = 0.0;
    for (int q = 0; q < NT / 64; q++) s += ws[q];
    *part_m = s;
  }
}

__device__ __forceinline__ void logdet_sum(const double* __restrict__ part, int32_t n,
                                           const unsigned long long* info, double* out, double* sh) {
  double s = 0.0;
  for (int i = threadIdx.x; i < n; i += NT) s += part[i];
  sh[threadIdx.x] = s;
  __syncthreads();
  for (int o = NT / 2; o > 0; o >>= 1) {
    if (threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = (*info == ~0ull) ? 2.0 * sh[0] : __builtin_nan("");
}

template <int T>
__global__ __launch_bounds__(NT) void logdet_partial_kernel(const double* __restrict__ tiles,
                                                            const int32_t* __restrict__ trow_ptr, double* part) {
  constexpr int TT = T * T;
  __shared__ double ws[NT / 64];
  const int m = blockIdx.x;
  logdet_row<T>(tiles + (int64_t)(trow_ptr[m + 1] - 1) * TT, part + m, ws);
}

__global__ __launch_bounds__(NT) void logdet_final_kernel(const double* __restrict__ part, int32_t n,
                                                          const unsigned long long* info, double* out) {
  __shared__ double sh[NT];
  logdet_sum(part, n, info, out, sh);
}

template <int T>
__global__ __launch_bounds__(NT) void logdet_partial_batch_kernel(const BatchDesc* __restrict__ desc,
                                                                  const int2* __restrict__ rmap) {
  constexpr int TT = T * T;
  __shared__ double ws[NT / 64];
  const int2 mr = rmap[blockIdx.x];
  const BatchDesc& d = desc[mr.x];
  logdet_row<T>(d.tiles + (int64_t)(d.trow_ptr[mr.y + 1] - 1) * TT, d.ldpart + mr.y, ws);
}

__global__ __launch_bounds__(NT) void logdet_final_batch_kernel(const BatchDesc* __restrict__ desc, double* out) {
  __shared__ double sh[NT];
  const BatchDesc& d = desc[blockIdx.x];
  logdet_sum(d.ldpart, d.ntr, d.info, out + blockIdx.x, sh);
}

hipError_t launch_logdet(int T, const double* tiles, const int32_t* trow_ptr, int32_t ntr, double* part,
                         const unsigned long long* info, double* out, hipStream_t st) {
  if (T == 64)
    hipLaunchKernelGGL(logdet_partial_kernel<64>, dim3(ntr), dim3(NT), 0, st, tiles, trow_ptr, part);
  else
    hipLaunchKernelGGL(logdet_partial_kernel<32>, dim3(ntr), dim3(NT), 0, st, tiles, trow_ptr, part);
  hipLaunchKernelGGL(logdet_final_kernel, dim3(1), dim3(NT), 0, st, part, ntr, info, out);
  return hipGetLastError();
}

// Per-tile-row partial sums of the log-determinant for callers that cannot
// allocate device memory (launch_logdet_static): a fixed array of the
// library, one copy per GPU, held until the process ends.  Host code never
// passes the array's name to a kernel (on the host it is only a stand-in
// for the symbol): it uses the device address that hipGetSymbolAddress
// returns, looked up once per device with that device current.  Every call
// on one GPU shares the array; each launch overwrites the partials of its
// own rows before the final sum reads them, so nothing needs clearing, and
// calls that overlap on one GPU race.
static __device__ __align__(256) double scratch[STATIC_LOGDET_ROWS];

namespace {
std::mutex g_scratch_mu;
double* g_scratch_ptr[64] = {};
}  // namespace

hipError_t static_scratch(double** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!ptr) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = static_cast<double*>(ptr);
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}

hipError_t launch_logdet_static(int T, const double* tiles, const int32_t* trow_ptr, int32_t ntr,
                                const unsigned long long* info, double* out, hipStream_t st) {
  if (ntr < 1 || ntr > STATIC_LOGDET_ROWS) return hipErrorInvalidValue;
  double* part = nullptr;
  hipError_t e = static_scratch(&part);
  if (e != hipSuccess) return e;
  return launch_logdet(T, tiles, trow_ptr, ntr, part, info, out, st);
}

hipError_t launch_logdet_batch(int T, const BatchDesc* desc, int32_t count, const int2* rmap, int64_t total_rows,
                               double* out, hipStream_t st) {
  if (count <= 0 || total_rows <= 0) return hipSuccess;
  if (T == 64)
    hipLaunchKernelGGL(logdet_partial_batch_kernel<64>, dim3((unsigned)total_rows), dim3(NT), 0, st, desc, rmap);
  else
    hipLaunchKernelGGL(logdet_partial_batch_kernel<32>, dim3((unsigned)total_rows), dim3(NT), 0, st, desc, rmap);
  hipLaunchKernelGGL(logdet_final_batch_kernel, dim3((unsigned)count), dim3(NT), 0, st, desc, out);
  return hipGetLastError();
}

// ------------------------------------------------------------ pack / unpack

__global__ void pack_kernel(int T, const double* __restrict__ B, int64_t ldb, int nrhs, const int64_t* __restrict__ perm,
                            const int64_t* __restrict__ row_base, const int32_t* __restrict__ row_cnt, int32_t ntr,
                            double* Y) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t vb = (int64_t)T * nrhs;
  if (e >= vb * ntr) return;
  const int64_t m = e / vb, rem = e % vb;
  const int c = (int)(rem / T), r = (int)(rem % T);
  Y[e] = r < row_cnt[m] ? B[perm[row_base[m] + r] + c * ldb] : 0.0;
}

__global__ void unpack_kernel(int T, const double* __restrict__ Z, int nrhs, const int64_t* __restrict__ perm,
                              const int64_t* __restrict__ row_base, const int32_t* __restrict__ row_cnt, int32_t ntr,
                              const unsigned long long* info, double* B, int64_t ldb) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t vb = (int64_t)T * nrhs;
  if (e >= vb * ntr) return;
  const int64_t m = e / vb, rem = e % vb;
  const int c = (int)(rem / T), r = (int)(rem % T);
  if (r < row_cnt[m]) B[perm[row_base[m] + r] + c * ldb] = (*info == ~0ull) ? Z[e] : __builtin_nan("");
}

hipError_t launch_pack(int T, const double* B, int64_t ldb, int nrhs, const int64_t* perm, const int64_t* row_base,
                       const int32_t* row_cnt, int32_t ntr, double* Y, hipStream_t st) {
  const int64_t n = (int64_t)T * nrhs * ntr;
  hipLaunchKernelGGL(pack_kernel, dim3((unsigned)((n + NT - 1) / NT)), dim3(NT), 0, st, T, B, ldb, nrhs, perm, row_base,
                     row_cnt, ntr, Y);
  return hipGetLastError();
}

hipError_t launch_unpack(int T, const double* Z, int nrhs, const int64_t* perm, const int64_t* row_base,
                         const int32_t* row_cnt, int32_t ntr, const unsigned long long* info, double* B, int64_t ldb,
                         hipStream_t st) {
  const int64_t n = (int64_t)T * nrhs * ntr;
  hipLaunchKernelGGL(unpack_kernel, dim3((unsigned)((n + NT - 1) / NT)), dim3(NT), 0, st, T, Z, nrhs, perm, row_base,
                     row_cnt, ntr, info, B, ldb);
  return hipGetLastError();
}

}  // namespace stiles

// ------------------------------------------------- refinement (mixed mode)

namespace stiles {

// Residual items on MFMA: each tile of the item is staged in LDS
// (with |.| in absmode), multiplied with the vector block (A x for row items,
// A^T x for column items; a diagonal tile adds its strict lower part
// transposed), and the item's partial written once.
template <int T>
__global__ __launch_bounds__(NT) void residual_mma_kernel(const double* __restrict__ orig,
                                                          const int32_t* __restrict__ rtile,
                                                          const int32_t* __restrict__ tcol,
                                                          const int32_t* __restrict__ ccol_tile,
                                                          const int32_t* __restrict__ ccol_row,
                                                          const int32_t* __restrict__ items,
                                                          const double* __restrict__ X, double* part, double* apart,
                                                          int nrhs, int absmode) {
  // operands straight from global memory into registers (SolveOps layout),
  // two tiles in flight; wave w owns rows 16 w .. 16 w + 15 of the T x 16 result.
  // With apart (residual pass), the row sums of |A| over the same operands
  // are accumulated too (one pass over A gives both).
  typedef SolveOps<T> O;
  constexpr int TT = T * T, NS = O::NS;
  const int q = blockIdx.x;
  const int m = items[4 * q], kind = items[4 * q + 1], lo = items[4 * q + 2], hi = items[4 * q + 3];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const bool act = 16 * wave < T;
  const int col = lane & 15, g = lane >> 4, r = O::a_row(wave, lane);
  const int64_t vb = (int64_t)T * nrhs;
  const int ncol = absmode ? 1 : nrhs;
  const bool trans = kind == 1;
  v4d acc = v4d{0.0, 0.0, 0.0, 0.0};
  double rs = 0.0;   // this lane's share of the row sum of |A| (apart)
  if (!act) return;
  double a[2][NS], b[2][NS];
  // operands of item entry e into slot u
  auto load = [&](int u, int e) {
    const int tile = kind == 0 ? rtile[e] : ccol_tile[e];
    const int src = kind == 0 ? tcol[tile] : ccol_row[e];
    O::load_a(a[u], orig + (int64_t)tile * TT, trans, wave, lane);
    if (absmode) {
#pragma unroll
      for (int s = 0; s < NS; s++) b[u][s] = col == 0 ? 1.0 : 0.0;
    } else {
      O::load_b(b[u], X + src * vb, nrhs, lane);
    }
  };
  auto use = [&](int u, int e) {
    if (absmode) {
#pragma unroll
      for (int s = 0; s < NS; s++) a[u][s] = fabs(a[u][s]);
    } else if (apart) {
#pragma unroll
      for (int s = 0; s < NS; s++) rs += fabs(a[u][s]);
    }
    acc = O::mma(acc, a[u], b[u]);
    const int tile = kind == 0 ? rtile[e] : -1;
    if (kind == 0 && tcol[tile] == m) {
      // diagonal tile: only its lower triangle is stored; add the strict
      // lower part transposed (A(r, k) = L(k, r), zero on the diagonal)
      double at[NS];
      O::load_a(at, orig + (int64_t)tile * TT, true, wave, lane);
#pragma unroll
      for (int s = 0; s < NS; s++) {
        const double v = O::k_of(s, g) == r ? 0.0 : at[s];
        at[s] = absmode ? fabs(v) : v;
        if (apart && !absmode) rs += fabs(v);
      }
      acc = O::mma(acc, at, b[u]);
    }
  };
  if (lo < hi) load(0, lo);
  for (int e = lo; e < hi; e += 2) {
    if (e + 1 < hi) load(1, e + 1);
    use(0, e);
    if (e + 1 < hi) {
      if (e + 2 < hi) load(0, e + 2);
      use(1, e + 1);
    }
  }
  double* out = part + (int64_t)q * vb;
  if (col < ncol) {
    v2d* o = reinterpret_cast<v2d*>(out + O::elem(wave, lane, T));
    o[0] = v2d{acc[0], acc[1]};
    o[1] = v2d{acc[2], acc[3]};
  }
  if (apart) {
    // the four lanes of a row (k groups g = 0..3) hold its whole sum
    rs += __shfl_xor(rs, 16, 64);
    rs += __shfl_xor(rs, 32, 64);
    if (g == 0) apart[(int64_t)q * T + r] = rs;
  }
}

__global__ void residual_combine_kernel(int T, const int32_t* __restrict__ item_ptr, const double* __restrict__ part,
                                        const double* __restrict__ B, double* R, int nrhs, int absmode,
                                        const double* __restrict__ apart, double* D) {
  const int m = blockIdx.x;
  const int64_t vb = (int64_t)T * nrhs;
  const int ncol = absmode ? 1 : nrhs;
  for (int e = threadIdx.x; e < T * ncol; e += blockDim.x) {
    double s = 0.0;
    for (int q = item_ptr[m]; q < item_ptr[m + 1]; q++) s += part[(int64_t)q * vb + e];
    R[m * vb + e] = absmode ? s : B[m * vb + e] - s;
  }
  if (apart) {
    for (int e = threadIdx.x; e < T; e += blockDim.x) {
      double s = 0.0;
      for (int q = item_ptr[m]; q < item_ptr[m + 1]; q++) s += apart[(int64_t)q * T + e];
      D[(int64_t)m * T + e] = s;
    }
  }
}

hipError_t launch_residual(int T, const double* orig, const int32_t* rtile, const int32_t* tcol,
                           const int32_t* ccol_tile, const int32_t* ccol_row, const int32_t* items, int32_t nitems,
                           const int32_t* item_ptr, int32_t ntr, const double* X, const double* B, double* part,
                           double* R, int nrhs, int absmode, hipStream_t st, double* apart, double* D) {
  if (absmode) apart = nullptr;
  if (nitems > 0) {
    if (T == 64)
      hipLaunchKernelGGL(residual_mma_kernel<64>, dim3(nitems), dim3(NT), 0, st, orig, rtile, tcol, ccol_tile, ccol_row,
                         items, X, part, apart, nrhs, absmode);
    else
      hipLaunchKernelGGL(residual_mma_kernel<32>, dim3(nitems), dim3(NT), 0, st, orig, rtile, tcol, ccol_tile, ccol_row,
                         items, X, part, apart, nrhs, absmode);
  }
  hipLaunchKernelGGL(residual_combine_kernel, dim3(ntr), dim3(NT), 0, st, T, item_ptr, part, B, R, nrhs, absmode,
                     apart, D);
  return hipGetLastError();
}

// ------------------------------------------------ out-of-core factorization
// S = Lc Lc^T (lower part, c x c, row-major) for the dense lower-triangular
// trailing block Lc of a factor stored in row-profile order: Lc(i, t) =
// L[rp[r0 + i] + (c0 + t - f[r0 + i])], t <= i.  16 x 16 tiles of S per
// workgroup, 64 columns of both row panels staged in LDS per step.
__global__ __launch_bounds__(256) void gram_lower_kernel(int32_t c, const double* __restrict__ L,
                                                         const int64_t* __restrict__ rp, const int64_t* __restrict__ f,
                                                         int64_t r0, int64_t c0, double* __restrict__ S) {
  const int bi = blockIdx.y, bj = blockIdx.x;
  if (bj > bi) return;
  __shared__ double A[16][65], B[16][65];
  const int ty = threadIdx.x >> 4, tx = threadIdx.x & 15;
  const int ri = 16 * bi + ty, rj = 16 * bj + ty;   // rows staged by this thread
  const int64_t oi = ri < c ? rp[r0 + ri] + c0 - f[r0 + ri] : 0;
  const int64_t oj = rj < c ? rp[r0 + rj] + c0 - f[r0 + rj] : 0;
  const int tmax = min(c, 16 * bj + 16);            // Lc(j, t) = 0 for t > j
  double acc = 0.0;
  for (int t0 = 0; t0 < tmax; t0 += 64) {
#pragma unroll
    for (int q = tx; q < 64; q += 16) {
      const int t = t0 + q;
      A[ty][q] = (ri < c && t <= ri) ? L[oi + t] : 0.0;
      B[ty][q] = (rj < c && t <= rj) ? L[oj + t] : 0.0;
    }
    __syncthreads();
#pragma unroll 8
    for (int q = 0; q < 64; q++) acc = fma(A[ty][q], B[tx][q], acc);
    __syncthreads();
  }
  const int i = 16 * bi + ty, j = 16 * bj + tx;
  if (i < c && j <= i) S[(int64_t)i * c + j] = acc;
}

hipError_t launch_gram_lower(int32_t c, const double* L, const int64_t* rp, const int64_t* f, int64_t r0, int64_t c0,
                             double* S, hipStream_t st) {
  if (c <= 0) return hipSuccess;
  const unsigned nb = (unsigned)((c + 15) / 16);
  hipLaunchKernelGGL(gram_lower_kernel, dim3(nb, nb), dim3(256), 0, st, c, L, rp, f, r0, c0, S);
  return hipGetLastError();
}

// acc += 2 sum_r log L(r, r) over rows [r0, r1) of a factor in row-profile
// order (diagonal = last entry of a row); one workgroup, fixed summation
// order (per-thread strided sums, then a tree), so the result is
// reproducible.  NaN when a pivot is not positive.
__global__ __launch_bounds__(256) void logdet_rows_kernel(const double* __restrict__ L, const int64_t* __restrict__ rp,
                                                          int64_t r0, int64_t r1, double* acc) {
  __shared__ double red[256];
  double s = 0.0;
  for (int64_t r = r0 + threadIdx.x; r < r1; r += 256) {
    const double d = L[rp[r + 1] - 1];
    s += d > 0.0 ? 2.0 * log(d) : NAN;
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) *acc += red[0];
}

hipError_t launch_logdet_rows(const double* L, const int64_t* rp, int64_t r0, int64_t r1, double* acc, hipStream_t st) {
  hipLaunchKernelGGL(logdet_rows_kernel, dim3(1), dim3(256), 0, st, L, rp, r0, r1, acc);
  return hipGetLastError();
}

// Per-column max |R| and max |X| over the tile-row blocks (T x nrhs each).
// Block (x, c) covers 16 tile rows of column c and reduces in LDS before one
// atomic per value.  Maxima are taken on the bit patterns of |v|
// (non-negative doubles order like their bits), so a NaN propagates.
__global__ __launch_bounds__(NT) void norms_kernel(int32_t ntr, int T, int nrhs, const double* __restrict__ R,
                                                   const double* __restrict__ X, unsigned long long* stats) {
  __shared__ unsigned long long sr[NT], sx[NT];
  const int c = blockIdx.y;
  const int64_t vb = (int64_t)T * nrhs;
  const int m0 = blockIdx.x * 16;
  unsigned long long rm = 0, xm = 0;
  for (int idx = threadIdx.x; idx < 16 * T; idx += NT) {
    const int m = m0 + idx / T, r = idx % T;
    if (m < ntr) {
      const int64_t e = (int64_t)m * vb + (int64_t)c * T + r;
      const unsigned long long ur = (unsigned long long)__double_as_longlong(fabs(R[e]));
      const unsigned long long ux = (unsigned long long)__double_as_longlong(fabs(X[e]));
      rm = ur > rm ? ur : rm;
      xm = ux > xm ? ux : xm;
    }
  }
  sr[threadIdx.x] = rm;
  sx[threadIdx.x] = xm;
  __syncthreads();
  for (int o = NT / 2; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) {
      sr[threadIdx.x] = sr[threadIdx.x + o] > sr[threadIdx.x] ? sr[threadIdx.x + o] : sr[threadIdx.x];
      sx[threadIdx.x] = sx[threadIdx.x + o] > sx[threadIdx.x] ? sx[threadIdx.x + o] : sx[threadIdx.x];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    atomicMax(stats + 2 * c, sr[0]);
    atomicMax(stats + 2 * c + 1, sx[0]);
  }
}

hipError_t launch_norms(int T, int32_t ntr, int nrhs, const double* R, const double* X, unsigned long long* stats,
                        hipStream_t st) {
  if (ntr <= 0 || nrhs <= 0) return hipSuccess;
  hipLaunchKernelGGL(norms_kernel, dim3((unsigned)((ntr + 15) / 16), (unsigned)nrhs), dim3(NT), 0, st, ntr, T, nrhs, R,
                     X, stats);
  return hipGetLastError();
}

// X(:, c) += D(:, c) (assign = 0) or X(:, c) = D(:, c) (assign = 1) for the
// right-hand sides c whose bit is set in `mask`; blocks of T x nrhs, so
// element e belongs to column (e / T) mod nrhs
__global__ void colmask_kernel(int64_t n, int T, int nrhs, double* X, const double* __restrict__ D, uint32_t mask,
                               int assign) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n) return;
  const int c = (int)((e / T) % nrhs);
  if (!((mask >> c) & 1u)) return;
  X[e] = assign ? D[e] : X[e] + D[e];
}

hipError_t launch_axpy(int T, int32_t ntr, int nrhs, double* X, const double* D, uint32_t mask, hipStream_t st) {
  const int64_t n = (int64_t)T * nrhs * ntr;
  hipLaunchKernelGGL(colmask_kernel, dim3((unsigned)((n + NT - 1) / NT)), dim3(NT), 0, st, n, T, nrhs, X, D, mask, 0);
  return hipGetLastError();
}

hipError_t launch_copy_cols(int T, int32_t ntr, int nrhs, double* X, const double* P, uint32_t mask, hipStream_t st) {
  const int64_t n = (int64_t)T * nrhs * ntr;
  hipLaunchKernelGGL(colmask_kernel, dim3((unsigned)((n + NT - 1) / NT)), dim3(NT), 0, st, n, T, nrhs, X, P, mask, 1);
  return hipGetLastError();
}

}  // namespace stiles
