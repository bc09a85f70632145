// gfx950 kernels of the Slow Momentum hot path.
//
// k_local_step         Algorithm 1 lines 3-5 for all workers (Table C.1 rows SGD, Adam)
// k_outer_step         lines 6-8 + copy into every replica (+ "average" buffer strategy)
// k_local_outer_step   the last local step of an outer iteration fused with the outer step
// k_outer_big, k_local_outer_big   the same two on pieces of 49 152 to 65 536 elements
//                      (many workers)
// k_init_broadcast     Algorithm 1 "Input": x_{0,0} into x0 and every replica
// k_outer_noavg        lines 7-8 per worker, without line 6 (Section 6)
// k_mix_step        mixing step of stochastic gradient push (Algorithm C.1)
// k_local_mix_step     a local step and the mixing step that follows it, fused
// k_team_mix           both on short lists, a wave per worker
// k_team_outer         the outer step and the fused last step, in the same way
// k_local_mix_paced    the fused one on 16 384-element pieces of long lists, the chip on one
//                      worker at a time
// k_debias             de-biased parameters of stochastic gradient push (Algorithm C.1)
//
// All of them are pure streams: every byte is read once and written once, no
// element is reused, so there is no dense contraction and the matrix cores are
// not involved.  The shape that measured fastest on MI355X for this read/write
// mix:
//   * one 16-byte vector per lane and per stream -- a wavefront instruction is
//     one contiguous 1 KiB burst;
//   * small workgroups that load, compute, store and retire (no loop): their
//     stores do not hold a wave slot, reads and writes of neighbouring
//     workgroups interleave, and the set of addresses in flight is a compact
//     window that moves through memory in order;
//   * on lists past the caches fewer of them per CU than the 32 that fit: 20 (SGD with kept
//     tiles up to 4 GB: 28) in the local step (its first step under "reset": 26 with Adam, no
//     cap with SGD) and the
//     outer step without the average, 16 in the outer step and the fused last step
//     with few workers.  The kernels that copy, mix or de-bias have no cap;
//   * non-temporal loads and stores, but for what the next call can find in a cache (lists
//     that fit the last-level cache, and the kept tiles of longer ones: cache_rule);
//   * workgroup -> tile mapping that gives each XCD one contiguous range of
//     tiles (workgroups are dealt to the 8 XCDs round-robin), from its start and from its
//     end by turns;
//   * tile descriptors and pointer tables read with scalar loads: they are
//     uniform over the workgroup, so they live in SGPRs, not in LDS.
//
// Compiled with -ffp-contract=off: products and sums are rounded separately,
// in the order written here, which is the order of Table C.1 and Eq. (2)-(3).
#include "slowmo_kernels.h"

#include <cstddef>
#include <mutex>
#include <type_traits>

// Device memory of the allocation-free entry point (slowmo_debias_static): the
// table its kernel reads.  One copy per GPU, held until the process ends.  In
// host code this name is only a handle for hipGetSymbolAddress -- the address
// kernels and copies use is the one static_scratch() returns.
static __device__ __align__(256) unsigned char scratch[slowmo::kStaticScratchBytes];

namespace slowmo {

namespace {

constexpr int kMaxDevices = 64;
void *g_scratch_ptr[kMaxDevices] = {};
std::mutex g_scratch_mutex;

}  // namespace

hipError_t static_scratch(int device, void **ptr) {
  *ptr = nullptr;
  if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[device]) {
    int current = -1;
    hipError_t e = hipGetDevice(&current);
    if (e != hipSuccess) return e;
    if (current != device) return hipErrorInvalidDevice;  // each GPU has its own copy and address
    void *p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch_ptr[device] = p;
  }
  *ptr = g_scratch_ptr[device];
  return hipSuccess;
}

namespace {

constexpr int kXcd = 8;  // XCDs per MI355X; workgroups are dealt to them round-robin

typedef float V4 __attribute__((ext_vector_type(4)));
typedef uint32_t U2 __attribute__((ext_vector_type(2)));

// Pointers that were themselves loaded from memory (replica and gradient
// tables) have no known address space, and the compiler would use flat
// accesses for them.  They are global memory: say so, to get global_load /
// global_store.
#define SLOWMO_GLOBAL __attribute__((address_space(1)))
// Vectors with the alignment of their elements: one global_load_dwordx4 /
// global_store_dwordx4 takes any 4-byte aligned address (any 2-byte aligned one
// for the 8 bytes of four bf16), so tensors packed back to back run on the same
// instructions as aligned ones.
typedef float V4u __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t U2u __attribute__((ext_vector_type(2), aligned(2)));
typedef SLOWMO_GLOBAL V4u GV4;
typedef SLOWMO_GLOBAL U2u GU2;

template <typename T>
__device__ __forceinline__ SLOWMO_GLOBAL T *as_global(const void *p) {
  return (SLOWMO_GLOBAL T *)(reinterpret_cast<uintptr_t>(p));
}

template <bool NT>
__device__ __forceinline__ V4 ld4(const float *p) {
  const GV4 *q = as_global<V4u>(p);
  if constexpr (NT) return __builtin_nontemporal_load(q);
  return *q;
}
template <bool NT>
__device__ __forceinline__ void st4(float *p, V4 v) {
  GV4 *q = as_global<V4u>(p);
  if constexpr (NT) {
    __builtin_nontemporal_store(v, q);
  } else {
    *q = v;
  }
}

// Stores one vector per lane to p + e0 (p uniform over the wave, e0 the lane's
// element).  With THROUGH, and where the wave's vectors cover whole 128-byte lines,
// the store is "nt sc1" (without NT "sc1"): streaming, and written through the XCD's L2 at
// once instead of when the line is evicted (the rule that sets it: cache_rule).  Lines
// that two waves share must stay in the L2 until both halves are there (tensors
// packed back to back: 2.61 ms "nt", 3.00 ms "nt sc1").  Only the buffer form lets a
// builtin ask for it.
constexpr int kNt = 2, kSc1 = 16;   // bits of the buffer store's cache policy
template <bool NT, bool THROUGH>
__device__ __forceinline__ void st4_at(float *p, int e0, V4 v) {
  if (THROUGH && (reinterpret_cast<uintptr_t>(p) & 127) == 0) {
    typedef uint32_t U4 __attribute__((ext_vector_type(4)));
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(p, 0, 0x7ffffff0, 0x00027000);
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(U4, v), rsrc, 4 * e0, 0, kSc1 + (NT ? kNt : 0));
  } else {
    st4<NT>(p + e0, v);
  }
}

// The same for a place in a state arena, every slice of which starts at a
// multiple of 256 bytes.
template <bool NT, bool THROUGH>
__device__ __forceinline__ void st4_arena(float *p, int e0, V4 v) {
  if constexpr (THROUGH) {
    typedef uint32_t U4 __attribute__((ext_vector_type(4)));
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(p, 0, 0x7ffffff0, 0x00027000);
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(U4, v), rsrc, 4 * e0, 0, kSc1 + (NT ? kNt : 0));
  } else {
    st4<NT>(p + e0, v);
  }
}

// The lanes of a tile of n elements.  n >= 4: lane t owns the vector at element 4t;
// the last one of a ragged tile moves back to n - 4, so it takes part in the same
// instructions as the others, and loads, computes and stores the elements it shares
// with its neighbour as the neighbour does.  (A path of its own for that lane is a
// second walk for its wave, and the loads it held cost every wave registers: fused
// last step 95-131 VGPRs against 59-68 so.  20 tensors of 50 001 elements, m = 32:
// fused last step 132 -> 115 us with SGD and fp32, 179 -> 155 us with Adam and bf16
// gradients, gossip step 68 -> 51 us.)  Both lanes read before either writes because they are lanes
// of one wave: a workgroup must be a single one.  n < 4 (ONE): one element per lane.
static_assert(kLocalBlock == 64 && kOuterBlock == 64, "a tile belongs to one wave");
// (t: the lane, which is the thread except where a workgroup's waves take tiles of their
// own.)
__device__ __forceinline__ int lane_element(int n, int t) { return 4 * t < n - 4 ? 4 * t : n - 4; }
__device__ __forceinline__ int lane_element(int n) {
  return lane_element(n, static_cast<int>(threadIdx.x));
}
__device__ __forceinline__ bool lane_idle(int n, int t) { return (n >= 4 ? 4 * t : t) >= n; }
__device__ __forceinline__ bool lane_idle(int n) { return lane_idle(n, static_cast<int>(threadIdx.x)); }

template <bool ONE, bool NT>
__device__ __forceinline__ V4 ldv(const float *p) {
  if constexpr (ONE) {
    const float f = *as_global<float>(p);
    return V4{f, f, f, f};
  } else {
    return ld4<NT>(p);
  }
}
template <bool ONE, bool NT>
__device__ __forceinline__ void stv(float *p, V4 v) {
  if constexpr (ONE) {
    *as_global<float>(p) = v.x;
  } else {
    st4<NT>(p, v);
  }
}

// Gradients: fp32 as is, bf16 widened exactly (the 16 bits become the high half
// of an fp32 word).  The vector (ONE: the element) at element e0 of g.
template <bool BF16, bool ONE, bool NT>
__device__ __forceinline__ V4 ldgv(const void *g, int e0) {
  if constexpr (BF16) {
    V4 r;
    if constexpr (ONE) {
      const float f =
          __uint_as_float(static_cast<uint32_t>(as_global<uint16_t>(g)[e0]) << 16);
      r = V4{f, f, f, f};
    } else {
      const GU2 *q = reinterpret_cast<const GU2 *>(as_global<uint16_t>(g) + e0);
      const U2 w = NT ? __builtin_nontemporal_load(q) : *q;
      r.x = __uint_as_float(w.x << 16);
      r.y = __uint_as_float(w.x & 0xffff0000u);
      r.z = __uint_as_float(w.y << 16);
      r.w = __uint_as_float(w.y & 0xffff0000u);
    }
    return r;
  } else {
    return ldv<ONE, NT>(static_cast<const float *>(g) + e0);
  }
}
template <bool BF16>
__device__ __forceinline__ const void *grad_at(const void *g, int64_t j) {
  return static_cast<const char *>(g) + j * (BF16 ? 2 : 4);
}

__device__ __forceinline__ int piece_of(const TileRef &t) { return t.k & ~kTileKept; }
__device__ __forceinline__ bool is_kept(const TileRef &t) { return (t.k & kTileKept) != 0; }

// Tile of workgroup b.  Workgroup b runs on XCD b mod 8; with the remap, XCD c
// walks the contiguous tile range [c * chunk, (c + 1) * chunk), so each XCD's
// L2 and TLB see one compact window of every stream instead of a 1-in-8 comb.
__device__ __forceinline__ int tile_of(int b, int chunk, int run) {
  // run == 0: workgroup b takes tile b.  run == chunk: every XCD has one
  // contiguous eighth of the tiles (the default; no division, which would be a
  // chain of some 40 instructions in front of a wave's first load).  Else, if > 0,
  // the workgroups of one XCD (b % 8) take runs of `run` consecutive tiles, the
  // 8 XCDs side by side.
  if (run == 0) return b;
  const unsigned q = static_cast<unsigned>(b) / kXcd, x = static_cast<unsigned>(b) % kXcd;
  if (run == chunk) return static_cast<int>(x * static_cast<unsigned>(chunk) + q);
  // The same eighths from their ends (run == -chunk).  Every sweep over the tiles goes the
  // other way than the one before it: what that one touched last is still in the caches.
  if (run < 0) return static_cast<int>((x + 1) * static_cast<unsigned>(chunk) - 1 - q);
  const unsigned r = static_cast<unsigned>(run);
  return static_cast<int>((q / r) * (kXcd * r) + x * r + q % r);
}

// Keep the accesses of one branch apart from those of the other: the compiler would merge
// a plain and a non-temporal load into one plain load, in front of the branch (own_path, on
// the pointer before the accesses) or behind it (own_value, on what was loaded).
template <typename P>
__device__ __forceinline__ void own_path(P &p) {
  asm volatile("" : "+s"(p));
}
__device__ __forceinline__ void own_value(V4 &v) { asm volatile("" : "+v"(v)); }

// ---- per-element arithmetic -------------------------------------------------

struct SgdP {
  float lr, mu, wd;
};
// Table C.1, SGD row, with the coupled weight-decay term.
template <bool FIRST>
__device__ __forceinline__ void sgd_elem(float &x, float &h, float g, const SgdP &p) {
  float grad = g + p.wd * x;
  float hn = FIRST ? grad : p.mu * h + grad;
  float dir = p.mu * hn + grad;
  h = hn;
  x = x - p.lr * dir;
}

struct AdamP {
  float lr, wd, b1, b2, omb1, omb2, rc1, rc2, eps;
};
// Table C.1, Adam row.  The two bias corrections are multiplications by
// reciprocals computed on the host in fp64; the root and the final quotient
// use the hardware's 1-ulp approximations, which keeps the kernel far from
// the VALU limit (an error of a few 1e-7 relative on the step, i.e. below
// 1e-9 absolute per step at the learning rates in use).
template <bool FIRST>
__device__ __forceinline__ void adam_elem(float &x, float &h, float &v, float g, const AdamP &p) {
  float grad = g + p.wd * x;
  float gsq = grad * grad;
  float hn = FIRST ? p.omb1 * grad : p.b1 * h + p.omb1 * grad;
  float vn = FIRST ? p.omb2 * gsq : p.b2 * v + p.omb2 * gsq;
  float hhat = hn * p.rc1;
  float vhat = vn * p.rc2;
  float den = __builtin_amdgcn_sqrtf(vhat) + p.eps;
  float dir = hhat * __builtin_amdgcn_rcpf(den);
  h = hn;
  v = vn;
  x = x - p.lr * dir;
}

// One base-optimizer step of four elements.
template <int BASE, bool FIRST>
__device__ __forceinline__ void step4(V4 &xv, V4 &hv, V4 &vv, V4 gv, const SgdP &sp,
                                      const AdamP &ap) {
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    float xe = xv[c], he = FIRST ? 0.f : hv[c];
    if constexpr (BASE == 0) {
      sgd_elem<FIRST>(xe, he, gv[c], sp);
    } else {
      float ve = FIRST ? 0.f : vv[c];
      adam_elem<FIRST>(xe, he, ve, gv[c], ap);
      vv[c] = ve;
    }
    xv[c] = xe;
    hv[c] = he;
  }
}

struct OuterP {
  float lr, alpha_lr, beta, m_f, alpha;
};
// gamma_t of one tensor: lr * lr_scale, and (alpha * gamma_t), each rounded once.
__device__ __forceinline__ OuterP for_tensor(OuterP p, float lr_scale) {
  p.lr = p.lr * lr_scale;
  p.alpha_lr = p.alpha * p.lr;
  return p;
}
// Algorithm 1 lines 6-8 for one element, given the ordered sum s of the
// replicas.  Returns x_{t+1,0}.
__device__ __forceinline__ float outer_elem(float s, float x0, float &u, const OuterP &p) {
  float xbar = s / p.m_f;
  float diff = x0 - xbar;
  float un = p.beta * u + diff / p.lr;
  u = un;
  return x0 - p.alpha_lr * un;
}

// The same for four elements; u is updated in place.
__device__ __forceinline__ V4 outer4(V4 s, V4 x0, V4 &u, const OuterP &p) {
  V4 xn;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    float ue = u[c];
    xn[c] = outer_elem(s[c], x0[c], ue, p);
    u[c] = ue;
  }
  return xn;
}

// Makes the (uniform) table words behind a tile arrive together: without it the
// compiler moves the loads of those that are not needed for the bounds check
// behind its branch, one more trip to the scalar cache in front of a wave's
// first vector load.
template <typename T>
__device__ __forceinline__ void have_now(const T &a) {
  asm volatile("" ::"s"(a));
}

// ---- local step ---------------------------------------------------------------
// One workgroup = one tile = up to 4 * blockDim elements of one (worker, tensor).

// One lane's vector at e0 of a tile.  FIRST: the stored buffers are to be read as
// zero (not loaded).  LAST: the buffers are dead after this step (the reset policy
// discards them before their next use), so they are not stored.  NT, THROUGH: the
// accesses to the replica and the buffers; NTG: those to the gradient.
template <int BASE, bool BF16, bool FIRST, bool LAST, bool NT, bool THROUGH, bool NTG>
__device__ __forceinline__ void local_lane(float *x, float *h, float *v, const void *g, int e0,
                                           const SgdP &sp, const AdamP &ap) {
  V4 xv = ld4<NT>(x + e0), hv, vv;
  // With only two loads per wave (buffers read as zero) the step measures 2.5 %
  // faster when the second load is issued after the first has returned
  // (2.125 -> 2.072 ms, m = 32, 25.6 M elements, four alternating runs); with
  // three or four loads the same wait changes nothing or costs 1-2 %.
  if constexpr (FIRST) asm volatile("s_waitcnt vmcnt(0)" : "+v"(xv)::"memory");
  const V4 gv = ldgv<BF16, false, NTG>(g, e0);
  if constexpr (!FIRST) hv = ld4<NT>(h + e0);
  if constexpr (!FIRST && BASE == 1) vv = ld4<NT>(v + e0);
  step4<BASE, FIRST>(xv, hv, vv, gv, sp, ap);
  st4_at<NT, THROUGH>(x, e0, xv);
  if constexpr (!LAST) st4_arena<NT, THROUGH>(h, e0, hv);
  if constexpr (!LAST && BASE == 1) st4_arena<NT, THROUGH>(v, e0, vv);
}

// Bound by memory.  What a call finds in the 256 MB last-level cache is what the call
// before left there, and non-temporal loads leave nothing: a call over a list that
// fits reads it through plain loads, and one over a longer list reads the kept tiles
// (kTileKept, see cache_rule) through plain loads and everything else past the cache,
// so that the kept lines are still there when the next call comes.  The kept tiles lie
// between the others, so that cache and memory serve the call side by side.
// ResNet-18-shaped, m = 8 (1.1 GB): 294 -> 258 us, 7.2 TB/s; 25.6 M elements, m = 1, Adam and
// bf16 gradients (358 MB) 111 -> 92 us; ResNet-50-shaped, m = 32 (9.8 GB) 2546 -> 2490 us.
template <int BASE, bool BF16, bool FIRST, bool LAST, bool NT, bool THROUGH>
__global__ __launch_bounds__(kLocalBlock) void k_local_step(
    const TileRef *__restrict__ tiles, const SlotInfo *__restrict__ slots,
    const void *const *__restrict__ gtab, float *__restrict__ hbase, float *__restrict__ vbase,
    int ntiles, int chunk, int remap, SgdP sp, AdamP ap) {
  const int tile = tile_of(blockIdx.x, chunk, remap);
  if (tile >= ntiles) return;
  const TileRef t = tiles[tile];         // uniform: scalar loads
  const SlotInfo s = slots[t.owner];
  const void *const g0 = gtab[t.owner];
  have_now(s.x), have_now(s.so), have_now(s.lr_scale), have_now(g0);
  // per-tensor hyper-parameters (uniform over the workgroup)
  sp.lr = sp.lr * s.lr_scale;
  sp.wd = s.wd;
  ap.lr = ap.lr * s.lr_scale;
  ap.wd = s.wd;
  const int64_t go = static_cast<int64_t>(piece_of(t)) * kLocalTile;  // offset in the tensor
  const void *g = grad_at<BF16>(g0, go);
  float *x = s.x + go;
  float *h = hbase + s.so + go;
  float *v = BASE == 1 ? vbase + s.so + go : nullptr;
  const int64_t left = s.numel - go;
  const int n = left < kLocalTile ? static_cast<int>(left) : kLocalTile;
  if (lane_idle(n)) return;
  if (n >= 4) {
    const int e0 = lane_element(n);
    if (NT && THROUGH && is_kept(t)) {
      own_path(x), own_path(h);
      if constexpr (BASE == 1) own_path(v);
      local_lane<BASE, BF16, FIRST, LAST, false, THROUGH, NT>(x, h, v, g, e0, sp, ap);
    } else {
      local_lane<BASE, BF16, FIRST, LAST, NT, THROUGH, NT>(x, h, v, g, e0, sp, ap);
    }
  } else {
    const int e0 = static_cast<int>(threadIdx.x);
    V4 xv = ldv<true, NT>(x + e0), hv, vv;
    if constexpr (!FIRST) hv = ldv<true, NT>(h + e0);
    if constexpr (!FIRST && BASE == 1) vv = ldv<true, NT>(v + e0);
    const V4 gv = ldgv<BF16, true, NT>(g, e0);
    step4<BASE, FIRST>(xv, hv, vv, gv, sp, ap);
    stv<true, NT>(x + e0, xv);
    if constexpr (!LAST) stv<true, NT>(h + e0, hv);
    if constexpr (!LAST && BASE == 1) stv<true, NT>(v + e0, vv);
  }
}

// ---- outer step -----------------------------------------------------------------
// One workgroup = one tile = up to 4 * blockDim elements of one tensor; a lane owns
// the same elements in all m replicas, x0 and u.

#ifndef SLOWMO_OUTER_UNROLL
#define SLOWMO_OUTER_UNROLL 8
#endif
#ifndef SLOWMO_OUTER_NTL
#define SLOWMO_OUTER_NTL 1
#endif
#ifndef SLOWMO_OUTER_NTS
#define SLOWMO_OUTER_NTS 1
#endif
#define SLOWMO_STR2(x) #x
#define SLOWMO_STR(x) SLOWMO_STR2(x)
#define SLOWMO_PRAGMA_UNROLL_OUTER _Pragma(SLOWMO_STR(unroll SLOWMO_OUTER_UNROLL))

// Buffer strategy "average" for this lane's elements of one arena (h or v):
// every worker's value becomes the ordered mean over the workers.
template <bool ONE, bool NTL, bool NTS>
__device__ __forceinline__ void average_arena(float *__restrict__ b0, int64_t stride, int m,
                                              float m_f, int e0) {
  V4 acc = ldv<ONE, NTL>(b0 + e0);
  SLOWMO_PRAGMA_UNROLL_OUTER
  for (int i = 1; i < m; ++i) acc = acc + ldv<ONE, NTL>(b0 + i * stride + e0);
  V4 mean;
#pragma unroll
  for (int c = 0; c < 4; ++c) mean[c] = acc[c] / m_f;
  SLOWMO_PRAGMA_UNROLL_OUTER
  for (int i = 0; i < m; ++i) stv<ONE, NTS>(b0 + i * stride + e0, mean);
}

// One lane's vector (ONE: element) at e0 of the tile at element eo of a tensor; xp:
// its m replicas; x0, u, h0, v0: the tile's place in the arenas.  NT: the accesses to the
// replicas and buffers (in a kept tile they are plain, as the local step's); NTO: those to
// x0 and u.
template <bool NT, bool NTO, int AVG, bool ONE>
__device__ __forceinline__ void outer_lane(float *const *__restrict__ xp, int64_t eo, float *x0,
                                           float *u, float *h0, float *v0, int64_t d_pad, int m,
                                           const OuterP &p, int e0) {
  constexpr bool NTL = NT && SLOWMO_OUTER_NTL, NTS = NT && SLOWMO_OUTER_NTS;
  // line 6: ordered sum over the replicas, i = 0, 1, ..., m-1
  V4 acc = ldv<ONE, NTL>(xp[0] + eo + e0);
  SLOWMO_PRAGMA_UNROLL_OUTER
  for (int i = 1; i < m; ++i) acc = acc + ldv<ONE, NTL>(xp[i] + eo + e0);
  const V4 x0v = ldv<ONE, NTO>(x0 + e0);
  V4 uv = ldv<ONE, NTO>(u + e0);
  const V4 xn = outer4(acc, x0v, uv, p);
  stv<ONE, NTO>(u + e0, uv);
  stv<ONE, NTO>(x0 + e0, xn);
  SLOWMO_PRAGMA_UNROLL_OUTER
  for (int i = 0; i < m; ++i) stv<ONE, NTS>(xp[i] + eo + e0, xn);
  // line 2 of the next outer iteration, strategy "average"
  if constexpr (AVG >= 1) average_arena<ONE, NTL, NTS>(h0, d_pad, m, p.m_f, e0);
  if constexpr (AVG >= 2) average_arena<ONE, NTL, NTS>(v0, d_pad, m, p.m_f, e0);
}

// AVG: 0 = lines 6-8 only; 1 = also average h over the workers; 2 = h and v.  KEPT: some
// of the tiles are kept (an instance of its own: with both walks in one the others would
// pay with registers, fused last step 64 -> 94).
template <bool NT, int AVG, bool KEPT>
__global__ __launch_bounds__(kOuterBlock) void k_outer_step(
    const TileRef *__restrict__ tiles, const TensorInfo *__restrict__ tensors,
    float *const *__restrict__ xtab_t, float *__restrict__ x0base, float *__restrict__ ubase,
    float *__restrict__ hbase, float *__restrict__ vbase, int64_t d_pad, int ntiles, int chunk,
    int remap, int m, OuterP p0) {
  const int tile = tile_of(blockIdx.x, chunk, remap);
  if (tile >= ntiles) return;
  const TileRef t = tiles[tile];         // uniform: scalar loads
  const TensorInfo ti = tensors[t.owner];
  const OuterP p = for_tensor(p0, ti.lr_scale);
  float *const *__restrict__ xp = xtab_t + static_cast<int64_t>(t.owner) * m;  // m replica pointers
  const int64_t eo = static_cast<int64_t>(piece_of(t)) * kOuterTile;  // offset of the tile in its tensor
  const int64_t left = ti.numel - eo;
  const int n = left < kOuterTile ? static_cast<int>(left) : kOuterTile;
  if (lane_idle(n)) return;
  float *x0 = x0base + ti.fo + eo, *u = ubase + ti.fo + eo;
  float *h0 = AVG >= 1 ? hbase + ti.fo + eo : nullptr, *v0 = AVG >= 2 ? vbase + ti.fo + eo : nullptr;
  if (n >= 4) {
    if (NT && KEPT && is_kept(t)) {
      own_path(xp);
      if constexpr (AVG >= 1) own_path(h0);
      if constexpr (AVG >= 2) own_path(v0);
      outer_lane<false, NT, AVG, false>(xp, eo, x0, u, h0, v0, d_pad, m, p, lane_element(n));
    } else {
      outer_lane<NT, NT, AVG, false>(xp, eo, x0, u, h0, v0, d_pad, m, p, lane_element(n));
    }
  } else {
    outer_lane<NT, NT, AVG, true>(xp, eo, x0, u, h0, v0, d_pad, m, p, static_cast<int>(threadIdx.x));
  }
}

// ---- common starting point (Algorithm 1, "Input") ------------------------------
// x_{0,0} is worker 0's replica: copy it into x0 (one copy, or one per worker
// when every worker keeps its own) and into the replicas of workers 1..m-1.
template <bool NT>
__global__ __launch_bounds__(kOuterBlock) void k_init_broadcast(
    const TileRef *__restrict__ tiles, const TensorInfo *__restrict__ tensors,
    float *const *__restrict__ xtab_t, float *__restrict__ x0base, int64_t d_pad, int x0_copies,
    int ntiles, int chunk, int remap, int m) {
  const int tile = tile_of(blockIdx.x, chunk, remap);
  if (tile >= ntiles) return;
  const TileRef t = tiles[tile];
  const TensorInfo ti = tensors[t.owner];
  const int64_t eo = static_cast<int64_t>(piece_of(t)) * kOuterTile;  // offset of the tile in its tensor
  const int64_t left = ti.numel - eo;
  const int n = left < kOuterTile ? static_cast<int>(left) : kOuterTile;
  if (lane_idle(n)) return;
  float *const *__restrict__ xp = xtab_t + static_cast<int64_t>(t.owner) * m;
  float *x0 = x0base + ti.fo + eo;
  if (n >= 4) {
    const int e0 = lane_element(n);
    const V4 v = ld4<NT>(xp[0] + eo + e0);
    for (int c = 0; c < x0_copies; ++c) st4<NT>(x0 + c * d_pad + e0, v);
#pragma unroll 8
    for (int i = 1; i < m; ++i) st4<NT>(xp[i] + eo + e0, v);
  } else {
    const int e0 = static_cast<int>(threadIdx.x);
    const V4 v = ldv<true, NT>(xp[0] + eo + e0);
    for (int c = 0; c < x0_copies; ++c) stv<true, NT>(x0 + c * d_pad + e0, v);
    for (int i = 1; i < m; ++i) stv<true, NT>(xp[i] + eo + e0, v);
  }
}

// ---- outer step without the exact average (Section 6) ---------------------------
// Same tiling as the local step: one workgroup = 256 elements of one (worker,
// tensor); 3 streams read, 3 written.  "xbar" is the worker's own replica
// (a one-term sum divided by 1, which is exact).
template <bool NT, bool THROUGH, bool KEPT>
__global__ __launch_bounds__(kLocalBlock) void k_outer_noavg(
    const TileRef *__restrict__ tiles, const SlotInfo *__restrict__ slots,
    float *__restrict__ x0base, float *__restrict__ ubase, int ntiles, int chunk, int remap,
    OuterP p0) {
  const int tile = tile_of(blockIdx.x, chunk, remap);
  if (tile >= ntiles) return;
  const TileRef t = tiles[tile];
  const SlotInfo s = slots[t.owner];
  const OuterP p = for_tensor(p0, s.lr_scale);
  const int64_t go = static_cast<int64_t>(piece_of(t)) * kLocalTile;
  float *x = s.x + go;
  float *x0 = x0base + s.so + go;
  float *u = ubase + s.so + go;
  const int64_t left = s.numel - go;
  const int n = left < kLocalTile ? static_cast<int>(left) : kLocalTile;
  if (lane_idle(n)) return;
  if (n >= 4) {
    const int e0 = lane_element(n);
    V4 xv;
    if (NT && KEPT && is_kept(t)) {
      own_path(x);
      xv = ld4<false>(x + e0);
      own_value(xv);
    } else {
      xv = ld4<NT>(x + e0);
    }
    const V4 x0v = ld4<NT>(x0 + e0);
    V4 uv = ld4<NT>(u + e0);
    const V4 xn = outer4(xv, x0v, uv, p);
    st4_arena<NT, THROUGH>(u, e0, uv);
    st4_arena<NT, THROUGH>(x0, e0, xn);
    if (NT && KEPT && is_kept(t)) {
      st4_at<false, THROUGH>(x, e0, xn);
    } else {
      st4_at<NT, THROUGH>(x, e0, xn);
    }
  } else {
    const int e0 = static_cast<int>(threadIdx.x);
    const V4 xv = ldv<true, NT>(x + e0), x0v = ldv<true, NT>(x0 + e0);
    V4 uv = ldv<true, NT>(u + e0);
    const V4 xn = outer4(xv, x0v, uv, p);
    stv<true, NT>(u + e0, uv);
    stv<true, NT>(x0 + e0, xn);
    stv<true, NT>(x + e0, xn);
  }
}

// ---- last local step + outer step without the average, fused ----------------------
// The local step's tiles, the arithmetic of both kernels; the stepped x stays in registers.  Bound by
// memory: 8 of the pair's 34 to 52 bytes per worker and element less, and a launch.  Rounds with tau = 1
// and 3, one kernel over two, SGD and Adam, both gradient types: up to 1.6 M elements of all workers
// 0.45-0.86 and 0.80-0.96, 3 to 10 M 0.60-0.89 and 0.87-0.94, 25 to 160 M 0.74-0.92 and 0.84-0.96
// (4 x 40 M, SGD, tau = 1 908 -> 730 us).  NTO: the accesses to x0 and u.
template <int BASE, bool BF16, bool FIRST, bool LAST, bool NT, bool NTO, bool THROUGH, bool NTG>
__device__ __forceinline__ void local_noavg_lane(float *x, float *h, float *v, const void *g, float *x0,
                                                 float *u, int e0, const SgdP &sp, const AdamP &ap,
                                                 const OuterP &p) {
  V4 xv = ld4<NT>(x + e0), hv, vv;
  if constexpr (!FIRST) hv = ld4<NT>(h + e0);
  if constexpr (!FIRST && BASE == 1) vv = ld4<NT>(v + e0);
  const V4 gv = ldgv<BF16, false, NTG>(g, e0);
  const V4 x0v = ld4<NTO>(x0 + e0);
  V4 uv = ld4<NTO>(u + e0);
  step4<BASE, FIRST>(xv, hv, vv, gv, sp, ap);
  const V4 xn = outer4(xv, x0v, uv, p);
  if constexpr (!LAST) st4_arena<NT, THROUGH>(h, e0, hv);
  if constexpr (!LAST && BASE == 1) st4_arena<NT, THROUGH>(v, e0, vv);
  st4_arena<NTO, THROUGH>(u, e0, uv);
  st4_arena<NTO, THROUGH>(x0, e0, xn);
  st4_at<NT, THROUGH>(x, e0, xn);
}

template <int BASE, bool BF16, bool FIRST, bool LAST, bool NT, bool NTO, bool THROUGH>
__global__ __launch_bounds__(kLocalBlock) void k_local_noavg(
    const TileRef *__restrict__ tiles, const SlotInfo *__restrict__ slots,
    const void *const *__restrict__ gtab, int ntiles, int chunk, int remap,
    float *__restrict__ hbase, float *__restrict__ vbase, float *__restrict__ x0base,
    float *__restrict__ ubase, SgdP sp, AdamP ap, OuterP p0) {
  const int tile = tile_of(blockIdx.x, chunk, remap);
  if (tile >= ntiles) return;
  const TileRef t = tiles[tile];
  const SlotInfo s = slots[t.owner];
  const void *const g0 = gtab[t.owner];
  have_now(s.x), have_now(s.so), have_now(s.lr_scale), have_now(g0);
  const OuterP p = for_tensor(p0, s.lr_scale);
  sp.lr = sp.lr * s.lr_scale;
  sp.wd = s.wd;
  ap.lr = ap.lr * s.lr_scale;
  ap.wd = s.wd;
  const int64_t go = static_cast<int64_t>(piece_of(t)) * kLocalTile;
  const void *g = grad_at<BF16>(g0, go);
  float *x = s.x + go;
  float *h = hbase + s.so + go;
  float *v = BASE == 1 ? vbase + s.so + go : nullptr;
  float *x0 = x0base + s.so + go, *u = ubase + s.so + go;
  const int64_t left = s.numel - go;
  const int n = left < kLocalTile ? static_cast<int>(left) : kLocalTile;
  if (lane_idle(n)) return;
  if (n >= 4) {
    const int e0 = lane_element(n);
    if (NT && THROUGH && is_kept(t)) {
      own_path(x), own_path(h);
      if constexpr (BASE == 1) own_path(v);
      local_noavg_lane<BASE, BF16, FIRST, LAST, false, NTO, THROUGH, NT>(x, h, v, g, x0, u, e0, sp, ap, p);
    } else {
      local_noavg_lane<BASE, BF16, FIRST, LAST, NT, NTO, THROUGH, NT>(x, h, v, g, x0, u, e0, sp, ap, p);
    }
  } else {
    const int e0 = static_cast<int>(threadIdx.x);
    V4 xv = ldv<true, NT>(x + e0), hv, vv;
    if constexpr (!FIRST) hv = ldv<true, NT>(h + e0);
    if constexpr (!FIRST && BASE == 1) vv = ldv<true, NT>(v + e0);
    const V4 gv = ldgv<BF16, true, NT>(g, e0), x0v = ldv<true, NTO>(x0 + e0);
    V4 uv = ldv<true, NTO>(u + e0);
    step4<BASE, FIRST>(xv, hv, vv, gv, sp, ap);
    const V4 xn = outer4(xv, x0v, uv, p);
    if constexpr (!LAST) stv<true, NT>(h + e0, hv);
    if constexpr (!LAST && BASE == 1) stv<true, NT>(v + e0, vv);
    stv<true, NTO>(u + e0, uv);
    stv<true, NTO>(x0 + e0, xn);
    stv<true, NT>(x + e0, xn);
  }
}

// ---- last local step + outer step, fused ---------------------------------------
// For one tile (256 elements of one tensor): for every worker in order, the
// base-optimizer step on that worker's (x, h[, v], g) -- the same arithmetic
// as k_local_step -- with the new x kept in registers and added to the ordered
// sum; then lines 6-8 and the write of x_{t+1,0} into all replicas.  The
// replicas are read once and written once (the unfused pair writes and
// re-reads them), and under "reset" / "average" the per-worker buffers of this
// step are never written.
#ifndef SLOWMO_FUSED_NTL
#define SLOWMO_FUSED_NTL 1
#endif
#ifndef SLOWMO_FUSED_UNROLL
#define SLOWMO_FUSED_UNROLL 8
#endif
// One lane's vector (ONE: element) at e0 of the tile at element eo of a tensor; xp:
// its replicas, gp: its gradients (worker i: gp[i * n_tensors]); x0, u, h0, v0:
// the tile's place in the arenas (worker i's buffers: + i * d_pad).  NT: the accesses to
// the replicas and buffers (plain in a kept tile); NTO: those to the gradients, x0 and u.
template <int BASE, bool BF16, bool FIRST, int POLICY, bool NT, bool NTO, bool ONE>
__device__ __forceinline__ void local_outer_lane(float *const *__restrict__ xp,
                                                 const void *const *__restrict__ gp, int64_t eo,
                                                 float *x0, float *u, float *h0, float *v0,
                                                 int64_t d_pad, int n_tensors, int m,
                                                 const SgdP &sp, const AdamP &ap, const OuterP &p,
                                                 int e0) {
  constexpr bool NTL = NT && SLOWMO_FUSED_NTL;
  V4 acc, acch, accv;
  // Adam with fp32 gradients and averaged buffers holds the most per worker: 8 of them
  // are 135 VGPRs, 3 waves per SIMD (lists that fit the caches, 4 workers of 1 M
  // elements: 21.7 us); 6 are 94 and 5 waves (19.2 us).
  constexpr int kUnroll =
      BASE == 1 && !BF16 && !FIRST && POLICY == 2 ? 6 : SLOWMO_FUSED_UNROLL;
#pragma unroll kUnroll
  for (int i = 0; i < m; ++i) {
    float *hi = h0 + i * d_pad + e0;
    float *vi = BASE == 1 ? v0 + i * d_pad + e0 : nullptr;
    V4 xv = ldv<ONE, NTL>(xp[i] + eo + e0), hv, vv;
    if constexpr (!FIRST) hv = ldv<ONE, NTL>(hi);
    if constexpr (!FIRST && BASE == 1) vv = ldv<ONE, NTL>(vi);
    const V4 gv =
        ldgv<BF16, ONE, NTO>(grad_at<BF16>(gp[static_cast<int64_t>(i) * n_tensors], eo), e0);
    step4<BASE, FIRST>(xv, hv, vv, gv, sp, ap);
    if constexpr (POLICY == 1) {
      stv<ONE, NT>(hi, hv);
      if constexpr (BASE == 1) stv<ONE, NT>(vi, vv);
    }
    if constexpr (POLICY == 2) {
      acch = (i == 0) ? hv : acch + hv;
      if constexpr (BASE == 1) accv = (i == 0) ? vv : accv + vv;
    }
    acc = (i == 0) ? xv : acc + xv;
  }
  const V4 x0v = ldv<ONE, NTO>(x0 + e0);
  V4 uv = ldv<ONE, NTO>(u + e0);
  const V4 xn = outer4(acc, x0v, uv, p);
  stv<ONE, NTO>(u + e0, uv);
  stv<ONE, NTO>(x0 + e0, xn);
#pragma unroll 8
  for (int i = 0; i < m; ++i) stv<ONE, NT>(xp[i] + eo + e0, xn);
  if constexpr (POLICY == 2) {
    V4 mh, mv;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      mh[c] = acch[c] / p.m_f;
      if constexpr (BASE == 1) mv[c] = accv[c] / p.m_f;
    }
#pragma unroll 8
    for (int i = 0; i < m; ++i) {
      stv<ONE, NT>(h0 + i * d_pad + e0, mh);
      if constexpr (BASE == 1) stv<ONE, NT>(v0 + i * d_pad + e0, mv);
    }
  }
}

template <int BASE, bool BF16, bool FIRST, int POLICY, bool NT, bool KEPT>
__global__ __launch_bounds__(kOuterBlock) void k_local_outer_step(
    const TileRef *__restrict__ tiles, const TensorInfo *__restrict__ tensors,
    float *const *__restrict__ xtab_t, const void *const *__restrict__ gtab,
    float *__restrict__ x0base, float *__restrict__ ubase, float *__restrict__ hbase,
    float *__restrict__ vbase, int64_t d_pad, int n_tensors, int ntiles, int chunk, int remap,
    int m, SgdP sp, AdamP ap, OuterP p0) {
  const int tile = tile_of(blockIdx.x, chunk, remap);
  if (tile >= ntiles) return;
  const TileRef t = tiles[tile];
  const TensorInfo ti = tensors[t.owner];
  const OuterP p = for_tensor(p0, ti.lr_scale);
  sp.lr = sp.lr * ti.lr_scale;
  sp.wd = ti.wd;
  ap.lr = ap.lr * ti.lr_scale;
  ap.wd = ti.wd;
  const int64_t eo = static_cast<int64_t>(piece_of(t)) * kOuterTile;  // offset of the tile in its tensor
  const int64_t left = ti.numel - eo;
  const int n = left < kOuterTile ? static_cast<int>(left) : kOuterTile;
  if (lane_idle(n)) return;
  float *const *__restrict__ xp = xtab_t + static_cast<int64_t>(t.owner) * m;
  const void *const *__restrict__ gp = gtab + t.owner;
  float *x0 = x0base + ti.fo + eo;
  float *u = ubase + ti.fo + eo;
  float *h0 = hbase + ti.fo + eo;
  float *v0 = BASE == 1 ? vbase + ti.fo + eo : nullptr;
  if (n >= 4) {
    const int e0 = lane_element(n);
    if (NT && KEPT && is_kept(t)) {
      own_path(xp), own_path(h0);
      if constexpr (BASE == 1) own_path(v0);
      local_outer_lane<BASE, BF16, FIRST, POLICY, false, NT, false>(xp, gp, eo, x0, u, h0, v0, d_pad,
                                                                    n_tensors, m, sp, ap, p, e0);
    } else {
      local_outer_lane<BASE, BF16, FIRST, POLICY, NT, NT, false>(xp, gp, eo, x0, u, h0, v0, d_pad,
                                                                 n_tensors, m, sp, ap, p, e0);
    }
  } else {
    local_outer_lane<BASE, BF16, FIRST, POLICY, NT, NT, true>(
        xp, gp, eo, x0, u, h0, v0, d_pad, n_tensors, m, sp, ap, p, static_cast<int>(threadIdx.x));
  }
}

// ---- big tiles: the two kernels above on whole pieces of 4096 VPT elements ---------
// One 1024-thread workgroup = 4096 VPT elements of one tensor, all workers;
// lane t owns the vectors [v * 4096 + 4t, + 4), v = 0..VPT-1, of every stream.  All
// 16 waves of the workgroup read 192 to 256 KiB of replica 0, then of replica 1, ...:
// measured, a memory region that is visited in pieces of this size serves the
// many-stream walk about 10 % faster than 1 KiB pieces from unrelated waves
// (m = 32).  The pieces are full, so there is no tail path.  Same arithmetic, same order of the sum, same
// results as the ordinary tiles.  Streams are addressed as a uniform base (the
// piece of vector v) plus the lane's offset, which keeps the addresses in
// scalar registers: the 128 vector registers a 1024-thread workgroup can have
// per lane hold the 16 accumulators and the operands of a few vectors.
constexpr int kBigStride = 4 * kBigBlock;  // floats between a lane's consecutive vectors

// The waves of a workgroup begin each worker together: one that runs ahead opens another
// region's pages for its 16 KiB only.  Fused last step, m = 32 2247 -> 2203 us, m = 8
// (11.7 M elements) 289 -> 280 us.
__device__ __forceinline__ void together() { __builtin_amdgcn_s_barrier(); }

template <int VPT>
__global__ __launch_bounds__(kBigBlock) void k_outer_big(
    const TileRef *__restrict__ tiles, const TensorInfo *__restrict__ tensors,
    float *const *__restrict__ xtab_t, float *__restrict__ x0base, float *__restrict__ ubase,
    int ntiles, int chunk, int remap, int m, OuterP p0) {
  const int tile = tile_of(blockIdx.x, chunk, remap);
  if (tile >= ntiles) return;
  const TileRef t = tiles[tile];
  const TensorInfo ti = tensors[t.owner];
  const OuterP p = for_tensor(p0, ti.lr_scale);
  const int64_t eo = static_cast<int64_t>(t.k) * big_tile(VPT);
  float *const *__restrict__ xp = xtab_t + static_cast<int64_t>(t.owner) * m;
  float *x0 = x0base + ti.fo + eo;
  float *u = ubase + ti.fo + eo;
  const int lane = 4 * static_cast<int>(threadIdx.x);
  constexpr int HALF = VPT / 2;
  V4 acc[VPT];
  for (int i = 0; i < m; ++i) {       // line 6: ordered sum, i = 0, 1, ..., m-1
    together();
    const float *x = xp[i] + eo;
#pragma unroll
    for (int v0 = 0; v0 < VPT; v0 += HALF) {
      V4 xv[HALF];
#pragma unroll
      for (int v = 0; v < HALF; ++v) xv[v] = ld4<true>(x + (v0 + v) * kBigStride + lane);
#pragma unroll
      for (int v = 0; v < HALF; ++v) acc[v0 + v] = (i == 0) ? xv[v] : acc[v0 + v] + xv[v];
    }
  }
#pragma unroll
  for (int v = 0; v < VPT; ++v) {
    const V4 x0v = ld4<true>(x0 + v * kBigStride + lane);
    V4 uv = ld4<true>(u + v * kBigStride + lane);
    const V4 xn = outer4(acc[v], x0v, uv, p);
    st4<true>(u + v * kBigStride + lane, uv);
    st4<true>(x0 + v * kBigStride + lane, xn);
    acc[v] = xn;
  }
  for (int i = 0; i < m; ++i) {
    float *x = xp[i] + eo;
#pragma unroll
    for (int v = 0; v < VPT; ++v) st4<true>(x + v * kBigStride + lane, acc[v]);
  }
}

// POLICY 0 (reset: the buffers of this step are not stored) or 1 (maintain).
// A worker's step runs over SUB vectors at a time: their operands are loaded,
// stepped, added to the sum and dropped before the next SUB are loaded.  No instance that the
// rules choose uses scratch memory.
template <int BASE, bool BF16, bool FIRST, int POLICY, int VPT>
__global__ __launch_bounds__(kBigBlock) void k_local_outer_big(
    const TileRef *__restrict__ tiles, const TensorInfo *__restrict__ tensors,
    float *const *__restrict__ xtab_t, const void *const *__restrict__ gtab,
    float *__restrict__ x0base, float *__restrict__ ubase, float *__restrict__ hbase,
    float *__restrict__ vbase, int64_t d_pad, int n_tensors, int ntiles, int chunk, int remap,
    int m, SgdP sp, AdamP ap, OuterP p0) {
  static_assert(POLICY == 0 || POLICY == 1, "no buffer average on big tiles");
  const int tile = tile_of(blockIdx.x, chunk, remap);
  if (tile >= ntiles) return;
  const TileRef t = tiles[tile];
  const TensorInfo ti = tensors[t.owner];
  const OuterP p = for_tensor(p0, ti.lr_scale);
  sp.lr = sp.lr * ti.lr_scale;
  sp.wd = ti.wd;
  ap.lr = ap.lr * ti.lr_scale;
  ap.wd = ti.wd;
  const int64_t eo = static_cast<int64_t>(t.k) * big_tile(VPT);
  float *const *__restrict__ xp = xtab_t + static_cast<int64_t>(t.owner) * m;
  const void *const *__restrict__ gp = gtab + t.owner;       // worker i: gp[i * n_tensors]
  float *x0 = x0base + ti.fo + eo;
  float *u = ubase + ti.fo + eo;
  float *h0 = hbase + ti.fo + eo;                              // worker i: h0 + i * d_pad
  float *v0 = BASE == 1 ? vbase + ti.fo + eo : nullptr;
  constexpr int gsize = BF16 ? 2 : 4;
  // With two narrow streams and registers to spare the compiler would issue most loads of a worker
  // first, take all 128 registers and spill up to 32 bytes per lane: it stays within SUB then.  Fused
  // last step at tau = 1, bf16 gradients: 12 vectors (8.2 and 20 M elements) SGD m = 8 144 -> 139
  // and 358 -> 347 us, m = 32 489 -> 477 and 1182 -> 1148, Adam m = 32 543 -> 517 and 1233 -> 1182
  // (3 vectors at a time; 2 are 4-9 % slower); 14 vectors (25.6 M) SGD m = 8 453 -> 428, m = 32
  // 1492 -> 1443, Adam m = 32 1528 -> 1486.
  constexpr bool APART = FIRST && BF16 && VPT < kBigVpt;
  constexpr int SUB = APART && VPT % 3 == 0 ? 3 : 2;
  const int lane = 4 * static_cast<int>(threadIdx.x);
  V4 acc[VPT];
  for (int i = 0; i < m; ++i) {
    together();
    const float *xi = xp[i] + eo;
    float *hi = h0 + i * d_pad;
    float *vi = BASE == 1 ? v0 + i * d_pad : nullptr;
    const char *gi = static_cast<const char *>(gp[static_cast<int64_t>(i) * n_tensors]) + eo * gsize;
#pragma unroll
    for (int s0 = 0; s0 < VPT; s0 += SUB) {
      V4 xv[SUB], hv[SUB], vv[SUB], gv[SUB];
      if constexpr (APART) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int v = 0; v < SUB; ++v) {
        const int off = (s0 + v) * kBigStride;
        xv[v] = ld4<true>(xi + off + lane);
        if constexpr (!FIRST) hv[v] = ld4<true>(hi + off + lane);
        if constexpr (!FIRST && BASE == 1) vv[v] = ld4<true>(vi + off + lane);
        gv[v] = ldgv<BF16, false, true>(gi + static_cast<int64_t>(off) * gsize, lane);
      }
      if constexpr (APART) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int v = 0; v < SUB; ++v) {
        step4<BASE, FIRST>(xv[v], hv[v], vv[v], gv[v], sp, ap);
        if constexpr (POLICY == 1) {
          const int off = (s0 + v) * kBigStride;
          st4<true>(hi + off + lane, hv[v]);
          if constexpr (BASE == 1) st4<true>(vi + off + lane, vv[v]);
        }
        acc[s0 + v] = (i == 0) ? xv[v] : acc[s0 + v] + xv[v];
      }
    }
  }
#pragma unroll
  for (int v = 0; v < VPT; ++v) {
    const V4 x0v = ld4<true>(x0 + v * kBigStride + lane);
    V4 uv = ld4<true>(u + v * kBigStride + lane);
    const V4 xn = outer4(acc[v], x0v, uv, p);
    st4<true>(u + v * kBigStride + lane, uv);
    st4<true>(x0 + v * kBigStride + lane, xn);
    acc[v] = xn;
  }
  for (int i = 0; i < m; ++i) {
    float *x = xp[i] + eo;
#pragma unroll
    for (int v = 0; v < VPT; ++v) st4<true>(x + v * kBigStride + lane, acc[v]);
  }
}

// ---- mixing step of stochastic gradient push (Algorithm C.1) ---------------------
// x^{(i)} <- p(i,i) x^{(i)} + p(i,j) x^{(j)}, j = in_peer(i), in place; one
// workgroup = 256 elements of one tensor, all workers.  See MixEntry, MixSend.  Every entry overwrites one worker
// with a * own + b * src, both operands being values from before the step.
// An operand that the previous entry already loaded (it is the previous
// entry's source) or that opened the current cycle is taken from a register
// instead of memory, so a replica is read once unless a sender has several
// receivers that are not neighbours in the order.  The loads of a batch of
// entries are issued together; all of them read old values, which stay in
// memory until their own entry comes, so issuing them early is safe.  Plain
// (cached) loads for the source operand measured faster than non-temporal ones.
#ifndef SLOWMO_MIX_BATCH
#define SLOWMO_MIX_BATCH 4
#endif
#ifndef SLOWMO_MIX_OWN_NT
#define SLOWMO_MIX_OWN_NT 1
#endif
#ifndef SLOWMO_MIX_SRC_NT
#define SLOWMO_MIX_SRC_NT 0
#endif
constexpr int kMixBatch = SLOWMO_MIX_BATCH;

// The saved registers of the mixing kernels: kMixSaved vectors, read and
// written with a register number 1..kMixSaved that is uniform over the
// workgroup (named members, so that they live in registers).
struct SavedRegs {
  V4 r1, r2, r3, r4;
  __device__ __forceinline__ void clear(const V4 &z) { r1 = r2 = r3 = r4 = z; }
  __device__ __forceinline__ void put(int k, const V4 &v) {
    if (k == 1) {
      r1 = v;
    } else if (k == 2) {
      r2 = v;
    } else if (k == 3) {
      r3 = v;
    } else if (k == 4) {
      r4 = v;
    }
  }
  __device__ __forceinline__ V4 get(int k, V4 v) const {   // v: the result for k == 0
    if (k == 1) {
      v = r1;
    } else if (k == 2) {
      v = r2;
    } else if (k == 3) {
      v = r3;
    } else if (k == 4) {
      v = r4;
    }
    return v;
  }
};
static_assert(kMixSaved == 4, "SavedRegs has four members");
// an entry's operand that is in a register already (not read from memory)
__device__ __forceinline__ bool mix_own_in_register(int32_t flags) {
  return (flags & kMixOwnFromS) || mix_own_saved(flags);
}
__device__ __forceinline__ bool mix_src_in_register(int32_t flags) {
  return (flags & (kMixSrcFromS | kMixSrcFromFirst)) || mix_src_saved(flags);
}

// The byte of a kernel's arguments at which the one of type T lies, each at a multiple of its alignment.
template <typename T, typename K>
struct ArgPlace;
template <typename T, typename... A>
struct ArgPlace<T, void (*)(A...)> {
  static constexpr size_t find() {
    size_t at = 0, found = ~size_t{0};
    ((at = (at + alignof(A) - 1) / alignof(A) * alignof(A), found = std::is_same_v<A, T> ? at : found,
      at += sizeof(A)),
     ...);
    return found;
  }
};

// The entries a workgroup takes.  They lie in the kernel's arguments (a MixInline behind the first
// kMixHead bytes, which are the same in all gossip kernels: check_mix_place) or, from more than
// kMixInline workers on, in a table; constant memory in both cases, so that an entry is a scalar
// load.  Blocks of one launch are dealt group after group (blockIdx.y).
// An upload of the entries in front of every launch was 2-4 us of copy and 13-18 us of gaps on
// the stream, and a wait of the host for the one four calls before.
// (the arguments' entries lie at multiples of 8 bytes only, which a scalar load does not mind)
typedef uint32_t U4 __attribute__((ext_vector_type(4), aligned(4)));
typedef const __attribute__((address_space(4))) U4 MixSendC;
typedef const __attribute__((address_space(4))) uint32_t WordC;
struct MixRange {
  MixSendC *seq;
  int len;
};
struct MixStep {
  int node, src;
  float a, b;
  int32_t flags;
};
__device__ __forceinline__ MixStep mix_entry(MixSendC *seq, int i) {
  const U4 w = seq[i];
  return {static_cast<int>(w.x & 0xffffu), static_cast<int>(w.x >> 16), __uint_as_float(w.y),
          __uint_as_float(w.z), static_cast<int32_t>(w.w)};
}
struct MixPlace {              // the part of a MixArgs that the kernels get beside the MixInline
  const MixSend *table;
  const uint32_t *groups;
  int32_t n_groups, first, len;
};
constexpr uintptr_t kMixHead = 3 * sizeof(void *) + 4 * sizeof(int);  // tiles, tensors, xtab_t, ntiles ... m
__device__ __forceinline__ MixRange mix_range(const MixPlace &p) {
  const uintptr_t args = (uintptr_t)__builtin_amdgcn_kernarg_segment_ptr() + kMixHead;
  MixSendC *seq = (MixSendC *)(p.table ? reinterpret_cast<uintptr_t>(p.table)
                                       : args + offsetof(MixInline, entry));
  if (p.n_groups == 0) return {seq + p.first, p.len};
  WordC *groups = (WordC *)(p.table ? reinterpret_cast<uintptr_t>(p.groups)
                                    : args + offsetof(MixInline, group));
  const uint32_t g = groups[blockIdx.y];
  return {seq + (g & 0xffffu), static_cast<int>(g >> 16)};
}

// One lane's vector (ONE: element) at e0 of the tile at element eo of a tensor whose
// replicas are xp.
template <bool NT, bool ONE>
__device__ __forceinline__ void mix_lane(float *const *__restrict__ xp,
                                         MixSendC *seq, int len, int64_t eo,
                                         int e0) {
  V4 S = {0.f, 0.f, 0.f, 0.f}, first = S;
  SavedRegs H;
  H.clear(S);
  for (int base = 0; base < len; base += kMixBatch) {
    V4 own[kMixBatch], sv[kMixBatch];
    float *ptr[kMixBatch];
#pragma unroll
    for (int q = 0; q < kMixBatch; ++q) {
      if (base + q < len) {
        const MixStep en = mix_entry(seq, base + q);
        ptr[q] = xp[en.node] + eo + e0;
        if (!mix_own_in_register(en.flags)) own[q] = ldv<ONE, NT && SLOWMO_MIX_OWN_NT>(ptr[q]);
        if (!(en.flags & kMixNoSrc) && !mix_src_in_register(en.flags))
          sv[q] = ldv<ONE, NT && SLOWMO_MIX_SRC_NT>(xp[en.src] + eo + e0);
      }
    }
#pragma unroll
    for (int q = 0; q < kMixBatch; ++q) {
      if (base + q < len) {
        const MixStep en = mix_entry(seq, base + q);
        const V4 o = (en.flags & kMixOwnFromS) ? S : H.get(mix_own_saved(en.flags), own[q]);
        if (en.flags & kMixSaveFirst) first = o;
        if (en.flags & kMixNoSrc) {
          stv<ONE, NT>(ptr[q], en.a * o);
        } else {
          H.put(mix_save(en.flags), S);
          if (en.flags & kMixSrcFromFirst) {
            S = first;
          } else if (!(en.flags & kMixSrcFromS)) {
            S = H.get(mix_src_saved(en.flags), sv[q]);
          }
          stv<ONE, NT>(ptr[q], en.a * o + en.b * S);
        }
      }
    }
  }
}

// Kept tiles go like the others.  Read and written as such they cost this kernel, which moves
// nothing but replicas, 1.05-1.29 times its time up to 1 GB (rounds of 4 local and 4 gossip steps,
// 2 to 32 workers, 1.00-1.10; 2 GB 0.99-1.02) and gain nothing beyond (5 to 20 GB 0.99-1.00).
template <bool NT>
__global__ __launch_bounds__(kOuterBlock) void k_mix_step(
    const TileRef *__restrict__ tiles, const TensorInfo *__restrict__ tensors,
    float *const *__restrict__ xtab_t, int ntiles, int chunk, int remap, int m, MixInline,
    MixPlace place) {
  const int tile = tile_of(blockIdx.x, chunk, remap);
  if (tile >= ntiles) return;
  const TileRef t = tiles[tile];
  const TensorInfo ti = tensors[t.owner];
  const int64_t eo = static_cast<int64_t>(piece_of(t)) * kOuterTile;  // offset of the tile in its tensor
  const int64_t left = ti.numel - eo;
  const int n = left < kOuterTile ? static_cast<int>(left) : kOuterTile;
  if (lane_idle(n)) return;
  float *const *__restrict__ xp = xtab_t + static_cast<int64_t>(t.owner) * m;
  const MixRange r = mix_range(place);
  if (n >= 4) {
    mix_lane<NT, false>(xp, r.seq, r.len, eo, lane_element(n));
  } else {
    mix_lane<NT, true>(xp, r.seq, r.len, eo, static_cast<int>(threadIdx.x));
  }
}

// ---- local step + mixing step, fused ---------------------------------------------
// Stochastic gradient push as base optimizer runs a mixing step after every
// local step (Algorithm C.1).  Done as two kernels, the replicas are written by
// the first and read again by the second.  Here one workgroup takes a tile of
// one tensor through all workers in the mixing order: a worker's base-optimizer
// step (the arithmetic of k_local_step) is computed when its value is first
// needed and the stepped x stays in registers for the mix, so x is read once
// and written once per step (8 bytes per worker and element less).  keep = 0: the buffers
// are dead after this step (last one before a reset) and are not stored (rounds under "reset", tau = 1, 2
// and 4, 3 to 300 M elements of all workers: SGD, fp32 0.81-0.85, 0.89-0.93, 0.94-0.96 of the time; Adam,
// bf16 0.69-0.77, 0.82-0.88, 0.91-0.95).  A worker
// whose stepped value is needed as a source before its own turn, and is not
// the next in the order, is stepped again from memory at its own turn: its x,
// h and v in memory stay untouched until then.
template <int BASE, bool BF16, bool FIRST, bool NT, bool NTG, bool ONE>
__device__ __forceinline__ void step_from_memory(const float *xi, const float *hi, const float *vi,
                                                 const void *gi, int e0, const SgdP &sp,
                                                 const AdamP &ap, V4 &xv, V4 &hv, V4 &vv) {
  xv = ldv<ONE, NT>(xi + e0);
  if constexpr (!FIRST) hv = ldv<ONE, NT>(hi + e0);
  if constexpr (!FIRST && BASE == 1) vv = ldv<ONE, NT>(vi + e0);
  const V4 gv = ldgv<BF16, ONE, NTG>(gi, e0);
  step4<BASE, FIRST>(xv, hv, vv, gv, sp, ap);
}

// One lane's vector (ONE: element) at e0 of a tile; pointers as in local_outer_lane.  NT:
// the accesses to the replicas and buffers (plain in a kept tile); NTG: the gradients'.
template <int BASE, bool BF16, bool FIRST, bool NT, bool NTG, bool ONE>
__device__ __forceinline__ void local_mix_lane(float *const *__restrict__ xp,
                                               const void *const *__restrict__ gp, int64_t eo,
                                               float *h0, float *v0, int64_t d_pad, int n_tensors,
                                               MixSendC *seq, int len, bool keep, const SgdP &sp,
                                               const AdamP &ap, int e0) {
  V4 Sx = {0.f, 0.f, 0.f, 0.f}, Sh = Sx, Sv = Sx, first = Sx;
  SavedRegs Hx, Hh, Hv;           // saved stepped workers: new x, h and v
  Hx.clear(Sx);
  Hh.clear(Sx);
  Hv.clear(Sx);
#pragma unroll 1
  for (int i = 0; i < len; ++i) {
    const MixStep en = mix_entry(seq, i);
    float *xi = xp[en.node] + eo;
    float *hi = h0 + en.node * d_pad;
    float *vi = BASE == 1 ? v0 + en.node * d_pad : nullptr;
    V4 xo, ho, vo;
    if (mix_own_in_register(en.flags)) {       // in a saved register, else held in S
      xo = Hx.get(mix_own_saved(en.flags), Sx);
      ho = Hh.get(mix_own_saved(en.flags), Sh);
      vo = Hv.get(mix_own_saved(en.flags), Sv);
    } else {
      const void *gi = grad_at<BF16>(gp[static_cast<int64_t>(en.node) * n_tensors], eo);
      step_from_memory<BASE, BF16, FIRST, NT, NTG, ONE>(xi, hi, vi, gi, e0, sp, ap, xo, ho, vo);
    }
    if (keep) {
      stv<ONE, NT>(hi + e0, ho);
      if constexpr (BASE == 1) stv<ONE, NT>(vi + e0, vo);
    }
    if (en.flags & kMixSaveFirst) first = xo;
    if (en.flags & kMixNoSrc) {
      stv<ONE, NT>(xi + e0, en.a * xo);
    } else {
      Hx.put(mix_save(en.flags), Sx);
      Hh.put(mix_save(en.flags), Sh);
      Hv.put(mix_save(en.flags), Sv);
      if (en.flags & kMixSrcFromFirst) {
        Sx = first;
      } else if (mix_src_saved(en.flags)) {
        Sx = Hx.get(mix_src_saved(en.flags), Sx);
        Sh = Hh.get(mix_src_saved(en.flags), Sh);
        Sv = Hv.get(mix_src_saved(en.flags), Sv);
      } else if (!(en.flags & kMixSrcFromS)) {
        const void *gs = grad_at<BF16>(gp[static_cast<int64_t>(en.src) * n_tensors], eo);
        step_from_memory<BASE, BF16, FIRST, NT, NTG, ONE>(
            xp[en.src] + eo, h0 + en.src * d_pad, BASE == 1 ? v0 + en.src * d_pad : nullptr, gs,
            e0, sp, ap, Sx, Sh, Sv);
      }
      stv<ONE, NT>(xi + e0, en.a * xo + en.b * Sx);
    }
  }
}

template <int BASE, bool BF16, bool FIRST, bool NT, bool KEPT>
__global__ __launch_bounds__(kOuterBlock) void k_local_mix_step(
    const TileRef *__restrict__ tiles, const TensorInfo *__restrict__ tensors,
    float *const *__restrict__ xtab_t, int ntiles, int chunk, int remap, int m, MixInline,
    MixPlace place, const void *const *__restrict__ gtab, float *__restrict__ hbase,
    float *__restrict__ vbase, int64_t d_pad, int n_tensors, int keep, SgdP sp, AdamP ap) {
  const int tile = tile_of(blockIdx.x, chunk, remap);
  if (tile >= ntiles) return;
  const TileRef t = tiles[tile];
  const TensorInfo ti = tensors[t.owner];
  sp.lr = sp.lr * ti.lr_scale;
  sp.wd = ti.wd;
  ap.lr = ap.lr * ti.lr_scale;
  ap.wd = ti.wd;
  const int64_t eo = static_cast<int64_t>(piece_of(t)) * kOuterTile;  // offset of the tile in its tensor
  const int64_t left = ti.numel - eo;
  const int n = left < kOuterTile ? static_cast<int>(left) : kOuterTile;
  if (lane_idle(n)) return;
  float *const *__restrict__ xp = xtab_t + static_cast<int64_t>(t.owner) * m;
  const void *const *__restrict__ gp = gtab + t.owner;       // worker i: gp[i * n_tensors]
  float *h0 = hbase + ti.fo + eo;                              // worker i: h0 + i * d_pad
  float *v0 = BASE == 1 ? vbase + ti.fo + eo : nullptr;
  const MixRange r = mix_range(place);
  if (n >= 4) {
    const int e0 = lane_element(n);
    if (NT && KEPT && is_kept(t)) {
      own_path(xp), own_path(h0);
      if constexpr (BASE == 1) own_path(v0);
      local_mix_lane<BASE, BF16, FIRST, false, NT, false>(xp, gp, eo, h0, v0, d_pad, n_tensors, r.seq,
                                                          r.len, keep, sp, ap, e0);
    } else {
      local_mix_lane<BASE, BF16, FIRST, NT, NT, false>(xp, gp, eo, h0, v0, d_pad, n_tensors, r.seq,
                                                       r.len, keep, sp, ap, e0);
    }
  } else {
    local_mix_lane<BASE, BF16, FIRST, NT, NT, true>(xp, gp, eo, h0, v0, d_pad, n_tensors, r.seq, r.len,
                                                    keep, sp, ap, static_cast<int>(threadIdx.x));
  }
}

// ---- teams: a wave per worker -----------------------------------------------------
// A wave that walks all workers of a tile waits for its loads worker after worker, about 1 us
// each, and a short list has no other waves to fill the time.  A team is one workgroup with a
// wave for every worker of the tile (R of them per wave from 17 on): all loads are in flight
// at once, and the stepped replicas meet in LDS.  Fused gossip step, SGD, cycle of 8 workers
// 256 tiles 8.6 -> 3.5 us, 1024 tiles 11.7 -> 7.3; 32 workers 33 -> 7.7 and 43 -> 24.5 us.
constexpr int kTeamWaves = 16;
// (wave number and lane of a thread; uniform over the wave)
__device__ __forceinline__ int team_wave() {
  return __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / 64);
}
__device__ __forceinline__ int team_lane() { return static_cast<int>(threadIdx.x) % 64; }

// Gossip step in place; BASE 2: by itself, else after the local step.  Everything is read before
// the barrier and the replicas are written behind it, so any order would do.
template <int BASE, bool BF16, bool FIRST, bool NT, int R, bool ONE>
__device__ __forceinline__ void team_mix_lane(V4 (*shared)[64], float *const *__restrict__ xp,
                                              const void *const *__restrict__ gp, int64_t eo,
                                              float *h0, float *v0, int64_t d_pad, int n_tensors,
                                              MixSendC *seq, int len, int waves, bool keep,
                                              const SgdP &sp, const AdamP &ap, bool on, int e0) {
  const int wave = team_wave(), t64 = team_lane();
  V4 x[R], h[R], v[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int k = wave + r * waves;
    if (k < len && on) {
      const MixStep en = mix_entry(seq, k);
      const float *xi = xp[en.node] + eo;
      if constexpr (BASE == 2) {
        x[r] = ldv<ONE, NT>(xi + e0);
      } else {
        float *hi = h0 + en.node * d_pad, *vi = BASE == 1 ? v0 + en.node * d_pad : nullptr;
        const void *gi = grad_at<BF16>(gp[static_cast<int64_t>(en.node) * n_tensors], eo);
        step_from_memory<BASE, BF16, FIRST, NT, NT, ONE>(xi, hi, vi, gi, e0, sp, ap, x[r], h[r], v[r]);
        if (keep) {
          stv<ONE, NT>(hi + e0, h[r]);
          if constexpr (BASE == 1) stv<ONE, NT>(vi + e0, v[r]);
        }
      }
      shared[k][t64] = x[r];
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int k = wave + r * waves;
    if (k < len && on) {
      const MixStep en = mix_entry(seq, k);
      V4 mixed = en.a * x[r];
      if (!(en.flags & kMixNoSrc)) mixed = mixed + en.b * shared[en.src][t64];
      stv<ONE, NT>(xp[en.node] + eo + e0, mixed);
    }
  }
}

template <int BASE, bool BF16, bool FIRST, bool NT, int R>
__global__ __launch_bounds__(64 * kTeamWaves) void k_team_mix(
    const TileRef *__restrict__ tiles, const TensorInfo *__restrict__ tensors,
    float *const *__restrict__ xtab_t, int ntiles, int chunk, int remap, int m, MixInline,
    MixPlace place, const void *const *__restrict__ gtab, float *__restrict__ hbase,
    float *__restrict__ vbase, int64_t d_pad, int n_tensors, int keep, SgdP sp, AdamP ap) {
  extern __shared__ V4 team_rows[];      // one row of 64 vectors per worker of the team
  V4 (*const shared)[64] = reinterpret_cast<V4 (*)[64]>(team_rows);
  const int tile = tile_of(blockIdx.x, chunk, remap);
  if (tile >= ntiles) return;
  const TileRef t = tiles[tile];
  const TensorInfo ti = tensors[t.owner];
  sp.lr = sp.lr * ti.lr_scale;
  sp.wd = ti.wd;
  ap.lr = ap.lr * ti.lr_scale;
  ap.wd = ti.wd;
  const int64_t eo = static_cast<int64_t>(piece_of(t)) * kOuterTile;
  const int64_t left = ti.numel - eo;
  const int n = left < kOuterTile ? static_cast<int>(left) : kOuterTile;
  float *const *__restrict__ xp = xtab_t + static_cast<int64_t>(t.owner) * m;
  const void *const *__restrict__ gp = BASE < 2 ? gtab + t.owner : nullptr;
  float *h0 = BASE < 2 ? hbase + ti.fo + eo : nullptr;
  float *v0 = BASE == 1 ? vbase + ti.fo + eo : nullptr;
  const MixRange o = mix_range(place);
  const int waves = static_cast<int>(blockDim.x) / 64, t64 = team_lane();
  const bool on = !lane_idle(n, t64);
  if (n >= 4) {
    team_mix_lane<BASE, BF16, FIRST, NT, R, false>(shared, xp, gp, eo, h0, v0, d_pad, n_tensors, o.seq,
                                                   o.len, waves, keep, sp, ap, on, lane_element(n, t64));
  } else {
    team_mix_lane<BASE, BF16, FIRST, NT, R, true>(shared, xp, gp, eo, h0, v0, d_pad, n_tensors, o.seq,
                                                  o.len, waves, keep, sp, ap, on, t64);
  }
}

// Outer step; BASE 0, 1: after the last local step, 2: by itself, 3: by itself with averages of v
// too.  POLICY as in k_local_outer_step (by itself: 2 averages the buffers).  The ordered sums go
// element by element: thread q takes column q of the tile's 256, over the workers in LDS.  Fused
// last step under "maintain" with Adam and bf16 gradients, 256 tiles, 8 workers 5.8 -> 4.4 us, 32 workers 23.5 -> 9.6
// us; outer step with averaged h and v after a local step, 256 tiles, 16 workers 24 -> 16 us.
template <int BASE, bool BF16, bool FIRST, int POLICY, bool NT, int R, bool ONE>
__device__ __forceinline__ void team_outer_lane(
    V4 (*shared)[64], float *const *__restrict__ xp, const void *const *__restrict__ gp, int64_t eo,
    float *x0, float *u, float *h0, float *v0, int64_t d_pad, int n_tensors, int m,
    int waves, const SgdP &sp, const AdamP &ap, const OuterP &p, int n) {
  constexpr bool STEP = BASE < 2, TWO = BASE == 1 || BASE == 3;
  constexpr int kSums = POLICY != 2 ? 1 : TWO ? 3 : 2;
  const int wave = team_wave(), t64 = team_lane();
  const bool on = !lane_idle(n, t64);
  const int e0 = ONE ? t64 : lane_element(n, t64);
  // Column q of the tile: component q % 4 of lane q / 4.  Lanes at a ragged end share elements;
  // x0 and u are read before the barrier and written behind it.
  const int q0 = static_cast<int>(threadIdx.x), step = 64 * waves;
  const auto column = [&](int q, bool *used) {
    const int l = q / 4, c = q % 4;
    *used = !lane_idle(n, l) && (!ONE || c == 0);
    return ONE ? l : lane_element(n, l) + c;
  };
  float x0v[4], uv[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int q = q0 + k * step;
    bool used;
    const int e = column(q, &used);
    if (q < kOuterTile && used) {
      x0v[k] = *as_global<float>(x0 + e);
      uv[k] = *as_global<float>(u + e);
    }
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int i = wave + r * waves;
    if (i < m && on) {
      const float *xi = xp[i] + eo;
      float *hi = STEP || POLICY == 2 ? h0 + i * d_pad : nullptr;
      float *vi = TWO ? v0 + i * d_pad : nullptr;
      V4 x, h, v;
      if constexpr (STEP) {
        const void *gi = grad_at<BF16>(gp[static_cast<int64_t>(i) * n_tensors], eo);
        step_from_memory<BASE, BF16, FIRST, NT, NT, ONE>(xi, hi, vi, gi, e0, sp, ap, x, h, v);
        if constexpr (POLICY == 1) {
          stv<ONE, NT>(hi + e0, h);
          if constexpr (TWO) stv<ONE, NT>(vi + e0, v);
        }
      } else {
        x = ldv<ONE, NT>(xi + e0);
        if constexpr (POLICY == 2) h = ldv<ONE, NT>(hi + e0);
        if constexpr (POLICY == 2 && TWO) v = ldv<ONE, NT>(vi + e0);
      }
      shared[i][t64] = x;
      if constexpr (kSums >= 2) shared[m + i][t64] = h;
      if constexpr (kSums >= 3) shared[2 * m + i][t64] = v;
    }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int q = q0 + k * step;
    bool used;
    const int e = column(q, &used);
    if (q < kOuterTile && used) {
#pragma unroll
      for (int s = 0; s < kSums; ++s) {
        float *col = reinterpret_cast<float *>(shared[s * m]) + q;
        float acc = col[0];
#pragma unroll 8
        for (int i = 1; i < m; ++i) acc = acc + col[i * kOuterTile];
        // the result takes the place of worker 0's value, which nobody else reads
        if (s == 0) {
          float ue = uv[k];
          const float xn = outer_elem(acc, x0v[k], ue, p);
          *as_global<float>(u + e) = ue;
          *as_global<float>(x0 + e) = xn;
          col[0] = xn;
        } else {
          col[0] = acc / p.m_f;
        }
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int i = wave + r * waves;
    if (i < m && on) {
      stv<ONE, NT>(xp[i] + eo + e0, shared[0][t64]);
      if constexpr (kSums >= 2) stv<ONE, NT>(h0 + i * d_pad + e0, shared[m][t64]);
      if constexpr (kSums >= 3) stv<ONE, NT>(v0 + i * d_pad + e0, shared[2 * m][t64]);
    }
  }
}

template <int BASE, bool BF16, bool FIRST, int POLICY, bool NT, int R>
__global__ __launch_bounds__(64 * kTeamWaves) void k_team_outer(
    const TileRef *__restrict__ tiles, const TensorInfo *__restrict__ tensors,
    float *const *__restrict__ xtab_t, const void *const *__restrict__ gtab,
    float *__restrict__ x0base, float *__restrict__ ubase, float *__restrict__ hbase,
    float *__restrict__ vbase, int64_t d_pad, int n_tensors, int ntiles, int chunk, int remap,
    int m, SgdP sp, AdamP ap, OuterP p0) {
  extern __shared__ V4 team_rows[];      // a row of 64 vectors per worker, of x, of h and of v
  V4 (*const shared)[64] = reinterpret_cast<V4 (*)[64]>(team_rows);
  const int tile = tile_of(blockIdx.x, chunk, remap);
  if (tile >= ntiles) return;
  const TileRef t = tiles[tile];
  const TensorInfo ti = tensors[t.owner];
  const OuterP p = for_tensor(p0, ti.lr_scale);
  sp.lr = sp.lr * ti.lr_scale;
  sp.wd = ti.wd;
  ap.lr = ap.lr * ti.lr_scale;
  ap.wd = ti.wd;
  const int64_t eo = static_cast<int64_t>(piece_of(t)) * kOuterTile;
  const int64_t left = ti.numel - eo;
  const int n = left < kOuterTile ? static_cast<int>(left) : kOuterTile;
  float *const *__restrict__ xp = xtab_t + static_cast<int64_t>(t.owner) * m;
  const void *const *__restrict__ gp = BASE < 2 ? gtab + t.owner : nullptr;
  float *x0 = x0base + ti.fo + eo, *u = ubase + ti.fo + eo;
  float *h0 = BASE < 2 || POLICY == 2 ? hbase + ti.fo + eo : nullptr;
  float *v0 = BASE == 1 || BASE == 3 ? vbase + ti.fo + eo : nullptr;
  const int waves = static_cast<int>(blockDim.x) / 64;
  if (n >= 4) {
    team_outer_lane<BASE, BF16, FIRST, POLICY, NT, R, false>(shared, xp, gp, eo, x0, u, h0, v0, d_pad,
                                                             n_tensors, m, waves, sp, ap, p, n);
  } else {
    team_outer_lane<BASE, BF16, FIRST, POLICY, NT, R, true>(shared, xp, gp, eo, x0, u, h0, v0, d_pad,
                                                            n_tensors, m, waves, sp, ap, p, n);
  }
}

// ---- paced walks over all workers ------------------------------------------------
// The kernels that take a tile through all workers are bound by the memory's
// pages: their waves are spread over 2m+4 to 5m streams, each in another place,
// and the same bytes that run at 0.79 of peak when the chip is busy in a few
// compact windows run at 0.64.  A paced walk keeps those windows compact.  One
// 512-thread workgroup per CU stays for the whole launch and takes 16 384 elements
// (64 KiB of a stream, 8 vectors per lane) at a time; the workgroups of one XCD
// take neighbouring tiles, and at every worker they wait for each other, so that
// an XCD reads and writes 2 MiB of one worker's streams, then 2 MiB of the next
// worker's.  Inside a workgroup each stream is loaded in one burst, and nothing is
// stored before all its waves have their operands.  Measured on the access
// pattern of the gossip step (m = 32, 25 M elements, streams at random offsets): single
// waves 0.64, bursts alone 0.68, with the barrier inside the workgroup 0.72, paced
// 0.775 of 8 TB/s; 1024 threads or other vector counts are 0.03-0.06 lower.
//
// The pace is a matter of speed only: no result depends on it, and no wait is
// without end.  A workgroup that has waited `spins` polls (kPaceSpins, about 0.3 ms: some of
// the others are not running, another kernel has their CUs) waits no more in this
// launch.

// Counters in the workspace, zero between launches: per XCD one for arrivals and,
// 256 bytes on, one for the step everybody may begin; after the XCDs' one that
// counts the workgroups that are done.
struct Pacer {
  uint32_t *arrive, *go;
  uint32_t members, step;
  int spins;
  bool on;
  __device__ __forceinline__ Pacer(uint32_t *base, int xcd, int members_, int spins_)
      : arrive(base + xcd * kPaceStride), go(arrive + kPaceStride / 2),
        members(static_cast<uint32_t>(members_)), step(0), spins(spins_), on(true) {}
  // Called by all threads of the workgroup.
  __device__ __forceinline__ void next() {
    ++step;
    __builtin_amdgcn_s_barrier();
    if (threadIdx.x == 0) {
      const uint32_t before =
          __hip_atomic_fetch_add(arrive, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (before == step * members - 1) {
        __hip_atomic_store(go, step, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      } else if (on) {
        int polls = 0;
        while (__hip_atomic_load(go, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < step) {
          if (++polls >= spins) {
            on = false;
            break;
          }
          __builtin_amdgcn_s_sleep(8);
        }
      }
    }
    __builtin_amdgcn_s_barrier();
  }
  // The last workgroup of the launch clears the counters for the next one: by
  // then every other one has finished its last access to them.
  __device__ __forceinline__ static void leave(uint32_t *base, uint32_t workgroups) {
    if (threadIdx.x != 0) return;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    uint32_t *done = base + kXcd * kPaceStride;
    const uint32_t before =
        __hip_atomic_fetch_add(done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (before != workgroups - 1) return;
    for (int c = 0; c < 2 * kXcd; ++c)
      __hip_atomic_store(base + c * (kPaceStride / 2), 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(done, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
};

constexpr int kPV = kPacedVpt;
constexpr int kPacedStride = 4 * kPacedBlock;  // floats between a lane's consecutive vectors
struct PV {                                    // a lane's elements of one stream
  V4 v[kPV];
};
// keeps the bursts apart and in order
__device__ __forceinline__ void burst_end() { asm volatile("" ::: "memory"); }
__device__ __forceinline__ void loads_done() {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
}
__device__ __forceinline__ void paced_load(PV &r, const float *p, int lane) {
#pragma unroll
  for (int k = 0; k < kPV; ++k) r.v[k] = ld4<true>(p + k * kPacedStride + lane);
  burst_end();
}
template <bool BF16>
__device__ __forceinline__ void paced_load_grad(PV &r, const void *g, int lane) {
#pragma unroll
  for (int k = 0; k < kPV; ++k) r.v[k] = ldgv<BF16, false, true>(grad_at<BF16>(g, k * kPacedStride), lane);
  burst_end();
}
__device__ __forceinline__ void paced_store(float *p, int lane, const PV &r) {
#pragma unroll
  for (int k = 0; k < kPV; ++k) st4<true>(p + k * kPacedStride + lane, r.v[k]);
  burst_end();
}
// One worker's base-optimizer step: x, h and v come back stepped, all waves of the
// workgroup have their operands.
template <int BASE, bool BF16, bool FIRST>
__device__ __forceinline__ void paced_step(PV &x, PV &h, PV &v, const float *xi, const float *hi,
                                           const float *vi, const void *gi, int lane,
                                           const SgdP &sp, const AdamP &ap) {
  PV g;
  paced_load(x, xi, lane);
  if constexpr (!FIRST) paced_load(h, hi, lane);
  if constexpr (!FIRST && BASE == 1) paced_load(v, vi, lane);
  paced_load_grad<BF16>(g, gi, lane);
  loads_done();
#pragma unroll
  for (int k = 0; k < kPV; ++k) step4<BASE, FIRST>(x.v[k], h.v[k], v.v[k], g.v[k], sp, ap);
}

// k_local_mix_step on paced tiles.  A worker's buffers are stored as soon as its
// step is taken for good: at its own turn, or where it is stepped as a source and
// kept in a register until then (kMixSrcDone), so only x is carried from entry to
// entry: the held source in registers, the value that opened the cycle and the
// first saved value in LDS (64 KiB each), the second saved value in registers.
template <int BASE, bool BF16, bool FIRST>
__global__ __launch_bounds__(kPacedBlock) void k_local_mix_paced(
    const TileRef *__restrict__ tiles, const TensorInfo *__restrict__ tensors,
    float *const *__restrict__ xtab_t, int ntiles, int chunk, int members, int m, MixInline,
    MixPlace place, int spins, int keep, const void *const *__restrict__ gtab, float *__restrict__ hbase,
    float *__restrict__ vbase, int64_t d_pad, int n_tensors, const TileRef *__restrict__ rest,
    int nrest, uint32_t *pace, SgdP sp0, AdamP ap0) {
  static_assert(kPacedSaved == 2, "one saved value in LDS, one in registers");
  __shared__ V4 kept[2][kPV][kPacedBlock];     // [0]: opened the cycle, [1]: saved value 1
  const int xcd = static_cast<int>(blockIdx.x) % kXcd, rank = static_cast<int>(blockIdx.x) / kXcd;
  const int lane = 4 * static_cast<int>(threadIdx.x);
  const int mine = ntiles - xcd * chunk < chunk ? ntiles - xcd * chunk : chunk;  // this XCD's tiles
  Pacer pacer(pace, xcd, members, spins);
  const MixRange order = mix_range(place);
  MixSendC *const seq = order.seq;
  const int len = order.len;
  for (int at = 0; at + rank < mine; at += members) {
    const bool paced = at + members <= mine;   // the last, partly filled row of tiles runs free
    const TileRef t = tiles[xcd * chunk + at + rank];
    const TensorInfo ti = tensors[t.owner];
    SgdP sp = sp0;
    AdamP ap = ap0;
    sp.lr = sp.lr * ti.lr_scale;
    sp.wd = ti.wd;
    ap.lr = ap.lr * ti.lr_scale;
    ap.wd = ti.wd;
    const int64_t eo = static_cast<int64_t>(t.k) * kPacedTile;
    float *const *__restrict__ xp = xtab_t + static_cast<int64_t>(t.owner) * m;
    const void *const *__restrict__ gp = gtab + t.owner;     // worker i: gp[i * n_tensors]
    float *h0 = hbase + ti.fo + eo;                            // worker i: h0 + i * d_pad
    float *v0 = BASE == 1 ? vbase + ti.fo + eo : nullptr;
    PV S, saved2, x, h, v;
#pragma unroll 1
    for (int i = 0; i < len; ++i) {
      const MixStep en = mix_entry(seq, i);
      if (paced) pacer.next();
      float *xi = xp[en.node] + eo;
      PV mixed;                                // a * own, then + b * source
      if (mix_own_in_register(en.flags)) {
        const int k = mix_own_saved(en.flags);
        if (k == 1) {
#pragma unroll
          for (int q = 0; q < kPV; ++q) x.v[q] = kept[1][q][threadIdx.x];
        } else if (k == 2) {
          x = saved2;
        } else {
          x = S;
        }
      } else {
        float *hi = h0 + en.node * d_pad, *vi = BASE == 1 ? v0 + en.node * d_pad : nullptr;
        paced_step<BASE, BF16, FIRST>(
            x, h, v, xi, hi, vi, grad_at<BF16>(gp[static_cast<int64_t>(en.node) * n_tensors], eo),
            lane, sp, ap);
        if (keep) {
          paced_store(hi, lane, h);
          if constexpr (BASE == 1) paced_store(vi, lane, v);
        }
      }
      if (en.flags & kMixSaveFirst) {
#pragma unroll
        for (int q = 0; q < kPV; ++q) kept[0][q][threadIdx.x] = x.v[q];
      }
#pragma unroll
      for (int q = 0; q < kPV; ++q) mixed.v[q] = en.a * x.v[q];
      if (!(en.flags & kMixNoSrc)) {
        const int put = mix_save(en.flags);
        if (put == 1) {
#pragma unroll
          for (int q = 0; q < kPV; ++q) kept[1][q][threadIdx.x] = S.v[q];
        } else if (put == 2) {
          saved2 = S;
        }
        const int get = mix_src_saved(en.flags);
        if (en.flags & kMixSrcFromFirst) {
#pragma unroll
          for (int q = 0; q < kPV; ++q) S.v[q] = kept[0][q][threadIdx.x];
        } else if (get == 1) {
#pragma unroll
          for (int q = 0; q < kPV; ++q) S.v[q] = kept[1][q][threadIdx.x];
        } else if (get == 2) {
          S = saved2;
        } else if (!(en.flags & kMixSrcFromS)) {
          float *hs = h0 + en.src * d_pad, *vs = BASE == 1 ? v0 + en.src * d_pad : nullptr;
          paced_step<BASE, BF16, FIRST>(
              S, h, v, xp[en.src] + eo, hs, vs,
              grad_at<BF16>(gp[static_cast<int64_t>(en.src) * n_tensors], eo), lane, sp, ap);
          if (keep && (en.flags & kMixSrcDone)) {
            paced_store(hs, lane, h);
            if constexpr (BASE == 1) paced_store(vs, lane, v);
          }
        }
#pragma unroll
        for (int q = 0; q < kPV; ++q) mixed.v[q] = mixed.v[q] + en.b * S.v[q];
      }
      paced_store(xi, lane, mixed);
    }
  }
  // The ordinary tiles that the pieces leave over go, one per wave, to the workgroups that
  // have no piece in the last row (if all have one: to all), an eighth to each XCD.
  const int busy = (mine > 0 ? mine : 0) % members;  // workgroups with a piece in the last row
  if (nrest > 0 && rank >= busy) {
    const int share = (nrest + kXcd - 1) / kXcd, end = nrest < (xcd + 1) * share ? nrest : (xcd + 1) * share;
    constexpr int kWaves = kPacedBlock / 64;
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / 64);
    const int t64 = static_cast<int>(threadIdx.x) % 64;
    for (int r = xcd * share + (rank - busy) * kWaves + wave; r < end; r += (members - busy) * kWaves) {
      const TileRef t = rest[r];
      const TensorInfo ti = tensors[t.owner];
      SgdP sp = sp0;
      AdamP ap = ap0;
      sp.lr = sp.lr * ti.lr_scale;
      sp.wd = ti.wd;
      ap.lr = ap.lr * ti.lr_scale;
      ap.wd = ti.wd;
      const int64_t eo = static_cast<int64_t>(piece_of(t)) * kOuterTile;
      const int64_t left = ti.numel - eo;
      const int n = left < kOuterTile ? static_cast<int>(left) : kOuterTile;
      if (lane_idle(n, t64)) continue;
      float *const *__restrict__ xp = xtab_t + static_cast<int64_t>(t.owner) * m;
      const void *const *__restrict__ gp = gtab + t.owner;
      float *h0 = hbase + ti.fo + eo;
      float *v0 = BASE == 1 ? vbase + ti.fo + eo : nullptr;
      if (n >= 4) {
        local_mix_lane<BASE, BF16, FIRST, true, true, false>(xp, gp, eo, h0, v0, d_pad, n_tensors, seq,
                                                             len, keep, sp, ap, lane_element(n, t64));
      } else {
        local_mix_lane<BASE, BF16, FIRST, true, true, true>(xp, gp, eo, h0, v0, d_pad, n_tensors, seq,
                                                            len, keep, sp, ap, t64);
      }
    }
  }
  Pacer::leave(pace, gridDim.x);
}

// z^{(i)} = x^{(i)} / w_i (Algorithm C.1, last line), one workgroup per local tile.  NTL:
// the loads; NT: the stores.  The weights change with every gossip step and lie in the kernel's
// arguments (a DebiasWeights behind the first kDebiasHead bytes) where there are at most kMixInline of them,
// so that only new destinations are uploaded.
constexpr uintptr_t kDebiasHead = 4 * sizeof(void *) + 4 * sizeof(int);
template <bool NTL, bool NT, bool KEPT>
__global__ __launch_bounds__(kLocalBlock) void k_debias(
    const TileRef *__restrict__ tiles, const SlotInfo *__restrict__ slots,
    float *const *__restrict__ ztab, const float *__restrict__ w, int n_tensors, int ntiles,
    int chunk, int remap, DebiasWeights) {
  const int tile = tile_of(blockIdx.x, chunk, remap);
  if (tile >= ntiles) return;
  const TileRef t = tiles[tile];
  const SlotInfo s = slots[t.owner];
  WordC *weights = (WordC *)(w ? reinterpret_cast<uintptr_t>(w)
                               : (uintptr_t)__builtin_amdgcn_kernarg_segment_ptr() + kDebiasHead);
  const float wi = __uint_as_float(weights[t.owner / n_tensors]);
  const int64_t go = static_cast<int64_t>(piece_of(t)) * kLocalTile;
  const float *x = s.x + go;
  float *z = ztab[t.owner] + go;
  const int64_t left = s.numel - go;
  const int n = left < kLocalTile ? static_cast<int>(left) : kLocalTile;
  if (lane_idle(n)) return;
  if (n >= 4) {
    const int e0 = lane_element(n);
    V4 xv;
    if (NTL && KEPT && is_kept(t)) {
      own_path(x);
      xv = ld4<false>(x + e0);
      own_value(xv);
    } else {
      xv = ld4<NTL>(x + e0);
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) xv[c] = xv[c] / wi;
    st4_at<NT, NT>(z, e0, xv);
  } else {
    const int e0 = static_cast<int>(threadIdx.x);
    V4 xv = ldv<true, NTL>(x + e0);
#pragma unroll
    for (int c = 0; c < 4; ++c) xv[c] = xv[c] / wi;
    stv<true, NT>(z + e0, xv);
  }
}

struct Grid {
  int chunk;
  int run;  // tiles per XCD turn; 0 = no remap, -chunk = each XCD's eighth backward
  unsigned blocks;
};
Grid make_grid(int ntiles, const LaunchTuning &t) {
  Grid g;
  g.chunk = (ntiles + kXcd - 1) / kXcd;
  g.run = !t.xcd_remap ? 0 : (t.xcd_run > 0 && t.xcd_run < g.chunk ? t.xcd_run : g.chunk);
  if (t.backward && g.run == g.chunk) {
    g.run = -g.chunk;
    g.blocks = static_cast<unsigned>(kXcd) * static_cast<unsigned>(g.chunk);
  } else if (g.run == 0) {
    g.blocks = static_cast<unsigned>(ntiles);
  } else {
    int64_t span = static_cast<int64_t>(kXcd) * g.run;
    if ((ntiles + span - 1) / span * span > INT32_MAX) {  // keep workgroup ids within int
      g.run = g.chunk;
      span = static_cast<int64_t>(kXcd) * g.run;
    }
    g.blocks = static_cast<unsigned>((ntiles + span - 1) / span * span);
  }
  return g;
}

template <int BASE, bool BF16, bool FIRST, bool LAST>
hipError_t launch_local_t(const LocalArgs &a, const LaunchTuning &t, hipStream_t s) {
  const Grid g = make_grid(a.ntiles, t);
  // The first step's waves wait between their two loads and have one in flight at a
  // time: under the cap that is too little.  SGD with fp32 / bf16 gradients, 25.5 M
  // elements, m = 32: 2.10 / 1.95 ms with it, 1.91-2.01 / 1.79 ms without (without
  // the wait 2.03-2.08 / 1.78 ms, cap or not).  Adam stores three streams in that
  // step and likes the middle, 26 wavefronts: 2.36-2.45 ms with the cap, 2.36
  // without, 2.23-2.25 so.
  const unsigned lds = !FIRST ? t.local_lds : BASE == 1 ? t.local_lds * 3 / 4 : 0;
  const SgdP sp{a.lr, a.mu, a.wd};
  const AdamP ap{a.lr, a.wd, a.b1, a.b2, a.omb1, a.omb2, a.rc1, a.rc2, a.eps};
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(g.blocks), dim3(kLocalBlock), lds, s, a.tiles, a.slots, a.gtab,
                       a.h, a.v, a.ntiles, g.chunk, g.run, sp, ap);
  };
  if (!t.local_nt) {
    if (t.write_through) {
      launch(k_local_step<BASE, BF16, FIRST, LAST, false, true>);
    } else {
      launch(k_local_step<BASE, BF16, FIRST, LAST, false, false>);
    }
  } else if (t.write_through) {
    launch(k_local_step<BASE, BF16, FIRST, LAST, true, true>);
  } else {
    launch(k_local_step<BASE, BF16, FIRST, LAST, true, false>);
  }
  return hipGetLastError();
}

template <int BASE, bool BF16>
hipError_t launch_local_b(const LocalArgs &a, bool first, bool last, const LaunchTuning &t,
                          hipStream_t s) {
  if (first) {
    return last ? launch_local_t<BASE, BF16, true, true>(a, t, s)
                : launch_local_t<BASE, BF16, true, false>(a, t, s);
  }
  return last ? launch_local_t<BASE, BF16, false, true>(a, t, s)
              : launch_local_t<BASE, BF16, false, false>(a, t, s);
}

}  // namespace

hipError_t launch_local_step(const LocalArgs &a, int base, bool bf16, bool first, bool last,
                             const LaunchTuning &t, hipStream_t s) {
  if (a.ntiles <= 0) return hipSuccess;
  if (base == 0) {
    return bf16 ? launch_local_b<0, true>(a, first, last, t, s)
                : launch_local_b<0, false>(a, first, last, t, s);
  }
  return bf16 ? launch_local_b<1, true>(a, first, last, t, s)
              : launch_local_b<1, false>(a, first, last, t, s);
}

template <int AVG>
hipError_t launch_outer_t(const OuterArgs &a, const LaunchTuning &t, hipStream_t s) {
  const Grid g = make_grid(a.ntiles, t);
  const OuterP p{a.lr, 0.f, a.beta, a.m_f, a.alpha};
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(g.blocks), dim3(kOuterBlock), t.outer_lds, s, a.tiles, a.tensors,
                       a.xtab_t, a.x0, a.u, a.avg_h, a.avg_v, a.d_pad, a.ntiles, g.chunk, g.run, a.m, p);
  };
  if (!t.outer_nt) {
    launch(k_outer_step<false, AVG, false>);
  } else if (t.kept_outer) {
    launch(k_outer_step<true, AVG, true>);
  } else {
    launch(k_outer_step<true, AVG, false>);
  }
  return hipGetLastError();
}

hipError_t launch_outer_step(const OuterArgs &a, const LaunchTuning &t, hipStream_t s) {
  if (a.ntiles <= 0) return hipSuccess;
  if (!a.avg_h) return launch_outer_t<0>(a, t, s);
  return a.avg_v ? launch_outer_t<2>(a, t, s) : launch_outer_t<1>(a, t, s);
}

hipError_t launch_outer_big(const OuterArgs &a, const LaunchTuning &t, hipStream_t s) {
  if (a.ntiles <= 0) return hipSuccess;
  if (a.avg_h || a.avg_v || !t.nontemporal) return hipErrorInvalidValue;
  const Grid g = make_grid(a.ntiles, t);
  const OuterP p{a.lr, 0.f, a.beta, a.m_f, a.alpha};
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(g.blocks), dim3(kBigBlock), 0, s, a.tiles, a.tensors, a.xtab_t,
                       a.x0, a.u, a.ntiles, g.chunk, g.run, a.m, p);
  };
  switch (t.big_vpt) {
    case 16: launch(k_outer_big<16>); break;
    case 14: launch(k_outer_big<14>); break;
    case 12: launch(k_outer_big<12>); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

namespace {

template <int BASE, bool BF16, bool FIRST>
hipError_t launch_fused_big_t(const LocalArgs &l, const OuterArgs &o, int n_tensors, int policy,
                              const LaunchTuning &t, hipStream_t s) {
  const Grid g = make_grid(o.ntiles, t);
  const SgdP sp{l.lr, l.mu, l.wd};
  const AdamP ap{l.lr, l.wd, l.b1, l.b2, l.omb1, l.omb2, l.rc1, l.rc2, l.eps};
  const OuterP p{o.lr, 0.f, o.beta, o.m_f, o.alpha};
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(g.blocks), dim3(kBigBlock), 0, s, o.tiles, o.tensors, o.xtab_t,
                       l.gtab, o.x0, o.u, l.h, l.v, o.d_pad, n_tensors, o.ntiles, g.chunk, g.run, o.m,
                       sp, ap, p);
  };
  if (policy != 0) {
    if (t.big_vpt != kBigVpt) return hipErrorInvalidValue;
    launch(k_local_outer_big<BASE, BF16, FIRST, 1, kBigVpt>);
    return hipGetLastError();
  }
  switch (t.big_vpt) {
    case 16: launch(k_local_outer_big<BASE, BF16, FIRST, 0, 16>); break;
    case 14: launch(k_local_outer_big<BASE, BF16, FIRST, 0, 14>); break;
    case 12: launch(k_local_outer_big<BASE, BF16, FIRST, 0, 12>); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int BASE, bool BF16>
hipError_t launch_fused_big_f(const LocalArgs &l, const OuterArgs &o, int n_tensors, bool first,
                              int policy, const LaunchTuning &t, hipStream_t s) {
  return first ? launch_fused_big_t<BASE, BF16, true>(l, o, n_tensors, policy, t, s)
               : launch_fused_big_t<BASE, BF16, false>(l, o, n_tensors, policy, t, s);
}

}  // namespace

hipError_t launch_local_outer_big(const LocalArgs &l, const OuterArgs &o, int32_t n_tensors,
                                  int base, bool bf16, bool first, int policy,
                                  const LaunchTuning &t, hipStream_t s) {
  if (o.ntiles <= 0) return hipSuccess;
  if ((policy != 0 && policy != 1) || !t.nontemporal) return hipErrorInvalidValue;
  if (base == 0) {
    return bf16 ? launch_fused_big_f<0, true>(l, o, n_tensors, first, policy, t, s)
                : launch_fused_big_f<0, false>(l, o, n_tensors, first, policy, t, s);
  }
  return bf16 ? launch_fused_big_f<1, true>(l, o, n_tensors, first, policy, t, s)
              : launch_fused_big_f<1, false>(l, o, n_tensors, first, policy, t, s);
}

namespace {

template <int BASE, bool BF16, bool FIRST, int POLICY>
hipError_t launch_fused_t(const LocalArgs &l, const OuterArgs &o, int n_tensors,
                          const LaunchTuning &t, hipStream_t s) {
  const Grid g = make_grid(o.ntiles, t);
  const SgdP sp{l.lr, l.mu, l.wd};
  const AdamP ap{l.lr, l.wd, l.b1, l.b2, l.omb1, l.omb2, l.rc1, l.rc2, l.eps};
  const OuterP p{o.lr, 0.f, o.beta, o.m_f, o.alpha};
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(g.blocks), dim3(kOuterBlock), t.last_lds, s, o.tiles, o.tensors,
                       o.xtab_t, l.gtab, o.x0, o.u, l.h, l.v, o.d_pad, n_tensors, o.ntiles, g.chunk,
                       g.run, o.m, sp, ap, p);
  };
  if (!t.last_nt) {
    launch(k_local_outer_step<BASE, BF16, FIRST, POLICY, false, false>);
  } else if (t.kept_tiles > 1 || (t.kept_tiles && last_keeps(o.ntiles, POLICY == 1))) {
    launch(k_local_outer_step<BASE, BF16, FIRST, POLICY, true, true>);
  } else {
    launch(k_local_outer_step<BASE, BF16, FIRST, POLICY, true, false>);
  }
  return hipGetLastError();
}

template <int BASE, bool BF16, bool FIRST>
hipError_t launch_fused_p(const LocalArgs &l, const OuterArgs &o, int n_tensors, int policy,
                          const LaunchTuning &t, hipStream_t s) {
  switch (policy) {
    case 0: return launch_fused_t<BASE, BF16, FIRST, 0>(l, o, n_tensors, t, s);
    case 1: return launch_fused_t<BASE, BF16, FIRST, 1>(l, o, n_tensors, t, s);
    default: return launch_fused_t<BASE, BF16, FIRST, 2>(l, o, n_tensors, t, s);
  }
}

template <int BASE, bool BF16>
hipError_t launch_fused_f(const LocalArgs &l, const OuterArgs &o, int n_tensors, bool first,
                          int policy, const LaunchTuning &t, hipStream_t s) {
  return first ? launch_fused_p<BASE, BF16, true>(l, o, n_tensors, policy, t, s)
               : launch_fused_p<BASE, BF16, false>(l, o, n_tensors, policy, t, s);
}

}  // namespace

hipError_t launch_local_outer_step(const LocalArgs &l, const OuterArgs &o, int32_t n_tensors,
                                   int base, bool bf16, bool first, int policy,
                                   const LaunchTuning &t, hipStream_t s) {
  if (o.ntiles <= 0) return hipSuccess;
  if (base == 0) {
    return bf16 ? launch_fused_f<0, true>(l, o, n_tensors, first, policy, t, s)
                : launch_fused_f<0, false>(l, o, n_tensors, first, policy, t, s);
  }
  return bf16 ? launch_fused_f<1, true>(l, o, n_tensors, first, policy, t, s)
              : launch_fused_f<1, false>(l, o, n_tensors, first, policy, t, s);
}

hipError_t launch_init_broadcast(const OuterArgs &a, int32_t x0_copies, const LaunchTuning &t,
                                 hipStream_t s) {
  if (a.ntiles <= 0) return hipSuccess;
  const Grid g = make_grid(a.ntiles, t);
  if (t.nontemporal) {
    hipLaunchKernelGGL((k_init_broadcast<true>), dim3(g.blocks), dim3(kOuterBlock), 0, s, a.tiles,
                       a.tensors, a.xtab_t, a.x0, a.d_pad, x0_copies, a.ntiles, g.chunk,
                       g.run, a.m);
  } else {
    hipLaunchKernelGGL((k_init_broadcast<false>), dim3(g.blocks), dim3(kOuterBlock), 0, s, a.tiles,
                       a.tensors, a.xtab_t, a.x0, a.d_pad, x0_copies, a.ntiles, g.chunk,
                       g.run, a.m);
  }
  return hipGetLastError();
}

namespace {

MixPlace mix_place(const MixArgs &a) { return {a.table, a.groups, a.n_groups, a.first, a.len}; }
const MixInline &mix_inline(const MixArgs &a) {
  static const MixInline none{};
  return a.order ? *a.order : none;
}
// x: the blocks of one group (a multiple of the XCDs, so that every group is dealt to them
// alike), y: the groups
dim3 mix_blocks(const MixArgs &a, const Grid &g) {
  return dim3(g.blocks, static_cast<unsigned>(a.n_groups > 0 ? a.n_groups : 1));
}

template <typename K>
constexpr void check_mix_place(K) {
  static_assert(ArgPlace<MixInline, K>::find() == kMixHead, "the kernel reads its entries behind kMixHead bytes");
}

}  // namespace

hipError_t launch_mix_step(const MixArgs &a, const LaunchTuning &t, hipStream_t s) {
  if (a.ntiles <= 0 || (a.len <= 0 && a.n_groups <= 0)) return hipSuccess;
  const Grid g = make_grid(a.ntiles, t);
  auto launch = [&](auto kernel) {
    check_mix_place(kernel);
    hipLaunchKernelGGL(kernel, mix_blocks(a, g), dim3(kOuterBlock), 0, s, a.tiles, a.tensors,
                       a.xtab_t, a.ntiles, g.chunk, g.run, a.m, mix_inline(a), mix_place(a));
  };
  if (t.local_nt) {
    launch(k_mix_step<true>);
  } else {
    launch(k_mix_step<false>);
  }
  return hipGetLastError();
}

namespace {

template <int BASE, bool BF16, bool FIRST>
hipError_t launch_local_mix_t(const LocalArgs &l, const MixArgs &x, int64_t d_pad, int n_tensors,
                              const LaunchTuning &t, hipStream_t s) {
  const Grid g = make_grid(x.ntiles, t);
  const SgdP sp{l.lr, l.mu, l.wd};
  const AdamP ap{l.lr, l.wd, l.b1, l.b2, l.omb1, l.omb2, l.rc1, l.rc2, l.eps};
  auto launch = [&](auto kernel) {
    check_mix_place(kernel);
    hipLaunchKernelGGL(kernel, mix_blocks(x, g), dim3(kOuterBlock), 0, s, x.tiles, x.tensors,
                       x.xtab_t, x.ntiles, g.chunk, g.run, x.m, mix_inline(x), mix_place(x), l.gtab,
                       l.h, l.v, d_pad, n_tensors, l.keep, sp, ap);
  };
  if (!t.mix_nt) {
    launch(k_local_mix_step<BASE, BF16, FIRST, false, false>);
  } else if (t.kept_mix > 1 || (t.kept_mix && mix_keeps(x.ntiles, BASE == 1))) {
    launch(k_local_mix_step<BASE, BF16, FIRST, true, true>);
  } else {
    launch(k_local_mix_step<BASE, BF16, FIRST, true, false>);
  }
  return hipGetLastError();
}

template <int BASE, bool BF16>
hipError_t launch_local_mix_f(const LocalArgs &l, const MixArgs &x, int64_t d_pad, int n_tensors,
                              bool first, const LaunchTuning &t, hipStream_t s) {
  return first ? launch_local_mix_t<BASE, BF16, true>(l, x, d_pad, n_tensors, t, s)
               : launch_local_mix_t<BASE, BF16, false>(l, x, d_pad, n_tensors, t, s);
}

}  // namespace

hipError_t launch_local_mix_step(const LocalArgs &l, const MixArgs &x, int64_t d_pad,
                                 int32_t n_tensors, int base, bool bf16, bool first,
                                 const LaunchTuning &t, hipStream_t s) {
  if (x.ntiles <= 0 || (x.len <= 0 && x.n_groups <= 0)) return hipSuccess;
  if (base == 0) {
    return bf16 ? launch_local_mix_f<0, true>(l, x, d_pad, n_tensors, first, t, s)
                : launch_local_mix_f<0, false>(l, x, d_pad, n_tensors, first, t, s);
  }
  return bf16 ? launch_local_mix_f<1, true>(l, x, d_pad, n_tensors, first, t, s)
              : launch_local_mix_f<1, false>(l, x, d_pad, n_tensors, first, t, s);
}

namespace {

template <int BASE, bool BF16, bool FIRST>
hipError_t launch_mix_paced_t(const LocalArgs &l, const MixArgs &x, int64_t d_pad, int n_tensors,
                              const PacedArgs &p, hipStream_t s) {
  const SgdP sp{l.lr, l.mu, l.wd};
  const AdamP ap{l.lr, l.wd, l.b1, l.b2, l.omb1, l.omb2, l.rc1, l.rc2, l.eps};
  check_mix_place(&k_local_mix_paced<BASE, BF16, FIRST>);
  hipLaunchKernelGGL((k_local_mix_paced<BASE, BF16, FIRST>), dim3(kXcd * p.members),
                     dim3(kPacedBlock), 0, s, p.tiles, x.tensors, x.xtab_t, p.ntiles,
                     (p.ntiles + kXcd - 1) / kXcd, p.members, x.m, mix_inline(x), mix_place(x), p.spins,
                     l.keep, l.gtab, l.h, l.v, d_pad, n_tensors, p.rest, p.nrest, p.counters, sp, ap);
  return hipGetLastError();
}

template <int BASE, bool BF16>
hipError_t launch_mix_paced_f(const LocalArgs &l, const MixArgs &x, int64_t d_pad, int n_tensors,
                              bool first, const PacedArgs &p, hipStream_t s) {
  return first ? launch_mix_paced_t<BASE, BF16, true>(l, x, d_pad, n_tensors, p, s)
               : launch_mix_paced_t<BASE, BF16, false>(l, x, d_pad, n_tensors, p, s);
}

}  // namespace

hipError_t launch_local_mix_paced(const LocalArgs &l, const MixArgs &x, int64_t d_pad,
                                  int32_t n_tensors, int base, bool bf16, bool first,
                                  const PacedArgs &p, hipStream_t s) {
  if (p.ntiles <= 0 || x.len <= 0) return hipSuccess;
  if (base == 0) {
    return bf16 ? launch_mix_paced_f<0, true>(l, x, d_pad, n_tensors, first, p, s)
                : launch_mix_paced_f<0, false>(l, x, d_pad, n_tensors, first, p, s);
  }
  return bf16 ? launch_mix_paced_f<1, true>(l, x, d_pad, n_tensors, first, p, s)
              : launch_mix_paced_f<1, false>(l, x, d_pad, n_tensors, first, p, s);
}

namespace {

// waves of a team of n workers, R workers per wave
int team_waves(int n, int R) { return (n + R - 1) / R; }
// bytes of LDS: a row per worker (and per sum), no more, so that small teams leave room for others
unsigned team_lds(int n) { return static_cast<unsigned>(n * 64 * sizeof(V4)); }

template <int BASE, bool BF16, bool FIRST>
hipError_t launch_team_mix_t(const LocalArgs *l, const MixArgs &x, int64_t d_pad, int n_tensors,
                             const LaunchTuning &t, hipStream_t s) {
  const Grid g = make_grid(x.ntiles, t);
  const LocalArgs a = l ? *l : LocalArgs{};
  const SgdP sp{a.lr, a.mu, a.wd};
  const AdamP ap{a.lr, a.wd, a.b1, a.b2, a.omb1, a.omb2, a.rc1, a.rc2, a.eps};
  auto launch = [&](auto kernel, int R) {
    check_mix_place(kernel);
    hipLaunchKernelGGL(kernel, mix_blocks(x, g), dim3(64 * team_waves(x.team, R)), team_lds(x.team),
                       s, x.tiles, x.tensors, x.xtab_t, x.ntiles, g.chunk, g.run, x.m, mix_inline(x),
                       mix_place(x), a.gtab, a.h, a.v, d_pad, n_tensors, a.keep, sp, ap);
  };
  const bool nt = BASE == 2 ? t.local_nt : t.mix_nt;
  if (x.team <= kTeamWaves) {
    nt ? launch(k_team_mix<BASE, BF16, FIRST, true, 1>, 1)
       : launch(k_team_mix<BASE, BF16, FIRST, false, 1>, 1);
  } else {
    nt ? launch(k_team_mix<BASE, BF16, FIRST, true, 2>, 2)
       : launch(k_team_mix<BASE, BF16, FIRST, false, 2>, 2);
  }
  return hipGetLastError();
}

template <int BASE, bool BF16, bool FIRST, int POLICY>
hipError_t launch_team_outer_t(const LocalArgs *l, const OuterArgs &o, int n_tensors,
                               const LaunchTuning &t, hipStream_t s) {
  const Grid g = make_grid(o.ntiles, t);
  const LocalArgs a = l ? *l : LocalArgs{};
  const SgdP sp{a.lr, a.mu, a.wd};
  const AdamP ap{a.lr, a.wd, a.b1, a.b2, a.omb1, a.omb2, a.rc1, a.rc2, a.eps};
  const OuterP p{o.lr, 0.f, o.beta, o.m_f, o.alpha};
  float *h = BASE < 2 ? a.h : o.avg_h, *v = BASE < 2 ? a.v : o.avg_v;
  constexpr int kSums = POLICY != 2 ? 1 : BASE == 1 || BASE == 3 ? 3 : 2;
  auto launch = [&](auto kernel, int R) {
    hipLaunchKernelGGL(kernel, dim3(g.blocks), dim3(64 * team_waves(o.m, R)), team_lds(o.m * kSums), s, o.tiles, o.tensors,
                       o.xtab_t, a.gtab, o.x0, o.u, h, v, o.d_pad, n_tensors, o.ntiles, g.chunk, g.run,
                       o.m, sp, ap, p);
  };
  const bool nt = BASE < 2 ? t.last_nt : t.outer_nt;
  if (o.m <= kTeamWaves) {
    nt ? launch(k_team_outer<BASE, BF16, FIRST, POLICY, true, 1>, 1)
       : launch(k_team_outer<BASE, BF16, FIRST, POLICY, false, 1>, 1);
  } else {
    nt ? launch(k_team_outer<BASE, BF16, FIRST, POLICY, true, 2>, 2)
       : launch(k_team_outer<BASE, BF16, FIRST, POLICY, false, 2>, 2);
  }
  return hipGetLastError();
}

template <int BASE, bool BF16, bool FIRST>
hipError_t launch_team_outer_p(const LocalArgs *l, const OuterArgs &o, int n_tensors, int policy,
                               const LaunchTuning &t, hipStream_t s) {
  switch (policy) {
    case 0: return launch_team_outer_t<BASE, BF16, FIRST, 0>(l, o, n_tensors, t, s);
    case 1: return launch_team_outer_t<BASE, BF16, FIRST, 1>(l, o, n_tensors, t, s);
    default: return launch_team_outer_t<BASE, BF16, FIRST, 2>(l, o, n_tensors, t, s);
  }
}

}  // namespace

hipError_t launch_team_mix(const LocalArgs *l, const MixArgs &x, int64_t d_pad, int32_t n_tensors,
                           int base, bool bf16, bool first, const LaunchTuning &t, hipStream_t s) {
  if (x.ntiles <= 0 || x.team <= 0) return hipSuccess;
  if (x.team > kTeamMost) return hipErrorInvalidValue;
  if (!l) return launch_team_mix_t<2, false, false>(l, x, d_pad, n_tensors, t, s);
  const auto by_first = [&](auto b, auto h) {
    return first ? launch_team_mix_t<decltype(b)::value, decltype(h)::value, true>(l, x, d_pad, n_tensors, t, s)
                 : launch_team_mix_t<decltype(b)::value, decltype(h)::value, false>(l, x, d_pad, n_tensors, t, s);
  };
  using std::integral_constant;
  using std::bool_constant;
  if (base == 0)
    return bf16 ? by_first(integral_constant<int, 0>{}, bool_constant<true>{})
                : by_first(integral_constant<int, 0>{}, bool_constant<false>{});
  return bf16 ? by_first(integral_constant<int, 1>{}, bool_constant<true>{})
              : by_first(integral_constant<int, 1>{}, bool_constant<false>{});
}

hipError_t launch_team_outer(const LocalArgs *l, const OuterArgs &o, int32_t n_tensors, int base,
                             bool bf16, bool first, int policy, const LaunchTuning &t, hipStream_t s) {
  if (o.ntiles <= 0) return hipSuccess;
  if (o.m > kTeamMost) return hipErrorInvalidValue;
  if (!l) {
    if (!o.avg_h) return launch_team_outer_t<2, false, false, 0>(l, o, n_tensors, t, s);
    return o.avg_v ? launch_team_outer_t<3, false, false, 2>(l, o, n_tensors, t, s)
                   : launch_team_outer_t<2, false, false, 2>(l, o, n_tensors, t, s);
  }
  const auto by_first = [&](auto b, auto h) {
    return first ? launch_team_outer_p<decltype(b)::value, decltype(h)::value, true>(l, o, n_tensors, policy, t, s)
                 : launch_team_outer_p<decltype(b)::value, decltype(h)::value, false>(l, o, n_tensors, policy, t, s);
  };
  using std::integral_constant;
  using std::bool_constant;
  if (base == 0)
    return bf16 ? by_first(integral_constant<int, 0>{}, bool_constant<true>{})
                : by_first(integral_constant<int, 0>{}, bool_constant<false>{});
  return bf16 ? by_first(integral_constant<int, 1>{}, bool_constant<true>{})
              : by_first(integral_constant<int, 1>{}, bool_constant<false>{});
}

hipError_t launch_debias(const DebiasArgs &a, const LaunchTuning &t, hipStream_t s) {
  if (a.ntiles <= 0) return hipSuccess;
  const Grid g = make_grid(a.ntiles, t);
  auto launch = [&](auto kernel) {
    static_assert(ArgPlace<DebiasWeights, decltype(kernel)>::find() == kDebiasHead,
                  "the kernel reads its weights behind kDebiasHead bytes");
    hipLaunchKernelGGL(kernel, dim3(g.blocks), dim3(kLocalBlock), 0, s,
                       a.tiles, a.slots, a.ztab, a.w, a.n_tensors, a.ntiles, g.chunk, g.run,
                       a.inl ? *a.inl : DebiasWeights{});
  };
  if (!t.nontemporal) {
    launch(k_debias<false, false, false>);
  } else if (!t.mix_nt) {
    launch(k_debias<false, true, false>);
  } else if (t.kept_local) {
    launch(k_debias<true, true, true>);
  } else {
    launch(k_debias<true, true, false>);
  }
  return hipGetLastError();
}

namespace {

template <int BASE, bool BF16, bool FIRST, bool LAST>
hipError_t launch_local_noavg_t(const LocalArgs &a, const OuterNoAvgArgs &o, const LaunchTuning &t,
                                hipStream_t s) {
  const Grid g = make_grid(a.ntiles, t);
  const SgdP sp{a.lr, a.mu, a.wd};
  const AdamP ap{a.lr, a.wd, a.b1, a.b2, a.omb1, a.omb2, a.rc1, a.rc2, a.eps};
  const OuterP p{o.lr, 0.f, o.beta, 1.0f, o.alpha};
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(g.blocks), dim3(kLocalBlock), t.noavg_lds, s, a.tiles, a.slots,
                       a.gtab, a.ntiles, g.chunk, g.run, a.h, a.v, o.x0, o.u, sp, ap, p);
  };
  const NoAvgAccess by = noavg_access(t.local_nt, t.outer_nt, t.write_through);
  if (by.local_nt) {
    by.through ? launch(k_local_noavg<BASE, BF16, FIRST, LAST, true, true, true>)
               : launch(k_local_noavg<BASE, BF16, FIRST, LAST, true, true, false>);
  } else if (by.outer_nt) {
    by.through ? launch(k_local_noavg<BASE, BF16, FIRST, LAST, false, true, true>)
               : launch(k_local_noavg<BASE, BF16, FIRST, LAST, false, true, false>);
  } else {
    by.through ? launch(k_local_noavg<BASE, BF16, FIRST, LAST, false, false, true>)
               : launch(k_local_noavg<BASE, BF16, FIRST, LAST, false, false, false>);
  }
  return hipGetLastError();
}

template <int BASE, bool BF16>
hipError_t launch_local_noavg_b(const LocalArgs &a, const OuterNoAvgArgs &o, bool first, bool last,
                                const LaunchTuning &t, hipStream_t s) {
  if (first) {
    return last ? launch_local_noavg_t<BASE, BF16, true, true>(a, o, t, s)
                : launch_local_noavg_t<BASE, BF16, true, false>(a, o, t, s);
  }
  return last ? launch_local_noavg_t<BASE, BF16, false, true>(a, o, t, s)
              : launch_local_noavg_t<BASE, BF16, false, false>(a, o, t, s);
}

}  // namespace

hipError_t launch_local_noavg_step(const LocalArgs &a, const OuterNoAvgArgs &o, int base, bool bf16,
                                   bool first, bool last, const LaunchTuning &t, hipStream_t s) {
  if (a.ntiles <= 0) return hipSuccess;
  if (base == 0) {
    return bf16 ? launch_local_noavg_b<0, true>(a, o, first, last, t, s)
                : launch_local_noavg_b<0, false>(a, o, first, last, t, s);
  }
  return bf16 ? launch_local_noavg_b<1, true>(a, o, first, last, t, s)
              : launch_local_noavg_b<1, false>(a, o, first, last, t, s);
}

hipError_t launch_outer_noavg_step(const OuterNoAvgArgs &a, const LaunchTuning &t, hipStream_t s) {
  if (a.ntiles <= 0) return hipSuccess;
  const Grid g = make_grid(a.ntiles, t);
  const OuterP p{a.lr, 0.f, a.beta, 1.0f, a.alpha};
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(g.blocks), dim3(kLocalBlock), t.noavg_lds, s, a.tiles, a.slots,
                       a.x0, a.u, a.ntiles, g.chunk, g.run, p);
  };
  if (!t.outer_nt) {
    launch(k_outer_noavg<false, false, false>);
  } else if (!t.noavg_through) {
    launch(k_outer_noavg<true, false, false>);
  } else if (t.kept_local) {
    launch(k_outer_noavg<true, true, true>);
  } else {
    launch(k_outer_noavg<true, true, false>);
  }
  return hipGetLastError();
}

}  // namespace slowmo
