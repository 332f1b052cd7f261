// engine.hip -- GPU contraction of PACI tensor networks (Sec. III of
// arXiv:1807.02119) for CDNA4 (gfx950).
//
// One persistent kernel executes the task groups of a device program (see
// program.h).  Ready tasks sit in a device queue: a workgroup claims the next
// queue slot, waits until a task id has been written there, runs the task,
// and when it finishes the last task of a group it appends every task of the
// knot's next group to the queue.  Completion is published with a release at
// device scope and taken with an acquire before a task reads its inputs, so
// data written on one XCD is visible on another.  Every task is enqueued
// exactly once and only after its predecessors finished, so every claimed
// slot is eventually filled and the kernel drains for any grid size.
//
// Work done by tasks:
//   setup   edge weights x_e = e^{J_e} (or the Jones couplings -t^{-eps_e},
//           Sec. II), merged weights x_m = prod x_e over parallel edges, and
//           every vertex tensor F_v(s_v, s_w...) = prod_j T_{v wj}(s_v, s_wj)
//           with T = 1 + (x - 1) delta (Eqs. 3, 5); a vertex spin private to
//           its tensor is summed here.
//   step    C[b,m,n] = sum_k A[b,m,k] B[b,k,n] (one pairwise contraction of
//           Eq. 6).  Operands are gathered from where their strides put
//           them (decoded from digit strides, or from offset tables in LDS),
//           so the permutation that brings A and B into GEMM order is fused
//           into the loads and never materialised.  Tensors
//           that live inside one serial task are kept in that workgroup's LDS.
//           Each tensor is a raw mantissa array R with an int64 exponent e
//           (true = R 2^e) and a shift s = frexp exponent of max(|Re|,|Im|)
//           over R; the consumer scales by 2^-(sA+sB) while accumulating, so
//           every product stays bounded by the contracted extent and Z never
//           overflows.
//   final   Z = prod over components of (scalar R 2^e) times the
//           simplification factors (loops x_e, spikes x_m + q - 1) and q per
//           isolated spin, renormalised after every product.
#include <hip/hip_runtime.h>
#include <type_traits>

#include <climits>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <map>
#include <mutex>
#include <algorithm>
#include <new>

#include "checks.h"
#include "decode.h"
#include "internal.h"

namespace kn {

template <class T>
struct alignas(2 * sizeof(T)) Cx {
  T re, im;
};

struct DevProg {
  const ImgHeader* h;
  const TaskDesc* tasks;
  const GroupDesc* groups;
  const KnotDesc* knots;
  const TensorDesc* tens;
  const StepDesc* steps;
  const VtxDesc* vtx;
  const int32_t* vslot;
  const MEdge* medges;
  const int32_t* members;
  const Factor* factors;
  const int32_t* strides;
  const int8_t* eps;
  const int32_t* comps;
  const int32_t* pins;
  int32_t* ctrl;
  int32_t* queue;
  int32_t* pending;
  TensorState* ts;
  Cx<double>* weights;  // x_e (n_edges) then x_m (n_medges)
  Cx<double>* mgrad;    // d log Z / d J per merged edge (gradient plans)
  kn_scalar* zslice;    // result of every slice (sliced plans)
  int32_t* uslice;      // the slice each knot descriptor is running
};

__device__ inline DevProg make_prog(const uint8_t* img, uint8_t* state) {
  DevProg p;
  p.h = reinterpret_cast<const ImgHeader*>(img);
  const ImgHeader& h = *p.h;
  p.tasks = reinterpret_cast<const TaskDesc*>(img + h.o_tasks);
  p.groups = reinterpret_cast<const GroupDesc*>(img + h.o_groups);
  p.knots = reinterpret_cast<const KnotDesc*>(img + h.o_knots);
  p.tens = reinterpret_cast<const TensorDesc*>(img + h.o_tensors);
  p.steps = reinterpret_cast<const StepDesc*>(img + h.o_steps);
  p.vtx = reinterpret_cast<const VtxDesc*>(img + h.o_vtx);
  p.vslot = reinterpret_cast<const int32_t*>(img + h.o_vslot);
  p.medges = reinterpret_cast<const MEdge*>(img + h.o_medges);
  p.members = reinterpret_cast<const int32_t*>(img + h.o_members);
  p.factors = reinterpret_cast<const Factor*>(img + h.o_factors);
  p.strides = reinterpret_cast<const int32_t*>(img + h.o_strides);
  p.eps = reinterpret_cast<const int8_t*>(img + h.o_eps);
  p.comps = reinterpret_cast<const int32_t*>(img + h.o_comps);
  p.pins = reinterpret_cast<const int32_t*>(img + h.o_pins);
  p.ctrl = reinterpret_cast<int32_t*>(state);
  p.queue = reinterpret_cast<int32_t*>(state + h.o_queue);
  p.pending = reinterpret_cast<int32_t*>(state + h.o_pending);
  p.ts = reinterpret_cast<TensorState*>(state + h.o_tstate);
  p.weights = reinterpret_cast<Cx<double>*>(state + h.o_weights);
  p.mgrad = reinterpret_cast<Cx<double>*>(state + h.o_mgrad);
  p.zslice = reinterpret_cast<kn_scalar*>(state + h.o_zslice);
  p.uslice = reinterpret_cast<int32_t*>(state + h.o_uslice);
  return p;
}

// The plan constants of a knot (derived merged edges, FAC_CONST factors).
__device__ inline const Cx<double>* plan_consts(const DevProg& p, const KnotDesc& kd) {
  return reinterpret_cast<const Cx<double>*>(reinterpret_cast<const uint8_t*>(p.h) +
                                              p.h->o_consts) +
         kd.const_off;
}

__device__ inline Cx<double> cmul(Cx<double> a, Cx<double> b) {
  return {fma(a.re, b.re, -a.im * b.im), fma(a.re, b.im, a.im * b.re)};
}

// z <- z * f with z = (mantissa, exponent) renormalised to max(|re|,|im|) in [0.5, 1)
__device__ inline void acc_mul(Cx<double>& z, int64_t& e, Cx<double> f) {
  z = cmul(z, f);
  double m = fmax(fabs(z.re), fabs(z.im));
  if (m == 0.0 || !isfinite(m)) return;
  int s;
  frexp(m, &s);
  z.re = ldexp(z.re, -s);
  z.im = ldexp(z.im, -s);
  e += s;
}

__device__ inline int32_t shift_of(int32_t s) { return s == kShiftNone ? 0 : s; }

// Tensor data: the workgroup's LDS arena or the global arena (generic pointer).
template <class T>
__device__ inline Cx<T>* tptr(const TensorDesc& d, Cx<T>* arena, Cx<T>* lds) {
  return d.lds_off >= 0 ? lds + d.lds_off : arena + d.off;
}

// Operand pointers with their address space fixed at compile time: LDS
// operands are read with LDS instructions and global ones with global
// instructions.  A generic (flat) load shares the vector-memory counter with
// stores, so a flat operand load would wait for every earlier output store.
template <class T>
using LdsCx = __attribute__((address_space(3))) Cx<T>;
template <class T>
using GlbCx = __attribute__((address_space(1))) Cx<T>;

// Loads of complex entries through address-space-qualified pointers
// (member-wise, merged into one wide access by the compiler).
template <class P>
__device__ inline auto ldc(P p) {
  using T = decltype(+p->re);
  return Cx<T>{p->re, p->im};
}

// Output entries.  Tile tasks write tensor entries in global memory through the
// L2 to memory (system-scope cache policy, sc0 sc1) instead of leaving dirty
// lines there: a task that finishes then has little left to write back when
// it releases its results at device scope (the release itself is
// unchanged), which makes the per-task release noticeably cheaper.  One
// entry is one store instruction (16 bytes in complex128, 8 in complex64),
// so the lanes of a wavefront that write consecutive entries write whole
// lines.  The stores are buffer stores with the cache policy as an operand,
// through a buffer resource whose base is the start of the output range a
// workgroup or wavefront writes (uniform over the wavefront); offsets are
// byte offsets from it, below kOutRangeBytes (the planner keeps every
// range a step writes from one base below that size), and a store past the
// range is dropped by the hardware bounds check rather than written.
constexpr int32_t kOutRangeBytes = 0x7fffffff;
constexpr int32_t kRawBufferWord3 = 0x00020000;  // raw buffer, 32-bit elements
constexpr int32_t kWriteThrough = 1 | 16;        // sc0 | sc1: system scope

template <class T>
struct GlbOut {
  __amdgpu_buffer_rsrc_t r;
  __device__ explicit GlbOut(GlbCx<T>* base)
      : r(__builtin_amdgcn_make_buffer_rsrc((void*)base, 0, kOutRangeBytes, kRawBufferWord3)) {}
};

__device__ inline void put(const GlbOut<double>& o, int32_t i, Cx<double> v) {
  typedef double D2 __attribute__((ext_vector_type(2)));
  typedef uint32_t U4 __attribute__((ext_vector_type(4)));
  const D2 x = {v.re, v.im};
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(U4, x), o.r, i * 16, 0, kWriteThrough);
}
__device__ inline void put(const GlbOut<float>& o, int32_t i, Cx<float> v) {
  typedef float F2 __attribute__((ext_vector_type(2)));
  typedef uint32_t U2 __attribute__((ext_vector_type(2)));
  const F2 x = {v.re, v.im};
  __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(U2, x), o.r, i * 8, 0, kWriteThrough);
}
// Serial tasks store plainly: most of what they write is read again by the
// same workgroup, and scattered entries written through cost the task more
// than the release then does (256-knot batch 930 -> 820 us, mixed-q values 1187
// -> 1040 us).
template <class T>
__device__ inline void put(GlbCx<T>* p, int32_t i, Cx<T> v) {
  p[i].re = v.re;
  p[i].im = v.im;
}
template <class T>
__device__ inline void put(LdsCx<T>* p, int32_t i, Cx<T> v) {
  p[i].re = v.re;
  p[i].im = v.im;
}

// Tensor states: those produced by the running serial task are cached in LDS,
// the rest live in global memory.
struct States {
  TensorState* g;
  int32_t* sh;  // LDS
  int64_t* ex;  // LDS
  int32_t lo, len;
  __device__ inline bool local(int32_t t) const { return (uint32_t)(t - lo) < (uint32_t)len; }
  __device__ inline void get(int32_t t, int32_t& shift, int64_t& e) const {
    if (local(t)) {
      shift = sh[t - lo];
      e = ex[t - lo];
    } else {
      shift = g[t].shift;
      e = g[t].exp2;
    }
  }
  // A state beyond what LDS holds that the running serial task may have
  // updated by atomics at the L2.  (Every lane of such a load is a request of
  // its own: tile tasks, which read their operands' states in all threads,
  // spent 10 us more each with it.)
  __device__ inline void get_late(int32_t t, int32_t& shift, int64_t& e) const {
    shift = __hip_atomic_load(&g[t].shift, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    e = __hip_atomic_load(&g[t].exp2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __device__ inline void set(int32_t t, int32_t shift, int64_t e) const {
    if (local(t)) {
      sh[t - lo] = shift;
      ex[t - lo] = e;
    } else {
      g[t].shift = shift;
      g[t].exp2 = e;
    }
  }
};

// threadIdx.x as a value of this task: without it every expression of the
// thread's index alone is computed before the task loop and held in registers
// (or scratch memory) through all of it.
__device__ inline int32_t task_tid() {
  int32_t t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

// ------------------------------------------------------------------ reductions

template <class T>
__device__ inline T wave_max(T v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
  return v;
}

// Maximum of an integer over the wavefront, in lane 63 (row shifts, then row
// broadcasts; a lane without a source keeps its own value).
__device__ inline int32_t wave_max_last(int32_t v) {
#define KN_DPP_MAX(ctrl, rows) \
  v = max(v, __builtin_amdgcn_update_dpp(v, v, ctrl, rows, 0xf, false))
  KN_DPP_MAX(0x111, 0xf);  // row_shr:1
  KN_DPP_MAX(0x112, 0xf);  // row_shr:2
  KN_DPP_MAX(0x114, 0xf);  // row_shr:4
  KN_DPP_MAX(0x118, 0xf);  // row_shr:8
  KN_DPP_MAX(0x142, 0xa);  // row_bcast:15 into rows 1 and 3
  KN_DPP_MAX(0x143, 0xc);  // row_bcast:31 into rows 2 and 3
#undef KN_DPP_MAX
  return v;
}

// Inclusive sum over the lanes up to this one.
__device__ inline int32_t wave_scan(int32_t v) {
#define KN_DPP_ADD(ctrl, rows) v += __builtin_amdgcn_update_dpp(0, v, ctrl, rows, 0xf, false)
  KN_DPP_ADD(0x111, 0xf);
  KN_DPP_ADD(0x112, 0xf);
  KN_DPP_ADD(0x114, 0xf);
  KN_DPP_ADD(0x118, 0xf);
  KN_DPP_ADD(0x142, 0xa);
  KN_DPP_ADD(0x143, 0xc);
#undef KN_DPP_ADD
  return v;
}

// The lane in [lo, hi) whose run of items holds item x, from the inclusive
// sums `end` of the lanes' runs; x does not decrease from lane to lane and is
// below hi's last sum.  The runs that end within the wavefront's 64 items are
// counted one by one (few of them mostly; a bisection over the lanes is six
// dependent shuffles).
__device__ inline int32_t lane_of(int32_t end, int32_t x, int32_t lo, int32_t hi) {
  const int32_t lane = threadIdx.x & 63;
  const int32_t x_first = __builtin_amdgcn_readlane(x, 0), x_last = __builtin_amdgcn_readlane(x, 63);
  int32_t j = lo + __popcll(__ballot(lane >= lo && lane < hi && end <= x_first));
  int32_t at = j;
  for (int32_t e = __builtin_amdgcn_readlane(end, j); e <= x_last; e = __builtin_amdgcn_readlane(end, j)) {
    at += x >= e ? 1 : 0;
    ++j;
  }
  return at;
}

template <class T>
__device__ inline T block_max(T v, T* red) {
  v = wave_max(v);
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  if (lane == 0) red[wv] = v;
  __syncthreads();
  T r = red[0];
#pragma unroll
  for (int i = 1; i < kBlock / 64; ++i) r = fmax(r, red[i]);
  return r;
}

// ------------------------------------------------------------------ setup

// Lane u's value of an integer held per lane (uniform result).
__device__ inline int32_t rl(int32_t v, int32_t lane) { return __builtin_amdgcn_readlane(v, lane); }

// Indices below 2^15 are divided by q in 24-bit arithmetic (full rate; a
// 32-bit multiply takes four times as long): with m = ceil(2^18 / q) the
// product x m is below 2^32, and m q exceeds 2^18 by less than q <= 8, so
// x m / 2^18 exceeds x / q by less than 1 / q.
constexpr int32_t kSmallIndex = 1 << 15;
__device__ inline uint32_t small_magic(int32_t q) { return ((1u << 18) + (uint32_t)q - 1) / (uint32_t)q; }

// QDiv(q) without a 64-bit integer division: 2^(31 + l) / q is below 2^32 and,
// where it is no integer, at least 1 / q away from one, far more than the
// rounding of the quotient in double precision for q < 2^20.
__device__ inline QDiv qdiv_of(int32_t q) {
  const int32_t l = 32 - __clz(q - 1);
  return QDiv(q, (uint32_t)(__builtin_ldexp(1.0, 31 + l) / (double)q) + 1u, l - 1);
}

template <class T>
__device__ __attribute__((always_inline)) void knot_setup(const DevProg& p, const KnotDesc& kd, Cx<T>* arena, Cx<T>* lds,
                           LdsCx<double>* s_w, int32_t w_cap, const double* J, const States& st, int32_t slice) {
  const int tid = task_tid();
  const ImgHeader& h = *p.h;
  Cx<double>* xe = p.weights + kd.w_off;
  Cx<double>* xm = xe + kd.n_edges;
  // x_e = e^{J_e}, or the Jones coupling -t^{-eps_e} (Sec. II)
  const Cx<double> t{kd.t_re, kd.t_im};
  const double tn = t.re * t.re + t.im * t.im;
  const Cx<double> tinv{t.re / tn, -t.im / tn};
  for (int e = tid; e < kd.n_edges; e += kBlock) {
    Cx<double> x;
    if (J) {
      double jr = J[2 * (kd.edge_off + e)], ji = J[2 * (kd.edge_off + e) + 1];
      double er = exp(jr);
      double sn, cs;
      sincos(ji, &sn, &cs);
      x = {er * cs, er * sn};
    } else {
      Cx<double> b = p.eps[kd.edge_off + e] > 0 ? tinv : t;
      x = {-b.re, -b.im};
    }
    xe[e] = x;
  }
  __syncthreads();
  for (int m = tid; m < kd.n_medges; m += kBlock) {
    const MEdge me = p.medges[kd.medge_off + m];
    Cx<double> x{1.0, 0.0};
    if (me.n_members < 0) x = plan_consts(p, kd)[me.member_off];  // derived edge
    for (int i = 0; i < me.n_members; ++i) x = cmul(x, xe[p.members[me.member_off + i]]);
    xm[m] = x;
  }
  __syncthreads();
  // the weights of the vertices' slots (each merged edge is absorbed once), in
  // slot order, to LDS: the loop over a vertex's entries then reads no global
  // memory (a load there would also wait for the entries stored before it)
  const VtxDesc* vtx = p.vtx + kd.vtx_off;
  const int32_t slot0 = kd.n_vtx ? vtx[0].slot_off : 0;
  const int32_t n_slot = kd.n_vtx ? vtx[kd.n_vtx - 1].slot_off + vtx[kd.n_vtx - 1].n_slots - slot0 : 0;
  for (int32_t i = tid; i < min(n_slot, w_cap); i += kBlock) {
    const Cx<double> x = xm[p.vslot[slot0 + i]];
    s_w[i].re = x.re;
    s_w[i].im = x.im;
  }
  __syncthreads();
  // vertex tensors, 64 vertices at a time: lane l of every wavefront loads the
  // records of vertex l of the block, and the block's entries, vertex after
  // vertex, are shared out to the wavefronts 64 at a time, each lane with the
  // vertex of its entry (a vertex has 9 to 81 entries mostly: one vertex at a
  // time left most lanes idle, and its 300 or so instructions were what setup
  // took).
  const int lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int q = kd.q;
  const uint32_t m18 = small_magic(q);
  VtxDesc next{};
  if (lane < kd.n_vtx) next = vtx[lane];
  for (int v0 = 0; v0 < kd.n_vtx; v0 += 64) {
    const VtxDesc my = next;
    TensorDesc td{};
    if (v0 + lane < kd.n_vtx) {
      td = p.tens[my.tensor];
      // entries are products of <= 8 weights: no scaling needed
      if (wv == 0) st.set(my.tensor, 0, 0);
    }
    next = VtxDesc{};
    if (v0 + 64 + lane < kd.n_vtx) next = vtx[v0 + 64 + lane];
    const int32_t e_end = wave_scan(td.size);
    const int32_t total = rl(e_end, 63);
    for (int32_t x0 = 64 * wv; x0 < total; x0 += kBlock) {
      const int32_t x = min(x0 + lane, total - 1);
      const int u = lane_of(e_end, x, 0, 64);
      const int32_t n_slots = __shfl(my.n_slots, u, 64), keep = __shfl(my.keep_center, u, 64);
      const int32_t slot = __shfl(my.slot_off, u, 64) - slot0;
      const int32_t i = x - (__shfl(e_end, u, 64) - __shfl(td.size, u, 64));
      // digits of entry i, 3 bits each: last neighbour slot fastest (first
      // here); a kept centre is the leading index (what is left after the
      // slot digits), a private centre is summed over.  A reverse-pass seed
      // (keep_center < 0, no slots, one entry) takes the kept branch with an
      // empty product: the scalar 1.
      uint32_t dig = 0, rem = (uint32_t)i;
      for (int j = 0; j < n_slots; ++j) {
        const uint32_t up = rem < (uint32_t)kSmallIndex ? __umul24(rem, m18) >> 18 : rem / (uint32_t)q;
        dig |= (rem - up * (uint32_t)q) << (3 * j);
        rem = up;
      }
      const int a_lo = keep ? (int)rem : 0;
      const int a_hi = keep ? a_lo + 1 : q;
      const int32_t pin_off = __shfl(my.pin_off, u, 64), n_pins = __shfl(my.n_pins, u, 64);
      Cx<double> acc{0.0, 0.0};
      for (int a = a_lo; a < a_hi; ++a) {
        Cx<double> prod{1.0, 0.0};
        for (int j = 0; j < n_slots; ++j) {
          const int32_t sl = slot + n_slots - 1 - j;
          if ((int)((dig >> (3 * j)) & 7) != a) continue;
          Cx<double> w;
          if (sl < w_cap) w = Cx<double>{s_w[sl].re, s_w[sl].im};
          else w = xm[p.vslot[slot0 + sl]];
          prod = cmul(prod, w);
        }
        // slices: an edge to a fixed spin contributes x_m where this spin
        // takes the fixed value (digit j of the slice number, base q)
        for (int j = 0; j < n_pins; ++j) {
          const int32_t* pn = p.pins + 2 * (pin_off + j);
          int sv = slice;
          for (int r = 0; r < pn[1]; ++r) sv /= q;
          if (sv % q == a) prod = cmul(prod, xm[pn[0]]);
        }
        acc.re += prod.re;
        acc.im += prod.im;
      }
      const int32_t lds_off = __shfl(td.lds_off, u, 64);
      const int32_t off_lo = __shfl((int32_t)td.off, u, 64), off_hi = __shfl((int32_t)(td.off >> 32), u, 64);
      if (x0 + lane < total) {
        const Cx<T> v{(T)acc.re, (T)acc.im};
        if (lds_off >= 0) put((LdsCx<T>*)(lds + lds_off), i, v);
        else put((GlbCx<T>*)(arena + (int64_t)(((uint64_t)(uint32_t)off_hi << 32) | (uint32_t)off_lo)), i, v);
      }
    }
  }
}

// ------------------------------------------------------------------ step

// Lanes per output: enough to give each of the nthr threads work, at most 64
// (one wavefront, reduced with shuffles) and at most the contracted extent.
__device__ inline int32_t lanes_per_output(int64_t outs, int32_t nk, int32_t nthr = kBlock) {
  int32_t L = 1;
  while (L < 64 && 2 * L <= nk && outs * L < nthr) L *= 2;
  return L;
}

// The shift of a tensor whose entries are all subnormal: that of the least
// normal number.  Its own exponent would make 2^-(sA+sB) overflow beside a
// tensor of shift 0; no shift at all would leave the products subnormal, with
// the few bits a subnormal has.
template <class T>
constexpr int32_t kMinShift = sizeof(T) == 8 ? -1021 : -125;

template <class T>
__device__ inline int32_t frexp_shift(T m) {
  if (!(m > 0)) return kShiftNone;
  int32_t s;
  if constexpr (sizeof(T) == 8) s = __builtin_amdgcn_frexp_exp(m);
  else s = __builtin_amdgcn_frexp_expf(m);
  return max(s, kMinShift<T>);
}

// Scale 2^-(sA+sB) applied to the products, and the exponent of C.
template <class T>
__device__ inline T step_scale(const States& st, int32_t a, int32_t b, int64_t& e_out) {
  int32_t sa, sb;
  int64_t ea, eb;
  st.get(a, sa, ea);
  st.get(b, sb, eb);
  const int32_t sh = shift_of(sa) + shift_of(sb);
  e_out = ea + eb + sh;
  return (T)ldexp(1.0, -sh);
}

// ---- serial runs
//
// The steps of a serial task are small (a few tens of outputs, a contracted
// extent of 3 or 9), so what bounds a run is the latency of each step's chain
// of some hundreds of dependent instructions, and how many steps run at once,
// not products or memory.  Hence:
//   - no gather tables: an entry's offsets in A and B are decoded from its
//     index digit by digit, the strides of each digit held in LDS.  Tables of
//     the offsets were generated entry by entry before a run and cost a quarter
//     of its time;
//   - the outputs of a dependency level, step after step, are shared out to the
//     wavefronts 64 at a time, each lane with the step of its output: a level
//     of 64 steps of 9 to 27 outputs takes each wavefront three rounds, not
//     the eight steps one after another that it took a wavefront per step;
//   - a lane computes a tile of up to 3 x 3 outputs that share rows and columns,
//     where a level has more outputs than the workgroup has lanes;
//   - only a level ends with a barrier: an output's shift is the maximum over
//     its entries, kept by an LDS atomic.
// Steps with a long contracted index (for their outputs) run as units: 2^l
// lanes share an output, and units of up to about kUnitMacs multiply-adds are
// taken by the wavefronts in turn.
// Figures: the launch of one 574-crossing knot (q = 3, complex128) 480 -> 200 us,
// of one 157-crossing knot with q = 5 170 -> 105 us; a 263-step run of the
// 256-knot batch 440 -> 250 us (LDS arena of 96 KiB but for the last).
constexpr int32_t kUnitMacs = 1024;
constexpr float kStageMacs = 4096.0f;
constexpr int32_t kDigCap = kTabBuf / 2;  // digit strides (pairs) of a chunk
static_assert(kDescBuf == 64, "lane j holds step j of a chunk");

// A flat step as its lanes read it from LDS.
struct alignas(16) FlatRec {
  int32_t o_start;     // its first output among those of the chunk's flat steps
  int32_t i_start;     // its first item among theirs
  int32_t dig_off;     // its digit strides
  int32_t ranks;       // as in StepDesc
  int32_t nn, nm;      // columns and rows
  int32_t sn, sm;      // columns (rows) per value of the highest column (row) digit
  int32_t ha, hb, hc;  // homes
  int32_t ia, ib, ic;  // states of A, B and C in the state arrays
};
static_assert(sizeof(FlatRec) == kFlatRecBytes, "LDS layout");

// A unit: a run of one step's outputs (uniform over the wavefront).
template <class T>
struct UnitCtx {
  int2 dig;            // lane d: strides in A and B of output digit d, then of
                       // contracted digits from lane R, least significant first
  int32_t R, rk, q;    // output digits, contracted digits
  int32_t nkq, qi;     // contracted extent = nkq values of its upper digits x qi
  int32_t log_l;       // lanes per output
  int32_t o0, o1;      // outputs of this unit
  int32_t ha, hb, hc;  // homes of A, B and C
  bool small;          // every index is below kSmallIndex
  uint32_t m18;
  T scale;
  QDiv D;
};

// Offsets in A and B of index x < q^n over n digits from d0.  Called with every
// lane of the wavefront on, like all code that reads other lanes' registers (one
// copied or spilled under a partial mask would hold nothing of the lanes that
// are off).  Four digits at a time without a branch: a taken branch costs a lone
// wavefront as much as several digits, and the digits past the last are zero.
template <class T>
__device__ inline int2 unit_offsets(const UnitCtx<T>& u, int32_t x, int32_t d0, int32_t n) {
  int2 off{0, 0};
  if (u.small) {
    for (int32_t d = d0; d < d0 + n; d += 4) {
#pragma unroll
      for (int32_t i = 0; i < 4; ++i) {
        const uint32_t up = __umul24((uint32_t)x, u.m18) >> 18;
        const uint32_t r = (uint32_t)x - __umul24(up, (uint32_t)u.q);
        off.x += (int32_t)__umul24(r, (uint32_t)rl(u.dig.x, d + i));
        off.y += (int32_t)__umul24(r, (uint32_t)rl(u.dig.y, d + i));
        x = (int32_t)up;
      }
    }
  } else {
    for (int32_t d = d0; d < d0 + n; ++d) {
      const int32_t up = u.D.div(x);
      const int32_t r = x - up * u.q;
      off.x += r * rl(u.dig.x, d);
      off.y += r * rl(u.dig.y, d);
      x = up;
    }
  }
  return off;
}

template <class T>
__device__ inline void cfma(Cx<T>& c, Cx<T> a, Cx<T> b) {
  c.re = fma(a.re, b.re, c.re);
  c.im = fma(a.re, b.im, c.im);
  c.re = fma(-a.im, b.im, c.re);
  c.im = fma(a.im, b.re, c.im);
}

// N entries of an operand from entry `off` of the arena it lives in (home < 0:
// LDS), `stride` apart.  The branch is uniform; each side keeps its own address
// space (a generic load would wait for every earlier store), and one copy of
// the code around it serves all four combinations of homes: a run's code is
// fetched anew in every launch, and four copies of it were a good part of the
// time of a single small knot.
template <int N, class T>
__device__ inline void load_entries(Cx<T>* arena, Cx<T>* lds, int32_t home, int32_t off, int32_t stride,
                                    Cx<T> (&v)[N]) {
  if (home < 0) {
    const LdsCx<T>* p = (const LdsCx<T>*)(lds + (-1 - home)) + off;
#pragma unroll
    for (int j = 0; j < N; ++j) v[j] = ldc(p + j * stride);
  } else {
    const GlbCx<T>* p = (const GlbCx<T>*)(arena + home) + off;
#pragma unroll
    for (int j = 0; j < N; ++j) v[j] = ldc(p + j * stride);
  }
}

// NO outputs per lane (base + slot, and base + slot + one round): the loads
// of three contracted entries of all of them are issued before their products.
// 2^log_l lanes share an output's contracted entries.  Returns the largest
// magnitude stored by this lane.
template <int NO, class T>
__device__ __attribute__((always_inline)) T unit_round(const UnitCtx<T>& u, Cx<T>* arena, Cx<T>* lds,
                                                               int32_t base, int32_t lane) {
  const int32_t lsub = lane & ((1 << u.log_l) - 1);
  const int32_t nslot = 64 >> u.log_l;
  const int32_t o = base + (lane >> u.log_l);
  const int32_t a0 = rl(u.dig.x, u.R), b0 = rl(u.dig.y, u.R);
  int2 f[NO];
  Cx<T> c[NO];
#pragma unroll
  for (int i = 0; i < NO; ++i) {
    // (lanes past the end repeat the last output and store nothing)
    f[i] = unit_offsets(u, min(o + i * nslot, u.o1 - 1), 0, u.R);
    c[i] = Cx<T>{0, 0};
  }
  for (int32_t kk0 = 0; kk0 < u.nkq; kk0 += 1 << u.log_l) {
    // (every lane decodes, for the strides are read from other lanes'
    // registers; one past the end repeats the last entry and adds nothing)
    const int32_t kk = min(kk0 + lsub, u.nkq - 1);
    const int2 kf = u.nkq > 1 ? unit_offsets(u, kk, u.R + 1, u.rk - 1) : int2{0, 0};
    if (kk0 + lsub >= u.nkq) continue;
    // the entries of the lowest contracted digit at value kk of the others
    int32_t d = 0;
#pragma unroll 1
    for (; d + 3 <= u.qi; d += 3) {
      Cx<T> va[NO][3], vb[NO][3];
#pragma unroll
      for (int i = 0; i < NO; ++i) {
        load_entries<3>(arena, lds, u.ha, f[i].x + kf.x + d * a0, a0, va[i]);
        load_entries<3>(arena, lds, u.hb, f[i].y + kf.y + d * b0, b0, vb[i]);
      }
#pragma unroll
      for (int j = 0; j < 3; ++j)
#pragma unroll
        for (int i = 0; i < NO; ++i) cfma(c[i], va[i][j], vb[i][j]);
    }
#pragma unroll 1
    for (; d < u.qi; ++d) {
      Cx<T> va[NO][1], vb[NO][1];
#pragma unroll
      for (int i = 0; i < NO; ++i) {
        load_entries<1>(arena, lds, u.ha, f[i].x + kf.x + d * a0, 0, va[i]);
        load_entries<1>(arena, lds, u.hb, f[i].y + kf.y + d * b0, 0, vb[i]);
      }
#pragma unroll
      for (int i = 0; i < NO; ++i) cfma(c[i], va[i][0], vb[i][0]);
    }
  }
  for (int32_t m = (1 << u.log_l) >> 1; m >= 1; m >>= 1) {
#pragma unroll
    for (int i = 0; i < NO; ++i) {
      c[i].re += __shfl_xor(c[i].re, m, 64);
      c[i].im += __shfl_xor(c[i].im, m, 64);
    }
  }
  T top = 0;
#pragma unroll
  for (int i = 0; i < NO; ++i) {
    const int32_t oi = o + i * nslot;
    if (lsub == 0 && oi < u.o1) {
      c[i].re *= u.scale;
      c[i].im *= u.scale;
      if (u.hc >= 0) put((GlbCx<T>*)(arena + u.hc), oi, c[i]);
      else put((LdsCx<T>*)(lds + (-1 - u.hc)), oi, c[i]);
      top = fmax(top, fmax(fabs(c[i].re), fabs(c[i].im)));
    }
  }
  return top;
}

// x / d for 0 <= x < 2^15 and d >= 1: x + 0.5 is 0.5 or more away from a
// multiple of d, so its quotient 0.5 / d from an integer, and the product with
// the approximate reciprocal (1 ulp) is off by less than 2^-7 / d.
__device__ inline int32_t small_div(int32_t x, int32_t d) {
  return (int32_t)(((float)x + 0.5f) * __builtin_amdgcn_rcpf((float)d));
}

// Rows (columns) of the tiles of a level's items, for steps of digits < q.
__device__ inline int32_t flat_tile(int32_t q) { return q == 2 || q == 4 ? 2 : 3; }

// One item of a flat step, `r` of the lane: a tile of outputs of one batch
// entry, in up to NT rows (columns) that differ in the highest row (column)
// digit alone; NT = 1: one output.  F says where the operands of all the lanes
// are: 0 LDS, 1 the global arena, 2 either (generic loads, which wait for
// earlier stores too).
//
// A lane's gathered entries are what bounds a level of many outputs (a load of
// 64 scattered entries occupies the memory pipeline for some 40 clocks, at 16
// for its products): a row's entry is multiplied with NT columns' and a
// column's with NT rows'.
template <int F, int NT, class T>
__device__ inline void flat_item(const FlatRec& r, const int2* s_dig, int32_t x, int32_t q, uint32_t m18,
                                 Cx<T>* arena, Cx<T>* lds, const States& st, bool write) {
  const int2* dg = s_dig + r.dig_off;
  const int32_t rb = r.ranks & 255, rm = (r.ranks >> 8) & 255, rk = (r.ranks >> 16) & 255,
                rn = (r.ranks >> 24) & 255;
  const int32_t R = rb + rm + rn;
  int32_t o = x, i0 = 0, j0 = 0, ni = 1, nj = 1;
  if (NT > 1) {
    // the tile's first row and column in the highest digits, and its output
    // where these are zero
    const int32_t bn = rn > 0 ? (q + NT - 1) / NT : 1, bm = rm > 0 ? (q + NT - 1) / NT : 1;
    const int32_t y = small_div(x, bn), z = small_div(y, bm);
    const int32_t u = small_div(z, r.sn), b = small_div(u, r.sm);
    o = (b * r.nm + (u - b * r.sm)) * r.nn + (z - u * r.sn);
    j0 = (x - y * bn) * NT;
    i0 = (y - z * bm) * NT;
    ni = rm > 0 ? min(NT, q - i0) : 1;
    nj = rn > 0 ? min(NT, q - j0) : 1;
  }
  int32_t fa = 0, fb = 0;
  uint32_t y = (uint32_t)o;
  // (the digits past the last are zero)
  for (int32_t d = 0; __any(d < R); d += 4) {
    int2 s4[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) s4[i] = dg[min(d + i, R)];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t up = __umul24(y, m18) >> 18;
      const uint32_t v = y - __umul24(up, (uint32_t)q);
      fa += (int32_t)__umul24(v, (uint32_t)s4[i].x);
      fb += (int32_t)__umul24(v, (uint32_t)s4[i].y);
      y = up;
    }
  }
  // strides of the contracted digits and of the highest row and column digits
  // (where there is none: other steps', not used)
  const int2 s0 = dg[R], s1 = dg[R + 1], s2 = dg[R + 2];
  const int32_t row = dg[max(rn + rm - 1, 0)].x, col = dg[max(rn - 1, 0)].y;
  const int32_t q0 = rk > 0 ? q : 1, q1 = rk > 1 ? q : 1, q2 = rk > 2 ? q : 1;
  if (NT > 1) {
    fa += i0 * row;
    fb += j0 * col;
    o += i0 * r.sm * r.nn + j0 * r.sn;
  }
  T mag = 0;
  Cx<T> c[NT][NT];
#pragma unroll
  for (int i = 0; i < NT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) c[i][j] = Cx<T>{0, 0};
  auto run = [&](auto pa, auto pb) {
    auto macs = [&](auto nk_, auto pa1, auto pb1) {
      constexpr int NK = decltype(nk_)::value;
      Cx<T> va[NK][NT], vb[NK][NT];
#pragma unroll
      for (int k = 0; k < NK; ++k)
#pragma unroll
        for (int i = 0; i < NT; ++i) {
          va[k][i] = vb[k][i] = Cx<T>{0, 0};
          if (i == 0 || i < ni) va[k][i] = ldc(pa1 + (k * s0.x + i * row));
          if (i == 0 || i < nj) vb[k][i] = ldc(pb1 + (k * s0.y + i * col));
        }
#pragma unroll
      for (int k = 0; k < NK; ++k)
#pragma unroll
        for (int i = 0; i < NT; ++i)
#pragma unroll
          for (int j = 0; j < NT; ++j) cfma(c[i][j], va[k][i], vb[k][j]);
    };
    // (two contracted entries at a time where three would take more registers
    // than there are)
    constexpr int NKT = NT == 3 ? 2 : 3;
#pragma unroll 1
    for (int32_t k2 = 0; k2 < q2; ++k2) {
      auto pa1 = pa;
      auto pb1 = pb;
#pragma unroll 1
      for (int32_t k1 = 0; k1 < q1; ++k1) {
        int32_t k0 = 0;
#pragma unroll 1
        for (; k0 + NKT <= q0; k0 += NKT) macs(std::integral_constant<int, NKT>{}, pa1 + k0 * s0.x, pb1 + k0 * s0.y);
#pragma unroll 1
        for (; k0 < q0; ++k0) macs(std::integral_constant<int, 1>{}, pa1 + k0 * s0.x, pb1 + k0 * s0.y);
        pa1 += s1.x;
        pb1 += s1.y;
      }
      pa += s2.x;
      pb += s2.y;
    }
  };
  if constexpr (F == 0)
    run((const LdsCx<T>*)(lds + (-1 - r.ha)) + fa, (const LdsCx<T>*)(lds + (-1 - r.hb)) + fb);
  else if constexpr (F == 1)
    run((const GlbCx<T>*)(arena + r.ha) + fa, (const GlbCx<T>*)(arena + r.hb) + fb);
  else
    run((const Cx<T>*)(r.ha < 0 ? lds + (-1 - r.ha) : arena + r.ha) + fa,
        (const Cx<T>*)(r.hb < 0 ? lds + (-1 - r.hb) : arena + r.hb) + fb);
  if (write) {
    const int32_t sh = shift_of(st.sh[r.ia]) + shift_of(st.sh[r.ib]);
    const T scale = (T)ldexp(1.0, -sh);
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j) {
        if (i < ni && j < nj) {
          c[i][j].re *= scale;
          c[i][j].im *= scale;
          const int32_t oj = o + i * r.sm * r.nn + j * r.sn;
          if (r.hc < 0) put((LdsCx<T>*)(lds + (-1 - r.hc)), oj, c[i][j]);
          else put((GlbCx<T>*)(arena + r.hc), oj, c[i][j]);
          mag = fmax(mag, fmax(fabs(c[i][j].re), fabs(c[i][j].im)));
        }
      }
    __hip_atomic_fetch_max((__attribute__((address_space(3))) int32_t*)&st.sh[r.ic], frexp_shift<T>(mag),
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (o == 0) st.ex[r.ic] = st.ex[r.ia] + st.ex[r.ib] + sh;
  }
}

// Serial steps [first, first + count).
//
// A larger step first has its operands that live in the global arena
// copied to the staging area after the LDS arena (A first, each when it fits):
// one burst of independent coalesced loads by the whole workgroup, after which
// the step's gathers read LDS.
template <class T>
__device__ __attribute__((always_inline)) void serial_steps(const DevProg& p, int32_t first, int32_t count, int32_t q,
                             Cx<T>* arena, Cx<T>* lds, int2* s_dig, FlatRec* s_rec,
                             const States& st, int32_t made, int64_t* ph) {
  const int32_t tid = task_tid();
  const int32_t lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  constexpr int32_t kWaves = kBlock / 64;
  int64_t tk = ph ? wall_clock64() : 0;
  auto lap = [&](int i) {
    if (ph) {
      const int64_t t = wall_clock64();
      ph[i] += t - tk;
      tk = t;
    }
  };
  const QDiv D = qdiv_of(q);
  // the staging area follows the tensor arena
  const int32_t stage_off = p.h->lds_bytes / (int32_t)sizeof(Cx<T>);
  const int32_t stage_elems = stage_bytes(p.h->lds_bytes) / (int32_t)sizeof(Cx<T>);
  const int32_t end = first + count;
  const uint32_t m18 = small_magic(q);
  const int32_t nt = flat_tile(q), q_tiles = (q + nt - 1) / nt;
  int32_t ce = 0;
  StepDesc next{};
  if (first + lane < end) next = p.steps[first + lane];
  for (int32_t s = first; s < end; s += ce) {
    // lane j: step s + j (loaded while the chunk before it ran)
    const bool have = s + lane < end;
    const StepDesc d = next;
    const int32_t rb = d.ranks & 255, rm = (d.ranks >> 8) & 255, rk = (d.ranks >> 16) & 255,
                  rn = (d.ranks >> 24) & 255;
    const int32_t R = rb + rm + rn;
    const int32_t n_dig = have ? R + rk : 0;
    const int32_t dig_end = wave_scan(n_dig);
    // the steps whose digits fit (a step has at most 62)
    const uint64_t fits = __ballot(have && dig_end <= kDigCap);
    ce = __popcll(fits);
    const int32_t dig_off = dig_end - n_dig;
    const int32_t outs = d.nb * d.nm * d.nn;
    // units: runs of whole wavefronts of outputs
    int32_t run = max(outs, 1), units = 0;
    const int32_t nkq = rk > 0 ? D.div(d.nk) : 1;
    int32_t log_l = 0;
    // lanes per output: to fill a wavefront, and the workgroup where the
    // contracted index is long enough to be worth a reduction over lanes
    while (log_l < 6 && (2 << log_l) <= nkq &&
           ((int64_t)outs << log_l) < (d.nk >> log_l >= 16 ? kBlock : 64))
      ++log_l;
    const int32_t pack = R | rk << 8 | log_l << 16 | (outs <= kSmallIndex && nkq <= kSmallIndex ? 1 << 24 : 0);
    // flat: a contracted index that a lane runs through by itself, of at most
    // two spins, or three where the outputs fill the workgroup (2187 outputs of
    // 27 entries took 27 us as units, 6 flat; with a limit of 64 entries, so
    // that 5^3 and 6^3 were units, mixed-q values took 1110 us for 940), and
    // every state in LDS
    auto made_here = [&](int32_t t) { return (uint32_t)(t - st.lo) < (uint32_t)made; };
    auto in_lds = [&](int32_t t) { return st.local(t) || !made_here(t); };
    const bool flat = lane < ce && (rk <= 2 || (rk == 3 && outs >= kBlock)) && outs <= kSmallIndex && in_lds(d.a) && in_lds(d.b) && st.local(d.c);
    const int32_t sn = rn > 0 ? D.div(d.nn) : 1, sm = rm > 0 ? D.div(d.nm) : 1;
    const int32_t items = d.nb * sn * sm * (rn > 0 ? q_tiles : 1) * (rm > 0 ? q_tiles : 1);
    const int32_t f_end = wave_scan(flat ? outs : 0), i_end = wave_scan(flat ? items : 0);
    if (wv == 0 && flat) {
      FlatRec r;
      r.o_start = f_end - outs;
      r.i_start = i_end - items;
      r.dig_off = dig_off;
      r.ranks = d.ranks;
      r.nn = d.nn;
      r.nm = d.nm;
      r.sn = sn;
      r.sm = sm;
      r.ha = d.home_a;
      r.hb = d.home_b;
      r.hc = d.home_c;
      r.ia = st.local(d.a) ? d.a - st.lo : kStateCap + 2 * lane;
      r.ib = st.local(d.b) ? d.b - st.lo : kStateCap + 2 * lane + 1;
      r.ic = d.c - st.lo;
      s_rec[lane] = r;
    }
    if (lane < ce && !flat) {
      const float macs = (float)outs * (float)d.nk;
      const int32_t wide = 64 >> log_l;  // outputs of a wavefront
      const int32_t want = (int32_t)fminf(macs * (1.0f / kUnitMacs), (float)((outs + wide - 1) / wide));
      if (want > 1) run = ((outs + want - 1) / want + wide - 1) & -wide;
      units = (outs + run - 1) / run;
    }
    const bool large = lane < ce && d.nk > 1 && (flat ? (float)outs * (float)d.nk >= kStageMacs : units > 1);
    const int32_t u_sum = wave_scan(units);
    const int32_t u_end = lane < ce ? u_sum : INT32_MAX;
    const int32_t prev_lvl = __shfl_up(d.lvl, 1, 64);
    uint64_t starts = __ballot(lane < ce && (lane == 0 || d.lvl != prev_lvl));
    // states of operands made before this task (final) are fetched now; those
    // of tensors it makes itself are in LDS (or, past what LDS holds, global)
    if (wv < 2 && lane < ce) {
      const int32_t t = wv ? d.b : d.a;
      if (!made_here(t)) {
        const TensorState x = p.ts[t];
        st.sh[kStateCap + 2 * lane + wv] = x.shift;
        st.ex[kStateCap + 2 * lane + wv] = x.exp2;
      }
    }
    // digit strides: entry i belongs to step j (the steps whose digits end
    // before it, counted by bisection over the lanes)
    const int32_t n_ent = rl(dig_end, ce - 1);
    for (int32_t i = tid; i < ((n_ent + 63) & ~63); i += kBlock) {
      int32_t j = 0;
#pragma unroll
      for (int32_t h = 32; h >= 1; h >>= 1)
        if (__shfl(dig_end, j + h - 1, 64) <= i) j += h;
      const int32_t jr = __shfl(d.ranks, j, 64), jo = __shfl(dig_off, j, 64), js = __shfl(d.str, j, 64);
      const int32_t b = jr & 255, m = (jr >> 8) & 255, k = (jr >> 16) & 255, n = (jr >> 24) & 255;
      int32_t x = i - jo;
      // strides: A_b A_m A_k B_b B_k B_n, most significant spin first
      int32_t ia = -1, ib = -1;
      if (x < n) {
        ib = 2 * b + m + 2 * k + n - 1 - x;
      } else if ((x -= n) < m) {
        ia = b + m - 1 - x;
      } else if ((x -= m) < b) {
        ia = b - 1 - x;
        ib = b + m + k + b - 1 - x;
      } else {
        x -= b;
        ia = b + m + k - 1 - x;
        ib = 2 * b + m + 2 * k - 1 - x;
      }
      if (i < n_ent) {
        const int32_t* sp = p.strides + js;
        s_dig[i] = int2{ia >= 0 ? sp[ia] : 0, ib >= 0 ? sp[ib] : 0};
      }
    }
    next = StepDesc{};
    if (s + ce + lane < end) next = p.steps[s + ce + lane];
    __syncthreads();
    lap(1);
    int32_t ha = d.home_a, hb = d.home_b;
    while (starts) {
      const int32_t j0 = __ffsll((unsigned long long)starts) - 1;
      starts &= starts - 1;
      const int32_t j1 = starts ? __ffsll((unsigned long long)starts) - 1 : ce;
      // larger steps with operands in the global arena
      uint64_t stage = __ballot(lane >= j0 && lane < j1 && large && (ha >= 0 || hb >= 0));
      if (stage) {
        LdsCx<T>* stg = (LdsCx<T>*)(lds + stage_off);
        int32_t used = 0;
        do {
          const int32_t j = __ffsll((unsigned long long)stage) - 1;
          stage &= stage - 1;
          const int32_t bk = rl(d.nb, j) * rl(d.nk, j);
#pragma unroll
          for (int op = 0; op < 2; ++op) {
            const int32_t h = op ? rl(hb, j) : rl(ha, j);
            if (h < 0) continue;
            const int64_t n = (int64_t)bk * (op ? rl(d.nn, j) : rl(d.nm, j));
            if (n > stage_elems - used) continue;
            const GlbCx<T>* src = (const GlbCx<T>*)(arena + h);
            for (int32_t i = tid; i < (int32_t)n; i += kBlock) put(stg + used, i, ldc(src + i));
            const int32_t home = -1 - (stage_off + used);
            if (op) hb = lane == j ? home : hb;
            else ha = lane == j ? home : ha;
            if (tid == 0) (op ? s_rec[j].hb : s_rec[j].ha) = home;
            used += (int32_t)n;
          }
        } while (stage);
        __syncthreads();
      }
      // flat steps: a lane takes the outputs of an item, or, where a level has
      // no more outputs than the workgroup has lanes, a single one
      const int32_t of0 = j0 ? rl(f_end, j0 - 1) : 0, of1 = rl(f_end, j1 - 1);
      const bool single = of1 - of0 <= kBlock;
      const int32_t l_end = single ? f_end : i_end;
      const int32_t x1 = single ? of1 : rl(i_end, j1 - 1);
      for (int32_t x0 = (single ? of0 : j0 ? rl(i_end, j0 - 1) : 0) + 64 * wv; x0 < x1; x0 += kBlock) {
        const int32_t x = min(x0 + lane, x1 - 1);
        const FlatRec r = s_rec[lane_of(l_end, x, j0, j1)];
        const int32_t i = x - (single ? r.o_start : r.i_start);
        const bool write = x0 + lane < x1;
        auto item = [&](auto f_) {
          constexpr int F = decltype(f_)::value;
          if (single) flat_item<F, 1, T>(r, s_dig, i, q, m18, arena, lds, st, write);
          else if (nt == 2) flat_item<F, 2, T>(r, s_dig, i, q, m18, arena, lds, st, write);
          else flat_item<F, 3, T>(r, s_dig, i, q, m18, arena, lds, st, write);
        };
        if (!__any(r.ha >= 0 || r.hb >= 0)) item(std::integral_constant<int, 0>{});
        else if (!__any(r.ha < 0 || r.hb < 0)) item(std::integral_constant<int, 1>{});
        else item(std::integral_constant<int, 2>{});
      }
      const int32_t u0 = j0 ? rl(u_end, j0 - 1) : 0, u1 = rl(u_end, j1 - 1);
      if (u0 < u1) {
        // lane j: the scale 2^-sh of step j; its output's exponent
        int32_t sh = 0;
        if (lane >= j0 && lane < j1 && !flat) {
          int32_t sa, sb;
          int64_t ea, eb;
          auto state = [&](int32_t t, int32_t e, int32_t& shift, int64_t& ex) {
            if (st.local(t) || !made_here(t)) {
              const int32_t i = st.local(t) ? t - st.lo : kStateCap + e;
              shift = st.sh[i];
              ex = st.ex[i];
            } else {
              st.get_late(t, shift, ex);
            }
          };
          state(d.a, 2 * lane, sa, ea);
          state(d.b, 2 * lane + 1, sb, eb);
          sh = shift_of(sa) + shift_of(sb);
          if (wv == 0) {
            if (st.local(d.c)) st.ex[d.c - st.lo] = ea + eb + sh;
            else
              __hip_atomic_store(&st.g[d.c].exp2, ea + eb + sh, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          }
        }
        // the digit strides of a wavefront's next unit are loaded while it
        // computes the one before
        auto step_of = [&](int32_t x) { return (int32_t)__popcll(__ballot(u_end <= x)); };
        auto digits_of = [&](int32_t j) {
          return s_dig[rl(dig_off, j) + min(lane, max((rl(pack, j) & 255) + ((rl(pack, j) >> 8) & 255) - 1, 0))];
        };
        int32_t x = u0 + wv;
        int32_t j = min(step_of(x), ce - 1);
        int2 dig_next = digits_of(j);
        for (; x < u1; x += kWaves) {
          const int2 dig = dig_next;
          const int32_t j_next = min(step_of(x + kWaves), ce - 1);
          dig_next = digits_of(j_next);
          const int32_t part = x - (j ? rl(u_end, j - 1) : 0);
          const int32_t pk = rl(pack, j);
          const int32_t uR = pk & 255, urk = (pk >> 8) & 255;
          const int32_t len = rl(run, j);
          const UnitCtx<T> u{dig, uR, urk, q, rl(nkq, j), urk > 0 ? q : 1, (pk >> 16) & 255, part * len,
                             min(rl(outs, j), part * len + len), rl(ha, j), rl(hb, j), rl(d.home_c, j),
                             (pk >> 24) != 0, m18,
                             (T)ldexp(1.0, -rl(sh, j)), D};
          const int32_t nslot = 64 >> u.log_l;
          T top = 0;
          int32_t at = u.o0;
  #pragma unroll 1
          for (; at + nslot < u.o1; at += 2 * nslot) top = fmax(top, unit_round<2>(u, arena, lds, at, lane));
          if (at < u.o1) top = fmax(top, unit_round<1>(u, arena, lds, at, lane));
          const int32_t mx = wave_max_last(frexp_shift<T>(top));
          const int32_t tc = rl(d.c, j);
          if (lane == 63) {
            if (st.local(tc))
              __hip_atomic_fetch_max((__attribute__((address_space(3))) int32_t*)&st.sh[tc - st.lo],
                                     mx, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            else
              __hip_atomic_fetch_max(&st.g[tc].shift, mx, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          }
          j = j_next;
        }
      }
      lap(2);
      __syncthreads();
      lap(3);
    }
  }
}

// Output shift of a tiled step: every tile of an unsplit step folds its max
// into C's shift, and tile 0 writes C's exponent.
template <class T>
__device__ inline void tile_publish(const DevProg& p, int32_t c, int32_t tile_id, T lm, int64_t ec,
                                    T* s_red) {
  lm = block_max<T>(lm, s_red);
  if (threadIdx.x == 0) {
    const int32_t sh = frexp_shift<T>(lm);
    if (sh != kShiftNone)
      __hip_atomic_fetch_max(&p.ts[c].shift, sh, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (tile_id == 0) p.ts[c].exp2 = ec;
  }
}

// Offsets in A and B of an index over a list of spins, in LDS: one entry per
// value of the lowest spins (together `n_lo` values) and one per value of the
// rest that a task meets, added up on use.  Few enough of either to be made in
// a round or two by the workgroup whatever the index's range: one table of the
// whole range seldom fits LDS for a wide step, whose offsets were then decoded
// spin by spin, from strides in global memory, at every use.
struct SplitTab {
  const int2* lo;
  const int2* hi;   // of value h at h - h0; null: decoded
  int32_t h0;
  QDiv by;          // n_lo
  const int2* str;  // strides of the upper spins, least significant first
  int32_t n;        // upper spins
  QDiv D;
  __device__ inline int2 at(int32_t i) const {
    int32_t h = by.div(i);
    int2 off = lo[i - h * by.q];
    if (hi) {
      off.x += hi[h - h0].x;
      off.y += hi[h - h0].y;
    } else {
      for (int32_t d = 0; d < n; ++d) {
        const int32_t up = D.div(h);
        off.x += (h - up * D.q) * str[d].x;
        off.y += (h - up * D.q) * str[d].y;
        h = up;
      }
    }
    return off;
  }
};

// Most entries of a split table's two parts (two tables fit LDS).
constexpr int32_t kSplitLo = 2048, kSplitHi = 6144;

// The table of indices [i0, i1) over n spins whose strides in A and B are
// str[d], least significant spin d = 0, at `mem` (LDS, next free entry in
// `used`).  The caller synchronises before the table is read.
__device__ inline SplitTab split_tab(int2* mem, int32_t& used, int32_t tid, int32_t i0, int32_t i1,
                                     const int2* str, int32_t n, const QDiv& D) {
  int32_t r = 0, n_lo = 1;
  while (r < n && n_lo * D.q <= kSplitLo && (r == 0 || n_lo < i1 - i0)) {
    n_lo *= D.q;
    ++r;
  }
  const QDiv by = qdiv_of(max(n_lo, 2));  // (n = 0: the index is 0)
  const int32_t h0 = by.div(i0), n_hi = by.div(i1 - 1) - h0 + 1;
  const bool both = n_hi <= kSplitHi;
  int2* lo = mem + used;
  int2* hi = lo + n_lo;
  const int32_t all = n_lo + (both ? n_hi : 0);
  used += all;
  for (int32_t i = tid; i < all; i += kBlock) {
    const bool low = i < n_lo;
    int32_t x = low ? i : h0 + (i - n_lo);
    const int32_t d1 = low ? r : n;
    int2 off{0, 0};
    for (int32_t d = low ? 0 : r; d < d1; ++d) {
      const int32_t up = D.div(x);
      const int32_t v = x - up * D.q;
      off.x += v * str[d].x;
      off.y += v * str[d].y;
      x = up;
    }
    lo[i] = off;
  }
  return SplitTab{lo, both ? hi : nullptr, h0, by, str + r, n - r, D};
}

// STEP_TILES: `tile` consecutive outputs of C (row-major over b, m, n), over
// contracted range ks of the split.  Bound by the memory its operands come
// from (a contracted index of 1 or 3, mostly), as long as enough loads are in
// flight: offsets come from split tables in LDS, and
//   - up to 64 contracted entries: lane k holds the offsets of entry k, a
//     thread computes two outputs together and issues the loads of three
//     entries of both before their products; a B of fewer entries than the
//     tile has outputs is first copied to LDS (half of the gathered loads were
//     B's, and a gathered load occupies the memory pipeline whether or not it
//     hits), and the thread then computes four (a step of 9 x 531441 outputs
//     over 3 entries: products 18.7 -> 15.1 us a task; half the copy rate of the
//     card when every compute unit runs such tasks);
//   - more of them: L lanes share an output, four entries each per round;
//   - one output over a long segment (the scalar product that ends a knot's
//     contraction, split over many tasks): all wavefronts, an equal part of
//     the segment each; thread 0 adds the partial sums in wavefront order.
//
// ph (traced launches, thread 0; else null; ph[3] holds the task's start):
// from the start to the end of the tables and operand states, then the
// products, then the publish.
template <class T>
__device__ __attribute__((always_inline)) void tile_step(const DevProg& p, const StepDesc& s, int32_t tile_id, int32_t q,
                          Cx<T>* arena, uint8_t* smem, int32_t smem_bytes, const States& st, T* s_red, int64_t* ph) {
  const int32_t tid = task_tid();
  const int32_t lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  constexpr int32_t kWaves = kBlock / 64;
  const QDiv D = qdiv_of(q);
  const int32_t rb = s.ranks & 255, rm = (s.ranks >> 8) & 255, rk = (s.ranks >> 16) & 255,
                rn = (s.ranks >> 24) & 255;
  const int64_t outs = (int64_t)s.nb * s.nm * s.nn;
  const int32_t base = s.n_tiles / s.n_ks;
  const int32_t ks = tile_id / base, t = tile_id - ks * base;
  const int32_t k0 = ks * s.kseg, k1 = min(s.nk, k0 + s.kseg), nk = k1 - k0;
  const int32_t o0 = t * s.tile;
  const int32_t o1 = (int32_t)min((int64_t)o0 + s.tile, outs);
  // LDS: partial sums of the wavefronts, strides, tables
  constexpr int32_t kTileFixed = kWaves * (int32_t)sizeof(Cx<double>) + 64 * (int32_t)sizeof(int2);
  LdsCx<double>* part = (LdsCx<double>*)smem;
  int2* dig = reinterpret_cast<int2*>(smem + kWaves * sizeof(Cx<double>));
  const int32_t R = rb + rm + rn;
  // strides in A and B of the output's spins n, m, b and of the contracted
  // ones, least significant first (stored: A_b A_m A_k B_b B_k B_n, most first)
  if (tid < R + rk) {
    int32_t x = tid, ia = -1, ib = -1;
    if (x < rn) {
      ib = 2 * rb + rm + 2 * rk + rn - 1 - x;
    } else if ((x -= rn) < rm) {
      ia = rb + rm - 1 - x;
    } else if ((x -= rm) < rb) {
      ia = rb - 1 - x;
      ib = rb + rm + rk + rb - 1 - x;
    } else {
      x -= rb;
      ia = rb + rm + rk - 1 - x;
      ib = 2 * rb + rm + 2 * rk - 1 - x;
    }
    const int32_t* sp = p.strides + s.str;
    dig[tid] = int2{ia >= 0 ? sp[ia] : 0, ib >= 0 ? sp[ib] : 0};
  }
  int64_t ec;
  const T scale = step_scale<T>(st, s.a, s.b, ec);
  __syncthreads();
  int2* mem = dig + 64;
  int32_t used = 0;
  const SplitTab to = split_tab(mem, used, tid, o0, o1, dig, R, D);
  const SplitTab tk_ = split_tab(mem, used, tid, k0, k1, dig + R, rk, D);
  // B, if it has no more entries than the tile has outputs and fits
  const int32_t L = lanes_per_output(o1 - o0, nk);
  const int64_t size_b = (int64_t)s.nb * s.nk * s.nn;
  LdsCx<T>* stg = (LdsCx<T>*)(mem + ((used + 1) & ~1));
  const bool b_lds = L == 1 && nk <= 64 && size_b <= o1 - o0 &&
                     size_b * (int32_t)sizeof(Cx<T>) <= smem_bytes - (kTileFixed + 8 * (used + 1));
  if (b_lds)
    for (int32_t i = tid; i < (int32_t)size_b; i += kBlock) put(stg, i, ldc((const GlbCx<T>*)(arena + s.home_b) + i));
  __syncthreads();
  int64_t tk = 0;
  if (ph) {
    tk = wall_clock64();
    ph[0] = tk - ph[3];
  }
  Cx<T>* pc = s.n_ks > 1 ? arena + s.partial + (int64_t)ks * outs : arena + s.home_c;
  const GlbCx<T>* pa = (const GlbCx<T>*)(arena + s.home_a);
  const GlbCx<T>* pb = (const GlbCx<T>*)(arena + s.home_b);
  const GlbOut<T> out((GlbCx<T>*)pc + o0);
  const Cx<T> zero{0, 0};
  T lm = 0;
  auto store = [&](int32_t o, Cx<T> c) {
    c.re *= scale;
    c.im *= scale;
    put(out, o - o0, c);
    lm = fmax(lm, fmax(fabs(c.re), fabs(c.im)));
  };
  // sum over the entries k_first, k_first + L, ... < k_end, four per round
  auto dot = [&](int2 f, int32_t k, int32_t k_end, int32_t L) {
    Cx<T> c = zero, c2 = zero;
    for (; k < k_end; k += 4 * L) {
      Cx<T> x[4], y[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        x[j] = y[j] = zero;
        if (k + j * L < k_end) {
          const int2 e = tk_.at(k + j * L);
          x[j] = ldc(pa + (f.x + e.x));
          y[j] = ldc(pb + (f.y + e.y));
        }
      }
      cfma(c, x[0], y[0]);
      cfma(c2, x[1], y[1]);
      cfma(c, x[2], y[2]);
      cfma(c2, x[3], y[3]);
    }
    return Cx<T>{c.re + c2.re, c.im + c2.im};
  };
  // the products of a short contracted index, NO outputs per thread at once
  auto short_k = [&](auto no_, auto qb) {
    constexpr int NO = decltype(no_)::value;
    const int2 dk = lane < nk ? tk_.at(k0 + lane) : int2{0, 0};
    // (a wavefront leaves the loop as a whole: macs reads all lanes' dk)
    for (int32_t ow = o0 + 64 * wv; ow < o1; ow += NO * kBlock) {
      const int32_t o = ow + lane;
      int2 f[NO];
      Cx<T> c[NO];
#pragma unroll
      for (int j = 0; j < NO; ++j) {
        f[j] = to.at(min(o + j * kBlock, o1 - 1));
        c[j] = zero;
      }
      auto macs = [&](auto nk_, int32_t k) {
        constexpr int NK = decltype(nk_)::value;
        Cx<T> x[NO][NK], y[NO][NK];
        int2 e[NK];
#pragma unroll
        for (int i = 0; i < NK; ++i) e[i] = int2{rl(dk.x, k + i), rl(dk.y, k + i)};
#pragma unroll
        for (int j = 0; j < NO; ++j)
#pragma unroll
          for (int i = 0; i < NK; ++i) {
            x[j][i] = y[j][i] = zero;
            if (o + j * kBlock < o1) {
              x[j][i] = ldc(pa + (f[j].x + e[i].x));
              y[j][i] = ldc(qb + (f[j].y + e[i].y));
            }
          }
#pragma unroll
        for (int i = 0; i < NK; ++i)
#pragma unroll
          for (int j = 0; j < NO; ++j) cfma(c[j], x[j][i], y[j][i]);
      };
      int32_t k = 0;
#pragma unroll 1
      for (; k + 3 <= nk; k += 3) macs(std::integral_constant<int, 3>{}, k);
#pragma unroll 1
      for (; k < nk; ++k) macs(std::integral_constant<int, 1>{}, k);
#pragma unroll
      for (int j = 0; j < NO; ++j)
        if (o + j * kBlock < o1) store(o + j * kBlock, c[j]);
    }
  };
  if (o1 - o0 == 1 && nk >= 2 * kBlock) {
    const int32_t run = (nk + kWaves - 1) / kWaves;
    const int32_t kw0 = min(k1, k0 + wv * run), kw1 = min(k1, kw0 + run);
    Cx<T> c = dot(to.at(o0), kw0 + lane, kw1, 64);
    for (int32_t m = 32; m >= 1; m >>= 1) {
      c.re += __shfl_xor(c.re, m, 64);
      c.im += __shfl_xor(c.im, m, 64);
    }
    if (lane == 0) {
      part[wv].re = c.re;
      part[wv].im = c.im;
    }
    __syncthreads();
    if (tid == 0) {
      c = zero;
      for (int i = 0; i < kWaves; ++i) {
        c.re += (T)part[i].re;
        c.im += (T)part[i].im;
      }
      store(o0, c);
    }
  } else if (L == 1 && nk <= 64) {
    if (b_lds) short_k(std::integral_constant<int, 4>{}, (const LdsCx<T>*)stg);
    else short_k(std::integral_constant<int, 2>{}, pb);
  } else {
    const int32_t lsub = tid & (L - 1);
    for (int32_t o = o0 + tid / L; o < o1; o += kBlock / L) {
      Cx<T> c = dot(to.at(o), k0 + lsub, k1, L);
      for (int32_t m = L >> 1; m >= 1; m >>= 1) {
        c.re += __shfl_xor(c.re, m, 64);
        c.im += __shfl_xor(c.im, m, 64);
      }
      if (lsub == 0) store(o, c);
    }
  }
  if (ph) {
    const int64_t t2 = wall_clock64();
    ph[1] = t2 - tk;
    tk = t2;
  }
  if (s.n_ks == 1) tile_publish<T>(p, s.c, tile_id, lm, ec, s_red);
  if (ph) ph[2] = wall_clock64() - tk;
}

// Matrix-core products for the GEMM blocks: D = A B + C on one 16 x 16
// tile per wavefront, K = 4 (v_mfma_f64_16x16x4f64 / v_mfma_f32_16x16x4f32).
// Operands: lane l holds A[l % 16][l / 16] and B[l / 16][l % 16]; the four
// accumulator registers of lane l hold column l % 16 of D, at rows row(l, r)
// (measured lane layouts of the two instructions on gfx950).
template <class T>
struct Mfma;
template <>
struct Mfma<double> {
  typedef double V __attribute__((ext_vector_type(4)));
  static __device__ inline V mac(double a, double b, V c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ inline int32_t row(int32_t l, int32_t r) { return (l >> 4) + 4 * r; }
};
template <>
struct Mfma<float> {
  typedef float V __attribute__((ext_vector_type(4)));
  static __device__ inline V mac(float a, float b, V c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ inline int32_t row(int32_t l, int32_t r) { return 4 * (l >> 4) + r; }
};

// STEP_GEMM / STEP_GEMM64: output blocks of 32 x 32 or 64 x 64 entries of C[b]
// over contracted range ks of the split, `tile` consecutive blocks per task.
//
// gemm_block computes BR rows and BC columns of C[b] from (m0, n0).  Chunks of
// 16 contracted entries of A (BR rows) and B (BC columns) are gathered into
// LDS (row pitch BR + 1 or BC + 1 entries), in two buffers in turn, the next
// chunk's operands loaded into registers while the current one is multiplied:
// one barrier per chunk.  The products run on the matrix cores, a complex
// 16 x 16 tile taking four real MFMAs per 4 contracted entries,
//   Re += Re A Re B, Re += (-Im A) Im B, Im += Re A Im B, Im += Im A Re B.
// Regions of 64 x 32 and more: the eight wavefronts share the tiles out, 4 x 2
// (8 x 1 for 128 x 32).  32 x 32: a wavefront has the real or the imaginary part of one of the four
// tiles, its two products in accumulators of their own; the imaginary parts go
// through LDS to the wavefront that holds the tile's real part, which stores
// whole entries.  Either way consecutive MFMAs do not wait on each other.
//
// A gathered entry is multiplied with BC columns or BR rows, so a 128 x 128
// region gathers half as much per product as a 64 x 64 block.  Gathers are
// what bounds wide steps: their operands are stored in the order of the steps
// that made them, so a wavefront's 64 entries come from up to 64 lines.
// Rates per compute unit in complex128: K = 2187 240 GFLOP/s (280 is a large
// library product's), K = 243 210, K = 81 170, K = 27 90-115, K = 9 45; the wide
// grid walk 22.6 -> 20.6 ms with regions and two buffers.
template <class T>
struct GemmCtx {
  const GlbCx<T>* A;
  const GlbCx<T>* B;
  GlbCx<T>* C;
  const int32_t* str;   // the step's strides (LDS): A_b A_m A_k B_b B_k B_n
  const int32_t* ktab;  // contracted offsets of A and B in turn (LDS), or null: decode
  int32_t rb, rm, rk, rn;
  int32_t nm, nn, k0, kl;
  T scale;
  uint8_t* buf;         // LDS of the chunk buffers and row and column offsets
  QDiv D;
};

// Contracted entries per chunk: half for the largest region, whose accumulators
// leave registers for half the operands in flight.
template <int BR, int BC>
constexpr int32_t gemm_chunk() {
  return BR * BC >= 128 * 128 ? kGemmChunk / 2 : kGemmChunk;
}
// LDS bytes gemm_block uses.
template <class T, int BR, int BC>
constexpr int32_t gemm_lds() {
  return 2 * gemm_chunk<BR, BC>() * (BR + 1 + BC + 1) * (int32_t)sizeof(Cx<T>) + (BR + BC) * 4;
}

template <class T, int BR, int BC>
__device__ __attribute__((always_inline)) T gemm_block(const GemmCtx<T>& g, int32_t b, int32_t m0, int32_t n0) {
  constexpr int32_t BK = gemm_chunk<BR, BC>(), PA = BR + 1, PB = BC + 1;
  constexpr int32_t LR = kBlock / BK;           // rows (columns) loaded at once
  constexpr int32_t NLA = BR / LR, NLB = BC / LR;
  constexpr bool kParts = BR == 32;             // a wavefront has one part of one tile
  constexpr int32_t WR = BR == 128 && BC == 32 ? 8 : 4, WC = 8 / WR;  // wavefronts by rows, columns
  constexpr int32_t NR = kParts ? 1 : BR / (16 * WR), NC = kParts ? 1 : BC / (16 * WC);  // tiles each
  static_assert(kBlock == 512 && BR % LR == 0 && BC % LR == 0 && BR % 32 == 0 && BC % 32 == 0 &&
                    (kParts ? BC == 32 : BR % (16 * WR) == 0 && BC % (16 * WC) == 0),
                "thread layout: eight wavefronts");
  using M = Mfma<T>;
  using V = typename M::V;
  const int32_t tid = task_tid();
  Cx<T>* As = reinterpret_cast<Cx<T>*>(g.buf);
  Cx<T>* Bs = As + 2 * BK * PA;
  int32_t* rtab = reinterpret_cast<int32_t*>(Bs + 2 * BK * PB);
  int32_t* ctab = rtab + BR;
  // offsets of the rows of A and the columns of B, -1 past the edge
  const int32_t* sab = g.str;
  const int32_t* sam = sab + g.rb;
  const int32_t* sak = sam + g.rm;
  const int32_t* sbb = sak + g.rk;
  const int32_t* sbk = sbb + g.rb;
  const int32_t* sbn = sbk + g.rk;
  if (tid < BR) {
    const int32_t m = m0 + tid;
    rtab[tid] = m < g.nm ? group_off(b, sab, g.rb, g.D) + group_off(m, sam, g.rm, g.D) : -1;
  } else if (tid < BR + BC) {
    const int32_t n = n0 + tid - BR;
    ctab[tid - BR] = n < g.nn ? group_off(b, sbb, g.rb, g.D) + group_off(n, sbn, g.rn, g.D) : -1;
  }
  __syncthreads();
  // this thread's loads: contracted entry kk of rows / columns lr + LR i
  const int32_t kk = tid & (BK - 1), lr = tid / BK;
  int32_t ra[NLA], cb[NLB];
#pragma unroll
  for (int i = 0; i < NLA; ++i) ra[i] = rtab[lr + LR * i];
#pragma unroll
  for (int i = 0; i < NLB; ++i) cb[i] = ctab[lr + LR * i];
  // this wavefront's tiles (the first at row qr, column qc), the part it has
  // of them (kParts), and its lane
  const int32_t lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool imag = kParts && wv >= 4;
  const int32_t qr = kParts ? ((wv >> 1) & 1) * 16 : (wv / WC) * 16 * NR;
  const int32_t qc = kParts ? (wv & 1) * 16 : (wv % WC) * 16 * NC;
  const int32_t l16 = lane & 15, lk = lane >> 4;
  struct Ops {
    Cx<T> a[NLA], b[NLB];
  };
  auto load = [&](int32_t c0) -> Ops {
    const int32_t k = c0 + kk;
    Ops x;
#pragma unroll
    for (int i = 0; i < NLA; ++i) x.a[i] = Cx<T>{0, 0};
#pragma unroll
    for (int i = 0; i < NLB; ++i) x.b[i] = Cx<T>{0, 0};
    if (k < g.kl) {
      int32_t oa, ob;
      if (g.ktab) {
        oa = g.ktab[2 * k];
        ob = g.ktab[2 * k + 1];
      } else {
        oa = group_off(g.k0 + k, sak, g.rk, g.D);
        ob = group_off(g.k0 + k, sbk, g.rk, g.D);
      }
#pragma unroll
      for (int i = 0; i < NLA; ++i)
        if (ra[i] >= 0) x.a[i] = ldc(g.A + ra[i] + oa);
#pragma unroll
      for (int i = 0; i < NLB; ++i)
        if (cb[i] >= 0) x.b[i] = ldc(g.B + cb[i] + ob);
    }
    return x;
  };
  // accumulators: the real and imaginary part of each tile, or the two
  // products of one part of one tile
  V acc0[NR][NC], acc1[NR][NC];
#pragma unroll
  for (int i = 0; i < NR; ++i)
#pragma unroll
    for (int j = 0; j < NC; ++j) {
      acc0[i][j] = V{0, 0, 0, 0};
      acc1[i][j] = V{0, 0, 0, 0};
    }
  // products of 4 contracted entries from row kr of the staged chunk
  auto products = [&](const Cx<T>* Ac, const Cx<T>* Bc, int32_t kr) {
    Cx<T> a[NR], bb[NC];
#pragma unroll
    for (int i = 0; i < NR; ++i) a[i] = Ac[(kr + lk) * PA + qr + 16 * i + l16];
#pragma unroll
    for (int j = 0; j < NC; ++j) bb[j] = Bc[(kr + lk) * PB + qc + 16 * j + l16];
    if constexpr (kParts) {
      acc0[0][0] = M::mac(a[0].re, imag ? bb[0].im : bb[0].re, acc0[0][0]);
      acc1[0][0] = M::mac(imag ? a[0].im : -a[0].im, imag ? bb[0].re : bb[0].im, acc1[0][0]);
    } else {
      // the four contributions in turn over the tiles: an accumulator is
      // used again only after every other one
#pragma unroll
      for (int i = 0; i < NR; ++i)
#pragma unroll
        for (int j = 0; j < NC; ++j) acc0[i][j] = M::mac(a[i].re, bb[j].re, acc0[i][j]);
#pragma unroll
      for (int i = 0; i < NR; ++i)
#pragma unroll
        for (int j = 0; j < NC; ++j) acc1[i][j] = M::mac(a[i].re, bb[j].im, acc1[i][j]);
#pragma unroll
      for (int i = 0; i < NR; ++i)
#pragma unroll
        for (int j = 0; j < NC; ++j) acc0[i][j] = M::mac(-a[i].im, bb[j].im, acc0[i][j]);
#pragma unroll
      for (int i = 0; i < NR; ++i)
#pragma unroll
        for (int j = 0; j < NC; ++j) acc1[i][j] = M::mac(a[i].im, bb[j].re, acc1[i][j]);
    }
  };
  Ops x = load(0);
  int32_t cur = 0;
  for (int32_t c0 = 0; c0 < g.kl; c0 += BK) {
    Cx<T>* Ac = As + cur * BK * PA;
    Cx<T>* Bc = Bs + cur * BK * PB;
#pragma unroll
    for (int i = 0; i < NLA; ++i) Ac[kk * PA + lr + LR * i] = x.a[i];
#pragma unroll
    for (int i = 0; i < NLB; ++i) Bc[kk * PB + lr + LR * i] = x.b[i];
    // a buffer is written again two chunks on, past the barrier that every
    // wavefront reaches only once it has read it
    __syncthreads();
    if (c0 + BK < g.kl) x = load(c0 + BK);
    // only the groups of 4 contracted entries this chunk holds (a short
    // contracted index, K = 3 or 9, would otherwise multiply zero padding)
    const int32_t kv = min(BK, g.kl - c0);
#pragma unroll 1
    for (int32_t j4 = 0; j4 < kv; j4 += 4) products(Ac, Bc, j4);
    cur ^= 1;
  }
  __syncthreads();  // the next block's offsets and chunks overwrite this one's
  // this wavefront's rows of C from C[b, m0 + qr, n0] (at most 32 rows: the
  // planner keeps 64 rows of C within one output range)
  const GlbOut<T> out(g.C + ((int64_t)b * g.nm + m0 + qr) * g.nn + n0);
  T lm = 0;
  if constexpr (kParts) {
    // register r of lane l of tile t at 256 t + 64 r + l of the first buffer
    static_assert(4 * 4 * 64 * sizeof(T) <= 2 * BK * PA * sizeof(Cx<T>), "exchange fits in As");
    T* xch = reinterpret_cast<T*>(As) + (wv & 3) * 256;
    if (imag) {
#pragma unroll
      for (int rr = 0; rr < 4; ++rr) xch[64 * rr + lane] = acc0[0][0][rr] + acc1[0][0][rr];
    }
    __syncthreads();
    if (!imag) {
      acc0[0][0] += acc1[0][0];
#pragma unroll
      for (int rr = 0; rr < 4; ++rr) acc1[0][0][rr] = xch[64 * rr + lane];
    }
    __syncthreads();
  }
  if (!imag) {
#pragma unroll
    for (int i = 0; i < NR; ++i)
#pragma unroll
      for (int j = 0; j < NC; ++j) {
        const int32_t nc = qc + 16 * j + l16;
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) {
          const int32_t mr = 16 * i + M::row(lane, rr);
          if (m0 + qr + mr < g.nm && n0 + nc < g.nn) {
            const T vr = acc0[i][j][rr] * g.scale, vi = acc1[i][j][rr] * g.scale;
            put(out, mr * g.nn + nc, Cx<T>{vr, vi});
            lm = fmax(lm, fmax(fabs(vr), fabs(vi)));
          }
        }
      }
  }
  return lm;
}

// One task of a STEP_GEMM (W = false) or STEP_GEMM64 step.  The blocks of a
// batch index are counted two rows of blocks at a time, column after column, so
// that consecutive blocks make up a larger region (four of 64 x 64: 128 x 128;
// two: 128 x 64; four of 32 x 32: 64 x 64, or 128 x 32 in a single column; two:
// 64 x 32), and a task of several blocks computes such regions: fewer gathers
// per product, and one round of barriers in place of several.  A task of
// single blocks (a step with few blocks, spread over the device) computes just
// that block.  The contracted offsets come from a table generated in LDS when
// the range fits, else they are decoded from the strides.
template <class T, bool W>
__device__ __attribute__((always_inline)) void gemm_tile(const DevProg& p, const StepDesc& s, int32_t tile_id, int32_t q,
                          Cx<T>* __restrict__ arena, uint8_t* smem, int32_t smem_bytes,
                          const States& st, T* s_red, int64_t* ph) {
  constexpr int32_t BM = W ? 64 : 32;
  const int32_t tid = task_tid();
  const int32_t rb = s.ranks & 255, rm = (s.ranks >> 8) & 255, rk = (s.ranks >> 16) & 255,
                rn = (s.ranks >> 24) & 255;
  // LDS: the step's strides, the contracted offsets, then gemm_block's own
  constexpr int32_t kStr = 128;  // the decoded groups' ranks are below 32
  constexpr int32_t kOwn = W ? (gemm_lds<T, 128, 128>() > gemm_lds<T, 128, 64>() ? gemm_lds<T, 128, 128>() : gemm_lds<T, 128, 64>())
                             : (gemm_lds<T, 64, 64>() > gemm_lds<T, 128, 32>() ? gemm_lds<T, 64, 64>() : gemm_lds<T, 128, 32>());
  static_assert(kOwn + kStr * 4 + 8 * 1024 <= kLdsLimit, "a region and 1024 contracted offsets fit");
  int32_t* str = reinterpret_cast<int32_t*>(smem + kOwn);
  int32_t* ktab = str + kStr;
  const int32_t kcap = (smem_bytes - kOwn - kStr * 4) / 8;
  const int32_t n_str = 2 * rb + rm + 2 * rk + rn;
  for (int32_t i = tid; i < n_str; i += kBlock) str[i] = p.strides[s.str + i];
  // this task: contracted range ks of the split, blocks [blk0, blk1) of the
  // nb * n_mb * n_nb blocks (s.tile blocks per task)
  const int32_t mb_nb = s.n_mb * s.n_nb;
  const int32_t nblk = s.nb * mb_nb;
  const int32_t per = s.tile;
  const int32_t base = (nblk + per - 1) / per;
  const int32_t ks = tile_id / base;
  const int32_t blk0 = (tile_id - ks * base) * per, blk1 = min(nblk, blk0 + per);
  const int32_t k0 = ks * s.kseg, k1 = min(s.nk, k0 + s.kseg), kl = k1 - k0;
  int64_t ec;
  const T scale = step_scale<T>(st, s.a, s.b, ec);
  const int64_t outs = (int64_t)s.nb * s.nm * s.nn;
  GemmCtx<T> g{(const GlbCx<T>*)(arena + s.home_a),
               (const GlbCx<T>*)(arena + s.home_b),
               (GlbCx<T>*)(s.n_ks > 1 ? arena + s.partial + (int64_t)ks * outs : arena + s.home_c),
               str, kl <= kcap ? ktab : nullptr, rb, rm, rk, rn, s.nm, s.nn, k0, kl, scale, smem,
               qdiv_of(q)};
  __syncthreads();
  if (g.ktab) {
    for (int32_t i = tid; i < kl; i += kBlock) {
      ktab[2 * i] = group_off(k0 + i, str + rb + rm, rk, g.D);
      ktab[2 * i + 1] = group_off(k0 + i, str + 2 * rb + rm + rk, rk, g.D);
    }
  }
  T lm = 0;
  int64_t tk = 0;
  if (ph) {
    tk = wall_clock64();
    ph[0] = tk - ph[3];
  }
  const int32_t paired = (s.n_mb & ~1) * s.n_nb;  // blocks in pairs of rows of blocks
  for (int32_t blk = blk0; blk < blk1;) {
    const int32_t b = blk / mb_nb;
    const int32_t r = blk - b * mb_nb;
    int32_t mblk, nbk;
    int32_t take = 1;
    if (r < paired) {
      const int32_t pr = r / (2 * s.n_nb), rest = r - pr * 2 * s.n_nb;
      mblk = 2 * pr + (rest & 1);
      nbk = rest >> 1;
      if ((rest & 1) == 0) {
        const bool four = W || s.n_nb > 1 ? nbk + 1 < s.n_nb : r + 4 <= paired;
        if (blk + 4 <= blk1 && four) take = 4;
        else if (blk + 2 <= blk1) take = 2;
      }
    } else {
      mblk = s.n_mb - 1;
      nbk = r - paired;
    }
    T m;
    const int32_t m0 = mblk * BM, n0 = nbk * BM;
    if constexpr (W) {
      if (take == 4) m = gemm_block<T, 128, 128>(g, b, m0, n0);
      else if (take == 2) m = gemm_block<T, 128, 64>(g, b, m0, n0);
      else m = gemm_block<T, 64, 64>(g, b, m0, n0);
    } else {
      if (take == 4 && s.n_nb > 1) m = gemm_block<T, 64, 64>(g, b, m0, n0);
      else if (take == 4) m = gemm_block<T, 128, 32>(g, b, m0, n0);
      else if (take == 2) m = gemm_block<T, 64, 32>(g, b, m0, n0);
      else m = gemm_block<T, 32, 32>(g, b, m0, n0);
    }
    lm = fmax(lm, m);
    blk += take;
  }
  if (ph) {
    const int64_t t = wall_clock64();
    ph[1] = t - tk;
    tk = t;
  }
  if (s.n_ks == 1) tile_publish<T>(p, s.c, tile_id, lm, ec, s_red);
  if (ph) ph[2] = wall_clock64() - tk;
}

// Outputs [part * kReduceChunk, ...) of a split step: C = sum over the n_ks
// partial results, in split order (the same bits on every run).
template <class T>
__device__ __attribute__((always_inline)) void reduce_step(const DevProg& p, const StepDesc& s, int32_t part, Cx<T>* arena,
                            const States& st, T* s_red) {
  const int64_t outs = (int64_t)s.nb * s.nm * s.nn;
  const int64_t o0 = (int64_t)part * kReduceChunk;
  const int64_t o1 = o0 + kReduceChunk < outs ? o0 + kReduceChunk : outs;
  const GlbCx<T>* P = (const GlbCx<T>*)(arena + s.partial);
  const GlbOut<T> C((GlbCx<T>*)(arena + s.home_c) + o0);
  T lm = 0;
  for (int64_t o = o0 + threadIdx.x; o < o1; o += kBlock) {
    T cr = 0, ci = 0;
    for (int32_t j = 0; j < s.n_ks; j += 8) {
      Cx<T> v[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        v[i] = Cx<T>{0, 0};
        if (j + i < s.n_ks) v[i] = ldc(P + (int64_t)(j + i) * outs + o);
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        cr += v[i].re;
        ci += v[i].im;
      }
    }
    put(C, (int32_t)(o - o0), Cx<T>{cr, ci});
    lm = fmax(lm, fmax(fabs(cr), fabs(ci)));
  }
  int64_t ec;
  step_scale<T>(st, s.a, s.b, ec);
  tile_publish<T>(p, s.c, part, lm, ec, s_red);
}

// ------------------------------------------------------------------ final

template <class T>
__device__ __attribute__((always_inline)) void knot_final(const DevProg& p, const KnotDesc& kd, Cx<T>* arena, Cx<T>* lds,
                           kn_scalar* zout, const States& st, int32_t slice) {
  // the first wavefront: lane l multiplies values l, l + 64, ... of the
  // components, the factors and q for each isolated spin, then the lanes'
  // products are multiplied pairwise (one thread for all of them: 9 us of a
  // 574-crossing knot's 218)
  const int32_t lane = task_tid();
  if (lane >= 64) return;
  const ImgHeader& h = *p.h;
  const Cx<double>* xe = p.weights + kd.w_off;
  const Cx<double>* xm = xe + kd.n_edges;
  Cx<double> z{1.0, 0.0};
  int64_t e = 0;
  const int32_t n_val = kd.n_comps + kd.n_factors + kd.n_iso;
  for (int32_t i = lane; i < n_val; i += 64) {
    Cx<double> x{(double)kd.q, 0.0};
    if (i < kd.n_comps) {
      const int32_t t = p.comps[kd.comp_off + i];
      const Cx<T> r = *tptr<T>(p.tens[t], arena, lds);
      int32_t sh;
      int64_t et;
      if (st.local(t)) st.get(t, sh, et);
      else st.get_late(t, sh, et);
      e += et;
      x = Cx<double>{(double)r.re, (double)r.im};
    } else if (i - kd.n_comps < kd.n_factors) {
      const Factor f = p.factors[kd.factor_off + i - kd.n_comps];
      x = f.kind == FAC_LOOP ? xe[f.id] : f.kind == FAC_CONST ? plan_consts(p, kd)[f.id] : xm[f.id];
      if (f.kind == FAC_LEAF) x.re += (double)(kd.q - 1);
      if (f.kind == FAC_PAIR) {  // equal fixed values: x_m, else 1
        int sa = slice, sb = slice;
        for (int r = 0; r < f.a; ++r) sa /= kd.q;
        for (int r = 0; r < f.b; ++r) sb /= kd.q;
        if (sa % kd.q != sb % kd.q) x = Cx<double>{1.0, 0.0};
      }
    }
    acc_mul(z, e, x);
  }
  for (int32_t m = 32; m >= 1; m >>= 1) {
    if (m >= n_val) continue;  // (those lanes' products are 1)
    const Cx<double> y{__shfl_xor(z.re, m, 64), __shfl_xor(z.im, m, 64)};
    e += __shfl_xor(e, m, 64);
    acc_mul(z, e, y);
  }
  if (lane != 0) return;
  kn_scalar out;
  if (__hip_atomic_load(&p.ctrl[CTRL_ERROR], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) {
    out.re = out.im = __builtin_nan("");
    out.exp2 = 0;
  } else {
    out.re = z.re;
    out.im = z.im;
    out.exp2 = (z.re == 0.0 && z.im == 0.0) ? 0 : e;
  }
  // a slice's value goes to the slice array; sum_slices adds them up
  if (kd.n_slices > 1) p.zslice[kd.out_slot + slice] = out;
  else zout[kd.out_slot] = out;
}

__device__ inline Cx<double> cdiv(Cx<double> a, Cx<double> b) {
  const double s = fmax(fabs(b.re), fabs(b.im));
  const Cx<double> bs{b.re / s, b.im / s};
  const double d = bs.re * bs.re + bs.im * bs.im;
  return {(a.re * bs.re + a.im * bs.im) / (d * s), (a.im * bs.re - a.re * bs.im) / (d * s)};
}

// d log Z / d J_e for every original edge of a gradient plan (after the
// reverse steps).  For the merged edge m in slot j of vertex tensor
// F_v(s_v, s_w1..) = prod_l T_ml(s_v, s_wl) (Eq. 5; a private s_v summed),
//   dF_v/dx_m = delta(s_v, s_wj) prod_{l != j} T_ml(s_v, s_wl),
// so d log S / d J_m = x_m sum_i dS/dF_v[i] dF_v/dx_m[i] / S, S the scalar of
// the vertex's component.  A spike factor x_m + q - 1 gives
// x_m / (x_m + q - 1), a loop factor x_e gives 1, and each original edge takes
// the value of its merged edge (x_m is the product of its members' e^{J}).
// One wavefront per vertex tensor; the whole workgroup calls this, after the
// persistent kernel (what it reads, the adjoints and their components' scalars
// with their states, is then in global memory).
template <class T>
__device__ void knot_gradient(const DevProg& p, const KnotDesc& kd, const Cx<T>* arena,
                              double* grad) {
  const ImgHeader& h = *p.h;
  const Cx<double>* xm = p.weights + kd.w_off + kd.n_edges;
  Cx<double>* mg = p.mgrad + kd.medge_off;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int q = kd.q;
  constexpr int kMaxSlots = 7;
  for (int v = wv; v < kd.n_vtx; v += kBlock / 64) {
    const VtxDesc vd = p.vtx[kd.vtx_off + v];
    if (vd.keep_center < 0 || vd.adjoint < 0 || vd.n_slots == 0) continue;
    const int ns = vd.n_slots;
    const int32_t* slot_me = p.vslot + vd.slot_off;
    Cx<double> x[kMaxSlots];
#pragma unroll
    for (int j = 0; j < kMaxSlots; ++j) x[j] = j < ns ? xm[slot_me[j]] : Cx<double>{1.0, 0.0};
    int32_t qn = 1;
    for (int j = 0; j < ns; ++j) qn *= q;
    // (adjoints of vertex tensors live in global memory)
    const TensorDesc td = p.tens[vd.adjoint];
    const Cx<T>* fb = arena + td.off;
    double ar[kMaxSlots], ai[kMaxSlots];
#pragma unroll
    for (int j = 0; j < kMaxSlots; ++j) ar[j] = ai[j] = 0.0;
    // entry i in F_v's order (kept centre leading, last slot fastest) sits at
    // sum of digit x stride in the adjoint's storage order
    const int32_t* astr = p.strides + vd.adj_str;
    const int32_t* sstr = astr + (vd.keep_center ? 1 : 0);
    for (int i = lane; i < td.size; i += 64) {
      int dig[kMaxSlots];
      int rem = i;
      int32_t off = 0;
#pragma unroll
      for (int j = kMaxSlots - 1; j >= 0; --j) {
        if (j < ns) {
          dig[j] = rem % q;
          rem /= q;
          off += dig[j] * sstr[j];
        } else {
          dig[j] = -1;
        }
      }
      const int centre = rem;  // kept centre (leading index); unused when private
      if (vd.keep_center) off += centre * astr[0];
      const Cx<T> f = fb[off];
#pragma unroll
      for (int j = 0; j < kMaxSlots; ++j) {
        if (j >= ns) continue;
        const int a = vd.keep_center ? centre : dig[j];
        if (dig[j] != a) continue;
        Cx<double> prod{(double)f.re, (double)f.im};
#pragma unroll
        for (int l = 0; l < kMaxSlots; ++l)
          if (l != j && l < ns && dig[l] == a) prod = cmul(prod, x[l]);
        ar[j] += prod.re;
        ai[j] += prod.im;
      }
    }
#pragma unroll
    for (int j = 0; j < kMaxSlots; ++j) {
      for (int o = 32; o >= 1; o >>= 1) {
        ar[j] += __shfl_xor(ar[j], o, 64);
        ai[j] += __shfl_xor(ai[j], o, 64);
      }
    }
    if (lane == 0) {
      const int64_t ef = p.ts[vd.adjoint].exp2;
      const int32_t root = p.comps[kd.comp_off + vd.comp];
      const Cx<T> r = arena[p.tens[root].off];
      const int64_t er = p.ts[root].exp2;
      const Cx<double> rs{(double)r.re, (double)r.im};
#pragma unroll
      for (int j = 0; j < kMaxSlots; ++j) {
        if (j >= ns) continue;
        Cx<double> g = cdiv(cmul(Cx<double>{ar[j], ai[j]}, x[j]), rs);
        g.re = ldexp(g.re, (int)(ef - er));
        g.im = ldexp(g.im, (int)(ef - er));
        mg[slot_me[j]] = g;
      }
    }
  }
  for (int i = tid; i < kd.n_factors; i += kBlock) {
    const Factor f = p.factors[kd.factor_off + i];
    if (f.kind == FAC_LEAF) {
      const Cx<double> x = xm[f.id];
      mg[f.id] = cdiv(x, Cx<double>{x.re + (double)(q - 1), x.im});
    }
  }
  __syncthreads();
  double* g = grad + 2 * (int64_t)kd.edge_off;
  for (int m = tid; m < kd.n_medges; m += kBlock) {
    const MEdge me = p.medges[kd.medge_off + m];
    const Cx<double> v = mg[m];
    for (int i = 0; i < me.n_members; ++i) {
      const int32_t e = p.members[me.member_off + i];
      g[2 * e] = v.re;
      g[2 * e + 1] = v.im;
    }
  }
  for (int i = tid; i < kd.n_factors; i += kBlock) {
    const Factor f = p.factors[kd.factor_off + i];
    if (f.kind == FAC_LOOP) {
      g[2 * f.id] = 1.0;
      g[2 * f.id + 1] = 0.0;
    }
  }
}

// ------------------------------------------------------------------ kernels

// Reset the runtime state of an image: control words, ready queue seeded
// with the knots' first groups, pending counters, tensor states; the results
// (every output scalar and slice value) start as NaN, so a knot whose final
// task never runs (the engine gave up on a queue slot) reads as NaN.
__global__ void clear_state(const uint8_t* __restrict__ img, uint8_t* __restrict__ state,
                            kn_scalar* __restrict__ zout) {
  const ImgHeader& h = *reinterpret_cast<const ImgHeader*>(img);
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const kn_scalar nan{__builtin_nan(""), __builtin_nan(""), 0};
  if (i < h.n_outputs) zout[i] = nan;
  if (i < h.n_zslice) reinterpret_cast<kn_scalar*>(state + h.o_zslice)[i] = nan;
  if (i < h.n_knots)
    reinterpret_cast<int32_t*>(state + h.o_uslice)[i] =
        reinterpret_cast<const KnotDesc*>(img + h.o_knots)[i].slice;
  int32_t* ctrl = reinterpret_cast<int32_t*>(state);
  if (i < CTRL_WORDS) ctrl[i] = (i == CTRL_TAIL) ? h.n_roots : 0;
  if (i < h.n_queue) {
    const int32_t* roots = reinterpret_cast<const int32_t*>(img + h.o_roots);
    reinterpret_cast<int32_t*>(state + h.o_queue)[i] = i < h.n_roots ? roots[i] : -1;
  }
  if (i < h.n_groups) {
    const GroupDesc* g = reinterpret_cast<const GroupDesc*>(img + h.o_groups);
    reinterpret_cast<int32_t*>(state + h.o_pending)[i] = g[i].n_pred;
  }
  if (i < h.n_tensors) {
    TensorState* ts = reinterpret_cast<TensorState*>(state + h.o_tstate);
    ts[i].shift = kShiftNone;
    ts[i].pad = 0;
    ts[i].exp2 = 0;
  }
}

// Z of a sliced plan = the sum of its slices' values: one thread per knot
// descriptor, the first slice of each plan adds up the plan's slices (they
// are consecutive), aligned to the largest exponent.
__global__ void sum_slices(const uint8_t* __restrict__ img, uint8_t* __restrict__ state,
                           kn_scalar* __restrict__ zout) {
  const ImgHeader& h = *reinterpret_cast<const ImgHeader*>(img);
  const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= h.n_knots) return;
  const KnotDesc* kds = reinterpret_cast<const KnotDesc*>(img + h.o_knots);
  const KnotDesc kd = kds[i];
  if (kd.n_slices <= 1 || kd.slice != 0) return;  // the plan's first chain adds its slices
  const kn_scalar* zs = reinterpret_cast<const kn_scalar*>(state + h.o_zslice) + kd.out_slot;
  int64_t emax = INT64_MIN;
  bool bad = false;
  for (int32_t j = 0; j < kd.n_slices; ++j) {
    const kn_scalar z = zs[j];
    if (!isfinite(z.re) || !isfinite(z.im)) bad = true;
    if (z.re != 0.0 || z.im != 0.0) emax = max(emax, z.exp2);
  }
  kn_scalar out{0.0, 0.0, 0};
  if (bad) {
    out.re = out.im = __builtin_nan("");
  } else if (emax != INT64_MIN) {
    double re = 0.0, im = 0.0;
    for (int32_t j = 0; j < kd.n_slices; ++j) {
      const kn_scalar z = zs[j];
      const int64_t d = z.exp2 - emax;  // <= 0
      if (d < -1100) continue;
      re += ldexp(z.re, (int)d);
      im += ldexp(z.im, (int)d);
    }
    const double m = fmax(fabs(re), fabs(im));
    if (m > 0.0) {
      int s;
      frexp(m, &s);
      out.re = ldexp(re, -s);
      out.im = ldexp(im, -s);
      out.exp2 = emax + s;
    }
  }
  zout[kd.plan_slot] = out;
}

// d log Z / d J of every knot of a gradient image: one workgroup per knot,
// launched after the persistent kernel on the same stream.
template <class T>
__global__ __launch_bounds__(kBlock) void gradient_kernel(const uint8_t* __restrict__ img,
                                                          uint8_t* __restrict__ state,
                                                          Cx<T>* __restrict__ arena,
                                                          double* __restrict__ grad) {
  const DevProg p = make_prog(img, state);
  const KnotDesc kd = p.knots[blockIdx.x];
  if (!kd.grad) return;
  knot_gradient<T>(p, kd, arena, grad);
}

// The checking build (KN_DEVICE_CHECKS) checks each task and its steps just
// before running it (checks.h) and skips a task that fails; it also fills the
// guard zone after the arena before a launch and checks it after.
#ifdef KN_DEVICE_CHECKS
constexpr bool kChecks = true;
#else
constexpr bool kChecks = false;
#endif

// Record an error: the first code wins, with the task, step and detail.
__device__ inline void report(const DevProg& p, int32_t code, int32_t task, int32_t step,
                              int32_t info) {
  int32_t expect = 0;
  if (__hip_atomic_compare_exchange_strong(&p.ctrl[CTRL_ERROR], &expect, code, __ATOMIC_RELAXED,
                                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
    __hip_atomic_store(&p.ctrl[CTRL_ERR_TASK], task, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&p.ctrl[CTRL_ERR_STEP], step, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&p.ctrl[CTRL_ERR_INFO], info, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// Checks of task ti before it runs (whole workgroup): thread 0 checks the
// record, then the threads share out its steps; the lowest failing step is
// reported.  True when the task may run.
template <class T>
__device__ bool task_ok(const DevProg& p, int32_t ti, int32_t* s_code, int32_t* s_step) {
  const ImageView v{p.h, p.tasks, p.groups, p.knots, p.tens, p.steps, p.vtx, p.strides, p.comps};
  const int64_t lds_elems = p.h->lds_bytes / (int64_t)sizeof(Cx<T>);
  if (threadIdx.x == 0) {
    *s_code = task_record_check(v, ti, lds_elems);
    *s_step = INT32_MAX;
  }
  __syncthreads();
  if (*s_code != CHK_OK) {
    if (threadIdx.x == 0) report(p, *s_code, ti, -1, 0);
    __syncthreads();
    return false;
  }
  const TaskDesc td = p.tasks[ti];
  const int32_t q = p.knots[td.knot].q;
  const int32_t n = td.kind == TASK_SERIAL ? td.count : 1;
  for (int32_t i = threadIdx.x; i < n; i += kBlock) {
    const StepDesc& d = p.steps[td.first + i];
    int32_t rc = step_check(d, p.tens, p.h->n_tensors, p.strides, p.h->n_strides, q,
                            p.h->arena_elems, lds_elems);
    if (td.kind == TASK_SERIAL && d.mode != STEP_SERIAL) rc = CHK_TASK;
    if (rc != CHK_OK) atomicMin(s_step, td.first + i);
  }
  __syncthreads();
  const int32_t bad = *s_step;
  if (bad != INT32_MAX && threadIdx.x == 0) {
    const StepDesc& d = p.steps[bad];
    int32_t rc = step_check(d, p.tens, p.h->n_tensors, p.strides, p.h->n_strides, q,
                            p.h->arena_elems, lds_elems);
    if (rc == CHK_OK) rc = CHK_TASK;
    report(p, rc, ti, bad, 0);
  }
  __syncthreads();
  return bad == INT32_MAX;
}

// Guard zone after the arena: filled before a launch, checked after it.
__global__ void fill_guard(uint8_t* __restrict__ ws) {
  const ImgHeader& h = *reinterpret_cast<const ImgHeader*>(ws);
  uint32_t* g = reinterpret_cast<uint32_t*>(ws + h.guard_off);
  for (int32_t i = threadIdx.x; i < (int32_t)(kGuardBytes / 4); i += blockDim.x) g[i] = kGuardWord;
}

__global__ void check_guard(const uint8_t* __restrict__ ws, uint8_t* __restrict__ state) {
  const ImgHeader& h = *reinterpret_cast<const ImgHeader*>(ws);
  const uint32_t* g = reinterpret_cast<const uint32_t*>(ws + h.guard_off);
  DevProg p;
  p.ctrl = reinterpret_cast<int32_t*>(state);
  for (int32_t i = threadIdx.x; i < (int32_t)(kGuardBytes / 4); i += blockDim.x)
    if (g[i] != kGuardWord) report(p, CHK_GUARD, -1, -1, i);
}

// Bound on the wait for a queue slot, in ticks of the 100 MHz device clock
// (20 s, far beyond any launch's critical path): a slot that is never filled
// (a planner bug) ends the kernel with the error flag set instead of hanging
// the device; the knots left unfinished keep the NaN that clear_state wrote.
constexpr int64_t kWaitTicks = 20LL * 100000000LL;

extern __shared__ __align__(16) uint8_t kn_dyn_smem[];

template <class T>
__global__ __launch_bounds__(kBlock, 2) void engine(const uint8_t* __restrict__ img,
                                                 uint8_t* __restrict__ state,
                                                 Cx<T>* __restrict__ arena,
                                                 const double* __restrict__ J,
                                                 kn_scalar* __restrict__ zout,
                                                 TraceRec* __restrict__ trace) {
  __shared__ int32_t s_task;
  __shared__ T s_red[kBlock / 64];
  __shared__ int64_t s_ph[4];
  __shared__ int32_t s_chk[2];
  int32_t* s_tab = reinterpret_cast<int32_t*>(kn_dyn_smem + kLdsTab);
  int32_t* s_shift = reinterpret_cast<int32_t*>(kn_dyn_smem + kLdsShift);
  int64_t* s_exp = reinterpret_cast<int64_t*>(kn_dyn_smem + kLdsExp);
  FlatRec* s_rec = reinterpret_cast<FlatRec*>(kn_dyn_smem + kLdsRec);
  Cx<T>* lds = reinterpret_cast<Cx<T>*>(kn_dyn_smem + kLdsArena);
  const DevProg p = make_prog(img, state);
  const int32_t n_queue = p.h->n_queue;
  const int tid = threadIdx.x;
  for (;;) {
    int64_t t_claim = 0;
    if (tid == 0) {
      if (trace) t_claim = wall_clock64();
      const int32_t slot = atomicAdd(&p.ctrl[CTRL_HEAD], 1);
      int32_t t = -1;
      if (slot < n_queue) {
        int32_t nap = 1;
        const int64_t t_wait = wall_clock64();
        while ((t = __hip_atomic_load(&p.queue[slot], __ATOMIC_RELAXED,
                                      __HIP_MEMORY_SCOPE_AGENT)) < 0) {
          if (nap < 16) {
            __builtin_amdgcn_s_sleep(1);
            ++nap;
          } else {
            __builtin_amdgcn_s_sleep(8);
            // after an error the slot may never be filled: give up at once
            if (__hip_atomic_load(&p.ctrl[CTRL_ERROR], __ATOMIC_RELAXED,
                                  __HIP_MEMORY_SCOPE_AGENT) != 0)
              break;
          }
          if (wall_clock64() - t_wait > kWaitTicks) {
            report(p, CHK_QUEUE_WAIT, -1, -1, slot);
            break;
          }
        }
      }
      s_task = t;
      // One acquire for the workgroup, whose wavefronts share their L1; the
      // barrier orders the others' loads after it.  These cache operations are
      // served one after another per XCD, 50 ns each: with one per wavefront
      // (and one to release) a task spent up to 28 us on them when all
      // compute units were busy, 3 us so.
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    }
    __syncthreads();
    const int32_t ti = s_task;
    __syncthreads();
    if (ti < 0) break;
    const int64_t t_start = (trace && tid == 0) ? wall_clock64() : 0;
    const TaskDesc td = p.tasks[ti];
    // a sliced unit that starts its next slice after this task (its final task)
    int32_t next_slice = -1;
    // the checking build skips a task that fails its checks and only
    // publishes it, so the launch still drains
    const bool run = !kChecks || task_ok<T>(p, ti, &s_chk[0], &s_chk[1]);
    if (!run) {
      // skipped: it writes nothing, and its knot's result stays NaN
    } else if (td.kind == TASK_SERIAL) {
      const KnotDesc kd = p.knots[td.knot];
      const int32_t slice = p.uslice[td.knot];
      const States st{p.ts, s_shift, s_exp, td.state_lo, min(td.state_len, kStateCap)};
      // an output's shift is the maximum over its step's units
      for (int32_t i = tid; i < st.len; i += kBlock) s_shift[i] = kShiftNone;
      __syncthreads();
      int64_t ph_buf[4] = {0, 0, 0, 0};
      int64_t* ph = (trace && tid == 0) ? ph_buf : nullptr;
      if (td.flags & TF_SETUP) {
        // (the staging area is free while the vertex tensors are built)
        knot_setup<T>(p, kd, arena, lds, (LdsCx<double>*)(kn_dyn_smem + kLdsArena + p.h->lds_bytes),
                      stage_bytes(p.h->lds_bytes) / (int32_t)sizeof(Cx<double>), J, st, slice);
        __syncthreads();
      }
      if (ph) ph[0] = wall_clock64() - t_start;
      serial_steps<T>(p, td.first, td.count, kd.q, arena, lds, reinterpret_cast<int2*>(s_tab),
                      s_rec, st, td.state_len, ph);
      if (td.flags & TF_FINAL) knot_final<T>(p, kd, arena, lds, zout, st, slice);
      if (ph)
        for (int i = 0; i < 4; ++i) s_ph[i] = ph[i];
      // states of this task's tensors go back to global memory for later groups
      for (int32_t i = tid; i < st.len; i += kBlock) {
        p.ts[st.lo + i].shift = s_shift[i];
        p.ts[st.lo + i].exp2 = s_exp[i];
      }
      // the last task of a slice whose chain has more: every group and tensor
      // of the unit is done with, so its counters and tensor states are reset
      // for the next slice here (published with this task's release below)
      if ((td.flags & TF_FINAL) && kd.n_slices > 1 && slice + kd.slice_step < kd.n_slices) {
        next_slice = slice + kd.slice_step;
        __syncthreads();
        for (int32_t g = tid; g < kd.n_groups; g += kBlock)
          p.pending[kd.group_off + g] = p.groups[kd.group_off + g].n_pred;
        for (int32_t t = tid; t < kd.n_tensors; t += kBlock) {
          p.ts[kd.tensor_off + t].shift = kShiftNone;
          p.ts[kd.tensor_off + t].exp2 = 0;
        }
        if (tid == 0) p.uslice[td.knot] = next_slice;
      }
    } else {
      const States st{p.ts, s_shift, s_exp, 0, 0};
      // traced launches: thread 0 writes the phases straight into s_ph
      int64_t* ph = (trace && tid == 0) ? s_ph : nullptr;
      if (ph) {
        for (int i = 0; i < 3; ++i) ph[i] = 0;
        ph[3] = t_start;
      }
      const StepDesc sd = p.steps[td.first];
      const int32_t q = p.knots[td.knot].q;
      const int32_t dyn = kLdsLimit;
      if (td.kind == TASK_REDUCE)
        reduce_step<T>(p, sd, td.count, arena, st, s_red);
      else if (sd.mode == STEP_GEMM)
        gemm_tile<T, false>(p, sd, td.count, q, arena, kn_dyn_smem, dyn, st, s_red, ph);
      else if (sd.mode == STEP_GEMM64)
        gemm_tile<T, true>(p, sd, td.count, q, arena, kn_dyn_smem, dyn, st, s_red, ph);
      else
        tile_step<T>(p, sd, td.count, q, arena, kn_dyn_smem, dyn, st, s_red, ph);
      if (ph) ph[3] = 0;
    }
    // ---- publish; the last task of a group releases the knot's next group.
    // Every wavefront waits for its own stores to complete: the barrier does
    // not wait for them, and the release below, by one wavefront for all,
    // only waits for that wavefront's.
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid < 64) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      int32_t n_enq = 0, first = 0, base = 0;
      if (tid == 0) {
        // the group to start: the unit's first again, for its next slice, or
        // the next one where this was the last task of its predecessor
        int32_t start = -1;
        const int32_t next = p.groups[td.group].next;
        if (next_slice >= 0) start = p.knots[td.knot].group_off;
        else if (next >= 0 && __hip_atomic_fetch_add(&p.pending[next], -1, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT) == 1)
          start = next;
        if (start >= 0) {
          const GroupDesc g = p.groups[start];
          n_enq = g.n_tasks;
          first = g.first_task;
          base = atomicAdd(&p.ctrl[CTRL_TAIL], n_enq);
        }
        if (trace) {
          TraceRec r{t_claim, t_start, wall_clock64(), ti, (int32_t)blockIdx.x, {0, 0, 0, 0}};
          for (int i = 0; i < 4; ++i) r.ph[i] = s_ph[i];
          trace[ti] = r;
        }
      }
      n_enq = __builtin_amdgcn_readfirstlane(n_enq);
      if (n_enq) {
        first = __builtin_amdgcn_readfirstlane(first);
        base = __builtin_amdgcn_readfirstlane(base);
        // the other tasks of the finished group, through its counter
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "agent");
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        for (int32_t i = tid; i < n_enq; i += 64)
          __hip_atomic_store(&p.queue[base + i], first + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
  }
}

// ------------------------------------------------------------------ host side

// Pool of host buffers for batch images.  Page-locked memory (hipHostMalloc)
// makes an image upload a DMA transfer with no staging copy on the CPU; it is
// slow to allocate, so buffers are kept and reused (best fit by capacity).
// Without a usable device the buffers are ordinary heap memory.
namespace {

std::mutex g_buf_mu;
std::multimap<size_t, std::pair<uint8_t*, bool>> g_buf_free;  // capacity -> (buffer, pinned)

}  // namespace

uint8_t* host_buf_get(size_t bytes, size_t* capacity, bool* pinned) {
  {
    std::lock_guard<std::mutex> lock(g_buf_mu);
    auto it = g_buf_free.lower_bound(bytes);
    if (it != g_buf_free.end() && it->first <= 2 * bytes + (1u << 20)) {
      *capacity = it->first;
      *pinned = it->second.second;
      uint8_t* p = it->second.first;
      g_buf_free.erase(it);
      return p;
    }
  }
  const size_t cap = (std::max<size_t>(bytes, 1) + (1u << 20) - 1) & ~size_t((1u << 20) - 1);
  void* p = nullptr;
  if (hipHostMalloc(&p, cap, hipHostMallocDefault) == hipSuccess && p) {
    *capacity = cap;
    *pinned = true;
    return static_cast<uint8_t*>(p);
  }
  (void)hipGetLastError();  // no device: fall back to the heap
  p = std::malloc(cap);
  if (!p) return nullptr;
  *capacity = cap;
  *pinned = false;
  return static_cast<uint8_t*>(p);
}

void host_buf_put(uint8_t* p, size_t capacity, bool pinned) {
  if (!p) return;
  std::lock_guard<std::mutex> lock(g_buf_mu);
  g_buf_free.emplace(capacity, std::make_pair(p, pinned));
  // keep the pool bounded: drop the largest buffers beyond 8
  while (g_buf_free.size() > 8) {
    auto last = std::prev(g_buf_free.end());
    if (last->second.second) (void)hipHostFree(last->second.first);
    else std::free(last->second.first);
    g_buf_free.erase(last);
  }
}

namespace {

int device_cus() {
  static int cus = 0;
  static std::once_flag once;
  std::call_once(once, [] {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) dev = 0;
    int v = 0;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v <= 0)
      v = 256;
    cus = v;
  });
  return cus;
}

template <class T>
kn_status launch_engine(const ImgHeader& h, uint8_t* ws, hipStream_t st, const double* J,
                        kn_scalar* z, double* grad, int32_t grid_override, TraceRec* trace) {
  const size_t dyn = kLdsLimit;
  static std::once_flag once;
  static bool attr_ok = true;
  std::call_once(once, [] {
    attr_ok = hipFuncSetAttribute(reinterpret_cast<const void*>(engine<T>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize,
                                  kLdsLimit) == hipSuccess;
  });
  if (!attr_ok) return KN_E_DEVICE;
  // default: one workgroup per compute unit (measured faster than filling
  // each CU with as many as fit: a workgroup running a knot's critical chain
  // then has its CU to itself)
  int32_t grid = grid_override;
  if (grid <= 0) grid = device_cus();
  if (grid > h.n_queue) grid = h.n_queue;
  if (grid < 1) grid = 1;
  hipLaunchKernelGGL(engine<T>, dim3(grid), dim3(kBlock), dyn, st, ws, ws + h.state_off,
                     reinterpret_cast<Cx<T>*>(ws + h.arena_off), J, z, trace);
  if (hipGetLastError() != hipSuccess) return KN_E_DEVICE;
  if (grad) {
    hipLaunchKernelGGL(gradient_kernel<T>, dim3(h.n_knots), dim3(kBlock), 0, st, ws,
                       ws + h.state_off, reinterpret_cast<Cx<T>*>(ws + h.arena_off), grad);
    if (hipGetLastError() != hipSuccess) return KN_E_DEVICE;
  }
  if (h.sliced) {
    hipLaunchKernelGGL(sum_slices, dim3((h.n_knots + 255) / 256), dim3(256), 0, st, ws,
                       ws + h.state_off, z);
    if (hipGetLastError() != hipSuccess) return KN_E_DEVICE;
  }
  return KN_OK;
}

kn_status launch(const ImgHeader& h, uint8_t* ws, hipStream_t st, const double* J,
                 kn_scalar* z, double* grad, int32_t grid_override, TraceRec* trace = nullptr) {
  int64_t n_clear = CTRL_WORDS;
  n_clear = std::max<int64_t>(n_clear, h.n_tasks);
  n_clear = std::max<int64_t>(n_clear, h.n_groups);
  n_clear = std::max<int64_t>(n_clear, h.n_tensors);
  n_clear = std::max<int64_t>(n_clear, h.n_knots);
  n_clear = std::max<int64_t>(n_clear, h.n_queue);
  n_clear = std::max<int64_t>(n_clear, h.n_zslice);
  hipLaunchKernelGGL(clear_state, dim3((unsigned)((n_clear + 255) / 256)), dim3(256), 0, st, ws,
                     ws + h.state_off, z);
  if (hipGetLastError() != hipSuccess) return KN_E_DEVICE;
  if (kChecks) {
    hipLaunchKernelGGL(fill_guard, dim3(1), dim3(256), 0, st, ws);
    if (hipGetLastError() != hipSuccess) return KN_E_DEVICE;
  }
  const kn_status rc = h.precision == 1
                           ? launch_engine<float>(h, ws, st, J, z, grad, grid_override, trace)
                           : launch_engine<double>(h, ws, st, J, z, grad, grid_override, trace);
  if (rc != KN_OK || !kChecks) return rc;
  hipLaunchKernelGGL(check_guard, dim3(1), dim3(256), 0, st, ws, ws + h.state_off);
  if (hipGetLastError() != hipSuccess) return KN_E_DEVICE;
  return KN_OK;
}

bool aligned256(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 255) == 0; }

}  // namespace
}  // namespace kn

using namespace kn;

namespace {

kn_status contract_plan(const kn_plan* p, const double* J, void* workspace,
                        size_t workspace_bytes, void* stream, kn_scalar* z_dev, double* grad) {
  if (!p || !workspace || !z_dev) return KN_E_INVALID;
  const Bytes& image = plan_image(p);
  if (image.empty()) return KN_E_BUDGET;
  if (J && p->k.jones_only) return KN_E_UNSUPPORTED;
  if (!aligned256(workspace)) return KN_E_INVALID;
  const ImgHeader& h = *reinterpret_cast<const ImgHeader*>(image.data());
  if ((int64_t)workspace_bytes < h.workspace_bytes) return KN_E_BUDGET;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  if (hipMemcpyAsync(workspace, image.data(), (size_t)h.image_bytes, hipMemcpyHostToDevice, st) !=
      hipSuccess)
    return KN_E_DEVICE;
  return launch(h, reinterpret_cast<uint8_t*>(workspace), st, J, z_dev, grad, 0);
}

}  // namespace

extern "C" kn_status kn_contract(const kn_plan* p, const double* J, void* workspace,
                                 size_t workspace_bytes, void* stream, kn_scalar* z_dev) {
  return contract_plan(p, J, workspace, workspace_bytes, stream, z_dev, nullptr);
}

// ------------------------------------------------------------------ fixed scratch
// Workspace of kn_contract_noalloc: one library-owned array per device, in
// place of the caller's workspace, so that the call allocates nothing.  In
// host code `scratch` names a host-side stand-in, never the device memory:
// its device address is looked up once per device (hipGetSymbolAddress) and
// only that address is handed to the kernels.
static __device__ __align__(256) uint8_t scratch[KN_NOALLOC_MAX_BYTES];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_dev[kMaxDevices];  // device address of `scratch` per device (null: not looked up)

// Device address of the current device's copy of `scratch`.
kn_status scratch_address(void** out) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return KN_E_DEVICE;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_dev[dev]) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) {
      (void)hipGetLastError();
      return KN_E_DEVICE;
    }
    g_scratch_dev[dev] = ptr;
  }
  *out = g_scratch_dev[dev];
  return KN_OK;
}

}  // namespace

extern "C" kn_status kn_contract_noalloc(const kn_plan* p, const double* J, void* stream,
                                         kn_scalar* z_dev) {
  if (!p || !z_dev) return KN_E_INVALID;
  const Bytes& image = plan_image(p);
  if (image.empty()) return KN_E_BUDGET;
  const ImgHeader& h = *reinterpret_cast<const ImgHeader*>(image.data());
  if (h.workspace_bytes > (int64_t)KN_NOALLOC_MAX_BYTES) return KN_E_BUDGET;
  void* ws = nullptr;
  const kn_status rc = scratch_address(&ws);
  if (rc != KN_OK) return rc;
  return contract_plan(p, J, ws, KN_NOALLOC_MAX_BYTES, stream, z_dev, nullptr);
}

extern "C" kn_status kn_batch_create(const kn_plan* const* plans, int32_t n, kn_batch** out) {
  if (!out) return KN_E_INVALID;
  *out = nullptr;
  if (!plans || n <= 0) return KN_E_INVALID;
  std::vector<const PlanKnot*> ks;
  bool jones_only = false, gradient = true;
  for (int32_t i = 0; i < n; ++i) {
    if (!plans[i] || !plans[i]->laid_out) return KN_E_INVALID;
    if (plans[i]->k.precision != plans[0]->k.precision) return KN_E_INVALID;
    jones_only |= plans[i]->k.jones_only;
    gradient &= plans[i]->k.gradient;
    ks.push_back(&plans[i]->k);
  }
  kn_batch* b = new (std::nothrow) kn_batch();
  if (!b) return KN_E_NOMEM;
  try {
    const int64_t nb = build_image_into(
        ks, [&](size_t bytes) { return b->image.allocate(bytes); }, nullptr);
    if (nb < 0) {
      delete b;
      return nb == -2 ? KN_E_NOMEM : KN_E_BUDGET;
    }
    b->precision = plans[0]->k.precision;
    b->jones_only = jones_only;
    b->gradient = gradient;
    int64_t off = 0;
    double flops = 0, bytes = 0;
    for (int32_t i = 0; i < n; ++i) {
      b->edge_offset.push_back(off);
      off += plans[i]->k.n_edges;
      flops += plans[i]->stats.flops;
      bytes += plans[i]->stats.bytes;
    }
    const ImgHeader& h = *reinterpret_cast<const ImgHeader*>(b->image.data());
    b->stats.workspace_bytes = (uint64_t)h.workspace_bytes;
    b->stats.image_bytes = (uint64_t)h.image_bytes;
    b->stats.n_tasks = h.n_tasks;
    b->stats.n_knots = n;
    b->stats.flops = flops;
    b->stats.bytes = bytes;
    b->stats.total_edges = off;
    b->stats.grid = 0;
  } catch (const std::bad_alloc&) {
    delete b;
    return KN_E_NOMEM;
  }
  *out = b;
  return KN_OK;
}

extern "C" kn_status kn_batch_info(const kn_batch* b, kn_batch_stats* out) {
  if (!b || !out) return KN_E_INVALID;
  *out = b->stats;
  int32_t grid = b->grid_override > 0 ? b->grid_override : 0;
  out->grid = grid;
  return KN_OK;
}

extern "C" kn_status kn_batch_edge_offset(const kn_batch* b, int32_t i, int64_t* off) {
  if (!b || !off || i < 0 || i >= (int32_t)b->edge_offset.size()) return KN_E_INVALID;
  *off = b->edge_offset[i];
  return KN_OK;
}

extern "C" kn_status kn_batch_upload(const kn_batch* b, void* workspace, size_t workspace_bytes,
                                     void* stream) {
  if (!b || !workspace) return KN_E_INVALID;
  if (!aligned256(workspace)) return KN_E_INVALID;
  const ImgHeader& h = *reinterpret_cast<const ImgHeader*>(b->image.data());
  if ((int64_t)workspace_bytes < h.workspace_bytes) return KN_E_BUDGET;
  if (hipMemcpyAsync(workspace, b->image.data(), (size_t)h.image_bytes, hipMemcpyHostToDevice,
                     reinterpret_cast<hipStream_t>(stream)) != hipSuccess)
    return KN_E_DEVICE;
  return KN_OK;
}

namespace {

kn_status contract_batch(const kn_batch* b, const double* J, void* workspace,
                         size_t workspace_bytes, void* stream, kn_scalar* z_dev, double* grad) {
  if (!b || !workspace || !z_dev) return KN_E_INVALID;
  if (J && b->jones_only) return KN_E_UNSUPPORTED;
  if (!aligned256(workspace)) return KN_E_INVALID;
  const ImgHeader& h = *reinterpret_cast<const ImgHeader*>(b->image.data());
  if ((int64_t)workspace_bytes < h.workspace_bytes) return KN_E_BUDGET;
  if (b->trace && b->trace_bytes < (size_t)h.n_tasks * sizeof(TraceRec)) return KN_E_BUDGET;
  return launch(h, reinterpret_cast<uint8_t*>(workspace), reinterpret_cast<hipStream_t>(stream), J,
                z_dev, grad, b->grid_override, reinterpret_cast<TraceRec*>(b->trace));
}

}  // namespace

extern "C" kn_status kn_batch_contract(const kn_batch* b, const double* J, void* workspace,
                                       size_t workspace_bytes, void* stream, kn_scalar* z_dev) {
  return contract_batch(b, J, workspace, workspace_bytes, stream, z_dev, nullptr);
}

extern "C" kn_status kn_batch_contract_backward(const kn_batch* b, const double* J,
                                                void* workspace, size_t workspace_bytes,
                                                void* stream, kn_scalar* z_dev, double* grad_dev) {
  if (!b || !grad_dev) return KN_E_INVALID;
  if (!b->gradient) return KN_E_UNSUPPORTED;
  return contract_batch(b, J, workspace, workspace_bytes, stream, z_dev, grad_dev);
}

extern "C" kn_status kn_batch_image(const kn_batch* b, const void** data, size_t* bytes) {
  if (!b || !data || !bytes) return KN_E_INVALID;
  *data = b->image.data();
  *bytes = b->image.size();
  return KN_OK;
}

extern "C" kn_status kn_batch_set_grid(kn_batch* b, int32_t grid) {
  if (!b || grid < 0) return KN_E_INVALID;
  b->grid_override = grid;
  return KN_OK;
}

extern "C" kn_status kn_batch_set_trace(kn_batch* b, void* trace_dev, size_t bytes) {
  if (!b) return KN_E_INVALID;
  b->trace = trace_dev;
  b->trace_bytes = trace_dev ? bytes : 0;
  return KN_OK;
}

extern "C" void kn_batch_free(kn_batch* b) { delete b; }

extern "C" kn_status kn_backward_workspace(const kn_plan* p, uint64_t* bytes) {
  if (!p || !bytes) return KN_E_INVALID;
  if (!p->k.gradient) return KN_E_UNSUPPORTED;
  *bytes = p->stats.workspace_bytes;
  return KN_OK;
}

extern "C" kn_status kn_contract_backward(const kn_plan* p, const double* J, void* workspace,
                                          size_t workspace_bytes, void* stream, kn_scalar* z_dev,
                                          double* grad_dev) {
  if (!p || !grad_dev) return KN_E_INVALID;
  if (!p->k.gradient) return KN_E_UNSUPPORTED;
  return contract_plan(p, J, workspace, workspace_bytes, stream, z_dev, grad_dev);
}

// ------------------------------------------------------------------ status

extern "C" int32_t kn_device_checks(void) { return kChecks ? 1 : 0; }

extern "C" kn_status kn_workspace_status(const void* workspace, void* stream, int32_t* status) {
  if (!workspace || !status) return KN_E_INVALID;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  ImgHeader h;
  int32_t w[CTRL_ERR_INFO + 1];
  if (hipMemcpyAsync(&h, workspace, sizeof(h), hipMemcpyDeviceToHost, st) != hipSuccess ||
      hipStreamSynchronize(st) != hipSuccess)
    return KN_E_DEVICE;
  if (h.magic != kMagic) return KN_E_INVALID;
  if (hipMemcpyAsync(w, reinterpret_cast<const uint8_t*>(workspace) + h.state_off, sizeof(w),
                     hipMemcpyDeviceToHost, st) != hipSuccess ||
      hipStreamSynchronize(st) != hipSuccess)
    return KN_E_DEVICE;
  status[0] = w[CTRL_ERROR];
  status[1] = w[CTRL_ERR_TASK];
  status[2] = w[CTRL_ERR_STEP];
  status[3] = w[CTRL_ERR_INFO];
  return KN_OK;
}
