// gfx950 kernels of the LQ-SGD compressor (Algorithm 1 of the paper, loop body).
//
// Three streaming sweeps over the W x (rows x cols) gradient data, each one
// batched launch over all layers and workers, and small kernels on the
// rows x r / cols x r factors between them:
//
//   add_project   M = G + E (stored over E), P partials = M Q        12 B / element
//   orth          sum partials, Gram-Schmidt, absmax                 factors only
//   exchange(P)   log-quantise, pack, dequantise, mean over workers  factors only
//   back_project  Q partials = M^T P-bar                              4 B / element
//   reduce_q      sum partials, absmax                               factors only
//   exchange(Q)   as exchange(P)                                     factors only
//   residual      E = M - P-bar Q-bar^T (and G-hat once per layer)    8 B / element
//
// Lanes own columns in every sweep (one float4 per lane per row: a wavefront
// reads 1 KiB of a row per instruction; one column per lane where rows are at
// most 64 columns, no multiple of four of them); the r-wide factor slice of a lane's
// columns lives in registers; rows of the other factor are wave-uniform.
// All reductions have a fixed order, so results are bit-identical run to run.
#include "lqsgd_kernels.h"

#include <hip/hip_cooperative_groups.h>

#include <algorithm>
#include <cfloat>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <type_traits>

// The kernels are templates and most of the build is their instantiation, so the file is compiled
// several times side by side, each time with the launchers of one part (LQSGD_PART = 0 .. 5) and
// with them the kernels that those launch.  Without the macro it is one whole translation unit.
#ifdef LQSGD_PART
#define LQSGD_HAS(part) (LQSGD_PART == (part))
#else
#define LQSGD_HAS(part) 1
#endif

#if LQSGD_HAS(0)
// Blocks of lqsgd_step_static (see static_scratch() below): device memory that is part of
// the code object, one copy per GPU.  In host code these names are handles for hipGetSymbolAddress,
// never addresses.
static __device__ __align__(256) unsigned char scratch[LQSGD_STATIC_SCRATCH_BYTES];
static __device__ __align__(256) unsigned char operands[LQSGD_STATIC_OPERAND_BYTES];
static __device__ __align__(256) unsigned char grams[LQSGD_STATIC_GRAM_BYTES];
#endif

namespace lqsgd {
namespace {

// ---------------------------------------------------------------------------
// small helpers
// ---------------------------------------------------------------------------
// Loads through a pointer in the constant address space are assumed not to
// change while the kernel runs; with a wave-uniform address they become
// scalar loads (one fetch per wavefront, no vector register traffic).  Used
// for factor rows that an earlier kernel wrote.
typedef const float __attribute__((address_space(4)))* const_fp;

// Streaming hints: data that is read once (gradients, residual) is loaded
// with the non-temporal hint so that it does not displace the factor panels.
#ifndef LQSGD_NT_G
#define LQSGD_NT_G 1
#endif
#ifndef LQSGD_NT_E          // residual sweeps (eager schedule); sweep 0 follows its store policy, see add_project_kernel
#define LQSGD_NT_E 1
#endif
#ifndef LQSGD_NT_M
#define LQSGD_NT_M 1
#endif
#ifndef LQSGD_RT           // rows a wavefront carries through one column pass of sweep 0 (rank <= 8)
#define LQSGD_RT 8
#endif
#ifndef LQSGD_BM_U
#define LQSGD_BM_U 8   // pairs of rows per step of the matrix-core sweep 1 (4: 829 us, 8: 750 us, 16: 833 us at 8192^2 x 16)
#endif
#ifndef LQSGD_BQ_LATE      // matrix-core sweep 0, fused mode: fetch the P product's Q slice after the G-hat part
#define LQSGD_BQ_LATE 1
#endif
#ifndef LQSGD_B_U          // rows a wavefront of sweep 1 has in flight
#define LQSGD_B_U 8
#endif
#ifndef LQSGD_B_INTERLEAVE  // sweep 1: row blocks of at least this many rows are split between the wavefronts in groups of LQSGD_B_U rows
#define LQSGD_B_INTERLEAVE 512
#endif
[[maybe_unused]] constexpr int kCus = 256;
// Dynamic LDS that sweep 0 asks for, and does not use, to keep it at two workgroups a CU, two wavefronts a SIMD: where rows
// fill a wavefront's pass more of them read slower (ResNet-18 set, r = 4: 187 / 174.7 / 177 / 177 us at 1 / 2 / 3 / 4).  Rows
// much narrower than a pass wait for memory instead, and take what the registers allow (1000000 x 16, r = 4, W = 8: 1980 us
// at two, 1560 without the limit, one group of rows an item).  (The registers are shared out for three, and rank pad 8 needs
// those of two: for four, rank pad 2 gets 117 instead of 142 of them and 8192^2 x 16 takes 2190 instead of 2085 us.)  Sweep 1
// takes what they allow everywhere (those narrow rows 434 us at four, 344 without a limit; the ResNet-18 set 64.5 and 64.9).
[[maybe_unused]] constexpr unsigned kTwoPerCu = 56 * 1024;
// The same for the residual sweep: three (ResNet-18 set 141 / 136 / 143 / 142 us at 2 / 3 / 4 / 8; with non-temporal stores 176,
// with plain loads 147; narrow rows see Plan::build).
[[maybe_unused]] constexpr unsigned kThreePerCu = 48 * 1024;

template <int V>
struct Pk {
  float v[V];
};

// Every tensor the kernels touch lives in device memory, but a pointer fetched from a pointer table
// (the caller's gradient and output tensors) is a generic one as far as the compiler knows, and it
// would use flat-address instructions for it, which complete out of order with the global ones and
// force every wait to be a wait for everything.  The streaming loads and stores say "global" outright.
template <typename T>
__device__ __forceinline__ const T __attribute__((address_space(1)))* gptr(const void* p) {
  return (const T __attribute__((address_space(1)))*)p;
}
template <typename T>
__device__ __forceinline__ T __attribute__((address_space(1)))* gptr(void* p) {
  return (T __attribute__((address_space(1)))*)p;
}

// x where `on`, else +0: a bit mask instead of a select, so that the compiler cannot turn the
// unconditional load that produced x back into a branch around a conditional one
__device__ __forceinline__ float keep_if(float x, bool on) {
  return __uint_as_float(__float_as_uint(x) & (on ? 0xffffffffu : 0u));
}

// Four floats at (wave-uniform row base) + (per-lane byte offset).  Rows of any length: the row only has to start at a
// multiple of the element size (global memory takes 16-byte accesses at any 4-byte address), so widths that are no
// multiple of four stream like the others and only the last group of a row is taken apart.  Against 4-byte accesses
// (3 x (64 x 27 .. 1000 x 2049)): sweep 1 28 -> 14 us at r = 4; sweep 0 1100 -> 59 us at r = 20, where such rows took a
// loop of one wavefront sum per row and rank.
typedef float v4fu __attribute__((ext_vector_type(4), aligned(4)));
template <bool NT>
__device__ __forceinline__ Pk<4> ldrow(const char* rowbase, unsigned boff) {
  const auto* p = gptr<v4fu>(rowbase + boff);
  const v4fu t = NT ? __builtin_nontemporal_load(p) : *p;
  return Pk<4>{{t.x, t.y, t.z, t.w}};
}
// The same for a row of bfloat16 values (gradients handed over in bfloat16): boff is the byte
// offset the fp32 loaders would use; a bfloat16 is the upper half of the float it stands for.
typedef unsigned int v2uu __attribute__((ext_vector_type(2), aligned(2)));
template <bool NT>
__device__ __forceinline__ Pk<2> ldrow_bf16_packed(const char* rowbase, unsigned boff) {
  const auto* p = gptr<v2uu>(rowbase + (boff >> 1));
  const v2uu t = NT ? __builtin_nontemporal_load(p) : *p;
  return Pk<2>{{__uint_as_float(t.x), __uint_as_float(t.y)}};
}
__device__ __forceinline__ Pk<4> unpack_bf16(float lo, float hi) {
  const unsigned x = __float_as_uint(lo), y = __float_as_uint(hi);
  return Pk<4>{{__uint_as_float(x << 16), __uint_as_float(x & 0xffff0000u), __uint_as_float(y << 16), __uint_as_float(y & 0xffff0000u)}};
}
// Gradient row in either format.
template <bool NT, bool GB16>
__device__ __forceinline__ Pk<4> ldgrad(const char* rowbase, unsigned boff) {
  if constexpr (GB16) {
    const Pk<2> t = ldrow_bf16_packed<NT>(rowbase, boff);
    return unpack_bf16(t.v[0], t.v[1]);
  } else {
    return ldrow<NT>(rowbase, boff);
  }
}
// Start of gradient row `off / cols` given its element offset.
template <bool GB16>
__device__ __forceinline__ const char* grad_row(const float* G, size_t off) {
  return reinterpret_cast<const char*>(G) + off * (GB16 ? 2 : 4);
}
template <bool GB16>
__device__ __forceinline__ float grad_elem(const float* G, size_t idx) {
  if constexpr (GB16) return __uint_as_float((unsigned)gptr<unsigned short>(G)[idx] << 16);
  else return gptr<float>(G)[idx];
}

template <bool NT>
__device__ __forceinline__ void strow(char* rowbase, unsigned boff, const Pk<4>& x) {
  const v4fu t = {x.v[0], x.v[1], x.v[2], x.v[3]};
  auto* p = gptr<v4fu>(rowbase + boff);
  if constexpr (NT) __builtin_nontemporal_store(t, p);
  else *p = t;
}

// Rows whose width is no multiple of four.  A lane's group of columns c .. c + 3 may hang over the end of its row: it is
// then loaded from edge_col(c), the row's last four columns, like every other lane's and without a branch, and
// edge_fix() moves the values into place, zeros behind them.  (Element loads under a branch for the last lane cost
// sweep 0 a second memory round trip per pass: 40 us against 29 us on 3 x (64 x 27 .. 1000 x 2049).)  A store
// writes the existing elements only.
__device__ __forceinline__ int edge_col(int c, int cols) { return max(0, min(c, cols - 4)); }
// Shapes of a layer's rows, a constant in every kernel's inner loops (a test inside ldedge would part the loads).
enum RowKind { kAligned = 0, kRagged = 1, kNarrow = 2 };   // cols % 4 == 0; the rest; the rest below four columns
constexpr int kOneColumnPerLane = 2;                       // LayerDesc::kind, see narrow_rows
template <int KIND, bool NT, bool GB16>
__device__ __forceinline__ Pk<4> ldedge(const char* rowbase, int c, int cols) {
  if constexpr (KIND == kNarrow) {               // element loads, the surplus ones repeat the last element
    Pk<4> r;
#pragma unroll
    for (int v = 0; v < 4; ++v) r.v[v] = grad_elem<GB16>(reinterpret_cast<const float*>(rowbase), min(v, cols - 1));
    return r;
  } else {
    return ldgrad<NT, GB16>(rowbase, (unsigned)(KIND == kAligned ? c : edge_col(c, cols)) * 4u);
  }
}
// N values per column, four columns loaded from edge_col(c) on -> those of columns c .. c + 3.
template <int N>
__device__ __forceinline__ void edge_fix(float (&x)[4 * N], int c, int cols) {
  const int sh = c - edge_col(c, cols), n = cols - c;
#pragma unroll
  for (int i = 0; i < 4 * N; ++i) x[i] = (sh & 1) ? (i + N < 4 * N ? x[i + N] : 0.0f) : x[i];
#pragma unroll
  for (int i = 0; i < 4 * N; ++i) x[i] = (sh & 2) ? (i + 2 * N < 4 * N ? x[i + 2 * N] : 0.0f) : x[i];
#pragma unroll
  for (int i = 0; i < 4 * N; ++i) x[i] = i < n * N ? x[i] : 0.0f;
}
// Stores the first n (<= 0: none, >= 4: all) elements of a group.
template <bool NT>
__device__ __forceinline__ void stgroup(char* rowbase, unsigned boff, int n, const Pk<4>& x) {
  if (n >= 4) {
    strow<NT>(rowbase, boff, x);
  } else {
#pragma unroll
    for (int v = 0; v < 3; ++v)
      if (v < n) gptr<float>(rowbase + boff)[v] = x.v[v];
  }
}

// Output of the reconstruction G-hat = P-bar Q-bar^T (Eq. (7)): either stored as it is, or applied
// to the caller's parameters, w <- w - eta G-hat (Algorithm 1, "Model update"; Eq. (2)).
template <int KIND>
__device__ __forceinline__ void emit_ghat(float* __restrict__ rowbase, int c, int cols, Pk<4> gh, int update, float eta, const Pk<4>& w) {
  char* row = reinterpret_cast<char*>(rowbase);
  const int n = KIND == kAligned ? 4 : cols - c;
  if (update) {
#pragma unroll
    for (int v = 0; v < 4; ++v) gh.v[v] = fmaf(-eta, gh.v[v], w.v[v]);
    stgroup<false>(row, (unsigned)c * 4u, n, gh);
  } else {
    stgroup<true>(row, (unsigned)c * 4u, n, gh);
  }
}
// The parameters that emit_ghat updates: fetched well ahead of it, or a row waits for them alone.
template <int KIND>
__device__ __forceinline__ Pk<4> load_params(const float* rowbase, int c, int cols) {
  Pk<4> w = ldedge<KIND, false, false>(reinterpret_cast<const char*>(rowbase), c, cols);
  if (KIND != kAligned && c + 4 > cols) edge_fix<1>(w.v, c, cols);
  return w;
}

// The factors as the sweeps read them: rows of RP ranks, zero beyond a layer's rank.  Where every layer fills the
// register pad that is the aggregate itself, elsewhere a copy that whoever writes the aggregate writes beside it
// (DevArgs::Pop / Qop), so that a lane's slice is whole 16-byte loads at every rank.  With tightly packed rows of
// 7 ranks sweep 0 spent 32 four-byte loads per lane and column pass on it: ResNet-18 set, W = 8, bfloat16 gradients,
// 405 us; 16-byte loads: 178 us.
__device__ __forceinline__ const float* p_operand(const DevArgs& a, const LayerDesc& ld) {
  return a.Pop + ld.pop_off;
}
__device__ __forceinline__ const float* q_operand(const DevArgs& a, const LayerDesc& ld) {
  return a.Qop + ld.qop_off;
}

// Factor slice of four consecutive columns starting at column c, as s[v*RP + k].
template <int RP>
__device__ __forceinline__ void load_slice(const float* __restrict__ F, int c, float (&s)[4 * RP]) {
  const auto* base = gptr<v4fu>(F + (size_t)c * RP);
#pragma unroll
  for (int i = 0; i < RP; ++i) {
    const v4fu t = base[i];
    s[4 * i + 0] = t.x; s[4 * i + 1] = t.y; s[4 * i + 2] = t.z; s[4 * i + 3] = t.w;
  }
}
// f(integral_constant<int, 0>) ... f(integral_constant<int, N - 1>), in order.
template <int N, int I = 0, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<N, I + 1>(f);
  }
}

// Row of a rows x r factor into p[k] (zero beyond r), plain loads.
template <int RP>
__device__ __forceinline__ void load_row(const float* __restrict__ F, int row, int r, bool exact, float (&p)[RP]) {
  if (exact) {
    const float* b = F + (size_t)row * RP;
#pragma unroll
    for (int k = 0; k < RP; ++k) p[k] = b[k];
  } else {
    const float* b = F + (size_t)row * r;
#pragma unroll
    for (int k = 0; k < RP; ++k) p[k] = keep_if(b[k], k < r);
  }
}

// The first r of the RP values to one place, in one store (RP <= 4).
template <int RP>
__device__ __forceinline__ void store_row(float* to, int r, const float (&p)[RP]) {
  static_for<RP>([&](auto n) __attribute__((always_inline)) {
    if (r == n.value + 1) {
#pragma unroll
      for (int k = 0; k <= n.value; ++k) to[k] = p[k];
    }
  });
}

// Wave-uniform row of a factor operand written by an earlier kernel: scalar loads.
template <int RP>
__device__ __forceinline__ void load_row_uniform(const float* F, int row, float (&p)[RP]) {
  const_fp b = (const_fp)(F + (size_t)row * RP);
#pragma unroll
  for (int k = 0; k < RP; ++k) p[k] = b[k];
}

// Sum of N per-lane values over the 64 lanes of a wavefront, N a power of two.
// Each butterfly step exchanges half of the still-live values, so the cost is
// about N shuffles instead of 6 N.  On return lane l holds, in v[0 .. max(1,N/64)),
// the totals of the values with index l*(N/64)+i (N >= 64), or of index
// l >> (6 - log2 N) replicated over 64/N neighbouring lanes (N < 64).
template <int NT, int LIVE, int OFF>
__device__ __forceinline__ void transpose_reduce(float (&v)[NT], int lane) {
  if constexpr (OFF >= 1) {
    if constexpr (LIVE > 1) {
      constexpr int H = LIVE / 2;
      const bool hi = (lane & OFF) != 0;
#pragma unroll
      for (int i = 0; i < H; ++i) {
        const float keep = hi ? v[i + H] : v[i];
        const float send = hi ? v[i] : v[i + H];
        v[i] = keep + __shfl_xor(send, OFF, kWave);
      }
      transpose_reduce<NT, H, OFF / 2>(v, lane);
    } else {
      v[0] += __shfl_xor(v[0], OFF, kWave);
      transpose_reduce<NT, 1, OFF / 2>(v, lane);
    }
  }
}

__device__ __forceinline__ void wave_lds_fence() {
  // LDS traffic between the lanes of one wavefront: the hardware keeps DS
  // operations of a wavefront in order; this only stops the compiler.
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Sums over the lanes of a wavefront, partners 32, 16, .. 1 apart, without LDS.  swap32_add: lanes 0 - 31 get x + its partner,
// lanes 32 - 63 y + its partner; swap16_add: the same within each 32 lanes; row_sums: the sum over each row of 16 lanes.
__device__ __forceinline__ float swap32_add(float x, float y) {
  const auto t = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
  return __uint_as_float(t[0]) + __uint_as_float(t[1]);
}
__device__ __forceinline__ float swap16_add(float x, float y) {
  const auto t = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
  return __uint_as_float(t[0]) + __uint_as_float(t[1]);
}
__device__ __forceinline__ float row_sums(float x) {
  // each step leaves a row periodic, so that a rotation by half a period is the partner's value
#define LQSGD_ROR_ADD(N) \
  x += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x120 + (N), 0xf, 0xf, true))
  LQSGD_ROR_ADD(8);
  LQSGD_ROR_ADD(4);
  LQSGD_ROR_ADD(2);
  LQSGD_ROR_ADD(1);
#undef LQSGD_ROR_ADD
  return x;
}
// The sums of four values: c[0], c[2], c[1], c[3] in rows 0, 1, 2, 3.
__device__ __forceinline__ float four_lane_sums(const float (&c)[4]) {
  return row_sums(swap16_add(swap32_add(c[0], c[1]), swap32_add(c[2], c[3])));
}

__device__ __forceinline__ float wave_max(float x) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) x = fmaxf(x, __shfl_xor(x, off, kWave));
  return x;
}

constexpr int log2c(int n) { return n <= 1 ? 0 : 1 + log2c(n / 2); }

// The absmax cells that later kernels of the iteration raise with atomic maxima start from zero:
// absmax(Q_w) always (sweep 1 or the reduce that follows it), absmax of the raw P_w in the
// aggregate-first order.  Called by the first workgroup of sweep 0, which nothing of this iteration
// that touches those cells can overtake.
__device__ __forceinline__ void zero_absmax_cells(const DevArgs& a, int nthreads) {
  for (int i = threadIdx.x; i < a.W * a.L; i += nthreads) {
    a.scaleQ[i] = 0.0f;
    if (a.agg_first) a.scaleP[i] = 0.0f;
  }
}

// ---------------------------------------------------------------------------
// sweep 0: M = G + E (Eq. (9)),  P_w partial = M_w Q  (Algorithm 1, "P <- G'Q")
// One wavefront per work item: rows [row0, row0+nrows) x columns [col0, col1),
// RT rows at a time; a lane accumulates RT x r partial dot products over its
// columns, one butterfly per row group adds them over the lanes.
// ---------------------------------------------------------------------------
template <int RP, int RT, bool FULL, int KIND, bool FUSE, bool GB16, bool NTS>
__device__ __forceinline__ void add_project_cols(const char* const (&gr)[RT], char* const (&mr)[RT],
                                                 const float* __restrict__ Q, const float (&pb)[RT * RP], int nr,
                                                 int cbeg, int cend, int cols, float (&acc)[RT * RP]) {
  for (int c = cbeg; c < cend; c += kWave * 4) {
    float q[4 * RP];
    const unsigned boff = (unsigned)c * 4u;
    Pk<4> g[RT], e[RT];
    load_slice<RP>(Q, KIND == kAligned ? c : edge_col(c, cols), q);
#pragma unroll
    for (int t = 0; t < RT; ++t) {               // rows beyond nr repeat the last one: loaded, never stored
      g[t] = ldedge<KIND, LQSGD_NT_G != 0, GB16>(gr[t], c, cols);
      e[t] = ldedge<KIND, NTS, false>(mr[t], c, cols);
    }
    // All requests stay ahead of the arithmetic (left to itself the compiler trades loads in flight for
    // registers; at ranks 1 and 2 it has them and does better alone).
    if constexpr (RP >= 4) __builtin_amdgcn_sched_barrier(0);
    if (KIND != kAligned && c + 4 > cols) {
      edge_fix<RP>(q, c, cols);
#pragma unroll
      for (int t = 0; t < RT; ++t) { edge_fix<1>(g[t].v, c, cols); edge_fix<1>(e[t].v, c, cols); }
    }
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      Pk<4> m;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        float ev = e[t].v[v];
        if constexpr (FUSE) {
          // the buffer still holds last iteration's M: E = M - P-bar Q-bar^T (Eq. (8)),
          // with the same operation order as the stand-alone residual sweep
          float gh = 0.0f;
#pragma unroll
          for (int k = 0; k < RP; ++k) gh = fmaf(pb[t * RP + k], q[v * RP + k], gh);
          ev = ev - gh;
        }
        m.v[v] = g[t].v[v] + ev;
      }
      if constexpr (KIND != kAligned) e[t] = m;               // stored below, all rows in one branch
      else if (FULL || t < nr) strow<NTS>(mr[t], boff, m);
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int k = 0; k < RP; ++k) acc[t * RP + k] = fmaf(m.v[v], q[v * RP + k], acc[t * RP + k]);
    }
    if constexpr (KIND != kAligned) {
      if (c + 4 <= cols) {
#pragma unroll
        for (int t = 0; t < RT; ++t)
          if (FULL || t < nr) strow<NTS>(mr[t], boff, e[t]);
      } else {
#pragma unroll
        for (int t = 0; t < RT; ++t)
          if (FULL || t < nr) stgroup<NTS>(mr[t], boff, cols & 3, e[t]);
      }
    }
  }
}

template <int RP, int RT, int KIND, bool FUSE, bool GB16, bool NTS>
__device__ __forceinline__ void add_project_tile(const float* __restrict__ G, float* __restrict__ M,
                                                 const float* __restrict__ Q, const float* Pb,
                                                 float* __restrict__ Pp, int cols, int r, int row0, int nrows,
                                                 int col0, int col1, int lane) {
  constexpr int N = RT * RP;
  for (int rg = 0; rg < nrows; rg += RT) {
    const int nr = min(RT, nrows - rg);
    float acc[N];
    float pb[N];
#pragma unroll
    for (int i = 0; i < N; ++i) acc[i] = 0.0f;
    const char* gr[RT];
    char* mr[RT];
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      const int row = row0 + rg + min(t, nr - 1);
      const size_t off = (size_t)row * cols;
      gr[t] = grad_row<GB16>(G, off);
      mr[t] = reinterpret_cast<char*>(M + off);
      if constexpr (FUSE) {
        float p[RP];
        load_row_uniform<RP>(Pb, row, p);
#pragma unroll
        for (int k = 0; k < RP; ++k) pb[t * RP + k] = p[k];
      } else {
#pragma unroll
        for (int k = 0; k < RP; ++k) pb[t * RP + k] = 0.0f;
      }
    }
    if (nr == RT)
      add_project_cols<RP, RT, true, KIND, FUSE, GB16, NTS>(gr, mr, Q, pb, nr, col0 + lane * 4, col1, cols, acc);
    else
      add_project_cols<RP, RT, false, KIND, FUSE, GB16, NTS>(gr, mr, Q, pb, nr, col0 + lane * 4, col1, cols, acc);
    transpose_reduce<N, N, 32>(acc, lane);
    constexpr int NPL = (N >= kWave) ? N / kWave : 1;
#pragma unroll
    for (int i = 0; i < NPL; ++i) {
      int idx;
      bool writer;
      if constexpr (N >= kWave) {
        idx = lane * NPL + i;
        writer = true;
      } else {
        idx = lane >> (6 - log2c(N));
        writer = (lane & (kWave / N - 1)) == 0;
      }
      const int t = idx / RP, k = idx - t * RP;
      if (writer && t < nr && k < r) Pp[(size_t)(row0 + rg + t) * r + k] = acc[i];
    }
  }
}

// Sweeps 0 and 2 over rows of at most 64 columns that are no multiple of four (input layers, class counts): a lane has
// one column, so that a pass of 4-byte loads covers a row, and the P products of a row are added by one butterfly over the
// lanes (and sweep 1, back_project_tile, holds one column per lane too).  Four columns on a lane, as in wider rows, would
// leave most lanes idle, and on the matrix cores most of a 32-column block; and the order of these sums is part of the results: ranks are often clipped to the width of such a
// layer, its factor is then close to singular, and Gram-Schmidt magnifies what another order changes (64 x 27 at r = 27:
// single values of G-hat 2e-4 of its root mean square).  It is not slower:
// sweep 0 of the ResNet-18 set at r = 50 366 us (four columns on the matrix cores 368); 4 x (100000 x 21), W = 8, r = 4, four
// columns per lane and one: sweep 0 407 and 299 us, sweep 1 169 and 73, finished residual 593 and 184.
// `nrows` rows from row0 on, at most R; ADD: M = G + E and the P partials; FUSE: E is still last iteration's M;
// EMIT: G-hat goes out.  ADD is false in the sweeps that only finish E (HASM) or only write G-hat.
template <int RP, int R, bool ADD, bool FUSE, bool HASM, bool EMIT, bool GB16>
__device__ __forceinline__ void narrow_rows(const float* __restrict__ G, float* __restrict__ M, const float* Q, const float* Pb,
                                            float* __restrict__ Pp, float* __restrict__ ghat, int cols, int r, int row0, int nrows,
                                            int lane, int update, float eta) {
  constexpr int RT = R * RP <= kWave ? R : kWave / RP;                     // rows of a butterfly
  const bool on = lane < cols;
  const int c = min(lane, cols - 1);             // the other lanes repeat the last column, and count as zeros
  float q[RP], g[R], e[R], w[R], p[RT * RP];
  auto fetch_p = [&](int t0) __attribute__((always_inline)) {
#pragma unroll
    for (int t1 = 0; t1 < RT; ++t1) {
      float x[RP];
      load_row_uniform<RP>(Pb, row0 + min(t0 + t1, nrows - 1), x);
#pragma unroll
      for (int k = 0; k < RP; ++k) p[t1 * RP + k] = x[k];
    }
  };
  if constexpr (FUSE || !ADD) fetch_p(0);
  if constexpr (RP >= 4) {
#pragma unroll
    for (int i = 0; i < RP / 4; ++i) {
      const Pk<4> t = ldrow<false>(reinterpret_cast<const char*>(Q), (unsigned)(c * RP + 4 * i) * 4u);
#pragma unroll
      for (int v = 0; v < 4; ++v) q[4 * i + v] = t.v[v];
    }
  } else {
#pragma unroll
    for (int k = 0; k < RP; ++k) q[k] = gptr<float>(Q)[c * RP + k];
  }
#pragma unroll
  for (int t = 0; t < R; ++t) {                  // rows beyond nrows repeat the last one: loaded, never stored
    const size_t at = (size_t)(row0 + min(t, nrows - 1)) * cols + c;
    if constexpr (ADD) g[t] = grad_elem<GB16>(G, at);
    if constexpr (HASM) e[t] = gptr<float>(M)[at];
    if constexpr (EMIT) w[t] = update && ghat ? gptr<float>(ghat)[at] : 0.0f;
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int k = 0; k < RP; ++k) q[k] = keep_if(q[k], on);
#pragma unroll
  for (int t0 = 0; t0 < R; t0 += RT) {
    float acc[RT * RP];
    if constexpr (FUSE || !ADD)
      if (t0 > 0) fetch_p(t0);
#pragma unroll
    for (int t1 = 0; t1 < RT; ++t1) {
      const int t = t0 + t1;
      float m = HASM ? e[t] : 0.0f;
      const size_t at = (size_t)(row0 + t) * cols + c;
      const bool mine = on && t < nrows;
      if constexpr (FUSE || !ADD) {              // the same operation order as everywhere: G-hat in rank order, then E
        float gh = 0.0f;
#pragma unroll
        for (int k = 0; k < RP; ++k) gh = fmaf(p[t1 * RP + k], q[k], gh);
        m = m - gh;
        if (EMIT && ghat && mine) gptr<float>(ghat)[at] = update ? fmaf(-eta, gh, w[t]) : gh;
      }
      if constexpr (ADD) m = g[t] + m;
      if (HASM && mine) gptr<float>(M)[at] = m;
      m = keep_if(m, on);
#pragma unroll
      for (int k = 0; k < RP; ++k) acc[t1 * RP + k] = fmaf(m, q[k], 0.0f);
    }
    if constexpr (ADD) {
      constexpr int N = RT * RP;
      transpose_reduce<N, N, 32>(acc, lane);     // N <= 64: lane l has value l / (64 / N)
      const int idx = lane >> (6 - log2c(N)), t = t0 + idx / RP, k = idx & (RP - 1);
      if ((lane & (kWave / N - 1)) == 0 && t < nrows && k < r) Pp[(size_t)(row0 + t) * r + k] = acc[0];
    }
  }
}

// Rows row0 .. rend of a wavefront; in sweep 0, whose loads are what it waits for, 16 at a time as long as there are as many.
// (Not at rank pad 8: 16 rows there cost the aligned rows in the same kernel, bfloat16 gradients, ResNet-18 set 184 against 172 us.)
template <int RP, bool ADD, bool FUSE, bool HASM, bool EMIT, bool GB16>
__device__ __forceinline__ void narrow_item(const float* __restrict__ G, float* __restrict__ M, const float* Q, const float* Pb,
                                            float* __restrict__ Pp, float* __restrict__ ghat, int cols, int r, int row0, int rend,
                                            int lane, int update, float eta) {
  for (; ADD && RP <= 4 && row0 + 16 <= rend; row0 += 16)
    narrow_rows<RP, 16, ADD, FUSE, HASM, EMIT, GB16>(G, M, Q, Pb, Pp, ghat, cols, r, row0, 16, lane, update, eta);
  for (; row0 < rend; row0 += 8)
    narrow_rows<RP, 8, ADD, FUSE, HASM, EMIT, GB16>(G, M, Q, Pb, Pp, ghat, cols, r, row0, min(8, rend - row0), lane, update, eta);
}

// FUSE: the residual update of the previous iteration has been deferred; the
// buffer holds M_{t-1} and this sweep forms E_{t-1} = M_{t-1} - P-bar Q-bar^T on
// the fly (Q-bar is the warm-start Q this sweep multiplies by anyway).
// NTS: the residual slabs are streamed -- E (or last iteration's M) is read with the non-temporal
// hint and M is written with non-temporal stores; chosen by the host from the size of the working set.
template <int RP, bool FUSE, bool GB16, bool NTS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, RP >= 8 ? 2 : 3))) void add_project_kernel(DevArgs a, const Tile* __restrict__ tiles, int ntiles, int reverse) {
  constexpr int RT = LQSGD_RT;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & (kWave - 1);
  if (blockIdx.x == 0) zero_absmax_cells(a, 256);
  const int t = blockIdx.x * 4 + wave;
  if (t >= ntiles) return;
  const Tile tl = tiles[reverse ? ntiles - 1 - t : t];
  const int layer = tl.lw / a.W, worker = tl.lw - layer * a.W;
  const LayerDesc& ld = a.layers[layer];
  const float* G = a.grads[(size_t)worker * a.n_all + ld.gidx];
  float* M = a.E + (size_t)worker * a.m_stride + ld.m_off;
  const float* Q = q_operand(a, ld);
  const float* Pb = p_operand(a, ld);
  float* Pp = a.Ppart + (size_t)worker * a.ppart_stride + ld.ppart_off + (size_t)tl.aux * ld.np_pad;
  const int col0 = tl.aux * ld.segw;
  const int col1 = min(ld.cols, col0 + ld.segw);
  if (ld.kind == kAligned)
    add_project_tile<RP, RT, kAligned, FUSE, GB16, NTS>(G, M, Q, Pb, Pp, ld.cols, ld.r, tl.row0, tl.nrows, col0, col1, lane);
  else if (ld.kind == kRagged)
    add_project_tile<RP, RT, kRagged, FUSE, GB16, NTS>(G, M, Q, Pb, Pp, ld.cols, ld.r, tl.row0, tl.nrows, col0, col1, lane);
  else                                           // one segment
    narrow_item<RP, true, FUSE, true, false, GB16>(G, M, Q, Pb, Pp, nullptr, ld.cols, ld.r, tl.row0, tl.row0 + tl.nrows, lane, 0, 0.0f);
}

// ---------------------------------------------------------------------------
// LogQuantize of Section 4.1 for one value and for a packed group of 8, as the
// exchange kernel uses them.
// The code of u = |x|/s is the number of decision thresholds <= u, i.e.
// nearest-level rounding in the q-domain of Eq. (5): a hardware log2 gives the
// level, and the thresholds on its two sides move it to the exact count.
// ---------------------------------------------------------------------------
// s_thr points at threshold 0; s_thr[-1] and s_thr[lv] are NaN, which no comparison holds for.
// ONESTEP: the estimate is known to be within one level (DevArgs::quant_fast), else it is walked all the way.
template <bool ONESTEP>
__device__ __forceinline__ int quantise_one(float u, float alpha, float qscale, int lv, const float* s_thr) {
  const float t = __log2f(fmaf(alpha, u, 1.0f)) * qscale;
  int k = (int)(t + 0.5f);
  k = max(0, min(lv, k));
  if constexpr (ONESTEP) {
    const float below = s_thr[k - 1], above = s_thr[k];
    k += (above <= u ? 1 : 0) - (below > u ? 1 : 0);
  } else {
    while (k < lv && s_thr[k] <= u) ++k;
    while (k > 0 && s_thr[k - 1] > u) --k;
  }
  return k;
}

// One group of kXGroup consecutive factor elements of one worker: LogQuantize against the worker's
// absmax s (codes: number of thresholds <= |x| / s; sign bit only on a non-zero code), the packed
// group (`bits` magnitude bytes, one sign byte) stored, and the dequantised values (Eq. (6): +-s level_k) in val.
// FAST: the estimate of a code is within one level (ONESTEP above), and the quotient comes from the reciprocal of s, taken once,
// and a remainder step (Markstein, "Computation of elementary functions on the IBM RISC System/6000", 1990: correctly
// rounded like the division it replaces, given a correctly rounded reciprocal and no under- or overflow: s_fast).
template <bool FAST>
__device__ __forceinline__ void quantise_group(const float (&x)[kXGroup], float s, int bits, int lv, float alpha, float qscale,
                                               const float* s_thr, const float* s_lev, uint8_t* mp, uint8_t* sp,
                                               float (&val)[kXGroup]) {
  unsigned long long magbits = 0;
  unsigned sgnbits = 0;
  const float rs = 1.0f / s;
#pragma unroll
  for (int i = 0; i < kXGroup; ++i) {
    const float ax = fabsf(x[i]);
    float u;
    if constexpr (FAST) {
      const float q = ax * rs;
      u = fmaf(fmaf(-q, s, ax), rs, q);
    } else {
      u = ax / s;
    }
    const int k = (s > 0.0f) ? quantise_one<FAST>(u, alpha, qscale, lv, s_thr) : 0;
    magbits |= (unsigned long long)k << (i * bits);
    const bool neg = x[i] < 0.0f && k > 0;
    if (neg) sgnbits |= 1u << i;
    const float v = s * s_lev[k];
    val[i] = neg ? -v : v;
  }
  if (bits == 8) {
    *reinterpret_cast<unsigned long long*>(mp) = magbits;
  } else if (bits == 4) {
    *reinterpret_cast<unsigned*>(mp) = (unsigned)magbits;
  } else if (bits == 2) {
    *reinterpret_cast<unsigned short*>(mp) = (unsigned short)magbits;
  } else {
    for (int bb = 0; bb < bits; ++bb) mp[bb] = (uint8_t)(magbits >> (8 * bb));
  }
  *sp = (uint8_t)sgnbits;
}

// ---------------------------------------------------------------------------
// orth: P_w = sum of the column-segment partials; modified Gram-Schmidt
// (Algorithm 1, "Orthonormalize"), right-looking: column j is normalised, then
// removed from every later column, which applies the projections to a column
// in the same order as the left-looking form.  Ends with absmax(P_w) -> scaleP.
// In the aggregate-first order (orth_shared) the same kernels run once per layer
// on the aggregated factor: input = one plane at P-bar, output in place, the
// un-orthonormalised aggregate kept where `Ppre` points, no absmax.
//
// orth, rows on lanes: one workgroup per (layer, worker) for layers of at most
// BS * RPT rows; a lane keeps its RPT rows in registers through all passes and
// only the block-wide sums go through LDS (one barrier per column).  Rank pads 1
// and 2: two columns leave nothing to gain from columns on lanes.
// ---------------------------------------------------------------------------
template <int RP, int RPT, int BS>
__global__ __launch_bounds__(BS) void orth_reg_kernel(DevArgs a) {
  constexpr int NW = BS / kWave;
  constexpr int LG = log2c(RP);
  __shared__ float red[2][NW][RP];
  __shared__ float redmax[NW];
  const int lw = blockIdx.x;
  const int layer = lw / a.W, worker = lw - layer * a.W;
  const LayerDesc& ld = a.layers[layer];
  const int rows = ld.rows, r = ld.r, nseg = a.orth_shared ? 1 : ld.nseg;
  const bool exact = (r == RP);
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
  const float* Pp = a.Ppart + (size_t)worker * a.ppart_stride + (a.orth_shared ? ld.p_off : ld.ppart_off);
  float* pre = a.Ppre + (size_t)worker * a.p_stride + ld.p_off;
  float* orth = a.Porth + (size_t)worker * a.p_stride + ld.p_off;

  float v[RPT][RP];
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    const int row = tid + i * BS;
#pragma unroll
    for (int k = 0; k < RP; ++k) v[i][k] = 0.0f;
    if (row < rows) {
      for (int s = 0; s < nseg; ++s) {
        float t[RP];
        load_row<RP>(Pp + (size_t)s * ld.np_pad, row, r, exact, t);
#pragma unroll
        for (int k = 0; k < RP; ++k) v[i][k] += t[k];
      }
#pragma unroll
      for (int k = 0; k < RP; ++k)
        if (k < r) pre[(size_t)row * r + k] = v[i][k];
    }
  }

#pragma unroll
  for (int j = 0; j < RP; ++j) {
    if (j < r) {
      float s[RP];
#pragma unroll
      for (int k = 0; k < RP; ++k) s[k] = 0.0f;
#pragma unroll
      for (int i = 0; i < RPT; ++i)
#pragma unroll
        for (int k = 0; k < RP; ++k) s[k] = fmaf(v[i][j], v[i][k], s[k]);
      transpose_reduce<RP, RP, 32>(s, lane);
      const int b = j & 1;
      if ((lane & (kWave / RP - 1)) == 0) red[b][wave][lane >> (6 - LG)] = s[0];
      __syncthreads();
#pragma unroll
      for (int k = 0; k < RP; ++k) {
        float t = 0.0f;
#pragma unroll
        for (int wv = 0; wv < NW; ++wv) t += red[b][wv][k];
        s[k] = t;
      }
      const float nrm2 = s[j];
      const float inv = (nrm2 > FLT_MIN) ? 1.0f / sqrtf(nrm2) : 0.0f;
#pragma unroll
      for (int i = 0; i < RPT; ++i) {
        const float qv = v[i][j] * inv;
        v[i][j] = qv;
#pragma unroll
        for (int k = j + 1; k < RP; ++k) v[i][k] = fmaf(-(s[k] * inv), qv, v[i][k]);
      }
    }
  }

  float mx = 0.0f;
  float* copy = a.orth_shared && a.padded ? a.Pop + ld.pop_off : nullptr;
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    const int row = tid + i * BS;
    if (row < rows) {
#pragma unroll
      for (int k = 0; k < RP; ++k)
        if (k < r) {
          orth[(size_t)row * r + k] = v[i][k];
          if (copy) copy[(size_t)row * RP + k] = v[i][k];
          mx = fmaxf(mx, fabsf(v[i][k]));
        }
    }
  }
  mx = wave_max(mx);
  if (lane == 0) redmax[wave] = mx;
  __syncthreads();
  if (tid == 0 && !a.orth_shared) {
    float m = redmax[0];
#pragma unroll
    for (int wv = 1; wv < NW; ++wv) m = fmaxf(m, redmax[wv]);
    a.scaleP[(size_t)worker * a.L + layer] = m;
  }
}

// ---------------------------------------------------------------------------
// orth, rows on lanes, one workgroup per (layer, worker), with the sums of
// slices of 256 rows (orth_coop_kernel, orth_wide_kernel; rank pads 1 to 4), to
// the last bit: the products of 256 neighbouring rows, a butterfly over each 64
// of them, the four wavefronts in pairs, then the slices one after the other.  A
// thread holds rows t, t + 1024, .., so that wavefronts 4 q .. 4 q + 3 have slice
// q of each block of 1024.
//
// What bounds it: reading the planes on one CU, then for each column two
// barriers and up to 44 additions in a row (1 to 2 us).  The slices' way costs
// about 20 us for the cooperative launch and 2 to 3 a column.  Gram-Schmidt, us,
// in one cooperative launch / here: 4096 x 1024, W = 16, r = 4 33 / 11,
// 8192^2, W = 16, r = 1 32 / 12, r = 4 42 / 24; 11264 x 8192, r = 3 43 / 27.  (With
// its values stored one at a time, 4 bytes of every row, 8192 x 1024, r = 4 took
// 28 us instead of 17.)
// ---------------------------------------------------------------------------
template <int RP, int RPT>
__global__ __launch_bounds__(1024) void orth_tall_kernel(DevArgs a) {
  constexpr int BS = 1024, NW = BS / kWave, NS = 4 * RPT;       // slices held
  constexpr int GROUPS = RPT * RP / 4;                          // of four values that are summed together
  static_assert(RPT * RP % 4 == 0 && GROUPS <= 16 && NS <= kWave && RP <= NW, "");
  __shared__ __attribute__((aligned(16))) float part[RP][NS][4];
  __shared__ float tot[RP];
  __shared__ float redmax[NW];
  const int lw = blockIdx.x;
  const int layer = lw / a.W, worker = lw - layer * a.W;
  const LayerDesc& ld = a.layers[layer];
  const int rows = ld.rows, r = ld.r, nseg = a.orth_shared ? 1 : ld.nseg, nslice = (rows + 255) >> 8;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const float* Pp = a.Ppart + (size_t)worker * a.ppart_stride + (a.orth_shared ? ld.p_off : ld.ppart_off);
  float* pre = a.Ppre + (size_t)worker * a.p_stride + ld.p_off;
  float* orth = a.Porth + (size_t)worker * a.p_stride + ld.p_off;

  // the planes added in order, many rows in flight; rows beyond the factor re-read its last one and count as zeros
  constexpr int CH = RPT * RP > 40 ? (RPT + 1) / 2 : RPT;
  int row0 = tid;
  auto hide_row = [&]() __attribute__((always_inline)) { asm volatile("" : "+v"(row0)); };   // (else all addresses stay in registers, and some spill)
  float v[RPT][RP];
#pragma unroll
  for (int i = 0; i < RPT; ++i)
#pragma unroll
    for (int k = 0; k < RP; ++k) v[i][k] = 0.0f;
  auto add_planes = [&](auto width) __attribute__((always_inline)) {   // (rows of r values in one load)
    constexpr int N = decltype(width)::value + 1;
    for (int s = 0; s < nseg; ++s) {
      const float* src = Pp + (size_t)s * ld.np_pad;
      hide_row();
#pragma unroll
      for (int i0 = 0; i0 < RPT; i0 += CH) {
        float t[CH][N];
#pragma unroll
        for (int i = 0; i < CH; ++i)
          if (i0 + i < RPT) {
            const float* from = src + min(row0 + (i0 + i) * BS, rows - 1) * N;
#pragma unroll
            for (int k = 0; k < N; ++k) t[i][k] = from[k];
          }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < CH; ++i)
#pragma unroll
          for (int k = 0; k < N; ++k)
            if (i0 + i < RPT) v[i0 + i][k] += t[i][k];
      }
    }
  };
  static_for<RP>([&](auto width) __attribute__((always_inline)) {
    if (r == width.value + 1) add_planes(width);
  });
  hide_row();
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    const int row = row0 + i * BS;
    if (row < rows) store_row<RP>(pre + row * r, r, v[i]);
#pragma unroll
    for (int k = 0; k < RP; ++k) v[i][k] = row < rows ? v[i][k] : 0.0f;
  }

  // the value whose sum this lane writes: the n-th of the thread's, row n / RP of it, column n % RP
  const int q = lane >> 4, n = 4 * (lane & 15) + (q == 1 ? 2 : q == 2 ? 1 : q);
#pragma unroll
  for (int j = 0; j < RP; ++j) {
    if (j < r) {
      float mine = 0.0f;
#pragma unroll
      for (int g = 0; g < GROUPS; ++g) {
        float x;
        if constexpr (RP == 1) {                   // (see column_products)
          auto squares = [&](int i) __attribute__((always_inline)) {
            const auto t = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[i][0]), __float_as_uint(v[i + 1][0]), false, false);
            const float lo = __uint_as_float(t[0]), hi = __uint_as_float(t[1]);
            return fmaf(lo, lo, hi * hi);
          };
          x = row_sums(swap16_add(squares(4 * g), squares(4 * g + 2)));
        } else {
          float c[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) c[e] = v[(4 * g + e) / RP][j] * v[(4 * g + e) / RP][(4 * g + e) % RP];
          x = four_lane_sums(c);
        }
        mine = (lane & 15) == g ? x : mine;
      }
      if ((lane & 15) < GROUPS) part[n % RP][4 * (n / RP) + (wave >> 2)][wave & 3] = mine;
      __syncthreads();
      if (wave < RP) {                             // a column each
        float x = 0.0f;
        if (lane < nslice) {
          const float4 w = *reinterpret_cast<const float4*>(part[wave][lane]);
          x = (w.x + w.y) + (w.z + w.w);
        }
        float sum = 0.0f;
#pragma unroll
        for (int sl = 0; sl < NS; ++sl) sum += __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(x), sl));   // (zeros beyond nslice)
        if (lane == 0) tot[wave] = sum;
      }
      __syncthreads();
      const float nrm2 = tot[j];
      const float inv = (nrm2 > FLT_MIN) ? 1.0f / sqrtf(nrm2) : 0.0f;
      float f[RP];
#pragma unroll
      for (int k = j + 1; k < RP; ++k) f[k] = -(tot[k] * inv);
#pragma unroll
      for (int i = 0; i < RPT; ++i) {
        const float qv = v[i][j] * inv;
        v[i][j] = qv;
#pragma unroll
        for (int k = j + 1; k < RP; ++k)
          if (k < r) v[i][k] = fmaf(f[k], qv, v[i][k]);
      }
    }
  }

  float mx = 0.0f;
  float* copy = a.orth_shared && a.padded ? a.Pop + ld.pop_off : nullptr;
  hide_row();
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    const int row = row0 + i * BS;
    if (row < rows) {
      store_row<RP>(orth + row * r, r, v[i]);
      if (copy) store_row<RP>(copy + row * RP, r, v[i]);
#pragma unroll
      for (int k = 0; k < RP; ++k) mx = fmaxf(mx, fabsf(v[i][k]));   // (zeros beyond r)
    }
  }
  mx = wave_max(mx);
  if (lane == 0) redmax[wave] = mx;
  __syncthreads();
  if (tid == 0 && !a.orth_shared) {
    float m = redmax[0];
#pragma unroll
    for (int wv = 1; wv < NW; ++wv) m = fmaxf(m, redmax[wv]);
    a.scaleP[(size_t)worker * a.L + layer] = m;
  }
}

// ---------------------------------------------------------------------------
// orth, one workgroup per (layer, worker), columns on lanes: lane (g, k) of a
// wavefront holds RPT rows of column k (C columns, 64 / C groups of rows), so a
// column's products with all later ones are RPT multiply-adds per lane and no
// sum over lanes at all: the column goes round its wavefront through LDS (its
// lane writes, all read the same words), the groups and wavefronts add up one
// value per column.  What bounds a column is this chain of LDS round trips and
// the one barrier; with rows on lanes (orth_reg_kernel) it is a butterfly over
// up to 64 values.  The loop over the columns is rolled: no register index
// depends on it, and the code stays a few KB at any rank (a workgroup runs it
// once).
//
// Every sum is the one that rows on lanes gives, to the last bit: products of
// rows t, t + 256, ... in a chain for each thread t < 256, a butterfly (32, 16,
// .. 1) over each 64 of these threads, then their wavefronts in order
// (t, t + 1024, ... and 16 wavefronts where WV = 16).  Where a factor is close
// to singular -- ranks clipped to a layer's width, later iterations of a high
// rank -- Gram-Schmidt magnifies the rounding of its sums by the factor's
// condition number, a thousand times and more: with the same products added in
// another order single values of G-hat move by 1e-4 of its root mean square, in
// one of eight runs of the ResNet-18 set at r = 50 by 3e-3.  So which rows a lane
// holds, and the order in which it goes through them, follow that tree: a lane
// holds the LL threads of one of its subtrees, in bit-reversed order, so that
// neighbouring partial sums always meet first.
// It serves heights from 513 rows on at rank pad 4 and from 2049 on at rank pad 8
// (130 factors of 10000 rows at r = 4: 27 us, rows on lanes 36), and up to 64
// rows at rank pad 32 where a set has more factors than CUs; elsewhere whole
// columns per wavefront (orth_colwave_kernel) are faster: their lanes end with
// their columns, here half of them work on columns that are done.
// ---------------------------------------------------------------------------
constexpr int bit_reverse(int x, int bits) { return bits == 0 ? 0 : ((x & 1) << (bits - 1)) | bit_reverse(x >> 1, bits - 1); }
constexpr int trailing_zeros(int x) { return (x & 1) ? 0 : 1 + trailing_zeros(x >> 1); }

template <int C, int WV, int NI, int NW>
__global__ __launch_bounds__(64 * NW) void orth_col_kernel(DevArgs a) {
  constexpr int G = kWave / C;
  constexpr int SUB = NW / WV;                   // wavefronts here per 64 threads of the tree
  constexpr int SP = SUB * G;                    // subtrees of 64 threads
  constexpr int LL = kWave / SP;                 // threads of a lane's subtree
  constexpr int RPT = LL * NI;                   // NI rows each
  constexpr int STEP = WV > 4 ? kWave * WV : 256;
  static_assert(NW % WV == 0 && SP <= kWave && RPT % 4 == 0 && (WV >= 4 || NI == 1), "");
  constexpr int PS = NW + 4;                     // pitch of a column's partials: 16-byte reads of 16 lanes hit all banks once
  __shared__ __attribute__((aligned(16))) float bc[NW][G][RPT];
  __shared__ __attribute__((aligned(16))) float part[2][C][PS];
  __shared__ float redmax[NW];
  const int lw = blockIdx.x;
  const int layer = lw / a.W, worker = lw - layer * a.W;
  const LayerDesc& ld = a.layers[layer];
  const int rows = ld.rows, r = ld.r, nseg = a.orth_shared ? 1 : ld.nseg;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int k = lane & (C - 1), g = lane / C;
  const float* Pp = a.Ppart + (size_t)worker * a.ppart_stride + (a.orth_shared ? ld.p_off : ld.ppart_off);
  float* pre = a.Ppre + (size_t)worker * a.p_stride + ld.p_off;
  float* orth = a.Porth + (size_t)worker * a.p_stride + ld.p_off;
  int row0 = (wave / SUB) * kWave + g * SUB + wave % SUB;
  // Many rows per lane: the optimiser would keep all their addresses in registers from one use to the next, and spill.
  auto hide_row = [&]() __attribute__((always_inline)) { if constexpr (RPT > 32) asm volatile("" : "+v"(row0)); };
  // row of the lane's value i, from row0
  auto row_of = [](int i) __attribute__((always_inline)) { return bit_reverse(i / NI, log2c(LL)) * SP + (i % NI) * STEP; };
  const bool col = k < r;
  const int kread = min(k, r - 1);

  float v[RPT];
#pragma unroll
  for (int i = 0; i < RPT; ++i) v[i] = 0.0f;
  // Elements beyond the factor re-read the last one of their row or column, in a line that is read anyhow (its first element would be
  // one more line in every load); they count as zeros from here on.
  for (int s = 0; s < nseg; ++s) {
    const float* src = Pp + (size_t)s * ld.np_pad;
    hide_row();
    constexpr int CH = RPT % 16 == 0 ? 16 : RPT % 14 == 0 ? 14 : RPT % 11 == 0 ? 11 : RPT;      // loads in flight
    static_assert(RPT % CH == 0, "");
#pragma unroll
    for (int i0 = 0; i0 < RPT; i0 += CH) {
      float t[CH];
#pragma unroll
      for (int i = 0; i < CH; ++i) {
        t[i] = src[min(row0 + row_of(i0 + i), rows - 1) * r + kread];
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < CH; ++i) v[i0 + i] += t[i];
    }
  }
  hide_row();
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    const int row = row0 + row_of(i);
    if (col && row < rows) pre[row * r + k] = v[i];
    else v[i] = 0.0f;
  }

  for (int j = 0; j < r; ++j) {
    constexpr bool KEEP = NW <= 8 || RPT <= 32;  // the column stays in registers between its two uses, or is read twice
    float4* mine = reinterpret_cast<float4*>(bc[wave][g]);
    if (k == j) {
#pragma unroll
      for (int i = 0; i < RPT / 4; ++i) mine[i] = make_float4(v[4 * i], v[4 * i + 1], v[4 * i + 2], v[4 * i + 3]);
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");   // DS operations of a wavefront stay in order
    __builtin_amdgcn_wave_barrier();
    auto fetch = [&](int i, float (&t)[4]) __attribute__((always_inline)) {
      const float4 x = mine[i];
      t[0] = x.x; t[1] = x.y; t[2] = x.z; t[3] = x.w;
    };
    float b[KEEP ? RPT / 4 : 1][4];
    float level[log2c(LL) + 1];                  // one open partial sum per level of the subtree
    float chain = 0.0f;
#pragma unroll
    for (int i = 0; i < RPT / 4; ++i) {
      float t[4];
      fetch(i, t);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int n = 4 * i + e, p = n / NI;     // value, thread of the subtree
        chain = fmaf(t[e], v[n], n % NI == 0 ? 0.0f : chain);
        if (n % NI == NI - 1) {                  // thread p is complete: close what ends with it
          const int top = trailing_zeros(p + 1);
          float sum = chain;
#pragma unroll
          for (int l = 0; l < log2c(LL); ++l)
            if (l < top) sum = level[l] + sum;
          level[top] = sum;
        }
        if constexpr (KEEP) b[i][e] = t[e];
      }
    }
    float s = level[log2c(LL)];
#pragma unroll
    for (int off = kWave / 2; off >= C; off >>= 1) s += __shfl_xor(s, off, kWave);
    float* mypart = part[j & 1][k];
    if (g == 0) mypart[wave] = s;
    __syncthreads();
    float pw[NW];
#pragma unroll
    for (int w = 0; w < NW; w += 4) {
      const float4 t = *reinterpret_cast<const float4*>(mypart + w);
      pw[w] = t.x; pw[w + 1] = t.y; pw[w + 2] = t.z; pw[w + 3] = t.w;
    }
#pragma unroll
    for (int wv = 0; wv < WV; ++wv)
#pragma unroll
      for (int h = SUB / 2; h >= 1; h /= 2)
#pragma unroll
        for (int i = 0; i < h; ++i) pw[wv * SUB + i] += pw[wv * SUB + i + h];
    s = pw[0];
#pragma unroll
    for (int wv = 1; wv < WV; ++wv) s += pw[wv * SUB];
    const float nrm2 = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(s), j));
    const float inv = (nrm2 > FLT_MIN) ? 1.0f / sqrtf(nrm2) : 0.0f;
    const float f = -(s * inv);
    if (k > j) {
#pragma unroll
      for (int i = 0; i < RPT / 4; ++i) {
        float t[4];
        if constexpr (KEEP) {
#pragma unroll
          for (int e = 0; e < 4; ++e) t[e] = b[i][e];
        } else {
          fetch(i, t);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float qv = t[e] * inv;
          v[4 * i + e] = fmaf(f, qv, v[4 * i + e]);
        }
      }
    } else if (k == j) {
#pragma unroll
      for (int i = 0; i < RPT; ++i) v[i] *= inv;
    }
  }

  float mx = 0.0f;
  float* copy = a.orth_shared && a.padded ? a.Pop + ld.pop_off : nullptr;   // the sweeps' copy of an orthonormalised aggregate
  hide_row();
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    const int row = row0 + row_of(i);
    if (col && row < rows) {
      orth[row * r + k] = v[i];
      if (copy) copy[row * C + k] = v[i];
      mx = fmaxf(mx, fabsf(v[i]));
    }
  }
  mx = wave_max(mx);
  if (lane == 0) redmax[wave] = mx;
  __syncthreads();
  if (tid == 0 && !a.orth_shared) {
    float m = redmax[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) m = fmaxf(m, redmax[w]);
    a.scaleP[(size_t)worker * a.L + layer] = m;
  }
}

// ---------------------------------------------------------------------------
// orth, one workgroup per (layer, worker), whole columns to a wavefront: its
// lanes hold the rows (lane l: rows l, l + 64, ..), and it owns blocks of BC
// neighbouring columns.  A finished column goes to the other wavefronts through
// LDS, where each column has a place of its own or, where the factor is larger
// than LDS, one in a ring; a wavefront waits for a column by its number, takes
// its products with its own later columns and removes it from them, and when
// its next block is complete it finishes that block at once.  There is no
// barrier between columns; the inverse of a column's norm follows the column,
// so that products with it are taken while it is computed.
//
// What bounds it: about 40 vector instructions for each pair of columns on one
// CU (30 of 47 us at 512 rows, r = 50), then the chain from column to column,
// a trip through LDS for every BC of them.  Gram-Schmidt of a set, microseconds
// before (columns on lanes, orth_col_kernel) and now: ResNet-18 set, W = 8,
// r = 7 12.1 -> 10.2, r = 16 20.4 -> 14.1, r = 32 40 -> 26, r = 50 94 -> 49;
// ragged set, r = 20 44 -> 23; 2 x (1000 x 640), W = 4, r = 50 179 -> 61;
// 2 x (1700 x 640), r = 20 73 -> 33; 640 factors of 250 rows at r = 64
// 210 -> 121.  (8 or 4 wavefronts instead of 16 at r = 32: 31 and 39 us; blocks
// of 1 and 4 columns at r = 50 56 and 53; pauses in the waiting loops, or a
// higher priority for the wavefront next in line while it waits: no gain.)
//
// The sums are those of orth_col_kernel, to the last bit: c[w] is the chain of
// rows l + 64 w, + 256, .., the reduction adds lanes 32, 16, .. 1 apart, the
// NB wavefronts of that order come last, one after the other or in pairs.
// Waits end: a column waits only for columns before it, its wavefront publishes
// in order, and all wavefronts of a workgroup are resident.
// ---------------------------------------------------------------------------
// Sum over the lanes of each c[w], then over w.
template <int NB, bool PAIRS>
__device__ __forceinline__ float column_total(const float (&c)[NB]) {
  float x;
  if constexpr (NB == 4) {
    x = four_lane_sums(c);
  } else {
    const float u = NB == 2 ? swap32_add(c[0], c[NB - 1]) : swap32_add(c[0], c[0]);
    x = row_sums(swap16_add(u, u));
  }
  auto at = [&](int l) __attribute__((always_inline)) { return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(x), l)); };
  if constexpr (NB == 4) {
    return PAIRS ? (at(0) + at(32)) + (at(16) + at(48)) : ((at(0) + at(32)) + at(16)) + at(48);
  } else {
    return NB == 2 ? at(0) + at(32) : at(0);
  }
}

// C: rank pad.  Up to 64 NB rows (NI = 1) or 256 NI (NB = 4).  BC: neighbouring columns of a wavefront.  NIC: 256-row blocks of the
// factor that go through LDS at once on their way in and out.  SLOTS: columns in LDS (C: each its own).
template <int C, int NB, int NI, int NW, int BC, int NIC, int SLOTS, bool PAIRS>
__global__ __launch_bounds__(64 * NW) void orth_colwave_kernel(DevArgs a) {
  constexpr int NT = 64 * NW, CPW = C / NW, RPT = NB * NI, BR = kWave * NB;      // BR: rows of a block
  constexpr int CPIN = NIC * BR + 1, CP = NI * BR;                           // pitches of a column, floats
  constexpr int POOL = C * CPIN > SLOTS * CP ? C * CPIN : SLOTS * CP;
  static_assert(CPW >= 1 && CPW % BC == 0 && NI % NIC == 0 && (NI == 1 || NB == 4) && (SLOTS == C || (SLOTS % 2 == 0 && BC <= SLOTS / 2)), "");
  __shared__ __attribute__((aligned(16))) float pool[POOL];
  __shared__ float s_inv[C];
  __shared__ int ready;                          // columns published
  __shared__ float redmax[NW];
  const int lw = blockIdx.x;
  const int layer = lw / a.W, worker = lw - layer * a.W;
  const LayerDesc& ld = a.layers[layer];
  const int rows = ld.rows, r = ld.r, nseg = a.orth_shared ? 1 : ld.nseg;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const float* Pp = a.Ppart + (size_t)worker * a.ppart_stride + (a.orth_shared ? ld.p_off : ld.ppart_off);
  float* pre = a.Ppre + (size_t)worker * a.p_stride + ld.p_off;
  float* orth = a.Porth + (size_t)worker * a.p_stride + ld.p_off;
  auto col_of = [&](int s) __attribute__((always_inline)) { return (s / BC * NW + wave) * BC + s % BC; };
  const unsigned magic = r > 1 ? 0xffffffffu / (unsigned)r + 1u : 0u;
  // row and column of element e of the factor (e < 2^17, r <= 64: exact)
  auto row_of = [&](int e) __attribute__((always_inline)) { return r > 1 ? (int)__umulhi((unsigned)e, magic) : e; };

  // ---- the factor: planes added in memory order, columns handed out through LDS
  constexpr int F4 = (NIC * BR * C / 4 + NT - 1) / NT;
  float v[CPW][RPT];
  if (tid == 0) ready = 0;
  if (tid < C) s_inv[tid] = -1.0f;               // (no norm's inverse)
#pragma unroll
  for (int ch = 0; ch < NI / NIC; ++ch) {
    const int row0 = ch * NIC * BR, el0 = row0 * r, el1 = min(rows, row0 + NIC * BR) * r;   // el0 is a multiple of 4
    if (ch > 0) __syncthreads();
    if (el0 < el1) {
      float4 acc[F4], x[F4];
#pragma unroll
      for (int i = 0; i < F4; ++i) acc[i] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      for (int s = 0; s < nseg; ++s) {
        const float* src = Pp + (size_t)s * ld.np_pad;
#pragma unroll
        for (int i = 0; i < F4; ++i) {
          const int e = el0 + 4 * (tid + NT * i);
          x[i] = *reinterpret_cast<const float4*>(src + (e < el1 ? e : 0));
        }
#pragma unroll
        for (int i = 0; i < F4; ++i) { acc[i].x += x[i].x; acc[i].y += x[i].y; acc[i].z += x[i].z; acc[i].w += x[i].w; }
      }
#pragma unroll
      for (int i = 0; i < F4; ++i) {
        const int e = el0 + 4 * (tid + NT * i);
        if (e < el1) {                           // (what lies beyond goes to rows that are not the factor's and count as zeros)
          const float t[4] = {acc[i].x, acc[i].y, acc[i].z, acc[i].w};
          int row = row_of(e), k = e - row * r;
          row -= row0;
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            pool[k * CPIN + row] = t[q];
            if (++k == r) { k = 0; ++row; }
          }
          if (e + 4 <= el1) *reinterpret_cast<float4*>(pre + e) = acc[i];
          else
            for (int q = 0; q < el1 - e; ++q) pre[e + q] = t[q];
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int s = 0; s < CPW; ++s) {
      const int k = col_of(s);
#pragma unroll
      for (int i = 0; i < NIC; ++i)
#pragma unroll
        for (int w = 0; w < NB; ++w) {
          const float t = pool[k * CPIN + i * BR + w * kWave + lane];
          v[s][(ch * NIC + i) * NB + w] = (k < r && row0 + i * BR + w * kWave + lane < rows) ? t : 0.0f;
        }
    }
  }
  __syncthreads();

  typedef volatile int __attribute__((address_space(3)))* lds_word;    // (a generic pointer's accesses have no order among DS ones)
  const lds_word flag = (lds_word)&ready;
  typedef volatile float __attribute__((address_space(3)))* lds_float;
  const lds_float invs = (lds_float)s_inv;
  auto dot = [&](const float (&x)[RPT], const float (&y)[RPT]) __attribute__((always_inline)) {
    float c[NB];
#pragma unroll
    for (int w = 0; w < NB; ++w) c[w] = 0.0f;
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int w = 0; w < NB; ++w) c[w] = fmaf(x[i * NB + w], y[i * NB + w], c[w]);
    return column_total<NB, PAIRS>(c);
  };
  auto update = [&](float (&y)[RPT], const float (&x)[RPT], float sum, float inv) __attribute__((always_inline)) {
    const float f = -(sum * inv);
#pragma unroll
    for (int i = 0; i < RPT; ++i) y[i] = fmaf(f, x[i] * inv, y[i]);
  };
  // Finishes the wavefront's columns s0 .. s0 + BC - 1, from which all earlier ones have been removed: hands each out, the inverse
  // of its norm after it, removes it from those after it, and normalises it.
  auto finish = [&](auto s0) __attribute__((always_inline)) {
    static_for<BC>([&](auto c) __attribute__((always_inline)) {
      constexpr int s = s0.value + c.value;
      const int k = col_of(s);
      if (k < r) {
        float* to = pool + (SLOTS == C ? k : k % SLOTS) * CP + lane * NB;
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
          for (int w = 0; w < NB; ++w) to[i * BR + w] = v[s][i * NB + w];
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");   // DS operations of a wavefront stay in order
        __builtin_amdgcn_wave_barrier();
        *flag = k + 1;
        float sum[BC];
#pragma unroll
        for (int d = c.value; d < BC; ++d) sum[d] = dot(v[s], v[s0.value + d]);
        const float nrm2 = sum[c.value];
        const float inv = (nrm2 > FLT_MIN) ? 1.0f / sqrtf(nrm2) : 0.0f;
        invs[k] = inv;
#pragma unroll
        for (int d = c.value + 1; d < BC; ++d) update(v[s0.value + d], v[s], sum[d], inv);
#pragma unroll
        for (int i = 0; i < RPT; ++i) v[s][i] *= inv;
      }
    });
  };
  if (wave == 0) finish(std::integral_constant<int, 0>{});
  for (int j = 0; j + 1 < r; ++j) {
    if constexpr (SLOTS < C) {
      if (j > 0 && j % (SLOTS / 2) == 0) __syncthreads();    // columns before j are done with, and so are their places
    }
    if (col_of(CPW - BC) <= j) {                 // the wavefront's columns are all done
      if constexpr (SLOTS < C) continue;
      else break;
    }
    while (__builtin_amdgcn_readfirstlane(*flag) <= j) {}
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    float b[RPT];
    const float* from = pool + (SLOTS == C ? j : j % SLOTS) * CP + lane * NB;
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int w = 0; w < NB; ++w) b[i * NB + w] = from[i * BR + w];
    float inv = -1.0f;
    static_for<CPW / BC>([&](auto q) __attribute__((always_inline)) {
      constexpr int s0 = q.value * BC;
      const int k0 = col_of(s0);
      if (k0 > j && k0 < r) {
        if (k0 == j + 1) __builtin_amdgcn_s_setprio(3);
        float sum[BC];
#pragma unroll
        for (int c = 0; c < BC; ++c) sum[c] = dot(b, v[s0 + c]);
        while (inv < 0.0f) inv = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(invs[j])));
#pragma unroll
        for (int c = 0; c < BC; ++c) update(v[s0 + c], b, sum[c], inv);
        if (k0 == j + 1) {
          finish(std::integral_constant<int, s0>{});
          __builtin_amdgcn_s_setprio(0);
        }
      }
    });
  }

  // ---- back to memory, in its order
  float mx = 0.0f;
  float* copy = a.orth_shared && a.padded ? a.Pop + ld.pop_off : nullptr;   // the sweeps' copy of an orthonormalised aggregate
#pragma unroll
  for (int ch = 0; ch < NI / NIC; ++ch) {
    const int row0 = ch * NIC * BR, el0 = row0 * r, el1 = min(rows, row0 + NIC * BR) * r;
    __syncthreads();
#pragma unroll
    for (int s = 0; s < CPW; ++s) {
      const int k = col_of(s);
#pragma unroll
      for (int i = 0; i < NIC; ++i)
#pragma unroll
        for (int w = 0; w < NB; ++w) pool[k * CPIN + i * BR + w * kWave + lane] = v[s][(ch * NIC + i) * NB + w];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < F4; ++i) {
      const int e = el0 + 4 * (tid + NT * i);
      if (e < el1) {
        float t[4];
        int row = row_of(e), k = e - row * r;
#pragma unroll
        for (int q = 0; q < 4; ++q) {              // (rows beyond the factor's are zeros)
          t[q] = pool[k * CPIN + row - row0];
          mx = fmaxf(mx, fabsf(t[q]));
          if (copy && e + q < el1) copy[row * C + k] = t[q];
          if (++k == r) { k = 0; ++row; }
        }
        if (e + 4 <= el1) *reinterpret_cast<float4*>(orth + e) = make_float4(t[0], t[1], t[2], t[3]);
        else
          for (int q = 0; q < el1 - e; ++q) orth[e + q] = t[q];
      }
    }
  }
  mx = wave_max(mx);
  if (lane == 0) redmax[wave] = mx;
  __syncthreads();
  if (tid == 0 && !a.orth_shared) {
    float m = redmax[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) m = fmaxf(m, redmax[w]);
    a.scaleP[(size_t)worker * a.L + layer] = m;
  }
}

// ---------------------------------------------------------------------------
// orth, many workgroups per (layer, worker): for tall factors with few
// (layer, worker) pairs, where one workgroup each would leave the chip idle.
// The rows are cut into slices of 256; launch j (j = 0 .. r) applies the update
// of column j-1 to its slice (using the block-wide totals of launch j-1, added
// up over the slices in slice order) and then forms its slice's partial dot
// products of column j with the columns after it.  The grid-wide dependency
// between columns is the kernel boundary.  Launch 0 sums the sweep-0 partials,
// launch r finishes with absmax(P_w) through an integer atomic max.
// only_if (optional): one word per (layer, worker) pair, written by an earlier
// kernel; the launches skip the pairs whose lowest bit is zero, and do nothing
// where the first word is.
// ---------------------------------------------------------------------------
// The factor and the slice that workgroup `block` has: the slices of all factors in a row, a layer's workers one after the other.
// (A grid of the tallest factor's slices for every factor is mostly empty where heights differ, and too many for one cooperative
// launch: 10 layers of up to 6848 rows, r = 21, W = 4, 1080 workgroups for 284 slices, Gram-Schmidt 150 us in three launches, 79 in
// one; 4000 x 300 beside 10 x (500 x 600), r = 40, W = 8 477 and 160.)
__device__ __forceinline__ void slice_of(const DevArgs& a, int block, int nslice_max, int& lw, int& slice) {
  if (a.slices == a.L * nslice_max) {            // all as tall
    lw = block / nslice_max;
    slice = block - lw * nslice_max;
    return;
  }
  const int lane = threadIdx.x & (kWave - 1);
  int layer = -1;
  for (int base = 0; base < a.L; base += kWave) {
    const bool at_or_before = base + lane < a.L && a.W * a.layers[base + lane].slice0 <= block;
    const int n = __popcll(__ballot(at_or_before));
    layer += n;
    if (n < kWave) break;
  }
  layer = __builtin_amdgcn_readfirstlane(layer);
  const int in_layer = block - a.W * a.layers[layer].slice0, n = (a.layers[layer].rows + 255) >> 8;
  const int worker = in_layer / n;
  lw = layer * a.W + worker;
  slice = in_layer - worker * n;
}

// Products of a column with all columns, summed over a wavefront's lanes as transpose_reduce does.  A single product (RP = 1) meets
// its partner's before it is rounded.
template <int RP>
__device__ __forceinline__ void column_products(float vj, const float (&v)[RP], float (&s)[RP], int lane) {
#pragma unroll
  for (int k = 0; k < RP; ++k) s[k] = vj * v[k];
  if constexpr (RP == 1) {
    s[0] = fmaf(vj, v[0], __shfl_xor(s[0], 32, kWave));
    transpose_reduce<1, 1, 16>(s, lane);
  } else {
    transpose_reduce<RP, RP, 32>(s, lane);
  }
}

template <int RP>
__global__ __launch_bounds__(256) void orth_wide_kernel(DevArgs a, int j, int nslice_max, const int* only_if) {
  __shared__ float red[4][RP];
  __shared__ float redmax[4];
  if (only_if && only_if[0] == 0) return;        // no pair has to be done column by column
  int lw, slice;
  slice_of(a, blockIdx.x, nslice_max, lw, slice);
  if (only_if && (only_if[lw] & 1) == 0) return; // this pair was finished by the Cholesky-QR kernels
  const int layer = lw / a.W, worker = lw - layer * a.W;
  const LayerDesc& ld = a.layers[layer];
  const int rows = ld.rows, r = ld.r;
  const int nslice = (rows + 255) >> 8;
  if (j > r) return;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
  const int row = slice * 256 + tid;
  const bool live = row < rows;
  float* pre = a.Ppre + (size_t)worker * a.p_stride + ld.p_off;
  float* orth = a.Porth + (size_t)worker * a.p_stride + ld.p_off;
  float* part = a.orth_part;    // [2][L*W][nslice_max][RP]
  const size_t pstride = (size_t)a.L * a.W * nslice_max * RP;
  float v[RP];
#pragma unroll
  for (int k = 0; k < RP; ++k) v[k] = 0.0f;
  if (j == 0) {
    if (slice == 0 && tid == 0 && !a.orth_shared) a.scaleP[(size_t)worker * a.L + layer] = 0.0f;
    if (live) {
      if (only_if) {
        // The Cholesky-QR kernels have left the sum of the planes in `pre`, and where Gram-Schmidt
        // runs in place (the plane is the output) they have overwritten the plane itself.
#pragma unroll
        for (int k = 0; k < RP; ++k)
          if (k < r) v[k] = pre[(size_t)row * r + k];
      } else {
        const float* Pp = a.Ppart + (size_t)worker * a.ppart_stride + (a.orth_shared ? ld.p_off : ld.ppart_off);
        const int nseg = a.orth_shared ? 1 : ld.nseg;
        for (int s = 0; s < nseg; ++s) {
          const float* src = Pp + (size_t)s * ld.np_pad + (size_t)row * r;
#pragma unroll
          for (int k = 0; k < RP; ++k)
            if (k < r) v[k] += src[k];
        }
      }
#pragma unroll
      for (int k = 0; k < RP; ++k)
        if (k < r) {
          pre[(size_t)row * r + k] = v[k];
          orth[(size_t)row * r + k] = v[k];
        }
    }
  } else {
    const int c = j - 1;                         // the column this launch finishes
    const float* pin = part + (size_t)(c & 1) * pstride + (size_t)lw * nslice_max * RP;
    float tot[RP];
#pragma unroll
    for (int k = 0; k < RP; ++k) tot[k] = 0.0f;
    for (int s = 0; s < nslice; ++s) {
#pragma unroll
      for (int k = 0; k < RP; ++k) tot[k] += pin[(size_t)s * RP + k];
    }
    float nrm2 = 0.0f;
#pragma unroll
    for (int k = 0; k < RP; ++k)
      if (k == c) nrm2 = tot[k];
    const float inv = (nrm2 > FLT_MIN) ? 1.0f / sqrtf(nrm2) : 0.0f;
    if (live) {
      float* dst = orth + (size_t)row * r;
#pragma unroll
      for (int k = 0; k < RP; ++k)
        if (k < r) v[k] = dst[k];
      float qv = 0.0f;
#pragma unroll
      for (int k = 0; k < RP; ++k)
        if (k == c) qv = v[k] * inv;
#pragma unroll
      for (int k = 0; k < RP; ++k) {
        if (k == c) v[k] = qv;
        else if (k > c && k < r) v[k] = fmaf(-(tot[k] * inv), qv, v[k]);
      }
#pragma unroll
      for (int k = 0; k < RP; ++k)
        if (k >= c && k < r) dst[k] = v[k];
    }
  }
  if (j < r) {
    // partial <column j, column k> over this slice, every k (entries k < j are not used)
    float vj = 0.0f;
#pragma unroll
    for (int k = 0; k < RP; ++k)
      if (k == j) vj = v[k];
    float s[RP];
    column_products<RP>(vj, v, s, lane);
    if ((lane & (kWave / RP - 1)) == 0) red[wave][lane >> (6 - log2c(RP))] = s[0];
    __syncthreads();
    if (tid < RP)
      part[(size_t)(j & 1) * pstride + ((size_t)lw * nslice_max + slice) * RP + tid] =
          (red[0][tid] + red[1][tid]) + (red[2][tid] + red[3][tid]);
  } else {
    float mx = 0.0f;
#pragma unroll
    for (int k = 0; k < RP; ++k)
      if (k < r) mx = fmaxf(mx, fabsf(v[k]));
    mx = wave_max(mx);
    if (lane == 0) redmax[wave] = mx;
    __syncthreads();
    if (tid == 0 && !a.orth_shared) {
      const float m = fmaxf(fmaxf(redmax[0], redmax[1]), fmaxf(redmax[2], redmax[3]));
      atomicMax(reinterpret_cast<unsigned int*>(a.scaleP + (size_t)worker * a.L + layer), __float_as_uint(m));
    }
  }
}

// ---------------------------------------------------------------------------
// orth, many workgroups per (layer, worker), one launch: the same slicing as
// orth_wide_kernel, but every workgroup keeps its 256 rows in registers through
// all columns, and the slices of a (layer, worker) pair exchange their partial
// dot products through a table in memory while the kernel runs.  The kernel is
// launched cooperatively, so all workgroups are resident and no slice waits
// for one that cannot start.
// A table entry is 64 bits: the partial <column j, column k> of one slice and a
// tag naming the launch and the column, written with ONE device-scope atomic
// store.  A reader polls an entry until it carries the tag it expects: value
// and "ready" arrive together, there is no counter and no fence (a device-
// scope fence writes back and invalidates a die's whole L2: ~100 us per column
// measured; the runtime's grid barrier ~65 us).  All entries of a pair are
// polled in parallel (one or a few per thread), collected in LDS and added up
// in slice order.  The table is double-buffered by column parity: a slice can
// only write column j + 2 after it has read every slice's column j + 1, which
// they write only after they have finished reading column j.
// Every wait is bounded; if one ever expires the workgroup raises the status
// word and carries on, so the kernel always ends.
// ---------------------------------------------------------------------------
[[maybe_unused]] constexpr unsigned kTablePolls = 1u << 20;      // default bound of a wait (about a second)
constexpr int kCoopMaxSlices = 64;               // rows <= 16384 per factor in this form

__device__ __forceinline__ unsigned long long table_load(const unsigned long long* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The columns of one slice, all r of them: v holds the slice's rows (one per thread) and leaves
// orthonormalised.  red [4 RP], tot_s [RP] and gather_s [kCoopMaxSlices RP] are LDS.
template <int RP>
__device__ __forceinline__ void coop_columns(float (&v)[RP], int r, int lw, int slice, int nslice, int nslice_max, int max_rank,
                                             unsigned long long* table, unsigned long long epoch, int* status,
                                             unsigned max_polls, size_t pstride, float* red, float* tot_s, float* gather_s) {
  constexpr int EPT = (kCoopMaxSlices * RP + 255) / 256;     // table entries a thread collects per column
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
  const int nent = nslice * RP;
  for (int j = 0; j < r; ++j) {                  // r is the same for every slice of the pair
    const unsigned tag = (unsigned)(epoch * (unsigned long long)max_rank + (unsigned long long)(j + 1));
    unsigned long long* tab = table + (size_t)(j & 1) * pstride + (size_t)lw * nslice_max * RP;
    float vj = 0.0f;
#pragma unroll
    for (int k = 0; k < RP; ++k)
      if (k == j) vj = v[k];
    float s[RP];
    column_products<RP>(vj, v, s, lane);
    if ((lane & (kWave / RP - 1)) == 0) red[wave * RP + (lane >> (6 - log2c(RP)))] = s[0];
    __syncthreads();
    if (tid < RP) {
      const float val = (red[tid] + red[RP + tid]) + (red[2 * RP + tid] + red[3 * RP + tid]);
      __hip_atomic_store(tab + (size_t)slice * RP + tid, ((unsigned long long)tag << 32) | __float_as_uint(val),
                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // collect every slice's entry for this column
    unsigned long long x[EPT];
#pragma unroll
    for (int i = 0; i < EPT; ++i) {
      const int e = tid + i * 256;
      x[i] = (e < nent) ? table_load(tab + e) : ((unsigned long long)tag << 32);
    }
#pragma unroll
    for (int i = 0; i < EPT; ++i) {
      const int e = tid + i * 256;
      unsigned polls = 0;
      while ((unsigned)(x[i] >> 32) != tag) {
        if (++polls >= max_polls) {
          __hip_atomic_store(status, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
          break;
        }
        __builtin_amdgcn_s_sleep(1);
        x[i] = table_load(tab + e);
      }
      if (e < nent) gather_s[e] = __uint_as_float((unsigned)x[i]);
    }
    __syncthreads();
    if (tid < RP) {
      float t = 0.0f;
      for (int sl = 0; sl < nslice; ++sl) t += gather_s[sl * RP + tid];
      tot_s[tid] = t;
    }
    __syncthreads();
    const float nrm2 = tot_s[j];
    const float inv = (nrm2 > FLT_MIN) ? 1.0f / sqrtf(nrm2) : 0.0f;
    float qv = 0.0f;
#pragma unroll
    for (int k = 0; k < RP; ++k)
      if (k == j) qv = v[k] * inv;
#pragma unroll
    for (int k = 0; k < RP; ++k) {
      if (k == j) v[k] = qv;
      else if (k > j && k < r) v[k] = fmaf(-(tot_s[k] * inv), qv, v[k]);
    }
    __syncthreads();                             // red, gather_s and tot_s are reused by the next column
  }
}

template <int RP>
__global__ __launch_bounds__(256) void orth_coop_kernel(DevArgs a, int nslice_max, int max_rank,
                                                        unsigned long long* table, unsigned long long epoch,
                                                        int* status, unsigned max_polls) {
  __shared__ float red[4 * RP];
  __shared__ float tot_s[RP];
  __shared__ float gather_s[kCoopMaxSlices * RP];
  __shared__ float redmax[4];
  int lw, slice;
  slice_of(a, blockIdx.x, nslice_max, lw, slice);
  const int layer = lw / a.W, worker = lw - layer * a.W;
  const LayerDesc& ld = a.layers[layer];
  const int rows = ld.rows, r = ld.r;
  const int nslice = (rows + 255) >> 8;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
  const int row = slice * 256 + tid;
  const bool live = row < rows;
  float* pre = a.Ppre + (size_t)worker * a.p_stride + ld.p_off;
  float* orth = a.Porth + (size_t)worker * a.p_stride + ld.p_off;
  const size_t pstride = (size_t)a.L * a.W * nslice_max * RP;   // [2][L*W][nslice_max][RP] entries
  float v[RP];
#pragma unroll
  for (int k = 0; k < RP; ++k) v[k] = 0.0f;
  // The absmax cell is shared by all slices: zeroed here with a device-scope store, raised with
  // atomics at the end.  Every slice reads slice 0's first table entry before it gets there.
  if (slice == 0 && tid == 0 && !a.orth_shared) {
    __hip_atomic_store(a.scaleP + (size_t)worker * a.L + layer, 0.0f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __builtin_amdgcn_s_waitcnt(0x0F70);          // vmcnt(0): acknowledged before this slice publishes anything
  }
  if (live) {
    const float* Pp = a.Ppart + (size_t)worker * a.ppart_stride + (a.orth_shared ? ld.p_off : ld.ppart_off);
    const int nseg = a.orth_shared ? 1 : ld.nseg;
    for (int s = 0; s < nseg; ++s) {
      const float* src = Pp + (size_t)s * ld.np_pad + (size_t)row * r;
#pragma unroll
      for (int k = 0; k < RP; ++k)
        if (k < r) v[k] += src[k];
    }
#pragma unroll
    for (int k = 0; k < RP; ++k)
      if (k < r) pre[(size_t)row * r + k] = v[k];
  }
  coop_columns<RP>(v, r, lw, slice, nslice, nslice_max, max_rank, table, epoch, status, max_polls, pstride, red, tot_s,
                   gather_s);
  float mx = 0.0f;
  if (live) {
#pragma unroll
    for (int k = 0; k < RP; ++k)
      if (k < r) {
        orth[(size_t)row * r + k] = v[k];
        mx = fmaxf(mx, fabsf(v[k]));
      }
  }
  mx = wave_max(mx);
  if (lane == 0) redmax[wave] = mx;
  __syncthreads();
  if (tid == 0 && !a.orth_shared) {
    const float m = fmaxf(fmaxf(redmax[0], redmax[1]), fmaxf(redmax[2], redmax[3]));
    atomicMax(reinterpret_cast<unsigned int*>(a.scaleP + (size_t)worker * a.L + layer), __float_as_uint(m));
  }
}

// ---------------------------------------------------------------------------
// exchange: LogQuantize (Eq. (5) discretised to 2^b levels, Section 4.1),
// pack, LogDequantize (Eq. (6)) and the mean over workers that stands in for
// the All-Reduce.
//   kQuantOnly: factors -> packets      kMeanOnly: packets -> mean
//   kFused:     factors -> packets and mean in one pass
// A workgroup takes kXBlockGroups groups of 8 consecutive factor elements; a
// lane handles one (group, worker) pair -- b magnitude bytes + 1 sign byte --
// eight workers at a time; the dequantised values meet in LDS, where thread e
// adds up element e of the workgroup's 256 over the workers in worker order.
// What bounds it at high ranks is the quantiser's arithmetic (see quantise_group).
// ---------------------------------------------------------------------------
template <int MODE>
__global__ __launch_bounds__(256) void exchange_kernel(DevArgs a, const XTile* __restrict__ tiles, int phase) {
  __shared__ float s_tab[258];                         // thresholds, NaN before and after them
  __shared__ float s_lev[256];
  __shared__ __attribute__((aligned(16))) float s_val[8][kXGroup * kXBlockGroups];   // [worker slot][element]
  const int bits = phase ? a.bits_q : a.bits_p;
  const int lv = (1 << bits) - 1;
  const int tid = threadIdx.x;
  float thr0 = 0.0f, lev0 = 0.0f;
  if (bits > 0) {
    thr0 = gptr<float>(phase ? a.thrQ : a.thrP)[min(tid, max(lv - 1, 0))];
    lev0 = gptr<float>(phase ? a.levQ : a.levP)[min(tid, lv)];
  }
  const XTile tl = tiles[blockIdx.x];
  const LayerDesc& ld = a.layers[tl.layer];
  const int n_el = phase ? ld.nq_el : ld.np_el;
  const int gl = tid & (kXBlockGroups - 1);
  const int slot = tid / kXBlockGroups;            // worker slot
  const int g = tl.grp0 + gl;
  const int e0 = g * kXGroup;
  const bool gvalid = e0 < n_el;
  const int nvalid = gvalid ? min(kXGroup, n_el - e0) : 0;
  const size_t fstride = phase ? a.q_stride : a.p_stride;
  const float* fac = (phase ? a.Qw + ld.q_off : a.Porth + ld.p_off) + e0;
  uint8_t* mag = (phase ? a.magQ + ld.magq_off : a.magP + ld.magp_off) + (size_t)g * bits;
  uint8_t* sgn = (phase ? a.sgnQ + ld.sgnq_off : a.sgnP + ld.sgnp_off) + g;
  const size_t mstride = phase ? a.magq_stride : a.magp_stride;
  const size_t sstride = phase ? a.sgnq_stride : a.sgnp_stride;
  const float* scale = phase ? a.scaleQ : a.scaleP;
  const float qscale = phase ? a.qscale_q : a.qscale_p;

  // A worker's group and its absmax.  The first ones are requested before the tables are waited for, and each worker's while the
  // one before it is quantised: at low ranks this kernel is nothing but a chain of trips to memory.
  float4 lo = make_float4(0.0f, 0.0f, 0.0f, 0.0f), hi = lo;
  float s_next = 0.0f;
  auto request = [&](int w) __attribute__((always_inline)) {
    if (gvalid && w < a.W) {
      if (MODE != kMeanOnly || bits == 0) {
        lo = reinterpret_cast<const float4*>(fac + (size_t)w * fstride)[0];
        hi = reinterpret_cast<const float4*>(fac + (size_t)w * fstride)[1];
      }
      if (bits > 0) s_next = scale[(size_t)w * a.L + tl.layer];
    }
  };
  request(slot);
  __builtin_amdgcn_sched_barrier(0);
  if (bits > 0) {
    if (tid < lv) s_tab[1 + tid] = thr0;
    if (tid <= lv) s_lev[tid] = lev0;
    if (tid < 2) s_tab[tid * (lv + 1)] = __uint_as_float(0x7fc00000u);
    __syncthreads();
  }

  float acc = 0.0f;
  for (int wbase = 0; wbase < a.W; wbase += 8) {
    const int w = wbase + slot;
    float val[kXGroup];
#pragma unroll
    for (int i = 0; i < kXGroup; ++i) val[i] = 0.0f;
    float x[kXGroup] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
    const float s = s_next;
    request(w + 8);
    if (gvalid && w < a.W) {
      if (MODE != kMeanOnly || bits == 0) {
#pragma unroll
        for (int i = 0; i < kXGroup; ++i)
          if (i >= nvalid) x[i] = 0.0f;
      }
      if (bits == 0) {
#pragma unroll
        for (int i = 0; i < kXGroup; ++i) val[i] = x[i];
      } else {
        if (MODE != kMeanOnly) {
          uint8_t* mp = mag + (size_t)w * mstride;
          uint8_t* sp = sgn + (size_t)w * sstride;
          // (s between 2^-60 and 2^60: neither the reciprocal nor a remainder that matters leaves the normal range)
          if (a.quant_fast && s > 0x1p-60f && s < 0x1p60f)
            quantise_group<true>(x, s, bits, lv, a.alpha, qscale, s_tab + 1, s_lev, mp, sp, val);
          else
            quantise_group<false>(x, s, bits, lv, a.alpha, qscale, s_tab + 1, s_lev, mp, sp, val);
        } else {
          unsigned long long magbits = 0;
          const uint8_t* mp = mag + (size_t)w * mstride;
          for (int bb = 0; bb < bits; ++bb) magbits |= (unsigned long long)mp[bb] << (8 * bb);
          const unsigned sgnbits = sgn[(size_t)w * sstride];
#pragma unroll
          for (int i = 0; i < kXGroup; ++i) {
            const int k = (int)((magbits >> (i * bits)) & (unsigned long long)lv);
            const float v = s * s_lev[k];
            val[i] = ((sgnbits >> i) & 1u) ? -v : v;
          }
        }
      }
    }
    if (MODE != kQuantOnly) {
      float4* mine = reinterpret_cast<float4*>(s_val[slot] + gl * kXGroup);
      mine[0] = make_float4(val[0], val[1], val[2], val[3]);
      mine[1] = make_float4(val[4], val[5], val[6], val[7]);
      __syncthreads();
      const int nw = min(8, a.W - wbase);
      for (int sidx = 0; sidx < nw; ++sidx) acc += s_val[sidx][tid];
      __syncthreads();
    }
  }
  if (MODE != kQuantOnly) {
    const int e = tl.grp0 * kXGroup + tid;       // a workgroup's elements are consecutive, one per thread
    if (e < n_el) {
      const float mean = acc / (float)a.W;
      (phase ? a.Qbar + ld.q_off : a.Pbar + ld.p_off)[e] = mean;
      if (a.padded) {    // the sweeps' copy with rows of rank_pad ranks
        const unsigned row = (unsigned)e / (unsigned)ld.r;
        float* pad = phase ? a.Qop + ld.qop_off : a.Pop + ld.pop_off;
        pad[(size_t)row * a.rank_pad + ((unsigned)e - row * (unsigned)ld.r)] = mean;
      }
    }
  }
}

// ---------------------------------------------------------------------------
// sweep 1: Q_w partial = M_w^T P-bar over a row block (Algorithm 1,
// "Q <- G'^T P").  One workgroup per (row block, chunk of 256 columns, or of 64
// with one column per lane); its four wavefronts split the rows and their partial
// sums meet in LDS, where they are added in wavefront order (aligned rows whose
// rank fills its pad) or as (0 + 2) + (1 + 3).
// ---------------------------------------------------------------------------
// Columns a lane of sweep 1 holds.
template <int KIND>
constexpr int lane_cols() { return KIND == kNarrow ? 1 : 4; }
template <int RP, int KIND, bool WHOLE_GROUP>
__device__ __forceinline__ void back_project_rows(const float* __restrict__ M, const float* Pb, int cols,
                                                  int ra, int rb, int c, float (&acc)[lane_cols<KIND>() * RP]) {
  constexpr int U = LQSGD_B_U, V = lane_cols<KIND>();
  auto load = [&](int row) __attribute__((always_inline)) {
    const float* p = M + (size_t)row * cols;
    if constexpr (V == 1) return Pk<1>{{gptr<float>(p)[c]}};
    else return ldedge<KIND, LQSGD_NT_M != 0, false>(reinterpret_cast<const char*>(p), c, cols);
  };
  int i = ra;
  for (; i + U <= rb; i += U) {
    Pk<V> m[U];
#pragma unroll
    for (int u = 0; u < U; ++u) m[u] = load(i + u);
    if constexpr (KIND == kRagged) {
      if (c + 4 > cols) {
#pragma unroll
        for (int u = 0; u < U; ++u) edge_fix<1>(m[u].v, c, cols);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float p[RP];
      load_row_uniform<RP>(Pb, i + u, p);
#pragma unroll
      for (int v = 0; v < V; ++v)
#pragma unroll
        for (int k = 0; k < RP; ++k) acc[v * RP + k] = fmaf(m[u].v[v], p[k], acc[v * RP + k]);
    }
  }
  if constexpr (WHOLE_GROUP) {
    // The last, partial group in flight as a whole, from three rows on: those beyond it repeat its last one and are left out.  One at
    // a time, each a trip to memory, they were most of a small item (a step, us: 731 x 300 and 300 x 600, r = 7, W = 3 47.2 -> 45.4;
    // 401 x 400, 3 of them, r = 6, W = 9 54.3 -> 52.5; 1000^2, 8 of them, r = 8, W = 8 245 -> 240).  Lower rank pads lose a wavefront
    // a SIMD to its registers (3001 x 5000, r = 4, W = 4 410 -> 414) and gain nothing.
    if (rb - i > 2) {
      Pk<V> m[U];
#pragma unroll
      for (int u = 0; u < U; ++u) m[u] = load(min(i + u, rb - 1));
      if constexpr (KIND == kRagged) {
        if (c + 4 > cols) {
#pragma unroll
          for (int u = 0; u < U; ++u) edge_fix<1>(m[u].v, c, cols);
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (i + u < rb) {
          float p[RP];
          load_row_uniform<RP>(Pb, i + u, p);
#pragma unroll
          for (int v = 0; v < V; ++v)
#pragma unroll
            for (int k = 0; k < RP; ++k) acc[v * RP + k] = fmaf(m[u].v[v], p[k], acc[v * RP + k]);
        }
      i = rb;
    }
  }
  for (; i < rb; ++i) {
    Pk<V> m = load(i);
    if constexpr (KIND == kRagged)
      if (c + 4 > cols) edge_fix<1>(m.v, c, cols);
    float p[RP];
    load_row_uniform<RP>(Pb, i, p);
#pragma unroll
    for (int v = 0; v < V; ++v)
#pragma unroll
      for (int k = 0; k < RP; ++k) acc[v * RP + k] = fmaf(m.v[v], p[k], acc[v * RP + k]);
  }
}

template <int RP, int KIND>
__device__ __forceinline__ void back_project_tile(const DevArgs& a, const LayerDesc& ld, const Tile& tl, int layer, int worker,
                                                  float* comb, float* redmax, int wave, int lane) {
  constexpr int V = lane_cols<KIND>(), NV = V * RP;
  const int cols = ld.cols, r = ld.r;
  const float* M = a.E + (size_t)worker * a.m_stride + ld.m_off;
  const float* Pb = p_operand(a, ld);
  const int c0 = tl.aux * (kWave * V);
  const int c = c0 + lane * V;
  const bool active = c < cols;
  const int per = (tl.nrows + 3) >> 2;
  const int ra = min(tl.row0 + wave * per, tl.row0 + tl.nrows);
  const int rb = min(ra + per, tl.row0 + tl.nrows);
  float acc[NV];
#pragma unroll
  for (int i = 0; i < NV; ++i) acc[i] = 0.0f;
  if (active) {
    if (tl.nrows >= LQSGD_B_INTERLEAVE) {
      // Tall row blocks: the four wavefronts take groups of 8 rows in turn instead of a quarter of
      // the block each, so that they read rows close to each other at any time (four streams
      // hundreds of rows apart read the 8192^2 set at 6.0 TB/s, interleaved at 6.6 TB/s).
      const int rend = tl.row0 + tl.nrows;
      for (int g0 = tl.row0 + wave * LQSGD_B_U; g0 < rend; g0 += 4 * LQSGD_B_U)
        back_project_rows<RP, KIND, false>(M, Pb, cols, g0, min(g0 + LQSGD_B_U, rend), c, acc);
    } else {
      back_project_rows<RP, KIND, RP >= 8>(M, Pb, cols, ra, rb, c, acc);
    }
  }
  // A layer whose rows fit one row block: this item holds the whole sum, Q_w is stored directly
  // and its absmax raised here (the cell was zeroed by sweep 0); otherwise a partial plane per
  // row block, added up by reduce_q_kernel.
  const bool direct = ld.direct_q != 0;
  float* Qp = direct ? a.Qw + (size_t)worker * a.q_stride + ld.q_off
                     : a.Qpart + (size_t)worker * a.qpart_stride + ld.qpart_off + (size_t)(tl.row0 / ld.rbb) * ld.nq_pad;
  float mx = 0.0f;
  // comb[wave][column][rank]; afterwards the workgroup adds the four partials of every output
  // element: the chunk's slice of the factor is contiguous from column c0.
  {
    float* mine = comb + (size_t)wave * (kWave * NV) + lane * NV;
    if constexpr (NV % 4 == 0) {
#pragma unroll
      for (int i = 0; i < NV / 4; ++i)
        reinterpret_cast<float4*>(mine)[i] = make_float4(acc[4 * i], acc[4 * i + 1], acc[4 * i + 2], acc[4 * i + 3]);
    } else {
#pragma unroll
      for (int i = 0; i < NV; ++i) mine[i] = acc[i];
    }
  }
  __syncthreads();
  const int tid = wave * kWave + lane;
  const int ncol = min(kWave * V, cols - c0);
  if (KIND == kAligned && r == RP) {
    const int nout = ncol * RP;                  // floats this chunk owns: a multiple of four
#pragma unroll
    for (int j = 0; j < (NV + 15) / 16; ++j) {   // 64 * NV / 4 float4 outputs over 256 lanes
      const int o = (j * 256 + tid) * 4;
      if (o < nout) {
        float4 s = reinterpret_cast<const float4*>(comb + o)[0];
#pragma unroll
        for (int wv = 1; wv < 4; ++wv) {
          const float4 t = reinterpret_cast<const float4*>(comb + (size_t)wv * (kWave * NV) + o)[0];
          s.x += t.x; s.y += t.y; s.z += t.z; s.w += t.w;
        }
        reinterpret_cast<float4*>(Qp + (size_t)c0 * RP + o)[0] = s;
        mx = fmaxf(fmaxf(mx, fmaxf(fabsf(s.x), fabsf(s.y))), fmaxf(fabsf(s.z), fabsf(s.w)));
      }
    }
  } else {
    const int nout = ncol * r;
    for (int o = tid; o < nout; o += 256) {
      const int cc = (int)((unsigned)o / (unsigned)r);
      const float* src = comb + cc * RP + (o - cc * r);
      constexpr size_t P = (size_t)kWave * NV;
      const float s = (src[0] + src[2 * P]) + (src[P] + src[3 * P]);
      Qp[(size_t)c0 * r + o] = s;
      mx = fmaxf(mx, fabsf(s));
    }
  }
  if (direct) {     // workgroup-uniform
    mx = wave_max(mx);
    if (lane == 0) redmax[wave] = mx;
    __syncthreads();
    if (wave == 0 && lane == 0) {
      const float m = fmaxf(fmaxf(redmax[0], redmax[1]), fmaxf(redmax[2], redmax[3]));
      atomicMax(reinterpret_cast<unsigned int*>(a.scaleQ + (size_t)worker * a.L + layer), __float_as_uint(m));
    }
  }
}

// ---------------------------------------------------------------------------
// 1-D tensors: plain mean over the workers (Eq. (1)).  Runs as extra
// workgroups at the end of sweep 1's grid.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void vector_mean_tile(const DevArgs& a, const VTile& tl) {
  const VecDesc& vd = a.vecs[tl.vec];
  auto* extra = gptr<float>(a.ghat ? a.ghat[vd.gidx] : nullptr);
  const float wf = (float)a.W;
  for (int i = 0; i < 4; ++i) {
    const int e = tl.el0 + i * 256 + threadIdx.x;
    if (e < vd.len) {
      float s = 0.0f;
      if (a.g_bf16) {
        for (int w = 0; w < a.W; ++w) s += grad_elem<true>(a.grads[(size_t)w * a.n_all + vd.gidx], (size_t)e);
      } else {
        for (int w = 0; w < a.W; ++w) s += grad_elem<false>(a.grads[(size_t)w * a.n_all + vd.gidx], (size_t)e);
      }
      s /= wf;
      a.vmean[vd.off + e] = s;
      if (extra) extra[e] = a.update ? fmaf(-a.eta, s, extra[e]) : s;
    }
  }
}

template <int RP>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 8))) void back_project_kernel(DevArgs a, const Tile* __restrict__ tiles, int ntiles,
                                                           const VTile* __restrict__ vtiles, int reverse) {
  __shared__ __attribute__((aligned(16))) float comb[4 * kWave * 4 * RP];
  __shared__ float redmax[4];
  if ((int)blockIdx.x >= ntiles) {
    vector_mean_tile(a, vtiles[blockIdx.x - ntiles]);
    return;
  }
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & (kWave - 1);
  const Tile tl = tiles[reverse ? ntiles - 1 - blockIdx.x : blockIdx.x];
  const int layer = tl.lw / a.W, worker = tl.lw - layer * a.W;
  const LayerDesc& ld = a.layers[layer];
  if (ld.kind == kAligned)
    back_project_tile<RP, kAligned>(a, ld, tl, layer, worker, comb, redmax, wave, lane);
  else if (ld.bcw != kWave)
    back_project_tile<RP, kRagged>(a, ld, tl, layer, worker, comb, redmax, wave, lane);
  else
    back_project_tile<RP, kNarrow>(a, ld, tl, layer, worker, comb, redmax, wave, lane);
}

// ---------------------------------------------------------------------------
// sweep 1 on the matrix cores, for rank pad 32, where 4 x r accumulators per
// lane no longer fit the vector register file.
// v_mfma_f32_32x32x2_f32 computes D[32 x 32] += A[32 x 2] B[2 x 32] with
//   A: lane l holds A[i = l % 32][k = l / 32]
//   B: lane l holds B[k = l / 32][j = l % 32]
//   D: lane l, register v holds D[i = 8 (v / 4) + 4 (l / 32) + v % 4][j = l % 32]
// Here j = rank, k = two gradient rows per instruction, i = gradient column.
// Which column an index i stands for is free, as long as the result is read
// back the same way: lane (i, k) loads the float4 of columns 4 i .. 4 i + 3 of
// its row (so a half-wavefront reads 512 contiguous bytes of a row, a
// wavefront two rows, a workgroup 2 KiB of each row), and component s of that
// float4 feeds matrix instruction s, whose block D_s then belongs to columns
// 4 i + s.  No transposition and no LDS; a 32 x 32 block of Q_w accumulates in
// 16 registers.
// ---------------------------------------------------------------------------
typedef float v16f __attribute__((ext_vector_type(16)));

// NB blocks of 32 ranks (rank pad 64: NB = 2): one pass over M feeds both.
// NB = 2: the rows of P-bar come through LDS, kPRows at a time, once for the four wavefronts of the workgroup, with 16 rows in
// flight; enter(row) makes `row` and those behind it the ones that `ps` holds, together with the other wavefronts.  (From L2 they
// are two requests of 4 bytes a lane beside one of 16 for M, and take registers that 8 rows in flight were left with: ResNet-18
// set, r = 50, W = 8 168 -> 162 us, 8 x (512 x 4608), r = 64 238 -> 211, 16 x 1024^2 185 -> 173, 8192^2, W = 8 663 - 689 ->
// 633 - 644.)  NB = 1: straight from L2, one request beside one (through LDS 16 x 1024^2, W = 8 128 -> 136 us,
// ResNet-18 set 92 -> 90).
constexpr int kPRows = 256;
// few: rank pad 64, a list that waits for single items (see the end).
template <int NB, int KIND, bool SHORT, typename Enter>
__device__ __forceinline__ void back_project_mfma_tile(const DevArgs& a, const LayerDesc& ld, const Tile& tl, int worker,
                                                       int c0, int lane, bool few, const float* ps, float* stage, Enter&& enter) {
  constexpr int U = LQSGD_BM_U;                     // pairs of rows per step
  constexpr bool SHARE = NB == 2;
  static_assert(kPRows % (2 * U) == 0, "");
  const int cols = ld.cols, r = ld.r;
  const int li = lane & 31, h = lane >> 5;
  const int cl = c0 + 4 * li;                      // first of this lane's four columns
  const float* M = a.E + (size_t)worker * a.m_stride + ld.m_off;
  const int rend = tl.row0 + tl.nrows;
  v16f acc[NB][4];                                  // [block of 32 ranks][column residue]
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[nb][s][i] = 0.0f;
  const float* Pb = p_operand(a, ld) + li;         // this lane's rank of each block: rows of 32 NB, zero beyond r
  Pk<4> am[U], an[U];
  float bp[NB][U], bn[NB][U];
  auto fetch = [&](int rb, Pk<4>* m, float (*p)[U]) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int row = min(rb + 2 * u + h, rend - 1);        // (clamped in the last, partial group only)
      m[u] = ldedge<KIND, LQSGD_NT_M != 0, false>(reinterpret_cast<const char*>(M + (size_t)row * cols), cl, cols);
      if constexpr (!SHARE) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) p[nb][u] = Pb[(size_t)row * (32 * NB) + 32 * nb];
      }
    }
  };
  auto read_p = [&](int rb, float (*p)[U]) __attribute__((always_inline)) {
    if constexpr (SHARE) {
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) p[nb][u] = ps[(((rb - tl.row0) & (kPRows - 1)) + 2 * u + h) * (32 * NB) + 32 * nb + li];
    }
  };
  auto multiply = [&](Pk<4>* m, float (*p)[U]) __attribute__((always_inline)) {
    if constexpr (KIND != kAligned) {
#pragma unroll
      for (int u = 0; u < U; ++u) edge_fix<1>(m[u].v, cl, cols);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int s = 0; s < 4; ++s)
          acc[nb][s] = __builtin_amdgcn_mfma_f32_32x32x2f32(m[u].v[s], p[nb][u], acc[nb][s], 0, 0, 0);
  };
  // a row that does not exist counts as zeros on both sides (0 x Inf would not be zero)
  auto last_group = [&](int rb, Pk<4>* m, float (*p)[U]) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool ok = rb + 2 * u + h < rend;
#pragma unroll
      for (int s = 0; s < 4; ++s) m[u].v[s] = keep_if(m[u].v[s], ok);
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) p[nb][u] = keep_if(p[nb][u], ok);
    }
    multiply(m, p);
  };
  // Short items of NB = 2: every prefetch is of rows that are still to come, and the last group, whole or partial, is left to the code
  // behind the loop (64 layers of 32 x 2048, r = 50, W = 8, two groups an item 88 -> 82 us, 32 layers of 65 rows 85 -> 82; with
  // 8 rows in flight and P-bar from L2 80 and 79).
  if constexpr (SHORT) {
    int rb = tl.row0;
    fetch(rb, am, bp);
    enter(rb);
    for (; rb + 2 * U < rend; rb += 2 * U) {
      fetch(rb + 2 * U, an, bn);
      __builtin_amdgcn_sched_barrier(0);           // (see below)
      read_p(rb, bp);
      multiply(am, bp);
#pragma unroll
      for (int u = 0; u < U; ++u) am[u] = an[u];
    }
    read_p(rb, bp);
    last_group(rb, am, bp);
  } else {
  // Whole groups of 2 U rows with the next group's loads issued before this group's matrix instructions, so that a
  // wavefront overlaps its own loads with its own arithmetic (the last prefetch re-reads the last group: every load
  // stays unconditional and in bounds), then the rows that are left.
  int rb = tl.row0;
  if (rend - rb >= 2 * U) {
    const int last = rb + (tl.nrows / (2 * U) - 1) * (2 * U);   // first row of the last whole group
    fetch(rb, am, bp);
    if constexpr (SHARE) enter(rb);
    for (; rb <= last; rb += 2 * U) {
      if constexpr (SHARE)
        if (rb > tl.row0 && (rb - tl.row0) % kPRows == 0) enter(rb);
      fetch(min(rb + 2 * U, last), an, bn);
      // the requests above stay ahead of the arithmetic below (left to itself the compiler moves the
      // P-bar loads down to their first use, and every group of matrix instructions then waits for
      // its operand and, requests completing in order, for the whole prefetch in front of it)
      __builtin_amdgcn_sched_barrier(0);
      read_p(rb, bp);
      multiply(am, bp);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        am[u] = an[u];
        if constexpr (!SHARE) {
#pragma unroll
          for (int nb = 0; nb < NB; ++nb) bp[nb][u] = bn[nb][u];
        }
      }
    }
  }
  if (rb < rend) {
    fetch(rb, am, bp);
    if constexpr (SHARE)
      if ((rb - tl.row0) % kPRows == 0) enter(rb);
    read_p(rb, bp);
    last_group(rb, am, bp);
  }
  }
  // Where the sums leave: straight from the registers, 4 bytes a lane, or through LDS, 64 columns at a time, whose rows of r ranks are
  // one run of memory there as in Q_w or its partial plane, so that a store is 1 KiB and there are no tests but at its end.  With an
  // address and a test of its own for each of the 64 NB values the register form was a fifth of an item of 256 rows, and most of the
  // code, which a short item runs once.  Whole strips of long items at rank pad 64 do without both (a wave-uniform row of Q_w plus
  // one byte offset a lane; sweep 1, us, ResNet-18 set, W = 8, r = 50 156 -> 130, 12 x (512 x 4608) 313 -> 292, 8192^2, W = 4, r = 64
  // 323 -> 308; through LDS, behind a barrier of the workgroup, 149, 297 and 310).  The others go through LDS, at rank pad 64 in lists of up
  // to two items a CU, which wait for single items (a step, us, r = 50, W = 8 registers / LDS: 20 x (100 x 300) 130.5 / 129.3, 64 x 512, 30 of
  // them 113.2 / 111.7; but the ResNet-18 set, 1800 items, 476 / 488, for the barrier).
  // Where a layer has one row block these are the sums themselves, and their absmax is taken here if a quantiser reads it, a pass over a copy less (a step:
  // ResNet-18 set, W = 8, r = 50 482 -> 476, r = 32 350 -> 347, 8 x (256 x 4096), r = 50 366 -> 349, 2 x (60 x 300), r = 20 48.3 -> 44.7).
  const bool through_lds = NB == 1 || few;
  if (SHARE && through_lds) __syncthreads();     // (the rows of P-bar make room)
  const bool direct = ld.direct_q != 0;
  float* Qp = direct ? a.Qw + (size_t)worker * a.q_stride + ld.q_off
                     : a.Qpart + (size_t)worker * a.qpart_stride + ld.qpart_off + (size_t)(tl.row0 / ld.rbb) * ld.nq_pad;
  float mx = 0.0f;
  const bool raise = direct && a.bits_q > 0;
  auto absmax = [&]() __attribute__((always_inline)) {           // (values beyond the columns or ranks are zeros)
    if (raise) {
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
          for (int v = 0; v < 16; ++v) mx = fmaxf(mx, fabsf(acc[nb][s][v]));
    }
  };
  if constexpr (NB == 2 && !SHORT && KIND == kAligned) {
    unsigned lane_off = (unsigned)(16 * h * r + li) * 4u;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
      if (32 * nb + li < r) {
#pragma unroll
        for (int v = 0; v < 16; ++v)
#pragma unroll
          for (int s = 0; s < 4; ++s) {
            const int col = c0 + 32 * (v >> 2) + 4 * (v & 3) + s;
            char* at = reinterpret_cast<char*>(Qp + (unsigned)(col * r + 32 * nb));
            asm volatile("" : "+v"(lane_off));   // (else the optimiser adds it to Qp first, and has 64-bit sums to do again)
            *gptr<float>(at + lane_off) = acc[nb][s][v];
          }
      }
    absmax();
  } else if (!through_lds) {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int col = c0 + 4 * (8 * (v >> 2) + 4 * h + (v & 3)) + s;
          if (col < cols && 32 * nb + li < r) Qp[(size_t)col * r + 32 * nb + li] = acc[nb][s][v];
        }
    absmax();
  } else {
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      const int c = c0 + 64 * half;
      if (c < cols) {
        wave_lds_fence();
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
          if (32 * nb + li < r) {
            float* to = stage + 16 * h * r + 32 * nb + li;
#pragma unroll
            for (int v = 8 * half; v < 8 * half + 8; ++v)
#pragma unroll
              for (int s = 0; s < 4; ++s) to[(32 * ((v >> 2) & 1) + 4 * (v & 3) + s) * r] = acc[nb][s][v];
          }
        wave_lds_fence();
        const int n = min(64, cols - c) * r;
        float* dst = Qp + (size_t)c * r;
#pragma unroll 4
        for (int e = 4 * lane; e < n; e += 4 * kWave) {
          const float4 t = *reinterpret_cast<const float4*>(stage + e);
          if (e + 4 <= n) {
            *reinterpret_cast<float4*>(dst + e) = t;
            mx = fmaxf(mx, fmaxf(fmaxf(fabsf(t.x), fabsf(t.y)), fmaxf(fabsf(t.z), fabsf(t.w))));
          } else {
            const float x[4] = {t.x, t.y, t.z, t.w};
#pragma unroll
            for (int q = 0; q < 3; ++q)
              if (e + q < n) {
                dst[e + q] = x[q];
                mx = fmaxf(mx, fabsf(x[q]));
              }
          }
        }
      }
    }
  }
  if (raise) {
    mx = wave_max(mx);
    if (lane == 0) atomicMax(reinterpret_cast<unsigned int*>(a.scaleQ + (size_t)worker * a.L + tl.lw / a.W), __float_as_uint(mx));
  }
}

template <int NB>
__global__ __launch_bounds__(256, 2) void back_project_mfma_kernel(DevArgs a, const Tile* __restrict__ tiles, int ntiles,
                                                                const VTile* __restrict__ vtiles, int reverse) {
  if ((int)blockIdx.x >= ntiles) {
    vector_mean_tile(a, vtiles[blockIdx.x - ntiles]);
    return;
  }
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & (kWave - 1);
  const Tile tl = tiles[reverse ? ntiles - 1 - blockIdx.x : blockIdx.x];
  const int layer = tl.lw / a.W, worker = tl.lw - layer * a.W;
  const LayerDesc& ld = a.layers[layer];
  const int c0 = tl.aux * kMfmaCols + wave * 128;
  const bool few = ntiles <= 2 * kCus;
  // rows of P-bar (NB = 2), at the end 64 columns' sums of each wavefront
  constexpr int STAGE = 64 * 32 * NB;
  static_assert(kPRows * 32 * NB >= 4 * STAGE, "");
  __shared__ __attribute__((aligned(16))) float ps[NB == 2 ? kPRows * 32 * NB : 4 * STAGE];
  float* stage = ps + wave * STAGE;
  // strips of which all 128 columns exist need no care at their end, whatever the alignment of the rows
  auto run = [&](auto short_tag, const float* ps, auto&& enter) __attribute__((always_inline)) {
    constexpr bool SHORT = decltype(short_tag)::value;
    if (c0 + 128 <= ld.cols) back_project_mfma_tile<NB, kAligned, SHORT>(a, ld, tl, worker, c0, lane, few, ps, stage, enter);
    else if (ld.cols >= 4) back_project_mfma_tile<NB, kRagged, SHORT>(a, ld, tl, worker, c0, lane, few, ps, stage, enter);
    else back_project_mfma_tile<NB, kNarrow, SHORT>(a, ld, tl, worker, c0, lane, few, ps, stage, enter);
  };
  if constexpr (NB == 2) {
    const int tid = threadIdx.x, rend = tl.row0 + tl.nrows;
    // rows of P-bar are contiguous: a linear copy, 16 bytes a thread and request
    auto enter = [&](int row) __attribute__((always_inline)) {
      const float* src = p_operand(a, ld) + (size_t)row * (32 * NB);
      const int n4 = min(kPRows, rend - row) * (8 * NB);
      if (row > tl.row0) __syncthreads();
      auto copy = [&](auto n_tag, const int i0) __attribute__((always_inline)) {
        constexpr int N = decltype(n_tag)::value;
        Pk<4> x[N];
#pragma unroll
        for (int i = 0; i < N; ++i) x[i] = ldrow<false>(reinterpret_cast<const char*>(src), (unsigned)min(tid + 256 * (i0 + i), n4 - 1) * 16u);
#pragma unroll
        for (int i = 0; i < N; ++i)
          if (tid + 256 * (i0 + i) < n4)
            reinterpret_cast<float4*>(ps)[tid + 256 * (i0 + i)] = make_float4(x[i].v[0], x[i].v[1], x[i].v[2], x[i].v[3]);
      };
      // no more requests than the rows take: an item of 32 rows is over after few others
      if (n4 <= 512) {
        copy(std::integral_constant<int, 2>{}, 0);
      } else {
        copy(std::integral_constant<int, 8>{}, 0);
        if (n4 > 2048) copy(std::integral_constant<int, 8>{}, 8);
      }
      __syncthreads();
    };
    if (c0 < ld.cols && tl.nrows < 128) run(std::true_type{}, ps, enter);
    else if (c0 < ld.cols) run(std::false_type{}, ps, enter);
    else {                                       // no columns: only its share of the copies
      for (int row = tl.row0; row < rend; row += kPRows) enter(row);
      if (few) __syncthreads();                  // (the others' before they hand out their sums)
    }
  } else {
    if (c0 < ld.cols) run(std::false_type{}, nullptr, [](int) {});
  }
}

// ---------------------------------------------------------------------------
// reduce_q: Q_w = sum over row blocks of the partials (fixed order), and
// absmax(Q_w) -> scaleQ.  The max over workgroups goes through an integer
// atomic max on the float's bit pattern (non-negative floats order like
// unsigned integers), which is exact and order-independent.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void reduce_q_kernel(DevArgs a, const RTile* __restrict__ tiles, int phase) {
  __shared__ float redmax[4];
  const RTile tl = tiles[blockIdx.x];
  const int layer = tl.lw / a.W, worker = tl.lw - layer * a.W;
  const LayerDesc& ld = a.layers[layer];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
  float mx = 0.0f;
  // phase 1: Q_w from the row-block planes; phase 0 (aggregate-first order only): the raw P_w from
  // the column-segment planes, which is then what the P exchange quantises
  const int n_el = phase ? ld.nq_el : ld.np_el;
  const float* planes = phase ? a.Qpart + (size_t)worker * a.qpart_stride + ld.qpart_off
                              : a.Ppart + (size_t)worker * a.ppart_stride + ld.ppart_off;
  float* out = phase ? a.Qw + (size_t)worker * a.q_stride + ld.q_off : a.Ppre + (size_t)worker * a.p_stride + ld.p_off;
  const int nplanes = phase ? ld.nrb : ld.nseg;
  const size_t pitch = phase ? ld.nq_pad : ld.np_pad;
  for (int off = tid * 4; off < tl.n; off += 1024) {
    const int e = tl.el0 + off;                    // < n_el, and so are the elements of its float4 that are kept
    const float* Qp = planes + e;
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    // planes are added in order; eight loads are in flight at a time
    int rb = 0;
    for (; rb + 8 <= nplanes; rb += 8) {
      float4 t[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) t[i] = *reinterpret_cast<const float4*>(Qp + (size_t)(rb + i) * pitch);
#pragma unroll
      for (int i = 0; i < 8; ++i) { s.x += t[i].x; s.y += t[i].y; s.z += t[i].z; s.w += t[i].w; }
    }
    for (; rb < nplanes; ++rb) {
      const float4 t = *reinterpret_cast<const float4*>(Qp + (size_t)rb * pitch);
      s.x += t.x; s.y += t.y; s.z += t.z; s.w += t.w;
    }
    float* dst = out + e;
    const int nv = min(4, n_el - e);
    if (nv == 4) {
      *reinterpret_cast<float4*>(dst) = s;
      mx = fmaxf(mx, fmaxf(fmaxf(fabsf(s.x), fabsf(s.y)), fmaxf(fabsf(s.z), fabsf(s.w))));
    } else {
      const float vals[4] = {s.x, s.y, s.z, s.w};
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (i < nv) {
          dst[i] = vals[i];
          mx = fmaxf(mx, fabsf(vals[i]));
        }
    }
  }
  mx = wave_max(mx);
  if (lane == 0) redmax[wave] = mx;
  __syncthreads();
  if (tid == 0) {
    const float m = fmaxf(fmaxf(redmax[0], redmax[1]), fmaxf(redmax[2], redmax[3]));
    atomicMax(reinterpret_cast<unsigned int*>((phase ? a.scaleQ : a.scaleP) + (size_t)worker * a.L + layer),
              __float_as_uint(m));
  }
}

// ---------------------------------------------------------------------------
// sweep 2: E_w = M_w - P-bar Q-bar^T (Eq. (7), (8)) and / or G-hat = P-bar Q-bar^T.
//   kResidual      E for every worker                          (8 B / element)
//   kResidualGhat  E for every worker, G-hat from worker 0's items
//   kGhatOnly      G-hat only, one item list per layer (4 B / element / W);
//                  used when the residual update is deferred into the next
//                  iteration's sweep 0
// The four wavefronts of a workgroup split the rows of the item.
// ---------------------------------------------------------------------------
enum ResidualMode { kResidual = 0, kResidualGhat = 1, kGhatOnly = 2 };

template <int RP, int MODE, int KIND>
__device__ __forceinline__ void residual_rows(float* __restrict__ M, const float* Pb, float* __restrict__ ghat,
                                              int cols, int ra, int rb, int c,
                                              const float (&q)[4 * RP], int update, float eta) {
  constexpr int U = 8;
  // what this pass reads besides the factors: M, or the parameters it updates
  const bool reads = MODE != kGhatOnly || update;
  const float* in = MODE != kGhatOnly ? M : ghat;
  const unsigned boff = (unsigned)c * 4u;
  const int n = KIND == kAligned ? 4 : cols - c;
  for (int i = ra; i < rb; i += U) {
    const int nu = min(U, rb - i);
    Pk<4> m[U];
    if (reads) {      // fetched for all U rows before the arithmetic starts (rows beyond nu repeat the last one)
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const char* p = reinterpret_cast<const char*>(in + (size_t)(i + min(u, nu - 1)) * cols);
        m[u] = ldedge<KIND, LQSGD_NT_M != 0, false>(p, c, cols);
      }
      __builtin_amdgcn_sched_barrier(0);
      if (n < 4) {
#pragma unroll
        for (int u = 0; u < U; ++u) edge_fix<1>(m[u].v, c, cols);
      }
    }
    Pk<4> wp[MODE == kResidualGhat ? U : 1];
    if (MODE == kResidualGhat && ghat && update) {
#pragma unroll
      for (int u = 0; u < U; ++u) wp[MODE == kResidualGhat ? u : 0] = load_params<KIND>(ghat + (size_t)(i + min(u, nu - 1)) * cols, c, cols);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (u < nu) {
        float p[RP];
        load_row_uniform<RP>(Pb, i + u, p);
        Pk<4> gh, e;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          float s = 0.0f;
#pragma unroll
          for (int k = 0; k < RP; ++k) s = fmaf(p[k], q[v * RP + k], s);
          gh.v[v] = s;
          if constexpr (MODE != kGhatOnly) e.v[v] = m[u].v[v] - s;
        }
        if constexpr (MODE != kGhatOnly)
          stgroup<false>(reinterpret_cast<char*>(M + (size_t)(i + u) * cols), boff, n, e);
        if constexpr (MODE == kGhatOnly) {
          if (update) {
#pragma unroll
            for (int v = 0; v < 4; ++v) gh.v[v] = fmaf(-eta, gh.v[v], m[u].v[v]);
          }
          stgroup<true>(reinterpret_cast<char*>(ghat + (size_t)(i + u) * cols), boff, n, gh);
        } else if (MODE == kResidualGhat && ghat) {
          emit_ghat<KIND>(ghat + (size_t)(i + u) * cols, c, cols, gh, update, eta, wp[MODE == kResidualGhat ? u : 0]);
        }
      }
    }
  }
}

template <int RP, int MODE, int KIND>
__device__ __forceinline__ void residual_tile(const DevArgs& a, const LayerDesc& ld, const Tile& tl, int worker,
                                              float* __restrict__ ghat, int wave, int lane) {
  const int cols = ld.cols;
  float* M = a.E + (size_t)worker * a.m_stride + ld.m_off;
  const float* Pb = p_operand(a, ld);
  const int c = tl.aux * (kWave * 4) + lane * 4;
  const int per = (tl.nrows + 3) >> 2;
  const int ra = min(tl.row0 + wave * per, tl.row0 + tl.nrows);
  const int rb = min(ra + per, tl.row0 + tl.nrows);
  if constexpr (KIND == kNarrow) {
    narrow_item<RP, false, false, MODE != kGhatOnly, MODE != kResidual, false>(nullptr, M, q_operand(a, ld), Pb, nullptr, ghat, cols,
                                                                               ld.r, ra, rb, lane, a.update, a.eta);
    return;
  }
  if (c >= cols) return;
  float q[4 * RP];
  load_slice<RP>(q_operand(a, ld), KIND == kAligned ? c : edge_col(c, cols), q);
  if (KIND != kAligned && c + 4 > cols) edge_fix<RP>(q, c, cols);
  residual_rows<RP, MODE, KIND>(M, Pb, ghat, cols, ra, rb, c, q, a.update, a.eta);
}

template <int RP, int MODE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 8))) void residual_kernel(DevArgs a, const Tile* __restrict__ tiles, int ntiles, int reverse) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & (kWave - 1);
  const Tile tl = tiles[reverse ? ntiles - 1 - blockIdx.x : blockIdx.x];
  const int layer = tl.lw / a.W, worker = tl.lw - layer * a.W;
  const LayerDesc& ld = a.layers[layer];
  float* ghat = nullptr;
  if (MODE != kResidual && worker == 0 && a.ghat) ghat = a.ghat[ld.gidx];
  if (MODE == kGhatOnly && !ghat) return;
  if (ld.kind == kAligned)
    residual_tile<RP, MODE, kAligned>(a, ld, tl, worker, ghat, wave, lane);
  else if (ld.kind != kOneColumnPerLane)
    residual_tile<RP, MODE, kRagged>(a, ld, tl, worker, ghat, wave, lane);
  else
    residual_tile<RP, MODE, kNarrow>(a, ld, tl, worker, ghat, wave, lane);
}

// ---------------------------------------------------------------------------
// Sweeps on the matrix cores by 64-column blocks per wavefront: the residual and G-hat
// passes at rank pads 16 to 64, sweep 0 of few items at 64 and of half-empty rounds at 16
// (DevArgs::by_blocks); the other sweeps 0 further below.
// One workgroup per 32 rows x one column segment; its four
// wavefronts take the 64-column blocks of the segment in turn, so that the
// workgroup touches 1 KiB of every row at about the same time (with one item
// per wavefront, each walking its own segment in 256-byte runs, the same data
// movement reached only 4.3 TB/s; this order reaches 5.4-5.8), and their P
// partials meet in LDS, added in wavefront order.  A 32 x 64 tile is loaded and
// stored in "row layout" (float4 per lane, 16 lanes = 256 contiguous bytes of a
// row, 4 rows per instruction).
//
//   G-hat tile = P-bar[32 x r] Q-bar^T[r x 64]: i = row, j = column, k = rank.
//     Lane (i, h) holds P-bar[row i][h r/2 .. h r/2 + r/2) -- a contiguous run of
//     its factor row, so the wavefront reads one contiguous block of P-bar;
//     lane (h, j) holds Q-bar[col j][the same ranks].  Which rank a step k
//     stands for is free as long as both operands agree.
//   P tile += M[32 x 64] Q[64 x r]: i = row, j = rank, k = column.  Lanes index
//     rows here while memory runs along columns, so M goes through a
//     wave-private LDS tile ([row][column], pitch 68 floats): written in row
//     layout, read back as lane (i, h) -> columns 32 h .. 32 h + 31 of row i.
//   The G-hat block comes out of the matrix cores in their D layout (lanes =
//   columns); it takes the same LDS tile the other way to meet G and M in row
//   layout for  M_new = G + (M_old - G-hat).
// Modes: kMAdd (first iteration: M = G + E), kMAddFused (deferred residual),
// kMResidual / kMResidualGhat (the residual sweep; G-hat uses the very same
// instruction sequence as in kMAddFused and in mfma_ghat_kernel, which kMGhatOnly
// launches, so deferring the residual does not change a bit of the result).
// ---------------------------------------------------------------------------
enum MfmaMode { kMAdd = 0, kMAddFused = 1, kMResidual = 2, kMResidualGhat = 3, kMGhatOnly = 4 };
constexpr int kLP = 68;   // LDS pitch (floats): 16-byte aligned rows, 4-bank skew per row


template <int RP, int MODE, bool GB16, bool NTS>
__device__ __forceinline__ void mfma_tile(const float* __restrict__ G, float* __restrict__ M,
                                          const float* Q, const float* Pb, float* __restrict__ Pp,
                                          float* __restrict__ ghat_out, int cols, int r, int row0, int nrows,
                                          int col0, int col1, int lane, int wave, float (*lds_all)[32 * kLP],
                                          int update, float eta) {
  float* lds = lds_all[wave];
  constexpr bool ADD = (MODE == kMAdd || MODE == kMAddFused);
  constexpr bool NEEDG = (MODE != kMAdd);
  constexpr int KH = RP / 2;                       // ranks per half-wavefront
  constexpr int NB = (RP + 31) / 32;               // blocks of 32 ranks in the P product (2 at rank pad 64)
  // (the rows of Q and Pb hold RP ranks; r is only the row length of the P partials this item writes)
  const int li = lane & 31, h = lane >> 5;
  const int sr = lane >> 4, c4 = (lane & 15) * 4;  // row layout: rows 4 i + sr, columns c4 .. c4 + 3
  float pa[KH];
  if constexpr (NEEDG) {
    const int row = row0 + li;
    if (li < nrows) {
      const float4* src = reinterpret_cast<const float4*>(Pb + (size_t)row * RP + KH * h);
#pragma unroll
      for (int t = 0; t < KH / 4; ++t) {
        const float4 x = src[t];
        pa[4 * t] = x.x; pa[4 * t + 1] = x.y; pa[4 * t + 2] = x.z; pa[4 * t + 3] = x.w;
      }
    } else {
#pragma unroll
      for (int k = 0; k < KH; ++k) pa[k] = 0.0f;
    }
  }
  v16f accP[NB], accP2[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int i = 0; i < 16; ++i) { accP[nb][i] = 0.0f; accP2[nb][i] = 0.0f; }

  // the four wavefronts take the 64-column blocks of the segment in turn, so that together they
  // touch 1 KiB of each row at about the same time (a wavefront on its own reads 256-byte runs)
  // One 64-column block.  FULL: all 32 rows and all 64 columns of the block exist (every block of a
  // large layer except on its edges): no bounds tests, so nothing branches around a load.
  auto block = [&](auto full_tag, const int c) {
    constexpr bool FULL = decltype(full_tag)::value;
    constexpr int KIND = kRagged;                // of edge blocks (takes aligned rows too)
    const int cl = c + c4;
    // Edge blocks: this lane's row number is hidden from the optimiser, which otherwise computes the addresses of all
    // rows once, ahead of the loop over the blocks, and keeps them in registers that the whole blocks need (rank pad
    // 16, deferred residual: 92 values spilled; 8192^2, W = 8, when that set took this form, sweep 0 1098 -> 1220 us).
    int sr_ = sr;
    if constexpr (!FULL) asm volatile("" : "+v"(sr_));
    const int ncol = FULL ? 4 : cols - cl;       // columns of this lane's group that exist
    Pk<4> g[8], e[8];
    // FULL blocks address memory as a wave-uniform base (scalar registers) plus one byte offset per
    // lane that is the same for every row group and block: lo = this lane's place in 4 rows.
    const unsigned lo = (unsigned)(sr * cols + c4) * 4u;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int rr = 4 * i + sr_;
      // (edge blocks: rows beyond nrows repeat the last one, and are never stored)
      const size_t off = FULL ? (size_t)(row0 + 4 * i) * cols + c : (size_t)(row0 + min(rr, nrows - 1)) * cols;
      if constexpr (FULL) {
        if constexpr (ADD) g[i] = ldgrad<LQSGD_NT_G != 0, GB16>(grad_row<GB16>(G, off), lo);
        e[i] = ldrow<(ADD ? NTS : LQSGD_NT_E != 0)>(reinterpret_cast<const char*>(M + off), lo);
      } else {
        if constexpr (ADD) g[i] = ldedge<KIND, LQSGD_NT_G != 0, GB16>(grad_row<GB16>(G, off), cl, cols);
        e[i] = ldedge<KIND, (ADD ? NTS : LQSGD_NT_E != 0), false>(reinterpret_cast<const char*>(M + off), cl, cols);
      }
    }
    if constexpr (!FULL) {
      if (ncol < 4) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          if constexpr (ADD) edge_fix<1>(g[i].v, cl, cols);
          edge_fix<1>(e[i].v, cl, cols);
        }
      }
    }
    Pk<4> wp[8];                                 // the parameters to update
    if constexpr (MODE == kMResidualGhat) {
      if (update && ghat_out) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          if constexpr (FULL) wp[i] = load_params<kAligned>(ghat_out + (size_t)(row0 + 4 * i) * cols + c, (int)(lo >> 2), 0);
          else wp[i] = load_params<KIND>(ghat_out + (size_t)(row0 + min(4 * i + sr_, nrows - 1)) * cols, cl, cols);
        }
      }
    }
    float bq[NB][32];
    auto load_bq = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int kk = 0; kk < 32; ++kk) {
          const int col = c + 32 * h + kk;
          const int rk = 32 * nb + li;
          if constexpr (FULL)
            bq[nb][kk] = *gptr<float>(reinterpret_cast<const char*>(Q + (size_t)c * RP) + (kk * RP + 32 * nb) * 4 +
                                      (unsigned)(32 * h * RP + li) * 4u);
          else
            bq[nb][kk] = (col < col1 && rk < RP) ? Q[(size_t)col * RP + rk] : 0.0f;
        }
    };
    // In the fused mode the Q slice of the P product is fetched only after the G-hat part, when
    // the registers of its operands are free again (fetched up front it does not fit the register file).
    constexpr bool BQ_LATE = ADD && NEEDG && LQSGD_BQ_LATE;
    if constexpr (ADD && !BQ_LATE) load_bq();
    if constexpr (NEEDG) {
      float qb[2][KH];
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const int col = c + 32 * b + li;
        if constexpr (FULL) {
          const char* base = reinterpret_cast<const char*>(Q + (size_t)(c + 32 * b) * RP);
#pragma unroll
          for (int t = 0; t < KH / 4; ++t) {
            const Pk<4> x = ldrow<false>(base + 16 * t, (unsigned)(li * RP + KH * h) * 4u);
            qb[b][4 * t] = x.v[0]; qb[b][4 * t + 1] = x.v[1]; qb[b][4 * t + 2] = x.v[2]; qb[b][4 * t + 3] = x.v[3];
          }
        } else if (col < col1) {
          const float4* src = reinterpret_cast<const float4*>(Q + (size_t)col * RP + KH * h);
#pragma unroll
          for (int t = 0; t < KH / 4; ++t) {
            const float4 x = src[t];
            qb[b][4 * t] = x.x; qb[b][4 * t + 1] = x.y; qb[b][4 * t + 2] = x.z; qb[b][4 * t + 3] = x.w;
          }
        } else {
#pragma unroll
          for (int k = 0; k < KH; ++k) qb[b][k] = 0.0f;
        }
      }
      // the two 32-column blocks accumulate in turn: two independent chains on the matrix pipe
      v16f gh0, gh1;
#pragma unroll
      for (int i = 0; i < 16; ++i) { gh0[i] = 0.0f; gh1[i] = 0.0f; }
#pragma unroll
      for (int k = 0; k < KH; ++k) {
        gh0 = __builtin_amdgcn_mfma_f32_32x32x2f32(pa[k], qb[0][k], gh0, 0, 0, 0);
        gh1 = __builtin_amdgcn_mfma_f32_32x32x2f32(pa[k], qb[1][k], gh1, 0, 0, 0);
      }
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        lds[(8 * (v >> 2) + 4 * h + (v & 3)) * kLP + li] = gh0[v];
        lds[(8 * (v >> 2) + 4 * h + (v & 3)) * kLP + 32 + li] = gh1[v];
      }
      wave_lds_fence();
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int rr = 4 * i + sr_;
        const float4 t = *reinterpret_cast<const float4*>(lds + rr * kLP + c4);
        e[i].v[0] -= t.x; e[i].v[1] -= t.y; e[i].v[2] -= t.z; e[i].v[3] -= t.w;
        if (MODE == kMResidualGhat && ghat_out) {
          if constexpr (FULL) {
            const Pk<4> o{{t.x, t.y, t.z, t.w}};
            emit_ghat<kAligned>(ghat_out + (size_t)(row0 + 4 * i) * cols + c, (int)(lo >> 2), 0, o, update, eta, wp[i]);
          } else if (rr < nrows) {
            const Pk<4> o{{t.x, t.y, t.z, t.w}};
            if (ncol > 0) emit_ghat<KIND>(ghat_out + (size_t)(row0 + rr) * cols, cl, cols, o, update, eta, wp[i]);
          }
        }
      }
      wave_lds_fence();
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int rr = 4 * i + sr_;
      Pk<4> m;
#pragma unroll
      for (int v = 0; v < 4; ++v) m.v[v] = ADD ? g[i].v[v] + e[i].v[v] : e[i].v[v];
      if constexpr (FULL)
        strow<NTS>(reinterpret_cast<char*>(M + (size_t)(row0 + 4 * i) * cols + c), lo, m);
      else if (rr < nrows)
        stgroup<NTS>(reinterpret_cast<char*>(M + (size_t)(row0 + rr) * cols), (unsigned)cl * 4u, ncol, m);

      if constexpr (ADD)
        *reinterpret_cast<float4*>(lds + rr * kLP + c4) = make_float4(m.v[0], m.v[1], m.v[2], m.v[3]);
    }
    if constexpr (BQ_LATE) {
      __builtin_amdgcn_sched_barrier(0);
      load_bq();
    }
    if constexpr (ADD) {
      wave_lds_fence();
      // two accumulators (even / odd float4 of the lane's run of columns): two independent chains
#pragma unroll
      for (int t = 0; t < 8; t += 2) {
        const float4 a0 = *reinterpret_cast<const float4*>(lds + li * kLP + 32 * h + 4 * t);
        const float4 a1 = *reinterpret_cast<const float4*>(lds + li * kLP + 32 * h + 4 * t + 4);
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
          accP[nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0.x, bq[nb][4 * t + 0], accP[nb], 0, 0, 0);
          accP2[nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1.x, bq[nb][4 * t + 4], accP2[nb], 0, 0, 0);
          accP[nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0.y, bq[nb][4 * t + 1], accP[nb], 0, 0, 0);
          accP2[nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1.y, bq[nb][4 * t + 5], accP2[nb], 0, 0, 0);
          accP[nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0.z, bq[nb][4 * t + 2], accP[nb], 0, 0, 0);
          accP2[nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1.z, bq[nb][4 * t + 6], accP2[nb], 0, 0, 0);
          accP[nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0.w, bq[nb][4 * t + 3], accP[nb], 0, 0, 0);
          accP2[nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1.w, bq[nb][4 * t + 7], accP2[nb], 0, 0, 0);
        }
      }
      wave_lds_fence();
    }
  };
  const bool small_offsets = cols < (1 << 26);   // byte offsets within 4 rows fit 32 bits
  for (int c = col0 + 64 * wave; c < col1; c += 256) {
    if (nrows == 32 && c + 64 <= col1 && small_offsets)
      block(std::true_type{}, c);
    else
      block(std::false_type{}, c);
  }
  if constexpr (ADD) {
    // P partial of the item = sum over the four wavefronts, added in wavefront order
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int v = 0; v < 16; ++v)
        lds[(8 * (v >> 2) + 4 * h + (v & 3)) * kLP + 32 * nb + li] = accP[nb][v] + accP2[nb][v];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4 * NB; ++i) {
      const int e = (int)threadIdx.x + 256 * i;
      const int rr = e / (32 * NB), k = e % (32 * NB);
      const float t = ((lds_all[0][rr * kLP + k] + lds_all[1][rr * kLP + k]) + lds_all[2][rr * kLP + k]) +
                      lds_all[3][rr * kLP + k];
      if (rr < nrows && k < r) Pp[(size_t)(row0 + rr) * r + k] = t;
    }
  }
}

constexpr int kLP32 = 36;   // LDS pitch (floats) of a 32 x 32 block: 16-byte aligned rows

// ---------------------------------------------------------------------------
// The add modes at rank pad 64 with the factor operand shared through LDS.
//
// The 32 x 64 form above fetches 16 KB of Q per wavefront and block from L2 -- once as the G-hat operand, 16 bytes
// of 64 different rows per instruction, once as the P operand, 4 bytes a lane: 80 memory instructions beside the 24 of
// the streams -- and has registers for one wavefront per SIMD: that is what bounded it, not the matrix rate.  Here a
// workgroup of eight wavefronts takes 64 rows: wavefront w works on the 32 rows w / 4 and on the 64 columns w % 4 of a
// round of 256, so that every row of Q in a round serves two wavefronts and comes once, coalesced, through LDS.
// Both matrix operands are read from there: 16-byte chunk x of row c lies at x ^ (c % 16), so that a read of 64 rows'
// chunks and a read of one row's ranks both hit all banks.  The next round's rows of Q, G and E are requested
// when this round's M is formed and arrive behind its P product and the next G-hat; one register set of each is
// enough, which leaves room for two wavefronts per SIMD.  Sums are those of the form above, to the bit.
// Microseconds, before and now: 8192^2, W = 16, r = 64 3720 / 3020; ResNet-18 set, W = 8, r = 50 373 / 277; 16 x (512 x 4096),
// W = 8 970 / 676; ragged set (64 x 27 .. 1000 x 2049), W = 4, r = 50 88 / 67.  At 8192^2 the matrix pipes are busy 67 % of
// the time, at a clock that falls from 2.4 to 2.1 GHz under them.
// ---------------------------------------------------------------------------
template <int MODE, bool GB16, bool NTS>
__device__ __forceinline__ void mfma_pair_tile(const float* __restrict__ G, float* __restrict__ M, const float* Q, const float* Pb,
                                               float* __restrict__ Pp, int cols, int r, int item_row0, int item_rows,
                                               int col0, int col1, int lane, int wave, char* qs, float (*lds_all)[32 * kLP]) {
  static_assert(MODE == kMAdd || MODE == kMAddFused, "add modes");
  constexpr bool NEEDG = MODE == kMAddFused;
  constexpr int RP = 64, KH = 32, NB = 2;
  constexpr int EARLY = NEEDG ? 12 : 16;           // requests of a block, of 16, that go out with the round before it
  constexpr int KIND = kRagged;                    // of edge blocks (takes aligned rows too)
  const int tid = threadIdx.x, li = lane & 31, h = lane >> 5;
  const int ph = wave & 3;
  const int row0 = item_row0 + 32 * (wave >> 2), nrows = min(32, item_rows - 32 * (wave >> 2));   // (nrows <= 0: none)
  float* lds = lds_all[wave];
  float pa[KH];
  if constexpr (NEEDG) {
#pragma unroll
    for (int k = 0; k < KH; ++k) pa[k] = 0.0f;
    if (li < nrows) {
      const char* src = reinterpret_cast<const char*>(Pb + (size_t)row0 * RP);
#pragma unroll
      for (int t = 0; t < KH / 4; ++t) {
        const Pk<4> x = ldrow<false>(src + 16 * t, (unsigned)(li * RP + KH * h) * 4u);
        pa[4 * t] = x.v[0]; pa[4 * t + 1] = x.v[1]; pa[4 * t + 2] = x.v[2]; pa[4 * t + 3] = x.v[3];
      }
    }
  }
  v16f accP[NB], accP2[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int i = 0; i < 16; ++i) { accP[nb][i] = 0.0f; accP2[nb][i] = 0.0f; }

  // 256 rows of Q: thread t moves chunk t % 16 of rows t / 16 + 32 i
  Pk<4> st[8];
  const int qrow = tid >> 4;
  char* const qdst = qs + qrow * (RP * 4) + ((((tid & 15) ^ (qrow & 15))) << 4);
  auto fetch_q = [&](auto full_tag, const int tid, const int c0, const int i0, const int i1) __attribute__((always_inline)) {
    unsigned lq = (unsigned)tid * 16u;
    asm volatile("" : "+v"(lq));
#pragma unroll
    for (int i = i0; i < i1; ++i) {
      if constexpr (decltype(full_tag)::value) {
        st[i] = ldrow<false>(reinterpret_cast<const char*>(Q + (size_t)(c0 + 32 * i) * RP), lq);
      } else {
        const int c = c0 + (tid >> 4) + 32 * i;
        st[i] = ldrow<false>(reinterpret_cast<const char*>(Q + (size_t)min(c, col1 - 1) * RP), (unsigned)(tid & 15) * 16u);
#pragma unroll
        for (int v = 0; v < 4; ++v) st[i].v[v] = keep_if(st[i].v[v], c < col1);
      }
    }
  };
  auto place_q = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 8; ++i)
      *reinterpret_cast<float4*>(qdst + i * (32 * RP * 4)) = make_float4(st[i].v[0], st[i].v[1], st[i].v[2], st[i].v[3]);
  };

  Pk<4> g[8], e[8];
  // A lane's place in 4 rows of a whole block is one offset from a wave-uniform base.  It is hidden from the optimiser, which
  // otherwise keeps the sums of the two for all rows, 64 bits each, in registers across the rounds.
  auto place = [&](const int ln) __attribute__((always_inline)) {
    unsigned lo = (unsigned)((ln >> 4) * cols + (ln & 15) * 4) * 4u;
    asm volatile("" : "+v"(lo));
    return lo;
  };
  // Requests k0 .. k1 of the 16 of a whole block: G and E of the block's rows 4 i + sr in turn.  real false: of the first
  // rows of Q instead, for a round that has no next one (a branch around a request would part the loop in two).
  auto fetch = [&](const bool real, const int ln, const int c, const int k0, const int k1) __attribute__((always_inline)) {
    unsigned lo = place(ln);
    if (!real) lo = (unsigned)ln * 16u;
#pragma unroll
    for (int k = k0; k < k1; ++k) {
      const int i = k >> 1;
      const size_t off = (size_t)(row0 + 4 * i) * cols + c;
      const char* base = (k & 1) ? reinterpret_cast<const char*>(M + off) : grad_row<GB16>(G, off);
      if (!real) base = reinterpret_cast<const char*>(Q);
      if (k & 1) {
        e[i] = ldrow<NTS>(base, lo);
      } else if constexpr (GB16) {                 // kept packed (two registers) until the block is worked on
        const Pk<2> x = ldrow_bf16_packed<LQSGD_NT_G != 0>(base, lo);
        g[i].v[0] = x.v[0]; g[i].v[1] = x.v[1];
      } else {
        g[i] = ldgrad<LQSGD_NT_G != 0, GB16>(base, lo);
      }
    }
  };
  auto fetch_edge = [&](const int ln, const int c) __attribute__((always_inline)) {
    const int sr = ln >> 4, cl = c + (ln & 15) * 4;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const size_t off = (size_t)(row0 + min(4 * i + sr, nrows - 1)) * cols;   // rows beyond nrows repeat the last one, and are never stored
      g[i] = ldedge<KIND, LQSGD_NT_G != 0, GB16>(grad_row<GB16>(G, off), cl, cols);
      e[i] = ldedge<KIND, NTS, false>(reinterpret_cast<const char*>(M + off), cl, cols);
    }
    if (cl + 4 > cols) {
#pragma unroll
      for (int i = 0; i < 8; ++i) { edge_fix<1>(g[i].v, cl, cols); edge_fix<1>(e[i].v, cl, cols); }
    }
  };
  // M of the block that g and e hold, to memory and to this wavefront's LDS tile
  // (late: the block's last requests are made here, between the matrix instructions)
  auto form = [&](auto full_tag, auto late_tag, const int ln, const int c) __attribute__((always_inline)) {
    constexpr bool FULL = decltype(full_tag)::value;
    const int li = ln & 31, h = ln >> 5, sr = ln >> 4, c4 = (ln & 15) * 4;
    if constexpr (NEEDG) {
      // rows li and 32 + li of this wavefront's part of Q, ranks 32 h .. 32 h + 31
      unsigned qb = (unsigned)((64 * ph + li) * (RP * 4) + (((8 * h) ^ (li & 15)) << 4));
      asm volatile("" : "+v"(qb));                 // (the exclusive ors below stay here, and out of registers across the rounds)
      v16f gh0, gh1;
#pragma unroll
      for (int i = 0; i < 16; ++i) { gh0[i] = 0.0f; gh1[i] = 0.0f; }
#pragma unroll
      for (int t = 0; t < KH / 4; ++t) {
        const float4 q0 = *reinterpret_cast<const float4*>(qs + (qb ^ (16 * t)));
        const float4 q1 = *reinterpret_cast<const float4*>(qs + (qb ^ (16 * t)) + 32 * RP * 4);
        gh0 = __builtin_amdgcn_mfma_f32_32x32x2f32(pa[4 * t], q0.x, gh0, 0, 0, 0);
        gh1 = __builtin_amdgcn_mfma_f32_32x32x2f32(pa[4 * t], q1.x, gh1, 0, 0, 0);
        gh0 = __builtin_amdgcn_mfma_f32_32x32x2f32(pa[4 * t + 1], q0.y, gh0, 0, 0, 0);
        gh1 = __builtin_amdgcn_mfma_f32_32x32x2f32(pa[4 * t + 1], q1.y, gh1, 0, 0, 0);
        gh0 = __builtin_amdgcn_mfma_f32_32x32x2f32(pa[4 * t + 2], q0.z, gh0, 0, 0, 0);
        gh1 = __builtin_amdgcn_mfma_f32_32x32x2f32(pa[4 * t + 2], q1.z, gh1, 0, 0, 0);
        gh0 = __builtin_amdgcn_mfma_f32_32x32x2f32(pa[4 * t + 3], q0.w, gh0, 0, 0, 0);
        gh1 = __builtin_amdgcn_mfma_f32_32x32x2f32(pa[4 * t + 3], q1.w, gh1, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (decltype(late_tag)::value) {
          if (t < 16 - EARLY) fetch(true, ln, c, EARLY + t, EARLY + t + 1);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        lds[(8 * (v >> 2) + 4 * h + (v & 3)) * kLP + li] = gh0[v];
        lds[(8 * (v >> 2) + 4 * h + (v & 3)) * kLP + 32 + li] = gh1[v];
      }
      wave_lds_fence();
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float4 t = *reinterpret_cast<const float4*>(lds + (4 * i + sr) * kLP + c4);
        e[i].v[0] -= t.x; e[i].v[1] -= t.y; e[i].v[2] -= t.z; e[i].v[3] -= t.w;
      }
      wave_lds_fence();
    }
    const unsigned lo = FULL ? place(ln) : 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      Pk<4> m, gv = g[i];
      if constexpr (GB16 && FULL) gv = unpack_bf16(g[i].v[0], g[i].v[1]);
#pragma unroll
      for (int v = 0; v < 4; ++v) m.v[v] = gv.v[v] + e[i].v[v];
      if constexpr (FULL)
        strow<NTS>(reinterpret_cast<char*>(M + (size_t)(row0 + 4 * i) * cols + c), lo, m);
      else if (4 * i + sr < nrows)
        stgroup<NTS>(reinterpret_cast<char*>(M + (size_t)(row0 + 4 * i + sr) * cols), (unsigned)(c + c4) * 4u, cols - c - c4, m);
      *reinterpret_cast<float4*>(lds + (4 * i + sr) * kLP + c4) = make_float4(m.v[0], m.v[1], m.v[2], m.v[3]);
    }
    wave_lds_fence();
  };
  // between(j): called after the j-th of eight groups of matrix instructions
  auto product = [&](const int ln, auto&& between) __attribute__((always_inline)) {
    const int li = ln & 31, h = ln >> 5;
    // ranks li and 32 + li of row 32 h + kk of this wavefront's part of Q
    unsigned bq = (unsigned)((64 * ph + 32 * h) * (RP * 4) + li * 4);
    asm volatile("" : "+v"(bq));
    auto q_at = [&](int nb, int kk) __attribute__((always_inline)) {
      return *reinterpret_cast<const float*>(qs + (bq ^ (16 * (kk & 7))) + kk * (RP * 4) + (nb ^ ((kk >> 3) & 1)) * 128);
    };
#pragma unroll
    for (int t = 0; t < 8; t += 2) {
      const float4 a0 = *reinterpret_cast<const float4*>(lds + li * kLP + 32 * h + 4 * t);
      const float4 a1 = *reinterpret_cast<const float4*>(lds + li * kLP + 32 * h + 4 * t + 4);
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        accP[nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0.x, q_at(nb, 4 * t + 0), accP[nb], 0, 0, 0);
        accP2[nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1.x, q_at(nb, 4 * t + 4), accP2[nb], 0, 0, 0);
        accP[nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0.y, q_at(nb, 4 * t + 1), accP[nb], 0, 0, 0);
        accP2[nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1.y, q_at(nb, 4 * t + 5), accP2[nb], 0, 0, 0);
        accP[nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0.z, q_at(nb, 4 * t + 2), accP[nb], 0, 0, 0);
        accP2[nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1.z, q_at(nb, 4 * t + 6), accP2[nb], 0, 0, 0);
        accP[nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0.w, q_at(nb, 4 * t + 3), accP[nb], 0, 0, 0);
        accP2[nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1.w, q_at(nb, 4 * t + 7), accP2[nb], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);         // (keeps the reads of all steps from being drawn together: registers)
        between(t + nb);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };

  int c0 = col0;
  const bool small_offsets = cols < (1 << 26);     // byte offsets within 4 rows fit 32 bits
  // whole rounds: 64 rows x 256 columns, the next one's requests ahead of this one's P product
  const int whole = item_rows == 64 && small_offsets ? (col1 - col0) / 256 : 0;
  if (whole > 0) {
    fetch_q(std::true_type{}, tid, c0, 0, 8);
    __builtin_amdgcn_sched_barrier(0);
    fetch(true, lane, c0 + 64 * ph, 0, EARLY);
    const int cend = col0 + 256 * whole;
    do {
      place_q();
      __syncthreads();
      form(std::true_type{}, std::bool_constant<NEEDG>{}, lane, c0 + 64 * ph);
      c0 += 256;
      // The next round's requests go out between the matrix instructions, a few at a time: made in one go, 24 a wavefront,
      // they fill what a CU can have outstanding, and all eight wavefronts wait for room before their next matrix instruction.
      // The rows of Q first: requests complete in order, and these are needed first.
      product(lane, [&](const int j) __attribute__((always_inline)) {
        if (j < 4) fetch_q(std::true_type{}, tid, min(c0, cend - 256), 2 * j, 2 * j + 2);
        else fetch(c0 < cend, lane, c0 + 64 * ph, (j - 4) * (EARLY / 4), (j - 3) * (EARLY / 4));
      });
      __syncthreads();
    } while (c0 < cend);
  }
  for (; c0 < col1; c0 += 256) {                   // (the same number of rounds, and of barriers, for all wavefronts)
    const int c = c0 + 64 * ph;
    // The lane number is hidden from the optimiser, which otherwise keeps addresses of these rounds in registers that the
    // whole rounds need.
    int ln = lane, td = tid;
    asm volatile("" : "+v"(ln), "+v"(td));
    fetch_q(std::false_type{}, td, c0, 0, 8);
    place_q();
    __syncthreads();
    if (nrows > 0 && c < col1) {
      if (nrows == 32 && c + 64 <= col1 && small_offsets) {
        fetch(true, ln, c, 0, 16);
        form(std::true_type{}, std::false_type{}, ln, c);
      } else {
        fetch_edge(ln, c);
        form(std::false_type{}, std::false_type{}, ln, c);
      }
      product(ln, [](int) {});
    }
    __syncthreads();
  }
  // P partial of the item = sum over the four wavefronts of its rows, added in wavefront order
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int v = 0; v < 16; ++v)
      lds[(8 * (v >> 2) + 4 * h + (v & 3)) * kLP + 32 * nb + li] = accP[nb][v] + accP2[nb][v];
  __syncthreads();
  const float (*const part)[32 * kLP] = lds_all + (wave & 4);
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int rr = ((tid & 255) >> 6) + 4 * i, k = tid & 63;
    const float t = ((part[0][rr * kLP + k] + part[1][rr * kLP + k]) + part[2][rr * kLP + k]) + part[3][rr * kLP + k];
    if (rr < nrows && k < r) Pp[(size_t)(row0 + rr) * r + k] = t;
  }
}

template <int MODE, bool GB16, bool NTS>
__global__ __launch_bounds__(512, 2) void mfma_pair_kernel(DevArgs a, const Tile* __restrict__ tiles, int ntiles, int reverse) {
  __shared__ __attribute__((aligned(256))) char qs[256 * 64 * 4];
  __shared__ __attribute__((aligned(16))) float lds_all[8][32 * kLP];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & (kWave - 1);
  if (blockIdx.x == 0) zero_absmax_cells(a, 512);
  const Tile tl = tiles[reverse ? ntiles - 1 - (int)blockIdx.x : (int)blockIdx.x];   // one item per workgroup
  const int layer = tl.lw / a.W, worker = tl.lw - layer * a.W;
  const LayerDesc& ld = a.layers[layer];
  const float* G = a.grads[(size_t)worker * a.n_all + ld.gidx];
  float* M = a.E + (size_t)worker * a.m_stride + ld.m_off;
  float* Pp = a.Ppart + (size_t)worker * a.ppart_stride + ld.ppart_off + (size_t)tl.aux * ld.np_pad;
  const int col0 = tl.aux * ld.segw;
  const int col1 = min(ld.cols, col0 + ld.segw);
  if (ld.kind == kOneColumnPerLane) {            // eight of the item's rows per wavefront
    const int nr = min(8, tl.nrows - 8 * wave);
    if (nr > 0)
      narrow_rows<64, 8, true, MODE == kMAddFused, true, false, GB16>(G, M, q_operand(a, ld), p_operand(a, ld), Pp, nullptr,
                                                                      ld.cols, ld.r, tl.row0 + 8 * wave, nr, lane, 0, 0.0f);
    return;
  }
  mfma_pair_tile<MODE, GB16, NTS>(G, M, q_operand(a, ld), p_operand(a, ld), Pp, ld.cols, ld.r, tl.row0, tl.nrows,
                                  col0, col1, lane, wave, qs, lds_all);
}

// ---------------------------------------------------------------------------
// The add modes at rank pads 16 and 32, loads and matrix work split differently over the wavefronts of a workgroup.
//
// What bounds this sweep is the order in which its streams reach memory (8192 columns, nothing but its loads and stores,
// microseconds per million elements: pieces of 32 columns a wavefront, 64 rows a workgroup 2.4, 32 rows 2.15; 32 rows in
// pieces of 256 columns with a barrier a round 1.95 - 2.05).  So in a round of 32 rows x 256 columns wavefront w loads and
// stores rows 8 w .. 8 w + 7, 1 KiB each, and multiplies columns 64 w .. 64 w + 63; G-hat and M change hands in an LDS
// tile.  G and E of the next round are requested between the matrix instructions of this one, the 64 rows of Q that
// a wavefront multiplies with come once, coalesced, through LDS of its own (they used to come twice from L2, in 40 requests a
// wavefront and round, most of them 4 bytes a lane) and are read there in both operand layouts: chunk x of 16 bytes of row c
// lies in row c ^ (c / 16 % 2) at x ^ (c / 2 % 8), so that a read of 32 rows' chunks and a read of two rows' ranks both hit all
// banks.  Two workgroups a CU, so that one's barriers and first requests hide behind the other's work: with eight wavefronts to a
// workgroup, one to a CU and requests two rounds ahead, items of few rounds wait (16 x 1024^2, W = 8 304 / 354 us; 8192^2,
// W = 4 615 / 593).  At rank pad 32 blocks of 32 columns accumulate on their own and are added at the end in their order, at rank
// pad 16 a wavefront's 64 columns.
// Microseconds at r = 32 unless said otherwise, W = 8, with 32 x 32 blocks per wavefront / now: ResNet-18 set 239 / 216, with
// bfloat16 gradients 233 / 189; 8192^2, W = 16 2431 / 2246; 4 x (3000 x 5000), r = 20 1892 / 1273; 32 x (512 x 4608) 1446 / 1342;
// sets as small as 4 x 1024^2, W = 2 29 / 27.  At r = 16, with 32 x 64 blocks per wavefront / now: ResNet-18 set 209 / 201, at r = 12
// with bfloat16 gradients 218 / 162; 8192^2 1091 / 1025; 4 x (3000 x 5000) 1283 / 1246; ragged set (64 x 27 .. 1000 x 2049), r = 12,
// W = 4 52 / 42; 4 x 1024^2, W = 2 28.6 / 24.7.
// Lists that have a CU an item lost in first iterations and where rounds are cut short, and go by blocks there (mfma_sweep32_kernel).
// Sets measured that lost and still do, a step: r = 32 16 x (512 x 576) 230 / 235, 24 x (512 x 320) 226 / 229, r = 16 8 x (512 x 2304)
// 298 / 303 (all in sweep 1 behind it); a first iteration's sweep 0 at r = 32: 16 x (512 x 2048) 318 / 334
// (ResNet-18 set 214 / 211, at r = 16 194 / 191).
// ---------------------------------------------------------------------------
constexpr int kLP256 = 260;  // LDS pitch (floats) of the 32 x 256 tile: 16-byte aligned rows, 4-bank skew per row

template <int RP, int MODE, bool GB16, bool NTS>
__device__ __forceinline__ void mfma_round_tile(const float* __restrict__ G, float* __restrict__ M, const float* Q, const float* Pb,
                                                float* __restrict__ Pp, int cols, int r, int row0, int nrows, int col0, int col1,
                                                int lane, int wave, char* qs, float* tile) {
  static_assert((RP == 16 || RP == 32) && (MODE == kMAdd || MODE == kMAddFused), "add modes at rank pads 16 and 32");
  constexpr bool NEEDG = MODE == kMAddFused;
  constexpr int KH = RP / 2;
  constexpr int NP = RP == 32 ? 2 : 1;             // sums of P a wavefront keeps: of each block of 32 columns, or of all 64
  constexpr int LPR = RP / 4, RPQ = 64 / LPR;      // 16-byte chunks of a row of Q, rows that a request moves
  constexpr int NBK = 2, RPW = 8;                  // blocks of 32 columns that a wavefront multiplies, rows that it moves
  constexpr int KIND = kRagged;                    // of edge rounds (takes aligned rows too)
  qs += wave * (NBK * 32 * RP * 4);
  float pa[KH];
  if constexpr (NEEDG) {
    const int li = lane & 31, h = lane >> 5;
#pragma unroll
    for (int k = 0; k < KH; ++k) pa[k] = 0.0f;
    if (li < nrows) {
      const char* src = reinterpret_cast<const char*>(Pb + (size_t)row0 * RP);
#pragma unroll
      for (int t = 0; t < KH / 4; ++t) {
        const Pk<4> x = ldrow<false>(src + 16 * t, (unsigned)(li * RP + KH * h) * 4u);
        pa[4 * t] = x.v[0]; pa[4 * t + 1] = x.v[1]; pa[4 * t + 2] = x.v[2]; pa[4 * t + 3] = x.v[3];
      }
    }
  }
  v16f accP[NP], accP2[NP];
#pragma unroll
  for (int b = 0; b < NP; ++b)
#pragma unroll
    for (int i = 0; i < 16; ++i) { accP[b][i] = 0.0f; accP2[b][i] = 0.0f; }

  // its rows of Q: request i moves rows RPQ i .. RPQ i + RPQ - 1, 16 bytes a lane
  constexpr int NQ = 64 / RPQ;
  Pk<4> st[NQ];
  auto fetch_q = [&](auto full_tag, const int ln, const int c0) __attribute__((always_inline)) {
    unsigned lq = (unsigned)ln * 16u;
    asm volatile("" : "+v"(lq));
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
      if constexpr (decltype(full_tag)::value) {
        st[i] = ldrow<false>(reinterpret_cast<const char*>(Q + (size_t)(c0 + RPQ * i) * RP), lq);
      } else {
        const int c = c0 + RPQ * i + ln / LPR;
        st[i] = ldrow<false>(reinterpret_cast<const char*>(Q + (size_t)min(c, col1 - 1) * RP), (unsigned)(ln % LPR) * 16u);
#pragma unroll
        for (int v = 0; v < 4; ++v) st[i].v[v] = keep_if(st[i].v[v], c < col1);
      }
    }
  };
  auto place_q = [&](const int ln) __attribute__((always_inline)) {
    // (rank pad 16: chunk x of row c lies at x ^ (c / 4 % 4))
    const unsigned w = RP == 32 ? (unsigned)((ln >> 3) * (RP * 4) + (((ln & 7) ^ (ln >> 4)) << 4))
                                : (unsigned)((ln >> 2) * (RP * 4) + (((ln & 3) ^ (ln >> 4)) << 4));
#pragma unroll
    for (int i = 0; i < NQ; ++i)
      *reinterpret_cast<float4*>(qs + (RP == 32 ? w ^ (128u * ((i >> 1) & 1)) ^ (64u * (i & 1)) : w) + i * (RPQ * RP * 4)) =
          make_float4(st[i].v[0], st[i].v[1], st[i].v[2], st[i].v[3]);
    wave_lds_fence();
  };
  // Requests k0 .. k1 of the round at c0, whole or partial: G and E of this wavefront's rows in turn, lo(c0) its lane's place.
  // real false: of the first rows of Q instead, for a round that has no next one (a branch around a request would part the
  // loop in two).  Addresses count from back columns before c0, so that a partial round's last lanes, which load the row's last
  // four columns (edge_col), stay at or behind them.
  auto place = [&](const bool real, const int c0, const int back) __attribute__((always_inline)) {
    unsigned lo = (unsigned)(real ? min(back + 4 * lane, back + col1 - 4 - c0) : 4 * lane) * 4u;
    asm volatile("" : "+v"(lo));
    return lo;
  };
  auto fetch = [&](const bool real, const unsigned lo, const int c0, const int back, Pk<4>* g, Pk<4>* e, const int k0, const int k1) __attribute__((always_inline)) {
#pragma unroll
    for (int k = k0; k < k1; ++k) {
      const int i = k >> 1;
      const size_t off = (size_t)(row0 + RPW * wave + i) * cols + (c0 - back);
      const char* base = (k & 1) ? reinterpret_cast<const char*>(M + off) : grad_row<GB16>(G, off);
      if (!real) base = reinterpret_cast<const char*>(Q);
      if (k & 1) {
        e[i] = ldrow<NTS>(base, lo);
      } else if constexpr (GB16) {                 // kept packed (two registers) until the round is worked on
        const Pk<2> x = ldrow_bf16_packed<LQSGD_NT_G != 0>(base, lo);
        g[i].v[0] = x.v[0]; g[i].v[1] = x.v[1];
      } else {
        g[i] = ldgrad<LQSGD_NT_G != 0, GB16>(base, lo);
      }
    }
  };
  auto fetch_edge = [&](const int ln, const int c0, Pk<4>* g, Pk<4>* e) __attribute__((always_inline)) {
    const int cl = c0 + 4 * ln;
#pragma unroll
    for (int i = 0; i < RPW; ++i) {
      const size_t off = (size_t)(row0 + min(RPW * wave + i, nrows - 1)) * cols;   // rows beyond nrows repeat the last one, and are never stored
      g[i] = ldedge<KIND, LQSGD_NT_G != 0, GB16>(grad_row<GB16>(G, off), cl, cols);
      e[i] = ldedge<KIND, NTS, false>(reinterpret_cast<const char*>(M + off), cl, cols);
    }
    if (cl + 4 > cols) {
#pragma unroll
      for (int i = 0; i < RPW; ++i) { edge_fix<1>(g[i].v, cl, cols); edge_fix<1>(e[i].v, cl, cols); }
    }
  };
  // G-hat of this wavefront's 64 columns, into the tile
  auto reconstruct = [&](const int ln) __attribute__((always_inline)) {
    const int li = ln & 31, h = ln >> 5;
    // row li of this wavefront's rows of Q, ranks KH h .. KH h + KH - 1
    const unsigned qb = RP == 32 ? (unsigned)((li ^ (li >> 4)) * (RP * 4) + (((4 * h) ^ ((li >> 1) & 7)) << 4))
                                 : (unsigned)(li * (RP * 4) + (((2 * h) ^ ((li >> 2) & 3)) << 4));
    v16f gh[NBK];
#pragma unroll
    for (int b = 0; b < NBK; ++b)
#pragma unroll
      for (int i = 0; i < 16; ++i) gh[b][i] = 0.0f;
#pragma unroll
    for (int t = 0; t < KH / 4; ++t) {
      float4 q[NBK];
#pragma unroll
      for (int b = 0; b < NBK; ++b) q[b] = *reinterpret_cast<const float4*>(qs + (qb ^ (16 * t)) + b * (32 * RP * 4));
#pragma unroll
      for (int b = 0; b < NBK; ++b) gh[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(pa[4 * t], q[b].x, gh[b], 0, 0, 0);
#pragma unroll
      for (int b = 0; b < NBK; ++b) gh[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(pa[4 * t + 1], q[b].y, gh[b], 0, 0, 0);
#pragma unroll
      for (int b = 0; b < NBK; ++b) gh[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(pa[4 * t + 2], q[b].z, gh[b], 0, 0, 0);
#pragma unroll
      for (int b = 0; b < NBK; ++b) gh[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(pa[4 * t + 3], q[b].w, gh[b], 0, 0, 0);
    }
#pragma unroll
    for (int b = 0; b < NBK; ++b)
#pragma unroll
      for (int v = 0; v < 16; ++v) tile[(8 * (v >> 2) + 4 * h + (v & 3)) * kLP256 + 32 * (NBK * wave + b) + li] = gh[b][v];
  };
  // M of this wavefront's eight rows, to memory and into the tile
  auto form = [&](auto full_tag, const int ln, const int c0, Pk<4>* g, Pk<4>* e) __attribute__((always_inline)) {
    constexpr bool FULL = decltype(full_tag)::value;
    float* mine = tile + RPW * wave * kLP256 + 4 * ln;
#pragma unroll
    for (int i = 0; i < RPW; ++i) {
      if constexpr (NEEDG) {
        const float4 t = *reinterpret_cast<const float4*>(mine + i * kLP256);
        e[i].v[0] -= t.x; e[i].v[1] -= t.y; e[i].v[2] -= t.z; e[i].v[3] -= t.w;
      }
      Pk<4> m, gv = g[i];
      if constexpr (GB16 && FULL) gv = unpack_bf16(g[i].v[0], g[i].v[1]);
#pragma unroll
      for (int v = 0; v < 4; ++v) m.v[v] = gv.v[v] + e[i].v[v];
      if constexpr (FULL)
        strow<NTS>(reinterpret_cast<char*>(M + (size_t)(row0 + RPW * wave + i) * cols + c0), (unsigned)ln * 16u, m);
      else if (RPW * wave + i < nrows)
        stgroup<NTS>(reinterpret_cast<char*>(M + (size_t)(row0 + RPW * wave + i) * cols), (unsigned)(c0 + 4 * ln) * 4u, cols - c0 - 4 * ln, m);
      *reinterpret_cast<float4*>(mine + i * kLP256) = make_float4(m.v[0], m.v[1], m.v[2], m.v[3]);
    }
  };
  // P += M Q over this wavefront's 64 columns; between(j): called after the j-th of 4 NBK groups of matrix instructions
  auto product = [&](const int ln, auto&& between) __attribute__((always_inline)) {
    const int li = ln & 31, h = ln >> 5;
    if constexpr (RP == 16) {
      // rank li % 16 of row 32 h + kk (lanes 16 .. 31: columns of the block that nobody reads)
      const char* bq = qs + 32 * h * (RP * 4) + (li & 3) * 4;
      const unsigned ch = (unsigned)((li >> 2) & 3);
      auto q_at = [&](int kk) __attribute__((always_inline)) {
        return *reinterpret_cast<const float*>(bq + ((ch ^ ((kk >> 2) & 3)) << 4) + kk * (RP * 4));
      };
      const float* src = tile + li * kLP256 + 64 * wave + 32 * h;
#pragma unroll
      for (int t = 0; t < 8; t += 2) {
        const float4 a0 = *reinterpret_cast<const float4*>(src + 4 * t);
        const float4 a1 = *reinterpret_cast<const float4*>(src + 4 * t + 4);
        accP[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0.x, q_at(4 * t + 0), accP[0], 0, 0, 0);
        accP2[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1.x, q_at(4 * t + 4), accP2[0], 0, 0, 0);
        accP[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0.y, q_at(4 * t + 1), accP[0], 0, 0, 0);
        accP2[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1.y, q_at(4 * t + 5), accP2[0], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        between(t);
        __builtin_amdgcn_sched_barrier(0);
        accP[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0.z, q_at(4 * t + 2), accP[0], 0, 0, 0);
        accP2[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1.z, q_at(4 * t + 6), accP2[0], 0, 0, 0);
        accP[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0.w, q_at(4 * t + 3), accP[0], 0, 0, 0);
        accP2[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1.w, q_at(4 * t + 7), accP2[0], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        between(t + 1);
        __builtin_amdgcn_sched_barrier(0);
      }
      wave_lds_fence();
      return;
    } else {
    // rank li of row 16 h + kk of this wavefront's rows of Q
    unsigned bq = (unsigned)(16 * h * (RP * 4) + 128 * h + li * 4);
    asm volatile("" : "+v"(bq));                   // (the exclusive ors below stay here, and out of registers across the rounds)
    auto q_at = [&](int b, int kk) __attribute__((always_inline)) {
      return *reinterpret_cast<const float*>(qs + (bq ^ (128u * (kk & 1)) ^ (16u * ((kk >> 1) & 7))) + (32 * b + (kk & ~1)) * (RP * 4));
    };
    const float* src = tile + li * kLP256 + 32 * NBK * wave + 16 * h;
#pragma unroll
    for (int t = 0; t < 4; t += 2)                 // two accumulators a block (even / odd float4 of the lane's run of columns)
#pragma unroll
      for (int b = 0; b < NBK; ++b) {
        const float4 a0 = *reinterpret_cast<const float4*>(src + 32 * b + 4 * t);
        const float4 a1 = *reinterpret_cast<const float4*>(src + 32 * b + 4 * t + 4);
        accP[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0.x, q_at(b, 4 * t + 0), accP[b], 0, 0, 0);
        accP2[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1.x, q_at(b, 4 * t + 4), accP2[b], 0, 0, 0);
        accP[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0.y, q_at(b, 4 * t + 1), accP[b], 0, 0, 0);
        accP2[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1.y, q_at(b, 4 * t + 5), accP2[b], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        between(NBK * t + 2 * b);
        __builtin_amdgcn_sched_barrier(0);
        accP[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0.z, q_at(b, 4 * t + 2), accP[b], 0, 0, 0);
        accP2[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1.z, q_at(b, 4 * t + 6), accP2[b], 0, 0, 0);
        accP[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0.w, q_at(b, 4 * t + 3), accP[b], 0, 0, 0);
        accP2[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1.w, q_at(b, 4 * t + 7), accP2[b], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        between(NBK * t + 2 * b + 1);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    wave_lds_fence();
  };

  int c0 = col0;
  // Layers narrower than a round: the item's rows are one run of memory, which the threads share in pieces of 16 bytes whatever
  // the width.  (A row a request leaves most lanes with another lane's address, and such layers are nothing but partial rounds.
  // Sweep 0, W = 8, 32 x 64 or 32 x 32 blocks per wavefront / a row a request / now: r = 16 64 x (512 x 64) 96 / 134 / 100 us,
  // 64 x (512 x 96) 138 / 149 / 113, 48 x (512 x 128) 91 / 118 / 92, 32 x (512 x 130) 80 / 86 / 69, 40 x (512 x 192) 92 / 117 / 87,
  // at r = 32 135 / 152 / 116, 145 / 167 / 129, 124 / 132 / 105, 118 / 97 / 80, 130 / 128 / 102.)
  auto narrow = [&](auto n_tag, const int n4) __attribute__((always_inline)) {
    constexpr int N = decltype(n_tag)::value;
    int ln = lane, tid = threadIdx.x;              // hidden from the optimiser (see mfma_pair_tile)
    asm volatile("" : "+v"(ln), "+v"(tid));
    const bool mine = 32 * NBK * wave < cols;
    const char* gb = grad_row<GB16>(G, (size_t)row0 * cols);
    char* mb = reinterpret_cast<char*>(M + (size_t)row0 * cols);
    Pk<4> g[N], e[N];
    if (mine) fetch_q(std::false_type{}, ln, 32 * NBK * wave);
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const unsigned lo = (unsigned)min(tid + 256 * i, n4 - 1) * 16u;
      g[i] = ldgrad<LQSGD_NT_G != 0, GB16>(gb, lo);
      e[i] = ldrow<NTS>(mb, lo);
    }
    if (mine) {
      place_q(ln);
      if constexpr (NEEDG) reconstruct(ln);
    }
    if constexpr (!NEEDG)                          // columns of a wavefront's block that do not exist (G-hat is zero there)
      for (int x = tid; x < 32 * 64; x += 256) {
        const int col = cols + (x & 63);
        if (col < (cols + 63) / 64 * 64) tile[(x >> 6) * kLP256 + col] = 0.0f;
      }
    __syncthreads();
    const float inv = 1.0f / (float)cols;          // (at most 32 rows: half a column is far more than the product's rounding)
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int x = tid + 256 * i;
      if (x < n4) {
        const int row = (int)(((float)(4 * x) + 0.5f) * inv), col = 4 * x - row * cols;
        float* at = tile + row * kLP256 + col;
        Pk<4> m;
        if (cols % 4 == 0) {
          if constexpr (NEEDG) {
            const float4 t = *reinterpret_cast<const float4*>(at);
            e[i].v[0] -= t.x; e[i].v[1] -= t.y; e[i].v[2] -= t.z; e[i].v[3] -= t.w;
          }
#pragma unroll
          for (int v = 0; v < 4; ++v) m.v[v] = g[i].v[v] + e[i].v[v];
          *reinterpret_cast<float4*>(at) = make_float4(m.v[0], m.v[1], m.v[2], m.v[3]);
        } else {
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            float* const a1 = at + v + (col + v >= cols ? kLP256 - cols : 0);
            if constexpr (NEEDG) e[i].v[v] -= *a1;
            m.v[v] = g[i].v[v] + e[i].v[v];
            *a1 = m.v[v];
          }
        }
        strow<NTS>(mb, (unsigned)x * 16u, m);
      }
    }
    __syncthreads();
    if (mine) product(ln, [](int) {});
  };
  if (cols < 256 && nrows * cols % 4 == 0) {       // (else the last piece would reach beyond the layer)
    const int n4 = nrows * cols / 4;
    if (n4 <= 512) narrow(std::integral_constant<int, 2>{}, n4);
    else if (n4 <= 1024) narrow(std::integral_constant<int, 4>{}, n4);
    else narrow(std::integral_constant<int, 8>{}, n4);
    c0 = col1;
  }
  // whole rounds: 32 rows x 256 columns
  const int cend = nrows == 32 ? col0 + (col1 - col0) / 256 * 256 : col0;
  Pk<4> g[RPW], e[RPW];
  if (c0 < cend) {
    // The tile needs two barriers a round: G-hat is complete before rows are read, M before columns are.  A wavefront's
    // next G-hat goes to columns that only it reads, and no row is written before all have passed the first barrier again.
    fetch_q(std::true_type{}, lane, c0 + 32 * NBK * wave);
    __builtin_amdgcn_sched_barrier(0);
    fetch(true, place(true, c0, 0), c0, 0, g, e, 0, 2 * RPW);
    __builtin_amdgcn_sched_barrier(0);
    do {
      place_q(lane);
      fetch_q(std::true_type{}, lane, min(c0 + 256, cend - 256) + 32 * NBK * wave);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (NEEDG) reconstruct(lane);
      __syncthreads();
      form(std::true_type{}, lane, c0, g, e);
      c0 += 256;
      // A round without G-hat is short, and its requests all go out at once (a first iteration of the ResNet-18 set, W = 8: 237 us
      // spread as below, 208 at once).  With G-hat spread ones are as fast in large sets and faster in small ones (1024 x 576,
      // r = 20 58 / 62, 4 x 1024^2 79 / 85).
      // The partial round behind the whole ones is requested with the last of them, in a round without G-hat (sweep 0 of a first
      // iteration, W = 8, us: r = 32 24 x (512 x 320) 104 / 98, 24 x (512 x 448) 120 / 107, 16 x (512 x 832) 126 / 119, 8 x (512 x 4096)
      // 340 / 308; r = 16 86 / 78, 97 / 91, 118 / 110, 303 / 289; with G-hat 24 x (512 x 448), r = 32 130 / 133).
      const bool real = c0 < (NEEDG ? cend : col1);
      const unsigned lo = place(real, c0, 256);
      if constexpr (!NEEDG) fetch(real, lo, c0, 256, g, e, 0, 2 * RPW);
      __syncthreads();
      product(lane, [&](const int j) __attribute__((always_inline)) {
        if constexpr (NEEDG) fetch(real, lo, c0, 256, g, e, 2 * j, 2 * j + 2);
      });
    } while (c0 < cend);
  }
  for (; c0 < col1; c0 += 256) {                   // (the same number of rounds, and of barriers, for all wavefronts)
    int ln = lane;                                 // hidden from the optimiser (see mfma_pair_tile)
    asm volatile("" : "+v"(ln));
    const bool mine = c0 + 32 * NBK * wave < col1;
    if (!NEEDG && c0 == cend && cend > col0) {     // requested by the last whole round
      if constexpr (GB16)
#pragma unroll
        for (int i = 0; i < RPW; ++i) g[i] = unpack_bf16(g[i].v[0], g[i].v[1]);
      if (c0 + 4 * ln + 4 > cols) {
#pragma unroll
        for (int i = 0; i < RPW; ++i) { edge_fix<1>(g[i].v, c0 + 4 * ln, cols); edge_fix<1>(e[i].v, c0 + 4 * ln, cols); }
      }
    } else {
      fetch_edge(ln, c0, g, e);
    }
    if (mine) {
      fetch_q(std::false_type{}, ln, c0 + 32 * NBK * wave);
      place_q(ln);
      if constexpr (NEEDG) reconstruct(ln);
    }
    __syncthreads();
    form(std::false_type{}, ln, c0, g, e);
    __syncthreads();
    if (mine) product(ln, [](int) {});
  }
  __syncthreads();
  // P partial of the item = sum over the eight blocks of a round (rank pad 16: the four wavefronts), added in their order
  const int li = lane & 31, h = lane >> 5;
#pragma unroll
  for (int b = 0; b < NP; ++b) {
    float* part = tile + (NP * wave + b) * (32 * kLP32);
#pragma unroll
    for (int v = 0; v < 16; ++v) part[(8 * (v >> 2) + 4 * h + (v & 3)) * kLP32 + li] = accP[b][v] + accP2[b][v];
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int x = (int)threadIdx.x + 256 * i, rr = x >> 5, k = x & 31;
    float t = tile[rr * kLP32 + k];
#pragma unroll
    for (int wv = 1; wv < 4 * NP; ++wv) t += tile[wv * (32 * kLP32) + rr * kLP32 + k];
    if (rr < nrows && k < r) Pp[(size_t)(row0 + rr) * r + k] = t;
  }
}

template <int RP, int MODE, bool GB16, bool NTS>
__global__ __launch_bounds__(256, RP == 16 && MODE == kMAdd ? 3 : 2) void mfma_round_kernel(DevArgs a, const Tile* __restrict__ tiles, int ntiles, int reverse) {
  __shared__ __attribute__((aligned(256))) char qs[8 * 32 * RP * 4];
  __shared__ __attribute__((aligned(16))) float tile[8 * 32 * kLP32];   // 32 x kLP256 in the rounds, the partial sums after them
  static_assert(32 * kLP256 <= 8 * 32 * kLP32, "");
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & (kWave - 1);
  if (blockIdx.x == 0) zero_absmax_cells(a, 256);
  const Tile tl = tiles[reverse ? ntiles - 1 - (int)blockIdx.x : (int)blockIdx.x];   // one item per workgroup
  const int layer = tl.lw / a.W, worker = tl.lw - layer * a.W;
  const LayerDesc& ld = a.layers[layer];
  const float* G = a.grads[(size_t)worker * a.n_all + ld.gidx];
  float* M = a.E + (size_t)worker * a.m_stride + ld.m_off;
  float* Pp = a.Ppart + (size_t)worker * a.ppart_stride + ld.ppart_off + (size_t)tl.aux * ld.np_pad;
  const int col0 = tl.aux * ld.segw;
  const int col1 = min(ld.cols, col0 + ld.segw);
  if (ld.kind == kOneColumnPerLane) {            // eight of the item's rows per wavefront
    const int nr = min(8, tl.nrows - 8 * wave);
    if (nr > 0)
      narrow_rows<RP, 8, true, MODE == kMAddFused, true, false, GB16>(G, M, q_operand(a, ld), p_operand(a, ld), Pp, nullptr, ld.cols,
                                                                      ld.r, tl.row0 + 8 * wave, nr, lane, 0, 0.0f);
    return;
  }
  mfma_round_tile<RP, MODE, GB16, NTS>(G, M, q_operand(a, ld), p_operand(a, ld), Pp, ld.cols, ld.r, tl.row0, tl.nrows,
                                   col0, col1, lane, wave, qs, tile);
}

// ---------------------------------------------------------------------------
// Sweep 0 at rank pad 32 for lists that have a CU an item (DevArgs::by_blocks): 32 x 32 blocks per wavefront.
//
// Such a list takes as long as its longest item, and an item as long as its chain of round trips to memory: a round of
// mfma_round_kernel pays two barriers, and one that is cut short a round trip of its own.  Here eight wavefronts walk the
// item's blocks on their own, 256 columns apart, with the next block's G, E and operands requested ahead; rows of Q come from
// L2 in operand layout, too many requests for a full chip.  Blocks of 32 columns accumulate and are added in the same order as
// there, and G-hat comes out of the same sequence of matrix instructions: the same bits.
// Sweep 0, r = 32, by rounds / here, us.  Deferred residual: 4 x (256 x 320), W = 4 16.7 / 12.9; 8 x (256 x 576), W = 4 23.0 / 19.3;
// 16 x (64 x 128), W = 4 9.9 / 8.2; 4 x (31 x 2048), W = 4 25.4 / 24.1; 16 x (20 x 2000), W = 8 32.1 / 27.7; 1000 x 1024, W = 4
// 27.2 / 24.5.  First iterations: 8 x (256 x 320), W = 4 15.7 / 11.7; 8 x (256 x 576), W = 4 20.4 / 16.3; 4 x (256 x 1024), W = 4
// 21.0 / 19.4; 8 x (256 x 1024), W = 4 28.6 / 25.5.  Where the rounds are whole or nearly, they win with the deferred residual (4 x (256 x 1024), W = 4
// 22.6 / 25.0; 2 x (64 x 988), W = 4 21.6 / 22.8).
// Row layout: 8 lanes = 128 contiguous bytes of a row, 8 rows per instruction.
// ---------------------------------------------------------------------------
template <int MODE, bool GB16>
__device__ __forceinline__ void mfma_tile32(const float* __restrict__ G, float* __restrict__ M,
                                            const float* Q, const float* Pb, float* __restrict__ Pp,
                                            int cols, int r, int row0, int nrows, int col0, int col1,
                                            int lane, int wave, float (*lds_all)[32 * kLP32]) {
  static_assert(MODE == kMAdd || MODE == kMAddFused, "add modes");
  constexpr int RP = 32;
  float* lds = lds_all[wave];
  constexpr bool NEEDG = (MODE != kMAdd);
  constexpr int KH = RP / 2;
  const int li = lane & 31, h = lane >> 5;
  const int sr = lane >> 3, c4 = (lane & 7) * 4;   // row layout: rows 8 i + sr, columns c4 .. c4 + 3
  float pa[KH];
  if constexpr (NEEDG) {
    const int row = row0 + li;
    if (li < nrows) {
      const float4* src = reinterpret_cast<const float4*>(Pb + (size_t)row * RP + KH * h);
#pragma unroll
      for (int t = 0; t < KH / 4; ++t) {
        const float4 x = src[t];
        pa[4 * t] = x.x; pa[4 * t + 1] = x.y; pa[4 * t + 2] = x.z; pa[4 * t + 3] = x.w;
      }
    } else {
#pragma unroll
      for (int k = 0; k < KH; ++k) pa[k] = 0.0f;
    }
  }
  v16f accP, accP2;
#pragma unroll
  for (int i = 0; i < 16; ++i) { accP[i] = 0.0f; accP2[i] = 0.0f; }

  // the G and E (or old M) values of one 32 x 32 block at an edge of the layer
  auto fetch = [&](const int c, Pk<4>* g, Pk<4>* e) {
    const int cl = c + c4;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const size_t off = (size_t)(row0 + min(8 * i + sr, nrows - 1)) * cols;   // rows beyond nrows: never stored
      g[i] = ldedge<kRagged, LQSGD_NT_G != 0, GB16>(grad_row<GB16>(G, off), cl, cols);
      e[i] = ldedge<kRagged, false, false>(reinterpret_cast<const char*>(M + off), cl, cols);
    }
    if (cl + 4 > cols) {
#pragma unroll
      for (int i = 0; i < 4; ++i) { edge_fix<1>(g[i].v, cl, cols); edge_fix<1>(e[i].v, cl, cols); }
    }
  };
  auto block = [&](const int c, Pk<4>* g, Pk<4>* e) {
    const int cl = c + c4;
    if constexpr (NEEDG) {
      float qb[KH];
      const int col = c + li;
      if (col < col1) {
        const float4* src = reinterpret_cast<const float4*>(Q + (size_t)col * RP + KH * h);
#pragma unroll
        for (int t = 0; t < KH / 4; ++t) {
          const float4 x = src[t];
          qb[4 * t] = x.x; qb[4 * t + 1] = x.y; qb[4 * t + 2] = x.z; qb[4 * t + 3] = x.w;
        }
      } else {
#pragma unroll
        for (int k = 0; k < KH; ++k) qb[k] = 0.0f;
      }
      v16f gh;
#pragma unroll
      for (int i = 0; i < 16; ++i) gh[i] = 0.0f;
#pragma unroll
      for (int k = 0; k < KH; ++k) gh = __builtin_amdgcn_mfma_f32_32x32x2f32(pa[k], qb[k], gh, 0, 0, 0);
#pragma unroll
      for (int v = 0; v < 16; ++v) lds[(8 * (v >> 2) + 4 * h + (v & 3)) * kLP32 + li] = gh[v];
      wave_lds_fence();
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float4 t = *reinterpret_cast<const float4*>(lds + (8 * i + sr) * kLP32 + c4);
        e[i].v[0] -= t.x; e[i].v[1] -= t.y; e[i].v[2] -= t.z; e[i].v[3] -= t.w;
      }
      wave_lds_fence();
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int rr = 8 * i + sr;
      Pk<4> m;
#pragma unroll
      for (int v = 0; v < 4; ++v) m.v[v] = g[i].v[v] + e[i].v[v];
      if (rr < nrows)
        stgroup<false>(reinterpret_cast<char*>(M + (size_t)(row0 + rr) * cols), (unsigned)cl * 4u, cols - cl, m);
      *reinterpret_cast<float4*>(lds + rr * kLP32 + c4) = make_float4(m.v[0], m.v[1], m.v[2], m.v[3]);
    }
    // the Q slice of the P product is fetched only now: the registers of the G-hat operands are free again
    float bq[16];
#pragma unroll
    for (int kk = 0; kk < 16; ++kk) {
      const int col = c + 16 * h + kk;
      bq[kk] = col < col1 ? Q[(size_t)col * RP + li] : 0.0f;
    }
    wave_lds_fence();
    {
      const float4 a0 = *reinterpret_cast<const float4*>(lds + li * kLP32 + 16 * h);
      const float4 a1 = *reinterpret_cast<const float4*>(lds + li * kLP32 + 16 * h + 4);
      const float4 a2 = *reinterpret_cast<const float4*>(lds + li * kLP32 + 16 * h + 8);
      const float4 a3 = *reinterpret_cast<const float4*>(lds + li * kLP32 + 16 * h + 12);
      accP = __builtin_amdgcn_mfma_f32_32x32x2f32(a0.x, bq[0], accP, 0, 0, 0);
      accP2 = __builtin_amdgcn_mfma_f32_32x32x2f32(a1.x, bq[4], accP2, 0, 0, 0);
      accP = __builtin_amdgcn_mfma_f32_32x32x2f32(a0.y, bq[1], accP, 0, 0, 0);
      accP2 = __builtin_amdgcn_mfma_f32_32x32x2f32(a1.y, bq[5], accP2, 0, 0, 0);
      accP = __builtin_amdgcn_mfma_f32_32x32x2f32(a0.z, bq[2], accP, 0, 0, 0);
      accP2 = __builtin_amdgcn_mfma_f32_32x32x2f32(a1.z, bq[6], accP2, 0, 0, 0);
      accP = __builtin_amdgcn_mfma_f32_32x32x2f32(a0.w, bq[3], accP, 0, 0, 0);
      accP2 = __builtin_amdgcn_mfma_f32_32x32x2f32(a1.w, bq[7], accP2, 0, 0, 0);
      accP = __builtin_amdgcn_mfma_f32_32x32x2f32(a2.x, bq[8], accP, 0, 0, 0);
      accP2 = __builtin_amdgcn_mfma_f32_32x32x2f32(a3.x, bq[12], accP2, 0, 0, 0);
      accP = __builtin_amdgcn_mfma_f32_32x32x2f32(a2.y, bq[9], accP, 0, 0, 0);
      accP2 = __builtin_amdgcn_mfma_f32_32x32x2f32(a3.y, bq[13], accP2, 0, 0, 0);
      accP = __builtin_amdgcn_mfma_f32_32x32x2f32(a2.z, bq[10], accP, 0, 0, 0);
      accP2 = __builtin_amdgcn_mfma_f32_32x32x2f32(a3.z, bq[14], accP2, 0, 0, 0);
      accP = __builtin_amdgcn_mfma_f32_32x32x2f32(a2.w, bq[11], accP, 0, 0, 0);
      accP2 = __builtin_amdgcn_mfma_f32_32x32x2f32(a3.w, bq[15], accP2, 0, 0, 0);
    }
    wave_lds_fence();
  };
  // Interior blocks (all 32 rows and 32 columns exist) run without bounds tests, as a software
  // pipeline inside the wavefront: the next block's G and E are requested before this block's matrix
  // instructions, and the next block's G-hat operand from Q as soon as this block's G-hat is done.
  // Requests complete in order, so everything a block waits for is requested before the prefetch.
  int c = col0 + 32 * wave;
  if (nrows == 32 && c + 32 <= col1 && cols < (1 << 26)) {   // (byte offsets within 8 rows fit 32 bits)
    const int last = c + ((col1 - 32 - c) / 256) * 256;   // this wavefront's last whole block
    Pk<4> g[4], e[4], gn[4], en[4];
    float qb[KH], bq[16];
    // Addresses are a wave-uniform base (scalar registers, advanced by scalar adds) plus a byte
    // offset per lane that does not change from block to block.
    const unsigned goff = (unsigned)(sr * cols + c4) * 4u;      // lane's place in a slab of 8 rows
    const unsigned qboff = (unsigned)(li * RP + KH * h) * 4u;   // ... in 32 rows of Q (G-hat operand)
    const unsigned bqoff = (unsigned)(16 * h * RP + li) * 4u;   // ... in 32 rows of Q (P operand)
    auto fetch_ge = [&](const int cb, Pk<4>* gg, Pk<4>* ee) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const size_t off = (size_t)(row0 + 8 * i) * cols + cb;
        if constexpr (GB16) {   // kept packed (two registers) until the block is worked on
          const Pk<2> t = ldrow_bf16_packed<LQSGD_NT_G != 0>(grad_row<GB16>(G, off), goff);
          gg[i].v[0] = t.v[0]; gg[i].v[1] = t.v[1];
        } else {
          gg[i] = ldgrad<LQSGD_NT_G != 0, GB16>(grad_row<GB16>(G, off), goff);
        }
        ee[i] = ldrow<false>(reinterpret_cast<const char*>(M + off), goff);
      }
    };
    auto fetch_qb = [&](const int cb) {
      const char* base = reinterpret_cast<const char*>(Q + (size_t)cb * RP);
#pragma unroll
      for (int t = 0; t < KH / 4; ++t) {
        const Pk<4> x = ldrow<false>(base + 16 * t, qboff);
        qb[4 * t] = x.v[0]; qb[4 * t + 1] = x.v[1]; qb[4 * t + 2] = x.v[2]; qb[4 * t + 3] = x.v[3];
      }
    };
    fetch_ge(c, g, e);
    if constexpr (NEEDG) fetch_qb(c);
    // one block; MORE: another whole block follows (a constant, so that no branch joins two
    // request histories and every wait counts exactly)
    auto step = [&](auto more_tag, const int c, Pk<4>* g, Pk<4>* e, Pk<4>* gn, Pk<4>* en) {
      constexpr bool more = decltype(more_tag)::value;
      {
        const char* base = reinterpret_cast<const char*>(Q + (size_t)c * RP);
#pragma unroll
        for (int kk = 0; kk < 16; ++kk) bq[kk] = *gptr<float>(base + kk * RP * 4 + bqoff);
      }
      if constexpr (more) fetch_ge(c + 256, gn, en);
      __builtin_amdgcn_sched_barrier(0);   // the requests above stay ahead of the arithmetic below
      if constexpr (NEEDG) {
        v16f gh;
#pragma unroll
        for (int i = 0; i < 16; ++i) gh[i] = 0.0f;
#pragma unroll
        for (int k = 0; k < KH; ++k) gh = __builtin_amdgcn_mfma_f32_32x32x2f32(pa[k], qb[k], gh, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (more) fetch_qb(c + 256);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int v = 0; v < 16; ++v) lds[(8 * (v >> 2) + 4 * h + (v & 3)) * kLP32 + li] = gh[v];
        wave_lds_fence();
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float4 t = *reinterpret_cast<const float4*>(lds + (8 * i + sr) * kLP32 + c4);
          e[i].v[0] -= t.x; e[i].v[1] -= t.y; e[i].v[2] -= t.z; e[i].v[3] -= t.w;
        }
        wave_lds_fence();
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int rr = 8 * i + sr;
        Pk<4> m, gv = g[i];
        if constexpr (GB16) gv = unpack_bf16(g[i].v[0], g[i].v[1]);
#pragma unroll
        for (int v = 0; v < 4; ++v) m.v[v] = gv.v[v] + e[i].v[v];
        strow<false>(reinterpret_cast<char*>(M + (size_t)(row0 + 8 * i) * cols + c), goff, m);
        *reinterpret_cast<float4*>(lds + rr * kLP32 + c4) = make_float4(m.v[0], m.v[1], m.v[2], m.v[3]);
      }
      wave_lds_fence();
      {
        const float4 a0 = *reinterpret_cast<const float4*>(lds + li * kLP32 + 16 * h);
        const float4 a1 = *reinterpret_cast<const float4*>(lds + li * kLP32 + 16 * h + 4);
        const float4 a2 = *reinterpret_cast<const float4*>(lds + li * kLP32 + 16 * h + 8);
        const float4 a3 = *reinterpret_cast<const float4*>(lds + li * kLP32 + 16 * h + 12);
        accP = __builtin_amdgcn_mfma_f32_32x32x2f32(a0.x, bq[0], accP, 0, 0, 0);
        accP2 = __builtin_amdgcn_mfma_f32_32x32x2f32(a1.x, bq[4], accP2, 0, 0, 0);
        accP = __builtin_amdgcn_mfma_f32_32x32x2f32(a0.y, bq[1], accP, 0, 0, 0);
        accP2 = __builtin_amdgcn_mfma_f32_32x32x2f32(a1.y, bq[5], accP2, 0, 0, 0);
        accP = __builtin_amdgcn_mfma_f32_32x32x2f32(a0.z, bq[2], accP, 0, 0, 0);
        accP2 = __builtin_amdgcn_mfma_f32_32x32x2f32(a1.z, bq[6], accP2, 0, 0, 0);
        accP = __builtin_amdgcn_mfma_f32_32x32x2f32(a0.w, bq[3], accP, 0, 0, 0);
        accP2 = __builtin_amdgcn_mfma_f32_32x32x2f32(a1.w, bq[7], accP2, 0, 0, 0);
        accP = __builtin_amdgcn_mfma_f32_32x32x2f32(a2.x, bq[8], accP, 0, 0, 0);
        accP2 = __builtin_amdgcn_mfma_f32_32x32x2f32(a3.x, bq[12], accP2, 0, 0, 0);
        accP = __builtin_amdgcn_mfma_f32_32x32x2f32(a2.y, bq[9], accP, 0, 0, 0);
        accP2 = __builtin_amdgcn_mfma_f32_32x32x2f32(a3.y, bq[13], accP2, 0, 0, 0);
        accP = __builtin_amdgcn_mfma_f32_32x32x2f32(a2.z, bq[10], accP, 0, 0, 0);
        accP2 = __builtin_amdgcn_mfma_f32_32x32x2f32(a3.z, bq[14], accP2, 0, 0, 0);
        accP = __builtin_amdgcn_mfma_f32_32x32x2f32(a2.w, bq[11], accP, 0, 0, 0);
        accP2 = __builtin_amdgcn_mfma_f32_32x32x2f32(a3.w, bq[15], accP2, 0, 0, 0);
      }
      wave_lds_fence();
    };
    // two blocks per trip, the two register sets changing roles (no copies, so nothing waits for
    // a prefetch before its values are needed)
    for (; c + 256 < last; c += 512) {
      step(std::true_type{}, c, g, e, gn, en);
      step(std::true_type{}, c + 256, gn, en, g, e);
    }
    if (c < last) {
      step(std::true_type{}, c, g, e, gn, en);
      step(std::false_type{}, c + 256, gn, en, g, e);
      c += 512;
    } else {
      step(std::false_type{}, c, g, e, gn, en);
      c += 256;
    }
  }
  for (; c < col1; c += 256) {
    Pk<4> g[4], e[4];
    fetch(c, g, e);
    block(c, g, e);
  }
  // P partial of the item = sum over the eight wavefronts, added in wavefront order
#pragma unroll
  for (int v = 0; v < 16; ++v) lds[(8 * (v >> 2) + 4 * h + (v & 3)) * kLP32 + li] = accP[v] + accP2[v];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int e = (int)threadIdx.x + 512 * i;
    const int rr = e >> 5, k = e & 31;
    float t = lds_all[0][rr * kLP32 + k];
#pragma unroll
    for (int wv = 1; wv < 8; ++wv) t += lds_all[wv][rr * kLP32 + k];
    if (rr < nrows && k < r) Pp[(size_t)(row0 + rr) * r + k] = t;
  }
}

template <int MODE, bool GB16>
__global__ __launch_bounds__(512, 2) void mfma_sweep32_kernel(DevArgs a, const Tile* __restrict__ tiles, int ntiles, int reverse) {
  __shared__ __attribute__((aligned(16))) float lds_all[8][32 * kLP32];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & (kWave - 1);
  if (blockIdx.x == 0) zero_absmax_cells(a, 512);
  const Tile tl = tiles[reverse ? ntiles - 1 - (int)blockIdx.x : (int)blockIdx.x];   // one item per workgroup
  const int layer = tl.lw / a.W, worker = tl.lw - layer * a.W;
  const LayerDesc& ld = a.layers[layer];
  const float* G = a.grads[(size_t)worker * a.n_all + ld.gidx];
  float* M = a.E + (size_t)worker * a.m_stride + ld.m_off;
  float* Pp = a.Ppart + (size_t)worker * a.ppart_stride + ld.ppart_off + (size_t)tl.aux * ld.np_pad;
  const int col0 = tl.aux * ld.segw;
  const int col1 = min(ld.cols, col0 + ld.segw);
  if (ld.kind == kOneColumnPerLane) {            // four of the item's rows per wavefront
    const int nr = min(4, tl.nrows - 4 * wave);
    if (nr > 0)
      narrow_rows<32, 4, true, MODE == kMAddFused, true, false, GB16>(G, M, q_operand(a, ld), p_operand(a, ld), Pp, nullptr,
                                                                      ld.cols, ld.r, tl.row0 + 4 * wave, nr, lane, 0, 0.0f);
    return;
  }
  mfma_tile32<MODE, GB16>(G, M, q_operand(a, ld), p_operand(a, ld), Pp, ld.cols, ld.r, tl.row0, tl.nrows,
                                   col0, col1, lane, wave, lds_all);
}

// Wavefronts per SIMD the register allocation aims for: two at rank pad 16, one from rank pad 32 on, where two would spill.
template <int RP, int MODE, bool GB16 = false, bool NTS = false>
__global__ __launch_bounds__(256, RP <= 16 ? 2 : 1) void mfma_sweep_kernel(DevArgs a, const Tile* __restrict__ tiles, int ntiles, int two, int reverse) {
  __shared__ __attribute__((aligned(16))) float lds_all[4][32 * kLP];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & (kWave - 1);
  if ((MODE == kMAdd || MODE == kMAddFused) && blockIdx.x == 0) zero_absmax_cells(a, 256);
  const int block = reverse ? ntiles + two - 1 - (int)blockIdx.x : (int)blockIdx.x;
  const HalfItem it = RP == 64 ? half_item(block, two) : HalfItem{block, 0};
  Tile tl = tiles[it.item];
  if constexpr (RP == 64) {
    tl.row0 += 32 * it.half;
    tl.nrows = min(32, tl.nrows - 32 * it.half);
  }
  const int layer = tl.lw / a.W, worker = tl.lw - layer * a.W;
  const LayerDesc& ld = a.layers[layer];
  const float* G = (MODE == kMAdd || MODE == kMAddFused) ? a.grads[(size_t)worker * a.n_all + ld.gidx] : nullptr;
  float* M = a.E + (size_t)worker * a.m_stride + ld.m_off;
  float* Pp = a.Ppart + (size_t)worker * a.ppart_stride + ld.ppart_off + (size_t)tl.aux * ld.np_pad;
  float* ghat_out = nullptr;
  if (MODE == kMResidualGhat && worker == 0 && a.ghat) ghat_out = a.ghat[ld.gidx];
  const int col0 = tl.aux * ld.segw;
  const int col1 = min(ld.cols, col0 + ld.segw);
  if (ld.kind == kOneColumnPerLane) {            // eight of the item's rows per wavefront
    constexpr bool ADD = MODE == kMAdd || MODE == kMAddFused;
    const int nr = min(8, tl.nrows - 8 * wave);
    if (nr > 0)
      narrow_rows<RP, 8, ADD, MODE == kMAddFused, true, MODE == kMResidualGhat, GB16>(
          G, M, q_operand(a, ld), p_operand(a, ld), Pp, ghat_out, ld.cols, ld.r, tl.row0 + 8 * wave, nr, lane, a.update, a.eta);
    return;
  }
  mfma_tile<RP, MODE, GB16, NTS>(G, M, q_operand(a, ld), p_operand(a, ld), Pp, ghat_out, ld.cols, ld.r, tl.row0,
                                 tl.nrows, col0, col1, lane, wave, lds_all, a.update, a.eta);
}

// ---------------------------------------------------------------------------
// The G-hat pass on the matrix cores: G-hat = P-bar Q-bar^T of one layer, or the
// parameters it updates.  One workgroup per block of rows x 256 columns; a
// wavefront keeps the rows of Q-bar of its 64 columns in registers and goes down
// the rows 32 at a time.  The 32 rows of P-bar come once, coalesced, through LDS
// for all four wavefronts, the next ones requested while these are multiplied.
// (Sweep 2's blocks, which this pass used to share, fetch 64 rows of Q-bar for
// every 32 x 64 of G-hat, 16 bytes of 64 rows at a time.)  The block leaves in
// the matrix cores' own layout, 128 bytes of two rows a store, non-temporal
// unless it is parameters that the next pass of the network reads (plain stores:
// ResNet-18 set, r = 50 24.6 us, r = 32 16.3).  The products are those of
// mfma_tile in the same order, so G-hat is what the other passes subtract, to
// the last bit.  Blocks of sweep 2 / this kernel, us: ResNet-18 set, r = 50
// 35.4 -> 22.3, r = 32 20.4 -> 14.2, r = 16 15.7 -> 12.4, ragged set, r = 20
// 13.2 -> 9.2, 2 x (208 x 2000), r = 41 19.7 -> 9.0, 8192^2, r = 64 139 -> 85,
// r = 32 67 -> 51.  Bound by the stores where items are many, else by the chain
// of one item: tile, layer, factors, products, stores.
// ---------------------------------------------------------------------------
template <int RP, bool UPDATE>
__global__ __launch_bounds__(256) void mfma_ghat_kernel(DevArgs a, const Tile* __restrict__ tiles) {
  constexpr int KH = RP / 2, PITCH = RP + 4, F4 = (8 * RP + 255) / 256;      // pitch: 16 rows' reads of 16 bytes hit all banks once
  __shared__ __attribute__((aligned(16))) float ps[2][32 * PITCH];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & (kWave - 1), tid = threadIdx.x;
  const Tile tl = tiles[blockIdx.x];
  const LayerDesc& ld = a.layers[tl.lw / a.W];
  float* out = a.ghat ? a.ghat[ld.gidx] : nullptr;
  if (!out) return;
  const float* Q = q_operand(a, ld);
  const float* Pb = p_operand(a, ld);
  const int cols = ld.cols;
  if (ld.kind == kOneColumnPerLane) {            // eight rows a wavefront at a time
    for (int i = 8 * wave; i < tl.nrows; i += 32)
      narrow_rows<RP, 8, false, false, false, true, false>(nullptr, nullptr, Q, Pb, nullptr, out, cols, ld.r, tl.row0 + i,
                                                           min(8, tl.nrows - i), lane, a.update, a.eta);
    return;
  }
  const int li = lane & 31, h = lane >> 5;
  const int c = tl.aux * kGhatCols + 64 * wave;
  // the block's rows of P-bar, 16 bytes a thread and request; the last one again where they end
  const char* src = reinterpret_cast<const char*>(Pb + (size_t)tl.row0 * RP);
  const int n4 = tl.nrows * (RP / 4);
  Pk<4> x[F4];
  auto request = [&](int t) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < F4; ++i) x[i] = ldrow<false>(src, (unsigned)min(t * 8 * RP + tid + 256 * i, n4 - 1) * 16u);
  };
  auto to_lds = [&](float* to) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < F4; ++i) {
      const int e = tid + 256 * i;
      if (8 * RP >= 256 || e < 8 * RP)
        *reinterpret_cast<float4*>(to + e / (RP / 4) * PITCH + e % (RP / 4) * 4) = make_float4(x[i].v[0], x[i].v[1], x[i].v[2], x[i].v[3]);
    }
  };
  request(0);
  float qb[2][KH];
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const int first = min(c, cols - 1), col = min(32 * b + li, cols - 1 - first);
#pragma unroll
    for (int t = 0; t < KH / 4; ++t) {
      const Pk<4> q = ldrow<false>(reinterpret_cast<const char*>(Q + (size_t)first * RP) + 16 * t, (unsigned)(col * RP + KH * h) * 4u);
#pragma unroll
      for (int v = 0; v < 4; ++v) qb[b][4 * t + v] = q.v[v];
    }
  }
  to_lds(ps[0]);
  __syncthreads();
  const int nt = (tl.nrows + 31) / 32;
  const bool small = cols < (1 << 26);           // byte offsets within 8 rows fit 32 bits
  unsigned lane_off = (unsigned)(4 * h * cols + li) * 4u;
  for (int t = 0; t < nt; ++t) {
    if (t + 1 < nt) request(t + 1);
    const int left = tl.nrows - 32 * t;
    float* o = out + (size_t)(tl.row0 + 32 * t) * cols + c;
    const bool whole = left >= 32 && c + 64 <= cols && small;
    if (c < cols) {
      float w[UPDATE ? 2 : 1][16];
      auto parameters = [&](auto whole_tag) __attribute__((always_inline)) {
#pragma unroll
        for (int v = 0; v < 16; ++v)
#pragma unroll
          for (int b = 0; b < 2; ++b) {
            const int row = 8 * (v >> 2) + (v & 3);
            if constexpr (decltype(whole_tag)::value) {
              w[b][v] = *gptr<const float>(reinterpret_cast<const char*>(o + (size_t)row * cols + 32 * b) + lane_off);
            } else {
              const size_t at = (size_t)min(row + 4 * h, left - 1) * cols + min(32 * b + li, cols - 1 - c);
              w[b][v] = o[at];
            }
          }
      };
      if constexpr (UPDATE) {
        if (whole) parameters(std::true_type{}); else parameters(std::false_type{});
      }
      float pa[KH];
#pragma unroll
      for (int k = 0; k < KH / 4; ++k) {
        const float4 p = *reinterpret_cast<const float4*>(ps[t & 1] + li * PITCH + KH * h + 4 * k);
        pa[4 * k] = p.x; pa[4 * k + 1] = p.y; pa[4 * k + 2] = p.z; pa[4 * k + 3] = p.w;
      }
      v16f gh[2];
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int i = 0; i < 16; ++i) gh[b][i] = 0.0f;
#pragma unroll
      for (int k = 0; k < KH; ++k)
#pragma unroll
        for (int b = 0; b < 2; ++b) gh[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(pa[k], qb[b][k], gh[b], 0, 0, 0);
      if constexpr (UPDATE) {
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
          for (int v = 0; v < 16; ++v) gh[b][v] = fmaf(-a.eta, gh[b][v], w[b][v]);
      }
      if (whole) {
#pragma unroll
        for (int v = 0; v < 16; ++v)
#pragma unroll
          for (int b = 0; b < 2; ++b) {
            char* at = reinterpret_cast<char*>(o + (size_t)(8 * (v >> 2) + (v & 3)) * cols + 32 * b);
            asm volatile("" : "+v"(lane_off));   // (one offset for all rows, not a 64-bit address for each)
            if constexpr (!UPDATE) __builtin_nontemporal_store(gh[b][v], gptr<float>(at + lane_off));
            else *gptr<float>(at + lane_off) = gh[b][v];
          }
      } else {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int row = 8 * (v >> 2) + 4 * h + (v & 3);
#pragma unroll
          for (int b = 0; b < 2; ++b)
            if (row < left && c + 32 * b + li < cols) o[(size_t)row * cols + 32 * b + li] = gh[b][v];
        }
      }
    }
    if (t + 1 < nt) {
      to_lds(ps[(t + 1) & 1]);
      __syncthreads();
    }
  }
}

// Copies of the aggregated factors with rows of RP ranks (zero beyond the layer's rank), as the sweeps
// read them.  blockIdx.y = layer; which: 0 = P-bar, 1 = Q-bar.
__global__ __launch_bounds__(256) void pad_factor_kernel(DevArgs a, int RP, int which) {
  const LayerDesc& ld = a.layers[blockIdx.y];
  const int n = which ? ld.cols : ld.rows, r = ld.r;
  const float* src = which ? a.Qbar + ld.q_off : a.Pbar + ld.p_off;
  float* dst = which ? a.Qop + ld.qop_off : a.Pop + ld.pop_off;
  const long long total = (long long)n * RP;
  for (long long e = blockIdx.x * 256 + threadIdx.x; e < total; e += gridDim.x * 256) {
    const long long row = e / RP;
    const int k = (int)(e - row * RP);
    dst[e] = k < r ? src[row * r + k] : 0.0f;
  }
}

// ---------------------------------------------------------------------------
// orth of tall factors at rank pads >= 8: Cholesky-QR, applied twice.
// The column-by-column form above pays one exchange between the slices of a
// factor per column (about 10 us each: r = 32 columns cost 0.33 ms on a factor
// of 8192 rows, where all the arithmetic is a few microseconds).  Here the
// slices exchange the r x r Gram matrix G = P^T P once per pass instead:
//   G = R^T R (Cholesky),  P <- P R^-1.
// In exact arithmetic R is the triangular factor of the QR decomposition of P,
// so P R^-1 is what Gram-Schmidt (Algorithm 1's Orthogonalize) returns; in
// float32 one pass loses orthogonality in proportion to cond(P)^2, and a second
// pass on its result restores it to rounding level (the usual "CholeskyQR2").
// That only holds while cond(P)^2 stays well below 1/epsilon: if a pivot of
// either factorisation falls below kCholPivotFloor of its column's squared
// norm (or a column is zero), the pair is done again from the start by the
// column-by-column form, whose result does not depend on conditioning in that
// way.  Every slice of a pair factorises the same total, so all take the same
// decision.
// Steps of a pass, per workgroup (= 256 rows, one per thread, in registers):
//   * the slice's Gram matrix on the matrix cores (rows are re-read from the
//     plane this workgroup has just written, in "lane = column" layout), the
//     four wavefronts' parts added in wavefront order;
//   * exchange: entry e of the total is owned by slice e / ceil(NE / nslice),
//     which collects that entry from every slice, adds them up in slice order
//     and publishes the total; every slice then collects all totals.  Entries
//     are tagged 64-bit words as in orth_coop_kernel: two round trips per pass
//     instead of one per column, and no workgroup reads more than 2 NE words;
//   * wavefront 0 factorises (lane l keeps row l of G in registers; right-
//     looking elimination with lane broadcasts), every thread then applies
//     R^-1 to its row by forward substitution, reading R from LDS.
// phase -1 runs all of it in one cooperative launch.  Without one, phases 0, 1
// and 2 are three ordinary launches that pass the slices' Gram matrices through
// plain memory and add them up in the same order, so that both forms
// give the same bits; pairs that need the column-by-column form raise redo[pair]
// and the guarded orth_wide_kernel launches that follow do them.  A launch reads the
// matrices of one plane (parts_in, all slices of the pair) and writes its own slice's to
// another (parts_out): the workgroups of a launch have no order, and slices beyond what the
// chip holds start after others have ended, so that a matrix of the second pass must not
// lie where a slice may still have to read the first pass's.
// ---------------------------------------------------------------------------
// On the CPU, in float32, two passes stay as close to the float64 Gram-Schmidt as float32 Gram-Schmidt
// itself down to pivot ratios of about 1e-6 (both 1e-6 .. 1e-5 away at ratios 2e-4 .. 1e-5); the floor
// keeps two orders of magnitude from where the factorisation starts to break down.
constexpr float kCholPivotFloor = 1e-4f;

template <int RP>
struct CholShape {
  static_assert(RP == 8 || RP == 16 || RP == 32 || RP == 64, "rank pads with a Cholesky-QR form");
  static constexpr int NB = RP <= 32 ? 1 : 3;                       // 32 x 32 blocks kept: (0,0) or (0,0), (0,1), (1,1)
  static constexpr int NE = RP <= 32 ? RP * RP : 3 * 1024;          // entries exchanged
  static constexpr int QN = (NE + 255) / 256;                       // ... per thread
  static constexpr int GN = (NE + kCoopMaxSlices + 255) / 256;      // entries a thread collects as an owner
  static constexpr int kPoolA = 4 * NE, kPoolB = (kCoopMaxSlices + 5) * RP;
  static constexpr int POOL = kPoolA > kPoolB ? kPoolA : kPoolB;    // LDS floats
};

// Where <column i, column j>, i <= j, sits among the exchanged entries.
template <int RP>
__device__ __forceinline__ int chol_entry(int i, int j) {
  if constexpr (RP <= 32) {
    return i * RP + j;
  } else {
    return j < 32 ? i * 32 + j : (i < 32 ? 1024 + i * 32 + (j - 32) : 2048 + (i - 32) * 32 + (j - 32));
  }
}

// The Gram matrix of the slice's 256 rows of `orth`: on return thread t holds entries t, t + 256, ...
// in gsum.  pool: 4 NE floats of LDS, free again on return.
template <int RP>
__device__ __forceinline__ void chol_slice_gram(const float* orth, int rows, int r, int row0, float* pool,
                                                float (&gsum)[CholShape<RP>::QN]) {
  using S = CholShape<RP>;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
  const int li = lane & 31, h = lane >> 5;
  v16f acc[S::NB];
#pragma unroll
  for (int b = 0; b < S::NB; ++b)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[b][i] = 0.0f;
  constexpr int U = 16;                           // row pairs loaded ahead of their matrix instructions
  const int c0 = min(li, r - 1), c1 = min(32 + li, r - 1);
  const bool ok0 = li < r, ok1 = 32 + li < r;
#pragma unroll 1
  for (int b = 0; b < 32 / U; ++b) {
    float x0[U], x1[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int row = row0 + wave * 64 + 2 * (b * U + u) + h;
      const float* src = orth + (size_t)min(row, rows - 1) * r;      // every load is in bounds; masked below
      x0[u] = keep_if(src[c0], ok0 && row < rows);
      if constexpr (RP == 64) x1[u] = keep_if(src[c1], ok1 && row < rows);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(x0[u], x0[u], acc[0], 0, 0, 0);
      if constexpr (RP == 64) {
        acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(x0[u], x1[u], acc[1], 0, 0, 0);
        acc[2] = __builtin_amdgcn_mfma_f32_32x32x2f32(x1[u], x1[u], acc[2], 0, 0, 0);
      }
    }
  }
  // D layout: register v of lane (li, h) is element (8 (v / 4) + 4 h + v % 4, li) of the block
  float* mine = pool + wave * S::NE;
#pragma unroll
  for (int b = 0; b < S::NB; ++b)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int m = 8 * (v >> 2) + 4 * h + (v & 3);
      if constexpr (RP <= 32) {
        if (m < RP && li < RP) mine[m * RP + li] = acc[b][v];
      } else {
        mine[b * 1024 + m * 32 + li] = acc[b][v];
      }
    }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < S::QN; ++q) {
    const int e = tid + 256 * q;
    gsum[q] = (e < S::NE) ? (pool[e] + pool[S::NE + e]) + (pool[2 * S::NE + e] + pool[3 * S::NE + e]) : 0.0f;
  }
  __syncthreads();
}

__device__ __forceinline__ unsigned long long table_wait(const unsigned long long* p, unsigned long long x, unsigned tag,
                                                         int* status, unsigned max_polls) {
  unsigned polls = 0;
  while ((unsigned)(x >> 32) != tag) {
    if (++polls >= max_polls) {
      __hip_atomic_store(status, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
      break;
    }
    __builtin_amdgcn_s_sleep(1);
    x = table_load(p);
  }
  return x;
}

// The slices' Gram matrices -> their total, in LDS at pool + 2 NE, through the tagged table
// `tab` ([nslice_max + 1][NE]: one plane per slice, the totals in the last one).
template <int RP>
__device__ __forceinline__ void chol_exchange(const float (&gsum)[CholShape<RP>::QN], unsigned long long* tab, int slice,
                                              int nslice, int nslice_max, unsigned tag_part, unsigned tag_total, float* pool,
                                              int* status, unsigned max_polls) {
  using S = CholShape<RP>;
  const int tid = threadIdx.x;
#pragma unroll
  for (int q = 0; q < S::QN; ++q) {
    const int e = tid + 256 * q;
    if (e < S::NE)
      __hip_atomic_store(tab + (size_t)slice * S::NE + e, ((unsigned long long)tag_part << 32) | __float_as_uint(gsum[q]),
                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  // the entries this slice owns, from every slice: item = (entry, slice)
  const int share = (S::NE + nslice - 1) / nslice;
  const int e0 = slice * share;
  const int cnt = max(0, min(S::NE - e0, share));
  const int nitem = cnt * nslice;                  // <= NE + nslice
  unsigned long long x[S::GN];
  const unsigned long long* src[S::GN];
#pragma unroll
  for (int i = 0; i < S::GN; ++i) {
    const int it = tid + 256 * i;
    const int el = it / nslice, sl = it - el * nslice;
    src[i] = tab + (size_t)sl * S::NE + e0 + el;
    x[i] = (it < nitem) ? table_load(src[i]) : ((unsigned long long)tag_part << 32);
  }
#pragma unroll
  for (int i = 0; i < S::GN; ++i) {
    const int it = tid + 256 * i;
    if (it < nitem) {
      x[i] = table_wait(src[i], x[i], tag_part, status, max_polls);
      pool[it] = __uint_as_float((unsigned)x[i]);
    }
  }
  __syncthreads();
  unsigned long long* totals = tab + (size_t)nslice_max * S::NE;
  for (int el = tid; el < cnt; el += 256) {
    float t = 0.0f;
    for (int sl = 0; sl < nslice; ++sl) t += pool[el * nslice + sl];
    __hip_atomic_store(totals + e0 + el, ((unsigned long long)tag_total << 32) | __float_as_uint(t), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
  }
  unsigned long long y[S::QN];
#pragma unroll
  for (int q = 0; q < S::QN; ++q) {
    const int e = tid + 256 * q;
    y[q] = (e < S::NE) ? table_load(totals + e) : ((unsigned long long)tag_total << 32);
  }
#pragma unroll
  for (int q = 0; q < S::QN; ++q) {
    const int e = tid + 256 * q;
    if (e < S::NE) {
      y[q] = table_wait(totals + e, y[q], tag_total, status, max_polls);
      pool[2 * S::NE + e] = __uint_as_float((unsigned)y[q]);
    }
  }
  __syncthreads();
}

// The same total from the slices' matrices in plain memory (written by an earlier launch).
template <int RP>
__device__ __forceinline__ void chol_sum_parts(const float* parts, int nslice, float* pool) {
  using S = CholShape<RP>;
  const int tid = threadIdx.x;
#pragma unroll
  for (int q = 0; q < S::QN; ++q) {
    const int e = tid + 256 * q;
    if (e < S::NE) {
      float t = 0.0f;
      for (int sl = 0; sl < nslice; ++sl) t += parts[(size_t)sl * S::NE + e];
      pool[2 * S::NE + e] = t;
    }
  }
  __syncthreads();
}

__device__ __forceinline__ float lane_value(float x, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), l));
}

// One wavefront: G (total, at T) = L L^T.  Lane l works on row l.  Leaves L at Ls ([RP][RP], row
// major, lower triangle; the diagonal holds 1 / L_jj; rows and columns >= r are those of the
// identity) and returns whether every pivot stayed above the floor -- the same in every lane.
template <int RP>
__device__ __forceinline__ bool chol_factor(const float* T, float* Ls, int r, int lane) {
  const int l = min(lane, RP - 1);
  float g[RP];
#pragma unroll
  for (int k = 0; k < RP; ++k) g[k] = T[chol_entry<RP>(min(k, l), max(k, l))];
  float diag0 = 0.0f;
#pragma unroll
  for (int k = 0; k < RP; ++k)
    if (k == l) diag0 = g[k];
  bool ok = true;
  static_for<RP>([&](auto J) {
    constexpr int j = decltype(J)::value;
    if (j < r) {
      const float d = lane_value(g[j], j), d0 = lane_value(diag0, j);
      ok = ok && (d0 > FLT_MIN) && (d > kCholPivotFloor * d0);        // false for NaN as well
      const float rinv = 1.0f / sqrtf(d);
      const float lj = (lane >= j) ? g[j] * rinv : 0.0f;               // column j of L
#pragma unroll
      for (int k = j + 1; k < RP; ++k) g[k] = fmaf(-lj, lane_value(lj, k), g[k]);
      g[j] = (lane == j) ? rinv : lj;
    } else {
      g[j] = (lane == j) ? 1.0f : 0.0f;
    }
  });
  if (lane < RP) {
#pragma unroll
    for (int k = 0; k < RP; ++k) Ls[lane * RP + k] = g[k];
  }
  return ok;
}

// p <- p R^-1 with R = L^T: forward substitution along the row.
template <int RP>
__device__ __forceinline__ void chol_solve_row(float (&p)[RP], const float* Ls, int r) {
  static_for<RP>([&](auto J) {
    constexpr int j = decltype(J)::value;
    if (j < r) {                                   // p[j] is zero beyond the rank and stays so
      float acc = p[j];
#pragma unroll
      for (int i = 0; i < j; ++i) acc = fmaf(-p[i], Ls[j * RP + i], acc);
      p[j] = acc * Ls[j * RP + j];
    }
  });
}

// The slice's block of P_w = the sum of the sweep-0 planes, written to `pre` and `orth`.  The block is
// one contiguous run of nflt floats in every plane and in both outputs, so the threads walk it in
// 16-byte pieces, fully coalesced (a thread per row would touch 64 cache lines per load).
template <int RP>
__device__ __forceinline__ void chol_sum_planes(const float* planes, int nseg, size_t plane_stride, float* pre_s, float* orth_s,
                                                int nflt) {
  const int tid = threadIdx.x;
  const bool vec = (((reinterpret_cast<uintptr_t>(planes) | reinterpret_cast<uintptr_t>(pre_s) |
                      reinterpret_cast<uintptr_t>(orth_s)) & 15) == 0) && (plane_stride & 3) == 0;
  if (vec) {
    constexpr int NI = RP / 4;
    float4 acc[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i) acc[i] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    for (int sg = 0; sg < nseg; ++sg) {
      const float* src = planes + (size_t)sg * plane_stride;
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const int f = 4 * (tid + 256 * i);
        if (f + 4 <= nflt) {
          const float4 t = *reinterpret_cast<const float4*>(src + f);
          acc[i].x += t.x; acc[i].y += t.y; acc[i].z += t.z; acc[i].w += t.w;
        }
      }
    }
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int f = 4 * (tid + 256 * i);
      if (f + 4 <= nflt) {
        *reinterpret_cast<float4*>(pre_s + f) = acc[i];
        *reinterpret_cast<float4*>(orth_s + f) = acc[i];
      }
    }
    const int f = (nflt & ~3) + tid;               // what is left of a block whose length is no multiple of 4
    if (tid < (nflt & 3)) {
      float t = 0.0f;
      for (int sg = 0; sg < nseg; ++sg) t += planes[(size_t)sg * plane_stride + f];
      pre_s[f] = t;
      orth_s[f] = t;
    }
  } else {
    float acc[RP];
#pragma unroll
    for (int i = 0; i < RP; ++i) acc[i] = 0.0f;
    for (int sg = 0; sg < nseg; ++sg) {
      const float* src = planes + (size_t)sg * plane_stride;
#pragma unroll
      for (int i = 0; i < RP; ++i) {
        const int f = tid + 256 * i;
        if (f < nflt) acc[i] += src[f];
      }
    }
#pragma unroll
    for (int i = 0; i < RP; ++i) {
      const int f = tid + 256 * i;
      if (f < nflt) {
        pre_s[f] = acc[i];
        orth_s[f] = acc[i];
      }
    }
  }
}

// Row `row` of a rows x r factor (zero beyond r and for a thread without a row): loads of RP values that may
// run into what follows the row (kFactorSlack).
template <int RP>
__device__ __forceinline__ void chol_load_row(const float* F, int row, int rows, int r, float (&v)[RP]) {
  load_row<RP>(F, min(row, rows - 1), r, r == RP, v);
  const bool live = row < rows;
#pragma unroll
  for (int k = 0; k < RP; ++k) v[k] = keep_if(v[k], live);
}

template <int RP>
__device__ __forceinline__ void chol_store_row(float* F, int row, int rows, int r, const float (&v)[RP]) {
  if (row >= rows) return;
  if (r == RP) {
    float* b = F + (size_t)row * RP;
#pragma unroll
    for (int k = 0; k < RP; k += 4) *reinterpret_cast<float4*>(b + k) = make_float4(v[k], v[k + 1], v[k + 2], v[k + 3]);
  } else if ((r & 1) == 0) {
    float* b = F + (size_t)row * r;
#pragma unroll
    for (int k = 0; k < RP; k += 2)
      if (k < r) *reinterpret_cast<float2*>(b + k) = make_float2(v[k], v[k + 1]);
  } else {
    float* b = F + (size_t)row * r;
#pragma unroll
    for (int k = 0; k < RP; ++k)
      if (k < r) b[k] = v[k];
  }
}

template <int RP>
__global__ __launch_bounds__(256, 2) void orth_chol_kernel(DevArgs a, int nslice_max, int max_rank, int phase,
                                                        unsigned long long* ctable, const float* parts_in, float* parts_out, int* redo,
                                                        unsigned long long epoch, unsigned max_polls) {
  using S = CholShape<RP>;
  __shared__ __attribute__((aligned(16))) float pool[S::POOL];
  __shared__ float redmax[4];
  __shared__ int flag;
  int lw, slice;
  slice_of(a, blockIdx.x, nslice_max, lw, slice);
  const int layer = lw / a.W, worker = lw - layer * a.W;
  const LayerDesc& ld = a.layers[layer];
  const int rows = ld.rows, r = ld.r;
  const int nslice = (rows + 255) >> 8;
  if (phase == 2 && (redo[lw] & 1)) return;       // raised in phase 1, or by a faster slice just now: the pair is done again anyway
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
  const int row = slice * 256 + tid;
  float* pre = a.Ppre + (size_t)worker * a.p_stride + ld.p_off;
  float* orth = a.Porth + (size_t)worker * a.p_stride + ld.p_off;
  float* scale = a.scaleP + (size_t)worker * a.L + layer;
  unsigned long long* tab = ctable + (size_t)lw * (nslice_max + 1) * S::NE;
  const size_t parts = (size_t)lw * nslice_max * S::NE;
  float* Ls = pool;                              // [RP][RP], once the total has been read out of pool + 2 NE
  float v[RP];
#pragma unroll
  for (int k = 0; k < RP; ++k) v[k] = 0.0f;
  if (phase <= 0) {
    if (slice == 0 && tid == 0) {
      if (phase == 0) {
        redo[lw] = 0;
        if (!a.orth_shared) *scale = 0.0f;
      } else if (!a.orth_shared) {
        // shared by all slices, raised with atomics at the end; every slice reads an entry that
        // slice 0 publishes after this store before it gets there
        __hip_atomic_store(scale, 0.0f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __builtin_amdgcn_s_waitcnt(0x0F70);      // vmcnt(0)
      }
    }
    {
      const float* Pp = a.Ppart + (size_t)worker * a.ppart_stride + (a.orth_shared ? ld.p_off : ld.ppart_off);
      const size_t base = (size_t)slice * 256 * r;
      chol_sum_planes<RP>(Pp + base, a.orth_shared ? 1 : ld.nseg, (size_t)ld.np_pad, pre + base, orth + base,
                          min(256, rows - slice * 256) * r);
    }
  }
  float gsum[S::QN];
  bool good = true;
  if (phase == 0) {
    __syncthreads();                             // the rows above, for the loads in "lane = column" layout
    chol_slice_gram<RP>(orth, rows, r, slice * 256, pool, gsum);
  } else {
    const int first = phase < 0 ? 0 : phase - 1, last = phase < 0 ? 1 : phase - 1;
    for (int pass = first; pass <= last; ++pass) {
      if (phase < 0) {
        __syncthreads();
        chol_slice_gram<RP>(orth, rows, r, slice * 256, pool, gsum);
        const unsigned tag = (unsigned)(epoch * 4ull) + 2u * (unsigned)pass;
        chol_exchange<RP>(gsum, tab, slice, nslice, nslice_max, tag + 1u, tag + 2u, pool, a.status, max_polls);
      } else {
        chol_sum_parts<RP>(parts_in + parts, nslice, pool);
      }
      if (wave == 0) {
        const bool ok = chol_factor<RP>(pool + 2 * S::NE, Ls, r, lane);
        if (lane == 0) flag = ok ? 1 : 0;
      }
      __syncthreads();
      good = flag != 0;
      if (!good) break;
      // the thread's row as the previous step left it in memory (not kept in registers across the
      // factorisation, which needs them)
      chol_load_row<RP>(orth, row, rows, r, v);
      chol_solve_row<RP>(v, Ls, r);
      chol_store_row<RP>(orth, row, rows, r, v);
      __syncthreads();                           // Ls and flag are written again by the next pass
    }
    if (phase == 1 && good) chol_slice_gram<RP>(orth, rows, r, slice * 256, pool, gsum);
  }
  if (phase == 0 || (phase == 1 && good)) {
#pragma unroll
    for (int q = 0; q < S::QN; ++q) {
      const int e = tid + 256 * q;
      if (e < S::NE) parts_out[parts + (size_t)slice * S::NE + e] = gsum[q];
    }
    return;
  }
  if (!good) {
    if (phase > 0) {
      if (slice == 0 && tid == 0) {
        atomicOr(redo + lw, 1);
        atomicOr(redo, 2);                       // some pair
      }
      return;
    }
    // one launch: column by column from the sum of the planes, as orth_coop_kernel does
    chol_load_row<RP>(pre, row, rows, r, v);
    const size_t pstride = (size_t)a.L * a.W * nslice_max * RP;
    coop_columns<RP>(v, r, lw, slice, nslice, nslice_max, max_rank, a.orth_table, epoch, a.status, max_polls, pstride,
                     pool + kCoopMaxSlices * RP, pool + (kCoopMaxSlices + 4) * RP, pool);
    chol_store_row<RP>(orth, row, rows, r, v);
  }
  float mx = 0.0f;
#pragma unroll
  for (int k = 0; k < RP; ++k)
    if (k < r) mx = fmaxf(mx, fabsf(v[k]));
  mx = wave_max(mx);
  if (lane == 0) redmax[wave] = mx;
  __syncthreads();
  if (tid == 0 && !a.orth_shared) {
    const float m = fmaxf(fmaxf(redmax[0], redmax[1]), fmaxf(redmax[2], redmax[3]));
    atomicMax(reinterpret_cast<unsigned int*>(scale), __float_as_uint(m));
  }
}

}  // namespace

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
// Every launcher notes the device function it has just launched, template arguments included, in
// the form a profiler's kernel list shows it (without namespaces and parameter list), so that a
// timing slot of the API can be matched to a profile.
__attribute__((format(printf, 1, 2))) void note_kernel(const char* fmt, ...);
#if LQSGD_HAS(0)
static thread_local char g_launched[96] = "";
void note_kernel(const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  std::vsnprintf(g_launched, sizeof g_launched, fmt, ap);
  va_end(ap);
}
const char* last_launched_kernel() { return g_launched; }
#endif
static inline const char* tf(bool b) { return b ? "true" : "false"; }

// Rank pads of the vector sweeps: up to 8 (sweep 1: up to 16); higher ones run on the matrix cores.
#define LQSGD_RP_SWITCH8(RPV, CALL)           \
  switch (RPV) {                              \
    case 1: { constexpr int RP = 1; CALL; } break;   \
    case 2: { constexpr int RP = 2; CALL; } break;   \
    case 4: { constexpr int RP = 4; CALL; } break;   \
    case 8: { constexpr int RP = 8; CALL; } break;   \
    default: return hipErrorInvalidValue;     \
  }
#define LQSGD_RP_SWITCH16(RPV, CALL)                    \
  if ((RPV) == 16) { constexpr int RP = 16; CALL; } else \
    LQSGD_RP_SWITCH8(RPV, CALL)

#define LQSGD_RP_SWITCH(RPV, CALL)            \
  switch (RPV) {                              \
    case 1: { constexpr int RP = 1; CALL; } break;   \
    case 2: { constexpr int RP = 2; CALL; } break;   \
    case 4: { constexpr int RP = 4; CALL; } break;   \
    case 8: { constexpr int RP = 8; CALL; } break;   \
    case 16: { constexpr int RP = 16; CALL; } break; \
    case 32: { constexpr int RP = 32; CALL; } break; \
    default: return hipErrorInvalidValue;     \
  }

// The Gram-Schmidt kernels also exist at rank pad 64 (the streaming sweeps run on the matrix cores there).
#define LQSGD_RP_SWITCH_ORTH(RPV, CALL)                 \
  if ((RPV) == 64) { constexpr int RP = 64; CALL; } else \
    LQSGD_RP_SWITCH(RPV, CALL)

#if LQSGD_HAS(1)
hipError_t launch_add_project(int rp, const DevArgs& a, const Tile* tiles, int ntiles, int fuse_residual, int narrow_rows,
                              int reverse, hipStream_t s) {
  if (ntiles <= 0) return hipSuccess;
  const dim3 grid((ntiles + 3) / 4), block(256);
  const unsigned lds = narrow_rows ? 0 : kTwoPerCu;
#define LQSGD_LAUNCH_A(FUSE, GB) \
  if (a.nt_store) { LQSGD_RP_SWITCH8(rp, (add_project_kernel<RP, FUSE, GB, true><<<grid, block, lds, s>>>(a, tiles, ntiles, reverse))); } \
  else { LQSGD_RP_SWITCH8(rp, (add_project_kernel<RP, FUSE, GB, false><<<grid, block, lds, s>>>(a, tiles, ntiles, reverse))); }
  if (a.g_bf16) {
    if (fuse_residual) { LQSGD_LAUNCH_A(true, true) } else { LQSGD_LAUNCH_A(false, true) }
  } else if (fuse_residual) {
    LQSGD_LAUNCH_A(true, false)
  } else {
    LQSGD_LAUNCH_A(false, false)
  }
#undef LQSGD_LAUNCH_A
  note_kernel("add_project_kernel<%d, %s, %s, %s>", rp, tf(fuse_residual), tf(a.g_bf16), tf(a.nt_store));
  return hipGetLastError();
}
#endif

#if LQSGD_HAS(4)
// Rows on lanes, rank pads 1 and 2.
template <int RP>
bool launch_orth_reg(const DevArgs& a, int max_rows, dim3 grid, hipStream_t s) {
#define LQSGD_LAUNCH_OR(RPT, BS)                                  \
  if (max_rows <= (RPT) * (BS)) {                                 \
    orth_reg_kernel<RP, RPT, BS><<<grid, dim3(BS), 0, s>>>(a);    \
    note_kernel("orth_reg_kernel<%d, %d, %d>", RP, RPT, BS);      \
    return true;                                                  \
  }
  LQSGD_LAUNCH_OR(2, 256)
  LQSGD_LAUNCH_OR(8, 256)
  LQSGD_LAUNCH_OR(4, 1024)
  LQSGD_LAUNCH_OR(11, 1024)
#undef LQSGD_LAUNCH_OR
  return false;
}

// One workgroup each with the sums of slices, rank pads 1 to 4.
template <int RP>
bool launch_orth_tall(const DevArgs& a, int max_rows, dim3 grid, hipStream_t s) {
#define LQSGD_LAUNCH_OT(RPT)                                      \
  if (max_rows <= (RPT) * 1024) {                                 \
    orth_tall_kernel<RP, RPT><<<grid, dim3(1024), 0, s>>>(a);     \
    note_kernel("orth_tall_kernel<%d, %d>", RP, RPT);             \
    return true;                                                  \
  }
  if constexpr (RP > 1) { LQSGD_LAUNCH_OT(2) }
  LQSGD_LAUNCH_OT(4)
  LQSGD_LAUNCH_OT(8)
  if constexpr (RP == 4) { LQSGD_LAUNCH_OT(11) }
  else { LQSGD_LAUNCH_OT(12) }
#undef LQSGD_LAUNCH_OT
  return false;
}

// Whole columns to a wavefront (OW) or columns on lanes (OC); the sums are those of 256 threads with rows on lanes (1024
// threads beyond 2048 rows), their wavefronts added in pairs from rank pad 16 and 513 rows on.
template <int C>
bool launch_orth_col(const DevArgs& a, int max_rows, dim3 grid, hipStream_t s) {
#define LQSGD_LAUNCH_OC(ROWS, WV, NI, NW)                                                            \
  if (max_rows <= (ROWS)) {                                                                          \
    static_assert((ROWS) <= ((WV) > 4 ? 64 * (WV) : (NI) > 1 ? 256 : 64 * (WV)) * (NI), "");         \
    orth_col_kernel<C, WV, NI, NW><<<grid, dim3(64 * (NW)), 0, s>>>(a);                              \
    note_kernel("orth_col_kernel<%d, %d, %d, %d>", C, WV, NI, NW);                                   \
    return true;                                                                                     \
  }
#define LQSGD_LAUNCH_OW(ROWS, NB, NI, NW, BC, NIC, SLOTS, PAIRS)                                                \
  if (max_rows <= (ROWS)) {                                                                                     \
    static_assert((ROWS) == 64 * (NB) * (NI), "");                                                              \
    orth_colwave_kernel<C, NB, NI, NW, BC, NIC, SLOTS, PAIRS><<<grid, dim3(64 * (NW)), 0, s>>>(a);              \
    note_kernel("orth_colwave_kernel<%d, %d, %d, %d, %d, %d, %d, %s>", C, NB, NI, NW, BC, NIC, SLOTS, tf(PAIRS)); \
    return true;                                                                                                \
  }
  // More factors than CUs: what counts is the work of a factor, not its chain (640 of them, one wavefront a column or block / as
  // chosen: 512 rows at r = 16 27 / 24 us, 120 rows 18 / 14; 60 rows at r = 40 41 / 37; 64 rows at r = 30 28 / 23.5.  168 of them at
  // r = 16 14.1 / 15.1).
  const bool many = grid.x > kCus;
  if constexpr (C == 4) {
    LQSGD_LAUNCH_OW(512, 4, 2, 4, 1, 2, 4, false)        // (500 rows 8.6 -> 8.3 us, but 1000 rows 8.1 -> 9.0, 1700 9.7 -> 12.4)
    LQSGD_LAUNCH_OC(1024, 4, 4, 8)
    LQSGD_LAUNCH_OC(2048, 4, 8, 8)
    LQSGD_LAUNCH_OC(4096, 16, 4, 16)
    LQSGD_LAUNCH_OC(8192, 16, 8, 16)
    LQSGD_LAUNCH_OC(11264, 16, 11, 16)
  } else if constexpr (C == 8) {
    LQSGD_LAUNCH_OW(256, 4, 1, 8, 1, 1, 8, false)
    LQSGD_LAUNCH_OW(512, 4, 2, 8, 1, 2, 8, false)
    LQSGD_LAUNCH_OW(1024, 4, 4, 8, 1, 4, 8, false)
    LQSGD_LAUNCH_OW(2048, 4, 8, 8, 1, 4, 8, false)
    LQSGD_LAUNCH_OC(4096, 16, 4, 16)
  } else if constexpr (C == 16) {
    if (!many) {
      LQSGD_LAUNCH_OW(128, 2, 1, 16, 1, 1, 16, false)
      LQSGD_LAUNCH_OW(256, 4, 1, 16, 1, 1, 16, false)
      LQSGD_LAUNCH_OW(512, 4, 2, 16, 1, 2, 16, false)
      LQSGD_LAUNCH_OW(1024, 4, 4, 16, 1, 2, 16, true)
      LQSGD_LAUNCH_OW(1792, 4, 7, 16, 1, 7, 16, true)
    }
    LQSGD_LAUNCH_OW(128, 2, 1, 8, 2, 1, 16, false)
    LQSGD_LAUNCH_OW(256, 4, 1, 8, 2, 1, 16, false)
    LQSGD_LAUNCH_OW(512, 4, 2, 8, 2, 2, 16, false)
    LQSGD_LAUNCH_OW(1024, 4, 4, 8, 2, 2, 16, true)
    LQSGD_LAUNCH_OW(1792, 4, 7, 8, 2, 7, 16, true)
  } else if constexpr (C == 32) {
    if (many) { LQSGD_LAUNCH_OC(64, 1, 1, 4) }
    LQSGD_LAUNCH_OW(64, 1, 1, 16, 2, 1, 32, false)
    LQSGD_LAUNCH_OW(128, 2, 1, 16, 2, 1, 32, false)
    LQSGD_LAUNCH_OW(256, 4, 1, 16, 2, 1, 32, false)
    LQSGD_LAUNCH_OW(512, 4, 2, 16, 2, 2, 32, false)
    LQSGD_LAUNCH_OW(1024, 4, 4, 16, 2, 2, 32, true)
    LQSGD_LAUNCH_OW(1792, 4, 7, 16, 2, 1, 16, true)
  } else {
    if (many) { LQSGD_LAUNCH_OW(64, 1, 1, 8, 2, 1, 64, false) }
    LQSGD_LAUNCH_OW(64, 1, 1, 16, 2, 1, 64, false)
    LQSGD_LAUNCH_OW(128, 2, 1, 16, 2, 1, 64, false)
    LQSGD_LAUNCH_OW(256, 4, 1, 16, 2, 1, 64, false)
    LQSGD_LAUNCH_OW(512, 4, 2, 16, 2, 2, 64, false)
    LQSGD_LAUNCH_OW(1024, 4, 4, 16, 2, 2, 32, true)
  }
#undef LQSGD_LAUNCH_OC
#undef LQSGD_LAUNCH_OW
  return false;
}

// One cooperative launch if every workgroup of the grid can be resident at once; returns false
// (nothing launched) otherwise, and the caller takes the one-launch-per-column path.
template <int RP>
bool try_orth_coop(int nslice, int max_rank, const DevArgs& a, int nblocks, CoopState* cs, hipStream_t s) {
  if (cs->capacity < 0) {                        // resident workgroups of this kernel on the context's device
    int dev = 0, coop = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, orth_coop_kernel<RP>, 256, 0) != hipSuccess) {
      (void)hipGetLastError();
      cs->capacity = 0;
    } else {
      cs->capacity = coop ? cus * per_cu : 0;
    }
  }
  if (nblocks > cs->capacity) return false;
  DevArgs args = a;
  unsigned long long* table = a.orth_table;
  unsigned long long n = cs->epoch;
  int* status = a.status;
  unsigned max_polls = cs->max_polls ? cs->max_polls : kTablePolls;
  void* params[] = {&args, &nslice, &max_rank, &table, &n, &status, &max_polls};
  const hipError_t e = hipLaunchCooperativeKernel(reinterpret_cast<void*>(orth_coop_kernel<RP>), dim3(nblocks), dim3(256),
                                                  params, 0, s);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  cs->epoch += 1;                                // the tags of a launch are epoch * max_rank + 1 ... + max_rank
  note_kernel("orth_coop_kernel<%d>", RP);
  return true;
}

bool launch_orth_coop(int rp, int nslice, int max_rank, const DevArgs& a, int nblocks, CoopState* cs, hipStream_t s) {
#ifdef LQSGD_TUNING
  static const bool enabled = [] { const char* e = std::getenv("LQSGD_ORTH_COOP"); return !(e && e[0] == '0'); }();
  if (!enabled) return false;
#endif
  if (!cs || !a.orth_table || !a.status || nslice > kCoopMaxSlices) return false;
  // Under stream capture the launch would be replayed with this launch's epoch baked in, and the
  // tags of one replay would be indistinguishable from the next one's: take the per-column path.
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &cap) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  if (cap != hipStreamCaptureStatusNone) return false;
  switch (rp) {
    case 1: return try_orth_coop<1>(nslice, max_rank, a, nblocks, cs, s);
    case 2: return try_orth_coop<2>(nslice, max_rank, a, nblocks, cs, s);
    case 4: return try_orth_coop<4>(nslice, max_rank, a, nblocks, cs, s);
    // (rank pads 8 to 32 come here only from sets far too large for one cooperative launch, see setup_device)
    case 64: return try_orth_coop<64>(nslice, max_rank, a, nblocks, cs, s);
    default: return false;
  }
}
#endif

#if LQSGD_HAS(5)
// The Cholesky-QR form in one cooperative launch; false (nothing launched) if the grid cannot be
// resident at once or the stream is being captured.
template <int RP>
bool try_orth_chol_coop(int nslice, int max_rank, const DevArgs& a, int nblocks, CoopState* cs, hipStream_t s) {
  if (cs->chol_capacity < 0) {
    int dev = 0, coop = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, orth_chol_kernel<RP>, 256, 0) != hipSuccess) {
      (void)hipGetLastError();
      cs->chol_capacity = 0;
    } else {
      cs->chol_capacity = coop ? cus * per_cu : 0;
    }
  }
  if (nblocks > cs->chol_capacity) return false;
  DevArgs args = a;
  int phase = -1;
  unsigned long long* table = a.chol_table;
  const float* in = nullptr;
  float* out = nullptr;
  int* redo = a.chol_redo;
  unsigned long long n = cs->epoch;
  unsigned max_polls = cs->max_polls ? cs->max_polls : kTablePolls;
  void* params[] = {&args, &nslice, &max_rank, &phase, &table, &in, &out, &redo, &n, &max_polls};
  const hipError_t e = hipLaunchCooperativeKernel(reinterpret_cast<void*>(orth_chol_kernel<RP>), dim3(nblocks), dim3(256),
                                                  params, 0, s);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  cs->epoch += 1;                                // tags of this launch: 4 epoch + 1 .. + 4, and the columns' as above
  note_kernel("orth_chol_kernel<%d>", RP);
  return true;
}

bool launch_orth_chol_coop(int rp, int nslice, int max_rank, const DevArgs& a, int nblocks, CoopState* cs, hipStream_t s) {
  if (!cs || !a.chol_table || !a.orth_table || !a.status || nslice > kCoopMaxSlices) return false;
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &cap) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  if (cap != hipStreamCaptureStatusNone) return false;      // a replay would repeat this launch's tags
  switch (rp) {
    case 8: return try_orth_chol_coop<8>(nslice, max_rank, a, nblocks, cs, s);
    case 16: return try_orth_chol_coop<16>(nslice, max_rank, a, nblocks, cs, s);
    case 32: return try_orth_chol_coop<32>(nslice, max_rank, a, nblocks, cs, s);
    case 64: return try_orth_chol_coop<64>(nslice, max_rank, a, nblocks, cs, s);
    default: return false;
  }
}

// Three launches of the Cholesky-QR kernel, then the column-by-column launches for the pairs that raised their word.
template <int RP>
void launch_orth_chol_split(int nslice, int max_rank, const DevArgs& a, int nblocks, hipStream_t s) {
  float* const planes[4] = {nullptr, a.chol_part, a.chol_part2, nullptr};
  for (int phase = 0; phase < 3; ++phase)
    orth_chol_kernel<RP><<<dim3(nblocks), dim3(256), 0, s>>>(a, nslice, max_rank, phase, nullptr, planes[phase], planes[phase + 1], a.chol_redo, 0ull, 0u);
  for (int j = 0; j <= max_rank; ++j)
    orth_wide_kernel<RP><<<dim3(nblocks), dim3(256), 0, s>>>(a, j, nslice, a.chol_redo);
  note_kernel("orth_chol_kernel<%d> x 3 launches", RP);
}

int chol_entries(int rp) {
  return rp == 8 ? CholShape<8>::NE : rp == 16 ? CholShape<16>::NE : rp == 32 ? CholShape<32>::NE : rp == 64 ? CholShape<64>::NE : 0;
}

// The Cholesky-QR Gram-Schmidt of every pair: in one cooperative launch, or else in several launches.
hipError_t launch_orth_chol(int rp, int nslice, int max_rank, const DevArgs& a, int nblocks, CoopState* coop, hipStream_t s) {
  if (launch_orth_chol_coop(rp, nslice, max_rank, a, nblocks, coop, s)) return hipSuccess;
  if (rp == 8) launch_orth_chol_split<8>(nslice, max_rank, a, nblocks, s);
  else if (rp == 16) launch_orth_chol_split<16>(nslice, max_rank, a, nblocks, s);
  else if (rp == 32) launch_orth_chol_split<32>(nslice, max_rank, a, nblocks, s);
  else launch_orth_chol_split<64>(nslice, max_rank, a, nblocks, s);
  return hipGetLastError();
}
#endif

hipError_t launch_orth_chol(int rp, int nslice, int max_rank, const DevArgs& a, int nblocks, CoopState* coop, hipStream_t s);

#if LQSGD_HAS(4)
hipError_t launch_orth(int rp, int max_rows, int max_rank, int64_t plane_rows, const DevArgs& a, CoopState* coop, bool* copied, hipStream_t s) {
  *copied = a.L <= 0;
  if (a.L <= 0) return hipSuccess;
  const dim3 grid(a.L * a.W);
  const int nslice = (max_rows + 255) / 256;
  // More rows than one workgroup holds, or tall factors and too few (layer, worker) pairs to fill the CUs with one workgroup each:
  // many workgroups per factor, or, at rank pads 1 to 4, one that adds in their order (orth_tall_kernel: a cooperative launch alone
  // costs about 20 us, its launches one by one 9 us a column; W = 4, r = 4, slices / one workgroup, us: 2048 x 1024 29 / 8.6, 8192 x 1024
  // 33 / 15, 8192^2 35 / 24).  It reads all planes on one CU, the slices on 8 to 44, so that many planes of many rows go to them: up to
  // 2^17 rows of planes one workgroup is the faster one or as fast (W = 1 and 4, slices / one workgroup, us: 2048 rows x 32 planes,
  // r = 4 45 / 27, 4096 x 32, r = 1 35 / 27, r = 4 50 / 44, 8192 x 16, r = 2 34 / 29, r = 4, W = 4 41 / 34, though W = 1 43 / 49, 11264 x 8, r = 4
  // 36 / 32), beyond it the slices soon are (8192 x 32, r = 2 38 / 41, r = 4 46 / 53, 11264 x 32, r = 2 38 / 59, 8192 x 126, r = 1 55 / 90,
  // r = 4 95 / 166).  A bound of the waits that was set from outside asks for the form that waits: same bits, and its expiry
  // can be tested at any height.
  // The limits keep each factor with the order of sums that it has had: one workgroup of columns on lanes would hold up to 8192 rows at
  // pad 8 (130 factors of 8000 rows: 121 us, Cholesky-QR 186) and 4096 at pad 16 (3000 rows: 119 and 125), with results that
  // differ by their rounding times the factor's condition number, which at those ranks can be a thousand.
  const bool fits = max_rows <= (rp <= 4 ? 11264 : rp == 8 ? 4096 : rp <= 32 ? 1792 : 1024);
  const bool few = nslice >= 8 && grid.x < kCus / 2;
  if (rp <= 4 && fits && few && plane_rows <= (1 << 17) && !(coop && coop->max_polls)) {
    const bool tall = rp == 1 ? launch_orth_tall<1>(a, max_rows, grid, s) : rp == 2 ? launch_orth_tall<2>(a, max_rows, grid, s)
                                                                                    : launch_orth_tall<4>(a, max_rows, grid, s);
    if (!tall) return hipErrorInvalidValue;
    *copied = true;
    return hipGetLastError();
  }
  if (a.orth_part && (!fits || few)) {
#ifdef LQSGD_TUNING
    static const bool chol = [] { const char* e = std::getenv("LQSGD_ORTH_CHOL"); return !(e && e[0] == '0'); }();
#else
    constexpr bool chol = true;
#endif
    if (chol && rp >= 8 && a.chol_part && a.chol_part2 && a.chol_redo) {
      return launch_orth_chol(rp, nslice, max_rank, a, a.W * a.slices, coop, s);
    }
    // (no Cholesky-QR buffers, or a pad below 8)
    if (launch_orth_coop(rp, nslice, max_rank, a, a.W * a.slices, coop, s)) return hipSuccess;
    for (int j = 0; j <= max_rank; ++j) {
      LQSGD_RP_SWITCH_ORTH(rp, (orth_wide_kernel<RP><<<dim3(a.W * a.slices), dim3(256), 0, s>>>(a, j, nslice, nullptr)));
    }
    note_kernel("orth_wide_kernel<%d> x %d launches", rp, max_rank + 1);
    return hipGetLastError();
  }
  bool done = false;
  switch (rp) {
    case 1: done = launch_orth_reg<1>(a, max_rows, grid, s); break;
    case 2: done = launch_orth_reg<2>(a, max_rows, grid, s); break;
    case 4: done = launch_orth_col<4>(a, max_rows, grid, s); break;
    case 8: done = launch_orth_col<8>(a, max_rows, grid, s); break;
    case 16: done = launch_orth_col<16>(a, max_rows, grid, s); break;
    case 32: done = launch_orth_col<32>(a, max_rows, grid, s); break;
    case 64: done = launch_orth_col<64>(a, max_rows, grid, s); break;
    default: return hipErrorInvalidValue;
  }
  if (!done) return hipErrorInvalidValue;        // (without slices' buffers: a caller this library does not have)
  *copied = true;
  return hipGetLastError();
}
#endif

#if LQSGD_HAS(0)
hipError_t launch_exchange(int mode, int phase, const DevArgs& a, const XTile* tiles, int ntiles, hipStream_t s) {
  if (ntiles <= 0) return hipSuccess;
  const dim3 grid(ntiles), block(256);
  switch (mode) {
    case kQuantOnly: exchange_kernel<kQuantOnly><<<grid, block, 0, s>>>(a, tiles, phase); break;
    case kMeanOnly: exchange_kernel<kMeanOnly><<<grid, block, 0, s>>>(a, tiles, phase); break;
    case kFused: exchange_kernel<kFused><<<grid, block, 0, s>>>(a, tiles, phase); break;
    default: return hipErrorInvalidValue;
  }
  note_kernel("exchange_kernel<%d>", mode);
  return hipGetLastError();
}
#endif

#if LQSGD_HAS(1)
hipError_t launch_back_project(int rp, const DevArgs& a, const Tile* tiles, int ntiles, const VTile* vtiles, int nvtiles,
                               int reverse, hipStream_t s) {
  if (ntiles + nvtiles <= 0) return hipSuccess;
  const dim3 grid(ntiles + nvtiles), block(256);
  LQSGD_RP_SWITCH16(rp, (back_project_kernel<RP><<<grid, block, 0, s>>>(a, tiles, ntiles, vtiles, reverse)));
  note_kernel("back_project_kernel<%d>", rp);
  return hipGetLastError();
}

hipError_t launch_back_project_mfma(int rp, const DevArgs& a, const Tile* tiles, int ntiles, const VTile* vtiles, int nvtiles,
                                    int reverse, hipStream_t s) {
  if (ntiles + nvtiles <= 0) return hipSuccess;
  if (rp == 64)
    back_project_mfma_kernel<2><<<dim3(ntiles + nvtiles), dim3(256), 0, s>>>(a, tiles, ntiles, vtiles, reverse);
  else
    back_project_mfma_kernel<1><<<dim3(ntiles + nvtiles), dim3(256), 0, s>>>(a, tiles, ntiles, vtiles, reverse);
  note_kernel("back_project_mfma_kernel<%d>", rp == 64 ? 2 : 1);
  return hipGetLastError();
}
#endif

#if LQSGD_HAS(0)
hipError_t launch_reduce_q(int phase, const DevArgs& a, const RTile* tiles, int ntiles, hipStream_t s) {
  if (ntiles <= 0) return hipSuccess;
  reduce_q_kernel<<<dim3(ntiles), dim3(256), 0, s>>>(a, tiles, phase);
  note_kernel("reduce_q_kernel");
  return hipGetLastError();
}
#endif

#if LQSGD_HAS(1)
hipError_t launch_residual(int rp, int mode, const DevArgs& a, const Tile* tiles, int ntiles, int narrow_rows, int reverse,
                           hipStream_t s) {
  if (ntiles <= 0) return hipSuccess;
  const dim3 grid(ntiles), block(256);
  const unsigned lds = narrow_rows ? 0 : kThreePerCu;
  switch (mode) {
    case kResidual: LQSGD_RP_SWITCH8(rp, (residual_kernel<RP, kResidual><<<grid, block, lds, s>>>(a, tiles, ntiles, reverse))); break;
    case kResidualGhat: LQSGD_RP_SWITCH8(rp, (residual_kernel<RP, kResidualGhat><<<grid, block, lds, s>>>(a, tiles, ntiles, reverse))); break;
    case kGhatOnly: LQSGD_RP_SWITCH8(rp, (residual_kernel<RP, kGhatOnly><<<grid, block, 0, s>>>(a, tiles, ntiles, reverse))); break;
    default: return hipErrorInvalidValue;
  }
  note_kernel("residual_kernel<%d, %d>", rp, mode);
  return hipGetLastError();
}
#endif

// Rank pad 64: items go to mfma_pair_kernel, a workgroup each, unless there is a CU for either half of every item (items of at most
// 32 rows count as two halves all the same): the 32-row form then has twice the workgroups and takes one round of them (sweep 0,
// microseconds, 32-row form / 64-row form: 64 items, 4096 x 2048, W = 1 66 / 85; 128 items, 4 x 1024^2, W = 2 42 / 49, 4096 x 3072,
// W = 1 59 / 68; 132 items, 2 x (2100 x 1500), W = 2 107 / 77; 192 items, 4 x 1024^2, W = 3 71 / 51).  Lists of short items
// lose nothing by the count, W = 8, r = 50 beside a 64 x 512 layer: 144 items, 17 x (32 x 2048) 67 / 61; 168 items, 20 x (20 x 2048)
// 74 / 65; 200 items, 24 x (32 x 1024) 40 / 38; 520 items, 64 x (32 x 2048) 169 / 155 (first iterations 123 / 130).
template <int RP, int MODE>
void launch_mfma_add(const DevArgs& a, const Tile* tiles, int ntiles, int two, int reverse, hipStream_t s) {
  const dim3 grid(ntiles + two);
  const bool nt = MODE == kMAddFused ? a.nt_fused : a.nt_store;
  if constexpr (RP == 64) {
    if (2 * ntiles > kCus) {
#define LQSGD_LAUNCH_MP(GB, NT) mfma_pair_kernel<MODE, GB, NT><<<dim3(ntiles), dim3(512), 0, s>>>(a, tiles, ntiles, reverse)
      if (a.g_bf16) {
        if (nt) { LQSGD_LAUNCH_MP(true, true); } else { LQSGD_LAUNCH_MP(true, false); }
      } else {
        if (nt) { LQSGD_LAUNCH_MP(false, true); } else { LQSGD_LAUNCH_MP(false, false); }
      }
#undef LQSGD_LAUNCH_MP
      note_kernel("mfma_pair_kernel<%d, %s, %s>", MODE, tf(a.g_bf16), tf(nt));
      return;
    }
  }
  if constexpr (RP == 32) {
    if (a.by_blocks > (MODE == kMAddFused ? 1 : 0)) {
      if (a.g_bf16) mfma_sweep32_kernel<MODE, true><<<grid, dim3(512), 0, s>>>(a, tiles, ntiles, reverse);
      else mfma_sweep32_kernel<MODE, false><<<grid, dim3(512), 0, s>>>(a, tiles, ntiles, reverse);
      note_kernel("mfma_sweep32_kernel<%d, %s>", MODE, tf(a.g_bf16));
      return;
    }
  }
  if constexpr (RP == 16) {
    if (a.by_blocks > (MODE == kMAddFused ? 0 : 1)) {
      mfma_sweep_kernel<RP, MODE><<<grid, dim3(256), 0, s>>>(a, tiles, ntiles, two, reverse);
      note_kernel("mfma_sweep_kernel<%d, %d, false, false>", RP, MODE);
      return;
    }
  }
#define LQSGD_LAUNCH_MA(GB, NT)                                                                                            \
  if constexpr (RP <= 32) mfma_round_kernel<RP, MODE, GB, NT><<<grid, dim3(256), 0, s>>>(a, tiles, ntiles, reverse);     \
  else mfma_sweep_kernel<RP, MODE, GB, NT><<<grid, dim3(256), 0, s>>>(a, tiles, ntiles, two, reverse)
  if (a.g_bf16) {
    if (nt) { LQSGD_LAUNCH_MA(true, true); } else { LQSGD_LAUNCH_MA(true, false); }
  } else {
    if (nt) { LQSGD_LAUNCH_MA(false, true); } else { LQSGD_LAUNCH_MA(false, false); }
  }
#undef LQSGD_LAUNCH_MA
  if constexpr (RP <= 32) note_kernel("mfma_round_kernel<%d, %d, %s, %s>", RP, MODE, tf(a.g_bf16), tf(nt));
  else note_kernel("mfma_sweep_kernel<%d, %d, %s, %s>", RP, MODE, tf(a.g_bf16), tf(nt));
}

template <int RP>
hipError_t launch_mfma_sweep_rp(int mode, const DevArgs& a, const Tile* tiles, int ntiles, int two, int reverse, hipStream_t s) {
  const dim3 grid(ntiles + two), block(256);
  switch (mode) {
    case kMAdd: launch_mfma_add<RP, kMAdd>(a, tiles, ntiles, two, reverse, s); return hipGetLastError();
    case kMAddFused: launch_mfma_add<RP, kMAddFused>(a, tiles, ntiles, two, reverse, s); return hipGetLastError();
    case kMResidual: mfma_sweep_kernel<RP, kMResidual><<<grid, block, 0, s>>>(a, tiles, ntiles, two, reverse); break;
    case kMResidualGhat: mfma_sweep_kernel<RP, kMResidualGhat><<<grid, block, 0, s>>>(a, tiles, ntiles, two, reverse); break;
    case kMGhatOnly:
      if (a.update) mfma_ghat_kernel<RP, true><<<dim3(ntiles), block, 0, s>>>(a, tiles);
      else mfma_ghat_kernel<RP, false><<<dim3(ntiles), block, 0, s>>>(a, tiles);
      note_kernel("mfma_ghat_kernel<%d, %s>", RP, tf(a.update));
      return hipGetLastError();
    default: return hipErrorInvalidValue;
  }
  note_kernel("mfma_sweep_kernel<%d, %d, false, false>", RP, mode);
  return hipGetLastError();
}

// rank pads 16 and 32 in one part, 64 in another: about the same time to compile
hipError_t launch_mfma_sweep64(int mode, const DevArgs& a, const Tile* tiles, int ntiles, int two, int reverse, hipStream_t s);
#if LQSGD_HAS(3)
hipError_t launch_mfma_sweep64(int mode, const DevArgs& a, const Tile* tiles, int ntiles, int two, int reverse, hipStream_t s) {
  return launch_mfma_sweep_rp<64>(mode, a, tiles, ntiles, two, reverse, s);
}
#endif
#if LQSGD_HAS(2)
hipError_t launch_mfma_sweep(int rp, int mode, const DevArgs& a, const Tile* tiles, int ntiles, int two, int reverse,
                             hipStream_t s) {
  if (ntiles <= 0) return hipSuccess;
  if (rp == 16) return launch_mfma_sweep_rp<16>(mode, a, tiles, ntiles, 0, reverse, s);
  if (rp == 32) return launch_mfma_sweep_rp<32>(mode, a, tiles, ntiles, 0, reverse, s);
  if (rp == 64) return launch_mfma_sweep64(mode, a, tiles, ntiles, two, reverse, s);
  return hipErrorInvalidValue;
}
#endif

#if LQSGD_HAS(0)
// ---------------------------------------------------------------------------
// Scratch memory for the entry point that allocates nothing: three blocks per GPU,
// part of the loaded code object, held until the process ends.  The names below
// are host-side handles only; the blocks' device addresses are asked for once per
// device and those addresses are what kernels and copies use.  (The arrays themselves
// are defined at file scope, at the top of this file.)
// ---------------------------------------------------------------------------

hipError_t static_scratch(int device, void** scratch_ptr, void** operands_ptr, void** grams_ptr) {
  constexpr int kMaxDev = 64;
  static void* addr[kMaxDev][3] = {};           // per device; the caller serialises calls
  if (device < 0 || device >= kMaxDev) return hipErrorInvalidDevice;
  if (!addr[device][2]) {
    int cur = -1;
    hipError_t e = hipGetDevice(&cur);
    if (e != hipSuccess) return e;
    if (cur != device) return hipErrorInvalidDevice;     // the address belongs to the device that is current
    void *p = nullptr, *q = nullptr, *g = nullptr;
    if ((e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch))) != hipSuccess) return e;
    if ((e = hipGetSymbolAddress(&q, HIP_SYMBOL(operands))) != hipSuccess) return e;
    if ((e = hipGetSymbolAddress(&g, HIP_SYMBOL(grams))) != hipSuccess) return e;
    if (!p || !q || !g) return hipErrorInvalidSymbol;
    addr[device][0] = p;
    addr[device][1] = q;
    addr[device][2] = g;
  }
  *scratch_ptr = addr[device][0];
  *operands_ptr = addr[device][1];
  *grams_ptr = addr[device][2];
  return hipSuccess;
}

namespace {
__global__ __launch_bounds__(256) void fill_zero_kernel(uint4* p, size_t n16) {
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n16; i += (size_t)gridDim.x * 256)
    p[i] = make_uint4(0u, 0u, 0u, 0u);
}
}  // namespace

hipError_t launch_fill_zero(void* p, size_t bytes, hipStream_t s) {
  if (bytes == 0) return hipSuccess;
  if ((reinterpret_cast<uintptr_t>(p) | bytes) & 15u) return hipErrorInvalidValue;
  const size_t n16 = bytes / 16;
  const unsigned grid = (unsigned)std::min<size_t>(2048, (n16 + 255) / 256);
  fill_zero_kernel<<<dim3(grid), dim3(256), 0, s>>>(static_cast<uint4*>(p), n16);
  return hipGetLastError();
}

// Pointers carried in the kernel's arguments, written to the device table in stream order: the table of the launches
// already enqueued needs no wait, and the copy no staging memory.
struct PointerBatch { const void* p[kPointerBatch]; };
__global__ __launch_bounds__(256) void write_pointers_kernel(PointerBatch b, const void** dst, int n) {
  for (int i = threadIdx.x; i < n; i += 256) dst[i] = b.p[i];
}
hipError_t launch_write_pointers(const void** dst, const void* const* src, size_t n, hipStream_t s) {
  for (size_t i = 0; i < n; i += kPointerBatch) {
    PointerBatch b;
    const int m = (int)std::min<size_t>(kPointerBatch, n - i);
    for (int k = 0; k < m; ++k) b.p[k] = src[i + k];
    for (int k = m; k < kPointerBatch; ++k) b.p[k] = nullptr;
    write_pointers_kernel<<<dim3(1), dim3(256), 0, s>>>(b, dst + i, m);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_pad_factor(int RP, int which, const DevArgs& a, hipStream_t s) {
  if (a.L <= 0 || !a.padded) return hipSuccess;
  pad_factor_kernel<<<dim3(64, a.L), dim3(256), 0, s>>>(a, RP, which);
  return hipGetLastError();
}
#endif

}  // namespace lqsgd
