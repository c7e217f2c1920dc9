// Several gates in one pass over the state. The calls that are given a list of operations
// (qd_circuit_apply, qd_density_apply_ops, the block building of qd_fuse) cut it into groups whose
// target digits all lie in one window of the register; a workgroup stages a tile, the amplitudes of
// that window with every other digit fixed, in LDS, applies the group's gates to it one after the
// other and writes it back. Each gate does the arithmetic of the one-gate kernels (the same fused
// multiply-adds in the same order, in the state's precision, rounded to it after every gate).
//
// Why: one gate a pass is bound by HBM on a large state (a gate of d_T <= 4 has 1-4 flops per byte it
// moves) and by the launch on a small one. A group costs one pass plus, for each gate, one trip through
// LDS (2 x 16 bytes per amplitude at 128 bytes per clock and CU) behind a chain of scalar loads, LDS reads
// and a barrier: of about 0.5 us on a small state; on a large one the LDS pipes are active 30 to 50 % of
// the time of a long pass and HBM moves 1.5 to 3 TB/s (5.1 in a pass of few gates).
// Measured, complex128, named gates, one call each before: 200 gates on 2.5e5 amplitudes 1078 -> 207 us,
// 60 gates on 1.1e8 amplitudes (1.7 GB) 30.0 -> 4.0 ms in 3 passes, 100 gates on 3^15 7.0 -> 1.25 ms;
// 24 gates with their channels on a density matrix of 2.7e7 elements, kernels 4.5 -> 1.8 ms.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <numeric>
#include <vector>

#include "qd_internal.h"
#include "qd_stream.h"

namespace qd {
namespace win {

template <typename R> struct CxW;
template <> struct CxW<double> { using T = double2; };
template <> struct CxW<float> { using T = float2; };

constexpr uint32_t kTile = 4096;       // complex128 amplitudes of a tile (64 KB of LDS: two workgroups per CU)
constexpr int kInserts = 7;            // targets and controls of one gate inside the window
constexpr int kMaxDt = 16;             // amplitudes a thread mixes (16, 12 and 1..9)
constexpr int kOutCtl = 8;             // controls of one gate outside the window
constexpr int kOutDiag = 4;            // diagonal targets of one gate outside the window
constexpr int kMaxOps = 64;            // gates of one pass
constexpr int kMaxRuns = 1024;         // runs of a tile

// One gate of a pass, as the kernel's scalar loads read it: two lines of 64 bytes. LDS positions are
// in bytes (a tile is at most 64 KB). Slice j of the gate is the j-th amplitude of the window whose
// target digits are 0 and whose control digits hold their values: each of those digits, of range d and
// LDS stride s amplitudes, is inserted into j by ascending stride.
struct Op {
  uint32_t dT;             // amplitudes per slice (the in-window targets)
  uint32_t kind;           // kMove: every entry 1, kMono: one entry per column, kDense: dT x dT
  uint32_t nsl;            // slices of the tile
  uint32_t mat;            // first value of its table
  Insert ins[2];           // digits to insert (all zero: none)
  uint32_t nins, nco, nod; // how many of them; controls and diagonal targets outside the window
  uint32_t fill;
  uint32_t off[kMaxDt];    // column y: LDS offset it is read from | the one row y (dense) or its row is written to << 16
};
struct Rest {              // what few gates need
  Insert more[kInserts - 2];
  uint32_t co[kOutCtl];    // digit number | value << 16
  uint32_t od[kOutDiag];   // digit number | weight in the table << 16
};
enum { kMove = 0, kMono = 1, kDense = 2 };
static_assert(sizeof(Op) == 128, "two lines");

struct Digit {          // a digit outside the window that some gate of the group looks at
  Magic32 stride, dim;  // (x / stride) mod dim
};

struct Args {
  SliceMap tiles;       // tile -> global offset of its origin
  Magic32 bl;           // division by the run length
  uint32_t E, nh, ndig, nops, nwarm;
  const int64_t* hoff;  // global offset of each run from the tile's origin
  const Digit* digits;
};

template <typename C>
__device__ __forceinline__ C& at(unsigned char* lds, uint32_t pos) { return *reinterpret_cast<C*>(lds + pos); }

template <typename C>
__device__ __forceinline__ uint32_t slice_at(const Op* __restrict__ op, const Rest* __restrict__ rest, uint32_t nins, uint32_t j) {
  uint32_t b = j;
  auto insert = [&](const Insert& d) {
    const uint32_t q = __umulhi(b, d.mul) + (b & d.self);
    b += q * d.grow + d.add;
  };
  insert(op->ins[0]);   // an entry of zeros inserts nothing: the common gates need no branch
  insert(op->ins[1]);
#pragma unroll 1
  for (uint32_t i = 2; i < nins; ++i) insert(rest->more[i - 2]);
  return b * uint32_t(sizeof(C));
}

// One gate on the tile: a thread takes every blockDim-th slice. (Two slices at a time, their reads on
// their way together, measured 5-10 % slower.)
template <typename R, int DT, int KIND>
__device__ __forceinline__ void gate(unsigned char* lds, const Op* __restrict__ op, const Rest* __restrict__ rest,
                                     const R* __restrict__ m) {
  using C = typename CxW<R>::T;
  const uint32_t nsl = op->nsl, nins = op->nins;
#pragma unroll 1
  for (uint32_t j = threadIdx.x; j < nsl; j += blockDim.x) {
    const uint32_t b = slice_at<C>(op, rest, nins, j);
    C x[DT];
#pragma unroll
    for (int y = 0; y < DT; ++y) x[y] = at<C>(lds, b + (op->off[y] & 0xFFFFu));
    if constexpr (KIND == kDense) {
      auto row = [&](int r) {
        R re = R(0), im = R(0);
#pragma unroll
        for (int c = 0; c < DT; ++c) {
          const R ur = m[2 * (r * DT + c)], ui = m[2 * (r * DT + c) + 1];
          re = fma(ur, x[c].x, re);
          re = fma(-ui, x[c].y, re);
          im = fma(ur, x[c].y, im);
          im = fma(ui, x[c].x, im);
        }
        C v;
        v.x = re;
        v.y = im;
        at<C>(lds, b + (op->off[r] >> 16)) = v;
      };
      // a row of U at a time in scalar registers (all of it would not fit)
      if constexpr (DT * sizeof(R) <= 24) {
#pragma unroll
        for (int r = 0; r < DT; ++r) row(r);
      } else {
#pragma unroll 1
        for (int r = 0; r < DT; ++r) row(r);
      }
    } else {
#pragma unroll
      for (int y = 0; y < DT; ++y) {
        C v = x[y];
        if constexpr (KIND == kMono) {
          const R pr = m[2 * y], pi = m[2 * y + 1];
          v.x = fma(pr, x[y].x, -pi * x[y].y);
          v.y = fma(pr, x[y].y, pi * x[y].x);
        }
        at<C>(lds, b + (op->off[y] >> 16)) = v;
      }
    }
  }
}

template <typename R, int DT>
__device__ __forceinline__ void gate_of(unsigned char* lds, const Op* __restrict__ op, const Rest* __restrict__ rest,
                                        const R* __restrict__ m) {
  const uint32_t kind = op->kind;
  if (kind == kDense) gate<R, DT, kDense>(lds, op, rest, m);
  else if (kind == kMono) gate<R, DT, kMono>(lds, op, rest, m);
  else gate<R, DT, kMove>(lds, op, rest, m);
}

template <typename R, bool NT>
__global__ __launch_bounds__(1024) void k_window(R* psi_raw, Args a, const Op* __restrict__ ops, const Rest* __restrict__ rests,
                                                 const R* __restrict__ tab) {
  using C = typename CxW<R>::T;
  extern __shared__ __align__(16) unsigned char lds[];
  int64_t* s_h = reinterpret_cast<int64_t*>(lds + a.E * uint32_t(sizeof(C)));   // where each run begins
  __shared__ uint32_t s_dig[QD_MAX_QUDITS];
  C* __restrict__ psi = reinterpret_cast<C*>(psi_raw);
  const uint32_t tid = threadIdx.x, bs = blockDim.x, lane = tid & 63u;
  int64_t g0 = a.tiles.base;
  {
    uint32_t rem = blockIdx.x;
#pragma unroll
    for (int g = 0; g < kMaxGroups; ++g)
      if (g < int(a.tiles.ng)) {
        const uint32_t q = g + 1 < int(a.tiles.ng) ? magic_div(rem, a.tiles.gmag[g]) : 0u;
        g0 += int64_t(rem - q * a.tiles.gdim[g]) * a.tiles.gstride[g];
        rem = q;
      }
  }
  for (uint32_t h = tid; h < a.nh; h += bs) s_h[h] = g0 + a.hoff[h];
  if (tid < a.ndig) {
    const Digit d = a.digits[tid];
    const uint32_t q = magic_div(uint32_t(g0), d.stride);
    s_dig[tid] = q - magic_div(q, d.dim) * d.dim.d;
  }
  __syncthreads();
  // the gates' lines and tables into the scalar cache, each wave its share, while the tile is on its way:
  // gate by gate they would be a chain of misses (0.5-1 us each right after the upload)
  const uint32_t* __restrict__ warm = reinterpret_cast<const uint32_t*>(ops);
  for (uint32_t l = __builtin_amdgcn_readfirstlane(tid >> 6) * 4; l < a.nwarm; l += (bs >> 6) * 4) {
    const uint32_t w0 = warm[16 * l], w1 = warm[16 * min(l + 1, a.nwarm - 1)], w2 = warm[16 * min(l + 2, a.nwarm - 1)],
                   w3 = warm[16 * min(l + 3, a.nwarm - 1)];
    __asm__ volatile("" ::"s"(w0), "s"(w1), "s"(w2), "s"(w3));
  }
  constexpr int U = 4;   // amplitudes in flight per thread
  for (uint32_t e0 = tid; e0 < a.E; e0 += U * bs) {
    C v[U];
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const uint32_t e = min(e0 + uint32_t(k) * bs, a.E - 1), h = magic_div(e, a.bl);
      const C* p = psi + (s_h[h] + int64_t(e - h * a.bl.d));
      v[k] = NT ? ld_stream(p) : *p;
    }
#pragma unroll
    for (int k = 0; k < U; ++k)
      if (e0 + uint32_t(k) * bs < a.E) at<C>(lds, (e0 + uint32_t(k) * bs) * uint32_t(sizeof(C))) = v[k];
  }
  // lane i of every wave: whether gate i acts on this tile (its controls outside the window), and where
  // its table begins (its diagonal targets outside)
  bool act = lane < a.nops;
  uint32_t tofs = 0;
  if (act && a.ndig) {
    const Rest* o = rests + lane;
    const uint32_t nco = ops[lane].nco, nod = ops[lane].nod;
    for (uint32_t c = 0; c < nco; ++c) act = act && s_dig[o->co[c] & 0xFFFFu] == o->co[c] >> 16;
    for (uint32_t c = 0; c < nod; ++c) tofs += s_dig[o->od[c] & 0xFFFFu] * (o->od[c] >> 16);
  }
  const uint64_t on = __ballot(act);
  __syncthreads();
  for (uint32_t i = 0; i < a.nops; ++i) {
    const Op* __restrict__ op = ops + i;
    const Rest* __restrict__ rest = rests + i;
    if (on >> i & 1u) {
      const R* __restrict__ m = tab + op->mat + 2 * __builtin_amdgcn_readlane(tofs, i);
      switch (op->dT) {
        case 1: gate<R, 1, kMono>(lds, op, rest, m); break;
        case 2: gate_of<R, 2>(lds, op, rest, m); break;
        case 3: gate_of<R, 3>(lds, op, rest, m); break;
        case 4: gate_of<R, 4>(lds, op, rest, m); break;
        case 5: gate_of<R, 5>(lds, op, rest, m); break;
        case 6: gate_of<R, 6>(lds, op, rest, m); break;
        case 7: gate_of<R, 7>(lds, op, rest, m); break;
        case 8: gate_of<R, 8>(lds, op, rest, m); break;
        case 9: gate_of<R, 9>(lds, op, rest, m); break;
        case 12: gate_of<R, 12>(lds, op, rest, m); break;
        case 16: gate_of<R, 16>(lds, op, rest, m); break;
        default: break;
      }
      __syncthreads();
    }
  }
  for (uint32_t e0 = tid; e0 < a.E; e0 += bs) {
    const uint32_t h = magic_div(e0, a.bl);
    C* p = psi + (s_h[h] + int64_t(e0 - h * a.bl.d));
    if constexpr (NT) st_stream(p, at<C>(lds, e0 * uint32_t(sizeof(C))));
    else *p = at<C>(lds, e0 * uint32_t(sizeof(C)));
  }
}

// ------------------------------------------------------------------------------------------ planner
static bool slice_size(int d) { return (d >= 1 && d <= 9) || d == 12 || d == 16; }

struct Gate {           // a gate as the planner sees it
  uint64_t nd = 0, dg = 0;   // qudits it changes, qudits it only looks at (controls, diagonal targets)
  const GateRef* g = nullptr;
  int cls = 0, dT = 0;
  double act = 1.0;          // share of the amplitudes whose control digits match
  bool fits = false;         // some window can hold it
  bool exact = false;        // it only moves amplitudes: no rounding
};

struct Pass {
  std::vector<int> gates;    // in the order they are applied
  uint64_t window = 0;       // qudits of the window (the suffix included); 0: gates run one by one
  int pq = 0;                // first qudit of the suffix
  uint64_t E = 0;
};

// Whether some window can hold the gate, whichever of its qudits lie inside: the limits of Op (a diagonal
// gate, all of whose targets may lie inside, has at most 16 phases).
static bool can_hold(const Register& r, const Gate& p) {
  const GateRef& g = *p.g;
  if (g.m > kOutCtl || g.k + g.m > kInserts) return false;
  if (p.cls != QD_CLASS_DIAGONAL) return slice_size(p.dT);
  if (g.k > kOutDiag) return false;
  for (int sub = 1; sub < 1 << g.k; ++sub) {
    int d = 1;
    for (int j = 0; j < g.k; ++j)
      if (sub >> j & 1) d *= r.dims[g.t[j]];
    if (!slice_size(d)) return false;
  }
  return true;
}

static uint64_t span_of(const Register& r, uint64_t m) {
  uint64_t p = 1;
  for (int q = 0; q < r.n; ++q)
    if (m >> q & 1) p *= uint64_t(r.dims[q]);
  return p;
}

static uint64_t suffix_mask(const Register& r, int pq) {
  uint64_t m = 0;
  for (int q = pq; q < r.n; ++q) m |= uint64_t(1) << q;
  return m;
}

// Cost in microseconds, from the measured kernels: a launch and its gap, a pass at 5.5 TB/s (one gate;
// the matching part) or 5 TB/s (a window, whole), and for each gate of a window a trip through LDS.
static double cost_alone(const Gate& p, double bytes) { return 4.5 + p.act * bytes / 5.5e6; }
static double cost_inside(const Gate& p, double bytes, double D) {
  const double flops = p.cls == QD_CLASS_DENSE ? 8.0 * p.dT * D : 0.0;
  return 0.5 + p.act * (bytes / 50e6 + flops / 60e6);
}
static double cost_window(double bytes) { return 5.5 + bytes / 5e6; }

// Cuts the list into passes whose windows hold at most emax amplitudes: a pass takes the first gate not
// yet placed and every later one that fits its window and commutes with the gates it moves ahead of;
// with `in_order` (complex64) no gate that rounds moves ahead of another, so that a circuit leaves the bits
// that its gates leave one by one: what a program reads back in 64 bits would show the difference. Moves
// alone still change places. (3^13, 100 named gates: 932 us one by one, 290 so.)
// *cost receives the estimate of all passes.
static std::vector<Pass> plan_passes(const Register& r, const std::vector<Gate>& gate, int pq0, uint64_t emax, double bytes,
                                     bool in_order, double* cost) {
  const size_t n = gate.size();
  const uint64_t suf0 = suffix_mask(r, pq0), all = r.n == 64 ? ~uint64_t(0) : (uint64_t(1) << r.n) - 1;
  std::vector<Pass> passes;
  std::vector<char> placed(n, 0);
  *cost = 0.0;
  for (size_t first = 0; first < n;) {
    Pass ps;
    ps.pq = pq0;
    uint64_t w = suf0 | gate[first].nd, E = span_of(r, w), skip_nd = 0, skip_any = 0;
    bool rounds = false;   // a gate left behind rounds
    ps.gates.push_back(int(first));
    placed[first] = 1;
    if (gate[first].fits && E <= emax)
      for (size_t i = first + 1, looked = 0; i < n && int(ps.gates.size()) < kMaxOps && looked < 512; ++i) {
        if (placed[i]) continue;
        ++looked;
        const Gate& it = gate[i];
        if (it.fits && !((it.nd | it.dg) & skip_nd) && !(it.nd & skip_any) && !(in_order && rounds && !it.exact)) {
          const uint64_t grow = (it.nd & ~w) ? span_of(r, it.nd & ~w) : 1;
          if (E * grow <= emax) {
            w |= it.nd;
            E *= grow;
            ps.gates.push_back(int(i));
            placed[i] = 1;
            continue;
          }
        }
        skip_nd |= it.nd;
        skip_any |= it.nd | it.dg;
        rounds = rounds || !it.exact;
        if ((skip_nd & all) == all) break;
      }
    double one = 0.0, together = cost_window(bytes);
    for (int g : ps.gates) {
      one += cost_alone(gate[size_t(g)], bytes);
      together += cost_inside(gate[size_t(g)], bytes, double(r.D));
    }
    if (ps.gates.size() > 1 && together < one) {
      // room that is left makes the runs longer
      while (ps.pq > 0) {
        const uint64_t bit = uint64_t(1) << (ps.pq - 1);
        if (!(w & bit)) {
          if (E * uint64_t(r.dims[ps.pq - 1]) > emax) break;
          E *= uint64_t(r.dims[ps.pq - 1]);
          w |= bit;
        }
        --ps.pq;
      }
      ps.window = w;
      ps.E = E;
    }
    *cost += ps.window ? together : one;
    passes.push_back(std::move(ps));
    while (first < n && placed[first]) ++first;
  }
  return passes;
}

static bool build_op(const Register& r, const Gate& p, uint64_t window, const std::vector<int>& order,
                     const uint32_t* lst, uint32_t amp, uint64_t E, std::vector<int>* digits, Op* op, Rest* rest,
                     std::vector<double>* tab) {
  const GateRef& gr = *p.g;
  std::memset(op, 0, sizeof(*op));
  std::memset(rest, 0, sizeof(*rest));
  auto inside = [&](int q) { return (window >> q & 1) != 0; };
  auto digit = [&](int q) {
    for (size_t i = 0; i < digits->size(); ++i)
      if ((*digits)[i] == q) return uint32_t(i);
    digits->push_back(q);
    return uint32_t(digits->size() - 1);
  };
  bool fixed[QD_MAX_QUDITS] = {}, target[QD_MAX_QUDITS] = {};
  uint32_t value[QD_MAX_QUDITS] = {};
  uint64_t act = 1;
  for (int j = 0; j < gr.m; ++j) {
    const int c = gr.c[j];
    if (inside(c)) {
      fixed[c] = true;
      act *= uint64_t(r.dims[c]);
      value[c] = uint32_t(gr.v[j]);
    } else {
      rest->co[op->nco++] = digit(c) | uint32_t(gr.v[j]) << 16;
    }
  }
  const bool diag = p.cls == QD_CLASS_DIAGONAL;
  int in[kInserts], out[kInserts], nin = 0, nout = 0;   // target positions, in listed order
  int dIn = 1, dOut = 1;
  for (int j = 0; j < gr.k; ++j) {
    const int t = gr.t[j];
    if (inside(t)) {
      in[nin++] = j;
      dIn *= r.dims[t];
      target[t] = true;
    } else {
      if (!diag || nout == kOutDiag) return false;
      out[nout++] = j;
      dOut *= r.dims[t];
    }
  }
  if (!slice_size(dIn)) return false;
  op->dT = uint32_t(dIn);
  op->nsl = uint32_t(E / (uint64_t(dIn) * act));
  op->kind = p.cls == QD_CLASS_DENSE ? kDense : kMono;
  uint32_t roff[kMaxDt];
  for (int y = 0; y < dIn; ++y) {
    uint32_t off = 0;
    for (int i = nin - 1, rem = y; i >= 0; --i) {
      const int t = gr.t[in[i]];
      off += uint32_t(rem % r.dims[t]) * lst[t] * amp;
      rem /= r.dims[t];
    }
    roff[y] = off;
    op->off[y] = off | off << 16;
  }
  op->mat = uint32_t(tab->size());
  if (op->kind == kDense) {
    tab->insert(tab->end(), gr.U, gr.U + 2 * size_t(dIn) * size_t(dIn));
  } else if (!diag) {
    op->kind = kMove;
    for (int y = 0; y < dIn; ++y)
      for (int row = 0; row < dIn; ++row) {   // column y holds one entry
        const double* e = gr.U + 2 * (size_t(row) * dIn + y);
        if (e[0] == 0.0 && e[1] == 0.0) continue;
        op->off[y] = roff[y] | roff[row] << 16;
        if (e[0] != 1.0 || e[1] != 0.0) op->kind = kMono;
        tab->push_back(e[0]);
        tab->push_back(e[1]);
      }
  } else {
    // phases by (outside digits, inside digits)
    uint32_t w = uint32_t(dIn);
    for (int i = nout - 1; i >= 0; --i) {
      const int t = gr.t[out[i]];
      rest->od[op->nod++] = digit(t) | w << 16;
      w *= uint32_t(r.dims[t]);
    }
    int mul[QD_MAX_QUDITS];
    for (int j = gr.k - 1, m = 1; j >= 0; --j) {
      mul[j] = m;
      m *= r.dims[gr.t[j]];
    }
    for (int o = 0; o < dOut; ++o)
      for (int y = 0; y < dIn; ++y) {
        int loc = 0;
        for (int i = nout - 1, rem = o; i >= 0; --i) {
          const int j = out[i], d = r.dims[gr.t[j]];
          loc += rem % d * mul[j];
          rem /= d;
        }
        for (int i = nin - 1, rem = y; i >= 0; --i) {
          const int j = in[i], d = r.dims[gr.t[j]];
          loc += rem % d * mul[j];
          rem /= d;
        }
        const double* e = gr.U + 2 * size_t(loc) * size_t(p.dT + 1);
        tab->push_back(e[0]);
        tab->push_back(e[1]);
      }
  }
  for (int q : order) {   // by ascending LDS stride
    if (!fixed[q] && !target[q]) continue;
    const uint32_t st = lst[q];
    (op->nins < 2 ? op->ins[op->nins] : rest->more[op->nins - 2]) = make_insert(st, uint32_t(r.dims[q]), value[q]);
    ++op->nins;
  }
  return true;
}

// LDS order of a window: the suffix from the lowest digit up, then its other qudits
static std::vector<int> window_order(const Register& r, const Pass& ps, uint32_t* lst) {
  std::vector<int> order;
  uint32_t st = 1;
  for (int q = r.n - 1; q >= 0; --q)
    if (q >= ps.pq || (ps.window >> q & 1)) {
      order.push_back(q);
      lst[q] = st;
      st *= uint32_t(r.dims[q]);
    }
  return order;
}

}  // namespace win

using namespace win;

// Applies the gates in order (up to exchanges of neighbours that commute exactly: no qudit in common
// that either of them changes). Gates run one by one, as qd_apply_gate launches them, on registers of
// 2^32 amplitudes or more, while the stream is captured (a group's tables are uploaded from a buffer
// that later calls write again), where the costs above say so and where the buffer cannot be allocated.
int apply_gate_list(qd_state* s, const std::vector<GateRef>& list) {
  const Register& r = s->reg;
  const size_t n = list.size();
  auto alone = [&](size_t i) -> int {
    const GateRef& g = list[i];
    GatePlan p;
    plan_gate(r, s->prec, g.t, g.k, g.c, g.v, g.m, g.U, &p);
    int rc = launch_gate(s, p);
    if (rc == QD_OK && last_kernel()[0]) ++s->launches, ++s->trips;
    return rc;
  };
  if (n < 2 || uint64_t(r.D) > 0xFFFFFFFFull || stream_captured(s->stream)) {
    for (size_t i = 0; i < n; ++i) {
      int rc = alone(i);
      if (rc) return rc;
    }
    return QD_OK;
  }
  const bool dbl = s->prec == QD_C128;
  const uint32_t amp = uint32_t(amp_bytes(s->prec));
  const double bytes = 2.0 * double(r.D) * double(amp);
  std::vector<Gate> gate(n);
  for (size_t i = 0; i < n; ++i) {
    Gate& p = gate[i];
    p.g = &list[i];
    p.dT = 1;
    for (int j = 0; j < p.g->k; ++j) p.dT *= r.dims[p.g->t[j]];
    p.cls = classify(p.g->U, p.dT);
    if (p.cls == QD_CLASS_MONOMIAL) {
      p.exact = true;
      for (int e = 0; e < p.dT * p.dT; ++e)
        p.exact = p.exact && p.g->U[2 * e + 1] == 0.0 && (p.g->U[2 * e] == 0.0 || p.g->U[2 * e] == 1.0);
      // one that rounds is mixed as a dense gate wherever the gate by itself would be
      if (!dbl && !p.exact) {
        GatePlan alone_plan;
        plan_gate(r, s->prec, p.g->t, p.g->k, p.g->c, p.g->v, p.g->m, p.g->U, &alone_plan);
        if (route_gate(r, s->prec, alone_plan) == QD_ROUTE_DIRECT && alone_plan.dT <= 9) p.cls = QD_CLASS_DENSE;
      }
    }
    for (int j = 0; j < p.g->k; ++j) (p.cls == QD_CLASS_DIAGONAL ? p.dg : p.nd) |= uint64_t(1) << p.g->t[j];
    for (int j = 0; j < p.g->m; ++j) {
      p.dg |= uint64_t(1) << p.g->c[j];
      p.act /= r.dims[p.g->c[j]];
    }
    p.fits = can_hold(r, p);
  }
  // the shortest suffix staged: two lines of amplitudes, one where the state stays in the caches
  const uint64_t minrun = bytes > 64e6 ? (dbl ? 16 : 32) : 8;
  int pq0 = r.n;
  for (uint64_t run = 1; pq0 > 0 && run < minrun;) run *= uint64_t(r.dims[--pq0]);
  // A tile of 64 KB, or the whole state; below 256 tiles of that size smaller ones that give every CU
  // one (2^18 complex128 amplitudes, 200 gates: 284 us with 1024 of them a tile, 356 with 4096; 2^20: 212
  // and 170). A large state also tries 32 KB, which leaves more workgroups on a CU and measured 0.82 to
  // 1.0 of the time in LDS, and takes it where the passes it adds cost less.
  const uint64_t most = dbl ? kTile : 2 * kTile, D = uint64_t(r.D);
  const uint64_t emax = D <= most ? most : std::min(most, std::max<uint64_t>(1024, D / 256));
  double cost = 0.0;
  std::vector<Pass> passes = plan_passes(r, gate, pq0, emax, bytes, !dbl, &cost);
  if (D >= 512 * most) {
    double half = 0.0;
    std::vector<Pass> other = plan_passes(r, gate, pq0, most / 2, bytes, !dbl, &half);
    if (0.94 * half < cost) passes.swap(other);
  }

  // a pass is uploaded and launched as soon as its tables are made, so the GPU works while the next
  // ones are prepared
  std::vector<char> blob;
  std::vector<int> digits;
  std::vector<Op> ops;
  std::vector<Rest> rest;
  std::vector<double> tab;
  std::vector<int64_t> hoff;
  auto put = [&](const void* p, size_t bytes_) {
    const size_t at = (blob.size() + 63) & ~size_t(63);
    blob.resize(at + bytes_);
    std::memcpy(blob.data() + at, p, bytes_);
    return at;
  };
  auto one_by_one = [&](const Pass& ps) -> int {
    int rc = QD_OK;
    for (size_t i = 0; i < ps.gates.size() && !rc; ++i) rc = alone(size_t(ps.gates[i]));
    return rc;
  };
  for (const Pass& ps : passes) {
    bool ok = ps.window != 0;
    Args a;
    uint32_t lst[QD_MAX_QUDITS] = {};
    std::vector<int> order;
    uint64_t BL = 1, nh = 1;
    if (ok) {
      order = window_order(r, ps, lst);
      int role[QD_MAX_QUDITS] = {};
      for (int q : order) role[q] = 1;
      BL = uint64_t(ps.pq > 0 ? r.strides[ps.pq - 1] : r.D);
      nh = ps.E / BL;
      ok = nh <= uint64_t(kMaxRuns) && fill_slicemap(make_groups(r, role, nullptr, 0, r.n), 0, &a.tiles) == QD_OK;
      digits.clear();
      tab.clear();
      ops.resize(ps.gates.size());
      rest.resize(ps.gates.size());
      for (size_t i = 0; i < ops.size() && ok; ++i)
        ok = build_op(r, gate[size_t(ps.gates[i])], ps.window, order, lst, amp, ps.E, &digits, &ops[i], &rest[i], &tab);
    }
    if (!ok) {
      int rc = one_by_one(ps);
      if (rc) return rc;
      continue;
    }
    hoff.resize(nh);
    for (uint64_t h = 0; h < nh; ++h) {
      uint64_t rem = h;
      int64_t off = 0;
      for (int q : order) {
        if (q >= ps.pq) continue;
        off += int64_t(rem % uint64_t(r.dims[q])) * r.strides[q];
        rem /= uint64_t(r.dims[q]);
      }
      hoff[size_t(h)] = off;
    }
    Digit dg[QD_MAX_QUDITS];
    for (size_t i = 0; i < digits.size(); ++i)
      dg[i] = Digit{make_magic32(uint32_t(r.strides[digits[i]])), make_magic32(uint32_t(r.dims[digits[i]]))};
    blob.clear();
    const size_t o_h = put(hoff.data(), hoff.size() * sizeof(int64_t));
    const size_t o_d = put(dg, digits.size() * sizeof(Digit));
    const size_t o_rest = put(rest.data(), rest.size() * sizeof(Rest));
    const size_t o_op = put(ops.data(), ops.size() * sizeof(Op));
    size_t o_tab = 0;
    if (dbl) {
      o_tab = put(tab.data(), tab.size() * sizeof(double));
    } else {
      const std::vector<float> f(tab.begin(), tab.end());
      o_tab = put(f.data(), f.size() * sizeof(float));
    }
    blob.resize((blob.size() + 63) & ~size_t(63));   // the last line is touched whole
    char *host = nullptr, *dev = nullptr;
    int rc = ring_reserve(&s->ring, s->stream, blob.size(), &host, &dev);
    if (rc == QD_ENOMEM) {   // no room for the tables: gates one by one need none
      rc = one_by_one(ps);
      if (rc) return rc;
      continue;
    }
    if (rc) return rc;
    std::memcpy(host, blob.data(), blob.size());
    rc = ring_commit(&s->ring, s->stream, host, dev, blob.size());
    if (rc) return rc;
    a.bl = make_magic32(uint32_t(BL));
    a.E = uint32_t(ps.E);
    a.nh = uint32_t(nh);
    a.ndig = uint32_t(digits.size());
    a.nops = uint32_t(ops.size());
    // gates and tables lie together; of the 16 KB scalar cache that two CUs share, at most 12 are filled ahead
    a.nwarm = uint32_t(std::min<size_t>((blob.size() - o_op) / 64, 192));
    a.hoff = reinterpret_cast<const int64_t*>(dev + o_h);
    a.digits = reinterpret_cast<const Digit*>(dev + o_d);
    const size_t lds = size_t(ps.E) * amp + nh * sizeof(int64_t);
    // 128 bytes of amplitudes a thread and gate: each gate costs a wave its scalar loads and branches
    // however little it mixes (1.1e8 amplitudes, 60 gates: 4.3 ms with 8 complex128 amplitudes a thread,
    // 6.0 with 4, 10 with 2); with less than two tiles per CU the waves are needed for latency instead
    const uint64_t per = a.tiles.count < 512 ? 2 : (dbl ? 8 : 16);
    const unsigned threads = unsigned(std::min<uint64_t>(1024, std::max<uint64_t>(64, (ps.E / per + 63) / 64 * 64)));
    // a state that the last-level cache (256 MB) holds between passes is not streamed past it: 100 named gates
    // on 3^15 1252 -> 1165 us, on 2^24 1192 -> 1161, on 4^12 1388 -> 1366
    const bool nt = bytes > 2.0 * double(256 << 20);
    auto launch = [&](auto kern, auto real) -> int {
      using R = decltype(real);
      if (lds > (size_t(48) << 10))
        QD_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, int(lds)));
      hipLaunchKernelGGL(kern, dim3(a.tiles.count), dim3(threads), lds, s->stream, reinterpret_cast<R*>(s->data), a,
                         reinterpret_cast<const Op*>(dev + o_op), reinterpret_cast<const Rest*>(dev + o_rest),
                         reinterpret_cast<const R*>(dev + o_tab));
      QD_HIP(hipGetLastError());
      return QD_OK;
    };
    rc = dbl ? (nt ? launch(k_window<double, true>, double()) : launch(k_window<double, false>, double()))
             : (nt ? launch(k_window<float, true>, float()) : launch(k_window<float, false>, float()));
    if (rc) return rc;
    set_last_kernel(dbl ? "k_window<double>" : "k_window<float>");
    s->launches += int64_t(ps.gates.size());   // counted as the passes it stands for
    ++s->trips;
  }
  return QD_OK;
}

}  // namespace qd
