// Gate-application kernels for gfx950 and their launcher.
//
// One generalized gate (Sec. 2.1) applied in place: every slice of the register (the d_T
// amplitudes that share all non-target digits) whose control digits match is multiplied by U.
// That is the Kronecker-embedded Moment operator I (x) U (x) I of Sec. 3.5 applied to the state
// vector, at O(D d_T) cost.
//
// Kernel families (HBM-bound up to d_T of about 32: 8 d_T flops per 2 x 16 bytes moved):
//   k_slices_direct  one slice per thread. Used when every target has a stride >= run_min (or at
//                    least one line, for controls inside a line that leave lines inactive), so the
//                    lanes of a wavefront take consecutive low digits and each load instruction
//                    reads one contiguous run.
//   k_slices_tiled   a low-stride target: the workgroup stages a tile of whole slices in LDS with
//                    contiguous coalesced loads (runs of the low suffix of the register), mixes
//                    each slice inside LDS and writes the tile back coalesced.
//   k_diag           diagonal gates (Z_d, controlled phases): elementwise, consecutive lanes on
//                    consecutive amplitudes whatever the target strides.
//   k_dense_mfma     dense gates of d_T >= 10: tiles of slices as complex GEMMs on the matrix cores.
//   k_dense_generic  registers of 2^32 amplitudes or more (64-bit indices), any d_T <= 1024: slices
//                    gathered into LDS, U read from device memory.
// The slice kernels take U (dense) or a destination/phase table (monomial: X_{+a}, controlled
// shifts, qudit swaps) inside the kernel arguments.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstddef>
#include <cstdio>
#include <cstring>
#include <numeric>
#include <vector>

#include "qd_internal.h"
#include "qd_stream.h"

namespace qd {

template <typename R> struct CxT;
template <> struct CxT<double> { using T = double2; };
template <> struct CxT<float> { using T = float2; };

// ------------------------------------------------------------------------------------------ index maps
__device__ __forceinline__ int64_t sm_offset(const SliceMap& sm, uint32_t idx) {
  int64_t off = sm.base;
  uint32_t rem = idx;
#pragma unroll
  for (int g = 0; g < kMaxGroups; ++g) {
    if (g < int(sm.ng)) {
      const uint32_t q = (g + 1 < int(sm.ng)) ? magic_div(rem, sm.gmag[g]) : 0u;
      const uint32_t r = rem - q * sm.gdim[g];
      off += int64_t(r) * sm.gstride[g];
      rem = q;
    }
  }
  return off;
}

__device__ __forceinline__ int64_t sm_offset_loc(const SliceMap& sm, uint32_t idx, uint32_t* loc) {
  int64_t off = sm.base;
  uint32_t rem = idx, l = 0;
#pragma unroll
  for (int g = 0; g < kMaxGroups; ++g) {
    if (g < int(sm.ng)) {
      const uint32_t q = (g + 1 < int(sm.ng)) ? magic_div(rem, sm.gmag[g]) : 0u;
      const uint32_t r = rem - q * sm.gdim[g];
      off += int64_t(r) * sm.gstride[g];
      l += r * sm.lmul[g];
      rem = q;
    }
  }
  *loc = l;
  return off;
}

__device__ __forceinline__ int64_t sm64_offset(const SliceMap64& sm, uint64_t idx) {
  int64_t off = sm.base;
  uint64_t rem = idx;
  for (uint32_t g = 0; g < sm.ng; ++g) {
    const uint64_t q = rem / sm.gdim[g];
    off += int64_t(rem - q * sm.gdim[g]) * sm.gstride[g];
    rem = q;
  }
  return off;
}

// ------------------------------------------------------------------------------------------ gate ops
template <typename R, int DT> struct DenseOp { R u[2 * DT * DT]; };
template <typename R, int DT> struct MonoOp { R ph[2 * DT]; int32_t dst[DT]; };

// doff[c] = toff[dst[c]] for monomial gates (filled by the host so no kernel indexes its
// arguments with a run-time value); unused by dense gates.

// put: a result into the state in HBM (ST: streaming store) or into LDS
template <bool ST, typename C>
__device__ __forceinline__ void put(C* p, int64_t i, C v) {
  if constexpr (ST) st_stream(p + i, v);
  else p[i] = v;
}

// get: an amplitude from HBM (ST: streaming load)
template <bool ST, typename C>
__device__ __forceinline__ C get(const C* p) {
  if constexpr (ST) return ld_stream(p);
  else return *p;
}

template <bool ST, typename C, typename R, int DT>
__device__ __forceinline__ void mix_store(C* p, int64_t base, const int64_t* toff, const int64_t*,
                                          const DenseOp<R, DT>& op, const C (&x)[DT]) {
#pragma unroll
  for (int r = 0; r < DT; ++r) {
    R re = R(0), im = R(0);
#pragma unroll
    for (int c = 0; c < DT; ++c) {
      const R ur = op.u[2 * (r * DT + c)], ui = op.u[2 * (r * DT + c) + 1];
      re = fma(ur, x[c].x, re);
      re = fma(-ui, x[c].y, re);
      im = fma(ur, x[c].y, im);
      im = fma(ui, x[c].x, im);
    }
    C y;
    y.x = re;
    y.y = im;
    put<ST>(p, base + toff[r], y);
  }
}

template <bool ST, typename C, typename R, int DT>
__device__ __forceinline__ void mix_store(C* p, int64_t base, const int64_t*, const int64_t* doff,
                                          const MonoOp<R, DT>& op, const C (&x)[DT]) {
#pragma unroll
  for (int c = 0; c < DT; ++c) {
    const R pr = op.ph[2 * c], pi = op.ph[2 * c + 1];
    C y;
    y.x = fma(pr, x[c].x, -pi * x[c].y);
    y.y = fma(pr, x[c].y, pi * x[c].x);
    put<ST>(p, base + doff[c], y);
  }
}

// ------------------------------------------------------------------------------------------ direct
// Controls whose stride is below one 128-byte line leave lines partly active, and controls of
// larger stride that is not a whole number of lines leave the lines at both ends of every active
// run partly active. HBM is written in whole lines here (a partial line costs a read-modify-write),
// so both cases are applied with whole-line writes: amplitudes of inactive slices that share a line
// with active ones are read and written back unchanged, and lines with no active amplitude at all
// are not touched.
enum { kDirectPlain = 0, kDirectPred = 1, kDirectEdge = 2 };

template <typename R, int DT, typename OP>
struct DirectArgs {
  R* psi;
  SliceMap sm;
  int64_t toff[DT];
  int64_t doff[DT];
  OP op;
  // kDirectPred: the low-stride controls are free digits of sm (singleton groups whose lmul weights
  // give their local index); a slice is mixed when that index equals vloc, else written unchanged.
  // Lines holding no amplitude where those controls all have their values are left untouched when
  // lper > 1: line L holds one iff bit (L mod lper) of lmask is set (the pattern of the low control
  // digits repeats every lper lines).
  uint32_t vloc;
  uint32_t lper;
  Magic32 lpm;
  uint64_t lmask;
  // kDirectEdge (every target above the lowest control): sm enumerates the active slices, grouped
  // into blocks of nA = blen consecutive indices (the blen contiguous amplitudes where the lowest
  // control holds its value, all higher digits fixed, each a slice base). Each block gets W lanes,
  // LINE times the most lines a block can touch, taking the amplitudes of those lines in order;
  // lanes outside the block rewrite their amplitudes unchanged (in every target plane whose line
  // holds amplitudes of the block).
  uint32_t nA;
  uint32_t W;
  Magic32 wm;
  uint32_t blen;
  uint32_t nvirt;
  int64_t D;
};

template <typename R> struct LineAmps;   // amplitudes per 128-byte line
template <> struct LineAmps<double> { static constexpr int value = 8; };
template <> struct LineAmps<float> { static constexpr int value = 16; };
template <typename R> constexpr int kLineShift = sizeof(R) == 8 ? 3 : 4;

// Outputs of one slice where every lane stores position y at the same instruction: the mixed
// values where the slice is active, its inputs otherwise (a monomial U picks, for each output row,
// the column whose entry lands there: dst is uniform, so the tests are scalar).
template <typename C, typename R, int DT>
__device__ __forceinline__ void mix_select(const DenseOp<R, DT>& op, const C (&x)[DT], bool act, C (&out)[DT]) {
#pragma unroll
  for (int r = 0; r < DT; ++r) {
    R re = R(0), im = R(0);
#pragma unroll
    for (int c = 0; c < DT; ++c) {
      const R ur = op.u[2 * (r * DT + c)], ui = op.u[2 * (r * DT + c) + 1];
      re = fma(ur, x[c].x, re);
      re = fma(-ui, x[c].y, re);
      im = fma(ur, x[c].y, im);
      im = fma(ui, x[c].x, im);
    }
    out[r].x = act ? re : x[r].x;
    out[r].y = act ? im : x[r].y;
  }
}

template <typename C, typename R, int DT>
__device__ __forceinline__ void mix_select(const MonoOp<R, DT>& op, const C (&x)[DT], bool act, C (&out)[DT]) {
#pragma unroll
  for (int y = 0; y < DT; ++y) out[y] = x[y];
#pragma unroll
  for (int c = 0; c < DT; ++c) {
    const R pr = op.ph[2 * c], pi = op.ph[2 * c + 1];
    C v;
    v.x = fma(pr, x[c].x, -pi * x[c].y);
    v.y = fma(pr, x[c].y, pi * x[c].x);
#pragma unroll
    for (int y = 0; y < DT; ++y)
      if (op.dst[c] == y) {
        out[y].x = act ? v.x : out[y].x;
        out[y].y = act ? v.y : out[y].y;
      }
  }
}

template <typename R, int DT, typename OP, int SPT, int MODE, bool ST>
__global__ __launch_bounds__(256) void k_slices_direct(DirectArgs<R, DT, OP> a) {
  using C = typename CxT<R>::T;
  C* __restrict__ psi = reinterpret_cast<C*>(a.psi);
  const uint64_t bs = blockDim.x;
  if constexpr (MODE != kDirectPlain) {
    // one slice or edge position per thread; position y of every lane is loaded and stored by
    // one instruction, so each instruction writes whole lines wherever its lanes are consecutive
    int64_t pos;
    bool act = true;
    uint32_t valid = (1u << DT) - 1u;
    if constexpr (MODE == kDirectPred) {
      const uint64_t i = uint64_t(blockIdx.x) * bs + threadIdx.x;
      if (i >= a.sm.count) return;
      uint32_t loc;
      pos = sm_offset_loc(a.sm, uint32_t(i), &loc);
      act = loc == a.vloc;
      if (!act && a.lper > 1) {
        valid = 0;
#pragma unroll
        for (int y = 0; y < DT; ++y) {
          const uint32_t L = uint32_t((pos + a.toff[y]) >> kLineShift<R>);
          if ((a.lmask >> (L - magic_div(L, a.lpm) * a.lper)) & 1u) valid |= 1u << y;
        }
        if (!valid) return;
      }
    } else {
      // the block's lanes walk its lines in order: lane j takes amplitude L0 + j, L0 the start of
      // the line holding the block's first amplitude, so every instruction writes whole lines
      constexpr int LINE = LineAmps<R>::value;
      const uint32_t vi = uint32_t(blockIdx.x) * uint32_t(bs) + threadIdx.x;
      if (vi >= a.nvirt) return;
      const uint32_t b = magic_div(vi, a.wm);
      const int64_t start = sm_offset(a.sm, b * a.nA);
      const int64_t end = start + a.blen - 1;
      pos = (start & ~int64_t(LINE - 1)) + int64_t(vi - b * a.W);
      if (pos > (end | int64_t(LINE - 1))) return;
      act = pos >= start && pos <= end;
      if (!act) {
        // outside the block: rewritten unchanged where its line (in each target plane) holds
        // amplitudes of the block
        valid = 0;
#pragma unroll
        for (int y = 0; y < DT; ++y) {
          const int64_t q = pos + a.toff[y];
          if ((q >> kLineShift<R>) >= ((start + a.toff[y]) >> kLineShift<R>) &&
              (q >> kLineShift<R>) <= ((end + a.toff[y]) >> kLineShift<R>) && q < a.D)
            valid |= 1u << y;
        }
        if (!valid) return;
      }
    }
    C x[DT], out[DT];
#pragma unroll
    for (int y = 0; y < DT; ++y) {
      x[y].x = R(0);
      x[y].y = R(0);
      if (valid & (1u << y)) x[y] = get<ST>(psi + pos + a.toff[y]);
    }
    mix_select<C, R, DT>(a.op, x, act, out);
#pragma unroll
    for (int y = 0; y < DT; ++y)
      if (valid & (1u << y)) put<ST>(psi, pos + a.toff[y], out[y]);
  } else {
    const uint64_t first = uint64_t(blockIdx.x) * bs * SPT + threadIdx.x;
    int64_t base[SPT];
    C x[SPT][DT];
#pragma unroll
    for (int s = 0; s < SPT; ++s) {
      const uint64_t i = first + s * bs;
      base[s] = i < a.sm.count ? sm_offset(a.sm, uint32_t(i)) : -1;
    }
#pragma unroll
    for (int s = 0; s < SPT; ++s)
      if (base[s] >= 0) {
#pragma unroll
        for (int y = 0; y < DT; ++y) x[s][y] = get<ST>(psi + base[s] + a.toff[y]);
      }
#pragma unroll
    for (int s = 0; s < SPT; ++s)
      if (base[s] >= 0) mix_store<ST, C, R, DT>(psi, base[s], a.toff, a.doff, a.op, x[s]);
  }
}

// Dense gates of d_T = 12 or 16 whose targets all have strides >= run_min: one slice per thread as
// in k_slices_direct, with U (too large for the kernel arguments in complex128) staged in LDS and
// read by broadcast; the slice map and target offsets are staged too, before the first store.
struct LuHead {
  SliceMap sm;
  int64_t toff[16];
  // followed by 2 DT^2 values of R (U, row-major interleaved)
};

template <typename R, int DT, bool ST>
__global__ __launch_bounds__(256) void k_slices_direct_lu(R* psi_raw, const unsigned char* desc) {
  using C = typename CxT<R>::T;
  __shared__ R su[2 * DT * DT];
  __shared__ SliceMap smap;
  __shared__ int64_t st[DT];
  static_assert(sizeof(SliceMap) % 4 == 0, "slice map copied in 4-byte words");
  const LuHead& h = *reinterpret_cast<const LuHead*>(desc);
  const R* ug = reinterpret_cast<const R*>(desc + sizeof(LuHead));
  const uint32_t tid = threadIdx.x;
  for (uint32_t i = tid; i < 2u * DT * DT; i += blockDim.x) su[i] = ug[i];
  for (uint32_t i = tid; i < sizeof(SliceMap) / 4; i += blockDim.x)
    reinterpret_cast<uint32_t*>(&smap)[i] = reinterpret_cast<const uint32_t*>(&h.sm)[i];
  if (tid < uint32_t(DT)) st[tid] = h.toff[tid];
  __syncthreads();
  C* __restrict__ psi = reinterpret_cast<C*>(psi_raw);
  const uint64_t i = uint64_t(blockIdx.x) * blockDim.x + tid;
  if (i >= smap.count) return;
  const int64_t b = sm_offset(smap, uint32_t(i));
  C x[DT];
#pragma unroll
  for (int y = 0; y < DT; ++y) x[y] = get<ST>(psi + b + st[y]);
#pragma unroll
  for (int r = 0; r < DT; ++r) {
    __asm__ volatile("" ::: "memory");   // U is read from LDS here (held in registers it would take hundreds)
    R re = R(0), im = R(0);
#pragma unroll
    for (int c = 0; c < DT; ++c) {
      const R ur = su[2 * (r * DT + c)], ui = su[2 * (r * DT + c) + 1];
      re = fma(ur, x[c].x, re);
      re = fma(-ui, x[c].y, re);
      im = fma(ur, x[c].y, im);
      im = fma(ui, x[c].x, im);
    }
    C yv;
    yv.x = re;
    yv.y = im;
    put<ST>(psi, b + st[r], yv);
  }
}

// ------------------------------------------------------------------------------------------ tiled
// The arguments are read where they lie, in the kernel argument segment, by scalar loads: as a by-value
// parameter the slice maps and U overflowed the scalar registers, and spilled values were read back lane
// by lane (250-370 of them). Slices are found by inserting the target and control digits into the slice
// number, which takes four instructions a digit. Dense U comes a row at a time by scalar loads (broadcast
// from LDS its reads took more of the LDS pipe than the amplitudes'). Measured, with the smaller tiles of
// tile_geometry: 9 x 9 gates on 3^16 474 -> 260 us (complex128), 177 -> 131 (complex64); qutrits on the
// hybrid register 594 -> 557 us and 430 -> 280; a qubit on 2^25 207 -> 178 and 134 -> 96.
template <typename R, int DT, typename OP>
struct TileArgs {
  R* psi;
  SliceMap tiles;                 // tile index -> global offset of the tile's origin
  uint32_t BL;                    // run length (amplitudes of the low suffix)
  uint32_t dH;                    // number of runs (product of the high targets' dims)
  Magic32 blm;                    // division by BL
  int64_t hoff[kMaxTileRuns];     // global offset of run h from the tile origin
  uint32_t nsl, nins;             // slices of a tile; digits inserted into a slice number ...
  Insert ins[14];                 // ... to make its LDS index (a tile of 2^13 amplitudes has at most 13 digits)
  uint32_t toff[DT];              // LDS offset of target combination y
  uint32_t doff[DT];              // monomial: LDS offset of the row column y moves to
  uint32_t nsc;                   // controls inside the suffix that the tile leaves out, and for
  Magic32 scm[kMaxTileCtl];       // each, by increasing stride s: division by s,
  uint32_t scmul[kMaxTileCtl];    // s (d_c - 1) and
  uint32_t scadd[kMaxTileCtl];    // v s (v: the control value)
  OP op;
};

#define QD_KARG const __attribute__((address_space(4)))   // kernel argument memory

template <typename M>
__device__ __forceinline__ Magic32 karg_magic(M* m) {
  Magic32 r;
  r.mul = m->mul;
  r.sh1 = m->sh1;
  r.sh2 = m->sh2;
  r.d = m->d;
  return r;
}

// Bytes [BEGIN, END) of the arguments into the scalar cache, every line asked for at once: read where they are
// needed they are a chain of misses, which bounds the kernel on small registers (9 x 9 gates on 3^9: 7.9 ->
// 5.8 us in complex128, 8.7 -> 6.5 in complex64; 3 x 3 on 3^9 4.9 -> 4.3).
template <uint32_t BEGIN, uint32_t END, typename A>
__device__ __forceinline__ void warm_lines(A* a) {
  QD_KARG uint32_t* w = (QD_KARG uint32_t*)a;
  uint32_t t = w[END / 4 - 1];
#pragma unroll
  for (uint32_t i = BEGIN / 4; i < END / 4; i += 16) t ^= w[i];
  __asm__ volatile("" ::"s"(t));
}

// Amplitudes a thread moves per tile: the tile holds at most 256 * kTileEpt<R> amplitudes.
template <typename R> struct TileEpt;
template <> struct TileEpt<double> { static constexpr int value = 8; };
template <> struct TileEpt<float> { static constexpr int value = 16; };

template <typename OP> struct DenseDim { static constexpr int value = 0; };
template <typename R, int DT> struct DenseDim<DenseOp<R, DT>> { static constexpr int value = DT; };

template <typename R, int DT, typename OP, bool ST>
__global__ __launch_bounds__(256) void k_slices_tiled(TileArgs<R, DT, OP>) {
  using C = typename CxT<R>::T;
  constexpr int EPT = TileEpt<R>::value;
  constexpr bool kDense = DenseDim<OP>::value > 0;
  constexpr bool kRows = kDense && DT * sizeof(R) > 24;   // a row of U at a time (all of it would not fit the scalar registers)
  using Args = TileArgs<R, DT, OP>;
  QD_KARG Args* a = (QD_KARG Args*)__builtin_amdgcn_kernarg_segment_ptr();
  const bool cold = blockIdx.x < 1024;   // later workgroups find what their predecessors on the CU have read
  if (cold) warm_lines<0, offsetof(Args, op)>(a);
  extern __shared__ __align__(16) unsigned char lds_raw[];
  __shared__ int64_t s_hoff[kMaxTileRuns];
  C* lds = reinterpret_cast<C*>(lds_raw);
  C* __restrict__ psi = reinterpret_cast<C*>(a->psi);
  const uint32_t bs = blockDim.x, tid = threadIdx.x, BL = a->BL, E = BL * a->dH;
  const Magic32 blm = karg_magic(&a->blm), sc0 = karg_magic(&a->scm[0]), sc1 = karg_magic(&a->scm[1]);
  const uint32_t m0 = a->scmul[0], m1 = a->scmul[1], d0 = a->scadd[0], d1 = a->scadd[1];
  if (tid < kMaxTileRuns) s_hoff[tid] = a->hoff[tid];
  __syncthreads();
  // Offset of the staged amplitude idx from the tile's origin: its run, and the offset inside the run,
  // where each left-out control digit is re-inserted at its value, smallest stride first (w = q s + r
  // becomes q s d_c + v s + r; an entry of zeros inserts nothing).
  auto place = [&](uint32_t idx) {
    const uint32_t h = magic_div(idx, blm);
    uint32_t w = idx - h * BL;
    w += magic_div(w, sc0) * m0 + d0;
    w += magic_div(w, sc1) * m1 + d1;
    return s_hoff[h] + int64_t(w);
  };
  const bool whole = a->dH == 1 && a->nsc == 0;   // the tile is one run of the state
  // most gates insert one or two digits (an entry of zeros inserts nothing)
  const uint32_t nsl = a->nsl, nins = a->nins;
  const uint32_t i0m = a->ins[0].mul, i0s = a->ins[0].self, i0g = a->ins[0].grow, i0a = a->ins[0].add;
  const uint32_t i1m = a->ins[1].mul, i1s = a->ins[1].self, i1g = a->ins[1].grow, i1a = a->ins[1].add;
  const uint32_t ntiles = a->tiles.count;
  for (uint32_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    int64_t g0 = a->tiles.base;
    {
      uint32_t rem = tile;   // uniform: scalar arithmetic
      const uint32_t ng = a->tiles.ng;
      for (uint32_t g = 0; g < ng; ++g) {
        const uint32_t q = g + 1 < ng ? magic_div(rem, karg_magic(&a->tiles.gmag[g])) : 0u;
        g0 += int64_t(rem - q * a->tiles.gdim[g]) * a->tiles.gstride[g];
        rem = q;
      }
    }
    // The per-element indices are recomputed in the load and in the store stage from opaque copies of
    // the thread index: kept live across the LDS mix they would take about 3 EPT registers and cut the
    // workgroups per CU for the wider gates. Every load of the tile is issued before the first LDS write;
    // in a tile of one run none has a branch of its own (a lane past the end repeats the last amplitude),
    // which took a complex64 qubit gate on 2^25 amplitudes from 149 to 103 us. (In other tiles the addresses
    // held for that took the registers of a third of the waves: 295 -> 361 us.)
    // (real and imaginary parts in separate scalar arrays so they stay in registers)
    uint32_t tl = tid;
    __asm__ volatile("" : "+v"(tl));
    R vr[EPT], vi[EPT];
    C* __restrict__ p0 = psi + g0;
    // uniform base, 32-bit offset: one address register a load
    auto byte_at = [&](uint32_t idx) {
      return reinterpret_cast<C*>(reinterpret_cast<unsigned char*>(p0) + idx * uint32_t(sizeof(C)));
    };
    if (whole) {
#pragma unroll
      for (int e = 0; e < EPT; ++e)
        if (uint32_t(e) * bs < E) {
          const C t = get<ST>(byte_at(min(tl + e * bs, E - 1)));
          vr[e] = t.x;
          vi[e] = t.y;
        }
    } else {
#pragma unroll
      for (int e = 0; e < EPT; ++e)
        if (tl + e * bs < E) {
          const C t = get<ST>(p0 + place(tl + e * bs));
          vr[e] = t.x;
          vi[e] = t.y;
        }
    }
    if constexpr (kRows) {
      // U's, while the tile is on its way
      if (cold) warm_lines<offsetof(Args, op), offsetof(Args, op) + sizeof(OP)>(a);
    }
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      const uint32_t idx = tl + e * bs;
      if (idx < E) {
        C t;
        t.x = vr[e];
        t.y = vi[e];
        lds[idx] = t;
      }
    }
    __syncthreads();
#pragma unroll 1
    for (uint32_t j = tid; j < nsl; j += bs) {
      uint32_t b = j;
      b += (__umulhi(b, i0m) + (b & i0s)) * i0g + i0a;
      b += (__umulhi(b, i1m) + (b & i1s)) * i1g + i1a;
#pragma unroll 1
      for (uint32_t i = 2; i < nins; ++i) b += (__umulhi(b, a->ins[i].mul) + (b & a->ins[i].self)) * a->ins[i].grow + a->ins[i].add;
      C x[DT];
#pragma unroll
      for (int y = 0; y < DT; ++y) x[y] = lds[b + a->toff[y]];
      if constexpr (kDense) {
        auto row = [&](int r) {
          R re = R(0), im = R(0);
#pragma unroll
          for (int c = 0; c < DT; ++c) {
            const R ur = a->op.u[2 * (r * DT + c)], ui = a->op.u[2 * (r * DT + c) + 1];
            re = fma(ur, x[c].x, re);
            re = fma(-ui, x[c].y, re);
            im = fma(ur, x[c].y, im);
            im = fma(ui, x[c].x, im);
          }
          C yv;
          yv.x = re;
          yv.y = im;
          lds[b + a->toff[r]] = yv;
        };
        if constexpr (!kRows) {
#pragma unroll
          for (int r = 0; r < DT; ++r) row(r);
        } else {
#pragma unroll 1
          for (int r = 0; r < DT; ++r) row(r);
        }
      } else {
#pragma unroll
        for (int c = 0; c < DT; ++c) {
          const R pr = a->op.ph[2 * c], pi = a->op.ph[2 * c + 1];
          C y;
          y.x = fma(pr, x[c].x, -pi * x[c].y);
          y.y = fma(pr, x[c].y, pi * x[c].x);
          lds[b + a->doff[c]] = y;
        }
      }
    }
    __syncthreads();
    uint32_t ts = tid;
    __asm__ volatile("" : "+v"(ts));
#pragma unroll
    for (int e = 0; e < EPT; ++e)
      if (uint32_t(e) * bs < E) {
        const C t = lds[min(ts + e * bs, E - 1)];
        vr[e] = t.x;
        vi[e] = t.y;
      }
    auto put_back = [&](int e, C* p) {
      C t;
      t.x = vr[e];
      t.y = vi[e];
      put<ST>(p, 0, t);
    };
    if (whole) {
#pragma unroll
      for (int e = 0; e < EPT; ++e)
        if (ts + e * bs < E) put_back(e, byte_at(ts + e * bs));
    } else {
#pragma unroll
      for (int e = 0; e < EPT; ++e)
        if (ts + e * bs < E) put_back(e, p0 + place(ts + e * bs));
    }
    if (tile + gridDim.x < ntiles) __syncthreads();
  }
}

// ------------------------------------------------------------------------------------------ diagonal
template <typename R>
struct DiagArgs {
  R* psi;
  SliceMap sm;                     // over all non-control qudits; targets are singleton groups
  R ph[2 * kMaxInlineTable];       // phase of target combination loc
};

template <typename R, int SPT, bool ST>
__global__ __launch_bounds__(256) void k_diag(DiagArgs<R> a) {
  using C = typename CxT<R>::T;
  C* __restrict__ psi = reinterpret_cast<C*>(a.psi);
  const uint64_t bs = blockDim.x;
  const uint64_t first = uint64_t(blockIdx.x) * bs * SPT + threadIdx.x;
  int64_t off[SPT];
  uint32_t loc[SPT];
  C x[SPT];
#pragma unroll
  for (int s = 0; s < SPT; ++s) {
    const uint64_t i = first + s * bs;
    off[s] = i < a.sm.count ? sm_offset_loc(a.sm, uint32_t(i), &loc[s]) : -1;
  }
#pragma unroll
  for (int s = 0; s < SPT; ++s)
    if (off[s] >= 0) x[s] = get<ST>(psi + off[s]);
#pragma unroll
  for (int s = 0; s < SPT; ++s)
    if (off[s] >= 0) {
      const R pr = a.ph[2 * loc[s]], pi = a.ph[2 * loc[s] + 1];
      C y;
      y.x = fma(pr, x[s].x, -pi * x[s].y);
      y.y = fma(pr, x[s].y, pi * x[s].x);
      put<ST>(psi, off[s], y);
    }
}

// ------------------------------------------------------------------------------------------ generic
struct GenericHead {
  SliceMap64 sm;
  int32_t dT;
  int32_t nsw;        // slices per workgroup iteration
  // followed by int64_t toff[dT] and then 2 dT^2 values of R (U, row-major interleaved)
};

template <typename R>
__global__ __launch_bounds__(256) void k_dense_generic(R* psi_raw, const unsigned char* desc) {
  using C = typename CxT<R>::T;
  extern __shared__ __align__(16) unsigned char lds_raw[];
  C* xs = reinterpret_cast<C*>(lds_raw);
  const GenericHead& h = *reinterpret_cast<const GenericHead*>(desc);
  // the slice map is read into LDS before the first store (read later from global memory it would
  // be fetched again by vector loads, the stores could alias it)
  __shared__ SliceMap64 smap;
  static_assert(sizeof(SliceMap64) % 4 == 0, "slice map copied in 4-byte words");
  for (uint32_t i = threadIdx.x; i < sizeof(SliceMap64) / 4; i += blockDim.x)
    reinterpret_cast<uint32_t*>(&smap)[i] = reinterpret_cast<const uint32_t*>(&h.sm)[i];
  const int64_t* toff = reinterpret_cast<const int64_t*>(desc + sizeof(GenericHead));
  const R* U = reinterpret_cast<const R*>(desc + sizeof(GenericHead) + sizeof(int64_t) * h.dT);
  C* psi = reinterpret_cast<C*>(psi_raw);
  const uint32_t dT = uint32_t(h.dT), nsw = uint32_t(h.nsw), tot = dT * nsw;
  const uint64_t count = h.sm.count;
  __syncthreads();
  for (uint64_t s0 = uint64_t(blockIdx.x) * nsw; s0 < count; s0 += uint64_t(gridDim.x) * nsw) {
    for (uint32_t e = threadIdx.x; e < tot; e += blockDim.x) {
      const uint32_t j = e / dT, y = e - j * dT;
      if (s0 + j < count) xs[e] = ld_stream(psi + (sm64_offset(smap, s0 + j) + toff[y]));
    }
    __syncthreads();
    for (uint32_t e = threadIdx.x; e < tot; e += blockDim.x) {
      const uint32_t j = e / dT, row = e - j * dT;
      if (s0 + j >= count) continue;
      R re = R(0), im = R(0);
      const R* u = U + 2 * size_t(row) * dT;
      const C* x = xs + j * dT;
      for (uint32_t c = 0; c < dT; ++c) {
        re = fma(u[2 * c], x[c].x, re);
        re = fma(-u[2 * c + 1], x[c].y, re);
        im = fma(u[2 * c], x[c].y, im);
        im = fma(u[2 * c + 1], x[c].x, im);
      }
      C y;
      y.x = re;
      y.y = im;
      st_stream(psi + (sm64_offset(smap, s0 + j) + toff[row]), y);
    }
    __syncthreads();
  }
}

// ------------------------------------------------------------------------------------------ matrix cores
// Dense gates with d_T >= kGemmMin on registers below 2^32 amplitudes: per tile of ns slices,
// Y = U X as a complex GEMM on the matrix cores in the state's own precision (16x16x4 FP64 or FP32
// products: FP64 inputs and sums for complex128, FP32 for complex64; four products per complex one).
// Bound: HBM up to d_T of about 32, the matrix cores above (8 d_T flops per 2 x 16 bytes; 72 TFLOP/s
// FP64 as a large product reaches it on this card).
//   - X (all d_T amplitudes of ns slices) is staged in LDS once, pitch ns + 1 so that both loading
//     orders and the operand reads spread over the banks; every output of those slices is made by
//     this workgroup, so the results go from the accumulators straight back to HBM.
//   - The matrix cores sum the four products of a K step as a chain of fused multiply-adds in ascending K
//     (checked bit for bit against such chains in both precisions). complex64 takes two columns a step,
//     real and imaginary part by turns: every output is then the very sum that a thread of the
//     vector-unit kernels makes, column by column in listed order, and no bit of a complex64 state
//     depends on the kernel that a gate takes. Its operands cost twice the LDS reads, which is why
//     complex128, where the order moves a result by 1e-16, takes four columns a step: all their real
//     parts, then all their imaginary ones (4^12, d_T = 64 and 256: complex64 124 -> 141, 552 -> 702 us,
//     complex128 would go 187 -> 201, 842 -> 996).
//   - U is stored by the host in operand order (lane l of a K step holds row l & 15 and, in complex128,
//     column 4 k + (l >> 4), in complex64 one part of column 2 k + (l >> 5)), one coalesced load per
//     lane and step, four steps ahead. It is read from L2 by every workgroup: at 16 slices or more per
//     tile that is at most 1 KB per 256 matrix-core cycles of a SIMD. So U takes no LDS and d_T is
//     bounded by X alone.
//   - A job is one 16-row tile of U times CG column tiles; the waves of a workgroup share them.
// The operands of a product may change places, which transposes the result: with kMfmaYF the 16
// consecutive lanes of a store hold consecutive target combinations (a target has the smallest
// stride) instead of consecutive slices, so both kinds of gate store runs.
// Measured, complex128 (kernel time; before: a vector-unit GEMM with U and X in LDS up to d_T = 64,
// above it a kernel that read U from L2 for every product): on 3^14 amplitudes d_T = 27 76 -> 49 us,
// 81 880 -> 92 us, 243 5220 -> 195 us (48 TFLOP/s); on 4^12 amplitudes d_T = 64 360 -> 189 us, 256
// 16.4 -> 0.60 ms (57 TFLOP/s); on the hybrid register of 1.1e8 amplitudes d_T = 27 1083 -> 757 us
// (4.5 TB/s), 54 2160 -> 1119 us. complex64 on 4^12: 64 205 -> 141 us, 256 15.2 -> 0.70 ms.
// Lines that belong to several runs (a target or control stride that is no multiple of a line) are read
// and written with plain accesses, so that the cache merges their parts: streaming stores cost up to a
// line each (d_T = 27 on 3^16, lowest targets of stride 3, 27 and 3^13: complex64 464, 384, 249 -> 236,
// 233, 225 us, complex128 480, 450, 410 -> 367, 348, 341). Whole lines stream: 395 against 413 us for
// d_T = 64 with stride 16 on 4^13 in complex64, 774 against 823 for d_T = 27 on the hybrid register.
constexpr int kGemmMin = 10;
constexpr int kGemmMax = 64;

struct MfmaArgs {
  SliceMap sm;                        // slices: the non-target digits (controls fixed)
  Magic32 div;                        // division by ns, or by KP when target combinations are fastest
  uint32_t dT, KP, RT, ns, njobs;     // KP: d_T rounded up to whole K steps; RT: 16-row tiles of U; jobs per tile
  const unsigned char* desc;          // uint64_t[d_T], by ascending offset: the offset and (upper half) the
                                      // column; then (16-byte aligned) RT x K steps x 64 entries of U in operand order
};

template <typename R> struct Mfma16;
template <> struct Mfma16<double> {
  typedef double V4 __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ V4 mul(double a, double b, V4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
  static __device__ __forceinline__ uint32_t row(uint32_t i, uint32_t q) { return 4u * i + q; }
};
template <> struct Mfma16<float> {
  typedef float V4 __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ V4 mul(float a, float b, V4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
  static __device__ __forceinline__ uint32_t row(uint32_t i, uint32_t q) { return 4u * q + i; }
};

enum { kMfmaYF, kMfmaLines, kMfmaParts };
template <typename R> constexpr uint32_t kMfmaStep = sizeof(R) == 8 ? 4 : 2;   // columns of U a K step

template <typename R, int CG, int MODE>
__global__ __launch_bounds__(1024) void k_dense_mfma(R* psi_raw, MfmaArgs a) {
  using C = typename CxT<R>::T;
  using M = Mfma16<R>;
  using V4 = typename M::V4;
  constexpr bool YF = MODE == kMfmaYF;
  extern __shared__ __align__(16) unsigned char lds_raw[];
  C* __restrict__ psi = reinterpret_cast<C*>(psi_raw);
  const uint32_t dT = a.dT, KP = a.KP, ns = a.ns, P = ns + 1, bs = blockDim.x, tid = threadIdx.x;
  C* xs = reinterpret_cast<C*>(lds_raw);                        // KP x ns, element (y, j) at y P + j
  int64_t* sb = reinterpret_cast<int64_t*>(xs + KP * P + (KP * P & 1u));   // ns slice bases
  uint64_t* to = reinterpret_cast<uint64_t*>(sb + ns);          // d_T target offsets (low half) and columns
  const uint64_t* tg = reinterpret_cast<const uint64_t*>(a.desc);
  // an entry of U in operand order: both parts of one column, or one part (kMfmaStep columns a step)
  using U = typename std::conditional<kMfmaStep<R> == 4, C, R>::type;
  const U* ug = reinterpret_cast<const U*>(a.desc + ((sizeof(int64_t) * dT + 15) & ~size_t(15)));
  const uint32_t s0 = blockIdx.x * ns, nsv = min(ns, a.sm.count - s0);   // nsv: slices of this tile
  // a column past the last slice repeats it (read, multiplied and not stored): no load is conditional
  for (uint32_t j = tid; j < ns; j += bs) sb[j] = sm_offset(a.sm, s0 + min(j, nsv - 1));
  for (uint32_t i = tid; i < dT; i += bs) to[i] = tg[i];
  __syncthreads();
  constexpr int B = 8;   // loads in flight per thread
  const uint32_t tot = KP * ns;
  for (uint32_t e0 = tid; e0 < tot; e0 += B * bs) {
    C v[B];
    uint32_t at[B];
    int64_t off[B];
    bool pad[B];
#pragma unroll
    for (int k = 0; k < B; ++k) {
      const uint32_t e = min(e0 + uint32_t(k) * bs, tot - 1);   // past the end: the last element again
      const uint32_t q = magic_div(e, a.div), r = e - q * a.div.d;
      const uint32_t y = YF ? r : q, j = YF ? q : r;
      pad[k] = y >= dT;
      const uint64_t t = to[pad[k] ? dT - 1 : y];
      at[k] = (pad[k] ? y : uint32_t(t >> 32)) * P + j;
      off[k] = sb[j] + uint32_t(t);
    }
#pragma unroll
    for (int k = 0; k < B; ++k) v[k] = MODE == kMfmaParts ? psi[off[k]] : ld_stream(psi + off[k]);
#pragma unroll
    for (int k = 0; k < B; ++k) {
      if (pad[k]) v[k].x = v[k].y = R(0);
      xs[at[k]] = v[k];
    }
  }
  __syncthreads();
  const uint32_t lane = tid & 63u, lq = lane >> 4, lr = lane & 15u, nw = bs >> 6;
  const uint32_t KS = KP / kMfmaStep<R>;
  for (uint32_t job = tid >> 6; job < a.njobs; job += nw) {   // wave-uniform
    const uint32_t cj = job / a.RT, rt = job - cj * a.RT;
    const U* up = ug + size_t(rt) * KS * 64 + lane;
    const C* xp = xs + (kMfmaStep<R> == 4 ? lq : lq >> 1) * P + cj * (16u * CG) + lr;
    V4 re[CG], im[CG];
#pragma unroll
    for (int g = 0; g < CG; ++g) {
      re[g] = V4{R(0), R(0), R(0), R(0)};
      im[g] = re[g];
    }
    constexpr uint32_t N = 4;
    auto ldu = [&](U (&u)[N], uint32_t k0) {   // N steps of U (past the last one: that one again)
#pragma unroll
      for (uint32_t k = 0; k < N; ++k) u[k] = up[64 * min(k0 + k, KS - 1)];
    };
    auto mul = [&](R u, R x, V4 c) { return YF ? M::mul(x, u, c) : M::mul(u, x, c); };
    auto step = [&](U u, uint32_t ks) {
      C x[CG];
#pragma unroll
      for (int g = 0; g < CG; ++g) x[g] = xp[ks * kMfmaStep<R> * P + 16 * g];
      if constexpr (kMfmaStep<R> == 4) {
#pragma unroll
        for (int g = 0; g < CG; ++g) {
          re[g] = mul(u.x, x[g].x, re[g]);
          im[g] = mul(u.x, x[g].y, im[g]);
        }
#pragma unroll
        for (int g = 0; g < CG; ++g) {
          re[g] = mul(-u.y, x[g].y, re[g]);
          im[g] = mul(u.y, x[g].x, im[g]);
        }
      } else {
        const bool odd = (lq & 1u) != 0;   // this lane holds an imaginary part of U
        const R v = odd ? -u : u;
#pragma unroll
        for (int g = 0; g < CG; ++g) {
          re[g] = mul(v, odd ? x[g].y : x[g].x, re[g]);
          im[g] = mul(u, odd ? x[g].x : x[g].y, im[g]);
        }
      }
    };
    auto many = [&](const U (&u)[N], uint32_t k0) {
#pragma unroll
      for (uint32_t k = 0; k < N; ++k)
        if (k0 + k < KS) step(u[k], k0 + k);
    };
    U ua[N], ub[N];
    ldu(ua, 0);
    for (uint32_t ks = 0; ks < KS; ks += 2 * N) {
      ldu(ub, ks + N);
      many(ua, ks);
      ldu(ua, ks + 2 * N);
      many(ub, ks + N);
    }
    // lane lr of a store holds consecutive slices (or consecutive target combinations): the four rows
    // of a register tile are four stores
    int64_t ro[4];
    bool rv[4];
#pragma unroll
    for (uint32_t i = 0; i < 4; ++i) {
      const uint32_t y = rt * 16u + (YF ? lr : M::row(i, lq));
      rv[i] = y < dT;
      ro[i] = uint32_t(to[min(y, dT - 1)]);
    }
#pragma unroll
    for (int g = 0; g < CG; ++g) {
      const uint32_t c0 = (cj * CG + uint32_t(g)) * 16u;
#pragma unroll
      for (uint32_t i = 0; i < 4; ++i) {
        const uint32_t j = c0 + (YF ? M::row(i, lq) : lr);
        const int64_t o = sb[min(j, ns - 1)] + ro[i];
        C v;
        v.x = re[g][i];
        v.y = im[g][i];
        if (rv[i] && j < nsv) {
          // runs of target combinations end inside lines too
          if constexpr (MODE == kMfmaLines) st_stream(psi + o, v);
          else psi[o] = v;
        }
      }
    }
  }
}

// ------------------------------------------------------------------------------------------ launch helpers
// Name of the kernel instance the calling thread's last gate launch used (qd_last_kernel).
static thread_local const char* g_last_kernel = "";

template <typename R> constexpr const char* real_name() { return sizeof(R) == 8 ? "double" : "float"; }
template <typename OP> struct OpName;
template <typename R, int DT> struct OpName<DenseOp<R, DT>> { static constexpr const char* value = "DenseOp"; };
template <typename R, int DT> struct OpName<MonoOp<R, DT>> { static constexpr const char* value = "MonoOp"; };

// "<kernel><R, DT[, Op<R, DT>][, SPT, mode]>", formatted once per instance
enum { kKnDirect, kKnTiled, kKnDiag, kKnGeneric, kKnGemm, kKnLu };
template <int KIND, typename R, int DT = 0, typename OP = void, int SPT = 0, int MODE = 0>
static const char* label() {
  static thread_local char buf[160] = {0};
  if (!buf[0]) {
    static const char* kn[] = {"k_slices_direct", "k_slices_tiled", "k_diag", "k_dense_generic", "k_dense_mfma",
                               "k_slices_direct_lu"};
    static const char* modes[] = {"plain", "pred", "edge"};
    const char* rn = real_name<R>();
    if constexpr (KIND == kKnDirect)
      std::snprintf(buf, sizeof(buf), "%s<%s, %d, %s<%s, %d>, %d, %s>", kn[KIND], rn, DT, OpName<OP>::value, rn, DT, SPT,
                    modes[MODE]);
    else if constexpr (KIND == kKnTiled)
      std::snprintf(buf, sizeof(buf), "%s<%s, %d, %s<%s, %d>>", kn[KIND], rn, DT, OpName<OP>::value, rn, DT);
    else if constexpr (KIND == kKnLu)
      std::snprintf(buf, sizeof(buf), "%s<%s, %d>", kn[KIND], rn, DT);
    else
      std::snprintf(buf, sizeof(buf), "%s<%s>", kn[KIND], rn);
  }
  return buf;
}

static inline unsigned grid_for(uint64_t items, uint64_t per_block) {
  const uint64_t g = (items + per_block - 1) / per_block;
  return unsigned(std::max<uint64_t>(1, g));
}

static int check_launch(const char* what) {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, what);
  return QD_OK;
}

// Which lines of `line` amplitudes hold an amplitude where every control of stride below one line
// has its value. Those control digits repeat with period P = lcm(s_c d_c), so the lines repeat with
// period lcm(P, line) / line; for a period of 2..64 lines, *per is set to it and bit j of *mask
// tells whether line j of a period holds such an amplitude (else *per = 1: treat every line so).
static void line_pattern(const Register& r, const GatePlan& p, int64_t line, uint32_t* per, uint64_t* mask) {
  *per = 1;
  *mask = 1;
  uint64_t P = 1;
  for (int j = 0; j < p.m; ++j) {
    const int c = p.controls[j];
    if (r.strides[c] < line) P = std::lcm(P, uint64_t(r.strides[c]) * uint64_t(r.dims[c]));
  }
  const uint64_t per_lines = std::lcm(P, uint64_t(line)) / uint64_t(line);
  if (per_lines < 2 || per_lines > 64) return;
  uint64_t m = 0;
  for (uint64_t L = 0; L < per_lines; ++L)
    for (uint64_t i = L * uint64_t(line); i < (L + 1) * uint64_t(line); ++i) {
      bool all = true;
      for (int j = 0; j < p.m && all; ++j) {
        const int c = p.controls[j];
        if (r.strides[c] < line) all = (i / uint64_t(r.strides[c])) % uint64_t(r.dims[c]) == uint64_t(p.cvals[j]);
      }
      if (all) {
        m |= uint64_t(1) << L;
        break;
      }
    }
  if (m == (per_lines == 64 ? ~uint64_t(0) : (uint64_t(1) << per_lines) - 1)) return;   // every line
  *per = uint32_t(per_lines);
  *mask = m;
}

// target offsets: y in mixed radix over the targets in listed order, t_0 most significant
static void target_offsets(const Register& r, const GatePlan& p, int64_t* toff) {
  for (int y = 0; y < p.dT; ++y) {
    int rem = y;
    int64_t off = 0;
    for (int j = p.k - 1; j >= 0; --j) {
      const int d = r.dims[p.targets[j]];
      off += int64_t(rem % d) * r.strides[p.targets[j]];
      rem /= d;
    }
    toff[y] = off;
  }
}

template <typename R, int DT>
static void fill_dense(const GatePlan& p, DenseOp<R, DT>* op) {
  for (int i = 0; i < 2 * DT * DT; ++i) op->u[i] = R(p.U[i]);
}
template <typename R, int DT>
static void fill_mono(const GatePlan& p, MonoOp<R, DT>* op) {
  for (int i = 0; i < DT; ++i) {
    op->dst[i] = p.dst[i];
    op->ph[2 * i] = R(p.ph[2 * i]);
    op->ph[2 * i + 1] = R(p.ph[2 * i + 1]);
  }
}

// LDS tile geometry: the low suffix L = {pq, ..., n-1} of the register holds every target whose
// stride is below run_min and is grown towards longer contiguous runs while the tile (dH runs of
// BL amplitudes) fits the LDS budget. Controls inside L (at most kMaxTileCtl; their strides are at
// least one 128-byte line, smaller ones having been folded into the targets) are left out of the
// tile: it stages only the amplitudes whose control digits match, so a control that falls inside
// L costs 1/d_c of a pass as it does above L. Returns false when no target is low (the direct
// kernel applies) or the tile would not fit.
bool tile_geometry(const Register& r, const GatePlan& p, int prec, TileGeom* g) {
  const TuneParams& tp = tune();
  int64_t min_stride = INT64_MAX;
  int min_t = -1;
  for (int j = 0; j < p.k; ++j)
    if (r.strides[p.targets[j]] < min_stride) {
      min_stride = r.strides[p.targets[j]];
      min_t = p.targets[j];
    }
  const TuneEntry e = entry_for(prec, min_stride);
  if (!e.tiled) return false;
  {
    // Controls inside a line that leave whole lines without a matching amplitude: the predicated
    // direct kernel skips those lines and the tile kernel would move them. With every target at
    // least a line apart the direct kernel's lanes still take whole lines, so it runs such gates.
    const int64_t line = prec == QD_C128 ? 8 : 16;
    uint32_t per = 1;
    uint64_t mask = 1;
    if (min_stride >= line) line_pattern(r, p, line, &per, &mask);
    if (per > 1) return false;
  }
  int low_idx = min_t;
  for (int j = 0; j < p.k; ++j)
    if (r.strides[p.targets[j]] < tp.run_min) low_idx = std::min(low_idx, int(p.targets[j]));
  const uint64_t ept = prec == QD_C128 ? TileEpt<double>::value : TileEpt<float>::value;
  const uint64_t emax = std::min<uint64_t>(uint64_t(e.tile_elems) * (prec == QD_C128 ? 1u : 2u),
                                           uint64_t(e.block) * ept);
  const int64_t line = prec == QD_C128 ? 8 : 16;   // amplitudes per 128-byte line
  bool is_t[QD_MAX_QUDITS] = {}, is_c[QD_MAX_QUDITS] = {};
  for (int j = 0; j < p.k; ++j) is_t[p.targets[j]] = true;
  for (int j = 0; j < p.m; ++j) is_c[p.controls[j]] = r.strides[p.controls[j]] >= line;
  auto grow = [&](bool compact) -> bool {
    int pq = low_idx, nsc = 0;
    uint64_t BL = 1, dH = 1;
    for (int i = pq; i < r.n; ++i) {
      if (compact && is_c[i]) ++nsc;
      else BL *= uint64_t(r.dims[i]);
    }
    if (nsc > kMaxTileCtl) return false;
    for (int i = 0; i < pq; ++i)
      if (is_t[i]) dH *= r.dims[i];
    // A tuned tile or one that the caller has set is filled. Otherwise growth stops at 9 KB: more, smaller
    // tiles keep the memory system busier than few large ones (complex128: 648 against 1296 amplitudes 565
    // and 615 us on the hybrid register of 1.1e8, 1024 against 2048 178 and 197 us on 2^25), while tiles
    // below that size leave the workgroups short of loads (243 against 729 amplitudes 384 and 243 us on
    // 3^16; complex64: 729 against 2187 221 and 132 us).
    // A register of fewer than 192 tiles of that size (of 256 CUs) takes smaller ones, down to one amplitude
    // a thread: complex64, radix 8 on 2^15 amplitudes 7.2 -> 5.2 us with 64 tiles instead of 8, 9 x 9 gates on
    // 3^9 6.4 -> 6.0; tiles of 64 amplitudes are slower again (5.7 and 6.1).
    const bool fill = e.tuned || tp.tile_elems_set;
    const uint64_t enough = fill ? emax : 9216 / amp_bytes(prec);
    while (pq > 0 && BL * dH < enough) {
      const int q = pq - 1;
      const bool drop = compact && is_c[q];
      if (drop && nsc == kMaxTileCtl) break;
      const uint64_t nBL = drop ? BL : BL * r.dims[q];
      const uint64_t ndH = is_t[q] ? dH / r.dims[q] : dH;
      if (nBL * ndH > emax) break;
      if (!fill && BL * dH >= 256 && nBL * ndH * 192 > uint64_t(r.D)) break;
      pq = q;
      BL = nBL;
      dH = ndH;
      nsc += drop ? 1 : 0;
    }
    if (dH > uint64_t(kMaxTileRuns) || BL * dH > emax) return false;
    g->pq = pq;
    g->BL = BL;
    g->dH = dH;
    g->nsc = 0;
    for (int i = r.n - 1; i >= pq && compact; --i)
      if (is_c[i]) g->sc[g->nsc++] = i;
    return true;
  };
  return grow(true) || grow(false);
}

// The route of a gate; *g is its tile where that is QD_ROUTE_TILED.
static int route_gate(const Register& r, int prec, const GatePlan& p, TileGeom* g) {
  const bool fast = uint64_t(r.D) <= 0xFFFFFFFFull;
  if (!fast) return QD_ROUTE_GENERIC;
  if (p.cls == QD_CLASS_DIAGONAL && p.dT <= kMaxInlineTable) return QD_ROUTE_DIAG;
  const bool mono = p.cls == QD_CLASS_MONOMIAL &&
                    (p.dT <= 9 || p.dT == 12 || p.dT == 16);
  const bool dense = p.cls != QD_CLASS_DIAGONAL && p.dT <= kMaxInlineDense;
  if (!mono && !dense) {
    if (p.dT < kGemmMin || p.dT > kGemmMax) return QD_ROUTE_GENERIC;
    // d_T = 12 or 16 with every target stride at or above the tiling threshold: one slice per thread
    if (p.dT == 12 || p.dT == 16) {
      int64_t tmin = INT64_MAX;
      for (int j = 0; j < p.k; ++j) tmin = std::min<int64_t>(tmin, r.strides[p.targets[j]]);
      if (tmin >= tune().run_min) return QD_ROUTE_DIRECT;
    }
    return QD_ROUTE_GEMM;
  }
  return tile_geometry(r, p, prec, g) ? QD_ROUTE_TILED : QD_ROUTE_DIRECT;
}

int route_gate(const Register& r, int prec, const GatePlan& p) {
  TileGeom g;
  return route_gate(r, prec, p, &g);
}

template <int DT>
static void fill_doff(const GatePlan& p, const int64_t* toff, int64_t* doff) {
  for (int c = 0; c < DT; ++c) doff[c] = p.dst.empty() ? 0 : toff[p.dst[c]];
}

// Whether a pass goes by the caches (streaming loads and stores) or leaves its lines in them.
//   - Touched amplitudes of at most 256 MB (the size of the card's last-level cache) stay there for the
//     next pass: plain accesses win 4 to 20 % (complex128: a qubit of 2^24 94 -> 86 us, pairs 106 -> 88,
//     qutrits of 3^15 90 to 102 -> 77 to 79; complex64: 2^25 97 -> 89, 3^15 50 to 59 -> 44) and lose as
//     much right above it (2^25 complex128 175 -> 190, 2^26 complex64 180 -> 196). Passes of 32 MB or
//     less stay streaming: what the L2s (8 x 4 MB) hold is written back at the end of each kernel
//     anyway, and 2^20 in complex128 lost 1 to 2 of 14 us.
//   - Above it, one slice a thread whose planes begin inside 64-byte sectors: the ends of a wave's runs
//     share sectors with the next wave's, and a streaming store of part of one costs a whole one.
//     complex64, where a wave writes 512 bytes, always wins by plain accesses (9 x 9 gates on 3^17 475
//     and 533 -> 404 and 395 us, a unit of 7^9 148 -> 120). complex128 wins up to strides of 512 and not
//     above, over 150 gates on thirteen registers: plain against streaming 0.79 to 0.95 at 18 to 125, 0.96 to
//     1.03 at 243 and 343, 0.98 to 1.07 at 625 to 3675, up to 1.13 above (3^16, stride 27, 9 x 9 308 -> 256 us;
//     stride 729 246 -> 262). Above 2 GB the caches hold the shared sectors for less: 0.94 and 1.01 at 49 and
//     25, but 1.06 and 1.07 at 343 and 125 (7^10 1922 -> 2032 us, 5^12 1674 -> 1797).
static bool streaming(const qd_state* s, const GatePlan& p, uint64_t touched, bool direct) {
  const uint64_t amp = uint64_t(amp_bytes(s->prec));
  if (touched * amp <= uint64_t(32) << 20) return true;
  if (touched * amp <= uint64_t(256) << 20) return false;
  if (!direct) return true;
  bool sectors = true;
  int64_t lowest = INT64_MAX;
  for (int j = 0; j < p.k + p.m; ++j) {
    const int64_t st = s->reg.strides[j < p.k ? p.targets[j] : p.controls[j - p.k]];
    sectors = sectors && uint64_t(st) * amp % 64 == 0;
    lowest = std::min(lowest, st);
  }
  return sectors || (s->prec == QD_C128 && lowest > (touched * amp > uint64_t(2) << 30 ? 64 : 512));
}

// tile: the tile of a gate of route QD_ROUTE_TILED, else null
template <typename R, int DT, typename OP>
static int launch_slices(qd_state* s, const GatePlan& p, const OP& op, const TileGeom* tile) {
  const Register& r = s->reg;
  const TuneParams& tp = tune();
  int role[QD_MAX_QUDITS] = {};
  for (int j = 0; j < p.k; ++j) role[p.targets[j]] = 1;
  for (int j = 0; j < p.m; ++j) role[p.controls[j]] = 1;

  int64_t min_stride = INT64_MAX;
  for (int j = 0; j < p.k; ++j) min_stride = std::min<int64_t>(min_stride, r.strides[p.targets[j]]);
  const TuneEntry ent = entry_for(s->prec, min_stride);
  if (tile) {
    const TileGeom& tg = *tile;
    const int pq = tg.pq;
    const uint64_t BL = tg.BL, dH = tg.dH;
    {
      TileArgs<R, DT, OP> a;
      std::memset(&a, 0, sizeof(a));
      a.psi = reinterpret_cast<R*>(s->data);
      a.op = op;
      a.BL = uint32_t(BL);
      a.dH = uint32_t(dH);
      a.blm = make_magic32(uint32_t(BL));
      // LDS strides of the suffix: the register's, with the left-out controls' digits removed
      bool out[QD_MAX_QUDITS] = {};
      for (int j = 0; j < tg.nsc; ++j) out[tg.sc[j]] = true;
      Register lr = r;
      {
        int64_t st = 1;
        for (int i = r.n - 1; i >= pq; --i) {
          lr.strides[i] = st;
          if (!out[i]) st *= r.dims[i];
        }
      }
      int64_t tbase = 0, ibase = 0;
      for (int j = 0; j < p.m; ++j) {
        const int c = p.controls[j];
        if (c < pq) tbase += int64_t(p.cvals[j]) * r.strides[c];
        else if (!out[c]) ibase += int64_t(p.cvals[j]) * lr.strides[c];
      }
      a.nsc = uint32_t(tg.nsc);
      for (int j = 0; j < tg.nsc; ++j) {
        const int c = tg.sc[j];
        int v = 0;
        for (int q = 0; q < p.m; ++q)
          if (p.controls[q] == c) v = p.cvals[q];
        a.scm[j] = make_magic32(uint32_t(r.strides[c]));
        a.scmul[j] = uint32_t(r.strides[c] * (r.dims[c] - 1));
        a.scadd[j] = uint32_t(int64_t(v) * r.strides[c]);
      }
      int rc = fill_slicemap(make_groups(r, role, nullptr, 0, pq), tbase, &a.tiles);
      if (rc) return rc;
      // the suffix's free digits, held to the limits of a slice map
      SliceMap inner;
      rc = fill_slicemap(make_groups(lr, role, nullptr, pq, r.n), ibase, &inner);
      if (rc) return rc;
      a.nsl = inner.count;
      // run offsets: h in mixed radix over the high targets in listed order
      int hmul[QD_MAX_QUDITS] = {};
      {
        int m = 1;
        for (int j = p.k - 1; j >= 0; --j)
          if (p.targets[j] < pq) {
            hmul[j] = m;
            m *= r.dims[p.targets[j]];
          }
      }
      for (uint32_t h = 0; h < a.dH; ++h) {
        int64_t off = 0;
        for (int j = 0; j < p.k; ++j)
          if (p.targets[j] < pq) off += int64_t((h / hmul[j]) % r.dims[p.targets[j]]) * r.strides[p.targets[j]];
        a.hoff[h] = off;
      }
      for (int y = 0; y < DT; ++y) {
        int rem = y;
        int64_t off = 0;
        for (int j = p.k - 1; j >= 0; --j) {
          const int t = p.targets[j];
          const int dg = rem % r.dims[t];
          rem /= r.dims[t];
          off += t < pq ? int64_t(dg) * hmul[j] * int64_t(BL) : int64_t(dg) * lr.strides[t];
        }
        a.toff[y] = uint32_t(off);
      }
      for (int c = 0; c < DT; ++c) a.doff[c] = p.dst.empty() ? 0 : a.toff[p.dst[c]];
      // a slice: the suffix's digits, targets at 0 and controls at their values (run 0 of the high targets)
      for (int i = r.n - 1; i >= pq; --i) {
        if (out[i] || role[i] == 0) continue;
        int v = 0;
        for (int j = 0; j < p.m; ++j)
          if (p.controls[j] == i) v = p.cvals[j];
        a.ins[a.nins++] = make_insert(uint32_t(lr.strides[i]), uint32_t(r.dims[i]), uint32_t(v));
      }
      if (a.tiles.count == 0 || a.nsl == 0) return QD_OK;
      const size_t lds = size_t(BL * dH) * sizeof(R) * 2;
      // workgroups walk the tiles; at most 2^22 of them keep the grid inside 32-bit work-item counts
      const unsigned grid = unsigned(std::min<uint64_t>(a.tiles.count, uint64_t(1) << 22));
      if (streaming(s, p, a.tiles.count * BL * dH, false))
        hipLaunchKernelGGL((k_slices_tiled<R, DT, OP, true>), dim3(grid), dim3(ent.block), lds, s->stream, a);
      else
        hipLaunchKernelGGL((k_slices_tiled<R, DT, OP, false>), dim3(grid), dim3(ent.block), lds, s->stream, a);
      g_last_kernel = label<kKnTiled, R, DT, OP>();
      return check_launch("k_slices_tiled");
    }
  }

  // ---- direct: one slice per thread
  DirectArgs<R, DT, OP> a;
  std::memset(&a, 0, sizeof(a));
  a.psi = reinterpret_cast<R*>(s->data);
  a.op = op;
  const int64_t line = LineAmps<R>::value;
  // controls below one line are free digits of the slice map, tested per slice (kDirectPred)
  uint32_t lmul[QD_MAX_QUDITS] = {};
  int nlow = 0, c0 = -1;
  {
    uint32_t w = 1;
    for (int j = p.m - 1; j >= 0; --j) {
      const int c = p.controls[j];
      if (r.strides[c] < line) {
        role[c] = 2;
        lmul[c] = w;
        a.vloc += uint32_t(p.cvals[j]) * w;
        w *= uint32_t(r.dims[c]);
        ++nlow;
      } else if (c0 < 0 || r.strides[c] < r.strides[c0]) {
        c0 = c;
      }
    }
  }
  int64_t base = 0;
  for (int j = 0; j < p.m; ++j)
    if (role[p.controls[j]] == 1) base += int64_t(p.cvals[j]) * r.strides[p.controls[j]];
  int rc = fill_slicemap(make_groups(r, role, nlow ? lmul : nullptr, 0, r.n), base, &a.sm);
  if (rc) return rc;
  target_offsets(r, p, a.toff);
  fill_doff<DT>(p, a.toff, a.doff);
  if (a.sm.count == 0) return QD_OK;
  int bs = ent.block, spt = ent.spt;
  // Untuned complex128 gates of d_T <= 4 whose planes all begin on a line: with target strides of 4096
  // or more workgroups of one wave, one slice a thread (537 against 593 us for a qubit of the hybrid
  // register, 333 against 371 on 2^26; two slices for d_T = 4, where one lost up to 14 % at the highest
  // strides of 4^13: 375 to 414 against 400 to 409 us with 256 threads), with strides of 256 to 4095 128
  // threads (587 against 606). Where runs begin inside lines (3^16) each workgroup shares the lines at its
  // ends with others, and larger ones stay ahead (271 against 289 us). On what the caches hold the smaller
  // workgroups only add launches: they lose below 32 MB touched for a qubit (2^21 with a control, 16 MB: 6.2
  // against 8.2 us; 2^21, 32 MB: 13.1 against 12.0) and below 64 MB for d_T = 3 (38 MB: 9.9 against 12.1) and 4
  // (16 MB: 6.4 against 8.0; 64 MB: 21.0 against 18.6), but for d_T = 4 with strides of 256 to 4095 (2^21 with
  // a control 7.6 against 5.7, without 11.4 against 11.9).
  const uint64_t touched = uint64_t(a.sm.count) * DT * sizeof(R) * 2;
  const bool large = touched >= uint64_t(DT == 2 ? 32 : 64) << 20 || (DT == 4 && min_stride < 4096);
  if (!ent.tuned && !tp.direct_block_set && !tp.direct_spt_set && DT <= 4 && s->prec == QD_C128 && min_stride >= 256 &&
      large) {
    bool lines = true;
    for (int j = 0; j < p.k; ++j) lines = lines && r.strides[p.targets[j]] % line == 0;
    for (int j = 0; j < p.m; ++j) lines = lines && r.strides[p.controls[j]] % line == 0;
    if (lines) {
      bs = min_stride >= 4096 ? 64 : 128;
      spt = min_stride >= 4096 && DT < 4 ? 1 : 2;
    }
  }
  const bool st = streaming(s, p, uint64_t(a.sm.count) * DT, nlow == 0);
  auto launch = [&](auto k, uint64_t items, uint64_t per_thread) {
    hipLaunchKernelGGL(k, dim3(grid_for(items, uint64_t(bs) * per_thread)), dim3(bs), 0, s->stream, a);
  };
  if (nlow) {
    line_pattern(r, p, line, &a.lper, &a.lmask);
    if (a.lper > 1) a.lpm = make_magic32(a.lper);
    if (st) launch(k_slices_direct<R, DT, OP, 1, kDirectPred, true>, a.sm.count, 1);
    else launch(k_slices_direct<R, DT, OP, 1, kDirectPred, false>, a.sm.count, 1);
    g_last_kernel = label<kKnDirect, R, DT, OP, 1, kDirectPred>();
    return check_launch("k_slices_direct");
  }
  // the lowest control's active runs end inside lines: edge lanes rewrite the rest of those lines
  bool above = c0 >= 0;
  for (int j = 0; j < p.k && above; ++j) above = r.strides[p.targets[j]] > r.strides[c0];
  if (above && r.strides[c0] % line != 0) {
    const int64_t sc = r.strides[c0];
    uint64_t nA = 1;   // every qudit below the control is free (the targets are above it)
    for (int i = r.n - 1; i >= 0 && r.strides[i] < sc; --i) nA *= uint64_t(r.dims[i]);
    const uint64_t nblk = a.sm.count / nA;
    const uint64_t W = (uint64_t(sc) + 2 * uint64_t(line) - 2) / uint64_t(line) * uint64_t(line);   // lines a block can touch
    if (nblk * nA == a.sm.count && nblk * W <= 0xFFFFFFFFull) {
      a.nA = uint32_t(nA);
      a.W = uint32_t(W);
      a.wm = make_magic32(uint32_t(W));
      a.blen = uint32_t(sc);
      a.nvirt = uint32_t(nblk * W);
      a.D = r.D;
      // (its edge lanes complete the lines, so only the touched size decides)
      if (streaming(s, p, uint64_t(a.sm.count) * DT, false)) launch(k_slices_direct<R, DT, OP, 1, kDirectEdge, true>, a.nvirt, 1);
      else launch(k_slices_direct<R, DT, OP, 1, kDirectEdge, false>, a.nvirt, 1);
      g_last_kernel = label<kKnDirect, R, DT, OP, 1, kDirectEdge>();
      return check_launch("k_slices_direct");
    }
  }
  // Several slices per thread only up to d_T = 4: beyond, two slices' operands and the gate's
  // kernel arguments overflow the scalar registers and the spilled values are read back per FMA.
  if (spt >= 4 && DT <= 4) {
    if (st) launch(k_slices_direct<R, DT, OP, 4, kDirectPlain, true>, a.sm.count, 4);
    else launch(k_slices_direct<R, DT, OP, 4, kDirectPlain, false>, a.sm.count, 4);
    g_last_kernel = label<kKnDirect, R, DT, OP, 4, kDirectPlain>();
  } else if (spt >= 2 && DT <= 4) {
    if (st) launch(k_slices_direct<R, DT, OP, 2, kDirectPlain, true>, a.sm.count, 2);
    else launch(k_slices_direct<R, DT, OP, 2, kDirectPlain, false>, a.sm.count, 2);
    g_last_kernel = label<kKnDirect, R, DT, OP, 2, kDirectPlain>();
  } else {
    if (st) launch(k_slices_direct<R, DT, OP, 1, kDirectPlain, true>, a.sm.count, 1);
    else launch(k_slices_direct<R, DT, OP, 1, kDirectPlain, false>, a.sm.count, 1);
    g_last_kernel = label<kKnDirect, R, DT, OP, 1, kDirectPlain>();
  }
  return check_launch("k_slices_direct");
}

template <typename R, int DT>
static int launch_dense_t(qd_state* s, const GatePlan& p, const TileGeom* tile) {
  DenseOp<R, DT> op;
  fill_dense<R, DT>(p, &op);
  return launch_slices<R, DT>(s, p, op, tile);
}

template <typename R, int DT>
static int launch_mono_t(qd_state* s, const GatePlan& p, const TileGeom* tile) {
  MonoOp<R, DT> op;
  fill_mono<R, DT>(p, &op);
  return launch_slices<R, DT>(s, p, op, tile);
}

template <typename R>
static int launch_diag(qd_state* s, const GatePlan& p) {
  const Register& r = s->reg;
  int role[QD_MAX_QUDITS] = {};
  uint32_t lmul[QD_MAX_QUDITS] = {};
  uint32_t m = 1;
  for (int j = p.k - 1; j >= 0; --j) {
    role[p.targets[j]] = 2;
    lmul[p.targets[j]] = m;
    m *= uint32_t(r.dims[p.targets[j]]);
  }
  for (int j = 0; j < p.m; ++j) role[p.controls[j]] = 1;
  DiagArgs<R> a;
  std::memset(&a, 0, sizeof(a));
  a.psi = reinterpret_cast<R*>(s->data);
  int64_t base = 0;
  for (int j = 0; j < p.m; ++j) base += int64_t(p.cvals[j]) * r.strides[p.controls[j]];
  int rc = fill_slicemap(make_groups(r, role, lmul, 0, r.n), base, &a.sm);
  if (rc) return rc;
  for (int i = 0; i < 2 * p.dT; ++i) a.ph[i] = R(p.ph[i]);
  if (a.sm.count == 0) return QD_OK;
  const int bs = tune().diag_block;
  const dim3 grid(grid_for(a.sm.count, uint64_t(bs) * 2));
  if (streaming(s, p, a.sm.count, false)) hipLaunchKernelGGL((k_diag<R, 2, true>), grid, dim3(bs), 0, s->stream, a);
  else hipLaunchKernelGGL((k_diag<R, 2, false>), grid, dim3(bs), 0, s->stream, a);
  g_last_kernel = label<kKnDiag, R>();
  return check_launch("k_diag");
}

template <typename R>
static int launch_generic(qd_state* s, const GatePlan& p) {
  const Register& r = s->reg;
  int role[QD_MAX_QUDITS] = {};
  for (int j = 0; j < p.k; ++j) role[p.targets[j]] = 1;
  for (int j = 0; j < p.m; ++j) role[p.controls[j]] = 1;
  int64_t base = 0;
  for (int j = 0; j < p.m; ++j) base += int64_t(p.cvals[j]) * r.strides[p.controls[j]];
  const size_t bytes = sizeof(GenericHead) + sizeof(int64_t) * p.dT + sizeof(R) * 2 * size_t(p.dT) * p.dT;
  std::vector<unsigned char> buf(bytes, 0);
  auto* h = reinterpret_cast<GenericHead*>(buf.data());
  fill_slicemap64(make_groups(r, role, nullptr, 0, r.n), base, &h->sm);
  h->dT = p.dT;
  h->nsw = std::max(1, 1024 / p.dT);
  target_offsets(r, p, reinterpret_cast<int64_t*>(buf.data() + sizeof(GenericHead)));
  R* U = reinterpret_cast<R*>(buf.data() + sizeof(GenericHead) + sizeof(int64_t) * p.dT);
  for (size_t i = 0; i < 2 * size_t(p.dT) * p.dT; ++i) U[i] = R(p.U[i]);
  if (h->sm.count == 0) return QD_OK;
  void* dev = nullptr;
  int rc = ring_push(s, buf.data(), bytes, &dev);
  if (rc) return rc;
  const uint64_t iters = (h->sm.count + h->nsw - 1) / h->nsw;
  const unsigned grid = unsigned(std::min<uint64_t>(iters, 65536));
  const size_t lds = size_t(h->nsw) * p.dT * sizeof(R) * 2;
  hipLaunchKernelGGL((k_dense_generic<R>), dim3(grid), dim3(256), lds, s->stream, reinterpret_cast<R*>(s->data),
                     static_cast<const unsigned char*>(dev));
  g_last_kernel = label<kKnGeneric, R>();
  return check_launch("k_dense_generic");
}

template <typename R>
static int launch_gemm(qd_state* s, const GatePlan& p);

template <typename R, int DT>
static int launch_direct_lu(qd_state* s, const GatePlan& p) {
  const Register& r = s->reg;
  int role[QD_MAX_QUDITS] = {};
  for (int j = 0; j < p.k; ++j) role[p.targets[j]] = 1;
  for (int j = 0; j < p.m; ++j) role[p.controls[j]] = 1;
  int64_t base = 0;
  for (int j = 0; j < p.m; ++j) base += int64_t(p.cvals[j]) * r.strides[p.controls[j]];
  const size_t bytes = sizeof(LuHead) + sizeof(R) * 2 * size_t(DT) * DT;
  std::vector<unsigned char> buf(bytes, 0);
  auto* h = reinterpret_cast<LuHead*>(buf.data());
  if (fill_slicemap(make_groups(r, role, nullptr, 0, r.n), base, &h->sm) != QD_OK) return launch_gemm<R>(s, p);
  target_offsets(r, p, h->toff);
  R* U = reinterpret_cast<R*>(buf.data() + sizeof(LuHead));
  for (size_t i = 0; i < 2 * size_t(DT) * DT; ++i) U[i] = R(p.U[i]);
  if (h->sm.count == 0) return QD_OK;
  void* dev = nullptr;
  int rc = ring_push(s, buf.data(), bytes, &dev);
  if (rc) return rc;
  auto launch = [&](auto k) {
    hipLaunchKernelGGL(k, dim3(grid_for(h->sm.count, 256)), dim3(256), 0, s->stream, reinterpret_cast<R*>(s->data),
                       static_cast<const unsigned char*>(dev));
  };
  if (streaming(s, p, uint64_t(h->sm.count) * DT, true)) launch(k_slices_direct_lu<R, DT, true>);
  else launch(k_slices_direct_lu<R, DT, false>);
  g_last_kernel = label<kKnLu, R, DT>();
  return check_launch("k_slices_direct_lu");
}

// Tile of the matrix-core kernel: ns slices (a multiple of 16), CG column tiles per job and the waves
// of a workgroup. X takes KP (ns + 1) amplitudes of LDS: the widest tile within 40 KB (four workgroups
// per CU, so that one's loads and stores overlap the others' products), else the widest within 80 KB
// (two per CU), else 16 slices in up to 150 KB; where fewer than two workgroups per CU would be left the
// tile is halved. One case lies beyond that: complex128 with d_T > 568 holds 8 slices.
struct MfmaTile {
  uint32_t ns = 0, lds = 0;
  int cg = 1, waves = 4;
};

static MfmaTile mfma_tile(uint32_t dT, uint32_t KP, size_t amp, uint64_t count) {
  auto bytes = [&](uint32_t ns) { return size_t(KP) * (ns + 1) * amp + amp + sizeof(int64_t) * (ns + dT); };
  MfmaTile t;
  for (size_t cap : {size_t(40) << 10, size_t(80) << 10, size_t(150) << 10}) {
    for (uint32_t ns : {128u, 64u, 32u, 16u})
      if (bytes(ns) <= cap) {
        t.ns = ns;
        break;
      }
    if (t.ns) break;
  }
  if (!t.ns) t.ns = 8;
  while (t.ns > 16 && (count + t.ns - 1) / t.ns < 512) t.ns /= 2;
  t.lds = uint32_t(bytes(t.ns));
  const uint32_t RT = (dT + 15) / 16, CT = std::max(1u, t.ns / 16);
  double best = 0.0;
  for (int cg : {2, 1}) {
    if (uint32_t(cg) > CT) continue;
    for (int w : {16, 8, 4}) {
      const uint32_t jobs = RT * (CT / cg), rounds = (jobs + w - 1) / w;
      if ((w > 4 && jobs < uint32_t(w)) || (w == 16 && t.lds < (uint32_t(80) << 10))) continue;
      const double eff = double(jobs) / double(rounds * w);   // share of the waves at work
      if (eff > best + 0.05) {
        best = eff;
        t.cg = cg;
        t.waves = w;
      }
    }
  }
  return t;
}

template <typename R>
static int launch_gemm(qd_state* s, const GatePlan& p) {
  using C = typename CxT<R>::T;
  const Register& r = s->reg;
  int role[QD_MAX_QUDITS] = {};
  for (int j = 0; j < p.k; ++j) role[p.targets[j]] = 1;
  for (int j = 0; j < p.m; ++j) role[p.controls[j]] = 1;
  int64_t base = 0;
  for (int j = 0; j < p.m; ++j) base += int64_t(p.cvals[j]) * r.strides[p.controls[j]];
  const std::vector<Group> groups = make_groups(r, role, nullptr, 0, r.n);
  MfmaArgs a;
  if (int(groups.size()) > kMaxGroups || fill_slicemap(groups, base, &a.sm) != QD_OK) return launch_generic<R>(s, p);
  if (a.sm.count == 0) return QD_OK;
  const uint32_t dT = uint32_t(p.dT), KP = (dT + kMfmaStep<R> - 1) / kMfmaStep<R> * kMfmaStep<R>, KS = KP / kMfmaStep<R>, RT = (dT + 15) / 16;
  const MfmaTile t = mfma_tile(dT, KP, sizeof(C), a.sm.count);
  const uint64_t ntiles = (uint64_t(a.sm.count) + t.ns - 1) / t.ns;
  int64_t tmin = INT64_MAX;
  for (int j = 0; j < p.k; ++j) tmin = std::min<int64_t>(tmin, r.strides[p.targets[j]]);
  const bool yf = groups.empty() || tmin < groups[0].stride;   // groups[0]: the lowest free run
  bool lines = streaming(s, p, uint64_t(a.sm.count) * dT, false);   // and every run of slices begins and ends on a line
  for (int j = 0; j < p.k + p.m; ++j)
    lines = lines && r.strides[j < p.k ? p.targets[j] : p.controls[j - p.k]] % LineAmps<R>::value == 0;
  a.dT = dT;
  a.KP = KP;
  a.RT = RT;
  a.ns = t.ns;
  a.njobs = RT * (std::max(1u, t.ns / 16) / uint32_t(t.cg));
  a.div = make_magic32(yf ? KP : t.ns);
  // the target combinations by ascending offset: the rows of U in that order, its columns as listed
  std::vector<int64_t> toff(dT);
  target_offsets(r, p, toff.data());
  std::vector<int32_t> ord(dT);
  std::iota(ord.begin(), ord.end(), 0);
  std::sort(ord.begin(), ord.end(), [&](int32_t x, int32_t y) { return toff[x] < toff[y]; });
  const size_t uoff = (sizeof(int64_t) * dT + 15) & ~size_t(15);
  constexpr uint32_t parts = kMfmaStep<R> / 2;   // of an entry, in one lane
  const size_t bytes = uoff + sizeof(R) * size_t(RT) * KS * 64 * parts;
  char* host = nullptr;
  char* dev = nullptr;
  int rc = ring_reserve(&s->ring, s->stream, bytes, &host, &dev);
  if (rc) return rc;
  uint64_t* tg = reinterpret_cast<uint64_t*>(host);
  for (uint32_t i = 0; i < dT; ++i) tg[i] = uint64_t(toff[ord[i]]) | uint64_t(ord[i]) << 32;   // offsets are below 2^32
  R* ug = reinterpret_cast<R*>(host + uoff);
  for (uint32_t rt = 0; rt < RT; ++rt)
    for (uint32_t ks = 0; ks < KS; ++ks)
      for (uint32_t l = 0; l < 64; ++l) {
        const uint32_t row = rt * 16 + (l & 15u), col = ks * kMfmaStep<R> + (parts == 2 ? l >> 4 : l >> 5);
        const uint32_t part = parts == 2 ? 0 : l >> 4 & 1u;
        for (uint32_t i = 0; i < parts; ++i)
          *ug++ = row < dT && col < dT ? R(p.U[2 * (size_t(ord[row]) * dT + col) + part + i]) : R(0);
      }
  rc = ring_commit(&s->ring, s->stream, host, dev, bytes);
  if (rc) return rc;
  a.desc = reinterpret_cast<const unsigned char*>(dev);
  auto launch = [&](auto k) -> int {
    if (t.lds > (size_t(64) << 10))
      QD_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize, int(t.lds)));
    hipLaunchKernelGGL(k, dim3(unsigned(ntiles)), dim3(64 * t.waves), t.lds, s->stream, reinterpret_cast<R*>(s->data), a);
    return check_launch("k_dense_mfma");
  };
  g_last_kernel = label<kKnGemm, R>();
  if (t.cg == 2)
    return yf ? launch(k_dense_mfma<R, 2, kMfmaYF>) : lines ? launch(k_dense_mfma<R, 2, kMfmaLines>) : launch(k_dense_mfma<R, 2, kMfmaParts>);
  return yf ? launch(k_dense_mfma<R, 1, kMfmaYF>) : lines ? launch(k_dense_mfma<R, 1, kMfmaLines>) : launch(k_dense_mfma<R, 1, kMfmaParts>);
}

template <typename R>
static int launch_gate_t(qd_state* s, const GatePlan& p) {
  TileGeom geom;
  const int route = route_gate(s->reg, s->prec, p, &geom);
  const TileGeom* tile = route == QD_ROUTE_TILED ? &geom : nullptr;
  // the generic kernel is left with registers of 2^32 amplitudes or more (launch_gemm also hands it
  // gates whose free digits fall into more groups than a slice map holds)
  if (route == QD_ROUTE_GENERIC)
    return uint64_t(s->reg.D) <= 0xFFFFFFFFull && p.dT >= kGemmMin ? launch_gemm<R>(s, p) : launch_generic<R>(s, p);
  if (route == QD_ROUTE_GEMM) return launch_gemm<R>(s, p);
  if (route == QD_ROUTE_DIAG) return launch_diag<R>(s, p);
  // On the slice-per-thread kernel a monomial U up to d_T = 9 runs as a dense one: each thread then
  // issues all its loads before its stores, which measured faster than storing every output as soon
  // as its one input arrives (a ququart shift 607 -> 588 us on a 1.7 GB state; with a control below
  // one line 720 -> 575 us), and the zero entries add exact zeros.
  if (p.cls == QD_CLASS_MONOMIAL && !(route == QD_ROUTE_DIRECT && p.dT <= kMaxInlineDense)) {
    switch (p.dT) {
      case 2: return launch_mono_t<R, 2>(s, p, tile);
      case 3: return launch_mono_t<R, 3>(s, p, tile);
      case 4: return launch_mono_t<R, 4>(s, p, tile);
      case 5: return launch_mono_t<R, 5>(s, p, tile);
      case 6: return launch_mono_t<R, 6>(s, p, tile);
      case 7: return launch_mono_t<R, 7>(s, p, tile);
      case 8: return launch_mono_t<R, 8>(s, p, tile);
      case 9: return launch_mono_t<R, 9>(s, p, tile);
      case 12: return launch_mono_t<R, 12>(s, p, tile);
      case 16: return launch_mono_t<R, 16>(s, p, tile);
      default: break;
    }
  }
  switch (p.dT) {
    case 2: return launch_dense_t<R, 2>(s, p, tile);
    case 3: return launch_dense_t<R, 3>(s, p, tile);
    case 4: return launch_dense_t<R, 4>(s, p, tile);
    case 5: return launch_dense_t<R, 5>(s, p, tile);
    case 6: return launch_dense_t<R, 6>(s, p, tile);
    case 7: return launch_dense_t<R, 7>(s, p, tile);
    case 8: return launch_dense_t<R, 8>(s, p, tile);
    case 9: return launch_dense_t<R, 9>(s, p, tile);
    case 12: return launch_direct_lu<R, 12>(s, p);
    case 16: return launch_direct_lu<R, 16>(s, p);
    default: return launch_generic<R>(s, p);
  }
}

int launch_gate(qd_state* s, const GatePlan& p) {
  g_last_kernel = "";
  return s->prec == QD_C128 ? launch_gate_t<double>(s, p) : launch_gate_t<float>(s, p);
}

const char* last_kernel() { return g_last_kernel; }
void set_last_kernel(const char* name) { g_last_kernel = name; }

}  // namespace qd
