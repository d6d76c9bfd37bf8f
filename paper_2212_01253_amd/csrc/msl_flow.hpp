// Dataflow schedule: the middle passes of a phase in one launch,
// handed from pass to pass through memory without a barrier.
//
// A wavefront (workgroup) keeps its line for the whole launch.  Every pass
// needs one element of every line of the pass before, so instead of a grid
// barrier the elements themselves carry the news: an exchange field holds a
// sentinel (kUnset, a NaN no pass writes) until its producer has stored the
// element, and a consumer reads its line again until no element is unset.
// A pass then costs one trip of the data to the coherence point and back,
// where separate launches cost that, the end and start of a kernel, and the
// reload of everything a kernel can keep.  It is bound by that chain: of the
// 4.4 k cycles of a 64x64 pass 2.4 k compute (one wavefront per busy SIMD, LDS
// exchanges included), 1.4 k wait for the input; 256x256 5.8 k, 3.3 k and 1.9 k;
// 512x512 10.9 k, 6.2 k and 3.8 k.  Measured, forward per slice, one launch per
// pass and this: 64x64 3.5 and 2.2 us, 128x128 3.8 and 2.5, 256x256 3.8 and 2.7,
// 512x512 6.3 and 4.8; gradient of 256x256x1024 10.7 and 7.5 ms, of
// 512x512x2048 33.7 and 30.9 ms (there the reverse sweep and the recompute
// beside it, 9.6 us a slice, gain nothing over their per-pass launches).
// The exact propagator (a row and a column pass per slice; a column lane keeps its elements of the 2-D
// factor in registers for the whole launch), per slice: 64x64 7.1 and 3.2 us, 256x256 8.6 and 4.2,
// 512x512 12.8 and 7.6, its adjoint 15.9 and 4.7, 16.6 and 6.9, 20.1 and 14.1.  The forward that evaluates
// T from the stacks: 64x64 4.4 and 2.3, 256x256 5.5 and 3.0.
// Lines of 1024 points take two wavefronts and stay with the per-pass launches.
//
// Four exchange fields rotate: pass i reads X[i % 4], writes X[(i + 1) % 4] and
// returns its share of X[(i - 1) % 4] to kUnset.
//  * Nobody still reads X[(i - 1) % 4] then: the workgroup has held whole lines
//    of pass i's input, an element from every line of pass i - 1, and each of
//    those was stored after its producer had read all it needed of
//    X[(i - 1) % 4].
//  * X[(i - 1) % 4] is written next in pass i + 2 and read in pass i + 3.  The new
//    elements have to come after the resets, and a reader's first look too, or it
//    could take the old value.
//  * Where every workgroup takes part in every pass, the resets follow the pass's output and are
//    complete before the workgroup computes pass i + 1 (it waits for its own
//    stores): who writes in pass i + 2 has read pass i + 1's output, who reads in
//    pass i + 3 has read it in pass i + 2.
//  * Where the axes have different numbers of line groups some workgroups sit out every second
//    pass: one that sits out pass i + 2 has seen nothing after pass i's output when it looks
//    for pass i + 2's in pass i + 3, and one that resets in pass i and sits out pass i + 1 tells nobody in
//    between that its resets are done.  There (flow_resets_early) the resets are issued
//    once the workgroup holds its input (after the barrier of the first transform's first exchange),
//    and are complete before any of its output is stored: pass i's output carries the news.
//    The wait is hidden by the second transform; it is not taken on the other grids, where it
//    would stand between the last exchange and the stores that everybody waits for.  512x256 with
//    this order, forward and adjoint per slice (one launch per pass): 4.3 and 6.7 us (5.4 and 9.7), exact
//    5.9 and 9.1 (10.4 and 17.3); 64x512 3.0 and 4.6 (4.6 and 9.1).
// flow_check.cpp follows both orders through the passes of all grids.
// A launch finds all four fields unset but X[0], which its first pass does not
// read and its pass 1 resets, and leaves them so but for X[n - 1], the last
// pass's input: the next launch on the same fields starts its rotation there
// (FlowArgs::rot), and only the first one of a call needs them filled.
// All exchange accesses are agent-scope atomics of one 8-byte element
// (written through to and read from the coherence point of the XCDs' L2s).
//
// The wait is bounded as in the persistent schedule: after `spin_limit` polls
// a wavefront raises the launch's error word and the workspace's status word
// and stops waiting for good.  The unset elements it read are NaN, but what was stored before
// or does not depend on them is not, so the call ends with a kernel that fills its outputs
// with NaN if an error word is raised (k_flow_fold): such a result cannot pass for valid.
#pragma once

#include "msl_flow_host.hpp"

namespace msl {

// Keeps a kernel argument in scalar registers for the whole launch (left alone, the compiler
// reads it again from memory in every pass, on the path between two passes).
template <typename V>
__device__ __forceinline__ void pin(V& v) {
  asm volatile("" : "+s"(v));
}

// Makes the compiler derive what depends on v anew in every pass: left alone it keeps every address
// of both axes' passes in registers, and 512-point lines (8 points per lane) spill.
__device__ __forceinline__ void fresh(int& v) { asm volatile("" : "+v"(v)); }

constexpr bool flow_exact(int k) { return k == FLOW_XFWD || k == FLOW_XREV; }
constexpr bool flow_rev(int k) { return k == FLOW_REV || k == FLOW_XREV; }
constexpr bool flow_pack(int k) { return k == FLOW_FWD || k == FLOW_REV; }

// Slice of pass p of the phase.
template <int K>
__device__ __forceinline__ int flow_slice(const PhaseSpec& ph, int p) {
  const int q = flow_rev(K) ? p - (ph.leading ? 1 : 0) : p, s = flow_exact(K) ? q >> 1 : q;
  return flow_rev(K) ? ph.s1 - 1 - s : ph.s0 + s;
}

// Descriptor of pass p of the phase: slice, cycle position and the fields that only this pass reads or
// writes (the exact propagator's column passes have none).
template <int K, int AXIS>
__device__ __forceinline__ PassDesc flow_desc(const PhaseSpec& ph, int p) {
  PassDesc d{};
  const int s = flow_slice<K>(ph, p);
  d.slice = s;
  d.axis = AXIS;
  d.tab = (flow_exact(K) ? s : s >> 1) & (DITHER - 1);   // tab_of
  if (flow_exact(K) && AXIS == COL) return d;
  const int lay = !flow_exact(K) && (s & 1) ? LAY_C : LAY_T;   // seg_lay
  if constexpr (!flow_rev(K)) {
    d.mid = MID_T_FWD;
    if (ph.kind == PH_FWD_RECOMP) {
      d.psi_store = ph.seg + (int64_t)(s - ph.s0 - 1) * ph.m;
      d.store_lay = lay;
    } else {
      d.psi_store = ckpt_slot(ph, s);
      d.store_lay = LAY_R;
    }
  } else {
    d.mid = MID_T_ADJ;
    if (s == ph.s0) {
      d.psi_load = ph.ckpt_c;
      d.load_lay = LAY_R;
    } else {
      d.psi_load = ph.seg + (int64_t)(s - ph.s0 - 1) * ph.m;
      d.load_lay = ph.seg_row_major ? LAY_R : lay;
    }
  }
  return d;
}

// Exchange layout: 4x4 tiles of 128 bytes, 2x2 tiles inside (row pairs
// contiguous), so two neighbouring rows of a row pass cover whole 64-byte
// halves and two neighbouring columns 32 bytes of each half.
template <int N, int AXIS, int P>
__device__ __forceinline__ LineAddr flow_at(const Ctx& c, int line, int j) {
  constexpr uint32_t L = (uint32_t)(N / P);
  static_assert(L % 4 == 0, "a step along the line keeps the place in the tile");
  const uint32_t r = AXIS == ROW ? (uint32_t)line : (uint32_t)j, q = AXIS == ROW ? (uint32_t)j : (uint32_t)line;
  const uint32_t tile = (r >> 2) * ((uint32_t)c.nz >> 2) + (q >> 2);
  const uint32_t in = ((r & 2u) << 2) + ((q & 2u) << 1) + ((r & 1u) << 1) + (q & 1u);
  return LineAddr{(tile << 4) + in, AXIS == ROW ? 4 * L : L * (uint32_t)c.nz};
}

// Byte offsets of a lane's static inputs from the uniform bases of a pass (its
// rows of the tables, its slice of the pack): computed once, so that a pass
// issues its loads as base + 32-bit offset without address arithmetic.
template <int N, int P>
struct FlowOffs {
  using T = LineTw<N, P>;
  uint32_t w[T::NPW > 0 ? T::NPW : 1][P - 1];
  uint32_t wl[T::R0LAST ? T::Q : 1][T::R0LAST ? T::R0 - 1 : 1];
  uint32_t h, tm;
};

template <typename V>
__device__ __forceinline__ V ld_off(const void* base, uint32_t off) {
  return *reinterpret_cast<const V*>(static_cast<const char*>(base) + off);
}

template <int N, int AXIS, int P, int K>
__device__ __forceinline__ void flow_offs(const Ctx& c, int line, int j, FlowOffs<N, P>& o) {
  using T = LineTw<N, P>;
  constexpr int L = N / P;
#pragma unroll
  for (int s = 0, NS = T::R0LAST ? P : T::R0; s < T::NPW; ++s, NS *= P)
#pragma unroll
    for (int r = 1; r < P; ++r) o.w[s][r - 1] = 8u * (uint32_t)((j % NS) * r * (N / (P * NS)));
  if constexpr (T::R0LAST) {
#pragma unroll
    for (int q = 0; q < T::Q; ++q)
#pragma unroll
      for (int r = 1; r < T::R0; ++r) o.wl[q][r - 1] = 8u * (uint32_t)((j + L * q) * r);
  }
  o.h = 8u * (uint32_t)j;
  if constexpr (flow_pack(K)) o.tm = 8u * line_at<N, AXIS, P>(c, pack_lay<AXIS>(c), line, j).base;
  else o.tm = 4u * line_at<N, AXIS, P>(c, LAY_R, line, j).base;
}

// The two halves of load_static of a middle pass, from those offsets: the
// tables' rows, and what belongs to the slice (T - 1; in the reverse sweep the
// entrance field).
template <int N, int AXIS, int P, bool H1D>
__device__ __forceinline__ void flow_tables(const Ctx& c, int tab, const FlowOffs<N, P>& o, LineIn<N, P>& in) {
  using T = LineTw<N, P>;
  constexpr uint32_t L = N / P;
  const uint32_t row = (uint32_t)tab * (uint32_t)N;
  const float2* const tw = (AXIS == ROW ? c.twz : c.twy) + row;
  const float2* const h = (AXIS == ROW ? c.hz : c.hy) + row;
#pragma unroll
  for (int s = 0; s < T::NPW; ++s)
#pragma unroll
    for (int r = 1; r < P; ++r) in.tw.w[s][r - 1] = ld_off<float2>(tw, o.w[s][r - 1]);
  if constexpr (T::R0LAST) {
#pragma unroll
    for (int q = 0; q < T::Q; ++q)
#pragma unroll
      for (int r = 1; r < T::R0; ++r) in.tw.wl[q][r - 1] = ld_off<float2>(tw, o.wl[q][r - 1]);
  }
  in.tw.rs2 = rs2_at(tab);
  if constexpr (H1D) {
#pragma unroll
    for (int t = 0; t < P; ++t) in.hh[t] = ld_off<float2>(h, o.h + 8u * L * (uint32_t)t);
  }
}

template <int N, int AXIS, int KIND, int P>
__device__ __forceinline__ void flow_slice_in(const Ctx& c, const PassDesc& pd, int line, int j,
                                              const FlowOffs<N, P>& o, LineIn<N, P>& in) {
  constexpr uint32_t L = N / P;
  if (flow_exact(KIND) && AXIS == COL) return;
  if constexpr (flow_pack(KIND)) {
    const float2* const tm = c.dbT + (int64_t)pd.slice * c.m;
#pragma unroll
    for (int t = 0; t < P; ++t) {
      const float2 q = ld_off<float2>(tm, o.tm + 16u * L * (uint32_t)t);   // 2x2 tiles along the line's axis
      in.dl[t] = q.x;
      in.bt[t] = q.y;
    }
  } else {
    const float* const dp = c.delta + (int64_t)pd.slice * c.m;
    const float* const bp = c.beta + (int64_t)pd.slice * c.m;
    const uint32_t step = 4u * L * (AXIS == ROW ? 1u : (uint32_t)c.nz);
#pragma unroll
    for (int t = 0; t < P; ++t) {
      in.dl[t] = ld_off<float>(dp, o.tm + step * (uint32_t)t);
      in.bt[t] = ld_off<float>(bp, o.tm + step * (uint32_t)t);
    }
  }
  if constexpr (flow_rev(KIND)) {
    const LineAddr a = line_at<N, AXIS, P>(c, pd.load_lay, line, j);
#pragma unroll
    for (int t = 0; t < P; ++t) in.ps[t] = ld_off<float2>(pd.psi_load, 8u * (a.base + (uint32_t)t * a.stride));
  }
}

// One element of an exchange field at byte offset off.
__device__ __forceinline__ float2 flow_ld(const float2* x, uint32_t off) {
  return field_ld<true>(reinterpret_cast<const float2*>(reinterpret_cast<const char*>(x) + off));
}
__device__ __forceinline__ void flow_st(float2* x, uint32_t off, float2 v) {
  field_st<true>(reinterpret_cast<float2*>(reinterpret_cast<char*>(x) + off), v);
}

// How the lanes of a workgroup hold its lines at a pass's two ends.  G = 1: as
// between the transforms, one wavefront per line or less.  G > 1 (lines of one
// wavefront each): thread t holds line t mod G at lane t / G, so neighbouring
// threads cover whole tiles of the exchange field; the first exchange of the
// first transform and the last one of the last transform carry the line over
// to its wavefront and back (their first and last butterflies are the same in
// both mappings), each with a workgroup barrier.
template <int N, int P, int G>
struct FlowEnds {
  LineLds sh;   // exchange buffers of the line held at the ends
  int j;        // lane in it
  LineTw<N, P> tw;   // the last stage's twiddles for that lane (w[NPW - 1] only)
};

// Waits until this wavefront's stores (and loads) are complete.
__device__ __forceinline__ void flow_wait() {
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

// fft_line within a wavefront (radix P throughout) whose input (IN) or output
// (OUT) is held as FlowEnds says.  EARLY: the wavefront's stores are complete before its workgroup
// meets for the last exchange of the output (G > 1).
template <int N, bool INV, int P, int G, bool IN, bool OUT, bool EARLY>
__device__ __forceinline__ void flow_fft(float2 (&v)[P], const LineLds& sh, int j, const LineTw<N, P>& tw,
                                         const FlowEnds<N, P, G>& e) {
  if constexpr (G == 1 || (!IN && !OUT)) {
    fft_line<N, INV, P, true>(v, sh, j, tw);
  } else {
    using T = LineTw<N, P>;
    constexpr int L = N / P, NX = T::NST;
    static_assert(T::R0 == P && L == 64, "radix P throughout, one wavefront per line");
    const LineLds& si = IN ? e.sh : sh;
    dft_p<P, INV>(v, tw.rs2);
    {
      const uint32_t wb = lds_base<N, P>(si, (uint32_t)(P * (IN ? e.j : j)));
#pragma unroll
      for (int r = 0; r < P; ++r) si.a[lds_slot<N, P>(wb, (uint32_t)r)] = v[r];
    }
    if constexpr (IN) __syncthreads();
    else line_sync<true>();
    const uint32_t rb = lds_base<N, P>(sh, (uint32_t)j), eb = lds_base<N, P>(e.sh, (uint32_t)e.j);
#pragma unroll
    for (int s = 0, NS = P; s < NX; ++s, NS *= P) {
      const bool out = OUT && s == NX - 1;
      if (out) {
        if constexpr (EARLY) flow_wait();
        __syncthreads();
      }
      const LineLds& b = out ? e.sh : sh;
      const float2* const rd = (s & 1) ? b.b : b.a;
#pragma unroll
      for (int t = 0; t < P; ++t) v[t] = rd[lds_slot<N, P>(out ? eb : rb, (uint32_t)(t * L))];
#pragma unroll
      for (int r = 1; r < P; ++r) v[r] = cmul<INV>(v[r], out ? e.tw.w[s][r - 1] : tw.w[s][r - 1]);
      dft_p<P, INV>(v, tw.rs2);
      if (s + 1 < NX) {
        float2* const wr = (s & 1) ? sh.a : sh.b;
        const uint32_t wb = lds_base<N, P>(sh, (uint32_t)((j / NS) * NS * P + (j % NS)));
#pragma unroll
        for (int r = 0; r < P; ++r) wr[lds_slot<N, P>(wb, (uint32_t)(r * NS))] = v[r];
        line_sync<true>();
      }
    }
  }
}

template <int N, int P, int G, bool IN, bool OUT, bool EARLY>
__device__ __forceinline__ void flow_prop(LineIn<N, P>& in, const LineLds& sh, int j, const FlowEnds<N, P, G>& e,
                                          bool conj) {
  flow_fft<N, false, P, G, IN, false, EARLY>(in.v, sh, j, in.tw, e);
#pragma unroll
  for (int t = 0; t < P; ++t) in.v[t] = cmul_dyn(in.v[t], in.hh[t], conj);
  flow_fft<N, true, P, G, false, OUT, EARLY>(in.v, sh, j, in.tw, e);
}

// One pass of this workgroup's lines (group `unit` of the pass; this lane's
// line and lane between the transforms, eline and e.j at the ends); in: the
// slice's inputs, already requested.  prefetch() requests the next pass's.
template <int N, int P, int AXIS, int KIND, int T, int G, bool FRESH, bool EARLY, class Prefetch>
__device__ __forceinline__ void flow_pass(const Ctx& c, const FlowArgs& a, int i, int unit, int line, int j,
                                          const LineLds& sh, const FlowOffs<N, P>& o, LineIn<N, P>& in, int eline,
                                          FlowEnds<N, P, G>& e, int& dead, Prefetch prefetch) {
  if constexpr (FRESH) {
    fresh(line);
    fresh(j);
    fresh(eline);
    fresh(e.j);
  }
  const bool first = i == 0, last = i == a.n - 1;
  const int x = a.rot + i;
  float2* const rd = a.x + (int64_t)(x & 3) * c.m;
  float2* const wr = a.x + (int64_t)((x + 1) & 3) * c.m;
  float2* const old = a.x + (int64_t)((x + 3) & 3) * c.m;
  const LineAddr xa = flow_at<N, AXIS, P>(c, eline, e.j);
  const LineAddr fa = line_at<N, AXIS, P>(c, KIND == FLOW_STACK ? (int)LAY_R : (int)LAY_T, eline, e.j);   // the working field's
  const uint32_t xo = 8u * xa.base;
  // the reset's share is contiguous (whole 128-byte lines): line by line it cost 0.5 k cycles a pass of
  // 256x256, 1 k of 512x512
  const uint32_t ro = 8u * ((uint32_t)unit * (uint32_t)(T * P) + (threadIdx.x & ~63u) * (uint32_t)P + (threadIdx.x & 63u));
  const PassDesc pd = flow_desc<KIND, AXIS>(a.ph, a.p0 + i);
  flow_tables<N, AXIS, P, !flow_exact(KIND)>(c, pd.tab, o, in);
  if constexpr (G > 1) {
    using TW = LineTw<N, P>;
    const float2* const tw = (AXIS == ROW ? c.twz : c.twy) + (uint32_t)pd.tab * (uint32_t)N;
#pragma unroll
    for (int r = 1; r < P; ++r) e.tw.w[TW::NPW - 1][r - 1] = ld_off<float2>(tw, 8u * (uint32_t)(e.j * r));
  }
  if (first) {
#pragma unroll
    for (int t = 0; t < P; ++t) in.v[t] = a.ph.field[fa.base + (uint32_t)t * fa.stride];
  } else {
    for (int q = 0; q < a.nap; ++q) __builtin_amdgcn_s_sleep(4);
    unsigned spins = 0;
    for (;;) {
      bool miss = false;
#pragma unroll
      for (int t = 0; t < P; ++t) in.v[t] = flow_ld(rd, xo + 8u * (uint32_t)t * xa.stride);
#pragma unroll
      for (int t = 0; t < P; ++t) miss = miss | (__float_as_uint(in.v[t].x) == kUnset);
      if (dead || __ballot(miss) == 0) break;
      if (++spins > a.spin_limit) {
        __hip_atomic_store(a.err, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        *a.status = 1u;
        dead = 1;
      } else if ((spins & 63u) == 0u) {
        dead = __builtin_amdgcn_readfirstlane(
            (int)__hip_atomic_load(a.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
      }
    }
  }
  if constexpr (!EARLY) flow_wait();   // the resets of the pass before are complete
  auto reset = [&]() {
    if (first) return;
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    const float q = __uint_as_float(kUnset);
#pragma unroll
    for (int t = 0; t < P; ++t) flow_st(old, ro + 512u * (uint32_t)t, make_float2(q, q));
  };
  constexpr int TS = flow_pack(KIND) ? TS_PACK : TS_RUNTIME;
  if constexpr (!flow_exact(KIND)) {
    flow_prop<N, P, G, true, false, EARLY>(in, sh, j, e, flow_rev(KIND));
    if constexpr (EARLY) reset();
    mid_line<N, AXIS, TS, P>(c, pd, line, j, in);
    prefetch();
    flow_prop<N, P, G, false, true, EARLY>(in, sh, j, e, flow_rev(KIND));
  } else if constexpr (AXIS == COL) {
    flow_fft<N, false, P, G, true, false, EARLY>(in.v, sh, j, in.tw, e);
    if constexpr (EARLY) reset();
#pragma unroll
    for (int t = 0; t < P; ++t) in.v[t] = cmul_comp_dyn(in.v[t], in.hh[t], in.hl[t], flow_rev(KIND));
    prefetch();
    flow_fft<N, true, P, G, false, true, EARLY>(in.v, sh, j, in.tw, e);
  } else {
    constexpr float inv_n = 1.0f / (float)N;
    flow_fft<N, true, P, G, true, false, EARLY>(in.v, sh, j, in.tw, e);
    if constexpr (EARLY) reset();
#pragma unroll
    for (int t = 0; t < P; ++t) in.v[t] = make_float2(in.v[t].x * inv_n, in.v[t].y * inv_n);
    mid_line<N, AXIS, TS, P>(c, pd, line, j, in);
    prefetch();
    flow_fft<N, false, P, G, false, true, EARLY>(in.v, sh, j, in.tw, e);
  }
  if constexpr (EARLY && G == 1) flow_wait();   // (G > 1: before the last exchange)
  if (last) {
#pragma unroll
    for (int t = 0; t < P; ++t) a.ph.field[fa.base + (uint32_t)t * fa.stride] = in.v[t];
  } else {
#pragma unroll
    for (int t = 0; t < P; ++t) {
      float2 v = in.v[t];
      if (__float_as_uint(v.x) == kUnset) v.x = __builtin_nanf("");
      flow_st(wr, xo + 8u * (uint32_t)t * xa.stride, v);
    }
  }
  if constexpr (!EARLY) reset();
}

// Middle passes of one phase over an NY x NZ grid by workgroups of T threads:
// row passes T / LZ lines of NZ points each, column passes T / LY lines of NY
// points; workgroups beyond a pass's line groups sit it out.
template <int NZ, int NY, int PZ, int PY, int KIND, int T>
__global__ void __launch_bounds__(T, 2) k_flow(Ctx c_, FlowArgs a_) {
  Ctx c = c_;
  FlowArgs a = a_;
  c.ny = NY;
  c.nz = NZ;
  c.m = (int64_t)NY * NZ;
  a.ph.m = c.m;
  if constexpr (!flow_pack(KIND)) c.dbT = nullptr;
  else pin(c.dbT);
  pin(c.twz);
  pin(c.twy);
  if constexpr (!flow_exact(KIND)) {
    pin(c.hz);
    pin(c.hy);
  }
  if constexpr (!flow_pack(KIND)) {
    pin(c.delta);
    pin(c.beta);
  }
  pin(a.x);
  pin(a.rot);
  pin(a.nap);
  pin(a.ph.field);
  pin(a.n);
  pin(a.p0);
  pin(a.ph.s0);
  pin(a.spin_limit);
  if constexpr (flow_rev(KIND)) {
    pin(a.ph.s1);
    pin(a.ph.seg);
    pin(a.ph.leading);
    pin(c.gdelta);
    pin(c.gbeta);
    pin(c.gT);
  } else {
    pin(a.ph.ckpt);
    pin(a.ph.seg);
    pin(a.ph.ckpt_every);
    pin(a.ph.kind);
  }
  constexpr int LZ = NZ / PZ, LY = NY / PY, GZ = T / LZ, GY = T / LY;
  constexpr int LDSZ = 2 * GZ * NZ, LDSY = 2 * GY * NY;
  static_assert(GZ >= 1 && GY >= 1 && GZ <= NY && GY <= NZ, "whole lines per workgroup");
  __shared__ float2 lds[LDSZ > LDSY ? LDSZ : LDSY];
  const int tid = threadIdx.x;
  constexpr int UZ = NY / GZ, UY = NZ / GY;  // line groups of a row pass, of a column pass
  // the wavefronts of a workgroup part at a pass's last exchange and meet at the next pass's first one;
  // where that one may use a buffer the last exchange is still read from, they meet between the passes
  constexpr bool FR = PZ == 8 || PY == 8, EARLY = flow_resets_early(NZ, NY);
  static_assert(UZ == flow_row_units(NZ, NY) && UY == flow_col_units(NZ, NY), "the order flow_check.cpp follows");
  constexpr bool kMeet = T > 64 && (NZ != NY || LineTw<NZ, PZ>::NST % 2 == 1);
  constexpr int NB = UZ > UY ? UZ : UY;  // the launch's grid
  const int b = xcd_group(blockIdx.x, gridDim.x);
  // lines shorter than a wavefront interleave in it; one-wavefront lines take a wavefront each
  constexpr int EZ = LZ == 64 ? GZ : 1, EY = LY == 64 ? GY : 1;   // FlowEnds mapping
  static_assert(T == 64 || (LZ == 64 && LY == 64), "several wavefronts: one line each");
  const int gz = T == 64 ? tid % GZ : tid / 64, jz = T == 64 ? tid / GZ : tid % 64;
  const int gy = T == 64 ? tid % GY : tid / 64, jy = T == 64 ? tid / GY : tid % 64;
  const int row = b * GZ + gz, col = b * GY + gy;
  const int ez = T == 64 ? gz : tid % GZ, ey = T == 64 ? gy : tid % GY;
  FlowEnds<NZ, PZ, EZ> endz;
  FlowEnds<NY, PY, EY> endy;
  endz.sh = line_buffers<NZ, PZ>(lds, ez, GZ);
  endy.sh = line_buffers<NY, PY>(lds, ey, GY);
  endz.j = T == 64 ? jz : tid / GZ;
  endy.j = T == 64 ? jy : tid / GY;
  const LineLds shz = line_buffers<NZ, PZ>(lds, gz, GZ);
  const LineLds shy = line_buffers<NY, PY>(lds, gy, GY);
  LineIn<NZ, PZ> inz;
  LineIn<NY, PY> iny;
  FlowOffs<NZ, PZ> oz;
  FlowOffs<NY, PY> oy;
  // a workgroup that sits out the passes of one axis loads the static inputs of a line that exists
  const int rowl = (UZ == NB || b < UZ) ? row : gz, coll = (UY == NB || b < UY) ? col : gy;
  flow_offs<NZ, ROW, PZ, KIND>(c, rowl, jz, oz);
  flow_offs<NY, COL, PY, KIND>(c, coll, jy, oy);
  if constexpr (flow_exact(KIND)) {   // one 2-D factor for all slices
#pragma unroll
    for (int t = 0; t < PY; ++t) {
      const uint32_t e = (uint32_t)(jy + t * LY) * NZ + (uint32_t)coll;
      iny.hh[t] = c.H_hi[e];
      iny.hl[t] = c.H_lo[e];
    }
  }
  int dead = __builtin_amdgcn_readfirstlane(
      (int)__hip_atomic_load(a.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
  auto load_row = [&](int i) {
    flow_slice_in<NZ, ROW, KIND, PZ>(c, flow_desc<KIND, ROW>(a.ph, a.p0 + i), rowl, jz, oz, inz);
  };
  auto load_col = [&](int i) {
    flow_slice_in<NY, COL, KIND, PY>(c, flow_desc<KIND, COL>(a.ph, a.p0 + i), coll, jy, oy, iny);
  };
  // pass 0 is a column pass; past the last pass the prefetch repeats a slice of the launch
  const int n = a.n;
  load_col(0);
  for (int i = 0;;) {
    int nx = i + 1 < n ? i + 1 : i;
    if (UY == NB || b < UY)
      flow_pass<NY, PY, COL, KIND, T, EY, FR, EARLY>(c, a, i, b, col, jy, shy, oy, iny, b * GY + ey, endy, dead, [&]() { load_row(nx); });
    else
      load_row(nx);
    if (++i >= n) break;
    if (kMeet) __syncthreads();
    nx = i + 1 < n ? i + 1 : i;
    if (UZ == NB || b < UZ)
      flow_pass<NZ, PZ, ROW, KIND, T, EZ, FR, EARLY>(c, a, i, b, row, jz, shz, oz, inz, b * GZ + ez, endz, dead, [&]() { load_col(nx); });
    else
      load_col(nx);
    if (++i >= n) break;
    if (kMeet) __syncthreads();
  }
}

}  // namespace msl
