// Resident solves: the whole time loop of a 2D instance in one launch.
//
// A domain is a group of workgroups, on one accelerator complex die (XCD) or
// over all of them.  Its members run every pass of an instance's steps over
// the instance's tiles and meet at a barrier between two passes.  What a pass
// hands to the next (the packed spectra) is complete (s_waitcnt) before the
// barrier and read past the vector L1; within one die it travels through that
// die's L2, across dies it is written through at agent scope as well.  The
// state and the medium of a row are only touched by the compute unit that
// owns it.  No cache is written back or invalidated between passes: an
// agent-scope release or acquire fence costs 15-20 us with 256 workgroups
// running (every wavefront's write-back and invalidate queue up at the L2);
// this barrier alone, in a build whose passes do nothing else, costs 0.40 us
// with the 8 members of 64^2, 0.65 us with 32 members on a die and 1.5 us over
// all eight.  A pass of its own launch costs 5.5-9 us at 64^2 to 512^2, whatever
// the grid.
//
// Tiles are cut for latency: four values per lane (eight for columns of 512
// points), the two parts of every pass (axis components, absorption terms, or
// the two outputs of the transposed density update) on different wavefronts,
// so that no wavefront runs more than two transforms between two barriers,
// and as few wavefronts per compute unit as there are compute units for.
// What bounds it is the chain of one wavefront: some 4 cycles per
// instruction, four exchanges per transform (4000-4500 of the 6100 cycles of a
// pass at 128^2), and the barrier (stores complete after 0.27 us, a load from
// the L2 takes 0.09 us).  So what does not change
// through the time loop is not formed in it (the columns' multipliers stay in
// registers), and the loads of a pass's own rows stand between the two halves
// of the barrier.
//
// Per step of the time loop, launches, resident without these two, and as it
// is, the barrier's words on lines of their own too (us): lossless forward 64^2
// 22.5, 10.7, 8.4; lossy forward 64^2 32.9, 15.3, 12.5, 128^2 36.7, 20.8,
// 15.2, 256 x 64 40.6, 20.0, 15.0, 256^2 43.9, 28.9, 23.3, 512^2 53.7, 39.8,
// 34.5; the adjoint within 5% of the forward.
//
// Membership is dynamic, so that a domain never waits for a workgroup that
// is not running: a domain's roll is closed when it is complete or after a
// bounded time, and a workgroup that comes later leaves at once.  Every
// member is then resident until the queue is empty.  Every wait is bounded; a
// member whose wait runs out leaves, and every instance that not all members
// of a domain took to its end, begun or not, stays marked (kSolveOpen).
#pragma once

#include <type_traits>

#include "passes_col.h"
#include "passes_row.h"
#include "solve.h"

// The results equal the per-launch passes' bitwise.  There the compiler
// contracts products into the sums they feed (a product of two into the
// first, unless it has more uses); here, where the same expressions stand in
// other surroundings, the contractions are written out.
#pragma clang fp contract(off)

namespace pat {

// ---------------------------------------------------------------- pointwise
__device__ __forceinline__ float2 fma2(float2 a, float2 b, float2 c) {
  return f2(fmaf(a.x, b.x, c.x), fmaf(a.y, b.y, c.y));
}
__device__ __forceinline__ float2 neg2(float2 a) { return f2(-a.x, -a.y); }
// u <- Qsg (Qsg u - B d p); the first step starts from u = (B/2) d p
__device__ __forceinline__ float2 velocity(float2 u, float2 d, float2 b, float2 qs, bool first) {
  const float2 db = mul2(b, d);
  const float2 u0 = first ? scl2(0.5f, db) : u;
  return mul2(qs, fma2(qs, u0, neg2(db)));
}
// ubar -= d+ gbar; feed B Qsg ubar (last step: B Qsg ubar (1 - Qsg/2)) in d,
// ubar <- Qsg^2 ubar
__device__ __forceinline__ void adj_velocity(float2& u, float2& d, float2 b, float2 qs, bool last) {
  const float2 ub = u - d;
  const float2 bq = mul2(b, mul2(qs, ub));
  d = last ? mul2(bq, f2(fmaf(-0.5f, qs.x, 1.f), fmaf(-0.5f, qs.y, 1.f))) : bq;
  u = mul2(mul2(qs, qs), ub);
}
// p = c0^2 sum rho + c0^2 tau A1 - c0^2 eta A2
__device__ __forceinline__ float2 pressure(float2 c2, float2 rs, float2 ct, float2 a1, float2 ce, float2 a2) {
  return fma2(neg2(ce), a2, fma2(c2, rs, mul2(ct, a1)));
}
// transposed density update of one component, r1 = rhobar + (q - A2):
// gbar / (dt rho0) = A1 - Q r1, rhobar <- Q^2 r1
__device__ __forceinline__ float2 adj_density(float2& r, float2 a2, float2 a1, float2 qq) {
  const float2 r1 = r + a2;
  r = mul2(mul2(qq, qq), r1);
  return fma2(neg2(qq), r1, a1);
}
// ... lossless: gbar = -dt rho0 Q r1, r1 = rhobar + c0^2 v
__device__ __forceinline__ float2 adj_density_ll(float2& r, float2 c2, float2 v, float2 dr, float2 qq) {
  const float2 r1 = fma2(c2, v, r);
  r = mul2(mul2(qq, qq), r1);
  return f2(0.f, 0.f) - mul2(dr, mul2(qq, r1));
}

// ---------------------------------------------------------------- transforms
// twmul (fft.h) with its contraction written out: the first of the two
// low-order products into the second, or (FA < 0) the second into the first
template <int SIGN, int FA>
__device__ __forceinline__ float2 tw_times(float2 x, const Tw w) {
  const float wi = (SIGN < 0) ? w.hi : -w.hi;
  float tr, ti;
  if constexpr (SIGN < 0) {
    tr = fmaf(x.x, w.lr, -(x.y * w.li));
    ti = FA < 0 ? fmaf(x.y, w.lr, x.x * w.li) : fmaf(x.x, w.li, x.y * w.lr);
  } else {
    tr = FA < 0 ? fmaf(x.y, w.li, x.x * w.lr) : fmaf(x.x, w.lr, x.y * w.li);
    ti = fmaf(x.y, w.lr, -(x.x * w.li));
  }
  return make_float2(fmaf(x.x, w.hr, fmaf(-x.y, wi, tr)), fmaf(x.x, wi, fmaf(x.y, w.hr, ti)));
}

// A transform on half as many values per thread (four) and twice as many
// threads, with the same butterflies and roundings as the eight-value
// transform (M, 8): the eight values of one of its threads t (T8 = M / 8)
// are held by two lanes of a wavefront 32 apart, half h = 0 those at
// t + T8 m, m < 4, half 1 those at m >= 4.  A radix-8 butterfly is its
// radix-2 layer across the two lanes (v_permlane32_swap), then a radix-4
// butterfly in each; smaller last stages likewise.
//
// After the swap both lanes hold half 0's value in x and half 1's in y.
__device__ __forceinline__ void half_pair(float2 v, float2& x, float2& y) {
  const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v.x), __float_as_uint(v.x), false, false);
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v.y), __float_as_uint(v.y), false, false);
  x = make_float2(__uint_as_float(a[0]), __uint_as_float(b[0]));
  y = make_float2(__uint_as_float(a[1]), __uint_as_float(b[1]));
}
// half 1's x and half 0's y change places
__device__ __forceinline__ void half_cross(float2& x, float2& y) {
  const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(x.x), __float_as_uint(y.x), false, false);
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x.y), __float_as_uint(y.y), false, false);
  x = make_float2(__uint_as_float(a[0]), __uint_as_float(b[0]));
  y = make_float2(__uint_as_float(a[1]), __uint_as_float(b[1]));
}
// values at 4 h + i (i = 0..3) <-> values at 2 i + h, in registers 0, 2, 1, 3
__device__ __forceinline__ void half_shuffle(float2 (&v)[4]) {
  half_cross(v[0], v[1]);
  half_cross(v[2], v[3]);
  const float2 w = v[1];
  v[1] = v[2];
  v[2] = w;
}
__device__ __forceinline__ float2 sel2(bool c, float2 a, float2 b) { return make_float2(c ? a.x : b.x, c ? a.y : b.y); }

template <int M, int SIGN, int L, int STOP = M, int FA = SIGN, bool PRE = false>
struct PairStage {
  static constexpr int T = M / 8;
  static constexpr int R = fft_radix(M, 8, L);
  static constexpr bool LAST = (L * R == M);
  static_assert(R == 8 || LAST, "only the last stage may be shorter");

  __device__ __forceinline__ static void run(float2 (&v)[4], float2* lds, int t, bool h, const Tw* tw) {
    const float sg = h ? -1.f : 1.f;
    if constexpr (R == 8) {
      const int j = t & (L - 1);
      if constexpr (!PRE && L > 1) {
        const Tw* w = tw + staged_off(M, 8, L) + j;
        v[0] = sel2(h, tw_times<SIGN, FA>(v[0], w[h ? 3 * L : 0]), v[0]);
#pragma unroll
        for (int i = 1; i < 4; ++i) v[i] = tw_times<SIGN, FA>(v[i], w[(h ? 3 + i : i - 1) * L]);
      }
      if constexpr (!PRE) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          float2 x, y;
          half_pair(v[i], x, y);
          v[i] = make_float2(fmaf(sg, y.x, x.x), fmaf(sg, y.y, x.y));
        }
      }
      v[1] = sel2(h, mul_w8<SIGN>(v[1]), v[1]);
      v[2] = sel2(h, mul_si<SIGN>(v[2]), v[2]);
      v[3] = sel2(h, mul_w83<SIGN>(v[3]), v[3]);
      Dft<4, SIGN>::run(v);
      half_unshuffle(v);  // outputs 2 i + h -> 4 h + i
      if constexpr (!LAST) {
        const int base = (t - j) * 8 + j + (h ? 4 * L : 0);
#pragma unroll
        for (int i = 0; i < 4; ++i) lds[pad8(base + i * L)] = v[i];
        if constexpr (L * R != STOP) {
          WaveSync::sync();
          read(v, lds, t, h);
          WaveSync::sync();
          PairStage<M, SIGN, L * R, STOP, FA>::run(v, lds, t, h, tw);
        }
      }
    } else if constexpr (R == 4) {
      half_shuffle(v);  // butterfly h: values h + 2 i
      const int j = (t + (h ? T : 0)) & (L - 1);
#pragma unroll
      for (int i = 1; i < 4; ++i) v[i] = tw_times<SIGN, FA>(v[i], tw[staged_off(M, 8, L) + (i - 1) * L + j]);
      Dft<4, SIGN>::run(v);
      half_unshuffle(v);
    } else {
      static_assert(R == 2, "radix");
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int j = (t + T * i) & (L - 1);
        float2 x, y;
        half_pair(sel2(h, tw_times<SIGN, FA>(v[i], tw[staged_off(M, 8, L) + j]), v[i]), x, y);
        v[i] = make_float2(fmaf(sg, y.x, x.x), fmaf(sg, y.y, x.y));
      }
    }
  }
  // the radix-2 layer of the first stage (PRE: done by this) on the products
  // a b: half 0's product contracted into the sum, half 1's rounded
  __device__ __forceinline__ static void products(const float2 (&a)[4], const float2 (&b)[4], float2 (&v)[4], bool h) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float2 ax, ay, bx, by;
      half_pair(a[i], ax, ay);
      half_pair(b[i], bx, by);
      const float2 y = f2(ay.x * by.x, ay.y * by.y);
      v[i] = f2(fmaf(ax.x, bx.x, h ? -y.x : y.x), fmaf(ax.y, bx.y, h ? -y.y : y.y));
    }
  }
  __device__ __forceinline__ static void read(float2 (&v)[4], const float2* lds, int t, bool h) {
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = lds[pad8(t + T * ((h ? 4 : 0) + i))];
  }
  __device__ __forceinline__ static void half_unshuffle(float2 (&v)[4]) {
    const float2 w = v[1];
    v[1] = v[2];
    v[2] = w;
    half_cross(v[0], v[1]);
    half_cross(v[2], v[3]);
  }
};

// The eight-value transform (FftStage) with the same written-out contraction.
template <int M, int SIGN, int L, int STOP = M, int FA = SIGN>
struct WideStage {
  static constexpr int T = M / 8;
  static constexpr int R = fft_radix(M, 8, L), NB = 8 / R;
  static constexpr bool LAST = (L * R == M);

  __device__ __forceinline__ static void run(float2 (&v)[8], float2* lds, int t, int, const Tw* tw) {
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int k = t + T * b, j = k & (L - 1);
      float2 x[R];
#pragma unroll
      for (int i = 0; i < R; ++i) x[i] = v[b + i * NB];
      if constexpr (L > 1) {
#pragma unroll
        for (int i = 1; i < R; ++i) x[i] = tw_times<SIGN, FA>(x[i], tw[staged_off(M, 8, L) + (i - 1) * L + j]);
      }
      Dft<R, SIGN>::run(x);
#pragma unroll
      for (int i = 0; i < R; ++i) {
        if constexpr (LAST) v[b + i * NB] = x[i];
        else lds[pad8((k - j) * R + j + i * L)] = x[i];
      }
    }
    if constexpr (!LAST && L * R != STOP) {
      WaveSync::sync();
#pragma unroll
      for (int m = 0; m < 8; ++m) v[m] = lds[pad8(t + T * m)];
      WaveSync::sync();
      WideStage<M, SIGN, L * R, STOP, FA>::run(v, lds, t, 0, tw);
    }
  }
};
template <bool PAIR, int M, int SIGN, int L, int STOP = M, int FA = SIGN>
struct SolveStage : PairStage<M, SIGN, L, STOP, FA> {};
template <int M, int SIGN, int L, int STOP, int FA>
struct SolveStage<false, M, SIGN, L, STOP, FA> : WideStage<M, SIGN, L, STOP, FA> {};

// The untangling of one bin k: packed bin X and its mirror bin Y -> the input
// of the half-length complex transform, and that transform's output Z (mirror
// Y) -> the packed bin.  Bin 0 carries (X[0], X[N/2]).
template <int N>
__device__ __forceinline__ float2 c2r_bin(float2 X, float2 Y, int k, const RowTw<N>& tw) {
  if (k == 0) return f2(X.x + X.y, X.x - X.y);
  Y = conjf2(Y);
  return X + Y + mul_si<+1>(tw_times<+1, +1>(X - Y, tw.u[k]));
}
template <int N>
__device__ __forceinline__ float2 r2c_bin(float2 Z, float2 Y, int k, const RowTw<N>& tw) {
  if (k == 0) return f2(Z.x + Z.y, Z.x - Z.y);
  Y = conjf2(Y);
  return 0.5f * (Z + Y + mul_si<-1>(tw_times<-1, -1>(Z - Y, tw.u[k])));
}

// Sensor gather (gather_row) by the T lanes of a row.
template <int T>
__device__ __forceinline__ void solve_gather(const DevPlan& P, int n, const float* Lf, int row, int t) {
  WaveSync::sync();
  const int e1 = gld(P.g_ptr, row + 1);
  float* out = P.partial + (long)n * P.nslots;
  for (int e0 = gld(P.g_ptr, row) + t; e0 < e1; e0 += 4 * T) {
    GTap tp[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) tp[u] = gld(P.g_tap, e0 + u * T < e1 ? e0 + u * T : e0);
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (e0 + u * T < e1) gst(out, tp[u].slot, fmaf(tp[u].w0, Lf[tp[u].x0], tp[u].w1 * Lf[tp[u].x0 + 1]));
  }
  WaveSync::sync();
}

// ---------------------------------------------------------------- geometry
template <int NX, int NY>
struct SolveGeo {
  static constexpr int WHOLE = solve_whole(NX, NY);
  static constexpr int NW = solve_nw(NX, NY), NTH = 64 * NW;
  // rows: TR threads of the eight-value transform, RPW rows per wavefront
  static constexpr int M = NX / 2, ER = 4, TR = M / 8, RL = M / ER;
  static constexpr int RPW = 64 / RL;          // rows per wavefront
  static constexpr int units = NY / RPW;       // wavefront row units
  static constexpr int groups = units / (NW / 2);
  // columns, likewise
  static constexpr bool PC = solve_pair_col(NY);
  static constexpr int EC = PC ? 4 : 8, TC = NY / 8, CL = NY / EC;
  static constexpr int LDT = NY + NY / 8 - 1;  // column stride in LDS (padded exchange, odd)
  static_assert(RL <= 64 && CL <= 64 && units % (NW / 2) == 0, "a row or column must fit a wavefront");
  // exchange region of a wavefront: its rows, or its share of the columns
  static constexpr int rreg = RPW * RowGeo<NX>::LDR, creg = (64 / CL) * LDT;
  static constexpr int region = rreg > creg ? rreg : creg;
};

struct SolveShared {
  uint32_t fail;  // barrier at which a wait ran out (0: none)
  int rank, n, xr, nx;
  uint32_t claim;
};
template <int NX, int NY>
struct SolveLds {
  using G = SolveGeo<NX, NY>;
  float2 ex[G::NW * G::region];
  float2 px[G::NW * 64 * (G::EC > G::ER ? G::EC : G::ER)];  // what the two parts of a tile hand each other
  RowTw<NX> row_tw;
  alignas(16) Tw col_tw[staged_len(NY, 8)];
  SolveShared c;
};

// ---------------------------------------------------------------- domain
#define PAT_AGENT_LD(p) __hip_atomic_load((p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
#define PAT_AGENT_ST(p, v) __hip_atomic_store((p), (v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
#define PAT_AGENT_ADD(p, v) __hip_atomic_fetch_add((p), (v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)

template <int WHOLE>
struct Domain {
  SolveDom* d;
  SolveShared* sh;
  int rank, n;    // this member, of n
  int x, xr, nx;  // this member's die, its place there, members there
  uint32_t* flag; // the flags of this die's members
  uint32_t dies;  // dies with members
  uint32_t epoch;
  int polls;      // left to a wait; 0 once one ran out

  __device__ __forceinline__ static bool reached(const uint32_t* w, uint32_t epoch) {
    return (int32_t)(PAT_AGENT_LD(w) - epoch) >= 0;
  }

  // The barrier between two passes, in two halves: arrive() once this block's
  // stores of the pass are issued, wait() before its first load of what other
  // members stored.  Loads of the block's own rows go between the two.
  __device__ __forceinline__ void arrive() {
    ++epoch;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (n > 1 && threadIdx.x < 64) {
      const int lane = (int)threadIdx.x;
      if (!WHOLE || xr != 0) {
        if (lane == 0) PAT_AGENT_ST(&flag[solve_flag(xr)], epoch);
      } else {
        // the first member of a die waits for its others
        for (int k = 1; k < nx; k += 64) poll(&flag[solve_flag(k + lane < nx ? k + lane : k)]);
        // (a copy per die: its members poll lines that no other die's poll)
        if (lane < kSolveXcds) PAT_AGENT_ST(&d[lane].lead[x * kSolveLine], epoch);
      }
    }
  }
  __device__ __forceinline__ void wait() {
    if (n > 1) {
      if (threadIdx.x < 64) {
        const int lane = (int)threadIdx.x;
        if (!WHOLE) poll(&flag[solve_flag(lane < nx ? lane : xr)]);
        else poll(&d[x].lead[((dies >> (lane & 7)) & 1 ? (lane & 7) : x) * kSolveLine]);
      }
      __syncthreads();
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  }
  // until every lane's word has reached this barrier; marks the block when that never happens
  __device__ __forceinline__ void poll(const uint32_t* w) {
    int spin = 0;
    while (!__all(reached(w, epoch)) && ++spin < polls) {
    }
    if (spin >= polls) {
      if (polls != 0 && (threadIdx.x & 63) == 0) sh->fail = epoch;
      polls = 0;
    }
  }
  // Whether a wait of this block ran out before the last arrive(), whose
  // block barrier makes every wavefront see it alike (one that runs out
  // meanwhile in the first wavefront carries the current epoch).
  __device__ __forceinline__ bool failed() const {
    const uint32_t f = (uint32_t)__builtin_amdgcn_readfirstlane((int)sh->fail);
    return f != 0 && (int32_t)(f - epoch) < 0;
  }
};

// Joins a domain of this block's die (WHOLE: the one domain); false for a
// block that is not needed.
template <int WHOLE>
__device__ __forceinline__ bool join_domain(const SolveArgs& a, SolveShared& sh, Domain<WHOLE>& dm) {
  const int x = (int)(__builtin_amdgcn_s_getreg(20 | (31 << 11)) & (kSolveXcds - 1));  // XCC_ID
  if (threadIdx.x == 0) {
    sh.fail = 0u;
    sh.n = 0;
    const uint32_t ticket = PAT_AGENT_ADD(&a.ctl->ticket[WHOLE ? 0 : x][0], 1u);
    const int k = (int)(ticket / (uint32_t)a.members);
    if (k < a.domains) {
      SolveDom* d = &a.doms[WHOLE ? 0 : x * a.domains + k];
      const uint32_t old = PAT_AGENT_ADD(&d->roll, 1u);
      if (!(old & kSolveClosed)) {
        sh.rank = (int)old;
        sh.xr = WHOLE ? (int)PAT_AGENT_ADD(&d->count[x], 1u) : (int)old;
        __hip_atomic_fetch_add(&d->ready, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
        int spin = 0;
        uint32_t v = 1;
        if (old == 0) {
          // The first member closes the roll: complete, or once it has waited
          // as long as the solve would take longer with the members there
          // (n of m take ceil(m / n) times the time), or when no instance is left.
          const uint64_t t0 = wall_clock64();
          for (;;) {
            v = PAT_AGENT_LD(&d->roll);
            const uint64_t more = ((uint32_t)a.members + v - 1) / v - 1, waited = wall_clock64() - t0;
            if (more == 0 || waited >= more * a.solve_ticks || waited >= kSolveRollTicks ||
                PAT_AGENT_LD(&a.ctl->claimed) >= (uint32_t)a.first[kSolveXcds])
              break;
          }
          v = __hip_atomic_fetch_or(&d->roll, kSolveClosed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          while (__hip_atomic_load(&d->ready, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT) < v && ++spin < a.polls) {
          }
          // (a member that has not counted itself yet: the domain does not start)
          if (spin >= a.polls) v = 0;
          PAT_AGENT_ST(&d->n, v ? v : kSolveClosed);
        } else {
          while (!(v = PAT_AGENT_LD(&d->n)) && ++spin < a.polls) {
          }
          if (v == kSolveClosed) v = 0;
        }
        sh.n = (int)v;  // 0: gave up
        sh.nx = WHOLE ? (int)PAT_AGENT_LD(&d->count[x]) : (int)v;
      }
      sh.claim = WHOLE ? 0u : (uint32_t)(x * a.domains + k);
    }
  }
  __syncthreads();
  if (sh.n == 0) return false;
  dm.d = &a.doms[__builtin_amdgcn_readfirstlane((int)sh.claim)];
  dm.sh = &sh;
  dm.rank = __builtin_amdgcn_readfirstlane(sh.rank);
  dm.n = __builtin_amdgcn_readfirstlane(sh.n);
  dm.x = x;
  dm.xr = __builtin_amdgcn_readfirstlane(sh.xr);
  dm.nx = __builtin_amdgcn_readfirstlane(sh.nx);
  dm.dies = 0;
  dm.flag = a.doms[WHOLE ? x : (int)(dm.d - a.doms)].flag;
  if (WHOLE)
    for (int y = 0; y < kSolveXcds; ++y) {
      const int c = __builtin_amdgcn_readfirstlane((int)PAT_AGENT_LD(&dm.d->count[y]));
      if (c > 0) dm.dies |= 1u << y;
    }
  dm.epoch = 0;
  dm.polls = a.polls;
  __syncthreads();
  return true;
}

// The domain's next instance: its own die's list first, then the others'.
// -1: every list is empty.
template <int WHOLE>
__device__ __forceinline__ int claim_instance(const SolveArgs& a, Domain<WHOLE>& dm, uint32_t seq) {
  if (threadIdx.x == 0) {
    uint32_t got = 0;
    if (dm.rank == 0) {
      for (int k = 0; k < kSolveXcds && !got; ++k) {
        const int y = (dm.x + k) & (kSolveXcds - 1);
        const int beg = a.first[y], len = a.first[y + 1] - beg;
        if (len <= 0) continue;
        const uint32_t i = PAT_AGENT_ADD(&a.ctl->head[y][0], 1u);
        if (i < (uint32_t)len) got = (uint32_t)beg + i + 1;
      }
      if (got) PAT_AGENT_ADD(&a.ctl->claimed, 1u);
      dm.sh->claim = got;
      if (dm.n > 1) PAT_AGENT_ST(&dm.d->claim, (seq << 16) | got);
    } else {
      int spin = 0;
      uint32_t v;
      while (((v = PAT_AGENT_LD(&dm.d->claim)) >> 16) != (seq & 0xffffu))
        if (++spin > a.polls) {
          v = 0;
          break;
        }
      dm.sh->claim = v & 0xffffu;
    }
  }
  __syncthreads();
  const int got = (int)dm.sh->claim - 1;
  __syncthreads();
  return __builtin_amdgcn_readfirstlane(got);
}

// ---------------------------------------------------------------- passes
// The plan record, through the constant address space: its fields are scalar
// loads (the kernel writes memory, but never a record) that stay in scalar
// registers through the time loop.  Read again in every pass, the dependent
// loads (sizes, then pointers, then data) took some 1500 cycles of it.
__device__ __forceinline__ const DevPlan* constant(const DevPlan* p) {
#if defined(__HIP_DEVICE_COMPILE__)
  const uint64_t v = (uint64_t)p;
  const uint64_t u = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(v >> 32)) << 32 |
                     (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
  return (const DevPlan*)(const __attribute__((address_space(4))) DevPlan*)u;
#else
  return p;
#endif
}
// spectra: loads past the L1; across dies the stores are written through
template <int WHOLE>
__device__ __forceinline__ void put(float2* p, long i, float2 v) {
  if constexpr (WHOLE) gst_agent(p, i, v);
  else gst(p, i, v);
}
__device__ __forceinline__ int opaque(int t) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("" : "+v"(t));  // a pass's index arithmetic stays in that pass
#endif
  return t;
}

// Real transforms of the rows of one wavefront (c2r and r2c on pairs of lanes).
template <class G, int NX>
__device__ __forceinline__ void solve_mirror(const float2 (&r)[G::ER], float2 (&y)[G::ER], int t, int h) {
  // element 4 h + i of lane t: element 3 - i of lane T - t's other half, or
  // for t = 0 element 4 - i of its own other half (i = 0: itself)
  constexpr int T = G::TR;
  const int lane = (int)(threadIdx.x & 63);
  const int src = ((lane & 31 & ~(T - 1)) | ((T - t) & (T - 1)) | (h ? 0 : 32)) << 2;
  float2 q[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    q[i].x = __int_as_float(__builtin_amdgcn_ds_bpermute(src, __float_as_int(r[3 - i].x)));
    q[i].y = __int_as_float(__builtin_amdgcn_ds_bpermute(src, __float_as_int(r[3 - i].y)));
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) y[i] = sel2(t == 0, i == 0 ? r[0] : q[i > 0 ? i - 1 : 0], q[i]);
}
template <class G, int NX>
__device__ __forceinline__ void solve_c2r(float2 (&r)[G::ER], float2* L, int t, int h, const RowTw<NX>& tw) {
  float2 y[G::ER];
  solve_mirror<G, NX>(r, y, t, h);
#pragma unroll
  for (int m = 0; m < G::ER; ++m) r[m] = c2r_bin(r[m], y[m], t + G::TR * (m + (h ? 4 : 0)), tw);
  WaveSync::sync();  // earlier readers of the row's region are done
  PairStage<G::M, +1, 1>::run(r, L, t, h, tw.s);
}
template <class G, int NX>
__device__ __forceinline__ void solve_r2c_bins(float2 (&r)[G::ER], int t, int h, const RowTw<NX>& tw) {
  float2 y[G::ER];
  solve_mirror<G, NX>(r, y, t, h);
#pragma unroll
  for (int m = 0; m < G::ER; ++m) r[m] = r2c_bin(r[m], y[m], t + G::TR * (m + (h ? 4 : 0)), tw);
}
template <class G, int NX>
__device__ __forceinline__ void solve_r2c(float2 (&r)[G::ER], float2* L, int t, int h, const RowTw<NX>& tw) {
  PairStage<G::M, -1, 1>::run(r, L, t, h, tw.s);
  solve_r2c_bins<G, NX>(r, t, h, tw);
}
// ... of the products a b (the adjoint's state and density passes, whose
// products the compiler contracts into the first butterflies)
template <class G, int NX>
__device__ __forceinline__ void solve_r2c_products(const float2 (&a)[G::ER], const float2 (&b)[G::ER],
                                                   float2 (&r)[G::ER], float2* L, int t, int h, const RowTw<NX>& tw) {
  using St = PairStage<G::M, -1, 1, G::M, -1, true>;
  St::products(a, b, r, h);
  St::run(r, L, t, h, tw.s);
  solve_r2c_bins<G, NX>(r, t, h, tw);
}

// One row pass: part j (component or term) of the rows of one wavefront.
// Arithmetic as the row pass of the same kind (passes_row.h).
template <int NX, int NY, int K>
__device__ __forceinline__ void solve_row_part(const DevPlan& P, int unit, int j, int it, int wave,
                                               Domain<solve_whole(NX, NY)>& dm, bool first_unit, SolveLds<NX, NY>& sh) {
  using G = SolveGeo<NX, NY>;
  constexpr int E = G::ER, T = G::TR, M = G::M, RL = G::RL;
  const int lane = opaque((int)(threadIdx.x & 63));
  const int h = lane >> 5, l = lane & 31;
  const int rl = l / T, t = l % T, tr = h * T + t;  // tr: lane of the row
  const int row = unit * G::RPW + rl;
  const int e0 = t + (h ? 4 * T : 0);               // this lane's elements: e0 + T m
  const long base = (long)row * M + e0;
  float2* L = sh.ex + wave * G::region + rl * RowGeo<NX>::LDR;
  float* Lf = reinterpret_cast<float*>(L);
  float2* mine = sh.px + wave * 64 * E;
  const float2* other = sh.px + (wave ^ (G::NW / 2)) * 64 * E;
  const auto& tws = sh.row_tw;
  // the spectrum of the pass before: after every load of this member's own
  auto lds = [&](const float2* a, float2(&v)[E]) {
    if (first_unit) dm.wait();
#pragma unroll
    for (int m = 0; m < E; ++m) v[m] = gld_agent(a, base + T * m);
  };
  auto ldf = [&](const float* a, float2(&v)[E]) {
#pragma unroll
    for (int m = 0; m < E; ++m) v[m] = ld2(a, base + T * m);
  };
  auto stf = [&](float* a, const float2(&v)[E]) {
#pragma unroll
    for (int m = 0; m < E; ++m) st2(a, base + T * m, v[m]);
  };
  // PML factor of axis j at this lane's points
  auto pml = [&](const float* const* tab, float2(&q)[E]) {
    if (j == 0) {
#pragma unroll
      for (int m = 0; m < E; ++m) q[m] = ld2(tab[0], e0 + T * m);
    } else {
      const float f = gld(tab[1], row);
#pragma unroll
      for (int m = 0; m < E; ++m) q[m] = f2(f, f);
    }
  };
  auto zero = [&](float2(&v)[E]) {
#pragma unroll
    for (int m = 0; m < E; ++m) v[m] = f2(0.f, 0.f);
  };
  auto send = [&](const float2(&v)[E]) {
#pragma unroll
    for (int m = 0; m < E; ++m) mine[lane + 64 * m] = v[m];
  };
  auto receive = [&](float2(&v)[E]) {
#pragma unroll
    for (int m = 0; m < E; ++m) v[m] = other[lane + 64 * m];
  };
  // real row -> its packed spectrum in S
  auto out = [&](float2(&v)[E], float2* S) {
    solve_r2c<G, NX>(v, L, t, h, tws);
#pragma unroll
    for (int m = 0; m < E; ++m) put<G::WHOLE>(S, base + T * m, v[m]);
  };
  auto out_products = [&](const float2(&a)[E], const float2(&b)[E], float2* S) {
    float2 v[E];
    solve_r2c_products<G, NX>(a, b, v, L, t, h, tws);
#pragma unroll
    for (int m = 0; m < E; ++m) put<G::WHOLE>(S, base + T * m, v[m]);
  };
  // the pressure of this row: finite check, sensors, spectrum
  auto record = [&](float2(&p)[E]) {
#pragma unroll
    for (int m = 0; m < E; ++m) {
      check_finite(P, p[m]);
      L[e0 + T * m] = p[m];
    }
    solve_gather<RL>(P, it + 1, Lf, row, tr);
    out(p, P.S[0]);
  };

  if constexpr (K == R_FWD_1 || K == R_ADJ_1) {
    const bool first = (it == 0), last = (K == R_ADJ_1) && (it == P.nt - 2);
    float2 d[E], b[E], u[E], qs[E];
    ldf(P.B[j], b);
    if (first) zero(u);
    else ldf(P.u[j], u);
    pml(P.Qsg, qs);
    lds(P.S[1 + j], d);
    solve_c2r<G, NX>(d, L, t, h, tws);
#pragma unroll
    for (int m = 0; m < E; ++m) {
      if constexpr (K == R_FWD_1) {
        u[m] = velocity(u[m], d[m], b[m], qs[m], first);
        d[m] = u[m];
      } else {
        adj_velocity(u[m], d[m], b[m], qs[m], last);
      }
    }
    if (K == R_FWD_1 || !last) stf(P.u[j], u);
    out(d, P.S[1 + j]);
  } else if constexpr (K == R_FWD_2 || K == R_FWD_2LL) {
    float2 g[E], r[E], dr[E], q[E], v[E];
    ldf(P.r[j], r);
    ldf(P.dtr0, dr);
    pml(P.Q, q);
    float2 c2[E];
    if constexpr (K == R_FWD_2LL) ldf(P.c2, c2);
    lds(P.S[1 + j], g);
    solve_c2r<G, NX>(g, L, t, h, tws);
    // rho_j <- Q (Q rho_j - t_j), t_j = dt rho0 g_j
#pragma unroll
    for (int m = 0; m < E; ++m) {
      g[m] = mul2(dr[m], g[m]);
      r[m] = mul2(q[m], fma2(q[m], r[m], neg2(g[m])));
    }
    stf(P.r[j], r);
    if constexpr (K == R_FWD_2) {
      // part 0: the divergence sum; part 1: the density sum
      if (j == 0) send(r);
      else send(g);
      __syncthreads();
      receive(v);
#pragma unroll
      for (int m = 0; m < E; ++m) v[m] = j == 0 ? g[m] + v[m] : v[m] + r[m];
      out(v, P.S[1 + j]);
    } else {
      // part 1: the density sum and the equation of state
      if (j == 0) send(r);
      __syncthreads();
      if (j == 1) {
        receive(v);
#pragma unroll
        for (int m = 0; m < E; ++m) v[m] = mul2(c2[m], v[m] + r[m]);
        record(v);
      }
    }
  } else if constexpr (K == R_FWD_3) {
    // part 0 transforms A1, part 1 A2 for part 0's equation of state
    float2 a[E], c2[E], r0[E], r1[E], ct[E], ce[E];
    if (j == 0) {
      ldf(P.c2, c2);
      ldf(P.r[0], r0);
      ldf(P.r[1], r1);
      if (!P.alpha_uniform) {
        ldf(P.c2tau, ct);
        ldf(P.c2eta, ce);
      } else {
        absorption_coefs<E>(P, c2, ct, ce);
      }
    }
    lds(P.S[1 + j], a);
    solve_c2r<G, NX>(a, L, t, h, tws);
    if (j == 1) send(a);
    __syncthreads();
    if (j == 0) {
      float2 v[E];
      receive(v);
#pragma unroll
      for (int m = 0; m < E; ++m) a[m] = pressure(c2[m], r0[m] + r1[m], ct[m], a[m], ce[m], v[m]);
      record(a);
    }
  } else if constexpr (K == R_ADJ_3 || K == R_ADJ_32LL) {
    // both parts form v (the transposed state's input); part 0 the eta term
    // (or the x density), part 1 the tau term (the y density)
    const bool first = (it == 0);
    const int nsamp = P.nt - 1 - it;
    float2 v[E], c2[E], cf[E], q[E], r[E];
    ldf(P.c2, c2);
    if constexpr (K == R_ADJ_3) {
      if (!P.alpha_uniform) ldf(j == 0 ? P.c2eta : P.c2tau, cf);
    } else {
      ldf(P.dtr0, cf);
      pml(P.Q, q);
      if (first) zero(r);
      else ldf(P.r[j], r);
    }
    const int sp0 = gld(P.s_ptr, row) + tr, sp1 = gld(P.s_ptr, row + 1);
    const float* sc = P.sc + (long)nsamp * P.ngroups;
    int sx = -1;
    float sv = 0.f;
    if (sp0 < sp1) {
      sx = gld(P.s_grp, sp0).x;
      sv = gld(sc, sp0);
    }
    if constexpr (K == R_ADJ_3) {
      if (P.alpha_uniform) {
        float2 ct[E], ce[E];
        absorption_coefs<E>(P, c2, ct, ce);
#pragma unroll
        for (int m = 0; m < E; ++m) cf[m] = j == 0 ? ce[m] : ct[m];
      }
    }
    if (first) zero(v);
    else lds(P.S[0], v);
    if (!first) solve_c2r<G, NX>(v, L, t, h, tws);
#pragma unroll
    for (int m = 0; m < E; ++m) L[e0 + T * m] = v[m];
    WaveSync::sync();
    if (sx >= 0) {
      Lf[sx] += sv;
      for (int g0 = sp0 + RL; g0 < sp1; g0 += 4 * RL) {
        int gx[4];
        float gs[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int g = g0 + u * RL < sp1 ? g0 + u * RL : sp0;
          gx[u] = gld(P.s_grp, g).x;
          gs[u] = gld(sc, g);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (g0 + u * RL < sp1) Lf[gx[u]] += gs[u];
      }
    }
    WaveSync::sync();
#pragma unroll
    for (int m = 0; m < E; ++m) v[m] = L[e0 + T * m];
    WaveSync::sync();
    if constexpr (K == R_ADJ_3) {
#pragma unroll
      for (int m = 0; m < E; ++m) c2[m] = mul2(c2[m], v[m]);
      if (j == 0) stf(P.q, c2);
      out_products(cf, v, P.S[1 + j]);
    } else {
#pragma unroll
      for (int m = 0; m < E; ++m) {
        v[m] = adj_density_ll(r[m], c2[m], v[m], cf[m], q[m]);
      }
      stf(P.r[j], r);
      out(v, P.S[1 + j]);
    }
  } else if constexpr (K == R_ADJ_2) {
    // part 0 transforms A2, part 1 A1; both then update their component
    const bool first = (it == 0);
    float2 a[E], v[E], q[E], dr[E], qq[E], r[E];
    ldf(P.q, q);
    ldf(P.dtr0, dr);
    pml(P.Q, qq);
    if (first) zero(r);
    else ldf(P.r[j], r);
    lds(P.S[1 + j], a);
    solve_c2r<G, NX>(a, L, t, h, tws);
    send(a);
    __syncthreads();
    receive(v);
#pragma unroll
    for (int m = 0; m < E; ++m) {
      const float2 a2 = q[m] - (j == 0 ? a[m] : v[m]), a1 = j == 0 ? v[m] : a[m];
      v[m] = adj_density(r[m], a2, a1, qq[m]);
    }
    stf(P.r[j], r);
    out_products(dr, v, P.S[1 + j]);
  }
}

// Row pass of every unit of this member: wavefronts 0 .. NW/2 - 1 run part 0,
// the others part 1 of the same rows.
template <int NX, int NY, int K>
__device__ __forceinline__ void solve_row(const DevPlan& P, int it, Domain<solve_whole(NX, NY)>& dm,
                                          SolveLds<NX, NY>& sh) {
  using G = SolveGeo<NX, NY>;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int j = wave / (G::NW / 2);
  for (int g = dm.rank; g < G::groups; g += dm.n) {
    if (g != dm.rank) __syncthreads();  // what the parts handed each other has been read
    solve_row_part<NX, NY, K>(P, g * (G::NW / 2) + wave % (G::NW / 2), j, it, wave, dm, g == dm.rank, sh);
  }
}

// The multipliers of one column pass at this lane's elements: at its x-bin
// and, for the packed column 0, the second factor of its mirror bins.  A
// member keeps the tiles it has through the time loop, and their multipliers
// stay in registers (unit: whose they are).
template <int E>
struct ColMult {
  float2 mv[E], mN[E];
  int unit;
  __device__ __forceinline__ float2 at(int m) const { return mv[m]; }
  __device__ __forceinline__ float2 mirror(int m) const { return mN[m]; }
  __device__ __forceinline__ void set(int m, float2 v) { mv[m] = v; }
  __device__ __forceinline__ void set_mirror(int m, float2 v) { mN[m] = v; }
};
template <int E>
struct RealMult {  // Laplacians: real
  float mv[E], mN[E];
  int unit;
  __device__ __forceinline__ float2 at(int m) const { return f2(mv[m], 0.f); }
  __device__ __forceinline__ float2 mirror(int m) const { return f2(mN[m], 0.f); }
  __device__ __forceinline__ void set(int m, float2 v) { mv[m] = v.x; }
  __device__ __forceinline__ void set_mirror(int m, float2 v) { mN[m] = v.x; }
};
template <int E, int FAM>
using MultOf = typename std::conditional<FAM == F_ABS, RealMult<E>, ColMult<E>>::type;

// One column pass over tile `tile` of NTHT threads (mapping and transforms as
// colm_pass): part j's input, multiplier and output.
//   MODE 0  S[1 + j] <- m_j S[0]        MODE 1  S[1 + j] <- m_j S[1 + j]
//   MODE 2  S[0] <- m_0 S[1] + m_1 S[2], the parts in the two halves of the block
// SWAP (Laplacians): part 0 applies |k|^(y-1), part 1 |k|^(y-2)/dt.
template <int NX, int NY, int MODE, int FAM, int SWAP>
__device__ __forceinline__ void solve_col_part(const DevPlan& P, int tile, int j, int unit,
                                               Domain<solve_whole(NX, NY)>& dm, bool first_unit, SolveLds<NX, NY>& sh,
                                               MultOf<SolveGeo<NX, NY>::EC, FAM>& cm) {
  using G = SolveGeo<NX, NY>;
  constexpr int NTHT = MODE == 2 ? G::NTH / 2 : G::NTH;
  constexpr int E = G::EC, TC = G::TC, LDT = G::LDT, TILE = NTHT / G::CL, M = G::M;
  constexpr bool PC = G::PC;
  auto sync = [] {
    if constexpr (NTHT == 64) WaveSync::sync();
    else __syncthreads();
  };
  const int tid = opaque((int)threadIdx.x - (MODE == 2 ? j * NTHT : 0));
  // pairs of lanes: half h of the wavefront holds the elements from 4 h on
  const int h = PC ? (tid >> 5) & 1 : 0, q = PC ? (tid >> 6) * 32 + (tid & 31) : tid;
  const int ca = q % TILE, ta = q / TILE, cb = q / TC, tb = q % TC;
  const int ea = ta + (h ? 4 * TC : 0), eb = tb + (h ? 4 * TC : 0);  // this lane's elements: ea / eb + TC m
  float2* ex = sh.ex + (MODE == 2 ? j * (G::NW / 2) * G::region : 0);
  float2* La = ex + ca * LDT;
  float2* Lb = ex + cb * LDT;
  const int c0 = tile * TILE;
  const bool valid = M >= TILE || ca < M;  // lanes past a narrow grid's last column
  const int ka = c0 + (valid ? ca : 0), kb = c0 + ((M >= TILE || cb < M) ? cb : 0);
  const bool special = tile == 0, fix = special && cb == 0;  // packed column 0

  // multipliers of this lane's elements (mapping B), at x-bin kb and, for the
  // packed column 0, at x-bin NX / 2
  constexpr bool DERIV = FAM != F_ABS;
  // packed column 0 holds C = A + iB: 1/2 (m0 + mN) C + 1/2 (m0 - mN) conj(C(-k)),
  // mN = g sh; mN[] takes the second factor there
  auto packed = [&](int m, float g, float2 sh) {
    const float2 gg = f2(g, g), p = 0.5f * fma2(gg, sh, cm.at(m)), q = 0.5f * fma2(neg2(gg), sh, cm.at(m));
    cm.set_mirror(m, q);
    cm.set(m, sel2(fix, p, cm.at(m)));
  };
  if (cm.unit != unit) {
    cm.unit = unit;
    const float k2x = gld(P.ksq[0], kb), k2N = gld(P.ksq[0], M);
    float k2[E];
#pragma unroll
    for (int m = 0; m < E; ++m) k2[m] = gld(P.ksq[1], eb + TC * m);
    if constexpr (DERIV) {
      const float2* const* tab = FAM == F_A ? P.shA : P.shB;
      float2 sx[E], sN;
      if (j == 0) {
        const float2 f = gld(tab[0], kb);
        sN = gld(tab[0], M);
#pragma unroll
        for (int m = 0; m < E; ++m) sx[m] = f;
      } else {
#pragma unroll
        for (int m = 0; m < E; ++m) sx[m] = gld(tab[1], eb + TC * m);
      }
#pragma unroll
      for (int m = 0; m < E; ++m) {
        cm.set(m, scl2(sinc_sqrt(P.kap2 * (k2x + k2[m])) * P.scale, sx[m]));
        if (special) packed(m, sinc_sqrt(P.kap2 * (k2N + k2[m])) * P.scale, j == 0 ? sN : sx[m]);
      }
    } else {
      const bool l1 = (j == 0) != (SWAP != 0);
      const float e = l1 ? P.ym2h : P.ym1h;
      auto lapl = [&](float q) {
        const float lk = __builtin_amdgcn_logf(q);
        const float w = lk > -INFINITY ? __builtin_amdgcn_exp2f(e * lk) : 0.f;
        return l1 ? w * P.inv_dt : w;
      };
#pragma unroll
      for (int m = 0; m < E; ++m) {
        cm.set(m, f2(lapl(k2x + k2[m]) * P.scale, 0.f));
        if (special) packed(m, lapl(k2N + k2[m]), f2(P.scale, 0.f));
      }
    }
  }
  if (first_unit) dm.wait();
  const float2* src = MODE == 0 ? P.S[0] : P.S[1 + j];
  float2 v[E], s[E];
#pragma unroll
  for (int m = 0; m < E; ++m) v[m] = gld_agent(src, (long)(ea + TC * m) * M + ka);
  SolveStage<PC, NY, -1, 1, 8>::run(v, La, ta, h, nullptr);
  sync();
#pragma unroll
  for (int m = 0; m < E; ++m) s[m] = Lb[pad8(eb + TC * m)];
  WaveSync::sync();
  SolveStage<PC, NY, -1, 8>::run(s, Lb, tb, h, sh.col_tw);
  float2 w[E];  // the mirror bins' product at the packed column 0
  if (special) {
    if (fix) {
#pragma unroll
      for (int m = 0; m < E; ++m) Lb[eb + TC * m] = s[m];
    }
    WaveSync::sync();
#pragma unroll
    for (int m = 0; m < E; ++m) w[m] = cmul(cm.mirror(m), conjf2(Lb[(NY - (eb + TC * m)) & (NY - 1)]));
    WaveSync::sync();
  }
#pragma unroll
  for (int m = 0; m < E; ++m) v[m] = cmul(cm.at(m), s[m]);
  if (fix && (MODE != 2 || j == 0)) {
#pragma unroll
    for (int m = 0; m < E; ++m) v[m] = v[m] + w[m];
  }
  if constexpr (MODE == 2) {
    if (j == 1) {
#pragma unroll
      for (int m = 0; m < E; ++m) sh.px[tid + NTHT * m] = v[m];
      if (special) {
#pragma unroll
        for (int m = 0; m < E; ++m) sh.px[NTHT * E + tid + NTHT * m] = w[m];
      }
    }
    __syncthreads();
    if (j == 0) {
#pragma unroll
      for (int m = 0; m < E; ++m) v[m] = v[m] + sh.px[tid + NTHT * m];
      if (fix) {
#pragma unroll
        for (int m = 0; m < E; ++m) v[m] = v[m] + sh.px[NTHT * E + tid + NTHT * m];
      }
    }
  }
  // (mode 2: part 1 runs the inverse along for the block's barriers)
  constexpr int LS = fft_last_span(NY, 8);
  SolveStage<PC, NY, +1, 1, LS>::run(v, Lb, tb, h, sh.col_tw);
  sync();
#pragma unroll
  for (int m = 0; m < E; ++m) s[m] = La[pad8(ea + TC * m)];
  SolveStage<PC, NY, +1, LS, NY, -1>::run(s, nullptr, ta, h, sh.col_tw);  // (the other contraction)
  if (valid && (MODE != 2 || j == 0)) {
    float2* dst = MODE == 2 ? P.S[0] : P.S[1 + j];
#pragma unroll
    for (int m = 0; m < E; ++m) put<G::WHOLE>(dst, (long)(ea + TC * m) * M + ka, s[m]);
  }
}

template <int NX, int NY, int MODE, int FAM, int SWAP = 0>
__device__ __forceinline__ void solve_col(const DevPlan& P, Domain<solve_whole(NX, NY)>& dm, SolveLds<NX, NY>& sh,
                                          MultOf<SolveGeo<NX, NY>::EC, FAM>& cm) {
  using G = SolveGeo<NX, NY>;
  constexpr int NTHT = MODE == 2 ? G::NTH / 2 : G::NTH;
  constexpr int TILE = NTHT / G::CL, tiles = (G::M + TILE - 1) / TILE;
  constexpr int units = MODE == 2 ? tiles : 2 * tiles;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  for (int u = dm.rank; u < units; u += dm.n) {
    if (u != dm.rank) __syncthreads();  // the previous tile's last reads of the regions
    const int j = MODE == 2 ? wave / (G::NW / 2) : (u >= tiles ? 1 : 0);
    solve_col_part<NX, NY, MODE, FAM, SWAP>(P, MODE == 2 ? u : u - j * tiles, j, u, dm, u == dm.rank, sh, cm);
  }
}

// ---------------------------------------------------------------- the kernel
// Steps [s0, s1) (s1 < 0: to the last) of direction DIR of every queued
// instance, between the launches of the initial and the final pass.  At most
// 168 registers, three wavefronts per SIMD: with 188 only two domains over
// every die fit side by side, and the members that a third one missed cost it
// its speed (three 512^2 adjoints and three 64^2 forwards on streams of their
// own, 200 steps: 43 ms, 14 ms with 168; launches 21 ms).
template <int NX, int NY, int DIR, int LOSSY>
__global__ void __launch_bounds__((SolveGeo<NX, NY>::NTH), 3) k_solve(SolveArgs a) {
  using G = SolveGeo<NX, NY>;
  constexpr int WHOLE = G::WHOLE;
  __shared__ SolveLds<NX, NY> sh;
  Domain<WHOLE> dm;
  if (!join_domain<WHOLE>(a, sh.c, dm)) return;
  load_row_twiddles<NX, G::NTH>(sh.row_tw, a.tw);
  load_table<staged_len(NY, 8), G::NTH>(sh.col_tw, a.tw, [](int i) { return staged_src<NY, 8>(i); });
  __syncthreads();
  for (uint32_t seq = 1;; ++seq) {
    const int inst = claim_instance<WHOLE>(a, dm, seq);
    if (inst < 0) return;
    const DevPlan& P = *constant(a.list ? a.list[inst] : a.one);
    const int s1 = a.s1 < 0 ? P.nt - 1 : a.s1;
    ColMult<G::EC> ma, mb;
    RealMult<G::EC> ml;
    ma.unit = mb.unit = ml.unit = -1;
    for (int it = a.s0; it < s1; ++it) {
      if constexpr (DIR == 0) {
        solve_col<NX, NY, 0, F_A>(P, dm, sh, ma);
        dm.arrive();
        solve_row<NX, NY, R_FWD_1>(P, it, dm, sh);
        dm.arrive();
        solve_col<NX, NY, 1, F_B>(P, dm, sh, mb);
        dm.arrive();
        if constexpr (LOSSY) {
          solve_row<NX, NY, R_FWD_2>(P, it, dm, sh);
          dm.arrive();
          solve_col<NX, NY, 1, F_ABS, 0>(P, dm, sh, ml);
          dm.arrive();
          solve_row<NX, NY, R_FWD_3>(P, it, dm, sh);
        } else {
          solve_row<NX, NY, R_FWD_2LL>(P, it, dm, sh);
        }
        dm.arrive();
      } else {
        if constexpr (LOSSY) {
          solve_row<NX, NY, R_ADJ_3>(P, it, dm, sh);
          dm.arrive();
          solve_col<NX, NY, 1, F_ABS, 1>(P, dm, sh, ml);
          dm.arrive();
          solve_row<NX, NY, R_ADJ_2>(P, it, dm, sh);
        } else {
          solve_row<NX, NY, R_ADJ_32LL>(P, it, dm, sh);
        }
        dm.arrive();
        solve_col<NX, NY, 1, F_A>(P, dm, sh, ma);
        dm.arrive();
        solve_row<NX, NY, R_ADJ_1>(P, it, dm, sh);
        dm.arrive();
        solve_col<NX, NY, 2, F_B>(P, dm, sh, mb);
        dm.arrive();
      }
      if (dm.failed()) return;
    }
    if (threadIdx.x == 0) PAT_AGENT_ADD((uint32_t*)P.bad + kBadOpen, solve_share(dm.rank, dm.n));
  }
}

// kernels of one column length NY and direction, by row length
template <int NY, int DIR>
hipError_t launch_solve_nd(int nx, int lossy, const SolveArgs& a, hipStream_t st) {
#define PAT_SOLVE(N, LS)                                                                               \
  hipLaunchKernelGGL((k_solve<N, NY, DIR, LS>),                                                        \
                     dim3((solve_whole(N, NY) ? 1 : kSolveXcds) * a.members * a.domains),              \
                     dim3(SolveGeo<N, NY>::NTH), 0, st, a)
#define PAT_SOLVE_NX(N)         \
  case N:                       \
    if (lossy) PAT_SOLVE(N, 1); \
    else PAT_SOLVE(N, 0);       \
    break;
  switch (nx) {
    PAT_SOLVE_NX(32)
    PAT_SOLVE_NX(64)
    PAT_SOLVE_NX(128)
    PAT_SOLVE_NX(256)
    PAT_SOLVE_NX(512)
    default: return hipErrorInvalidValue;
  }
#undef PAT_SOLVE_NX
#undef PAT_SOLVE
  return hipGetLastError();
}

}  // namespace pat
