// Row-tile sparse product W = opscale * (Q X) * diag(xmult) over a matrix's
// row groups (Alg 1's operator application): the same W, fused inner products
// and early subtraction as the row-group product of k_rowgroup.hip, with the
// probe rows that a tile of kTileGroups groups references gathered once into
// LDS.
//
// What bounds the row-group product is its gathers: each group of 4 rows
// fetches its union columns' probe rows from the L2 by itself (covariance of
// 5e5 scattered points, 48.8 entries per row, 64 FP32 probes: 10.4e6 rows of
// 256 bytes per launch, 9.8 TB/s of L2 -> L1 reads in 0.28 ms), although 16
// neighbouring groups reference mostly the same rows.  Here a 256-thread block
// takes a tile (64 rows) and a panel of the probe columns (16 lanes of CPL
// columns, 128 bytes per probe row), moves the tile's union (about 300 rows
// there, against 1330 gathers of its groups) straight into LDS with 16-byte
// loads and serves every group from LDS: a group is 16 lanes, each with CPL
// columns of the group's 4 rows, so an LDS read feeds 4 rows.  The entries (a
// 16-bit index into the tile's union and 4 values) are loaded one per lane and
// handed round the 16 lanes by the DPP row broadcast inside the multiply-add,
// so no LDS access or shuffle is spent on them.  A tile's union, entries and
// window vector are read while the tile before it is finished, its sizes one
// tile further ahead.
//
// Measured against the row-group product (mean per launch, us): the
// covariance above 279 -> 209, a grid covariance of 78 entries per row (n =
// 1.08e6, 30 FP32 probes) 355 -> 243, 23 000 scattered points with 30 FP64
// probes 69 -> 21.  What bounds it now is vector issue: 76e6 wave instructions
// on the first, 65% of them the multiply-adds (41% of those on the zeros of
// rows that lack a column), 0.7 of the cycles at 4.6 clocks each, at 3 blocks of
// 4 waves per CU (LDS); on the last, with one tile per block, the chain of
// latencies (vector instructions in a quarter of the cycles).  Tried and not
// kept: 64 FP32 columns per panel (two blocks per CU: 294 against 215 us), one
// round of entries in flight ahead (274: a round of memory latency each 16
// entries).
//
// A row's sum sees its nonzero terms in CSR order (a zero value adds an exact
// zero): W is the CSR product's W.  Only the grouping of the FP64 partial sums
// differs.
#include <algorithm>
#include <climits>
#include <map>
#include <mutex>
#include <type_traits>

#include "ld_kernels.h"

namespace ld {

constexpr int kTileLanes = 16;                              // lanes per group: a DPP row
static_assert(kTileGroups * kTileLanes == kThreads, "one 16-lane row per group");
static_assert(kRowGroup == 4, "four rows per group");
constexpr int kTileSort = 8192;  // most union columns of a tile's groups together (the build)

struct TileDesc {
  int64_t n;
  const int* gp;
  const void* val;       // kRowGroup values per union column, in the element type
  const uint16_t* lidx;  // per union column of a group: its index in the tile's union
  const uint16_t* self;  // per group: index of its first row in the tile's union
  const int* tcol;       // [tile][ust] union columns of the tile, then its last one
  const int* tcnt;       // [tile]
  TileShape shape;
  int ust, umax;
  const void* X;
  void* W;
  const double* xmult;
  double opscale;
  const void* fx[2];
  const double* fmult[2];
  double* part;
  int ld, voff, il, npan;
  const void* sx;
  const double* smult;
  const double* sd;
};

// acc += (lane J of the 16-lane row's a) * x; every lane of the row is active.
// The no-op covers the wait states between a vector write of the broadcast
// operand and its DPP read, which the compiler does not see inside the block;
// volatile keeps the block out of the divergent code around it.  The sums are
// early-clobber: the first ones are written before the last operands are read.
template <int J>
__device__ inline void fmac_row(float (&acc)[4][1], const float (&a)[4], const float (&x)[1]) {
  asm volatile("s_nop 1\n\t"
      "v_fmac_f32_dpp %0, %4, %8 row_newbcast:%9 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %1, %5, %8 row_newbcast:%9 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %2, %6, %8 row_newbcast:%9 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %3, %7, %8 row_newbcast:%9 row_mask:0xf bank_mask:0xf"
      : "+&v"(acc[0][0]), "+&v"(acc[1][0]), "+&v"(acc[2][0]), "+&v"(acc[3][0])
      : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(x[0]), "n"(J));
}
template <int J>
__device__ inline void fmac_row(float (&acc)[4][2], const float (&a)[4], const float (&x)[2]) {
  asm volatile("s_nop 1\n\t"
      "v_fmac_f32_dpp %0, %8, %12 row_newbcast:%14 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %1, %8, %13 row_newbcast:%14 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %2, %9, %12 row_newbcast:%14 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %3, %9, %13 row_newbcast:%14 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %4, %10, %12 row_newbcast:%14 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %5, %10, %13 row_newbcast:%14 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %6, %11, %12 row_newbcast:%14 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %7, %11, %13 row_newbcast:%14 row_mask:0xf bank_mask:0xf"
      : "+&v"(acc[0][0]), "+&v"(acc[0][1]), "+&v"(acc[1][0]), "+&v"(acc[1][1]), "+&v"(acc[2][0]),
        "+&v"(acc[2][1]), "+&v"(acc[3][0]), "+&v"(acc[3][1])
      : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(x[0]), "v"(x[1]), "n"(J));
}
template <int J>
__device__ inline void fmac_row(double (&acc)[4][1], const double (&a)[4], const double (&x)[1]) {
  asm volatile("s_nop 1\n\t"
      "v_fmac_f64_dpp %0, %4, %8 row_newbcast:%9 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %1, %5, %8 row_newbcast:%9 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %2, %6, %8 row_newbcast:%9 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %3, %7, %8 row_newbcast:%9 row_mask:0xf bank_mask:0xf"
      : "+&v"(acc[0][0]), "+&v"(acc[1][0]), "+&v"(acc[2][0]), "+&v"(acc[3][0])
      : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(x[0]), "n"(J));
}
template <int J>
__device__ inline void fmac_row(double (&acc)[4][2], const double (&a)[4], const double (&x)[2]) {
  asm volatile("s_nop 1\n\t"
      "v_fmac_f64_dpp %0, %8, %12 row_newbcast:%14 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %1, %8, %13 row_newbcast:%14 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %2, %9, %12 row_newbcast:%14 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %3, %9, %13 row_newbcast:%14 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %4, %10, %12 row_newbcast:%14 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %5, %10, %13 row_newbcast:%14 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %6, %11, %12 row_newbcast:%14 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %7, %11, %13 row_newbcast:%14 row_mask:0xf bank_mask:0xf"
      : "+&v"(acc[0][0]), "+&v"(acc[0][1]), "+&v"(acc[1][0]), "+&v"(acc[1][1]), "+&v"(acc[2][0]),
        "+&v"(acc[2][1]), "+&v"(acc[3][0]), "+&v"(acc[3][1])
      : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(x[0]), "v"(x[1]), "n"(J));
}
// lane J of the 16-lane row
template <int J>
__device__ inline int row_lane(int v) {
  return __builtin_amdgcn_update_dpp(0, v, 0x150 + J, 0xf, 0xf, true);
}

template <int N, typename F>
__device__ inline void unroll_n(F f) {
  if constexpr (N > 0) {
    unroll_n<N - 1>(f);
    f(std::integral_constant<int, N - 1>{});
  }
}

// CPL contiguous elements
template <typename T, int CPL>
struct Cols {
  T v[CPL];
  __device__ inline void load(const T* p) {
    if constexpr (CPL == 1) {
      v[0] = p[0];
    } else {
      typedef T tv __attribute__((ext_vector_type(CPL)));
      const tv t = *reinterpret_cast<const tv*>(p);
#pragma unroll
      for (int e = 0; e < CPL; ++e) v[e] = t[e];
    }
  }
  __device__ inline void load_nt(const T* p) {
    typedef T tv __attribute__((ext_vector_type(CPL)));
    const tv t = __builtin_nontemporal_load(reinterpret_cast<const tv*>(p));
#pragma unroll
    for (int e = 0; e < CPL; ++e) v[e] = t[e];
  }
  __device__ inline void store_nt(T* p) const {
    typedef T tv __attribute__((ext_vector_type(CPL)));
    tv t;
#pragma unroll
    for (int e = 0; e < CPL; ++e) t[e] = v[e];
    __builtin_nontemporal_store(t, reinterpret_cast<tv*>(p));
  }
};

// One entry of a group per lane, as loaded: its 4 values and its column's
// index in the tile's union.  Lanes past the group's last entry hold entries
// of a later group (the arrays end in kTilePad unused entries), which the
// product replaces by zero values on the group's own first row.
template <typename VT>
struct TileEntry {
  VT t[4];
  int idx;
  __device__ inline void load(const VT* vals, const uint16_t* lidx) {
    idx = lidx[0];
    if constexpr (sizeof(VT) == 4) {
      const float4 q = *reinterpret_cast<const float4*>(vals);
      t[0] = q.x; t[1] = q.y; t[2] = q.z; t[3] = q.w;
    } else {
      const double2 p = reinterpret_cast<const double2*>(vals)[0];
      const double2 q = reinterpret_cast<const double2*>(vals)[1];
      t[0] = p.x; t[1] = p.y; t[2] = q.x; t[3] = q.y;
    }
  }
};

// 16 bytes per lane straight into LDS: lane i of the wave writes lds + 16 i.
__device__ inline void load_lds16(const void* src, void* lds) {
  __builtin_amdgcn_global_load_lds(
      (const __attribute__((address_space(1))) void*)src,
      (__attribute__((address_space(3))) void*)lds, 16, 0, 0);
}

// Waits for the wave's vector memory loads (vmcnt 0, the other counters
// untouched); the compiler's own wait placement sees it.
__device__ inline void wait_vm() { __builtin_amdgcn_s_waitcnt(0x0f70); }

template <typename VT, typename T, int CPL, int NF>
__device__ inline void tile_body(const TileDesc& q, int bk0, int nb0) {
  using A = typename std::conditional<sizeof(VT) == 8 || sizeof(T) == 8, double, float>::type;
  constexpr int PC = kTileLanes * CPL;           // columns of a panel
  constexpr int PB = PC * (int)sizeof(T);        // bytes of a probe row in the panel
  constexpr int CH = PB / 16;                    // 16-byte chunks of it
  constexpr int VEC = 16 / (int)sizeof(T);
  constexpr int RPW = 64 / CH, NW = kThreads / 64;  // union rows a wave loads at a time
  constexpr int EB = sizeof(VT) == 8 && sizeof(T) == 4 ? 4 : 6;  // rounds of 16 entries in flight
  constexpr int TB = 10;  // loads in flight per lane: 320 union rows of 128 bytes per round
  constexpr int G = kRowGroup;
  extern __shared__ __align__(16) char xs_raw[];
  T* xt = reinterpret_cast<T*>(xs_raw);
  const int nbk = nb0 / q.npan;
  const int pan = bk0 / nbk, bk = bk0 - pan * nbk;
  const int tid = threadIdx.x, grp = tid / kTileLanes, l = tid % kTileLanes;
  const int ld = q.ld, pc0 = pan * PC;
  const int col = pc0 + l * CPL;                 // this lane's first column
  const bool on = col < ld;                      // ld is a multiple of 4: all CPL or none
  const int wv = __builtin_amdgcn_readfirstlane(tid / 64), wl = tid % 64, ch = wl % CH;  // load phase
  const bool chon = pc0 + ch * VEC < ld;
  A sc[CPL];
  double scf[CPL];
#pragma unroll
  for (int e = 0; e < CPL; ++e) {
    sc[e] = on ? A(q.opscale * (q.xmult ? q.xmult[col + e] : 1.0)) : A(0);
    scf[e] = (on && q.sx) ? q.sd[col + e] * (q.smult ? q.smult[col + e] : 1.0) : 0.0;
  }
  double dacc[NF > 0 ? NF : 1][CPL];
#pragma unroll
  for (int v = 0; v < (NF > 0 ? NF : 1); ++v)
#pragma unroll
    for (int e = 0; e < CPL; ++e) dacc[v][e] = 0.0;
  const int64_t ng = (q.n + G - 1) / G;
  const int ntile = (int)q.shape.ntile, nn = (int)q.n;  // n < 2^31
  const VT* vals = static_cast<const VT*>(q.val);
  const T* X = static_cast<const T*>(q.X);
  const T* sx = static_cast<const T*>(q.sx);
  T* W = static_cast<T*>(q.W);
  // a zero the compiler does not see through: the tile's size is loaded per
  // lane and made uniform only where it is used, not waited for in meta
  int vzero;
  asm volatile("v_mov_b32 %0, 0" : "=v"(vzero));
  // a tile's size, its group of this lane and the first TB union columns this
  // lane loads: read one tile ahead, so that a tile waits for one round of
  // memory (its union, entries and window vector together)
  struct Meta {
    int nu, ub, ue, sl;
    int g;
    int tc[TB];
  };
  auto meta = [&](int j) -> Meta {
    Meta m;
    // past the last tile: the last one again, without groups
    const int t0 = q.il ? j * nbk + bk : chunk_of(j, bk, nbk), tile = min(t0, ntile - 1);
    m.g = t0 < ntile ? (int)tile_group(q.shape, ng, tile, grp) : -1;
    m.nu = q.tcnt[tile + vzero];
    // ust is a multiple of the RPW * NW rows a load takes
    const int* tc = q.tcol + (size_t)tile * q.ust;
#pragma unroll
    for (int u = 0; u < TB; ++u)
      m.tc[u] = (tc + min(u * NW * RPW, q.ust - NW * RPW))[wv * RPW + wl / CH];
    const int g = max(m.g, 0);
    m.ub = q.gp[g];
    m.ue = q.gp[g + 1];
    m.sl = q.self[g];
    return m;
  };
  // the tile's union into LDS: each wave takes RPW rows at a time, a row's
  // CH 16-byte chunks on consecutive lanes (the order they have in LDS); the
  // last ones of a tile may be repeats of its last column
  auto gather = [&](const Meta& m, int j) {
    if (!chon) return;
    const int nu = __builtin_amdgcn_readfirstlane(m.nu);
    const T* xp = X + pc0 + ch * VEC;
#pragma unroll
    for (int u = 0; u < TB; ++u) {
      const int r0 = (u * NW + wv) * RPW;
      if (r0 < nu) load_lds16(xp + (size_t)m.tc[u] * ld, xs_raw + (size_t)r0 * PB);
    }
    if (nu > TB * NW * RPW) {
      // (past the last tile the last one again, as in meta)
      const int tile = min(q.il ? j * nbk + bk : chunk_of(j, bk, nbk), ntile - 1);
      const int* tc = q.tcol + (size_t)tile * q.ust;
      for (int rb = TB * NW * RPW; rb < nu; rb += TB * NW * RPW) {
        int c[TB];
#pragma unroll
        for (int u = 0; u < TB; ++u)
          if (rb + u * NW * RPW < q.ust) c[u] = tc[rb + (u * NW + wv) * RPW + wl / CH];
        wait_vm();
#pragma unroll
        for (int u = 0; u < TB; ++u) {
          const int r0 = rb + (u * NW + wv) * RPW;
          if (r0 < nu) load_lds16(xp + (size_t)c[u] * ld, xs_raw + (size_t)r0 * PB);
        }
      }
    }
  };
  // the next EB rounds of the group's entries (all of them on a covariance of
  // scattered points, most often) and its rows of the window vector, read
  // with the union
  TileEntry<VT> ent[EB];
  auto entries = [&](auto& en, int k, int rounds) {
    constexpr int N = sizeof(en) / sizeof(en[0]);
    const VT* v = vals + (size_t)4 * (k + l);
    const uint16_t* x = q.lidx + (k + l);
#pragma unroll
    for (int b = 0; b < N; ++b)
      if (b < rounds) en[b].load(v + b * 4 * kTileLanes, x + b * kTileLanes);
  };
  // entries of the wave's longest group, made uniform
  auto longest = [&](const Meta& m) -> int {
    const int c = m.g >= 0 ? m.ue - m.ub : 0;
    return max(max(__builtin_amdgcn_readlane(c, 0), __builtin_amdgcn_readlane(c, 16)),
               max(__builtin_amdgcn_readlane(c, 32), __builtin_amdgcn_readlane(c, 48)));
  };
  Cols<T, CPL> xn[G];
  auto window = [&](int g) {
    if (sx && g >= 0 && on) {
#pragma unroll
      for (int r = 0; r < G; ++r)
        xn[r].load_nt(sx + (size_t)min(g * G + r, nn - 1) * ld + col);  // read once per step
    }
  };
  Meta nx = meta(0);
  wait_vm();
  gather(nx, 0);
  int cnt_n = longest(nx);
  entries(ent, nx.ub, (cnt_n + kTileLanes - 1) / kTileLanes);
  window(nx.g);
  Meta cur = nx;
  nx = meta(1);
  for (int j = 0; j * nbk < ntile; ++j) {
    const int g = cur.g, sl = cur.sl, ub = cur.ub, ue = g >= 0 ? cur.ue : ub, cnt = cnt_n;
    wait_vm();  // this wave's rows are in LDS
    __syncthreads();
    A acc[G][CPL];
#pragma unroll
    for (int r = 0; r < G; ++r)
#pragma unroll
      for (int e = 0; e < CPL; ++e) acc[r][e] = A(0);
    const int lo = l * CPL * (int)sizeof(T);
    // one round: lane J of the row holds entry base + J; left: entries of the
    // wave's longest group from base on
    auto round = [&](const TileEntry<VT>& en, int base, int left) {
      const bool mine = base + l < ue;
      const int off = (mine ? en.idx : sl) * PB;
      A a[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) a[r] = mine ? A(en.t[r]) : A(0);
      // N entries from the round's entry H on, their LDS reads in flight
      auto part = [&](auto h0, auto n0) {
        constexpr int H = decltype(h0)::value, N = decltype(n0)::value;
        Cols<T, CPL> x[N];
        unroll_n<N>([&](auto jj) {
          constexpr int J = decltype(jj)::value;
          x[J].load(reinterpret_cast<const T*>(xs_raw + row_lane<H + J>(off) + lo));
        });
        unroll_n<N>([&](auto jj) {
          constexpr int J = decltype(jj)::value;
          A xa[CPL];
#pragma unroll
          for (int e = 0; e < CPL; ++e) xa[e] = A(x[J].v[e]);
          fmac_row<H + J>(acc, a, xa);
        });
      };
      std::integral_constant<int, 0> i0;
      std::integral_constant<int, 8> i8;
      part(i0, i8);
      if (left > 8) part(i8, i8);
    };
#pragma unroll
    for (int b = 0; b < EB; ++b)
      if (b * kTileLanes < cnt) round(ent[b], ub + b * kTileLanes, cnt - b * kTileLanes);
    for (int b0 = EB * kTileLanes; b0 < cnt; b0 += 2 * kTileLanes) {
      TileEntry<VT> more[2];
      entries(more, ub + b0, (cnt - b0 + kTileLanes - 1) / kTileLanes);
      wait_vm();
      round(more[0], ub + b0, cnt - b0);
      if (b0 + kTileLanes < cnt) round(more[1], ub + b0 + kTileLanes, cnt - b0 - kTileLanes);
    }
    // the rows' own entries of the tile (a group's rows are consecutive in
    // the union): the newest window vector is X itself
    Cols<T, CPL> xd[NF > 0 ? G : 1], xs[G];
    if constexpr (NF > 0) {
#pragma unroll
      for (int r = 0; r < G; ++r)
        xd[r].load(xt + min(sl + r, q.umax - 1) * PC + l * CPL);
    }
#pragma unroll
    for (int r = 0; r < G; ++r) xs[r] = xn[r];
    __syncthreads();
    // the next tile's reads, in flight during this one's epilogue
    cur = nx;
    if ((j + 1) * nbk < ntile) gather(cur, j + 1);
    cnt_n = longest(cur);
    entries(ent, cur.ub, (cnt_n + kTileLanes - 1) / kTileLanes);
    window(cur.g);
    nx = meta(j + 2);
    if (g >= 0 && on) {
      size_t at = (size_t)(g * G) * ld + col;
#pragma unroll
      for (int r = 0; r < G; ++r, at += ld) {
        if (g * G + r >= nn) break;
        Cols<T, CPL> out;
        if (sx) {
#pragma unroll
          for (int e = 0; e < CPL; ++e)
            out.v[e] = T(fma(-scf[e], double(xs[r].v[e]), double(acc[r][e] * sc[e])));
        } else {
#pragma unroll
          for (int e = 0; e < CPL; ++e) out.v[e] = T(acc[r][e] * sc[e]);
        }
        out.store_nt(W + at);
        if constexpr (NF > 0) {
#pragma unroll
          for (int v = 0; v < NF; ++v) {
            Cols<T, CPL> x = xd[r];
            if (v < NF - 1) x.load(static_cast<const T*>(q.fx[v]) + at);
#pragma unroll
            for (int e = 0; e < CPL; ++e)
              dacc[v][e] = fma(double(x.v[e]), double(out.v[e]), dacc[v][e]);
          }
        }
      }
    }
  }
  if constexpr (NF > 0) {
    // the block's column sums: groups in order
    double* red = reinterpret_cast<double*>(xs_raw);
#pragma unroll
    for (int v = 0; v < NF; ++v) {
#pragma unroll
      for (int e = 0; e < CPL; ++e) red[grp * PC + l * CPL + e] = dacc[v][e];
      __syncthreads();
      for (int i = tid; i < PC; i += kThreads) {
        double s = 0.0;
        for (int k = 0; k < kTileGroups; ++k) s += red[k * PC + i];
        const int c = pc0 + i;
        if (c < ld)
          q.part[((size_t)(q.voff + v) * ld + c) * nbk + bk] =
              s * (q.fmult[v] ? q.fmult[v][c] : 1.0);
      }
      __syncthreads();
    }
  }
}

template <typename VT, typename T, int CPL, int NF>
__global__ __launch_bounds__(kThreads, 3) void k_spmm_tile(BatchArgs<TileDesc> bt) {
  int r = 0;
  while (r + 1 < bt.count && (int)blockIdx.x >= bt.off[r + 1]) ++r;
  tile_body<VT, T, CPL, NF>(bt.d[r], (int)blockIdx.x - bt.off[r], bt.off[r + 1] - bt.off[r]);
}

// Columns per lane: one for FP64 blocks; two for FP32 blocks (a probe row of
// a panel is then 128 bytes, one cache line), one where the block has at most
// 16 columns.
static int tile_cpl(int ld, int xbytes) { return xbytes == 4 && ld > kTileLanes ? 2 : 1; }

static size_t tile_lds(int rows, int ld, int xbytes) {
  const size_t pb = (size_t)kTileLanes * tile_cpl(ld, xbytes) * xbytes;
  const size_t red = (size_t)kThreads * 2 * sizeof(double);
  // the load phase writes whole waves' rows: up to 1024 bytes past the union
  return std::max(red, (size_t)rows * pb + 1024);
}

// LDS classes by the blocks a CU holds (4, 3, 2 or 1 of its 128 pieces of 1280
// bytes): requests of one launch share a class, so the launch's LDS (the
// class's bound) and a request's grid do not depend on what it is batched with.
constexpr size_t kTileLdsClass[] = {32 * 1280, 42 * 1280, 64 * 1280, 128 * 1280};
static int tile_class(int rows, int ld, int xbytes) {
  const size_t need = tile_lds(rows, ld, xbytes);
  for (int c = 0; c < 4; ++c)
    if (need <= kTileLdsClass[c]) return c;
  return -1;
}
static int tile_class(const SpmmItem& it) {
  return tile_class(it.rg.tile.umax, it.g.ld, it.g.xbytes);
}
int tile_blocks(int rows, int ld, int xbytes) {
  const int c = tile_class(rows, ld, xbytes);
  return c < 0 ? 0 : 4 - c;
}
int tile_panels(int ld, int xbytes) {
  const int pc = kTileLanes * tile_cpl(ld, xbytes);
  return (ld + pc - 1) / pc;
}

int spmm_tile_key(const SpmmItem& it) {
  if (it.g.rg != 2 || !it.rg.tile.tcol || it.g.ld < kTileMinCols) return 0;
  const int c = tile_class(it);
  return c < 0 ? 0 : 1 + c + 8 * tile_cpl(it.g.ld, it.g.xbytes);
}

static int tile_resident(const void* fn, size_t lds) {
  static std::mutex mu;
  static std::map<std::pair<const void*, size_t>, int> cache;
  std::lock_guard<std::mutex> lk(mu);
  auto it = cache.find({fn, lds});
  if (it != cache.end()) return it->second;
  int dev = 0, cus = 0, per_cu = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
    cus = 256;
  (void)hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, kThreads, lds) != hipSuccess ||
      per_cu < 1)
    per_cu = 1;
  const int r = std::min(kMaxBlocks, std::max(1, per_cu * cus));
  cache[{fn, lds}] = r;
  return r;
}

template <typename VT, typename T, int CPL, int NF>
static hipError_t tile_launch(hipStream_t st, SpmmItem* items, const int* idx, int cnt) {
  auto fn = k_spmm_tile<VT, T, CPL, NF>;
  const size_t lds = kTileLdsClass[tile_class(items[idx[0]])];
  const int resident = tile_resident((const void*)fn, lds);
  BatchArgs<TileDesc> bt{};
  bt.count = cnt;
  int off = 0;
  for (int q = 0; q < cnt; ++q) {
    SpmmItem& it = items[idx[q]];
    TileDesc& d = bt.d[q];
    const RowTiles& rt = it.rg.tile;
    d.npan = tile_panels(it.g.ld, it.g.xbytes);
    // one resident wave of blocks over all panels, a multiple of 8 per panel
    // from 8 up (see chunk_of)
    int nb = (int)std::min<int64_t>(rt.shape.ntile, std::max(1, resident / d.npan));
    if (nb >= 8) nb &= ~7;
    it.nblk = nb;
    d.n = it.g.n;
    d.gp = it.rg.gp;
    d.val = sizeof(VT) == 4 ? static_cast<const void*>(it.rg.val)
                            : static_cast<const void*>(it.rg.val64);
    d.lidx = rt.lidx;
    d.self = rt.self;
    d.tcol = rt.tcol;
    d.tcnt = rt.tcnt;
    d.shape = rt.shape;
    d.ust = rt.ust;
    d.umax = rt.umax;
    d.X = it.X;
    d.W = it.W;
    d.xmult = it.xmult;
    d.opscale = it.opscale;
    for (int v = 0; v < 2; ++v) {
      d.fx[v] = v < it.nf ? it.fused.x[v] : nullptr;
      d.fmult[v] = v < it.nf ? it.fused.mult[v] : nullptr;
    }
    d.part = it.part;
    d.ld = it.g.ld;
    d.voff = it.voff;
    d.il = it.g.xil;
    d.sx = it.sx;
    d.smult = it.smult;
    d.sd = it.sd;
    bt.off[q] = off;
    off += nb * d.npan;
  }
  bt.off[cnt] = off;
  hipLaunchKernelGGL(fn, dim3(off), dim3(kThreads), lds, st, bt);
  return hipGetLastError();
}

hipError_t launch_spmm_tile_group(hipStream_t st, SpmmItem* items, const int* idx, int cnt) {
  if (!items || !idx || cnt < 1 || cnt > kMaxBatch) return hipErrorInvalidValue;
  const SpmmItem& it = items[idx[0]];
  const int key = spmm_tile_key(it);
  for (int q = 0; q < cnt; ++q) {
    const SpmmItem& x = items[idx[q]];
    const bool ok = (x.g.xbytes == 4 && (x.vt == VT_F32 || x.vt == VT_F64)) ||
                    (x.g.xbytes == 8 && x.vt == VT_F64);
    const void* val = x.vt == VT_F32 ? static_cast<const void*>(x.rg.val)
                                     : static_cast<const void*>(x.rg.val64);
    const RowTiles& t = x.rg.tile;
    if (key == 0 || spmm_tile_key(x) != key || !ok || x.g.xbytes != it.g.xbytes ||
        x.vt != it.vt || x.nf != it.nf || !x.rg.gp || !val || !t.lidx || !t.self || !t.tcnt ||
        t.ust < 1 || t.ust % kTileLoadRows != 0 || t.umax < 1 || t.umax > t.ust || t.shape.ntile < 1 || reinterpret_cast<uintptr_t>(val) % 16 != 0 ||
        reinterpret_cast<uintptr_t>(x.X) % 16 != 0 || reinterpret_cast<uintptr_t>(x.W) % 16 != 0 ||
        x.g.ld * x.g.xbytes % 16 != 0)
      return hipErrorInvalidValue;
  }
  const int nf = it.nf;
  auto by_nf = [&](auto v, auto t, auto c) -> hipError_t {
    using VT = decltype(v);
    using T = decltype(t);
    constexpr int CC = decltype(c)::value;
    if (nf == 0) return tile_launch<VT, T, CC, 0>(st, items, idx, cnt);
    if (nf == 1) return tile_launch<VT, T, CC, 1>(st, items, idx, cnt);
    return tile_launch<VT, T, CC, 2>(st, items, idx, cnt);
  };
  std::integral_constant<int, 1> one;
  std::integral_constant<int, 2> two;
  if (it.g.xbytes == 8) return by_nf(double{}, double{}, one);
  const bool wide = tile_cpl(it.g.ld, 4) == 2;
  if (it.vt == VT_F64) return wide ? by_nf(double{}, float{}, two) : by_nf(double{}, float{}, one);
  return wide ? by_nf(float{}, float{}, two) : by_nf(float{}, float{}, one);
}

// ---------------------------------------------------------------------------
// Tiles of a matrix's row groups on the device, one block per tile: the
// groups' sorted union columns concatenated in LDS, sorted (bitonic) and made
// unique.  Pass 1 counts (tcnt[tile]; -1 when the tile's groups hold more
// than kTileSort columns together); pass 2, with ust at least every count,
// writes the unions, each group entry's index in its tile's union and the
// index of each group's first row.
// ---------------------------------------------------------------------------
template <bool FILL>
__global__ __launch_bounds__(kThreads) void k_tile_build(int64_t n, TileShape shape,
                                                         const int* __restrict__ gp,
                                                         const int* __restrict__ col, int ust,
                                                         int* __restrict__ tcnt,
                                                         int* __restrict__ tcol,
                                                         uint16_t* __restrict__ lidx,
                                                         uint16_t* __restrict__ self) {
  __shared__ int key[kTileSort];
  __shared__ int uq[FILL ? kTileMaxUnion : 1];
  __shared__ int scan[kThreads];
  __shared__ int gb[kTileGroups], gn[kTileGroups + 1];
  __shared__ int64_t gid[kTileGroups];
  const int64_t tile = blockIdx.x, ng = (n + kRowGroup - 1) / kRowGroup;
  const int t = threadIdx.x;
  if (t < kTileGroups) {
    const int64_t g = tile_group(shape, ng, tile, t);
    gid[t] = g;
    gb[t] = g >= 0 ? gp[g] : 0;
    scan[t] = g >= 0 ? gp[g + 1] - gb[t] : 0;
  }
  __syncthreads();
  if (t == 0) {
    int64_t s = 0;
    for (int k = 0; k < kTileGroups; ++k) {
      gn[k] = (int)min(s, (int64_t)INT_MAX);
      s += scan[k];
    }
    gn[kTileGroups] = (int)min(s, (int64_t)INT_MAX);
  }
  __syncthreads();
  const int total = gn[kTileGroups];
  if (total > kTileSort) {
    if (!FILL && t == 0) tcnt[tile] = -1;
    return;
  }
  int np = 1;
  while (np < total) np <<= 1;
  for (int i = t; i < np; i += kThreads) key[i] = INT_MAX;
  __syncthreads();
  for (int k = 0; k < kTileGroups; ++k)
    for (int i = t; i < gn[k + 1] - gn[k]; i += kThreads) key[gn[k] + i] = col[gb[k] + i];
  __syncthreads();
  for (int len = 2; len <= np; len <<= 1)
    for (int d = len >> 1; d > 0; d >>= 1) {
      for (int i = t; i < np / 2; i += kThreads) {
        const int a = 2 * i - (i & (d - 1)), b = a + d;
        const int x = key[a], y = key[b];
        if ((x > y) == ((a & len) == 0)) {
          key[a] = y;
          key[b] = x;
        }
      }
      __syncthreads();
    }
  // unique columns: each thread counts a contiguous part, then a scan
  const int per = (total + kThreads - 1) / kThreads, i0 = min(total, t * per),
            i1 = min(total, i0 + per);
  int c = 0;
  for (int i = i0; i < i1; ++i) c += (i == 0 || key[i] != key[i - 1]) ? 1 : 0;
  scan[t] = c;
  __syncthreads();
  for (int d = 1; d < kThreads; d <<= 1) {
    const int v = t >= d ? scan[t - d] : 0;
    __syncthreads();
    scan[t] += v;
    __syncthreads();
  }
  const int nu = scan[kThreads - 1];
  if constexpr (!FILL) {
    if (t == 0) tcnt[tile] = nu;
  } else {
    if (nu > kTileMaxUnion || nu > ust) return;  // the host sized ust from pass 1's counts
    int at = scan[t] - c;
    for (int i = i0; i < i1; ++i)
      if (i == 0 || key[i] != key[i - 1]) {
        uq[at] = key[i];
        tcol[(size_t)tile * ust + at] = key[i];
        ++at;
      }
    // the rest of the tile's list repeats its last column (the load phase
    // reads whole waves' rows)
    for (int i = nu + t; i < ust; i += kThreads) tcol[(size_t)tile * ust + i] = key[total - 1];
    __syncthreads();
    auto find = [&](int cc) -> int {
      int lo = 0, hi = nu - 1;
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (uq[mid] < cc) lo = mid + 1; else hi = mid;
      }
      return lo;
    };
    for (int k = 0; k < kTileGroups; ++k)
      for (int i = t; i < gn[k + 1] - gn[k]; i += kThreads)
        lidx[gb[k] + i] = (uint16_t)find(col[gb[k] + i]);
    if (t < kTileGroups && gid[t] >= 0) self[gid[t]] = (uint16_t)find((int)(gid[t] * kRowGroup));
  }
}

hipError_t launch_tile_count(hipStream_t st, int64_t n, const TileShape& s, const int* gp,
                             const int* col, int* tcnt) {
  if (n < 1 || s.ntile < 1 || s.ntile > INT_MAX || !gp || !col || !tcnt)
    return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_tile_build<false>, dim3((unsigned)s.ntile), dim3(kThreads), 0, st, n, s, gp,
                     col, 0, tcnt, nullptr, nullptr, nullptr);
  return hipGetLastError();
}

hipError_t launch_tile_fill(hipStream_t st, int64_t n, const TileShape& s, const int* gp,
                            const int* col, int ust, int* tcol, uint16_t* lidx, uint16_t* self) {
  if (n < 1 || s.ntile < 1 || s.ntile > INT_MAX || !gp || !col || ust < 1 ||
      !tcol || !lidx || !self ||
      ust % kTileLoadRows != 0)
    return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_tile_build<true>, dim3((unsigned)s.ntile), dim3(kThreads), 0, st, n, s, gp,
                     col, ust, nullptr, tcol, lidx, self);
  return hipGetLastError();
}

}  // namespace ld
