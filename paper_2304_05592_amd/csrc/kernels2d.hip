// 2D time-step kernels for gfx950: forward, adjoint with imaging, Born.
//
// One workgroup (4 x wave64) updates one tile of TZ rows x 64 columns of one shot.  The
// tile of the field at the previous time level plus a 4-cell halo is staged in LDS
// ((TZ + 8) x 72 floats); each wave updates TZ/4 consecutive rows, one column per lane, so
// every global access is a 256-byte coalesced row segment.  Damping is evaluated from the
// grid indices (no array), the source is injected by the threads owning its nodes, the
// receivers whose base node lies in the tile are sampled from LDS, and the adjoint's
// receiver injection is gathered per touched point into LDS (no atomics, fixed order).
//
// Discretisation (row k of A u = s, see awe.h), written in increment form:
//   incr = coef * (L_h u^{k-1} + s^{k-1} - (eta/dt) (u^{k-1} - u^{k-2})),
//   u^k  = 2 u^{k-1} - u^{k-2} + incr,      coef = dt^2 / (m + eta dt / 2),
// with the Laplacian summed as sum_r c_r ((u_{+r} - u) + (u_{-r} - u)) so that a smooth
// field loses few digits to cancellation.  incr equals u^k - 2u^{k-1} + u^{k-2} exactly
// before rounding, which gives the imaging condition and the Born source without the
// cancellation of a second time difference.
//
// Fields are read and written through buffer resources (bufio.h): a lane's byte offset within
// a row is fixed (kOOB for a column outside the grid: its loads read 0, its stores are
// dropped, and it costs no memory traffic) and the row's offset is wave-uniform, so rows cost
// no vector instructions for addresses, clamps or masks.  Rows outside the grid, and levels
// that are zero by definition, are read through a resource of size 0.
#include "awe_internal.h"
#include "bufio.h"
#include "codec.h"

namespace awe {

namespace {

__device__ __forceinline__ int xcd_tile(int bid, int n) {
  // Workgroups are dispatched round-robin over the 8 XCDs; give each XCD a contiguous
  // range of tiles so that neighbouring tiles share its L2.
  const int q = n >> 3, r = n & 7, x = bid & 7;
  return x * q + min(x, r) + (bid >> 3);
}

__device__ __forceinline__ int border_dist(int i, int n, int nbl) {
  return max(max(nbl - i, i - (n - 1 - nbl)), 0);
}

template <int TZ>
struct T2 {
  static constexpr int W = kTX + 2 * kHalo;  // 72
  static constexpr int H = TZ + 2 * kHalo;
  static constexpr int NW = TZ >= 32 ? 8 : 4;  // waves per workgroup
  static constexpr int NT = 64 * NW;           // threads per workgroup
  static constexpr int RPT = TZ / NW;          // rows per thread
  static_assert(TZ % NW == 0, "tile rows must split evenly over the waves");
};

// Plane offsets of this thread's side-halo cells of a tile staged with an HW-cell halo: cell e
// of the 2 HW columns left and right of the 64-column body of each of the H rows, starting at
// row z0 - HW (kOOB outside the grid or past the last cell).
template <int NT, int H, int HW>
struct SideHalo {
  static constexpr int NE = H * 2 * HW;
  static constexpr int NH = (NE + NT - 1) / NT;
};

template <int NT, int H, int HW>
__device__ __forceinline__ void side_cell(int i, int* r, int* c) {
  constexpr int NE = SideHalo<NT, H, HW>::NE;
  const int e = min((int)threadIdx.x + i * NT, NE - 1);
  *r = e / (2 * HW);
  const int cc = e - *r * (2 * HW);
  *c = cc < HW ? cc : kTX + cc;          // columns 0 .. HW-1 and 64+HW .. 64+2HW-1
}

template <int NT, int H, int HW>
__device__ __forceinline__ void side_offsets(int (&ho)[(SideHalo<NT, H, HW>::NH)], int nx, int nz, int px,
                                             int x0, int z0) {
#pragma unroll
  for (int i = 0; i < SideHalo<NT, H, HW>::NH; ++i) {
    // a slot past the last side cell takes the last cell (side_cell clamps): it loads and
    // writes the same value as that cell's owner, so the staging needs no condition
    int r, c;
    side_cell<NT, H, HW>(i, &r, &c);
    ho[i] = col_off(x0 - HW + c, z0 - HW + r, nx, nz, px, 4);
  }
}

// Stage rows z0-HW .. z0+TZ+HW-1, columns x0-HW .. x0+63+HW of a field into LDS (W = 64 + 2 HW
// columns, H rows), zero outside the grid: the 64-column body of each row is one aligned
// 256-byte row segment per wave (row offset wave-uniform, column offset cx = 4 x or kOOB), the
// side cells follow from their precomputed offsets.  All loads are issued before the first LDS
// write.
// The staging is split in two: `issue` loads this thread's cells into registers, `commit` writes
// them to LDS.  A kernel issues its tile before its other prefetches: loads complete in issue
// order, so the LDS writes then wait for the tile's loads alone, not for every prefetch.
template <int NT, int NW, int H, int HW>
struct Staged {
  static constexpr int NB = H / NW, NH = SideHalo<NT, H, HW>::NH;
  float vb[NB], vh[NH];
};

template <int NT, int NW, int H, int HW>
__device__ __forceinline__ void stage_issue(Staged<NT, NW, H, HW>& s, const Planes& f, int cx,
                                            const int (&ho)[(SideHalo<NT, H, HW>::NH)], int z0) {
  // every wave stages whole rows: no row condition, so no branch separates the loads from
  // their use (a branch would make the compiler wait for all loads at its start)
  static_assert(H % NW == 0, "staged rows must split evenly over the waves");
  const int wv = wave_id();
#pragma unroll
  for (int i = 0; i < Staged<NT, NW, H, HW>::NB; ++i) s.vb[i] = ldp(f, cx, z0 - HW + wv + i * NW);
#pragma unroll
  for (int i = 0; i < Staged<NT, NW, H, HW>::NH; ++i) s.vh[i] = ldp_at(f, ho[i]);
}

template <int NT, int NW, int H, int HW, int W>
__device__ __forceinline__ void stage_commit(float (*L)[W], const Staged<NT, NW, H, HW>& s) {
  const int lane = threadIdx.x & 63, wv = wave_id();
#pragma unroll
  for (int i = 0; i < Staged<NT, NW, H, HW>::NB; ++i) L[wv + i * NW][lane + HW] = s.vb[i];
  // unconditional: threads past the last side cell write that cell's own value again (a
  // condition here would let the compiler sink the load into it and wait for every load)
#pragma unroll
  for (int i = 0; i < Staged<NT, NW, H, HW>::NH; ++i) {
    int r, c;
    side_cell<NT, H, HW>(i, &r, &c);
    L[r][c] = s.vh[i];
  }
}

template <int TZ>
using Side4 = SideHalo<T2<TZ>::NT, T2<TZ>::H, kHalo>;

// The previous level with a 4-cell halo (one-step kernels): issue, then commit to LDS.
template <int TZ>
using Tile4 = Staged<T2<TZ>::NT, T2<TZ>::NW, T2<TZ>::H, kHalo>;

template <int TZ>
__device__ __forceinline__ void tile_issue(Tile4<TZ>& t, const Planes& f, int cx, const int (&ho)[Side4<TZ>::NH],
                                           int z0) {
  stage_issue<T2<TZ>::NT, T2<TZ>::NW, T2<TZ>::H, kHalo>(t, f, cx, ho, z0);
}

template <int TZ>
__device__ __forceinline__ void tile_commit(float (*L)[T2<TZ>::W], const Tile4<TZ>& t) {
  stage_commit<T2<TZ>::NT, T2<TZ>::NW, T2<TZ>::H, kHalo, T2<TZ>::W>(L, t);
}

// Difference-form Laplacian at *p in an LDS array with row stride `stride` (x neighbours at
// +-1, z neighbours at +-stride); the order of the sum is fixed for every 2D kernel.
__device__ __forceinline__ float lap_ptr(const float* p, int stride, const float* c) {
  const float u = p[0];
  float s = 0.f;
#pragma unroll
  for (int r = kHalo; r >= 1; --r) {
    s += c[r] * ((p[-r] - u) + (p[r] - u));
    s += c[r] * ((p[-r * stride] - u) + (p[r * stride] - u));
  }
  return s;
}

// Increment coef (L u + s - (eta/dt)(u - u_prev)) of one update; the new level is
// (u + u - u_prev) + increment.
__device__ __forceinline__ float step_incr(float u, float um2, float cfv, float lap, float eta) {
  return cfv * (lap - eta * (u - um2));
}

// Source term weight * sample, fused explicitly: left to the compiler, a product hoisted out of the
// source's condition would be rounded by itself in some kernels and not in others.
__device__ __forceinline__ float add_source(float lap, float w, float q) { return __builtin_fmaf(w, q, lap); }

template <int TZ>
__device__ __forceinline__ float lap_at(const float (*L)[T2<TZ>::W], int lr, int lc,
                                        const float* c) {
  return lap_ptr(&L[lr + kHalo][lc + kHalo], T2<TZ>::W, c);
}

template <int TZ>
__device__ __forceinline__ float interp_lds(const float (*L)[T2<TZ>::W], int i, int k, int x0,
                                            int z0, const float* w) {
  const int C = i - x0 + kHalo, R = k - z0 + kHalo;
  return w[0] * L[R][C] + w[1] * L[R][C + 1] + w[2] * L[R + 1][C] + w[3] * L[R + 1][C + 1];
}

__device__ __forceinline__ float* fbuf(unsigned char* ws, const ShotDev& S, int b) {
  return reinterpret_cast<float*>(ws + S.fld) + (long long)b * S.npts;
}

// Where a one-level forward step reads level k of shot S.  kStoreF32R: the FULL FP32 store keeps
// every level bit for bit, so the step reads its two previous levels from it (written by the
// launch before, with ordinary stores that leave them in the caches) and the rotating buffers
// are not needed; otherwise the rotating buffers, or a checkpoint slot restored by reference.
template <int SK>
__device__ __forceinline__ const float* fwd_src(const StepArgs& a, const ShotDev& S, int k) {
  if (SK == kStoreF32R) return reinterpret_cast<const float*>(a.ws + S.store) + (long long)k * S.npts;
  return fwd_level(a, S, k);
}

// Column offset of a checkpoint slot's stores in kernels of one column per lane.  Two-level steps on 128-column
// tiles read a slot by column pairs, so where nx is odd the column after the last is written too: its lane read
// only zeros, so the value is 0.  (The rotating buffers are cleared as a whole before a solve.)
__device__ __forceinline__ int slot_col(int x, int nx) { return x < nx + (nx & 1) ? 4 * x : kOOB; }

// Bytes of the rotating buffer a one-level forward step writes level k into: with kStoreF32R only
// the last level goes there too (the receivers' last sample is taken from it), so the other
// levels' buffer stores are dropped by the range check.
template <int SK>
__device__ __forceinline__ int fwd_ring_bytes(const ShotDev& S, int k, int bytes) {
  return SK != kStoreF32R || k == S.nt - 1 ? bytes : 0;
}

// ------------------------------------------------------------------------------ forward
// Produces u^k (k = step - off) for every shot in the tile list; samples d^{k-1}.
template <int TZ, int SK>
__global__ __launch_bounds__(T2<TZ>::NT) void fwd2d_kernel(StepArgs a) {
  constexpr int RPT = T2<TZ>::RPT;
  __shared__ float L[T2<TZ>::H][T2<TZ>::W];
  const int tid = xcd_tile(blockIdx.x, a.ntiles);
  const TileDev T = a.t.tiles[a.tile_base + tid];
  const ShotDev& S = a.t.shots[T.shot];
  const int k = a.step - S.off;
  if (k < 1 || k >= S.nt) return;
  const int nx = S.nx, nz = S.nz, px = S.px;
  const int row4 = 4 * px;
  // levels below 1 are zero (initial state); their buffers may hold older levels after a
  // checkpoint restore of a state before this shot's start, so they are not read
  const Planes u1 = planes(fwd_src<SK>(a, S, k - 1), nz, k >= 2 ? nz : 0, row4);
  const Planes u2 = planes(fwd_src<SK>(a, S, k - 2), nz, k >= 3 ? nz : 0, row4);
  const Planes cf = planes(a.ws + S.coef, nz, nz, row4);
  const brsrc rout = make_rsrc(fbuf(a.ws, S, fwd_buf(k)), fwd_ring_bytes<SK>(S, k, nz * row4));
  const int lane = threadIdx.x & 63, wv = wave_id();
  const int x = T.x0 + lane;
  const int cx = x < nx ? 4 * x : kOOB;

  int ho[Side4<TZ>::NH];
  side_offsets<T2<TZ>::NT, T2<TZ>::H, kHalo>(ho, nx, nz, px, T.x0, T.z0);
  Tile4<TZ> tile;
  tile_issue<TZ>(tile, u1, cx, ho, T.z0);
  float pu2[RPT], pcf[RPT];
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    const int z = T.z0 + wv * RPT + i;
    pu2[i] = ldp(u2, cx, z);
    pcf[i] = ldp(cf, cx, z);
  }
  tile_commit<TZ>(L, tile);
  __syncthreads();

  if (a.d != nullptr) {
    for (int t = threadIdx.x; t < T.gat_count; t += T2<TZ>::NT) {
      const RecDev R = a.t.recs[T.gat_begin + t];
      a.d[S.d + (long long)(k - 1) * S.nrec + R.r] = interp_lds<TZ>(L, R.i, R.k, T.x0, T.z0, R.w);
    }
  }

  const float qk = a.q[S.q + k - 1];
  const int dx = border_dist(x, nx, a.nbl);
  // shot fields used in the row loop, in registers: a reload after a store would wait for every
  // store in flight
  const int src_i = S.src_i, src_k = S.src_k;
  const float sw0 = S.src_w[0], sw1 = S.src_w[1], sw2 = S.src_w[2], sw3 = S.src_w[3];
  const long long npts = S.npts;
  // FULL store: level k (FP32) or level k-1 (16 bits, quantised with its finished scale)
  constexpr bool F32 = SK == kStoreF32 || SK == kStoreF32R;
  const brsrc rst = F32
      ? make_rsrc(reinterpret_cast<float*>(a.ws + S.store) + (long long)k * npts, nz * row4)
      : make_rsrc(reinterpret_cast<unsigned short*>(a.ws + S.store) + (long long)(k - 1) * npts,
                  SK == kStoreBF16 || SK == kStoreFP16 ? nz * row4 / 2 : 0);
  // checkpoint store fused into the step that reaches the stored state: (u^k, u^{k-1}) into slot
  const bool to_slot = SK == kStoreNone && a.st_slot >= 0;
  float* sl = reinterpret_cast<float*>(a.ws + S.store) + (long long)(to_slot ? a.st_slot : 0) * 2 * npts;
  const brsrc rsl0 = make_rsrc(sl, to_slot ? nz * row4 : 0);
  const brsrc rsl1 = make_rsrc(sl + npts, to_slot ? nz * row4 : 0);
  const int cs = slot_col(x, nx);
  const int cx2 = x < nx ? 2 * x : kOOB;
  constexpr bool S16 = SK == kStoreBF16 || SK == kStoreFP16;
  float* scl = S16 ? reinterpret_cast<float*>(a.ws + S.scale) : nullptr;
  const float inv_prev = S16 && k >= 2 ? inv_scale(level_scale(scl, k - 1)) : 0.f;
  // probed gradient: the r FP64 sums B_j of this shot, and this level's coefficients
  double* pb = SK == kStoreProbe ? reinterpret_cast<double*>(a.ws + S.store) : nullptr;
  const float* pc = SK == kStoreProbe ? a.probe_c + k : nullptr;
  float lmax = 0.f;
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    // every lane computes; outside the grid u, u^{k-2} and coef read 0 (so the new value is 0)
    // and the stores are dropped
    const int lr = wv * RPT + i;
    const int z = T.z0 + lr;
    const float u = L[lr + kHalo][lane + kHalo];
    float lap = lap_at<TZ>(L, lr, lane, a.c);
    const int bx = x - src_i, bz = z - src_k;
    if ((unsigned)bx < 2u && (unsigned)bz < 2u) {
      const int w = bx + 2 * bz;
      lap = add_source(lap, w == 0 ? sw0 : w == 1 ? sw1 : w == 2 ? sw2 : sw3, qk);
    }
    const int dz = border_dist(z, nz, a.nbl);
    const float eta = a.eta_dt * (float)(dx * dx + dz * dz);
    const float incr = step_incr(u, pu2[i], pcf[i], lap, eta);
    const float un = (u + u - pu2[i]) + incr;
    const int zo = z * row4;
    stb(rout, un, cx, zo);
    if (to_slot) {
      stb(rsl0, un, cs, zo);
      stb(rsl1, u, cs, zo);
    }
    // a stored level the next launch reads back stays in the caches; otherwise it is written once
    // and read thousands of launches later
    if (SK == kStoreF32) stb_nt(rst, un, cx, zo);
    if (SK == kStoreF32R) stb(rst, un, cx, zo);
    if (S16) {
      lmax = fmaxf(lmax, fabsf(un));
      if (k >= 2) stb16_nt(rst, enc16(u * inv_prev, SK == kStoreBF16), cx2, zo / 2);
    }
    if (SK == kStoreProbe && x < nx && z < nz) {
      // u^k - 2u^{k-1} + u^{k-2} = incr (increment form of the step)
      const long long p = (long long)z * px + x;
      probe_add(probe_sums(pb, p, a.probe_r), a.probe_r, pc, (double)incr, true, nullptr, 0.0, false, a.probe_pitch);
    }
  }
  if (S16) block_max_to_slot<T2<TZ>::NW, false>(lmax, scl, k);
}

// ------------------------------------------------------------------------------ adjoint
// Produces w^j (j = step - off) from w^{j+1} (LDS) and w^{j+2}; injects P_r^T dd^j; samples
// v^j = R(x_s) w^{j+1} / h^ndim; IMG adds u^j * (w^j - 2w^{j+1} + w^{j+2}) into the FP64
// accumulator (u^j from the FULL store or from the recomputed forward buffers).
template <int TZ, int IMG>
__global__ __launch_bounds__(T2<TZ>::NT) void adj2d_kernel(StepArgs a) {
  constexpr int RPT = T2<TZ>::RPT;
  __shared__ float L[T2<TZ>::H][T2<TZ>::W];
  __shared__ float INJ[TZ][kTX];
  const int tid = xcd_tile(blockIdx.x, a.ntiles);
  const TileDev T = a.t.tiles[a.tile_base + tid];
  const ShotDev& S = a.t.shots[T.shot];
  const int j = a.step - S.off;
  if (j < 1 || j >= S.nt) return;
  const int nx = S.nx, nz = S.nz, px = S.px;
  const int row4 = 4 * px;
  const Planes w1 = planes(fbuf(a.ws, S, adj_buf(j + 1)), nz, nz, row4);
  const Planes w2 = planes(fbuf(a.ws, S, adj_buf(j + 2)), nz, nz, row4);
  const Planes cf = planes(a.ws + S.coef, nz, nz, row4);
  const brsrc rout = make_rsrc(fbuf(a.ws, S, adj_buf(j)), nz * row4);
  // imaging: u^j from the FULL store (FP32, or 16 bits with the level's scale) or the forward
  // buffers, and the FP64 accumulator
  constexpr bool I16 = IMG == kImgFullBF16 || IMG == kImgFullFP16;
  constexpr bool IACC = IMG != kImgNone && IMG != kImgProbe;  // imaging into the FP64 accumulator
  const void* ubase = IMG == kImgBuffers ? (const void*)fwd_level(a, S, j)
                      : IMG == kImgFull32 ? (const void*)(reinterpret_cast<const float*>(a.ws + S.store) + (long long)j * S.npts)
                      : (const void*)(reinterpret_cast<const unsigned short*>(a.ws + S.store) + (long long)j * S.npts);
  const Planes uj = planes(ubase, nz, IACC ? nz : 0, I16 ? row4 / 2 : row4);
  const float usc = I16 ? level_scale(reinterpret_cast<const float*>(a.ws + S.scale), j) : 1.f;
  const Planes acc = planes(a.ws + S.acc, nz, IACC ? nz : 0, 2 * row4);
  const brsrc racc = make_rsrc(a.ws + S.acc, IACC ? 2 * nz * row4 : 0);
  // probed gradient: the r FP64 sums A_j of this shot (after its B_j), and this level's coefficients
  double* pa = IMG == kImgProbe ? reinterpret_cast<double*>(a.ws + S.store) + (long long)a.probe_r * S.npts : nullptr;
  const float* pc = IMG == kImgProbe ? a.probe_c + j : nullptr;
  const int lane = threadIdx.x & 63, wv = wave_id();
  const int x = T.x0 + lane;
  const int cx = x < nx ? 4 * x : kOOB;
  const int cxu = x < nx ? (I16 ? 2 : 4) * x : kOOB;
  const int cx8 = x < nx ? 8 * x : kOOB;
  const bool has_inj = T.inj_count > 0 && a.dd != nullptr;  // no residual: nothing to inject

  int ho[Side4<TZ>::NH];
  side_offsets<T2<TZ>::NT, T2<TZ>::H, kHalo>(ho, nx, nz, px, T.x0, T.z0);
  Tile4<TZ> tile;
  tile_issue<TZ>(tile, w1, cx, ho, T.z0);
  float pw2[RPT], pcf[RPT], pu[RPT];
  double pacc[RPT];
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    const int z = T.z0 + wv * RPT + i;
    pw2[i] = ldp(w2, cx, z);
    pcf[i] = ldp(cf, cx, z);
    if (I16) pu[i] = dec16(ldp16_nt(uj, cxu, z), IMG == kImgFullBF16) * usc;
    else if (IMG == kImgFull32) pu[i] = ldp_nt(uj, cxu, z);
    else if (IACC) pu[i] = ldp(uj, cxu, z);
    if (IACC) pacc[i] = ldp64(acc, cx8, z);
    if (has_inj) INJ[wv * RPT + i][lane] = 0.f;
  }
  tile_commit<TZ>(L, tile);
  __syncthreads();

  if (has_inj) {
    const float* ddj = a.dd + S.d + (long long)j * S.nrec;
    for (int t = threadIdx.x; t < T.inj_count; t += T2<TZ>::NT) {
      const InjPoint P = a.t.inj_pts[T.inj_begin + t];
      float s = 0.f;
      for (int e = 0; e < P.e_count; ++e) {
        const InjEntry E = a.t.inj_ent[P.e_begin + e];
        s += E.w * ddj[E.r];
      }
      INJ[P.lz][P.lx] = s;
    }
    __syncthreads();
  }
  if (a.v != nullptr && a.tile_base + tid == S.src_tile && threadIdx.x == 0)
    a.v[S.q + j] = interp_lds<TZ>(L, S.src_i, S.src_k, T.x0, T.z0, S.src_w);

  const int dx = border_dist(x, nx, a.nbl);
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    // every lane computes; outside the grid the stores are dropped
    const int lr = wv * RPT + i;
    const int z = T.z0 + lr;
    const float w = L[lr + kHalo][lane + kHalo];
    float lap = lap_at<TZ>(L, lr, lane, a.c);
    if (has_inj) lap += INJ[lr][lane];
    const int dz = border_dist(z, nz, a.nbl);
    const float eta = a.eta_dt * (float)(dx * dx + dz * dz);
    const float incr = step_incr(w, pw2[i], pcf[i], lap, eta);
    const int zo = z * row4;
    const float wn = (w + w - pw2[i]) + incr;
    stb(rout, wn, cx, zo);
    if (IACC) stb64(racc, pacc[i] + (double)pu[i] * (double)incr, cx8, 2 * zo);
    if (IMG == kImgProbe && x < nx && z < nz) {
      const long long p = (long long)z * px + x;
      probe_add(probe_sums(pa, p, a.probe_r), a.probe_r, pc, (double)wn, true, nullptr, 0.0, false, a.probe_pitch);
    }
  }
}

// ------------------------------------------------------------------------------ Born
// Produces u^k and du^k together; samples (J dm)^{k-1} = R du^{k-1}.
template <int TZ>
__global__ __launch_bounds__(T2<TZ>::NT) void born2d_kernel(StepArgs a) {
  constexpr int RPT = T2<TZ>::RPT;
  __shared__ float LU[T2<TZ>::H][T2<TZ>::W];
  __shared__ float LD[T2<TZ>::H][T2<TZ>::W];
  const int tid = xcd_tile(blockIdx.x, a.ntiles);
  const TileDev T = a.t.tiles[a.tile_base + tid];
  const ShotDev& S = a.t.shots[T.shot];
  const int k = a.step - S.off;
  if (k < 1 || k >= S.nt) return;
  const int nx = S.nx, nz = S.nz, px = S.px;
  const int row4 = 4 * px;
  const Planes u1 = planes(fbuf(a.ws, S, fwd_buf(k - 1)), nz, nz, row4);
  const Planes u2 = planes(fbuf(a.ws, S, fwd_buf(k - 2)), nz, nz, row4);
  const Planes d1 = planes(fbuf(a.ws, S, adj_buf(k - 1)), nz, nz, row4);
  const Planes d2 = planes(fbuf(a.ws, S, adj_buf(k - 2)), nz, nz, row4);
  const Planes cf = planes(a.ws + S.coef, nz, nz, row4);
  const Planes dm = planes(a.dm + S.m, nz, nz, 4LL * nx);   // caller's layout: rows of nx
  const brsrc ruo = make_rsrc(fbuf(a.ws, S, fwd_buf(k)), nz * row4);
  const brsrc rdo = make_rsrc(fbuf(a.ws, S, adj_buf(k)), nz * row4);
  const int lane = threadIdx.x & 63, wv = wave_id();
  const int x = T.x0 + lane;
  const int cx = x < nx ? 4 * x : kOOB;

  int ho[Side4<TZ>::NH];
  side_offsets<T2<TZ>::NT, T2<TZ>::H, kHalo>(ho, nx, nz, px, T.x0, T.z0);
  Tile4<TZ> tu, td;
  tile_issue<TZ>(tu, u1, cx, ho, T.z0);
  tile_issue<TZ>(td, d1, cx, ho, T.z0);
  float pu2[RPT], pd2[RPT], pcf[RPT], pdm[RPT];
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    const int z = T.z0 + wv * RPT + i;
    pu2[i] = ldp(u2, cx, z);
    pd2[i] = ldp(d2, cx, z);
    pcf[i] = ldp(cf, cx, z);
    pdm[i] = ldp(dm, cx, z);
  }
  tile_commit<TZ>(LU, tu);
  tile_commit<TZ>(LD, td);
  __syncthreads();

  if (a.d != nullptr) {
    for (int t = threadIdx.x; t < T.gat_count; t += T2<TZ>::NT) {
      const RecDev R = a.t.recs[T.gat_begin + t];
      a.d[S.d + (long long)(k - 1) * S.nrec + R.r] = interp_lds<TZ>(LD, R.i, R.k, T.x0, T.z0, R.w);
    }
  }

  const int src_i = S.src_i, src_k = S.src_k;   // in registers (see the forward kernel)
  const float sw0 = S.src_w[0], sw1 = S.src_w[1], sw2 = S.src_w[2], sw3 = S.src_w[3];
  const float qk = a.q[S.q + k - 1];
  const int dx = border_dist(x, nx, a.nbl);
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    // every lane computes; outside the grid the stores are dropped
    const int lr = wv * RPT + i;
    const int z = T.z0 + lr;
    const int dz = border_dist(z, nz, a.nbl);
    const float eta = a.eta_dt * (float)(dx * dx + dz * dz);
    const int zo = z * row4;
    // background field
    const float u = LU[lr + kHalo][lane + kHalo];
    float lap = lap_at<TZ>(LU, lr, lane, a.c);
    const int bx = x - src_i, bz = z - src_k;
    if ((unsigned)bx < 2u && (unsigned)bz < 2u) {
      const int w = bx + 2 * bz;
      lap = add_source(lap, w == 0 ? sw0 : w == 1 ? sw1 : w == 2 ? sw2 : sw3, qk);
    }
    const float incr = pcf[i] * (lap - eta * (u - pu2[i]));
    stb(ruo, (u + u - pu2[i]) + incr, cx, zo);
    // scattered field, source -dm (u^k - 2u^{k-1} + u^{k-2}) / dt^2 = -dm incr / dt^2
    const float du = LD[lr + kHalo][lane + kHalo];
    const float lapd = lap_at<TZ>(LD, lr, lane, a.c) - pdm[i] * incr * a.inv_dt2;
    const float incd = pcf[i] * (lapd - eta * (du - pd2[i]));
    stb(rdo, (du + du - pd2[i]) + incd, cx, zo);
  }
}

// ------------------------------------------------------------------------------ two steps per launch
// A tile of TZ rows x 64 V columns (V = 1, 2).  Level n-1 is staged with an 8-cell halo (LDS L1); the first
// step computes level n on the tile plus a 4-cell halo (LDS LE: everything the second step's
// stencil needs), the second step computes level n+1 (forward) or n-1 (adjoint) on the tile.  Both
// steps do exactly the arithmetic of the one-step kernels, in the same order, so results are
// bitwise identical; HBM traffic per two steps falls from 2 x (3 reads + 1 write) to 3 reads +
// 2 writes.
//
// Vector issue is most of a forward launch's time (at one wave instruction per cycle and compute unit 61 % of
// one with FP32 store, 70 % without) and 45 % of a reverse launch's, so the work per point is cut: a lane owns V adjacent columns (V = 2: 8-byte global and LDS
// accesses, one set of address and row work for two points) and RA or RB consecutive rows, whose
// z-neighbours it reads from LDS once (N + 8 reads for N rows instead of 9 N); along x a difference
// u(b) - u(a) that serves the stencils of two of its points is formed once.  A row of the tile is one
// wave, so row offsets stay wave-uniform.  Rows are kept apart for the scheduler: mixed, they took 125
// registers instead of 80 (24-row forward, V = 2) and lost more to occupancy than they gained.
// V = 1 (64-column tiles) wastes fewer columns where the width is no multiple of 128 and shortens the
// chain of a small launch; wide_tiles holds the rule.
// Measured, 16 shots of 730 x 421, us per launch of two levels, against one column and row at a time:
// forward without store 23.4 -> 21.3 (V = 2), with FP32 store 24.7 -> 23.3, reverse with imaging 41.4 ->
// 38.0; one shot of 281 x 181, against one level per launch twice: forward 7.4 -> 4.0.  Lane-operations per
// point and level with the halos' (SQ_INSTS_VALU, 16 shots of 730 x 421): forward with FP32 store 79 -> 60,
// reverse with imaging 93 -> 68.

// V adjacent columns of a lane.
template <int V>
struct VecOf {
  typedef float f32 __attribute__((ext_vector_type(V)));
  typedef double f64 __attribute__((ext_vector_type(V)));
};
template <int V>
using fv = typename VecOf<V>::f32;
template <int V>
using dv = typename VecOf<V>::f64;

template <int V, int AUX = 0>
__device__ __forceinline__ fv<V> ldv(brsrc r, int voff, int soff) {
  if constexpr (V == 2) return __builtin_bit_cast(fv<V>, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, AUX));
  else return __builtin_bit_cast(fv<V>, __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, AUX));
}
template <int V, int AUX = 0>
__device__ __forceinline__ fv<V> ldpv(const Planes& f, int voff, int z) {
  return ldv<V, AUX>(f.r, voff, slice_off(f, z));
}
template <int V>
__device__ __forceinline__ fv<V> ldpv_at(const Planes& f, int off) {
  return ldv<V>(f.r, off, f.nzv > 0 ? 0 : kZOOB);
}
template <int V, int AUX = 0>
__device__ __forceinline__ void stv(brsrc r, fv<V> v, int voff, int soff) {
  typedef unsigned u2 __attribute__((ext_vector_type(2)));
  if constexpr (V == 2) __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, v), r, voff, soff, AUX);
  else __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v[0]), r, voff, soff, AUX);
}
// V 16-bit codes, two to a 32-bit word (byte offsets as in ldv, stv).
template <int V>
__device__ __forceinline__ unsigned ldpv16(const Planes& f, int voff, int z) {
  if constexpr (V == 2) return __builtin_amdgcn_raw_buffer_load_b32(f.r, voff, slice_off(f, z), kNT);
  else return ldp16_nt(f, voff, z);
}
template <int V>
__device__ __forceinline__ fv<V> dec16v(unsigned b, int bf16, float scale) {
  fv<V> r;
#pragma unroll
  for (int i = 0; i < V; ++i) r[i] = dec16((unsigned short)(b >> (16 * i)), bf16) * scale;
  return r;
}
template <int V>
__device__ __forceinline__ void stv16(brsrc r, fv<V> v, float inv, int bf16, int voff, int soff) {
  unsigned b = enc16(v[0] * inv, bf16);
  if constexpr (V == 2) {
    b |= (unsigned)enc16(v[1] * inv, bf16) << 16;
    __builtin_amdgcn_raw_buffer_store_b32(b, r, voff, soff, kNT);
  } else {
    stb16_nt(r, (unsigned short)b, voff, soff);
  }
}
template <int V>
__device__ __forceinline__ float absmax(float m, fv<V> v) {
#pragma unroll
  for (int i = 0; i < V; ++i) m = fmaxf(m, fabsf(v[i]));
  return m;
}
template <int V>
__device__ __forceinline__ dv<V> ldpacc(const Planes& f, int voff, int z) {
  if constexpr (V == 2) return ldp64x2(f, voff, z);
  else return dv<V>{ldp64(f, voff, z)};
}
template <int V>
__device__ __forceinline__ void stacc(brsrc r, dv<V> v, int voff, int soff) {
  if constexpr (V == 2) stb64x2(r, v, voff, soff);
  else stb64(r, v[0], voff, soff);
}
template <int V>
__device__ __forceinline__ fv<V>& lds(float& p) {
  return *reinterpret_cast<fv<V>*>(&p);
}
template <int V>
__device__ __forceinline__ const fv<V>& lds(const float& p) {
  return *reinterpret_cast<const fv<V>*>(&p);
}

template <int TZ, int V>
struct F2 {
  static constexpr int TX = 64 * V;
  static constexpr int W1 = TX + 4 * kHalo;       // level n-1 with an 8-cell halo
  static constexpr int H1 = TZ + 4 * kHalo;
  static constexpr int WE = TX + 2 * kHalo;       // first-step level on tile + 4
  static constexpr int HE = TZ + 2 * kHalo;
  static constexpr int NW = 8;                    // waves per workgroup
  static constexpr int NT = 64 * NW;
  static constexpr int RA = HE / NW;              // first-step rows of a wave (body columns)
  static constexpr int RB = TZ / NW;              // second-step rows of a wave
  static_assert(HE % NW == 0 && TZ % NW == 0, "rows must split evenly over the waves");
  // groups of V columns in the halo columns: NSE of the first step (4 + 4 columns of HE rows), NS1 of
  // the staged level (8 + 8 columns of H1 rows); thread t takes group t
  static constexpr int NSE = HE * 2 * kHalo / V, NS1 = H1 * 4 * kHalo / V;
  static constexpr int MS1 = (NS1 + NT - 1) / NT;
  static_assert(NSE <= NT, "one halo group per thread");
};

// Row and column of group e of the halo columns of a region with HW halo columns per side.
template <int V, int HW>
__device__ __forceinline__ void side_cols(int e, int* r, int* c) {
  constexpr int N = 2 * HW / V;
  *r = e / N;
  const int k = V * (e - *r * N);
  *c = k < HW ? k : 64 * V + k;
}

// Level n-1 with an 8-cell halo: rows z0-8 .. z0+TZ+7, whole rows per wave plus the halo columns.
// Issue before the other prefetches, commit to LDS (see Staged).
template <int TZ, int V>
struct Tile8 {
  using G = F2<TZ, V>;
  static constexpr int NB = G::H1 / G::NW;
  static_assert(G::H1 % G::NW == 0, "staged rows must split evenly over the waves");
  fv<V> vb[NB], vh[G::MS1];

  __device__ __forceinline__ void issue(const Planes& f, int cx, int x0, int z0, int nx, int nz, int px) {
    const int wv = wave_id();
#pragma unroll
    for (int i = 0; i < NB; ++i) vb[i] = ldpv<V>(f, cx, z0 - 2 * kHalo + wv + i * G::NW);
#pragma unroll
    for (int i = 0; i < G::MS1; ++i) {
      int r, c;
      side_cols<V, 2 * kHalo>(min((int)threadIdx.x + i * G::NT, G::NS1 - 1), &r, &c);
      vh[i] = ldpv_at<V>(f, col_off(x0 - 2 * kHalo + c, z0 - 2 * kHalo + r, nx, nz, px, 4));
    }
  }
  __device__ __forceinline__ void commit(float (*L)[G::W1]) const {
    const int lane = threadIdx.x & 63, wv = wave_id();
#pragma unroll
    for (int i = 0; i < NB; ++i) lds<V>(L[wv + i * G::NW][2 * kHalo + V * lane]) = vb[i];
    // unconditional: threads past the last group write that group again (see stage_commit)
#pragma unroll
    for (int i = 0; i < G::MS1; ++i) {
      int r, c;
      side_cols<V, 2 * kHalo>(min((int)threadIdx.x + i * G::NT, G::NS1 - 1), &r, &c);
      lds<V>(L[r][c]) = vh[i];
    }
  }
};

// Laplacians of the V columns at p (an LDS array of row stride W) in N consecutive rows, p at
// the first; u receives the centre values.  The order of each sum is that of lap_ptr; along x a
// difference is formed once for the points it belongs to ((a - u) + (b - u) = (b - u) - (u - a)).
template <int V, int N, int W>
__device__ __forceinline__ void lap_rows(const float* p, fv<V> (&lap)[N], fv<V> (&u)[N], const float* c) {
  fv<V> P[N + 2 * kHalo];
#pragma unroll
  for (int i = 0; i < N + 2 * kHalo; ++i) P[i] = lds<V>(p[(i - kHalo) * W]);
#pragma unroll
  for (int n = 0; n < N; ++n) {
    __builtin_amdgcn_sched_barrier(0);   // one row after the other
    const float* q = p + n * W;
    float X[2 * kHalo + V];        // columns x-4 .. x+V+3
#pragma unroll
    for (int k = 0; k < 2 * kHalo + V; k += V) {
      const fv<V> v = k == kHalo ? P[n + kHalo] : lds<V>(q[k - kHalo]);
#pragma unroll
      for (int i = 0; i < V; ++i) X[k + i] = v[i];
    }
    u[n] = P[n + kHalo];
    float s[V] = {};
#pragma unroll
    for (int r = kHalo; r >= 1; --r) {
      float D[2 * kHalo + V];      // D[k] = X[k + r] - X[k] at the columns and r to their left
#pragma unroll
      for (int k = kHalo - r; k < kHalo + V; ++k) D[k] = X[k + r] - X[k];
#pragma unroll
      for (int i = 0; i < V; ++i) {
        s[i] += c[r] * (D[kHalo + i] - D[kHalo + i - r]);
        s[i] += c[r] * ((P[n + kHalo - r][i] - P[n + kHalo][i]) + (P[n + kHalo + r][i] - P[n + kHalo][i]));
      }
    }
#pragma unroll
    for (int i = 0; i < V; ++i) lap[n][i] = s[i];
  }
}

// Squared border distances of a lane's columns.
template <int V>
struct Damp {
  float d2[V];
  __device__ __forceinline__ Damp(int x, int nx, int nbl) {
#pragma unroll
    for (int i = 0; i < V; ++i) {
      const float d = (float)border_dist(x + i, nx, nbl);
      d2[i] = d * d;
    }
  }
};

// One update of V columns at border distance dz: (increment, new level).  The sum of the squared distances
// is the integers' sum bit for bit (both far below 2^24).
template <int V>
__device__ __forceinline__ void step_cols(fv<V> u, fv<V> um2, fv<V> cf, fv<V> lap, const Damp<V>& d, int dz,
                                          float eta_dt, fv<V>* incr, fv<V>* un) {
  const float fz = (float)dz * (float)dz;
#pragma unroll
  for (int i = 0; i < V; ++i) {
    const float inc = step_incr(u[i], um2[i], cf[i], lap[i], eta_dt * (d.d2[i] + fz));
    (*incr)[i] = inc;
    (*un)[i] = (u[i] + u[i] - um2[i]) + inc;
  }
}

// Source term of the columns x, x + 1, ... at row z.
struct Source {
  int i, k;
  float w0, w1, w2, w3;
  __device__ __forceinline__ explicit Source(const ShotDev& S)
      : i(S.src_i), k(S.src_k), w0(S.src_w[0]), w1(S.src_w[1]), w2(S.src_w[2]), w3(S.src_w[3]) {}
  template <int V>
  __device__ __forceinline__ void add(fv<V>* lap, int x, int z, float q) const {
    if ((unsigned)(z - k) < 2u) {
      const float a = z == k ? w0 : w2, b = z == k ? w1 : w3;
      const int b0 = x - i;
      if ((unsigned)(b0 + V - 1) < (unsigned)(V + 1)) {
#pragma unroll
        for (int c = 0; c < V; ++c)
          if ((unsigned)(b0 + c) < 2u) (*lap)[c] = add_source((*lap)[c], b0 + c == 0 ? a : b, q);
      }
    }
  }
};

// probe_add for V columns: sum j of adjacent points is adjacent (x is a multiple of V, and a second
// column may lie in the row's padding, whose terms are zero).
template <int V>
__device__ __forceinline__ void probe_cols(double* sum, int r, const float* c1, fv<V> v1, bool t1, const float* c2,
                                           fv<V> v2, bool t2, long long pitch) {
  constexpr int kGroup = kProbeGroup / V;   // as many bytes in flight as probe_add
  for (int j0 = 0; j0 < r; j0 += kGroup) {
    dv<V> t[kGroup];
    const int n = min(r - j0, kGroup);
    dv<V>* s = reinterpret_cast<dv<V>*>(sum + j0 * 64);
#pragma unroll
    for (int u = 0; u < kGroup; ++u)
      if (u < n) t[u] = __builtin_nontemporal_load(s + u * (64 / V));
#pragma unroll
    for (int u = 0; u < kGroup; ++u)
      if (u < n) {
        if (t1) {
          const double c = c1[(j0 + u) * pitch];
#pragma unroll
          for (int i = 0; i < V; ++i) t[u][i] += c * (double)v1[i];
        }
        if (t2) {
          const double c = c2[(j0 + u) * pitch];
#pragma unroll
          for (int i = 0; i < V; ++i) t[u][i] += c * (double)v2[i];
        }
      }
#pragma unroll
    for (int u = 0; u < kGroup; ++u)
      if (u < n) __builtin_nontemporal_store(t[u], s + u * (64 / V));
  }
}

template <int W>
__device__ __forceinline__ float interp_at(const float (*L)[W], int R, int C, const float* w) {
  return w[0] * L[R][C] + w[1] * L[R][C + 1] + w[2] * L[R + 1][C] + w[3] * L[R + 1][C + 1];
}

// Samples the tile's receivers from an LDS level whose cell (0, 0) is the grid point (zl, xl).
template <int NT, int W>
__device__ __forceinline__ void gather(const StepArgs& a, const TileDev& T, const ShotDev& S, const float (*L)[W],
                                       int zl, int xl, int level) {
  for (int t = threadIdx.x; t < T.gat_count; t += NT) {
    const RecDev R = a.t.recs[T.gat_begin + t];
    a.d[S.d + (long long)level * S.nrec + R.r] = interp_at<W>(L, R.k - zl, R.i - xl, R.w);
  }
}

// Forward: levels k and k+1 (k = step - off); SK = kStoreNone, kStoreF32, kStoreBF16 / kStoreFP16 or
// kStoreProbe (both levels' increments added to the probe sums in one FP64 read-modify-write, level k
// first), or kStoreSlot (a checkpoint advance: reads a slot by reference, the state reached may go into one).
// A 16-bit store takes the levels k-2 and k-1, whose scales the launch before finished, from the values the
// first step has in registers, and this launch's maxima go to the levels' slots: the gradient of
// 3 shots of 261 x 185 (501 samples) 4.94 -> 3.27 ms against one level per launch.
// a.single: level k alone.
template <int TZ, int V, int SK>
__global__ __launch_bounds__((F2<TZ, V>::NT)) void fwd2d2_kernel(StepArgs a) {
  using G = F2<TZ, V>;
  constexpr bool PRB = SK == kStoreProbe;
  constexpr bool S16 = SK == kStoreBF16 || SK == kStoreFP16;
  constexpr int RA = G::RA, RB = G::RB;
  __shared__ __align__(16) float L1[G::H1][G::W1];
  __shared__ __align__(16) float LE[G::HE][G::WE];
  __shared__ float RED[S16 ? 2 * G::NW : 1];
  __shared__ __align__(16) float INC1[PRB ? TZ : 1][G::TX];  // probe: level k's increment on the tile
  const int tid = xcd_tile(blockIdx.x, a.ntiles);
  const TileDev T = a.t.tiles[a.tile_base + tid];
  const ShotDev& S = a.t.shots[T.shot];
  const int k = a.step - S.off;
  const bool act1 = k >= 1 && k <= S.nt - 1;
  const bool act2 = !a.single && k + 1 >= 1 && k + 1 <= S.nt - 1;
  if (!act1 && !act2) return;
  const int nx = S.nx, nz = S.nz, px = S.px;
  const int row4 = 4 * px;
  // levels below 1 are zero (see fwd2d_kernel); kStoreSlot may follow a restore by reference, whose look-up
  // the other kinds are spared (it delays the tile's loads)
  constexpr bool SLOT = SK == kStoreSlot;
  const Planes u1 = planes(SLOT ? fwd_level(a, S, k - 1) : fbuf(a.ws, S, fwd_buf(k - 1)), nz, k >= 2 ? nz : 0, row4);
  const Planes u2 = planes(SLOT ? fwd_level(a, S, k - 2) : fbuf(a.ws, S, fwd_buf(k - 2)), nz, k >= 3 ? nz : 0, row4);
  const Planes cf = planes(a.ws + S.coef, nz, nz, row4);
  const long long npts = S.npts;
  // new levels k and k+1 (a level outside 1..nt-1 belongs to an inactive step: no records)
  const brsrc ro1 = make_rsrc(fbuf(a.ws, S, fwd_buf(k)), act1 ? nz * row4 : 0);
  const brsrc ro2 = make_rsrc(fbuf(a.ws, S, fwd_buf(k + 1)), act2 ? nz * row4 : 0);
  float* st = reinterpret_cast<float*>(a.ws + S.store);
  const brsrc rs1 = make_rsrc(st + (long long)(SK == kStoreF32 && act1 ? k : 0) * npts,
                              SK == kStoreF32 && act1 ? nz * row4 : 0);
  const brsrc rs2 = make_rsrc(st + (long long)(SK == kStoreF32 && act2 ? k + 1 : 0) * npts,
                              SK == kStoreF32 && act2 ? nz * row4 : 0);
  // checkpoint slot: the last level, and the one before it (level k-1 when this launch ends at k)
  const bool to_slot = SLOT && a.st_slot >= 0;
  float* sl = st + (long long)(to_slot ? a.st_slot : 0) * 2 * npts;
  const int slb = to_slot ? nz * row4 : 0;
  const brsrc rsl0 = make_rsrc(sl, a.single ? 0 : slb);
  const brsrc rslv = make_rsrc(a.single ? sl : sl + npts, slb), rslu = make_rsrc(sl + npts, a.single ? slb : 0);
  // 16-bit store: the levels k-1 and k-2
  unsigned short* st16 = reinterpret_cast<unsigned short*>(a.ws + S.store);
  const bool has1 = S16 && k >= 2, has2 = S16 && k >= 3;
  const brsrc rq1 = make_rsrc(st16 + (has1 ? k - 1 : 0) * npts, has1 ? nz * row4 / 2 : 0);
  const brsrc rq2 = make_rsrc(st16 + (has2 ? k - 2 : 0) * npts, has2 ? nz * row4 / 2 : 0);
  float* scl = S16 ? reinterpret_cast<float*>(a.ws + S.scale) : nullptr;
  const float inv1 = has1 ? inv_scale(level_scale(scl, k - 1)) : 0.f;
  const float inv2 = has2 ? inv_scale(level_scale(scl, k - 2)) : 0.f;
  const int lane = threadIdx.x & 63, wv = wave_id();
  const int x = T.x0 + V * lane;
  const int cx = x < nx ? 4 * x : kOOB;
  const int cx2 = x < nx ? 2 * x : kOOB;
  const int cs = V == 1 ? slot_col(x, nx) : cx;
  const int zE = T.z0 - kHalo;           // row 0 of the first-step region

  // the level k-1 tile first, then level k-2 and coef of this thread's first-step points and coef
  // of its tile points
  Tile8<TZ, V> tile;
  tile.issue(u1, cx, T.x0, T.z0, nx, nz, px);
  fv<V> pm2[RA], pcf[RA], tcf[RB];
#pragma unroll
  for (int i = 0; i < RA; ++i) {
    pm2[i] = ldpv<V>(u2, cx, zE + wv * RA + i);
    pcf[i] = ldpv<V>(cf, cx, zE + wv * RA + i);
  }
  const bool side = (int)threadIdx.x < G::NSE;
  int sr, sc;
  side_cols<V, kHalo>(min((int)threadIdx.x, G::NSE - 1), &sr, &sc);
  const int sx = T.x0 - kHalo + sc, sz = zE + sr;
  const int so = side ? col_off(sx, sz, nx, nz, px, 4) : kOOB;
  const fv<V> sm2 = ldpv_at<V>(u2, so), scf = ldpv_at<V>(cf, so);
#pragma unroll
  for (int i = 0; i < RB; ++i) tcf[i] = ldpv<V>(cf, cx, T.z0 + wv * RB + i);
  tile.commit(L1);
  __syncthreads();

  if (act1 && a.d != nullptr) gather<G::NT, G::W1>(a, T, S, L1, T.z0 - 2 * kHalo, T.x0 - 2 * kHalo, k - 1);
  // shot fields used after stores, in registers (see fwd2d_kernel)
  const Source src(S);
  const float q1 = act1 ? a.q[S.q + k - 1] : 0.f, q2 = act2 ? a.q[S.q + k] : 0.f;
  const Damp<V> damp(x, nx, a.nbl);
  // first step: level k on the tile + 4-cell halo (zero outside the grid, where u, u^{k-2} and coef
  // read 0)
  {
    fv<V> lap[RA], u[RA];
    float lmax = 0.f;
    lap_rows<V, RA, G::W1>(&L1[wv * RA + kHalo][2 * kHalo + V * lane], lap, u, a.c);
#pragma unroll
    for (int i = 0; i < RA; ++i) {
      const int r = wv * RA + i, z = zE + r;
      if (act1) src.add<V>(&lap[i], x, z, q1);
      fv<V> incr, v;
      step_cols<V>(u[i], pm2[i], pcf[i], lap[i], damp, border_dist(z, nz, a.nbl), a.eta_dt, &incr, &v);
      // rows of the tile store level k (the others' stores drop)
      const int zo = (unsigned)(r - kHalo) < (unsigned)TZ && z < nz ? z * row4 : kZOOB;
      stv<V>(ro1, v, cx, zo);
      if (SK == kStoreF32) stv<V, kNT>(rs1, v, cx, zo);
      if (SLOT) {
        stv<V>(rslv, v, cs, zo);
        stv<V>(rslu, u[i], cs, zo);
      }
      if (S16) {   // rows of other tiles count too: their points are the level's
        lmax = absmax<V>(lmax, v);
        const int z2 = zo == kZOOB ? kZOOB : zo / 2;
        stv16<V>(rq1, u[i], inv1, SK == kStoreBF16, cx2, z2);
        stv16<V>(rq2, pm2[i], inv2, SK == kStoreBF16, cx2, z2);
      }
      if (PRB && (unsigned)(r - kHalo) < (unsigned)TZ) lds<V>(INC1[r - kHalo][V * lane]) = incr;
      lds<V>(LE[r][kHalo + V * lane]) = v;
    }
    if (S16 && (lmax = wave_max(lmax), lane == 0)) RED[wv] = lmax;
  }
  if (side) {
    fv<V> lap[1], u[1], incr, v;
    lap_rows<V, 1, G::W1>(&L1[sr + kHalo][sc + kHalo], lap, u, a.c);
    if (act1) src.add<V>(&lap[0], sx, sz, q1);
    step_cols<V>(u[0], sm2, scf, lap[0], Damp<V>(sx, nx, a.nbl), border_dist(sz, nz, a.nbl), a.eta_dt, &incr, &v);
    lds<V>(LE[sr][sc]) = v;
  }
  __syncthreads();

  if (S16 && act1 && threadIdx.x == 0) max_to_slot<G::NW>(RED, scl, k);
  if (act2 && a.d != nullptr) gather<G::NT, G::WE>(a, T, S, LE, zE, T.x0 - kHalo, k);
  if (!act2 && !PRB) return;  // probe: level k's increments are still to be added
  // second step: level k+1 on the tile (every lane computes; stores outside the grid drop, as
  // do those of an inactive level k+1)
  double* pb = PRB ? reinterpret_cast<double*>(a.ws + S.store) : nullptr;
  const float* pc1 = PRB ? a.probe_c + k : nullptr;
  const float* pc2 = PRB ? a.probe_c + k + 1 : nullptr;
  fv<V> lap[RB], u[RB];
  float lmax = 0.f;
  lap_rows<V, RB, G::WE>(&LE[wv * RB + kHalo][kHalo + V * lane], lap, u, a.c);
#pragma unroll
  for (int i = 0; i < RB; ++i) {
    const int lr = wv * RB + i, z = T.z0 + lr;
    const fv<V> um2 = lds<V>(L1[lr + 2 * kHalo][2 * kHalo + V * lane]);
    src.add<V>(&lap[i], x, z, q2);
    fv<V> incr, un;
    step_cols<V>(u[i], um2, tcf[i], lap[i], damp, border_dist(z, nz, a.nbl), a.eta_dt, &incr, &un);
    const int zo = z * row4;
    stv<V>(ro2, un, cx, zo);
    if (SK == kStoreF32) stv<V, kNT>(rs2, un, cx, zo);
    if (SLOT) stv<V>(rsl0, un, cs, zo);
    if (S16) lmax = absmax<V>(lmax, un);
    if (PRB && z < nz) {
      // the same two FP64 additions, in the same order, as two one-level launches
      const fv<V> i1 = lds<V>(INC1[lr][V * lane]);
      if (x < nx)
        probe_cols<V>(probe_sums(pb, (long long)z * px + x, a.probe_r), a.probe_r, pc1, i1, act1, pc2, incr, act2,
                   a.probe_pitch);
    }
  }
  if (S16) {
    if (lmax = wave_max(lmax), lane == 0) RED[G::NW + wv] = lmax;
    __syncthreads();
    if (threadIdx.x == 0) max_to_slot<G::NW>(RED + G::NW, scl, k + 1);
  }
}

// ------------------------------------------------------------------------------ T forward steps per launch
// A launch of few tiles is bound by the launch itself (1.8 us) and by the chain of one tile, so small
// forward solves take T levels per launch: level i of the launch is computed on the tile plus 4 (T - i)
// cells, one LDS array per level, each point with the arithmetic of the one-level kernel in the same order
// (so the results are bitwise the same).  Rows of a region split evenly over the eight waves; the columns
// beside the tile go to all threads, a point each.  Three levels beat four: us per level at two, three, four
// levels per launch, without a store, one shot of 281 x 181 2.11, 1.76, 1.75; of 480 x 280 2.39, 2.07, 2.20;
// of 730 x 421 2.66, 2.37, 2.36; two of 730 x 421 3.37, 3.11, 3.22; the added halo takes the rest.
template <int TZ, int T>
struct FM {
  static constexpr int NW = 8, NT = 64 * NW;
  static constexpr int halo(int i) { return kHalo * (T - i); }
  static constexpr int W(int i) { return kTX + 2 * halo(i); }
  static constexpr int H(int i) { return TZ + 2 * halo(i); }
  static constexpr int off(int i) { return i == 0 ? 0 : off(i - 1) + W(i - 1) * H(i - 1); }   // LDS floats below
  static constexpr int rows(int i) { return H(i) / NW; }                                      // of a wave
  static constexpr int cells(int i) { return 2 * halo(i) * H(i); }                            // beside the tile
  static constexpr int per(int i) { return (cells(i) + NT - 1) / NT; }                        // of a thread
  static_assert(TZ % NW == 0 && 2 * kHalo % NW == 0, "rows must split evenly over the waves");
  // row and column of cell e of region i
  static __device__ __forceinline__ void cell(int i, int e, int* r, int* c) {
    const int n = 2 * halo(i);
    *r = e / n;
    const int k = e - *r * n;
    *c = k < halo(i) ? k : kTX + k;
  }
};

// Levels k .. k + T - 1 (k = step - off; levels below 1 are zero), the last of them T m levels below the
// sweep's last.  Only the last two go to the rotating buffers: those of the sweep's last two levels, or the
// other two when m is odd (flip = 2), so that no launch writes a buffer it reads.
// SK = kStoreNone or kStoreF32.
template <int TZ, int T, int SK>
__global__ __launch_bounds__((FM<TZ, T>::NT)) void fwd2dm_kernel(StepArgs a) {
  using G = FM<TZ, T>;
  __shared__ float L[G::off(T)];
  const int tid = xcd_tile(blockIdx.x, a.ntiles);
  const TileDev Tl = a.t.tiles[a.tile_base + tid];
  const ShotDev& S = a.t.shots[Tl.shot];
  const int k = a.step - S.off;
  if (k + T - 1 < 1) return;
  const int nx = S.nx, nz = S.nz, px = S.px;
  const int row4 = 4 * px;
  const int b = S.nt - 1 + a.flip;
  const Planes u1 = planes(fbuf(a.ws, S, fwd_buf(b + 2)), nz, k >= 2 ? nz : 0, row4);
  const Planes u2 = planes(fbuf(a.ws, S, fwd_buf(b + 1)), nz, k >= 3 ? nz : 0, row4);
  const Planes cf = planes(a.ws + S.coef, nz, nz, row4);
  const brsrc ro = make_rsrc(fbuf(a.ws, S, fwd_buf(b)), nz * row4);
  const brsrc rp = make_rsrc(fbuf(a.ws, S, fwd_buf(b - 1)), nz * row4);
  const long long npts = S.npts;
  float* st = reinterpret_cast<float*>(a.ws + S.store);
  const int lane = threadIdx.x & 63, wv = wave_id();
  const int x = Tl.x0 + lane;
  const int cx = x < nx ? 4 * x : kOOB;

  float v0[G::rows(0)], s0[G::per(0)];
#pragma unroll
  for (int n = 0; n < G::rows(0); ++n) v0[n] = ldp(u1, cx, Tl.z0 - G::halo(0) + wv + n * G::NW);
  auto cell_off = [&](int i, int n) {
    int r, c;
    G::cell(i, min((int)threadIdx.x + n * G::NT, G::cells(i) - 1), &r, &c);
    return col_off(Tl.x0 - G::halo(i) + c, Tl.z0 - G::halo(i) + r, nx, nz, px, 4);
  };
#pragma unroll
  for (int n = 0; n < G::per(0); ++n) s0[n] = ldp_at(u1, cell_off(0, n));
  // level k-2 of the first region, and coef of every region
  float um2[G::rows(1)], sm2[G::per(1)], pc[T + 1][G::rows(1)], sc[T + 1][G::per(1)];
#pragma unroll
  for (int n = 0; n < G::rows(1); ++n) um2[n] = ldp(u2, cx, Tl.z0 - G::halo(1) + wv * G::rows(1) + n);
#pragma unroll
  for (int n = 0; n < G::per(1); ++n) sm2[n] = ldp_at(u2, cell_off(1, n));
#pragma unroll
  for (int i = 1; i <= T; ++i) {
#pragma unroll
    for (int n = 0; n < G::rows(i); ++n) pc[i][n] = ldp(cf, cx, Tl.z0 - G::halo(i) + wv * G::rows(i) + n);
#pragma unroll
    for (int n = 0; n < G::per(i); ++n) sc[i][n] = ldp_at(cf, cell_off(i, n));
  }
#pragma unroll
  for (int n = 0; n < G::rows(0); ++n) L[(wv + n * G::NW) * G::W(0) + G::halo(0) + lane] = v0[n];
#pragma unroll
  for (int n = 0; n < G::per(0); ++n) {   // threads past the last cell write it again
    int r, c;
    G::cell(0, min((int)threadIdx.x + n * G::NT, G::cells(0) - 1), &r, &c);
    L[r * G::W(0) + c] = s0[n];
  }
  __syncthreads();

  const Source src(S);
  const Damp<1> damp(x, nx, a.nbl);
  auto level = [&](auto I) __attribute__((always_inline)) {
    constexpr int i = decltype(I)::value, h = G::halo(i), N = G::rows(i), W = G::W(i), W1 = G::W(i - 1);
    constexpr int W2 = i >= 2 ? G::W(i - 2) : 0, o2 = i >= 2 ? G::off(i - 2) : 0;
    const int lv = k + i - 1;
    const bool act = lv >= 1;
    float* L0 = &L[G::off(i - 1)];
    if (act && a.d != nullptr)
      gather<G::NT, W1>(a, Tl, S, reinterpret_cast<const float (*)[W1]>(L0), Tl.z0 - G::halo(i - 1),
                        Tl.x0 - G::halo(i - 1), lv - 1);
    const float q = act ? a.q[S.q + lv - 1] : 0.f;
    const brsrc rs = make_rsrc(st + (long long)(SK == kStoreF32 && act ? lv : 0) * npts,
                               SK == kStoreF32 && act ? nz * row4 : 0);
    fv<1> lap[N], u[N];
    lap_rows<1, N, W1>(L0 + (wv * N + kHalo) * W1 + h + kHalo + lane, lap, u, a.c);
#pragma unroll
    for (int n = 0; n < N; ++n) {
      const int r = wv * N + n, z = Tl.z0 - h + r;
      fv<1> m2, incr, v;
      if constexpr (i == 1) m2[0] = um2[n];
      else m2[0] = L[o2 + (r + 2 * kHalo) * W2 + h + 2 * kHalo + lane];
      if (act) src.add<1>(&lap[n], x, z, q);
      step_cols<1>(u[n], m2, fv<1>{pc[i][n]}, lap[n], damp, border_dist(z, nz, a.nbl), a.eta_dt, &incr, &v);
      if (!act) v[0] = 0.f;
      if constexpr (i < T) L[G::off(i) + r * W + h + lane] = v[0];
      const int zo = (unsigned)(r - h) < (unsigned)TZ && z < nz ? z * row4 : kZOOB;
      if (SK == kStoreF32) stb_nt(rs, v[0], cx, zo);
      if (i == T) stb(ro, v[0], cx, zo);
      if (i == T - 1) stb(rp, v[0], cx, zo);
    }
    if constexpr (i < T) {
#pragma unroll
      for (int n = 0; n < G::per(i); ++n) {
        const int e = (int)threadIdx.x + n * G::NT;
        if (e < G::cells(i)) {
          int r, c;
          G::cell(i, e, &r, &c);
          const int xs = Tl.x0 - h + c, zs = Tl.z0 - h + r;
          fv<1> l1[1], u1c[1], m2, incr, v;
          lap_rows<1, 1, W1>(L0 + (r + kHalo) * W1 + c + kHalo, l1, u1c, a.c);
          if constexpr (i == 1) m2[0] = sm2[n];
          else m2[0] = L[o2 + (r + 2 * kHalo) * W2 + c + 2 * kHalo];
          if (act) src.add<1>(&l1[0], xs, zs, q);
          step_cols<1>(u1c[0], m2, fv<1>{sc[i][n]}, l1[0], Damp<1>(xs, nx, a.nbl), border_dist(zs, nz, a.nbl),
                       a.eta_dt, &incr, &v);
          L[G::off(i) + r * W + c] = act ? v[0] : 0.f;
        }
      }
      __syncthreads();
    }
  };
  level(std::integral_constant<int, 1>{});
  level(std::integral_constant<int, 2>{});
  level(std::integral_constant<int, 3>{});
  static_assert(T == 3, "one call per level");
}

// Residual injected at the points [begin, begin + count) of a tile's list, into LDS at the points'
// tile coordinates.
template <int NT, int W>
__device__ __forceinline__ void inject(const StepArgs& a, const InjPoint* pts, int begin, int count, const float* dd,
                                       float (*L)[W]) {
  for (int t = threadIdx.x; t < count; t += NT) {
    const InjPoint Pt = pts[begin + t];
    float sum = 0.f;
    for (int e = 0; e < Pt.e_count; ++e) {
      const InjEntry E = a.t.inj_ent[Pt.e_begin + e];
      sum += E.w * dd[E.r];
    }
    L[Pt.lz][Pt.lx] = sum;
  }
}

// Adjoint: levels j and j-1 (j = step - off), receiver residual injected in both steps,
// imaging of both steps accumulated (in step order) into one FP64 read-modify-write.
// IMG = kImgNone, kImgFull32, kImgFullBF16, kImgFullFP16, kImgBuffers or kImgProbe (both levels added to the
// probe sums A_j in one FP64 read-modify-write, level j first).  a.single: level j alone.
//
// The injected residual takes no LDS of its own: the first step's lies where the point's new level
// goes (LE), which its own thread reads before it writes; the second step's in L1, of which the
// second step needs only its own points' values, held in registers by then.
template <int TZ, int V, int IMG>
__global__ __launch_bounds__((F2<TZ, V>::NT)) void adj2d2_kernel(StepArgs a) {
  using G = F2<TZ, V>;
  constexpr int RA = G::RA, RB = G::RB;
  // kImgBuffers: the two levels come from the recomputed forward buffers (or the slot restored
  // by reference) instead of the FULL store, as in a checkpointed gradient's paired reversals
  constexpr bool IBUF = IMG == kImgBuffers;
  constexpr bool I16 = IMG == kImgFullBF16 || IMG == kImgFullFP16;
  constexpr bool IACC = IMG == kImgFull32 || I16 || IBUF;
  constexpr bool PRB = IMG == kImgProbe;
  __shared__ __align__(16) float L1[G::H1][G::W1];
  __shared__ __align__(16) float LE[G::HE][G::WE];
  __shared__ __align__(16) float INC1[IACC ? TZ : 1][G::TX];
  const int tid = xcd_tile(blockIdx.x, a.ntiles);
  const TileDev T = a.t.tiles[a.tile_base + tid];
  const ShotDev& S = a.t.shots[T.shot];
  const int j = a.step - S.off;
  const bool act1 = j >= 1 && j <= S.nt - 1;
  const bool act2 = !a.single && j - 1 >= 1 && j - 1 <= S.nt - 1;
  if (!act1 && !act2) return;
  const int nx = S.nx, nz = S.nz, px = S.px;
  const int row4 = 4 * px;
  const Planes w1 = planes(fbuf(a.ws, S, adj_buf(j + 1)), nz, nz, row4);
  const Planes w2 = planes(fbuf(a.ws, S, adj_buf(j + 2)), nz, nz, row4);
  const Planes cf = planes(a.ws + S.coef, nz, nz, row4);
  // new levels j and j-1 (a level of an inactive step gets no records: its stores drop)
  const brsrc ro1 = make_rsrc(fbuf(a.ws, S, adj_buf(j)), act1 ? nz * row4 : 0);
  const brsrc ro2 = make_rsrc(fbuf(a.ws, S, adj_buf(j - 1)), act2 ? nz * row4 : 0);
  // imaging: stored u^j and u^{j-1} (levels of inactive steps read 0) and the FP64 accumulator
  const long long lvl = S.npts * (I16 ? 2 : 4);   // bytes of a stored level
  const unsigned char* ust = a.ws + S.store;
  const bool img1 = IACC && act1, img2 = IACC && act2;
  const Planes us1 = planes(IBUF ? (const void*)fwd_level(a, S, j) : ust + (img1 ? j : 0) * lvl, nz, img1 ? nz : 0,
                            I16 ? row4 / 2 : row4);
  const Planes us2 = planes(IBUF ? (const void*)fwd_level(a, S, j - 1) : ust + (img2 ? j - 1 : 0) * lvl, nz,
                            img2 ? nz : 0, I16 ? row4 / 2 : row4);
  const float* scl = reinterpret_cast<const float*>(a.ws + S.scale);
  const float usc1 = I16 && act1 ? level_scale(scl, j) : 0.f, usc2 = I16 && act2 ? level_scale(scl, j - 1) : 0.f;
  const Planes acc = planes(a.ws + S.acc, nz, IACC ? nz : 0, 2 * row4);
  const brsrc racc = make_rsrc(a.ws + S.acc, IACC ? 2 * nz * row4 : 0);
  const int lane = threadIdx.x & 63, wv = wave_id();
  const int x = T.x0 + V * lane;
  const int cx = x < nx ? 4 * x : kOOB;
  const int cx8 = x < nx ? 8 * x : kOOB;
  const int cx2 = x < nx ? 2 * x : kOOB;
  const int zE = T.z0 - kHalo;
  const bool inj1 = act1 && a.dd != nullptr && T.ext_count > 0;
  const bool inj2 = act2 && a.dd != nullptr && T.inj_count > 0;

  // Imaging inputs: issued with the first step's, or - where the registers they would hold through it
  // cost a workgroup per CU (100 instead of 79 at 24 rows of column pairs) - after it, behind the second
  // step's arithmetic: 16 shots of 1104 x 592 84.9 -> 77.5 us per launch, of 730 x 421 40.1 -> 38.0;
  // narrow or low tiles lose up to 7 % by it.
  constexpr bool LATE = TZ >= (V == 2 ? 16 : 32);
  fv<V> pu1[RB], pu2[RB];
  unsigned ph1[RB], ph2[RB];   // 16-bit codes
  dv<V> pacc[RB];
  auto load_img = [&]() {
#pragma unroll
    for (int i = 0; i < RB; ++i) {
      const int z = T.z0 + wv * RB + i;
      if (I16) {
        ph1[i] = ldpv16<V>(us1, cx2, z);
        ph2[i] = ldpv16<V>(us2, cx2, z);
      } else {
        pu1[i] = ldpv<V, kNT>(us1, cx, z);
        pu2[i] = ldpv<V, kNT>(us2, cx, z);
      }
      pacc[i] = ldpacc<V>(acc, cx8, z);
    }
  };
  Tile8<TZ, V> tile;
  tile.issue(w1, cx, T.x0, T.z0, nx, nz, px);
  fv<V> pm2[RA], pcf[RA], tcf[RB];
#pragma unroll
  for (int i = 0; i < RA; ++i) {
    const int r = wv * RA + i;
    pm2[i] = ldpv<V>(w2, cx, zE + r);
    pcf[i] = ldpv<V>(cf, cx, zE + r);
    if (inj1) lds<V>(LE[r][kHalo + V * lane]) = fv<V>{};
  }
  const bool side = (int)threadIdx.x < G::NSE;
  int sr, sc;
  side_cols<V, kHalo>(min((int)threadIdx.x, G::NSE - 1), &sr, &sc);
  const int sx = T.x0 - kHalo + sc, sz = zE + sr;
  const int so = side ? col_off(sx, sz, nx, nz, px, 4) : kOOB;
  const fv<V> sm2 = ldpv_at<V>(w2, so), scf = ldpv_at<V>(cf, so);
  if (inj1 && side) lds<V>(LE[sr][sc]) = fv<V>{};
#pragma unroll
  for (int i = 0; i < RB; ++i) {
    const int z = T.z0 + wv * RB + i;
    tcf[i] = ldpv<V>(cf, cx, z);
  }
  if (IACC && !LATE) load_img();
  tile.commit(L1);
  __syncthreads();

  if (inj1) {
    inject<G::NT, G::WE>(a, a.t.ext_pts, T.ext_begin, T.ext_count, a.dd + S.d + (long long)j * S.nrec, LE);
    __syncthreads();
  }
  const bool src_here = a.v != nullptr && a.tile_base + tid == S.src_tile && threadIdx.x == 0;
  if (act1 && src_here)
    a.v[S.q + j] = interp_at<G::W1>(L1, S.src_k - T.z0 + 2 * kHalo, S.src_i - T.x0 + 2 * kHalo, S.src_w);
  const Damp<V> damp(x, nx, a.nbl);
  // first step: level j on the tile + 4-cell halo
  {
    fv<V> lap[RA], u[RA];
    lap_rows<V, RA, G::W1>(&L1[wv * RA + kHalo][2 * kHalo + V * lane], lap, u, a.c);
#pragma unroll
    for (int i = 0; i < RA; ++i) {
      const int r = wv * RA + i, z = zE + r;
      fv<V>* le = &lds<V>(LE[r][kHalo + V * lane]);
      if (inj1) {
        const fv<V> s = *le;
        lap[i] += s;
      }
      fv<V> incr, v;
      step_cols<V>(u[i], pm2[i], pcf[i], lap[i], damp, border_dist(z, nz, a.nbl), a.eta_dt, &incr, &v);
      const bool on = (unsigned)(r - kHalo) < (unsigned)TZ;
      stv<V>(ro1, v, cx, on && z < nz ? z * row4 : kZOOB);
      if (IACC && on) lds<V>(INC1[r - kHalo][V * lane]) = incr;
      *le = v;
    }
  }
  if (side) {
    fv<V> lap[1], u[1], incr, v;
    lap_rows<V, 1, G::W1>(&L1[sr + kHalo][sc + kHalo], lap, u, a.c);
    fv<V>* le = &lds<V>(LE[sr][sc]);
    if (inj1) {
      const fv<V> s = *le;
      lap[0] += s;
    }
    step_cols<V>(u[0], sm2, scf, lap[0], Damp<V>(sx, nx, a.nbl), border_dist(sz, nz, a.nbl), a.eta_dt, &incr, &v);
    *le = v;
  }
  if (IACC && LATE) {
    __builtin_amdgcn_sched_barrier(0);
    load_img();
  }
  fv<V> um2[RB];
#pragma unroll
  for (int i = 0; i < RB; ++i)
    um2[i] = lds<V>(L1[wv * RB + i + 2 * kHalo][2 * kHalo + V * lane]);
  __syncthreads();

  if (inj2) {   // the tile's rows of L1 (cell (0, 0) = tile point (0, 0)) now take the second residual
#pragma unroll
    for (int i = 0; i < RB; ++i) lds<V>(L1[wv * RB + i][V * lane]) = fv<V>{};
    __syncthreads();
    inject<G::NT, G::W1>(a, a.t.inj_pts, T.inj_begin, T.inj_count, a.dd + S.d + (long long)(j - 1) * S.nrec, L1);
    __syncthreads();
  }
  if (act2 && src_here) a.v[S.q + j - 1] = interp_at<G::WE>(LE, S.src_k - zE, S.src_i - T.x0 + kHalo, S.src_w);
  // second step: level j-1 on the tile; imaging of both steps (every lane computes; outside
  // the grid the stores drop)
  double* pa = PRB ? reinterpret_cast<double*>(a.ws + S.store) + (long long)a.probe_r * S.npts : nullptr;
  const float* pc1 = PRB ? a.probe_c + j : nullptr;
  const float* pc2 = PRB ? a.probe_c + j - 1 : nullptr;
  if (!act2 && !IACC && !PRB) return;
  fv<V> lap[RB], u[RB];
  lap_rows<V, RB, G::WE>(&LE[wv * RB + kHalo][kHalo + V * lane], lap, u, a.c);
#pragma unroll
  for (int i = 0; i < RB; ++i) {
    const int lr = wv * RB + i, z = T.z0 + lr;
    if (inj2) {
      const fv<V> s = lds<V>(L1[lr][V * lane]);
      lap[i] += s;
    }
    fv<V> incr, wn;
    step_cols<V>(u[i], um2[i], tcf[i], lap[i], damp, border_dist(z, nz, a.nbl), a.eta_dt, &incr, &wn);
    stv<V>(ro2, wn, cx, z * row4);
    if (IACC) {
      const fv<V> i1 = lds<V>(INC1[lr][V * lane]);
      dv<V> ac = pacc[i];
      if (I16) {
        pu1[i] = dec16v<V>(ph1[i], IMG == kImgFullBF16, usc1);
        pu2[i] = dec16v<V>(ph2[i], IMG == kImgFullBF16, usc2);
      }
#pragma unroll
      for (int c = 0; c < V; ++c) {
        if (act1) ac[c] = ac[c] + (double)pu1[i][c] * (double)i1[c];
        if (act2) ac[c] = ac[c] + (double)pu2[i][c] * (double)incr[c];
      }
      stacc<V>(racc, ac, cx8, 2 * z * row4);
    }
    if (PRB && z < nz) {
      // the same two FP64 additions, in the same order, as two one-level launches
      if (x < nx)
        probe_cols<V>(probe_sums(pa, (long long)z * px + x, a.probe_r), a.probe_r, pc1, u[i], act1, pc2, wn, act2,
                   a.probe_pitch);
    }
  }
}

// Born, two levels per launch: u and du at levels k and k+1 (k = step - off), each point with
// the arithmetic of born2d_kernel in the same order (so the results are bitwise those of two
// one-level launches); samples (J dm)^{k-1} and (J dm)^k.  Per two levels the launch reads
// u^{k-1}, u^{k-2}, du^{k-1}, du^{k-2}, coef and dm once and writes four levels: 40 B per point
// instead of 2 x 32.  a.single: level k alone.  Column pairs would cost this kernel, which holds two
// fields, more in occupancy than they save: 43.1 us per launch instead of 39.5 (16 shots of 730 x 421).
template <int TZ>
__global__ __launch_bounds__((F2<TZ, 1>::NT)) void born2d2_kernel(StepArgs a) {
  constexpr int V = 1;
  using G = F2<TZ, V>;
  constexpr int RA = G::RA, RB = G::RB;
  __shared__ __align__(16) float L1U[G::H1][G::W1];
  __shared__ __align__(16) float L1D[G::H1][G::W1];
  __shared__ __align__(16) float LEU[G::HE][G::WE];
  __shared__ __align__(16) float LED[G::HE][G::WE];
  const int tid = xcd_tile(blockIdx.x, a.ntiles);
  const TileDev T = a.t.tiles[a.tile_base + tid];
  const ShotDev& S = a.t.shots[T.shot];
  const int k = a.step - S.off;
  const bool act1 = k >= 1 && k <= S.nt - 1;
  const bool act2 = !a.single && k + 1 >= 1 && k + 1 <= S.nt - 1;
  if (!act1 && !act2) return;
  const int nx = S.nx, nz = S.nz, px = S.px;
  const int row4 = 4 * px;
  // levels below 1 are zero
  const Planes u1 = planes(fbuf(a.ws, S, fwd_buf(k - 1)), nz, k >= 2 ? nz : 0, row4);
  const Planes u2 = planes(fbuf(a.ws, S, fwd_buf(k - 2)), nz, k >= 3 ? nz : 0, row4);
  const Planes d1 = planes(fbuf(a.ws, S, adj_buf(k - 1)), nz, k >= 2 ? nz : 0, row4);
  const Planes d2 = planes(fbuf(a.ws, S, adj_buf(k - 2)), nz, k >= 3 ? nz : 0, row4);
  const Planes cf = planes(a.ws + S.coef, nz, nz, row4);
  const Planes dmp = planes(a.dm + S.m, nz, nz, 4LL * nx);   // caller's layout: rows of nx
  // new levels k and k+1 (a level outside 1..nt-1 belongs to an inactive step: no records)
  const brsrc uo1 = make_rsrc(fbuf(a.ws, S, fwd_buf(k)), act1 ? nz * row4 : 0);
  const brsrc uo2 = make_rsrc(fbuf(a.ws, S, fwd_buf(k + 1)), act2 ? nz * row4 : 0);
  const brsrc do1 = make_rsrc(fbuf(a.ws, S, adj_buf(k)), act1 ? nz * row4 : 0);
  const brsrc do2 = make_rsrc(fbuf(a.ws, S, adj_buf(k + 1)), act2 ? nz * row4 : 0);
  const int lane = threadIdx.x & 63, wv = wave_id();
  const int x = T.x0 + V * lane;
  const int cx = x < nx ? 4 * x : kOOB;
  const int zE = T.z0 - kHalo;

  // the two level k-1 tiles first, then the first step's other inputs on its points and coef and
  // dm of the tile points
  Tile8<TZ, V> tu, td;
  tu.issue(u1, cx, T.x0, T.z0, nx, nz, px);
  td.issue(d1, cx, T.x0, T.z0, nx, nz, px);
  fv<V> pu2[RA], pd2[RA], pcf[RA], pdm[RA], tcf[RB], tdm[RB];
#pragma unroll
  for (int i = 0; i < RA; ++i) {
    const int z = zE + wv * RA + i;
    pu2[i] = ldpv<V>(u2, cx, z);
    pd2[i] = ldpv<V>(d2, cx, z);
    pcf[i] = ldpv<V>(cf, cx, z);
    #pragma unroll
    for (int c = 0; c < V; ++c) pdm[i][c] = ldp(dmp, x + c < nx ? 4 * (x + c) : kOOB, z);   // rows of nx
  }
  const bool side = (int)threadIdx.x < G::NSE;
  int sr, sc;
  side_cols<V, kHalo>(min((int)threadIdx.x, G::NSE - 1), &sr, &sc);
  const int sx = T.x0 - kHalo + sc, sz = zE + sr;
  const int so = side ? col_off(sx, sz, nx, nz, px, 4) : kOOB;
  const fv<V> su2 = ldpv_at<V>(u2, so), sd2 = ldpv_at<V>(d2, so), scf = ldpv_at<V>(cf, so);
  fv<V> sdm;
#pragma unroll
  for (int c = 0; c < V; ++c) sdm[c] = ldp_at(dmp, side ? col_off(sx + c, sz, nx, nz, nx, 4) : kOOB);
#pragma unroll
  for (int i = 0; i < RB; ++i) {
    const int z = T.z0 + wv * RB + i;
    tcf[i] = ldpv<V>(cf, cx, z);
    #pragma unroll
    for (int c = 0; c < V; ++c) tdm[i][c] = ldp(dmp, x + c < nx ? 4 * (x + c) : kOOB, z);
  }
  tu.commit(L1U);
  td.commit(L1D);
  __syncthreads();

  if (act1 && a.d != nullptr) gather<G::NT, G::W1>(a, T, S, L1D, T.z0 - 2 * kHalo, T.x0 - 2 * kHalo, k - 1);
  const Source src(S);   // in registers (see the forward kernel)
  const float q1 = act1 ? a.q[S.q + k - 1] : 0.f, q2 = act2 ? a.q[S.q + k] : 0.f;
  const Damp<V> damp(x, nx, a.nbl);
  // scattered field's source: -dm (u^k - 2u^{k-1} + u^{k-2}) / dt^2 = -dm incr / dt^2
  auto scatter = [&](fv<V>* lapd, fv<V> dm, fv<V> incr) {
#pragma unroll
    for (int i = 0; i < V; ++i) (*lapd)[i] = (*lapd)[i] - dm[i] * incr[i] * a.inv_dt2;
  };
  // first step: levels k of u and du on the tile + 4-cell halo
  {
    fv<V> lap[RA], u[RA], inc[RA];
    lap_rows<V, RA, G::W1>(&L1U[wv * RA + kHalo][2 * kHalo + V * lane], lap, u, a.c);
#pragma unroll
    for (int i = 0; i < RA; ++i) {
      const int r = wv * RA + i, z = zE + r;
      if (act1) src.add<V>(&lap[i], x, z, q1);
      fv<V> v;
      step_cols<V>(u[i], pu2[i], pcf[i], lap[i], damp, border_dist(z, nz, a.nbl), a.eta_dt, &inc[i], &v);
      stv<V>(uo1, v, cx, (unsigned)(r - kHalo) < (unsigned)TZ && z < nz ? z * row4 : kZOOB);
      lds<V>(LEU[r][kHalo + V * lane]) = v;
    }
    lap_rows<V, RA, G::W1>(&L1D[wv * RA + kHalo][2 * kHalo + V * lane], lap, u, a.c);
#pragma unroll
    for (int i = 0; i < RA; ++i) {
      const int r = wv * RA + i, z = zE + r;
      scatter(&lap[i], pdm[i], inc[i]);
      fv<V> incd, v;
      step_cols<V>(u[i], pd2[i], pcf[i], lap[i], damp, border_dist(z, nz, a.nbl), a.eta_dt, &incd, &v);
      stv<V>(do1, v, cx, (unsigned)(r - kHalo) < (unsigned)TZ && z < nz ? z * row4 : kZOOB);
      lds<V>(LED[r][kHalo + V * lane]) = v;
    }
  }
  if (side) {
    const Damp<V> sdamp(sx, nx, a.nbl);
    const int dz = border_dist(sz, nz, a.nbl);
    fv<V> lap[1], u[1], incr, incd, v;
    lap_rows<V, 1, G::W1>(&L1U[sr + kHalo][sc + kHalo], lap, u, a.c);
    if (act1) src.add<V>(&lap[0], sx, sz, q1);
    step_cols<V>(u[0], su2, scf, lap[0], sdamp, dz, a.eta_dt, &incr, &v);
    lds<V>(LEU[sr][sc]) = v;
    lap_rows<V, 1, G::W1>(&L1D[sr + kHalo][sc + kHalo], lap, u, a.c);
    scatter(&lap[0], sdm, incr);
    step_cols<V>(u[0], sd2, scf, lap[0], sdamp, dz, a.eta_dt, &incd, &v);
    lds<V>(LED[sr][sc]) = v;
  }
  __syncthreads();

  if (act2 && a.d != nullptr) gather<G::NT, G::WE>(a, T, S, LED, zE, T.x0 - kHalo, k);
  if (!act2) return;
  // second step: levels k+1 on the tile (every lane computes; stores outside the grid drop)
  fv<V> lap[RB], u[RB], inc[RB];
  lap_rows<V, RB, G::WE>(&LEU[wv * RB + kHalo][kHalo + V * lane], lap, u, a.c);
#pragma unroll
  for (int i = 0; i < RB; ++i) {
    const int lr = wv * RB + i, z = T.z0 + lr;
    const fv<V> um2 = lds<V>(L1U[lr + 2 * kHalo][2 * kHalo + V * lane]);
    src.add<V>(&lap[i], x, z, q2);
    fv<V> v;
    step_cols<V>(u[i], um2, tcf[i], lap[i], damp, border_dist(z, nz, a.nbl), a.eta_dt, &inc[i], &v);
    stv<V>(uo2, v, cx, z * row4);
  }
  lap_rows<V, RB, G::WE>(&LED[wv * RB + kHalo][kHalo + V * lane], lap, u, a.c);
#pragma unroll
  for (int i = 0; i < RB; ++i) {
    const int lr = wv * RB + i, z = T.z0 + lr;
    const fv<V> dm2 = lds<V>(L1D[lr + 2 * kHalo][2 * kHalo + V * lane]);
    scatter(&lap[i], tdm[i], inc[i]);
    fv<V> incd, v;
    step_cols<V>(u[i], dm2, tcf[i], lap[i], damp, border_dist(z, nz, a.nbl), a.eta_dt, &incd, &v);
    stv<V>(do2, v, cx, z * row4);
  }
}

template <int TZ>
hipError_t fwd2d_tz(const StepArgs& a, int store, hipStream_t s) {
  switch (store) {
    case kStoreNone: fwd2d_kernel<TZ, kStoreNone><<<a.ntiles, T2<TZ>::NT, 0, s>>>(a); break;
    case kStoreF32: fwd2d_kernel<TZ, kStoreF32><<<a.ntiles, T2<TZ>::NT, 0, s>>>(a); break;
    case kStoreF32R: fwd2d_kernel<TZ, kStoreF32R><<<a.ntiles, T2<TZ>::NT, 0, s>>>(a); break;
    case kStoreBF16: fwd2d_kernel<TZ, kStoreBF16><<<a.ntiles, T2<TZ>::NT, 0, s>>>(a); break;
    case kStoreFP16: fwd2d_kernel<TZ, kStoreFP16><<<a.ntiles, T2<TZ>::NT, 0, s>>>(a); break;
    case kStoreProbe: fwd2d_kernel<TZ, kStoreProbe><<<a.ntiles, T2<TZ>::NT, 0, s>>>(a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int TZ>
hipError_t adj2d_tz(const StepArgs& a, hipStream_t s) {
  switch (a.image_src) {
    case kImgNone: adj2d_kernel<TZ, kImgNone><<<a.ntiles, T2<TZ>::NT, 0, s>>>(a); break;
    case kImgFull32: adj2d_kernel<TZ, kImgFull32><<<a.ntiles, T2<TZ>::NT, 0, s>>>(a); break;
    case kImgBuffers: adj2d_kernel<TZ, kImgBuffers><<<a.ntiles, T2<TZ>::NT, 0, s>>>(a); break;
    case kImgFullBF16: adj2d_kernel<TZ, kImgFullBF16><<<a.ntiles, T2<TZ>::NT, 0, s>>>(a); break;
    case kImgFullFP16: adj2d_kernel<TZ, kImgFullFP16><<<a.ntiles, T2<TZ>::NT, 0, s>>>(a); break;
    case kImgProbe: adj2d_kernel<TZ, kImgProbe><<<a.ntiles, T2<TZ>::NT, 0, s>>>(a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int TZ, int V>
hipError_t fwd2d2_tz(const StepArgs& a, int store, hipStream_t s) {
  switch (store) {
    case kStoreSlot: fwd2d2_kernel<TZ, V, kStoreSlot><<<a.ntiles, F2<TZ, V>::NT, 0, s>>>(a); break;
    case kStoreNone: fwd2d2_kernel<TZ, V, kStoreNone><<<a.ntiles, F2<TZ, V>::NT, 0, s>>>(a); break;
    case kStoreF32: fwd2d2_kernel<TZ, V, kStoreF32><<<a.ntiles, F2<TZ, V>::NT, 0, s>>>(a); break;
    case kStoreBF16: fwd2d2_kernel<TZ, V, kStoreBF16><<<a.ntiles, F2<TZ, V>::NT, 0, s>>>(a); break;
    case kStoreFP16: fwd2d2_kernel<TZ, V, kStoreFP16><<<a.ntiles, F2<TZ, V>::NT, 0, s>>>(a); break;
    case kStoreProbe: fwd2d2_kernel<TZ, V, kStoreProbe><<<a.ntiles, F2<TZ, V>::NT, 0, s>>>(a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int TZ, int V>
hipError_t adj2d2_tz(const StepArgs& a, hipStream_t s) {
  switch (a.image_src) {
    case kImgNone: adj2d2_kernel<TZ, V, kImgNone><<<a.ntiles, F2<TZ, V>::NT, 0, s>>>(a); break;
    case kImgFull32: adj2d2_kernel<TZ, V, kImgFull32><<<a.ntiles, F2<TZ, V>::NT, 0, s>>>(a); break;
    case kImgFullBF16: adj2d2_kernel<TZ, V, kImgFullBF16><<<a.ntiles, F2<TZ, V>::NT, 0, s>>>(a); break;
    case kImgFullFP16: adj2d2_kernel<TZ, V, kImgFullFP16><<<a.ntiles, F2<TZ, V>::NT, 0, s>>>(a); break;
    case kImgBuffers: adj2d2_kernel<TZ, V, kImgBuffers><<<a.ntiles, F2<TZ, V>::NT, 0, s>>>(a); break;
    case kImgProbe: adj2d2_kernel<TZ, V, kImgProbe><<<a.ntiles, F2<TZ, V>::NT, 0, s>>>(a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace

namespace {
template <int V>
hipError_t fwd2d2_v(const StepArgs& a, int tz, int store, hipStream_t s) {
  switch (tz) {
    case 8: return fwd2d2_tz<8, V>(a, store, s);
    case 16: return fwd2d2_tz<16, V>(a, store, s);
    case 24: return fwd2d2_tz<24, V>(a, store, s);
    case 32: return fwd2d2_tz<32, V>(a, store, s);
  }
  return hipErrorInvalidValue;
}

template <int V>
hipError_t adj2d2_v(const StepArgs& a, int tz, hipStream_t s) {
  switch (tz) {
    case 8: return adj2d2_tz<8, V>(a, s);
    case 16: return adj2d2_tz<16, V>(a, s);
    case 24: return adj2d2_tz<24, V>(a, s);
    case 32: return adj2d2_tz<32, V>(a, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_fwd2d2(const StepArgs& a, int tx, int tz, int store, hipStream_t s) {
  if (a.ntiles <= 0) return hipSuccess;
  return tx == 64 ? fwd2d2_v<1>(a, tz, store, s) : tx == 128 ? fwd2d2_v<2>(a, tz, store, s) : hipErrorInvalidValue;
}

hipError_t launch_fwd2dm(const StepArgs& a, int tz, int store, hipStream_t s) {
  if (a.ntiles <= 0) return hipSuccess;
  auto go = [&](auto TZ) -> hipError_t {
    constexpr int tz = decltype(TZ)::value;
    if (store == kStoreNone) fwd2dm_kernel<tz, kManyLevels, kStoreNone><<<a.ntiles, FM<tz, kManyLevels>::NT, 0, s>>>(a);
    else if (store == kStoreF32) fwd2dm_kernel<tz, kManyLevels, kStoreF32><<<a.ntiles, FM<tz, kManyLevels>::NT, 0, s>>>(a);
    else return hipErrorInvalidValue;
    return hipGetLastError();
  };
  switch (tz) {
    case 8: return go(std::integral_constant<int, 8>{});
    case 16: return go(std::integral_constant<int, 16>{});
    case 24: return go(std::integral_constant<int, 24>{});
  }
  return hipErrorInvalidValue;
}

hipError_t launch_adj2d2(const StepArgs& a, int tx, int tz, hipStream_t s) {
  if (a.ntiles <= 0) return hipSuccess;
  return tx == 64 ? adj2d2_v<1>(a, tz, s) : tx == 128 ? adj2d2_v<2>(a, tz, s) : hipErrorInvalidValue;
}

hipError_t launch_born2d2(const StepArgs& a, int tz, hipStream_t s) {
  if (a.ntiles <= 0) return hipSuccess;
  switch (tz) {
    case 8: born2d2_kernel<8><<<a.ntiles, F2<8, 1>::NT, 0, s>>>(a); break;
    case 16: born2d2_kernel<16><<<a.ntiles, F2<16, 1>::NT, 0, s>>>(a); break;
    case 24: born2d2_kernel<24><<<a.ntiles, F2<24, 1>::NT, 0, s>>>(a); break;
    case 32: born2d2_kernel<32><<<a.ntiles, F2<32, 1>::NT, 0, s>>>(a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_fwd2d(const StepArgs& a, int tz, int store, hipStream_t s) {
  if (a.ntiles <= 0) return hipSuccess;
  switch (tz) {
    case 8: return fwd2d_tz<8>(a, store, s);
    case 12: return fwd2d_tz<12>(a, store, s);
    case 16: return fwd2d_tz<16>(a, store, s);
    case 20: return fwd2d_tz<20>(a, store, s);
    case 24: return fwd2d_tz<24>(a, store, s);
    case 32: return fwd2d_tz<32>(a, store, s);
    case 64: return fwd2d_tz<64>(a, store, s);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_adj2d(const StepArgs& a, int tz, hipStream_t s) {
  if (a.ntiles <= 0) return hipSuccess;
  switch (tz) {
    case 8: return adj2d_tz<8>(a, s);
    case 12: return adj2d_tz<12>(a, s);
    case 16: return adj2d_tz<16>(a, s);
    case 20: return adj2d_tz<20>(a, s);
    case 24: return adj2d_tz<24>(a, s);
    case 32: return adj2d_tz<32>(a, s);
    case 64: return adj2d_tz<64>(a, s);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_born2d(const StepArgs& a, int tz, hipStream_t s) {
  if (a.ntiles <= 0) return hipSuccess;
  switch (tz) {
    case 8: born2d_kernel<8><<<a.ntiles, T2<8>::NT, 0, s>>>(a); break;
    case 12: born2d_kernel<12><<<a.ntiles, T2<12>::NT, 0, s>>>(a); break;
    case 16: born2d_kernel<16><<<a.ntiles, T2<16>::NT, 0, s>>>(a); break;
    case 20: born2d_kernel<20><<<a.ntiles, T2<20>::NT, 0, s>>>(a); break;
    case 24: born2d_kernel<24><<<a.ntiles, T2<24>::NT, 0, s>>>(a); break;
    case 32: born2d_kernel<32><<<a.ntiles, T2<32>::NT, 0, s>>>(a); break;
    case 64: born2d_kernel<64><<<a.ntiles, T2<64>::NT, 0, s>>>(a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace awe
