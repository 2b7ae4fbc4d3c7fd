// nh_brick.hpp -- implicit-Euler steps of grids that fit the chip with few cells
// per thread: the whole state of the single-reduction CG iteration of
// nh_kernels.hpp -- x, p, u = r/D, w/D = A u / D, s/D = A p / D -- and the
// operator -- the six face weights, D and 1/D of every cell -- stay in the
// registers of the workgroup that owns the cell, for FP32 and FP64, any lateral
// closure and the Robin face. A launch runs several consecutive steps.
//
// A workgroup of NT threads owns a brick of TX x TY columns (TX TY = NT) of at
// most ZC cells, one column per thread. An iteration is: the elementwise
// updates in registers; the new u of the brick and of its halo ring into LDS;
// one workgroup barrier; the stencil, 1/D and the three FP64 sums; w/D on the
// brick's faces to memory; the team reduction.
//
// On these grids an iteration is bound by the latency of that exchange and not
// by work or traffic, so everything else is kept out of the loop, and the
// exchange is one store and one load deep:
//  - w/D is the only vector exchanged. A workgroup keeps u, s, p and x of its
//    halo cells too and advances them by the same fused operations as their
//    owner, so it holds the same bits; at the end of a step it knows its halo of
//    the new state, and the next step and the gradient need no exchange for it.
//  - Halo values travel as words that carry the reduction's tag (value or half
//    of it | tag << 32), so a store need not complete before the workgroup's sum
//    is published, and halo values and slots are polled together. Banks
//    alternate with the reduction's epoch: a bank is rewritten two reductions
//    later, which a workgroup reaches only after every reader has published the
//    one in between, computed from what it read.
// A brick that holds the whole grid has no exchange at all, only two workgroup
// barriers per iteration. (The streaming kernel marches a tile plane by plane
// through memory and recomputes the weights, seven divisions per cell and
// iteration.)
//
// The arithmetic is that of the streaming and resident kernels (diag_w, apply_w,
// the same fused updates, FP64 sums), so FP32 results are the same bits.
#pragma once

#include "nh_kernels.hpp"

namespace nh {

constexpr int kBrickSteps = 12;             // steps per launch (their fields travel as kernel arguments)

// The steps of a launch. Where a step's adaptive initial guess compares the
// iteration counts of probe steps, bit d of here says that the probe of order d
// is an earlier step of this launch (else its count is read from gi).
template <typename R>
struct BrickSteps {
  StepVar<R> v[kBrickSteps];
  unsigned char here[kBrickSteps];
  int count;
};

// Buffer access to one vector of n elements: a lane's byte offset (kOffLane:
// reads 0, writes nothing) plus a uniform offset, so that no per-lane 64-bit
// addresses are kept through the solve (a launch's vectors stay below 2^31 bytes).
template <typename R>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t brick_rsrc(const R* p, long long n) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<R*>(p), 0, p ? (int)(n * (long long)sizeof(R)) : 0, 0x00020000);
}
template <int CPOL, typename R>
__device__ __forceinline__ R brick_ld(__amdgpu_buffer_rsrc_t r, unsigned voff, int soff) {
  if constexpr (sizeof(R) == 4) {
    return (R)__uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, CPOL));
  } else {
    const auto v = __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, CPOL);
    return (R)__hiloint2double((int)v[1], (int)v[0]);
  }
}
template <int CPOL, typename R>
__device__ __forceinline__ void brick_st(__amdgpu_buffer_rsrc_t r, unsigned voff, int soff, R v) {
  if constexpr (sizeof(R) == 4) {
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint((float)v), r, voff, soff, CPOL);
  } else {
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    const u2 w = {(unsigned)__double2loint((double)v), (unsigned)__double2hiint((double)v)};
    __builtin_amdgcn_raw_buffer_store_b64(w, r, voff, soff, CPOL);
  }
}

// Tagged halo words, 2 sizeof(R) bytes per cell: FP32 (value, tag); FP64 (low
// half, tag, high half, tag), each 8-byte word valid by itself.
template <typename R>
__device__ __forceinline__ void halo_st(__amdgpu_buffer_rsrc_t r, unsigned voff, int soff, R v, unsigned tag) {
  if constexpr (sizeof(R) == 4) {
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    __builtin_amdgcn_raw_buffer_store_b64(u2{__float_as_uint((float)v), tag}, r, voff, soff, kCpolSc1);
  } else {
    typedef unsigned u4 __attribute__((ext_vector_type(4)));
    __builtin_amdgcn_raw_buffer_store_b128(
        u4{(unsigned)__double2loint((double)v), tag, (unsigned)__double2hiint((double)v), tag}, r, voff, soff, kCpolSc1);
  }
}
template <typename R>
__device__ __forceinline__ bool halo_ld(__amdgpu_buffer_rsrc_t r, unsigned voff, int soff, R& v, unsigned tag) {
  if constexpr (sizeof(R) == 4) {
    const auto x = __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, kCpolSc1);
    v = (R)__uint_as_float(x[0]);
    return x[1] == tag;
  } else {
    const auto x = __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, kCpolSc1);
    v = (R)__hiloint2double((int)x[2], (int)x[0]);
    return (x[1] == tag) & (x[3] == tag);
  }
}

template <typename F>
struct BrickHalo {
  static constexpr bool kAny = true;
  F poll_f;
  template <int NV> __device__ bool poll(__amdgpu_buffer_rsrc_t, unsigned tag) const { return poll_f(tag); }
  __device__ void ready() const {}
};

template <typename R, int ZC, int NT>
__global__ void __launch_bounds__(NT, 1) brick_steps_kernel(StepArgs<R> S, BrickSteps<R> tab) {
  constexpr int PLX = NT == 512 ? 660 : 396;               // max (TX+2)*(TY+2), TX 16, 32 or 64
  constexpr int RG = NT == 512 ? 144 : 136;                // max 2*(TX+TY)
  constexpr int KR = (RG * ZC + NT - 1) / NT;              // halo ring cells per thread
  constexpr unsigned SZ = sizeof(R);
  __shared__ R lu[ZC * PLX];
  __shared__ RedBuf rb;
  const Geom& g = S.g;
  const int tid = threadIdx.x, rank = blockIdx.x;
  const Tile T = tile_of(g, rank);
  const int PW = g.TX + 2, PL = PW * (g.TY + 2);
  const int tx = tid & (g.TX - 1), ty = tid >> g.txs;
  const int cx = min(g.TX, g.nx - T.x0), cy = min(g.TY, g.ny - T.y0), tzn = T.z1 - T.z0;
  const bool own = tx < cx && ty < cy;
  const int gx = T.x0 + tx, gy = T.y0 + ty;
  const int nxy = (int)g.nxy;
  const int oslot = (ty + 1) * PW + tx + 1;
  const R sx = S.sx, sy = S.sy, sz = S.sz;
  // byte offsets: of this thread's column in plane 0, and of plane z of the brick
  const unsigned vo = own ? SZ * (unsigned)(gx + g.nx * gy) : kOffLane;
  auto po = [&](int z) { return (T.z0 + z) * nxy * (int)SZ; };

  // a tile of another workgroup lies across this side (a side that wraps onto
  // the brick itself is served by its own threads' second LDS store)
  const bool per = g.periodic != 0;
  const bool rxm = T.x0 > 0 || (per && g.ntx > 1), rxp = T.x0 + cx < g.nx || (per && g.ntx > 1);
  const bool rym = T.y0 > 0 || (per && g.nty > 1), ryp = T.y0 + cy < g.ny || (per && g.nty > 1);
  const bool rzm = T.z0 > 0, rzp = T.z1 < g.nz;
  // faces to publish: the lateral edges' columns on every plane, all columns on
  // the first and last plane where a brick lies below or above
  const bool edge = own && ((tx == 0 && rxm) || (tx == cx - 1 && rxp) || (ty == 0 && rym) || (ty == cy - 1 && ryp));
  const unsigned vt = own ? 2 * vo : kOffLane;             // (tagged words are twice as wide)
  const unsigned ve = edge ? vt : kOffLane, vlo = rzm ? vt : ve, vhi = rzp ? vt : ve;
  const unsigned vtop = tzn == 1 && rzm ? vlo : vhi;
  auto vpub = [&](int z) -> unsigned {
    return z + 1 == tzn ? vtop : (z == 0 ? vlo : (z < tzn ? ve : kOffLane));
  };
  int wslx = oslot, wsly = oslot;           // the wrapped copies of this column's cell in LDS
  if (own && per && g.ntx == 1) {
    if (gx == 0) wslx = (ty + 1) * PW + cx + 1;
    if (gx == g.nx - 1) wslx = (ty + 1) * PW;
  }
  if (own && per && g.nty == 1) {
    if (gy == 0) wsly = (cy + 1) * PW + tx + 1;
    if (gy == g.ny - 1) wsly = tx + 1;
  }
  const bool wraps = per && (g.ntx == 1 || g.nty == 1);

  // the halo ring cells this thread loads: byte offset of the tagged word and LDS slot (-1: none)
  unsigned rg[KR];
  int rl[KR];
  {
    const int pr = 2 * (cx + cy);
#pragma unroll
    for (int k = 0; k < KR; ++k) {
      const int e = tid + k * NT;
      rg[k] = kOffLane;
      rl[k] = -1;
      if (e >= pr * tzn) continue;
      const int z = e / pr;
      int h = e - z * pr, hx, hy, slot;
      bool in;
      if (h < cx) { in = rym; hx = T.x0 + h; hy = T.y0 > 0 ? T.y0 - 1 : g.ny - 1; slot = h + 1; }
      else if ((h -= cx) < cx) { in = ryp; hx = T.x0 + h; hy = T.y0 + cy < g.ny ? T.y0 + cy : 0; slot = (cy + 1) * PW + h + 1; }
      else if ((h -= cx) < cy) { in = rxm; hx = T.x0 > 0 ? T.x0 - 1 : g.nx - 1; hy = T.y0 + h; slot = (h + 1) * PW; }
      else { h -= cy; in = rxp; hx = T.x0 + cx < g.nx ? T.x0 + cx : 0; hy = T.y0 + h; slot = (h + 1) * PW + cx + 1; }
      if (in) {
        rg[k] = 2 * SZ * (unsigned)(hx + g.nx * hy + (T.z0 + z) * nxy);
        rl[k] = z * PL + slot;
      }
    }
  }
  // LDS slots that no cell fills stay zero (beyond a wall: weight 0 times a finite difference)
  for (int e = tid; e < ZC * PL; e += NT) lu[e] = R(0);

  // the operator: face weights, D and 1/D (a cell that is absent reads alpha = 0: weights 0, D = 1)
  const __amdgpu_buffer_rsrc_t ra = brick_rsrc(S.alpha, g.ng);
  const int dxm = gx > 0 ? -1 : g.nx - 1, dxp = gx + 1 < g.nx ? 1 : 1 - g.nx;
  const int dym = gy > 0 ? -g.nx : g.nx * (g.ny - 1), dyp = gy + 1 < g.ny ? g.nx : g.nx * (1 - g.ny);
  const unsigned vxm = own && (gx > 0 || per) ? vo + SZ * (unsigned)dxm : kOffLane;
  const unsigned vxp = own && (gx + 1 < g.nx || per) ? vo + SZ * (unsigned)dxp : kOffLane;
  const unsigned vym = own && (gy > 0 || per) ? vo + SZ * (unsigned)dym : kOffLane;
  const unsigned vyp = own && (gy + 1 < g.ny || per) ? vo + SZ * (unsigned)dyp : kOffLane;
  auto ia_at = [&](bool in, unsigned v, int z) -> R {
    return inv_alpha<R>(in ? brick_ld<0, R>(ra, v, po(z)) : R(0));
  };
  R wxm[ZC], wxp[ZC], wym[ZC], wyp[ZC], wz[ZC + 1], D[ZC], rD[ZC];
  {
    R ic = ia_at(true, vo, 0);
    wz[0] = face_w<R>(ic, ia_at(rzm, vo, -1));
#pragma unroll
    for (int z = 0; z < ZC; ++z) {
      const bool in = z < tzn;
      wxm[z] = face_w<R>(ic, ia_at(in, vxm, z));
      wxp[z] = face_w<R>(ic, ia_at(in, vxp, z));
      wym[z] = face_w<R>(ic, ia_at(in, vym, z));
      wyp[z] = face_w<R>(ic, ia_at(in, vyp, z));
      const R iz = ia_at(in && T.z0 + z + 1 < g.nz, vo, z + 1);
      wz[z + 1] = face_w<R>(ic, iz);
      ic = z + 1 < tzn ? iz : inv_alpha<R>(R(0));
      const R w[6] = {wxm[z], wxp[z], wym[z], wyp[z], z < tzn ? wz[z] : R(0), wz[z + 1]};
      D[z] = diag_w<R>(sx, sy, sz, w);
      if (T.z0 + z == g.nz - 1 && S.sb != R(0)) D[z] = add_rn(D[z], S.sb);
      rD[z] = rcp<R>(D[z]);
    }
  }

  R x[ZC], p[ZC], u[ZC], wr[ZC], s[ZC];
  // the same of the halo: ring cells [0, KR), then the cells below and above the brick
  constexpr int KH = KR + 2;
  R hx[KH], hp[KH], hu[KH], hw[KH], hs[KH];
#pragma unroll
  for (int k = 0; k < KH; ++k) hx[k] = hp[k] = hu[k] = hw[k] = hs[k] = R(0);
  auto put = [&](const R (&v)[ZC]) {
    if (own) {
#pragma unroll
      for (int z = 0; z < ZC; ++z) {
        lu[z * PL + oslot] = v[z];
        if (wraps) {
          lu[z * PL + wslx] = v[z];
          lu[z * PL + wsly] = v[z];
        }
      }
    }
  };
  // values of a state on the halo (complete since an earlier launch or step; 0 where there is no cell)
  auto ld_halo = [&](const R* q, R (&h)[KH]) {
    const __amdgpu_buffer_rsrc_t r = brick_rsrc(q, g.ng);
#pragma unroll
    for (int k = 0; k < KR; ++k) h[k] = brick_ld<kCpolSc1, R>(r, rg[k] / 2, 0);
    h[KR] = rzm ? brick_ld<kCpolSc1, R>(r, vo, po(-1)) : R(0);
    h[KR + 1] = rzp ? brick_ld<kCpolSc1, R>(r, vo, po(tzn)) : R(0);
  };
  // tagged halo values of bank b (0, 1: w/D by epoch parity; 2: u0); true once this lane has all of its own
  auto bank_of = [&](int b) {
    return __builtin_amdgcn_make_buffer_rsrc((char*)S.halo + (size_t)b * (2 * SZ) * (size_t)g.ng, 0,
                                             (int)(2 * SZ * g.ng), 0x00020000);
  };
  auto ld_tagged = [&](int b, unsigned tag, R (&h)[KH]) -> bool {
    const __amdgpu_buffer_rsrc_t r = bank_of(b);
    bool all = true;                        // (no branches: one round trip)
#pragma unroll
    for (int k = 0; k < KR; ++k) {
      const bool got = halo_ld<R>(r, rg[k], 0, h[k], tag);
      all &= got | (rl[k] < 0);
    }
    const bool gm = halo_ld<R>(r, rzm ? vt : kOffLane, rzm ? 2 * po(-1) : 0, h[KR], tag);
    const bool gp = halo_ld<R>(r, rzp ? vt : kOffLane, rzp ? 2 * po(tzn) : 0, h[KR + 1], tag);
    all &= (gm | !rzm | !own) & (gp | !rzp | !own);
    return all;
  };
  auto put_halo = [&](const R (&h)[KH]) {
#pragma unroll
    for (int k = 0; k < KR; ++k)
      if (rl[k] >= 0) lu[rl[k]] = h[k];
  };
  // A v of cell z of the vector v in registers, its plane (with halo) in LDS
  auto apply = [&](int z, const R (&v)[ZC], const R (&h)[KH]) -> R {
    const R* pl = lu + z * PL + oslot;
    const R w[6] = {wxm[z], wxp[z], wym[z], wyp[z], wz[z], wz[z + 1]};
    const R n[6] = {pl[-1], pl[1], pl[-PW], pl[PW], z == 0 ? h[KR] : v[z > 0 ? z - 1 : 0],
                    z + 1 == tzn ? h[KR + 1] : v[z + 1 < ZC ? z + 1 : ZC - 1]};
    R Av = apply_w<R>(sx, sy, sz, w, v[z], n);
    if (z > 0 && z >= tzn) Av = R(0);       // (no branch: the planes' LDS reads overlap)
    if (T.z0 + z == g.nz - 1 && S.sb != R(0)) Av = fma_r(S.sb, v[z], Av);
    return Av;
  };

  unsigned long long red = tab.v[0].epoch_base;
  bool ok = true;
  // iteration counts of this launch's latest probe of each order. Every wave has
  // them from the team reductions, so a step needs nothing of the step before it
  // from LDS (there is no barrier between two forward steps).
  int pc0 = 0, pc1 = 0, pc2 = 0;
  __syncthreads();
  for (int st = 0; st < tab.count; ++st) {
    const StepVar<R>& V = tab.v[st];
    // ---- initial guess (guess_order with the counts of this launch's probes)
    int order = V.gmode;
    if (order < 0) {
      const int here = tab.here[st];
      const int c0 = here & 1 ? pc0 : V.gi[V.gp[0]], c1 = here & 2 ? pc1 : V.gi[V.gp[1]],
                c2 = here & 4 ? pc2 : V.gi[V.gp[2]];
      order = 2;
      int best = c2;
      if (c1 < best) { order = 1; best = c1; }
      if (c0 < best) order = 0;
    }
    if (order == 3) order = V.xprev && V.xprev2 ? 3 : 0;
    else if (!V.xprev || !V.xprev2) order = 0;
    else if (order == 2 && !V.xprev3) order = 1;
    order = __builtin_amdgcn_readfirstlane(order);         // (uniform: it selects the vectors to load)
    const R* h2 = order >= 1 ? V.xprev2 : nullptr;
    const R* h3 = order == 2 ? V.xprev3 : nullptr;
    R e1, e2;
    guess_coef<R>(order, e1, e2);
    auto x0_of = [&](R a1, R a2, R a3) -> R {
      if (!h2) return a1;
      R v = mul_rn(e2, a2);
      if (h3) v = add_rn(v, a3);
      return fma_r(e1, a1, v);
    };
    // ---- set-up: r = b - A x0, u = r / D (h1, which b needs, in s). In the launch's
    // first step h1 comes from memory, then x and its halo still hold it.
    {
      const __amdgpu_buffer_rsrc_t r1 = brick_rsrc(V.xprev, g.ng), r2 = brick_rsrc(h2, g.ng), r3 = brick_rsrc(h3, g.ng);
#pragma unroll
      for (int z = 0; z < ZC; ++z) {
        // (a null vector's resource covers nothing: it reads 0)
        const unsigned v = z < tzn ? vo : kOffLane;
        if (st == 0) x[z] = brick_ld<kCpolSc1, R>(r1, v, po(z));
        p[z] = h2 ? brick_ld<kCpolSc1, R>(r2, v, po(z)) : R(0);
        u[z] = h3 ? brick_ld<kCpolSc1, R>(r3, v, po(z)) : R(0);
      }
    }
    if (st == 0 && V.xprev) ld_halo(V.xprev, hx);
    if (h2) ld_halo(h2, hp);
    if (h3) ld_halo(h3, hs);
    const R top = own && T.z0 == 0 ? V.top_src[gx + g.nx * gy] : R(0);
#pragma unroll
    for (int z = 0; z < ZC; ++z) {
      s[z] = x[z];
      x[z] = x0_of(x[z], p[z], u[z]);
    }
#pragma unroll
    for (int k = 0; k < KH; ++k) hx[k] = x0_of(hx[k], hp[k], hs[k]);
    put(x);
    put_halo(hx);
    __syncthreads();
    double v4[4] = {0.0, 0.0, 0.0, 0.0};    // |b|^2, r.u, |r|^2, u.A u
    const unsigned tag0 = __builtin_amdgcn_readfirstlane((unsigned)(red + 1));
    {
      const __amdgpu_buffer_rsrc_t rb2 = bank_of(2);
#pragma unroll
      for (int z = 0; z < ZC; ++z) {
        const R Av = apply(z, x, hx);
        R b = s[z];
        if (T.z0 + z == 0) b += V.top_scale * top;
        const R r = b - Av;
        u[z] = r * rD[z];
        const double bd = b, rd = r;
        v4[0] += bd * bd;
        v4[1] += rd * (double)u[z];
        v4[2] += rd * rd;
        if (S.team > 1) halo_st<R>(rb2, vpub(z), 2 * po(z), u[z], tag0);
      }
    }
    __syncthreads();                        // LDS holds x0 no longer
    // ---- w0 = A u0
    put(u);
    if (S.team > 1) {
      long long t0 = 0;
      while (true) {
        asm volatile("" ::: "memory");      // every pass loads anew
        if (ld_tagged(2, tag0, hu)) break;
        const long long now = wall_clock64();
        if (t0 == 0) t0 = now;
        if (now - t0 > S.timeout_ticks) { ok = false; break; }
      }
    }
    put_halo(hu);
    __syncthreads();
    {
      const __amdgpu_buffer_rsrc_t rw = bank_of((int)(tag0 & 1));
#pragma unroll
      for (int z = 0; z < ZC; ++z) wr[z] = s[z] = p[z] = R(0);
#pragma unroll
      for (int z = 0; z < ZC; ++z) {
        const R w = apply(z, u, hu);
        wr[z] = w * rD[z];
        v4[3] += (double)u[z] * (double)w;
        if (S.team > 1) halo_st<R>(rw, vpub(z), 2 * po(z), wr[z], tag0);
      }
    }
#pragma unroll
    for (int k = 0; k < KH; ++k) hs[k] = hp[k] = R(0);
    {
      // (waits for the stores: past this reduction the states of earlier steps are complete)
      auto f = [&](unsigned tag) { return ld_tagged((int)(tag & 1), tag, hw); };
      ok = team_sum<R, 4, NT, false>(S, rank, red, v4, rb, BrickHalo<decltype(f)>{f}, ok);
    }
    const double bb = v4[0];
    double gam = v4[1], rr = v4[2];
    int it = 0, status = kOk;
    if (ok && bb == 0.0) {
#pragma unroll
      for (int z = 0; z < ZC; ++z) x[z] = R(0);
#pragma unroll
      for (int k = 0; k < KH; ++k) hx[k] = R(0);
      rr = 0.0;
    } else if (ok && rr > S.rtol2 * bb) {
      double a_cg = gam / v4[3], b_cg = 0.0;
      while (ok) {
        if (it >= S.max_iter) { status |= kNoConv; break; }
        const R a = (R)a_cg, b = (R)b_cg;
        // (first iteration: b = 0 and p = s = 0, so s = w and p = u exactly)
#pragma unroll
        for (int z = 0; z < ZC; ++z) {
          s[z] = fma_r(b, s[z], wr[z]);
          p[z] = fma_r(b, p[z], u[z]);
          u[z] = fma_r(-a, s[z], u[z]);
          x[z] = fma_r(a, p[z], x[z]);
        }
        put(u);
        if (S.team > 1) {
#pragma unroll
          for (int k = 0; k < KH; ++k) {
            hs[k] = fma_r(b, hs[k], hw[k]);
            hp[k] = fma_r(b, hp[k], hu[k]);
            hu[k] = fma_r(-a, hs[k], hu[k]);
            hx[k] = fma_r(a, hp[k], hx[k]);
          }
          put_halo(hu);
        }
        __syncthreads();
        const unsigned tag = __builtin_amdgcn_readfirstlane((unsigned)(red + 1));
        const __amdgpu_buffer_rsrc_t rw = bank_of((int)(tag & 1));
        double acc[3] = {0.0, 0.0, 0.0};
#pragma unroll
        for (int z = 0; z < ZC; ++z) {
          const R w = apply(z, u, hu);
          wr[z] = w * rD[z];
          if (S.team > 1) halo_st<R>(rw, vpub(z), 2 * po(z), wr[z], tag);
          const double ud = u[z], rd = (double)D[z] * ud;
          acc[0] += rd * ud;
          acc[1] += (double)w * ud;
          acc[2] += rd * rd;
        }
        {
          auto f = [&](unsigned t) { return ld_tagged((int)(t & 1), t, hw); };
          ok = team_sum<R, 3, NT, false, BrickHalo<decltype(f)>, false>(S, rank, red, acc, rb,
                                                                        BrickHalo<decltype(f)>{f}, ok);
        }
        ++it;
        rr = acc[2];
        if (!(rr > S.rtol2 * bb)) break;
        const double gn = acc[0], dn = acc[1];
        cg_scalars(gn, dn, gam, a_cg, b_cg);
      }
    }
    if (!(bb < INFINITY) || !(rr < INFINITY) || rr != rr) status |= kNonFinite;
    if (!ok) status |= kTimeout;

    // ---- the state, the surface frame, the checkpoint
    {
      const __amdgpu_buffer_rsrc_t rx = brick_rsrc(V.x, g.ng), rc = brick_rsrc(V.ckpt_out, g.ng);
#pragma unroll
      for (int z = 0; z < ZC; ++z)
        if (z < tzn) {
          brick_st<kCpolSc1, R>(rx, vo, po(z), x[z]);
          if (V.ckpt_out) brick_st<0, R>(rc, vo, po(z), x[z]);
        }
    }
    if (own && V.surf_out && T.z0 == 0) V.surf_out[gx + g.nx * gy] = S.mode == kForward ? x[0] : V.surf_scale * x[0];
    const double relres = bb > 0.0 ? sqrt(rr / bb) : 0.0;
    if (tid == 0 && rank == 0 && V.out_iters) {
      V.out_iters[0] = it;
      V.out_relres[0] = relres;
      V.out_status[0] = status;
    }
    {
      const int n = __builtin_amdgcn_readfirstlane(it);
      if (V.gmode == 0) pc0 = n;
      if (V.gmode == 1) pc1 = n;
      if (V.gmode == 2) pc2 = n;
    }
    if (!ok) return;                        // a wait timed out: every workgroup leaves within its own time limit
    if (S.mode == kAdjoint && V.T_grad) {
      // G_p -= sum_f s_f (a_q/(a_p+a_q))^2 (T_p-T_q)(mu_p-mu_q), as GradOp
      put(x);
      put_halo(hx);
      __syncthreads();
      const __amdgpu_buffer_rsrc_t rt = brick_rsrc(V.T_grad, g.ng);
#pragma unroll
      for (int z = 0; z < ZC; ++z) {
        asm volatile("" ::: "memory");      // one cell's loads at a time
        if (own && z < tzn) {
          const int k = T.z0 + z;
          const R* pl = lu + z * PL + oslot;
          const R nzm = z == 0 ? hx[KR] : x[z > 0 ? z - 1 : 0];
          const R nzp = z + 1 == tzn ? hx[KR + 1] : x[z + 1 < ZC ? z + 1 : ZC - 1];
          const double ia = ia_at(true, vo, z), m = x[z], t = brick_ld<0, R>(rt, vo, po(z));
          double acc = 0.0;
          // the face towards the cell at offset v of plane zq (in: the plane exists), mu there mq
          auto term = [&](R sf, unsigned v, int zq, bool in, R mq) {
            const double w = ia / (ia + (double)ia_at(in, v, zq));
            const R tq = in ? brick_ld<0, R>(rt, v, po(zq)) : R(0);
            acc += (double)sf * (w * w) * ((t - (double)tq) * (m - (double)mq));
          };
          term(sx, vxm, z, true, pl[-1]);
          term(sx, vxp, z, true, pl[1]);
          term(sy, vym, z, true, pl[-PW]);
          term(sy, vyp, z, true, pl[PW]);
          term(sz, vo, z - 1, k > 0, nzm);
          term(sz, vo, z + 1, k + 1 < g.nz, nzp);
          double* G = S.G + (gx + g.nx * gy) + (long long)k * nxy;
          *G = *G - acc;
        }
      }
      __syncthreads();
    }
  }
}

}  // namespace nh
