// nh_jacobi.hpp -- the paper's fixed-K Jacobi inner solver (eq. jacobi_iter,
// App. D.2) with temporal blocking, for thin grids (nz <= 32) in FP32, several
// implicit-Euler steps per launch.
//
// An exchange between workgroups costs 1.5-2 us on this chip, more than a sweep
// of a small grid, so a step that exchanges after every sweep is bound by it
// (75x50x24 in the streaming kernel: 7.1 us per sweep with a team reduction each). Here each workgroup
// owns an interior tile of kJacIX x IY columns and computes on the tile widened
// by kJacS columns on every lateral side (an extended tile of kJacEX x (IY + 6)
// columns, two threads per column, each with half of the column's cells, their
// face coefficients, 1/D and b in registers). A phase runs kJacS sweeps
// exchanging the tile through LDS only: after j sweeps the j outermost rings of
// the extended tile hold wrong values (they miss neighbours outside it), so after
// kJacS sweeps exactly the interior is right. The halo columns are computed again
// by every tile that needs them; the small interiors (64x64: 96 workgroups of
// 24 x 2 columns) buy short sweeps with CUs that would be idle, and grids with
// more columns take taller tiles.
//
// Within a sweep the +-x neighbours come from the neighbouring lanes (a row of
// the extended tile is half a wave), the +-y neighbours through LDS (two
// buffers in turn: one barrier per sweep), the +-z neighbours from registers
// but for the cell where the column is split.
//
// Between phases there is no barrier across workgroups: a phase stores its
// interior into a tagged buffer, one 64-bit word per cell holding the value and
// the phase's tag, stored and loaded device-coherent, and the next phase's halo
// loads (all cells of a thread in one pass) are repeated until every word
// carries the expected tag; the interior is still in registers. A
// workgroup can run at most one phase ahead of another whose columns it reads,
// because that one reads its columns too (within kJacS columns of each other's
// interior, which is what `need` limits the loads to), so the two
// alternating buffers are never overwritten while still being read. Tags grow
// from launch to launch (the host clears the buffers before they wrap), so a
// stale word never matches. The last phase of a step is published the same way: its
// halo is what the next step starts from and what the gradient pass reads.
// The residual sums of the steps are added up once, at the end of a launch.
//
// Measured on 64x64x16, K = 50, periodic: 1.46 us per sweep (phases of three
// sweeps, 0.78 us each, and 1.5 us of exchange; a sweep is bound by its
// instructions, 8 cells of ~17 for two waves per SIMD, and one LDS round trip),
// 3.66 with 24 workgroups of 24 x 8 columns, four neighbours of a cell read
// through LDS, b and 1/D in LDS, halo words awaited one by one and a reduction
// per step. 75x50x24: 2.0 us, 7.1 in the streaming kernel, 13.7 there before its
// team reduction became one exchange (each with the steps' set-up; the sweeps
// alone, from K = 75 to 150: 1.8, 6.7 and 12.5 us).
#pragma once

#include "nh_kernels.hpp"

namespace nh {

constexpr int kJacEX = 32;                  // columns of the extended tile in x: half a wave
constexpr int kJacS = 3;                    // sweeps per phase = halo width
constexpr int kJacIX = 24;                  // interior columns in x
static_assert(kJacIX + 2 * kJacS <= kJacEX, "a row of the extended tile is half a wave");
constexpr int kJacNZ = 16;                  // largest nz of jacobi_steps_kernel
constexpr int kJacNZDeep = 32;              // and of jacobi_deep_kernel
constexpr int jac_threads(int parts, int iy) { return parts * kJacEX * (iy + 2 * kJacS); }

// The steps of a launch take their per-step fields from tab.v (the rest of S
// is the same for all of them).
constexpr int kJacBatch = 12;               // steps per launch (their fields travel as kernel arguments)

struct JacSteps {
  StepVar<float> v[kJacBatch];
  int count;
};

__device__ __forceinline__ float lane_below(float v) {     // the value of the lane before (wave_shr:1)
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x138, 0xf, 0xf, false));
}
__device__ __forceinline__ float lane_above(float v) {     // the value of the lane after (wave_shl:1)
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x130, 0xf, 0xf, false));
}

struct JacNo { static constexpr bool value = false; };
struct JacYes { static constexpr bool value = true; };

// LDS of one workgroup: P threads per column with H cells each, IY interior
// rows. b and 1/D of a thread's cells live in LDS where its registers are few
// (128 with more than 768 threads, 168 with more than 512).
template <int H, int P, int IY>
struct JacLds {
  static constexpr int kC = kJacEX * (IY + 2 * kJacS);
  static constexpr int kNT = jac_threads(P, IY);
  static constexpr bool kB = kNT > 512 && (H > 8 || kNT > 768);
  static constexpr bool kRd = kNT > 768;
  alignas(16) float xs[2][P * H * kC];      // the exchanged iterate, two buffers of [4 planes][column][plane]
  alignas(16) float b[kB ? H * kNT : 4];    // [4 cells][thread][cell]
  alignas(16) float rd[kRd ? H * kNT : 4];
  RedBuf rb;
};

// nz <= P H cells per column. WFORM: the coefficients are face weights from
// 1/alpha, rounded as the streaming kernel's sweep rounds (diag_w, apply_w);
// else face conductances summed face by face.
template <int H, int P, int IY, bool WFORM, bool TRACE>
__device__ __forceinline__ void jacobi_tb_steps(const StepArgs<float>& S, const StepVar<float>* steps, int count,
                                                int rank, JacLds<H, P, IY>& sh) {
  using L = JacLds<H, P, IY>;
  constexpr int C = L::kC, NT = L::kNT;
  typedef float f4 __attribute__((ext_vector_type(4)));
  // slot of cell (plane k, column q): four cells of a column side by side, so a
  // thread's accesses are 16 bytes wide and those of a wave contiguous
  auto at = [](int k, int q) { return ((k >> 2) * C + q) * 4 + (k & 3); };
  static_assert(H % 4 == 0, "whole groups of four cells");
  float* const xs = sh.xs[0];
  RedBuf& rb = sh.rb;
  const Geom& g = S.g;
  const int tid = threadIdx.x;
  const int part = __builtin_amdgcn_readfirstlane(tid / C);   // (uniform: C is a multiple of 64)
  const int c = tid - part * C, k0 = part * H;
  const int lx = c % kJacEX, ly = c / kJacEX;
  const int x0 = (rank % S.jtx) * kJacIX, y0 = (rank / S.jtx) * IY;   // first interior column
  const int ix = min(kJacIX, g.nx - x0), iy = min(IY, g.ny - y0);     // interior extents inside the grid
  const int ux = x0 - kJacS + lx, uy = y0 - kJacS + ly;               // unwrapped grid column
  int gx = ux, gy = uy;
  bool valid;
  if (g.periodic) {
    gx = ((gx % g.nx) + g.nx) % g.nx;
    gy = ((gy % g.ny) + g.ny) % g.ny;
    valid = true;
  } else {
    valid = gx >= 0 && gx < g.nx && gy >= 0 && gy < g.ny;
  }
  const int col = valid ? gx + g.nx * gy : 0;
  const bool inner = lx >= kJacS && lx < kJacS + ix && ly >= kJacS && ly < kJacS + iy;
  // halo columns whose values can reach the interior within a phase
  const bool need = valid && !inner && lx < 2 * kJacS + ix && ly < 2 * kJacS + iy;
  const bool hl = lx > 0, hr = lx < kJacEX - 1, hd = ly > 0, hu = c + kJacEX < C;
  const bool hb = part > 0, ha = part < P - 1;   // another thread of the column holds cell k0-1 / k0+H
  const int nz = g.nz, nxy = (int)g.nxy;
  bool ok = true;
  int ntr = 0;
  auto stamp = [&]() {
    if (TRACE && S.trace && rank == S.trace_rank && tid == 0 && ntr < S.trace_cap) S.trace[ntr++] = wall_clock64();
  };
  stamp();

  // byte offsets of the column in a state and in a tagged buffer; plane k adds k planes
  const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc((void*)S.alpha, 0, (int)(4 * g.ng), 0x00020000);
  const unsigned vcol = valid ? 4u * (unsigned)col : kOffLane;
  auto plane = [&](int i) { return 4 * nxy * (k0 + i); };

  // coefficients of the own cells from the neighbours' alpha, exchanged through
  // LDS (WFORM: 1/alpha, +inf where there is no cell: weight 0)
  float cxm[H], cxp[H], cym[H], cyp[H], cz[H], rdr[L::kRd ? 1 : H], x[H], br[L::kB ? 1 : H];
  auto rd = [&](int i) -> float& { return L::kRd ? sh.rd[((i >> 2) * NT + tid) * 4 + (i & 3)] : rdr[L::kRd ? 0 : i]; };
  auto b = [&](int i) -> float& { return L::kB ? sh.b[((i >> 2) * NT + tid) * 4 + (i & 3)] : br[L::kB ? 0 : i]; };
  float czb = 0.f;                          // the face below the first own cell
  {
    float a[H];
#pragma unroll
    for (int i = 0; i < H; ++i) {
      a[i] = k0 + i < nz ? plane_ld_at(ra, vcol, plane(i)) : 0.f;
      if (WFORM) a[i] = inv_alpha<float>(a[i]);
    }
#pragma unroll
    for (int i = 0; i < H; ++i) xs[at(k0 + i, c)] = a[i];
    __syncthreads();
    const float none = WFORM ? INFINITY : 0.f;
    auto coef = [&](float s, float p, float q) -> float {
      if (WFORM) return face_w<float>(p, q);
      return p > 0.f ? face<float>(s, p, q) : 0.f;         // (p > 0: no face divides by zero)
    };
    if (hb) czb = coef(S.sz, a[0], xs[at(k0 - 1, c)]);
#pragma unroll
    for (int i = 0; i < H; ++i) {
      const int k = k0 + i;
      cxm[i] = coef(S.sx, a[i], hl ? xs[at(k, c - 1)] : none);
      cxp[i] = coef(S.sx, a[i], hr ? xs[at(k, c + 1)] : none);
      cym[i] = coef(S.sy, a[i], hd ? xs[at(k, c - kJacEX)] : none);
      cyp[i] = coef(S.sy, a[i], hu ? xs[at(k, c + kJacEX)] : none);
      cz[i] = coef(S.sz, a[i], i + 1 < H ? a[i + 1 < H ? i + 1 : 0] : (ha ? xs[at(k + 1, c)] : none));
      const float czm = i > 0 ? cz[i > 0 ? i - 1 : 0] : czb;
      float D;
      if (WFORM) {
        const float w[6] = {cxm[i], cxp[i], cym[i], cyp[i], czm, cz[i]};
        D = diag_w<float>(S.sx, S.sy, S.sz, w);
        if (k0 + i == nz - 1 && S.sb != 0.f) D = add_rn(D, S.sb);
      } else {
        D = diag_of<float>(cxm[i], cxp[i], cym[i], cyp[i], czm, cz[i], k0 + i == nz - 1 ? S.sb : 0.f);
      }
      rd(i) = valid && k0 + i < nz ? rcp<float>(D) : 1.f;
    }
    __syncthreads();                        // alpha reads done before the first exchange of x
  }
  stamp();

  const int K = S.jacobi_k;
  const int phases = (K + kJacS - 1) / kJacS;
  int buf = 0;                              // LDS buffer of the next exchange
  for (int st = 0; st < count; ++st) {
    const StepVar<float>& V = steps[st];
    int col_l = col;                        // (laundered: no 64-bit addresses held from step to step)
    asm volatile("" : "+v"(col_l));
    // b = h1 + the top source; x^(0) = h1 (in the launch's first step from
    // memory, then in x from the last step's end)
    if (st == 0) {
      const __amdgpu_buffer_rsrc_t r1 =
          __builtin_amdgcn_make_buffer_rsrc((void*)V.xprev, 0, V.xprev ? (int)(4 * g.ng) : 0, 0x00020000);
#pragma unroll
      for (int i = 0; i < H; ++i) x[i] = k0 + i < nz ? plane_ld_at(r1, vcol, plane(i)) : 0.f;
    }
    const float top = valid && part == 0 ? V.top_src[col_l] : 0.f;
#pragma unroll
    for (int i = 0; i < H; ++i) {
      float bi = x[i];
      if (k0 + i == 0) bi += V.top_scale * top;
      b(i) = bi;
    }
    for (int ph = 0; ph < phases; ++ph) {
      const int ns = min(kJacS, K - ph * kJacS);
      const bool last_phase = ph == phases - 1;
      double vb = 0.0, vr = 0.0;            // |b|^2 and |b - A x|^2 of the last sweep's input
      // One sweep. DIAG: add up |b|^2 and the residual of its input (only the
      // step's last sweep does; predicated, the FP64 sums would double the
      // instructions of every sweep).
      auto sweep = [&](auto diag) {
        constexpr bool DIAG = decltype(diag)::value;
        // one base per sweep and constant offsets from it (laundered: hoisted,
        // each cell's addresses would hold registers through the launch)
        int cb = buf * (P * H * C) + 4 * (part * (H / 4) * C + c), tl = 4 * tid;
        asm volatile("" : "+v"(cb));
        asm volatile("" : "+v"(tl));
        float* xp = xs + cb;
        buf ^= 1;
#pragma unroll
        for (int q = 0; q < H / 4; ++q) *(f4*)(xp + 4 * q * C) = f4{x[4 * q], x[4 * q + 1], x[4 * q + 2], x[4 * q + 3]};
        __syncthreads();
        // a missing neighbour reads a cell whose face coefficient is 0
        const float* pd = xp + (hd ? -4 * kJacEX : 0);
        const float* pu = xp + (hu ? 4 * kJacEX : 0);
        const float xbelow = hb ? xp[-4 * C + 3] : x[0], xabove = ha ? xp[H * C] : x[H - 1];
        float vm = xbelow;                  // the cell below, before its update
#pragma unroll
        for (int q = 0; q < H / 4; ++q) {
          if (NT > 768 && q > 0) asm volatile("" ::: "memory");   // fewer reads in flight, fewer registers
          const f4 fd = *(const f4*)(pd + 4 * q * C), fu = *(const f4*)(pu + 4 * q * C);
          f4 fb, fr;
          if (L::kB) fb = *(const f4*)(sh.b + 4 * q * NT + tl);
          if (L::kRd) fr = *(const f4*)(sh.rd + 4 * q * NT + tl);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int i = 4 * q + e;
            const float v = x[i];
            const float xl = lane_below(v), xr = lane_above(v);
            const float xa = i + 1 < H ? x[i + 1 < H ? i + 1 : 0] : xabove;
            const float czm = i > 0 ? cz[i > 0 ? i - 1 : 0] : czb;
            const float sbk = k0 + i == nz - 1 ? S.sb : 0.f;
            const float bi = L::kB ? fb[e] : b(i);
            float r;
            if (WFORM) {
              const float w[6] = {cxm[i], cxp[i], cym[i], cyp[i], czm, cz[i]};
              const float n[6] = {xl, xr, fd[e], fu[e], vm, xa};
              r = bi - fma_r(sbk, v, apply_w<float>(S.sx, S.sy, S.sz, w, v, n));
            } else {
              float s = cxm[i] * (v - xl);
              s += cxp[i] * (v - xr);
              s += cym[i] * (v - fd[e]);
              s += cyp[i] * (v - fu[e]);
              s += czm * (v - vm);
              s += cz[i] * (v - xa);
              s = fma_r(sbk, v, s);
              r = bi - (v + s);
            }
            x[i] = v + r * (L::kRd ? fr[e] : rd(i));
            vm = v;
            if (DIAG && inner && k0 + i < nz) {
              vb += (double)bi * (double)bi;
              vr += (double)r * (double)r;
            }
          }
        }
      };
      for (int j = 0; j < ns - (last_phase ? 1 : 0); ++j) sweep(JacNo{});
      if (last_phase) sweep(JacYes{});
      stamp();
      // publish the interior; then the next phase's halo
      const unsigned tag = V.jtag + (unsigned)ph;
      const __amdgpu_buffer_rsrc_t rt =
          __builtin_amdgcn_make_buffer_rsrc(S.jt[tag & 1], 0, (int)(8 * g.ng), 0x00020000);
      unsigned v2 = 2u * vcol;              // (a lane that stores or loads has a valid column)
      asm volatile("" : "+v"(v2));
      const unsigned vneed = need ? v2 : kOffLane, vinner = inner ? v2 : kOffLane;
      const bool more = !last_phase || st + 1 < count || (S.mode == kAdjoint && V.T_grad);
      if (more) {
        typedef unsigned u2 __attribute__((ext_vector_type(2)));
#pragma unroll
        for (int i = 0; i < H; ++i)
          if (k0 + i < nz)
            __builtin_amdgcn_raw_buffer_store_b64(u2{__float_as_uint(x[i]), tag}, rt, vinner, 2 * plane(i), kCpolSc1);
      }
      if (last_phase) {
        double sums[2] = {vb, vr};
        wave_sums<2>(sums);
        if ((tid & 63) == 0) {
          rb.red[tid >> 6][0] = sums[0];
          rb.red[tid >> 6][1] = sums[1];
        }
        const __amdgpu_buffer_rsrc_t rx =
            __builtin_amdgcn_make_buffer_rsrc(V.x, 0, (int)(4 * g.ng), 0x00020000);
        const __amdgpu_buffer_rsrc_t rc =
            __builtin_amdgcn_make_buffer_rsrc(V.ckpt_out, 0, V.ckpt_out ? (int)(4 * g.ng) : 0, 0x00020000);
        const unsigned vi = inner ? vcol : kOffLane;
#pragma unroll
        for (int i = 0; i < H; ++i)
          if (k0 + i < nz) {
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(x[i]), rx, vi, plane(i), 0);
            if (V.ckpt_out) __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(x[i]), rc, vi, plane(i), 0);
          }
        if (V.surf_out && inner && part == 0) V.surf_out[col_l] = S.mode == kForward ? x[0] : V.surf_scale * x[0];
      }
      if (more) {
        // all of a thread's halo cells in one round trip
        constexpr int PG = H;
#pragma unroll
        for (int i0 = 0; i0 < H; i0 += PG) {
          long long t0 = 0;
          while (true) {
            asm volatile("" ::: "memory");  // every pass loads anew
            bool all = true;
            unsigned w[PG];
#pragma unroll
            for (int i = 0; i < PG; ++i) {
              // (planes past the grid and lanes that need nothing load nothing; no branch among the loads)
              const int k = k0 + i0 + i;
              const auto t = __builtin_amdgcn_raw_buffer_load_b64(rt, k < nz ? vneed : kOffLane,
                                                                  k < nz ? 2 * plane(i0 + i) : 0, kCpolSc1);
              w[i] = t[0];
              all &= (t[1] == tag) | !need | (k >= nz);
            }
            if (all || !ok) {
              if (need) {
#pragma unroll
                for (int i = 0; i < PG; ++i) x[i0 + i] = __uint_as_float(w[i]);
              }
              break;
            }
            const long long now = wall_clock64();
            if (t0 == 0) t0 = now;
            if (now - t0 > S.timeout_ticks) ok = false;    // (after a time-out, wait no more)
          }
        }
      }
      stamp();
    }
    if (S.mode == kAdjoint && V.T_grad) {
      // gradient of the interior (GradOp), its cells dealt to all threads: mu
      // with its halo in LDS, alpha and T from memory
      float* xb = xs + buf * (P * H * C);
      buf ^= 1;
      int cb = 4 * (part * (H / 4) * C + c);
      asm volatile("" : "+v"(cb));
#pragma unroll
      for (int q = 0; q < H / 4; ++q)
        *(f4*)(xb + cb + 4 * q * C) = f4{x[4 * q], x[4 * q + 1], x[4 * q + 2], x[4 * q + 3]};
      __syncthreads();
      const int ncell = ix * iy * nz;
      const double sx = S.sx, sy = S.sy, sz = S.sz;
      int e = tid;
      asm volatile("" : "+v"(e));
#pragma unroll 1
      for (; e < ncell; e += NT) {
        const int k = e / (ix * iy), r = e - k * (ix * iy);
        const int jy = r / ix, jx = r - jy * ix;
        const int px = x0 + jx, py = y0 + jy;
        const int p = px + g.nx * py + k * nxy;
        const int q = (jy + kJacS) * kJacEX + jx + kJacS;
        const double ia = inv_alpha<float>(S.alpha[p]), mc = xb[at(k, q)], t = V.T_grad[p];
        double acc = 0.0;
        auto term = [&](double sf, bool in, int pq, float mq) {
          if (NT > 768) asm volatile("" ::: "memory");   // fewer loads in flight, fewer registers
          const double w = ia / (ia + (double)inv_alpha<float>(in ? S.alpha[pq] : 0.f));
          const float tq = in ? V.T_grad[pq] : 0.f;
          acc += sf * (w * w) * ((t - (double)tq) * (mc - (double)mq));
        };
        const bool per = g.periodic != 0;
        term(sx, per || px > 0, px > 0 ? p - 1 : p + g.nx - 1, xb[at(k, q - 1)]);
        term(sx, per || px + 1 < g.nx, px + 1 < g.nx ? p + 1 : p + 1 - g.nx, xb[at(k, q + 1)]);
        term(sy, per || py > 0, py > 0 ? p - g.nx : p + g.nx * (g.ny - 1), xb[at(k, q - kJacEX)]);
        term(sy, per || py + 1 < g.ny, py + 1 < g.ny ? p + g.nx : p - g.nx * (g.ny - 1), xb[at(k, q + kJacEX)]);
        term(sz, k > 0, p - nxy, k > 0 ? xb[at(k - 1, q)] : 0.f);
        term(sz, k + 1 < nz, p + nxy, k + 1 < nz ? xb[at(k + 1, q)] : 0.f);
        S.G[p] = S.G[p] - acc;
      }
#pragma unroll
      for (int q = 0; q < H / 4; ++q) {     // (back from LDS: no registers held through the pass)
        const f4 t = *(const f4*)(xb + cb + 4 * q * C);
#pragma unroll
        for (int e = 0; e < 4; ++e) x[4 * q + e] = t[e];
      }
    }
    __syncthreads();                        // rb.red is complete
    int tl = tid;
    asm volatile("" : "+v"(tl));
    if (tl < 2) {
      double s = 0.0;
      for (int w = 0; w < NT / 64; ++w) s += rb.red[w][tl];
      st_out(S.jpart + ((size_t)st * S.team + rank) * 2 + tl, s);
    }
    __syncthreads();                        // and free again
  }
  // the steps' residuals, once every workgroup has stored its sums
  unsigned long long red = steps[0].epoch_base;
  double none[1] = {0.0};
  ok = team_sum<float, 1, NT, false>(S, rank, red, none, rb, NoNeighbours(), ok);
  if (rank == 0) {
    for (int st = tid >> 6; st < count; st += NT / 64) {
      double v2[2] = {0.0, 0.0};
      for (int r = tid & 63; r < S.team; r += 64) {
        const double* q = S.jpart + ((size_t)st * S.team + r) * 2;
        v2[0] += ld_out(q);
        v2[1] += ld_out(q + 1);
      }
      wave_sums<2>(v2);
      if ((tid & 63) == 0 && steps[st].out_iters) {
        const double bb = v2[0], rr = v2[1];
        int status = kOk;
        if (!(bb < INFINITY) || !(rr < INFINITY)) status |= kNonFinite;
        if (!ok) status |= kTimeout;
        steps[st].out_iters[0] = ok ? K : 0;
        steps[st].out_relres[0] = bb > 0.0 ? sqrt(rr / bb) : 0.0;
        steps[st].out_status[0] = status;
      }
    }
  }
}

// nz <= 16: interior tiles of 24 x IY columns, two threads per column (64x64x16,
// three sweeps: 2.3 us with two or one thread per column, 3.4 with four; the
// exchange 1.5 us with two, 1.9 with one).
template <int IY>
__global__ void __launch_bounds__(jac_threads(2, IY), 1) jacobi_steps_kernel(StepArgs<float> S, JacSteps tab) {
  __shared__ JacLds<kJacNZ / 2, 2, IY> sh;
  jacobi_tb_steps<kJacNZ / 2, 2, IY, false, false>(S, tab.v, tab.count, blockIdx.x, sh);
}

// One step, with phase stamps.
template <int IY>
__global__ void __launch_bounds__(jac_threads(2, IY), 1) jacobi_step_kernel(StepArgs<float> S) {
  __shared__ JacLds<kJacNZ / 2, 2, IY> sh;
  const StepVar<float> V = step_var(S);
  jacobi_tb_steps<kJacNZ / 2, 2, IY, false, true>(S, &V, 1, blockIdx.x, sh);
}

// nz <= P H: more threads or more cells per thread.
template <int H, int P, int IY>
__global__ void __launch_bounds__(jac_threads(P, IY), 1) jacobi_deep_kernel(StepArgs<float> S, JacSteps tab) {
  __shared__ JacLds<H, P, IY> sh;
  jacobi_tb_steps<H, P, IY, true, false>(S, tab.v, tab.count, blockIdx.x, sh);
}

}  // namespace nh
