// HIP kernels of the Riccati-sweep iteration for gfx950 (arXiv:2205.15000).
//
//   interp_kernel       Delta(p_k, slot), a(slot) = v_k.A(slot) on the rotated
//                       lattices (Sec. III.A bilinear interpolation)
//   sweep_kernel        gamma forward / gamma~ backward along every segment
//                       (App. C), Green's functions (Sec. II.A) and per-node
//                       pole sums; one group of G lanes per segment and
//                       direction, EPL energies per lane, all angles in one
//                       launch
//   rotate_back_kernel  rotated lattice -> reference cells, angle sums,
//                       gap update (Eq. gapeq_fixpoint), current
//                       (Eq. current_density), free-energy density
//   ldos_back_kernel    rotate-back of the per-energy LDOS values
//   curl / reductions / Picard helpers (App. D, App. E)
#include <algorithm>

#include "kernels.hpp"
#include "plan.hpp"
#include "sweep.hpp"

namespace qc {

// --------------------------------------------------------------------------
// interpolation pre-pass
// --------------------------------------------------------------------------
template <typename T>
__device__ __forceinline__ void interp_slot(const InterpArgs& a, int64_t s, node4<T>* __restrict__ nodes) {
  if (s >= a.nslot) return;
  const int k = a.slot_angle[s];
  const double px = a.px[s], py = a.py[s];
  int di[4], ai[4];
  double dw[4], aw[4];
  delta_stencil(a.geom, px, py, a.fb[s], di, dw);
  a_stencil(a.geom, px, py, ai, aw);
  double dx = 0.0, dy = 0.0;
  for (int c = 0; c < 4; ++c) {
    const int idx = di[c];
    const double w = dw[c];
    double vx = 0.0, vy = 0.0;
    for (int g = 0; g < a.ncomp; ++g) {
      const double ex = a.eta[2 * (g * a.n_theta + k)], ey = a.eta[2 * (g * a.n_theta + k) + 1];
      const double fx = a.delta[2 * (static_cast<int64_t>(g) * a.ncell + idx)];
      const double fy = a.delta[2 * (static_cast<int64_t>(g) * a.ncell + idx) + 1];
      vx += ex * fx - ey * fy;
      vy += ex * fy + ey * fx;
    }
    dx += vx * w;
    dy += vy * w;
  }
  double ax = 0.0, ay = 0.0;
  for (int c = 0; c < 4; ++c) {
    ax += a.A[ai[c]] * aw[c];
    ay += a.A[a.ncell + ai[c]] * aw[c];
  }
  node4<T> v;
  v.dx = static_cast<T>(dx);
  v.dy = static_cast<T>(dy);
  v.a = static_cast<T>(a.cosk[k] * ax + a.sink[k] * ay + a.aext[s]);
  v.pad = T(0);
  nodes[s] = v;
}

template <typename T>
__global__ void __launch_bounds__(256) interp_kernel(InterpArgs a, node4<T>* __restrict__ nodes) {
  interp_slot<T>(a, static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x, nodes);
}

// Single order-parameter component: Delta and A_ind packed per cell in the
// sweep precision, so the gathers of a slot touch one 16 B (FP32) or 32 B
// (FP64) record per corner and the FP32 grid stays resident in L2.  Cells
// outside the grain carry a NaN in Re Delta: the masked interpolation reads
// the mask from the same record instead of a separate dependent load.
template <typename T>
__device__ __forceinline__ cell4<T> cell_values(const InterpArgs& a, int64_t i) {
  cell4<T> c;
  c.dx = a.geom.mask[i] ? static_cast<T>(a.delta[2 * i]) : __builtin_nan("");
  c.dy = static_cast<T>(a.delta[2 * i + 1]);
  c.ax = static_cast<T>(a.A[i]);
  c.ay = static_cast<T>(a.A[a.ncell + i]);
  return c;
}
template <typename T>
__device__ __forceinline__ void pack_cell(const InterpArgs& a, int64_t i, cell4<T>* __restrict__ cells) {
  if (i < a.ncell) cells[i] = cell_values<T>(a, i);
}
template <typename T>
__global__ void __launch_bounds__(256) pack_cells_kernel(InterpArgs a, cell4<T>* __restrict__ cells) {
  pack_cell<T>(a, static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x, cells);
}

// Same stencils as interp_kernel (identical floating-point operations for the
// weights): masked bilinear for Delta with the nearest-grain-cell fallback,
// clamped bilinear for A_ind.  Away from the array edge the two stencils
// share their corners, and the four records serve both.
// PACKED: the cells from the packed records, or straight from the fields (the
// same values).
template <typename T, bool PACKED>
__device__ __forceinline__ void interp1_block(const InterpArgs& a, int block, const cell4<T>* __restrict__ cells,
                                              node4<T>* __restrict__ nodes) {
  auto cell_at = [&](int64_t i) {
    if constexpr (PACKED) return cells[i];
    return cell_values<T>(a, i);
  };
  // one wave per segment: its record is read once (scalar loads), and each
  // lane takes every 64th slot of the segment
  const int64_t seg = __builtin_amdgcn_readfirstlane(block * 4 + static_cast<int>(threadIdx.x >> 6));
  if (seg >= a.nseg) return;
  const SegGeo sgeo = a.seg_geo[seg];
  const int nsl = sgeo.n > 0 ? sgeo.n : 1;
  const GridGeom& gg = a.geom;
  const int k = sgeo.k;
  const double epx = a.cosk[k], epy = a.sink[k];
  for (int t = static_cast<int>(threadIdx.x & 63); t < nsl; t += 64) {
    const int64_t s = sgeo.slot0 + t;
    const int fb = a.fb[s];
    // the slot position as the plan forms it, so the corner choice below is
    // the one the nearest-cell fallback was decided on
    const double sp = sgeo.n > 0 ? rn_node_s(static_cast<double>(sgeo.jf + t), a.half, gg.h) : sgeo.smid;
    const double px = rn_point(a.cx, sgeo.u, epy, sp, epx);
    const double py = rn_point(a.cy, sgeo.u, -epx, sp, epy);
    const double fx = (px - gg.x0) / gg.h - 0.5, fy = (py - gg.y0) / gg.h - 0.5;
    const int i0 = static_cast<int>(__builtin_floor(fx)), j0 = static_cast<int>(__builtin_floor(fy));
    const double wx = fx - i0, wy = fy - j0;
    double w[4];
    w[0] = (1 - wx) * (1 - wy);
    w[1] = wx * (1 - wy);
    w[2] = (1 - wx) * wy;
    w[3] = wx * wy;
    cell4<T> v[4];
    double tot = 0.0;
    for (int c = 0; c < 4; ++c) {
      const int ci = i0 + (c & 1), cj = j0 + (c >> 1);
      const bool in = ci >= 0 && ci < gg.nx && cj >= 0 && cj < gg.ny;
      const int lc = min(max(ci, 0), gg.nx - 1), lj = min(max(cj, 0), gg.ny - 1);
      v[c] = cell_at(static_cast<int64_t>(lj) * gg.nx + lc);
      const bool ok = in && v[c].dx == v[c].dx;  // NaN marks cells outside the grain
      if (!ok) w[c] = 0.0;
      tot += w[c];
    }
    const double ex = a.eta[2 * k], ey = a.eta[2 * k + 1];
    double dx = 0.0, dy = 0.0;
    if (fb >= 0) {
      const cell4<T> f = cell_at(fb);
      const double fx0 = static_cast<double>(f.dx), fy0 = static_cast<double>(f.dy);
      dx = ex * fx0 - ey * fy0;
      dy = ex * fy0 + ey * fx0;
    } else {
      if (tot > 0.0)
        for (int c = 0; c < 4; ++c) w[c] /= tot;
      for (int c = 0; c < 4; ++c) {
        if (w[c] == 0.0) continue;  // a dropped corner may hold the NaN marker
        const double cx = static_cast<double>(v[c].dx), cy = static_cast<double>(v[c].dy);
        dx += (ex * cx - ey * cy) * w[c];
        dy += (ex * cy + ey * cx) * w[c];
      }
    }
    // A_ind: clamped bilinear
    const double fxa = __builtin_fmin(__builtin_fmax(fx, 0.0), gg.nx - 1.0);
    const double fya = __builtin_fmin(__builtin_fmax(fy, 0.0), gg.ny - 1.0);
    const int i0a = min(static_cast<int>(__builtin_floor(fxa)), gg.nx - 2);
    const int j0a = min(static_cast<int>(__builtin_floor(fya)), gg.ny - 2);
    const double wxa = fxa - i0a, wya = fya - j0a;
    double aw[4];
    aw[0] = (1 - wxa) * (1 - wya);
    aw[1] = wxa * (1 - wya);
    aw[2] = (1 - wxa) * wya;
    aw[3] = wxa * wya;
    double ax = 0.0, ay = 0.0;
    if (i0a == i0 && j0a == j0) {
      for (int c = 0; c < 4; ++c) {
        ax += static_cast<double>(v[c].ax) * aw[c];
        ay += static_cast<double>(v[c].ay) * aw[c];
      }
    } else {
      const int64_t b0 = static_cast<int64_t>(j0a) * gg.nx + i0a;
      for (int c = 0; c < 4; ++c) {
        const cell4<T> u = cell_at(b0 + (c & 1) + (c >> 1) * gg.nx);
        ax += static_cast<double>(u.ax) * aw[c];
        ay += static_cast<double>(u.ay) * aw[c];
      }
    }
    node4<T> o;
    o.dx = static_cast<T>(dx);
    o.dy = static_cast<T>(dy);
    // external field: symmetric, Landau or solenoid gauge (App. B; Eq. solenoid_gauge)
    double ex_x = 0.0, ex_y = 0.0;
    const double rx = px - a.cx, ry = py - a.cy;
    if (a.gauge == 0) {
      ex_x = -0.5 * a.bfield * ry;
      ex_y = 0.5 * a.bfield * rx;
    } else if (a.gauge == 1) {
      ex_x = -a.bfield * ry;
    } else {
      const double r2 = rx * rx + ry * ry;
      if (r2 > 0.0) {
        ex_x = -0.5 * a.flux * ry / r2;
        ex_y = 0.5 * a.flux * rx / r2;
      }
    }
    o.a = static_cast<T>(epx * (ax + ex_x) + epy * (ay + ex_y));
    o.pad = T(0);
    nodes[s] = o;
  }
}
template <typename T, bool PACKED>
__global__ void __launch_bounds__(256) interp1_kernel(InterpArgs a, const cell4<T>* __restrict__ cells,
                                                      node4<T>* __restrict__ nodes) {
  interp1_block<T, PACKED>(a, static_cast<int>(blockIdx.x), cells, nodes);
}

// --------------------------------------------------------------------------
// Riccati sweep
//
// Lane group of G lanes per segment, EPL consecutive energies per lane
// (energy e = lane * EPL + i).  Step t (t = 0..n) joins value slot t-1 and t;
// a boundary point takes the value of the nearest slot (App. C), so the
// half-step value is the mean of the two slot values with V(-1) = V(0) and
// V(n) = V(n-1).  gamma runs t = 0..n, gamma~ t = n..0 with D -> -D*.  The
// partial end steps (t = 0 and t = n) are peeled off the loops, so interior
// steps use per-energy constants formed once for the full step h.
//
// Two waves share a bundle of 64/G segments, one per direction: wave 0
// marches gamma from R_min, wave 1 gamma~ from R_max, both at once.  Each
// leaves its values at every second node of its own first half in the spill
// array; the waves meet at a barrier when both have reached the middle, and
// on its second half each reads the other's values, takes one step of the
// other march for the node between two stored ones (the same step on the
// same inputs, so the same value), and forms the node sums there.
//
// What bounds it: with every node spilled by one wave that marched gamma and
// then gamma~, the sweep of the 400 x 400 d-wave square (64 angles, 64 poles)
// moved 5.7 GB (FP32) or 11.2 GB (FP64) at 4.1 TB/s, 85% of what a large copy
// reaches on this card: it was bound by the spill's traffic.  Two waves halve
// the serial chain (n + 1 steps instead of 2 n + 2); every second node halves
// the traffic for half a march more arithmetic (26 of about 90 VALU
// instructions per node and pole), and the sweep is bound by VALU issue.
// Measured there: 1.41 -> 0.98 ms mixed, 2.84 -> 2.04 ms FP64 (sweeps alone;
// 1.05 to 1.09 and 2.10 ms inside iterations, at a lower clock); on smaller
// grains, which the chain's latency bounds, 565 -> 330 us (200 x 200 disc, 48
// poles, FP64) and 29 -> 17 us (32 x 32 disc).
//
// Per node and pole (Sec. II.A): X = gamma gamma~, g = -i pi (1-X)/(1+X),
// f = -2 i pi gamma/(1+X), f~ = 2 i pi gamma~/(1+X); the pole sums are
// formed from 1/(1+X) alone (identities at node_sums below).
// --------------------------------------------------------------------------
// Memory instructions stay on their side of this point (arithmetic may move
// across it): the wait counts of the loops below depend on their order.
__device__ __forceinline__ void vmem_order() { __builtin_amdgcn_sched_barrier(0x387); }

// The direction of one wave: DIR = +1 marches gamma, DIR = -1 gamma~.  In
// the order of the march the nodes are j = 0..n-1, node j at slot j or
// n - 1 - j.  Lanes that are not live only meet the barrier.
template <typename T, int EPL, int MODE, int DIR>
__device__ __forceinline__ void sweep_march(const SweepArgs& a, bool live, int64_t wseg, int lane, int G, int lg,
                                            const node4<T>* __restrict__ nodes, const cpx<T>* __restrict__ bc_prev,
                                            cpx<T>* __restrict__ bc_next, cpx<T>* __restrict__ bc_mirror, cpx<T>* gbase, int64_t gmul,
                                            T* __restrict__ ebuf, double* __restrict__ lsum) {
  constexpr T sd = T(DIR);  // D -> -D* for gamma~
  if (!live) wseg = 0;
  const int64_t seg = a.order ? static_cast<int64_t>(a.order[wseg]) : wseg;
  const int64_t slot0 = a.seg_slot0[seg];
  const int n = a.seg_n[seg];
  const int last = n > 0 ? n - 1 : 0;
  // nodes of the first half: gamma takes floor(n/2) of them, gamma~ the rest
  // (a boundary-only sweep has no second half)
  const int n1 = MODE == 2 ? n : (DIR > 0 ? n >> 1 : n - (n >> 1));
  const T hfull = static_cast<T>(a.h);
  const T q = static_cast<T>(a.q);
  const int e0 = lane * EPL;
  // The lane marches the energies es .. es + EPL - 1.  Its own start at e0;
  // a lane at the end of the range (e0 + EPL > n_e) starts early enough that
  // all EPL exist (the host never launches EPL > n_e).  The energies below
  // e0 belong to the lane before it, whose values it reproduces exactly
  // (same constants, same start): its loads and stores then cover EPL
  // consecutive entries, and its duplicates carry no weight and write no
  // end values.
  const int es = min(e0, a.n_e - EPL);
  bool own[EPL];
  for (int i = 0; i < EPL; ++i) own[i] = es + i >= e0;

  // The Matsubara sweeps (modes 0 and 3) have purely imaginary energies.
  constexpr bool kReal = MODE == 1 || MODE == 2;
  T ex[EPL], ey[EPL];
  // interior steps (length h): Kx = (-h Im z - 1)/2 and its square per energy
  T kxi[EPL], kx2i[EPL];
  for (int i = 0; i < EPL; ++i) {
    const int e = es + i;
    ex[i] = kReal ? static_cast<T>(a.eps[2 * (a.e_off + e)]) : T(0);
    ey[i] = static_cast<T>(a.eps[2 * (a.e_off + e) + 1]);
    kxi[i] = fmaT(T(-0.5) * hfull, ey[i], T(-0.5));
    kx2i[i] = kxi[i] * kxi[i];
  }
  const T hh = T(0.5) * hfull, hq8 = T(0.125) * hfull, hqa = T(0.25) * q * hfull;

  // Step with the half-step values (mean of two slots).  End steps take
  // every constant from their length.
  auto end_step = [&](cpx<T>* gv, const node4<T>& v, T hs) {
    const T h8 = T(0.125) * hs;
    StepC<T> c;
    c.c2x = h8 * (v.dy + v.dy);
    c.c2y = h8 * (sd * (v.dx + v.dx));
    c.U0x = T(-4) * c.c2x;
    c.U0y = T(4) * c.c2y;
    const T qa = T(0.5) * q * (v.a + v.a);
    for (int i = 0; i < EPL; ++i) {
      const T kx = fmaT(T(-0.5) * hs, ey[i], T(-0.5));
      gv[i] = riccati_step_c(gv[i], c, kx, kx * kx, T(0.5) * hs * (qa + ex[i]));
    }
  };
  auto full_step = [&](cpx<T>* gv, const node4<T>& pv, const node4<T>& cv, T s) {
    StepC<T> c;
    c.c2x = hq8 * (pv.dy + cv.dy);
    c.c2y = hq8 * (s * (pv.dx + cv.dx));
    c.U0x = T(-4) * c.c2x;
    c.U0y = T(4) * c.c2y;
    // (the product alone, rounded once: an fma keeps the compiler from
    // contracting it into the sums that riccati_steps forms with it)
    const T hq = fmaT(hqa, pv.a + cv.a, T(0));
    T ky[EPL];
    for (int i = 0; i < EPL; ++i) ky[i] = kReal ? fmaT(hh, ex[i], hq) : hq;
    riccati_steps<T, EPL, !kReal>(gv, c, kxi, kx2i, ky);
  };
  auto mid_step = [&](cpx<T>* gv, const node4<T>& pv, const node4<T>& cv) { full_step(gv, pv, cv, sd); };
  // a step of the other direction, from node cv back to node pv
  auto back_step = [&](cpx<T>* gv, const node4<T>& pv, const node4<T>& cv) { full_step(gv, pv, cv, -sd); };

  // slot of node j of the march, clamped to the segment's slots; unsigned
  // 32-bit offsets widen to the 64-bit address without a sign extension
  auto slot = [&](int j) { return static_cast<uint32_t>(DIR > 0 ? min(j, last) : max(last - j, 0)); };
  const node4<T>* const nseg = nodes + slot0;
  // spill of this segment, slot t at gseg[t * n_e]: the grain's array
  // (gmul = n_e) or a wave pair's own scratch (gmul = 0); this lane's entries
  // start at glane
  cpx<T>* const glane = gbase + slot0 * gmul + es;

  // ---- first half: start value, first partial step, nodes 0 .. n1 - 1
  cpx<T> g[EPL];
  node4<T> prev;
  if (live) {
    prev = nseg[slot(0)];
    {
      const int64_t tb = seg * 4;
      const double* tw = (DIR > 0 ? a.tap_start_w : a.tap_end_w) + tb;
      const int32_t* ts = (DIR > 0 ? a.tap_start_seg : a.tap_end_seg) + tb;
      const double wsum = tw[0] + tw[1] + tw[2] + tw[3];
      if (a.bc_valid && wsum > 0.0) {
        for (int i = 0; i < EPL; ++i) g[i] = mk(T(0), T(0));
        for (int c = 0; c < 4; ++c) {
          const T w = static_cast<T>(tw[c]);
          const cpx<T>* src = bc_prev + static_cast<int64_t>(ts[c]) * a.n_e_tot + a.e_off;
          for (int i = 0; i < EPL; ++i) {
            const cpx<T> v = src[es + i];
            g[i] = mk(g[i].x + w * v.x, g[i].y + w * v.y);
          }
        }
      } else {
        const T qa = q * prev.a;
        // (the real part from memory in every mode: a zero the compiler knows
        // would be shared by the energies and change which products it fuses)
        for (int i = 0; i < EPL; ++i) {
          const T er = static_cast<T>(a.eps[2 * (a.e_off + es + i)]);
          g[i] = bulk_root(qa + er, ey[i], sd * prev.dx, prev.dy);
        }
      }
    }
    // the partial step next to the start (the whole segment if n = 0)
    end_step(g, prev, static_cast<T>(DIR > 0 || n == 0 ? a.seg_hfirst[seg] : a.seg_hlast[seg]));
    // Slot values are loaded one step ahead, so the load overlaps a step.  A
    // node's value is stored at the start of the next step, beside that
    // step's load: the wait for the load then finds the store done too (a
    // store issued at the end of a step would be waited for right away).
    // Every lane stores all its EPL entries (a duplicate writes the value its
    // owner writes).
    if (n1 > 0) {
      node4<T> nxt = nseg[slot(1)];
      int j = 0;  // the node g stands at
      auto store_g = [&]() {
        cpx<T>* dst = glane + static_cast<int64_t>(slot(j)) * a.n_e;
        if (MODE != 2)
          for (int i = 0; i < EPL; ++i) dst[i] = g[i];
      };
      auto step = [&]() {
        const node4<T> cur = nxt;
        nxt = nseg[slot(j + 2)];
        mid_step(g, prev, cur);
        prev = cur;
        ++j;
      };
      // stored: node 0 and every second node counted back from n1 - 2
      store_g();
      if (!(n1 & 1)) step();
      while (j + 2 < n1) {
        step();
        store_g();
        step();
      }
    }
  }
  // ---- the waves of the pair meet: the other's first half is in the spill
  if (MODE != 2) __syncthreads();
  if (!live) return;

  // pole weights R_p of the lane's energies (0 for duplicates), kept in FP64:
  // the gap denominator holds them exactly, and rounding them to FP32 in
  // the node sums would bias every gap update the same way
  double rw[EPL];
  for (int i = 0; i < EPL; ++i)
    rw[i] = (MODE == 0 && own[i]) ? a.rp[a.e_off + es + i] : 0.0;

  // Per node and pole (Sec. II.A), with X = gamma gamma~ and I = 1/(1+X):
  //   f + conj f~ = -2 i pi [Re((gamma + gamma~) I) + i Im((gamma - gamma~) I)],
  //   Re g = pi Im((1-X)/(1+X)) = 2 pi Im I,
  //   (D* f + D f~) / (pi + i g) = i (D gamma~ - D* gamma)  since pi + i g = 2 pi I,
  // so the Eilenberger free-energy term needs no division.
  //
  // Node sums through LDS (MODE 0, G >= 8).  The wave's buffer holds two
  // nodes x four components x 64 lanes; slot b of component c of lane l is
  // lsum[b * 256 + c * 64 + l].  Lanes of one wave see each other's LDS
  // writes in issue order; the fences keep the compiler from moving the
  // accesses across each other.  Every lane of a group then takes one
  // (node, component) output and a block of 8 partials, and P = G / 8
  // neighbouring lanes finish it with quad moves.
  auto lds_reduce = [&](int64_t node0, int cnt) {
    const int l64 = threadIdx.x & 63;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    const int lp = lg - 3;  // log2 P
    const int o = lane >> lp, r = lane & ((1 << lp) - 1);
    const double2* src = reinterpret_cast<const double2*>(lsum + o * 64 + (l64 - lane));
    // partials of lanes 8 r .. 8 r + 7 of the group
    const double2 x0 = src[r << 2];
    double v = x0.x + x0.y;
    for (int j = 1; j < 4; ++j) {
      const double2 x = src[(r << 2) + j];
      v += x.x + x.y;
    }
    if (lp >= 1) v += dpp_f64<0xB1>(v);   // quad_perm [1,0,3,2]
    if (lp >= 2) v += dpp_f64<0x4E>(v);   // quad_perm [2,3,0,1]
    if (lp >= 3) v += dpp_f64<0x141>(v);  // row_half_mirror: lane 0 of 8 adds lane 7
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    // slot b = o >> 2 holds the b-th node of the pair; component o & 3
    if (r == 0 && (o >> 2) < cnt) a.node_out[(node0 + DIR * (o >> 2)) * 4 + (o & 3)] = a.twopi_tt * v;
  };
  // sums at one node from this wave's value g and the other direction's go;
  // k counts the nodes of the second half visited before this one (the same
  // for every group of the wave, since all groups start it together)
  auto node_sums = [&](int64_t node, const node4<T>& nv, const cpx<T>* go, int k) {
    if (MODE == 0) {
      double sfx, sfy, sg, si;
      if constexpr (sizeof(T) == 4) {
        // mixed precision: each pole's terms are formed from the FP32
        // marches, weighted by R_p and summed over poles in FP64
        for (int i = 0; i < EPL; ++i) {
          const cpx<T> gg = DIR > 0 ? g[i] : go[i], gt = DIR > 0 ? go[i] : g[i];
          const T xx = fmaT(gg.x, gt.x, -(gg.y * gt.y));
          const T xy = fmaT(gg.x, gt.y, gg.y * gt.x);
          const T dxr = T(1) + xx;
          // I = 1/(1+X) = (dxr - i xy) u with u = 1 / |1+X|^2
          const T u = drcp(fmaT(dxr, dxr, xy * xy));
          const T ix = dxr * u, iy = xy * u;  // I = ix - i iy
          const T sxs = gg.x + gt.x, sys = gg.y + gt.y;
          const T dxs = gg.x - gt.x, dys = gg.y - gt.y;
          const double tfx = static_cast<double>(fmaT(sxs, ix, sys * iy));     // Re((gamma + gamma~) I)
          const double tfy = static_cast<double>(fmaT(dys, ix, -(dxs * iy)));  // Im((gamma - gamma~) I)
          const double tg = static_cast<double>(iy);                           // -Im I
          const double ti = static_cast<double>(fmaT(nv.dx, dys, -(nv.dy * sxs)));  // Im(D* gamma - D gamma~)
          if (i == 0) {
            sfx = rw[0] * tfx;
            sfy = rw[0] * tfy;
            sg = -rw[0] * tg;
            si = rw[0] * ti;
          } else {
            sfx = __builtin_fma(rw[i], tfx, sfx);
            sfy = __builtin_fma(rw[i], tfy, sfy);
            sg = __builtin_fma(-rw[i], tg, sg);
            si = __builtin_fma(rw[i], ti, si);
          }
        }
      } else {
        T pfx = T(0), pfy = T(0), pg = T(0), p1 = T(0), p2 = T(0);
        for (int i = 0; i < EPL; ++i) {
          const cpx<T> gg = DIR > 0 ? g[i] : go[i], gt = DIR > 0 ? go[i] : g[i];
          const T xx = fmaT(gg.x, gt.x, -(gg.y * gt.y));
          const T xy = fmaT(gg.x, gt.y, gg.y * gt.x);
          const T dxr = T(1) + xx;
          // I = 1/(1+X) = (dxr - i xy) u / R with u = R / |1+X|^2 (R the pole weight)
          const T r = static_cast<T>(rw[i]);
          const T u = r * drcp(fmaT(dxr, dxr, xy * xy));
          const T sxs = gg.x + gt.x, sys = gg.y + gt.y;
          const T dxs = gg.x - gt.x, dys = gg.y - gt.y;
          pfx = fmaT(u, fmaT(sxs, dxr, sys * xy), pfx);     // R Re((gamma + gamma~) I)
          pfy = fmaT(u, fmaT(dys, dxr, -(dxs * xy)), pfy);  // R Im((gamma - gamma~) I)
          pg = fmaT(-u, xy, pg);                            // R Im I
          p1 = fmaT(r, dys, p1);
          p2 = fmaT(r, sxs, p2);
        }
        sfx = pfx;
        sfy = pfy;
        sg = pg;
        // Im(D* gamma - D gamma~) summed over the lane's poles
        si = fmaT(nv.dx, p1, -(nv.dy * p2));
      }
      // S_f = -2 i pi t~ (sfx + i sfy), S_g = 2 pi t~ sg, S_I = 2 pi t~ si
      if (G >= 8) {
        // the lane's four partials go to LDS, where the group sums them
        // when a pair of nodes is there (see the loop below)
        const int b = k & 1;
        double* w = lsum + b * 256 + (threadIdx.x & 63);
        w[0] = sfy;
        w[64] = -sfx;
        w[128] = sg;
        w[192] = si;
      } else if (G >= 4) {
        // lane q of the group (q < 4) ends with component q of the node's sums
        const double v = group_sum4_scatter(sfy, -sfx, sg, si, G, lane);
        if (lane < 4) a.node_out[node * 4 + scatter_index(lane)] = a.twopi_tt * v;
      } else {
        const double ox = group_sum(sfy, G), oy = group_sum(sfx, G);
        const double oz = group_sum(sg, G), ow = group_sum(si, G);
        if (lane == 0) {
          double4 o;
          o.x = a.twopi_tt * ox;
          o.y = -a.twopi_tt * oy;
          o.z = a.twopi_tt * oz;
          o.w = a.twopi_tt * ow;
          reinterpret_cast<double4*>(a.node_out)[node] = o;
        }
      }
    } else {
      // MODE 1: N/N_F = -Im g / pi = Re((1-X)/(1+X)) = 2 Re I - 1 per energy;
      // MODE 3: (1-X)/(1+X) = 2 I - 1 per energy, complex (g = -i pi times it)
      T* dst = ebuf + (MODE == 1 ? 1 : 2) * (node * a.n_e + es);
      for (int i = 0; i < EPL; ++i) {
        if (!own[i]) continue;
        const cpx<T> gg = DIR > 0 ? g[i] : go[i], gt = DIR > 0 ? go[i] : g[i];
        const T xx = fmaT(gg.x, gt.x, -(gg.y * gt.y));
        const T xy = fmaT(gg.x, gt.y, gg.y * gt.x);
        const T dxr = T(1) + xx;
        const T ri = drcp(fmaT(dxr, dxr, xy * xy));
        if (MODE == 1) {
          dst[i] = fmaT(T(2) * dxr, ri, T(-1));
        } else {
          dst[2 * i] = fmaT(T(2) * dxr, ri, T(-1));
          dst[2 * i + 1] = T(-2) * xy * ri;
        }
      }
    }
  };
  // ---- second half: nodes n1 .. n - 1 in pairs, slot values and the other
  // direction's values read one pair ahead (those come back from HBM)
  if (MODE != 2) {
    int j = n1;
    node4<T> vA = nseg[slot(j)], vB = nseg[slot(j + 1)];
    cpx<T> oB[EPL];
    auto load_row = [&](cpx<T>* gv, int jj) {
      const cpx<T>* row = glane + static_cast<int64_t>(slot(jj)) * a.n_e;
      for (int i = 0; i < EPL; ++i) gv[i] = row[i];
    };
    load_row(oB, j + 1);
    for (; j + 1 < n; j += 2) {
      const node4<T> cA = vA, cB = vB;
      cpx<T> gA[EPL], gB[EPL];
      for (int i = 0; i < EPL; ++i) gA[i] = gB[i] = oB[i];
      // The sums of the pair before this one: reduced and stored here, ahead
      // of the loads for the next pair, so that the wait for those loads
      // finds this store done (issued at the end of a turn, its latency
      // would be waited for at the start of the next).
      if (MODE == 0 && G >= 8 && j > n1) lds_reduce(slot0 + slot(j - 2), 2);
      vA = nseg[slot(j + 2)];
      vB = nseg[slot(j + 3)];
      load_row(oB, j + 3);
      vmem_order();
      mid_step(g, prev, cA);
      back_step(gA, cA, cB);  // node j was not stored: one step from node j + 1
      node_sums(slot0 + slot(j), cA, gA, 0);
      mid_step(g, cA, cB);
      node_sums(slot0 + slot(j + 1), cB, gB, 1);
      prev = cB;
    }
    if (MODE == 0 && G >= 8 && j > n1) lds_reduce(slot0 + slot(j - 2), 2);
    if (j < n) {  // an odd count leaves the last node alone (the other direction's first, always stored)
      if (n > 1) mid_step(g, prev, vA);  // n = 1: the first partial step already reached the node
      node_sums(slot0 + slot(j), vA, oB, 0);
      prev = vA;
      if (MODE == 0 && G >= 8) lds_reduce(slot0 + slot(j), 1);
    }
  }
  // the partial step to the far end
  if (n > 0) end_step(g, prev, static_cast<T>(DIR > 0 ? a.seg_hlast[seg] : a.seg_hfirst[seg]));
  // end values for the next sweep (the LDOS output pass writes them only
  // when iterating to convergence: bc_next given)
  if (MODE == 0 || MODE == 2 || (MODE == 1 && bc_next)) {
    cpx<T>* dst = bc_next + seg * a.n_e_tot + a.e_off + es;
    for (int i = 0; i < EPL; ++i)
      if (own[i]) dst[i] = g[i];
    // gamma~ along a line is the conjugate of gamma along the reversed line
    // (even order parameter), at a real energy e of gamma at -e: the end
    // values of the upper angle of a pair
    if (MODE != 1 && a.mirror) {
      cpx<T>* mdst = bc_mirror + static_cast<int64_t>(a.mirror[seg]) * a.n_e_tot;
      for (int i = 0; i < EPL; ++i) {
        const int e = a.e_off + es + i;
        if (own[i]) mdst[MODE == 2 && a.partner ? a.partner[e] : e] = mk(g[i].x, -g[i].y);
      }
    }
  }
}

// one bundle of 64/G segments by the two waves of a 128-thread block
template <typename T, int EPL, int MODE>
__device__ __forceinline__ void sweep_bundle(const SweepArgs& a, int64_t wseg0, int G, int lg, const SweepBufs& b,
                                             cpx<T>* gbase, int64_t gmul, double* lsum) {
  const int l64 = threadIdx.x & 63;
  const int dir = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
  const int64_t wseg = wseg0 + (l64 >> lg);
  const bool live = wseg < a.nseg;
  const int lane = l64 & (G - 1);
  const node4<T>* nodes = static_cast<const node4<T>*>(b.nodes);
  T* ebuf = static_cast<T*>(b.ebuf);
  // (the branch is uniform over each wave, and each wave meets the one barrier once)
  if (dir == 0)
    sweep_march<T, EPL, MODE, 1>(a, live, wseg, lane, G, lg, nodes, static_cast<const cpx<T>*>(b.bc_g_prev),
                                 static_cast<cpx<T>*>(b.bc_g_next), static_cast<cpx<T>*>(b.bc_gt_next), gbase, gmul,
                                 ebuf, lsum);
  else
    sweep_march<T, EPL, MODE, -1>(a, live, wseg, lane, G, lg, nodes, static_cast<const cpx<T>*>(b.bc_gt_prev),
                                  static_cast<cpx<T>*>(b.bc_gt_next), static_cast<cpx<T>*>(b.bc_g_next), gbase, gmul,
                                  ebuf, lsum);
}

template <typename T, int EPL, int MODE>
__global__ void __launch_bounds__(128)
sweep_kernel(SweepArgs a, SweepBufs b) {
  double* lsum = nullptr;
  if constexpr (MODE == 0) {
    __shared__ double red[2 * 512];  // two nodes x four sums x 64 lanes per wave
    lsum = red + (threadIdx.x >> 6) * 512;
  }
  cpx<T>* const gbuf = static_cast<cpx<T>*>(b.gbuf);
  // The launch order is longest first.  In a launch that fills the device's
  // wave slots a few times, the longest segments finish last; the first
  // nlong of them march with twice the lanes and half the energies per lane,
  // so they finish in about half the time.  The split falls on a wave
  // boundary (nlong * 2G is a multiple of 64), so each wave takes one shape.
  int64_t w = blockIdx.x, first = 0;
  if constexpr (MODE == 0 && EPL % 2 == 0) {
    first = a.nlong;
    const int64_t wl = (a.nlong << (a.log2g + 1)) >> 6;
    if (w < wl) {
      sweep_bundle<T, EPL / 2, MODE>(a, w << (5 - a.log2g), 2 * a.G, a.log2g + 1, b, gbuf, a.n_e, lsum);
      return;
    }
    w -= wl;
  }
  sweep_bundle<T, EPL, MODE>(a, first + (w << (6 - a.log2g)), a.G, a.log2g, b, gbuf, a.n_e, lsum);
}

// Batched grains: one persistent launch.  Every block (a wave pair) pulls
// tiles (a grain and a bundle of 64/G of its segments) from a queue sorted by
// cost until the queue is empty; every block reaches that exit.  The spill of
// a tile lives only between the two halves of its marches, so each block
// keeps it in its own slice of `spill` (wave_elems records; segment k of the
// tile at k * maxn * n_e), reused tile after tile: the spill memory is set by
// the resident blocks, not by the number or size of the grains.
template <typename T, int EPL>
__global__ void __launch_bounds__(128)
batch_sweep_kernel(const BatchGrainDev* __restrict__ grains,
                                                          const int2* __restrict__ tiles, int ntiles,
                                                          int* __restrict__ counter, cpx<T>* __restrict__ spill,
                                                          int64_t wave_elems) {
  const int l64 = threadIdx.x & 63;
  cpx<T>* const wspill = spill + static_cast<int64_t>(blockIdx.x) * wave_elems;
  __shared__ double red[2 * 512];  // node-sum exchange, two nodes x four sums x 64 lanes per wave
  __shared__ int next;
  while (true) {
    if (threadIdx.x == 0) next = atomicAdd(counter, 1);
    __syncthreads();
    // the tile index is uniform: the grain's arguments become scalar loads
    const int t = __builtin_amdgcn_readfirstlane(next);
    __syncthreads();  // (read by both waves before the next tile overwrites it)
    if (t >= ntiles) break;
    const int2 tile = tiles[t];
    const BatchGrainDev& gd = grains[tile.x];
    const int lg = gd.a.log2g;
    sweep_bundle<T, EPL, 0>(gd.a, tile.y, gd.a.G, lg, gd.b,
                            wspill + static_cast<int64_t>(l64 >> lg) * gd.a.maxn * gd.a.n_e, 0,
                            red + (threadIdx.x >> 6) * 512);
  }
}

// (curl A)_z by central differences, one-sided at the grid's edges
__device__ __forceinline__ double curl_at(const double* __restrict__ A, int64_t c, int nx, int ny, double h) {
  const int i = static_cast<int>(c % nx), j = static_cast<int>(c / nx);
  const double* ax = A;
  const double* ay = A + static_cast<int64_t>(nx) * ny;
  double dyx, dxy;  // d_x A_y, d_y A_x
  if (i == 0)
    dyx = (ay[c + 1] - ay[c]) / h;
  else if (i == nx - 1)
    dyx = (ay[c] - ay[c - 1]) / h;
  else
    dyx = (ay[c + 1] - ay[c - 1]) / (2 * h);
  if (j == 0)
    dxy = (ax[c + nx] - ax[c]) / h;
  else if (j == ny - 1)
    dxy = (ax[c] - ax[c - nx]) / h;
  else
    dxy = (ax[c + nx] - ax[c - nx]) / (2 * h);
  return dyx - dxy;
}

// --------------------------------------------------------------------------
// rotate back + angle sums + gap / current / free energy
// --------------------------------------------------------------------------
// A block of W waves shares 64 grain cells: wave w takes the angles
// k = w, w + W, ... for all of them, so each load of a wave gathers
// the lattice corners of 64 neighbouring cells at one angle; the waves'
// partial angle sums meet in LDS.
constexpr int kBackFields = 12;  // 2 x (up to 4 components) + jx, jy, I, <|Delta|^2>

// Bilinear weights and slots of a cell's corner record ix on one angle's
// lattice; corners that are not nodes read one of the record's that is, with
// weight 0, so the four gathers issue together and only nodes are read.
// Returns the factor that renormalises the weights.
__device__ __forceinline__ double back_weights(int4 ix, double epx, double epy, double rx, double ry, double h,
                                               double half, double w[4], int sl[4]) {
  // lattice coordinates (line u, node v) of the cell centre
  const double u = rn_lattice(rx, epy, ry, -epx, h, half);
  const double v = rn_lattice(rx, epx, ry, epy, h, half);
  const double wu = u - __builtin_floor(u), wv = v - __builtin_floor(v);
  w[0] = (1 - wu) * (1 - wv);
  w[1] = wu * (1 - wv);
  w[2] = (1 - wu) * wv;
  w[3] = wu * wv;
  sl[0] = ix.x;
  sl[1] = ix.y;
  sl[2] = ix.z;
  sl[3] = ix.w;
  if (ix.y == -2) {  // no lattice corner is a node: the nearest node alone
    w[0] = 1.0;
    w[1] = w[2] = w[3] = 0.0;
  }
  const int any = record_node(ix.x, ix.y, ix.z, ix.w);
  double tot = 0.0;
  for (int q = 0; q < 4; ++q) {
    if (sl[q] < 0) {
      w[q] = 0.0;
      sl[q] = any;
    }
    tot += w[q];
  }
  return (ix.x | ix.y | ix.z | ix.w) < 0 ? 1.0 / tot : 1.0;
}

// NC = 1: one order-parameter component (its arrays in fixed registers);
// NC = 4: a.ncomp <= 4 components
// UPDATE: the Picard step of size one in place (Delta += Delta_new - Delta)
// instead of Delta_new: a cell's Delta is read by the cell's own thread only
template <int NC, int W, bool UPDATE>
__device__ __forceinline__ void rotate_back_block(const BackArgs& a, int64_t block,
                                                  double (*__restrict__ part)[kBackFields][64]) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int64_t c = block * 64 + lane;
  const bool live = c < a.ncg;
  const int cell = live ? a.grain_cells[c] : 0;
  constexpr int MAXC = NC;
  const int ncomp = NC == 1 ? 1 : a.ncomp;
  double nx_[MAXC], ny_[MAXC], dx_[MAXC], dy_[MAXC];
  for (int g = 0; g < ncomp; ++g) {
    nx_[g] = 0.0;
    ny_[g] = 0.0;
    dx_[g] = a.delta[2 * (static_cast<int64_t>(g) * a.ncell + cell)];
    dy_[g] = a.delta[2 * (static_cast<int64_t>(g) * a.ncell + cell) + 1];
  }
  // cell centre relative to the grid centre, as the plan forms it
  const double rx = rn_cell_offset(a.x0, static_cast<double>(cell % a.nx), a.h, a.cx);
  const double ry = rn_cell_offset(a.y0, static_cast<double>(cell / a.nx), a.h, a.cy);
  const double4* nsum = reinterpret_cast<const double4*>(a.node_out);
  double jx = 0.0, jy = 0.0, icell = 0.0, d2avg = 0.0;
  // angle kk's share of the sums from the node sums gathered at its corners
  // (sgn: the sign of S_g, -1 for the reversed direction of a pair)
  auto add_angle = [&](int kk, double cfx, double cfy, double cg, double ci) {
    const double wk = a.wk[kk];
    double dkx = 0.0, dky = 0.0;
    for (int g = 0; g < ncomp; ++g) {
      const double ex = a.eta[2 * (g * a.n_theta + kk)], ey = a.eta[2 * (g * a.n_theta + kk) + 1];
      const double px = wk * ex, py = -wk * ey;  // wk conj(eta)
      nx_[g] += px * cfx - py * cfy;
      ny_[g] += px * cfy + py * cfx;
      dkx += ex * dx_[g] - ey * dy_[g];
      dky += ex * dy_[g] + ey * dx_[g];
    }
    jx += a.four_q * wk * a.cosk[kk] * cg;
    jy += a.four_q * wk * a.sink[kk] * cg;
    icell += wk * ci;
    d2avg += wk * (dkx * dkx + dky * dky);
  };
  // with pair_fold each gather of a lower angle serves its upper angle too
  const int kend = a.pair_fold ? a.pair_k0 : a.n_theta;
  // the corner record of the wave's next angle is loaded one iteration
  // ahead, so only the node-sum gathers wait in each iteration
  int k = live ? wv : kend;
  int4 ixn = make_int4(0, 0, 0, 0);
  if (k < kend) ixn = a.rb4[static_cast<int64_t>(k) * a.ncg + c];
  for (; k < kend; k += W) {
    const int4 ix = ixn;
    if (k + W < kend) ixn = a.rb4[static_cast<int64_t>(k + W) * a.ncg + c];
    double w[4];
    int sl[4];
    const double rt = back_weights(ix, a.cosk[k], a.sink[k], rx, ry, a.h, a.half, w, sl);
    double cfx = 0.0, cfy = 0.0, cg = 0.0, ci = 0.0;
    for (int qd = 0; qd < 4; ++qd) {
      const double4 vv = nsum[sl[qd]];
      const double wq = w[qd] * rt;
      cfx += vv.x * wq;
      cfy += vv.y * wq;
      cg += vv.z * wq;
      ci += vv.w * wq;
    }
    // S_g of the reversed direction changes sign; S_f and S_I do not
    add_angle(k, cfx, cfy, k >= a.pair_k0 ? -cg : cg, ci);
    if (a.pair_fold) add_angle(k + a.pair_k0, cfx, cfy, -cg, ci);
  }
  if (wv > 0) {
    double* p = &part[wv - 1][0][lane];
    for (int g = 0; g < ncomp; ++g) {
      p[64 * (2 * g)] = nx_[g];
      p[64 * (2 * g + 1)] = ny_[g];
    }
    p[64 * 8] = jx;
    p[64 * 9] = jy;
    p[64 * 10] = icell;
    p[64 * 11] = d2avg;
  }
  __syncthreads();
  if (wv > 0) return;
  double om = 0.0;
  if (live) {
    for (int w = 0; w < W - 1; ++w) {
      const double* p = &part[w][0][lane];
      for (int g = 0; g < ncomp; ++g) {
        nx_[g] += p[64 * (2 * g)];
        ny_[g] += p[64 * (2 * g + 1)];
      }
      jx += p[64 * 8];
      jy += p[64 * 9];
      icell += p[64 * 10];
      d2avg += p[64 * 11];
    }
    for (int g = 0; g < ncomp; ++g) {
      const double vx = nx_[g] / a.den[g], vy = ny_[g] / a.den[g];
      double* const o = a.delta_new + 2 * (static_cast<int64_t>(g) * a.ncell + cell);
      o[0] = UPDATE ? dx_[g] + (vx - dx_[g]) : vx;
      o[1] = UPDATE ? dy_[g] + (vy - dy_[g]) : vy;
      om += (dx_[g] * dx_[g] + dy_[g] * dy_[g]) * a.logt[g];
    }
    om += a.twopi_rz * d2avg - icell;
    a.j[cell] = jx;
    a.j[a.ncell + cell] = jy;
    if (a.omega) a.omega[cell] = om;
    a.omega_cell[c] = om;
  }
  if (a.sums) {
    const double so = group_sum(om, 64), sx = group_sum(live ? jx : 0.0, 64), sy = group_sum(live ? jy : 0.0, 64);
    if (lane == 0) {
      a.sums[block] = so;
      a.sums[2 * a.nparts + block] = sx;
      a.sums[3 * a.nparts + block] = sy;
    }
  }
}

template <int NC, int W>
__global__ void __launch_bounds__(64 * W) rotate_back_kernel(BackArgs a) {
  __shared__ double part[W - 1][kBackFields][64];
  const int nblk = static_cast<int>((a.ncg + 63) / 64);
  if (static_cast<int>(blockIdx.x) >= nblk) {  // zeros off the grain, partial sums over the grid
    const int b = blockIdx.x - nblk;
    const int64_t cell = static_cast<int64_t>(b) * (64 * W) + threadIdx.x;
    if (a.sums) {
      // (every block of these leaves its share of the entries without one at zero)
      const int others = gridDim.x - nblk;
      for (int i = static_cast<int>(cell); i < a.nparts; i += others * 64 * W) {
        for (int r = 0; r < 4; ++r)
          if (i >= (r == 1 ? others : nblk)) a.sums[r * a.nparts + i] = 0.0;
      }
      double v = 0.0;
      if (a.curl_A && cell < a.ncell) {
        v = curl_at(a.curl_A, cell, a.nx, static_cast<int>(a.ncell / a.nx), a.h);
        v *= v;
      }
      v = group_sum(v, 64);
      double* const sh = &part[0][0][0];
      if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
      __syncthreads();
      if (threadIdx.x == 0) {
        for (int w = 1; w < W; ++w) v += sh[w];
        a.sums[a.nparts + b] = v;
      }
    }
    if (!a.zero_mask || cell >= a.ncell || a.zero_mask[cell]) return;
    for (int g = 0; g < a.ncomp; ++g)
      reinterpret_cast<double2*>(a.delta_new)[g * a.ncell + cell] = make_double2(0.0, 0.0);
    a.j[cell] = 0.0;
    a.j[a.ncell + cell] = 0.0;
    if (a.omega) a.omega[cell] = 0.0;
    return;
  }
  // each XCD takes a contiguous band of grain cells: neighbouring cells share
  // lattice corners, which then meet in the same L2
  rotate_back_block<NC, W, false>(a, xcd_block(blockIdx.x, nblk), part);
}

// Batched grains: the passes around the sweep, every grain's blocks in one
// launch (tiles: the grain and the block of the grain).  A launch per grain
// left most of the device idle and cost its latency each time: eight grains
// of 64 x 64 to 176 x 176 took 45 launches and 290 us an iteration beside
// the sweeps, 66 us now.
template <typename T>
__global__ void __launch_bounds__(256) batch_pack_kernel(const BatchGrainDev* __restrict__ grains,
                                                         const int2* __restrict__ tiles) {
  const int2 t = tiles[blockIdx.x];
  const BatchGrainDev& gd = grains[__builtin_amdgcn_readfirstlane(t.x)];
  pack_cell<T>(gd.ia, static_cast<int64_t>(t.y) * 256 + threadIdx.x, static_cast<cell4<T>*>(gd.cells));
}
// (one or several components: without or with the packed cells)
template <typename T>
__global__ void __launch_bounds__(256) batch_interp_kernel(const BatchGrainDev* __restrict__ grains,
                                                           const int2* __restrict__ tiles,
                                                           int* __restrict__ counters) {
  // (the tile counters of the sweeps that follow)
  if (blockIdx.x == 0 && threadIdx.x < kBatchCounters) counters[threadIdx.x] = 0;
  const int2 t = tiles[blockIdx.x];
  const BatchGrainDev& gd = grains[__builtin_amdgcn_readfirstlane(t.x)];
  node4<T>* nodes = static_cast<node4<T>*>(const_cast<void*>(gd.b.nodes));
  if (gd.cells)
    interp1_block<T, true>(gd.ia, __builtin_amdgcn_readfirstlane(t.y), static_cast<const cell4<T>*>(gd.cells), nodes);
  else
    interp_slot<T>(gd.ia, static_cast<int64_t>(t.y) * 256 + threadIdx.x, nodes);
}
template <int NC, int W>
__global__ void __launch_bounds__(64 * W) batch_back_kernel(const BatchGrainDev* __restrict__ grains,
                                                            const int2* __restrict__ tiles) {
  __shared__ double part[W - 1][kBackFields][64];
  const int2 t = tiles[xcd_block(blockIdx.x, gridDim.x)];
  const BatchGrainDev& gd = grains[__builtin_amdgcn_readfirstlane(t.x)];
  rotate_back_block<NC, W, true>(gd.ra, __builtin_amdgcn_readfirstlane(t.y), part);
}

// Fields of a batched grain: Delta on the grain and zero off it, A as given
// or (no screening) zero
__global__ void __launch_bounds__(256) batch_set_kernel(const double2* __restrict__ delta,
                                                        const double* __restrict__ A,
                                                        const uint8_t* __restrict__ mask, int64_t ncell, int ncomp,
                                                        double2* __restrict__ delta_out, double* __restrict__ A_out) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= ncell) return;
  for (int g = 0; g < ncomp; ++g)
    delta_out[g * ncell + i] = mask[i] ? delta[g * ncell + i] : make_double2(0.0, 0.0);
  A_out[i] = A ? A[i] : 0.0;
  A_out[ncell + i] = A ? A[ncell + i] : 0.0;
}

// Rotate-back and angle sums of the per-node, per-energy values of sweep mode
// 1 (LDOS) or 3 (CPLX: -i pi times the average of a complex value).  A row of
// a node holds M = n_e (CPLX: 2 n_e) reals; a thread takes V consecutive ones
// (16 B loads where the row length allows) of one cell, tpc threads a cell.
// The corner weights of up to sixteen angles are formed at a time, each by one
// thread, from the 16 B corner records that the sweep's rotate-back reads, and
// shared through LDS.  The sums meet in LDS too, so that a lower angle's sum
// reaches its partner energy and the output, energy by energy, is written
// along the cells.
// Bound by VALU (a conversion and an FP64 fma per corner and energy) and the
// gathers of the rows through L2.  With one thread per (cell, energy), stored
// indices and weights (48 B per angle and thread), and the partner energy
// gathered as well, the kernel waited on those loads: 926 us for 43264 cells x
// 64 angle pairs x 64 energies; 247 us with a thread's own weights, some 40 of
// its 100 instructions an angle, and 218 us shared (185 and 149 us for 22500
// cells x 128 angles).
template <typename T, int V>
struct __attribute__((aligned(V * sizeof(T) < 16 ? V * sizeof(T) : 16))) vecn {
  T v[V];
};
template <typename T, int V, bool CPLX>
__global__ void __launch_bounds__(256) ldos_back_kernel(LdosBackArgs a, const T* __restrict__ ebuf, int tpc, int cpb,
                                                        int kpb) {
  extern __shared__ double sums[];
  const int M = (CPLX ? 2 : 1) * a.n_e;
  const int lc = static_cast<int>(threadIdx.x) / tpc, te = static_cast<int>(threadIdx.x) - lc * tpc;
  const int mbase = static_cast<int>(blockIdx.y) * tpc * V, m0 = mbase + te * V;
  const int64_t c0 = xcd_block(blockIdx.x, gridDim.x) * cpb, c = c0 + lc;
  const bool fold = a.fold_k0 > 0;
  const int width = tpc * V, pitch = width + 1;
  double acc[V], accp[V];
  for (int i = 0; i < V; ++i) acc[i] = accp[i] = 0.0;
  // corner records of kpb angles x cpb cells, one thread each, read by the
  // threads of the cell
  double2* const w01 = reinterpret_cast<double2*>(sums);
  double2* const w23 = w01 + kpb * cpb;
  int4* const rows = reinterpret_cast<int4*>(w23 + kpb * cpb);
  const bool live = lc < cpb && c < a.ncg && m0 < M;
  // with fold_k0 each lower angle's corners serve its upper angle too, at
  // the partner energy (N of the reversed direction at e is N at -e)
  const int kend = fold ? a.fold_k0 : a.n_theta;
  for (int k0 = 0; k0 < kend; k0 += kpb) {
    const int nk = min(kpb, kend - k0);
    if (k0 > 0) __syncthreads();  // (the records before these are read)
    for (int t = threadIdx.x; t < nk * cpb; t += 256) {
      const int kk = t / cpb, k = k0 + kk;
      const int64_t cc = c0 + t - kk * cpb;
      if (cc >= a.ncg) continue;
      const int cell = a.grain_cells[cc];
      const double rx = rn_cell_offset(a.x0, static_cast<double>(cell % a.nx), a.h, a.cx);
      const double ry = rn_cell_offset(a.y0, static_cast<double>(cell / a.nx), a.h, a.cy);
      double w[4];
      int sl[4];
      const double rt = back_weights(a.rb4[static_cast<int64_t>(k) * a.ncg + cc], a.cosk[k], a.sink[k], rx, ry, a.h,
                                     a.half, w, sl);
      w01[t] = make_double2(w[0] * rt, w[1] * rt);
      w23[t] = make_double2(w[2] * rt, w[3] * rt);
      rows[t] = make_int4(sl[0], sl[1], sl[2], sl[3]);
    }
    __syncthreads();
    if (!live) continue;
    for (int kk = 0; kk < nk; ++kk) {
      const double2 wa = w01[kk * cpb + lc], wb = w23[kk * cpb + lc];
      const int4 r = rows[kk * cpb + lc];
      const double w[4] = {wa.x, wa.y, wb.x, wb.y};
      const int sl[4] = {r.x, r.y, r.z, r.w};
      vecn<T, V> x[4];
      for (int q = 0; q < 4; ++q)
        x[q] = *reinterpret_cast<const vecn<T, V>*>(ebuf + static_cast<int64_t>(sl[q]) * M + m0);
      const double wk = a.wk[k0 + kk], wp = fold ? a.wk[k0 + kk + a.fold_k0] : 0.0;
      for (int i = 0; i < V; ++i) {
        double v = 0.0;
        for (int q = 0; q < 4; ++q) v += static_cast<double>(x[q].v[i]) * w[q];
        acc[i] += wk * v;
        if (fold) accp[i] += wp * v;
      }
    }
  }
  __syncthreads();  // (the sums take the records' place)
  if (lc < cpb)
    for (int i = 0; i < V; ++i) {
      sums[lc * pitch + te * V + i] = acc[i];
      if (fold) sums[(cpb + lc) * pitch + te * V + i] = accp[i];
    }
  __syncthreads();
  const int ne = (CPLX ? width / 2 : width);  // energies of this block
  for (int t = threadIdx.x; t < cpb * ne; t += 256) {
    const int le = t / cpb, l = t - le * cpb;
    const int e = (CPLX ? mbase / 2 : mbase) + le;
    if (c0 + l >= a.ncg || e >= a.n_e) continue;
    const int64_t cell = a.grain_cells[c0 + l];
    if constexpr (CPLX) {
      const double pi = 3.14159265358979323846;
      double* o = a.out + 2 * (static_cast<int64_t>(a.e_off + e) * a.ncell + cell);
      o[0] = pi * sums[l * pitch + 2 * le + 1];  // -i pi (re + i im)
      o[1] = -pi * sums[l * pitch + 2 * le];
    } else {
      double v = sums[l * pitch + le];
      if (fold) v += sums[(cpb + l) * pitch + (a.e_partner[a.e_off + e] - a.e_off)];
      const int64_t eo = a.e_map ? a.e_map[a.e_off + e] : a.e_off + e;
      a.out[eo * a.ncell + cell] = v;
    }
  }
}

// --------------------------------------------------------------------------
// grid helpers: zero fill, curl + magnetic energy, block reductions
// --------------------------------------------------------------------------
__global__ void fill_kernel(double* __restrict__ p, int64_t n, double v) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

__global__ void __launch_bounds__(256) curl_kernel(const double* __restrict__ A, double* __restrict__ B,
                                                   int nx, int ny, double h) {
  const int64_t c = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (c < static_cast<int64_t>(nx) * ny) B[c] = curl_at(A, c, nx, ny, h);
}

// Block partial sums: kind 0 of x (gathered through idx when given), kind 1
// of the square of curl A (x = A), formed where it is summed.  One partial
// per block written to part[blockIdx.x]; the host adds them in order.
// Up to two sums per launch: blockIdx.y picks the row (BlockSumRow r0, r1);
// each row's partials are those a launch of its own would give.
__global__ void __launch_bounds__(256) block_sum_kernel(BlockSumRow r0, BlockSumRow r1) {
  const BlockSumRow& r = blockIdx.y == 0 ? r0 : r1;
  __shared__ double sh[256];
  double acc = 0.0;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < r.n;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    if (r.mode == 1) {
      const double v = curl_at(r.x, i, r.nx, r.ny, r.h);
      acc += v * v;
    } else {
      acc += r.x[r.idx ? r.idx[i] : i];
    }
  }
  sh[threadIdx.x] = acc;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) r.part[blockIdx.x] = sh[0];
}

// Block partials to pinned host memory, visible there when the stream has been
// waited for.  A launch: as a copy call these few KB took some 8 us more (sweep of
// the 32 x 32 disc 59 -> 50 us, ten iterations on 40 x 40 983 -> 850 us).
__global__ void __launch_bounds__(256) parts_to_host_kernel(const double* __restrict__ part, int n,
                                                            double* __restrict__ host) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) host[i] = part[i];
}

// Luttinger-Ward free energy (Sec. II): the propagator term at one
// coupling lambda, 2 sum_G den_G Re(conj(Delta_G) Delta_new_G[lambda Delta])
// with den_G the gap-equation denominator, weighted into acc per grain cell
__global__ void __launch_bounds__(256) lw_accumulate_kernel(const double* __restrict__ delta,
                                                            const double* __restrict__ dnew,
                                                            const int32_t* __restrict__ grain_cells, int64_t ncg,
                                                            int ncomp, int64_t ncell, const double* __restrict__ den,
                                                            double w, int first, double* __restrict__ acc) {
  const int64_t c = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (c >= ncg) return;
  const int64_t cell = grain_cells[c];
  double v = 0.0;
  for (int g = 0; g < ncomp; ++g) {
    const int64_t o = 2 * (static_cast<int64_t>(g) * ncell + cell);
    v += den[g] * (delta[o] * dnew[o] + delta[o + 1] * dnew[o + 1]);
  }
  v *= 2.0 * w;
  acc[c] = first ? v : acc[c] + v;
}

// The terms of the free-energy density before the propagator term,
// sum_G |Delta_G|^2 ln(t / t_c,G) + 2 pi sum_p (R_p / z_p) <|Delta(p)|^2>,
// minus the lambda integral of the propagator term
__global__ void __launch_bounds__(256) lw_finish_kernel(const double* __restrict__ delta,
                                                        const int32_t* __restrict__ grain_cells, int64_t ncg,
                                                        int ncomp, int64_t ncell, int n_theta,
                                                        const double* __restrict__ eta, const double* __restrict__ wk,
                                                        const double* __restrict__ logt, double twopi_rz,
                                                        const double* __restrict__ acc,
                                                        double* __restrict__ omega_cell, double* __restrict__ omega) {
  const int64_t c = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (c >= ncg) return;
  const int64_t cell = grain_cells[c];
  double dx[4], dy[4], base = 0.0;
  for (int g = 0; g < ncomp; ++g) {
    dx[g] = delta[2 * (static_cast<int64_t>(g) * ncell + cell)];
    dy[g] = delta[2 * (static_cast<int64_t>(g) * ncell + cell) + 1];
    base += (dx[g] * dx[g] + dy[g] * dy[g]) * logt[g];
  }
  double d2 = 0.0;
  for (int k = 0; k < n_theta; ++k) {
    double px = 0.0, py = 0.0;
    for (int g = 0; g < ncomp; ++g) {
      const double ex = eta[2 * (g * n_theta + k)], ey = eta[2 * (g * n_theta + k) + 1];
      px += ex * dx[g] - ey * dy[g];
      py += ex * dy[g] + ey * dx[g];
    }
    d2 += wk[k] * (px * px + py * py);
  }
  const double om = base + twopi_rz * d2 - acc[c];
  omega_cell[c] = om;
  if (omega) omega[cell] = om;
}

__global__ void __launch_bounds__(256) scale_kernel(const double* __restrict__ x, double s, int64_t n,
                                                    double* __restrict__ y) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) y[i] = s * x[i];
}

// CongAcc (App. E): dot products m.m, m.d, d.d of component comp of x, with
// d = xnew - xold and m the component's moving average.
__device__ __forceinline__ void congacc_dots_block(const CongFields& f, int comp, double (*__restrict__ sm)[256],
                                                   double* __restrict__ part) {
  const int nd = 2 * f.ncomp;
  const bool in_a = comp >= nd;  // components 2 G + (0 re, 1 im) of Delta, then A_x, A_y
  const int64_t n = in_a ? f.ncell : f.ncg, base = (in_a ? comp - nd : comp / 2) * f.ncell;
  const int stride = in_a ? 1 : 2, c = in_a ? 0 : comp & 1;
  const int32_t* idx = in_a ? nullptr : f.grain_cells;
  const double *xnew = in_a ? f.anew : f.dnew, *xold = in_a ? f.a : f.delta, *m = in_a ? f.ma : f.md;
  double a0 = 0.0, a1 = 0.0, a2 = 0.0;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    const int64_t k = (base + (idx ? idx[i] : i)) * stride + c;
    const double d = xnew[k] - xold[k], mv = m[k];
    a0 += mv * mv;
    a1 += mv * d;
    a2 += d * d;
  }
  sm[0][threadIdx.x] = a0;
  sm[1][threadIdx.x] = a1;
  sm[2][threadIdx.x] = a2;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w)
      for (int j = 0; j < 3; ++j) sm[j][threadIdx.x] += sm[j][threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0)
    for (int j = 0; j < 3; ++j) part[3 * (static_cast<int64_t>(comp) * gridDim.x + blockIdx.x) + j] = sm[j][0];
}

// Partial p-norms of (new - old) and of old over `n` elements of `stride`
// doubles each (stride 2: complex modulus).  p = 1, 2, or 0 (max).
// Elements may be gathered through idx (grain cells) when idx != nullptr,
// for `nrep` consecutive fields of `field_stride` elements.
// nf (up to three) independent fields per launch, picked by blockIdx.y, and
// after them the CongAcc dot products of every component
__global__ void __launch_bounds__(256) diff_norm_kernel(int nf, DiffNormArgs a0, DiffNormArgs a1, DiffNormArgs a2,
                                                        CongFields f, double* __restrict__ cong_part) {
  __shared__ double sm[3][256];
  if (static_cast<int>(blockIdx.y) >= nf) {
    congacc_dots_block(f, blockIdx.y - nf, sm, cong_part);
    return;
  }
  const DiffNormArgs& a = blockIdx.y == 0 ? a0 : (blockIdx.y == 1 ? a1 : a2);
  double *const s0 = sm[0], *const s1 = sm[1];
  double acc0 = 0.0, acc1 = 0.0;
  const int64_t total = a.n * a.nrep;
  for (int64_t t = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; t < total;
       t += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    const int64_t r = t / a.n, i = t - r * a.n;
    const int64_t e = r * a.field_stride + (a.idx ? a.idx[i] : i);
    double dn = 0.0, dd = 0.0;
    for (int c = 0; c < a.stride; ++c) {
      const int64_t k = e * a.stride + c;
      const double vn = a.xnew[k], vo = a.xold[k];
      const double d = vn - vo;
      if (a.vel) {  // the heavy-ball step
        const double step = (1.0 - a.beta) * a.vel[k] + a.alpha * d;
        a.vel[k] = step;
        a.update[k] = vo + step;
      } else if (a.update) {
        a.update[k] = vo + a.alpha * d;  // the Picard step
      }
      // the global error is of g(x) - x, before any step (Alg. 1)
      dn += d * d;
      dd += vo * vo;
    }
    if (a.p == 2) {
      acc0 += dn;
      acc1 += dd;
    } else if (a.p == 1) {
      acc0 += __builtin_sqrt(dn);
      acc1 += __builtin_sqrt(dd);
    } else {
      acc0 = fmax(acc0, __builtin_sqrt(dn));
      acc1 = fmax(acc1, __builtin_sqrt(dd));
    }
  }
  s0[threadIdx.x] = acc0;
  s1[threadIdx.x] = acc1;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < s) {
      if (a.p == 0) {
        s0[threadIdx.x] = fmax(s0[threadIdx.x], s0[threadIdx.x + s]);
        s1[threadIdx.x] = fmax(s1[threadIdx.x], s1[threadIdx.x + s]);
      } else {
        s0[threadIdx.x] += s0[threadIdx.x + s];
        s1[threadIdx.x] += s1[threadIdx.x + s];
      }
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    a.part[2 * blockIdx.x] = s0[0];
    a.part[2 * blockIdx.x + 1] = s1[0];
  }
}

// x <- x + alpha (g - x) on n doubles (gathered through idx when given, for
// nrep fields of field_stride elements with `stride` doubles each)
__global__ void __launch_bounds__(256) picard_kernel(double* __restrict__ x, const double* __restrict__ gx,
                                                     const int32_t* __restrict__ idx, int64_t n, int nrep,
                                                     int64_t field_stride, int stride, double alpha) {
  const int64_t t = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (t >= n * nrep) return;
  const int64_t r = t / n, i = t - r * n;
  const int64_t e = r * field_stride + (idx ? idx[i] : i);
  for (int c = 0; c < stride; ++c) {
    const double v = x[e * stride + c];
    x[e * stride + c] = v + alpha * (gx[e * stride + c] - v);
  }
}

// Barzilai-Borwein dot products (App. E) over one field of the concatenated
// x: with d = scale (xnew - xold) and dp the previous iteration's d, block
// partials of dp.dp, dp.(d - dp) and (d - dp).(d - dp); dp <- d.
__global__ void __launch_bounds__(256) bb_dots_kernel(const double* __restrict__ xnew,
                                                      const double* __restrict__ xold,
                                                      const int32_t* __restrict__ idx, int64_t n, int nrep,
                                                      int64_t field_stride, int stride, double scale,
                                                      double* __restrict__ dprev, double* __restrict__ part) {
  __shared__ double sm[3][256];
  double a0 = 0.0, a1 = 0.0, a2 = 0.0;
  const int64_t total = n * nrep;
  for (int64_t t = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; t < total;
       t += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    const int64_t r = t / n, i = t - r * n;
    const int64_t e = r * field_stride + (idx ? idx[i] : i);
    for (int c = 0; c < stride; ++c) {
      const int64_t k = e * stride + c;
      const double d = scale * (xnew[k] - xold[k]);
      const double pv = dprev[k];
      const double q = d - pv;
      a0 += pv * pv;
      a1 += pv * q;
      a2 += q * q;
      dprev[k] = d;
    }
  }
  sm[0][threadIdx.x] = a0;
  sm[1][threadIdx.x] = a1;
  sm[2][threadIdx.x] = a2;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w)
      for (int c = 0; c < 3; ++c) sm[c][threadIdx.x] += sm[c][threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0)
    for (int c = 0; c < 3; ++c) part[3 * blockIdx.x + c] = sm[c][0];
}

// CongAcc step of every component: m <- w m + (1 - w) d, x += a m, with
// d = gx - x; Delta on the grain cells, then A everywhere.
__global__ void __launch_bounds__(256) congacc_update_kernel(CongFields f, CongCoef cf) {
  const int64_t t = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  const int64_t nd = f.ncg * f.ncomp;
  if (t >= nd + 2 * f.ncell) return;
  auto step = [&](int comp, int64_t k, double* x, const double* gx, double* m) {
    const double w = cf.w[comp];
    const double mn = w * m[k] + (1.0 - w) * (gx[k] - x[k]);
    m[k] = mn;
    x[k] += cf.a[comp] * mn;
  };
  if (t < nd) {
    const int64_t r = t / f.ncg, e = r * f.ncell + f.grain_cells[t - r * f.ncg];
    for (int c = 0; c < 2; ++c) step(2 * static_cast<int>(r) + c, 2 * e + c, f.delta, f.dnew, f.md);
  } else {
    const int64_t k = t - nd;
    step(2 * f.ncomp + (k >= f.ncell ? 1 : 0), k, f.a, f.anew, f.ma);
  }
}

// --------------------------------------------------------------------------
// issue-rate probe: eight independent chains of one FP32 operation per lane
// (op 0 fma, 1 rsq, 2 sqrt, 3 rcp), for the roofline of the sweep kernels
// --------------------------------------------------------------------------
template <int OP>
__device__ __forceinline__ float rate_op(float a, float s) {
  if (OP == 0) return __builtin_fmaf(a, s, 0.5f);
  if (OP == 1) return __builtin_amdgcn_rsqf(a);
  if (OP == 2) return __builtin_amdgcn_sqrtf(a);
  return __builtin_amdgcn_rcpf(a);
}
template <int OP>
__global__ void __launch_bounds__(256) valu_rate_kernel(float* __restrict__ out, int iters, float s) {
  float v[8];
  for (int i = 0; i < 8; ++i) v[i] = 1.0f + 1e-3f * static_cast<float>(threadIdx.x) + 0.1f * static_cast<float>(i);
  for (int k = 0; k < iters; ++k)
    for (int i = 0; i < 8; ++i) v[i] = rate_op<OP>(v[i], s);
  float t = 0.0f;
  for (int i = 0; i < 8; ++i) t += v[i];
  out[static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x] = t;
}

// --------------------------------------------------------------------------
// launch wrappers
// --------------------------------------------------------------------------
static inline unsigned nblk(int64_t n, int b = 256) { return static_cast<unsigned>((n + b - 1) / b); }

template <typename T>
void launch_interp(const InterpArgs& a, void* cells, void* nodes, hipStream_t st) {
  if (a.nslot == 0) return;
  // One component: over packed cells, or on small grids, where a launch costs
  // more than the packing saves, straight from the fields (a sweep, FP64 and
  // mixed, packed and straight: 60.3 / 57.6 and 58.9 / 57.4 us on 32 x 32, 72.5
  // / 68 and 70.6 / 66.9 on 64 x 64, 91.5 / 79 on 96 x 96 either way, 111 / 91
  // and 111 / 92.4 on 128 x 128, 161 / 128 and 167 / 139 on 200 x 200).
  if (cells && a.ncomp == 1) {
    const dim3 grid(static_cast<unsigned>((a.nseg + 3) / 4));
    auto* out = static_cast<node4<T>*>(nodes);
    if (a.ncell > 96 * 96) {
      hipLaunchKernelGGL(pack_cells_kernel<T>, dim3(nblk(a.ncell)), dim3(256), 0, st, a,
                         static_cast<cell4<T>*>(cells));
      hipLaunchKernelGGL((interp1_kernel<T, true>), grid, dim3(256), 0, st, a, static_cast<const cell4<T>*>(cells), out);
    } else {
      hipLaunchKernelGGL((interp1_kernel<T, false>), grid, dim3(256), 0, st, a, nullptr, out);
    }
  } else {
    hipLaunchKernelGGL(interp_kernel<T>, dim3(nblk(a.nslot)), dim3(256), 0, st, a, static_cast<node4<T>*>(nodes));
  }
}
template void launch_interp<double>(const InterpArgs&, void*, void*, hipStream_t);
template void launch_interp<float>(const InterpArgs&, void*, void*, hipStream_t);

template <typename T, int EPL, int MODE>
static void launch_sweep_t(const SweepArgs& a, const SweepBufs& b, hipStream_t st) {
  const bool split = MODE == 0 && EPL % 2 == 0 && a.nlong > 0;
  const int64_t nl = split ? a.nlong : 0;
  // one block of two waves per bundle of 64/G segments
  const int64_t bundles = nl * 2 * a.G / 64 + ((a.nseg - nl) * a.G + 63) / 64;
  hipLaunchKernelGGL((sweep_kernel<T, EPL, MODE>), dim3(static_cast<unsigned>(bundles)), dim3(128), 0, st, a, b);
}

template <typename T, int MODE>
static void launch_sweep_m(int epl, const SweepArgs& a, const SweepBufs& b, hipStream_t st) {
  switch (epl) {
    case 1: launch_sweep_t<T, 1, MODE>(a, b, st); break;
    case 2: launch_sweep_t<T, 2, MODE>(a, b, st); break;
    case 3: launch_sweep_t<T, 3, MODE>(a, b, st); break;
    case 4: launch_sweep_t<T, 4, MODE>(a, b, st); break;
    default: launch_sweep_t<T, 8, MODE>(a, b, st); break;
  }
}

template <typename T>
void launch_sweep(int mode, int epl, const SweepArgs& a, const SweepBufs& b, hipStream_t st) {
  if (a.nseg == 0) return;
  if (mode == 0)
    launch_sweep_m<T, 0>(epl, a, b, st);
  else if (mode == 1)
    launch_sweep_m<T, 1>(epl, a, b, st);
  else if (mode == 2)
    launch_sweep_m<T, 2>(epl, a, b, st);
  else
    launch_sweep_m<T, 3>(epl, a, b, st);
}
template void launch_sweep<double>(int, int, const SweepArgs&, const SweepBufs&, hipStream_t);
template void launch_sweep<float>(int, int, const SweepArgs&, const SweepBufs&, hipStream_t);

template <typename T, int EPL>
static int64_t wave_slots_t() {
  int dev = 0, blocks = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, sweep_kernel<T, EPL, 0>, 128, 0) != hipSuccess) return 0;
  return static_cast<int64_t>(blocks) * 2 * cus;
}

template <typename T>
int64_t sweep_wave_slots(int epl) {
  switch (epl) {
    case 1: return wave_slots_t<T, 1>();
    case 2: return wave_slots_t<T, 2>();
    case 3: return wave_slots_t<T, 3>();
    case 4: return wave_slots_t<T, 4>();
    default: return wave_slots_t<T, 8>();
  }
}
template int64_t sweep_wave_slots<double>(int);
template int64_t sweep_wave_slots<float>(int);

template <typename T>
void launch_batch_sweep(int epl, const BatchGrainDev* grains, const int2* tiles, int ntiles, int* counter, int nblocks,
                        void* spill, int64_t wave_elems, hipStream_t st) {
  cpx<T>* sp = static_cast<cpx<T>*>(spill);
#define QC_BATCH(E)                                                                                                  \
  hipLaunchKernelGGL((batch_sweep_kernel<T, E>), dim3(nblocks), dim3(128), 0, st, grains, tiles, ntiles, counter, sp, \
                     wave_elems)
  switch (epl) {
    case 1: QC_BATCH(1); break;
    case 2: QC_BATCH(2); break;
    case 3: QC_BATCH(3); break;
    case 4: QC_BATCH(4); break;
    default: QC_BATCH(8); break;
  }
#undef QC_BATCH
}
template void launch_batch_sweep<double>(int, const BatchGrainDev*, const int2*, int, int*, int, void*, int64_t,
                                         hipStream_t);
template void launch_batch_sweep<float>(int, const BatchGrainDev*, const int2*, int, int*, int, void*, int64_t,
                                        hipStream_t);

void launch_valu_rate(int op, float* out, int nblocks, int iters, hipStream_t st) {
  switch (op) {
    case 0: hipLaunchKernelGGL(valu_rate_kernel<0>, dim3(nblocks), dim3(256), 0, st, out, iters, 0.999f); break;
    case 1: hipLaunchKernelGGL(valu_rate_kernel<1>, dim3(nblocks), dim3(256), 0, st, out, iters, 0.999f); break;
    case 2: hipLaunchKernelGGL(valu_rate_kernel<2>, dim3(nblocks), dim3(256), 0, st, out, iters, 0.999f); break;
    default: hipLaunchKernelGGL(valu_rate_kernel<3>, dim3(nblocks), dim3(256), 0, st, out, iters, 0.999f); break;
  }
}

template <int W>
static void launch_back_w(const BackArgs& a, hipStream_t st) {
  int64_t nb = (a.ncg + 63) / 64;
  if (a.zero_mask || a.sums) nb += (a.ncell + 64 * W - 1) / (64 * W);
  const dim3 grid(static_cast<unsigned>(nb));
  if (a.ncomp == 1)
    hipLaunchKernelGGL((rotate_back_kernel<1, W>), grid, dim3(64 * W), 0, st, a);
  else if constexpr (W <= 8)
    hipLaunchKernelGGL((rotate_back_kernel<4, W>), grid, dim3(64 * W), 0, st, a);
}
// Waves a block by the number of blocks of 64 cells.  A launch is bound by the
// gathers while its blocks fill the wave slots (1024 blocks of four waves, at
// four waves a SIMD): more waves a block then only add partial sums (400 x 400:
// 84, 90 and 105 us with 4, 8 and 16).  With fewer blocks it is the chain of a
// wave's angles, which more waves shorten: 24 and 22 us with 4 and 8 on the
// 200 x 200 disc (491 blocks), 16 and 13 us at 249 blocks, and down to a block
// a compute unit 16 waves beat 8 or equal them (12.2 -> 10.3 us at 89 blocks, 6.3 -> 5.6 us
// at 13).  Several components leave no registers for 16 (24 and 18 us with 4
// and 8 at 100 blocks).
static int back_waves(int64_t blocks, int ncomp) { return blocks >= 1024 ? 4 : blocks > 256 || ncomp > 1 ? 8 : 16; }
void launch_rotate_back(const BackArgs& a, hipStream_t st) {
  if (a.ncg == 0 && !a.zero_mask && !a.sums) return;
  switch (back_waves((a.ncg + 63) / 64, a.ncomp)) {
    case 4: launch_back_w<4>(a, st); break;
    case 8: launch_back_w<8>(a, st); break;
    default: launch_back_w<16>(a, st); break;
  }
}
template <typename T>
void launch_batch_interp(const BatchGrainDev* grains, const int2* pack, int npack, const int2* interp, int ninterp,
                         int* counters, hipStream_t st) {
  if (npack > 0) hipLaunchKernelGGL(batch_pack_kernel<T>, dim3(npack), dim3(256), 0, st, grains, pack);
  if (ninterp > 0) hipLaunchKernelGGL(batch_interp_kernel<T>, dim3(ninterp), dim3(256), 0, st, grains, interp, counters);
}
template void launch_batch_interp<float>(const BatchGrainDev*, const int2*, int, const int2*, int, int*, hipStream_t);
template void launch_batch_interp<double>(const BatchGrainDev*, const int2*, int, const int2*, int, int*, hipStream_t);
void launch_batch_back(bool several, const BatchGrainDev* grains, const int2* tiles, int n, hipStream_t st) {
  if (n == 0) return;
  const int w = back_waves(n, several ? 2 : 1);
  const dim3 grid(n), block(64 * w);
  if (several) {
    if (w == 4)
      hipLaunchKernelGGL((batch_back_kernel<4, 4>), grid, block, 0, st, grains, tiles);
    else
      hipLaunchKernelGGL((batch_back_kernel<4, 8>), grid, block, 0, st, grains, tiles);
  } else if (w == 4) {
    hipLaunchKernelGGL((batch_back_kernel<1, 4>), grid, block, 0, st, grains, tiles);
  } else if (w == 8) {
    hipLaunchKernelGGL((batch_back_kernel<1, 8>), grid, block, 0, st, grains, tiles);
  } else {
    hipLaunchKernelGGL((batch_back_kernel<1, 16>), grid, block, 0, st, grains, tiles);
  }
}
void launch_batch_set(const double* delta, const double* A, const uint8_t* mask, int64_t ncell, int ncomp,
                      double* delta_out, double* A_out, hipStream_t st) {
  if (ncell > 0)
    hipLaunchKernelGGL(batch_set_kernel, dim3(nblk(ncell)), dim3(256), 0, st, reinterpret_cast<const double2*>(delta),
                       A, mask, ncell, ncomp, reinterpret_cast<double2*>(delta_out), A_out);
}

template <typename T, int V, bool CPLX>
static void launch_back_v(const LdosBackArgs& a, const void* ebuf, hipStream_t st) {
  const int M = (CPLX ? 2 : 1) * a.n_e;
  const int tpc = std::min(M / V, 256), cpb = 256 / tpc;
  const dim3 grid(static_cast<unsigned>((a.ncg + cpb - 1) / cpb), static_cast<unsigned>((M / V + tpc - 1) / tpc));
  // records of sixteen angles at a time, or as many as leave up to 512 of them
  const int kpb = std::min(std::max(512 / cpb, 1), 16);
  const size_t lds = std::max(sizeof(double) * cpb * (tpc * V + 1) * (a.fold_k0 > 0 ? 2 : 1),
                              static_cast<size_t>(48) * kpb * cpb);
  hipLaunchKernelGGL((ldos_back_kernel<T, V, CPLX>), grid, dim3(256), lds, st, a, static_cast<const T*>(ebuf), tpc, cpb,
                     kpb);
}
// the widest loads (up to 16 B) that the row length allows
template <typename T, bool CPLX>
static void launch_back_t(const LdosBackArgs& a, const void* ebuf, hipStream_t st) {
  if (a.ncg == 0) return;
  const int M = (CPLX ? 2 : 1) * a.n_e;
  if (sizeof(T) == 4 && M % 4 == 0)
    launch_back_v<T, 4, CPLX>(a, ebuf, st);
  else if (M % 2 == 0)
    launch_back_v<T, 2, CPLX>(a, ebuf, st);
  else
    launch_back_v<T, 1, CPLX>(a, ebuf, st);
}
template <typename T>
void launch_ldos_back(const LdosBackArgs& a, const void* ebuf, hipStream_t st) {
  launch_back_t<T, false>(a, ebuf, st);
}
template void launch_ldos_back<double>(const LdosBackArgs&, const void*, hipStream_t);
template void launch_ldos_back<float>(const LdosBackArgs&, const void*, hipStream_t);

template <typename T>
void launch_green_back(const LdosBackArgs& a, const void* ebuf, hipStream_t st) {
  launch_back_t<T, true>(a, ebuf, st);
}
template void launch_green_back<double>(const LdosBackArgs&, const void*, hipStream_t);
template void launch_green_back<float>(const LdosBackArgs&, const void*, hipStream_t);

void launch_fill(double* p, int64_t n, double v, hipStream_t st) {
  if (n > 0) hipLaunchKernelGGL(fill_kernel, dim3(nblk(n)), dim3(256), 0, st, p, n, v);
}
void launch_curl(const double* A, double* B, int nx, int ny, double h, hipStream_t st) {
  hipLaunchKernelGGL(curl_kernel, dim3(nblk(static_cast<int64_t>(nx) * ny)), dim3(256), 0, st, A, B, nx, ny, h);
}
void launch_block_sum(const double* x, const int32_t* idx, int64_t n, double* part, int nparts, hipStream_t st) {
  const BlockSumRow r{x, idx, n, part, 0, 0, 0, 0.0};
  hipLaunchKernelGGL(block_sum_kernel, dim3(nparts), dim3(256), 0, st, r, r);
}
void launch_parts_to_host(const double* part, int n, double* host, hipStream_t st) {
  hipLaunchKernelGGL(parts_to_host_kernel, dim3(nblk(n)), dim3(256), 0, st, part, n, host);
}
void launch_block_sum2(const BlockSumRow& r0, const BlockSumRow& r1, int nparts, hipStream_t st) {
  hipLaunchKernelGGL(block_sum_kernel, dim3(nparts, 2), dim3(256), 0, st, r0, r1);
}
void launch_diff_norm(const DiffNormArgs* a, int count, const CongFields* f, double* cong_part, int nparts,
                      hipStream_t st) {
  if (count < 1 || count > 3) return;
  const int rows = count + (f ? 2 * f->ncomp + 2 : 0);
  hipLaunchKernelGGL(diff_norm_kernel, dim3(nparts, rows), dim3(256), 0, st, count, a[0], a[count > 1 ? 1 : 0],
                     a[count > 2 ? 2 : 0], f ? *f : CongFields{}, cong_part);
}
void launch_congacc_update(const CongFields& f, const CongCoef& cf, hipStream_t st) {
  const int64_t n = f.ncg * f.ncomp + 2 * f.ncell;
  if (n > 0) hipLaunchKernelGGL(congacc_update_kernel, dim3(nblk(n)), dim3(256), 0, st, f, cf);
}
void launch_bb_dots(const double* xnew, const double* xold, const int32_t* idx, int64_t n, int nrep,
                    int64_t field_stride, int stride, double scale, double* dprev, double* part, int nparts,
                    hipStream_t st) {
  hipLaunchKernelGGL(bb_dots_kernel, dim3(nparts), dim3(256), 0, st, xnew, xold, idx, n, nrep, field_stride, stride,
                     scale, dprev, part);
}
void launch_picard(double* x, const double* gx, const int32_t* idx, int64_t n, int nrep, int64_t field_stride,
                   int stride, double alpha, hipStream_t st) {
  if (n * nrep > 0)
    hipLaunchKernelGGL(picard_kernel, dim3(nblk(n * nrep)), dim3(256), 0, st, x, gx, idx, n, nrep, field_stride,
                       stride, alpha);
}
void launch_lw_accumulate(const double* delta, const double* delta_new, const int32_t* grain_cells, int64_t ncg,
                          int ncomp, int64_t ncell, const double* den, double w, int first, double* acc,
                          hipStream_t st) {
  if (ncg > 0)
    hipLaunchKernelGGL(lw_accumulate_kernel, dim3(nblk(ncg)), dim3(256), 0, st, delta, delta_new, grain_cells, ncg,
                       ncomp, ncell, den, w, first, acc);
}
void launch_lw_finish(const double* delta, const int32_t* grain_cells, int64_t ncg, int ncomp, int64_t ncell,
                      int n_theta, const double* eta, const double* wk, const double* logt, double twopi_rz,
                      const double* acc, double* omega_cell, double* omega, hipStream_t st) {
  if (ncg > 0)
    hipLaunchKernelGGL(lw_finish_kernel, dim3(nblk(ncg)), dim3(256), 0, st, delta, grain_cells, ncg, ncomp, ncell,
                       n_theta, eta, wk, logt, twopi_rz, acc, omega_cell, omega);
}
void launch_scale(const double* x, double s, int64_t n, double* y, hipStream_t st) {
  if (n > 0) hipLaunchKernelGGL(scale_kernel, dim3(nblk(n)), dim3(256), 0, st, x, s, n, y);
}
}  // namespace qc
