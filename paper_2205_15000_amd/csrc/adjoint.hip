// Reverse mode of one iteration map (FP64): gradients of a real loss of
// (Delta_new, j, Omega) with respect to Delta_G(R) and A_ind(R), the
// boundary store held fixed (start values from specular taps are inputs;
// start values that are bulk roots of the end values are differentiated).
//
// Complex gradients follow dL = Re(conj(G_x) dx), i.e. G_x = dL/dRe x +
// i dL/dIm x.  For y = F(x, x*): G_x = conj(dF/dx) G_y + dF/dx* conj(G_y).
//
// Implicit-midpoint step (App. C) y = F(g; D, z, h) solves
//   y - g - h f((g+y)/2) = 0,  f(m) = i (D* m^2 + 2 z m + D),
// so with m = (g+y)/2, f' = i (2 D* m + 2 z) and Q = 1 - h f'/2:
//   dF/dg = (1 + h f'/2)/Q,  dF/dD = i h/Q,  dF/dD* = i h m^2/Q,  dF/dz = 2 i h m/Q.
// Bulk root y = -D/(z+s), s = z + D* y: dy/dD = -1/(2s), dy/dD* = -y^2/(2s),
// dy/dz = -y/s.
#include "kernels.hpp"
#include "sweep.hpp"

namespace qc {

using C = cpx<double>;

__device__ __forceinline__ C cconj(C a) { return mk(a.x, -a.y); }
__device__ __forceinline__ C cdivd(C a, C b) {
  const double r = drcp(b.x * b.x + b.y * b.y);
  return mk((a.x * b.x + a.y * b.y) * r, (a.y * b.x - a.x * b.y) * r);
}
__device__ __forceinline__ C cscale(double s, C a) { return mk(s * a.x, s * a.y); }

// Sums over the segment's lane group of the three slot gradients (Re, Im of
// G_Delta and the gradient of a), written to o[0..2] by the group's first lanes.
__device__ __forceinline__ void put_slot_grad(double* o, double rx, double ry, double ra, int G, int lane) {
  if (G >= 4) {
    const double v = group_sum4_scatter(rx, ry, ra, 0.0, G, lane);
    const int qq = scatter_index(lane);
    if (lane < 4 && qq < 3) o[qq] = v;
  } else {
    rx = group_sum(rx, G);
    ry = group_sum(ry, G);
    ra = group_sum(ra, G);
    if (lane == 0) {
      o[0] = rx;
      o[1] = ry;
      o[2] = ra;
    }
  }
}

// One step y = F(g; D, z, h) taken backwards for one energy: the adjoint l of
// y becomes that of g.  With M = 2m = g + y, Q as above and u = l Q / |Q|^2
// (= conj(1/Q) l) the four derivatives share all their products:
//   adjoint of g   conj(2/Q - 1) l                       = 2u - l,
//   gradient of D  conj(ih/Q) l + (ih m^2/Q) conj(l)     = ih (m v - u),  v = m conj(u),
//   gradient of z  Re(conj(l) 2ih m/Q)                   = -2h Im v,
// so the sums over the energies are taken of u, M (M conj(u)) and
// Im(M conj(u)) and the factors are put on once per step.  hd = (h/2) D and
// hz = h Re z are the step's, qx = 1 + h Im z the energy's.
struct StepSum {
  C u = {0.0, 0.0}, mmu = {0.0, 0.0};
  double mu = 0.0;
};
__device__ __forceinline__ C step_back(C g, C y, C l, C hd, double hz, double qx, StepSum& sum) {
  const C M = g + y;
  const double Qx = fmaT(hd.x, M.y, fmaT(-hd.y, M.x, qx));
  const double Qy = -fmaT(hd.x, M.x, fmaT(hd.y, M.y, hz));
  const double r = drcp(fmaT(Qx, Qx, Qy * Qy));
  const C u = mk(r * fmaT(Qx, l.x, -(Qy * l.y)), r * fmaT(Qx, l.y, Qy * l.x));
  const C mu = mk(fmaT(M.x, u.x, M.y * u.y), fmaT(M.y, u.x, -(M.x * u.y)));  // M conj(u)
  sum.u = sum.u + u;
  sum.mmu.x = fmaT(M.x, mu.x, fmaT(-M.y, mu.y, sum.mmu.x));
  sum.mmu.y = fmaT(M.x, mu.y, fmaT(M.y, mu.x, sum.mmu.y));
  sum.mu += mu.y;
  return mk(fmaT(2.0, u.x, -l.x), fmaT(2.0, u.y, -l.y));
}

// adjoint of y = bulk root(z, d) (start value) with adjoint gy: adds to
// G_d (complex) and to the real gradient of z's real part
__device__ __forceinline__ void bulk_adj(C y, C z, C d, C gy, C& gd, double& gzr) {
  const C s = z + cconj(d) * y;
  const C i2s = cdivd(mk(-0.5, 0.0), s);   // -1/(2s)
  const C dd = i2s;
  const C ddc = y * y * i2s;
  const C dz = cscale(2.0, y * i2s);       // -y/s
  gd = gd + cconj(dd) * gy + ddc * cconj(gy);
  gzr += (cconj(gy) * dz).x;
}

// Node-local gradients of the per-node sums (Sec. II.A, Sec. II), without the
// pole weight: with P = 1 + gamma gamma~, D the node's order parameter and
// pt = 2 pi t~,
//   S_f = -i pt R (u + conj v),  S_g = (pt/2) R Im((1-X)/(1+X)),  S_I = pt R Im(D* g - D g~)
// the adjoint of gamma is conj[(F - conj(F) g~^2 - 2 kg g~)/P^2 + ki conj(D)]
// and that of gamma~ conj[(conj(F) - F g^2 - 2 kg g)/P^2 - ki D], with
// F = -i pt conj(G_f) and kg = i c/2, ki = i k: constants of the node.
struct NodeConst {
  C f, add;  // F (conj(F) for gamma~) and conj(ki conj D) (-conj(ki D))
  double c;
};
template <int DIR>
__device__ __forceinline__ NodeConst node_const(C dn, const double4& gs, double pt) {
  const double k = -pt * gs.w;
  NodeConst n;
  n.f = mk(-pt * gs.y, DIR * (-pt * gs.x));
  n.add = DIR > 0 ? mk(k * dn.y, -k * dn.x) : mk(k * dn.y, k * dn.x);
  n.c = -pt * gs.z;
  return n;
}
// l plus r times the adjoint, of the own value's function by the other's value o
__device__ __forceinline__ C node_adj(C own, C o, const NodeConst& n, double r, C l) {
  const double Px = fmaT(own.x, o.x, fmaT(-own.y, o.y, 1.0)), Py = fmaT(own.x, o.y, own.y * o.x);
  const double ip = drcp(fmaT(Px, Px, Py * Py));
  // T = f - o (conj(f) o + i c)
  const double ax = fmaT(n.f.x, o.x, n.f.y * o.y), ay = fmaT(n.f.x, o.y, fmaT(-n.f.y, o.x, n.c));
  const double tx = fmaT(-o.x, ax, fmaT(o.y, ay, n.f.x)), ty = fmaT(-o.x, ay, fmaT(-o.y, ax, n.f.y));
  // conj(T) P^2 / |P|^4
  const double qx = fmaT(Px, Px, -(Py * Py)), qy = 2.0 * (Px * Py), w = r * (ip * ip);
  return mk(fmaT(w, fmaT(tx, qx, ty * qy), fmaT(r, n.add.x, l.x)),
            fmaT(w, fmaT(tx, qy, -(ty * qx)), fmaT(r, n.add.y, l.y)));
}

// Reverse mode of one march: DIR = +1 that of gamma, -1 that of gamma~.  In
// the order of the march the nodes are j = 0..n-1 (node j at slot j or
// n - 1 - j), step j joins nodes j - 1 and j, step 0 comes from the start
// value and step n goes to the far end, which nothing reads: its adjoint is
// zero.  The wave marches its own function once (forward sweep order), then
// walks back: at every node the other function, marched along in the same
// direction, gives the local gradients of the sums; the adjoint of the own
// function takes them up and passes through the step before.
//
// The own values on the way back: CK > 0 keeps the value entering every block
// of CK nodes and marches a block again into a per-thread scratch when the
// walk reaches it; CK = 0 keeps every node's value.  Both do the same steps on
// the same inputs.
//
// The two directions share no intermediate value, so each is a wave of its
// own (they write gradients of their own, which the gather adds).  One wave
// that marched gamma, then gamma~ with the adjoint of gamma, then the adjoint
// of gamma~ from values marched again took three passes over the segment
// instead of two and had 1.6 waves a SIMD at 38% of the issue rate.  Bound by
// FP64 issue: two marches, one marched again, a step and a node taken back
// (step_back, node_adj: some 70 operations for 130 before).  200 x 200 disc,
// 48 poles, checkpoints: 2.42 ms before, 1.65 ms as two waves, 1.38 ms with
// the shorter step, 1.20 ms with two waves a SIMD (adjoint_kernel); d-wave
// 400 x 400, 64 poles: 7.9 ms.
template <int EPL, int DIR>
__device__ __forceinline__ void adjoint_march(const AdjArgs& a, int64_t seg, int lane, int64_t thr,
                                              const node4<double>* __restrict__ nodes, const C* __restrict__ bc_prev_own,
                                              const C* __restrict__ bc_prev_oth, C* keep, int CK,
                                              const int64_t* __restrict__ ckbase, C* scr, int64_t nthr,
                                              const double4* __restrict__ gS, double* __restrict__ gV) {
  constexpr double sd = DIR;  // D -> -D* for gamma~
  const int64_t slot0 = a.seg_slot0[seg];
  const int n = a.seg_n[seg];
  const int last = n > 0 ? n - 1 : 0;
  const double hfull = a.h, q = a.q;
  const int e0 = lane * EPL;
  // a lane's energies beyond the last one repeat it with no weight (their
  // adjoint stays zero) and store nothing
  auto energy = [&](int i) { return min(e0 + i, a.n_e - 1); };
  auto ok = [&](int i) { return e0 + i < a.n_e; };
  double ey[EPL], rw[EPL];
  for (int i = 0; i < EPL; ++i) {
    ey[i] = a.eps[2 * energy(i) + 1];  // (Matsubara poles: no real part)
    rw[i] = ok(i) ? a.rp[energy(i)] : 0.0;
  }
  double* const out = gV + (DIR > 0 ? 0 : 3);
  auto slot = [&](int j) { return static_cast<uint32_t>(DIR > 0 ? min(max(j, 0), last) : max(min(last - j, last), 0)); };
  const node4<double>* const nseg = nodes + slot0;
  if (n == 0) {  // no node: nothing reads this segment's marches
    put_slot_grad(out + slot0 * 6, 0.0, 0.0, 0.0, a.G, lane);
    return;
  }
  const double h_in = DIR > 0 ? a.seg_hfirst[seg] : a.seg_hlast[seg];
  const double h_out = DIR > 0 ? a.seg_hlast[seg] : a.seg_hfirst[seg];
  const int64_t tb = seg * 4;
  // start value of the own (OWN) or the other march, from the taps or the
  // bulk root; returns whether it came from the taps
  auto start = [&](C* v, bool own_march) {
    const bool at_min = own_march == (DIR > 0);  // gamma starts at s_min
    const double* tw = (at_min ? a.tap_start_w : a.tap_end_w) + tb;
    const int32_t* ts = (at_min ? a.tap_start_seg : a.tap_end_seg) + tb;
    const C* bc = own_march ? bc_prev_own : bc_prev_oth;
    const bool taps = a.bc_valid && tw[0] + tw[1] + tw[2] + tw[3] > 0.0;
    const node4<double> v0 = nseg[slot(own_march ? 0 : n - 1)];
    for (int i = 0; i < EPL; ++i) {
      if (taps) {
        v[i] = mk(0.0, 0.0);
        for (int c = 0; c < 4; ++c)
          v[i] = v[i] + cscale(tw[c], bc[static_cast<int64_t>(ts[c]) * a.n_e_tot + energy(i)]);
      } else {
        v[i] = bulk_root(q * v0.a, ey[i], at_min ? v0.dx : -v0.dx, v0.dy);
      }
    }
    return taps;
  };
  // full step between neighbouring slots; s = sd the own march, -sd the other
  auto full_step = [&](C* v, const node4<double>& p, const node4<double>& c, double s) {
    StepC<double> k = step_consts(0.5 * (s * (p.dx + c.dx)), 0.5 * (p.dy + c.dy), hfull);
    const double ky = 0.5 * hfull * (q * (0.5 * (p.a + c.a)));
    double kx[EPL], kx2[EPL];  // (formed here: held, they cost occupancy)
    for (int i = 0; i < EPL; ++i) {
      kx[i] = fmaT(-0.5 * hfull, ey[i], -0.5);
      kx2[i] = kx[i] * kx[i];
    }
    riccati_steps<double, EPL, true>(v, k, kx, kx2, &ky);
  };
  // partial step next to an end, with the value of the slot there
  auto end_step = [&](C* v, const node4<double>& p, double hs, double s) {
    const StepC<double> k = step_consts(s * p.dx, p.dy, hs);
    for (int i = 0; i < EPL; ++i) v[i] = riccati_step_z(v[i], k, hs, q * p.a, ey[i]);
  };
  const int64_t cb = CK > 0 ? ckbase[seg] : 0;
  auto scr_at = [&](int pos, int i) -> C& { return scr[(static_cast<int64_t>(pos) * EPL + i) * nthr + thr]; };
  auto keep_at = [&](int64_t row, int i) -> C& { return keep[row * a.n_e + energy(i)]; };

  // ---- the own march: its values kept
  C x[EPL];
  const bool taps = start(x, true);
  {
    node4<double> prev = nseg[slot(0)], nxt = nseg[slot(1)];
    end_step(x, prev, h_in, sd);
    for (int j = 0;; ++j) {  // x at node j
      if (CK == 0) {
        for (int i = 0; i < EPL; ++i)
          if (ok(i)) keep_at(slot0 + slot(j), i) = x[i];
      } else if ((j + 1) % CK == 0 && j + 1 < n) {
        for (int i = 0; i < EPL; ++i)
          if (ok(i)) keep_at(cb + (j + 1) / CK, i) = x[i];
      }
      if (j == n - 1) break;
      const node4<double> cur = nxt;
      nxt = nseg[slot(j + 2)];
      full_step(x, prev, cur, sd);
      prev = cur;
    }
  }

  // (a lane may read what another lane of its wave kept: the last energy)
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");

  // ---- back along the segment
  int loaded = -1;
  // own value at node j < n - 1 (start value for j = -1)
  auto recall = [&](C* v, int j) {
    if (j < 0) {
      start(v, true);
      return;
    }
    if (CK == 0) {
      for (int i = 0; i < EPL; ++i) v[i] = keep_at(slot0 + slot(j), i);
      return;
    }
    const int kb = j / CK, s0 = kb * CK;
    if (kb != loaded) {  // march block kb again, up to node j
      loaded = kb;
      C r[EPL];
      if (kb == 0) {
        start(r, true);
      } else {
        for (int i = 0; i < EPL; ++i) r[i] = keep_at(cb + kb, i);
      }
      node4<double> prev = nseg[slot(s0 - 1)], nxt = nseg[slot(s0)];
      for (int s = s0; s <= j; ++s) {
        const node4<double> cur = nxt;
        nxt = nseg[slot(s + 1)];
        if (s == 0)
          end_step(r, cur, h_in, sd);
        else
          full_step(r, prev, cur, sd);
        prev = cur;
        for (int i = 0; i < EPL; ++i) scr_at(s - s0, i) = r[i];
      }
    }
    for (int i = 0; i < EPL; ++i) v[i] = scr_at(j - s0, i);
  };
  C y[EPL], lam[EPL];
  start(y, false);
  for (int i = 0; i < EPL; ++i) lam[i] = mk(0.0, 0.0);
  const double pt = a.twopi_tt;  // 2 pi t~
  // Step j gives half of its slot gradient to slot j - 1 and half to slot j
  // (step 0 both to slot 0); `carry` holds the half of the step just taken
  // that belongs to the next slot.
  C carry = mk(0.0, 0.0);
  double carrya = 0.0;
  node4<double> cur = nseg[slot(n - 1)], nxt = nseg[slot(n - 2)];
  double4 gsn = gS[slot0 + slot(n - 1)];
  end_step(y, cur, h_out, -sd);
  for (int j = n - 1; j >= 0; --j) {  // x, y at node j; cur, nxt the slots j and j - 1
    const double4 gs = gsn;
    gsn = gS[slot0 + slot(j - 1)];
    C xl[EPL];
    recall(xl, j - 1);
    const node4<double> lo = nxt;
    nxt = nseg[slot(j - 2)];
    const C dn = mk(cur.dx, cur.dy);
    C acc = carry;
    double acca = carrya;
    // half-step values of step j (slot 0's alone for j = 0)
    const node4<double>& lw = j > 0 ? lo : cur;
    const double za = q * (0.5 * (lw.a + cur.a)), hs = j > 0 ? hfull : h_in;
    const C hd = mk(0.25 * hs * (sd * (lw.dx + cur.dx)), 0.25 * hs * (lw.dy + cur.dy));
    const NodeConst nc = node_const<DIR>(dn, gs, pt);
    StepSum sum;
    C si = mk(0.0, 0.0);
    for (int i = 0; i < EPL; ++i) {
      lam[i] = node_adj(x[i], y[i], nc, rw[i], lam[i]);
      if (DIR > 0) {
        si.x = fmaT(rw[i], y[i].y - x[i].y, si.x);
        si.y = fmaT(rw[i], x[i].x + y[i].x, si.y);
      }
      lam[i] = step_back(xl[i], x[i], lam[i], hd, hs * za, fmaT(hs, ey[i], 1.0), sum);
    }
    if (DIR > 0) acc = acc + cscale(-pt * gs.w, si);  // D in S_I: ki g - conj(ki g~)
    C stepD = mk(-hs * fmaT(0.25, sum.mmu.y, -sum.u.y), hs * fmaT(0.25, sum.mmu.x, -sum.u.x));
    const double stepa = -hs * q * sum.mu;
    if (DIR < 0) stepD = mk(-stepD.x, stepD.y);  // gradient of D from that of -D*
    acc = acc + cscale(0.5, stepD);
    acca += 0.5 * stepa;
    carry = cscale(0.5, stepD);
    carrya = 0.5 * stepa;
    if (j == 0) {
      acc = acc + carry;
      acca += carrya;
      if (!taps) {  // the march started at the bulk root of this slot's values
        C gd = mk(0.0, 0.0);
        double gz = 0.0;
        for (int i = 0; i < EPL; ++i)
          if (ok(i)) bulk_adj(xl[i], mk(q * cur.a, ey[i]), mk(sd * cur.dx, cur.dy), lam[i], gd, gz);
        acc = acc + (DIR > 0 ? gd : mk(-gd.x, gd.y));
        acca += q * gz;
      }
    }
    put_slot_grad(out + (slot0 + slot(j)) * 6, acc.x, acc.y, acca, a.G, lane);
    if (j > 0) full_step(y, lo, cur, -sd);
    for (int i = 0; i < EPL; ++i) x[i] = xl[i];
    cur = lo;
  }
}

// blocks of two waves: the two directions of one bundle of 64/G segments.
// Three energies a lane need 261 registers and are held to the 256 that leave
// room for a second wave on the SIMD (nothing is spilled: 1.38 -> 1.20 ms);
// four and eight need more than can be taken away.
template <int EPL>
__global__ void __launch_bounds__(128, EPL == 3 ? 2 : 1) adjoint_kernel(AdjArgs a, AdjBufs b) {
  const int l64 = threadIdx.x & 63;
  const int dir = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
  const int64_t wseg = (static_cast<int64_t>(blockIdx.x) << (6 - a.log2g)) + (l64 >> a.log2g);
  if (wseg >= a.nseg) return;  // whole lane groups leave together (G | 64)
  const int lane = l64 & (a.G - 1);
  const int64_t seg = a.order ? static_cast<int64_t>(a.order[wseg]) : wseg;
  const int64_t thr = static_cast<int64_t>(blockIdx.x) * 128 + threadIdx.x;
  const node4<double>* nodes = static_cast<const node4<double>*>(b.nodes);
  const C* bg = static_cast<const C*>(b.bc_g_prev);
  const C* bgt = static_cast<const C*>(b.bc_gt_prev);
  const double4* gS = static_cast<const double4*>(b.gS);
  if (dir == 0)
    adjoint_march<EPL, 1>(a, seg, lane, thr, nodes, bg, bgt, static_cast<C*>(b.keep_g), b.ck, b.ckbase,
                          static_cast<C*>(b.scr), b.nthr, gS, b.gV);
  else
    adjoint_march<EPL, -1>(a, seg, lane, thr, nodes, bgt, bg, static_cast<C*>(b.keep_gt), b.ck, b.ckbase,
                           static_cast<C*>(b.scr), b.nthr, gS, b.gV);
}

// The cell gradients a rotated lattice gathers, one record per grain cell:
// (G_{Delta_new,G} / den_G for every component, G_jx, G_jy).
__global__ void __launch_bounds__(256) cell_grad_kernel(BackAdjArgs a) {
  const int64_t c = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (c >= a.ncg) return;
  const int64_t cell = a.grain_cells[c];
  double* const o = a.gC + c * (2 * a.ncomp + 2);
  for (int g = 0; g < a.ncomp; ++g) {
    o[2 * g] = a.gdn ? a.gdn[2 * (g * a.ncell + cell)] / a.den[g] : 0.0;
    o[2 * g + 1] = a.gdn ? a.gdn[2 * (g * a.ncell + cell) + 1] / a.den[g] : 0.0;
  }
  o[2 * a.ncomp] = a.gj ? a.gj[cell] : 0.0;
  o[2 * a.ncomp + 1] = a.gj ? a.gj[a.ncell + cell] : 0.0;
}

// Gradients of the per-node sums from the cell gradients: the transpose of
// the rotate-back gather, formed as a gather per slot over the cells whose
// rotate-back stencil uses it (no atomics; each slot written once).
// Bound by its table (12 B an entry, about eight entries a slot with paired
// angles).  Four lanes share a slot: the lanes of a wave then read the table
// in order, where a lane per slot walked its own row, 64 rows at once in the
// cache, and waited for each entry's cell, gradient and two divisions in turn
// (135 us, 60 us now with the records, on the 200 x 200 disc;
// 1347 and 310 us on d-wave 400 x 400).
constexpr int kBtLanes = 4;
__global__ void __launch_bounds__(256) back_adjoint_kernel(BackAdjArgs a) {
  const int64_t t = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  const int64_t s = t / kBtLanes;
  const int lane = static_cast<int>(t & (kBtLanes - 1));
  if (s >= a.nslot) return;  // whole groups of four leave together
  const int k = a.slot_angle[s];
  const double ck = a.cosk[k], sk = a.sink[k];
  double ex[4], ey[4];
  for (int g = 0; g < a.ncomp; ++g) {
    ex[g] = a.eta[2 * (g * a.n_theta + k)];
    ey[g] = a.eta[2 * (g * a.n_theta + k) + 1];
  }
  double sx = 0.0, sy = 0.0, sj = 0.0, sw = 0.0;
  const int64_t end = a.bt_ptr[s + 1];
  for (int64_t e = a.bt_ptr[s] + lane; e < end; e += kBtLanes) {
    const double w = a.bt_w[e];
    const double* const r = a.gC + static_cast<int64_t>(a.bt_c[e]) * (2 * a.ncomp + 2);
    // G_{S_f} = wk sum_G eta_G G_{Num_G}, G_{Num_G} = G_{Delta_new,G} / den_G
    double fx = 0.0, fy = 0.0;
    for (int g = 0; g < a.ncomp; ++g) {
      fx += ex[g] * r[2 * g] - ey[g] * r[2 * g + 1];
      fy += ex[g] * r[2 * g + 1] + ey[g] * r[2 * g];
    }
    sx += w * fx;
    sy += w * fy;
    sj += w * (ck * r[2 * a.ncomp] + sk * r[2 * a.ncomp + 1]);
    sw += w;
  }
  const double v = group_sum4_scatter(sx, sy, sj, sw, kBtLanes, lane);
  const int qq = scatter_index(lane);
  const double f = qq < 2 ? 1.0 : qq == 2 ? a.four_q : -a.h2 * a.gomega;  // omega = ... - I
  a.gS[4 * s + qq] = a.wk[k] * f * v;
}

// Gradients on the reference grid from the slot gradients: the transpose of
// the interpolation pre-pass, as a gather per cell over the slots whose
// stencils use it (each cell written once, zero where none does).  Sixteen
// lanes share a cell, lane q taking every 16th entry of its lists; their
// partial sums are combined with DPP moves.  Bound by the lists (12 B an
// entry, four Delta and four A entries a slot) and the gathers of gV: with
// paired angles it stops at the lower angles' entries instead of reading the
// upper ones' zeros (208 -> 113 us on the 200 x 200 disc).
constexpr int kItLanes = 16;
__global__ void __launch_bounds__(256) interp_adjoint_kernel(InterpAdjArgs a) {
  const int64_t t = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  const int64_t cell = t / kItLanes;
  const int q = static_cast<int>(t & (kItLanes - 1));
  if (cell >= a.ncell) return;  // whole groups of sixteen leave together
  double dx[4] = {0.0, 0.0, 0.0, 0.0}, dy[4] = {0.0, 0.0, 0.0, 0.0};
  for (int64_t e = a.it_dptr[cell] + q; e < a.it_dend[cell]; e += kItLanes) {
    const int64_t s = a.it_ds[e];
    const double w = a.it_dw[e];
    const int k = a.slot_angle[s];
    const double* r = a.gV + s * 6;  // the parts of the two marches
    const double gx = r[0] + r[3], gy = r[1] + r[4];
    for (int g = 0; g < a.ncomp; ++g) {
      // y = eta w x  ->  G_x += conj(eta) w G_y
      const double ex = a.eta[2 * (g * a.n_theta + k)], ey = a.eta[2 * (g * a.n_theta + k) + 1];
      dx[g] += w * (ex * gx + ey * gy);
      dy[g] += w * (ex * gy - ey * gx);
    }
  }
  double ax = 0.0, ay = 0.0;
  for (int64_t e = a.it_aptr[cell] + q; e < a.it_aend[cell]; e += kItLanes) {
    const int64_t s = a.it_as[e];
    const double wg = a.it_aw[e] * (a.gV[s * 6 + 2] + a.gV[s * 6 + 5]);
    const int k = a.slot_angle[s];
    ax += wg * a.cosk[k];
    ay += wg * a.sink[k];
  }
  for (int g = 0; g < a.ncomp; ++g) {
    dx[g] = group_sum(dx[g], kItLanes);
    dy[g] = group_sum(dy[g], kItLanes);
  }
  ax = group_sum(ax, kItLanes);
  ay = group_sum(ay, kItLanes);
  if (q != 0) return;
  for (int g = 0; g < a.ncomp; ++g) {
    a.gdelta[2 * (g * a.ncell + cell)] = dx[g];
    a.gdelta[2 * (g * a.ncell + cell) + 1] = dy[g];
  }
  a.gA[cell] = ax;
  a.gA[a.ncell + cell] = ay;
}

// explicit dependence of Omega on Delta at the cells:
// G_{Delta_G} += h^2 gOmega (2 ln(t/t_cG) Delta_G + 2 c sum_k w_k conj(eta_G,k) Delta_k)
__global__ void __launch_bounds__(256) omega_delta_adjoint_kernel(OmegaAdjArgs a) {
  const int64_t c = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (c >= a.ncg) return;
  const int cell = a.grain_cells[c];
  constexpr int MAXC = 4;
  double dx[MAXC], dy[MAXC], ox[MAXC], oy[MAXC];
  for (int g = 0; g < a.ncomp; ++g) {
    dx[g] = a.delta[2 * (static_cast<int64_t>(g) * a.ncell + cell)];
    dy[g] = a.delta[2 * (static_cast<int64_t>(g) * a.ncell + cell) + 1];
    ox[g] = 2.0 * a.logt[g] * dx[g];
    oy[g] = 2.0 * a.logt[g] * dy[g];
  }
  for (int k = 0; k < a.n_theta; ++k) {
    double kx = 0.0, ky = 0.0;
    for (int g = 0; g < a.ncomp; ++g) {
      const double ex = a.eta[2 * (g * a.n_theta + k)], ey = a.eta[2 * (g * a.n_theta + k) + 1];
      kx += ex * dx[g] - ey * dy[g];
      ky += ex * dy[g] + ey * dx[g];
    }
    const double s = 2.0 * a.twopi_rz * a.wk[k];
    for (int g = 0; g < a.ncomp; ++g) {
      const double ex = a.eta[2 * (g * a.n_theta + k)], ey = a.eta[2 * (g * a.n_theta + k) + 1];
      ox[g] += s * (ex * kx + ey * ky);
      oy[g] += s * (ex * ky - ey * kx);
    }
  }
  const double f = a.h2 * a.gomega;
  for (int g = 0; g < a.ncomp; ++g) {
    a.gdelta[2 * (static_cast<int64_t>(g) * a.ncell + cell)] += f * ox[g];
    a.gdelta[2 * (static_cast<int64_t>(g) * a.ncell + cell) + 1] += f * oy[g];
  }
}

// transpose of the curl B = d_x A_y - d_y A_x (central, one-sided at the
// edges): gA += s * D^T B
__global__ void __launch_bounds__(256) curl_adjoint_kernel(const double* __restrict__ B, double* __restrict__ gA,
                                                           int nx, int ny, double h, double s) {
  const int64_t c = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (c >= static_cast<int64_t>(nx) * ny) return;
  const int i = static_cast<int>(c % nx), j = static_cast<int>(c / nx);
  // d_x A_y at column i' uses A_y[i] with weights: collect from B at i' = i-1, i, i+1
  double gy = 0.0;
  for (int ip = i - 1; ip <= i + 1; ++ip) {
    if (ip < 0 || ip >= nx) continue;
    double w = 0.0;
    if (ip == 0) {
      w = (i == 1 ? 1.0 : (i == 0 ? -1.0 : 0.0)) / h;
    } else if (ip == nx - 1) {
      w = (i == nx - 1 ? 1.0 : (i == nx - 2 ? -1.0 : 0.0)) / h;
    } else {
      w = (i == ip + 1 ? 1.0 : (i == ip - 1 ? -1.0 : 0.0)) / (2 * h);
    }
    gy += w * B[static_cast<int64_t>(j) * nx + ip];
  }
  double gx = 0.0;
  for (int jp = j - 1; jp <= j + 1; ++jp) {
    if (jp < 0 || jp >= ny) continue;
    double w = 0.0;
    if (jp == 0) {
      w = (j == 1 ? 1.0 : (j == 0 ? -1.0 : 0.0)) / h;
    } else if (jp == ny - 1) {
      w = (j == ny - 1 ? 1.0 : (j == ny - 2 ? -1.0 : 0.0)) / h;
    } else {
      w = (j == jp + 1 ? 1.0 : (j == jp - 1 ? -1.0 : 0.0)) / (2 * h);
    }
    gx -= w * B[static_cast<int64_t>(jp) * nx + i];
  }
  gA[c] += s * gx;
  gA[static_cast<int64_t>(nx) * ny + c] += s * gy;
}

static inline unsigned nb(int64_t n) { return static_cast<unsigned>((n + 255) / 256); }

void launch_adjoint(int epl, const AdjArgs& a, const AdjBufs& b, hipStream_t st) {
  if (a.nseg == 0) return;
  const dim3 grid(static_cast<unsigned>((a.nseg * a.G + 63) / 64));
  switch (epl) {
    case 1: hipLaunchKernelGGL(adjoint_kernel<1>, grid, dim3(128), 0, st, a, b); break;
    case 2: hipLaunchKernelGGL(adjoint_kernel<2>, grid, dim3(128), 0, st, a, b); break;
    case 3: hipLaunchKernelGGL(adjoint_kernel<3>, grid, dim3(128), 0, st, a, b); break;
    case 4: hipLaunchKernelGGL(adjoint_kernel<4>, grid, dim3(128), 0, st, a, b); break;
    default: hipLaunchKernelGGL(adjoint_kernel<8>, grid, dim3(128), 0, st, a, b); break;
  }
}
void launch_back_adjoint(const BackAdjArgs& a, hipStream_t st) {
  if (a.nslot == 0) return;
  if (a.ncg > 0) hipLaunchKernelGGL(cell_grad_kernel, dim3(nb(a.ncg)), dim3(256), 0, st, a);
  hipLaunchKernelGGL(back_adjoint_kernel, dim3(nb(a.nslot * kBtLanes)), dim3(256), 0, st, a);
}
void launch_interp_adjoint(const InterpAdjArgs& a, hipStream_t st) {
  if (a.ncell > 0) hipLaunchKernelGGL(interp_adjoint_kernel, dim3(nb(a.ncell * kItLanes)), dim3(256), 0, st, a);
}
void launch_omega_delta_adjoint(const OmegaAdjArgs& a, hipStream_t st) {
  hipLaunchKernelGGL(omega_delta_adjoint_kernel, dim3(nb(a.ncg)), dim3(256), 0, st, a);
}
void launch_curl_adjoint(const double* B, double* gA, int nx, int ny, double h, double s, hipStream_t st) {
  hipLaunchKernelGGL(curl_adjoint_kernel, dim3(nb(static_cast<int64_t>(nx) * ny)), dim3(256), 0, st, B, gA, nx, ny,
                     h, s);
}

}  // namespace qc
