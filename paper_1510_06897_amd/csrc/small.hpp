// Plain recurrence step of one small problem (fewer than 64K sites and workgroups, 8 or 16 sites per
// workgroup), the same sums as step_kernel in the same order, bitwise.
//
// A launch this small is one wave's latency chain.  step_kernel reads its arguments in ten dependent
// rounds of scalar loads (role -> vector address, item fields behind branches) and takes seven integer
// divisions by run-time extents before its first vector load.  Here the host resolves the vectors, every
// argument is read in one burst at the start, the divisions are multiplications by reciprocals from the
// host, and all vector loads are issued before the first is waited for.  Overlap operator as a replayed
// graph, step_kernel -> this kernel (an empty launch in a graph is 2.2 us): 4^4 FP64 degree 63 262 ->
// 211 us (3.3 us per step), 8^3 x 16 FP32 degree 199 1065 -> 817 us (4.1), 11 x 7 x 9 x 13 FP32 3 vectors
// degree 99 778 -> 715 us (7.0).
#pragma once

#include "kernels.hpp"

namespace ovl {

// n / d for n, d < 2^16 by one high multiplication: m = ceil(2^32 / d), exact as n (m d - 2^32) < 2^32
struct SmallDiv {
  uint32_t d, m;  // m = 0: d = 1
};
inline SmallDiv small_div(int d) {
  return SmallDiv{(uint32_t)d, d == 1 ? 0u : (uint32_t)(0xffffffffu / (uint32_t)d + 1u)};
}
__device__ __forceinline__ uint32_t operator/(uint32_t n, const SmallDiv &q) {
  return q.m ? __umulhi(n, q.m) : n;
}

template <class C>
struct SmallArgs {
  const void *U, *v, *src, *w;  // src, w null: absent
  void *out;
  C kd, kh, a, t;
  SmallDiv lx, ly, lz, nrhs;
  int lt, remap, blocks;
  int v_g5, y_g5, src_g5;
};

template <class C, class SE, class LE, int SPB, int NQ, bool R12>
__global__ void __launch_bounds__(NQ * SPB) step_small_kernel(SmallArgs<C> p) {
  __shared__ cx<C> part[NQ][12][SPB];  // directional partial sums
  // every argument in scalar registers now: one round of loads
  asm volatile("" ::"s"(p.U), "s"(p.v), "s"(p.src), "s"(p.w), "s"(p.out), "s"(p.lt), "s"(p.remap),
               "s"(p.blocks));
  asm volatile("" ::"s"(p.lx.d), "s"(p.lx.m), "s"(p.ly.d), "s"(p.ly.m), "s"(p.lz.d), "s"(p.lz.m),
               "s"(p.nrhs.d), "s"(p.nrhs.m));
  asm volatile("" ::"s"(p.kd), "s"(p.kh), "s"(p.a), "s"(p.t), "s"(p.v_g5), "s"(p.y_g5), "s"(p.src_g5));
  const uint32_t gb = (uint32_t)xcd_block(blockIdx.x, p.blocks, p.remap);
  const uint32_t b = gb / p.nrhs, r = gb - b * p.nrhs.d;
  Ext4 ex;
  ex.lx = p.lx.d;
  ex.ly = p.ly.d;
  ex.lz = p.lz.d;
  ex.lt = p.lt;
  ex.sy = ex.lx;
  ex.sz = ex.lx * ex.ly;
  ex.st = ex.sz * ex.lz;
  ex.V = ex.st * ex.lt;
  const int V = ex.V;
  const int q = threadIdx.x / SPB, sl = threadIdx.x % SPB;
  const int dq = q & 3;
  const bool owner = q < 4;  // owns spin component q after the exchange
  const uint32_t site0 = b * SPB + sl;
  const bool active = site0 < (uint32_t)V;
  const uint32_t site = active ? site0 : 0u;
  Coord4 c4;
  {
    const uint32_t yy = site / p.lx, zz = yy / p.ly, tt = zz / p.lz;
    c4.x = (int)(site - yy * p.lx.d);
    c4.y = (int)(yy - zz * p.ly.d);
    c4.z = (int)(zz - tt * p.lz.d);
    c4.t = (int)tt;
  }
  int fwd, bwd;
  dir_neighbours(ex, c4, (int)site, dq, fwd, bwd);
  constexpr uint32_t ls = 64u * elem_traits<LE>::bytes;  // link component stride
  const uint32_t cs = (uint32_t)V * elem_traits<SE>::bytes, vb = 12u * cs;
  const int64_t ro = (int64_t)r * 12 * V;
  const rsrc_t v = make_rsrc((const SE *)p.v + ro, vb);
  const rsrc_t sr = make_rsrc((const SE *)(p.src ? p.src : p.v) + ro, p.src ? vb : 0u);
  const rsrc_t w = make_rsrc((const SE *)(p.w ? p.w : p.v) + ro, p.w ? vb : 0u);
  const rsrc_t o = make_rsrc((SE *)p.out + ro, vb);
  const rsrc_t U = make_rsrc(p.U, link_bytes(V, ls));
  const bool vg5 = p.v_g5 != 0, lower = q >= 2;
  const DirCoef<C> k = dir_coef<C>(dq);
  const uint32_t lane_links = (uint32_t)dq * 9u * 64u;
  const uint32_t e0 = (uint32_t)(3 * q) * (uint32_t)V + site;  // element of component 3q
  cx<C> acc[12];
#pragma unroll
  for (int i = 0; i < 12; ++i) acc[i] = mk<C>(0, 0);
  cx<C> vx[3], srcx[3], wx[3];
  auto own = [&]() {  // (with eight threads per site the upper four read past the vector: zero)
#pragma unroll
    for (int c = 0; c < 3; ++c) vx[c] = bldv<C, SE>(v, e0 + c * V);
#pragma unroll
    for (int c = 0; c < 3; ++c) srcx[c] = bldv<C, SE>(sr, e0 + c * V);
#pragma unroll
    for (int c = 0; c < 3; ++c) wx[c] = bldv<C, SE>(w, e0 + c * V);
  };
  if (NQ == 8) {
    const bool bw = q >= 4;
    cx<C> u[2][3], d[2][3], m[3][3], mm[3][3];
    load_spinor<C, SE>(v, cs, bw ? bwd : fwd, vg5, u, d);
    load_link3<C, LE>(U, ls, lane_links + link_lane(bw ? bwd : site), R12, m);
    own();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int x = 0; x < 3; ++x)
#pragma unroll
      for (int y = 0; y < 3; ++y) mm[x][y] = bw ? mk<C>(m[y][x].re, -m[y][x].im) : m[x][y];
    hop_apply<C, false>(acc, u, d, mm, k, bw ? C(-1) : C(1));
  } else {
    cx<C> u[2][3], d[2][3], m[3][3], u2[2][3], d2[2][3], m2[3][3];
    load_spinor<C, SE>(v, cs, fwd, vg5, u, d);
    load_link3<C, LE>(U, ls, lane_links + link_lane(site), R12, m);
    load_spinor<C, SE>(v, cs, bwd, vg5, u2, d2);
    load_link3<C, LE>(U, ls, lane_links + link_lane(bwd), R12, m2);
    own();
    __builtin_amdgcn_sched_barrier(0);
    hop_apply<C, false>(acc, u, d, m, k, C(1));
    hop_apply<C, true>(acc, u2, d2, m2, k, C(-1));
  }
#pragma unroll
  for (int i = 0; i < 12; ++i) part[q][i][sl] = acc[i];
  __syncthreads();
  if (!active || !owner) return;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    cx<C> hop = part[0][3 * q + c][sl] + part[1][3 * q + c][sl] + part[2][3 * q + c][sl] +
                part[3][3 * q + c][sl];
    if (NQ == 8)
      hop = hop + (part[4][3 * q + c][sl] + part[5][3 * q + c][sl] + part[6][3 * q + c][sl] +
                   part[7][3 * q + c][sl]);
    const C kd = p.kd, kh = p.kh;
    const cx<C> x = (vg5 && lower) ? -vx[c] : vx[c];
    // the roundings of step_kernel, spelled out
    cx<C> y = mk<C>(fma(kd, x.re, kh * hop.re), fma(kd, x.im, kh * hop.im));
    if (p.y_g5 && lower) y = -y;
    const C a = (p.src_g5 && lower) ? -p.a : p.a;
    cx<C> res = mk<C>(fma(a, srcx[c].re, y.re), fma(a, srcx[c].im, y.im));
    res = mk<C>(fma(p.t, wx[c].re, res.re), fma(p.t, wx[c].im, res.im));
    bstv<C, SE>(o, e0 + c * V, res);
  }
}

}  // namespace ovl
