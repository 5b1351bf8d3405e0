// Leaf-to-root walks of the kinematic-tree models whose constraint blocks are full poses, full
// relative poses, rods and centre-of-mass rows.
//
// The step J^T (J J^T + lambda I)^-1 F does not change when a block's rows are replaced by T^-1 of
// them (with lambda I replaced by lambda T^-1 T^-T). The passes here use the rows in which the
// Jacobian is cheapest: the body twist of the block's end frame f,
//   POSE  rows [R_f^T (p_f - p_ref); w],       w = log(R_ref^T R_f)^v
//   REL   rows [R_rel^T (p_rel - p_ref); w],   T_rel = T_a^-1 T_b, w = log(R_ref^T R_rel)^v
// T is orthogonal in the linear rows and J_r^-1(w) in the angular ones (J_r w = w, so the angular
// residual is w itself), lambda T^-1 T^-T is lambda on the linear rows and lambda J_r J_r^T on the
// angular ones, and ||F|| is the same in both bases. DIST, COM and HULL rows keep their form.
//
// With X_j = (R, p) the pose of frame f in the frame of joint j, the column of a revolute joint about
// axis a is [R^T (e_a x p); R^T e_a]: row a of R, and a combination of its two other rows (6
// multiplications), where world rows cost a cross product and two matrix products. X is built from
// the leaf to the root, X <- O_j Q_j X: the origin translation is then an addition of constants, no
// stack of link frames is kept, and the chains of the two arms (or legs) are independent work that
// hides each other's latency. The centre of mass comes from the same walk: h_j, the first moment of
// the subtree of j in its frame, h_parent += O_j Q_j h_j with the constant parts folded on the host (in
// FP32 steps an FP32 recursion: the humanoid's CoM columns are off by 1.0e-8 root mean square, against
// 3.6e-8 for differences of whole-body prefix sums).
// J^T y is the recursion of the wrench y up the chain: force and moment are rotated and shifted, and
// the joint's entry is the moment's axis component, so no column is formed a second time.
//
// Walk order: Topo::walk, pairs of joints of the two sides, every joint after its children.
#pragma once

#include "kin.hpp"
#include "trig.hpp"

namespace mc {

template <class Topo>
struct Leaf {
  static constexpr bool trig = true;
  using KI = KInfo<Topo>;
  static constexpr int NJ = Topo::NJ, NB = Topo::NB, NF = Topo::NF, M = Topo::M, D = Topo::NJ;
  static constexpr uint32_t ALL = ~uint32_t(0);
  static constexpr bool com = Topo::has_com;

  // ---------------------------------------------------------------- structure
  static constexpr bool in_rows(uint32_t rm, int r) { return (rm >> r) & 1u; }
  static constexpr bool sel(uint32_t rm, int b) { return (KI::brmask(b) & rm) != 0; }
  // Ends: the frames whose poses the walk carries. End 2b is frame fa of block b, end 2b + 1 frame fb.
  static constexpr int NE = 2 * NB;
  static constexpr bool is_pose(int b) { return Topo::btype[b] == B_POSE; }
  static constexpr bool is_rel(int b) { return Topo::btype[b] == B_REL; }
  static constexpr bool is_dist(int b) { return Topo::btype[b] == B_DIST; }
  static constexpr bool end_used(int e) {
    const int b = e / 2;
    return e % 2 == 0 ? (is_pose(b) || is_rel(b) || is_dist(b)) : (is_rel(b) || is_dist(b));
  }
  static constexpr int end_frame(int e) { return e % 2 == 0 ? Topo::bfa[e / 2] : Topo::bfb[e / 2]; }
  static constexpr int end_link(int e) { return Topo::frame_link[end_frame(e)]; }
  // the chain of an end ends below this link (-1: the world): the last common ancestor of a block's ends
  static constexpr int stop_link(int b) {
    if (is_pose(b)) return -1;
    for (int k = end_link(2 * b); k >= 0; k = Topo::parent[k])
      if (KI::anc(k, end_link(2 * b + 1))) return k;
    return -1;
  }
  static constexpr bool on(int e, int j) {  // joint j is on the chain of end e
    if (!end_used(e) || !KI::anc(j, end_link(e))) return false;
    const int s = stop_link(e / 2);
    return !(s >= 0 && KI::anc(j, s));
  }
  static constexpr bool has_chain(int e) { return end_link(e) != stop_link(e / 2); }
  struct Pos { int v[NJ]; };
  static constexpr Pos pos_table() {
    Pos t{};
    for (int j = 0; j < NJ; ++j) t.v[j] = -1;
    for (int g = 0; g < Topo::NG; ++g)
      for (int k = 0; k < 2; ++k)
        if (Topo::walk[g][k] >= 0) t.v[Topo::walk[g][k]] = 2 * g + k;
    return t;
  }
  static constexpr Pos POS = pos_table();
  static constexpr int pos(int j) { return POS.v[j]; }  // slot of joint j in the walk
  // the joint after which both chains of block b are complete
  static constexpr int last_joint(int b) {
    int best = -1;
    for (int j = 0; j < NJ; ++j)
      if ((on(2 * b, j) || on(2 * b + 1, j)) && (best < 0 || pos(j) > pos(best))) best = j;
    return best;
  }
  static constexpr bool first_child(int j) {
    for (int k = 0; k < NJ; ++k)
      if (k != j && Topo::parent[k] == Topo::parent[j] && pos(k) < pos(j)) return false;
    return true;
  }
  static constexpr bool has_child(int j) {
    for (int k = 0; k < NJ; ++k)
      if (Topo::parent[k] == j) return true;
    return false;
  }
  static constexpr bool order_ok() {
    for (int j = 0; j < NJ; ++j) {
      if (pos(j) < 0) return false;
      if (Topo::parent[j] >= 0 && pos(Topo::parent[j]) / 2 <= pos(j) / 2) return false;
    }
    return true;
  }
  // the end whose chain carries the world rotation for the CoM column of joint j (-1: none does)
  static constexpr int com_end(int j) {
    for (int e = 0; e < NE; ++e)
      if (on(e, j) && !is_dist(e / 2)) return e;
    return -1;
  }
  // links whose world rotation (two rows) a root-to-leaf walk provides: joints on no chain, the links
  // where relative chains stop, and their ancestors
  static constexpr bool pw_needed(int l) {
    if (com_end(l) < 0) return true;
    for (int b = 0; b < NB; ++b)
      if (is_rel(b) && stop_link(b) == l) return true;
    return false;
  }
  static constexpr bool pw_walk(int j) {
    for (int l = 0; l < NJ; ++l)
      if (pw_needed(l) && KI::anc(j, l)) return true;
    return false;
  }
  // ends of pose blocks in the rows rm that continue as one from joint j on: the end that stands for e there
  static constexpr int leader(uint32_t rm, int e, int j) {
    for (int k = 0; k < e; ++k)
      if (on(k, j) && is_pose(k / 2) && is_pose(e / 2) && sel(rm, k / 2)) return k;
    return e;
  }
  static constexpr int child_on(int e, int j) {  // the joint below j on the chain of e (-1: e starts at j)
    for (int k = 0; k < NJ; ++k)
      if (Topo::parent[k] == j && on(e, k)) return k;
    return -1;
  }
  static constexpr bool com_block(int b) { return Topo::btype[b] == B_COM || Topo::btype[b] == B_HULL; }
  static constexpr bool com_rows(uint32_t rm) {
    for (int b = 0; b < NB; ++b)
      if (com_block(b) && sel(rm, b)) return true;
    return false;
  }

  // Per-iteration data from the residual pass for the step passes.
  template <class S>
  struct SD {
    S PW[NB][6];    // POSE: first two rows of the end frame's world rotation (CoM columns)
    S rel[NB][12];  // REL: T_a^-1 T_b (rotation, translation)
    S Rb[NB][9];    // REL: rotation of frame b in the frame of the link where the chains meet
    S u[NB][3];     // DIST: unit vector from end a to end b in that link's frame
    S H[NB][3];     // HULL: the lane's 2 x 2 row map [h0 h1; 0 h2]
    uint32_t drop = 0;
  };

  // The change of row basis T at a point, for callers that need the scene's own rows (POSE rows with their linear part
  // in the world's axes, REL rows in frame a's, both constant rotations of them): y' = T^T y.
  struct Basis {
    double R[NB][9];  // POSE: rotation of the end frame; REL: R_a^T R_b
    double w[NB][3];
  };

  // ---------------------------------------------------------------- joint data
  template <class T>
  struct JD {
    T q, s, c;   // coordinate, sine, cosine
    T o[3];      // origin translation
    T R[9];      // origin rotation (when the topology has rotated origins)
    T hc[3];     // first moment of the link and of its children's origins
    T m;         // subtree mass (prismatic and root joints)
  };
  static constexpr int STRIDE = Topo::origin_rot ? 16 : 8;
  static_assert(!(Topo::origin_rot && com), "the packed constants hold rotations or moments");
  // What the walk reads ahead besides the joints' own data: frames of the ends that start at a group
  template <class T>
  struct Frames {
    T p[NE][3], R[NE][9];
  };
  // Constants of the joints of group g, with wide scalar loads.
  template <class T, int g>
  static __device__ __forceinline__ void load_consts(JD<T>* r, Frames<T>& fr, const TP<T>& P0) {
    // (V8 is read behind the first four elements of a rotated joint's sixteen, which start at a multiple of 64 bytes)
    typedef T V8 __attribute__((ext_vector_type(8), aligned(16)));  // (an alias declaration would drop the alignment)
    static_assert(alignof(V8) <= 4 * sizeof(T), "V8 is read at c + 4");
    using V4 = T __attribute__((ext_vector_type(4)));
    using V2 = T __attribute__((ext_vector_type(2)));
    const TP<T>& P = fresh_const(P0);
    sfor<0, 2>([&](auto K) {
      constexpr int kk = decltype(K)::value, j = Topo::walk[g][kk];
      if constexpr (j >= 0) {
        const T* c = P.jc + (2 * g + kk) * STRIDE;
        JD<T>& d = r[kk];
        if constexpr (Topo::origin_rot) {
          const V4 a = *(const V4*)c;
          const V8 b = *(const V8*)(c + 4);
          for (int k = 0; k < 3; ++k) d.o[k] = a[k];
          d.R[0] = a[3];
          for (int k = 0; k < 8; ++k) d.R[1 + k] = b[k];
        } else if constexpr (std::is_same<T, float>::value) {
          const V8 a = *(const V8*)c;
          for (int k = 0; k < 3; ++k) {
            d.o[k] = a[k];
            d.hc[k] = a[3 + k];
          }
          d.m = a[6];
        } else {
          const V4 a = *(const V4*)c;
          const V2 b = *(const V2*)(c + 4);
          for (int k = 0; k < 3; ++k) d.o[k] = a[k];
          d.hc[0] = a[3];
          d.hc[1] = b[0];
          d.hc[2] = b[1];
          if constexpr (Topo::jtype[j] == PRI || Topo::parent[j] < 0) d.m = c[6];
        }
        sfor<0, NE>([&](auto E) {
          constexpr int e = decltype(E)::value;
          if constexpr (on(e, j) && end_link(e) == j) {
            for (int k = 0; k < 3; ++k) fr.p[e][k] = P.fp[end_frame(e)][k];
            if constexpr (Topo::frame_rot)
              for (int k = 0; k < 9; ++k) fr.R[e][k] = P.fR[end_frame(e)][k];
          }
        });
      }
    });
  }
  // sines and cosines (coordinates of prismatic joints) of a compile-time list of joints, outside the walk: read together
  template <class S, class List, class Q, class TR>
  static __device__ __forceinline__ void load_list(const Q& q0, const TR& tr0, JD<S>* d) {
    const Q q = q0.fresh();
    const TR tr = tr0.fresh();
    double x[List::N];
    sfor<0, List::N>([&](auto I) {
      constexpr int i = decltype(I)::value, j = List::at(i);
      if constexpr (TR::tile) {
        const auto v = tr.get(j);
        d[i].q = d[i].s = v.x;
        d[i].c = v.y;
      } else {
        x[i] = q.get(j);
      }
    });
    if constexpr (!TR::tile) {
      sfor<0, List::N>([&](auto I) {
        constexpr int i = decltype(I)::value;
        double s, c;
        sincos_tab<std::is_same<S, double>::value && TR::exact>(x[i], tr.tab, s, c);
        d[i].q = S(x[i]);
        d[i].s = S(s);
        d[i].c = S(c);
      });
    }
  }

  // c a - s b and c b + s a. In FP64 the cosine's product is the one that is not rounded by itself: it is the larger one for
  // most joints, and a rounding at the size of the result is the least there is.
  template <class T>
  static __device__ __forceinline__ void rotate(const JD<T>& d, T a, T b, T& x, T& y) {
    if constexpr (std::is_same<T, double>::value) {
      x = __builtin_fma(d.c, a, -(d.s * b));
      y = __builtin_fma(d.c, b, d.s * a);
    } else {
      x = d.c * a - d.s * b;
      y = d.s * a + d.c * b;
    }
  }
  // v <- O_j Q_j v for a free vector
  template <int j, class T>
  static __device__ __forceinline__ void up_vec(const JD<T>& d, T* v) {
    constexpr int ax = Topo::axis[j], i = (ax + 1) % 3, k = (ax + 2) % 3;
    if constexpr (Topo::jtype[j] == REV) {
      rotate(d, v[i], v[k], v[i], v[k]);
    }
    if constexpr (Topo::origin_rot) {
      T t[3];
      matvec3(d.R, v, t);
      for (int r = 0; r < 3; ++r) v[r] = t[r];
    }
  }
  template <int j, class T>
  static __device__ __forceinline__ void up_point(const JD<T>& d, T* p) {
    constexpr int ax = Topo::axis[j], i = (ax + 1) % 3, k = (ax + 2) % 3;
    if constexpr (std::is_same<T, double>::value && Topo::jtype[j] == REV && !Topo::origin_rot) {
      const T a = p[i], b = p[k];  // (the origin inside the products' sum: two roundings in place of three)
      p[i] = __builtin_fma(d.c, a, __builtin_fma(-d.s, b, d.o[i]));
      p[k] = __builtin_fma(d.c, b, __builtin_fma(d.s, a, d.o[k]));
      p[ax] += d.o[ax];
    } else {
      if constexpr (Topo::jtype[j] == PRI) p[ax] += d.q;
      up_vec<j>(d, p);
      for (int r = 0; r < 3; ++r) p[r] += d.o[r];
    }
  }
  // R <- O_j Q_j R (columns of R are free vectors); identity: R is the identity before
  template <int j, bool identity, class T>
  static __device__ __forceinline__ void up_rot(const JD<T>& d, T* R) {
    constexpr int ax = Topo::axis[j], i = (ax + 1) % 3, k = (ax + 2) % 3;
    if constexpr (Topo::jtype[j] == REV) {
      if constexpr (identity) {
        R[3 * i + i] = d.c;
        R[3 * i + k] = -d.s;
        R[3 * k + i] = d.s;
        R[3 * k + k] = d.c;
      } else {
        for (int m = 0; m < 3; ++m) {
          rotate(d, R[3 * i + m], R[3 * k + m], R[3 * i + m], R[3 * k + m]);
        }
      }
    }
    if constexpr (Topo::origin_rot) {
      T t[9];
      matmul3(d.R, R, t);
      for (int r = 0; r < 9; ++r) R[r] = t[r];
    }
  }
  // first moment of the subtree of j in its frame; hs[l + 1] holds the sum of the children of link l
  template <int j, class T>
  static __device__ __forceinline__ void subtree_h(const T (*hs)[3], const JD<T>& d, T* h) {
    if constexpr (has_child(j)) {
      for (int r = 0; r < 3; ++r) h[r] = hs[j + 1][r] + d.hc[r];
    } else {
      for (int r = 0; r < 3; ++r) h[r] = d.hc[r];
    }
  }
  template <int j, class T>
  static __device__ __forceinline__ void push_h(T (*hs)[3], const JD<T>& d, T* h) {
    if constexpr (Topo::jtype[j] == PRI) h[Topo::axis[j]] += d.m * d.q;
    up_vec<j>(d, h);
    constexpr int par = Topo::parent[j];
    for (int r = 0; r < 3; ++r) {
      if constexpr (par < 0) h[r] += d.m * d.o[r];
      if constexpr (first_child(j)) hs[par + 1][r] = h[r];
      else hs[par + 1][r] += h[r];
    }
  }

  // The walk: visit(ic<j>, data, frames) for the joints of each group in turn, ahead<g>() where group g's loads are issued.
  // A single wave per SIMD has nothing else to hide a load behind, and scalar and LDS reads share one counter
  // that can only be waited down to zero together: so each group is a stage that first issues every read the
  // stages after it need (joint constants of the next group; with stored sines those of the next group, else
  // the table entries of the group after the next and the coordinates of the one behind it) and then computes;
  // the scheduler may not move anything across the two marks. A stage waits once, for reads a whole stage old.
  template <class T, bool STORE, class Q, class TR, class V, class A>
  static __device__ __forceinline__ void walk(const Q& q0, const TP<T>& P, const TR& tr0, V&& visit, A&& ahead) {
    constexpr int NG = Topo::NG;
    constexpr bool read = TR::tile && !STORE;
    const Q q = q0.fresh();
    const TR tr = tr0.fresh();
    JD<T> d[NG][2];
    Frames<T> fr;
    double x[NG][2], kr[NG][2];
    SinTabE t[NG][2];
    auto slots = [&](auto G, auto&& fn) {
      constexpr int g = decltype(G)::value;
      if constexpr (g < NG) {
        if constexpr (Topo::walk[g][0] >= 0) fn(ic<Topo::walk[g][0]>{}, ic<0>{});
        if constexpr (Topo::walk[g][1] >= 0) fn(ic<Topo::walk[g][1]>{}, ic<1>{});
      }
    };
    auto fetch_tile = [&](auto G) {
      constexpr int g = decltype(G)::value;
      slots(G, [&](auto J, auto K) {
        if constexpr (TR::tile) {
          constexpr int j = decltype(J)::value, k = decltype(K)::value;
          const auto v = tr.get(j);
          d[g][k].q = d[g][k].s = v.x;
          d[g][k].c = v.y;
        }
      });
    };
    auto fetch_q = [&](auto G) {
      constexpr int g = decltype(G)::value;
      slots(G, [&](auto J, auto K) { x[g][decltype(K)::value] = q.get(decltype(J)::value); });
    };
    auto fetch_tab = [&](auto G) {
      constexpr int g = decltype(G)::value;
      slots(G, [&](auto J, auto K) {
        constexpr int k = decltype(K)::value;
        if constexpr (Topo::jtype[decltype(J)::value] == REV) t[g][k] = sin_tab_entry(x[g][k], tr.tab, kr[g][k]);
      });
    };
    auto finish_trig = [&](auto G) {
      constexpr int g = decltype(G)::value;
      slots(G, [&](auto J, auto K) {
        constexpr int j = decltype(J)::value, k = decltype(K)::value;
        if constexpr (Topo::jtype[j] == PRI) {
          d[g][k].q = T(x[g][k]);
          if constexpr (TR::tile) tr.set(j, float(x[g][k]), 0.f);
        } else {
          double sn, cs;
          sincos_finish<std::is_same<T, double>::value && TR::exact>(x[g][k], kr[g][k], t[g][k], sn, cs);
          d[g][k].s = T(sn);
          d[g][k].c = T(cs);
          if constexpr (TR::tile) tr.set(j, float(sn), float(cs));
        }
      });
    };
    // rotated origins in FP64 are 24 scalar registers a joint: read at their own stage
    constexpr bool late = Topo::origin_rot && std::is_same<T, double>::value;
    if constexpr (!late) load_consts<T, 0>(d[0], fr, P);
    if constexpr (read) {
      fetch_tile(ic<0>{});
    } else {
      fetch_q(ic<0>{});
      fetch_q(ic<1>{});
      fetch_q(ic<2>{});
      __builtin_amdgcn_sched_barrier(0);
      fetch_tab(ic<0>{});
      fetch_tab(ic<1>{});
      __builtin_amdgcn_sched_barrier(0);
      finish_trig(ic<0>{});
    }
    sfor<0, NG>([&](auto G) {
      constexpr int g = decltype(G)::value;
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (late) load_consts<T, g>(d[g], fr, P);
      else if constexpr (g + 1 < NG) load_consts<T, (g + 1 < NG ? g + 1 : g)>(d[g + 1 < NG ? g + 1 : g], fr, P);
      ahead(G);
      if constexpr (read) {
        fetch_tile(ic<g + 1>{});
      } else {
        fetch_tab(ic<g + 2>{});
        fetch_q(ic<g + 3>{});
      }
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (!read) finish_trig(ic<g + 1>{});
      slots(G, [&](auto J, auto K) { visit(J, d[g][decltype(K)::value], fr); });
    });
    __builtin_amdgcn_sched_barrier(0);
  }

  template <int e, class T>
  static __device__ __forceinline__ void start_end(const Frames<T>& fr, Rig<T>& X) {
    for (int k = 0; k < 9; ++k) X.R[k] = Topo::frame_rot ? fr.R[e][k] : ((k % 4 == 0) ? T(1) : T(0));
    for (int k = 0; k < 3; ++k) X.p[k] = fr.p[e][k];
  }

  // ---------------------------------------------------------------- residual
  // constants of the blocks that end at a group, read at its start
  struct BlockConsts {
    double Rt[NB][9], p[NB][3], fa[NB][3], len[NB];
  };
  template <int g>
  static __device__ __forceinline__ void load_blocks(BlockConsts& bc, const TP<double>& P0) {
    sfor<0, NB>([&](auto BI) {
      constexpr int b = decltype(BI)::value;
      if constexpr (!com_block(b)) {
        if constexpr (pos(last_joint(b)) / 2 == g) {
          const TP<double>& P = fresh_const(P0);
          if constexpr (is_dist(b)) {
            bc.len[b] = P.target[b][0];
            for (int k = 0; k < 3; ++k) bc.fa[b][k] = P.fp[end_frame(2 * b)][k];
          } else {
            for (int k = 0; k < 9; ++k) bc.Rt[b][k] = P.refRt[b][k];
            for (int k = 0; k < 3; ++k) bc.p[b][k] = P.refp[b][k];
          }
        }
      }
    });
  }
  template <int b, bool WITH_F, class S>
  static __device__ __forceinline__ void finish_block(Rig<double>* X, const BlockConsts& bc, S* F, double& n2, SD<S>& sd,
                                                      double (*sc)[4], Basis* basis) {
    constexpr int r0 = KI::brow0(b);
    Rig<double>& A = X[2 * b];
    static_assert(has_chain(2 * b) || is_dist(b), "a chain that ends where it starts: rods only");
    static_assert(!end_used(2 * b + 1) || has_chain(2 * b + 1), "second ends have a chain");
    if constexpr (!has_chain(2 * b))
      for (int k = 0; k < 3; ++k) A.p[k] = bc.fa[b][k];
    if constexpr (is_pose(b) || is_rel(b)) {
      double dp[3], Rr[9];
      const double* Rt = bc.Rt[b];
      if constexpr (is_pose(b)) {
        for (int k = 0; k < 3; ++k) dp[k] = A.p[k] - bc.p[b][k];
        for (int k = 0; k < 9; ++k) Rr[k] = A.R[k];
        if constexpr (com)
          for (int k = 0; k < 6; ++k) sd.PW[b][k] = to_step<S>(A.R[k]);
      } else {
        const Rig<double>& B = X[2 * b + 1];
        const double t[3] = {B.p[0] - A.p[0], B.p[1] - A.p[1], B.p[2] - A.p[2]};
        for (int i = 0; i < 3; ++i) {
          const double pr = A.R[i] * t[0] + A.R[3 + i] * t[1] + A.R[6 + i] * t[2];
          sd.rel[b][9 + i] = to_step<S>(pr);
          dp[i] = pr - bc.p[b][i];
          for (int k = 0; k < 3; ++k)
            Rr[3 * i + k] = A.R[i] * B.R[k] + A.R[3 + i] * B.R[3 + k] + A.R[6 + i] * B.R[6 + k];
        }
        for (int k = 0; k < 9; ++k) sd.rel[b][k] = to_step<S>(Rr[k]);
        if constexpr (com)
          for (int k = 0; k < 9; ++k) sd.Rb[b][k] = to_step<S>(B.R[k]);
      }
      if constexpr (WITH_F) {
        if (basis)
          for (int k = 0; k < 9; ++k) basis->R[b][k] = Rr[k];
        // sin(theta) times the axis and cos(theta) of R_ref^T Rr, from the entries they need
        auto re = [&](int i, int k) { return Rt[3 * i] * Rr[k] + Rt[3 * i + 1] * Rr[3 + k] + Rt[3 * i + 2] * Rr[6 + k]; };
        sc[b][0] = 0.5 * (re(2, 1) - re(1, 2));
        sc[b][1] = 0.5 * (re(0, 2) - re(2, 0));
        sc[b][2] = 0.5 * (re(1, 0) - re(0, 1));
        sc[b][3] = 0.5 * (re(0, 0) + re(1, 1) + re(2, 2) - 1.0);
        for (int k = 0; k < 3; ++k) {
          F[r0 + k] = to_step<S>(Rr[k] * dp[0] + Rr[3 + k] * dp[1] + Rr[6 + k] * dp[2]);
          n2 += dp[k] * dp[k];
        }
      }
    } else if constexpr (is_dist(b)) {
      const Rig<double>& B = X[2 * b + 1];
      const double dv[3] = {B.p[0] - A.p[0], B.p[1] - A.p[1], B.p[2] - A.p[2]};
      const double len = sqrt(dv[0] * dv[0] + dv[1] * dv[1] + dv[2] * dv[2]);
      if constexpr (WITH_F) {
        const double e = len - bc.len[b];
        F[r0] = to_step<S>(e);
        n2 += e * e;
      }
      const double il = 1.0 / len;
      for (int k = 0; k < 3; ++k) sd.u[b][k] = to_step<S>(dv[k] * il);
    }
  }

  // theta / sin(theta) of every pose block. Near the manifold (theta < pi/2, sin^2 < 0.01) the series of asin(s) / s, to
  // s^14 (remainder below 2e-18); else from the angle itself, which a wave computes only where some lane needs it (each
  // lane's value depends on its own angle alone).
  static __device__ __forceinline__ void angle_factors(const double (*sc)[4], double* f) {
    double s2[NB];
    bool far = false;
    sfor<0, NB>([&](auto BI) {
      constexpr int b = decltype(BI)::value;
      if constexpr (is_pose(b) || is_rel(b)) {
        s2[b] = sc[b][0] * sc[b][0] + sc[b][1] * sc[b][1] + sc[b][2] * sc[b][2];
        double p = __builtin_fma(s2[b], 143.0 / 10240.0, 231.0 / 13312.0);
        p = __builtin_fma(p, s2[b], 63.0 / 2816.0);
        p = __builtin_fma(p, s2[b], 35.0 / 1152.0);
        p = __builtin_fma(p, s2[b], 5.0 / 112.0);
        p = __builtin_fma(p, s2[b], 3.0 / 40.0);
        p = __builtin_fma(p, s2[b], 1.0 / 6.0);
        f[b] = __builtin_fma(p, s2[b], 1.0);
        far = far || !(sc[b][3] > 0.0 && s2[b] < 0.01);
      }
    });
    if (__any(far)) {
      sfor<0, NB>([&](auto BI) {
        constexpr int b = decltype(BI)::value;
        if constexpr (is_pose(b) || is_rel(b)) {
          const double sn = sqrt(s2[b]);
          const double g = angle_from_sincos(sn, sc[b][3]) / sn;
          f[b] = (sc[b][3] > 0.0 && s2[b] < 0.01) ? f[b] : g;
        }
      });
    }
  }

  // Residual pass in FP64: returns ||F(q)||^2; F in the rows above and the step data, in precision S.
  // (every row is evaluated: RM is the Direct passes' row selection)
  template <class S, uint32_t RM = ALL, class Q, class TR>
  static __device__ __forceinline__ double residual(const Q& q, const Consts& P, S* F, SD<S>& sd, const TR& tr) {
    return residual_pass<S, true>(q, P, F, sd, tr);
  }
  // with the change of row basis
  template <class Q, class TR>
  static __device__ __forceinline__ void residual_basis(const Q& q, const Consts& P, double* F, SD<double>& sd, Basis& bs,
                                                        const TR& tr) {
    residual_pass<double, true>(q, P, F, sd, tr, &bs);
  }
  // the step data alone
  template <class S, class Q, class TR>
  static __device__ __forceinline__ void step_data(const Q& q, const Consts& P, SD<S>& sd, const TR& tr) {
    S F[M];
    residual_pass<S, false>(q, P, F, sd, tr);
  }
  template <class S, bool WITH_F, class Q, class TR>
  static __device__ __forceinline__ double residual_pass(const Q& q, const Consts& P, S* F, SD<S>& sd, const TR& tr,
                                                         Basis* basis = nullptr) {
    Rig<double> X[NE];
    double hs[NJ + 1][3];
    double sc[NB][4];
    double n2 = 0.0;
    BlockConsts bc;
    walk<double, true>(
        q, P.d, tr,
        [&](auto J, const JD<double>& d, const Frames<double>& fr) {
          constexpr int j = decltype(J)::value;
          sfor<0, NE>([&](auto E) {
            constexpr int e = decltype(E)::value;
            if constexpr (on(e, j)) {
              if constexpr (end_link(e) == j) start_end<e>(fr, X[e]);
              up_point<j>(d, X[e].p);
              if constexpr (!is_dist(e / 2)) up_rot<j, !Topo::frame_rot && end_link(e) == j>(d, X[e].R);
            }
          });
          if constexpr (com) {
            double h[3];
            subtree_h<j>(hs, d, h);
            push_h<j>(hs, d, h);
          }
          sfor<0, NB>([&](auto BI) {
            constexpr int b = decltype(BI)::value;
            if constexpr (last_joint(b) == j) finish_block<b, WITH_F>(X, bc, F, n2, sd, sc, basis);
          });
        },
        [&](auto G) { load_blocks<decltype(G)::value>(bc, P.d); });
    if constexpr (com && (WITH_F || has_hull())) {
      // (pinned ahead of the branch below: the compiler would sink the whole moment recursion past it)
      const TP<double>& Pd = fresh_const(P.d);
      const double x = opaque(hs[0][0] * Pd.inv_total_mass), y = opaque(hs[0][1] * Pd.inv_total_mass);
      sfor<0, NB>([&](auto BI) {
        constexpr int b = decltype(BI)::value;
        if constexpr (Topo::btype[b] == B_COM && WITH_F) {
          constexpr int r0 = KI::brow0(b);
          const double e0 = x - Pd.target[b][0], e1 = y - Pd.target[b][1];
          F[r0] = to_step<S>(e0);
          F[r0 + 1] = to_step<S>(e1);
          n2 += e0 * e0 + e1 * e1;
        } else if constexpr (Topo::btype[b] == B_HULL) {
          Kin<Topo>::template hull_rows<S, b>(x, y, P, F, n2, sd);  // (its row map is step data)
        }
      });
    }
    if constexpr (!WITH_F) return 0.0;
    double fa[NB];
    angle_factors(sc, fa);
    sfor<0, NB>([&](auto BI) {
      constexpr int b = decltype(BI)::value;
      if constexpr (is_pose(b) || is_rel(b)) {
        for (int k = 0; k < 3; ++k) {
          const double w = fa[b] * sc[b][k];
          if (basis) basis->w[b][k] = w;
          F[KI::brow0(b) + 3 + k] = to_step<S>(w);
          n2 += w * w;
        }
      }
    });
    return n2;
  }

  // y' = T^T c (FORWARD) or its inverse c = T^-T y', in place: the rotations R^T and R on the linear rows, the inverse left
  // Jacobian J_l^-1(w) and J_l(w) on the angular ones (J_l = I + B [w]x + C [w]x^2, J_l^-1 = I - [w]x / 2 + beta [w]x^2).
  template <bool FORWARD, class TR>
  static __device__ __forceinline__ void change_rows(const Basis& bs, const TR& tr, double* y) {
    sfor<0, NB>([&](auto BI) {
      constexpr int b = decltype(BI)::value, r0 = KI::brow0(b);
      if constexpr (is_pose(b) || is_rel(b)) {
        const double* R = bs.R[b];
        const double* w = bs.w[b];
        double l[3];
        for (int k = 0; k < 3; ++k)
          l[k] = FORWARD ? R[k] * y[r0] + R[3 + k] * y[r0 + 1] + R[6 + k] * y[r0 + 2]
                         : R[3 * k] * y[r0] + R[3 * k + 1] * y[r0 + 1] + R[3 * k + 2] * y[r0 + 2];
        for (int k = 0; k < 3; ++k) y[r0 + k] = l[k];
        const double t2 = w[0] * w[0] + w[1] * w[1] + w[2] * w[2];
        double B, C;  // of J_l; for the inverse B = -1/2, C = beta
        if (t2 < 0.1) {  // series to theta^10, remainders below 1e-17
          if constexpr (FORWARD) {
            C = 1.0 / 12 + t2 * (1.0 / 720 + t2 * (1.0 / 30240 + t2 * (1.0 / 1209600 + t2 * (1.0 / 47900160 + t2 * (691.0 / 1307674368000.0)))));
          } else {
            B = 0.5 - t2 * (1.0 / 24 - t2 * (1.0 / 720 - t2 * (1.0 / 40320 - t2 * (1.0 / 3628800 - t2 / 479001600.0))));
            C = 1.0 / 6 - t2 * (1.0 / 120 - t2 * (1.0 / 5040 - t2 * (1.0 / 362880 - t2 * (1.0 / 39916800 - t2 / 6227020800.0))));
          }
        } else {
          const double th = sqrt(t2);
          double sn, cs;
          sincos_tab(th, tr.tab, sn, cs);
          if constexpr (FORWARD) {
            C = 1.0 / t2 - (1.0 + cs) / (2.0 * th * sn);
          } else {
            B = (1.0 - cs) / t2;
            C = (th - sn) / (t2 * th);
          }
        }
        if constexpr (FORWARD) B = -0.5;
        double* a = y + r0 + 3;
        double c1[3], c2[3];
        cross3(w, a, c1);
        cross3(w, c1, c2);
        for (int k = 0; k < 3; ++k) a[k] += B * c1[k] + C * c2[k];
      }
    });
  }
  // Take the base point's choice of rows (dropped rows, polygon row map) into sd: the smooth piece that is active there.
  static __device__ __forceinline__ void freeze_rows(SD<double>& sd, const SD<double>& base) {
    sd.drop = base.drop;
    sfor<0, NB>([&](auto BI) {
      constexpr int b = decltype(BI)::value;
      if constexpr (Topo::btype[b] == B_HULL)
        for (int k = 0; k < 3; ++k) sd.H[b][k] = base.H[b][k];
    });
  }

  // ---------------------------------------------------------------- step passes
  static constexpr int pw_count() {
    int n = 0;
    for (int j = 0; j < NJ; ++j) n += pw_walk(j) ? 1 : 0;
    return n;
  }
  struct PwList {
    static constexpr int N = pw_count();
    static constexpr int at(int i) {
      for (int j = 0; j < NJ; ++j)
        if (pw_walk(j) && i-- == 0) return j;
      return -1;
    }
  };
  // First two rows of the world rotation of the links in pw_walk (root to leaf).
  template <class S, class Q, class TR>
  static __device__ __forceinline__ void world_rows(const Q& q, const TR& tr, S (*pw)[6]) {
    constexpr int N = PwList::N;
    JD<S> d[N];
    load_list<S, PwList>(q, tr, d);
    sfor<0, N>([&](auto I) {
      constexpr int n = decltype(I)::value, j = PwList::at(n);
      constexpr int par = Topo::parent[j], ax = Topo::axis[j], i = (ax + 1) % 3, k = (ax + 2) % 3;
      S* w = pw[j];
      for (int r = 0; r < 6; ++r) w[r] = par < 0 ? (r % 4 == 0 ? S(1) : S(0)) : pw[par < 0 ? 0 : par][r];
      if constexpr (Topo::jtype[j] == REV) {
        for (int r = 0; r < 2; ++r) {
          const S a = w[3 * r + i], b = w[3 * r + k];
          w[3 * r + i] = a * d[n].c + b * d[n].s;
          w[3 * r + k] = b * d[n].c - a * d[n].s;
        }
      }
    });
  }
  // Two world rows, divided by the total mass, in the basis of the end that carries joint j's CoM column
  template <int e, class S>
  static __device__ __forceinline__ void com_basis(const SD<S>& sd, const S (*pw)[6], S iM, S* out) {
    constexpr int b = e / 2;
    if constexpr (is_pose(b)) {
      for (int r = 0; r < 6; ++r) out[r] = sd.PW[b][r] * iM;
    } else {
      constexpr int s = stop_link(b);
      for (int r = 0; r < 2; ++r)
        for (int m = 0; m < 3; ++m)
          out[3 * r + m] = iM * (pw[s][3 * r] * sd.Rb[b][m] + pw[s][3 * r + 1] * sd.Rb[b][3 + m] + pw[s][3 * r + 2] * sd.Rb[b][6 + m]);
    }
  }
  // pose of the end frame in its link's frame; the first end of a relative pose carries frame b
  template <int e, class S>
  static __device__ __forceinline__ void start_step(const Frames<S>& fr, const SD<S>& sd, Rig<S>& X) {
    if constexpr (is_rel(e / 2) && e % 2 == 0) {
      const S* R = sd.rel[e / 2];
      if constexpr (Topo::frame_rot) {
        matmul3(fr.R[e], R, X.R);
        S t[3];
        matvec3(fr.R[e], R + 9, t);
        for (int k = 0; k < 3; ++k) X.p[k] = fr.p[e][k] + t[k];
      } else {
        for (int k = 0; k < 9; ++k) X.R[k] = R[k];
        for (int k = 0; k < 3; ++k) X.p[k] = fr.p[e][k] + R[9 + k];
      }
    } else {
      start_end<e>(fr, X);
    }
  }
  static constexpr bool starts_identity(int e) {
    return !Topo::frame_rot && !(is_rel(e / 2) && e % 2 == 0);
  }
  // DIST: the block's direction in the frames of the joints on the chain of its end e, walked down from the
  // link where the chains meet
  static constexpr int chain_len(int e) {
    int n = 0;
    for (int j = 0; j < NJ; ++j) n += on(e, j) ? 1 : 0;
    return n;
  }
  template <int e>
  struct ChainList {  // the chain of end e, root first
    static constexpr int N = chain_len(e);
    static constexpr int at(int i) {
      for (int j = 0; j < NJ; ++j)
        if (on(e, j) && i-- == 0) return j;
      return -1;
    }
  };
  template <uint32_t RM, class S, class Q, class TR>
  static __device__ __forceinline__ void dist_dirs(const Q& q, const TR& tr, const SD<S>& sd, S (*u)[NJ][3]) {
    static_assert(!Topo::origin_rot || !has_dist(), "rods on topologies without rotated origins");
    sfor<0, NE>([&](auto E) {
      constexpr int e = decltype(E)::value;
      if constexpr (end_used(e)) {
        if constexpr (is_dist(e / 2) && has_chain(e) && sel(RM, e / 2)) {
          using List = ChainList<e>;
          constexpr int N = List::N;
          JD<S> d[N];
          load_list<S, List>(q, tr, d);
          S v[3] = {sd.u[e / 2][0], sd.u[e / 2][1], sd.u[e / 2][2]};
          sfor<0, N>([&](auto I) {
            constexpr int n = decltype(I)::value, j = List::at(n);
            constexpr int ax = Topo::axis[j], i = (ax + 1) % 3, k = (ax + 2) % 3;
            if constexpr (Topo::jtype[j] == REV) {
              const S a = v[i], b = v[k];
              v[i] = a * d[n].c + b * d[n].s;
              v[k] = b * d[n].c - a * d[n].s;
            }
            for (int r = 0; r < 3; ++r) u[e][j][r] = v[r];
          });
        }
      }
    });
  }
  static constexpr bool has_hull() {
    for (int b = 0; b < NB; ++b)
      if (Topo::btype[b] == B_HULL) return true;
    return false;
  }
  static constexpr bool has_dist() {
    for (int b = 0; b < NB; ++b)
      if (is_dist(b)) return true;
    return false;
  }
  // a joint on the first chain of a relative pose moves the pose the other way: the whole column is negated
  static constexpr bool negated(int j) {
    for (int b = 0; b < NB; ++b)
      if (is_rel(b) && on(2 * b, j)) return true;
    return false;
  }

  // no joint before j in the walk has both rows
  static constexpr bool first_touch(int r1, int r2, int j) {
    for (int l = 0; l < NJ; ++l)
      if (pos(l) < pos(j) && KI::rdep(r1, l) && KI::rdep(r2, l)) return false;
    return true;
  }
  // Gram pass: G = sum of J_j J_j^T over all columns (packed lower triangle), optionally v = J g.
  template <class S, uint32_t RM = ALL, class Q, class TR>
  static __device__ __forceinline__ void gram(const Q& q, const Consts& P, const SD<S>& sd, const TR& tr, S* G) {
    gram_pass<S, false, RM>(q, P, sd, tr, G, (const S*)nullptr, (S*)nullptr);
  }
  template <class S, class Q, class TR, class GV>
  static __device__ __forceinline__ void gram_jv(const Q& q, const Consts& P, const SD<S>& sd, const TR& tr, S* G, GV g, S* v) {
    gram_pass<S, true>(q, P, sd, tr, G, g, v);
  }
  template <class S, bool WITH_V, uint32_t RM = ALL, class Q, class TR, class GV>
  static __device__ __forceinline__ void gram_pass(const Q& q, const Consts& P, const SD<S>& sd, const TR& tr, S* G, GV g, S* v) {
    const TP<S>& T = tp<S>(P);
    sfor<0, M>([&](auto I) {  // entries that only fill in during the factorisation
      constexpr int i = decltype(I)::value;
      sfor<0, i + 1>([&](auto K) {
        constexpr int k = decltype(K)::value;
        if constexpr (KI::LP.nz[i][k] && !KI::gnz(i, k) && in_rows(RM, i) && in_rows(RM, k)) G[pidx(i, k)] = S(0);
      });
    });
    constexpr bool wc = com && com_rows(RM);
    S pw[NJ][6], cb[NE][6], iM = S(0);
    if constexpr (wc) {
      iM = T.inv_total_mass;
      world_rows<S>(q, tr, pw);
    }
    S du[NE][NJ][3];
    dist_dirs<RM>(q, tr, sd, du);
    Rig<S> X[NE];
    S hs[NJ + 1][3];
    walk<S, false>(q, T, tr, [&](auto J, const JD<S>& d, const Frames<S>& fr) {
      constexpr int j = decltype(J)::value;
      constexpr int ax = Topo::axis[j], i1 = (ax + 1) % 3, k1 = (ax + 2) % 3;
      constexpr bool rev = Topo::jtype[j] == REV;
      constexpr int ce = wc ? com_end(j) : -1;
      constexpr bool neg = negated(j);
      S col[M];
      sfor<0, NE>([&](auto E) {
        constexpr int e = decltype(E)::value;
        if constexpr (on(e, j)) {
          if constexpr (sel(RM, e / 2) || e == ce) {
            constexpr int b = e / 2, r0 = KI::brow0(b);
            if constexpr (end_link(e) == j) {
              start_step<e>(fr, sd, X[e]);
              if constexpr (wc && !is_dist(b)) com_basis<e>(sd, pw, iM, cb[e]);
            }
            if constexpr (sel(RM, b)) {
              const S* R = X[e].R;
              const S* p = X[e].p;
              if constexpr (is_dist(b)) {
                S val;
                if constexpr (rev) val = p[i1] * du[e][j][k1] - p[k1] * du[e][j][i1];
                else val = du[e][j][ax];
                col[r0] = (e % 2 == 0) ? -val : val;
              } else {
                constexpr bool id = starts_identity(e) && end_link(e) == j;
                if constexpr (rev) {
                  if constexpr (id) {
                    col[r0 + ax] = S(0);
                    col[r0 + i1] = -p[k1];
                    col[r0 + k1] = p[i1];
                  } else {
                    for (int m = 0; m < 3; ++m) col[r0 + m] = p[i1] * R[3 * k1 + m] - p[k1] * R[3 * i1 + m];
                  }
                  for (int m = 0; m < 3; ++m) col[r0 + 3 + m] = R[3 * ax + m];
                } else {
                  for (int m = 0; m < 3; ++m) col[r0 + m] = R[3 * ax + m];
                }
              }
            }
          }
        }
      });
      if constexpr (wc) {
        S h[3];
        subtree_h<j>(hs, d, h);
        S c0, c1;
        if constexpr (ce >= 0) {
          const S* R = X[ce].R;
          S t[3];
          if constexpr (rev) {
            for (int m = 0; m < 3; ++m) t[m] = h[i1] * R[3 * k1 + m] - h[k1] * R[3 * i1 + m];
          } else {
            for (int m = 0; m < 3; ++m) t[m] = d.m * R[3 * ax + m];
          }
          c0 = cb[ce][0] * t[0] + cb[ce][1] * t[1] + cb[ce][2] * t[2];
          c1 = cb[ce][3] * t[0] + cb[ce][4] * t[1] + cb[ce][5] * t[2];
        } else {
          if constexpr (rev) {
            c0 = iM * (h[i1] * pw[j][k1] - h[k1] * pw[j][i1]);
            c1 = iM * (h[i1] * pw[j][3 + k1] - h[k1] * pw[j][3 + i1]);
          } else {
            c0 = iM * d.m * pw[j][ax];
            c1 = iM * d.m * pw[j][3 + ax];
          }
        }
        if constexpr (neg) {
          c0 = -c0;
          c1 = -c1;
        }
        sfor<0, NB>([&](auto BI) {
          constexpr int b = decltype(BI)::value, r0 = KI::brow0(b);
          if constexpr (Topo::btype[b] == B_COM) {
            col[r0] = c0;
            col[r0 + 1] = c1;
          } else if constexpr (Topo::btype[b] == B_HULL) {
            col[r0] = sd.H[b][0] * c0 + sd.H[b][1] * c1;
            col[r0 + 1] = sd.H[b][2] * c1;
          }
        });
        push_h<j>(hs, d, h);
      }
      S gj = S(0);
      if constexpr (WITH_V) gj = neg ? -S(g[j]) : S(g[j]);
      sfor<0, M>([&](auto I) {
        constexpr int i = decltype(I)::value;
        if constexpr (KI::rdep(i, j) && in_rows(RM, i)) {
          sfor<0, i + 1>([&](auto K) {
            constexpr int k = decltype(K)::value;
            if constexpr (KI::rdep(k, j) && in_rows(RM, k)) {
              if constexpr (first_touch(i, k, j)) G[pidx(i, k)] = col[i] * col[k];
              else G[pidx(i, k)] += col[i] * col[k];
            }
          });
          if constexpr (WITH_V) {
            if constexpr (first_touch(i, i, j)) v[i] = col[i] * gj;
            else v[i] += col[i] * gj;
          }
        }
      });
      sfor<0, NE>([&](auto E) {
        constexpr int e = decltype(E)::value;
        if constexpr (on(e, j)) {
          if constexpr (sel(RM, e / 2) || e == ce) {
            up_point<j>(d, X[e].p);
            if constexpr (!is_dist(e / 2)) up_rot<j, starts_identity(e) && end_link(e) == j>(d, X[e].R);
          }
        }
      });
    }, [](auto) {});
  }

  // G += lambda T^-1 T^-T (see the header): J_r J_r^T = a I + (1 - a) / theta^2 w w^T with a = (2 sin(theta/2) / theta)^2.
  template <class S, uint32_t RM = ALL, class TR>
  static __device__ __forceinline__ void add_lambda(S* G, const S* F, S lambda, const TR& tr) {
    sfor<0, M>([&](auto I) {
      constexpr int i = decltype(I)::value;
      constexpr int b = KI::row_block(i);
      if constexpr (in_rows(RM, i)) {
        if constexpr ((is_pose(b) || is_rel(b)) && KI::row_comp(i) == 3) {
          const S t2 = F[i] * F[i] + F[i + 1] * F[i + 1] + F[i + 2] * F[i + 2];
          S a, c;
          if (t2 < S(1e-2)) {  // series of a and of (1 - a) / theta^2
            c = S(1.0 / 12) - t2 * (S(1.0 / 360) - t2 * (S(1.0 / 20160) - t2 * S(1.0 / 1814400)));
            a = S(1) - t2 * c;
          } else {
            double sn, cs;
            sincos_tab(0.5 * sqrt(double(t2)), tr.tab, sn, cs);
            const double aa = 4.0 * sn * sn / double(t2);
            a = S(aa);
            c = S((1.0 - aa) / double(t2));
          }
          for (int x = 0; x < 3; ++x)
            for (int y = 0; y <= x; ++y) G[pidx(i + x, i + y)] += lambda * ((x == y ? a : S(0)) + c * F[i + x] * F[i + y]);
        } else if constexpr (!((is_pose(b) || is_rel(b)) && KI::row_comp(i) > 3)) {
          G[pidx(i, i)] += lambda;
        }
      }
    });
  }

  // J^T y: out[j] assigned from the leaves to the root.
  template <class S, uint32_t RM = ALL, class Q, class TR, class OUT>
  static __device__ __forceinline__ void jty(const Q& q, const Consts& P, const SD<S>& sd, const TR& tr, const S* y, OUT&& out) {
    const TP<S>& T = tp<S>(P);
    constexpr bool wc = com && com_rows(RM);
    S pw[NJ][6], yc[2] = {S(0), S(0)};
    if constexpr (wc) {
      const S iM = T.inv_total_mass;
      sfor<0, NB>([&](auto BI) {
        constexpr int b = decltype(BI)::value, r0 = KI::brow0(b);
        if constexpr (Topo::btype[b] == B_COM) {
          yc[0] += iM * y[r0];
          yc[1] += iM * y[r0 + 1];
        } else if constexpr (Topo::btype[b] == B_HULL) {
          yc[0] += iM * sd.H[b][0] * y[r0];
          yc[1] += iM * (sd.H[b][1] * y[r0] + sd.H[b][2] * y[r0 + 1]);
        }
      });
      world_rows<S>(q, tr, pw);
    }
    S du[NE][NJ][3];
    dist_dirs<RM>(q, tr, sd, du);
    S f[NE][3], n[NE][3], cg[NE][3];  // force, moment, CoM row direction, per end
    S dp[NE][3];                      // DIST: the end's position
    S hs[NJ + 1][3];
    walk<S, false>(q, T, tr, [&](auto J, const JD<S>& d, const Frames<S>& fr) {
      constexpr int j = decltype(J)::value;
      constexpr int ax = Topo::axis[j], i1 = (ax + 1) % 3, k1 = (ax + 2) % 3;
      constexpr bool rev = Topo::jtype[j] == REV;
      constexpr int ce = wc ? com_end(j) : -1;
      S acc = S(0);
      sfor<0, NE>([&](auto E) {
        constexpr int e = decltype(E)::value;
        if constexpr (on(e, j)) {
          constexpr int b = e / 2, r0 = KI::brow0(b);
          if constexpr (is_dist(b)) {
            if constexpr (sel(RM, b)) {
              if constexpr (end_link(e) == j)
                for (int k = 0; k < 3; ++k) dp[e][k] = fr.p[e][k];
              S val;
              if constexpr (rev) val = dp[e][i1] * du[e][j][k1] - dp[e][k1] * du[e][j][i1];
              else val = du[e][j][ax];
              acc += (e % 2 == 0 ? -val : val) * y[r0];
              up_point<j>(d, dp[e]);
            }
          } else if constexpr (sel(RM, b) || e == ce) {
            constexpr int le = sel(RM, b) ? leader(RM, e, j) : e;
            if constexpr (end_link(e) == j) {
              Rig<S> X;
              start_step<e>(fr, sd, X);
              constexpr bool id = starts_identity(e);
              if constexpr (sel(RM, b)) {
                S yl[3], ya[3];
                for (int k = 0; k < 3; ++k) {
                  yl[k] = negated(j) ? -y[r0 + k] : y[r0 + k];
                  ya[k] = negated(j) ? -y[r0 + 3 + k] : y[r0 + 3 + k];
                }
                if constexpr (id) {
                  for (int k = 0; k < 3; ++k) {
                    f[e][k] = yl[k];
                    n[e][k] = ya[k];
                  }
                } else {
                  matvec3(X.R, yl, f[e]);
                  matvec3(X.R, ya, n[e]);
                }
                S t[3];
                cross3(X.p, f[e], t);
                for (int k = 0; k < 3; ++k) n[e][k] += t[k];
              }
              if constexpr (e == ce) {
                S gb[3];  // the rows' world direction in the end's basis
                if constexpr (is_pose(b)) {
                  for (int m = 0; m < 3; ++m) gb[m] = sd.PW[b][m] * yc[0] + sd.PW[b][3 + m] * yc[1];
                } else {
                  constexpr int s = stop_link(b);
                  S gs[3];
                  for (int m = 0; m < 3; ++m) gs[m] = pw[s][m] * yc[0] + pw[s][3 + m] * yc[1];
                  for (int m = 0; m < 3; ++m)
                    gb[m] = sd.Rb[b][m] * gs[0] + sd.Rb[b][3 + m] * gs[1] + sd.Rb[b][6 + m] * gs[2];
                }
                if constexpr (id) {
                  for (int m = 0; m < 3; ++m) cg[e][m] = gb[m];
                } else {
                  matvec3(X.R, gb, cg[e]);
                }
              }
            }
            if constexpr (sel(RM, b)) {
              if constexpr (le != e) {
                // where the chains of two ends meet, their wrenches continue as one
                constexpr int below = child_on(e, j);
                constexpr bool merged = below >= 0 && leader(RM, e, below < 0 ? j : below) != e;
                if constexpr (!merged) {
                  for (int k = 0; k < 3; ++k) {
                    f[le][k] += f[e][k];
                    n[le][k] += n[e][k];
                  }
                }
              }
            }
          }
        }
      });
      sfor<0, NE>([&](auto E) {
        constexpr int e = decltype(E)::value;
        if constexpr (on(e, j) && !is_dist(e / 2)) {
          if constexpr (sel(RM, e / 2) && leader(RM, e, j) == e) {
            if constexpr (rev) {
              acc += n[e][ax];
            } else {
              acc += f[e][ax];
              n[e][i1] -= d.q * f[e][k1];  // q e_ax x f
              n[e][k1] += d.q * f[e][i1];
            }
            up_vec<j>(d, f[e]);
            up_vec<j>(d, n[e]);
            S t[3];
            cross3(d.o, f[e], t);
            for (int k = 0; k < 3; ++k) n[e][k] += t[k];
          }
        }
      });
      if constexpr (wc) {
        S h[3];
        subtree_h<j>(hs, d, h);
        S g3[3];
        if constexpr (ce >= 0) {
          for (int m = 0; m < 3; ++m) g3[m] = cg[ce][m];
        } else {
          for (int m = 0; m < 3; ++m) g3[m] = pw[j][m] * yc[0] + pw[j][3 + m] * yc[1];
        }
        if constexpr (rev) acc += h[i1] * g3[k1] - h[k1] * g3[i1];
        else acc += d.m * g3[ax];
        if constexpr (ce >= 0) up_vec<j>(d, cg[ce]);
        push_h<j>(hs, d, h);
      }
      out[j] = acc;
    }, [](auto) {});
  }
};

// The topologies with a walk order take their step passes from it. (The other arms keep the direct
// passes: their rows are single components, bounded or masked, which the body basis mixes.)
template <> struct StepOf<Kin<TopoDual14Rel>> { using type = Leaf<TopoDual14Rel>; };
template <> struct StepOf<Kin<TopoHumanoid36>> { using type = Leaf<TopoHumanoid36>; };
template <> struct StepOf<Kin<TopoDigit36>> { using type = Leaf<TopoDigit36>; };

}  // namespace mc
