// Device pieces of the Gauss-Radau collocation step shared by the
// propagation and adjoint kernels: perturber chains into LDS, the force
// of Eqs. A.1 + A.3, its Jacobians, and the corrector sweep.
#pragma once

#include "kete_internal.hpp"

namespace kete {

constexpr int kNodes = 9;   // s_0 = 0, s_1..s_7, and s = 1 (step end)
constexpr double kInf = 1e300;

// Eq. A.4 (App. A.3) of J2 body q in vector form.  With d = x - x_m the
// object's offset from the body (Eq. A.4's r is -d, the sign of Eq. A.2's
// Newtonian term), z = d . p along the unit pole p and k = (3/2) J2 mu R^2,
// the componentwise expression in the body's equatorial frame reads
//   a = -k / |d|^5 [(1 - 5 z^2 / |d|^2) d + 2 z p].
// id = 1 / |d|.
__device__ __forceinline__ void j2_add(double k, const double* p, const double d[3], double id, double a[3]) {
    const double id2 = id * id;
    const double s = -k * (id2 * id2 * id);
    const double z = fma(d[0], p[0], fma(d[1], p[1], d[2] * p[2]));
    const double c = s * fma(-5.0 * z * id2, z, 1.0);
    const double e = 2.0 * s * z;
#pragma unroll
    for (int i = 0; i < 3; ++i) a[i] = fma(c, d[i], fma(e, p[i], a[i]));
}

// Its Jacobian da/dx, added to Jx (symmetric, the Hessian of the J2
// potential):
//   -k [A I + B d d^T + C (d p^T + p d^T) + E p p^T],
//   A = |d|^-5 - 5 z^2 |d|^-7, B = 35 z^2 |d|^-9 - 5 |d|^-7,
//   C = -10 z |d|^-7, E = 2 |d|^-5.
__device__ __forceinline__ void j2_jac_add(const EphemArgs& E, int q, const double d[3], double id, double Jx[9]) {
    const double* p = E.j2p[q];
    const double k = E.j2k[q];
    const double id2 = id * id, id5 = id2 * id2 * id, id7 = id5 * id2;
    const double z = fma(d[0], p[0], fma(d[1], p[1], d[2] * p[2]));
    const double A = -k * (id5 - 5.0 * z * z * id7);
    const double B = -k * (35.0 * z * z * id7 * id2 - 5.0 * id7);
    const double C = -k * (-10.0 * z * id7);
    const double Ee = -k * 2.0 * id5;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j)
            Jx[3 * i + j] += (i == j ? A : 0.0) + B * d[i] * d[j] + C * (d[i] * p[j] + p[i] * d[j]) + Ee * p[i] * p[j];
}

// Acceleration at one node from the LDS perturber table e[b][6]:
// Eq. A.1 with the attractive sign, plus Eq. A.3 (eps = 0) where kgr != 0
// and Eq. A.4 for the J2 bodies.
__device__ __forceinline__ void accel(const double* __restrict__ e, const EphemArgs& E,
                                      const double X[3], const double V[3], double F[3]) {
    double ax = 0.0, ay = 0.0, az = 0.0;
    for (int b = 0; b < E.n_body; ++b) {
        const double* pb = e + 6 * b;
        const double rx = X[0] - pb[0], ry = X[1] - pb[1], rz = X[2] - pb[2];
        const double r2 = fma(rx, rx, fma(ry, ry, rz * rz));
        const double ir = rsqrt(r2);
        const double ir3 = ir * ir * ir;
        const double gm = E.gm[b];
        double f = -gm * ir3;
        const double k = E.kgr[b];
        if (k != 0.0) {
            const double wx = V[0] - pb[3], wy = V[1] - pb[4], wz = V[2] - pb[5];
            const double w2 = fma(wx, wx, fma(wy, wy, wz * wz));
            const double rw = fma(rx, wx, fma(ry, wy, rz * wz));
            const double g = k * ir3;
            f = fma(g, 4.0 * gm * ir - w2, f);
            const double q = 4.0 * g * rw;
            ax = fma(q, wx, ax); ay = fma(q, wy, ay); az = fma(q, wz, az);
        }
        ax = fma(f, rx, ax); ay = fma(f, ry, ay); az = fma(f, rz, az);
    }
    F[0] = ax; F[1] = ay; F[2] = az;
    for (int q = 0; q < E.n_j2; ++q) {
        const double* pb = e + 6 * E.j2_body[q];
        const double d[3] = {X[0] - pb[0], X[1] - pb[1], X[2] - pb[2]};
        j2_add(E.j2k[q], E.j2p[q], d, rsqrt(fma(d[0], d[0], fma(d[1], d[1], d[2] * d[2]))), F);
    }
}

// Perturber positions and velocities at the 9 node times of a step
// (t + s_n h, and t_end for s = 1), one Clenshaw chain per lane, from the
// LDS window of segments [seg_lo, seg_hi]; results in ephW[n][b][6].
__device__ __forceinline__ void node_ephemeris(const double* __restrict__ coefL, int bstride, const EphemArgs& E,
                                               const RadauConst& rc, int seg_lo, int seg_hi, double t, double h,
                                               double t_end, int lane, double* __restrict__ ephW) {
    const int nb = E.n_body, deg1 = E.deg1, cps = 3 * deg1;
    const int nchain = kNodes * nb * 3;
    for (int c = lane; c < nchain; c += kWave) {
        const int n = c / (nb * 3);
        const int r = c - n * nb * 3;
        const int b = r / 3, i = r - 3 * b;
        const double tt = (n == kNodes - 1) ? t_end : t + rc.s[n] * h;
        const int k = seg_index(tt, E.t_start, E.inv_seg, seg_lo, seg_hi);
        const double tau = 2.0 * (tt - (E.t_start + (double)k * E.seg_days)) * E.inv_seg - 1.0;
        double pv, dv;
        clenshaw(coefL + b * bstride + (k - seg_lo) * cps + i * deg1, deg1, tau, pv, dv);
        ephW[(n * nb + b) * 6 + i] = pv;
        ephW[(n * nb + b) * 6 + 3 + i] = dv * 2.0 * E.inv_seg;
    }
    wave_lds_sync();
}

// Stage the Chebyshev segments [seg_lo, seg_hi] of every body into LDS
// (cooperatively by `nthreads` threads; the caller synchronizes).
__device__ __forceinline__ void stage_window(const EphemArgs& E, int seg_lo, int seg_hi, int bstride, int tid,
                                             int nthreads, double* __restrict__ coefL) {
    const int cps = 3 * E.deg1;
    const int per_body = (seg_hi - seg_lo + 1) * cps;
    const int total = E.n_body * per_body;
    for (int i = tid; i < total; i += nthreads) {
        const int b = i / per_body, r = i - b * per_body;
        coefL[b * bstride + r] = E.coef[((size_t)b * E.n_seg + seg_lo) * cps + r];
    }
}

// The collocation corrector: fixed-point sweeps over the 7 nodes
// (Gauss-Seidel: each node sees the increments already updated) until the
// change of b6 relative to |a| is below 1e-16, stops decreasing after the
// third sweep, or max_iter sweeps ran.  Returns the sweep count; b6 gets
// the final highest coefficient.
__device__ __forceinline__ int corrector(const RadauConst& rc, const EphemArgs& E, const double* __restrict__ ephW,
                                         const double x0[3], const double v0[3], const double F0[3], double h,
                                         bool active, int max_iter, double D[7][3], double b6[3],
                                         unsigned long long& lane_iters) {
    const double hh = h * h;
#pragma unroll
    for (int m = 0; m < 7; ++m) { D[m][0] = D[m][1] = D[m][2] = 0.0; }
    b6[0] = b6[1] = b6[2] = 0.0;
    double pc = 1e300, pcl;
    int it = 0;
    do {
        pcl = pc;
        ++it;
        // An opaque zero row offset keeps the collocation constants in the
        // kernel-argument segment (scalar loads per node) instead of being
        // hoisted into vector registers.
        int z;
        asm volatile("s_mov_b32 %0, 0" : "=s"(z));
#pragma unroll
        for (int n = 1; n <= 7; ++n) {
            const int nz = n + z;
            const double sh = rc.s[nz] * h;
            double X[3], V[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                double acc = rc.half_s2[nz] * F0[c];
#pragma unroll
                for (int m = 0; m < 7; ++m) acc = fma(rc.A[nz][m], D[m][c], acc);
                X[c] = fma(hh, acc, fma(sh, v0[c], x0[c]));
            }
            if (E.has_gr) {
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    double av = rc.s[nz] * F0[c];
#pragma unroll
                    for (int m = 0; m < 7; ++m) av = fma(rc.B[nz][m], D[m][c], av);
                    V[c] = fma(h, av, v0[c]);
                }
            } else {
                V[0] = v0[0]; V[1] = v0[1]; V[2] = v0[2];
            }
            double F[3];
            accel(ephW + n * E.n_body * 6, E, X, V, F);
#pragma unroll
            for (int c = 0; c < 3; ++c) D[n - 1][c] = F[c] - F0[c];
        }
        double db = 0.0, fm = 0.0;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            double b = 0.0;
#pragma unroll
            for (int m = 0; m < 7; ++m) b = fma(rc.E6[m + z], D[m][c], b);
            db = fmax(db, fabs(b - b6[c]));
            b6[c] = b;
            fm = fmax(fm, fabs(D[6][c] + F0[c]));
        }
        const double lpc = (active && fm > 0.0) ? db / fm : 0.0;
        pc = wave_max(lpc);
        lane_iters += __popcll(__ballot(active));
    } while (!(pc < 1e-16) && !(it > 2 && pcl <= pc) && it < max_iter);
    return it;
}

// ---------------------------------------------------------------- lane groups
// A body is spread over a lane group: the group's lanes own the collocation
// nodes 1..7 (one or more lanes per node), every lane keeps the body's state,
// and one corrector sweep updates all nodes at once from the previous
// sweep's increments (a Jacobi sweep of the same fixed-point map, converging
// to the same collocation solution).
constexpr int kGroup = 8;

// Lanes of a wavefront by body, G lanes per body.  G = 7: 9 bodies, lanes
// 7g..7g+6 for body g, and lane 63 joins body 8 as its eighth lane.  G = 8:
// 8 bodies, lanes 8g..8g+7.  G = 14, 56: 4 bodies or one with kLanes = 2 or
// 8 adjacent lanes per node, which share the node's force sum, and
// lanes 56..63 joining the last body.  gl is the lane's node less one; lanes
// with gl = 7 repeat node 7, so every node has exactly one owning set of
// lanes and the code below needs no other distinction.  sub numbers the
// lanes of a node.
template <int G>
struct GroupMap {
    static_assert(G == 7 || G == 8 || G == 14 || G == 56, "lanes per body");
    static constexpr int kLanes = G == 8 ? 1 : G / 7;
    static constexpr int kBodies = G == 8 ? 8 : 64 / G;      // bodies per wavefront
    int grp, gl, sub;
    __device__ __forceinline__ explicit GroupMap(int lane) {
        sub = 0;
        if constexpr (G == 8) {
            grp = lane >> 3;
            gl = lane & 7;
        } else {
            const bool in = lane < kBodies * G;
            grp = in ? lane / G : kBodies - 1;
            gl = in ? (lane - grp * G) / kLanes : 7;
            if constexpr (kLanes > 1) sub = lane & (kLanes - 1);
        }
    }
};

// Constants of one node.
struct NodeRow {
    double s, hs2, A[7], B[7];
    double pad_[2];       // 144-byte rows: the 8 rows start in distinct LDS banks
};

// Constants of the grouped kernels, copied to LDS from the device table that
// fill_group_const describes (GroupConst's doubles in order).
struct GroupConst {
    double Ap[7][8], Bp[7][8];      // dense output
    NodeRow row[kGroup];            // by gl
    double s[7];                    // nodes 1..7
    double Lden[7], L1[7];          // extrapolated corrector start
    double A8[8], B8[7];            // step end: weights of D_1..D_7 (A8[7]: of F_0)
};
static_assert(sizeof(GroupConst) == kGroupConstDoubles * sizeof(double), "the device table is one GroupConst");

__device__ __forceinline__ void load_group_const(const double* __restrict__ src, GroupConst* dst, int tid,
                                                 int nthreads) {
    double* d = &dst->Ap[0][0];
    for (int i = tid; i < kGroupConstDoubles; i += nthreads) d[i] = src[i];
}

// Wave-wide reductions of values that are equal within each group, as a
// butterfly of lane permutations that stay in the vector unit: DPP quad
// permutes (lanes xor 1, xor 2), the half-row and row mirrors (lane i with
// 7 - i, with 15 - i) and the row-pair and half-wave swaps (xor 16, xor
// 32).  Aligned 8-lane groups need only the last three steps.
struct PermDouble {
    unsigned lo, hi;
};
__device__ __forceinline__ PermDouble split_double(double x) {
    const unsigned long long u = __double_as_longlong(x);
    return PermDouble{(unsigned)u, (unsigned)(u >> 32)};
}
__device__ __forceinline__ double join_double(unsigned lo, unsigned hi) {
    return __longlong_as_double(((long long)hi << 32) | lo);
}
template <int CTRL>
__device__ __forceinline__ double dpp_double(double x) {
    const PermDouble d = split_double(x);
    return join_double((unsigned)__builtin_amdgcn_update_dpp(0, (int)d.lo, CTRL, 0xF, 0xF, false),
                       (unsigned)__builtin_amdgcn_update_dpp(0, (int)d.hi, CTRL, 0xF, 0xF, false));
}
// the other operand of a max/min step across rows (xor 16) and halves (xor 32)
__device__ __forceinline__ double swap16_double(double x) {
    const PermDouble d = split_double(x);
    const auto lo = __builtin_amdgcn_permlane16_swap(d.lo, d.lo, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(d.hi, d.hi, false, false);
    // both results hold each lane's own value in one and its xor-16 partner in the other
    const double a = join_double(lo[0], hi[0]), b = join_double(lo[1], hi[1]);
    return ((threadIdx.x >> 4) & 1) ? a : b;
}
__device__ __forceinline__ double swap32_double(double x) {
    const PermDouble d = split_double(x);
    const auto lo = __builtin_amdgcn_permlane32_swap(d.lo, d.lo, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap(d.hi, d.hi, false, false);
    const double a = join_double(lo[0], hi[0]), b = join_double(lo[1], hi[1]);
    return ((threadIdx.x >> 5) & 1) ? a : b;
}
template <int G = kGroup, bool MAX = true>
__device__ __forceinline__ double groups_reduce(double x) {
    auto op = [](double a, double b) { return MAX ? fmax(a, b) : fmin(a, b); };
    if constexpr (G != 8) {
        x = op(x, dpp_double<0xB1>(x));      // lane xor 1
        x = op(x, dpp_double<0x4E>(x));      // lane xor 2
        x = op(x, dpp_double<0x141>(x));     // 7 - lane within 8
    }
    x = op(x, dpp_double<0x140>(x));         // 15 - lane within 16
    x = op(x, swap16_double(x));
    x = op(x, swap32_double(x));
    return uniform(x);
}
template <int G = kGroup>
__device__ __forceinline__ double groups_max(double x) { return groups_reduce<G, true>(x); }
template <int G = kGroup>
__device__ __forceinline__ double groups_min(double x) { return groups_reduce<G, false>(x); }

// Sum over the L adjacent lanes of a node (every lane gets the same bits:
// each step adds the same two values on both sides).
template <int L>
__device__ __forceinline__ void node_sum(double a[3]) {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        if constexpr (L > 1) a[c] += dpp_double<0xB1>(a[c]);
        if constexpr (L > 2) a[c] += dpp_double<0x4E>(a[c]);
        if constexpr (L > 4) a[c] += dpp_double<0x141>(a[c]);
    }
}

// Perturber table of the grouped integrators: per node and slot 8 doubles
// (x, y, z, GM, vx, vy, vz, GM/c^2).  GM values are written once per
// launch (g8_table_init); node_ephemeris8 fills positions, and velocities
// only for the slots that carry the Eq. A.3 term (zero for the others).
// Slots past the last body stand for massless ones far away, which add
// exactly nothing: with one lane per node the bodies without the term are
// padded to whole fours, else the slots to whole rounds of the lanes.
constexpr int kSlot = 8;
__host__ __device__ inline int g8_slots(int n_body, int n_gr, int lanes) {
    return lanes == 1 ? n_gr + ((n_body - n_gr + 3) & ~3) : (n_body + lanes - 1) / lanes * lanes;
}
// Doubles per node row: 4 (4 slots + 1) dwords, so the 8 rows read together
// by an 8-lane group fall in distinct LDS banks.
__host__ __device__ inline int g8_row(int slots) { return slots * kSlot + 2; }

// Exchange rows of the grouped corrector, after the wave's node table:
// per group three rows (x, y, z) of 8 doubles, lane gl writing column gl,
// padded to 26 doubles so that the 16-byte reads of the groups of a
// wavefront fall in distinct LDS banks.
constexpr int kXchGroup = 26;
// Constants {k, pole} of the bodies with the Eq. A.4 term, after the
// exchange rows: 8 entries by slot for those that carry the Eq. A.3 term too
// (they have the first slots; zero for the others), then KETE_MAX_J2 by
// index for the rest.
constexpr int kJ2Doubles = 4 * (8 + KETE_MAX_J2);
// Doubles of LDS per wavefront: node table, exchange rows of its bodies, J2
// constants.
__host__ __device__ inline int g8_wave_doubles(int slots, int bodies) {
    return kNodes * g8_row(slots) + bodies * kXchGroup + kJ2Doubles;
}
template <int G>
inline int g8_wave_doubles(const EphemArgs& E) {
    return g8_wave_doubles(g8_slots(E.n_body, E.n_gr, GroupMap<G>::kLanes), GroupMap<G>::kBodies);
}

// One wavefront's LDS areas, and the shape of its table.
struct G8Lds {
    double* e8;             // node table
    double* xg;             // this group's exchange rows
    const double* j2;       // J2 constants
    int row;                // doubles per node row
};
template <int G>
__device__ __forceinline__ G8Lds g8_lds(const EphemArgs& E, double* base, int grp) {
    const int slots = g8_slots(E.n_body, E.n_gr, GroupMap<G>::kLanes);
    G8Lds s;
    s.e8 = base;
    s.row = g8_row(slots);
    s.xg = base + kNodes * s.row + grp * kXchGroup;
    s.j2 = base + kNodes * s.row + GroupMap<G>::kBodies * kXchGroup;
    return s;
}

// The entries of the table and of the J2 constants that hold for the whole
// launch; one wavefront.
template <int G>
__device__ __forceinline__ void g8_table_init(const EphemArgs& E, int lane, double* __restrict__ base) {
    const int slots = g8_slots(E.n_body, E.n_gr, GroupMap<G>::kLanes);
    const int row = g8_row(slots);
    const int n = lane < kNodes ? lane : 0;      // lanes past the nodes repeat node 0
    double* r = base + n * row;
#pragma unroll
    for (int b = 0; b < KETE_MAX_BODIES; ++b) {
        if (b >= E.n_body) break;
        double* q = r + body_slot(E, b) * kSlot;
        q[3] = E.gm[b];
        q[4] = q[5] = q[6] = 0.0;
        q[7] = E.kgr[b];
    }
    for (int sl = E.n_body; sl < slots; ++sl) {
        double* q = r + sl * kSlot;
        q[0] = 1e6;
        for (int k = 1; k < kSlot; ++k) q[k] = 0.0;
    }
    double* j2 = base + kNodes * row + GroupMap<G>::kBodies * kXchGroup;
    if (lane < kJ2Doubles) j2[lane] = 0.0;
    wave_lds_sync();
#pragma unroll
    for (int q = 0; q < KETE_MAX_J2; ++q) {
        if (q >= E.n_j2) break;
        double* d = j2 + 4 * (q < E.n_j2g ? q : 8 + q);
        d[0] = E.j2k[q];
        d[1] = E.j2p[q][0]; d[2] = E.j2p[q][1]; d[3] = E.j2p[q][2];
    }
    wave_lds_sync();
}

// Publish this lane's increment dn (node gl + 1) and read the increments
// D[m] of nodes m + 1 = 1..7 of the group.  Every lane of the wavefront
// takes part (the lanes of a node write the same values).
__device__ __forceinline__ void g8_exchange(double* __restrict__ xg, int gl, const double dn[3], double D[7][3]) {
    wave_lds_sync();                        // earlier reads of the rows are done
    xg[gl] = dn[0];
    xg[8 + gl] = dn[1];
    xg[16 + gl] = dn[2];
    wave_lds_sync();
#pragma unroll
    for (int c = 0; c < 3; ++c) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const double2 v = *reinterpret_cast<const double2*>(xg + 8 * c + 2 * k);
            D[2 * k][c] = v.x;
            if (2 * k + 1 < 7) D[2 * k + 1][c] = v.y;
        }
    }
}

// Coefficients of one coordinate's segment, read together.  DEG1 = 0 takes
// the count at run time and pads with zeros to the largest, which leaves the
// Clenshaw recurrences' values as they are.
template <int DEG1>
struct ChainCoef {
    static constexpr int kN = DEG1 > 0 ? DEG1 : KETE_MAX_DEGREE + 1;
    double c[kN];
    __device__ __forceinline__ void load(const double* __restrict__ p, int deg1) {
#pragma unroll
        for (int k = 0; k < kN; ++k) c[k] = (DEG1 > 0 || k < deg1) ? p[k] : 0.0;
    }
    __device__ __forceinline__ double value(double tau) const {
        const double t2 = tau + tau;
        double b2 = c[kN - 1], b1 = fma(t2, b2, c[kN - 2]);
#pragma unroll
        for (int k = kN - 3; k >= 1; --k) {
            const double b0 = fma(t2, b1, c[k] - b2);
            b2 = b1; b1 = b0;
        }
        return fma(tau, b1, c[0] - b2);
    }
    __device__ __forceinline__ void value_slope(double tau, double& p, double& dp) const {
        const double t2 = tau + tau;
        double b2 = c[kN - 1], b1 = fma(t2, b2, c[kN - 2]);
        double d2 = 0.0, d1 = 2.0 * b2;
#pragma unroll
        for (int k = kN - 3; k >= 1; --k) {
            const double b0 = fma(t2, b1, c[k] - b2);
            const double d0 = fma(t2, d1, 2.0 * b1 - d2);
            b2 = b1; b1 = b0; d2 = d1; d1 = d0;
        }
        p = fma(tau, b1, c[0] - b2);
        dp = fma(tau, d1, b1 - d2);
    }
};

// Perturber states at the node times of a step.  Lane k of each 8 takes
// node (k & 7) + 1 (node 8 is the step end) and finds that node's segment
// and tau once; the 3 n_body coordinates are spread over the 8 eights (eight
// g takes coordinates g, g + 8, ...), two of a lane's chains in flight.
// Coordinates of the slots with the Eq. A.3 term come first and also get the
// velocity (derivative chain); a pair of passes holding any of them
// evaluates derivatives in every lane so the wavefront does not diverge.
// Node 0 (the step start, needed before the first step or when the caller
// asks) takes one more pass with coordinate = lane.  The node of a lane here
// follows lane & 7 whatever the lane's body group.
//
// The coefficients come straight from the table (156 KB for ten bodies and a
// year: it stays in each XCD's L2), a step's chains reading two or three
// segments of it.  Staged in LDS instead they tied the wavefronts of a block
// to one window of a few segments: barriers at its ends, where every step
// also had to land (750,000 bodies for a year: 28.3 ms a launch, 20.9 so).
template <int NB, int NGR, int DEG1>
__device__ __forceinline__ void node_ephemeris8(const EphemArgs& E, const GroupConst& K, const G8Lds& T, double t,
                                                double h, double t_end, bool node0, int lane) {
    const int nb = NB > 0 ? NB : E.n_body;
    const int ngr = NB > 0 ? NGR : E.n_gr;
    const int deg1 = DEG1 > 0 ? DEG1 : E.deg1;
    const int cps = 3 * deg1, nc = 3 * nb, ngc = 3 * ngr;
    // A body's segments begin at a 64-bit offset (a table may pass 2^31 values),
    // one multiply-add where a body has fewer than 2^32 (group_shape).
    const size_t bstride = (size_t)E.n_seg * cps;
    auto body_offset = [&](int b) {
        return DEG1 > 0 ? (size_t)(unsigned)b * (unsigned)bstride : (size_t)b * bstride;
    };
    const double sc = 2.0 * E.inv_seg;
    auto chains = [&](int n, double tt, int c0, int cstep, int npass) {
        const int k = seg_index(tt, E.t_start, E.inv_seg, 0, E.n_seg - 1);
        const double tau = 2.0 * (tt - (E.t_start + (double)k * E.seg_days)) * E.inv_seg - 1.0;
        const double* cb = E.coef + (size_t)k * cps;
        double* row = T.e8 + n * T.row;
        auto at = [&](int c) {                     // coefficients of coordinate c
            const int qc = c < nc ? c : nc - 1, sl = qc / 3;
            return cb + body_offset(slot_body(E, sl)) + (unsigned)((qc - 3 * sl) * deg1);
        };
#pragma unroll 1
        for (int j = 0; j < npass; j += 2) {
            const int ca = c0 + cstep * j, cc = ca + cstep;
            const int sa = ca / 3, ia = ca - 3 * sa, sb = cc / 3, ib = cc - 3 * sb;
            ChainCoef<DEG1> A, B;
            A.load(at(ca), deg1);
            B.load(at(cc), deg1);
            if (cstep * j < ngc) {                 // wave-uniform: the pair holds derivative chains
                double pa, da, pb, db;
                A.value_slope(tau, pa, da);
                B.value_slope(tau, pb, db);
                if (ca < nc) row[sa * kSlot + ia] = pa;
                if (ca < ngc) row[sa * kSlot + 4 + ia] = da * sc;
                if (cc < nc) row[sb * kSlot + ib] = pb;
                if (cc < ngc) row[sb * kSlot + 4 + ib] = db * sc;
            } else {
                const double pa = A.value(tau), pb = B.value(tau);
                if (ca < nc) row[sa * kSlot + ia] = pa;
                if (cc < nc) row[sb * kSlot + ib] = pb;
            }
        }
    };
    const int nl = lane & (kGroup - 1);
    chains(nl + 1, nl == kGroup - 1 ? t_end : fma(K.row[nl].s, h, t), lane / kGroup, kGroup,
           (nc + kGroup - 1) / kGroup);
    if (node0) chains(0, t, lane, kWave, 1);
    wave_lds_sync();
}

// Adds to a[] the terms of M slots, pb + m step: Eq. A.1, with GR Eq. A.3
// (nothing for slots whose GM/c^2 is zero), and for the first MJ of them
// Eq. A.4 with the constants jc + 4 m jstep (see j2_add; its part along r
// joins the coefficient of r).  The M slots advance side by side: a slot's
// chain (offset, inverse distance, coefficient) is some 20 dependent
// operations, and one after another they left a lone wavefront waiting.
template <int M, bool GR, int MJ = 0>
__device__ __forceinline__ void force_terms(const double* __restrict__ pb, int step, const double* __restrict__ jc,
                                            int jstep, const double X[3], const double V[3], double a[3]) {
    static_assert(MJ <= M, "J2 slots are among the slots");
    double r[M][3], gm[M], ir[M], ir3[M], f[M], w[M][3], kg[M];
#pragma unroll
    for (int m = 0; m < M; ++m) {
        const double2 xy = *reinterpret_cast<const double2*>(pb + m * step);
        const double2 zg = *reinterpret_cast<const double2*>(pb + m * step + 2);
        r[m][0] = X[0] - xy.x; r[m][1] = X[1] - xy.y; r[m][2] = X[2] - zg.x;
        gm[m] = zg.y;
        if constexpr (GR) {
            const double2 vxy = *reinterpret_cast<const double2*>(pb + m * step + 4);
            const double2 vzk = *reinterpret_cast<const double2*>(pb + m * step + 6);
            w[m][0] = V[0] - vxy.x; w[m][1] = V[1] - vxy.y; w[m][2] = V[2] - vzk.x;
            kg[m] = vzk.y;
        }
    }
#pragma unroll
    for (int m = 0; m < M; ++m) ir[m] = rsqrt_pos(fma(r[m][0], r[m][0], fma(r[m][1], r[m][1], r[m][2] * r[m][2])));
#pragma unroll
    for (int m = 0; m < M; ++m) {
        ir3[m] = ir[m] * ir[m] * ir[m];
        f[m] = -gm[m] * ir3[m];
    }
    if constexpr (GR) {
#pragma unroll
        for (int m = 0; m < M; ++m) {
            const double w2 = fma(w[m][0], w[m][0], fma(w[m][1], w[m][1], w[m][2] * w[m][2]));
            const double rw = fma(r[m][0], w[m][0], fma(r[m][1], w[m][1], r[m][2] * w[m][2]));
            const double g = kg[m] * ir3[m];
            f[m] = fma(g, 4.0 * gm[m] * ir[m] - w2, f[m]);
            const double q = 4.0 * g * rw;
#pragma unroll
            for (int c = 0; c < 3; ++c) a[c] = fma(q, w[m][c], a[c]);
        }
    }
#pragma unroll
    for (int m = 0; m < MJ; ++m) {
        const double2 kp = *reinterpret_cast<const double2*>(jc + 4 * m * jstep);
        const double2 pq = *reinterpret_cast<const double2*>(jc + 4 * m * jstep + 2);
        const double p[3] = {kp.y, pq.x, pq.y};
        const double ir2 = ir[m] * ir[m];
        const double s = -kp.x * (ir3[m] * ir2);
        const double z = fma(r[m][0], p[0], fma(r[m][1], p[1], r[m][2] * p[2]));
        f[m] = fma(s, fma(-5.0 * z * ir2, z, 1.0), f[m]);
        const double e = 2.0 * s * z;
#pragma unroll
        for (int c = 0; c < 3; ++c) a[c] = fma(e, p[c], a[c]);
    }
#pragma unroll
    for (int m = 0; m < M; ++m)
#pragma unroll
        for (int c = 0; c < 3; ++c) a[c] = fma(f[m], r[m][c], a[c]);
}

// Eq. A.4 of the J2 bodies outside the first slots (none in the default
// model), from the table row.
__device__ __forceinline__ void j2_extra(const EphemArgs& E, const double* __restrict__ row, int q, const double X[3],
                                         double a[3]) {
    const double* pb = row + kSlot * E.j2_slot[q];
    const double d[3] = {X[0] - pb[0], X[1] - pb[1], X[2] - pb[2]};
    j2_add(E.j2k[q], E.j2p[q], d, rsqrt_pos(fma(d[0], d[0], fma(d[1], d[1], d[2] * d[2]))), a);
}

// Force of Eqs. A.1 + A.3 + A.4 at one node from its table row: with L = 1
// lane per node every slot; else lane sub takes slots sub, sub + L, ... (the
// same kind of round in every lane: slots with the Eq. A.3 term come first,
// those with the Eq. A.4 term first among them) and the lanes' sums are
// added.  NB = 0 takes the counts at run time.
template <int NB, int NGR, int NJ2, int L>
__device__ __forceinline__ void accel8(const double* __restrict__ row, const G8Lds& T, const EphemArgs& E, int sub,
                                       const double X[3], const double V[3], double F[3]) {
    F[0] = F[1] = F[2] = 0.0;
    const double* pb = row + kSlot * sub;
    const double* jc = T.j2 + 4 * sub;
    if constexpr (NB > 0) {
        constexpr int kRounds = (NB + L - 1) / L, kGr = (NGR + L - 1) / L, kJ = (NJ2 + L - 1) / L;
        constexpr int kPlain = kRounds - kGr;
        // at most two slots with the Eq. A.3 term side by side, and four without
        constexpr int kGrA = kGr > 2 ? 2 : kGr, kJa = kJ > kGrA ? kGrA : kJ;
        if constexpr (kGrA > 0) force_terms<kGrA, true, kJa>(pb, kSlot * L, jc, L, X, V, F);
        if constexpr (kGr > kGrA)
            force_terms<kGr - kGrA, true, kJ - kJa>(pb + kSlot * L * kGrA, kSlot * L, jc + 4 * L * kGrA, L, X, V, F);
        constexpr int kHalf = kPlain > 4 ? (kPlain + 1) / 2 : kPlain;
        if constexpr (kHalf > 0) force_terms<kHalf, false>(pb + kSlot * L * kGr, kSlot * L, jc, 0, X, V, F);
        if constexpr (kPlain > kHalf)
            force_terms<kPlain - kHalf, false>(pb + kSlot * L * (kGr + kHalf), kSlot * L, jc, 0, X, V, F);
    } else {
        const int rounds = g8_slots(E.n_body, E.n_gr, L) / L, gr = (E.n_gr + L - 1) / L, nj = (E.n_j2g + L - 1) / L;
        int k = 0;
        for (; k < nj; ++k) force_terms<1, true, 1>(pb + kSlot * L * k, 0, jc + 4 * L * k, 0, X, V, F);
        for (; k + 1 < gr; k += 2) force_terms<2, true>(pb + kSlot * L * k, kSlot * L, jc, 0, X, V, F);
        for (; k < gr; ++k) force_terms<1, true>(pb + kSlot * L * k, 0, jc, 0, X, V, F);
        for (; k + 3 < rounds; k += 4) force_terms<4, false>(pb + kSlot * L * k, kSlot * L, jc, 0, X, V, F);
        for (; k < rounds; ++k) force_terms<1, false>(pb + kSlot * L * k, 0, jc, 0, X, V, F);
        if (sub == 0)
            for (int q = E.n_j2g; q < E.n_j2; ++q) j2_extra(E, row, q, X, F);
    }
    node_sum<L>(F);
}

// The same force computed by a group together: its lanes take slots gl L +
// sub, ... (lanes with gl = 7 none); the partial sums meet in the group's
// exchange rows and every lane adds them in the same order, so all lanes of
// the group return the same total.  The whole wavefront takes part.
template <int L>
__device__ __forceinline__ void accel8_group(const double* __restrict__ row, const G8Lds& T, const EphemArgs& E,
                                             const double X[3], const double V[3], int gl, int sub, double F[3]) {
    double part[3] = {0.0, 0.0, 0.0};
    const int lane_slot = gl * L + sub;
    for (int s0 = 0; s0 < E.n_body; s0 += 7 * L) {
        const int sl = s0 + lane_slot;
        if (gl < 7 && sl < E.n_body) {
            if (s0 < E.n_gr) force_terms<1, true>(row + kSlot * sl, 0, T.j2, 0, X, V, part);
            else force_terms<1, false>(row + kSlot * sl, 0, T.j2, 0, X, V, part);
        }
    }
    if (lane_slot < E.n_j2 && gl < 7) {        // J2 body q by lane q of the group
        const bool first = lane_slot < E.n_j2g;
        const double* pb = row + kSlot * (first ? lane_slot : (int)((E.j2_slots >> (4 * lane_slot)) & 15u));
        const double* jc = T.j2 + 4 * (first ? lane_slot : 8 + lane_slot);
        const double d[3] = {X[0] - pb[0], X[1] - pb[1], X[2] - pb[2]};
        const double id = rsqrt_pos(fma(d[0], d[0], fma(d[1], d[1], d[2] * d[2])));
        j2_add(jc[0], jc + 1, d, id, part);
    }
    node_sum<L>(part);
    double D[7][3];
    g8_exchange(T.xg, gl, part, D);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        double f = D[0][c];
#pragma unroll
        for (int m = 1; m < 7; ++m) f += D[m][c];
        F[c] = f;
    }
}

// Jacobians Jx = da/dx, Jv = da/dv (row-major 3x3) from the grouped
// table e8 (one node) of the force of accel8, Eq. A.4 included.  The Newtonian part is
// symmetric and accumulated once per pair (i <= j); the Eq. A.3 part,
// with P = s1 r + 4 (r.w) w and s1 = 4 mu / r - w^2, is
//   Jx += k [(-3 P / r^5 - 4 mu r / r^6) r^T + 4 w w^T / r^3 + s1 I / r^3]
//   Jv += k / r^3 [-2 r w^T + 4 w r^T + 4 (r.w) I].
// NB = 0 takes the counts at run time.
template <int NB, int NGR>
__device__ __forceinline__ void accel_jac8(const double* __restrict__ e8, const EphemArgs& E, const double X[3],
                                           const double V[3], double Jx[9], double Jv[9]) {
    const int nb = NB > 0 ? NB : E.n_body;
    const int ngr = NB > 0 ? NGR : E.n_gr;
    double S[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};   // xx xy xz yy yz zz
    double dg = 0.0;
#pragma unroll
    for (int i = 0; i < 9; ++i) { Jx[i] = 0.0; Jv[i] = 0.0; }
#pragma unroll
    for (int sl = 0; sl < (NB > 0 ? NB : KETE_MAX_BODIES); ++sl) {
        if (NB == 0 && sl >= nb) break;
        const double* pb = e8 + kSlot * sl;
        const double2 pxy = *reinterpret_cast<const double2*>(pb);
        const double2 pzg = *reinterpret_cast<const double2*>(pb + 2);
        const double r[3] = {X[0] - pxy.x, X[1] - pxy.y, X[2] - pzg.x};
        const double r2 = fma(r[0], r[0], fma(r[1], r[1], r[2] * r[2]));
        const double ir = rsqrt_pos(r2);
        const double ir2 = ir * ir, ir3 = ir2 * ir, ir5 = ir3 * ir2;
        const double gm = pzg.y;
        const double sN = 3.0 * gm * ir5;
        const double a[3] = {sN * r[0], sN * r[1], sN * r[2]};
        S[0] = fma(a[0], r[0], S[0]); S[1] = fma(a[0], r[1], S[1]); S[2] = fma(a[0], r[2], S[2]);
        S[3] = fma(a[1], r[1], S[3]); S[4] = fma(a[1], r[2], S[4]); S[5] = fma(a[2], r[2], S[5]);
        dg = fma(-gm, ir3, dg);
        if (sl < ngr) {
            const double2 vxy = *reinterpret_cast<const double2*>(pb + 4);
            const double2 vzk = *reinterpret_cast<const double2*>(pb + 6);
            const double k = vzk.y;
            const double w[3] = {V[0] - vxy.x, V[1] - vxy.y, V[2] - vzk.x};
            const double w2 = fma(w[0], w[0], fma(w[1], w[1], w[2] * w[2]));
            const double rw = fma(r[0], w[0], fma(r[1], w[1], r[2] * w[2]));
            const double s1 = 4.0 * gm * ir - w2;
            const double kr3 = k * ir3;
            const double c1 = -3.0 * k * ir5, c2 = -4.0 * k * gm * ir3 * ir3, c4 = 4.0 * kr3;
            double u[3], v[3], pr[3], qw[3];
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                const double P = fma(s1, r[i], 4.0 * rw * w[i]);
                u[i] = fma(c1, P, c2 * r[i]);
                v[i] = c4 * w[i];
                pr[i] = -2.0 * kr3 * r[i];
                qw[i] = c4 * w[i];
            }
#pragma unroll
            for (int i = 0; i < 3; ++i)
#pragma unroll
                for (int j = 0; j < 3; ++j) {
                    Jx[3 * i + j] = fma(u[i], r[j], fma(v[i], w[j], Jx[3 * i + j]));
                    Jv[3 * i + j] = fma(pr[i], w[j], fma(qw[i], r[j], Jv[3 * i + j]));
                }
            const double dx = kr3 * s1, dv = c4 * rw;
            Jx[0] += dx; Jx[4] += dx; Jx[8] += dx;
            Jv[0] += dv; Jv[4] += dv; Jv[8] += dv;
        }
    }
    Jx[0] += S[0] + dg; Jx[1] += S[1]; Jx[2] += S[2];
    Jx[3] += S[1]; Jx[4] += S[3] + dg; Jx[5] += S[4];
    Jx[6] += S[2]; Jx[7] += S[4]; Jx[8] += S[5] + dg;
    for (int q = 0; q < E.n_j2; ++q) {
        const double* pb = e8 + kSlot * E.j2_slot[q];
        const double d[3] = {X[0] - pb[0], X[1] - pb[1], X[2] - pb[2]};
        j2_jac_add(E, q, d, rsqrt_pos(fma(d[0], d[0], fma(d[1], d[1], d[2] * d[2]))), Jx);
    }
}

// Step-size factor (eps / e)^(1/7) of the IAS15 control, in single
// precision: the factor only sets the next trial step.
__device__ __forceinline__ double step_factor(double q) {
    const float qf = (float)fmin(fmax(q, 1e-35), 1e35);
    return (double)exp2f(log2f(qf) * (1.0f / 7.0f));
}

// Starting increment of this lane's node for a step q times the previous
// accepted one: that step's collocation polynomial of the force
// increments (values Dp at its nodes, 0 at its start) evaluated at the new
// node's time sig = 1 + q s_n of the old step, less its value at sig = 1.
// The Lagrange basis of the 8 nodes is formed from prefix and suffix
// products of (sig - s_k).
__device__ __forceinline__ void extrapolate_increment(const GroupConst& K, double* __restrict__ xg, int gl,
                                                      const double Dp[3], double q, double dn[3]) {
    double D[7][3];
    g8_exchange(xg, gl, Dp, D);
    const double sig = fma(q, K.row[gl].s, 1.0);
    double dk[8], pre[8];
    dk[0] = sig;
#pragma unroll
    for (int k = 1; k < 8; ++k) dk[k] = sig - K.s[k - 1];
    pre[0] = 1.0;
#pragma unroll
    for (int k = 1; k < 8; ++k) pre[k] = pre[k - 1] * dk[k - 1];
    double suf = 1.0;
    dn[0] = dn[1] = dn[2] = 0.0;
#pragma unroll
    for (int m = 7; m >= 1; --m) {
        const double w = fma(pre[m] * suf, K.Lden[m - 1], -K.L1[m - 1]);
#pragma unroll
        for (int c = 0; c < 3; ++c) dn[c] = fma(w, D[m - 1][c], dn[c]);
        suf *= dk[m];
    }
}

// Corrector of the lane groups (see above).  Each lane keeps only its own
// node's increment dn; the other nodes' increments are read from the group's
// lanes when the predictor sums and b6 are formed.  With q > 0 the iteration
// starts from the previous step's increments Dp extrapolated
// (extrapolate_increment), otherwise from zero.  A body is done when the
// change of its b6 relative to |a| is below 1e-16, or has stopped decreasing
// after the third sweep (corrector()'s rule, body by body); the wavefront
// sweeps until all of its bodies are, which a vote tells without a reduction
// over the lanes.  On return dn holds the converged increment of this lane's
// node, b6 the highest coefficient and d6 the increment of node 7 (all
// lanes).
template <int NB, int NGR, int NJ2, int L>
__device__ __forceinline__ int corrector_g8(const RadauConst& rc, const GroupConst& K, const EphemArgs& E,
                                            const G8Lds& T, int gl, int sub, const double x0[3], const double v0[3],
                                            const double F0[3], double h, bool active, int max_iter, double dn[3],
                                            double b6[3], double d6[3], const double Dp[3], double q) {
    const NodeRow& R = K.row[gl];
    const double hh = h * h, sh = R.s * h;
    const double* en = T.e8 + (gl < 7 ? gl + 1 : 7) * T.row;
    const bool started = q > 0.0;           // wave-uniform
    if (started) extrapolate_increment(K, T.xg, gl, Dp, q, dn);
    else dn[0] = dn[1] = dn[2] = 0.0;
    b6[0] = b6[1] = b6[2] = 0.0;
    double last = 1e300;
    bool done = !active;
    int it = 0;
    for (;;) {
        double ax[3], av[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) { ax[c] = R.hs2 * F0[c]; av[c] = R.s * F0[c]; }
        if (it > 0 || started) {
            double D[7][3], bb[3] = {0.0, 0.0, 0.0};
            g8_exchange(T.xg, gl, dn, D);
#pragma unroll
            for (int m = 0; m < 7; ++m) {
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    const double d = D[m][c];
                    ax[c] = fma(R.A[m], d, ax[c]);
                    av[c] = fma(R.B[m], d, av[c]);
                    bb[c] = fma(rc.E6[m], d, bb[c]);
                }
            }
            double db = 0.0, fm = 0.0;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                db = fmax(db, fabs(bb[c] - b6[c]));
                b6[c] = bb[c];
                fm = fmax(fm, fabs(D[6][c] + F0[c]));
            }
            // the ratio only steers the stopping rule: the reciprocal estimate
            // suffices (a body whose ratio is not a number holds no one up)
            const double pc = fm > 0.0 ? db * __builtin_amdgcn_rcp(fm) : 0.0;
            if (it > 0) {
                done = done || !(pc >= 1e-16) || (it > 2 && last <= pc);
                if (__ballot(!done) == 0ull || it >= max_iter) break;
            }
            last = pc;
        }
        ++it;
        double X[3], V[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) X[c] = fma(hh, ax[c], fma(sh, v0[c], x0[c]));
        if (NB > 0 ? NGR > 0 : E.has_gr) {
#pragma unroll
            for (int c = 0; c < 3; ++c) V[c] = fma(h, av[c], v0[c]);
        } else {
            V[0] = v0[0]; V[1] = v0[1]; V[2] = v0[2];
        }
        double F[3];
        accel8<NB, NGR, NJ2, L>(en, T, E, sub, X, V, F);
#pragma unroll
        for (int c = 0; c < 3; ++c) dn[c] = F[c] - F0[c];
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) d6[c] = T.xg[8 * c + 6];       // as published last
    return it;
}

// Step end of a group-integrated body from the converged increments.
__device__ __forceinline__ void step_end_g8(const GroupConst& K, double* __restrict__ xg, int gl, const double dn[3],
                                            double h, double x0[3], double v0[3], const double F0[3]) {
    double ax[3], av[3];
    double D[7][3];
    g8_exchange(xg, gl, dn, D);
#pragma unroll
    for (int c = 0; c < 3; ++c) { ax[c] = K.A8[7] * F0[c]; av[c] = F0[c]; }
#pragma unroll
    for (int m = 0; m < 7; ++m) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const double d = D[m][c];
            ax[c] = fma(K.A8[m], d, ax[c]);
            av[c] = fma(K.B8[m], d, av[c]);
        }
    }
    const double hh = h * h;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        x0[c] = fma(hh, ax[c], fma(h, v0[c], x0[c]));
        v0[c] = fma(h, av[c], v0[c]);
    }
}

// Stepping state of a group-integrated body (replicated in its lanes).
struct G8State {
    double x0[3], v0[3], F0[3];
    double Dp[3] = {0.0, 0.0, 0.0};   // this lane's increment in the last accepted step
    double hprev = 0.0;               // that step (0: none yet)
    double t, hw, hp_new;
    bool active, haveF0;
    int status;
};
struct G8Count {
    unsigned long long steps = 0, iter = 0, rej = 0, lsteps = 0, liter = 0, chain = 0, vchain = 0, lpred = 0;
};

// Largest ratio of a step to the previous accepted one for which the
// corrector starts from the extrapolated increments.
constexpr double kPredMaxRatio = 3.0;

struct G8NoVisit {
    template <class... A>
    __device__ __forceinline__ void operator()(A&&...) const {}
};

// Integrate [S.t, tb] with wave-shared adaptive steps (the bodies of the
// wavefront take the smallest step any of them asks for).  Correctors start
// from the previous step extrapolated unless p.zero_start.
// visit(ts, te, h, dn, S) is called by every lane after each accepted step,
// before S moves to the step end te (dn: this lane's converged increment).
template <int NB, int NGR, int NJ2, int DEG1, int G, class Params, class Visit = G8NoVisit>
__device__ __forceinline__ void g8_integrate(const Params& p, const GroupConst& K, const G8Lds& T,
                                             const GroupMap<G>& M, int lane, double tb, G8State& S, G8Count& C,
                                             Visit&& visit = Visit(), double t_stop = kInf) {
    constexpr int L = GroupMap<G>::kLanes;
    const EphemArgs& E = p.eph;
    const RadauConst& rc = p.rc;
    const int nb = E.n_body, gl = M.gl, sub = M.sub;
    if (__ballot(S.active) == 0ull) { S.t = tb; return; }
    while (S.t != tb) {
        if (S.t >= t_stop) return;          // a recompute ends where the recorded run took its checkpoint
        const double dir = tb > S.t ? 1.0 : -1.0;
        double hmag = S.hw;
        if (p.h_max > 0.0 && hmag > p.h_max) hmag = p.h_max;
        double h = dir * hmag;
        bool landed = false;
        if (fabs(h) >= fabs(tb - S.t)) { h = tb - S.t; landed = true; }
        // (times and steps are the same in every lane: kept in scalar registers)
        h = uniform(h);
        if ((long)C.steps >= p.max_steps) {
            if (S.active) { S.status = KETE_ST_MAX_STEPS; S.active = false; }
            S.t = tb;
            return;
        }
        const double t_end = uniform(landed ? tb : S.t + h);
        // (node 0, for the force there, before the first step only)
        const int n0 = S.haveF0 ? 1 : 0;
        node_ephemeris8<NB, NGR, DEG1>(E, K, T, S.t, h, t_end, n0 == 0, lane);
        C.chain += (kNodes - n0) * E.n_gr * 3;
        C.vchain += (kNodes - n0) * (nb - E.n_gr) * 3;
        if (!S.haveF0) { accel8_group<L>(T.e8, T, E, S.x0, S.v0, gl, sub, S.F0); S.haveF0 = true; }

        double q = 0.0;                       // wave-uniform, like h and S.hprev
        if (!p.zero_start && S.hprev != 0.0) q = h / S.hprev;
        if (!(q <= kPredMaxRatio)) q = 0.0;
        q = uniform(q);
        double dn[3], b6p[3], d6[3];
        const int it = corrector_g8<NB, NGR, NJ2, L>(rc, K, E, T, gl, sub, S.x0, S.v0, S.F0, h, S.active, p.max_iter,
                                                     dn, b6p, d6, S.Dp, q);
        C.iter += it;
        const unsigned long long n_act = __popcll(__ballot(S.active && gl == 0 && sub == 0));
        C.liter += (unsigned long long)it * n_act;
        if (q > 0.0) C.lpred += n_act;

        double fm = 0.0, bm = 0.0;
#pragma unroll
        for (int c = 0; c < 3; ++c) { fm = fmax(fm, fabs(d6[c] + S.F0[c])); bm = fmax(bm, fabs(b6p[c])); }
        // (the reciprocal estimate suffices: the factor only sets the next step)
        double hl = (bm > 0.0 && fm > 0.0 && bm < kInf && fm < kInf)
                        ? fabs(h) * step_factor(p.eps * fm * __builtin_amdgcn_rcp(bm))
                        : fabs(h) / p.safety;
        if (!S.active) hl = kInf;
        if (S.active && hl < p.h_min) { S.status = KETE_ST_STEP_UNDERFLOW; S.active = false; hl = kInf; }
        const double hn = groups_min<G>(hl);
        if (!(hn < kInf)) { S.t = tb; return; }
        if (hn < p.safety * fabs(h)) {       // reject and retry from the same state
            S.hw = hn;
            ++C.rej;
            continue;
        }
        visit(S.t, t_end, h, dn, S);
#pragma unroll
        for (int c = 0; c < 3; ++c) S.Dp[c] = dn[c];
        S.hprev = h;
        step_end_g8(K, T.xg, gl, dn, h, S.x0, S.v0, S.F0);
        S.t = t_end;
        ++C.steps;
        C.lsteps += n_act;
        if (S.active && !(isfinite(S.x0[0]) && isfinite(S.x0[1]) && isfinite(S.x0[2]) && isfinite(S.v0[0]) &&
                          isfinite(S.v0[1]) && isfinite(S.v0[2]))) {
            S.status = KETE_ST_NONFINITE; S.active = false;
        }
        accel8_group<L>(T.e8 + 8 * T.row, T, E, S.x0, S.v0, gl, sub, S.F0);
        if (landed) {
            S.hw = uniform(fmin(S.hw, hn));
        } else {
            S.hw = uniform(fmin(hn, fabs(h) / p.safety));
            S.hp_new = fmin(S.hp_new, fmin(hl, fabs(h) / p.safety));
        }
    }
}

// Component c (0..2) of a vector and gl (0..5) of a state.  The components
// are made opaque first: selects between plain array elements are merged
// into one load at a selected address, which keeps the whole array in
// scratch memory, read again by every sweep (a third of the integrator's
// time).
__device__ __forceinline__ double vector_component(const double x[3], int c) {
    double a = x[0], b = x[1], d = x[2];
    asm("" : "+v"(a));
    asm("" : "+v"(b));
    asm("" : "+v"(d));
    return c == 0 ? a : c == 1 ? b : d;
}
__device__ __forceinline__ double state_component(const double x0[3], const double v0[3], int gl) {
    const double a = vector_component(x0, gl), b = vector_component(v0, gl - 3);
    return gl < 3 ? a : b;
}

// The node increments of component c of a step, and F_0's, as the dense
// output reads them: from the group's exchange rows, where each lane
// publishes its node's increment dn first.  The whole wavefront calls it.
__device__ __forceinline__ void dense_increments(double* __restrict__ xg, int gl, int c, const double dn[3],
                                                 const double F0[3], double D[8]) {
    wave_lds_sync();                        // earlier reads of the exchange rows are done
    xg[gl] = dn[0];
    xg[8 + gl] = dn[1];
    xg[16 + gl] = dn[2];
    wave_lds_sync();
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const double2 d = *reinterpret_cast<const double2*>(xg + 8 * c + 2 * k);
        D[2 * k] = d.x;
        D[2 * k + 1] = d.y;
    }
    D[7] = vector_component(F0, c);
}

// sum_m w[m] D[m] + w[7] F_0 from eight weights in LDS.
__device__ __forceinline__ double dense_sum(const double* __restrict__ w, const double D[8]) {
    const double2* q = reinterpret_cast<const double2*>(w);
    const double2 q0 = q[0], q1 = q[1], q2 = q[2], q3 = q[3];
    double a = q3.y * D[7];
    a = fma(q0.x, D[0], a);
    a = fma(q0.y, D[1], a);
    a = fma(q1.x, D[2], a);
    a = fma(q1.y, D[3], a);
    a = fma(q2.x, D[4], a);
    a = fma(q2.y, D[5], a);
    return fma(q3.x, D[6], a);
}

// This lane's component of the collocation polynomial at fraction sig of the
// step, which differs between the 8-lane groups: lane gl of a group evaluates
// the weights alpha and beta of node gl + 1 (lane 7 those of F_0) into the
// group's 16 slots wt, and each lane forms the component it stands for
// (velocity if vel) from them and D (dense_increments).  The whole wavefront
// calls it.
__device__ __forceinline__ double dense_component8(const GroupConst& K, double* __restrict__ wt, int gl, bool vel,
                                                   double sig, double h, double xc, double vc, const double D[8]) {
    const double* am = K.Ap[gl < 7 ? gl : 6];
    const double* bm = K.Bp[gl < 7 ? gl : 6];
    double a = am[7], b = bm[7];
#pragma unroll
    for (int k = 6; k >= 0; --k) { a = fma(a, sig, am[k]); b = fma(b, sig, bm[k]); }
    a *= sig * sig;
    b *= sig;
    wave_lds_sync();                        // earlier reads of wt are done
    wt[gl] = gl < 7 ? a : 0.5 * sig * sig;
    wt[8 + gl] = gl < 7 ? b : sig;
    wave_lds_sync();
    const double s = dense_sum(wt + (vel ? 8 : 0), D);
    return vel ? fma(h, s, vc) : fma(h * h, s, fma(sig * h, vc, xc));
}

// Dense output of a step for a wavefront's objects: the cursor's epochs that
// lie inside the step [ts, te] are read off its collocation polynomial
// (te, not ts + h, which rounds below a landing time)
// and put(e, value) gets component gl (0..5) of each object's state; the
// cursor moves past them.  The step is the same for every
// object, so its weights are too: the 16 lanes of a quarter of the wavefront
// evaluate one epoch's (slots 0..6 alpha_m(sig) = sum_k Ap[m][k] sig^(k+2)
// and 7 sig^2 / 2 of the force at the step start; 8..14 beta_m(sig) = sum_k
// Bp[m][k] sig^(k+1) and 15 sig), four epochs at a time, into the
// wavefront's slots wt[64]; then each lane forms the one component it
// writes, eight multiply-adds an epoch, from the weights and the node
// increments of its group in the exchange rows xg.  (Every lane forming
// all six components, one epoch's 14 weights at a time, took 250 vector
// instructions an epoch, a fifth of the integrator's with epochs 3 days apart.)
constexpr int kDenseRound = 4;              // epochs per round
constexpr int kDenseWeights = 16 * kDenseRound;
// The cursor keeps 64 epochs' times in the lanes, so that a step seldom
// loads: a load waits for the states stored before it.
struct EpochCursor {
    const double* t_out;
    int next, end;          // wave-uniform
    int base = 0;           // lane l holds t_out[base + l] (the last epoch past the end)
    double buf = 0.0;
    __device__ __forceinline__ EpochCursor(const double* t, int first, int last, int lane)
        : t_out(t), next(first), end(last) { load(lane); }
    __device__ __forceinline__ void load(int lane) {
        base = next;
        const int e = next + lane;
        if (next < end) buf = t_out[e < end ? e : end - 1];
    }
    __device__ __forceinline__ double time() const {           // of epoch `next`
        return lane_value(buf, __builtin_amdgcn_readfirstlane(next - base));
    }
    __device__ __forceinline__ double time_ahead(int k) const { return __shfl(buf, next - base + k, kWave); }
    __device__ __forceinline__ void advance(int n, int lane) {
        next += n;
        if (next - base > kWave - 4) load(lane);
    }
};
template <class Put>
__device__ __forceinline__ void dense_epochs(const GroupConst& K, double* __restrict__ wt, double* __restrict__ xg,
                                             int gl, int lane, double ts, double te, double h, const double dn[3],
                                             const double x0[3], const double v0[3], const double F0[3],
                                             EpochCursor& ec, Put&& put) {
    if (ec.next >= ec.end) return;
    const double t_first = ec.time();
    if (!(h > 0.0 ? t_first <= te : t_first >= te)) return;
    // this lane's component: coordinate c of the position or velocity
    const bool vel = gl >= 3;
    const int c = vel ? (gl < 6 ? gl - 3 : 2) : gl;
    double D[8];
    dense_increments(xg, gl, c, dn, F0, D);
    const double xc = vector_component(x0, c);
    const double vc = vector_component(v0, c);
    const double hc = vel ? h : h * h;
    const int m = lane & 15;
    const double* pm = &K.Ap[0][0] + 8 * (m < 7 ? m : m < 15 ? m - 1 : 13);
    for (;;) {
        const int el = ec.next + (lane >> 4), e0 = ec.next;
        const double tk = ec.time_ahead(lane >> 4);
        const int n = __popcll(__ballot(el < ec.end && (h > 0.0 ? tk <= te : tk >= te))) >> 4;
        const double sig = (tk - ts) / h;
        ec.advance(n, lane);
        double w = pm[7];
#pragma unroll
        for (int k = 6; k >= 0; --k) w = fma(w, sig, pm[k]);
        w *= m < 8 ? sig * sig : sig;
        if (m == 7) w = 0.5 * sig * sig;
        if (m == 15) w = sig;
        wave_lds_sync();                    // earlier reads of wt are done
        wt[lane] = w;
        wave_lds_sync();
#pragma unroll
        for (int k = 0; k < kDenseRound; ++k) {
            if (k >= n) break;
            const double a = dense_sum(wt + 16 * k + (vel ? 8 : 0), D);
            const double sg = wt[16 * k + 15];
            put(e0 + k, vel ? fma(hc, a, vc) : fma(hc, a, fma(sg * h, vc, xc)));
        }
        if (n < kDenseRound || ec.next >= ec.end) break;
    }
}

}  // namespace kete
