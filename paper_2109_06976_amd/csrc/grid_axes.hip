// Spatial algebra along common axes (gfx950), shared by the kernels with one lane per body
// (grid_team.hip) and one lane per problem (grid_serial.hip).
//
// Every quantity of a (knot, base branch) problem is expressed along one set of axes, those of the
// branch's first body, but about the origin of the body that it belongs to. Moving a spatial vector
// from a body to its parent is then one cross product with the offset r between the origins (6 FMA
// against 24 for a full transform), and the offsets stay as short as the links, which keeps
// float32 as accurate as it is in body axes. Gravity enters as the base acceleration turned
// into these axes.
//
// With z_i the joint axis, S_i = (z_i, 0) for a revolute joint or (0, z_i) for a prismatic one,
// v_l, a_l the velocity and acceleration of the parent taken at the origin of i, and
//   psd_i = v_l x S_i,   pdd_i = a_l x S_i + v_l x psd_i,
// the derivatives of inverse dynamics need only quantities of the subtree of j (superscript c):
// the inertia I^c_j, the force f^c_j and B^c_j with B v = v x* I v, and with
//   F1_j = I^c_j S_j,  b_j = B^c_j^T S_j,
//   u_j = 2 B^c_j psd_j + I^c_j pdd_j + S_j x* f^c_j,   w_j = 2 (B^c_j S_j + I^c_j psd_j)
// they are, for i = j or i an ancestor of j,
//   M_ij = S_i . F1_j,   dtau_i/dq_j = S_i . u_j,   dtau_i/dqd_j = S_i . w_j,
//   dtau_j/dq_i = 2 b_j . psd_i + F1_j . pdd_i,
//   dtau_j/dqd_i = 2 (b_j . S_i + F1_j . psd_i)         (i an ancestor of j),
// all other entries zero: one column of two six-vectors moved up the ancestor path replaces a
// sweep over the tree per column (Algorithm 1 evaluates the same derivatives column by column).
// For particles of mass m at p (from the origin) moving at u, B = [[sum m ((p . u) 1 - u p^T),
// 0], [-(sum m u) x, 0]], so B^c travels as K = sum m u p^T (9 floats) and the momentum
// l = sum m u, and the rotational inertia travels as P = sum m p p^T (J = tr(P) 1 - P):
//   about an origin moved by -r: P' = P + (h + m r) r^T + r h^T, h' = h + m r, K' = K + l r^T.

namespace gridv {

struct BatchArgs {
    int nknots;
    const float* q;
    const float* qd;      // unused by M^-1
    const float* u;       // tau (dFD, FD), qdd (ID, dID, VJP), unused (M^-1)
    const float* u2;      // g (VJP)
    float* o0;            // qdd (dFD, FD), tau (ID), M^-1 (M^-1), dtau/dq (dID), qbar (VJP)
    float* o1;            // M^-1 (dFD), dtau/dqd (dID), qdbar (VJP)
    float* o2;            // dqdd/dq (dFD), taubar (VJP)
    float* o3;            // dqdd/dqd (dFD)
};

// ..Q, ..V: half of dID (dtau/dq; dtau/dqd) and of dFD (qdd and dqdd/dq; M^-1 and dqdd/dqd)
enum Op : int {
    kFdGrad = 0, kFd = 1, kMinv = 2, kIdGrad = 3, kVjp = 4, kId = 5,
    kIdGradQ = 6, kIdGradV = 7, kFdGradQ = 8, kFdGradV = 9
};

// a workgroup's LDS, one array for all the calls of a kernel that want the same size
template <int FLOATS>
__device__ __forceinline__ float* lds()
{
    __shared__ __align__(16) float p[FLOATS];
    return p;
}

// 16 bytes at a 4-byte aligned address (global memory takes them at any dword)
struct __attribute__((packed, aligned(4))) F4 {
    float x, y, z, w;
};

struct __attribute__((packed, aligned(4))) F2 {
    float x, y;
};

// V (1, 2, 4) floats at a 4-byte aligned address
template <int V>
__device__ __forceinline__ void store(float* p, const float* x)
{
    if constexpr (V == 4)
        *reinterpret_cast<F4*>(p) = F4{x[0], x[1], x[2], x[3]};
    else if constexpr (V == 2)
        *reinterpret_cast<F2*>(p) = F2{x[0], x[1]};
    else
        p[0] = x[0];
}

struct V3 {
    float x, y, z;
};

__device__ __forceinline__ V3 operator+(V3 a, V3 b) { return {a.x + b.x, a.y + b.y, a.z + b.z}; }
__device__ __forceinline__ V3 operator-(V3 a, V3 b) { return {a.x - b.x, a.y - b.y, a.z - b.z}; }
__device__ __forceinline__ V3 operator*(V3 a, float s) { return {a.x * s, a.y * s, a.z * s}; }
__device__ __forceinline__ float dot(V3 a, V3 b) { return a.x * b.x + a.y * b.y + a.z * b.z; }
__device__ __forceinline__ V3 cross(V3 a, V3 b)
{
    return {a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x};
}
__device__ __forceinline__ V3 sel(bool c, V3 a, V3 b)
{
    return {c ? a.x : b.x, c ? a.y : b.y, c ? a.z : b.z};
}

struct Six {        // spatial vector [angular; linear]
    V3 a, l;
};

struct Sym {        // symmetric 3x3
    float xx, yy, zz, xy, xz, yz;
};

struct Mat {        // 3x3 by columns
    V3 c0, c1, c2;
};

__device__ __forceinline__ V3 mul(const Sym& s, V3 v)
{
    return {s.xx * v.x + s.xy * v.y + s.xz * v.z, s.xy * v.x + s.yy * v.y + s.yz * v.z,
            s.xz * v.x + s.yz * v.y + s.zz * v.z};
}
__device__ __forceinline__ V3 mul(const Mat& m, V3 v)
{
    return m.c0 * v.x + m.c1 * v.y + m.c2 * v.z;
}
__device__ __forceinline__ V3 tmul(const Mat& m, V3 v) { return {dot(m.c0, v), dot(m.c1, v), dot(m.c2, v)}; }

// rigid-body inertia: mass, first moment h, second moment P about the origin
// I x = [J w + h x v; m v + w x h], J = tr(P) 1 - P
__device__ __forceinline__ Six inertia(float m, V3 h, const Sym& J, Six x)
{
    return {mul(J, x.a) + cross(h, x.l), x.l * m + cross(x.a, h)};
}
__device__ __forceinline__ Sym second_to_inertia(const Sym& P)
{
    return {P.yy + P.zz, P.xx + P.zz, P.xx + P.yy, -P.xy, -P.xz, -P.yz};
}
// B x = [tr(K) w - K w; w x l] (only the angular part of x enters)
__device__ __forceinline__ Six bmul(const Mat& K, V3 l, V3 w)
{
    const float tr = K.c0.x + K.c1.y + K.c2.z;
    return {w * tr - mul(K, w), cross(w, l)};
}

// K = sum m u p^T = v h^T + w x P of a body moving at (w, v)
__device__ __forceinline__ Mat momentum_moment(Six v, V3 h, const Sym& P)
{
    return {v.l * h.x + cross(v.a, V3{P.xx, P.xy, P.xz}), v.l * h.y + cross(v.a, V3{P.xy, P.yy, P.yz}),
            v.l * h.z + cross(v.a, V3{P.xz, P.yz, P.zz})};
}

// second moment P of mass m and first moment h, about an origin moved by -r (h is moved too)
__device__ __forceinline__ void move_moments(Sym& P, V3& h, float m, V3 r)
{
    const V3 g = h + r * m;
    P = Sym{P.xx + g.x * r.x + r.x * h.x, P.yy + g.y * r.y + r.y * h.y,
            P.zz + g.z * r.z + r.z * h.z, P.xy + g.x * r.y + r.x * h.y,
            P.xz + g.x * r.z + r.x * h.z, P.yz + g.y * r.z + r.y * h.z};
    h = g;
}

// R P R^T
__device__ __forceinline__ Sym turn(const Mat& R, const Sym& P)
{
    const V3 c0 = mul(R, V3{P.xx, P.xy, P.xz}), c1 = mul(R, V3{P.xy, P.yy, P.yz}),
             c2 = mul(R, V3{P.xz, P.yz, P.zz});
    const V3 r0{R.c0.x, R.c1.x, R.c2.x}, r1{R.c0.y, R.c1.y, R.c2.y}, r2{R.c0.z, R.c1.z, R.c2.z};
    return {dot(r0, V3{c0.x, c1.x, c2.x}), dot(r1, V3{c0.y, c1.y, c2.y}),
            dot(r2, V3{c0.z, c1.z, c2.z}), dot(r1, V3{c0.x, c1.x, c2.x}),
            dot(r2, V3{c0.x, c1.x, c2.x}), dot(r2, V3{c0.y, c1.y, c2.y})};
}

}  // namespace gridv
