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
// they are, for i = j or i an ancestor of j (the analytical derivatives by spatial vector algebra of
// Singh, Russell and Wensing, RA-L 2022; the particle form of B below is this library's),
//   M_ij = S_i . F1_j,   dtau_i/dq_j = S_i . u_j,   dtau_i/dqd_j = S_i . w_j,
//   dtau_j/dq_i = 2 b_j . psd_i + F1_j . pdd_i,
//   dtau_j/dqd_i = 2 (b_j . S_i + F1_j . psd_i)         (i an ancestor of j),
// all other entries zero: one column of two six-vectors moved up the ancestor path replaces a
// sweep over the tree per column (Algorithm 1 evaluates the same derivatives column by column).
// For particles of mass m at p (from the origin) moving at u, B = [[sum m ((p . u) 1 - u p^T),
// 0], [-(sum m u) x, 0]], so B^c travels as K = sum m u p^T (9 floats) and the momentum
// l = sum m u. With D = (h + m r) r^T + r h^T, about an origin moved by -r:
//   J' = J + tr(D) 1 - D, h' = h + m r, K' = K + l r^T.
//
// Rounding. In body axes a row of M begins with constants of the model and small inertias keep
// their relative accuracy; along common axes every quantity is a turned one. So that nothing is
// lost by it: the inertia J is stored and summed as the model gives it (not as the second moment,
// which would have to be rounded and turned back); sine and cosine are brought to unit length and
// the rotations kept orthonormal (in double, or by one orthonormalisation), since errors of scale
// would add up along the chain; the rows of M are formed in double, whose FMA issues at the rate of
// float's, beginning with the body's own part as a constant (M_ii) or a turned constant; short
// branches turn in double; M = L^T D L without square roots. 2-norm errors against 64 bits, in 1e-7, in body axes (the quad layout)
// and here: M^-1 of quad12 0.80 and 0.78, chain7 7.8 and 5.9, humanoid30 6.1 and 4.9; qdd 0.98 and
// 0.90, 9.4 and 7.2, 7.7 and 6.3; dqdd/dq 3.1 and 2.95, 26 and 19.5, 21 and 17.7 (without these: M^-1
// 2.25, 8.2 and 7.8). It costs 3 to 5% of a launch: humanoid30 at 4096 knots 23.5 and 24.2 us, chain7 at
// 65536 20.2 and 21.0. Short branches turned in float: quad12 dqdd/dq 3.16, a launch 2 to 4% shorter.

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

// vectors and matrices of float (V3, Mat) and of double (V3D, MatD)
template <class T>
struct Vec {
    T x, y, z;
};
using V3 = Vec<float>;
using V3D = Vec<double>;

template <class T>
__device__ __forceinline__ Vec<T> operator+(Vec<T> a, Vec<T> b) { return {a.x + b.x, a.y + b.y, a.z + b.z}; }
template <class T>
__device__ __forceinline__ Vec<T> operator-(Vec<T> a, Vec<T> b) { return {a.x - b.x, a.y - b.y, a.z - b.z}; }
__device__ __forceinline__ V3 operator*(V3 a, float s) { return {a.x * s, a.y * s, a.z * s}; }
__device__ __forceinline__ V3D operator*(V3D a, double s) { return {a.x * s, a.y * s, a.z * s}; }
template <class T>
__device__ __forceinline__ T dot(Vec<T> a, Vec<T> b) { return a.x * b.x + a.y * b.y + a.z * b.z; }
template <class T>
__device__ __forceinline__ Vec<T> cross(Vec<T> a, Vec<T> b)
{
    return {a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x};
}
__device__ __forceinline__ V3D wide(V3 a) { return {a.x, a.y, a.z}; }
__device__ __forceinline__ V3 narrow(V3D a) { return {(float)a.x, (float)a.y, (float)a.z}; }

struct Six {        // spatial vector [angular; linear]
    V3 a, l;
};

struct Sym {        // symmetric 3x3
    float xx, yy, zz, xy, xz, yz;
};

__device__ __forceinline__ Sym operator+(const Sym& a, const Sym& b)
{
    return {a.xx + b.xx, a.yy + b.yy, a.zz + b.zz, a.xy + b.xy, a.xz + b.xz, a.yz + b.yz};
}
__device__ __forceinline__ Sym operator-(const Sym& a, const Sym& b)
{
    return {a.xx - b.xx, a.yy - b.yy, a.zz - b.zz, a.xy - b.xy, a.xz - b.xz, a.yz - b.yz};
}

template <class T>
struct Matrix {     // 3x3 by columns
    Vec<T> c0, c1, c2;
};
using Mat = Matrix<float>;
using MatD = Matrix<double>;

// Branches of few bodies, whose own rounding is what is left of the error and which have registers
// to spare, turn each body's quantities in double; others in float (a chain of 7 and a branch of 18
// lose nothing by it)
template <int B>
constexpr bool kFineBranch = B <= 5;
template <bool kFine>
struct AxesOf {
    using T = float;
    static __device__ __forceinline__ Mat of(const MatD& m)
    {
        return {narrow(m.c0), narrow(m.c1), narrow(m.c2)};
    }
};
template <>
struct AxesOf<true> {
    using T = double;
    static __device__ __forceinline__ MatD of(const MatD& m) { return m; }
};

template <class T>
__device__ __forceinline__ Vec<T> mul(const Sym& s, Vec<T> v)
{
    return {s.xx * v.x + s.xy * v.y + s.xz * v.z, s.xy * v.x + s.yy * v.y + s.yz * v.z,
            s.xz * v.x + s.yz * v.y + s.zz * v.z};
}
template <class T>
__device__ __forceinline__ Vec<T> mul(const Matrix<T>& m, Vec<T> v)
{
    return m.c0 * v.x + m.c1 * v.y + m.c2 * v.z;
}
template <class T>
__device__ __forceinline__ Vec<T> tmul(const Matrix<T>& m, Vec<T> v) { return {dot(m.c0, v), dot(m.c1, v), dot(m.c2, v)}; }

// rigid-body inertia: mass, first moment h, rotational inertia J about the origin
// I x = [J w + h x v; m v + w x h]
__device__ __forceinline__ Six inertia(float m, V3 h, const Sym& J, Six x)
{
    return {mul(J, x.a) + cross(h, x.l), x.l * m + cross(x.a, h)};
}
// the second moment sum m p p^T of a body with half = tr(J) / 2
__device__ __forceinline__ Sym second_moment(const Sym& J, float half)
{
    return {half - J.xx, half - J.yy, half - J.zz, -J.xy, -J.xz, -J.yz};
}
// B x = [tr(K) w - K w; w x l] (only the angular part of x enters)
__device__ __forceinline__ Six bmul(const Mat& K, V3 l, V3 w)
{
    const float tr = K.c0.x + K.c1.y + K.c2.z;
    return {w * tr - mul(K, w), cross(w, l)};
}

// K = sum m u p^T = v h^T + w x P of a body moving at (w, v), P its second moment
__device__ __forceinline__ Mat momentum_moment(Six v, V3 h, const Sym& P)
{
    return {v.l * h.x + cross(v.a, V3{P.xx, P.xy, P.xz}), v.l * h.y + cross(v.a, V3{P.xy, P.yy, P.yz}),
            v.l * h.z + cross(v.a, V3{P.xz, P.yz, P.zz})};
}

// inertia J of mass m and first moment h, about an origin moved by -r (h is moved too)
__device__ __forceinline__ void move_inertia(Sym& J, V3& h, float m, V3 r)
{
    const V3 g = h + r * m;
    const float dx = g.x * r.x + r.x * h.x, dy = g.y * r.y + r.y * h.y, dz = g.z * r.z + r.z * h.z;
    J = Sym{J.xx + (dy + dz), J.yy + (dx + dz), J.zz + (dx + dy), J.xy - (g.x * r.y + r.x * h.y),
            J.xz - (g.x * r.z + r.x * h.z), J.yz - (g.y * r.z + r.y * h.z)};
    h = g;
}

// body axes along the parent's: the columns of E^T for E = E_z(q) E_T with rows e0, e1, e2 of E_T,
// from the hardware sine and cosine (argument in revolutions reduced to [0, 1)) brought to unit
// length by one Newton step; E_T alone for a prismatic joint
template <class T>
__device__ __forceinline__ Matrix<T> joint_axes(bool prismatic, float q, Vec<T> e0, Vec<T> e1, Vec<T> e2)
{
    if (prismatic)
        return {e0, e1, e2};
    const float rev = __builtin_amdgcn_fractf(q * 0.159154943091895336f);
    const float s = __builtin_amdgcn_sinf(rev), c = __builtin_amdgcn_cosf(rev);
    const float d = -0.5f * __builtin_fmaf(s, s, __builtin_fmaf(c, c, -1.0f));
    const T sn = s + (T)s * d, co = c + (T)c * d;
    return {e0 * co + e1 * sn, e1 * co - e0 * sn, e2};
}

__device__ __forceinline__ MatD wide(const Mat& m) { return {wide(m.c0), wide(m.c1), wide(m.c2)}; }
__device__ __forceinline__ MatD wide(const MatD& m) { return m; }
__device__ __forceinline__ V3 narrow(V3 a) { return a; }

// R J R^T
template <class T>
__device__ __forceinline__ Sym turn(const Matrix<T>& R, const Sym& J)
{
    using V = Vec<T>;
    const V c0 = mul(R, V{J.xx, J.xy, J.xz}), c1 = mul(R, V{J.xy, J.yy, J.yz}),
            c2 = mul(R, V{J.xz, J.yz, J.zz});
    const V r0{R.c0.x, R.c1.x, R.c2.x}, r1{R.c0.y, R.c1.y, R.c2.y}, r2{R.c0.z, R.c1.z, R.c2.z};
    return {(float)dot(r0, V{c0.x, c1.x, c2.x}), (float)dot(r1, V{c0.y, c1.y, c2.y}),
            (float)dot(r2, V{c0.z, c1.z, c2.z}), (float)dot(r1, V{c0.x, c1.x, c2.x}),
            (float)dot(r2, V{c0.x, c1.x, c2.x}), (float)dot(r2, V{c0.y, c1.y, c2.y})};
}
// M = L^T D L along ancestor paths, L with a unit diagonal, in place: L below the diagonal, dinv = 1 / D
// (one rounding where the square root of D takes three)
template <class S>
__device__ __forceinline__ void ltdl_factor(float (&L)[S::B][S::B], float (&dinv)[S::B])
{
    constexpr int B = S::B;
#pragma unroll
    for (int k = B - 1; k >= 0; --k) {
        float d = __builtin_amdgcn_rcpf(L[k][k]);
        d += d * __builtin_fmaf(-L[k][k], d, 1.0f);
        dinv[k] = d;
        float row[B];
#pragma unroll
        for (int a = 0; a < k; ++a) {
            if ((S::anc[k] >> a) & 1ull) {
                row[a] = L[k][a] * d;
#pragma unroll
                for (int b = 0; b <= a; ++b)
                    if (b == a || ((S::anc[a] >> b) & 1ull))
                        L[a][b] -= row[a] * L[k][b];
            }
        }
#pragma unroll
        for (int a = 0; a < k; ++a)
            if ((S::anc[k] >> a) & 1ull)
                L[k][a] = row[a];
    }
}

// x <- M^-1 x
template <class S>
__device__ __forceinline__ void ltdl_solve(const float (&L)[S::B][S::B], const float (&dinv)[S::B],
                                           float (&x)[S::B])
{
    constexpr int B = S::B;
#pragma unroll
    for (int k = B - 1; k >= 0; --k)
#pragma unroll
        for (int a = 0; a < k; ++a)
            if ((S::anc[k] >> a) & 1ull)
                x[a] -= L[k][a] * x[k];
#pragma unroll
    for (int k = 0; k < B; ++k) {
        float t = x[k] * dinv[k];
#pragma unroll
        for (int a = 0; a < k; ++a)
            if ((S::anc[k] >> a) & 1ull)
                t -= L[k][a] * x[a];
        x[k] = t;
    }
}

}  // namespace gridv
