// One lane per (knot, branch) problem (gfx950): grid_fdgrad_serial, the batch forms of ID, FD, M^-1,
// dID and the adjoint VJP, and M^-1 alone by two routes.
//
// Every lane of a wavefront works on the same branch of the same robot for a different knot,
// so all model constants are instruction literals, nothing crosses lanes, and no work is
// repeated: the fewest instructions per knot of all the builds (the throughput form; its
// latency is one lane's whole chain). Per problem, float32 (Sec. IV-B), in the formulation of
// grid_axes.hip:
//   1. outward: axes, velocities, accelerations at qdd = 0, forces, inertias
//   2. inward: M by the subtrees' inertias and the bias forces; M = L^T D L along ancestor paths,
//      qdd = M^-1 (tau - c), M^-1 by B solves
//   3. outward: accelerations at qdd
//   4. inward: the derivatives from the subtrees' inertias, momenta and forces, each column moved
//      up its ancestor path; dqdd/du_j = -M^-1 dtau/du_j by the two triangular solves
//
// 65536 knots of chain7 are one wavefront per SIMD: bound by issue and by its stores, which do not
// overlap with it, since all wavefronts run in step (9 us at the rate of a copy). 37.1 us per launch
// with a derivative sweep per column, 21.0 here with half the instructions; quad12 44.7 and 32 (writes
// at 4.0 TB/s), at 16384 knots 19.7 and 10.5. FD / M^-1 / dID / VJP of chain7 at 32768 knots 13 / 11 /
// 19 / 19 us with one lane per body, 6.2 / 6.2 / 10.3 / 15.3 here.

namespace grids {

using grid::kConstStride;
using grid::prismatic;
using grid::s_index;
using grid::x_mv;
using grid::xt_fv;

template <class S>
__device__ __forceinline__ constexpr bool in_subtree(int i, int j)   // i == j or j an ancestor
{
    return i == j || ((S::anc[i] >> j) & 1ull);
}

struct RB {         // rigid-body inertia about the frame origin
    float m, h[3], I[6];   // I: xx yy zz xy xz yz
};

__device__ __forceinline__ RB rb_to_parent(const float* E, const float* r, const RB& c)
{
    const float Ib[3][3] = {{c.I[0], c.I[3], c.I[4]}, {c.I[3], c.I[1], c.I[5]},
                            {c.I[4], c.I[5], c.I[2]}};
    float T[3][3];    // Ibar E
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b)
            T[a][b] = Ib[a][0] * E[b] + Ib[a][1] * E[3 + b] + Ib[a][2] * E[6 + b];
    float ht[3];
#pragma unroll
    for (int a = 0; a < 3; ++a)
        ht[a] = E[a] * c.h[0] + E[3 + a] * c.h[1] + E[6 + a] * c.h[2];
    const float rh = r[0] * ht[0] + r[1] * ht[1] + r[2] * ht[2];
    const float rr = r[0] * r[0] + r[1] * r[1] + r[2] * r[2];
    RB o;
    o.m = c.m;
#pragma unroll
    for (int a = 0; a < 3; ++a)
        o.h[a] = ht[a] + c.m * r[a];
    const int ia[6] = {0, 1, 2, 0, 0, 1};
    const int ib[6] = {0, 1, 2, 1, 2, 2};
#pragma unroll
    for (int e = 0; e < 6; ++e) {
        const int a = ia[e], b = ib[e];
        const float etib = E[a] * T[0][b] + E[3 + a] * T[1][b] + E[6 + a] * T[2][b];
        const float diag = (a == b) ? 2.0f * rh + c.m * rr : 0.0f;
        o.I[e] = etib + diag - r[a] * ht[b] - ht[a] * r[b] - c.m * r[a] * r[b];
    }
    return o;
}

__device__ __forceinline__ void rb_add(RB& x, const RB& y)
{
    x.m += y.m;
#pragma unroll
    for (int a = 0; a < 3; ++a)
        x.h[a] += y.h[a];
#pragma unroll
    for (int e = 0; e < 6; ++e)
        x.I[e] += y.I[e];
}

// X_i = (E_i, r_i) of one body at joint position qi: E = E_z(q) E_T (hardware sin and cos,
// argument in revolutions reduced to [0, 1)), r = r_T; prismatic: E = E_T, r = r_T + q E_T^T e_z
template <class I>
__device__ __forceinline__ void serial_transform(int i, float qi, float (&E)[9], float (&R)[3])
{
    const float* c = I::consts() + i * kConstStride;
    if (prismatic<I>(i)) {
#pragma unroll
        for (int k = 0; k < 9; ++k)
            E[k] = c[k];
#pragma unroll
        for (int k = 0; k < 3; ++k)
            R[k] = c[9 + k] + qi * c[6 + k];
        return;
    }
    const float rev = __builtin_amdgcn_fractf(qi * 0.159154943091895336f);
    const float s = __builtin_amdgcn_sinf(rev);
    const float co = __builtin_amdgcn_cosf(rev);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        E[k] = co * c[k] + s * c[3 + k];
        E[3 + k] = co * c[3 + k] - s * c[k];
        E[6 + k] = c[6 + k];
        R[k] = c[9 + k];
    }
}

// M by composite rigid bodies, factored: I^c_i = I_i + sum over children of X^T I^c X as
// (mass, first moment, rotational inertia); M_ii = S^T I^c_i S and M_ki = S^T (X^T ... I^c_i S)
// up the ancestor path of i; then M = L^T L in place (Lf, dinv = 1 / L_kk)
template <class I>
__device__ __forceinline__ void serial_mass_factor(const float (&E)[I::S::B][9],
                                                   const float (&R)[I::S::B][3],
                                                   float (&Lf)[I::S::B][I::S::B],
                                                   float (&dinv)[I::S::B])
{
    using S = typename I::S;
    constexpr int B = S::B;
    const float* C = I::consts();
    RB Ic[B];
#pragma unroll
    for (int i = 0; i < B; ++i) {
        const float* c = C + i * kConstStride;
        Ic[i].m = c[21];
#pragma unroll
        for (int k = 0; k < 3; ++k)
            Ic[i].h[k] = c[18 + k];
#pragma unroll
        for (int k = 0; k < 6; ++k)
            Ic[i].I[k] = c[12 + k];
    }
#pragma unroll
    for (int i = B - 1; i >= 0; --i) {
        // I^c_i S: [Ibar e_z; -(h x e_z)] for S = (e_z, 0), [h x e_z; m e_z] for (0, e_z)
        float f[6] = {Ic[i].I[4], Ic[i].I[5], Ic[i].I[2], -Ic[i].h[1], Ic[i].h[0], 0.0f};
        if (prismatic<I>(i)) {
            f[0] = Ic[i].h[1];
            f[1] = -Ic[i].h[0];
            f[2] = 0.0f;
            f[3] = 0.0f;
            f[4] = 0.0f;
            f[5] = Ic[i].m;
        }
        Lf[i][i] = f[s_index(prismatic<I>(i))];
        // up the ancestor path (ancestors have smaller indices): f into the parent
        // frame of k, M_{lambda(k), i} = S^T f
#pragma unroll
        for (int k = B - 1; k >= 0; --k) {
            if (k <= i && (k == i || gridq::is_anc<S>(k, i)) && S::parent[k] >= 0) {
                float y[6];
                xt_fv(E[k], R[k], f, y);
#pragma unroll
                for (int e = 0; e < 6; ++e)
                    f[e] = y[e];
                const int pk = S::parent[k] < 0 ? 0 : S::parent[k];
                Lf[i][pk] = f[s_index(prismatic<I>(pk))];
            }
        }
        const int p = S::parent[i];
        if (p >= 0)
            rb_add(Ic[p], rb_to_parent(E[i], R[i], Ic[i]));
    }
    gridq::ltl_factor<S>(Lf, dinv);
}

constexpr int cmax(int a) { return a; }
template <class... T>
constexpr int cmax(int a, int b, T... rest) { return cmax(a > b ? a : b, rest...); }

// the workgroup is one wavefront: ordering its own LDS traffic needs no workgroup barrier
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int K>
struct Int {
    static constexpr int v = K;
};

// f(Int<0>), f(Int<1>), .. f(Int<N - 1>)
template <int N, int K = 0, class F>
__device__ __forceinline__ void static_for(const F& f)
{
    if constexpr (K < N) {
        f(Int<K>{});
        static_for<N, K + 1>(f);
    }
}

// Outputs. A lane that wrote the entries of its own knot would put 64 addresses N^2 floats apart
// into each store, so the B x B block of a matrix is staged in LDS ([knot][B][B]: the lane stride
// B^2 is odd for odd B, no bank conflicts) and the wavefront writes its knots' contiguous blocks
// with 16-byte stores when the branch is the whole robot, else its B rows of N floats per knot,
// zeros in the other branches' columns included.

// copy the [nv][N][N] floats of the wavefront's valid knots: 16 bytes per lane and step (global
// memory takes them at any 4-byte aligned address); several steps in flight, since one at a time
// waits for LDS and for memory in turn
template <int N>
__device__ __forceinline__ void flush_whole(float* dst, const float* src, int nv, int lane)
{
    constexpr int STEPS = (64 * N * N / 4 + 63) / 64;
    const int cnt = nv * N * N, n4 = cnt / 4;
#pragma unroll
    for (int s = 0; s < STEPS; ++s) {
        const int e = s * 64 + lane;
        if (e < n4) {
            const float4 v = reinterpret_cast<const float4*>(src)[e];
            reinterpret_cast<gridv::F4*>(dst)[e] = gridv::F4{v.x, v.y, v.z, v.w};
        }
    }
    if (4 * n4 + lane < cnt)                             // up to three floats left
        dst[4 * n4 + lane] = src[4 * n4 + lane];
}

// the branch's rows of a knot as V-float pieces, LPK of them; a lane keeps its place in the knot
// and strides over the knots, KPI at a time (one address computation per lane)
template <class I>
struct RowPieces {
    static constexpr int B = I::S::B, N = I::N;
    static constexpr int V = N % 4 == 0 ? 4 : (N % 2 == 0 ? 2 : 1);
    static constexpr int PPR = N / V;                    // pieces per row
    static constexpr int LPK = B * PPR;
    static constexpr int KPI = LPK <= 64 ? 64 / LPK : 0; // 0: a knot takes several steps
};

// write the blocks of the wavefront's nv valid knots, NM matrices; `d0`, `d1` are the blocks of
// its first knot
template <class I, int NM>
__device__ __forceinline__ void flush_blocks(float* d0, float* d1, const float* t0,
                                             const float* t1, int nv, int lane)
{
    using RP = RowPieces<I>;
    constexpr int B = RP::B, N = RP::N, V = RP::V;
    if constexpr (B == N) {
        flush_whole<N>(d0, t0, nv, lane);
        if constexpr (NM > 1)
            flush_whole<N>(d1, t1, nv, lane);
    } else {
        constexpr int KPI = RP::KPI > 0 ? RP::KPI : 1;
        constexpr int TURNS = RP::KPI > 0 ? 1 : (RP::LPK + 63) / 64;
#pragma unroll
        for (int turn = 0; turn < TURNS; ++turn) {
            const int e = turn * 64 + lane;
            const int kk = RP::KPI > 0 ? lane / RP::LPK : 0, rem = e - kk * RP::LPK;
            if (RP::KPI > 0 ? kk >= KPI : rem >= RP::LPK)
                continue;
            const int i = rem / RP::PPR, c = (rem - i * RP::PPR) * V;
            bool in[V];
            int at[V];
#pragma unroll
            for (int w = 0; w < V; ++w) {
                // the local column: the branch's bodies below c (local order follows the robot's)
                in[w] = I::contains(c + w);
                at[w] = i * B + (in[w] ? __popcll(I::mask & ((1ull << (c + w)) - 1)) : 0);
            }
            const int off = I::body_of(i) * N + c;
#pragma unroll 5
            for (int k = kk; k < nv; k += KPI) {
                float x[V], y[V];
#pragma unroll
                for (int w = 0; w < V; ++w) {
                    x[w] = in[w] ? t0[k * B * B + at[w]] : 0.0f;
                    y[w] = NM > 1 && in[w] ? t1[k * B * B + at[w]] : 0.0f;
                }
                gridv::store<V>(d0 + k * N * N + off, x);
                if constexpr (NM > 1)
                    gridv::store<V>(d1 + k * N * N + off, y);
            }
        }
    }
}

// LDS: the tiles of one matrix, or of two at a time where they are small (the addresses are then
// computed once), and what a lane parks while it factors M and writes M^-1: 16 floats for every
// body but the first. Without parking a branch of 7 bodies holds 330 floats there, which move
// through the accumulation registers and scratch memory (65536 knots 21.4 us, 20.2 with it, the rows
// of M in float32 then); one of 3 bodies has room (7.0 us at 128 knots, 7.7 with it), and so have
// the halves of dFD (7 bodies at 32768 knots 14.3, 22.8 with it: the LDS then leaves room for too few
// wavefronts)
template <class I, int OP>
struct SerialLds {
    static constexpr int B = I::S::B;
    static constexpr bool kPark = B > 4 && (OP == gridv::kFdGrad || OP == gridv::kVjp);
    static constexpr bool kTiles = OP != gridv::kFd && OP != gridv::kVjp && OP != gridv::kId;
    static constexpr int NT = !kTiles ? 0 : (B <= 4 && (OP == gridv::kFdGrad || OP == gridv::kIdGrad) ? 2 : 1);
    static constexpr int tile = 64 * B * B;
    static constexpr int floats = NT * tile + (kPark ? 16 * 64 * (B - 1) : 0) + 4;
};
template <class I, int OP>
constexpr int serial_floats()
{
    return SerialLds<I, OP>::floats;
}

// x <- M^-1 x, entry k of x zero unless bit k of MASK is set (MASK holds the ancestors of its
// bodies); entries up to LAST only
template <class S, unsigned long long MASK, int LAST>
__device__ __forceinline__ void solve_masked(const float (&L)[S::B][S::B],
                                             const float (&dinv)[S::B], float (&x)[S::B])
{
    constexpr int B = S::B;
    static_for<B>([&](auto kk) {
        constexpr int k = B - 1 - decltype(kk)::v;
        if constexpr ((MASK >> k) & 1ull) {
#pragma unroll
            for (int a = 0; a < k; ++a)
                if ((S::anc[k] >> a) & 1ull)
                    x[a] -= L[k][a] * x[k];
        }
    });
    static_for<LAST + 1>([&](auto kk) {
        constexpr int k = decltype(kk)::v;
        float t = ((MASK >> k) & 1ull) ? x[k] * dinv[k] : 0.0f;
#pragma unroll
        for (int a = 0; a < k; ++a)
            if ((S::anc[k] >> a) & 1ull)
                t -= L[k][a] * x[a];
        x[k] = t;
    });
}

// j, its ancestors and its subtree
template <class S>
constexpr unsigned long long relatives(int j)
{
    unsigned long long m = S::anc[j] | (1ull << j);
    for (int i = 0; i < S::B; ++i)
        if ((S::anc[i] >> j) & 1ull)
            m |= 1ull << i;
    return m;
}

// One lane per (knot, branch) problem. Along the first body's axes (grid_axes.hip) its rotation is
// the identity and its joint axis e_z, so that what concerns it folds.
template <class I, int OP>
__device__ __forceinline__ void run_serial(const gridv::BatchArgs& A, int block, float* pool)
{
    using namespace gridv;
    using S = typename I::S;
    constexpr int B = S::B;
    constexpr int N = I::N;
    using Y = SerialLds<I, OP>;
    constexpr bool kVel = OP != kMinv;
    constexpr bool kIdDer = OP == kIdGrad || OP == kIdGradQ || OP == kIdGradV;
    constexpr bool kMass = !kIdDer && OP != kId;
    constexpr bool kFdDer = OP == kFdGrad || OP == kFdGradQ || OP == kFdGradV;
    constexpr bool kQ = OP != kIdGradV && OP != kFdGradV;   // dq's matrix is wanted, dqd's
    constexpr bool kV = OP != kIdGradQ && OP != kFdGradQ;
    constexpr bool kBias = OP == kFdGrad || OP == kFdGradQ || OP == kFd;
    constexpr bool kDer = kIdDer || kFdDer || OP == kVjp;
    constexpr bool kPark = Y::kPark;
    constexpr bool kFine = kFineBranch<B>;
    const int lane = (int)threadIdx.x;
    const int kraw = block * 64 + lane;
    const bool valid = kraw < A.nknots;
    const int knot = valid ? kraw : A.nknots - 1;       // tail lanes recompute the last knot
    const int nv = min(64, A.nknots - block * 64);
    const float* C = I::consts();                       // literals: folded into the code
    const long vbase = (long)knot * N;
    const long mb = (long)block * 64 * N * N;           // the wavefront's first output block
    float* const mine = pool + lane * B * B;
    float4* const park = reinterpret_cast<float4*>(pool + Y::NT * Y::tile) + lane;
    const auto zero3 = V3{0.0f, 0.0f, 0.0f};

    float qd[B], uu[B];
    V3 z[B], r[B], h[B];
    Sym J[B];
    Six vl[B], psd[B], al[B];                           // vl, al: the parent's, at this origin
    Six own[B];                                         // the body's own inertia on a revolute S_i
    const auto pri = [](int i) { return prismatic<I>(i); };
    const auto add_S = [&](int i, Six y, float s) {
        if (pri(i))
            return Six{y.a, y.l + z[i] * s};
        return Six{y.a + z[i] * s, y.l};
    };
    const auto cross_S = [&](int i, Six x) {
        if (pri(i))
            return Six{zero3, cross(x.a, z[i])};
        return Six{cross(x.a, z[i]), cross(x.l, z[i])};
    };
    const auto dot_S = [&](int i, Six f) { return pri(i) ? dot(z[i], f.l) : dot(z[i], f.a); };
    const auto mass_of = [&](int i) { return C[i * kConstStride + 21]; };

    // ------------------------------------------------------------ outward: axes, velocities,
    // the parents' accelerations (at qdd = 0 for dFD and FD, else at the given qdd), inertias
    Six F[B];
    {
        MatD R[B];
        Six a[B], v[B];
        static_for<B>([&](auto ii) {
            constexpr int i = decltype(ii)::v;
            constexpr int p = S::parent[i];
            const float* c = C + i * kConstStride;
            const long o = vbase + I::body[i];
            const float qi = A.q[o];
            qd[i] = kVel ? A.qd[o] : 0.0f;
            uu[i] = kVel ? A.u[o] : 0.0f;
            using AX = AxesOf<kFine>;                   // the type that turns a body's quantities
            using VT = Vec<typename AX::T>;
            const auto X = joint_axes(pri(i), qi, VT{c[0], c[1], c[2]}, VT{c[3], c[4], c[5]},
                                      VT{c[6], c[7], c[8]});
            const Sym JT{c[12], c[13], c[14], c[15], c[16], c[17]};   // Ibar
            if constexpr (p < 0) {
                z[i] = V3{0.0f, 0.0f, 1.0f};
                r[i] = zero3;
                J[i] = JT;
                h[i] = V3{c[18], c[19], c[20]};
                own[i] = Six{{c[16], c[17], c[14]}, {-c[19], c[18], 0.0f}};
                al[i] = Six{zero3, narrow(tmul(X, VT{I::a0()[0], I::a0()[1], I::a0()[2]}))};
                vl[i] = Six{zero3, zero3};
                psd[i] = vl[i];
                v[i] = pri(i) ? Six{zero3, {0.0f, 0.0f, qd[i]}} : Six{{0.0f, 0.0f, qd[i]}, zero3};
                a[i] = al[i];
                if constexpr (!kBias) {
                    if (pri(i))
                        a[i].l.z += uu[i];
                    else
                        a[i].a.z = uu[i];
                }
            } else {
                if constexpr (S::parent[p] < 0) {       // the first body's axes
                    R[i] = wide(X);
                    r[i] = V3{c[9], c[10], c[11]};
                } else {
                    const MatD Y = wide(X);
                    R[i] = MatD{mul(R[p], Y.c0), mul(R[p], Y.c1), mul(R[p], Y.c2)};
                    r[i] = narrow(mul(AX::of(R[p]), VT{c[9], c[10], c[11]}));
                }
                const auto Ai = AX::of(R[i]);
                z[i] = narrow(Ai.c2);
                if (pri(i))
                    r[i] = r[i] + z[i] * qi;
                J[i] = turn(Ai, JT);
                h[i] = narrow(mul(Ai, VT{c[18], c[19], c[20]}));
                if constexpr (kFine)
                    own[i] = Six{narrow(mul(Ai, VT{c[16], c[17], c[14]})),
                                 narrow(mul(Ai, VT{-c[19], c[18], 0.0f}))};
                vl[i] = Six{v[p].a, v[p].l + cross(v[p].a, r[i])};
                psd[i] = cross_S(i, vl[i]);
                v[i] = add_S(i, vl[i], qd[i]);
                al[i] = Six{a[p].a, a[p].l + cross(a[p].a, r[i])};
                a[i] = Six{al[i].a + psd[i].a * qd[i], al[i].l + psd[i].l * qd[i]};
                if constexpr (!kBias)
                    a[i] = add_S(i, a[i], uu[i]);
                if constexpr (kPark) {
                    park[64 * (4 * i - 4)] = float4{J[i].xx, J[i].yy, J[i].zz, J[i].xy};
                    park[64 * (4 * i - 3)] = float4{J[i].xz, J[i].yz, h[i].x, h[i].y};
                    park[64 * (4 * i - 2)] = float4{h[i].z, psd[i].a.x, psd[i].a.y, psd[i].a.z};
                    park[64 * (4 * i - 1)] = float4{psd[i].l.x, psd[i].l.y, psd[i].l.z, qd[i]};
                }
            }
            if constexpr (kBias || OP == kId) {         // f = I a + v x* (I v)
                const Six Ia = inertia(mass_of(i), h[i], J[i], a[i]);
                const Six Iv = inertia(mass_of(i), h[i], J[i], v[i]);
                F[i] = Six{Ia.a + cross(v[i].a, Iv.a) + cross(v[i].l, Iv.l),
                           Ia.l + cross(v[i].a, Iv.l)};
            }
        });
    }

    if constexpr (OP == kId) {
        static_for<B>([&](auto ii) {
            constexpr int i = B - 1 - decltype(ii)::v;
            constexpr int p = S::parent[i];
            if (valid)
                A.o0[vbase + I::body[i]] = dot_S(i, F[i]);
            if constexpr (p >= 0)
                F[p] = Six{F[p].a + F[i].a + cross(r[i], F[i].l), F[p].l + F[i].l};
        });
        return;
    }

    // ------------------------------------------------------------ inward: M by the subtrees'
    // inertias, the bias forces, the factor
    float Lf[B][B], dinv[B], x[B];
    if constexpr (kMass) {
        Sym Jc[B];                                      // of the bodies below
        V3 hc[B];
        float mc[B];
#pragma unroll
        for (int i = 0; i < B; ++i) {
            Jc[i] = Sym{0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
            hc[i] = kFine ? zero3 : h[i];
            mc[i] = mass_of(i);
        }
        static_for<B>([&](auto ii) {
            constexpr int i = B - 1 - decltype(ii)::v;
            constexpr int p = S::parent[i];
            // the row of M in double; the body's own part of M_ii is a constant
            const V3D zi = wide(z[i]), below = mul(Jc[i], zi);
            Lf[i][i] = pri(i) ? mc[i] : (float)(C[i * kConstStride + 14] + dot(zi, below));
            const V3 ht = kFine ? hc[i] + h[i] : hc[i];
            V3D fa, fl;
            if (pri(i)) {
                fa = cross(wide(ht), zi);
                fl = zi * mc[i];
            } else {
                fa = below + (kFine ? wide(own[i].a) : mul(J[i], zi));
                fl = cross(zi, wide(hc[i]));
                if constexpr (kFine)
                    fl = fl + wide(own[i].l);
            }
            static_for<i>([&](auto tt) {                // the ancestors, nearest first
                constexpr int k = i - decltype(tt)::v;  // i, then each ancestor but the root
                if constexpr (k == i || ((S::anc[i] >> k) & 1ull)) {
                    constexpr int q = S::parent[k];
                    if constexpr (q >= 0) {
                        fa = fa + cross(wide(r[k]), fl);
                        Lf[i][q] = (float)dot(wide(z[q]), pri(q) ? fl : fa);
                    }
                }
            });
            if constexpr (kBias) {
                x[i] = uu[i] - dot_S(i, F[i]);
                if constexpr (p >= 0)
                    F[p] = Six{F[p].a + F[i].a + cross(r[i], F[i].l), F[p].l + F[i].l};
            }
            if constexpr (p >= 0) {
                Jc[i] = Jc[i] + J[i];
                hc[i] = ht;
                move_inertia(Jc[i], hc[i], mc[i], r[i]);
                Jc[p] = Jc[p] + Jc[i];
                hc[p] = hc[p] + hc[i];
                mc[p] += mc[i];
            }
        });
        if constexpr (OP == kVjp) {
#pragma unroll
            for (int i = 0; i < B; ++i)
                x[i] = A.u2[vbase + I::body[i]];
        }
        ltdl_factor<S>(Lf, dinv);
        if constexpr (kBias || OP == kVjp) {
            ltdl_solve<S>(Lf, dinv, x);           // qdd, or taubar
            if (valid) {
                float* out = OP == kVjp ? A.o2 : A.o0;
#pragma unroll
                for (int i = 0; i < B; ++i)
                    out[vbase + I::body[i]] = x[i];
            }
        }
    }
    if constexpr (OP == kFd)
        return;

    if constexpr (OP == kFdGrad || OP == kFdGradV || OP == kMinv) {
        // M^-1: entries (i, j), i <= j, to both mirrored positions (exactly symmetric)
        static_for<B>([&](auto jj) {
            constexpr int j = decltype(jj)::v;
            float m[B];
#pragma unroll
            for (int i = 0; i < B; ++i)
                m[i] = (i == j) ? 1.0f : 0.0f;
            solve_masked<S, S::anc[j] | (1ull << j), j>(Lf, dinv, m);
#pragma unroll
            for (int i = 0; i <= j; ++i) {
                mine[i * B + j] = m[i];
                mine[j * B + i] = m[i];
            }
        });
        wave_lds_sync();
        flush_blocks<I, 1>((OP == kMinv ? A.o0 : A.o1) + mb, nullptr, pool, nullptr, nv, lane);
        if constexpr (OP == kMinv)
            return;
        wave_lds_sync();
    }
    if constexpr (OP == kFdGrad || OP == kFdGradQ) {
        // the parents' accelerations at qdd
        Six d[B];
        static_for<B>([&](auto ii) {
            constexpr int i = decltype(ii)::v;
            constexpr int p = S::parent[i];
            if constexpr (p < 0) {
                d[i] = pri(i) ? Six{zero3, {0.0f, 0.0f, x[i]}} : Six{{0.0f, 0.0f, x[i]}, zero3};
            } else {
                d[i] = Six{d[p].a, d[p].l + cross(d[p].a, r[i])};
                al[i] = Six{al[i].a + d[i].a, al[i].l + d[i].l};
                d[i] = add_S(i, d[i], x[i]);
            }
        });
    }

    // ------------------------------------------------------------ inward: dtau/dq, dtau/dqd from
    // the subtrees' inertias, momenta and forces
    if constexpr (kDer) {
        float Dq[B][B], Dv[B][B];                       // [column][row]
        float gq[B], gv[B];                             // VJP: the products with taubar
        Six pdd[B];
        Mat K[B];
        V3 l[B];
        float mc[B];
#pragma unroll
        for (int i = 0; i < B; ++i)
            mc[i] = mass_of(i);
        static_for<B>([&](auto ii) {
            constexpr int i = decltype(ii)::v;
            if constexpr (kPark && i > 0) {
                const float4 a = park[64 * (4 * i - 4)], b = park[64 * (4 * i - 3)],
                             c = park[64 * (4 * i - 2)], d = park[64 * (4 * i - 1)];
                J[i] = Sym{a.x, a.y, a.z, a.w, b.x, b.y};
                h[i] = V3{b.z, b.w, c.x};
                psd[i] = Six{{c.y, c.z, c.w}, {d.x, d.y, d.z}};
                qd[i] = d.w;
            }
            const float qdd = kFdDer ? (kBias ? x[i] : 0.0f) : uu[i];
            const Six v = add_S(i, vl[i], qd[i]);
            const float* c = C + i * kConstStride;
            const float half = (float)(0.5 * ((double)c[12] + c[13] + c[14]));
            K[i] = momentum_moment(v, h[i], second_moment(J[i], half));
            l[i] = v.l * mass_of(i) + cross(v.a, h[i]);
            Six a = add_S(i, Six{al[i].a + psd[i].a * qd[i], al[i].l + psd[i].l * qd[i]}, qdd);
            const Six Ia = inertia(mass_of(i), h[i], J[i], a), Bv = bmul(K[i], l[i], v.a);
            F[i] = Six{Ia.a + Bv.a, Ia.l + Bv.l};
            const Six s = cross_S(i, al[i]);
            pdd[i] = S::parent[i] < 0 ? s
                                      : Six{s.a + cross(vl[i].a, psd[i].a),
                                            s.l + cross(vl[i].a, psd[i].l) + cross(vl[i].l, psd[i].a)};
            gq[i] = 0.0f;
            gv[i] = 0.0f;
        });
        static_for<B>([&](auto jj) {
            constexpr int j = B - 1 - decltype(jj)::v;
            constexpr int p = S::parent[j];
            Six f, u, w;
            V3 b;
            if (pri(j)) {
                f = Six{cross(h[j], z[j]), z[j] * mc[j]};
                b = cross(l[j], z[j]);
            } else {
                f = Six{mul(J[j], z[j]), cross(z[j], h[j])};
                b = z[j] * (K[j].c0.x + K[j].c1.y + K[j].c2.z) - tmul(K[j], z[j]);
            }
            {
                const Six Ip = inertia(mc[j], h[j], J[j], pdd[j]);
                const Six Sf = pri(j) ? Six{cross(z[j], F[j].l), zero3}
                                      : Six{cross(z[j], F[j].a), cross(z[j], F[j].l)};
                u = Six{Ip.a + Sf.a, Ip.l + Sf.l};
                w = Six{zero3, zero3};
                if constexpr (p >= 0) {                 // psd of the first body is zero
                    const Six Bp = bmul(K[j], l[j], psd[j].a);
                    u = Six{Bp.a * 2.0f + u.a, Bp.l * 2.0f + u.l};
                    w = inertia(mc[j], h[j], J[j], psd[j]);
                }
                if (!pri(j)) {
                    const Six Bs = bmul(K[j], l[j], z[j]);
                    w = Six{w.a + Bs.a, w.l + Bs.l};
                }
                w = Six{w.a * 2.0f, w.l * 2.0f};
            }
            const auto put = [&](int i, int c, float xq, float xv) {   // row i, column c
                if constexpr (OP == kVjp) {
                    gq[c] += xq * x[i];
                    gv[c] += xv * x[i];
                } else {
                    Dq[c][i] = xq;
                    Dv[c][i] = xv;
                }
            };
            put(j, j, dot_S(j, u), dot_S(j, w));
            const V3 b2 = b * 2.0f;
            static_for<j>([&](auto tt) {
                constexpr int k = j - decltype(tt)::v;
                if constexpr (k == j || ((S::anc[j] >> k) & 1ull)) {
                    constexpr int q = S::parent[k];
                    if constexpr (q >= 0) {
                        u.a = u.a + cross(r[k], u.l);
                        w.a = w.a + cross(r[k], w.l);
                        f.a = f.a + cross(r[k], f.l);
                        put(q, j, dot_S(q, u), dot_S(q, w));
                        float y = dot(f.a, pdd[q].a) + dot(f.l, pdd[q].l);
                        float t = pri(q) ? 0.0f : dot(b2, z[q]);
                        if constexpr (S::parent[q] >= 0) {
                            y += dot(b2, psd[q].a);
                            t += 2.0f * (dot(f.a, psd[q].a) + dot(f.l, psd[q].l));
                        }
                        put(j, q, y, t);
                    }
                }
            });
            if constexpr (p >= 0) {
                K[p].c0 = K[p].c0 + K[j].c0 + l[j] * r[j].x;
                K[p].c1 = K[p].c1 + K[j].c1 + l[j] * r[j].y;
                K[p].c2 = K[p].c2 + K[j].c2 + l[j] * r[j].z;
                l[p] = l[p] + l[j];
                F[p] = Six{F[p].a + F[j].a + cross(r[j], F[j].l), F[p].l + F[j].l};
                move_inertia(J[j], h[j], mc[j], r[j]);
                J[p] = J[p] + J[j];
                h[p] = h[p] + h[j];
                mc[p] += mc[j];
            }
        });
        if constexpr (OP == kVjp) {
            if (valid) {
#pragma unroll
                for (int i = 0; i < B; ++i) {
                    A.o0[vbase + I::body[i]] = -gq[i];
                    A.o1[vbase + I::body[i]] = -gv[i];
                }
            }
            return;
        }
        float* const o0 = (kFdDer ? A.o2 : A.o0) + mb;
        float* const o1 = (kFdDer ? A.o3 : A.o1) + mb;
        const auto columns = [&](float (&D)[B][B], float* to) {
            static_for<B>([&](auto jj) {
                constexpr int j = decltype(jj)::v;
                constexpr unsigned long long m = relatives<S>(j);
                if constexpr (kFdDer)
                    solve_masked<S, m, B - 1>(Lf, dinv, D[j]);
#pragma unroll
                for (int i = 0; i < B; ++i)
                    to[i * B + j] = kFdDer ? -D[j][i] : (((m >> i) & 1ull) ? D[j][i] : 0.0f);
            });
        };
        if constexpr (kQ)
            columns(Dq, mine);
        if constexpr (!kQ || !kV) {
            if constexpr (kV)
                columns(Dv, mine);
            wave_lds_sync();
            flush_blocks<I, 1>(kQ ? o0 : o1, nullptr, pool, nullptr, nv, lane);
        } else if constexpr (Y::NT == 2) {
            columns(Dv, mine + Y::tile);
            wave_lds_sync();
            flush_blocks<I, 2>(o0, o1, pool, pool + Y::tile, nv, lane);
        } else {
            wave_lds_sync();
            flush_blocks<I, 1>(o0, nullptr, pool, nullptr, nv, lane);
            wave_lds_sync();
            columns(Dv, mine);
            wave_lds_sync();
            flush_blocks<I, 1>(o1, nullptr, pool, nullptr, nv, lane);
        }
    }
}

// ------------------------------------------------------------------ M^-1 alone, two routes
//
// One lane per (knot, branch) problem, as build 5, computing only M^-1, by either route:
//   kDirect = false: M by composite rigid bodies, M = L^T L along ancestor paths, and the B
//     columns of M^-1 by two triangular solves each (the route every fused build takes);
//   kDirect = true: the paper's direct inverse (Sec. IV-B): the articulated-body recursion
//     with zero velocity and gravity and the identity as its B right-hand sides. Inward,
//     U_i = IA_i S_i, D_i = S_i^T U_i, row_i = (e_i^T - S_i^T F_i) / D_i over the columns
//     of the subtree of i, IA_lambda += X^T (IA_i - U_i U_i^T / D_i) X and
//     F_lambda += X^T (F_i + U_i row_i); outward, per column c, A = X_i P_lambda,
//     row_i -= U_i^T A / D_i and P_i = A + S_i row_i; M^-1 = [row_i]. The articulated
//     inertias do not depend on the right-hand sides, so they come first, and then each
//     column runs its inward and outward steps (the same arithmetic, fewer live values).
// Both write the upper triangle of the branch's block to both mirrored positions (exactly
// symmetric) and zeros in the other branches' columns, one float per store.

// articulated-body inertia [[A, B], [B^T, C]] in a body frame: A, C symmetric (xx yy zz xy xz
// yz), B row-major
struct AB {
    float A[6], B[9], C[6];
};

__device__ __forceinline__ constexpr int sym3(int a, int b)
{
    return a == b ? a : (a + b == 1 ? 3 : (a + b == 2 ? 4 : 5));
}

// X^T Ia X for X = [E 0; -E r~ E]: with A' = E^T A E, B' = E^T B E, C' = E^T C E,
//   C'' = C', B'' = B' + r~ C', A'' = A' + G + G^T - r~ C' r~, G = r~ B'^T
// (X = diag(E, E) [1 0; -r~ 1]; for a rigid body this is the transform rb_to_parent writes out)
__device__ __forceinline__ AB ab_to_parent(const float* E, const float* r, const AB& x)
{
    float A1[6], C1[6], B1[3][3];
    {
        float Ta[3][3], Tb[3][3], Tc[3][3];    // A E, B E, C E
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                Ta[a][b] = x.A[sym3(a, 0)] * E[b] + x.A[sym3(a, 1)] * E[3 + b] +
                           x.A[sym3(a, 2)] * E[6 + b];
                Tb[a][b] = x.B[3 * a] * E[b] + x.B[3 * a + 1] * E[3 + b] + x.B[3 * a + 2] * E[6 + b];
                Tc[a][b] = x.C[sym3(a, 0)] * E[b] + x.C[sym3(a, 1)] * E[3 + b] +
                           x.C[sym3(a, 2)] * E[6 + b];
            }
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                B1[a][b] = E[a] * Tb[0][b] + E[3 + a] * Tb[1][b] + E[6 + a] * Tb[2][b];
                if (a <= b) {
                    A1[sym3(a, b)] = E[a] * Ta[0][b] + E[3 + a] * Ta[1][b] + E[6 + a] * Ta[2][b];
                    C1[sym3(a, b)] = E[a] * Tc[0][b] + E[3 + a] * Tc[1][b] + E[6 + a] * Tc[2][b];
                }
            }
    }
    const float rt[3][3] = {{0.0f, -r[2], r[1]}, {r[2], 0.0f, -r[0]}, {-r[1], r[0], 0.0f}};
    float W[3][3], G[3][3];                    // r~ C', r~ B'^T
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            W[a][b] = rt[a][0] * C1[sym3(0, b)] + rt[a][1] * C1[sym3(1, b)] +
                      rt[a][2] * C1[sym3(2, b)];
            G[a][b] = rt[a][0] * B1[b][0] + rt[a][1] * B1[b][1] + rt[a][2] * B1[b][2];
        }
    AB o;
#pragma unroll
    for (int e = 0; e < 6; ++e)
        o.C[e] = C1[e];
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            o.B[3 * a + b] = B1[a][b] + W[a][b];
            if (a <= b) {
                const float wr = W[a][0] * rt[0][b] + W[a][1] * rt[1][b] + W[a][2] * rt[2][b];
                o.A[sym3(a, b)] = A1[sym3(a, b)] + G[a][b] + G[b][a] - wr;
            }
        }
    return o;
}

template <class I, bool kDirect>
__device__ __forceinline__ void run_minv(const grid::Args& A, int block)
{
    using S = typename I::S;
    constexpr int B = S::B;
    constexpr int N = I::N;
    const int lane = (int)threadIdx.x;
    const int kraw = block * 64 + lane;
    const bool valid = kraw < A.nknots;
    const int knot = valid ? kraw : A.nknots - 1;
    const long mbase = (long)knot * N * N;
    float E[B][9], R[B][3];
#pragma unroll
    for (int i = 0; i < B; ++i)
        serial_transform<I>(i, A.q[(long)knot * N + I::body[i]], E[i], R[i]);
    const auto put = [&](int i, int c, float x) {   // entry (i, c), i <= c, and its mirror
        if (valid) {
            A.Minv[mbase + (long)I::body[i] * N + I::body[c]] = x;
            A.Minv[mbase + (long)I::body[c] * N + I::body[i]] = x;
        }
    };
    if constexpr (!kDirect) {
        float Lf[B][B], dinv[B];
        serial_mass_factor<I>(E, R, Lf, dinv);
#pragma unroll
        for (int c = 0; c < B; ++c) {
            float mc[B];
#pragma unroll
            for (int i = 0; i < B; ++i)
                mc[i] = (i == c) ? 1.0f : 0.0f;
            gridq::ltl_solve<S>(Lf, dinv, mc);
#pragma unroll
            for (int i = 0; i <= c; ++i)
                put(i, c, mc[i]);
        }
    } else {
        const float* C = I::consts();
        float U[B][6], dv[B];
        {
            // inward: the articulated inertias, U_i = IA_i S_i and 1 / D_i (no right-hand side
            // enters them)
            AB Ia[B];
#pragma unroll
            for (int i = 0; i < B; ++i) {   // I_i = [[Ibar, h~], [-h~, m 1]]
                const float* c = C + i * kConstStride;
                const float h0 = c[18], h1 = c[19], h2 = c[20], m = c[21];
#pragma unroll
                for (int k = 0; k < 6; ++k)
                    Ia[i].A[k] = c[12 + k];
                const float hb[9] = {0.0f, -h2, h1, h2, 0.0f, -h0, -h1, h0, 0.0f};
#pragma unroll
                for (int k = 0; k < 9; ++k)
                    Ia[i].B[k] = hb[k];
                const float cm[6] = {m, m, m, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int k = 0; k < 6; ++k)
                    Ia[i].C[k] = cm[k];
            }
#pragma unroll
            for (int i = B - 1; i >= 0; --i) {
                const AB& x = Ia[i];
                if (prismatic<I>(i)) {        // IA_i e_6 = [B[:, 2]; C[:, 2]]
                    const float u[6] = {x.B[2], x.B[5], x.B[8], x.C[4], x.C[5], x.C[2]};
#pragma unroll
                    for (int k = 0; k < 6; ++k)
                        U[i][k] = u[k];
                } else {                      // IA_i e_3 = [A[:, 2]; B[2, :]]
                    const float u[6] = {x.A[4], x.A[5], x.A[2], x.B[6], x.B[7], x.B[8]};
#pragma unroll
                    for (int k = 0; k < 6; ++k)
                        U[i][k] = u[k];
                }
                dv[i] = 1.0f / U[i][s_index(prismatic<I>(i))];
                const int p = S::parent[i];
                if (p < 0)
                    continue;
                AB y = x;                     // IA_i - U_i U_i^T / D_i
                const float* Ua = U[i];
                const float* Ul = U[i] + 3;
#pragma unroll
                for (int a = 0; a < 3; ++a)
#pragma unroll
                    for (int b = 0; b < 3; ++b) {
                        y.B[3 * a + b] -= Ua[a] * Ul[b] * dv[i];
                        if (a <= b) {
                            y.A[sym3(a, b)] -= Ua[a] * Ua[b] * dv[i];
                            y.C[sym3(a, b)] -= Ul[a] * Ul[b] * dv[i];
                        }
                    }
                const AB z = ab_to_parent(E[i], R[i], y);
                const int pp = p < 0 ? 0 : p;
#pragma unroll
                for (int k = 0; k < 6; ++k) {
                    Ia[pp].A[k] += z.A[k];
                    Ia[pp].C[k] += z.C[k];
                }
#pragma unroll
                for (int k = 0; k < 9; ++k)
                    Ia[pp].B[k] += z.B[k];
            }
        }
        // the right-hand sides one column c at a time (the recursion is linear in them): F_i
        // of column c is nonzero only on the ancestor path of c, so inward it is one 6-vector
        // carried from c to the root; outward every body takes its row entry
#pragma unroll
        for (int c = 0; c < B; ++c) {
            float row[B];
            {
                float f[6] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int i = B - 1; i >= 0; --i) {
                    if (!in_subtree<S>(c, i)) {
                        row[i] = 0.0f;
                        continue;
                    }
                    row[i] = ((c == i ? 1.0f : 0.0f) - f[s_index(prismatic<I>(i))]) * dv[i];
                    if (S::parent[i] >= 0) {
                        float col[6];
#pragma unroll
                        for (int k = 0; k < 6; ++k)
                            col[k] = f[k] + U[i][k] * row[i];
                        xt_fv(E[i], R[i], col, f);
                    }
                }
            }
            float P[B][6];
#pragma unroll
            for (int i = 0; i < B; ++i) {
                const int p = S::parent[i];
                float Av[6] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
                float x = row[i];
                if (p >= 0) {
                    x_mv(E[i], R[i], P[p < 0 ? 0 : p], Av);
                    float ua = 0.0f;
#pragma unroll
                    for (int k = 0; k < 6; ++k)
                        ua += U[i][k] * Av[k];
                    x -= ua * dv[i];
                }
#pragma unroll
                for (int k = 0; k < 6; ++k)
                    P[i][k] = Av[k];
                P[i][s_index(prismatic<I>(i))] += x;
                if (i <= c)
                    put(i, c, x);
            }
        }
    }
    if (valid && N > B) {
        // this branch's rows hold zeros in the other branches' columns
#pragma unroll
        for (int i = 0; i < B; ++i)
#pragma unroll
            for (int c2 = 0; c2 < N; ++c2)
                if (!I::contains(c2))
                    A.Minv[mbase + (long)I::body[i] * N + c2] = 0.0f;
    }
}

}  // namespace grids

// kernels of a one-robot module (a module of several robots defines GRID_PIPE_ONLY and its
// own entry point, grid_fdgrad_pipe_mixed)
#ifndef GRID_PIPE_ONLY

// (a robot with a branch of more than 8 bodies has none of the three: they would hold most of
// a problem in scratch memory)
#if !GRID_LONG_BRANCH

// defined by the generated epilogue: workgroup -> (branch, 64 knots)
template <int OP>
__device__ void grid_dispatch_s(const gridv::BatchArgs& args, int block);

extern "C" __global__ void __launch_bounds__(64) grid_fdgrad_serial(grid::Args args)
{
    const gridv::BatchArgs a{args.nknots, args.q, args.qd, args.tau, nullptr,
                        args.qdd, args.Minv, args.dqdd_dq, args.dqdd_dqd};
    grid_dispatch_s<gridv::kFdGrad>(a, (int)blockIdx.x);
}

// dFD by two wavefronts: qdd and dqdd/dq; M^-1 and dqdd/dqd. Each repeats the axes, the inertias
// and the factor, 27 % more instructions in all, but runs 0.6 of them: chain7 at 32768 knots 18.7
// us by one wavefront, 14.3 by two, at 65536 20.2 and 24.0
extern "C" __global__ void __launch_bounds__(64) grid_fdgrad_serial_halves(grid::Args args)
{
    const gridv::BatchArgs a{args.nknots, args.q, args.qd, args.tau, nullptr,
                        args.qdd, args.Minv, args.dqdd_dq, args.dqdd_dqd};
    const int half = (int)gridDim.x / 2, b = (int)blockIdx.x;
    if (b < half)
        grid_dispatch_s<gridv::kFdGradQ>(a, b);
    else
        grid_dispatch_s<gridv::kFdGradV>(a, b - half);
}

// the standalone algorithms in the same layout (their arguments as gridq::OpArgs)
struct SerialOpArgs {
    int nknots;
    const float *q, *qd, *u, *u2;
    float *out0, *out1, *out2;
};

extern "C" __global__ void __launch_bounds__(64) grid_serial_fd(SerialOpArgs x)
{
    const gridv::BatchArgs a{x.nknots, x.q, x.qd, x.u, nullptr, x.out0, nullptr, nullptr, nullptr};
    grid_dispatch_s<gridv::kFd>(a, (int)blockIdx.x);
}

extern "C" __global__ void __launch_bounds__(64) grid_serial_minv(SerialOpArgs x)
{
    const gridv::BatchArgs a{x.nknots, x.q,     nullptr, nullptr, nullptr,
                             x.out0,   nullptr, nullptr, nullptr};
    grid_dispatch_s<gridv::kMinv>(a, (int)blockIdx.x);
}

extern "C" __global__ void __launch_bounds__(64) grid_serial_idgrad(SerialOpArgs x)
{
    const gridv::BatchArgs a{x.nknots, x.q, x.qd, x.u, nullptr, x.out0, x.out1, nullptr, nullptr};
    grid_dispatch_s<gridv::kIdGrad>(a, (int)blockIdx.x);
}

// dID by two wavefronts, one matrix each: chain7 at 32768 knots 11.9 us by one, 9.8 by two, at
// 65536 13.5 and 16.4
extern "C" __global__ void __launch_bounds__(64) grid_serial_idgrad_halves(SerialOpArgs x)
{
    const int half = (int)gridDim.x / 2, b = (int)blockIdx.x;
    if (b < half) {
        const gridv::BatchArgs a{x.nknots, x.q, x.qd, x.u, nullptr, x.out0, nullptr, nullptr, nullptr};
        grid_dispatch_s<gridv::kIdGradQ>(a, b);
    } else {
        const gridv::BatchArgs a{x.nknots, x.q, x.qd, x.u, nullptr, nullptr, x.out1, nullptr, nullptr};
        grid_dispatch_s<gridv::kIdGradV>(a, b - half);
    }
}

// against the quad layout's (grid_ops.hip): chain7 at 32768 and 65536 knots 4.2 and 6.4 us there,
// 4.3 and 4.5 here; quad12 at 8192, 16384 and 32768 3.0 / 3.7 / 5.3 and 3.2 / 3.1 / 3.2
extern "C" __global__ void __launch_bounds__(64) grid_serial_id(SerialOpArgs x)
{
    const gridv::BatchArgs a{x.nknots, x.q, x.qd, x.u, nullptr, x.out0, nullptr, nullptr, nullptr};
    grid_dispatch_s<gridv::kId>(a, (int)blockIdx.x);
}

extern "C" __global__ void __launch_bounds__(64) grid_serial_vjp(SerialOpArgs x)
{
    const gridv::BatchArgs a{x.nknots, x.q, x.qd, x.u, x.u2, x.out0, x.out1, x.out2, nullptr};
    grid_dispatch_s<gridv::kVjp>(a, (int)blockIdx.x);
}

#endif  // GRID_LONG_BRANCH

// defined by the generated epilogue: workgroup -> (branch, 64 knots), M^-1 by either route
template <bool kDirect>
__device__ void grid_dispatch_minv(const grid::Args& args, int block);

// M^-1 alone, one lane per knot: composite bodies and the L^T L factor
extern "C" __global__ void __launch_bounds__(64) grid_minv_serial(grid::Args args)
{
    grid_dispatch_minv<false>(args, (int)blockIdx.x);
}

// M^-1 alone, one lane per knot: the direct articulated-body inverse (Sec. IV-B)
extern "C" __global__ void __launch_bounds__(64) grid_minv_direct(grid::Args args)
{
    grid_dispatch_minv<true>(args, (int)blockIdx.x);
}

#endif  // GRID_PIPE_ONLY
