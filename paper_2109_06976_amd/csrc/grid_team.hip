// One lane per body (gfx950): grid_fdgrad_team and the batch forms of FD, M^-1, dID and the
// adjoint VJP.
//
// A problem is one (knot, base branch). Its B bodies sit on B adjacent lanes of a wavefront, so
// a wavefront holds as many knots as fit, with all branches of one shape side by side
// (Group<g>: NB branches of shape S). Each lane keeps its own body's quantities in registers
// and meets the others through LDS; a workgroup is one wavefront, so no barrier is needed.
//
// The formulation is that of grid_axes.hip. M^-1 comes from M = L^T L (sparse along ancestor
// paths), which every lane of a problem factors for itself from the rows of M in LDS: 57 (7-body chain) to 324 (18-body tree) FMAs in
// registers against one LDS round trip per level for a shared factor. Lane j then solves for
// column j of M^-1, dqdd/dq and dqdd/dqd.
//
// Bound by the latency of its chain of LDS exchanges up to a few wavefronts per SIMD, by VALU
// issue beyond. humanoid30: 236 us per launch at 4096 knots and 648 at 16384 on the kernels it
// took the place of, 28 and 82 here; chain7 at 4096 knots 11.4 and 10.7, quad12 7.8 and 6.8.
// FD / M^-1 / dID / VJP against the quad layout's (grid_ops.hip): humanoid30 at 4096 knots 46 /
// 31 / 192 / 68 and 12 / 12 / 18 / 18 us, at 128 9.8 / 9.7 / 11.3 / 14.1 and 8.7 / 8.0 / 11.1 /
// 12.0; chain7 at 32768 29 / 16 / 77 / 53 and 13 / 11 / 19 / 19.

namespace gridt {

using grids::wave_lds_sync;

using namespace gridv;

// compile-time facts of a shape
template <class S>
struct Tree {
    static constexpr int depth(int i)
    {
        int d = 0;
        for (int p = S::parent[i]; p >= 0; p = S::parent[p])
            ++d;
        return d;
    }
    static constexpr int max_depth()
    {
        int d = 0;
        for (int i = 0; i < S::B; ++i)
            d = depth(i) > d ? depth(i) : d;
        return d;
    }
    // ancestor of i at distance t + 1
    static constexpr int anc_at(int i, int t)
    {
        int p = S::parent[i];
        for (int k = 0; k < t; ++k)
            p = S::parent[p];
        return p;
    }
    // most children that a body of depth lev - 1 has
    static constexpr int max_children(int lev)
    {
        int m = 0;
        for (int p = 0; p < S::B; ++p) {
            int c = 0;
            for (int i = 0; i < S::B; ++i)
                c += (S::parent[i] == p && depth(i) == lev) ? 1 : 0;
            m = c > m ? c : m;
        }
        return m;
    }
    static constexpr bool chain()
    {
        return max_depth() == S::B - 1;
    }
};

constexpr int up4(int x) { return (x + 3) / 4 * 4; }

template <class G>
struct Lay {
    using S = typename G::S;
    static constexpr int B = S::B;
    static constexpr int NB = G::NB;
    static constexpr int N = G::N;
    static constexpr int KPB = 64 / (NB * B);          // knots per wavefront
    static constexpr int SL = KPB * NB;                // problems per wavefront
    static constexpr int NE = SL * B + 1;              // bodies, and an entry of zeros
    static constexpr int MD = Tree<S>::max_depth();
    static constexpr int AW = MD > 0 ? (MD + 3) / 4 : 1;
    static constexpr int RS = up4(MD + 1);             // a row of M: self, then ancestors
    static constexpr int BS = up4(B);
    static constexpr bool FULL = NB * B == N;          // the group is the whole robot
    // floats: six fields of a float4 per body (z and a scalar, r, psd, pdd), a vector per
    // problem, then one region that the level exchange (seven fields), M and the columns of
    // dtau use in turn; the output tiles take the place of everything at the end
    static constexpr int oX = 6 * 4 * NE;
    static constexpr int oU = oX + up4(SL * BS);
    static constexpr int exch = 7 * 4 * NE;
    static constexpr int rows = SL * B * RS;
    static constexpr int cols = 2 * SL * B * BS;
    static constexpr int tile = FULL ? up4(KPB * N * N) : up4(SL * B * B);
    static constexpr int mx(int a, int b) { return a > b ? a : b; }
    static constexpr int floats = mx(oU + mx(mx(exch, rows), cols), 3 * tile);
};

template <class G>
constexpr int team_floats()
{
    return Lay<G>::floats;
}

__device__ __forceinline__ void flush_block(float* dst, const float* src, int cnt, int lane)
{
    const int n4 = cnt / 4;
    for (int e = lane; e < n4; e += 64) {
        const float4 v = reinterpret_cast<const float4*>(src)[e];
        reinterpret_cast<F4*>(dst)[e] = F4{v.x, v.y, v.z, v.w};
    }
    for (int e = 4 * n4 + lane; e < cnt; e += 64)
        dst[e] = src[e];
}

// NM matrices' tiles ([knot][N][N], or the branch's blocks [problem][B][B] when the group is not
// the whole robot: then its rows, zeros in the other branches' columns) to global memory
template <class G, int NM>
__device__ __forceinline__ void flush_tiles(const float* pool, float* d0, float* d1, float* d2,
                                            int block, int nv, int lane)
{
    using Y = Lay<G>;
    constexpr int B = Y::B, N = Y::N, NB = Y::NB;
    const long kb = (long)block * Y::KPB * N * N;
    if constexpr (Y::FULL) {
        flush_block(d0 + kb, pool, nv * N * N, lane);
        if constexpr (NM > 1)
            flush_block(d1 + kb, pool + Y::tile, nv * N * N, lane);
        if constexpr (NM > 2)
            flush_block(d2 + kb, pool + 2 * Y::tile, nv * N * N, lane);
    } else {
        // RPI rows of N floats per step; a lane keeps its column and, per branch, that column's
        // place in the tile and the offsets of its rows (loaded once, not per knot)
        constexpr int RPI = 64 / N, STEPS = (B + RPI - 1) / RPI;
        const int lr = lane / N, lc = lane - lr * N;
        int row[NB][STEPS], col[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            col[b] = G::colmap()[b * N + lc];
#pragma unroll
            for (int k = 0; k < STEPS; ++k) {
                const int i = k * RPI + lr;
                row[b][k] = G::rowmap()[b * B + (i < B ? i : 0)] * N + lc;
            }
        }
        if (lr >= RPI)
            return;
#pragma unroll
        for (int ks = 0; ks < Y::KPB; ++ks) {
            if (ks >= nv)
                return;
            float* const p0 = d0 + kb + ks * N * N;
            float* const p1 = NM > 1 ? d1 + kb + ks * N * N : nullptr;
            float* const p2 = NM > 2 ? d2 + kb + ks * N * N : nullptr;
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const bool in = col[b] >= 0;
                const float* src = pool + (ks * NB + b) * B * B + lr * B + (in ? col[b] : 0);
#pragma unroll
                for (int k = 0; k < STEPS; ++k) {
                    if (k * RPI + RPI > B && k * RPI + lr >= B)
                        break;
                    const float* x = src + k * RPI * B;
                    p0[row[b][k]] = in ? x[0] : 0.0f;
                    if constexpr (NM > 1)
                        p1[row[b][k]] = in ? x[Y::tile] : 0.0f;
                    if constexpr (NM > 2)
                        p2[row[b][k]] = in ? x[2 * Y::tile] : 0.0f;
                }
            }
        }
    }
}

template <class G, int OP>
__device__ __forceinline__ void run_team(const BatchArgs& A, int block, float* pool)
{
    using S = typename G::S;
    using Y = Lay<G>;
    using T = Tree<S>;
    constexpr int B = Y::B, NB = Y::NB, N = Y::N, MD = Y::MD, NE = Y::NE, BS = Y::BS;
    constexpr int DZ = NE - 1;                         // the entry of zeros
    constexpr bool kVel = OP != kMinv;
    constexpr bool kMass = OP != kIdGrad;
    constexpr bool kBias = OP == kFdGrad || OP == kFd;
    constexpr bool kDer = OP == kFdGrad || OP == kIdGrad || OP == kVjp;
    constexpr bool kPrism = G::prism;

    const int lane = (int)threadIdx.x;
    // lanes past the last problem repeat lanes of that problem: same values, same addresses
    const int id = lane < Y::SL * B ? lane : lane - B * ((lane - Y::SL * B) / B + 1);
    const int slot = id / B;
    const int i = id - slot * B;
    const int ks = slot / NB, br = slot - ks * NB;
    const int kraw = block * Y::KPB + ks;
    const int nv = min(Y::KPB, A.nknots - block * Y::KPB);
    const bool valid = kraw < A.nknots;
    const int knot = valid ? kraw : A.nknots - 1;      // tail problems recompute the last knot
    const int sb = slot * B;                           // the problem's first entry
    const int me = sb + i;

    float4* const fZ = reinterpret_cast<float4*>(pool);        // z, scalar (qd or qdd)
    float4* const fR = fZ + NE;                                // r, 1 for a prismatic joint
    float4* const fP0 = fR + NE;                               // psd
    float4* const fP1 = fP0 + NE;
    float4* const fQ0 = fP1 + NE;                              // pdd
    float4* const fQ1 = fQ0 + NE;
    float* const sx = pool + Y::oX + slot * BS;
    float4* const fU = reinterpret_cast<float4*>(pool + Y::oU);
    float* const sM = pool + Y::oU;
    float* const sT = pool + Y::oU;
    constexpr int TQ = Y::SL * B * BS;                 // from a column of dtau/dq to dtau/dqd's

    // ------------------------------------------------------------ the lane's body
    const int4 ti = reinterpret_cast<const int4*>(G::ints())[(br * B + i) * 3];
    const int body = ti.x, depth = ti.y, rank = ti.z, nchild = ti.w;
    const long vo = (long)knot * N + body;
    const float qi = A.q[vo];
    const float qd = kVel ? A.qd[vo] : 0.0f;
    const float ui = kVel ? A.u[vo] : 0.0f;
    int anc[MD > 0 ? MD : 1];                          // entries of the ancestors, parent first
    {
        const int* aw = G::ints() + (br * B + i) * 12 + 4;
#pragma unroll
        for (int t = 0; t < MD; ++t)
            anc[t] = t < depth ? sb + ((aw[t / 4] >> (8 * (t % 4))) & 255) : DZ;
    }
    const int parent = MD > 0 ? anc[0] : DZ;           // entry; the root's is the zeros
    const float4* tf = reinterpret_cast<const float4*>(G::table()) + (br * B + i) * 6;
    const float4 t0 = tf[0], t1 = tf[1], t2 = tf[2], t3 = tf[3], t4 = tf[4], t5 = tf[5];
    const V3 e0{t0.x, t0.y, t0.z}, e1{t0.w, t1.x, t1.y}, e2{t1.z, t1.w, t2.x};   // rows of E_T
    const V3 rT{t2.y, t2.z, t2.w};
    const Sym PT{t3.x, t3.y, t3.z, t3.w, t4.x, t4.y};
    const V3 hT{t4.z, t4.w, t5.x};
    const float m = t5.y, mC = t5.z;
    const bool pr = kPrism && t5.w != 0.0f;

    // body axes along the parent's: the rows of E = E_z(q) E_T, or E_T
    float sn = 0.0f, co = 1.0f;
    if (!pr) {
        const float rev = __builtin_amdgcn_fractf(qi * 0.159154943091895336f);
        sn = __builtin_amdgcn_sinf(rev);
        co = __builtin_amdgcn_cosf(rev);
    }
    Mat R{e0 * co + e1 * sn, e1 * co - e0 * sn, e2};
    V3 rb = tmul(R, rT);                               // r in body axes
    if (kPrism && pr)
        rb.z += qi;
    V3 a0 = {0.0f, 0.0f, 0.0f};                        // -g along the first body's axes
    if constexpr (kVel) {
        const V3 g{G::a0()[0], G::a0()[1], G::a0()[2]};
        a0 = tmul(R, g);
    }
    if (depth == 0)
        R = Mat{{1.0f, 0.0f, 0.0f}, {0.0f, 1.0f, 0.0f}, {0.0f, 0.0f, 1.0f}};
    // products along the path to the first body, by doubling
#pragma unroll
    for (int s = 1; s < MD; s *= 2) {
        fU[me] = float4{R.c0.x, R.c0.y, R.c0.z, R.c1.x};
        fU[NE + me] = float4{R.c1.y, R.c1.z, R.c2.x, R.c2.y};
        fU[2 * NE + me] = float4{R.c2.z, 0.0f, 0.0f, 0.0f};
        wave_lds_sync();
        if (depth > s) {                               // an ancestor below the first body
            const int k = anc[s - 1];
            const float4 x = fU[k], y = fU[NE + k];
            const float z = fU[2 * NE + k].x;
            const Mat Q{{x.x, x.y, x.z}, {x.w, y.x, y.y}, {y.z, y.w, z}};
            R = Mat{mul(Q, R.c0), mul(Q, R.c1), mul(Q, R.c2)};
        }
        wave_lds_sync();
    }
    const V3 z = R.c2;
    const V3 r = depth == 0 ? V3{0.0f, 0.0f, 0.0f} : mul(R, rb);
    fZ[me] = float4{z.x, z.y, z.z, qd};
    fR[me] = float4{r.x, r.y, r.z, pr ? 1.0f : 0.0f};
    if (lane == 0) {
        const float4 zero{0.0f, 0.0f, 0.0f, 0.0f};
        fZ[DZ] = zero;
        fR[DZ] = zero;
        fP0[DZ] = zero;
        fP1[DZ] = zero;
        fQ0[DZ] = zero;
        fQ1[DZ] = zero;
    }
    if constexpr (kVel) {                              // the first body's lane has -g
        if (depth == 0)
            fU[me] = float4{a0.x, a0.y, a0.z, 0.0f};
    }
    wave_lds_sync();
    if constexpr (kVel) {
        const float4 g = fU[sb];
        a0 = V3{g.x, g.y, g.z};
    }

    // sum over the strict ancestors k of S_k s_k, moved to this body's origin (s_k: the scalar
    // beside z_k)
    const auto path_sum = [&]() {
        Six x{{0.0f, 0.0f, 0.0f}, {0.0f, 0.0f, 0.0f}};
        V3 D = r;
#pragma unroll
        for (int t = 0; t < MD; ++t) {
            const float4 zk = fZ[anc[t]], rk = fR[anc[t]];
            const V3 s{zk.x * zk.w, zk.y * zk.w, zk.z * zk.w};
            if (kPrism && rk.w != 0.0f) {
                x.l = x.l + s;
            } else {
                x.a = x.a + s;
                x.l = x.l + cross(s, D);
            }
            D = D + V3{rk.x, rk.y, rk.z};
        }
        return x;
    };
    // y += S_i s
    const auto add_S = [&](Six y, float s) {
        if (kPrism && pr)
            return Six{y.a, y.l + z * s};
        return Six{y.a + z * s, y.l};
    };
    // x x S_i
    const auto cross_S = [&](Six x) {
        if (kPrism && pr)
            return Six{{0.0f, 0.0f, 0.0f}, cross(x.a, z)};
        return Six{cross(x.a, z), cross(x.l, z)};
    };

    Six vl{}, psd{}, al{};                             // v_lambda, psd, a_lambda (at this origin)
    if constexpr (kVel) {
        vl = path_sum();
        psd = cross_S(vl);
        fP0[me] = float4{psd.a.x, psd.a.y, psd.a.z, psd.l.x};
        fP1[me] = float4{psd.l.y, psd.l.z, 0.0f, 0.0f};
        if constexpr (!kBias)
            fQ1[me] = float4{ui, 0.0f, 0.0f, 0.0f};    // the given qdd
        wave_lds_sync();
        // a_lambda with qdd = 0 (dFD, FD) or the given qdd: a0 + sum of psd_k qd_k + S_k qdd_k
        al = Six{{0.0f, 0.0f, 0.0f}, a0};
        V3 D = r;
#pragma unroll
        for (int t = 0; t < MD; ++t) {
            const float4 zk = fZ[anc[t]], rk = fR[anc[t]], p0 = fP0[anc[t]], p1 = fP1[anc[t]];
            Six x{{p0.x * zk.w, p0.y * zk.w, p0.z * zk.w}, {p0.w * zk.w, p1.x * zk.w, p1.y * zk.w}};
            if constexpr (!kBias) {
                const float a = fQ1[anc[t]].x;
                const V3 s{zk.x * a, zk.y * a, zk.z * a};
                if (kPrism && rk.w != 0.0f)
                    x.l = x.l + s;
                else
                    x.a = x.a + s;
            }
            al = Six{al.a + x.a, al.l + x.l + cross(x.a, D)};
            D = D + V3{rk.x, rk.y, rk.z};
        }
    }

    // ------------------------------------------------------------ the body's own inertia
    Sym P = turn(R, PT);
    V3 h = mul(R, hT);
    const Sym P1 = P;                                  // the body alone (for the qdd increment)
    const V3 h1 = h;
    Mat K{};
    V3 l{};
    Six F{};
    if constexpr (kVel) {
        const Six v = add_S(vl, qd);
        l = v.l * m + cross(v.a, h);
        K = momentum_moment(v, h, P);
        Six a = Six{al.a + psd.a * qd, al.l + psd.l * qd};
        if constexpr (!kBias)
            a = add_S(a, ui);
        const Six Ia = inertia(m, h, second_to_inertia(P), a), Bv = bmul(K, l, v.a);
        F = Six{Ia.a + Bv.a, Ia.l + Bv.l};
    }

    // ------------------------------------------------------------ sums over subtrees
    // leaves to root, level by level; siblings take turns (their rank)
    constexpr int NF = kDer ? 7 : (kVel ? 4 : 3);      // float4 fields exchanged
#pragma unroll
    for (int lev = MD; lev >= 1; --lev) {
#pragma unroll
        for (int c = 0; c < T::max_children(lev); ++c) {
            if (depth == lev && rank == c) {
                Sym Q = P;
                V3 g = h;
                move_moments(Q, g, mC, r);
                float o[28] = {Q.xx, Q.yy, Q.zz, Q.xy, Q.xz, Q.yz, g.x, g.y, g.z};
                if constexpr (kVel) {
                    const V3 n = F.a + cross(r, F.l);
                    const float f[6] = {n.x, n.y, n.z, F.l.x, F.l.y, F.l.z};
#pragma unroll
                    for (int e = 0; e < 6; ++e)
                        o[9 + e] = f[e];
                }
                if constexpr (kDer) {
                    const V3 k0 = K.c0 + l * r.x, k1 = K.c1 + l * r.y, k2 = K.c2 + l * r.z;
                    const float f[12] = {k0.x, k0.y, k0.z, k1.x, k1.y, k1.z,
                                         k2.x, k2.y, k2.z, l.x,  l.y,  l.z};
#pragma unroll
                    for (int e = 0; e < 12; ++e)
                        o[15 + e] = f[e];
                }
#pragma unroll
                for (int e = 0; e < NF; ++e)
                    fU[e * NE + parent] = float4{o[4 * e], o[4 * e + 1], o[4 * e + 2], o[4 * e + 3]};
            }
            wave_lds_sync();
            if (depth == lev - 1 && nchild > c) {
                float o[28];
#pragma unroll
                for (int e = 0; e < NF; ++e) {
                    const float4 x = fU[e * NE + me];
                    o[4 * e] = x.x;
                    o[4 * e + 1] = x.y;
                    o[4 * e + 2] = x.z;
                    o[4 * e + 3] = x.w;
                }
                P = Sym{P.xx + o[0], P.yy + o[1], P.zz + o[2], P.xy + o[3], P.xz + o[4], P.yz + o[5]};
                h = h + V3{o[6], o[7], o[8]};
                if constexpr (kVel)
                    F = Six{F.a + V3{o[9], o[10], o[11]}, F.l + V3{o[12], o[13], o[14]}};
                if constexpr (kDer) {
                    K.c0 = K.c0 + V3{o[15], o[16], o[17]};
                    K.c1 = K.c1 + V3{o[18], o[19], o[20]};
                    K.c2 = K.c2 + V3{o[21], o[22], o[23]};
                    l = l + V3{o[24], o[25], o[26]};
                }
            }
            wave_lds_sync();
        }
    }

    // S_k . f for the body k beside z_k, and for this body
    const auto dot_S = [&](float4 zk, float4 rk, Six f) {
        const V3 zz{zk.x, zk.y, zk.z};
        return kPrism && rk.w != 0.0f ? dot(zz, f.l) : dot(zz, f.a);
    };
    const auto dot_me = [&](Six f) { return kPrism && pr ? dot(z, f.l) : dot(z, f.a); };

    // F1 = I^c S and M's row of this body
    const Sym J = second_to_inertia(P);
    const Six F1 = kPrism && pr ? Six{cross(h, z), z * mC} : Six{mul(J, z), cross(z, h)};
    float Lf[B][B], dinv[B];
    if constexpr (kMass) {
        float* row = sM + me * Y::RS;
        row[0] = dot_me(F1);
        V3 n = F1.a, s = r;
#pragma unroll
        for (int t = 0; t < MD; ++t) {
            n = n + cross(s, F1.l);
            const float4 zk = fZ[anc[t]], rk = fR[anc[t]];
            const float x = dot_S(zk, rk, Six{n, F1.l});
            if (t < depth)
                row[1 + t] = x;
            s = V3{rk.x, rk.y, rk.z};
        }
        if constexpr (kBias)
            sx[i] = ui - dot_me(F);                    // tau - c
        if constexpr (OP == kVjp)
            sx[i] = A.u2[vo];
        wave_lds_sync();
        // every lane factors its problem's M
#pragma unroll
        for (int k = 0; k < B; ++k) {
            float rowk[Y::RS];
#pragma unroll
            for (int e = 0; e < (T::depth(k) + 4) / 4; ++e) {
                const float4 x = reinterpret_cast<const float4*>(sM + (sb + k) * Y::RS)[e];
                rowk[4 * e] = x.x;
                rowk[4 * e + 1] = x.y;
                rowk[4 * e + 2] = x.z;
                rowk[4 * e + 3] = x.w;
            }
            Lf[k][k] = rowk[0];
#pragma unroll
            for (int t = 0; t < T::depth(k); ++t)
                Lf[k][T::anc_at(k, t)] = rowk[1 + t];
        }
        gridq::ltl_factor<S>(Lf, dinv);
    }

    // ------------------------------------------------------------ qdd, or taubar
    float xi = 0.0f;                                   // this joint's qdd (dFD, FD), taubar (VJP)
    if constexpr (OP != kMinv && OP != kIdGrad) {
        float x[BS];
#pragma unroll
        for (int e = 0; e < BS / 4; ++e) {
            const float4 y = reinterpret_cast<const float4*>(sx)[e];
            x[4 * e] = y.x;
            x[4 * e + 1] = y.y;
            x[4 * e + 2] = y.z;
            x[4 * e + 3] = y.w;
        }
        float xs[B];
#pragma unroll
        for (int k = 0; k < B; ++k)
            xs[k] = x[k];
        gridq::ltl_solve<S>(Lf, dinv, xs);
        wave_lds_sync();
        if (i == 0) {
#pragma unroll
            for (int k = 0; k < B; ++k)
                sx[k] = xs[k];
        }
        wave_lds_sync();
        xi = sx[i];
        if (valid)
            (OP == kVjp ? A.o2 : A.o0)[vo] = xi;
    }
    if constexpr (OP == kFd)
        return;

    if constexpr (OP == kFdGrad) {
        // the increment from qdd = 0 to qdd: Da_lambda, Df, summed over subtrees
        fZ[me] = float4{z.x, z.y, z.z, xi};
        wave_lds_sync();
        const Six da = path_sum();
        al = Six{al.a + da.a, al.l + da.l};
        Six f = inertia(m, h1, second_to_inertia(P1), add_S(da, xi));
#pragma unroll
        for (int lev = MD; lev >= 1; --lev) {
#pragma unroll
            for (int c = 0; c < T::max_children(lev); ++c) {
                if (depth == lev && rank == c) {
                    const V3 n = f.a + cross(r, f.l);
                    fU[parent] = float4{n.x, n.y, n.z, f.l.x};
                    fU[NE + parent] = float4{f.l.y, f.l.z, 0.0f, 0.0f};
                }
                wave_lds_sync();
                if (depth == lev - 1 && nchild > c) {
                    const float4 x = fU[me], y = fU[NE + me];
                    f = Six{f.a + V3{x.x, x.y, x.z}, f.l + V3{x.w, y.x, y.y}};
                }
                wave_lds_sync();
            }
        }
        F = Six{F.a + f.a, F.l + f.l};
    }

    // ------------------------------------------------------------ dtau/dq, dtau/dqd
    if constexpr (kDer) {
        Six pdd;
        {
            const Six x = cross_S(al);
            pdd = Six{x.a + cross(vl.a, psd.a), x.l + cross(vl.a, psd.l) + cross(vl.l, psd.a)};
        }
        fQ0[me] = float4{pdd.a.x, pdd.a.y, pdd.a.z, pdd.l.x};
        fQ1[me] = float4{pdd.l.y, pdd.l.z, 0.0f, 0.0f};
        if constexpr (!T::chain()) {                   // entries off the ancestor paths
            for (int e = lane; e < Y::cols / 4; e += 64)
                reinterpret_cast<float4*>(sT)[e] = float4{0.0f, 0.0f, 0.0f, 0.0f};
        }
        Six u, w;
        V3 b;
        {
            const Six Bp = bmul(K, l, psd.a), Ip = inertia(mC, h, J, pdd);
            const Six Sf = kPrism && pr ? Six{cross(z, F.l), {0.0f, 0.0f, 0.0f}}
                                        : Six{cross(z, F.a), cross(z, F.l)};
            u = Six{Bp.a * 2.0f + Ip.a + Sf.a, Bp.l * 2.0f + Ip.l + Sf.l};
            const Six Iq = inertia(mC, h, J, psd);
            if (kPrism && pr) {
                w = Six{Iq.a * 2.0f, Iq.l * 2.0f};
                b = cross(l, z);
            } else {
                const Six Bs = bmul(K, l, z);
                w = Six{(Bs.a + Iq.a) * 2.0f, (Bs.l + Iq.l) * 2.0f};
                b = z * (K.c0.x + K.c1.y + K.c2.z) - tmul(K, z);
            }
        }
        wave_lds_sync();
        float* const col = sT + me * BS;               // this body's column
        col[i] = dot_me(u);
        col[TQ + i] = dot_me(w);
        Six g = F1;
        V3 s = r;
        const V3 b2 = b * 2.0f;
#pragma unroll
        for (int t = 0; t < MD; ++t) {
            u.a = u.a + cross(s, u.l);
            w.a = w.a + cross(s, w.l);
            g.a = g.a + cross(s, g.l);
            const float4 zk = fZ[anc[t]], rk = fR[anc[t]], p0 = fP0[anc[t]], p1 = fP1[anc[t]],
                         q0 = fQ0[anc[t]], q1 = fQ1[anc[t]];
            const V3 pa{p0.x, p0.y, p0.z}, pl{p0.w, p1.x, p1.y};
            const V3 qa{q0.x, q0.y, q0.z}, ql{q0.w, q1.x, q1.y};
            const float bs = kPrism && rk.w != 0.0f ? 0.0f : dot(b, V3{zk.x, zk.y, zk.z});
            const float x0 = dot_S(zk, rk, u), x1 = dot_S(zk, rk, w);
            const float y0 = dot(b2, pa) + dot(g.a, qa) + dot(g.l, ql);
            const float y1 = 2.0f * (bs + dot(g.a, pa) + dot(g.l, pl));
            if (t < depth) {
                const int k = anc[t] - sb;
                col[k] = x0;
                col[TQ + k] = x1;
                float* const row = sT + anc[t] * BS + i;
                row[0] = y0;
                row[TQ] = y1;
            }
            s = V3{rk.x, rk.y, rk.z};
        }
        wave_lds_sync();
    }

    // ------------------------------------------------------------ columns, outputs
    float cq[B], cqd[B];                               // this joint's columns of dtau
    if constexpr (kDer) {
        const float* col = sT + me * BS;
        float x[BS], y[BS];
#pragma unroll
        for (int e = 0; e < BS / 4; ++e) {
            const float4 a = reinterpret_cast<const float4*>(col)[e];
            const float4 c = reinterpret_cast<const float4*>(col + TQ)[e];
            x[4 * e] = a.x;
            x[4 * e + 1] = a.y;
            x[4 * e + 2] = a.z;
            x[4 * e + 3] = a.w;
            y[4 * e] = c.x;
            y[4 * e + 1] = c.y;
            y[4 * e + 2] = c.z;
            y[4 * e + 3] = c.w;
        }
#pragma unroll
        for (int k = 0; k < B; ++k) {
            cq[k] = x[k];
            cqd[k] = y[k];
        }
    }
    if constexpr (OP == kVjp) {
        // qbar = -(dtau/dq)^T taubar, qdbar = -(dtau/dqd)^T taubar
        float s0 = 0.0f, s1 = 0.0f;
#pragma unroll
        for (int k = 0; k < B; ++k) {
            const float w = sx[k];
            s0 += cq[k] * w;
            s1 += cqd[k] * w;
        }
        if (valid) {
            A.o0[vo] = -s0;
            A.o1[vo] = -s1;
        }
        return;
    }
    wave_lds_sync();                                   // everything in LDS has been read
    // where entry (row k, this lane's column) of a tile goes
    constexpr int TS = Y::tile;
    float* tl = pool + (Y::FULL ? ks * N * N : slot * B * B);
    constexpr int LD = Y::FULL ? N : B;
    const int cj = Y::FULL ? body : i;
    int rows[B];
#pragma unroll
    for (int k = 0; k < B; ++k)
        rows[k] = (Y::FULL && NB > 1) ? G::rowmap()[br * B + k] : k;
    if constexpr (Y::FULL && NB > 1) {                 // zeros between branches
        constexpr int NM = OP == kFdGrad ? 3 : (OP == kIdGrad ? 2 : 1);
        for (int e = lane; e < NM * TS / 4; e += 64)
            reinterpret_cast<float4*>(pool)[e] = float4{0.0f, 0.0f, 0.0f, 0.0f};
        wave_lds_sync();
    }
    if constexpr (OP == kIdGrad) {
#pragma unroll
        for (int k = 0; k < B; ++k) {
            tl[rows[k] * LD + cj] = cq[k];
            tl[TS + rows[k] * LD + cj] = cqd[k];
        }
        wave_lds_sync();
        flush_tiles<G, 2>(pool, A.o0, A.o1, nullptr, block, nv, lane);
        return;
    }
    if constexpr (kMass) {
        float mc[B];
#pragma unroll
        for (int k = 0; k < B; ++k)
            mc[k] = (k == i) ? 1.0f : 0.0f;
        gridq::ltl_solve<S>(Lf, dinv, mc);
        // entries (k, i), k <= i, to both mirrored positions: exactly symmetric
#pragma unroll
        for (int k = 0; k < B; ++k) {
            if (k <= i) {
                tl[rows[k] * LD + cj] = mc[k];
                tl[cj * LD + rows[k]] = mc[k];
            }
        }
    }
    if constexpr (OP == kMinv) {
        wave_lds_sync();
        flush_tiles<G, 1>(pool, A.o0, nullptr, nullptr, block, nv, lane);
        return;
    }
    if constexpr (OP == kFdGrad) {
        gridq::ltl_solve<S>(Lf, dinv, cq);
#pragma unroll
        for (int k = 0; k < B; ++k)
            tl[TS + rows[k] * LD + cj] = -cq[k];
        gridq::ltl_solve<S>(Lf, dinv, cqd);
#pragma unroll
        for (int k = 0; k < B; ++k)
            tl[2 * TS + rows[k] * LD + cj] = -cqd[k];
        wave_lds_sync();
        flush_tiles<G, 3>(pool, A.o1, A.o2, A.o3, block, nv, lane);
    }
}

}  // namespace gridt

// kernels of a one-robot module (a module of several robots defines GRID_PIPE_ONLY and its
// own entry point, grid_fdgrad_pipe_mixed)
#ifndef GRID_PIPE_ONLY

// defined by the generated epilogue: workgroup -> (group of branches, knots)
template <int OP>
__device__ void grid_dispatch_t(const gridv::BatchArgs& args, int block);

extern "C" __global__ void __launch_bounds__(64) grid_fdgrad_team(grid::Args args)
{
    const gridv::BatchArgs a{args.nknots, args.q, args.qd, args.tau, nullptr,
                        args.qdd, args.Minv, args.dqdd_dq, args.dqdd_dqd};
    grid_dispatch_t<gridt::kFdGrad>(a, (int)blockIdx.x);
}

extern "C" __global__ void __launch_bounds__(64) grid_team_fd(gridq::OpArgs x)
{
    const gridv::BatchArgs a{x.nknots, x.q, x.qd, x.u, nullptr, x.out0, nullptr, nullptr, nullptr};
    grid_dispatch_t<gridt::kFd>(a, (int)blockIdx.x);
}

extern "C" __global__ void __launch_bounds__(64) grid_team_minv(gridq::OpArgs x)
{
    const gridv::BatchArgs a{x.nknots, x.q, nullptr, nullptr, nullptr, x.out0, nullptr, nullptr, nullptr};
    grid_dispatch_t<gridt::kMinv>(a, (int)blockIdx.x);
}

extern "C" __global__ void __launch_bounds__(64) grid_team_idgrad(gridq::OpArgs x)
{
    const gridv::BatchArgs a{x.nknots, x.q, x.qd, x.u, nullptr, x.out0, x.out1, nullptr, nullptr};
    grid_dispatch_t<gridt::kIdGrad>(a, (int)blockIdx.x);
}

extern "C" __global__ void __launch_bounds__(64) grid_team_vjp(gridq::OpArgs x)
{
    const gridv::BatchArgs a{x.nknots, x.q, x.qd, x.u, x.u2, x.out0, x.out1, x.out2, nullptr};
    grid_dispatch_t<gridt::kVjp>(a, (int)blockIdx.x);
}

#endif  // GRID_PIPE_ONLY
