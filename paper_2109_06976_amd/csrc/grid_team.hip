// One lane per body (gfx950): grid_fdgrad_team and the batch forms of FD, M^-1, dID and the
// adjoint VJP.
//
// A problem is one (knot, base branch). Its B bodies sit on B adjacent lanes of a wavefront, so
// a wavefront holds as many knots as fit, with all branches of one shape side by side
// (Group<g>: NB branches of shape S). Each lane keeps its own body's quantities in registers
// and meets the others through LDS; a workgroup is one wavefront, so no barrier is needed.
//
// The formulation is that of grid_axes.hip. M^-1 comes from M = L^T D L (sparse along ancestor
// paths), which every lane of a problem factors for itself from the rows of M in LDS: 57 (7-body chain) to 324 (18-body tree) FMAs in
// registers against one LDS round trip per level for a shared factor. Lane j then solves for
// column j of M^-1, dqdd/dq and dqdd/dqd.
//
// Bound by the latency of its chain of LDS exchanges up to a few wavefronts per SIMD, by VALU
// issue beyond. humanoid30: 236 us per launch at 4096 knots and 648 at 16384 on the kernels it
// took the place of, 24.2 and 69.0 here (74.6 and 83.6 at 16384 where a run's outputs do not stay
// in the caches); chain7 at 4096 knots 11.4 and 9.0, quad12 7.8 and 6.6.
// FD / M^-1 / dID / VJP against the quad layout's (grid_ops.hip): humanoid30 at 4096 knots 46 /
// 31 / 192 / 68 and 10.3 / 10.8 / 15.6 / 16.1 us, at 128 9.8 / 9.7 / 11.3 / 14.1 and 7.4 / 6.9 / 9.2 /
// 10.5; chain7 dID at 8192 8.4 and 7.9. (Where a comment below gives figures of an alternative, both
// sides are of this kernel with the rows of M in float32, 3 to 5% faster.)


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
    static constexpr int children(int p)
    {
        int c = 0;
        for (int i = p + 1; i < S::B; ++i)
            c += S::parent[i] == p ? 1 : 0;
        return c;
    }
    // Segments: a body with one child shares its child's. The tier of a segment is 0 without
    // branches below it, else one more than the highest tier among those.
    static constexpr int end_of(int i)
    {
        for (int k = i + 1; k < S::B; ++k)
            if (S::parent[k] == i && children(i) == 1)
                i = k;
        return i;
    }
    static constexpr int tier(int i)
    {
        const int e = end_of(i);
        int t = 0;
        for (int k = e + 1; k < S::B; ++k) {
            if (S::parent[k] == e) {
                const int x = tier(k) + 1;
                t = x > t ? x : t;
            }
        }
        return t;
    }
    static constexpr int tiers()
    {
        return tier(0) + 1;
    }
    // bodies in the longest segment of a tier
    static constexpr int longest(int tr)
    {
        int m = 0;
        for (int i = 0; i < S::B; ++i) {
            const bool head = S::parent[i] < 0 || children(S::parent[i]) != 1;
            if (head && tier(i) == tr) {
                const int n = depth(end_of(i)) - depth(i) + 1;
                m = n > m ? n : m;
            }
        }
        return m;
    }
    // most segments that hang from one body
    static constexpr int most_hanging()
    {
        int m = 0;
        for (int i = 0; i < S::B; ++i)
            m = children(i) > 1 && children(i) > m ? children(i) : m;
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
    static constexpr int GB = NB * B;                  // the group's rows of a knot's matrix
    static constexpr bool FULL = GB == N;              // the group is the whole robot
    // floats: six fields of a float4 per body (z and a scalar, r, psd, pdd), a vector per
    // problem, then one region that the level exchange (seven fields), M and the columns of
    // dtau use in turn; the output tiles take the place of everything at the end: all three
    // where they fit, else one after the other
    static constexpr int oX = 6 * 4 * NE;
    static constexpr int oU = oX + up4(SL * BS);
    static constexpr int exch = 7 * 4 * NE;
    static constexpr int rows = SL * B * RS;
    static constexpr int cols = 2 * SL * B * BS;
    static constexpr int tile = up4(KPB * GB * N);
    static constexpr int mx(int a, int b) { return a > b ? a : b; }
    static constexpr int base = oU + mx(mx(exch, rows), cols);
    static constexpr int NT = 3 * tile <= base ? 3 : 1;
    static constexpr int floats = mx(base, NT * tile);
    // floats that a flushed piece holds: no piece crosses the end of a run of adjacent rows
    static constexpr int piece()
    {
        int w = GB * N % 4 == 0 ? 4 : (GB * N % 2 == 0 ? 2 : 1);
        for (int k = 0; k < G::NR; ++k)
            while (G::run_row[k] * N % w != 0)
                w /= 2;
        return w;
    }
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

// rows of other groups before row `row` of the group's (its place in the robot, less `row`)
template <class G>
__device__ __forceinline__ int rows_before(int row)
{
    int n = 0;
#pragma unroll
    for (int r = 0; r < G::NR; ++r)
        n += row >= G::run_row[r] ? G::run_gap[r] : 0;
    return n;
}

// a matrix's tile ([knot][the group's rows in the robot's order][N]) to global memory, in pieces
// of up to four floats whatever the rows (row by row, with a lane per float, it took three to
// four times the instructions: humanoid30 at 16384 knots 82.5 us a launch, 79.2 so)
template <class G>
__device__ __forceinline__ void flush_tile(float* d, const float* tile, int block, int nv, int lane)
{
    using Y = Lay<G>;
    constexpr int N = Y::N;
    d += (long)block * Y::KPB * N * N;
    if constexpr (Y::FULL) {
        flush_block(d, tile, nv * N * N, lane);
    } else {
        constexpr int W = Y::piece(), PK = Y::GB * N / W, STEPS = (Y::KPB * PK + 63) / 64;
#pragma unroll
        for (int k = 0; k < STEPS; ++k) {
            const int e = k * 64 + lane;
            const int ks = e / PK, p = (e - ks * PK) * W;
            const int off = ks * N * N + p + rows_before<G>(p / N) * N;
            if (e < nv * PK) {
                float x[W];
                if constexpr (W == 4) {
                    const float4 v = reinterpret_cast<const float4*>(tile)[e];
                    x[0] = v.x;
                    x[1] = v.y;
                    x[2] = v.z;
                    x[3] = v.w;
                } else {
#pragma unroll
                    for (int w = 0; w < W; ++w)
                        x[w] = tile[e * W + w];
                }
                store<W>(d + off, x);
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
    constexpr int MK = T::most_hanging();
    constexpr int DZ = NE - 1;                         // the entry of zeros
    constexpr bool kVel = OP != kMinv;
    constexpr bool kMass = OP != kIdGrad;
    constexpr bool kFdDer = OP == kFdGrad || OP == kFdGradQ || OP == kFdGradV;
    constexpr bool kBias = OP == kFdGrad || OP == kFdGradQ || OP == kFd;
    constexpr bool kDer = kFdDer || OP == kIdGrad || OP == kVjp;
    constexpr bool kQ = OP != kFdGradV, kV = OP != kFdGradQ;   // dq's matrix is wanted, dqd's
    constexpr bool kForce = kVel && kQ;
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
    const int body = ti.x, depth = ti.y;
    // place in its segment from the top, bodies below it there, the segment's tier, and for a
    // segment's first body the tier of the segment that it hangs from
    const int pos = ti.z & 255, rem = (ti.z >> 8) & 255, tier = (ti.z >> 16) & 255,
              above = (ti.z >> 24) & 255;
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
    int hang[MK > 0 ? MK : 1];                         // entries of the segments that hang here
#pragma unroll
    for (int c = 0; c < MK; ++c) {
        const int k = G::hanging()[(br * B + i) * MK + c];
        hang[c] = k < 0 ? DZ : sb + k;
    }
    const float4* tf = reinterpret_cast<const float4*>(G::table()) + (br * B + i) * 6;
    const float4 t0 = tf[0], t1 = tf[1], t2 = tf[2], t3 = tf[3], t4 = tf[4], t5 = tf[5];
    const V3 rT{t2.y, t2.z, t2.w};
    const Sym JT{t3.x, t3.y, t3.z, t3.w, t4.x, t4.y};
    const float half = 0.5f * (JT.xx + JT.yy + JT.zz);   // for the second moment
    const V3 hT{t4.z, t4.w, t5.x};
    const float m = t5.y, mC = t5.z;
    const bool pr = kPrism && t5.w != 0.0f;

    Mat R = joint_axes(pr, qi, V3{t0.x, t0.y, t0.z}, V3{t0.w, t1.x, t1.y}, V3{t1.z, t1.w, t2.x});
    V3 rb = tmul(R, rT);                               // r in body axes
    if (kPrism && pr)
        rb.z += qi;
    V3 a0 = {0.0f, 0.0f, 0.0f};                        // -g along the first body's axes
    if constexpr (kVel) {
        a0 = tmul(R, V3{G::a0()[0], G::a0()[1], G::a0()[2]});
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
    {                                                  // orthonormal again
        const auto unit = [](V3 v) {
            const float d = __builtin_fmaf(v.x, v.x, __builtin_fmaf(v.y, v.y, __builtin_fmaf(v.z, v.z, -1.0f)));
            return v * (1.0f - 0.5f * d);
        };
        R.c2 = unit(R.c2);
        R.c0 = unit(R.c0 - R.c2 * dot(R.c0, R.c2));
        R.c1 = cross(R.c2, R.c0);
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

    // from the ancestor at distance 1, 2, 4, .. to this body
    V3 ds[5];
    {
        V3 D = r;
#pragma unroll
        for (int t = 0; t < MD; ++t) {
            if (t == 0 || t == 1 || t == 3 || t == 7 || t == 15)
                ds[t == 0 ? 0 : t == 1 ? 1 : t == 3 ? 2 : t == 7 ? 3 : 4] = D;
            const float4 rk = fR[anc[t]];
            D = D + V3{rk.x, rk.y, rk.z};
        }
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
        if constexpr (!kBias && kForce)
            fQ1[me] = float4{ui, 0.0f, 0.0f, 0.0f};    // the given qdd
        wave_lds_sync();
    }
    if constexpr (kForce) {
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
    Sym J = turn(R, JT);
    V3 h = mul(R, hT);
    const Six self{mul(R, V3{JT.xz, JT.yz, JT.zz}), mul(R, V3{-hT.y, hT.x, 0.0f})};
    const Sym J1 = J;                                  // the body alone (for the qdd increment)
    const V3 h1 = h;
    Mat K{};
    V3 l{};
    Six F{};
    if constexpr (kVel) {
        const Six v = add_S(vl, qd);
        l = v.l * m + cross(v.a, h);
        K = momentum_moment(v, h, second_moment(J, half));
    }
    if constexpr (kForce) {
        const Six v = add_S(vl, qd);
        Six a = Six{al.a + psd.a * qd, al.l + psd.l * qd};
        if constexpr (!kBias)
            a = add_S(a, ui);
        const Six Ia = inertia(m, h, J, a), Bv = bmul(K, l, v.a);
        F = Six{Ia.a + Bv.a, Ia.l + Bv.l};
    }

    // ------------------------------------------------------------ sums over subtrees
    // Within the segments of a tier by doubling: after the step of distance s a body holds the
    // sum over 2 s bodies from it on, about its own origin. Then a segment's last body takes
    // the sums of those that hang from it. `put` writes a body's fields, moved up by d, and
    // `add` takes them. Level by level, one body of each chain at work, it took as many
    // exchanges as the tree is deep, and one more for every further sibling: humanoid30 at 4096
    // and 16384 knots 27.2 and 79.2 us a launch, 24.0 and 70.0 so; chain7 at 16384 14.7 and 12.9.
    const auto sum_up = [&](auto nf, const auto& put, const auto& add) {
        constexpr int NF = decltype(nf)::v;            // float4 fields exchanged
        const auto send = [&](int to, V3 d) {
            float o[4 * NF];
            put(o, d);
#pragma unroll
            for (int e = 0; e < NF; ++e)
                fU[e * NE + to] = float4{o[4 * e], o[4 * e + 1], o[4 * e + 2], o[4 * e + 3]};
        };
        const auto receive = [&](int from) {
            float o[4 * NF];
#pragma unroll
            for (int e = 0; e < NF; ++e) {
                const float4 x = fU[e * NE + from];
                o[4 * e] = x.x;
                o[4 * e + 1] = x.y;
                o[4 * e + 2] = x.z;
                o[4 * e + 3] = x.w;
            }
            add(o);
        };
        grids::static_for<T::tiers()>([&](auto tt) {
            constexpr int tr = decltype(tt)::v, len = T::longest(tr);
            if constexpr (tr > 0) {
                if (above == tr)
                    send(me, r);
                wave_lds_sync();
                if (tier == tr) {
#pragma unroll
                    for (int c = 0; c < MK; ++c)
                        if (hang[c] != DZ)
                            receive(hang[c]);
                }
                wave_lds_sync();
            }
            grids::static_for<5>([&](auto kk) {
                constexpr int k = decltype(kk)::v, s = 1 << k;
                if constexpr (s < len) {
                    if (tier == tr && pos >= s)
                        send(anc[s - 1], ds[k]);
                    wave_lds_sync();
                    if (tier == tr && rem >= s)
                        receive(me);
                    wave_lds_sync();
                }
            });
        });
    };
    constexpr int NF = kDer ? (kForce ? 7 : 6) : (kForce ? 4 : 3);
    constexpr int KO = kForce ? 16 : 10;               // where K and l begin
    float ms = m;                                      // the mass that J and h stand for
    sum_up(
        grids::Int<NF>{},
        [&](float (&o)[4 * NF], V3 d) {
            Sym Q = J;
            V3 g = h;
            move_inertia(Q, g, ms, d);
            const float f[10] = {Q.xx, Q.yy, Q.zz, Q.xy, Q.xz, Q.yz, g.x, g.y, g.z, ms};
#pragma unroll
            for (int e = 0; e < 10; ++e)
                o[e] = f[e];
            if constexpr (kForce) {
                const V3 n = F.a + cross(d, F.l);
                const float y[6] = {n.x, n.y, n.z, F.l.x, F.l.y, F.l.z};
#pragma unroll
                for (int e = 0; e < 6; ++e)
                    o[10 + e] = y[e];
            }
            if constexpr (kDer) {
                const V3 k0 = K.c0 + l * d.x, k1 = K.c1 + l * d.y, k2 = K.c2 + l * d.z;
                const float y[12] = {k0.x, k0.y, k0.z, k1.x, k1.y, k1.z,
                                     k2.x, k2.y, k2.z, l.x,  l.y,  l.z};
#pragma unroll
                for (int e = 0; e < 12; ++e)
                    o[KO + e] = y[e];
            }
#pragma unroll
            for (int e = kDer ? KO + 12 : (kForce ? 16 : 10); e < 4 * NF; ++e)
                o[e] = 0.0f;
        },
        [&](const float (&o)[4 * NF]) {
            J = J + Sym{o[0], o[1], o[2], o[3], o[4], o[5]};
            h = h + V3{o[6], o[7], o[8]};
            ms += o[9];
            if constexpr (kForce)
                F = Six{F.a + V3{o[10], o[11], o[12]}, F.l + V3{o[13], o[14], o[15]}};
            if constexpr (kDer) {
                K.c0 = K.c0 + V3{o[KO], o[KO + 1], o[KO + 2]};
                K.c1 = K.c1 + V3{o[KO + 3], o[KO + 4], o[KO + 5]};
                K.c2 = K.c2 + V3{o[KO + 6], o[KO + 7], o[KO + 8]};
                l = l + V3{o[KO + 9], o[KO + 10], o[KO + 11]};
            }
        });

    // S_k . f for the body k beside z_k, and for this body
    const auto dot_S = [&](float4 zk, float4 rk, Six f) {
        const V3 zz{zk.x, zk.y, zk.z};
        return kPrism && rk.w != 0.0f ? dot(zz, f.l) : dot(zz, f.a);
    };
    const auto dot_me = [&](Six f) { return kPrism && pr ? dot(z, f.l) : dot(z, f.a); };

    // F1 = I^c S and M's row of this body
    const Six F1 = kPrism && pr ? Six{cross(h, z), z * mC} : Six{mul(J, z), cross(z, h)};
    float Lf[B][B], dinv[B];
    if constexpr (kMass) {
        float* row = sM + me * Y::RS;
        // in double; the body's own part of M_ii is a constant, of the others a turned one
        const V3D zd = wide(z), below = mul(J - J1, zd);
        V3D n = below + wide(self.a), fl = cross(zd, wide(h - h1)) + wide(self.l);
        if (kPrism && pr) {
            n = cross(wide(h), zd);
            fl = zd * mC;
        }
        row[0] = kPrism && pr ? mC : (float)(JT.zz + dot(zd, below));
        V3 s = r;
#pragma unroll
        for (int t = 0; t < MD; ++t) {
            n = n + cross(wide(s), fl);
            const float4 zk = fZ[anc[t]], rk = fR[anc[t]];
            const float x = (float)dot(V3D{zk.x, zk.y, zk.z}, kPrism && rk.w != 0.0f ? fl : n);
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
        ltdl_factor<S>(Lf, dinv);
    }

    // ------------------------------------------------------------ qdd, or taubar
    float xi = 0.0f;                                   // this joint's qdd (dFD, FD), taubar (VJP)
    if constexpr (kBias || OP == kVjp) {
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
        ltdl_solve<S>(Lf, dinv, xs);
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

    if constexpr (kBias) {
        // the increment from qdd = 0 to qdd: Da_lambda, Df, summed over subtrees
        fZ[me] = float4{z.x, z.y, z.z, xi};
        wave_lds_sync();
        const Six da = path_sum();
        al = Six{al.a + da.a, al.l + da.l};
        Six f = inertia(m, h1, J1, add_S(da, xi));
        sum_up(
            grids::Int<2>{},
            [&](float (&o)[8], V3 d) {
                const V3 n = f.a + cross(d, f.l);
                const float y[8] = {n.x, n.y, n.z, f.l.x, f.l.y, f.l.z, 0.0f, 0.0f};
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    o[e] = y[e];
            },
            [&](const float (&o)[8]) {
                f = Six{f.a + V3{o[0], o[1], o[2]}, f.l + V3{o[3], o[4], o[5]}};
            });
        F = Six{F.a + f.a, F.l + f.l};
    }

    // ------------------------------------------------------------ dtau/dq, dtau/dqd
    if constexpr (kDer) {
        Six pdd{};
        if constexpr (kQ) {
            const Six x = cross_S(al);
            pdd = Six{x.a + cross(vl.a, psd.a), x.l + cross(vl.a, psd.l) + cross(vl.l, psd.a)};
        }
        if constexpr (kQ) {
            fQ0[me] = float4{pdd.a.x, pdd.a.y, pdd.a.z, pdd.l.x};
            fQ1[me] = float4{pdd.l.y, pdd.l.z, 0.0f, 0.0f};
        }
        if constexpr (!T::chain()) {                   // entries off the ancestor paths
            wave_lds_sync();                           // M's rows, in the same place, have been read
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
        if constexpr (kQ)
            col[i] = dot_me(u);
        if constexpr (kV)
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
                float* const row = sT + anc[t] * BS + i;
                if constexpr (kQ) {
                    col[k] = x0;
                    row[0] = y0;
                }
                if constexpr (kV) {
                    col[TQ + k] = x1;
                    row[TQ] = y1;
                }
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
    constexpr int TS = Y::NT == 3 ? Y::tile : 0;
    float* const tl = pool + ks * Y::GB * N;
    int rows[B];
#pragma unroll
    for (int k = 0; k < B; ++k)
        rows[k] = (NB == 1 || G::in_order) ? br * B + k : G::rowmap()[br * B + k];
    int own = br * B + i;
    if constexpr (NB > 1 && !G::in_order)
        own = G::rowmap()[own];
    constexpr int NM = OP == kFdGrad ? 3 : (OP == kIdGrad || OP == kFdGradV ? 2 : 1);
    if constexpr (B < N) {                             // zeros in the other branches' columns
        for (int e = lane; e < (Y::NT == 3 ? NM : 1) * Y::tile / 4; e += 64)
            reinterpret_cast<float4*>(pool)[e] = float4{0.0f, 0.0f, 0.0f, 0.0f};
        wave_lds_sync();
    }
    float* const dst[3] = {OP == kFdGradQ ? A.o2 : (kFdDer ? A.o1 : A.o0),
                           OP == kFdGrad ? A.o2 : (OP == kFdGradV ? A.o3 : A.o1), A.o3};
    // matrix `mat` is in its tile
    const auto tile_done = [&](int mat) {
        if constexpr (Y::NT == 3) {
            if (mat == NM - 1) {
                wave_lds_sync();
#pragma unroll
                for (int k = 0; k < NM; ++k)
                    flush_tile<G>(dst[k], pool + k * TS, block, nv, lane);
            }
        } else {
            wave_lds_sync();
            flush_tile<G>(dst[mat], pool, block, nv, lane);
            wave_lds_sync();
        }
    };
    const auto put_column = [&](int mat, const float (&x)[B], float sign) {
#pragma unroll
        for (int k = 0; k < B; ++k)
            tl[mat * TS + rows[k] * N + body] = sign * x[k];
        tile_done(mat);
    };
    if constexpr (OP == kIdGrad) {
        put_column(0, cq, 1.0f);
        put_column(1, cqd, 1.0f);
        return;
    }
    if constexpr (kMass && kV) {
        float mc[B];
#pragma unroll
        for (int k = 0; k < B; ++k)
            mc[k] = (k == i) ? 1.0f : 0.0f;
        ltdl_solve<S>(Lf, dinv, mc);
        // entries (k, i), k <= i, to both mirrored positions: exactly symmetric
#pragma unroll
        for (int k = 0; k < B; ++k) {
            if (k <= i) {
                tl[rows[k] * N + body] = mc[k];
                tl[own * N + rows[k] + rows_before<G>(rows[k])] = mc[k];
            }
        }
        tile_done(0);
    }
    if constexpr (kFdDer && kQ) {
        ltdl_solve<S>(Lf, dinv, cq);
        put_column(kV ? 1 : 0, cq, -1.0f);
    }
    if constexpr (kFdDer && kV) {
        ltdl_solve<S>(Lf, dinv, cqd);
        put_column(kQ ? 2 : 1, cqd, -1.0f);
    }
}

}  // namespace gridt

// defined by the generated epilogue: workgroup -> (group of branches, knots)
template <int OP>
__device__ void grid_dispatch_t(const gridv::BatchArgs& args, int block);

#ifdef GRID_PIPE_ONLY

// dFD lives in the module with the three-role kernel, compiled for instruction-level parallelism:
// humanoid30 at 128, 4096 and 16384 knots 11.4 / 24.1 / 70.2 us by the default schedule, 11.2 / 23.5
// / 69.1 by that; chain7 at 1024 and 16384 7.6 / 12.9 and 7.2 / 12.7. dID has fewer wavefronts per
// SIMD by it (humanoid30 at 4096 knots 15.2 and 18.3) and stays with the other algorithms
extern "C" __global__ void __launch_bounds__(64) grid_fdgrad_team(grid::Args args)
{
    const gridv::BatchArgs a{args.nknots, args.q, args.qd, args.tau, nullptr,
                        args.qdd, args.Minv, args.dqdd_dq, args.dqdd_dqd};
    grid_dispatch_t<gridt::kFdGrad>(a, (int)blockIdx.x);
}

// dFD by two wavefronts: qdd and dqdd/dq; M^-1 and dqdd/dqd, which needs neither accelerations nor
// forces. humanoid30 at 128, 1024, 1536 and 2048 knots 14.5 / 16.4 / 17.0 / 18.0 us by one, 11.8 /
// 14.2 / 16.1 / 18.1 by two; chain7 at 1024 and 4096 8.9 / 9.5 and 7.85 / 9.0, at 8192 and 16384
// 10.4 / 13.7 and 10.7 / 14.0

#if GRID_LANE_PER_BODY
extern "C" __global__ void __launch_bounds__(64) grid_fdgrad_team_halves(grid::Args args)
{
    const gridv::BatchArgs a{args.nknots, args.q, args.qd, args.tau, nullptr,
                        args.qdd, args.Minv, args.dqdd_dq, args.dqdd_dqd};
    const int half = (int)gridDim.x / 2, b = (int)blockIdx.x;
    if (b < half)
        grid_dispatch_t<gridv::kFdGradQ>(a, b);
    else
        grid_dispatch_t<gridv::kFdGradV>(a, b - half);
}
#endif

#else

// (reached by robots with a branch of more than 8 bodies)
#if GRID_LONG_BRANCH

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

#endif  // GRID_LONG_BRANCH
#if GRID_LANE_PER_BODY

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

#endif  // GRID_LANE_PER_BODY

#endif  // GRID_PIPE_ONLY
