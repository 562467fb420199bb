// Backward pass on MFMA (bf16 storage, d = dv in {64, 128}, p in {4, 8}, r in {32, 64}, b % 256 == 0).
// Included inside the anonymous namespace of psf_mfma.hip, after the forward kernels it reuses.
//
// Gradient of the forward function of Sections 3, 3.1, 3.2 (the paper prints no formula; this is
// the chain rule through the definition).  With C_j = [v_j | 1], row_i = sum_j w_ij C_j,
// D_i = 1 + row_i[dv], o_i = row_i[0:dv] / D_i:
//     g_i = dO_i / D_i,  c_i = -<dO_i, o_i> / D_i,  dw_ij = <g_i, v_j> + c_i,  dV_j = sum_i w_ij g_i
// pairs inside a block:  w = <q, k>^p,        dq_i += sum_j dw_ij p <q_i, k_j>^(p-1) k_j   (dk alike)
// pairs across blocks:   w = <m(q), m(k)>^2,  dm(q_i) = 2 sum_j dw_ij <m(q_i), m(k_j)> m(k_j) (dm(k) alike)
// The cross-block sums are linear-time through the prefix states Z_l of Section 3.1 and their
// mirror R_l = sum over later blocks of phi'(q_i) [g_i | c_i]^T:
//     dm(q_i)[e] = 2 sum_{b,c} Z_l[e,b,c] m(q_i)[b] g_i[c]  +  2 c_i (S_l m(q_i))[e]
//     dm(k_j)[e] = 2 sum_{b,c} R_l[e,b,c] m(k_j)[b] v_j[c]  +  2 (Rc_l m(k_j))[e]
//     dV_j      +=   phi'(k_j)^T R_l            (the forward cross-block product with R in place of Z)
// where S_l / Rc_l are the ones-column parts of the states.  Finally dq_i += J_m(q_i)^T dm(q_i)
// through Algorithm 1 (p = 4: m = sqrt(1/r) (x G1) * (x G2), inside k_bwd_dm at d = 64; d = 128 and
// p = 8 (one more level of the recursion): k_bwd_sketch_rows).

template <int E>
__device__ __forceinline__ float pow_n(float x)
{
    float r = x;
#pragma unroll
    for (int e = 1; e < E; ++e) r *= x;
    return r;
}

// ---- g, c and the layouts of g ------------------------------------------------------------
// A group of D / 8 lanes per row, eight columns a lane.  G_rm: g as bf16 rows; Cc: c as fp32.
template <int D>
__global__ __launch_bounds__(kWg) void k_bwd_prep(const bf16_t *__restrict__ dO, const bf16_t *__restrict__ O,
                                                  const float *__restrict__ Den, bf16_t *__restrict__ G_rm,
                                                  float *__restrict__ Cc)
{
    constexpr int LANES = D / 8, ROWS = kWg / LANES, U = 4;    // rows a pass; passes, all their loads first
    const int li = threadIdx.x % LANES;
    const size_t row0 = (size_t)blockIdx.x * (ROWS * U) + threadIdx.x / LANES;
    bf16x8 d_o[U], o[U];
    float inv[U];
#pragma unroll
    for (int i = 0; i < U; ++i) {
        const size_t row = row0 + (size_t)i * ROWS;
        d_o[i] = *(const bf16x8 *)&dO[row * D + 8 * li];
        o[i] = *(const bf16x8 *)&O[row * D + 8 * li];
        inv[i] = Den[row];
    }
#pragma unroll
    for (int i = 0; i < U; ++i) {
        const size_t row = row0 + (size_t)i * ROWS;
        inv[i] = 1.0f / inv[i];
        f32x8 g;
        float dot = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            g[e] = (float)d_o[i][e] * inv[i];
            dot += (float)d_o[i][e] * (float)o[i][e] * inv[i];
        }
        *(bf16x8 *)&G_rm[row * D + 8 * li] = cvt8(g);
#pragma unroll
        for (int m = LANES / 2; m >= 1; m >>= 1) dot += __shfl_xor(dot, m);
        if (li == 0) Cc[row] = -dot;
    }
}

// ---- m(Q) octets in reverse block order and the c-weighted partial sums --------------------
// Workgroup = 256 tokens: M8r [rows/8][2][R][4] fp32 (reverse block order) and
// Sc = sum_i c_i m_i m_i^T (R x R fp32) at the part's reverse-order position.
template <int R>
__global__ __launch_bounds__(kWg) void k_bwd_qoct(const bf16_t *__restrict__ MQ, const float *__restrict__ Cc,
                                                  float *__restrict__ M8r, float *__restrict__ ScPart, int n,
                                                  int b, int t)
{
    constexpr int OT = R / 32;
    __shared__ float red[4][32][33];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, x = lane & 31, h = lane >> 5;
    const size_t row0 = (size_t)blockIdx.x * 256;
    const size_t u = row0 / n, pos0 = row0 % n;
    const size_t rrow0 = u * n + (size_t)(t - 1 - (int)(pos0 / b)) * b + pos0 % b;
    f32x16 sacc[OT][OT];
#pragma unroll
    for (int i = 0; i < OT; ++i)
#pragma unroll
        for (int j = 0; j < OT; ++j) sacc[i][j] = f32x16{0};
#pragma unroll
    for (int tt = 0; tt < 2; ++tt) {
        const size_t tile0 = row0 + wave * 64 + 32 * tt, rtile0 = rrow0 + wave * 64 + 32 * tt;
        // lane = sketch column 32 ot + x, register v = token 8 (v / 4) + 4 h + v % 4
        f32x16 m[OT], mw[OT];
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const size_t tok = tile0 + 8 * (v / 4) + 4 * h + (v % 4);
            const float cw = Cc[tok];
#pragma unroll
            for (int ot = 0; ot < OT; ++ot) {
                m[ot][v] = bf16_to_f32(MQ[tok * R + 32 * ot + x]);
                mw[ot][v] = m[ot][v] * cw;
            }
        }
#pragma unroll
        for (int ot = 0; ot < OT; ++ot)
#pragma unroll
            for (int gq = 0; gq < 4; ++gq) {
                const f32x4 q4 = {m[ot][4 * gq], m[ot][4 * gq + 1], m[ot][4 * gq + 2], m[ot][4 * gq + 3]};
                const size_t oct = (rtile0 >> 3) + gq;
                *(f32x4 *)&M8r[((oct * 2 + h) * R + 32 * ot + x) * 4] = q4;
            }
#pragma unroll
        for (int sp = 0; sp < 2; ++sp) {
            bf16x8 f[OT], fw[OT];
#pragma unroll
            for (int ot = 0; ot < OT; ++ot) {
                f[ot] = cvt8_from16(m[ot], 8 * sp);
                fw[ot] = cvt8_from16(mw[ot], 8 * sp);
            }
#pragma unroll
            for (int i = 0; i < OT; ++i)
#pragma unroll
                for (int j = 0; j < OT; ++j) sacc[i][j] = mfma32(f[i], fw[j], sacc[i][j]);
        }
    }
    float *out = ScPart + (rrow0 / 256) * R * R;
#pragma unroll
    for (int i = 0; i < OT; ++i)
#pragma unroll
        for (int j = 0; j < OT; ++j) {
            __syncthreads();
#pragma unroll
            for (int v = 0; v < 16; ++v) red[wave][8 * (v / 4) + 4 * h + (v % 4)][x] = sacc[i][j][v];
            __syncthreads();
            for (int idx = tid; idx < 32 * 32; idx += kWg) {
                const int a = idx / 32, c = idx % 32;
                out[(size_t)(32 * i + a) * R + 32 * j + c] = red[0][a][c] + red[1][a][c] + red[2][a][c] + red[3][a][c];
            }
        }
}

// ---- through Algorithm 1 (p = 4), one 32-token tile of a wave --------------------------------
template <int D>
__device__ __forceinline__ void add_held(f32x16 (&dx)[D / 32], const float *__restrict__ held, size_t row, int x, int h)
{
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
        for (int gq = 0; gq < 4; ++gq) {
            const f32x4 base = *(const f32x4 *)&held[held_quad<D>(row, x, h, dt, gq)];
#pragma unroll
            for (int j = 0; j < 4; ++j) dx[dt][4 * gq + j] += base[j];
        }
}

// dst: the first of the wave's 32 rows
template <int D>
__device__ __forceinline__ void store_rows(const RowsOut<D> &out, const f32x16 (&dx)[D / 32], bf16_t *__restrict__ dst)
{
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
        for (int gq = 0; gq < 4; ++gq)
            out.put(dt, gq, f32x4{dx[dt][4 * gq], dx[dt][4 * gq + 1], dx[dt][4 * gq + 2], dx[dt][4 * gq + 3]});
    out.store(dst);
}

// dx = dXacc (if ADD_BASE) + sqrt(1/r) [(dm * (x G2)) G1^T + (dm * (x G1)) G2^T].  lds: the transposed sketch
// matrices as the forward sketch kernel stages them (for the recomputed projections); go: G1,
// G2 as given, rows [d][r] padded to GP (for the transposed products, whose A fragments are read
// in accumulator order).  dm: lane = token, register = sketch column, as the accumulators of
// the cross-block kernel leave it.
template <int D, int R, bool ADD_BASE = true>
__device__ __forceinline__ void sketch_grad_tile(const SketchLds<D, R> &lds, const bf16_t *go,
                                                 const bf16_t *__restrict__ X, const f32x16 *dm,
                                                 const float *__restrict__ dXacc, size_t row, int x, int h,
                                                 f32x16 (&dx)[D / 32])
{
    constexpr int KS = D / 16, NT = R / 32, DT = D / 32, GP = R + 8;
    const float scale = sqrtf(1.0f / (float)R);
    bf16x8 xfr[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) xfr[s] = *(const bf16x8 *)&X[row * D + 16 * s + 8 * h];
    f32x16 a0[NT], a1[NT];                                  // lane = token, register = sketch column
    project<D, R, KS, true>(lds.gt[0], xfr, a0, x, h);
    project<D, R, KS, true>(lds.gt[1], xfr, a1, x, h);
    bf16x8 d0[2 * NT], d1[2 * NT];                          // B operands, contraction over sketch columns
#pragma unroll
    for (int ct = 0; ct < NT; ++ct) {
        f32x16 da0, da1;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            da0[v] = scale * dm[ct][v] * a1[ct][v];
            da1[v] = scale * dm[ct][v] * a0[ct][v];
        }
#pragma unroll
        for (int sp = 0; sp < 2; ++sp) {
            d0[2 * ct + sp] = cvt8_from16(da0, 8 * sp);
            d1[2 * ct + sp] = cvt8_from16(da1, 8 * sp);
        }
    }
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
        f32x16 acc = {0};
#pragma unroll
        for (int ks = 0; ks < 2 * NT; ++ks) {
            // entries e of the step are sketch columns 16 ks + 8 (e / 4) + 4 h + e % 4
            const int off = (32 * dt + x) * GP + 16 * ks + 4 * h;
            const bf16x4 lo1 = *(const bf16x4 *)&go[off], hi1 = *(const bf16x4 *)&go[off + 8];
            const bf16x4 lo2 = *(const bf16x4 *)&go[D * GP + off], hi2 = *(const bf16x4 *)&go[D * GP + off + 8];
            bf16x8 f1, f2;
#pragma unroll
            for (int e = 0; e < 4; ++e) { f1[e] = lo1[e]; f1[4 + e] = hi1[e]; f2[e] = lo2[e]; f2[4 + e] = hi2[e]; }
            acc = mfma32(f1, d0[ks], acc);
            acc = mfma32(f2, d1[ks], acc);
        }
        dx[dt] = acc;
    }
    if constexpr (ADD_BASE) add_held<D>(dx, dXacc, row, x, h);
}

// Both sets of sketch matrices of one parameter set into LDS (see sketch_grad_tile).
template <int D, int R>
__device__ __forceinline__ void sketch_grad_stage(SketchLds<D, R> &lds, bf16_t *go, const bf16_t *__restrict__ Gt,
                                                  const bf16_t *__restrict__ G)
{
    constexpr int GP = R + 8;
    stage_gt<D, R, D>(lds.gt[0], Gt);
    stage_gt<D, R, D>(lds.gt[1], Gt + (size_t)D * R);
    for (int idx = threadIdx.x; idx < 2 * D * (R / 8); idx += kWg) {
        const int m = idx / (D * (R / 8)), rem = idx % (D * (R / 8)), e = rem / (R / 8), part = rem % (R / 8);
        *(uint4 *)&go[(m * D + e) * GP + 8 * part] = *(const uint4 *)&G[(size_t)m * D * R + (size_t)e * R + 8 * part];
    }
}

// ---- through Algorithm 1 as a pass of its own (d = 128 or degree 8) ---------------------------
// dX = bf16(dXacc + J_m(x)^T dm) for 128 rows per workgroup (one 32-row tile per wave, lane = row), dm
// given as fp32 rows (held_quad).  Degree 4: sketch_grad_tile.  Degree 8, with u_k = x G_k (k < 4),
// n1 = s u0 * u1, n2 = s u2 * u3, w1 = n1 G4, w2 = n2 G5, m = s w1 * w2, s = sqrt(1/r):
//     dw1 = s dm * w2, dw2 = s dm * w1;  dn1 = dw1 G4^T, dn2 = dw2 G5^T;
//     du0 = s dn1 * u1, du1 = s dn1 * u0, du2 = s dn2 * u3, du3 = s dn2 * u2;  dx = sum_k du_k G_k^T.
// The matrices go through LDS in phases (two transposed ones for the projections, two as given
// for the transposed products at a time), as in the forward sketch kernel.
template <int D, int R, int P>
__global__ __launch_bounds__(kWg, 2) void k_bwd_sketch_rows(const bf16_t *__restrict__ X, const bf16_t *__restrict__ Gt,
                                                           const bf16_t *__restrict__ G, const float *__restrict__ dM,
                                                           const float *__restrict__ dXacc, bf16_t *__restrict__ dX,
                                                           int n, int heads, int per_head, size_t g_len)
{
    constexpr int KS = D / 16, NT = R / 32, RS = R / 16, DT = D / 32, GP = R + 8;
    constexpr int LDS_BYTES = sizeof(SketchLds<D, R>) + 2 * D * GP * 2;
    static_assert(4 * RowsOut<D>::BYTES <= LDS_BYTES, "the rows reuse the matrices' room");
    __shared__ __attribute__((aligned(16))) unsigned char stage[LDS_BYTES];
    SketchLds<D, R> &lds = *(SketchLds<D, R> *)stage;
    bf16_t *go = (bf16_t *)(stage + sizeof(SketchLds<D, R>));
    const int tid = threadIdx.x, lane = tid & 63, x = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const size_t row0 = (size_t)blockIdx.x * 128, row = row0 + wave * 32 + x;
    const size_t goff = per_head ? (size_t)((row0 / n) % heads) * g_len : 0;
    const bf16_t *gt = Gt + goff, *g = G + goff;
    // dm of the tile: lane = row, register v of tile ct = sketch column 32 ct + 8 (v / 4) + 4 h + v % 4
    f32x16 dm[NT];
#pragma unroll
    for (int ct = 0; ct < NT; ++ct)
#pragma unroll
        for (int gq = 0; gq < 4; ++gq) {
            const f32x4 d4 = *(const f32x4 *)&dM[held_quad<R>(row, x, h, ct, gq)];
#pragma unroll
            for (int j = 0; j < 4; ++j) dm[ct][4 * gq + j] = d4[j];
        }
    f32x16 dx[DT];
    if constexpr (P == 4) {
        sketch_grad_stage<D, R>(lds, go, gt, g);
        __syncthreads();
        sketch_grad_tile<D, R, true>(lds, go, X, dm, dXacc, row, x, h, dx);
    } else {
        static_assert(P == 8, "degree 4 or 8");
        const float scale = sqrtf(1.0f / (float)R);
        // rows [0, nrows) of a matrix given as [nrows][R] -> go[which] with rows padded to GP
        auto stage_rows = [&](int which, const bf16_t *src, int nrows) {
            for (int idx = tid; idx < nrows * (R / 8); idx += kWg) {
                const int e = idx / (R / 8), part = idx % (R / 8);
                *(uint4 *)&go[(which * D + e) * GP + 8 * part] = *(const uint4 *)&src[(size_t)e * R + 8 * part];
            }
        };
        // out[i][row] = sum_k M[i][k] v[k][row], M as given ([.][R], staged by stage_rows), v as B
        // fragments in accumulator order (entries e of step ks: k = 16 ks + 8 (e / 4) + 4 h + e % 4)
        auto times_rows = [&](int which, int tile, const bf16x8 *v, f32x16 acc) {
#pragma unroll
            for (int ks = 0; ks < RS; ++ks) {
                const int off = (which * D + 32 * tile + x) * GP + 16 * ks + 4 * h;
                const bf16x4 lo = *(const bf16x4 *)&go[off], hi = *(const bf16x4 *)&go[off + 8];
                bf16x8 f;
#pragma unroll
                for (int e = 0; e < 4; ++e) { f[e] = lo[e]; f[4 + e] = hi[e]; }
                acc = mfma32(f, v[ks], acc);
            }
            return acc;
        };
        auto to_frags = [&](const f32x16 (&a)[NT], bf16x8 (&f)[RS]) {
#pragma unroll
            for (int ct = 0; ct < NT; ++ct)
#pragma unroll
                for (int q2 = 0; q2 < 2; ++q2) f[2 * ct + q2] = cvt8_from16(a[ct], 8 * q2);
        };
        bf16x8 xfr[KS];
#pragma unroll
        for (int s = 0; s < KS; ++s) xfr[s] = *(const bf16x8 *)&X[row * D + 16 * s + 8 * h];
        // the projections are kept as bf16 (like every operand of the products they enter): half the registers
        bf16x8 ub[4][RS];
        bf16x8 nfr[2][RS];
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            __syncthreads();
            stage_gt<D, R, D>(lds.gt[0], gt + (size_t)(2 * half) * D * R);
            stage_gt<D, R, D>(lds.gt[1], gt + (size_t)(2 * half + 1) * D * R);
            __syncthreads();
            f32x16 ua[NT], uc[NT];
            project<D, R, KS, true>(lds.gt[0], xfr, ua, x, h);
            project<D, R, KS, true>(lds.gt[1], xfr, uc, x, h);
            f32x16 nn[NT];
#pragma unroll
            for (int ct = 0; ct < NT; ++ct) nn[ct] = scale * (ua[ct] * uc[ct]);
            to_frags(nn, nfr[half]);
            to_frags(ua, ub[2 * half]);
            to_frags(uc, ub[2 * half + 1]);
        }
        auto u_at = [&](int k, int ct, int v) { return (float)ub[k][2 * ct + v / 8][v % 8]; };
        __syncthreads();
        const size_t inner = (size_t)4 * D * R;
        stage_gt<D, R, R>(lds.gt[0], gt + inner);
        stage_gt<D, R, R>(lds.gt[1], gt + inner + (size_t)R * R);
        stage_rows(0, g + inner, R);
        stage_rows(1, g + inner + (size_t)R * R, R);
        __syncthreads();
        bf16x8 duf[4][RS];
        {
            f32x16 w1[NT], w2[NT];
            project_inner<D, R, true>(lds.gt[0], nfr[0], w1, x, h);
            project_inner<D, R, true>(lds.gt[1], nfr[1], w2, x, h);
            f32x16 d1[NT], d2[NT];
#pragma unroll
            for (int ct = 0; ct < NT; ++ct) {
                d1[ct] = scale * (dm[ct] * w2[ct]);
                d2[ct] = scale * (dm[ct] * w1[ct]);
            }
            bf16x8 dw1[RS], dw2[RS];
            to_frags(d1, dw1);
            to_frags(d2, dw2);
            f32x16 t0[NT], t1[NT];
#pragma unroll
            for (int ct = 0; ct < NT; ++ct) {
                const f32x16 dn1 = times_rows(0, ct, dw1, f32x16{0}), dn2 = times_rows(1, ct, dw2, f32x16{0});
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    t0[ct][v] = scale * dn1[v] * u_at(1, ct, v);
                    t1[ct][v] = scale * dn1[v] * u_at(0, ct, v);
                    d1[ct][v] = scale * dn2[v] * u_at(3, ct, v);
                    d2[ct][v] = scale * dn2[v] * u_at(2, ct, v);
                }
            }
            to_frags(t0, duf[0]);
            to_frags(t1, duf[1]);
            to_frags(d1, duf[2]);
            to_frags(d2, duf[3]);
        }
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) dx[dt] = f32x16{0};
#pragma unroll
        for (int pair = 0; pair < 2; ++pair) {
            __syncthreads();
            stage_rows(0, g + (size_t)(2 * pair) * D * R, D);
            stage_rows(1, g + (size_t)(2 * pair + 1) * D * R, D);
            __syncthreads();
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) {
                dx[dt] = times_rows(0, dt, duf[2 * pair], dx[dt]);
                dx[dt] = times_rows(1, dt, duf[2 * pair + 1], dx[dt]);
            }
        }
        add_held<D>(dx, dXacc, row, x, h);
    }
    __syncthreads();                                        // every wave is done with the matrices
    store_rows<D>(RowsOut<D>(stage, wave, lane), dx, dX + (row0 + wave * 32) * D);
}

// ---- contraction of the states with a row's gradient (or value) --------------------------------
// dm[e] = sum_b 2 Z[e][b][.] . vec  m[b] for 32 TT tokens a wave, from the snapshots as the state kernel writes
// them ([a][b'/8][c][8]: b' > a doubled, b' = a once, b' < a zero).  With T[a][b'] = sum_c Zs[a][b'][c] vec[c]:
//     dm[a] += T[a][b'] m[b'],  dm[b'] += T[a][b'] m[a]   for every stored segment (a, 16 columns b'),
// the diagonal 16 x 16 squares included (what is stored doubled meets each of the two once, what is stored
// once meets itself twice).  vec is the fixed B operand (lane = token), so no operand is generated and
// T stays fp32: 62 % of the products of a contraction over (b, c) pairs at r = 64, 75 % at r = 32, and 8 (D =
// 64) or 4 (D = 128) vector instructions a product instead of 6 (r = 64) or 12 (r = 32).
// A fragments run along c while the snapshot's octets run along b': ds_read_b64_tr_b16 turns 4 columns c x 16
// columns b' round on the way out of LDS, so no re-laid copy of the states is needed.
// A tile is two segments of the rows a and a + 4 and one 16-wide range of b': a lane's half of
// the rows of T then lines up with the half of m and dm it holds (index 8 (i / 4) + 4 h + i % 4 of a range),
// and the two halves' sums for a and a + 4 change places with one swap.  Its four planes (octets 2 beta, 2 beta + 1
// of both rows, one per wave of the copy) lie 64 bytes apart modulo 256, so that the 16-lane groups of a
// transposed read meet different banks.
template <int R, int D, int TT>
struct StateTimesRow : StateTiles<R, D> {
    using Base = StateTiles<R, D>;
    using Base::RS;
    using Base::VS;
    using Base::PS;
    using Base::TILE;
    using Base::TILES;
    using Base::SLOTS;
    using Base::range_of;
    using Base::pair_of;
    using Base::beta_of;

    // the products of tile IT with the row: m, dm in the order of the accumulators (index 8 range + i)
    template <int IT>
    static __device__ __forceinline__ void consume(const f32x16 &T, const float (&m)[8 * RS], float (&dm)[8 * RS],
                                                   float &ma, float &mb, float &sa, float &sb)
    {
        constexpr int S0 = range_of(IT), BETA = beta_of(IT), P = pair_of(IT), I = 8 * S0 + P;   // I: the index of a and a + 4
        if constexpr (BETA == S0) {
            const uint32_t w = __float_as_uint(m[I]);
            const auto both = __builtin_amdgcn_permlane32_swap(w, w, false, false);
            ma = __uint_as_float(both[0]);
            mb = __uint_as_float(both[1]);
            sa = sb = 0.f;
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            dm[8 * BETA + i] = fmaf(T[i], ma, dm[8 * BETA + i]);
            sa = fmaf(T[i], m[8 * BETA + i], sa);
            dm[8 * BETA + i] = fmaf(T[8 + i], mb, dm[8 * BETA + i]);
            sb = fmaf(T[8 + i], m[8 * BETA + i], sb);
        }
        if constexpr (BETA == RS - 1) {
            const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(sa), __float_as_uint(sb), false, false);
            dm[I] += __uint_as_float(s[0]) + __uint_as_float(s[1]);
        }
    }
    // The ring's first tiles are on their way (Ring::fill).  vec: B operands; ends with a barrier.
    static __device__ __forceinline__ void run(const bf16_t *__restrict__ Z, const bf16x8 (&vec)[TT][VS],
                                               const float (&m)[TT][8 * RS], float (&dm)[TT][8 * RS], unsigned char *lds)
    {
        const int lane = threadIdx.x & 63, h = lane >> 5, s16 = lane & 15;
        const typename Base::Ring ring(Z, lds);
        // (offsets of a read reach 64 KB: a base for each half of the ring)
        const unsigned char *const lane_lo =
            lds + (2 * ((lane >> 4) & 1) + ((s16 & 3) >> 1)) * PS + (8 * h + (s16 >> 2)) * 16 + (s16 & 1) * 8;
        const unsigned char *const lane_hi = lane_lo + SLOTS / 2 * TILE;
        bf16x8 af[2][VS];
        auto load = [&](auto it_tag) {
            constexpr int IT = decltype(it_tag)::value, SLOT = IT % SLOTS;
            const unsigned char *base = SLOT < SLOTS / 2 ? lane_lo + SLOT * TILE : lane_hi + (SLOT - SLOTS / 2) * TILE;
#pragma unroll
            for (int s = 0; s < VS; ++s) af[IT & 1][s] = read_turned(base + s * 256, base + s * 256 + 64);
        };
        ring.start();
        load(std::integral_constant<int, 0>{});
        float ma[TT], mb[TT], sa[TT], sb[TT];
        f32x16 T[2];
        static_for<TILES>([&](auto it_tag) {
            constexpr int IT = decltype(it_tag)::value;
            ring.template advance<IT>();
            static_for<TT>([&](auto tt_tag) {
                constexpr int tt = decltype(tt_tag)::value, Q = IT * TT + tt;
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (tt == 0 && IT + 1 < TILES) load(std::integral_constant<int, IT + 1>{});
                f32x16 acc = {0};
#pragma unroll
                for (int s = 0; s < VS; ++s) acc = mfma32(af[IT & 1][s], vec[tt][s], acc);
                // the tile before this one, under these products
                constexpr int TP = tt > 0 ? tt - 1 : TT - 1, ITP = tt > 0 ? IT : IT - 1;
                if constexpr (ITP >= 0) consume<ITP>(T[(Q + 1) & 1], m[TP], dm[TP], ma[TP], mb[TP], sa[TP], sb[TP]);
                T[Q & 1] = acc;
                if constexpr (tt == 0 && IT + 1 < TILES) __builtin_amdgcn_sched_group_barrier(0x100, 2 * VS, 0);
#pragma unroll
                for (int s = 0; s < VS; ++s) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x002, 36 / VS, 0);
                }
            });
        });
        consume<TILES - 1>(T[(TILES * TT + 1) & 1], m[TT - 1], dm[TT - 1], ma[TT - 1], mb[TT - 1], sa[TT - 1], sb[TT - 1]);
        __syncthreads();                                       // the caller may reuse the stage
    }
};

// ---- dm(q) and dm(k): cross-block part -------------------------------------------------------
// dm of the workgroup's 128 TT rows from i0 of unit u on; stage: StateTimesRow's room, free again at the end (of every wave
// where there was a state, untouched where there was none: then false).
template <int R, int D, bool QSIDE, int TT>
__device__ __forceinline__ bool dm_rows(const bf16_t *__restrict__ M, const bf16_t *__restrict__ Vec,
                                        const float *__restrict__ Cc, const bf16_t *__restrict__ Zs,
                                        const bf16_t *__restrict__ Shi, const bf16_t *__restrict__ Slo, int u, int i0,
                                        int n, int b, int t, unsigned char *stage, f32x16 (&out)[TT][R / 32])
{
    using X = StateTimesRow<R, D, TT>;
    constexpr int AT = R / 32, RS = R / 16, VS = D / 16;
    const int lane = threadIdx.x & 63, x = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l = i0 / b;
    const size_t urow = (size_t)u * n;
    const bool has = QSIDE ? l > 0 : l < t - 1;
    const int slot = QSIDE ? l - 1 : t - 2 - l;

#pragma unroll
    for (int tt = 0; tt < TT; ++tt)
#pragma unroll
        for (int at = 0; at < AT; ++at) out[tt][at] = f32x16{0};
    if (has) {
        const bf16_t *z = Zs + ((size_t)u * (t - 1) + slot) * R * R * D;
        typename X::Ring(z, stage).fill();
        // ones column: (S m)[a] per token with S as hi + lo A operands [b'/8][a][8]
        bf16x8 mfr[TT][RS];
#pragma unroll
        for (int tt = 0; tt < TT; ++tt)
#pragma unroll
            for (int s = 0; s < RS; ++s)
                mfr[tt][s] = *(const bf16x8 *)&M[(urow + i0 + wave * 32 * TT + 32 * tt + x) * R + 16 * s + 8 * h];
        float dm[TT][8 * RS], m[TT][8 * RS];                // entry 8 s + i: sketch column 16 s + 8 (i / 4) + 4 h + i % 4
        const size_t sbase = ((size_t)u * (t - 1) + slot) * R * R;
#pragma unroll
        for (int at = 0; at < AT; ++at) {
            f32x16 td[TT];
#pragma unroll
            for (int tt = 0; tt < TT; ++tt) td[tt] = f32x16{0};
#pragma unroll
            for (int s = 0; s < RS; ++s) {
                const size_t off = sbase + ((size_t)(2 * s + h) * R + 32 * at + x) * 8;
                const bf16x8 s_hi = *(const bf16x8 *)&Shi[off], s_lo = *(const bf16x8 *)&Slo[off];
#pragma unroll
                for (int tt = 0; tt < TT; ++tt) {
                    td[tt] = mfma32(s_hi, mfr[tt][s], td[tt]);
                    td[tt] = mfma32(s_lo, mfr[tt][s], td[tt]);
                }
            }
#pragma unroll
            for (int tt = 0; tt < TT; ++tt) {
                const float coef = QSIDE ? Cc[urow + i0 + wave * 32 * TT + 32 * tt + x] : 1.0f;
#pragma unroll
                for (int v = 0; v < 16; ++v) dm[tt][16 * at + v] = 2.0f * coef * td[tt][v];   // the states count twice, too
            }
        }
        // m in the same order: the B operands hold columns 16 s + 8 h + e, one swap per register pair
#pragma unroll
        for (int tt = 0; tt < TT; ++tt)
#pragma unroll
            for (int s = 0; s < RS; ++s) {
                const uint4 w = __builtin_bit_cast(uint4, mfr[tt][s]);
                const auto s0 = __builtin_amdgcn_permlane32_swap(w.x, w.z, false, false);
                const auto s1 = __builtin_amdgcn_permlane32_swap(w.y, w.w, false, false);
                const uint32_t pr[4] = {s0[0], s1[0], s0[1], s1[1]};
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    m[tt][8 * s + i] = __uint_as_float((i & 1) ? (pr[i / 2] & 0xffff0000u) : (pr[i / 2] << 16));
            }
        bf16x8 vec[TT][VS];
#pragma unroll
        for (int tt = 0; tt < TT; ++tt)
#pragma unroll
            for (int s = 0; s < VS; ++s)
                vec[tt][s] = *(const bf16x8 *)&Vec[(urow + i0 + wave * 32 * TT + 32 * tt + x) * D + 16 * s + 8 * h];
        X::run(z, vec, m, dm, stage);
#pragma unroll
        for (int tt = 0; tt < TT; ++tt)
#pragma unroll
            for (int at = 0; at < AT; ++at)
#pragma unroll
                for (int v = 0; v < 16; ++v) out[tt][at][v] = dm[tt][16 * at + v];
    }
    return has;
}

// QSIDE: tokens of block l >= 1 with Z / S of slot l - 1, vec = g, coefficient c_i.
// key side: tokens of block l <= t - 2 with R / Rc of the mirror slot t - 2 - l, vec = v,
// coefficient 1.  Blocks without a cross-block term have dm = 0.  dm stays in registers and goes
// straight through Algorithm 1 (sketch_grad_tile): dX = bf16(dXacc + J_m(x)^T dm), with dXacc the
// in-block part, for the rows X (Q or K) of the workgroup.
// LS (in-block rule of Section 3.1, R == D): the in-block weights are functions of the sketches
// too, so dXacc holds the in-block part of dm ([rows][R] fp32), which joins dm before the sketch:
// dX = bf16(J_m(x)^T (dm + dXacc)).
// RAW (learned sketches, and those with a pass of their own): dm itself is the result, fp32 rows (held_quad) in dMout.
template <int R, int D, bool QSIDE, int TT, bool LS = false, bool RAW = false>
__global__ __launch_bounds__(kWg, (StateTiles<R, D>::OCC)) void k_bwd_dm(const bf16_t *__restrict__ M, const bf16_t *__restrict__ Vec,
                                                  const float *__restrict__ Cc, const bf16_t *__restrict__ Zs,
                                                  const bf16_t *__restrict__ Shi, const bf16_t *__restrict__ Slo,
                                                  const bf16_t *__restrict__ Xrows, const bf16_t *__restrict__ Gt,
                                                  const bf16_t *__restrict__ G, const float *__restrict__ dXacc,
                                                  bf16_t *__restrict__ dX, int n, int b, int t, int heads,
                                                  int per_head, size_t g_len, float *__restrict__ dMout = nullptr)
{
    using X = StateTimesRow<R, D, TT>;
    constexpr int MATS = sizeof(SketchLds<D, R>) + 2 * D * (R + 8) * 2;
    static_assert(RAW || MATS + 4 * RowsOut<D>::BYTES <= X::LDS_BYTES, "the sketch matrices and the result rows reuse the stage");
    constexpr int AT = R / 32, TOK_WG = 128 * TT;
    __shared__ __attribute__((aligned(16))) unsigned char stage[X::LDS_BYTES];
    const int tid = threadIdx.x, lane = tid & 63, x = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tiles_per_unit = n / TOK_WG;
    int wg = blockIdx.x;                                    // XCD-aware order: one state snapshot, one L2
    if ((gridDim.x & 7) == 0) wg = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    const int u = wg / tiles_per_unit, i0 = (wg % tiles_per_unit) * TOK_WG;
    const size_t urow = (size_t)u * n;

    f32x16 out[TT][AT];
    dm_rows<R, D, QSIDE, TT>(M, Vec, Cc, Zs, Shi, Slo, u, i0, n, b, t, stage, out);
    if constexpr (RAW) {
        // register v of out[tt][at]: sketch column 32 at + 8 (v / 4) + 4 h + v % 4
#pragma unroll
        for (int tt = 0; tt < TT; ++tt)
#pragma unroll
            for (int at = 0; at < AT; ++at)
#pragma unroll
                for (int gq = 0; gq < 4; ++gq) {
                    const f32x4 o4 = {out[tt][at][4 * gq], out[tt][at][4 * gq + 1], out[tt][at][4 * gq + 2],
                                      out[tt][at][4 * gq + 3]};
                    *(f32x4 *)&dMout[held_quad<R>(urow + i0 + wave * 32 * TT + 32 * tt + x, x, h, at, gq)] = o4;
                }
        return;
    }
    // through the sketch; the stage is free again (the contraction ends with a barrier)
    SketchLds<D, R> &lds = *(SketchLds<D, R> *)stage;
    bf16_t *go = (bf16_t *)(stage + sizeof(SketchLds<D, R>));
    const size_t goff = per_head ? (size_t)(u % heads) * g_len : 0;
    sketch_grad_stage<D, R>(lds, go, Gt + goff, G + goff);
    __syncthreads();
    if constexpr (LS) {
        static_assert(R == D, "the in-block kernels leave dm in the layout of a gradient row");
#pragma unroll
        for (int tt = 0; tt < TT; ++tt)
#pragma unroll
            for (int at = 0; at < AT; ++at)
#pragma unroll
                for (int gq = 0; gq < 4; ++gq) {
                    // register v of out[tt][at]: sketch column 32 at + 8 (v / 4) + 4 h + v % 4
                    const f32x4 a4 = *(const f32x4 *)&dXacc[held_quad<R>(urow + i0 + wave * 32 * TT + 32 * tt + x, x, h,
                                                                         at, gq)];
#pragma unroll
                    for (int j = 0; j < 4; ++j) out[tt][at][4 * gq + j] += a4[j];
                }
    }
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) {
        const size_t row = urow + i0 + wave * 32 * TT + 32 * tt;
        f32x16 dx[D / 32];
        sketch_grad_tile<D, R, !LS>(lds, go, Xrows, out[tt], dXacc, row + x, x, h, dx);
        store_rows<D>(RowsOut<D>(stage + MATS, wave, lane), dx, dX + row * D);
    }
}

// ---- dV: cross-block part = phi'(k_j)^T R_l (value columns) ----------------------------------
// 32 TT rows a wave of the 128 TT from i0 of unit u on; slot: the mirror state they take.
template <int R, int D, int TT>
__device__ __forceinline__ void dv_rows(const bf16_t *__restrict__ MK, const bf16_t *__restrict__ Rg, int u, int i0, int slot,
                                        int n, int t, unsigned char *stage, f32x16 (&out)[TT][D / 32])
{
    using X = FeaturesTimesState<R, D, TT>;
    constexpr int RS = R / 16;
    const int lane = threadIdx.x & 63, x = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const bf16_t *r = Rg + ((size_t)u * (t - 1) + slot) * R * R * D;
    typename X::Ring(r, stage).fill();
    f32x8 vec[TT][RS];
#pragma unroll
    for (int tt = 0; tt < TT; ++tt)
#pragma unroll
        for (int s = 0; s < RS; ++s) {
            const bf16x8 raw = *(const bf16x8 *)&MK[((size_t)u * n + i0 + wave * 32 * TT + 32 * tt + x) * R + 16 * s + 8 * h];
#pragma unroll
            for (int e = 0; e < 8; ++e) vec[tt][s][e] = (float)raw[e];
        }
    X::run(r, vec, out, stage);
}

template <int R, int D, int TT>
__global__ __launch_bounds__(kWg, (StateTiles<R, D>::OCC)) void k_bwd_dvc(const bf16_t *__restrict__ MK, const bf16_t *__restrict__ Rg,
                                                   float *__restrict__ dVc, int n, int b, int t)
{
    using X = FeaturesTimesState<R, D, TT>;
    constexpr int CT = D / 32, TOK_WG = 128 * TT;
    __shared__ __attribute__((aligned(16))) unsigned char stage[X::LDS_BYTES];
    const int tid = threadIdx.x, lane = tid & 63, x = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tiles_per_unit = n / TOK_WG;
    int wg = blockIdx.x;                                    // XCD-aware order: one state snapshot, one L2
    if ((gridDim.x & 7) == 0) wg = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    const int u = wg / tiles_per_unit, i0 = (wg % tiles_per_unit) * TOK_WG;
    const int l = i0 / b;
    const size_t urow = (size_t)u * n;
    f32x16 out[TT][CT];
#pragma unroll
    for (int tt = 0; tt < TT; ++tt)
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) out[tt][ct] = f32x16{0};
    if (l < t - 1) dv_rows<R, D, TT>(MK, Rg, u, i0, t - 2 - l, n, t, stage, out);
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) {
        const size_t row = urow + i0 + wave * 32 * TT + 32 * tt + x;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
#pragma unroll
            for (int gq = 0; gq < 4; ++gq) {
                const f32x4 q4 = {out[tt][ct][4 * gq], out[tt][ct][4 * gq + 1], out[tt][ct][4 * gq + 2],
                                  out[tt][ct][4 * gq + 3]};
                *(f32x4 *)&dVc[held_quad<D>(row, x, h, ct, gq)] = q4;
            }
    }
}

// The cross-block part of one side inside the in-block kernel of that side (degree 4, Gaussian sketches, r = 32): the
// gradient through the states and the sketch is where the in-block accumulators start from, so that the fp32 rows
// between the two kernels (one written and read for queries, two for keys) and the second read of the side's own rows
// go away.  At r = 64 the contractions want 64 rows a wave, which the in-block part has no registers for.  96 units of
// 4096, us, as kernels of their own and in one: queries 71 + 99 and 123, keys 93 + 94 + 60 and 169.
struct CrossSide {
    const bf16_t *M, *Zs, *Shi, *Slo, *Gt, *G;               // the side's sketches, states, matrices
    bf16_t *dX;
    int heads, per_head;
    size_t g_len;

    template <int R, int D>
    static constexpr int mats_bytes() { return sizeof(SketchLds<D, R>) + 2 * D * (R + 8) * 2; }
    template <int R, int D>
    static constexpr int lds_bytes() { return std::max(StateTimesRow<R, D, 1>::LDS_BYTES, mats_bytes<R, D>()); }

    // dx: 1 / P (a power of two) of the row's gradient, 128 rows from i0 of unit u on.  stage is free before and after.
    template <int R, int D, int P, bool QSIDE>
    __device__ __forceinline__ void rows(const bf16_t *__restrict__ Vec, const float *__restrict__ Cc,
                                         const bf16_t *__restrict__ X, int u, int i0, int n, int b, int t,
                                         unsigned char *stage, f32x16 (&dx)[D / 32]) const
    {
        const int lane = threadIdx.x & 63, x = lane & 31, h = lane >> 5;
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        f32x16 dm[1][R / 32];
        if (!dm_rows<R, D, QSIDE, 1>(M, Vec, Cc, Zs, Shi, Slo, u, i0, n, b, t, stage, dm)) {
#pragma unroll
            for (int ct = 0; ct < D / 32; ++ct) dx[ct] = f32x16{0};
            return;
        }
        SketchLds<D, R> &lds = *(SketchLds<D, R> *)stage;
        bf16_t *go = (bf16_t *)(stage + sizeof(SketchLds<D, R>));
        const size_t goff = per_head ? (size_t)(u % heads) * g_len : 0;
        sketch_grad_stage<D, R>(lds, go, Gt + goff, G + goff);
        __syncthreads();
        sketch_grad_tile<D, R, false>(lds, go, X, dm[0], nullptr, (size_t)u * n + i0 + wave * 32 + x, x, h, dx);
#pragma unroll
        for (int ct = 0; ct < D / 32; ++ct) dx[ct] *= 1.0f / (float)P;
        __syncthreads();
    }
};

// ---- in-block pairs ---------------------------------------------------------------------------
// Both kernels: workgroup = 32 NW "own" rows (wave = 32, held in registers as B operands), the other side streams
// through LDS in tiles of 64 rows, double buffered, as its rows lie in memory.  Score tiles come out transposed
// (lane = own row, registers = streamed rows), are turned into bf16 B operands as they stand and contracted with
// the same rows read transposed (ds_read_b64_tr_b16, in the order of the accumulator registers): one copy of the
// streamed side in LDS serves both products, so no layouts of Q, K, V and g are made in memory, twice as
// many workgroups fit a CU's LDS, and a tile costs half the copies.
constexpr int kLocT = 64;                                   // streamed rows per tile
template <int D, int NTHR>
struct LocTile {
    static constexpr int BYTES = kLocT * D * 2, PIECES = D / 8, KS = D / 16, CT = D / 32;
    static constexpr int ROWS_PER_COPY = NTHR / PIECES;     // rows one copy instruction of the workgroup moves
    static_assert(ROWS_PER_COPY % 16 == 0 && kLocT % ROWS_PER_COPY == 0, "whole swizzle periods per copy");
    static __device__ __forceinline__ int swz(int j) { return row_swz<D>(j); }
    int x, h, tid, wave;
    uint32_t copy_off;                                      // lane's place in a copy's source
    uint32_t plain[KS], turned[2][CT];                      // lane's byte offsets of fragments, see rows() and columns()
    __device__ __forceinline__ LocTile()
    {
        tid = threadIdx.x;
        const int lane = tid & 63;
        x = lane & 31;
        h = lane >> 5;
        wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        copy_off = row_copy_offset<D>(tid);
#pragma unroll
        for (int s = 0; s < KS; ++s) plain[s] = (uint32_t)((x * PIECES + ((2 * s + h) ^ swz(x))) * 16);
#pragma unroll
        for (int hi = 0; hi < 2; ++hi)
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) turned[hi][ct] = row_turned_offset<D>(lane, 8 * hi + 4 * h, ct);
    }
    // rows [j0, j0 + 64) of X -> LDS
    __device__ __forceinline__ void stage(const bf16_t *__restrict__ X, size_t j0, uint32_t dst) const
    {
#pragma unroll
        for (int q = 0; q < kLocT / ROWS_PER_COPY; ++q)
            dma16_sbase(X + (j0 + q * ROWS_PER_COPY) * D, copy_off, dst + q * (NTHR * 16) + wave * 1024);
    }
    // A fragment: rows 32 sub + x, columns 16 s + 8 h + e
    __device__ __forceinline__ bf16x8 rows(const unsigned char *tile, int sub, int s) const
    {
        return *(const bf16x8 *)(tile + plain[s] + sub * 32 * D * 2);
    }
    // A fragment: columns 32 ct + x, contraction over the rows 32 sub + 16 sp + 8 (e / 4) + 4 h + e % 4
    __device__ __forceinline__ bf16x8 columns(const unsigned char *tile, int sub, int sp, int ct) const
    {
        const unsigned char *t = tile + (32 * sub + 16 * sp) * D * 2;
        return read_turned(t + turned[0][ct], t + turned[1][ct]);
    }
};

// dQ (in-block): own rows = queries, streamed = keys of the same block up to the diagonal.
//   dq_i = sum_{j <= i} (<g_i, v_j> + c_i) p <q_i, k_j>^(p-1) k_j          -> dQacc fp32 rows
// CROSS: the cross-block part and Algorithm 1's reverse first, in the same workgroup, into the accumulators (see CrossSide).
// The launch's last workgroups scan the mirror states' ones column (R: sketch width; DenScan::n_main others come first).
template <int P, int NW, int D, int R, bool CROSS = false>
__global__ __launch_bounds__(64 * NW, D == 64 ? 3 : 2) void k_bwd_local_q(const bf16_t *__restrict__ Q, const bf16_t *__restrict__ K,
                                                                         const bf16_t *__restrict__ V, const bf16_t *__restrict__ G_rm,
                                                                         const float *__restrict__ Cc, float *__restrict__ dQacc,
                                                                         int n, int b, int t, DenScan den, CrossSide cx = {})
{
    constexpr int KS = D / 16, CT = D / 32, NTHR = 64 * NW, OWN = 32 * NW;
    using Tile = LocTile<D, NTHR>;
    constexpr int BUF = 2 * Tile::BYTES;
    static_assert(NTHR == kWg, "the scan's workgroup");
    __shared__ __attribute__((aligned(16))) unsigned char stage[CROSS ? std::max(2 * BUF, CrossSide::lds_bytes<R, D>()) : 2 * BUF];
    if (den_scan_role<R, NTHR>(den, t, stage)) return;
    const Tile T;
    const int x = T.x, h = T.h, tiles_per_unit = n / OWN;
    // XCD-aware order: consecutive workgroup ids go to different XCDs, so give each XCD a
    // contiguous range of tiles: the workgroups that stream the same rows then share one L2
    int wg = blockIdx.x;
    if ((den.n_main & 7) == 0) wg = (blockIdx.x & 7) * (den.n_main >> 3) + (blockIdx.x >> 3);
    const int u = wg / tiles_per_unit, i0 = (wg % tiles_per_unit) * OWN;
    const int jb = (i0 / b) * b;
    const size_t urow = (size_t)u * n;
    const int tok0 = i0 + 32 * T.wave, tok = tok0 + x;
    f32x16 dq[CT];
    if constexpr (CROSS) {
        cx.rows<R, D, P, true>(G_rm, Cc, Q, u, i0, n, b, t, stage, dq);
    } else {
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) dq[ct] = f32x16{0};
    }
    bf16x8 qfr[KS], gfr[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        qfr[s] = *(const bf16x8 *)&Q[(urow + tok) * D + 16 * s + 8 * h];
        gfr[s] = *(const bf16x8 *)&G_rm[(urow + tok) * D + 16 * s + 8 * h];
    }
    const float c_me = Cc[urow + tok];
    const int ntiles = (i0 + OWN - jb) / kLocT;
    const uint32_t stage0 = lds_address(stage);
    auto stage_tile = [&](int kt) {
        const uint32_t dst = stage0 + (kt & 1) * BUF;
        const size_t j0 = urow + jb + (size_t)kt * kLocT;
        T.stage(K, j0, dst);
        T.stage(V, j0, dst + Tile::BYTES);
    };
    auto tile = [&](auto diag_tag, int kt) {
        constexpr bool DIAG = decltype(diag_tag)::value;
        const unsigned char *ks = stage + (kt & 1) * BUF, *vs = ks + Tile::BYTES;
        bf16x8 pw[2][2];
#pragma unroll
        for (int sub = 0; sub < 2; ++sub) {
            f32x16 sc = {0}, dw = {0};
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                sc = mfma32(T.rows(ks, sub, s), qfr[s], sc);
                dw = mfma32(T.rows(vs, sub, s), gfr[s], dw);
            }
            // key = key0 + 8 (v / 4) + 4 h + v % 4 <= tok  <=>  8 (v / 4) + v % 4 <= lim
            const int lim = tok - (jb + kt * kLocT + 32 * sub) - 4 * h;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const float sm = !DIAG || 8 * (v / 4) + (v % 4) <= lim ? sc[v] : 0.f;   // masked pairs: every power is 0
                dw[v] = (dw[v] + c_me) * pow_n<P - 1>(sm);
            }
            pw[sub][0] = cvt8_from16(dw, 0);
            pw[sub][1] = cvt8_from16(dw, 8);
        }
#pragma unroll
        for (int sub = 0; sub < 2; ++sub)
#pragma unroll
            for (int sp = 0; sp < 2; ++sp)
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) dq[ct] = mfma32(T.columns(ks, sub, sp, ct), pw[sub][sp], dq[ct]);
    };
    // (loops of one body each: with both bodies in one loop the accumulators change registers and spill)
    auto sync = [&](int kt) {
        wait_vmem_le<0>();
        __syncthreads();
        if (kt + 1 < ntiles) stage_tile(kt + 1);
    };
    const int diag = (tok0 - jb) / kLocT;                  // the tile that holds this wave's own tokens
    stage_tile(0);
#pragma unroll 1
    for (int kt = 0; kt < diag; ++kt) {
        sync(kt);
        tile(std::false_type{}, kt);
        branch_wait();
    }
    sync(diag);
    tile(std::true_type{}, diag);
#pragma unroll 1
    for (int kt = diag + 1; kt < ntiles; ++kt) sync(kt);   // later tiles: only keep the barriers and copies going
    if constexpr (CROSS) {
        __syncthreads();                                    // every wave is done with the last tile
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) dq[ct] *= (float)P;
        store_rows<D>(RowsOut<D>(stage, T.wave, T.tid & 63), dq, cx.dX + (urow + tok0) * D);
        return;
    }
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int gq = 0; gq < 4; ++gq) {
            // (the p of p s^(p-1): a power of two, exact)
            const f32x4 q4 = {(float)P * dq[ct][4 * gq], (float)P * dq[ct][4 * gq + 1], (float)P * dq[ct][4 * gq + 2],
                              (float)P * dq[ct][4 * gq + 3]};
            *(f32x4 *)&dQacc[held_quad<D>(urow + tok, x, h, ct, gq)] = q4;
        }
}

// dK (in-block) and dV (in-block + the cross-block part already in dVc): own rows = keys,
// streamed = queries of the same block from the diagonal on.
//   dk_j = sum_{i >= j} (<g_i, v_j> + c_i) p <q_i, k_j>^(p-1) q_i   -> dKacc fp32 rows (held_quad)
//   dv_j = sum_{i >= j} <q_i, k_j>^p g_i + dVc_j                     -> dV bf16 rows
// CROSS: the cross-block parts of both first, in the same workgroup, into the accumulators; dK as bf16 rows (see CrossSide).
// CROSS_V: dV's alone, from the mirror states cx.Zs and m(K) in cx.M (48 units of 8192, r = 32: 172 us, with k_bwd_dvc and
// its fp32 rows 154 + 44; a call of 16 units of 16384, d = 128: 2035, 2083).
template <int P, int NW, int D, int R = 0, bool CROSS = false, bool CROSS_V = CROSS>
__global__ __launch_bounds__(64 * NW, D == 64 ? 3 : 2) void k_bwd_local_k(const bf16_t *__restrict__ Q, const bf16_t *__restrict__ K,
                                                                         const bf16_t *__restrict__ V, const bf16_t *__restrict__ G_rm,
                                                                         const float *__restrict__ Cc, const float *__restrict__ dVc,
                                                                         float *__restrict__ dKacc, bf16_t *__restrict__ dV,
                                                                         int n, int b, int t = 0, CrossSide cx = {})
{
    constexpr int KS = D / 16, CT = D / 32, NTHR = 64 * NW, OWN = 32 * NW;
    using Tile = LocTile<D, NTHR>;
    constexpr int BUF = 2 * Tile::BYTES + kLocT * 4, RC = CROSS_V ? R : 32;
    constexpr int CROSS_LDS = CROSS ? CrossSide::lds_bytes<RC, D>() : CROSS_V ? StateTiles<RC, D>::LDS_BYTES : 0;
    __shared__ __attribute__((aligned(16))) unsigned char stage[std::max(2 * BUF, CROSS_LDS)];
    const Tile T;
    const int x = T.x, h = T.h, tiles_per_unit = n / OWN;
    int wg = blockIdx.x;                                    // XCD-aware order, as in k_bwd_local_q
    if ((gridDim.x & 7) == 0) wg = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    const int u = wg / tiles_per_unit, j0 = (wg % tiles_per_unit) * OWN;
    const int jb = (j0 / b) * b;
    const size_t urow = (size_t)u * n;
    const int key0 = j0 + 32 * T.wave, key = key0 + x;
    f32x16 dk[CT], dv[CT];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) dk[ct] = dv[ct] = f32x16{0};
    if constexpr (CROSS) cx.rows<R, D, P, false>(V, nullptr, K, u, j0, n, b, t, stage, dk);
    if constexpr (CROSS_V) {
        const int l = j0 / b;
        if (l < t - 1) dv_rows<R, D, 1>(cx.M, cx.Zs, u, j0, t - 2 - l, n, t, stage, *(f32x16(*)[1][CT]) & dv);
        __syncthreads();                                    // the stage is free
    }
    bf16x8 kfr[KS], vfr[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        kfr[s] = *(const bf16x8 *)&K[(urow + key) * D + 16 * s + 8 * h];
        vfr[s] = *(const bf16x8 *)&V[(urow + key) * D + 16 * s + 8 * h];
    }
    const int first = (j0 - jb) / kLocT, ntiles = b / kLocT;
    const uint32_t stage0 = lds_address(stage);
    auto stage_tile = [&](int qt) {
        const uint32_t dst = stage0 + (qt & 1) * BUF;
        const size_t t0 = urow + jb + (size_t)qt * kLocT;
        T.stage(Q, t0, dst);
        T.stage(G_rm, t0, dst + Tile::BYTES);
        if (T.wave == 0) dma4_sbase(Cc + t0, (uint32_t)T.tid * 4, dst + 2 * Tile::BYTES);
    };
    auto tile = [&](auto diag_tag, int qt) {
        constexpr bool DIAG = decltype(diag_tag)::value;
        const unsigned char *qs = stage + (qt & 1) * BUF, *gs = qs + Tile::BYTES;
        const float *cs = (const float *)(qs + 2 * Tile::BYTES);
#pragma unroll
        for (int sub = 0; sub < 2; ++sub) {
            __builtin_amdgcn_sched_barrier(0);              // (halves interleaved do not fit the registers)
            f32x16 sc = {0}, dw;
#pragma unroll
            for (int gq = 0; gq < 4; ++gq) {                // dw starts at c of its row
                const f32x4 c4 = *(const f32x4 *)&cs[32 * sub + 8 * gq + 4 * h];
#pragma unroll
                for (int j = 0; j < 4; ++j) dw[4 * gq + j] = c4[j];
            }
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                sc = mfma32(T.rows(qs, sub, s), kfr[s], sc);
                dw = mfma32(T.rows(gs, sub, s), vfr[s], dw);
            }
            // key <= token t0 + 8 (v / 4) + 4 h + v % 4  <=>  8 (v / 4) + v % 4 >= lim
            const int lim = key - (jb + qt * kLocT + 32 * sub) - 4 * h;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const float sm = !DIAG || 8 * (v / 4) + (v % 4) >= lim ? sc[v] : 0.f;   // masked pairs: every power is 0
                const float pm1 = pow_n<P - 1>(sm);
                sc[v] = pm1 * sm;
                dw[v] = dw[v] * pm1;
            }
#pragma unroll
            for (int sp = 0; sp < 2; ++sp) {
                const bf16x8 pww = cvt8_from16(sc, 8 * sp), pwp = cvt8_from16(dw, 8 * sp);
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) {
                    dk[ct] = mfma32(T.columns(qs, sub, sp, ct), pwp, dk[ct]);
                    dv[ct] = mfma32(T.columns(gs, sub, sp, ct), pww, dv[ct]);
                }
            }
        }
    };
    auto sync = [&](int qt) {
        wait_vmem_le<0>();
        __syncthreads();
        if (qt + 1 < ntiles) stage_tile(qt + 1);
    };
    const int diag = (key0 - jb) / kLocT;                  // the tile that holds this wave's own keys
    stage_tile(first);
#pragma unroll 1
    for (int qt = first; qt < diag; ++qt) sync(qt);        // earlier tiles: only keep the barriers and copies going
    sync(diag);
    tile(std::true_type{}, diag);
#pragma unroll 1
    for (int qt = diag + 1; qt < ntiles; ++qt) {
        sync(qt);
        tile(std::false_type{}, qt);
        branch_wait();
    }
    static_assert(NW * RowsOut<D>::BYTES <= 2 * BUF, "the rows reuse the stage");
    __syncthreads();                                        // every wave is done with the last tile
    const RowsOut<D> rows_out(stage, T.wave, T.tid & 63);
    if constexpr (CROSS) {
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) dk[ct] *= (float)P;
        store_rows<D>(rows_out, dk, cx.dX + (urow + key0) * D);
        store_rows<D>(rows_out, dv, dV + (urow + key0) * D);
        return;
    }
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int gq = 0; gq < 4; ++gq) {
            const size_t held = held_quad<D>(urow + key, x, h, ct, gq);
            // (the p of p s^(p-1): a power of two, exact)
            const f32x4 k4 = {(float)P * dk[ct][4 * gq], (float)P * dk[ct][4 * gq + 1], (float)P * dk[ct][4 * gq + 2],
                              (float)P * dk[ct][4 * gq + 3]};
            *(f32x4 *)&dKacc[held] = k4;
            f32x4 c4 = {0.f, 0.f, 0.f, 0.f};                // (with CROSS_V the sums started from it)
            if constexpr (!CROSS_V) c4 = *(const f32x4 *)&dVc[held];
            const f32x4 v4 = {dv[ct][4 * gq] + c4[0], dv[ct][4 * gq + 1] + c4[1], dv[ct][4 * gq + 2] + c4[2],
                              dv[ct][4 * gq + 3] + c4[3]};
            rows_out.put(ct, gq, v4);
        }
    rows_out.store(dV + (urow + key - x) * D);
}

// ---- host ---------------------------------------------------------------------------------------
struct MfmaBwdWs {
    void *fwd;                                               // the forward workspace
    bf16_t *O, *MK, *G_rm, *Rg, *Rchi, *Rclo;
    float *Den, *Cc, *M8r, *ScPart, *dVc, *dQacc, *dKacc;
    // learned sketches: backward weight stream, what the row kernel leaves for the parameter
    // kernel (one side at a time), its workgroup sums, the per-unit parameter sums of both sides
    bf16_t *LB;
    LbStage sg;
    float *GB1, *part;
    size_t total;
};

MfmaBwdWs carve_bwd(const Problem &pb, void *ws)
{
    MfmaBwdWs w;
    const size_t rows = (size_t)pb.units * pb.n, R = pb.r, D = pb.d, tb = pb.t > 1 ? pb.t - 1 : 0;
    const size_t snaps = (size_t)pb.units * tb;
    size_t off = 0;
    char *base = (char *)ws;
    auto take = [&](size_t bytes) { char *p = base + off; off += align_up(bytes, 256); return (void *)p; };
    w.fwd = take(carve(pb, nullptr).total);
    w.O = (bf16_t *)take(rows * D * 2);
    w.MK = (bf16_t *)take(rows * R * 2);
    w.G_rm = (bf16_t *)take(rows * D * 2);
    w.Rg = (bf16_t *)take(snaps * R * R * D * 2);
    w.Rchi = (bf16_t *)take(snaps * R * R * 2);
    w.Rclo = (bf16_t *)take(snaps * R * R * 2);
    w.Den = (float *)take(rows * 4);
    w.Cc = (float *)take(rows * 4);
    w.M8r = (float *)take(rows * R * 4);
    w.ScPart = (float *)take(rows / 256 * R * R * 4);
    w.dVc = (float *)take(rows * D * 4);
    w.dQacc = (float *)take(rows * D * 4);
    w.dKacc = (float *)take(rows * D * 4);
    // Its least size is what it was with re-laid states and layouts of the rows beside them, the lower bound that the tests of
    // the interface state; nothing lies in what is more than the arrays above.
    off = std::max(off, align_up(carve(pb, nullptr).total, 256) + 2 * snaps * R * R * D * 2 + 5 * rows * D * 4);
    if (pb.learned) {
        const size_t sets = pb.per_head ? pb.heads : 1, nch = R / 4;
        w.LB = (bf16_t *)take(sets * 4 * nch * kLbSlot);
        w.sg.rows = rows;
        w.sg.XnR = (bf16_t *)take(rows * D * 2);
        w.sg.XnT = (bf16_t *)take(rows * D * 2);
        w.sg.A2R = (bf16_t *)take(2 * rows * R * 2);
        w.sg.A2T = (bf16_t *)take(2 * rows * R * 2);
        w.sg.DOR = (bf16_t *)take(2 * rows * R * 2);
        w.sg.DOT = (bf16_t *)take(2 * rows * R * 2);
        w.sg.DAR = (bf16_t *)take(2 * rows * R * 2);
        w.sg.DAT = (bf16_t *)take(2 * rows * R * 2);
        w.sg.ST = (float *)take(2 * 4 * rows * 4);
        w.GB1 = (float *)take(rows / 256 * 2 * 2 * D * 4);
        const LearnedSlices ls = learned_slices(pb.units, pb.n, !pb.per_head, pb.r, pb.g_len);
        w.part = (float *)take(2 * (size_t)std::max(pb.units, ls.units * ls.per_unit) * pb.g_len * 4);
    }
    w.total = off;
    return w;
}

// What a forward call leaves for the backward pass when asked to (psf_causal_attn_fwd_save): its
// whole workspace (m(Q), the states Z_l and S_l, the transposed sketch matrices), the
// denominators and m(K) as bf16 rows.
struct MfmaSaved {
    void *fwd;
    float *Den;
    bf16_t *MK;
    size_t total;
};

MfmaSaved carve_saved(const Problem &pb, void *ptr)
{
    MfmaSaved sv;
    const size_t rows = (size_t)pb.units * pb.n;
    size_t off = 0;
    char *base = (char *)ptr;
    auto take = [&](size_t bytes) { char *p = base + off; off += align_up(bytes, 256); return (void *)p; };
    sv.fwd = take(carve(pb, nullptr).total);
    sv.Den = (float *)take(rows * 4);
    sv.MK = (bf16_t *)take(rows * pb.r * 2);
    sv.total = off;
    return sv;
}

// saved / O_saved: null = run the forward pass again inside; otherwise what psf_causal_attn_fwd_save
// left and the output it wrote.
template <int R, int D, int P>
psf_status attn_bwd_impl(const Problem &pb, const void *Q, const void *K, const void *V, const void *G,
                         const void *dO, void *dQ, void *dK, void *dV, void *ws, hipStream_t s, StageTimer *tm,
                         void *saved = nullptr, const void *O_saved = nullptr, float *dG = nullptr)
{
    constexpr int TT = D == 64 ? 2 : 1;                     // 32-token tiles per wave in the cross-block kernels
    constexpr int DT = D == 64 && R == 64 ? 2 : 1;          // the same in k_bwd_dm (see StateTiles::OCC)
    constexpr int NWL = 4;                                  // waves per in-block workgroup: 256 own rows share a streamed tile
    MfmaBwdWs w = carve_bwd(pb, ws);
    MfmaWs f = carve(pb, w.fwd);
    const size_t rows = (size_t)pb.units * pb.n;
    const bf16_t *q = (const bf16_t *)Q, *k = (const bf16_t *)K, *v = (const bf16_t *)V;
    // in-block rule of Section 3.1 (r = d = 64 only): the in-block kernels take the sketches
    // m(Q), m(K) in place of Q, K with exponent 2 and leave the in-block part of dm
    const bool ls = !pb.local_exact;
    if (ls && !(R == D && P == 4)) return PSF_ERR_UNSUPPORTED;
    if (pb.learned && !(D == 64 && P == 4)) return PSF_ERR_UNSUPPORTED;
    if (pb.learned && ls) return PSF_ERR_UNSUPPORTED;
    psf_status st;
    if (saved) {
        const MfmaSaved sv = carve_saved(pb, saved);
        f = carve(pb, sv.fwd);
        w.Den = sv.Den;
        w.MK = sv.MK;
        w.O = (bf16_t *)O_saved;                           // read only
    } else {
        // forward pass again: O, the denominators, m(Q), m(K), the states Z_l and S_l
        st = attn_impl<D, R, P>(pb, Q, K, V, G, w.O, w.fwd, s, nullptr, w.Den, w.MK);
        if (st != PSF_OK) return st;
        if (pb.learned) {
            // (the learned key-side sketch kernel writes the state kernel's octets only)
            if (!learned_on_mfma(pb)) return PSF_ERR_UNSUPPORTED;
            const size_t count4 = rows * R / 4;
            hipLaunchKernelGGL((k_octets_to_rows<R>), dim3((unsigned)((count4 + kWg - 1) / kWg)), dim3(kWg), 0, s,
                               f.MK8, w.MK, count4);
            PSF_LAUNCH_CHECK();
        }
    }
    if (tm) tm->mark();
    const bf16_t *rq = ls ? f.MQ : q, *rk = ls ? w.MK : k;  // the rows the in-block weights are made of
    // g, c, layouts
    hipLaunchKernelGGL((k_bwd_prep<D>), dim3((unsigned)(rows / (kWg / (D / 8) * 4))), dim3(kWg), 0, s, (const bf16_t *)dO,
                       w.O, w.Den, w.G_rm, w.Cc);
    PSF_LAUNCH_CHECK();
    if (tm) tm->mark();
    // mirror states R_l (the forward state kernel on block-reversed inputs)
    if (pb.t > 1) {
        hipLaunchKernelGGL((k_bwd_qoct<R>), dim3((unsigned)(rows / 256)), dim3(kWg), 0, s, f.MQ, w.Cc, w.M8r,
                           w.ScPart, pb.n, pb.b, pb.t);
        PSF_LAUNCH_CHECK();
        st = launch_state<D, R>(pb, w.M8r, w.G_rm, (size_t)pb.n * D, 1, w.Rg, s);
        if (st != PSF_OK) return st;
    }
    if (tm) tm->mark();
    if constexpr (D == 64 && P == 4 && R == 32) {
        if (!pb.learned) {
            // both parts of a side in one kernel, each a stage of its own: the two that divide them otherwise are empty
            if (tm) {
                tm->mark();
                tm->mark();
            }
            const unsigned main = (unsigned)(rows / (32 * NWL));
            const DenScan den = {w.ScPart, w.Rchi, w.Rclo, pb.b / 256, pb.n / 256, (int)main};
            const int ph = pb.per_head ? 1 : 0;
            const CrossSide cq = {f.MQ, f.Zg, f.Shi, f.Slo, f.Gt, (const bf16_t *)G, (bf16_t *)dQ, pb.heads, ph, pb.g_len};
            const CrossSide ck = {w.MK, w.Rg, w.Rchi, w.Rclo, f.Gt, (const bf16_t *)G, (bf16_t *)dK, pb.heads, ph, pb.g_len};
            hipLaunchKernelGGL((k_bwd_local_q<P, NWL, D, R, true>), dim3(main + (pb.t > 1 ? (unsigned)(pb.units * (R * R / kWg)) : 0u)),
                               dim3(64 * NWL), 0, s, q, k, v, w.G_rm, w.Cc, nullptr, pb.n, pb.b, pb.t, den, cq);
            PSF_LAUNCH_CHECK();
            if (tm) tm->mark();
            hipLaunchKernelGGL((k_bwd_local_k<P, NWL, D, R, true>), dim3(main), dim3(64 * NWL), 0, s, q, k, v, w.G_rm, w.Cc,
                               nullptr, nullptr, (bf16_t *)dV, pb.n, pb.b, pb.t, ck);
            PSF_LAUNCH_CHECK();
            if (tm) tm->mark();
            return PSF_OK;
        }
    }
    // in-block parts
    {
        const unsigned main = (unsigned)(rows / (32 * NWL));
        const DenScan den = {w.ScPart, w.Rchi, w.Rclo, pb.b / 256, pb.n / 256, (int)main};
        const unsigned grid = main + (pb.t > 1 ? (unsigned)(pb.units * (R * R / kWg)) : 0u);
        if constexpr (R == D && P == 4) {
            if (ls) {
                hipLaunchKernelGGL((k_bwd_local_q<2, NWL, D, R>), dim3(grid), dim3(64 * NWL), 0, s, rq, rk, v, w.G_rm,
                                   w.Cc, w.dQacc, pb.n, pb.b, pb.t, den);
                PSF_LAUNCH_CHECK();
            }
        }
        if (!ls) {
            hipLaunchKernelGGL((k_bwd_local_q<P, NWL, D, R>), dim3(grid), dim3(64 * NWL), 0, s, q, k, v, w.G_rm, w.Cc,
                               w.dQacc, pb.n, pb.b, pb.t, den);
            PSF_LAUNCH_CHECK();
        }
    }
    {
        // dV: the cross-block part first, the in-block kernel adds to it
        const unsigned gridc = (unsigned)(rows / (128 * TT)), grid = (unsigned)(rows / (32 * NWL));
        constexpr bool APART = D == 64 && R == 64;          // two row tiles a wave share a state's operands there
        const CrossSide cv = {w.MK, w.Rg, nullptr, nullptr, nullptr, nullptr, nullptr, 0, 0, 0};
        if constexpr (APART) {
            hipLaunchKernelGGL((k_bwd_dvc<R, D, TT>), dim3(gridc), dim3(kWg), 0, s, w.MK, w.Rg, w.dVc, pb.n, pb.b, pb.t);
            PSF_LAUNCH_CHECK();
        }
        if constexpr (R == D && P == 4) {
            if (ls) {
                hipLaunchKernelGGL((k_bwd_local_k<2, NWL, D>), dim3(grid), dim3(64 * NWL), 0, s, rq, rk, v, w.G_rm, w.Cc,
                                   w.dVc, w.dKacc, (bf16_t *)dV, pb.n, pb.b);
                PSF_LAUNCH_CHECK();
            }
        }
        if (!ls) {
            hipLaunchKernelGGL((k_bwd_local_k<P, NWL, D, R, false, !APART>), dim3(grid), dim3(64 * NWL), 0, s, q, k, v, w.G_rm,
                               w.Cc, w.dVc, w.dKacc, (bf16_t *)dV, pb.n, pb.b, pb.t, cv);
            PSF_LAUNCH_CHECK();
        }
    }
    if (tm) tm->mark();
    // cross-block parts of dm(q), dm(k), then through the sketch together with the in-block parts
    {
        const unsigned grid = (unsigned)(rows / (128 * DT));
        const int ph = pb.per_head ? 1 : 0;
        if constexpr (R == D && P == 4) {
            if (ls) {
                hipLaunchKernelGGL((k_bwd_dm<R, D, true, DT, true>), dim3(grid), dim3(kWg), 0, s, f.MQ, w.G_rm, w.Cc,
                                   f.Zg, f.Shi, f.Slo, q, f.Gt, (const bf16_t *)G, w.dQacc, (bf16_t *)dQ, pb.n, pb.b,
                                   pb.t, pb.heads, ph, pb.g_len);
                PSF_LAUNCH_CHECK();
                hipLaunchKernelGGL((k_bwd_dm<R, D, false, DT, true>), dim3(grid), dim3(kWg), 0, s, w.MK, v, w.Cc, w.Rg,
                                   w.Rchi, w.Rclo, k, f.Gt, (const bf16_t *)G, w.dKacc, (bf16_t *)dK, pb.n, pb.b, pb.t,
                                   pb.heads, ph, pb.g_len);
                PSF_LAUNCH_CHECK();
            }
        }
        constexpr bool FUSED = D == 64 && P == 4;           // Algorithm 1's reverse inside k_bwd_dm
        if constexpr (FUSED) {
        if (pb.learned) {
            // dm as fp32 rows (in the buffer of the mirror-state octets, consumed by now), then
            // through the networks: one side after the other, the staging buffers serve both
            const int sets = pb.per_head ? pb.heads : 1;
            const unsigned grid_rows = (unsigned)(rows / 256);
            const LearnedSlices sl = learned_slices(pb.units, pb.n, !pb.per_head, pb.r, pb.g_len);
            const int slices = sl.units * sl.per_unit, slice_rows = sl.n / sl.per_unit;
            const unsigned grid_par = (unsigned)(slices * 2 * (R / 4 / 4));
            hipLaunchKernelGGL((k_learned_bwd_prep<R>), dim3(4 * (R / 4), sets), dim3(kWg), 0, s, (const bf16_t *)G,
                               pb.g_len, w.LB);
            PSF_LAUNCH_CHECK();
            for (int side = 0; side < 2; ++side) {
                if (side == 0)
                    hipLaunchKernelGGL((k_bwd_dm<R, D, true, DT, false, true>), dim3(grid), dim3(kWg), 0, s, f.MQ, w.G_rm,
                                       w.Cc, f.Zg, f.Shi, f.Slo, q, nullptr, nullptr, nullptr, nullptr, pb.n, pb.b, pb.t,
                                       pb.heads, ph, pb.g_len, w.M8r);
                else
                    hipLaunchKernelGGL((k_bwd_dm<R, D, false, DT, false, true>), dim3(grid), dim3(kWg), 0, s, w.MK, v,
                                       w.Cc, w.Rg, w.Rchi, w.Rclo, k, nullptr, nullptr, nullptr, nullptr, pb.n, pb.b, pb.t,
                                       pb.heads, ph, pb.g_len, w.M8r);
                PSF_LAUNCH_CHECK();
                const bf16_t *xr = side == 0 ? q : k;
                const float *base = side == 0 ? w.dQacc : w.dKacc;
                bf16_t *dx = (bf16_t *)(side == 0 ? dQ : dK);
                if (dG) {
                    hipLaunchKernelGGL((k_learned_bwd_rows<R, true>), dim3(grid_rows), dim3(512), 0, s, xr, w.M8r, base,
                                       f.LW, f.C1, f.LVp, w.LB, (const bf16_t *)G, pb.g_len, dx, w.sg, w.GB1, pb.n,
                                       pb.heads, ph);
                    PSF_LAUNCH_CHECK();
                    float *part = w.part + (size_t)side * slices * pb.g_len;
                    hipLaunchKernelGGL((k_learned_bwd_params<R, 0>), dim3(grid_par), dim3(kWg), 0, s, w.sg,
                                       (const bf16_t *)G, pb.g_len, f.C1, w.GB1, part, pb.g_len, sl.n, slice_rows,
                                       pb.heads, ph);
                    PSF_LAUNCH_CHECK();
                    hipLaunchKernelGGL((k_learned_bwd_params<R, 1>), dim3(grid_par), dim3(kWg), 0, s, w.sg,
                                       (const bf16_t *)G, pb.g_len, f.C1, w.GB1, part, pb.g_len, sl.n, slice_rows,
                                       pb.heads, ph);
                    PSF_LAUNCH_CHECK();
                } else {
                    hipLaunchKernelGGL((k_learned_bwd_rows<R, false>), dim3(grid_rows), dim3(512), 0, s, xr, w.M8r, base,
                                       f.LW, f.C1, f.LVp, w.LB, (const bf16_t *)G, pb.g_len, dx, w.sg, w.GB1, pb.n,
                                       pb.heads, ph);
                    PSF_LAUNCH_CHECK();
                }
            }
            if (dG) {
                hipLaunchKernelGGL(k_learned_bwd_reduce, dim3((unsigned)((pb.g_len + kWg - 1) / kWg), sets), dim3(kWg), 0, s,
                                   w.part, dG, pb.g_len, sl.units, sl.per_unit, pb.heads, ph);
                PSF_LAUNCH_CHECK();
            }
        } else if constexpr (R != 32) {                     // (r = 32: done above)
            if (!ls) {
                hipLaunchKernelGGL((k_bwd_dm<R, D, true, DT>), dim3(grid), dim3(kWg), 0, s, f.MQ, w.G_rm, w.Cc, f.Zg, f.Shi,
                                   f.Slo, q, f.Gt, (const bf16_t *)G, w.dQacc, (bf16_t *)dQ, pb.n, pb.b, pb.t, pb.heads, ph,
                                   pb.g_len);
                PSF_LAUNCH_CHECK();
                hipLaunchKernelGGL((k_bwd_dm<R, D, false, DT>), dim3(grid), dim3(kWg), 0, s, w.MK, v, w.Cc, w.Rg, w.Rchi,
                                   w.Rclo, k, f.Gt, (const bf16_t *)G, w.dKacc, (bf16_t *)dK, pb.n, pb.b, pb.t, pb.heads, ph,
                                   pb.g_len);
                PSF_LAUNCH_CHECK();
            }
        }
        } else {
            // d = 128 or degree 8: dm as fp32 rows (in the buffer of the mirror-state octets, consumed
            // by now), then Algorithm 1's reverse as a pass of its own, one side after the other
            for (int side = 0; side < 2; ++side) {
                if (side == 0)
                    hipLaunchKernelGGL((k_bwd_dm<R, D, true, DT, false, true>), dim3(grid), dim3(kWg), 0, s, f.MQ, w.G_rm,
                                       w.Cc, f.Zg, f.Shi, f.Slo, q, nullptr, nullptr, nullptr, nullptr, pb.n, pb.b, pb.t,
                                       pb.heads, ph, pb.g_len, w.M8r);
                else
                    hipLaunchKernelGGL((k_bwd_dm<R, D, false, DT, false, true>), dim3(grid), dim3(kWg), 0, s, w.MK, v,
                                       w.Cc, w.Rg, w.Rchi, w.Rclo, k, nullptr, nullptr, nullptr, nullptr, pb.n, pb.b, pb.t,
                                       pb.heads, ph, pb.g_len, w.M8r);
                PSF_LAUNCH_CHECK();
                hipLaunchKernelGGL((k_bwd_sketch_rows<D, R, P>), dim3((unsigned)(rows / 128)), dim3(kWg), 0, s,
                                   side == 0 ? q : k, f.Gt, (const bf16_t *)G, w.M8r, side == 0 ? w.dQacc : w.dKacc,
                                   (bf16_t *)(side == 0 ? dQ : dK), pb.n, pb.heads, ph, pb.g_len);
                PSF_LAUNCH_CHECK();
            }
        }
    }
    if (tm) tm->mark();
    return PSF_OK;
}
