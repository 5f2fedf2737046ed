// bwd_small.hpp -- the block-form backward for noisy blocks of nl = 1, 2, 4, 8 or 16 positions
// (included by bwd_kernels.hip): clean chunks of 32 positions, each with the 32 / nl noisy
// blocks inside it, where one padded unit per noisy block would do 32 / nl times the work and
// walk 32 / nl times the serial steps.
//
// Let a chunk start from S0 with the clean Delta (rows Delta_j), and let the noisy block of
// row t start at row p = p(t).  Its seed is the clean state before p,
//     seed_t = gp_t S0 + sum_(j < p) m_tj k_j Delta_j^T,  gp_t = gamma_(p-1), m_tj = gamma_(p-1) / gamma_j
// (gp = 1 and no sum for p = 0), so no noisy block needs a state of its own:
//     X~ = K~ seed = gp (K~ S0) + Nk Delta,  Nk = (K~ K^T) o m;  R~ = V~ - Gamma~ X~;  Delta~ = T~ R~
// with T~ block diagonal.  With Pn = (K~ Q~^T) restricted to a noisy block,
//     dDelta~ = D~ s Pn dO~,  dR~ = T~^T dDelta~ = dV~,
// and the gradient of a noisy block's seed is a sum of outer products of its rows,
//     sum_t q~_t a_t^T + k~_t b_t^T,  a_t = s gamma~_n dO~_t,  b_t = -gamma~_t dR~_t.
// seed_t a_t = gp_t S0 a_t + sum_j FA_tj k_j with FA_tj = m_tj (a_t . Delta_j), likewise FB with b:
//     dQ~ = seed a + dPh K~,  dK~ = seed b + dPh^T Q~ + (dKK + dKK^T) K~,  dPh = s (dO~ Delta~^T) D~.
// To the clean chunk the rows (q~_t, a_t), (k~_t, b_t) are further readouts of the state before
// p(t): they add to its gradients
//     dDelta += XD = Nq^T a + Nk^T b  (Nq = (Q~ K^T) o m),   dK += FA^T Q~ + FB^T K~,
//     dS0 += Q~^T gp a + K~^T gp b,   and, with W = Nq o FA' + Nk o FB' (FA', FB' before the mask),
//     gp_t (q~_t . S0 a_t + k~_t . S0 b_t) + sum_j W_tj on the cumulative gate of position p(t) - 1,
//     - W_tj on that of j.
// dg is the sum of these from the chunk's end back, where every W_tj cancels but for the positions
// between j and p: both come from one W_tj, and j = p - 1 is in neither, since under a strong decay
// what is left is of the decay's order (a row sum formed as q~ . (FA K), with FA rounded to fp16,
// left 2^-11 of W whatever the gates: a tenth of dg at g = -5).
// This kernel writes XD for the clean pass, starts the clean dk
// and dg with its shares, and runs the clean preparation (the dh-independent part of dS0, U K)
// with dDelta's share XD included; the clean pass then adds to dk and dg.
//
// Measured at 2048 (chunk, head) units (1 x 4096 tokens, 16 heads), nl = 4: 189 us, against
// 621 us for 16384 padded units of the per-block kernel (1110 us before that ran twice on a CU).
// Bound by the latency of its phases: one workgroup per CU (159 KB of LDS), persistent, the
// next unit's rows in flight during the second half of each unit.  Everything that needs only
// a wave's own 16 columns runs without a barrier from the solves to the chunk's c term.

struct SmallSmem {
    _Float16 S0[DD * LDH];
    _Float16 Q[NP * LDH];     // clean q; then, fp32, T~ (later dA) and M~^T
    _Float16 K[NP * LDH];
    _Float16 V[NP * LDH];     // clean v, then Delta~
    _Float16 dO[NP * LDH];    // clean dO; then, fp32, dT and W
    _Float16 Dl[NP * LDH];    // clean Delta
    _Float16 Qn[NP * LDH], Kn[NP * LDH];
    _Float16 Rn[NP * LDH];    // noisy v, then R~
    _Float16 dOn[NP * LDH];
    _Float16 dDn[NP * LDH];   // dDelta~
    _Float16 Bn[NP * LDH];    // b = -Gamma~ dR~
    _Float16 Mc[NP * LDM], Mn[NP * LDM];   // (I + A)^-1 of the clean chunk and of the noisy blocks
    _Float16 Ph[NP * LDM];    // clean P; then dKK + dKK^T
    _Float16 Pn[NP * LDM];    // Pn; then dPh
    _Float16 Nq[NP * LDM], Nk[NP * LDM], FA[NP * LDM], FB[NP * LDM];
    float KK[NP * LDF];       // K~ K~^T
    float G[NP], G2[NP], gam[NP], bet[NP];         // the clean chunk's cumulative gates
    float Gn[NP], G2n[NP], gamn[NP], betn[NP];     // cumulative inside each noisy block
    float Dn[NP], sg[NP];     // gamma~_n / gamma~, s gamma~_n
    float Gp[NP], gp[NP];     // log gamma_(p-1), gamma_(p-1)
    float dB[NP];
    // per-wave partial sums over columns, added in a fixed order at the end: the gate terms of
    // dA, gp q~ . S0 a, gp k~ . S0 b, dDelta~ . Delta~, and the column sums of W
    float part[kWaves][NP], pA[kWaves][NP], pB[kWaves][NP], pW[kWaves][NP], pC[kWaves][NP];
    // row sums of W, a's and b's, over 16 columns each, but for column p - 1, which is in pD
    float pR[2][2][NP], pD[2][NP];
};
static_assert(sizeof(SmallSmem) <= 160 * 1024, "one workgroup's LDS");
static_assert(2 * NP * LDF * 4 <= NP * LDH * 2, "two fp32 matrices in the room of a row block");

// One unit's inputs in registers.
template <typename Od> struct SmallRows {
    BlockRows<Od, true> c, n;
    SeedRegs seed;
};

template <typename Od> __global__ void __launch_bounds__(512) bdgdn_bwd_small_kernel(BwdArgs a)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    SmallSmem &sm = *reinterpret_cast<SmallSmem *>(smem_raw);
    float *const Tf = reinterpret_cast<float *>(sm.Q), *const Mt = Tf + NP * LDF;
    float *const dT = reinterpret_cast<float *>(sm.dO), *const Wm = dT + NP * LDF;
    _Float16 *const Dln = sm.V, *const Wh = sm.Ph, *const dPh = sm.Pn;
    const int nl = a.nl, r = a.h_v / a.h_qk;
    const float s = a.scale, sigma = a.range[0], inv = a.range[1];
    const f32x4 z = {0.f, 0.f, 0.f, 0.f};
    const long qks = (long)a.h_qk * DD, vs = (long)a.h_v * DD;
    // workgroup w takes the (chunk, q/k head) groups w, w + gridDim.x, ..., each as its r
    // consecutive units (unit_of)
    auto next_unit = [&](long t) { return (t + 1) % r ? t + 1 : t + 1 + (long)(gridDim.x - 1) * r; };
    auto load = [&](long t, int tid, SmallRows<Od> &x) {
        long gb, p0;
        int h, hq, vi, n, nvalid;
        const long uw = unit_of(a, t, gb, h, hq, vi);
        block_unit(a, gb, n, p0, nvalid);
        x.c = load_block<Od, true>(stream_ptrs<Od>(a, false, p0, h, hq), a.h_qk, a.h_v, nvalid, tid);
        x.n = load_block<Od, true>(stream_ptrs<Od>(a, true, p0, h, hq), a.h_qk, a.h_v, nvalid, tid);
        x.seed = load_seed(a.seeds + (size_t)uw * DD * DD, tid);
    };
    SmallRows<Od> in;
    long u = (long)blockIdx.x * r;
    load(u, threadIdx.x, in);
    for (;;) {
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));   // lane-dependent addresses recomputed per unit, not kept live
        const int lane = tid & 63, g4 = lane >> 4, rr = lane & 15;
        const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), c0 = 16 * wave, col = c0 + rr;
        long gb, p0;
        int h, hq, vi, seq, nvalid;
        const long uw = unit_of(a, u, gb, h, hq, vi);
        block_unit(a, gb, seq, p0, nvalid);
        const StreamPtrs pc = stream_ptrs<Od>(a, false, p0, h, hq), pn = stream_ptrs<Od>(a, true, p0, h, hq);
        const bool add_qk = vi > 0;
        // ---- the unit's rows, seed and gates into LDS
        store_rows(sm.Q, in.c.q, tid);
        store_rows(sm.K, in.c.k, tid);
        store_rows(sm.V, in.c.v, tid);
        store_rows(sm.dO, in.c.dout, tid, sigma);
        store_rows(sm.Qn, in.n.q, tid);
        store_rows(sm.Kn, in.n.k, tid);
        store_rows(sm.Rn, in.n.v, tid);
        store_rows(sm.dOn, in.n.dout, tid, sigma);
        store_seed(sm.S0, in.seed, tid);
        if (tid < NP) {
            sm.bet[tid] = in.c.b;
            sm.G[tid] = ut::gate_floor(in.c.g);
            sm.betn[tid] = in.n.b;
            sm.Gn[tid] = ut::gate_floor(in.n.g);
        }
        if (tid < kWaves * NP) {
            sm.part[tid / NP][tid % NP] = 0.f;
            sm.pC[tid / NP][tid % NP] = 0.f;
        }
        __syncthreads();
        if (wave == 0) {
            const float x = ut::scan32(lane < NP ? sm.G[lane] : 0.f, lane);
            const int p = lane & ~(nl - 1);
            const float before = __shfl(x, p > 0 ? p - 1 : 0);
            if (lane < NP) {
                sm.G[lane] = x;
                sm.G2[lane] = x * kLog2e;
                sm.gam[lane] = ex(x);
                sm.Gp[lane] = p > 0 ? before : 0.f;
                sm.gp[lane] = p > 0 ? ex(before) : 1.f;
            }
        } else if (wave == 1) {
            // inside each noisy block: a scan over its nl positions, and its total
            float x = lane < NP ? sm.Gn[lane] : 0.f;
            for (int o = 1; o < nl; o <<= 1) {
                const float y = __shfl_up(x, o);
                if ((lane & (nl - 1)) >= o) x += y;
            }
            const float end = __shfl(x, lane | (nl - 1));
            if (lane < NP) {
                sm.Gn[lane] = x;
                sm.G2n[lane] = x * kLog2e;
                sm.gamn[lane] = ex(x);
                sm.Dn[lane] = ex(end - x);
                sm.sg[lane] = s * ex(end);
            }
        }
        __syncthreads();
        // ---- the solves (waves 0, 1) and the Gram tiles with the clean keys and inside the
        // noisy blocks (waves 2 .. 7)
        if (wave < 2) {
            ut::QE kq[2][DD / 16];
            const _Float16 *K = wave == 0 ? sm.K : sm.Kn;
#pragma unroll
            for (int rb = 0; rb < 2; ++rb)
#pragma unroll
                for (int kb = 0; kb < DD / 16; ++kb)
                    kq[rb][kb] = *reinterpret_cast<const f16x4 *>(K + (16 * rb + rr) * LDH + 16 * kb + 4 * g4);
            ut::Consts cs;
            ut::make_consts(cs, lane);
            // the clean chunk is one group of 32
            ut::solve_t<2, DD / 16, false, true>(kq, wave == 0 ? sm.G2 : sm.G2n, wave == 0 ? sm.bet : sm.betn,
                                                 wave == 0 ? sm.Mc : sm.Mn, LDM, cs, lane, wave == 0 ? NP : nl);
        } else {
            for (int e = wave - 2; e < 20; e += 6) {
                const int gram = e >> 2, m0 = 16 * ((e >> 1) & 1), n0 = 16 * (e & 1), i = n0 + rr;
                const _Float16 *A = gram == 0 ? sm.Q : (gram == 2 ? sm.Qn : sm.Kn);
                const _Float16 *B = gram < 3 ? sm.K : (gram == 3 ? sm.Qn : sm.Kn);
                const f32x4 c = tile_mma<_Float16, DD>(z, A + m0 * LDH, LDH, B + n0 * LDH, LDH, lane);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int t = m0 + 4 * g4 + j;
                    if (gram == 0) {
                        sm.Ph[t * LDM + i] = (_Float16)(i <= t ? c[j] * ex(sm.G[t] - sm.G[i]) : 0.f);
                    } else if (gram == 4) {
                        sm.KK[t * LDF + i] = c[j];
                    } else if (gram == 3) {
                        sm.Pn[t * LDM + i] = (_Float16)((t ^ i) < nl ? c[j] : 0.f);
                    } else {
                        const float m = i < (t & ~(nl - 1)) ? ex(sm.Gp[t] - sm.G[i]) : 0.f;
                        (gram == 1 ? sm.Nk : sm.Nq)[t * LDM + i] = (_Float16)(c[j] * m);
                    }
                }
            }
        }
        // R = V - Gamma K S0 (operands of T R) and K~ S0, this wave's columns
        f16x4 rq[2];
        f32x4 xn[2];
        {
            f16x4 s0q[8];
#pragma unroll
            for (int kb = 0; kb < 8; ++kb) s0q[kb] = op_tr(sm.S0, LDH, 16 * kb, c0, lane);
#pragma unroll
            for (int tm = 0; tm < 2; ++tm) {
                f32x4 x = z;
                xn[tm] = z;
#pragma unroll
                for (int kb = 0; kb < 8; kb += 2) {
                    x = mfma2(op_row(sm.K, LDH, 16 * tm, 16 * kb, lane), op_row(sm.K, LDH, 16 * tm, 16 * kb + 16, lane),
                              s0q[kb], s0q[kb + 1], x);
                    xn[tm] = mfma2(op_row(sm.Kn, LDH, 16 * tm, 16 * kb, lane),
                                   op_row(sm.Kn, LDH, 16 * tm, 16 * kb + 16, lane), s0q[kb], s0q[kb + 1], xn[tm]);
                }
                rq[tm] = h4(f4(op_tr(sm.V, LDH, 16 * tm, c0, lane)) - ld4(sm.gam + 16 * tm + 4 * g4) * x);
            }
        }
        __syncthreads();
        // ---- this wave's columns, without a barrier: Delta, R~, Delta~, dDelta~, dV~, b, XD, the
        // clean preparation
        float roww[2][4];   // dDelta~ . Delta~ of row 16 tm + 4 g + j
        {
            const f32x4 b0 = ld4(sm.bet + 4 * g4), b1 = ld4(sm.bet + 16 + 4 * g4);
            const f32x4 bn0 = ld4(sm.betn + 4 * g4), bn1 = ld4(sm.betn + 16 + 4 * g4);
            // a (not b, a result of other fp16 products) in two fp16 parts; ga, gb: gp a, gp b
            f16x4 dl[2], rn[2], dd[2], aq[2], al[2], bq[2], ga[2], gal[2], gb[2];
            f32x4 dn[2];
#pragma unroll
            for (int tm = 0; tm < 2; ++tm) {
                dl[tm] = h4(mfma2(scale4(op_row(sm.Mc, LDM, 16 * tm, 0, lane), b0),
                                  scale4(op_row(sm.Mc, LDM, 16 * tm, 16, lane), b1), rq[0], rq[1], z));
                put_tile(sm.Dl, LDH, 16 * tm, col, dl[tm], g4);
            }
#pragma unroll
            for (int tm = 0; tm < 2; ++tm) {
                const f32x4 x = apply(sm.Nk, 16 * tm, dl, ld4(sm.gp + 16 * tm + 4 * g4) * xn[tm], lane);
                rn[tm] = h4(f4(op_tr(sm.Rn, LDH, 16 * tm, c0, lane)) - ld4(sm.gamn + 16 * tm + 4 * g4) * x);
            }
            const f16x4 dob[2] = {op_tr(sm.dOn, LDH, 0, c0, lane), op_tr(sm.dOn, LDH, 16, c0, lane)};
#pragma unroll
            for (int tm = 0; tm < 2; ++tm) {
                put_tile(sm.Rn, LDH, 16 * tm, col, rn[tm], g4);
                dn[tm] = mfma2(scale4(op_row(sm.Mn, LDM, 16 * tm, 0, lane), bn0),
                               scale4(op_row(sm.Mn, LDM, 16 * tm, 16, lane), bn1), rn[0], rn[1], z);
                put_tile(Dln, LDH, 16 * tm, col, h4(dn[tm]), g4);
                const f32x4 d = s * ld4(sm.Dn + 16 * tm + 4 * g4) * apply(sm.Pn, 16 * tm, dob, z, lane);
                dd[tm] = h4(d);
                put_tile(sm.dDn, LDH, 16 * tm, col, dd[tm], g4);
#pragma unroll
                for (int j = 0; j < 4; ++j) roww[tm][j] = d[j] * dn[tm][j];
                // a = s gamma~_n dO~ differs by block, so that it can't be put on a product of dO~ as the
                // block by block backward does
                const f32x4 x = ld4(sm.sg + 16 * tm + 4 * g4) * f4(dob[tm]);
                aq[tm] = h4(x);
                al[tm] = h4(x - f4(aq[tm]));
                const f32x4 y = ld4(sm.gp + 16 * tm + 4 * g4) * x;
                ga[tm] = h4(y);
                gal[tm] = h4(y - f4(ga[tm]));
            }
#pragma unroll
            for (int tm = 0; tm < 2; ++tm) {   // dR~ = T~^T dDelta~ (T~^T_ri = beta~_r M~_ir)
                const float b = sm.betn[16 * tm + rr];
                const f32x4 bb = {b, b, b, b};
                const f32x4 c = mfma2(scale4(op_tr(sm.Mn, LDM, 0, 16 * tm, lane), bb),
                                      scale4(op_tr(sm.Mn, LDM, 16, 16 * tm, lane), bb), dd[0], dd[1], z);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int t = 16 * tm + 4 * g4 + j;
                    if (t < nvalid) pn.dv[(long)t * vs + col] = c[j] * inv;
                }
                const f32x4 x = -ld4(sm.gamn + 16 * tm + 4 * g4) * c;
                bq[tm] = h4(x);
                gb[tm] = h4(ld4(sm.gp + 16 * tm + 4 * g4) * x);
                put_tile(sm.Bn, LDH, 16 * tm, col, bq[tm], g4);
            }
            // XD (for the clean pass), Y = s P^T dO + XD, -Gamma T^T Y
            const f16x4 doc[2] = {op_tr(sm.dO, LDH, 0, c0, lane), op_tr(sm.dO, LDH, 16, c0, lane)};
            f16x4 yq[2], drq[2], sd[2];
            f32x4 *xd = reinterpret_cast<f32x4 *>(a.xd + (size_t)uw * NP * DD) + wave * 64 + lane;
#pragma unroll
            for (int tm = 0; tm < 2; ++tm) {
                f32x4 x = apply_t(sm.Nq, LDM, 16 * tm, aq, z, lane);
                x = apply_t(sm.Nq, LDM, 16 * tm, al, x, lane);
                x = apply_t(sm.Nk, LDM, 16 * tm, bq, x, lane);
                xd[tm * 8 * 64] = x;
                yq[tm] = h4(s * apply_t(sm.Ph, LDM, 16 * tm, doc, z, lane) + x);
            }
#pragma unroll
            for (int tm = 0; tm < 2; ++tm) {
                const float b = sm.bet[16 * tm + rr];
                const f32x4 bb = {b, b, b, b}, gm = ld4(sm.gam + 16 * tm + 4 * g4);
                const f32x4 c = mfma2(scale4(op_tr(sm.Mc, LDM, 0, 16 * tm, lane), bb),
                                      scale4(op_tr(sm.Mc, LDM, 16, 16 * tm, lane), bb), yq[0], yq[1], z);
                drq[tm] = h4(-gm * c);
                sd[tm] = scale4(doc[tm], s * gm);
            }
            // c term: K^T (-Gamma dR0) + Q^T (s Gamma dO) + Q~^T (gp a) + K~^T (gp b)
            f16x4 *ct = reinterpret_cast<f16x4 *>(a.cterm + (size_t)uw * DD * DD) + wave * 64 + lane;
#pragma unroll
            for (int tm = 0; tm < 8; ++tm) {
                f32x4 c = apply_t(sm.K, LDH, 16 * tm, drq, z, lane);
                c = apply_t(sm.Q, LDH, 16 * tm, sd, c, lane);
                c = apply_t(sm.Qn, LDH, 16 * tm, ga, c, lane);
                c = apply_t(sm.Qn, LDH, 16 * tm, gal, c, lane);
                ct[tm * 8 * 64] = h4(apply_t(sm.Kn, LDH, 16 * tm, gb, c, lane));
            }
            // U K = Gamma diag(beta) M^T (D K)
            const float Ge = sm.G[NP - 1];
            f16x4 kd[2];
#pragma unroll
            for (int tm = 0; tm < 2; ++tm) {
                f32x4 d;
#pragma unroll
                for (int j = 0; j < 4; ++j) d[j] = ex(Ge - sm.G[16 * tm + 4 * g4 + j]);
                kd[tm] = scale4(op_tr(sm.K, LDH, 16 * tm, c0, lane), d);
            }
            _Float16 *uk = a.uk + (size_t)uw * NP * DD;
#pragma unroll
            for (int tm = 0; tm < 2; ++tm) {
                // the transpose from the swapped operands, in the scan's order
                const float f = sm.gam[16 * tm + rr] * sm.bet[16 * tm + rr];
                const f32x4 u = mfma2(kd[0], kd[1], op_tr(sm.Mc, LDM, 0, 16 * tm, lane),
                                      op_tr(sm.Mc, LDM, 16, 16 * tm, lane), z);
                put_uk(uk, tm, wave, lane, h4(f * u));
            }
            if (tid == 0) a.gnb[uw] = ex(Ge);
        }
        __syncthreads();
        // ---- Gram tiles over the columns: FA and dPh (waves 0 .. 3), FB and dT (waves 4 .. 7), with
        // the row and column sums of W; fp32 copies of T~ and M~^T
        {
            const int m0 = 16 * ((wave >> 1) & 1), n0 = 16 * (wave & 1), i = n0 + rr;
            const bool lo = wave < 4;
            const f32x4 f = tile_mma<_Float16, DD>(z, (lo ? sm.dOn : sm.Bn) + m0 * LDH, LDH, sm.Dl + n0 * LDH, LDH, lane);
            const f32x4 e = tile_mma<_Float16, DD>(z, (lo ? sm.dOn : sm.dDn) + m0 * LDH, LDH,
                                                   (lo ? Dln : sm.Rn) + n0 * LDH, LDH, lane);
            // the Gram entries of W again in fp32: at g = -8 those of Nq and Nk are below fp16's normal range
            const f32x4 gr = tile_mma<_Float16, DD>(z, (lo ? sm.Qn : sm.Kn) + m0 * LDH, LDH, sm.K + n0 * LDH, LDH, lane);
            float colw = 0.f;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int t = m0 + 4 * g4 + j;
                const float m = i < (t & ~(nl - 1)) ? ex(sm.Gp[t] - sm.G[i]) : 0.f, x = lo ? sm.sg[t] * f[j] : f[j];
                float w = x * m * gr[j];
                if (i + 1 == (t & ~(nl - 1))) {
                    sm.pD[wave >> 2][t] = w;
                    w = 0.f;
                }
                colw += w;
                const float roww = row_total(w);
                if (rr == 15) sm.pR[wave >> 2][wave & 1][t] = roww;
                (lo ? sm.FA : sm.FB)[t * LDM + i] = (_Float16)(x * m);
                if (lo)
                    dPh[t * LDM + i] = (_Float16)((t ^ i) < nl ? s * e[j] * sm.Dn[i] : 0.f);
                else
                    dT[t * LDF + i] = e[j];
            }
            colw += __shfl_xor(colw, 16);
            colw += __shfl_xor(colw, 32);
            if (g4 == 0) sm.pC[wave][i] = colw;
        }
        for (int e = tid; e < NP * NP; e += 64 * kWaves) {
            const int t = e / NP, i = e % NP;
            const float m = (float)sm.Mn[t * LDM + i];
            Tf[t * LDF + i] = m * sm.betn[i];
            Mt[i * LDF + t] = m;
        }
        // the next unit's rows, in flight from here on
        const long un = next_unit(u);
        const bool more = un < a.n_units;
        if (more) load(un, tid, in);
        __syncthreads();
        // ---- dQ~, dK~ but for the dKK term, the clean dK's share; W = dT T~^T (transposed), dbeta~
        float rowa[2][4], rowb[2][4];
        f32x4 dk[2];
        const f16x4 knq[2] = {op_tr(sm.Kn, LDH, 0, c0, lane), op_tr(sm.Kn, LDH, 16, c0, lane)};
        {
            const f16x4 kq[2] = {op_tr(sm.K, LDH, 0, c0, lane), op_tr(sm.K, LDH, 16, c0, lane)};
            const f16x4 qnq[2] = {op_tr(sm.Qn, LDH, 0, c0, lane), op_tr(sm.Qn, LDH, 16, c0, lane)};
#pragma unroll
            for (int tm = 0; tm < 2; ++tm) {
                const f32x4 gq = ld4(sm.gp + 16 * tm + 4 * g4);
                f32x4 ca = tile_mma<_Float16, DD>(z, sm.dOn + 16 * tm * LDH, LDH, sm.S0 + c0 * LDH, LDH, lane);
                ca = gq * ld4(sm.sg + 16 * tm + 4 * g4) * ca;
                f32x4 cb = gq * tile_mma<_Float16, DD>(z, sm.Bn + 16 * tm * LDH, LDH, sm.S0 + c0 * LDH, LDH, lane);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    rowa[tm][j] = ca[j] * (float)qnq[tm][j];
                    rowb[tm][j] = cb[j] * (float)knq[tm][j];
                }
                ca = apply(dPh, 16 * tm, knq, apply(sm.FA, 16 * tm, kq, ca, lane), lane);
                dk[tm] = apply_t(dPh, LDM, 16 * tm, qnq, apply(sm.FB, 16 * tm, kq, cb, lane), lane);
                const f32x4 xk = apply_t(sm.FB, LDM, 16 * tm, knq, apply_t(sm.FA, LDM, 16 * tm, qnq, z, lane), lane);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int t = 16 * tm + 4 * g4 + j;
                    if (t < nvalid) {
                        put_qk(add_qk, pn.dq + (long)t * qks + col, ca[j] * inv);
                        put_qk(add_qk, pc.dk + (long)t * qks + col, xk[j] * inv);
                    }
                }
            }
        }
        if (wave < 4) {
            const int m0 = 16 * (wave >> 1), n0 = 16 * (wave & 1);
            const f32x4 c = tile_mma<float, NP>(z, dT + m0 * LDF, LDF, Tf + n0 * LDF, LDF, lane);
#pragma unroll
            for (int j = 0; j < 4; ++j) Wm[(n0 + rr) * LDF + m0 + 4 * g4 + j] = c[j];
        } else if (tid < 256 + NP) {
            const int i = tid - 256;
            float v = 0.f;
            for (int t = 0; t < NP; ++t) v = fmaf(dT[t * LDF + i], Mt[i * LDF + t], v);
            sm.dB[i] = v;
        }
        __syncthreads();
        // dA = -M~^T W, the entries below the diagonal inside a noisy block, over T~
        if (wave < 4) {
            const int m0 = 16 * (wave >> 1), n0 = 16 * (wave & 1);
            const f32x4 c = tile_mma<float, NP>(z, Mt + m0 * LDF, LDF, Wm + n0 * LDF, LDF, lane);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int t = m0 + 4 * g4 + j, i = n0 + rr;
                Tf[t * LDF + i] = t > i && (t ^ i) < nl ? -c[j] : 0.f;
            }
        }
        __syncthreads();
        // dbeta~_r += sum_c dA_rc F_rc; gate terms of A; dKK + dKK^T
#pragma unroll 1
        for (int it = 0; it < 2; ++it) {
            const int t = 16 * it + 2 * wave + (lane >> 5), c = lane & 31;
            float bt = 0.f, wa = 0.f, sym = 0.f;
            if ((t ^ c) < nl) {
                if (t > c) {
                    const float da = Tf[t * LDF + c], e = ex(sm.Gn[t] - sm.Gn[c]), f = e * sm.KK[t * LDF + c];
                    bt = da * f;
                    wa = da * sm.betn[t] * f;
                    sym = da * sm.betn[t] * e;
                } else if (c > t) {
                    sym = Tf[c * LDF + t] * sm.betn[c] * ex(sm.Gn[c] - sm.Gn[t]);
                }
            }
            Wh[t * LDM + c] = (_Float16)sym;
            const float wc = wa + __shfl_xor(wa, 32);
            const float br = half_total(bt, lane), wr = half_total(wa, lane);
            if (c == 0) {
                lds_add(&sm.dB[t], br);
                lds_add(&sm.part[wave][t], wr);
            }
            if (lane < 32 && wc != 0.f) lds_add(&sm.part[wave][c], -wc);
        }
        __syncthreads();
#pragma unroll
        for (int tm = 0; tm < 2; ++tm) {
            const f32x4 c = apply(Wh, 16 * tm, knq, dk[tm], lane);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int t = 16 * tm + 4 * g4 + j;
                if (t < nvalid) put_qk(add_qk, pn.dk + (long)t * qks + col, c[j] * inv);
                const float xa = row_total(rowa[tm][j]), xb = row_total(rowb[tm][j]), xw = row_total(roww[tm][j]);
                if (rr == 15) {
                    sm.pA[wave][t] = xa;
                    sm.pB[wave][t] = xb;
                    sm.pW[wave][t] = xw;
                }
            }
        }
        __syncthreads();
        if (wave < 2) {
            float xa = 0.f, xb = 0.f, xw = 0.f, xp = 0.f, xc = 0.f;
            if (lane < NP) {
#pragma unroll
                for (int w = 0; w < kWaves; ++w) {
                    xa += sm.pA[w][lane];
                    xb += sm.pB[w][lane];
                    xw += sm.pW[w][lane];
                    xp += sm.part[w][lane];
                    xc += sm.pC[w][lane];
                }
                xa += sm.pR[0][0][lane] + sm.pR[0][1][lane];
                xb += sm.pR[1][0][lane] + sm.pR[1][1][lane];
                if (wave == 0 && lane >= nl) {   // the noisy gates' terms hold all of the seed
                    xa += sm.pD[0][lane];
                    xb += sm.pD[1][lane];
                }
            }
            if (wave == 0) {
                // noisy: row terms summed from the block's end back, the block-end terms of all its rows,
                // and of dDelta~ . Delta~, a block-end term less a row term, the rows before
                float x = xp + xb, e = xa, before = __shfl_up(xw, 1);
                if ((lane & (nl - 1)) == 0) before = 0.f;
                for (int o = 1; o < nl; o <<= 1) {
                    const float y = __shfl_down(x, o), w = __shfl_up(before, o);
                    if ((lane & (nl - 1)) + o < nl) x += y;
                    if ((lane & (nl - 1)) >= o) before += w;
                    e += __shfl_xor(e, o);
                }
                if (lane < nvalid) {
                    pn.dg[(long)lane * a.h_v] = (x + e + before) * inv;
                    pn.db[(long)lane * a.h_v] = sm.dB[lane] * inv;
                }
            } else {
                // clean: the seed terms of a noisy block on the position before it
                float v = xa + xb;
                for (int o = 1; o < nl; o <<= 1) v += __shfl_xor(v, o);
                const float next = __shfl_down(v, 1);
                float x = lane < NP ? -xc : 0.f;
                if (lane + 1 < NP && ((lane + 1) & (nl - 1)) == 0) x += next;
#pragma unroll
                for (int o = 1; o < NP; o <<= 1) {
                    const float y = __shfl_down(x, o);
                    if (lane + o < NP) x += y;
                }
                if (lane < nvalid) pc.dg[(long)lane * a.h_v] = x * inv;
            }
        }
        if (!more) break;
        u = un;
        __syncthreads();   // LDS is free for the next unit
    }
}
