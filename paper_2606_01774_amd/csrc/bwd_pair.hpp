// bwd_pair.hpp -- the block-form backward for noisy blocks of two sub-blocks (blocks of 2 L
// positions, L = a.L <= 32, the clean stream cut into sub-blocks of L; included by
// bwd_kernels.hip): one workgroup of sixteen waves per (block, q/k head), its v-heads in turn.
//
// The noisy block runs from the clean seed S0 through its halves a and b,
//     S~1 = ea S0 + K~a^T Da Delta~a,  S~2 = eb S~1 + K~b^T Db Delta~b   (ea, eb: gamma~_n of a half),
// and every position of both halves reads S~2.  Neither S~1, S~2 nor their gradients are
// formed: with N = K~b K~a^T, f = s ea eb,
//     X~a = K~a S0,  X~b = ea K~b S0 + N Da Delta~a,
//     dDelta~b = Db s (K~b Q~a^T dO~a + K~b Q~b^T dO~b),                 Bb = -Gamma~b T~b^T dDelta~b,
//     dDelta~a = Da (eb s (K~a Q~a^T dO~a + K~a Q~b^T dO~b) + N^T Bb),   Ba = -Gamma~a T~a^T dDelta~a,
//     dS0 = f (Q~a^T dO~a + Q~b^T dO~b) + ea K~b^T Bb + K~a^T Ba,
// and with F_xa = s eb (dO~x Delta~a^T) Da, F_xb = s (dO~x Delta~b^T) Db, H = (Bb Delta~a^T) Da,
//     dQ~x = f dO~x S0^T + F_xa K~a + F_xb K~b,
//     dK~a = Ba S0^T + F_aa^T Q~a + F_ba^T Q~b + H^T K~b + (dKK + dKK^T)_a K~a,
//     dK~b = ea Bb S0^T + H K~a + F_ab^T Q~a + F_bb^T Q~b + (dKK + dKK^T)_b K~b,
// six products with S0 or S0^T of 32 rows each, where the states form took sixteen.  Waves
// 0 .. 7 work on half a and 8 .. 15 on half b, wave w % 8 on columns 16 (w % 8) ..; half b's
// backward runs beside half a's forward, half a's backward beside half b's forward.
//
// The gate gradients of a half: its rows' terms as in a block of its own, and on its last
// position <gamma~_n dS~, seed>, which is sum over the rows of q~ . (dQ~'s terms with the half's
// seed), for half a also that of k~b . (ea Bb S0^T).  The terms dDelta~ . Delta~ of the rows, added on
// the last position and taken off at their own, are summed over the rows before each position, in
// fp32: a difference would leave their rounding under strong decays, and factors rounded to fp16
// more of it (dg~ 15 % further from 64 bits at gates of -1 to -5).
//
// One workgroup per CU (157 KB of LDS), bound by what it waits for: 30 us a unit, of which
// its 430 KB of HBM traffic are 22 at a large copy's rate, which do not overlap the barriers
// (9.5 k clocks to the end of the solves, 10 k for the columns' products and the clean
// preparation, 10 k for the tiles over the columns).  At 2 x 16384 tokens, 32 v-heads over 16
// q/k heads, blocks of 64 (16384 units): 3300 -> 1990 us against one workgroup of eight waves
// forming S~1, S~2 and their gradients.  Loading the next unit's inputs during the last phases
// from a persistent grid took 2040 us (they don't fit beside the last phases: nine registers
// spilled, and waves stall at the issue of loads).

struct PairSmem {
    _Float16 Qn[2 * NP * LDH], Kn[2 * NP * LDH];   // rows 0 .. 31 half a, 32 .. 63 half b
    _Float16 Rn[2 * NP * LDH];    // v, then R~, then the partial sums
    _Float16 dOn[2 * NP * LDH];   // then, fp32, W of both halves
    _Float16 X1[2 * NP * LDH];    // clean q, then Delta~, then (fp32) dA
    _Float16 X2[2 * NP * LDH];    // clean k, then dDelta~
    _Float16 X3[2 * NP * LDH];    // clean dO, then Ba, Bb
    _Float16 Mn[2][NP * LDM];
    _Float16 N[NP * LDM];         // N, then H
    _Float16 Pn[4][NP * LDM];     // K~x Q~y^T at 2 x + y, then F_xy, then (0, 1) dKK + dKK^T
    _Float16 Mc[2][NP * LDM], Ph[2][NP * LDM];   // clean; then both, fp32, dT
    float KK[2][NP * LDF];        // first the waves' tiles being turned over
    float Gn[2][NP], G2n[2][NP], gamn[2][NP], betn[2][NP], Dn[2][NP];
    float G[2][NP], G2[2][NP], gam[2][NP], bet[2][NP];
    float dB[2][NP];
};
// per-wave partial sums over columns (in Rn): by row the gate terms of dA, k~ . (dK~'s seed
// terms) and dDelta~ . Delta~; over all rows a wave's share of the seed terms of a's and b's last
// position; by eight rows dbeta from dT
struct PairSums {
    float part[16][NP], b[16][NP], w[16][NP], end[2][16], db[2][4][NP];
};
static_assert(sizeof(PairSmem) <= 160 * 1024, "one workgroup's LDS");
static_assert(sizeof(PairSums) <= 2 * NP * LDH * 2 && 2 * NP * LDF * 4 <= 4 * NP * LDM * 2 &&
                  16 * 256 * 2 <= 2 * NP * LDF * 4,
              "shared rooms");

// 64 rows (two halves of up to 32, L apart) of a stream, one row of 16 threads
template <typename In>
__device__ __forceinline__ Row8<In> load_row64(const In *src, long stride, int L, int nva, int nvb, int tid)
{
    const int row = tid >> 4, x = row >> 5, r = row & 31, c = (tid & 15) * 8;
    Row8<In> v;
    if (r < (x ? nvb : nva))
        v.load(src + (long)(x * L + r) * stride + c);
    else
        v.zero();
    return v;
}
template <typename In> __device__ __forceinline__ void store_row64(_Float16 *dst, const Row8<In> &v, int tid, float sg = 1.f)
{
    *reinterpret_cast<f16x8 *>(dst + (tid >> 4) * LDH + (tid & 15) * 8) = v.h(sg);
}

// Where a noisy block of two halves lies: the block of 2 L positions m, its first row p0, the
// global index ga of its first sub-block, its halves' rows (nvb may be 0).
struct PairUnit {
    long p0, ga;
    int nva, nvb;
};
__device__ __forceinline__ PairUnit pair_unit(const BwdArgs &a, unsigned m)
{
    const int L2 = 2 * a.L;
    PairUnit u;
    int nv;   // its rows
    if (a.seg) {
        // a segment's noisy block: the last sequence n with segp[n] <= m, its noisy block
        // (blk0 / 2) + m - segp[n] (blk0 and the segment length are even)
        int lo = 0, hi = a.n_chains / a.h_v;
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (a.segp[mid] <= (int)m)
                lo = mid;
            else
                hi = mid;
        }
        const long lm = (long)m - a.segp[lo];
        const long r0 = a.cu ? a.cu[lo] : (long)lo * a.T, r1 = a.cu ? a.cu[lo + 1] : r0 + a.T;
        u.p0 = r0 + (a.blk0 + 2 * lm) * a.L;
        const long rem = r1 - u.p0;
        nv = rem < 0 ? 0 : (rem < L2 ? (int)rem : L2);
        u.ga = a.seg[lo] + 2 * lm;
    } else if (a.cu) {
        u.p0 = (long)m * L2;   // documents start on block boundaries
        int lo = 0, hi = a.n_docs;   // the last document with cu[d] <= p0
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (a.cu[mid] <= u.p0)
                lo = mid;
            else
                hi = mid;
        }
        const long rem = a.cu[lo + 1] - u.p0;
        nv = (int)(rem < L2 ? rem : L2);
        u.ga = u.p0 / a.L;
    } else {
        const unsigned nb2 = (a.T + L2 - 1) / L2, n = m / nb2, b = m % nb2;
        u.p0 = (long)n * a.T + (long)b * L2;
        const int rem = a.T - (int)b * L2;
        nv = rem < L2 ? rem : L2;
        u.ga = (long)n * a.nblk + 2 * b;
    }
    u.nva = nv < a.L ? nv : a.L;
    u.nvb = nv - u.nva;
    return u;
}
// a unit's inputs: rows, gates, the seed's columns (unturned)
template <typename Od, bool PREP> struct PairRows {
    Row8<__bf16> q, k, v, qc, kc;
    Row8<Od> d, dc;
    float g, b;   // wave 0 of a half: noisy, wave 1: clean
    f16x4 s0[8];
    // the noisy q and k only for the first v-head (they stay in LDS)
    __device__ __forceinline__ void load(const BwdArgs &a, const PairUnit &u, int h, int hq, bool qk, int tid)
    {
        const long qks = (long)a.h_qk * DD, vs = (long)a.h_v * DD;
        const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), x = wave >> 3, w = wave & 7;
        const StreamPtrs pn = stream_ptrs<Od>(a, true, u.p0, h, hq), pc = stream_ptrs<Od>(a, false, u.p0, h, hq);
        load_cols(s0, a.seeds + (size_t)(u.ga * a.h_v + h) * DD * DD, 16 * w, lane);
        q = load_row64(pn.q, qks, a.L, qk ? u.nva : 0, qk ? u.nvb : 0, tid);
        k = load_row64(pn.k, qks, a.L, qk ? u.nva : 0, qk ? u.nvb : 0, tid);
        v = load_row64(pn.v, vs, a.L, u.nva, u.nvb, tid);
        d = load_row64(static_cast<const Od *>(pn.dout), vs, a.L, u.nva, u.nvb, tid);
        if constexpr (PREP) {
            qc = load_row64(pc.q, qks, a.L, u.nva, u.nvb, tid);
            kc = load_row64(pc.k, qks, a.L, u.nva, u.nvb, tid);
            dc = load_row64(static_cast<const Od *>(pc.dout), vs, a.L, u.nva, u.nvb, tid);
        }
        const bool on = w < (PREP ? 2 : 1) && lane < (x ? u.nvb : u.nva);
        const long o = (long)(x * a.L + lane) * a.h_v;
        const StreamPtrs &p = w ? pc : pn;
        g = on ? p.g[o] : 0.f;
        b = on ? p.beta[o] : 0.f;
    }
};

template <typename Od, bool PREP> __global__ void __launch_bounds__(1024) bdgdn_bwd_pair_kernel(BwdArgs a)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    PairSmem &sm = *reinterpret_cast<PairSmem *>(smem_raw);
    PairSums &ps = *reinterpret_cast<PairSums *>(sm.Rn);
    const int r = a.h_v / a.h_qk;
    const float s = a.scale, sigma = a.range[0], inv = a.range[1];
    const f32x4 z = {0.f, 0.f, 0.f, 0.f};
    const long qks = (long)a.h_qk * DD, vs = (long)a.h_v * DD;
    const unsigned m = blockIdx.x / (unsigned)a.h_qk, hq = blockIdx.x % (unsigned)a.h_qk;   // (block, q/k head)
    const PairUnit un = pair_unit(a, m);
    for (int vi = 0; vi < r; ++vi) {
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));   // lane-dependent addresses recomputed per unit, not kept live
        const int lane = tid & 63, g4 = lane >> 4, rr = lane & 15;
        const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), x = wave >> 3, w = wave & 7;
        const int c0 = 16 * w, col = c0 + rr, nvb = un.nvb, nvx = x ? nvb : un.nva;
        const int h = (int)hq * r + vi;
        const long ua = un.ga * a.h_v + h, ux = x ? ua + a.h_v : ua;
        const StreamPtrs pn = stream_ptrs<Od>(a, true, un.p0, h, hq);
        const bool add_qk = vi > 0;
        const _Float16 *seed = a.seeds + (size_t)ua * DD * DD;
        // ---- rows, gates and the seed's columns
        f16x4 s0c[8];
        {
            PairRows<Od, PREP> in;
            in.load(a, un, h, hq, vi == 0, tid);
            if (vi == 0) {
                store_row64(sm.Qn, in.q, tid);
                store_row64(sm.Kn, in.k, tid);
            }
            store_row64(sm.Rn, in.v, tid);
            store_row64(sm.dOn, in.d, tid, sigma);
            if constexpr (PREP) {
                store_row64(sm.X1, in.qc, tid);
                store_row64(sm.X2, in.kc, tid);
                store_row64(sm.X3, in.dc, tid, sigma);
                if (w == 1) {
                    cum_to_lds(in.g, sm.G[x], sm.G2[x], sm.gam[x], lane);
                    if (lane < NP) sm.bet[x][lane] = in.b;
                }
            }
            if (w == 0) {
                const float c = cum_to_lds(in.g, sm.Gn[x], sm.G2n[x], sm.gamn[x], lane);
                const float end = ut::lane_value(c, NP - 1);
                if (lane < NP) {
                    sm.betn[x][lane] = in.b;
                    sm.Dn[x][lane] = ex(end - c);
                }
            }
            _Float16 *Z = reinterpret_cast<_Float16 *>(sm.KK) + 256 * wave;
#pragma unroll
            for (int kb = 0; kb < 8; ++kb) s0c[kb] = turn(Z, in.s0[kb], lane);
        }
        __syncthreads();
        const float ea = ex(sm.Gn[0][NP - 1]), eb = ex(sm.Gn[1][NP - 1]), f = s * ea * eb;
        _Float16 *const Kx = sm.Kn + x * NP * LDH, *const Rx = sm.Rn + x * NP * LDH;
        // ---- K~x S0 (first: its operands are free for the solve's registers)
        f32x4 x0[2];
#pragma unroll
        for (int tm = 0; tm < 2; ++tm) {
            x0[tm] = rows_times(Kx, 16 * tm, s0c, lane);
            settle(x0[tm]);
        }
        reread();
        // ---- the solves (waves 0, 8 noisy, 1, 9 clean) and Gram tiles
        if (w == 0) {
            solve_block(Kx, sm.G2n[x], sm.betn[x], sm.Mn[x], lane);
        } else if (w == 1) {
            if constexpr (PREP) solve_block(sm.X2 + x * NP * LDH, sm.G2[x], sm.bet[x], sm.Mc[x], lane);
        } else {
            for (int e = w - 2 + 6 * x; e < (PREP ? 36 : 28); e += 12) {
                const int gram = e >> 2, m0 = 16 * ((e >> 1) & 1), n0 = 16 * (e & 1), i = n0 + rr;
                // K~a K~a^T, K~b K~b^T, N; K~x Q~y^T; P of the clean halves
                const int ax = gram < 3 ? (gram > 0) : (gram < 7 ? (gram - 3) >> 1 : gram - 7);
                const int bx = gram < 3 ? gram == 1 : (gram < 7 ? (gram - 3) & 1 : gram - 7);
                const _Float16 *A = (gram < 7 ? sm.Kn : sm.X1) + ax * NP * LDH;
                const _Float16 *B = (gram < 3 ? sm.Kn : (gram < 7 ? sm.Qn : sm.X2)) + bx * NP * LDH;
                const f32x4 c = tile_mma<_Float16, DD>(z, A + m0 * LDH, LDH, B + n0 * LDH, LDH, lane);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int t = m0 + 4 * g4 + j;
                    if (gram < 2)
                        sm.KK[gram][t * LDF + i] = c[j];
                    else if (gram < 7)
                        (gram == 2 ? sm.N : sm.Pn[gram - 3])[t * LDM + i] = (_Float16)c[j];
                    else
                        sm.Ph[ax][t * LDM + i] = (_Float16)(i <= t ? c[j] * ex(sm.G[ax][t] - sm.G[ax][i]) : 0.f);
                }
            }
        }
        __syncthreads();
        // ---- this wave's columns: the clean preparation of its half; half a: R~a, Delta~a, half b:
        // dDelta~b, dV~b, Bb
        f32x4 acc[8];   // half a: its clean c term, completed below
        f32x4 first[2];   // Delta~a (half a), dDelta~b (half b): fp32 for the row sums with the other
        f16x4 dd[2], bq[2];
#pragma unroll
        for (int tm = 0; tm < 8; ++tm) acc[tm] = z;
        if constexpr (PREP) {
            const _Float16 *Qc = sm.X1 + x * NP * LDH, *Kc = sm.X2 + x * NP * LDH, *dOc = sm.X3 + x * NP * LDH;
            const f16x4 doc[2] = {op_tr(dOc, LDH, 0, c0, lane), op_tr(dOc, LDH, 16, c0, lane)};
            f16x4 yq[2], drq[2], sd[2], kd[2];
            const float Ge = sm.G[x][NP - 1];
#pragma unroll
            for (int tm = 0; tm < 2; ++tm) yq[tm] = h4(s * apply_t(sm.Ph[x], LDM, 16 * tm, doc, z, lane));
#pragma unroll
            for (int tm = 0; tm < 2; ++tm) {
                const f32x4 gm = ld4(sm.gam[x] + 16 * tm + 4 * g4);
                drq[tm] = h4(-gm * apply_Tt(sm.Mc[x], sm.bet[x], 16 * tm, yq, lane));
                sd[tm] = scale4(doc[tm], s * gm);
                f32x4 d;
#pragma unroll
                for (int j = 0; j < 4; ++j) d[j] = ex(Ge - sm.G[x][16 * tm + 4 * g4 + j]);
                kd[tm] = scale4(op_tr(Kc, LDH, 16 * tm, c0, lane), d);
            }
            if (nvx > 0) {   // U K, transposed as the scan reads it
                _Float16 *uk = a.uk + (size_t)ux * NP * DD;
#pragma unroll
                for (int tm = 0; tm < 2; ++tm) {
                    const float fu = sm.gam[x][16 * tm + rr] * sm.bet[x][16 * tm + rr];
                    const f32x4 u = mfma2(kd[0], kd[1], op_tr(sm.Mc[x], LDM, 0, 16 * tm, lane),
                                          op_tr(sm.Mc[x], LDM, 16, 16 * tm, lane), z);
                    put_uk(uk, tm, w, lane, h4(fu * u));
                }
                if (w == 0 && lane == 0) a.gnb[ux] = ex(Ge);
            }
            f16x4 *ct = reinterpret_cast<f16x4 *>(a.cterm + (size_t)ux * DD * DD) + w * 64 + lane;
#pragma unroll
            for (int tm = 0; tm < 8; ++tm) {
                const f32x4 c = apply_t(Qc, LDH, 16 * tm, sd, apply_t(Kc, LDH, 16 * tm, drq, z, lane), lane);
                if (x == 0)
                    acc[tm] = c;
                else if (nvb > 0)   // no noisy block is seeded at half b's start: its whole term
                    ct[tm * 8 * 64] = h4(c);
            }
        }
        if (x == 0) {
#pragma unroll
            for (int tm = 0; tm < 2; ++tm)
                bq[tm] = h4(f4(op_tr(Rx, LDH, 16 * tm, c0, lane)) - ld4(sm.gamn[0] + 16 * tm + 4 * g4) * x0[tm]);   // R~a
#pragma unroll
            for (int tm = 0; tm < 2; ++tm) {
                put_tile(Rx, LDH, 16 * tm, col, bq[tm], g4);
                first[tm] = apply_T(sm.Mn[0], sm.betn[0], 16 * tm, bq, lane);
            }
        } else {
            const f16x4 da[2] = {op_tr(sm.dOn, LDH, 0, c0, lane), op_tr(sm.dOn, LDH, 16, c0, lane)};
            const f16x4 db[2] = {op_tr(sm.dOn, LDH, 32, c0, lane), op_tr(sm.dOn, LDH, 48, c0, lane)};
#pragma unroll
            for (int tm = 0; tm < 2; ++tm) {
                first[tm] = s * ld4(sm.Dn[1] + 16 * tm + 4 * g4) *
                            apply(sm.Pn[3], 16 * tm, db, apply(sm.Pn[2], 16 * tm, da, z, lane), lane);
                dd[tm] = h4(first[tm]);
            }
        }
        // dR~ = T~^T dDelta~ (= dV~) and B = -Gamma~ dR~ of this wave's half
        auto half_back = [&]() {
#pragma unroll
            for (int tm = 0; tm < 2; ++tm) {
                const f32x4 c = apply_Tt(sm.Mn[x], sm.betn[x], 16 * tm, dd, lane);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int t = 16 * tm + 4 * g4 + j;
                    if (t < nvx) pn.dv[(long)(x * a.L + t) * vs + col] = c[j] * inv;
                }
                bq[tm] = h4(-ld4(sm.gamn[x] + 16 * tm + 4 * g4) * c);
            }
        };
        if (x) half_back();
        __syncthreads();   // the clean rows are read: Delta~, dDelta~, B in their place
#pragma unroll
        for (int tm = 0; tm < 2; ++tm) {
            if (x == 0) {
                put_tile(sm.X1, LDH, 16 * tm, col, h4(first[tm]), g4);
            } else {
                put_tile(sm.X2, LDH, NP + 16 * tm, col, dd[tm], g4);
                put_tile(sm.X3, LDH, NP + 16 * tm, col, bq[tm], g4);
            }
        }
        __syncthreads();
        // ---- half b: R~b, Delta~b; half a: dDelta~a, dV~a, Ba
        if (x) {
            // N Da Delta~a: the decays on Delta~a's rows
            f16x4 da[2], rn[2];
#pragma unroll
            for (int tm = 0; tm < 2; ++tm)
                da[tm] = scale4(op_tr(sm.X1, LDH, 16 * tm, c0, lane), ld4(sm.Dn[0] + 16 * tm + 4 * g4));
#pragma unroll
            for (int tm = 0; tm < 2; ++tm)
                rn[tm] = h4(f4(op_tr(Rx, LDH, 16 * tm, c0, lane)) -
                            ld4(sm.gamn[1] + 16 * tm + 4 * g4) * apply(sm.N, 16 * tm, da, ea * x0[tm], lane));
#pragma unroll
            for (int tm = 0; tm < 2; ++tm) {
                put_tile(Rx, LDH, 16 * tm, col, rn[tm], g4);
                const f32x4 d = apply_T(sm.Mn[1], sm.betn[1], 16 * tm, rn, lane);
                put_tile(sm.X1, LDH, NP + 16 * tm, col, h4(d), g4);
                first[tm] *= d;
            }
        } else {
            const f16x4 da[2] = {op_tr(sm.dOn, LDH, 0, c0, lane), op_tr(sm.dOn, LDH, 16, c0, lane)};
            const f16x4 db[2] = {op_tr(sm.dOn, LDH, 32, c0, lane), op_tr(sm.dOn, LDH, 48, c0, lane)};
            const f16x4 bb[2] = {op_tr(sm.X3, LDH, 32, c0, lane), op_tr(sm.X3, LDH, 48, c0, lane)};
#pragma unroll
            for (int tm = 0; tm < 2; ++tm) {
                const f32x4 c = apply(sm.Pn[1], 16 * tm, db, apply(sm.Pn[0], 16 * tm, da, z, lane), lane);
                const f32x4 d = ld4(sm.Dn[0] + 16 * tm + 4 * g4) * apply_t(sm.N, LDM, 16 * tm, bb, s * eb * c, lane);
                dd[tm] = h4(d);
                first[tm] *= d;
                put_tile(sm.X2, LDH, 16 * tm, col, dd[tm], g4);
            }
            half_back();
#pragma unroll
            for (int tm = 0; tm < 2; ++tm) put_tile(sm.X3, LDH, 16 * tm, col, bq[tm], g4);
        }
#pragma unroll
        for (int tm = 0; tm < 2; ++tm) settle(first[tm]);   // now dDelta~ . Delta~, this column's terms
        __syncthreads();
        // ---- half a's waves: the c term of sub-block a; half b's: the Gram tiles over the columns
        float *const dT = reinterpret_cast<float *>(sm.Mc);
        if (x == 0) {
            const f32x4 ff = {f, f, f, f}, ee = {ea, ea, ea, ea};
            const f16x4 da[2] = {scale4(op_tr(sm.dOn, LDH, 0, c0, lane), ff), scale4(op_tr(sm.dOn, LDH, 16, c0, lane), ff)};
            const f16x4 db[2] = {scale4(op_tr(sm.dOn, LDH, 32, c0, lane), ff), scale4(op_tr(sm.dOn, LDH, 48, c0, lane), ff)};
            const f16x4 bb[2] = {scale4(op_tr(sm.X3, LDH, 32, c0, lane), ee), scale4(op_tr(sm.X3, LDH, 48, c0, lane), ee)};
            f16x4 *ct = reinterpret_cast<f16x4 *>(a.cterm + (size_t)ua * DD * DD) + w * 64 + lane;
#pragma unroll
            for (int tm = 0; tm < 8; ++tm) {
                f32x4 c = PREP ? acc[tm] : f4(ct[tm * 8 * 64]);
                c = apply_t(sm.Kn, LDH, 16 * tm, bq, c, lane);
                c = apply_t(sm.Kn + NP * LDH, LDH, 16 * tm, bb, c, lane);
                c = apply_t(sm.Qn, LDH, 16 * tm, da, c, lane);
                ct[tm * 8 * 64] = h4(apply_t(sm.Qn + NP * LDH, LDH, 16 * tm, db, c, lane));
            }
        } else {
            for (int e = w; e < 28; e += 8) {
                const int gram = e >> 2, m0 = 16 * ((e >> 1) & 1), n0 = 16 * (e & 1), i = n0 + rr;
                // F_aa, F_ab, F_ba, F_bb; H; dT of half a, of half b
                const int ax = gram < 4 ? gram >> 1 : (gram == 4 ? 1 : gram - 5);
                const int bx = gram < 4 ? gram & 1 : (gram == 4 ? 0 : gram - 5);
                const _Float16 *A = (gram < 4 ? sm.dOn : (gram == 4 ? sm.X3 : sm.X2)) + ax * NP * LDH;
                const _Float16 *B = (gram < 5 ? sm.X1 : sm.Rn) + bx * NP * LDH;
                const f32x4 c = tile_mma<_Float16, DD>(z, A + m0 * LDH, LDH, B + n0 * LDH, LDH, lane);
                const float g = gram < 4 ? (bx ? s : s * eb) * sm.Dn[bx][i] : sm.Dn[0][i];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int t = m0 + 4 * g4 + j;
                    if (gram < 5)
                        (gram < 4 ? sm.Pn[gram] : sm.N)[t * LDM + i] = (_Float16)(c[j] * g);
                    else
                        dT[(gram - 5) * NP * LDF + t * LDF + i] = c[j];
                }
            }
        }
        // products with S0^T of this half's rows
        float *const dqx = pn.dq + (long)x * a.L * qks + col, *const dkx = pn.dk + (long)x * a.L * qks + col;
        // dq, dk so far (the v-heads before), to be added to
        auto so_far = [&](f32x4 (&o)[2], const float *p) {
#pragma unroll
            for (int tm = 0; tm < 2; ++tm) {
                o[tm] = z;
                if (add_qk) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const int t = 16 * tm + 4 * g4 + j;
                        if (t < nvx) o[tm][j] = p[(long)t * qks];
                    }
                }
            }
        };
        f32x4 old[2];
        so_far(old, dqx);
        f32x4 ca[2], cb[2];
        {
            f16x8 s0r[4];
            load_rows16(s0r, seed, c0, lane);
#pragma unroll
            for (int tm = 0; tm < 2; ++tm) {
                ca[tm] = f * rows_times(sm.dOn + x * NP * LDH, 16 * tm, s0r, lane);
                cb[tm] = (x ? ea : 1.f) * rows_times(sm.X3 + x * NP * LDH, 16 * tm, s0r, lane);
                settle(ca[tm]);
                settle(cb[tm]);
            }
            reread();
        }
        __syncthreads();
        // ---- dQ~; dK~ but for the dKK term; the dA products; the row sums
        float *const Wm = reinterpret_cast<float *>(sm.dOn) + x * NP * LDF;
        float *const dA = reinterpret_cast<float *>(sm.X1) + x * NP * LDF;
        if (w < 4)
            dA_first(dT + x * NP * LDF, sm.Mn[x], sm.betn[x], Wm, w, lane);
        else {
            // dbeta_i += sum_t dT_ti M_ti, eight rows a wave
            const int i = lane & 31, t0 = 8 * (w - 4) + 4 * (lane >> 5);
            float v = 0.f;
#pragma unroll
            for (int t = 0; t < 4; ++t) v = fmaf(dT[x * NP * LDF + (t0 + t) * LDF + i], (float)sm.Mn[x][(t0 + t) * LDM + i], v);
            v += __shfl_xor(v, 32);
            if (lane < NP) {
                ps.db[x][w - 4][lane] = v;
                if (w == 4) sm.dB[x][lane] = 0.f;
            }
        }
        if (lane < NP) ps.part[wave][lane] = 0.f;
        auto rows = [&](f16x4 (&o)[2], const _Float16 *X, int m0) {
            o[0] = op_tr(X, LDH, m0, c0, lane);
            o[1] = op_tr(X, LDH, m0 + 16, c0, lane);
        };
        float e1 = 0.f, e2 = 0.f;
#pragma unroll
        for (int tm = 0; tm < 2; ++tm) {
            float s4[4];
            f16x4 o[2];
            const f16x4 qx = op_tr(sm.Qn, LDH, x * NP + 16 * tm, c0, lane), kx = op_tr(sm.Kn, LDH, x * NP + 16 * tm, c0, lane);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                e1 = fmaf(ca[tm][j], (float)qx[j], e1);
                if (x) e1 = fmaf(cb[tm][j], (float)kx[j], e1);
            }
            rows(o, sm.Kn, 0);
            ca[tm] = apply(sm.Pn[2 * x], 16 * tm, o, ca[tm], lane);
            if (x) cb[tm] = apply(sm.N, 16 * tm, o, cb[tm], lane);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                e2 = fmaf(ca[tm][j], (float)qx[j], e2);
                s4[j] = cb[tm][j] * (float)kx[j];
            }
            rows(o, sm.Kn, NP);
            ca[tm] = apply(sm.Pn[2 * x + 1], 16 * tm, o, ca[tm], lane);
            if (!x) cb[tm] = apply_t(sm.N, LDM, 16 * tm, o, cb[tm], lane);
            rows(o, sm.Qn, 0);
            cb[tm] = apply_t(sm.Pn[x], LDM, 16 * tm, o, cb[tm], lane);
            rows(o, sm.Qn, NP);
            cb[tm] = apply_t(sm.Pn[2 + x], LDM, 16 * tm, o, cb[tm], lane);
            reread();
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int t = 16 * tm + 4 * g4 + j;
                if (t < nvx) dqx[(long)t * qks] = fmaf(ca[tm][j], inv, old[tm][j]);
                const float t4 = row_total(s4[j]), w4 = row_total(first[tm][j]);
                if (rr == 15) {
                    ps.b[wave][t] = t4;
                    ps.w[wave][t] = w4;
                }
            }
        }
        e1 = wave_total(e1);
        e2 = wave_total(e2);
        if (lane == 0) {
            ps.end[0][wave] = e1;
            ps.end[1][wave] = e2;
        }
        so_far(old, dkx);
        __syncthreads();
        if (w < 4) dA_second(sm.Mn[x], Wm, dA, w, lane);
        __syncthreads();
        dA_terms(dA, sm.KK[x], sm.Gn[x], sm.betn[x], sm.Pn[x], sm.dB[x], ps.part[wave], w, lane);
        __syncthreads();
#pragma unroll
        for (int tm = 0; tm < 2; ++tm) {
            const f16x4 kq[2] = {op_tr(Kx, LDH, 0, c0, lane), op_tr(Kx, LDH, 16, c0, lane)};
            const f32x4 c = apply(sm.Pn[x], 16 * tm, kq, cb[tm], lane);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int t = 16 * tm + 4 * g4 + j;
                if (t < nvx) dkx[(long)t * qks] = fmaf(c[j], inv, old[tm][j]);
            }
        }
        if (w == 0) {
            // dg of a half: row terms summed from its end back, the block-end terms of all rows, and of
            // dDelta~ . Delta~, a block-end term less a row term, what is left: the rows before
            float g = 0.f, db = 0.f, before = 0.f;
            if (lane < NP) {
                db = ((ps.db[x][0][lane] + ps.db[x][1][lane]) + (ps.db[x][2][lane] + ps.db[x][3][lane])) + sm.dB[x][lane];
#pragma unroll
                for (int v = 0; v < 8; ++v) {
                    g += ps.part[8 * x + v][lane] + ps.b[8 * x + v][lane];
                    if (lane > 0) before += ps.w[8 * x + v][lane - 1];
                }
            }
            const float e = lane < 16 ? ps.end[x][lane] : 0.f;
            g = back_sum32(g, lane) + wave_total(e) + ut::scan32(before, lane);
            if (lane < nvx) {
                const long o = (long)(x * a.L + lane) * a.h_v;
                pn.dg[o] = g * inv;
                pn.db[o] = db * inv;
            }
        }
        if (vi + 1 < r) __syncthreads();   // LDS is free for the next v-head
    }
}
