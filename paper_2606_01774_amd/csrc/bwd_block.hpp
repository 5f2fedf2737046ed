// bwd_block.hpp -- the noisy and clean block kernels of the block-form backward (included by
// bwd_kernels.hip): one workgroup of eight waves per (block, q/k head), its v-heads in turn.
//
// Both are bound by the latency of their phases (solve, Gram tiles, fp32 products of dA, each
// behind a barrier) and by the LDS reads of the 32-row operands, not by MFMA or HBM.  So they
// are cut to half of a CU's LDS and of its registers (80 KB, 128 VGPRs), and two workgroups
// run on a CU, one computing while the other loads or waits at a barrier.  The two 128 x 128
// states never lie in LDS: wave w needs 16 columns and 16 rows of each, 8 tiles of 16 x 16
// fp16, which it loads straight into operand registers, the tiles of the other orientation
// turned over through 512 bytes of its own.  Everything that needs only a wave's 16 columns
// runs without a barrier; the noisy block-end gradient s Q~^T dO~ is never formed, K~ dS~
// coming from the Gram tiles K~ Q~^T.  At 4 x 4096 tokens, 16 heads, blocks of 32 (8192
// units): noisy 640 -> 456 us, clean 520 -> 358 us (425 and 340 on the fastest of the boxes they were
// measured on), against one workgroup of 160 KB per CU with
// both states in LDS.  Registers are what the form hangs on: with 17 of them spilled the
// kernels wrote 300 and 270 MB of scratch and took 490 and 416 us, hence settle() and reread();
// one is still spilled where the noisy kernel prepares the clean block too (8 bytes a lane).

// a 16 x 32 by 32 x 16 product from operand quads over k = 0 .. 15 and 16 .. 31 (one
// 16x16x32 step: A and B agree on which k each slot holds)
__device__ __forceinline__ f32x4 mfma2(f16x4 a0, f16x4 a1, f16x4 b0, f16x4 b1, f32x4 c)
{
    const f16x8 a = __builtin_shufflevector(a0, a1, 0, 1, 2, 3, 4, 5, 6, 7);
    const f16x8 b = __builtin_shufflevector(b0, b1, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}
// rows m0 .. of a [32][32] matrix, and rows m0 .. of its transpose, times the k-quads b
__device__ __forceinline__ f32x4 apply(const _Float16 *X, int m0, const f16x4 (&b)[2], f32x4 c, int lane)
{
    return mfma2(op_row(X, LDM, m0, 0, lane), op_row(X, LDM, m0, 16, lane), b[0], b[1], c);
}
__device__ __forceinline__ f32x4 apply_t(const _Float16 *X, int ld, int m0, const f16x4 (&b)[2], f32x4 c, int lane)
{
    return mfma2(op_tr(X, ld, 0, m0, lane), op_tr(X, ld, 16, m0, lane), b[0], b[1], c);
}
// T rows m0 .. (T_ri = M_ri beta_i), and T^T rows m0 .., times the k-quads b
__device__ __forceinline__ f32x4 apply_T(const _Float16 *M, const float *bet, int m0, const f16x4 (&b)[2], int lane)
{
    const f32x4 z = {0.f, 0.f, 0.f, 0.f};
    return mfma2(scale4(op_row(M, LDM, m0, 0, lane), ld4(bet + 4 * (lane >> 4))),
                 scale4(op_row(M, LDM, m0, 16, lane), ld4(bet + 16 + 4 * (lane >> 4))), b[0], b[1], z);
}
__device__ __forceinline__ f32x4 apply_Tt(const _Float16 *M, const float *bet, int m0, const f16x4 (&b)[2], int lane)
{
    const f32x4 z = {0.f, 0.f, 0.f, 0.f};
    const float x = bet[m0 + (lane & 15)];
    const f32x4 bb = {x, x, x, x};
    return mfma2(scale4(op_tr(M, LDM, 0, m0, lane), bb), scale4(op_tr(M, LDM, 16, m0, lane), bb), b[0], b[1], z);
}
__device__ __forceinline__ f32x4 f4(f16x4 v) { return f32x4{(float)v[0], (float)v[1], (float)v[2], (float)v[3]}; }
// a C tile (rows m0 + 4 g + j, column c) into a row-major fp16 matrix
__device__ __forceinline__ void put_tile(_Float16 *X, int ld, int m0, int c, f16x4 v, int g4)
{
#pragma unroll
    for (int j = 0; j < 4; ++j) X[(m0 + 4 * g4 + j) * ld + c] = v[j];
}
// A 16 x 16 tile turned over through this wave's 256 elements at Z: lane (g, n) gives row (or
// column) n, entries 4 g .. 4 g + 3, and receives column (or row) n.  A wave's LDS operations
// run in order, so the next tile may be written as soon as this read is issued.
__device__ __forceinline__ f16x4 turn(_Float16 *Z, f16x4 v, int lane)
{
    *reinterpret_cast<f16x4 *>(Z + 16 * (lane & 15) + 4 * (lane >> 4)) = v;
    return op_tr(Z, 16, 0, 0, lane);
}
// rows m0 .. m0 + 15 of a [32][128] LDS matrix times the natural-order k-octets b (a 16-row slice
// of a row-major state: X S^T)
__device__ __forceinline__ f32x4 rows_times(const _Float16 *X, int m0, const f16x8 (&b)[4], int lane)
{
    f32x4 c = {0.f, 0.f, 0.f, 0.f};
    const _Float16 *p = X + (m0 + (lane & 15)) * LDH + 8 * (lane >> 4);
#pragma unroll
    for (int j = 0; j < 4; ++j)
        c = __builtin_amdgcn_mfma_f32_16x16x32_f16(*reinterpret_cast<const f16x8 *>(p + 32 * j), b[j], c, 0, 0, 0);
    return c;
}
// the same times quads b (k = 16 kb + 4 g + e)
__device__ __forceinline__ f32x4 rows_times(const _Float16 *X, int m0, const f16x4 (&b)[8], int lane)
{
    f32x4 c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kb = 0; kb < 8; kb += 2)
        c = mfma2(op_row(X, LDH, m0, 16 * kb, lane), op_row(X, LDH, m0, 16 * kb + 16, lane), b[kb], b[kb + 1], c);
    return c;
}
// wave w's columns of a row-major state as k-quads (rows), unturned; and its rows
__device__ __forceinline__ void load_cols(f16x4 (&x)[8], const _Float16 *S, int c0, int lane)
{
#pragma unroll
    for (int kb = 0; kb < 8; ++kb)
        x[kb] = *reinterpret_cast<const f16x4 *>(S + (16 * kb + (lane & 15)) * DD + c0 + 4 * (lane >> 4));
}
__device__ __forceinline__ void load_rows16(f16x8 (&x)[4], const _Float16 *S, int c0, int lane)
{
#pragma unroll
    for (int j = 0; j < 4; ++j)
        x[j] = *reinterpret_cast<const f16x8 *>(S + (c0 + (lane & 15)) * DD + 32 * j + 8 * (lane >> 4));
}
// LDS values read before are read again after (not kept in registers from one product to the next)
__device__ __forceinline__ void reread() { asm volatile("" ::: "memory"); }
// x computed here, so that its operands' registers are free from here on
template <typename T> __device__ __forceinline__ void settle(T &x) { asm volatile("" : "+v"(x)); }
// 32 lanes' inclusive sum from lane 31 back
__device__ __forceinline__ float back_sum32(float x, int lane)
{
#pragma unroll
    for (int o = 1; o < NP; o <<= 1) {
        const float y = __shfl_down(x, o);
        if (lane + o < NP) x += y;
    }
    return x;
}
// Cumulative log-gates of a block from the gate of each lane (wave 0 or 1, lanes 0 .. 31).
__device__ __forceinline__ float cum_to_lds(float g, float *G, float *G2, float *gam, int lane)
{
    const float x = ut::scan32(lane < NP ? ut::gate_floor(g) : 0.f, lane);
    if (lane < NP) {
        G[lane] = x;
        G2[lane] = x * kLog2e;
        gam[lane] = ex(x);
    }
    return x;
}
__device__ __forceinline__ void solve_block(const _Float16 *K, const float *G2, const float *bet, _Float16 *M, int lane)
{
    ut::QE kq[2][DD / 16];
#pragma unroll
    for (int rb = 0; rb < 2; ++rb)
#pragma unroll
        for (int kb = 0; kb < DD / 16; ++kb) kq[rb][kb] = op_row(K, LDH, 16 * rb, 16 * kb, lane);
    ut::Consts cs;
    ut::make_consts(cs, lane);
    ut::solve_t<2, DD / 16, false>(kq, G2, bet, M, LDM, cs, lane);
}
// Tile e (0 .. 3) of W^T = (dT T^T)^T in fp32 MFMA, T from the fp16 M; then of dA = -(M^T W)
// below the diagonal.  Exact products of fp16 values in fp32, as from fp32 copies.
__device__ __forceinline__ void dA_first(const float *dT, const _Float16 *M, const float *bet, float *W, int e, int lane)
{
    const int m0 = 16 * (e >> 1), n0 = 16 * (e & 1), rr = lane & 15, g4 = lane >> 4;
    f32x4 c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < NP; k += 4)
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(dT[(m0 + rr) * LDF + k + g4],
                                                 (float)M[(n0 + rr) * LDM + k + g4] * bet[k + g4], c, 0, 0, 0);
#pragma unroll
    for (int j = 0; j < 4; ++j) W[(n0 + rr) * LDF + m0 + 4 * g4 + j] = c[j];
}
__device__ __forceinline__ void dA_second(const _Float16 *M, const float *W, float *dA, int e, int lane)
{
    const int m0 = 16 * (e >> 1), n0 = 16 * (e & 1), rr = lane & 15, g4 = lane >> 4;
    f32x4 c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < NP; k += 4)
        c = __builtin_amdgcn_mfma_f32_16x16x4f32((float)M[(k + g4) * LDM + m0 + rr], W[(n0 + rr) * LDF + k + g4], c, 0,
                                                 0, 0);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int r = m0 + 4 * g4 + j, i = n0 + rr;
        dA[r * LDF + i] = r > i ? -c[j] : 0.f;
    }
}
// dbeta_i += sum_r dT_ri M_ri (lane i of one wave)
__device__ __forceinline__ float dbeta_T(const float *dT, const _Float16 *M, int i)
{
    float v = 0.f;
#pragma unroll
    for (int r = 0; r < NP; ++r) v = fmaf(dT[r * LDF + i], (float)M[r * LDM + i], v);
    return v;
}
// From dA: dbeta_r += sum_c dA_rc F_rc; the gate terms of A (row + , column -) into this wave's
// part; dKK + dKK^T with dKK_rc = dA_rc beta_r gamma_r / gamma_c.
__device__ __forceinline__ void dA_terms(const float *dA, const float *KK, const float *G, const float *bet, _Float16 *Wh,
                                         float *dB, float *part, int wave, int lane)
{
#pragma unroll 1
    for (int it = 0; it < 2; ++it) {
        const int r = 16 * it + 2 * wave + (lane >> 5), c = lane & 31;
        float bt = 0.f, wa = 0.f, sym = 0.f;
        if (r > c) {
            const float da = dA[r * LDF + c], e = ex(G[r] - G[c]), f = e * KK[r * LDF + c];
            bt = da * f;
            wa = da * bet[r] * f;
            sym = da * bet[r] * e;
        } else if (c > r) {
            sym = dA[c * LDF + r] * bet[c] * ex(G[c] - G[r]);
        }
        Wh[r * LDM + c] = (_Float16)sym;
        const float wc = wa + __shfl_xor(wa, 32);
        const float br = half_total(bt, lane), wr = half_total(wa, lane);
        if (c == 0) {
            lds_add(&dB[r], br);
            lds_add(&part[r], wr);
        }
        if (lane < 32 && wc != 0.f) lds_add(&part[c], -wc);
    }
}

struct NoisySmem {
    _Float16 Qn[NP * LDH], Kn[NP * LDH];
    _Float16 Rn[NP * LDH];    // noisy v, then R~
    _Float16 dOn[NP * LDH];   // then, fp32, W
    _Float16 Q[NP * LDH];     // clean q, then Delta~, then (fp32) dA
    _Float16 K[NP * LDH];     // clean k, then dDelta~
    _Float16 dO[NP * LDH];    // clean dO, then -Gamma~ dR~
    _Float16 Mc[NP * LDM], Ph[NP * LDM];   // clean M and P; then both fp32 dT, then Ph dKK + dKK^T
    _Float16 Mn[NP * LDM];
    _Float16 Pn[NP * LDM];    // K~ Q~^T, then dPh
    float KK[NP * LDF];       // first the waves' tiles being turned over
    float G[NP], G2[NP], gam[NP], bet[NP];
    float Gn[NP], G2n[NP], gamn[NP], betn[NP], Dn[NP];
    float dB[NP];
    // per-wave partial sums, added in a fixed order: gate terms of dA, q~ . seed a, k~ . seed b,
    // dDelta~ . Delta~ (as in bwd_small.hpp, with one noisy block per chunk)
    float part[kWaves][NP], pA[kWaves][NP], pB[kWaves][NP], pW[kWaves][NP];
};
static_assert(sizeof(NoisySmem) <= 80 * 1024, "two workgroups per CU");
static_assert(NP * LDF * 4 <= 2 * NP * LDM * 2 && kWaves * 256 * 2 <= NP * LDF * 4, "shared rooms");

// Phase 1: every noisy block, and (PREP) the part of the clean block of the same position that
// does not depend on the state gradient at its end; both enter the state gradient at the
// block's start, whose sum is written to cterm.  Without PREP (a further noisy view) the
// seed's gradient is added to cterm.
template <typename Od, bool PREP> __global__ void __launch_bounds__(512, 4) bdgdn_bwd_noisy_kernel(BwdArgs a)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    NoisySmem &sm = *reinterpret_cast<NoisySmem *>(smem_raw);
    _Float16 *const Dln = sm.Q, *const dDn = sm.K, *const Bn = sm.dO, *const dPh = sm.Pn, *const Wh = sm.Ph;
    float *const dT = reinterpret_cast<float *>(sm.Mc), *const Wm = reinterpret_cast<float *>(sm.dOn);
    float *const dA = reinterpret_cast<float *>(sm.Q);
    const int r = a.h_v / a.h_qk;
    const float s = a.scale, sigma = a.range[0], inv = a.range[1];
    const f32x4 z = {0.f, 0.f, 0.f, 0.f};
    const long qks = (long)a.h_qk * DD, vs = (long)a.h_v * DD;
    const int gb = blockIdx.x / a.h_qk, hq = blockIdx.x % a.h_qk;
    long p0;
    int n, nvalid;
    block_unit(a, gb, n, p0, nvalid);
    for (int vi = 0; vi < r; ++vi) {
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));   // lane-dependent addresses recomputed per unit, not kept live
        const int lane = tid & 63, g4 = lane >> 4, rr = lane & 15;
        const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), c0 = 16 * wave, col = c0 + rr;
        const int h = hq * r + vi;
        const long uw = (long)gb * a.h_v + h;
        const StreamPtrs pn = stream_ptrs<Od>(a, true, p0, h, hq);
        const bool add_qk = vi > 0;
        const _Float16 *seed = a.seeds + (size_t)uw * DD * DD;
        // ---- rows, gates and the seed's columns
        f16x4 s0c[8];
        {
            load_cols(s0c, seed, c0, lane);
            const BlockRows<Od, true> nin = load_block<Od, true>(pn, a.h_qk, a.h_v, nvalid, tid);
            BlockRows<Od, false> cin;
            if constexpr (PREP)
                cin = load_block<Od, false>(stream_ptrs<Od>(a, false, p0, h, hq), a.h_qk, a.h_v, nvalid, tid);
            // clean gates by wave 0 (lanes of tid < 32 hold them), noisy ones read by wave 1
            float gn = 0.f, bn = 0.f;
            if (wave == 1 && lane < nvalid) {
                gn = pn.g[(long)lane * a.h_v];
                bn = pn.beta[(long)lane * a.h_v];
            }
            store_rows(sm.Qn, nin.q, tid);
            store_rows(sm.Kn, nin.k, tid);
            store_rows(sm.Rn, nin.v, tid);
            store_rows(sm.dOn, nin.dout, tid, sigma);
            if constexpr (PREP) {
                store_rows(sm.Q, cin.q, tid);
                store_rows(sm.K, cin.k, tid);
                store_rows(sm.dO, cin.dout, tid, sigma);
                if (wave == 0) {
                    cum_to_lds(cin.g, sm.G, sm.G2, sm.gam, lane);
                    if (lane < NP) sm.bet[lane] = cin.b;
                }
            }
            if (wave == 1) {
                const float x = cum_to_lds(lane < NP ? gn : 0.f, sm.Gn, sm.G2n, sm.gamn, lane);
                const float end = ut::lane_value(x, NP - 1);
                if (lane < NP) {
                    sm.betn[lane] = bn;
                    sm.Dn[lane] = ex(end - x);
                }
            }
            if (tid < kWaves * NP) sm.part[tid / NP][tid % NP] = 0.f;
            _Float16 *Z = reinterpret_cast<_Float16 *>(sm.KK) + 256 * wave;
#pragma unroll
            for (int kb = 0; kb < 8; ++kb) s0c[kb] = turn(Z, s0c[kb], lane);
        }
        __syncthreads();
        const float Gn_ = sm.Gn[NP - 1], sgn = s * ex(Gn_);   // s gamma~_n
        // ---- R~ = V~ - Gamma~ K~ S0 (first: its operands are free for the solve's registers)
        f16x4 rn[2];
#pragma unroll
        for (int tm = 0; tm < 2; ++tm) {
            const f32x4 x = rows_times(sm.Kn, 16 * tm, s0c, lane);
            rn[tm] = h4(f4(op_tr(sm.Rn, LDH, 16 * tm, c0, lane)) - ld4(sm.gamn + 16 * tm + 4 * g4) * x);
            settle(rn[tm]);
        }
        reread();
        // ---- the solves (wave 1 noisy, wave 0 clean) and Gram tiles (P, K~ Q~^T, K~ K~^T)
        if (wave == 1) {
            solve_block(sm.Kn, sm.G2n, sm.betn, sm.Mn, lane);
        } else if (PREP && wave == 0) {
            solve_block(sm.K, sm.G2, sm.bet, sm.Mc, lane);
        } else if (wave >= 2) {
            for (int e = wave - 2; e < (PREP ? 12 : 8); e += 6) {
                const int gram = e >> 2, m0 = 16 * ((e >> 1) & 1), n0 = 16 * (e & 1), i = n0 + rr;
                const _Float16 *A = gram == 2 ? sm.Q : sm.Kn, *B = gram == 2 ? sm.K : (gram == 1 ? sm.Qn : sm.Kn);
                const f32x4 c = tile_mma<_Float16, DD>(z, A + m0 * LDH, LDH, B + n0 * LDH, LDH, lane);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int t = m0 + 4 * g4 + j;
                    if (gram == 0)
                        sm.KK[t * LDF + i] = c[j];
                    else if (gram == 1)
                        sm.Pn[t * LDM + i] = (_Float16)c[j];
                    else
                        sm.Ph[t * LDM + i] = (_Float16)(i <= t ? c[j] * ex(sm.G[t] - sm.G[i]) : 0.f);
                }
            }
        }
        __syncthreads();
        // ---- this wave's columns: Delta~, dDelta~, dV~, b = -Gamma~ dR~, the c term, U K
        float roww[2][4];
        f16x4 dl[2], dd[2], bq[2];
        {
            const f16x4 dob[2] = {op_tr(sm.dOn, LDH, 0, c0, lane), op_tr(sm.dOn, LDH, 16, c0, lane)};
#pragma unroll
            for (int tm = 0; tm < 2; ++tm) {
                put_tile(sm.Rn, LDH, 16 * tm, col, rn[tm], g4);
                const f32x4 dn = apply_T(sm.Mn, sm.betn, 16 * tm, rn, lane);
                dl[tm] = h4(dn);
                const f32x4 d = s * ld4(sm.Dn + 16 * tm + 4 * g4) * apply(sm.Pn, 16 * tm, dob, z, lane);
                dd[tm] = h4(d);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    roww[tm][j] = d[j] * dn[j];
                    settle(roww[tm][j]);
                }
            }
#pragma unroll
            for (int tm = 0; tm < 2; ++tm) {
                const f32x4 c = apply_Tt(sm.Mn, sm.betn, 16 * tm, dd, lane);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int t = 16 * tm + 4 * g4 + j;
                    if (t < nvalid) pn.dv[(long)t * vs + col] = c[j] * inv;
                }
                bq[tm] = h4(-ld4(sm.gamn + 16 * tm + 4 * g4) * c);
            }
            f16x4 *ct = reinterpret_cast<f16x4 *>(a.cterm + (size_t)uw * DD * DD) + wave * 64 + lane;
            if constexpr (PREP) {
                // dh-independent terms of the clean block: s Q^T Gamma dO - K^T Gamma T^T (s P^T dO)
                const f16x4 doc[2] = {op_tr(sm.dO, LDH, 0, c0, lane), op_tr(sm.dO, LDH, 16, c0, lane)};
                f16x4 yq[2], drq[2], sd[2], kd[2];
                const float Ge = sm.G[NP - 1];
#pragma unroll
                for (int tm = 0; tm < 2; ++tm) yq[tm] = h4(s * apply_t(sm.Ph, LDM, 16 * tm, doc, z, lane));
#pragma unroll
                for (int tm = 0; tm < 2; ++tm) {
                    const f32x4 gm = ld4(sm.gam + 16 * tm + 4 * g4);
                    drq[tm] = h4(-gm * apply_Tt(sm.Mc, sm.bet, 16 * tm, yq, lane));
                    sd[tm] = scale4(doc[tm], s * gm);
                    f32x4 d;
#pragma unroll
                    for (int j = 0; j < 4; ++j) d[j] = ex(Ge - sm.G[16 * tm + 4 * g4 + j]);
                    kd[tm] = scale4(op_tr(sm.K, LDH, 16 * tm, c0, lane), d);
                }
                // U K = Gamma diag(beta) M^T (D K)
                _Float16 *uk = a.uk + (size_t)uw * NP * DD;
#pragma unroll
                for (int tm = 0; tm < 2; ++tm) {
                    // the transpose from the swapped operands, in the scan's order
                    const float f = sm.gam[16 * tm + rr] * sm.bet[16 * tm + rr];
                    const f32x4 u = mfma2(kd[0], kd[1], op_tr(sm.Mc, LDM, 0, 16 * tm, lane),
                                          op_tr(sm.Mc, LDM, 16, 16 * tm, lane), z);
                    put_uk(uk, tm, wave, lane, h4(f * u));
                }
                // the c term; s gamma~_n on the fp32 product, not on the fp16 rows
#pragma unroll
                for (int tm = 0; tm < 8; ++tm) {
                    f32x4 c = sgn * apply_t(sm.Qn, LDH, 16 * tm, dob, z, lane);
                    c = apply_t(sm.K, LDH, 16 * tm, drq, c, lane);
                    c = apply_t(sm.Q, LDH, 16 * tm, sd, c, lane);
                    ct[tm * 8 * 64] = h4(apply_t(sm.Kn, LDH, 16 * tm, bq, c, lane));
                }
                if (tid == 0) a.gnb[uw] = ex(Ge);
            } else {
#pragma unroll
                for (int tm = 0; tm < 8; ++tm) {
                    const f32x4 c = sgn * apply_t(sm.Qn, LDH, 16 * tm, dob, z, lane);
                    ct[tm * 8 * 64] = h4(f4(ct[tm * 8 * 64]) + apply_t(sm.Kn, LDH, 16 * tm, bq, c, lane));
                }
            }
        }
        f16x8 s0r[4];   // the seed's rows, for the products with S0^T below
        load_rows16(s0r, seed, c0, lane);
        __syncthreads();   // the clean rows are read: Delta~, dDelta~, b in their place
#pragma unroll
        for (int tm = 0; tm < 2; ++tm) {
            put_tile(Dln, LDH, 16 * tm, col, dl[tm], g4);
            put_tile(dDn, LDH, 16 * tm, col, dd[tm], g4);
            put_tile(Bn, LDH, 16 * tm, col, bq[tm], g4);
        }
        __syncthreads();
        // ---- dPh = s (dO~ Delta~^T) D~ (waves 0 .. 3), dT = dDelta~ R~^T (waves 4 .. 7); products with S0^T
        {
            const int m0 = 16 * ((wave >> 1) & 1), n0 = 16 * (wave & 1), i = n0 + rr;
            const bool lo = wave < 4;
            const f32x4 e = tile_mma<_Float16, DD>(z, (lo ? sm.dOn : dDn) + m0 * LDH, LDH, (lo ? Dln : sm.Rn) + n0 * LDH,
                                                   LDH, lane);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int t = m0 + 4 * g4 + j;
                if (lo)
                    dPh[t * LDM + i] = (_Float16)(s * e[j] * sm.Dn[i]);
                else
                    dT[t * LDF + i] = e[j];
            }
        }
        float rowa[2][4], rowb[2][4];
        f32x4 ca[2], cb[2];
        const f16x4 knq[2] = {op_tr(sm.Kn, LDH, 0, c0, lane), op_tr(sm.Kn, LDH, 16, c0, lane)};
        const f16x4 qnq[2] = {op_tr(sm.Qn, LDH, 0, c0, lane), op_tr(sm.Qn, LDH, 16, c0, lane)};
#pragma unroll
        for (int tm = 0; tm < 2; ++tm) {
            ca[tm] = sgn * rows_times(sm.dOn, 16 * tm, s0r, lane);
            cb[tm] = rows_times(Bn, 16 * tm, s0r, lane);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                rowa[tm][j] = ca[tm][j] * (float)qnq[tm][j];
                rowb[tm][j] = cb[tm][j] * (float)knq[tm][j];
            }
        }
        __syncthreads();
        // ---- dQ~; dK~ but for the dKK term; the dA products
        if (wave < 4)
            dA_first(dT, sm.Mn, sm.betn, Wm, wave, lane);
        else if (wave == 4 && lane < NP)
            sm.dB[lane] = dbeta_T(dT, sm.Mn, lane);
#pragma unroll
        for (int tm = 0; tm < 2; ++tm) {
            const f32x4 c = apply(dPh, 16 * tm, knq, ca[tm], lane);
            cb[tm] = apply_t(dPh, LDM, 16 * tm, qnq, cb[tm], lane);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int t = 16 * tm + 4 * g4 + j;
                if (t < nvalid) put_qk(add_qk, pn.dq + (long)t * qks + col, c[j] * inv);
                const float xa = row_total(rowa[tm][j]), xb = row_total(rowb[tm][j]), xw = row_total(roww[tm][j]);
                if (rr == 15) {
                    sm.pA[wave][t] = xa;
                    sm.pB[wave][t] = xb;
                    sm.pW[wave][t] = xw;
                }
            }
        }
        __syncthreads();
        if (wave < 4) dA_second(sm.Mn, Wm, dA, wave, lane);
        __syncthreads();
        dA_terms(dA, sm.KK, sm.Gn, sm.betn, Wh, sm.dB, sm.part[wave], wave, lane);
        __syncthreads();
#pragma unroll
        for (int tm = 0; tm < 2; ++tm) {
            const f32x4 c = apply(Wh, 16 * tm, knq, cb[tm], lane);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int t = 16 * tm + 4 * g4 + j;
                if (t < nvalid) put_qk(add_qk, pn.dk + (long)t * qks + col, c[j] * inv);
            }
        }
        if (wave == 0) {
            // dg: row terms summed from the block's end back, the block-end terms of all rows, and of
            // dDelta~ . Delta~, a block-end term less a row term, what is left: the rows before
            float x = 0.f, e = 0.f, before = 0.f;
            if (lane < NP) {
#pragma unroll
                for (int w = 0; w < kWaves; ++w) {
                    x += sm.part[w][lane] + sm.pB[w][lane];
                    e += sm.pA[w][lane];
                    if (lane > 0) before += sm.pW[w][lane - 1];
                }
            }
            x = back_sum32(x, lane) + wave_total(e) + ut::scan32(before, lane);
            if (lane < nvalid) {
                pn.dg[(long)lane * a.h_v] = x * inv;
                pn.db[(long)lane * a.h_v] = sm.dB[lane] * inv;
            }
        }
        if (vi + 1 < r) __syncthreads();   // LDS is free for the next v-head
    }
}

struct CleanSmem {
    _Float16 Q[NP * LDH], K[NP * LDH];
    _Float16 R[NP * LDH];     // v, then R
    _Float16 dO[NP * LDH];    // then, fp32, W
    _Float16 Dl[NP * LDH];    // first the waves' tiles being turned over
    _Float16 dDl[NP * LDH];   // then, fp32, dA
    _Float16 dR[NP * LDH];    // -Gamma dR
    _Float16 Mh[NP * LDM], Ph[NP * LDM], dPh[NP * LDM], Wh[NP * LDM];
    float KK[NP * LDF], dT[NP * LDF];
    float G[NP], G2[NP], gam[NP], bet[NP], dB[NP];
    // per-wave partial sums of the gate gradient, which is summed from the block's end back: what a
    // position would add and take off again is left out, since under strong decays the rest is of the
    // decay's order and its rounding is not
    float part[kWaves][NP];
};
static_assert(sizeof(CleanSmem) <= 80 * 1024, "two workgroups per CU");

// Phase 3: every clean block, in parallel, from its seed and the gradient at its end (dh,
// written by the scan); one workgroup per (block, q/k head).  SMALL: the chunk's small noisy
// blocks have left their shares: xd, of dDelta, and the starting values of dk and dg, to which
// this pass adds.
template <typename Od, bool SMALL> __global__ void __launch_bounds__(512, 4) bdgdn_bwd_clean_kernel(BwdArgs a)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    CleanSmem &sm = *reinterpret_cast<CleanSmem *>(smem_raw);
    float *const Wm = reinterpret_cast<float *>(sm.dO), *const dA = reinterpret_cast<float *>(sm.dDl);
    const int r = a.h_v / a.h_qk;
    const float s = a.scale, inv = a.range[1];
    const f32x4 z = {0.f, 0.f, 0.f, 0.f};
    const long qks = (long)a.h_qk * DD, vs = (long)a.h_v * DD;
    const int gb = blockIdx.x / a.h_qk, hq = blockIdx.x % a.h_qk;
    long p0;
    int n, nvalid;
    block_unit(a, gb, n, p0, nvalid);
    for (int vi = 0; vi < r; ++vi) {
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));   // lane-dependent addresses recomputed per unit, not kept live
        const int lane = tid & 63, g4 = lane >> 4, rr = lane & 15;
        const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), c0 = 16 * wave, col = c0 + rr;
        const int h = hq * r + vi;
        const long uw = (long)gb * a.h_v + h;
        const StreamPtrs p = stream_ptrs<Od>(a, false, p0, h, hq);
        const bool add_qk = vi > 0;
        const _Float16 *seed = a.seeds + (size_t)uw * DD * DD;
        const f16x4 *dh = reinterpret_cast<const f16x4 *>(a.dh + (size_t)uw * DD * DD) + lane;   // 64 tiles
        _Float16 *Z = sm.Dl + 256 * wave;
        // ---- rows and gates; the columns of the seed and of dh
        f16x4 s0c[8], dsc[8];
        {
            load_cols(s0c, seed, c0, lane);
#pragma unroll
            for (int kb = 0; kb < 8; ++kb) dsc[kb] = dh[(kb * 8 + wave) * 64];
            const BlockRows<Od, true> in = load_block<Od, true>(p, a.h_qk, a.h_v, nvalid, tid);
            store_rows(sm.Q, in.q, tid);
            store_rows(sm.K, in.k, tid);
            store_rows(sm.R, in.v, tid);
            store_rows(sm.dO, in.dout, tid, a.range[0]);
            if (wave == 0) {
                cum_to_lds(in.g, sm.G, sm.G2, sm.gam, lane);
                if (lane < NP) sm.bet[lane] = in.b;
            }
            if (tid < kWaves * NP) sm.part[tid / NP][tid % NP] = 0.f;
#pragma unroll
            for (int kb = 0; kb < 8; ++kb) s0c[kb] = turn(Z, s0c[kb], lane);
        }
        __syncthreads();
        const float Ge = sm.G[NP - 1];
        // this lane's shares of the gate gradient: rowg[tm][j] for row 16 tm + 4 g + j, dlast for
        // the last position
        float rowg[2][4], dlast = 0.f;
        // ---- R = V - Gamma K S0, K dS (first: their operands are free for the solve's registers)
        f16x4 rq[2];
        f32x4 kds[2];
#pragma unroll
        for (int tm = 0; tm < 2; ++tm) {
            const f32x4 x = rows_times(sm.K, 16 * tm, s0c, lane);
            kds[tm] = rows_times(sm.K, 16 * tm, dsc, lane);
            rq[tm] = h4(f4(op_tr(sm.R, LDH, 16 * tm, c0, lane)) - ld4(sm.gam + 16 * tm + 4 * g4) * x);
        }
        {   // gamma_n <dS_n, S0>
            float w = 0.f;
#pragma unroll
            for (int kb = 0; kb < 8; ++kb)
#pragma unroll
                for (int j = 0; j < 4; ++j) w = fmaf((float)dsc[kb][j], (float)s0c[kb][j], w);
            dlast = ex(Ge) * w;
        }
        settle(dlast);
#pragma unroll
        for (int tm = 0; tm < 2; ++tm) {
            settle(rq[tm]);
            settle(kds[tm]);
        }
        reread();
        // ---- the solve (wave 0) and Gram tiles: K K^T (waves 1 .. 3), P = (Q K^T) o Mc (waves 4 .. 7, which
        // keep their tile of Q K^T in fp32 for its gate terms: at g = -8 an entry of P is below fp16's
        // normal range, and with it dg was 7e-4 of its 2-norm off, where 3e-4 are left)
        const int m0 = 16 * ((wave >> 1) & 1), n0 = 16 * (wave & 1);
        f32x4 qk = z;
        if (wave == 0) {
            solve_block(sm.K, sm.G2, sm.bet, sm.Mh, lane);
        } else if (wave < 4) {
            for (int e = wave - 1; e < 4; e += 3) {
                const int mk = 16 * (e >> 1), nk = 16 * (e & 1);
                const f32x4 c = tile_mma<_Float16, DD>(z, sm.K + mk * LDH, LDH, sm.K + nk * LDH, LDH, lane);
#pragma unroll
                for (int j = 0; j < 4; ++j) sm.KK[(mk + 4 * g4 + j) * LDF + nk + rr] = c[j];
            }
        } else {
            qk = tile_mma<_Float16, DD>(z, sm.Q + m0 * LDH, LDH, sm.K + n0 * LDH, LDH, lane);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int t = m0 + 4 * g4 + j, i = n0 + rr;
                sm.Ph[t * LDM + i] = (_Float16)(i <= t ? qk[j] * ex(sm.G[t] - sm.G[i]) : 0.f);
            }
        }
        reread();
        // the rows of the seed and of dh, for the products with S0^T and dS^T
        f16x8 s0r[4];
        f16x4 dsr[8];
        load_rows16(s0r, seed, c0, lane);
#pragma unroll
        for (int kb = 0; kb < 8; ++kb) dsr[kb] = dh[(wave * 8 + kb) * 64];
#pragma unroll
        for (int kb = 0; kb < 8; ++kb) dsr[kb] = turn(Z, dsr[kb], lane);
        __syncthreads();
        // ---- this wave's columns: Delta, dDelta = s P^T dO + D K dS (+ xd), dR = T^T dDelta = dV
        {
            const f16x4 doc[2] = {op_tr(sm.dO, LDH, 0, c0, lane), op_tr(sm.dO, LDH, 16, c0, lane)};
            f16x4 dd[2];
#pragma unroll
            for (int tm = 0; tm < 2; ++tm) {
                put_tile(sm.R, LDH, 16 * tm, col, rq[tm], g4);
                const f16x4 dl = h4(apply_T(sm.Mh, sm.bet, 16 * tm, rq, lane));
                put_tile(sm.Dl, LDH, 16 * tm, col, dl, g4);
                f32x4 d = s * apply_t(sm.Ph, LDM, 16 * tm, doc, z, lane);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int t = 16 * tm + 4 * g4 + j;
                    const float w = ex(Ge - sm.G[t]) * kds[tm][j];
                    d[j] += w;
                    // the last position's own term would be taken off itself
                    rowg[tm][j] = t < nvalid - 1 ? -w * (float)dl[j] : 0.f;
                    dlast -= rowg[tm][j];
                }
                if constexpr (SMALL)
                    d += (reinterpret_cast<const f32x4 *>(a.xd + (size_t)uw * NP * DD) + tid)[tm * 8 * 64];
                dd[tm] = h4(d);
                put_tile(sm.dDl, LDH, 16 * tm, col, dd[tm], g4);
            }
#pragma unroll
            for (int tm = 0; tm < 2; ++tm) {
                const f32x4 c = apply_Tt(sm.Mh, sm.bet, 16 * tm, dd, lane);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int t = 16 * tm + 4 * g4 + j;
                    if (t < nvalid) p.dv[(long)t * vs + col] = c[j] * inv;
                }
                put_tile(sm.dR, LDH, 16 * tm, col, h4(-ld4(sm.gam + 16 * tm + 4 * g4) * c), g4);
            }
        }
        __syncthreads();
        // ---- E = dO Delta^T (waves 4 .. 7): the gradient of Q K^T into dPh, the gates of Mc; dT =
        // dDelta R^T (waves 0 .. 3); products with S0^T and dS^T
        {
            const int i = n0 + rr;
            const bool hi = wave >= 4;
            const f32x4 e = tile_mma<_Float16, DD>(z, (hi ? sm.dO : sm.dDl) + m0 * LDH, LDH, (hi ? sm.Dl : sm.R) + n0 * LDH,
                                                   LDH, lane);
            float colw = 0.f;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int t = m0 + 4 * g4 + j;
                if (hi) {
                    const float d = i <= t ? s * e[j] * ex(sm.G[t] - sm.G[i]) : 0.f;
                    // the diagonal, in the row and the column sum of one position, is in neither
                    const float w = i < t ? d * qk[j] : 0.f;
                    sm.dPh[t * LDM + i] = (_Float16)d;
                    if (m0)
                        rowg[1][j] += w;
                    else
                        rowg[0][j] += w;
                    colw += w;
                } else {
                    sm.dT[t * LDF + i] = e[j];
                }
            }
            if (hi) {
                colw += __shfl_xor(colw, 16);
                colw += __shfl_xor(colw, 32);
                if (g4 == 0) lds_add(&sm.part[wave][i], -colw);
            }
        }
        f32x4 ca[2], cb[2];
        const f16x4 kq[2] = {op_tr(sm.K, LDH, 0, c0, lane), op_tr(sm.K, LDH, 16, c0, lane)};
        const f16x4 qq[2] = {op_tr(sm.Q, LDH, 0, c0, lane), op_tr(sm.Q, LDH, 16, c0, lane)};
#pragma unroll
        for (int tm = 0; tm < 2; ++tm) {
            ca[tm] = s * ld4(sm.gam + 16 * tm + 4 * g4) * rows_times(sm.dO, 16 * tm, s0r, lane);
            cb[tm] = rows_times(sm.dR, 16 * tm, s0r, lane);
            const f32x4 cd = rows_times(sm.Dl, 16 * tm, dsr, lane);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                rowg[tm][j] += ca[tm][j] * (float)qq[tm][j] + cb[tm][j] * (float)kq[tm][j];
                cb[tm][j] += ex(Ge - sm.G[16 * tm + 4 * g4 + j]) * cd[j];
            }
        }
        __syncthreads();
        // ---- dQ; dK but for the dKK term; the dA products
        if (wave < 4)
            dA_first(sm.dT, sm.Mh, sm.bet, Wm, wave, lane);
        else if (wave == 4 && lane < NP)
            sm.dB[lane] = dbeta_T(sm.dT, sm.Mh, lane);
#pragma unroll
        for (int tm = 0; tm < 2; ++tm) {
            const f32x4 c = apply(sm.dPh, 16 * tm, kq, ca[tm], lane);
            cb[tm] = apply_t(sm.dPh, LDM, 16 * tm, qq, cb[tm], lane);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int t = 16 * tm + 4 * g4 + j;
                if (t < nvalid) put_qk(add_qk, p.dq + (long)t * qks + col, c[j] * inv);
            }
        }
        {   // the row gate terms: this wave's partial sums
            const float dl = wave_total(dlast);
#pragma unroll
            for (int tm = 0; tm < 2; ++tm)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int t = 16 * tm + 4 * g4 + j;
                    const float x = row_total(rowg[tm][j]);
                    if (rr == 15) sm.part[wave][t] += t == NP - 1 ? x + dl : x;
                }
        }
        __syncthreads();
        if (wave < 4) dA_second(sm.Mh, Wm, dA, wave, lane);
        __syncthreads();
        dA_terms(dA, sm.KK, sm.G, sm.bet, sm.Wh, sm.dB, sm.part[wave], wave, lane);
        __syncthreads();
#pragma unroll
        for (int tm = 0; tm < 2; ++tm) {
            const f32x4 c = apply(sm.Wh, 16 * tm, kq, cb[tm], lane);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int t = 16 * tm + 4 * g4 + j;
                if (t < nvalid) put_qk(SMALL || add_qk, p.dk + (long)t * qks + col, c[j] * inv);
            }
        }
        if (wave == 0) {   // dg = reverse cumulative sum of the gate terms
            float x = 0.f;
            if (lane < NP) {
#pragma unroll
                for (int w = 0; w < kWaves; ++w) x += sm.part[w][lane];
            }
            x = back_sum32(x, lane);
            if (lane < nvalid) {
                put_qk(SMALL, p.dg + (long)lane * a.h_v, x * inv);
                p.db[(long)lane * a.h_v] = sm.dB[lane] * inv;
            }
        }
        if (vi + 1 < r) __syncthreads();   // LDS is free for the next v-head
    }
}
