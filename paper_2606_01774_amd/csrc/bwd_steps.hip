// bwd_steps.hip -- the per-step fp32 backward of the two-stream training forward, parallel
// over blocks (Appendix "Backward primitives": eq. per-step-bwd, eq. noisy-readout-bwd,
// eq. dh-block-recursion), for the shapes outside the block-form backward of
// bwd_kernels.hip: fp32 inputs, d_k or d_v of 64, odd blocks of 33 to 63 positions.
//
// Forward step i (alpha = exp g):  u = v - alpha S^T k,  S' = alpha S + beta k u^T.
// Backward from the gradient dS' of S' (a clean step first adds s q do^T to it):
//     w = dS'^T k,  dv = beta w,  dbeta = w . u,  dk = beta (dS' u - alpha S w),
//     dS = alpha (dS' - beta k w^T),  clean: dq = s S' do.
// Neither recurrence needs the other's states: S runs forwards from k, v, gates; dS runs
// backwards from k, q, do, gates and the noisy seeds' gradients.  So only those two walks
// are serial, and everything else is done for all blocks at once:
//   1. states: the clean state before every block (one wave per 4 columns of a chain);
//   2. noisy blocks in parallel from their seeds: every gradient, and the seed's gradient;
//   3. reverse: the gradient dh of the state at every block's end (one wave per 4 columns),
//      stored over the seed gradients it has consumed;
//   4. clean blocks in parallel from the state at their start and dh.
// A block (2, 4) is two walks over its positions: forwards for u (and the clean dq), then
// backwards for w, dv, dbeta, dk and dg.  The second needs the state before each position, which
// a step of the first cannot be run back to (it would divide by alpha): four positions at a time
// it is rebuilt from the block's seed or the state kept at the block's middle by the steps' stored
// u, S' = alpha S + beta k u^T, which sums over nothing.  The gate gradient is the inner product
// dg = <dS^, alpha S> (dS^ the gradient of the decayed state), every term of which carries alpha: a
// running sum dg_(i-1) = dg_i + do.o - dv.v over the block, though it needs no states, leaves the
// rounding of terms of order one in a result of order alpha (7e-4 of it at g = -8, 40 times it at
// g = -20).
//
// Layout: 16 lanes of a DPP row share a column's rows (d_k / 16 consecutive rows each), so a
// column sum over rows is four DPP adds; the four DPP rows hold different columns.  Row sums
// over columns go over the DPP rows by permlane swaps and over waves through LDS, in a fixed
// order (deterministic, no atomics; the v-heads of a q/k head are added in turn).
//
// What bounds it: the instructions of the two serial walks, one wave in order (0.11 us per
// step forwards, 0.15 us backwards), and in the block kernels a walk of a block each way and the
// states rebuilt in between.
// Measured at 1 x 256 + 256 tokens, 2 heads, d = 64, L = 16 in fp32: states 28 to 32 us by box, noisy
// 27 us, reverse 38 us, clean 25 us; the one-wave walk of bwd_generic.hip, whose steps waited
// for loads and for two butterflies over the columns each, 4.04 ms.  The walks' 4-column
// tiles and per-chunk row pointers: 41 + 53 us with a 64-bit row product per position.
#include "bwd.hpp"
#include "common.hpp"
#include "kernels.hpp"
#include "ut.hpp"

namespace bdgdn {

namespace {

constexpr int kSpan = 4;        // positions per row-sum exchange between the waves of a block
constexpr int kMaxL = 64;
constexpr int kStepStreams = 5; // the clean stream and up to four noisy views

struct StepStream {
    const void *q, *k, *v;
    const float *g, *beta;
    const void *dout;
    float *dq, *dk, *dv, *dg, *db;
};

struct StepArgs {
    StepStream st[kStepStreams];   // 0 clean, 1 .. n_views noisy
    int n_views;
    const int32_t *cu;             // packed documents, or null
    int n_seq;
    const float *h0, *dht;
    float *dh0;
    float *seeds;                  // [block][h_v][d_v][d_k]: the clean state before each block
    float *dh;                     // same: the seed's gradient, then the gradient at the block's end
    int T, L, nblk, h_qk, h_v;
    float scale;
};

// NR consecutive elements, loaded as a whole.
template <typename T, int NR> struct alignas(sizeof(T) * NR > 16 ? 16 : sizeof(T) * NR) Vec {
    T v[NR];
};
template <typename T, int NR> __device__ __forceinline__ Vec<T, NR> ldv(const T *p)
{
    return *reinterpret_cast<const Vec<T, NR> *>(p);
}

// x summed over the 16 lanes of each DPP row, in every lane
__device__ __forceinline__ float row16_sum(float x)
{
    x += ut::dpp<0x128>(x);   // row_ror:8
    x += ut::dpp<0x124>(x);
    x += ut::dpp<0x122>(x);
    x += ut::dpp<0x121>(x);
    return x;
}
// a in the lower and b in the upper 32 lanes, each summed with the other half's value
__device__ __forceinline__ float swap32_sum(float a, float b)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, a), __builtin_bit_cast(unsigned, b),
                                                    false, false);
    return __builtin_bit_cast(float, (unsigned)r[0]) + __builtin_bit_cast(float, (unsigned)r[1]);
}
// the same between neighbouring DPP rows: a in the even rows, b in the odd rows
__device__ __forceinline__ float swap16_sum(float a, float b)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, a), __builtin_bit_cast(unsigned, b),
                                                    false, false);
    return __builtin_bit_cast(float, (unsigned)r[0]) + __builtin_bit_cast(float, (unsigned)r[1]);
}
__device__ __forceinline__ float rows4_sum(float x)
{
    x = swap32_sum(x, x);
    return swap16_sum(x, x);
}
// x[m] (m < NR) summed over the four DPP rows; lane (cg, rl) ends with the sums of rows
// cg NR / 4 .. cg NR / 4 + NR / 4 - 1 of its NR rows in y
template <int NR> __device__ __forceinline__ void rows4_scatter(const float (&x)[NR], float (&y)[NR / 4])
{
    float z[NR / 2];
#pragma unroll
    for (int m = 0; m < NR / 2; ++m) z[m] = swap32_sum(x[m], x[m + NR / 2]);
#pragma unroll
    for (int m = 0; m < NR / 4; ++m) y[m] = swap16_sum(z[m], z[m + NR / 4]);
}

// A chain's first row, length and the workspace unit of its first block.
__device__ __forceinline__ void chain_span(const StepArgs &a, int seq, long &base, long &len, long &blk0)
{
    if (a.cu) {
        base = a.cu[seq];
        len = (long)a.cu[seq + 1] - base;
        blk0 = base / a.L;   // documents start on block boundaries
    } else {
        base = (long)seq * a.T;
        len = a.T;
        blk0 = (long)seq * a.nblk;
    }
}

// The (chain, 4-column tile) of a one-wave workgroup: the tiles of a chain on one XCD
// (workgroups are dealt to the 8 XCDs in turn), so that they share its k and q rows in L2.
template <int DV> __device__ __forceinline__ bool walk_unit(const StepArgs &a, int &seq, int &h, int &tile)
{
    constexpr int NT = DV / 4;
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int chain = slot / NT * 8 + xcd;
    tile = slot % NT;
    seq = chain / a.h_v;
    h = chain % a.h_v;
    return chain < a.n_seq * a.h_v;
}
template <int DV> unsigned walk_grid(const StepArgs &a)
{
    const long chains = (long)a.n_seq * a.h_v;
    return (unsigned)((chains + 7) / 8 * 8 * (DV / 4));
}

}  // namespace

// Phase 1: the clean state before every block of each chain, column-major.  Bound by the
// instructions of one step after another (one wave per 4 columns, P positions of loads in
// flight behind the P being walked).
template <typename In, int DK, int DV>
__global__ void __launch_bounds__(64) bdgdn_bwd_steps_states_kernel(StepArgs a)
{
    constexpr int NR = DK / 16, P = 8;
    int seq, h, tile;
    if (!walk_unit<DV>(a, seq, h, tile)) return;
    const int lane = threadIdx.x, rl = lane & 15, col = 4 * tile + (lane >> 4), hq = h / (a.h_v / a.h_qk);
    long base, len, blk0;
    chain_span(a, seq, base, len, blk0);
    float S[NR];
#pragma unroll
    for (int m = 0; m < NR; ++m)
        S[m] = a.h0 ? a.h0[((long)(seq * a.h_v + h) * DK + rl * NR + m) * DV + col] : 0.f;
    if (len <= 0) return;
    // uniform row pointers and one lane offset each
    const In *kp = static_cast<const In *>(a.st[0].k) + (base * a.h_qk + hq) * DK;
    const In *vp = static_cast<const In *>(a.st[0].v) + (base * a.h_v + h) * DV;
    const unsigned ko = rl * NR, vo = col;
    const long qks = (long)a.h_qk * DK, vs = (long)a.h_v * DV;
    const float *gp = a.st[0].g + base * a.h_v + h, *bp = a.st[0].beta + base * a.h_v + h;
    struct Buf {
        Vec<In, NR> k[P];
        In v[P];
    };
    // the P positions from the running row pointers on (whole chunks without a row index)
    const In *kc = kp, *vc = vp;
    auto fetch = [&](Buf &b, long i0) {
        if (i0 + P <= len) {
#pragma unroll
            for (int j = 0; j < P; ++j) {
                b.k[j] = ldv<In, NR>(kc + j * qks + ko);
                b.v[j] = (vc + j * vs)[vo];
            }
            kc += P * qks;
            vc += P * vs;
        } else {
#pragma unroll
            for (int j = 0; j < P; ++j) {
                const long i = i0 + j < len ? i0 + j : len - 1;
                b.k[j] = ldv<In, NR>(kp + i * qks + ko);
                b.v[j] = (vp + i * vs)[vo];
            }
        }
    };
    auto gate_row = [&](long i0) { return (i0 + lane < len ? i0 + lane : len - 1) * a.h_v; };
    // gates of 64 positions, one a lane, the next 64 in flight
    float ng = gp[gate_row(0)], nb = bp[gate_row(0)], al = 0.f, be = 0.f;
    int left = 0;      // positions to the next block start
    float *seed = a.seeds + ((blk0 * a.h_v + h) * DV + col) * (long)DK + rl * NR;
    auto walk = [&](const Buf &b, long i0) {
        if ((i0 & 63) == 0) {
            al = expf(ng);
            be = nb;
            ng = gp[gate_row(i0 + 64)];
            nb = bp[gate_row(i0 + 64)];
        }
#pragma unroll
        for (int j = 0; j < P; ++j) {
            if (i0 + j >= len) break;
            if (left == 0) {
#pragma unroll
                for (int m = 0; m < NR; m += 4) st4(seed + m, S[m], S[m + 1], S[m + 2], S[m + 3]);
                seed += (long)a.h_v * DV * DK;
                left = a.L;
            }
            --left;
            const int at = (int)(i0 & 63) + j;
            const float alpha = ut::lane_value(al, at), beta = ut::lane_value(be, at);
            float k[NR], x = 0.f;
#pragma unroll
            for (int m = 0; m < NR; ++m) {
                k[m] = to_f(b.k[j].v[m]);
                x = fmaf(k[m], S[m], x);
            }
            const float bu = beta * (to_f(b.v[j]) - alpha * row16_sum(x));
#pragma unroll
            for (int m = 0; m < NR; ++m) S[m] = fmaf(alpha, S[m], k[m] * bu);   // the rounding of the product is the small one
        }
    };
    Buf b0, b1;
    fetch(b0, 0);
    for (long i = 0; i < len; i += 2 * P) {
        fetch(b1, i + P);
        walk(b0, i);
        if (i + P >= len) break;
        fetch(b0, i + 2 * P);
        walk(b1, i + P);
    }
}

// Phase 3: the reverse walk of the clean state gradient: dh at every block's end over the
// block's seed gradient (read before), the seed gradient added at the block's start; dh0.
template <typename In, typename Out, int DK, int DV>
__global__ void __launch_bounds__(64) bdgdn_bwd_steps_reverse_kernel(StepArgs a)
{
    constexpr int NR = DK / 16, P = 8;
    int seq, h, tile;
    if (!walk_unit<DV>(a, seq, h, tile)) return;
    const int lane = threadIdx.x, rl = lane & 15, col = 4 * tile + (lane >> 4), hq = h / (a.h_v / a.h_qk);
    long base, len, blk0;
    chain_span(a, seq, base, len, blk0);
    float dS[NR];
    const long edge = ((long)(seq * a.h_v + h) * DK + rl * NR) * DV + col;   // of h0, dht, dh0
#pragma unroll
    for (int m = 0; m < NR; ++m) dS[m] = a.dht ? a.dht[edge + (long)m * DV] : 0.f;
    if (len > 0) {
        const In *kp = static_cast<const In *>(a.st[0].k) + (base * a.h_qk + hq) * DK;
        const In *qp = static_cast<const In *>(a.st[0].q) + (base * a.h_qk + hq) * DK;
        const Out *dp = static_cast<const Out *>(a.st[0].dout) + (base * a.h_v + h) * DV;
        const unsigned ko = rl * NR, vo = col;
        const long qks = (long)a.h_qk * DK, vs = (long)a.h_v * DV;
        const float *gp = a.st[0].g + base * a.h_v + h, *bp = a.st[0].beta + base * a.h_v + h;
        struct Buf {
            Vec<In, NR> k[P], q[P];
            Out d[P];
        };
        // position j of the walk is row len - 1 - j
        const In *kc = kp + (len - 1) * qks, *qc = qp + (len - 1) * qks;
        const Out *dc = dp + (len - 1) * vs;
        auto fetch = [&](Buf &b, long j0) {
            if (j0 + P <= len) {
#pragma unroll
                for (int j = 0; j < P; ++j) {
                    b.k[j] = ldv<In, NR>(kc - j * qks + ko);
                    b.q[j] = ldv<In, NR>(qc - j * qks + ko);
                    b.d[j] = (dc - j * vs)[vo];
                }
                kc -= P * qks;
                qc -= P * qks;
                dc -= P * vs;
                return;
            }
#pragma unroll
            for (int j = 0; j < P; ++j) {
                const long i = len - 1 - j0 - j > 0 ? len - 1 - j0 - j : 0;
                b.k[j] = ldv<In, NR>(kp + i * qks + ko);
                b.q[j] = ldv<In, NR>(qp + i * qks + ko);
                b.d[j] = (dp + i * vs)[vo];
            }
        };
        auto gate_row = [&](long j0) { return (len - 1 - j0 - lane > 0 ? len - 1 - j0 - lane : 0) * a.h_v; };
        float ng = gp[gate_row(0)], nb = bp[gate_row(0)], al = 0.f, be = 0.f;
        const long unit = (long)a.h_v * DV * DK;
        const long nblk = (len + a.L - 1) / a.L;
        float *slot = a.dh + (((blk0 + nblk - 1) * a.h_v + h) * DV + col) * (long)DK + rl * NR;   // the last block's
        int left = (int)(len - (nblk - 1) * a.L);   // positions of the current block still to walk
        float cur[NR];   // the seed gradient of the current block
        bool ends = true;   // the next position is its block's last
        auto walk = [&](const Buf &b, long j0) {
            if ((j0 & 63) == 0) {
                al = expf(ng);
                be = nb;
                ng = gp[gate_row(j0 + 64)];
                nb = bp[gate_row(j0 + 64)];
            }
#pragma unroll
            for (int j = 0; j < P; ++j) {
                if (j0 + j >= len) break;
                if (ends) {   // the seed gradient out of the block's slot, dh into it
#pragma unroll
                    for (int m = 0; m < NR; m += 4) {
                        const f32x4 y = *reinterpret_cast<const f32x4 *>(slot + m);
#pragma unroll
                        for (int e = 0; e < 4; ++e) cur[m + e] = y[e];
                    }
#pragma unroll
                    for (int m = 0; m < NR; m += 4) st4(slot + m, dS[m], dS[m + 1], dS[m + 2], dS[m + 3]);
                    ends = false;
                }
                const int at = (int)(j0 & 63) + j;
                const float alpha = ut::lane_value(al, at), beta = ut::lane_value(be, at);
                const float d = a.scale * to_f(b.d[j]);
                float k[NR], w = 0.f;
#pragma unroll
                for (int m = 0; m < NR; ++m) {
                    k[m] = to_f(b.k[j].v[m]);
                    dS[m] = fmaf(to_f(b.q[j].v[m]), d, dS[m]);
                    w = fmaf(k[m], dS[m], w);
                }
                const float bw = beta * row16_sum(w);
#pragma unroll
                for (int m = 0; m < NR; ++m) dS[m] = alpha * fmaf(-k[m], bw, dS[m]);
                if (--left == 0) {   // the block's start: the noisy seeds' gradient joins
#pragma unroll
                    for (int m = 0; m < NR; ++m) dS[m] += cur[m];
                    slot -= unit;
                    left = a.L;
                    ends = true;
                }
            }
        };
        Buf b0, b1;
        fetch(b0, 0);
        for (long j = 0; j < len; j += 2 * P) {
            fetch(b1, j + P);
            walk(b0, j);
            if (j + P >= len) break;
            fetch(b0, j + 2 * P);
            walk(b1, j + P);
        }
    }
    if (a.dh0) {
#pragma unroll
        for (int m = 0; m < NR; ++m) a.dh0[edge + (long)m * DV] = dS[m];
    }
}

namespace {

// LDS of a block kernel with W = DV / 16 waves: the block's rows, its per-column u and w, the
// row-sum exchange and the per-position sums over columns (one entry per wave).
template <typename In, typename Out, int DK, int DV> struct BlockLds {
    static constexpr int W = DV / 16;
    In *q, *k;       // [L][DK]
    Out *d;          // [L][DV]
    float *u, *w;    // [L][DV]: u holds v until u replaces it
    float *red;      // [W][kSpan][DK]
    float *pb, *pg;  // [L][W]: w . u, <dS^, alpha S>
    float *al, *be;  // [kMaxL]
    static size_t bytes(int L)
    {
        return (size_t)L * (2 * DK * sizeof(In) + DV * sizeof(Out) + 2 * DV * 4 + 2 * W * 4) + W * kSpan * DK * 4 +
               2 * kMaxL * 4;
    }
    __device__ BlockLds(unsigned char *p, int L)
    {
        u = reinterpret_cast<float *>(p);
        w = u + L * DV;
        red = w + L * DV;
        pb = red + W * kSpan * DK;
        pg = pb + L * W;
        al = pg + L * W;
        be = al + kMaxL;
        q = reinterpret_cast<In *>(be + kMaxL);
        k = q + L * DK;
        d = reinterpret_cast<Out *>(k + L * DK);
    }
};

template <typename In, typename Out, int DK, int DV> struct Block {
    static constexpr int NR = DK / 16, W = DV / 16, NT = 64 * W;
    typedef BlockLds<In, Out, DK, DV> Lds;
    const StepArgs &a;
    Lds s;
    int tid, lane, wave, rl, col;   // col: this lane's first of 4 columns
    int n;                          // positions of the block
    f32x4 S[NR];

    __device__ Block(const StepArgs &a_, unsigned char *smem) : a(a_), s(smem, a_.L)
    {
        tid = threadIdx.x;
        lane = tid & 63;
        wave = tid >> 6;
        rl = lane & 15;
        col = 16 * wave + 4 * (lane >> 4);
    }
    // rows of [n][D] elements into LDS, 16 bytes a thread
    template <typename T, int D> __device__ __forceinline__ void stage(T *dst, const T *src, long stride) const
    {
        constexpr int E = 16 / sizeof(T);
        for (int e = tid; e < n * (D / E); e += NT) {
            const int r = e / (D / E), c = e % (D / E) * E;
            *reinterpret_cast<Vec<T, E> *>(dst + r * D + c) = ldv<T, E>(src + r * stride + c);
        }
    }
    __device__ __forceinline__ void load_state(f32x4 (&x)[NR], const float *p) const   // column-major
    {
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int m = 0; m < NR; m += 4) {
                const f32x4 y = *reinterpret_cast<const f32x4 *>(p + (long)(col + c) * DK + rl * NR + m);
#pragma unroll
                for (int e = 0; e < 4; ++e) x[m + e][c] = y[e];
            }
    }
    __device__ __forceinline__ void load_k(float (&x)[NR], const In *rows, int i) const
    {
        const Vec<In, NR> y = ldv<In, NR>(rows + i * DK + rl * NR);
#pragma unroll
        for (int m = 0; m < NR; ++m) x[m] = to_f(y.v[m]);
    }
    template <typename T> __device__ __forceinline__ void load_c(float (&x)[4], const T *rows, int i) const
    {
        const Vec<T, 4> y = ldv<T, 4>(rows + i * DV + col);
#pragma unroll
        for (int c = 0; c < 4; ++c) x[c] = to_f(y.v[c]);
    }
    // this wave's sums over its columns of the row vector x of position i0 + slot
    __device__ __forceinline__ void put_rows(const float (&x)[NR], int slot)
    {
        float y[NR / 4];
        rows4_scatter<NR>(x, y);
        float *p = s.red + (wave * kSpan + slot) * DK + rl * NR + (lane >> 4) * (NR / 4);
#pragma unroll
        for (int m = 0; m < NR / 4; ++m) p[m] = y[m];
    }
    // the waves' row sums of positions i0 .. i0 + cnt - 1 to dst (rows of stride ld): stored,
    // or added to what this same thread stored before
    __device__ __forceinline__ void flush(float *dst, long ld, int i0, int cnt, bool add)
    {
        __syncthreads();
        for (int e = tid; e < cnt * DK; e += NT) {
            const int sl = e / DK, r = e % DK;
            float x = 0.f;
#pragma unroll
            for (int v = 0; v < W; ++v) x += s.red[(v * kSpan + sl) * DK + r];
            float *p = dst + (long)(i0 + sl) * ld + r;
            *p = add ? *p + x : x;
        }
        __syncthreads();
    }

    __device__ __forceinline__ void copy(f32x4 (&x)[NR], const f32x4 (&y)[NR]) const
    {
#pragma unroll
        for (int m = 0; m < NR; ++m)
#pragma unroll
            for (int c = 0; c < 4; ++c) x[m][c] = y[m][c];
    }
    __device__ __forceinline__ void store_state(float *p, const f32x4 (&x)[NR]) const
    {
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int m = 0; m < NR; m += 4)
                st4(p + (long)(col + c) * DK + rl * NR + m, x[m][c], x[m + 1][c], x[m + 2][c], x[m + 3][c]);
    }
    // X, the state before position i, taken on to that before position end by the stored u
    __device__ __forceinline__ void advance(f32x4 (&X)[NR], int i, int end) const
    {
#pragma unroll 1
        for (; i < end; ++i) {
            float k[NR], u[4];
            load_k(k, s.k, i);
            load_c(u, s.u, i);
            const float alpha = s.al[i], beta = s.be[i];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const float bu = beta * u[c];
#pragma unroll
                for (int m = 0; m < NR; ++m) X[m][c] = fmaf(alpha, X[m][c], k[m] * bu);
            }
        }
    }

    // The block of stream st (clean, or a noisy view) for v-head h: rows from row p0; seed: the
    // state at its start; spare: a state's room (the block's slot of dh, free meanwhile) for the
    // state at its middle; dS: clean, the gradient at its end (in); noisy, the gradient of its
    // seed (out).  add: dq, dk add to an earlier v-head's.
    template <bool CLEAN>
    __device__ void run(const StepStream &st, long p0, int h, int hq, const float *seed, float *spare,
                        f32x4 (&dS)[NR], bool add)
    {
        const int half = n / 2 / kSpan * kSpan;   // 0: a short block, no middle state
        const long qks = (long)a.h_qk * DK, vs = (long)a.h_v * DV;
        const long qo = (p0 * a.h_qk + hq) * DK, vo = (p0 * a.h_v + h) * DV, go = p0 * a.h_v + h;
        stage<In, DK>(s.q, static_cast<const In *>(st.q) + qo, qks);
        stage<In, DK>(s.k, static_cast<const In *>(st.k) + qo, qks);
        stage<Out, DV>(s.d, static_cast<const Out *>(st.dout) + vo, vs);
        for (int e = tid; e < n * (DV / 4); e += NT) {   // v as fp32
            const int r = e / (DV / 4), c = e % (DV / 4) * 4;
            const Vec<In, 4> x = ldv<In, 4>(static_cast<const In *>(st.v) + vo + r * vs + c);
            st4(s.u + r * DV + c, to_f(x.v[0]), to_f(x.v[1]), to_f(x.v[2]), to_f(x.v[3]));
        }
        if (tid < n) {
            s.al[tid] = expf(st.g[go + (long)tid * a.h_v]);
            s.be[tid] = st.beta[go + (long)tid * a.h_v];
        }
        load_state(S, seed);
        __syncthreads();
        float *dq = st.dq + qo, *dk = st.dk + qo;
        // forwards: u over v; clean: dq
        for (int i0 = 0; i0 < n; i0 += kSpan) {
            const int cnt = n - i0 < kSpan ? n - i0 : kSpan;
            if (i0 > 0 && i0 == half) store_state(spare, S);
            for (int j = 0; j < cnt; ++j) {
                const int i = i0 + j;
                float k[NR], u[4];
                load_k(k, s.k, i);
                load_c(u, s.u, i);
                const float alpha = s.al[i], beta = s.be[i];
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    float x = 0.f;
#pragma unroll
                    for (int m = 0; m < NR; ++m) x = fmaf(k[m], S[m][c], x);
                    u[c] -= alpha * row16_sum(x);
                    const float bu = beta * u[c];
#pragma unroll
                    for (int m = 0; m < NR; ++m) S[m][c] = fmaf(alpha, S[m][c], k[m] * bu);
                }
                if (rl == 0) st4(s.u + i * DV + col, u[0], u[1], u[2], u[3]);
                if constexpr (CLEAN) read_out(i, j);
            }
            if constexpr (CLEAN) flush(dq, qks, i0, cnt, add);
        }
        if constexpr (!CLEAN) {
            // every position reads the end state: dq_i = s S~ do_i, dS~ = s sum q_i do_i^T
#pragma unroll
            for (int m = 0; m < NR; ++m)
#pragma unroll
                for (int c = 0; c < 4; ++c) dS[m][c] = 0.f;
            for (int i0 = 0; i0 < n; i0 += kSpan) {
                const int cnt = n - i0 < kSpan ? n - i0 : kSpan;
                for (int j = 0; j < cnt; ++j) {
                    read_out(i0 + j, j);
                    add_outer(dS, i0 + j);
                }
                flush(dq, qks, i0, cnt, add);
            }
        }
        // backwards: w, dbeta, dk, dg; S: the state before the span, from that before position from
        int from = half;
        load_state(S, half > 0 ? spare : seed);   // spare: written by this lane
        for (int i0 = (n - 1) / kSpan * kSpan; i0 >= 0; i0 -= kSpan) {
            const int cnt = n - i0 < kSpan ? n - i0 : kSpan;
            if (i0 < from) {
                from = 0;
                load_state(S, seed);
            }
            f32x4 X[NR];   // the state before the span, then before each of its positions
            copy(X, S);
            advance(X, from, i0);
            f32x4 B[NR];
            copy(B, X);
            for (int j = cnt - 1; j >= 0; --j) {
                const int i = i0 + j;
                advance(X, i0, i);
                if constexpr (CLEAN) add_outer(dS, i);
                float k[NR], u[4], w[4], e[NR], gs[4] = {0.f, 0.f, 0.f, 0.f}, b = 0.f;
                load_k(k, s.k, i);
                load_c(u, s.u, i);
                const float alpha = s.al[i], beta = s.be[i];
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    float x = 0.f;
#pragma unroll
                    for (int m = 0; m < NR; ++m) x = fmaf(k[m], dS[m][c], x);
                    w[c] = row16_sum(x);
                    b = fmaf(w[c], u[c], b);
                }
#pragma unroll
                for (int m = 0; m < NR; ++m) {
                    float t[4];
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const float sh = alpha * X[m][c], d = fmaf(-k[m], beta * w[c], dS[m][c]);
                        t[c] = fmaf(dS[m][c], u[c], -sh * w[c]);
                        gs[c] = fmaf(d, sh, gs[c]);
                        dS[m][c] = alpha * d;
                    }
                    e[m] = beta * ((t[0] + t[1]) + (t[2] + t[3]));
                }
                // both sums over the wave's columns: gg ends in the lower, b in the upper 32 lanes
                float gg = row16_sum((gs[0] + gs[1]) + (gs[2] + gs[3]));
                gg = swap32_sum(gg, b);
                gg = swap16_sum(gg, gg);
                if (rl == 0) st4(s.w + i * DV + col, w[0], w[1], w[2], w[3]);
                if ((lane & 31) == 0) (lane ? s.pb : s.pg)[i * W + wave] = gg;
                put_rows(e, j);
                copy(X, B);
            }
            flush(dk, qks, i0, cnt, add);
        }
        // dv = beta w, by floats (the gradients may lie at any of them); dbeta and dg from the waves' sums
        for (int e = tid; e < n * DV; e += NT) {
            const int r = e / DV, c = e % DV;
            st.dv[vo + r * vs + c] = s.be[r] * s.w[r * DV + c];
        }
        if (tid < n) {
            float b = 0.f, x = 0.f;
#pragma unroll
            for (int v = 0; v < W; ++v) {
                b += s.pb[tid * W + v];
                x += s.pg[tid * W + v];
            }
            st.db[go + (long)tid * a.h_v] = b;
            st.dg[go + (long)tid * a.h_v] = x;
        }
        __syncthreads();   // LDS is free for the next v-head or view
    }
    // dq of position i from the state in S, into exchange slot j
    __device__ __forceinline__ void read_out(int i, int j)
    {
        float d[4], p[NR];
        load_c(d, s.d, i);
#pragma unroll
        for (int m = 0; m < NR; ++m) {
            p[m] = a.scale * (fmaf(S[m][0], d[0], S[m][1] * d[1]) + fmaf(S[m][2], d[2], S[m][3] * d[3]));
        }
        put_rows(p, j);
    }
    __device__ __forceinline__ void add_outer(f32x4 (&dS)[NR], int i)
    {
        float q[NR], d[4];
        load_k(q, s.q, i);
        load_c(d, s.d, i);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const float x = a.scale * d[c];
#pragma unroll
            for (int m = 0; m < NR; ++m) dS[m][c] = fmaf(q[m], x, dS[m][c]);
        }
    }
};

// First row and positions of global block blk.
__device__ __forceinline__ void block_span(const StepArgs &a, long blk, long &p0, int &n)
{
    long rem;
    if (a.cu) {
        p0 = blk * a.L;
        int lo = 0, hi = a.n_seq;   // the last document with cu[d] <= p0
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (a.cu[mid] <= p0)
                lo = mid;
            else
                hi = mid;
        }
        rem = a.cu[lo + 1] - p0;
    } else {
        const long s = blk / a.nblk, b = blk % a.nblk;
        p0 = s * a.T + b * a.L;
        rem = a.T - b * a.L;
    }
    n = (int)(rem < a.L ? rem : a.L);
}

}  // namespace

// Phases 2 and 4: one workgroup per (block, q/k head) runs the v-heads in turn, and the
// noisy views of each; phase 2 leaves the sum of the views' seed gradients in dh, phase 4
// reads the gradient at the block's end there.
template <typename In, typename Out, int DK, int DV, bool CLEAN>
__global__ void __launch_bounds__(4 * DV) bdgdn_bwd_steps_block_kernel(StepArgs a)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    typedef Block<In, Out, DK, DV> B;
    B b(a, smem_raw);
    const long blk = blockIdx.x / a.h_qk;
    const int hq = blockIdx.x % a.h_qk, r = a.h_v / a.h_qk;
    long p0;
    block_span(a, blk, p0, b.n);
    if (b.n <= 0) return;
    for (int vi = 0; vi < r; ++vi) {
        const int h = hq * r + vi;
        const long so = (blk * a.h_v + h) * (long)DV * DK;
        f32x4 dS[B::NR];
        if constexpr (CLEAN) {
            b.load_state(dS, a.dh + so);
            b.template run<true>(a.st[0], p0, h, hq, a.seeds + so, a.dh + so, dS, vi > 0);
        } else {
            f32x4 acc[B::NR] = {};
            for (int v = 1; v <= a.n_views; ++v) {
                b.template run<false>(a.st[v], p0, h, hq, a.seeds + so, a.dh + so, dS, vi > 0);
#pragma unroll
                for (int m = 0; m < B::NR; ++m)
#pragma unroll
                    for (int c = 0; c < 4; ++c) acc[m][c] += dS[m][c];
            }
            b.store_state(a.dh + so, acc);
        }
    }
}

namespace {

template <typename In, typename Out, int DK, int DV> hipError_t launch(const StepArgs &a, long blocks, hipStream_t s)
{
    const int lds = (int)BlockLds<In, Out, DK, DV>::bytes(a.L);
    auto ks = bdgdn_bwd_steps_states_kernel<In, DK, DV>;
    auto kr = bdgdn_bwd_steps_reverse_kernel<In, Out, DK, DV>;
    auto kn = bdgdn_bwd_steps_block_kernel<In, Out, DK, DV, false>;
    auto kc = bdgdn_bwd_steps_block_kernel<In, Out, DK, DV, true>;
    for (const void *f : {reinterpret_cast<const void *>(kn), reinterpret_cast<const void *>(kc)}) {
        const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
    }
    const dim3 walk(walk_grid<DV>(a)), units((unsigned)(blocks * a.h_qk)), nt(4 * DV);
    hipError_t e;
    hipLaunchKernelGGL(ks, walk, dim3(64), 0, s, a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(kn, units, nt, lds, s, a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(kr, walk, dim3(64), 0, s, a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(kc, units, nt, lds, s, a);
    return hipGetLastError();
}

size_t up256(size_t x) { return (x + 255) & ~(size_t)255; }

}  // namespace

size_t bwd_steps_workspace(long total_blocks, int h_v, int dk, int dv)
{
    const size_t states = (size_t)total_blocks * h_v * dk * dv * sizeof(float);
    const size_t need = 2 * up256(states);
    return need <= kStepsMaxBytes ? need : 0;
}

// The line between this schedule and the serial walk is workspace alone: at every size
// measured this one is faster (7 x at 3 x 63 positions in blocks of 16, 27 x at 1 x 256 in
// blocks of 16, 38 x at 2 x 369 in blocks of 4), so it runs whenever the caller gives it its
// two states per (block, v-head), but where these are more than kStepsMaxBytes, the most that a
// call asks for here (d = 128, 16 v-heads, blocks of 16: past 16384 positions): there the
// walk runs whatever the workspace.
hipError_t launch_bwd_steps(bool f32_in, bool f32_out, const GenBwdCall &c, hipStream_t s)
{
    StepArgs a = {};
    a.st[0] = StepStream{c.q, c.k, c.v, c.g, c.beta, c.dout, c.dq, c.dk, c.dv, c.dg, c.db};
    a.st[1] = StepStream{c.qn, c.kn, c.vn, c.gn, c.betan, c.doutn, c.dqn, c.dkn, c.dvn, c.dgn, c.dbn};
    a.n_views = 1 + c.n_more;
    if (!bwd_generic_supported(f32_in, c.d_k, c.d_v, c.L, a.n_views)) return hipErrorInvalidValue;
    for (int i = 0; i < c.n_more; ++i) {
        const BwdView &w = c.more[i];
        a.st[2 + i] = StepStream{w.q, w.k, w.v, w.g, w.beta, w.dout, w.dq, w.dk, w.dv, w.dg, w.db};
    }
    a.cu = c.cu;
    a.n_seq = c.n_seq;
    a.h0 = c.h0; a.dht = c.dht; a.dh0 = c.dh0;
    const size_t states = (size_t)c.total_blocks * c.h_v * c.d_k * c.d_v * sizeof(float);
    a.seeds = static_cast<float *>(c.workspace);
    a.dh = reinterpret_cast<float *>(static_cast<unsigned char *>(c.workspace) + up256(states));
    a.T = c.T; a.L = c.L; a.nblk = (c.T + c.L - 1) / c.L;
    a.h_qk = c.h_qk; a.h_v = c.h_v;
    a.scale = c.scale;
#define BDGDN_DIMS(IN, OUT)                                                                     \
    {                                                                                           \
        if (c.d_k == 64)                                                                        \
            return c.d_v == 64 ? launch<IN, OUT, 64, 64>(a, c.total_blocks, s)                  \
                               : launch<IN, OUT, 64, 128>(a, c.total_blocks, s);                \
        return c.d_v == 64 ? launch<IN, OUT, 128, 64>(a, c.total_blocks, s)                     \
                           : launch<IN, OUT, 128, 128>(a, c.total_blocks, s);                   \
    }
    if (f32_in) BDGDN_DIMS(float, float)
    if (f32_out) BDGDN_DIMS(__bf16, float)
    BDGDN_DIMS(__bf16, __bf16)
#undef BDGDN_DIMS
}

}  // namespace bdgdn
