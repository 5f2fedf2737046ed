// bwd_kernels.hip -- backward of the two-stream training forward (Appendix "Backward
// primitives": the block-level chain rule eq. dh-block-recursion, the noisy block-end
// readout backward eq. noisy-readout-bwd, and the clean chunk backward), for gfx950.
//
// The per-step backward of the paper (eq. per-step-bwd) needs every per-step state; here
// each block is differentiated in its block (WY) form instead, which needs only the
// block's seed state S0.  For one block of n positions from S0, with local cumulative
// log-gates G (gamma = exp G, gamma_n the last), D_i = gamma_n / gamma_i and
//   A_ri = beta_r (gamma_r/gamma_i) k_r.k_i (i < r),  M = (I + A)^-1,  T = M diag(beta),
//   X = K S0,  R = V - Gamma X,  Delta = T R,  S_n = gamma_n S0 + K^T D Delta,
//   clean:  O = s (Gamma Q S0 + P Delta),  P = Q K^T o Mc,  Mc_ri = gamma_r/gamma_i (i <= r)
//   noisy:  O~ = s Q S_n  (every position reads the block-end state),
// and the gradient dS_n of the block-end state (clean: the gradient arriving from the later
// blocks; noisy: s Q^T dO~), the backward is
//   E = dO Delta^T,  dDelta = [clean] s P^T dO + D K dS_n,  dR = T^T dDelta = dV,
//   dQ = [clean] s Gamma dO S0^T + (s E o Mc) K   |  [noisy] s gamma_n dO S0^T + s (E D) K,
//   dK = [clean] (s E o Mc)^T Q + D Delta dS_n^T - Gamma dR S0^T + (dKK + dKK^T) K,
//   dT = dDelta R^T,  dbeta_i = sum_r dT_ri M_ri + sum_i' dA_ii' F_ii',
//   dA = strictly lower part of -M^T (dT diag beta) M^T,  dKK_ri = dA_ri beta_r gamma_r/gamma_i,
//   dS0 = gamma_n dS_n + [clean] s Q^T Gamma dO - K^T Gamma dR,
// with the gate gradients collected on the local cumulative gates (dG) and dg = the
// reverse cumulative sum of dG inside the block.  The chain rule across blocks:
// dh_(b-1) = dS0(clean block b) + dS0(noisy block b), since the noisy block b is seeded with
// the clean state at the end of block b - 1.
//
// Three phases after the clean scan has written every block's seed (launch_scan_states, fp16):
//  1. every noisy block in parallel (bwd_block.hpp; bwd_pair.hpp for blocks of 34 .. 64 in two
//     halves, bwd_small.hpp for several small blocks in a clean chunk): its gradients and its
//     seed's gradient, plus the part of the clean block at the same position that does not
//     depend on the state gradient dh.  With dDelta = s P^T dO + D K dh and dR = T^T dDelta,
//       dS0 = gamma_n dh + s Q^T Gamma dO - K^T Gamma T^T (s P^T dO) - K^T (U K) dh,  U = Gamma T^T D,
//     so that part is s Q^T Gamma dO - K^T Gamma T^T (s P^T dO), and U K (32 x 128, U_ij = T_ji
//     gamma_i gamma_n / gamma_j, upper triangular with |U_ij| <= |T_ji|) and gamma_n go to the
//     scan; the noisy and the clean part sum to c_b, the dh-independent part of dh_(b-1);
//  2. the reverse scan of the clean state gradient over the blocks of each (sequence,
//     v-head), 16 columns a wave (bwd_scan.hip): dh_(b-1) = gamma_n dh_b + c_b - K^T (U K) dh_b;
//  3. every clean block in parallel from its seed and the gradient at its end (bwd_block.hpp).
// In time segments (BwdArgs::seg; the strided clean checkpoints of the checkpoint build) the
// same three phases run over one segment of every chain at a time, last segment first: the
// seeds come from the segment's checkpoint, the scan starts from the gradient the later
// segment left in the carry and leaves its own there, and the units are numbered inside the
// segment by the segment tables (bdgdn_bwd_seg_plan_kernel).
// Products are MFMA tiles on fp16 operands with fp32 accumulation: k-contiguous operands by
// 16-byte LDS reads, the others by the LDS transpose load, and results that are the next
// product's operand kept in registers; M = (I + A)^-1 by the register-resident doubling solve
// (ut::solve_t), the dA products in fp32 MFMA.  Blocks are padded to 32 positions with
// identity steps (k = 0, beta = 0, g = 0), which change nothing.
#include "common.hpp"
#include "bwd.hpp"
#include "kernels.hpp"
#include "ut.hpp"

namespace bdgdn {

namespace {

constexpr int NP = 32;           // positions per (padded) block
constexpr int DD = 128;          // d_k = d_v
constexpr int LDH = DD + 8;      // f16 row stride of [*][128] LDS matrices
constexpr int LDF = NP + 1;      // fp32 row stride of [32][32] LDS matrices
constexpr int LDM = NP + 8;      // f16 row stride of [32][32] LDS matrices
constexpr int kWaves = 8;

typedef __fp16 fp16x4_t __attribute__((__vector_size__(4 * sizeof(__fp16))));

// Operands of v_mfma_f32_16x16x16f16, lane (g, n) = (lane / 16, lane % 16): A row n with
// k = 4 g .. 4 g + 3, B column n with the same k, C column n with rows 4 g .. 4 g + 3.  A C
// tile kept in registers is therefore the B operand of a product contracting over its rows.
//
// A from a row-major matrix with k contiguous (one 8-byte read).
__device__ __forceinline__ f16x4 op_row(const _Float16 *X, int ld, int m0, int k0, int lane)
{
    return *reinterpret_cast<const f16x4 *>(X + (m0 + (lane & 15)) * ld + k0 + 4 * (lane >> 4));
}
// X[k0 + 4 g + e][c0 + n] of a row-major matrix: the B operand X (k = row) or the A operand
// X^T, by the LDS transpose load ds_read_b64_tr_b16 (lane L reads the 8 bytes at row
// k0 + L / 4, columns c0 + 4 (L % 4); each 16-lane group receives the columns of the 4 x 16
// block its lanes read).
__device__ __forceinline__ f16x4 op_tr(const _Float16 *X, int ld, int k0, int c0, int lane)
{
    const _Float16 *p = X + (k0 + (lane >> 2)) * ld + c0 + 4 * (lane & 3);
    return __builtin_bit_cast(f16x4, __builtin_amdgcn_ds_read_tr16_b64_v4f16(
                                         (__attribute__((address_space(3))) fp16x4_t *)(p)));
}
__device__ __forceinline__ f16x4 h4(f32x4 v)
{
    return f16x4{(_Float16)v[0], (_Float16)v[1], (_Float16)v[2], (_Float16)v[3]};
}
__device__ __forceinline__ f16x4 scale4(f16x4 v, f32x4 f)
{
    return f16x4{(_Float16)((float)v[0] * f[0]), (_Float16)((float)v[1] * f[1]), (_Float16)((float)v[2] * f[2]),
                 (_Float16)((float)v[3] * f[3])};
}
__device__ __forceinline__ f32x4 ld4(const float *p) { return *reinterpret_cast<const f32x4 *>(p); }

__device__ __forceinline__ float ex(float x) { return __expf(x); }

// v added to *dst (LDS) atomically.
__device__ __forceinline__ void lds_add(float *dst, float v) { atomicAdd(dst, v); }

// Sum over the 16 lanes of each lane row (the columns of a C tile row), by DPP row shifts:
// valid in lane 15 of the row.
__device__ __forceinline__ float row_total(float v)
{
    v += ut::dpp<0x111>(v);
    v += ut::dpp<0x112>(v);
    v += ut::dpp<0x114>(v);
    v += ut::dpp<0x118>(v);
    return v;
}
// Sums over lanes 0 .. 31 and 32 .. 63, each returned to the lanes of its half.
__device__ __forceinline__ float half_total(float v, int lane)
{
    const float t = row_total(v);
    const float h0 = ut::lane_value(t, 15) + ut::lane_value(t, 31);
    const float h1 = ut::lane_value(t, 47) + ut::lane_value(t, 63);
    return lane < 32 ? h0 : h1;
}
__device__ __forceinline__ float wave_total(float v)
{
    const float t = row_total(v);
    return (ut::lane_value(t, 15) + ut::lane_value(t, 31)) + (ut::lane_value(t, 47) + ut::lane_value(t, 63));
}

// One thread's share of a 32 x 128 row block (row tid / 16, the 8 values from 8 (tid % 16)),
// loaded into registers ahead of its store to LDS as fp16, so that all loads of a unit are
// in flight together.
template <typename In> struct Row8;
template <> struct Row8<__bf16> {
    bf16x8 v;
    __device__ __forceinline__ void load(const __bf16 *p) { v = *reinterpret_cast<const bf16x8 *>(p); }
    __device__ __forceinline__ void zero()
    {
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = (__bf16)0.f;
    }
    __device__ __forceinline__ f16x8 h(float sg = 1.f) const
    {
        f16x8 r;
#pragma unroll
        for (int j = 0; j < 8; ++j) r[j] = (_Float16)((float)v[j] * sg);
        return r;
    }
};
template <> struct Row8<float> {
    f32x4 lo, hi;
    __device__ __forceinline__ void load(const float *p)
    {
        lo = ld4(p);
        hi = ld4(p + 4);
    }
    __device__ __forceinline__ void zero() { lo = hi = f32x4{0.f, 0.f, 0.f, 0.f}; }
    __device__ __forceinline__ f16x8 h(float sg = 1.f) const
    {
        f16x8 r;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            r[j] = (_Float16)(lo[j] * sg);
            r[4 + j] = (_Float16)(hi[j] * sg);
        }
        return r;
    }
};
template <typename In> __device__ __forceinline__ Row8<In> load_rows(const In *src, long stride, int nvalid, int tid)
{
    const int r = tid >> 4, c = (tid & 15) * 8;
    Row8<In> x;
    if (r < nvalid)
        x.load(src + (long)r * stride + c);
    else
        x.zero();
    return x;
}
template <typename In> __device__ __forceinline__ void store_rows(_Float16 *dst, const Row8<In> &x, int tid,
                                                                  float sg = 1.f)
{
    const int r = tid >> 4, c = (tid & 15) * 8;
    *reinterpret_cast<f16x8 *>(dst + r * LDH + c) = x.h(sg);
}

// The fp16 seed state (128 x 128, 32 KB): four 16-byte pieces per thread.
struct SeedRegs {
    f16x8 v[4];
};
__device__ __forceinline__ SeedRegs load_seed(const _Float16 *src, int tid)
{
    SeedRegs x;
#pragma unroll
    for (int it = 0; it < 4; ++it) x.v[it] = *reinterpret_cast<const f16x8 *>(src + (tid + 512 * it) * 8);
    return x;
}
__device__ __forceinline__ void store_seed(_Float16 *dst, const SeedRegs &x, int tid)
{
#pragma unroll
    for (int it = 0; it < 4; ++it) {
        const int e = (tid + 512 * it) * 8;
        *reinterpret_cast<f16x8 *>(dst + (e / DD) * LDH + e % DD) = x.v[it];
    }
}
struct StreamPtrs {
    const __bf16 *q, *k, *v;   // first row of the block (q/k head hq, v head h)
    const float *g, *beta;     // first row (head h), stride h_v
    const void *dout;          // first row (head h)
    float *dq, *dk, *dv, *dg, *db;   // first row of the gradients
};

// A block's inputs in registers (V only with WITH_V); g, b: the gate and step size of
// position tid (tid < 32).
template <typename Od, bool WITH_V> struct BlockRows {
    Row8<__bf16> q, k, v;
    Row8<Od> dout;
    float g, b;
};
template <typename Od, bool WITH_V>
__device__ __forceinline__ BlockRows<Od, WITH_V> load_block(const StreamPtrs &p, int h_qk, int h_v, int nvalid, int tid)
{
    const long qks = (long)h_qk * DD, vs = (long)h_v * DD;
    BlockRows<Od, WITH_V> x;
    x.q = load_rows(p.q, qks, nvalid, tid);
    x.k = load_rows(p.k, qks, nvalid, tid);
    if constexpr (WITH_V) x.v = load_rows(p.v, vs, nvalid, tid);
    x.dout = load_rows(static_cast<const Od *>(p.dout), vs, nvalid, tid);
    const bool ok = tid < NP && tid < nvalid;
    x.g = ok ? p.g[(long)tid * h_v] : 0.f;
    x.b = ok ? p.beta[(long)tid * h_v] : 0.f;
    return x;
}

}  // namespace

// Rows 16 tm .. of U K, columns 16 w .. 16 w + 15, into the order the scan reads as operands: 16 x 32
// tiles (tm, w / 2), lane (g, n) holding row n, columns 4 g .. 4 g + 3 of both 16-column halves.
// x: lane (g, n)'s four entries (a C tile of (U K)^T).
__device__ __forceinline__ void put_uk(_Float16 *uk, int tm, int w, int lane, f16x4 x)
{
    *reinterpret_cast<f16x4 *>(uk + ((4 * tm + (w >> 1)) * 64 + lane) * 8 + 4 * (w & 1)) = x;
}

// q/k gradient x into *dst: stored for the first v-head of a q/k head, added for the others
// (a workgroup runs the v-heads of a q/k head one after the other, and the same thread
// writes the same element for each, so the sum has a fixed order; see unit_of).
__device__ __forceinline__ void put_qk(bool add, float *dst, float x)
{
    if (add)
        *dst += x;
    else
        *dst = x;
}

namespace {

// Unit t of the (block, v-head) units ordered so that the r = h_v / h_qk v-heads of a q/k
// head (consecutive v-heads) are consecutive: t = ((gblk h_qk) + hq) r + i, v-head h = hq r + i.
// Each workgroup runs the units of a (block, q/k head) one after the other, so that its dq, dk
// rows are stored by the first (i = 0) and added to by the others: a fixed summation order,
// no atomics, nothing to clear.  Returns the unit's index in the per-(block, v-head) arrays.
__device__ __forceinline__ long unit_of(const BwdArgs &a, long t, long &gblk, int &h, int &hq, int &i)
{
    // a launch has fewer than 2^32 units: 32-bit division
    const unsigned r = a.h_v / a.h_qk, ti = (unsigned)t, gi = ti / r;
    i = (int)(ti % r);
    gblk = gi / (unsigned)a.h_qk;
    hq = (int)(gi % (unsigned)a.h_qk);
    h = hq * r + i;
    return gblk * a.h_v + h;
}

// The (sequence, first row, rows) of global block gblk: packed documents start on block
// boundaries, so a block lies inside one document.
__device__ __forceinline__ void block_unit(const BwdArgs &a, long gblk, int &n, long &p0, int &nvalid)
{
    if (a.seg) {
        // a segment's unit: the last sequence n with seg[n] <= gblk (one with no blocks in
        // the segment has seg[n] == seg[n + 1] and is passed over), block blk0 + gblk - seg[n]
        int lo = 0, hi = a.n_chains / a.h_v;
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (a.seg[mid] <= gblk)
                lo = mid;
            else
                hi = mid;
        }
        n = lo;
        const long r0 = a.cu ? a.cu[n] : (long)n * a.T, r1 = a.cu ? a.cu[n + 1] : r0 + a.T;
        p0 = r0 + (a.blk0 + gblk - a.seg[n]) * a.L;
        const long rem = r1 - p0;
        nvalid = rem < 0 ? 0 : (rem < a.L ? (int)rem : a.L);
    } else if (a.cu) {
        p0 = gblk * a.L;
        int lo = 0, hi = a.n_docs;   // the last document with cu[d] <= p0
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (a.cu[mid] <= p0)
                lo = mid;
            else
                hi = mid;
        }
        n = lo;
        const long rem = a.cu[lo + 1] - p0;
        nvalid = (int)(rem < a.L ? rem : a.L);
    } else {
        // a launch has fewer than 2^32 units: 32-bit division
        n = (int)((unsigned)gblk / (unsigned)a.nblk);
        const int b = (int)((unsigned)gblk % (unsigned)a.nblk);
        p0 = (long)n * a.T + (long)b * a.L;
        const int rem = a.T - b * a.L;
        nvalid = rem < a.L ? rem : a.L;
    }
}

template <typename Od>
__device__ __forceinline__ StreamPtrs stream_ptrs(const BwdArgs &a, bool noisy, long p0, int h, int hq)
{
    const long qks = (long)a.h_qk * DD, vs = (long)a.h_v * DD;
    StreamPtrs p;
    p.q = static_cast<const __bf16 *>(noisy ? a.qn : a.q) + p0 * qks + hq * DD;
    p.k = static_cast<const __bf16 *>(noisy ? a.kn : a.k) + p0 * qks + hq * DD;
    p.v = static_cast<const __bf16 *>(noisy ? a.vn : a.v) + p0 * vs + h * DD;
    p.g = (noisy ? a.gn : a.g) + p0 * a.h_v + h;
    p.beta = (noisy ? a.betan : a.beta) + p0 * a.h_v + h;
    p.dout = static_cast<const Od *>(noisy ? a.doutn : a.dout) + p0 * vs + h * DD;
    p.dq = (noisy ? a.dqn : a.dq) + p0 * qks + hq * DD;
    p.dk = (noisy ? a.dkn : a.dk) + p0 * qks + hq * DD;
    p.dv = (noisy ? a.dvn : a.dv) + p0 * vs + h * DD;
    p.dg = (noisy ? a.dgn : a.dg) + p0 * a.h_v + h;
    p.db = (noisy ? a.dbn : a.db) + p0 * a.h_v + h;
    return p;
}

}  // namespace

#include "bwd_block.hpp"
#include "bwd_pair.hpp"
#include "bwd_small.hpp"

// The range of the upstream gradients (dO, dO~ of every view, dht): each block's max |x| over
// its grid-stride share of every array into part[blockIdx.x].  With Od = bf16 the output
// gradients are bf16 (dht is always fp32).
__device__ __forceinline__ float absmax4(f32x4 v)
{
    return fmaxf(fmaxf(fabsf(v[0]), fabsf(v[1])), fmaxf(fabsf(v[2]), fabsf(v[3])));
}
__device__ __forceinline__ float absmax8(bf16x8 v)
{
    float m = 0.f;
#pragma unroll
    for (int j = 0; j < 8; ++j) m = fmaxf(m, fabsf((float)v[j]));
    return m;
}
// max |x| over this block's contiguous segment of x[0 .. n), eight 16-byte loads in flight
// per thread
template <typename V, typename F>
__device__ __forceinline__ float range_max(const V *x, long n, float m, const F &absmax)
{
    const long seg = (n + gridDim.x - 1) / gridDim.x;
    const long end = min(n, seg * (blockIdx.x + 1));
    long e = seg * blockIdx.x + threadIdx.x;
    for (; e + 7 * 256 < end; e += 8 * 256) {
        V v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = x[e + u * 256];
#pragma unroll
        for (int u = 0; u < 8; ++u) m = fmaxf(m, absmax(v[u]));
    }
    for (; e < end; e += 256) m = fmaxf(m, absmax(x[e]));
    return m;
}
template <typename Od>
__global__ void __launch_bounds__(256) bdgdn_bwd_range_kernel(RangeArgs r)
{
    __shared__ float red[4];
    float m = 0.f;
    for (int i = 0; i < r.count; ++i) {
        const long n8 = r.n[i] / 8;   // 8-element vectors (every length is a multiple of 128)
        if (sizeof(Od) == 2 && !(i == r.count - 1 && r.last_f32))
            m = range_max(static_cast<const bf16x8 *>(r.arr[i]), n8, m, absmax8);
        else
            m = range_max(static_cast<const f32x4 *>(r.arr[i]), 2 * n8, m, absmax4);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) r.part[blockIdx.x] = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
}

// The blocks' maxima reduced to the power-of-two scale sigma that puts the largest upstream
// gradient in [4, 8), and its inverse: range[0] = sigma, range[1] = 1 / sigma (both 1 when
// every gradient is zero or one is not finite).  Every gradient is linear in the upstream
// gradients, so the block kernels work on sigma times them (fp16 operands keep their relative
// precision whatever the loss scale) and divide their fp32 results by sigma, exactly.
__global__ void __launch_bounds__(256) bdgdn_bwd_scale_kernel(const float *part, int n, float *range)
{
    __shared__ float red[4];
    float m = 0.f;
    bool bad = false;
    for (int i = threadIdx.x; i < n; i += 256) {
        const float v = part[i];
        bad |= !isfinite(v);
        m = fmaxf(m, v);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
    const bool any_bad = __syncthreads_or(bad);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        m = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
        float sg = 1.f;
        if (!any_bad && m > 0.f) {
            int e;
            frexpf(m, &e);                       // m in [2^(e-1), 2^e)
            const int k = min(max(3 - e, -120), 120);
            sg = ldexpf(1.f, k);                 // sigma m in [4, 8)
        }
        range[0] = sg;
        range[1] = 1.f / sg;
    }
}

hipError_t launch_bwd_range(bool bf16_out, const RangeArgs &r, hipStream_t s)
{
    if (r.count < 1 || r.count > kRangeArrays) return hipErrorInvalidValue;
    if (bf16_out)
        hipLaunchKernelGGL(bdgdn_bwd_range_kernel<__bf16>, dim3(kRangeBlocks), dim3(256), 0, s, r);
    else
        hipLaunchKernelGGL(bdgdn_bwd_range_kernel<float>, dim3(kRangeBlocks), dim3(256), 0, s, r);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(bdgdn_bwd_scale_kernel, dim3(1), dim3(256), 0, s, r.part, kRangeBlocks, r.range);
    return hipGetLastError();
}


// The segment tables: wave k scans the sequences, 64 at a time, summing the blocks of each inside
// segment k (and its noisy blocks of two sub-blocks, the last one possibly half).
__global__ void __launch_bounds__(64) bdgdn_bwd_seg_plan_kernel(const int32_t *cu, int n_seq, int T, int L,
                                                                int seg_len, int *seg, int *segp)
{
    const int k = blockIdx.x, lane = threadIdx.x;
    int *o = seg + (long)k * (n_seq + 1), *op = segp + (long)k * (n_seq + 1);
    int acc = 0, accp = 0;   // of the sequences before n0
    for (int n0 = 0; n0 <= n_seq; n0 += 64) {
        const int n = n0 + lane;
        int cnt = 0;
        if (n < n_seq) {
            const long len = cu ? (long)cu[n + 1] - cu[n] : T;
            const long nb = (len + L - 1) / L, rest = nb - (long)k * seg_len;
            cnt = rest <= 0 ? 0 : (rest < seg_len ? (int)rest : seg_len);
        }
        const int cntp = (cnt + 1) / 2;
        int x = cnt, xp = cntp;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int y = __shfl_up(x, d), yp = __shfl_up(xp, d);
            if (lane >= d) {
                x += y;
                xp += yp;
            }
        }
        if (n <= n_seq) {
            o[n] = acc + x - cnt;
            op[n] = accp + xp - cntp;
        }
        acc += __shfl(x, 63);
        accp += __shfl(xp, 63);
    }
}

hipError_t launch_bwd_seg_plan(const int32_t *cu, int n_seq, int T, int L, int seg_len, int n_seg, int *seg,
                               int *segp, hipStream_t s)
{
    if (n_seg <= 0 || n_seq <= 0 || L <= 0 || seg_len <= 0) return hipErrorInvalidValue;
    hipLaunchKernelGGL(bdgdn_bwd_seg_plan_kernel, dim3(n_seg), dim3(64), 0, s, cu, n_seq, T, L, seg_len, seg, segp);
    return hipGetLastError();
}

hipError_t launch_bwd(bool bf16_out, const BwdArgs &a, const BwdView *more, int n_more, int n_chains,
                      long n_block_units, long n_pair_units, hipStream_t s)
{
    if (n_more < 0 || (n_more > 0 && !more)) return hipErrorInvalidValue;
    if (a.nl > 0 && (n_more > 0 || n_pair_units > 0 || a.L != NP || NP % a.nl != 0 || !a.xd)) return hipErrorInvalidValue;
    // one workgroup per (block, q/k head), running its r v-heads in turn (unit_of)
    const int r = a.h_v / a.h_qk;
    const long groups = n_block_units / r, pair_groups = n_pair_units / r;
    BwdArgs a2 = a;
    a2.n_units = n_block_units;
    // the noisy stream of a: its pointers replaced by those of view i
    auto with_view = [&](const BwdView &w) {
        BwdArgs b = a2;
        b.qn = w.q; b.kn = w.k; b.vn = w.v; b.gn = w.g; b.betan = w.beta; b.doutn = w.dout;
        b.dqn = w.dq; b.dkn = w.dk; b.dvn = w.dv; b.dgn = w.dg; b.dbn = w.db;
        return b;
    };
    // the persistent small-block kernel: one workgroup per CU (its LDS allows no more)
    int dev = 0, n_cu = 0;
    hipError_t err = hipGetDevice(&dev);
    if (err == hipSuccess) err = hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev);
    if (err != hipSuccess) return err;
    const unsigned pgrid = (unsigned)(groups < n_cu ? groups : (n_cu > 0 ? n_cu : 1));
    auto run = [&](auto noisy, auto noisy_more, auto pair, auto pair_more, auto small, auto clean, auto clean_small) {
        for (const void *f : {reinterpret_cast<const void *>(noisy), reinterpret_cast<const void *>(noisy_more),
                              reinterpret_cast<const void *>(pair), reinterpret_cast<const void *>(pair_more),
                              reinterpret_cast<const void *>(small), reinterpret_cast<const void *>(clean),
                              reinterpret_cast<const void *>(clean_small)}) {
            const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
            if (e != hipSuccess) return e;
        }
        hipError_t e;
        if (a.nl > 0) {   // small noisy blocks in clean chunks
            if (groups > 0) {
                hipLaunchKernelGGL(small, dim3(pgrid), dim3(512), sizeof(SmallSmem), s, a2);
                if ((e = hipGetLastError()) != hipSuccess) return e;
            }
        } else if (pair_groups > 0) {   // noisy blocks of two sub-blocks
            hipLaunchKernelGGL(pair, dim3((unsigned)pair_groups), dim3(1024), sizeof(PairSmem), s, a2);
            if ((e = hipGetLastError()) != hipSuccess) return e;
            for (int i = 0; i < n_more; ++i) {   // in stream order: each adds its seed gradients
                hipLaunchKernelGGL(pair_more, dim3((unsigned)pair_groups), dim3(1024), sizeof(PairSmem), s,
                                   with_view(more[i]));
                if ((e = hipGetLastError()) != hipSuccess) return e;
            }
        } else if (groups > 0) {
            hipLaunchKernelGGL(noisy, dim3((unsigned)groups), dim3(512), sizeof(NoisySmem), s, a2);
            if ((e = hipGetLastError()) != hipSuccess) return e;
            for (int i = 0; i < n_more; ++i) {   // in stream order: each adds its seed gradients
                hipLaunchKernelGGL(noisy_more, dim3((unsigned)groups), dim3(512), sizeof(NoisySmem), s,
                                   with_view(more[i]));
                if ((e = hipGetLastError()) != hipSuccess) return e;
            }
        }
        if ((e = launch_bwd_scan(a, s)) != hipSuccess) return e;
        if (groups > 0) {
            hipLaunchKernelGGL(a.nl > 0 ? clean_small : clean, dim3((unsigned)groups), dim3(512),
                               sizeof(CleanSmem), s, a2);
            if ((e = hipGetLastError()) != hipSuccess) return e;
        }
        return hipSuccess;
    };
    return bf16_out ? run(bdgdn_bwd_noisy_kernel<__bf16, true>, bdgdn_bwd_noisy_kernel<__bf16, false>,
                          bdgdn_bwd_pair_kernel<__bf16, true>, bdgdn_bwd_pair_kernel<__bf16, false>,
                          bdgdn_bwd_small_kernel<__bf16>, bdgdn_bwd_clean_kernel<__bf16, false>,
                          bdgdn_bwd_clean_kernel<__bf16, true>)
                    : run(bdgdn_bwd_noisy_kernel<float, true>, bdgdn_bwd_noisy_kernel<float, false>,
                          bdgdn_bwd_pair_kernel<float, true>, bdgdn_bwd_pair_kernel<float, false>,
                          bdgdn_bwd_small_kernel<float>, bdgdn_bwd_clean_kernel<float, false>,
                          bdgdn_bwd_clean_kernel<float, true>);
}

}  // namespace bdgdn
