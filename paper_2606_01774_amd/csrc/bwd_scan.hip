// bwd_scan.hip -- phase 2 of the block-form backward (bwd_kernels.hip), for gfx950.
//
// The reverse scan of the clean state gradient over the blocks of a (sequence,
// v-head) (a chain), one wave per 16 columns (the columns are independent):
//   dh_(b-1) = gamma_n dh_b + cterm_b - K^T Z,  Z = (U K) dh_b  (32 x 16),
// writing dh_b (the gradient at the end of block b; fp16, the precision phase 3 uses it in,
// tile-native) over cterm_b, which only this scan reads, for phase 3, and dh0 (fp32).
//
// A wave holds its 128 x 16 of dh as eight C tiles, which are the B operands of (U K) dh, and Z's
// tiles those of K^T Z: nothing passes between waves and no step has a barrier.  U K comes in
// operand order from phase 1; K's rows go through the wave's own LDS to be read transposed, as
// the bf16 they are, against Z in two bf16 parts (16 bits, more than the fp16 Z of the other
// products).  Bound by the step's chain of instructions on the one wave of a SIMD where chains
// are few, by the traffic of U K, K, cterm and dh (80 KB per block) where they are many.  The
// operands of the next two blocks are in flight, which takes a loop without a branch between
// the sets: behind one the waits also drained the set just asked for (1.0 us a step).
// Measured per call, against four waves per 32 columns with dh and Z passed through LDS and two
// barriers a step: 128 steps of 16 chains 144 -> 90 us, of 64 chains 180 -> 166 us, 512 steps of 64
// chains 661 -> 625 us (4.3 TB/s).
#include "bwd.hpp"
#include "common.hpp"

namespace bdgdn {

namespace {

constexpr int NP = 32, DD = 128;   // positions per (padded) block, d_k = d_v
constexpr int kScanSets = 3;   // register sets of one block's operands (81 VGPRs each)

__device__ __forceinline__ f16x4 h4(f32x4 v)
{
    return f16x4{(_Float16)v[0], (_Float16)v[1], (_Float16)v[2], (_Float16)v[3]};
}
__device__ __forceinline__ bf16x8 tr_bf16(const __bf16 *K, int tm, int lane)
{
    // rows 4 g + e and 16 + 4 g + e of column 16 tm + n (the A operand K^T), by transpose loads from
    // the swizzled rows: the 32-byte piece m of row r lies at piece m ^ (r & 7)
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    const int r = lane >> 2;
    s16x4 x[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int row = 16 * h + r;
        const __bf16 *p = K + row * DD + 16 * (tm ^ (row & 7)) + 4 * (lane & 3);
        x[h] = __builtin_bit_cast(s16x4, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                                             (__attribute__((address_space(3))) s16x4 *)(p)));
    }
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(x[0], x[1], 0, 1, 2, 3, 4, 5, 6, 7));
}
}  // namespace

__global__ void __launch_bounds__(64, 1) bdgdn_bwd_scan_kernel(BwdArgs a)
{
    constexpr int NT = DD / 16;   // waves per chain
    __shared__ __align__(16) __bf16 sK[NP * DD];
    const int lane = threadIdx.x, g4 = lane >> 4, rr = lane & 15;
    // the waves of a chain on one XCD (workgroups are dealt to the 8 XCDs in turn), so that
    // they read its U K and K rows through one L2
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int chain = (slot / NT) * 8 + xcd, strip = slot % NT;
    if (chain >= a.n_chains) return;
    const int n = chain / a.h_v, h = chain % a.h_v, hq = h / (a.h_v / a.h_qk);
    long r0, r1;
    if (a.cu) {
        r0 = a.cu[n];
        r1 = a.cu[n + 1];
    } else {
        r0 = (long)n * a.T;
        r1 = r0 + a.T;
    }
    const int nb = (int)((r1 - r0 + a.L - 1) / a.L);
    // the blocks walked, blo .. bhi - 1, and the workspace unit of block b, gb0 + b: all the
    // chain's blocks by global index (documents start on block boundaries), or those of one
    // time segment numbered from seg[n]; the walk starts from dht where the chain ends in it,
    // else from the gradient the next segment left in carry, and ends in dh0 at the chain's
    // start, else in carry
    int blo = 0, bhi = nb;
    long gb0 = a.cu ? r0 / a.L : (long)n * a.nblk;
    bool from_dht = true, to_dh0 = true;
    if (a.seg) {
        blo = a.blk0;
        bhi = nb < a.blk0 + a.seg_len ? nb : a.blk0 + a.seg_len;
        // no blocks of this chain in the segment: nothing to do, but for an empty chain,
        // whose dh0 is dht, in the first segment
        if (bhi <= blo && !(nb == 0 && a.blk0 == 0)) return;
        gb0 = a.seg[n] - blo;
        from_dht = nb <= a.blk0 + a.seg_len;
        to_dh0 = a.blk0 == 0;
    }
    const size_t SS = (size_t)DD * DD;
    const long qks = (long)a.h_qk * DD;
    f32x4 dh[NT];   // rows 16 tm + 4 g + j of column 16 strip + rr
    const size_t so = ((size_t)n * a.h_v + h) * SS + 4 * g4 * DD + 16 * strip + rr;   // this lane's first element
    float *carry = a.seg ? a.carry + so : nullptr;
    // the carry holds dh as the walk keeps it (times sigma)
    const float *src = !from_dht ? carry : (a.dht ? a.dht + so : nullptr);
    const float sg = from_dht ? a.range[0] : 1.f;
#pragma unroll
    for (int tm = 0; tm < NT; ++tm) dh[tm] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (src) {
#pragma unroll
        for (int tm = 0; tm < NT; ++tm)
#pragma unroll
            for (int j = 0; j < 4; ++j) dh[tm][j] = src[(16 * tm + j) * DD] * sg;
    }
    // wait for these loads here, once: left pending into the loop, they would make every
    // step wait for all outstanding loads (the prefetch of the next blocks included)
#pragma unroll
    for (int tm = 0; tm < NT; ++tm) asm volatile("" : "+v"(dh[tm]));
    // one block's operands: U K (operand order: 16 x 32 tiles of rows tm, columns 32 j), K's rows
    // (row 4 i + lane / 16, 16-byte chunk lane % 16), cterm's tiles (tm, strip), gamma_n
    struct Ops {
        f16x8 uk[8];
        bf16x8 k[8];
        f16x4 cs[8];
        float gn;
    };
    const unsigned kr = lane >> 4, kc = lane & 15;
    // uniform addresses per block, and 32-bit byte offsets a lane that never change
    unsigned ko[8];
    auto k_rows = [&](int nvalid) {
        // rows past the block's end: the last one again (their rows of U K, so of Z, are zero)
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int row = 4 * i + (int)kr < nvalid ? 4 * i + (int)kr : nvalid - 1;
            ko[i] = 2 * ((unsigned)row * (unsigned)qks + 8 * kc);
        }
    };
    const unsigned uo[2] = {16u * lane, 16u * lane + 4096u};
    unsigned co[4];   // tiles 2 t and 2 t + 1 of a state's column strip, 4096 bytes apart
#pragma unroll
    for (int t = 0; t < 4; ++t) co[t] = 512u * strip + 8u * lane + 8192u * t + 4096u;
    auto fetch = [&](int b, Ops &o) {
        const size_t unit = (size_t)(gb0 + b) * a.h_v + h;
        const char *u = reinterpret_cast<const char *>(a.uk + unit * NP * DD);
#pragma unroll
        for (int i = 0; i < 8; ++i) o.uk[i] = *reinterpret_cast<const f16x8 *>(u + uo[i >> 2] + 1024 * (i & 3));
        const char *k = reinterpret_cast<const char *>(static_cast<const __bf16 *>(a.k) + (r0 + (long)b * a.L) * qks +
                                                       hq * DD);
#pragma unroll
        for (int i = 0; i < 8; ++i) o.k[i] = *reinterpret_cast<const bf16x8 *>(k + ko[i]);
        const char *c = reinterpret_cast<const char *>(a.cterm + unit * SS);
#pragma unroll
        for (int tm = 0; tm < NT; ++tm)
            o.cs[tm] = *reinterpret_cast<const f16x4 *>(c + co[tm >> 1] + (tm & 1 ? 0 : -4096));
        // a vector load (the index made lane-opaque): a scalar load would be counted with the
        // LDS operations, whose waits would wait for it
        unsigned z;
        asm volatile("v_mov_b32 %0, 0" : "=v"(z));
        o.gn = *reinterpret_cast<const float *>(reinterpret_cast<const char *>(a.gnb + unit) + z);
    };
    auto step = [&](int b, const Ops &cur, Ops &nxt) {
        // K's rows to LDS, the 32-byte pieces of a row swizzled for the transpose loads
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int row = 4 * i + (int)kr;
            *reinterpret_cast<bf16x8 *>(sK + row * DD + 16 * ((int)(kc >> 1) ^ (row & 7)) + 8 * (kc & 1)) = cur.k[i];
        }
        bf16x8 kt[NT];   // read back transposed while (U K) dh is on its way
#pragma unroll
        for (int tm = 0; tm < NT; ++tm) kt[tm] = tr_bf16(sK, tm, lane);
        // dh_b in fp16: block b's cterm slot (tile-native), which this lane has read, and operands
        char *dhb = reinterpret_cast<char *>(a.dh + ((size_t)(gb0 + b) * a.h_v + h) * SS);
        f16x4 hv[NT];
#pragma unroll
        for (int tm = 0; tm < NT; ++tm) hv[tm] = h4(dh[tm]);
        f32x4 zt[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const f16x8 d = __builtin_shufflevector(hv[2 * j], hv[2 * j + 1], 0, 1, 2, 3, 4, 5, 6, 7);
            zt[0] = __builtin_amdgcn_mfma_f32_16x16x32_f16(cur.uk[j], d, zt[0], 0, 0, 0);
            zt[1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(cur.uk[4 + j], d, zt[1], 0, 0, 0);
        }
#pragma unroll
        for (int tm = 0; tm < NT; ++tm) {
#pragma unroll
            for (int j = 0; j < 4; ++j) dh[tm][j] = fmaf(cur.gn, dh[tm][j], (float)cur.cs[tm][j]);
            *reinterpret_cast<f16x4 *>(dhb + co[tm >> 1] + (tm & 1 ? 0 : -4096)) = hv[tm];
        }
#pragma unroll
        for (int tm = 0; tm < NT; ++tm) asm volatile("" : "+v"(kt[tm]));   // all at hand here, not one by one
        bf16x8 zh, zl;   // -Z in two parts
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float z = -zt[t][j];
                zh[4 * t + j] = (__bf16)z;
                // an infinite Z stays one: its second part is zero, not inf - inf
                const float zf = (float)zh[4 * t + j];
                zl[4 * t + j] = (__bf16)(z == zf ? 0.f : z - zf);
            }
#pragma unroll
        for (int tm = 0; tm < NT; ++tm) dh[tm] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kt[tm], zh, dh[tm], 0, 0, 0);
#pragma unroll
        for (int tm = 0; tm < NT; ++tm) dh[tm] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kt[tm], zl, dh[tm], 0, 0, 0);
        // unconditional (the first block again at the end): behind a branch the loads in flight
        // would not be counted, and each step would wait for its successor's operands too
        fetch(b - kScanSets + 1 > blo ? b - kScanSets + 1 : blo, nxt);
        // the sets' loads stay apart and in order, so that a wait for one leaves the next in flight
        __builtin_amdgcn_sched_barrier(0);
    };
    // three sets: block b's operands were loaded two steps earlier
    Ops o0, o1, o2;
    if (bhi > blo) {
        // the chain's last block may be partial; the ones before it are whole
        k_rows((int)(r1 - r0 - (long)(bhi - 1) * a.L < a.L ? r1 - r0 - (long)(bhi - 1) * a.L : a.L));
        fetch(bhi - 1, o0);
        __builtin_amdgcn_sched_barrier(0);
        if (bhi - 1 > blo) k_rows(a.L);
        fetch(bhi - 2 > blo ? bhi - 2 : blo, o1);
        __builtin_amdgcn_sched_barrier(0);
        // whole rounds of the three sets without a branch inside, then the rest
        int b = bhi - 1;
        for (; b - 2 >= blo; b -= 3) {
            step(b, o0, o2);
            step(b - 1, o1, o0);
            step(b - 2, o2, o1);
        }
        if (b >= blo) step(b, o0, o2);
        if (b - 1 >= blo) step(b - 1, o1, o0);
    }
    float *d0 = !to_dh0 ? carry : (a.dh0 ? a.dh0 + so : nullptr);
    if (d0) {
        const float f = to_dh0 ? a.range[1] : 1.f;
#pragma unroll
        for (int tm = 0; tm < NT; ++tm)
#pragma unroll
            for (int j = 0; j < 4; ++j) d0[(16 * tm + j) * DD] = dh[tm][j] * f;
    }
}

hipError_t launch_bwd_scan(const BwdArgs &a, hipStream_t s)
{
    // a wave per 16 columns of a chain, the chains padded to the XCDs
    hipLaunchKernelGGL(bdgdn_bwd_scan_kernel, dim3((a.n_chains + 7) / 8 * 8 * (DD / 16)), dim3(64), 0, s, a);
    return hipGetLastError();
}

}  // namespace bdgdn
