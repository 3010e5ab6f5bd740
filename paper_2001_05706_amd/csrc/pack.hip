// pack.hip -- conversions between the canonical FP64 layout of the ABI and
// the packed per-parity layouts of the kernels, and the bandwidth-reference
// copy kernel.  Links are compressed to 12 reals (two rows) when recon = 12,
// as in the caption of Table 2.
#include "wl_kernels.h"

namespace wl {

__device__ __forceinline__ size_t lex_site(const SysDesc &d, const Site &s)
{
    return (size_t)s.x + (size_t)d.L[0] * (s.y + (size_t)d.L[1] * (s.z + (size_t)d.L[2] * s.t));
}

// Canonical <-> packed spinors.  Bound by HBM: 192 bytes per canonical site and
// the packed site once each.  The sites 2 cb and 2 cb + 1 (one of each parity)
// are neighbours in the canonical layout, so the sites of consecutive
// checkerboard indices are one contiguous piece of it.  A thread that reads or
// writes its own site touches 16 bytes of 64 different lines per instruction;
// here a block moves its piece of the canonical field in 16-byte elements,
// consecutive lanes on consecutive elements, and turns it into sites through
// LDS.  12 x 24^3x48, FP32: one parity packed in 241 us (1.15 GB) instead of 347,
// unpacked with the other parity zeroed in 375 us (1.9 GB) instead of 325 + 220.
//
// A site's row in LDS is padded to 112 bytes (FP32 arithmetic) or 208 (FP64):
// 16-byte accesses of lanes one or two rows apart then fall on different banks.
constexpr int kPackBlock = 256;   // threads, and checkerboard sites of a map block
template <class T> constexpr int kPackRow = sizeof(T) == 4 ? 28 : 26;

// which of the sites 2 cb, 2 cb + 1 has the parity `parity`
__device__ __forceinline__ int pair_slot(const SysDesc &sd, int cb, int parity)
{
    return cb_coords(sd, cb, parity).x & 1;
}

// The first number of the pair (2 c0, 2 c0 + 1) of vector vd in the canonical layout
__device__ __forceinline__ double *canon_pair(const PackArgs &a, const VecDesc &vd, const SysDesc &sd, int c0)
{
    return const_cast<double *>(a.canon[vd.sys]) + ((size_t)vd.rhs * (size_t)sd.Vh + (size_t)c0) * 48;
}

// BOTH: blocks of 128 indices, both parities (f, fn: even; f2, fn2: odd);
// otherwise blocks of 256 indices of the parity a.parity.
template <int P, bool BOTH>
__global__ __launch_bounds__(kPackBlock) void k_pack_spinor(PackArgs a)
{
    using T = typename SpinorFmt<P>::real;
    using CH = typename SpinorFmt<P>::chunk;
    constexpr int ROW = kPackRow<T>, NCB = BOTH ? kPackBlock / 2 : kPackBlock;
    __shared__ __align__(16) T s_site[kPackBlock * ROW];
    __shared__ unsigned long long s_slot[kPackBlock / 64];  // pair_slot of the block's indices, a bit each
    const int tid = (int)threadIdx.x;
    const int lb = xcd_remap(blockIdx.x, BOTH ? 2 * a.nblocks : a.nblocks);
    const BlkMap bm = a.map[BOTH ? lb >> 1 : lb];
    const VecDesc vd = a.vec[bm.v];
    const SysDesc sd = a.sys[vd.sys];
    const int c0 = bm.lblk * kPackBlock + (BOTH ? (lb & 1) * NCB : 0);
    const int n = min(NCB, sd.Vh - c0);  // checkerboard indices of this block
    if (n <= 0) return;
    const int j = BOTH ? tid & (NCB - 1) : tid, par = BOTH ? tid / NCB : a.parity;
    const int slot = pair_slot(sd, min(c0 + j, sd.Vh - 1), par);
    if constexpr (!BOTH) {
        const unsigned long long m = __ballot(slot);
        if ((tid & 63) == 0) s_slot[tid >> 6] = m;
        __syncthreads();
    }
    const double *src = canon_pair(a, vd, sd, c0);
    const int nel = (BOTH ? 24 : 12) * n;
    double2 w[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) {
        const int i = k * kPackBlock + tid;
        size_t e = (size_t)i;
        if constexpr (!BOTH) {
            const int q = i / 12;  // index within the block; element i % 12 of its site of this parity
            e = (size_t)(i + 12 * q + 12 * (int)((s_slot[q >> 6] >> (q & 63)) & 1));
        }
        if (i < nel) w[k] = ld_canon(src + 2 * e);
    }
#pragma unroll
    for (int k = 0; k < 12; ++k) {
        const int i = k * kPackBlock + tid;
        if (i < nel) {
            T *d = s_site + (i / 12) * ROW + 2 * (i % 12);
            d[0] = (T)w[k].x;
            d[1] = (T)w[k].y;
        }
    }
    __syncthreads();
    if (j >= n) return;
    T v[24];
    const T *r = s_site + (BOTH ? 2 * j + slot : j) * ROW;
#pragma unroll
    for (int k = 0; k < 24; ++k) v[k] = r[k];
    void *f = BOTH && par ? a.f2 : a.f;
    float *fn = BOTH && par ? a.fn2 : a.fn;
    store_spinor<P>((CH *)f + (size_t)vd.site_off * SpinorFmt<P>::nchunk, fn ? fn + vd.site_off : nullptr, sd.stride,
                    c0 + j, v);
}

// Blocks of 128 indices; every canonical element of both sites is written.
// BOTH: the even field f and the odd field f2; otherwise the field f of parity
// a.parity and zeros on the other parity.
template <int P, bool BOTH>
__global__ __launch_bounds__(kPackBlock) void k_unpack_spinor(PackArgs a)
{
    using T = typename SpinorFmt<P>::real;
    using CH = typename SpinorFmt<P>::chunk;
    constexpr int ROW = kPackRow<T>, NCB = kPackBlock / 2;
    __shared__ __align__(16) T s_site[kPackBlock * ROW];
    const int tid = (int)threadIdx.x;
    const int lb = xcd_remap(blockIdx.x, 2 * a.nblocks);
    const BlkMap bm = a.map[lb >> 1];
    const VecDesc vd = a.vec[bm.v];
    const SysDesc sd = a.sys[vd.sys];
    const int c0 = bm.lblk * kPackBlock + (lb & 1) * NCB;
    const int n = min(NCB, sd.Vh - c0);
    if (n <= 0) return;
    const int j = tid & (NCB - 1), half = tid / NCB;
    if (j < n) {
        const int par = BOTH ? half : (half ? 1 - a.parity : a.parity);
        const int cb = c0 + j;
        T v[24];
        if (BOTH || half == 0) {
            const void *f = BOTH && half ? a.f2 : a.f;
            const float *fn = BOTH && half ? a.fn2 : a.fn;
            load_spinor<P>((const CH *)f + (size_t)vd.site_off * SpinorFmt<P>::nchunk, fn ? fn + vd.site_off : nullptr,
                           sd.stride, cb, v);
        } else {
#pragma unroll
            for (int k = 0; k < 24; ++k) v[k] = 0;
        }
        T *r = s_site + (2 * j + pair_slot(sd, cb, par)) * ROW;
#pragma unroll
        for (int k = 0; k < 24; ++k) r[k] = v[k];
    }
    __syncthreads();
    double *dst = canon_pair(a, vd, sd, c0);
#pragma unroll
    for (int k = 0; k < 12; ++k) {
        const int i = k * kPackBlock + tid;
        if (i < 24 * n) {
            const T *r = s_site + (i / 12) * ROW + 2 * (i % 12);
            st_canon(dst + 2 * (size_t)i, (double)r[0], (double)r[1]);
        }
    }
}

template <int P, int R>
__global__ __launch_bounds__(256) void k_pack_gauge(const double *U, void *out, SysDesc d)
{
    const int tid = blockIdx.x * blockDim.x + threadIdx.x;
    if (tid >= 2 * d.Vh) return;
    const int parity = tid / d.Vh, cb = tid - parity * d.Vh;
    const Site st = cb_coords(d, cb, parity);
    const size_t s = lex_site(d, st);
    constexpr int NCH = LinkFmt<P, R>::nchunk;
    using CH = typename LinkFmt<P, R>::chunk;
    for (int mu = 0; mu < 4; ++mu) {
        double u[18];
        const double *src = U + (s * 4 + mu) * 18;
        for (int k = 0; k < 18; ++k) u[k] = src[k];
        store_link<P, R>((CH *)out + (size_t)((parity * 4 + mu) * NCH) * d.gstride, d.gstride, cb, u);
    }
}

// Reference copy for the achievable-bandwidth figure: one 16-byte element per
// thread with non-temporal loads and stores (the fastest plain copy measured
// on gfx950: one element per thread beats grid-stride loops and unrolling)
__global__ __launch_bounds__(256) void k_copy_bw(const float4 *__restrict__ in, float4 *__restrict__ out, size_t n)
{
    const size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    if (i < n) WL_NT_STORE(nt_f4, WL_NT_LOAD(nt_f4, in + i), out + i);
}

// The same copy with ordinary (cached) loads and stores: operands small enough
// for the last-level cache stay there between launches.
__global__ __launch_bounds__(256) void k_copy_cached(const float4 *__restrict__ in, float4 *__restrict__ out, size_t n)
{
    const size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    if (i < n) out[i] = in[i];
}

// Read-only reference: each thread sums four 16-byte elements a grid apart
// with ordinary loads; the sum is stored only when it equals a value a zeroed
// buffer never produces, so no store reaches memory.
__global__ __launch_bounds__(256) void k_read_cached(const float4 *__restrict__ in, float *__restrict__ out, size_t n)
{
    const size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x, st = (size_t)gridDim.x * blockDim.x;
    float s = 0.f;
#pragma unroll
    for (int k = 0; k < 4; ++k)
        if (i + k * st < n) {
            const float4 v = in[i + k * st];
            s += (v.x + v.y) + (v.z + v.w);
        }
    if (s == 1.0f) out[blockIdx.x] = s;
}

template <int P>
static hipError_t launch_pack_t(bool unpack, const PackArgs &a, hipStream_t s)
{
    // (the map's blocks hold kPackBlock indices; the kernels take 128 at a time
    // except when they read one parity)
    const dim3 b(kPackBlock), whole(a.nblocks), halves(2 * a.nblocks);
    if (unpack && a.both)
        hipLaunchKernelGGL((k_unpack_spinor<P, true>), halves, b, 0, s, a);
    else if (unpack)
        hipLaunchKernelGGL((k_unpack_spinor<P, false>), halves, b, 0, s, a);
    else if (a.both)
        hipLaunchKernelGGL((k_pack_spinor<P, true>), halves, b, 0, s, a);
    else
        hipLaunchKernelGGL((k_pack_spinor<P, false>), whole, b, 0, s, a);
    return hipGetLastError();
}

static hipError_t launch_pack_any(bool unpack, int prec, const PackArgs &a, int block, hipStream_t s)
{
    if (block != kPackBlock) return hipErrorInvalidValue;
    switch (prec) {
    case P_F64: return launch_pack_t<P_F64>(unpack, a, s);
    case P_F32: return launch_pack_t<P_F32>(unpack, a, s);
    case P_F16: return launch_pack_t<P_F16>(unpack, a, s);
    case P_BF16: return launch_pack_t<P_BF16>(unpack, a, s);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_pack_spinor(int prec, const PackArgs &a, int block, hipStream_t s)
{
    return launch_pack_any(false, prec, a, block, s);
}

hipError_t launch_unpack_spinor(int prec, const PackArgs &a, int block, hipStream_t s)
{
    return launch_pack_any(true, prec, a, block, s);
}

hipError_t launch_pack_gauge(int prec, int recon, const double *U, void *out, const SysDesc &d, hipStream_t s)
{
    const int n = 2 * d.Vh, blk = 256, grid = (n + blk - 1) / blk;
    if (prec == P_F64 && recon == 18) hipLaunchKernelGGL((k_pack_gauge<P_F64, 18>), dim3(grid), dim3(blk), 0, s, U, out, d);
    else if (prec == P_F64 && recon == 12) hipLaunchKernelGGL((k_pack_gauge<P_F64, 12>), dim3(grid), dim3(blk), 0, s, U, out, d);
    else if (prec == P_F32 && recon == 18) hipLaunchKernelGGL((k_pack_gauge<P_F32, 18>), dim3(grid), dim3(blk), 0, s, U, out, d);
    else if (prec == P_F32 && recon == 12) hipLaunchKernelGGL((k_pack_gauge<P_F32, 12>), dim3(grid), dim3(blk), 0, s, U, out, d);
    else if (prec == P_F16 && recon == 12) hipLaunchKernelGGL((k_pack_gauge<P_F16, 12>), dim3(grid), dim3(blk), 0, s, U, out, d);
    else if (prec == P_BF16 && recon == 12) hipLaunchKernelGGL((k_pack_gauge<P_BF16, 12>), dim3(grid), dim3(blk), 0, s, U, out, d);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_copy_bw(int mode, const void *in, void *out, size_t bytes, hipStream_t s)
{
    const size_t n = bytes / sizeof(float4);
    const int blk = 256;
    // the read-only kernel takes four elements per thread and stores at most
    // one float per block into `out` (which holds `bytes` bytes)
    const size_t grid = mode == 2 ? (n / 4 + blk - 1) / blk : (n + blk - 1) / blk;
    if (grid > 0x7FFFFFFFu || grid == 0) return hipErrorInvalidValue;
    if (mode == 0)
        hipLaunchKernelGGL(k_copy_bw, dim3((unsigned)grid), dim3(blk), 0, s, (const float4 *)in, (float4 *)out, n);
    else if (mode == 1)
        hipLaunchKernelGGL(k_copy_cached, dim3((unsigned)grid), dim3(blk), 0, s, (const float4 *)in, (float4 *)out, n);
    else if (mode == 2)
        hipLaunchKernelGGL(k_read_cached, dim3((unsigned)grid), dim3(blk), 0, s, (const float4 *)in, (float *)out, n);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace wl
