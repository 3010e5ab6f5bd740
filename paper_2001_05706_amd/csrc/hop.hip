// hop.hip -- the single-parity Wilson hopping kernel (the D-slash of Table 2)
// with a fused linear-combination epilogue and optional fused |out|^2.
//
// One thread per output site of one vector (variant 11: eight, one a direction).
// Per direction the neighbour spinor is spin-projected to two components (12 flop),
// both are multiplied by the link (2 x 66 flop) rebuilt from 12 reals when recon = 12,
// and the result is spin-reconstructed into the accumulator (24 flop): 1320 flop per
// site.  Each link is used once per hop and right-hand side; neighbour
// spinors are shared by up to 8 output sites through L2, which the XCD-aware
// block order keeps on one die.
#include <algorithm>

#include <hip/hip_ext.h>

#include "wl_reduce.h"
#include "wl_kernels.h"

namespace wl {

// Launch variants the autotuner chooses from, with the block size:
//   fence: directions whose operands may be in flight together per wave
//   waves: occupancy target (waves per SIMD), which caps registers at 512/waves
//   nt:    non-temporal link loads or cached ones (cached win wherever a cache
//          line of links is shared: by the right-hand sides of a set, and by
//          neighbouring waves whose backward-link rows start mid line)
//   0: fence 2, 4 waves (FP64: 2), non-temporal links
//   1: fence 1, 5 waves (FP64: 3), non-temporal links
//   2: fence 1, 6 waves (FP64: 3), non-temporal links
//   3: fence 2, 4 waves (FP64: 2), cached links
//   4: fence 4, 4 waves, cached links -- twice the bytes in flight per wave
//   5: fence 4, 5 waves, cached links
//   6: as 3, but the waves of a block serve consecutive right-hand sides of one
//      system on the same 64 sites, so the links they share hit in the CU's L1
//      (multi-RHS sets; launched on the layouts of `ExecSet::layout(-G)`)
//   7: each thread serves two right-hand sides of one system at its site: the
//      neighbour index and each link (with its recon-12 row) are formed once
//      for both; one direction in flight, 3 waves (multi-RHS sets; pair layouts)
//   8: the waves of a block serve consecutive right-hand sides of one system on
//      the same 64 sites (as 6), and the block's 8 x 64 links are read, rebuilt
//      to 18 reals and stored in LDS once, together with the neighbour indices,
//      before any wave starts its hop: no right-hand side repeats a link load,
//      the recon-12 arithmetic or the site-coordinate arithmetic (FP32 and
//      half-precision storage; not with the clover epilogue)
//   9: pencil blocks (k_hop_pencil): the waves of a block take the same 64
//      positions of consecutive time slices and pass each other their time
//      neighbours through LDS; fence 2, non-temporal links
//  10: pencil blocks with cached links; fence 4 for FP16/BF16, 2 for FP32
//      (FP32 and half-precision storage, Wilson epilogue; lattices whose time
//      slices hold a multiple of 64 sites)
//  11: the eight directions of 64 sites on the eight waves of a block (k_hop_split)
// Variants 4 and 5 exist for FP16/BF16 storage only (FP32 and FP64 operands of
// four directions do not fit the registers).
template <int SP, int VAR> struct HopVar {
    static constexpr bool half = SP == P_F16 || SP == P_BF16;
    static constexpr int fence = VAR == 0 || VAR == 3 || VAR == 6 || VAR == 9
                                     ? 2
                                     : (VAR == 4 || VAR == 5 || VAR == 10 ? (half ? 4 : 2) : 1);
    static constexpr int waves = SP == P_F64 ? (VAR == 0 || VAR >= 3 ? 2 : 3)
                                             : (VAR == 7 ? 3 : VAR == 0 || VAR == 3 || VAR == 4 || VAR == 6 || VAR >= 9
                                                                   ? 4
                                                                   : VAR == 2 ? 6 : 5);
    static constexpr bool nt = VAR < 3 || VAR == 9;
    static constexpr bool rhs_waves = VAR == 6;
    static constexpr bool rhs_pairs = VAR == 7;
    // largest block: 1024 threads (16 waves on one CU, 4 per SIMD) where the
    // occupancy target already allows 4 waves per SIMD; 512 otherwise
    static constexpr int max_block = waves >= 4 && VAR < 6 ? 1024 : 512;
};
constexpr int kHopVariants = 12;

// What a hop's epilogue ends in, one instantiation each: EP_CANON stores the
// canonical FP64 field instead of the packed one.  (Bit 2, variant 11 only: the
// input and X0 are read from the canonical field too.)
enum { EP_WILSON = 0, EP_CLOVER = 1, EP_CANON = 2, EP_CLOVER_CANON = 3, EP_DIRECT = 4 };

// The fields of the output parity a block computes: the launch's first slot,
// or for the odd blocks of a twin launch the second one.  X and Xn point into
// the kernel's argument block, so that an index that varies at run time still
// reads them with scalar loads.
struct HopIO {
    int parity;
    const void *in;
    const float *in_norm;
    void *out;
    float *out_norm;
    const void *const *X;
    const float *const *Xn;
};

// Epilogue field X[j] at site cb, before its half-precision norm is applied.
// Each X field is read once per launch; for sets whose fields are large
// against the last-level cache the read is non-temporal, so that it does not
// push out the links that the solver's next hops re-read from that cache.
template <int SP>
__device__ __forceinline__ void load_x(const HopArgs &a, const HopIO &f, int j, size_t voff, const VecDesc &vd,
                                       const SysDesc &sd, int cb, typename SpinorFmt<SP>::real x[24],
                                       typename SpinorFmt<SP>::real *nx)
{
    using CH = typename SpinorFmt<SP>::chunk;
    const CH *base = (const CH *)f.X[j] + voff;
    const float *nrm = f.Xn[j] ? f.Xn[j] + vd.site_off : nullptr;
    if (a.stream)
        load_spinor_raw<SP, true>(base, nrm, sd.stride, cb, x, nx);
    else
        load_spinor_raw<SP, false>(base, nrm, sd.stride, cb, x, nx);
}

// An FP64 result rounded to the field a.lo (as k_convert rounds; plain stores: the
// next hop reads it).  A reliable update's residual is only wanted in the sloppy
// precision: storing it in FP64 and converting it cost the 32^3x64 FP16 solve a
// further 400 MB (201 written, 201 read) and a launch, about 90 us of each update's 750.
__device__ __forceinline__ void store_lo(const HopArgs &a, const VecDesc &vd, const SysDesc &sd, int cb, const double o[24])
{
    float y[24];
#pragma unroll
    for (int k = 0; k < 24; ++k) y[k] = (float)o[k];
    if (a.lo_prec == P_F32) {
        store_spinor<P_F32>((float4 *)a.lo + (size_t)vd.site_off * 6, nullptr, sd.stride, cb, y);
    } else {
        uint4 *base = (uint4 *)a.lo + (size_t)vd.site_off * 3;
        if (a.lo_prec == P_F16) {
            // FP16 rounds the exact product y / m once, BF16 the FP32 product: kept
            // apart, or the compiler forms products for both ahead of the branch
#pragma unroll
            for (int k = 0; k < 24; ++k) asm("" : "+v"(y[k]));
            store_spinor<P_F16>(base, a.lo_norm + vd.site_off, sd.stride, cb, y);
        } else
            store_spinor<P_BF16>(base, a.lo_norm + vd.site_off, sd.stride, cb, y);
    }
}

// Everything after the hopping sum at one output site of one vector: the
// linear-combination epilogue, the store, and the site's reduction values.
// acc holds H psi (FP16/BF16: already multiplied by the system's c).  CANON:
// the result stays in acc, rounded as the packed field would hold it.
template <int SP, bool CLOV, bool CANON = false>
__device__ __forceinline__ void hop_epilogue(const HopArgs &a, const HopIO &f, const VecDesc &vd, const SysDesc &sd,
                                             int cb, typename SpinorFmt<SP>::real acc[24], double rv[3])
{
    using T = typename SpinorFmt<SP>::real;
    using CH = typename SpinorFmt<SP>::chunk;
    constexpr int NC = SpinorFmt<SP>::nchunk;
    const size_t voff = (size_t)vd.site_off * NC;
    const double *cf = a.epi.coef + vd.sys * 5;
    constexpr bool HALF = SP == P_F16 || SP == P_BF16;
    // acc = c H psi from here on (half precision: c rode on the accumulation)
    if constexpr (!HALF) {
        const T c = (T)cf[4];
#pragma unroll
        for (int k = 0; k < 24; ++k) acc[k] *= c;
    }

    // clover term of this system at the output site (FP16/BF16 launches read the FP16 copy)
    constexpr int CP = clover_prec<SP>();
    const bool clov = CLOV && a.epi.clov != 0 && sd.clov != nullptr;
    T o[24];
    if (a.epi.nx >= 1) {
        // operand values before their site norm; the norm joins the coefficient
        T x[24], n0 = 1;
        bool raw = true;
        if constexpr (CLOV) {
            if (clov && (a.epi.clov & EPI_CLOV_X0)) {
                load_spinor<SP>((const CH *)f.X[0] + voff, f.Xn[0] ? f.Xn[0] + vd.site_off : nullptr,
                                sd.stride, cb, x);
                clover_apply<CP>(clover_parity<CP>(sd.clov, f.parity, sd.stride), sd.stride, cb, x);
                n0 = 1;
                raw = false;
            }
        }
        if (raw) load_x<SP>(a, f, 0, voff, vd, sd, cb, x, &n0);
        const T s0 = (T)cf[0] * n0;
#pragma unroll
        for (int k = 0; k < 24; ++k) o[k] = fmadd(x[k], s0, acc[k]);
    } else {
#pragma unroll
        for (int k = 0; k < 24; ++k) o[k] = acc[k];
    }
    if (a.epi.g5) {
#pragma unroll
        for (int k = 12; k < 24; ++k) o[k] = -o[k];
    }
    if constexpr (CLOV) {
        if (clov && (a.epi.clov & EPI_CLOV_INV))
            clover_apply<CP>(clover_parity<CP>(sd.clovinv, f.parity, sd.stride), sd.stride, cb, o);
    }
    for (int j = 1; j < a.epi.nx; ++j) {
        T x[24], nj;
        load_x<SP>(a, f, j, voff, vd, sd, cb, x, &nj);
        const T sj = (T)cf[j] * nj;
#pragma unroll
        for (int k = 0; k < 24; ++k) o[k] = fmadd(x[k], sj, o[k]);
    }
    if constexpr (CANON) {
        round_spinor<SP>(o);
#pragma unroll
        for (int k = 0; k < 24; ++k) acc[k] = o[k];
        return;
    }
    if (SP == P_F64 && a.lo) {
        if constexpr (SP == P_F64) store_lo(a, vd, sd, cb, o);
    } else {
        store_spinor<SP, true>((CH *)f.out + voff, f.out_norm ? f.out_norm + vd.site_off : nullptr, sd.stride, cb, o);
    }
    if (a.red.kind != RED_NONE) {
        if (a.red.mode == RM_NORM) {
            rv[0] = site_norm2(o);
        } else {
            // the X field was read above; this re-read hits in cache.  The
            // products are linear in x: its site norm scales the site sums.
            const int j = a.red.mode == RM_DOT_X1 ? 1 : 0;
            T x[24], nx;
            load_spinor_raw<SP>((const CH *)f.X[j] + voff, f.Xn[j] ? f.Xn[j] + vd.site_off : nullptr,
                                sd.stride, cb, x, &nx);
            if (a.red.mode == RM_DOT_X1) {
                site_cdot(x, o, rv[0], rv[1]);
            } else {
                site_cdot(o, x, rv[0], rv[1]);
                rv[2] = site_norm2(o);
            }
            rv[0] *= (double)nx;
            rv[1] *= (double)nx;
        }
    }
}

// EP_CANON: a wave stores the canonical sites of its 64 consecutive checkerboard
// indices, through LDS private to the wave, consecutive lanes on consecutive 16
// bytes.  A single-parity launch also zeroes the sites of the other parity, so
// the wave writes one contiguous 24 KB; a launch that leaves them writes
// 192-byte pieces.  Whole lines matter: with 64 bytes of a site per step
// (a third of the LDS) the 32^3x64 FP16 hop with this epilogue took 190 us,
// with whole lines 139, the packed hop and a separate unpack 158 (cold operands).
// The row pitch puts the 16-byte accesses of neighbouring lanes on different banks.
template <class T> constexpr int kStageRow = sizeof(T) == 4 ? 24 : 26;
template <class T> constexpr int kStageBytes = 64 * kStageRow<T> * (int)sizeof(T);  // per wave

template <class T>
__device__ __forceinline__ void store_canon(const HopArgs &a, const HopIO &f, const VecDesc &vd, const SysDesc &sd,
                                            int cb, bool live, const T o[24], void *stage)
{
    const int lane = (int)threadIdx.x & 63;
    const int c0 = __builtin_amdgcn_readfirstlane(cb - lane);
    const int n = live ? min(64, sd.Vh - c0) : 0;  // sites of the wave (uniform)
    if (n <= 0) return;
    // which site of each pair is the output's
    const unsigned long long slots = __ballot(cb_coords(sd, min(cb, sd.Vh - 1), f.parity).x & 1);
    double *base = a.canon + ((size_t)vd.rhs * (size_t)sd.Vh + (size_t)c0) * 48;
    const T *st = (const T *)stage;
    T *row = (T *)stage + lane * kStageRow<T>;
    wave_lds_fence();  // an earlier vector's sites may still be read
#pragma unroll
    for (int k = 0; k < 24; ++k) row[k] = o[k];
    wave_lds_fence();
    if (a.canon_zero) {
#pragma unroll
        for (int i = 0; i < 24; ++i) {
            const int e = i * 64 + lane, j = e / 24, r = e % 24;  // pair, 16-byte element of the pair
            const int q = r < 12 ? r : r - 12;
            const bool mine = (int)((slots >> (j & 63)) & 1) == (r >= 12);
            const T *w = st + j * kStageRow<T> + 2 * q;
            if (j < n) st_canon(base + 2 * e, mine ? (double)w[0] : 0.0, mine ? (double)w[1] : 0.0);
        }
    } else {
#pragma unroll
        for (int i = 0; i < 12; ++i) {
            const int e = i * 64 + lane, j = e / 12, q = e % 12;
            const T *w = st + j * kStageRow<T> + 2 * q;
            if (j < n)
                st_canon(base + 48 * j + 24 * (int)((slots >> (j & 63)) & 1) + 2 * q, (double)w[0], (double)w[1]);
        }
    }
}

template <int SP>
__device__ __forceinline__ HopSite hop_input(const HopArgs &a, const HopIO &f, const VecDesc &vd, const SysDesc &sd)
{
    using CH = typename SpinorFmt<SP>::chunk;
    constexpr bool HALF = SP == P_F16 || SP == P_BF16;
    HopSite hs;
    hs.in = (const CH *)f.in + (size_t)vd.site_off * SpinorFmt<SP>::nchunk;
    hs.in_norm = f.in_norm ? f.in_norm + vd.site_off : nullptr;
    hs.stride = sd.stride;
    hs.gauge = sd.gauge;
    hs.gstride = sd.gstride;
    hs.scale = HALF ? (float)a.epi.coef[vd.sys * 5 + 4] : 1.0f;
    return hs;
}

template <int SP, int GP, int R, bool DAG, int VAR, int EP>
__global__ __launch_bounds__((HopVar<SP, VAR>::max_block)) __attribute__((amdgpu_waves_per_eu(HopVar<SP, VAR>::waves)))
void k_hop(HopArgs a)
{
    using T = typename SpinorFmt<SP>::real;
    constexpr bool CLOV = EP == EP_CLOVER || EP == EP_CLOVER_CANON, CANON = EP >= EP_CANON;

    constexpr bool RW = HopVar<SP, VAR>::rhs_waves;
    constexpr bool PAIR = HopVar<SP, VAR>::rhs_pairs;
    const int lb = xcd_remap(blockIdx.x, a.nblocks);
    // a twin launch's odd blocks compute the other output parity from the second
    // field slot (the selection is uniform over the block)
    const bool second = a.twin && (lb & 1);
    const HopIO f = second ? HopIO{1 - a.parity, a.in_b, a.in_norm_b, a.out_b, a.out_norm_b, a.X_b, a.Xn_b}
                           : HopIO{a.parity, a.in, a.in_norm, a.out, a.out_norm, a.epi.X, a.epi.Xn};
    const BlkMap bm = a.map[a.twin ? lb >> 1 : lb];
    int v = bm.v, cb;
    bool valid = true;
    if constexpr (RW) {
        // wave w serves vector bm.v + w (when it is a further rhs of the same system) on 64 sites
        // wave-uniform: keep the vector's descriptors in scalar registers
        const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
        v = bm.v + w;
        valid = v < a.nvec && a.vec[v].sys == a.vec[bm.v].sys && (!a.active || a.active[v]);
        cb = bm.lblk * 64 + ((int)threadIdx.x & 63);
    } else if constexpr (PAIR) {
        cb = bm.lblk * (int)blockDim.x + (int)threadIdx.x;
    } else {
        if (a.active && !a.active[a.one ? 0 : bm.v]) return;
        cb = bm.lblk * (int)blockDim.x + (int)threadIdx.x;
    }
    // (single-vector sets: the indices are known, so the descriptor loads do
    // not wait for the block map)
    const VecDesc vd = a.vec[a.one ? 0 : (valid ? v : bm.v)];
    const SysDesc sd = a.sys[a.one ? 0 : vd.sys];
    // the block's start stamp goes to memory at once, after the descriptor
    // loads are issued (held in registers across the body, or read before
    // them, it costs the FP16 kernel four registers and a spill)
    if (a.stamps && threadIdx.x == 0) a.stamps[2 * lb] = (unsigned long long)wall_clock64();

    if constexpr (PAIR) {
        // vectors bm.v and bm.v + 1 (when that is a further rhs of the same
        // system); an absent second vector is computed from the first and not stored
        const int v1 = bm.v + 1;
        const bool has1 = v1 < a.nvec && a.vec[v1].sys == vd.sys;
        const bool live0 = !a.active || a.active[bm.v];
        const bool live1 = has1 && (!a.active || a.active[v1]);
        if (!live0 && !live1) return;
        const VecDesc vd1 = a.vec[has1 ? v1 : bm.v];
        double rv0[3] = {0.0, 0.0, 0.0}, rv1[3] = {0.0, 0.0, 0.0};
        T acc0[24], acc1[24];
        if (cb < sd.Vh) {
            const HopSite hs0 = hop_input<SP>(a, f, vd, sd), hs1 = hop_input<SP>(a, f, vd1, sd);
            hop_site2<SP, GP, R, DAG, HopVar<SP, VAR>::nt>(sd, hs0, hs1, f.parity, cb, acc0, acc1);
            if (live0) hop_epilogue<SP, CLOV, CANON>(a, f, vd, sd, cb, acc0, rv0);
            if (live1) hop_epilogue<SP, CLOV, CANON>(a, f, vd1, sd, cb, acc1, rv1);
        }
        if constexpr (CANON) {
            extern __shared__ uint4 s_stage[];
            void *stage = (char *)s_stage + (threadIdx.x >> 6) * kStageBytes<T>;
            store_canon<T>(a, f, vd, sd, cb, live0, acc0, stage);
            store_canon<T>(a, f, vd1, sd, cb, live1, acc1, stage);
        }
        // live0 and live1 are uniform over the block
        if (a.red.kind != RED_NONE && live0) block_reduce_store_n(a.red, vd.pslot0, bm.lblk, rv0);
        if (a.red.kind != RED_NONE && live1) block_reduce_store_n(a.red, vd1.pslot0, bm.lblk, rv1);
    } else {
        double rv[3] = {0.0, 0.0, 0.0};
        T acc[24];
        if (valid && cb < sd.Vh) {
            const HopSite hs = hop_input<SP>(a, f, vd, sd);
            hop_site<SP, GP, R, DAG, HopVar<SP, VAR>::fence, HopVar<SP, VAR>::nt>(sd, hs, f.parity, cb, acc);
            hop_epilogue<SP, CLOV, CANON>(a, f, vd, sd, cb, acc, rv);
        }
        if constexpr (CANON) {
            extern __shared__ uint4 s_stage[];
            store_canon<T>(a, f, vd, sd, cb, valid, acc, (char *)s_stage + (threadIdx.x >> 6) * kStageBytes<T>);
        }
        if constexpr (RW) {
            if (a.red.kind != RED_NONE && valid) wave_reduce_store_n(a.red, vd.pslot0, bm.lblk, rv);
        } else {
            if (a.red.kind != RED_NONE) block_reduce_store_n(a.red, vd.pslot0, bm.lblk, rv);
        }
    }
    if (a.stamps) {
        // the block's work ends when its last wave ends
        __syncthreads();
        if (threadIdx.x == 0) a.stamps[2 * lb + 1] = (unsigned long long)wall_clock64();
    }
}

// Variant 8.  LDS holds, per direction d = 2 mu + (backward), the rebuilt link
// of each of the block's 64 sites as 9 complex numbers ([d][element][site], so
// a wave's 64 lanes read 64 consecutive float2) and the neighbour's
// checkerboard index with the antiperiodic sign in bit 31: 38.9 KB per block.
constexpr int kLdsLinkBytes = 8 * 9 * 64 * (int)sizeof(float2) + 8 * 64 * (int)sizeof(int);

template <int GP, int R, int MU, int DIR>
__device__ __forceinline__ void stage_dir(const SysDesc &sd, const HopSite &hs, int parity, const Site &st, int cb,
                                          int lane, bool nt, float2 (*su)[64], int *sn)
{
    bool flip;
    const int ncb = neighbour<MU, DIR>(sd, st, cb, flip);
    cpx<float> u[3][3];
    if (nt)
        hop_link<GP, R, MU, DIR, true>(hs, parity, cb, ncb, u);
    else
        hop_link<GP, R, MU, DIR, false>(hs, parity, cb, ncb, u);
#pragma unroll
    for (int k = 0; k < 9; ++k) su[k][lane] = float2{u[k / 3][k % 3].re, u[k / 3][k % 3].im};
    sn[lane] = (int)((unsigned)ncb | (flip ? 0x80000000u : 0u));
}

template <int SP, int MU, int DIR, bool DAG>
__device__ __forceinline__ void lds_dir(const HopSite &hs, int lane, const float2 (*su)[64], const int *sn,
                                        float acc[24])
{
    constexpr int SG = (DIR > 0) == DAG ? +1 : -1;
    const int nn = sn[lane];
    cpx<float> h0[3], h1[3];
    const float f = project_neighbour<SP, MU, SG>(hs, nn & 0x7fffffff, nn < 0, h0, h1);
    cpx<float> u[3][3];
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        const float2 w = su[k][lane];
        u[k / 3][k % 3] = cpx<float>{w.x, w.y};
    }
    hop_accumulate<SP, MU, DIR, SG>(u, h0, h1, f, acc);
}

template <int SP, int GP, int R, bool DAG, bool CANON>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(4))) void k_hop_lds(HopArgs a)
{
    static_assert(SP != P_F64, "variant 8 stages FP32 links");
    extern __shared__ uint4 s_dyn[];
    auto s_u = reinterpret_cast<float2(*)[9][64]>(s_dyn);
    auto s_n = reinterpret_cast<int(*)[64]>(s_u + 8);
    const int lb = xcd_remap(blockIdx.x, a.nblocks);
    const bool second = a.twin && (lb & 1);
    const HopIO f = second ? HopIO{1 - a.parity, a.in_b, a.in_norm_b, a.out_b, a.out_norm_b, a.X_b, a.Xn_b}
                           : HopIO{a.parity, a.in, a.in_norm, a.out, a.out_norm, a.epi.X, a.epi.Xn};
    const BlkMap bm = a.map[a.twin ? lb >> 1 : lb];
    const int lane = (int)threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int nw = (int)blockDim.x >> 6;
    const int sys = a.vec[bm.v].sys;
    auto live = [&](int v) { return v < a.nvec && a.vec[v].sys == sys && (!a.active || a.active[v]); };
    // a block whose right-hand sides have all converged has nothing to do
    bool any = false;
    for (int k = 0; k < nw; ++k) any = any || live(bm.v + k);
    if (!any) return;
    const SysDesc sd = a.sys[sys];
    const int cb = bm.lblk * 64 + lane;
    if (a.stamps && threadIdx.x == 0) a.stamps[2 * lb] = (unsigned long long)wall_clock64();

    // stage: wave w rebuilds the links of directions w, w + nw, ... (all waves
    // take part, also those whose right-hand side is idle).  When the block
    // holds every right-hand side of its system, no other block reads these
    // links (in a twin launch its twin does): they are loaded non-temporally.
    const bool nt = !a.twin && a.vec[bm.v].rhs == 0 && (bm.v + nw >= a.nvec || a.vec[bm.v + nw].sys != sys);
    if (cb < sd.Vh) {
        const Site st = cb_coords(sd, cb, f.parity);
        HopSite hl;
        hl.gauge = sd.gauge;
        hl.gstride = sd.gstride;
        for (int d = w; d < 8; d += nw) {
            switch (d) {
            case 0: stage_dir<GP, R, 0, +1>(sd, hl, f.parity, st, cb, lane, nt, s_u[0], s_n[0]); break;
            case 1: stage_dir<GP, R, 0, -1>(sd, hl, f.parity, st, cb, lane, nt, s_u[1], s_n[1]); break;
            case 2: stage_dir<GP, R, 1, +1>(sd, hl, f.parity, st, cb, lane, nt, s_u[2], s_n[2]); break;
            case 3: stage_dir<GP, R, 1, -1>(sd, hl, f.parity, st, cb, lane, nt, s_u[3], s_n[3]); break;
            case 4: stage_dir<GP, R, 2, +1>(sd, hl, f.parity, st, cb, lane, nt, s_u[4], s_n[4]); break;
            case 5: stage_dir<GP, R, 2, -1>(sd, hl, f.parity, st, cb, lane, nt, s_u[5], s_n[5]); break;
            case 6: stage_dir<GP, R, 3, +1>(sd, hl, f.parity, st, cb, lane, nt, s_u[6], s_n[6]); break;
            default: stage_dir<GP, R, 3, -1>(sd, hl, f.parity, st, cb, lane, nt, s_u[7], s_n[7]); break;
            }
        }
    }
    __syncthreads();

    const int v = bm.v + w;
    const bool valid = live(v);
    double rv[3] = {0.0, 0.0, 0.0};
    float acc[24];
    if (valid && cb < sd.Vh) {
        const VecDesc vd = a.vec[v];
        const HopSite hs = hop_input<SP>(a, f, vd, sd);
#pragma unroll
        for (int k = 0; k < 24; ++k) acc[k] = 0.f;
        // two directions' operands in flight per wave, as variant 6
        lds_dir<SP, 0, +1, DAG>(hs, lane, s_u[0], s_n[0], acc);
        lds_dir<SP, 0, -1, DAG>(hs, lane, s_u[1], s_n[1], acc);
        sched_fence(acc);
        lds_dir<SP, 1, +1, DAG>(hs, lane, s_u[2], s_n[2], acc);
        lds_dir<SP, 1, -1, DAG>(hs, lane, s_u[3], s_n[3], acc);
        sched_fence(acc);
        lds_dir<SP, 2, +1, DAG>(hs, lane, s_u[4], s_n[4], acc);
        lds_dir<SP, 2, -1, DAG>(hs, lane, s_u[5], s_n[5], acc);
        sched_fence(acc);
        lds_dir<SP, 3, +1, DAG>(hs, lane, s_u[6], s_n[6], acc);
        lds_dir<SP, 3, -1, DAG>(hs, lane, s_u[7], s_n[7], acc);
        sched_fence(acc);
        hop_epilogue<SP, false, CANON>(a, f, vd, sd, cb, acc, rv);
    }
    if constexpr (CANON) {
        __syncthreads();  // the waves' stages take the place of the links
        if (valid) store_canon<float>(a, f, a.vec[v], sd, cb, true, acc, (char *)s_dyn + w * kStageBytes<float>);
    }
    if (a.red.kind != RED_NONE && valid) wave_reduce_store_n(a.red, a.vec[v].pslot0, bm.lblk, rv);
    if (a.stamps) {
        __syncthreads();
        if (threadIdx.x == 0) a.stamps[2 * lb + 1] = (unsigned long long)wall_clock64();
    }
}

// Variants 9 and 10: pencil blocks.  The nw = block / 64 waves of a block
// take the same 64 positions of nw consecutive time slices of one vector
// (wave j: slice t0 + j; the set's slices hold a multiple of 64 sites and nw
// divides the time extent).  In the checkerboard index the time neighbours of
// output site cb are the input sites cb +- (sites per slice), at the same
// position: the input row at wave j's own sites is the forward time
// neighbour of wave j - 1 and the backward one of wave j + 1.  Each wave puts
// that row into LDS once; inside the block the time directions read it there,
// and only the outer slices fetch a time row from memory.  (The stand-alone
// hop fetches every input spinor about twice, and the second fetch is the
// time rows'.)  LDS holds per wave the row's raw chunks, [chunk][lane], and
// for FP16/BF16 its norms.  Every direction runs the per-site arithmetic of
// hop_site in its order, so the result equals the other variants' bit for bit.
template <int SP> struct PencilRow {
    using CH = typename SpinorFmt<SP>::chunk;
    static constexpr int NC = SpinorFmt<SP>::nchunk;
    static constexpr bool HALF = SP == P_F16 || SP == P_BF16;
    static constexpr int chunk_bytes = NC * 64 * (int)sizeof(CH);
    static constexpr int bytes = chunk_bytes + (HALF ? 64 * (int)sizeof(float) : 0);
};

// the time direction DIR of output site cb from the neighbour row in LDS
// (interior slices of the block: no wrap, no boundary sign)
template <int SP, int GP, int R, int DIR, bool DAG, bool NT>
__device__ __forceinline__ void pencil_t(const HopSite &hs, int parity, int cb, int ncb, const unsigned char *row,
                                         int lane, float acc[24])
{
    using P = PencilRow<SP>;
    constexpr int SG = (DIR > 0) == DAG ? +1 : -1;
    const typename P::CH *src = reinterpret_cast<const typename P::CH *>(row);
    cpx<float> h0[3], h1[3];
    float f;
    if constexpr (P::HALF) {
        uint32_t q[12];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const uint4 w = src[c * 64 + lane];
            q[4 * c] = w.x;
            q[4 * c + 1] = w.y;
            q[4 * c + 2] = w.z;
            q[4 * c + 3] = w.w;
        }
        const float nrm = reinterpret_cast<const float *>(row + P::chunk_bytes)[lane];
        project_half<SP, 3, SG>(q, h0, h1);
        f = nrm * hs.scale;
    } else {
        float v[24];
#pragma unroll
        for (int c = 0; c < 6; ++c) {
            const float4 w = src[c * 64 + lane];
            v[4 * c] = w.x;
            v[4 * c + 1] = w.y;
            v[4 * c + 2] = w.z;
            v[4 * c + 3] = w.w;
        }
        project<3, SG>(v, h0, h1);
        f = 1.f;
    }
    cpx<float> u[3][3];
    hop_link<GP, R, 3, DIR, NT>(hs, parity, cb, ncb, u);
    hop_accumulate<SP, 3, DIR, SG>(u, h0, h1, f, acc);
}

template <int SP, int GP, int R, bool DAG, int VAR, bool CANON>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(HopVar<SP, VAR>::waves)))
void k_hop_pencil(HopArgs a)
{
    static_assert(SP != P_F64, "pencil rows hold FP32 or half-precision spinors");
    using P = PencilRow<SP>;
    using CH = typename P::CH;
    constexpr int FENCE = HopVar<SP, VAR>::fence;
    constexpr bool NT = HopVar<SP, VAR>::nt;
    extern __shared__ uint4 s_pencil[];
    unsigned char *rows = reinterpret_cast<unsigned char *>(s_pencil);

    const int lb = xcd_remap(blockIdx.x, a.nblocks);
    const bool second = a.twin && (lb & 1);
    const HopIO f = second ? HopIO{1 - a.parity, a.in_b, a.in_norm_b, a.out_b, a.out_norm_b, a.X_b, a.Xn_b}
                           : HopIO{a.parity, a.in, a.in_norm, a.out, a.out_norm, a.epi.X, a.epi.Xn};
    const BlkMap bm = a.map[a.twin ? lb >> 1 : lb];
    if (a.active && !a.active[a.one ? 0 : bm.v]) return;  // uniform over the block
    const VecDesc vd = a.vec[a.one ? 0 : bm.v];
    const SysDesc sd = a.sys[a.one ? 0 : vd.sys];
    if (a.stamps && threadIdx.x == 0) a.stamps[2 * lb] = (unsigned long long)wall_clock64();
    const int lane = (int)threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int nw = (int)blockDim.x >> 6;
    const int slice = sd.Lxh * sd.L[1] * sd.L[2], nch = slice >> 6;
    const int pz = bm.lblk / nch;
    const int cb = (pz * nw + w) * slice + (bm.lblk - pz * nch) * 64 + lane;
    const HopSite hs = hop_input<SP>(a, f, vd, sd);

    // this wave's row: the input site at the thread's own index
    unsigned char *own = rows + w * P::bytes;
#pragma unroll
    for (int c = 0; c < P::NC; ++c)
        reinterpret_cast<CH *>(own)[c * 64 + lane] = ld_field<false>(row_elem<CH>(hs.in, c, hs.stride, cb));
    if constexpr (P::HALF)
        reinterpret_cast<float *>(own + P::chunk_bytes)[lane] = ld_field<false>(row_elem<float>(hs.in_norm, 0, 0, cb));

    float acc[24];
#pragma unroll
    for (int k = 0; k < 24; ++k) acc[k] = 0.f;
    const Site st = cb_coords(sd, cb, f.parity);
    hop_dir<SP, GP, R, 0, +1, DAG, NT>(sd, hs, f.parity, st, cb, acc);
    hop_dir<SP, GP, R, 0, -1, DAG, NT>(sd, hs, f.parity, st, cb, acc);
    if constexpr (FENCE <= 2) sched_fence(acc);
    hop_dir<SP, GP, R, 1, +1, DAG, NT>(sd, hs, f.parity, st, cb, acc);
    hop_dir<SP, GP, R, 1, -1, DAG, NT>(sd, hs, f.parity, st, cb, acc);
    sched_fence(acc);
    __syncthreads();  // every wave's row is in LDS
    hop_dir<SP, GP, R, 2, +1, DAG, NT>(sd, hs, f.parity, st, cb, acc);
    hop_dir<SP, GP, R, 2, -1, DAG, NT>(sd, hs, f.parity, st, cb, acc);
    if constexpr (FENCE <= 2) sched_fence(acc);
    if (w + 1 < nw)
        pencil_t<SP, GP, R, +1, DAG, NT>(hs, f.parity, cb, cb + slice, rows + (w + 1) * P::bytes, lane, acc);
    else
        hop_dir<SP, GP, R, 3, +1, DAG, NT>(sd, hs, f.parity, st, cb, acc);
    if (w > 0)
        pencil_t<SP, GP, R, -1, DAG, NT>(hs, f.parity, cb, cb - slice, rows + (w - 1) * P::bytes, lane, acc);
    else
        hop_dir<SP, GP, R, 3, -1, DAG, NT>(sd, hs, f.parity, st, cb, acc);
    sched_fence(acc);

    double rv[3] = {0.0, 0.0, 0.0};
    hop_epilogue<SP, false, CANON>(a, f, vd, sd, cb, acc, rv);
    if constexpr (CANON) {
        __syncthreads();  // the waves' stages take the place of the rows
        store_canon<float>(a, f, vd, sd, cb, true, acc, rows + w * kStageBytes<float>);
    }
    if (a.red.kind != RED_NONE) block_reduce_store_n(a.red, vd.pslot0, bm.lblk, rv);
    if (a.stamps) {
        __syncthreads();
        if (threadIdx.x == 0) a.stamps[2 * lb + 1] = (unsigned long long)wall_clock64();
    }
}

// Variant 11: the eight directions of 64 sites of one vector on the eight waves
// of a block.  Wave d loads its direction's link and neighbour spinor, projects
// and multiplies; the products meet in LDS, where each of the first waves adds a
// few reals of every site over the directions in the order of hop_site (so the
// result equals the other variants' bit for bit) and applies the epilogue to them.
// For small and ordinary lattices, where the hop is one round of latencies after
// another: a wave waits for one round of loads instead of four, eight times as
// many waves are under way, and the eight readers of a spinor ask for it at the
// same time.  Warm D-slash against the best per-site variant: 8^3x16 FP32 3.5 us
// instead of 6.6, 12x14x10x18 FP64 4.9 instead of 10.5, 16^3x32 FP32 6.7 instead
// of 8.8, 24^3x48 FP32 30.5 instead of 37; at 32^3x64 the products' way through
// LDS costs more than the loads it hides (FP16 64 us against 52).
template <int SP> struct SplitHop {
    using T = typename SpinorFmt<SP>::real;
    static constexpr bool half = SP == P_F16 || SP == P_BF16;
    static constexpr int rows = half ? 13 : 12;     // reals per direction and site in LDS (half precision: and its factor)
    static constexpr int per_wave = half ? 8 : 4;   // reals of a site that one wave finishes: whole chunk rows
    static constexpr int finishers = 24 / per_wave;
    static constexpr int buf = 8 * rows * 64;       // T's of the products
    static constexpr int waves = SP == P_F64 ? 4 : 8;  // per SIMD
};

// Output real k of direction mu with projector sign sg: the product real it comes
// from (0-5: U h0, 6-11: U h1) and whether it is subtracted; see reconstruct_add.
struct SplitSrc {
    int idx;
    bool neg;
};
constexpr SplitSrc split_src(int mu, int sg, int k)
{
    if (k < 12) return {k, false};
    const bool lower = k >= 18;  // spin 3
    const int q = (k - 12) % 6, c = 2 * (q / 2), ri = q & 1;
    switch (mu) {
    case 0: return {(lower ? 0 : 6) + c + 1 - ri, (sg > 0) == (ri == 1)};
    case 1: return {(lower ? 0 : 6) + c + ri, (sg > 0) == lower};
    case 2: return {(lower ? 6 : 0) + c + 1 - ri, ((sg > 0) == (ri == 1)) != lower};
    default: return {(lower ? 6 : 0) + c + ri, sg < 0};
    }
}

// reals w * per_wave ... of a packed FP32 or FP64 site, plain stores (the next
// launch reads them)
template <int SP>
__device__ __forceinline__ void split_store(void *base, int stride, int cb, int w, const typename SplitHop<SP>::T *o)
{
    if constexpr (SP == P_F64) {
        st_out<false>(row_elem<double2>(base, 2 * w, stride, cb), double2{o[0], o[1]});
        st_out<false>(row_elem<double2>(base, 2 * w + 1, stride, cb), double2{o[2], o[3]});
    } else {
        st_out<false>(row_elem<float4>(base, w, stride, cb), float4{o[0], o[1], o[2], o[3]});
    }
}

// U P v of direction MU, DIR for a neighbour's FP32 or FP64 spinor v
template <int SP, int MU, int DIR, bool DAG, class T>
__device__ __forceinline__ void split_multiply(const T v[24], bool flip, const cpx<T> u[3][3], T *out)
{
    constexpr int SG = (DIR > 0) == DAG ? +1 : -1;
    cpx<T> h0[3], h1[3], g[3];
    project<MU, SG>(v, h0, h1);
    if (flip) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            h0[c] = {-h0[c].re, -h0[c].im};
            h1[c] = {-h1[c].re, -h1[c].im};
        }
    }
    su3_mul<(DIR < 0), T>(u, h0, g);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        out[(2 * c) * 64] = g[c].re;
        out[(2 * c + 1) * 64] = g[c].im;
    }
    su3_mul<(DIR < 0), T>(u, h1, g);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        out[(6 + 2 * c) * 64] = g[c].re;
        out[(7 + 2 * c) * 64] = g[c].im;
    }
}

// Site `lex` of the canonical field `base`, rounded as packing it rounds: FP64 and
// FP32 the 24 reals; FP16/BF16 the packed words and the norm
template <int SP>
__device__ __forceinline__ void canon_site(const double *base, int lex, typename SplitHop<SP>::T v[24], uint32_t q[12],
                                           float *norm)
{
    const WL_G double *p = (const WL_G double *)base + (size_t)lex * 24;
#pragma unroll
    for (int k = 0; k < 12; ++k) {
        const nt_d2u w = *(const WL_G nt_d2u *)(p + 2 * k);
        v[2 * k] = (typename SplitHop<SP>::T)w.x;
        v[2 * k + 1] = (typename SplitHop<SP>::T)w.y;
    }
    if constexpr (SplitHop<SP>::half) quantize_site<SP>(v, q, norm);
}

// U P psi of direction MU, DIR at the lane's site into its column of `out`; DIRECT:
// psi is the vector of the canonical field that starts at `canon`
template <int SP, int GP, int R, int MU, int DIR, bool DAG, bool DIRECT = false, class T>
__device__ __forceinline__ void split_product(const SysDesc &sd, const HopSite &hs, int parity, const Site &st, int cb,
                                              T *out, const double *canon = nullptr)
{
    constexpr int SG = (DIR > 0) == DAG ? +1 : -1;
    bool flip;
    const int ncb = neighbour<MU, DIR>(sd, st, cb, flip);
    cpx<T> h0[3], h1[3], g[3], u[3][3];
    T f;
    if constexpr (DIRECT) {
        // the neighbour is the site of its pair with the x of its own parity
        T v[24];
        uint32_t q[12];
        float m;
        canon_site<SP>(canon, 2 * ncb + ((MU == 0 ? st.x + 1 : st.x) & 1), v, q, &m);
        hop_link<GP, R, MU, DIR, false>(hs, parity, cb, ncb, u);
        if constexpr (SplitHop<SP>::half) {
            project_half<SP, MU, SG>(q, h0, h1);
            f = (flip ? -m : m) * (T)hs.scale;
        } else {
            project<MU, SG>(v, h0, h1);
            if (flip) {
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    h0[c] = {-h0[c].re, -h0[c].im};
                    h1[c] = {-h1[c].re, -h1[c].im};
                }
            }
            f = 1;
        }
    } else {
        f = project_neighbour<SP, MU, SG>(hs, ncb, flip, h0, h1);
        hop_link<GP, R, MU, DIR, false>(hs, parity, cb, ncb, u);
    }
    su3_mul<(DIR < 0), T>(u, h0, g);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        out[(2 * c) * 64] = g[c].re;
        out[(2 * c + 1) * 64] = g[c].im;
    }
    su3_mul<(DIR < 0), T>(u, h1, g);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        out[(6 + 2 * c) * 64] = g[c].re;
        out[(7 + 2 * c) * 64] = g[c].im;
    }
    if constexpr (SplitHop<SP>::half) out[12 * 64] = f;
}

// reals W * per_wave ... of the hopping sum of the lane's site
template <int SP, bool DAG, int W, int D>
__device__ __forceinline__ void split_add(const typename SplitHop<SP>::T *b, typename SplitHop<SP>::T *acc)
{
    using S = SplitHop<SP>;
    using T = typename S::T;
    constexpr int mu = D >> 1, SG = ((D & 1) == 0) == DAG ? +1 : -1;
    const T *g = b + D * S::rows * 64;
    T f = 0;
    if constexpr (S::half) f = g[12 * 64];
#pragma unroll
    for (int i = 0; i < S::per_wave; ++i) {
        const SplitSrc e = split_src(mu, SG, W * S::per_wave + i);
        const T x = g[e.idx * 64];
        if constexpr (S::half)
            acc[i] = fmadd(x, e.neg ? -f : f, acc[i]);
        else
            acc[i] = e.neg ? acc[i] - x : acc[i] + x;
    }
}

template <int SP, bool DAG, int W>
__device__ __forceinline__ void split_sum(const typename SplitHop<SP>::T *b, typename SplitHop<SP>::T *acc)
{
#pragma unroll
    for (int i = 0; i < SplitHop<SP>::per_wave; ++i) acc[i] = 0;
    split_add<SP, DAG, W, 0>(b, acc);
    split_add<SP, DAG, W, 1>(b, acc);
    split_add<SP, DAG, W, 2>(b, acc);
    split_add<SP, DAG, W, 3>(b, acc);
    split_add<SP, DAG, W, 4>(b, acc);
    split_add<SP, DAG, W, 5>(b, acc);
    split_add<SP, DAG, W, 6>(b, acc);
    split_add<SP, DAG, W, 7>(b, acc);
}

// reals w * per_wave ... of a packed site before its norm is applied
template <int SP, bool NT>
__device__ __forceinline__ void split_load(const void *base, int stride, int cb, int w, typename SplitHop<SP>::T *x)
{
    if constexpr (SP == P_F64) {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const double2 v = ld_field<NT>(row_elem<double2>(base, 2 * w + c, stride, cb));
            x[2 * c] = v.x;
            x[2 * c + 1] = v.y;
        }
    } else if constexpr (SP == P_F32) {
        const float4 v = ld_field<NT>(row_elem<float4>(base, w, stride, cb));
        x[0] = v.x;
        x[1] = v.y;
        x[2] = v.z;
        x[3] = v.w;
    } else {
        const uint4 v = ld_field<NT>(row_elem<uint4>(base, w, stride, cb));
        const uint32_t q[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            x[2 * k] = half_part<SP, 0>(q[k]);
            x[2 * k + 1] = half_part<SP, 1>(q[k]);
        }
    }
}

// The 24 reals of a site as far as finishing wave W needs them for its rows of the
// clover term: the six complex numbers of the block (or, half precision, blocks)
// that its reals belong to, norm applied.
template <int SP, int W, class T>
__device__ __forceinline__ void split_load_blocks(const void *base, const float *norm, int stride, int cb, T x[24])
{
    constexpr int PW = SplitHop<SP>::per_wave;
    if constexpr (SP == P_F64 || SP == P_F32) {
        constexpr int b = W * PW / 12, per = 12 / PW;
#pragma unroll
        for (int c = 0; c < per; ++c) split_load<SP, false>(base, stride, cb, b * per + c, x + (b * per + c) * PW);
    } else {
        load_spinor<SP>(base, norm, stride, cb, x);
    }
}

// y = the rows W * per_wave ... of the packed clover term applied to x, in the
// order of clover_apply
template <int SP, int W, class T>
__device__ __forceinline__ void split_clover(const void *base, int stride, int cb, const T x[24], T *y)
{
    constexpr int PW = SplitHop<SP>::per_wave, CP = clover_prec<SP>();
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const int lo = W * PW > 12 * b ? W * PW : 12 * b, hi = W * PW + PW < 12 * b + 12 ? W * PW + PW : 12 * b + 12;
        if (lo >= hi) continue;
        T m[36];
        clover_block<CP>(base, stride, cb, b, m);
#pragma unroll
        for (int i = 0; i < 6; ++i) {
            const int k = 12 * b + 2 * i;
            if (k < lo || k >= hi) continue;
            T yr, yi;
            clover_row(m, x + 12 * b, i, yr, yi);
            y[k - W * PW] = yr;
            y[k - W * PW + 1] = yi;
        }
    }
}

#define WL_EACH_DIR(w, CALL)          \
    switch (w) {                      \
    case 0: CALL(0, +1); break;       \
    case 1: CALL(0, -1); break;       \
    case 2: CALL(1, +1); break;       \
    case 3: CALL(1, -1); break;       \
    case 4: CALL(2, +1); break;       \
    case 5: CALL(2, -1); break;       \
    case 6: CALL(3, +1); break;       \
    default: CALL(3, -1); break;      \
    }

#define WL_EACH_FINISHER(w, CALL)                                          \
    switch (w) {                                                           \
    case 0: CALL(0); break;                                                \
    case 1: CALL(1); break;                                                \
    case 2: CALL(2); break;                                                \
    case 3: if constexpr (!S::half) CALL(3 % S::finishers); break;         \
    case 4: if constexpr (!S::half) CALL(4 % S::finishers); break;         \
    default: if constexpr (!S::half) CALL(5 % S::finishers); break;        \
    }

template <int SP, int GP, int R, bool DAG, int EP>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(EP & EP_DIRECT ? 2 : EP & EP_CLOVER ? 4 : SplitHop<SP>::waves)))
void k_hop_split(HopArgs a)
{
    constexpr bool CLOV = (EP & 1) != 0, CANON = (EP & 2) != 0, DIRECT = (EP & EP_DIRECT) != 0;
    using S = SplitHop<SP>;
    using T = typename S::T;
    using CH = typename SpinorFmt<SP>::chunk;
    constexpr int PW = S::per_wave, CP = clover_prec<SP>();
    extern __shared__ uint4 s_split[];
    __shared__ float s_max[S::half ? S::finishers : 1][64];
    T *prod = reinterpret_cast<T *>(s_split);

    const int lb = xcd_remap(blockIdx.x, a.nblocks);
    const bool second = a.twin && (lb & 1);
    const HopIO f = second ? HopIO{1 - a.parity, a.in_b, a.in_norm_b, a.out_b, a.out_norm_b, a.X_b, a.Xn_b}
                           : HopIO{a.parity, a.in, a.in_norm, a.out, a.out_norm, a.epi.X, a.epi.Xn};
    const BlkMap bm = a.map[a.twin ? lb >> 1 : lb];
    if (a.active && !a.active[a.one ? 0 : bm.v]) return;
    const VecDesc vd = a.vec[a.one ? 0 : bm.v];
    const SysDesc sd = a.sys[a.one ? 0 : vd.sys];
    if (a.stamps && threadIdx.x == 0) a.stamps[2 * lb] = (unsigned long long)wall_clock64();
    const int lane = (int)threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int cb = bm.lblk * 64 + lane;
    const bool live = cb < sd.Vh;
    const int ccb = live ? cb : sd.Vh - 1;  // lanes past the end repeat the last site and store nothing
    const Site st = cb_coords(sd, ccb, f.parity);
    const HopSite hs = hop_input<SP>(a, f, vd, sd);
    const double *canon = DIRECT ? a.canon_in + (size_t)vd.rhs * (size_t)sd.Vh * 48 : nullptr;
    {
        T *out = prod + w * S::rows * 64 + lane;
#define WL_PROD(MU, DIR) split_product<SP, GP, R, MU, DIR, DAG, DIRECT>(sd, hs, f.parity, st, ccb, out, canon)
        WL_EACH_DIR(w, WL_PROD)
#undef WL_PROD
    }
    const double *cf = a.epi.coef + vd.sys * 5;
    const int nx = a.epi.nx;
    const size_t voff = (size_t)vd.site_off * SpinorFmt<SP>::nchunk;
    auto load = [&](int j, T *x, T &n) {
        const CH *xb = (const CH *)f.X[j] + voff;
        n = 1;
        if (a.stream) {
            split_load<SP, true>(xb, sd.stride, ccb, w, x);
            if constexpr (S::half) n = ld_field<true>(row_elem<float>(f.Xn[j] + vd.site_off, 0, 0, ccb));
        } else {
            split_load<SP, false>(xb, sd.stride, ccb, w, x);
            if constexpr (S::half) n = ld_field<false>(row_elem<float>(f.Xn[j] + vd.site_off, 0, 0, ccb));
        }
    };
    // the first two epilogue operands are on their way while the products meet
    T x0[PW], x1[PW], n0 = 1, n1 = 1;
    // (DIRECT: X0 is the input at the output site, and there is no other)
    T xc[24];
    if (w < S::finishers) {
        if constexpr (DIRECT) {
            if (nx >= 1) {
                uint32_t q[12];
                float m = 1.f;
                canon_site<SP>(canon, 2 * ccb + (st.x & 1), xc, q, &m);
                n0 = (T)m;
                if constexpr (S::half) {
#pragma unroll
                    for (int k = 0; k < 12; ++k) {
                        xc[2 * k] = half_part<SP, 0>(q[k]);
                        xc[2 * k + 1] = half_part<SP, 1>(q[k]);
                    }
                }
#define WL_OWN(W)                                     \
    _Pragma("unroll") for (int i = 0; i < PW; ++i) x0[i] = xc[W * PW + i]
                WL_EACH_FINISHER(w, WL_OWN)
#undef WL_OWN
            }
        } else {
            if (nx >= 1) load(0, x0, n0);
            if (nx >= 2) load(1, x1, n1);
        }
    }
    __syncthreads();
    double rv[3] = {0.0, 0.0, 0.0};
    T o[PW];
    if (w < S::finishers) {
        const T *q = prod + lane;
#define WL_SUM(W) split_sum<SP, DAG, W>(q, o)
        WL_EACH_FINISHER(w, WL_SUM)
#undef WL_SUM
        if constexpr (!S::half) {
            const T c = (T)cf[4];
#pragma unroll
            for (int i = 0; i < PW; ++i) o[i] *= c;
        }
        bool plain = nx >= 1;
        if constexpr (CLOV) {
            if (nx >= 1 && (a.epi.clov & EPI_CLOV_X0) && sd.clov) {
                plain = false;
                const void *cl = clover_parity<CP>(sd.clov, f.parity, sd.stride);
                const float *xn = f.Xn[0] ? f.Xn[0] + vd.site_off : nullptr;
                T xs[24], y[PW];
                if constexpr (DIRECT) {
#pragma unroll
                    for (int k = 0; k < 24; ++k) xs[k] = S::half ? xc[k] * n0 : xc[k];
                }
#define WL_CLOV(W)                                                                           \
    {                                                                                        \
        if constexpr (!DIRECT)                                                               \
            split_load_blocks<SP, W>((const CH *)f.X[0] + voff, xn, sd.stride, ccb, xs);     \
        split_clover<SP, W>(cl, sd.stride, ccb, xs, y);                                      \
    }
                WL_EACH_FINISHER(w, WL_CLOV)
#undef WL_CLOV
                const T s0 = (T)cf[0];
#pragma unroll
                for (int i = 0; i < PW; ++i) o[i] = fmadd(y[i], s0, o[i]);
            }
        }
        if (plain) {
            const T s0 = (T)cf[0] * n0;
#pragma unroll
            for (int i = 0; i < PW; ++i) o[i] = fmadd(x0[i], s0, o[i]);
        }
        if (a.epi.g5) {
#pragma unroll
            for (int i = 0; i < PW; ++i)
                if (w * PW + i >= 12) o[i] = -o[i];
        }
    }
    if constexpr (CLOV) {
        if ((a.epi.clov & EPI_CLOV_INV) && sd.clovinv) {  // uniform over the block
            // the rows of A^-1 need the whole block of the site: exchanged through LDS
            T *site = prod + S::buf;
            if (w < S::finishers) {
#pragma unroll
                for (int i = 0; i < PW; ++i) site[(w * PW + i) * 64 + lane] = o[i];
            }
            __syncthreads();
            if (w < S::finishers) {
                T xs[24];
#pragma unroll
                for (int k = 0; k < 24; ++k) xs[k] = site[k * 64 + lane];
                const void *cl = clover_parity<CP>(sd.clovinv, f.parity, sd.stride);
#define WL_CLOV_INV(W) split_clover<SP, W>(cl, sd.stride, ccb, xs, o)
                WL_EACH_FINISHER(w, WL_CLOV_INV)
#undef WL_CLOV_INV
            }
            if constexpr (CANON) __syncthreads();  // the stage of the canonical store lies there too
        }
    }
    if (w < S::finishers) {
        if (nx >= 2) {
            const T s1 = (T)cf[1] * n1;
#pragma unroll
            for (int i = 0; i < PW; ++i) o[i] = fmadd(x1[i], s1, o[i]);
        }
        for (int j = 2; j < nx; ++j) {
            T x[PW], n;
            load(j, x, n);
            const T sj = (T)cf[j] * n;
#pragma unroll
            for (int i = 0; i < PW; ++i) o[i] = fmadd(x[i], sj, o[i]);
        }
        if (a.red.kind != RED_NONE && live) {
            T s = 0;
#pragma unroll
            for (int i = 0; i < PW; ++i) s = fmadd(o[i], o[i], s);
            if (a.red.mode == RM_NORM) {
                rv[0] = (double)s;
            } else {
                // <X1, o> or <o, X0>; linear in x: its site norm scales the sums
                const bool dot1 = a.red.mode == RM_DOT_X1;
                T cr = 0, ci = 0;
#pragma unroll
                for (int i = 0; i < PW; i += 2) {
                    const T xr = dot1 ? x1[i] : x0[i], xi = dot1 ? x1[i + 1] : x0[i + 1];
                    cr = fmadd(xr, o[i], cr);
                    cr = fmadd(xi, o[i + 1], cr);
                    ci = fmadd(xr, o[i + 1], ci);
                    ci = fmadd(-xi, o[i], ci);
                }
                const double nx1 = (double)(dot1 ? n1 : n0);
                rv[0] = (double)cr * nx1;
                rv[1] = (dot1 ? (double)ci : -(double)ci) * nx1;
                rv[2] = (double)s;
            }
        }
    }
    if constexpr (S::half) {
        // the site's norm is the largest of its 24 reals
        float m = 0.f;
        if (w < S::finishers) {
#pragma unroll
            for (int i = 0; i < PW; ++i) m = fmaxf(m, fabsf(o[i]));
            s_max[w][lane] = m;
        }
        __syncthreads();
        if (w < S::finishers) {
            m = fmaxf(fmaxf(s_max[0][lane], s_max[1][lane]), s_max[2][lane]);
            const float inv = m > 0.f ? 1.0f / m : 0.f;
            uint32_t qw[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) qw[k] = pack2<SP>(o[2 * k] * inv, o[2 * k + 1] * inv);
            if constexpr (CANON) {
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    o[2 * k] = lo16_to_float<SP>(qw[k]) * m;
                    o[2 * k + 1] = hi16_to_float<SP>(qw[k]) * m;
                }
            } else if (live) {
                st_out<true>(row_elem<uint4>((CH *)f.out + voff, w, sd.stride, cb), uint4{qw[0], qw[1], qw[2], qw[3]});
                if (w == 0) st_out<true>(row_elem<float>(f.out_norm + vd.site_off, 0, 0, cb), m);
            }
        }
    } else if constexpr (!CANON) {
        if (w < S::finishers && live) {
            void *out = (CH *)f.out + voff;
            if constexpr (SP == P_F64) {
                if (a.lo) {  // FP32 (the host offers this variant no half-precision one)
                    st_out<false>(row_elem<float4>((float4 *)a.lo + (size_t)vd.site_off * 6, w, sd.stride, cb),
                                  float4{(float)o[0], (float)o[1], (float)o[2], (float)o[3]});
                } else {
                    st_out<true>(row_elem<double2>(out, 2 * w, sd.stride, cb), double2{o[0], o[1]});
                    st_out<true>(row_elem<double2>(out, 2 * w + 1, sd.stride, cb), double2{o[2], o[3]});
                }
            } else {
                st_out<true>(row_elem<float4>(out, w, sd.stride, cb), float4{o[0], o[1], o[2], o[3]});
            }
        }
    }
    if constexpr (CANON) {
        // the block's 64 pairs in whole lines (see store_canon), staged behind the products
        T *site = prod + S::buf;
        const unsigned long long slots = __ballot(st.x & 1);  // the same in every wave
        if (w < S::finishers) {
#pragma unroll
            for (int i = 0; i < PW; ++i) site[lane * kStageRow<T> + w * PW + i] = o[i];
        }
        __syncthreads();
        const int ns = min(64, sd.Vh - bm.lblk * 64);
        double *base = a.canon + ((size_t)vd.rhs * (size_t)sd.Vh + (size_t)bm.lblk * 64) * 48;
        if (a.canon_zero) {
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                const int e = i * 512 + (int)threadIdx.x, j = e / 24, r = e % 24;
                const int k = r < 12 ? r : r - 12;
                const bool mine = (int)((slots >> j) & 1) == (r >= 12);
                const T *p = site + j * kStageRow<T> + 2 * k;
                if (j < ns) st_canon(base + 2 * e, mine ? (double)p[0] : 0.0, mine ? (double)p[1] : 0.0);
            }
        } else {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int e = i * 512 + (int)threadIdx.x, j = e / 12, k = e % 12;
                if (j < ns) {
                    const T *p = site + j * kStageRow<T> + 2 * k;
                    st_canon(base + 48 * j + 24 * (int)((slots >> j) & 1) + 2 * k, (double)p[0], (double)p[1]);
                }
            }
        }
    }
    if (a.red.kind != RED_NONE) block_reduce_store_n(a.red, vd.pslot0, bm.lblk, rv);
    if (a.stamps) {
        __syncthreads();
        if (threadIdx.x == 0) a.stamps[2 * lb + 1] = (unsigned long long)wall_clock64();
    }
}

// The four launches of a CGNR iteration of a small set (FP32 and FP64, Wilson;
// steps of Cg::iterations), on the blocks of variant 11.  A small iteration lasts
// as long as its launches: the two update kernels and the two finishing launches
// between the hops took as long as the hops.  Here
//   HI_P, HI_R  the input is in + z in2 (z = beta or -alpha, finished here from
//               the previous launch's partials), formed at every neighbour;
//   HI_Q, HI_S  that field is formed again at the output sites and stored, with
//               x, as the epilogue's X0, and the hop's norm (HI_S: and |r|^2) goes
//               to the partials.
// CGNR to 1e-10: 8^3x16 FP32 2070 -> 1790 us, 4^3x8 FP32 1850 -> 1590.
template <int SP, int GP, int R, bool DAG, bool COMB>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(SP == P_F64 ? 2 : 4)))
void k_hop_iter(HopArgs a)
{
    using S = SplitHop<SP>;
    using T = typename S::T;
    using CH = typename SpinorFmt<SP>::chunk;
    static_assert(!S::half, "half-precision fields round when they are stored");
    constexpr int PW = S::per_wave;
    extern __shared__ uint4 s_split[];
    T *prod = reinterpret_cast<T *>(s_split);

    const int lb = xcd_remap(blockIdx.x, a.nblocks);
    const BlkMap bm = a.map[lb];
    const int vi = a.one ? 0 : bm.v;
    if (a.active && !a.active[vi]) return;
    const VecDesc vd = a.vec[vi];
    const SysDesc sd = a.sys[a.one ? 0 : vd.sys];
    const int lane = (int)threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int cb = bm.lblk * 64 + lane;
    const bool live = cb < sd.Vh;
    const int ccb = live ? cb : sd.Vh - 1;
    const Site st = cb_coords(sd, ccb, a.parity);
    const HopIO f{a.parity, a.in, nullptr, a.out, nullptr, a.epi.X, a.epi.Xn};
    const HopSite hs = hop_input<SP>(a, f, vd, sd);
    const size_t voff = (size_t)vd.site_off * SpinorFmt<SP>::nchunk;
    const CH *in2 = (const CH *)a.in2 + voff;
    T *pout = prod + w * S::rows * 64 + lane;
    if constexpr (COMB) {
        // every load of the wave's direction goes out, then the scalar is finished
        T v[24], v2[24];
        cpx<T> u[3][3];
        bool flip;
        int ncb;
#define WL_LOAD(MU, DIR)                                    \
    {                                                       \
        ncb = neighbour<MU, DIR>(sd, st, ccb, flip);        \
        load_spinor<SP>(hs.in, nullptr, sd.stride, ncb, v); \
        load_spinor<SP>(in2, nullptr, sd.stride, ncb, v2);  \
        hop_link<GP, R, MU, DIR, false>(hs, a.parity, ccb, ncb, u); \
    }
        WL_EACH_DIR(w, WL_LOAD)
#undef WL_LOAD
        // HI_P (no adjoint) beta, HI_R (adjoint) -alpha
        const T z = DAG ? (T)(-fold_alpha(a.fold, vi, bm.lblk)) : (T)fold_beta(a.fold, vi, bm.lblk);
#pragma unroll
        for (int k = 0; k < 24; ++k) v[k] = fmadd(z, v2[k], v[k]);
#define WL_PROD(MU, DIR) split_multiply<SP, MU, DIR, DAG>(v, flip, u, pout)
        WL_EACH_DIR(w, WL_PROD)
#undef WL_PROD
    } else {
#define WL_PROD(MU, DIR) split_product<SP, GP, R, MU, DIR, DAG>(sd, hs, a.parity, st, ccb, pout)
        WL_EACH_DIR(w, WL_PROD)
#undef WL_PROD
    }
    // own-site fields: HI_Q s, p, x; HI_S r, q
    T x0[PW], x1[PW], x2[PW];
    double z1 = 0.0, z2 = 0.0;
    if constexpr (!COMB) {
        if (w < S::finishers) {
            split_load<SP, false>((const CH *)a.epi.X[0] + voff, sd.stride, ccb, w, x0);
            split_load<SP, false>((const CH *)a.epi.X[1] + voff, sd.stride, ccb, w, x1);
            if constexpr (!DAG) split_load<SP, false>((const CH *)a.epi.X[2] + voff, sd.stride, ccb, w, x2);
        }
        z2 = a.fold.sc[(size_t)SC_ALPHA * a.nvec + vi];
        if constexpr (!DAG) z1 = a.fold.sc[(size_t)SC_BETA * a.nvec + vi];
    }
    __syncthreads();
    double rv = 0.0, rr = 0.0;
    if (w < S::finishers) {
        T o[PW], n[PW];
        const T *q = prod + lane;
#define WL_SUM(W) split_sum<SP, DAG, W>(q, o)
        WL_EACH_FINISHER(w, WL_SUM)
#undef WL_SUM
        const T c = (T)a.epi.coef[vd.sys * 5 + 4];
#pragma unroll
        for (int i = 0; i < PW; ++i) o[i] *= c;
        if constexpr (!COMB) {
            if constexpr (DAG) {
                const T al = (T)(-z2);
#pragma unroll
                for (int i = 0; i < PW; ++i) n[i] = fmadd(al, x1[i], x0[i]);  // r - alpha q
            } else {
                const T be = (T)z1, al = (T)z2;
#pragma unroll
                for (int i = 0; i < PW; ++i) {
                    x2[i] = fmadd(al, x1[i], x2[i]);  // x + alpha p
                    n[i] = fmadd(be, x1[i], x0[i]);   // s + beta p
                }
                if (live) split_store<SP>((CH *)a.out3 + voff, sd.stride, cb, w, x2);
            }
            if (live) split_store<SP>((CH *)a.out2 + voff, sd.stride, cb, w, n);
            const T c0 = (T)a.epi.coef[vd.sys * 5];
#pragma unroll
            for (int i = 0; i < PW; ++i) o[i] = fmadd(n[i], c0, o[i]);
            if (live) {
                T s1 = 0, s2 = 0;
#pragma unroll
                for (int i = 0; i < PW; ++i) {
                    s1 = fmadd(o[i], o[i], s1);
                    s2 = fmadd(n[i], n[i], s2);
                }
                rv = (double)s1;
                rr = (double)s2;
            }
        }
        if (live) split_store<SP>((CH *)f.out + voff, sd.stride, cb, w, o);
    }
    if constexpr (!COMB) {
        block_reduce_store(a.red, vd.pslot0, bm.lblk, rv);
        if constexpr (DAG) {
            const double bs = block_sum(rr);
            if (threadIdx.x == 0) a.partials2[vd.pslot0 + bm.lblk] = bs;
        }
    }
}

// With events, the dispatch itself records them at the kernel's start and end
// (the kernel-timing form of the launch), so the measured interval is the
// kernel alone.
template <class K>
static void dispatch(K kernel, const HopArgs &a, int block, hipStream_t s, hipEvent_t e0, hipEvent_t e1,
                     unsigned lds = 0)
{
    if (e0)
        hipExtLaunchKernelGGL(kernel, dim3(a.nblocks), dim3(block), lds, s, e0, e1, 0, a);
    else
        hipLaunchKernelGGL(kernel, dim3(a.nblocks), dim3(block), lds, s, a);
}

template <int SP, int GP, int R, int VAR, int EP>
static hipError_t launch_hop_ep(bool dag, const HopArgs &a, int block, hipStream_t s, hipEvent_t e0, hipEvent_t e1)
{
    const unsigned lds = EP >= EP_CANON ? (unsigned)(block / 64) * kStageBytes<typename SpinorFmt<SP>::real> : 0;
    if (dag)
        dispatch(k_hop<SP, GP, R, true, VAR, EP>, a, block, s, e0, e1, lds);
    else
        dispatch(k_hop<SP, GP, R, false, VAR, EP>, a, block, s, e0, e1, lds);
    return hipGetLastError();
}

template <int SP, int GP, int R, int VAR>
static hipError_t launch_hop_v(bool dag, bool clov, const HopArgs &a, int block, hipStream_t s, hipEvent_t e0,
                               hipEvent_t e1)
{
    // the clover epilogue is a separate instantiation: it needs registers the Wilson
    // kernels do not, more than the one-direction variants 1 and 2 leave
    if (clov) {
        if constexpr (VAR == 1 || VAR == 2) return hipErrorInvalidValue;
        else
            return a.canon ? launch_hop_ep<SP, GP, R, VAR, EP_CLOVER_CANON>(dag, a, block, s, e0, e1)
                           : launch_hop_ep<SP, GP, R, VAR, EP_CLOVER>(dag, a, block, s, e0, e1);
    }
    return a.canon ? launch_hop_ep<SP, GP, R, VAR, EP_CANON>(dag, a, block, s, e0, e1)
                   : launch_hop_ep<SP, GP, R, VAR, EP_WILSON>(dag, a, block, s, e0, e1);
}

template <int SP, int GP, int R, bool CANON>
static hipError_t launch_hop_lds(bool dag, const HopArgs &a, int block, hipStream_t s, hipEvent_t e0, hipEvent_t e1)
{
    const unsigned lds = std::max(kLdsLinkBytes, CANON ? block / 64 * kStageBytes<float> : 0);
    if (dag)
        dispatch(k_hop_lds<SP, GP, R, true, CANON>, a, block, s, e0, e1, lds);
    else
        dispatch(k_hop_lds<SP, GP, R, false, CANON>, a, block, s, e0, e1, lds);
    return hipGetLastError();
}

template <int SP, int GP, int R, int VAR, bool CANON>
static hipError_t launch_hop_pencil(bool dag, const HopArgs &a, int block, hipStream_t s, hipEvent_t e0, hipEvent_t e1)
{
    const unsigned lds = (unsigned)(block / 64) * std::max(PencilRow<SP>::bytes, CANON ? kStageBytes<float> : 0);
    if (dag)
        dispatch(k_hop_pencil<SP, GP, R, true, VAR, CANON>, a, block, s, e0, e1, lds);
    else
        dispatch(k_hop_pencil<SP, GP, R, false, VAR, CANON>, a, block, s, e0, e1, lds);
    return hipGetLastError();
}

template <int SP, int GP, int R, int EP>
static hipError_t launch_hop_split(bool dag, const HopArgs &a, hipStream_t s, hipEvent_t e0, hipEvent_t e1)
{
    using S = SplitHop<SP>;
    const unsigned lds = (unsigned)(S::buf + (EP != EP_WILSON ? 64 * kStageRow<typename S::T> : 0)) * (unsigned)sizeof(typename S::T);
    if (dag)
        dispatch(k_hop_split<SP, GP, R, true, EP>, a, 512, s, e0, e1, lds);
    else
        dispatch(k_hop_split<SP, GP, R, false, EP>, a, 512, s, e0, e1, lds);
    return hipGetLastError();
}

template <int SP, int GP, int R>
hipError_t launch_hop_t(int var, bool dag, bool clov, const HopArgs &a, int block, hipStream_t s,
                               hipEvent_t e0, hipEvent_t e1)
{
    if (a.canon_in && var != 11) return hipErrorInvalidValue;
    if (a.lo && (SP != P_F64 || a.canon)) return hipErrorInvalidValue;
    switch (var) {
    case 0: return launch_hop_v<SP, GP, R, 0>(dag, clov, a, block, s, e0, e1);
    case 1: return launch_hop_v<SP, GP, R, 1>(dag, clov, a, block, s, e0, e1);
    case 2: return launch_hop_v<SP, GP, R, 2>(dag, clov, a, block, s, e0, e1);
    case 3: return launch_hop_v<SP, GP, R, 3>(dag, clov, a, block, s, e0, e1);
    case 4:
        if constexpr (SplitHop<SP>::half) return launch_hop_v<SP, GP, R, 4>(dag, clov, a, block, s, e0, e1);
        return hipErrorInvalidValue;
    case 5:
        if constexpr (SplitHop<SP>::half) return launch_hop_v<SP, GP, R, 5>(dag, clov, a, block, s, e0, e1);
        return hipErrorInvalidValue;
    case 6: return launch_hop_v<SP, GP, R, 6>(dag, clov, a, block, s, e0, e1);
    case 7:
        if constexpr (SP != P_F64) return launch_hop_v<SP, GP, R, 7>(dag, clov, a, block, s, e0, e1);
        return hipErrorInvalidValue;
    case 8:
        if constexpr (SP != P_F64) {
            if (clov || block % 64 != 0 || block > 1024) return hipErrorInvalidValue;
            return a.canon ? launch_hop_lds<SP, GP, R, true>(dag, a, block, s, e0, e1)
                           : launch_hop_lds<SP, GP, R, false>(dag, a, block, s, e0, e1);
        }
        return hipErrorInvalidValue;
    case 11:
        if (block != 64) return hipErrorInvalidValue;  // 64 sites on 512 threads
        if (a.canon_in && (!a.canon || a.epi.nx > 1)) return hipErrorInvalidValue;
        if (a.lo && a.lo_prec != P_F32) return hipErrorInvalidValue;
        if (a.canon_in)
            return clov ? launch_hop_split<SP, GP, R, EP_CLOVER_CANON | EP_DIRECT>(dag, a, s, e0, e1)
                        : launch_hop_split<SP, GP, R, EP_CANON | EP_DIRECT>(dag, a, s, e0, e1);
        if (clov)
            return a.canon ? launch_hop_split<SP, GP, R, EP_CLOVER_CANON>(dag, a, s, e0, e1)
                           : launch_hop_split<SP, GP, R, EP_CLOVER>(dag, a, s, e0, e1);
        return a.canon ? launch_hop_split<SP, GP, R, EP_CANON>(dag, a, s, e0, e1)
                       : launch_hop_split<SP, GP, R, EP_WILSON>(dag, a, s, e0, e1);
    case 9:
    case 10:
        if constexpr (SP != P_F64) {
            // 2 to 8 slices per block, one vector per block
            if (clov || block % 64 != 0 || block < 128 || block > 512) return hipErrorInvalidValue;
            if (var == 9)
                return a.canon ? launch_hop_pencil<SP, GP, R, 9, true>(dag, a, block, s, e0, e1)
                               : launch_hop_pencil<SP, GP, R, 9, false>(dag, a, block, s, e0, e1);
            return a.canon ? launch_hop_pencil<SP, GP, R, 10, true>(dag, a, block, s, e0, e1)
                           : launch_hop_pencil<SP, GP, R, 10, false>(dag, a, block, s, e0, e1);
        }
        return hipErrorInvalidValue;
    }
    return hipErrorInvalidValue;
}

// One launch of the CGNR iteration of small sets
template <int SP, int GP, int R>
hipError_t launch_hop_iter_t(int step, const HopArgs &a, hipStream_t s)
{
    if constexpr (SP == P_F64 || SP == P_F32) {
        const unsigned lds = (unsigned)SplitHop<SP>::buf * (unsigned)sizeof(typename SplitHop<SP>::T);
        switch (step) {
        case HI_P: dispatch(k_hop_iter<SP, GP, R, false, true>, a, 512, s, nullptr, nullptr, lds); break;
        case HI_Q: dispatch(k_hop_iter<SP, GP, R, false, false>, a, 512, s, nullptr, nullptr, lds); break;
        case HI_R: dispatch(k_hop_iter<SP, GP, R, true, true>, a, 512, s, nullptr, nullptr, lds); break;
        case HI_S: dispatch(k_hop_iter<SP, GP, R, true, false>, a, 512, s, nullptr, nullptr, lds); break;
        default: return hipErrorInvalidValue;
        }
        return hipGetLastError();
    }
    return hipErrorInvalidValue;
}

// The kernels of one storage format are compiled in a source of their own (hop_*.hip,
// which define WL_HOP_FORMAT and include this file), so that the formats build in
// parallel; this file by itself compiles the dispatch over them.
#ifdef WL_HOP_FORMAT
template hipError_t launch_hop_t<WL_HOP_FORMAT>(int var, bool dag, bool clov, const HopArgs &a, int block,
                                                hipStream_t s, hipEvent_t e0, hipEvent_t e1);
template hipError_t launch_hop_iter_t<WL_HOP_FORMAT>(int step, const HopArgs &a, hipStream_t s);
#else
#define WL_HOP_EXTERN(...)                                                                                          \
    extern template hipError_t launch_hop_t<__VA_ARGS__>(int var, bool dag, bool clov, const HopArgs &a, int block, \
                                                         hipStream_t s, hipEvent_t e0, hipEvent_t e1);              \
    extern template hipError_t launch_hop_iter_t<__VA_ARGS__>(int step, const HopArgs &a, hipStream_t s)
WL_HOP_EXTERN(P_F64, P_F64, 18);
WL_HOP_EXTERN(P_F64, P_F64, 12);
WL_HOP_EXTERN(P_F32, P_F32, 18);
WL_HOP_EXTERN(P_F32, P_F32, 12);
WL_HOP_EXTERN(P_F16, P_F16, 12);
WL_HOP_EXTERN(P_BF16, P_BF16, 12);
#undef WL_HOP_EXTERN

// 4 and 5 are for half precision; FP64 has no variants 8-10, which stage FP32 or
// half-precision data in LDS, and no 7: its two FP64 accumulators fit only at 2 waves
// per SIMD (12-RHS recon-12 D-slash 700 us against 672 for variants 3 and 6)
bool hop_has_variant(int prec, int var)
{
    if (var == 4 || var == 5) return prec == P_F16 || prec == P_BF16;
    return var >= 0 && var < kHopVariants && !(prec == P_F64 && var >= 7 && var <= 10);
}
int hop_variants() { return kHopVariants; }

hipError_t launch_hop(int prec, int recon, bool dag, bool clov, int var, const HopArgs &a, int block, hipStream_t s,
                      hipEvent_t e0, hipEvent_t e1)
{
    if (prec == P_F64 && recon == 18) return launch_hop_t<P_F64, P_F64, 18>(var, dag, clov, a, block, s, e0, e1);
    if (prec == P_F64 && recon == 12) return launch_hop_t<P_F64, P_F64, 12>(var, dag, clov, a, block, s, e0, e1);
    if (prec == P_F32 && recon == 18) return launch_hop_t<P_F32, P_F32, 18>(var, dag, clov, a, block, s, e0, e1);
    if (prec == P_F32 && recon == 12) return launch_hop_t<P_F32, P_F32, 12>(var, dag, clov, a, block, s, e0, e1);
    if (prec == P_F16 && recon == 12) return launch_hop_t<P_F16, P_F16, 12>(var, dag, clov, a, block, s, e0, e1);
    if (prec == P_BF16 && recon == 12) return launch_hop_t<P_BF16, P_BF16, 12>(var, dag, clov, a, block, s, e0, e1);
    return hipErrorInvalidValue;
}

hipError_t launch_hop_iter(int prec, int recon, int step, const HopArgs &a, hipStream_t s)
{
    if (prec == P_F64 && recon == 18) return launch_hop_iter_t<P_F64, P_F64, 18>(step, a, s);
    if (prec == P_F64 && recon == 12) return launch_hop_iter_t<P_F64, P_F64, 12>(step, a, s);
    if (prec == P_F32 && recon == 18) return launch_hop_iter_t<P_F32, P_F32, 18>(step, a, s);
    if (prec == P_F32 && recon == 12) return launch_hop_iter_t<P_F32, P_F32, 12>(step, a, s);
    return hipErrorInvalidValue;
}
#endif

}  // namespace wl
