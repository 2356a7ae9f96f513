// wl_eo.hip -- even-odd (red-black) decomposition of the Wilson operator.
//
// With sites coloured by the parity of x + y + z + t, the hopping term only
// couples opposite parities, so D = 1 - kappa H reads, in (even, odd) blocks,
//   D = [[1, -kappa H_eo], [-kappa H_oe, 1]],
// and D x = b is equivalent to the Schur system on the even sites
//   M x_e = b_e + kappa H_eo b_o,   M = 1 - kappa^2 H_eo H_oe,
// followed by x_o = b_o + kappa H_oe x_e.  (The paper leaves
// preconditioning out, Sec. II-C; this is the standard first step, with the
// same solution.)
//
// Half fields hold the sites of one parity in the packed spinor format with
// V/2 sites: the site x + Lx (y + Ly (z + Lz t)) of parity p sits at half
// index (x + Lx (y + ...)) / 2.  Every extent must be even (a hop that wraps
// around an odd extent would keep the parity).  Links stay in the full
// packed layout.
#include <type_traits>

#include "wl_stencil_dev.h"

namespace wl {

// Copy whole packed sites between the full layout and the two half layouts
// (raw 16-byte chunks and, for 16-bit formats, the scale: bit-exact).
template <int P, bool SPLIT>
__global__ void eo_copy_kernel(uint32_t V, int nrhs, const void *__restrict__ full_in, void *__restrict__ full_out,
                               void *__restrict__ even, void *__restrict__ odd, FastDiv fx, FastDiv fy, FastDiv fz,
                               int Lx, int Ly, int Lz)
{
    const uint32_t s = blockIdx.x * blockDim.x + threadIdx.x;
    const int r = blockIdx.y;
    if (s >= V)
        return;
    const uint32_t q1 = fdiv(s, fx);
    const int x = (int)(s - q1 * (uint32_t)Lx);
    const uint32_t q2 = fdiv(q1, fy);
    const int y = (int)(q1 - q2 * (uint32_t)Ly);
    const uint32_t q3 = fdiv(q2, fz);
    const int z = (int)(q2 - q3 * (uint32_t)Lz);
    const int t = (int)q3;
    const int par = (x + y + z + t) & 1;
    const uint32_t Vh = V / 2, i = s >> 1;
    constexpr int NCH = Traits<P>::NCH;
    const uint4 *src;
    uint4 *dst;
    uint32_t sv, dv, si, di;
    char *half = reinterpret_cast<char *>(par ? odd : even);
    if constexpr (SPLIT) {
        src = reinterpret_cast<const uint4 *>(full_in);
        dst = reinterpret_cast<uint4 *>(half);
        sv = V;
        dv = Vh;
        si = s;
        di = i;
    } else {
        src = reinterpret_cast<const uint4 *>(half);
        dst = reinterpret_cast<uint4 *>(full_out);
        sv = Vh;
        dv = V;
        si = i;
        di = s;
    }
#pragma unroll
    for (int k = 0; k < NCH; ++k)
        dst[((size_t)r * NCH + k) * dv + di] = src[((size_t)r * NCH + k) * sv + si];
    if constexpr (Traits<P>::SCALED) {
        const float *ss = reinterpret_cast<const float *>(reinterpret_cast<const char *>(src) + (size_t)nrhs * NCH * sv * 16);
        float *ds = reinterpret_cast<float *>(reinterpret_cast<char *>(dst) + (size_t)nrhs * NCH * dv * 16);
        ds[(size_t)r * dv + di] = ss[(size_t)r * sv + si];
    }
}

hipError_t launch_eo_copy(int prec, bool split, const int *L, int nrhs, const void *full_in, void *full_out,
                          void *even, void *odd, hipStream_t st)
{
    const uint32_t V = (uint32_t)L[0] * L[1] * L[2] * L[3];
    const FastDiv fx = make_fastdiv((uint32_t)L[0]), fy = make_fastdiv((uint32_t)L[1]),
                  fz = make_fastdiv((uint32_t)L[2]);
    dim3 g((V + 255) / 256, nrhs), b(256);
#define WL_EO_COPY(PP)                                                                                         \
    if (split)                                                                                                 \
        hipLaunchKernelGGL((eo_copy_kernel<PP, true>), g, b, 0, st, V, nrhs, full_in, full_out, even, odd, fx, \
                           fy, fz, L[0], L[1], L[2]);                                                          \
    else                                                                                                       \
        hipLaunchKernelGGL((eo_copy_kernel<PP, false>), g, b, 0, st, V, nrhs, full_in, full_out, even, odd,    \
                           fx, fy, fz, L[0], L[1], L[2]);
    switch (prec) {
    case F64: WL_EO_COPY(F64) break;
    case F32: WL_EO_COPY(F32) break;
    case BF16S: WL_EO_COPY(BF16S) break;
    case F16S: WL_EO_COPY(F16S) break;
    default: return hipErrorInvalidValue;
    }
#undef WL_EO_COPY
    return hipGetLastError();
}

// The raw data of one hop: the neighbour spinor nb of the half field `in`
// (the other parity) and the link of site ls in the full layout.
template <int P>
__device__ __forceinline__ void eo_raw_load(const EoParams &p, uint32_t nb, uint32_t ls, int mu, int rhs, RawHop<P> &r)
{
    using C = typename std::remove_reference<decltype(r.sp[0])>::type;
    using K = typename std::remove_reference<decltype(r.lk[0])>::type;
    constexpr int NCH = Traits<P>::NCH, NU = Traits<P>::LINK_UNITS;
    const C *b = reinterpret_cast<const C *>(p.in) + (size_t)rhs * NCH * p.Vh + nb;
#pragma unroll
    for (int k = 0; k < NCH; ++k)
        r.sp[k] = b[(size_t)k * p.Vh];
    if constexpr (Traits<P>::SCALED)
        r.sc = scale_ptr<P>(p.in, p.Vh, p.nrhs)[(size_t)rhs * p.Vh + nb];
    const K *u = reinterpret_cast<const K *>(p.U) + (size_t)mu * NU * p.V + ls;
#pragma unroll
    for (int k = 0; k < NU; ++k)
        r.lk[k] = u[(size_t)k * p.V];
}

// The eight hops of a half-lattice site: neighbour (half index), link site
// (full index) and boundary sign of hop h = 2 mu + (0 forward, 1 backward).
struct EoHops {
    uint32_t nb[8], ls[8];
    float sg[8];
};

// In the half layout the y, z and t neighbours keep their half x coordinate,
// so they lie a half stride away; the x neighbours are the same half index or
// the next one, by the parity of the row.
__device__ __forceinline__ void eo_make_hops(const EoParams &p, uint32_t i, EoHops &h, uint32_t &s)
{
    const uint32_t lxh = (uint32_t)p.L[0] / 2;
    const uint32_t q1 = fdiv(i, p.fxh);
    const uint32_t k = i - q1 * lxh;
    const uint32_t q2 = fdiv(q1, p.fy);
    const int y = (int)(q1 - q2 * (uint32_t)p.L[1]);
    const uint32_t q3 = fdiv(q2, p.fz);
    const int z = (int)(q2 - q3 * (uint32_t)p.L[2]);
    const int t = (int)q3;
    const uint32_t odd = (uint32_t)(y + z + t + p.parity) & 1u;  // x = 2 k + odd
    const uint32_t x = 2 * k + odd;
    s = x + (uint32_t)p.L[0] * q1;
    const uint32_t row = q1 * lxh;
    const uint32_t kf = odd ? (k + 1 == lxh ? 0 : k + 1) : k, kb = odd ? k : (k == 0 ? lxh - 1 : k - 1);
    const bool xf = (int)x == p.L[0] - 1, xb = x == 0;
    h.nb[0] = row + kf;
    h.nb[1] = row + kb;
    h.ls[1] = xb ? s + (uint32_t)p.L[0] - 1 : s - 1;
    h.sg[0] = xf && p.bc[0] < 0 ? -1.f : 1.f;
    h.sg[1] = xb && p.bc[0] < 0 ? -1.f : 1.f;
    const int c[3] = {y, z, t};
    uint32_t st = (uint32_t)p.L[0];
#pragma unroll
    for (int m = 0; m < 3; ++m) {
        const int L = p.L[m + 1];
        const bool wf = c[m] == L - 1, wb = c[m] == 0, anti = p.bc[m + 1] < 0;
        const uint32_t span = (uint32_t)(L - 1) * st;
        h.nb[2 * m + 2] = wf ? i - span / 2 : i + st / 2;
        h.nb[2 * m + 3] = wb ? i + span / 2 : i - st / 2;
        h.ls[2 * m + 3] = wb ? s + span : s - st;
        h.sg[2 * m + 2] = wf && anti ? -1.f : 1.f;
        h.sg[2 * m + 3] = wb && anti ? -1.f : 1.f;
        st *= (uint32_t)L;
    }
#pragma unroll
    for (int m = 0; m < 4; ++m)
        h.ls[2 * m] = s;
}

// One hop of raw data into acc, in the arithmetic type of the format (FP16
// too: this path never rounds a projected spinor or a rebuilt row to f16).
template <int P, int DAG, int H>
__device__ __forceinline__ void eo_compute_hop(const RawHop<P> &r, float sg, cx<typename Traits<P>::real> (&acc)[12],
                                               typename Traits<P>::real one)
{
    using T = typename Traits<P>::real;
    constexpr int MU = H / 2, SF = DAG ? 1 : -1, SIG = (H % 2 == 0) ? SF : -SF;
    cx<T> ps[12], u[9], h[6], g[6];
    decode<P>(r, ps, u);
    project<MU, SIG>(ps, h, one);
    if constexpr (H % 2)
        su3_adj_mv(u, h, g);
    else
        su3_mv(u, h, g);
    if constexpr (Traits<P>::SCALED)
        accum<MU, SIG>(acc, g, (T)sg * r.sc);
    else
        accum<MU, SIG>(acc, g, (T)sg);
}

// Hops loaded G at a time, the next G while the current ones are computed
// (as the pipelined full-lattice stencil).
template <int P>
struct EoG {
    static constexpr int G = P == F64 ? 1 : 2;
};
template <int P, int H>
__device__ __forceinline__ void eo_load_group(const EoParams &p, int rhs, const EoHops &hp, RawHop<P> (&buf)[2 * EoG<P>::G])
{
    constexpr int G = EoG<P>::G, slot = ((H / G) % 2) * G;
#pragma unroll
    for (int j = 0; j < G; ++j)
        eo_raw_load<P>(p, hp.nb[H + j], hp.ls[H + j], (H + j) / 2, rhs, buf[slot + j]);
    __builtin_amdgcn_sched_barrier(0);  // keep the loads ahead of the hops before them
}
template <int P, int DAG, int H>
__device__ __forceinline__ void eo_pipe(const EoParams &p, int rhs, const EoHops &hp, RawHop<P> (&buf)[2 * EoG<P>::G],
                                        cx<typename Traits<P>::real> (&acc)[12])
{
    constexpr int G = EoG<P>::G;
    if constexpr (H < 8) {
        if constexpr (H % G == 0 && H + G < 8)
            eo_load_group<P, H + G>(p, rhs, hp, buf);
        eo_compute_hop<P, DAG, H>(buf[((H / G) % 2) * G + H % G], hp.sg[H], acc, (typename Traits<P>::real)p.one);
        eo_pipe<P, DAG, H + 1>(p, rhs, hp, buf, acc);
    }
}

// out(parity) = c_self * self + c_hop * H_{parity, other} in, with optional
// fused reductions over out: |out|^2 (RED_NORM), <v, out> (RED_DOTV, v =
// dotv) or <self, out> and |out|^2 (RED_DOTIN_NORM); with self the Schur
// input, the BiCGStab sets RED_BICG and RED_SR.
//
// Bound by bandwidth: each half-lattice hop needs every link of the lattice
// (forward ones of its own sites, backward ones of the other parity's) and
// two or three half fields.  Workgroups are handed out round-robin over the
// XCDs, each with its own L2; in plain order a tile's z and t neighbours, and
// the other half of the link lines it uses, were fetched by other XCDs again.
// The tile order keeps them on one XCD (eo_order), the right-hand sides of a
// tile run back to back there, and the loads of the next hops are in flight
// while the current ones are computed.  A Schur application (two hops) at
// 32^3 x 64 went from 457 to 279 us in FP32 (4.7 TB/s of the bytes it needs;
// a copy reaches 5.65), 1000 to 588 us in FP64 and 190 to 133 us in FP16.
template <int P, int DAG, int RED>
__global__ __launch_bounds__(256) void eo_hop_kernel(EoParams p)
{
    using T = typename Traits<P>::real;
    constexpr int NV = red_nval(RED);
    __shared__ double lds[(NV > 0 ? NV : 1) * 4];
    uint32_t bt = blockIdx.x;
    int rhs = 0;
    if (p.ng > 1) {
        const uint32_t k = bt >> 3, q = fdiv(k, p.f_ng);
        rhs = (int)(k - q * p.ng);
        bt = (q << 3) | (bt & 7u);
    }
    if (p.skip && p.skip[rhs].frozen)
        return;
    const uint32_t i = p.xcd >= 2 ? slab_site(bt, threadIdx.x, blockDim.x, p.slab)
                                  : tile_of(bt, (uint32_t)p.nblk, p.xcd) * blockDim.x + threadIdx.x;
    double red[NV > 0 ? NV : 1] = {};
    if (i < p.Vh) {
        EoHops hp;
        uint32_t s;
        eo_make_hops(p, i, hp, s);
        cx<T> acc[12];
#pragma unroll
        for (int n = 0; n < 12; ++n)
            acc[n] = cx<T>{T(0), T(0)};
        RawHop<P> buf[2 * EoG<P>::G];
        eo_load_group<P, 0>(p, rhs, hp, buf);
        eo_pipe<P, DAG, 0>(p, rhs, hp, buf, acc);
        const T ch = (T)p.c_hop, cs = (T)p.c_self;
        cx<T> o[12], sf[12];
        if (p.self) {
            load_site<P>(p.self, p.Vh, p.nrhs, i, rhs, sf);
#pragma unroll
            for (int n = 0; n < 12; ++n)
                o[n] = cx<T>{fma(ch, acc[n].re, cs * sf[n].re), fma(ch, acc[n].im, cs * sf[n].im)};
        } else {
#pragma unroll
            for (int n = 0; n < 12; ++n) {
                sf[n] = cx<T>{T(0), T(0)};
                o[n] = cx<T>{ch * acc[n].re, ch * acc[n].im};
            }
        }
        if constexpr (!Traits<P>::SCALED && (RED == RED_NONE || RED == RED_NORM)) {
            if (p.res) {  // the residual of (c_self + c_hop H) in = res
                cx<T> b[12];
                load_site<P>(p.res, p.Vh, p.nrhs, i, rhs, b);
#pragma unroll
                for (int n = 0; n < 12; ++n)
                    o[n] = cx<T>{b[n].re - o[n].re, b[n].im - o[n].im};
            }
        }
        store_site_q<P, true>(p.out, p.Vh, p.nrhs, i, rhs, o);
        if constexpr (RED == RED_NORM || RED == RED_DOTIN_NORM) {
            double n2 = 0.0;
#pragma unroll
            for (int n = 0; n < 12; ++n)
                n2 = fma((double)o[n].re, (double)o[n].re, fma((double)o[n].im, (double)o[n].im, n2));
            red[NV - 1] = n2;
        }
        if constexpr (RED == RED_DOTV || RED == RED_DOTIN_NORM) {
            cx<T> v[12];
            if constexpr (RED == RED_DOTV)
                load_site<P>(p.dotv, p.Vh, p.nrhs, i, rhs, v);
            else
#pragma unroll
                for (int n = 0; n < 12; ++n)
                    v[n] = sf[n];
            double re = 0.0, im = 0.0;
#pragma unroll
            for (int n = 0; n < 12; ++n) {
                re = fma((double)v[n].re, (double)o[n].re, fma((double)v[n].im, (double)o[n].im, re));
                im = fma((double)v[n].re, (double)o[n].im, fma(-(double)v[n].im, (double)o[n].re, im));
            }
            red[0] = re;
            red[1] = im;
        }
        if constexpr (RED == RED_BICG) {  // self = the Schur input s, dotv = rh
            cx<T> v[12];
            load_site<P>(p.dotv, p.Vh, p.nrhs, i, rhs, v);
            bicg_values(sf, o, v, red);
        }
        if constexpr (RED == RED_SR) {  // self = the Schur input v; dotv, dotv2, dotv3 = rh, r, u
            cx<T> a[12], b[12], c[12];
            load_site<P>(p.dotv, p.Vh, p.nrhs, i, rhs, a);
            load_site<P>(p.dotv2, p.Vh, p.nrhs, i, rhs, b);
            load_site<P>(p.dotv3, p.Vh, p.nrhs, i, rhs, c);
            sr_values(sf, o, a, b, c, red);
        }
    }
    if constexpr (NV > 0) {
        const double sum = block_sum<NV>(red, lds);
        if ((int)threadIdx.x < NV)
            p.partials[((size_t)threadIdx.x * p.nrhs + rhs) * p.nblk + bt] = sum;
    }
}

// Sites per workgroup.  256, so that a workgroup holds the y neighbours of
// most of its rows; 64 below 2^16 half-lattice sites, where the chip has more
// wavefront slots than the lattice has wavefronts (8^3 x 16, FP64: 11.4 us
// with 64, 15.9 us with 256; 16^3 x 32, FP32: 16.4 and 16.2 us; 32^3 x 64,
// FP32: 291 and 279 us, all per Schur application of two hops).
static int eo_block(uint32_t Vh) { return Vh >= (1u << 16) ? 256 : 64; }

// Tile order: z-slabs per XCD for the lattices that do not fit the L2s
// together, else (or where the extents do not divide) a contiguous range per
// XCD.  Measured contiguous against slabs: 307 and 279 us at 32^3 x 64 in
// FP32, 674 and 588 us in FP64; 77.3 and 73.3 us at 24^3 x 48 (202 and 174 us
// for three right-hand sides); but 16.2 and 19.3 us at 16^3 x 32 in FP32,
// where only FP64 gains (40.3 and 35.6 us).  In plain order these took 313 to
// 338, 727, 103 and 19.2 us.  Cutting the slabs in y too was slower in every case.
static int eo_order(int prec, const int *H, uint32_t Vh, int block)
{
    return (prec == F64 || Vh >= (1u << 17)) && slab_ok(H, block, 2) ? 2 : 1;
}

int eo_partials(uint32_t Vh, int nrhs)
{
    const int b = eo_block(Vh), n = (int)((Vh + b - 1) / b);
    return nrhs > 1 ? (n + 7) & ~7 : n;
}

EoParams eo_params(const wl_op *op, int parity, int nrhs)
{
    EoParams p{};
    p.U = op->U;
    for (int i = 0; i < 4; ++i) {
        p.L[i] = op->g.dims[i];
        p.bc[i] = op->g.bc[i];
    }
    p.parity = parity;
    p.nrhs = nrhs;
    return p;
}

hipError_t launch_eo_hop(int prec, int dagger, int red, EoParams p, hipStream_t st)
{
    if (p.L[0] % 2 != 0 || p.L[1] % 2 != 0 || p.L[2] % 2 != 0 || p.L[3] % 2 != 0)
        return hipErrorInvalidValue;
    p.V = (uint32_t)p.L[0] * p.L[1] * p.L[2] * p.L[3];
    p.Vh = p.V / 2;
    p.fxh = make_fastdiv((uint32_t)(p.L[0] / 2));
    p.fy = make_fastdiv((uint32_t)p.L[1]);
    p.fz = make_fastdiv((uint32_t)p.L[2]);
    if (p.res && (prec > F32 || (red != RED_NONE && red != RED_NORM)))
        return hipErrorInvalidValue;
    const int block = eo_block(p.Vh);
    p.nblk = eo_partials(p.Vh, p.nrhs);
    p.ng = (uint32_t)p.nrhs;
    p.f_ng = make_fastdiv(p.ng);
    p.one = 1.0f;
    const int H[4] = {p.L[0] / 2, p.L[1], p.L[2], p.L[3]};
    p.xcd = eo_order(prec, H, p.Vh, block);
    if (p.xcd >= 2) {
        SlabOrder &o = p.slab;
        o.zs = (uint32_t)H[2] / 8;
        o.plane_n = (uint32_t)H[0] * (uint32_t)H[1];
        o.slice_n = o.plane_n * o.zs;
        o.chunk_n = o.slice_n * (uint32_t)H[3];
        o.xy = o.plane_n;
        o.vslice = o.xy * (uint32_t)H[2];
        o.f_chunk = make_fastdiv(o.chunk_n);
        o.f_slice = make_fastdiv(o.slice_n);
        o.f_plane = make_fastdiv(o.plane_n);
    }
    if ((uint64_t)p.nblk * p.ng > 0x7fffffffull)
        return hipErrorInvalidValue;
    dim3 g((uint32_t)p.nblk * p.ng), b(block);
#define WL_EO_RED(PP, DD)                                                                                      \
    switch (red) {                                                                                             \
    case RED_NONE: hipLaunchKernelGGL((eo_hop_kernel<PP, DD, RED_NONE>), g, b, 0, st, p); break;              \
    case RED_NORM: hipLaunchKernelGGL((eo_hop_kernel<PP, DD, RED_NORM>), g, b, 0, st, p); break;              \
    case RED_DOTV: hipLaunchKernelGGL((eo_hop_kernel<PP, DD, RED_DOTV>), g, b, 0, st, p); break;              \
    case RED_DOTIN_NORM: hipLaunchKernelGGL((eo_hop_kernel<PP, DD, RED_DOTIN_NORM>), g, b, 0, st, p); break;  \
    case RED_BICG: hipLaunchKernelGGL((eo_hop_kernel<PP, DD, RED_BICG>), g, b, 0, st, p); break;              \
    case RED_SR: hipLaunchKernelGGL((eo_hop_kernel<PP, DD, RED_SR>), g, b, 0, st, p); break;                  \
    default: return hipErrorInvalidValue;                                                                      \
    }
    switch (prec * 2 + (dagger ? 1 : 0)) {
    case 0: WL_EO_RED(F64, 0) break;
    case 1: WL_EO_RED(F64, 1) break;
    case 2: WL_EO_RED(F32, 0) break;
    case 3: WL_EO_RED(F32, 1) break;
    case 4: WL_EO_RED(BF16S, 0) break;
    case 5: WL_EO_RED(BF16S, 1) break;
    case 6: WL_EO_RED(F16S, 0) break;
    case 7: WL_EO_RED(F16S, 1) break;
    default: return hipErrorInvalidValue;
    }
#undef WL_EO_RED
    return hipGetLastError();
}

}  // namespace wl
