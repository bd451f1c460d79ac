// C ABI, context layer: errors, the context (gauge copies, workspace), layout
// conversion kernels, timing and launch configuration.
#include "wl_internal.h"

// ------------------------------------------------------------------ errors
thread_local std::string wli::g_err;

wl_status wli::fail(wl_status st, const char *fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
    return st;
}

#define HIP_TRY(call)                                                                            \
    do {                                                                                         \
        hipError_t e_ = (call);                                                                  \
        if (e_ != hipSuccess) return fail(WL_ERR_HIP, "%s failed: %s", #call, hipGetErrorString(e_)); \
    } while (0)

wl_status wli::ensure_buf(wl_ctx *c, int slot, size_t bytes) {
    if (c->buf_bytes[slot] >= bytes) return WL_OK;
    if (c->buf[slot]) {
        HIP_TRY(hipDeviceSynchronize());
        HIP_TRY(hipFree(c->buf[slot]));
        c->buf[slot] = nullptr;
        c->buf_bytes[slot] = 0;
    }
    hipError_t e = hipMalloc(&c->buf[slot], bytes);
    if (e != hipSuccess) {
        c->buf[slot] = nullptr;
        (void)hipGetLastError();
        return fail(WL_ERR_NOMEM, "hipMalloc of %zu bytes failed: %s", bytes, hipGetErrorString(e));
    }
    c->buf_bytes[slot] = bytes;
    return WL_OK;
}

wl_status wli::ensure_pinned(wl_ctx *c, size_t bytes) {
    if (c->host_pinned_bytes >= bytes) return WL_OK;
    if (c->host_pinned) HIP_TRY(hipHostFree(c->host_pinned));
    c->host_pinned = nullptr;
    c->host_pinned_bytes = 0;
    HIP_TRY(hipHostMalloc(&c->host_pinned, bytes, hipHostMallocDefault));
    c->host_pinned_bytes = bytes;
    return WL_OK;
}

// ------------------------------------------------------------------ small kernels (layout conversion)
// canonical FP64 spinor <-> internal, through LDS.  A block takes a run of `ns`
// consecutive canonical sites (of both parities for a FULL field) with all their
// right-hand sides: at most PACK_POINTS points.  The canonical side moves as contiguous
// 16-byte units (ns * 192 bytes a right-hand side), the internal side a point per thread
// (consecutive points, rhs fastest); between them a point occupies 13 units of LDS, so
// that the 16 points of a 16-byte access fall into different banks.
// Bound by HBM.  12 right-hand sides at 16^3x32 in FP32, 453 MB each way: pack 89 us
// (5.1 TB/s; 102 us with a thread reading its point's 192 bytes by itself, each line
// fetched for half its bytes) and unpack 69 us (6.6 TB/s, non-temporal stores; 139 us).
constexpr int PACK_POINTS = 128;
struct PackArgs {
    Geom g;
    size_t half_bytes;
    int subset, nrhs;
    int ns;      // canonical sites of a block (even)
    long nsite;  // canonical sites of the field
    FastDiv f_run;  // 12 ns: 16-byte units of a block's run of one right-hand side
};

// unit e of the block's canonical runs: its right-hand side, site in the run and component
__device__ __forceinline__ void pack_unit(const PackArgs &a, int e, int &rhs, int &u, int &sl) {
    rhs = fdiv(e, a.f_run);
    u = e - rhs * a.f_run.d;
    sl = u / 12;
}
constexpr int PACK_BURST = 12;  // a thread's loads, all in flight at once

// internal point of thread `e` of the block's nloc * nrhs points: its half, its index
// there and its place in LDS; false past the end
__device__ __forceinline__ bool pack_point(const PackArgs &a, long s0, int nloc, int e, int &h, long &pt, int &slot) {
    if (e >= nloc * a.nrhs) return false;
    int sl = e / a.nrhs;
    const int rhs = e - sl * a.nrhs;
    h = 0;
    if (a.subset == WL_FULL) {
        // the even sites of the run first: site i of a parity is canonical site 2 i or 2 i + 1
        const int nh = nloc >> 1;
        if (sl >= nh) h = 1, sl -= nh;
        const int i = (int)(s0 >> 1) + sl;
        pt = (long)i * a.nrhs + rhs;
        const int r = fdiv(i, a.g.f_lxh), r2 = fdiv(r, a.g.f_ly), t = fdiv(r2, a.g.f_lz);
        const int y = r - r2 * a.g.L[1], z = r2 - t * a.g.L[2];
        sl = 2 * sl + ((y + z + t + h) & 1);
    } else {
        pt = (s0 + sl) * a.nrhs + rhs;
    }
    slot = sl * a.nrhs + rhs;
    return true;
}

template <int SP>
__global__ void __launch_bounds__(PACK_POINTS) k_pack(const PackArgs a, void *dst, const double *src) {
    using T = typename SpinorIO<SP>::real;
    __shared__ double2 lds[PACK_POINTS * 13];
    const long s0 = (long)blockIdx.x * a.ns;
    const int nloc = (int)min((long)a.ns, a.nsite - s0);
    int h, slot;
    long pt;
    const int total = a.nrhs * a.f_run.d;
    for (int e0 = threadIdx.x; e0 < total; e0 += PACK_BURST * PACK_POINTS) {
        v2d d[PACK_BURST];
        int to[PACK_BURST];
#pragma unroll
        for (int k = 0; k < PACK_BURST; ++k) {
            const int e = e0 + k * PACK_POINTS;
            int rhs, u, sl;
            pack_unit(a, e, rhs, u, sl);
            to[k] = e < total && sl < nloc ? (sl * a.nrhs + rhs) * 13 + (u - 12 * sl) : -1;
            if (to[k] >= 0) d[k] = ((const v2d *)src)[((long)rhs * a.nsite + s0) * 12 + u];
        }
#pragma unroll
        for (int k = 0; k < PACK_BURST; ++k)
            if (to[k] >= 0) lds[to[k]] = make_double2(d[k].x, d[k].y);
    }
    __syncthreads();
    if (!pack_point(a, s0, nloc, threadIdx.x, h, pt, slot)) return;
    cpx<T> v[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) {
        const double2 d = lds[slot * 13 + k];
        v[k] = {(T)d.x, (T)d.y};
    }
    SpinorIO<SP>::store((char *)dst + h * a.half_bytes, pt, v);
}

// a thread per internal point, which reads its point's 192 bytes itself (see pack_direct)
constexpr int PACK_DIRECT_BLOCK = 256;
template <int SP>
__global__ void __launch_bounds__(PACK_DIRECT_BLOCK) k_pack_direct(const PackArgs a, void *dst, const double *src) {
    using T = typename SpinorIO<SP>::real;
    const int h = blockIdx.y;
    const long pt = (long)blockIdx.x * PACK_DIRECT_BLOCK + threadIdx.x;
    if (pt >= (long)a.g.vh * a.nrhs) return;
    const int i = (int)(pt / a.nrhs), rhs = (int)(pt - (long)i * a.nrhs);
    long site = i;
    if (a.subset == WL_FULL) {
        int c[4];
        eo_coords(a.g, i, h, c);
        site = c[0] + (long)a.g.L[0] * (c[1] + (long)a.g.L[1] * (c[2] + (long)a.g.L[2] * c[3]));
    }
    const double2 *from = (const double2 *)src + (rhs * a.nsite + site) * 12;
    cpx<T> v[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) {
        const double2 d = from[k];
        v[k] = {(T)d.x, (T)d.y};
    }
    SpinorIO<SP>::store((char *)dst + h * a.half_bytes, pt, v);
}

template <int SP>
__global__ void __launch_bounds__(PACK_POINTS) k_unpack(const PackArgs a, double *dst, const void *src) {
    using T = typename SpinorIO<SP>::real;
    __shared__ double2 lds[PACK_POINTS * 13];
    const long s0 = (long)blockIdx.x * a.ns;
    const int nloc = (int)min((long)a.ns, a.nsite - s0);
    int h, slot;
    long pt;
    if (pack_point(a, s0, nloc, threadIdx.x, h, pt, slot)) {
        cpx<T> v[12];
        SpinorIO<SP>::load((const char *)src + h * a.half_bytes, pt, v);
#pragma unroll
        for (int k = 0; k < 12; ++k) lds[slot * 13 + k] = make_double2((double)v[k].re, (double)v[k].im);
    }
    __syncthreads();
    const int total = a.nrhs * a.f_run.d;
    for (int e = threadIdx.x; e < total; e += PACK_POINTS) {
        int rhs, u, sl;
        pack_unit(a, e, rhs, u, sl);
        if (sl >= nloc) continue;
        const double2 d = lds[(sl * a.nrhs + rhs) * 13 + (u - 12 * sl)];
        __builtin_nontemporal_store(v2d{d.x, d.y}, (v2d *)dst + ((long)rhs * a.nsite + s0) * 12 + u);
    }
}

// Whether a thread reads its point's 192 bytes itself (k_pack_direct) instead of going through
// LDS.  LDS pays where the source's lines would come from HBM more than once (many sites
// in flight, both parities of a line read by different blocks) and the launch is long enough
// for two phases a block; a half field's wave reads whole stretches anyway.  Times of direct
// over LDS, 18 counts of right-hand sides on 7 lattices from 8^4 to 32^4:
//   full fields, FP64 and FP32: below 72,000 points 0.77 to 1.02 (once 1.13), from there 0.92 to
//     1.37 (16^3x32, 12 rhs, FP32 103 against 89 us), 33 rhs 0.83 to 1.16; 16-bit formats: below
//     330,000 points 0.79 to 1.23, 2 and 3 rhs 0.86 to 1.18, the rest 0.96 to 1.45;
//   half fields: below 700,000 points or 12 rhs (16-bit: 24) 0.72 to 1.12 (0.92 in the middle), the
//     rest 0.93 to 1.26 (16^3x32, 24 rhs, FP32 105 against 85 us).
static bool pack_direct(int prec, int subset, int nrhs, long vh) {
    const bool narrow = prec != WL_F64 && prec != WL_F32;
    const long points = vh * nrhs * (subset == WL_FULL ? 2 : 1);
    if (subset != WL_FULL) return points < 700000 || nrhs < (narrow ? 24 : 12);
    return narrow ? points < 330000 || nrhs == 2 || nrhs == 3 : points < 72000 || (nrhs > 32 && nrhs % 2);
}
static PackArgs pack_args(const wl_ctx *c, int subset, size_t hb, int nrhs, dim3 *grid) {
    PackArgs a;
    a.g = c->g;
    a.half_bytes = hb;
    a.subset = subset;
    a.nrhs = nrhs;
    a.ns = PACK_POINTS / nrhs & ~1;  // nrhs <= 64
    a.nsite = subset == WL_FULL ? c->V : c->Vh;
    a.f_run = make_fastdiv(12 * a.ns);
    *grid = dim3((unsigned)((a.nsite + a.ns - 1) / a.ns));
    return a;
}

// FP64 18-real internal links -> another link format, one thread per (slab, site)
template <int GP, int R>
__global__ void __launch_bounds__(256) k_link_convert(void *dst, size_t dslab, const void *src, size_t sslab,
                                                      int vh) {
    using T = typename LinkIO<GP, R>::real;
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    const int slab = blockIdx.y;
    if (i >= vh) return;
    cpx<double> u[9];
    LinkIO<WL_F64, 18>::load((const char *)src + slab * sslab, i, u);
    cpx<T> w[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) w[k] = {(T)u[k].re, (T)u[k].im};
    LinkIO<GP, R>::store((char *)dst + slab * dslab, i, w);
}

template <template <int> class K, typename... A>
static hipError_t launch_prec(int prec, dim3 grid, int block, hipStream_t s, A... args) {
    switch (prec) {
    case WL_F64: hipLaunchKernelGGL(K<WL_F64>::fn, grid, dim3(block), 0, s, args...); break;
    case WL_F32: hipLaunchKernelGGL(K<WL_F32>::fn, grid, dim3(block), 0, s, args...); break;
    case WL_F16N: hipLaunchKernelGGL(K<WL_F16N>::fn, grid, dim3(block), 0, s, args...); break;
    case WL_BF16N: hipLaunchKernelGGL(K<WL_BF16N>::fn, grid, dim3(block), 0, s, args...); break;
    case WL_I16N: hipLaunchKernelGGL(K<WL_I16N>::fn, grid, dim3(block), 0, s, args...); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}
template <int SP> struct PackDirectK { static constexpr auto fn = k_pack_direct<SP>; };
template <int SP> struct PackK { static constexpr auto fn = k_pack<SP>; };
template <int SP> struct UnpackK { static constexpr auto fn = k_unpack<SP>; };

// ------------------------------------------------------------------ context API
extern "C" const char *wl_last_error(void) { return g_err.c_str(); }
extern "C" const char *wl_version(void) { return "wilson-gfx950 0.1"; }

extern "C" wl_status wl_ctx_create(const int dims[4], const double phases[8], const double *gauge_host,
                                   wl_ctx **out) {
    g_err.clear();
    if (!dims || !phases || !gauge_host || !out) return fail(WL_ERR_ARG, "null argument");
    *out = nullptr;
    long V = 1;
    for (int m = 0; m < 4; ++m) {
        if (dims[m] < 2 || dims[m] % 2 || dims[m] > 4096)
            return fail(WL_ERR_DIMS, "extent %d of direction %d must be even and in [2, 4096]", dims[m], m);
        V *= dims[m];
        if (V > (1L << 28)) return fail(WL_ERR_DIMS, "volume exceeds 2^28 sites");
    }
    for (int k = 0; k < 8; ++k)
        if (!std::isfinite(phases[k])) return fail(WL_ERR_ARG, "non-finite boundary phase");
    int ndev = 0;
    hipError_t e = hipGetDeviceCount(&ndev);
    if (e != hipSuccess || ndev < 1) {
        (void)hipGetLastError();
        return fail(WL_ERR_HIP, "no HIP device available (%s)", hipGetErrorString(e));
    }
    int device = 0;
    HIP_TRY(hipGetDevice(&device));
    // the allocation-free entry points' scratch address on this device (once per device)
    if (wl_status sst = scratch_setup(device)) return sst;
    wl_ctx *c = new wl_ctx();
    std::memcpy(c->dims, dims, sizeof c->dims);
    std::memcpy(c->phases, phases, sizeof c->phases);
    c->V = V;
    c->Vh = V / 2;
    c->device = device;
    Geom &g = c->g;
    for (int m = 0; m < 4; ++m) g.L[m] = dims[m];
    g.lxh = dims[0] / 2;
    g.vh = (int)c->Vh;
    g.sy = g.lxh;
    g.sz = g.lxh * dims[1];
    g.st = g.lxh * dims[1] * dims[2];
    g.f_lxh = make_fastdiv(g.lxh);
    g.f_ly = make_fastdiv(dims[1]);
    g.f_lz = make_fastdiv(dims[2]);
    g.f_sz = make_fastdiv(g.sz);
    g.phase_mask = 0;
    for (int m = 0; m < 4; ++m) {
        g.zr[m] = phases[2 * m];
        g.zi[m] = phases[2 * m + 1];
        if (!(phases[2 * m] == 1.0 && phases[2 * m + 1] == 0.0)) g.phase_mask |= 1 << m;
    }
    // host packing of the canonical FP64 gauge field into the FP64 18-real internal layout
    const size_t slab = LinkIO<WL_F64, 18>::bytes_per_link * (size_t)padded(c->Vh);
    std::vector<double> host(slab / sizeof(double) * 8);
    for (long lex = 0; lex < V; ++lex) {
        long r = lex;
        const int x = (int)(r % dims[0]);
        r /= dims[0];
        const int y = (int)(r % dims[1]);
        r /= dims[1];
        const int z = (int)(r % dims[2]);
        const int t = (int)(r / dims[2]);
        const int par = (x + y + z + t) & 1;
        const long i = lex >> 1;
        for (int mu = 0; mu < 4; ++mu)
            for (int k = 0; k < 9; ++k) {
                const double *src = gauge_host + ((lex * 4 + mu) * 9 + k) * 2;
                // slab (par, mu); block i / 64, unit k, lane i % 64 (double2 units)
                double *dst = host.data() + (size_t)(par * 4 + mu) * (slab / sizeof(double)) +
                              ((size_t)((i >> 6) * 9 + k) * 64 + (i & 63)) * 2;
                dst[0] = src[0];
                dst[1] = src[1];
            }
    }
    void *d = nullptr;
    e = hipMalloc(&d, slab * 8);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        delete c;
        return fail(WL_ERR_NOMEM, "hipMalloc of gauge field failed: %s", hipGetErrorString(e));
    }
    e = hipMemcpy(d, host.data(), slab * 8, hipMemcpyHostToDevice);
    if (e != hipSuccess) {
        (void)hipFree(d);
        delete c;
        return fail(WL_ERR_HIP, "gauge upload failed: %s", hipGetErrorString(e));
    }
    c->gauge[WL_F64][0] = d;
    e = hipHostMalloc((void **)&c->red_pinned, RED_PINNED * sizeof(double), hipHostMallocDefault);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        c->red_pinned = nullptr;
        wl_ctx_destroy(c);
        return fail(WL_ERR_NOMEM, "pinned host memory: %s", hipGetErrorString(e));
    }
    // measured defaults (MI355X, 24^3x48 and 32^3x64 lattices): two threads per point
    c->cfg[WL_F64] = {hop_default_block(WL_F64), 1, 2, WL_TCHUNK_AUTO, -1};
    c->cfg[WL_F32] = {hop_default_block(WL_F32), 1, 2, WL_TCHUNK_AUTO, -1};
    // 16-bit storage: few registers per thread, so without a cap so many waves are in flight
    // that their neighbour spinors crowd each other out of L2; about 4 waves per SIMD measured
    // best (FP16 half-dslash at 32^3x64: 82 -> 67 us)
    c->cfg[WL_F16N] = {256, 1, 1, WL_TCHUNK_AUTO, -1, 1, 0, 4};
    c->cfg[WL_BF16N] = {256, 1, 1, WL_TCHUNK_AUTO, -1, 1, 0, 4};
    c->cfg[WL_I16N] = {256, 1, 1, WL_TCHUNK_AUTO, -1, 1, 0, 4};
    c->slab[WL_F64][0] = slab;
    *out = c;
    return WL_OK;
}

extern "C" wl_status wl_ctx_destroy(wl_ctx *c) {
    if (!c) return WL_OK;
    (void)hipDeviceSynchronize();
    for (hipEvent_t e : c->event_pool) (void)hipEventDestroy(e);
    if (c->cg_exec) (void)hipGraphExecDestroy(c->cg_exec);
    if (c->cg_graph) (void)hipGraphDestroy(c->cg_graph);
    for (hipEvent_t e : c->handoff)
        if (e) (void)hipEventDestroy(e);
    if (c->own_stream) (void)hipStreamDestroy(c->own_stream);
    for (hipEvent_t e : c->halo_ev)
        if (e) (void)hipEventDestroy(e);
    if (c->comm_stream) (void)hipStreamDestroy(c->comm_stream);
    for (int p = 0; p < 5; ++p)
        for (int r = 0; r < 2; ++r)
            if (c->gauge[p][r]) (void)hipFree(c->gauge[p][r]);
    for (int s = 0; s < S_NSLOTS; ++s)
        if (c->buf[s]) (void)hipFree(c->buf[s]);
    if (c->host_pinned) (void)hipHostFree(c->host_pinned);
    if (c->red_pinned) (void)hipHostFree(c->red_pinned);
    delete c;
    return WL_OK;
}

wl_status wli::get_links(wl_ctx *c, int prec, int recon, const void **ptr, size_t *slab) {
    if (!recon_ok(prec, recon)) return fail(WL_ERR_UNSUPPORTED, "link format prec %d / recon %d not supported", prec, recon);
    const int ri = recon == 12 ? 1 : 0;
    if (!c->gauge[prec][ri]) {
        const size_t sl = link_bytes(prec, recon) * (size_t)padded(c->Vh);
        void *d = nullptr;
        hipError_t e = hipMalloc(&d, sl * 8);
        if (e != hipSuccess) {
            (void)hipGetLastError();
            return fail(WL_ERR_NOMEM, "hipMalloc of link copy failed: %s", hipGetErrorString(e));
        }
        dim3 grid((unsigned)((c->Vh + 255) / 256), 8);
        const void *src = c->gauge[WL_F64][0];
        const size_t ss = c->slab[WL_F64][0];
        const int vh = (int)c->Vh;
        if (prec == WL_F64 && recon == 12) hipLaunchKernelGGL((k_link_convert<WL_F64, 12>), grid, dim3(256), 0, 0, d, sl, src, ss, vh);
        else if (prec == WL_F32 && recon == 18) hipLaunchKernelGGL((k_link_convert<WL_F32, 18>), grid, dim3(256), 0, 0, d, sl, src, ss, vh);
        else if (prec == WL_F32 && recon == 12) hipLaunchKernelGGL((k_link_convert<WL_F32, 12>), grid, dim3(256), 0, 0, d, sl, src, ss, vh);
        else if (prec == WL_F16N) hipLaunchKernelGGL((k_link_convert<WL_F16N, 12>), grid, dim3(256), 0, 0, d, sl, src, ss, vh);
        else if (prec == WL_BF16N) hipLaunchKernelGGL((k_link_convert<WL_BF16N, 12>), grid, dim3(256), 0, 0, d, sl, src, ss, vh);
        else if (prec == WL_I16N) hipLaunchKernelGGL((k_link_convert<WL_I16N, 12>), grid, dim3(256), 0, 0, d, sl, src, ss, vh);
        HIP_TRY(hipGetLastError());
        HIP_TRY(hipDeviceSynchronize());
        c->gauge[prec][ri] = d;
        c->slab[prec][ri] = sl;
    }
    *ptr = c->gauge[prec][ri];
    *slab = c->slab[prec][ri];
    return WL_OK;
}

extern "C" wl_status wl_ctx_prepare_links(wl_ctx *c, wl_prec prec, int recon) {
    g_err.clear();
    if (!c) return fail(WL_ERR_ARG, "null context");
    if (!prec_ok(prec)) return fail(WL_ERR_ARG, "bad precision %d", (int)prec);
    const void *p;
    size_t s;
    return get_links(c, prec, recon, &p, &s);
}

extern "C" wl_status wl_spinor_bytes(const wl_ctx *c, wl_subset subset, wl_prec prec, int nrhs, size_t *bytes) {
    g_err.clear();
    wl_status st = check_field_args(c, subset, prec, nrhs);
    if (st) return st;
    if (!bytes) return fail(WL_ERR_ARG, "null output");
    *bytes = half_bytes(c, prec, nrhs) * (subset == WL_FULL ? 2 : 1);
    return WL_OK;
}

extern "C" wl_status wl_pack_spinor(const wl_ctx *c, void *dst, const double *src, wl_subset subset, wl_prec prec,
                                    int nrhs, void *stream) {
    g_err.clear();
    wl_status st = check_field_args(c, subset, prec, nrhs);
    if (st) return st;
    if (!dst || !src) return fail(WL_ERR_ARG, "null field pointer");
    if (!aligned16(dst) || !aligned16(src)) return fail(WL_ERR_ARG, "field pointers must be 16-byte aligned");
    const int nh = subset == WL_FULL ? 2 : 1;
    const size_t hb = half_bytes(c, prec, nrhs);
    if (overlap(dst, hb * nh, src, (size_t)c->Vh * nh * nrhs * 24 * 8)) return fail(WL_ERR_ARG, "dst and src overlap");
    dim3 grid;
    const PackArgs a = pack_args(c, subset, hb, nrhs, &grid);
    if (pack_direct(prec, subset, nrhs, c->Vh)) {
        grid = dim3((unsigned)((c->Vh * nrhs + PACK_DIRECT_BLOCK - 1) / PACK_DIRECT_BLOCK), nh);
        HIP_TRY((launch_prec<PackDirectK>(prec, grid, PACK_DIRECT_BLOCK, (hipStream_t)stream, a, dst, src)));
        return WL_OK;
    }
    HIP_TRY((launch_prec<PackK>(prec, grid, PACK_POINTS, (hipStream_t)stream, a, dst, src)));
    return WL_OK;
}

extern "C" wl_status wl_unpack_spinor(const wl_ctx *c, double *dst, const void *src, wl_subset subset, wl_prec prec,
                                      int nrhs, void *stream) {
    g_err.clear();
    wl_status st = check_field_args(c, subset, prec, nrhs);
    if (st) return st;
    if (!dst || !src) return fail(WL_ERR_ARG, "null field pointer");
    if (!aligned16(dst) || !aligned16(src)) return fail(WL_ERR_ARG, "field pointers must be 16-byte aligned");
    const int nh = subset == WL_FULL ? 2 : 1;
    const size_t hb = half_bytes(c, prec, nrhs);
    if (overlap(dst, (size_t)c->Vh * nh * nrhs * 24 * 8, src, hb * nh)) return fail(WL_ERR_ARG, "dst and src overlap");
    dim3 grid;
    const PackArgs a = pack_args(c, subset, hb, nrhs, &grid);
    HIP_TRY((launch_prec<UnpackK>(prec, grid, PACK_POINTS, (hipStream_t)stream, a, dst, src)));
    return WL_OK;
}

VecArgs wli::vec_args(const wl_ctx *c, int prec, int nrhs) {
    VecArgs a;
    std::memset(&a, 0, sizeof a);
    a.n = c->Vh * (long)nrhs;
    a.nrhs = nrhs;
    (void)prec;
    return a;
}
void wli::set_vec(VecArgs &a, int k, const void *base, size_t hb) {
    a.v[k][0] = (void *)base;
    a.v[k][1] = (char *)base + hb;
}

extern "C" wl_status wl_convert_spinor(const wl_ctx *c, void *dst, wl_prec dprec, const void *src, wl_prec sprec,
                                       wl_subset subset, int nrhs, void *stream) {
    g_err.clear();
    wl_status st = check_field_args(c, subset, sprec, nrhs);
    if (st) return st;
    if (!prec_ok(dprec)) return fail(WL_ERR_ARG, "bad precision %d", (int)dprec);
    if (!dst || !src || !aligned16(dst) || !aligned16(src)) return fail(WL_ERR_ARG, "null or misaligned field pointer");
    const int nh = subset == WL_FULL ? 2 : 1;
    if (overlap(dst, half_bytes(c, dprec, nrhs) * nh, src, half_bytes(c, sprec, nrhs) * nh))
        return fail(WL_ERR_ARG, "dst and src overlap");
    VecArgs a = vec_args(c, sprec, nrhs);
    set_vec(a, 0, src, half_bytes(c, sprec, nrhs));
    set_vec(a, 1, dst, half_bytes(c, dprec, nrhs));
    HIP_TRY(blas_convert(dprec, sprec, false, a, nh, (hipStream_t)stream));
    return WL_OK;
}

const char *wli::launch_problem(int block, int tps, int nt, int rpt, int occ, int sweep) {
    if (block < 64 || block > 256 || block % 64) return "block not in {64, 128, 192, 256}";
    if (occ < 0 || occ > 8) return "occ not in 0..8";
    if (sweep < 0 || sweep > 65536) return "sweep not in 0..65536";
    if (tps != 1 && tps != 2) return "tps not in {1, 2}";
    if (nt < -1 || nt > 1) return "nt not in {-1, 0, 1}";
    if (rpt < 1 || rpt > 4) return "rpt not in 1..4";
    if (rpt > 1 && tps != 1) return "rpt > 1 needs tps = 1";
    return nullptr;
}

// ------------------------------------------------------------------ timing API
extern "C" wl_status wl_timing_enable(wl_ctx *c, int enable) {
    g_err.clear();
    if (!c) return fail(WL_ERR_ARG, "null context");
    if (enable < 0) return fail(WL_ERR_ARG, "enable = %d < 0", enable);
    HIP_TRY(hipDeviceSynchronize());
    c->timed.clear();
    c->pool_used = 0;
    c->timing = enable != 0;
    c->timing_stride = enable > 0 ? enable : 1;
    c->timing_seq = 0;
    return WL_OK;
}

extern "C" wl_status wl_timing_read(wl_ctx *c, wl_prec prec, int recon, int dagger, int epilogue, int *count,
                                    double *total_ms) {
    g_err.clear();
    if (!c || !count || !total_ms) return fail(WL_ERR_ARG, "null argument");
    if (!prec_ok(prec) || !recon_ok(prec, recon) || epilogue < 0 || epilogue > 7)
        return fail(WL_ERR_ARG, "bad kernel selector");
    const int key = timing_key(prec, recon, dagger != 0, epilogue);
    int n = 0;
    double ms = 0.0;
    for (auto &t : c->timed) {
        if (t.key != key) continue;
        HIP_TRY(hipEventSynchronize(t.ev[1]));
        float m = 0.f;
        HIP_TRY(hipEventElapsedTime(&m, t.ev[0], t.ev[1]));
        ms += m;
        ++n;
    }
    *count = n;
    *total_ms = ms;
    return WL_OK;
}

// ------------------------------------------------------------------ launch configuration
extern "C" wl_status wl_ctx_set_launch(wl_ctx *c, wl_prec prec, const wl_launch *l) {
    g_err.clear();
    if (!c || !l) return fail(WL_ERR_ARG, "null argument");
    if (!prec_ok(prec)) return fail(WL_ERR_ARG, "bad precision %d", (int)prec);
    if (const char *why = launch_problem(l->block, l->tps, l->nt, l->rpt, l->occ, l->sweep))
        return fail(WL_ERR_ARG, "launch (block %d, tps %d, nt %d, rpt %d, occ %d, sweep %d): %s", l->block, l->tps,
                    l->nt, l->rpt, l->occ, l->sweep, why);
    LaunchCfg &g = c->cfg[prec];
    g.block = l->block;
    g.swizzle = l->swizzle ? 1 : 0;
    g.tps = l->tps;
    g.tchunk = l->tchunk;
    g.nt = l->nt;
    g.rpt = l->rpt;
    g.occ = l->occ;
    g.sweep = l->sweep;
    return WL_OK;
}

extern "C" wl_status wl_ctx_get_launch(const wl_ctx *c, wl_prec prec, wl_launch *l) {
    g_err.clear();
    if (!c || !l) return fail(WL_ERR_ARG, "null argument");
    if (!prec_ok(prec)) return fail(WL_ERR_ARG, "bad precision %d", (int)prec);
    const LaunchCfg &g = c->cfg[prec];
    l->block = g.block;
    l->swizzle = g.swizzle;
    l->tps = g.tps;
    l->tchunk = g.tchunk;
    l->nt = g.nt;
    l->rpt = g.rpt;
    l->occ = g.occ;
    l->sweep = g.sweep;
    return WL_OK;
}
