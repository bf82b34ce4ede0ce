// C ABI of the non-ideal DDF lattice Boltzmann library (declared in lbm.h):
// context management, launches of the step kernels, moments, population
// access, conservation sums and the stand-alone codec.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdlib>
#include <cstdio>
#include <cstring>
#include <new>

#include "lbm.h"
#include "lbm_internal.hpp"
#include "lbm_block2d.hpp"
#include <algorithm>
#include <type_traits>

using namespace lbm;

// ---------------------------------------------------------------------------
// Deterministic FP64 reductions: per-block partials (wavefront shuffles, then
// LDS), then a single block summing the partials in a fixed order.
// ---------------------------------------------------------------------------
namespace lbm {
// the counts of non-finite and inadmissible cells for the FP64 inputs of
// lbm_init (rho, u, T given; P from eq. Pvdw), columns 5 and 6 of the partials,
// the others zero
template <int D>
__global__ void __launch_bounds__(BX) k_check_inputs(long long N, Phys<double> ph, const double *rho,
                                                            const double *u, const double *T, double *partials) {
    double acc[RED_VALS] = {0, 0, 0, 0, 0, 0, 0};
    for (long long c = blockIdx.x * (long long)BX + threadIdx.x; c < N; c += (long long)gridDim.x * BX) {
        const double r = rho[c], t = T[c];
        double uu[3] = {0, 0, 0};
        bool bad = !isfinite(r) || !isfinite(t);
        for (int a = 0; a < D; a++) {
            uu[a] = u[a * N + c];
            bad = bad || !isfinite(uu[a]);
        }
        acc[5] += bad ? 1.0 : 0.0;
        if (!bad) {
            const double P = ph.pr ? pr_eos(ph, r, t).P : vdw_pressure(ph, r, t);
            acc[6] += admissible<D>(r, P / r, uu, ph.b) ? 0.0 : 1.0;
        }
    }
    block_partials(acc, partials);
}

// wavefront k sums column k, lane l the partials l, l + 64, ... (one lane per
// column reading 1024 partials one after the other took 148 us; now 12 us for 2048)
__global__ void __launch_bounds__(64 * RED_VALS) k_reduce_final(int nblocks, const double *partials, double *out) {
    const int k = threadIdx.x >> 6, lane = threadIdx.x & 63;
    double s = 0;
    for (int b = lane; b < nblocks; b += 64) s += partials[(long long)b * RED_VALS + k];
    s = wave_sum(s);
    if (lane == 0) out[k] = s;
}

// population decode / encode between the storage form and FP64: the (f, g) pair
// of a direction in one access, the caller's two arrays in whole lines.  Bound
// by HBM (333 x 201 x 97 cells, FP16, 3.5 GB: read 1.27 ms and write 0.98 ms
// with f and g apart, now 0.82 and 0.74; non-temporal stores of the read-out
// 0.96).  The way in takes the non-temporal hint on both sides: the data come
// from elsewhere and are read once.  With the hint on the loads alone, or on
// neither, that write takes 0.87 and 0.73 ms, and after other traffic 128 x 9 x
// 291 cells in BF16 41 and 63 us, with both 36 (f and g apart 61).
template <int D, class S>
__global__ void __launch_bounds__(BX) k_get_pops(Grid g, RefPops ref, const typename S::T *__restrict__ fi,
                                                 double *__restrict__ fo, double *__restrict__ go, SetForm form) {
    using C = typename S::C;
    constexpr int Q = Lattice<D>::Q;
    const int pull = form.pull();
    int x, y, z;
    if (!flat_cell(g, x, y, z)) return;
    long long c = cell_index<D>(g, x, y, z);
#pragma unroll
    for (int i = 0; i < Q; i++) {
        const PopPair<typename S::T> p = load_pair(fi, arrived_index<D>(g, i, x, y, z, pull));
        fo[i * g.N + c] = (double)S::load(&p.f, 0, (C)ref.f[i]);
        go[i * g.N + c] = (double)S::load(&p.g, 0, (C)ref.g[i]);
    }
}
template <int D, class S>
__global__ void __launch_bounds__(BX) k_set_pops(Grid g, RefPops ref, const double *__restrict__ fi,
                                                 const double *__restrict__ gi, typename S::T *__restrict__ fo,
                                                 int *form) {
    using C = typename S::C;
    constexpr int Q = Lattice<D>::Q;
    int x, y, z;
    if (!flat_cell(g, x, y, z)) return;
    mark_form(form, 0);
    long long c = cell_index<D>(g, x, y, z);
    const long long xy = x + (long long)g.nx * y;
#pragma unroll
    for (int i = 0; i < Q; i++)
        store_pair_nt(fo, pop_index<Q>(g, i, z, xy),
                      S::enc((C)__builtin_nontemporal_load(&fi[i * g.N + c]), (C)ref.f[i]),
                      S::enc((C)__builtin_nontemporal_load(&gi[i * g.N + c]), (C)ref.g[i]));
}

__global__ void k_codec_encode(int kind, const float *x, const float *ref, uint16_t *out, long long n) {
    long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (i >= n) return;
    float d = x[i] - ref[i];
    out[i] = kind == LBM_STORE_BF16 ? f32_to_bf16_rne(d) : f32_to_f16_rne(d);
}
__global__ void k_codec_decode(int kind, const uint16_t *code, const float *ref, float *out, long long n) {
    long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (i >= n) return;
    out[i] = ref[i] + (kind == LBM_STORE_BF16 ? bf16_to_f32(code[i]) : f16_to_f32(code[i]));
}
// HBM bandwidth probes (the practical ceiling the step's kernels are
// measured against): 16-byte accesses per lane, grid-stride loops, stores
// and loads with the non-temporal hint.  The read probe folds its loads into
// one value that is stored only if it equals an arbitrary constant, so the
// loads cannot be dropped.
__global__ void __launch_bounds__(256) k_probe_read(const u32x4 *__restrict__ src, long long n,
                                                    u32x4 *__restrict__ sink) {
    u32x4 acc = {0u, 0u, 0u, 0u};
    for (long long i = blockIdx.x * 256ll + threadIdx.x; i < n; i += (long long)gridDim.x * 256)
        acc ^= __builtin_nontemporal_load(&src[i]);
    const unsigned a = acc.x, b = acc.y, c = acc.z, d = acc.w;
    if ((a ^ b ^ c ^ d) == 0x9e3779b9u) sink[0] = acc;
}
__global__ void __launch_bounds__(256) k_probe_write(u32x4 *__restrict__ dst, long long n) {
    for (long long i = blockIdx.x * 256ll + threadIdx.x; i < n; i += (long long)gridDim.x * 256) {
        const unsigned k = (unsigned)i;
        __builtin_nontemporal_store((u32x4){k, k + 1u, k + 2u, k + 3u}, &dst[i]);
    }
}
__global__ void __launch_bounds__(256) k_probe_copy(const u32x4 *__restrict__ src, u32x4 *__restrict__ dst,
                                                    long long n) {
    for (long long i = blockIdx.x * 256ll + threadIdx.x; i < n; i += (long long)gridDim.x * 256)
        __builtin_nontemporal_store(__builtin_nontemporal_load(&src[i]), &dst[i]);
}
}  // namespace lbm

// ---------------------------------------------------------------------------
// host helpers
// ---------------------------------------------------------------------------
// the flat grid of flat_cell()
static dim3 flat_grid(const lbm_ctx *c) {
    const long long plane = (long long)c->p.nx * c->p.ny;
    return dim3((unsigned)((plane + BX - 1) / BX), (unsigned)c->p.nz);
}

// compute units of the current device; if it cannot be queried, those of a whole MI355X
static int compute_units() {
    int dev = 0, ncu = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && ncu > 0)
        return ncu;
    (void)hipGetLastError();
    return 256;
}

static thread_local char g_last_error[256] = "";

int lbm_note(hipError_t e) {
    if (e == hipSuccess) return LBM_OK;
    std::snprintf(g_last_error, sizeof(g_last_error), "%s: %s", hipGetErrorName(e), hipGetErrorString(e));
    return LBM_EDEVICE;
}

static int hip_status(hipError_t e) { return lbm_note(e); }

static int last_launch() { return hip_status(hipGetLastError()); }

template <class C> static Phys<C> make_phys(const lbm_params &p) {
    Phys<C> ph;
    ph.a = (C)p.a; ph.b = (C)p.b; ph.R = (C)p.R; ph.cv = (C)p.cv;
    ph.mu = (C)p.mu; ph.eta = (C)p.eta; ph.k = (C)p.k; ph.kappa = (C)p.kappa;
    ph.inv_cv = (C)(1.0 / p.cv);
    ph.k_over_mu = (C)(p.k / p.mu);
    ph.eta_over_mu = (C)(p.eta / p.mu);
    ph.sgn_eps = (C)p.upwind_eps;
    ph.sc_cmu = (C)p.sc_cmu;
    ph.sc_ceta = (C)p.sc_ceta;
    ph.sc_ck = (C)p.sc_ck;
    ph.pr = lbm_eos_is_pr(p.eos) ? 1 : 0;
    ph.pr_m = p.pr_m;
    ph.pr_Tc = p.pr_Tc;
    ph.pr_c0 = p.pr_c0;
    ph.pr_c1 = p.pr_c1;
    return ph;
}

// reference populations of the 16-bit forms: rest equilibria at (ref_rho,
// ref_T) (Psi(0) = 1 - theta, Psi(+-1) = theta/2 at u = 0), computed in FP64.
static void make_ref(const lbm_params &p, int D, RefPops &ref) {
    std::memset(&ref, 0, sizeof(ref));
    if (!(p.ref_rho > 0 && p.ref_T > 0)) return;
    double r = p.ref_rho, t = p.ref_T;
    double P = r * p.R * t / (1.0 - p.b * r) - p.a * r * r;
    double th = P / r;
    double e = p.cv * t - p.a * r;
    int Q = D == 2 ? 9 : 27;
    // per axis at u = 0: p(0) = 1 - th, p(+-1) = th/2; q(0) = th - 3 th^2,
    // q(+-1) = 3 th^2 / 2
    for (int i = 0; i < Q; i++) {
        int cc[3] = {cx_of(i), cy_of(i), D == 3 ? cz_of(i) : 0};
        double pa[3], qa[3];
        for (int a = 0; a < D; a++) {
            pa[a] = cc[a] ? 0.5 * th : 1.0 - th;
            qa[a] = cc[a] ? 1.5 * th * th : th - 3.0 * th * th;
        }
        double prod = 1.0, s = 0.0;
        for (int a = 0; a < D; a++) prod *= pa[a];
        for (int b = 0; b < D; b++) {
            double t2 = qa[b];
            for (int a = 0; a < D; a++)
                if (a != b) t2 *= pa[a];
            s += t2;
        }
        double feq = r * prod;
        ref.f[i] = (float)feq;
        ref.g[i] = (float)(feq * (e - 0.5 * D * th) + 0.5 * r * s);
    }
}

// ---------------------------------------------------------------------------
// dispatch over (lattice, storage)
// ---------------------------------------------------------------------------
// tile of the fused step.  The FP32 and 16-bit forms take a wide 64 x 4 tile
// (fewer x-shifted row fragments per plane; measured faster than 32 x 8 for
// FP32 and, fix-up pass included, for BF16).  FP64, bound by arithmetic and by
// latency, takes 32 x 8: the fewest ring cells per cell of 256 (a 16 x 8 tile
// left two of a compute unit's four SIMDs idle).
template <class S, bool MLP>
using TileOf = typename std::conditional<std::is_same<S, StoreF64>::value, Tile<32, 8>, Tile<64, 4>>::type;

template <int D, class S> struct Impl {
    using C = typename S::C;
    using T = typename S::T;
    // the fused step's surrogate form (van der Waals with the network)
    static bool mlp(const lbm_ctx *c) { return std::is_same<C, float>::value && c->p.eos == LBM_EOS_MLP; }

    // complete moments of the current state into the side channel's plane
    // layers (a step writes every other layer before the fix-up reads it);
    // inbound slots of both buffers start at zero (slots behind a zero-gradient
    // wall are never written afterwards, the fix-up pass adds them as zeros)
    static int fused_prepare(lbm_ctx *c) { return mlp(c) ? fused_prepare_t<true>(c) : fused_prepare_t<false>(c); }
    template <bool M> static int fused_prepare_t(lbm_ctx *c) {
        using TL = TileOf<S, M>;
        if (!c->fused || c->b2_threads) return LBM_OK;
        for (int s = 0; s < 2; s++)
            if (hipMemsetAsync(c->IN[s], 0, c->in_bytes, c->stream) != hipSuccess)
                return lbm_note(hipGetLastError());
        C rs[4];
        ref_sums(c, rs);
        const bool thin_x = c->p.nx % TL::TX == 1, thin_y = c->p.ny % TL::TY == 1;
        if (thin_x) thin_y ? moments_replay<TL, 3, 3>(c, rs) : moments_replay<TL, 3, 2>(c, rs);
        else thin_y ? moments_replay<TL, 2, 3>(c, rs) : moments_replay<TL, 2, 2>(c, rs);
        c->mc_pending = false;
        return last_launch();
    }
    template <class TL, int NX, int NY> static void moments_replay(lbm_ctx *c, const C rs[4]) {
        hipLaunchKernelGGL((k_fused_moments<D, S, TL, NX, NY>), flat_grid(c), dim3(BX), 0, c->stream, c->grid, c->ref,
                           rs[0], rs[1], rs[2], rs[3], c->nseg, (const T *)c->f[c->cur], (C *)c->Mc[c->mcc],
                           c->pulled);
    }
    // sums of the reference populations in the compute type as hi + lo
    // pairs {f_hi, f_lo, g_hi, g_lo} (FP64 sums of the stored references)
    static void ref_sums(const lbm_ctx *c, C rs[4]) {
        double sf = 0, sg = 0;
        for (int i = 0; i < c->Q; i++) {
            sf += (double)(C)c->ref.f[i];
            sg += (double)(C)c->ref.g[i];
        }
        rs[0] = (C)sf;
        rs[1] = (C)(sf - (double)rs[0]);
        rs[2] = (C)sg;
        rs[3] = (C)(sg - (double)rs[2]);
    }
    // full tiles and periodic x, y: the instance without wall and
    // partial-tile handling.  With 16-bit storage and the explicit EOS that
    // instance also completes its input moments itself (kfold) and on D3Q27
    // needs z segments of at least 6 planes; shorter ones take the general
    // instance.
    static constexpr bool fold_storage = sizeof(T) == 2;
    template <bool M> static bool fast_instance(const lbm_ctx *c) {
        using TL = TileOf<S, M>;
        const bool fast = c->p.nx % TL::TX == 0 && c->p.ny % TL::TY == 0 && c->p.bc[0] == LBM_BC_PERIODIC &&
                          c->p.bc[1] == LBM_BC_PERIODIC;
        if (!fast || M || !fold_storage || D == 2) return fast;
        return c->p.nz / c->nseg >= 6;
    }
    // D2Q9: every instance, on tiles of at least 2 x 2 cells
    static bool kfold(const lbm_ctx *c) {
        using TL = TileOf<S, false>;
        if (mlp(c) || !c->fused || c->b2_threads) return false;
        return D == 2 ? c->p.nx % TL::TX != 1 && c->p.ny % TL::TY != 1 : fold_storage && fast_instance<false>(c);
    }
    // the fused step proper (kind 0 of step_timed)
    static void fused_main(lbm_ctx *c) { mlp(c) ? fused_main_t<true>(c) : fused_main_t<false>(c); }
    template <bool M> static void fused_main_t(lbm_ctx *c) {
        using TL = TileOf<S, M>;
        FusedArgs<C, T> a;
        a.g = c->grid;
        a.ph = make_phys<C>(c->p);
        a.ref = c->ref;
        a.ntx = c->ntx;
        a.nty = c->nty;
        a.nseg = c->nseg;
        a.nsub = c->nsub;
        a.nlay = c->nlay;
        a.chunk = c->chunk;
        a.pull = c->pulled;
        {
            C rs[4];
            ref_sums(c, rs);
            a.rsf_hi = rs[0];
            a.rsf_lo = rs[1];
            a.rsg_hi = rs[2];
            a.rsg_lo = rs[3];
        }
        const int nxt = 1 - c->cur;
        a.fi = (const T *)c->f[c->cur];
        a.fo = (T *)c->f[nxt];
        a.Mci = (const C *)c->Mc[c->mcc];
        a.Mco = (C *)c->Mc[1 - c->mcc];
        a.INo = (C *)c->IN[1 - c->mcc];
        a.INi = (const C *)c->IN[c->mcc];
        a.Tin = (const C *)c->Tsur;
        a.Acc = (const unsigned *)c->Acc;
        a.accw = 2 * ((c->p.nx + 63) / 64);
        a.inv_cv_d = 1.0 / (double)(float)c->p.cv;
        const dim3 grid((unsigned)(c->ntx * c->nty * c->nseg * c->nsub));
        constexpr bool SUR = M && std::is_same<C, float>::value;
        // Three instances are scheduled better with the tests of the shared marches
        // in them and are taken with them always (us per step of lattices that do
        // not share, without and with): the general one of FP64 (100 x 75 x 60
        // cells 132.6 and 130.6, 200 x 200 x 100 995 and 976), the full-tile ones
        // of FP16 with the explicit EOS (256^3 1297 and 1255) and of FP32 with the
        // surrogate (256^3 2197 and 2181).  The others without (full tiles, FP32
        // 128^3 258 and 276, FP64 128^3 481 and 487; general, FP16 250 x 200 x 100
        // 536 and 556).
        auto launch = [&](auto FAST, auto FOLD) {
            constexpr bool always = D == 3 && (FAST.value ? (M ? std::is_same<S, StoreF32>::value
                                                               : std::is_same<S, StoreF16>::value)
                                                          : std::is_same<S, StoreF64>::value);
            if (D == 3 && (always || c->nsub > 1))
                hipLaunchKernelGGL((k_fused<D, S, TL, SUR, FAST.value, FOLD.value, D == 3>), grid, dim3(TL::NT), 0,
                                   c->stream, a);
            else
                hipLaunchKernelGGL((k_fused<D, S, TL, SUR, FAST.value, FOLD.value, always>), grid, dim3(TL::NT), 0,
                                   c->stream, a);
        };
        constexpr std::integral_constant<bool, !M && (D == 2 || fold_storage)> folding{};
        constexpr std::integral_constant<bool, !M && D == 2> folding_general{};
        if (fast_instance<M>(c)) launch(std::true_type(), folding);
        else if (folding_general.value && !kfold(c)) launch(std::false_type(), std::false_type());
        else launch(std::false_type(), folding_general);
        c->cur = nxt;
        c->pulled = 1;
        c->mc_pending = true;
    }
    // the surrogate pass completes the side channel itself (the fix-up's
    // work): the surrogate form on 64 x 4 tiles, every tile at least 2 x 2
    static bool fold(const lbm_ctx *c) {
        return mlp(c) && c->p.nx >= 2 && c->p.ny >= 2 && c->p.nx % 64 != 1 && c->p.ny % 4 != 1;
    }
    // completes the output moments (kind 1 of step_timed) and flips the state;
    // after a folding step only the segment-end planes (the next step adds
    // the perimeter cells' slots on load).  In the surrogate form with the
    // completion in its pass, only the segment-end planes too, and the state
    // stays pending: the pass adds the perimeter cells' slots and writes the
    // complete moments to the other buffer.
    static void fused_fixup(lbm_ctx *c) { mlp(c) ? fused_fixup_t<true>(c) : fused_fixup_t<false>(c); }
    template <bool M> static void fused_fixup_t(lbm_ctx *c) {
        using TL = TileOf<S, M>;
        if (!c->mc_pending) return;
        const int nxt = 1 - c->mcc;
        const int rows0 = fold(c) || kfold(c) ? 0 : c->p.nz, ends = D == 3 ? 2 * c->nseg : 0;
        const long long per = (long long)c->ntx * c->nty * TL::PMAX, plane = (long long)c->p.nx * c->p.ny;
        // rows of the perimeter cells, then segment ends [e0, e0 + erows)
        auto launch = [&](int rows, int e0, int erows) {
            if (rows + erows == 0) return;
            const long long n = std::max(rows ? per : 0, erows ? plane : 0);
            hipLaunchKernelGGL((k_fused_fixup<D, TL, C>), dim3((unsigned)((n + BX - 1) / BX), (unsigned)(rows + erows)),
                               dim3(BX), 0, c->stream, c->grid, c->ntx, c->nty, c->nseg, rows, e0, (C *)c->Mc[nxt],
                               (const C *)c->IN[nxt]);
        };
        constexpr int MAX_ROWS = 65535;  // of a grid's second extent
        if (rows0 + ends <= MAX_ROWS) {
            launch(rows0, 0, ends);
        } else {  // tall lattices of many segments
            launch(rows0, 0, 0);
            for (int e0 = 0; e0 < ends; e0 += MAX_ROWS) launch(0, e0, std::min(MAX_ROWS, ends - e0));
        }
        if (fold(c)) return;
        c->mcc = nxt;
        c->mc_pending = false;
    }
    // surrogate form: T of every cell by the network pass (kind 2 of
    // step_timed), ahead of the fused step that reads it
    static void fused_eos(lbm_ctx *c) {
        if constexpr (std::is_same<C, float>::value) {
            if (!mlp(c)) return;
            const int zchunk = c->zchunk;
            const dim3 grid((unsigned)((c->p.nx + 63) / 64), (unsigned)((c->p.ny + 3) / 4),
                            (unsigned)((c->p.nz + zchunk - 1) / zchunk));
            FoldArgs fa{nullptr, nullptr, c->ntx, c->nty, c->nseg};
            if (fold(c) && c->mc_pending) {
                // partial sums and slots of the last fused step in (its
                // segment-end planes completed by the fix-up), complete
                // moments out to the buffer that step read
                fa.IN = (const float *)c->IN[1 - c->mcc];
                fa.Mco = (float *)c->Mc[c->mcc];
                hipLaunchKernelGGL((k_eos_surrogate<D, true>), grid, dim3(256), 0, c->stream, c->grid,
                                   make_phys<float>(c->p), (const float *)c->Mc[1 - c->mcc], (float *)c->Tsur,
                                   c->mlp_params, c->mlp_w2b, c->mlp_norm, (float)c->p.mlp_tol, c->mlp_counters,
                                   zchunk, fa, (unsigned long long *)c->Acc);
                c->mc_pending = false;
            } else {
                hipLaunchKernelGGL((k_eos_surrogate<D, false>), grid, dim3(256), 0, c->stream, c->grid,
                                   make_phys<float>(c->p), (const float *)c->Mc[c->mcc], (float *)c->Tsur,
                                   c->mlp_params, c->mlp_w2b, c->mlp_norm, (float)c->p.mlp_tol, c->mlp_counters,
                                   zchunk, fa, (unsigned long long *)c->Acc);
            }
        }
    }
    static void fused_launch(lbm_ctx *c) {
        fused_eos(c);
        fused_main(c);
        fused_fixup(c);
    }

    // counts of non-finite and inadmissible cells of the inputs (blocking)
    static int check_inputs(lbm_ctx *c, const double *rho, const double *u, const double *Tf) {
        hipLaunchKernelGGL((k_check_inputs<D>), dim3(READ_BLOCKS), dim3(BX), 0, c->stream,
                           (long long)c->grid.N, make_phys<double>(c->p), rho, u, Tf, c->red_partials);
        hipLaunchKernelGGL(k_reduce_final, dim3(1), dim3(64 * RED_VALS), 0, c->stream, READ_BLOCKS, c->red_partials,
                           c->red_out);
        int rc = last_launch();
        if (rc) return rc;
        double tmp[RED_VALS];
        if (hipMemcpyAsync(tmp, c->red_out, sizeof(tmp), hipMemcpyDeviceToHost, c->stream) != hipSuccess ||
            hipStreamSynchronize(c->stream) != hipSuccess)
            return lbm_note(hipGetLastError());
        return tmp[5] > 0 ? LBM_ENAN : (tmp[6] > 0 ? LBM_EUNSTABLE : LBM_OK);
    }
    static int init(lbm_ctx *c, const double *rho, const double *u, const double *Tf) {
        int rc0 = check_inputs(c, rho, u, Tf);
        if (rc0) return rc0;
        hipLaunchKernelGGL((k_init<D, S>), flat_grid(c), dim3(BX), 0, c->stream, c->grid, make_phys<double>(c->p),
                           c->ref, rho, u, Tf, (T *)c->f[c->cur], form_flag(c, c->cur));
        c->pulled = 0;
        int rc = last_launch();
        return rc ? rc : fused_prepare(c);
    }
    // the form flag of buffer b (null where the host's flag holds), the form of
    // the current set
    static int *form_flag(const lbm_ctx *c, int b) { return c->form ? (int *)c->form + 16 * b : nullptr; }
    static SetForm set_form(const lbm_ctx *c) { return SetForm{c->pulled, form_flag(c, c->cur)}; }
    static MomSrc<C> field_moments(lbm_ctx *c) {
        return MomSrc<C>{get_fields<C>(c).rho, (long long)c->p.nx * c->p.ny, (long long)c->grid.N, D + 1};
    }
    // moments and fields of every cell (multi-kernel step)
    static int fields_pass(lbm_ctx *c) {
        moments_launch(c);
        lap_launch(c, field_moments(c));
        const int rc = fields_launch(c);
        return rc ? rc : last_launch();
    }
    static void moments_launch(lbm_ctx *c) {
        hipLaunchKernelGGL((k_moments<D, S>), flat_grid(c), dim3(BX), 0, c->stream, c->grid, c->ref,
                           (const T *)c->f[c->cur], get_fields<C>(c), set_form(c));
    }
    static void lap_launch(lbm_ctx *c, const MomSrc<C> &m) {
        hipLaunchKernelGGL((k_lap<D, C>), flat_grid(c), dim3(BX), 0, c->stream, c->grid, m, get_fields<C>(c).lap);
    }
    static bool warm_start(const lbm_ctx *c) { return c->p.eos == LBM_EOS_PR_PREV && c->T_valid; }
    static int fields_launch(lbm_ctx *c) {
        int rc = LBM_OK;
        if (lbm_eos_uses_mlp(c->p.eos)) rc = launch_fields_mlp<D, C>(c, get_fields<C>(c));
        else
            hipLaunchKernelGGL((k_fields<D, C>), flat_grid(c), dim3(BX), 0, c->stream, c->grid, make_phys<C>(c->p),
                               field_moments(c), get_fields<C>(c), warm_start(c) ? 1 : 0, c->mlp_counters);
        c->T_valid = true;
        return rc;
    }
    // The moments of the current state for a read-back.  The fused step's side
    // channel holds them (20 bytes per cell against the 2 Q populations that
    // k_moments reads, 5.1 ms at 512^3 cells in BF16); where the next step would
    // complete them on load, k_complete does so into the field arrays (1.5 ms).
    static MomSrc<C> state_moments(lbm_ctx *c) {
        if (!c->fused || c->b2_threads) {
            moments_launch(c);
            return field_moments(c);
        }
        const long long plane = (long long)c->p.nx * c->p.ny;
        const bool pending = c->mc_pending;  // surrogate form: its pass completes them
        const int at = pending ? 1 - c->mcc : c->mcc;
        if (!pending && !kfold(c)) return MomSrc<C>{(const C *)c->Mc[at], 5 * plane, plane, 4};
        using TL = TileOf<S, false>;
        static_assert(std::is_same<TL, TileOf<S, true>>::value, "one tile for both forms");
        hipLaunchKernelGGL((k_complete<D, TL, C>), flat_grid(c), dim3(BX), 0, c->stream, c->grid, c->ntx, c->nty,
                           c->nseg, (const C *)c->Mc[at], (const C *)c->IN[at], get_fields<C>(c));
        return field_moments(c);
    }
    // rho, u, T, P to the caller's arrays (any null) or the conservation sums
    // to the partials
    static int read_back(lbm_ctx *c, const ReadOut &o) {
        const MomSrc<C> m = state_moments(c);
        lap_launch(c, m);
        Fields<C> fl = get_fields<C>(c);
        if (lbm_eos_uses_mlp(c->p.eos)) {
            const int rc = launch_readback_mlp<D, C>(c, m, fl, o);
            if (rc) return rc;
        } else {
            const int warm = warm_start(c) ? 1 : 0;
            if (o.partials)
                hipLaunchKernelGGL((k_readback<D, C, true>), dim3(READ_BLOCKS), dim3(BX), 0, c->stream, c->grid,
                                   make_phys<C>(c->p), m, fl.lap, fl.T, warm, o);
            else
                hipLaunchKernelGGL((k_readback<D, C, false>), dim3(READ_BLOCKS), dim3(BX), 0, c->stream, c->grid,
                                   make_phys<C>(c->p), m, fl.lap, fl.T, warm, o);
            c->T_valid = c->T_valid || lbm_eos_is_pr(c->p.eos);
        }
        return last_launch();
    }
    // shock-capturing passes over the fields of the step; returns the filtered
    // (|grad^4 S|, |grad^4 |grad s||) arrays, or nulls when the scheme is off
    static void sc_passes(lbm_ctx *c, const C **fS, const C **fs) {
        *fS = *fs = nullptr;
        if (!c->sc) return;
        Fields<C> fl = get_fields<C>(c);
        const dim3 gr = flat_grid(c);
        hipLaunchKernelGGL((k_sc_grad<D, C>), gr, dim3(BX), 0, c->stream, c->grid, make_phys<C>(c->p), fl);
        hipLaunchKernelGGL((k_sc_d4<D, C>), gr, dim3(BX), 0, c->stream, c->grid, fl.sc[0], fl.sc[1], fl.sc[2],
                           fl.sc[3]);
        // filter weights exp(-j^2 / (2 sigma^2)), |j| <= 4, sigma = 1.2, normalised
        ScFilter<C> f;
        double w[2 * SC_RADIUS + 1], ws = 0;
        for (int j = -SC_RADIUS; j <= SC_RADIUS; j++) ws += (w[j + SC_RADIUS] = std::exp(-(double)(j * j) / 2.88));
        for (int j = 0; j <= 2 * SC_RADIUS; j++) f.w[j] = (C)(w[j] / ws);
        int src = 2;
        for (int a = 0; a < D; a++) {
            const int dst = 2 - src;
            hipLaunchKernelGGL((k_sc_filter<D, C>), gr, dim3(BX), 0, c->stream, c->grid, a, f, fl.sc[src],
                               fl.sc[src + 1], fl.sc[dst], fl.sc[dst + 1]);
            src = dst;
        }
        *fS = fl.sc[src];
        *fs = fl.sc[src + 1];
    }
    static Walls walls(const lbm_ctx *c) {
        Walls w;
        for (int s = 0; s < 2; s++) {
            for (int a = 0; a < 3; a++) w.u[s][a] = c->p.wall_u[s][a];
            w.T[s] = c->p.wall_T[s];
        }
        return w;
    }
    // collide into buffer nxt (multi-kernel path): the post-collision set, or
    // with x walls the arrived one and then what the wall ghosts emit
    static void collide_launch(lbm_ctx *c, Fields<C> fl, const C *fS, const C *fs, int nxt) {
        const Walls w = walls(c);
        if (c->grid.wallx)
            hipLaunchKernelGGL((k_collide<D, S, true>), flat_grid(c), dim3(BX), 0, c->stream, c->grid,
                               make_phys<C>(c->p), c->ref, (const T *)c->f[c->cur], fl, (T *)c->f[nxt], fS, fs, w,
                               (C *)c->ghost, set_form(c), form_flag(c, nxt));
        else
            hipLaunchKernelGGL((k_collide<D, S, false>), flat_grid(c), dim3(BX), 0, c->stream, c->grid,
                               make_phys<C>(c->p), c->ref, (const T *)c->f[c->cur], fl, (T *)c->f[nxt], fS, fs, w,
                               (C *)c->ghost, set_form(c), form_flag(c, nxt));
        if (c->grid.wallx)
            hipLaunchKernelGGL((k_wall_emit<D, S>), dim3((unsigned)((c->p.ny + 63) / 64), (unsigned)c->p.nz, 2u),
                               dim3(64), 0, c->stream, c->grid, make_phys<C>(c->p), c->ref, w, fl,
                               (const C *)c->ghost, (T *)c->f[nxt], (T *)c->g[nxt]);
    }
    // Whether and how small D2Q9 lattices take several steps in one launch.  A
    // region has at most 1024 cells (FP32; 128 registers per thread) or 512
    // (FP64, x walls).  The whole lattice where it fits (us per step, FP64 and
    // FP32: 64 x 4 cells 1.6 and 1.3, fused 8.8 and 8.9; with x walls 2.6 and
    // 2.4, multi-kernel 20); else all rows of `own` columns and a halo of 4 per
    // step, by the shortest time per step of the model below (4 us per launch,
    // then a step's latency, which grows with the wavefronts per SIMD: fitted to
    // those and 512 x 4 2.1 and 1.8, 1000 x 4 2.2 and 1.9, 400 x 16 3.7 and 3.1,
    // 800 x 32 FP32 5.1; x walls, up to 1 us longer, take the same numbers).  It
    // is taken below 8 us, with x walls below 16: a step of the other path takes
    // 9 us and more there, 20 and more.  Up to 64 (32) rows, a choice: a region
    // of one step would fit up to 85 (42), but from 64 (32) on most of it is
    // halo and little is gained (us per step, other path against this one: FP32
    // 64 x 64 10.6 and 6.2, 1000 x 64 11.5 and 9.8, 2048 x 64 13.5 and 11.0;
    // FP64 1000 x 32 12.2 and 10.3; x walls 4096 x 32 FP32 23.4 and 15.0, FP64
    // 28.9 and 18.6).
    static void block2d_plan(lbm_ctx *c) {
        c->b2_threads = 0;
        const bool wide = std::is_same<C, double>::value;
        if (D != 2 || sizeof(T) == 2 || c->p.eos != LBM_EOS_VDW || c->sc || (!c->fused && !c->grid.wallx)) return;
        const int cap = wide || c->grid.wallx ? 512 : 1024, nx = c->p.nx, ny = c->p.ny;
        auto plan = [&](int threads, int own, int halo, int steps) {
            c->b2_threads = threads;
            c->b2_own = own;
            c->b2_halo = halo;
            c->b2_steps = steps;
        };
        if ((long long)nx * ny <= cap) return plan(nx * ny, nx, 0, 1024);
        if (ny > cap / 16) return;
        const double launch = 4.0, base = wide ? 1.0 : 0.95, per = wide ? 0.65 : 0.45;
        const int ncu = compute_units();
        double best = c->grid.wallx ? 16.0 : 8.0;
        for (int k = 1; k <= 16; k++)
            for (int own = 4; (own + 8 * k) * ny <= cap; own += 4) {
                const int threads = (own + 8 * k) * ny;
                const double rounds = std::ceil(((nx + own - 1) / own) / (double)ncu);
                const double t = rounds * (launch / k + base + per * ((threads + 255) / 256));
                if (t >= best) continue;
                best = t;
                plan(threads, own, 4 * k, k);
            }
    }
    template <bool WALL, int NT> static void block2d_run(lbm_ctx *c, int steps) {
        if constexpr (D == 2 && sizeof(T) != 2) {
            Block2DArgs<C, T> a;
            a.g = c->grid;
            a.ph = make_phys<C>(c->p);
            a.ref = c->ref;
            a.w = walls(c);
            a.own = c->b2_own;
            a.halo = c->b2_halo;
            a.steps = steps;
            a.pull = c->pulled;
            C rs[4];
            ref_sums(c, rs);
            a.rsf_hi = rs[0];
            a.rsf_lo = rs[1];
            a.rsg_hi = rs[2];
            a.rsg_lo = rs[3];
            a.fi = (const T *)c->f[c->cur];
            a.fo = (T *)c->f[1 - c->cur];
            hipLaunchKernelGGL((k_block2d<S, WALL, NT>), dim3((unsigned)((c->p.nx + a.own - 1) / a.own)),
                               dim3((unsigned)((c->b2_threads + 63) / 64 * 64)), 0, c->stream, a);
        }
    }
    // at most b2_steps steps
    static void block2d_launch(lbm_ctx *c, int steps) {
        constexpr int BIG = std::is_same<C, double>::value ? 512 : 1024;
        const bool small = c->b2_threads <= 256;
        if (c->grid.wallx) small ? block2d_run<true, 256>(c, steps) : block2d_run<true, 512>(c, steps);
        else small ? block2d_run<false, 256>(c, steps) : block2d_run<false, BIG>(c, steps);
        c->cur = 1 - c->cur;
        c->pulled = c->grid.wallx ? 0 : 1;
    }
    static int block2d_step(lbm_ctx *c, int n) {
        const long long every = c->p.check_every;
        while (n > 0) {
            // the steps up to the next check
            int m = every > 0 ? (int)std::min<long long>(n, every - c->steps_done % every) : n;
            n -= m;
            // As many launches, or one more, as turn the two buffers like m
            // single steps would: a captured call of an even number of steps
            // ends in the buffer it began in and can be replayed, as on the
            // other paths.
            int launches = (m + c->b2_steps - 1) / c->b2_steps;
            if ((launches ^ m) & 1) launches++;
            for (; m > 0; launches--) {
                const int k = (m + launches - 1) / launches;
                block2d_launch(c, k);
                const int rc = last_launch();
                if (rc) return rc;
                m -= k;
                c->steps_done += k;
            }
            if (every > 0 && c->steps_done % every == 0) {
                double tmp[RED_VALS];
                const int rc = conservation(c, tmp);
                if (rc) return rc;
            }
        }
        return LBM_OK;
    }
    static int step(lbm_ctx *c, int n) {
        if (c->b2_threads) return block2d_step(c, n);
        Fields<C> fl = get_fields<C>(c);
        for (int s = 0; s < n; s++) {
            int rc;
            if (c->fused) {
                fused_launch(c);
                rc = last_launch();
            } else {
                rc = fields_pass(c);
                if (rc) return rc;
                const C *fS, *fs;
                sc_passes(c, &fS, &fs);
                int nxt = 1 - c->cur;
                collide_launch(c, fl, fS, fs, nxt);
                rc = last_launch();
                c->cur = nxt;
            }
            if (rc) return rc;
            c->steps_done++;
            if (c->p.check_every > 0 && c->steps_done % c->p.check_every == 0) {
                double tmp[RED_VALS];
                rc = conservation(c, tmp);
                if (rc) return rc;
            }
        }
        return LBM_OK;
    }
    // n steps with events between the launches: host_ms[k] receives the
    // average duration of kernel kind k (moments, laplacian, fields, collide)
    static int step_timed(lbm_ctx *c, int n, double *host_ms) {
        hipEvent_t ev[5];
        for (int k = 0; k < 5; k++)
            if (hipEventCreate(&ev[k]) != hipSuccess) return LBM_EDEVICE;
        if (c->b2_threads) {  // one kind, its time per step
            (void)hipEventRecord(ev[0], c->stream);
            int rc = LBM_OK;
            for (int left = n; left > 0 && rc == LBM_OK; left -= c->b2_steps) {
                block2d_launch(c, std::min(left, c->b2_steps));
                rc = last_launch();
            }
            (void)hipEventRecord(ev[1], c->stream);
            float ms = 0;
            if (rc == LBM_OK && (hipEventSynchronize(ev[1]) != hipSuccess ||
                                 hipEventElapsedTime(&ms, ev[0], ev[1]) != hipSuccess))
                rc = LBM_EDEVICE;
            for (int k = 0; k < 5; k++) (void)hipEventDestroy(ev[k]);
            for (int k = 0; k < LBM_NUM_KERNELS; k++) host_ms[k] = k == 0 && n > 0 ? (double)ms / n : 0.0;
            return rc;
        }
        if (c->fused) {
            // kinds: 0 k_fused, 1 k_fused_fixup, 2 k_eos_surrogate
            double acc[3] = {0, 0, 0};
            const int kind_of[3] = {2, 0, 1};
            int rc = LBM_OK;
            for (int s = 0; s < n && rc == LBM_OK; s++) {
                (void)hipEventRecord(ev[0], c->stream);
                fused_eos(c);
                (void)hipEventRecord(ev[1], c->stream);
                fused_main(c);
                (void)hipEventRecord(ev[2], c->stream);
                fused_fixup(c);
                (void)hipEventRecord(ev[3], c->stream);
                rc = last_launch();
                for (int k = 0; k < 3 && rc == LBM_OK; k++) {
                    float ms = 0;
                    if (hipEventSynchronize(ev[k + 1]) != hipSuccess ||
                        hipEventElapsedTime(&ms, ev[k], ev[k + 1]) != hipSuccess)
                        rc = LBM_EDEVICE;
                    acc[kind_of[k]] += ms;
                }
            }
            for (int k = 0; k < 5; k++) (void)hipEventDestroy(ev[k]);
            for (int k = 0; k < LBM_NUM_KERNELS; k++) host_ms[k] = (k < 3 && n > 0) ? acc[k] / n : 0.0;
            if (!mlp(c)) host_ms[2] = 0.0;
            return rc;
        }
        double acc[4] = {0, 0, 0, 0};
        Fields<C> fl = get_fields<C>(c);
        int rc = LBM_OK;
        for (int s = 0; s < n && rc == LBM_OK; s++) {
            (void)hipEventRecord(ev[0], c->stream);
            moments_launch(c);
            (void)hipEventRecord(ev[1], c->stream);
            lap_launch(c, field_moments(c));
            (void)hipEventRecord(ev[2], c->stream);
            rc = fields_launch(c);
            const C *fS, *fs;
            sc_passes(c, &fS, &fs);  // timed with the fields kind
            (void)hipEventRecord(ev[3], c->stream);
            int nxt = 1 - c->cur;
            collide_launch(c, fl, fS, fs, nxt);
            (void)hipEventRecord(ev[4], c->stream);
            if (rc == LBM_OK) rc = last_launch();
            c->cur = nxt;
            if (hipEventSynchronize(ev[4]) != hipSuccess) rc = LBM_EDEVICE;
            for (int k = 0; k < 4 && rc == LBM_OK; k++) {
                float ms = 0;
                if (hipEventElapsedTime(&ms, ev[k], ev[k + 1]) != hipSuccess) rc = LBM_EDEVICE;
                acc[k] += ms;
            }
        }
        for (int k = 0; k < 5; k++) (void)hipEventDestroy(ev[k]);
        for (int k = 0; k < 4; k++) host_ms[k] = n > 0 ? acc[k] / n : 0.0;
        return rc;
    }
    static int moments(lbm_ctx *c, double *rho, double *u, double *Tf, double *P) {
        return read_back(c, ReadOut{rho, u, Tf, P, nullptr});
    }
    static int get_pops(lbm_ctx *c, double *f, double *g) {
        hipLaunchKernelGGL((k_get_pops<D, S>), flat_grid(c), dim3(BX), 0, c->stream, c->grid, c->ref,
                           (const T *)c->f[c->cur], f, g, set_form(c));
        return last_launch();
    }
    static int set_pops(lbm_ctx *c, const double *f, const double *g) {
        hipLaunchKernelGGL((k_set_pops<D, S>), flat_grid(c), dim3(BX), 0, c->stream, c->grid, c->ref, f, g,
                           (T *)c->f[c->cur], form_flag(c, c->cur));
        c->pulled = 0;
        int rc = last_launch();
        return rc ? rc : fused_prepare(c);
    }
    static void tiles(lbm_ctx *c) {
        mlp(c) ? tiles_t<true>(c) : tiles_t<false>(c);
        c->folded = fold(c);
        c->zchunk = eos_chunk(c);
    }
    // Resident workgroups of the fused step: compute units x the kernel's
    // occupancy (of the general instance; on D3Q27 the LDS gives every instance
    // of a storage form the same); 0 if the device cannot be queried
    template <bool M> static long long resident_groups() {
        using TL = TileOf<S, M>;
        int dev = 0, ncu = 0, nb = 0;
        const bool known =
            hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess &&
            hipOccupancyMaxActiveBlocksPerMultiprocessor(
                &nb, k_fused<D, S, TL, M && std::is_same<C, float>::value, false, !M && D == 2, D == 3>, TL::NT, 0) ==
                hipSuccess &&
            ncu > 0 && nb > 0;
        if (!known) (void)hipGetLastError();
        return known ? (long long)ncu * nb : 0;
    }
    // Workgroups per tile and segment.  A march takes about its planes plus four
    // (the prologue), and two planes more where several share a segment; more of
    // them pay where the tiles and segments leave compute units without work
    // (us per step, FP32, 1 against the number taken: 11 x 11 x 28 cells 204
    // against 47, 100 x 75 x 60 166 against 112).
    static int sub_marches(const lbm_ctx *c, long long ntiles, long long res) {
        if (!res) return 1;
        const int planes = (c->p.nz + c->nseg - 1) / c->nseg;
        auto cost = [&](int m) {
            const long long rounds = (ntiles * c->nseg * m + res - 1) / res;
            return rounds * ((planes + m - 1) / m + (m > 1 ? 2 : 0) + 4);
        };
        int best = 1;
        for (int m = 2; m <= planes; m++)
            if (cost(m) < cost(best)) best = m;
        return cost(best) * 20 <= cost(1) * 19 ? best : 1;
    }
    // Planes per workgroup of the surrogate pass.  64 x 4 columns march through
    // the fewest chunks of at most 58 planes, as even as nz allows (longer chunks
    // spread the prologue -- rho region of four planes, two Laplacians, the
    // permuted weights -- over more planes: at 512^3, 32 -> 56 took the pass 2.98
    // -> 2.88 ms, nine chunks of 57 and 56 instead of nine of 56 and one of 8
    // 2.39 -> 2.36 ms; the end-plane bitmask of the completing pass spans a chunk
    // plus 6 planes, at most 64).  Where these leave compute units without work
    // (two workgroups each), the count with the shortest march and its prologue of
    // about five planes; a cell's value does not depend on its chunk.
    static int eos_chunk(const lbm_ctx *c) {
        constexpr int ZCHUNK_MAX = 58;
        static_assert(ZCHUNK_MAX + 6 <= 64, "end-plane bitmask of the surrogate pass");
        const int nz = c->p.nz;
        if (D == 2) return 1;
        int n = (nz + ZCHUNK_MAX - 1) / ZCHUNK_MAX, dev = 0, ncu = 0;
        const long long cols = (long long)((c->p.nx + 63) / 64) * ((c->p.ny + 3) / 4);
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || ncu < 1) {
            (void)hipGetLastError();
        } else if (cols * n < 2 * ncu) {
            auto march = [&](int k) { return ((cols * k + 2 * ncu - 1) / (2 * ncu)) * ((nz + k - 1) / k + 5); };
            for (int k = n + 1; k <= nz; k++)
                if (march(k) < march(n)) n = k;
        }
        return (nz + n - 1) / n;
    }
    template <bool M> static void tiles_t(lbm_ctx *c) {
        using TL = TileOf<S, M>;
        c->ntx = (c->p.nx + TL::TX - 1) / TL::TX;
        c->nty = (c->p.ny + TL::TY - 1) / TL::TY;
        const long long ntiles = (long long)c->ntx * c->nty;
        if (D == 2) {
            c->nseg = 1;
        } else if (c->p.zsegments > 0) {
            c->nseg = c->p.zsegments;
        } else {
            // segments of at least 16 planes; the count minimises the
            // workgroup rounds times the planes per segment (no half-empty
            // last round).  Among equal costs: segments of at least 64
            // planes where there are such (the prologue, about 8 planes of
            // loads, stays small), the first count giving 8 workgroups per
            // resident slot, else the longest of them -- a march of one or
            // two rounds ends on its slowest workgroups (512^3, 16-bit: one
            // segment, two rounds, 9.6 ms; four segments 9.0 ms); without
            // such segments the first count reaching 1024 workgroups.
            // If the device cannot be queried, the first count giving 1024
            // workgroups.
            const int smax = std::max(1, c->p.nz / 16);
            const long long res = resident_groups<M>();
            if (std::is_same<C, double>::value && res && ntiles * smax < res) {
                // FP64 where such segments leave compute units without work:
                // the shortest march with its prologue of about four planes
                // (100 x 75 x 60 cells: 6 segments 146 us per step, 3 shared by
                // two workgroups each 159).  The other forms keep the count,
                // which the last bits of their sums depend on.
                const int nz = c->p.nz;
                auto march = [&](int s) { return ((ntiles * s + res - 1) / res) * ((nz + s - 1) / s + 4); };
                c->nseg = 1;
                for (int s = 2; s <= std::max(1, nz / 4); s++)
                    if (march(s) < march(c->nseg)) c->nseg = s;
            } else if (!res) {
                c->nseg = std::max(1, std::min((int)((1024 + ntiles - 1) / ntiles), smax));
            } else {
                const int nz = c->p.nz;
                auto cost = [&](int s) { return ((ntiles * s + res - 1) / res) * ((nz + s - 1) / s); };
                long long best_cost = -1;
                for (int s = 1; s <= smax; s++) best_cost = best_cost < 0 ? cost(s) : std::min(best_cost, cost(s));
                int best = -1;
                for (int s = 1; s <= smax && nz / s >= 64; s++) {
                    if (cost(s) != best_cost) continue;
                    best = s;
                    if (ntiles * s >= 8 * res) break;
                }
                if (best < 0) {
                    for (int s = 1; s <= smax; s++) {
                        if (cost(s) != best_cost) continue;
                        best = s;
                        if (ntiles * s >= 1024) break;
                    }
                }
                c->nseg = best;
            }
        }
        c->nlay = D == 3 ? c->p.nz + 2 * c->nseg : 1;
        c->nsub = D == 3 ? sub_marches(c, ntiles, resident_groups<M>()) : 1;
        const long long total = ntiles * c->nseg * c->nsub;
        c->chunk = total % 8 == 0 ? (int)(total / 8) : 0;
        c->mc_bytes = sizeof(C) * 5 * (size_t)c->nlay * c->p.nx * c->p.ny;
        c->in_bytes = sizeof(C) * (size_t)ntiles * c->nlay * 5 * TL::NR;
    }
    static int conservation(lbm_ctx *c, double *host_out) {
        int rc = read_back(c, ReadOut{nullptr, nullptr, nullptr, nullptr, c->red_partials});
        if (rc) return rc;
        hipLaunchKernelGGL(k_reduce_final, dim3(1), dim3(64 * RED_VALS), 0, c->stream, READ_BLOCKS, c->red_partials,
                           c->red_out);
        rc = last_launch();
        if (rc) return rc;
        double tmp[RED_VALS];
        if (hipMemcpyAsync(tmp, c->red_out, sizeof(tmp), hipMemcpyDeviceToHost, c->stream) != hipSuccess ||
            hipStreamSynchronize(c->stream) != hipSuccess)
            return LBM_EDEVICE;
        host_out[0] = tmp[0];
        for (int a = 0; a < D; a++) host_out[1 + a] = tmp[1 + a];
        host_out[D + 1] = tmp[4];
        host_out[D + 2] = tmp[5];
        host_out[D + 3] = tmp[6];
        return tmp[5] > 0 ? LBM_ENAN : (tmp[6] > 0 ? LBM_EUNSTABLE : LBM_OK);
    }
};

#define DISPATCH(ctx, CALL)                                                                    \
    do {                                                                                       \
        const int st_ = (ctx)->p.storage;                                                      \
        if ((ctx)->D == 2) {                                                                   \
            if (st_ == LBM_STORE_F64) return Impl<2, StoreF64>::CALL;                          \
            if (st_ == LBM_STORE_F32) return Impl<2, StoreF32>::CALL;                          \
            if (st_ == LBM_STORE_BF16) return Impl<2, StoreBF16>::CALL;                        \
            return Impl<2, StoreF16>::CALL;                                                    \
        }                                                                                      \
        if (st_ == LBM_STORE_F64) return Impl<3, StoreF64>::CALL;                              \
        if (st_ == LBM_STORE_F32) return Impl<3, StoreF32>::CALL;                              \
        if (st_ == LBM_STORE_BF16) return Impl<3, StoreBF16>::CALL;                            \
        return Impl<3, StoreF16>::CALL;                                                        \
    } while (0)

#define DISPATCH_VOID(ctx, CALL)                                                               \
    do {                                                                                       \
        const int st_ = (ctx)->p.storage;                                                      \
        if ((ctx)->D == 2) {                                                                   \
            if (st_ == LBM_STORE_F64) Impl<2, StoreF64>::CALL;                                 \
            else if (st_ == LBM_STORE_F32) Impl<2, StoreF32>::CALL;                            \
            else if (st_ == LBM_STORE_BF16) Impl<2, StoreBF16>::CALL;                          \
            else Impl<2, StoreF16>::CALL;                                                      \
        } else {                                                                               \
            if (st_ == LBM_STORE_F64) Impl<3, StoreF64>::CALL;                                 \
            else if (st_ == LBM_STORE_F32) Impl<3, StoreF32>::CALL;                            \
            else if (st_ == LBM_STORE_BF16) Impl<3, StoreBF16>::CALL;                          \
            else Impl<3, StoreF16>::CALL;                                                      \
        }                                                                                      \
    } while (0)

// ---------------------------------------------------------------------------
// exported entry points
// ---------------------------------------------------------------------------
extern "C" {

const char *lbm_strerror(int s) {
    switch (s) {
        case LBM_OK: return "ok";
        case LBM_EINVAL: return "invalid argument";
        case LBM_ENOMEM: return "device allocation failed";
        case LBM_EDEVICE: return "HIP runtime or kernel launch error";
        case LBM_EUNSTABLE: return "state left the admissible set";
        case LBM_ENAN: return "non-finite value in the state";
        case LBM_ESTATE: return "call out of order";
        default: return "unknown status";
    }
}

static int validate(const lbm_params *p) {
    if (!p) return LBM_EINVAL;
    if (p->lattice != 2 && p->lattice != 3) return LBM_EINVAL;
    if (p->nx < 1 || p->ny < 1 || p->nz < 1) return LBM_EINVAL;
    if (p->lattice == 2 && p->nz != 1) return LBM_EINVAL;
    if (p->ny > 65535 || p->nz > 65535) return LBM_EINVAL;
    for (int a = 0; a < 3; a++)
        if (p->bc[a] != LBM_BC_PERIODIC && p->bc[a] != LBM_BC_ZEROGRAD && !(a == 0 && p->bc[a] == LBM_BC_WALL))
            return LBM_EINVAL;
    if (p->bc[0] == LBM_BC_WALL) {
        if (p->bc[1] != LBM_BC_PERIODIC || p->bc[2] != LBM_BC_PERIODIC) return LBM_EINVAL;
        for (int s = 0; s < 2; s++)
            if (!(p->wall_T[s] > 0) || !std::isfinite(p->wall_u[s][0]) || !std::isfinite(p->wall_u[s][1]) ||
                !std::isfinite(p->wall_u[s][2]))
                return LBM_EINVAL;
    }
    if (p->storage < LBM_STORE_F64 || p->storage > LBM_STORE_F16) return LBM_EINVAL;
    if (p->eos < LBM_EOS_VDW || p->eos > LBM_EOS_PR_MLP) return LBM_EINVAL;
    if (lbm_eos_uses_mlp(p->eos) && p->storage == LBM_STORE_F64) return LBM_EINVAL;
    if (lbm_eos_is_pr(p->eos) && !(p->pr_Tc > 0 && p->pr_c0 > 0 && p->pr_c1 >= 0 && std::isfinite(p->pr_m) &&
                                   p->b > 0 && p->a >= 0))
        return LBM_EINVAL;
    if (!(p->cv > 0) || !(p->mu > 0) || !(p->R > 0)) return LBM_EINVAL;
    if (!(p->upwind_eps >= 0)) return LBM_EINVAL;
    if (p->zsegments < 0 || p->zsegments > p->nz) return LBM_EINVAL;
    if (p->check_every < 0) return LBM_EINVAL;
    if (!(p->sc_cmu >= 0 && p->sc_ceta >= 0 && p->sc_ck >= 0) || !std::isfinite(p->sc_cmu) ||
        !std::isfinite(p->sc_ceta) || !std::isfinite(p->sc_ck))
        return LBM_EINVAL;
    if ((long long)p->nx * p->ny > (1LL << 30)) return LBM_EINVAL;
    if ((p->storage == LBM_STORE_BF16 || p->storage == LBM_STORE_F16) && !(p->ref_rho > 0 && p->ref_T > 0))
        return LBM_EINVAL;
    if (!(p->ref_rho >= 0 && p->ref_T >= 0)) return LBM_EINVAL;
    return LBM_OK;
}

int lbm_create(const lbm_params *params, lbm_ctx **out) {
    if (!out) return LBM_EINVAL;
    *out = nullptr;
    int rc = validate(params);
    if (rc) return rc;
    lbm_ctx *c = new (std::nothrow) lbm_ctx();
    if (!c) return LBM_ENOMEM;
    c->p = *params;
    c->D = params->lattice;
    c->Q = c->D == 2 ? 9 : 27;
    c->stream = (hipStream_t)params->stream;
    c->grid.nx = params->nx; c->grid.ny = params->ny; c->grid.nz = params->nz;
    c->grid.clampx = params->bc[0] != LBM_BC_PERIODIC; c->grid.clampy = params->bc[1]; c->grid.clampz = params->bc[2];
    c->grid.wallx = params->bc[0] == LBM_BC_WALL;
    c->grid.N = (long long)params->nx * params->ny * params->nz;
    const long long N = c->grid.N;
    int sb = params->storage == LBM_STORE_F64 ? 8 : (params->storage == LBM_STORE_F32 ? 4 : 2);
    c->store_bytes = sb;
    int cb = params->storage == LBM_STORE_F64 ? 8 : 4;
    make_ref(*params, c->D, c->ref);
    size_t pop_bytes = (size_t)c->Q * N * sb;
    c->sc = params->sc_cmu > 0 || params->sc_ceta > 0 || params->sc_ck > 0;
    // the single-pass step covers periodic z (and every D = 2 lattice)
    // with the van der Waals equation of state, without shock capturing
    c->fused = (c->D == 2 || params->bc[2] == LBM_BC_PERIODIC) && !c->sc && !lbm_eos_is_pr(params->eos) &&
               params->bc[0] != LBM_BC_WALL;
    if (c->fused) {
        auto tiles = [&]() { DISPATCH_VOID(c, tiles(c)); };
        tiles();
        // its buffer resources (one plane of populations, one side-channel
        // layer, one layer of inbound slots) must stay below 2^31 bytes;
        // larger planes take the multi-kernel path
        const long long plane = (long long)params->nx * params->ny, lim = 1LL << 31;
        if (2LL * c->Q * plane * sb >= lim || 5 * plane * cb >= lim || (long long)(c->in_bytes / c->nlay) >= lim)
            c->fused = false;
    }
    if (!c->fused) c->folded = false;
    auto plan2d = [&]() { DISPATCH_VOID(c, block2d_plan(c)); };
    plan2d();
    auto kfolded = [&]() -> bool { DISPATCH(c, kfold(c)); };
    c->kfolded = kfolded();
    // field arrays: rho, J[D], G, lap (all that a read-back of the fused path
    // uses); the multi-kernel path's also u[D], F[D], Lam[D], T, P, h, cs2, with
    // Peng-Robinson e(rho, T), and the four shock-capturing work arrays when
    // that scheme is on
    size_t nfield = (size_t)(3 + c->D);
    if (!c->fused) nfield += (size_t)(4 + 3 * c->D + (lbm_eos_is_pr(params->eos) ? 1 : 0) + (c->sc ? 4 : 0));
    const size_t field_bytes = nfield * N * cb;
    // The large buffers come from one allocation, carved at 2 MiB boundaries:
    // the population sets (one buffer per ping-pong slot holds both sets, f_i
    // and g_i side by side; the g pointer is the f buffer offset by one
    // element), the field arrays, the wall ghosts, and the fused step's side
    // channel, inbound slots, surrogate temperatures and their acceptance bits;
    // the form flags of the multi-kernel step (with x walls every set is arrived).
    struct Part {
        void **dst;
        size_t bytes;
    };
    const bool mlpT = c->fused && params->eos == LBM_EOS_MLP;
    const Part parts[] = {{&c->f[0], 2 * pop_bytes},
                          {&c->f[1], 2 * pop_bytes},
                          {&c->work, field_bytes},
                          {&c->ghost, c->grid.wallx ? (size_t)2 * params->ny * params->nz * c->Q * cb : 0},
                          {&c->form, !c->fused && !c->grid.wallx ? 2 * 16 * sizeof(int) : 0},
                          {&c->Mc[0], c->fused ? c->mc_bytes : 0},
                          {&c->Mc[1], c->fused ? c->mc_bytes : 0},
                          {&c->IN[0], c->fused ? c->in_bytes : 0},
                          {&c->IN[1], c->fused ? c->in_bytes : 0},
                          {&c->Tsur, mlpT ? sizeof(float) * (size_t)N : 0},
                          {&c->Acc, mlpT ? 8 * (size_t)((params->nx + 63) / 64) * params->ny * params->nz : 0}};
    constexpr size_t ALIGN = (size_t)1 << 21;
    size_t total = 0;
    for (const Part &pt : parts) total += (pt.bytes + ALIGN - 1) / ALIGN * ALIGN;
    bool ok = hipMalloc(&c->block, total) == hipSuccess &&
              hipMalloc((void **)&c->red_partials, sizeof(double) * RED_VALS * READ_BLOCKS) == hipSuccess &&
              hipMalloc((void **)&c->red_out, sizeof(double) * RED_VALS) == hipSuccess &&
              hipMalloc((void **)&c->mlp_counters, LBM_COUNTER_BYTES) == hipSuccess &&
              hipMalloc((void **)&c->mlp_params, sizeof(float) * (LBM_MLP_NPARAMS + 64)) == hipSuccess &&
              hipMalloc((void **)&c->mlp_norm, sizeof(float) * 16) == hipSuccess &&
              hipMalloc((void **)&c->mlp_w2b, sizeof(uint16_t) * 64 * 64) == hipSuccess;
    if (!ok) {
        lbm_note(hipGetLastError());
        lbm_destroy(c);
        return LBM_ENOMEM;
    }
    {
        char *q = (char *)c->block;
        for (const Part &pt : parts) {
            *pt.dst = pt.bytes ? q : nullptr;
            q += (pt.bytes + ALIGN - 1) / ALIGN * ALIGN;
        }
        for (int k = 0; k < 2; k++) c->g[k] = (char *)c->f[k] + sb;
    }
    (void)hipMemsetAsync(c->mlp_counters, 0, LBM_COUNTER_BYTES, c->stream);
    c->cur = 0;
    c->mcc = 0;
    c->mc_pending = false;
    c->initialized = false;
    c->mlp_ready = false;
    *out = c;
    return LBM_OK;
}

void lbm_destroy(lbm_ctx *c) {
    if (!c) return;
    // errors here have nowhere to go (the call returns nothing); the context
    // is released regardless
    if (c->stream) (void)hipStreamSynchronize(c->stream);
    else (void)hipDeviceSynchronize();
    // the large buffers are carved from c->block
    void *ptrs[] = {c->block, c->red_partials, c->red_out, c->mlp_counters, c->mlp_params, c->mlp_norm, c->mlp_w2b};
    for (void *p : ptrs)
        if (p) (void)hipFree(p);
    delete c;
}

static int init_dispatch(lbm_ctx *c, const double *rho, const double *u, const double *Tf) {
    DISPATCH(c, init(c, rho, u, Tf));
}

int lbm_init(lbm_ctx *c, const double *rho, const double *u, const double *Tf) {
    if (!c || !rho || !u || !Tf) return LBM_EINVAL;
    c->cur = 0;
    c->mcc = 0;
    c->mc_pending = false;
    c->initialized = false;
    const int rc = init_dispatch(c, rho, u, Tf);
    c->initialized = rc == LBM_OK;
    c->steps_done = 0;
    c->T_valid = false;
    return rc;
}

int lbm_step(lbm_ctx *c, int n) {
    if (!c) return LBM_EINVAL;
    if (!c->initialized) return LBM_ESTATE;
    if (n < 0) return LBM_EINVAL;
    if (lbm_eos_uses_mlp(c->p.eos) && !c->mlp_ready) return LBM_ESTATE;
    DISPATCH(c, step(c, n));
}

int lbm_moments(lbm_ctx *c, double *rho, double *u, double *Tf, double *P) {
    if (!c) return LBM_EINVAL;
    if (!c->initialized) return LBM_ESTATE;
    if (lbm_eos_uses_mlp(c->p.eos) && !c->mlp_ready) return LBM_ESTATE;
    DISPATCH(c, moments(c, rho, u, Tf, P));
}

int lbm_get_populations(lbm_ctx *c, double *f, double *g) {
    if (!c || !f || !g) return LBM_EINVAL;
    if (!c->initialized) return LBM_ESTATE;
    DISPATCH(c, get_pops(c, f, g));
}

int lbm_set_populations(lbm_ctx *c, const double *f, const double *g) {
    if (!c || !f || !g) return LBM_EINVAL;
    c->initialized = true;
    c->steps_done = 0;
    c->T_valid = false;
    DISPATCH(c, set_pops(c, f, g));
}

int lbm_conservation(lbm_ctx *c, double *host_out) {
    if (!c || !host_out) return LBM_EINVAL;
    if (!c->initialized) return LBM_ESTATE;
    if (lbm_eos_uses_mlp(c->p.eos) && !c->mlp_ready) return LBM_ESTATE;
    DISPATCH(c, conservation(c, host_out));
}

int lbm_synchronize(lbm_ctx *c) {
    if (!c) return LBM_EINVAL;
    return hip_status(c->stream ? hipStreamSynchronize(c->stream) : hipDeviceSynchronize());
}

int lbm_step_timed(lbm_ctx *c, int n, double *host_ms, int nslots) {
    if (!c || !host_ms || n < 0) return LBM_EINVAL;
    if (!c->initialized) return LBM_ESTATE;
    if (lbm_eos_uses_mlp(c->p.eos) && !c->mlp_ready) return LBM_ESTATE;
    if (nslots < LBM_NUM_KERNELS) return LBM_EINVAL;
    DISPATCH(c, step_timed(c, n, host_ms));
}

const char *lbm_last_error(void) { return g_last_error; }

const char *lbm_kernel_name(const lbm_ctx *c, int k) {
    static const char *names[LBM_NUM_KERNELS] = {"k_moments", "k_lap", "k_fields", "k_collide"};
    if (c && c->b2_threads) return k == 0 ? "k_block2d" : "";
    if (c && c->fused)  // folded: the surrogate pass does the fix-up's work but on the segment-end planes
        return k == 0 ? "k_fused"
                      : (k == 1 ? ((c->folded || c->kfolded) && c->p.lattice == 2 ? "" : "k_fused_fixup")
                                : (k == 2 && c->p.eos == LBM_EOS_MLP ? "k_eos_surrogate" : ""));
    return k >= 0 && k < LBM_NUM_KERNELS ? names[k] : "";
}

int lbm_is_fused(const lbm_ctx *c) { return c && c->fused ? 1 : 0; }

double lbm_bytes_per_cell(const lbm_ctx *c) {
    if (!c) return 0.0;
    return 2.0 * 2.0 * c->Q * c->store_bytes;
}

int lbm_hbm_probe(int kind, const void *src, void *dst, int64_t bytes, int blocks_per_cu, int iters, void *stream,
                  double *host_ms) {
    if (kind < 0 || kind > 2 || bytes <= 0 || bytes % 16 || blocks_per_cu < 1 || blocks_per_cu > 64 || iters < 1 ||
        !host_ms || !dst || (kind != 1 && !src))
        return LBM_EINVAL;
    int dev = 0, ncu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || ncu < 1)
        return lbm_note(hipGetLastError());
    hipStream_t s = (hipStream_t)stream;
    const long long n = bytes / 16;
    const dim3 grid((unsigned)(ncu * blocks_per_cu));
    hipEvent_t e0, e1;
    if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) return lbm_note(hipGetLastError());
    auto launch = [&]() {
        if (kind == 0)
            hipLaunchKernelGGL(k_probe_read, grid, dim3(256), 0, s, (const u32x4 *)src, n, (u32x4 *)dst);
        else if (kind == 1)
            hipLaunchKernelGGL(k_probe_write, grid, dim3(256), 0, s, (u32x4 *)dst, n);
        else
            hipLaunchKernelGGL(k_probe_copy, grid, dim3(256), 0, s, (const u32x4 *)src, (u32x4 *)dst, n);
    };
    launch();  // warm-up
    (void)hipEventRecord(e0, s);
    for (int k = 0; k < iters; k++) launch();
    (void)hipEventRecord(e1, s);
    int rc = last_launch();
    float ms = 0;
    if (rc == LBM_OK && (hipEventSynchronize(e1) != hipSuccess || hipEventElapsedTime(&ms, e0, e1) != hipSuccess))
        rc = lbm_note(hipGetLastError());
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    *host_ms = (double)ms / iters;
    return rc;
}

int lbm_codec_encode(int kind, const float *x, const float *ref, uint16_t *out, int64_t n, void *stream) {
    if ((kind != LBM_STORE_BF16 && kind != LBM_STORE_F16) || n < 0) return LBM_EINVAL;
    if (n == 0) return LBM_OK;
    if (!x || !ref || !out) return LBM_EINVAL;
    hipLaunchKernelGGL(k_codec_encode, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, (hipStream_t)stream, kind, x,
                       ref, out, (long long)n);
    return last_launch();
}

int lbm_codec_decode(int kind, const uint16_t *code, const float *ref, float *out, int64_t n, void *stream) {
    if ((kind != LBM_STORE_BF16 && kind != LBM_STORE_F16) || n < 0) return LBM_EINVAL;
    if (n == 0) return LBM_OK;
    if (!code || !ref || !out) return LBM_EINVAL;
    hipLaunchKernelGGL(k_codec_decode, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, (hipStream_t)stream, kind,
                       code, ref, out, (long long)n);
    return last_launch();
}

}  // extern "C"
