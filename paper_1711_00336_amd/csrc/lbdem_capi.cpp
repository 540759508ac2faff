// Host runtime and C ABI of the coupled LBM-DEM library (include/lbdem.h).
// One domain = one set of device arrays on one HIP stream; a step is the
// kernel sequence of Alg. 1 (Rettinger & Ruede, Sec. 3.3), optionally
// captured once into a HIP graph and replayed.
#include "../../include/lbdem.h"
#include "lbdem_internal.h"

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <string>
#include <type_traits>
#include <vector>

using namespace lbdem;

namespace {

thread_local std::string g_thread_err = "";

void *(*g_alloc)(size_t, void *) = nullptr;
void (*g_free)(void *, void *) = nullptr;
void *g_alloc_ctx = nullptr;

struct DevAlloc {
    void *(*alloc)(size_t, void *);
    void (*free_fn)(void *, void *);
    void *ctx;
};

// particles from which the slots are ordered in blocks of cells by default
constexpr int64_t kBlockedFrom = (int64_t)1 << 18;

struct HipError {
    hipError_t e;
    const char *what;
};

inline void hip_check(hipError_t e, const char *what)
{
    if (e != hipSuccess) throw HipError{e, what};
}

struct Oom {
    size_t bytes;
};

// a request the explicit coupling cannot advance stably (LBDEM_E_UNSTABLE)
struct Unstable : std::runtime_error {
    using std::runtime_error::runtime_error;
};

}  // namespace

struct lbdem_domain {
    lbdem_params prm;
    DevAlloc al{};
    hipStream_t stream = nullptr;
    bool own_stream = false;
    int prec = LBDEM_FP64;
    int device = 0;             // the HIP device current at creation
    Geo geo{};
    Phys phys{};
    Tune tune{-1, -1, -1, -1};
    int64_t version = 0;        // bumped whenever captured steps become stale
    std::string err;
    int64_t step_host = 0;

    // cell arrays (one of the two precisions is used)
    void *df[2] = {nullptr, nullptr};
    int cur = 0;
    void *j = nullptr, *uprev = nullptr, *dudt = nullptr, *gradp = nullptr;
    void *epsp = nullptr, *fam = nullptr, *uf = nullptr, *facc = nullptr;
    void *curl = nullptr;       // lift only
    // bins
    int *cnt = nullptr, *start = nullptr, *list = nullptr, *bsum = nullptr, *loc = nullptr;
    int64_t list_cap = 0;
    int64_t nlist_rows = 0;     // particle rows the Verlet-list buffer holds
    // blocked slot order
    Order ord{};
    int64_t ord_rows_cap = 0;
    // particles
    Parts pt{};
    double dmax = 0.0;
    // misc
    int *flags = nullptr;
    long long *stepc = nullptr;
    double *diag_part = nullptr, *diag_out = nullptr, *tmp = nullptr;
    int64_t tmp_len = 0;
    std::vector<void *> owned;

    // captured steps, keyed by (PDF buffer, DEM record buffer)
    bool use_graphs = true;
    int rswap = 0;
    hipGraphExec_t graph[2][2] = {{nullptr, nullptr}, {nullptr, nullptr}};

    // the captured steps no longer hold; a batch finds that out from version
    void drop_graphs()
    {
        version += 1;
        for (auto &row : graph)
            for (auto &g : row)
                if (g) {
                    (void)hipGraphExecDestroy(g);
                    g = nullptr;
                }
    }

    // timing
    bool timing = false;
    struct Ev {
        hipEvent_t a, b;
        int cls;
    };
    std::vector<Ev> ev_pool;
    size_t ev_used = 0;
    double cls_ms[kTimingClasses] = {0};
    int64_t cls_n[kTimingClasses] = {0};

    size_t rsize() const { return prec == LBDEM_FP64 ? sizeof(double) : sizeof(float); }

    void *dalloc(size_t bytes)
    {
        if (bytes == 0) bytes = 256;
        void *p = nullptr;
        if (al.alloc) {
            p = al.alloc(bytes, al.ctx);
            if (!p) throw Oom{bytes};
            // vector loads of packed records and counts assume hipMalloc's alignment
            if (reinterpret_cast<uintptr_t>(p) % 256 != 0) {
                if (al.free_fn) al.free_fn(p, al.ctx);
                throw std::runtime_error("the caller allocator returned a block not aligned to 256 bytes");
            }
        } else {
            hipError_t e = hipMalloc(&p, bytes);
            if (e != hipSuccess) {
                (void)hipGetLastError();
                throw Oom{bytes};
            }
        }
        owned.push_back(p);
        return p;
    }
    void dfree(void *p)
    {
        if (!p) return;
        auto it = std::find(owned.begin(), owned.end(), p);
        if (it != owned.end()) owned.erase(it);
        if (al.free_fn) al.free_fn(p, al.ctx);
        else (void)hipFree(p);
    }

    Desc desc() const
    {
        Desc D{};
        D.g = geo;
        D.p = phys;
        D.t = tune;
        D.b = Bins{cnt, start, list, bsum, loc, flags + 1};
        D.pt = pt;
        D.o = ord;
        // default: the blocked order once the particles outgrow an XCD's cache
        D.t.dem_order = tune.dem_order >= 0 ? tune.dem_order : (pt.np >= kBlockedFrom ? 1 : 0);
        D.flags = flags;
        D.stepc = stepc;
        return D;
    }

    template <typename R>
    Cells<R> cells() const
    {
        Cells<R> C{};
        C.df_src = (R *)df[cur];
        C.df_dst = (R *)df[cur ^ 1];
        C.j = (R *)j;
        C.uprev = (R *)uprev;
        C.un = (R *)fam;
        C.dudt = (R *)dudt;
        C.gradp = (R *)gradp;
        C.epsp = (R *)epsp;
        C.fam = (R *)fam;
        C.uf = (R *)uf;
        C.facc = (R *)facc;
        C.curl = (R *)curl;
        return C;
    }

    double *scratch(int64_t n)
    {
        if (n > tmp_len) {
            dfree(tmp);
            tmp = (double *)dalloc(sizeof(double) * (size_t)n);
            tmp_len = n;
        }
        return tmp;
    }

    void ev_begin(int cls, hipEvent_t &b_out)
    {
        if (ev_used == ev_pool.size()) {
            Ev e{};
            hip_check(hipEventCreate(&e.a), "hipEventCreate");
            hip_check(hipEventCreate(&e.b), "hipEventCreate");
            ev_pool.push_back(e);
        }
        Ev &e = ev_pool[ev_used++];
        e.cls = cls;
        hip_check(hipEventRecord(e.a, stream), "hipEventRecord");
        b_out = e.b;
    }
};

namespace {

lbdem_status fail(lbdem_domain_t h, lbdem_status st, const std::string &msg)
{
    if (h) h->err = msg;
    else g_thread_err = msg;
    return st;
}

template <typename F>
lbdem_status guarded(lbdem_domain_t h, F &&f)
{
    try {
        return f();
    } catch (const HipError &e) {
        return fail(h, LBDEM_E_DEVICE, std::string(e.what) + ": " + hipGetErrorString(e.e));
    } catch (const Oom &o) {
        return fail(h, LBDEM_E_OOM, "device allocation of " + std::to_string(o.bytes) + " bytes failed");
    } catch (const Unstable &e) {
        return fail(h, LBDEM_E_UNSTABLE, e.what());
    } catch (const std::exception &e) {
        return fail(h, LBDEM_E_INVALID, e.what());
    }
}

// timed launch of one kernel class
template <typename F>
void launch_cls(lbdem_domain_t h, int cls, F &&f)
{
    if (!h->timing) {
        f();
        return;
    }
    hipEvent_t b;
    h->ev_begin(cls, b);
    f();
    hip_check(hipEventRecord(b, h->stream), "hipEventRecord");
}

void harvest_timing(lbdem_domain_t h)
{
    for (size_t i = 0; i < h->ev_used; ++i) {
        float ms = 0.f;
        hip_check(hipEventElapsedTime(&ms, h->ev_pool[i].a, h->ev_pool[i].b), "hipEventElapsedTime");
        h->cls_ms[h->ev_pool[i].cls] += ms;
        h->cls_n[h->ev_pool[i].cls] += 1;
    }
    h->ev_used = 0;
}

// constants for n / d = (umulhi(n, m) + n) >> s, valid for 0 <= n < 2^31
void set_fastdiv(uint32_t d, uint32_t &m, uint32_t &s)
{
    s = 0;
    while ((1ull << s) < d) ++s;
    m = (uint32_t)((((uint64_t)1 << 32) * ((1ull << s) - d)) / d + 1);
}

void resolve_phys(lbdem_domain_t h)
{
    const lbdem_params &p = h->prm;
    Phys &P = h->phys;
    P.tau = p.tau;
    P.omega = 1.0 / p.tau;
    P.rho_f = p.rho_f;
    P.mu = p.rho_f * (p.tau - 0.5) / 3.0;  // Eq. visc_tau with tau_e = tau
    for (int a = 0; a < 3; ++a) {
        P.g[a] = p.gravity[a];
        P.fb[a] = p.body_force[a];
    }
    P.e_n = p.e_n;
    P.mu_c = p.mu_c;
    P.h_c = p.h_c;
    P.h_min = p.h_min;
    P.lub_stab = p.lub_stab;
    P.use_lub = p.use_lub;
    P.use_am = p.use_am;
    P.use_lift = p.use_lift ? 1 : 0;
    P.use_eilers = p.use_eilers ? 1 : 0;
    P.use_les = p.use_les ? 1 : 0;
    P.lub_contact = p.lub_contact ? 1 : 0;
    P.n_int = p.n_int;
    P.n_dem = p.n_dem;
    P.dt_int = 1.0 / p.n_int;
    P.dt_dem = P.dt_int / p.n_dem;
    P.T_c = p.T_c > 0.0 ? p.T_c : 20.0 * P.dt_dem;
    // Eq. damping_to_stiffness and Eq. collision_time solved for the pair's
    // k_n and xi_n: k_n = m_ij (pi^2 + ln^2 e_n)/T_c^2, xi_n = -2 ln(e_n) m_ij/T_c
    const double L = std::log(p.e_n);
    P.kn_per_m = (M_PI * M_PI + L * L) / (P.T_c * P.T_c);
    P.xi_per_m = -2.0 * L / P.T_c;
    P.c_am = p.c_am;
    // a particle may move at most `skin` per axis within one subcycle (else the
    // step is flagged unstable); Verlet lists carry `vskin` beyond the
    // interaction reach and are rebuilt ahead of a subcycle in which a particle
    // could get vskin/2 away from where it was at the build, so every pair
    // within reach stays listed (vskin/2 must exceed sqrt(3) skin for lists to
    // outlive a subcycle). A fifth of a tenth of a cell per subcycle is far
    // above the settling speeds of these workloads (1e-4 cells per step at
    // most), and a thin skin keeps the lists close to the pairs within reach.
    P.skin = 0.02;
    P.vskin = 0.1;
    P.rbin = 1;
}

void update_search(lbdem_domain_t h)
{
    Phys &P = h->phys;
    // list build runs on current bins: reach d_max + h_c + Verlet skin
    const double reach = h->dmax + (P.use_lub ? std::max(P.h_c, 0.0) : 0.0) + P.vskin;
    P.reach_max = reach;
    P.rbin = std::max(1, (int)std::ceil(reach));
    if (P.rbin > 8) throw std::runtime_error("interaction reach d_max + h_c exceeds the 8-cell search limit");
}

// block shape of the blocked slot order; (re)allocates the row arrays
void set_order_shape(lbdem_domain_t h, int bx, int by, int bz)
{
    Order &O = h->ord;
    const int ob[3] = {bx, by, bz};
    int64_t rows = (int64_t)ob[1] * ob[2];
    for (int a = 0; a < 3; ++a) {
        O.ob[a] = ob[a];
        O.nb[a] = (h->geo.n[a] + ob[a] - 1) / ob[a];
        rows *= O.nb[a];
    }
    O.nrows = rows;
    if (rows > h->ord_rows_cap) {
        h->dfree(O.rowoff);
        h->dfree(O.rowsum);
        O.rowoff = (int *)h->dalloc(sizeof(int) * (size_t)rows);
        O.rowsum = (int *)h->dalloc(sizeof(int) * (size_t)(rows / kScanPerBlock + 2));
        h->ord_rows_cap = rows;
    }
}

// Verlet-list capacity per particle: twice the mean number of neighbours
// within the list reach (d_max + h_c + skin) at the domain's mean particle
// density, plus 24; a particle with more neighbours raises FLAG_NLIST when a
// step builds its list
void ensure_lists(lbdem_domain_t h)
{
    Parts &P = h->pt;
    const Phys &ph = h->phys;
    const double reach = h->dmax + (ph.use_lub ? std::max(ph.h_c, 0.0) : 0.0) + ph.vskin;
    const double dens = (double)P.np / (double)h->geo.nc;
    int need = (int)std::ceil(2.0 * dens * (4.0 / 3.0) * M_PI * reach * reach * reach) + 24;
    need = std::min(std::max((need + 3) & ~3, 32), 4096);
    if (P.nlist && need <= P.nbr && h->nlist_rows >= P.cap) return;
    h->dfree(P.nlist);
    P.nlist = nullptr;
    P.nbr = std::max(need, P.nbr);
    // no stale count may meet the new, unwritten lists (a build that flags an
    // overflow leaves the remaining particles as they were)
    hip_check(hipMemsetAsync(P.nnb, 0, sizeof(int) * (size_t)P.cap, h->stream), "hipMemsetAsync");
    P.nlist = (int *)h->dalloc(sizeof(int) * (size_t)P.nbr * (size_t)((P.cap + 63) / 64 * 64));
    h->nlist_rows = P.cap;
}

void update_body_force(lbdem_domain_t h, const std::vector<double> &d, const std::vector<double> &rho)
{
    const lbdem_params &p = h->prm;
    if (!p.body_force_auto) return;
    bool all_per = p.periodic[0] && p.periodic[1] && p.periodic[2];
    double s = 0.0;
    if (all_per)
        for (size_t i = 0; i < d.size(); ++i) s += (rho[i] - p.rho_f) * (M_PI * d[i] * d[i] * d[i] / 6.0);
    s /= (double)h->geo.nc;
    for (int a = 0; a < 3; ++a) h->phys.fb[a] = all_per ? -s * p.gravity[a] : 0.0;
}

// Fused substeps alternate between the two record buffers: after an odd number
// of them the records are in the other one. Returns whether a step changes it.
bool step_swaps_records(lbdem_domain_t h)
{
    return dem_substep_fused(h->desc()) && (h->phys.n_int & h->phys.n_dem & 1);
}

void swap_records(lbdem_domain_t h)
{
    h->rswap ^= 1;
    std::swap(h->pt.pk, h->pt.pk2);
}

template <typename R>
void rebuild_particle_fields(lbdem_domain_t h)
{
    launch_set_int(h->pt.need, 1, h->stream);
    launch_set_int(h->pt.need + 1, 1, h->stream);
    launch_zero_int(h->cnt, h->geo.nc, h->stream);
    launch_bin_count(h->desc(), h->stream);
    launch_bin_build(h->desc(), h->stream);
    launch_reorder(h->desc(), h->stream);
    // once more with the lengths known. Lists that overflow here need not do so
    // in the first step, which builds its own: particles may yet be added, and
    // the capacity goes by their number
    if (dem_sorts_lengths(h->desc())) {
        launch_nlist<R>(h->desc(), h->stream, false);
        launch_reorder(h->desc(), h->stream);
    }
    launch_set_int(h->pt.need + 1, 0, h->stream);
    launch_gather_eps<R>(h->desc(), h->cells<R>(), h->stream);
    hip_check(hipGetLastError(), "particle field rebuild");
}

void rebuild(lbdem_domain_t h)
{
    if (h->prec == LBDEM_FP64) rebuild_particle_fields<double>(h);
    else rebuild_particle_fields<float>(h);
}

// reallocate particle arrays for capacity `cap`, keeping nothing
void alloc_particles(lbdem_domain_t h, int64_t cap)
{
    Parts &P = h->pt;
    std::vector<double **> vec = {&P.x, &P.u, &P.w, &P.a, &P.x2, &P.u2, &P.w2, &P.a2, &P.Fam, &P.Fd, &P.Fc,
                                  &P.Fdem, &P.Tdem, &P.ustart, &P.xstart, &P.Fam_id, &P.Fd_id, &P.Fpr_id, &P.Fc_id};
    h->dfree(P.Fl);
    h->dfree(P.Fl_id);
    P.Fl = P.Fl_id = nullptr;
    if (h->phys.use_lift) {
        vec.push_back(&P.Fl);
        vec.push_back(&P.Fl_id);
    }
    double **sca[] = {&P.d, &P.rho, &P.d2, &P.rho2};
    int **ints[] = {&P.id, &P.id2, &P.nnb2, &P.pos2};
    for (double **v : vec) { h->dfree(*v); *v = nullptr; }
    for (double **v : sca) { h->dfree(*v); *v = nullptr; }
    for (int **v : ints) { h->dfree(*v); *v = nullptr; }
    h->dfree(P.sb);
    h->dfree(P.sw);
    h->dfree(P.swf);
    h->dfree(h->list);
    P.sb = nullptr;
    P.sw = nullptr;
    P.swf = nullptr;
    h->list = nullptr;
    P.cap = std::max<int64_t>(cap, 1);
    const size_t c = (size_t)P.cap;
    for (double **v : vec) {
        *v = (double *)h->dalloc(sizeof(double) * 3 * c);
        hip_check(hipMemsetAsync(*v, 0, sizeof(double) * 3 * c, h->stream), "hipMemsetAsync");
    }
    for (double **v : sca) {
        *v = (double *)h->dalloc(sizeof(double) * c);
        hip_check(hipMemsetAsync(*v, 0, sizeof(double) * c, h->stream), "hipMemsetAsync");
    }
    for (int **v : ints) {
        *v = (int *)h->dalloc(sizeof(int) * c);
        hip_check(hipMemsetAsync(*v, 0, sizeof(int) * c, h->stream), "hipMemsetAsync");
    }
    h->dfree(P.nlist);
    h->dfree(P.nnb);
    h->dfree(P.xbuild);
    P.nlist = nullptr;
    P.nbr = 0;
    h->nlist_rows = 0;
    P.nnb = (int *)h->dalloc(sizeof(int) * c);
    P.xbuild = (double *)h->dalloc(sizeof(double) * 3 * c);
    hip_check(hipMemsetAsync(P.nnb, 0, sizeof(int) * c, h->stream), "hipMemsetAsync");
    hip_check(hipMemsetAsync(P.xbuild, 0, sizeof(double) * 3 * c, h->stream), "hipMemsetAsync");
    P.sb = (int *)h->dalloc(sizeof(int) * 3 * c);
    hip_check(hipMemsetAsync(P.sb, 0, sizeof(int) * 3 * c, h->stream), "hipMemsetAsync");
    if (h->prec == LBDEM_FP32_DEV) {
        P.swf = (float *)h->dalloc(sizeof(float) * 9 * c);
        hip_check(hipMemsetAsync(P.swf, 0, sizeof(float) * 9 * c, h->stream), "hipMemsetAsync");
    } else {
        P.sw = (double *)h->dalloc(sizeof(double) * 9 * c);
        hip_check(hipMemsetAsync(P.sw, 0, sizeof(double) * 9 * c, h->stream), "hipMemsetAsync");
    }
    h->list = (int *)h->dalloc(sizeof(int) * c);
    h->list_cap = P.cap;
    h->dfree(P.pk);
    h->dfree(P.pk2);
    P.pk = P.pk2 = nullptr;
    const size_t rec = h->prec == LBDEM_FP32_DEV ? sizeof(DemRec<float>) : sizeof(DemRec<double>);
    for (void **q : {&P.pk, &P.pk2}) {
        *q = h->dalloc(rec * c);
        hip_check(hipMemsetAsync(*q, 0, rec * c, h->stream), "hipMemsetAsync");
    }
    h->dfree(h->ord.porder);
    h->ord.porder = (int *)h->dalloc(sizeof(int) * c);
    hip_check(hipMemsetAsync(h->ord.porder, 0, sizeof(int) * c, h->stream), "hipMemsetAsync");
}

// host AoS [n][3] <-> device SoA [3][cap]
void upload_vec(lbdem_domain_t h, double *dev, const double *host, int64_t n)
{
    if (n == 0) return;
    std::vector<double> buf(3 * (size_t)n);
    for (int64_t i = 0; i < n; ++i)
        for (int a = 0; a < 3; ++a) buf[a * n + i] = host ? host[3 * i + a] : 0.0;
    for (int a = 0; a < 3; ++a)
        hip_check(hipMemcpyAsync(dev + a * h->pt.cap, buf.data() + a * n, sizeof(double) * n, hipMemcpyHostToDevice,
                                 h->stream), "upload");
    hip_check(hipStreamSynchronize(h->stream), "sync");
}

struct HostParticles {
    std::vector<double> x, u, w, a, d, rho;
};

// Particle state in insertion order, [n][3] vectors and [n] scalars, to host
// or device memory (null pointers are skipped): one kernel reorders the slots
// into the permutation targets, then each array is one copy. Four vectors of
// 3.17 M spheres to the host: 31 ms (9.9 GB/s, the copy to pageable memory),
// 205 ms when the host transposed and scattered every vector itself.
// Work that the caller has pending on the default stream may still write the
// destination (a fill, a copy to pinned memory): the copies wait for it, as a
// copy on that stream would.
void read_particle_state(lbdem_domain_t h, hipMemcpyKind kind, double *x, double *u, double *w, double *a, double *d,
                         double *rho)
{
    const int64_t n = h->pt.np;
    const Parts &P = h->pt;
    double *dst[6] = {x, u, w, a, d, rho};
    const double *src[6] = {P.x2, P.u2, P.w2, P.a2, P.d2, P.rho2};
    int what = 0;
    for (int t = 0; t < 6; ++t) what |= dst[t] ? 1 << t : 0;
    if (n == 0 || what == 0) return;
    launch_pack_particles(h->desc(), what, h->stream);
    hip_check(hipGetLastError(), "particle read-out");
    hip_check(hipStreamSynchronize(nullptr), "sync");
    for (int t = 0; t < 6; ++t)
        if (dst[t])
            hip_check(hipMemcpyAsync(dst[t], src[t], sizeof(double) * (size_t)(t < 4 ? 3 * n : n), kind, h->stream),
                      "copy");
    hip_check(hipStreamSynchronize(h->stream), "sync");
}

// forces by insertion index [3][cap] -> host [n][3], through a permutation target
void download_vec(lbdem_domain_t h, const double *dev, double *host, int64_t n)
{
    if (n == 0 || !host) return;
    launch_pack_vec(dev, h->pt.cap, n, h->pt.x2, h->stream);
    hip_check(hipGetLastError(), "particle read-out");
    hip_check(hipMemcpyAsync(host, h->pt.x2, sizeof(double) * 3 * (size_t)n, hipMemcpyDeviceToHost, h->stream),
              "copy");
    hip_check(hipStreamSynchronize(h->stream), "sync");
}

HostParticles fetch_particles(lbdem_domain_t h)
{
    HostParticles hp;
    const int64_t n = h->pt.np;
    hp.x.resize(3 * n);
    hp.u.resize(3 * n);
    hp.w.resize(3 * n);
    hp.a.resize(3 * n);
    hp.d.resize(n);
    hp.rho.resize(n);
    read_particle_state(h, hipMemcpyDeviceToHost, hp.x.data(), hp.u.data(), hp.w.data(), hp.a.data(), hp.d.data(),
                        hp.rho.data());
    return hp;
}

void put_particles(lbdem_domain_t h, const HostParticles &hp)
{
    h->drop_graphs();
    const int64_t n = (int64_t)hp.d.size();
    if (n > h->pt.cap) alloc_particles(h, std::max<int64_t>(n, 2 * h->pt.cap));
    h->pt.np = n;
    upload_vec(h, h->pt.x, hp.x.data(), n);
    upload_vec(h, h->pt.u, hp.u.data(), n);
    upload_vec(h, h->pt.w, hp.w.data(), n);
    upload_vec(h, h->pt.a, hp.a.empty() ? nullptr : hp.a.data(), n);
    if (n) {
        hip_check(hipMemcpy(h->pt.d, hp.d.data(), sizeof(double) * n, hipMemcpyHostToDevice), "upload");
        hip_check(hipMemcpy(h->pt.rho, hp.rho.data(), sizeof(double) * n, hipMemcpyHostToDevice), "upload");
        std::vector<int> id(n);
        for (int64_t i = 0; i < n; ++i) id[i] = (int)i;
        hip_check(hipMemcpy(h->pt.id, id.data(), sizeof(int) * n, hipMemcpyHostToDevice), "upload");
    }
    h->dmax = 0.0;
    for (double v : hp.d) h->dmax = std::max(h->dmax, v);
    update_search(h);
    ensure_lists(h);
    update_body_force(h, hp.d, hp.rho);
}

// Stability estimate of the explicit fluid-particle coupling. Over one
// interaction subcycle the drag with F_const frozen relaxes the slip with
// the particle response time tau_p = rho_p d^2 / (18 mu f(eps)) (Table 1
// drag at Re -> 0, f the Tenneti factor, Stokes for eps = 0); the added
// mass, evaluated with the previous subcycle's du_p/dt, lags by one
// subcycle. The slip error then obeys lambda^2 - (1 - r - a) lambda - a = 0
// with r = dt_int / tau_p and a = C_am rho_f / rho_p, whose roots stay
// inside the unit circle only for r < 2 - 2a. The solid fraction in f is
// eps_ref = max(V_max/8, <eps_p>): a lone sphere sees V/8 of itself through
// the kernel, a suspension at least its mean solid fraction. Returns the
// largest stable dt_int, min over particles of (2 - 2a) tau_p (infinity
// without particles).
double tenneti_stokes_factor(double ep)
{
    // Table 1 drag factor (1 - eps)^2 [1/(1-eps)^3 + 5.81 eps/(1-eps)^3
    // + 0.48 eps^(1/3)/(1-eps)^4] at Re = 0
    const double e1 = 1.0 - ep;
    return e1 * e1 * ((1.0 + 5.81 * ep) / (e1 * e1 * e1) + 0.48 * std::cbrt(ep) / (e1 * e1 * e1 * e1));
}

double stable_dt_int(const lbdem_params &p, int64_t n, const double *d, const double *rho)
{
    if (n <= 0) return HUGE_VAL;
    const double mu = p.rho_f * (p.tau - 0.5) / 3.0;
    double vmax = 0.0, vsum = 0.0;
    for (int64_t i = 0; i < n; ++i) {
        const double V = M_PI * d[i] * d[i] * d[i] / 6.0;
        vmax = std::max(vmax, V);
        vsum += V;
    }
    const double nc = (double)p.n[0] * p.n[1] * p.n[2];
    const double eref = std::min(std::max(vmax / 8.0, vsum / nc), 0.99);
    const double f = tenneti_stokes_factor(eref);
    double dt = HUGE_VAL;
    for (int64_t i = 0; i < n; ++i) {
        const double taup = rho[i] * d[i] * d[i] / (18.0 * mu * f);
        const double a = p.use_am ? p.c_am * p.rho_f / rho[i] : 0.0;
        dt = std::min(dt, (2.0 - 2.0 * a) * taup);
    }
    return dt;
}

void check_particles(lbdem_domain_t h, int64_t n, const double *x, const double *d, const double *rho)
{
    for (int64_t i = 0; i < n; ++i) {
        if (!(d[i] > 0.0) || !(rho[i] > 0.0) || !std::isfinite(d[i]) || !std::isfinite(rho[i]))
            throw std::runtime_error("particle " + std::to_string(i) + ": diameter and density must be > 0");
        for (int a = 0; a < 3; ++a) {
            const double v = x[3 * i + a];
            const double L = h->geo.n[a];
            if (!std::isfinite(v)) throw std::runtime_error("particle " + std::to_string(i) + ": non-finite position");
            if (h->geo.per[a] ? !(v >= 0.0 && v < L) : !(v > 0.0 && v < L))
                throw std::runtime_error("particle " + std::to_string(i) + ": centre outside the domain");
        }
    }
}

// One coupled step, Alg. 1. The volume-fraction update that closes
// subcycle k and the added-mass spreading that opens subcycle k+1 use the
// same positions and bins, so they share one gather pass. With lift, the
// subcycle's u_f and curl need the new volume fraction first, so the two
// passes run apart with the curl pass between them.
template <typename R>
void enqueue_step(lbdem_domain_t h)
{
    hipStream_t s = h->stream;
    const Cells<R> C = h->cells<R>();
    const int nint = h->phys.n_int;
    const bool lift = h->phys.use_lift != 0;
    launch_cls(h, 11, [&] { launch_reorder(h->desc(), s); });
    launch_cls(h, 1, [&] { launch_moments<R>(h->desc(), C, s); });
    launch_cls(h, 2, [&] { launch_cellfields<R>(h->desc(), C, s); });
    if (lift) launch_cls(h, 12, [&] { launch_curl<R>(h->desc(), C, s); });
    launch_cls(h, 3, [&] { launch_part_am<R>(h->desc(), C, s); });
    launch_cls(h, 5, [&] { launch_gather_am<R>(h->desc(), C, s); });
    for (int k = 0; k < nint; ++k) {
        const int last_sub = k == nint - 1;
        // the lists before the drag spreading, which clears the requests served
        launch_cls(h, 8, [&] { launch_nlist<R>(h->desc(), s); });
        launch_cls(h, 4, [&] { launch_part_drag<R>(h->desc(), C, last_sub, s); });
        Desc fd = h->desc();
        fd.clear = k == 0 ? 3 : 1;
        launch_cls(h, 6, [&] { launch_gather_fd<R>(fd, C, s); });
        for (int sub = 0; sub < h->phys.n_dem; ++sub) {
            const int last_dem = sub == h->phys.n_dem - 1;
            if (dem_subcycle_single(h->desc()) && sub > 0) break;  // substep 0 ran them all
            if (dem_substep_fused(h->desc())) {
                launch_cls(h, 9, [&] { launch_dem_substep_fused<R>(h->desc(), C, k, sub, s); });
            } else {
                launch_cls(h, 9, [&] { launch_dem_force<R>(h->desc(), C, s); });
                launch_cls(h, 10, [&] { launch_integrate<R>(h->desc(), C, last_dem, last_sub, s); });
            }
        }
        if (dem_substep_fused(h->desc()) && (h->phys.n_dem & 1)) swap_records(h);
        launch_cls(h, 11, [&] { launch_bin_build(h->desc(), s); });
        if (!last_sub && lift) {
            launch_cls(h, 7, [&] { launch_gather_eps_uf<R>(h->desc(), C, s); });
            launch_cls(h, 12, [&] { launch_curl<R>(h->desc(), C, s); });
            launch_cls(h, 3, [&] { launch_part_am<R>(h->desc(), C, s); });
            launch_cls(h, 5, [&] { launch_gather_am<R>(h->desc(), C, s); });
        } else if (!last_sub) {
            launch_cls(h, 7, [&] { launch_gather_eps_am<R>(h->desc(), C, s); });
        } else {
            launch_cls(h, 7, [&] { launch_gather_eps<R>(h->desc(), C, s); });
        }
    }
    launch_cls(h, 0, [&] { launch_stream_collide<R>(h->desc(), C, s); });
    hip_check(hipGetLastError(), "kernel launch");
    h->cur ^= 1;
    h->step_host += 1;
}

// one step, replayed from a captured graph when possible (kernel arguments,
// including the buffer pointers of the step, are baked into the graph; the
// host-side buffer bookkeeping is advanced exactly as a direct launch would)
template <typename R>
void run_step(lbdem_domain_t h)
{
    if (!h->use_graphs || h->timing) {
        enqueue_step<R>(h);
        return;
    }
    hipGraphExec_t &ge = h->graph[h->cur][h->rswap];
    if (!ge) {
        hipGraph_t g = nullptr;
        hip_check(hipStreamBeginCapture(h->stream, hipStreamCaptureModeThreadLocal), "hipStreamBeginCapture");
        try {
            enqueue_step<R>(h);
        } catch (...) {
            hipGraph_t dummy = nullptr;
            (void)hipStreamEndCapture(h->stream, &dummy);
            if (dummy) (void)hipGraphDestroy(dummy);
            throw;
        }
        hip_check(hipStreamEndCapture(h->stream, &g), "hipStreamEndCapture");
        // undo the bookkeeping of the capture; the launch below redoes it
        h->cur ^= 1;
        h->step_host -= 1;
        if (step_swaps_records(h)) swap_records(h);
        hipError_t e = hipGraphInstantiate(&ge, g, nullptr, nullptr, 0);
        (void)hipGraphDestroy(g);
        hip_check(e, "hipGraphInstantiate");
    }
    hip_check(hipGraphLaunch(ge, h->stream), "hipGraphLaunch");
    h->cur ^= 1;
    h->step_host += 1;
    if (step_swaps_records(h)) swap_records(h);
}

template <typename R>
void read_field_impl(lbdem_domain_t h, int field, double *dev_out)
{
    const int64_t nc = h->geo.nc;
    const R *src = nullptr, *vec4 = nullptr;
    int ncomp = 1;
    switch (field) {
    case LBDEM_FIELD_DRHO:
        // moments of the current state
        launch_moments<R>(h->desc(), h->cells<R>(), h->stream);
        launch_vec4_w_to_double<R>((const R *)h->j, dev_out, nc, h->stream);
        hip_check(hipGetLastError(), "read_field");
        return;
    case LBDEM_FIELD_EPS_F:
        launch_fluid_fraction<R>((const R *)h->epsp, dev_out, nc, h->stream);
        hip_check(hipGetLastError(), "read_field");
        return;
    case LBDEM_FIELD_J: vec4 = (const R *)h->j; break;
    case LBDEM_FIELD_F_ACC: src = (const R *)h->facc; ncomp = 3; break;
    case LBDEM_FIELD_DUDT: vec4 = (const R *)h->dudt; break;
    case LBDEM_FIELD_GRADP: vec4 = (const R *)h->gradp; break;
    case LBDEM_FIELD_CURL: vec4 = (const R *)h->curl; break;
    case LBDEM_FIELD_UPREV: src = (const R *)h->uprev; ncomp = 3; break;
    case LBDEM_FIELD_PDF: src = (const R *)h->df[h->cur]; ncomp = 19; break;
    default: throw std::runtime_error("unknown field id");
    }
    if (vec4) launch_vec4_to_double<R>(vec4, dev_out, nc, h->stream);
    else launch_to_double<R>(src, dev_out, ncomp * nc, h->stream);
    hip_check(hipGetLastError(), "read_field");
}

int field_ncomp(int field)
{
    switch (field) {
    case LBDEM_FIELD_DRHO:
    case LBDEM_FIELD_EPS_F: return 1;
    case LBDEM_FIELD_PDF: return 19;
    default: return 3;
    }
}

}  // namespace

// ===========================================================================
// C ABI
// ===========================================================================
extern "C" {

const char *lbdem_last_error(lbdem_domain_t h) { return h ? h->err.c_str() : g_thread_err.c_str(); }

lbdem_status lbdem_params_default(lbdem_params *p)
{
    if (!p) return fail(nullptr, LBDEM_E_INVALID, "null params");
    std::memset(p, 0, sizeof(*p));
    p->n[0] = p->n[1] = p->n[2] = 32;
    p->periodic[0] = p->periodic[1] = p->periodic[2] = 1;
    p->tau = 0.8;
    p->rho_f = 1.0;
    p->e_n = 0.88;
    p->mu_c = 0.25;
    p->T_c = 0.0;
    p->h_c = 0.5;
    p->h_min = 1e-5;
    p->lub_stab = 1;
    p->use_lub = 1;
    p->use_am = 1;
    p->n_int = 10;
    p->n_dem = 1;
    p->c_am = 0.5;
    p->precision = LBDEM_FP64;
    p->lub_contact = 1;
    return LBDEM_OK;
}

lbdem_status lbdem_set_allocator(void *(*alloc)(size_t, void *), void (*free_fn)(void *, void *), void *ctx)
{
    if ((alloc == nullptr) != (free_fn == nullptr))
        return fail(nullptr, LBDEM_E_INVALID, "allocator and free must both be set or both NULL");
    g_alloc = alloc;
    g_free = free_fn;
    g_alloc_ctx = ctx;
    return LBDEM_OK;
}

lbdem_status lbdem_stability_limit(const lbdem_params *p, int64_t n, const double *d, const double *rho_p,
                                   double *dt_int_max)
{
    if (!p || !dt_int_max || n < 0 || (n > 0 && (!d || !rho_p))) return fail(nullptr, LBDEM_E_INVALID, "null argument");
    if (!(p->tau > 0.5) || !(p->rho_f > 0.0)) return fail(nullptr, LBDEM_E_INVALID, "tau must be > 1/2, rho_f > 0");
    for (int64_t i = 0; i < n; ++i)
        if (!(d[i] > 0.0) || !(rho_p[i] > 0.0) || !std::isfinite(d[i]) || !std::isfinite(rho_p[i]))
            return fail(nullptr, LBDEM_E_INVALID, "diameter and density must be > 0");
    *dt_int_max = stable_dt_int(*p, n, d, rho_p);
    const double dt = p->n_int >= 1 ? 1.0 / p->n_int : 1.0;
    return dt < *dt_int_max ? LBDEM_OK : LBDEM_E_UNSTABLE;
}

lbdem_status lbdem_create(const lbdem_params *p, void *hip_stream, lbdem_domain_t *out)
{
    if (!p || !out) return fail(nullptr, LBDEM_E_INVALID, "null argument");
    *out = nullptr;
    if (!(p->tau > 0.5) || !std::isfinite(p->tau)) return fail(nullptr, LBDEM_E_INVALID, "tau must be > 1/2");
    for (int a = 0; a < 3; ++a)
        if (p->n[a] < 1) return fail(nullptr, LBDEM_E_INVALID, "grid sizes must be >= 1");
    if (p->n_int < 1 || p->n_dem < 1) return fail(nullptr, LBDEM_E_INVALID, "n_int and n_dem must be >= 1");
    if (p->precision != LBDEM_FP64 && p->precision != LBDEM_FP32_DEV)
        return fail(nullptr, LBDEM_E_INVALID, "unknown precision");
    if (!(p->e_n > 0.0 && p->e_n <= 1.0)) return fail(nullptr, LBDEM_E_INVALID, "e_n must be in (0, 1]");
    if (!(p->rho_f > 0.0)) return fail(nullptr, LBDEM_E_INVALID, "rho_f must be > 0");
    const int64_t nc = (int64_t)p->n[0] * p->n[1] * p->n[2];
    if (nc > ((int64_t)1 << 31) - 1) return fail(nullptr, LBDEM_E_INVALID, "too many cells (max 2^31-1)");
    if ((nc + kScanPerBlock - 1) / kScanPerBlock > 1024 * 64)
        return fail(nullptr, LBDEM_E_INVALID, "too many cells for the bin scan");

    lbdem_domain_t h = new lbdem_domain();
    h->prm = *p;
    h->al = DevAlloc{g_alloc, g_free, g_alloc_ctx};
    h->prec = p->precision;
    h->use_graphs = (p->flags & LBDEM_FLAG_NO_GRAPH) == 0;
    for (int a = 0; a < 3; ++a) {
        h->geo.n[a] = p->n[a];
        h->geo.len[a] = (double)p->n[a];
        h->geo.half[a] = 0.5 * (double)p->n[a];
        h->geo.per[a] = p->periodic[a] ? 1 : 0;
    }
    h->geo.nc = nc;
    set_fastdiv((uint32_t)p->n[0], h->geo.mx, h->geo.sx);
    set_fastdiv((uint32_t)p->n[0] * (uint32_t)p->n[1], h->geo.mxy, h->geo.sxy);
    resolve_phys(h);
    lbdem_status st = guarded(nullptr, [&]() -> lbdem_status {
        hip_check(hipGetDevice(&h->device), "hipGetDevice");
        if (hip_stream) h->stream = (hipStream_t)hip_stream;
        else {
            hip_check(hipStreamCreateWithFlags(&h->stream, hipStreamNonBlocking), "hipStreamCreate");
            h->own_stream = true;
        }
        const size_t rs = h->rsize();
        h->df[0] = h->dalloc(rs * 19 * nc);
        h->df[1] = h->dalloc(rs * 19 * nc);
        h->uprev = h->dalloc(rs * 3 * nc);
        h->epsp = h->dalloc(rs * nc);
        for (void **q : {&h->j, &h->dudt, &h->gradp, &h->fam, &h->uf, &h->facc, &h->curl}) {
            if (q == &h->curl && !h->phys.use_lift) continue;
            const size_t ncomp = q == &h->facc || (q == &h->uf && h->prec == LBDEM_FP64) ? 3 : 4;
            *q = h->dalloc(rs * ncomp * nc);
            hip_check(hipMemsetAsync(*q, 0, rs * ncomp * nc, h->stream), "memset");
        }
        h->cnt = (int *)h->dalloc(sizeof(int) * nc);
        h->start = (int *)h->dalloc(sizeof(int) * (nc + 1));
        h->bsum = (int *)h->dalloc(sizeof(int) * ((nc + kScanPerBlock - 1) / kScanPerBlock + 1));
        h->loc = (int *)h->dalloc(sizeof(int) * nc);
        h->flags = (int *)h->dalloc(sizeof(int) * 4);
        h->stepc = (long long *)h->dalloc(sizeof(long long) * 2);
        h->pt.need = (int *)h->dalloc(sizeof(int) * 4);
        hip_check(hipMemsetAsync(h->pt.need, 0, sizeof(int) * 4, h->stream), "memset");
        h->diag_part = (double *)h->dalloc(sizeof(double) * 12 * 1024);
        h->diag_out = (double *)h->dalloc(sizeof(double) * 16);
        for (void *q : {h->df[0], h->df[1]}) hip_check(hipMemsetAsync(q, 0, rs * 19 * nc, h->stream), "memset");
        hip_check(hipMemsetAsync(h->epsp, 0, rs * nc, h->stream), "memset");
        hip_check(hipMemsetAsync(h->uprev, 0, rs * 3 * nc, h->stream), "memset");
        hip_check(hipMemsetAsync(h->cnt, 0, sizeof(int) * nc, h->stream), "memset");
        hip_check(hipMemsetAsync(h->start, 0, sizeof(int) * (nc + 1), h->stream), "memset");
        hip_check(hipMemsetAsync(h->flags, 0, sizeof(int) * 4, h->stream), "memset");
        hip_check(hipMemsetAsync(h->stepc, 0, sizeof(long long) * 2, h->stream), "memset");
        set_order_shape(h, 32, 32, 32);
        alloc_particles(h, 64);
        h->pt.np = 0;
        update_search(h);
        ensure_lists(h);
        rebuild(h);
        hip_check(hipStreamSynchronize(h->stream), "create sync");
        return LBDEM_OK;
    });
    if (st != LBDEM_OK) {
        lbdem_destroy(h);
        return st;
    }
    *out = h;
    return LBDEM_OK;
}

lbdem_status lbdem_destroy(lbdem_domain_t h)
{
    if (!h) return LBDEM_OK;
    if (h->stream) (void)hipStreamSynchronize(h->stream);
    h->drop_graphs();
    for (auto &e : h->ev_pool) {
        (void)hipEventDestroy(e.a);
        (void)hipEventDestroy(e.b);
    }
    std::vector<void *> all = h->owned;
    for (void *p : all) h->dfree(p);
    if (h->own_stream && h->stream) (void)hipStreamDestroy(h->stream);
    delete h;
    return LBDEM_OK;
}

lbdem_status lbdem_add_particles(lbdem_domain_t h, int64_t n, const double *x, const double *u, const double *omega,
                                 const double *d, const double *rho_p)
{
    if (!h) return fail(nullptr, LBDEM_E_INVALID, "null handle");
    if (n < 0 || (n > 0 && (!x || !d || !rho_p))) return fail(h, LBDEM_E_INVALID, "bad particle arrays");
    if (n == 0) return LBDEM_OK;
    return guarded(h, [&]() -> lbdem_status {
        check_particles(h, n, x, d, rho_p);
        if (h->pt.np + n > ((int64_t)1 << 31) - 1) throw std::runtime_error("too many particles");
        hip_check(hipStreamSynchronize(h->stream), "sync");
        int fl = 0;
        hip_check(hipMemcpy(&fl, h->flags, sizeof(int), hipMemcpyDeviceToHost), "flags");
        if (fl) return fail(h, LBDEM_E_STATE, "the domain has flagged instability; restore a state first");
        HostParticles hp = fetch_particles(h);
        const int64_t n0 = h->pt.np;
        {
            std::vector<double> dd(hp.d), rr(hp.rho);
            dd.insert(dd.end(), d, d + n);
            rr.insert(rr.end(), rho_p, rho_p + n);
            const double lim = stable_dt_int(h->prm, n0 + n, dd.data(), rr.data());
            if (!(h->phys.dt_int < lim))
                throw Unstable("explicit coupling estimated unstable: dt_int = " + std::to_string(h->phys.dt_int) +
                               " >= (2 - 2a) tau_p = " + std::to_string(lim) + "; raise n_int");
        }
        hp.x.insert(hp.x.end(), x, x + 3 * n);
        if (u) hp.u.insert(hp.u.end(), u, u + 3 * n); else hp.u.resize(3 * (n0 + n), 0.0);
        if (omega) hp.w.insert(hp.w.end(), omega, omega + 3 * n); else hp.w.resize(3 * (n0 + n), 0.0);
        hp.a.resize(3 * (n0 + n), 0.0);
        hp.d.insert(hp.d.end(), d, d + n);
        hp.rho.insert(hp.rho.end(), rho_p, rho_p + n);
        put_particles(h, hp);
        rebuild(h);
        hip_check(hipStreamSynchronize(h->stream), "sync");
        return LBDEM_OK;
    });
}

lbdem_status lbdem_step(lbdem_domain_t h, int64_t nsteps)
{
    if (!h) return fail(nullptr, LBDEM_E_INVALID, "null handle");
    if (nsteps < 0) return fail(h, LBDEM_E_INVALID, "nsteps < 0");
    return guarded(h, [&]() -> lbdem_status {
        for (int64_t s = 0; s < nsteps; ++s) {
            if (h->prec == LBDEM_FP64) run_step<double>(h);
            else run_step<float>(h);
        }
        return LBDEM_OK;
    });
}

lbdem_status lbdem_sync(lbdem_domain_t h)
{
    if (!h) return fail(nullptr, LBDEM_E_INVALID, "null handle");
    return guarded(h, [&]() -> lbdem_status {
        hip_check(hipStreamSynchronize(h->stream), "hipStreamSynchronize");
        if (h->timing) harvest_timing(h);
        int fl = 0;
        hip_check(hipMemcpy(&fl, h->flags, sizeof(int), hipMemcpyDeviceToHost), "flags");
        if (fl) {
            std::string m = "unstable:";
            if (fl & FLAG_WALL) m += " particle through a wall;";
            if (fl & FLAG_SKIN) m += " particle moved beyond the search skin within a subcycle;";
            if (fl & FLAG_NONFINITE) m += " non-finite particle state;";
            if (fl & FLAG_EPS) m += " fluid fraction <= 0;";
            if (fl & FLAG_NLIST) m += " more neighbours within the interaction reach than the list holds;";
            if (fl & FLAG_FLUID_NONFINITE) m += " non-finite fluid state (PDFs);";
            if (fl & FLAG_MACH) m += " fluid velocity |u| > 0.1 (lattice Mach number limit);";
            return fail(h, LBDEM_E_UNSTABLE, m);
        }
        return LBDEM_OK;
    });
}

lbdem_status lbdem_read_field(lbdem_domain_t h, int field, int mem_kind, double *out)
{
    if (!h || !out) return fail(h, LBDEM_E_INVALID, "null argument");
    if (field < 0 || field > LBDEM_FIELD_CURL) return fail(h, LBDEM_E_INVALID, "unknown field");
    if (field == LBDEM_FIELD_CURL && !h->curl) return fail(h, LBDEM_E_STATE, "the curl is kept only with use_lift");
    return guarded(h, [&]() -> lbdem_status {
        const int64_t n = field_ncomp(field) * h->geo.nc;
        double *dst = mem_kind == LBDEM_MEM_DEVICE ? out : h->scratch(n);
        if (h->prec == LBDEM_FP64) read_field_impl<double>(h, field, dst);
        else read_field_impl<float>(h, field, dst);
        if (mem_kind != LBDEM_MEM_DEVICE)
            hip_check(hipMemcpyAsync(out, dst, sizeof(double) * n, hipMemcpyDeviceToHost, h->stream), "copy");
        hip_check(hipStreamSynchronize(h->stream), "sync");
        return LBDEM_OK;
    });
}

lbdem_status lbdem_read_particles(lbdem_domain_t h, int mem_kind, double *x, double *u, double *omega, double *accel)
{
    if (!h) return fail(nullptr, LBDEM_E_INVALID, "null handle");
    return guarded(h, [&]() -> lbdem_status {
        read_particle_state(h, mem_kind == LBDEM_MEM_DEVICE ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost, x, u,
                            omega, accel, nullptr, nullptr);
        hip_check(hipStreamSynchronize(h->stream), "sync");
        return LBDEM_OK;
    });
}

lbdem_status lbdem_read_particle_forces(lbdem_domain_t h, double *F_am, double *F_d, double *F_pr, double *F_const)
{
    if (!h) return fail(nullptr, LBDEM_E_INVALID, "null handle");
    return guarded(h, [&]() -> lbdem_status {
        hip_check(hipStreamSynchronize(h->stream), "sync");
        const int64_t n = h->pt.np;
        download_vec(h, h->pt.Fam_id, F_am, n);
        download_vec(h, h->pt.Fd_id, F_d, n);
        download_vec(h, h->pt.Fpr_id, F_pr, n);
        download_vec(h, h->pt.Fc_id, F_const, n);
        return LBDEM_OK;
    });
}

lbdem_status lbdem_read_particle_lift(lbdem_domain_t h, double *F_l)
{
    if (!h) return fail(nullptr, LBDEM_E_INVALID, "null handle");
    if (!h->pt.Fl_id) return fail(h, LBDEM_E_STATE, "the domain runs without lift");
    return guarded(h, [&]() -> lbdem_status {
        hip_check(hipStreamSynchronize(h->stream), "sync");
        download_vec(h, h->pt.Fl_id, F_l, h->pt.np);
        return LBDEM_OK;
    });
}

lbdem_status lbdem_diagnostics(lbdem_domain_t h, lbdem_diag *out)
{
    if (!h || !out) return fail(h, LBDEM_E_INVALID, "null argument");
    return guarded(h, [&]() -> lbdem_status {
        Desc D = h->desc();
        const int nb = diag_blocks(D);
        if (h->prec == LBDEM_FP64) {
            Cells<double> C = h->cells<double>();
            launch_diag<double>(D, C, C.df_src, h->diag_part, nb, h->diag_out, h->stream);
        } else {
            Cells<float> C = h->cells<float>();
            launch_diag<float>(D, C, C.df_src, h->diag_part, nb, h->diag_out, h->stream);
        }
        hip_check(hipGetLastError(), "diag");
        double v[12];
        hip_check(hipMemcpyAsync(v, h->diag_out, sizeof(v), hipMemcpyDeviceToHost, h->stream), "diag copy");
        hip_check(hipStreamSynchronize(h->stream), "sync");
        const double nc = (double)h->geo.nc, np = (double)h->pt.np;
        out->mass_dev = v[0];
        for (int a = 0; a < 3; ++a) {
            out->mom_fluid[a] = v[1 + a];
            out->mom_part[a] = v[8 + a];
        }
        out->mean_eps_f = v[4] / nc;
        out->min_eps_f = v[5];
        out->u_ps = (np > 0 ? v[11] / np : 0.0) - v[6] / nc;
        out->max_u = v[7];
        out->step = h->step_host;
        out->np = h->pt.np;
        return LBDEM_OK;
    });
}

lbdem_status lbdem_diagnostics_noalloc(lbdem_domain_t h, lbdem_diag *out)
{
    if (!h || !out) return fail(h, LBDEM_E_INVALID, "null argument");
    return guarded(h, [&]() -> lbdem_status {
        int cur = -1;
        hip_check(hipGetDevice(&cur), "hipGetDevice");
        if (cur != h->device) hip_check(hipSetDevice(h->device), "hipSetDevice");
        struct Restore {
            int dev;
            bool on;
            ~Restore()
            {
                if (on) (void)hipSetDevice(dev);
            }
        } restore{cur, cur != h->device};
        double *sc = diag_scratch_on_device(h->device);
        if (!sc) throw HipError{hipErrorInvalidSymbol, "looking up the diagnostics scratch"};
        Desc D = h->desc();
        const int nb = diag_blocks(D);
        if ((int64_t)nb * kDiagValues + 16 > kDiagScratchDoubles)
            throw std::runtime_error("diagnostics reduction of " + std::to_string(nb) +
                                     " blocks exceeds the static scratch of " +
                                     std::to_string(kDiagMaxBlocks) + " blocks");
        double *part = sc, *res = sc + (int64_t)nb * kDiagValues;
        if (h->prec == LBDEM_FP64) {
            Cells<double> C = h->cells<double>();
            launch_diag<double>(D, C, C.df_src, part, nb, res, h->stream);
        } else {
            Cells<float> C = h->cells<float>();
            launch_diag<float>(D, C, C.df_src, part, nb, res, h->stream);
        }
        hip_check(hipGetLastError(), "diag");
        double v[kDiagValues];
        hip_check(hipMemcpyAsync(v, res, sizeof(v), hipMemcpyDeviceToHost, h->stream), "diag copy");
        hip_check(hipStreamSynchronize(h->stream), "sync");
        const double nc = (double)h->geo.nc, np = (double)h->pt.np;
        out->mass_dev = v[0];
        for (int a = 0; a < 3; ++a) {
            out->mom_fluid[a] = v[1 + a];
            out->mom_part[a] = v[8 + a];
        }
        out->mean_eps_f = v[4] / nc;
        out->min_eps_f = v[5];
        out->u_ps = (np > 0 ? v[11] / np : 0.0) - v[6] / nc;
        out->max_u = v[7];
        out->step = h->step_host;
        out->np = h->pt.np;
        return LBDEM_OK;
    });
}

int64_t lbdem_num_cells(lbdem_domain_t h) { return h ? h->geo.nc : 0; }
int64_t lbdem_num_particles(lbdem_domain_t h) { return h ? h->pt.np : 0; }

lbdem_status lbdem_get_state(lbdem_domain_t h, lbdem_state_view *v)
{
    if (!h || !v) return fail(h, LBDEM_E_INVALID, "null argument");
    if (v->np < h->pt.np) {
        const int64_t need = h->pt.np;
        v->np = need;
        return fail(h, LBDEM_E_INVALID, "particle arrays too small");
    }
    return guarded(h, [&]() -> lbdem_status {
        const int64_t nc = h->geo.nc;
        if (v->df) {
            double *tmp = h->scratch(19 * nc);
            if (h->prec == LBDEM_FP64) launch_to_double<double>((const double *)h->df[h->cur], tmp, 19 * nc, h->stream);
            else launch_to_double<float>((const float *)h->df[h->cur], tmp, 19 * nc, h->stream);
            hip_check(hipMemcpyAsync(v->df, tmp, sizeof(double) * 19 * nc, hipMemcpyDeviceToHost, h->stream), "copy");
            hip_check(hipStreamSynchronize(h->stream), "sync");
        }
        if (v->uprev) {
            double *tmp = h->scratch(3 * nc);
            if (h->prec == LBDEM_FP64) launch_to_double<double>((const double *)h->uprev, tmp, 3 * nc, h->stream);
            else launch_to_double<float>((const float *)h->uprev, tmp, 3 * nc, h->stream);
            hip_check(hipMemcpyAsync(v->uprev, tmp, sizeof(double) * 3 * nc, hipMemcpyDeviceToHost, h->stream), "copy");
            hip_check(hipStreamSynchronize(h->stream), "sync");
        }
        v->step = h->step_host;
        v->np = h->pt.np;
        read_particle_state(h, hipMemcpyDeviceToHost, v->x, v->u, v->omega, v->accel, v->d, v->rho_p);
        return LBDEM_OK;
    });
}

lbdem_status lbdem_set_state(lbdem_domain_t h, const lbdem_state_view *v)
{
    if (!h || !v || !v->df || !v->uprev) return fail(h, LBDEM_E_INVALID, "null argument");
    if (v->np < 0 || (v->np > 0 && (!v->x || !v->u || !v->omega || !v->d || !v->rho_p)))
        return fail(h, LBDEM_E_INVALID, "bad particle arrays");
    return guarded(h, [&]() -> lbdem_status {
        const int64_t nc = h->geo.nc, n = v->np;
        for (int64_t i = 0; i < n; ++i)
            for (int a = 0; a < 3; ++a) {
                const double x = v->x[3 * i + a];
                if (!std::isfinite(x) || (h->geo.per[a] ? !(x >= 0.0 && x < h->geo.n[a]) : !(x > 0.0 && x < h->geo.n[a])))
                    throw std::runtime_error("particle " + std::to_string(i) + ": centre outside the domain");
            }
        hip_check(hipStreamSynchronize(h->stream), "sync");
        double *tmp = h->scratch(19 * nc);
        hip_check(hipMemcpy(tmp, v->df, sizeof(double) * 19 * nc, hipMemcpyHostToDevice), "copy");
        if (h->prec == LBDEM_FP64) launch_from_double<double>(tmp, (double *)h->df[h->cur], 19 * nc, h->stream);
        else launch_from_double<float>(tmp, (float *)h->df[h->cur], 19 * nc, h->stream);
        hip_check(hipStreamSynchronize(h->stream), "sync");
        hip_check(hipMemcpy(tmp, v->uprev, sizeof(double) * 3 * nc, hipMemcpyHostToDevice), "copy");
        if (h->prec == LBDEM_FP64) launch_from_double<double>(tmp, (double *)h->uprev, 3 * nc, h->stream);
        else launch_from_double<float>(tmp, (float *)h->uprev, 3 * nc, h->stream);
        hip_check(hipStreamSynchronize(h->stream), "sync");
        HostParticles hp;
        hp.x.assign(v->x, v->x + 3 * n);
        hp.u.assign(v->u, v->u + 3 * n);
        hp.w.assign(v->omega, v->omega + 3 * n);
        if (v->accel) hp.a.assign(v->accel, v->accel + 3 * n); else hp.a.assign(3 * n, 0.0);
        hp.d.assign(v->d, v->d + n);
        hp.rho.assign(v->rho_p, v->rho_p + n);
        put_particles(h, hp);
        h->step_host = v->step;
        launch_set_step(h->stepc, (long long)v->step, h->stream);
        hip_check(hipMemsetAsync(h->flags, 0, sizeof(int) * 4, h->stream), "memset");
        rebuild(h);
        hip_check(hipStreamSynchronize(h->stream), "sync");
        return LBDEM_OK;
    });
}

namespace {
struct BlobHeader {
    char magic[8];
    int32_t version, precision;
    int32_t n[3], periodic[3];
    int64_t step, np;
};
}  // namespace

lbdem_status lbdem_save_state(lbdem_domain_t h, void *blob, size_t *size)
{
    if (!h || !size) return fail(h, LBDEM_E_INVALID, "null argument");
    const int64_t nc = h->geo.nc, n = h->pt.np;
    const size_t need = sizeof(BlobHeader) + sizeof(double) * (size_t)(22 * nc + 14 * n);
    if (!blob) {
        *size = need;
        return LBDEM_OK;
    }
    if (*size < need) return fail(h, LBDEM_E_INVALID, "blob too small");
    BlobHeader hd{};
    std::memcpy(hd.magic, "LBDEMST1", 8);
    hd.version = 1;
    hd.precision = h->prec;
    for (int a = 0; a < 3; ++a) {
        hd.n[a] = h->geo.n[a];
        hd.periodic[a] = h->geo.per[a];
    }
    hd.step = h->step_host;
    hd.np = n;
    std::memcpy(blob, &hd, sizeof(hd));
    double *p = (double *)((char *)blob + sizeof(hd));
    lbdem_state_view v{};
    v.df = p;
    v.uprev = p + 19 * nc;
    double *q = p + 22 * nc;
    v.x = q; v.u = q + 3 * n; v.omega = q + 6 * n; v.accel = q + 9 * n; v.d = q + 12 * n; v.rho_p = q + 13 * n;
    v.np = n;
    *size = need;
    return lbdem_get_state(h, &v);
}

lbdem_status lbdem_load_state(lbdem_domain_t h, const void *blob, size_t size)
{
    if (!h || !blob) return fail(h, LBDEM_E_INVALID, "null argument");
    if (size < sizeof(BlobHeader)) return fail(h, LBDEM_E_INVALID, "blob too small");
    BlobHeader hd;
    std::memcpy(&hd, blob, sizeof(hd));
    if (std::memcmp(hd.magic, "LBDEMST1", 8) != 0 || hd.version != 1) return fail(h, LBDEM_E_INVALID, "not a state blob");
    for (int a = 0; a < 3; ++a)
        if (hd.n[a] != h->geo.n[a] || hd.periodic[a] != h->geo.per[a])
            return fail(h, LBDEM_E_INVALID, "blob shape does not match the domain");
    const int64_t nc = h->geo.nc, n = hd.np;
    if (n < 0 || size < sizeof(BlobHeader) + sizeof(double) * (size_t)(22 * nc + 14 * n))
        return fail(h, LBDEM_E_INVALID, "blob truncated");
    const double *p = (const double *)((const char *)blob + sizeof(hd));
    lbdem_state_view v{};
    v.df = (double *)p;
    v.uprev = (double *)(p + 19 * nc);
    const double *q = p + 22 * nc;
    v.x = (double *)q; v.u = (double *)(q + 3 * n); v.omega = (double *)(q + 6 * n);
    v.accel = (double *)(q + 9 * n); v.d = (double *)(q + 12 * n); v.rho_p = (double *)(q + 13 * n);
    v.np = n;
    v.step = hd.step;
    return lbdem_set_state(h, &v);
}

}  // extern "C"

// --------------------------------------------------------------------------
// autotuner: time the gather tile variants on the domain's current state
// with the volume-fraction gather (idempotent: it rewrites the same field)
// and keep the fastest. Variants give bit-identical results.
// --------------------------------------------------------------------------
// slots into the current choice of order, lists rebuilt for it
template <typename R>
static void reorder_now(lbdem_domain_t h)
{
    launch_set_int(h->pt.need + 1, 1, h->stream);
    launch_reorder(h->desc(), h->stream);
    launch_nlist<R>(h->desc(), h->stream);
    launch_set_int(h->pt.need, 0, h->stream);
    launch_set_int(h->pt.need + 1, 0, h->stream);
    hip_check(hipGetLastError(), "reordering");
}

template <typename R>
static void autotune_impl(lbdem_domain_t h)
{
    hipEvent_t a, b;
    hip_check(hipEventCreate(&a), "hipEventCreate");
    hip_check(hipEventCreate(&b), "hipEventCreate");
    // the density default is kept unless another variant is at least 3 %
    // faster (timings of near-equal variants flip from run to run)
    const double dens = h->geo.nc > 0 ? (double)h->pt.np / (double)h->geo.nc : 0.0;
    const int def = dens < 0.3 ? 0 : (dens < 1.0 ? 1 : 2);
    float t[kGatherVariants];
    for (int v = 0; v < kGatherVariants; ++v) {
        h->tune.gather = v;
        float tmin = 1e30f;
        for (int rep = 0; rep < 6; ++rep) {
            hip_check(hipEventRecord(a, h->stream), "hipEventRecord");
            launch_gather_eps<R>(h->desc(), h->cells<R>(), h->stream);
            hip_check(hipEventRecord(b, h->stream), "hipEventRecord");
            hip_check(hipEventSynchronize(b), "hipEventSynchronize");
            float ms = 0.f;
            hip_check(hipEventElapsedTime(&ms, a, b), "hipEventElapsedTime");
            if (rep > 0) tmin = std::min(tmin, ms);
            if (rep > 0 && v > 0 && ms > 1.5f * *std::min_element(t, t + v)) break;  // out of the running
        }
        t[v] = tmin;
    }
    int best_v = def;
    for (int v = 0; v < kGatherVariants; ++v)
        if (t[v] < 0.97f * t[best_v]) best_v = v;
    h->tune.gather = best_v;

    // Slot order (each particle's force is the same in every order). Blocks of
    // 32^3 or 16^3 cells, whichever the DEM force pass takes less time with; row
    // by row below kBlockedFrom particles, where the order changed a step by less
    // than the timings differ (396 k dense spheres: 11.9 ms row by row, 11.6 in
    // blocks of 32^3, 12.0 in 16^3; 3.17 M: 98, 94 and 92 ms).
    h->tune.dem_order = h->pt.np >= kBlockedFrom ? 1 : 0;
    if (h->pt.np > 0) {
        float t[2] = {0.f, 0.f};
        const int edge[2] = {32, 16};
        const int n = h->tune.dem_order ? 2 : 1;
        for (int c = 0; c < n; ++c) {
            set_order_shape(h, edge[c], edge[c], edge[c]);
            reorder_now<R>(h);
            t[c] = 1e30f;
            for (int rep = 0; n > 1 && rep < 4; ++rep) {
                hip_check(hipEventRecord(a, h->stream), "hipEventRecord");
                launch_dem_force<R>(h->desc(), h->cells<R>(), h->stream);
                hip_check(hipEventRecord(b, h->stream), "hipEventRecord");
                hip_check(hipEventSynchronize(b), "hipEventSynchronize");
                float ms = 0.f;
                hip_check(hipEventElapsedTime(&ms, a, b), "hipEventElapsedTime");
                if (rep > 0) t[c] = std::min(t[c], ms);
            }
        }
        // (near-equal timings flip from run to run)
        if (n > 1 && !(t[1] < 0.97f * t[0])) {
            set_order_shape(h, edge[0], edge[0], edge[0]);
            reorder_now<R>(h);
        }
        hip_check(hipStreamSynchronize(h->stream), "sync");
    }

    // residency of the streaming cell passes, timed on the moments pass and
    // the stream-collide (both rewrite the same outputs from the same inputs;
    // the stream-collide's step count is restored afterwards)
    {
        const int cand[] = {-1, 0, 3, 4, 5, 6};
        float best_t = 1e30f;
        int best = -1;
        const Cells<R> C = h->cells<R>();
        for (int cw : cand) {
            h->tune.cell_waves = cw;
            float tmin = 1e30f;
            for (int rep = 0; rep < 4; ++rep) {
                hip_check(hipEventRecord(a, h->stream), "hipEventRecord");
                launch_moments<R>(h->desc(), C, h->stream);
                launch_stream_collide<R>(h->desc(), C, h->stream);
                hip_check(hipEventRecord(b, h->stream), "hipEventRecord");
                hip_check(hipEventSynchronize(b), "hipEventSynchronize");
                float ms = 0.f;
                hip_check(hipEventElapsedTime(&ms, a, b), "hipEventElapsedTime");
                if (rep > 0) tmin = std::min(tmin, ms);
            }
            if (tmin < 0.97f * best_t) {
                best_t = tmin;
                best = cw;
            }
        }
        h->tune.cell_waves = best;
        launch_set_step(h->stepc, (long long)h->step_host, h->stream);
        hip_check(hipStreamSynchronize(h->stream), "sync");
    }
    (void)hipEventDestroy(a);
    (void)hipEventDestroy(b);
    h->drop_graphs();
}

extern "C" {

lbdem_status lbdem_autotune(lbdem_domain_t h, int32_t *gather_variant)
{
    if (!h) return fail(nullptr, LBDEM_E_INVALID, "null handle");
    return guarded(h, [&]() -> lbdem_status {
        hip_check(hipStreamSynchronize(h->stream), "sync");
        if (h->prec == LBDEM_FP64) autotune_impl<double>(h);
        else autotune_impl<float>(h);
        if (gather_variant) *gather_variant = h->tune.gather;
        return LBDEM_OK;
    });
}

lbdem_status lbdem_get_tuning(lbdem_domain_t h, lbdem_tuning *out)
{
    if (!h || !out) return fail(h, LBDEM_E_INVALID, "null argument");
    out->gather_variant = h->tune.gather;
    out->dem_order = h->tune.dem_order;
    for (int a = 0; a < 3; ++a) out->dem_block[a] = h->ord.ob[a];
    out->cell_waves = h->tune.cell_waves;
    out->fuse_substep = h->tune.fuse;
    return LBDEM_OK;
}

lbdem_status lbdem_set_tuning(lbdem_domain_t h, const lbdem_tuning *t)
{
    if (!h || !t) return fail(h, LBDEM_E_INVALID, "null argument");
    if (t->gather_variant < -1 || t->gather_variant >= kGatherVariants)
        return fail(h, LBDEM_E_INVALID, "unknown gather variant");
    if (t->dem_order < -1 || t->dem_order > 1) return fail(h, LBDEM_E_INVALID, "dem_order must be -1, 0 or 1");
    if (t->cell_waves < -1 || t->cell_waves > 16)
        return fail(h, LBDEM_E_INVALID, "cell_waves must be -1 (default), 0 (no cap) or 1..16");
    for (int a = 0; a < 3; ++a)
        if (t->dem_block[a] < 1 || t->dem_block[a] > 256)
            return fail(h, LBDEM_E_INVALID, "DEM block edges must be in 1..256 cells");
    if (t->fuse_substep < -1 || t->fuse_substep > 1)
        return fail(h, LBDEM_E_INVALID, "fuse_substep must be -1, 0 or 1");
    return guarded(h, [&]() -> lbdem_status {
        hip_check(hipStreamSynchronize(h->stream), "sync");
        h->tune.gather = t->gather_variant;
        h->tune.dem_order = t->dem_order;
        h->tune.cell_waves = t->cell_waves;
        h->tune.fuse = t->fuse_substep;
        set_order_shape(h, t->dem_block[0], t->dem_block[1], t->dem_block[2]);
        launch_set_int(h->pt.need + 1, 1, h->stream);  // the next step starts in the new order
        hip_check(hipStreamSynchronize(h->stream), "sync");
        h->drop_graphs();
        return LBDEM_OK;
    });
}

lbdem_status lbdem_set_gather_variant(lbdem_domain_t h, int32_t variant)
{
    if (!h) return fail(nullptr, LBDEM_E_INVALID, "null handle");
    if (variant < -1 || variant >= kGatherVariants) return fail(h, LBDEM_E_INVALID, "unknown gather variant");
    return guarded(h, [&]() -> lbdem_status {
        hip_check(hipStreamSynchronize(h->stream), "sync");
        h->tune.gather = variant;
        h->drop_graphs();
        return LBDEM_OK;
    });
}

lbdem_status lbdem_set_timing(lbdem_domain_t h, int on)
{
    if (!h) return fail(nullptr, LBDEM_E_INVALID, "null handle");
    return guarded(h, [&]() -> lbdem_status {
        hip_check(hipStreamSynchronize(h->stream), "sync");
        if (h->timing) harvest_timing(h);
        h->timing = on != 0;
        for (int c = 0; c < kTimingClasses; ++c) {
            h->cls_ms[c] = 0.0;
            h->cls_n[c] = 0;
        }
        return LBDEM_OK;
    });
}

lbdem_status lbdem_kernel_time(lbdem_domain_t h, int cls, double *ms_total, int64_t *launches)
{
    if (!h || cls < 0 || cls >= kTimingClasses) return fail(h, LBDEM_E_INVALID, "bad argument");
    return guarded(h, [&]() -> lbdem_status {
        hip_check(hipStreamSynchronize(h->stream), "sync");
        if (h->timing) harvest_timing(h);
        if (ms_total) *ms_total = h->cls_ms[cls];
        if (launches) *launches = h->cls_n[cls];
        return LBDEM_OK;
    });
}

}  // extern "C"

// ===========================================================================
// Batching: independent domains advanced together. One batch step is a
// single captured HIP graph whose branches (one per worker stream) each run
// the full step of a share of the domains, so small domains overlap on the
// device. Domains keep their own parameters (n_int, precision, tuning).
// ===========================================================================
struct lbdem_batch {
    std::vector<lbdem_domain_t> doms;
    hipStream_t master = nullptr;
    bool own_master = false;
    std::vector<hipStream_t> workers;
    hipEvent_t fork = nullptr;
    std::vector<hipEvent_t> join;
    std::vector<std::pair<std::string, hipGraphExec_t>> graphs;
    bool tuned = false;
};

namespace {

std::string batch_key(lbdem_batch_t b)
{
    std::string k;
    for (lbdem_domain_t d : b->doms)
        k += std::to_string(d->cur) + ":" + std::to_string(d->rswap) + ":" + std::to_string(d->version) + ";";
    return k;
}

void advance_bookkeeping(lbdem_domain_t d, int dir)
{
    d->cur ^= 1;
    d->step_host += dir;
    if (step_swaps_records(d)) swap_records(d);
}

void batch_drop_graphs(lbdem_batch_t b)
{
    for (auto &g : b->graphs) (void)hipGraphExecDestroy(g.second);
    b->graphs.clear();
}

void batch_enqueue(lbdem_batch_t b)
{
    const int S = (int)b->workers.size();
    hip_check(hipEventRecord(b->fork, b->master), "hipEventRecord");
    for (hipStream_t w : b->workers) hip_check(hipStreamWaitEvent(w, b->fork, 0), "hipStreamWaitEvent");
    for (size_t i = 0; i < b->doms.size(); ++i) {
        lbdem_domain_t d = b->doms[i];
        hipStream_t saved = d->stream;
        d->stream = b->workers[i % S];
        try {
            if (d->prec == LBDEM_FP64) enqueue_step<double>(d);
            else enqueue_step<float>(d);
        } catch (...) {
            d->stream = saved;
            throw;
        }
        d->stream = saved;
    }
    for (int w = 0; w < S; ++w) {
        hip_check(hipEventRecord(b->join[w], b->workers[w]), "hipEventRecord");
        hip_check(hipStreamWaitEvent(b->master, b->join[w], 0), "hipStreamWaitEvent");
    }
}

}  // namespace

extern "C" {

lbdem_status lbdem_batch_create(int32_t n, const lbdem_params *p, void *hip_stream, lbdem_batch_t *out)
{
    if (!p || !out || n < 1) return fail(nullptr, LBDEM_E_INVALID, "bad batch arguments");
    *out = nullptr;
    lbdem_batch_t b = new lbdem_batch();
    lbdem_status st = guarded(nullptr, [&]() -> lbdem_status {
        if (hip_stream) b->master = (hipStream_t)hip_stream;
        else {
            hip_check(hipStreamCreateWithFlags(&b->master, hipStreamNonBlocking), "hipStreamCreate");
            b->own_master = true;
        }
        const int S = std::min<int>(n, 4);
        for (int w = 0; w < S; ++w) {
            hipStream_t s;
            hip_check(hipStreamCreateWithFlags(&s, hipStreamNonBlocking), "hipStreamCreate");
            b->workers.push_back(s);
            hipEvent_t e;
            hip_check(hipEventCreateWithFlags(&e, hipEventDisableTiming), "hipEventCreate");
            b->join.push_back(e);
        }
        hip_check(hipEventCreateWithFlags(&b->fork, hipEventDisableTiming), "hipEventCreate");
        for (int i = 0; i < n; ++i) {
            lbdem_domain_t d = nullptr;
            lbdem_status s2 = lbdem_create(&p[i], (void *)b->master, &d);
            if (s2 != LBDEM_OK)
                return fail(nullptr, s2, "domain " + std::to_string(i) + ": " + g_thread_err);
            b->doms.push_back(d);
        }
        return LBDEM_OK;
    });
    if (st != LBDEM_OK) {
        lbdem_batch_destroy(b);
        return st;
    }
    *out = b;
    return LBDEM_OK;
}

lbdem_status lbdem_batch_domain(lbdem_batch_t b, int32_t i, lbdem_domain_t *out)
{
    if (!b || !out || i < 0 || i >= (int32_t)b->doms.size()) return fail(nullptr, LBDEM_E_INVALID, "bad domain index");
    *out = b->doms[i];
    return LBDEM_OK;
}

lbdem_status lbdem_batch_autotune(lbdem_batch_t b)
{
    if (!b) return fail(nullptr, LBDEM_E_INVALID, "null batch");
    for (size_t i = 0; i < b->doms.size(); ++i) {
        lbdem_status st = lbdem_autotune(b->doms[i], nullptr);
        if (st != LBDEM_OK) return fail(nullptr, st, "domain " + std::to_string(i) + ": " + b->doms[i]->err);
    }
    batch_drop_graphs(b);
    b->tuned = true;
    return LBDEM_OK;
}

lbdem_status lbdem_batch_step(lbdem_batch_t b, int64_t nsteps)
{
    if (!b || nsteps < 0) return fail(nullptr, LBDEM_E_INVALID, "bad batch step arguments");
    return guarded(nullptr, [&]() -> lbdem_status {
        for (int64_t s = 0; s < nsteps; ++s) {
            const std::string key = batch_key(b);
            hipGraphExec_t ge = nullptr;
            for (auto &g : b->graphs)
                if (g.first == key) ge = g.second;
            if (!ge) {
                hipGraph_t g = nullptr;
                hip_check(hipStreamBeginCapture(b->master, hipStreamCaptureModeThreadLocal), "hipStreamBeginCapture");
                try {
                    batch_enqueue(b);
                } catch (...) {
                    hipGraph_t dummy = nullptr;
                    (void)hipStreamEndCapture(b->master, &dummy);
                    if (dummy) (void)hipGraphDestroy(dummy);
                    throw;
                }
                hip_check(hipStreamEndCapture(b->master, &g), "hipStreamEndCapture");
                for (lbdem_domain_t d : b->doms) advance_bookkeeping(d, -1);
                hipError_t e = hipGraphInstantiate(&ge, g, nullptr, nullptr, 0);
                (void)hipGraphDestroy(g);
                hip_check(e, "hipGraphInstantiate");
                if (b->graphs.size() >= 4) batch_drop_graphs(b);
                b->graphs.emplace_back(key, ge);
            }
            hip_check(hipGraphLaunch(ge, b->master), "hipGraphLaunch");
            for (lbdem_domain_t d : b->doms) advance_bookkeeping(d, +1);
        }
        return LBDEM_OK;
    });
}

lbdem_status lbdem_batch_sync(lbdem_batch_t b)
{
    if (!b) return fail(nullptr, LBDEM_E_INVALID, "null batch");
    for (size_t i = 0; i < b->doms.size(); ++i) {
        lbdem_status st = lbdem_sync(b->doms[i]);
        if (st != LBDEM_OK) return fail(nullptr, st, "domain " + std::to_string(i) + ": " + b->doms[i]->err);
    }
    return LBDEM_OK;
}

int32_t lbdem_batch_size(lbdem_batch_t b) { return b ? (int32_t)b->doms.size() : 0; }

lbdem_status lbdem_batch_destroy(lbdem_batch_t b)
{
    if (!b) return LBDEM_OK;
    if (b->master) (void)hipStreamSynchronize(b->master);
    batch_drop_graphs(b);
    for (lbdem_domain_t d : b->doms) lbdem_destroy(d);
    for (hipStream_t s : b->workers) (void)hipStreamDestroy(s);
    for (hipEvent_t e : b->join) (void)hipEventDestroy(e);
    if (b->fork) (void)hipEventDestroy(b->fork);
    if (b->own_master && b->master) (void)hipStreamDestroy(b->master);
    delete b;
    return LBDEM_OK;
}

}  // extern "C"
