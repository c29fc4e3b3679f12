// C ABI of libsoptx: handle lifetime, argument validation, device uploads and
// kernel dispatch.  Every numeric step runs in the HIP kernels of kernels.hip.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <map>
#include <mutex>
#include <new>
#include <tuple>
#include <vector>

#include "../../include/soptx.h"
#include "../../include/soptx_debug.h"
#include "host_util.h"
#include "internal.h"
#include "kernels.h"

using namespace soptx;

namespace soptx {

// Per-(device, stream, use) scratch; see host_util.h.
namespace {
struct Workspace {
    double *buf = nullptr;
    size_t n = 0;
};
std::mutex g_ws_mu;
std::map<std::tuple<int, hipStream_t, int>, Workspace> g_ws;
// Buffers replaced by larger ones.  They are kept, not freed: a HIP graph
// captured with a call on this stream holds their addresses, and a replay
// after a larger call must still find valid memory there (it also spares
// the host a synchronisation before the free)
std::vector<double *> g_ws_retired;
}  // namespace

int get_workspace(int device, hipStream_t st, size_t n, double **out, int use) {
    std::lock_guard<std::mutex> lk(g_ws_mu);
    try {
        Workspace &w = g_ws[std::make_tuple(device, st, use)];
        if (w.n < n) {
            g_ws_retired.reserve(g_ws_retired.size() + 1);
            const size_t cap = n < 4096 ? 4096 : n;
            double *p = nullptr;
            if (hipMalloc(&p, cap * sizeof(double)) != hipSuccess) {
                (void)hipGetLastError();  // not for the next launch to report
                return SOPTX_E_OOM;
            }
            if (w.buf) g_ws_retired.push_back(w.buf);
            w.buf = p;
            w.n = cap;
        }
        *out = w.buf;
    } catch (...) {
        return SOPTX_E_OOM;
    }
    return SOPTX_OK;
}

}  // namespace soptx


namespace {
// soptx_debug_fail_optional: how many allocations that a call can do without
// still succeed, and how many then fail
std::mutex g_fail_mu;
int g_fail_skip = 0, g_fail_count = 0;
bool fail_optional() {
    std::lock_guard<std::mutex> lk(g_fail_mu);
    if (g_fail_count == 0) return false;
    if (g_fail_skip > 0) {
        g_fail_skip--;
        return false;
    }
    g_fail_count--;
    return true;
}

// A record in host memory that kernels write (a stop of the CG), with an event;
// up to kKept of them are kept between calls, each for its device.  Coherent
// memory: the host reads what a kernel wrote once an event behind that kernel
// has passed.  host is null where none could be had.
struct StopRecord {
    double *host = nullptr, *dev = nullptr;
    hipEvent_t event = nullptr;
    int device;
    hipStream_t stream;
    StopRecord(int d, hipStream_t st) : device(d), stream(st) {
        if (fail_optional()) return;
        {
            std::lock_guard<std::mutex> lk(mu());
            for (Kept &k : kept())
                if (k.host && k.device == device) {
                    host = k.host;
                    dev = k.dev;
                    event = k.event;
                    k.host = nullptr;
                    break;
                }
        }
        if (!host) {
            void *p = nullptr, *q = nullptr;
            if (hipHostMalloc(&p, 64, hipHostMallocMapped | hipHostMallocCoherent) != hipSuccess) {
                (void)hipGetLastError();
                return;
            }
            if (hipHostGetDevicePointer(&q, p, 0) != hipSuccess ||
                hipEventCreateWithFlags(&event, hipEventDisableTiming) != hipSuccess) {
                (void)hipHostFree(p);
                (void)hipGetLastError();
                return;
            }
            host = static_cast<double *>(p);
            dev = static_cast<double *>(q);
        }
        host[0] = host[1] = host[2] = 0.0;
    }
    ~StopRecord() {
        if (!host) return;
        // kernels of a call that failed may still write the record: they end first
        (void)hipStreamSynchronize(stream);
        {
            std::lock_guard<std::mutex> lk(mu());
            for (Kept &k : kept())
                if (!k.host) {
                    k = Kept{host, dev, event, device};
                    return;
                }
        }
        (void)hipEventDestroy(event);
        (void)hipHostFree(host);
    }
    StopRecord(const StopRecord &) = delete;
    StopRecord &operator=(const StopRecord &) = delete;

private:
    struct Kept {
        double *host, *dev;
        hipEvent_t event;
        int device;
    };
    static constexpr int kKept = 32;
    static std::mutex &mu() {
        static std::mutex m;
        return m;
    }
    static Kept (&kept())[kKept] {
        static Kept k[kKept] = {};
        return k;
    }
};
}  // namespace

struct soptx_pattern_s {
    int elem = 0, dim = 0, nen = 0, ref_method = 0, device = 0, nq = 0;
    int64_t n_nodes = 0, n_cells = 0, ndof = 0, nnz = 0, ngroups = 0, nsig = 0;
    int emax = 0, kmax = 0;
    int64_t stage = 0;
    int32_t *row_ptr = nullptr, *col_idx = nullptr, *cells = nullptr;
    double *geo = nullptr;
    int32_t *grp_info = nullptr, *grp_nodes = nullptr, *grp_elems = nullptr;
    uint16_t *grp_n2l = nullptr;
    int32_t *grp_rows = nullptr;
    int32_t *grp_rank_off = nullptr;  // canonical-order plans only
    uint8_t *grp_rank = nullptr;
    int64_t n_rank_bytes = 0;
    int32_t *elem_by_rank = nullptr;  // canonical-order plans only: rank -> element
    double *geo_rank = nullptr;       // geo with its columns in rank order
    int n_cu = 0;
    int32_t *sig_info = nullptr, *sig_pos_ptr = nullptr, *sig_contrib = nullptr, *sig_pairs = nullptr;
    int32_t *sig_witems = nullptr, *sig_witem_ptr = nullptr;
    uint16_t *pos = nullptr, *nb_tdeg = nullptr;
    int32_t *nb_tslot = nullptr;
    int32_t *nb = nullptr;
    double *M = nullptr;
    float *M32 = nullptr;
    double *qw = nullptr, *qgrad = nullptr, *cgrad = nullptr, *xref = nullptr;
    // per-quadrature-point assembly (handles built by soptx_build_pattern_general)
    bool affine = true, general = false;
    double *coords = nullptr;
    int32_t *gptr = nullptr, *gent = nullptr, *gnode = nullptr;
    double *qgeo = nullptr;  // general Q1: per-point geometry of the row-block kernels
    // Q2 hexahedra: row groups and per-point geometry of the fused assembly
    int32_t *rg_info = nullptr, *rg_rows = nullptr, *rg_vis = nullptr, *rg_pairs = nullptr, *rg_ext = nullptr;
    uint16_t *rg_code = nullptr;
    double *geo27 = nullptr;
    int64_t n_row_groups = 0;
    int max_items = 0;       // largest number of work items of a signature
    float *qgrad32 = nullptr;
    soptx_pattern_stats stats{};
    std::vector<void *> allocs;
};

struct soptx_host_plan_s {
    HostPlan hp;
};

// A Dirichlet mask bound to a pattern: for every group of the plan whose
// blocks hold a fixed row or column, the offset of its bits (one byte per
// (node, neighbour position), see dirichlet_entry), -1 for the others.
struct soptx_dirichlet_s {
    soptx_pattern h = nullptr;
    int device = 0;
    int64_t n_fixed = 0, n_groups = 0;
    int32_t *off = nullptr;
    uint8_t *bits = nullptr;
    std::vector<void *> allocs;
    int64_t device_bytes = 0;
};

namespace {

template <class T>
int upload(soptx_pattern_s *h, const std::vector<T> &v, T **dst, hipStream_t st) {
    return upload_vector(h->allocs, v, dst, st, &h->stats.device_bytes);
}

void free_handle(soptx_pattern_s *h) {
    if (!h) return;
    for (void *p : h->allocs) (void)hipFree(p);
    delete h;
}

// the code an affine-only call returns on a handle with general elements
int not_affine(const soptx_pattern_s *h) {
    return h->elem == SOPTX_HEX27 ? SOPTX_E_UNSUPPORTED_ELEM : SOPTX_E_NONAFFINE;
}

int check_material(const soptx_material *m) {
    if (!m) return SOPTX_E_INVALID_ARG;
    if (!(m->E0 > m->Emin) || !(m->Emin >= 0.0) || !(m->nu > -1.0 && m->nu < 0.5) || !(m->p >= 1.0) ||
        !std::isfinite(m->E0) || !std::isfinite(m->p))
        return SOPTX_E_INVALID_ARG;
    return SOPTX_OK;
}

// Lame constants at unit modulus; 2D plane stress uses lambda* = nu/(1-nu^2)
void lame(const soptx_pattern_s *h, const soptx_material *m, double *lam, double *mu) {
    const double nu = m->nu;
    *mu = 1.0 / (2.0 * (1.0 + nu));
    if (h->dim == 2 && !m->plane_strain) *lam = nu / (1.0 - nu * nu);
    else *lam = nu / ((1.0 + nu) * (1.0 - 2.0 * nu));
}

int int_exponent(double p) {
    if (p == std::floor(p) && p >= 0.0 && p <= 16.0) return (int)p;
    return -1;
}

// SOPTX_BF16_FP32ACC is refused: bf16-rounded inputs miss the FP32 form's
// bound on K by two to three orders of magnitude
bool valid_prec(int32_t prec) { return prec == SOPTX_FP64 || prec == SOPTX_FP32; }

}  // namespace

extern "C" {

const char *soptx_status_string(int s) {
    switch (s) {
    case SOPTX_OK: return "ok";
    case SOPTX_E_INVALID_ARG: return "invalid argument";
    case SOPTX_E_UNSUPPORTED_ELEM: return "unsupported element type";
    case SOPTX_E_BAD_MESH: return "bad mesh (node index out of range or repeated in a cell)";
    case SOPTX_E_JACOBIAN: return "element with non-positive Jacobian determinant";
    case SOPTX_E_NONAFFINE: return "element map is not affine";
    case SOPTX_E_OVERFLOW: return "size exceeds the int32 index range";
    case SOPTX_E_OOM: return "out of memory";
    case SOPTX_E_DEVICE: return "HIP device or launch error";
    case SOPTX_E_SCRATCH: return "input exceeds the fixed scratch of an allocation-free call";
    default: return "unknown status";
    }
}

int soptx_validate_mesh(const soptx_mesh *mesh) { return validate_mesh(mesh); }

int soptx_reference_tensor(int32_t elem, int32_t ref_method, double *M_out) {
    if (!M_out) return SOPTX_E_INVALID_ARG;
    if (elem_dim(elem) < 0) return SOPTX_E_UNSUPPORTED_ELEM;
    return reference_tensor(elem, ref_method, M_out);
}

// The row groups' tables and geometry of a Q2 mesh.  SOPTX_E_OOM: the device
// has no room beside the pattern; nothing of them is held, and the assembly
// forms element matrices.
static int row_group_tables(soptx_pattern_s *h, const HostPlan &hp, hipStream_t st) {
    const size_t held = h->allocs.size();
    const int64_t bytes0 = h->stats.device_bytes;
    const size_t bytes = (size_t)hp.n_cells * 27 * 10 * sizeof(double);
    void *geo = nullptr;
    int rc = fail_optional() ? SOPTX_E_OOM : SOPTX_OK;
    if (!rc) {
        h->allocs.reserve(held + 7);
        if (hipMalloc(&geo, bytes) != hipSuccess) rc = SOPTX_E_OOM;
        else h->allocs.push_back(geo);
    }
    if (!rc) rc = upload(h, hp.rg_info, &h->rg_info, st);
    if (!rc) rc = upload(h, hp.rg_rows, &h->rg_rows, st);
    if (!rc) rc = upload(h, hp.rg_vis, &h->rg_vis, st);
    if (!rc) rc = upload(h, hp.rg_pairs, &h->rg_pairs, st);
    if (!rc) rc = upload(h, hp.rg_ext, &h->rg_ext, st);
    if (!rc) rc = fail_optional() ? SOPTX_E_OOM : upload(h, hp.rg_code, &h->rg_code, st);
    if (rc == SOPTX_E_OOM) {
        (void)hipGetLastError();  // not for the next launch to report
        for (size_t k = held; k < h->allocs.size(); k++) (void)hipFree(h->allocs[k]);
        h->allocs.resize(held);
        h->stats.device_bytes = bytes0;
        h->rg_info = h->rg_rows = h->rg_vis = h->rg_pairs = h->rg_ext = nullptr;
        h->rg_code = nullptr;
    }
    if (rc) return rc;
    h->stats.device_bytes += (int64_t)bytes;
    h->geo27 = static_cast<double *>(geo);
    if (launch_hex27_geometry(h->cells, h->coords, hp.n_cells, h->geo27, st) != hipSuccess) return SOPTX_E_DEVICE;
    h->n_row_groups = (int64_t)hp.rg_info.size() / 4;
    return SOPTX_OK;
}

static int build_pattern(const soptx_mesh *mesh, int32_t ref_method, bool general, soptx_pattern *out,
                         void *stream) {
    if (!out) return SOPTX_E_INVALID_ARG;
    *out = nullptr;
    if (ref_method != SOPTX_REF_SYMBOLIC && ref_method != SOPTX_REF_QUADRATURE) return SOPTX_E_INVALID_ARG;
    HostPlan hp;
    int rc;
    try {
        rc = build_host_plan(mesh, hp, general);
    } catch (const std::bad_alloc &) {
        return SOPTX_E_OOM;
    } catch (...) {
        return SOPTX_E_INVALID_ARG;
    }
    if (rc) return rc;
    hipStream_t st = static_cast<hipStream_t>(stream);
    soptx_pattern_s *h = new (std::nothrow) soptx_pattern_s();
    if (!h) return SOPTX_E_OOM;
    try {
        h->elem = hp.elem; h->dim = hp.dim; h->nen = hp.nen; h->ref_method = ref_method;
        h->n_nodes = hp.n_nodes; h->n_cells = hp.n_cells; h->ndof = hp.ndof; h->nnz = hp.nnz;
        h->ngroups = hp.n_groups(); h->nsig = hp.n_sigs(); h->emax = hp.ne_max; h->kmax = hp.kmax; h->stage = hp.stage_max;
        h->affine = hp.affine; h->general = hp.general;
        for (int64_t sg = 0; sg < hp.n_sigs(); sg++) {
            const int deg = hp.sig_info[4 * sg + 1], posoff = hp.sig_info[4 * sg + 2];
            int n = 0;
            while (n <= deg && hp.sig_pairs[2 * (size_t)posoff + 2 * n] >= 0) n++;
            h->max_items = std::max({h->max_items, n, hp.sig_witem_ptr[sg + 1] - hp.sig_witem_ptr[sg]});
        }
        if (hipGetDevice(&h->device) != hipSuccess) { free_handle(h); return SOPTX_E_DEVICE; }
        if (hipDeviceGetAttribute(&h->n_cu, hipDeviceAttributeMultiprocessorCount, h->device) != hipSuccess)
            h->n_cu = 0;
        // reference data
        const int nen = hp.nen, dim = hp.dim;
        std::vector<double> M((size_t)nen * nen * dim * dim);
        rc = reference_tensor(hp.elem, ref_method, M.data());
        if (rc) { free_handle(h); return rc; }
        std::vector<float> M32(M.begin(), M.end());
        std::vector<double> qw, qg;
        rc = reference_qp_grads(hp.elem, qw, qg);
        if (rc) { free_handle(h); return rc; }
        h->nq = (int)qw.size();
        std::vector<float> qg32(qg.begin(), qg.end());
        // centroid gradients and reference node coordinates (rigid-motion removal)
        std::vector<double> xref((size_t)nen * dim, 0.0), cg((size_t)nen * dim, 0.0);
        {
            static const int E[6][2] = {{0, 1}, {0, 2}, {0, 3}, {1, 2}, {1, 3}, {2, 3}};
            for (int i = 0; i < nen; i++) {
                if (hp.elem == SOPTX_QUAD4 || hp.elem == SOPTX_HEX8) {
                    for (int m = 0; m < dim; m++) xref[i * dim + m] = corner_bit(hp.elem, i, m);
                } else if (hp.elem == SOPTX_HEX27) {
                    for (int m = 0; m < dim; m++) xref[i * dim + m] = 0.5 * lattice_index(i, m);
                } else if (hp.elem == SOPTX_TRI3) {
                    if (i > 0) xref[i * dim + i - 1] = 1.0;
                } else {
                    auto v = [&](int vv, int m) { return (vv > 0 && vv - 1 == m) ? 1.0 : 0.0; };
                    for (int m = 0; m < 3; m++)
                        xref[i * dim + m] = i < 4 ? v(i, m) : 0.5 * (v(E[i - 4][0], m) + v(E[i - 4][1], m));
                }
            }
            // weighted mean of the quadrature-point gradients: the reference
            // gradient at the centroid (the rules are symmetric and the
            // gradients multilinear / affine)
            double wsum = 0.0;
            for (size_t q = 0; q < qw.size(); q++) wsum += qw[q];
            for (size_t q = 0; q < qw.size(); q++)
                for (int k = 0; k < nen * dim; k++) cg[k] += qw[q] / wsum * qg[q * nen * dim + k];
        }
        // pattern / plan uploads
        std::vector<int32_t> cells(mesh->cells, mesh->cells + (size_t)mesh->n_cells * nen);
        if ((rc = upload(h, hp.row_ptr, &h->row_ptr, st)) || (rc = upload(h, hp.col_idx, &h->col_idx, st)) ||
            (rc = upload(h, cells, &h->cells, st)) || (rc = upload(h, hp.geo, &h->geo, st))) {
            free_handle(h); return rc;
        }
        const int64_t base_bytes = h->stats.device_bytes;
        if ((rc = upload(h, hp.grp_info, &h->grp_info, st)) || (rc = upload(h, hp.grp_nodes, &h->grp_nodes, st)) ||
            (rc = upload(h, hp.grp_elems, &h->grp_elems, st)) || (rc = upload(h, hp.grp_n2l, &h->grp_n2l, st)) ||
            (rc = upload(h, hp.grp_rows, &h->grp_rows, st)) ||
            (hp.canonical && (rc = upload(h, hp.grp_rank_off, &h->grp_rank_off, st))) ||
            (hp.canonical && (rc = upload(h, hp.grp_rank, &h->grp_rank, st))) ||
            (hp.canonical && (rc = upload(h, hp.elem_by_rank, &h->elem_by_rank, st))) ||
            (hp.canonical && (rc = upload(h, hp.geo_rank, &h->geo_rank, st))) ||
            (rc = upload(h, hp.sig_info, &h->sig_info, st)) || (rc = upload(h, hp.sig_pos_ptr, &h->sig_pos_ptr, st)) ||
            (rc = upload(h, hp.sig_contrib, &h->sig_contrib, st)) || (rc = upload(h, hp.sig_pairs, &h->sig_pairs, st)) ||
            (rc = upload(h, hp.sig_witems, &h->sig_witems, st)) || (rc = upload(h, hp.sig_witem_ptr, &h->sig_witem_ptr, st))) {
            free_handle(h); return rc;
        }
        h->stats.plan_bytes = h->stats.device_bytes - base_bytes;
        h->n_rank_bytes = (int64_t)hp.grp_rank.size();
        if ((rc = upload(h, hp.pos, &h->pos, st)) || (rc = upload(h, hp.nb_tslot, &h->nb_tslot, st)) ||
            (rc = upload(h, hp.nb, &h->nb, st)) || (rc = upload(h, hp.nb_tdeg, &h->nb_tdeg, st)) || (rc = upload(h, M, &h->M, st)) ||
            (rc = upload(h, M32, &h->M32, st)) ||
            (rc = upload(h, qw, &h->qw, st)) || (rc = upload(h, qg, &h->qgrad, st)) ||
            (rc = upload(h, qg32, &h->qgrad32, st)) || (rc = upload(h, cg, &h->cgrad, st)) ||
            (rc = upload(h, xref, &h->xref, st))) {
            free_handle(h); return rc;
        }
        if (hp.general) {
            std::vector<double> xy(mesh->coords, mesh->coords + (size_t)mesh->n_nodes * dim);
            if ((rc = upload(h, xy, &h->coords, st)) || (rc = upload(h, hp.gptr, &h->gptr, st)) ||
                (rc = upload(h, hp.gent, &h->gent, st)) || (rc = upload(h, hp.gnode, &h->gnode, st)) ||
                (!hp.qgeo.empty() && (rc = upload(h, hp.qgeo, &h->qgeo, st)))) {
                free_handle(h);
                return rc;
            }
        }
        if (!hp.rg_info.empty() && (rc = row_group_tables(h, hp, st)) && rc != SOPTX_E_OOM) {
            free_handle(h);
            return rc;
        }
        if (hipStreamSynchronize(st) != hipSuccess) { free_handle(h); return SOPTX_E_DEVICE; }
        const int64_t ncontrib = hp.n_cells * (int64_t)nen * nen;
        h->stats.ndof = hp.ndof; h->stats.nnz = hp.nnz; h->stats.n_cells = hp.n_cells; h->stats.n_nodes = hp.n_nodes;
        h->stats.n_groups = h->ngroups; h->stats.n_signatures = h->nsig; h->stats.n_contributions = ncontrib;
        for (int64_t g = 0; g < h->ngroups; g++)
            h->stats.n_groups_diag += (hp.grp_info[g * kGrpInfo + kGrpInfo - 1] & kGrpDiag) ? 1 : 0;
        for (int32_t ro : hp.grp_rank_off) h->stats.n_groups_ranked += ro >= 0 ? 1 : 0;
    } catch (const std::bad_alloc &) {
        free_handle(h);
        return SOPTX_E_OOM;
    }
    *out = h;
    return SOPTX_OK;
}

int soptx_build_pattern_ex(const soptx_mesh *mesh, int32_t ref_method, soptx_pattern *out, void *stream) {
    return build_pattern(mesh, ref_method, false, out, stream);
}

int soptx_build_pattern(const soptx_mesh *mesh, soptx_pattern *out, void *stream) {
    return soptx_build_pattern_ex(mesh, SOPTX_REF_SYMBOLIC, out, stream);
}

int soptx_build_pattern_general(const soptx_mesh *mesh, soptx_pattern *out, void *stream) {
    return build_pattern(mesh, SOPTX_REF_SYMBOLIC, true, out, stream);
}

static int asm_params(soptx_pattern h, const soptx_material *m, const void *d_rho, double *d_K_vals, int32_t prec,
                      hipStream_t st, AsmParams &P);
static int assemble_general_ke(soptx_pattern h, const soptx_material *m, const double *d_rho, double *d_K_vals,
                               hipStream_t st);

// which assembly general handles of Q1 elements run (soptx_debug_set_general_variant)
static std::atomic<int> g_general_variant{-1};

// the form of soptx_assemble_general on this handle: 1 = in LDS with the
// blocks' sums in registers (k_assemble_point), 2 = in LDS with the sums in
// the stage (k_assemble_quad), 3 = Q2 hexahedra by row groups
// (k_assemble_hex27), 0 = element matrices through memory
static int general_form(soptx_pattern h) {
    const int v = g_general_variant.load();
    if (h->n_row_groups > 0 && v != 0) return 3;
    if (!h->qgeo || v == 0) return 0;
    if (v != 1 && assemble_point_fits(h->elem, h->n_cells, h->stage, h->kmax, h->max_items)) return 1;
    if (assemble_quad_fits(h->elem, h->stage, h->kmax)) return 2;
    return 0;
}

int soptx_assemble_general(soptx_pattern h, const soptx_material *m, const double *d_rho, const uint8_t *d_dirichlet,
                           double *d_K_vals, void *stream) {
    if (!h) return SOPTX_E_INVALID_ARG;
    if (!h->general) return SOPTX_E_INVALID_ARG;
    int rc = check_material(m);
    if (rc) return rc;
    if ((h->n_cells > 0 && !d_rho) || (h->nnz > 0 && !d_K_vals)) return SOPTX_E_INVALID_ARG;
    if (h->nnz == 0) return SOPTX_OK;
    if (h->elem != SOPTX_QUAD4 && h->elem != SOPTX_HEX8 && h->elem != SOPTX_HEX27) return SOPTX_E_UNSUPPORTED_ELEM;
    DeviceGuard dg(h->device);
    if (!dg.ok) return SOPTX_E_DEVICE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int form = general_form(h);
    if (form == 3) {
        Hex27Params P{};
        P.info = h->rg_info; P.rows = h->rg_rows; P.vis = h->rg_vis; P.pairs = h->rg_pairs; P.ext = h->rg_ext;
        P.code = h->rg_code; P.geo = h->geo27; P.rho = d_rho; P.K = d_K_vals;
        P.n_groups = (int)h->n_row_groups; P.n_cu = h->n_cu;
        P.E0 = m->E0; P.Emin = m->Emin; P.p = m->p; P.ip = int_exponent(m->p);
        lame(h, m, &P.lam, &P.mu);
        if (launch_assemble_hex27(P, st) != hipSuccess) return SOPTX_E_DEVICE;
    } else if (form) {
        AsmParams P{};
        if ((rc = asm_params(h, m, d_rho, d_K_vals, kF64, st, P))) return rc;
        P.qgeo = h->qgeo;
        const hipError_t e = form == 1 ? launch_assemble_point(h->elem, P, h->ngroups, st)
                                       : launch_assemble_quad(h->elem, P, h->ngroups, st);
        if (e != hipSuccess) return SOPTX_E_DEVICE;
    } else {
        rc = assemble_general_ke(h, m, d_rho, d_K_vals, st);
        if (rc) return rc;
    }
    if (d_dirichlet && launch_dirichlet(h->dim, h->row_ptr, h->nb_tslot, h->nb_tdeg, d_dirichlet, d_K_vals, h->ndof, st) != hipSuccess)
        return SOPTX_E_DEVICE;
    return SOPTX_OK;
}

// the element-matrix path: every element's matrix to memory, then one
// gather per block of K in ascending element order
static int assemble_general_ke(soptx_pattern h, const soptx_material *m, const double *d_rho, double *d_K_vals,
                               hipStream_t st) {
    int rc;
    const int nen = h->nen, dim = h->dim;
    double *ke = nullptr;
    rc = get_workspace(h->device, st, (size_t)h->n_cells * nen * nen * dim * dim, &ke, 4);
    if (rc) return rc;
    double lam, mu;
    lame(h, m, &lam, &mu);
    GenParams G{};
    G.cells = h->cells; G.coords = h->coords; G.rho = d_rho; G.qw = h->qw; G.qgrad = h->qgrad;
    G.n_cells = h->n_cells; G.nq = h->nq; G.E0 = m->E0; G.Emin = m->Emin; G.p = m->p; G.ip = int_exponent(m->p);
    G.lam = lam; G.mu = mu; G.ke = ke;
    G.gptr = h->gptr; G.gent = h->gent; G.gnode = h->gnode; G.row_ptr = h->row_ptr; G.K = d_K_vals;
    G.n_blocks = h->nnz / (dim * dim);
    if (launch_assemble_general(h->elem, G, st) != hipSuccess) return SOPTX_E_DEVICE;
    return SOPTX_OK;
}

int soptx_pattern_info(soptx_pattern h, int64_t *ndof, int64_t *nnz, const int32_t **d_row_ptr,
                       const int32_t **d_col_idx) {
    if (!h) return SOPTX_E_INVALID_ARG;
    if (ndof) *ndof = h->ndof;
    if (nnz) *nnz = h->nnz;
    if (d_row_ptr) *d_row_ptr = h->row_ptr;
    if (d_col_idx) *d_col_idx = h->col_idx;
    return SOPTX_OK;
}

int soptx_pattern_copy(soptx_pattern h, int32_t *h_row_ptr, int32_t *h_col_idx) {
    if (!h) return SOPTX_E_INVALID_ARG;
    DeviceGuard dg(h->device);
    if (!dg.ok) return SOPTX_E_DEVICE;
    if (h_row_ptr && hipMemcpy(h_row_ptr, h->row_ptr, sizeof(int32_t) * (h->ndof + 1), hipMemcpyDeviceToHost) != hipSuccess)
        return SOPTX_E_DEVICE;
    if (h_col_idx && h->nnz > 0 &&
        hipMemcpy(h_col_idx, h->col_idx, sizeof(int32_t) * h->nnz, hipMemcpyDeviceToHost) != hipSuccess)
        return SOPTX_E_DEVICE;
    return SOPTX_OK;
}

int soptx_pattern_stats_get(soptx_pattern h, soptx_pattern_stats *out) {
    if (!h || !out) return SOPTX_E_INVALID_ARG;
    *out = h->stats;
    return SOPTX_OK;
}

// Parameters of the assembly kernel.  A canonical-order plan reads its
// geometry in rank order (geo_rank, built with the plan) and the caller's
// densities through its rank -> element map.
static int asm_params(soptx_pattern h, const soptx_material *m, const void *d_rho, double *d_K_vals, int32_t prec,
                      hipStream_t st, AsmParams &P) {
    P.grp_info = h->grp_info; P.grp_nodes = h->grp_nodes; P.grp_elems = h->grp_elems; P.grp_n2l = h->grp_n2l;
    P.grp_rows = h->grp_rows; P.n_groups = h->ngroups; P.n_cu = h->n_cu;
    P.grp_rank_off = h->grp_rank_off; P.grp_rank = h->grp_rank;
    P.sig_info = h->sig_info; P.sig_pos_ptr = h->sig_pos_ptr; P.sig_contrib = h->sig_contrib;
    P.sig_pairs = h->sig_pairs; P.sig_witems = h->sig_witems; P.sig_witem_ptr = h->sig_witem_ptr;
    P.geo = h->geo; P.rho = d_rho;
    if (h->elem_by_rank) {
        // canonical order: the geometry columns in rank order (a copy made
        // with the plan); the densities read through the rank -> element map
        P.geo = h->geo_rank;
        P.elem_by_rank = h->elem_by_rank;
    }
    P.M = h->M; P.M32 = h->M32; P.K = d_K_vals;
    P.n_cells = h->n_cells; P.E0 = m->E0; P.Emin = m->Emin; P.p = m->p; P.ip = int_exponent(m->p);
    lame(h, m, &P.lam, &P.mu);
    P.kmax = h->kmax; P.stage = h->stage;
    return SOPTX_OK;
}

int soptx_assemble(soptx_pattern h, const soptx_material *m, const void *d_rho, const uint8_t *d_dirichlet,
                   double *d_K_vals, int32_t prec, void *stream) {
    if (!h || !valid_prec(prec)) return SOPTX_E_INVALID_ARG;
    if (!h->affine) return not_affine(h);
    int rc = check_material(m);
    if (rc) return rc;
    if ((h->n_cells > 0 && !d_rho) || (h->nnz > 0 && !d_K_vals)) return SOPTX_E_INVALID_ARG;
    if (h->nnz == 0) return SOPTX_OK;
    DeviceGuard dg(h->device);
    if (!dg.ok) return SOPTX_E_DEVICE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    AsmParams P{};
    if ((rc = asm_params(h, m, d_rho, d_K_vals, prec, st, P))) return rc;
    if (launch_assemble(h->elem, prec, P, h->ngroups, st) != hipSuccess) return SOPTX_E_DEVICE;
    if (d_dirichlet && launch_dirichlet(h->dim, h->row_ptr, h->nb_tslot, h->nb_tdeg, d_dirichlet, d_K_vals, h->ndof, st) != hipSuccess)
        return SOPTX_E_DEVICE;
    return SOPTX_OK;
}

int soptx_apply_dirichlet(soptx_pattern h, const uint8_t *d_dirichlet, double *d_K_vals, void *stream) {
    if (!h || !d_dirichlet || (h->nnz > 0 && !d_K_vals)) return SOPTX_E_INVALID_ARG;
    if (h->nnz == 0) return SOPTX_OK;
    DeviceGuard dg(h->device);
    if (!dg.ok) return SOPTX_E_DEVICE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (launch_dirichlet(h->dim, h->row_ptr, h->nb_tslot, h->nb_tdeg, d_dirichlet, d_K_vals, h->ndof, st) != hipSuccess)
        return SOPTX_E_DEVICE;
    return SOPTX_OK;
}

int soptx_spmv(soptx_pattern h, const double *d_K_vals, const double *d_x, double *d_y, void *stream) {
    if (!h || (h->nnz > 0 && (!d_K_vals || !d_x)) || (h->ndof > 0 && !d_y)) return SOPTX_E_INVALID_ARG;
    if (h->ndof == 0) return SOPTX_OK;
    DeviceGuard dg(h->device);
    if (!dg.ok) return SOPTX_E_DEVICE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (launch_spmv(h->dim, h->row_ptr, h->nb, d_K_vals, d_x, d_y, nullptr, h->n_nodes, st) != hipSuccess)
        return SOPTX_E_DEVICE;
    return SOPTX_OK;
}

// which iteration small systems run (soptx_debug_set_pcg_variant)
static std::atomic<int> g_pcg_variant{-1};

int soptx_debug_fail_optional(int32_t skip, int32_t n) {
    if (skip < 0 || n < 0) return SOPTX_E_INVALID_ARG;
    std::lock_guard<std::mutex> lk(g_fail_mu);
    g_fail_skip = skip;
    g_fail_count = n;
    return SOPTX_OK;
}

int soptx_debug_set_pcg_variant(int32_t v) {
    if (v != -1 && v != 0) return SOPTX_E_INVALID_ARG;
    g_pcg_variant = v;
    return SOPTX_OK;
}

int soptx_pcg(soptx_pattern h, const double *d_K_vals, const double *d_f, double *d_u, double rtol,
              int32_t max_iter, int32_t *h_iters, double *h_relres, void *stream) {
    if (!h || !h_iters || !h_relres || max_iter < 0 || !(rtol >= 0.0)) return SOPTX_E_INVALID_ARG;
    if (h->ndof > 0 && (!d_K_vals || !d_f || !d_u)) return SOPTX_E_INVALID_ARG;
    *h_iters = 0;
    *h_relres = 0.0;
    if (h->ndof == 0) return SOPTX_OK;
    DeviceGuard dg(h->device);
    if (!dg.ok) return SOPTX_E_DEVICE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int64_t n = h->ndof;
    const int64_t nbv = cg_vec_blocks(h->dim, n);            // blocks of the vector kernels
    const int64_t nbs = spmv_blocks(h->dim, h->n_nodes);      // blocks of the SpMV
    const int64_t npart = std::max<int64_t>(3 * nbv, nbs);
    // Small systems run two launches per iteration that form the scalars
    // themselves: each of their blocks re-reads the other launch's partials,
    // which pays while that is a few MB (nbs * nbv doubles); both forms give the
    // same bits.
    bool small = g_pcg_variant.load() != 0 && nbs * nbv <= (int64_t)1 << 22;
    // r, z, p, q, the node blocks of the preconditioner (DIM doubles per dof),
    // partials, 2 x 8 scalars, a stop record; small systems: a second p (where
    // there is memory for it)
    const size_t base = (4 + (size_t)h->dim) * (size_t)n + (size_t)npart + 2 * (size_t)nbv + 20;
    double *ws = nullptr;
    if (small) small = !fail_optional() && get_workspace(h->device, st, base + (size_t)n, &ws, 1) == SOPTX_OK;
    int rc = SOPTX_OK;
    if (!small && (rc = get_workspace(h->device, st, base, &ws, 1))) return rc;
    double *r = ws, *z = r + n, *p = z + n, *q = p + n, *binv = q + n, *part = binv + h->dim * n,
           *part2 = part + npart, *sc = part2 + 2 * nbv, *fin = sc + 16, *p2 = fin + 4;
    double hs[8];
    auto scalars = [&]() {
        if (hipMemcpyAsync(hs, sc, sizeof(hs), hipMemcpyDeviceToHost, st) != hipSuccess) return false;
        return hipStreamSynchronize(st) == hipSuccess;
    };
    // r = f - K u, z = B^-1 r, p = z
    if (launch_block_inv(h->dim, h->row_ptr, h->nb, d_K_vals, binv, h->n_nodes, st) != hipSuccess ||
        launch_spmv(h->dim, h->row_ptr, h->nb, d_K_vals, d_u, q, nullptr, h->n_nodes, st) != hipSuccess ||
        launch_cg_vec(h->dim, 0, d_f, d_u, r, z, p, q, binv, sc, part, n, st) != hipSuccess ||
        launch_cg_scalars(0, part, (int)nbv, sc, st) != hipSuccess ||
        launch_cg_scalars(3, part + 2 * nbv, (int)nbv, sc, st) != hipSuccess || !scalars())
        return SOPTX_E_DEVICE;
    const double rr0 = hs[4];
    if (!(rr0 > 0.0)) {  // u already solves the system (or the data hold a NaN)
        *h_relres = rr0 == 0.0 ? 0.0 : NAN;
        return SOPTX_OK;
    }
    // the residual is measured against ||f|| (against ||r_0|| when f = 0): from
    // u = 0 the two agree, and a start near the solution then needs fewer steps
    const double ref = hs[6] > 0.0 ? hs[6] : rr0;
    if (!(std::sqrt(rr0 / ref) > rtol)) {
        *h_relres = std::sqrt(rr0 / ref);
        return SOPTX_OK;
    }
    // the residual is checked every kCheck iterations
    constexpr int kCheck = 8;
    int it = 0;
    double rel = 1.0;
    // two launches per iteration
    auto pcg_small = [&](StopRecord &rec) -> int {
        CgStep A{};
        A.row_ptr = h->row_ptr; A.nb = h->nb; A.K = d_K_vals; A.binv = binv;
        A.u = d_u; A.r = r; A.z = z; A.q = q; A.p[0] = p; A.p[1] = p2;
        A.pq_part = part; A.rz_part = part2; A.n_pq = (int)nbs; A.n_rz = (int)nbv;
        A.sc = sc; A.fin = fin; A.host = rec.dev; A.ref = ref; A.rtol = rtol; A.n_nodes = h->n_nodes;
        // the record of a stop starts as "none"
        if (launch_cg_clear(fin, 4, st) != hipSuccess) return SOPTX_E_DEVICE;
        // The launches of kAhead iterations past a check are enqueued before
        // its result is waited for, so the device does not idle meanwhile.
        constexpr int kAhead = 4;
        bool waiting = false;
        for (it = 0; it < max_iter; it++) {
            const bool check = it > 0 && it % kCheck == 0;
            if (launch_cg_step(h->dim, A, it, check, st) != hipSuccess) return SOPTX_E_DEVICE;
            if (check) {
                if (hipEventRecord(rec.event, st) != hipSuccess) return SOPTX_E_DEVICE;
                waiting = true;
            }
            if (launch_cg_step_vec(h->dim, A, it, st) != hipSuccess) return SOPTX_E_DEVICE;
            if (waiting && it % kCheck == kAhead) {
                waiting = false;
                if (hipEventSynchronize(rec.event) != hipSuccess) return SOPTX_E_DEVICE;
                if (rec.host[0] != 0.0) break;
            }
        }
        if (launch_cg_step_end(A, max_iter, st) != hipSuccess || hipStreamSynchronize(st) != hipSuccess)
            return SOPTX_E_DEVICE;
        *h_iters = (int32_t)rec.host[1];
        *h_relres = std::sqrt(rec.host[2] / ref);
        return SOPTX_OK;
    };
    if (small && max_iter > 0) {
        StopRecord rec(h->device, st);
        if (rec.host) return pcg_small(rec);
    }
    while (it < max_iter) {
        if (launch_spmv(h->dim, h->row_ptr, h->nb, d_K_vals, p, q, part, h->n_nodes, st) != hipSuccess ||
            launch_cg_scalars(1, part, (int)nbs, sc, st) != hipSuccess ||
            launch_cg_vec(h->dim, 1, d_f, d_u, r, z, p, q, binv, sc, part, n, st) != hipSuccess ||
            launch_cg_scalars(2, part, (int)nbv, sc, st) != hipSuccess ||
            launch_cg_p(p, z, sc, n, st) != hipSuccess)
            return SOPTX_E_DEVICE;
        it++;
        if (it % kCheck == 0 || it == max_iter) {
            if (!scalars()) return SOPTX_E_DEVICE;
            rel = std::sqrt(hs[3] / ref);
            if (!(rel > rtol)) break;  // converged, or broke down (NaN)
        }
    }
    *h_iters = it;
    *h_relres = rel;
    return SOPTX_OK;
}

// The element-energy kernel of soptx_evaluate and soptx_step: dc, and with
// d_c the fixed-order block partials of c and f^T u in the per-stream
// workspace or the fixed scratch (*ws, *nblk of each) for a finalize.
// Arguments are checked by the callers; the device is current.
static int launch_energies(soptx_pattern h, const soptx_material *m, const void *d_rho, const double *d_u,
                           const double *d_f, void *d_dc, double *d_c, int32_t prec, hipStream_t st, bool noalloc,
                           double **ws_out, int *nblk_out) {
    const int64_t nblk64 = std::max<int64_t>(1, (h->n_cells + 255) / 256);
    if (noalloc && d_c && nblk64 > kNoAllocBlocks) return SOPTX_E_SCRATCH;
    const int nblk = (int)nblk64;
    double *ws = nullptr;
    if (d_c) {
        // block partials of c, then of f^T u
        if (noalloc) {
            if (noalloc_scratch(h->device, &ws) != hipSuccess) return SOPTX_E_DEVICE;
        } else {
            const int rc = get_workspace(h->device, st, 2 * (size_t)nblk, &ws, 0);
            if (rc) return rc;
        }
    }
    EnergyParams P{};
    P.cells = h->cells; P.geo = h->geo; P.rho = d_rho; P.u = d_u;
    P.qw = h->qw; P.qgrad = h->qgrad; P.qgrad32 = h->qgrad32; P.cgrad = h->cgrad; P.xref = h->xref;
    P.dc = d_dc;
    P.f = d_c ? d_f : nullptr;
    P.ndof = h->ndof;
    P.partials = d_c ? ws : nullptr;
    P.axis_aligned = h->ngroups > 0 && h->stats.n_groups_diag == h->ngroups;
    P.n_cells = h->n_cells; P.E0 = m->E0; P.Emin = m->Emin; P.p = m->p; P.ip = int_exponent(m->p);
    lame(h, m, &P.lam, &P.mu);
    if (launch_energy(h->elem, prec, P, st) != hipSuccess) return SOPTX_E_DEVICE;
    *ws_out = ws;
    *nblk_out = nblk;
    return SOPTX_OK;
}

// soptx_evaluate and its allocation-free variant: the same kernels; the block
// partials of c go to the per-stream workspace or to the fixed scratch
static int evaluate_impl(soptx_pattern h, const soptx_material *m, const void *d_rho, const double *d_u,
                         const double *d_f, void *d_dc, double *d_c, int32_t prec, void *stream, bool noalloc) {
    if (!h || !valid_prec(prec)) return SOPTX_E_INVALID_ARG;
    if (!h->affine) return not_affine(h);
    int rc = check_material(m);
    if (rc) return rc;
    if (h->n_cells > 0 && (!d_rho || !d_u)) return SOPTX_E_INVALID_ARG;
    if (!d_dc && !d_c) return SOPTX_E_INVALID_ARG;
    if (noalloc && d_c && std::max<int64_t>(1, (h->n_cells + 255) / 256) > kNoAllocBlocks) return SOPTX_E_SCRATCH;
    DeviceGuard dg(h->device);
    if (!dg.ok) return SOPTX_E_DEVICE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    double *ws = nullptr;
    int nblk = 0;
    if ((rc = launch_energies(h, m, d_rho, d_u, d_f, d_dc, d_c, prec, st, noalloc, &ws, &nblk))) return rc;
    if (d_c && launch_finalize(ws, nblk, d_f ? 1 : 0, d_c, st) != hipSuccess) return SOPTX_E_DEVICE;
    return SOPTX_OK;
}

int soptx_evaluate(soptx_pattern h, const soptx_material *m, const void *d_rho, const double *d_u,
                   const double *d_f, void *d_dc, double *d_c, int32_t prec, void *stream) {
    return evaluate_impl(h, m, d_rho, d_u, d_f, d_dc, d_c, prec, stream, false);
}

int soptx_evaluate_noalloc(soptx_pattern h, const soptx_material *m, const void *d_rho, const double *d_u,
                           const double *d_f, void *d_dc, double *d_c, int32_t prec, void *stream) {
    return evaluate_impl(h, m, d_rho, d_u, d_f, d_dc, d_c, prec, stream, true);
}

int soptx_evaluate_general(soptx_pattern h, const soptx_material *m, const double *d_rho, const double *d_u,
                           const double *d_f, double *d_dc, double *d_c, void *stream) {
    if (!h || !h->general) return SOPTX_E_INVALID_ARG;
    int rc = check_material(m);
    if (rc) return rc;
    if (h->n_cells > 0 && (!d_rho || !d_u)) return SOPTX_E_INVALID_ARG;
    if (!d_dc && !d_c) return SOPTX_E_INVALID_ARG;
    if (h->elem != SOPTX_QUAD4 && h->elem != SOPTX_HEX8 && h->elem != SOPTX_HEX27) return SOPTX_E_UNSUPPORTED_ELEM;
    DeviceGuard dg(h->device);
    if (!dg.ok) return SOPTX_E_DEVICE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int per = h->elem == SOPTX_HEX27 ? kEnergyWideElems : 256;  // elements per partial
    const int nblk = std::max(1, (int)((h->n_cells + per - 1) / per));
    double *ws = nullptr;
    if (d_c) {
        rc = get_workspace(h->device, st, 2 * (size_t)nblk, &ws, 0);
        if (rc) return rc;
    }
    GenEnergyParams P{};
    P.cells = h->cells; P.coords = h->coords; P.rho = d_rho; P.u = d_u; P.qw = h->qw; P.qgrad = h->qgrad;
    P.dc = d_dc; P.f = d_c ? d_f : nullptr; P.ndof = h->ndof; P.partials = d_c ? ws : nullptr;
    P.n_cells = h->n_cells; P.nq = h->nq; P.E0 = m->E0; P.Emin = m->Emin; P.p = m->p; P.ip = int_exponent(m->p);
    lame(h, m, &P.lam, &P.mu);
    if (launch_energy_general(h->elem, P, st) != hipSuccess) return SOPTX_E_DEVICE;
    if (d_c && launch_finalize(ws, nblk, d_f ? 1 : 0, d_c, st) != hipSuccess) return SOPTX_E_DEVICE;
    return SOPTX_OK;
}

int soptx_sensitivity(soptx_pattern h, const soptx_material *m, const void *d_rho, const double *d_u,
                      void *d_dc, int32_t prec, void *stream) {
    if (h && h->n_cells > 0 && !d_dc) return SOPTX_E_INVALID_ARG;
    if (h && !h->affine) return not_affine(h);
    if (h && h->n_cells == 0) return (h && valid_prec(prec) && check_material(m) == 0) ? SOPTX_OK : SOPTX_E_INVALID_ARG;
    return soptx_evaluate(h, m, d_rho, d_u, nullptr, d_dc, nullptr, prec, stream);
}

int soptx_compliance(soptx_pattern h, const soptx_material *m, const void *d_rho, const double *d_u,
                     const double *d_f, double *d_c, int32_t prec, void *stream) {
    if (!d_c) return SOPTX_E_INVALID_ARG;
    return soptx_evaluate(h, m, d_rho, d_u, d_f, nullptr, d_c, prec, stream);
}

static int check_backward(soptx_pattern h, const soptx_material *m, const void *d_rho, const double *d_Kbar,
                          const void *d_drho, int32_t prec) {
    if (!h || !valid_prec(prec)) return SOPTX_E_INVALID_ARG;
    if (!h->affine) return not_affine(h);
    const int rc = check_material(m);
    if (rc) return rc;
    if (h->n_cells > 0 && (!d_rho || !d_Kbar || !d_drho)) return SOPTX_E_INVALID_ARG;
    return SOPTX_OK;
}

// The scratch of the backward on the plan's node groups: the parts of each
// element (one per local node) and a word of its fixed dofs.  0 where the
// element-by-element kernel runs in any case: 2D meshes whose calls cost their
// launches (two or three against one, and the group's chain of tables, rows
// and sums), up to a size that depends on the element and on whether the
// numbering keeps an element's rows near each other (a plan in the given
// order).  Element kernel against node groups, us without and with a mask,
// FP64:
//   quadrilaterals, given order: 2,500 cells 8.5 / 8.5, 14.6 / 11.0;
//     5,000 8.4 / 8.6, 14.5 / 11.3; 10,000 10.6 / 8.9, 16.5 / 11.3
//   canonical order: 400 9.1 / 8.7, 15.1 / 11.0; 2,500 14.7 / 9.2, 23.7 / 12.0
//   triangles, given order: 20,000 5.7 / 9.3, 9.1 / 12.0; 60,000 7.3 / 10.7,
//     10.5 / 13.4; 100,000 11.6 / 13.4, 16.1 / 16.1; 115,000 13.7 / 13.6, 18.7 / 16.4
//   canonical order: 5,000 7.3 / 9.7, 11.2 / 12.4; 7,200 10.1 / 9.7, 14.8 / 12.3
// In 3D the groups are the faster form from one element on (31.5 / 7.4, 64.9 /
// 9.9; 343 hexahedra 75 / 10, 137 / 12).
static int64_t backward_scratch_doubles(soptx_pattern h) {
    if (!h->affine) return 0;
    const bool canonical = h->elem_by_rank != nullptr;
    int64_t element_cells = 0;
    if (h->elem == SOPTX_QUAD4) element_cells = canonical ? 400 : 5000;
    if (h->elem == SOPTX_TRI3) element_cells = canonical ? 7000 : 100000;
    if (h->n_cells <= element_cells) return 0;
    return h->n_cells * (h->nen + 1);
}

int soptx_assemble_backward(soptx_pattern h, const soptx_material *m, const void *d_rho,
                            const uint8_t *d_dirichlet, const double *d_Kbar, void *d_drho, int32_t prec,
                            void *stream) {
    const int rc = check_backward(h, m, d_rho, d_Kbar, d_drho, prec);
    if (rc) return rc;
    if (h->n_cells == 0) return SOPTX_OK;
    DeviceGuard dg(h->device);
    if (!dg.ok) return SOPTX_E_DEVICE;
    BwdParams P{};
    P.cells = h->cells; P.row_ptr = h->row_ptr; P.pos = h->pos; P.geo = h->geo; P.rho = d_rho;
    P.Kbar = d_Kbar; P.M = h->M; P.M32 = h->M32; P.drho = d_drho; P.mask = d_dirichlet;
    P.n_cells = h->n_cells; P.E0 = m->E0; P.Emin = m->Emin; P.p = m->p; P.ip = int_exponent(m->p);
    lame(h, m, &P.lam, &P.mu);
    if (launch_backward(h->elem, prec, P, static_cast<hipStream_t>(stream)) != hipSuccess) return SOPTX_E_DEVICE;
    return SOPTX_OK;
}

int soptx_backward_scratch_size(soptx_pattern h, int64_t *bytes) {
    if (!h || !bytes) return SOPTX_E_INVALID_ARG;
    *bytes = backward_scratch_doubles(h) * (int64_t)sizeof(double);
    return SOPTX_OK;
}

int soptx_assemble_backward_scratch(soptx_pattern h, const soptx_material *m, const void *d_rho,
                                    const uint8_t *d_dirichlet, const double *d_Kbar, void *d_drho, int32_t prec,
                                    void *d_scratch, int64_t scratch_bytes, void *stream) {
    int rc = check_backward(h, m, d_rho, d_Kbar, d_drho, prec);
    if (rc) return rc;
    const int64_t need = backward_scratch_doubles(h);
    if (need == 0) return soptx_assemble_backward(h, m, d_rho, d_dirichlet, d_Kbar, d_drho, prec, stream);
    if (!d_scratch || reinterpret_cast<uintptr_t>(d_scratch) % sizeof(double) ||
        scratch_bytes < need * (int64_t)sizeof(double))
        return SOPTX_E_INVALID_ARG;
    DeviceGuard dg(h->device);
    if (!dg.ok) return SOPTX_E_DEVICE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    double *part = static_cast<double *>(d_scratch);
    BwdGroupParams B{};
    if ((rc = asm_params(h, m, d_rho, nullptr, prec, st, B.A))) return rc;
    B.Kbar = d_Kbar; B.mask = d_dirichlet; B.cells = h->cells; B.part = part;
    B.fixed = reinterpret_cast<uint32_t *>(part + h->n_cells * h->nen); B.drho = d_drho;
    if (launch_backward_group(h->elem, prec, B, h->ngroups, st) != hipSuccess) return SOPTX_E_DEVICE;
    return SOPTX_OK;
}

int soptx_build_dirichlet(soptx_pattern h, const uint8_t *h_mask, soptx_dirichlet *out, void *stream) {
    if (!out) return SOPTX_E_INVALID_ARG;
    *out = nullptr;
    if (!h || (h->ndof > 0 && !h_mask)) return SOPTX_E_INVALID_ARG;
    if (!h->affine) return not_affine(h);
    DeviceGuard dg(h->device);
    if (!dg.ok) return SOPTX_E_DEVICE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    soptx_dirichlet_s *bc = new (std::nothrow) soptx_dirichlet_s();
    if (!bc) return SOPTX_E_OOM;
    bc->h = h;
    bc->device = h->device;
    auto fail = [&](int code) {
        for (void *p : bc->allocs) (void)hipFree(p);
        delete bc;
        return code;
    };
    try {
        const int dim = h->dim, d2 = dim * dim;
        const int64_t G = h->ngroups;
        for (int64_t r = 0; r < h->ndof; r++) bc->n_fixed += h_mask[r] ? 1 : 0;
        // the plan's group tables and the neighbour lists, back from the device
        std::vector<int32_t> gi((size_t)G * kGrpInfo), si((size_t)h->nsig * 4), gn((size_t)G * kGroupNodes),
            rp((size_t)h->ndof + 1), nb((size_t)(h->nnz / d2));
        auto down = [&](std::vector<int32_t> &v, const int32_t *d) {
            return v.empty() || hipMemcpy(v.data(), d, v.size() * sizeof(int32_t), hipMemcpyDeviceToHost) == hipSuccess;
        };
        if (!down(gi, h->grp_info) || !down(si, h->sig_info) || !down(gn, h->grp_nodes) || !down(rp, h->row_ptr) ||
            !down(nb, h->nb))
            return fail(SOPTX_E_DEVICE);
        // canonical-order plans: the kernel's position p of a node is the CSR
        // position rank[p][lane] where the group has a rank table
        std::vector<int32_t> roff(h->grp_rank_off ? (size_t)G : 0);
        std::vector<uint8_t> rank(h->grp_rank ? (size_t)h->n_rank_bytes : 0);
        if (!down(roff, h->grp_rank_off) ||
            (!rank.empty() && hipMemcpy(rank.data(), h->grp_rank, rank.size(), hipMemcpyDeviceToHost) != hipSuccess))
            return fail(SOPTX_E_DEVICE);
        std::vector<int32_t> off((size_t)G, -1);
        std::vector<uint8_t> bits;
        if (bc->n_fixed > 0) {
            for (int64_t g = 0; g < G; g++) {
                const int nn = gi[(size_t)(kGrpInfo * g + 1)];
                const int deg = si[(size_t)(4 * gi[(size_t)(kGrpInfo * g)] + 1)];
                std::vector<uint8_t> gb((size_t)nn * deg, 0);
                bool any = false;
                for (int l = 0; l < nn; l++) {
                    const int64_t n = gn[(size_t)(g * kGroupNodes + l)];
                    int row = 0;
                    for (int a = 0; a < dim; a++) row |= h_mask[dim * n + a] ? 1 << a : 0;
                    const int64_t b0 = rp[(size_t)(dim * n)] / d2;
                    for (int p = 0; p < deg; p++) {
                        const int ro = roff.empty() ? -1 : roff[(size_t)g];
                        const int q = ro < 0 ? p : rank[(size_t)ro + (size_t)p * kGroupNodes + l];
                        const int64_t J = nb[(size_t)(b0 + q)];
                        int col = 0;
                        for (int c = 0; c < dim; c++) col |= h_mask[dim * J + c] ? 1 << (3 + c) : 0;
                        const int v = row | col | (J == n ? 64 : 0);
                        any = any || (row | col) != 0;
                        gb[(size_t)l * deg + p] = (uint8_t)v;
                    }
                }
                if (any) {
                    if (bits.size() + gb.size() >= (size_t)INT32_MAX) return fail(SOPTX_E_OVERFLOW);
                    off[(size_t)g] = (int32_t)bits.size();
                    bits.insert(bits.end(), gb.begin(), gb.end());
                    bc->n_groups++;
                }
            }
        }
        int rc;
        if ((rc = upload_vector(bc->allocs, off, &bc->off, st, &bc->device_bytes)) ||
            (rc = upload_vector(bc->allocs, bits, &bc->bits, st, &bc->device_bytes)))
            return fail(rc);
        if (hipStreamSynchronize(st) != hipSuccess) return fail(SOPTX_E_DEVICE);
    } catch (const std::bad_alloc &) {
        return fail(SOPTX_E_OOM);
    }
    *out = bc;
    return SOPTX_OK;
}

int soptx_dirichlet_info(soptx_dirichlet bc, int64_t *n_fixed, int64_t *n_groups) {
    if (!bc) return SOPTX_E_INVALID_ARG;
    if (n_fixed) *n_fixed = bc->n_fixed;
    if (n_groups) *n_groups = bc->n_groups;
    return SOPTX_OK;
}

void soptx_destroy_dirichlet(soptx_dirichlet bc) {
    if (!bc) return;
    DeviceGuard dg(bc->device);
    for (void *p : bc->allocs) (void)hipFree(p);
    delete bc;
}

int soptx_step(soptx_pattern h, soptx_dirichlet bc, const soptx_material *m, const void *d_rho, const double *d_u,
               const double *d_f, double *d_K_vals, void *d_dc, double *d_c, int32_t prec, void *stream) {
    if (!h || !valid_prec(prec)) return SOPTX_E_INVALID_ARG;
    if (!h->affine) return not_affine(h);
    int rc = check_material(m);
    if (rc) return rc;
    if (bc && bc->h != h) return SOPTX_E_INVALID_ARG;
    if ((h->n_cells > 0 && !d_rho) || (h->nnz > 0 && !d_K_vals)) return SOPTX_E_INVALID_ARG;
    if (h->n_cells > 0 && (d_dc || d_c) && !d_u) return SOPTX_E_INVALID_ARG;
    DeviceGuard dg(h->device);
    if (!dg.ok) return SOPTX_E_DEVICE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    // element energies and dc first (the kernel of soptx_evaluate; it does
    // not read K), so that the assembly kernel can add the partials of c in
    // the step where its store waves have nothing to store yet: the same
    // function and order as soptx_evaluate's finalize, one launch fewer
    double *ws = nullptr;
    int nblk = 0;
    if ((d_dc || d_c) && (rc = launch_energies(h, m, d_rho, d_u, d_f, d_dc, d_c, prec, st, false, &ws, &nblk)))
        return rc;
    // assembly with the Dirichlet table applied while the blocks are staged
    if (h->ngroups > 0) {
        AsmParams P{};
        if ((rc = asm_params(h, m, d_rho, d_K_vals, prec, st, P))) return rc;
        P.bc_off = (bc && bc->n_groups > 0) ? bc->off : nullptr;
        P.bc_bits = bc ? bc->bits : nullptr;
        if (d_c) {
            P.fin_partials = ws;
            P.fin_n = nblk;
            P.fin_with_f = d_f ? 1 : 0;
            P.fin_c = d_c;
        }
        if (launch_assemble(h->elem, prec, P, h->ngroups, st, true) != hipSuccess) return SOPTX_E_DEVICE;
    } else if (d_c && launch_finalize(ws, nblk, d_f ? 1 : 0, d_c, st) != hipSuccess) {
        return SOPTX_E_DEVICE;
    }
    return SOPTX_OK;
}

void soptx_destroy_pattern(soptx_pattern h) {
    if (!h) return;
    DeviceGuard dg(h->device);
    free_handle(h);
}

// ----------------------------------------------------------- host-only debug

int soptx_debug_set_general_variant(int32_t v) {
    if (v < -1 || v > 1) return SOPTX_E_INVALID_ARG;
    g_general_variant.store(v);
    return SOPTX_OK;
}

int soptx_debug_general_path(soptx_pattern h, int32_t *form) {
    if (!h || !form || !h->general) return SOPTX_E_INVALID_ARG;
    *form = general_form(h);
    return SOPTX_OK;
}

int soptx_debug_set_assembly_variant(int32_t v) {
    if (v < -1 || v > 1) return SOPTX_E_INVALID_ARG;
    set_assembly_variant(v);
    return SOPTX_OK;
}

int soptx_debug_host_plan(const soptx_mesh *mesh, soptx_host_plan *out) {
    return soptx_debug_host_plan_ex(mesh, 0, out);
}

int soptx_debug_host_plan_ex(const soptx_mesh *mesh, int32_t general, soptx_host_plan *out) {
    if (!out) return SOPTX_E_INVALID_ARG;
    *out = nullptr;
    soptx_host_plan_s *p = new (std::nothrow) soptx_host_plan_s();
    if (!p) return SOPTX_E_OOM;
    int rc;
    try {
        rc = build_host_plan(mesh, p->hp, general != 0);
    } catch (...) {
        rc = SOPTX_E_OOM;
    }
    if (rc) { delete p; return rc; }
    *out = p;
    return SOPTX_OK;
}

int soptx_debug_host_plan_array(soptx_host_plan p, const char *name, const void **data, int64_t *count,
                                int32_t *elem_bytes) {
    if (!p || !name || !data || !count || !elem_bytes) return SOPTX_E_INVALID_ARG;
    const HostPlan &hp = p->hp;
#define SOPTX_ARR(N)                                            \
    if (std::strcmp(name, #N) == 0) {                           \
        *data = hp.N.data();                                    \
        *count = (int64_t)hp.N.size();                         \
        *elem_bytes = (int32_t)sizeof(hp.N[0]);                 \
        return SOPTX_OK;                                        \
    }
    SOPTX_ARR(row_ptr) SOPTX_ARR(col_idx) SOPTX_ARR(geo) SOPTX_ARR(sig_info) SOPTX_ARR(sig_pos_ptr)
    SOPTX_ARR(sig_contrib) SOPTX_ARR(sig_pairs) SOPTX_ARR(sig_witems) SOPTX_ARR(sig_witem_ptr) SOPTX_ARR(grp_info) SOPTX_ARR(grp_nodes) SOPTX_ARR(grp_elems)
    SOPTX_ARR(grp_n2l) SOPTX_ARR(grp_rows) SOPTX_ARR(grp_rank_off) SOPTX_ARR(grp_rank) SOPTX_ARR(elem_by_rank)
    SOPTX_ARR(pos)
    SOPTX_ARR(nb_tslot) SOPTX_ARR(nb_tdeg)
    SOPTX_ARR(gptr) SOPTX_ARR(gent) SOPTX_ARR(gnode) SOPTX_ARR(qgeo)
    SOPTX_ARR(rg_info) SOPTX_ARR(rg_rows) SOPTX_ARR(rg_vis) SOPTX_ARR(rg_pairs) SOPTX_ARR(rg_code) SOPTX_ARR(rg_ext)
#undef SOPTX_ARR
    return SOPTX_E_INVALID_ARG;
}

int soptx_debug_host_plan_scalars(soptx_host_plan p, int64_t *out8) {
    if (!p || !out8) return SOPTX_E_INVALID_ARG;
    const HostPlan &hp = p->hp;
    out8[0] = hp.ndof; out8[1] = hp.nnz; out8[2] = hp.n_groups(); out8[3] = hp.n_sigs();
    out8[4] = hp.emax; out8[5] = hp.kmax; out8[6] = hp.dim; out8[7] = hp.nen;
    return SOPTX_OK;
}

void soptx_debug_host_plan_free(soptx_host_plan p) { delete p; }

}  // extern "C"
