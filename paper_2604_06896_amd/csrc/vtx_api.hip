// Host side of the libvtx C ABI: validation and staging of the half-edge
// table, workspace ownership, the relaxation and CG drivers (device loops
// replayed as HIP graphs, the host reading their state now and then), and the
// hypergradient entry point.
#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstddef>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "vtx_launch.h"

namespace vtx {
// Rebuild the tissue's fused-evaluation tables after its topology changed
// (on stream s, in order with the change).
int tissue_topology_changed(vtx_tissue t, hipStream_t s);
}

using namespace vtx;

// ------------------------------------------------- allocation-free scratch
// Fixed device scratch of vtx_energy_forces_noalloc: the per-tile partial
// sums and two loop control blocks of one fused evaluation, for tissues of
// up to kNoAllocVerts vertices (a 3-valent periodic tissue has half as many
// cells).  Every GPU the library runs on holds one copy until the process
// ends.  In host code `scratch` names a host-side stand-in; its device
// address comes from hipGetSymbolAddress (noalloc_scratch).
namespace {
constexpr int64_t kNoAllocVerts = 1 << 18;
constexpr size_t kNoAllocMpartBytes = 16 * (size_t)((kNoAllocVerts + kTileV - 1) / kTileV);
constexpr size_t kNoAllocCtlOffset = (kNoAllocMpartBytes + 255) & ~(size_t)255;
constexpr size_t kNoAllocBytes = kNoAllocCtlOffset + ((2 * sizeof(LoopCtl) + 255) & ~(size_t)255);
}  // namespace

static __device__ __align__(256) unsigned char scratch[kNoAllocBytes];

// Clears the two control blocks in the scratch (a kernel, not a memset, so a
// caller may capture the call in a graph).
__global__ void k_clear_ctl(LoopCtl *ctl) {
    const int n = (int)(2 * sizeof(LoopCtl) / sizeof(uint32_t));
    uint32_t *w = reinterpret_cast<uint32_t *>(ctl);
    for (int i = threadIdx.x; i < n; i += blockDim.x) w[i] = 0u;
}

struct vtx_tissue_s {
    DevTissue d;
    Workspace w;
    TileTables tiles;    // fused evaluation; rebuilt in stream order after topology changes
    int64_t n_vert, n_cell, n_edge, n_he;
    double *ep_buf;      // two position buffers for EP (double-sized)
    HessRows hess;       // one-launch CG step; allocated at the first solve that takes it
    int64_t t1_cap;
};

namespace {

thread_local std::string g_err = "no error";

int fail(int code, const char *fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
    return code;
}

#define HIPCHK(x)                                                                          \
    do {                                                                                   \
        hipError_t e_ = (x);                                                               \
        if (e_ != hipSuccess)                                                              \
            return fail(VTX_E_HIP, "%s failed: %s", #x, hipGetErrorString(e_));            \
    } while (0)

int check_launch(const char *what) {
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(VTX_E_HIP, "%s: %s", what, hipGetErrorString(e));
    return VTX_OK;
}

bool mode_ok(int m) { return m == VTX_F32 || m == VTX_F64 || m == VTX_MIXED; }

ParamsRaw raw(const vtx_params *p) {
    ParamsRaw r{p->KA, p->A0, p->KP, p->P0, p->lam, p->KA_s, p->A0_s, p->KP_s, p->P0_s, p->lam_s};
    return r;
}

// Largest tissue of the one-launch relaxation step, which computes each cell
// six times, without T1 and with, and its launches per captured graph.  Us a
// step of 300, against the loop of two launches (three with T1), in FP64, MIXED
// and FP32:
//   cells    without T1                             with T1 (no exchange)
//    5000     6.4/14.1   6.2/13.3   6.2/13.5   10.5/18.5  10.3/18.6   9.6/17.3 (41 exchanges)
//   20000     7.4/14.1   7.3/13.0   6.1/13.0    8.6/16.5   8.4/16.4   7.5/15.9
//   48400    11.6/14.8  11.5/13.0   8.7/14.2   14.4/15.9  13.9/15.6  12.7/16.6
//   53824    12.4/14.1  12.2/13.7  10.9/13.2   16.8/15.2  16.5/15.7  15.7/15.6
//   65536    14.3/14.1  13.8/14.6  12.0/13.8   19.6/17.6  18.9/17.0  16.8/15.8
// and 29/17 at 120000 cells without T1 in FP64.
constexpr int64_t kStepMaxVerts = 131072, kStepMaxVertsT1 = 98304;
constexpr int kStepChunk = 60;

// The same for the one-launch CG step (an even number of launches, so that
// every replay starts on the same vectors): what 256 blocks of 256 vertices
// hold.  Against the six-launch step, one solve: 9.7 and 36.8 ms at 5000
// cells, 54 and 91 at 32000.
constexpr int64_t kCgStepMaxVerts = 65536;
constexpr int kCgChunk = 256;
// Every vertex's rows have as many slots per lane as the largest cell needs
// (its sides - 2), and a step reads the columns of all of them (16 B a vertex
// and slot, 144 B of memory): limited to 1.5 million in all (24 MB, 216 MB).
// Against the six-launch step, a us per iteration with one cell of many sides:
// 20.5 and 23.7 (32000 cells, 24 sides: 1.4 million), 26.9 and 25.5 (32 sides:
// 1.9), 26.0 and 28.2 (20000 cells, 40 sides: 1.5), 39.2 and 34.8 (64: 2.5),
// 42.2 and 45.5 (5000 cells, 100 sides: 1.0).
constexpr int64_t kCgStepMaxSlots = 1500000;
static_assert(kCgStepMaxVerts <= (int64_t)kCgBlocks * kCgVerts, "vertices of a workgroup");

// Host copy of the staged layouts.
struct Staged {
    std::vector<int32_t> he_edge, edge_he, row_ptr, row_cap, corner, corner_he, nsides, cell_he;
    std::vector<int32_t> star, star_he;
};

int validate_and_stage(const int32_t *he, int64_t n_he, int64_t n_vert, int64_t n_cell,
                       Staged &S) {
    if (n_he <= 0 || n_he % 2 || n_vert <= 0 || n_cell <= 0)
        return fail(VTX_E_ARG, "bad sizes n_he=%lld n_vert=%lld n_cell=%lld", (long long)n_he,
                    (long long)n_vert, (long long)n_cell);
    if (n_vert >= (int64_t)kIdMask || n_he >= (int64_t)INT32_MAX / 2 || n_cell >= INT32_MAX)
        return fail(VTX_E_CAPACITY, "tissue too large (n_vert must be < 2^28)");
    auto R = [&](int64_t h, int c) { return he[8 * h + c]; };
    for (int64_t h = 0; h < n_he; ++h) {
        for (int c : {HP, HN, HT})
            if (R(h, c) < 0 || R(h, c) >= n_he)
                return fail(VTX_E_TOPOLOGY, "half-edge %lld: index out of range", (long long)h);
        if (R(h, HS) < 0 || R(h, HS) >= n_vert || R(h, HG) < 0 || R(h, HG) >= n_vert)
            return fail(VTX_E_TOPOLOGY, "half-edge %lld: vertex out of range", (long long)h);
        if (R(h, HF) < 0 || R(h, HF) >= n_cell)
            return fail(VTX_E_TOPOLOGY, "half-edge %lld: face out of range", (long long)h);
        if (R(h, HOX) < -1 || R(h, HOX) > 1 || R(h, HOY) < -1 || R(h, HOY) > 1)
            return fail(VTX_E_TOPOLOGY, "half-edge %lld: offset not in {-1,0,1}", (long long)h);
        const int64_t t = R(h, HT);
        if (t == h || R(t, HT) != h)
            return fail(VTX_E_TOPOLOGY, "half-edge %lld: twin is not an involution", (long long)h);
        if (R(t, HS) != R(h, HG) || R(t, HG) != R(h, HS) || R(t, HOX) != -R(h, HOX) ||
            R(t, HOY) != -R(h, HOY))
            return fail(VTX_E_TOPOLOGY, "half-edge %lld: twin does not reverse it", (long long)h);
        if (R(R(h, HN), HP) != h || R(R(h, HP), HN) != h)
            return fail(VTX_E_TOPOLOGY, "half-edge %lld: prev/next not inverse", (long long)h);
        if (R(R(h, HN), HS) != R(h, HG))
            return fail(VTX_E_TOPOLOGY, "half-edge %lld: source(next) != target", (long long)h);
        if (R(R(h, HN), HF) != R(h, HF))
            return fail(VTX_E_TOPOLOGY, "half-edge %lld: next leaves the face", (long long)h);
        if (R(h, HS) == R(h, HG))
            return fail(VTX_E_TOPOLOGY, "half-edge %lld joins a vertex to itself", (long long)h);
    }
    // edges: ascending lower half-edge id
    S.he_edge.assign(n_he, -1);
    S.edge_he.clear();
    for (int64_t h = 0; h < n_he; ++h) {
        const int64_t t = R(h, HT);
        if (h < t) {
            S.he_edge[h] = S.he_edge[t] = (int32_t)S.edge_he.size();
            S.edge_he.push_back((int32_t)h);
        }
    }
    // faces
    std::vector<int64_t> count(n_cell, 0);
    S.cell_he.assign(n_cell, -1);
    for (int64_t h = 0; h < n_he; ++h) {
        const int c = R(h, HF);
        if (S.cell_he[c] < 0) S.cell_he[c] = (int32_t)h;
        ++count[c];
    }
    S.nsides.assign(n_cell, 0);
    S.row_ptr.assign(n_cell + 1, 0);
    for (int64_t c = 0; c < n_cell; ++c) {
        if (S.cell_he[c] < 0) return fail(VTX_E_TOPOLOGY, "cell %lld has no half-edge", (long long)c);
        int64_t n = 0, h = S.cell_he[c];
        int sx = 0, sy = 0;
        do {
            sx += R(h, HOX);
            sy += R(h, HOY);
            h = R(h, HN);
            ++n;
        } while (h != S.cell_he[c] && n <= n_he);
        if (n != count[c])
            return fail(VTX_E_TOPOLOGY, "cell %lld is not a single cycle", (long long)c);
        if (n < 3) return fail(VTX_E_TOPOLOGY, "cell %lld has fewer than 3 sides", (long long)c);
        if (sx || sy)
            return fail(VTX_E_TOPOLOGY, "cell %lld: image offsets do not close", (long long)c);
        S.nsides[c] = (int32_t)n;
        S.row_ptr[c + 1] = S.row_ptr[c] + (int32_t)n;
    }
    S.row_cap.assign(S.nsides.begin(), S.nsides.end());
    // corner rows: compact rows, room to re-compact them with kRowSlack spare
    // slots each, then a relocation pool of n_he + 1024 slots
    const int64_t cap_total = 2 * n_he + kRowSlack * n_cell + 1024;
    if (cap_total >= INT32_MAX) return fail(VTX_E_CAPACITY, "tissue too large");
    S.corner.assign(cap_total, 0);
    S.corner_he.assign(cap_total, 0);
    for (int64_t c = 0; c < n_cell; ++c) {
        int64_t h = S.cell_he[c], k = S.row_ptr[c];
        int wx = 0, wy = 0;
        do {
            if (wx < -1 || wx > 1 || wy < -1 || wy > 1)
                return fail(VTX_E_CAPACITY, "cell %lld spans more than one periodic image",
                            (long long)c);
            S.corner[k] = pack_id(R(h, HS), wx, wy);
            S.corner_he[k] = (int32_t)h;
            wx += R(h, HOX);
            wy += R(h, HOY);
            h = R(h, HN);
            ++k;
        } while (h != S.cell_he[c]);
    }
    // vertex stars
    std::vector<int32_t> out_he(n_vert, -1), out_n(n_vert, 0);
    for (int64_t h = 0; h < n_he; ++h) {
        const int v = R(h, HS);
        if (out_he[v] < 0) out_he[v] = (int32_t)h;
        ++out_n[v];
    }
    S.star.assign(9 * n_vert, 0);
    S.star_he.assign(3 * n_vert, 0);
    for (int64_t v = 0; v < n_vert; ++v) {
        if (out_n[v] != 3)
            return fail(VTX_E_TOPOLOGY, "vertex %lld has %d edges (3 required)", (long long)v,
                        out_n[v]);
        int64_t h = out_he[v];
        for (int k = 0; k < 3; ++k) {
            if (R(h, HS) != v)
                return fail(VTX_E_TOPOLOGY, "vertex %lld: star does not close", (long long)v);
            S.star_he[k * n_vert + v] = (int32_t)h;
            S.star[star_nb_at(n_vert, k, v)] = pack_id(R(h, HG), R(h, HOX), R(h, HOY));
            S.star[star_cell_at(n_vert, k, v)] = R(h, HF);
            S.star[star_edge_at(n_vert, k, v)] = S.he_edge[h];
            h = R(R(h, HP), HT);
        }
        if (h != out_he[v])
            return fail(VTX_E_TOPOLOGY, "vertex %lld: star does not close", (long long)v);
    }
    return VTX_OK;
}

template <typename T>
int upload(T **dst, const std::vector<T> &src) {
    HIPCHK(hipMalloc((void **)dst, std::max<size_t>(1, src.size()) * sizeof(T)));
    if (!src.empty()) HIPCHK(hipMemcpy(*dst, src.data(), src.size() * sizeof(T), hipMemcpyHostToDevice));
    return VTX_OK;
}

int upload_into(int32_t *dst, const std::vector<int32_t> &src) {
    HIPCHK(hipMemcpy(dst, src.data(), src.size() * sizeof(int32_t), hipMemcpyHostToDevice));
    return VTX_OK;
}

void free_tissue(vtx_tissue t) {
    if (!t) return;
    DevTissue &d = t->d;
    void *ptrs[] = {d.he, d.he_edge, d.edge_he, d.row_ptr, d.row_cap, d.pool_top, d.corner,
                    d.corner_he, d.nsides,
                    d.cell_he, d.star, d.star_he, t->w.xbuf,
                    t->w.cap, t->w.cell_aux, t->w.partials, t->w.partials2, t->w.mpart,
                    t->w.t1_list,
                    t->w.ctl, t->w.cg, t->w.scal, t->w.one, t->w.step, t->w.step_part, t->w.step_tab,
                    t->w.cg_state, t->w.max_sides, t->hess.col, t->hess.top, t->hess.bottom,
                    t->hess.halo, t->hess.n_halo,
                    t->ep_buf,
                    t->tiles.cells, t->tiles.info, t->tiles.halo, t->tiles.cstart,
                    t->tiles.corners, t->tiles.fstar, t->tiles.fe};
    for (void *p : ptrs)
        if (p) (void)hipFree(p);
    if (t->w.ctl_host) (void)hipHostFree(t->w.ctl_host);
    if (t->w.step_host) (void)hipHostFree(t->w.step_host);
    if (t->w.cg_host) (void)hipHostFree(t->w.cg_host);
    if (t->w.cap_stream) (void)hipStreamDestroy(t->w.cap_stream);
    delete t;
}

int reset_ctl(vtx_tissue t, int which, const LoopCtl &init, hipStream_t s) {
    t->w.ctl_host[which] = init;
    HIPCHK(hipMemcpyAsync(t->w.ctl + which, t->w.ctl_host + which, sizeof(LoopCtl),
                          hipMemcpyHostToDevice, s));
    HIPCHK(hipStreamSynchronize(s));
    return VTX_OK;
}

int read_ctl(vtx_tissue t, int which, hipStream_t s) {
    HIPCHK(hipMemcpyAsync(t->w.ctl_host + which, t->w.ctl + which, sizeof(LoopCtl),
                          hipMemcpyDeviceToHost, s));
    HIPCHK(hipStreamSynchronize(s));
    return VTX_OK;
}

hipError_t fetch_ctl(vtx_tissue t, hipStream_t s) {
    return hipMemcpyAsync(t->w.ctl_host, t->w.ctl, sizeof(LoopCtl), hipMemcpyDeviceToHost, s);
}

size_t pos_bytes(vtx_tissue t, int mode) {
    return (size_t)t->n_vert * 2 * (mode == VTX_F32 ? sizeof(float) : sizeof(double));
}

// Device loop driver: runs steps of `body` on the device until the control
// block (copied by `read` into host memory, then asked by `done`) reports
// done, looked at after every look() steps.  Steps run as replays of a graph
// of `chunk` of them, captured when it is first needed, and what is left
// before a look, if less than two thirds of it, by direct launches, a
// multiple of 6 (k counts from 0 in both: for bodies that depend on k mod 2
// and 3).
template <typename Body, typename Read, typename Done, typename Look>
int run_loop(vtx_tissue t, int chunk, int64_t max_steps, hipStream_t s, Body body, Read read,
             Done done, Look look) {
    hipGraph_t g = nullptr;
    hipGraphExec_t ge = nullptr;
    auto replay = [&]() {
        hipError_t e = hipSuccess;
        if (!ge) {
            e = hipStreamBeginCapture(t->w.cap_stream, hipStreamCaptureModeThreadLocal);
            if (e != hipSuccess) return e;
            for (int k = 0; k < chunk; ++k) body(k, t->w.cap_stream);
            e = hipStreamEndCapture(t->w.cap_stream, &g);
            if (e == hipSuccess) e = hipGraphInstantiate(&ge, g, nullptr, nullptr, 0);
        }
        return e == hipSuccess ? hipGraphLaunch(ge, s) : e;
    };
    int rc = VTX_OK;
    for (int64_t queued = 0;;) {
        hipError_t e = hipSuccess;
        int64_t left = look();
        for (; left > 0 && e == hipSuccess; left -= chunk) {
            if (3 * left < 2 * (int64_t)chunk) {
                const int n = (int)(left + 5) / 6 * 6;
                for (int k = 0; k < n; ++k) body(k, s);
                e = hipGetLastError();
                queued += n;
                break;
            }
            e = replay();
            queued += chunk;
        }
        if (e == hipSuccess) e = read();
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        if (e != hipSuccess) {
            rc = fail(VTX_E_HIP, "device loop: %s", hipGetErrorString(e));
            break;
        }
        if (done()) break;
        if (queued >= max_steps + 2 * (int64_t)chunk) {
            rc = fail(VTX_E_HIP, "device loop did not report completion");
            break;
        }
    }
    if (ge) (void)hipGraphExecDestroy(ge);
    if (g) (void)hipGraphDestroy(g);
    return rc;
}

// Steps before the next look at a relaxation: those that it takes unless it
// converges, up to kLook.  Capturing a step costs as much as launching it
// (1.7 us), so the graph is short; replays follow each other without a gap
// that would show (500 steps of 3000 cells: 3.06 ms with graphs of 252 and a
// look after each, 2.59 with graphs of 60, 2.64 with direct launches only,
// which are bound by the host).
constexpr int64_t kLook = 252;
int64_t relax_look(const vtx_relax_opts *o, int chunk, int64_t iters) {
    if (o->chunk > 0) return chunk;
    return std::max<int64_t>(6, std::min(kLook, o->max_iter - iters + 1));
}

// The table of k_relax_step, kept from the first use on: three int4 for each of
// four lanes a vertex, in whole blocks.  False where the device has no room.
bool step_reserve(vtx_tissue t) {
    if (t->w.step_tab) return true;
    const size_t blocks = (4 * (size_t)t->n_vert + kBlock - 1) / kBlock;
    if (hipMalloc((void **)&t->w.step_tab, 3 * 16 * (size_t)kBlock * blocks) == hipSuccess)
        return true;
    t->w.step_tab = nullptr;
    (void)hipGetLastError();  // not an error of the call, which takes the other loop
    return false;
}

// The loop of one-launch steps (k_relax_step): no nudge, tissues of up to
// kStepMaxVerts vertices, their table reserved.
int relax_steps(vtx_tissue t, int mode, void *X, const vtx_params *p, const vtx_relax_opts *o,
                const RelaxArgs &ra, hipStream_t s, vtx_relax_result &r, int &overflow) {
    StepCtl &h = *t->w.step_host;
    h = StepCtl{};
    h.s[0].status = VTX_NOT_CONVERGED;
    HIPCHK(hipMemcpyAsync(t->w.step, &h, sizeof h, hipMemcpyHostToDevice, s));
    HIPCHK(hipStreamSynchronize(s));
    // (a multiple of 6: every replay starts at launch index 0 mod 2 and mod 3)
    const int chunk = ((o->chunk > 0 ? o->chunk : kStepChunk) + 5) / 6 * 6;
    // an iteration with a T1 pass takes three launches
    const int64_t most = ra.t1_enable ? 3 * std::min(o->max_iter, INT64_MAX / 4) : o->max_iter;
    int rc = run_loop(
        t, chunk, most + 1, s,
        [&](int k, hipStream_t cs) {
            launch_relax_step(t->d, t->w, mode, X, t->w.xbuf, raw(p), ra, o->tol, o->patience,
                              o->max_iter, k, cs);
        },
        [&]() { return hipMemcpyAsync(&h, t->w.step, sizeof h, hipMemcpyDeviceToHost, s); },
        [&]() { return h.s[0].done != 0; }, [&]() { return relax_look(o, chunk, h.s[0].iter); });
    const StepState &f = h.s[0];
    // (a loop without an exchange, and without an error, left the topology)
    if (ra.t1_enable && (rc || f.n_t1 > 0 || f.t1_overflow)) {
        const int rt = vtx::tissue_topology_changed(t, s);
        if (!rc) rc = rt;
    }
    if (rc) return rc;
    if (f.result_buf == 1)
        HIPCHK(hipMemcpyAsync(X, t->w.xbuf, pos_bytes(t, mode), hipMemcpyDeviceToDevice, s));
    r.iters = f.iter;
    r.n_t1 = f.n_t1;
    r.n_stretch = f.n_stretch;
    r.max_f = f.last_maxf;
    r.status = f.status;
    overflow = f.t1_overflow;
    return VTX_OK;
}

// The relaxation loop on the whole GPU: captured graphs of `chunk`
// iterations.  Leaves the result (all but the energy) in r and the T1 pass's
// overflow code in `overflow`, and the final positions in X.
int relax_grid(vtx_tissue t, int mode, void *X, const vtx_params *p, const vtx_relax_opts *o,
               const RelaxArgs &ra, hipStream_t s, vtx_relax_result &r, int &overflow) {
    if (!ra.nudge && t->n_vert <= (ra.t1_enable ? kStepMaxVertsT1 : kStepMaxVerts) &&
        step_reserve(t))
        return relax_steps(t, mode, X, p, o, ra, s, r, overflow);
    LoopCtl c{};
    c.status = VTX_NOT_CONVERGED;
    c.max_iter = o->max_iter;
    c.patience = o->patience;
    c.tol = o->tol;
    int rc = reset_ctl(t, 0, c, s);
    if (rc) return rc;
    if (ra.nudge == 2) {
        double *mean = (double *)((char *)t->w.ctl + offsetof(LoopCtl, nudge_mean));
        launch_mean_pos(t->w, VTX_F64, (int)t->n_vert, o->g_lin, mean, s);
        if ((rc = check_launch("nudge mean"))) return rc;
    }
    const int chunk = o->chunk > 0 ? o->chunk + (o->chunk & 1) : kStepChunk;  // (even: every
                                            // replay starts on the caller's buffer)
    void *bufs[2] = {X, t->w.xbuf};
    rc = run_loop(t, chunk, o->max_iter, s, [&](int k, hipStream_t cs) {
        const int cur = k & 1;
        launch_relax_iter(t->d, t->w, mode, bufs[cur], bufs[cur ^ 1], cur, raw(p), ra, cs);
    }, [&]() { return fetch_ctl(t, s); }, [&]() { return t->w.ctl_host[0].done != 0; },
       [&]() { return relax_look(o, chunk, t->w.ctl_host[0].iter); });
    const LoopCtl &h = t->w.ctl_host[0];
    // (a loop without an exchange, and without an error, left the topology)
    if (ra.t1_enable && (rc || h.n_t1 > 0 || h.t1_overflow)) {
        const int rt = vtx::tissue_topology_changed(t, s);
        if (!rc) rc = rt;
    }
    if (rc) return rc;
    if (h.result_buf == 1)
        HIPCHK(hipMemcpyAsync(X, t->w.xbuf, pos_bytes(t, mode), hipMemcpyDeviceToDevice, s));
    r.iters = h.iter;
    r.n_t1 = h.n_t1;
    r.n_stretch = h.n_stretch;
    r.max_f = h.last_maxf;
    r.status = h.status;
    overflow = h.t1_overflow;
    return VTX_OK;
}

int relax_impl(vtx_tissue t, int mode, void *X, const vtx_params *p, const vtx_relax_opts *o,
               vtx_relax_result *res, hipStream_t s) {
    if (!(o->eta > 0) || !(o->tol >= 0) || o->patience < 1 || o->max_iter < 1)
        return fail(VTX_E_ARG, "relax options: eta > 0, tol >= 0, patience >= 1, max_iter >= 1");
    RelaxArgs ra{};
    ra.eta = o->eta;
    ra.t1_enable = o->t1_enable != 0;
    ra.l_min = o->l_min;
    ra.l_new = o->l_new;
    ra.beta = o->beta;
    ra.X_target = o->X_target;
    ra.g_lin = o->g_lin;
    ra.nudge = o->beta != 0.0 ? (o->X_target ? 1 : (o->g_lin ? 2 : 0)) : 0;
    if (o->beta != 0.0 && ra.nudge == 0)
        return fail(VTX_E_ARG, "a nudge needs X_target or g_lin");
    if (ra.nudge && ra.t1_enable) return fail(VTX_E_ARG, "a nudge cannot be combined with T1");
    if (ra.t1_enable && !(o->l_min > 0 && o->l_new > 0))
        return fail(VTX_E_ARG, "T1 needs l_min > 0 and l_new > 0");
    vtx_relax_result r{};
    int overflow = 0;
    // A tissue that fits one workgroup's LDS runs its whole loop there.  Us a
    // step of 500 against the one-launch step, FP64, MIXED and FP32: without T1
    // 3.1/5.6, 2.8/5.7, 2.5/5.1 at 200 cells, 5.2/5.9, 4.5/5.9, 3.5/5.4 at 700,
    // 6.0/6.0, 5.3/6.1, 4.2/5.4 at 1024; with T1 3.7/6.4, 3.5/6.3, 2.8/6.1, then
    // 6.1/6.7, 5.5/6.8, 4.4/6.9, then 7.0/7.0, 6.2/7.0, 5.3/6.7.
    const vtx_relax_result *one = nullptr;
    int rc = relax_one(t->d, t->w, mode, X, raw(p), ra, o->tol, o->patience, o->max_iter, s, &one);
    if (rc) return rc;
    if (!one && (rc = relax_grid(t, mode, X, p, o, ra, s, r, overflow))) return rc;
    // energy (and nudge energy) at the returned positions
    launch_eval(t->d, t->w, mode, X, raw(p), t->w.scal + 4, nullptr, nullptr, s);
    if (ra.nudge == 1) launch_v2v(t->d, t->w, mode, X, o->X_target, t->w.scal + 5, nullptr, s);
    if (ra.nudge == 2)
        launch_dot_pos(t->w, mode, (int)t->n_vert, (const double *)o->g_lin, X, t->w.scal + 5, s);
    if ((rc = check_launch("final energy"))) return rc;
    double e[2] = {0, 0};
    if (one) HIPCHK(hipMemcpyAsync(&r, one, sizeof r, hipMemcpyDeviceToHost, s));
    HIPCHK(hipMemcpyAsync(e, t->w.scal + 4, 2 * sizeof(double), hipMemcpyDeviceToHost, s));
    HIPCHK(hipStreamSynchronize(s));
    // (waited for: the next call on the tissue may come on another stream)
    if (one && ra.t1_enable && (r.n_t1 > 0 || r.status == VTX_E_CAPACITY)) {
        if ((rc = vtx::tissue_topology_changed(t, s))) return rc;
        HIPCHK(hipStreamSynchronize(s));
    }
    if (r.status == VTX_E_CAPACITY) overflow = 3;
    const bool nonfinite = r.status == VTX_E_NONFINITE;
    r.energy = e[0] + (ra.nudge ? o->beta * e[1] : 0.0);
    if (r.status < 0) r.status = VTX_NOT_CONVERGED;
    if (res) *res = r;
    if (overflow == 1) return fail(VTX_E_CAPACITY, "T1 pass: too many pending re-checks");
    if (overflow == 2)
        return fail(VTX_E_CAPACITY, "T1 pass: corner-row pool exhausted or a cell spans two images");
    if (overflow == 3)
        return fail(VTX_E_CAPACITY, "T1 pass: too many pending re-checks, corner-row pool exhausted "
                                    "or a cell spans two images");
    if (nonfinite) return fail(VTX_E_NONFINITE, "non-finite forces in relaxation");
    return VTX_OK;
}

}  // namespace

namespace vtx {
const DevTissue &tissue_dev(vtx_tissue t) { return t->d; }
const Workspace &tissue_ws(vtx_tissue t) { return t->w; }
int64_t tissue_size(vtx_tissue t) { return t->n_vert; }
int64_t tissue_cells(vtx_tissue t) { return t->n_cell; }
double *tissue_ep_buf(vtx_tissue t) { return t->ep_buf; }
const TileTables &tissue_tiles(vtx_tissue t) { return t->tiles; }
int set_error(int code, const char *msg) { return fail(code, "%s", msg); }
int tissue_topology_changed(vtx_tissue t, hipStream_t s) {
    launch_tile_build(t->d, t->tiles, s);
    return check_launch("tile tables");
}
}  // namespace vtx

extern "C" {

const char *vtx_last_error(void) { return g_err.c_str(); }

int vtx_tissue_create(const int32_t *he, int64_t n_he, int64_t n_vert, int64_t n_cell, double Lx,
                      double Ly, vtx_tissue *out) {
    if (!he || !out) return fail(VTX_E_ARG, "null argument");
    if (!(Lx > 0) || !(Ly > 0) || !std::isfinite(Lx) || !std::isfinite(Ly))
        return fail(VTX_E_ARG, "box sides must be positive and finite");
    *out = nullptr;
    Staged S;
    int rc = validate_and_stage(he, n_he, n_vert, n_cell, S);
    if (rc) return rc;
    vtx_tissue t = new vtx_tissue_s();
    std::memset(&t->d, 0, sizeof t->d);
    std::memset(&t->w, 0, sizeof t->w);
    t->ep_buf = nullptr;
    t->hess = HessRows{};
    t->n_vert = n_vert;
    t->n_cell = n_cell;
    t->n_he = n_he;
    t->n_edge = (int64_t)S.edge_he.size();
    DevTissue &d = t->d;
    d.n_vert = (int32_t)n_vert;
    d.n_cell = (int32_t)n_cell;
    d.n_edge = (int32_t)t->n_edge;
    d.n_he = (int32_t)n_he;
    d.Lx = Lx;
    d.Ly = Ly;
    std::vector<int32_t> hev(he, he + 8 * n_he);
#define UP(dst, v)                       \
    if ((rc = upload(&dst, v))) {        \
        free_tissue(t);                  \
        return rc;                       \
    }
    UP(d.he, hev);
    UP(d.he_edge, S.he_edge);
    UP(d.edge_he, S.edge_he);
    UP(d.row_ptr, S.row_ptr);
    UP(d.row_cap, S.row_cap);
    {
        const std::vector<int32_t> pt{(int32_t)(n_he + kRowSlack * n_cell)};
        UP(d.pool_top, pt);
    }
    d.pool_start = (int32_t)(n_he + kRowSlack * n_cell);
    d.corner_cap = (int32_t)S.corner.size();
    UP(d.corner, S.corner);
    UP(d.corner_he, S.corner_he);
    UP(d.nsides, S.nsides);
    UP(d.cell_he, S.cell_he);
    UP(d.star, S.star);
    UP(d.star_he, S.star_he);
#undef UP
    int64_t t1cap = 1;
    while (t1cap < t->n_edge) t1cap <<= 1;
    t->t1_cap = t1cap;
    const int64_t nb = std::max<int64_t>(
        1024, (std::max(n_vert, std::max(n_cell, t->n_edge)) + kBlock - 1) / kBlock);
    Workspace &w = t->w;
    hipError_t e = hipSuccess;
    auto A = [&](void **p, size_t bytes) {
        if (e == hipSuccess) e = hipMalloc(p, std::max<size_t>(bytes, 16));
    };
    A(&w.xbuf, 16 * (size_t)n_vert);
    A((void **)&w.cap, 16 * (size_t)n_cell);
    A((void **)&w.cell_aux, 16 * (size_t)n_cell);
    A((void **)&w.partials, 16 * (size_t)nb);
    A((void **)&w.partials2, 16 * (size_t)nb);
    A((void **)&w.mpart, 16 * (size_t)nb);
    A((void **)&w.t1_list, 4 * (size_t)t1cap);
    A((void **)&w.ctl, 2 * sizeof(LoopCtl));
    A((void **)&w.cg, 6 * 16 * (size_t)n_vert);  // CG: 4 vectors, MINRES: 6
    A((void **)&w.scal, 16 * sizeof(double));
    A(&w.one, kOneBytes);
    A((void **)&w.step, sizeof(StepCtl));
    A((void **)&w.step_part,
      2 * 4 * sizeof(double) * (size_t)((4 * std::min(n_vert, kStepMaxVerts) + kBlock - 1) / kBlock));
    A((void **)&w.cg_state, 2 * sizeof(CgState));
    A((void **)&w.max_sides, sizeof(int32_t));
    A((void **)&t->ep_buf, 2 * 16 * (size_t)n_vert);
    const size_t n_tiles = (size_t)n_tiles_for(n_vert);
    A((void **)&t->tiles.cells, 4 * (size_t)kTileCap * n_tiles);
    A((void **)&t->tiles.info, 16 * n_tiles);
    A((void **)&t->tiles.halo, 4 * (size_t)kHaloCap * n_tiles);
    A((void **)&t->tiles.cstart, 2 * (size_t)kCstartPad * n_tiles);
    A((void **)&t->tiles.corners, 2 * (size_t)kCornerCap * n_tiles);
    A((void **)&t->tiles.fstar, 16 * (size_t)n_vert);
    A((void **)&t->tiles.fe, 8 * (size_t)n_vert);
    if (e == hipSuccess) e = hipHostMalloc((void **)&w.ctl_host, 2 * sizeof(LoopCtl), 0);
    if (e == hipSuccess) e = hipHostMalloc((void **)&w.step_host, sizeof(StepCtl), 0);
    if (e == hipSuccess) e = hipHostMalloc((void **)&w.cg_host, 2 * sizeof(CgState), 0);
    if (e == hipSuccess) e = hipStreamCreateWithFlags(&w.cap_stream, hipStreamNonBlocking);
    if (e == hipSuccess) {
        LoopCtl z{};
        w.ctl_host[0] = z;
        w.ctl_host[1] = z;
        e = hipMemcpy(w.ctl, w.ctl_host, 2 * sizeof(LoopCtl), hipMemcpyHostToDevice);
    }
    if (e == hipSuccess) {
        launch_tile_build(d, t->tiles, nullptr);
        e = hipGetLastError();
        if (e == hipSuccess) e = hipDeviceSynchronize();
    }
    if (e != hipSuccess) {
        free_tissue(t);
        return fail(VTX_E_HIP, "workspace allocation: %s", hipGetErrorString(e));
    }
    *out = t;
    return VTX_OK;
}

int vtx_tissue_destroy(vtx_tissue t) {
    if (!t) return fail(VTX_E_ARG, "null tissue");
    (void)hipDeviceSynchronize();
    free_tissue(t);
    return VTX_OK;
}

int vtx_tissue_sizes(vtx_tissue t, int64_t *n_vert, int64_t *n_cell, int64_t *n_edge,
                     int64_t *n_he) {
    if (!t) return fail(VTX_E_ARG, "null tissue");
    if (n_vert) *n_vert = t->n_vert;
    if (n_cell) *n_cell = t->n_cell;
    if (n_edge) *n_edge = t->n_edge;
    if (n_he) *n_he = t->n_he;
    return VTX_OK;
}

int vtx_tissue_tile_stats(vtx_tissue t, int64_t *stats) {
    if (!t || !stats) return fail(VTX_E_ARG, "null argument");
    const int64_t nt = n_tiles_for(t->n_vert);
    std::vector<int4> info((size_t)nt);
    HIPCHK(hipDeviceSynchronize());
    HIPCHK(hipMemcpy(info.data(), t->tiles.info, sizeof(int4) * (size_t)nt,
                     hipMemcpyDeviceToHost));
    for (int k = 0; k < 5; ++k) stats[k] = 0;
    stats[0] = nt;
    for (const int4 &i : info) {
        stats[1] += i.x;
        stats[2] += i.y;
        stats[3] += i.w;
        stats[4] += i.z;
    }
    return VTX_OK;
}

int vtx_tissue_get_topology(vtx_tissue t, int32_t *he_out) {
    if (!t || !he_out) return fail(VTX_E_ARG, "null argument");
    HIPCHK(hipDeviceSynchronize());
    HIPCHK(hipMemcpy(he_out, t->d.he, 8 * sizeof(int32_t) * t->n_he, hipMemcpyDeviceToHost));
    return VTX_OK;
}

int vtx_tissue_set_topology(vtx_tissue t, const int32_t *he) {
    if (!t || !he) return fail(VTX_E_ARG, "null argument");
    Staged S;
    int rc = validate_and_stage(he, t->n_he, t->n_vert, t->n_cell, S);
    if (rc) return rc;
    if ((int64_t)S.edge_he.size() != t->n_edge) return fail(VTX_E_TOPOLOGY, "edge count changed");
    HIPCHK(hipDeviceSynchronize());
    std::vector<int32_t> hev(he, he + 8 * t->n_he);
    DevTissue &d = t->d;
    if ((rc = upload_into(d.he, hev)) || (rc = upload_into(d.he_edge, S.he_edge)) ||
        (rc = upload_into(d.edge_he, S.edge_he)) || (rc = upload_into(d.row_ptr, S.row_ptr)) ||
        (rc = upload_into(d.row_cap, S.row_cap)) ||
        (rc = upload_into(d.pool_top, std::vector<int32_t>{d.pool_start})) ||
        (rc = upload_into(d.corner, S.corner)) || (rc = upload_into(d.corner_he, S.corner_he)) ||
        (rc = upload_into(d.nsides, S.nsides)) || (rc = upload_into(d.cell_he, S.cell_he)) ||
        (rc = upload_into(d.star, S.star)) || (rc = upload_into(d.star_he, S.star_he)))
        return rc;
    // synchronous like the uploads: the tables are complete on return, for
    // callers on any stream
    if ((rc = vtx::tissue_topology_changed(t, nullptr))) return rc;
    HIPCHK(hipDeviceSynchronize());
    return VTX_OK;
}

int vtx_energy_forces(vtx_tissue t, int32_t mode, const void *X, const vtx_params *p,
                      double *E_dev, void *F, double *maxf_dev, void *stream) {
    if (!t || !X || !p || !mode_ok(mode)) return fail(VTX_E_ARG, "bad argument");
    launch_eval_fused(t->d, t->w, t->tiles, mode, X, raw(p), E_dev, F, maxf_dev,
                      (hipStream_t)stream);
    return check_launch("vtx_energy_forces");
}

}  // extern "C"

namespace {
// Device address of `scratch` on the current device, looked up once per
// device (with that device current) and kept; NULL on failure.
unsigned char *noalloc_scratch(int *err) {
    static std::mutex mu;
    static unsigned char *addr[64] = {nullptr};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess || dev < 0 || dev >= 64) {
        *err = fail(VTX_E_HIP, "hipGetDevice: %s", hipGetErrorString(e));
        return nullptr;
    }
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[dev]) {
        void *ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr) {
            *err = fail(VTX_E_HIP, "hipGetSymbolAddress(scratch): %s", hipGetErrorString(e));
            return nullptr;
        }
        addr[dev] = (unsigned char *)ptr;
    }
    return addr[dev];
}
}  // namespace

extern "C" {

int vtx_energy_forces_noalloc(vtx_tissue t, int32_t mode, const void *X, const vtx_params *p,
                              double *E_dev, void *F, double *maxf_dev, void *stream) {
    if (!t || !X || !p || !mode_ok(mode)) return fail(VTX_E_ARG, "bad argument");
    if (t->n_vert > kNoAllocVerts)
        return fail(VTX_E_CAPACITY,
                    "vtx_energy_forces_noalloc: %lld vertices exceed its fixed scratch (at most "
                    "%lld vertices)",
                    (long long)t->n_vert, (long long)kNoAllocVerts);
    int rc = VTX_OK;
    unsigned char *base = noalloc_scratch(&rc);
    if (!base) return rc;
    hipStream_t s = (hipStream_t)stream;
    Workspace w{};
    w.mpart = (double *)base;
    w.ctl = (LoopCtl *)(base + kNoAllocCtlOffset);
    hipLaunchKernelGGL(k_clear_ctl, dim3(1), dim3(64), 0, s, w.ctl);
    launch_eval_fused(t->d, w, t->tiles, mode, X, raw(p), E_dev, F, maxf_dev, s);
    return check_launch("vtx_energy_forces_noalloc");
}

int vtx_cell_coeffs(vtx_tissue t, int32_t mode, const void *X, const vtx_params *p,
                    void *coeffs, void *stream) {
    if (!t || !X || !p || !coeffs || !mode_ok(mode)) return fail(VTX_E_ARG, "bad argument");
    launch_cell_pass(t->d, t->w, mode, X, raw(p), coeffs, (hipStream_t)stream);
    return check_launch("vtx_cell_coeffs");
}

int vtx_vertex_forces(vtx_tissue t, int32_t mode, const void *X, const vtx_params *p,
                      const void *coeffs, void *F, double *maxf_dev, void *stream) {
    if (!t || !X || !p || !coeffs || !mode_ok(mode)) return fail(VTX_E_ARG, "bad argument");
    launch_vertex_pass(t->d, t->w, mode, X, raw(p), coeffs, F, maxf_dev, (hipStream_t)stream);
    return check_launch("vtx_vertex_forces");
}

int vtx_cell_geometry(vtx_tissue t, int32_t mode, const void *X, double *A_dev, double *P_dev,
                      void *stream) {
    if (!t || !X || !mode_ok(mode)) return fail(VTX_E_ARG, "bad argument");
    launch_cell_exact(t->d, mode, X, A_dev, P_dev, (hipStream_t)stream);
    return check_launch("vtx_cell_geometry");
}

int vtx_edge_lengths(vtx_tissue t, int32_t mode, const void *X, double *len_dev, void *stream) {
    if (!t || !X || !len_dev || !mode_ok(mode)) return fail(VTX_E_ARG, "bad argument");
    launch_edge_len(t->d, mode, X, len_dev, (hipStream_t)stream);
    return check_launch("vtx_edge_lengths");
}

int vtx_relax(vtx_tissue t, int32_t mode, void *X, const vtx_params *p, const vtx_relax_opts *o,
              vtx_relax_result *res, void *stream) {
    if (!t || !X || !p || !o || !mode_ok(mode)) return fail(VTX_E_ARG, "bad argument");
    return relax_impl(t, mode, X, p, o, res, (hipStream_t)stream);
}

int vtx_t1(vtx_tissue t, int32_t mode, void *X, const vtx_params *p, double l_min, double l_new,
           int64_t *n_swap, int64_t *n_stretch, void *stream) {
    if (!t || !X || !p || !mode_ok(mode)) return fail(VTX_E_ARG, "bad argument");
    if (!(l_min > 0) || !(l_new > 0)) return fail(VTX_E_ARG, "l_min and l_new must be > 0");
    hipStream_t s = (hipStream_t)stream;
    LoopCtl z{};
    int rc = reset_ctl(t, 1, z, s);
    if (rc) return rc;
    launch_t1(t->d, t->w, mode, X, raw(p), l_min, l_new, s);
    if ((rc = check_launch("vtx_t1"))) return rc;
    if ((rc = read_ctl(t, 1, s))) return rc;
    const LoopCtl h = t->w.ctl_host[1];
    if ((h.n_t1 > 0 || h.t1_overflow) && (rc = vtx::tissue_topology_changed(t, s))) return rc;
    if (n_swap) *n_swap = h.n_t1;
    if (n_stretch) *n_stretch = h.n_stretch;
    LoopCtl z2{};  // the evaluation control block must never stay `done`
    if ((rc = reset_ctl(t, 1, z2, s))) return rc;
    if (h.t1_overflow) return fail(VTX_E_CAPACITY, "T1 pass overflow (%d)", h.t1_overflow);
    return VTX_OK;
}

int vtx_hvp(vtx_tissue t, int32_t mode, const void *X, const vtx_params *p, const double *v,
            double *Hv, void *stream) {
    if (!t || !X || !p || !v || !Hv || !mode_ok(mode)) return fail(VTX_E_ARG, "bad argument");
    hipStream_t s = (hipStream_t)stream;
    launch_cell_coeffs(t->d, t->w, mode, X, raw(p), s);
    launch_hvp(t->d, t->w, mode, X, raw(p), v, Hv, nullptr, nullptr, s);
    return check_launch("vtx_hvp");
}

int vtx_v2v(vtx_tissue t, int32_t mode, const void *X, const void *X_target, double *C_dev,
            double *grad, void *stream) {
    if (!t || !X || !X_target || !mode_ok(mode)) return fail(VTX_E_ARG, "bad argument");
    launch_v2v(t->d, t->w, mode, X, X_target, C_dev, grad, (hipStream_t)stream);
    return check_launch("vtx_v2v");
}

// Memory for rows of `width` slots per lane: kept for later solves, grown when
// a larger cell appears.  False, with none held, where the device has no room.
static bool hess_reserve(vtx_tissue t, int width) {
    HessRows &H = t->hess;
    if (width <= H.width) return true;
    void *old[] = {H.col, H.top, H.bottom, H.halo, H.n_halo};
    H = HessRows{};
    for (void *q : old)
        if (q) (void)hipFree(q);
    hess_plan(t->n_vert, H);
    width = std::max(width, 6);  // six: cells of up to eight sides
    const size_t n = 4 * (size_t)width * (size_t)H.verts * (size_t)H.blocks;
    hipError_t e = hipMalloc((void **)&H.col, 4 * n);
    if (e == hipSuccess) e = hipMalloc((void **)&H.top, 16 * n);
    if (e == hipSuccess) e = hipMalloc((void **)&H.bottom, 16 * n);
    if (e == hipSuccess) e = hipMalloc((void **)&H.halo, 4 * (size_t)kCgHalo * (size_t)H.blocks);
    if (e == hipSuccess) e = hipMalloc((void **)&H.n_halo, 4 * (size_t)H.blocks);
    if (e == hipSuccess) {
        H.width = width;
        return true;
    }
    (void)hipGetLastError();  // not an error of the call, which takes the other loop
    for (void *q : {(void *)H.col, (void *)H.top, (void *)H.bottom, (void *)H.halo,
                    (void *)H.n_halo})
        if (q) (void)hipFree(q);
    H = HessRows{};
    return false;
}

// CG by one launch per iteration (k_cg_step) on the rows of the Hessian,
// FP64; the solution is left in w.cg, not yet projected.  *taken is false, and
// nothing done, where the rows would be too wide or have no room.
static int cg_steps(vtx_tissue t, const void *X, const vtx_params *p, const double *b, double tol,
                    int64_t max_iter, hipStream_t s, vtx_grad_result *r, bool *taken) {
    *taken = false;
    CgState &h = t->w.cg_host[0];
    launch_max_sides(t->d, t->w, s);
    int rc;
    if ((rc = check_launch("largest cell"))) return rc;
    h = CgState{};
    HIPCHK(hipMemcpyAsync(t->w.cg_state, &h, sizeof h, hipMemcpyHostToDevice, s));
    int32_t sides = 0;
    HIPCHK(hipMemcpyAsync(&sides, t->w.max_sides, sizeof sides, hipMemcpyDeviceToHost, s));
    HIPCHK(hipStreamSynchronize(s));
    const int width = sides - 2;
    if (width * t->n_vert > kCgStepMaxSlots || !hess_reserve(t, width)) return VTX_OK;
    *taken = true;
    const HessRows &H = t->hess;
    HessRows use = H;
    use.width = width;  // slots in use now
    launch_hess_rows(t->d, t->w, use, X, raw(p), s);
    launch_cg_step_init(t->w, (int)t->n_vert, b, s);
    if ((rc = check_launch("Hessian rows"))) return rc;
    rc = run_loop(
        t, kCgChunk, max_iter + 2, s,
        [&](int k, hipStream_t cs) { launch_cg_step(t->d, t->w, use, tol, max_iter, k, cs); },
        [&]() { return hipMemcpyAsync(&h, t->w.cg_state, sizeof h, hipMemcpyDeviceToHost, s); },
        [&]() { return h.done != 0; }, []() { return (int64_t)kCgChunk; });
    if (rc) return rc;
    r->cg_iters = h.it;
    r->cg_rel_res = h.rel_res;
    r->status = h.status;
    return VTX_OK;
}

// Solves H x = P b at X (H restricted to the zero-mean subspace) by CG or
// MINRES on the device, x left projected in the first workspace vector, then
// contracts it with the mixed derivatives of theta into g unless g is NULL.
static int solve_hessian(vtx_tissue t, int mode, const void *X, const vtx_params *p,
                         const double *b, bool minres, double tol, int64_t max_iter, int theta,
                         double *g, hipStream_t s, vtx_grad_result *r) {
    const int nv = (int)t->n_vert;
    // an FP64 tissue that fits one workgroup's LDS is solved there (against
    // the one-launch step: 1.0 and 3.1 ms at 200 cells, 4.6 and 4.9-5.3 at 1000)
    const vtx_grad_result *one = nullptr;
    int rc = solve_one(t->d, t->w, mode, X, raw(p), b, minres, tol, max_iter, theta, g, s, &one);
    if (rc) return rc;
    if (one) {
        HIPCHK(hipMemcpyAsync(r, one, sizeof *r, hipMemcpyDeviceToHost, s));
        HIPCHK(hipStreamSynchronize(s));
        return VTX_OK;
    }
    launch_cell_coeffs(t->d, t->w, mode, X, raw(p), s);
    bool taken = false;
    if (mode == VTX_F64 && !minres && t->n_vert <= kCgStepMaxVerts &&
        (rc = cg_steps(t, X, p, b, tol, max_iter, s, r, &taken)))
        return rc;
    if (taken) {
        launch_project(t->w, nv, t->w.cg, s);
        if (g) launch_contract(t->d, mode, X, raw(p), theta, t->w.cg, g, s);
        return check_launch("CG solve");
    }
    LoopCtl c{};
    c.status = VTX_CG_MAXITER;
    c.tol = tol;
    c.max_iter = max_iter;
    c.solver = minres ? 1 : 0;
    if ((rc = reset_ctl(t, 0, c, s))) return rc;
    if (minres) launch_minres_init(t->w, nv, b, s);
    else launch_cg_init(t->w, nv, b, s);
    if ((rc = check_launch("Krylov init"))) return rc;
    if ((rc = read_ctl(t, 0, s))) return rc;
    if (!t->w.ctl_host[0].done) {
        rc = run_loop(t, 32, max_iter, s, [&](int, hipStream_t cs) {
            if (minres) launch_minres_iter(t->d, t->w, mode, X, raw(p), cs);
            else launch_cg_iter(t->d, t->w, mode, X, raw(p), cs);
        }, [&]() { return fetch_ctl(t, s); }, [&]() { return t->w.ctl_host[0].done != 0; },
           []() { return (int64_t)32; });
        if (rc) return rc;
    }
    const LoopCtl &h = t->w.ctl_host[0];
    launch_project(t->w, nv, t->w.cg, s);
    if (g) launch_contract(t->d, mode, X, raw(p), theta, t->w.cg, g, s);
    r->cg_iters = h.cg_iter;
    r->cg_rel_res = h.rel_res;
    r->status = h.status;
    return check_launch("Krylov solve");
}

int vtx_param_grad(vtx_tissue t, int32_t mode, const void *X_star, const vtx_params *p,
                   const double *dC_dX, const void *X_target, const vtx_grad_opts *o,
                   double *dC_dtheta, vtx_grad_result *res, void *stream) {
    if (!t || !X_star || !p || !o || !dC_dtheta || !mode_ok(mode))
        return fail(VTX_E_ARG, "bad argument");
    if (o->theta != VTX_THETA_LAMBDA && o->theta != VTX_THETA_P0)
        return fail(VTX_E_ARG, "unknown theta selector");
    hipStream_t s = (hipStream_t)stream;
    vtx_grad_result r{};
    int rc;
    if (o->method == VTX_GRAD_ADJOINT || o->method == VTX_GRAD_ADJOINT_MINRES) {
        if (!dC_dX) return fail(VTX_E_ARG, "the adjoint needs dC_dX");
        if (!(o->cg_tol > 0) || o->cg_max_iter < 1) return fail(VTX_E_ARG, "bad Krylov options");
        if ((rc = solve_hessian(t, mode, X_star, p, dC_dX, o->method == VTX_GRAD_ADJOINT_MINRES,
                                o->cg_tol, o->cg_max_iter, o->theta, dC_dtheta, s, &r)))
            return rc;
        HIPCHK(hipStreamSynchronize(s));
    } else if (o->method == VTX_GRAD_EP_CENTRED || o->method == VTX_GRAD_EP_FORWARD) {
        const bool centred = o->method == VTX_GRAD_EP_CENTRED;
        if (!(o->beta != 0.0)) return fail(VTX_E_ARG, "EP needs beta != 0");
        if (o->ep_relax.t1_enable) return fail(VTX_E_ARG, "EP relaxations cannot use T1");
        if (!X_target && !dC_dX) return fail(VTX_E_ARG, "EP needs X_target or dC_dX");
        const size_t pb = pos_bytes(t, mode);
        char *Xp = (char *)t->ep_buf, *Xm = Xp + 16 * (size_t)t->n_vert;
        HIPCHK(hipMemcpyAsync(Xp, X_star, pb, hipMemcpyDeviceToDevice, s));
        HIPCHK(hipMemcpyAsync(Xm, X_star, pb, hipMemcpyDeviceToDevice, s));
        vtx_relax_opts ro = o->ep_relax;
        ro.X_target = X_target;
        ro.g_lin = X_target ? nullptr : dC_dX;
        ro.beta = centred ? 0.5 * o->beta : o->beta;
        if ((rc = relax_impl(t, mode, Xp, p, &ro, &r.ep_plus, s))) return rc;
        if (centred) {
            ro.beta = -0.5 * o->beta;
            if ((rc = relax_impl(t, mode, Xm, p, &ro, &r.ep_minus, s))) return rc;
        }
        launch_ep(t->d, mode, Xp, Xm, raw(p), o->theta, o->beta, dC_dtheta, s);
        if ((rc = check_launch("EP estimate"))) return rc;
        HIPCHK(hipStreamSynchronize(s));
        r.status = combine_status(r.ep_plus.status, r.ep_minus.status);
    } else {
        return fail(VTX_E_ARG, "unknown hypergradient method");
    }
    if (res) *res = r;
    return VTX_OK;
}

int vtx_param_sens(vtx_tissue t, int32_t mode, const void *X_star, const vtx_params *p,
                   const double *d, const double *dC_dX, const vtx_grad_opts *o, double *dC_dd,
                   double *dX_dd, vtx_grad_result *res, void *stream) {
    if (!t || !X_star || !p || !d || !dC_dX || !o || !dC_dd || !mode_ok(mode))
        return fail(VTX_E_ARG, "bad argument");
    if (mode == VTX_F32) return fail(VTX_E_ARG, "sensitivities need double positions");
    if (o->theta != VTX_THETA_LAMBDA && o->theta != VTX_THETA_P0)
        return fail(VTX_E_ARG, "unknown theta selector");
    if (!(o->cg_tol > 0) || o->cg_max_iter < 1) return fail(VTX_E_ARG, "bad CG options");
    hipStream_t s = (hipStream_t)stream;
    const int nv = (int)t->n_vert;
    double *rhs = t->ep_buf;  // [n_vert][2]
    launch_sens_rhs(t->d, t->w, X_star, raw(p), o->theta, d, rhs, s);
    vtx_grad_result r{};
    int rc = solve_hessian(t, mode, X_star, p, rhs, o->method == VTX_GRAD_ADJOINT_MINRES,
                           o->cg_tol, o->cg_max_iter, o->theta, nullptr, s, &r);
    if (rc) return rc;
    launch_dot_pos(t->w, VTX_F64, nv, dC_dX, t->w.cg, dC_dd, s);
    if (dX_dd)
        HIPCHK(hipMemcpyAsync(dX_dd, t->w.cg, 16 * (size_t)nv, hipMemcpyDeviceToDevice, s));
    if ((rc = check_launch("sensitivity"))) return rc;
    HIPCHK(hipStreamSynchronize(s));
    if (res) *res = r;
    return VTX_OK;
}

}  // extern "C"
