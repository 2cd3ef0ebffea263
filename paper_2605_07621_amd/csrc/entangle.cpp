// Entanglement spectrum of a state in the bipartite layout: the spectrum
// xi_{q,i} = -log lambda_{q,i} of the entanglement Hamiltonian
// H_E = -log rho_L, rho_L = Tr_R |psi><psi| (the paper's figure on the
// distributed entanglement spectrum).  rho_L is block diagonal over the
// sectors of the cut, rho_L^q = Psi_q Psi_q^T, and its nonzero eigenvalues
// are those of the smaller Gram matrix of the block, Psi_q Psi_q^T or
// Psi_q^T Psi_q.  Per block: the Gram matrix with rocBLAS syrk (a plain
// dense contraction), its eigenvalues with rocSOLVER syevd, both on the
// device; the sector weights W_q, their participation numbers and the
// process-resolved sums W_P on the host.
#include <hip/hip_runtime.h>
#include <rocblas/rocblas.h>
#include <rocsolver/rocsolver.h>

#include <algorithm>
#include <cmath>
#include <exception>
#include <map>
#include <mutex>
#include <numeric>
#include <string>
#include <thread>
#include <vector>

#include "ecut_internal.h"
#include "runtime.h"

using namespace ecut;

namespace {

// A rocBLAS handle with a stream of its own.  The eigensolver is a chain of
// thousands of small launches per matrix size, so the sizes run side by side,
// each chain on a lane: the lanes of a call are taken from a process-wide pool
// and go back to it; the pool keeps at most LANES_KEPT idle ones per device.
constexpr int LANES = 4;          // per call: the hardware queues of a process
constexpr size_t LANES_KEPT = 8;

struct Lane {
    rocblas_handle h = nullptr;
    hipStream_t st = nullptr;
    hipEvent_t ev = nullptr;
};

std::mutex g_lane_mu;
std::map<int, std::vector<Lane>> g_lanes;   // idle lanes by device

void drop_lane(Lane &l) {
    if (l.h) (void)rocblas_destroy_handle(l.h);
    if (l.ev) (void)hipEventDestroy(l.ev);
    if (l.st) (void)hipStreamDestroy(l.st);
    l = Lane{};
}

// The lanes of one call on the current device.  The destructor waits for their
// work (it reads and writes the caller's memory) before it hands them back.
struct LaneSet {
    int dev = -1;
    std::vector<Lane> lanes;
    bool direct = false;        // the one lane's handle is on the caller's stream
    hipStream_t caller = nullptr;

    ecut_status take(int n) {
        if (hipGetDevice(&dev) != hipSuccess) return fail(ECUT_EDEVICE, "hipGetDevice");
        {
            std::lock_guard<std::mutex> g(g_lane_mu);
            auto &idle = g_lanes[dev];
            while ((int)lanes.size() < n && !idle.empty()) {
                lanes.push_back(idle.back());
                idle.pop_back();
            }
        }
        while ((int)lanes.size() < n) {
            Lane l;
            const bool ok = hipStreamCreateWithFlags(&l.st, hipStreamNonBlocking) == hipSuccess &&
                            hipEventCreateWithFlags(&l.ev, hipEventDisableTiming) == hipSuccess &&
                            rocblas_create_handle(&l.h) == rocblas_status_success &&
                            rocblas_set_stream(l.h, l.st) == rocblas_status_success;
            if (!ok) {
                drop_lane(l);
                return fail(ECUT_EDEVICE, "rocblas_create_handle");
            }
            lanes.push_back(l);
        }
        return ECUT_OK;
    }

    // one lane: its chain runs on the caller's stream itself
    ecut_status on_stream(hipStream_t st) {
        if (rocblas_set_stream(lanes[0].h, st) != rocblas_status_success) return fail(ECUT_EDEVICE, "rocblas_set_stream");
        direct = true;
        caller = st;
        return ECUT_OK;
    }

    ~LaneSet() {
        if (direct) {
            (void)hipStreamSynchronize(caller);
            if (rocblas_set_stream(lanes[0].h, lanes[0].st) != rocblas_status_success) {
                drop_lane(lanes[0]);
                lanes.clear();
            }
        }
        for (Lane &l : lanes) (void)hipStreamSynchronize(l.st);
        std::lock_guard<std::mutex> g(g_lane_mu);
        auto &idle = g_lanes[dev];
        for (Lane &l : lanes) {
            if (idle.size() < LANES_KEPT) idle.push_back(l);
            else drop_lane(l);
        }
    }
};

int64_t schmidt_count(const ecut_sectors *s) {
    int64_t n = 0;
    for (const BlockDev &B : s->blocks) n += std::min(B.d_l, B.d_r);
    return n;
}

// parts of a largest-first bin packing of the blocks by dimension
std::vector<int32_t> pack_blocks(const ecut_sectors *s, int32_t n_parts) {
    std::vector<int32_t> order(s->blocks.size()), part(s->blocks.size(), 0);
    std::iota(order.begin(), order.end(), 0);
    auto dimq = [&](int32_t q) { return (int64_t)s->blocks[q].d_l * s->blocks[q].d_r; };
    std::stable_sort(order.begin(), order.end(), [&](int32_t a, int32_t b) { return dimq(a) > dimq(b); });
    std::vector<int64_t> load(n_parts, 0);
    for (int32_t q : order) {
        const int32_t p = (int32_t)(std::min_element(load.begin(), load.end()) - load.begin());
        part[q] = p;
        load[p] += dimq(q);
    }
    return part;
}

// the blocks by the size of their Gram matrix (m = min(d_L, d_R) > 0), in
// block order inside each size
std::map<int, std::vector<int32_t>> gram_groups(const ecut_sectors *s) {
    std::map<int, std::vector<int32_t>> g;
    for (int32_t q = 0; q < (int32_t)s->blocks.size(); ++q) {
        const int m = std::min(s->blocks[q].d_l, s->blocks[q].d_r);
        if (m > 0) g[m].push_back(q);
    }
    return g;
}

// The groups of equal sizes dealt to lanes: the longest chain first, each to
// the lane with the least work so far (the solver's launches grow with the size,
// not with the number of blocks).  A lane's groups run one after the other in
// one Gram buffer and one off-diagonal buffer, as large as its largest group
// needs.  Side by side the lanes need more than one chain does; where that is
// past LANES_EXTRA, fewer lanes run, down to one, so that a large spectrum fits
// where the largest group and its eigenvalues fit (32 sites in halves: 2.1 GB
// instead of 4.8 for every block at once).  A short spectrum is one chain on the
// caller's stream: a lane costs threads, events and slower launches (sizes 1, 6,
// 15 and 20, 12-site spin chain: 834 us in one chain, 908 on four lanes; 1, 4 and
// 6: 247 against 343; one size of 252: 5.8 against 6.3 ms on a lane's own stream;
// the sizes of an 8-site spatial Hubbard cut, 87 rows: 1.60 against 1.25 ms).
constexpr int LANES_MIN_ROWS = 64;   // sum of the sizes from which lanes run
constexpr size_t LANES_EXTRA = (size_t)1 << 27;   // doubles, 1 GiB

struct Group {
    int m;
    std::vector<int32_t> q;
    int64_t off;     // its eigenvalues in the list of all
    int32_t info;    // its first status word
};

struct Schedule {
    std::vector<Group> groups;                 // by size, ascending
    std::vector<std::vector<int>> todo;        // per lane: groups, largest first
    std::vector<size_t> gram, diag;            // per lane: doubles of its buffers
    size_t doubles = 0;                        // of all lanes' buffers
};

Schedule lane_schedule(const ecut_sectors *s) {
    Schedule S;
    int64_t off = 0;
    int32_t info = 0;
    size_t largest = 0;
    for (const auto &kv : gram_groups(s)) {
        const size_t m = (size_t)kv.first, c = kv.second.size();
        S.groups.push_back(Group{kv.first, kv.second, off, info});
        off += (int64_t)(c * m);
        info += (int32_t)c;
        largest = std::max(largest, c * m * m);
    }
    int64_t rows = 0;
    for (const Group &W : S.groups) rows += W.m;
    const int most = rows < LANES_MIN_ROWS ? 1 : std::max(1, std::min<int>(LANES, (int)S.groups.size()));
    for (int n = most; n >= 1; --n) {
        std::vector<int64_t> load(n, 0);
        S.todo.assign(n, {});
        S.gram.assign(n, 0);
        S.diag.assign(n, 0);
        for (int g = (int)S.groups.size() - 1; g >= 0; --g) {
            const size_t lane = std::min_element(load.begin(), load.end()) - load.begin();
            const size_t m = (size_t)S.groups[g].m, c = S.groups[g].q.size();
            load[lane] += (int64_t)m;
            S.todo[lane].push_back(g);
            S.gram[lane] = std::max(S.gram[lane], c * m * m);
            S.diag[lane] = std::max(S.diag[lane], c * m);
        }
        const size_t grams = std::accumulate(S.gram.begin(), S.gram.end(), (size_t)0);
        S.doubles = grams + std::accumulate(S.diag.begin(), S.diag.end(), (size_t)0);
        if (grams - largest <= LANES_EXTRA) break;
    }
    return S;
}

}  // namespace

extern "C" {

// Workspace: every lane's Gram matrices and the eigensolver's off-diagonals, the
// eigenvalues and one status word of every block.
size_t ecut_entanglement_sizes(const ecut_sectors *s, size_t *n_lambda) {
    if (!s) return 0;
    const size_t nl = (size_t)schmidt_count(s);
    if (n_lambda) *n_lambda = nl;
    return lane_schedule(s).doubles + nl + (s->blocks.size() + 1) / 2 + 1;
}

ecut_status ecut_entanglement_spectrum(const ecut_sectors *s, const double *psi_d, double cutoff, int32_t n_parts,
                                       const int32_t *part_of_block, double *lambda, double *xi, double *w_q,
                                       int32_t *chi_q, double *w_p, ecut_entanglement *summary, double *workspace_d,
                                       void *stream) {
    if (!s || !psi_d || !workspace_d || !lambda || !w_q || !chi_q || !summary)
        return fail(ECUT_EINVAL, "null argument");
    if (!s->on_device) return fail(ECUT_EINVAL, "handle was built with ECUT_BUILD_HOST_ONLY");
    if (n_parts < 1 || (n_parts > 1 && !w_p)) return fail(ECUT_EINVAL, "n_parts must be >= 1 (and w_p set)");
    if (!(cutoff >= 0.0)) return fail(ECUT_EINVAL, "cutoff must be >= 0");
    const int32_t nb = (int32_t)s->blocks.size();
    if (part_of_block)
        for (int32_t q = 0; q < nb; ++q)
            if (part_of_block[q] < 0 || part_of_block[q] >= n_parts) return fail(ECUT_EINVAL, "part_of_block out of range");
    for (const BlockDev &B : s->blocks)
        if (std::min(B.d_l, B.d_r) > (1 << 24)) return fail(ECUT_EUNSUPPORTED, "block too large for the Gram matrix");
    const hipStream_t hs = (hipStream_t)stream;
    // refused before the lanes join the caller's capture: they go back to the
    // pool for other threads' calls
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(hs, &cap) == hipSuccess && cap != hipStreamCaptureStatusNone)
        return fail(ECUT_EDEVICE, "the spectrum synchronises its stream and cannot be captured");
    const Schedule S = lane_schedule(s);
    const int64_t n_lam = schmidt_count(s);
    LaneSet set;
    ecut_status st = set.take((int)S.todo.size());
    if (st != ECUT_OK) return st;
    hipError_t le = hipSuccess;
    if (set.lanes.size() == 1) {
        st = set.on_stream(hs);
        if (st != ECUT_OK) return st;
    } else {   // the lanes start after the caller's work on its stream
        le = hipEventRecord(set.lanes[0].ev, hs);
        for (Lane &l : set.lanes)
            if (le == hipSuccess) le = hipStreamWaitEvent(l.st, set.lanes[0].ev, 0);
        if (le != hipSuccess) return hip_fail(le, "entanglement lanes");
    }
    // per group of equal-size blocks: their Gram matrices side by side
    // (rocBLAS syrk each), one batched eigensolve; the eigenvalues of every
    // group side by side, one copy to the host at the end
    double *Dg = workspace_d + S.doubles;
    rocblas_int *info = (rocblas_int *)(Dg + n_lam);
    const double one = 1.0, zero = 0.0;
    std::vector<double *> Gm, Ed;   // the lanes' buffers
    double *p = workspace_d;
    for (size_t lane = 0; lane < S.todo.size(); ++lane) {
        Gm.push_back(p);
        Ed.push_back(p + S.gram[lane]);
        p += S.gram[lane] + S.diag[lane];
    }
    // one thread per lane: the chains are so many launches that one thread's
    // launch rate would bound them (14-site spatial Hubbard cut, 64 blocks of
    // up to 1,225 x 1,225: one chain 82 ms, four lanes from one thread 62, from
    // four 55; 12 sites 26 -> 14.5 ms)
    struct Err {
        const char *what;
        int status;
    };
    std::vector<Err> err(set.lanes.size(), Err{nullptr, 0});
    auto enqueue = [&](size_t lane) {   // on a thread of its own: reports by err only
        if (hipSetDevice(set.dev) != hipSuccess) {
            err[lane] = Err{"hipSetDevice", 0};
            return;
        }
        const rocblas_handle h = set.lanes[lane].h;
        double *G = Gm[lane], *E = Ed[lane];
        for (const int g : S.todo[lane]) {
            const Group &W = S.groups[g];
            const int m = W.m, c = (int)W.q.size();
            for (int i = 0; i < c; ++i) {
                const BlockDev &B = s->blocks[W.q[i]];
                // Psi_q is row-major d_L x d_R: column-major it is A (d_R x d_L, lda = d_R)
                const double *A = psi_d + B.offset;
                const bool left = B.d_l <= B.d_r;   // Psi Psi^T = A^T A (d_L x d_L), else Psi^T Psi = A A^T
                const rocblas_status rs =
                    rocblas_dsyrk(h, rocblas_fill_upper, left ? rocblas_operation_transpose : rocblas_operation_none, m,
                                  left ? B.d_r : B.d_l, &one, A, B.d_r, &zero, G + (size_t)i * m * m, m);
                if (rs != rocblas_status_success) {
                    err[lane] = Err{"rocblas_dsyrk", (int)rs};
                    return;
                }
            }
            const rocblas_status rs = rocsolver_dsyevd_strided_batched(
                h, rocblas_evect_none, rocblas_fill_upper, m, G, m, (rocblas_stride)m * m, Dg + W.off, m, E, m,
                info + W.info, c);
            if (rs != rocblas_status_success) {
                err[lane] = Err{"rocsolver_dsyevd_strided_batched", (int)rs};
                return;
            }
        }
    };
    std::vector<std::thread> threads(set.lanes.size());
    for (size_t lane = 1; lane < set.lanes.size(); ++lane) {
        try {
            threads[lane] = std::thread(enqueue, lane);
        } catch (const std::exception &) {   // no thread to be had: this one does its work
            enqueue(lane);
        }
    }
    enqueue(0);
    for (std::thread &t : threads)
        if (t.joinable()) t.join();
    for (const Err &e : err)
        if (e.what) return fail(ECUT_EDEVICE, std::string(e.what) + ": status " + std::to_string(e.status));
    for (Lane &l : set.lanes) {   // the copies below follow every lane
        if (set.direct) break;
        if (le == hipSuccess) le = hipEventRecord(l.ev, l.st);
        if (le == hipSuccess) le = hipStreamWaitEvent(hs, l.ev, 0);
    }
    if (le != hipSuccess) return hip_fail(le, "entanglement lanes");
    std::vector<double> ev((size_t)n_lam);
    const int32_t n_info = S.groups.empty() ? 0 : S.groups.back().info + (int32_t)S.groups.back().q.size();
    std::vector<rocblas_int> inf((size_t)std::max(n_info, 1), 0);
    hipError_t e = n_lam ? hipMemcpyAsync(ev.data(), Dg, sizeof(double) * n_lam, hipMemcpyDeviceToHost, hs) : hipSuccess;
    if (e == hipSuccess && n_info)
        e = hipMemcpyAsync(inf.data(), info, sizeof(rocblas_int) * n_info, hipMemcpyDeviceToHost, hs);
    if (e == hipSuccess) e = hipStreamSynchronize(hs);
    if (e != hipSuccess) return fail(ECUT_EDEVICE, std::string("entanglement spectrum: ") + hipGetErrorString(e));
    // each block's eigenvalues, descending, at its place in block order
    std::vector<int64_t> lam_off((size_t)nb + 1, 0);
    for (int32_t q = 0; q < nb; ++q)
        lam_off[q + 1] = lam_off[q] + std::min(s->blocks[q].d_l, s->blocks[q].d_r);
    for (const Group &W : S.groups) {
        const int m = W.m;
        for (size_t i = 0; i < W.q.size(); ++i) {
            const int32_t q = W.q[i];
            if (inf[W.info + i] != 0) return fail(ECUT_ENOTCONV, "rocsolver_dsyevd did not converge on block " + std::to_string(q));
            for (int k = 0; k < m; ++k) lambda[lam_off[q] + k] = ev[(size_t)(W.off + (int64_t)i * m + m - 1 - k)];
        }
    }
    int64_t off_l = n_lam;
    // normalise to the state's norm: the eigenvalues of rho_L of psi / |psi|
    const double norm2 = std::accumulate(lambda, lambda + off_l, 0.0);
    if (!(norm2 > 0.0)) return fail(ECUT_EINVAL, "the state is zero");
    off_l = 0;
    int64_t chi_sum = 0;
    double w2 = 0.0;
    for (int32_t q = 0; q < nb; ++q) {
        const BlockDev &B = s->blocks[q];
        const int m = std::min(B.d_l, B.d_r);
        double wq = 0.0;
        int32_t chi = 0;
        for (int i = 0; i < m; ++i) {
            double &l = lambda[off_l + i];
            l /= norm2;
            wq += l;
            if (l > cutoff) ++chi;
            if (xi) xi[off_l + i] = l > 0.0 ? -std::log(l) : INFINITY;
        }
        w_q[q] = wq;
        chi_q[q] = chi;
        chi_sum += chi;
        w2 += wq * wq;
        off_l += m;
    }
    double c2 = 0.0;
    for (int32_t q = 0; q < nb; ++q) {
        const double c = chi_sum > 0 ? (double)chi_q[q] / (double)chi_sum : 0.0;
        c2 += c * c;
    }
    std::vector<int32_t> part = part_of_block ? std::vector<int32_t>(part_of_block, part_of_block + nb)
                                              : pack_blocks(s, n_parts);
    if (w_p) {
        std::fill(w_p, w_p + n_parts, 0.0);
        for (int32_t q = 0; q < nb; ++q) w_p[part[q]] += w_q[q] * w_q[q];
    }
    ecut_entanglement R{};
    R.n_blocks = nb;
    R.n_parts = n_parts;
    R.n_lambda = off_l;
    R.norm2 = norm2;
    R.weight_ipr = w2 > 0.0 ? 1.0 / w2 : 0.0;
    R.n_eff = c2 > 0.0 ? 1.0 / c2 : 0.0;
    R.entropy = 0.0;
    for (int64_t i = 0; i < off_l; ++i)
        if (lambda[i] > 0.0) R.entropy -= lambda[i] * std::log(lambda[i]);
    *summary = R;
    return ECUT_OK;
}

}  // extern "C"
