// C ABI of libecut: handle life cycle, device upload, H*psi, batched H*psi
// and the canonical <-> bipartite permutations.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstring>
#include <map>
#include <mutex>
#include <new>
#include <string>
#include <thread>
#include <vector>

#include "ecut_internal.h"
#include "kernels.h"
#include "runtime.h"

static ecut_status check_dev(const ecut_sectors *s);   // handle on the current device

namespace ecut {

static thread_local std::string g_err;

void set_error(const std::string &msg) { g_err = msg; }

ecut_status fail(ecut_status st, const std::string &msg) {
    g_err = msg;
    return st;
}

ecut_status hip_fail(hipError_t e, const char *what) {
    return fail(ECUT_EDEVICE, std::string(what) + ": " + hipGetErrorString(e));
}

// ---------------------------------------------------------------- per-device resources
namespace {
struct DevRes {
    uint64_t *binom = nullptr;
    int n_cu = 0;
    size_t max_lds = 0;
    bool lds_set = false;
};
std::mutex g_dev_mu;
std::map<int, DevRes> g_dev;
}  // namespace

static std::atomic<size_t> g_last_max_lds{0};   // read by launches on any thread

ecut_status device_res(int *dev_out, const uint64_t **binom_out, int *n_cu_out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
    std::lock_guard<std::mutex> g(g_dev_mu);
    DevRes &R = g_dev[dev];
    if (!R.binom) {
        std::vector<uint64_t> t(65 * 65);
        for (int n = 0; n <= 64; ++n)
            for (int k = 0; k <= 64; ++k) t[n * 65 + k] = binom(n, k);
        void *p = nullptr;
        e = hipMalloc(&p, t.size() * sizeof(uint64_t));
        if (e != hipSuccess) return hip_fail(e, "hipMalloc(binomial table)");
        e = hipMemcpy(p, t.data(), t.size() * sizeof(uint64_t), hipMemcpyHostToDevice);
        if (e != hipSuccess) return hip_fail(e, "hipMemcpy(binomial table)");
        R.binom = (uint64_t *)p;
        hipDeviceProp_t prop;
        e = hipGetDeviceProperties(&prop, dev);
        if (e != hipSuccess) return hip_fail(e, "hipGetDeviceProperties");
        R.n_cu = prop.multiProcessorCount;
        R.max_lds = prop.sharedMemPerBlock;
        // Raising the dynamic-LDS cap is only a request: where the runtime
        // does not take the attribute, launches up to the device limit work
        // without it, so a refusal is cleared and ignored.
        e = set_hub_lds_limits((size_t)prop.sharedMemPerBlock > 65536 ? prop.sharedMemPerBlock : 65536);
        if (e != hipSuccess) (void)hipGetLastError();
        R.lds_set = e == hipSuccess;
    }
    if (dev_out) *dev_out = dev;
    if (binom_out) *binom_out = R.binom;
    if (n_cu_out) *n_cu_out = R.n_cu;
    g_last_max_lds = R.max_lds;
    return ECUT_OK;
}

// ---------------------------------------------------------------- upload
namespace {
struct Arena {
    size_t off = 0;
    struct Piece {
        size_t off;
        const void *src;
        size_t bytes;
    };
    std::vector<Piece> pieces;
    template <class T>
    size_t add(const std::vector<T> &v) {
        size_t o = off;
        size_t b = v.size() * sizeof(T);
        if (b) pieces.push_back({o, v.data(), b});
        off += (b + 255) & ~(size_t)255;
        if (b == 0) off += 256;   // keep a distinct, valid address
        return o;
    }
};
}  // namespace

// ---------------------------------------------------------------- table memory
// The sector tables of a handle come from the caller's allocator when one is
// set (ecut_set_allocator), else from hipMalloc.  Each allocation remembers
// the pair that made it, so it is released through that pair even after the
// caller installs another one.
namespace {
struct MetaAlloc {
    ecut_alloc_fn alloc = nullptr;
    ecut_free_fn free = nullptr;
    void *user = nullptr;
};
std::mutex g_alloc_mu;
MetaAlloc g_alloc;
std::map<void *, std::pair<MetaAlloc, size_t>> g_alloc_owner;   // live allocations of callers' allocators
}  // namespace

static ecut_status table_alloc(void **p, size_t bytes, int device) {
    MetaAlloc a;
    {
        std::lock_guard<std::mutex> g(g_alloc_mu);
        a = g_alloc;
    }
    if (!a.alloc) {
        const hipError_t e = hipMalloc(p, bytes);
        if (e != hipSuccess) return fail(ECUT_ENOMEM, std::string("hipMalloc(sector tables): ") + hipGetErrorString(e));
        return ECUT_OK;
    }
    void *m = a.alloc(bytes, device, a.user);
    if (!m) return fail(ECUT_ENOMEM, "the caller's allocator returned NULL for the sector tables");
    if ((uintptr_t)m & 255) {
        a.free(m, bytes, device, a.user);
        return fail(ECUT_EINVAL, "the caller's allocator returned memory that is not 256-byte aligned");
    }
    std::lock_guard<std::mutex> g(g_alloc_mu);
    g_alloc_owner[m] = {a, bytes};
    *p = m;
    return ECUT_OK;
}

static void table_free(void *p, int device) {
    MetaAlloc a;
    size_t bytes = 0;
    {
        std::lock_guard<std::mutex> g(g_alloc_mu);
        auto it = g_alloc_owner.find(p);
        if (it != g_alloc_owner.end()) {
            a = it->second.first;
            bytes = it->second.second;
            g_alloc_owner.erase(it);
        }
    }
    if (!a.free) {   // made by hipMalloc (the wait inside hipFree happens outside the lock)
        (void)hipFree(p);
        return;
    }
    // hipFree waits for the device; a caller's free may hand the memory out
    // again at once, so kernels still reading the tables must finish first
    (void)hipDeviceSynchronize();
    a.free(p, bytes, device, a.user);
}

void release_device(ecut_sectors *s) {
    if (s->dev_mem) {
        int cur = 0;
        hipGetDevice(&cur);
        if (s->device >= 0 && s->device != cur) (void)hipSetDevice(s->device);
        table_free(s->dev_mem, s->device >= 0 ? s->device : cur);
        if (s->device >= 0 && s->device != cur) (void)hipSetDevice(cur);
    }
    s->dev_mem = nullptr;
    s->on_device = false;
}

ecut_status upload(ecut_sectors *s) {
    int dev = 0;
    ecut_status st = device_res(&dev, nullptr, nullptr);
    if (st != ECUT_OK) return st;
    Arena A;
    const size_t o_blocks = A.add(s->blocks);
    const size_t o_lw = A.add(s->lwords), o_rw = A.add(s->rwords);
    const size_t o_hlp = A.add(s->hl_ptr), o_hlc = A.add(s->hl_col), o_hlv = A.add(s->hl_val);
    const size_t o_hrp = A.add(s->hr_ptr), o_hrc = A.add(s->hr_col), o_hrv = A.add(s->hr_val);
    const size_t o_dl = A.add(s->diag_l), o_dr = A.add(s->diag_r);
    const size_t o_xd = A.add(s->xdiag), o_xb = A.add(s->xbond), o_maps = A.add(s->maps), o_xdl = A.add(s->xdl);
    std::vector<ItemDev> row_items(std::max(s->items_cap, s->items.size()), ItemDev{0, 0, 0, 0, 0, 0});
    std::copy(s->items.begin(), s->items.end(), row_items.begin());   // capacity for any tile size
    const size_t o_items = A.add(row_items);
    size_t o_lc = 0, o_le = 0, o_lr = 0, o_hc = 0, o_he = 0, o_seg = 0, o_xbh = 0, o_cf = 0, o_u = 0, o_rw16 = 0,
           o_rw32 = 0, o_cor = 0, o_order = 0;
    if (s->hub_ok) {
        o_lc = A.add(s->hub_lo_cnt);
        o_le = A.add(s->hub_lo_ent);
        o_lr = A.add(s->hub_lo_rank);
        o_hc = A.add(s->hub_hi_cnt);
        o_he = A.add(s->hub_hi_ent);
        o_seg = A.add(s->hub_seg_off);
        o_xbh = A.add(s->hub_xb);
        o_cf = A.add(s->hub_coef);
        o_u = A.add(s->hub_u);
        o_rw16 = A.add(s->hub_rw16);
        o_rw32 = A.add(s->hub_rw32);
        o_cor = A.add(s->hub_col_of_rank);
        o_order = A.add(s->row_order);
    }
    size_t o_hcc = 0, o_hsc = 0, o_hhw = 0, o_hhc = 0, o_hhe = 0, o_hlw = 0, o_hlcn = 0, o_hle = 0, o_hit = 0;
    std::vector<HubItem> items_cap;   // must outlive the copies below
    if (s->hub_ok) {
        o_hcc = A.add(s->hc_cls);
        o_hsc = A.add(s->hc_segcol);
        o_hhw = A.add(s->hc_hiw);
        o_hhc = A.add(s->hc_hicnt);
        o_hhe = A.add(s->hc_hient);
        o_hlw = A.add(s->hc_low);
        o_hlcn = A.add(s->hc_locnt);
        o_hle = A.add(s->hc_loent);
        items_cap.assign(std::max(s->hub_items_cap, s->hub_items_ord.size()), HubItem{0, 0, 0, -1});
        std::copy(s->hub_items_ord.begin(), s->hub_items_ord.end(), items_cap.begin());
        o_hit = A.add(items_cap);
    }
    size_t o_srl = 0, o_srh = 0, o_sfm = 0, o_sfc = 0, o_hbm = 0, o_hbb = 0, o_hbc = 0;
    if (s->spin_ok || s->hubrow_ok || s->sp2_ok) {
        o_srl = A.add(s->spin_rank_lo);
        o_srh = A.add(s->spin_rank_hi);
    }
    if (s->hubrow_ok) {
        o_hbm = A.add(s->hrow_bmask);
        o_hbb = A.add(s->hrow_bbetw);
        o_hbc = A.add(s->hrow_bcoef);
    }
    size_t o_spr = 0, o_spb = 0, o_spp = 0, o_spc = 0, o_spv = 0, o_spt = 0, o_sptb = 0, o_flat = 0;
    if (s->spin_ok || s->sp2_ok) {
        o_sfm = A.add(s->spin_fmask);
        o_sfc = A.add(s->spin_fcoef);
        o_spr = A.add(s->sp_level_rows);
        o_spb = A.add(s->sp_lblocks);
        o_spp = A.add(s->sp_pptr);
        o_spc = A.add(s->sp_pcol);
        o_spv = A.add(s->sp_pval);
        o_spt = A.add(s->sp_tab);
        o_sptb = A.add(s->sp_tbase);
        o_flat = A.add(s->flat_base);
    }
    size_t o_3si = 0, o_3li = 0, o_3lo = 0, o_3hn = 0, o_3hc = 0;
    if (s->hub3_ok) {
        o_3si = A.add(s->h3_seginfo);
        o_3li = A.add(s->h3_loinfo);
        o_3lo = A.add(s->h3_looff);
        o_3hn = A.add(s->h3_hnb);
        o_3hc = A.add(s->h3_hcnt);
    }
    size_t o_5us = 0, o_5uh = 0, o_5ul = 0, o_5ux = 0, o_5it = 0;
    if (s->hubseg_ok) {
        o_5us = A.add(s->hs_useg);
        o_5uh = A.add(s->hs_uhnb);
        o_5ul = A.add(s->hs_ulo);
        o_5ux = A.add(s->hs_ucross);
        o_5it = A.add(s->hs_items);
    }
    size_t o_6k = 0, o_6v = 0, o_6r = 0, o_6p = 0, o_6c = 0, o_6w = 0, o_hp = 0;
    if (s->hub6_ok) {
        o_6k = A.add(s->h6_col);
        o_6v = A.add(s->h6_val);
        o_6r = A.add(s->level_rows);
        o_6p = A.add(s->h6_pptr);
        o_6c = A.add(s->h6_pcol);
        o_6w = A.add(s->h6_pval);
        o_hp = A.add(s->hp_panels);
    }
    void *mem = nullptr;
    st = table_alloc(&mem, A.off, dev);
    if (st != ECUT_OK) return st;
    // one host image of the whole block, one copy (each copy of pageable
    // memory is a synchronous call with its own staging)
    std::vector<char> image(A.off, 0);
    for (auto &p : A.pieces) std::memcpy(image.data() + p.off, p.src, p.bytes);
    hipError_t e = hipMemcpy(mem, image.data(), A.off, hipMemcpyHostToDevice);
    if (e != hipSuccess) {
        table_free(mem, dev);
        return hip_fail(e, "hipMemcpy(sector tables)");
    }
    char *b = (char *)mem;
    ProblemDev &P = s->prob;
    P = ProblemDev{};
    P.kind = s->kind;
    P.n_blocks = (int32_t)s->blocks.size();
    P.n_xdiag = (int32_t)s->xdiag.size();
    P.n_xbond = (int32_t)s->xbond.size();
    P.blocks = (const BlockDev *)(b + o_blocks);
    P.lwords = (const uint32_t *)(b + o_lw);
    P.rwords = (const uint32_t *)(b + o_rw);
    P.hl_ptr = (const int32_t *)(b + o_hlp);
    P.hl_col = (const int32_t *)(b + o_hlc);
    P.hl_val = (const double *)(b + o_hlv);
    P.hr_ptr = (const int32_t *)(b + o_hrp);
    P.hr_col = (const int32_t *)(b + o_hrc);
    P.hr_val = (const double *)(b + o_hrv);
    P.diag_l = (const double *)(b + o_dl);
    P.diag_r = (const double *)(b + o_dr);
    P.xdiag = (const XDiagDev *)(b + o_xd);
    P.xdl = (const double *)(b + o_xdl);
    P.n_xr = (int32_t)s->xr_site.size();
    for (int g = 0; g < P.n_xr; ++g) P.xr_site[g] = s->xr_site[g];
    P.xr_lo = P.n_xr > 0 ? P.xr_site[0] : 0;
    P.xr_contig = 1;
    for (int g = 1; g < P.n_xr; ++g)
        if (P.xr_site[g] != P.xr_lo + g) P.xr_contig = 0;
    P.xbond = (const XBondDev *)(b + o_xb);
    P.maps = (const int32_t *)(b + o_maps);
    P.dim = s->dim;
    P.xscale = 1.0;
    P.rows_split = rows_split_of(s);
    if (s->spin_ok || s->sp2_ok) {
        P.spin_ok = (s->spin_ok && s->tune.variant == 0) ? 1 : 0;
        P.n_rflip = (int32_t)s->spin_fmask.size();
        P.max_d_r = s->max_d_r;
        P.rank_lo = (const int32_t *)(b + o_srl);
        P.rank_hi = (const int32_t *)(b + o_srh);
        P.rflip_mask = (const uint32_t *)(b + o_sfm);
        P.rflip_coef = (const double *)(b + o_sfc);
        s->dev_sp_rows = (int32_t *)(b + o_spr);
        s->dev_sp_lblocks = (SpinLBlock *)(b + o_spb);
        s->dev_sp_pptr = (const int32_t *)(b + o_spp);
        s->dev_sp_pcol = (const int32_t *)(b + o_spc);
        s->dev_sp_pval = (const double *)(b + o_spv);
        s->dev_sp_tab = (const uint16_t *)(b + o_spt);
        s->dev_sp_tbase = (const int64_t *)(b + o_sptb);
        P.sp_tab = s->dev_sp_tab;
        P.sp_tbase = s->dev_sp_tbase;
        P.flat_base = (const int32_t *)(b + o_flat);
        P.flat_groups = s->flat_base.empty() ? 0 : s->flat_base.back();
    }
    s->dev_items = (ItemDev *)(b + o_items);
    if (s->hub_ok) {
        HubDev &H = P.hub;
        H = s->hub;
        H.lo_cnt = (const int32_t *)(b + o_lc);
        H.lo_ent = (const int32_t *)(b + o_le);
        H.lo_rank = (const int32_t *)(b + o_lr);
        H.hi_cnt = (const int32_t *)(b + o_hc);
        H.hi_ent = (const int32_t *)(b + o_he);
        H.seg_off = (const int32_t *)(b + o_seg);
        H.xb = (const int32_t *)(b + o_xbh);
        H.coef = (const double *)(b + o_cf);
        H.u = (const double *)(b + o_u);
        H.rwords16 = s->hub_rw16.empty() ? nullptr : (const uint16_t *)(b + o_rw16);
        if (s->hubrow_ok) {
            H.n_dbond = (int32_t)s->hrow_bmask.size();
            H.dbond_mask = (const uint32_t *)(b + o_hbm);
            H.dbond_betw = (const uint32_t *)(b + o_hbb);
            H.dbond_coef = (const double *)(b + o_hbc);
            H.rank_lo = (const int32_t *)(b + o_srl);
            H.rank_hi = (const int32_t *)(b + o_srh);
        }
        H.rwords32 = (const uint32_t *)(b + o_rw32);
        H.col_of_rank = (const int32_t *)(b + o_cor);
        s->dev_row_order = (int32_t *)(b + o_order);
        H.cls = (const int32_t *)(b + o_hcc);
        H.cls_segcol = (const int32_t *)(b + o_hsc);
        H.cls_hiw = (const int32_t *)(b + o_hhw);
        H.cls_hicnt = (const int32_t *)(b + o_hhc);
        H.cls_hient = (const int32_t *)(b + o_hhe);
        H.cls_low = (const int32_t *)(b + o_hlw);
        H.cls_locnt = (const int32_t *)(b + o_hlcn);
        H.cls_loent = (const int32_t *)(b + o_hle);
        s->dev_hub_items = (HubItem *)(b + o_hit);
    }
    if (s->hub3_ok) {
        Hub3Args &A3 = s->h3;
        A3 = Hub3Args{};
        A3.hop = s->hub.hop0;
        A3.u0 = s->hub.u0;
        A3.hl_ptr = P.hl_ptr;
        A3.hl_col = P.hl_col;
        A3.hl_val = P.hl_val;
        A3.n_rows = s->blocks[0].d_l;
        A3.lwords = P.lwords;
        A3.cls = P.hub.cls;
        A3.seginfo = (const int4 *)(b + o_3si);
        A3.loinfo = (const int4 *)(b + o_3li);
        A3.looff = (const int32_t *)(b + o_3lo);
        A3.hnb = (const int32_t *)(b + o_3hn);
        A3.hcnt = (const int32_t *)(b + o_3hc);
        A3.items = s->dev_hub_items;
        A3.n_items = (int32_t)s->hub_items.size();
        A3.dR = s->blocks[0].d_r;
        A3.h = s->hub.h;
        A3.hs = s->h3_hs;
        A3.max_tile = s->h3_max_tile;
        A3.max_nseg = s->hub.max_nseg;
        A3.max_l = 0;
        for (size_t ci = 0; ci + 7 < s->hc_cls.size(); ci += 8) A3.max_l = std::max(A3.max_l, s->hc_cls[ci]);
    }
    if (s->hubseg_ok) {
        HubSegArgs &G = s->hseg;
        G = HubSegArgs{};
        G.hop = s->hub.hop0;
        G.u0 = s->hub.u0;
        G.lwords = P.lwords;
        G.cls = P.hub.cls;
        G.seginfo = (const int4 *)(b + o_3si);
        G.loinfo = (const int4 *)(b + o_3li);
        G.looff = (const int32_t *)(b + o_3lo);
        G.hnb = (const int32_t *)(b + o_3hn);
        G.hcnt = (const int32_t *)(b + o_3hc);
        G.useg = (const int4 *)(b + o_5us);
        G.uhnb = (const int32_t *)(b + o_5uh);
        G.ulo = (const int32_t *)(b + o_5ul);
        G.ucross = (const int32_t *)(b + o_5ux);
        G.items = (const HubSegItem *)(b + o_5it);
        G.n_items = (int32_t)s->hs_items.size();
        G.dR = s->blocks[0].d_r;
        G.h = s->hub.h;
        G.hs = s->h3_hs;
        G.uhs = s->hs_uhs;
    }
    if (s->hub6_ok) {
        const BlockDev &B0 = s->blocks[0];
        HubUArgs &U = s->h6u;
        U = HubUArgs{};
        // level order: a row's neighbours sit in the levels beside it; the
        // left operator's CSR in that order
        U.hl_ptr = (const int32_t *)(b + o_6p);
        U.hl_col = (const int32_t *)(b + o_6c);
        U.hl_val = (const double *)(b + o_6w);
        U.rows = (const int32_t *)(b + o_6r);
        U.uniform = 1;
        for (double v : s->hl_val) U.uniform = U.uniform && v == s->hl_val[0];
        U.hop = s->hl_val.empty() ? 0.0 : s->hl_val[0];
        U.n_rows = B0.d_l;
        U.dR = B0.d_r;
        HubPArgs &Pn = s->hp;
        Pn = HubPArgs{};
        Pn.panels = (const int32_t *)(b + o_hp);
        Pn.hop = U.hop;
        Pn.n_rows = B0.d_l;
        Pn.dR = B0.d_r;
        Pn.n_panels = (int32_t)(s->hp_panels.size() / HUBP_PANEL_INTS);
        HubDArgs &D = s->h6d;
        D = HubDArgs{};
        D.n_slots = s->h6_maxq;
        D.col = (const int32_t *)(b + o_6k);
        D.val = s->h6_uniform ? nullptr : (const double *)(b + o_6v);
        D.hop = s->h6_hop;
        D.lwords = P.lwords;
        D.rwords = P.hub.rwords32;
        D.u = P.hub.u;
        D.u0 = s->hub.u0;
        D.uniform_u = s->hub.uniform_u;
        D.n_rows = B0.d_l;
        D.dR = B0.d_r;
    }
    s->dev_mem = mem;
    s->dev_bytes = A.off;
    s->device = dev;
    s->on_device = true;
    P.flat = flat_on(s) ? (s->hub_spatial ? 2 : 1) : 0;
    return ECUT_OK;
}

static bool default_tuning(const ApplyTuning &T) {
    return T.grid == 0 && T.n_xcd == 0 && T.order == 0 && T.variant == 0 && T.tile == 0;
}

// The default tuning of a spin or spatial Hubbard cut whose tables the flat
// kernel can read (flat_base is built for vectors it is the better kernel for)
bool flat_on(const ecut_sectors *s) {
    return s->on_device && s->kernel != 1 && !s->flat_base.empty() && default_tuning(s->tune);
}

// Variant 2 of a spin or spatial Hubbard cut, and the default tuning of the
// vectors too long for the flat kernel
bool two_pass_rows(const ecut_sectors *s, const ApplyTuning &T) {
    if (s->kernel == 1 || !s->sp2_ok) return false;
    if (T.variant == 2) return true;
    if (!s->flat_base.empty() || !default_tuning(T)) return false;
    // on the spatial Hubbard cut every row is an item of its own, on threads
    // for the longest one: by default only where the mean row is a quarter of
    // it (14 sites at half filling, 719 of 1,225: 240 against 396 us on the
    // row kernel; 16 sites with 5 + 5 particles, 320 of 4,900: 1.74 against 0.75 ms)
    // and fills the 128 threads of the smallest group (13 sites at half filling
    // cut after 7, mean row 183: 84 against 103 us; after 8, 49: 196 against 102;
    // after 10, 5: 1,700 against 106; cut after 7 with 6 + 5 particles, 145: 75
    // against 81; with 5 + 5, 115: 70 against 63)
    // spin rows shorter than half a wave on average stay on the one-pass kernel,
    // several rows a group (right part of 7 sites, 23-site chain, mean row 22: 62
    // against 67 us; 24 sites with 9 up spins, 26: 59 both; 24 sites cut after
    // 16, 42: 117 against 87)
    int64_t rows = 0;
    for (const BlockDev &B : s->blocks) rows += B.d_l;
    if (!s->hub_spatial) return s->dim >= rows * SPIN_MIN_MEAN_ROW;
    return s->dim >= rows * s->max_d_r / 4 && s->dim >= rows * HUBSP_MIN_MEAN_ROW;
}

// Many short rows (one particle or hole of the down spin, or none): the fused
// and the two-pass kernels give every row lanes of its own, the class tiles
// pack rows.  The line is in the number of rows: 15 sites with 7 + 1 particles
// (6,435 rows of 15) fused 14.6 against 15.5 us, 16 sites with 6 + 1 (8,008 of 16)
// 17.3 against 15.3, with 8 + 0 (12,870 of 1) 25.6 against 10.3; 18 sites with
// 9 + 1 (48,620 of 18) 150 against 68, 20 with 10 + 1 (184,756 of 20), two passes,
// 264 against 214.
static bool hub_short_rows(const ecut_sectors *s) {
    return s->hub2_ok && s->blocks[0].d_r < HUB_SHORT_ROW && s->blocks[0].d_l >= HUB_SHORT_ROW_MIN_ROWS;
}

// The default tuning, and the two-pass tuning, of a Hubbard up/down problem
// short enough for the fused kernel.  With one hop value (no value table to
// read) it wins at 853,776 amplitudes (13.3 against 17 us, one launch instead of
// two) and is level at 2.9M (37 us both); with signed hops it wins at 213,444
// (7.5 against 10), is level at 853,776 (20 us both) and loses at 2.9M (56
// against 48).
bool hub_fused_size(const ecut_sectors *s) {
    return s->kernel == 1 && s->hub6_ok && s->dim <= (s->h6_uniform ? HUBF_MAX_DIM_UNIFORM : HUBF_MAX_DIM);
}
// Variant 6 with no other field set leaves the choice to the library too; with
// any of them it names the two passes and their launch shape.
bool hub_fused(const ecut_sectors *s) {
    const ApplyTuning &T = s->tune;
    return hub_fused_size(s) && T.grid == 0 && T.n_xcd == 0 && T.order == 0 && T.tile == 0 &&
           (T.variant == 6 || (T.variant == 0 && !hub_short_rows(s)));
}

// The default tuning above those sizes: the two-pass kernels, which beat the
// one-pass class tiles at every size measured (12-site chain 16.4 against 22.4
// us, 14-site 180 against 325, 14-site ring 186 against 481); long vectors take
// the class tiles for the right pass where they exist (16-site chain: 2.2 against
// 2.8 ms; 4 + 8 particles, 23.4M amplitudes, 300 against 365 us, where the one-pass
// class tiles take 344; 8 + 4, 371 against 402; 15 sites, 19.3M, 5 + 7 264 against
// 290, but 7 + 5 312 against 297).
ApplyTuning hub_tuning(const ecut_sectors *s) {
    if (s->kernel != 1 || !default_tuning(s->tune) || !s->hub6_ok || hub_short_rows(s)) return s->tune;
    if (s->hub3_ok && s->dim >= HUB7_MIN_DIM) return ApplyTuning{8, 8, 0, 7, 0};
    return ApplyTuning{0, 8, 0, 6, 0};
}

int32_t max_tile_elems(const ecut_sectors *s) {
    int64_t m = 0;
    for (auto &it : s->items) m = std::max<int64_t>(m, (int64_t)(it.row1 - it.row0) * s->blocks[it.block].d_r);
    return (int32_t)m;
}

// The generic kernel's items are row tiles of about 2,048 amplitudes, and at
// least one row: a problem of few or long rows has too few of them to fill the
// device.  Such a problem's items are cut into slices of at least one pass of
// a work group until the launch has about ROWS_MIN_GROUPS groups.  Problems the
// spin kernel can take keep whole items (the generic kernel is their fallback
// tuning, with rows staged in LDS).
int32_t rows_split_of(const ecut_sectors *s) {
    if (s->kernel == 1 || s->spin_ok || s->item_slots <= 0) return 1;
    int64_t tile = 0;
    const bool own = s->hub_spatial || s->wide_rows;   // items may hold the two-pass kernels' rows
    for (const ItemDev &it : own ? s->generic_items : s->items)
        tile = std::max<int64_t>(tile, (int64_t)(it.row1 - it.row0) * s->blocks[it.block].d_r);
    const int64_t n = own ? (int64_t)s->generic_items.size() : s->item_slots;
    const int64_t most = (tile + ROWS_THREADS - 1) / ROWS_THREADS;
    return (int32_t)std::max<int64_t>(1, std::min<int64_t>(most, std::min<int64_t>(ROWS_MIN_GROUPS / n, 65535)));
}

// Item counts of the two-pass kernels for the current tuning: the left pass
// takes `grid` rows of the level order (0 = HUBU_ROWS) per item over slabs of
// 64 lanes x 1 or 2 columns; the right pass `tile` rows (0 = HUBD_ROWS) x
// HUBD_THREADS columns per item.
static int32_t hub6_rows_d(const ApplyTuning &T) { return T.tile > 0 ? T.tile : HUBD_ROWS; }

void hub6_shape(const ecut_sectors *s, HubUArgs &U, HubDArgs &D) {
    const int32_t dR = s->blocks[0].d_r, nr = s->blocks[0].d_l;
    const int32_t cols = (dR > 1 ? 2 : 1) * 64;
    const ApplyTuning T = hub_tuning(s);
    U.rows_per_item = T.grid > 0 ? T.grid : HUBU_ROWS;
    U.n_rgroups = (nr + U.rows_per_item - 1) / U.rows_per_item;
    U.slab_ways = (T.variant == 7 && T.tile > 0) ? T.tile : 1;
    U.n_slabs = ((dR + cols - 1) / cols + U.slab_ways - 1) / U.slab_ways;
    U.n_items = U.n_slabs * U.n_rgroups;
    // the fused kernel takes single rows: the shorter the items, the more of
    // them to fill the device
    D.rows_per_item = hub_fused(s) ? 1 : hub6_rows_d(T);
    D.n_chunks = (dR + HUBD_THREADS - 1) / HUBD_THREADS;
    D.n_items = ((nr + D.rows_per_item - 1) / D.rows_per_item) * D.n_chunks;
}

// The left operator's pass runs on panels where they exist, unless the tuning
// names the general pass's shape: rows per item, items in launch order, or
// slabs side by side.  The default takes them where a solve's three vectors no
// longer share the last-level cache and panels are long: a panel's low hops cost no load, but its few waves must keep
// the high hops' panels in L2, and with many high sites those are most of the
// loads.  Whole applications, general pass -> panels, by mean rows a panel:
// 16 sites 8 + 8 particles (50 rows) 2,029 -> 1,950 us, 8 + 5 859 -> 818, 6 + 6 (32)
// 855 -> 840, 5 + 8 (20) 716 -> 738, 4 + 8 (11) 298 -> 340; 15 sites 7 + 7 (25)
// 562 -> 549, 5 + 7 (14) 255 -> 277; 17 sites 8 + 4 (48) 977 -> 947, 6 + 4 (27) 499 ->
// 504; 18 sites 9 + 4 (48) 2,563 -> 2,511, but 2,516 with 8 rows an item, 7 + 4 (33)
// level, 6 + 4 (23) 984 -> 1,019; 20 sites 10 + 3 (45) 3,917 -> 3,985.  At the line in
// size, 14 sites 7 + 7 (27; 11.8M amplitudes): 180 -> 172 on three vectors in turn,
// 125 -> 133 on one pair; below, 16 sites 8 + 3 (50; 7.2M) 89 -> 97 on one pair.
static bool panels_by_default(const ecut_sectors *s) {
    const int64_t panels = (int64_t)s->hp_panels.size() / HUBP_PANEL_INTS;
    return s->n_sites <= 17 && s->dim >= HUBP_MIN_DIM &&
           s->blocks[0].d_l >= panels * (s->n_sites <= 16 ? HUBP_MIN_MEAN : HUBP_MIN_MEAN_17);
}
static bool left_on_panels(const ecut_sectors *s) {
    const ApplyTuning &T = s->tune;
    if (default_tuning(T)) return s->hp_lo > 0 && panels_by_default(s);
    return s->hp_lo > 0 && T.grid == 0 && T.n_xcd != 1 && !(T.variant == 7 && T.tile > 0);
}

static hipError_t launch_left(const ecut_sectors *s, const HubUArgs &U, int n_xcd, hipStream_t st) {
    if (!left_on_panels(s)) return launch_hub6_left(U, n_xcd, st);
    HubPArgs A = s->hp;
    A.x = U.x;
    A.y = U.y;
    return launch_hubP(A, s->hp_lo, st);
}

static HubFArgs hub_fused_args(const ecut_sectors *s, const ProblemDev &P) {
    HubUArgs U = s->h6u;
    HubFArgs F{};
    F.d = s->h6d;
    hub6_shape(s, U, F.d);
    F.d.x = P.x;
    F.d.y = P.y;
    F.d.z = P.z;
    F.d.partials = P.partials;
    F.d.xscale = P.xscale;
    F.d.zcoef = P.zcoef;
    F.d.dscale = P.dscale;
    F.hl_ptr = P.hl_ptr;
    F.hl_col = P.hl_col;
    F.hl_val = P.hl_val;
    return F;
}

// One application on a stream, with the Lanczos epilogue fields of `P`
// already filled in by the caller.
ecut_status launch_apply(const ecut_sectors *s, const ProblemDev &P, hipStream_t st) {
    int dev = 0, n_cu = 0;
    ecut_status rs = device_res(&dev, nullptr, &n_cu);
    if (rs != ECUT_OK) return rs;
    hipError_t e;
    if (hub_fused(s)) {
        e = launch_hubF(hub_fused_args(s, P), st);
    } else if (s->kernel == 1) {
        const ApplyTuning T = hub_tuning(s);
        const int n_xcd = T.n_xcd > 0 ? T.n_xcd : 8;
        if ((T.variant == 0 || T.variant == 3) && s->hub3_ok) {
            const size_t lds = hub3_lds_bytes(s);
            if (lds > g_last_max_lds) return fail(ECUT_EUNSUPPORTED, "class tiles exceed the device's LDS per work group");
            const int grid = T.grid > 0 ? T.grid : n_cu * hub_blocks_per_cu(3, lds);
            Hub3Args A3 = s->h3;
            A3.x = P.x;
            A3.y = P.y;
            A3.z = P.z;
            A3.partials = P.partials;
            A3.items = s->dev_hub_items;
            A3.n_items = (int32_t)s->hub_items_ord.size();
            A3.xscale = P.xscale;
            A3.zcoef = P.zcoef;
            A3.dscale = P.dscale;
            const int slab_grid = 8 * std::max(1, (n_cu / 8) * hub_blocks_per_cu(4, 0));
            e = launch_hub3(s, A3, grid, n_xcd, T.variant == 3, slab_grid, st);
        } else if ((T.variant == 6 && s->hub6_ok) || (T.variant == 7 && s->hub3_ok)) {
            // left operator on flat slab items of `grid` rows (0 = HUBU_ROWS)
            HubUArgs U = s->h6u;
            HubDArgs D = s->h6d;
            hub6_shape(s, U, D);
            U.x = D.x = P.x;
            U.y = D.y = P.y;
            e = launch_left(s, U, n_xcd, st);
            if (e == hipSuccess && T.variant == 6) {
                D.z = P.z;
                D.partials = P.partials;
                D.xscale = P.xscale;
                D.zcoef = P.zcoef;
                D.dscale = P.dscale;
                e = launch_hubD_only(D, n_xcd, st);
            } else if (e == hipSuccess) {
                // right operator, diagonal and epilogue on class tiles (the
                // left operator's sum is already in y)
                const size_t lds = hub3_lds_bytes(s);
                if (e == hipSuccess && lds > g_last_max_lds)
                    return fail(ECUT_EUNSUPPORTED, "class tiles exceed the device's LDS per work group");
                Hub3Args A3 = s->h3;
                A3.x = P.x;
                A3.y = P.y;
                A3.z = P.z;
                A3.partials = P.partials;
                A3.items = s->dev_hub_items;
                A3.n_items = (int32_t)s->hub_items_ord.size();
                A3.xscale = P.xscale;
                A3.zcoef = P.zcoef;
                A3.dscale = P.dscale;
                const int grid = n_cu * hub_blocks_per_cu(3, lds);
                if (e == hipSuccess) e = launch_hub3(s, A3, grid, n_xcd, true, 0, st);
            }
        } else if (T.variant == 5 && s->hubseg_ok) {
            const size_t lds = (size_t)s->hs_max_tile * 8;
            if (lds > g_last_max_lds) return fail(ECUT_EUNSUPPORTED, "segment tiles exceed the device's LDS per work group");
            const int grid = T.grid > 0 ? T.grid : n_cu * hub_blocks_per_cu(5, lds);
            HubSegArgs G = s->hseg;
            G.x = P.x;
            G.y = P.y;
            G.z = P.z;
            G.partials = P.partials;
            G.xscale = P.xscale;
            G.zcoef = P.zcoef;
            G.dscale = P.dscale;
            e = launch_hubseg(s, G, grid, n_xcd == 1 ? 1 : 8, st);
        } else if (T.variant == 4 && s->hubrow_ok) {
            if (((uintptr_t)P.x | (uintptr_t)P.y | (uintptr_t)P.z) & 15)
                return fail(ECUT_EINVAL, "the whole-row kernel needs 16-byte aligned vectors");
            e = launch_hubrow(s, P, s->dev_row_order, s->blocks[0].d_l, T.grid, n_xcd == 8 ? 8 : 1,
                              T.tile > 0 ? T.tile : 1024, n_cu, st);
        } else if ((T.variant == 0 || T.variant == 2) && s->hub2_ok) {
            const size_t lds = hub2_lds_bytes(s);
            if (lds > g_last_max_lds) return fail(ECUT_EUNSUPPORTED, "class tiles exceed the device's LDS per work group");
            const int grid = T.grid > 0 ? T.grid : n_cu * hub_blocks_per_cu(2, lds);
            e = launch_hub2(s, P, s->dev_hub_items, (int)s->hub_items_ord.size(), grid, n_xcd, st);
        } else {
            if (hub_lds_bytes(s) > g_last_max_lds)
                return fail(ECUT_EUNSUPPORTED, "Hubbard kernel tables exceed the device's LDS per work group");
            const int grid = T.grid > 0 ? T.grid : n_cu;
            e = launch_hub(s, P, s->dev_row_order, s->blocks[0].d_l, grid, n_xcd, st);
        }
    } else if (two_pass_rows(s, s->tune)) {
        SpinLArgs L{};
        L.x = P.x;
        L.y = P.y;
        L.hl_ptr = s->dev_sp_pptr;
        L.hl_col = s->dev_sp_pcol;
        L.hl_val = s->dev_sp_pval;
        L.rows = s->dev_sp_rows;
        L.blocks = s->dev_sp_lblocks;
        L.n_blocks = (int32_t)s->sp_lblocks.size();
        L.n_items = s->sp_lblocks.empty() ? 0
                                          : s->sp_lblocks.back().item0 +
                                                s->sp_lblocks.back().n_rgroups * s->sp_lblocks.back().n_slabs;
        L.rows_per_item = s->tune.grid > 0 ? s->tune.grid : HUBU_ROWS;
        e = launch_spin2(L, P, s->dev_sp_tab, s->dev_sp_tbase, s->dev_items, s->sp_n_one, (int)s->items.size(),
                         s->max_d_r, s->tune.n_xcd == 1 ? 1 : 8, s->hub_spatial, st);
    } else if (P.flat) {
        e = launch_flat(P, st);
    } else if (P.spin_ok) {
        int grid = s->tune.grid;
        if (s->tune.order == 1) grid = std::max(8, ((grid > 0 ? grid : 2048) / 8) * 8);   // keeps chunk c on XCD c
        e = launch_spin(nullptr, P, s->dev_items, (int)s->items.size(), max_tile_elems(s), s->max_d_r, grid, st);
    } else {
        e = launch_rows(nullptr, P, s->dev_items, (int)s->items.size(), max_tile_elems(s), P.rows_split, st);
    }
    if (e != hipSuccess) return hip_fail(e, "kernel launch (apply_H)");
    return ECUT_OK;
}

// the kernels launch_apply runs, in the order of its branches
static const char *kernel_names(const ecut_sectors *s) {
    if (hub_fused(s)) return "k_hubF";
    if (s->kernel == 1) {
        const ApplyTuning T = hub_tuning(s);
        const bool panels = left_on_panels(s);
        if ((T.variant == 0 || T.variant == 3) && s->hub3_ok) return T.variant == 3 ? "k_upslab+k_hub3" : "k_hub3";
        if (T.variant == 6 && s->hub6_ok) return panels ? "k_hubP+k_hubD" : "k_hubU+k_hubD";
        if (T.variant == 7 && s->hub3_ok) return panels ? "k_hubP+k_hub3" : "k_hubU+k_hub3";
        if (T.variant == 5 && s->hubseg_ok) return "k_hubseg";
        if (T.variant == 4 && s->hubrow_ok) return "k_hubrow";
        return (T.variant == 0 || T.variant == 2) && s->hub2_ok ? "k_hub2" : "k_hub";
    }
    if (two_pass_rows(s, s->tune)) return "k_spinL+k_spinR";
    if (!s->flat_base.empty() && default_tuning(s->tune)) return "k_flat";
    return s->spin_ok && s->tune.variant == 0 ? "k_spin" : "k_rows";
}

bool own_launch(const ecut_sectors *s) { return s->kernel == 1 || two_pass_rows(s, s->tune); }

bool hub6_batchable(const ecut_sectors *s) {
    return s->kernel == 1 && s->hub6_ok && hub_tuning(s).variant == 6 && s->h6_maxq <= HUBD_BATCH_SLOTS;
}

void hub6_batch_add(HubBatch &b, const ecut_sectors *s, const ProblemDev &P) {
    if (hub_fused(s)) {
        b.f.push_back(hub_fused_args(s, P));
        b.off_f.push_back(b.off_f.back() + b.f.back().d.n_items);
        return;
    }
    HubUArgs U = s->h6u;
    HubDArgs D = s->h6d;
    hub6_shape(s, U, D);
    U.x = D.x = P.x;
    U.y = D.y = P.y;
    D.z = P.z;
    D.partials = P.partials;
    D.xscale = P.xscale;
    D.zcoef = P.zcoef;
    D.dscale = P.dscale;
    if (left_on_panels(s)) {
        // left pass of its own: the merged launch of the general left passes
        // gets no item of this problem
        HubPArgs A = s->hp;
        A.x = P.x;
        A.y = P.y;
        b.p.push_back(A);
        b.p_lo.push_back(s->hp_lo);
        U.n_items = 0;
    }
    b.u.push_back(U);
    b.d.push_back(D);
    b.off_u.push_back(b.off_u.back() + U.n_items);
    b.off_d.push_back(b.off_d.back() + D.n_items);
}

HubBatchLayout hub6_batch_layout(const HubBatch &b, size_t base) {
    auto al = [](size_t o) { return (o + 255) & ~(size_t)255; };
    HubBatchLayout l;
    l.u = al(base);
    l.d = al(l.u + b.u.size() * sizeof(HubUArgs));
    l.off_u = al(l.d + b.d.size() * sizeof(HubDArgs));
    l.off_d = al(l.off_u + b.off_u.size() * sizeof(int32_t));
    l.f = al(l.off_d + b.off_d.size() * sizeof(int32_t));
    l.off_f = al(l.f + b.f.size() * sizeof(HubFArgs));
    l.bytes = l.off_f + b.off_f.size() * sizeof(int32_t);
    return l;
}

void hub6_batch_pack(const HubBatch &b, const HubBatchLayout &l, char *buf) {
    std::memcpy(buf + l.u, b.u.data(), b.u.size() * sizeof(HubUArgs));
    std::memcpy(buf + l.d, b.d.data(), b.d.size() * sizeof(HubDArgs));
    std::memcpy(buf + l.off_u, b.off_u.data(), b.off_u.size() * sizeof(int32_t));
    std::memcpy(buf + l.off_d, b.off_d.data(), b.off_d.size() * sizeof(int32_t));
    std::memcpy(buf + l.f, b.f.data(), b.f.size() * sizeof(HubFArgs));
    std::memcpy(buf + l.off_f, b.off_f.data(), b.off_f.size() * sizeof(int32_t));
}

hipError_t hub6_batch_launch(const HubBatch &b, const HubBatchLayout &l, const void *dev, hipStream_t st) {
    if (b.empty()) return hipSuccess;
    const char *d = (const char *)dev;
    hipError_t e = launch_hubF_batch((const HubFArgs *)(d + l.f), (const int32_t *)(d + l.off_f), (int)b.f.size(),
                                           b.off_f.back(), st);
    for (size_t k = 0; k < b.p.size() && e == hipSuccess; ++k) e = launch_hubP(b.p[k], b.p_lo[k], st);
    if (e != hipSuccess) return e;
    return launch_hub6_batch((const HubUArgs *)(d + l.u), (const HubDArgs *)(d + l.d), (const int32_t *)(d + l.off_u),
                             (const int32_t *)(d + l.off_d), (int)b.u.size(), b.off_u.back(), b.off_d.back(), st);
}

// number of partial slots the apply kernel writes
int32_t apply_partial_slots(const ecut_sectors *s) {
    if (flat_on(s)) return s->prob.flat_groups;
    if (s->kernel != 1) return s->item_slots * ((s->spin_ok || two_pass_rows(s, s->tune)) ? 1 : s->prob.rows_split);
    const ApplyTuning T = hub_tuning(s);
    if (T.variant == 5 && s->hubseg_ok) return s->hs_n_slots;
    if (T.variant == 7 && s->hub3_ok) return (int32_t)s->hub_items.size();
    if (T.variant == 6 && s->hub6_ok) {
        HubUArgs U{};
        HubDArgs D{};
        hub6_shape(s, U, D);
        return D.n_items;
    }
    const bool tiles = ((T.variant == 0 || T.variant == 3) && (s->hub3_ok || s->hub2_ok)) ||
                       (T.variant == 2 && s->hub2_ok);   // variants 1 and 4: one slot per row
    return tiles ? (int32_t)s->hub_items.size() : s->blocks[0].d_l;
}

// Slots the generic row kernel writes: one a slice of its items.  From the host
// tables alone, so that a host-only handle gives the sizes of a device handle.
static int32_t rows_partial_slots(const ecut_sectors *s) {
    if (s->spin_ok) return 0;   // whole items, counted by item_slots_cap
    const bool own = s->hub_spatial || s->wide_rows;   // items may hold the two-pass kernels' rows
    return (own ? (int32_t)s->generic_items.size() : s->item_slots) * rows_split_of(s);
}

// workspace size: any kernel of the problem may run on the same workspace
int32_t apply_partial_slots_max(const ecut_sectors *s) {
    // the two-pass kernels use the most slots with one row per right-pass item
    const int32_t h6 = s->hub6_ok ? s->blocks[0].d_l * ((s->blocks[0].d_r + HUBD_THREADS - 1) / HUBD_THREADS) : 0;
    return s->kernel == 1 ? std::max<int32_t>(std::max<int32_t>(std::max<int32_t>(s->blocks[0].d_l,
                                                                                    (int32_t)s->hub_items.size()),
                                                                  s->hubseg_ok ? s->hs_n_slots : 0),
                                              h6)
                          : std::max(std::max(std::max(s->item_slots_cap, s->item_slots), rows_partial_slots(s)),
                                     s->flat_base.empty() ? 0 : s->flat_base.back());
}

// ---------------------------------------------------------------- staging buffers
ecut_status Staging::reserve(size_t bytes) {
    int cur = 0;
    hipGetDevice(&cur);
    if (device >= 0 && device != cur) release();
    if (bytes <= cap && dev) return ECUT_OK;
    ecut_status st = wait();
    if (st != ECUT_OK) return st;
    // kernels launched earlier may still read the old descriptors
    if (dev && hipDeviceSynchronize() != hipSuccess) return fail(ECUT_EDEVICE, "hipDeviceSynchronize(descriptor buffer)");
    if (dev) hipFree(dev);
    if (host) hipHostFree(host);
    dev = host = nullptr;
    cap = 0;
    size_t c = 4096;
    while (c < bytes) c *= 2;
    hipError_t e = hipMalloc(&dev, c);
    if (e != hipSuccess) return fail(ECUT_ENOMEM, "hipMalloc(descriptor buffer)");
    e = hipHostMalloc(&host, c, hipHostMallocDefault);
    if (e != hipSuccess) return fail(ECUT_ENOMEM, "hipHostMalloc(descriptor staging)");
    if (!ev) {
        e = hipEventCreateWithFlags(&ev, hipEventDisableTiming);
        if (e != hipSuccess) return hip_fail(e, "hipEventCreate");
    }
    cap = c;
    device = cur;
    return ECUT_OK;
}

ecut_status Staging::wait() {
    if (pending && ev) {
        hipError_t e = hipEventSynchronize(ev);
        pending = false;
        if (e != hipSuccess) return hip_fail(e, "hipEventSynchronize(descriptor buffer)");
    }
    return ECUT_OK;
}

ecut_status Staging::upload(size_t bytes, hipStream_t st) {
    hipError_t e = hipMemcpyAsync(dev, host, bytes, hipMemcpyHostToDevice, st);
    if (e != hipSuccess) return hip_fail(e, "hipMemcpyAsync(descriptors)");
    e = hipEventRecord(ev, st);
    if (e != hipSuccess) return hip_fail(e, "hipEventRecord");
    pending = true;
    return ECUT_OK;
}

void Staging::release() {
    if (pending && ev) hipEventSynchronize(ev);
    pending = false;
    if (dev) hipFree(dev);
    if (host) hipHostFree(host);
    if (ev) hipEventDestroy(ev);
    dev = host = nullptr;
    ev = nullptr;
    cap = 0;
    device = -1;
}

void make_rows_batch(const std::vector<ProblemDev> &probs, const std::vector<ItemDev> &items_in,
                     const std::vector<int32_t> &tiles, const std::vector<char> &flat, RowsBatch &b) {
    // the spin kernel takes the problems whose tuning selects it (as their
    // own ecut_apply_H does), the generic row kernel the others; the order
    // of the queue is kept within each group
    std::vector<ItemDev> items;
    items.reserve(items_in.size());
    b = RowsBatch{};
    for (const ItemDev &it : items_in)
        if (probs[it.prob].spin_ok) {
            items.push_back(it);
            b.spin_tile = std::max(b.spin_tile, tiles[it.prob]);
            b.spin_src = std::max(b.spin_src, probs[it.prob].max_d_r);
            if (b.first_spin < 0) b.first_spin = it.prob;
        }
    b.n_spin = (int)items.size();
    for (const ItemDev &it : items_in)
        if (!probs[it.prob].spin_ok) {
            items.push_back(it);
            b.rows_tile = std::max(b.rows_tile, tiles[it.prob]);
            b.rows_split = std::max(b.rows_split, probs[it.prob].rows_split);
        }
    b.n_items = (int)items.size();
    for (size_t k = 0; k < flat.size(); ++k) {
        if (!flat[k] || probs[k].flat_groups <= 0) continue;
        const int t = probs[k].flat == 2;
        if (b.flat_off[t].empty()) b.flat_off[t].push_back(0);
        b.flat_idx[t].push_back((int32_t)k);
        b.flat_off[t].push_back(b.flat_off[t].back() + probs[k].flat_groups);
    }
    b.pb = (probs.size() * sizeof(ProblemDev) + 255) & ~(size_t)255;
    size_t bytes = b.pb + items.size() * sizeof(ItemDev);
    for (int t = 0; t < 2; ++t) {
        b.o_flat[t] = bytes = (bytes + 15) & ~(size_t)15;
        bytes += (b.flat_idx[t].size() + b.flat_off[t].size()) * sizeof(int32_t);
    }
    b.buf.assign(bytes, 0);
    std::memcpy(b.buf.data(), probs.data(), probs.size() * sizeof(ProblemDev));
    std::memcpy(b.buf.data() + b.pb, items.data(), items.size() * sizeof(ItemDev));
    for (int t = 0; t < 2; ++t) {
        char *o = b.buf.data() + b.o_flat[t];
        std::memcpy(o, b.flat_idx[t].data(), b.flat_idx[t].size() * sizeof(int32_t));
        std::memcpy(o + b.flat_idx[t].size() * sizeof(int32_t), b.flat_off[t].data(), b.flat_off[t].size() * sizeof(int32_t));
    }
    if (b.first_spin >= 0) b.spin_single = probs[b.first_spin];
    if (!probs.empty()) b.rows_single = probs[0];
}

hipError_t launch_rows_batch(const RowsBatch &b, const void *dev, hipStream_t st) {
    const ProblemDev *probs_d = (const ProblemDev *)dev;
    const ItemDev *items_d = (const ItemDev *)((const char *)dev + b.pb);
    hipError_t e = hipSuccess;
    if (b.n_spin > 0) e = launch_spin(probs_d, b.spin_single, items_d, b.n_spin, b.spin_tile, b.spin_src, 0, st);
    if (e == hipSuccess && b.n_spin < b.n_items)
        e = launch_rows(probs_d, b.rows_single, items_d + b.n_spin, b.n_items - b.n_spin, b.rows_tile, b.rows_split, st);
    for (int t = 0; t < 2 && e == hipSuccess; ++t) {
        const int n = (int)b.flat_idx[t].size();
        const int32_t *idx = (const int32_t *)((const char *)dev + b.o_flat[t]);
        if (n > 0) e = launch_flat_batch(probs_d, idx, idx + n, n, b.flat_off[t].back(), t == 1, st);
    }
    return e;
}

ecut_status make_batch_plan(int32_t n, const ecut_sectors *const *s, const double *const *psi_d,
                            double *const *y_d, BatchPlan &pl) {
    if (n < 0 || (n > 0 && (!s || !psi_d || !y_d))) return fail(ECUT_EINVAL, "bad batch arguments");
    pl = BatchPlan{};
    if (n == 0) return ECUT_OK;
    std::vector<ProblemDev> probs(n);
    std::vector<ItemDev> items;
    std::vector<int32_t> tiles(n, 0);
    std::vector<char> flat(n, 0);   // problems on the flat kernel
    bool any_flat = false;
    for (int32_t k = 0; k < n; ++k) {
        ecut_status st = check_dev(s[k]);
        if (st != ECUT_OK) return st;
        if (!psi_d[k] || !y_d[k] || psi_d[k] == y_d[k]) return fail(ECUT_EINVAL, "bad vector in batch");
    }
    for (int32_t k = 0; k < n; ++k) {
        probs[k] = s[k]->prob;
        probs[k].x = psi_d[k];
        probs[k].y = y_d[k];
        probs[k].z = nullptr;
        probs[k].xscale = 1.0;
        probs[k].zcoef = 0.0;
        probs[k].partials = nullptr;
        if (probs[k].flat) {
            flat[k] = 1;
            any_flat = true;
            continue;
        }
        tiles[k] = max_tile_elems(s[k]);
        if (hub6_batchable(s[k])) {
            hub6_batch_add(pl.hub, s[k], probs[k]);   // one merged launch per pass for all of them
        } else if (own_launch(s[k])) {
            pl.own.push_back(probs[k]);               // other Hubbard tunings and two-pass spin keep their own kernels
            pl.own_s.push_back(s[k]);
        } else {
            for (const ItemDev &it : s[k]->items) items.push_back(ItemDev{k, it.block, it.row0, it.row1, it.slot, 0});
        }
    }
    if (!items.empty() || any_flat) {
        // one queue over all problems, largest tiles first (stable: problem order breaks ties)
        std::stable_sort(items.begin(), items.end(), [&](const ItemDev &a, const ItemDev &b) {
            const int64_t wa = (int64_t)(a.row1 - a.row0) * s[a.prob]->blocks[a.block].d_r;
            const int64_t wb = (int64_t)(b.row1 - b.row0) * s[b.prob]->blocks[b.block].d_r;
            return wa > wb;
        });
        make_rows_batch(probs, items, tiles, flat, pl.rows);
        pl.has_rows = true;
        pl.buf = pl.rows.buf;
    }
    if (!pl.hub.empty()) {
        pl.hub_l = hub6_batch_layout(pl.hub, pl.buf.size());
        pl.buf.resize(pl.hub_l.bytes);
        hub6_batch_pack(pl.hub, pl.hub_l, pl.buf.data());
    }
    return ECUT_OK;
}

ecut_status launch_batch_plan(const BatchPlan &pl, const void *dev, hipStream_t st) {
    for (size_t k = 0; k < pl.own.size(); ++k) {
        ecut_status rs = launch_apply(pl.own_s[k], pl.own[k], st);
        if (rs != ECUT_OK) return rs;
    }
    hipError_t e = hipSuccess;
    if (pl.has_rows) e = launch_rows_batch(pl.rows, dev, st);
    if (e == hipSuccess) e = hub6_batch_launch(pl.hub, pl.hub_l, dev, st);
    if (e != hipSuccess) return hip_fail(e, "kernel launch (batched apply_H)");
    return ECUT_OK;
}

}  // namespace ecut

using namespace ecut;

// ---------------------------------------------------------------- ABI
extern "C" {

const char *ecut_last_error(void) { return g_err.c_str(); }

const char *ecut_version(void) { return "ecut 0.1 (gfx950)"; }

ecut_status ecut_set_allocator(ecut_alloc_fn alloc, ecut_free_fn free_fn, void *user) {
    if ((alloc == nullptr) != (free_fn == nullptr)) return fail(ECUT_EINVAL, "alloc and free must both be set or both be NULL");
    std::lock_guard<std::mutex> g(g_alloc_mu);
    g_alloc = MetaAlloc{alloc, free_fn, user};
    return ECUT_OK;
}

ecut_status ecut_build_sectors(const ecut_model_desc *model, const ecut_cut_desc *cut, ecut_qnum q, uint32_t flags,
                               ecut_sectors **out) {
    if (!out) return fail(ECUT_EINVAL, "out is NULL");
    *out = nullptr;
    if (flags & ~(uint32_t)ECUT_BUILD_HOST_ONLY) return fail(ECUT_EINVAL, "unknown flags");
    ecut_sectors *s = new (std::nothrow) ecut_sectors();
    if (!s) return fail(ECUT_ENOMEM, "host allocation");
    ecut_status st;
    try {
        st = build_host(model, cut, q, s);
    } catch (const std::bad_alloc &) {
        st = fail(ECUT_ENOMEM, "host allocation during sector build");
    }
    if (st == ECUT_OK && !(flags & ECUT_BUILD_HOST_ONLY)) st = upload(s);
    if (st != ECUT_OK) {
        delete s;
        return st;
    }
    *out = s;
    return ECUT_OK;
}

void ecut_sectors_free(ecut_sectors *s) {
    if (!s) return;
    release_device(s);
    delete s;
}

const char *ecut_apply_kernels(const ecut_sectors *s) { return s ? kernel_names(s) : ""; }

ecut_status ecut_sectors_get_info(const ecut_sectors *s, ecut_sectors_info *info) {
    if (!s || !info) return fail(ECUT_EINVAL, "null argument");
    ecut_sectors_info I{};
    I.dim = s->dim;
    I.n_blocks = (int32_t)s->blocks.size();
    I.n_left_sites = (int32_t)s->lsites.size();
    I.n_right_sites = (int32_t)s->rsites.size();
    I.max_d_r = s->max_d_r;
    I.n_cut_bonds = s->n_cut_bonds;
    I.n_cross_offdiag = 2 * (int32_t)s->xbond.size();
    I.n_cross_diag = (int32_t)s->xdiag.size();
    I.kernel = s->kernel;
    I.kernel_flags = (s->hub2_ok ? 1 : 0) | (s->hub3_ok ? 2 : 0) | (s->spin_ok ? 4 : 0) | (s->hubrow_ok ? 8 : 0) |
                     (s->hubseg_ok ? 16 : 0) | (s->hub6_ok ? 32 : 0) |
                     (s->sp2_ok && !s->wide_rows ? 64 : 0);
    I.device_bytes = (int64_t)s->dev_bytes;
    I.n_eff = s->n_eff;
    *info = I;
    return ECUT_OK;
}

ecut_status ecut_sectors_blocks(const ecut_sectors *s, int64_t *blocks) {
    if (!s || !blocks) return fail(ECUT_EINVAL, "null argument");
    for (size_t b = 0; b < s->blocks.size(); ++b) {
        const BlockDev &B = s->blocks[b];
        blocks[5 * b + 0] = B.q_l;
        blocks[5 * b + 1] = B.q_r;
        blocks[5 * b + 2] = B.d_l;
        blocks[5 * b + 3] = B.d_r;
        blocks[5 * b + 4] = B.offset;
    }
    return ECUT_OK;
}

ecut_status ecut_sectors_words(const ecut_sectors *s, int32_t block, uint32_t *l_words, uint32_t *r_words) {
    if (!s) return fail(ECUT_EINVAL, "null handle");
    if (block < 0 || block >= (int32_t)s->blocks.size()) return fail(ECUT_EINVAL, "block out of range");
    const BlockDev &B = s->blocks[block];
    if (l_words) std::memcpy(l_words, s->lwords.data() + B.lbase, sizeof(uint32_t) * (size_t)B.d_l);
    if (r_words) {
        if (s->hub_ok) std::memcpy(r_words, s->hub_rw32.data(), sizeof(uint32_t) * (size_t)B.d_r);   // column order
        else std::memcpy(r_words, s->rwords.data() + B.rbase, sizeof(uint32_t) * (size_t)B.d_r);
    }
    return ECUT_OK;
}

// Position and fermion sign of every canonical index of a spatial Hubbard
// cut, on the host's threads (the layout map of the device kernel).
static void hubsp_positions(const ecut_sectors *s, int64_t *pos, int8_t *sign) {
    const int nL = (int)s->lsites.size(), nR = (int)s->rsites.size();
    uint32_t lmask = 0, rmask = 0;
    for (int k : s->lsites) lmask |= 1u << k;
    for (int k : s->rsites) rmask |= 1u << k;
    const int64_t nd_words = (int64_t)binom(s->n_sites, s->n_dn);
    const int la0 = s->blocks.front().q_l, lb0 = s->blocks.front().q_l2;
    const int nb_b = s->blocks.back().q_l2 - lb0 + 1;
    auto compact = [](uint32_t w, uint32_t mask) {
        uint32_t out = 0;
        int k = 0;
        for (uint32_t m = mask; m; m &= m - 1u, ++k) out |= ((w >> __builtin_ctz(m)) & 1u) << k;
        return out;
    };
    auto work = [&](int64_t i0, int64_t i1) {
        for (int64_t i = i0; i < i1; ++i) {
            const uint32_t up = (uint32_t)colex_unrank(i / nd_words, s->n_up);
            const uint32_t dn = (uint32_t)colex_unrank(i % nd_words, s->n_dn);
            const uint32_t ul = compact(up, lmask), dl = compact(dn, lmask), ur = compact(up, rmask),
                           dr = compact(dn, rmask);
            const int a = __builtin_popcount(ul), b = __builtin_popcount(dl);
            const BlockDev &B = s->blocks[(size_t)((a - la0) * nb_b + (b - lb0))];
            const int64_t row = colex_rank(ul) * (int64_t)binom(nL, b) + colex_rank(dl);
            const int64_t col = colex_rank(ur) * (int64_t)binom(nR, s->n_dn - b) + colex_rank(dr);
            if (pos) pos[i] = B.offset + row * B.d_r + col;
            if (sign) {
                int par = __builtin_popcount(ur) * b;
                for (uint32_t m = lmask; m; m &= m - 1u) {
                    const uint32_t below = (m & (0u - m)) - 1u;
                    const int sb = __builtin_ctz(m);
                    if ((up >> sb) & 1u) par += __builtin_popcount(up & rmask & below);
                    if ((dn >> sb) & 1u) par += __builtin_popcount(dn & rmask & below);
                }
                sign[i] = (par & 1) ? -1 : 1;
            }
        }
    };
    const int64_t dim = s->dim;
    const unsigned hw = std::max(1u, std::min(64u, std::thread::hardware_concurrency()));
    const int64_t chunk = std::max<int64_t>(1 << 14, (dim + hw - 1) / hw);
    std::vector<std::thread> th;
    for (int64_t i0 = 0; i0 < dim; i0 += chunk) th.emplace_back(work, i0, std::min(dim, i0 + chunk));
    for (auto &t : th) t.join();
}

ecut_status ecut_canonical_signs(const ecut_sectors *s, int8_t *sign) {
    if (!s || !sign) return fail(ECUT_EINVAL, "null argument");
    if (s->hub_spatial) hubsp_positions(s, nullptr, sign);
    else std::fill(sign, sign + s->dim, (int8_t)1);
    return ECUT_OK;
}

ecut_status ecut_sectors_labels(const ecut_sectors *s, int32_t *labels) {
    if (!s || !labels) return fail(ECUT_EINVAL, "null argument");
    for (size_t b = 0; b < s->blocks.size(); ++b) {
        const BlockDev &B = s->blocks[b];
        labels[4 * b + 0] = B.q_l;
        labels[4 * b + 1] = B.q_l2;
        labels[4 * b + 2] = B.q_r;
        labels[4 * b + 3] = B.q_r2;
    }
    return ECUT_OK;
}

ecut_status ecut_canonical_positions(const ecut_sectors *s, int64_t *pos) {
    if (!s || !pos) return fail(ECUT_EINVAL, "null argument");
    if (s->hub_spatial) {
        hubsp_positions(s, pos, nullptr);
        return ECUT_OK;
    }
    if (s->kind == ECUT_HUBBARD) {
        // canonical index = up rank * d_R + down rank (up-major integer order)
        const int64_t dR = s->blocks[0].d_r;
        for (int64_t i = 0; i < s->dim; ++i) pos[i] = (i / dR) * dR + hub_column(s, i % dR);
        return ECUT_OK;
    }
    // Chunks of the canonical order on the host's threads: each chunk unranks
    // its first word and steps to the next word of the same popcount (the
    // smallest larger one: move the lowest movable set bit up by one and put
    // the set bits below it back at the bottom).
    const int qmin = s->blocks[0].q_l;
    const int64_t dim = s->dim;
    const unsigned hw = std::max(1u, std::min(64u, std::thread::hardware_concurrency()));
    const int64_t chunk = std::max<int64_t>(1 << 16, (dim + hw - 1) / hw);
    auto work = [&](int64_t i0, int64_t i1) {
        uint64_t w = colex_unrank(i0, s->n_up);
        for (int64_t i = i0; i < i1; ++i) {
            uint64_t l = 0, r = 0;
            for (size_t k = 0; k < s->lsites.size(); ++k) l |= ((w >> s->lsites[k]) & 1ull) << k;
            for (size_t k = 0; k < s->rsites.size(); ++k) r |= ((w >> s->rsites[k]) & 1ull) << k;
            const BlockDev &B = s->blocks[__builtin_popcountll(l) - qmin];
            pos[i] = B.offset + colex_rank(l) * B.d_r + colex_rank(r);
            if (w != 0 && i + 1 < i1) {
                const int t = __builtin_ctzll(w);                  // lowest set bit
                const int run = __builtin_ctzll(~(w >> t));        // set bits from there up
                w = (w & ~(((1ull << run) - 1) << t)) | (1ull << (t + run)) | ((1ull << (run - 1)) - 1);
            }
        }
    };
    std::vector<std::thread> th;
    for (int64_t i0 = 0; i0 < dim; i0 += chunk) th.emplace_back(work, i0, std::min(dim, i0 + chunk));
    for (auto &t : th) t.join();
    return ECUT_OK;
}

static ecut_status check_dev(const ecut_sectors *s) {
    if (!s) return fail(ECUT_EINVAL, "null handle");
    if (!s->on_device) return fail(ECUT_EINVAL, "handle was built with ECUT_BUILD_HOST_ONLY");
    int cur = -1;
    hipGetDevice(&cur);
    if (cur != s->device) return fail(ECUT_EINVAL, "handle lives on another device");
    return ECUT_OK;
}

static HubSpPerm hubsp_perm(const ecut_sectors *s, const uint64_t *binom_d) {
    HubSpPerm A{};
    A.blocks = s->prob.blocks;
    A.binom = binom_d;
    A.dim = s->dim;
    A.n_dn_words = (int64_t)binom(s->n_sites, s->n_dn);
    for (int k : s->lsites) A.lmask |= 1u << k;
    for (int k : s->rsites) A.rmask |= 1u << k;
    A.n_up = s->n_up;
    A.n_dn = s->n_dn;
    A.nL = (int32_t)s->lsites.size();
    A.nR = (int32_t)s->rsites.size();
    A.la0 = s->blocks.front().q_l;
    A.lb0 = s->blocks.front().q_l2;
    A.nb_b = s->blocks.back().q_l2 - A.lb0 + 1;
    return A;
}

static ecut_status permute(const ecut_sectors *s, const double *in, double *out, bool to_bip, void *stream) {
    ecut_status st = check_dev(s);
    if (st != ECUT_OK) return st;
    if (!in || !out) return fail(ECUT_EINVAL, "null vector");
    if (in == out) return fail(ECUT_EINVAL, "in and out must differ");
    hipStream_t hs = (hipStream_t)stream;
    hipError_t e;
    if (s->hub_spatial) {
        const uint64_t *bt = nullptr;
        st = device_res(nullptr, &bt, nullptr);
        if (st != ECUT_OK) return st;
        e = launch_perm_hubsp(hubsp_perm(s, bt), in, out, to_bip, hs);
    } else if (s->kind == ECUT_HUBBARD && s->hub_ok) {
        e = launch_perm_cols(s->prob.hub.col_of_rank, s->blocks[0].d_l, s->blocks[0].d_r, in, out, to_bip, hs);
    } else if (s->kind == ECUT_HUBBARD) {
        e = hipMemcpyAsync(out, in, sizeof(double) * (size_t)s->dim, hipMemcpyDeviceToDevice, hs);
    } else {
        const uint64_t *bt = nullptr;
        st = device_res(nullptr, &bt, nullptr);
        if (st != ECUT_OK) return st;
        e = launch_perm(s, bt, s->prob.blocks, in, out, to_bip, hs);
    }
    if (e != hipSuccess) return hip_fail(e, to_bip ? "ecut_import" : "ecut_export");
    return ECUT_OK;
}

ecut_status ecut_apply_cdag(const ecut_sectors *src, const ecut_sectors *dst, int32_t site, int32_t spin,
                            int32_t dagger, const double *x_d, double *y_d, void *stream) {
    ecut_status st = check_dev(src);
    if (st == ECUT_OK) st = check_dev(dst);
    if (st != ECUT_OK) return st;
    if (!x_d || !y_d || (const double *)y_d == x_d) return fail(ECUT_EINVAL, "null or overlapping vectors");
    if (src->kind != ECUT_HUBBARD || dst->kind != ECUT_HUBBARD || src->cut_kind != ECUT_CUT_UPDN ||
        dst->cut_kind != ECUT_CUT_UPDN)
        return fail(ECUT_EUNSUPPORTED, "c+ / c is built for Hubbard sectors with the up/down cut");
    if (src->n_sites != dst->n_sites) return fail(ECUT_EINVAL, "the two sectors belong to lattices of different size");
    if (site < 0 || site >= src->n_sites || spin < 0 || spin > 1) return fail(ECUT_EINVAL, "site or spin out of range");
    const int d = dagger ? 1 : -1;
    const int want_up = src->n_up + (spin == 0 ? d : 0), want_dn = src->n_dn + (spin == 1 ? d : 0);
    if (dst->n_up != want_up || dst->n_dn != want_dn)
        return fail(ECUT_EINVAL, "the destination sector must hold the source's particles with one more (c+) or one "
                                 "fewer (c) of the given spin");
    const uint64_t *bt = nullptr;
    st = device_res(nullptr, &bt, nullptr);
    if (st != ECUT_OK) return st;
    CdagArgs A{};
    A.x = x_d;
    A.y = y_d;
    A.dim = dst->dim;
    A.dR_dst = dst->blocks[0].d_r;
    A.dR_src = src->blocks[0].d_r;
    A.dst_lwords = dst->prob.lwords;
    A.dst_rwords = dst->hub_ok ? dst->prob.hub.rwords32 : dst->prob.rwords;
    A.src_col_of_rank = src->hub_ok ? src->prob.hub.col_of_rank : nullptr;
    A.binom = bt;
    A.site = site;
    A.spin = spin;
    A.dagger = dagger ? 1 : 0;
    if (A.dim == 0) return ECUT_OK;
    const hipError_t e = launch_cdag(A, (hipStream_t)stream);
    if (e != hipSuccess) return hip_fail(e, "kernel launch (apply_cdag)");
    return ECUT_OK;
}

ecut_status ecut_import(const ecut_sectors *s, const double *canon_d, double *bip_d, void *stream) {
    return permute(s, canon_d, bip_d, true, stream);
}

ecut_status ecut_export(const ecut_sectors *s, const double *bip_d, double *canon_d, void *stream) {
    return permute(s, bip_d, canon_d, false, stream);
}

ecut_status ecut_apply_H(const ecut_sectors *s, const double *psi_d, double *y_d, void *stream) {
    ecut_status st = check_dev(s);
    if (st != ECUT_OK) return st;
    if (!psi_d || !y_d) return fail(ECUT_EINVAL, "null vector");
    if (psi_d == y_d) return fail(ECUT_EINVAL, "psi and y must not overlap");
    ProblemDev P = s->prob;
    P.x = psi_d;
    P.y = y_d;
    P.z = nullptr;
    P.xscale = 1.0;
    P.zcoef = 0.0;
    P.partials = nullptr;
    return launch_apply(s, P, (hipStream_t)stream);
}

ecut_status ecut_apply_H_batch(int32_t n, const ecut_sectors *const *s, const double *const *psi_d,
                               double *const *y_d, void *stream) {
    BatchPlan pl;
    ecut_status st = make_batch_plan(n, s, psi_d, y_d, pl);
    if (st != ECUT_OK || n == 0) return st;
    // a descriptor buffer whose previous batch has been copied (a ring of a
    // few per thread, so the call waits only when all of them are in flight)
    static thread_local Staging ring[4];
    static thread_local int next = 0;
    Staging *S = nullptr;
    for (int k = 0; k < 4 && !S; ++k) {
        Staging &c = ring[(next + k) % 4];
        if (!c.pending || hipEventQuery(c.ev) == hipSuccess) S = &c;
    }
    if (!S) S = &ring[next % 4];   // every buffer busy: the oldest use is waited for
    next = (int)(S - ring + 1) % 4;
    if (!pl.buf.empty()) {
        st = S->reserve(pl.buf.size());
        if (st == ECUT_OK) st = S->wait();
        if (st != ECUT_OK) return st;
        std::memcpy(S->host, pl.buf.data(), pl.buf.size());
        hipError_t e = hipMemcpyAsync(S->dev, S->host, pl.buf.size(), hipMemcpyHostToDevice, (hipStream_t)stream);
        if (e != hipSuccess) return hip_fail(e, "hipMemcpyAsync(batch descriptors)");
    }
    st = launch_batch_plan(pl, S->dev, (hipStream_t)stream);
    if (st != ECUT_OK) return st;
    if (!pl.buf.empty()) {
        hipError_t e = hipEventRecord(S->ev, (hipStream_t)stream);
        if (e != hipSuccess) return hip_fail(e, "hipEventRecord");
        S->pending = true;
    }
    return ECUT_OK;
}

}  // extern "C"
