// Per-precision handle of libflood: device allocation and layout, the batched
// step scheduler (HIP graphs + double-buffered completion poll), the particle
// filter cycle, ledger/field access, snapshots and kernel timing.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <vector>

#include "flood_internal.h"
#include "flood_runtime.h"
#include "flood_validate.h"

static_assert(flood::kMaxSections == flood::kMaxSectionsAbi, "one limit on sections");
#include "flood_tune.h"

namespace flood {

#define HIPCHK(expr)                                                              \
    do {                                                                          \
        hipError_t e_ = (expr);                                                   \
        if (e_ != hipSuccess) {                                                   \
            err = std::string(#expr) + " failed: " + hipGetErrorString(e_);       \
            return FLOOD_EHIP;                                                    \
        }                                                                         \
    } while (0)

#define CHK(expr)                           \
    do {                                    \
        flood_status s_ = (expr);           \
        if (s_ != FLOOD_OK) return s_;      \
    } while (0)

template <typename T> struct Impl : ImplBase {
    using HB = typename HBits<T>::type;

    struct Cat {
        int ny = 0, nx = 0, N = 0, n_chunks = 0, tile_rows = 4, cpb = 1, march_rows = 32;
        double dx = 0;
        flood_params p{};
        std::vector<double> rain;
        double* d_rain = nullptr;
        int edge_kind[4] = {0, 0, 0, 0};
        double edge_slope[4] = {0, 0, 0, 0};
        CatchDev<T> dev{};
        size_t state_elems = 0, strip_w = 0, strip_n = 0;
        T* peak_tmp = nullptr;    // resampling scratch of the running maximum
        int n_classes = 0;        // land cover: 0 none
        double rain_cells = 0.0;  // rain-receiving cell count (land cover: sum of runoff coefficients)
        // inflow hydrographs
        int n_series = 0;
        double* d_inflow_q = nullptr;
        std::vector<int8_t> h_inflow_id;   // host copy of dev.inflow_id (empty: no inflow link)
        double wq[kMaxSeries] = {0, 0, 0, 0};
        // streamflow sections (configuration, not state: not in snapshots)
        int n_sec = 0;
        int32_t* d_sec_offs = nullptr;
        int32_t* d_sec_code = nullptr;
        int32_t* d_sec_index = nullptr;
        size_t sec_cap = 0;
    };

    hipStream_t st = nullptr;
    hipStream_t own_stream = nullptr;  // created when the caller passes the null stream
    int mi = 1;
    int variant = 1;          // 1 tiled step kernel; mi == 1: 2 row march, 3 vectorised row march
    int march_seg = 2;        // members per wavefront of the row-marching kernel
    int march_order = 1;      // wavefront order of the row-marching kernel
    int march_narrow = -1;    // strips of one cell a lane in the vectorised row march: as measured, -1 by rule
    int forced_order = -1;    // >= 0: the only order the tuner tries
    int march_bands = 0;      // order 4: bands of rows of strips (multiple of 8); 0: from the L2 size
    int march_nt = 1;         // non-temporal state streams in the vectorised row-marching kernel
    bool nt_forced = false;
    int total_waves = 0;      // waves of one row-marching launch
    int n_catch = 0, n_total = 0;
    std::vector<Cat> cats;
    std::vector<void*> allocs;

    double *t = nullptr, *s = nullptr, *mu = nullptr, *logw = nullptr, *vrain = nullptr, *vout = nullptr,
           *vclamp = nullptr;
    int64_t* steps = nullptr;
    int64_t* step_lim = nullptr;   // per-member step limit of the current flood_step_n call
    // step log opened by flood_log_steps: [n_total][log_cap] lengths and end times
    double *dtlog = nullptr, *telog = nullptr;
    int64_t* log_n = nullptr;
    int32_t log_cap = 0;
    double *clsn = nullptr, *drain = nullptr, *vdrain = nullptr;   // land cover per member; drained volume
    double* vin = nullptr;    // inflow volume per member
    bool any_land = false;
    bool any_inflow = false;
    // land cover and inflow links exist in the vectorised row-march kernel only
    bool vector_only() const { return any_land || any_inflow; }
    int32_t *par = nullptr, *fault = nullptr, *status = nullptr;
    HB* hbins = nullptr;
    MemberStep<T>* ms = nullptr;
    double* d_tend = nullptr;
    int32_t* d_count = nullptr;
    double* h_tend = nullptr;      // pinned
    int32_t* h_count = nullptr;    // pinned [2 slots][4]: a batch's counts
    int32_t* d_hcount = nullptr;   // the same in the device's view
    int32_t* h_cnt3 = nullptr;     // pinned [2 slots][4]: the adjoint forward's batch counts
    int last_adj_groups = 0, last_adj_group_size = 0, last_adj_segments = 0;
    hipEvent_t ev[2] = {nullptr, nullptr};

    // particle filter scratch
    double *d_y = nullptr, *d_obs = nullptr, *d_sigma = nullptr, *d_beta = nullptr, *d_neff = nullptr;
    int32_t *d_grc = nullptr, *d_anc = nullptr, *d_src = nullptr, *d_dst = nullptr, *d_flag = nullptr;
    int max_gauges = 0;
    double* d_stage = nullptr;     // field staging, max over catchments of (ny+1)*(nx+1) doubles
    size_t stage_elems = 0;
    // Results leave through a pinned block that the kernels write straight into: the
    // pages of a caller's array are then touched by the CPU, while the GPU fills the
    // next slot, instead of being pinned for a copy of their own (8.4 MB: 170 us over the
    // link and 270 us on the CPU, overlapped, against 490 us after the kernel).
    static constexpr int kOutSlots = 3;
    static constexpr size_t kOutElems = (size_t)1 << 18;   // doubles a slot (2 MiB)
    double* h_out = nullptr;       // pinned [kOutSlots][kOutElems]
    double* d_hout = nullptr;      // its device address
    hipEvent_t ev_out[kOutSlots] = {};

    // captured batches of G steps (and of kShort, for the end of a call)
    hipGraph_t graph[2] = {nullptr, nullptr};
    hipGraphExec_t gexec[2] = {nullptr, nullptr};
    int G = 16;
    static constexpr int kShort = 4;
    bool use_graph = true;

    // second copies for steps that plan themselves (see StepPlan), and that plan's catchments
    double *t2 = nullptr, *dt_last = nullptr;
    int64_t* steps2 = nullptr;
    int32_t *par2 = nullptr, *fault2 = nullptr;
    HB* hbins4 = nullptr;            // copies 1 to 3 of the depth-maximum bins
    PlanCatch* d_pc = nullptr;

    // kernel timing
    bool timing_on = false;      // per-launch events (graph capture off while on)
    bool timing_batch = false;   // events around each batch of G steps (graph path kept)
    std::vector<int32_t> tev_steps;   // step launches between each pair of events
    std::vector<hipEvent_t> tev;
    size_t tev_used = 0;
    double t_ms = 0.0;
    int64_t t_launches = 0;

    StepLaunch<T> SL{};
    PlanLaunch<T> PL{};

    // Adjoint scratch kept on the handle between flood_adjoint calls: the tape,
    // its clamp flags, the two adjoint copies, the Manning accumulators and the
    // checkpoints (up to half the device memory that was free).  Allocating and
    // freeing that much per call costs seconds once the memory has been used and
    // freed before.  Released by adjoint_release and the destructor.
    struct Scratch {
        void* p = nullptr;
        size_t bytes = 0;
    };
    Scratch adj_tape, adj_clamp, adj_lam, adj_nacc;
    std::vector<Scratch> adj_ckpt;
    Scratch adj_row;            // one member's row of a state array, for reordering members
    int32_t* d_order = nullptr; // [kMaxMembers + 1]: a member order and a set flag

    size_t adj_held() const {
        size_t b = adj_tape.bytes + adj_clamp.bytes + adj_lam.bytes + adj_nacc.bytes;
        for (const Scratch& c : adj_ckpt) b += c.bytes;
        return b;
    }

    // at least `bytes` in b: the held block if it is large enough, else a new one
    flood_status adj_reserve(Scratch& b, size_t bytes, std::string& err) {
        bytes = std::max<size_t>(bytes, 16);
        if (b.p && b.bytes >= bytes) return FLOOD_OK;
        if (b.p) {
            HIPCHK(hipStreamSynchronize(st));
            (void)hipFree(b.p);
            b.p = nullptr;
            b.bytes = 0;
        }
        if (hipMalloc(&b.p, bytes) != hipSuccess) {
            (void)hipGetLastError();
            b.p = nullptr;
            err = "hipMalloc of " + std::to_string(bytes) + " bytes failed in flood_adjoint";
            return FLOOD_ENOMEM;
        }
        b.bytes = bytes;
        return FLOOD_OK;
    }

    void adj_free_all() {
        (void)hipStreamSynchronize(st);
        for (Scratch* b : {&adj_tape, &adj_clamp, &adj_lam, &adj_nacc, &adj_row})
            if (b->p) (void)hipFree(b->p);
        for (Scratch& c : adj_ckpt)
            if (c.p) (void)hipFree(c.p);
        adj_tape = adj_clamp = adj_lam = adj_nacc = adj_row = Scratch{};
        adj_ckpt.clear();
    }

    // Reorder the members of catchment c (members in planes): slot i takes the member
    // held in slot order[i], with everything that belongs to it (its state, edge
    // strips, running maximum, outflow accumulators, depth-maximum bins, time,
    // parameters, weight, ledger, copy index, fault flag).  Rows of the large arrays
    // move along the cycles of the order through one row of staging.  Of the two
    // state copies only the one holding the member's state moves (into the same copy
    // of its new slot, whose copy index moves with it); the other is the next step's
    // output and holds nothing.
    flood_status reorder_members(int c, const std::vector<int32_t>& order, std::string& err) {
        Cat& C = cats[c];
        const int N = C.N, off = C.dev.member_off;
        const size_t ncell = (size_t)C.ny * C.nx, nb = 2 * ((size_t)C.nx + C.ny);
        struct Rows {
            void* base[2];   // the two state copies, or one array (base[1] null)
            size_t bytes;    // per member
        };
        std::vector<Rows> rows;
        rows.push_back({{C.dev.h[0], C.dev.h[1]}, ncell * sizeof(T)});
        rows.push_back({{C.dev.qx[0], C.dev.qx[1]}, ncell * sizeof(T)});
        rows.push_back({{C.dev.qy[0], C.dev.qy[1]}, ncell * sizeof(T)});
        rows.push_back({{C.dev.qw[0], C.dev.qw[1]}, (size_t)C.ny * sizeof(T)});
        rows.push_back({{C.dev.qn[0], C.dev.qn[1]}, (size_t)C.nx * sizeof(T)});
        if (C.dev.peak) rows.push_back({{C.dev.peak, nullptr}, ncell * sizeof(T)});
        rows.push_back({{C.dev.out_acc, nullptr}, nb * sizeof(double)});
        if (C.dev.drain_acc) rows.push_back({{C.dev.drain_acc, nullptr}, (size_t)kBins * sizeof(double)});
        CHK(adj_reserve(adj_row, ncell * sizeof(T) > nb * sizeof(double) ? ncell * sizeof(T) : nb * sizeof(double), err));
        // the state copy of each slot's member before the move
        std::vector<int32_t> hp(N);
        HIPCHK(hipMemcpyAsync(hp.data(), par + off, (size_t)N * sizeof(int32_t), hipMemcpyDeviceToHost, st));
        HIPCHK(hipStreamSynchronize(st));
        auto row = [&](const Rows& r, int i, int slot_of_member) {
            const int k = r.base[1] ? hp[slot_of_member] : 0;
            return static_cast<char*>(r.base[k]) + (size_t)i * r.bytes;
        };
        std::vector<char> seen(N, 0);
        for (int i0 = 0; i0 < N; ++i0) {
            if (seen[i0] || order[i0] == i0) {
                seen[i0] = 1;
                continue;
            }
            for (const Rows& r : rows) {
                HIPCHK(hipMemcpyAsync(adj_row.p, row(r, i0, i0), r.bytes, hipMemcpyDeviceToDevice, st));
                int i = i0;
                while (order[i] != i0) {
                    HIPCHK(hipMemcpyAsync(row(r, i, order[i]), row(r, order[i], order[i]), r.bytes,
                                          hipMemcpyDeviceToDevice, st));
                    i = order[i];
                }
                HIPCHK(hipMemcpyAsync(row(r, i, i0), adj_row.p, r.bytes, hipMemcpyDeviceToDevice, st));
            }
            for (int i = i0; !seen[i]; i = order[i]) seen[i] = 1;
        }
        // per-member scalars through the host
        HIPCHK(hipStreamSynchronize(st));
        auto scal = [&](void* base, size_t bytes) -> flood_status {
            std::vector<char> a((size_t)N * bytes), b((size_t)N * bytes);
            char* p = static_cast<char*>(base) + (size_t)off * bytes;
            HIPCHK(hipMemcpy(a.data(), p, a.size(), hipMemcpyDeviceToHost));
            for (int i = 0; i < N; ++i) std::memcpy(&b[(size_t)i * bytes], &a[(size_t)order[i] * bytes], bytes);
            HIPCHK(hipMemcpy(p, b.data(), b.size(), hipMemcpyHostToDevice));
            return FLOOD_OK;
        };
        for (double* a : {t, s, mu, logw, vrain, vout, vclamp, drain, vdrain, vin}) CHK(scal(a, sizeof(double)));
        CHK(scal(steps, sizeof(int64_t)));
        CHK(scal(clsn, kMaxClasses * sizeof(double)));
        CHK(scal(par, sizeof(int32_t)));
        CHK(scal(fault, sizeof(int32_t)));
        // depth-maximum bins: slot i's maximum is member order[i]'s
        if (!d_order) CHK(dalloc(&d_order, (size_t)kMaxMembers + 1, err));
        std::vector<int32_t> ho(order);
        ho.push_back(1);
        HIPCHK(hipMemcpy(d_order, ho.data(), ho.size() * sizeof(int32_t), hipMemcpyHostToDevice));
        launch_permute_bins<HB>(off, N, n_total, hbins, d_order, d_order + N, st);
        HIPCHK(hipGetLastError());
        HIPCHK(hipStreamSynchronize(st));
        return FLOOD_OK;
    }

    void get_adjoint_info(int32_t* groups, int32_t* group_size, int32_t* segments) const override {
        if (groups) *groups = last_adj_groups;
        if (group_size) *group_size = last_adj_group_size;
        if (segments) *segments = last_adj_segments;
    }

    flood_status adjoint_release(std::string& err) override {
        (void)err;
        adj_free_all();
        return FLOOD_OK;
    }

    ~Impl() override {
        (void)hipStreamSynchronize(st);
        adj_free_all();
        invalidate_graph();
        for (auto e : ev)
            if (e) (void)hipEventDestroy(e);
        for (auto e : tev) (void)hipEventDestroy(e);
        for (auto e : ev_out)
            if (e) (void)hipEventDestroy(e);
        if (h_out) (void)hipHostFree(h_out);
        for (void* p : allocs) (void)hipFree(p);
        if (dtlog) (void)hipFree(dtlog);
        if (telog) (void)hipFree(telog);
        if (h_tend) (void)hipHostFree(h_tend);
        if (h_count) (void)hipHostFree(h_count);
        if (h_cnt3) (void)hipHostFree(h_cnt3);
        if (snap.p) (void)hipFree(snap.p);
        if (own_stream) (void)hipStreamDestroy(own_stream);
    }

    template <typename X> flood_status dalloc(X** p, size_t n, std::string& err) {
        if (n == 0) n = 1;
        hipError_t e = hipMalloc((void**)p, n * sizeof(X));
        if (e != hipSuccess) {
            *p = nullptr;
            err = "hipMalloc of " + std::to_string(n * sizeof(X)) + " bytes failed: " + hipGetErrorString(e);
            (void)hipGetLastError();
            return e == hipErrorOutOfMemory ? FLOOD_ENOMEM : FLOOD_EHIP;
        }
        allocs.push_back((void*)*p);
        return FLOOD_OK;
    }

    static int ilog2(int v) {
        int l = 0;
        while ((1 << l) < v) ++l;
        return l;
    }

    // Wavefronts that a step over the members of a catchment takes in strips of whole
    // vectors, two rows tall, and whether strips of one cell a lane are the better ones:
    // where those do not fill the chip's 1024 SIMDs, the four times (FP64: twice) as many
    // wavefronts are shorter chains of arithmetic, and in FP32 no lanes idle beside a
    // narrow grid.  A step in FP32: 97 x 83 x 5 7.2 us from 10.5, 128 x 128 x 4 7.2 from 9.1, 512 x
    // 512 x 2 9.9 from 12.5, 256 x 256 x 16 13.4 from 12.7; in FP64 128 x 128 x 4 7.6 from 9.4,
    // 256 x 256 x 4 10.2 from 10.2.  By rule where nothing is measured; else both compete
    // (narrow_competes), but for small FP32 ensembles (below).
    static size_t wide_pairs(int ny, int nx, int members) {
        const int w = 64 * march_vec<T>();
        return (size_t)((nx + w - 1) / w) * ((ny + 1) / 2) * members;
    }
    static bool narrow_pays(size_t pairs) { return pairs < (sizeof(T) == 4 ? 1024 : 512); }
    bool narrow_ok() const { return mi == 1 && !any_land && !any_inflow; }
    // FP32 ensembles of up to 2^20 member cells: always in narrow strips, whose clamp ledger
    // adds in double as that of the tiled kernel does, which stepped them before.  At the
    // top of that range wide strips are the faster ones (256 x 256 x 16, above), and passed
    // over all the same.
    bool small_fp32() const {
        size_t cells = 0;
        for (const Cat& c : cats) cells += (size_t)c.ny * c.nx * c.N;
        return sizeof(T) == 4 && cells <= (size_t)1 << 20;
    }
    bool adj_tiled = false;   // adjoints in the tiled form although the steps march
    // The rain-multiplier gradients of the two adjoint forms differ by some 1e-7 in FP32:
    // the tiled one sums tiles in single precision, the row march in double.  Handles
    // that name no kernel keep the form, and so the sums, of the step kernel that was
    // measured the fastest before ragged rows and narrow strips could march: the tiled one
    // up to 2^20 member cells, then the scalar march (tiled adjoints too) where strips of 256
    // cells leave more lanes idle than its strips of 62.  Of 190 shapes of 9,000 to 6 million
    // member cells timed, 185 fall on the side that the trial took.
    bool tiled_adjoint_by_shape() const {
        if (sizeof(T) != 4 || !narrow_ok()) return false;
        if (small_fp32()) return true;
        double wide = 0.0, slim = 0.0, cells = 0.0;
        bool long_rows = true;
        for (const Cat& c : cats) {
            const double rows = (double)c.ny * c.N;
            wide += rows * (256 * ((c.nx + 255) / 256));
            slim += rows * (62 * ((c.nx + 61) / 62));
            cells += rows * c.nx;
            long_rows = long_rows && c.nx > 256;
        }
        return wide > slim * (cells < 2.6e6 && long_rows ? 1.4 : cells < 4.2e6 ? 1.04 : 1.02);
    }

    // Rows that a lane's drained depth is summed over in single precision: 4 up to 4.5
    // million member cells, 8 beyond.  The sum once ended where a strip did; of 65 shapes of
    // 3.7 to 54 million member cells a free choice took strips of 4 rows at six of the nine up
    // to 4.5 million, at 12 of the 32 from there to 12.2 million and at none of the 24 beyond.
    // The drained volume is off by 0.8 to 1.3e-8 with 4 rows and by 1.9 to 2.4e-8 with 8
    // (against FP64 sums of the same depths).
    static constexpr double kDrainCells = 4.5e6;

    // tile / grouping geometry of every catchment and the launch descriptor
    void layout_launch() {
        int begin = 0, waves = 0;
        SL.n_catch = n_catch;
        SL.n_total = n_total;
        double all_cells = 0.0;
        for (const Cat& c : cats) all_cells += (double)c.ny * c.nx * c.N;
        SL.drain_rows = all_cells <= kDrainCells ? 4 : 8;
        size_t pairs = 0;
        for (const Cat& c : cats) pairs += wide_pairs(c.ny, c.nx, c.N);
        SL.narrow = variant == 3 && narrow_ok() &&
                    (small_fp32() || (march_narrow >= 0 ? march_narrow != 0 : narrow_pays(pairs)));
        for (int i = 0; i < n_catch; ++i) {
            Cat& c = cats[i];
            CatchDev<T>& d = c.dev;
            const int txc = std::max(1, kBlock / (mi * c.tile_rows));
            d.tx_log2 = ilog2(txc);
            const int ty = (kBlock / mi) >> d.tx_log2;
            d.tiles_x = (c.nx + txc - 1) / txc;
            d.tiles_y = (c.ny + ty - 1) / ty;
            d.chunks_per_group = std::max(1, std::min(c.cpb, c.n_chunks));
            d.groups = (c.n_chunks + d.chunks_per_group - 1) / d.chunks_per_group;
            d.n_blocks = d.tiles_x * d.tiles_y * d.groups;
            d.block_begin = begin;
            begin += d.n_blocks;
            d.march_rows = std::max(1, std::min(c.march_rows, c.ny));
            const int strip_w = variant != 3 ? 62 : SL.narrow ? 64 : 64 * march_vec<T>();
            d.strips_x = (c.nx + strip_w - 1) / strip_w;
            d.strips_xa = (c.nx + 62 * adj_vec<T>() - 1) / (62 * adj_vec<T>());
            d.strips_y = (c.ny + d.march_rows - 1) / d.march_rows;
            d.index = i;
            d.wave_begin = waves;
            {
                // order 4: enough bands that one band's bed and roughness (2 values
                // per cell) stay within about 1 MiB, a quarter of one XCD's L2,
                // while the units of the band pass through it
                int bands = march_bands;
                if (bands <= 0) {
                    const double shared_bytes = (double)c.ny * c.nx * 2.0 * sizeof(T);
                    bands = (int)std::ceil(shared_bytes / (1 << 20) / 8.0) * 8;
                }
                d.march_bands = std::max(8, std::min(bands, (d.strips_y + 7) / 8 * 8));
            }
            d.n_waves = march_waves(d.strips_x, d.strips_y, variant == 3 ? c.N : (c.N + march_seg - 1) / march_seg,
                                    march_order, d.march_bands);
            d.march_order = march_order;
            waves += d.n_waves;
            SL.c[i] = d;
        }
        SL.total_blocks = begin;
        total_waves = waves;
        if (!nt_forced) {
            // What a step reads and writes: where it fits the 256 MB last-level cache,
            // plain accesses leave the new state there for the next step (1024 x 1024 x 8,
            // 202 MB: 51 us a step against 57 us; 512 x 512 x 16: 34 against 39 us); beyond
            // it, accesses marked non-temporal are the faster ones (1024 x 1024 x 16, 403 MB:
            // 101 against 106 us; 2000 x 2000 x 96: 2.07 against 2.19 ms)
            double moved = 0.0;
            for (const Cat& c : cats) moved += (double)c.ny * c.nx * (6.0 * c.N + 2.0) * sizeof(T);
            march_nt = moved > 230e6 ? 1 : 0;
        }
        SL.ms = ms;
        SL.hbins = hbins;
        SL.vclamp = vclamp;
    }

    // One instantiation of the row march serves catchments with land cover or without: a
    // handle that holds both kinds steps them in two launches.
    void launch_marchv_kind(const StepLaunch<T>& L, bool land) {
        StepLaunch<T> K = L;
        int waves = 0;
        bool peak = false;
        K.n_catch = 0;
        for (int i = 0; i < L.n_catch; ++i) {
            if ((L.c[i].cls != nullptr) != land) continue;
            CatchDev<T>& d = K.c[K.n_catch++];
            d = L.c[i];
            d.wave_begin = waves;
            waves += d.n_waves;
            peak |= d.peak != nullptr;
        }
        if (K.n_catch == 0) return;
        launch_marchv<T>(K, march_nt,
                         (land ? 1 : 0) | (any_inflow ? 2 : 0) | (vector_ok() || K.narrow ? 0 : 4) |
                             (peak ? 8 : 0),
                         waves, st);
    }

    void launch_steps(const StepLaunch<T>& L) {
        if (variant == 3 && !L.recompute) {
            launch_marchv_kind(L, false);
            if (any_land) launch_marchv_kind(L, true);
        } else if (variant == 2 && !L.recompute) {
            launch_march<T>(L, march_seg, total_waves, st);
        } else {
            launch_step_mi<T>(mi, L, st);
        }
    }

    bool vector_ok() const {
        for (const Cat& c : cats)
            if (c.nx % march_vec<T>() != 0) return false;
        return mi == 1;
    }

    void invalidate_graph() {
        for (int k = 0; k < 2; ++k) {
            if (gexec[k]) (void)hipGraphExecDestroy(gexec[k]);
            if (graph[k]) (void)hipGraphDestroy(graph[k]);
            gexec[k] = nullptr;
            graph[k] = nullptr;
        }
    }

    // Whether the steps plan themselves: the row march, in batches of whole rounds of
    // four.  At every size: calls of flood_step over 512 x 512 x 16 8.9 -> 7.6 ms,
    // 1024 x 1024 x 16 with inflow 26.7 -> 22.7 ms, 1024 x 1024 x 32 91 -> 79 ms, and 2000 x
    // 2000 x 96, where the planning of 200,000 wavefronts is hidden behind their loads,
    // 310 -> 308 ms.
    bool self_planned() const { return variant == 3 && G % 4 == 0; }

    // step i of a batch
    void launch_one(int i) {
        if (!self_planned()) {
            launch_plan<T>(PL, st);
            launch_steps(SL);
            return;
        }
        StepLaunch<T> L = SL;
        StepPlan<T>& P = L.plan;
        HB* bins[4];
        for (int k = 0; k < 4; ++k) bins[k] = k ? hbins4 + (size_t)(k - 1) * kBins * n_total : hbins;
        const bool o = i & 1;
        P.pc = d_pc;
        P.t_end = d_tend;
        P.t_in = o ? t2 : t;
        P.t_out = o ? t : t2;
        P.steps_in = o ? steps2 : steps;
        P.steps_out = o ? steps : steps2;
        P.par_in = o ? par2 : par;
        P.par_out = o ? par : par2;
        P.fault_in = o ? fault2 : fault;
        P.fault_out = o ? fault : fault2;
        P.bins_in = bins[i & 3];
        P.bins_out = bins[(i + 1) & 3];
        P.bins_clear = bins[(i + 2) & 3];
        P.s = s;
        P.mu = mu;
        P.clsn = PL.clsn;
        P.drain = PL.drain;
        P.lim = step_lim;
        P.vrain = vrain;
        P.vin = vin;
        P.dt_last = dt_last;
        P.dtlog = dtlog;
        P.telog = telog;
        P.log_n = log_n;
        P.dtlog_cap = log_cap;
        P.status = status;
        launch_steps(L);
    }

    flood_status init(int nc, const flood_grid* grids, const flood_params* params, const int32_t* members,
                      const double* const* n_scale, const double* const* rain_mult, hipStream_t stream,
                      std::string& err) {
        st = stream;
        if (!st) {
            // A blocking stream stays ordered with the legacy null stream and, unlike it,
            // can be captured into a graph.
            HIPCHK(hipStreamCreate(&own_stream));
            st = own_stream;
        }
        n_catch = nc;
        if (const char* mb = std::getenv("FLOOD_MARCH_BANDS")) {
            const int v = std::atoi(mb);
            if (v >= 8 && v <= 1024) march_bands = v / 8 * 8;
        }
        if (const char* mo = std::getenv("FLOOD_MARCH_ORDER")) {   // restricts the tuner to one order
            march_order = std::min(4, std::max(0, std::atoi(mo)));
            forced_order = march_order;
        }
        if (const char* nt = std::getenv("FLOOD_MARCH_NT")) {
            march_nt = std::atoi(nt) ? 1 : 0;
            nt_forced = true;
        }
        const char* ng = std::getenv("FLOOD_NO_GRAPH");
        use_graph = !(ng && ng[0] == '1');
        if (const char* gs = std::getenv("FLOOD_GRAPH_STEPS")) {   // steps per captured batch
            const int v = std::atoi(gs);
            if (v >= 1 && v <= 4096) G = v;
        }
        cats.resize(nc);
        int off = 0;
        for (int i = 0; i < nc; ++i) {
            Cat& c = cats[i];
            c.ny = grids[i].ny;
            c.nx = grids[i].nx;
            c.dx = grids[i].dx;
            c.N = members[i];
            c.p = params[i];
            c.rain.assign(params[i].rain_rate, params[i].rain_rate + params[i].n_rain);
            for (int e = 0; e < 4; ++e) {
                c.edge_kind[e] = grids[i].edge_kind[e];
                c.edge_slope[e] = grids[i].edge_slope[e];
            }
            c.dev.member_off = off;
            off += c.N;
            max_gauges = std::max(max_gauges, 64);
            stage_elems = std::max(stage_elems, (size_t)(c.ny + 1) * (c.nx + 1));
            stage_elems = std::max(stage_elems, (size_t)c.N * 64);
            stage_elems = std::max(stage_elems, (size_t)std::max(c.N, kProdPad) + 16);   // weights, percentiles
        }
        n_total = off;

        // kernel configuration: explicit values, else the tuner's choice
        TuneKey key{};
        key.real_bytes = (int)sizeof(T);
        key.n_catch = nc;
        for (int i = 0; i < nc; ++i) {
            key.ny[i] = cats[i].ny;
            key.nx[i] = cats[i].nx;
            key.members[i] = cats[i].N;
            key.kind[i] = (grids[i].land_class && params[i].n_classes > 0 ? 1 : 0) | (params[i].n_inflow > 0 ? 2 : 0);
        }
        TuneChoice ch = tune_default(key);
        if (params[0].member_interleave) ch.mi = params[0].member_interleave;
        mi = ch.mi;
        variant = params[0].step_kernel ? params[0].step_kernel : ch.variant;
        march_seg = params[0].march_members ? params[0].march_members : ch.march_seg;
        // asked for by number, the vectorised kernel needs whole vectors in every row;
        // chosen by the library it takes any row length
        if (params[0].step_kernel == 3 && !vector_ok()) {
            err = "the vectorised kernel needs member_interleave 1 and nx a multiple of " +
                  std::to_string(march_vec<T>());
            return FLOOD_EINVAL;
        }
        if (mi != 1) variant = 1;
        // land cover runs on the vectorised row-march kernel only (per-member class
        // tables in scalar registers)
        any_land = false;
        any_inflow = false;
        for (int i = 0; i < nc; ++i) {
            any_land |= grids[i].land_class != nullptr && params[i].n_classes > 0;
            any_inflow |= params[i].n_inflow > 0;
        }
        if (any_land || any_inflow) {
            const char* what = any_land ? "land cover" : "inflow links";
            if (mi != 1 || !vector_ok()) {
                err = std::string(what) + " need member_interleave 1 and nx a multiple of " +
                      std::to_string(march_vec<T>());
                return FLOOD_EINVAL;
            }
            if (params[0].step_kernel == 1 || params[0].step_kernel == 2) {
                err = std::string(what) + " run on step kernel 3 only";
                return FLOOD_EINVAL;
            }
            variant = 3;
        }
        for (int i = 0; i < nc; ++i) {
            cats[i].tile_rows = params[i].tile_rows ? params[i].tile_rows : ch.tile_rows;
            cats[i].cpb = params[i].chunks_per_block ? params[i].chunks_per_block : ch.cpb;
            cats[i].march_rows = params[i].march_rows ? params[i].march_rows : ch.march_rows;
            while (cats[i].tile_rows * mi > kBlock) cats[i].tile_rows >>= 1;
        }

        // per-catchment device arrays
        for (int i = 0; i < nc; ++i) {
            Cat& c = cats[i];
            CatchDev<T>& d = c.dev;
            c.n_chunks = (c.N + mi - 1) / mi;
            const size_t ncell = (size_t)c.ny * c.nx;
            c.state_elems = (size_t)c.n_chunks * ncell * mi;
            c.strip_w = (size_t)c.n_chunks * c.ny * mi;
            c.strip_n = (size_t)c.n_chunks * c.nx * mi;
            d.ny = c.ny;
            d.nx = c.nx;
            d.n_members = c.N;
            d.n_chunks = c.n_chunks;
            d.dx = c.dx;
            d.hdry = (T)c.p.h_dry;
            d.g = (T)c.p.g;
            for (int e = 0; e < 4; ++e) {
                d.edge_open[e] = c.edge_kind[e] == FLOOD_EDGE_OPEN;
                d.edge_slope[e] = (T)c.edge_slope[e];
            }
            for (int k = 0; k < 2; ++k) {
                CHK(dalloc(&d.h[k], c.state_elems + kRowPad, err));
                CHK(dalloc(&d.qx[k], c.state_elems + kRowPad, err));
                CHK(dalloc(&d.qy[k], c.state_elems + kRowPad, err));
                CHK(dalloc(&d.qw[k], c.strip_w + kRowPad, err));
                CHK(dalloc(&d.qn[k], c.strip_n + kRowPad, err));
                HIPCHK(hipMemsetAsync(d.h[k], 0, c.state_elems * sizeof(T), st));
                HIPCHK(hipMemsetAsync(d.qx[k], 0, c.state_elems * sizeof(T), st));
                HIPCHK(hipMemsetAsync(d.qy[k], 0, c.state_elems * sizeof(T), st));
                HIPCHK(hipMemsetAsync(d.qw[k], 0, c.strip_w * sizeof(T), st));
                HIPCHK(hipMemsetAsync(d.qn[k], 0, c.strip_n * sizeof(T), st));
            }
            T* zz;
            T* nn;
            CHK(dalloc(&zz, ncell + kRowPad, err));
            CHK(dalloc(&nn, ncell + kRowPad, err));
            {
                std::vector<T> hz(ncell), hn(ncell);
                for (size_t j = 0; j < ncell; ++j) {
                    hz[j] = (T)grids[i].dem[j];
                    hn[j] = (T)grids[i].manning_n[j];
                }
                HIPCHK(hipMemcpyAsync(zz, hz.data(), ncell * sizeof(T), hipMemcpyHostToDevice, st));
                HIPCHK(hipMemcpyAsync(nn, hn.data(), ncell * sizeof(T), hipMemcpyHostToDevice, st));
                HIPCHK(hipStreamSynchronize(st));
            }
            d.z = zz;
            d.n = nn;
            // land cover: class map, runoff coefficients, draining classes
            c.n_classes = (grids[i].land_class && params[i].n_classes > 0) ? params[i].n_classes : 0;
            d.cls = nullptr;
            d.drain_acc = nullptr;
            d.drain_mask = 0;
            for (int k = 0; k < kMaxClasses; ++k) d.class_rc[k] = T(1);
            c.rain_cells = (double)ncell;
            if (c.n_classes) {
                uint8_t* dc;
                CHK(dalloc(&dc, ncell, err));
                HIPCHK(hipMemcpy(dc, grids[i].land_class, ncell, hipMemcpyHostToDevice));
                d.cls = dc;
                CHK(dalloc(&d.drain_acc, (size_t)c.N * kBins, err));
                HIPCHK(hipMemsetAsync(d.drain_acc, 0, (size_t)c.N * kBins * sizeof(double), st));
                for (int k = 0; k < c.n_classes; ++k) {
                    d.class_rc[k] = (T)params[i].class_runoff[k];
                    if (params[i].class_drain[k]) d.drain_mask |= 1 << k;
                }
                double rcs = 0.0;   // cell order, as the rain volume of the ledger is summed
                for (size_t j = 0; j < ncell; ++j) rcs += params[i].class_runoff[grids[i].land_class[j]];
                c.rain_cells = rcs;
            }
            // inflow links: series of each edge link in the out_acc order (N, S, W, E)
            d.inflow_id = nullptr;
            c.n_series = params[i].n_inflow > 0 ? params[i].n_series : 0;
            if (c.n_series) {
                const int nbl = 2 * (c.nx + c.ny);
                std::vector<int8_t> id(nbl, -1);
                for (int k = 0; k < kMaxSeries; ++k) c.wq[k] = 0.0;
                for (int k = 0; k < params[i].n_inflow; ++k) {
                    const int32_t* f = params[i].inflow + 3 * k;
                    const int e = f[0], pos = f[1];
                    const int at = e == 0 ? pos : e == 2 ? c.nx + pos : e == 3 ? 2 * c.nx + pos : 2 * c.nx + c.ny + pos;
                    id[at] = (int8_t)f[2];
                    c.wq[f[2]] += c.dx;
                }
                c.h_inflow_id = id;
                int8_t* did;
                CHK(dalloc(&did, (size_t)nbl, err));
                HIPCHK(hipMemcpy(did, id.data(), nbl, hipMemcpyHostToDevice));
                d.inflow_id = did;
                const size_t nq = (size_t)c.n_series * std::max(c.p.n_rain, 0);
                CHK(dalloc(&c.d_inflow_q, std::max<size_t>(nq, 1), err));
                if (nq) HIPCHK(hipMemcpy(c.d_inflow_q, params[i].inflow_q, nq * sizeof(double), hipMemcpyHostToDevice));
            }
            if (c.p.track_peak) {
                CHK(dalloc(&d.peak, c.state_elems + kRowPad, err));
                CHK(dalloc(&c.peak_tmp, c.state_elems, err));
                HIPCHK(hipMemsetAsync(d.peak, 0, c.state_elems * sizeof(T), st));
            } else {
                d.peak = nullptr;
            }
            const int nb = 2 * (c.nx + c.ny);
            CHK(dalloc(&d.out_acc, (size_t)c.N * nb, err));
            HIPCHK(hipMemsetAsync(d.out_acc, 0, (size_t)c.N * nb * sizeof(double), st));
            CHK(dalloc(&c.d_rain, std::max<size_t>(c.rain.size(), 1), err));
            if (!c.rain.empty())
                HIPCHK(hipMemcpyAsync(c.d_rain, c.rain.data(), c.rain.size() * sizeof(double), hipMemcpyHostToDevice,
                                      st));
        }

        // per-member arrays
        CHK(dalloc(&t, n_total, err));
        CHK(dalloc(&s, n_total, err));
        CHK(dalloc(&mu, n_total, err));
        CHK(dalloc(&logw, n_total, err));
        CHK(dalloc(&vrain, n_total, err));
        CHK(dalloc(&vout, n_total, err));
        CHK(dalloc(&vclamp, n_total, err));
        CHK(dalloc(&steps, n_total, err));
        CHK(dalloc(&step_lim, n_total, err));
        CHK(dalloc(&log_n, n_total, err));
        CHK(dalloc(&clsn, (size_t)n_total * kMaxClasses, err));
        CHK(dalloc(&drain, n_total, err));
        CHK(dalloc(&vdrain, n_total, err));
        CHK(dalloc(&vin, n_total, err));
        CHK(dalloc(&par, n_total, err));
        CHK(dalloc(&fault, n_total, err));
        CHK(dalloc(&status, 1, err));
        CHK(dalloc(&hbins, (size_t)kBins * n_total, err));
        CHK(dalloc(&hbins4, (size_t)3 * kBins * n_total, err));
        CHK(dalloc(&t2, n_total, err));
        CHK(dalloc(&dt_last, n_total, err));
        CHK(dalloc(&steps2, n_total, err));
        CHK(dalloc(&par2, n_total, err));
        CHK(dalloc(&fault2, n_total, err));
        CHK(dalloc(&d_pc, nc, err));
        CHK(dalloc(&ms, n_total, err));
        CHK(dalloc(&d_tend, 1, err));
        CHK(dalloc(&d_count, 3, err));
        {
            std::vector<double> hs(n_total), hm(n_total), hl(n_total), z0(n_total, 0.0);
            std::vector<double> hcn((size_t)n_total * kMaxClasses, 0.0), hdr(n_total, 0.0);
            for (int i = 0; i < nc; ++i) {
                const Cat& c = cats[i];
                for (int m = 0; m < c.N; ++m) {
                    const int g = c.dev.member_off + m;
                    hs[g] = (n_scale && n_scale[i] && !c.n_classes) ? n_scale[i][m] : 1.0;
                    hm[g] = (rain_mult && rain_mult[i]) ? rain_mult[i][m] : 1.0;
                    hl[g] = -std::log((double)c.N);
                    if (c.n_classes) {
                        for (int k = 0; k < c.n_classes; ++k)
                            hcn[(size_t)g * kMaxClasses + k] = params[i].member_class_n[(size_t)m * c.n_classes + k];
                        hdr[g] = params[i].member_drain ? params[i].member_drain[m] : 0.0;
                    }
                }
            }
            HIPCHK(hipMemcpy(clsn, hcn.data(), hcn.size() * sizeof(double), hipMemcpyHostToDevice));
            HIPCHK(hipMemcpy(drain, hdr.data(), n_total * sizeof(double), hipMemcpyHostToDevice));
            HIPCHK(hipMemcpy(s, hs.data(), n_total * sizeof(double), hipMemcpyHostToDevice));
            HIPCHK(hipMemcpy(mu, hm.data(), n_total * sizeof(double), hipMemcpyHostToDevice));
            HIPCHK(hipMemcpy(logw, hl.data(), n_total * sizeof(double), hipMemcpyHostToDevice));
            HIPCHK(hipMemcpy(t, z0.data(), n_total * sizeof(double), hipMemcpyHostToDevice));
        }
        HIPCHK(hipMemsetAsync(vrain, 0, n_total * sizeof(double), st));
        HIPCHK(hipMemsetAsync(vout, 0, n_total * sizeof(double), st));
        HIPCHK(hipMemsetAsync(vclamp, 0, n_total * sizeof(double), st));
        HIPCHK(hipMemsetAsync(vdrain, 0, n_total * sizeof(double), st));
        HIPCHK(hipMemsetAsync(vin, 0, n_total * sizeof(double), st));
        HIPCHK(hipMemsetAsync(steps, 0, n_total * sizeof(int64_t), st));
        HIPCHK(hipMemsetAsync(log_n, 0, n_total * sizeof(int64_t), st));
        launch_step_limit(n_total, steps, -1, step_lim, st);
        HIPCHK(hipMemsetAsync(par, 0, n_total * sizeof(int32_t), st));
        HIPCHK(hipMemsetAsync(fault, 0, n_total * sizeof(int32_t), st));
        HIPCHK(hipMemsetAsync(status, 0, sizeof(int32_t), st));
        HIPCHK(hipMemsetAsync(hbins, 0, (size_t)kBins * n_total * sizeof(HB), st));
        HIPCHK(hipMemsetAsync(hbins4, 0, (size_t)3 * kBins * n_total * sizeof(HB), st));
        HIPCHK(hipMemsetAsync(dt_last, 0, n_total * sizeof(double), st));
        HIPCHK(hipMemsetAsync(ms, 0, n_total * sizeof(MemberStep<T>), st));

        // scratch
        CHK(dalloc(&d_y, (size_t)kMaxMembers * 4096, err));
        CHK(dalloc(&d_obs, 4096, err));
        CHK(dalloc(&d_sigma, 4096, err));
        CHK(dalloc(&d_beta, kMaxMembers, err));
        CHK(dalloc(&d_neff, 1, err));
        CHK(dalloc(&d_grc, 2 * 4096, err));
        CHK(dalloc(&d_anc, kMaxMembers, err));
        CHK(dalloc(&d_src, kMaxMembers, err));
        CHK(dalloc(&d_dst, kMaxMembers, err));
        CHK(dalloc(&d_flag, 1, err));
        CHK(dalloc(&d_stage, stage_elems, err));
        HIPCHK(hipHostMalloc((void**)&h_tend, sizeof(double), hipHostMallocDefault));
        HIPCHK(hipHostMalloc((void**)&h_count, 8 * sizeof(int32_t), hipHostMallocDefault));
        std::memset(h_count, 0, 8 * sizeof(int32_t));
        HIPCHK(hipHostGetDevicePointer((void**)&d_hcount, h_count, 0));
        HIPCHK(hipHostMalloc((void**)&h_out, kOutSlots * kOutElems * sizeof(double), hipHostMallocDefault));
        HIPCHK(hipHostGetDevicePointer((void**)&d_hout, h_out, 0));
        for (auto& e : ev_out) HIPCHK(hipEventCreateWithFlags(&e, hipEventDisableTiming));
        HIPCHK(hipEventCreateWithFlags(&ev[0], hipEventDisableTiming));
        HIPCHK(hipEventCreateWithFlags(&ev[1], hipEventDisableTiming));

        // initial depths
        for (int i = 0; i < nc; ++i) {
            if (!grids[i].h0) continue;
            const Cat& c = cats[i];
            const size_t ncell = (size_t)c.ny * c.nx;
            std::vector<double> h0(ncell);
            for (size_t j = 0; j < ncell; ++j) h0[j] = (double)grids[i].h0[j];
            HIPCHK(hipMemcpyAsync(d_stage, h0.data(), ncell * sizeof(double), hipMemcpyHostToDevice, st));
            for (int m = 0; m < c.N; ++m) {
                launch_set_field<T>(mi, c.dev, m, nullptr, FLOOD_FIELD_H, d_stage, st);
                if (c.dev.peak) launch_set_field<T>(mi, c.dev, m, nullptr, FLOOD_FIELD_PEAK, d_stage, st);
            }
            HIPCHK(hipStreamSynchronize(st));
        }

        // planner descriptor
        PL.n_catch = nc;
        PL.n_total = n_total;
        for (int i = 0; i < nc; ++i) {
            const Cat& c = cats[i];
            PlanCatch& pc = PL.c[i];
            pc.member_off = c.dev.member_off;
            pc.n_members = c.N;
            pc.n_rain = c.p.n_rain;
            pc.rain = c.d_rain;
            pc.rain_interval = c.p.rain_interval;
            pc.alpha = c.p.cfl_alpha;
            pc.hdry = c.p.h_dry;
            pc.dt_cap = c.p.dt_cap;
            pc.dt_fixed = c.p.dt_fixed;
            pc.g = c.p.g;
            pc.dx = c.dx;
            pc.ncells = c.rain_cells;
            pc.inflow_q = c.d_inflow_q;
            pc.n_series = c.n_series;
            for (int k = 0; k < kMaxSeries; ++k) pc.wq[k] = c.wq[k];
        }
        HIPCHK(hipMemcpy(d_pc, PL.c, nc * sizeof(PlanCatch), hipMemcpyHostToDevice));
        PL.t_end = d_tend;
        PL.dt_last = dt_last;
        PL.t = t;
        PL.s = s;
        PL.mu = mu;
        PL.par = par;
        PL.steps = steps;
        PL.fault = fault;
        PL.status = status;
        PL.vrain = vrain;
        PL.vin = vin;
        PL.hbins = hbins;
        PL.ms = ms;
        PL.dtlog = nullptr;
        PL.telog = nullptr;
        PL.log_n = log_n;
        PL.dtlog_cap = 0;
        PL.step_lim = step_lim;
        PL.clsn = any_land ? clsn : nullptr;
        PL.drain = any_land ? drain : nullptr;
        PL.m_begin = 0;
        PL.m_end = n_total;
        PL.ms_log = nullptr;
        PL.rdt_log = nullptr;
        PL.tag_log = nullptr;
        PL.any_log = nullptr;
        PL.tag_value = -1;
        SL.recompute = 0;
        SL.clamp_out = nullptr;
        SL.plan = StepPlan<T>{};
        layout_launch();
        for (int i = 0; i < nc; ++i) launch_hmax_init<T>(mi, cats[i].dev, par, hbins, n_total, st);
        HIPCHK(hipGetLastError());
        HIPCHK(hipStreamSynchronize(st));

        // measured choice of tile rows / chunks per workgroup when not given
        bool autotune = false;
        for (int i = 0; i < nc; ++i)
            autotune |= (params[i].tile_rows == 0 || params[i].chunks_per_block == 0 ||
                         (mi == 1 && (params[i].step_kernel == 0 || params[i].march_rows == 0 ||
                                      params[i].march_members == 0)));
        if (autotune && tune_enabled()) CHK(autotune_geometry(key, params, err));
        return FLOOD_OK;
    }

    // time candidate (tile rows, chunks per workgroup) pairs on the real state
    // without advancing it: each trial launches one step kernel that reads the
    // current copy and writes the other copy, which is dead until the next step.
    flood_status autotune_geometry(const TuneKey& key, const flood_params* params, std::string& err) {
        adj_tiled = params[0].step_kernel == 0 && tiled_adjoint_by_shape();
        TuneChoice cached;
        if (tune_lookup(key, mi, params[0].step_kernel, cached)) {
            if (!params[0].step_kernel && mi == 1 && !vector_only()) variant = cached.variant;
            if (!params[0].march_members) march_seg = cached.march_seg;
            march_order = forced_order >= 0 ? forced_order : cached.march_order;
            march_narrow = cached.march_narrow;
            for (int i = 0; i < n_catch; ++i) {
                if (!params[i].tile_rows) cats[i].tile_rows = cached.tile_rows;
                if (!params[i].chunks_per_block) cats[i].cpb = cached.cpb;
                if (!params[i].march_rows)
                    cats[i].march_rows = (i < 8 && cached.march_rows_c[i] > 0) ? cached.march_rows_c[i]
                                                                               : cached.march_rows;
            }
            layout_launch();
            return FLOOD_OK;
        }
        // a synthetic step plan: every member active with a representative step
        std::vector<MemberStep<T>> hms(n_total);
        for (int i = 0; i < n_catch; ++i)
            for (int m = 0; m < cats[i].N; ++m) {
                MemberStep<T>& x = hms[cats[i].dev.member_off + m];
                const double dt = 0.5, dx = cats[i].dx, g = cats[i].p.g;
                x.dtdx = (T)(dt / dx);
                x.gdtdx = (T)(g * dt / dx);
                x.gdt = (T)(g * dt);
                x.s2dt = (T)dt;
                x.capf = (T)(dx / (4 * dt));
                x.rinc = (T)1e-5;
                x.dxdt = dx * dt;
                x.active = 1;
                x.parity = 0;
            }
        std::vector<MemberStep<T>> saved(n_total);
        std::vector<double> saved_clamp(n_total);
        HIPCHK(hipMemcpy(saved.data(), ms, n_total * sizeof(MemberStep<T>), hipMemcpyDeviceToHost));
        HIPCHK(hipMemcpy(saved_clamp.data(), vclamp, n_total * sizeof(double), hipMemcpyDeviceToHost));
        std::vector<int32_t> hpar(n_total);
        HIPCHK(hipMemcpy(hpar.data(), par, n_total * sizeof(int32_t), hipMemcpyDeviceToHost));
        for (int m = 0; m < n_total; ++m) hms[m].parity = hpar[m];
        HIPCHK(hipMemcpy(ms, hms.data(), n_total * sizeof(MemberStep<T>), hipMemcpyHostToDevice));
        std::vector<std::vector<HB>> bins_saved(1);
        bins_saved[0].resize((size_t)kBins * n_total);
        HIPCHK(hipMemcpy(bins_saved[0].data(), hbins, bins_saved[0].size() * sizeof(HB), hipMemcpyDeviceToHost));
        // the outflow and drainage accumulators are touched by trial steps: save, restore after
        std::vector<std::vector<double>> acc_saved(n_catch), dacc_saved(n_catch);
        for (int i = 0; i < n_catch; ++i) {
            const size_t n = (size_t)cats[i].N * 2 * (cats[i].nx + cats[i].ny);
            acc_saved[i].resize(n);
            HIPCHK(hipMemcpy(acc_saved[i].data(), cats[i].dev.out_acc, n * sizeof(double), hipMemcpyDeviceToHost));
            if (cats[i].dev.drain_acc) {
                dacc_saved[i].resize((size_t)cats[i].N * kBins);
                HIPCHK(hipMemcpy(dacc_saved[i].data(), cats[i].dev.drain_acc, dacc_saved[i].size() * sizeof(double),
                                 hipMemcpyDeviceToHost));
            }
        }
        // trial launches must not touch the running maxima
        std::vector<T*> peaks(n_catch);
        for (int i = 0; i < n_catch; ++i) {
            peaks[i] = cats[i].dev.peak;
            cats[i].dev.peak = nullptr;
        }
        hipEvent_t a, b;
        HIPCHK(hipEventCreate(&a));
        HIPCHK(hipEventCreate(&b));
        int max_chunks = 1;
        for (int i = 0; i < n_catch; ++i) max_chunks = std::max(max_chunks, cats[i].n_chunks);
        std::vector<int> cpbs;
        for (int v = 1; v < max_chunks; v *= 2) cpbs.push_back(v);
        cpbs.push_back(max_chunks);
        struct Cand {
            int variant, rows, cpb, mrows, seg, order, narrow = 0;
        };
        std::vector<Cand> cands;
        // Left to itself the library steps members in planes with the vectorised row
        // march, of any row length: no other kernel was faster at any size, on the
        // smallest grids 7 us a step against 8.4 and a planner launch for the tiled one.
        // That serves interleaved members, and it and the scalar march whoever asks for
        // them by number.
        const bool want1 = !vector_only() && (params[0].step_kernel == 1 || mi != 1);
        const bool want2 = !vector_only() && mi == 1 && params[0].step_kernel == 2;
        const bool want3 = mi == 1 && (params[0].step_kernel == 0 || params[0].step_kernel == 3);
        if (want1)
            for (int r : {1, 2, 4, 8})
                for (int cp : cpbs)
                    if (r * mi <= kBlock) cands.push_back({1, r, cp, cats[0].march_rows, march_seg, march_order});
        if (want2) {
            std::vector<int> segs;
            if (params[0].march_members)
                segs.push_back(params[0].march_members);
            else
                segs = {1, 2, 4, 8};
            for (int od : {0, 1, 2, 3, 4})
                for (int sg : segs)
                    if (forced_order < 0 || od == forced_order)
                    for (int mr : {8, 16, 32, 64, 128})
                        cands.push_back({2, cats[0].tile_rows, cats[0].cpb, mr, sg, od});
        }
        if (want3) {
            const std::vector<int> heights = strip_heights(any_land ? SL.drain_rows : 0, false);
            for (int od : {0, 1, 2, 3, 4})
                if ((forced_order < 0 || od == forced_order) && !(narrow_ok() && small_fp32()))
                    for (int mr : heights) cands.push_back({3, cats[0].tile_rows, cats[0].cpb, mr, 1, od, 0});
            if (narrow_ok() && narrow_competes(key))
                for (int od : {0, 1, 2, 3, 4})
                    if (forced_order < 0 || od == forced_order)
                        for (int mr : {1, 2, 4, 8, 16}) cands.push_back({3, cats[0].tile_rows, cats[0].cpb, mr, 1, od, 1});
        }
        Cand bc = cands.empty()
                      ? Cand{variant, cats[0].tile_rows, cats[0].cpb, cats[0].march_rows, march_seg, march_order}
                      : cands[0];
        // two rounds: every candidate timed once (after a warm-up launch), then the
        // candidates within 8 % of the fastest timed again as the minimum of five
        // launches, which separates geometries a few per cent apart
        auto time_cand = [&](const Cand& cd, int reps, float* out) -> flood_status {
            variant = cd.variant;
            march_seg = cd.seg;
            march_order = cd.order;
            march_narrow = cd.narrow;
            for (int i = 0; i < n_catch; ++i) {
                if (!params[i].tile_rows) cats[i].tile_rows = cd.rows;
                if (!params[i].chunks_per_block) cats[i].cpb = cd.cpb;
                if (!params[i].march_rows) cats[i].march_rows = cd.mrows;
            }
            layout_launch();
            launch_steps(SL);  // warm-up
            float best_rep = 1e30f;
            for (int rep = 0; rep < reps; ++rep) {
                HIPCHK(hipEventRecord(a, st));
                launch_steps(SL);
                HIPCHK(hipEventRecord(b, st));
                HIPCHK(hipEventSynchronize(b));
                float ms_el = 0;
                HIPCHK(hipEventElapsedTime(&ms_el, a, b));
                best_rep = std::min(best_rep, ms_el);
            }
            // kernels whose steps do not plan themselves need a planner launch before each
            // (4-5 us for few members, with a launch gap of 4 us), which the trial leaves out
            if (!self_planned()) best_rep += 8e-3f;
            *out = best_rep;
            return FLOOD_OK;
        };
        std::vector<float> first(cands.size(), 1e30f);
        float best1 = 1e30f;
        for (size_t i = 0; i < cands.size(); ++i) {
            CHK(time_cand(cands[i], 1, &first[i]));
            best1 = std::min(best1, first[i]);
        }
        float best = 1e30f;
        std::vector<std::pair<float, size_t>> round2;
        for (size_t i = 0; i < cands.size(); ++i) {
            if (first[i] > 1.08f * best1) continue;
            float t5;
            CHK(time_cand(cands[i], 5, &t5));
            round2.push_back({t5, i});
            if (t5 < best) {
                best = t5;
                bc = cands[i];
            }
        }
        // trial launches step every member, but in an assimilation window members
        // finish at different times; order 4 keeps the XCDs evenly loaded then, so
        // it is taken when it is within 1 % of the fastest
        if (bc.variant >= 2 && bc.order != 4) {
            const float best_all = best;
            int pick = -1;
            float pick_t = 1e30f;
            for (const auto& r : round2) {
                const Cand& cd = cands[r.second];
                if (cd.variant == bc.variant && cd.narrow == bc.narrow && cd.order == 4 && cd.seg == bc.seg && r.first <= 1.01f * best_all &&
                    r.first < pick_t) {
                    pick = (int)r.second;
                    pick_t = r.first;
                }
            }
            if (pick >= 0) {
                bc = cands[pick];
                best = pick_t;
            }
        }
        // geometries of the same kernel and order within 1 % of the fastest are
        // indistinguishable by timing; the tallest strip re-reads the fewest halo rows
        for (const auto& r : round2) {
            const Cand& cd = cands[r.second];
            if (r.first <= 1.01f * best && cd.variant == bc.variant && cd.order == bc.order && cd.variant >= 2 &&
                cd.narrow == bc.narrow && cd.seg == bc.seg && cd.mrows > bc.mrows)
                bc = cd;
        }
        variant = bc.variant;
        march_seg = bc.seg;
        march_order = bc.order;
        march_narrow = bc.narrow;
        for (int i = 0; i < n_catch; ++i) {
            if (!params[i].tile_rows) cats[i].tile_rows = bc.rows;
            if (!params[i].chunks_per_block) cats[i].cpb = bc.cpb;
            if (!params[i].march_rows) cats[i].march_rows = bc.mrows;
        }
        layout_launch();
        // catchments of different sizes in one launch: each one's rows per strip
        // refined in turn (the others held), timing the whole batched launch; a
        // change is kept only when it is more than 1 % faster
        if (n_catch > 1 && variant >= 2) {
            const std::vector<int> rows_set = variant == 3 ? strip_heights(any_land ? SL.drain_rows : 0, true)
                                                           : std::vector<int>{8, 16, 32, 64, 128};
            auto time_layout = [&](float* out) -> flood_status {
                layout_launch();
                launch_steps(SL);   // warm-up
                float b5 = 1e30f;
                for (int rep = 0; rep < 5; ++rep) {
                    HIPCHK(hipEventRecord(a, st));
                    launch_steps(SL);
                    HIPCHK(hipEventRecord(b, st));
                    HIPCHK(hipEventSynchronize(b));
                    float el = 0;
                    HIPCHK(hipEventElapsedTime(&el, a, b));
                    b5 = std::min(b5, el);
                }
                *out = b5;
                return FLOOD_OK;
            };
            float t_cur;
            CHK(time_layout(&t_cur));
            for (int i = 0; i < n_catch; ++i) {
                if (params[i].march_rows) continue;
                const int keep = cats[i].march_rows;
                int best_r = keep;
                for (int mr : rows_set) {
                    if (mr == keep) continue;
                    cats[i].march_rows = mr;
                    float t;
                    CHK(time_layout(&t));
                    if (t < 0.99f * t_cur) {
                        t_cur = t;
                        best_r = mr;
                    }
                }
                cats[i].march_rows = best_r;
            }
            layout_launch();
        }
        (void)hipEventDestroy(a);
        (void)hipEventDestroy(b);
        // the launch descriptors are built from the catchments again once the running
        // maxima are back (trial launches ran without them)
        for (int i = 0; i < n_catch; ++i) cats[i].dev.peak = peaks[i];
        layout_launch();
        HIPCHK(hipMemcpy(ms, saved.data(), n_total * sizeof(MemberStep<T>), hipMemcpyHostToDevice));
        HIPCHK(hipMemcpy(vclamp, saved_clamp.data(), n_total * sizeof(double), hipMemcpyHostToDevice));
        HIPCHK(hipMemcpy(hbins, bins_saved[0].data(), bins_saved[0].size() * sizeof(HB), hipMemcpyHostToDevice));
        for (int i = 0; i < n_catch; ++i) {
            HIPCHK(hipMemcpy(cats[i].dev.out_acc, acc_saved[i].data(), acc_saved[i].size() * sizeof(double),
                             hipMemcpyHostToDevice));
            if (cats[i].dev.drain_acc)
                HIPCHK(hipMemcpy(cats[i].dev.drain_acc, dacc_saved[i].data(), dacc_saved[i].size() * sizeof(double),
                                 hipMemcpyHostToDevice));
        }
        TuneChoice c;
        c.mi = mi;
        c.tile_rows = bc.rows;
        c.cpb = bc.cpb;
        c.variant = bc.variant;
        c.march_rows = bc.mrows;
        c.march_seg = bc.seg;
        c.march_order = bc.order;
        c.march_narrow = bc.narrow;
        for (int i = 0; i < n_catch && i < 8; ++i) c.march_rows_c[i] = cats[i].march_rows;
        // only a search over the full candidate set is remembered: a handle that
        // pinned part of the geometry measured a subset, whose best need not be
        // the best for a later handle of the same shape
        bool free_search = forced_order < 0;
        for (int i = 0; i < n_catch; ++i)
            free_search &= params[i].tile_rows == 0 && params[i].chunks_per_block == 0 &&
                           params[i].step_kernel == 0 && params[i].march_rows == 0 &&
                           params[i].march_members == 0;
        if (free_search) tune_store(key, c);
        return FLOOD_OK;
    }

    // ---------------------------------------------------------------------
    // stepping
    // ---------------------------------------------------------------------
    flood_status ensure_graph(std::string& err) {
        if (!use_graph || gexec[0] || timing_on) return FLOOD_OK;
        for (int k = 0; k < 2; ++k) {
            const int n = k ? kShort : G;
            if (k && (G % kShort || G == kShort)) break;   // batches of G only
            hipError_t e = hipStreamBeginCapture(st, hipStreamCaptureModeThreadLocal);
            if (e != hipSuccess) {
                (void)hipGetLastError();
                invalidate_graph();
                use_graph = false;
                return FLOOD_OK;
            }
            for (int i = 0; i < n; ++i) launch_one(i);
            e = hipStreamEndCapture(st, &graph[k]);
            if (e == hipSuccess && graph[k]) e = hipGraphInstantiate(&gexec[k], graph[k], nullptr, nullptr, 0);
            if (e != hipSuccess || !gexec[k]) {
                (void)hipGetLastError();
                gexec[k] = nullptr;
                invalidate_graph();
                use_graph = false;
                return FLOOD_OK;
            }
        }
        (void)err;
        return FLOOD_OK;
    }

    flood_status next_event_pair(int32_t launches) {
        while (tev.size() < tev_used + 2) {
            hipEvent_t e;
            if (hipEventCreate(&e) != hipSuccess) return FLOOD_EHIP;
            tev.push_back(e);
        }
        if (tev_steps.size() < tev_used / 2 + 1) tev_steps.resize(tev_used / 2 + 1);
        tev_steps[tev_used / 2] = launches;
        return FLOOD_OK;
    }

    // n steps of every member (G, or kShort where there is a graph for it); the counts
    // after them go straight into the pinned block (no copy command per batch)
    flood_status launch_batch(int slot, int n, std::string& err) {
        if (timing_batch) {
            if (next_event_pair(n)) { err = "hipEventCreate failed"; return FLOOD_EHIP; }
            HIPCHK(hipEventRecord(tev[tev_used], st));
        }
        hipGraphExec_t ge = timing_on ? nullptr : gexec[n == G ? 0 : 1];
        if (ge) {
            HIPCHK(hipGraphLaunch(ge, st));
        } else {
            for (int i = 0; i < n; ++i) {
                if (timing_on) {
                    if (next_event_pair(1)) { err = "hipEventCreate failed"; return FLOOD_EHIP; }
                    if (!self_planned()) launch_plan<T>(PL, st);
                    HIPCHK(hipEventRecord(tev[tev_used], st));
                    if (self_planned())
                        launch_one(i);
                    else
                        launch_steps(SL);
                    HIPCHK(hipEventRecord(tev[tev_used + 1], st));
                    tev_used += 2;
                } else {
                    launch_one(i);
                }
            }
        }
        if (timing_batch) {
            HIPCHK(hipEventRecord(tev[tev_used + 1], st));
            tev_used += 2;
        }
        launch_count_active(n_total, t, fault, d_tend, status, steps, step_lim, dt_last, d_hcount + 4 * slot, st);
        HIPCHK(hipGetLastError());
        HIPCHK(hipEventRecord(ev[slot], st));
        return FLOOD_OK;
    }

    flood_status step(double t_end, int64_t max_steps, std::string& err) override {
        CHK(ensure_graph(err));
        // a status word is only read for batches launched by this call
        std::memset(h_count, 0, 8 * sizeof(int32_t));
        *h_tend = t_end;
        HIPCHK(hipMemcpyAsync(d_tend, h_tend, sizeof(double), hipMemcpyHostToDevice, st));
        launch_step_limit(n_total, steps, max_steps, step_lim, st);
        // Up to two batches are in flight, so that the device does not wait for the host.
        // The first runs alone (a call that needs one batch launches no more); after it
        // the steps still needed are estimated from the step lengths, and what is
        // launched beyond them is kept to a short batch.  (Two full batches past the end
        // were 20 of 224 launches of a 600-s call on 128 x 128 cells.)
        const int small = (gexec[1] || (!gexec[0] && self_planned() && G > kShort)) ? kShort : G;
        int64_t launched = 0;
        const int64_t most = (int64_t)50000000;
        int64_t pending[2] = {0, 0};      // steps of the batch in each slot, 0: none in flight
        int slot = 0;                     // the slot to wait for next
        auto put = [&](int sl, int n) -> flood_status {
            CHK(launch_batch(sl, n, err));
            pending[sl] = n;
            launched += n;
            return FLOOD_OK;
        };
        CHK(put(0, max_steps > 0 && max_steps <= small ? small : G));
        for (;;) {
            HIPCHK(hipEventSynchronize(ev[slot]));
            pending[slot] = 0;
            if (h_count[4 * slot] == 0) break;
            if (launched > most) {
                err = "step limit exceeded before every member reached t_end";
                return FLOOD_ESTATE;
            }
            // steps needed after the batch just finished, less those already on their way
            int64_t need = (int64_t)h_count[4 * slot + 2] - pending[slot ^ 1];
            if (pending[slot ^ 1] == 0) {
                CHK(put(slot, need > small ? G : small));
                need -= pending[slot];
                if (need > 0) CHK(put(slot ^ 1, need > small ? G : small));
            } else {
                if (need > 0) CHK(put(slot, need > small ? G : small));
                slot ^= 1;
            }
        }
        HIPCHK(hipStreamSynchronize(st));
        if (timing_on || timing_batch) {
            for (size_t i = 0; i < tev_used; i += 2) {
                float el = 0;
                HIPCHK(hipEventElapsedTime(&el, tev[i], tev[i + 1]));
                t_ms += el;
                t_launches += tev_steps[i / 2];
            }
            tev_used = 0;
        }
        // status words of the batches this call launched
        const int stat = h_count[1] | h_count[4 + 1];
        if (stat) {
            err = "a member's depth became non-finite or too large to advance its clock; it was frozen";
            return FLOOD_ENUMERIC;
        }
        return FLOOD_OK;
    }

    // ---------------------------------------------------------------------
    // particle filter
    // ---------------------------------------------------------------------
    flood_status check_catch(int c, std::string& err) const {
        if (c < 0 || c >= n_catch) {
            err = "catchment index out of range";
            return FLOOD_EINVAL;
        }
        return FLOOD_OK;
    }

    flood_status common_time(int c, double* tc, std::string& err) {
        const Cat& C = cats[c];
        std::vector<double> ht(C.N);
        std::vector<int32_t> hf(C.N);
        HIPCHK(hipStreamSynchronize(st));
        HIPCHK(hipMemcpy(ht.data(), t + C.dev.member_off, C.N * sizeof(double), hipMemcpyDeviceToHost));
        HIPCHK(hipMemcpy(hf.data(), fault + C.dev.member_off, C.N * sizeof(int32_t), hipMemcpyDeviceToHost));
        for (int m = 0; m < C.N; ++m) {
            if (hf[m]) {
                err = "a member of this catchment is faulted";
                return FLOOD_ESTATE;
            }
            if (ht[m] != ht[0]) {
                err = "members are not at a common time";
                return FLOOD_ESTATE;
            }
        }
        *tc = ht[0];
        return FLOOD_OK;
    }

    flood_status assimilate(int c, int K, const int32_t* grc, const double* obs, const double* sigma,
                            int with_sections, double alpha, double neff_frac, double u0, const double* beta,
                            double* neff_out, int32_t* anc_out, int32_t* res_out, std::string& err) override {
        CHK(check_catch(c, err));
        const Cat& C = cats[c];
        // observation vector: K gauge depths, then the registered sections' discharges
        const int S = with_sections ? C.n_sec : 0;
        const int KT = K + S;
        CHK(check_observations(C.ny, C.nx, C.N, K, S, grc, obs, sigma, alpha, neff_frac, u0, beta, err));
        double tc;
        CHK(common_time(c, &tc, err));
        const int off = C.dev.member_off;
        const int nb = 2 * (C.nx + C.ny);
        launch_flush_outflow(C.N, nb, C.dev.out_acc, vout + off, st);
        if (C.dev.drain_acc) launch_flush_outflow(C.N, kBins, C.dev.drain_acc, vdrain + off, st);
        if (K > 0) HIPCHK(hipMemcpyAsync(d_grc, grc, 2 * K * sizeof(int32_t), hipMemcpyHostToDevice, st));
        if (KT > 0) {
            HIPCHK(hipMemcpyAsync(d_obs, obs, KT * sizeof(double), hipMemcpyHostToDevice, st));
            HIPCHK(hipMemcpyAsync(d_sigma, sigma, KT * sizeof(double), hipMemcpyHostToDevice, st));
        }
        if (beta) HIPCHK(hipMemcpyAsync(d_beta, beta, C.N * sizeof(double), hipMemcpyHostToDevice, st));
        launch_gauges<T>(mi, C.dev, par, K, d_grc, d_y, KT, st);
        launch_sections<T>(mi, C.dev, par, S, C.d_sec_offs, C.d_sec_code, C.d_sec_index, d_y, KT, K, st);
        PfArgs a{};
        a.N = C.N;
        a.K = KT;
        a.alpha = alpha;
        a.vin = vin + off;
        a.y = d_y;
        a.d = d_obs;
        a.sigma = d_sigma;
        a.neff_frac = neff_frac;
        a.u0 = u0;
        a.beta = beta ? d_beta : nullptr;
        a.logw = logw + off;
        a.t = t + off;
        a.s = s + off;
        a.mu = mu + off;
        a.vrain = vrain + off;
        a.vout = vout + off;
        a.vclamp = vclamp + off;
        a.steps = steps + off;
        a.par = par + off;
        a.src_par = d_src;
        a.dst_par = d_dst;
        a.anc = d_anc;
        a.neff = d_neff;
        a.flag = d_flag;
        a.clsn = C.n_classes ? clsn + (size_t)off * kMaxClasses : nullptr;
        a.drain = C.n_classes ? drain + off : nullptr;
        a.vdrain = vdrain + off;
        launch_pf(a, st);
        launch_permute<T>(mi, C.dev, d_anc, d_src, d_dst, d_flag, st);
        if (C.dev.peak) launch_permute_peak<T>(mi, C.dev, d_anc, d_flag, C.peak_tmp, st);
        launch_permute_bins<HB>(off, C.N, n_total, hbins, d_anc, d_flag, st);
        HIPCHK(hipGetLastError());
        double hn = 0;
        int32_t hflag = 0;
        HIPCHK(hipMemcpyAsync(&hn, d_neff, sizeof(double), hipMemcpyDeviceToHost, st));
        HIPCHK(hipMemcpyAsync(&hflag, d_flag, sizeof(int32_t), hipMemcpyDeviceToHost, st));
        if (anc_out) HIPCHK(hipMemcpyAsync(anc_out, d_anc, C.N * sizeof(int32_t), hipMemcpyDeviceToHost, st));
        HIPCHK(hipStreamSynchronize(st));
        if (neff_out) *neff_out = hn;
        if (res_out) *res_out = hflag;
        return FLOOD_OK;
    }

    // streamflow sections (Sec. 4.4): links in the host layouts, converted to
    // the device arrays (east / south edge links are the last cell's qx / qy;
    // west / north edge links live in the edge strips)
    flood_status set_sections(int c, int n, const int32_t* count, const int32_t* links, std::string& err) override {
        CHK(check_catch(c, err));
        Cat& C = cats[c];
        std::vector<int32_t> offs, code, index;
        CHK(parse_sections(C.ny, C.nx, n, count, links, offs, code, index, err));
        const size_t L = code.size();
        if (L > C.sec_cap) {
            CHK(dalloc(&C.d_sec_code, L, err));
            CHK(dalloc(&C.d_sec_index, L, err));
            C.sec_cap = L;
        }
        if (!C.d_sec_offs) CHK(dalloc(&C.d_sec_offs, (size_t)kMaxSections + 1, err));
        HIPCHK(hipMemcpyAsync(C.d_sec_offs, offs.data(), offs.size() * sizeof(int32_t), hipMemcpyHostToDevice, st));
        if (L) {
            HIPCHK(hipMemcpyAsync(C.d_sec_code, code.data(), L * sizeof(int32_t), hipMemcpyHostToDevice, st));
            HIPCHK(hipMemcpyAsync(C.d_sec_index, index.data(), L * sizeof(int32_t), hipMemcpyHostToDevice, st));
        }
        HIPCHK(hipStreamSynchronize(st));
        C.n_sec = n;
        return FLOOD_OK;
    }

    flood_status get_sections(int c, double* q_out, std::string& err) override {
        CHK(check_catch(c, err));
        const Cat& C = cats[c];
        if (!q_out) { err = "q_out is NULL"; return FLOOD_EINVAL; }
        if (C.n_sec == 0) { err = "no section is registered for this catchment"; return FLOOD_ESTATE; }
        launch_sections<T>(mi, C.dev, par, C.n_sec, C.d_sec_offs, C.d_sec_code, C.d_sec_index, d_y, C.n_sec, 0, st);
        HIPCHK(hipGetLastError());
        HIPCHK(hipMemcpyAsync(q_out, d_y, (size_t)C.N * C.n_sec * sizeof(double), hipMemcpyDeviceToHost, st));
        HIPCHK(hipStreamSynchronize(st));
        return FLOOD_OK;
    }

    flood_status adjoint(int c, double t_end, double sample_dt, int K, const int32_t* grc, const double* obs,
                         int ckpt_every, double* loss_out, double* grad_n_out, double* grad_mult_out,
                         std::string& err) override;

    // ---------------------------------------------------------------------
    // fields, parameters, ledger
    // ---------------------------------------------------------------------
    flood_status member_parity(int g, int* p, std::string& err) {
        int32_t v = 0;
        HIPCHK(hipStreamSynchronize(st));
        HIPCHK(hipMemcpy(&v, par + g, sizeof(int32_t), hipMemcpyDeviceToHost));
        *p = v;
        return FLOOD_OK;
    }

    static size_t field_size(const Cat& C, int which) {
        return (which == FLOOD_FIELD_H || which == FLOOD_FIELD_PEAK) ? (size_t)C.ny * C.nx
               : which == FLOOD_FIELD_QX                             ? (size_t)C.ny * (C.nx + 1)
                                                                     : (size_t)(C.ny + 1) * C.nx;
    }

    flood_status get_field(int c, int m, int which, double* out, std::string& err) override {
        CHK(check_catch(c, err));
        const Cat& C = cats[c];
        if (m < 0 || m >= C.N) { err = "member index out of range"; return FLOOD_EINVAL; }
        if (which < 0 || which > 3) { err = "which must be H, QX, QY or PEAK"; return FLOOD_EINVAL; }
        if (!out) { err = "host_out is NULL"; return FLOOD_EINVAL; }
        if (which == FLOOD_FIELD_PEAK && !C.dev.peak) {
            err = "the running maximum is kept only by handles created with track_peak = 1";
            return FLOOD_ESTATE;
        }
        return stage_out(
            field_size(C, which), kOutElems,
            [&](size_t e0, size_t n, double* dst) { launch_get_field<T>(mi, C.dev, m, par, which, e0, n, dst, st); },
            [&](size_t e0, size_t n, const double* src) { std::memcpy(out + e0, src, n * sizeof(double)); }, err);
    }

    // n elements in pieces of at most `per` through the pinned slots: fill(first, count,
    // dst) launches what writes a piece, drain(first, count, src) copies it out while
    // the GPU is on the next ones.  Ends synchronised.
    template <typename Fill, typename Drain>
    flood_status stage_out(size_t n, size_t per, Fill fill, Drain drain, std::string& err) {
        const size_t pieces = (n + per - 1) / per;
        hipError_t e = hipSuccess;
        for (size_t i = 0; i < pieces + kOutSlots && e == hipSuccess; ++i) {
            if (i >= (size_t)kOutSlots) {
                const size_t j = i - kOutSlots;
                if (j >= pieces) break;
                e = hipEventSynchronize(ev_out[j % kOutSlots]);
                if (e != hipSuccess) break;
                drain(j * per, std::min(per, n - j * per), h_out + (j % kOutSlots) * kOutElems);
            }
            if (i >= pieces) continue;
            fill(i * per, std::min(per, n - i * per), d_hout + (i % kOutSlots) * kOutElems);
            e = hipGetLastError();
            if (e == hipSuccess) e = hipEventRecord(ev_out[i % kOutSlots], st);
        }
        if (e != hipSuccess) {
            (void)hipStreamSynchronize(st);
            err = std::string(hipGetErrorString(e)) + " while results were copied out";
            return FLOOD_EHIP;
        }
        return FLOOD_OK;
    }

    // wet/dry decision of every link of one member for its next step
    flood_status get_wet_mask(int c, int m, uint8_t* wx, uint8_t* wy, std::string& err) override {
        CHK(check_catch(c, err));
        const Cat& C = cats[c];
        if (m < 0 || m >= C.N) { err = "member index out of range"; return FLOOD_EINVAL; }
        if (!wx || !wy) { err = "wet_x and wet_y are required"; return FLOOD_EINVAL; }
        int p;
        CHK(member_parity(C.dev.member_off + m, &p, err));
        const size_t nxl = (size_t)C.ny * (C.nx + 1), nyl = (size_t)(C.ny + 1) * C.nx;
        uint8_t* d = reinterpret_cast<uint8_t*>(d_stage);   // stage_elems doubles >= nxl + nyl bytes
        launch_wetmask<T>(mi, C.dev, m, p, d, d + nxl, st);
        HIPCHK(hipGetLastError());
        HIPCHK(hipMemcpyAsync(wx, d, nxl, hipMemcpyDeviceToHost, st));
        HIPCHK(hipMemcpyAsync(wy, d + nxl, nyl, hipMemcpyDeviceToHost, st));
        HIPCHK(hipStreamSynchronize(st));
        return FLOOD_OK;
    }

    // step log: capacity entries per member, counters restarted; 0 closes it
    flood_status log_steps(int32_t cap, std::string& err) override {
        HIPCHK(hipStreamSynchronize(st));
        if (dtlog) (void)hipFree(dtlog);
        if (telog) (void)hipFree(telog);
        dtlog = telog = nullptr;
        log_cap = 0;
        if (cap > 0) {
            const size_t n = (size_t)n_total * cap * sizeof(double);
            if (hipMalloc((void**)&dtlog, n) != hipSuccess || hipMalloc((void**)&telog, n) != hipSuccess) {
                (void)hipGetLastError();
                if (dtlog) (void)hipFree(dtlog);
                dtlog = nullptr;
                telog = nullptr;
                err = "hipMalloc of the step log failed";
                PL.dtlog = PL.telog = nullptr;
                PL.dtlog_cap = 0;
                invalidate_graph();
                return FLOOD_ENOMEM;
            }
            log_cap = cap;
        }
        HIPCHK(hipMemsetAsync(log_n, 0, n_total * sizeof(int64_t), st));
        PL.dtlog = dtlog;
        PL.telog = telog;
        PL.dtlog_cap = log_cap;
        invalidate_graph();   // the captured planner carries the log pointers
        HIPCHK(hipStreamSynchronize(st));
        return FLOOD_OK;
    }

    flood_status get_step_log(int c, double* dt_out, double* te_out, int64_t* count_out, std::string& err) override {
        CHK(check_catch(c, err));
        const Cat& C = cats[c];
        if (log_cap == 0) { err = "no step log is open (flood_log_steps)"; return FLOOD_ESTATE; }
        const int off = C.dev.member_off;
        const size_t n = (size_t)C.N * log_cap;
        HIPCHK(hipStreamSynchronize(st));
        if (dt_out) HIPCHK(hipMemcpy(dt_out, dtlog + (size_t)off * log_cap, n * sizeof(double), hipMemcpyDeviceToHost));
        if (te_out) HIPCHK(hipMemcpy(te_out, telog + (size_t)off * log_cap, n * sizeof(double), hipMemcpyDeviceToHost));
        if (count_out) HIPCHK(hipMemcpy(count_out, log_n + off, C.N * sizeof(int64_t), hipMemcpyDeviceToHost));
        return FLOOD_OK;
    }

    // depth maximum of every member of catchment c, or (m >= 0) of member m only
    flood_status recompute_hmax(int c, std::string& err, int m = -1) {
        const Cat& C = cats[c];
        if (m >= 0 && mi == 1) {
            // a one-member view: members in planes, so member m's plane is its own array
            CatchDev<T> one = C.dev;
            const size_t plane = (size_t)C.ny * C.nx;
            for (int k = 0; k < 2; ++k) one.h[k] = C.dev.h[k] + (size_t)m * plane;
            one.member_off = C.dev.member_off + m;
            one.n_members = 1;
            one.n_chunks = 1;
            launch_zero_bins<HB>(one.member_off, 1, n_total, hbins, st);
            launch_hmax_init<T>(mi, one, par, hbins, n_total, st);
        } else {
            launch_zero_bins<HB>(C.dev.member_off, C.N, n_total, hbins, st);
            launch_hmax_init<T>(mi, C.dev, par, hbins, n_total, st);
        }
        HIPCHK(hipGetLastError());
        return FLOOD_OK;
    }

    flood_status set_state(int c, int m, const double* hh, const double* qx, const double* qy, double tt,
                           std::string& err) override {
        CHK(check_catch(c, err));
        const Cat& C = cats[c];
        if (m < 0 || m >= C.N) { err = "member index out of range"; return FLOOD_EINVAL; }
        CHK(check_state_args(C.ny, C.nx, C.edge_kind, C.h_inflow_id.empty() ? nullptr : C.h_inflow_id.data(), hh, qx,
                             qy, tt, err));
        const int g = C.dev.member_off + m;
        const double* src[3] = {hh, qx, qy};
        for (int w = 0; w < 3; ++w) {
            HIPCHK(hipMemcpyAsync(d_stage, src[w], field_size(C, w) * sizeof(double), hipMemcpyHostToDevice, st));
            launch_set_field<T>(mi, C.dev, m, par, w, d_stage, st);
            if (w == FLOOD_FIELD_H && C.dev.peak) launch_set_field<T>(mi, C.dev, m, par, FLOOD_FIELD_PEAK, d_stage, st);
            HIPCHK(hipStreamSynchronize(st));
        }
        HIPCHK(hipMemcpy(t + g, &tt, sizeof(double), hipMemcpyHostToDevice));
        CHK(recompute_hmax(c, err, m));
        HIPCHK(hipStreamSynchronize(st));
        return FLOOD_OK;
    }

    flood_status set_params(int c, const float* manning, const double* n_scale, const double* rain_mult,
                            std::string& err) override {
        CHK(check_catch(c, err));
        const Cat& C = cats[c];
        const size_t ncell = (size_t)C.ny * C.nx;
        CHK(check_param_update(ncell, C.N, C.n_classes, manning, n_scale, rain_mult, err));
        HIPCHK(hipStreamSynchronize(st));
        if (manning) {
            std::vector<T> hn(ncell);
            for (size_t i = 0; i < ncell; ++i) hn[i] = (T)manning[i];
            HIPCHK(hipMemcpy(const_cast<T*>(C.dev.n), hn.data(), ncell * sizeof(T), hipMemcpyHostToDevice));
        }
        if (n_scale) HIPCHK(hipMemcpy(s + C.dev.member_off, n_scale, C.N * sizeof(double), hipMemcpyHostToDevice));
        if (rain_mult) HIPCHK(hipMemcpy(mu + C.dev.member_off, rain_mult, C.N * sizeof(double), hipMemcpyHostToDevice));
        return FLOOD_OK;
    }

    flood_status get_ledger(int c, double* storage, double* rain_in, double* outflow, double* clamp,
                            double* drained, double* inflow, double* tt, int64_t* stp, std::string& err) override {
        CHK(check_catch(c, err));
        const Cat& C = cats[c];
        const int off = C.dev.member_off;
        launch_flush_outflow(C.N, 2 * (C.nx + C.ny), C.dev.out_acc, vout + off, st);
        if (C.dev.drain_acc) launch_flush_outflow(C.N, kBins, C.dev.drain_acc, vdrain + off, st);
        if (storage) {
            HIPCHK(hipMemsetAsync(d_stage, 0, C.N * sizeof(double), st));
            launch_storage<T>(mi, C.dev, par, d_stage, st);
        }
        const struct { void* out; const void* src; } want[] = {
            {storage, d_stage},      {rain_in, vrain + off}, {outflow, vout + off}, {clamp, vclamp + off},
            {drained, vdrain + off}, {inflow, vin + off},    {tt, t + off},         {stp, steps + off}};
        PackList L{};
        void* out[8];
        L.n = C.N;
        for (const auto& x : want)
            if (x.out) {
                L.src[L.arrays] = static_cast<const uint64_t*>(x.src);
                out[L.arrays++] = x.out;
            }
        if (!L.arrays) {
            HIPCHK(hipStreamSynchronize(st));
            return FLOOD_OK;
        }
        return stage_out(
            1, 1, [&](size_t, size_t, double* dst) { launch_pack(L, reinterpret_cast<uint64_t*>(dst), st); },
            [&](size_t, size_t, const double* src) {
                for (int a = 0; a < L.arrays; ++a) std::memcpy(out[a], src + (size_t)a * C.N, (size_t)C.N * 8);
            }, err);
    }

    flood_status get_land_params(int c, double* cn, double* dr, std::string& err) override {
        CHK(check_catch(c, err));
        const Cat& C = cats[c];
        if (!C.n_classes) { err = "this catchment has no land cover"; return FLOOD_ESTATE; }
        const int off = C.dev.member_off;
        HIPCHK(hipStreamSynchronize(st));
        if (cn) {
            std::vector<double> all((size_t)C.N * kMaxClasses);
            HIPCHK(hipMemcpy(all.data(), clsn + (size_t)off * kMaxClasses, all.size() * sizeof(double),
                             hipMemcpyDeviceToHost));
            for (int m = 0; m < C.N; ++m)
                for (int k = 0; k < C.n_classes; ++k) cn[(size_t)m * C.n_classes + k] = all[(size_t)m * kMaxClasses + k];
        }
        if (dr) HIPCHK(hipMemcpy(dr, drain + off, C.N * sizeof(double), hipMemcpyDeviceToHost));
        return FLOOD_OK;
    }

    flood_status get_weights(int c, double* lw, double* rm, double* ns, std::string& err) override {
        CHK(check_catch(c, err));
        const Cat& C = cats[c];
        const int off = C.dev.member_off;
        HIPCHK(hipStreamSynchronize(st));
        if (lw) HIPCHK(hipMemcpy(lw, logw + off, C.N * sizeof(double), hipMemcpyDeviceToHost));
        if (rm) HIPCHK(hipMemcpy(rm, mu + off, C.N * sizeof(double), hipMemcpyDeviceToHost));
        if (ns) HIPCHK(hipMemcpy(ns, s + off, C.N * sizeof(double), hipMemcpyDeviceToHost));
        return FLOOD_OK;
    }

    // ---------------------------------------------------------------------
    // snapshots: raw device images of every array, after a shape header
    // ---------------------------------------------------------------------
    struct Blob {
        void* p;
        size_t bytes;
    };

    std::vector<Blob> blobs() {
        std::vector<Blob> v;
        for (auto& C : cats) {
            for (int k = 0; k < 2; ++k) {
                v.push_back({C.dev.h[k], C.state_elems * sizeof(T)});
                v.push_back({C.dev.qx[k], C.state_elems * sizeof(T)});
                v.push_back({C.dev.qy[k], C.state_elems * sizeof(T)});
                v.push_back({C.dev.qw[k], C.strip_w * sizeof(T)});
                v.push_back({C.dev.qn[k], C.strip_n * sizeof(T)});
            }
            v.push_back({const_cast<T*>(C.dev.n), (size_t)C.ny * C.nx * sizeof(T)});
            v.push_back({C.dev.out_acc, (size_t)C.N * 2 * (C.nx + C.ny) * sizeof(double)});
            if (C.dev.drain_acc) v.push_back({C.dev.drain_acc, (size_t)C.N * kBins * sizeof(double)});
            if (C.dev.peak) v.push_back({C.dev.peak, C.state_elems * sizeof(T)});
        }
        const size_t n = n_total;
        v.push_back({t, n * 8});
        v.push_back({s, n * 8});
        v.push_back({mu, n * 8});
        v.push_back({logw, n * 8});
        v.push_back({vrain, n * 8});
        v.push_back({vout, n * 8});
        v.push_back({vclamp, n * 8});
        v.push_back({steps, n * 8});
        v.push_back({clsn, n * kMaxClasses * 8});
        v.push_back({drain, n * 8});
        v.push_back({vdrain, n * 8});
        v.push_back({vin, n * 8});
        v.push_back({par, n * 4});
        v.push_back({fault, n * 4});
        v.push_back({hbins, (size_t)kBins * n * sizeof(HB)});
        return v;
    }

    // device snapshot (flood_device_snapshot): every blob of a file snapshot,
    // copied back to back into one device buffer held by the handle
    Scratch snap;
    bool snap_valid = false;

    // the blobs to (take) or from the snapshot, which lets them follow one another on
    // 256-byte boundaries
    flood_status copy_snapshot(const std::vector<Blob>& bl, bool take, std::string& err) {
        CopyList L;
        L.n = 0;
        L.clear = take ? nullptr : status;
        char* at = static_cast<char*>(snap.p);
        for (size_t i = 0; i < bl.size(); ++i) {
            if (bl[i].bytes) {
                CopyList::Item& it = L.item[L.n++];
                it.dst = take ? at : static_cast<char*>(bl[i].p);
                it.src = take ? static_cast<char*>(bl[i].p) : at;
                it.bytes = bl[i].bytes;
            }
            at += (bl[i].bytes + 255) / 256 * 256;
            if (L.n == kCopyList || i + 1 == bl.size()) {
                launch_copy_list(L, st);
                L.n = 0;
            }
        }
        HIPCHK(hipGetLastError());
        return FLOOD_OK;
    }

    flood_status device_snapshot(int op, std::string& err) override {
        if (op == FLOOD_SNAPSHOT_RELEASE) {
            HIPCHK(hipStreamSynchronize(st));
            if (snap.p) (void)hipFree(snap.p);
            snap = Scratch{};
            snap_valid = false;
            return FLOOD_OK;
        }
        const std::vector<Blob> bl = blobs();
        size_t total = 0;
        for (const Blob& b : bl) total += (b.bytes + 255) / 256 * 256;
        if (op == FLOOD_SNAPSHOT_TAKE) {
            if (!snap.p || snap.bytes < total) {
                HIPCHK(hipStreamSynchronize(st));
                if (snap.p) (void)hipFree(snap.p);
                snap = Scratch{};
                snap_valid = false;
                if (hipMalloc(&snap.p, total) != hipSuccess) {
                    (void)hipGetLastError();
                    snap.p = nullptr;
                    err = "hipMalloc of " + std::to_string(total) + " bytes for the device snapshot failed";
                    return FLOOD_ENOMEM;
                }
                snap.bytes = total;
            }
            CHK(copy_snapshot(bl, true, err));
            snap_valid = true;
            return FLOOD_OK;
        }
        if (!snap_valid) { err = "no device snapshot has been taken"; return FLOOD_ESTATE; }
        CHK(copy_snapshot(bl, false, err));   // and clears the status word
        return FLOOD_OK;
    }

    void header(std::vector<int64_t>& hd) const {
        hd = {0x464c4f4f44534e32LL, (int64_t)sizeof(T), mi, n_catch, n_total};
        for (auto& C : cats) {
            hd.push_back(C.ny);
            hd.push_back(C.nx);
            hd.push_back(C.N);
            hd.push_back(C.dev.peak ? 1 : 0);
            hd.push_back(C.n_classes);
            hd.push_back(C.n_series);
        }
    }

    // ensemble products of the running maximum depth (Sec. 4.4, Figs. 15-16)
    flood_status products(int c, double threshold, int n_pct, const double* pct, const double* weights,
                          double* prob_out, double* pct_out, std::string& err) override {
        CHK(check_catch(c, err));
        const Cat& C = cats[c];
        std::vector<double> w;
        CHK(check_products(C.N, threshold, n_pct, pct, weights, w, err));
        double W = 0.0;
        for (int m = 0; m < C.N; ++m) W += w[m];   // member order, as the kernel's sums
        if (!C.dev.peak) {
            err = "the running maximum is kept only by handles created with track_peak = 1";
            return FLOOD_ESTATE;
        }
        const size_t ncell = (size_t)C.ny * C.nx;
        // weights (zeros up to kProdPad) and percentiles
        double* const d_w = d_stage;
        double* const d_p = d_stage + std::max(C.N, kProdPad);
        w.resize(std::max(C.N, kProdPad), 0.0);
        w.insert(w.end(), pct, pct + n_pct);
        HIPCHK(hipMemcpyAsync(d_w, w.data(), w.size() * sizeof(double), hipMemcpyHostToDevice, st));
        HIPCHK(hipStreamSynchronize(st));   // w is this call's
        const int maps = pct_out ? n_pct : 0;
        if (!prob_out && !maps) return FLOOD_OK;
        const size_t per = kOutElems / ((prob_out ? 1 : 0) + maps) / 64 * 64;   // whole wavefronts of cells
        return stage_out(
            ncell, per,
            [&](size_t c0, size_t n, double* dst) {
                launch_products<T>(mi, C.dev, threshold, maps, d_p, d_w, W, c0, n, prob_out ? dst : nullptr,
                                   dst + (prob_out ? n : 0), st);
            },
            [&](size_t c0, size_t n, const double* src) {
                if (prob_out) {
                    std::memcpy(prob_out + c0, src, n * sizeof(double));
                    src += n;
                }
                for (int i = 0; i < maps; ++i)
                    std::memcpy(pct_out + i * ncell + c0, src + i * n, n * sizeof(double));
            }, err);
    }

    flood_status save(const char* path, std::string& err) override {
        HIPCHK(hipStreamSynchronize(st));
        FILE* f = std::fopen(path, "wb");
        if (!f) { err = std::string("cannot open ") + path; return FLOOD_EINVAL; }
        std::vector<int64_t> hd;
        header(hd);
        const int64_t nh = (int64_t)hd.size();
        bool ok = std::fwrite(&nh, 8, 1, f) == 1 && std::fwrite(hd.data(), 8, hd.size(), f) == hd.size();
        std::vector<char> buf;
        for (auto& b : blobs()) {
            if (!ok) break;
            buf.resize(b.bytes);
            if (hipMemcpy(buf.data(), b.p, b.bytes, hipMemcpyDeviceToHost) != hipSuccess) {
                std::fclose(f);
                err = "device read failed";
                return FLOOD_EHIP;
            }
            ok = std::fwrite(buf.data(), 1, b.bytes, f) == b.bytes;
        }
        ok = (std::fclose(f) == 0) && ok;
        if (!ok) { err = "write failed"; return FLOOD_EINVAL; }
        return FLOOD_OK;
    }

    flood_status load(const char* path, std::string& err) override {
        FILE* f = std::fopen(path, "rb");
        if (!f) { err = std::string("cannot open ") + path; return FLOOD_EINVAL; }
        std::vector<int64_t> hd, got;
        header(hd);
        int64_t nh = 0;
        bool ok = std::fread(&nh, 8, 1, f) == 1 && nh == (int64_t)hd.size();
        if (ok) {
            got.resize(nh);
            ok = std::fread(got.data(), 8, nh, f) == (size_t)nh && got == hd;
        }
        if (!ok) {
            std::fclose(f);
            err = "snapshot does not match this handle's shape";
            return FLOOD_EINVAL;
        }
        std::vector<std::vector<char>> data;
        for (auto& b : blobs()) {
            data.emplace_back(b.bytes);
            if (std::fread(data.back().data(), 1, b.bytes, f) != b.bytes) {
                std::fclose(f);
                err = "snapshot is truncated";
                return FLOOD_EINVAL;
            }
        }
        std::fclose(f);
        HIPCHK(hipStreamSynchronize(st));
        size_t i = 0;
        for (auto& b : blobs()) {
            HIPCHK(hipMemcpy(b.p, data[i].data(), b.bytes, hipMemcpyHostToDevice));
            ++i;
        }
        HIPCHK(hipMemset(status, 0, sizeof(int32_t)));
        return FLOOD_OK;
    }

    void get_config(int32_t* omi, int32_t* rows, int32_t* cpb, int32_t* gs, int32_t* vk, int32_t* mr,
                    int32_t* mseg, int32_t* mord) const override {
        if (mseg) *mseg = march_seg;
        if (mord) *mord = march_order;
        if (omi) *omi = mi;
        if (rows) *rows = cats[0].tile_rows;
        if (cpb) *cpb = std::min(cats[0].cpb, cats[0].n_chunks);
        if (gs) *gs = (use_graph && gexec[0]) ? G : 0;
        if (vk) *vk = variant;
        if (mr) *mr = std::min(cats[0].march_rows, cats[0].ny);
    }

    flood_status get_march_rows(int c, int32_t* rows, std::string& err) const override {
        CHK(check_catch(c, err));
        if (!rows) { err = "march_rows is NULL"; return FLOOD_EINVAL; }
        *rows = std::min(cats[c].march_rows, cats[c].ny);
        return FLOOD_OK;
    }

    flood_status timing(int mode, std::string& err) override {
        HIPCHK(hipStreamSynchronize(st));
        if (mode) {
            t_ms = 0.0;
            t_launches = 0;
            tev_used = 0;
        }
        timing_on = mode == FLOOD_TIMING_LAUNCH;
        timing_batch = mode == FLOOD_TIMING_BATCH;
        return FLOOD_OK;
    }

    void get_timing(double* avg, int64_t* n) const override {
        if (avg) *avg = t_launches ? t_ms / (double)t_launches : 0.0;
        if (n) *n = t_launches;
    }
};

// A view of members [g0, g0 + G) of catchment c (g0 a multiple of MI) over state
// arrays laid out like the catchment's, with its own tile grid (one workgroup
// per tile walking every chunk of the group).  The tile shape is fixed rather
// than taken from the tuned forward geometry: the adjoint's per-workgroup
// partial sums then group cells the same way on every handle of a given
// interleave, so its gradients do not depend on what the tuner picked.
constexpr int kAdjTileRows = 4;
constexpr int kAdjMarchRows = 8;
constexpr int kAdjMarchOrder = 4;   // recorded forward, recomputation: strips in bands over the XCDs (see march_wave)
// the reverse step: the member quads of a row of strips one after the other; at
// 1024 x 1024 x 16 in FP32 128 us a step against 134 with order 4 and 132 with 0 or 2
constexpr int kAdjReverseOrder = 3;
// Rows per strip on grids too small to fill the chip: a strip is a chain of rows,
// so strips are halved (down to 2 rows) while there are fewer of them than
// workgroups to go round (`per` of them make one).  From the grid alone for the
// reverse step, whose partial sums are taken by strip.  At 64 x 96 x 4 in FP64, 2
// rows against 8: reverse step 11.0 us against 22.1, recorded step 8.4 against 14.9.
static int adj_rows(int rows, int strips_x, int ny, int per) {
    while (rows > 2 && strips_x * ((ny + rows - 1) / rows) < 256 * per) rows /= 2;
    return rows;
}
constexpr size_t kAdjMaxGroup = 16;  // members of a row-march adjoint group at most

// Members of a row-march adjoint group: as many as a pool of tape blocks holds
// when each takes `steps` steps, plus its first state and two batches of bm
// launches of slack (between 1 and gmax).
static int adj_group_size(size_t pool, int steps, int bm, int gmax) {
    const size_t per = (size_t)std::max(steps, 0) + 1 + 2 * (size_t)bm;
    return (int)std::max<size_t>(1, std::min<size_t>(pool / per, (size_t)gmax));
}

// Rows per strip of a row-march view of G members, with the strip rows, bands
// and wavefront count that follow from them.
template <typename T>
static void set_march_rows(CatchDev<T>& v, int rows, int G) {
    v.march_rows = std::min(rows, v.ny);
    v.strips_y = (v.ny + v.march_rows - 1) / v.march_rows;
    v.march_bands = std::max(8, std::min((int)std::ceil((double)v.ny * v.nx * 2.0 * sizeof(T) / (1 << 20) / 8.0) * 8,
                                         (v.strips_y + 7) / 8 * 8));
    v.n_waves = march_waves(v.strips_x, v.strips_y, G, v.march_order, v.march_bands);
}

template <typename T>
static CatchDev<T> group_view(const CatchDev<T>& C, int mi, int g0, int G, T* const h[2], T* const qx[2],
                              T* const qy[2], T* const qw[2], T* const qn[2]) {
    CatchDev<T> v = C;
    v.peak = nullptr;   // tape, checkpoint and adjoint views; the recorded forward sets its own
    const int txc = std::max(1, kBlock / (mi * kAdjTileRows));
    int l = 0;
    while ((1 << l) < txc) ++l;
    v.tx_log2 = l;
    const int ty = (kBlock / mi) >> l;
    v.tiles_x = (C.nx + (1 << l) - 1) >> l;
    v.tiles_y = (C.ny + ty - 1) / ty;
    // row-march geometry (members in planes), likewise fixed
    const int strip_w = 64 * march_vec<T>();       // the recorded forward and tape recomputation (k_marchv)
    const int strip_wa = 62 * adj_vec<T>();        // the reverse step (k_adjv)
    // at most 16: the reverse step stages 4 x rows x 64 x V values in LDS
    int rows = adj_rows(kAdjMarchRows, (C.nx + strip_wa - 1) / strip_wa, C.ny, 1);
    if (const char* ar = std::getenv("FLOOD_ADJ_ROWS")) rows = std::min(16, std::max(1, std::atoi(ar)));
    v.march_rows = std::min(rows, C.ny);
    v.strips_x = (C.nx + strip_w - 1) / strip_w;
    v.strips_xa = (C.nx + strip_wa - 1) / strip_wa;
    v.strips_y = (C.ny + v.march_rows - 1) / v.march_rows;
    v.wave_begin = 0;
    v.march_order = kAdjMarchOrder;
    // bands of about 1 MiB of bed and roughness, as in the forward (a multiple of 8)
    v.march_bands = std::max(8, std::min((int)std::ceil((double)C.ny * C.nx * 2.0 * sizeof(T) / (1 << 20) / 8.0) * 8,
                                         (v.strips_y + 7) / 8 * 8));
    v.n_waves = march_waves(v.strips_x, v.strips_y, G, v.march_order, v.march_bands);
    v.member_off = C.member_off + g0;
    v.n_members = G;
    v.n_chunks = (G + mi - 1) / mi;
    v.groups = 1;
    v.chunks_per_group = v.n_chunks;
    v.n_blocks = v.tiles_x * v.tiles_y;
    v.block_begin = 0;
    for (int k = 0; k < 2; ++k) {
        v.h[k] = h[k];
        v.qx[k] = qx[k];
        v.qy[k] = qy[k];
        v.qw[k] = qw[k];
        v.qn[k] = qn[k];
    }
    return v;
}

template <typename T>
flood_status Impl<T>::adjoint(int c, double t_end, double sample_dt, int K, const int32_t* grc, const double* obs,
                              int ckpt_every, double* loss_out, double* grad_n_out, double* grad_mult_out,
                              std::string& err) {
    CHK(check_catch(c, err));
    Cat& C = cats[c];
    CHK(check_adjoint_args(C.ny, C.nx, C.n_classes, C.n_series, t_end, sample_dt, K, grc, obs, ckpt_every, err));
    double t0;
    CHK(common_time(c, &t0, err));
    int S = 0, gauges_distinct = 1;
    CHK(adjoint_samples(C.nx, t0, t_end, sample_dt, K, grc, obs, &S, &gauges_distinct, err));

    const size_t ncell = (size_t)C.ny * C.nx;
    const int N = C.N;
    // member groups sized so that the tape (ckpt_every + 1 states) fits in half the free memory
    size_t free_b = 0, total_b = 0;
    HIPCHK(hipMemGetInfo(&free_b, &total_b));
    free_b += adj_held();   // held from an earlier call: reused or replaced below
    const size_t per_member_state = (3 * ncell + C.ny + C.nx) * sizeof(T);
    const size_t per_member_slot = per_member_state + ncell;   // + clamp flags
    // members in planes with a vectorisable row length: the adjoint runs in
    // row-march form (forward, tape recomputation and reverse step), otherwise
    // in the tiled form that also serves interleaved members
    const bool march_adj = variant == 3 && vector_ok() && !adj_tiled;
    size_t env_group = 0;
    if (const char* eg = std::getenv("FLOOD_ADJ_GROUP")) {   // testing: force smaller member groups
        const long v = std::atol(eg);
        if (v > 0) env_group = (size_t)v;
    }
    // recording-forward launches per batch (a member takes at most one step per launch)
    const int Bm = std::min(8, ckpt_every);
    size_t G = 0;         // tiled form: members per group; row-march form: the most members a group takes
    size_t pool = 0;      // row-march form: tape blocks (one member state and its clamp flags each)
    int g_first = 0;      // row-march form: members of the first group
    if (march_adj) {
        // The row-march form keeps every step of its group's members in a pool of
        // tape blocks that takes most of the free memory: a member uses as many
        // blocks as it takes steps, so members that step less leave room for more
        // members in a group.  A group holds at most kAdjMaxGroup members (larger
        // launches gain little); their adjoint copies, checkpoints and
        // accumulators are kept outside the pool.
        G = std::min<size_t>((size_t)N, kAdjMaxGroup);
        if (env_group) G = std::min(G, env_group);
        const double spare = 0.85 * (double)free_b - (double)(G * 8 * per_member_state);
        pool = spare > 0.0 ? (size_t)(spare / (double)per_member_state) : 0;
        // A pool held from an earlier call is kept when it is nearly as large:
        // freeing and allocating a block of this size costs seconds, and the same
        // pool gives the same member groups on every call.
        const size_t held = adj_tape.bytes / per_member_state;
        if (adj_tape.p && held >= pool - pool / 16) pool = held;
        // never more than every member of the largest group taking ckpt_every steps
        pool = std::min(pool, G * ((size_t)ckpt_every + 1 + 2 * (size_t)Bm));
        if (const char* ep = std::getenv("FLOOD_ADJ_POOL")) {   // testing: a smaller pool
            const long v = std::atol(ep);
            if (v > 0) pool = std::min(pool, (size_t)v);
        }
        pool = std::min<size_t>(pool, (size_t)INT32_MAX);
        // a group needs its members' first states and two batches of steps
        if (pool < (size_t)(2 * Bm + 2)) { err = "adjoint tape does not fit in device memory"; return FLOOD_ENOMEM; }
        g_first = adj_group_size(pool, ckpt_every, Bm, (int)G);
    } else {
        // the tiled form keeps ckpt_every + 1 states per member in half the free memory
        G = (size_t)(0.5 * (double)free_b) / ((size_t)(ckpt_every + 1) * per_member_slot + 8 * per_member_state);
        G = std::min<size_t>(G, (size_t)N);
        if (env_group) G = std::min(G, env_group);
        G = (G / mi) * mi;
        if (G < (size_t)mi) { err = "adjoint tape does not fit in device memory"; return FLOOD_ENOMEM; }
        // as many groups as memory needs, all of one size: equal launches, and a
        // grouping that small changes of free memory do not move
        const size_t n_groups = ((size_t)N + G - 1) / G;
        G = (((size_t)N + n_groups - 1) / n_groups + mi - 1) / mi * mi;
    }

    // Several groups: the members are brought into the order of their expected step
    // counts, most steps first, so that a group's members take about as many steps
    // (every launch of a group runs until its slowest member is done) and each
    // group can be sized from the step counts of the one before it.  Eq. 4 ties
    // the step count to the depth, and the depth a member reaches to its current
    // depth and the rain it still receives: the key is the member's current maximum
    // depth plus its rain multiplier times the rain depth of the window.  Slots are
    // restored on every way out of the call; results do not depend on the order
    // (the loss is summed in member order, each member's gradient is its own).
    std::vector<int32_t> order(N), inv(N);
    for (int i = 0; i < N; ++i) order[i] = inv[i] = i;
    bool reordered = false;
    if (march_adj && N > g_first && !std::getenv("FLOOD_ADJ_NO_ORDER")) {
        const int off = C.dev.member_off;
        std::vector<HB> hb((size_t)kBins * n_total);
        std::vector<double> hmu(N);
        HIPCHK(hipStreamSynchronize(st));
        HIPCHK(hipMemcpy(hb.data(), hbins, hb.size() * sizeof(HB), hipMemcpyDeviceToHost));
        HIPCHK(hipMemcpy(hmu.data(), mu + off, N * sizeof(double), hipMemcpyDeviceToHost));
        double rain_depth = 0.0;   // rain depth of [t0, t_end] at multiplier 1
        const double ri = C.p.rain_interval;
        for (size_t j = 0; j < C.rain.size(); ++j) {
            const double a = std::max(t0, (double)j * ri), b = std::min(t_end, (double)(j + 1) * ri);
            if (b > a) rain_depth += C.rain[j] * (b - a);
        }
        std::vector<double> key(N);
        for (int m = 0; m < N; ++m) {
            HB mx = 0;
            for (int b = 0; b < kBins; ++b) mx = std::max(mx, hb[(size_t)b * n_total + off + m]);
            T hmax;
            std::memcpy(&hmax, &mx, sizeof(T));
            key[m] = (double)hmax + hmu[m] * rain_depth;
        }
        std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return key[a] > key[b]; });
        for (int i = 0; i < N; ++i) inv[order[i]] = i;
        for (int i = 0; i < N && !reordered; ++i) reordered = order[i] != i;
    }
    if (reordered) CHK(reorder_members(c, order, err));
    struct Restore {
        Impl* self;
        int c;
        const std::vector<int32_t>* inv;
        bool armed;
        ~Restore() {
            std::string e;
            if (armed) (void)self->reorder_members(c, *inv, e);
        }
    } restore{this, c, &inv, reordered};

    // device scratch owned by this call
    std::vector<void*> tmp;
    auto talloc = [&](size_t bytes, void** p) -> flood_status {
        hipError_t e = hipMalloc(p, std::max<size_t>(bytes, 16));
        if (e != hipSuccess) {
            (void)hipGetLastError();
            err = "hipMalloc of " + std::to_string(bytes) + " bytes failed in flood_adjoint";
            return FLOOD_ENOMEM;
        }
        tmp.push_back(*p);
        return FLOOD_OK;
    };
    struct Guard {
        std::vector<void*>& v;
        hipStream_t s;
        ~Guard() {
            (void)hipStreamSynchronize(s);
            for (void* p : v) (void)hipFree(p);
        }
    } guard{tmp, st};

    const int Gi = (int)G;
    const int chunksG = (Gi + mi - 1) / mi;
    const size_t elemsG = (size_t)chunksG * ncell * mi;
    const size_t wG = (size_t)chunksG * C.ny * mi, nG = (size_t)chunksG * C.nx * mi;
    const size_t slot_elems = 3 * elemsG + wG + nG;
    const int max_launch = 1 << 20;
    int32_t* d_grc2 = nullptr;
    double *d_obs2 = nullptr, *d_loss = nullptr, *d_nbar = nullptr, *d_mubar = nullptr, *d_gm = nullptr;
    CHK(talloc(2 * std::max(K, 1) * sizeof(int32_t), (void**)&d_grc2));
    CHK(talloc((size_t)S * std::max(K, 1) * sizeof(double), (void**)&d_obs2));
    CHK(talloc((size_t)N * sizeof(double), (void**)&d_loss));   // tiled form: misfit per member
    CHK(talloc(ncell * sizeof(double), (void**)&d_nbar));
    CHK(talloc((size_t)N * sizeof(double), (void**)&d_gm));
    if (K > 0) {
        HIPCHK(hipMemcpyAsync(d_grc2, grc, 2 * K * sizeof(int32_t), hipMemcpyHostToDevice, st));
        HIPCHK(hipMemcpyAsync(d_obs2, obs, (size_t)S * K * sizeof(double), hipMemcpyHostToDevice, st));
    }
    HIPCHK(hipMemsetAsync(d_loss, 0, (size_t)N * sizeof(double), st));
    HIPCHK(hipMemsetAsync(d_nbar, 0, ncell * sizeof(double), st));
    // Tape.  Row-march form: the pool of blocks, each field's blocks contiguous
    // (block b of the depth at b * ncell, of the west edge strip at b * ny, ...),
    // with a clamped depth kept as -0.  Tiled form: ckpt_every + 1 slots of the
    // group state and ckpt_every slots of clamp flags.  Then the adjoint ping-pong.
    T* tape = nullptr;
    uint8_t* clamp = nullptr;
    T* lam = nullptr;
    const size_t tape_elems = march_adj ? pool * (3 * ncell + C.ny + C.nx) : (size_t)(ckpt_every + 1) * slot_elems;
    if (!march_adj) {
        CHK(adj_reserve(adj_clamp, (size_t)ckpt_every * elemsG, err));
    } else if (adj_clamp.p) {   // held from a tiled-form call: counted as free above
        HIPCHK(hipStreamSynchronize(st));
        (void)hipFree(adj_clamp.p);
        adj_clamp.p = nullptr;
        adj_clamp.bytes = 0;
    }
    CHK(adj_reserve(adj_tape, tape_elems * sizeof(T), err));
    CHK(adj_reserve(adj_lam, 2 * slot_elems * sizeof(T), err));
    tape = static_cast<T*>(adj_tape.p);
    clamp = static_cast<uint8_t*>(adj_clamp.p);
    lam = static_cast<T*>(adj_lam.p);
    // per-launch record
    MemberStep<T>* ms_log = nullptr;
    double* rdt_log = nullptr;
    int32_t *tag_log = nullptr, *any_log = nullptr;
    int nblk;
    {
        T* none[2] = {nullptr, nullptr};
        const CatchDev<T> tv = group_view(C.dev, mi, 0, std::min(Gi, N), none, none, none, none, none);
        nblk = tv.tiles_x * tv.tiles_y;
        if (march_adj) nblk = tv.strips_xa * tv.strips_y;
    }
    CHK(talloc((size_t)nblk * Gi * sizeof(double), (void**)&d_mubar));
    // row-march form: per-member adjoint copy index, Manning-field accumulators,
    // member-local step records ([segment][slot][member]) and per-member counters
    int32_t* d_lpar = nullptr;
    int32_t* d_segcnt = nullptr;
    int32_t *d_smp = nullptr, *d_pend = nullptr;
    int32_t *d_curblk = nullptr, *d_pool = nullptr, *d_hcnt3 = nullptr;
    double* d_lossm = nullptr;
    T* d_nacc = nullptr;
    MemberStep<T>* rec_ms = nullptr;
    double* rec_rdt = nullptr;
    int32_t* rec_tag = nullptr;
    size_t rec_cap = 0;
    int32_t* seg_n = nullptr;
    size_t segn_cap = 0;
    std::vector<double> loss_slot(N, 0.0);   // each slot's misfit
    if (march_adj) {
        CHK(talloc((size_t)Gi * sizeof(int32_t), (void**)&d_lpar));
        CHK(talloc((size_t)Gi * sizeof(int32_t), (void**)&d_segcnt));
        CHK(talloc((size_t)Gi * sizeof(int32_t), (void**)&d_smp));
        CHK(talloc((size_t)Gi * sizeof(int32_t), (void**)&d_pend));
        CHK(talloc((size_t)Gi * sizeof(int32_t), (void**)&d_curblk));
        CHK(talloc(sizeof(int32_t), (void**)&d_pool));
        CHK(talloc((size_t)Gi * sizeof(double), (void**)&d_lossm));
        // one Manning-field accumulator per member quad
        CHK(adj_reserve(adj_nacc, (size_t)((Gi + 3) / 4) * ncell * sizeof(T), err));
        d_nacc = static_cast<T*>(adj_nacc.p);
        if (!h_cnt3) HIPCHK(hipHostMalloc((void**)&h_cnt3, 8 * sizeof(int32_t), hipHostMallocDefault));
        // the batch counts go straight into the pinned block (no copy command per batch)
        HIPCHK(hipHostGetDevicePointer((void**)&d_hcnt3, h_cnt3, 0));
    }
    // grow the member-local records to hold n entries (contents kept)
    auto grow_rec = [&](size_t n) -> flood_status {
        if (n <= rec_cap) return FLOOD_OK;
        size_t cap = std::max<size_t>(rec_cap * 2, n);
        MemberStep<T>* a;
        double* r;
        int32_t* g;
        CHK(talloc(cap * sizeof(MemberStep<T>), (void**)&a));
        CHK(talloc(cap * sizeof(double), (void**)&r));
        CHK(talloc(cap * sizeof(int32_t), (void**)&g));
        if (rec_cap) {
            HIPCHK(hipMemcpyAsync(a, rec_ms, rec_cap * sizeof(MemberStep<T>), hipMemcpyDeviceToDevice, st));
            HIPCHK(hipMemcpyAsync(r, rec_rdt, rec_cap * sizeof(double), hipMemcpyDeviceToDevice, st));
            HIPCHK(hipMemcpyAsync(g, rec_tag, rec_cap * sizeof(int32_t), hipMemcpyDeviceToDevice, st));
        }
        rec_ms = a;
        rec_rdt = r;
        rec_tag = g;
        rec_cap = cap;
        return FLOOD_OK;
    };
    auto grow_segn = [&](size_t n) -> flood_status {
        if (n <= segn_cap) return FLOOD_OK;
        size_t cap = std::max<size_t>(segn_cap * 2, n);
        int32_t* a;
        CHK(talloc(cap * sizeof(int32_t), (void**)&a));
        if (segn_cap) HIPCHK(hipMemcpyAsync(a, seg_n, segn_cap * sizeof(int32_t), hipMemcpyDeviceToDevice, st));
        seg_n = a;
        segn_cap = cap;
        return FLOOD_OK;
    };
    int n_segments = 0;
    size_t log_cap = 4096;
    auto grow_log = [&](size_t need) -> flood_status {
        if (need <= log_cap && ms_log) return FLOOD_OK;
        size_t cap = std::max(log_cap, (size_t)4096);
        while (cap < need) cap *= 2;
        MemberStep<T>* a;
        double* r;
        int32_t *tg, *an;
        CHK(talloc(cap * Gi * sizeof(MemberStep<T>), (void**)&a));
        CHK(talloc(cap * Gi * sizeof(double), (void**)&r));
        CHK(talloc(cap * Gi * sizeof(int32_t), (void**)&tg));
        CHK(talloc(cap * sizeof(int32_t), (void**)&an));
        HIPCHK(hipMemsetAsync(an, 0, cap * sizeof(int32_t), st));
        if (ms_log) {
            HIPCHK(hipMemcpyAsync(a, ms_log, log_cap * Gi * sizeof(MemberStep<T>), hipMemcpyDeviceToDevice, st));
            HIPCHK(hipMemcpyAsync(r, rdt_log, log_cap * Gi * sizeof(double), hipMemcpyDeviceToDevice, st));
            HIPCHK(hipMemcpyAsync(tg, tag_log, log_cap * Gi * sizeof(int32_t), hipMemcpyDeviceToDevice, st));
            HIPCHK(hipMemcpyAsync(an, any_log, log_cap * sizeof(int32_t), hipMemcpyDeviceToDevice, st));
        }
        ms_log = a;
        rdt_log = r;
        tag_log = tg;
        any_log = an;
        log_cap = cap;
        return FLOOD_OK;
    };

    // checkpoint i of a member group: the i-th held block, grown to a group state
    auto checkpoint = [&](int i, T** p) -> flood_status {
        if ((int)adj_ckpt.size() <= i) adj_ckpt.resize(i + 1);
        CHK(adj_reserve(adj_ckpt[i], slot_elems * sizeof(T), err));
        *p = static_cast<T*>(adj_ckpt[i].p);
        return FLOOD_OK;
    };

    const int off = C.dev.member_off;
    launch_flush_outflow(N, 2 * (C.nx + C.ny), C.dev.out_acc, vout + off, st);
    std::vector<double> gm_host(N, 0.0);

    // row-march form: the members' step counts at the start of the call, block
    // indices 0, 1, ... (a member's first block, and the pool's first free block)
    std::vector<int64_t> steps0;
    std::vector<int32_t> blk_iota;
    if (march_adj) {
        steps0.resize(N);
        HIPCHK(hipMemcpyAsync(steps0.data(), steps + off, (size_t)N * sizeof(int64_t), hipMemcpyDeviceToHost, st));
        HIPCHK(hipStreamSynchronize(st));
        blk_iota.resize((size_t)Gi + 1);
        for (int i = 0; i <= Gi; ++i) blk_iota[i] = i;
    }
    int g_next = march_adj ? g_first : Gi, groups_run = 0, group_most = 0;
    for (int g0 = 0, Gg = 0; g0 < N; g0 += Gg) {
        Gg = std::min(g_next, N - g0);
        ++groups_run;
        group_most = std::max(group_most, Gg);
        const int chunk0 = g0 / mi;
        auto at = [&](T* base) { return base + (size_t)chunk0 * ncell * mi; };
        auto atw = [&](T* base) { return base + (size_t)chunk0 * C.ny * mi; };
        auto atn = [&](T* base) { return base + (size_t)chunk0 * C.nx * mi; };
        T* mh[2] = {at(C.dev.h[0]), at(C.dev.h[1])};
        T* mqx[2] = {at(C.dev.qx[0]), at(C.dev.qx[1])};
        T* mqy[2] = {at(C.dev.qy[0]), at(C.dev.qy[1])};
        T* mqw[2] = {atw(C.dev.qw[0]), atw(C.dev.qw[1])};
        T* mqn[2] = {atn(C.dev.qn[0]), atn(C.dev.qn[1])};
        CatchDev<T> V = group_view(C.dev, mi, g0, Gg, mh, mqx, mqy, mqw, mqn);
        V.out_acc = C.dev.out_acc + (size_t)g0 * 2 * (C.nx + C.ny);
        V.peak = C.dev.peak ? at(C.dev.peak) : nullptr;   // the recorded forward advances the members
        // slot j of the tape as a view (copy 0 = slot j, copy 1 = slot j + 1)
        auto slot_view = [&](T* base, int j) {
            T* sh[2];
            T* sx[2];
            T* sy[2];
            T* sw[2];
            T* sn[2];
            for (int k = 0; k < 2; ++k) {
                T* b = base + (size_t)(j + k) * slot_elems;
                sh[k] = b;
                sx[k] = b + elemsG;
                sy[k] = b + 2 * elemsG;
                sw[k] = b + 3 * elemsG;
                sn[k] = b + 3 * elemsG + wG;
            }
            return group_view(C.dev, mi, g0, Gg, sh, sx, sy, sw, sn);
        };
        StepLaunch<T> SLg = SL;
        SLg.n_catch = 1;
        SLg.c[0] = V;
        // chunks per workgroup: as tuned for the tiled kernel, one where the steps march
        const int cpb = variant == 3 ? 1 : std::max(1, std::min(C.cpb, V.n_chunks));
        SLg.c[0].groups = (V.n_chunks + cpb - 1) / cpb;
        SLg.c[0].chunks_per_group = cpb;
        SLg.c[0].n_blocks = V.tiles_x * V.tiles_y * SLg.c[0].groups;
        SLg.total_blocks = SLg.c[0].n_blocks;
        SLg.recompute = 0;
        PlanLaunch<T> PLg = PL;
        PLg.step_lim = nullptr;
        PLg.dtlog = nullptr;
        PLg.telog = nullptr;
        PLg.m_begin = off + g0;
        PLg.m_end = off + g0 + Gg;
        if (march_adj) {
            // ---------------- row-march form ----------------
            // Recording forward: the step kernel writes each step of a member into
            // the next free block of the tape pool (the member's first state is in
            // block m, its latest in cur_blk[m]), so the last tape segment needs no
            // recomputation.  A segment ends when a member has taken ckpt_every
            // steps in it, the pool could run out or the rest fits into one more: every
            // member's latest state is then copied to its first block and to a
            // checkpoint.  Step records are member-local ([slot][member]) and carry
            // the blocks, and the members' sample times are scheduled on the
            // device, so the forward runs in batches of launches without a host
            // round trip per sample.
            const size_t plane = ncell;
            T* ph[2] = {tape, tape};
            T* pqx[2] = {tape + pool * ncell, tape + pool * ncell};
            T* pqy[2] = {tape + 2 * pool * ncell, tape + 2 * pool * ncell};
            T* pqw[2] = {tape + 3 * pool * ncell, tape + 3 * pool * ncell};
            T* pqn[2] = {pqw[0] + pool * C.ny, pqw[0] + pool * C.ny};
            const CatchDev<T> TV = group_view(C.dev, mi, g0, Gg, ph, pqx, pqy, pqw, pqn);
            // the recording forward also keeps the group's outflow and running maximum
            CatchDev<T> TVF = TV;
            TVF.out_acc = V.out_acc;
            TVF.peak = V.peak;
            const bool narrow = narrow_pays(wide_pairs(C.ny, C.nx, Gg));
            if (narrow) TVF.strips_x = (C.nx + 63) / 64;
            set_march_rows(TVF, adj_rows(kAdjMarchRows, TVF.strips_x * Gg, C.ny, 4), Gg);
            if (const char* fr = std::getenv("FLOOD_ADJ_FROWS")) set_march_rows(TVF, std::max(1, std::atoi(fr)), Gg);
            CatchDev<T> TVR = TV;   // tape recomputation: the forward's geometry
            TVR.strips_x = TVF.strips_x;
            TVR.march_rows = TVF.march_rows;
            TVR.strips_y = TVF.strips_y;
            TVR.march_bands = TVF.march_bands;
            TVR.n_waves = TVF.n_waves;
            const int tw = TVF.n_waves;
            // the group's first states (blocks 0 .. Gg - 1) to or from a checkpoint
            // laid out as a group state of Gi members
            auto ckpt_copy = [&](T* ck, bool save) -> flood_status {
                T* const fp[5] = {ph[0], pqx[0], pqy[0], pqw[0], pqn[0]};
                const size_t fo[5] = {0, elemsG, 2 * elemsG, 3 * elemsG, 3 * elemsG + wG};
                const size_t fe[5] = {plane, plane, plane, (size_t)C.ny, (size_t)C.nx};
                for (int f = 0; f < 5; ++f) {
                    T* d = save ? ck + fo[f] : fp[f];
                    const T* src = save ? fp[f] : ck + fo[f];
                    HIPCHK(hipMemcpyAsync(d, src, (size_t)Gg * fe[f] * sizeof(T), hipMemcpyDeviceToDevice, st));
                }
                return FLOOD_OK;
            };
            // member m's latest state is in its first block, and the pool's other blocks are free
            auto reset_blocks = [&]() -> flood_status {
                HIPCHK(hipMemcpyAsync(d_curblk, blk_iota.data(), (size_t)Gg * sizeof(int32_t), hipMemcpyHostToDevice,
                                      st));
                HIPCHK(hipMemcpyAsync(d_pool, &blk_iota[Gg], sizeof(int32_t), hipMemcpyHostToDevice, st));
                return FLOOD_OK;
            };
            StepLaunch<T> SLm = SL;
            SLm.n_catch = 1;
            SLm.c[0] = V;
            SLm.total_blocks = 0;
            SLm.recompute = 0;
            SLm.narrow = narrow;
            // launches per batch: a member takes at most one step per launch, so a
            // batch never takes a member past the segment's ckpt_every steps
            const int B = Bm;
            const size_t seg_recs = (size_t)ckpt_every * Gi;
            std::vector<int> seg_nmax;
            int seg = 0;
            CHK(grow_rec(seg_recs));
            auto rec_at = [&](int sg) { return rec_ms + (size_t)sg * seg_recs; };
            HIPCHK(hipMemsetAsync(rec_ms, 0, seg_recs * sizeof(MemberStep<T>), st));
            launch_snapshot<T>(mi, V, par, TV, st);
            T* ck0;
            CHK(checkpoint(0, &ck0));
            CHK(ckpt_copy(ck0, true));
            CHK(reset_blocks());
            HIPCHK(hipMemsetAsync(d_segcnt, 0, (size_t)Gi * sizeof(int32_t), st));
            HIPCHK(hipMemsetAsync(d_smp, 0, (size_t)Gi * sizeof(int32_t), st));
            HIPCHK(hipMemsetAsync(d_pend, 0xff, (size_t)Gi * sizeof(int32_t), st));
            HIPCHK(hipMemsetAsync(d_lossm, 0, (size_t)Gi * sizeof(double), st));
            PLg.seg_cnt = d_segcnt;
            PLg.cur_blk = d_curblk;
            PLg.pool_next = d_pool;
            PLg.rec_stride = Gi;
            PLg.any_log = nullptr;
            PLg.tag_value = -1;
            PLg.s_t0 = t0;
            PLg.s_dt = sample_dt;
            PLg.smp = d_smp;
            PLg.pend = d_pend;
            PLg.tape_h = tape;
            PLg.plane = plane;
            PLg.nx = C.nx;
            PLg.n_gauges = K;
            PLg.grc = d_grc2;
            PLg.obs = d_obs2;
            PLg.loss_m = d_lossm;
            auto set_seg = [&](int sg) {
                PLg.ms_log = rec_at(sg);
                PLg.rdt_log = rec_rdt + (size_t)sg * seg_recs;
                PLg.tag_log = rec_tag + (size_t)sg * seg_recs;
            };
            set_seg(0);
            *h_tend = t0 + (double)S * sample_dt;
            HIPCHK(hipMemcpyAsync(d_tend, h_tend, sizeof(double), hipMemcpyHostToDevice, st));
            StepLaunch<T> RF = SLm;
            RF.c[0] = TVF;
            RF.ms = ms;
            RF.clamp_out = nullptr;
            int64_t L = 0;
            auto launch_fwd_batch = [&](int slot, int n) -> flood_status {
                for (int i = 0; i < n; ++i) {
                    launch_plan<T>(PLg, st);
                    launch_marchv_rec<T>(RF, 1, tw, st);
                }
                L += n;
                launch_count_group(Gg, t + off + g0, fault + off + g0, d_tend, status, d_segcnt,
                                   dt_last + off + g0, d_smp, t0, sample_dt, d_hcnt3 + 4 * slot, st);
                HIPCHK(hipGetLastError());
                HIPCHK(hipEventRecord(ev[slot], st));
                return FLOOD_OK;
            };
            // end the current segment: its step counts, and every member's latest
            // state to its first block and to the next checkpoint
            auto roll = [&](int nmax) -> flood_status {
                HIPCHK(hipMemcpyAsync(seg_n + (size_t)seg * Gi, d_segcnt, (size_t)Gi * sizeof(int32_t),
                                      hipMemcpyDeviceToDevice, st));
                seg_nmax.push_back(nmax);
                ++seg;
                CHK(grow_rec((size_t)(seg + 1) * seg_recs));
                CHK(grow_segn((size_t)(seg + 1) * Gi));
                HIPCHK(hipMemsetAsync(rec_at(seg), 0, seg_recs * sizeof(MemberStep<T>), st));
                // a member's latest block is its own first block or one past the first Gg
                launch_tape_gather<T>(TV, d_curblk, TV, nullptr, st);
                T* ck;
                CHK(checkpoint(seg, &ck));
                CHK(ckpt_copy(ck, true));
                CHK(reset_blocks());
                HIPCHK(hipMemsetAsync(d_segcnt, 0, (size_t)Gi * sizeof(int32_t), st));
                set_seg(seg);
                return FLOOD_OK;
            };
            CHK(grow_segn((size_t)Gi));
            // Where the segments end.  All but the last are recomputed, so the last is
            // made as long as the tape allows: once the steps still needed fit into a
            // segment of their own, but not into the rest of this one, this one ends
            // there, instead of where it is full.  The need is an estimate (it grows as
            // the depth does); a margin, and ending one more segment early where it was
            // short, keep an estimate that fails as good as the full segments.  At
            // 1024 x 1024 x 16, 102 steps in segments of 100: 9 steps recomputed, not 96, and the
            // call takes 25.0 ms, not 29.7 (with 99 steps there is one segment either way).
            // A segment holds ckpt_every steps, or what is left for every member in the
            // pool, in whole batches.
            const int cap = (int)std::min<size_t>((size_t)ckpt_every, (pool - Gg) / Gg / B * B);
            const int last = std::max(1, cap - 1 - cap / 16);
            // harvested counts: mx steps in the segment, need steps to come; ahead: steps
            // of the batch in flight behind them
            int mx = 0, need = 0, ahead = 0;
            // steps of the next batch; 0: the segment ends here; -1: nothing left to launch
            auto next_batch = [&]() -> int {
                const int done = mx + ahead, rest = need - ahead;
                if (ahead && rest <= 0) return -1;
                int n = B;
                if (rest > 0) {
                    n = std::min(B, rest + 1);
                    if (done > 0 && done + rest > cap) {
                        if (rest <= last) return 0;
                        n = std::min(n, rest - last);
                    }
                }
                return std::min(n, cap - done);
            };
            // two batches in flight, but for the end of a segment and of the window
            CHK(launch_fwd_batch(0, std::min(B, cap)));
            int inflight = 1, next = 1, wait_slot = 0;
            int batch_n[2] = {std::min(B, cap), 0};
            for (bool first = true;; first = false) {
                if (inflight == 1 && !first) {
                    ahead = batch_n[wait_slot];
                    const int n = next_batch();
                    if (n > 0) {
                        CHK(launch_fwd_batch(next, n));
                        batch_n[next] = n;
                        next ^= 1;
                        inflight = 2;
                    }
                }
                HIPCHK(hipEventSynchronize(ev[wait_slot]));
                --inflight;
                const int32_t* cnt = h_cnt3 + 4 * wait_slot;
                const int active = cnt[0], stat = cnt[1];
                mx = cnt[2];
                need = cnt[3];
                wait_slot ^= 1;
                if (stat) {
                    HIPCHK(hipStreamSynchronize(st));
                    err = "a member's depth became non-finite or too large to advance its clock during the adjoint forward";
                    return FLOOD_ENUMERIC;
                }
                if (active == 0) {
                    if (inflight) {
                        HIPCHK(hipEventSynchronize(ev[wait_slot]));
                        mx = std::max(mx, (int)h_cnt3[4 * wait_slot + 2]);
                    }
                    break;
                }
                if (L > max_launch) {
                    HIPCHK(hipStreamSynchronize(st));
                    err = "adjoint forward exceeded the launch limit";
                    return FLOOD_ESTATE;
                }
                if (inflight == 0) {
                    ahead = 0;
                    int n = next_batch();
                    if (n <= 0) {
                        CHK(roll(mx));
                        mx = 0;
                        n = next_batch();
                    }
                    if (n <= 0) {   // cannot happen: a segment holds a step of every member
                        err = "adjoint tape segment overflow";
                        return FLOOD_ESTATE;
                    }
                    CHK(launch_fwd_batch(next, n));
                    batch_n[next] = n;
                    next ^= 1;
                    inflight = 1;
                }
            }
            launch_plan<T>(PLg, st);   // misfit of the samples completed by the last steps
            HIPCHK(hipMemcpyAsync(seg_n + (size_t)seg * Gi, d_segcnt, (size_t)Gi * sizeof(int32_t),
                                  hipMemcpyDeviceToDevice, st));
            seg_nmax.push_back(mx);
            // the members' end states back into the handle
            launch_tape_gather<T>(TV, d_curblk, V, par, st);
            {
                std::vector<double> lm(Gg);
                std::vector<int64_t> sn(Gg);
                HIPCHK(hipMemcpyAsync(lm.data(), d_lossm, Gg * sizeof(double), hipMemcpyDeviceToHost, st));
                HIPCHK(hipMemcpyAsync(sn.data(), steps + off + g0, Gg * sizeof(int64_t), hipMemcpyDeviceToHost, st));
                HIPCHK(hipStreamSynchronize(st));
                for (int m = 0; m < Gg; ++m) loss_slot[g0 + m] = lm[m];
                // the next group's members are expected to take no more steps than these
                int64_t most = 0;
                for (int m = 0; m < Gg; ++m) most = std::max(most, sn[m] - steps0[g0 + m]);
                g_next = adj_group_size(pool, (int)std::min<int64_t>(most, ckpt_every), Bm, Gi);
            }
            n_segments += (int)seg_nmax.size();

            // Reverse, segment by segment from the last, each member walking back
            // through its own steps (reverse launch i of a segment reverses step
            // n[k] - 1 - i of member k), so every launch carries every member that
            // has steps left.  Earlier segments are first recomputed from their
            // checkpoints, member by member in the same way, into the same blocks.
            HIPCHK(hipMemsetAsync(lam, 0, 2 * slot_elems * sizeof(T), st));
            HIPCHK(hipMemsetAsync(d_mubar, 0, (size_t)nblk * Gi * sizeof(double), st));
            HIPCHK(hipMemsetAsync(d_lpar, 0, (size_t)Gi * sizeof(int32_t), st));
            HIPCHK(hipMemsetAsync(d_nacc, 0, (size_t)((Gg + 3) / 4) * ncell * sizeof(T), st));
            T* lb[2] = {lam, lam + slot_elems};
            int rev_order = kAdjReverseOrder;
            if (const char* ao = std::getenv("FLOOD_ADJ_ORDER")) rev_order = std::min(4, std::max(0, std::atoi(ao)));
            const int last_seg = (int)seg_nmax.size() - 1;
            for (int sg = last_seg; sg >= 0; --sg) {
                const int nmax = seg_nmax[sg];
                const MemberStep<T>* recs = rec_at(sg);
                const int32_t* nseg = seg_n + (size_t)sg * Gi;
                if (nmax == 0) {   // no member stepped: only the adjoint copy indices move on
                    launch_adj_segment<T>(Gg, Gi, sg == last_seg ? nullptr : nseg + Gi, nseg, recs,
                                          rec_tag + (size_t)sg * seg_recs, 0, d_grc2, d_obs2, tape, plane, C.nx,
                                          d_lpar, lb[0], lb[1], st);
                    continue;
                }
                if (sg != (int)seg_nmax.size() - 1) {
                    CHK(ckpt_copy(static_cast<T*>(adj_ckpt[sg].p), false));
                    for (int r = 0; r < nmax; ++r) {
                        StepLaunch<T> R = SLm;
                        R.c[0] = TVR;
                        R.ms = recs + (size_t)r * Gi - (off + g0);
                        R.clamp_out = nullptr;
                        launch_marchv_rec<T>(R, 0, tw, st);
                    }
                }
                launch_adj_segment<T>(Gg, Gi, sg == last_seg ? nullptr : nseg + Gi, nseg, recs,
                                      rec_tag + (size_t)sg * seg_recs, K, d_grc2, d_obs2, tape, plane, C.nx, d_lpar,
                                      lb[0], lb[1], st);
                AdjvLaunch<T> A{};
                A.c = TV;
                A.c.march_order = rev_order;
                for (int w = 0; w < 2; ++w) {
                    A.lh[w] = lb[w];
                    A.lqx[w] = lb[w] + elemsG;
                    A.lqy[w] = lb[w] + 2 * elemsG;
                    A.lqw[w] = lb[w] + 3 * elemsG;
                    A.lqn[w] = lb[w] + 3 * elemsG + wG;
                }
                A.stride = Gi;
                A.n = nseg;
                A.lbase = d_lpar;
                A.rec = recs;
                A.rec_rdt = rec_rdt + (size_t)sg * seg_recs;
                A.rec_tag = rec_tag + (size_t)sg * seg_recs;
                A.n_gauges = K;
                A.grc = d_grc2;
                A.obs = d_obs2;
                A.nacc = d_nacc;
                A.mubar_part = d_mubar;
                for (int i = 0; i < nmax; ++i) {
                    A.i = i;
                    launch_adjoint_march<T>(A, st);
                }
                HIPCHK(hipGetLastError());
            }
            launch_nacc_reduce<T>((Gg + 3) / 4, ncell, d_nacc, d_nbar, st);
            launch_sum_parts(V.strips_xa * V.strips_y, Gg, d_mubar, d_gm + g0, st);
            HIPCHK(hipGetLastError());
            HIPCHK(hipStreamSynchronize(st));
            continue;
        }

        // ---------------- forward with record and checkpoints ----------------
        std::vector<T*> ckpts;
        int64_t L = 0;
        CHK(grow_log(4096));
        HIPCHK(hipMemsetAsync(any_log, 0, log_cap * sizeof(int32_t), st));
        for (int smp = 0; smp < S; ++smp) {
            *h_tend = t0 + (double)(smp + 1) * sample_dt;
            HIPCHK(hipMemcpyAsync(d_tend, h_tend, sizeof(double), hipMemcpyHostToDevice, st));
            HIPCHK(hipStreamSynchronize(st));
            for (;;) {
                const int B = 4;
                CHK(grow_log((size_t)L + B + 1));
                for (int i = 0; i < B; ++i) {
                    if (L % ckpt_every == 0) {
                        T* ck;
                        CHK(checkpoint((int)ckpts.size(), &ck));
                        ckpts.push_back(ck);
                        T* ch[2] = {ck, ck};
                        T* cx[2] = {ck + elemsG, ck + elemsG};
                        T* cyy[2] = {ck + 2 * elemsG, ck + 2 * elemsG};
                        T* cw[2] = {ck + 3 * elemsG, ck + 3 * elemsG};
                        T* cn[2] = {ck + 3 * elemsG + wG, ck + 3 * elemsG + wG};
                        CatchDev<T> D = group_view(C.dev, mi, g0, Gg, ch, cx, cyy, cw, cn);
                        launch_snapshot<T>(mi, V, par, D, st);
                    }
                    PLg.ms_log = ms_log + (size_t)L * Gi;
                    PLg.rdt_log = rdt_log + (size_t)L * Gi;
                    PLg.tag_log = tag_log + (size_t)L * Gi;
                    PLg.any_log = any_log + L;
                    PLg.tag_value = smp;
                    launch_plan<T>(PLg, st);
                    launch_step_mi<T>(mi, SLg, st);
                    ++L;
                }
                launch_count_active(Gg, t + off + g0, fault + off + g0, d_tend, status, nullptr, nullptr, nullptr, d_count, st);
                HIPCHK(hipGetLastError());
                HIPCHK(hipMemcpyAsync(h_count, d_count, 2 * sizeof(int32_t), hipMemcpyDeviceToHost, st));
                HIPCHK(hipStreamSynchronize(st));
                if (h_count[1]) {
                    err = "a member's depth became non-finite or too large to advance its clock during the adjoint forward";
                    return FLOOD_ENUMERIC;
                }
                if (h_count[0] == 0) break;
                if (L > max_launch) {
                    err = "adjoint forward exceeded the launch limit";
                    return FLOOD_ESTATE;
                }
            }
            launch_misfit<T>(mi, V, par, K, d_grc2, d_obs2 + (size_t)smp * K, d_loss + g0, st);
        }
        std::vector<int32_t> any_h(L);
        HIPCHK(hipMemcpyAsync(any_h.data(), any_log, L * sizeof(int32_t), hipMemcpyDeviceToHost, st));
        HIPCHK(hipStreamSynchronize(st));

        // ---------------- reverse sweep ----------------
        HIPCHK(hipMemsetAsync(lam, 0, 2 * slot_elems * sizeof(T), st));
        HIPCHK(hipMemsetAsync(d_mubar, 0, (size_t)nblk * Gi * sizeof(double), st));
        int cur = 0;
        auto lam_view = [&](int which, T** lh, T** lqx, T** lqy, T** lqw, T** lqn) {
            T* b = lam + (size_t)which * slot_elems;
            *lh = b;
            *lqx = b + elemsG;
            *lqy = b + 2 * elemsG;
            *lqw = b + 3 * elemsG;
            *lqn = b + 3 * elemsG + wG;
        };
        const int n_ck = (int)ckpts.size();
        for (int ck = n_ck - 1; ck >= 0; --ck) {
            const int64_t L0 = (int64_t)ck * ckpt_every;
            const int64_t L1 = std::min<int64_t>(L0 + ckpt_every, L);
            std::vector<int64_t> useful;
            for (int64_t l = L0; l < L1; ++l)
                if (any_h[l]) useful.push_back(l);
            if (useful.empty()) continue;
            HIPCHK(hipMemcpyAsync(tape, ckpts[ck], slot_elems * sizeof(T), hipMemcpyDeviceToDevice, st));
            const int n = (int)useful.size();
            for (int j = 0; j < n; ++j) {
                StepLaunch<T> R = SLg;
                R.recompute = 1;
                R.c[0] = slot_view(tape, j);
                R.c[0].groups = 1;
                R.c[0].chunks_per_group = R.c[0].n_chunks;
                R.c[0].n_blocks = R.c[0].tiles_x * R.c[0].tiles_y;
                R.total_blocks = R.c[0].n_blocks;
                R.ms = ms_log + (size_t)useful[j] * Gi - (off + g0);
                R.clamp_out = clamp + (size_t)j * elemsG;
                launch_step_mi<T>(mi, R, st);
            }
            for (int j = n - 1; j >= 0; --j) {
                const int64_t l = useful[j];
                CatchDev<T> after = slot_view(tape, j + 1);
                T *lh0, *lqx0, *lqy0, *lqw0, *lqn0, *lh1, *lqx1, *lqy1, *lqw1, *lqn1;
                lam_view(cur, &lh0, &lqx0, &lqy0, &lqw0, &lqn0);
                lam_view(cur ^ 1, &lh1, &lqx1, &lqy1, &lqw1, &lqn1);
                launch_inject<T>(mi, after, tag_log + (size_t)l * Gi, K, d_grc2, d_obs2, lh0, st);
                AdjLaunch<T> A{};
                A.c = slot_view(tape, j);
                A.lh[0] = lh0;
                A.lh[1] = lh1;
                A.lqx[0] = lqx0;
                A.lqx[1] = lqx1;
                A.lqy[0] = lqy0;
                A.lqy[1] = lqy1;
                A.lqw[0] = lqw0;
                A.lqw[1] = lqw1;
                A.lqn[0] = lqn0;
                A.lqn[1] = lqn1;
                A.clamp = clamp + (size_t)j * elemsG;
                A.ms = ms_log + (size_t)l * Gi;
                A.rdt = rdt_log + (size_t)l * Gi;
                A.nbar = d_nbar;
                A.mubar_part = d_mubar;
                launch_adjoint_step<T>(mi, A, st);
                cur ^= 1;
            }
            HIPCHK(hipGetLastError());
        }
        launch_sum_parts(nblk, Gg, d_mubar, d_gm + g0, st);
        HIPCHK(hipGetLastError());
        HIPCHK(hipStreamSynchronize(st));
    }
    if (!march_adj) {
        HIPCHK(hipMemcpyAsync(loss_slot.data(), d_loss, (size_t)N * sizeof(double), hipMemcpyDeviceToHost, st));
        HIPCHK(hipStreamSynchronize(st));
    }
    double loss_h = 0.0;
    for (int m = 0; m < N; ++m) loss_h += loss_slot[inv[m]];   // member order
    last_adj_groups = groups_run;
    last_adj_group_size = group_most;
    last_adj_segments = n_segments;
    if (grad_n_out) HIPCHK(hipMemcpyAsync(grad_n_out, d_nbar, ncell * sizeof(double), hipMemcpyDeviceToHost, st));
    std::vector<double> gm_slot(N);
    HIPCHK(hipMemcpyAsync(gm_slot.data(), d_gm, N * sizeof(double), hipMemcpyDeviceToHost, st));
    HIPCHK(hipStreamSynchronize(st));
    if (grad_mult_out)
        for (int i = 0; i < N; ++i) grad_mult_out[order[i]] = gm_slot[i];
    if (reordered) {
        restore.armed = false;
        CHK(reorder_members(c, inv, err));
    }
    if (loss_out) *loss_out = loss_h;
    (void)gm_host;
    return FLOOD_OK;
}

flood_status create_impl(flood_handle* h, int n_catch, const flood_grid* grids, const flood_params* params,
                         const int32_t* members, const double* const* n_scale, const double* const* rain_mult,
                         hipStream_t stream, std::string& err) {
    int ndev = 0;
    hipError_t e = hipGetDeviceCount(&ndev);
    if (e != hipSuccess || ndev < 1) {
        (void)hipGetLastError();
        err = "no HIP device available";
        return FLOOD_EHIP;
    }
    if (params[0].real_bytes == 8) {
        auto* I = new Impl<double>();
        h->impl.reset(I);
        flood_status st = I->init(n_catch, grids, params, members, n_scale, rain_mult, stream, err);
        if (st) h->impl.reset();
        return st;
    }
    auto* I = new Impl<float>();
    h->impl.reset(I);
    flood_status st = I->init(n_catch, grids, params, members, n_scale, rain_mult, stream, err);
    if (st) h->impl.reset();
    return st;
}

flood_status systematic_resample_impl(const double* w, int n, double u0, int32_t* anc, hipStream_t s) {
    double* dw = nullptr;
    int32_t* da = nullptr;
    if (hipMalloc((void**)&dw, n * sizeof(double)) != hipSuccess) return FLOOD_ENOMEM;
    if (hipMalloc((void**)&da, n * sizeof(int32_t)) != hipSuccess) {
        (void)hipFree(dw);
        return FLOOD_ENOMEM;
    }
    flood_status rc = FLOOD_OK;
    if (hipMemcpyAsync(dw, w, n * sizeof(double), hipMemcpyHostToDevice, s) != hipSuccess) rc = FLOOD_EHIP;
    if (!rc) {
        launch_systematic(n, dw, u0, da, s);
        if (hipGetLastError() != hipSuccess) rc = FLOOD_EHIP;
    }
    if (!rc && hipMemcpyAsync(anc, da, n * sizeof(int32_t), hipMemcpyDeviceToHost, s) != hipSuccess) rc = FLOOD_EHIP;
    if (!rc && hipStreamSynchronize(s) != hipSuccess) rc = FLOOD_EHIP;
    (void)hipFree(dw);
    (void)hipFree(da);
    return rc;
}

}  // namespace flood
