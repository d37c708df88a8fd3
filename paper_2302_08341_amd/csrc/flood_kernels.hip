// Forward kernels of libflood for gfx950: step planner, fused link + continuity
// step with the per-member depth maximum, and state utilities.
//
// The step is memory-bound (about 60 flops per 24 bytes per member-cell), so it
// uses plain vector ALU work with coalesced structure-of-arrays streams and no
// matrix cores.  All kernels are compiled with FP contraction off, so every
// link is evaluated with the same rounding wherever it is computed (a link
// shared by two cells is computed by both, identically).
#include <cfloat>
#include <cmath>
#include <type_traits>

#include "flood_device.h"

namespace flood {

// ---------------------------------------------------------------------------
// step planner: per-member Eq. 4 step, clipped to rain-block edges and t_end
// ---------------------------------------------------------------------------
// One wavefront per member: lane k folds depth-maximum bin k (kBins = 64) and
// the lanes share the gauge misfit; the plan itself is the same scalar work on
// every lane, written out by lane 0.
template <typename T>
__global__ __launch_bounds__(256) void k_plan(const PlanLaunch<T> P) {
    using HB = typename HBits<T>::type;
    static_assert(kBins == 64, "one depth-maximum bin per lane");
    const int lane = threadIdx.x & 63;
    const int m = P.m_begin + blockIdx.x * (blockDim.x >> 6) + (int)(threadIdx.x >> 6);
    if (m >= P.m_end) return;
    const bool w0 = lane == 0;
    int ci = 0;
    for (int i = 1; i < P.n_catch; ++i)
        if (m >= P.c[i].member_off) ci = i;
    const PlanCatch& C = P.c[ci];
    const int lm = m - P.m_begin;
    // The loads of the plan that depend on nothing else go out together, before
    // any store (a planner is a chain of memory round trips, not of arithmetic).
    const int par = P.par[m];
    const double t = P.t[m];
    const double t_end = *P.t_end;
    const int fault = P.fault[m];
    const int64_t st = P.steps[m];
    const bool at_lim = P.step_lim && st >= P.step_lim[m];
    HB hb = P.hbins[(size_t)lane * P.n_total + m];
    const int pend = P.pend ? P.pend[lm] : -1;
    const int cb = P.cur_blk ? P.cur_blk[lm] : 0;
    const int nsmp = P.s_dt > 0.0 ? P.smp[lm] : 0;
    const int nseg = P.seg_cnt ? P.seg_cnt[lm] : 0;
    const double sc = P.s[m];
    const double mu = P.mu[m];
    const double jf = floor(t / C.rain_interval);
    const double R = (jf >= 0.0 && jf < (double)C.n_rain) ? C.rain[(int64_t)jf] : 0.0;
    MemberStep<T> ms;
    ms.dtdx = ms.gdtdx = ms.gdt = ms.s2dt = ms.capf = ms.rinc = T(0);
    ms.dxdt = 0.0;
    ms.active = 0;
    ms.parity = par;
    ms.slot = ms.blk = ms.blk_next = -1;
    ms.seed = 0;
    for (int k = 0; k < kMaxClasses; ++k) ms.cn[k] = T(0);
    ms.drain = T(0);
    for (int k = 0; k < kMaxSeries; ++k) ms.qin[k] = T(0);
    if (pend >= 0) {
        // misfit of the state after the member's last step, which completed sample pend
        const T* h = P.tape_h + (size_t)cb * P.plane;
        double acc = 0.0;
        for (int q = lane; q < P.n_gauges; q += 64) {
            const double d = (double)h[(size_t)P.grc[2 * q] * P.nx + P.grc[2 * q + 1]] -
                             P.obs[(size_t)pend * P.n_gauges + q];
            acc += d * d;
        }
        for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
        if (w0) {
            P.loss_m[lm] += acc;
            P.pend[lm] = -1;
        }
    }
    if (fault || !(t < t_end) || at_lim) {
        if (w0) {
            P.ms[m] = ms;
            if (P.ms_log && !P.rec_stride) {
                P.ms_log[lm] = ms;
                P.rdt_log[lm] = 0.0;
                P.tag_log[lm] = -1;
            }
        }
        return;
    }
    for (int off = 32; off > 0; off >>= 1) {
        const HB o = __shfl_xor(hb, off, 64);
        hb = o > hb ? o : hb;
    }
    const T H = from_bits<T>(hb);
    const auto freeze = [&]() {
        if (w0) {
            P.fault[m] = 1;
            atomicOr(P.status, 1);
            P.ms[m] = ms;
            if (P.ms_log && !P.rec_stride) {
                P.ms_log[lm] = ms;
                P.rdt_log[lm] = 0.0;
                P.tag_log[lm] = -1;
            }
        }
    };
    if (!(H <= (sizeof(T) == 4 ? T(FLT_MAX) : T(DBL_MAX)))) {
        freeze();
        return;
    }
    double dt;
    if (C.dt_fixed > 0.0) {
        dt = C.dt_fixed;
    } else {
        double Hd = (double)H;
        if (Hd < C.hdry) Hd = C.hdry;
        dt = C.alpha * C.dx / sqrt(C.g * Hd);
        if (dt > C.dt_cap) dt = C.dt_cap;
    }
    const double edge = (jf + 1.0 > (double)C.n_rain) ? INFINITY : (jf + 1.0) * C.rain_interval;
    double tev = t_end < edge ? t_end : edge;
    const double ts = P.s_dt > 0.0 ? P.s_t0 + (double)(nsmp + 1) * P.s_dt : INFINITY;
    if (ts < tev) tev = ts;
    const double dt_free = dt;   // not cut to an event
    double tn;
    if (dt >= tev - t) {
        dt = tev - t;
        tn = tev;
    } else {
        tn = t + dt;
    }
    if (!(tn > t)) {
        // an Eq. 4 step below the resolution of the member's clock (a depth so
        // large that the member can no longer advance): a numeric fault too
        freeze();
        return;
    }
    // every lane has read its bin: clear it for the step's new maximum
    P.hbins[(size_t)lane * P.n_total + m] = 0;
    if (!w0) return;
    ms.dtdx = (T)(dt / C.dx);
    ms.gdtdx = (T)(C.g * dt / C.dx);
    ms.gdt = (T)(C.g * dt);
    ms.s2dt = (T)(sc * sc * dt);
    ms.capf = (T)(C.dx / (4.0 * dt));
    ms.rinc = (T)(mu * R * dt);
    ms.dxdt = C.dx * dt;
    ms.active = 1;
    {
        // the step's random bits follow from the member's time: a state set back
        // to an earlier time replays the same rounding
        const uint64_t tb = (uint64_t)__double_as_longlong(t);
        ms.seed = mix32((uint32_t)tb ^ mix32((uint32_t)(tb >> 32) + 0x632be5abu));
    }
    if (P.seg_cnt) {
        // the member's new state goes to the next free block of the tape
        ms.slot = nseg;
        P.seg_cnt[lm] = nseg + 1;
        ms.blk = cb;
        ms.blk_next = atomicAdd(P.pool_next, 1);
        P.cur_blk[lm] = ms.blk_next;
    }
    if (P.clsn)
        for (int k = 0; k < kMaxClasses; ++k) ms.cn[k] = (T)P.clsn[(size_t)m * kMaxClasses + k];
    if (P.drain) ms.drain = (T)(P.drain[m] * dt);
    if (C.n_series > 0) {
        // inflow hydrographs: the series value of the current rain block
        double vq = 0.0;
        for (int j = 0; j < C.n_series; ++j) {
            const double q = (jf >= 0.0 && jf < (double)C.n_rain) ? C.inflow_q[(size_t)j * C.n_rain + (int64_t)jf]
                                                                     : 0.0;
            ms.qin[j] = (T)q;
            vq += C.wq[j] * q;
        }
        P.vin[m] += vq * dt;
    }
    P.ms[m] = ms;
    int tag = (tn == t_end) ? P.tag_value : -1;
    if (P.s_dt > 0.0) {
        tag = (tn == ts) ? nsmp : -1;
        if (tag >= 0) {
            P.smp[lm] = tag + 1;
            P.pend[lm] = tag;
        }
    }
    if (P.ms_log) {
        const size_t li = P.rec_stride ? (size_t)ms.slot * P.rec_stride + lm : (size_t)lm;
        P.ms_log[li] = ms;
        P.rdt_log[li] = R * dt;
        P.tag_log[li] = tag;
        if (P.any_log) P.any_log[0] = 1;
    }
    if (P.dtlog) {
        const int64_t li = P.log_n[m];
        if (li < P.dtlog_cap) {
            P.dtlog[(size_t)m * P.dtlog_cap + li] = dt;
            P.telog[(size_t)m * P.dtlog_cap + li] = tn;
        }
        P.log_n[m] = li + 1;
    }
    P.t[m] = tn;
    P.dt_last[m] = dt_free;
    P.par[m] = ms.parity ^ 1;
    P.steps[m] = st + 1;
    P.vrain[m] += (double)ms.rinc * C.ncells * (C.dx * C.dx);
}

template <typename T> void launch_plan(const PlanLaunch<T>& P, hipStream_t s) {
    const int n = P.m_end - P.m_begin;
    if (n > 0) hipLaunchKernelGGL(k_plan<T>, dim3((n + 3) / 4), dim3(256), 0, s, P);
}

// ---------------------------------------------------------------------------
// fused step: every link around a cell from (h^n, q^n), continuity with the
// new discharges and the rain depth, per-member maximum of the new depth.
// One lane per (cell, member-in-chunk); a workgroup covers a tile of cells for
// `chunks_per_group` consecutive member chunks, reusing the shared bed and
// roughness of its cells from registers.
// ---------------------------------------------------------------------------
template <typename T, int MI>
__global__ __launch_bounds__(kBlock) void k_step(const StepLaunch<T> L) {
    using HB = typename HBits<T>::type;
    const int b = xcd_remap(blockIdx.x, gridDim.x);
    int ci = 0;
    for (int i = 1; i < L.n_catch; ++i)
        if (b >= L.c[i].block_begin) ci = i;
    const CatchDev<T>& C = L.c[ci];
    const int lb = b - C.block_begin;
    const int grp = lb % C.groups;
    const int tile = lb / C.groups;
    const int tyi = tile / C.tiles_x;
    const int txi = tile - tyi * C.tiles_x;
    const int txl = C.tx_log2;
    const int lane = threadIdx.x % MI;
    const int p = threadIdx.x / MI;
    const int TY = (kBlock / MI) >> txl;
    const int nx = C.nx, ny = C.ny;
    const int cx = (txi << txl) + (p & ((1 << txl) - 1));
    const int cy = tyi * TY + (p >> txl);
    const bool in = cx < nx && cy < ny;
    const int k0 = grp * C.chunks_per_group;
    const int k1 = min(k0 + C.chunks_per_group, C.n_chunks);
    const int mend = min(k1 * MI, C.n_members);
    // Recompute mode (adjoint tape): every member reads copy 0 and writes copy 1, members that
    // do not step copy their state across, clamp flags are recorded, ledgers and the depth
    // maximum are left alone.
    const bool rec = L.recompute != 0;
    int any = rec ? 1 : 0;
    for (int m = k0 * MI + (int)threadIdx.x; m < mend && !rec; m += kBlock) any |= L.ms[C.member_off + m].active;
    if (!__syncthreads_or(any)) return;

    // shared bed and roughness of this cell and its four neighbours
    const bool hasE = cx + 1 < nx, hasW = cx > 0, hasS = cy + 1 < ny, hasN = cy > 0;
    const T g = C.g;
    T dzE = 0, dzW = 0, dzS = 0, dzN = 0, GE = 0, GW = 0, GS = 0, GN = 0;
    if (in) {
        const size_t c0 = (size_t)cy * nx + cx;
        const T z0 = C.z[c0], n0 = C.n[c0];
        const T gb = g * (n0 * n0);
        if (hasE) {
            const T z1 = C.z[c0 + 1], n1 = C.n[c0 + 1];
            const T nf = T(0.5) * (n0 + n1);
            dzE = z1 - z0;
            GE = g * (nf * nf);
        } else {
            GE = gb;
        }
        if (hasW) {
            const T z1 = C.z[c0 - 1], n1 = C.n[c0 - 1];
            const T nf = T(0.5) * (n1 + n0);
            dzW = z0 - z1;
            GW = g * (nf * nf);
        } else {
            GW = gb;
        }
        if (hasS) {
            const T z1 = C.z[c0 + nx], n1 = C.n[c0 + nx];
            const T nf = T(0.5) * (n0 + n1);
            dzS = z1 - z0;
            GS = g * (nf * nf);
        } else {
            GS = gb;
        }
        if (hasN) {
            const T z1 = C.z[c0 - nx], n1 = C.n[c0 - nx];
            const T nf = T(0.5) * (n1 + n0);
            dzN = z0 - z1;
            GN = g * (nf * nf);
        } else {
            GN = gb;
        }
    }
    const T hdry = C.hdry;
    const int nb = 2 * (nx + ny);
    const int bin = blockIdx.x & (kBins - 1);
    const size_t plane = (size_t)ny * nx * MI;
    const size_t rowMI = (size_t)nx * MI;

    for (int k = k0; k < k1; ++k) {
        const int ml = k * MI + lane;
        MemberStep<T> ms;
        bool act = false;
        if (ml < C.n_members) {
            ms = L.ms[C.member_off + ml];
            act = in && ms.active;
        }
        T hn = T(0);
        if (rec && in && ml < C.n_members && !act) {
            const size_t idx = (size_t)k * plane + ((size_t)cy * nx + cx) * MI + lane;
            C.h[1][idx] = C.h[0][idx];
            C.qx[1][idx] = C.qx[0][idx];
            C.qy[1][idx] = C.qy[0][idx];
            if (!hasW) C.qw[1][((size_t)k * ny + cy) * MI + lane] = C.qw[0][((size_t)k * ny + cy) * MI + lane];
            if (!hasN) C.qn[1][((size_t)k * nx + cx) * MI + lane] = C.qn[0][((size_t)k * nx + cx) * MI + lane];
            L.clamp_out[idx] = 0;
        }
        if (act) {
            const int sp = rec ? 0 : ms.parity, dp = sp ^ 1;
            const T* __restrict__ hs = C.h[sp];
            const T* __restrict__ qxs = C.qx[sp];
            const T* __restrict__ qys = C.qy[sp];
            const size_t idx = (size_t)k * plane + ((size_t)cy * nx + cx) * MI + lane;
            const T h0 = hs[idx];
            const T hE = hasE ? hs[idx + MI] : T(0);
            const T hW = hasW ? hs[idx - MI] : T(0);
            const T hS = hasS ? hs[idx + rowMI] : T(0);
            const T hN = hasN ? hs[idx - rowMI] : T(0);
            const T qE = qxs[idx];
            const T qS = qys[idx];
            const T qW = hasW ? qxs[idx - MI] : C.qw[sp][((size_t)k * ny + cy) * MI + lane];
            const T qN = hasN ? qys[idx - rowMI] : C.qn[sp][((size_t)k * nx + cx) * MI + lane];
            T fE, fS, fW, fN;
            if (hasE)
                fE = link_in(qE, h0, hE, dzE, GE, ms, hdry);
            else
                fE = C.edge_open[1] ? link_open(qE, h0, GE, C.edge_slope[1], ms, hdry) : T(0);
            if (hasS)
                fS = link_in(qS, h0, hS, dzS, GS, ms, hdry);
            else
                fS = C.edge_open[2] ? link_open(qS, h0, GS, C.edge_slope[2], ms, hdry) : T(0);
            if (hasW)
                fW = link_in(qW, hW, h0, dzW, GW, ms, hdry);
            else
                fW = C.edge_open[3] ? -link_open(-qW, h0, GW, C.edge_slope[3], ms, hdry) : T(0);
            if (hasN)
                fN = link_in(qN, hN, h0, dzN, GN, ms, hdry);
            else
                fN = C.edge_open[0] ? -link_open(-qN, h0, GN, C.edge_slope[0], ms, hdry) : T(0);
            // Eq. 1 with the four links of Sec. 3.1 (west/east x-links, north/south y-links)
            const T dv = ((fW - fE) + fN) - fS;
            hn = depth_add(h0, ms.dtdx * dv + ms.rinc, ms.seed, (uint32_t)(cy * nx + cx));
            const bool clamped = hn < T(0);
            if (clamped) {
                if (!rec) atomicAdd(&L.vclamp[C.member_off + ml], -(double)hn * (C.dx * C.dx));
                hn = T(0);
            }
            if (rec) L.clamp_out[idx] = clamped ? 1 : 0;
            if (hn == T(0)) hn = T(0);  // canonical +0 for the bit-pattern maximum
            C.h[dp][idx] = hn;
            if (!rec && C.peak) C.peak[idx] = fmax(C.peak[idx], hn);
            C.qx[dp][idx] = fE;
            C.qy[dp][idx] = fS;
            if (!hasW) C.qw[dp][((size_t)k * ny + cy) * MI + lane] = fW;
            if (!hasN) C.qn[dp][((size_t)k * nx + cx) * MI + lane] = fN;
            if (!rec && !(hasE && hasW && hasS && hasN)) {
                double* acc = C.out_acc + (size_t)ml * nb;
                if (!hasN && C.edge_open[0]) acc[cx] += -(double)fN * ms.dxdt;
                if (!hasS && C.edge_open[2]) acc[nx + cx] += (double)fS * ms.dxdt;
                if (!hasW && C.edge_open[3]) acc[2 * nx + cy] += -(double)fW * ms.dxdt;
                if (!hasE && C.edge_open[1]) acc[2 * nx + ny + cy] += (double)fE * ms.dxdt;
            }
        }
        // depth maximum per member over the wavefront, on the IEEE bit pattern
        // (depths are >= 0, and a NaN or Inf compares above every finite depth)
        HB v = to_bits(hn);
#pragma unroll
        for (int off = MI; off < 64; off <<= 1) {
            const HB o = __shfl_xor(v, off, 64);
            v = o > v ? o : v;
        }
        if (!rec && (threadIdx.x & 63) < MI && ml < C.n_members && v != 0) {
            HB* a = L.hbins + (size_t)bin * L.n_total + C.member_off + ml;
            const HB cur = __hip_atomic_load(a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (v > cur) atomicMax(a, v);
        }
    }
}

template <typename T, int MI> void launch_step(const StepLaunch<T>& L, hipStream_t s) {
    hipLaunchKernelGGL((k_step<T, MI>), dim3(L.total_blocks), dim3(kBlock), 0, s, L);
}

template <typename T> void launch_step_mi(int mi, const StepLaunch<T>& L, hipStream_t s) {
    switch (mi) {
        case 1: launch_step<T, 1>(L, s); break;
        case 2: launch_step<T, 2>(L, s); break;
        case 4: launch_step<T, 4>(L, s); break;
        default: launch_step<T, 8>(L, s); break;
    }
}

// ---------------------------------------------------------------------------
// members still short of t_end
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_count_active(int n, const double* t, const int32_t* fault,
                                                      const double* t_end, const int32_t* status,
                                                      const int64_t* steps, const int64_t* lim, const double* dt,
                                                      int32_t* out) {
    __shared__ int part[4], mpart[4];
    int c = 0, need = 0;
    const double te = *t_end;
    for (int m = threadIdx.x; m < n; m += 256) {
        if (fault[m] || !(t[m] < te) || (lim && steps[m] >= lim[m])) continue;
        ++c;
        if (dt) {
            // an estimate: the step length follows the depth and shortens before block edges
            double k = dt[m] > 0.0 ? ceil((te - t[m]) / dt[m]) : 1.0;
            if (lim && (double)(lim[m] - steps[m]) < k) k = (double)(lim[m] - steps[m]);
            need = max(need, (int)fmin(k, 1e9));
        }
    }
    for (int off = 32; off > 0; off >>= 1) {
        c += __shfl_xor(c, off, 64);
        need = max(need, __shfl_xor(need, off, 64));
    }
    if ((threadIdx.x & 63) == 0) {
        part[threadIdx.x >> 6] = c;
        mpart[threadIdx.x >> 6] = need;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        out[0] = part[0] + part[1] + part[2] + part[3];
        out[1] = status[0];
        if (dt) out[2] = max(max(mpart[0], mpart[1]), max(mpart[2], mpart[3]));
    }
}

void launch_count_active(int n_total, const double* t, const int32_t* fault, const double* t_end,
                         const int32_t* status, const int64_t* steps, const int64_t* lim, const double* dt, int32_t* out,
                         hipStream_t s) {
    hipLaunchKernelGGL(k_count_active, dim3(1), dim3(256), 0, s, n_total, t, fault, t_end, status, steps, lim, dt, out);
}

__global__ __launch_bounds__(256) void k_count_group(int n, const double* t, const int32_t* fault,
                                                     const double* t_end, const int32_t* status,
                                                     const int32_t* seg_cnt, const double* dt, const int32_t* smp,
                                                     double s_t0, double s_dt,
                                                     int32_t* out) {
    __shared__ int part[4], mpart[4], npart[4];
    int c = 0, mx = 0, need = 0;
    const double te = *t_end;
    for (int m = threadIdx.x; m < n; m += 256) {
        mx = max(mx, seg_cnt[m]);
        if (fault[m] || !(t[m] < te)) continue;
        ++c;
        if (!(dt[m] > 0.0)) continue;
        // to the member's next sample, then whole sample intervals, at its last step length
        const double ts = fmin(s_t0 + (double)(smp[m] + 1) * s_dt, te);
        const double k = ceil((ts - t[m]) / dt[m]) + rint((te - ts) / s_dt) * ceil(s_dt / dt[m]);
        need = max(need, (int)fmin(k, 1e9));
    }
    for (int off = 32; off > 0; off >>= 1) {
        c += __shfl_xor(c, off, 64);
        mx = max(mx, __shfl_xor(mx, off, 64));
        need = max(need, __shfl_xor(need, off, 64));
    }
    if ((threadIdx.x & 63) == 0) {
        part[threadIdx.x >> 6] = c;
        mpart[threadIdx.x >> 6] = mx;
        npart[threadIdx.x >> 6] = need;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        out[0] = part[0] + part[1] + part[2] + part[3];
        out[1] = status[0];
        out[2] = max(max(mpart[0], mpart[1]), max(mpart[2], mpart[3]));
        out[3] = max(max(npart[0], npart[1]), max(npart[2], npart[3]));
    }
}

void launch_count_group(int G, const double* t, const int32_t* fault, const double* t_end, const int32_t* status,
                        const int32_t* seg_cnt, const double* dt, const int32_t* smp, double s_t0, double s_dt,
                        int32_t* out, hipStream_t s) {
    hipLaunchKernelGGL(k_count_group, dim3(1), dim3(256), 0, s, G, t, fault, t_end, status, seg_cnt, dt, smp, s_t0,
                       s_dt, out);
}

__global__ __launch_bounds__(256) void k_step_limit(int n, const int64_t* steps, int64_t add, int64_t* lim) {
    const int m = blockIdx.x * blockDim.x + threadIdx.x;
    if (m < n) lim[m] = add < 0 ? INT64_MAX : steps[m] + add;
}

void launch_step_limit(int n_total, const int64_t* steps, int64_t n, int64_t* lim, hipStream_t s) {
    hipLaunchKernelGGL(k_step_limit, dim3((n_total + 255) / 256), dim3(256), 0, s, n_total, steps, n, lim);
}

template <typename HB> __global__ __launch_bounds__(256) void k_zero_bins(int off, int n, int n_total, HB* bins) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n * kBins) return;
    bins[(size_t)(e / n) * n_total + off + e % n] = 0;
}

template <typename HB> void launch_zero_bins(int off, int n, int n_total, HB* bins, hipStream_t s) {
    hipLaunchKernelGGL(k_zero_bins<HB>, dim3((n * kBins + 255) / 256), dim3(256), 0, s, off, n, n_total, bins);
}

// After resampling slot j holds a copy of member anc[j]: its depth maximum follows.
template <typename HB>
__global__ __launch_bounds__(1024) void k_permute_bins(int off, int n, int n_total, HB* bins, const int32_t* anc,
                                                       const int32_t* flag) {
    if (flag[0] == 0) return;
    const int j = threadIdx.x;
    HB v = 0;
    if (j < n) {
        const int a = anc[j];
        for (int b = 0; b < kBins; ++b) {
            const HB x = bins[(size_t)b * n_total + off + a];
            v = x > v ? x : v;
        }
    }
    __syncthreads();
    if (j < n)
        for (int b = 0; b < kBins; ++b) bins[(size_t)b * n_total + off + j] = b == 0 ? v : HB(0);
}

template <typename HB>
void launch_permute_bins(int off, int n, int n_total, HB* bins, const int32_t* anc, const int32_t* flag,
                         hipStream_t s) {
    hipLaunchKernelGGL(k_permute_bins<HB>, dim3(1), dim3(((n + 63) / 64) * 64), 0, s, off, n, n_total, bins, anc,
                       flag);
}

template void launch_zero_bins<uint32_t>(int, int, int, uint32_t*, hipStream_t);
template void launch_zero_bins<unsigned long long>(int, int, int, unsigned long long*, hipStream_t);
template void launch_permute_bins<uint32_t>(int, int, int, uint32_t*, const int32_t*, const int32_t*, hipStream_t);
template void launch_permute_bins<unsigned long long>(int, int, int, unsigned long long*, const int32_t*,
                                                      const int32_t*, hipStream_t);

// ---------------------------------------------------------------------------
// element-wise helpers over one catchment: lane = (cell, member)
// ---------------------------------------------------------------------------
// Depth maximum of the current state into bin 0 (bins must be zero);
// blockIdx.y = member.
template <typename T, int MI>
__global__ __launch_bounds__(256) void k_hmax_init(const CatchDev<T> C, const int32_t* par,
                                                   typename HBits<T>::type* hbins, int n_total) {
    using HB = typename HBits<T>::type;
    const int m = blockIdx.y;
    const size_t ncell = (size_t)C.ny * C.nx;
    const T* h = C.h[par[C.member_off + m]];
    HB best = 0;
    for (size_t cell = (size_t)blockIdx.x * blockDim.x + threadIdx.x; cell < ncell;
         cell += (size_t)gridDim.x * blockDim.x) {
        const int r = (int)(cell / C.nx), c = (int)(cell % C.nx);
        const HB bv = to_bits(h[state_index<T, MI>(C, m, r, c)] + T(0));
        best = bv > best ? bv : best;
    }
    for (int off = 32; off > 0; off >>= 1) {
        const HB o = __shfl_xor(best, off, 64);
        best = o > best ? o : best;
    }
    if ((threadIdx.x & 63) == 0 && best != 0) atomicMax(hbins + C.member_off + m, best);
}

template <typename T>
void launch_hmax_init(int mi, const CatchDev<T>& C, const int32_t* par, typename HBits<T>::type* hbins,
                      int n_total, hipStream_t s) {
    const size_t ncell = (size_t)C.ny * C.nx;
    dim3 grid((unsigned)std::min<size_t>((ncell + 255) / 256, 512), C.n_members);
    switch (mi) {
        case 1: hipLaunchKernelGGL((k_hmax_init<T, 1>), grid, dim3(256), 0, s, C, par, hbins, n_total); break;
        case 2: hipLaunchKernelGGL((k_hmax_init<T, 2>), grid, dim3(256), 0, s, C, par, hbins, n_total); break;
        case 4: hipLaunchKernelGGL((k_hmax_init<T, 4>), grid, dim3(256), 0, s, C, par, hbins, n_total); break;
        default: hipLaunchKernelGGL((k_hmax_init<T, 8>), grid, dim3(256), 0, s, C, par, hbins, n_total); break;
    }
}

// Storage sum(h) dx^2 per member, added into out[member] (out must be zero).
// Bound by the read of the depths.  A few workgroups per member, each over many
// cells: their sums meet in atomics on one or two cache lines, about 20 ns apiece,
// and with one workgroup per 256 cells those were the whole time (1024 x 1024 x 16:
// 320 us then, 46 now; 2000 x 2000 x 96: 725, 257, 6.0 TB/s).  Independent partial
// sums for the cells of a vector; cells of a member lie `mi` apart.
template <typename T, int V>
__global__ __launch_bounds__(256) void k_storage(const CatchDev<T> C, int mi, const int32_t* par, double* out) {
    const int m = blockIdx.y;
    const size_t ncell = (size_t)C.ny * C.nx;
    const T* h = C.h[par[C.member_off + m]] + (size_t)(m / mi) * ncell * mi + m % mi;
    double acc[V] = {};
    const size_t nv = V == 1 ? ncell : ncell / V;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < nv; e += stride) {
        if constexpr (V > 1) {
            T v[V];
            vload<T, V>(h + e * V, v);
#pragma unroll
            for (int j = 0; j < V; ++j) acc[j] += (double)v[j];
        } else {
            acc[0] += (double)h[e * mi];
        }
    }
    double sum = 0.0;
#pragma unroll
    for (int j = 0; j < V; ++j) sum += acc[j];
    for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off, 64);
    __shared__ double part[4];
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = sum;
    __syncthreads();
    if (threadIdx.x == 0) atomicAdd(out + m, ((part[0] + part[1]) + (part[2] + part[3])) * (C.dx * C.dx));
}

template <typename T>
void launch_storage(int mi, const CatchDev<T>& C, const int32_t* par, double* out, hipStream_t s) {
    constexpr int V = march_vec<T>();
    const size_t ncell = (size_t)C.ny * C.nx;
    // whole vectors of cells in every member's plane
    const bool vec = mi == 1 && ncell % V == 0;
    const size_t per = (ncell / (vec ? V : 1) + 255) / 256;
    const size_t want = (size_t)std::max(8, 4096 / C.n_members);
    dim3 grid((unsigned)std::max<size_t>(1, std::min(per, want)), C.n_members);
    if (vec) hipLaunchKernelGGL((k_storage<T, V>), grid, dim3(256), 0, s, C, mi, par, out);
    else hipLaunchKernelGGL((k_storage<T, 1>), grid, dim3(256), 0, s, C, mi, par, out);
}

// Elements [e0, e0 + count) of one member's field in the host layout (H: ny*nx, QX:
// ny*(nx+1), QY: (ny+1)*nx), buf[0] the first of them.  The member's current copy is
// read from par (null: copy 0).
template <typename T>
__global__ __launch_bounds__(256) void k_field(const CatchDev<T> C, int mi, int m, const int32_t* par, int which,
                                               size_t e0, size_t count, double* buf, int to_state) {
    const int ny = C.ny, nx = C.nx;
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= count) return;
    const int p = par ? par[C.member_off + m] : 0;
    const size_t e = e0 + i;
    const size_t k = m / mi, lane = m % mi, ncell = (size_t)ny * nx;
    auto at = [&](T* base, size_t cell) { return base + (k * ncell + cell) * mi + lane; };
    T* ptr;
    if (which == 3) {
        ptr = at(C.peak, e);
    } else if (which == 0) {
        ptr = at(C.h[p], e);
    } else if (which == 1) {
        const size_t r = e / (nx + 1), c = e % (nx + 1);
        ptr = c == 0 ? C.qw[p] + (k * ny + r) * mi + lane : at(C.qx[p], r * nx + c - 1);
    } else {
        ptr = e < (size_t)nx ? C.qn[p] + (k * nx + e) * mi + lane : at(C.qy[p], e - nx);
    }
    if (to_state)
        *ptr = (T)buf[i] + T(0);
    else
        buf[i] = (double)*ptr;
}

template <typename T>
void launch_get_field(int mi, const CatchDev<T>& C, int member, const int32_t* par, int which, size_t e0, size_t count,
                      double* out, hipStream_t s) {
    hipLaunchKernelGGL((k_field<T>), dim3((unsigned)((count + 255) / 256)), dim3(256), 0, s, C, mi, member, par, which,
                       e0, count, out, 0);
}
template <typename T>
void launch_set_field(int mi, const CatchDev<T>& C, int member, const int32_t* par, int which, const double* in,
                      hipStream_t s) {
    const size_t n = (which == 0 || which == 3) ? (size_t)C.ny * C.nx
                     : which == 1               ? (size_t)C.ny * (C.nx + 1)
                                                : (size_t)(C.ny + 1) * C.nx;
    hipLaunchKernelGGL((k_field<T>), dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, C, mi, member, par, which, 0, n,
                       const_cast<double*>(in), 1);
}

// One launch for the some thirty arrays of a handle's state: as copy commands they
// took 2 to 5 us each with as much between them, which on a small grid was most of a
// snapshot's time.  Bound by the copy itself past some 10 MB (5.3 TB/s, read and
// written, at 2000 x 2000 x 96: 3.5 ms from 4.4; 1024 x 1024 x 16: 0.28 from 0.95).
// A workgroup copies 32 KiB of one array, 16 bytes a lane with eight in flight.
constexpr uint32_t kCopyBytes = 256 * 16 * 8;

__global__ __launch_bounds__(256) void k_copy_list(const CopyList L) {
    typedef uint32_t __attribute__((ext_vector_type(4))) u4;
    int i = 0;
    while (i + 1 < L.n && blockIdx.x >= L.item[i + 1].block0) ++i;
    const CopyList::Item& it = L.item[i];
    const uint64_t o = (uint64_t)(blockIdx.x - it.block0) * kCopyBytes;
    const uint64_t left = it.bytes - o;
    const char* src = static_cast<const char*>(it.src) + o;
    char* dst = static_cast<char*>(it.dst) + o;
    if (blockIdx.x == 0 && threadIdx.x == 0 && L.clear) *L.clear = 0;
    if (left >= kCopyBytes && (((uintptr_t)src | (uintptr_t)dst) & 15) == 0) {
        u4 v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = reinterpret_cast<const u4*>(src)[j * 256 + threadIdx.x];
#pragma unroll
        for (int j = 0; j < 8; ++j) reinterpret_cast<u4*>(dst)[j * 256 + threadIdx.x] = v[j];
        return;
    }
    const uint32_t words = (uint32_t)((left < kCopyBytes ? left : kCopyBytes) / 4);
    for (uint32_t w = threadIdx.x; w < words; w += 256)
        reinterpret_cast<uint32_t*>(dst)[w] = reinterpret_cast<const uint32_t*>(src)[w];
}

void launch_copy_list(CopyList& L, hipStream_t s) {
    uint32_t blocks = 0;
    for (int i = 0; i < L.n; ++i) {
        L.item[i].block0 = blocks;
        blocks += (uint32_t)((L.item[i].bytes + kCopyBytes - 1) / kCopyBytes);
    }
    if (blocks) hipLaunchKernelGGL(k_copy_list, dim3(blocks), dim3(256), 0, s, L);
}

__global__ __launch_bounds__(256) void k_pack(const PackList L, uint64_t* dst) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < L.n) dst[(size_t)blockIdx.y * L.n + i] = L.src[blockIdx.y][i];
}

void launch_pack(const PackList& L, uint64_t* dst, hipStream_t s) {
    hipLaunchKernelGGL(k_pack, dim3((L.n + 255) / 256, L.arrays), dim3(256), 0, s, L, dst);
}

// Wet/dry decision of every link of member m from its state in copy p, in the
// host link layouts (x-links [ny][nx+1], y-links [ny+1][nx]).  Interior links
// use link_depth, as the step does; an open edge link is wet when its inner
// cell's depth exceeds h_dry; walls and inflow links (prescribed discharge,
// no decision) are 0.  One lane per link.
template <typename T, int MI>
__global__ __launch_bounds__(256) void k_wetmask(const CatchDev<T> C, int m, int p, uint8_t* wx, uint8_t* wy) {
    const int ny = C.ny, nx = C.nx;
    const size_t nxl = (size_t)ny * (nx + 1), nyl = (size_t)(ny + 1) * nx;
    const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= nxl + nyl) return;
    const T* H = C.h[p];
    const T hdry = C.hdry;
    auto hat = [&](int r, int c) -> T { return H[state_index<T, MI>(C, m, r, c)]; };
    auto zat = [&](int r, int c) -> T { return C.z[(size_t)r * nx + c]; };
    // inflow link ids in the order N (c), S (nx + c), W (2 nx + r), E (2 nx + ny + r)
    auto inflow = [&](int i) -> bool { return C.inflow_id && C.inflow_id[i] >= 0; };
    uint8_t w = 0;
    if (e < nxl) {
        const int r = (int)(e / (nx + 1)), c = (int)(e % (nx + 1));
        if (c == 0)
            w = C.edge_open[3] && !inflow(2 * nx + r) && hat(r, 0) > hdry;
        else if (c == nx)
            w = C.edge_open[1] && !inflow(2 * nx + ny + r) && hat(r, nx - 1) > hdry;
        else
            w = link_depth(hat(r, c - 1), hat(r, c), zat(r, c) - zat(r, c - 1)) > hdry;
        wx[e] = w;
    } else {
        const size_t f = e - nxl;
        const int r = (int)(f / nx), c = (int)(f % nx);
        if (r == 0)
            w = C.edge_open[0] && !inflow(c) && hat(0, c) > hdry;
        else if (r == ny)
            w = C.edge_open[2] && !inflow(nx + c) && hat(ny - 1, c) > hdry;
        else
            w = link_depth(hat(r - 1, c), hat(r, c), zat(r, c) - zat(r - 1, c)) > hdry;
        wy[f] = w;
    }
}

template <typename T>
void launch_wetmask(int mi, const CatchDev<T>& C, int member, int p, uint8_t* wx, uint8_t* wy, hipStream_t s) {
    const size_t n = (size_t)C.ny * (C.nx + 1) + (size_t)(C.ny + 1) * C.nx;
    dim3 grid((unsigned)((n + 255) / 256));
    switch (mi) {
        case 1: hipLaunchKernelGGL((k_wetmask<T, 1>), grid, dim3(256), 0, s, C, member, p, wx, wy); break;
        case 2: hipLaunchKernelGGL((k_wetmask<T, 2>), grid, dim3(256), 0, s, C, member, p, wx, wy); break;
        case 4: hipLaunchKernelGGL((k_wetmask<T, 4>), grid, dim3(256), 0, s, C, member, p, wx, wy); break;
        default: hipLaunchKernelGGL((k_wetmask<T, 8>), grid, dim3(256), 0, s, C, member, p, wx, wy); break;
    }
}

// Observation operator: depth of every member at every gauge cell, [N*K].
template <typename T, int MI>
__global__ __launch_bounds__(256) void k_gauges(const CatchDev<T> C, const int32_t* par, int K, const int32_t* grc,
                                                double* y, int ys) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= C.n_members * K) return;
    const int m = e / K, k = e % K;
    const T* h = C.h[par[C.member_off + m]];
    y[(size_t)m * ys + k] = (double)h[state_index<T, MI>(C, m, grc[2 * k], grc[2 * k + 1])];
}

template <typename T>
void launch_gauges(int mi, const CatchDev<T>& C, const int32_t* par, int n_gauges, const int32_t* grc, double* y,
                   int ys, hipStream_t s) {
    dim3 grid((C.n_members * n_gauges + 255) / 256);
    if (grid.x == 0) return;
    switch (mi) {
        case 1: hipLaunchKernelGGL((k_gauges<T, 1>), grid, dim3(256), 0, s, C, par, n_gauges, grc, y, ys); break;
        case 2: hipLaunchKernelGGL((k_gauges<T, 2>), grid, dim3(256), 0, s, C, par, n_gauges, grc, y, ys); break;
        case 4: hipLaunchKernelGGL((k_gauges<T, 4>), grid, dim3(256), 0, s, C, par, n_gauges, grc, y, ys); break;
        default: hipLaunchKernelGGL((k_gauges<T, 8>), grid, dim3(256), 0, s, C, par, n_gauges, grc, y, ys); break;
    }
}

// Streamflow through sections (Sec. 4.4): one workgroup per (section, member)
// sums sign * q over the section's links in FP64 (lanes stride the links, then
// a fixed reduction tree), times dx.
template <typename T, int MI>
__global__ __launch_bounds__(256) void k_sections(const CatchDev<T> C, const int32_t* par, const int32_t* offs,
                                                  const int32_t* code, const int32_t* index, double* out,
                                                  int ostride, int ooff) {
    const int sec = blockIdx.x, m = blockIdx.y;
    const int p = par[C.member_off + m];
    const int chunk = m / MI, lane = m % MI;
    const size_t plane = (size_t)C.ny * C.nx * MI;
    double acc = 0.0;
    for (int l = offs[sec] + (int)threadIdx.x; l < offs[sec + 1]; l += 256) {
        const int cd = code[l], ix = index[l];
        double q;
        switch (cd & 3) {
            case 0: q = (double)C.qx[p][(size_t)chunk * plane + (size_t)ix * MI + lane]; break;
            case 1: q = (double)C.qy[p][(size_t)chunk * plane + (size_t)ix * MI + lane]; break;
            case 2: q = (double)C.qw[p][((size_t)chunk * C.ny + ix) * MI + lane]; break;
            default: q = (double)C.qn[p][((size_t)chunk * C.nx + ix) * MI + lane]; break;
        }
        acc += (cd & 4) ? -q : q;
    }
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
    __shared__ double part[4];
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) out[(size_t)m * ostride + ooff + sec] = ((part[0] + part[1]) + (part[2] + part[3])) * C.dx;
}

template <typename T>
void launch_sections(int mi, const CatchDev<T>& C, const int32_t* par, int n_sections, const int32_t* offs,
                     const int32_t* code, const int32_t* index, double* out, int ostride, int ooff, hipStream_t s) {
    if (n_sections <= 0 || C.n_members <= 0) return;
    const dim3 grid(n_sections, C.n_members);
    switch (mi) {
        case 1:
            hipLaunchKernelGGL((k_sections<T, 1>), grid, dim3(256), 0, s, C, par, offs, code, index, out, ostride, ooff);
            break;
        case 2:
            hipLaunchKernelGGL((k_sections<T, 2>), grid, dim3(256), 0, s, C, par, offs, code, index, out, ostride, ooff);
            break;
        case 4:
            hipLaunchKernelGGL((k_sections<T, 4>), grid, dim3(256), 0, s, C, par, offs, code, index, out, ostride, ooff);
            break;
        default:
            hipLaunchKernelGGL((k_sections<T, 8>), grid, dim3(256), 0, s, C, par, offs, code, index, out, ostride, ooff);
            break;
    }
}

// Fold the per-edge-link outflow accumulators into the per-member total.
__global__ __launch_bounds__(256) void k_flush_outflow(int nb, double* acc, double* vout) {
    const int m = blockIdx.x;
    double* a = acc + (size_t)m * nb;
    double s = 0.0;
    for (int i = threadIdx.x; i < nb; i += 256) {
        s += a[i];
        a[i] = 0.0;
    }
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    __shared__ double part[4];
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) vout[m] += (part[0] + part[1]) + (part[2] + part[3]);
}

void launch_flush_outflow(int n_members, int nb, double* out_acc, double* vout, hipStream_t s) {
    if (n_members > 0) hipLaunchKernelGGL(k_flush_outflow, dim3(n_members), dim3(256), 0, s, nb, out_acc, vout);
}

// explicit instantiations
template void launch_plan<float>(const PlanLaunch<float>&, hipStream_t);
template void launch_plan<double>(const PlanLaunch<double>&, hipStream_t);
template void launch_step_mi<float>(int, const StepLaunch<float>&, hipStream_t);
template void launch_step_mi<double>(int, const StepLaunch<double>&, hipStream_t);
template void launch_hmax_init<float>(int, const CatchDev<float>&, const int32_t*, uint32_t*, int, hipStream_t);
template void launch_hmax_init<double>(int, const CatchDev<double>&, const int32_t*, unsigned long long*, int,
                                       hipStream_t);
template void launch_storage<float>(int, const CatchDev<float>&, const int32_t*, double*, hipStream_t);
template void launch_storage<double>(int, const CatchDev<double>&, const int32_t*, double*, hipStream_t);
template void launch_get_field<float>(int, const CatchDev<float>&, int, const int32_t*, int, size_t, size_t, double*,
                                     hipStream_t);
template void launch_get_field<double>(int, const CatchDev<double>&, int, const int32_t*, int, size_t, size_t, double*,
                                      hipStream_t);
template void launch_set_field<float>(int, const CatchDev<float>&, int, const int32_t*, int, const double*, hipStream_t);
template void launch_set_field<double>(int, const CatchDev<double>&, int, const int32_t*, int, const double*, hipStream_t);
template void launch_wetmask<float>(int, const CatchDev<float>&, int, int, uint8_t*, uint8_t*, hipStream_t);
template void launch_wetmask<double>(int, const CatchDev<double>&, int, int, uint8_t*, uint8_t*, hipStream_t);
template void launch_gauges<float>(int, const CatchDev<float>&, const int32_t*, int, const int32_t*, double*, int,
                                   hipStream_t);
template void launch_gauges<double>(int, const CatchDev<double>&, const int32_t*, int, const int32_t*, double*, int,
                                    hipStream_t);
template void launch_sections<float>(int, const CatchDev<float>&, const int32_t*, int, const int32_t*,
                                     const int32_t*, const int32_t*, double*, int, int, hipStream_t);
template void launch_sections<double>(int, const CatchDev<double>&, const int32_t*, int, const int32_t*,
                                      const int32_t*, const int32_t*, double*, int, int, hipStream_t);

}  // namespace flood

namespace flood {

// ---------------------------------------------------------------------------
// Row-marching step for members stored in planes (MI = 1).
//
// One wavefront handles SEG members on a strip 62 cells wide and `march_rows`
// rows tall.  Lane l holds cell x0 - 1 + l: lanes 0 and 63 are halo cells that
// only supply their values to the neighbouring lanes, so horizontal neighbours
// (depth, bed, roughness, the east link of the lane to the left) come from
// lane shuffles.  Walking down the strip, the next row's depth, bed and
// roughness are loaded once and carried into the following iteration, and the
// new south link of a row is the north link of the next, so every state
// element is read once and written once; the bed and roughness rows are shared
// by the SEG members, whose independent streams keep more loads in flight per
// wavefront.  Whether a member steps is uniform across the wavefront, so idle
// members cost no divergence.  Each cell evaluates the same link functions on
// the same operands as k_step, so both kernels produce identical bits.
// ---------------------------------------------------------------------------
template <typename T, int SEG>
__global__ __launch_bounds__(kBlock) void k_march(const StepLaunch<T> L) {
    using HB = typename HBits<T>::type;
    const int lane = threadIdx.x & 63;
    // the wavefront index is uniform across the wavefront; saying so lets every
    // per-member quantity live in scalar registers
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int wg = xcd_remap(blockIdx.x, gridDim.x) * (kBlock / 64) + wave;
    int ci = 0;
    for (int i = 1; i < L.n_catch; ++i)
        if (wg >= L.c[i].wave_begin) ci = i;
    const CatchDev<T>& C = L.c[ci];
    const int local = wg - C.wave_begin;
    if (local >= C.n_waves) return;
    const int n_groups = (C.n_members + SEG - 1) / SEG;
    int kg, sx, sy;
    if (!march_wave(C, local, n_groups, kg, sx, sy)) return;
    MemberStep<T> ms[SEG];
    bool act[SEG];
    bool any = false;
#pragma unroll
    for (int s = 0; s < SEG; ++s) {
        const int k = kg * SEG + s;
        act[s] = false;
        if (k < C.n_members) {
            ms[s] = L.ms[C.member_off + k];
            act[s] = ms[s].active != 0;
        }
        any |= act[s];
    }
    if (!any) return;
    const int nx = C.nx, ny = C.ny;
    const int x = sx * 62 - 1 + lane;
    const bool inx = x >= 0 && x < nx;
    const bool own = lane >= 1 && lane <= 62 && inx;
    const bool hasE = x + 1 < nx, hasW = x > 0;
    const int r0 = sy * C.march_rows;
    const int r1 = min(r0 + C.march_rows, ny);
    const size_t plane = (size_t)ny * nx;
    const T* __restrict__ Z = C.z;
    const T* __restrict__ Nn = C.n;
    const T g = C.g, hdry = C.hdry;
    const int nb = 2 * (nx + ny);

    size_t c0 = (size_t)r0 * nx + x;
    T zc = inx ? Z[c0] : T(0);
    T nc = inx ? Nn[c0] : T(0);
    T zN = T(0), nN = T(0);
    if (inx && r0 > 0) {
        zN = Z[c0 - nx];
        nN = Nn[c0 - nx];
    }
    T hc[SEG], fN[SEG];
    HB vmax[SEG];
#pragma unroll
    for (int s = 0; s < SEG; ++s) {
        hc[s] = T(0);
        fN[s] = T(0);
        vmax[s] = 0;
        if (!act[s]) continue;
        const int k = kg * SEG + s;
        const int sp = ms[s].parity;
        const T* __restrict__ H = C.h[sp] + (size_t)k * plane;
        if (inx) {
            hc[s] = H[c0];
            if (r0 > 0) {
                const T nf = T(0.5) * (nN + nc);
                fN[s] = link_in(C.qy[sp][(size_t)k * plane + c0 - nx], H[c0 - nx], hc[s], zc - zN, g * (nf * nf),
                                ms[s], hdry);
            } else if (C.edge_open[0]) {
                fN[s] = -link_open(-C.qn[sp][(size_t)k * nx + x], hc[s], g * (nc * nc), C.edge_slope[0], ms[s], hdry);
            }
        }
    }
    for (int r = r0; r < r1; ++r) {
        const bool hasS = r + 1 < ny;
        T zs = T(0), ns = T(0);
        if (inx && hasS) {
            zs = Z[c0 + nx];
            ns = Nn[c0 + nx];
        }
        const T zE = __shfl_down(zc, 1, 64);
        const T nE = __shfl_down(nc, 1, 64);
        const T gb = g * (nc * nc);
        T nfE = T(0.5) * (nc + nE);
        const T GE = g * (nfE * nfE);
        const T nfS = T(0.5) * (nc + ns);
        const T GS = g * (nfS * nfS);
#pragma unroll
        for (int s = 0; s < SEG; ++s) {
            if (!act[s]) continue;
            const int k = kg * SEG + s;
            const MemberStep<T>& m = ms[s];
            const int sp = m.parity, dp = sp ^ 1;
            const size_t base = (size_t)k * plane;
            const T* __restrict__ H = C.h[sp] + base;
            T hs = T(0), qE = T(0), qS = T(0);
            if (inx) {
                qE = C.qx[sp][base + c0];
                qS = C.qy[sp][base + c0];
                if (hasS) hs = H[c0 + nx];
            }
            const T h0 = hc[s];
            const T hE = __shfl_down(h0, 1, 64);
            T fE;
            if (hasE)
                fE = link_in(qE, h0, hE, zE - zc, GE, m, hdry);
            else
                fE = C.edge_open[1] ? link_open(qE, h0, gb, C.edge_slope[1], m, hdry) : T(0);
            const T fWn = __shfl_up(fE, 1, 64);
            if (own) {
                T fW, fS;
                if (hasW)
                    fW = fWn;
                else
                    fW = C.edge_open[3] ? -link_open(-C.qw[sp][(size_t)k * ny + r], h0, gb, C.edge_slope[3], m, hdry)
                                        : T(0);
                if (hasS)
                    fS = link_in(qS, h0, hs, zs - zc, GS, m, hdry);
                else
                    fS = C.edge_open[2] ? link_open(qS, h0, gb, C.edge_slope[2], m, hdry) : T(0);
                const T dv = ((fW - fE) + fN[s]) - fS;
                T hn = depth_add(h0, m.dtdx * dv + m.rinc, m.seed, (uint32_t)(r * nx + x));
                if (hn < T(0)) {
                    atomicAdd(&L.vclamp[C.member_off + k], -(double)hn * (C.dx * C.dx));
                    hn = T(0);
                }
                if (hn == T(0)) hn = T(0);
                C.h[dp][base + c0] = hn;
                if (C.peak) C.peak[base + c0] = fmax(C.peak[base + c0], hn);
                C.qx[dp][base + c0] = fE;
                C.qy[dp][base + c0] = fS;
                if (!hasW) C.qw[dp][(size_t)k * ny + r] = fW;
                if (r == 0) C.qn[dp][(size_t)k * nx + x] = fN[s];
                if (!(hasE && hasW && hasS && r > 0)) {
                    double* acc = C.out_acc + (size_t)k * nb;
                    if (r == 0 && C.edge_open[0]) acc[x] += -(double)fN[s] * m.dxdt;
                    if (!hasS && C.edge_open[2]) acc[nx + x] += (double)fS * m.dxdt;
                    if (!hasW && C.edge_open[3]) acc[2 * nx + r] += -(double)fW * m.dxdt;
                    if (!hasE && C.edge_open[1]) acc[2 * nx + ny + r] += (double)fE * m.dxdt;
                }
                const HB hb = to_bits(hn);
                vmax[s] = hb > vmax[s] ? hb : vmax[s];
                fN[s] = fS;
            }
            hc[s] = hs;
        }
        zc = zs;
        nc = ns;
        c0 += nx;
    }
#pragma unroll
    for (int s = 0; s < SEG; ++s) {
        if (!act[s]) continue;
        HB v = vmax[s];
        for (int off = 32; off > 0; off >>= 1) {
            const HB o = __shfl_xor(v, off, 64);
            v = o > v ? o : v;
        }
        if (lane == 0 && v != 0) {
            HB* a = L.hbins + (size_t)(blockIdx.x & (kBins - 1)) * L.n_total + C.member_off + kg * SEG + s;
            const HB cur = __hip_atomic_load(a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (v > cur) atomicMax(a, v);
        }
    }
}

// ---------------------------------------------------------------------------
// Vectorised row-marching step (members in planes): each lane owns V adjacent
// cells and moves them with one V-wide load or store, so a wavefront streams a
// strip of 64 V cells per row.  Every lane owns cells: the strip starts at a
// multiple of 64 V cells, so with a row pitch that is a multiple of 16 cells its
// stores cover whole 64-byte blocks and no block is shared with a neighbouring
// strip.  Where nx is no multiple of V (EXT bit 2) the last lane of a row owns
// the remainder: it loads V cells all the same (the arrays are padded by kRowPad
// elements) and stores its own one by one.
//
// What bounds it is vector issue as much as HBM, so the row loop holds nothing
// but the links and the depth update of its own cells:
//  - row addresses are wavefront-uniform bases with one 32-bit lane offset;
//  - the cells beside the strip are loaded for two rows at a time by lanes 0, 1
//    (west) and 63, 62 (east), and the strip's west link is evaluated for both
//    rows at once (exactly as the strip to the west evaluates its last east link:
//    same operands, same order), as are the domain's west and east edge links.
//    (A batch of 16 or more rows per evaluation reads the neighbours' cells long
//    before the neighbours do: 17 % more HBM reads at 2000 x 2000 x 96.);
//  - the loads of the first row, of the row above the strip, of the cells beside
//    it and of the second row are all issued before the first is waited for;
//  - neighbouring lanes' values come by DPP shifts, the halo value entering as
//    the shift's fill;
//  - a cell's limiter product h capf serves its four links;
//  - two rows per loop iteration, so the register sets of the row in work and of
//    the row in flight swap roles without moves;
//  - clamped depths, which are rare, are handled under a wavefront-wide test.
// Same link functions and operands as k_step: identical bits.
//
// Measured against the form that kept pointers per stream, evaluated the west
// link in every row and rotated its registers (160 vector instructions per cell,
// 72-85 % of the cycles; now about 120): calls of flood_step over 512 x 512 x 16
// 10.0 -> 8.9 ms, 768 x 1536 x 24 with land cover and running maxima 37.4 ->
// 31.9 ms, 1024 x 1024 x 16 with inflow links 32.6 -> 26.7 ms, 701 x 503 x 12 (the
// scalar march before) 8.9 -> 8.1 ms.  2000 x 2000 x 96 stays at 2.0 ms a launch
// (311 -> 311 ms): there the six state streams of 9.2 GB are at the rate that the
// same streams reach without arithmetic.
// ---------------------------------------------------------------------------
// The next row's loads are issued before the current row's arithmetic.  Rows are
// clamped to the last one: values of the row below it are read but never used.
// All row traffic goes through buffer descriptors in scalar registers: a lane
// address is one 32-bit offset in a row plus a wavefront-uniform row offset, and
// lanes beyond the last column carry an offset past the buffer's end, which the
// hardware's range check turns into zero loads and dropped stores, so the row
// loop holds no branch around memory accesses and no address arithmetic, and
// the compiler's waits leave the next row's loads in flight (as pointers, the
// addresses of the nine row streams took 18 registers and spilled, and every row
// waited for all of its loads).
// REC = 0: the plain step between the member's two state copies.  REC = 1: tape
// recomputation for the adjoint (tape block ms.blk to block ms.blk_next, a
// clamped depth stored as -0, no ledger).  REC = 2: the adjoint's recording
// forward, the same blocks and marks with the plain step's ledger, depth-maximum
// bins and outflow.  EXT: bit 0 land cover, bit 1 inflow links, bit 2 nx not a
// multiple of V (neither of the former), bit 3 running maximum (of the catchments
// that keep one).
constexpr int kMarchLand = 1, kMarchInflow = 2, kMarchRagged = 4, kMarchPeak = 8;

// what a row of a strip needs from memory: its links, and the depth, bed and
// roughness (land cover: classes) of the row below it
template <typename T, int V, bool LC, bool PEAK>
struct MarchRow {
    T qE[V], qS[V], hs[V], zs[V];
    T ns[LC ? 1 : V];
    T pk[PEAK ? V : 1];
    uint32_t cs;   // land cover: classes of the row below, one byte per cell
};

// The step planned by the wavefronts that take it: each of a member's wavefronts
// folds the member's depth-maximum bins and forms the step's coefficients itself,
// in the same operations as k_plan, while its first rows are on their way; the
// member's first wavefront (lead) writes the member's new clock, ledger and log.
// A planner launch before every step costs its 4-7 us and a launch gap of 4 us
// (a third to a half of a step of 512 x 512 x 16 cells and less); folded in, the
// bins' reduction and one division for three quotients cost a wavefront about
// 300 cycles.
template <typename T> struct PlanHead {
    using HB = typename HBits<T>::type;
    double t, t_end;
    int64_t steps;
    int32_t par;
    HB hb;          // depth-maximum bin of this lane
};

// the member's clock; false (and, by the lead wavefront, the member's values
// carried over to the next launch) when it takes no step
template <typename T>
__device__ __forceinline__ bool plan_head(const StepPlan<T>& P, int m, int n_total, int lane, bool lead, PlanHead<T>& h) {
    h.t = P.t_in[m];
    h.t_end = *P.t_end;
    h.steps = P.steps_in[m];
    h.par = P.par_in[m];
    h.hb = P.bins_in[(size_t)lane * n_total + m];
    const int fault = P.fault_in[m];
    if (!fault && h.t < h.t_end && h.steps < P.lim[m]) return true;
    if (lead) {
        P.bins_out[(size_t)lane * n_total + m] = h.hb;
        P.bins_clear[(size_t)lane * n_total + m] = 0;
        if (lane == 0) {
            P.t_out[m] = h.t;
            P.steps_out[m] = h.steps;
            P.par_out[m] = h.par;
            P.fault_out[m] = fault;
        }
    }
    return false;
}

// the step's coefficients; false when the member is frozen (see k_plan)
template <typename T>
__device__ __forceinline__ bool plan_step(const StepPlan<T>& P, const PlanCatch& C, int m, int n_total, int lane, bool lead,
                                          const PlanHead<T>& h, MemberStep<T>& ms) {
    const T H = from_bits<T>(wave_max_bits(h.hb));
    const double t = h.t;
    const double jf = floor(t / C.rain_interval);
    const bool rains = jf >= 0.0 && jf < (double)C.n_rain;
    const double R = rains ? C.rain[(int64_t)jf] : 0.0;
    double dt;
    if (C.dt_fixed > 0.0) {
        dt = C.dt_fixed;
    } else {
        double Hd = (double)H;
        if (Hd < C.hdry) Hd = C.hdry;
        dt = C.alpha * C.dx / sqrt(C.g * Hd);
        if (dt > C.dt_cap) dt = C.dt_cap;
    }
    const double dt_free = dt;   // not cut to an event
    const double edge = (jf + 1.0 > (double)C.n_rain) ? INFINITY : (jf + 1.0) * C.rain_interval;
    const double tev = h.t_end < edge ? h.t_end : edge;
    double tn;
    if (dt >= tev - t) {
        dt = tev - t;
        tn = tev;
    } else {
        tn = t + dt;
    }
    const bool finite = H <= (sizeof(T) == 4 ? T(FLT_MAX) : T(DBL_MAX));
    if (!finite || !(tn > t)) {
        if (lead) {
            P.bins_out[(size_t)lane * n_total + m] = h.hb;
            P.bins_clear[(size_t)lane * n_total + m] = 0;
            if (lane == 0) {
                P.fault_out[m] = 1;
                atomicOr(P.status, 1);
                P.t_out[m] = t;
                P.steps_out[m] = h.steps;
                P.par_out[m] = h.par;
            }
        }
        return false;
    }
    // dt / dx, g dt / dx and dx / (4 dt), one division in three lanes
    const double num = lane == 0 ? dt : lane == 1 ? C.g * dt : C.dx;
    const double den = lane == 2 ? 4.0 * dt : C.dx;
    const T quo = (T)(num / den);
    const double sc = P.s[m], mu = P.mu[m];
    ms.dtdx = lane_pick(quo, 0);
    ms.gdtdx = lane_pick(quo, 1);
    ms.capf = lane_pick(quo, 2);
    ms.gdt = lane_pick((T)(C.g * dt), 0);
    ms.s2dt = lane_pick((T)(sc * sc * dt), 0);
    ms.rinc = lane_pick((T)(mu * R * dt), 0);
    ms.dxdt = C.dx * dt;
    ms.active = 1;
    ms.parity = h.par;
    ms.slot = ms.blk = ms.blk_next = -1;
    const uint64_t tb = (uint64_t)__double_as_longlong(t);
    ms.seed = (uint32_t)__builtin_amdgcn_readfirstlane(
        (int)mix32((uint32_t)tb ^ mix32((uint32_t)(tb >> 32) + 0x632be5abu)));
    for (int k = 0; k < kMaxClasses; ++k) ms.cn[k] = P.clsn ? (T)P.clsn[(size_t)m * kMaxClasses + k] : T(0);
    ms.drain = P.drain ? lane_pick((T)(P.drain[m] * dt), 0) : T(0);
    double vq = 0.0;
#pragma unroll
    for (int j = 0; j < kMaxSeries; ++j) {
        ms.qin[j] = T(0);
        if (j < C.n_series) {
            const double q = rains ? C.inflow_q[(size_t)j * C.n_rain + (int64_t)jf] : 0.0;
            ms.qin[j] = lane_pick((T)q, 0);
            vq += C.wq[j] * q;
        }
    }
    if (lead) {
        P.bins_clear[(size_t)lane * n_total + m] = 0;
        if (lane == 0) {
            P.t_out[m] = tn;
            P.steps_out[m] = h.steps + 1;
            P.par_out[m] = h.par ^ 1;
            P.fault_out[m] = 0;
            P.dt_last[m] = dt_free;
            if (C.n_series > 0) P.vin[m] += vq * dt;
            P.vrain[m] += (double)ms.rinc * C.ncells * (C.dx * C.dx);
            if (P.dtlog) {
                const int64_t li = P.log_n[m];
                if (li < P.dtlog_cap) {
                    P.dtlog[(size_t)m * P.dtlog_cap + li] = dt;
                    P.telog[(size_t)m * P.dtlog_cap + li] = tn;
                }
                P.log_n[m] = li + 1;
            }
        }
    }
    return true;
}

// PLAN: the step is planned here (REC = 0), else by k_plan into L.ms.
// V: cells per lane, 16 bytes of them, or one.  With one a strip is 64 cells wide: small
// grids, bound by the chain of a wavefront's arithmetic (0.35 us a row against 1.3 us)
// and by lanes that idle beside a row shorter than 256 cells, get more and shorter ones
// (97 x 83 x 5 in FP32 7.2 us a step from 10.5; see narrow_pays and narrow_competes for where the line lies).
// Wavefronts per SIMD the registers are budgeted for: four in FP32 (128 registers; three
// where inflow links meet another extension and four would spill), two in FP64.
template <typename T> constexpr int march_occupancy(int ext) {
    return sizeof(T) == 8 ? 2 : ((ext & kMarchInflow) && (ext & ~kMarchInflow)) ? 3 : 4;
}
template <typename T, int V, int NT, int REC, int EXT, bool PLAN>
__global__ __launch_bounds__(kBlock, march_occupancy<T>(EXT)) void k_marchv(const StepLaunch<T> L) {
    using HB = typename HBits<T>::type;
    constexpr bool lc = (EXT & kMarchLand) != 0, INFL = (EXT & kMarchInflow) != 0, RAG = (EXT & kMarchRagged) != 0,
                   PEAK = (EXT & kMarchPeak) != 0;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int wg = xcd_remap(blockIdx.x, gridDim.x) * (kBlock / 64) + wave;
    // strips of one cell a lane: the depth maxima of a workgroup's wavefronts (see the end)
    constexpr bool kCombine = V == 1 && REC != 1;
    __shared__ HB wg_max[kCombine ? kBlock / 64 : 1];
    __shared__ int wg_member[kCombine ? kBlock / 64 : 1];
    if constexpr (kCombine) {
        if (lane == 0) wg_member[wave] = -1;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");   // done before this wavefront can end
    }
    int ci = 0;
    for (int i = 1; i < L.n_catch; ++i)
        if (wg >= L.c[i].wave_begin) ci = i;
    const CatchDev<T>& C = L.c[ci];
    const int local = wg - C.wave_begin;
    if (local >= C.n_waves) return;
    int k, sx, sy;
    if (!march_wave(C, local, C.n_members, k, sx, sy)) return;
    const int mg = C.member_off + k;
    const bool lead = sx == 0 && sy == 0;
    MemberStep<T> ms;
    PlanHead<T> head;
    if constexpr (PLAN) {
        if (!plan_head<T>(L.plan, mg, L.n_total, lane, lead, head)) return;
        ms.parity = head.par;
    } else {
        ms = L.ms[mg];
        if (!ms.active) return;
    }
    const int nx = C.nx, ny = C.ny;
    const int x0 = sx * (64 * V);                          // first cell of the strip
    const int xl = x0 + V * lane;                          // first cell of this lane
    const bool own = xl < nx;                              // with nx % V == 0 all V cells or none
    const int tail = RAG ? nx - xl : V;                    // own cells of the lane, if below V
    const bool westw = sx == 0;                            // wavefront-uniform edge tests
    const bool eastw = sx == C.strips_x - 1;
    const uint32_t es = (uint32_t)sizeof(T);
    const uint32_t xo = own ? (uint32_t)xl * es : kPastEnd;   // offset in a row, bytes
    const int r0 = sy * C.march_rows;
    const int r1 = min(r0 + C.march_rows, ny);
    const size_t plane = (size_t)ny * nx;
    const uint32_t pitch = (uint32_t)nx * es;
    const uint32_t bytes = (uint32_t)plane * es;           // plane <= 2^28 cells
    // source and destination of this member's state: the two copies, or (tape
    // recording and recomputation) the member's tape block and the block of its new state
    Rows<T> H, QX, QY, Ho, QXo, QYo;
    const T *QWs, *QNs;
    T *QWo, *QNo;
    if constexpr (REC) {
        const size_t bs = (size_t)__builtin_amdgcn_readfirstlane(ms.blk);
        const size_t bd = (size_t)__builtin_amdgcn_readfirstlane(ms.blk_next);
        H.set(C.h[0] + bs * plane, bytes);
        QX.set(C.qx[0] + bs * plane, bytes);
        QY.set(C.qy[0] + bs * plane, bytes);
        Ho.set(C.h[0] + bd * plane, bytes);
        QXo.set(C.qx[0] + bd * plane, bytes);
        QYo.set(C.qy[0] + bd * plane, bytes);
        QWs = C.qw[0] + bs * ny;
        QWo = C.qw[0] + bd * ny;
        QNs = C.qn[0] + bs * nx;
        QNo = C.qn[0] + bd * nx;
    } else {
        const bool p1 = __builtin_amdgcn_readfirstlane(ms.parity) != 0;
        const size_t b = (size_t)k * plane;
        H.set((p1 ? C.h[1] : C.h[0]) + b, bytes);
        QX.set((p1 ? C.qx[1] : C.qx[0]) + b, bytes);
        QY.set((p1 ? C.qy[1] : C.qy[0]) + b, bytes);
        Ho.set((p1 ? C.h[0] : C.h[1]) + b, bytes);
        QXo.set((p1 ? C.qx[0] : C.qx[1]) + b, bytes);
        QYo.set((p1 ? C.qy[0] : C.qy[1]) + b, bytes);
        QWs = (p1 ? C.qw[1] : C.qw[0]) + (size_t)k * ny;
        QWo = (p1 ? C.qw[0] : C.qw[1]) + (size_t)k * ny;
        QNs = (p1 ? C.qn[1] : C.qn[0]) + (size_t)k * nx;
        QNo = (p1 ? C.qn[0] : C.qn[1]) + (size_t)k * nx;
    }
    Rows<T> Z, NM, PK;
    Rows<uint8_t> CLS;
    Z.set(C.z, bytes);
    if constexpr (lc)
        CLS.set(C.cls, (uint32_t)plane);
    else
        NM.set(C.n, bytes);
    // a catchment that keeps no maxima has an empty array: the range check drops the
    // accesses, whose whole offset is the lane's
    if constexpr (PEAK) {
        const bool kept = C.peak != nullptr;
        PK.set(kept ? C.peak + (size_t)k * plane : C.h[0], kept ? bytes : 0u);
    }
    const T g = C.g, hdry = C.hdry;
    // outflow through open edges (FP64 per member and edge link); inflow links are
    // not outflow: their volume is logged by the step planner
    double* acc = C.out_acc + (size_t)k * (2 * (nx + ny));
    // inflow links (edge links with a prescribed inward discharge): the series
    // index of an edge link in the out_acc order, or -1; the series value is
    // picked by a select chain (a per-lane index into the step record would
    // go through private memory)
    const int8_t* INF = INFL ? C.inflow_id : nullptr;
    auto inflow_q = [&](int id) -> T { return pick4(id, ms.qin[0], ms.qin[1], ms.qin[2], ms.qin[3]); };
    // land cover: the member's class table lives in lanes: 0-3 its Manning n of
    // each class, 4-7 the runoff coefficients, 8-11 the drainage depth of the
    // step for draining classes (0 for the others); a cell's entries are read
    // from those lanes with ds_bpermute, a cross-lane read served by the LDS
    // unit, instead of compare-and-select chains on the VALU.  Every lookup is
    // made where the whole wavefront is active (the early returns above are
    // wavefront-uniform).
    T tab = T(0);
    auto lut = [&](uint32_t c, int base) -> T { return lane_read(tab, (int)c + base); };
    auto rough = [&](uint32_t c) -> T { return lut(c, 0); };
    const uint32_t xc = own ? (uint32_t)xl : kPastEnd;
    auto classes = [&](uint32_t row) -> uint32_t {   // of the lane's V cells
        if constexpr (V == 4)
            return CLS.load32(xc, row);
        else
            return CLS.load16(xc, row);
    };
    auto rough4 = [&](uint32_t cw, T (&nv)[V]) {
#pragma unroll
        for (int j = 0; j < V; ++j) nv[j] = rough((cw >> (8 * j)) & 0xffu);
    };
    // Manning factor g nf^2 of a link, nf = (n1 + n2) / 2 (the halving, exact, is in g4)
    const T g4 = T(0.25) * g;
    auto mean_g = [&](T n1, T n2) -> T {
        const T n = n1 + n2;
        return g4 * (n * n);
    };
    // a lane's own cells of a row; at: the lane's offset in the array
    auto store_own = [&](auto nt, const Rows<T>& a, uint32_t at, const T (&d)[V]) {
        if (!RAG || !eastw) {
            a.template store<V, decltype(nt)::value>(at, d);
        } else {
#pragma unroll
            for (int j = 0; j < V; ++j) a.store1(j < tail ? at + j * es : kPastEnd, d[j]);
        }
    };
    constexpr std::integral_constant<bool, NT == 1> nts{};
    constexpr std::integral_constant<bool, false> cached{};

    // Cells beside the strip, for rows r (lanes 0 and 63) and r + 1 (lanes 1 and
    // 62), and what follows from them: the west link (lanes 0, 1; the domain's west
    // edge link when westw), the east cell's depth, bed and (land cover) roughness,
    // or (eastw) the domain's east edge link (lanes 63, 62).
    struct Beside {
        T h, z, q, qe, n;
        uint32_t cls;
    };
    Beside hx;
    T bW = T(0), bN = T(0), bE = T(0), bH = T(0), bZ = T(0);
    const int cw = westw ? 0 : x0 - 1, ce = eastw ? nx - 1 : x0 + 64 * V;
    const bool wl = lane < 2, el = lane > 61;
    const uint32_t hat = beside_cell(lane, (uint32_t)nx, (uint32_t)cw, (uint32_t)ce);   // from row r
    const uint32_t hv = beside_lane(lane) ? hat * es : kPastEnd;
    const uint32_t qv = wl ? (westw ? (uint32_t)lane * es : hv) : kPastEnd;
    const uint32_t qev = (el && eastw) ? hv : kPastEnd;
    Rows<T> QH;
    QH.set(westw ? QWs : QX.p, westw ? (uint32_t)ny * es : bytes);
    auto beside_load = [&](int r, uint32_t so) {
        const uint32_t at = beside_at(hv, so);
        hx.h = H.load1(at, 0);
        hx.z = Z.load1(at, 0);
        hx.q = QH.load1(beside_at(qv, westw ? (uint32_t)r * es : so), 0);
        hx.qe = QX.load1(beside_at(qev, so), 0);
        if constexpr (lc)
            hx.cls = CLS.load8(beside_at(beside_lane(lane) ? hat : kPastEnd, so / es), 0);
        else
            hx.n = NM.load1(at, 0);
    };
    // h0, z0, n0: the lane's first cell in row r, h1, z1, n1: in row r + 1
    auto beside = [&](T h0, T z0, T n0, T h1, T z1, T n1) {
        T nb = hx.n;
        if constexpr (lc) nb = rough(hx.cls);
        bN = nb;
        // the strip's first cell, row r in lane 0, row r + 1 in lane 1
        const T hs = lane_shr(h1, h0), zs = lane_shr(z1, z0), n2 = lane_shr(n1, n0);
        const T hf = lane == 0 ? h0 : hs, zf = lane == 0 ? z0 : zs, nf = lane == 0 ? n0 : n2;
        if (!westw)
            bW = link_core(hx.q, hx.h, hf, hx.h * ms.capf, hf * ms.capf, zf - hx.z, mean_g(nb, nf) * ms.s2dt, ms.gdtdx,
                           hdry);
        else
            bW = C.edge_open[3] ? -link_open(-hx.q, hx.h, g * (nb * nb), C.edge_slope[3], ms, hdry) : T(0);
        bH = hx.h;
        bZ = hx.z;
        if (eastw) bE = C.edge_open[1] ? link_open(hx.qe, hx.h, g * (nb * nb), C.edge_slope[1], ms, hdry) : T(0);
    };
    // The domain's west and east edge links of the rows passed, lane i those of row
    // rb + i, written out every 64 rows and at the strip's end.  Inflow links take
    // their prescribed discharge: the ids of row rb + i are in lane i too.
    T eW = T(0), eE = T(0);
    int idW = -1, idE = -1;
    auto edges_begin = [&](int rb) {
        if constexpr (INFL) {
            const int rr = min(rb + lane, ny - 1);
            idW = (INF && westw) ? (int)INF[2 * nx + rr] : -1;
            idE = (INF && eastw) ? (int)INF[2 * nx + ny + rr] : -1;
        }
    };
    auto edges_end = [&](int rb, int re) {
        const int rr = rb + lane;
        if (rr >= re) return;
        if (westw) {
            QWo[rr] = eW;
            if (REC != 1 && C.edge_open[3] && idW < 0) acc[2 * nx + rr] += -(double)eW * ms.dxdt;
        }
        if (eastw && REC != 1 && C.edge_open[1] && idE < 0) acc[2 * nx + ny + rr] += (double)eE * ms.dxdt;
    };

    // loads of the row at offset so, and of the row below it
    auto load_row = [&](uint32_t so, bool below, MarchRow<T, V, lc, PEAK>& m) {
        const uint32_t sb = below ? so + pitch : so;
        QX.template load<V, NT == 1>(xo, so, m.qE);
        QY.template load<V, NT == 1>(xo, so, m.qS);
        H.template load<V, false>(xo, sb, m.hs);
        Z.template load<V, false>(xo, sb, m.zs);
        if constexpr (lc)
            m.cs = classes(sb / es);
        else
            NM.template load<V, false>(xo, sb, m.ns);
        if constexpr (PEAK) PK.template load<V, false>(beside_at(xo, so), 0, m.pk);
    };
    // first loads, in one go: the strip's first row, the row above it (or the
    // domain's north edge), the cells beside the strip, the first row's links
    T hc[V], cc[V], zc[V], nc[V], fN[V];   // row in work: depths, limiter products, bed, (land cover) roughness
    MarchRow<T, V, lc, PEAK> a, b;
    a.cs = b.cs = 0;
    uint32_t ccw = 0;
    uint32_t so = (uint32_t)r0 * pitch;    // the row in work
    uint32_t vo = own ? xo + so : kPastEnd;   // this lane's cells in it, for the stores
    const uint32_t vp = own ? pitch : 0u;
    // inflow ids of the strip's north and south edge links, one byte per cell of
    // the lane (0xff: none)
    uint32_t nid4 = 0xffffffffu, sid4 = 0xffffffffu;
    if constexpr (INFL) {
        if (INF) {
            const int xa = min(xl, nx - V);   // inflow links need nx % V == 0
#pragma unroll
            for (int j = 0; j < V; ++j) {
                if (r0 == 0) nid4 = (nid4 & ~(0xffu << (8 * j))) | ((uint32_t)(uint8_t)INF[xa + j] << (8 * j));
                if (r1 == ny) sid4 = (sid4 & ~(0xffu << (8 * j))) | ((uint32_t)(uint8_t)INF[nx + xa + j] << (8 * j));
            }
        }
    }
    auto id_of = [](uint32_t w, int j) -> int { return (int)(int8_t)(uint8_t)((w >> (8 * j)) & 0xffu); };
    {
        T hN[V], zN[V], qN[V], nN[V];
        uint32_t cwN = 0;
        H.template load<V, false>(xo, so, hc);
        Z.template load<V, false>(xo, so, zc);
        if constexpr (lc)
            ccw = classes(so / es);
        else
            NM.template load<V, false>(xo, so, nc);
        Rows<T> qn;
        qn.set(QNs, pitch);
        if (r0 > 0) {
            H.template load<V, false>(xo, so - pitch, hN);
            Z.template load<V, false>(xo, so - pitch, zN);
            QY.template load<V, false>(xo, so - pitch, qN);
            if constexpr (lc)
                cwN = classes((so - pitch) / es);
            else
                NM.template load<V, false>(xo, so - pitch, nN);
        } else {
            qn.template load<V, false>(xo, 0, qN);
        }
        beside_load(r0, so);
        load_row(so, r0 + 1 < ny, a);
        if constexpr (PLAN) {
            if (!plan_step<T>(L.plan, L.plan.pc[C.index], mg, L.n_total, lane, lead, head, ms)) return;
        }
        if constexpr (lc) {
            const int c = lane & 3;
            T cn = ms.cn[0], rc = C.class_rc[0];
            cn = (c == 1) ? ms.cn[1] : cn;
            cn = (c == 2) ? ms.cn[2] : cn;
            cn = (c == 3) ? ms.cn[3] : cn;
            rc = (c == 1) ? C.class_rc[1] : rc;
            rc = (c == 2) ? C.class_rc[2] : rc;
            rc = (c == 3) ? C.class_rc[3] : rc;
            const T dk = ((C.drain_mask >> c) & 1) ? ms.drain : T(0);
            tab = lane < 4 ? cn : lane < 8 ? rc : lane < 12 ? dk : T(0);
        }
        if constexpr (lc) rough4(ccw, nc);
#pragma unroll
        for (int j = 0; j < V; ++j) cc[j] = hc[j] * ms.capf;
        if (r0 > 0) {
            if constexpr (lc) rough4(cwN, nN);
#pragma unroll
            for (int j = 0; j < V; ++j)
                fN[j] = link_core(qN[j], hN[j], hc[j], hN[j] * ms.capf, cc[j], zc[j] - zN[j], mean_g(nN[j], nc[j]) * ms.s2dt,
                                  ms.gdtdx, hdry);
        } else {
            // north edge of the domain: the links, their strip and the outflow through them
#pragma unroll
            for (int j = 0; j < V; ++j) {
                fN[j] = T(0);
                if (C.edge_open[0]) fN[j] = -link_open(-qN[j], hc[j], g * (nc[j] * nc[j]), C.edge_slope[0], ms, hdry);
                if constexpr (INFL) {
                    const int id = id_of(nid4, j);
                    if (id >= 0) fN[j] = inflow_q(id);
                }
            }
            Rows<T> qno;
            qno.set(QNo, pitch);
            store_own(cached, qno, xo, fN);
            if (own && REC != 1 && C.edge_open[0]) {
#pragma unroll
                for (int j = 0; j < V; ++j)
                    if ((!RAG || j < tail) && id_of(nid4, j) < 0) acc[xl + j] += -(double)fN[j] * ms.dxdt;
            }
        }
    }

    HB vmax = 0;
    // Depth that clamping added, per lane.  In double where a step may also run in the
    // tiled kernel, which adds cell by cell: the two then give one ledger.
    using Clamped = std::conditional_t<RAG || V == 1, double, T>;
    Clamped vcl = 0;
    T vdr = T(0);
    double vdrain = 0.0;
    uint32_t cell = (uint32_t)r0 * (uint32_t)nx + (uint32_t)xl;
    // one row: m holds its loads, nxt takes those of the next row; odd: the second
    // row of a pair; bi: the row's lane in the edge registers
    auto row = [&](int r, auto odd, int bi, MarchRow<T, V, lc, PEAK>& m, MarchRow<T, V, lc, PEAK>& nxt) {
        constexpr int o = decltype(odd)::value;
        load_row(r + 1 < r1 ? so + pitch : so, r + 2 < ny, nxt);
        T ns[V];
        if constexpr (lc) {
            rough4(m.cs, ns);
        } else {
#pragma unroll
            for (int j = 0; j < V; ++j) ns[j] = m.ns[j];
        }
        if constexpr (o == 0) {
            beside(hc[0], zc[0], nc[0], m.hs[0], m.zs[0], ns[0]);
            beside_load(r + 2, so + 2 * pitch);
        }
        // east neighbour of the lane's last cell = first cell of the next lane, lane 63's the halo cell
        const T hE = lane_shl(hc[0], lane_pick(bH, 63 - o));
        const T zE = lane_shl(zc[0], lane_pick(bZ, 63 - o));
        const T nE = lane_shl(nc[0], lane_pick(bN, 63 - o));
        T fE[V], fS[V], fW[V], cs[V];
#pragma unroll
        for (int j = 0; j < V; ++j) {
            const T h2 = (j + 1 < V) ? hc[j + 1] : hE;
            const T z2 = (j + 1 < V) ? zc[j + 1] : zE;
            const T c2 = (j + 1 < V) ? cc[j + 1] : hE * ms.capf;
            const T G = mean_g(nc[j], (j + 1 < V) ? nc[j + 1] : nE);
            fE[j] = link_core(m.qE[j], hc[j], h2, cc[j], c2, z2 - zc[j], G * ms.s2dt, ms.gdtdx, hdry);
        }
        T w = lane_pick(bW, o);
        if (eastw) {
            T e = lane_pick(bE, 63 - o);
            if constexpr (INFL) {
                const int id = __builtin_amdgcn_readlane(idE, bi);
                if (id >= 0) e = -inflow_q(id);
            }
#pragma unroll
            for (int j = RAG ? 0 : V - 1; j < V; ++j) fE[j] = (xl + j + 1 == nx) ? e : fE[j];
            eE = lane == bi ? e : eE;
        }
        if (westw) {
            if constexpr (INFL) {
                const int id = __builtin_amdgcn_readlane(idW, bi);
                if (id >= 0) w = inflow_q(id);
            }
            eW = lane == bi ? w : eW;
        }
        fW[0] = lane_shr(fE[V - 1], w);
#pragma unroll
        for (int j = 1; j < V; ++j) fW[j] = fE[j - 1];
#pragma unroll
        for (int j = 0; j < V; ++j) {
            cs[j] = m.hs[j] * ms.capf;
            fS[j] = link_core(m.qS[j], hc[j], m.hs[j], cc[j], cs[j], m.zs[j] - zc[j], mean_g(nc[j], ns[j]) * ms.s2dt,
                              ms.gdtdx, hdry);
        }
        if (r + 1 == ny) {
            // south edge of the domain
#pragma unroll
            for (int j = 0; j < V; ++j) {
                fS[j] = T(0);
                if (C.edge_open[2])
                    fS[j] = link_open(m.qS[j], hc[j], g * (nc[j] * nc[j]), C.edge_slope[2], ms, hdry);
                if constexpr (INFL) {
                    const int id = id_of(sid4, j);
                    if (id >= 0) fS[j] = -inflow_q(id);
                }
            }
        }
        T hn[V], inc[V];
#pragma unroll
        for (int j = 0; j < V; ++j) {
            const T dv = ((fW[j] - fE[j]) + fN[j]) - fS[j];
            T rn = ms.rinc;
            if constexpr (lc) rn = ms.rinc * lut((ccw >> (8 * j)) & 0xffu, 4);
            inc[j] = ms.dtdx * dv + rn;
        }
        if constexpr (RAG || V == 1) {
            // the first cell of the lane may be odd, so a pair's hash may serve two lanes
#pragma unroll
            for (int j = 0; j < V; ++j) hn[j] = depth_add(hc[j], inc[j], ms.seed, cell + (uint32_t)j);
            if (RAG && eastw) {
#pragma unroll
                for (int j = 0; j < V; ++j) hn[j] = j < tail ? hn[j] : T(0);
            }
        } else {
            depth_add_row<T, V>(hc, inc, ms.seed, cell, hn);
        }
        bool neg[V];
        bool any = false;
#pragma unroll
        for (int j = 0; j < V; ++j) {
            neg[j] = hn[j] < T(0);
            any |= neg[j];
        }
        if (__any(any)) {
#pragma unroll
            for (int j = 0; j < V; ++j) {
                vcl += neg[j] ? (Clamped)-hn[j] : Clamped(0);
                // the tape keeps a clamped depth as -0 (the clamp branch for the adjoint)
                hn[j] = neg[j] ? (REC ? -T(0) : T(0)) : hn[j];
            }
        }
        if constexpr (lc) {
            // drainage of draining classes, up to the water the cell holds; summed per
            // drain_rows rows of the grid, so that the sum is the same for every strip
            // height that is a multiple of them
            if ((r & (L.drain_rows - 1)) == 0) {
                vdrain += (double)vdr;
                vdr = T(0);
            }
#pragma unroll
            for (int j = 0; j < V; ++j) {
                const T loss = fmin(lut((ccw >> (8 * j)) & 0xffu, 8), hn[j]);
                hn[j] = hn[j] - loss;
                vdr += loss;
            }
        }
#pragma unroll
        for (int j = 0; j < V; ++j) {
            // -0 (tape marks only) must not enter the bit-pattern maximum
            const HB hb = REC ? to_bits(hn[j] + T(0)) : to_bits(hn[j]);
            vmax = hb > vmax ? hb : vmax;
        }
        store_own(nts, Ho, vo, hn);
        store_own(nts, QXo, vo, fE);
        store_own(nts, QYo, vo, fS);
        if constexpr (PEAK) {
            T pk[V];
#pragma unroll
            for (int j = 0; j < V; ++j) pk[j] = fmax(m.pk[j], REC ? hn[j] + T(0) : hn[j]);
            store_own(cached, PK, vo, pk);
        }
#pragma unroll
        for (int j = 0; j < V; ++j) {
            fN[j] = fS[j];
            hc[j] = m.hs[j];
            zc[j] = m.zs[j];
            cc[j] = cs[j];
            nc[j] = ns[j];
        }
        ccw = m.cs;
        so += pitch;
        vo += vp;
        cell += (uint32_t)nx;
    };
    constexpr std::integral_constant<int, 0> even{};
    constexpr std::integral_constant<int, 1> odd{};
    for (int rb = r0; rb < r1; rb += 64) {
        const int re = min(rb + 64, r1);
        edges_begin(rb);
        int r = rb;
        for (; r + 1 < re; r += 2) {
            row(r, even, r - rb, a, b);
            row(r + 1, odd, r + 1 - rb, b, a);
        }
        if (r < re) row(r, even, r - rb, a, b);   // the strip's last row (64 rows end even)
        if (westw || eastw) edges_end(rb, re);
    }
    if (REC != 1 && r1 == ny && C.edge_open[2] && own) {
#pragma unroll
        for (int j = 0; j < V; ++j)
            if ((!RAG || j < tail) && id_of(sid4, j) < 0) acc[nx + xl + j] += (double)fN[j] * ms.dxdt;
    }
    if constexpr (REC != 1) {
        // lanes beyond the last column hold no cells
        vmax = own ? vmax : HB(0);
        for (int off = 32; off > 0; off >>= 1) {
            const HB o = __shfl_xor(vmax, off, 64);
            vmax = o > vmax ? o : vmax;
        }
        if constexpr (lc) {
            double dr = own ? vdrain + (double)vdr : 0.0;
            for (int off = 32; off > 0; off >>= 1) dr += __shfl_xor(dr, off, 64);
            // spread over kBins accumulators per member: the wavefronts in flight
            // mostly belong to one member, so a single address would serialise them
            if (lane == 0 && dr != 0.0)
                atomicAdd(C.drain_acc + (size_t)k * kBins + (blockIdx.x & (kBins - 1)), dr * (C.dx * C.dx));
        }
        vcl = own ? vcl : Clamped(0);
        if (__any(vcl != Clamped(0))) {
            double cl = (double)vcl;
            for (int off = 32; off > 0; off >>= 1) cl += __shfl_xor(cl, off, 64);
            if (lane == 0) atomicAdd(&L.vclamp[mg], cl * (C.dx * C.dx));
        }
        if constexpr (kCombine) {
            // Small grids: what counts is the chain after the last row, and that atomics on
            // the bins of few members meet on few cache lines (15 ns apiece), so the
            // wavefronts of a member in a workgroup send one, without looking first.
            // Wavefronts that had nothing to step have ended; the barrier is among the others.
            if (lane == 0) {
                wg_max[wave] = vmax;
                wg_member[wave] = mg;
            }
            __syncthreads();
            bool first = true;
#pragma unroll
            for (int w = 0; w < kBlock / 64; ++w) {
                if (wg_member[w] != mg) continue;
                first = first && w >= wave;
                const HB o = wg_max[w];
                vmax = o > vmax ? o : vmax;
            }
            if (first && lane == 0 && vmax != 0)
                atomicMax((PLAN ? L.plan.bins_out : L.hbins) + (size_t)(blockIdx.x & (kBins - 1)) * L.n_total + mg, vmax);
        } else if (lane == 0 && vmax != 0) {
            HB* bin = (PLAN ? L.plan.bins_out : L.hbins) + (size_t)(blockIdx.x & (kBins - 1)) * L.n_total + mg;
            const HB cur = __hip_atomic_load(bin, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (vmax > cur) atomicMax(bin, vmax);
        }
    }
}

// ext: kMarch* bits; an instantiation carries only the code of the extensions it
// names, so the plain step keeps its register budget
template <typename T, int EXT>
static void launch_marchv_ext(const StepLaunch<T>& L, int nt, const dim3 grid, hipStream_t s) {
    constexpr int V = march_vec<T>();
    static_assert(sizeof(StepLaunch<T>) <= 4096, "kernel arguments");
    if constexpr (EXT == 0 || EXT == kMarchPeak)
        if (L.narrow) {
            if (L.plan.pc) hipLaunchKernelGGL((k_marchv<T, 1, 0, 0, EXT, true>), grid, dim3(kBlock), 0, s, L);
            else hipLaunchKernelGGL((k_marchv<T, 1, 0, 0, EXT, false>), grid, dim3(kBlock), 0, s, L);
            return;
        }
    if (L.plan.pc && nt)
        hipLaunchKernelGGL((k_marchv<T, V, 1, 0, EXT, true>), grid, dim3(kBlock), 0, s, L);
    else if (L.plan.pc)
        hipLaunchKernelGGL((k_marchv<T, V, 0, 0, EXT, true>), grid, dim3(kBlock), 0, s, L);
    else if (nt)
        hipLaunchKernelGGL((k_marchv<T, V, 1, 0, EXT, false>), grid, dim3(kBlock), 0, s, L);
    else
        hipLaunchKernelGGL((k_marchv<T, V, 0, 0, EXT, false>), grid, dim3(kBlock), 0, s, L);
}

template <typename T>
void launch_marchv(const StepLaunch<T>& L, int nt, int ext, int total_waves, hipStream_t s) {
    const int per = kBlock / 64;
    const dim3 grid((total_waves + per - 1) / per);
    switch (ext) {
        case 0: launch_marchv_ext<T, 0>(L, nt, grid, s); break;
        case 1: launch_marchv_ext<T, 1>(L, nt, grid, s); break;
        case 2: launch_marchv_ext<T, 2>(L, nt, grid, s); break;
        case 3: launch_marchv_ext<T, 3>(L, nt, grid, s); break;
        case 4: launch_marchv_ext<T, 4>(L, nt, grid, s); break;
        case 8: launch_marchv_ext<T, 8>(L, nt, grid, s); break;
        case 9: launch_marchv_ext<T, 9>(L, nt, grid, s); break;
        case 10: launch_marchv_ext<T, 10>(L, nt, grid, s); break;
        case 11: launch_marchv_ext<T, 11>(L, nt, grid, s); break;
        default: launch_marchv_ext<T, 12>(L, nt, grid, s); break;
    }
}

// Tape recomputation of the adjoint (record = 0): the same step, reading and
// writing tape blocks, marking clamped depths as -0, leaving the ledger, the
// outflow accumulators and the depth maximum alone; members that do not step in
// the launch are skipped.  Recording forward (record = 1): the same blocks and
// marks, plus everything the plain step
// updates (depth maximum bins, clamp and outflow ledgers, running maximum).
template <typename T, int V, int NT>
static void launch_marchv_rec_v(const StepLaunch<T>& L, int record, int total_waves, hipStream_t s) {
    const int per = kBlock / 64;
    const dim3 grid((total_waves + per - 1) / per);
    if (record && L.c[0].peak)
        hipLaunchKernelGGL((k_marchv<T, V, NT, 2, kMarchPeak, false>), grid, dim3(kBlock), 0, s, L);
    else if (record)
        hipLaunchKernelGGL((k_marchv<T, V, NT, 2, 0, false>), grid, dim3(kBlock), 0, s, L);
    else
        hipLaunchKernelGGL((k_marchv<T, V, 0, 1, 0, false>), grid, dim3(kBlock), 0, s, L);
}

template <typename T>
void launch_marchv_rec(const StepLaunch<T>& L, int record, int total_waves, hipStream_t s) {
    if (L.narrow) launch_marchv_rec_v<T, 1, 0>(L, record, total_waves, s);
    else launch_marchv_rec_v<T, march_vec<T>(), 1>(L, record, total_waves, s);
}

template void launch_marchv<float>(const StepLaunch<float>&, int, int, int, hipStream_t);
template void launch_marchv<double>(const StepLaunch<double>&, int, int, int, hipStream_t);
template void launch_marchv_rec<float>(const StepLaunch<float>&, int, int, hipStream_t);
template void launch_marchv_rec<double>(const StepLaunch<double>&, int, int, hipStream_t);

template <typename T> void launch_march(const StepLaunch<T>& L, int seg, int total_waves, hipStream_t s) {
    const int per = kBlock / 64;
    const dim3 grid((total_waves + per - 1) / per);
    switch (seg) {
        case 1: hipLaunchKernelGGL((k_march<T, 1>), grid, dim3(kBlock), 0, s, L); break;
        case 2: hipLaunchKernelGGL((k_march<T, 2>), grid, dim3(kBlock), 0, s, L); break;
        case 4: hipLaunchKernelGGL((k_march<T, 4>), grid, dim3(kBlock), 0, s, L); break;
        default: hipLaunchKernelGGL((k_march<T, 8>), grid, dim3(kBlock), 0, s, L); break;
    }
}

template void launch_march<float>(const StepLaunch<float>&, int, int, hipStream_t);
template void launch_march<double>(const StepLaunch<double>&, int, int, hipStream_t);


// ---------------------------------------------------------------------------
// Ensemble products of the running maximum depth (Sec. 4.4, Figs. 15-16): the
// weight of the members at or above the threshold, and for each p the smallest
// member value v_k whose weight, that of the members at or below it, reaches p W
// (inverted distribution function).  Every weight is summed in FP64 in member
// order.
//
// One wavefront covers 64 cells, a lane each.  A weight summed that way never
// falls when members join the sum (a rounded addition keeps the order of its
// operands), so it never falls along the sorted values, and the first value that
// reaches p W is found by bisection: the values of a cell are sorted in registers
// (odd-even merges) into LDS, read again into the registers in member order, and
// each of log2(NP) rounds forms the exact weight of one candidate per percentile.
// In the sort a NaN (of a member that failed) stands as infinity, the value of a
// percentile that no candidate reaches.  Bound by the compares, selects and FMAs
// of the rounds: 18 per member and percentile at 64 members, where every
// candidate's weight took 3 x 64.  Three percentiles in FP32: 512 x 512 x 64 63 us from 212,
// 256 x 256 x 128 47 from 162; in FP64 256 x 256 x 64 24 from 39.
// NP: members, rounded up to a power of two.  The registers hold NP values, so
// ensembles past 128 members (64 in FP64) take k_products_any.
// Cells [cell0, cell0 + count) of the grid: prob [count], pout [n_pct][count].
template <typename T> constexpr T kInf = std::numeric_limits<T>::infinity();

template <typename T> __device__ __forceinline__ void sort_pair(T& a, T& b) {
    T lo, hi;
    if constexpr (sizeof(T) == 4) {
        lo = __builtin_fminf(a, b);
        hi = __builtin_fmaxf(a, b);
    } else {
        lo = __builtin_fmin(a, b);
        hi = __builtin_fmax(a, b);
    }
    a = lo;
    b = hi;
}

// Batcher's odd-even merge sort of v[LO .. LO + N), ascending
template <int LO, int N, int R, typename T, int NP> __device__ __forceinline__ void merge_odd_even(T (&v)[NP]) {
    if constexpr (2 * R < N) {
        merge_odd_even<LO, N, 2 * R>(v);
        merge_odd_even<LO + R, N, 2 * R>(v);
#pragma unroll
        for (int i = LO + R; i + R < LO + N; i += 2 * R) sort_pair(v[i], v[i + R]);
    } else {
        sort_pair(v[LO], v[LO + R]);
    }
}
template <int LO, int N, typename T, int NP> __device__ __forceinline__ void sort_odd_even(T (&v)[NP]) {
    if constexpr (N > 1) {
        sort_odd_even<LO, N / 2>(v);
        sort_odd_even<LO + N / 2, N / 2>(v);
        merge_odd_even<LO, N, 1>(v);
    }
}

// Bisection of G percentiles at once.  v: the cell's values in member order, w:
// weights, zero past the last member; sorted: the values in ascending order, the
// last of which always reaches (all of W, or infinity).
template <int G, typename T, int NP>
__device__ __forceinline__ void find_percentiles(const T (&v)[NP], const T* sorted, int lane, const double* __restrict__ w,
                                                 const double* __restrict__ pct, double W, double (&out)[3]) {
    int pos[G];
#pragma unroll
    for (int i = 0; i < G; ++i) pos[i] = 0;
    for (int half = NP / 2; half >= 1; half /= 2) {
        T p[G];
        double cum[G];
#pragma unroll
        for (int i = 0; i < G; ++i) {
            p[i] = sorted[(pos[i] + half - 1) * 64 + lane];
            cum[i] = 0.0;
        }
        // w_m x 1 or x 0 in one FMA: the sum of the selected weights, rounded as the
        // plain additions are (weights are finite and >= 0)
#pragma unroll
        for (int m = 0; m < NP; ++m) {
            const double wm = w[m];
#pragma unroll
            for (int i = 0; i < G; ++i) cum[i] = __builtin_fma(wm, v[m] <= p[i] ? 1.0 : 0.0, cum[i]);
        }
#pragma unroll
        for (int i = 0; i < G; ++i)
            if (p[i] < kInf<T> && !(cum[i] >= pct[i] * W)) pos[i] += half;
    }
#pragma unroll
    for (int i = 0; i < G; ++i) out[i] = (double)sorted[pos[i] * 64 + lane];
}

template <typename T, int NP>
__global__ __launch_bounds__(64) void k_products(const CatchDev<T> C, int mi, double thr, int n_pct,
                                                 const double* __restrict__ pct, const double* __restrict__ w,
                                                 double W, size_t cell0, size_t count, double* __restrict__ prob,
                                                 double* __restrict__ pout) {
    __shared__ T sorted[NP * 64];
    const int lane = threadIdx.x;
    const size_t i = (size_t)blockIdx.x * 64 + lane;
    const size_t ncell = (size_t)C.ny * C.nx;
    const T* at = C.peak + (cell0 + (i < count ? i : count - 1)) * mi;
    const int N = C.n_members;
    // member m's value (mi, a power of two, members interleaved); places past the
    // last member read that one's
    auto value = [&](int m) -> T {
        const int k = m < N ? m : N - 1;
        return at[(size_t)(k & ~(mi - 1)) * ncell + (k & (mi - 1))];
    };
    T v[NP];
#pragma unroll
    for (int m = 0; m < NP; ++m) v[m] = value(m);
    if (n_pct > 0) {
#pragma unroll
        for (int m = 0; m < NP; ++m) v[m] = m < N && v[m] == v[m] ? v[m] : kInf<T>;
        sort_odd_even<0, NP>(v);
#pragma unroll
        for (int m = 0; m < NP; ++m) sorted[m * 64 + lane] = v[m];
        __asm__ volatile("" ::: "memory");   // loads again, from the caches, instead of twice the registers
#pragma unroll
        for (int m = 0; m < NP; ++m) v[m] = value(m);
    }
    if (prob) {
        double hit = 0.0;
#pragma unroll
        for (int m = 0; m < NP; ++m) hit = __builtin_fma(w[m], (double)v[m] >= thr ? 1.0 : 0.0, hit);
        if (i < count) prob[i] = hit / W;
    }
    double q[3];
    for (int p = 0; p < n_pct; p += 3) {
        const int g = n_pct - p;
        if (g >= 3) find_percentiles<3>(v, sorted, lane, w, pct + p, W, q);
        else if (g == 2) find_percentiles<2>(v, sorted, lane, w, pct + p, W, q);
        else find_percentiles<1>(v, sorted, lane, w, pct + p, W, q);
        if (i >= count) continue;
#pragma unroll
        for (int e = 0; e < 3; ++e)
            if (e < g) pout[(size_t)(p + e) * count + i] = q[e];
    }
}

// The same for any number of members.  A workgroup covers 64 cells with four
// wavefronts, one lane per cell in each: it stages its cells' member values in LDS
// where they fit, the first wavefront forms the weight of the members at or above
// the threshold, and the four share the candidates k: for each, the weight of the
// members at or below member k's value; the smallest value whose weight reaches
// p W is a minimum over the candidates that is the same in any order.
constexpr int kProdCells = 64;
constexpr int kProdWaves = 4;      // wavefronts per workgroup, splitting the candidates
constexpr int kProdMaxPct = 16;

constexpr int kProdUnroll = 8;   // percentile candidates evaluated per pass over the members

template <typename T, bool LDS>
__global__ __launch_bounds__(kProdCells * kProdWaves) void k_products_any(
    const CatchDev<T> C, int mi, double thr, int n_pct, const double* __restrict__ pct, const double* __restrict__ w,
    double W, size_t cell0, size_t count, double* __restrict__ prob, double* __restrict__ pout) {
    extern __shared__ unsigned char smem[];
    T* vals = reinterpret_cast<T*>(smem);
    const int N = C.n_members;
    const size_t ncell = (size_t)C.ny * C.nx;
    const int lane = (int)threadIdx.x % kProdCells;
    const int wave = (int)threadIdx.x / kProdCells;
    const size_t cell = (size_t)blockIdx.x * kProdCells + lane;   // of this range
    const bool in = cell < count;
    auto peak = [&](int m) -> T {
        return C.peak[(size_t)(m / mi) * ncell * mi + (cell0 + (in ? cell : 0)) * mi + m % mi];
    };
    auto value = [&](int m) -> T {
        if constexpr (LDS) return vals[(size_t)m * kProdCells + lane];
        else return peak(m);
    };
    if constexpr (LDS) {
        for (int m = wave; m < N; m += kProdWaves)
            vals[(size_t)m * kProdCells + lane] = in ? peak(m) : T(0);
    }
    __syncthreads();
    const bool want_pct = n_pct > 0 && pout != nullptr;   // the same for the whole grid
    double best[kProdMaxPct];
    double lim[kProdMaxPct];
    for (int i = 0; i < n_pct; ++i) {
        best[i] = INFINITY;
        lim[i] = pct[i] * W;
    }
    if (in) {
        if (wave == 0) {
            // w_m x 1 or x 0 in one FMA: the sum of the selected weights, rounded as
            // the plain additions are (weights are finite and >= 0)
            double hit = 0.0;
            for (int m = 0; m < N; ++m) hit = __builtin_fma(w[m], ((double)value(m) >= thr) ? 1.0 : 0.0, hit);
            if (prob) prob[cell] = hit / W;
        }
        // kProdUnroll candidates k per pass over the members: independent sums
        // (each still in member order), one read of each member value per pass;
        // the wavefronts take interleaved groups of candidates
        if (want_pct) {
            for (int k0 = wave * kProdUnroll; k0 < N; k0 += kProdWaves * kProdUnroll) {
                T vk[kProdUnroll];
                double cum[kProdUnroll];
#pragma unroll
                for (int q = 0; q < kProdUnroll; ++q) {
                    vk[q] = value(k0 + q < N ? k0 + q : N - 1);
                    cum[q] = 0.0;
                }
                for (int m = 0; m < N; ++m) {
                    const T vm = value(m);
                    const double wm = w[m];
#pragma unroll
                    for (int q = 0; q < kProdUnroll; ++q) cum[q] = __builtin_fma(wm, (vm <= vk[q]) ? 1.0 : 0.0, cum[q]);
                }
#pragma unroll
                for (int q = 0; q < kProdUnroll; ++q) {
                    if (k0 + q >= N) break;
                    for (int i = 0; i < n_pct; ++i)
                        if (cum[q] >= lim[i] && (double)vk[q] < best[i]) best[i] = (double)vk[q];
                }
            }
        }
    }
    if (!want_pct) return;   // uniform: no wavefront is left waiting at the barriers below
    // minimum over the wavefronts' candidates, through LDS (the staged values are done with)
    __syncthreads();
    double* red = reinterpret_cast<double*>(smem);   // [wave][percentile][lane]
    for (int i = 0; i < n_pct; ++i) red[((size_t)wave * n_pct + i) * kProdCells + lane] = best[i];
    __syncthreads();
    if (wave == 0 && in)
        for (int i = 0; i < n_pct; ++i) {
            double b = red[(size_t)i * kProdCells + lane];
            for (int v = 1; v < kProdWaves; ++v) {
                const double o = red[((size_t)v * n_pct + i) * kProdCells + lane];
                b = o < b ? o : b;
            }
            pout[(size_t)i * count + cell] = b;
        }
}

template <typename T, int NP>
static void launch_products_np(int mi, const CatchDev<T>& C, double thr, int n_pct, const double* pct, const double* w,
                               double W, size_t cell0, size_t count, double* prob, double* pout, hipStream_t s) {
    hipLaunchKernelGGL((k_products<T, NP>), dim3((unsigned)((count + 63) / 64)), dim3(64), 0, s, C, mi, thr, n_pct, pct,
                       w, W, cell0, count, prob, pout);
}

template <typename T>
void launch_products(int mi, const CatchDev<T>& C, double thr, int n_pct, const double* pct, const double* w,
                     double W, size_t cell0, size_t count, double* prob, double* pout, hipStream_t s) {
    const int N = C.n_members;
    if (N <= 16) return launch_products_np<T, 16>(mi, C, thr, n_pct, pct, w, W, cell0, count, prob, pout, s);
    if (N <= 32) return launch_products_np<T, 32>(mi, C, thr, n_pct, pct, w, W, cell0, count, prob, pout, s);
    if (N <= 64) return launch_products_np<T, 64>(mi, C, thr, n_pct, pct, w, W, cell0, count, prob, pout, s);
    if constexpr (sizeof(T) == 4)
        if (N <= 128) return launch_products_np<T, 128>(mi, C, thr, n_pct, pct, w, W, cell0, count, prob, pout, s);
    const dim3 grid((unsigned)((count + kProdCells - 1) / kProdCells));
    const dim3 block(kProdCells * kProdWaves);
    const size_t stage = (size_t)N * kProdCells * sizeof(T);
    const size_t red = (size_t)kProdWaves * std::max(n_pct, 1) * kProdCells * sizeof(double);
    if (stage <= 48 * 1024)
        hipLaunchKernelGGL((k_products_any<T, true>), grid, block, std::max(stage, red), s, C, mi, thr, n_pct, pct, w, W,
                           cell0, count, prob, pout);
    else
        hipLaunchKernelGGL((k_products_any<T, false>), grid, block, red, s, C, mi, thr, n_pct, pct, w, W, cell0, count,
                           prob, pout);
}

template void launch_products<float>(int, const CatchDev<float>&, double, int, const double*, const double*, double,
                                     size_t, size_t, double*, double*, hipStream_t);
template void launch_products<double>(int, const CatchDev<double>&, double, int, const double*, const double*, double,
                                      size_t, size_t, double*, double*, hipStream_t);

}  // namespace flood
