// k_step.hip -- the per-step hot kernel on gfx950: truncated LJ pair forces
// gathered over the Verlet list, fused with both velocity-Verlet half steps
// and the reductions that follow them (paper Sec. 3 "Code structure" and
// Fig. 1: force, finalize and integrate; Sec. 5: truncated pair forces).
//
// One launch per step s does, for every particle i:
//   F_i(x_s)      = sum_j fs(r_ij) r_ij over list partners with r_ij < r_c
//   finalize      v_s   = v' + dt/(2m) F_i              (completes step s)
//   observables   e_i, w_i (half of every pair), K_i, m v_i -> FP64 block partials
//   integrate     v'    = v_s + dt/(2m) F_i ; x_{s+1} = x_s + dt v'  (starts step s+1)
//   displacement  |x_{s+1} - x_ref|^2 -> max -> rebuild decision of step s+1
// Positions are read from one record buffer and written to the other, so no
// wave ever sees a partner that has already moved.
//
// Gather geometry: LANES lanes per particle, 64/LANES particles per
// wavefront; in the interleaved list layout a lane's entries come in groups
// of four, so every list load of a wave is one 1 KiB contiguous read. Each
// XCD gets a contiguous eighth of the particles.
#include "batch.h"
#include "step_common.h"

namespace ljmd {

// Word 3 of a buffer descriptor: raw bytes (32-bit data format), so that an
// access past num_records reads 0.
constexpr int kRawBuffer = 0x00027000;

// Housekeeping shared by both precisions: the rebuilt marker of this step and,
// after a rebuild, clearing the cell counters for the next binning.
// Cells [c_lo, c_hi) belong to this system; block bj of its nbj blocks
// clears every nbj-th stretch of them. rebuilt (may be NULL) receives the marker.
__device__ inline void step_housekeeping(const StepArgs &a, const Ctl *ctl, int64_t c_lo, int64_t c_hi,
                                         int bj, int nbj, int32_t *rebuilt) {
    const bool rb = rebuild_due(ctl, a.step, a.forced, a.dyn.thr2);
    if (rebuilt && bj == 0 && threadIdx.x == 0) *rebuilt = rb ? 1 : 0;
    if (rb) {
        const int64_t nthr = (int64_t)nbj * blockDim.x;
        for (int64_t c = c_lo + (int64_t)bj * blockDim.x + threadIdx.x; c < c_hi; c += nthr)
            a.st.cell_count[c] = 0;
    }
}

// ---------------------------------------------------------------- FP32 ---
// Q: a cubic box. Then the pair loop works in quanta: the raw wrapped
// fixed-point differences are the displacements, r_c^2 and sigma^2 are
// pre-divided by the squared quantum (exactly, in FP64, before one
// rounding), and the quantum goes into the force factor 24 eps / quantum
// (once per particle with one species, per pair with two). The energy and
// virial terms are summed per lane in FP32 over the lane's few dozen pairs
// before the FP64 reductions. The lists are padded and every slot holds a valid index,
// so the entries the unrolled loop reads past a list are loaded unclamped
// and skipped.
//
// OBS: accumulate the pair energy and virial terms and reduce the
// observable partials; steps whose observables nobody reads skip them.
// Records are addressed by 32-bit byte offsets (fewer than 2^28 slots).
//
// The body serves one block of one system: box holds its constants, ctl its
// control words, particles below i_end are real (the rest of the block is
// padding), and the block is number bj of the nbj blocks that share the
// clearing of its cells [c_lo, c_hi).
// TH: the thermostat resamples colliding particles' velocities after
// "finalize" (a separate instantiation, so that the plain NVE kernel keeps
// its register budget).
// BS: threads per block. SMALL: the form for boxes that leave the chip's wave
// slots mostly empty (see the pair loop).
template <int NS, int LANES, bool Q, bool OBS, bool TH = false, bool PLAIN = false, int BS = kBlock,
          bool SMALL = false>
__device__ inline void step_ds_body(const StepArgs &a, const BoxC &box, Ctl *ctl, int blk, int64_t i_end,
                                    int64_t c_lo, int64_t c_hi, int bj, int nbj, int32_t *rebuilt) {
    constexpr int P = kWave / LANES;
    constexpr int WPB = BS / kWave;
    const State &st = a.st;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t chunk = (int64_t)blk * WPB + wv;
    const int l = lane % LANES;
    const int64_t i = chunk * P + lane / LANES;
    const bool valid = i < i_end;
    // SMALL: loads through buffer descriptors, which the compiler keeps where
    // they are written (it sinks plain loads of read-only memory to their
    // first use, past scheduling barriers). Everything the wave reads outside
    // its trips is asked for at once, ahead of the halt check: own record,
    // list length, first list entries, and the step tail's operands.
    constexpr int UQ = 8;  // list entries of a lane per trip
    const int4 *__restrict__ rec = st.recq[a.cur];
    [[maybe_unused]] __amdgpu_buffer_rsrc_t rsrc_rec, rsrc_nb;
    int4 ri = make_int4(0, 0, 0, 0);
    int cnt = 0;
    [[maybe_unused]] int jn[UQ];
    [[maybe_unused]] int4 xr;
    [[maybe_unused]] DsState ds;
    // Two 16-byte group loads: entries m .. m + 7 of the lane.
    const int32_t *__restrict__ nb = st.nbr + chunk * (int64_t)(P * a.g.cap) + 4 * lane;
    auto entries = [&](int m, int (&jj)[UQ]) {
        if constexpr (SMALL) {
            const auto g0 = __builtin_amdgcn_raw_buffer_load_b128(rsrc_nb, lane << 4, m << 8, 0);
            const auto g1 = __builtin_amdgcn_raw_buffer_load_b128(rsrc_nb, (lane << 4) + 1024, m << 8, 0);
#pragma unroll
            for (int u = 0; u < 4; ++u) jj[u] = (int)g0[u], jj[4 + u] = (int)g1[u];
        } else {
            const int4 g0 = *reinterpret_cast<const int4 *>(nb + ((int64_t)(m >> 2) << 8));
            const int4 g1 = *reinterpret_cast<const int4 *>(nb + ((int64_t)((m >> 2) + 1) << 8));
            jj[0] = g0.x, jj[1] = g0.y, jj[2] = g0.z, jj[3] = g0.w;
            jj[4] = g1.x, jj[5] = g1.y, jj[6] = g1.z, jj[7] = g1.w;
        }
    };
    if constexpr (SMALL) {
        // Slots past the last particle read 0 (out of the descriptor's range).
        auto rsrc = [](const void *p, int64_t bytes) {
            return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, kRawBuffer);
        };
        const int64_t wchunk = __builtin_amdgcn_readfirstlane((int)chunk);
        rsrc_rec = rsrc(rec, a.g.n << 4);
        rsrc_nb = rsrc(st.nbr + wchunk * (P * a.g.cap), wchunk * P < a.g.n ? P * a.g.cap * 4 + kListPad * 4 : 0);
        const __amdgpu_buffer_rsrc_t rsrc_cnt = rsrc(st.nbr_cnt, a.g.n << 2), rsrc_xr = rsrc(st.xref, a.g.n << 4);
        const int o16 = (int)i << 4;
        const uint32_t c = __builtin_amdgcn_raw_buffer_load_b32(rsrc_cnt, (int)i << 2, 0, 0);
        const auto r = __builtin_amdgcn_raw_buffer_load_b128(rsrc_rec, o16, 0, 0);
        entries(0, jn);
        const auto x = __builtin_amdgcn_raw_buffer_load_b128(rsrc_xr, o16, 0, 0);
        float4 w[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const auto v = __builtin_amdgcn_raw_buffer_load_b128(rsrc(st.dsw[k], a.g.n << 4), o16, 0, 0);
            w[k] = make_float4(__uint_as_float(v[0]), __uint_as_float(v[1]), __uint_as_float(v[2]), __uint_as_float(v[3]));
        }
        // One word of every 64-byte line of the kernel arguments, so that the
        // constants of the step tail come from the scalar cache later on.
        const auto *arg = (const __attribute__((address_space(4))) int *)__builtin_amdgcn_kernarg_segment_ptr();
        constexpr int kArgLines = (int)((sizeof(StepArgs) + 63) / 64);
        int touch = 0;
#pragma unroll
        for (int k = 0; k < kArgLines; ++k) touch |= arg[k * 16];
        asm volatile("" ::"s"(touch));
        __builtin_amdgcn_sched_barrier(0);
        ri = make_int4((int)r[0], (int)r[1], (int)r[2], (int)r[3]);
        xr = make_int4((int)x[0], (int)x[1], (int)x[2], (int)x[3]);
        ds = ds_unpack(w[0], w[1], w[2]);
        cnt = valid ? (int)c : 0;
    }
    if (halted_record(ctl, a.step, bj == 0)) return;
    step_housekeeping(a, ctl, c_lo, c_hi, bj, nbj, rebuilt);
    // Own record (position and species). In the form for large boxes the
    // double-single state and the list reference are read by the step tail
    // after the pair loop: reading the state here as well and again there
    // costs a second fetch, because the list stream of the loop evicts it from
    // L2. (Staging the tail's operands in LDS with asynchronous loads issued
    // here measured 0.7 us slower per launch at N = 256,000.)
    if constexpr (!SMALL) {
        if (valid) {
            ri = rec[i];
            cnt = st.nbr_cnt[i];
        }
    }
    cnt = cnt < a.g.cap ? cnt : a.g.cap;
    const int iters = cnt > l ? (cnt - l + LANES - 1) / LANES : 0;
    const float qsx = box.qs_hi[0], qsy = box.qs_hi[1], qsz = box.qs_hi[2];
    const float qlx = box.qs_lo[0], qly = box.qs_lo[1], qlz = box.qs_lo[2];
    // Pair arithmetic: d = (q_i - q_j) * quantum (wrapping difference, i.e.
    // the minimum image), u = sigma^2 / r^2, s6 = u^3. With one species the
    // per-pair constants are factored out: the lanes accumulate
    //   f' = sum s6 (2 s6 - 1) / r^2 * d,  a12 = sum s6^2,  a6 = sum s6,  an = #pairs,
    // and F = 24 eps f', sum phi_s = 4 eps (a12 - a6) - an phi(r_c),
    // sum fs r^2 = 24 eps (2 a12 - a6). With two species every pair carries
    // its own constants. Forces are accumulated in FP32; outside the quanta
    // loop the energy and virial terms are summed in FP64.
    float fx = 0.f, fy = 0.f, fz = 0.f;
    double e = 0.0, w = 0.0, a12 = 0.0, a6 = 0.0;
    int an = 0;
    const float rc2_1 = a.pc.rc2f[0], sig2_1 = a.pc.sig2f[0];
    const PairRow<float> t_rc2(a.pc.rc2f, ri.w), t_sig2(a.pc.sig2f, ri.w), t_eps24(a.pc.eps24f, ri.w),
        t_eps4(a.pc.eps4f, ri.w), t_shift(a.pc.shiftf, ri.w);
    const float c2x = box.r2c[0], c2y = box.r2c[1], c2z = box.r2c[2];
    // Outside the quanta loop: four list entries per trip (one group load),
    // all record gathers in flight before the arithmetic of the first one.
    constexpr int U = 4;
    if constexpr (Q) {
        const float rc2q = box.rc2q[0], sig2q = box.sig2q[0];
        const PairRow<float> q_rc2(box.rc2q, ri.w), q_sig2(box.sig2q, ri.w), q_f(box.fq, ri.w);
        const char *__restrict__ recb = reinterpret_cast<const char *>(rec);
        // Per lane over a few dozen pairs, in FP32: one species, sum s6^2 and
        // sum s6; two species, the pair energies and virials themselves.
        float sa = 0.f, sb = 0.f;
        static_assert((size_t)4 * kWave <= kListPad, "list padding below the unroll depth");
        auto gather = [&](const int (&jj)[UQ], int4 (&rr)[UQ]) {
            if constexpr (SMALL) {
#pragma unroll
                for (int u = 0; u < UQ; ++u) {
                    if constexpr (NS == 1) {
                        const auto r = __builtin_amdgcn_raw_buffer_load_b96(rsrc_rec, jj[u] << 4, 0, 0);
                        rr[u] = make_int4((int)r[0], (int)r[1], (int)r[2], 0);
                    } else {
                        const auto r = __builtin_amdgcn_raw_buffer_load_b128(rsrc_rec, jj[u] << 4, 0, 0);
                        rr[u] = make_int4((int)r[0], (int)r[1], (int)r[2], (int)r[3]);
                    }
                }
                return;
            }
#pragma unroll
            for (int u = 0; u < UQ; ++u) rr[u] = *reinterpret_cast<const int4 *>(recb + ((uint32_t)jj[u] << 4));
        };
        // The lane's pairs of one trip, in list order. SMALL: a pair outside
        // takes a zero reciprocal instead of a branch (every term it adds is
        // zero, so the sums are the same): with one wave per SIMD nothing
        // hides the branches.
        auto pairs = [&](const int4 (&rr)[UQ], int m) {
#pragma unroll
            for (int u = 0; u < UQ; ++u) {
                const float dx = (float)(int32_t)((uint32_t)ri.x - (uint32_t)rr[u].x);
                const float dy = (float)(int32_t)((uint32_t)ri.y - (uint32_t)rr[u].y);
                const float dz = (float)(int32_t)((uint32_t)ri.z - (uint32_t)rr[u].z);
                const float r2 = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
                const int sj = rr[u].w;
                bool in = true;
                if constexpr (SMALL)
                    in = m + u < iters && r2 < (NS == 1 ? rc2q : q_rc2(sj));
                else if (!(m + u < iters && r2 < (NS == 1 ? rc2q : q_rc2(sj))))
                    continue;
                const float ir2 = in ? __builtin_amdgcn_rcpf(r2) : 0.0f;
                const float s2 = (NS == 1 ? sig2q : q_sig2(sj)) * ir2;
                const float s6 = s2 * s2 * s2;
                float t = (s6 * ir2) * fmaf(2.0f, s6, -1.0f);
                if constexpr (NS == 2) t *= q_f(sj);
                fx = fmaf(t, dx, fx);
                fy = fmaf(t, dy, fy);
                fz = fmaf(t, dz, fz);
                if constexpr (OBS) {
                    if constexpr (NS == 1) {
                        sa = fmaf(s6, s6, sa);
                        sb += s6;
                        an += in ? 1 : 0;
                    } else {
                        const float s12 = s6 * s6;
                        sa += fmaf(t_eps4(sj), s12 - s6, in ? -t_shift(sj) : 0.0f);
                        sb += t_eps24(sj) * fmaf(2.0f, s12, -s6);
                    }
                }
            }
        };
        if constexpr (SMALL) {
            // Software pipeline over the trips of the wave's longest list: the
            // records of one trip and the entries of the one after are in
            // flight while a trip's pairs are evaluated, so a wave that has
            // its SIMD to itself waits for about one memory latency in all
            // instead of two per trip.
            const int trips =
                (__builtin_amdgcn_readlane((int)wave_max_last((uint32_t)iters), kWave - 1) + UQ - 1) / UQ;
            if (trips > 0) {
                int4 ra[UQ], rb[UQ];
                gather(jn, ra);
                entries(UQ * min(1, trips - 1), jn);
                int t = 0;
                for (; t + 2 < trips; t += 2) {
                    gather(jn, rb);
                    entries(UQ * (t + 2), jn);
                    __builtin_amdgcn_sched_barrier(0);
                    pairs(ra, UQ * t);
                    __builtin_amdgcn_sched_barrier(0);
                    gather(jn, ra);
                    entries(UQ * min(t + 3, trips - 1), jn);
                    __builtin_amdgcn_sched_barrier(0);
                    pairs(rb, UQ * (t + 1));
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (t + 1 < trips) {
                    gather(jn, rb);
                    __builtin_amdgcn_sched_barrier(0);
                    pairs(ra, UQ * t);
                    pairs(rb, UQ * (t + 1));
                } else {
                    pairs(ra, UQ * t);
                }
            }
        } else {
            // What bounds the kernel here is the gathers: a compute unit's
            // cache takes one to two lanes of them per clock, hit or not (0.98
            // random, 1.93 in list order, against 4.2 from LDS), so the 19
            // million of N = 256,000 take 16 to 32 us by themselves. Fewer
            // vector instructions change nothing; branchless pairs, whose lanes all
            // stay active, cost 38 us. (The block's partners copied to LDS
            // gave 27.8 us, but making the lists of their places took 76 us
            // per list build.)
            // Eight entries per trip (two 16-byte group loads per lane) keep
            // more of the list stream in flight; groups past a list end read
            // padding or other lists (valid indices) and are skipped. (Masking
            // the loads of entries past a lane's list end instead, per entry,
            // serialised them: 38.5 us against 30.3 us per launch at
            // N = 256,000.)
            for (int m = 0; m < iters; m += UQ) {
                int jj[UQ];
                int4 rr[UQ];
                entries(m, jj);
                gather(jj, rr);
                pairs(rr, m);
            }
        }
        if constexpr (NS == 1) {
            a12 = (double)sa;
            a6 = (double)sb;
        } else {
            e = (double)sa;
            w = (double)sb;
        }
    } else {
    for (int m = 0; m < iters; m += U) {
        // One 16-byte group load per lane: its four entries m .. m+3 (entries
        // past the list end are valid indices and are skipped).
        static_assert(U == 4, "one entry group per trip");
        const int4 grp = *reinterpret_cast<const int4 *>(nb + ((int64_t)(m >> 2) << 8));
        const int jj[U] = {grp.x, grp.y, grp.z, grp.w};
        int4 rr[U];
#pragma unroll
        for (int u = 0; u < U; ++u) rr[u] = rec[jj[u]];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (m + u >= iters) continue;
            const int4 rj = rr[u];
            const float dx = (float)(int32_t)((uint32_t)ri.x - (uint32_t)rj.x) * qsx;
            const float dy = (float)(int32_t)((uint32_t)ri.y - (uint32_t)rj.y) * qsy;
            const float dz = (float)(int32_t)((uint32_t)ri.z - (uint32_t)rj.z) * qsz;
            // d carries the single-float quantum's relative rounding (a few
            // 1e-8, the same for every pair); r^2 takes it out exactly per axis.
            const float r2 = fmaf(dz * c2z, dz, fmaf(dy * c2y, dy, (dx * c2x) * dx));
            if constexpr (NS == 1) {
                if (r2 < rc2_1) {
                    const float ir2 = __builtin_amdgcn_rcpf(r2);
                    const float s2 = sig2_1 * ir2;
                    const float s6 = s2 * s2 * s2;
                    const float t = (s6 * ir2) * fmaf(2.0f, s6, -1.0f);
                    fx = fmaf(t, dx, fx);
                    fy = fmaf(t, dy, fy);
                    fz = fmaf(t, dz, fz);
                    a12 += (double)(s6 * s6);
                    a6 += (double)s6;
                    an += 1;
                }
            } else {
                const int sj = rj.w;
                if (r2 < t_rc2(sj)) {
                    const float ir2 = __builtin_amdgcn_rcpf(r2);
                    const float s2 = t_sig2(sj) * ir2;
                    const float s6 = s2 * s2 * s2;
                    const float s12 = s6 * s6;
                    const float c24 = t_eps24(sj);
                    const float fs = c24 * ((s6 * ir2) * fmaf(2.0f, s6, -1.0f));
                    fx = fmaf(fs, dx, fx);
                    fy = fmaf(fs, dy, fy);
                    fz = fmaf(fs, dz, fz);
                    e += (double)fmaf(t_eps4(sj), s12 - s6, -t_shift(sj));
                    w += (double)(c24 * fmaf(2.0f, s12, -s6));
                }
            }
        }
    }
    }
    if constexpr (LANES > 1) {
        // The particle's lanes exchange their sums: within a quad by DPP
        // moves (no LDS round trip), wider by shuffles.
        auto xsum = [](auto &v, int o) {
            using V = std::remove_reference_t<decltype(v)>;
            if (o == 1 || o == 2) {
                if constexpr (std::is_same_v<V, double>) v += o == 1 ? dpp_d<kDppXor1>(v) : dpp_d<kDppXor2>(v);
                else if constexpr (std::is_same_v<V, float>) v += o == 1 ? dpp_f<kDppXor1>(v) : dpp_f<kDppXor2>(v);
                else v += (V)(o == 1 ? dpp_u<kDppXor1>((uint32_t)v) : dpp_u<kDppXor2>((uint32_t)v));
            } else {
                v += __shfl_xor(v, o);
            }
        };
#pragma unroll
        for (int o = LANES / 2; o > 0; o >>= 1) {
            xsum(fx, o);
            xsum(fy, o);
            xsum(fz, o);
            if constexpr (NS == 1) {
                if constexpr (OBS) {
                    xsum(a12, o);
                    xsum(a6, o);
                    xsum(an, o);
                }
            } else {
                xsum(e, o);
                xsum(w, o);
            }
        }
    }
    if constexpr (NS == 1) {
        const float c24 = Q ? box.fq[0] : a.pc.eps24f[0];
        fx *= c24;
        fy *= c24;
        fz *= c24;
        e = a.pc.eps4[0] * (a12 - a6) - (double)an * a.pc.shift[0];
        w = a.pc.eps24[0] * (2.0 * a12 - a6);
    }
    double pu = 0.0, pw = 0.0, pk = 0.0, ppx = 0.0, ppy = 0.0, ppz = 0.0;
    uint32_t dm = 0u;
    if (valid && l == 0) {
        if constexpr (!SMALL) {
            xr = st.xref[i];
            ds = ds_load(st.dsw, i);
        }
        finish_ds<OBS, TH, PLAIN>(a, box, i, ri.w, xr, ds, fx, fy, fz, e, w, pu, pw, pk, ppx, ppy, ppz, dm);
    }
    block_finish<OBS, BS>(a, ctl, blk, pu, pw, pk, ppx, ppy, ppz, dm);
}

// PLAIN: the single-precision state (positions and velocities as single
// floats) instead of double-single.
template <int NS, int LANES, bool Q, bool OBS, bool TH, bool PLAIN>
__global__ __launch_bounds__(kBlock) void k_step_ds(StepArgs a) {
    static_assert(OBS || Q, "observables are skipped on the quanta path only");
    step_ds_body<NS, LANES, Q, OBS, TH, PLAIN>(a, a.box, a.st.ctl, xcd_remap(blockIdx.x, gridDim.x), a.g.n, 0,
                                               a.box.ncell, blockIdx.x, gridDim.x, rebuilt_mark(a));
}
// Two species, NVE: held to 64 VGPRs, eight waves per SIMD (unbounded it
// takes 65-66 and drops to seven; the 4M mixture's step kernel measured
// 727 -> 683 us). The thermostat's form would spill under that bound.
template <int LANES, bool Q, bool OBS, bool PLAIN>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(8))) void k_step_ds_mix(StepArgs a) {
    static_assert(OBS || Q, "observables are skipped on the quanta path only");
    step_ds_body<2, LANES, Q, OBS, false, PLAIN>(a, a.box, a.st.ctl, xcd_remap(blockIdx.x, gridDim.x), a.g.n, 0,
                                                 a.box.ncell, blockIdx.x, gridDim.x, rebuilt_mark(a));
}
template <int NS, int LANES, bool Q, bool OBS, bool TH, bool PLAIN>
constexpr void (*step_ds_kernel())(StepArgs) {
    if constexpr (NS == 2 && !TH)
        return k_step_ds_mix<LANES, Q, OBS, PLAIN>;
    else
        return k_step_ds<NS, LANES, Q, OBS, TH, PLAIN>;
}

// The form for small boxes, two lanes per particle (the default layout). A
// wave has its SIMD nearly to itself, so the kernel is a chain of latencies;
// at 7,000 particles cycle stamps put it at 14,400 cycles (8,300 in the pair
// loop, about six cycles per instruction; 20,100 and 11,700 before the loads
// were pipelined and asked for ahead).
template <int NS, bool OBS, bool TH, bool PLAIN>
__global__ __launch_bounds__(kBlockSmall) void k_step_ds_small(StepArgs a) {
    step_ds_body<NS, 2, true, OBS, TH, PLAIN, kBlockSmall, true>(a, a.box, a.st.ctl, xcd_remap(blockIdx.x, gridDim.x),
                                                                 a.g.n, 0, a.box.ncell, blockIdx.x, gridDim.x,
                                                                 rebuilt_mark(a));
}

// The form for large boxes in blocks of 256 threads (see fine_blocks); eight
// waves per SIMD but for the thermostat, whose form would spill.
template <int NS, bool OBS, bool TH, bool PLAIN>
__global__ __launch_bounds__(kBlockSmall, (TH ? 4 : 8)) void k_step_ds_fine(StepArgs a) {
    step_ds_body<NS, 2, true, OBS, TH, PLAIN, kBlockSmall>(a, a.box, a.st.ctl, xcd_remap(blockIdx.x, gridDim.x), a.g.n,
                                                           0, a.box.ncell, blockIdx.x, gridDim.x,
                                                           rebuilt_mark(a));
}

// A batch of independent one-species cubic systems, each over its own run of
// blocks (particle ranges padded to whole blocks): the block finds its
// system, then runs the same body with that system's box and control words.
template <int LANES, bool OBS>
__global__ __launch_bounds__(kBlock) void k_batch_step(StepArgs a, const SysC *sys, const int32_t *sys_of_g16) {
    const int blk = xcd_remap(blockIdx.x, gridDim.x);
    const int64_t first = (int64_t)blk * (kBlock / LANES);
    const SysC &y = sys[sys_of_g16[first >> 4]];
    step_ds_body<1, LANES, true, OBS>(a, y.box, a.st.ctl + y.id, blk, y.p_off + y.n, y.c_off, y.c_off + y.box.ncell,
                                 blk - y.b_off, y.nb, nullptr);
}

// ---------------------------------------------------------------- FP64 ---
// SMALL: the form for boxes that leave the chip's wave slots mostly empty, as
// in the single-precision body: loads through buffer descriptors, everything
// outside the trips asked for at once, one trip's records and the next trip's
// entries in flight while a trip's pairs are evaluated. The same sums in the
// same order.
template <int NS, int LANES, bool TH, bool SMALL>
__device__ inline void step_fp64_body(const StepArgs &a) {
    constexpr int P = kWave / LANES;
    constexpr int WPB = kBlockF64 / kWave;
    constexpr int U = 4;  // list entries of a lane per trip: one group load
    const State &st = a.st;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int blk = xcd_remap(blockIdx.x, gridDim.x);
    const int64_t chunk = (int64_t)blk * WPB + wv;
    const int l = lane % LANES;
    const int64_t i = chunk * P + lane / LANES;
    const bool valid = i < a.g.n;
    const double4 *__restrict__ rec = st.rec64[a.cur];
    const int32_t *__restrict__ nb = st.nbr + chunk * (int64_t)(P * a.g.cap) + 4 * lane;
    double4 ri = make_double4(0, 0, 0, 0);
    int cnt = 0;
    [[maybe_unused]] __amdgpu_buffer_rsrc_t rsrc_rec, rsrc_nb;
    [[maybe_unused]] int jn[U];
    [[maybe_unused]] double4 vel;
    [[maybe_unused]] int4 xr;
    auto entries = [&](int m, int (&jj)[U]) {
        if constexpr (SMALL) {
            const auto g = __builtin_amdgcn_raw_buffer_load_b128(rsrc_nb, lane << 4, m << 8, 0);
#pragma unroll
            for (int u = 0; u < U; ++u) jj[u] = (int)g[u];
        } else {
            const int4 g = *reinterpret_cast<const int4 *>(nb + ((int64_t)(m >> 2) << 8));
            jj[0] = g.x, jj[1] = g.y, jj[2] = g.z, jj[3] = g.w;
        }
    };
    auto load4 = [](const __amdgpu_buffer_rsrc_t &rs, int off) {
        const auto p = __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0);
        const auto q = __builtin_amdgcn_raw_buffer_load_b128(rs, off + 16, 0, 0);
        auto d = [](uint32_t lo, uint32_t hi) { return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo)); };
        return make_double4(d(p[0], p[1]), d(p[2], p[3]), d(q[0], q[1]), d(q[2], q[3]));
    };
    auto gather = [&](const int (&jj)[U], double4 (&rr)[U]) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if constexpr (SMALL) rr[u] = load4(rsrc_rec, jj[u] << 5);
            else rr[u] = rec[jj[u]];
        }
    };
    if constexpr (SMALL) {
        auto rsrc = [](const void *p, int64_t bytes) {
            return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, kRawBuffer);
        };
        const int64_t wchunk = __builtin_amdgcn_readfirstlane((int)chunk);
        rsrc_rec = rsrc(rec, a.g.n << 5);
        rsrc_nb = rsrc(st.nbr + wchunk * (P * a.g.cap), wchunk * P < a.g.n ? P * a.g.cap * 4 + kListPad * 4 : 0);
        const uint32_t c = __builtin_amdgcn_raw_buffer_load_b32(rsrc(st.nbr_cnt, a.g.n << 2), (int)i << 2, 0, 0);
        ri = load4(rsrc_rec, (int)i << 5);
        entries(0, jn);
        const auto x = __builtin_amdgcn_raw_buffer_load_b128(rsrc(st.xref, a.g.n << 4), (int)i << 4, 0, 0);
        vel = load4(rsrc(st.vel64, a.g.n << 5), (int)i << 5);
        // One word of every 64-byte line of the kernel arguments.
        const auto *arg = (const __attribute__((address_space(4))) int *)__builtin_amdgcn_kernarg_segment_ptr();
        int touch = 0;
#pragma unroll
        for (int k = 0; k < (int)((sizeof(StepArgs) + 63) / 64); ++k) touch |= arg[k * 16];
        asm volatile("" ::"s"(touch));
        __builtin_amdgcn_sched_barrier(0);
        xr = make_int4((int)x[0], (int)x[1], (int)x[2], (int)x[3]);
        cnt = valid ? (int)c : 0;
    }
    if (halted_record(a.st.ctl, a.step, blockIdx.x == 0)) return;
    step_housekeeping(a, a.st.ctl, 0, a.box.ncell, blockIdx.x, gridDim.x, rebuilt_mark(a));
    if constexpr (!SMALL) {
        if (valid) {
            ri = rec[i];
            cnt = st.nbr_cnt[i];
        }
    }
    const int si = (int)ri.w;
    cnt = cnt < a.g.cap ? cnt : a.g.cap;
    const int iters = cnt > l ? (cnt - l + LANES - 1) / LANES : 0;
    double fx = 0, fy = 0, fz = 0, e = 0, w = 0;
    const PairRow<double> t_rc2(a.pc.rc2, si), t_sig2(a.pc.sig2, si), t_eps24(a.pc.eps24, si),
        t_eps4(a.pc.eps4, si), t_shift(a.pc.shift, si);
    // The lane's pairs of one trip, in list order (entries past the list end
    // are valid indices and are skipped).
    auto pairs = [&](const double4 (&rr)[U], int m) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (m + u >= iters) continue;
            const double4 rj = rr[u];
            const double dx = disp_d(ri.x, rj.x, a.box.L[0], a.box.invL[0]);
            const double dy = disp_d(ri.y, rj.y, a.box.L[1], a.box.invL[1]);
            const double dz = disp_d(ri.z, rj.z, a.box.L[2], a.box.invL[2]);
            const double r2 = fma(dz, dz, fma(dy, dy, dx * dx));
            const int sj = (int)rj.w;
            if (r2 < (NS == 1 ? a.pc.rc2[0] : t_rc2(sj))) {
                // Reciprocal: hardware estimate refined by two Newton steps.
                double ir2 = __builtin_amdgcn_rcp(r2);
                ir2 = fma(ir2, fma(-r2, ir2, 1.0), ir2);
                ir2 = fma(ir2, fma(-r2, ir2, 1.0), ir2);
                const double s2 = (NS == 1 ? a.pc.sig2[0] : t_sig2(sj)) * ir2;
                const double s6 = s2 * s2 * s2;
                const double fs = (NS == 1 ? a.pc.eps24[0] : t_eps24(sj)) * s6 * fma(2.0, s6, -1.0) * ir2;
                fx = fma(fs, dx, fx);
                fy = fma(fs, dy, fy);
                fz = fma(fs, dz, fz);
                e += fma((NS == 1 ? a.pc.eps4[0] : t_eps4(sj)) * s6, s6 - 1.0,
                         -(NS == 1 ? a.pc.shift[0] : t_shift(sj)));
                w = fma(fs, r2, w);
            }
        }
    };
    if constexpr (SMALL) {
        const int trips = (__builtin_amdgcn_readlane((int)wave_max_last((uint32_t)iters), kWave - 1) + U - 1) / U;
        if (trips > 0) {
            double4 ra[U], rb[U];
            gather(jn, ra);
            entries(U * min(1, trips - 1), jn);
            int t = 0;
            for (; t + 2 < trips; t += 2) {
                gather(jn, rb);
                entries(U * (t + 2), jn);
                __builtin_amdgcn_sched_barrier(0);
                pairs(ra, U * t);
                __builtin_amdgcn_sched_barrier(0);
                gather(jn, ra);
                entries(U * min(t + 3, trips - 1), jn);
                __builtin_amdgcn_sched_barrier(0);
                pairs(rb, U * (t + 1));
                __builtin_amdgcn_sched_barrier(0);
            }
            if (t + 1 < trips) {
                gather(jn, rb);
                __builtin_amdgcn_sched_barrier(0);
                pairs(ra, U * t);
                pairs(rb, U * (t + 1));
            } else {
                pairs(ra, U * t);
            }
        }
    } else {
        for (int m = 0; m < iters; m += U) {
            int jj[U];
            double4 rr[U];
            entries(m, jj);
            gather(jj, rr);
            pairs(rr, m);
        }
    }
    if constexpr (LANES > 1) {
        // The particle's lanes exchange their sums: wide steps by shuffles,
        // within a quad by DPP moves (no LDS round trip).
        auto xsum = [](double &v) {
            if constexpr (LANES >= 16) v += __shfl_xor(v, 8);
            if constexpr (LANES >= 8) v += __shfl_xor(v, 4);
            if constexpr (LANES >= 4) v += dpp_d<kDppXor2>(v);
            v += dpp_d<kDppXor1>(v);
        };
        xsum(fx);
        xsum(fy);
        xsum(fz);
        xsum(e);
        xsum(w);
    }
    double pu = 0.0, pw = 0.0, pk = 0.0, ppx = 0.0, ppy = 0.0, ppz = 0.0;
    uint32_t dm = 0u;
    if (valid && l == 0) {
        if constexpr (!SMALL) {
            vel = st.vel64[i];
            xr = st.xref[i];
        }
        finish_fp64<TH>(a, a.box, i, ri, vel, xr, fx, fy, fz, e, w, pu, pw, pk, ppx, ppy, ppz, dm);
    }
    block_finish<true, kBlockF64>(a, a.st.ctl, blk, pu, pw, pk, ppx, ppy, ppz, dm);
}

template <int NS, int LANES, bool TH>
__global__ __launch_bounds__(kBlockF64) void k_step_fp64(StepArgs a) {
    step_fp64_body<NS, LANES, TH, false>(a);
}
// Small boxes, four lanes per particle (the default layout).
template <int NS, bool TH>
__global__ __launch_bounds__(kBlockF64) void k_step_fp64_small(StepArgs a) {
    step_fp64_body<NS, 4, TH, true>(a);
}

// Start of a run: "integrate" from the stored forces of the current step
// (the tail of a step with only its integrate half: a.mode is kIntegrate).
template <int PREC>
__device__ inline void integrate_body(const StepArgs &a, const BoxC &box, Ctl *ctl, int64_t i_end) {
    const State &st = a.st;
    if (halted(ctl)) return;
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    uint32_t dm = 0u;
    double pu, pw, pk, ppx, ppy, ppz;
    if (i < i_end) {
        if constexpr (PREC == LJMD_FP64) {
            const double4 f = st.frc64[i];
            finish_fp64<false>(a, box, i, st.rec64[a.cur][i], st.vel64[i], st.xref[i], f.x, f.y, f.z, 0.0, 0.0, pu, pw,
                               pk, ppx, ppy, ppz, dm);
        } else {
            const float4 f = st.frc32[i];
            finish_ds<false, false, PREC == LJMD_FP32>(a, box, i, st.recq[a.cur][i].w, st.xref[i],
                                                       ds_load(st.dsw, i), f.x, f.y, f.z, 0.0,
                                                       0.0, pu,
                                                       pw, pk, ppx, ppy, ppz, dm);
        }
    }
    dm = wave_max_u(dm);
    if ((threadIdx.x & 63) == 0 && dm > __float_as_uint(a.dyn.thr2)) {
        atomicMax(&ctl->maxd[(a.step + 1) & 1], dm);
        if (dm > 0x7f800000u) atomicOr(&ctl->flags, kErrNaN);
    }
}

template <int PREC>
__global__ __launch_bounds__(kBlock) void k_integrate(StepArgs a) {
    integrate_body<PREC>(a, a.box, a.st.ctl, a.g.n);
}

// Batch form: systems are padded to whole step-kernel blocks (at least 64
// slots), so the 64 slots of a wave lie inside one system.
__global__ __launch_bounds__(kBlock) void k_batch_integrate(StepArgs a, const SysC *sys, const int32_t *sys_of_g16,
                                                            int64_t nslots) {
    const int64_t w0 = (int64_t)blockIdx.x * kBlock + (threadIdx.x & ~(kWave - 1));
    if (w0 >= nslots) return;
    const SysC &y = sys[sys_of_g16[w0 >> 4]];
    integrate_body<LJMD_FP32_DS>(a, y.box, a.st.ctl + y.id, y.p_off + y.n);
}

// ------------------------------------------------------------------------
int step_blocks(const Geom &g) {
    const int per_block = (step_block_threads(g.prec) / kWave) * (kWave / g.lanes);
    return (int)((g.n + per_block - 1) / per_block);
}

static StepArgs make_args(const Launch &L, int64_t step, int forced, int mode, int slot) {
    StepArgs a;
    a.st = *L.st;
    a.g = *L.g;
    a.box = *L.box;
    a.pc = *L.pc;
    a.dyn = *L.dyn;
    a.cur = L.cur;
    a.forced = forced;
    a.mode = mode;
    a.slot = slot;
    a.step = step;
    return a;
}

// Whether the step kernel for large boxes runs in blocks of 256 threads
// (quarters) instead of 1024. Two blocks of 1024 fit a compute unit, so their
// kernel takes as long as the most loaded unit: 18.5 us with one block for
// each, 29.5 with two, 40 with three, 50 with four, whatever n in between.
// Quarters even that out, at a tenth more time for the same load (neighbouring
// particles in one block share its compute unit's cache). 1024 against 256
// threads: 68,000 particles 18.7 / 15.0 us, 90,000 18.4 / 15.9, 100,000 18.6 /
// 19.2, 133,000 28.2 / 22.8, 160,000 29.3 / 23.9, 200,000 29.2 / 28.2, 256,000
// 30.0 / 31.6, 270,000 39.1 / 34.5, 320,000 40.3 / 38.2, 360,000 40.4 / 41.7,
// 400,000 50.4 / 46.6; from 600,000 on (76.1 / 80.3) the blocks that follow
// the first round even it out.
// The thermostat's kernel holds 84 registers, more than two blocks of 1024
// leave room for: it always takes quarters (100,000 particles 21.0 / 20.6,
// 256,000 37.2 / 35.1, 1,000,000 158.8 / 137.8; see launch_step).
static bool fine_blocks(const Geom &g) {
    const int64_t ncu = g.ncu > 0 ? g.ncu : 256;
    const int64_t whole = (g.n + kBlock / 2 - 1) / (kBlock / 2), quarters = (g.n + kBlockSmall / 2 - 1) / (kBlockSmall / 2);
    const int64_t load = (whole + ncu - 1) / ncu, load4 = (quarters + ncu - 1) / ncu;
    return load <= 4 && 11 * load4 < 40 * load;
}

// The kernels in blocks of 1024 threads, and every other layout than two lanes
// in a cubic box. The thermostat has no such kernel for that layout.
template <int NS, int LN, bool TH, bool PL>
static hipError_t step_ds_launch(const Launch &L, dim3 grid, dim3 block, const StepArgs &a, bool quanta, bool obs) {
    if (!quanta) {
        launch_k(L, step_ds_kernel<NS, LN, false, true, TH, PL>(), grid, block, a);
        return hipGetLastError();
    }
    if constexpr (LN == 2 && TH) {
        return hipErrorInvalidDeviceFunction;
    } else {
        if (obs)
            launch_k(L, step_ds_kernel<NS, LN, true, true, TH, PL>(), grid, block, a);
        else
            launch_k(L, step_ds_kernel<NS, LN, true, false, TH, PL>(), grid, block, a);
        return hipGetLastError();
    }
}

hipError_t launch_step(const Launch &L, int64_t step, int forced, int mode, int slot) {
    if (L.g->all_pairs) return launch_allpairs_step(L, step, mode, slot);
    StepArgs a = make_args(L, step, forced, mode, slot);
    dim3 grid(step_blocks(*L.g)), block(step_block_threads(L.g->prec));
    const bool ds = L.g->prec != LJMD_FP64;
    const bool plain = L.g->prec == LJMD_FP32;
    const bool two = L.g->nspecies == 2;
    const bool quanta = ds && L.box->cubic && L.g->n < kQuantaMaxSlots;
    const bool obs = (mode & kObserve) != 0;
    // The thermostat acts on "finalize" only.
    const bool th = L.dyn->thermo_on && (mode & kFinalize);
    // At most two wavefronts per SIMD (256 particles per compute unit): nothing
    // hides a wave's chain of loads then, and 1024-thread blocks leave compute
    // units empty. Step kernel at 7,000 / 32,000 / 64,000 particles: 16.6 /
    // 16.8 / 17.9 us with the form for large boxes, 9.6 / 10.0 / 13.0 us with
    // this one; at 100,000 18.6 against 19.4 us, at 256,000 30.1 against 32.1.
    const bool few_waves = L.g->n <= (int64_t)256 * (L.g->ncu > 0 ? L.g->ncu : 256);
    const bool small = quanta && L.g->lanes == 2 && few_waves;
    if (small || (quanta && L.g->lanes == 2 && (th || fine_blocks(*L.g)))) {
        const dim3 gs((unsigned)L.g->max_blocks), bs(kBlockSmall);  // every row of partials is written
#define STEP_256(K, NS, OB)                                                          \
    do {                                                                             \
        if (th && plain)                                                             \
            launch_k(L, K<NS, OB, true, true>, gs, bs, a);                           \
        else if (th)                                                                 \
            launch_k(L, K<NS, OB, true, false>, gs, bs, a);                          \
        else if (plain)                                                              \
            launch_k(L, K<NS, OB, false, true>, gs, bs, a);                          \
        else                                                                         \
            launch_k(L, K<NS, OB, false, false>, gs, bs, a);                         \
    } while (0)
#define STEP_256_OBS(K)                      \
    do {                                     \
        if (two && obs) STEP_256(K, 2, true);  \
        else if (two) STEP_256(K, 2, false);   \
        else if (obs) STEP_256(K, 1, true);    \
        else STEP_256(K, 1, false);            \
    } while (0)
        if (small) STEP_256_OBS(k_step_ds_small);
        else STEP_256_OBS(k_step_ds_fine);
#undef STEP_256_OBS
#undef STEP_256
        return hipGetLastError();
    }
    // FP64, by the same rule (four waves per SIMD then): step kernel at 2,000 /
    // 32,000 / 64,000 particles 11.1 / 13.3 / 18.2 us with the other form, 9.2 /
    // 11.9 / 17.7 us with this one; at 256,000 48.7 against 49.8.
    if (!ds && L.g->lanes == 4 && few_waves) {
        if (two && th) launch_k(L, k_step_fp64_small<2, true>, grid, block, a);
        else if (two) launch_k(L, k_step_fp64_small<2, false>, grid, block, a);
        else if (th) launch_k(L, k_step_fp64_small<1, true>, grid, block, a);
        else launch_k(L, k_step_fp64_small<1, false>, grid, block, a);
        return hipGetLastError();
    }
#define STEP_TH(NS, LN, TH)                                                             \
    do {                                                                                \
        if (ds && plain)                                                                \
            return step_ds_launch<NS, LN, TH, true>(L, grid, block, a, quanta, obs);    \
        if (ds)                                                                         \
            return step_ds_launch<NS, LN, TH, false>(L, grid, block, a, quanta, obs);   \
        launch_k(L, k_step_fp64<NS, LN, TH>, grid, block, a);                           \
    } while (0)
#define STEP(NS, LN)              \
    do {                          \
        if (th)                   \
            STEP_TH(NS, LN, true);  \
        else                      \
            STEP_TH(NS, LN, false); \
    } while (0)
#define BY_LANES(NS)                          \
    switch (L.g->lanes) {                     \
        case 1: STEP(NS, 1); break;           \
        case 2: STEP(NS, 2); break;           \
        case 4: STEP(NS, 4); break;           \
        case 8: STEP(NS, 8); break;           \
        default: STEP(NS, 16); break;         \
    }
    if (two) {
        BY_LANES(2);
    } else {
        BY_LANES(1);
    }
#undef BY_LANES
#undef STEP
#undef STEP_TH
    return hipGetLastError();
}

hipError_t launch_integrate(const Launch &L, int64_t step) {
    StepArgs a = make_args(L, step, 0, kIntegrate, 0);
    dim3 grid((unsigned)((L.g->n + kBlock - 1) / kBlock)), block(kBlock);
    if (L.g->prec == LJMD_FP64)
        hipLaunchKernelGGL(k_integrate<LJMD_FP64>, grid, block, 0, L.stream, a);
    else if (L.g->prec == LJMD_FP32)
        hipLaunchKernelGGL(k_integrate<LJMD_FP32>, grid, block, 0, L.stream, a);
    else
        hipLaunchKernelGGL(k_integrate<LJMD_FP32_DS>, grid, block, 0, L.stream, a);
    return hipGetLastError();
}


hipError_t launch_batch_step(const Launch &L, const SysC *sys, const int32_t *sys_of_g16, int nblocks,
                             int64_t step, int forced, int mode, int slot) {
    StepArgs a = make_args(L, step, forced, mode, slot);
    const dim3 grid((unsigned)nblocks), block(kBlock);
#define BSTEP(LN)                                                                                        \
    do {                                                                                                 \
        if (mode & kObserve)                                                                             \
            hipLaunchKernelGGL((k_batch_step<LN, true>), grid, block, 0, L.stream, a, sys, sys_of_g16);  \
        else                                                                                             \
            hipLaunchKernelGGL((k_batch_step<LN, false>), grid, block, 0, L.stream, a, sys, sys_of_g16); \
    } while (0)
    switch (L.g->lanes) {
        case 1: BSTEP(1); break;
        case 2: BSTEP(2); break;
        case 4: BSTEP(4); break;
        case 8: BSTEP(8); break;
        default: BSTEP(16); break;
    }
#undef BSTEP
    return hipGetLastError();
}

hipError_t launch_batch_integrate(const Launch &L, const SysC *sys, const int32_t *sys_of_g16, int64_t nslots,
                                  int64_t step) {
    StepArgs a = make_args(L, step, 0, kIntegrate, 0);
    const dim3 grid((unsigned)((nslots + kBlock - 1) / kBlock)), block(kBlock);
    hipLaunchKernelGGL(k_batch_integrate, grid, block, 0, L.stream, a, sys, sys_of_g16, nslots);
    return hipGetLastError();
}

}  // namespace ljmd
