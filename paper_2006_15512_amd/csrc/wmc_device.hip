// Execution stage on gfx950 for one plan: the pairwise contractions of
// Algorithm 2 over the slices of Algorithm 3, all on the device.  Kernels
// and their numerics are in wmc_kernels.h.
#include <mutex>

#include "wmc_chain.h"

// Optional per-launch timing: an event is recorded on the stream after every
// launch; ms[k] accumulates launch k's duration over the slices.
struct LaunchTimer {
    std::vector<hipEvent_t> ev;
    float *ms = nullptr;
    int64_t cap = 0;
    size_t k = 0;
    hipStream_t st = nullptr;
    void mark() {
        if (!ms) return;
        if (k < ev.size()) (void)hipEventRecord(ev[k], st);
        ++k;
    }
};

// Weights into the workspace: the caller's 2 * n_user (or the network's),
// then the constant (1, 1) of auxiliary variables from the plan.
static hipError_t upload_weights(const wmc_plan_t &P, const double *weights, char *ws, hipStream_t st) {
    const double *w = weights ? weights : P.w.data();
    hipError_t e = hipSuccess;
    if (P.n_user > 0) e = hipMemcpyAsync(ws + P.off_w, w, sizeof(double) * 2 * (size_t)P.n_user, hipMemcpyHostToDevice, st);
    if (e == hipSuccess && P.n > P.n_user)
        e = hipMemcpyAsync(ws + P.off_w + sizeof(double) * 2 * (size_t)P.n_user, P.w.data() + 2 * (size_t)P.n_user,
                           sizeof(double) * 2 * (size_t)(P.n - P.n_user), hipMemcpyHostToDevice, st);
    return e;
}

// Lanes per summed-index group of a streaming node of the plan: the tuned
// split for FP64 nodes with K >= 16 (instances exist for K of 16 and 32).
template <typename T>
static inline int split_lanes_of(const wmc_plan_t &P, int nk) {
    return sizeof(T) == 8 && nk >= 4 && nk <= 5 ? P.tune.split_lanes : 0;
}

// Kernel family that runs a single node alone (mat: its matrix descriptor,
// or null), with the streaming kernels' arguments filled in when one of them
// is chosen.  The executor and wmc_plan_kernels share this choice.
template <typename T>
static int node_kernel(const wmc_plan_t &P, const NodeDesc &d, const GemmDesc *mat, Stream2Tab *tb, StreamMfmaArgs *ma) {
    if (mat) return gemm_persistent<T>(*mat) ? WMC_KERNEL_GEMM_P : WMC_KERNEL_GEMM;
    if (d.cls == WMC_CLASS_STREAM) {
        const wmc_tuning &tu = P.tune;
        if (tu.stream_mfma_min_bits > 0 && stream_mfma_args(d, ma, tu.stream_mfma_min_bits)) return WMC_KERNEL_STREAM_MFMA;
        if (stream2_args(d, &tb->a, tu.stream2_tile_bits, tu.stream2_min_thread_bits, tu.stream2_low_bits,
                         tu.stream2_vec != 0)) {
            const int lg = tb->a.vec ? 0 : split_lanes_of<T>(P, d.nk);
            // work items per workgroup: 256 threads, or 256 / lg lane groups
            if (stream2_tab(tb, lg > 0 ? 8 - (lg == 4 ? 2 : lg == 2 ? 1 : 3) : 8))
                return tb->a.vec ? WMC_KERNEL_STREAM2_VEC : lg > 0 ? WMC_KERNEL_STREAM2_SPLIT : WMC_KERNEL_STREAM2;
        }
    }
    return WMC_KERNEL_NODES;
}

// The same for node launch k (1 <= k < P.launches.size()) of the plan's
// general launch list.
template <typename T>
static int solo_kernel(const wmc_plan_t &P, size_t k, Stream2Tab *tb, StreamMfmaArgs *ma) {
    const Launch &Ln = P.launches[k];
    if (Ln.type != LAUNCH_GEMM && Ln.count != 1) return WMC_KERNEL_NODES;
    return node_kernel<T>(P, P.nodes[(size_t)Ln.first], Ln.type == LAUNCH_GEMM ? &P.gemms[(size_t)Ln.pad] : nullptr, tb,
                          ma);
}

// Launches one node alone on the kernel family `kern`; false if no instance
// covers it (nothing launched).
template <typename T>
static bool launch_node(const wmc_plan_t &P, int kern, const NodeDesc &d, const GemmDesc *mat, const GemmDesc *mat_dev,
                        const Stream2Tab &sa, const StreamMfmaArgs &ma, T *arena, wmc_meta *meta, hipStream_t st,
                        const SliceGroup sg, unsigned nz) {
    switch (kern) {
    case WMC_KERNEL_GEMM_P:
    case WMC_KERNEL_GEMM:
        launch_gemm<T>(*mat, mat_dev, arena, meta, st, sg, nz, GemmShape{P.tune.gemm_tpw_max_nt, P.tune.gemm_orient});
        return true;
    case WMC_KERNEL_STREAM_MFMA:
        launch_stream_mfma<T>(ma, d.nk, arena, meta, st, (unsigned)P.tune.stream_mfma_grid_cap, sg, nz);
        return true;
    case WMC_KERNEL_STREAM2:
    case WMC_KERNEL_STREAM2_SPLIT:
    case WMC_KERNEL_STREAM2_VEC:
        return launch_stream2<T>(sa, d.nk, arena, meta, st,
                                 kern == WMC_KERNEL_STREAM2_SPLIT ? split_lanes_of<T>(P, d.nk) : 0, sg, nz,
                                 (unsigned)P.tune.stream2_grid_cap);
    default: return false;
    }
}

// Node launches of the plan's general launch list on one slice group.
template <typename T>
static void general_launches(const wmc_plan_t &P, char *ws, T *arena, wmc_meta *meta, hipStream_t st,
                             const SliceGroup sg, unsigned nz, LaunchTimer *tm) {
    const NodeDesc *D = (const NodeDesc *)(ws + P.off_node);
    const GemmDesc *Gd = (const GemmDesc *)(ws + P.off_gemm);
    const int *TB = (const int *)(ws + P.off_tab);
    for (size_t k = 1; k < P.launches.size(); ++k) {
        const Launch &Ln = P.launches[k];
        Stream2Tab sa;
        StreamMfmaArgs ma;
        const int kern = solo_kernel<T>(P, k, &sa, &ma);
        const bool mat = Ln.type == LAUNCH_GEMM;
        if (!launch_node<T>(P, kern, P.nodes[(size_t)Ln.first], mat ? &P.gemms[(size_t)Ln.pad] : nullptr,
                            mat ? Gd + Ln.pad : nullptr, sa, ma, arena, meta, st, sg, nz))
            hipLaunchKernelGGL(k_nodes<T>, dim3(grid_for(Ln.work), 1, nz), dim3(WMC_BLOCK), 0, st, D + Ln.first,
                               Ln.count, (long long)Ln.work, arena, meta, sg,
                               P.tab_off[k] >= 0 ? TB + P.tab_off[k] : nullptr);
        if (tm) tm->mark();
    }
}

// Launches of the fused program on one slice group.
template <typename T>
static void fused_launches(const wmc_plan_t &P, char *ws, T *arena, wmc_meta *meta, hipStream_t st,
                           const SliceGroup sg, unsigned nz) {
    const FusedProgram &F = P.fused;
    char *img = ws + P.off_leaf;
    const NodeDesc *D = (const NodeDesc *)(img + F.o_node);
    const GemmDesc *Gd = (const GemmDesc *)(img + F.o_gemm);
    const int *TB = (const int *)(img + F.o_tab);
    for (const FusedLaunch &Ln : F.launches) {
        bool launched = false;
        if (Ln.type == FUSED_NODE || Ln.type == FUSED_GEMM) {
            Stream2Tab sa;
            StreamMfmaArgs ma;
            const NodeDesc &d = F.nodes[(size_t)Ln.node_first];
            const GemmDesc *mat = Ln.type == FUSED_GEMM ? &F.gemms[(size_t)Ln.gemm] : nullptr;
            launched = launch_node<T>(P, node_kernel<T>(P, d, mat, &sa, &ma), d, mat, mat ? Gd + Ln.gemm : nullptr, sa,
                                      ma, arena, meta, st, sg, nz);
        }
        const int *tab = Ln.tab >= 0 ? TB + Ln.tab : nullptr;
        if (!launched && !Ln.rec_count) {
            // nodes without chains: k_nodes' workgroups of 256 threads put a
            // node of 2^13 outputs on twice as many compute units
            hipLaunchKernelGGL(k_nodes<T>, dim3(grid_for(Ln.node_work), 1, nz), dim3(WMC_BLOCK), 0, st,
                               D + Ln.node_first, Ln.node_count, (long long)Ln.node_work, arena, meta, sg, tab);
        } else if (!launched) {
            FusedStepArgs a{};
            a.recs = (const ChainRec *)(img + F.o_recs) + Ln.rec_first;
            a.words = (const unsigned *)(img + F.o_words);
            a.cblocks = (unsigned)Ln.rec_count;
            a.nodes = D + Ln.node_first;
            a.nnodes = Ln.node_count;
            a.node_work = Ln.node_work;
            a.wave_node = tab;
            a.nblocks = Ln.node_count ? chain_node_blocks<WMC_CHAIN_LANE>(Ln.node_work) : 0;
            if (Ln.type == FUSED_CHAIN) launch_chain_big<T>(a, Ln.lds, arena, meta, st, sg, nz);
            else launch_fused_step<T, WMC_CHAIN_LANE>(a, Ln.lds, arena, meta, st, sg, nz);
        }
    }
}

// Launches of one slice group up to its roots' values: slices eta ... eta +
// nz - 1 side by side (grid dimension z).
template <typename T>
static void group_launches(const wmc_plan_t &P, char *ws, hipStream_t st, long long eta, unsigned nz, bool fused,
                           bool reset, LaunchTimer *tm = nullptr) {
    const FusedProgram &F = P.fused;
    wmc_meta *meta = (wmc_meta *)(ws + P.off_meta);
    char *img = ws + P.off_leaf;
    const LeafDesc *L = (const LeafDesc *)(fused ? img + F.o_leaf : img);
    const int *TB = (const int *)(fused ? img + F.o_tab : ws + P.off_tab);
    const int64_t leaf_tab = fused ? F.leaf_tab : P.leaf_tab;
    T *arena = (T *)(ws + P.off_arena);
    const SliceGroup sg{(long long)(P.arena_stride / sizeof(T)), (int)P.meta_stride, 0};
    const long long nmeta = (long long)(nz - 1) * P.meta_stride + (long long)P.T.size();
    hipLaunchKernelGGL(k_begin, dim3((unsigned)((nmeta + WMC_BLOCK - 1) / WMC_BLOCK)), dim3(WMC_BLOCK), 0, st, meta,
                       (int)nmeta, (wmc_acc *)(ws + P.off_acc), reset ? 1 : 0);
    if (tm) tm->mark();
    if (!P.leaves.empty())
        hipLaunchKernelGGL(k_leaves<T>, dim3(grid_for(P.leaf_work), 1, nz), dim3(WMC_BLOCK), 0, st, L,
                           (int)P.leaves.size(), (long long)P.leaf_work, (const double *)(ws + P.off_w), arena, meta, sg,
                           (unsigned long long)eta, leaf_tab >= 0 ? TB + leaf_tab : nullptr);
    if (tm) tm->mark();
    if (fused) fused_launches<T>(P, ws, arena, meta, st, sg, nz);
    else general_launches<T>(P, ws, arena, meta, st, sg, nz, tm);
}

// Slices [b, e) on the general launch list.
template <typename T>
static wmc_status run_slices(const wmc_plan_t &P, char *ws, hipStream_t st, long long b, long long e,
                             wmc_value *per_slice, LaunchTimer *tm, bool keep_sum) {
    wmc_acc *acc = (wmc_acc *)(ws + P.off_acc);
    // slices run in groups of up to P.group, side by side in every launch;
    // per-slice results need one slice at a time
    const long long G = per_slice ? 1 : (long long)P.group;
    for (long long eta = b; eta < e; eta += G) {
        const unsigned nz = (unsigned)std::min<long long>(G, e - eta);
        if (tm) {
            tm->k = 0;
            tm->mark();
        }
        group_launches<T>(P, ws, st, eta, nz, false, eta == b && !keep_sum, tm);
        hipLaunchKernelGGL(k_finish<T>, dim3(1), dim3(1), 0, st, (const T *)(ws + P.off_arena),
                           (long long)P.T[(size_t)P.root].off, (const wmc_meta *)(ws + P.off_meta), P.root, acc, (int)nz,
                           (long long)(P.arena_stride / sizeof(T)), (int)P.meta_stride);
        if (tm) tm->mark();
        HIP_TRY(hipGetLastError());
        if (tm) {
            HIP_TRY(hipEventSynchronize(tm->ev[tm->k - 1]));
            for (size_t q = 1; q < tm->k && (int64_t)(q - 1) < tm->cap; ++q) {
                float t = 0.f;
                HIP_TRY(hipEventElapsedTime(&t, tm->ev[q - 1], tm->ev[q]));
                tm->ms[q - 1] += t;
            }
        }
        if (per_slice) {
            wmc_acc h;
            HIP_TRY(hipMemcpyAsync(&h, acc, sizeof h, hipMemcpyDeviceToHost, st));
            HIP_TRY(hipStreamSynchronize(st));
            per_slice[eta - b] = make_value(h.last_m, h.last_e);
        }
    }
    return WMC_OK;
}

// Slices [b, e), at most P.log_slices, on the fused program, and once more on
// the launch list the groups with a slice whose chains left their range: *h is
// the sum after them.  *resident: whether the program's image is in ws.
template <typename T>
static wmc_status run_window(const wmc_plan_t &P, char *ws, hipStream_t st, long long b, long long e,
                             wmc_value *per_slice, bool keep_sum, bool *resident, wmc_acc *h) {
    const FusedProgram &F = P.fused;
    const T *arena = (const T *)(ws + P.off_arena);
    const wmc_meta *meta = (const wmc_meta *)(ws + P.off_meta);
    wmc_acc *acc = (wmc_acc *)(ws + P.off_acc);
    SliceVal *log = (SliceVal *)(ws + P.off_log);
    const long long astride = (long long)(P.arena_stride / sizeof(T)), n = e - b;
    const int mstride = (int)P.meta_stride;
    if (!*resident)
        HIP_TRY(hipMemcpyAsync(ws + P.off_leaf, F.image.data(), F.image.size(), hipMemcpyHostToDevice, st));
    *resident = true;
    for (long long eta = b; eta < e; eta += P.group) {
        const unsigned nz = (unsigned)std::min<long long>(P.group, e - eta);
        group_launches<T>(P, ws, st, eta, nz, true, eta == b && !keep_sum);
        hipLaunchKernelGGL(k_finish_fused<T>, dim3(1), dim3(nz > 1 ? WMC_BLOCK : WMC_WAVE), 0, st, arena, (long long)F.off[(size_t)P.root],
                           meta, P.root, acc, (int)nz, astride, mstride, (const int *)(ws + P.off_leaf + F.o_masks),
                           (int)F.masks.size(), log + (eta - b));
        HIP_TRY(hipGetLastError());
    }
    HIP_TRY(hipMemcpyAsync(h, acc, sizeof *h, hipMemcpyDeviceToHost, st));
    HIP_TRY(hipStreamSynchronize(st));
    if (!h->pad[0] && !per_slice) return WMC_OK;
    std::vector<SliceVal> v((size_t)n);
    HIP_TRY(hipMemcpyAsync(v.data(), log, sizeof(SliceVal) * (size_t)n, hipMemcpyDeviceToHost, st));
    HIP_TRY(hipStreamSynchronize(st));
    if (h->pad[0]) {
        long long first = n;
        HIP_TRY(hipMemcpyAsync(ws + P.off_leaf, P.desc_image.data(), P.desc_bytes, hipMemcpyHostToDevice, st));
        *resident = false;
        for (long long q = 0; q < n; q += P.group) {
            const unsigned nz = (unsigned)std::min<long long>(P.group, n - q);
            long long z = q;
            while (z < q + nz && v[(size_t)z].e != WMC_SLICE_OUT) ++z;
            if (z == q + nz) continue;
            first = std::min(first, z);
            group_launches<T>(P, ws, st, b + q, nz, false, false);
            hipLaunchKernelGGL(k_relog<T>, dim3((nz + 63) / 64), dim3(64), 0, st, arena,
                               (long long)P.T[(size_t)P.root].off, meta, P.root, (int)nz, astride, mstride, log + q);
        }
        hipLaunchKernelGGL(k_fold, dim3(1), dim3(1), 0, st, acc, log + first, (int)(n - first));
        HIP_TRY(hipGetLastError());
        HIP_TRY(hipMemcpyAsync(h, acc, sizeof *h, hipMemcpyDeviceToHost, st));
        if (per_slice)
            HIP_TRY(hipMemcpyAsync(v.data(), log, sizeof(SliceVal) * (size_t)n, hipMemcpyDeviceToHost, st));
        HIP_TRY(hipStreamSynchronize(st));
    }
    for (long long q = 0; per_slice && q < n; ++q) per_slice[q] = make_value(v[(size_t)q].m, v[(size_t)q].e);
    return WMC_OK;
}

// Slices [b, e) with the weights and the running sum *init (null: zero),
// into *h.
static wmc_status contract_range(const wmc_plan_t &P, const double *weights, char *ws, hipStream_t st, long long b,
                                 long long e, wmc_value *per_slice, const wmc_acc *init, wmc_acc *h,
                                 LaunchTimer *tm = nullptr) {
    HIP_TRY(upload_weights(P, weights, ws, st));
    if (init) HIP_TRY(hipMemcpyAsync(ws + P.off_acc, init, sizeof *init, hipMemcpyHostToDevice, st));
    if (P.fused.on && !tm) {  // a profile times the launch list it reports, node by node
        bool resident = false;
        for (long long q = b; q < e; q += P.log_slices) {
            const long long end = std::min<long long>(e, q + P.log_slices);
            const bool keep = init || q > b;
            wmc_value *out = per_slice ? per_slice + (q - b) : nullptr;
            const wmc_status s = P.precision == WMC_FP64 ? run_window<double>(P, ws, st, q, end, out, keep, &resident, h)
                                                         : run_window<float>(P, ws, st, q, end, out, keep, &resident, h);
            if (s != WMC_OK) return s;
        }
        return WMC_OK;
    }
    HIP_TRY(hipMemcpyAsync(ws + P.off_leaf, P.desc_image.data(), P.desc_bytes, hipMemcpyHostToDevice, st));
    const wmc_status s = P.precision == WMC_FP64 ? run_slices<double>(P, ws, st, b, e, per_slice, tm, init != nullptr)
                                                 : run_slices<float>(P, ws, st, b, e, per_slice, tm, init != nullptr);
    if (s != WMC_OK) return s;
    HIP_TRY(hipMemcpyAsync(h, ws + P.off_acc, sizeof *h, hipMemcpyDeviceToHost, st));
    HIP_TRY(hipStreamSynchronize(st));
    return WMC_OK;
}

extern "C" wmc_status wmc_contract_slices(const wmc_plan_t *plan, const double *weights, void *workspace,
                                          uint64_t workspace_bytes, void *stream, int64_t slice_begin,
                                          int64_t slice_end, wmc_value *out, wmc_value *per_slice) {
    if (!plan || !out) {
        wmc_set_error("wmc_contract: NULL plan or out");
        return WMC_ERR_INVALID_ARGUMENT;
    }
    const wmc_plan_t &P = *plan;
    const int64_t ns = (int64_t)1 << P.sliced.size();
    if (slice_begin < 0 || slice_end > ns || slice_begin > slice_end) {
        wmc_set_error("wmc_contract: slice range [%lld, %lld) outside [0, %lld)", (long long)slice_begin,
                      (long long)slice_end, (long long)ns);
        return WMC_ERR_INVALID_ARGUMENT;
    }
    if (weights)
        for (int64_t i = 0; i < 2 * (int64_t)P.n_user; ++i)
            if (!std::isfinite(weights[i])) {
                wmc_set_error("wmc_contract: weight %lld is not finite", (long long)i);
                return WMC_ERR_INVALID_ARGUMENT;
            }
    if (P.root < 0) {  // no variables and no clauses: the empty product
        *out = make_value(1.0, 0);
        if (per_slice)
            for (int64_t s = slice_begin; s < slice_end; ++s) per_slice[s - slice_begin] = *out;
        return WMC_OK;
    }
    if (!workspace || ((uintptr_t)workspace & 255u)) {
        wmc_set_error("wmc_contract: workspace is NULL or not 256-byte aligned");
        return WMC_ERR_INVALID_ARGUMENT;
    }
    if (workspace_bytes < P.workspace_bytes) {
        wmc_set_error("wmc_contract: workspace has %llu bytes, plan needs %llu", (unsigned long long)workspace_bytes,
                      (unsigned long long)P.workspace_bytes);
        return WMC_ERR_OUT_OF_MEMORY;
    }
    if (slice_begin == slice_end) {
        *out = make_value(0.0, 0);
        return WMC_OK;
    }
    hipStream_t st = (hipStream_t)stream;
    char *ws = (char *)workspace;
    wmc_acc h;
    const wmc_status s = contract_range(P, weights, ws, st, slice_begin, slice_end, per_slice, nullptr, &h);
    if (s != WMC_OK) return s;
    if (h.s == 0.0 && h.c == 0.0) {
        *out = make_value(0.0, 0);
    } else {
        *out = make_value(h.s + h.c, h.e);
    }
    return WMC_OK;
}

// Continue the running slice sum held in *state over the next `count`
// slices (Algorithm 3's loop over eta, split across calls).  The Neumaier
// pair and its exponent are restored into the device accumulator before the
// first slice and read back after the last, so a run split at any slice
// boundary gives the bits of one uninterrupted run.
extern "C" wmc_status wmc_contract_resume(const wmc_plan_t *plan, const double *weights, void *workspace,
                                          uint64_t workspace_bytes, void *stream, int64_t count,
                                          wmc_slice_state *state, wmc_value *out) {
    if (!plan || !state || !out) {
        wmc_set_error("wmc_contract_resume: NULL argument");
        return WMC_ERR_INVALID_ARGUMENT;
    }
    const wmc_plan_t &P = *plan;
    const int64_t ns = (int64_t)1 << P.sliced.size();
    if (state->next_slice == 0 && state->n_slices == 0) state->n_slices = ns;  // fresh state
    if (state->n_slices != ns || state->next_slice < 0 || state->next_slice > ns || count < 0 ||
        !std::isfinite(state->s) || !std::isfinite(state->c)) {
        wmc_set_error("wmc_contract_resume: state does not belong to this plan (next %lld of %lld slices, plan has %lld)",
                      (long long)state->next_slice, (long long)state->n_slices, (long long)ns);
        return WMC_ERR_INVALID_ARGUMENT;
    }
    if (weights)
        for (int64_t i = 0; i < 2 * (int64_t)P.n_user; ++i)
            if (!std::isfinite(weights[i])) {
                wmc_set_error("wmc_contract_resume: weight %lld is not finite", (long long)i);
                return WMC_ERR_INVALID_ARGUMENT;
            }
    if (!workspace || ((uintptr_t)workspace & 255u) || workspace_bytes < P.workspace_bytes) {
        wmc_set_error("wmc_contract_resume: workspace NULL, misaligned or below %llu bytes",
                      (unsigned long long)P.workspace_bytes);
        return WMC_ERR_OUT_OF_MEMORY;
    }
    const int64_t b = state->next_slice, e = std::min<int64_t>(ns, b + count);
    if (P.root >= 0 && e > b) {
        hipStream_t st = (hipStream_t)stream;
        char *ws = (char *)workspace;
        wmc_acc h;
        std::memset(&h, 0, sizeof h);
        h.s = state->s;
        h.c = state->c;
        h.e = state->e;
        const wmc_acc init = h;
        const wmc_status s = contract_range(P, weights, ws, st, b, e, nullptr, &init, &h);
        if (s != WMC_OK) return s;
        state->s = h.s;
        state->c = h.c;
        state->e = h.e;
    }
    state->next_slice = e;
    if (P.root < 0) {
        *out = make_value(1.0, 0);  // no variables and no clauses
    } else {
        *out = (state->s == 0.0 && state->c == 0.0) ? make_value(0.0, 0) : make_value(state->s + state->c, state->e);
    }
    return WMC_OK;
}

extern "C" wmc_status wmc_contract(const wmc_plan_t *plan, const double *weights, void *workspace,
                                   uint64_t workspace_bytes, void *stream, wmc_value *out) {
    if (!plan) {
        wmc_set_error("wmc_contract: NULL plan");
        return WMC_ERR_INVALID_ARGUMENT;
    }
    return wmc_contract_slices(plan, weights, workspace, workspace_bytes, stream, 0,
                               (int64_t)1 << plan->sliced.size(), out, nullptr);
}

// wmc_contract with per-launch timing: ms[k] (k < n_launches of
// wmc_plan_launches) receives the summed duration of launch k over all
// slices, measured with HIP events recorded on `stream` between launches.
extern "C" wmc_status wmc_contract_profile(const wmc_plan_t *plan, const double *weights, void *workspace,
                                           uint64_t workspace_bytes, void *stream, float *ms, int64_t cap,
                                           wmc_value *out) {
    if (!plan || !out || !ms) {
        wmc_set_error("wmc_contract_profile: NULL argument");
        return WMC_ERR_INVALID_ARGUMENT;
    }
    const wmc_plan_t &P = *plan;
    const int64_t n = (int64_t)P.launches.size() + 2;
    if (cap < n - 1) {
        wmc_set_error("wmc_contract_profile: need %lld slots", (long long)(n - 1));
        return WMC_ERR_OUT_OF_MEMORY;
    }
    if (P.root < 0 || !workspace || workspace_bytes < P.workspace_bytes)
        return wmc_contract(plan, weights, workspace, workspace_bytes, stream, out);
    hipStream_t st = (hipStream_t)stream;
    char *ws = (char *)workspace;
    LaunchTimer tm;
    tm.ms = ms;
    tm.cap = cap;
    tm.st = st;
    tm.ev.resize((size_t)n + 1);
    for (auto &e : tm.ev) HIP_TRY(hipEventCreate(&e));
    for (int64_t k = 0; k < cap; ++k) ms[k] = 0.f;
    wmc_acc h;
    const wmc_status s = contract_range(P, weights, ws, st, 0, 1ll << P.sliced.size(), nullptr, nullptr, &h, &tm);
    for (auto &e : tm.ev) (void)hipEventDestroy(e);
    if (s != WMC_OK) return s;
    *out = (h.s == 0.0 && h.c == 0.0) ? make_value(0.0, 0) : make_value(h.s + h.c, h.e);
    return WMC_OK;
}

// Kernel family of every launch wmc_contract issues for one slice, in the
// order of wmc_plan_launches (host only: the choice depends on the plan and,
// for the matrix kernel, on the current device's LDS size).
extern "C" wmc_status wmc_plan_kernels(const wmc_plan_t *plan, int32_t *kernel, int64_t cap, int64_t *n_out) {
    if (!plan) {
        wmc_set_error("wmc_plan_kernels: plan is NULL");
        return WMC_ERR_INVALID_ARGUMENT;
    }
    const wmc_plan_t &P = *plan;
    const int64_t n = (int64_t)P.launches.size() + 2;
    if (n_out) *n_out = n;
    if (!kernel) return WMC_OK;
    if (cap < n) {
        wmc_set_error("wmc_plan_kernels: need %lld slots", (long long)n);
        return WMC_ERR_OUT_OF_MEMORY;
    }
    kernel[0] = WMC_KERNEL_BEGIN;
    kernel[1] = WMC_KERNEL_LEAVES;
    Stream2Tab sa;
    StreamMfmaArgs ma;
    for (size_t k = 1; k < P.launches.size(); ++k)
        kernel[k + 1] = P.precision == WMC_FP64 ? solo_kernel<double>(P, k, &sa, &ma) : solo_kernel<float>(P, k, &sa, &ma);
    kernel[n - 1] = WMC_KERNEL_FINISH;
    return WMC_OK;
}

// Largest value a run list can deposit (every source bit set).
static unsigned long long deposit_all(const unsigned *runs, int n) {
    unsigned long long out = 0;
    for (int i = 0; i < n; ++i) out |= ((1ull << ((runs[i] >> 8) & 255u)) - 1ull) << (runs[i] >> 16);
    return out;
}

// Every index map of the kernels is a bit deposit, so the largest address a
// launch can form is the map of all ones: the OR of its table entries and
// tile bits.  Checked for every launch against the ranks of the tensors it
// reads and writes; every tensor against the arena.
template <typename T>
static bool validate_t(const wmc_plan_t &P, std::string *why) {
    char buf[160];
    auto fail = [&](size_t k, const char *what) {
        std::snprintf(buf, sizeof buf, "launch %zu: %s", k, what);
        *why = buf;
        return false;
    };
    auto rank = [&](int t) { return (int)P.T[(size_t)t].layout.size(); };
    auto fits = [](unsigned long long mx, int bits) { return bits >= 64 || (mx >> bits) == 0; };
    const uint64_t arena_elems = P.arena_bytes / (uint64_t)P.elem;
    for (size_t t = 0; t < P.T.size(); ++t)
        if (P.T[t].off < 0 || (uint64_t)P.T[t].off + (1ull << rank((int)t)) > arena_elems) {
            std::snprintf(buf, sizeof buf, "tensor %zu outside the arena", t);
            *why = buf;
            return false;
        }
    for (size_t k = 1; k < P.launches.size(); ++k) {
        const Launch &Ln = P.launches[k];
        Stream2Tab tb;
        StreamMfmaArgs ma;
        const int kern = solo_kernel<T>(P, k, &tb, &ma);
        if (kern == WMC_KERNEL_GEMM_P || kern == WMC_KERNEL_GEMM) {
            const GemmDesc &g = P.gemms[(size_t)Ln.pad];
            int top[GR_N] = {0};
            for (int q = 0; q < GR_N; ++q)
                for (int r = 0; r < g.nrun[q]; ++r) top[q] = std::max(top[q], (int)g.run[q][r][2] + (int)g.run[q][r][1]);
            const int ra = rank(g.ta), rb = rank(g.tb), rc = rank(g.tc);
            if (top[GR_MU_A] > ra - 4 - g.nk || top[GR_BETA_A] > ra - 4 - g.nk || top[GR_NU_B] > rb - g.nk ||
                top[GR_BETA_B] > rb - g.nk || top[GR_MU_C] > rc || top[GR_NU_C] > rc || top[GR_BETA_C] > rc ||
                ra != g.nk + g.nb + g.nm || rb != g.nk + g.nb + g.nn || rc != g.nb + g.nm + g.nn)
                return fail(k, "matrix node maps exceed its operands");
        } else if (kern == WMC_KERNEL_STREAM_MFMA) {
            unsigned long long c = 0, a = 0, b = 0;
            for (int q = 0; q < ma.nch; ++q)
                for (int v = 0; v < 16; ++v) {
                    c |= ma.tabc[q][v];
                    a |= ma.taba[q][v];
                    b |= ma.tabb[q][v];
                }
            for (int v = 0; v < 16; ++v) {
                a |= ma.lane_a[v] | ma.blk_a[v];
                b |= ma.lane_b[v] | ma.blk_b[v];
            }
            for (int t = 0; t < ma.nt; ++t) c |= 1ull << ma.tpos[t];
            const int nk = P.nodes[(size_t)Ln.first].nk;
            if (!fits(c, ma.rc) || ma.rc != rank(ma.tc) || !fits(a, rank(ma.ta) - nk) || !fits(b, rank(ma.tb) - nk))
                return fail(k, "matrix-core streaming tables exceed the node's tensors");
        } else if (kern == WMC_KERNEL_STREAM2 || kern == WMC_KERNEL_STREAM2_SPLIT || kern == WMC_KERNEL_STREAM2_VEC) {
            const Stream2Args &a = tb.a;
            unsigned long long c = 0, so = 0, oo = 0;
            for (int q = 0; q < tb.nch; ++q)
                for (int v = 0; v < 16; ++v) {
                    c |= tb.hr[q][v];
                    so |= tb.hs[q][v];
                    oo |= tb.ho[q][v];
                }
            for (int q = 0; q < 2; ++q)
                for (int v = 0; v < 16; ++v) {
                    c |= tb.lr[q][v];
                    so |= tb.ls[q][v];
                    oo |= tb.lo[q][v];
                }
            unsigned long long pq = 0;
            for (int t = 0; t < a.np; ++t) pq |= 1ull << a.pbit[t];
            for (int t = 0; t < a.nq; ++t) pq |= 1ull << a.qbit[t];
            c |= pq | (a.vec ? 1ull : 0ull);
            so |= deposit_all(a.srun, a.nsrun);
            oo |= deposit_all(a.orun, a.norun);
            const int nk = P.nodes[(size_t)Ln.first].nk;
            if (!fits(c, a.rc) || a.rc != rank(a.tc) || !fits(so, rank(a.ts) - nk) || !fits(oo, rank(a.to) - nk))
                return fail(k, "streaming tables exceed the node's tensors");
        } else {
            for (int32_t q = 0; q < Ln.count; ++q) {
                const NodeDesc &d = P.nodes[(size_t)(Ln.first + q)];
                if (d.rc != rank(d.tc) || !fits(deposit_all(d.ra, d.nra), rank(d.ta) - d.nk) ||
                    !fits(deposit_all(d.rb, d.nrb), rank(d.tb) - d.nk))
                    return fail(k, "node maps exceed the node's tensors");
            }
        }
    }
    return true;
}

bool wmc_validate_launches(const wmc_plan_t &P, std::string *why) {
    return (P.precision == WMC_FP64 ? validate_t<double>(P, why) : validate_t<float>(P, why)) &&
           wmc_validate_fused(P, why);
}

// ---------------------------------------------------------------------------
// Contraction without any device allocation: the workspace is a static
// device array of WMC_NOALLOC_SCRATCH_BYTES.  Host code never passes the
// array's name to a kernel or copy (on the host it is only a stand-in for
// the symbol); it passes the device address hipGetSymbolAddress returns,
// looked up once per device with that device current.  Every call on a
// device shares that device's array, so calls that overlap on one device
// race; k_begin clears the meta table and the accumulator at the start of
// every contraction, and nothing else in the workspace is read before it is
// written.
// ---------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[WMC_NOALLOC_SCRATCH_BYTES];

#define WMC_NOALLOC_MAX_DEVICES 64
static std::mutex g_scratch_mu;
static void *g_scratch_ptr[WMC_NOALLOC_MAX_DEVICES];

static wmc_status scratch_of_current_device(void **out) {
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= WMC_NOALLOC_MAX_DEVICES) {
        wmc_set_error("wmc_contract_noalloc: device %d beyond the %d supported", dev, WMC_NOALLOC_MAX_DEVICES);
        return WMC_ERR_UNSUPPORTED;
    }
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) {
            wmc_set_error("wmc_contract_noalloc: hipGetSymbolAddress(scratch) failed: %s", hipGetErrorString(e));
            return WMC_ERR_DEVICE;
        }
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return WMC_OK;
}

extern "C" wmc_status wmc_contract_noalloc(const wmc_plan_t *plan, const double *weights, void *stream,
                                           wmc_value *out) {
    if (!plan || !out) {
        wmc_set_error("wmc_contract_noalloc: NULL plan or out");
        return WMC_ERR_INVALID_ARGUMENT;
    }
    if (plan->workspace_bytes > WMC_NOALLOC_SCRATCH_BYTES) {
        wmc_set_error("wmc_contract_noalloc: plan needs a workspace of %llu bytes, the static scratch holds %llu",
                      (unsigned long long)plan->workspace_bytes, (unsigned long long)WMC_NOALLOC_SCRATCH_BYTES);
        return WMC_ERR_OUT_OF_MEMORY;
    }
    void *ws = nullptr;
    const wmc_status s = scratch_of_current_device(&ws);
    if (s != WMC_OK) return s;
    return wmc_contract(plan, weights, ws, WMC_NOALLOC_SCRATCH_BYTES, stream, out);
}
