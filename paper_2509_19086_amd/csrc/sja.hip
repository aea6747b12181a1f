// C ABI of the gap-job fit / slot-grant engine: argument validation, workspace
// bookkeeping and kernel launches.  See include/sja.h for the contract.
#include "sja_kernels.h"
#include "k_sets.h"
#include "k_pairs.h"

#include <math.h>

#include <mutex>
#include <new>
#include <vector>

using namespace sja;

// Built-in scratch for callers that cannot allocate a workspace (see
// sja_prepare_profiles_static).  Every GPU the library runs on holds its own
// copy of this array, at its own address, until the process ends.  In host
// code the name is only a handle for hipGetSymbolAddress: kernels are given
// the address that call returns, never the name.
static __device__ __align__(256) unsigned char scratch[SJA_STATIC_SCRATCH_BYTES];

namespace {

constexpr int kMaxDevices = 64;
void *g_scratch_ptr[kMaxDevices];          // device address of `scratch` on each GPU, once known
std::mutex g_scratch_mutex;

// Address of the built-in scratch on `device`, which must be the current device.
hipError_t static_scratch(int device, void **out)
{
    if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[device]) {
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        g_scratch_ptr[device] = p;
    }
    *out = g_scratch_ptr[device];
    return hipSuccess;
}

struct DeviceGuard {
    int prev = -1;
    bool switched = false;
    hipError_t err = hipSuccess;
    explicit DeviceGuard(int dev)
    {
        err = hipGetDevice(&prev);
        if (err == hipSuccess && prev != dev) {
            err = hipSetDevice(dev);
            switched = (err == hipSuccess);
        }
    }
    ~DeviceGuard()
    {
        if (switched) (void)hipSetDevice(prev);
    }
};

int fail(sja_ctx *ctx, int status, const char *what)
{
    if (ctx) snprintf(ctx->err, sizeof(ctx->err), "%s: %s", sja_status_string(status), what);
    return status;
}

int fail_hip(sja_ctx *ctx, hipError_t e, const char *what)
{
    if (ctx) snprintf(ctx->err, sizeof(ctx->err), "HIP error in %s: %s", what, hipGetErrorString(e));
    return SJA_ERR_HIP;
}

#define SJA_HIP(call, what)                                        \
    do {                                                           \
        hipError_t e__ = (call);                                   \
        if (e__ != hipSuccess) return fail_hip(ctx, e__, what);    \
    } while (0)

template <typename T>
T *ws_ptr(sja_ctx *ctx, size_t off) { return reinterpret_cast<T *>(ctx->ws + off); }

// The per-atom table of F is read while the area score or the hysteresis rule is in force
// (without either an atom's F is its own duration x peak); the per-segment area table only
// with the area score.
const long long *atom_area_of(const sja_ctx *ctx, const Layout &L)
{
    return (ctx->score_used == SJA_SCORE_AREA || ctx->hyst_used_n_caps > 0)
               ? reinterpret_cast<const long long *>(ctx->ws + L.atom_area) : nullptr;
}
const long long *pre_area_of(const sja_ctx *ctx, const Layout &L)
{
    return ctx->score_used == SJA_SCORE_AREA ? reinterpret_cast<const long long *>(ctx->ws + L.pre_area) : nullptr;
}

// Whether the keys never fall along a job's atoms: under the hysteresis rule a longer fit can end in a shorter cut if
// its minimum gain is above the distance of two capacities.
bool keys_rise(const sja_ctx *ctx)
{
    for (int i = 1; i < ctx->hyst_used_n_caps; ++i)
        if (int64_t(ctx->hyst_used_cap[i]) - ctx->hyst_used_cap[i - 1] < ctx->hyst_used_min_gain) return false;
    return true;
}

int check_params(sja_ctx *ctx, const sja_params *p, const int32_t *wait, const uint8_t *sla_class)
{
    if (!p) return fail(ctx, SJA_ERR_NULL, "params");
    if (p->policy < SJA_POLICY_EFFICIENCY || p->policy > SJA_POLICY_MIXED)
        return fail(ctx, SJA_ERR_POLICY, "unknown policy");
    if (p->wait_scale <= 0) return fail(ctx, SJA_ERR_POLICY, "wait_scale must be > 0");
    for (int i = 0; i < 3; ++i)
        if (p->sla_weight[i] < 0) return fail(ctx, SJA_ERR_POLICY, "sla_weight must be >= 0");
    if (p->max_rounds < 0) return fail(ctx, SJA_ERR_POLICY, "max_rounds must be >= 0");
    const bool needs_wait = p->policy == SJA_POLICY_FAIRNESS || p->policy == SJA_POLICY_MIXED;
    const bool needs_class = p->policy == SJA_POLICY_SLA || p->policy == SJA_POLICY_MIXED;
    if (needs_wait && !wait) return fail(ctx, SJA_ERR_NULL, "wait is required by this policy");
    if (needs_class && !sla_class) return fail(ctx, SJA_ERR_NULL, "sla_class is required by this policy");
    return SJA_OK;
}

PolicyDev to_dev(const sja_params *p)
{
    PolicyDev d;
    d.policy = p->policy;
    d.wait_scale = p->wait_scale;
    d.w0 = p->sla_weight[0];
    d.w1 = p->sla_weight[1];
    d.w2 = p->sla_weight[2];
    d.class0_override = p->class0_override;
    return d;
}

// Enqueues the pass over the cut matrix, which leaves partial bests per job tile.  The
// per-prefix keys live in the space the list building of sja_resolve uses for
// its atom keys (the two never run at the same time); `keys_ready` says that an
// earlier call with the same policy inputs left them there and nothing has
// written that space since.  The kernels do nothing for batches that another form serves, and take 3 us for every 16384
// blocks of that; fewer blocks with several tiles each made the batches that they do serve slower (8192 gaps
// of 65 capacities x 32768 jobs 528 us a select with a block to a tile, 590 with 2048 blocks and 536 with 16384; the loop
// takes registers).
int launch_matrix_pass(sja_ctx *ctx, hipStream_t st, const Layout &L, const sja_params *params, const int32_t *wait,
                       const uint8_t *sla_class, const int32_t *job_held, const uint8_t *gap_active, int unless_classes,
                       bool keys_ready)
{
    const int G = ctx->n_gaps, J = ctx->n_jobs, job_tiles = (J + kSelBlock - 1) / kSelBlock;
    const int32_t *plan = unless_classes == kNoClasses ? nullptr : ws_ptr<int32_t>(ctx, L.plan);
    unsigned long long *seg_key = ws_ptr<unsigned long long>(ctx, L.g_key_hi);
    if (job_tiles > 0 && !keys_ready) {
        const int per_wave = keys_jobs_per_wave(J, ctx->n_segments);
        const unsigned key_blocks = unsigned((J + 4 * per_wave - 1) / (4 * per_wave));
        hipLaunchKernelGGL(k_select_keys, dim3(key_blocks), dim3(256), 0, st, J, to_dev(params), ctx->seg_off, ws_ptr<int2>(ctx, L.atom_dp),
                           ws_ptr<int2>(ctx, L.atom_db), atom_area_of(ctx, L), ws_ptr<int32_t>(ctx, L.n_atoms), wait, sla_class,
                           ctx->pre_dur, ctx->pre_peak, pre_area_of(ctx, L), keys_dense(ctx->n_segments, ctx->hyst_used_n_caps > 0), per_wave, unless_classes, plan, seg_key);
        SJA_HIP(hipGetLastError(), "k_select_keys launch");
    }
    if (job_tiles > 0) {
        const int n_chunks = (G + kSelGapChunk - 1) / kSelGapChunk;
        const int tiles8 = (job_tiles + 7) / 8 * 8;
        const unsigned grid = unsigned(tiles8) * unsigned(n_chunks);
        const bool mixed = params->policy == SJA_POLICY_MIXED;
        auto kern = mixed ? k_select_pass<true> : k_select_pass<false>;
        hipLaunchKernelGGL(kern, dim3(grid), dim3(kSelBlock), 0, st, J, G, n_chunks,
                           to_dev(params), ctx->seg_off, seg_key, ctx->cut,
                           ws_ptr<int32_t>(ctx, L.gap_order), wait, sla_class, job_held, gap_active, unless_classes, plan,
                           ws_ptr<SelPartial>(ctx, L.sel_part));
        SJA_HIP(hipGetLastError(), "k_select_pass launch");
    }
    return SJA_OK;
}

// The select from the cut matrix; outputs may be user or workspace arrays.
int launch_select(sja_ctx *ctx, hipStream_t st, const sja_params *params, const int32_t *wait,
                  const uint8_t *sla_class, const int32_t *job_held, const uint8_t *gap_active,
                  int32_t *cand_job, int32_t *cand_cut, int64_t *cand_score, bool keys_ready = false)
{
    const Layout L = make_layout(ctx->n_gaps, ctx->n_jobs, ctx->n_segments);
    const int G = ctx->n_gaps, job_tiles = (ctx->n_jobs + kSelBlock - 1) / kSelBlock;
    if (G == 0) return SJA_OK;
    const int rc = launch_matrix_pass(ctx, st, L, params, wait, sla_class, job_held, gap_active, kNoClasses, keys_ready);
    if (rc != SJA_OK) return rc;
    hipLaunchKernelGGL(k_select_reduce, dim3((G + kReduceGaps - 1) / kReduceGaps), dim3(256), 0, st, G, job_tiles,
                       ws_ptr<SelPartial>(ctx, L.sel_part), cand_job, cand_cut, cand_score);
    SJA_HIP(hipGetLastError(), "k_select_reduce launch");
    return SJA_OK;
}


// One stable pass over the `width` bits of the keys at `shift` (at most 8), from buf[flip] to the other
// buffer; `launch` enqueues the scatter kernel of the kind the caller wants.
template <typename Launch>
int radix_pass(sja_ctx *ctx, hipStream_t st, const Layout &L, const int32_t *n_dev, int64_t n_host, int shift, int width,
               int &turn, bool &flip, unsigned long long *const buf[2], Launch &&launch)
{
    const int n_tiles = int((n_host + kKeyTile - 1) / kKeyTile);
    int32_t *hist = ws_ptr<int32_t>(ctx, L.g_hist);
    const unsigned long long *src = buf[flip ? 1 : 0];
    const unsigned digit_mask = (1u << width) - 1u;
    const bool few = n_tiles <= kKeyFewTiles;
    // the groups' sums of a pass and of the next one, by turns; the state of the rounds is not in use yet
    static_assert(size_t(kMaxClasses) * kListSplits * kWave * 16 >= 2 * size_t(kKeyGroupSums) * 4, "room for them");
    int32_t *sums = ws_ptr<int32_t>(ctx, L.g_state), *next_sums = sums + kKeyGroupSums;
    if (few && (turn++ & 1)) std::swap(sums, next_sums);
    hipLaunchKernelGGL(few ? k_keys_hist<true> : k_keys_hist<false>, dim3(n_tiles), dim3(kKeyThreads), 0, st, src, n_dev, shift, digit_mask,
                       hist, n_tiles, sums);
    SJA_HIP(hipGetLastError(), "k_keys_hist launch");
    if (!few)
        SJA_HIP(enqueue_scan(st, hist, (int64_t(1) << width) * n_tiles, ws_ptr<int32_t>(ctx, L.g_scan_tmp), nullptr),
                "radix scan launch");
    launch(few, dim3(n_tiles), src, buf[flip ? 0 : 1], shift, digit_mask, hist, n_tiles, sums, next_sums);
    SJA_HIP(hipGetLastError(), "k_keys_scatter launch");
    flip = !flip;
    return SJA_OK;
}

// Stable radix passes over 64-bit keys with a 32-bit payload each, lowest byte first; only the bytes named
// in byte_mask are sorted on (a byte that is the same in every key needs no pass).
int radix_sort_keys(sja_ctx *ctx, hipStream_t st, const Layout &L, const int32_t *n_dev, int64_t n_host,
                    unsigned byte_mask, int &turn, bool &flip, unsigned long long *const buf[2], uint32_t *const pay[2])
{
    for (int b = 0; b < 8 && n_host > 0; ++b) {
        if (!((byte_mask >> b) & 1u)) continue;
        const bool from = flip;
        const int rc = radix_pass(ctx, st, L, n_dev, n_host, 8 * b, 8, turn, flip, buf,
                                  [&](bool few, dim3 grid, const unsigned long long *src, unsigned long long *dst, int shift, unsigned mask,
                                      const int32_t *hist, int n_tiles, const int32_t *sums, int32_t *next_sums) {
                                      auto kern = few ? k_keys_scatter<true, true, NoRec> : k_keys_scatter<false, true, NoRec>;
                                      hipLaunchKernelGGL(kern, grid, dim3(kKeyThreads), 0, st, src, dst,
                                                         pay[from ? 1 : 0], pay[from ? 0 : 1], n_dev, shift, mask, hist, n_tiles, sums, next_sums,
                                                         static_cast<void *>(nullptr), static_cast<uint16_t *>(nullptr));
                                  });
        if (rc != SJA_OK) return rc;
    }
    return SJA_OK;
}

// The list entries by list block (they come in rank order), the last pass writes their records.
template <typename REC>
int radix_sort_entries(sja_ctx *ctx, hipStream_t st, const Layout &L, const int32_t *n_dev, int64_t n_host, int block_bits, int &turn,
                       unsigned long long *const buf[2], void *rec, uint16_t *rec_from = nullptr)
{
    bool flip = false;
    const int passes = (block_bits + 7) / 8, width = (block_bits + passes - 1) / passes;
    constexpr int first_bit = std::is_same<REC, Rec32Placed>::value ? kEntryPlacedBlockShift : kEntryBlockShift;
    for (int p = 0; p < passes; ++p) {
        const int rc = radix_pass(ctx, st, L, n_dev, n_host, first_bit + p * width, width, turn, flip, buf,
                                  [&](bool few, dim3 grid, const unsigned long long *src, unsigned long long *dst, int shift, unsigned mask,
                                      const int32_t *hist, int n_tiles, const int32_t *sums, int32_t *next_sums) {
                                      auto kern = p == passes - 1 ? (few ? k_keys_scatter<true, false, REC> : k_keys_scatter<false, false, REC>)
                                                                  : (few ? k_keys_scatter<true, false, NoRec> : k_keys_scatter<false, false, NoRec>);
                                      hipLaunchKernelGGL(kern, grid, dim3(kKeyThreads), 0, st, src, dst,
                                                         static_cast<const uint32_t *>(nullptr), static_cast<uint32_t *>(nullptr),
                                                         n_dev, shift, mask, hist, n_tiles, sums, next_sums, rec, rec_from);
                                  });
        if (rc != SJA_OK) return rc;
    }
    return SJA_OK;
}

int bits_for(int64_t n)
{
    int b = 1;
    while ((int64_t(1) << b) < n) ++b;
    return b;
}

// List-driven conflict rounds.  Returns SJA_OK with *done = true when it
// produced the grants, *done = false when the batch is outside what the lists
// serve (more than kMaxClasses capacities, or more list entries than the
// workspace holds) and the caller must take the matrix-scanning rounds; *tabled and *many_capacities say what
// it has seen of the plan by then.
int resolve_with_lists(sja_ctx *ctx, hipStream_t st, const Layout &L, const sja_params *params,
                       const int32_t *wait, const uint8_t *sla_class, int32_t *grant_job, int32_t *grant_cut,
                       int64_t *grant_score, int32_t *job_gap, int64_t cap, int32_t *rounds_and_stable, bool *done, bool *tabled, bool *many_capacities)
{
    *done = false;
    int32_t result[2] = {0, 0};
    const int G = ctx->n_gaps, J = ctx->n_jobs;
    const int sub_bound = int(fit_sub_bound(G, J));
    const int lb_bound = int(list_block_bound(G, J));
    const PolicyDev pol = to_dev(params);
    int32_t *plan = ws_ptr<int32_t>(ctx, L.plan);
    int32_t *abase = ws_ptr<int32_t>(ctx, L.g_abase);
    int32_t *tmp = ws_ptr<int32_t>(ctx, L.g_scan_tmp);
    int32_t *counters = ws_ptr<int32_t>(ctx, L.res_counters);      // [0..1] entries (64 bit), [2] atoms, [4..7] key bits
    constexpr int kCountTies = 13;
    constexpr int64_t kDigestFew = 1 << 20;         // atoms that 24 bits of their keys' digests tell apart well enough,
    constexpr int kDigestAlike = 8;                 // unless an atom shares them with so many others: a run of more than
                                                    // kTieRun would be likely, and the sort begun for nothing
    int32_t *list_off = ws_ptr<int32_t>(ctx, L.g_list_off);
    const int2 *atom_dp = ws_ptr<int2>(ctx, L.atom_dp);
    const int2 *atom_db = ws_ptr<int2>(ctx, L.atom_db);
    const int32_t *sub_begin = ws_ptr<int32_t>(ctx, L.sub_begin), *sub_end = ws_ptr<int32_t>(ctx, L.sub_end);
    int32_t *lb_begin = ws_ptr<int32_t>(ctx, L.lb_begin), *lb_end = ws_ptr<int32_t>(ctx, L.lb_end);
    int32_t *lb_off = ws_ptr<int32_t>(ctx, L.lb_off);
    const int32_t *ncap_tab = ws_ptr<int32_t>(ctx, L.ncap_tab);
    const int32_t *gap_w = ws_ptr<int32_t>(ctx, L.gap_w);
    unsigned long long *key_hi = ws_ptr<unsigned long long>(ctx, L.g_key_hi);
    unsigned long long *key_lo = ws_ptr<unsigned long long>(ctx, L.g_key_lo);
    uint32_t *perm[2] = {ws_ptr<uint32_t>(ctx, L.g_perm0), ws_ptr<uint32_t>(ctx, L.g_perm1)};
    int4 *info = ws_ptr<int4>(ctx, L.g_info);
    int32_t *chunk_at = ws_ptr<int32_t>(ctx, L.g_chunk_at);
    unsigned long long *ekey[2] = {ws_ptr<unsigned long long>(ctx, L.g_ekey0), ws_ptr<unsigned long long>(ctx, L.g_ekey1)};

    // 1. list blocks; reachable atoms per job -> compact atom ids
    int32_t *pos_block = ws_ptr<int32_t>(ctx, L.g_pos_block), *pos_tab = ws_ptr<int32_t>(ctx, L.g_pos_tab);
    const int32_t *class_begin = ws_ptr<int32_t>(ctx, L.class_begin);
    const int pos_entries = G > kEntryWinBig ? kPosTableMany : kPosTable;       // (a batch has room for as many as it has gaps, at least 4096)
    if (sub_bound <= kListBlocksOne) {
        hipLaunchKernelGGL(k_list_blocks, dim3(1 + pos_entries / 1024), dim3(1024), 0, st, lb_bound, G, pos_entries, plan, class_begin, sub_begin,
                           sub_end, gap_w, lb_begin, lb_end, pos_block, pos_tab);
    } else {
        hipLaunchKernelGGL(k_list_blocks_count, dim3((sub_bound + 1 + 255) / 256), dim3(256), 0, st, sub_bound + 1, plan, sub_begin,
                           sub_end, gap_w, lb_off);
        SJA_HIP(enqueue_scan(st, lb_off, int64_t(sub_bound) + 1, tmp, plan + kPlanListBlocks), "list block scan launch");
        const int items = sub_bound > pos_entries ? sub_bound : pos_entries;
        hipLaunchKernelGGL(k_list_blocks_write, dim3((items + 255) / 256), dim3(256), 0, st, lb_bound, G, pos_entries, plan, class_begin,
                           sub_begin, sub_end, gap_w, lb_off, lb_begin, lb_end, pos_block, pos_tab);
    }
    SJA_HIP(hipGetLastError(), "list block launch");
    hipLaunchKernelGGL(k_reach, dim3((J + 1 + 255) / 256), dim3(256), 0, st, J, plan, ncap_tab, int(ctx->reach_only), abase);
    SJA_HIP(hipGetLastError(), "k_reach launch");
    SJA_HIP(enqueue_scan(st, abase, int64_t(J) + 1, tmp, counters + 2), "atom scan launch");
    // policy keys of the atoms and the bytes in which they differ
    auto launch_keys = [&](bool first) {
        hipLaunchKernelGGL(k_atom_keys, dim3(J < 4 * 4096 ? (J + 3) / 4 : 4096), dim3(256), 0, st, J, pol, ctx->seg_off, atom_dp,
                           atom_area_of(ctx, L), abase, wait, sla_class, key_hi, key_lo, perm[0], info, ekey[0],
                           reinterpret_cast<unsigned long long *>(counters + 4), 
                           first && ctx->hyst_used_n_caps == 0 ? ekey[1] : nullptr, counters + 3);
        return hipGetLastError();
    };
    SJA_HIP(launch_keys(true), "k_atom_keys launch");
    char host_both[512] = {0};      // the plan, and the counters behind it
    const size_t apart = L.res_counters - L.plan;
    static_assert(sizeof(host_both) >= 256 + 64, "plan and counters");
    SJA_HIP(hipMemcpyAsync(host_both, plan, apart + 64, hipMemcpyDeviceToHost, st), "plan and count readback");
    SJA_HIP(hipStreamSynchronize(st), "count synchronise");
    int32_t host_plan[kPlanWords], host_counters[8];
    memcpy(host_plan, host_both, sizeof(host_plan));
    memcpy(host_counters, host_both + apart, sizeof(host_counters));
    const int64_t n_atoms = host_counters[2];
    const int n_subs = host_plan[kPlanListBlocks];          // list blocks from here on
    // runs of one capacity so short that the stepping form would begin anew every few positions
    *tabled = host_plan[kPlanTabled] != 0;
    *many_capacities = !*tabled && int64_t(host_plan[kPlanMarks]) * kShortRun > G;
    if (!host_plan[kPlanTabled] || n_subs > lb_bound || n_atoms > L.atom_cap) return SJA_OK;

    // 2. rank the atoms by policy key (descending key, ascending job id): stable passes over
    //    (inverted key, atom id) pairs; the entry buffers serve as second key buffers, they are
    //    not in use yet.  A secondary key only orders equal primary ones: the pairs are sorted by
    //    the primary key and their ties put in order; `both`: by the secondary key first
    const bool mixed = params->policy == SJA_POLICY_MIXED;
    bool flip = false;      // where the atom ids are: perm[flip]
    int turn = 0;           // of the sorts' passes
    // 24 or 32 bits, or no digest (the hysteresis rule gives many atoms of a job the same cut: long runs of equal keys, and
    // others among them).  8192 jobs of one profile, 2048 gaps: with 24 bits whatever the keys 770 us a resolve with waits
    // between 10^6 and 10^6 + 1000 and 930 under MIXED, by all bytes 600 and 620, so 530 and 525
    auto alike = [&](int found) {
        // of those looked at, every one but the first of each run was found: a share of 1 - (1 - exp(-x)) / x in runs that
        // leave x of their atoms on average
        const int shift = alike_shift(uint32_t(n_atoms));
        const double x = double(kDigestAlike) / double(1 << shift);
        return found > kDigestAlike && found > double(n_atoms >> shift) * (1.0 + expm1(-x) / x);
    };
    int digest_passes = n_atoms <= kDigestFew && !alike(host_counters[3] & 0xffff) ? 3 : 4;
    unsigned long long bits_hi = 0, bits_lo = 0;
    memcpy(&bits_hi, host_counters + 4, 8);
    memcpy(&bits_lo, host_counters + 6, 8);
    auto bytes_of = [](unsigned long long v) {
        unsigned m = 0;
        for (int b = 0; b < 8; ++b) if ((v >> (8 * b)) & 0xffull) m |= 1u << b;
        return m;
    };
    if (ctx->hyst_used_n_caps > 0 || (digest_passes == 4 && alike(host_counters[3] >> 16)) ||
        __builtin_popcount(bytes_of(bits_hi)) <= digest_passes)
        digest_passes = 0;
    auto rank_atoms = [&](bool both) -> int {
        const dim3 grid(unsigned((n_atoms + 255) / 256)), block(256);
        flip = false;
        if (n_atoms <= kKeyTile) {
            hipLaunchKernelGGL(k_sort_one, dim3(1), dim3(kSortOneThreads), 0, st, int(n_atoms), key_lo, mixed ? bytes_of(bits_lo) : 0u,
                               key_hi, bytes_of(bits_hi), perm[0]);
            SJA_HIP(hipGetLastError(), "k_sort_one launch");
            return SJA_OK;
        }
        // by the leading bits only, the rest where those are equal, if that takes fewer passes: three in place of six at
        // 2048 gaps x 8192 jobs (tick 1175 -> 1134 us), in place of eight under MIXED (three ticks 4655 -> 4245)
        const int passes = digest_passes;
        if (!both && passes) {
            for (int p = 0; p < passes; ++p) {
                const int rc = radix_pass(ctx, st, L, counters + 2, n_atoms, 64 - 8 * (passes - p), 8, turn, flip, ekey,
                                          [&](bool few, dim3 tiles, const unsigned long long *src, unsigned long long *dst, int shift, unsigned mask,
                                              const int32_t *hist, int n_tiles, const int32_t *sums, int32_t *next_sums) {
                                              hipLaunchKernelGGL((few ? k_keys_scatter<true, false, NoRec> : k_keys_scatter<false, false, NoRec>), tiles,
                                                                 dim3(kKeyThreads), 0, st, src, dst, static_cast<const uint32_t *>(nullptr),
                                                                 static_cast<uint32_t *>(nullptr), counters + 2, shift, mask, hist, n_tiles, sums, next_sums,
                                                                 static_cast<void *>(nullptr), static_cast<uint16_t *>(nullptr));
                                          });
                if (rc != SJA_OK) return rc;
            }
            hipLaunchKernelGGL(mixed ? k_fix_runs<true> : k_fix_runs<false>, grid, block, 0, st, counters + 2, ekey[flip ? 1 : 0], 64 - 8 * passes,
                               key_hi, key_lo, perm[flip ? 1 : 0], counters + kCountTies);
            SJA_HIP(hipGetLastError(), "k_fix_runs launch");
            return SJA_OK;
        }
        if (!both) {
            unsigned long long *kb[2] = {key_hi, ekey[0]};
            const int rc = radix_sort_keys(ctx, st, L, counters + 2, n_atoms, bytes_of(bits_hi), turn, flip, kb, perm);
            if (rc != SJA_OK || !mixed) return rc;
            hipLaunchKernelGGL(k_fix_ties, grid, block, 0, st, counters + 2, kb[flip ? 1 : 0], key_lo, perm[flip ? 1 : 0],
                               counters + kCountTies);
            SJA_HIP(hipGetLastError(), "k_fix_ties launch");
            return SJA_OK;
        }
        unsigned long long *kb[2] = {key_lo, ekey[0]};
        const int rc = radix_sort_keys(ctx, st, L, counters + 2, n_atoms, bytes_of(bits_lo), turn, flip, kb, perm);
        if (rc != SJA_OK) return rc;
        // the primary keys in the order reached so far
        unsigned long long *kh[2] = {ekey[1], ekey[0]};
        if (flip) { kh[0] = ekey[0]; kh[1] = ekey[1]; }      // buffer index must follow the id buffers
        hipLaunchKernelGGL(k_gather_keys, grid, block, 0, st, counters + 2, key_hi, perm[flip ? 1 : 0], kh[flip ? 1 : 0]);
        SJA_HIP(hipGetLastError(), "k_gather_keys launch");
        return radix_sort_keys(ctx, st, L, counters + 2, n_atoms, bytes_of(bits_hi), turn, flip, kh, perm);
    };

    // 3. list entries in rank order: counted, then written, then sorted by list block
    constexpr int waves_per_block = kEntryThreads / kWave;
    static_assert(SJA_MAX_GAPS / 64 + kMaxClasses + kMaxClasses * kListSplits <= kEntryMostBlocks, "a count per list block fits LDS");
    // (sub-blocks are shorter than 64 positions only in batches of fewer than 2048 such chunks)
    // windows in LDS: a block with 32768 of them has a compute unit to itself, and so has one with many list blocks
    const bool in_lds = n_subs <= kEntryBlocks && G <= kEntryWinBig, small = in_lds && G <= kEntryWinSmall;
    const int most = small ? kEntryGrid : kEntryGrid / 2;
    // 64 atoms a chunk; fewer where few atoms have many entries each, so that every wave has a chunk (131072 gaps x
    // 1024 jobs: 274 -> 114 us)
    int per_chunk = kWave;
    auto chunks_of = [&](int per) { return (n_atoms + per - 1) / per; };
    while (!in_lds && per_chunk > kEntryLeastAtoms && chunks_of(per_chunk / 2) <= int64_t(most) * waves_per_block &&
           chunks_of(per_chunk / 2) <= L.atom_cap / kWave)
        per_chunk /= 2;
    const int64_t n_chunks = chunks_of(per_chunk), want = (n_chunks + waves_per_block - 1) / waves_per_block;
    const unsigned entry_grid = unsigned(want < most ? want : most);
    auto launch_entries = [&](auto emit, int placed) {
        auto kern = small ? k_list_entries<decltype(emit)::value, kEntryWinSmall>
                          : in_lds ? k_list_entries<decltype(emit)::value, kEntryWinBig> : k_list_entries<decltype(emit)::value, 0>;
        hipLaunchKernelGGL(kern, dim3(entry_grid), dim3(kEntryThreads), 0, st, int(n_atoms), per_chunk, n_subs, G, pos_entries,
                           plan, class_begin, lb_begin, pos_block, pos_tab, gap_w, ws_ptr<int32_t>(ctx, L.gap_c), perm[flip ? 1 : 0], info, chunk_at,
                           list_off, reinterpret_cast<unsigned long long *>(counters), ekey[0], placed);
        return hipGetLastError();
    };
    long long n_entries = 0;
    for (bool both = false;;) {
        if (n_atoms > 0) {
            const int rc = rank_atoms(both);
            if (rc != SJA_OK) return rc;
            SJA_HIP(launch_entries(std::false_type{}, 0), "k_list_entries launch");
            SJA_HIP(enqueue_scan(st, chunk_at, n_chunks, tmp, nullptr), "entry scan launch");
        }
        int32_t h[kCountTies + 1] = {0};
        SJA_HIP(hipMemcpyAsync(h, counters, sizeof(h), hipMemcpyDeviceToHost, st), "entry count readback");
        SJA_HIP(hipStreamSynchronize(st), "entry count synchronise");
        memcpy(&n_entries, h, sizeof(n_entries));
        if (!h[kCountTies]) break;
        // a long run out of order: once more, by all of the primary key if that was not done and the run lacks it, else by both
        both = !digest_passes || !(h[kCountTies] & kRunsByKey);
        digest_passes = 0;
        hipLaunchKernelGGL(k_fill_i32, dim3(1), dim3(256), 0, st, counters, int64_t(2), 0);
        hipLaunchKernelGGL(k_fill_i32, dim3(1), dim3(256), 0, st, counters + kCountTies, int64_t(1), 0);
        hipLaunchKernelGGL(k_fill_i32, dim3((lb_bound + 2 + 255) / 256), dim3(256), 0, st, list_off, int64_t(lb_bound + 2), 0);
        SJA_HIP(launch_keys(false), "k_atom_keys launch");
    }
    if (n_entries > L.entry_cap || n_entries >= (1ll << 31)) return SJA_OK;
    SJA_HIP(enqueue_scan(st, list_off, int64_t(lb_bound) + 2, tmp, nullptr), "list offset scan launch");
    const int held_words = held_bitmap_words(J);
    const bool use_held = held_words <= kHeldMaxWords;
    const bool wide_records = int64_t(J) > (int64_t(1) << kRec32JobBits);
    // the block that runs rounds by itself: it needs the held bitmap, a thread per list block, and keys
    // that never fall along a job's atoms (a minimum gain above the distance of two capacities of the
    // hysteresis set can let a longer fit end in a shorter cut); and more than a few rounds to go, which cost no
    // more launched than the block needs to start and report (20 us of a Medium batch, 200 at 630 list blocks)
    const bool solo_fits = use_held && !wide_records && keys_rise(ctx) && n_subs <= kSoloMaxBlocks;
    const bool long_lists = n_entries >= int64_t(kFirstLong) * n_subs;
    const int solo_few = kSoloFewRounds + n_subs / kSoloBlocksPerRound;
    const int solo_first = n_subs <= kSoloFewBlocks ? kSoloFirstFew : kSoloFirstMany;
    const bool solo = solo_fits && cap >= solo_first + solo_few;
    const int solo_waves = (n_subs + kWave - 1) / kWave > kSoloMinWaves ? (n_subs + kWave - 1) / kWave : kSoloMinWaves;
    // and the calm rounds after it, in batches: with a place per record (Medium tick 1775 -> 1290 us)
    const int64_t list_room = L.entry_cap * 8 / (int64_t(n_subs > 0 ? n_subs : 1) * kSetsPieces * 6);
    const int list_jobs = int(list_room < kSetsListed ? list_room / 2 * 2 : kSetsListed);
    const bool sets = solo && n_subs <= kSetsMaxBlocks && J <= kPlacedJobs && (n_subs <= kSetsOneBlocks || list_jobs >= kSetsLeastListed);
    // (records of four bytes leave half of their space to the places; entry_cap is at least 192)
    void *rec = ws_ptr<void>(ctx, L.g_rec);
    uint16_t *rec_from = ws_ptr<uint16_t>(ctx, L.g_rec + align_up(size_t(L.entry_cap) * sizeof(Rec32)));
    if (n_entries > 0) {
        SJA_HIP(launch_entries(std::true_type{}, sets), "k_list_entries launch");
        const int block_bits = bits_for(n_subs > 1 ? n_subs : 2);
        const int rc = wide_records ? radix_sort_entries<Rec64>(ctx, st, L, counters, n_entries, block_bits, turn, ekey, rec)
                       : sets       ? radix_sort_entries<Rec32Placed>(ctx, st, L, counters, n_entries, block_bits, turn, ekey, rec, rec_from)
                                    : radix_sort_entries<Rec32>(ctx, st, L, counters, n_entries, block_bits, turn, ekey, rec);
        if (rc != SJA_OK) return rc;
    }

    // 4. rounds
    int32_t *cnt_lost = ws_ptr<int32_t>(ctx, L.g_cnt_lost), *cnt_cand = ws_ptr<int32_t>(ctx, L.g_cnt_cand);
    const int32_t *gap_order = ws_ptr<int32_t>(ctx, L.gap_order);
    unsigned long long *claim = ws_ptr<unsigned long long>(ctx, L.res_claim);
    int4 *state = ws_ptr<int4>(ctx, L.g_state);
    const int round_grid = (n_subs + kRoundBlock / kWave - 1) / (kRoundBlock / kWave);

    // one launch per round, in batches between looks at the flags
    // the first kHeldRounds rounds keep the held jobs as a bitmap too (two alternating copies), if it fits LDS
    uint32_t *held = ws_ptr<uint32_t>(ctx, L.g_held);
    const bool wide = !wide_records && n_subs <= kWideBlocks;
    auto launch_round = [&](int64_t k, int propose) {
        const bool with_bitmap = use_held && (solo || k <= kHeldRounds);
        if (k == 1 && long_lists && propose) {
            auto first = [&](auto kern, auto *records) {        // (round 1 marks the bitmap that round 2 reads)
                hipLaunchKernelGGL(kern, dim3(n_subs), dim3(kFirstThreads), 0, st, state, list_off, records, claim,
                                   with_bitmap ? held : static_cast<uint32_t *>(nullptr), lb_begin, lb_end, gap_order, cnt_cand);
            };
            if (wide_records)
                first(k_grant_first<Rec64>, static_cast<const Rec64 *>(rec));
            else
                first(k_grant_first<Rec32>, static_cast<const Rec32 *>(rec));
            return hipGetLastError();
        }
        if (wide && k <= kWideRounds && with_bitmap && propose) {
            const bool few = n_subs > kWideManyBlocks;
            hipLaunchKernelGGL(few ? k_grant_wide<kWideFewWaves> : k_grant_wide<kWideWaves>, dim3(n_subs),
                               dim3((few ? kWideFewWaves : kWideWaves) * kWave), 0, st, state, list_off, static_cast<const Rec32 *>(rec), claim,
                               int(k), held_words, held, lb_begin, lb_end, gap_order, cnt_lost, cnt_cand,
                               solo ? counters + 14 : static_cast<int32_t *>(nullptr));
            return hipGetLastError();
        }
        auto go = [&](auto kern, auto *records) {
            hipLaunchKernelGGL(kern, dim3(round_grid), dim3(kRoundBlock), 0, st, state, list_off, records, claim, int(k), propose, n_subs,
                               with_bitmap ? held_words : 0, with_bitmap ? held : static_cast<uint32_t *>(nullptr), lb_begin,
                               lb_end, gap_order, cnt_lost, cnt_cand, solo ? counters + 14 : static_cast<int32_t *>(nullptr));
        };
        if (wide_records)
            go(with_bitmap ? k_grant_round<true, Rec64> : k_grant_round<false, Rec64>, static_cast<const Rec64 *>(rec));
        else
            go(with_bitmap ? k_grant_round<true, Rec32> : k_grant_round<false, Rec32>, static_cast<const Rec32 *>(rec));
        return hipGetLastError();
    };
    std::vector<int32_t> h_told;
    int64_t launched = 0;        // kernels 1..launched have been enqueued
    int64_t next_check = 1;      // first round whose end is not yet decided
    int64_t open_left = cap;     // rounds that can still follow, as far as is known
    bool finished = false, sets_built = false;
    const bool few_blocks = n_subs <= kSetsOneBlocks;
    const int calm_shift = few_blocks ? kSoloCalmShiftFew : kSoloCalmShift, calm_pieces = few_blocks ? kSoloCalmPiecesFew : kSoloCalmPieces;
    const int64_t calm_rounds = int64_t(1) << calm_shift;
    int64_t calm_wait = calm_rounds;
    constexpr int64_t kLaunchedRounds = 64;
    int64_t batch = solo ? solo_first : kLaunchedRounds;   // rounds enqueued between looks at the flags; grows, a finished batch costs little
    const int64_t most_rounds = solo ? 256 : 1024;  // (a look at whether the block can go on costs three or four rounds)
    while (!finished) {
        const bool take_over = solo && cap - launched - batch >= solo_few;
        if (!take_over && batch < kLaunchedRounds) batch = kLaunchedRounds;
        const int64_t rounds = batch < open_left ? batch : open_left;
        const int64_t upto = (launched + rounds < cap) ? launched + rounds : cap;
        if (batch < most_rounds) batch = batch ? 2 * batch : solo_first;
        for (int64_t k = launched + 1; k <= upto; ++k) SJA_HIP(launch_round(k, 1), "k_grant_round launch");
        if (take_over) {
            int32_t h_out[4] = {0, 0, 0, 0};
            auto look = [&]() -> int {
                SJA_HIP(hipMemcpyAsync(h_out, counters + 8, sizeof(h_out), hipMemcpyDeviceToHost, st), "rounds readback");
                SJA_HIP(hipStreamSynchronize(st), "round synchronise");
                return SJA_OK;
            };
            auto solo_kern = n_subs <= kSoloSmallBlocks ? k_grant_solo<true> : k_grant_solo<false>;
            hipLaunchKernelGGL(solo_kern, dim3(1), dim3(solo_waves * kWave), 0, st, state, list_off, static_cast<const Rec32 *>(rec),
                               claim, int(upto), int(next_check), int(cap), n_subs, held_words, held, cnt_lost, cnt_cand,
                               sets && upto + calm_wait < INT32_MAX ? int(upto + calm_wait) : INT32_MAX, calm_shift, calm_pieces, counters + 14, counters + 8);
            SJA_HIP(hipGetLastError(), "k_grant_solo launch");
            SetsArgs args{};
            args.state = state;
            args.list_off = list_off;
            args.rec = static_cast<const Rec32 *>(rec);
            args.rec_from = rec_from;
            args.claim = claim;
            args.held = held;
            args.plan = plan;
            args.class_begin = class_begin;
            args.gap_cls = ws_ptr<int32_t>(ctx, L.gap_cls);
            args.lb_begin = lb_begin;
            args.lb_end = lb_end;
            args.gap_order = gap_order;
            args.place_of = pos_tab;           // the lists are built: the tables of positions are done with
            args.by_class = ws_ptr<int2>(ctx, L.gap_tile_key);
            // (the states' space behind those of the list blocks that there are)
            args.block = reinterpret_cast<SetsBlock *>(state + size_t(n_subs) * kWave);
            args.low = reinterpret_cast<int32_t *>(args.block + n_subs);
            args.classes = args.low + kMaxClasses;
            // (the records are sorted: the buffers of the entries are free)
            args.list_jobs = list_jobs;
            args.list = reinterpret_cast<uint32_t *>(ekey[0]);
            args.list_from = reinterpret_cast<uint16_t *>(args.list + size_t(n_subs) * kSetsPieces * list_jobs);
            static_assert((kListSplits * kMaxClasses + kMaxClasses - kSetsMaxBlocks) * kWave * sizeof(int4) >
                          size_t(kSetsMaxBlocks) * sizeof(SetsBlock) + (3 * kMaxClasses + 2) * 4, "room for them");
            args.out = counters + 8;
            args.cap = int(cap);
            args.n_gaps = G;
            args.n_lb = n_subs;
            args.held_words = held_words;
            args.build = !sets_built;
            // one launch that returns at once if the block has not left the rounds calm: 5 us, a look 20
            const bool sets_follow = sets && few_blocks;
            if (sets_follow) {
                hipLaunchKernelGGL(k_sets_one, dim3(1), dim3(kSetsThreads), 0, st, args);
                SJA_HIP(hipGetLastError(), "k_sets_one launch");
            }
            int rc = look();
            if (rc != SJA_OK) return rc;
            if (!sets_follow && h_out[kSoloDone] == kSoloCalm) {
                const dim3 blocks((n_subs + kSetsFormThreads / kWave - 1) / (kSetsFormThreads / kWave)), threads(kSetsFormThreads);
                hipLaunchKernelGGL(k_sets_open, blocks, threads, 0, st, args);
                hipLaunchKernelGGL(k_sets_begin, dim3(1), dim3(kSetsThreads), 0, st, args);
                // (a launch too many does nothing and takes 3 us)
                for (int pairs = 4; rc == SJA_OK; pairs = pairs < 32 ? 2 * pairs : 32) {
                    for (int k = 0; k < pairs; ++k) {
                        hipLaunchKernelGGL(k_sets_form, blocks, threads, 0, st, args);
                        hipLaunchKernelGGL(k_sets_play, dim3(1), dim3(kSetsThreads), 0, st, args);
                    }
                    SJA_HIP(hipGetLastError(), "k_sets_play launch");
                    rc = look();
                    if (h_out[kSoloDone] != kSetsRunning) break;
                }
                if (rc == SJA_OK && h_out[kSoloDone] == kSetsLeft) {
                    hipLaunchKernelGGL(k_sets_hand_back, blocks, threads, 0, st, args);
                    SJA_HIP(hipGetLastError(), "k_sets_hand_back launch");
                }
                if (rc != SJA_OK) return rc;
            }
            launched = h_out[kSoloRounds];
            if (h_out[kSoloDone] == kSetsLeft) {        // on with k_grant_solo, the longer the shorter it was calm
                sets_built = true;
                batch = 0;
                calm_wait = launched - upto < 4 * calm_wait ? 2 * calm_wait : calm_rounds;
            }
            next_check = h_out[kSoloDone] == kSoloPutOff ? launched : launched + 1;
            if (h_out[kSoloDone] == kSoloEnded) {
                result[0] = h_out[kSoloRounds];
                result[1] = h_out[kSoloStable];
                finished = true;
            }
            continue;
        }
        if (upto == cap) SJA_HIP(launch_round(cap + 1, 0), "k_grant_round launch");
        launched = upto;
        const int64_t known = (upto == cap) ? cap + 1 : upto;        // kernels that have run
        // what the host looks at lies side by side (the entries' buffer is free), a copy of its own took 10 us each
        const int64_t since = next_check, told = known + 1 - since;
        int32_t *told_at = reinterpret_cast<int32_t *>(ekey[0]);
        hipLaunchKernelGGL(k_count_open, dim3(1), dim3(1024), 0, st, lb_bound, plan, state, cnt_lost + since, cnt_cand + since, int(told), told_at);
        SJA_HIP(hipGetLastError(), "k_count_open launch");
        h_told.resize(size_t(1 + 2 * told));
        SJA_HIP(hipMemcpyAsync(h_told.data(), told_at, h_told.size() * 4, hipMemcpyDeviceToHost, st), "round counters");
        SJA_HIP(hipStreamSynchronize(st), "round synchronise");
        const int32_t *h_lost = h_told.data() + 1, *h_cand = h_lost + told;
        // every further round grants at least one open position: no point in enqueueing more than that
        open_left = int64_t(h_told[0]) + 1;
        for (int64_t r = since; r <= upto; ++r) {
            if (h_cand[r - since] == 0) { result[0] = int32_t(r); result[1] = 1; finished = true; break; }
            if (r + 1 > known) { next_check = r; break; }              // losers of r not counted yet
            if (h_lost[r - since] == 0) { result[0] = int32_t(r); result[1] = 1; finished = true; break; }
            if (r == cap) { result[0] = int32_t(cap); result[1] = 0; finished = true; break; }
            next_check = r + 1;
        }
    }
    hipLaunchKernelGGL(k_grant_finish, dim3(unsigned((int64_t(n_subs) * kWave + 255) / 256)), dim3(256), 0, st, lb_bound, pol,
                       plan, state, lb_begin, gap_w, ws_ptr<int32_t>(ctx, L.gap_c), ctx->seg_off, ws_ptr<int32_t>(ctx, L.n_atoms),
                       atom_dp, atom_db, atom_area_of(ctx, L), wait, sla_class, grant_job, grant_cut, grant_score, job_gap, result[0],
                       result[1], rounds_and_stable);
    SJA_HIP(hipGetLastError(), "k_grant_finish launch");
    *done = true;
    return SJA_OK;
}

// Gap ordering, capacity classes and chunk / sub-block plan of a batch of gaps.
int enqueue_gap_plan(sja_ctx *ctx, hipStream_t st, const Layout &L, int32_t n_gaps, const int32_t *W, const int32_t *C)
{
    const int J = ctx->n_jobs;
    const int gc = fit_chunk_len(n_gaps, J);
    const int chunk_bound = int(fit_chunk_bound(n_gaps, J));
    const int sb = fit_sub_len(n_gaps, J);
    const int sub_bound = int(fit_sub_bound(n_gaps, J));
    const dim3 per_gap((n_gaps + 255) / 256), b256(256);
    int32_t *rank = ws_ptr<int32_t>(ctx, L.gap_rank);
    int32_t *gw = ws_ptr<int32_t>(ctx, L.gap_w), *gcap = ws_ptr<int32_t>(ctx, L.gap_c);
    int32_t *plan = ws_ptr<int32_t>(ctx, L.plan);
    const int gap_tiles = (n_gaps + kGapTile - 1) / kGapTile;
    unsigned long long *tile_key = ws_ptr<unsigned long long>(ctx, L.gap_tile_key);
    int32_t *tile_idx = ws_ptr<int32_t>(ctx, L.gap_tile_idx);
    hipLaunchKernelGGL(k_gap_tile_sort, dim3(gap_tiles), dim3(kGapSortThreads), 0, st, n_gaps, W, C, tile_key, tile_idx,
                       plan, ws_ptr<int32_t>(ctx, L.class_dmax));
    SJA_HIP(hipGetLastError(), "k_gap_tile_sort launch");
    hipLaunchKernelGGL(k_gap_rank, dim3(gap_tiles * (kGapTile / kGapRankBlock)), dim3(kGapRankBlock * kGapRankGroups), 0, st, n_gaps, J,
                       gap_tiles, tile_key, tile_idx, W, C, rank, ws_ptr<int32_t>(ctx, L.gap_order), gw, gcap,
                       ws_ptr<int64_t>(ctx, L.gap_row));
    SJA_HIP(hipGetLastError(), "k_gap_rank launch");
    if (J > 0) {
        int32_t *marks = ws_ptr<int32_t>(ctx, L.class_marks);
        hipLaunchKernelGGL(k_gap_marks, per_gap, b256, 0, st, n_gaps, gcap, plan, marks);
        SJA_HIP(hipGetLastError(), "k_gap_marks launch");
        const int plan_blocks = (n_gaps + 255) / 256 < 64 ? (n_gaps + 255) / 256 : 64;
        hipLaunchKernelGGL(k_gap_plan, dim3(plan_blocks), b256, 0, st, n_gaps, gc, sb, chunk_bound, sub_bound, gcap, marks,
                           plan, ws_ptr<int32_t>(ctx, L.class_begin), ws_ptr<int32_t>(ctx, L.class_chunk0),
                           ws_ptr<int32_t>(ctx, L.class_sub0), ws_ptr<int32_t>(ctx, L.chunk_begin),
                           ws_ptr<int32_t>(ctx, L.chunk_end), ws_ptr<int32_t>(ctx, L.chunk_class),
                           ws_ptr<int32_t>(ctx, L.chunk_sub), ws_ptr<int32_t>(ctx, L.sub_begin),
                           ws_ptr<int32_t>(ctx, L.sub_end), ws_ptr<int32_t>(ctx, L.gap_cls),
                           ws_ptr<int32_t>(ctx, L.gap_run_end));
        SJA_HIP(hipGetLastError(), "k_gap_plan launch");
    }
    return SJA_OK;
}

// The start tables: what the stepping kernels still need.
int enqueue_starts(sja_ctx *ctx, hipStream_t st, const Layout &L)
{
    const int J = ctx->n_jobs;
    if (J == 0) return SJA_OK;
    hipLaunchKernelGGL(k_fit_starts, dim3((starts_tiles(J) + 7) / 8 * 8), dim3(256), 0, st, J, ws_ptr<int32_t>(ctx, L.plan),
                       ws_ptr<int32_t>(ctx, L.class_begin), ws_ptr<int32_t>(ctx, L.chunk_begin), ws_ptr<int32_t>(ctx, L.chunk_class),
                       ws_ptr<int32_t>(ctx, L.gap_w), ws_ptr<int32_t>(ctx, L.gap_c), ctx->seg_off, ws_ptr<int2>(ctx, L.atom_dp),
                       ws_ptr<int32_t>(ctx, L.n_atoms), ws_ptr<int32_t>(ctx, L.start_tab), ws_ptr<int32_t>(ctx, L.ncap_tab));
    SJA_HIP(hipGetLastError(), "k_fit_starts launch");
    ctx->reach_only = false;
    return SJA_OK;
}

// A batch served pair by pair.  The gaps' lists take the space of the list entries.
int pair_list_most(int64_t G, int64_t J) { return int(G < J ? G : J); }

// Pairs, and gaps x segments, from which on the atoms are found job by job: a launch more, and shorter searches, which pays the
// more the longer the profiles are.  A fit -> select and the resolve behind it, searched and so, us, means over batches of
// 2^19 to 2^19.5 pairs: 22 segments a job 28.4 / 31.1 and 112 / 114, 50 29.4 / 30.9 and 218 / 219, 120 34.2 / 32.1 and
// 140 / 138; of 2^20 to 2^21 pairs 22 segments 39.2 / 37.1 and 205 / 202, 120 51.2 / 39.1 and 203 / 189; of 2^18 pairs
// 50 23.7 / 28.3 and 79 / 84, 300 27.2 / 30.1 and 75 / 78.
constexpr int64_t kPairAtomsLeast = int64_t(1) << 19, kPairAtomsSegments = int64_t(1) << 25;

bool pairs_batch(const sja_ctx *ctx, const Layout &L, int64_t G, int64_t J)
{
    return ctx->resolve_mode == SJA_RESOLVE_LISTS && J > 0 && G <= kPairsGaps && J <= kPairsJobs && G * J <= kPairsMost &&
           pair_list_words(int(G), pair_list_most(G, J)) * 8 <= L.lb_begin - L.g_ekey0;
}

PairGaps pair_gaps(sja_ctx *ctx, const Layout &L)
{
    return {ws_ptr<int32_t>(ctx, L.gap_w), ws_ptr<int32_t>(ctx, L.gap_c), ws_ptr<int32_t>(ctx, L.gap_order)};
}

// The plan that a small batch went without.
int plan_pairs(sja_ctx *ctx, hipStream_t st, const Layout &L)
{
    int32_t *W = ws_ptr<int32_t>(ctx, L.res_cand_job), *C = ws_ptr<int32_t>(ctx, L.res_cand_cut);
    const size_t bytes = size_t(ctx->n_gaps) * 4;
    SJA_HIP(hipMemcpyAsync(W, ws_ptr<int32_t>(ctx, L.gap_w), bytes, hipMemcpyDeviceToDevice, st), "gap copy");
    SJA_HIP(hipMemcpyAsync(C, ws_ptr<int32_t>(ctx, L.gap_c), bytes, hipMemcpyDeviceToDevice, st), "gap copy");
    int rc = enqueue_gap_plan(ctx, st, L, ctx->n_gaps, W, C);
    if (rc == SJA_OK) rc = enqueue_starts(ctx, st, L);
    if (rc == SJA_OK) ctx->pairs = false;
    return rc;
}

// The atoms of every pair job by job, behind the gaps' lists, where there are enough pairs to pay for the launch and room
// for them; else null: each pair is searched where it is needed.
uint16_t *pair_atoms(sja_ctx *ctx, hipStream_t st, const Layout &L, int32_t n_gaps, const int32_t *W, const int32_t *C)
{
    const int J = ctx->n_jobs;
    const size_t at = align_up(L.g_ekey0 + pair_list_words(n_gaps, pair_list_most(n_gaps, J)) * 8);
    if (int64_t(n_gaps) * J < kPairAtomsLeast || int64_t(n_gaps) * ctx->n_segments < kPairAtomsSegments || at + size_t(n_gaps) * J * 2 > L.lb_begin) return nullptr;
    uint16_t *atoms = ws_ptr<uint16_t>(ctx, at);
    hipLaunchKernelGGL(k_pair_atoms, dim3((J + kAtomsJobs - 1) / kAtomsJobs, (n_gaps + kAtomsGaps - 1) / kAtomsGaps), dim3(kAtomsThreads), 0, st, n_gaps, J,
                       W, C, ctx->seg_off, ws_ptr<int2>(ctx, L.atom_dp), ws_ptr<int32_t>(ctx, L.n_atoms), atoms);
    return atoms;
}

int pair_threads(int J) { return J <= kWave ? kWave : J <= 4 * 256 ? 256 : kPairsMostThreads; }

int resolve_pairs(sja_ctx *ctx, hipStream_t st, const Layout &L, const sja_params *params, const int32_t *wait, const uint8_t *sla_class,
                  int32_t *grant_job, int32_t *grant_cut, int64_t *grant_score, int32_t *job_gap, int cap, int32_t *rounds_and_stable)
{
    const int G = ctx->n_gaps, J = ctx->n_jobs, most = pair_list_most(G, J);
    const PolicyDev pol = to_dev(params);
    const long long *area = atom_area_of(ctx, L);
    const int32_t *gap_w = ws_ptr<int32_t>(ctx, L.gap_w), *gap_c = ws_ptr<int32_t>(ctx, L.gap_c), *n_atoms = ws_ptr<int32_t>(ctx, L.n_atoms);
    const int2 *atom_dp = ws_ptr<int2>(ctx, L.atom_dp), *atom_db = ws_ptr<int2>(ctx, L.atom_db);
    int32_t *len = ws_ptr<int32_t>(ctx, L.gap_rank);
    unsigned long long *list = ws_ptr<unsigned long long>(ctx, L.g_ekey0);
    PairReplies from{};
    if (ctx->fitted) {
        from.cut = ctx->cut;
        from.pre_dur = ctx->pre_dur;
        from.pre_peak = ctx->pre_peak;
        from.pre_area = pre_area_of(ctx, L);
    } else {
        from.atoms = pair_atoms(ctx, st, L, G, gap_w, gap_c);
        SJA_HIP(hipGetLastError(), "k_pair_atoms launch");
    }
    auto order = [&](auto mixed) {
        constexpr bool M = decltype(mixed)::value;
        static_assert(kPairsJobs <= 4096, "the largest has room for every job");
        auto launch = [&](auto kern, int threads) {
            hipLaunchKernelGGL(kern, dim3(G), dim3(threads), 0, st, G, J, most, pol, from, gap_w, gap_c, ctx->seg_off, atom_dp, area, n_atoms, wait,
                               sla_class, len, list);
        };
        if (J <= 128) launch(k_order_pairs<M, 128, 64>, 64);
        else if (J <= 512) launch(k_order_pairs<M, 512, 256>, 256);
        else if (J <= 1024) launch(k_order_pairs<M, 1024, 512>, 512);
        else if (J <= 2048) launch(k_order_pairs<M, 2048, 1024>, 1024);
        else launch(k_order_pairs<M, 4096, 1024>, 1024);
    };
    if (params->policy == SJA_POLICY_MIXED) order(std::true_type{});
    else order(std::false_type{});
    SJA_HIP(hipGetLastError(), "k_order_pairs launch");
    const RoundsOut out{pol, gap_w, gap_c, ctx->seg_off, n_atoms, atom_dp, atom_db, area, wait, sla_class, grant_job, grant_cut, grant_score, job_gap,
                        rounds_and_stable};
    hipLaunchKernelGGL(k_rounds_pairs, dim3(1), dim3((G + kWave - 1) / kWave * kWave), 0, st, G, J, most, cap, len, list, out);
    SJA_HIP(hipGetLastError(), "k_rounds_pairs launch");
    SJA_HIP(hipStreamSynchronize(st), "final synchronise");
    return SJA_OK;
}

JobLimits job_limits(const sja_limits &l, const int32_t *power, const int32_t *deadline)
{
    JobLimits out;
    out.tau_min = l.tau_min;
    out.tau_max = l.tau_max;
    out.power_cap = l.power_cap;
    out.now = l.now;
    out.power = power;
    out.deadline = deadline;
    return out;
}

// The start and the end of the pair evaluation, for sja_last_fit_kernel_ms.
int mark_kernel(sja_ctx *ctx, hipStream_t st, bool end)
{
    if (!ctx->ev_start) {
        SJA_HIP(hipEventCreate(&ctx->ev_start), "hipEventCreate");
        SJA_HIP(hipEventCreate(&ctx->ev_stop), "hipEventCreate");
    }
    SJA_HIP(hipEventRecord(end ? ctx->ev_stop : ctx->ev_start, st), "hipEventRecord");
    ctx->timed = end;
    return SJA_OK;
}

// fit -> select of a small batch.
int launch_best_pairs(sja_ctx *ctx, hipStream_t st, const Layout &L, int32_t n_gaps, const int32_t *W, const int32_t *C,
                      const sja_params *params, const int32_t *wait, const uint8_t *sla_class, const int32_t *job_held,
                      const uint8_t *gap_active, int32_t *cand_job, int32_t *cand_cut, int64_t *cand_score)
{
    const int J = ctx->n_jobs;
    const bool mixed = params->policy == SJA_POLICY_MIXED;
    int rc = ctx->timing ? mark_kernel(ctx, st, false) : SJA_OK;
    if (rc != SJA_OK) return rc;
    const uint16_t *atoms = pair_atoms(ctx, st, L, n_gaps, W, C);
    SJA_HIP(hipGetLastError(), "k_pair_atoms launch");
    auto kern = atoms ? (mixed ? k_best_pairs<true, true> : k_best_pairs<false, true>) : (mixed ? k_best_pairs<true, false> : k_best_pairs<false, false>);
    hipLaunchKernelGGL(kern, dim3(n_gaps), dim3(pair_threads(J)), 0, st, J, to_dev(params), W, C, ctx->seg_off, ws_ptr<int2>(ctx, L.atom_dp),
                       ws_ptr<int2>(ctx, L.atom_db), atom_area_of(ctx, L), ws_ptr<int32_t>(ctx, L.n_atoms), wait, sla_class, job_held,
                       gap_active, pair_gaps(ctx, L), atoms, cand_job, cand_cut, cand_score);
    SJA_HIP(hipGetLastError(), "k_best_pairs launch");
    return ctx->timing ? mark_kernel(ctx, st, true) : SJA_OK;
}

// The best job per gap by atoms (k_floor.h).  The intermediate results take the space of the list entries, of the
// records and of the partials.
FloorArgs floor_args(sja_ctx *ctx, const Layout &L, int32_t n_gaps, int most_classes, const sja_params *params, const int32_t *wait, const uint8_t *sla_class,
                     const int32_t *job_held)
{
    FloorArgs args{};
    const int64_t room = L.entry_cap * 2 / (kFloorFirstBlocks + 3);
    args.pol = to_dev(params);
    args.n_jobs = ctx->n_jobs;
    args.n_gaps = n_gaps;
    args.most_classes = most_classes;
    args.room = int(room < kFloorBuckets ? room : kFloorBuckets);
    args.seg_off = ctx->seg_off;
    args.atom_dp = ws_ptr<int2>(ctx, L.atom_dp);
    args.atom_area = atom_area_of(ctx, L);
    args.n_atoms = ws_ptr<int32_t>(ctx, L.n_atoms);
    args.plan = ws_ptr<int32_t>(ctx, L.plan);
    args.class_begin = ws_ptr<int32_t>(ctx, L.class_begin);
    args.gap_w = ws_ptr<int32_t>(ctx, L.gap_w);
    args.gap_c = ws_ptr<int32_t>(ctx, L.gap_c);
    args.wait = wait;
    args.sla_class = sla_class;
    args.job_held = job_held;
    args.near = ws_ptr<ulonglong2>(ctx, L.g_ekey0);            // (an entry per segment: entry_cap has two of half its size)
    args.near_job = ws_ptr<ulonglong2>(ctx, L.g_rec);
    args.floors = ws_ptr<uint32_t>(ctx, L.g_ekey1);
    args.floor = args.floors + int64_t(kFloorFirstBlocks) * args.room;
    args.running = args.floor + args.room;
    args.bucket_pos = reinterpret_cast<int32_t *>(args.running + args.room);
    args.n_near = ws_ptr<int32_t>(ctx, L.g_list_off);
    static_assert(kMaxClasses * kListSplits > kFloorBlocks, "room for n_near");
    args.best = ws_ptr<unsigned long long>(ctx, L.sel_part);
    args.second = args.best + n_gaps;
    args.who = reinterpret_cast<int32_t *>(args.second + n_gaps);
    static_assert(sizeof(SelPartial) >= 20, "a partial per gap has room for them");
    return args;
}

// With `reach` the atoms that any class can reach are noted for the lists of sja_resolve, too.
int launch_floor(sja_ctx *ctx, hipStream_t st, const Layout &L, FloorArgs args, bool reach)
{
    const int J = ctx->n_jobs, blocks = floor_blocks_of(J, kFloorBlocks);
    const int floor_step = floor_step_of(J), floor_blocks = floor_blocks_of((J + floor_step - 1) / floor_step, kFloorFirstBlocks);
    if (reach) args.reach = ws_ptr<int32_t>(ctx, L.ncap_tab);
    const bool area = args.atom_area != nullptr;
    hipLaunchKernelGGL(area ? k_floor_first<true> : k_floor_first<false>, dim3(floor_blocks), dim3(kFloorThreads), 0, st, args, floor_step);
    SJA_HIP(hipGetLastError(), "k_floor_first launch");
    hipLaunchKernelGGL(k_floor_merge, dim3((args.room + kFloorMergeEntries - 1) / kFloorMergeEntries), dim3(kFloorMergeThreads), 0, st, args, floor_blocks);
    SJA_HIP(hipGetLastError(), "k_floor_merge launch");
    hipLaunchKernelGGL(area ? k_floor_filter<true> : k_floor_filter<false>, dim3(blocks), dim3(kFloorThreads), 0, st, args);
    SJA_HIP(hipGetLastError(), "k_floor_filter launch");
    if (args.pol.policy == SJA_POLICY_MIXED) {
        hipLaunchKernelGGL(k_floor_ties<true>, dim3(blocks), dim3(kTiesThreads), 0, st, args, 0);
        hipLaunchKernelGGL(k_floor_ties<true>, dim3(blocks), dim3(kTiesThreads), 0, st, args, 1);
    } else {
        hipLaunchKernelGGL(k_floor_ties<false>, dim3(blocks), dim3(kTiesThreads), 0, st, args, 0);
    }
    SJA_HIP(hipGetLastError(), "k_floor_ties launch");
    if (reach) ctx->reach_only = true;
    return SJA_OK;
}

// The running maximum; where the plan has no class tables the best over the partials of the other form's job_tiles.
int launch_floor_reduce(sja_ctx *ctx, hipStream_t st, const Layout &L, const FloorArgs &args, int job_tiles, bool from_matrix, const uint8_t *gap_active,
                        int32_t *cand_job, int32_t *cand_cut, int64_t *cand_score)
{
    auto kern = args.pol.policy == SJA_POLICY_MIXED ? k_floor_reduce<true> : k_floor_reduce<false>;
    static_assert(kReduceGaps <= kFloorTile, "a grid for either form");
    hipLaunchKernelGGL(kern, dim3((args.n_gaps + kReduceGaps - 1) / kReduceGaps), dim3(256), 0, st, args, floor_tile(args.n_gaps), job_tiles, int(from_matrix),
                       ws_ptr<SelPartial>(ctx, L.sel_part), ws_ptr<int32_t>(ctx, L.gap_cls), ws_ptr<int32_t>(ctx, L.gap_order), gap_active,
                       ws_ptr<int2>(ctx, L.atom_db), cand_job, cand_cut, cand_score);
    SJA_HIP(hipGetLastError(), "k_floor_reduce launch");
    return SJA_OK;
}

// Which form looks for the best job per gap where the plan has class tables and the keys rise.  k_range_select looks at the
// ends of every job in every chunk of positions, two gathers each; the k_floor_ kernels at all atoms once or twice and at
// those near the best again, and take 40 us of launches and short kernels, but no start tables after sja_fit_select.
// Near the best are many atoms where many jobs have equal keys, or where many capacities leave few buckets to each.
// k_range_select and they, us, fit -> select by EFFICIENCY of random jobs / of 16 profiles and equal waits / of 64 capacities:
// 30000 gaps x 8000 jobs 129 and 157 / 137 and 181 / 270 and 950, 8192 x 32768 183 and 172 / 187 and 252 / 534 and 980,
// 24000 x 32768 184 and 130 / 181 and 231 / 369 and 444, 32768 x 32768 220 and 135 / 223 and 238 / 449 and 502, 16384 x 65536
// 302 and 151 / 314 and 180 / 585 and 662, 32768 x 65536 345 and 158 / 352 and 192 / 797 and 746, the last of 512 segments
// a job instead of 128 364 and 249 / 374 and 335 / 1628 and 2348; by MIXED 227 and 130 / 475 and 218 / 450 and 201 at that size.
// (Of few jobs the chunks' rows stay in the caches: 150000 x 7000 416 and 324, 32000 x 3500 98 and 110.)
constexpr int64_t kFloorLeast = int64_t(1) << 30;
constexpr int kFloorLeastOfJobs = 6 << 10;
bool by_floor(int64_t n_gaps, int64_t n_jobs) { return n_gaps * n_jobs >= kFloorLeast && n_jobs >= kFloorLeastOfJobs; }

// A select goes along the matrix, which takes 1.05 us per million pairs besides the keys of all cuts whatever the jobs are
// like, or without it.  Matrix / k_range_select, us, random jobs and jobs of 16 profiles with equal waits, 4 to 8 capacities:
// 2048 gaps x 8192 jobs 63 / 67 and 89 / 156, 886 x 20000 57 / 80 and 87 / 102, 8192 x 8192 103 / 70 and 178 / 174, 20000 x 4000
// 111 / 60 and 202 / 104, 4096 x 36000 204 / 115 and 346 / 155.  The more capacities, the fewer gaps to a chunk: 300 x 450000 of
// 8 / 16 / 24 capacities 293 / 183, 312 / 326 and 303 / 381, 700 x 200000 of 16 / 24 243 / 223 and 248 / 273, 2100 x 65600 of 24 / 64
// 209 / 161 and 285 / 415, 4096 x 36000 of 24 / 64 301 / 227 and 300 / 505, 30000 x 8000 of 64 367 / 231.
// Matrix / k_range_select / k_floor_: 5000 x 27000 of 16 profiles 185 / 99 / 304, 9000 x 16400 219 / 155 / 249, of random jobs and 24
// capacities 234 / 156 / 296; 8192 x 32768 of 8 capacities 340 / 105 / 80 to 349 / 141 / 287, of 24 471 / 282 / 530; 16384 x 32768 of
// 24 593 / 259 / 226, of 64 1022 / 538 / 376.
constexpr int64_t kSelectByAtoms = int64_t(1) << 27, kSelectFloor = int64_t(1) << 28, kSelectFloorAnyClasses = int64_t(1) << 29;
constexpr int kSelectFloorGaps = 8 << 10, kSelectFloorClasses = 16;
struct SelectForm {
    bool by_atoms, floor;
    int most_classes;           // of the batches that go without the matrix
};
SelectForm select_form(int64_t n_gaps, int64_t n_jobs)
{
    const int64_t pairs = n_gaps * n_jobs;
    if (n_jobs >= kFloorLeastOfJobs && pairs >= kSelectFloorAnyClasses) return {true, true, kAnyClasses};
    if (n_jobs >= kFloorLeastOfJobs && pairs >= kSelectFloor && n_gaps >= kSelectFloorGaps) return {true, true, kSelectFloorClasses};
    int classes = kMaxClasses;
    while (3 * int64_t(classes) * classes > n_gaps) --classes;
    return {pairs >= kSelectByAtoms, false, classes};
}

// k_range_select, along the start tables: partials of as many tiles of jobs as returned.
int launch_ranges(sja_ctx *ctx, hipStream_t st, const Layout &L, int32_t n_gaps, int most_classes, const sja_params *params, const int32_t *wait,
                  const uint8_t *sla_class, const int32_t *job_held, const uint8_t *gap_active, int *tiles)
{
    const int J = ctx->n_jobs;
    const bool mixed = params->policy == SJA_POLICY_MIXED;
    const long long *atom_area = atom_area_of(ctx, L);
    const int64_t jobs_once = (J + kRangeThreads - 1) / kRangeThreads, chunks = (n_gaps + fit_chunk_len(n_gaps, J) - 1) / fit_chunk_len(n_gaps, J);
    const int chunk_bound = int(chunks) + most_classes;         // (of a batch that is served; 16000 blocks that return at once take 27 us)
    int batches = 1;
    while (batches < kRangeBatches && jobs_once * chunks >= 2 * batches * int64_t(kRangeBlocks)) batches *= 2;
    *tiles = int((jobs_once + batches - 1) / batches);
    auto kern = atom_area ? (mixed ? k_range_select<true, true> : k_range_select<false, true>)
                          : (mixed ? k_range_select<true, false> : k_range_select<false, false>);
    hipLaunchKernelGGL(kern, dim3(unsigned((*tiles + 7) / 8 * 8) * unsigned(chunk_bound)), dim3(kRangeThreads), 0, st, J, n_gaps,
                       chunk_bound, batches, most_classes, to_dev(params), ctx->seg_off, ws_ptr<int2>(ctx, L.atom_dp), atom_area,
                       ws_ptr<int32_t>(ctx, L.plan), ws_ptr<int32_t>(ctx, L.chunk_begin), ws_ptr<int32_t>(ctx, L.chunk_end),
                       ws_ptr<int32_t>(ctx, L.chunk_class), ws_ptr<int32_t>(ctx, L.start_tab), ws_ptr<int32_t>(ctx, L.ncap_tab),
                       ws_ptr<int32_t>(ctx, L.gap_w), ws_ptr<int32_t>(ctx, L.gap_order), wait, sla_class, job_held, gap_active,
                       ws_ptr<SelPartial>(ctx, L.sel_part));
    SJA_HIP(hipGetLastError(), "k_range_select launch");
    return SJA_OK;
}

int launch_range_reduce(sja_ctx *ctx, hipStream_t st, const Layout &L, int32_t n_gaps, int job_tiles, int range_tiles, int most_classes, bool from_matrix,
                        int32_t *cand_job, int32_t *cand_cut, int64_t *cand_score)
{
    hipLaunchKernelGGL(k_range_reduce, dim3((n_gaps + kReduceGaps - 1) / kReduceGaps), dim3(256), 0, st, n_gaps, job_tiles, range_tiles, most_classes, int(from_matrix),
                       ws_ptr<SelPartial>(ctx, L.sel_part), ws_ptr<int32_t>(ctx, L.plan), ws_ptr<int32_t>(ctx, L.gap_w),
                       ws_ptr<int32_t>(ctx, L.gap_c), ctx->seg_off, ws_ptr<int2>(ctx, L.atom_dp), ws_ptr<int2>(ctx, L.atom_db),
                       ws_ptr<int32_t>(ctx, L.n_atoms), cand_job, cand_cut, cand_score);
    SJA_HIP(hipGetLastError(), "k_range_reduce launch");
    return SJA_OK;
}

// The fused fit -> select pass over the planned batch of gaps (the plan of enqueue_gap_plan is in
// the workspace): candidates per gap among the jobs that job_held does not mark, for the gaps that
// gap_active does not switch off.  No cut matrix is read or written.  A batch has class tables or not, and either
// k_range_select or the k_floor_ kernels serve it, or k_fit_select; which, only the device knows, so both are launched and one
// returns at once, unless the caller has seen the plan (2500 gaps of 65 capacities x 1200 jobs: 6 us of a round of 290).
// k_fit_select has a block to a tile all the same: 32768 that return at once take 7 us, but 2048 blocks with a fixed share of
// the tiles each took 672 us where this takes 492 (32000 gaps of 65 capacities x 4500 jobs).
// starts: the start tables are still to be made, where they are needed.
enum class Tabled { Unknown, No, Yes };
int launch_fused(sja_ctx *ctx, hipStream_t st, const Layout &L, int32_t n_gaps, const sja_params *params,
                 const int32_t *wait, const uint8_t *sla_class, const int32_t *job_held, const uint8_t *gap_active,
                 int32_t *cand_job, int32_t *cand_cut, int64_t *cand_score, bool timed, bool starts, bool searched = false, Tabled tabled = Tabled::Unknown)
{
    const int J = ctx->n_jobs;
    const int job_tiles = (J + kFusedBlock - 1) / kFusedBlock;
    bool by_atoms = false;
    int range_tiles = 0;
    FloorArgs args{};
    if (job_tiles > 0 && searched) {
        const bool mixed = params->policy == SJA_POLICY_MIXED;
        const long long *atom_area = atom_area_of(ctx, L);
        auto kern = atom_area ? (mixed ? k_search_select<true, true> : k_search_select<false, true>)
                              : (mixed ? k_search_select<true, false> : k_search_select<false, false>);
        const int rows = (n_gaps + kSearchGaps - 1) / kSearchGaps;
        for (int first = 0; first < rows; first += kSearchRows) {
            const int n_rows = rows - first < kSearchRows ? rows - first : kSearchRows;
            hipLaunchKernelGGL(kern, dim3(job_tiles, n_rows), dim3(kFusedBlock), 0, st, J, n_gaps, first, to_dev(params), ctx->seg_off,
                               ws_ptr<int2>(ctx, L.atom_dp), atom_area, ws_ptr<int32_t>(ctx, L.n_atoms), ws_ptr<int32_t>(ctx, L.gap_w),
                               ws_ptr<int32_t>(ctx, L.gap_c), ws_ptr<int32_t>(ctx, L.gap_order), wait, sla_class, job_held, gap_active,
                               ws_ptr<SelPartial>(ctx, L.sel_part));
            SJA_HIP(hipGetLastError(), "k_search_select launch");
        }
    } else if (job_tiles > 0) {
        const int chunk_bound = int(fit_chunk_bound(n_gaps, J));
        const int tiles8 = (job_tiles + 7) / 8 * 8;
        const unsigned grid = unsigned(tiles8) * unsigned(chunk_bound);
        const bool mixed = params->policy == SJA_POLICY_MIXED;
        const long long *atom_area = atom_area_of(ctx, L);
        auto kern = atom_area ? (mixed ? k_fit_select<kFusedBlock, kFusedWindow, kFusedPeriod, true, true>
                                       : k_fit_select<kFusedBlock, kFusedWindow, kFusedPeriod, false, true>)
                              : (mixed ? k_fit_select<kFusedBlock, kFusedWindow, kFusedPeriod, true, false>
                                       : k_fit_select<kFusedBlock, kFusedWindow, kFusedPeriod, false, false>);
        const bool rise = keys_rise(ctx);
        const bool floor = rise && by_floor(n_gaps, J);
        int rc = starts && !floor ? enqueue_starts(ctx, st, L) : SJA_OK;
        if (rc == SJA_OK && timed) rc = mark_kernel(ctx, st, false);        // (from here on pairs are evaluated)
        if (rc != SJA_OK) return rc;
        if (rise && tabled != Tabled::No) {
            by_atoms = true;
            if (floor) {
                args = floor_args(ctx, L, n_gaps, kAnyClasses, params, wait, sla_class, job_held);
                rc = launch_floor(ctx, st, L, args, starts);
            } else {
                rc = launch_ranges(ctx, st, L, n_gaps, kAnyClasses, params, wait, sla_class, job_held, gap_active, &range_tiles);
            }
            if (rc != SJA_OK) return rc;
        }
        if (!rise || tabled != Tabled::Yes) {
            hipLaunchKernelGGL(kern, dim3(grid), dim3(kFusedBlock), 0, st, J, n_gaps, chunk_bound, int(!rise), to_dev(params),
                               ctx->seg_off, ws_ptr<int2>(ctx, L.atom_dp), atom_area, ws_ptr<int32_t>(ctx, L.n_atoms),
                               ws_ptr<int32_t>(ctx, L.plan), ws_ptr<int32_t>(ctx, L.chunk_begin),
                               ws_ptr<int32_t>(ctx, L.chunk_end), ws_ptr<int32_t>(ctx, L.chunk_class),
                               ws_ptr<int32_t>(ctx, L.chunk_sub), ws_ptr<int32_t>(ctx, L.start_tab),
                               ws_ptr<int32_t>(ctx, L.ncap_tab), ws_ptr<int32_t>(ctx, L.gap_w),
                               ws_ptr<int32_t>(ctx, L.gap_c), ws_ptr<int32_t>(ctx, L.gap_order),
                               ws_ptr<int32_t>(ctx, L.gap_run_end), wait, sla_class, job_held, gap_active,
                               ws_ptr<SelPartial>(ctx, L.sel_part));
            SJA_HIP(hipGetLastError(), "k_fit_select launch");
        }
        if (timed && (rc = mark_kernel(ctx, st, true)) != SJA_OK) return rc;
    }
    if (by_atoms && range_tiles == 0) return launch_floor_reduce(ctx, st, L, args, job_tiles, false, gap_active, cand_job, cand_cut, cand_score);
    if (by_atoms) return launch_range_reduce(ctx, st, L, n_gaps, job_tiles, range_tiles, kAnyClasses, false, cand_job, cand_cut, cand_score);
    hipLaunchKernelGGL(k_fused_reduce, dim3((n_gaps + kReduceGaps - 1) / kReduceGaps), dim3(256), 0, st, n_gaps, job_tiles,
                       ws_ptr<SelPartial>(ctx, L.sel_part), ctx->seg_off, ws_ptr<int2>(ctx, L.atom_db), cand_job,
                       cand_cut, cand_score);
    SJA_HIP(hipGetLastError(), "k_fused_reduce launch");
    return SJA_OK;
}

Hysteresis hysteresis_of(int32_t n_caps, int32_t min_gain, const int32_t *cap)
{
    Hysteresis h{};
    h.n_caps = n_caps;
    h.min_gain = min_gain;
    for (int i = 0; i < n_caps; ++i) h.cap[i] = cap[i];
    return h;
}

// sja_prepare_profiles and its variant on the built-in scratch: the same checks and the same
// kernel; only where the private tables live differs.
int prepare_into(sja_ctx *ctx, void *stream, int32_t n_jobs, int64_t n_segments,
                 const int64_t *seg_off, const int32_t *dur, const int32_t *mem,
                 const uint8_t *safe, const int32_t *progress, int32_t *pre_dur,
                 int32_t *pre_peak, int32_t *prev_safe, bool on_static_scratch)
{
    ctx->prepared = false;
    ctx->fitted = false;
    ctx->planned = false;
    if (n_jobs < 0 || n_jobs > SJA_MAX_JOBS) return fail(ctx, SJA_ERR_SIZE, "n_jobs");
    if (n_segments < 0 || n_segments > SJA_MAX_SEGMENTS) return fail(ctx, SJA_ERR_SIZE, "n_segments");
    if (!seg_off || !progress) return fail(ctx, SJA_ERR_NULL, "seg_off / progress");
    if (n_segments > 0 && (!dur || !mem || !safe || !pre_dur || !pre_peak || !prev_safe))
        return fail(ctx, SJA_ERR_NULL, "profile or output array");
    const Layout L = make_layout(0, n_jobs, n_segments);
    if (on_static_scratch) {
        if (L.total > size_t(SJA_STATIC_SCRATCH_BYTES))
            return fail(ctx, SJA_ERR_SIZE, "n_jobs / n_segments beyond what the built-in scratch holds "
                                           "(sja_workspace_bytes(0, n_jobs, n_segments) > SJA_STATIC_SCRATCH_BYTES)");
    } else if (!ctx->ws || ctx->ws_bytes < L.total) {
        return fail(ctx, SJA_ERR_WORKSPACE, "workspace too small for prepare");
    }

    DeviceGuard guard(ctx->device);
    SJA_HIP(guard.err, "hipSetDevice");
    if (on_static_scratch) {
        void *p = nullptr;
        SJA_HIP(static_scratch(ctx->device, &p), "hipGetSymbolAddress(scratch)");
        ctx->ws = static_cast<char *>(p);
        ctx->ws_bytes = size_t(SJA_STATIC_SCRATCH_BYTES);
    }
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (n_jobs > 0) {
        const int jobs_per_block = 256 / kWave;
        const dim3 grid((n_jobs + jobs_per_block - 1) / jobs_per_block), block(256);
        const bool by_area = ctx->score_mode == SJA_SCORE_AREA;
        const Hysteresis hyst = hysteresis_of(ctx->hyst_n_caps, ctx->hyst_min_gain, ctx->hyst_cap);
        long long *pre_area = by_area ? ws_ptr<long long>(ctx, L.pre_area) : nullptr;
        long long *atom_area = by_area || hyst.n_caps > 0 ? ws_ptr<long long>(ctx, L.atom_area) : nullptr;
        if (ctx->limits_on) {
            const JobLimits lim = job_limits(ctx->limits, ctx->lim_power, ctx->lim_deadline);
            hipLaunchKernelGGL(k_prepare<true>, grid, block, 0, st, lim, hyst, pre_area, atom_area, n_jobs, seg_off, dur, mem, safe, progress,
                               pre_dur, pre_peak, prev_safe, ws_ptr<int2>(ctx, L.atom_dp),
                               ws_ptr<int2>(ctx, L.atom_db), ws_ptr<int32_t>(ctx, L.n_atoms),
                               ws_ptr<int2>(ctx, L.first_dp));
        } else {
            hipLaunchKernelGGL(k_prepare<false>, grid, block, 0, st, JobLimits{}, hyst, pre_area, atom_area, n_jobs, seg_off, dur, mem, safe,
                               progress, pre_dur, pre_peak, prev_safe, ws_ptr<int2>(ctx, L.atom_dp),
                               ws_ptr<int2>(ctx, L.atom_db), ws_ptr<int32_t>(ctx, L.n_atoms),
                               ws_ptr<int2>(ctx, L.first_dp));
        }
        SJA_HIP(hipGetLastError(), "k_prepare launch");
    }
    ctx->limits_used = ctx->limits_on;
    ctx->score_used = ctx->score_mode;
    ctx->hyst_used_n_caps = ctx->hyst_n_caps;
    ctx->hyst_used_min_gain = ctx->hyst_min_gain;
    memcpy(ctx->hyst_used_cap, ctx->hyst_cap, sizeof(ctx->hyst_cap));
    ctx->limits_applied = ctx->limits;
    ctx->used_power = ctx->lim_power;
    ctx->used_deadline = ctx->lim_deadline;
    ctx->n_jobs = n_jobs;
    ctx->n_segments = n_segments;
    ctx->seg_off = seg_off;
    ctx->dur = dur;
    ctx->mem = mem;
    ctx->safe = safe;
    ctx->pre_dur = pre_dur;
    ctx->pre_peak = pre_peak;
    ctx->prev_safe = prev_safe;
    ctx->prepared = true;
    return SJA_OK;
}

}  // namespace

extern "C" {

const char *sja_status_string(int status)
{
    switch (status) {
    case SJA_OK: return "SJA_OK";
    case SJA_ERR_NULL: return "SJA_ERR_NULL";
    case SJA_ERR_SIZE: return "SJA_ERR_SIZE";
    case SJA_ERR_POLICY: return "SJA_ERR_POLICY";
    case SJA_ERR_STATE: return "SJA_ERR_STATE";
    case SJA_ERR_OVERFLOW: return "SJA_ERR_OVERFLOW";
    case SJA_ERR_WORKSPACE: return "SJA_ERR_WORKSPACE";
    case SJA_ERR_HIP: return "SJA_ERR_HIP";
    case SJA_ERR_NOT_IMPLEMENTED: return "SJA_ERR_NOT_IMPLEMENTED";
    default: return "SJA_ERR_UNKNOWN";
    }
}

const char *sja_last_error(const sja_ctx *ctx) { return ctx ? ctx->err : "null context"; }

int sja_create(sja_ctx **out, int device_id)
{
    if (!out) return SJA_ERR_NULL;
    *out = nullptr;
    if (device_id < 0) return SJA_ERR_SIZE;
    sja_ctx *ctx = new (std::nothrow) sja_ctx();
    if (!ctx) return SJA_ERR_WORKSPACE;
    memset(ctx, 0, sizeof(*ctx));
    ctx->device = device_id;
    *out = ctx;
    return SJA_OK;
}

int sja_destroy(sja_ctx *ctx)
{
    if (!ctx) return SJA_ERR_NULL;
    if (ctx->ev_start) (void)hipEventDestroy(ctx->ev_start);
    if (ctx->ev_stop) (void)hipEventDestroy(ctx->ev_stop);
    delete ctx;
    return SJA_OK;
}

size_t sja_workspace_bytes(int64_t n_gaps, int64_t n_jobs, int64_t n_segments)
{
    if (n_gaps < 0 || n_jobs < 0 || n_segments < 0) return 0;
    if (n_gaps > SJA_MAX_GAPS || n_jobs > SJA_MAX_JOBS || n_segments > SJA_MAX_SEGMENTS) return 0;
    return make_layout(n_gaps, n_jobs, n_segments).total;
}

int sja_set_workspace(sja_ctx *ctx, void *dev_ptr, size_t bytes)
{
    if (!ctx) return SJA_ERR_NULL;
    if (!dev_ptr && bytes) return fail(ctx, SJA_ERR_NULL, "workspace pointer");
    if (reinterpret_cast<uintptr_t>(dev_ptr) & 255) return fail(ctx, SJA_ERR_WORKSPACE, "workspace must be 256-byte aligned");
    ctx->ws = static_cast<char *>(dev_ptr);
    ctx->ws_bytes = bytes;
    ctx->prepared = false;   // private tables lived in the old workspace
    ctx->fitted = false;
    ctx->planned = false;
    return SJA_OK;
}

int sja_validate(sja_ctx *ctx, void *stream, int32_t n_jobs, int64_t n_segments, const int64_t *seg_off,
                 const int32_t *dur, const int32_t *mem, const int32_t *progress, const sja_params *params,
                 const int32_t *wait, const uint8_t *sla_class, uint32_t *problems)
{
    if (!ctx) return SJA_ERR_NULL;
    if (n_jobs < 0 || n_jobs > SJA_MAX_JOBS) return fail(ctx, SJA_ERR_SIZE, "n_jobs");
    if (n_segments < 0 || n_segments > SJA_MAX_SEGMENTS) return fail(ctx, SJA_ERR_SIZE, "n_segments");
    if (!seg_off || !problems) return fail(ctx, SJA_ERR_NULL, "seg_off / problems");
    if (n_jobs > 0 && !progress) return fail(ctx, SJA_ERR_NULL, "progress");
    if (n_segments > 0 && (!dur || !mem)) return fail(ctx, SJA_ERR_NULL, "dur / mem");
    PolicyDev pol{};
    if (params) {
        const int rc = check_params(ctx, params, wait, sla_class);
        if (rc != SJA_OK) return rc;
        pol = to_dev(params);
    }
    DeviceGuard guard(ctx->device);
    SJA_HIP(guard.err, "hipSetDevice");
    hipStream_t st = static_cast<hipStream_t>(stream);
    hipLaunchKernelGGL(k_fill_i32, dim3(1), dim3(64), 0, st, reinterpret_cast<int32_t *>(problems), int64_t(1), 0);
    SJA_HIP(hipGetLastError(), "k_fill_i32 launch");
    if (n_jobs > 0) {
        const int jobs_per_block = 256 / kWave;
        hipLaunchKernelGGL(k_validate, dim3((n_jobs + jobs_per_block - 1) / jobs_per_block), dim3(256), 0, st, n_jobs,
                           n_segments, seg_off, dur, mem, progress, params != nullptr, pol, wait, sla_class, problems);
        SJA_HIP(hipGetLastError(), "k_validate launch");
    }
    return SJA_OK;
}

int sja_enable_timing(sja_ctx *ctx, int on)
{
    if (!ctx) return SJA_ERR_NULL;
    ctx->timing = on != 0;
    ctx->timed = false;
    return SJA_OK;
}

int sja_set_resolve_mode(sja_ctx *ctx, int mode)
{
    if (!ctx) return SJA_ERR_NULL;
    if (mode != SJA_RESOLVE_LISTS && mode != SJA_RESOLVE_MATRIX && mode != SJA_RESOLVE_LISTS_LOOKUP)
        return fail(ctx, SJA_ERR_SIZE, "sja_set_resolve_mode: unknown mode");
    ctx->resolve_mode = mode;
    return SJA_OK;
}

int sja_last_fit_kernel_ms(sja_ctx *ctx, float *ms_host)
{
    if (!ctx) return SJA_ERR_NULL;
    if (!ms_host) return fail(ctx, SJA_ERR_NULL, "ms_host");
    if (!ctx->timed) return fail(ctx, SJA_ERR_STATE, "no timed sja_fit has run");
    SJA_HIP(hipEventSynchronize(ctx->ev_stop), "hipEventSynchronize");
    SJA_HIP(hipEventElapsedTime(ms_host, ctx->ev_start, ctx->ev_stop), "hipEventElapsedTime");
    return SJA_OK;
}

int sja_set_score(sja_ctx *ctx, int score)
{
    if (!ctx) return SJA_ERR_NULL;
    if (score != SJA_SCORE_RECTANGLE && score != SJA_SCORE_AREA) return fail(ctx, SJA_ERR_SIZE, "unknown score");
    ctx->score_mode = score;
    return SJA_OK;
}

int sja_set_limits(sja_ctx *ctx, const sja_limits *limits, const int32_t *power, const int32_t *deadline)
{
    if (!ctx) return SJA_ERR_NULL;
    if (!limits) {
        ctx->limits_on = false;
        ctx->lim_power = nullptr;
        ctx->lim_deadline = nullptr;
        return SJA_OK;
    }
    if (limits->tau_min < 0 || limits->tau_max < 0) return fail(ctx, SJA_ERR_SIZE, "tau_min / tau_max");
    ctx->limits = *limits;
    ctx->lim_power = power;
    ctx->lim_deadline = deadline;
    ctx->limits_on = true;
    return SJA_OK;
}

int sja_set_hysteresis(sja_ctx *ctx, int32_t n_caps, const int32_t *cap_set, int32_t min_gain)
{
    if (!ctx) return SJA_ERR_NULL;
    if (n_caps < 0 || n_caps > SJA_MAX_CAPS) return fail(ctx, SJA_ERR_SIZE, "n_caps");
    if (n_caps == 0) {
        ctx->hyst_n_caps = 0;
        return SJA_OK;
    }
    if (!cap_set) return fail(ctx, SJA_ERR_NULL, "cap_set");
    if (min_gain < 1) return fail(ctx, SJA_ERR_SIZE, "min_gain must be >= 1");
    for (int i = 1; i < n_caps; ++i)
        if (cap_set[i] < cap_set[i - 1]) return fail(ctx, SJA_ERR_SIZE, "cap_set must ascend");
    ctx->hyst_n_caps = n_caps;
    ctx->hyst_min_gain = min_gain;
    for (int i = 0; i < n_caps; ++i) ctx->hyst_cap[i] = cap_set[i];
    return SJA_OK;
}

int sja_prepare_profiles(sja_ctx *ctx, void *stream, int32_t n_jobs, int64_t n_segments,
                         const int64_t *seg_off, const int32_t *dur, const int32_t *mem,
                         const uint8_t *safe, const int32_t *progress, int32_t *pre_dur,
                         int32_t *pre_peak, int32_t *prev_safe)
{
    if (!ctx) return SJA_ERR_NULL;
    return prepare_into(ctx, stream, n_jobs, n_segments, seg_off, dur, mem, safe, progress, pre_dur, pre_peak,
                        prev_safe, false);
}

int sja_prepare_profiles_static(sja_ctx *ctx, void *stream, int32_t n_jobs, int64_t n_segments,
                                const int64_t *seg_off, const int32_t *dur, const int32_t *mem,
                                const uint8_t *safe, const int32_t *progress, int32_t *pre_dur,
                                int32_t *pre_peak, int32_t *prev_safe)
{
    if (!ctx) return SJA_ERR_NULL;
    return prepare_into(ctx, stream, n_jobs, n_segments, seg_off, dur, mem, safe, progress, pre_dur, pre_peak,
                        prev_safe, true);
}

int sja_fit(sja_ctx *ctx, void *stream, int32_t n_gaps, const int32_t *W, const int32_t *C,
            int32_t *cut, uint32_t *interest_bits)
{
    if (!ctx) return SJA_ERR_NULL;
    ctx->fitted = false;
    ctx->planned = false;
    ctx->timed = false;
    if (!ctx->prepared) return fail(ctx, SJA_ERR_STATE, "sja_fit before sja_prepare_profiles");
    if (n_gaps < 0 || n_gaps > SJA_MAX_GAPS) return fail(ctx, SJA_ERR_SIZE, "n_gaps");
    if (n_gaps > 0 && (!W || !C)) return fail(ctx, SJA_ERR_NULL, "W / C");
    const int J = ctx->n_jobs;
    if (n_gaps > 0 && J > 0 && !cut) return fail(ctx, SJA_ERR_NULL, "cut");
    const Layout L = make_layout(n_gaps, J, ctx->n_segments);
    if (!ctx->ws || ctx->ws_bytes < L.total) return fail(ctx, SJA_ERR_WORKSPACE, "workspace too small for this many gaps");

    DeviceGuard guard(ctx->device);
    SJA_HIP(guard.err, "hipSetDevice");
    hipStream_t st = static_cast<hipStream_t>(stream);
    const bool pairs = pairs_batch(ctx, L, n_gaps, J);
    if (n_gaps > 0) {
        const int words = (J + 31) / 32;
        const int chunk_bound = int(fit_chunk_bound(n_gaps, J));
        const dim3 b256(256);
        int32_t *gw = ws_ptr<int32_t>(ctx, L.gap_w), *gcap = ws_ptr<int32_t>(ctx, L.gap_c);
        int32_t *plan = ws_ptr<int32_t>(ctx, L.plan);
        int rc = SJA_OK;
        if (pairs) {
            if (ctx->timing && (rc = mark_kernel(ctx, st, false)) != SJA_OK) return rc;
            hipLaunchKernelGGL(k_fit_pairs, dim3((J + kPairsThreads - 1) / kPairsThreads, (n_gaps + kPairsQ - 1) / kPairsQ), dim3(kPairsThreads), 0, st,
                               n_gaps, J, W, C, ctx->seg_off, ws_ptr<int2>(ctx, L.atom_dp), ws_ptr<int2>(ctx, L.atom_db),
                               ws_ptr<int32_t>(ctx, L.n_atoms), pair_gaps(ctx, L), cut, interest_bits);
            SJA_HIP(hipGetLastError(), "k_fit_pairs launch");
            if (ctx->timing && (rc = mark_kernel(ctx, st, true)) != SJA_OK) return rc;
        } else {
            rc = enqueue_gap_plan(ctx, st, L, n_gaps, W, C);
            if (rc == SJA_OK) rc = enqueue_starts(ctx, st, L);
            if (rc != SJA_OK) return rc;
        }
        if (J > 0 && !pairs) {
            const int job_tiles = (J + kFitBlock - 1) / kFitBlock;
            const int tiles8 = (job_tiles + 7) / 8 * 8;
            const unsigned grid = unsigned(tiles8) * unsigned(chunk_bound);
            if (ctx->timing && (rc = mark_kernel(ctx, st, false)) != SJA_OK) return rc;
            hipLaunchKernelGGL((k_fit_main<kFitBlock, kFitWindow, kFitPeriod>), dim3(grid), dim3(kFitBlock), 0, st,
                               J, chunk_bound, ctx->seg_off, ws_ptr<int2>(ctx, L.atom_dp),
                               ws_ptr<int2>(ctx, L.atom_db), ws_ptr<int32_t>(ctx, L.n_atoms), plan,
                               ws_ptr<int32_t>(ctx, L.chunk_begin), ws_ptr<int32_t>(ctx, L.chunk_end),
                               ws_ptr<int32_t>(ctx, L.chunk_class), ws_ptr<int32_t>(ctx, L.chunk_sub),
                               ws_ptr<int32_t>(ctx, L.start_tab),
                               ws_ptr<int32_t>(ctx, L.ncap_tab), gw, gcap, ws_ptr<int64_t>(ctx, L.gap_row),
                               ws_ptr<int32_t>(ctx, L.gap_run_end), cut);
            SJA_HIP(hipGetLastError(), "k_fit_main launch");
            if (ctx->timing && (rc = mark_kernel(ctx, st, true)) != SJA_OK) return rc;
            if (interest_bits) {
                uint32_t *table = ws_ptr<uint32_t>(ctx, L.bits_table);
                int32_t *class_dmax = ws_ptr<int32_t>(ctx, L.class_dmax);
                hipLaunchKernelGGL(k_bits_table, dim3((words + 255) / 256, kMaxClasses), b256, 0, st, J, words, plan,
                                   ws_ptr<int32_t>(ctx, L.class_begin), gcap, ws_ptr<int2>(ctx, L.first_dp), table, class_dmax);
                SJA_HIP(hipGetLastError(), "k_bits_table launch");
                BitsArgs bits{};
                bits.bits = interest_bits;
                bits.first_dp = ws_ptr<int2>(ctx, L.first_dp);
                bits.table = table;
                bits.class_dmax = class_dmax;
                bits.gap_order = ws_ptr<int32_t>(ctx, L.gap_order);
                bits.gap_cls = ws_ptr<int32_t>(ctx, L.gap_cls);
                bits.n_gaps = n_gaps;
                bits.words = words;
                const int64_t col_tiles = (words + 256 * kBitsWords - 1) / (256 * kBitsWords);
                const int64_t row_tiles = (n_gaps + kBitsRows - 1) / kBitsRows;
                hipLaunchKernelGGL(k_fit_bits, dim3(unsigned(col_tiles * row_tiles)), b256, 0, st, bits, J, plan, gw, gcap);
                SJA_HIP(hipGetLastError(), "k_fit_bits launch");
                const int low_tiles = int((words + 255) / 256), low_rows = fit_low_rows(low_tiles, n_gaps);
                hipLaunchKernelGGL(k_fit_bits_low, dim3(low_tiles, (n_gaps + low_rows - 1) / low_rows), b256, 0, st,
                                   bits, J, low_rows, plan, gw);
                SJA_HIP(hipGetLastError(), "k_fit_bits launch");
            }
        }
    }
    ctx->n_gaps = n_gaps;
    ctx->cut = cut;
    ctx->fitted = true;
    ctx->planned = true;
    ctx->pairs = pairs;
    return SJA_OK;
}

int sja_store_reference(sja_ctx *ctx, void *stream, int32_t *cut)
{
    if (!ctx) return SJA_ERR_NULL;
    if (!ctx->planned) return fail(ctx, SJA_ERR_STATE, "sja_store_reference before sja_fit or sja_fit_select");
    const int G = ctx->n_gaps, J = ctx->n_jobs;
    if (G > 0 && J > 0 && !cut) return fail(ctx, SJA_ERR_NULL, "cut");
    const Layout L = make_layout(G, J, ctx->n_segments);
    if (!ctx->ws || ctx->ws_bytes < L.total) return fail(ctx, SJA_ERR_WORKSPACE, "workspace too small");
    DeviceGuard guard(ctx->device);
    SJA_HIP(guard.err, "hipSetDevice");
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int job_tiles = (J + kFitBlock - 1) / kFitBlock;
    if (G > 0 && job_tiles > 0) {
        if (ctx->pairs) {
            const int rc = plan_pairs(ctx, st, L);
            if (rc != SJA_OK) return rc;
        }
        const int chunk_bound = int(fit_chunk_bound(G, J));
        const int tiles8 = (job_tiles + 7) / 8 * 8;
        hipLaunchKernelGGL(k_store_reference<kFitBlock>, dim3(unsigned(tiles8) * unsigned(chunk_bound)), dim3(kFitBlock), 0, st,
                           J, chunk_bound, ws_ptr<int32_t>(ctx, L.plan), ws_ptr<int32_t>(ctx, L.chunk_begin),
                           ws_ptr<int32_t>(ctx, L.chunk_end), ws_ptr<int64_t>(ctx, L.gap_row), cut);
        SJA_HIP(hipGetLastError(), "k_store_reference launch");
    }
    if (cut == ctx->cut) ctx->fitted = false;      // the matrix of the last sja_fit no longer holds its replies
    return SJA_OK;
}

int sja_fit_select(sja_ctx *ctx, void *stream, int32_t n_gaps, const int32_t *W, const int32_t *C,
                   const sja_params *params, const int32_t *wait, const uint8_t *sla_class,
                   const int32_t *job_held, const uint8_t *gap_active, int32_t *cand_job, int32_t *cand_cut,
                   int64_t *cand_score)
{
    if (!ctx) return SJA_ERR_NULL;
    ctx->fitted = false;
    ctx->planned = false;
    ctx->timed = false;
    if (!ctx->prepared) return fail(ctx, SJA_ERR_STATE, "sja_fit_select before sja_prepare_profiles");
    if (n_gaps < 0 || n_gaps > SJA_MAX_GAPS) return fail(ctx, SJA_ERR_SIZE, "n_gaps");
    if (n_gaps > 0 && (!W || !C)) return fail(ctx, SJA_ERR_NULL, "W / C");
    int rc = check_params(ctx, params, wait, sla_class);
    if (rc != SJA_OK) return rc;
    if (n_gaps > 0 && (!cand_job || !cand_cut || !cand_score)) return fail(ctx, SJA_ERR_NULL, "candidate outputs");
    const int J = ctx->n_jobs;
    const Layout L = make_layout(n_gaps, J, ctx->n_segments);
    if (!ctx->ws || ctx->ws_bytes < L.total) return fail(ctx, SJA_ERR_WORKSPACE, "workspace too small for this many gaps");

    DeviceGuard guard(ctx->device);
    SJA_HIP(guard.err, "hipSetDevice");
    hipStream_t st = static_cast<hipStream_t>(stream);
    const bool pairs = pairs_batch(ctx, L, n_gaps, J);
    if (n_gaps > 0 && pairs) {
        rc = launch_best_pairs(ctx, st, L, n_gaps, W, C, params, wait, sla_class, job_held, gap_active, cand_job, cand_cut, cand_score);
        if (rc != SJA_OK) return rc;
    } else if (n_gaps > 0) {
        rc = enqueue_gap_plan(ctx, st, L, n_gaps, W, C);
        if (rc != SJA_OK) return rc;
        rc = launch_fused(ctx, st, L, n_gaps, params, wait, sla_class, job_held, gap_active, cand_job, cand_cut,
                          cand_score, ctx->timing, true);
        if (rc != SJA_OK) return rc;
    }
    ctx->n_gaps = n_gaps;
    ctx->cut = nullptr;
    ctx->planned = true;
    ctx->pairs = pairs;
    return SJA_OK;
}

int sja_select(sja_ctx *ctx, void *stream, const sja_params *params, const int32_t *wait,
               const uint8_t *sla_class, const int32_t *job_held, const uint8_t *gap_active,
               int32_t *cand_job, int32_t *cand_cut, int64_t *cand_score)
{
    if (!ctx) return SJA_ERR_NULL;
    if (!ctx->fitted) return fail(ctx, SJA_ERR_STATE, "sja_select before sja_fit");
    int rc = check_params(ctx, params, wait, sla_class);
    if (rc != SJA_OK) return rc;
    if (ctx->n_gaps > 0 && (!cand_job || !cand_cut || !cand_score)) return fail(ctx, SJA_ERR_NULL, "candidate outputs");
    const Layout L = make_layout(ctx->n_gaps, ctx->n_jobs, ctx->n_segments);
    if (!ctx->ws || ctx->ws_bytes < L.total) return fail(ctx, SJA_ERR_WORKSPACE, "workspace too small");
    DeviceGuard guard(ctx->device);
    SJA_HIP(guard.err, "hipSetDevice");
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (ctx->pairs && ctx->n_gaps > 0) {
        auto kern = params->policy == SJA_POLICY_MIXED ? k_select_pairs<true> : k_select_pairs<false>;
        hipLaunchKernelGGL(kern, dim3(ctx->n_gaps), dim3(pair_threads(ctx->n_jobs)), 0, st, ctx->n_jobs, to_dev(params), ctx->seg_off, ctx->pre_dur,
                           ctx->pre_peak, pre_area_of(ctx, L), ctx->cut, wait, sla_class, job_held, gap_active, cand_job, cand_cut,
                           cand_score);
        SJA_HIP(hipGetLastError(), "k_select_pairs launch");
        return SJA_OK;
    }
    const int G = ctx->n_gaps, J = ctx->n_jobs, job_tiles = (J + kSelBlock - 1) / kSelBlock;
    const SelectForm form = select_form(G, J);
    if (!keys_rise(ctx) || !form.by_atoms)
        return launch_select(ctx, st, params, wait, sla_class, job_held, gap_active, cand_job, cand_cut, cand_score);
    // along the plan of the fit, without reading the matrix; along the matrix if the plan has no class tables or too many classes
    FloorArgs args{};
    int range_tiles = 0;
    if (form.floor) {
        args = floor_args(ctx, L, G, form.most_classes, params, wait, sla_class, job_held);
        rc = launch_floor(ctx, st, L, args, false);
    } else {
        rc = launch_ranges(ctx, st, L, G, form.most_classes, params, wait, sla_class, job_held, gap_active, &range_tiles);
    }
    if (rc == SJA_OK) rc = launch_matrix_pass(ctx, st, L, params, wait, sla_class, job_held, gap_active, form.most_classes, false);
    if (rc != SJA_OK) return rc;
    return form.floor ? launch_floor_reduce(ctx, st, L, args, job_tiles, true, gap_active, cand_job, cand_cut, cand_score)
                      : launch_range_reduce(ctx, st, L, G, job_tiles, range_tiles, form.most_classes, true, cand_job, cand_cut, cand_score);
}

int sja_resolve(sja_ctx *ctx, void *stream, const sja_params *params, const int32_t *wait,
                const uint8_t *sla_class, int32_t *grant_job, int32_t *grant_cut,
                int64_t *grant_score, int32_t *job_gap, int32_t *rounds_used_and_stable)
{
    if (!ctx) return SJA_ERR_NULL;
    if (!ctx->planned) return fail(ctx, SJA_ERR_STATE, "sja_resolve before sja_fit or sja_fit_select");
    int rc = check_params(ctx, params, wait, sla_class);
    if (rc != SJA_OK) return rc;
    const int G = ctx->n_gaps, J = ctx->n_jobs;
    if (G > 0 && (!grant_job || !grant_cut || !grant_score)) return fail(ctx, SJA_ERR_NULL, "grant outputs");
    if (J > 0 && !job_gap) return fail(ctx, SJA_ERR_NULL, "job_gap");
    if (!rounds_used_and_stable) return fail(ctx, SJA_ERR_NULL, "rounds_used_and_stable");
    const Layout L = make_layout(G, J, ctx->n_segments);
    if (!ctx->ws || ctx->ws_bytes < L.total) return fail(ctx, SJA_ERR_WORKSPACE, "workspace too small");

    DeviceGuard guard(ctx->device);
    SJA_HIP(guard.err, "hipSetDevice");
    hipStream_t st = static_cast<hipStream_t>(stream);

    // every round that does not end the process grants at least one job, so it
    // ends by itself within min(G, J) + 1 rounds: a larger cap changes nothing
    const int64_t natural = int64_t(G < J ? G : J) + 1;
    const int64_t cap = (params->max_rounds > 0 && params->max_rounds < natural) ? params->max_rounds : natural;
    if (ctx->pairs && G > 0 && ctx->resolve_mode == SJA_RESOLVE_LISTS)
        return resolve_pairs(ctx, st, L, params, wait, sla_class, grant_job, grant_cut, grant_score, job_gap, int(cap), rounds_used_and_stable);
    if (ctx->pairs && G > 0 && ctx->resolve_mode != SJA_RESOLVE_MATRIX && (rc = plan_pairs(ctx, st, L)) != SJA_OK) return rc;

    int32_t *cand_job = ws_ptr<int32_t>(ctx, L.res_cand_job);
    int32_t *cand_cut = ws_ptr<int32_t>(ctx, L.res_cand_cut);
    int64_t *cand_score = ws_ptr<int64_t>(ctx, L.res_cand_score);
    uint8_t *active = ws_ptr<uint8_t>(ctx, L.res_active);
    unsigned long long *claim = ws_ptr<unsigned long long>(ctx, L.res_claim);
    int32_t *counters = ws_ptr<int32_t>(ctx, L.res_counters);

    ClearList clear{};
    int n_init = G > J ? G : J;
    if (G > 0 && J > 0) {
        auto also = [&, k = 0](size_t off, int64_t n) mutable {
            clear.p[k] = ws_ptr<int32_t>(ctx, off);
            clear.n[k++] = int(n);
            if (n > n_init) n_init = int(n);
        };
        also(L.res_counters, 16);
        also(L.g_list_off, list_block_bound(G, J) + 2);
        also(L.g_ekey1, 2 * (L.entry_cap < kAlikeSlots ? L.entry_cap : kAlikeSlots));      // (used if there are more atoms than that)
        also(L.g_cnt_lost, (G < J ? G : J) + 4);
        also(L.g_cnt_cand, (G < J ? G : J) + 4);
        also(L.g_state, 2 * kKeyGroupSums);        // (radix_pass)
        if (held_bitmap_words(J) <= kHeldMaxWords) also(L.g_held, 2 * held_bitmap_words(J));
    }
    if (n_init > 0) {
        hipLaunchKernelGGL(k_resolve_init, dim3((n_init + 255) / 256), dim3(256), 0, st, G, J, grant_job,
                           grant_cut, grant_score, job_gap, active, claim, clear);
        SJA_HIP(hipGetLastError(), "k_resolve_init launch");
    }
    int32_t result[2] = {0, 0};
    bool done = false, many_capacities = false, has_tables = false;
    Tabled tabled = Tabled::Unknown;
    if (G > 0 && J > 0 && ctx->resolve_mode != SJA_RESOLVE_MATRIX) {
        rc = resolve_with_lists(ctx, st, L, params, wait, sla_class, grant_job, grant_cut, grant_score, job_gap, cap,
                                rounds_used_and_stable, &done, &has_tables, &many_capacities);
        if (rc != SJA_OK) return rc;
        tabled = has_tables ? Tabled::Yes : Tabled::No;
    }
    if (done) {
        SJA_HIP(hipStreamSynchronize(st), "final synchronise");
        return SJA_OK;
    }
    // Rounds go out in batches between looks at their counters (a pair a round): a round after the last one finds
    // no candidate and changes nothing.  It costs little where pairs are searched; the other forms pay a full
    // pass over all pairs for it, so their batches are an eighth of the rounds done, and only while a pass takes
    // no longer than a few looks (3 rounds of 6000 gaps x 12000 jobs: 311 us one by one, 465 in batches of 2
    // and 4; 272 rounds of 700 x 2501: 12.0 ms one by one, 8.6 so).
    constexpr int kMostRounds = 8;
    constexpr int64_t kShortPass = int64_t(1) << 24;        // pairs; 40 us
    const bool searched = (many_capacities || ctx->pairs) && !ctx->fitted;
    auto batch_from = [&](int64_t r) -> int64_t {
        const int64_t n = searched ? r + 1 : int64_t(G) * J <= kShortPass ? r / 8 : 1;
        return n < 1 ? 1 : n < kMostRounds ? n : kMostRounds;
    };
    for (int64_t r = 1; r <= cap;) {
        const int64_t batch = batch_from(r);
        const int n = G == 0 ? 1 : int(cap - r + 1 < batch ? cap - r + 1 : batch);
        int32_t host_counters[2 * kMostRounds] = {0};
        for (int k = 0; k < n && G > 0; ++k) {
            // the round's selection over the still-active gaps and un-held jobs: from the cut matrix if
            // sja_fit left one, else by evaluating the pairs again (nothing is stored)
            if (ctx->fitted)
                rc = launch_select(ctx, st, params, wait, sla_class, job_gap, active, cand_job, cand_cut, cand_score,
                                   /*keys_ready=*/r + k > 1);
            else
                rc = launch_fused(ctx, st, L, G, params, wait, sla_class, job_gap, active, cand_job, cand_cut, cand_score,
                                  false, false, searched, tabled);
            if (rc != SJA_OK) return rc;
            const dim3 grid((G + 255) / 256), block(256);
            hipLaunchKernelGGL(k_claim, grid, block, 0, st, G, int(r) + k, active, cand_job, claim, counters + 2 * k);
            SJA_HIP(hipGetLastError(), "k_claim launch");
            hipLaunchKernelGGL(k_commit, grid, block, 0, st, G, int(r) + k, active, cand_job, cand_cut, cand_score,
                               claim, grant_job, grant_cut, grant_score, job_gap, counters + 2 * k);
            SJA_HIP(hipGetLastError(), "k_commit launch");
        }
        if (G > 0) {
            SJA_HIP(hipMemcpyAsync(host_counters, counters, size_t(n) * 8, hipMemcpyDeviceToHost, st), "counter readback");
            SJA_HIP(hipStreamSynchronize(st), "round synchronise");
        }
        for (int k = 0; k < n && !result[1]; ++k) {
            result[0] = int32_t(r) + k;
            if (host_counters[2 * k] == 0 || host_counters[2 * k + 1] == 0) result[1] = 1;
        }
        if (result[1]) break;
        r += n;
    }
    SJA_HIP(hipMemcpyAsync(rounds_used_and_stable, result, sizeof(result), hipMemcpyHostToDevice, st),
            "rounds writeback");
    SJA_HIP(hipStreamSynchronize(st), "final synchronise");
    return SJA_OK;
}

int sja_advance(sja_ctx *ctx, void *stream, int32_t n_gaps, const int32_t *W, const int32_t *C,
                const int32_t *grant_job, const int32_t *grant_cut, const int32_t *job_gap, int32_t *progress,
                int32_t *wait, int32_t wait_step, int64_t *metrics)
{
    if (!ctx) return SJA_ERR_NULL;
    if (!ctx->prepared) return fail(ctx, SJA_ERR_STATE, "sja_advance before sja_prepare_profiles");
    if (n_gaps < 0 || n_gaps > SJA_MAX_GAPS) return fail(ctx, SJA_ERR_SIZE, "n_gaps");
    if (wait_step < 0) return fail(ctx, SJA_ERR_SIZE, "wait_step");
    if (n_gaps > 0 && (!W || !C || !grant_job || !grant_cut)) return fail(ctx, SJA_ERR_NULL, "gap arrays");
    const int J = ctx->n_jobs;
    if (J > 0 && (!job_gap || !progress)) return fail(ctx, SJA_ERR_NULL, "job_gap / progress");
    if (!metrics) return fail(ctx, SJA_ERR_NULL, "metrics");
    const Layout L = make_layout(0, J, ctx->n_segments);
    if (!ctx->ws || ctx->ws_bytes < L.total) return fail(ctx, SJA_ERR_WORKSPACE, "workspace too small");

    DeviceGuard guard(ctx->device);
    SJA_HIP(guard.err, "hipSetDevice");
    hipStream_t st = static_cast<hipStream_t>(stream);
    // the profiles of the granted jobs change: whatever the last fit left no longer describes them
    ctx->fitted = false;
    ctx->planned = false;
    unsigned long long *m = reinterpret_cast<unsigned long long *>(metrics);
    hipLaunchKernelGGL(k_fill_i64, dim3(1), dim3(64), 0, st, 4, int64_t(0), metrics);
    SJA_HIP(hipGetLastError(), "k_fill_i64 launch");
    if (n_gaps > 0) {
        hipLaunchKernelGGL(k_advance_gaps, dim3((n_gaps + 255) / 256), dim3(256), 0, st, n_gaps, J, ctx->seg_off,
                           ctx->pre_dur, ctx->pre_peak, W, C, grant_job, grant_cut, job_gap, progress, m);
        SJA_HIP(hipGetLastError(), "k_advance_gaps launch");
    }
    if (J > 0) {
        const int jobs_per_block = 256 / kWave;
        const dim3 grid((J + jobs_per_block - 1) / jobs_per_block), block(256);
        const bool by_area = ctx->score_used == SJA_SCORE_AREA;
        const Hysteresis hyst = hysteresis_of(ctx->hyst_used_n_caps, ctx->hyst_used_min_gain, ctx->hyst_used_cap);
        long long *pre_area = by_area ? ws_ptr<long long>(ctx, L.pre_area) : nullptr;
        long long *atom_area = by_area || hyst.n_caps > 0 ? ws_ptr<long long>(ctx, L.atom_area) : nullptr;
        if (ctx->limits_used) {
            const JobLimits lim = job_limits(ctx->limits_applied, ctx->used_power, ctx->used_deadline);
            hipLaunchKernelGGL(k_advance_jobs<true>, grid, block, 0, st, lim, hyst, pre_area, atom_area, n_gaps, J, ctx->seg_off, ctx->dur,
                               ctx->mem, ctx->safe, grant_job, grant_cut, job_gap, progress, wait, wait_step,
                               ctx->pre_dur, ctx->pre_peak, ctx->prev_safe, ws_ptr<int2>(ctx, L.atom_dp),
                               ws_ptr<int2>(ctx, L.atom_db), ws_ptr<int32_t>(ctx, L.n_atoms),
                               ws_ptr<int2>(ctx, L.first_dp), m);
        } else {
            hipLaunchKernelGGL(k_advance_jobs<false>, grid, block, 0, st, JobLimits{}, hyst, pre_area, atom_area, n_gaps, J, ctx->seg_off,
                               ctx->dur, ctx->mem, ctx->safe, grant_job, grant_cut, job_gap, progress, wait,
                               wait_step, ctx->pre_dur, ctx->pre_peak, ctx->prev_safe,
                               ws_ptr<int2>(ctx, L.atom_dp), ws_ptr<int2>(ctx, L.atom_db),
                               ws_ptr<int32_t>(ctx, L.n_atoms), ws_ptr<int2>(ctx, L.first_dp), m);
        }
        SJA_HIP(hipGetLastError(), "k_advance_jobs launch");
    }
    return SJA_OK;
}

int sja_cover(sja_ctx *ctx, void *stream, int32_t n_gaps, const int32_t *C, const int32_t *grant_job,
              const int32_t *grant_cut, int32_t n_caps, const int32_t *cap_set, int32_t *cover, int32_t *slack)
{
    if (!ctx) return SJA_ERR_NULL;
    if (!ctx->prepared) return fail(ctx, SJA_ERR_STATE, "sja_cover before sja_prepare_profiles");
    if (n_gaps < 0 || n_gaps > SJA_MAX_GAPS) return fail(ctx, SJA_ERR_SIZE, "n_gaps");
    if (n_caps < 0) return fail(ctx, SJA_ERR_SIZE, "n_caps");
    if (n_gaps > 0 && (!C || !grant_job || !grant_cut || !cover || !slack)) return fail(ctx, SJA_ERR_NULL, "gap arrays");
    if (n_caps > 0 && !cap_set) return fail(ctx, SJA_ERR_NULL, "cap_set");
    DeviceGuard guard(ctx->device);
    SJA_HIP(guard.err, "hipSetDevice");
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (n_gaps > 0) {
        hipLaunchKernelGGL(k_cover, dim3((n_gaps + 255) / 256), dim3(256), 0, st, n_gaps, ctx->n_jobs, ctx->seg_off,
                           ctx->pre_peak, C, grant_job, grant_cut, n_caps, cap_set, cover, slack);
        SJA_HIP(hipGetLastError(), "k_cover launch");
    }
    return SJA_OK;
}

}  // extern "C"
