// Mixing diagnostic (Sec. 6.1): host side of gesmc_mixing.  Part of the
// library's translation unit (included by gesmc.hip after its entry points).
#pragma once

namespace {

constexpr uint32_t kMixMaxN = 1u << 14;  // pair ids below 2^27

// The diagnostic's device block.  After a call that finished (its stream is
// idle then) the context keeps a block of up to kMixKeepBytes for its next
// diagnostic, instead of gigabytes mapped and unmapped on each call: the
// driver clears freed memory before it maps it again, and calls that follow
// each other sooner than that wait.  n = 2^13, seven thinnings (2.9 GB), 400
// calls in a row, ms at the median and the 90th percentile: K = 200 21.9 and
// 163 without, 21.2 and 21.2 with it; K = 20 3.95 and 225, 3.27 and 3.30.
// It is returned with the context, for a larger block, as soon as another
// allocation of the context finds no memory, or by gesmc_set_allocator.  A block
// of the caller's allocator goes back with the call: it is there to be shared,
// and keeps what it gets itself.
constexpr uint64_t kMixKeepBytes = 4ull << 30;

struct MixBlock {
    gesmc_ctx *c;
    unsigned char *p = nullptr;
    uint64_t bytes = 0;

    gesmc_status take(uint64_t want) {
        if (c->mix_bytes < want) release_mix_block(c);
        bytes = want;
        if (!c->mix_blk) return dev_alloc(c, (void **)&p, want);
        p = c->mix_blk;
        bytes = c->mix_bytes;
        c->mix_blk = nullptr;
        c->mix_bytes = 0;
        return GESMC_OK;
    }
    void keep() {
        if (bytes > kMixKeepBytes || c->alloc_fn) return;
        c->mix_blk = p;
        c->mix_bytes = bytes;
        p = nullptr;
    }
    ~MixBlock() {
        if (p) dev_free(c, p);
    }
};

// The G-ES-MC chain of a diagnostic on the multi-kernel supersteps: the state
// stays in its records (buffer 0) between supersteps, whose order no sample
// depends on, and the host waits once per kMixPiece supersteps instead of
// loading, writing back and waiting for each (n = 2^13, m = 1.1e4, per
// superstep with its samples: 232 -> 200 us).
constexpr uint32_t kMixPiece = 64;

struct MixChain {
    Plan p;
    uint32_t m, n, k0, k1, pl, K, piece0;
    bool ahead;
    Level1 level1;
};

gesmc_status mix_chain_open(gesmc_ctx *c, hipStream_t s, MixChain *q, const unsigned long long *E) {
    GESMC_TRY(ensure_capacity(c, q->m, true));
    GESMC_TRY(ensure_counters(c, kMixPiece));
    q->p = perm_plan(c, q->m);
    q->p.dig_in_key = digit_in_key(q->p, q->n);
    q->ahead = GESMC_COUNT_AHEAD && q->p.bbits > 0 && q->p.b1 > 0 && q->p.ell > 0;
    q->piece0 = 0;
    GESMC_TRY(launch(c, s, KID_MISC, 0, k_zero_words, dim3(4), dim3(256), 0, c->err, (uint64_t)64));
    return launch(c, s, KID_LOAD, q->m, k_load, dim3(grid_stride_blocks(c, q->m)), dim3(kBlock), 0, E, q->m, q->n,
                  c->idx[0], c->key[0], c->err, 0u);
}

// Superstep t (in order from 0); after a piece's last one, waits and checks.
gesmc_status mix_chain_step(gesmc_ctx *c, hipStream_t s, MixChain *q, uint32_t t) {
    const uint32_t k = t - q->piece0;
    if (k == 0)
        GESMC_TRY(launch(c, s, KID_MISC, 0, k_zero_words, dim3(4), dim3(256), 0, (uint32_t *)c->ctr,
                         (uint64_t)kMixPiece * (sizeof(StepCounters) / 4)));
    c->ctr_step = c->ctr + k;
    GESMC_TRY(superstep_partitioned(c, s, q->p, t, q->k0, q->k1, q->pl, t == 0 ? ERR_DUP : ERR_INTERNAL, nullptr,
                                    q->n, 0, q->ahead && t + 1 < q->K, &q->level1));
    if (k + 1 < kMixPiece && t + 1 < q->K) return GESMC_OK;
    GESMC_TRY(check_hip(hipMemcpyAsync(c->h_err, c->err, 4, hipMemcpyDeviceToHost, s), "hipMemcpyAsync"));
    GESMC_TRY(check_hip(hipMemcpyAsync(c->h_ctr, c->ctr, sizeof(StepCounters) * (k + 1), hipMemcpyDeviceToHost, s),
                        "hipMemcpyAsync"));
    GESMC_TRY(check_hip(hipStreamSynchronize(s), "hipStreamSynchronize"));
    if (c->profile) collect_profile(c);
    GESMC_TRY(map_err(*c->h_err));
    adapt_decision_rounds(c, k + 1);
    q->piece0 = t + 1;
    return GESMC_OK;
}

gesmc_status mixing_impl(gesmc_ctx *c, void *stream, const uint64_t *d_in, uint64_t m64, uint32_t n, uint64_t seed,
                         uint32_t chain, uint32_t pl, uint32_t K, const uint32_t *thin, uint32_t nthin,
                         gesmc_mixing_result *out, double *ms_total) {
    if (!c || !thin || !out || (m64 > 0 && !d_in)) {
        set_error("null argument");
        return GESMC_E_INVAL;
    }
    if (chain > 1 || nthin == 0 || nthin > kMixMaxThin) {
        set_error("chain must be 0 or 1 and 1 <= nthin <= %u", kMixMaxThin);
        return GESMC_E_INVAL;
    }
    for (uint32_t q = 0; q < nthin; ++q)
        if (thin[q] == 0) {
            set_error("thinning values must be at least 1");
            return GESMC_E_INVAL;
        }
    if (n < 2 || n > kMixMaxN || m64 >= kMaxEdges) {
        set_error("the mixing diagnostic needs 2 <= n <= %u (dense pair counters) and m < 2^30", kMixMaxN);
        return GESMC_E_RANGE;
    }
    if (chain == 0 && (uint64_t)K > 0x100000000ull) {
        set_error("K exceeds the 32-bit superstep counter");
        return GESMC_E_INVAL;
    }
    GESMC_TRY(check_hip(hipSetDevice(c->device), "hipSetDevice"));
    hipStream_t s = (hipStream_t)stream;
    const uint32_t m = (uint32_t)m64, ell = m / 2;
    const uint64_t npairs = (uint64_t)n * (n - 1) / 2, words = (npairs + 31) / 32;
    // one block: the state, the current-sample bitmaps, the results, and per
    // thinning value the previous sample's list and bitmap, the tracked bitmap
    // and the counters, each on 256 bytes
    const uint64_t mm = std::max<uint32_t>(m, 1);
    auto pad = [](uint64_t b) { return (b + 255) & ~255ull; };
    const uint64_t lists = pad(mm * 8) + 2 * pad(words * 4);
    const uint64_t bytes = lists + pad(64) + nthin * (lists + pad(npairs * sizeof(MixCount)));
    MixBlock block{c};
    GESMC_TRY(block.take(bytes));
    unsigned char *const blk = block.p;
    uint64_t off = 0;
    auto take = [&](uint64_t b) {
        unsigned char *p = blk + off;
        off += pad(b);
        return p;
    };
    auto *E = (unsigned long long *)take(mm * 8);
    uint32_t *cur_bits[2] = {(uint32_t *)take(words * 4), (uint32_t *)take(words * 4)};
    auto *res = (unsigned long long *)take(64);
    std::vector<unsigned long long *> prev(nthin);
    std::vector<uint32_t *> prev_bits(nthin), ever(nthin);
    std::vector<MixCount *> cnt(nthin);
    for (uint32_t q = 0; q < nthin; ++q) {
        prev[q] = (unsigned long long *)take(mm * 8);
        prev_bits[q] = (uint32_t *)take(words * 4);
        ever[q] = (uint32_t *)take(words * 4);
        cnt[q] = (MixCount *)take(npairs * sizeof(MixCount));
    }
    GESMC_TRY(check_hip(hipMemsetAsync(blk, 0, bytes, s), "hipMemsetAsync"));
    // X_0: the input validated and canonicalised (a call with no superstep)
    GESMC_TRY(run_impl(c, stream, d_in, (uint64_t *)E, m, n, seed, 0, 0, pl, nullptr, nullptr, nullptr));
    const uint32_t gb = grid_stride_blocks(c, m);
    for (uint32_t q = 0; q < nthin && m > 0; ++q) {
        GESMC_TRY(launch(c, s, KID_MIX, m, k_mix_bits, dim3(gb), dim3(kBlock), 0, (const unsigned long long *)E, m, n,
                         prev_bits[q]));
        GESMC_TRY(launch(c, s, KID_MIX, m, k_mix_bits, dim3(gb), dim3(kBlock), 0, (const unsigned long long *)E, m, n,
                         ever[q]));
        GESMC_TRY(check_hip(hipMemcpyAsync(prev[q], E, m * 8ull, hipMemcpyDeviceToDevice, s), "hipMemcpyAsync"));
    }
    auto t_start = std::chrono::steady_clock::now();
    // small graphs run a superstep in one workgroup's LDS (run_impl)
    const bool resident = chain == 0 && c->strategy == 0 && m >= 2 &&
                          !(c->small_graphs && (m <= kMidMax || (m <= kCmpMax && n <= kCmpMaxN)));
    MixChain mc{Plan{}, m, n, (uint32_t)seed, (uint32_t)(seed >> 32), pl, K, 0, false, kLevel1Todo};
    if (resident && K > 0) GESMC_TRY(mix_chain_open(c, s, &mc, (const unsigned long long *)E));
    const unsigned long long *last = nullptr;  // a series' list of the sample before
    uint32_t nsample = 0;
    for (uint32_t t = 0; t < K; ++t) {
        if (resident) {
            GESMC_TRY(mix_chain_step(c, s, &mc, t));
        } else if (m >= 2) {
            if (chain == 0)
                GESMC_TRY(run_impl(c, stream, (const uint64_t *)E, (uint64_t *)E, m, n, seed, t, 1, pl, nullptr,
                                   nullptr, nullptr));
            else
                GESMC_TRY(run_es_impl(c, stream, (const uint64_t *)E, (uint64_t *)E, m, n, seed, (uint64_t)t * ell,
                                      ell, nullptr, nullptr));
        }
        const uint32_t tt = t + 1;
        MixSeries due;
        uint32_t ndue = 0;
        for (uint32_t q = 0; q < nthin; ++q) {
            if (tt % thin[q]) continue;
            due.prev[ndue] = prev[q];
            due.prev_bits[ndue] = prev_bits[q];
            due.ever[ndue] = ever[q];
            due.cnt[ndue] = cnt[q];
            ++ndue;
        }
        if (ndue == 0 || m == 0) continue;
        const unsigned long long *now = resident ? (const unsigned long long *)c->key[0] : E;
        uint32_t *bits = cur_bits[nsample & 1u];
        GESMC_TRY(launch(c, s, KID_MIX, m, k_mix_mark, dim3(gb), dim3(kBlock), 0, now, last, m, n, bits,
                         cur_bits[1u - (nsample & 1u)]));
        GESMC_TRY(launch(c, s, KID_MIX, (uint64_t)m * ndue, k_mix_sample, dim3(gb, ndue), dim3(kBlock), 0, now, m, n,
                         (const uint32_t *)bits, due));
        last = due.prev[0];  // holds this sample until its series is due again
        ++nsample;
    }
    for (uint32_t q = 0; q < nthin; ++q) {
        const uint32_t N = K / thin[q];
        unsigned long long h[6] = {0, 0, 0, 0, 0, 0};
        GESMC_TRY(check_hip(hipMemsetAsync(res, 0, 64, s), "hipMemsetAsync"));
        GESMC_TRY(launch(c, s, KID_MIX, npairs, k_mix_decide, dim3(grid_stride_blocks(c, npairs)), dim3(kBlock), 0,
                         (const MixCount *)cnt[q], (const uint32_t *)ever[q], npairs, N, res));
        GESMC_TRY(check_hip(hipMemcpyAsync(h, res, sizeof(h), hipMemcpyDeviceToHost, s), "hipMemcpyAsync"));
        GESMC_TRY(check_hip(hipStreamSynchronize(s), "hipStreamSynchronize"));
        gesmc_mixing_result &o = out[q];
        memset(&o, 0, sizeof(o));
        o.k = thin[q];
        o.transitions = N;
        o.tracked = h[0];
        o.non_independent = N > 0 ? h[1] : 0;
        o.n01 = h[2];
        o.n10 = h[3];
        o.n11 = h[4];
        o.n00 = (uint64_t)N * h[0] - h[2] - h[3] - h[4];
    }
    GESMC_TRY(check_hip(hipStreamSynchronize(s), "hipStreamSynchronize"));
    if (ms_total)
        *ms_total = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t_start).count();
    if (c->profile) collect_profile(c);
    block.keep();
    return GESMC_OK;
}

}  // namespace

extern "C" {

gesmc_status gesmc_mixing(gesmc_ctx *ctx, void *stream, const uint64_t *d_in, uint64_t m, uint32_t n, uint64_t seed,
                          uint32_t chain, uint32_t pl, uint32_t K, const uint32_t *thin, uint32_t nthin,
                          gesmc_mixing_result *out, double *ms_chain) {
    return mixing_impl(ctx, stream, d_in, m, n, seed, chain, pl, K, thin, nthin, out, ms_chain);
}

}  // extern "C"
