// ParES (Alg. 2): host side of gesmc_run_es and gesmc_es_draws.  Part of the
// library's translation unit (included by gesmc.hip after its entry points).
#pragma once

namespace {

// Switches per launch of k_es_chain (an epoch): the edge set is rebuilt
// between epochs, so that its used slots (live edges plus retired ones) stay
// below m + 2 * epoch, and its slot count (a power of two at least twice
// that) keeps the load at or below one half.
uint64_t es_epoch(uint32_t m) { return std::max<uint64_t>(m / 2, 65536); }

uint64_t es_slots(uint32_t m) {
    const uint64_t want = 2 * ((uint64_t)m + 2 * es_epoch(m));
    uint64_t T = 1024;
    while (T < want) T <<= 1;
    return T;
}

// Switches per window and passes over it; 0 switches (the chain on one
// workgroup) below kEsWindowEdges edges, where a window's launches cost more
// than the supersteps they replace.  Small graphs are bound by the launches, so
// their windows take a larger share of m and the more passes that share needs.
// Where the two shares cross depends on how many switches a pass changes.  us per
// m / 2 switches at m / 8 with 10 passes and m / 4 with 16: sparse G(n, p) m =
// 3.0e5 663 and 514, 1.0e6 943 and 814, 1.3e6 1011 and 927, 2.0e6 1326 and 1318;
// gamma = 2.05 and 2.01 2.7e5 1312 and 1540, 9.7e5 1903 and 2361, 1.3e6 2261 and
// 2889; G(n, 0.9) 5.4e5 1319 and 1495.  The line lies between the two.
constexpr uint32_t kEsWindowEdges = 4096;
constexpr uint32_t kEsSmallEdges = 1u << 20;
// At most 2^19 switches: the event lists and keys of a window then still sit
// in L2 and MALL (m = 6.7e6, ms per call at 2^17, 2^18, 2^19: 5.2, 4.3, 4.0).
constexpr uint32_t kEsWindowMax = 1u << 19;
uint32_t es_window(uint32_t m) {
    if (m < kEsWindowEdges) return 0;
    return std::min<uint32_t>(m < kEsSmallEdges ? m / 4 : m / 8, kEsWindowMax);
}
uint32_t es_passes(uint32_t m) { return m < kEsSmallEdges ? kEsPasses : 10u; }
// Nodes of an event list that a judgement walks before its window is given up.
// A walk is a chain of reads of 0.17 to 0.28 us a node and is repeated in seven
// passes or more, while the window (m / 4 switches) takes 4 sqrt(m) us on the
// chain: the two meet at about 2 sqrt(m) nodes.  Two stars of m / 2 edges each,
// lists of m / 16, us per m / 2 switches on the chain, with lists of any length
// below 4096, with this line: m = 8,192 870, 1542, 1041; 65,536 3429, 40116, 3803.
// Power laws down to gamma = 2.01 stay below it but for one window in 16 at n =
// 20,000.
uint32_t es_walk(uint32_t m) { return std::min<uint32_t>((uint32_t)(2.0 * std::sqrt((double)m)), 4096u); }
// Fewer switches than this (a short call, the rest of an epoch) go to the chain
// on one workgroup: it takes about 16 / sqrt(m) us a switch, and 0.055 to 0.033
// from m = 1.7e5 on, where its supersteps reach their 1024 switches and wait for
// HBM; a window's launches take 90 to 135 us whatever it holds.  Calls cross, in
// switches: m = 4,096 700 (r = 600: 181 us on the chain, 194 as a window; 1000:
// 262, 206), 16,384 1,250 (1000: 167, 208; 2000: 299, 202), 110,000 2,100 (2000:
// 198, 207; 3000: 261, 200), 1.0e6 3,500 (3000: 223, 249; 5000: 300, 241), 6.7e6
// 3,100 (3000: 547, 556; 5000: 616, 554).
uint32_t es_chain_below(uint32_t m) {
    return std::min<uint32_t>((uint32_t)(10.0 * std::sqrt((double)m)), m < 1u << 18 ? 2048u : 3072u);
}

// The window's arrays in one buffer (130 to 160 bytes a switch, and a word per edge).
gesmc_status es_ensure_window(gesmc_ctx *c, uint32_t m, uint32_t W, EsWindow *out) {
    uint32_t cells = 1024;
    while (cells < 4 * W) cells <<= 1;
    const uint64_t w = W;
    const uint64_t sizes[] = {w * 8,  w * 8,  w * 8,           w * 16, w * 16,     w * 2,
                              w,      cells * 4ull, w * 32, w * 16, kEsCtl * 4ull, cells / 8 * (kEsPasses - 1ull), 8ull, m * 4ull};
    uint64_t total = 0;
    for (uint64_t b : sizes) total += (b + 255) & ~255ull;
    if (total > c->es_cap_w) {
        if (c->es_win) dev_free(c, c->es_win);
        c->es_win = nullptr;
        c->es_cap_w = 0;
        GESMC_TRY(dev_alloc(c, (void **)&c->es_win, total));
        c->es_cap_w = total;
    }
    unsigned char *p = c->es_win;
    int k = 0;
    auto take = [&]() {
        unsigned char *q = p;
        p += (sizes[k++] + 255) & ~255ull;
        return q;
    };
    out->ij = (uint2 *)take();
    out->ulink = (uint32_t *)take();
    out->pred = (uint32_t *)take();
    out->src = (unsigned long long *)take();
    out->tgt = (unsigned long long *)take();
    out->pres = (uint8_t *)take();
    out->st = (uint8_t *)take();
    out->cell = (uint32_t *)take();
    out->link = (uint32_t *)take();
    out->pool = (uint32_t *)take();
    out->ctl = (uint32_t *)take();
    out->touched = (uint32_t *)take();
    out->gate = (uint32_t *)take();
    out->last = (uint32_t *)take();
    out->cap = W;
    out->cmask = cells - 1;
    out->passes = es_passes(m);
    out->walk = es_walk(m);
    return GESMC_OK;
}

constexpr size_t kEsCtrBytes = kEsCtrCopies * sizeof(EsCounters);

gesmc_status es_ensure(gesmc_ctx *c, uint32_t m) {
    const uint64_t cap = std::max<uint64_t>(m, 1024), T = es_slots(m);
    if (!c->es_ctr) {
        GESMC_TRY(dev_alloc(c, (void **)&c->es_ctr, kEsCtrBytes));
        if (hipHostMalloc((void **)&c->h_es_ctr, kEsCtrBytes, hipHostMallocDefault) != hipSuccess) {
            (void)hipGetLastError();
            c->h_es_ctr = nullptr;
            set_error("hipHostMalloc failed");
            return GESMC_E_NOMEM;
        }
    }
    if (cap > c->es_cap_m) {
        for (void **q : {(void **)&c->es_E, (void **)&c->es_slot}) {
            if (*q) dev_free(c, *q);
            *q = nullptr;
        }
        c->es_cap_m = 0;
        GESMC_TRY(dev_alloc(c, (void **)&c->es_E, cap * 8));
        GESMC_TRY(dev_alloc(c, (void **)&c->es_slot, cap * 4));
        c->es_cap_m = cap;
    }
    if (T > c->es_cap_T) {
        if (c->es_H) dev_free(c, c->es_H);
        c->es_H = nullptr;
        c->es_cap_T = 0;
        GESMC_TRY(dev_alloc(c, (void **)&c->es_H, T * 8));
        c->es_cap_T = T;
    }
    return GESMC_OK;
}

gesmc_status run_es_impl(gesmc_ctx *c, void *stream, const uint64_t *d_in, uint64_t *d_out, uint64_t m64, uint32_t n,
                         uint64_t seed, uint64_t k0, uint64_t r, uint8_t *d_outcome, gesmc_es_stats *stats) {
    if (!c) {
        set_error("null context");
        return GESMC_E_INVAL;
    }
    if (m64 > 0 && (!d_in || !d_out)) {
        set_error("null edge pointer");
        return GESMC_E_INVAL;
    }
    if (m64 >= kMaxEdges) {
        set_error("m = %llu exceeds the limit 2^30 - 1", (unsigned long long)m64);
        return GESMC_E_RANGE;
    }
    if (r > ~0ull - k0) {
        set_error("switch counter k0 + r overflows 64 bits");
        return GESMC_E_INVAL;
    }
    GESMC_TRY(check_hip(hipSetDevice(c->device), "hipSetDevice"));
    hipStream_t s = (hipStream_t)stream;
    const uint32_t m = (uint32_t)m64;
    GESMC_TRY(es_ensure(c, m));
    const uint32_t W = es_window(m), below = es_chain_below(m);
    bool windows = W > 0 && r >= below;
    EsWindow win{};
    if (windows) {
        const gesmc_status st = es_ensure_window(c, m, W, &win);
        if (st == GESMC_E_NOMEM)
            windows = false;  // the chain on one workgroup needs no more than the edge set
        else
            GESMC_TRY(st);
    }
    const uint64_t T = es_slots(m), epoch = es_epoch(m);
    const uint32_t mask = (uint32_t)(T - 1);
    const uint32_t s0 = (uint32_t)seed, s1 = (uint32_t)(seed >> 32);
    GESMC_TRY(check_hip(hipEventRecord(c->call_a, s), "hipEventRecord"));
    GESMC_TRY(launch(c, s, KID_MISC, 0, k_zero_words, dim3(4), dim3(256), 0, c->err, (uint64_t)64));
    GESMC_TRY(launch(c, s, KID_MISC, 0, k_zero_words, dim3(2), dim3(256), 0, (uint32_t *)c->es_ctr,
                     (uint64_t)(kEsCtrBytes / 4)));
    if (m > 0)
        GESMC_TRY(launch(c, s, KID_LOAD, m, k_load, dim3(grid_stride_blocks(c, m)), dim3(kBlock), 0,
                         (const unsigned long long *)d_in, m, n, c->es_slot, c->es_E, c->err, 0u));
    uint64_t launches = 0;
    if (windows) GESMC_TRY(launch(c, s, KID_MISC, 0, k_zero_words, dim3(1), dim3(64), 0, win.gate, (uint64_t)2));
    if (m >= 2) {
        for (uint64_t kb = k0; kb == k0 || kb - k0 < r; kb += epoch) {
            const uint64_t ke = kb + std::min<uint64_t>(epoch, r - (kb - k0));
            // (re)build the edge set from the edge list: all slots live, none retired
            GESMC_TRY(launch(c, s, KID_ES_BUILD, T, k_es_clear, dim3(grid_stride_blocks(c, T)), dim3(kBlock), 0,
                             c->es_H, T));
            GESMC_TRY(launch(c, s, KID_ES_BUILD, m, k_es_insert_all, dim3(grid_stride_blocks(c, m)), dim3(kBlock),
                             0, (const unsigned long long *)c->es_E, m, c->es_H, mask, c->es_slot, c->err));
            if (windows && ke - kb >= below)  // uses of earlier epochs must read as none
                GESMC_TRY(launch(c, s, KID_MISC, 0, k_zero_words, dim3(grid_stride_blocks(c, m)), dim3(kBlock), 0,
                                 win.last, (uint64_t)m));
            uint32_t tag = 1;  // of the window's uses: 2 W a window, below 2 (epoch + W) in an epoch
            // (by offset: a counter near 2^64 must not wrap past the epoch's end)
            for (uint64_t o = 0; o < ke - kb;) {
                const uint64_t wb = kb + o, rest = ke - wb;
                if (!windows || rest < below) {
                    GESMC_TRY(launch(c, s, KID_ES_CHAIN, rest, k_es_chain, dim3(1), dim3(kEsThreads), 0, c->es_E,
                                     c->es_slot, c->es_H, mask, m, s0, s1, wb, ke, k0, d_outcome, c->es_ctr, c->err,
                                     (const uint32_t *)nullptr, (uint32_t *)nullptr));
                    break;
                }
                const uint32_t nw = (uint32_t)std::min<uint64_t>(W, rest);
                const dim3 grid(ceil_div(nw, kBlock)), block(kBlock);
                GESMC_TRY(launch(c, s, KID_ES_CHAIN, nw, k_es_win_draw, grid, block, 0, win, nw, wb, m, s0, s1,
                                 tag));
                GESMC_TRY(launch(c, s, KID_ES_CHAIN, 0, k_es_win_link, grid, block, 0, win, nw, tag,
                                 (const unsigned long long *)c->es_E, (const unsigned long long *)c->es_H, mask,
                                 c->err));
                for (uint32_t t = 0; t < win.passes; ++t) {
                    GESMC_TRY(launch(c, s, KID_ES_CHAIN, 0, k_es_win_sources, grid, block, 0, win, nw, t,
                                     (const unsigned long long *)c->es_H, mask, c->err));
                    GESMC_TRY(launch(c, s, KID_ES_CHAIN, 0, k_es_win_decide, grid, block, 0, win, nw, t,
                                     (const uint32_t *)c->err));
                }
                GESMC_TRY(launch(c, s, KID_ES_CHAIN, 0, k_es_win_commit, grid, block, 0, win, nw, c->es_E,
                                 c->es_slot, c->es_H, mask, d_outcome ? d_outcome + (wb - k0) : nullptr, c->es_ctr,
                                 c->err));
                GESMC_TRY(launch(c, s, KID_ES_CHAIN, 0, k_es_chain, dim3(1), dim3(kEsThreads), 0, c->es_E,
                                 c->es_slot, c->es_H, mask, m, s0, s1, wb, wb + nw, k0, d_outcome, c->es_ctr, c->err,
                                 (const uint32_t *)(win.ctl + win.passes), win.gate));
                tag += 2 * W;
                o += nw;
            }
            ++launches;
            if (ke - k0 >= r) break;
        }
    }
    if (m > 0)
        GESMC_TRY(launch(c, s, KID_UNPERMUTE, m, k_es_out, dim3(grid_stride_blocks(c, m)), dim3(kBlock), 0,
                         (const unsigned long long *)c->es_E, m, (unsigned long long *)d_out,
                         (const uint32_t *)c->err));
    GESMC_TRY(check_hip(hipEventRecord(c->call_b, s), "hipEventRecord"));
    GESMC_TRY(check_hip(hipMemcpyAsync(c->h_err, c->err, 4, hipMemcpyDeviceToHost, s), "hipMemcpyAsync"));
    GESMC_TRY(check_hip(hipMemcpyAsync(c->h_es_ctr, c->es_ctr, kEsCtrBytes, hipMemcpyDeviceToHost, s),
                        "hipMemcpyAsync"));
    GESMC_TRY(check_hip(hipStreamSynchronize(s), "hipStreamSynchronize"));
    if (c->profile) collect_profile(c);
    GESMC_TRY(map_err(*c->h_err));
    if (stats) {
        EsCounters h = c->h_es_ctr[0];
        for (uint32_t q = 1; q < kEsCtrCopies; ++q) {
            const EsCounters &o = c->h_es_ctr[q];
            h.legal += o.legal;
            h.rej_loop += o.rej_loop;
            h.rej_exists += o.rej_exists;
            h.supersteps += o.supersteps;
            h.rounds += o.rounds;
            h.rounds_max = std::max(h.rounds_max, o.rounds_max);
        }
        memset(stats, 0, sizeof(*stats));
        stats->attempts = m >= 2 ? r : 0;
        stats->legal = h.legal;
        stats->rej_loop = h.rej_loop;
        stats->rej_exists = h.rej_exists;
        stats->supersteps = h.supersteps;
        stats->rounds_sum = h.rounds;
        stats->rounds_max = (uint32_t)h.rounds_max;
        stats->epochs = (uint32_t)launches;
        float ms = 0.f;
        if (hipEventElapsedTime(&ms, c->call_a, c->call_b) == hipSuccess)
            stats->ms_device = ms;
        else
            (void)hipGetLastError();
    }
    return GESMC_OK;
}

}  // namespace

extern "C" {

gesmc_status gesmc_run_es(gesmc_ctx *ctx, void *stream, const uint64_t *d_in, uint64_t *d_out, uint64_t m, uint32_t n,
                          uint64_t seed, uint64_t k0, uint64_t r, uint32_t flags, uint8_t *d_outcome,
                          gesmc_es_stats *stats) {
    if (flags != 0) {
        set_error("flags must be 0");
        return GESMC_E_INVAL;
    }
    return run_es_impl(ctx, stream, d_in, d_out, m, n, seed, k0, r, d_outcome, stats);
}

gesmc_status gesmc_es_draws(gesmc_ctx *c, void *stream, uint64_t m, uint64_t seed, uint64_t k0, uint64_t count,
                            uint64_t *d_i, uint64_t *d_j, uint8_t *d_g) {
    if (!c || (count > 0 && (!d_i || !d_j || !d_g))) {
        set_error("null argument");
        return GESMC_E_INVAL;
    }
    if (m < 2 || m >= kMaxEdges) {
        set_error("m = %llu: draws need 2 <= m < 2^30", (unsigned long long)m);
        return GESMC_E_RANGE;
    }
    if (count > ~0ull - k0) {
        set_error("switch counter k0 + count overflows 64 bits");
        return GESMC_E_INVAL;
    }
    GESMC_TRY(check_hip(hipSetDevice(c->device), "hipSetDevice"));
    hipStream_t s = (hipStream_t)stream;
    if (count > 0)
        GESMC_TRY(launch(c, s, KID_MISC, count, k_es_draws, dim3(grid_stride_blocks(c, count)), dim3(kBlock), 0, k0,
                         count, (uint32_t)m, (uint32_t)seed, (uint32_t)(seed >> 32), (unsigned long long *)d_i,
                         (unsigned long long *)d_j, d_g));
    GESMC_TRY(check_hip(hipStreamSynchronize(s), "hipStreamSynchronize"));
    if (c->profile) collect_profile(c);
    return GESMC_OK;
}

}  // extern "C"
