// mtpt_lists.h -- neighbour lists of the 3-d FP64 passes (included by
// mtpt_device.h).
//
// The mask variant of the tiled passes records, per plane of candidate rows,
// which candidates are neighbours; the row-sum pass then sums the kernel plane
// by plane and the transfer pass decodes the bits again: three loops each, as
// long as the wave's largest count in that plane (19 iterations a particle on
// the reacting workload, of 5.9 neighbours), with the software FP64
// exponential (about 25 instructions) in both and a division in the second.
// The list variant has one loop of 13 in each: the row-sum pass appends the
// LDS offset of every candidate within the cutoff to its lane's list in LDS,
// sums the kernel over that one list, and packs it for the transfer pass,
// whose neighbours' slots take two instructions to unpack instead of ten.
// For that both passes stage the same tiles in the same order, in workgroups
// of kListBlock threads (two per CU by LDS).  Both passes are bound by VALU
// issue and by the latency of their setup.  Reacting workload, row-sum and
// transfer launch, mask and list variant: 1e6 particles 126 -> 92 and 98 -> 85
// us, 8e6 817 -> 654 and 724 -> 677 us, 1e5 36 -> 25 and 22 -> 23 us.
// The FP32 passes gain nothing from it: their exponential is one instruction,
// so the second loop costs the row-sum pass what the lists save (3.2e7
// particles 1.40 -> 1.70 ms), and the transfer pass, with a third fewer
// instructions, still waits for its setup (2.11 -> 2.02 ms at best).
//
// A list holds the particle itself (its visit adds exactly zero in the
// transfer pass) and is in candidate order, so every sum is that of the mask
// variant bit for bit.  Packed: word 0 holds the count (6 bits) and two slots,
// the others three slots, each of 10 bits relative to the particle's first
// candidate row; words 0..5 are the masks' memory, word 6 is the permutation
// of the binning, free between the place pass and the next scatter.  A
// particle with more neighbours, or slots further apart, has the count
// kListNone, and the transfer pass scans its rows.  That is slower than the
// masks, so the host keeps the lists to sims with few such particles.
#pragma once

namespace mtpt {

__device__ __forceinline__ uint32_t* list_word(const SimArgs& a, int w)
{
    return w < kListWords - 1 ? reinterpret_cast<uint32_t*>(a.cmask) + static_cast<size_t>(w) * static_cast<size_t>(a.n)
                              : a.perm;
}

// A list tile is one tile of the mask variant's transfer pass, or two of them
// side by side (a.lsplit: the axis, kListWhole: one), and leaves their partial
// sums: the totals of a sim are then the same bit for bit whichever variant it
// takes, alone or in a pool.  The mask variant sums a tile by thread (particles
// v, v + kBlock, .. in the tile's order), by wave and over its kBlock / 64
// waves; here each half of the workgroup sums one transfer tile in that order,
// the masses handed over through LDS, or, of a tile of more particles than the
// workgroup has threads, read back.
// The sums of a transfer tile's kBlock threads (sum) to its place in a.partials.
template <int NS>
__device__ __forceinline__ void list_totals(const SimArgs& a, bool upper, const int* sub, const double* sum)
{
    constexpr int kWaves = kBlock / 64;
    __shared__ double red[NS][kListBlock / 64];
    const int tid = threadIdx.x;
#pragma unroll
    for (int c = 0; c < NS; ++c) {
        double x = sum[c];
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1)
            x += __shfl_down(x, off, 64);
        if ((tid & 63) == 0)
            red[c][tid >> 6] = x;
    }
    __syncthreads();
    // (the second tile may lie past the grid's edge)
    if (tid % kBlock != 0 || (upper && a.lsplit == kListWhole) || sub[0] * a.ttile[0] >= a.nc[0] ||
        sub[1] * a.ttile[1] >= a.nc[1] || sub[2] * a.ttile[2] >= a.nc[2])
        return;
    const size_t s = (static_cast<size_t>(sub[2]) * a.ttiles_y + sub[1]) * a.ttiles_x + sub[0];
#pragma unroll
    for (int c = 0; c < NS; ++c) {
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w)
            t += red[c][(upper ? kWaves : 0) + w];
        a.partials[s * NS + c] = t;
    }
}

// a particle without a list, of cnt neighbours, itself included
__device__ __forceinline__ void count_unlisted(const SimArgs& a, uint32_t cnt)
{
    atomicAdd(&a.st->unlisted, 1u);
    atomicMax(&a.st->most_pairs, cnt);
}

// words that a list of cnt entries takes
__device__ __forceinline__ uint32_t list_words(uint32_t cnt) { return cnt <= 2u ? 1u : 1u + cnt / 3u; }

// a particle's rows scanned whole in LDS (the rare particle without a list)
template <int NS, bool TRANSFER, int CAP, int SCAP, typename PR>
__device__ __forceinline__ void list_scan(const SimArgs& a, const double (*lpos)[CAP], const double* lsr,
                                          const double (*lms)[SCAP], const uint32_t (*cst)[TileLimits<3>::cols],
                                          int rbase, int cl, int ch, uint32_t li, const double* xi,
                                          Acc<0, NS, TRANSFER>& acc, PR rec)
{
    for (int pz = 0; pz < 3; ++pz)
        for (int dy = 0; dy < 3; ++dy) {
            const int sg = rbase + pz * TileLimits<3>::seg_y + dy;
            scan_row<3, 0, NS, TRANSFER, false>(
                a, [&](int d, uint32_t k) { return lpos[d][k]; }, [&](uint32_t k) { return lsr[k]; },
                [&](int c, uint32_t k) { return lms[c][k]; }, cst[sg][cl], cst[sg][ch], 0u, xi, -INFINITY, INFINITY,
                li, acc, rec);
        }
}

// Row sum, pair count and list of one particle per lane: LDS slot li, sorted
// slot i, candidates in columns cl..ch-1 of the halo rows from rbase on.
// Every lane of the wave calls it; act: the lane has a particle of its own.
template <bool EXPORT, int CAP, typename F>
__device__ __forceinline__ void list_rowsum(const SimArgs& a, const double (*lpos)[CAP],
                                            const uint32_t (*cst)[TileLimits<3>::cols], uint16_t (*found)[kListBlock],
                                            int rbase, int cl, int ch, uint32_t li, uint32_t i, bool act,
                                            const double* xi, Acc<0, 1, false>& acc, F export_slot)
{
    constexpr int kSY = TileLimits<3>::seg_y;
    constexpr uint32_t kT = sizeof(double);
    uint16_t* const list = &found[0][threadIdx.x];
    uint32_t at = 0;                        // entries, in units of found's row
    const uint32_t first = cst[rbase][cl];
    const uint32_t obs = li * kT;
#pragma unroll
    for (int pz = 0; pz < 3; ++pz) {
        const int s0 = rbase + pz * kSY;
        const uint32_t b0 = cst[s0][cl], l0 = cst[s0][ch] - b0;
        const uint32_t b1 = cst[s0 + 1][cl], l1 = cst[s0 + 1][ch] - b1;
        const uint32_t b2 = cst[s0 + 2][cl], l2 = cst[s0 + 2][ch] - b2;
        const uint32_t tot = act ? l0 + l1 + l2 : 0u;
        const uint32_t e0 = l0, e1 = l0 + l1;
        uint32_t ob0 = b0 * kT, ob1 = (b1 - l0) * kT, ob2 = (b2 - l0 - l1) * kT;
        asm volatile("" : "+v"(ob0), "+v"(ob1), "+v"(ob2));
        const uint32_t kmax = wave_max_u32(tot);
        // candidates k .. k + U - 1: their LDS reads first; a candidate past
        // the lane's rows reads the particle's own slot
        auto group = [&](auto width, uint32_t k) {
            constexpr int U = width;
            uint32_t off[U];
            double xj[U][3];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                off[u] = (k + u) * kT + (k + u < e0 ? ob0 : (k + u < e1 ? ob1 : ob2));
                off[u] = k + u < tot ? off[u] : obs;
#pragma unroll
                for (int d = 0; d < 3; ++d)
                    xj[u][d] = lds_at(lpos[d], static_cast<int>(off[u]));
            }
            uint64_t in[U];
#pragma unroll
            for (int u = 0; u < U; ++u)
                in[u] = within(a, Pair<3, double>::r2(xi, xj[u])) & __builtin_amdgcn_uicmp(k + u, tot, kIcmpUlt);
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (__builtin_amdgcn_inverse_ballot_w64(in[u])) {
                    list[at] = static_cast<uint16_t>(off[u]);
                    at += kListBlock;
                }
            // (a list past its end keeps overwriting the rows kept for that)
            at = min(at, static_cast<uint32_t>(kListMax + 1) * kListBlock);
        };
        uint32_t k = 0;
        for (; k + 4u <= kmax; k += 4u)
            group(std::integral_constant<int, 4>{}, k);
        if (k + 2u <= kmax) {
            group(std::integral_constant<int, 2>{}, k);
            k += 2u;
        }
        if (k < kmax)
            group(std::integral_constant<int, 1>{}, k);
    }
    uint32_t cnt = at / kListBlock;
    const bool over = cnt > static_cast<uint32_t>(kListMax);
    cnt = over ? 0u : cnt;
    // kernel values over the list and its words, three entries at a time (the
    // first word two); an entry past the lane's count is its own slot
    uint32_t far = 0;
    double s = 0.0;
    auto word = [&](uint32_t k0, int n, uint32_t lo) {
        uint32_t off[3], w = 0u;
        double xj[3][3];
#pragma unroll
        for (int u = 0; u < 3; ++u) {
            if (u >= n)
                break;
            off[u] = k0 + u < cnt ? list[(k0 + u) * kListBlock] : obs;
#pragma unroll
            for (int d = 0; d < 3; ++d)
                xj[u][d] = lds_at(lpos[d], static_cast<int>(off[u]));
        }
#pragma unroll
        for (int u = 0; u < 3; ++u) {
            if (u >= n)
                break;
            const double kv = Pair<3, double>::kernel(a, Pair<3, double>::r2(xi, xj[u]));
            s += k0 + u < cnt ? kv : 0.0;
            const uint32_t rel = off[u] / kT - first;
            far |= rel;
            w |= rel << (lo + 10u * u);
        }
        return w;
    };
    const uint32_t nw = list_words(wave_max_u32(cnt));
    const uint32_t w0 = cnt | word(0u, 2, 6u);
    for (uint32_t w = 1; w < nw; ++w) {
        const uint32_t v = word(3u * w - 1u, 3, 0u);
        if (!EXPORT && act)
            list_word(a, static_cast<int>(w))[i] = v;
    }
    const bool none = over || far > 1023u;
    if (!EXPORT && act)
        list_word(a, 0)[i] = none ? kListNone : w0;
    acc.s = s;
    acc.cnt = cnt;
    if (over) {
        acc = {};
        list_scan<1, false, CAP, 1>(a, lpos, nullptr, nullptr, cst, rbase, cl, ch, li, xi, acc,
                                    [&](uint32_t k) { if (act) export_slot(k); });
    } else if constexpr (EXPORT) {
        for (uint32_t k = 0; k < cnt; ++k) {
            const uint32_t slot = list[k * kListBlock] / kT;
            if (slot != li && act)
                export_slot(slot);
        }
    }
    if (!EXPORT && act && none)
        count_unlisted(a, acc.cnt);
}

// Mass increments of one particle per lane from its list (lw: its words but
// the last, loaded ahead).
template <int NS, bool EXPORT, int CAP, typename F>
__device__ __forceinline__ void list_transfer(const SimArgs& a, const double (*lpos)[CAP], const double (&lsr)[CAP],
                                              const double (*lms)[CAP], const uint32_t (*cst)[TileLimits<3>::cols],
                                              int rbase, int cl, int ch, uint32_t li, uint32_t i, bool act,
                                              uint32_t* lw, const double* xi, Acc<0, NS, true>& acc, F export_slot)
{
    constexpr uint32_t kT = sizeof(double);
    const bool none = (lw[0] & 63u) == kListNone;
    const uint32_t cnt = act && !none ? lw[0] & 63u : 0u;
    const uint32_t first = cst[rbase][cl] * kT;
    const uint32_t nw = list_words(wave_max_u32(cnt));
    if (nw == static_cast<uint32_t>(kListWords))
        lw[kListWords - 1] = act ? list_word(a, kListWords - 1)[i] : 0u;
    // n slots of word v from bit lo, entries k0 ..: an entry past the lane's
    // count visits the particle's own slot (r^2 = 0 and m_j - m_i = 0 give an
    // increment of exactly zero)
    auto visit = [&](uint32_t v, uint32_t k0, int n, uint32_t lo) {
        uint32_t off[3];
        double xj[3][3], sj[3], wt[3];
#pragma unroll
        for (int u = 0; u < 3; ++u) {
            if (u >= n)
                break;
            off[u] = k0 + u < cnt ? first + ((v >> (lo + 10u * u)) & 1023u) * kT : li * kT;
#pragma unroll
            for (int d = 0; d < 3; ++d)
                xj[u][d] = lds_at(lpos[d], static_cast<int>(off[u]));
            sj[u] = lds_at(&lsr[0], static_cast<int>(off[u]));
        }
#pragma unroll
        for (int u = 0; u < 3; ++u) {
            if (u >= n)
                break;
            if constexpr (EXPORT) {
                if (off[u] != li * kT && act)
                    export_slot(off[u] / kT);
            }
            wt[u] = Pair<3, double>::weight(Pair<3, double>::kernel(a, Pair<3, double>::r2(xi, xj[u])), acc.si, sj[u]);
        }
#pragma unroll
        for (int c = 0; c < NS; ++c) {
            double mj[3];
#pragma unroll
            for (int u = 0; u < 3; ++u)
                if (u < n)
                    mj[u] = lds_at(lms[c], static_cast<int>(off[u]));
#pragma unroll
            for (int u = 0; u < 3; ++u)
                if (u < n)
                    acc.dl[c] = __builtin_fma(wt[u], mj[u] - acc.mi[c], acc.dl[c]);
        }
    };
    visit(lw[0], 0u, 2, 6u);
#pragma unroll
    for (int w = 1; w < kListWords; ++w)
        if (static_cast<uint32_t>(w) < nw)
            visit(lw[w], 3u * w - 1u, 3, 0u);
    if (act && none)
        list_scan<NS, true, CAP, CAP>(a, lpos, &lsr[0], lms, cst, rbase, cl, ch, li, xi, acc,
                                      [&](uint32_t k) { export_slot(k); });
}

}  // namespace mtpt
