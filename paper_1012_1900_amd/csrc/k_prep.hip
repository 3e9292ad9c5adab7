// Normalisation, mask, gamma0 and ordered compaction (Algorithm A2 step 2, "Kernel 1"),
// plus the stand-alone pass-rate reduction.
//
// Three launches (one for small grids, k_prep_small), each a coalesced stream over the dose arrays; results cross blocks only
// at kernel boundaries or through atomic adds (a cross-block hand-over inside a kernel
// would need device-scope release fences, which write back the XCD's L2):
//   1. maximum and finiteness of D_r: one partial per block (block 0 also clears the
//      tile-group sums and the flags);
//   2. every block reduces those partials itself (a few KB from L2), derives the
//      threshold and the global 1/dD, then counts the masked nodes of its tile and their
//      max gamma0^2, checks D_e's finiteness, stores the tile's mask bits and count and
//      adds the count and the maximum into its tile group (about sqrt(tiles) / 8 tiles per
//      group, so no address sees many atomics); block 0 also stores the scalars and clears
//      the search counters;
//   3. ordered emit of the masked node indices from the mask bits: a block's first slot is
//      the sum of the groups before its own plus the tiles of its group before it; the
//      last block stores M and R^2.
// Each dose volume is read once by the compaction except D_r, read twice (its maximum sets
// the threshold that the mask needs); the emit reads one bit per node.
#include "internal.hpp"

namespace gammax {

namespace {

constexpr int WAVE = 64;

__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
    for (int o = WAVE / 2; o > 0; o >>= 1) v = max(v, (uint32_t)__shfl_xor((int)v, o));
    return v;
}
__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t v) {
    for (int o = WAVE / 2; o > 0; o >>= 1) v += (uint32_t)__shfl_xor((int)v, o);
    return v;
}

// Block-wide max and or over PREP_THREADS threads (result valid in every thread).
__device__ __forceinline__ void block_max_or(uint32_t& m, uint32_t& f) {
    __shared__ uint32_t s_m[PREP_THREADS / WAVE], s_f[PREP_THREADS / WAVE];
    m = wave_max_u32(m);
    f = __ballot(f != 0u) != 0ull ? 1u : 0u;
    const int w = threadIdx.x / WAVE;
    if ((threadIdx.x & (WAVE - 1)) == 0) {
        s_m[w] = m;
        s_f[w] = f;
    }
    __syncthreads();
    m = s_m[0];
    f = s_f[0];
    for (int j = 1; j < PREP_THREADS / WAVE; ++j) {
        m = max(m, s_m[j]);
        f |= s_f[j];
    }
    __syncthreads();
}

// 1. dose maximum and finiteness of D_r (WITH_EV: of D_e too), one partial per block (vb
// of vgrid).  The map's compaction checks D_e where it loads it (prep_count_body); there
// block 0 here clears the flags that the later kernels or into.
template <bool WITH_EV>
__device__ __forceinline__ void dose_max_body(const PrepArgs& a, int vb, int vgrid) {
    uint32_t best = 0u, bad = 0u;
    // DM_ITEMS nodes per thread per step, all loads of a step issued before the first use
    // (indices clamped to the last node; the clamped copies do not change a max or an or)
    constexpr int DM_ITEMS = 8;
    const int64_t step = (int64_t)vgrid * PREP_THREADS * DM_ITEMS;
    for (int64_t b0 = (int64_t)vb * PREP_THREADS * DM_ITEMS; b0 < a.n; b0 += step) {
        float r[DM_ITEMS], e[DM_ITEMS];
#pragma unroll
        for (int k = 0; k < DM_ITEMS; ++k) {
            const int64_t i = b0 + (int64_t)k * PREP_THREADS + threadIdx.x;
            const int64_t j = i < a.n ? i : a.n - 1;
            r[k] = a.ref[j];
            if (WITH_EV) e[k] = a.ev[j];
        }
#pragma unroll
        for (int k = 0; k < DM_ITEMS; ++k) {
            bad |= (!isfinite(r[k]) || (WITH_EV && !isfinite(e[k]))) ? 1u : 0u;
            best = max(best, float_to_ord(r[k]));
        }
    }
    block_max_or(best, bad);
    if (threadIdx.x == 0) {
        a.part[vb] = best;
        a.part[MAX_BLOCKS + vb] = bad;
        if (!WITH_EV && vb == 0) a.sc->flags = 0u;
    }
    if (a.super && vb == 0)
        for (int j = threadIdx.x; j < 2 * a.n_super; j += PREP_THREADS) a.super[j] = 0u;
}

__global__ __launch_bounds__(PREP_THREADS) void k_dose_max(PrepArgs a) {
    dose_max_body<false>(a, blockIdx.x, gridDim.x);
}
__global__ __launch_bounds__(PREP_THREADS) void k_dose_max_both(PrepArgs a) {
    dose_max_body<true>(a, blockIdx.x, gridDim.x);
}

// 1b. dose maximum and the global 1/dD only (no mask, no compaction): one block reduces
// the partials of k_dose_max.
__global__ __launch_bounds__(PREP_THREADS) void k_dose_finish(PrepArgs a, int nb_red) {
    uint32_t dm = 0u, bad = 0u;
    for (int j = threadIdx.x; j < nb_red; j += PREP_THREADS) {
        dm = max(dm, a.part[j]);
        bad |= a.part[MAX_BLOCKS + j];
    }
    block_max_or(dm, bad);
    if (threadIdx.x == 0) {
        const float dmax = ord_to_float(dm);
        a.sc->dmax_ord = dm;
        a.sc->flags = bad ? FLAG_NONFINITE : 0u;
        a.sc->thr_val = a.thr * dmax;
        a.sc->inv_dd = 1.0f / (a.dd * dmax);
    }
}

__device__ __forceinline__ bool node_masked(float dr, float thr_val, int local) {
    return dr >= thr_val && (!local || dr > 0.0f);
}

// The scalars that every map starts with, but flags and n_masked.
__device__ __forceinline__ void prep_scalars(Scalars* sc, uint32_t dm, float thr_val, float inv_dd) {
    sc->dmax_ord = dm;
    sc->thr_val = thr_val;
    sc->inv_dd = inv_dd;
    sc->r2_bits = 0u;
    sc->n_tail = 0u;
    sc->n_guard = 0u;
    sc->maxg2_bits = 0u;
    sc->n_fallback = 0u;
    sc->sort_overflow = 0u;
    sc->long_rows = 0u;
    sc->n_fallback_inline = 0u;
    sc->ticket = 0u;
    sc->n_pass = 0ull;
    sc->n_border = 0ull;
    sc->n_fp64 = 0ull;
    sc->n_cells = 0ull;
}

// 2. every block: the dose maximum from the partials, then per tile the masked count, max
// gamma0^2 and -1 for unmasked nodes.  Block 0 stores the scalars of this map.
__device__ __forceinline__ void prep_count_body(const PrepArgs& a, int nb_red, int vb) {
    // this tile's doses first (they do not depend on the dose maximum), then the partials:
    // all loads in flight together, indices clamped to valid entries
    const int64_t base = (int64_t)vb * PREP_TILE;
    float rr[PREP_ITEMS], ee[PREP_ITEMS];
#pragma unroll
    for (int k = 0; k < PREP_ITEMS; ++k) {
        const int64_t i = base + (int64_t)k * PREP_THREADS + threadIdx.x;
        const int64_t j = i < a.n ? i : a.n - 1;
        rr[k] = a.ref[j];
        ee[k] = a.ev[j];
    }
    constexpr int PR = MAX_BLOCKS / PREP_THREADS;
    uint32_t pm[PR], pb[PR];
#pragma unroll
    for (int r = 0; r < PR; ++r) {
        const int j = threadIdx.x + PREP_THREADS * r;
        const int jj = j < nb_red ? j : 0;
        pm[r] = a.part[jj];
        pb[r] = a.part[MAX_BLOCKS + jj];
    }
    uint32_t dm = 0u, bad = 0u;
#pragma unroll
    for (int r = 0; r < PR; ++r) {
        dm = max(dm, pm[r]);
        bad |= pb[r];
    }
    block_max_or(dm, bad);
    const float dmax = ord_to_float(dm);
    const float thr_val = a.thr * dmax;
    const float inv_dd_g = 1.0f / (a.dd * dmax);
    if (vb == 0) {
        for (int j = threadIdx.x; j < SUM_BINS; j += PREP_THREADS) a.sums[j] = BlockSums{};
        if (threadIdx.x == 0) {
            if (bad) atomicOr(&a.sc->flags, FLAG_NONFINITE);
            prep_scalars(a.sc, dm, thr_val, inv_dd_g);
            a.sc->n_masked = 0u;
        }
    }
    uint32_t cnt = 0u, best = 0u;
    bool bad_e = false;
    const int lane = threadIdx.x & (WAVE - 1);
#pragma unroll
    for (int k = 0; k < PREP_ITEMS; ++k) {
        const int64_t i = base + (int64_t)k * PREP_THREADS + threadIdx.x;
        bool m = false;
        if (i < a.n) {
            const float dr = rr[k];
            bad_e |= !isfinite(ee[k]);
            m = node_masked(dr, thr_val, a.local);
            if (m) {
                const float de = ee[k];
                const float g2 = gamma0_sq(de, dr, node_inv_dd(dr, inv_dd_g, a.dd, a.local));
                best = max(best, f2u(g2));
                ++cnt;
            } else {
                a.gamma[i] = -1.0f;
            }
        }
        // the mask bits of the wave's 64 consecutive nodes, for the emit
        const unsigned long long bal = __ballot(m);
        if (lane == 0) a.mbits[(base + (int64_t)k * PREP_THREADS + (threadIdx.x & ~(WAVE - 1))) / WAVE] = bal;
    }
    if (__ballot(bad_e) != 0ull && lane == 0) atomicOr(&a.sc->flags, FLAG_NONFINITE);
    __shared__ uint32_t s_cnt[PREP_THREADS / WAVE];
    cnt = wave_sum_u32(cnt);
    if ((threadIdx.x & (WAVE - 1)) == 0) s_cnt[threadIdx.x / WAVE] = cnt;
    uint32_t unused = 0u;
    block_max_or(best, unused);   // also orders s_cnt
    if (threadIdx.x == 0) {
        uint32_t c = 0u;
        for (int j = 0; j < PREP_THREADS / WAVE; ++j) c += s_cnt[j];
        a.blockcnt[vb] = c;
        const int grp = vb >> a.super_shift;
        if (c) atomicAdd(&a.super[grp], c);
        if (best) atomicMax(&a.super[a.n_super + grp], best);
    }
}

__global__ __launch_bounds__(PREP_THREADS) void k_prep_count(PrepArgs a, int nb_red) {
    prep_count_body(a, nb_red, blockIdx.x);
}

// 3. the masked nodes in grid order.
__device__ __forceinline__ void prep_emit_body(const PrepArgs& a, int vb) {
    const int64_t base = (int64_t)vb * PREP_TILE;
    __shared__ uint32_t s_wave[PREP_ITEMS][PREP_THREADS / WAVE];
    __shared__ uint32_t s_pre[PREP_THREADS / WAVE];
    const int lane = threadIdx.x & (WAVE - 1), w = threadIdx.x / WAVE;
    const unsigned long long lt = (lane == 0) ? 0ull : (~0ull >> (WAVE - lane));
    // this tile's mask bits (one word per wave and item), in flight while the prefix is summed
    unsigned long long bal[PREP_ITEMS];
#pragma unroll
    for (int k = 0; k < PREP_ITEMS; ++k) bal[k] = a.mbits[(base + (int64_t)k * PREP_THREADS) / WAVE + w];
    // first slot of this tile: the groups before its own, then its group's earlier tiles
    {
        const int grp = vb >> a.super_shift;
        uint32_t v = 0u;
        for (int j = threadIdx.x; j < grp; j += PREP_THREADS) v += a.super[j];
        for (int t = (grp << a.super_shift) + threadIdx.x; t < vb; t += PREP_THREADS) v += a.blockcnt[t];
        v = wave_sum_u32(v);
        if (lane == 0) s_pre[w] = v;
    }
    bool m[PREP_ITEMS];
#pragma unroll
    for (int k = 0; k < PREP_ITEMS; ++k) {
        m[k] = (bal[k] >> lane) & 1ull;
        if (lane == 0) s_wave[k][w] = (uint32_t)__popcll(bal[k]);
    }
    __syncthreads();
    uint32_t run = 0u;
    for (int j = 0; j < PREP_THREADS / WAVE; ++j) run += s_pre[j];
#pragma unroll
    for (int k = 0; k < PREP_ITEMS; ++k) {
        uint32_t off = run, tot = 0u;
        for (int j = 0; j < PREP_THREADS / WAVE; ++j) {
            const uint32_t c = s_wave[k][j];
            if (j < w) off += c;
            tot += c;
        }
        if (m[k]) a.nodes[off + (uint32_t)__popcll(bal[k] & lt)] = (uint32_t)(base + (int64_t)k * PREP_THREADS + threadIdx.x);
        run += tot;
    }
    if (vb == a.ntiles - 1) {
        // the last tile: M and R^2 (the maximum over the groups)
        uint32_t mx = 0u, none = 0u;
        for (int j = threadIdx.x; j < a.n_super; j += PREP_THREADS) mx = max(mx, a.super[a.n_super + j]);
        block_max_or(mx, none);
        if (threadIdx.x == 0) {
            a.sc->n_masked = run;
            a.sc->r2_bits = mx;
        }
    }
}

__global__ __launch_bounds__(PREP_THREADS) void k_prep_emit(PrepArgs a) { prep_emit_body(a, blockIdx.x); }

// The same, EMIT_TILES tiles per block (large grids): the prefix is summed once for all of them, a
// lane holds the mask word of one (tile, item) and their slots come from one scan.  A word
// without nodes costs a test.  One tile per block is bound by its chain of dependent loads,
// which a large grid runs several times per slot: 16.9 us at 192x256x256 (12288 tiles), 9.5 at
// 160x200x200 (6250), 7.0 at 117x171x171 (3342), 4.1 at 96x128x128 (1536); this takes 9.0, 6.4,
// 6.0 and 5.3.
constexpr int64_t EMIT_WIDE_MIN = 3072;   // tiles
constexpr int EMIT_TILES = 8, EMIT_WORDS = EMIT_TILES * PREP_ITEMS;   // words per wave
static_assert(EMIT_WORDS <= WAVE && WAVE % EMIT_WORDS == 0, "a lane per word");
__global__ __launch_bounds__(PREP_THREADS) void k_prep_emit_wide(PrepArgs a) {
    constexpr int W = PREP_THREADS / WAVE;
    __shared__ uint32_t s_cnt[EMIT_WORDS][W];
    __shared__ uint32_t s_pre[W];
    const int lane = threadIdx.x & (WAVE - 1), w = threadIdx.x / WAVE;
    const int t0 = blockIdx.x * EMIT_TILES;
    const int l = lane % EMIT_WORDS, tile = t0 + l / PREP_ITEMS;
    // lane l: the word of tile t0 + l / PREP_ITEMS, item l % PREP_ITEMS, this wave's nodes
    unsigned long long word = 0ull;
    if (tile < a.ntiles)
        word = a.mbits[((int64_t)tile * PREP_TILE + (int64_t)(l % PREP_ITEMS) * PREP_THREADS) / WAVE + w];
    {
        const int grp = t0 >> a.super_shift;
        uint32_t v = 0u;
        for (int j = threadIdx.x; j < grp; j += PREP_THREADS) v += a.super[j];
        for (int t = (grp << a.super_shift) + threadIdx.x; t < t0; t += PREP_THREADS) v += a.blockcnt[t];
        v = wave_sum_u32(v);
        if (lane == 0) s_pre[w] = v;
    }
    if (lane < EMIT_WORDS) s_cnt[l][w] = (uint32_t)__popcll(word);
    __syncthreads();
    uint32_t run = 0u;
    for (int j = 0; j < W; ++j) run += s_pre[j];
    // slots: the words in (tile, item) order, the waves' within a word
    uint32_t off = 0u, tot = 0u;
    for (int j = 0; j < W; ++j) {
        const uint32_t c = s_cnt[l][j];
        off += j < w ? c : 0u;
        tot += c;
    }
    uint32_t incl = tot;
    for (int o = 1; o < EMIT_WORDS; o <<= 1) {
        const uint32_t up = (uint32_t)__shfl_up((int)incl, o, EMIT_WORDS);
        incl += l >= o ? up : 0u;
    }
    off += run + incl - tot;
    const unsigned long long lt = (lane == 0) ? 0ull : (~0ull >> (WAVE - lane));
#pragma unroll 4
    for (int k = 0; k < EMIT_WORDS; ++k) {
        const unsigned long long bal =
            ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(word >> 32), k) << 32) |
            (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)word, k);
        if (bal == 0ull) continue;
        const uint32_t at = (uint32_t)__builtin_amdgcn_readlane((int)off, k);
        if ((bal >> lane) & 1ull)
            a.nodes[at + (uint32_t)__popcll(bal & lt)] =
                (uint32_t)((int64_t)(t0 + k / PREP_ITEMS) * PREP_TILE + (k % PREP_ITEMS) * PREP_THREADS + threadIdx.x);
    }
    if (t0 + EMIT_TILES >= a.ntiles) {
        uint32_t mx = 0u, none = 0u;
        for (int j = threadIdx.x; j < a.n_super; j += PREP_THREADS) mx = max(mx, a.super[a.n_super + j]);
        block_max_or(mx, none);
        if (threadIdx.x == EMIT_WORDS - 1) a.sc->n_masked = run + incl;
        if (threadIdx.x == 0) a.sc->r2_bits = mx;
    }
}

// 1-3 in one launch, for grids where the three launches cost more than the work in them: every
// block of 1024 nodes reads all of D_r itself (from L2 after the first), takes the maximum and
// counts the masked nodes before its own, so nothing crosses blocks but the largest gamma0^2
// and the finiteness of D_e, which go to the block's partial slot and are joined where the
// counts are.  Launch latency and one pass of dependent loads bound it: 4.5 us at 64x64 and 7.7
// at 173x200, against 10.0 and 10.5 in three launches and the gaps between them.
constexpr int SMALL_THREADS = 1024, SMALL_STEP = 8;
constexpr int SMALL_STEPS = (int)(PREP_SMALL_MAX / (SMALL_THREADS * SMALL_STEP));
static_assert(PREP_SMALL_MAX % (SMALL_THREADS * SMALL_STEP) == 0, "whole steps");
static_assert(PREP_SMALL_MAX / SMALL_THREADS <= SUM_BINS, "one partial slot per block");

__global__ __launch_bounds__(SMALL_THREADS) void k_prep_small(PrepArgs a) {
    constexpr int W = SMALL_THREADS / WAVE;
    __shared__ uint32_t s_a[W], s_b[W], s_c[W];
    const int lane = threadIdx.x & (WAVE - 1), w = threadIdx.x / WAVE;
    const int vb = blockIdx.x, n = (int)a.n;
    const int i = vb * SMALL_THREADS + (int)threadIdx.x;
    const float dr = a.ref[i < n ? i : n - 1], de = a.ev[i < n ? i : n - 1];
    float r[SMALL_STEPS][SMALL_STEP];
    // the bits as integers: the largest of them is the largest dose where one is not negative;
    // finiteness from the largest magnitude
    int32_t mi = INT32_MIN;
    uint32_t ma = 0u;
#pragma unroll
    for (int g = 0; g < SMALL_STEPS; ++g)
        if (g * SMALL_STEP * SMALL_THREADS < n)
#pragma unroll
            for (int k = 0; k < SMALL_STEP; ++k) {
                const int j = (g * SMALL_STEP + k) * SMALL_THREADS + (int)threadIdx.x;
                r[g][k] = a.ref[j < n ? j : n - 1];
            }
#pragma unroll
    for (int g = 0; g < SMALL_STEPS; ++g)
        if (g * SMALL_STEP * SMALL_THREADS < n)
#pragma unroll
            for (int k = 0; k < SMALL_STEP; ++k) {
                mi = max(mi, (int32_t)f2u(r[g][k]));
                ma = max(ma, f2u(r[g][k]) & 0x7fffffffu);
            }
    uint32_t dm = float_to_ord(u2f((uint32_t)mi));
    if (mi < 0) {   // this thread's doses are all negative: integers order those the other way
        for (int j = (int)threadIdx.x; j < n; j += SMALL_THREADS) dm = max(dm, float_to_ord(a.ref[j]));
    }
    dm = wave_max_u32(dm);
    bool bad = __ballot(!isfinite(u2f(ma)) || (i < n && !isfinite(de))) != 0ull;
    if (lane == 0) {
        s_a[w] = dm;
        s_b[w] = bad ? 1u : 0u;
    }
    __syncthreads();
    bad = false;
#pragma unroll
    for (int k = 0; k < W; ++k) {
        dm = max(dm, s_a[k]);
        bad |= s_b[k] != 0u;
    }
    const float dmax = ord_to_float(dm);
    const float thr_val = a.thr * dmax;
    const float inv_dd_g = 1.0f / (a.dd * dmax);
    // the masked nodes before this block's (block vb's nodes are step vb of the loop)
    uint32_t before = 0u;
#pragma unroll
    for (int g = 0; g < SMALL_STEPS; ++g)
        if (g * SMALL_STEP < vb)
#pragma unroll
            for (int k = 0; k < SMALL_STEP; ++k)
                if (g * SMALL_STEP + k < vb)
                    before += (uint32_t)__popcll(__ballot(node_masked(r[g][k], thr_val, a.local)));
    const bool m = i < n && node_masked(dr, thr_val, a.local);
    const unsigned long long bal = __ballot(m);
    uint32_t best = 0u;
    if (m) best = f2u(gamma0_sq(de, dr, node_inv_dd(dr, inv_dd_g, a.dd, a.local)));
    else if (i < n) a.gamma[i] = -1.0f;
    best = wave_max_u32(best);
    __syncthreads();   // (s_a, s_b are read)
    if (lane == 0) {
        s_a[w] = before;
        s_b[w] = (uint32_t)__popcll(bal);
        s_c[w] = best;
    }
    __syncthreads();
    uint32_t off = 0u, tot = 0u;
#pragma unroll
    for (int k = 0; k < W; ++k) {
        off += s_a[k] + (k < w ? s_b[k] : 0u);
        tot += s_a[k] + s_b[k];
        best = max(best, s_c[k]);
    }
    const unsigned long long lt = (lane == 0) ? 0ull : (~0ull >> (WAVE - lane));
    if (m) a.nodes[off + (uint32_t)__popcll(bal & lt)] = (uint32_t)i;
    // the partial slots: this block's, and block 0 those that no block has
    if (threadIdx.x == 0) {
        BlockSums b{};
        b.prep = (best & ~PREP_BAD) | (bad ? PREP_BAD : 0u);   // (a NaN of finite doses has either sign)
        a.sums[vb] = b;
    }
    if (vb == 0) {
        const int j = (int)gridDim.x + (int)threadIdx.x;
        if (j < SUM_BINS) a.sums[j] = BlockSums{};
    }
    // the scalars but n_masked: block 0; n_masked: the last block
    if (threadIdx.x == 0) {
        if (vb == 0) {
            a.sc->flags = 0u;
            prep_scalars(a.sc, dm, thr_val, inv_dd_g);
        }
        if (vb == (int)gridDim.x - 1) a.sc->n_masked = tot;
    }
}

// Same-address atomics from many blocks serialise (1024 blocks on three counters set the
// kernel's time: 25 us for 0.3 M nodes, 4.0 us now), so at most 256 blocks of 1024 threads run,
// each thread with PC_ITEMS loads in flight per step.
constexpr int PC_THREADS = 1024, PC_ITEMS = 8;
__global__ __launch_bounds__(PC_THREADS) void k_pass_count(const float* __restrict__ g, int64_t n,
                                                           unsigned long long* counts) {
    uint32_t ne = 0u, np = 0u, nb = 0u;
    const int64_t step = (int64_t)gridDim.x * PC_THREADS * PC_ITEMS;
    for (int64_t b0 = (int64_t)blockIdx.x * PC_THREADS * PC_ITEMS; b0 < n; b0 += step) {
        float v[PC_ITEMS];
#pragma unroll
        for (int k = 0; k < PC_ITEMS; ++k) {
            const int64_t i = b0 + (int64_t)k * PC_THREADS + threadIdx.x;
            v[k] = g[i < n ? i : n - 1];
        }
#pragma unroll
        for (int k = 0; k < PC_ITEMS; ++k) {
            const bool in = b0 + (int64_t)k * PC_THREADS + threadIdx.x < n && v[k] >= 0.0f;
            ne += in;
            np += in & (v[k] <= 1.0f);
            nb += in & (fabsf(v[k] - 1.0f) <= 1e-5f);
        }
    }
    // summed over the block, then one atomic per count
    __shared__ uint32_t s[3][PC_THREADS / WAVE];
    ne = wave_sum_u32(ne);
    np = wave_sum_u32(np);
    nb = wave_sum_u32(nb);
    const int w = threadIdx.x / WAVE;
    if ((threadIdx.x & (WAVE - 1)) == 0) {
        s[0][w] = ne;
        s[1][w] = np;
        s[2][w] = nb;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        unsigned long long t = 0ull;
        for (int j = 0; j < PC_THREADS / WAVE; ++j) t += s[threadIdx.x][j];
        if (t) atomicAdd(&counts[threadIdx.x], t);
    }
}

__global__ void k_zero3(unsigned long long* c) {
    if (threadIdx.x < 3) c[threadIdx.x] = 0ull;
}

int reduce_blocks(int64_t n) {
    int64_t b = (n + PREP_THREADS * 8 - 1) / (PREP_THREADS * 8);
    if (b > MAX_BLOCKS) b = MAX_BLOCKS;
    return (int)(b < 1 ? 1 : b);
}

// Batches: the same bodies, one block per (pair, block) item.
__global__ __launch_bounds__(PREP_THREADS) void k_batch_dose_max(const BatchPair* __restrict__ pairs,
                                                                 const uint2* __restrict__ items) {
    const uint2 w = items[blockIdx.x];
    const BatchPair& P = pairs[w.x];
    dose_max_body<false>(P.pa, (int)w.y, P.nbr);
}
__global__ __launch_bounds__(PREP_THREADS) void k_batch_prep_count(const BatchPair* __restrict__ pairs,
                                                                   const uint2* __restrict__ items) {
    const uint2 w = items[blockIdx.x];
    const BatchPair& P = pairs[w.x];
    prep_count_body(P.pa, P.nbr, (int)w.y);
}
__global__ __launch_bounds__(PREP_THREADS) void k_batch_prep_emit(const BatchPair* __restrict__ pairs,
                                                                  const uint2* __restrict__ items) {
    const uint2 w = items[blockIdx.x];
    const BatchPair& P = pairs[w.x];
    prep_emit_body(P.pa, (int)w.y);
}

}  // namespace

int prep_reduce_blocks(int64_t n) { return reduce_blocks(n); }

hipError_t launch_batch_prep(const BatchPair* pairs, const uint2* dm, int n_dm, const uint2* tiles, int n_tiles,
                             hipStream_t s) {
    if (n_dm <= 0 || n_tiles <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_batch_dose_max, dim3((unsigned)n_dm), dim3(PREP_THREADS), 0, s, pairs, dm);
    hipLaunchKernelGGL(k_batch_prep_count, dim3((unsigned)n_tiles), dim3(PREP_THREADS), 0, s, pairs, tiles);
    hipLaunchKernelGGL(k_batch_prep_emit, dim3((unsigned)n_tiles), dim3(PREP_THREADS), 0, s, pairs, tiles);
    return hipGetLastError();
}

int64_t prep_tiles(int64_t n) { return (n + PREP_TILE - 1) / PREP_TILE; }

void prep_groups(int64_t n, int* shift, int* n_super) {
    // 2^sh tiles per group with 4^(sh + 3) >= tiles: about sqrt(tiles) / 8 tiles share a
    // group counter (same-address atomics from blocks on every XCD serialise), and the
    // emit reads about 8 sqrt(tiles) group sums
    const int64_t t = prep_tiles(n);
    int sh = 0;
    while (((int64_t)1 << (2 * (sh + 3))) < t) ++sh;
    *shift = sh;
    *n_super = (int)((t + ((int64_t)1 << sh) - 1) >> sh);
}

int64_t prep_mbits_offset(int64_t n) {
    int sh = 0, ns = 0;
    prep_groups(n, &sh, &ns);
    return (prep_tiles(n) + 2 * (int64_t)ns + 1) & ~(int64_t)1;   // 8-byte aligned
}

int64_t prep_words(int64_t n) { return prep_mbits_offset(n) + 2 * prep_tiles(n) * (PREP_TILE / 64); }

hipError_t launch_prep(const PrepArgs& a, bool joined, hipStream_t s) {
    if (joined && a.n <= PREP_SMALL_MAX) {
        const unsigned nb = (unsigned)((a.n + SMALL_THREADS - 1) / SMALL_THREADS);
        hipLaunchKernelGGL(k_prep_small, dim3(nb), dim3(SMALL_THREADS), 0, s, a);
        return hipGetLastError();
    }
    const int nbr = reduce_blocks(a.n);
    const int64_t nb = prep_tiles(a.n);
    hipLaunchKernelGGL(k_dose_max, dim3(nbr), dim3(PREP_THREADS), 0, s, a);
    hipLaunchKernelGGL(k_prep_count, dim3((unsigned)nb), dim3(PREP_THREADS), 0, s, a, nbr);
    if (nb >= EMIT_WIDE_MIN)
        hipLaunchKernelGGL(k_prep_emit_wide, dim3((unsigned)((nb + EMIT_TILES - 1) / EMIT_TILES)), dim3(PREP_THREADS), 0,
                           s, a);
    else
        hipLaunchKernelGGL(k_prep_emit, dim3((unsigned)nb), dim3(PREP_THREADS), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_dose_partials(const PrepArgs& a, DosePartials* dp, hipStream_t s) {
    const int nbr = reduce_blocks(a.n);
    hipLaunchKernelGGL(k_dose_max_both, dim3(nbr), dim3(PREP_THREADS), 0, s, a);
    *dp = DosePartials{a.part, nbr, a.dd, a.thr, a.sc};
    return hipGetLastError();
}

hipError_t launch_dose_scalars(const PrepArgs& a, hipStream_t s) {
    DosePartials dp;
    const hipError_t e = launch_dose_partials(a, &dp, s);
    if (e != hipSuccess) return e;
    const int nbr = dp.n;
    hipLaunchKernelGGL(k_dose_finish, dim3(1), dim3(PREP_THREADS), 0, s, a, nbr);
    return hipGetLastError();
}

hipError_t launch_pass_count(const float* gamma, int64_t n, unsigned long long* counts3, hipStream_t s) {
    hipLaunchKernelGGL(k_zero3, dim3(1), dim3(64), 0, s, counts3);
    if (n > 0) {
        int64_t b = (n + PC_THREADS * PC_ITEMS - 1) / (PC_THREADS * PC_ITEMS);
        if (b > 256) b = 256;
        hipLaunchKernelGGL(k_pass_count, dim3((unsigned)b), dim3(PC_THREADS), 0, s, gamma, n, counts3);
    }
    return hipGetLastError();
}

}  // namespace gammax
