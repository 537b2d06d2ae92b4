// rk_tile.hip -- the fill by square tiles of spans.
//
// The table's (s, t) triangle is cut into square tiles of up to 16 x 16 spans: tile (S, T) holds
// the spans that start in block S and end in block T of `side` blocks of the chain each.  A tile
// reads only tiles to its left and below (S' >= S, T' <= T), so the tiles of one level T - S are
// independent and the fill is one launch per level, ceil(L / 16) of them, where a launch per
// span length costs L.  A workgroup owns one tile on 64 budgets (lane = m), one wave per end t:
//
//  1. Product: the splits i with both operands in earlier levels (side (S + 1) <= i <= side T), a
//     plain min-plus matrix product of 16 rows and 16 ends.  Its partial minima stay in LDS.
//  2. Solve: every wave walks its end t from the tile's last row s up to its first.  Splits
//     inside block S have their right operand Opt(i, t, m - x_i) among the wave's own earlier
//     rows (registers) and their left operand ap(s, i) in LDS; splits inside block T have
//     their left operand among the tile's other ends (LDS) and their right one in registers.
//
// What a cell needs at other budgets, Opt(s+1, t, m - xbar) of case 1 and Opt(i, t, m - x_i),
// lies in columns to the left, which other workgroups of the same launch compute at the same
// time.  Every Opt entry is written once per fill, as one 32-bit word; the fill's first kernel
// sets them all to UNSET, and a reader repeats its load until the word is set.  So no order
// between the stores of different words matters, and no fence, flag or cache maintenance is
// needed: readers and writers use relaxed atomics at device scope (a store is seen by
// another workgroup's load 0.35-0.5 us later, on one XCD or across).
//
// Measured against one launch per diagonal (4.5-10 us each, mostly latency), fill time at blocks
// x budgets x options: 8 x 501 x 3 42 -> 20 us, 64 x 1001 x 5 416 -> 165 us, 128 x 2001 x 8
// 1.08 -> 0.43 ms, 256 x 4001 x 8 3.51 -> 2.02 ms, 384 x 6001 x 16 8.2 -> 5.9 ms, 1000 x 601 x 4
// 24.7 -> 15.9 ms.
//
// Waits end: a workgroup waits only for columns to the left of its own in the same tile, and
// which columns it takes is decided when it starts: the tile's next ones, by a counter per
// tile.  So it waits only for workgroups that have started, in whatever order the XCDs
// start them and whatever else runs beside (another fill of this kind on another stream too,
// which could otherwise hold the place that a workgroup waited for needs).  As a last guard a
// wait gives up after SPIN_MAX loads, marks the table as failed (reads of it then return
// RK_E_INTERNAL) and goes on.
#include "rk_device.h"

#include <algorithm>
#include <type_traits>

namespace rk {

constexpr int32_t TB = 16;               // most blocks per tile side, waves per workgroup
constexpr int32_t TCI = 4;               // splits staged at a time by the product
constexpr int32_t TOPT = 4;               // options whose words are loaded together
constexpr int32_t TWIN = 4;              // most 64-column pieces of the case-1 window
constexpr int32_t UNSET = -1;            // an Opt entry not written yet in this fill
constexpr int32_t SPIN_MAX = 1 << 22;    // loads before a wait gives up (seconds)
constexpr int32_t TLIST_MIN = 40;        // splits from which the product sorts out those that matter
constexpr int32_t TPIECE = 128;          // splits sorted out at a time
constexpr int32_t TRI = TB * (TB - 1) / 2;

__device__ inline int32_t ld_dev(const int32_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline void st_dev(int32_t v, int32_t *p)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Read-only arrays of the chain, through the scalar cache where the address is wave-uniform
// whatever has been stored before.
typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(4))) i32x4 *opt_ptr;
typedef int32_t i32x2 __attribute__((ext_vector_type(2)));

// Summaries: the last value of every row of ap and of os in each group of `cpe` chunks, for the
// product to sort out its splits with.  They are kept in the left pads of the three tables,
// which nothing else of this fill uses: entry e of row r (e = 2 group for ap, 2 group + 1 for
// os) is word (e mod 64) n_rows + r of the 64 n_rows words that the pads of table e / 64 hold,
// so neighbouring rows' entries lie side by side.
constexpr int32_t SUM_GROUPS = 3 * 64 / 2;
__device__ inline int32_t *sum_at(const Tables &tb, int32_t e, int32_t r)
{
    const uint32_t w = (uint32_t)(e & 63) * (uint32_t)tb.inf_row + (uint32_t)r;
    return (e < 64 ? tb.opt : e < 128 ? tb.ap : tb.os) + (int64_t)(w >> 6) * tb.stride + (w & 63);
}
static_assert((int64_t)64 * RK_MAX_L * (RK_MAX_L + 1) / 2 < (int64_t(1) << 32), "summary words are counted in 32 bits");

// How many workgroups of the running launch have started on tile sb: in the slack rows before
// row 0, which nothing else of this fill uses.  The launch's last one sets it back to 0.
__device__ inline int32_t *started_at(const Tables &tb, int32_t sb) { return tb.opt - SLACK * (int64_t)tb.stride + sb; }
static_assert((RK_MAX_L + TB - 1) / TB <= TABLE_FAILED && TABLE_FAILED < SLACK * 64 && TABLE_FAILED <= 256,
              "the counters and the flag after them fit the slack rows (a row has 64 words at least), the counters "
              "k_tile_init's workgroup");

// The entries of the span rows of opt that a workgroup may wait for: UNSET.  The counters: 0.
// A workgroup that reads row r at other budgets does so only if its first column, less reach,
// lies below msa(r) (else the row is flat there), so nobody waits for a column from
// msa(r) + reach + 64 on.  Bound by its stores: the whole rows took 312 us at 384 blocks x 6001
// budgets (5.8 TB/s), a pass there 6.31 -> 6.16 ms without the rest.  Rows that one store of
// each thread covers are set whole: there the wait for msa costs more than the stores (1000
// blocks x 601 budgets 17.6 -> 17.8 ms with it).
__global__ __launch_bounds__(256) void k_tile_init(Tables tb, const int32_t *msa, int32_t reach, int32_t nb)
{
    typedef int32_t i32x4u __attribute__((ext_vector_type(4), aligned(4)));
    i32x4u *const row = (i32x4u *)(tb.opt + (int64_t)blockIdx.x * tb.stride);
    const i32x4u unset = {UNSET, UNSET, UNSET, UNSET};
    int32_t end = tb.stride;
    if (end - tb.padl > 4 * 256) end = (int32_t)min((int64_t)tb.padl + msa[blockIdx.x] + reach + 64, (int64_t)end);
    for (int32_t j = tb.padl / 4 + (int32_t)threadIdx.x; 4 * j < end; j += 256) row[j] = unset;
    if (blockIdx.x == 0 && (int32_t)threadIdx.x < nb) *started_at(tb, (int32_t)threadIdx.x) = 0;
    if (blockIdx.x == 0 && threadIdx.x == 0) tb.host[1] = *failed_at(tb) = 0;
}

// index in LDS of the left operand ap(s, s + u), s = S0 + ls, u = 0 .. 14 - ls
__device__ constexpr int32_t tri(int32_t ls, int32_t u) { return ls * (TB - 1) - ls * (ls - 1) / 2 + u; }

// FULL: sides of TB blocks, as a constant (as an argument it costs more scalar registers than there
// are: fill at 128 blocks x 2001 budgets 426 -> 432 us).
template <bool DIAG, int NW, bool FULL>
__global__ __launch_bounds__(TB * 64) void k_tile(DevChain ch, Tables tb, int32_t level, int32_t side_arg, int32_t n_chunks,
                                                  int32_t reach, int32_t flat_reach, int32_t cpe, int32_t m_ans)
{
    const int32_t side = FULL ? TB : side_arg;
    __shared__ __align__(16) int32_t cells[TB * TB * 64];  // the product's two staging buffers, then the tile
    __shared__ int32_t aps[(TRI + TB) * 64]; // left operands inside block S (reads run past a row's last)
    __shared__ int32_t win[NW ? TB * NW * 64 : 1];
    __shared__ int32_t prog[TB];             // rows each wave has finished
    __shared__ int32_t taken;
    __shared__ uint16_t list[DIAG ? 1 : RK_MAX_L];  // the product's splits, less i0
    __shared__ int32_t n_kept, ubs[DIAG ? 1 : TB * TB], keep[RK_MAX_L / 32 + 1];
    static_assert(TCI == 4 && TB == 16, "a wave stages four rows of one split");
    static_assert(2 * TCI * 2 * TB <= TB * TB, "two staging buffers fit the tile");

    const int32_t L = ch.L, K4 = ch.K4;
    int32_t chunk, sb;
    chunk_tile(blockIdx.x, (uint32_t)((L + side - 1) / side - level), &chunk, &sb);
    if (threadIdx.x == 0) {
        int32_t *const started = started_at(tb, sb);
        taken = __hip_atomic_fetch_add(started, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        // (as many workgroups as chunk_grid launches for each tile)
        if (taken == (n_chunks + 7) / 8 * 8 - 1) st_dev(0, started);
    }
    __syncthreads();
    chunk = __builtin_amdgcn_readfirstlane(taken);
    if (chunk >= n_chunks) return;
    const int32_t lane = (int32_t)(threadIdx.x & 63);
    const int32_t lt = __builtin_amdgcn_readfirstlane((int32_t)(threadIdx.x >> 6));
    const int32_t S0 = sb * side, T0 = S0 + level * side, t = T0 + lt;
    const int32_t t_end = min(T0 + side, L) - 1;  // the tile's last end
    const bool real = t <= t_end;
    const int32_t mb = chunk * 64, m = mb + lane;
    const int64_t stride = tb.stride;
    const uint32_t col = (uint32_t)(tb.padl + m) * 4u;
    const int32_t pitch = (int32_t)(stride * 4);
    bool dead = false;

    if (threadIdx.x < TB) prog[threadIdx.x] = 0;
    // entries read before they are written (and then not used) hold infinity
    for (int32_t j = (DIAG ? 0 : TRI * 64) + (int32_t)threadIdx.x; j < (TRI + TB) * 64; j += TB * 64) aps[j] = DINF;

    // Per row ls of this wave (lane ls; lane 16: the row below the tile): what the solve
    // reads per row, fetched once.
    int32_t r_lb, r_msa, r_P, r_need2, r_PT, r_x, r_need1max, r_P1;
    {
        const int32_t te = min(t, L - 1), s = min(S0 + min(lane, TB), te);
        const int64_t r = row_of(L, s, te);
        r_lb = ch.lb[r];
        r_msa = ch.msa[r];
        r_P = te + 1 < L ? ch.P[(int64_t)s * L + te + 1] : 0;
        r_need2 = te + 1 < L ? ch.need2[(int64_t)s * L + te + 1] : 0;
        r_PT = !DIAG && T0 + 1 < L ? ch.P[(int64_t)s * L + T0 + 1] : 0;
        r_x = ch.x[min(S0 + lane, L)];
        r_P1 = ch.P[(int64_t)s * L + min(s + 1, L - 1)];
        r_need1max = ch.need1max[s];
    }
    auto at = [](int32_t v, int32_t l) { return __builtin_amdgcn_readlane(v, l); };

    // from msa(S0, last end) on, every cell of the tile is lb
    const int32_t msa_tile = ch.msa[row_of(L, S0, t_end)];
    const bool closed_tile = mb >= msa_tile;

    const int32_t top = DIAG ? lt : side - 1;  // the wave's last row
    // the last values of the rows of ap and os (lane: ls), for the summaries
    int32_t end_a = 0, end_os = 0;
    auto last = [&](int32_t v, int32_t ls, int32_t &ends) {
        const int32_t end = __builtin_amdgcn_readlane(v, 63);
        ends = lane == ls ? end : ends;
    };
    auto summarize = [&]() {
        if (cpe > 0 && (chunk + 1 == n_chunks || (chunk + 1) % cpe == 0) && lane <= top) {
            const int32_t r = (int32_t)row_of(L, S0 + lane, t), e = 2 * (chunk / cpe);
            *sum_at(tb, e, r) = end_a;
            *sum_at(tb, e + 1, r) = end_os;
        }
    };
    auto answer = [&](int32_t v) {
        if (S0 == 0 && t == L - 1 && m == m_ans) __hip_atomic_store(tb.host, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    };

    // From msa(S0, last end) + reach on, all that the cells read is in closed form, too: the rows are written
    // as they are, with nothing to wait for (and nobody waits for these columns, see k_tile_init).
    // Bound by its stores.  Fills through the loop below -> so: 24 blocks x 200001 budgets with shifts of
    // up to 150 columns 395 -> 178 us, 64 x 400001 3.32 -> 1.83 ms, 384 x 6001 x 16 6.09 -> 5.72 ms.
    if (mb - flat_reach >= msa_tile) {
        if (!real) return;
        int64_t e = row_of(L, S0 + top, t) * stride + tb.padl + mb + lane;
        int32_t lb = 0;
#pragma unroll 1
        for (int32_t ls = top; ls >= 0; --ls) {
            lb = at(r_lb, ls);
            const bool only1 = (DIAG && ls == lt) || at(r_P1, ls) > 0;  // splits cost at least lb + r(F_s^0)
            const int32_t a = m >= at(r_need2, ls) ? min(at(r_P, ls) + lb, DINF) : DINF;
            __builtin_nontemporal_store(only1 ? lb | ONLY_CASE1 : lb, tb.opt + e);
            __builtin_nontemporal_store(a, tb.ap + e);
            __builtin_nontemporal_store(lb, tb.os + e);
            last(a, ls, end_a);
            end_os = lane == ls ? lb : end_os;
            e -= (int64_t)(L - (S0 + ls)) * (int32_t)stride;
        }
        summarize();
        answer(lb);
        return;
    }

    int32_t ost[TB - 1];  // Opt(T0 + 1 + v, t, m - x): right operands inside block T
    if (!DIAG && !closed_tile) {
        const int32_t s = S0 + lt;
        const int32_t *p = tb.ap + row_of(L, s, s) * stride;
        for (int32_t u = 0; u < side - 1 - lt; ++u, p += stride) aps[tri(lt, u) * 64 + lane] = ldb(p, col);
        for (int32_t u = max(side - 1 - lt, 0); u < TB - 1 - lt; ++u) aps[tri(lt, u) * 64 + lane] = DINF;
        if (real) {
#pragma unroll
            for (int32_t v = 0; v < TB - 1; ++v) ost[v] = v < lt ? ldb(tb.os + row_of(L, T0 + 1 + v, t) * stride, col) : DINF;
        }

        // The product's splits i0 .. T0, or those of them that can matter.  ap, Opt and with them
        // a candidate's value never rise with the budget.  So a cell's minimum is nowhere above
        // ub, the least of its candidates at the last budget of the chunks before, and a split
        // whose candidate at this group of chunks' last budget is no lower than ub in any of
        // the tile's cells can be left out, once the accumulators start from ub.
        const int32_t i0 = S0 + side, n_all = T0 - i0 + 1;
        const int32_t grp_e = 2 * (chunk / max(cpe, 1));  // the summaries' entry
        int32_t n_list = n_all;
        const bool listed = cpe > 0 && n_all >= TLIST_MIN;
        if (listed) {
            // TPIECE splits at a time through LDS, one cell and every fourth split per thread
            const int32_t cell = (int32_t)(threadIdx.x & 255), grp = lt >> 2, cr = cell >> 4, ck = cell & 15;
            i32x2 *const sa = (i32x2 *)cells, *const sbv = sa + TPIECE * (TB + 1);
            const int32_t ra = (int32_t)row_of(L, S0 + min(lt, side - 1), i0 - 1), rb = min(T0 + (lane & 15), t_end);
            // the entry before this group's and this group's
            auto both = [&](int32_t e, int32_t r) -> i32x2 {
                return i32x2{e > 1 ? *sum_at(tb, e - 2, r) : DINF, *sum_at(tb, e, r)};
            };
            auto stage = [&](int32_t p) {
                const int32_t np = min(n_all - p, TPIECE);
                __syncthreads();
                i32x2 va[TPIECE / 64], vb[TPIECE / 64];
#pragma unroll
                for (int32_t q = 0; q < TPIECE / 64; ++q) {
                    const int32_t ja = lane + 64 * q, jb = 64 * q + 4 * lt + (lane >> 4), i = i0 + p + min(jb, np - 1);
                    va[q] = both(grp_e, ra + p + min(ja, np - 1));
                    vb[q] = both(grp_e + 1, rb + (i * L - i * (i - 1) / 2 - i));
                }
#pragma unroll
                for (int32_t q = 0; q < TPIECE / 64; ++q) {
                    sa[(lane + 64 * q) * (TB + 1) + lt] = va[q];
                    sbv[(64 * q + 4 * lt + (lane >> 4)) * TB + (lane & 15)] = vb[q];
                }
                __syncthreads();
                return np;
            };
            if (threadIdx.x < 256) ubs[threadIdx.x] = DINF;
            if (threadIdx.x < RK_MAX_L / 32 + 1) keep[threadIdx.x] = 0;
            const i32x2 *const pa = sa + cr, *const pb = sbv + ck;
            int32_t ub = DINF, np = 0, last = (n_all - 1) / TPIECE * TPIECE;
            for (int32_t p = 0; p <= last; p += TPIECE) {
                np = stage(p);
#pragma unroll 4
                for (int32_t j = grp; j < np; j += 4) ub = min(ub, pa[j * (TB + 1)].x + pb[j * TB].x);
            }
            atomicMin(&ubs[cell], ub);
            __syncthreads();
            ub = ubs[cell];
            for (int32_t p = last; p >= 0; p -= TPIECE) {  // the last piece is still staged
                if (p != last) np = stage(p);
                uint32_t bits = 0;  // of the splits p + 4 b + grp
#pragma unroll 4
                for (int32_t j = grp; j < np; j += 4)
                    bits |= (uint32_t)(pa[j * (TB + 1)].y + pb[j * TB].y < ub) << (j / 4 % 32);
                static_assert(TPIECE <= 128, "one word of bits per piece and thread");
                // or over the wave, then over the waves of the group
#pragma unroll
                for (int32_t d = 1; d < 64; d *= 2) bits |= __shfl_xor(bits, d);
                if (lane < 32 && (bits >> lane & 1)) atomicOr(&keep[(p + 4 * lane + grp) / 32], 1 << ((p + 4 * lane + grp) % 32));
            }
            __syncthreads();
            if (lt == 0) {
                int32_t n = 0;
                for (int32_t j0 = 0; j0 < n_all; j0 += 64) {
                    const int32_t j = j0 + lane;
                    const bool k = j < n_all && (keep[j / 32] >> (j % 32) & 1);
                    const uint64_t mask = __ballot(k);
                    if (k) list[n + __popcll(mask & ((1ull << lane) - 1))] = (uint16_t)j;
                    n += __popcll(mask);
                }
                if (lane == 0) n_kept = n;
            }
        }
        // Wave w stages split w / 4 of the TCI, rows 4 q .. 4 q + 3 of either operand (q = w mod
        // 4), four rows of a column side by side, so that reading four takes one 16-byte LDS
        // read; it relaxes rows 4 wr .. and ends 4 wc .. of the tile.
        const int32_t wr = lt >> 2, wc = lt & 3;
        i32x4 acc[4];
        __syncthreads();
#pragma unroll
        for (int32_t r = 0; r < 4; ++r)
#pragma unroll
            for (int32_t k = 0; k < 4; ++k) acc[r][k] = listed ? ubs[(4 * wr + r) * TB + 4 * wc + k] : DINF;
        if (listed) n_list = __builtin_amdgcn_readfirstlane(n_kept);
        __syncthreads();
        // (rows and ends past the tile's last: the last again)
        const int32_t *const pa = tb.ap + row_of(L, min(S0 + 4 * wc, i0 - 1), i0 - 1) * stride;
        const int32_t *const pb = tb.os + min(T0 + 4 * wc, t_end) * stride;
        uint32_t ca[4], cb[4];  // byte offsets of the four rows from the first
        {
            uint32_t ra = 0;
#pragma unroll
            for (int32_t r = 0; r < 4; ++r) {
                ca[r] = ra * (uint32_t)pitch + col;
                cb[r] = (uint32_t)max(min(r, t_end - (T0 + 4 * wc)), 0) * (uint32_t)pitch + col;
                if (S0 + 4 * wc + r < i0 - 1) ra += (uint32_t)(L - 1 - (S0 + 4 * wc + r));
            }
        }
        i32x4 qa[2], qb[2];
        auto fetch = [&](int32_t c, i32x4 &xa, i32x4 &xb) {
            const int32_t e = min(c + wr, n_list - 1);  // past the end: the last split again
            const int32_t j = listed ? __builtin_amdgcn_readfirstlane(list[e]) : e, i = i0 + j;
            const int32_t *const a = pa + j * stride;
            const int32_t *const b = pb + (int64_t)(i * L - i * (i - 1) / 2 - i) * stride;
#pragma unroll
            for (int32_t r = 0; r < 4; ++r) {
                xa[r] = ldb(a, ca[r]);
                xb[r] = ldb(b, cb[r]);
            }
        };
        auto relax = [&](int32_t buf, i32x4 &xa, i32x4 &xb, int32_t next) {
            i32x4 *const as = (i32x4 *)cells + buf * (TCI * 2 * 4 * 64), *const bs = as + TCI * 4 * 64;
            as[lt * 64 + lane] = xa;
            bs[lt * 64 + lane] = xb;
            __syncthreads();
            if (next < n_list) fetch(next, xa, xb);
            const i32x4 *const aw = as + wr * 64 + lane, *const bw = bs + wc * 64 + lane;
#pragma unroll
            for (int32_t u = 0; u < TCI; u += 2) {
                const i32x4 a0 = aw[u * 4 * 64], b0 = bw[u * 4 * 64], a1 = aw[(u + 1) * 4 * 64], b1 = bw[(u + 1) * 4 * 64];
#pragma unroll
                for (int32_t r = 0; r < 4; ++r)
#pragma unroll
                    for (int32_t k = 0; k < 4; ++k) acc[r][k] = min(min(acc[r][k], a0[r] + b0[k]), a1[r] + b1[k]);
            }
        };
        if (n_list > 0) fetch(0, qa[0], qb[0]);
        if (n_list > TCI) fetch(TCI, qa[1], qb[1]);
        for (int32_t c = 0; c < n_list; c += 2 * TCI) {
            relax(0, qa[0], qb[0], c + 2 * TCI);
            if (c + TCI < n_list) relax(1, qa[1], qb[1], c + 3 * TCI);
        }
        __syncthreads();
#pragma unroll
        for (int32_t r = 0; r < 4; ++r)
#pragma unroll
            for (int32_t k = 0; k < 4; ++k) cells[((4 * wr + r) * TB + 4 * wc + k) * 64 + lane] = acc[r][k];
    }
    __syncthreads();
    if (!real) return;  // no barrier below

    // repeat get() (a round of loads; true: some word is still UNSET) until it is done
    auto settle = [&](auto &&get) {
        for (int32_t n = 0; get() && !dead;)
            if (++n > SPIN_MAX) {
                dead = true;
                if (lane == 0) {
                    st_dev(1, failed_at(tb));
                    __hip_atomic_store(tb.host + 1, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
                }
            }
    };
    // wait for rows up to ls of the waves lo .. hi - 1 of this workgroup
    auto wait_waves = [&](int32_t lo, int32_t hi, int32_t ls) {
        for (;;) {
            const int32_t p = lane >= lo && lane < hi
                                  ? __hip_atomic_load(&prog[lane & (TB - 1)], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)
                                  : TB;
            if (!__any(p < TB - ls)) break;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    };
    // Rows from the last to the first, and one more turn (ls = -1) that only completes the
    // first row's right operand.  The rows are a loop and not unrolled: unrolled, each wave
    // ran 80 KB of code once.  The kernel is bound by the instructions of this loop (16 waves
    // share four SIMDs), so it branches little and reads LDS in batches.
    int32_t os[TB];  // os[u] = Opt(s + u, t, m - x): right operands inside block S, u >= 1
#pragma unroll
    for (int32_t u = 0; u < TB; ++u) os[u] = DINF;
    int32_t a_prev = 0, os_prev = 0;  // ap and os values not stored yet
    // entries of rows (s, t), (s+1, t), (s+2, t) at this wave's first column; row (s-1, t) lies
    // L - s rows before (s, t)
    const int32_t stride32 = (int32_t)stride;
    int64_t e0 = row_of(L, S0 + top, t) * stride + tb.padl + mb, e1 = e0 + (int64_t)(L - 1 - (S0 + top)) * stride32, e2 = e1;
    // the window of case 1, columns m - 64 NH + 64 k of row (s+1, t); piece NH is this wave's own
    constexpr int32_t NH = NW - 1;
    int32_t *const wn = win + (NW ? lt * NW * 64 + lane : 0);
    const int32_t *const wm = wn + 64 * NH;  // column m
    const int32_t k0 = max(NH - chunk, 0);   // pieces left of column 0 are infinite
    if constexpr (NW > 0) {
#pragma unroll
        for (int32_t k = 0; k < NW; ++k)
            wn[64 * k] = DIAG || k < NH ? DINF : tb.opt[e1 + lane] & DINF;  // the row below the tile
    }
    int32_t best = DINF;
    for (int32_t ls = top; ls >= -1; --ls) {
        const int32_t s = S0 + ls, n_in = top - ls;  // splits s+1 .. s+n_in inside block S
        const bool rest = !DIAG || n_in > 0;  // row (s+1, t) exists
        const bool need_os = n_in > 0;        // ... and is one of this wave's
        const int32_t lsc = max(ls, 0);
        const int32_t lb = at(r_lb, lsc), x1 = at(r_x, ls + 1);
        const bool closed = ls < 0 || mb >= at(r_msa, lsc);
        // all columns of row (s+1, t) that this workgroup reads are past its msa (or there is none)
        const bool flat = !rest || mb - reach >= at(r_msa, ls + 1);
        const int32_t fv = rest ? at(r_lb, ls + 1) : 0;
        const int32_t *const row1 = tb.opt + e1 + lane;  // at column m
        const opt_ptr op = (opt_ptr)(uint64_t)ch.opt4 + max(s, 0) * K4;
        i32x4 o4[TOPT];
#pragma unroll
        for (int32_t j = 0; j < TOPT; ++j) o4[j] = op[j];  // xbar, r(F)+r(B), need1, 4 xbar

        // the loads of row (s+1, t): the window's pieces of other workgroups; without a window
        // the right operand's word and the first options'
        const bool wait = !flat && (need_os || !closed);
        constexpr int32_t NV = NW ? (NH ? NH : 1) : TOPT + 1;
        int32_t wv[NV];
        auto get = [&]() -> bool {
            int32_t bad = 0;
            if constexpr (NW > 0) {
#pragma unroll
                for (int32_t k = 0; k < NH; ++k)
                    if (k >= k0) bad |= wv[k] = ld_dev(row1 - 64 * (NH - k));
            } else {
                // (a scalar base and a 32-bit column)
                const int32_t *const row1c = tb.opt + (e1 - mb);
                auto word = [&](int32_t back, bool want) {
                    return want && m >= back ? ld_dev(row1c + (uint32_t)(m - back)) : DINF;
                };
                bad |= wv[TOPT] = word(x1, need_os);
#pragma unroll
                for (int32_t j = 0; j < TOPT; ++j) bad |= wv[j] = word(o4[j].x, !closed && m >= o4[j].z);
            }
            return __any(bad < 0);
        };
        auto finish = [&](bool again) {
            if (again) {
                settle(get);
                if (dead)
#pragma unroll
                    for (int32_t &v : wv) v = v < 0 ? DINF : v;
            }
#pragma unroll
            for (int32_t &v : wv) v &= DINF;  // (the mark)
        };
        const bool again = wait && get();
        // row s+1's ap and row s+2's os, after the loads they would otherwise hold up
        if (need_os) __builtin_nontemporal_store(a_prev, tb.ap + e1 + lane);
        if (n_in > 1) __builtin_nontemporal_store(os_prev, tb.os + e2 + lane);

        const int32_t *const as = aps + (tri(lsc, 0) * 64 + lane);
        int32_t b0 = DINF;
        if (!closed) {
            if constexpr (!DIAG) b0 = cells[(ls * TB + lt) * 64 + lane];
            if (DIAG && rest) wait_waves(ls, lt, ls);
            // splits inside block S, but for i = s + 1; in pieces whose reads are all in flight
            // (splits past the last have an infinite right operand)
            auto piece = [&](auto u0, auto u1) {
                if (decltype(u0)::value <= n_in)
#pragma unroll
                    for (int32_t u = decltype(u0)::value; u < decltype(u1)::value; u += 2)
                        b0 = min(min(b0, as[(u - 1) * 64] + os[u - 1]), as[u * 64] + os[u]);
            };
            piece(std::integral_constant<int, 2>{}, std::integral_constant<int, 8>{});
            piece(std::integral_constant<int, 8>{}, std::integral_constant<int, TB>{});
        }
#pragma unroll
        for (int32_t u = TB - 1; u > 1; --u) os[u] = os[u - 1];
        finish(again);
        if constexpr (NW > 0) {
            if (flat) {  // (columns left of 0 stay infinite: a flat row has none here, no row may)
#pragma unroll
                for (int32_t k = 0; k < NW; ++k)
                    if (!DIAG || k >= k0) wn[64 * k] = fv;
            } else if (wait) {
#pragma unroll
                for (int32_t k = 0; k < NH; ++k)
                    if (k >= k0) wn[64 * k] = wv[k];
            }
            __builtin_amdgcn_wave_barrier();
            os[1] = os_prev = wm[-x1];
        } else {
            os[1] = os_prev = flat ? fv : wv[TOPT];
        }
        last(os_prev, ls + 1, end_os);
        if (!need_os) os[1] = DINF;
        if (ls < 0) break;
        bool only1;  // no split reaches the value
        if (closed) {
            best = lb;
            only1 = !rest || at(r_P1, ls) > 0;  // splits cost at least lb + r(F_s^0)
        } else {
            b0 = min(b0, as[0] + os[1]);  // the splits; best: case 1
            best = DINF;
            // case 1
            const bool all = mb >= at(r_need1max, ls);
            for (int32_t o = 0;;) {
                int32_t v[TOPT];
#pragma unroll
                for (int32_t j = 0; j < TOPT; ++j)
                    if constexpr (NW > 0) v[j] = *(const int32_t *)((const char *)wm - o4[j].w) + o4[j].y;
                    else v[j] = (flat ? fv : wv[j]) + o4[j].y;
                if (!all)
#pragma unroll
                    for (int32_t j = 0; j < TOPT; ++j) v[j] = m >= o4[j].z ? v[j] : DINF;
#pragma unroll
                for (int32_t j = 0; j < TOPT; j += 2) best = min(min(best, v[j]), v[j + 1]);
                if ((o += TOPT) >= K4) break;
#pragma unroll
                for (int32_t j = 0; j < TOPT; ++j) o4[j] = op[o + j];
                if constexpr (NW == 0) finish(wait);
            }
            // splits inside block T: each costs at least lb(s,t) + P(s, T0+1)
            bool left = false;  // splits left out could reach the value
            if constexpr (!DIAG) {
                const int32_t bound = lb + at(r_PT, ls);
                if (lt > 0 && __any(min(best, b0) > bound)) {
                    wait_waves(0, lt, ls);
                    const int32_t *const ac = cells + (ls * TB * 64 + lane);
                    auto piece = [&](auto v0, auto v1) {
                        if (decltype(v0)::value < lt)
#pragma unroll
                            for (int32_t v = decltype(v0)::value; v < decltype(v1)::value; ++v)
                                b0 = min(b0, ac[v * 64] + ost[v]);
                    };
                    piece(std::integral_constant<int, 0>{}, std::integral_constant<int, 8>{});
                    piece(std::integral_constant<int, 8>{}, std::integral_constant<int, TB - 1>{});
                } else {
                    left = lt > 0 && best == bound;
                }
            }
            only1 = best < min(b0, DINF) && !left;
            best = min(min(best, b0), DINF);
        }
        st_dev(only1 ? best | ONLY_CASE1 : best, tb.opt + e0 + lane);
        if constexpr (NW > 0) wn[64 * NH] = best;
        a_prev = m >= at(r_need2, ls) ? min(at(r_P, ls) + best, DINF) : DINF;
        last(a_prev, ls, end_a);
        // (lt = 15 has no such left operand: its word is the next row's first, ap(s+1, s+1).  Either the wait
        // above has seen all other waves past that row, or this cell is closed and with it, msa never
        // falling in t nor rising in s, every cell of that row: then nobody reads the word.)
        if constexpr (DIAG) aps[tri(ls, n_in) * 64 + lane] = a_prev;
        else cells[(ls * TB + lt) * 64 + lane] = a_prev;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        if (lane == 0) __hip_atomic_store(&prog[lt], TB - ls, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        e2 = e1;
        e1 = e0;
        e0 -= (int64_t)(L - s) * stride32;
    }
    __builtin_nontemporal_store(os_prev, tb.os + e1 + lane);  // row S0
    summarize();
    answer(best);
}

// Tiles of equal sides, the fewest that hold L blocks: 17 blocks are two of 9, not 16 and 1 (a
// workgroup takes as long for one end as for 16, and a tile's rows follow one another).
static int32_t tile_side(int32_t L)
{
    const int32_t nb = (L + TB - 1) / TB;
    return (L + nb - 1) / nb;
}

// Two tiles of 9-12 blocks leave a third of the waves idle, which shows where the budgets are so many that
// neither launches nor the schedule (faster with this fill's marks) count.  Fill by diagonals -> by
// tiles, shifts of up to a few thousand columns, 1 to 20 options: 17 blocks x 50001 budgets 154-255 ->
// 181-249 us, x 100001 233-378 -> 305-428 us, x 300001 0.54-0.87 -> 0.81-1.15 ms; 20 x 100001 295-477 -> 349-493
// us, x 300001 0.70-1.11 -> 0.93-1.32 ms; 24 x 100001 391-675 -> 421-654 us, x 300001 0.99-1.71 -> 1.14-1.78 ms;
// 26 blocks and more: tiles as fast or faster, but for single options (at 33 x 300001 2.20 -> 2.49 ms).
// Columns past storing everything don't count, tiles write them faster (24 x 200001, small shifts: 333 -> 178 us).
bool tiles_pay(const DevChain &ch, int32_t W)
{
    const int32_t side = tile_side(ch.L);
    if (ch.L <= TB || ch.L > 2 * TB || side > 12) return true;
    const int64_t open = (int64_t)ch.h_msa[row_of(ch.L, 0, ch.L - 1)] + ch.reach;
    return std::min<int64_t>(W, open) < 50000 * (side - 7);
}

hipError_t launch_tiles(const DevChain &ch, const Tables &tb, int32_t m_ans, hipStream_t stream, int32_t *launches)
{
    const int32_t side = tile_side(ch.L);
    const int32_t nb = (ch.L + side - 1) / side, n_chunks = (tb.W + 63) / 64;
    // Case 1 reads its row at K shifts.  Staged in LDS that costs a load per 64 columns of reach
    // and cell, unstaged one per option (and one for the right operand), four at a time.  Reach 190
    // (staged) and 195 (not): 40 blocks x 4001 budgets with 2 options 128 and 145 us, with 24 147 and
    // 247 us, 128 blocks with 5 options 681 and 855 us, with 24 774 and 1249 us.  So the line lies too low
    // at any number of options; wider windows (4 KB a piece of the 160 KB LDS) are not built.
    const int32_t nw = ch.reach <= 64 * (TWIN - 1) ? 1 + (ch.reach + 63) / 64 : 0;
    // chunks per entry of the summaries (0: no pads to keep them in)
    const int32_t cpe = tb.padl >= 64 ? (n_chunks + SUM_GROUPS - 1) / SUM_GROUPS : 0;
    using Kernel = void (*)(DevChain, Tables, int32_t, int32_t, int32_t, int32_t, int32_t, int32_t, int32_t);
    static const Kernel kernels[3][TWIN + 1] = {
        {k_tile<true, 0, false>, k_tile<true, 1, false>, k_tile<true, 2, false>, k_tile<true, 3, false>, k_tile<true, 4, false>},
        {k_tile<false, 0, false>, k_tile<false, 1, false>, k_tile<false, 2, false>, k_tile<false, 3, false>,
         k_tile<false, 4, false>},
        {k_tile<false, 0, true>, k_tile<false, 1, true>, k_tile<false, 2, true>, k_tile<false, 3, true>, k_tile<false, 4, true>}};
    static_assert(TWIN == 4, "one kernel per window width");
    hipLaunchKernelGGL(k_tile_init, dim3((uint32_t)n_rows(ch.L)), dim3(256), 0, stream, tb, ch.msa, ch.reach, nb);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    for (int32_t level = 0; level < nb; ++level) {
        const dim3 grid(chunk_grid(n_chunks, nb - level));
        // tiles in closed form are left early where that lets other workgroups start; where all run at
        // once their stores would only come first (128 blocks x 2001 budgets 423 -> 428 us with it)
        const int32_t flat_reach = grid.x > 256 ? ch.reach : 1 << 30;
        hipLaunchKernelGGL(kernels[level == 0 ? 0 : side < TB ? 1 : 2][nw], grid, dim3(TB * 64), 0, stream, ch, tb, level, side, n_chunks,
                           ch.reach, flat_reach, cpe, m_ans);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    *launches = nb + 1;
    return hipSuccess;
}

}  // namespace rk
