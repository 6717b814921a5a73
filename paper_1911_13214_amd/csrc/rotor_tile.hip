// 4 x 4 tiles of pairs (Theorem 1, Section 4.2 of Beaumont et al., arXiv
// 1911.13214): the streamed order of small tables, tile-diagonal by
// tile-diagonal, and the diagonal blocks and edges of the blocked order.  The
// recurrence, the value paths and the saturated budgets are described at the
// head of rotor_fill.hip.
//
// Stages are cut into groups of 4; tile (R, C) holds the pairs (s, t) with s
// in group R and t in group C.  triangle_kernel fills the diagonal tiles
// (R, R), leaves included; then one launch of tile_kernel per C - R = 1, 2,
// ... fills the others, so a chain of L stages takes ceil(L / 4) dependent
// launches, and one more per further window of budgets where the chain's sizes
// are large against them (Window).  The splits k of a tile's cells fall in
//   middle  k in [4R + 4, 4C]: both operands in finished tiles, the same range
//           for every cell: a 4 x 4 register product, 8 loads per 16
//           candidates, on packed keys.  All but the first and last four (the
//           rim) read no tile of the tile-diagonal before: these inner splits
//           are taken one launch ahead by workgroups of their own;
//   low     k in [s, 4R + 3]: X in the diagonal tile R, Y a cell of the same
//           tile further down;
//   high    k in [4C + 1, t - 1]: X a cell of the same tile to the left, Y in
//           the diagonal tile C.
// Low and high splits (at most 6 per cell) and C_2 are taken row by row from
// the tile's bottom row up, left to right in a row: a row's cells meet as X
// in registers (same budget), and the rows above read them, shifted by the one w_a
// their row is always shifted by, from LDS, with one barrier per row.
// Measured on MI355X against one launch per t - s: L = 50, M = 500 202 -> 156 us,
// L = 339, M = 500 5.7 -> 2.0 ms.  A launch is bound by the finishing wave's
// dependent loads and about 2,500 instructions (8 to 12 us) and, in the middle
// levels of long chains and in batches, by bytes: L = 1001, M = 100 reads 2.6 per
// candidate past the L2 and moves 5.0 TB/s, 256 chains of L = 64, M = 640 4.9 TB/s
// (a large copy 4.7).
#include <climits>

#include "rotor_paths.h"

namespace rotor {
namespace {

constexpr int kG = kTileSide;
constexpr int kTileMaxWaves = 10;
constexpr int kPerBlock = kT / kG;  // tiles of a 16 x 16 block, each way
// tile-diagonals from this one on have middle splits besides the rim
constexpr int kInnerLevel = 3;
// Middle candidates as one key, value * 2^S + (k - first split of the run):
// the minimum is the smallest value and, among equal values, the smallest
// split.  A range longer than 2^S splits goes in runs of 2^S.
//
// 32 bits, for chains and block-diagonals with S = pbits >= kMinKeyBits; an
// infinite operand (all ones) stays all ones under the rotation and the
// saturating adds.
constexpr int kMinKeyBits = 4;
struct Key32 {
    typedef Narrow P;
    typedef uint32_t K;
    static constexpr int kPer = 2;  // splits relaxed together (one three-way minimum per pair)
    __device__ static K far() { return kInf32; }
    __device__ static K add(uint64_t prefix, int off, bool ok, int S)
    {
        return ok ? ((uint32_t)prefix << S) | (uint32_t)off : kInf32;
    }
    __device__ static K x(uint32_t v, K a, int S) { return sat_add(rot_left(v, S), a); }
    __device__ static K y(uint32_t v, int S) { return rot_left(v, S); }
    __device__ static void relax(K &k, K x, K y) { k = min(k, sat_add(x, y)); }
    // the result of a key: offset 0 is s' = first, offsets from `jump` on
    // `skip` further (jump = 0: none)
    __device__ static Narrow::Acc acc(K key, int S, int first, int jump, int skip, uint64_t prefix)
    {
        Narrow::Acc a;
        a.val = key == kInf32 ? kInf32 : (key >> S) + (uint32_t)prefix;
        const int off = (int)(key & ((1u << S) - 1u));
        a.sp = (uint32_t)(first + off + (jump > 0 && off >= jump ? skip : 0));
        return a;
    }
};

// Exact doubles, for every other block-diagonal: costs are below 2^44, so
// with S = 9 keys stay below 2^53.
constexpr int kKey64Bits = 9;
template <class Path>
struct Key64 {
    typedef Path P;
    typedef double K;
    static constexpr int kPer = 1;
    __device__ static K far() { return __builtin_inf(); }
    __device__ static K add(uint64_t prefix, int off, bool ok, int)
    {
        return ok ? (double)((prefix << kKey64Bits) + (uint64_t)off) : __builtin_inf();
    }
    __device__ static K x(typename P::Raw v, K a, int) { return __builtin_ldexp((double)v, kKey64Bits) + a; }
    __device__ static K y(typename P::Raw v, int) { return __builtin_ldexp((double)v, kKey64Bits); }
    __device__ static void relax(K &k, K x, K y) { k = min_f64(k, x + y); }
    __device__ static typename P::Acc acc(K key, int, int first, int jump, int skip, uint64_t prefix)
    {
        // below the least infinite sum: 2^32 - 1 as a value, or 2^53
        const double bound = P::kShadow ? 4294967295.0 * 512.0 : 9007199254740992.0;
        typename P::Acc a;
        P::init(a);
        if (key < bound) {
            const double q = __builtin_floor(key * (1.0 / 512.0));
            const uint64_t v = (uint64_t)q + prefix;
            const int off = (int)(key - q * 512.0);
            const uint32_t sp = (uint32_t)(first + off + (jump > 0 && off >= jump ? skip : 0));
            P::merge_later(a, P::kShadow ? (int64_t)((v << 32) | sp) : (int64_t)((v << 16) | sp));
        }
        return a;
    }
};

// Budgets of one pass over a tile: W from w0 on, 64 per wave, stored from
// `from` on.  A row's cells at budget m need the rows below at no more than m
// and no less than m - reach (the chain's reach: the largest sum of shifts
// down through the rows of a tile).  Where the reach is no more than `halo`, a
// tile's windows overlap by that much: a window computes its first halo budgets
// a second time, finds what it stores in itself and waits for no other, so all
// windows of a tile are filled in one launch.  Elsewhere the windows lie side by
// side, each one launch after the one below, and read what lies below them
// back from the tables.
struct Window {
    int W, halo, w0, from;
    bool back;  // what lies below w0 is read back
    int at;     // this lane's place in the window
    int m;      // its budget, w0 + at
    int mc;     // the budget it loads, at most M
};

// Fold in the stored() form of a result over any other splits.
template <class P>
__device__ __forceinline__ void merge_any(typename P::Acc &a, int64_t other)
{
    if constexpr (P::kShadow) {
        const uint64_t own = (uint64_t)P::stored(a);
        const uint64_t least = umin(own, (uint64_t)other);
        a.val = (uint32_t)(least >> 32);
        a.sp = (uint32_t)least;
    } else {
        P::merge_later(a, other);
    }
}

// Fold in a candidate of a smaller split than any met so far: ties go to it.
template <class P>
__device__ __forceinline__ void relax_earlier(typename P::Acc &a, typename P::X x, typename P::Y y, uint32_t sp)
{
    if constexpr (P::kShadow) {
        const uint32_t v = sat_add(x, y);
        const bool b = v <= a.val;
        a.val = b ? v : a.val;
        a.sp = b ? sp : a.sp;
    } else {
        P::relax(a, x, y, sp);
    }
}

// A finished row of a tile in LDS: kG cells side by side per budget, so that
// a lane writes and reads them as whole 16-byte words.
template <class P>
struct alignas(16) RowCells {
    typename P::Raw v[kG];
};

// The row `row` of the tile (cells t0 .. t0 + last, further columns repeat the
// last), as written to `buf`, at budgets w below the lane's: from LDS, or
// back from the tables where that is below the window.  A lane whose budget
// lies below w gets another cell of the row.
template <class P>
__device__ __forceinline__ RowCells<P> read_row(const RowCells<P> *buf, const Window &wn, int w, const int64_t *tab,
                                                const uint32_t *shadow, int64_t row, int last, int64_t pitch)
{
    const int idx = wn.at - w;
    RowCells<P> c = buf[max(idx, 0)];
    if (wn.back && idx < 0) {
#pragma unroll
        for (int j = 0; j < kG; ++j) {
            const int64_t o = (row + min(j, last)) * pitch;
            c.v[j] = P::load(tab + o, shadow + o, max(wn.mc - w, 0));
        }
    }
    return c;
}

template <class P>
__device__ __forceinline__ typename P::Raw inf_raw()
{
    if constexpr (P::kShadow)
        return kInf32;
    else
        return kInf;
}

// The final cell from its C_1 result: infinite below m_none (gate = false),
// C_2 where it is within reach (all_ok) and less.
template <class P>
struct FinalCell {
    typename P::Raw v;  // as the path loads it
    int16_t d;
    __device__ __forceinline__ FinalCell(typename P::Acc a, bool gate, bool all_ok, typename P::Raw c2, uint64_t ufub)
    {
        if constexpr (P::kShadow) {
            const uint32_t c1 = gate ? a.val : kInf32;
            const uint32_t c = all_ok ? sat_add(c2, (uint32_t)ufub) : kInf32;
            v = min(c, c1);
            d = v == kInf32 ? (int16_t)-1 : c < c1 ? (int16_t)0 : (int16_t)a.sp;
        } else {
            if (!gate)
                P::init(a);
            if (all_ok)
                P::relax_all(a, c2, ufub);
            const bool fin = P::finite(a);
            v = fin ? P::value(a) : kInf;
            d = !fin ? (int16_t)-1 : P::split(a) == kAllSplit ? (int16_t)0 : (int16_t)P::split(a);
        }
    }
    __device__ __forceinline__ FinalCell(typename P::Raw v_, int16_t d_) : v(v_), d(d_) {}
    __device__ __forceinline__ int64_t cost() const
    {
        if constexpr (P::kShadow)  // the infinity's low half is all ones already
            return (int64_t)(v | (uint64_t)(v == kInf32 ? 0x7FFFFFFFu : 0u) << 32);
        else
            return v;
    }
};

// Row pointers of the tables at cell (s, t0), advanced column by column.
struct RowStores {
    char *cost, *dec, *shadow;
    int64_t pitch;
    __device__ __forceinline__ RowStores(int64_t *tab, int16_t *dtab, const ChainWork &cw, int64_t row, int64_t pitch_)
        : cost((char *)(tab + row * pitch_)), dec((char *)(dtab + row * pitch_)),
          shadow((char *)(cw.shadow + row * pitch_)), pitch(pitch_)
    {
    }
    __device__ __forceinline__ void next()
    {
        cost += pitch * 8;
        dec += pitch * 2;
        shadow += pitch * 4;
    }
    // as store_cell: non-temporal where the fill never reads the cell back
    template <class P>
    __device__ __forceinline__ void store(const FinalCell<P> &f, uint32_t m) const
    {
        typedef __attribute__((address_space(1))) int64_t *g64;
        typedef __attribute__((address_space(1))) int16_t *g16;
        typedef __attribute__((address_space(1))) uint32_t *g32;
        const g64 c = (g64)(cost + m * 8u);
        const g16 d = (g16)(dec + m * 2u);
        if constexpr (P::kShadow) {
            __builtin_nontemporal_store(f.cost(), c);
            __builtin_nontemporal_store(f.d, d);
            *(g32)(shadow + m * 4u) = f.v;
        } else {
            *c = f.cost();
            *d = f.d;
        }
    }
};

// Addresses of the operands of tile (s0 .., t0 ..): rows (s0 + i, k) of X and
// (k + 1, t0 + j) of Y (columns past L: column L) for a split k.
template <class P>
struct TileRows {
    const char *base;
    int64_t rb;      // bytes of a row
    int64_t xd[kG];  // row (s0 + i, k) from row (s0, k)
    int64_t yd[kG];  // row (k + 1, t0 + j) from row (k + 1, t0)
    uint32_t mb;     // byte offset of the lane's budget
    int L, s0, t0;
    __device__ __forceinline__ TileRows(const int64_t *tab, const ChainWork &cw, int L_, int64_t pitch, int s0_, int t0_,
                                        int mc)
        : base(P::table(tab, cw.shadow)), rb(pitch * P::kBytes), mb((uint32_t)mc * P::kBytes), L(L_), s0(s0_), t0(t0_)
    {
        xd[0] = yd[0] = 0;
#pragma unroll
        for (int i = 1; i < kG; ++i) {
            xd[i] = xd[i - 1] + (int64_t)(L - s0 - i + 1) * rb;
            yd[i] = (int64_t)min(i, L - t0) * rb;
        }
    }
    __device__ __forceinline__ const char *x_row(int k) const { return base + row_of(L, s0, k) * rb; }
    __device__ __forceinline__ const char *y_row(int k) const { return base + row_of(L, k + 1, t0) * rb; }
    // w: the shift of Y, w_a^k
    __device__ __forceinline__ void load(typename P::Raw (&x)[kG], typename P::Raw (&y)[kG], const char *xr,
                                         const char *yr, int w) const
    {
        const uint32_t off = shifted_off<P::kBytes>(mb, w);
#pragma unroll
        for (int i = 0; i < kG; ++i)
            x[i] = P::load_off(xr + xd[i], mb);
#pragma unroll
        for (int j = 0; j < kG; ++j)
            y[j] = P::load_off(yr + yd[j], off);
    }
};

template <class Key>
struct TileKeys {
    typename Key::K k[kG][kG];
    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int i = 0; i < kG; ++i)
#pragma unroll
            for (int j = 0; j < kG; ++j)
                k[i][j] = Key::far();
    }
    // relax N splits: operands as loaded, a[n] the key term of split n
    template <int N>
    __device__ __forceinline__ void relax(const typename Key::P::Raw (&x)[N][kG], const typename Key::P::Raw (&y)[N][kG],
                                          const typename Key::K (&a)[N], int S)
    {
        typename Key::K xk[N][kG], yk[N][kG];
#pragma unroll
        for (int n = 0; n < N; ++n)
#pragma unroll
            for (int i = 0; i < kG; ++i) {
                xk[n][i] = Key::x(x[n][i], a[n], S);
                yk[n][i] = Key::y(y[n][i], S);
            }
#pragma unroll
        for (int i = 0; i < kG; ++i)
#pragma unroll
            for (int j = 0; j < kG; ++j)
#pragma unroll
                for (int n = 0; n < N; ++n)
                    Key::relax(k[i][j], xk[n][i], yk[n][j]);
    }
};

// Splits ka .. kb of tile (s0 .., t0 ..) folded into acc, with the u_f prefix
// of each row: per split 8 loads and 16 candidates per lane, in steps of
// Key::kPer splits, with AHEAD the operands of the next step loaded before a
// step is relaxed.
template <class Key, bool AHEAD>
__device__ __forceinline__ void tile_splits(typename Key::P::Acc (&acc)[kG][kG], const ChainRows &r,
                                            const ChainWork &cw, const TileRows<typename Key::P> &tr, int ka, int kb,
                                            int S, int mc)
{
    typedef typename Key::P P;
    typedef typename P::Raw Raw;
    typedef typename Key::K K;
    constexpr int N = Key::kPer;
    const char *x = tr.x_row(ka), *y = tr.y_row(ka);
    int64_t ystep = (int64_t)(tr.L - ka - 1) * tr.rb;
    const const_i64 pre = (const_i64)cw.pre;
    const int64_t pre_lo = pre[ka - 1];
    struct Step {
        Raw x[N][kG], y[N][kG];
        int w[N];
        int64_t p[N];
    };
    int k_load = ka;
    auto load = [&](Step &st) {
#pragma unroll
        for (int n = 0; n < N; ++n) {
            st.w[n] = r.wa[k_load - 1];
            st.p[n] = pre[k_load];
            tr.load(st.x[n], st.y[n], x, y, st.w[n]);
            if (k_load < kb) {  // splits past kb load kb again
                ++k_load;
                x += tr.rb;
                y += ystep;
                ystep -= tr.rb;
            }
        }
    };
    TileKeys<Key> keys;
    keys.clear();
    int run = ka;  // split of key offset 0
    auto relax = [&](const Step &st, int k) {
        K a[N];
#pragma unroll
        for (int n = 0; n < N; ++n)
            a[n] = Key::add((uint64_t)(st.p[n] - pre_lo), k + n - run, k + n <= kb && mc >= st.w[n], S);
        keys.relax(st.x, st.y, a, S);
    };
    Step a;
    [[maybe_unused]] Step b;
    if constexpr (AHEAD)
        load(a);
    for (int k = ka; k <= kb; k += 2 * N) {
        if constexpr (AHEAD) {
            load(b);
            relax(a, k);
            if (k + N <= kb) {
                load(a);
                relax(b, k + N);
            }
        } else {
            load(a);
            relax(a, k);
            if (k + N <= kb) {
                load(a);
                relax(a, k + N);
            }
        }
        if (k + 2 * N - run >= 1 << S || k + 2 * N > kb) {
#pragma unroll
            for (int i = 0; i < kG; ++i) {
                const uint64_t pfx = (uint64_t)(pre_lo - pre[tr.s0 + i - 1]);
#pragma unroll
                for (int j = 0; j < kG; ++j)
                    P::merge_later(acc[i][j], P::stored(Key::acc(keys.k[i][j], S, run + 1, 0, 0, pfx)));
            }
            keys.clear();
            run = k + 2 * N;
        }
    }
}

// The middle splits of a tile that read the tile-diagonal before its own: the
// first kG of the range [k_lo, k_hi] (Y in tile (R + 1, C)) and the last kG (X
// in tile (R, C - 1)), or the whole range where it is no longer than that.
// Key offsets 0 .. 3 and 4 .. 7.
template <class Key>
struct TileRim {
    typedef typename Key::P P;
    struct Half {
        typename P::Raw x[kG][kG], y[kG][kG];
        int w[kG];
    };
    int k_lo, k_hi, k2;  // offset o is split k_lo + o, or k2 + o from offset kG on
    __device__ __forceinline__ TileRim(int lo, int hi) : k_lo(lo), k_hi(hi), k2(max(lo + kG, hi - kG + 1) - kG) {}
    __device__ __forceinline__ int split(int o) const { return (o < kG ? k_lo : k2) + o; }
    template <int H>
    __device__ __forceinline__ void load(Half &a, const ChainRows &r, const TileRows<P> &tr) const
    {
        int k = min(split(H * kG), k_hi);
        const char *x = tr.x_row(k), *y = tr.y_row(k);
        int64_t ystep = (int64_t)(tr.L - k - 1) * tr.rb;
#pragma unroll
        for (int n = 0; n < kG; ++n) {
            a.w[n] = r.wa[k - 1];
            tr.load(a.x[n], a.y[n], x, y, a.w[n]);
            const bool more = k < k_hi;
            k += more ? 1 : 0;
            x += more ? tr.rb : 0;
            y += more ? ystep : 0;
            ystep -= tr.rb;
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    template <int H>
    __device__ __forceinline__ void relax(TileKeys<Key> &keys, const Half &a, const const_i64 pre, int S, int mc) const
    {
        typename Key::K add[kG];
#pragma unroll
        for (int n = 0; n < kG; ++n) {
            const int k = split(H * kG + n);
            add[n] = Key::add((uint64_t)(pre[min(k, k_hi)] - pre[k_lo - 1]), H * kG + n, k <= k_hi && mc >= a.w[n], S);
        }
        keys.relax(a.x, a.y, add, S);
    }
};

// Meet the workgroup with this wave's LDS accesses done; its global accesses
// may be under way (a plain barrier: __syncthreads would wait for them).
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Values that every lane needs, one per lane of a vector loaded once.
__device__ __forceinline__ int32_t lane_of(int32_t v, int l) { return __builtin_amdgcn_readlane(v, l); }
__device__ __forceinline__ uint64_t lane_of64(int64_t v, int l)
{
    return (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, l) |
           (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)v >> 32), l) << 32;
}

// Whether every cell of the tile is saturated at every budget from `base` on
// (G(s, t) falls as s grows, so the tile's first row has the largest).
__device__ inline bool tile_saturated(const ChainRows &r, const ChainWork &cw, int L, int s0, int t0, int base)
{
    const const_i32 gsat = (const_i32)cw.gsat + row_of(L, s0, t0);
    const int last = min(kG, L - t0 + 1) - 1;
    int32_t g = gsat[0];
    bool pos = true;
#pragma unroll
    for (int j = 0; j < kG; ++j) {
        g = max(g, gsat[min(j, last)]);
        pos = pos && r.uf[s0 + j - 1] > 0;
    }
    return pos && base >= g;
}

// Inner results at the budgets that a second window computes again (the first
// halo of every window but the first) are kept twice: in the cost slots, which
// the window that stores those cells overwrites, and for the three lower rows
// in the workspace's 2-byte section, which the tiles have no other use for: a
// slice of 64 of its rows per row group, half of it for each parity of the
// tile-diagonal.  Budgets come in waves of 64.
__device__ inline int halo_place(int base, int W, int halo)
{
    const int per = (W - halo) >> 6, own = halo >> 6;
    const int q = base >> 6, v = q / per, x = q - v * per;
    return v > 0 && x < own ? ((v - 1) * own + x) * 64 : -1;
}
constexpr int kHaloRows = (kG - 1) * kG;
constexpr int kHaloSlice = kG * kT;  // rows of the 2-byte section per row group
// places of a row's halos: room for halos of up to 2/3 of W - halo
__device__ inline int64_t halo_pitch_of(const ChainWork &cw) { return cw.hpitch * 2 / 3 / 64 * 64; }
static_assert(2 * kHaloRows * 2 * sizeof(int64_t) <= 3 * kHaloSlice * sizeof(int16_t), "both parities in a slice");
// the row groups of tiles off the diagonal are all but the last
constexpr bool slices_fit()
{
    for (int L = kBlock + 1; L <= 8 * kBlock; ++L)  // both sides grow alike
        if ((int64_t)((L + kG - 1) / kG - 1) * kHaloSlice > half_rows_of(L))
            return false;
    return true;
}
static_assert(slices_fit(), "a chain's slices in its part of the section");
__device__ inline int64_t *halo_of(const ChainWork &cw, int R, int level)
{
    return (int64_t *)(cw.half + (int64_t)R * (kHaloSlice * cw.hpitch)) +
           (level & 1) * (kHaloSlice * sizeof(int16_t) / sizeof(int64_t) / 2 * cw.hpitch);
}

// tile_inner's part for the edges of the blocked order: the splits of a tile of
// block (I, J) inside the block, less the rim, k in [4R + 8, 16I + 15] and [16J + 1,
// 4C - 4], and between them the middle products' result: a packed key in the
// cell's compact copy, or the path's stored() form in its cost slot, counting
// u_f from stage 16I + 16 on.
template <class Key>
__device__ __forceinline__ void edge_splits(typename Key::P::Acc (&acc)[kG][kG], const ChainRows &r,
                                            const ChainWork &cw, const TileRows<typename Key::P> &tr, int L,
                                            int64_t pitch, const int64_t *tab, int last, int S, int mc)
{
    typedef typename Key::P P;
    const int I = (tr.s0 - 1) / kT, J = (tr.t0 - 1) / kT;
    const int k_lo = (I + 1) * kT, k_hi = J * kT;  // the middle range
    const bool packed = P::kShadow && middle_packed(cw, J - I, k_hi - k_lo);
    const int Sm = k_hi > k_lo ? 32 - __clz(k_hi - k_lo) : 0;
    const const_i64 pre = (const_i64)cw.pre;
    const int64_t pre_lo = pre[k_lo - 1];
    constexpr bool kAheadE = sizeof(typename Key::K) == 4;  // registers
#pragma unroll
    for (int i = 0; i < kG; ++i)
#pragma unroll
        for (int j = 0; j < kG; ++j)
            P::init(acc[i][j]);
    if (tr.s0 + 2 * kG - 1 < k_lo)
        tile_splits<Key, kAheadE>(acc, r, cw, tr, tr.s0 + 2 * kG - 1, k_lo - 1, S, mc);
    if (packed) {
#pragma unroll
        for (int i = 0; i < kG; ++i) {
            const uint32_t *p = cw.shadow + row_of(L, tr.s0 + i, tr.t0) * pitch;
            const uint64_t pfx = (uint64_t)(pre_lo - pre[tr.s0 + i - 1]);
#pragma unroll
            for (int j = 0; j < kG; ++j) {
                const uint32_t key = load32(p, mc);
                const uint32_t split = (uint32_t)(k_lo + 1) + (key & ((1u << Sm) - 1u));
                P::merge_stored(acc[i][j], (int64_t)((uint64_t)(key == kInf32 ? kInf32 : key >> Sm) << 32 | split), pfx);
                p += j < last ? pitch : 0;
            }
        }
    } else {
#pragma unroll
        for (int i = 0; i < kG; ++i) {
            const int64_t *p = tab + row_of(L, tr.s0 + i, tr.t0) * pitch;
            const uint64_t pfx = (uint64_t)(pre_lo - pre[tr.s0 + i - 1]);
#pragma unroll
            for (int j = 0; j < kG; ++j) {
                P::merge_stored(acc[i][j], load64(p, mc), pfx);
                p += j < last ? pitch : 0;
            }
        }
    }
    if (k_hi + 1 < tr.t0 - kG)
        tile_splits<Key, kAheadE>(acc, r, cw, tr, k_hi + 1, tr.t0 - 1 - kG, S, mc);
}

// The inner middle splits [ka, kb] of tile (R, C) at the budgets of a
// workgroup, left in the cost slots of its cells in the path's stored() form.
// Waves hold 64 budgets each; n_kw waves of the same budgets take a part of
// the splits each, and their minima meet in LDS.  EDGE: edge_splits instead
// (n_kw = 1).
template <class Key, bool EDGE>
__device__ __forceinline__ void tile_inner(const ChainRows &r, const ChainWork &cw, int L, int M, int64_t pitch, int R,
                                           int C, int S, int m, int at, int W, int n_kw, int kw, int64_t *tab,
                                           int64_t *halo, int64_t halo_pitch, int W_T, int halo_T, char *lds)
{
    typedef typename Key::P P;
    typedef typename P::Acc Acc;
    const int s0 = R * kG + 1, t0 = C * kG + 1;
    const int last = min(kG, L - t0 + 1) - 1;
    const int mc = min(m, M);
    const bool works = __builtin_amdgcn_readfirstlane(m) <= M &&
                       !tile_saturated(r, cw, L, s0, t0, __builtin_amdgcn_readfirstlane(m));
    Acc acc[kG][kG];
#pragma unroll
    for (int i = 0; i < kG; ++i)
#pragma unroll
        for (int j = 0; j < kG; ++j)
            P::init(acc[i][j]);
    if constexpr (EDGE) {
        if (works) {
            const TileRows<P> tr(tab, cw, L, pitch, s0, t0, mc);
            edge_splits<Key>(acc, r, cw, tr, L, pitch, tab, last, S, mc);
        }
    } else if (works) {
        const int lo = s0 + 2 * kG - 1, hi = t0 - 1 - kG;
        const int chunk = (hi - lo + n_kw) / n_kw;
        const int ka = lo + kw * chunk, kb = min(hi, ka + chunk - 1);
        if (ka <= kb) {
            const TileRows<P> tr(tab, cw, L, pitch, s0, t0, mc);
            tile_splits<Key, true>(acc, r, cw, tr, ka, kb, S, mc);
        }
    }
    unsigned long long *const part = (unsigned long long *)lds + at;
    if (n_kw > 1) {
        if (kw == 0) {
#pragma unroll
            for (int i = 0; i < kG; ++i)
#pragma unroll
                for (int j = 0; j < kG; ++j)
                    part[(i * kG + j) * W] = (unsigned long long)P::stored(acc[i][j]);
        }
        __syncthreads();
        if (kw != 0 && works) {
#pragma unroll
            for (int i = 0; i < kG; ++i)
#pragma unroll
                for (int j = 0; j < kG; ++j)
                    atomicMin(&part[(i * kG + j) * W], (unsigned long long)P::stored(acc[i][j]));
        }
        __syncthreads();
    }
    if (kw == 0 && works && m <= M) {
        // a copy for the window that computes these budgets a second time,
        // whose cells may be final before it reads them
        int64_t *copy = halo;
        if (copy) {
            const int x = halo_place(m - at % 64, W_T, halo_T);
            copy = x >= 0 ? copy + x + at % 64 : nullptr;
        }
#pragma unroll
        for (int i = 0; i < kG; ++i) {
            const int64_t row = row_of(L, s0 + i, t0);
#pragma unroll
            for (int j = 0; j < kG; ++j) {
                const int64_t v = n_kw > 1 ? (int64_t)part[(i * kG + j) * W] : P::stored(acc[i][j]);
                if (j <= last)
                    tab[(row + j) * pitch + m] = v;
                if (i > 0 && copy)
                    copy[((i - 1) * kG + j) * halo_pitch] = v;
            }
        }
    }
}

// One window of tile (R, C), C > R: the splits of its cells that tile_inner
// did not take, C_2, the gates, the final cells.  Bound by latency and, from
// about five waves in a workgroup on, by instruction issue: the scalars of the
// tile come in two vector loads, then the operands in two batches.  has_inner:
// tile_inner has left its results.
template <class Key, bool INNER>
__device__ __forceinline__ void tile_finish(const ChainRows &r, const ChainWork &cw, int L, int M, int64_t pitch,
                                            int R, int C, int S, bool has_inner, const Window &wn, int64_t *tab,
                                            int16_t *dtab, char *lds)
{
    typedef typename Key::P P;
    typedef typename P::Raw Raw;
    typedef typename P::Acc Acc;
    const int s0 = R * kG + 1, t0 = C * kG + 1;
    const int last = min(kG, L - t0 + 1) - 1;  // last column of the tile
    const int m = wn.m, mc = wn.mc;
    const int lane = threadIdx.x & 63;
    // lanes 0-15: m_none of cell (lane / 4, lane % 4), 16-31: the least budget
    // of C_2; 32-35: w_a of stage s0 + i - 1 (the shift of row i as Y), 36-39:
    // w_abar of s0 + i, 40-43: w_a of t0 + j
    int32_t v32;
    {
        const int i = (lane >> 2) & 3, j = lane & 3;
        const int64_t cell = row_of(L, s0 + i, t0) + min(j, last);
        const int32_t *src = lane < 16 ? cw.gnone + cell : cw.gall + cell;
        const int32_t *wa = (const int32_t *)r.wa, *wabar = (const int32_t *)r.wabar;
        if (lane >= 32)
            src = lane < 36 ? wa + max(s0 + j - 2, 0) : lane < 40 ? wabar + (s0 + j - 1) : wa + (min(t0 + j, L) - 1);
        v32 = *src;
        if (lane >= 16 && lane < 32)
            v32 = max(v32, wabar[s0 + i - 1]);
    }
    // lanes 0-3: u_f up to stage s0 + i - 1, 4-7: up to t0 + j; 8-11: u_f + u_b
    // of s0 + i; 12-15: least times' u_f + u_b up to s0 + i - 1, 16-19: up to t0 + j
    int64_t v64;
    {
        const int j = lane & 3;
        const int tj = min(t0 + j, L);
        const int64_t *src = lane < 4 ? cw.pre + (s0 + j - 1)
                             : lane < 8 ? cw.pre + tj
                             : lane < 12 ? r.uf + (s0 + j - 1)
                             : lane < 16 ? cw.preall + (s0 + j - 1)
                                         : cw.preall + tj;
        v64 = *src;
        if (lane >= 8 && lane < 12)
            v64 += r.ub[s0 + j - 1];
    }
    RowCells<P> *const bufs = (RowCells<P> *)lds;
    const int base = __builtin_amdgcn_readfirstlane(m);
    const TileRows<P> tr(tab, cw, L, pitch, s0, t0, mc);
    const TileRim<Key> rim(s0 + kG - 1, t0 - 1);
    const const_i64 pre = (const_i64)cw.pre;
    // waves past M, and waves whose cells are all saturated, relax nothing
    const bool sat = base > M || tile_saturated(r, cw, L, s0, t0, base);
    const bool in = m <= M && m >= wn.from;
    if (sat) {
#pragma unroll 1
        for (int i = kG - 1;; --i) {
            RowStores st(tab, dtab, cw, row_of(L, s0 + i, t0), pitch);
            RowCells<P> c;
#pragma unroll
            for (int j = 0; j < kG; ++j) {
                const FinalCell<P> f((Raw)(lane_of64(v64, 16 + j) - lane_of64(v64, 12 + i)), 0);
                c.v[j] = f.v;
                if (j <= last && in)
                    st.store(f, m);
                st.next();
            }
            if (i == 0)
                return;
            bufs[(i & 1) * wn.W + wn.at] = c;
            lds_barrier();
        }
    }
    Acc acc[kG][kG];
    // operands: X of row i as Y of the rows u above (split k = s0 + i - 1), Y of
    // the high splits, C_2's of the row at hand
    Raw xl[kG][kG], yh[kG][kG];
    RowCells<P> c2;
    // loaded beside the rim where the keys leave registers for it
    constexpr bool kEarly = sizeof(typename Key::K) == 4;
    auto load_operands = [&]() {
        const char *x = tr.base + row_of(L, s0, s0) * tr.rb;  // (s0 + u, s0 + u)
#pragma unroll
        for (int u = 0; u + 1 < kG; ++u) {
#pragma unroll
            for (int i = u + 1; i < kG; ++i)
                xl[u][i] = P::load_off(x + (int64_t)(i - u - 1) * tr.rb, tr.mb);
            x += (int64_t)(L - s0 - u + 1) * tr.rb;
        }
        const char *y = tr.base + row_of(L, t0 + 1, t0 + 1) * tr.rb;  // (t0 + e + 1, t0 + e + 1)
#pragma unroll
        for (int e = 0; e + 1 < kG; ++e) {
            const uint32_t off = shifted_off<P::kBytes>(tr.mb, lane_of(v32, 40 + e));
#pragma unroll
            for (int j = e + 1; j < kG; ++j)
                yh[e][j] = P::load_off(e < last ? y + (int64_t)(min(j, last) - e - 1) * tr.rb : tr.base, off);
            y += (int64_t)(L - t0 - e) * tr.rb;
        }
        const char *p = tr.base + row_of(L, s0 + kG, t0) * tr.rb;
        const uint32_t off = shifted_off<P::kBytes>(tr.mb, lane_of(v32, 39));
#pragma unroll
        for (int j = 0; j < kG; ++j)
            c2.v[j] = P::load_off(p + tr.yd[j], off);
    };
    {
        typename TileRim<Key>::Half a, b;
        TileKeys<Key> keys;
        keys.clear();
        rim.template load<0>(a, r, tr);
        if constexpr (kEarly)
            load_operands();
        rim.template relax<0>(keys, a, pre, S, mc);
        __builtin_amdgcn_sched_barrier(0);
        rim.template load<1>(b, r, tr);
        [[maybe_unused]] int64_t inner[kG][kG];
        auto load_inner = [&]() {
            if (has_inner) {
                const int at = base < wn.from ? halo_place(base, wn.W, wn.halo) : -1;
                const int64_t hp = halo_pitch_of(cw);
#pragma unroll
                for (int i = 0; i < kG; ++i) {
                    // the first row of a halo is not needed
                    const bool copy = i > 0 && at >= 0;
                    const int64_t *q = copy ? halo_of(cw, R, C - R) + (i - 1) * kG * hp + at
                                            : tab + row_of(L, s0 + i, t0) * pitch + base;
                    const int64_t step = copy ? hp : pitch;
#pragma unroll
                    for (int j = 0; j < kG; ++j) {
                        inner[i][j] = load64(q, mc - base);
                        q += j < last ? step : 0;
                    }
                }
            } else {
#pragma unroll
                for (int i = 0; i < kG; ++i)
#pragma unroll
                    for (int j = 0; j < kG; ++j)
                        inner[i][j] = -1;  // all ones: above every stored form
            }
        };
        if constexpr (INNER && kEarly)
            load_inner();
        rim.template relax<1>(keys, b, pre, S, mc);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (!kEarly) {
            if constexpr (INNER)
                load_inner();
            load_operands();
        }
#pragma unroll
        for (int i = 0; i < kG; ++i) {
            const uint64_t pfx = lane_of64(v64, 3) - lane_of64(v64, i);
#pragma unroll
            for (int j = 0; j < kG; ++j) {
                acc[i][j] = Key::acc(keys.k[i][j], S, rim.k_lo + 1, kG, rim.k2 - rim.k_lo, pfx);
                if constexpr (INNER)
                    merge_any<P>(acc[i][j], inner[i][j]);
            }
        }
    }
#pragma unroll
    for (int i = kG - 1; i >= 0; --i) {
        __builtin_amdgcn_sched_barrier(0);
        const int s = s0 + i;
        const int64_t row = row_of(L, s, t0);
        const uint64_t pre_s = lane_of64(v64, i), ufub = lane_of64(v64, 8 + i);
        typename P::X xh[kG];
        RowCells<P> c;
        int16_t d[kG];
#pragma unroll
        for (int j = 0; j < kG; ++j) {
            Acc a = acc[i][j];
#pragma unroll
            for (int e = 0; e < j; ++e)
                P::relax(a, xh[e], P::yop(yh[e][j]), (uint32_t)(t0 + e + 1));
            const FinalCell<P> f(a, mc >= lane_of(v32, i * kG + j), mc >= lane_of(v32, 16 + i * kG + j), c2.v[j], ufub);
            c.v[j] = f.v;
            d[j] = f.d;
            if (j + 1 < kG)
                xh[j] = P::xop(f.v, lane_of64(v64, 4 + j) - pre_s, (uint32_t)(t0 + j + 1), mc >= lane_of(v32, 40 + j));
        }
        RowCells<P> *const buf = bufs + (i & 1) * wn.W;
        RowCells<P> v;
        int w = 0;
        if (i > 0) {
            buf[wn.at] = c;
            lds_barrier();
            // this row as Y of the rows above, and as C_2's operand of the next
            w = lane_of(v32, 32 + i);
            v = read_row<P>(buf, wn, w, tab, cw.shadow, row, last, pitch);
            c2 = read_row<P>(buf, wn, lane_of(v32, 35 + i), tab, cw.shadow, row, last, pitch);
        }
        if (in) {
            RowStores st(tab, dtab, cw, row, pitch);
#pragma unroll
            for (int j = 0; j < kG; ++j) {
                if (j <= last)
                    st.store(FinalCell<P>(c.v[j], d[j]), m);
                st.next();
            }
        }
#pragma unroll
        for (int u = 0; u < i; ++u) {
            const typename P::X x = P::xop(xl[u][i], pre_s - lane_of64(v64, u), (uint32_t)s, mc >= w);
#pragma unroll
            for (int j = 0; j < kG; ++j)
                relax_earlier<P>(acc[u][j], x, P::yop(v.v[j]), (uint32_t)s);
        }
    }
}

// The diagonal tile R: stages s0 .. s0 + last, leaves included (Eq.
// (DP:Init)); every split lies in the tile.  The rows above a row read it
// back shifted (sh), and meet it with their own cells to the left.
template <class P>
__device__ __forceinline__ void triangle_body(const ChainRows &r, const ChainWork &cw, int L, int M, int64_t pitch,
                                              int R, const Window &wn, int64_t *tab, int16_t *dtab, char *lds)
{
    typedef typename P::Acc Acc;
    const int s0 = R * kG + 1;
    const int last = min(kG, L - s0 + 1) - 1;
    const const_i64 pre = (const_i64)cw.pre;
    const const_i32 gall = (const_i32)cw.gall, gnone = (const_i32)cw.gnone;
    const int m = wn.m, mc = wn.mc;
    RowCells<P> sh[kG], c2;
#pragma unroll
    for (int i = kG - 1; i >= 0; --i) {
        if (i > last)
            continue;  // uniform: no such stage
        const int s = s0 + i;
        RowCells<P> *const buf = (RowCells<P> *)lds + (i & 1) * wn.W;
        const int64_t row = row_of(L, s, s);
        const int wab = r.wabar[s - 1];
        const uint64_t ufub = (uint64_t)(r.uf[s - 1] + r.ub[s - 1]);
        typename P::X x[kG];
        RowCells<P> c;
        RowStores st(tab, dtab, cw, row, pitch);
#pragma unroll
        for (int j = i; j < kG; ++j) {
            const int t = s0 + j;
            const int64_t cell = row + min(j, last) - i;
            Acc a;
            P::init(a);
#pragma unroll
            for (int e = i + 1; e <= j; ++e)
                P::relax(a, x[e - 1], P::yop(sh[e].v[j]), (uint32_t)(s0 + e));
            const bool all_ok = mc >= gall[cell] && (j == i || mc >= wab);
            const FinalCell<P> f = j == i ? FinalCell<P>(all_ok ? (typename P::Raw)ufub : inf_raw<P>(),
                                                         all_ok ? (int16_t)0 : (int16_t)-1)
                                          : FinalCell<P>(a, mc >= gnone[cell], all_ok, c2.v[j], ufub);
            if (j + 1 < kG) {
                const int tc = min(t, L);
                x[j] = P::xop(f.v, (uint64_t)(pre[tc] - pre[s - 1]), (uint32_t)(t + 1), mc >= r.wa[tc - 1]);
            }
            c.v[j] = f.v;
            if (j <= last && m <= M)
                st.store(f, m);
            st.next();
        }
        if (i > 0) {
            buf[wn.at] = c;
            lds_barrier();
            // columns below i hold nothing of this row
            sh[i] = read_row<P>(buf, wn, r.wa[s - 2], tab, cw.shadow, row - i, last, pitch);
            c2 = read_row<P>(buf, wn, r.wabar[s - 2], tab, cw.shadow, row - i, last, pitch);
        }
    }
}

// The passes of a workgroup over a tile's budgets from wn.w0 on, in turn;
// body(wn, R) fills one.  R is opaque in each pass, or the compiler computes
// every row address of the tile before the loop and spills them.
template <class F>
__device__ __forceinline__ void for_passes(Window &wn, int M, int passes, int R, F &&body)
{
    for (;;) {
        wn.m = wn.w0 + wn.at;
        wn.mc = min(wn.m, M);
        int tile = R;
        asm volatile("" : "+s"(tile));
        body(wn, tile);
        wn.w0 += wn.W;
        if (--passes == 0 || wn.w0 > M)
            return;
        wn.from = wn.w0;
        wn.back = true;
        __syncthreads();  // the cells below are read back, the LDS rows written again
    }
}

__global__ __launch_bounds__(kTileMaxWaves * 64) void triangle_kernel(const int64_t *__restrict__ params, int L, int M,
                                                                      int64_t pitch, int64_t rows,
                                                                      int64_t *__restrict__ cost,
                                                                      int16_t *__restrict__ dec, Work w)
{
    extern __shared__ __align__(16) char lds[];
    const int c = blockIdx.y;
    const int R = blockIdx.x;
    const ChainRows r = chain_rows(params, w, L, c);
    const ChainWork cw = chain_work(w, L, rows, pitch, c);
    int64_t *tab = cost + (int64_t)c * rows * pitch;
    int16_t *dtab = dec + (int64_t)c * rows * pitch;
    Window wn{(int)blockDim.x, 0, 0, 0, false, (int)threadIdx.x, 0, 0};
    for_passes(wn, M, INT_MAX, R, [&](const Window &wn, int tile) {
        if (cw.narrow(0))
            triangle_body<Narrow>(r, cw, L, M, pitch, tile, wn, tab, dtab, lds);
        else
            triangle_body<Wide>(r, cw, L, M, pitch, tile, wn, tab, dtab, lds);
    });
}

// f(std::integral_constant-like key type) for the key of the tile (R, C)
template <class F>
__device__ __forceinline__ void with_key(const ChainWork &cw, int R, int C, F &&f)
{
    const int bits = cw.pbits[block_diag(R * kG + 1, C * kG + 1)];
    if (bits >= kMinKeyBits)
        f(Key32{}, min(bits, 15));
    else if (bits >= 0)
        f(Key64<Narrow>{}, kKey64Bits);
    else
        f(Key64<Wide>{}, kKey64Bits);
}

// The tiles of one step of a chain: of tile-diagonal `step`, all of them
// (kAllTiles) or those inside the 16 x 16 diagonal blocks (kDiagonalBlocks); or, of
// the blocks (I, I + delta), the tiles a + b = step (kBlockEdges), a groups above
// the block's last and b right of its first.
struct TileSteps {
    TileSet set;
    int groups, delta;
    __host__ __device__ int count(int step) const
    {
        constexpr int B = kPerBlock;
        const int blocks = (groups + B - 1) / B;
        if (set == kAllTiles)
            return groups - step;
        if (set == kDiagonalBlocks)
            return step < B ? blocks * (B - step) : 0;
        return step < 2 * B - 1 ? (blocks - delta) * (step < B ? step + 1 : 2 * B - 1 - step) : 0;
    }
    // tile i of the step; past the chain when C >= groups
    __device__ void at(int step, int i, int &R, int &C) const
    {
        constexpr int B = kPerBlock;
        if (set == kAllTiles) {
            R = i;
            C = i + step;
        } else if (set == kDiagonalBlocks) {
            R = i / (B - step) * B + i % (B - step);
            C = R + step;
        } else {
            const int n = step < B ? step + 1 : 2 * B - 1 - step, I = i / n;
            const int a = max(0, step - B + 1) + (i - I * n);
            R = I * B + B - 1 - a;
            C = (I + delta) * B + step - a;
        }
    }
};

// One launch of a run of tile steps: step `front` is the one whose first window
// is finished.  Its workgroups for one chain, in order:
//   tiles * windows        a window of a tile of step `front` each; of a chain
//                          whose windows lie apart: window v of step front - v
//   next * chunks          the inner splits of a tile of step front + 1 at the
//                          budgets of `chunks` workgroups (not for those chains)
// and for chains whose windows lie apart
//   more * apart           the tiles that window v's step has more than `front`
//   apart_next * apart_chunks * apart   the inner splits of the step after each
//                          window's.
// So the order of chains whose windows overlap, the usual ones, is not
// stretched by the others'.
struct TileLaunch {
    TileSteps steps;
    int front;
    int first, last;  // the steps finished in this run
    int inner_from;   // steps from here on get inner splits
    int W, passes;    // budgets of a pass, passes in turn (where there is one window)
    int halo;         // largest reach of chains with overlapping windows (-1: no chain; INT_MAX: one window)
    int tiles, windows, next, chunks;
    int more, apart, apart_passes, apart_next, apart_chunks;
    int copy_W, copy_halo;  // overlapping windows that will read the inner results (copy_W = 0: none)
    int n_kw;               // waves that share the inner splits of the same budgets
};

// A workgroup either finishes a window of a tile or takes the inner splits of a
// tile of the step that follows, which read tiles of the steps before this one
// only: so that the products, most of the work, run beside the short dependent
// part.  INNER: some step finished has inner splits; WINDOWS: a tile's budgets are
// cut into windows.
template <bool INNER, bool EDGE, bool WINDOWS>
__global__ __launch_bounds__(kTileMaxWaves * 64, 3) void tile_kernel(const int64_t *__restrict__ params, int L, int M,
                                                                  int64_t pitch, int64_t rows, TileLaunch tl,
                                                                  int64_t *__restrict__ cost,
                                                                  int16_t *__restrict__ dec, Work w)
{
    extern __shared__ __align__(16) char lds[];
    const int c = blockIdx.y;
    const ChainRows r = chain_rows(params, w, L, c);
    const ChainWork cw = chain_work(w, L, rows, pitch, c);
    int64_t *tab = cost + (int64_t)c * rows * pitch;
    const int reach = WINDOWS ? cw.reach() : 0;  // here, beside the other scalars: a read further down waits alone
    int v = 0, i, chunk = 0;
    bool finishes = true, apart_only = false;
    int b = blockIdx.x;
    const int windows = WINDOWS ? tl.windows : 1;
    if (b < tl.tiles * windows) {
        v = WINDOWS ? b / tl.tiles : 0;
        i = b - v * tl.tiles;
    } else if ((b -= tl.tiles * windows) < tl.next * tl.chunks || !WINDOWS) {
        finishes = false;
        chunk = b / tl.next;
        i = b - chunk * tl.next;
    } else {
        apart_only = true;
        b -= tl.next * tl.chunks;
        finishes = b < tl.more * tl.apart;
        if (finishes) {
            v = b / tl.more;
            i = b - v * tl.more + tl.tiles;
        } else {
            b -= tl.more * tl.apart;
            const int q = b / tl.apart_next;
            i = b - q * tl.apart_next;
            v = q / tl.apart_chunks;
            chunk = q - v * tl.apart_chunks;
        }
    }
    const bool apart = WINDOWS && reach > tl.halo;
    const int step = tl.front - (apart ? v : 0) + (finishes ? 0 : 1);
    if (step < (finishes ? tl.first : tl.inner_from) || step > tl.last || i >= tl.steps.count(step) ||
        v >= (apart ? tl.apart : windows) || (apart_only ? !apart : apart && !finishes))
        return;
    int R, C;
    tl.steps.at(step, i, R, C);
    if (C >= tl.steps.groups)
        return;
    const int span = tl.W * tl.apart_passes;  // budgets of a window that lies apart
    if (finishes) {
        if ((int)threadIdx.x >= tl.W)
            return;
        int16_t *dtab = dec + (int64_t)c * rows * pitch;
        const bool has_inner = INNER && (EDGE || step >= kInnerLevel);
        Window wn{tl.W, tl.halo, v * (apart ? span : tl.W - tl.halo), 0, apart && v > 0, (int)threadIdx.x, 0, 0};
        if (v > 0)
            wn.from = wn.w0 + (apart ? 0 : tl.halo);
        with_key(cw, R, C, [&](auto key, int S) {
            for_passes(wn, M, apart ? tl.apart_passes : tl.passes, R, [&](const Window &wn, int tile) {
                tile_finish<decltype(key), INNER>(r, cw, L, M, pitch, tile, tile - R + C, S, has_inner, wn, tab, dtab,
                                                  lds);
            });
        });
    } else {
        const int Wi = blockDim.x / tl.n_kw;
        const int kw = __builtin_amdgcn_readfirstlane(threadIdx.x / Wi);
        const int at = threadIdx.x - kw * Wi;
        int m = chunk * Wi + at;
        if (apart)  // a wave past the window's budgets is idle, like one past M
            m = m < span ? v * span + m : M + 1;
        int64_t *halo = !apart && tl.copy_W > 0 ? halo_of(cw, R, C - R) : nullptr;
        with_key(cw, R, C, [&](auto key, int S) {
            tile_inner<decltype(key), EDGE>(r, cw, L, M, pitch, R, C, S, m, at, Wi, tl.n_kw, kw, tab, halo,
                                            halo_pitch_of(cw), tl.copy_W, tl.copy_halo, lds);
        });
    }
}

}  // namespace

// Windows of a step of `tiles` tiles over all chains.  Launches of few tiles
// cut the budgets, into small windows where they are few (sizes, and with them
// the reach, grow with the budgets); from 128 tiles on the chip is full
// without, and a workgroup of four waves walks its tile's budgets in turn
// (measured on MI355X, against overlapping windows: ten chains of L = 101, M = 500
// 0.77 -> 0.65 ms, 32 of L = 64, M = 640 0.81 -> 0.64 ms; one of L = 100, M = 1000,
// with one workgroup of 16 waves per tile 0.49 -> 0.32 ms).
struct WindowSize {
    int W, halo;
};
constexpr WindowSize kWindowSizes[] = {{320, 128}, {512, 192}, {640, 256}};
constexpr bool halos_fit()
{
    for (const WindowSize &s : kWindowSizes)
        if (s.W % 64 || s.halo % 64 || s.W > 64 * kTileMaxWaves || 3 * s.halo > 2 * (s.W - s.halo))
            return false;
    return true;
}
static_assert(halos_fit(), "whole waves, and places for the halos (halo_pitch_of)");

static void tile_windows(const Tables &tb, int64_t tiles, TileLaunch &tl)
{
    const int chunks = (tb.M + 64) / 64;  // of 64 budgets
    tl.passes = tl.windows = tl.apart = tl.apart_passes = 1;
    tl.halo = INT_MAX;
    if (tiles >= 128) {
        tl.passes = (chunks + 3) / 4;
        tl.W = 64 * ((chunks + tl.passes - 1) / tl.passes);
        return;
    }
    if (chunks <= 5) {
        tl.W = 64 * chunks;
        return;
    }
    const WindowSize size = kWindowSizes[chunks < 12 ? 0 : chunks < 48 ? 1 : 2];
    tl.W = size.W;
    // the workspace has a place for the halos' inner results from two blocks on
    tl.halo = -1;
    if (tb.L > kBlock) {
        tl.halo = size.halo;
        tl.windows = max(0, tb.M - size.halo) / (size.W - size.halo) + 1;
    }
    const int n = tb.M / size.W + 1;
    tl.apart_passes = tl.steps.set == kBlockEdges && n > 2 ? 2 : 1;
    tl.apart = (n + tl.apart_passes - 1) / tl.apart_passes;
    tl.windows = max(tl.windows, tl.apart);
}

TileRun::TileRun(const Tables &tables, TileSet set, int delta)
    : tb(tables), set_(set), delta_(delta), groups_((tables.L + kG - 1) / kG)
{
    front_ = first_ = set == kBlockEdges ? -1 : 0;
    last_ = set == kAllTiles ? groups_ - 1 : set == kDiagonalBlocks ? min(groups_, kPerBlock) - 1 : 2 * kPerBlock - 2;
}

int TileRun::step() const { return front_ <= last_ ? front_ : -1; }

bool TileRun::more() const { return front_ < last_ + n_apart_; }

void TileRun::launch(hipStream_t stream, const Work &w)
{
    if (set_ != kBlockEdges && front_ == 0) {
        const int W = 64 * min((tb.M + 64) / 64, 8);
        triangle_kernel<<<dim3(groups_, tb.n_chains), W, 2 * kG * sizeof(int64_t) * W, stream>>>(
            tb.params, tb.L, tb.M, tb.pitch, tb.rows, tb.cost, tb.dec, w);
        first_ = ++front_;
        return;
    }
    TileLaunch tl;
    tl.steps = TileSteps{set_, groups_, delta_};
    const bool edge = set_ == kBlockEdges;
    // windows of one size through a run; where a step's were all in one launch,
    // the next one may begin a new run
    if (n_apart_ == 1 && !edge)
        first_ = front_;
    tile_windows(tb, (int64_t)tl.steps.count(edge ? kPerBlock - 1 : first_) * tb.n_chains, tl);
    n_apart_ = tl.apart;
    TileLaunch next = tl;
    if (n_apart_ == 1 && !edge && front_ < last_)
        tile_windows(tb, (int64_t)tl.steps.count(front_ + 1) * tb.n_chains, next);
    tl.copy_W = next.windows > 1 && next.halo > 0 ? next.W : 0;
    tl.copy_halo = next.halo;
    tl.front = front_;
    tl.first = max(first_, 0);
    tl.last = last_;
    // the run before left those of this one's first step
    tl.inner_from = edge ? 0 : max(kInnerLevel, first_ + 1);
    auto finished = [&](int step) { return step >= tl.first && step <= last_ ? tl.steps.count(step) : 0; };
    auto inner = [&](int step) { return step >= tl.inner_from && step <= last_ ? tl.steps.count(step) : 0; };
    tl.tiles = finished(front_);
    tl.next = inner(front_ + 1);
    tl.more = tl.apart_next = 0;
    if (tl.halo < INT_MAX)
        for (int v = 0; v < tl.apart; ++v) {
            tl.more = max(tl.more, finished(front_ - v) - tl.tiles);
            tl.apart_next = max(tl.apart_next, inner(front_ + 1 - v));
        }
    const int chunks = (tb.M + 64) / 64;
    const bool finishes = tl.tiles + tl.more > 0;
    int waves = finishes ? tl.W / 64 : min(chunks, 4);
    tl.n_kw = 1;
    tl.chunks = tl.apart_chunks = 0;
    if (tl.next + tl.apart_next > 0) {
        // waves of the inner splits: about 1024, at least 4 splits each
        // (measured: 512 and 2048 lose 5% at L = 339, M = 500 and ten chains of
        // L = 101)
        const int step = min(front_ + 1, last_), most = edge ? 1 : kG * step - 3 * kG + 1;
        const int64_t units = (int64_t)tl.steps.count(step) * chunks * tb.n_chains;
        auto rounded = [&](int kw) { return (waves + kw - 1) / kw * kw; };
        while (tl.n_kw < 8 && units * tl.n_kw < 1024 && most >= 8 * tl.n_kw && rounded(2 * tl.n_kw) <= kTileMaxWaves)
            tl.n_kw *= 2;
        waves = rounded(tl.n_kw);
        const int bw = waves / tl.n_kw;
        tl.chunks = (chunks + bw - 1) / bw;
        tl.apart_chunks = (tl.W / 64 * tl.apart_passes + bw - 1) / bw;
    }
    const int threads = 64 * waves;
    const size_t lds = max(2 * kG * sizeof(int64_t) * (size_t)(finishes ? tl.W : 0),
                           tl.n_kw > 1 ? kG * kG * sizeof(int64_t) * (size_t)(threads / tl.n_kw) : 0);
    const int wgs = tl.tiles * tl.windows + tl.next * tl.chunks + tl.more * tl.apart +
                    tl.apart_next * tl.apart_chunks * tl.apart;
    const bool windows = tl.halo < INT_MAX, has_inner = front_ >= kInnerLevel;
    const auto kernel = edge ? (windows ? tile_kernel<true, true, true> : tile_kernel<true, true, false>)
                        : has_inner ? (windows ? tile_kernel<true, false, true> : tile_kernel<true, false, false>)
                                    : (windows ? tile_kernel<false, false, true> : tile_kernel<false, false, false>);
    if (wgs > 0)
        kernel<<<dim3(wgs, tb.n_chains), threads, lds, stream>>>(tb.params, tb.L, tb.M, tb.pitch, tb.rows, tl, tb.cost,
                                                                 tb.dec, w);
    ++front_;
}

}  // namespace rotor
