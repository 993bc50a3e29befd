// Negacyclic NTT / INTT building blocks for gfx950 (Sec. 2.2; Sec. 4.2
// "(I)NTT ... stages split into phases").
//
// Transform (bit-reversed evaluation order):
//     A[k] = sum_n a[n] * psi^((2*brev(k)+1)*n)  (mod q)
// computed by the merged Cooley-Tukey recursion: stage s (0 <= s < log N)
// pairs j and j + N/2^(s+1) inside block i = j >> (log N - s) with twiddle
// Psi[2^s + i] = psi^brev(2^s + i); the inverse runs Gentleman-Sande stages
// in reverse with inverse twiddles and folds N^-1 (and any constant that
// follows, Sec. 5.1 Seq.1/Seq.2) into its last stage.
//
// Decomposition of one limb of N = 2^LOG1 * 256 residues, viewed as a
// 2^LOG1 x 256 row-major matrix (index j = h*256 + l):
//   column pass: stages 0 .. LOG1-1 act on h for each column l;
//   row pass   : stages LOG1 .. log N - 1 act on l for each row h.
// Each pass is one kernel; 256 threads each hold 16 residues in VGPRs and
// run up to four radix-2 stages in registers ("round"), exchange once
// through LDS, and run the remaining stages.  One pass reads and writes the
// limb once; the 255 twiddles of the column pass are shared by every column
// (wave-uniform loads), the row pass reads each row's own 255 twiddles.
#pragma once
#include <type_traits>

#include "internal.h"
#include "modarith.h"

namespace ckks {

constexpr int ROW_LOG = 8;
constexpr int ROW = 1 << ROW_LOG;
constexpr int NTT_THREADS = 256;
constexpr int ROWS_PER_WG = NTT_THREADS / 16;  // row pass: 16 threads per row

// Layout of a forward column pass's output inside key switching and
// rescaling: rows in groups of four, a group column by column (element (h, l)
// at 1024 (h / 4) + 4 l + h mod 4).  A column pass leaves four consecutive rows
// of a column in a thread: one 16-byte store, 64 contiguous bytes per tile and
// row group, where row-major rows took four stores of 16 bytes per tile, each a
// request of its own to the L2 (nearly three quarters of the requests of a
// batch's conversions).  The row pass reads a row with a stride of 16 bytes,
// and its work-group's other rows find the same lines in the L1.
// N = 2^16: the conversions of 64 items of 4 to 24 limbs 359 -> 303 and 292 ->
// 243 us, their combine 259 -> 286, the batch 2024 -> 1968; one HMult + rescale
// at 24 limbs 80.2 -> 78.1, 25-30 system at 15 limbs 60.7 -> 59.2.
__host__ __device__ constexpr int quad_row(int h) { return ((h >> 2) << (ROW_LOG + 2)) + (h & 3); }

// ---------------------------------------------------------------------------
// Butterflies.  Twiddles are centred pairs (w, round(w 2^32 / q)) and a
// product (mulr) lands in (-3q/4, 3q/4) for any signed 32-bit operand.  Two
// classes of primes, chosen per work-group (uniform branch):
//   q < 2^30 ("wide"): forward values are signed 32-bit integers.  A stage
//     that first centres its a (two multiply-adds) and one that does not
//     alternate.  A centred a is at most q/2 + |x| q e / 2^32, where e =
//     |2^32/q - round(2^32/q)| <= 1/2 (the centring's quotient is that rounded
//     reciprocal), and a product t at most q/2 + |x| q / 2^33.  From any 32-bit
//     input a centring stage leaves at most (5/4 + e/2) q, the stage after it
//     (7/4 + e/2 + (5/4 + e/2) q / 2^33) q, and that is below 0.963 2^31 for
//     every q < 2^30, because e is near 0 where q is near 2^30; the largest is
//     2.17 q at e = 1/2, q = 2^32 / 4.5 = 0.889 2^30.  (With e = 1/2 at 2^30 it
//     would be 2.19 q, beyond 2^31: the class limit and the reciprocal belong
//     together.)  A butterfly is 3
//     instructions for the product, 2 for the sums and on average 1 for the
//     centring.  Inverse values lie in [0, 2q): the difference is signed by
//     itself and the product's multiply-add adds q: 3 + 1, and 3 for the sum
//     and its reduction.
//   q >= 2^30 (31-bit): no headroom for sums.  Forward values lie in [-q, q):
//     both operands are corrected to [0, q) (one min each), the sum takes -q
//     with it; inverse values are canonical: 9 instructions.
// Against Shoup's product in [0, 2q) these are 8 -> 6 and 11 -> 9 instructions
// forward, 9 -> 7 and 11 -> 9 inverse (a loop of forward butterflies: 9.1 ->
// 7.6 CU cycles per wave), and one table word per twiddle instead of two:
// HMult + rescale at N = 2^16, 24 limbs 86.5 -> 83.3 us, 64 of them at 4 to 24
// limbs 2302 -> 2205 us, 32 hoisted rotations 1114 -> 1071 us.
// Pass boundaries: a forward pass takes canonical or centred residues or
// another forward pass's values and leaves forward values (fwd_canon gives
// [0, q)); an inverse row pass hands the column pass values in the inverse
// range, an inverse column pass ends canonical.
// ---------------------------------------------------------------------------
__device__ __forceinline__ bool wide_prime(uint32_t q) { return q < (1u << 30); }

// in-register radix-2 stages over the low NS bits of the register index k
// (x[k], k < E; E = 16, or 4 in the wave-per-row passes).  tw(u, b) returns
// the twiddle of stage u for register block b = k >> (NS - u).
template <int NS, bool WIDE, class TW, int E>
__device__ __forceinline__ void ct_stages(uint32_t (&x)[E], const PrimeC& p, TW&& tw)
{
#pragma unroll
    for (int u = 0; u < NS; u++) {
        const int half = 1 << (NS - 1 - u), span = 2 * half;
#pragma unroll
        for (int b = 0; b < E / span; b++) {
            const int2 w = tw(u, b);
#pragma unroll
            for (int m = 0; m < half; m++) {
                const int k = b * span + m;
                const uint32_t t = (uint32_t)mulr((int32_t)x[k + half], w, p.nq);
                if constexpr (WIDE) {
                    const uint32_t a = (u & 1) ? x[k] : (uint32_t)centre((int32_t)x[k], p);
                    x[k] = a + t;
                    x[k + half] = a - t;
                } else {  // [-q, q) -> [-q, q)
                    const uint32_t a = fix_signed(x[k], p.q), c = fix_signed(t, p.q);
                    x[k] = a + c + p.nq;
                    x[k + half] = a - c;
                }
            }
        }
    }
}

// forward range -> a residue small enough for one signed sum with a canonical
// one: (-q, q)
template <bool WIDE>
__device__ __forceinline__ int32_t fwd_centre(uint32_t x, const PrimeC& p)
{
    return WIDE ? centre((int32_t)x, p) : (int32_t)fix_signed(x, p.q);
}
// forward range -> [0, q)
template <bool WIDE>
__device__ __forceinline__ uint32_t fwd_canon(uint32_t x, const PrimeC& p)
{
    return fix_signed(WIDE ? (uint32_t)centre((int32_t)x, p) : x, p.q);
}

// Gentleman-Sande inverse stages, u = NS-1 .. 0.  If FOLD, stage u == 0 also
// multiplies both outputs by a constant: c = (c, c_s, c w, (c w)_s) with w the
// stage-0 twiddle, and ends canonical.
template <int NS, bool WIDE, bool FOLD, class TW, int E>
__device__ __forceinline__ void gs_stages(uint32_t (&x)[E], const PrimeC& p, TW&& tw, int4 c = int4{0, 0, 0, 0})
{
    const uint32_t q2 = 2 * p.q;
#pragma unroll
    for (int u = NS - 1; u >= 0; u--) {
        const int half = 1 << (NS - 1 - u), span = 2 * half;
#pragma unroll
        for (int b = 0; b < E / span; b++) {
            const int2 w = (FOLD && u == 0) ? make_int2(c.z, c.w) : tw(u, b);
#pragma unroll
            for (int m = 0; m < half; m++) {
                const int k = b * span + m;
                const uint32_t a = x[k], y = x[k + half];
                const int32_t d = (int32_t)(a - y);  // (-2q, 2q), or (-q, q)
                if (FOLD && u == 0) {
                    // a + y less 2q (or q), so that the sum is a signed operand too
                    const int32_t s = (int32_t)(a + y + (WIDE ? 2 * p.nq : p.nq));
                    x[k] = fix_signed((uint32_t)mulr(s, make_int2(c.x, c.y), p.nq), p.q);
                    x[k + half] = fix_signed((uint32_t)mulr(d, w, p.nq), p.q);
                } else if constexpr (WIDE) {  // [0, 2q) -> [0, 2q)
                    x[k] = red2(a + y, q2);
                    x[k + half] = mulr_add(d, w, p.nq, p.q);
                } else {                      // [0, q) -> [0, q)
                    x[k] = red2(a + y, p.q);
                    x[k + half] = fix_signed((uint32_t)mulr(d, w, p.nq), p.q);
                }
            }
        }
    }
}

// Calls f(tag) with tag = std::integral_constant<bool, q < 2^30>: q is
// uniform across the work-group, so this is one branch and each prime class
// gets its own straight-line code (read the class as
// decltype(tag)::value).
template <class F>
__device__ __forceinline__ void by_class(uint32_t q, F&& f)
{
    if (wide_prime(q))
        f(std::integral_constant<bool, true>{});
    else
        f(std::integral_constant<bool, false>{});
}

// ---------------------------------------------------------------------------
// LDS exchange layouts (one padding slot per 16 entries keeps both access
// patterns free of bank conflicts).
// ---------------------------------------------------------------------------
// column pass: element (row h, column c) of a 2^LOG1 x C tile
template <int C>
__device__ __forceinline__ int col_lds(int h, int c) { return (h + (h >> 4)) * C + c; }
// row pass: element (row rr, column l) of a 16 x 256 tile
__device__ __forceinline__ int row_lds(int rr, int l) { return rr * (ROW + ROW / 16) + l + (l >> 4); }

// Column tile of CT threads (256, or 512 for 128-byte rows at N = 2^16):
// 16 residues per thread, R threads per column, C columns.
template <int LOG1, int CT = NTT_THREADS>
struct ColGeom {
    static constexpr int S1 = 1 << LOG1;        // points per column transform
    static constexpr int R = S1 / 16;           // threads per column
    static constexpr int C = CT / R;            // columns per work-group
    static constexpr int NS2 = LOG1 - 4;        // stages in the second round
    static constexpr int LDS = (S1 + S1 / 16) * C;
    static_assert(C <= ROW, "column tile wider than a row");
};
constexpr int ROW_LDS_WORDS = ROWS_PER_WG * (ROW + ROW / 16);

// Launch geometry shared by all passes: blockIdx.y = limb of the launch,
// blockIdx.x = tile (column block or row block) inside the limb.
template <int LOG1, int CT = NTT_THREADS>
__host__ __device__ constexpr int col_tiles() { return ROW / ColGeom<LOG1, CT>::C; }

// Column tile of a column-pass work-group.  Work-groups go to the 8 XCDs
// round-robin in launch order (blockIdx.x fastest), so tile = blockIdx.x
// would put the two 64-byte halves of a 128-byte line (tiles 2m, 2m+1 when
// a tile is 16 columns) on different XCDs and fetch every line twice; pair
// them on one XCD instead.
template <int LOG1, int CT = NTT_THREADS>
__device__ __forceinline__ int col_tile(int pair)
{
    constexpr int T = col_tiles<LOG1, CT>();
    if constexpr (T == 16)
        return pair ? 2 * (blockIdx.x & 7) + (blockIdx.x >> 3) : (int)blockIdx.x;
    else if constexpr (T == 32)  // 8-column tiles: four per 128-byte line
        return pair ? 4 * (blockIdx.x & 7) + (blockIdx.x >> 3) : (int)blockIdx.x;
    else
        return blockIdx.x;
}
template <int LOG1>
__host__ __device__ constexpr int row_tiles() { return (1 << LOG1) / ROWS_PER_WG; }

// ---------------------------------------------------------------------------
// Pass kernels.  Ld::at(item) / St::at(item) return copies whose pointers
// are advanced to batch item `item` (identity for a single operation).
// Ld::load(M, limb, j, pc), load16, loadv<E> (E residues from j0 on) and
// load_rc (row, column) produce input residues (fused prologues);
// St::store(M, limb, j, v, pc), store4 (a run of lifted residues) and
// store_fwd<E, W> (E forward values, with the operands that prefetch<E>
// requested) consume outputs (fused epilogues); St::final_const(M, limb) is the
// constant folded into the last inverse stage.  M.pid[limb] is the prime.
// ---------------------------------------------------------------------------
// Launch maps reach the kernels as a pointer to a map precomputed in device
// memory at context creation (every internal launch), or by value for the
// stand-alone NTT with its caller-chosen primes: limb l of the launch is limb
// l of the data, so the prime ids are all there is to pass, a byte each in
// words that are read by scalar loads (264 bytes of kernel argument; a whole
// LaunchMap, 3.6 KB, cost more per launch than the kernel's own start).
struct SameLimb {
    __device__ int operator[](int l) const { return l; }
};
struct PackedIds {
    uint32_t w[MAX_LAUNCH_LIMBS / 4];
    __device__ int operator[](int l) const { return (int)((w[l >> 2] >> (8 * (l & 3))) & 255u); }
};
struct IdMap {
    int32_t count;
    SameLimb in_off, out_off;
    PackedIds pid, cidx;  // the final constants are indexed by prime too
};
struct MapByVal {
    IdMap m;
    __device__ const IdMap* get() const { return &m; }
};
struct MapByPtr {
    const LaunchMap* p;
    __device__ const LaunchMap* get() const { return p; }
};
// batched launch: item blockIdx.z uses the map of its own level; an item
// whose level lies outside [lo, hi], whose key index lies outside
// [0, n_keys) or whose input slot lies outside [0, n_src) gets no map and is
// skipped by every pass (n_src == 0: the launch reads one shared input and
// ignores the slot)
__device__ __forceinline__ bool item_ok(const BatchItem& it, int lo, int hi, int n_keys, int n_src)
{
    return it.level >= lo && it.level <= hi && it.key >= 0 && it.key < n_keys &&
           (n_src == 0 || (it.src >= 0 && it.src < n_src));
}
struct MapDir {
    const LaunchMap* const* dir;
    const BatchItem* items;
    int lo, hi, n_keys, n_src;
    __device__ const LaunchMap* get() const
    {
        const BatchItem it = items[blockIdx.z];
        return item_ok(it, lo, hi, n_keys, n_src) ? dir[it.level] : nullptr;
    }
};

__device__ __forceinline__ PrimeC prime_c(const uint32_t* mods, const uint32_t* qinvs, const int32_t* rcs, int pid)
{
    const uint32_t q = mods[pid];
    return PrimeC{q, qinvs[pid], 0u - q, rcs[pid]};
}

struct NttTables {
    const int32_t* tw;      // [n_primes][N] Psi (forward) or Psi^-1 (inverse) as round(w 2^32 / q)
    const uint32_t* mods;   // [n_primes]
    const uint32_t* qinvs;  // [n_primes] q^-1 mod 2^32
    const int32_t* rcs;     // [n_primes] round(2^32 / q)
    int log_n;
    int xcd_pair;           // column-tile order (col_tile)
    __device__ PrimeC prime(int pid) const { return prime_c(mods, qinvs, rcs, pid); }
};

// a prime's twiddle table, read as pairs
struct TwTable {
    const int32_t* p;
    uint32_t q;
    __device__ __forceinline__ int2 operator[](int i) const { return const_from_quot(p[i], q); }
};

// Row-pass twiddles of a work-group's ROWS_PER_WG rows, staged in LDS (one
// slot per thread) for kernels that run the same row pass several times
// (KeyMult: once per digit).  Row i, slot s: s < 15 is the first round
// (stage u = log2(s+1), block s+1-2^u: read at (1 << u) - 1 + b); s >= 16 is
// the second round (stage u = log2(s)-4, local index (rp << u) + b: read at
// (16 << u) + (rp << u) + b).  Ends with a barrier.
constexpr int ROW_TW_SLOTS = 256;
template <int LOG1>
__device__ __forceinline__ void stage_row_twiddles(int2* tws, const int32_t* tw, int h0, uint32_t q)
{
    static_assert(NTT_THREADS == ROW_TW_SLOTS, "one slot per thread");
    const int sl = threadIdx.x;
    if (sl != 15) {
        const int lg = 31 - __clz(sl < 15 ? sl + 1 : sl);
        const int loc = sl < 15 ? sl + 1 - (1 << lg) : sl - (1 << lg);
#pragma unroll 4
        for (int i = 0; i < ROWS_PER_WG; i++)
            tws[i * ROW_TW_SLOTS + sl] = const_from_quot(tw[(1 << (LOG1 + lg)) + ((h0 + i) << lg) + loc], q);
    }
    __syncthreads();
}
__device__ __forceinline__ int2 row_tw1(const int2* tws, int rr, int u, int b) { return tws[rr * ROW_TW_SLOTS + (1 << u) - 1 + b]; }
__device__ __forceinline__ int2 row_tw2(const int2* tws, int rr, int rp, int u, int b)
{
    return tws[rr * ROW_TW_SLOTS + (16 << u) + (rp << u) + b];
}

// forward, column pass (stages 0 .. LOG1-1)
template <int LOG1, class MS, class Ld, class St, int CT = NTT_THREADS>
__global__ void __launch_bounds__(CT) k_fwd_cols(NttTables T, MS ms, Ld ld0, St st0)
{
    // grid.z = batch item; grid.y is sized for the largest map of a batch
    const auto* Mp = ms.get();
    if (!Mp || (int)blockIdx.y >= Mp->count) return;
    const auto& M = *Mp;
    const Ld ld = ld0.at(blockIdx.z);
    const St st = st0.at(blockIdx.z);
    using G = ColGeom<LOG1, CT>;
    __shared__ uint32_t lds[G::LDS];
    const int limb = blockIdx.y, pid = M.pid[limb];
    const PrimeC pc = T.prime(pid);
    const TwTable tw{T.tw + ((size_t)pid << T.log_n), pc.q};
    const int c = threadIdx.x % G::C, r = threadIdx.x / G::C;
    const int col = col_tile<LOG1, CT>(T.xcd_pair) * G::C + c;
    uint32_t x[16];
#pragma unroll
    for (int k = 0; k < 16; k++) x[k] = ld.load(M, limb, (r + G::R * k) * ROW + col, pc);
    by_class(pc.q, [&](auto tag) {
        constexpr bool W = decltype(tag)::value;
        ct_stages<4, W>(x, pc, [&](int u, int b) { return tw[(1 << u) + b]; });
        if constexpr (G::NS2 > 0) {
#pragma unroll
            for (int k = 0; k < 16; k++) lds[col_lds<G::C>(r + G::R * k, c)] = x[k];
            __syncthreads();
#pragma unroll
            for (int k = 0; k < 16; k++) x[k] = lds[col_lds<G::C>(16 * r + k, c)];
            ct_stages<G::NS2, W>(x, pc, [&](int u, int b) {
                return tw[(1 << (4 + u)) + (r << (4 - G::NS2 + u)) + b];
            });
#pragma unroll
            for (int k = 0; k < 16; k++) st.store(M, limb, (16 * r + k) * ROW + col, x[k], pc);
        } else {
#pragma unroll
            for (int k = 0; k < 16; k++) st.store(M, limb, (r + G::R * k) * ROW + col, x[k], pc);
        }
    });
}

// forward, row pass (stages LOG1 .. LOG1+7); the storer takes forward values
template <int LOG1, class MS, class Ld, class St>
__global__ void __launch_bounds__(NTT_THREADS) k_fwd_rows(NttTables T, MS ms, Ld ld0, St st0)
{
    // grid.z = batch item; grid.y is sized for the largest map of a batch
    const auto* Mp = ms.get();
    if (!Mp || (int)blockIdx.y >= Mp->count) return;
    const auto& M = *Mp;
    const Ld ld = ld0.at(blockIdx.z);
    const St st = st0.at(blockIdx.z);
    __shared__ uint32_t lds[ROW_LDS_WORDS];
    const int limb = blockIdx.y, pid = M.pid[limb];
    const PrimeC pc = T.prime(pid);
    const TwTable tw{T.tw + ((size_t)pid << T.log_n), pc.q};
    // a wave holds four rows; in row groups of four its neighbouring lanes are
    // the four rows of one column, so that a load is contiguous
    const int rp = Ld::kQuads ? (threadIdx.x >> 2) & 15 : threadIdx.x % 16;
    const int rr = Ld::kQuads ? (int)((threadIdx.x & 3) | (threadIdx.x >> 6 << 2)) : threadIdx.x / 16;
    const int h = blockIdx.x * ROWS_PER_WG + rr;  // 2^LOG1 rows, LOG1 >= 4: exact grid
    uint32_t x[16];
#pragma unroll
    for (int k = 0; k < 16; k++) x[k] = ld.load_rc(M, limb, h, rp + 16 * k);
    by_class(pc.q, [&](auto tag) {
        constexpr bool W = decltype(tag)::value;
        ct_stages<4, W>(x, pc, [&](int u, int b) { return tw[(1 << (LOG1 + u)) + (h << u) + b]; });
#pragma unroll
        for (int k = 0; k < 16; k++) lds[row_lds(rr, rp + 16 * k)] = x[k];
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 16; k++) x[k] = lds[row_lds(rr, 16 * rp + k)];
        ct_stages<4, W>(x, pc, [&](int u, int b) {
            return tw[(1 << (LOG1 + 4 + u)) + (h << (4 + u)) + (rp << u) + b];
        });
        st.template store_fwd<16, W>(M, limb, h * ROW + 16 * rp, x, pc,
                                     st.template prefetch<16>(M, limb, h * ROW + 16 * rp));
    });
}

// inverse, row pass (stages LOG1+7 .. LOG1)
template <int LOG1, class MS, class Ld, class St>
__global__ void __launch_bounds__(NTT_THREADS) k_inv_rows(NttTables T, MS ms, Ld ld0, St st0)
{
    // grid.z = batch item; grid.y is sized for the largest map of a batch
    const auto* Mp = ms.get();
    if (!Mp || (int)blockIdx.y >= Mp->count) return;
    const auto& M = *Mp;
    const Ld ld = ld0.at(blockIdx.z);
    const St st = st0.at(blockIdx.z);
    __shared__ uint32_t lds[ROW_LDS_WORDS];
    const int limb = blockIdx.y, pid = M.pid[limb];
    const PrimeC pc = T.prime(pid);
    const TwTable tw{T.tw + ((size_t)pid << T.log_n), pc.q};
    const int rp = threadIdx.x % 16, rr = threadIdx.x / 16;
    const int h = blockIdx.x * ROWS_PER_WG + rr;
    uint32_t x[16];
    ld.load16(M, limb, h * ROW + 16 * rp, pc, x);
    by_class(pc.q, [&](auto tag) {
        constexpr bool W = decltype(tag)::value;
        gs_stages<4, W, false>(x, pc, [&](int u, int b) {
            return tw[(1 << (LOG1 + 4 + u)) + (h << (4 + u)) + (rp << u) + b];
        });
#pragma unroll
        for (int k = 0; k < 16; k++) lds[row_lds(rr, 16 * rp + k)] = x[k];
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 16; k++) x[k] = lds[row_lds(rr, rp + 16 * k)];
        gs_stages<4, W, false>(x, pc, [&](int u, int b) { return tw[(1 << (LOG1 + u)) + (h << u) + b]; });
    });
#pragma unroll
    for (int k = 0; k < 16; k++) st.store(M, limb, h * ROW + rp + 16 * k, x[k], pc);
}

// ---------------------------------------------------------------------------
// Row passes with one wave per row (4 residues per thread, 4 rows per
// work-group): four radix-4 rounds with three exchanges between registers and
// lanes, no LDS.  Four times the waves of the 16-residue passes: more memory
// latency hidden per SIMD when a launch has few limbs.
// Round j of the forward pass holds the 4 points
// l = blk*2^(sh+2) + pp + k*2^sh (sh = 6 - 2j, blk = t >> sh); the inverse
// pass walks the same units in the opposite order (sh = 2j).
// ---------------------------------------------------------------------------
constexpr int ROWS4 = NTT_THREADS / 64;   // rows (waves) per work-group
// the wave's index in its work-group, as a scalar (the same in every lane)
__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)); }
template <int LOG1>
__host__ __device__ constexpr int row4_tiles() { return (1 << LOG1) / ROWS4; }

// 4 x 4 transpose across the lanes of each quad, in registers: lane a's
// register b becomes lane b's register a.  Two exchange stages with the
// partner lane (DPP quad permutes): first the entries whose lane and register
// indices differ in bit 0 (partner lane a^1, register b^1), then in bit 1.
__device__ __forceinline__ void quad_transpose(uint32_t (&x)[4], int lane)
{
    constexpr int SWAP1 = 1 | (0 << 2) | (3 << 4) | (2 << 6);  // quad_perm [1, 0, 3, 2]
    constexpr int SWAP2 = 2 | (3 << 2) | (0 << 4) | (1 << 6);  // quad_perm [2, 3, 0, 1]
    uint32_t y[4];
#pragma unroll
    for (int b = 0; b < 4; b++) y[b] = (uint32_t)__builtin_amdgcn_mov_dpp((int)x[b ^ 1], SWAP1, 0xF, 0xF, true);
#pragma unroll
    for (int b = 0; b < 4; b++) x[b] = ((b ^ lane) & 1) ? y[b] : x[b];
#pragma unroll
    for (int b = 0; b < 4; b++) y[b] = (uint32_t)__builtin_amdgcn_mov_dpp((int)x[b ^ 2], SWAP2, 0xF, 0xF, true);
#pragma unroll
    for (int b = 0; b < 4; b++) x[b] = ((b ^ lane) & 2) ? y[b] : x[b];
}

// Exchange of one register bit with one lane bit: of a pair (a: register bit
// 0, b: bit 1), a lane whose bit LB is 0 keeps a and takes its partner's a as
// its b, a lane whose bit is 1 keeps b and takes its partner's b as its a.
// Bits 5 and 4 are the two halves and the odd and even 16-lane rows, which
// v_permlane32_swap and v_permlane16_swap exchange between two registers; bits
// 3 and 2 stay in a 16-lane row: a DPP shift by 8 or 4 lanes, written to the
// banks of four lanes that take it.
// Row passes need no LDS with these, column passes one exchange through LDS and
// one barrier instead of three (a swap of two registers takes about 2.5 issue
// slots, a DPP move one; an LDS exchange of four points 8 LDS operations, their
// addresses and a wait): HMult + rescale at N = 2^16, 24 limbs 83.5 -> 81.2 us
// (row passes 1.1 of it), 25-30 system at 15 limbs 63.2 -> 60.9; 64 items of 4
// to 24 limbs 2130 -> 2040 us, where KeyMult goes from 750 to 692 us (95
// instead of 106 registers, no LDS).
template <int LB>
__device__ __forceinline__ void lane_swap(uint32_t& a, uint32_t& b)
{
    static_assert(LB >= 2 && LB <= 5, "lane bits 2..5");
    if constexpr (LB >= 4) {
        const auto r = LB == 5 ? __builtin_amdgcn_permlane32_swap(a, b, false, false)
                               : __builtin_amdgcn_permlane16_swap(a, b, false, false);
        a = r[0], b = r[1];
    } else {
        constexpr int D = 1 << LB;                                   // partner's distance
        constexpr int ZERO = LB == 3 ? 0x3 : 0x5, ONE = 0xF ^ ZERO;  // banks whose lane bit is 0 / 1
        const uint32_t b0 = b;
        b = (uint32_t)__builtin_amdgcn_update_dpp((int)b, (int)a, 0x100 + D, 0xF, ZERO, false);   // row_shl: lane + D
        a = (uint32_t)__builtin_amdgcn_update_dpp((int)a, (int)b0, 0x110 + D, 0xF, ONE, false);   // row_shr: lane - D
    }
}
// the two register bits of four points with lane bits LB + 1 and LB (LB even:
// 4 and 2 here, 0 is quad_transpose)
template <int LB>
__device__ __forceinline__ void lane_exchange(uint32_t (&x)[4], int lane)
{
    if constexpr (LB == 0) {
        quad_transpose(x, lane);
    } else {
        lane_swap<LB + 1>(x[0], x[2]);
        lane_swap<LB + 1>(x[1], x[3]);
        lane_swap<LB>(x[0], x[1]);
        lane_swap<LB>(x[2], x[3]);
    }
}

// Forward row pass of the row a wave holds: x[k] = row[t + 64 k] on entry,
// row[4 t + k] on exit (forward values); tw[j][i]: round j's twiddles (stage 0,
// then the two of stage 1).  Round j's register bits are point bits 7 - 2j and
// 6 - 2j; the lane bits 5 - 2j and 4 - 2j hold the next round's, so the rounds
// change places in registers.
template <bool W>
__device__ __forceinline__ void row4_fwd(uint32_t (&x)[4], const PrimeC& p, int t, const int2 (&tw)[4][3])
{
#pragma unroll
    for (int j = 0; j < 4; j++) {
        if (j == 1) lane_exchange<4>(x, t);
        if (j == 2) lane_exchange<2>(x, t);
        if (j == 3) lane_exchange<0>(x, t);
        ct_stages<2, W>(x, p, [&](int u, int b) { return tw[j][u ? 1 + b : 0]; });
    }
}

// Inverse row pass: x[k] = row[4 t + k] on entry, row[t + 64 k] on exit
// (inverse range); tw[j][i] as in row4_fwd for round j of the inverse; the
// forward pass's exchanges undone.
template <bool W>
__device__ __forceinline__ void row4_inv(uint32_t (&x)[4], const PrimeC& p, int t, const int2 (&tw)[4][3])
{
#pragma unroll
    for (int j = 0; j < 4; j++) {
        if (j == 1) lane_exchange<0>(x, t);
        if (j == 2) lane_exchange<2>(x, t);
        if (j == 3) lane_exchange<4>(x, t);
        gs_stages<2, W, false>(x, p, [&](int u, int b) { return tw[j][u ? 1 + b : 0]; });
    }
}

// the twiddles thread t uses in row h (forward: round j covers stages
// LOG1 + 2j, LOG1 + 2j + 1; inverse: the same stages in reverse order).
// h is the same in every lane of a wave, so each entry's address is a
// wave-uniform base plus a 32-bit lane offset (scalar-base loads).
template <int LOG1, bool INV>
__device__ __forceinline__ void row4_twiddles(const int32_t* tw, uint32_t q, int h, int t, int2 (&out)[4][3])
{
    int32_t ws[4][3];
#pragma unroll
    for (int j = 0; j < 4; j++) {
        const int g = INV ? 6 - 2 * j : 2 * j;         // stage offset of the round's first stage
        const uint32_t blk = (uint32_t)t >> (INV ? 2 * j : 6 - 2 * j);
        const int32_t* s0 = tw + ((1u << (LOG1 + g)) + ((uint32_t)h << g));
        const int32_t* s1 = tw + ((1u << (LOG1 + g + 1)) + ((uint32_t)h << (g + 1)));
        ws[j][0] = s0[blk];
#pragma unroll
        for (int b = 0; b < 2; b++) ws[j][1 + b] = s1[(blk << 1) + (uint32_t)b];
    }
#pragma unroll
    for (int j = 0; j < 4; j++)
#pragma unroll
        for (int i = 0; i < 3; i++) out[j][i] = const_from_quot(ws[j][i], q);
}

// Launch-map entries of a work-group's limb (scalar loads issued together;
// the entries of limbs at or above count are in bounds and unused).
struct LimbInfo {
    int count, pid;
    PrimeC pc;
};
template <class LM>
__device__ __forceinline__ LimbInfo limb_info(const NttTables& T, const LM& M, int limb)
{
    LimbInfo r;
    r.count = M.count;
    r.pid = M.pid[limb];
    r.pc = T.prime(r.pid);
    return r;
}

// Row passes with one wave per row: every operand (the row, the twelve
// twiddles of the four rounds, and what the epilogue reads) is requested
// before the first wait, so a work-group pays about one memory latency.
template <int LOG1, class MS, class Ld, class St>
__global__ void __launch_bounds__(NTT_THREADS) k_fwd_rows4(NttTables T, MS ms, Ld ld0, St st0)
{
    const auto* Mp = ms.get();
    if (!Mp) return;
    const auto& M = *Mp;
    const int limb = blockIdx.y;
    const LimbInfo I = limb_info(T, M, limb);
    if (limb >= I.count) return;
    const Ld ld = ld0.at(blockIdx.z);
    const St st = st0.at(blockIdx.z);
    const PrimeC pc = I.pc;
    const int t = threadIdx.x & 63, w = wave_id();
    const int h = blockIdx.x * ROWS4 + w;  // exact grid
    uint32_t x[4];
#pragma unroll
    for (int k = 0; k < 4; k++) x[k] = ld.load_rc(M, limb, h, t + 64 * k);
    if constexpr (Ld::kQuads && St::kInPlace) __syncthreads();  // the rows of a group are read before one is written
    int2 tw[4][3];
    row4_twiddles<LOG1, false>(T.tw + ((size_t)I.pid << T.log_n), pc.q, h, t, tw);
    const auto pre = st.template prefetch<4>(M, limb, h * ROW + 4 * t);
    by_class(pc.q, [&](auto tag) {
        constexpr bool W = decltype(tag)::value;
        row4_fwd<W>(x, pc, t, tw);
        st.template store_fwd<4, W>(M, limb, h * ROW + 4 * t, x, pc, pre);
    });
}

template <int LOG1, class MS, class Ld, class St>
__global__ void __launch_bounds__(NTT_THREADS) k_inv_rows4(NttTables T, MS ms, Ld ld0, St st0)
{
    const auto* Mp = ms.get();
    if (!Mp) return;
    const auto& M = *Mp;
    const int limb = blockIdx.y;
    const LimbInfo I = limb_info(T, M, limb);
    if (limb >= I.count) return;
    const Ld ld = ld0.at(blockIdx.z);
    const St st = st0.at(blockIdx.z);
    const PrimeC pc = I.pc;
    const int t = threadIdx.x & 63, w = wave_id();
    const int h = blockIdx.x * ROWS4 + w;
    uint32_t x[4];
    ld.template loadv<4>(M, limb, h * ROW + 4 * t, pc, x);
    int2 tw[4][3];
    row4_twiddles<LOG1, true>(T.tw + ((size_t)I.pid << T.log_n), pc.q, h, t, tw);
    by_class(pc.q, [&](auto tag) { row4_inv<decltype(tag)::value>(x, pc, t, tw); });
#pragma unroll
    for (int k = 0; k < 4; k++) st.store(M, limb, h * ROW + t + 64 * k, x[k], pc);
}

// ---------------------------------------------------------------------------
// Column passes with 4 residues per thread.  256 threads hold a tile of
// C = 1024 / 2^LOG1 columns; thread (c = tid % C, t = tid / C) holds four
// points of column c.  Radix-4 rounds (plus one radix-2 round when LOG1 is
// odd) exchange once through LDS, across the waves, and then between registers
// and lanes (col4_lane): four times the waves of the 16-residue passes.  In a radix-4 round with shift sh the thread's
// points are base + k 2^sh, base = ((t >> sh) << (sh + 2)) | (t mod 2^sh);
// the radix-2 round holds 4t + k.  The forward pass enters with points
// t + k TC (TC = 2^LOG1 / 4) and leaves with 4t + k; the inverse pass the
// other way round.  Tile-thread layout of lifted residues (inverse passes
// write it, BConv passes read it, of either width): thread tid of tile T keeps
// its four residues at T 1024 + 4 tid (tile_run).
// ---------------------------------------------------------------------------
template <int LOG1>
struct Col4 {
    static constexpr int S1 = 1 << LOG1;           // points per column
    static constexpr int TC = S1 / 4;              // threads per column
    static constexpr int C = NTT_THREADS / TC;     // columns per work-group
    static constexpr int TILES = ROW / C;          // tiles per limb
    static constexpr int TILE = NTT_THREADS * 4;   // residues per tile
    static constexpr int NR4 = LOG1 / 2;           // radix-4 rounds
    static constexpr bool ODD = (LOG1 & 1) != 0;   // plus one radix-2 round
    static constexpr int NR = NR4 + (ODD ? 1 : 0);
    // LDS word of point p, column c: an additive padding, so the four
    // points of a round sit at fixed offsets from the first, chosen by
    // simulating every round's accesses (at most 2-way bank conflicts)
    static constexpr int PS = LOG1 == 8 ? 4 : 2;
    static constexpr int PA = LOG1 == 8 ? 12 : (LOG1 == 4 ? 0 : C);
    static constexpr int WORDS = S1 * C + PA * (S1 >> PS);  // one buffer
    __device__ static int lds(int p, int c) { return p * C + c + PA * (p >> PS); }
    // words from point base to point base + k 2^sh, the same for every thread
    // where a step is a multiple of the padding's 2^PS points (one address and
    // constant offsets for a round's four accesses)
    __host__ __device__ static constexpr bool fixed(int sh) { return PA == 0 || sh >= PS; }
    __host__ __device__ static constexpr int stride(int sh) { return (C << sh) + (PA == 0 ? 0 : PA * ((1 << sh) >> PS)); }
    __device__ static int lds_k(int base, int sh, int k, int c)
    {
        return fixed(sh) ? lds(base, c) + k * stride(sh) : lds(base + (k << sh), c);
    }
    // shift of forward round j (-1: the radix-2 round) and of inverse round j
    __host__ __device__ static constexpr int fsh(int j) { return j < NR4 ? LOG1 - 2 - 2 * j : -1; }
    __host__ __device__ static constexpr int ish(int j) { return ODD ? (j == 0 ? -1 : 1 + 2 * (j - 1)) : 2 * j; }
    static_assert(C >= 1 && C * TC == NTT_THREADS, "column tile");
};
// where the points t + k TC (k < 4) of a column start in the tile-thread layout
template <int LOG1>
__device__ __forceinline__ int tile_run(int col, int t)
{
    using G = Col4<LOG1>;
    return (col / G::C) * G::TILE + (t * G::C + col % G::C) * 4;
}
__device__ __forceinline__ int col4_base(int t, int sh) { return sh < 0 ? 4 * t : (((t >> sh) << (sh + 2)) | (t & ((1 << sh) - 1))); }

// Column tile of a 4-residue column work-group: as col_tile, the tiles that
// share a 128-byte line run on one XCD.
template <int LOG1>
__device__ __forceinline__ int col4_tile(int pair)
{
    constexpr int T = Col4<LOG1>::TILES;
    if constexpr (T >= 16)
        return pair ? (T / 8) * (blockIdx.x & 7) + (blockIdx.x >> 3) : (int)blockIdx.x;
    else
        return blockIdx.x;
}

// A column pass uses the first 2^LOG1 - 1 twiddles of its prime's table
// (Psi[1 .. 2^LOG1 - 1], shared by every column): a work-group stages them
// in LDS once as pairs (one load per thread, 2 KB at N = 2^16) and every
// round reads them there.  Entry e of the staged copy is table entry e.  Ends with a
// barrier.
template <int LOG1, int NT>
__device__ __forceinline__ void col4_stage_twiddles(int2* twl, const int32_t* const (&tw)[NT], const PrimeC (&p)[NT])
{
#pragma unroll
    for (int i = 0; i < NT; i++)
        for (int e = threadIdx.x; e < (1 << LOG1); e += NTT_THREADS)
            twl[i * (1 << LOG1) + e] = const_from_quot(tw[i][e], p[i].q);
    __syncthreads();
}
// twiddle of stage u of round j (sh: the round's shift) for pair block b
template <int LOG1>
__device__ __forceinline__ int2 col4_tw(const int2* twl, int t, int sh, int u, int b)
{
    if (sh < 0) return twl[(1 << (LOG1 - 1)) + 2 * t + b];  // radix-2 round: stage LOG1-1
    const int s0 = LOG1 - 2 - sh, blk = t >> sh;             // radix-4 round: stages s0, s0 + 1
    return twl[(1 << (s0 + u)) + (blk << u) + b];
}

// Exchange before forward round J >= 2, or undone (INV) after the inverse of
// that round.  Thread index t of a column is the wave's two bits and the lane
// bits above the tile's columns; only the first exchange (point bits LOG1 - 3
// and LOG1 - 4, held by the waves) crosses waves and goes through LDS.  Round
// 2's point bits lie in lane bits 5 and 4, round 3's in 3 and 2; the radix-2
// round of an odd LOG1 takes one, lane bit 5 (LOG1 = 5) or 3 (LOG1 = 7), for
// the higher register bit, and then the register bits change places.
template <int LOG1, int J, bool INV>
__device__ __forceinline__ void col4_lane(uint32_t (&x)[4])
{
    using G = Col4<LOG1>;
    if constexpr (J >= 2 && J < G::NR) {
        if constexpr (G::fsh(J) >= 0) {
            lane_exchange<J == 2 ? 4 : 2>(x, 0);  // its own inverse
        } else {
            constexpr int LB = LOG1 == 5 ? 5 : 3;
            if constexpr (INV) {
                const uint32_t y = x[1];
                x[1] = x[2], x[2] = y;
            }
            lane_swap<LB>(x[0], x[2]);
            lane_swap<LB>(x[1], x[3]);
            if constexpr (!INV) {
                const uint32_t y = x[1];
                x[1] = x[2], x[2] = y;
            }
        }
    }
}

// Forward column pass of NT targets held by the work-group: x[i] enters with
// points t + k TC of column c, leaves with 4t + k (forward values); lds holds
// one buffer of Col4::WORDS words per target (a round stores its results
// where it read its inputs, so one barrier per exchange suffices), twl the
// staged twiddles of each target
// (2^LOG1 entries apart).
template <int LOG1, int NT>
__device__ __forceinline__ void col4_fwd(uint32_t (&x)[NT][4], const PrimeC (&p)[NT], uint32_t* lds,
                                         const int2* twl, int c, int t)
{
    using G = Col4<LOG1>;
#pragma unroll
    for (int j = 0; j < G::NR; j++) {
        const int sh = G::fsh(j), base = col4_base(t, sh);
        if (j == 1) {
            __syncthreads();
#pragma unroll
            for (int i = 0; i < NT; i++)
#pragma unroll
                for (int k = 0; k < 4; k++) x[i][k] = lds[i * G::WORDS + G::lds_k(base, sh, k, c)];
        } else if (j == 2) {
#pragma unroll
            for (int i = 0; i < NT; i++) col4_lane<LOG1, 2, false>(x[i]);
        } else if (j == 3) {
#pragma unroll
            for (int i = 0; i < NT; i++) col4_lane<LOG1, 3, false>(x[i]);
        }
#pragma unroll
        for (int i = 0; i < NT; i++) {
            const int2* tl = twl + i * (1 << LOG1);
            by_class(p[i].q, [&](auto tag) {
                constexpr bool W = decltype(tag)::value;
                if (sh < 0)
                    ct_stages<1, W>(x[i], p[i], [&](int, int b) { return col4_tw<LOG1>(tl, t, sh, 0, b); });
                else
                    ct_stages<2, W>(x[i], p[i], [&](int u, int b) { return col4_tw<LOG1>(tl, t, sh, u, b); });
            });
        }
        if (j == 0) {
#pragma unroll
            for (int i = 0; i < NT; i++)
#pragma unroll
                for (int k = 0; k < 4; k++) lds[i * G::WORDS + G::lds_k(base, sh, k, c)] = x[i][k];
        }
    }
}

// Inverse column pass of one limb: x enters with points 4t + k, leaves with
// t + k TC, canonical, the last stage folding the constant cst (as
// gs_stages with FOLD).  lds: one buffer of Col4::WORDS words; twl: the
// staged inverse twiddles.
template <int LOG1, bool W>
__device__ __forceinline__ void col4_inv(uint32_t (&x)[4], const PrimeC& p, uint32_t* lds, const int2* twl, int c, int t,
                                         int4 cst)
{
    using G = Col4<LOG1>;
#pragma unroll
    for (int j = 0; j < G::NR; j++) {
        const int sh = G::ish(j), base = col4_base(t, sh);
        const bool last = j == G::NR - 1;
        if (last) {
            __syncthreads();
#pragma unroll
            for (int k = 0; k < 4; k++) x[k] = lds[G::lds_k(base, sh, k, c)];
        } else if (j == 1) {
            col4_lane<LOG1, G::NR - 1, true>(x);
        } else if (j == 2) {
            col4_lane<LOG1, G::NR - 2, true>(x);
        }
        auto tw = [&](int u, int b) { return col4_tw<LOG1>(twl, t, sh, u, b); };
        if (sh < 0) {
            gs_stages<1, W, false>(x, p, [&](int, int b) { return tw(0, b); });
        } else if (last) {
            gs_stages<2, W, true>(x, p, tw, cst);
        } else {
            gs_stages<2, W, false>(x, p, tw);
        }
        if (j == G::NR - 2) {
#pragma unroll
            for (int k = 0; k < 4; k++) lds[G::lds_k(base, sh < 0 ? 0 : sh, k, c)] = x[k];
        }
    }
}

// forward column pass, 4 residues per thread; leaves forward values
template <int LOG1, class MS, class Ld, class St>
__global__ void __launch_bounds__(NTT_THREADS) k_fwd_cols4(NttTables T, MS ms, Ld ld0, St st0)
{
    using G = Col4<LOG1>;
    const auto* Mp = ms.get();
    if (!Mp) return;
    const auto& M = *Mp;
    const int limb = blockIdx.y;
    const LimbInfo I = limb_info(T, M, limb);
    if (limb >= I.count) return;
    const Ld ld = ld0.at(blockIdx.z);
    const St st = st0.at(blockIdx.z);
    __shared__ uint32_t lds[G::WORDS];
    __shared__ int2 twl[1 << LOG1];
    const int c = threadIdx.x % G::C, t = threadIdx.x / G::C;
    const int col = col4_tile<LOG1>(T.xcd_pair) * G::C + c;
    uint32_t x[1][4];
#pragma unroll
    for (int k = 0; k < 4; k++) x[0][k] = ld.load(M, limb, (t + k * G::TC) * ROW + col, I.pc);
    const int32_t* const tws[1] = {T.tw + ((size_t)I.pid << T.log_n)};
    const PrimeC pcs[1] = {I.pc};
    col4_stage_twiddles<LOG1, 1>(twl, tws, pcs);
    col4_fwd<LOG1, 1>(x, pcs, lds, twl, c, t);
#pragma unroll
    for (int k = 0; k < 4; k++) st.store(M, limb, (4 * t + k) * ROW + col, x[0][k], I.pc);
}

// inverse column pass, 4 residues per thread: reads the row-pass output,
// ends canonical with the constant folded, stores through St (tile-thread
// layout when St::kTileThread)
template <int LOG1, class MS, class Ld, class St>
__global__ void __launch_bounds__(NTT_THREADS) k_inv_cols4(NttTables T, MS ms, Ld ld0, St st0)
{
    using G = Col4<LOG1>;
    const auto* Mp = ms.get();
    if (!Mp) return;
    const auto& M = *Mp;
    const int limb = blockIdx.y;
    const LimbInfo I = limb_info(T, M, limb);
    if (limb >= I.count) return;
    const Ld ld = ld0.at(blockIdx.z);
    const St st = st0.at(blockIdx.z);
    __shared__ uint32_t lds[G::WORDS];
    __shared__ int2 twl[1 << LOG1];
    const PrimeC pc = I.pc;
    const int c = threadIdx.x % G::C, t = threadIdx.x / G::C;
    const int tile = col4_tile<LOG1>(T.xcd_pair), col = tile * G::C + c;
    uint32_t x[4];
#pragma unroll
    for (int k = 0; k < 4; k++) x[k] = ld.load(M, limb, (4 * t + k) * ROW + col, pc);
    const int4 cst = st.final_const(M, limb);
    const int32_t* const tws[1] = {T.tw + ((size_t)I.pid << T.log_n)};
    const PrimeC pcs[1] = {pc};
    col4_stage_twiddles<LOG1, 1>(twl, tws, pcs);
    by_class(pc.q, [&](auto tag) { col4_inv<LOG1, decltype(tag)::value>(x, pc, lds, twl, c, t, cst); });
    if constexpr (St::kTileThread) {
        st.store4(M, limb, tile * G::TILE + threadIdx.x * 4, x, pc);
    } else {
#pragma unroll
        for (int k = 0; k < 4; k++) st.store(M, limb, (t + k * G::TC) * ROW + col, x[k], pc);
    }
}

// inverse, column pass (stages LOG1-1 .. 0); the last stage multiplies by
// st.final_const(M, limb) (N^-1 times whatever constant follows) and ends
// canonical.
template <int LOG1, class MS, class Ld, class St, int CT = NTT_THREADS>
__global__ void __launch_bounds__(CT) k_inv_cols(NttTables T, MS ms, Ld ld0, St st0)
{
    // grid.z = batch item; grid.y is sized for the largest map of a batch
    const auto* Mp = ms.get();
    if (!Mp || (int)blockIdx.y >= Mp->count) return;
    const auto& M = *Mp;
    const Ld ld = ld0.at(blockIdx.z);
    const St st = st0.at(blockIdx.z);
    using G = ColGeom<LOG1, CT>;
    __shared__ uint32_t lds[G::LDS];
    const int limb = blockIdx.y, pid = M.pid[limb];
    const PrimeC pc = T.prime(pid);
    const TwTable tw{T.tw + ((size_t)pid << T.log_n), pc.q};
    const int c = threadIdx.x % G::C, r = threadIdx.x / G::C;
    const int col = col_tile<LOG1, CT>(T.xcd_pair) * G::C + c;
    const int4 cst = st.final_const(M, limb);
    uint32_t x[16];
    if constexpr (G::NS2 > 0) {
#pragma unroll
        for (int k = 0; k < 16; k++) x[k] = ld.load(M, limb, (16 * r + k) * ROW + col, pc);
    } else {
#pragma unroll
        for (int k = 0; k < 16; k++) x[k] = ld.load(M, limb, (r + G::R * k) * ROW + col, pc);
    }
    by_class(pc.q, [&](auto tag) {
        constexpr bool W = decltype(tag)::value;
        if constexpr (G::NS2 > 0) {
            gs_stages<G::NS2, W, false>(x, pc, [&](int u, int b) {
                return tw[(1 << (4 + u)) + (r << (4 - G::NS2 + u)) + b];
            });
#pragma unroll
            for (int k = 0; k < 16; k++) lds[col_lds<G::C>(16 * r + k, c)] = x[k];
            __syncthreads();
#pragma unroll
            for (int k = 0; k < 16; k++) x[k] = lds[col_lds<G::C>(r + G::R * k, c)];
        }
        gs_stages<4, W, true>(x, pc, [&](int u, int b) { return tw[(1 << u) + b]; }, cst);
    });
    if constexpr (St::kTileThread) {
        // points r + R (m + 4 k) of the column: run r + R m of the tile-thread layout
#pragma unroll
        for (int m = 0; m < 4; m++) {
            const uint32_t v[4] = {x[m], x[m + 4], x[m + 8], x[m + 12]};
            st.store4(M, limb, tile_run<LOG1>(col, r + G::R * m), v, pc);
        }
    } else {
#pragma unroll
        for (int k = 0; k < 16; k++) st.store(M, limb, (r + G::R * k) * ROW + col, x[k], pc);
    }
}

}  // namespace ckks
