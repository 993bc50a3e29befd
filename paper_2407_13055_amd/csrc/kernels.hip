// HIP kernels and launch sequences of the key-switching path (gfx950):
// ModUp -> KeyMult -> MAC -> automorphism -> ModDown (Sec. 2.3), rescale
// (Sec. 2.1), and the stand-alone NTT / BConv calls.
//
// Fusion (Sec. 5): the tensor product, the automorphism gather and the BConv
// constant multiplication ride on the INTT passes (Seq.1); the BConv matrix
// multiplication feeds the NTT column pass directly; KeyMult over all digits
// is one output-stationary kernel that also runs the NTT row pass, adds the
// HMult d0/d1 (or HRot phi(b)) term pre-multiplied by P so that ModDown
// returns it unchanged, and starts ModDown's INTT on the P rows (Par.1); the
// last NTT row pass of ModDown / rescale subtracts and scales in its
// epilogue (Seq.3).  Montgomery factors 2^-32 are folded into constants
// (Seq.2) so no pass converts in or out of Montgomery form.
#include <cstdlib>
#include <algorithm>
#include <cstring>
#include <vector>

#include "internal.h"
#include "ntt_core.h"
#include "xcd_rows.h"

namespace ckks {

thread_local KtEvents* g_kt = nullptr;

// ---------------------------------------------------------------------------
// loaders
// ---------------------------------------------------------------------------
__device__ __forceinline__ void load16_u32(const uint32_t* p, uint32_t (&x)[16])
{
    const uint4* v = reinterpret_cast<const uint4*>(p);
#pragma unroll
    for (int i = 0; i < 4; i++) {
        uint4 t = v[i];
        x[4 * i] = t.x, x[4 * i + 1] = t.y, x[4 * i + 2] = t.z, x[4 * i + 3] = t.w;
    }
}

__device__ __forceinline__ void store16_u32(uint32_t* p, const uint32_t (&x)[16])
{
    uint4* v = reinterpret_cast<uint4*>(p);
#pragma unroll
    for (int i = 0; i < 4; i++) v[i] = make_uint4(x[4 * i], x[4 * i + 1], x[4 * i + 2], x[4 * i + 3]);
}

// E contiguous residues (E a multiple of 4, p 16-byte aligned)
template <int E>
__device__ __forceinline__ void loadv_u32(const uint32_t* p, uint32_t (&x)[E])
{
    const uint4* v = reinterpret_cast<const uint4*>(p);
#pragma unroll
    for (int i = 0; i < E / 4; i++) {
        uint4 t = v[i];
        x[4 * i] = t.x, x[4 * i + 1] = t.y, x[4 * i + 2] = t.z, x[4 * i + 3] = t.w;
    }
}
template <int E>
__device__ __forceinline__ void storev_u32(uint32_t* p, const uint32_t (&x)[E])
{
    uint4* v = reinterpret_cast<uint4*>(p);
#pragma unroll
    for (int i = 0; i < E / 4; i++) v[i] = make_uint4(x[4 * i], x[4 * i + 1], x[4 * i + 2], x[4 * i + 3]);
}

// four residues read once by the whole launch (keys and plaintexts of hoisted
// rotations): non-temporal, so that they do not displace the shared rows in L2
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void load_once(const uint32_t* p, uint32_t (&x)[4])
{
    const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
    x[0] = v.x, x[1] = v.y, x[2] = v.z, x[3] = v.w;
}

// Galois element 5^(k mod N/2) mod 2N of a rotation by k slots (Sec. 2.2 Eq. 4)
__device__ __forceinline__ uint32_t galois_of(int k, int log_n)
{
    const uint32_t half = 1u << (log_n - 1), mask = (2u << log_n) - 1u;
    uint32_t e = (uint32_t)(((k % (int)half) + (int)half) % (int)half), g = 1, b = 5;
    for (; e; e >>= 1, b = (b * b) & mask)
        if (e & 1) g = (g * b) & mask;
    return g;
}

// The automorphism X -> X^g in the bit-reversed evaluation order (Eq. 4):
// natural slot k takes natural slot k' with 2k'+1 = g(2k+1) mod 2N.  An
// aligned group of four positions differs in the two top bits of k, and
// g N/4 = (g mod 4) N/4 (mod N): the four sources are one aligned group too,
// rotated among themselves.  So a thread's four residues are one 16-byte load
// and one address computation instead of four of each.
struct AutQuad {
    uint32_t off;   // first position of the source group
    uint32_t rot;   // natural index u of the group takes (g u + rot) mod 4
    bool neg;       // g = 3 (mod 4): conjugation
    // pos: a multiple of 4
    __device__ __forceinline__ AutQuad(uint32_t pos, uint32_t g, int log_n)
    {
        const uint32_t k = __brev(pos >> 2) >> (34 - log_n);                      // low log_n - 2 bits of the natural slot
        const uint32_t kp = (g * k + (g >> 1)) & ((1u << log_n) - 1u);
        off = (__brev(kp & ((1u << (log_n - 2)) - 1u)) >> (34 - log_n)) << 2;
        rot = kp >> (log_n - 2);
        neg = (g & 2u) != 0;
    }
    __device__ __forceinline__ void load(const uint32_t* row, uint32_t* x) const
    {
        const uint4 v = *reinterpret_cast<const uint4*>(row + off);
        arrange(v, x);
    }
    __device__ __forceinline__ void arrange(const uint4 v, uint32_t* x) const
    {
        // natural order within the group: positions 0, 2, 1, 3
        uint32_t w0 = v.x, w1 = neg ? v.w : v.z, w2 = v.y, w3 = neg ? v.z : v.w;
        const uint32_t r = neg ? 4u - rot : rot;
        if (r & 1u) {
            const uint32_t t = w0;
            w0 = w1, w1 = w2, w2 = w3, w3 = t;
        }
        const bool half = (r & 2u) != 0;
        x[0] = half ? w2 : w0;
        x[2] = half ? w3 : w1;
        x[1] = half ? w0 : w2;
        x[3] = half ? w1 : w3;
    }
};

// Every loader / storer carries, per pointer, the residue step between
// consecutive items of a batched launch (0 for a single operation); at(i)
// returns the copy for item i.
struct LdPlain {
    static constexpr bool kTileThread = false;
    const uint32_t* base;
    int log_n;
    size_t step = 0;
    __device__ LdPlain at(int i) const
    {
        LdPlain r = *this;
        r.base += (size_t)i * step;
        return r;
    }
    template <class LM>
    __device__ uint32_t load(const LM& M, int l, int j, PrimeC) const
    {
        return base[((size_t)M.in_off[l] << log_n) + j];
    }
    template <class LM>
    __device__ void load16(const LM& M, int l, int j, PrimeC, uint32_t (&x)[16]) const
    {
        load16_u32(base + ((size_t)M.in_off[l] << log_n) + j, x);
    }
    template <int E, class LM>
    __device__ void loadv(const LM& M, int l, int j, PrimeC, uint32_t (&x)[E]) const
    {
        loadv_u32<E>(base + ((size_t)M.in_off[l] << log_n) + j, x);
    }
    static constexpr bool kQuads = false;
    template <class LM>
    __device__ uint32_t load_rc(const LM& M, int l, int h, int col) const
    {
        return base[((size_t)M.in_off[l] << log_n) + (size_t)h * ROW + col];
    }
};

// a forward column pass's output (quad_row)
struct LdQuads {
    static constexpr bool kQuads = true;
    const uint32_t* base;
    int log_n;
    size_t step = 0;
    __device__ LdQuads at(int i) const
    {
        LdQuads r = *this;
        r.base += (size_t)i * step;
        return r;
    }
    template <class LM>
    __device__ uint32_t load_rc(const LM& M, int l, int h, int col) const
    {
        return (base + (((size_t)M.in_off[l] << log_n) + quad_row(h)))[4 * col];
    }
};

// the digit's own rows: a_a*a_b*2^-32 (HMult), d (KeySwitch), phi_g(a) (HRot)
template <Own OWN>
struct LdOwn {
    static constexpr bool kTileThread = false;
    const uint32_t* a0;
    const uint32_t* a1;
    uint32_t galois;
    int log_n;
    size_t step0 = 0, step1 = 0;
    const BatchItem* items = nullptr;  // batched HRot: Galois element per item
    __device__ LdOwn at(int i) const
    {
        LdOwn r = *this;
        const size_t src = items ? (size_t)items[i].src : (size_t)i;  // input slot of item i
        r.a0 += src * step0;
        if (a1) r.a1 += src * step1;
        if (items) r.galois = galois_of(items[i].rot, log_n);
        return r;
    }
    template <int E>
    __device__ void loadv(const LaunchMap& M, int l, int j, PrimeC pc, uint32_t (&x)[E]) const
    {
        const size_t off = (size_t)M.in_off[l] << log_n;
        if constexpr (OWN == Own::Tensor) {
            uint32_t y[E];
            loadv_u32<E>(a0 + off + j, x);
            loadv_u32<E>(a1 + off + j, y);
#pragma unroll
            for (int k = 0; k < E; k++) x[k] = mont(x[k], y[k], pc.q, pc.qinv);
        } else if constexpr (OWN == Own::Plain) {
            loadv_u32<E>(a0 + off + j, x);
        } else {
#pragma unroll
            for (int k = 0; k < E; k += 4) AutQuad(j + k, galois, log_n).load(a0 + off, x + k);
        }
    }
    __device__ void load16(const LaunchMap& M, int l, int j, PrimeC pc, uint32_t (&x)[16]) const
    {
        loadv<16>(M, l, j, pc, x);
    }
};

// ---------------------------------------------------------------------------
// storers
// ---------------------------------------------------------------------------
struct StPlain {
    static constexpr bool kTileThread = false, kInPlace = true;
    uint32_t* base;
    const int4* fc;  // final constant table (inverse passes), row cidx[l]
    int log_n;
    size_t step = 0;
    __device__ StPlain at(int i) const
    {
        StPlain r = *this;
        r.base += (size_t)i * step;
        return r;
    }
    template <class LM>
    __device__ void store(const LM& M, int l, int j, uint32_t v, PrimeC) const
    {
        base[((size_t)M.out_off[l] << log_n) + j] = v;
    }
    template <int E, class LM>
    __device__ void storev(const LM& M, int l, int j, const uint32_t (&x)[E], PrimeC) const
    {
        storev_u32<E>(base + ((size_t)M.out_off[l] << log_n) + j, x);
    }
    // epilogue operands requested ahead of the pass: none
    struct Pre {};
    template <int E, class LM>
    __device__ Pre prefetch(const LM&, int, int) const { return {}; }
    // canonical residues of forward values (class W)
    template <int E, bool W, class LM>
    __device__ void store_fwd(const LM& M, int l, int j, const uint32_t (&x)[E], PrimeC pc, Pre) const
    {
        uint32_t y[E];
#pragma unroll
        for (int k = 0; k < E; k++) y[k] = fwd_canon<W>(x[k], pc);
        storev<E>(M, l, j, y, pc);
    }
    template <class LM>
    __device__ int4 final_const(const LM& M, int l) const { return fc[M.cidx[l]]; }
};

// centred lift into int32 (input of a base conversion), tile-thread layout:
// four points of a column per 16-byte run (Col4)
struct StLift {
    static constexpr bool kTileThread = true;
    int32_t* base;
    const int4* fc;
    int log_n;
    size_t step = 0;
    __device__ StLift at(int i) const
    {
        StLift r = *this;
        r.base += (size_t)i * step;
        return r;
    }
    __device__ void store4(const LaunchMap& M, int l, int j, const uint32_t (&x)[4], PrimeC pc) const
    {
        uint32_t y[4];
#pragma unroll
        for (int k = 0; k < 4; k++) y[k] = (uint32_t)lift(x[k], pc.q);
        storev_u32<4>(reinterpret_cast<uint32_t*>(base) + ((size_t)M.out_off[l] << log_n) + j, y);
    }
    __device__ int4 final_const(const LaunchMap& M, int l) const { return fc[M.cidx[l]]; }
};

// out = (sub - v) * c  (ModDown: c = P^-1 R^2; rescale: c = q_last^-1); sub = 0 where sub_off < 0.
// v is a forward value: centred, its difference with the canonical sub lies
// in (-q, 2q) of a wide prime or (-q, q) of a 31-bit one, an operand of mulr.
struct StCombine {
    static constexpr bool kTileThread = false, kInPlace = false;
    uint32_t* out0;
    uint32_t* out1;
    const uint32_t* sub;
    const int2* cst;
    int log_n;
    size_t out_step = 0, sub_step = 0;
    __device__ StCombine at(int i) const
    {
        StCombine r = *this;
        r.out0 += (size_t)i * out_step;
        r.out1 += (size_t)i * out_step;
        r.sub += (size_t)i * sub_step;
        return r;
    }
    // the subtrahend row and the constant, requested ahead of the pass
    template <int E>
    struct PreE {
        uint32_t s[E];
        int2 c;
    };
    template <int E>
    __device__ PreE<E> prefetch(const LaunchMap& M, int l, int j) const
    {
        PreE<E> p;
        if (M.sub_off[l] >= 0) {
            loadv_u32<E>(sub + ((size_t)M.sub_off[l] << log_n) + j, p.s);
        } else {  // an output prime the input did not have (rational rescaling's added primes)
#pragma unroll
            for (int k = 0; k < E; k++) p.s[k] = 0;
        }
        p.c = cst[M.cidx[l]];
        return p;
    }
    template <int E, bool W>
    __device__ void store_fwd(const LaunchMap& M, int l, int j, const uint32_t (&x)[E], PrimeC pc,
                              const PreE<E>& p) const
    {
        uint32_t o[E];
#pragma unroll
        for (int k = 0; k < E; k++) {
            const int32_t d = (int32_t)(p.s[k] - (uint32_t)fwd_centre<W>(x[k], pc));
            o[k] = fix_signed((uint32_t)mulr(d, p.c, pc.nq), pc.q);
        }
        storev_u32<E>((M.grp[l] ? out1 : out0) + ((size_t)M.out_off[l] << log_n) + j, o);
    }
};

// ---------------------------------------------------------------------------
// BConv matrix multiplication feeding the NTT column pass (ModUp, ModDown).
// A work-group owns one column tile and up to TPW target primes that share
// their input rows (a digit's lifted rows, or one polynomial's lifted P
// rows).  The input rows stream through registers one at a time into int64
// accumulators of all TPW targets (lazy reduction, Sec. 4.2); each target
// is then reduced once (signed Montgomery), runs the column pass and is
// stored.  Column tile t runs on XCD t mod 8 for every target, so the
// reloads of a tile's inputs by other work-groups hit that XCD's L2.
// ---------------------------------------------------------------------------
// acc - t 2^32 if acc >= t 2^31, acc + t 2^32 if acc < -t 2^31, else acc.
// Adding a multiple of 2^32 touches only the high word, so the fix is a
// select of -t / t / 0 added there (no branch, no 64-bit add).
__device__ __forceinline__ int64_t range_fix(int64_t acc, int64_t t31, int64_t t32)
{
    const int32_t t = (int32_t)(t32 >> 32);
    int32_t adj = acc >= t31 ? -t : 0;
    adj = acc < -t31 ? t : adj;
    const uint32_t hi = (uint32_t)(acc >> 32) + (uint32_t)adj;
    return (int64_t)(((uint64_t)hi << 32) | (uint32_t)acc);
}

// Fused rescale (RS): the group's input rows are followed in y by row e =
// INTT(ks_{l-1}) P^-1 (lifted); the kernel also converts the P rows to
// q_{l-1} (times P^-1), forms t = lift(e - conv_{l-1} P^-1), which is the
// coefficient form of the ModDown output's last limb, and adds t * P to
// every target before the NTT, so the row pass can divide by P q_{l-1}.
struct BcRescale {
    const int32_t* mlast;  // [n_q][n_p] centred [Phat_k P^-1 R]_{q_i}; row l-1 is used
    const int32_t* pr;     // [n_q] centred [P R^-1]_{q_i}, indexed by target prime
    int n_p;
    int level;             // single operation: its level; batched: taken from the item
    int nofix = 0;         // every sum of the launch stays within t 2^31 (Ctx::up_nofix)
};

struct BcByPtr {
    const BcMap* p;
    __device__ const BcMap* get() const { return p; }
};
struct BcDir {
    const BcMap* const* dir;
    const BatchItem* items;
    int lo, hi, n_keys, n_src;
    __device__ const BcMap* get() const
    {
        const BatchItem it = items[blockIdx.z];
        return item_ok(it, lo, hi, n_keys, n_src) ? dir[it.level] : nullptr;
    }
};

// A BConv map read through a global-memory pointer: its wave-uniform fields
// then load through the scalar cache into SGPRs.  A map found in a launch
// directory arrives as a generic pointer read from memory, whose fields the
// compiler would otherwise read per lane, into VGPRs, with divergent branches
// on them.
using GlobalBcMap = const __attribute__((address_space(1))) BcMap;

template <int LOG1, int TPW, int NIN, bool RS, class BS, int CT = NTT_THREADS>
__global__ void __launch_bounds__(CT) k_bconv_ntt_cols(NttTables T, BS bs, const int32_t* y0,
                                                                const int32_t* mat, uint32_t* out0, BcRescale X,
                                                                size_t step, const BatchItem* items)
{
    const BcMap* Bp = bs.get();
    if (!Bp) return;
    GlobalBcMap& B = *(GlobalBcMap*)Bp;
    if ((int)blockIdx.y >= B.groups) return;
    const int32_t* y = y0 + (size_t)blockIdx.z * step;
    uint32_t* out = out0 + (size_t)blockIdx.z * step;
    using G = ColGeom<LOG1, CT>;
    __shared__ uint32_t lds[G::LDS];
    const int g = blockIdx.y;
    const int c = threadIdx.x % G::C, r = threadIdx.x / G::C;
    const int tile = col_tile<LOG1, CT>(T.xcd_pair);
    const int col = tile * G::C + c;
    const int n_in = B.n_in[g], n_tg = B.n_tg[g], first = B.first[g];
    const size_t n = (size_t)1 << T.log_n;
    // inputs in the tile-thread layout: this thread's 16 residues of row s are
    // four runs of four, s*N + tile_run(col, r + R m)
    const int32_t* src = y + (size_t)B.in_off[g] * n;
    auto load_row = [&](size_t row, uint32_t (&x)[16]) {
#pragma unroll
        for (int m = 0; m < 4; m++) {
            uint32_t v[4];
            loadv_u32<4>(reinterpret_cast<const uint32_t*>(src + row * n) + tile_run<LOG1>(col, r + G::R * m), v);
#pragma unroll
            for (int k = 0; k < 4; k++) x[m + 4 * k] = v[k];
        }
    };

    int64_t acc[TPW][16];
    int64_t t31[TPW], t32[TPW];
#pragma unroll
    for (int t = 0; t < TPW; t++) {
        const int tt = first + (t < n_tg ? t : 0);
        const uint32_t q = T.mods[B.pid[tt]];
        t31[t] = (int64_t)q << 31, t32[t] = (int64_t)q << 32;
#pragma unroll
        for (int k = 0; k < 16; k++) acc[t][k] = 0;
    }
    int64_t accl[RS ? 16 : 1];
    uint32_t ql = 0;
    int64_t l31 = 0, l32 = 0;
    const int ql_pid = RS ? (items ? items[blockIdx.z].level : X.level) - 1 : 0;  // prime id of q_{l-1}
    const int32_t* mlast = X.mlast + (size_t)ql_pid * X.n_p;
    if constexpr (RS) {
        ql = T.mods[ql_pid];
        l31 = (int64_t)ql << 31, l32 = (int64_t)ql << 32;
#pragma unroll
        for (int k = 0; k < 16; k++) accl[k] = 0;
    }
    // one input row at a time; the next row's load is in flight while this row is accumulated
    auto mac = [&](const uint32_t (&yv)[16], int s) {
        if (s >= 8 && (s & 3) == 0) {
#pragma unroll
            for (int t = 0; t < TPW; t++)
#pragma unroll
                for (int k = 0; k < 16; k++) acc[t][k] = range_fix(acc[t][k], t31[t], t32[t]);
            if constexpr (RS) {
#pragma unroll
                for (int k = 0; k < 16; k++) accl[k] = range_fix(accl[k], l31, l32);
            }
        }
#pragma unroll
        for (int t = 0; t < TPW; t++) {
            const int64_t mt = t < n_tg ? mat[B.mat_off[first + t] + s] : 0;
#pragma unroll
            for (int k = 0; k < 16; k++) acc[t][k] += (int64_t)(int32_t)yv[k] * mt;
        }
        if constexpr (RS) {
            const int64_t mt = mlast[s];
#pragma unroll
            for (int k = 0; k < 16; k++) accl[k] += (int64_t)(int32_t)yv[k] * mt;
        }
    };
    uint32_t e[RS ? 16 : 1];
    if constexpr (RS) load_row((size_t)n_in, e);  // last limb, used below
    {
        uint32_t ya[16], yb[16];
        if (n_in > 0) load_row(0, ya);
        int s = 0;
        for (; s + 1 < n_in; s += 2) {
            load_row((size_t)(s + 1), yb);
            mac(ya, s);
            if (s + 2 < n_in) load_row((size_t)(s + 2), ya);
            mac(yb, s + 1);
        }
        if (s < n_in) mac(ya, s);
    }
    int32_t tl[RS ? 16 : 1];
    if constexpr (RS) {
        const uint32_t qlinv = T.qinvs[ql_pid];
#pragma unroll
        for (int k = 0; k < 16; k++) {
            const uint32_t cl = canon_signed(smr64(range_fix(accl[k], l31, l32), ql, qlinv), ql);
            const int32_t ei = (int32_t)e[k];
            const uint32_t ec = ei < 0 ? (uint32_t)(ei + (int32_t)ql) : (uint32_t)ei;
            tl[k] = lift(sub_mod(ec, cl, ql), ql);
        }
    }

#pragma unroll
    for (int t = 0; t < TPW; t++) {
        if (t >= n_tg) break;
        const int tg = first + t;
        const int pid = B.pid[tg];
        const PrimeC pc = T.prime(pid);
        const uint32_t q = pc.q, qinv = pc.qinv;
        const TwTable tw{T.tw + ((size_t)pid << T.log_n), q};
        uint32_t x[16];
        if constexpr (RS) {
            const int64_t mp = X.pr[pid];
#pragma unroll
            for (int k = 0; k < 16; k++) acc[t][k] = range_fix(acc[t][k], t31[t], t32[t]) + (int64_t)tl[k] * mp;
        }
#pragma unroll
        for (int k = 0; k < 16; k++) x[k] = (uint32_t)smr64(range_fix(acc[t][k], t31[t], t32[t]), q, qinv);
        uint32_t* dst = out + (size_t)B.out_off[tg] * n + 4 * col;
        by_class(q, [&](auto tag) {
            constexpr bool W = decltype(tag)::value;
            ct_stages<4, W>(x, pc, [&](int u, int b) { return tw[(1 << u) + b]; });
            if constexpr (G::NS2 > 0) {
                if (t) __syncthreads();  // previous target's LDS reads are done
#pragma unroll
                for (int k = 0; k < 16; k++) lds[col_lds<G::C>(r + G::R * k, c)] = x[k];
                __syncthreads();
#pragma unroll
                for (int k = 0; k < 16; k++) x[k] = lds[col_lds<G::C>(16 * r + k, c)];
                ct_stages<G::NS2, W>(x, pc, [&](int u, int b) {
                    return tw[(1 << (4 + u)) + (r << (4 - G::NS2 + u)) + b];
                });
            }
        });
        // rows 16 r + k (a column of 16 points: r = 0), in row groups of four
#pragma unroll
        for (int m = 0; m < 4; m++) {
            const uint32_t v[4] = {x[4 * m], x[4 * m + 1], x[4 * m + 2], x[4 * m + 3]};
            storev_u32<4>(dst + quad_row(16 * r + 4 * m), v);
        }
    }
}

// The sums of one target to forward values of its column pass; a fused rescale
// adds tl times mp first.  A sum is at most t 2^32 (8 products, or t 2^31 after
// a fix and 4 more: |y| <= 2^30, |m| < t/2), and the rescaling's product adds
// less than t 2^29: the reduction leaves |x| < (1 + 1/8 + 1/2) t < 2^31 for a
// wide prime, a forward value as it is.  A 31-bit prime's forward values end
// at q, which takes the sum within t 2^31: it is there already when n_in input
// primes' n_in (q_s / 2) (t / 2) is (ModUp of digits of up to 8 primes below
// 2^30; nofix), otherwise a range fix takes it there.
template <bool RS>
__device__ __forceinline__ void bconv_reduce(const int64_t (&acc)[4], const int32_t (&tl)[RS ? 4 : 1], int64_t mp,
                                             const PrimeC& p, bool nofix, uint32_t (&x)[4])
{
    const int64_t t31 = (int64_t)p.q << 31, t32 = (int64_t)p.q << 32;
    if (wide_prime(p.q) || (!RS && nofix)) {
#pragma unroll
        for (int k = 0; k < 4; k++) {
            int64_t a = acc[k];
            if constexpr (RS) a += (int64_t)tl[k] * mp;
            x[k] = (uint32_t)smr64(a, p.q, p.qinv);
        }
    } else {
#pragma unroll
        for (int k = 0; k < 4; k++) {
            int64_t a = acc[k];
            if constexpr (RS) a = range_fix(a, t31, t32) + (int64_t)tl[k] * mp;
            x[k] = (uint32_t)smr64(range_fix(a, t31, t32), p.q, p.qinv);
        }
    }
}

// ---------------------------------------------------------------------------
// BConv + NTT column pass with 4 residues per thread (Col4 geometry; lifted
// inputs in the 4-residue tile-thread layout of k_inv_cols4).  The group's
// input rows are requested together (four at a time: 54-56 VGPRs, 8
// work-groups per CU; eight at a time needs 74-80), with its matrix
// constants and its targets' twiddles (staged in LDS); the TPW targets'
// column transforms then run round by round together, one barrier per
// exchange.  Same residues as k_bconv_ntt_cols.
// ---------------------------------------------------------------------------
template <int LOG1, int TPW, bool RS, class BS>
__global__ void __launch_bounds__(NTT_THREADS) k_bconv_ntt_cols4(NttTables T, BS bs, const int32_t* y0,
                                                                  const int32_t* mat, uint32_t* out0, BcRescale X,
                                                                  size_t step, const BatchItem* items)
{
    using G = Col4<LOG1>;
    constexpr int CH = 4;  // input rows in flight (<= BCONV_MAT_PAD)
    const BcMap* Bp = bs.get();
    if (!Bp) return;
    GlobalBcMap& B = *(GlobalBcMap*)Bp;
    const int g = blockIdx.y;  // grid.y <= MAX_BC_GROUPS: the entries read below are in bounds
    const int groups = B.groups, n_in = B.n_in[g], n_tg = B.n_tg[g], first = B.first[g], in_off = B.in_off[g];
    if (g >= groups) return;
    const int32_t* y = y0 + (size_t)blockIdx.z * step;
    uint32_t* out = out0 + (size_t)blockIdx.z * step;
    __shared__ uint32_t lds[TPW * G::WORDS];
    __shared__ int2 twl[TPW << LOG1];
    const int c = threadIdx.x % G::C, t = threadIdx.x / G::C;
    const int tile = col4_tile<LOG1>(T.xcd_pair), col = tile * G::C + c;
    const size_t n = (size_t)1 << T.log_n;
    // the group's input rows start at ybase (uniform); this thread's four
    // residues sit at toff in each (a 32-bit offset from a scalar base)
    const uint32_t* ybase = reinterpret_cast<const uint32_t*>(y + (size_t)in_off * n + tile * G::TILE);
    const uint32_t toff = threadIdx.x * 4;

    // targets (a group's missing targets repeat its first; they are not stored)
    PrimeC tp[TPW];
    const int32_t* tws[TPW];
    const int32_t* tm[TPW];
    int64_t t31[TPW], t32[TPW];
#pragma unroll
    for (int i = 0; i < TPW; i++) {
        const int k = first + (i < n_tg ? i : 0);
        const int pid = B.pid[k];
        tp[i] = T.prime(pid);
        tws[i] = T.tw + ((size_t)pid << T.log_n);
        tm[i] = mat + B.mat_off[k];
        t31[i] = (int64_t)tp[i].q << 31, t32[i] = (int64_t)tp[i].q << 32;
    }
    // fused rescale: row e (after the inputs) and the conversion to q_{l-1}
    const int ql_pid = RS ? (items ? items[blockIdx.z].level : X.level) - 1 : 0;
    const int32_t* mlast = X.mlast + (size_t)ql_pid * X.n_p;
    uint32_t e[RS ? 4 : 1];
    if constexpr (RS) loadv_u32<4>(ybase + (size_t)n_in * n + toff, e);
    uint32_t yv[CH][4];
    auto load_rows = [&](int s0) {  // rows past the inputs repeat the last one (their constants are zero)
#pragma unroll
        for (int s = 0; s < CH; s++) loadv_u32<4>(ybase + (size_t)min(s0 + s, n_in - 1) * n + toff, yv[s]);
    };
    if (n_in > 0) load_rows(0);
    col4_stage_twiddles<LOG1, TPW>(twl, tws, tp);

    int64_t acc[TPW][4];
#pragma unroll
    for (int i = 0; i < TPW; i++)
#pragma unroll
        for (int k = 0; k < 4; k++) acc[i][k] = 0;
    int64_t accl[RS ? 4 : 1];
    uint32_t ql = 0;
    int64_t l31 = 0, l32 = 0;
    if constexpr (RS) {
        ql = T.mods[ql_pid];
        l31 = (int64_t)ql << 31, l32 = (int64_t)ql << 32;
#pragma unroll
        for (int k = 0; k < 4; k++) accl[k] = 0;
    }
    // Chunks of CH input rows: the chunk's matrix constants are requested
    // together, zero past the group's inputs (every matrix ends with CH spare
    // entries, so those reads stay in bounds), so a chunk is CH multiply-adds
    // per residue without branches.  A group's missing targets accumulate its
    // first target's row, unstored.  The first chunk (the only one when a
    // digit has at most CH primes) runs straight from the rows loaded above.
    auto mac_chunk = [&](int s0) {
        int32_t mv[TPW][CH], ml[RS ? CH : 1];
#pragma unroll
        for (int s = 0; s < CH; s++) {
            const bool in = s0 + s < n_in;
#pragma unroll
            for (int i = 0; i < TPW; i++) {
                const int32_t m = tm[i][s0 + s];
                mv[i][s] = in ? m : 0;
            }
            if constexpr (RS) {
                const int32_t m = mlast[s0 + s];
                ml[s] = in ? m : 0;
            }
        }
#pragma unroll
        for (int s1 = 0; s1 < CH; s1++) {
            if ((s1 & 3) == 0 && s0 + s1 >= 8) {  // lazy reduction: range fix after 8 products, then every 4
#pragma unroll
                for (int i = 0; i < TPW; i++)
#pragma unroll
                    for (int k = 0; k < 4; k++) acc[i][k] = range_fix(acc[i][k], t31[i], t32[i]);
                if constexpr (RS) {
#pragma unroll
                    for (int k = 0; k < 4; k++) accl[k] = range_fix(accl[k], l31, l32);
                }
            }
#pragma unroll
            for (int i = 0; i < TPW; i++)
#pragma unroll
                for (int k = 0; k < 4; k++) acc[i][k] += (int64_t)(int32_t)yv[s1][k] * (int64_t)mv[i][s1];
            if constexpr (RS) {
#pragma unroll
                for (int k = 0; k < 4; k++) accl[k] += (int64_t)(int32_t)yv[s1][k] * (int64_t)ml[s1];
            }
        }
    };
    if (n_in > 0) mac_chunk(0);
    for (int s0 = CH; s0 < n_in; s0 += CH) {
        load_rows(s0);
        mac_chunk(s0);
    }
    int32_t tl[RS ? 4 : 1];
    if constexpr (RS) {
        const uint32_t qlinv = T.qinvs[ql_pid];
#pragma unroll
        for (int k = 0; k < 4; k++) {
            const uint32_t cl = canon_signed(smr64(range_fix(accl[k], l31, l32), ql, qlinv), ql);
            const int32_t ei = (int32_t)e[k];
            const uint32_t ec = ei < 0 ? (uint32_t)(ei + (int32_t)ql) : (uint32_t)ei;
            tl[k] = lift(sub_mod(ec, cl, ql), ql);
        }
    }
    uint32_t x[TPW][4];
#pragma unroll
    for (int i = 0; i < TPW; i++) {
        int64_t mp = 0;
        if constexpr (RS) mp = X.pr[B.pid[first + (i < n_tg ? i : 0)]];
        bconv_reduce<RS>(acc[i], tl, mp, tp[i], X.nofix != 0, x[i]);
    }
    col4_fwd<LOG1, TPW>(x, tp, lds, twl, c, t);
#pragma unroll
    for (int i = 0; i < TPW; i++) {
        if (i >= n_tg) break;
        storev_u32<4>(out + (size_t)B.out_off[first + i] * n + (quad_row(4 * t) + 4 * col), x[i]);
    }
}

// ---------------------------------------------------------------------------
// INTT column pass, BConv and NTT column pass in one launch, for conversions
// of a few rows (a rescaling's dropped primes, narrow digits).  All three act
// on the columns of one tile: a work-group runs its group's input rows through
// the inverse column pass one after the other, lifts each and adds it to its
// targets' sums, and goes on as k_bconv_ntt_cols4.  The input rows' passes are
// repeated by every group of targets; that is what the launch it saves must
// outweigh (fuse_list).  Launch limb in_off + s of M is input row s.
// ---------------------------------------------------------------------------
template <int LOG1, int TPW, bool RS>
__global__ void __launch_bounds__(NTT_THREADS) k_inv_bconv_ntt_cols4(NttTables Tf, NttTables Ti, const LaunchMap* Mp,
                                                                     const BcMap* Bp, const uint32_t* w0,
                                                                     const int4* fc, const int32_t* mat,
                                                                     uint32_t* out, BcRescale X)
{
    using G = Col4<LOG1>;
    const LaunchMap& M = *Mp;
    const BcMap& B = *Bp;
    const int g = blockIdx.y;  // grid.y = groups
    const int n_in = B.n_in[g], n_tg = B.n_tg[g], first = B.first[g], l0 = B.in_off[g];
    __shared__ uint32_t lds[TPW * G::WORDS];
    __shared__ int2 twl[TPW << LOG1];
    __shared__ int2 twi[1 << LOG1];
    const int c = threadIdx.x % G::C, t = threadIdx.x / G::C;
    const int tile = col4_tile<LOG1>(Tf.xcd_pair), col = tile * G::C + c;
    const size_t n = (size_t)1 << Tf.log_n;
    auto load_row = [&](int l, uint32_t (&x)[4]) {
        const uint32_t* src = w0 + (size_t)M.in_off[l] * n + col;
#pragma unroll
        for (int k = 0; k < 4; k++) x[k] = src[(4 * t + k) * ROW];
    };
    uint32_t nx[4];
    load_row(l0, nx);

    PrimeC tp[TPW];
    const int32_t* tws[TPW];
    const int32_t* tm[TPW];
    int64_t t31[TPW], t32[TPW];
#pragma unroll
    for (int i = 0; i < TPW; i++) {  // a group's missing targets repeat its first; they are not stored
        const int k = first + (i < n_tg ? i : 0);
        const int pid = B.pid[k];
        tp[i] = Tf.prime(pid);
        tws[i] = Tf.tw + ((size_t)pid << Tf.log_n);
        tm[i] = mat + B.mat_off[k];
        t31[i] = (int64_t)tp[i].q << 31, t32[i] = (int64_t)tp[i].q << 32;
    }
    const int ql_pid = RS ? X.level - 1 : 0;
    const int32_t* mlast = X.mlast + (size_t)ql_pid * X.n_p;
    PrimeC pl{};
    int64_t l31 = 0, l32 = 0;
    if constexpr (RS) pl = Tf.prime(ql_pid), l31 = (int64_t)pl.q << 31, l32 = (int64_t)pl.q << 32;

    int64_t acc[TPW][4], accl[RS ? 4 : 1];
#pragma unroll
    for (int i = 0; i < TPW; i++)
#pragma unroll
        for (int k = 0; k < 4; k++) acc[i][k] = 0;
    if constexpr (RS) {
#pragma unroll
        for (int k = 0; k < 4; k++) accl[k] = 0;
    }
    int32_t tl[RS ? 4 : 1];
    const int rows = n_in + (RS ? 1 : 0);  // fused rescale: row n_in is e (BcRescale)
    for (int s = 0; s < rows; s++) {
        uint32_t x[4];
#pragma unroll
        for (int k = 0; k < 4; k++) x[k] = nx[k];
        const int pid = M.pid[l0 + s];
        const PrimeC pc = Ti.prime(pid);
        const int4 cst = fc[M.cidx[l0 + s]];
        const int32_t* const twsi[1] = {Ti.tw + ((size_t)pid << Ti.log_n)};
        const PrimeC pci[1] = {pc};
        if (s + 1 < rows) load_row(l0 + s + 1, nx);
        if (s) __syncthreads();  // the previous row's reads of lds and twi are done
        else col4_stage_twiddles<LOG1, TPW>(twl, tws, tp);
        col4_stage_twiddles<LOG1, 1>(twi, twsi, pci);
        by_class(pc.q, [&](auto tag) { col4_inv<LOG1, decltype(tag)::value>(x, pc, lds, twi, c, t, cst); });
        int32_t y[4];
#pragma unroll
        for (int k = 0; k < 4; k++) y[k] = lift(x[k], pc.q);
        if (RS && s == n_in) {
            if constexpr (RS) {
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    const uint32_t cl = canon_signed(smr64(range_fix(accl[k], l31, l32), pl.q, pl.qinv), pl.q);
                    const uint32_t ec = y[k] < 0 ? (uint32_t)(y[k] + (int32_t)pl.q) : (uint32_t)y[k];
                    tl[k] = lift(sub_mod(ec, cl, pl.q), pl.q);
                }
            }
            break;
        }
        const bool fix = s >= 8 && (s & 3) == 0;
#pragma unroll
        for (int i = 0; i < TPW; i++) {
            const int64_t m = tm[i][s];
#pragma unroll
            for (int k = 0; k < 4; k++)
                acc[i][k] = (fix ? range_fix(acc[i][k], t31[i], t32[i]) : acc[i][k]) + (int64_t)y[k] * m;
        }
        if constexpr (RS) {
            const int64_t m = mlast[s];
#pragma unroll
            for (int k = 0; k < 4; k++) accl[k] = (fix ? range_fix(accl[k], l31, l32) : accl[k]) + (int64_t)y[k] * m;
        }
    }
    uint32_t x[TPW][4];
#pragma unroll
    for (int i = 0; i < TPW; i++) {
        int64_t mp = 0;
        if constexpr (RS) mp = X.pr[B.pid[first + (i < n_tg ? i : 0)]];
        bconv_reduce<RS>(acc[i], tl, mp, tp[i], X.nofix != 0, x[i]);
    }
    __syncthreads();  // the last row's reads of lds are done
    col4_fwd<LOG1, TPW>(x, tp, lds, twl, c, t);
#pragma unroll
    for (int i = 0; i < TPW; i++) {
        if (i >= n_tg) break;
        storev_u32<4>(out + (size_t)B.out_off[first + i] * n + (quad_row(4 * t) + 4 * col), x[i]);
    }
}

// ---------------------------------------------------------------------------
// KeyMult (Sec. 2.3; Par.1): one output row r of R_{Q_l P} for all digits.
// For each digit j: the digit's own rows come straight from the input; every
// other row finishes its ModUp NTT here (row pass) and is multiplied into the
// accumulators with evk_j.  Q rows then take the HMult / HRot term times P
// and are stored; P rows run ModDown's INTT row pass and are stored.
// All accumulated values carry a factor 2^-64 (two Montgomery products),
// removed by ModDown's constants.
// ---------------------------------------------------------------------------
struct KmArgs {
    const uint32_t* up;   // ModUp column-pass output: digit j, row r at (j*(level+alpha) + r) * N
    const uint32_t* evk;  // [dnum][2][n_q+n_p][N]
    const uint32_t* b0;
    const uint32_t* a0;
    const uint32_t* b1;
    const uint32_t* a1;
    uint32_t* ks_q;       // [2][level][N]
    uint32_t* ks_p;       // [2][n_p + rs][N] (after the INTT row pass)
    const uint32_t* p_mod_q;
    const uint2* rinv;
    const uint2* p_r2;
    const uint2* r1;      // [n_q + n_p] x -> x 2^32 (folds a 64-bit KeyMult sum, k_keymult4)
    uint32_t galois;
    int level, n_q, n_p;
    int base;             // prime id of the level's first limb (a window of the list; 0 in batched launches)
    int rs;               // rows dropped by a rescaling that follows (0: none): they take the INTT row
                          // pass into slots n_p.. of ks_p, in row order
    int dlo, dhi;         // rows kept by that rescaling: [dlo, dhi) (dhi < 0: level - 1, single rescaling)
    const int32_t* lv;    // batched launch on a windowed context: per-level window data (Ctx::lv_tab)
    // batched launch (items != nullptr): item blockIdx.z takes its level, key
    // and Galois element from items and advances the pointers by these steps;
    // an item whose level is outside [lo_level, level] or whose key index is
    // outside [0, n_keys) is skipped
    const BatchItem* items;
    size_t in_step, in2_step, ws_step, key_step, up_step;
    int lo_level, n_keys, n_src;
    int n_rot;            // rotations of a hoisted launch (XcdRows)
    bool once;            // hoisted: key rows are loaded past the caches (KEYS_ONCE_BYTES)
};

// End of a KeyMult row: Q rows store ks; P rows (and the dropped row q_{l-1}
// when rescale follows) start ModDown with the INTT row pass, then store.
template <int LOG1>
__device__ __forceinline__ void keymult_store(const NttTables& Ti, const KmArgs& A, int r, int pid, int h, int rp,
                                              int rr, const PrimeC& pc, uint32_t* lds, const uint32_t (&acc0)[16],
                                              const uint32_t (&acc1)[16])
{
    const int log_n = Ti.log_n;
    const size_t n = (size_t)1 << log_n;
    const int j0 = h * ROW + 16 * rp;
    const int dhi = A.dhi < 0 ? A.level - 1 : A.dhi;
    const bool dropped = A.rs && r < A.level && (r < A.dlo || r >= dhi);
    const bool to_coef = r >= A.level || dropped;
    if (!to_coef) {
        store16_u32(A.ks_q + (size_t)r * n + j0, acc0);
        store16_u32(A.ks_q + ((size_t)A.level + r) * n + j0, acc1);
    } else {
        const TwTable twi{Ti.tw + ((size_t)pid << log_n), pc.q};
        const int slot = r >= A.level ? r - A.level : A.n_p + (r < A.dlo ? r : A.dlo + (r - dhi));
#pragma unroll
        for (int poly = 0; poly < 2; poly++) {
            uint32_t x[16];
#pragma unroll
            for (int k = 0; k < 16; k++) x[k] = poly ? acc1[k] : acc0[k];
            by_class(pc.q, [&](auto tag) {
                constexpr bool W = decltype(tag)::value;
                gs_stages<4, W, false>(x, pc, [&](int u, int b) {
                    return twi[(1 << (LOG1 + 4 + u)) + (h << (4 + u)) + (rp << u) + b];
                });
#pragma unroll
                for (int k = 0; k < 16; k++) lds[row_lds(rr, 16 * rp + k)] = x[k];
                __syncthreads();
#pragma unroll
                for (int k = 0; k < 16; k++) x[k] = lds[row_lds(rr, rp + 16 * k)];
                __syncthreads();
                gs_stages<4, W, false>(x, pc, [&](int u, int b) { return twi[(1 << (LOG1 + u)) + (h << u) + b]; });
            });
            uint32_t* dst = A.ks_p + ((size_t)poly * (A.n_p + A.rs) + slot) * n + (size_t)h * ROW;
#pragma unroll
            for (int k = 0; k < 16; k++) dst[rp + 16 * k] = x[k];
        }
    }
}

// Batched KeyMult launch: the item's level, window, key, rotation and
// pointers replace the launch's; false if the item is skipped.
__device__ __forceinline__ bool km_item(KmArgs& A, int log_n, int item)
{
    if (!A.items) return true;
    const BatchItem it = A.items[item];
    const size_t z = (size_t)item;
    if (!item_ok(it, A.lo_level, A.level, A.n_keys, A.n_src)) return false;
    A.level = it.level;
    if (A.lv) {  // windowed context: the item's window, and its rescaling's dropped rows
        constexpr int S = MAX_PRIMES + 1;
        A.base = A.lv[it.level];
        if (A.base < 0) return false;  // no window with this many limbs
        if (A.rs) {
            A.rs = A.lv[S + it.level];
            if (A.rs == 0) return false;  // no window below to rescale to
            A.dlo = A.lv[2 * S + it.level];
            A.dhi = A.lv[3 * S + it.level];
        }
    }
    A.galois = galois_of(it.rot, log_n);
    A.evk += (size_t)it.key * A.key_step;
    const size_t src = (size_t)it.src;  // input slot
    A.b0 += src * A.in_step;
    A.a0 += src * A.in_step;
    if (A.b1) A.b1 += src * A.in2_step;
    if (A.a1) A.a1 += src * A.in2_step;
    A.up += z * A.up_step;
    A.ks_q += z * A.ws_step;
    A.ks_p += z * A.ws_step;
    return true;
}

template <int LOG1, Own OWN, Extra EX>
__global__ void __launch_bounds__(NTT_THREADS) k_keymult(NttTables Tf, NttTables Ti, KmArgs A)
{
    __shared__ uint32_t lds[ROW_LDS_WORDS];
    if (!km_item(A, Tf.log_n, blockIdx.z)) return;
    const int r = blockIdx.y;  // row in q_b..q_{b+l-1}, p_0..
    if (r >= A.level + A.n_p) return;
    // window digit j is the part of key digit kd + j inside the window;
    // the window starts woff primes into key digit kd
    const int woff = A.base % A.n_p, kd = A.base / A.n_p;
    const int beta = (woff + A.level + A.n_p - 1) / A.n_p;
    const int log_n = Tf.log_n;
    const int pid = r < A.level ? A.base + r : A.n_q + (r - A.level);  // also the key row
    const PrimeC pc = Tf.prime(pid);
    const uint32_t q = pc.q, qinv = pc.qinv;
    const int rp = (threadIdx.x >> 2) & 15, rr = (int)((threadIdx.x & 3) | (threadIdx.x >> 6 << 2));  // as k_fwd_rows
    const int h = blockIdx.x * ROWS_PER_WG + rr;
    const int j0 = h * ROW + 16 * rp;
    const size_t n = (size_t)1 << log_n;
    const int rows = A.level + A.n_p, key_rows = A.n_q + A.n_p;

    uint32_t acc0[16], acc1[16];
#pragma unroll
    for (int k = 0; k < 16; k++) acc0[k] = acc1[k] = 0;

    // The row's prime is the same for every digit: its row-pass twiddles are
    // staged in LDS once, ahead of the digit loop.
    __shared__ int2 tws[OWN == Own::Hoisted ? 1 : ROWS_PER_WG * ROW_TW_SLOTS];
    if constexpr (OWN != Own::Hoisted) stage_row_twiddles<LOG1>(tws, Tf.tw + ((size_t)pid << log_n), blockIdx.x * ROWS_PER_WG, q);

    for (int j = 0; j < beta; j++) {
        // this digit's key rows are loaded first and arrive while x is formed
        uint32_t kb[16], ka[16];
        load16_u32(A.evk + ((size_t)(2 * (kd + j)) * key_rows + pid) * n + j0, kb);
        load16_u32(A.evk + ((size_t)(2 * (kd + j) + 1) * key_rows + pid) * n + j0, ka);
        uint32_t x[16];
        const int lo = max(j * A.n_p - woff, 0), hi = min((j + 1) * A.n_p - woff, A.level);
        if (r >= lo && r < hi) {
            const size_t off = (size_t)r * n;
            if constexpr (OWN == Own::Tensor) {
                uint32_t y[16];
                load16_u32(A.a0 + off + j0, x);
                load16_u32(A.a1 + off + j0, y);
                if constexpr (EX == Extra::HMult) {
                    // + P*d0, + P*d1 (d0 = b_a b_b, d1 = b_a a_b + a_a b_b) while a_a, a_b
                    // are in registers: this row's inputs are read once
                    uint32_t ba[16], bb[16];
                    load16_u32(A.b0 + off + j0, ba);
                    load16_u32(A.b1 + off + j0, bb);
                    const uint32_t pq = A.p_mod_q[pid];
#pragma unroll
                    for (int k = 0; k < 16; k++) {
                        const uint32_t d0 = mont(ba[k], bb[k], q, qinv);
                        const uint32_t d1 = add_mod(mont(ba[k], y[k], q, qinv), mont(x[k], bb[k], q, qinv), q);
                        acc0[k] = add_mod(acc0[k], mont(d0, pq, q, qinv), q);
                        acc1[k] = add_mod(acc1[k], mont(d1, pq, q, qinv), q);
                    }
                }
#pragma unroll
                for (int k = 0; k < 16; k++) x[k] = mont(x[k], y[k], q, qinv);
            } else {
                if constexpr (OWN == Own::Plain) {
                    load16_u32(A.a0 + off + j0, x);
                } else {  // Gather, Hoisted: phi_g(a)
#pragma unroll
                    for (int k = 0; k < 16; k += 4) AutQuad(j0 + k, A.galois, log_n).load(A.a0 + off, x + k);
                }
                const uint2 c = A.rinv[pid];
#pragma unroll
                for (int k = 0; k < 16; k++) x[k] = mulc(x[k], c, q);
            }
        } else if constexpr (OWN == Own::Hoisted) {
            // ModUp row already in the evaluation domain: gather phi_g on load
            const uint32_t* src = A.up + (size_t)(j * rows + r) * n;
#pragma unroll
            for (int k = 0; k < 16; k += 4) AutQuad(j0 + k, A.galois, log_n).load(src, x + k);
        } else {
            const uint32_t* src = A.up + (size_t)(j * rows + r) * n + quad_row(h);
#pragma unroll
            for (int k = 0; k < 16; k++) x[k] = src[4 * (rp + 16 * k)];
            by_class(q, [&](auto tag) {
                constexpr bool W = decltype(tag)::value;
                ct_stages<4, W>(x, pc, [&](int u, int b) { return row_tw1(tws, rr, u, b); });
#pragma unroll
                for (int k = 0; k < 16; k++) lds[row_lds(rr, rp + 16 * k)] = x[k];
                __syncthreads();
#pragma unroll
                for (int k = 0; k < 16; k++) x[k] = lds[row_lds(rr, 16 * rp + k)];
                __syncthreads();
                ct_stages<4, W>(x, pc, [&](int u, int b) { return row_tw2(tws, rr, rp, u, b); });
#pragma unroll
                for (int k = 0; k < 16; k++) x[k] = fwd_canon<W>(x[k], pc);
            });
        }
#pragma unroll
        for (int k = 0; k < 16; k++) {
            acc0[k] = add_mod(acc0[k], mont(x[k], kb[k], q, qinv), q);
            acc1[k] = add_mod(acc1[k], mont(x[k], ka[k], q, qinv), q);
        }
    }

    if (r < A.level) {
        if constexpr (EX == Extra::HRot) {
            const uint2 c = A.p_r2[pid];
            uint32_t x[16];
#pragma unroll
            for (int k = 0; k < 16; k += 4) AutQuad(j0 + k, A.galois, log_n).load(A.b0 + (size_t)r * n, x + k);
#pragma unroll
            for (int k = 0; k < 16; k++) acc0[k] = add_mod(acc0[k], mulc(x[k], c, q), q);
        }
    }
    keymult_store<LOG1>(Ti, A, r, pid, h, rp, rr, pc, lds, acc0, acc1);
}

// ---------------------------------------------------------------------------
// KeyMult with one wave per 256-point row (4 residues per thread, ROWS4 rows
// per work-group): four times the waves of k_keymult, for launches with few
// rows in flight.  Same inputs, outputs and residues as k_keymult.
//  * The ModUp rows finish their NTT row pass as four radix-4 rounds with
//    three exchanges between registers and lanes (as k_fwd_rows4); the
//    row's twelve twiddles per thread stay in registers across the digits.
//  * The digit products of a coefficient are summed exactly in 64 bits and
//    reduced once: x 2^-32 of the sum is the same residue as the sum of
//    per-digit Montgomery products (KmSum below).
//  * P rows (and the rows a following rescaling drops) run ModDown's INTT
//    row pass the same way before they are stored.
// ---------------------------------------------------------------------------
// Sums of products x k of one coefficient, k a canonical key residue.  A wide
// prime (q < 2^30) takes x as the row pass leaves it, any forward value
// (|x| < 0.97 2^31): the sum is signed, a row product counts 2 quarters of
// q 2^32 and a product of canonical residues 1, and up to 6 quarters the signed
// Montgomery reduction ends in (-2q, 2q).  A 31-bit prime takes canonical x:
// four products below q^2 fit unsigned, and redc64 reduces a sum below
// 2q 2^32.  Before the limit is passed the sum is folded:
// hi 2^32 + lo -> lo + [hi 2^32]_q, counted 1.
template <bool W>
struct KmSum {
    static constexpr int ROW = W ? 2 : 1, CANON = 1, LIMIT = W ? 6 : 4;
    uint64_t s;
    __device__ __forceinline__ void mac(uint32_t x, uint32_t k)
    {
        if constexpr (W) s += (uint64_t)((int64_t)(int32_t)x * (int64_t)(int32_t)k);
        else s += (uint64_t)x * k;
    }
    __device__ __forceinline__ void fold(uint2 r1, uint32_t q)
    {
        // a wide prime's high word lies in (-2q, 2q): 2q more is the same residue
        const uint32_t hi = (uint32_t)(s >> 32) + (W ? 2 * q : 0u);
        s = (uint64_t)(uint32_t)s + mulc(hi, r1, q);
    }
    // sum x 2^-32 in [0, q)
    __device__ __forceinline__ uint32_t reduce(uint32_t q, uint32_t qinv) const
    {
        if constexpr (W) {
            const uint32_t r = (uint32_t)smr64((int64_t)s, q, qinv);
            return red2(min(r, r + 2 * q), q);
        } else {
            // m = lo qinv makes s - m q divisible by 2^32 with equal low words,
            // so the quotient is hi - mulhi(m, q), in (-q, 2q)
            const uint32_t lo = (uint32_t)s, hi = (uint32_t)(s >> 32);
            const uint32_t t = __umulhi(lo * qinv, q);
            const uint32_t r = hi >= t ? hi - t : hi - t + q;
            return red2(r, q);
        }
    }
};

// ONCE: the key rows are loaded past the caches (hoisted launches; a branch in
// the kernel instead costs 0.25 % of a call of 32 rotations at N = 2^16)
template <int LOG1, Own OWN, Extra EX, bool ONCE = false>
__global__ void __launch_bounds__(NTT_THREADS) k_keymult4(NttTables Tf, NttTables Ti, KmArgs A)
{
    // row in q_b..q_{b+l-1}, p_0..: the P rows (the longest work: every digit
    // needs its row pass, then two INTT row passes) take the first grid rows,
    // so they are dispatched first and do not form the launch's tail
    int gy = blockIdx.y, tile = blockIdx.x, item = blockIdx.z;
    if constexpr (OWN == Own::Hoisted) {
        const XcdRows X(XcdGrid{blockIdx.x, blockIdx.y, blockIdx.z}, gridDim.y, A.level + A.n_p, row4_tiles<LOG1>(), A.n_rot);
        if (X.row < 0) return;
        gy = X.row, tile = X.tile, item = X.rot;
    }
    if (!km_item(A, Tf.log_n, item)) return;
    if (gy >= A.level + A.n_p) return;
    const int r = (gy + A.level) % (A.level + A.n_p);
    const int woff = A.base % A.n_p, kd = A.base / A.n_p;  // as in k_keymult
    const int beta = (woff + A.level + A.n_p - 1) / A.n_p;
    const int log_n = Tf.log_n;
    const int pid = r < A.level ? A.base + r : A.n_q + (r - A.level);  // also the key row
    const PrimeC pc = Tf.prime(pid);
    const uint32_t q = pc.q, qinv = pc.qinv;
    const int t = threadIdx.x & 63, w = wave_id();
    const int h = tile * ROWS4 + w;
    const int j0 = h * ROW + 4 * t;  // this thread's residues: row h, positions 4t .. 4t+3
    // contiguous accesses as a wave-uniform pointer (through row h) plus the
    // lane's 32-bit offset 4t (scalar-base loads and stores)
    const size_t hrow = (size_t)h * ROW;
    const uint32_t l4 = 4u * (uint32_t)t;
    const size_t n = (size_t)1 << log_n;
    const int rows = A.level + A.n_p, key_rows = A.n_q + A.n_p;

    by_class(q, [&](auto tag) {
    constexpr bool W = decltype(tag)::value;
    using Sum = KmSum<W>;
    int2 twf[4][3];
    if constexpr (OWN != Own::Hoisted) row4_twiddles<LOG1, false>(Tf.tw + ((size_t)pid << log_n), q, h, t, twf);
    Sum s0[4], s1[4];
#pragma unroll
    for (int k = 0; k < 4; k++) s0[k].s = s1[k].s = 0;
    int terms = 0;  // what s0 / s1 hold, in KmSum's count
    const uint2 r1 = A.r1[pid];
    constexpr bool EXTRA = OWN == Own::Tensor && EX == Extra::HMult;

    [[maybe_unused]] const AutQuad quad((uint32_t)j0, A.galois, log_n);
    // The digit whose own rows this row is (none for P rows).
    int jown = -1;
    for (int j = 0; j < beta; j++)
        if (r >= max(j * A.n_p - woff, 0) && r < min((j + 1) * A.n_p - woff, A.level)) jown = j;
    struct Dig {
        uint32_t kb[4], ka[4], x[4];
    };
    auto issue = [&](int j, Dig& d) {
        const uint32_t* kb = A.evk + (((size_t)(2 * (kd + j)) * key_rows + pid) * n + hrow) + l4;
        const uint32_t* ka = A.evk + (((size_t)(2 * (kd + j) + 1) * key_rows + pid) * n + hrow) + l4;
        if constexpr (ONCE) {
            load_once(kb, d.kb);
            load_once(ka, d.ka);
        } else {
            loadv_u32<4>(kb, d.kb);
            loadv_u32<4>(ka, d.ka);
        }
        if (j == jown) return;
        if constexpr (OWN == Own::Hoisted) {  // ModUp row already in the evaluation domain: gather phi_g
            loadv_u32<4>(A.up + (size_t)(j * rows + r) * n + quad.off, d.x);
        } else {
            const uint32_t* src = A.up + (size_t)(j * rows + r) * n + quad_row(h);
#pragma unroll
            for (int k = 0; k < 4; k++) d.x[k] = src[l4 + 256u * k];
        }
    };
    // digit j from cur; requests digit j + 1 into nxt first
    auto step = [&](int j, const uint32_t (&xo)[4], Dig& cur, Dig& nxt) {
        if (j + 1 < beta) issue(j + 1, nxt);
        const bool own = j == jown;
        const int more = own || OWN == Own::Hoisted ? Sum::CANON : Sum::ROW;
        if (terms + more > Sum::LIMIT) {  // uniform across the row
#pragma unroll
            for (int k = 0; k < 4; k++) s0[k].fold(r1, q), s1[k].fold(r1, q);
            terms = 1;
        }
        terms += more;
        uint32_t x[4];
        if (own) {
#pragma unroll
            for (int k = 0; k < 4; k++) x[k] = xo[k];
        } else {
            if constexpr (OWN == Own::Hoisted) {
                quad.arrange(make_uint4(cur.x[0], cur.x[1], cur.x[2], cur.x[3]), x);
            } else {
#pragma unroll
                for (int k = 0; k < 4; k++) x[k] = cur.x[k];
                row4_fwd<W>(x, pc, t, twf);
                if constexpr (!W) {
#pragma unroll
                    for (int k = 0; k < 4; k++) x[k] = fwd_canon<W>(x[k], pc);
                }
            }
        }
#pragma unroll
        for (int k = 0; k < 4; k++) {
            s0[k].mac(x[k], cur.kb[k]);
            s1[k].mac(x[k], cur.ka[k]);
        }
    };
    Dig da, db;
    // The row's own input is read first and taken at once: the own digit's
    // operand stays (4 registers instead of 16), and P d0 and P d1 join the sums
    // (d0 = b_a b_b, d1 = b_a a_b + a_a b_b) while digit 0's rows arrive.
    uint32_t xo[4];
    if (jown >= 0) {
        const size_t off = (size_t)r * n + hrow;
        uint32_t o0[4], o1[4], o2[4], o3[4];
        if constexpr (OWN == Own::Tensor) {
            loadv_u32<4>(A.a0 + off + l4, o0);
            loadv_u32<4>(A.a1 + off + l4, o1);
            if constexpr (EXTRA) {
                loadv_u32<4>(A.b0 + off + l4, o2);
                loadv_u32<4>(A.b1 + off + l4, o3);
            }
        } else if constexpr (OWN == Own::Plain) {
            loadv_u32<4>(A.a0 + off + l4, o0);
        } else {  // Gather, Hoisted: phi_g(a)
            quad.load(A.a0 + (size_t)r * n, o0);
        }
        issue(0, da);
        if constexpr (OWN == Own::Tensor) {
            if constexpr (EXTRA) {
                const uint32_t pq = A.p_mod_q[pid];
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    const uint32_t d0 = mont(o2[k], o3[k], q, qinv);
                    const uint32_t d1 = add_mod(mont(o2[k], o1[k], q, qinv), mont(o0[k], o3[k], q, qinv), q);
                    s0[k].mac(d0, pq);
                    s1[k].mac(d1, pq);
                }
                terms += Sum::CANON;
            }
#pragma unroll
            for (int k = 0; k < 4; k++) xo[k] = mont(o0[k], o1[k], q, qinv);
        } else {
            const uint2 c = A.rinv[pid];
#pragma unroll
            for (int k = 0; k < 4; k++) xo[k] = mulc(o0[k], c, q);
        }
    } else {
        issue(0, da);
    }
    for (int j = 0; j < beta; j += 2) {  // two digits per trip: the buffers swap roles without copies
        step(j, xo, da, db);
        if (j + 1 < beta) step(j + 1, xo, db, da);
    }

    uint32_t acc0[4], acc1[4];
#pragma unroll
    for (int k = 0; k < 4; k++) acc0[k] = s0[k].reduce(q, qinv), acc1[k] = s1[k].reduce(q, qinv);
    if (r < A.level) {
        if constexpr (EX == Extra::HRot) {
            const uint2 c = A.p_r2[pid];
            uint32_t x[4];
            quad.load(A.b0 + (size_t)r * n, x);
#pragma unroll
            for (int k = 0; k < 4; k++) acc0[k] = add_mod(acc0[k], mulc(x[k], c, q), q);
        }
    }

    // Q rows store ks; P rows (and the rows a following rescaling drops) start
    // ModDown with the INTT row pass, then store
    const int dhi = A.dhi < 0 ? A.level - 1 : A.dhi;
    const bool dropped = A.rs && r < A.level && (r < A.dlo || r >= dhi);
    if (r < A.level && !dropped) {
        storev_u32<4>(A.ks_q + ((size_t)r * n + hrow) + l4, acc0);
        storev_u32<4>(A.ks_q + (((size_t)A.level + r) * n + hrow) + l4, acc1);
        return;
    }
    int2 twi[4][3];
    row4_twiddles<LOG1, true>(Ti.tw + ((size_t)pid << log_n), q, h, t, twi);
    const int slot = r >= A.level ? r - A.level : A.n_p + (r < A.dlo ? r : A.dlo + (r - dhi));
#pragma unroll
    for (int poly = 0; poly < 2; poly++) {
        uint32_t x[4];
#pragma unroll
        for (int k = 0; k < 4; k++) x[k] = poly ? acc1[k] : acc0[k];
        row4_inv<W>(x, pc, t, twi);
        uint32_t* dst = A.ks_p + ((size_t)poly * (A.n_p + A.rs) + slot) * n + (size_t)h * ROW;
#pragma unroll
        for (int k = 0; k < 4; k++) dst[t + 64 * k] = x[k];
    }
    });
}

// ---------------------------------------------------------------------------
// Key switching at N = 2^12 in four launches.  A limb is 16 KB, so one
// work-group of 16 waves holds a whole transform: its 16 rows are the waves'
// (one-wave-per-row passes), its columns of 16 points are a thread's each (four
// waves, one radix-16 round), with LDS between the two.  The sequence is
//   k_small_intt      ModUp's INTT of a limb, lifted
//   k_small_modup     a digit's conversion to one row and its NTT
//   k_small_keymult   a row of one polynomial over all digits; P rows (and
//                     dropped ones) go on to ModDown's lifted INTT
//   k_small_moddown   an output row's conversion, NTT and combine
// Nothing is large here: a dependent launch and its kernel's shortest chain take
// about 3.5 us together and a whole transform's chain little more, so the number
// of launches (seven, or five with narrow digits) was the time.  One launch for conversions and KeyMult
// (a row's digits and both polynomials in one work-group) took 15.6 us against
// the two launches' 10: a row's chain is issued by one CU.  HMult + rescale,
// seven launches -> four: 24 limbs in three digits 29.5 -> 25.4 us, 8 limbs in
// two 28.8 -> 23.0; HRot 29.1 -> 23.4 and 28.5 -> 21.4.  At N = 2^13 a limb's
// chain on one CU is twice as long, about what the launches cost: the general
// sequence stays.  Lifted limbs are row-major.
// ---------------------------------------------------------------------------
constexpr int SM_LOG1 = 4, SM_LOG_N = SM_LOG1 + ROW_LOG, SM_ROWS = 1 << SM_LOG1, SM_THREADS = 64 * SM_ROWS;
constexpr int SM_N = 1 << SM_LOG_N;

// the 15 twiddles of a 16-point column (the same in every thread), requested
// with a kernel's other operands, ahead of its first barrier
struct SmallColTw {
    int32_t w[SM_ROWS - 1];
    uint32_t q;
    __device__ __forceinline__ SmallColTw(const int32_t* tw, uint32_t q_) : q(q_)
    {
#pragma unroll
        for (int i = 0; i < SM_ROWS - 1; i++) w[i] = tw[1 + i];
    }
    __device__ __forceinline__ int2 operator()(int u, int b) const { return const_from_quot(w[(1 << u) - 1 + b], q); }
};

// inverse column of 16 points in a thread (rows k of column c), constant folded, canonical
template <bool W>
__device__ __forceinline__ void small_inv_col(const uint32_t* buf, int c, const PrimeC& pc, const SmallColTw& tw, int4 cst,
                                              uint32_t (&y)[16])
{
#pragma unroll
    for (int k = 0; k < 16; k++) y[k] = buf[k * ROW + c];
    gs_stages<4, W, true>(y, pc, tw, cst);
}
template <bool W>
__device__ __forceinline__ void small_fwd_col(uint32_t* buf, int c, const PrimeC& pc, const SmallColTw& tw)
{
    uint32_t y[16];
#pragma unroll
    for (int k = 0; k < 16; k++) y[k] = buf[k * ROW + c];
    ct_stages<4, W>(y, pc, tw);
#pragma unroll
    for (int k = 0; k < 16; k++) buf[k * ROW + c] = y[k];
}
__device__ __forceinline__ void small_store_lifted(int32_t* dst, int c, const uint32_t (&y)[16], uint32_t q)
{
#pragma unroll
    for (int k = 0; k < 16; k++) dst[k * ROW + c] = lift(y[k], q);
}

// n_in products of lifted rows y (SM_N apart) with constants m, four residues
// from index e on: range fixes after 8 products, then every 4
__device__ __forceinline__ void small_bconv_sums(const int32_t* y, int e, int n_in, const int32_t* m, uint32_t q,
                                                 int64_t (&acc)[4])
{
#pragma unroll
    for (int k = 0; k < 4; k++) acc[k] = 0;
    for (int s0 = 0; s0 < n_in; s0 += 4) {
        uint32_t v[4][4];
        int32_t mv[4];
#pragma unroll
        for (int s = 0; s < 4; s++) {  // past the inputs: the last row again, times zero (BCONV_MAT_PAD)
            loadv_u32<4>(reinterpret_cast<const uint32_t*>(y) + (size_t)min(s0 + s, n_in - 1) * SM_N + e, v[s]);
            const int32_t c = m[s0 + s];
            mv[s] = s0 + s < n_in ? c : 0;
        }
        if (s0 >= 8) {
#pragma unroll
            for (int k = 0; k < 4; k++) acc[k] = range_fix(acc[k], (int64_t)q << 31, (int64_t)q << 32);
        }
#pragma unroll
        for (int s = 0; s < 4; s++)
#pragma unroll
            for (int k = 0; k < 4; k++) acc[k] += (int64_t)(int32_t)v[s][k] * (int64_t)mv[s];
    }
}

template <class Ld>
__global__ void __launch_bounds__(SM_THREADS) k_small_intt(NttTables T, const LaunchMap* Mr, const LaunchMap* Mc, Ld ld,
                                                           const int4* fc, int32_t* out)
{
    __shared__ uint32_t buf[SM_N];
    const int limb = blockIdx.x, pid = Mr->pid[limb];
    const PrimeC pc = T.prime(pid);
    const int t = threadIdx.x & 63, h = wave_id();
    const int32_t* twt = T.tw + (size_t)pid * SM_N;
    const SmallColTw tw(twt, pc.q);
    uint32_t x[4];
    ld.template loadv<4>(*Mr, limb, h * ROW + 4 * t, pc, x);
    int2 twr[4][3];
    row4_twiddles<SM_LOG1, true>(twt, pc.q, h, t, twr);
    const int4 cst = fc[Mc->cidx[limb]];
    by_class(pc.q, [&](auto tag) {
        constexpr bool W = decltype(tag)::value;
        row4_inv<W>(x, pc, t, twr);
#pragma unroll
        for (int k = 0; k < 4; k++) buf[h * ROW + t + 64 * k] = x[k];
        __syncthreads();
        if (h < ROW / 64) {
            uint32_t y[16];
            small_inv_col<W>(buf, threadIdx.x, pc, tw, cst, y);
            small_store_lifted(out + (size_t)limb * SM_N, threadIdx.x, y, pc.q);
        }
    });
}

// stand-alone transforms of a limb, in place
__global__ void __launch_bounds__(SM_THREADS) k_small_ntt(NttTables T, IdMap M, uint32_t* data)
{
    __shared__ uint32_t buf[SM_N];
    const int limb = blockIdx.x, pid = M.pid[limb];
    const PrimeC pc = T.prime(pid);
    const int t = threadIdx.x & 63, h = wave_id(), c = threadIdx.x % ROW;
    const int32_t* twt = T.tw + (size_t)pid * SM_N;
    const SmallColTw tw(twt, pc.q);
    uint32_t* d = data + (size_t)limb * SM_N;
    uint32_t y[16], x[4];
    if (h < ROW / 64) {
#pragma unroll
        for (int k = 0; k < 16; k++) y[k] = d[k * ROW + c];
    }
    int2 twr[4][3];
    row4_twiddles<SM_LOG1, false>(twt, pc.q, h, t, twr);
    by_class(pc.q, [&](auto tag) {
        constexpr bool W = decltype(tag)::value;
        if (h < ROW / 64) {
            ct_stages<4, W>(y, pc, tw);
#pragma unroll
            for (int k = 0; k < 16; k++) buf[k * ROW + c] = y[k];
        }
        __syncthreads();  // every column is read before a row is written
#pragma unroll
        for (int k = 0; k < 4; k++) x[k] = buf[h * ROW + t + 64 * k];
        row4_fwd<W>(x, pc, t, twr);
#pragma unroll
        for (int k = 0; k < 4; k++) x[k] = fwd_canon<W>(x[k], pc);
    });
    storev_u32<4>(d + h * ROW + 4 * t, x);
}
__global__ void __launch_bounds__(SM_THREADS) k_small_intt_plain(NttTables T, IdMap M, uint32_t* data, const int4* ninv)
{
    __shared__ uint32_t buf[SM_N];
    const int limb = blockIdx.x, pid = M.pid[limb];
    const PrimeC pc = T.prime(pid);
    const int t = threadIdx.x & 63, h = wave_id(), c = threadIdx.x % ROW;
    const int32_t* twt = T.tw + (size_t)pid * SM_N;
    const SmallColTw tw(twt, pc.q);
    uint32_t* d = data + (size_t)limb * SM_N;
    uint32_t x[4];
    loadv_u32<4>(d + h * ROW + 4 * t, x);
    int2 twr[4][3];
    row4_twiddles<SM_LOG1, true>(twt, pc.q, h, t, twr);
    const int4 cst = ninv[pid];
    by_class(pc.q, [&](auto tag) {
        constexpr bool W = decltype(tag)::value;
        row4_inv<W>(x, pc, t, twr);
#pragma unroll
        for (int k = 0; k < 4; k++) buf[h * ROW + t + 64 * k] = x[k];
        __syncthreads();
        if (h < ROW / 64) {
            uint32_t y[16];
            small_inv_col<W>(buf, c, pc, tw, cst, y);
#pragma unroll
            for (int k = 0; k < 16; k++) d[k * ROW + c] = y[k];
        }
    });
}

// digit blockIdx.y to row blockIdx.x of the level (own rows: nothing to do);
// out: evaluation domain, digit j's row r at (j rows + r)
struct SmallUp {
    const int32_t* y;      // lifted limbs of the level
    const int32_t* mat;    // constants of the level: digit jk, prime pid at (jk n_primes + pid) n_p
    uint32_t* out;
    int level, base, n_q, n_p, n_primes, nofix;
};
__global__ void __launch_bounds__(SM_THREADS) k_small_modup(NttTables T, SmallUp U)
{
    __shared__ uint32_t buf[SM_N];
    const int r = blockIdx.x, j = blockIdx.y;
    const int woff = U.base % U.n_p, kd = U.base / U.n_p;
    const int lo = max(j * U.n_p - woff, 0), hi = min((j + 1) * U.n_p - woff, U.level);
    if (r >= lo && r < hi) return;
    const int pid = r < U.level ? U.base + r : U.n_q + (r - U.level);
    const PrimeC pc = T.prime(pid);
    const int t = threadIdx.x & 63, h = wave_id(), e = h * ROW + 4 * t;
    const int32_t* twt = T.tw + (size_t)pid * SM_N;
    const SmallColTw tw(twt, pc.q);
    int2 twr[4][3];
    row4_twiddles<SM_LOG1, false>(twt, pc.q, h, t, twr);
    int64_t acc[4];
    small_bconv_sums(U.y + (size_t)lo * SM_N, e, hi - lo, U.mat + ((size_t)(kd + j) * U.n_primes + pid) * U.n_p, pc.q, acc);
    uint32_t x[4];
    const int32_t none[1] = {0};
    bconv_reduce<false>(acc, none, 0, pc, U.nofix != 0, x);
    storev_u32<4>(buf + e, x);
    __syncthreads();
    by_class(pc.q, [&](auto tag) {
        constexpr bool W = decltype(tag)::value;
        if (h < ROW / 64) small_fwd_col<W>(buf, threadIdx.x, pc, tw);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 4; k++) x[k] = buf[h * ROW + t + 64 * k];
        row4_fwd<W>(x, pc, t, twr);
#pragma unroll
        for (int k = 0; k < 4; k++) x[k] = fwd_canon<W>(x[k], pc);
    });
    storev_u32<4>(U.out + (size_t)(j * (U.level + U.n_p) + r) * SM_N + e, x);
}

// row blockIdx.x of polynomial blockIdx.y (k_keymult4's sums over evaluation-
// domain rows); dn: ModDown's INTT column map, the constant of slot k at cidx[k]
template <Own OWN, Extra EX>
__global__ void __launch_bounds__(SM_THREADS) k_small_keymult(NttTables Ti, KmArgs A, const LaunchMap* dn, const int4* fc,
                                                              int32_t* dn_y)
{
    __shared__ uint32_t buf[SM_N];
    const int rows = A.level + A.n_p, key_rows = A.n_q + A.n_p;
    const int r = blockIdx.x, poly = blockIdx.y;
    const int woff = A.base % A.n_p, kd = A.base / A.n_p;
    const int beta = (woff + A.level + A.n_p - 1) / A.n_p;
    const int pid = r < A.level ? A.base + r : A.n_q + (r - A.level);
    const PrimeC pc = Ti.prime(pid);
    const uint32_t q = pc.q, qinv = pc.qinv;
    const int t = threadIdx.x & 63, h = wave_id(), e = h * ROW + 4 * t;
    const int32_t* twt = Ti.tw + (size_t)pid * SM_N;
    const SmallColTw tw(twt, q);
    const uint2 r1 = A.r1[pid];
    const int dhi = A.dhi < 0 ? A.level - 1 : A.dhi;
    const bool dropped = A.rs && r < A.level && (r < A.dlo || r >= dhi);
    by_class(q, [&](auto tag) {
        constexpr bool W = decltype(tag)::value;
        using Sum = KmSum<W>;
        Sum s[4];
#pragma unroll
        for (int k = 0; k < 4; k++) s[k].s = 0;
        int terms = 0;
        auto room = [&](int more) {  // uniform across the work-group
            if (terms + more > Sum::LIMIT) {
#pragma unroll
                for (int k = 0; k < 4; k++) s[k].fold(r1, q);
                terms = 1;
            }
            terms += more;
        };
        for (int j = 0; j < beta; j++) {
            uint32_t key[4], x[4];
            loadv_u32<4>(A.evk + ((size_t)(2 * (kd + j) + poly) * key_rows + pid) * SM_N + e, key);
            if (r >= max(j * A.n_p - woff, 0) && r < min((j + 1) * A.n_p - woff, A.level)) {  // the digit's own row
                const size_t off = (size_t)r * SM_N + e;
                if constexpr (OWN == Own::Tensor) {
                    uint32_t a0[4], a1[4];
                    loadv_u32<4>(A.a0 + off, a0);
                    loadv_u32<4>(A.a1 + off, a1);
                    if constexpr (EX == Extra::HMult) {  // P d0 or P d1, as k_keymult4
                        uint32_t b0[4], b1[4];
                        loadv_u32<4>(A.b0 + off, b0);
                        loadv_u32<4>(A.b1 + off, b1);
                        const uint32_t pq = A.p_mod_q[pid];
                        room(Sum::CANON);
#pragma unroll
                        for (int k = 0; k < 4; k++)
                            s[k].mac(poly ? add_mod(mont(b0[k], a1[k], q, qinv), mont(a0[k], b1[k], q, qinv), q)
                                          : mont(b0[k], b1[k], q, qinv), pq);
                    }
#pragma unroll
                    for (int k = 0; k < 4; k++) x[k] = mont(a0[k], a1[k], q, qinv);
                } else {
                    if constexpr (OWN == Own::Plain) loadv_u32<4>(A.a0 + off, x);
                    else AutQuad((uint32_t)e, A.galois, SM_LOG_N).load(A.a0 + (size_t)r * SM_N, x);
                    const uint2 ri = A.rinv[pid];
#pragma unroll
                    for (int k = 0; k < 4; k++) x[k] = mulc(x[k], ri, q);
                }
            } else {
                loadv_u32<4>(A.up + (size_t)(j * rows + r) * SM_N + e, x);
            }
            room(Sum::CANON);
#pragma unroll
            for (int k = 0; k < 4; k++) s[k].mac(x[k], key[k]);
        }
        uint32_t acc[4];
#pragma unroll
        for (int k = 0; k < 4; k++) acc[k] = s[k].reduce(q, qinv);
        if constexpr (EX == Extra::HRot) {
            if (r < A.level && poly == 0) {
                const uint2 cb = A.p_r2[pid];
                uint32_t x[4];
                AutQuad((uint32_t)e, A.galois, SM_LOG_N).load(A.b0 + (size_t)r * SM_N, x);
#pragma unroll
                for (int k = 0; k < 4; k++) acc[k] = add_mod(acc[k], mulc(x[k], cb, q), q);
            }
        }
        if (r < A.level && !dropped) {
            storev_u32<4>(A.ks_q + ((size_t)poly * A.level + r) * SM_N + e, acc);
            return;
        }
        const int slot = r >= A.level ? r - A.level : A.n_p + (r < A.dlo ? r : A.dlo + (r - dhi));
        int2 twr[4][3];
        row4_twiddles<SM_LOG1, true>(twt, q, h, t, twr);
        row4_inv<W>(acc, pc, t, twr);
#pragma unroll
        for (int k = 0; k < 4; k++) buf[h * ROW + t + 64 * k] = acc[k];
        __syncthreads();
        if (h < ROW / 64) {
            uint32_t y[16];
            small_inv_col<W>(buf, threadIdx.x, pc, tw, fc[dn->cidx[slot]], y);
            small_store_lifted(dn_y + (size_t)(poly * (A.n_p + A.rs) + slot) * SM_N, threadIdx.x, y, q);
        }
    });
}

struct SmallDown {
    const int32_t* y;      // lifted rows of the two polynomials, `rows` each
    const int32_t* mat;    // output row i's constants at mat + i stride
    int rows, n_in, stride;
};

// launch limb l of M (ModDown's combine map) is an output row of one polynomial
template <bool RS>
__global__ void __launch_bounds__(SM_THREADS) k_small_moddown(NttTables T, const LaunchMap* Mp, SmallDown S, StCombine st,
                                                              BcRescale X)
{
    __shared__ uint32_t buf[SM_N];
    const LaunchMap& M = *Mp;
    const int l = blockIdx.x, pid = M.pid[l], poly = M.grp[l], i = M.out_off[l];
    const PrimeC pc = T.prime(pid);
    const int t = threadIdx.x & 63, h = wave_id(), e = h * ROW + 4 * t;
    const int32_t* twt = T.tw + (size_t)pid * SM_N;
    const SmallColTw tw(twt, pc.q);
    const int32_t* y = S.y + (size_t)(poly * S.rows) * SM_N;
    int2 twr[4][3];
    row4_twiddles<SM_LOG1, false>(twt, pc.q, h, t, twr);
    const auto pre = st.template prefetch<4>(M, l, e);
    int64_t acc[4];
    small_bconv_sums(y, e, S.n_in, S.mat + (size_t)i * S.stride, pc.q, acc);
    int32_t tl[RS ? 4 : 1];
    int64_t mp = 0;
    if constexpr (RS) {  // t = lift(e - conv_{l-1} P^-1), the dropped limb of the result (BcRescale)
        const PrimeC pl = T.prime(X.level - 1);
        int64_t al[4];
        uint32_t er[4];
        loadv_u32<4>(reinterpret_cast<const uint32_t*>(y) + (size_t)S.n_in * SM_N + e, er);
        small_bconv_sums(y, e, S.n_in, X.mlast + (size_t)(X.level - 1) * X.n_p, pl.q, al);
#pragma unroll
        for (int k = 0; k < 4; k++) {
            const uint32_t cl = canon_signed(smr64(range_fix(al[k], (int64_t)pl.q << 31, (int64_t)pl.q << 32), pl.q, pl.qinv), pl.q);
            const int32_t ei = (int32_t)er[k];
            tl[k] = lift(sub_mod(ei < 0 ? (uint32_t)(ei + (int32_t)pl.q) : (uint32_t)ei, cl, pl.q), pl.q);
        }
        mp = X.pr[pid];
    }
    uint32_t x[4];
    bconv_reduce<RS>(acc, tl, mp, pc, false, x);
    storev_u32<4>(buf + e, x);
    __syncthreads();
    by_class(pc.q, [&](auto tag) {
        constexpr bool W = decltype(tag)::value;
        if (h < ROW / 64) small_fwd_col<W>(buf, threadIdx.x, pc, tw);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 4; k++) x[k] = buf[h * ROW + t + 64 * k];
        row4_fwd<W>(x, pc, t, twr);
        st.template store_fwd<4, W>(M, l, e, x, pc, pre);
    });
}

// ---------------------------------------------------------------------------
// Sum of plaintext-weighted rotations (Sec. 5 Par.4/Par.5, Eq. 5): one
// KeyMult pass over all rotations.  For row r, rotation i: the shared ModUp
// rows (evaluation domain) and the own digit's input row are gathered
// through phi_i, multiplied into rotation i's key rows, weighted by the
// plaintext row pt_i and accumulated; Q rows also take P * pt_i * phi_i(b).
// One ModDown follows.  items[i] = {level, key, rot, -}.
// ---------------------------------------------------------------------------
// One wave per 256-point row, 4 residues per thread, as k_keymult4; the key
// rows and the ModUp row of the next digit (of the next rotation after the
// last) are requested while a digit is multiplied.  Bound by the key and
// plaintext rows, read once each (2 beta + 1 rows per row and rotation): 32
// rotations at N = 2^16, 24 limbs, three digits (1.9 GB) take 330 us, 5.7 TB/s.
// 16 residues per thread with single gathers and a Montgomery product per term
// took 483 us, this kernel with cached key and plaintext loads 398 us.
template <int LOG1>
__global__ void __launch_bounds__(NTT_THREADS) k_keymult_sum(NttTables Tf, NttTables Ti, KmArgs A,
                                                              const uint32_t* pts, size_t pt_step, int n_rot)
{
    const XcdRows X(XcdGrid{blockIdx.x, blockIdx.y, blockIdx.z}, gridDim.y, A.level + A.n_p, row4_tiles<LOG1>(), 1);
    const int r = X.row;
    if (r < 0) return;
    const int woff = A.base % A.n_p, kd = A.base / A.n_p;  // as in k_keymult
    const int beta = (woff + A.level + A.n_p - 1) / A.n_p;
    const int log_n = Tf.log_n;
    const int pid = r < A.level ? A.base + r : A.n_q + (r - A.level);  // also the key and plaintext row
    const PrimeC pc = Tf.prime(pid);
    const uint32_t q = pc.q, qinv = pc.qinv;
    const int t = threadIdx.x & 63, w = wave_id();
    const int h = X.tile * ROWS4 + w;
    const uint32_t j0 = (uint32_t)(h * ROW + 4 * t);
    const size_t n = (size_t)1 << log_n, hrow = (size_t)h * ROW;
    const uint32_t l4 = 4u * (uint32_t)t;
    const int rows = A.level + A.n_p, key_rows = A.n_q + A.n_p;
    const uint2 r1 = A.r1[pid];
    const bool q_row = r < A.level;
    int jown = -1;
    for (int j = 0; j < beta; j++)
        if (r >= max(j * A.n_p - woff, 0) && r < min((j + 1) * A.n_p - woff, A.level)) jown = j;

    by_class(q, [&](auto tag) {
        constexpr bool W = decltype(tag)::value;
        using Sum = KmSum<W>;
        struct Dig {
            uint32_t kb[4], ka[4], x[4];
        };
        // the rotation in hand and the one whose first digit is requested next
        struct Rot {
            int i;
            const uint32_t* evk;
            AutQuad quad;
        };
        auto rotation = [&](int i) {  // the first rotation from i on that is not skipped (uniform across the launch)
            BatchItem it{};
            for (; i < n_rot; i++) {
                it = A.items[i];
                if (item_ok(it, A.level, A.level, A.n_keys, 0)) break;
            }
            const uint32_t g = i < n_rot ? galois_of(it.rot, log_n) : 1u;
            return Rot{i, A.evk + (i < n_rot ? (size_t)it.key * A.key_step : 0), AutQuad(j0, g, log_n)};
        };
        auto issue = [&](const Rot& R, int j, Dig& d) {
            load_once(R.evk + (((size_t)(2 * (kd + j)) * key_rows + pid) * n + hrow) + l4, d.kb);
            load_once(R.evk + (((size_t)(2 * (kd + j) + 1) * key_rows + pid) * n + hrow) + l4, d.ka);
            loadv_u32<4>((j == jown ? A.a0 + (size_t)r * n : A.up + (size_t)(j * rows + r) * n) + R.quad.off, d.x);
        };
        Sum t0[4], t1[4];
#pragma unroll
        for (int k = 0; k < 4; k++) t0[k].s = t1[k].s = 0;
        int total = 0;  // what t0 / t1 hold, in KmSum's count
        const uint2 own_c = q_row ? A.rinv[pid] : make_uint2(0, 0), pb_c = q_row ? A.p_r2[pid] : make_uint2(0, 0);
        Rot cur = rotation(0);
        Dig d;
        if (cur.i < n_rot) issue(cur, 0, d);
        while (cur.i < n_rot) {
            uint32_t pm[4], pb[4];
            load_once(pts + (size_t)cur.i * pt_step + ((size_t)pid * n + hrow) + l4, pm);
            if (q_row) loadv_u32<4>(A.b0 + (size_t)r * n + cur.quad.off, pb);
            const Rot next = rotation(cur.i + 1);
            Sum s0[4], s1[4];
#pragma unroll
            for (int k = 0; k < 4; k++) s0[k].s = s1[k].s = 0;
            int terms = 0;
            for (int j = 0; j < beta; j++) {
                Dig nd;
                const bool last = j + 1 == beta;
                if (!last || next.i < n_rot) issue(last ? next : cur, last ? 0 : j + 1, nd);
                if (terms + Sum::CANON > Sum::LIMIT) {
#pragma unroll
                    for (int k = 0; k < 4; k++) s0[k].fold(r1, q), s1[k].fold(r1, q);
                    terms = 1;
                }
                terms += Sum::CANON;
                uint32_t x[4];
                cur.quad.arrange(make_uint4(d.x[0], d.x[1], d.x[2], d.x[3]), x);
                if (j == jown) {  // the digit's own row: phi(a) times R^-1, as in ModUp's own rows
#pragma unroll
                    for (int k = 0; k < 4; k++) x[k] = mulc(x[k], own_c, q);
                }
#pragma unroll
                for (int k = 0; k < 4; k++) s0[k].mac(x[k], d.kb[k]), s1[k].mac(x[k], d.ka[k]);
                d = nd;
            }
            // the weighted sums: canonical products p s (and p P phi(b)), reduced once after the last rotation
            if (total + 2 * Sum::CANON > Sum::LIMIT) {
#pragma unroll
                for (int k = 0; k < 4; k++) t0[k].fold(r1, q), t1[k].fold(r1, q);
                total = 1;
            }
            total += 2 * Sum::CANON;
            uint32_t bx[4];
            if (q_row) cur.quad.arrange(make_uint4(pb[0], pb[1], pb[2], pb[3]), bx);
#pragma unroll
            for (int k = 0; k < 4; k++) {
                t0[k].mac(s0[k].reduce(q, qinv), pm[k]);
                t1[k].mac(s1[k].reduce(q, qinv), pm[k]);
                if (q_row) t0[k].mac(mulc(bx[k], pb_c, q), pm[k]);  // P phi(b), with the R^-2 of ks
            }
            cur = next;
        }
        // the sums carry the R^-2 of ks; their reduction takes one R more, given back here
        uint32_t acc0[4], acc1[4];
#pragma unroll
        for (int k = 0; k < 4; k++) {
            acc0[k] = mulc(t0[k].reduce(q, qinv), r1, q);
            acc1[k] = mulc(t1[k].reduce(q, qinv), r1, q);
        }
        if (q_row) {
            storev_u32<4>(A.ks_q + ((size_t)r * n + hrow) + l4, acc0);
            storev_u32<4>(A.ks_q + (((size_t)A.level + r) * n + hrow) + l4, acc1);
            return;
        }
        int2 twi[4][3];
        row4_twiddles<LOG1, true>(Ti.tw + ((size_t)pid << log_n), q, h, t, twi);
#pragma unroll
        for (int poly = 0; poly < 2; poly++) {
            uint32_t x[4];
#pragma unroll
            for (int k = 0; k < 4; k++) x[k] = poly ? acc1[k] : acc0[k];
            row4_inv<W>(x, pc, t, twi);
            uint32_t* dst = A.ks_p + ((size_t)poly * A.n_p + (r - A.level)) * n + hrow;
#pragma unroll
            for (int k = 0; k < 4; k++) dst[t + 64 * k] = x[k];
        }
    });
}

// ---------------------------------------------------------------------------
// stand-alone base conversion (coefficient domain), one launch: a thread
// holds BC_VEC coefficients, forms the centred products of the input rows
// (a multiplication by [Shat_s^-1]_s and the lift) as they arrive, and adds
// them to BC_TG targets' int64 sums with the range fixes of Sec. 4.2 (|y_s| <=
// 2^30, |M_s| < t/2: after 8 products, then every 4), one signed Montgomery
// reduction each.  The constants come by value (a kernel argument holds 512
// matrix entries: 8 inputs to 64 targets, 64 inputs to 8; a larger conversion
// is several launches), so nothing is set up on the device.  Bound by the
// launch and the load latency: 8 -> 24 primes at N = 2^16 take 6.8 us on the
// GPU (12.0 in the three launches of a lifted copy, set-up and one target per
// thread).  8 targets of 2 coefficients keep 32 sum registers and the most
// work-groups that the products' recomputation per target group is worth.
// ---------------------------------------------------------------------------
constexpr int BC_VEC = 2, BC_TG = 8, BC_CONSTS = 512;
struct BconvArgs {
    int n_in, n_tg, log_n;
    uint32_t iq[MAX_PRIMES];        // input primes
    uint2 ic[MAX_PRIMES];           // [Shat_s^-1]_s twisted
    uint32_t tq[MAX_PRIMES], tqinv[MAX_PRIMES];  // targets
    int32_t m[BC_CONSTS];           // [n_tg][n_in] centred [Shat_s 2^32]_t
};
static_assert(sizeof(BconvArgs) + 16 <= 4096, "the constants must fit a kernel argument");

__global__ void __launch_bounds__(256) k_bconv(BconvArgs A, const uint32_t* in, uint32_t* out)
{
    constexpr int CH = 4;  // input rows in flight
    const size_t n = (size_t)1 << A.log_n;
    const size_t j = ((size_t)blockIdx.x * 256 + threadIdx.x) * BC_VEC;  // exact grid
    const int t0 = blockIdx.y * BC_TG;
    int64_t acc[BC_TG][BC_VEC];
#pragma unroll
    for (int g = 0; g < BC_TG; g++)
#pragma unroll
        for (int k = 0; k < BC_VEC; k++) acc[g][k] = 0;
    for (int s0 = 0; s0 < A.n_in; s0 += CH) {
        uint2 v[CH];
#pragma unroll
        for (int i = 0; i < CH; i++)
            v[i] = *reinterpret_cast<const uint2*>(in + (size_t)min(s0 + i, A.n_in - 1) * n + j);
        if (s0 >= 8) {
#pragma unroll
            for (int g = 0; g < BC_TG; g++) {
                const uint32_t q = A.tq[min(t0 + g, A.n_tg - 1)];
#pragma unroll
                for (int k = 0; k < BC_VEC; k++)
                    acc[g][k] = range_fix(acc[g][k], (int64_t)q << 31, (int64_t)q << 32);
            }
        }
#pragma unroll
        for (int i = 0; i < CH; i++) {
            if (s0 + i >= A.n_in) break;
            const uint32_t q = A.iq[s0 + i];
            const uint2 c = A.ic[s0 + i];
            const int32_t y[BC_VEC] = {lift(mulc(v[i].x, c, q), q), lift(mulc(v[i].y, c, q), q)};
#pragma unroll
            for (int g = 0; g < BC_TG; g++) {  // past the last target: the last one again, not stored
                const int32_t m = A.m[min(t0 + g, A.n_tg - 1) * A.n_in + s0 + i];
#pragma unroll
                for (int k = 0; k < BC_VEC; k++) acc[g][k] += (int64_t)y[k] * m;
            }
        }
    }
#pragma unroll
    for (int g = 0; g < BC_TG; g++) {
        if (t0 + g >= A.n_tg) break;
        const uint32_t q = A.tq[t0 + g], qinv = A.tqinv[t0 + g];
        uint32_t r[BC_VEC];
#pragma unroll
        for (int k = 0; k < BC_VEC; k++)
            r[k] = canon_signed(smr64(range_fix(acc[g][k], (int64_t)q << 31, (int64_t)q << 32), q, qinv), q);
        *reinterpret_cast<uint2*>(out + (size_t)(t0 + g) * n + j) = make_uint2(r[0], r[1]);
    }
}

// ---------------------------------------------------------------------------
// launch helpers
// ---------------------------------------------------------------------------
static NttTables tables(const Ctx& c, bool inverse)
{
    return NttTables{inverse ? c.tw_inv : c.tw_fwd, c.mods, c.qinvs, c.rcs, c.log_n, c.xcd_pair};
}

#define CKKS_DISPATCH_LOG1(log1, CALL)                  \
    switch (log1) {                                     \
    case 4: { constexpr int L1 = 4; CALL; } break;      \
    case 5: { constexpr int L1 = 5; CALL; } break;      \
    case 6: { constexpr int L1 = 6; CALL; } break;      \
    case 7: { constexpr int L1 = 7; CALL; } break;      \
    case 8: { constexpr int L1 = 8; CALL; } break;      \
    default: return set_error(-5, "unsupported ring degree"); \
    }

// Forward column passes of 4 residues per thread (c4) store rows in runs of a
// tile's columns, 16 bytes at N = 2^16 and 32 at 2^15, where 16 residues give
// runs of 64 and 128; once the 16-residue work-groups fill the chip, that is
// what counts.  NTT of n limbs (both passes), 4 -> 16 residues: N = 2^16, 8
// limbs 9.0 -> 9.3 us, 16 11.8 -> 11.4, 48 22.3 -> 20.4, 128 36.9 -> 30.4; 2^15,
// 48 limbs 13.6 -> 13.8, 64 16.0 -> 16.0, 128 24.4 -> 23.7; 2^14 (64-byte runs)
// 128 limbs 15.7 -> 16.3.
template <int L1>
static bool fwd_cols16(long groups) { return L1 == 8 ? groups >= 256 : L1 == 7 ? groups >= 512 : false; }
template <int L1, class MS, class Ld, class St>
static void fwd_cols(const Ctx& c, MS ms, int n, Ld ld, St st, hipStream_t s, int items_n = 1, bool c4 = false)
{
    if (c4 && !fwd_cols16<L1>((long)col_tiles<L1>() * n * items_n)) {
        CKKS_LAUNCH((k_fwd_cols4<L1, MS, Ld, St>), dim3(Col4<L1>::TILES, n, items_n), dim3(NTT_THREADS), 0, s,
                    tables(c, false), ms, ld, st);
        return;
    }
    const int ct = c4 ? NTT_THREADS : c.col_threads;
    if constexpr (L1 >= 5) {
        if (ct == 512) {
            CKKS_LAUNCH((k_fwd_cols<L1, MS, Ld, St, 512>), dim3(col_tiles<L1, 512>(), n, items_n), dim3(512), 0, s,
                        tables(c, false), ms, ld, st);
            return;
        }
    }
    if constexpr (L1 >= 7) {
        if (ct == 128) {
            CKKS_LAUNCH((k_fwd_cols<L1, MS, Ld, St, 128>), dim3(col_tiles<L1, 128>(), n, items_n), dim3(128), 0, s,
                        tables(c, false), ms, ld, st);
            return;
        }
    }
    CKKS_LAUNCH((k_fwd_cols<L1, MS, Ld, St>), dim3(col_tiles<L1>(), n, items_n), dim3(NTT_THREADS), 0, s,
                       tables(c, false), ms, ld, st);
}
// row passes: 16 residues per thread, or one wave per row (4); single
// operations (items_n == 1) and batched launches have knobs of their own
static int row_ept(const Ctx& c, int items_n) { return items_n > 1 ? c.rows_ept : c.rows_ept1; }
template <int L1, class MS, class Ld, class St>
static void fwd_rows(const Ctx& c, MS ms, int n, Ld ld, St st, hipStream_t s, int items_n = 1)
{
    if (row_ept(c, items_n) == 4)
        CKKS_LAUNCH((k_fwd_rows4<L1, MS, Ld, St>), dim3(row4_tiles<L1>(), n, items_n), dim3(NTT_THREADS), 0,
                           s, tables(c, false), ms, ld, st);
    else
        CKKS_LAUNCH((k_fwd_rows<L1, MS, Ld, St>), dim3(row_tiles<L1>(), n, items_n), dim3(NTT_THREADS), 0,
                           s, tables(c, false), ms, ld, st);
}
template <int L1, class MS, class Ld, class St>
static void inv_rows(const Ctx& c, MS ms, int n, Ld ld, St st, hipStream_t s, int items_n = 1)
{
    if (row_ept(c, items_n) == 4)
        CKKS_LAUNCH((k_inv_rows4<L1, MS, Ld, St>), dim3(row4_tiles<L1>(), n, items_n), dim3(NTT_THREADS), 0,
                           s, tables(c, true), ms, ld, st);
    else
        CKKS_LAUNCH((k_inv_rows<L1, MS, Ld, St>), dim3(row_tiles<L1>(), n, items_n), dim3(NTT_THREADS), 0,
                           s, tables(c, true), ms, ld, st);
}
// Inverse column passes of 4 residues per thread, where they are asked for
// (c4), give way to 16 in large launches: 64-byte instead of 16-byte runs of a
// row per tile at N = 2^16.
//  * Lifted residues (key switching), from 11 work-groups per CU on, where the
//    launch is counted as sized for its top level (a batch at uneven levels
//    leaves up to half of it empty).  Batches of multiplications and rotations,
//    4 -> 16: 2070 to 2392 work-groups at uneven levels 167.4 -> 171.7 us (45
//    items at N = 2^13), 190.0 -> 193.1 (24 at 2^14), 198.0 -> 201.8 (13 at
//    2^15), at even levels 337.5 -> 341; 2688 and 2760 the same; 3072 and more
//    271.2 -> 269.9 (8 items of 4 to 24 limbs at 2^16), 374.2 -> 365.3 (26 at
//    2^15), 2070 -> 1995 (64 at 2^16).
//  * Row-major residues (stand-alone INTT): the stores have the same short runs,
//    and two work-groups per CU are enough.  INTT of n limbs (both passes) at
//    N = 2^16: 24 limbs 14.3 -> 14.8, 32 17.4 -> 17.1, 48 22.2 -> 21.7, 64 25.5 ->
//    24.2, 96 30.8 -> 28.2, 128 36.6 -> 33.4; at 2^15 128 limbs 25.0 -> 25.4.
template <int L1, class St>
static bool inv_cols16(long groups) { return St::kTileThread ? groups >= 2816 : L1 == 8 && groups >= 512; }
template <int L1, class MS, class Ld, class St>
static void inv_cols(const Ctx& c, MS ms, int n, Ld ld, St st, hipStream_t s, int items_n = 1, bool c4 = false)
{
    if (c4 && !inv_cols16<L1, St>((long)col_tiles<L1>() * n * items_n)) {
        CKKS_LAUNCH((k_inv_cols4<L1, MS, Ld, St>), dim3(Col4<L1>::TILES, n, items_n), dim3(NTT_THREADS), 0, s,
                    tables(c, true), ms, ld, st);
        return;
    }
    const int ct = c4 ? NTT_THREADS : c.col_threads;
    if constexpr (L1 >= 5) {
        if (ct == 512) {
            CKKS_LAUNCH((k_inv_cols<L1, MS, Ld, St, 512>), dim3(col_tiles<L1, 512>(), n, items_n), dim3(512), 0, s,
                        tables(c, true), ms, ld, st);
            return;
        }
    }
    if constexpr (L1 >= 7) {
        if (ct == 128) {
            CKKS_LAUNCH((k_inv_cols<L1, MS, Ld, St, 128>), dim3(col_tiles<L1, 128>(), n, items_n), dim3(128), 0, s,
                        tables(c, true), ms, ld, st);
            return;
        }
    }
    CKKS_LAUNCH((k_inv_cols<L1, MS, Ld, St>), dim3(col_tiles<L1>(), n, items_n), dim3(NTT_THREADS), 0, s,
                       tables(c, true), ms, ld, st);
}

static int launched(const char* what) { return check_hip(hipGetLastError(), what); }
static MapByPtr ptr(const MapRef& m) { return MapByPtr{m.dev}; }
// key switching's column passes (INTT columns + BConv + NTT columns) with 4
// residues per thread: single operations and batched launches apart
static bool col4(const Ctx& c, int items_n) { return (items_n > 1 ? c.col_ept : c.col_ept1) == 4; }

template <int L1, int TPW, bool RS, class BS>
static void bconv_ntt(const Ctx& c, BS bs, int groups, int items_n, const int32_t* y, const int32_t* mat,
                      uint32_t* out, const BcRescale& X, size_t step, const BatchItem* items, hipStream_t s, bool c4)
{
    if (c4) {
        CKKS_LAUNCH((k_bconv_ntt_cols4<L1, TPW, RS, BS>), dim3(Col4<L1>::TILES, groups, items_n), dim3(NTT_THREADS),
                    0, s, tables(c, false), bs, y, mat, out, X, step, items);
        return;
    }
    const int ct = c.col_threads;
    if constexpr (L1 >= 5) {
        if (ct == 512) {
            CKKS_LAUNCH((k_bconv_ntt_cols<L1, TPW, 0, RS, BS, 512>), dim3(col_tiles<L1, 512>(), groups, items_n),
                        dim3(512), 0, s, tables(c, false), bs, y, mat, out, X, step, items);
            return;
        }
    }
    if constexpr (L1 >= 7) {
        if (ct == 128) {
            CKKS_LAUNCH((k_bconv_ntt_cols<L1, TPW, 0, RS, BS, 128>), dim3(col_tiles<L1, 128>(), groups, items_n),
                        dim3(128), 0, s, tables(c, false), bs, y, mat, out, X, step, items);
            return;
        }
    }
    CKKS_LAUNCH((k_bconv_ntt_cols<L1, TPW, 0, RS, BS>), dim3(col_tiles<L1>(), groups, items_n),
                       dim3(NTT_THREADS), 0, s, tables(c, false), bs, y, mat, out, X, step, items);
}

// one launch of the BConv + NTT column pass (map by pointer, or per level)
// tpw: targets per work-group the maps were built with (Ctx::tpw_up / tpw_dn)
template <bool RS, class BS>
static int launch_bconv_ntt(const Ctx& c, int tpw, BS bs, int groups, int items_n, const int32_t* y,
                            const int32_t* mat, uint32_t* out, const BcRescale& X, size_t step,
                            const BatchItem* items, hipStream_t s, bool c4)
{
    const int log1 = c.log_n - ROW_LOG;
    if (tpw == 1) { CKKS_DISPATCH_LOG1(log1, (bconv_ntt<L1, 1, RS>(c, bs, groups, items_n, y, mat, out, X, step, items, s, c4))); }
    else if (tpw == 2) { CKKS_DISPATCH_LOG1(log1, (bconv_ntt<L1, 2, RS>(c, bs, groups, items_n, y, mat, out, X, step, items, s, c4))); }
    else { CKKS_DISPATCH_LOG1(log1, (bconv_ntt<L1, 4, RS>(c, bs, groups, items_n, y, mat, out, X, step, items, s, c4))); }
    return launched("bconv+ntt cols");
}

template <bool RS>
static int launch_bconv_list(const Ctx& c, int tpw, const std::vector<BcRef>& bs, const int32_t* y,
                             const int32_t* mat, uint32_t* out, const BcRescale& X, hipStream_t s, bool c4)
{
    for (const BcRef& B : bs)
        if (int e = launch_bconv_ntt<RS>(c, tpw, BcByPtr{B.dev}, B.groups, 1, y, mat, out, X, 0, nullptr, s, c4))
            return e;
    return 0;
}

// Conversions that run as one launch from the INTT row pass to the NTT column
// pass (k_inv_bconv_ntt_cols4) instead of two.  It saves a launch (about 3 us
// of a dependent sequence, as much host time) and costs the input rows' column
// passes again for every group of targets (a fused rescaling's row e among
// them) and a chain of them in every work-group.  HMult + rescale, neither
// conversion in one launch -> both that the rule takes: one-prime digits 29.6 ->
// 23.1 us at N = 2^13 and 30.5 -> 27.8 at 2^16 (3 limbs), 53.1 -> 52.4 at 2^16 (8
// limbs, ModDown alone); two-prime digits 30.1 -> 26.5 at 2^13 and 36.8 -> 34.8 at
// 2^15 (8 limbs), 39.0 -> 38.1 at 2^16 (6 limbs; the largest repeat, 18 2^16).
// Past the line 10 limbs in two-prime digits at 2^16 (ModDown, 30 2^16) 50.0 ->
// 51.0, 16 limbs at 2^15 (24 2^16) 52.5 -> 53.0; with four-prime digits 12 limbs
// 45.3 -> 50.2.  Rescalings convert 1 to 3 dropped primes to one window:
// rational 20.1 -> 18.6 us with 3 at N = 2^16, single 30.5 -> 26.1 at 24 limbs,
// 44.6 -> 38.8 at 48 and 20.6 -> 13.5 at 4.
constexpr int FUSE_MAX_IN = 2, RR_FUSE_MAX_IN = 3;
constexpr size_t FUSE_MAX_REPEAT = (size_t)5 << 18;
// targets per work-group of the rescalings' conversions: 1 repeats the input
// rows' passes twice as often, 4 leaves 5 work-groups per CU (rational
// rescaling 18.6 us with 2, 20.2 with 4)
constexpr int RS_TPW = 2;
// extra: rows that pass through the inverse columns besides the inputs
static bool fuse_list(const Ctx& c, const std::vector<BcRef>& bs, int extra)
{
    int n_in = 0, groups = 0;
    for (const BcRef& B : bs) n_in = std::max(n_in, B.n_in_max), groups += B.groups;
    return n_in <= FUSE_MAX_IN && (((size_t)(n_in + extra) * groups) << c.log_n) <= FUSE_MAX_REPEAT;
}

template <bool RS>
static int launch_inv_bconv_list(const Ctx& c, int tpw, const MapRef& cols, const std::vector<BcRef>& bs,
                                 const uint32_t* w0, const int4* fc, const int32_t* mat, uint32_t* out,
                                 const BcRescale& X, hipStream_t s)
{
    const int log1 = c.log_n - ROW_LOG;
    for (const BcRef& B : bs) {
#define CKKS_FUSED(TPW)                                                                                          \
    CKKS_DISPATCH_LOG1(log1, CKKS_LAUNCH((k_inv_bconv_ntt_cols4<L1, TPW, RS>), dim3(Col4<L1>::TILES, B.groups),    \
                                         dim3(NTT_THREADS), 0, s, tables(c, false), tables(c, true), cols.dev,   \
                                         B.dev, w0, fc, mat, out, X))
        if (tpw == 1) { CKKS_FUSED(1) }
        else if (tpw == 2) { CKKS_FUSED(2) }
        else { CKKS_FUSED(4) }
#undef CKKS_FUSED
    }
    return launched("intt cols + bconv + ntt cols");
}

// Single operations at N = 2^12 (the launch-bound ring) run whole limbs per
// work-group: key switching in four launches, rescalings in two, transforms in
// one.  A launch and its kernel's chain take about 3.5 us together, more than
// the second pass of a limb adds to a work-group's chain: NTT 7.5 -> 5.1, INTT 7.4 -> 5.1, rescaling
// 11.0 -> 9.8, rational rescaling 13.3 -> 10.7 us.
// The settings other than one wave per row and 4-residue columns keep the
// general passes.
static bool small_ring(const Ctx& c)
{
    return c.log_n == SM_LOG_N && c.rows_ept1 == 4 && c.km_ept1 == 4 && c.col_ept1 == 4;
}
// a rescaling at N = 2^12: INTT of the dropped rows (`drop` per polynomial,
// lifted into y), then every output row's conversion, NTT and combine
static int small_rescale(const Ctx& c, const MapRef& rows, const MapRef& cols, const MapRef& out, const uint32_t* in,
                         const int4* fc, int drop, const int32_t* mat, const StCombine& st, int32_t* y, hipStream_t s)
{
    KTimer t(c, "rescale_small", s);
    CKKS_LAUNCH((k_small_intt<LdPlain>), dim3(rows.n), dim3(SM_THREADS), 0, s, tables(c, true), rows.dev, cols.dev,
                (LdPlain{in, c.log_n}), fc, y);
    CKKS_LAUNCH((k_small_moddown<false>), dim3(out.n), dim3(SM_THREADS), 0, s, tables(c, false), out.dev,
                (SmallDown{y, mat, drop, drop, drop}), st, BcRescale{});
    return launched("rescale");
}

// ---------------------------------------------------------------------------
// stand-alone NTT / INTT over a list of limbs (caller-chosen primes: maps by
// value)
// ---------------------------------------------------------------------------
int launch_ntt(const Ctx& c, bool inverse, uint32_t* data, const int32_t* pids, int n_limbs, hipStream_t s)
{
    const int log1 = c.log_n - ROW_LOG;
    const bool c4 = col4(c, 1);
    for (int base = 0; base < n_limbs; base += MAX_LAUNCH_LIMBS) {
        const int n = n_limbs - base < MAX_LAUNCH_LIMBS ? n_limbs - base : MAX_LAUNCH_LIMBS;
        MapByVal M{};
        M.m.count = n;
        for (int l = 0; l < n; l++) M.m.pid.w[l >> 2] |= (uint32_t)pids[base + l] << (8 * (l & 3));
        M.m.cidx = M.m.pid;
        uint32_t* d = data + (size_t)base * c.n;
        if (small_ring(c)) {
            KTimer t(c, inverse ? "intt" : "ntt", s);
            if (inverse) CKKS_LAUNCH(k_small_intt_plain, dim3(n), dim3(SM_THREADS), 0, s, tables(c, true), M.m, d, c.ninv);
            else CKKS_LAUNCH(k_small_ntt, dim3(n), dim3(SM_THREADS), 0, s, tables(c, false), M.m, d);
            if (int e = launched("ntt")) return e;
            continue;
        }
        LdPlain ld{d, c.log_n};
        StPlain st{d, c.ninv, c.log_n};
        if (!inverse) {
            { KTimer t(c, "ntt_cols", s); CKKS_DISPATCH_LOG1(log1, (fwd_cols<L1>(c, M, n, ld, st, s, 1, c4))); }
            { KTimer t(c, "ntt_rows", s); CKKS_DISPATCH_LOG1(log1, (fwd_rows<L1>(c, M, n, ld, st, s))); }
        } else {
            { KTimer t(c, "intt_rows", s); CKKS_DISPATCH_LOG1(log1, (inv_rows<L1>(c, M, n, ld, st, s))); }
            { KTimer t(c, "intt_cols", s); CKKS_DISPATCH_LOG1(log1, (inv_cols<L1>(c, M, n, ld, st, s, 1, c4))); }
        }
        if (int e = launched("ntt")) return e;
    }
    return 0;
}

// ---------------------------------------------------------------------------
// stand-alone BConv (coefficient domain)
// ---------------------------------------------------------------------------
size_t bconv_ws_bytes(const Ctx& c, int n_in, int n_out)
{
    return 4096 + (size_t)n_in * n_out * 4 + ((size_t)n_in << c.log_n) * 4;
}

int launch_bconv(const Ctx& c, const uint32_t* in, const int32_t* in_ids, int n_in, uint32_t* out,
                 const int32_t* out_ids, int n_out, void*, hipStream_t s)
{
    KTimer tm(c, "bconv", s);
    const size_t n = (size_t)1 << c.log_n;
    const int per = std::min(MAX_PRIMES, BC_CONSTS / n_in);  // targets per launch (n_in <= MAX_PRIMES: 8 or more)
    BconvArgs A;
    A.n_in = n_in;
    A.log_n = c.log_n;
    for (int i = 0; i < n_in; i++) A.iq[i] = (uint32_t)c.mod[in_ids[i]];
    for (int t0 = 0; t0 < n_out; t0 += per) {
        A.n_tg = std::min(per, n_out - t0);
        bconv_consts(c, in_ids, n_in, out_ids + t0, A.n_tg, t0 ? nullptr : A.ic, A.m);
        for (int t = 0; t < A.n_tg; t++) {
            const uint32_t q = (uint32_t)c.mod[out_ids[t0 + t]];
            A.tq[t] = q, A.tqinv[t] = inv32(q);
        }
        CKKS_LAUNCH(k_bconv, dim3((unsigned)(n / (256 * BC_VEC)), (unsigned)((A.n_tg + BC_TG - 1) / BC_TG)), dim3(256), 0,
                    s, A, in, out + (size_t)t0 * n);
    }
    return launched("bconv");
}

// ---------------------------------------------------------------------------
// key switching: ModUp (INTT, BConv, NTT), KeyMult, ModDown
// ---------------------------------------------------------------------------
// workspace (units of N residues):
//   W0 [max(level, 2 (alpha+d))]      INTT row-pass output; later the P rows of ks (+ the d rows a
//                                     rescaling drops: 1, or a windowed level's dropped rows)
//   W1 [max(level, 2 (alpha+d))] int32  lifted ModUp input; later lifted ModDown input
//   W2 [max(beta (level+alpha), 2 level)]  ModUp column-pass output; later ModDown conv
//   W3 [2 level]                      ks on the Q rows
struct KsLayout {
    size_t w0, w1, w2, w3, total;  // offsets in residues
};
static KsLayout ks_layout(const Ctx& c, int level)
{
    const size_t n = (size_t)c.n;
    const int d = c.rs_drop_max(level);
    const size_t a = (size_t)(level > 2 * (c.n_p + d) ? level : 2 * (c.n_p + d));
    // ModUp rows of the largest level up to `level` (a window below the top
    // one can start inside a key digit and need one digit more)
    size_t up = 0;
    for (int l = 1; l <= level; l++)
        if (c.has_level(l) && (size_t)c.digits(l) * (l + c.n_p) > up) up = (size_t)c.digits(l) * (l + c.n_p);
    const size_t b = up > (size_t)2 * level ? up : (size_t)2 * level;
    KsLayout L;
    L.w0 = 0;
    L.w1 = L.w0 + a * n;
    L.w2 = L.w1 + a * n;
    L.w3 = L.w2 + b * n;
    L.total = L.w3 + (size_t)2 * level * n;
    return L;
}

size_t keyswitch_ws_bytes(const Ctx& c, int level) { return ks_layout(c, level).total * 4; }

static dim3 xcd_grid(int rows, int tiles, int n_rot)
{
    const XcdGrid g = XcdRows::grid((uint32_t)rows, (uint32_t)tiles, (uint32_t)n_rot);
    return dim3(g.x, g.y, g.z);
}

template <int L1, Own OWN, Extra EX>
static void keymult(const Ctx& c, int max_level, int items_n, const KmArgs& A, hipStream_t s)
{
    const int rows = max_level + c.n_p;
    if ((items_n == 1 ? c.km_ept1 : c.km_ept) != 4) {
        CKKS_LAUNCH((k_keymult<L1, OWN, EX>), dim3(row_tiles<L1>(), rows, items_n), dim3(NTT_THREADS), 0, s,
                    tables(c, false), tables(c, true), A);
        return;
    }
    if constexpr (OWN == Own::Hoisted) {
        const dim3 grid = xcd_grid(rows, row4_tiles<L1>(), items_n);
        if (A.once)
            CKKS_LAUNCH((k_keymult4<L1, OWN, EX, true>), grid, dim3(NTT_THREADS), 0, s, tables(c, false), tables(c, true), A);
        else
            CKKS_LAUNCH((k_keymult4<L1, OWN, EX>), grid, dim3(NTT_THREADS), 0, s, tables(c, false), tables(c, true), A);
    } else {
        CKKS_LAUNCH((k_keymult4<L1, OWN, EX>), dim3(row4_tiles<L1>(), rows, items_n), dim3(NTT_THREADS), 0, s,
                    tables(c, false), tables(c, true), A);
    }
}

template <Own OWN, Extra EX>
static int keymult_dispatch(const Ctx& c, int max_level, int items_n, const KmArgs& A, hipStream_t s)
{
    CKKS_DISPATCH_LOG1(c.log_n - ROW_LOG, (keymult<L1, OWN, EX>(c, max_level, items_n, A, s)));
    return 0;
}

// Largest launch sizes over the context's levels in [lo, hi] (batched grids).
struct KsGrid {
    int up_rows = 0, up_cols = 0, up_bc = 0, dn_cols = 0, dn_bc = 0, dn_rows = 0;
};
static bool ks_grid(const Ctx& c, int lo, int hi, bool rescale, KsGrid& g)
{
    for (int level = lo; level <= hi; level++) {
        if (!c.has_level(level) || (rescale && c.windowed && !c.rr_below[level])) continue;
        const KsPlan& P = c.ks_plan[rescale ? 1 : 0][level];
        if (P.up_bc.size() != 1 || P.dn_bc.size() != 1) return false;
        g.up_rows = std::max(g.up_rows, P.up_rows.n);
        g.up_cols = std::max(g.up_cols, P.up_cols.n);
        g.up_bc = std::max(g.up_bc, P.up_bc[0].groups);
        g.dn_cols = std::max(g.dn_cols, P.dn_cols.n);
        g.dn_bc = std::max(g.dn_bc, P.dn_bc[0].groups);
        g.dn_rows = std::max(g.dn_rows, P.dn_rows.n);
    }
    return true;
}

// Where the phases of a key switch find their maps, workspace and items.
// Single operation: this level's plan, z = 1.  Batched: the per-level
// directory, z = items, workspace slices ws_step apart.
struct KsRun {
    const Ctx* c;
    const KsPlan* P = nullptr;  // single
    const KsDir* D = nullptr;   // batched
    const BatchItem* items = nullptr;
    int zn = 1, lo = 1, hi = 1, nk = 1, ns = 1;
    KsGrid g;
    size_t wst = 0;
    uint32_t* w0;
    int32_t* w1;
    uint32_t* w2;
    uint32_t* w3;
};

#define KS_MAP(R, field, CALL)                                      \
    do {                                                            \
        if ((R).D) {                                                \
            MapDir ms{(R).D->field, (R).items, (R).lo, (R).hi, (R).nk, (R).ns}; \
            CALL;                                                   \
        } else {                                                    \
            MapByPtr ms{(R).P->field.dev};                          \
            CALL;                                                   \
        }                                                           \
    } while (0)

static KsRun ks_run(const Ctx& c, void* ws, int top)
{
    KsRun R;
    R.c = &c;
    const KsLayout L = ks_layout(c, top);
    uint32_t* W = static_cast<uint32_t*>(ws);
    R.w0 = W + L.w0;
    R.w1 = reinterpret_cast<int32_t*>(W + L.w1);
    R.w2 = W + L.w2;
    R.w3 = W + L.w3;
    return R;
}

// ModUp: INTT (row and column pass, with the prologue of `own`), BConv +
// NTT column pass.  Leaves the lifted digits in w1 and the new rows' column
// pass in w2.
static int modup_phase(const KsRun& R, Own own, const KsIn& in, size_t s0, size_t s1, hipStream_t s)
{
    const Ctx& c = *R.c;
    const int log1 = c.log_n - ROW_LOG;
    const bool c4 = col4(c, R.zn);
    {
        StPlain st{R.w0, nullptr, c.log_n, R.wst};
        const uint32_t gal = (uint32_t)in.galois;
        KTimer t(c, "modup_intt_rows", s);
        switch (own) {
        case Own::Tensor: { LdOwn<Own::Tensor> ld{in.a0, in.a1, gal, c.log_n, s0, s1, R.items}; KS_MAP(R, up_rows, CKKS_DISPATCH_LOG1(log1, (inv_rows<L1>(c, ms, R.g.up_rows, ld, st, s, R.zn)))); } break;
        case Own::Gather: { LdOwn<Own::Gather> ld{in.a0, in.a1, gal, c.log_n, s0, s1, R.items}; KS_MAP(R, up_rows, CKKS_DISPATCH_LOG1(log1, (inv_rows<L1>(c, ms, R.g.up_rows, ld, st, s, R.zn)))); } break;
        default:          { LdOwn<Own::Plain> ld{in.a0, in.a1, gal, c.log_n, s0, s1, R.items};  KS_MAP(R, up_rows, CKKS_DISPATCH_LOG1(log1, (inv_rows<L1>(c, ms, R.g.up_rows, ld, st, s, R.zn)))); } break;
        }
        if (int e = launched("modup intt rows")) return e;
    }
    BcRescale X{};
    X.nofix = c.up_nofix;
    const int4* up_c = own == Own::Tensor ? c.up_c_r : c.up_c;
    if (!R.D && c4 && fuse_list(c, R.P->up_bc, 0)) {
        KTimer t(c, "modup_cols", s);
        return launch_inv_bconv_list<false>(c, c.tpw_up, R.P->up_cols, R.P->up_bc, R.w0, up_c, c.up_mat, R.w2,
                                            X, s);
    }
    {
        LdPlain ld{R.w0, c.log_n, R.wst};
        StLift st{R.w1, up_c, c.log_n, R.wst};
        KTimer t(c, "modup_intt_cols", s);
        KS_MAP(R, up_cols, CKKS_DISPATCH_LOG1(log1, (inv_cols<L1>(c, ms, R.g.up_cols, ld, st, s, R.zn, c4))));
        if (int e = launched("modup intt cols")) return e;
    }
    {
        KTimer t(c, "modup_bconv_ntt_cols", s);
        int e;
        if (R.D) e = launch_bconv_ntt<false>(c, c.tpw_up, BcDir{R.D->up_bc, R.items, R.lo, R.hi, R.nk, R.ns}, R.g.up_bc, R.zn, R.w1, c.up_mat, R.w2, X, R.wst, R.items, s, c4);
        else e = launch_bconv_list<false>(c, c.tpw_up, R.P->up_bc, R.w1, c.up_mat, R.w2, X, s, c4);
        if (e) return e;
    }
    return 0;
}

// ModDown: INTT column pass of the P rows (+ row l-1 when rescaling), BConv
// P -> Q + NTT column pass, NTT row pass + combine into out0 / out1.
static int moddown_phase(const KsRun& R, int level, bool rescale, uint32_t* out0, uint32_t* out1, size_t out_step,
                         hipStream_t s)
{
    const Ctx& c = *R.c;
    const int log1 = c.log_n - ROW_LOG;
    const bool rr = rescale && c.windowed;  // merged ModDown + rational rescaling
    const bool c4 = col4(c, R.zn);
    const int4* dn_c = rr ? c.rr_c : c.dn_c;
    const int32_t* dn_mat = rr ? c.rr_mat : c.dn_mat;
    const BcRescale X{c.rs_mlast, c.rs_pr, c.n_p, level};
    if (!R.D && c4 && fuse_list(c, R.P->dn_bc, rescale && !rr ? 1 : 0)) {
        KTimer t(c, "moddown_cols", s);
        if (int e = rescale && !rr
                        ? launch_inv_bconv_list<true>(c, c.tpw_dn, R.P->dn_cols, R.P->dn_bc, R.w0, dn_c, dn_mat, R.w2, X, s)
                        : launch_inv_bconv_list<false>(c, c.tpw_dn, R.P->dn_cols, R.P->dn_bc, R.w0, dn_c, dn_mat, R.w2, X, s))
            return e;
    } else {
    {
        LdPlain ld{R.w0, c.log_n, R.wst};
        StLift st{R.w1, dn_c, c.log_n, R.wst};
        KTimer t(c, "moddown_intt_cols", s);
        KS_MAP(R, dn_cols, CKKS_DISPATCH_LOG1(log1, (inv_cols<L1>(c, ms, R.g.dn_cols, ld, st, s, R.zn, c4))));
        if (int e = launched("moddown intt cols")) return e;
    }
    {
        KTimer t(c, "moddown_bconv_ntt_cols", s);
        int e;
        if (R.D) {
            const BcDir bd{R.D->dn_bc, R.items, R.lo, R.hi, R.nk, R.ns};
            if (rescale && !rr) e = launch_bconv_ntt<true>(c, c.tpw_dn, bd, R.g.dn_bc, R.zn, R.w1, dn_mat, R.w2, X, R.wst, R.items, s, c4);
            else e = launch_bconv_ntt<false>(c, c.tpw_dn, bd, R.g.dn_bc, R.zn, R.w1, dn_mat, R.w2, X, R.wst, R.items, s, c4);
        } else {
            if (rescale && !rr) e = launch_bconv_list<true>(c, c.tpw_dn, R.P->dn_bc, R.w1, dn_mat, R.w2, X, s, c4);
            else e = launch_bconv_list<false>(c, c.tpw_dn, R.P->dn_bc, R.w1, dn_mat, R.w2, X, s, c4);
        }
        if (e) return e;
    }
    }
    {
        LdQuads ld{R.w2, c.log_n, R.wst};
        StCombine st{out0, out1, R.w3, rr ? c.rr_fin : rescale ? c.rs_fin : c.dn_pinv, c.log_n, out_step, R.wst};
        KTimer t(c, "moddown_ntt_rows_combine", s);
        KS_MAP(R, dn_rows, CKKS_DISPATCH_LOG1(log1, (fwd_rows<L1>(c, ms, R.g.dn_rows, ld, st, s, R.zn))));
        if (int e = launched("moddown ntt rows")) return e;
    }
    return 0;
}

static int keymult_launch(const Ctx& c, Own own, Extra extra, int top, int zn, const KmArgs& A, hipStream_t s)
{
    KTimer t(c, "keymult", s);
    int e;
    if (own == Own::Tensor && extra == Extra::HMult) e = keymult_dispatch<Own::Tensor, Extra::HMult>(c, top, zn, A, s);
    else if (own == Own::Plain && extra == Extra::None) e = keymult_dispatch<Own::Plain, Extra::None>(c, top, zn, A, s);
    else if (own == Own::Gather && extra == Extra::HRot) e = keymult_dispatch<Own::Gather, Extra::HRot>(c, top, zn, A, s);
    else if (own == Own::Hoisted && extra == Extra::HRot) e = keymult_dispatch<Own::Hoisted, Extra::HRot>(c, top, zn, A, s);
    else return set_error(-1, "unsupported key-switch variant");
    if (e) return e;
    return launched("keymult");
}

static KmArgs km_args(const Ctx& c, const KsRun& R, const KsIn& in, const uint32_t* evk, int level, bool rescale)
{
    KmArgs A{};
    A.up = R.w2;
    A.evk = evk;
    A.b0 = in.b0;
    A.a0 = in.a0;
    A.b1 = in.b1;
    A.a1 = in.a1;
    A.ks_q = R.w3;
    A.ks_p = R.w0;
    A.p_mod_q = c.p_mod_q;
    A.rinv = c.rinv;
    A.p_r2 = c.p_r2;
    A.r1 = c.r1;
    A.galois = (uint32_t)in.galois;
    A.level = level;
    A.n_q = c.n_q;
    A.n_p = c.n_p;
    A.base = c.wbase[level];  // batched launches run on prefix contexts only (base 0 at every level)
    A.rs = rescale ? c.rs_drop(level) : 0;
    A.dlo = c.windowed ? c.rr_dlo[level] : 0;
    A.dhi = c.windowed ? c.rr_dhi[level] : -1;
    A.lv = nullptr;  // set for batched launches on a windowed context
    A.lo_level = R.lo;
    A.n_keys = R.nk;
    A.n_src = R.ns;
    return A;
}

// One operation at N = 2^12 takes the four-launch sequence.
static bool small_switch(const Ctx& c, int level)
{
    // Up to four one-prime digits the general sequence's conversions fuse into
    // five launches of smaller work-groups.  HMult + rescale, general against
    // four launches, one-prime digits: 3 limbs 22.3 : 22.9 us, 4 23.3 : 23.6, 5
    // 24.4 : 24.2, 8 26.9 : 25.9, 12 34.6 : 28.8, 24 65.2 : 43.0, 48 153 : 73;
    // two-prime: 4 limbs 24.2 : 22.8, 8 25.4 : 23.9, 48 91 : 50; four-prime: 12
    // limbs 25.9 : 23.5, 48 60.5 : 38.1; eight: 24 limbs 27.2 : 25.5, 56 51.9 : 33.1.
    if (c.n_p == 1 && c.digits(level) <= 4) return false;
    return small_ring(c);
}

static int small_keyswitch(const Ctx& c, const KsRun& R, Own own, Extra extra, const KsIn& in, int level,
                           const uint32_t* evk, uint32_t* out0, uint32_t* out1, hipStream_t s, bool rescale)
{
    const KsPlan& P = *R.P;
    const bool rr = rescale && c.windowed;
    const int pst = c.n_p + (rescale ? c.rs_drop(level) : 0), wb = c.wbase[level];
    const NttTables Tf = tables(c, false), Ti = tables(c, true);
    const uint32_t gal = (uint32_t)in.galois;
    {
        KTimer t(c, "modup_intt", s);
        const int4* fc = own == Own::Tensor ? c.up_c_r : c.up_c;
#define CKKS_SMALL_INTT(OWN)                                                                                     \
    CKKS_LAUNCH((k_small_intt<LdOwn<OWN>>), dim3(level), dim3(SM_THREADS), 0, s, Ti, P.up_rows.dev, P.up_cols.dev,        \
                (LdOwn<OWN>{in.a0, in.a1, gal, c.log_n, 0, 0, nullptr}), fc, R.w1)
        if (own == Own::Tensor) CKKS_SMALL_INTT(Own::Tensor);
        else if (own == Own::Gather) CKKS_SMALL_INTT(Own::Gather);
        else CKKS_SMALL_INTT(Own::Plain);
#undef CKKS_SMALL_INTT
        if (int e = launched("modup intt")) return e;
    }
    {
        KTimer t(c, "modup", s);
        const SmallUp U{R.w1, c.up_mat + (size_t)level * c.dnum * c.n_primes * c.n_p, R.w2, level, wb, c.n_q, c.n_p,
                        c.n_primes, c.up_nofix};
        CKKS_LAUNCH(k_small_modup, dim3(level + c.n_p, c.digits(level)), dim3(SM_THREADS), 0, s, Tf, U);
        if (int e = launched("modup")) return e;
    }
    {
        KTimer t(c, "keymult", s);
        const KmArgs A = km_args(c, R, in, evk, level, rescale);
        const LaunchMap* dn = P.dn_cols.dev;
        const int4* fc = rr ? c.rr_c : c.dn_c;
        int32_t* dn_y = reinterpret_cast<int32_t*>(R.w0);
        const dim3 grid(level + c.n_p, 2);
        if (own == Own::Tensor && extra == Extra::HMult)
            CKKS_LAUNCH((k_small_keymult<Own::Tensor, Extra::HMult>), grid, dim3(SM_THREADS), 0, s, Ti, A, dn, fc, dn_y);
        else if (own == Own::Plain && extra == Extra::None)
            CKKS_LAUNCH((k_small_keymult<Own::Plain, Extra::None>), grid, dim3(SM_THREADS), 0, s, Ti, A, dn, fc, dn_y);
        else if (own == Own::Gather && extra == Extra::HRot)
            CKKS_LAUNCH((k_small_keymult<Own::Gather, Extra::HRot>), grid, dim3(SM_THREADS), 0, s, Ti, A, dn, fc, dn_y);
        else return set_error(-1, "unsupported key-switch variant");
        if (int e = launched("keymult")) return e;
    }
    {
        KTimer t(c, "moddown", s);
        const SmallDown S{reinterpret_cast<const int32_t*>(R.w0), rr ? c.rr_mat + c.rr_mat_off[level] : c.dn_mat + (size_t)wb * c.n_p,
                          pst, rr ? pst : c.n_p, rr ? pst : c.n_p};
        const StCombine st{out0, out1, R.w3, rr ? c.rr_fin : rescale ? c.rs_fin : c.dn_pinv, c.log_n};
        const BcRescale X{c.rs_mlast, c.rs_pr, c.n_p, level};
        if (rescale && !rr) CKKS_LAUNCH((k_small_moddown<true>), dim3(P.dn_rows.n), dim3(SM_THREADS), 0, s, Tf, P.dn_rows.dev, S, st, X);
        else CKKS_LAUNCH((k_small_moddown<false>), dim3(P.dn_rows.n), dim3(SM_THREADS), 0, s, Tf, P.dn_rows.dev, S, st, X);
        return launched("moddown");
    }
}

// Shared sequence of a single (b == nullptr) or batched key switch.
static int keyswitch_seq(const Ctx& c, Own own, Extra extra, const KsIn& in, int level, const KsBatch* b,
                         const uint32_t* evk, uint32_t* out0, uint32_t* out1, void* ws, hipStream_t s, bool rescale)
{
    const int rsi = rescale ? 1 : 0;
    const int top = b ? b->max_level : level;  // layout and grids are sized for this level
    KsRun R = ks_run(c, ws, top);
    if (b) {
        if (!ks_grid(c, rescale && !c.windowed ? 2 : 1, top, rescale, R.g) || !c.ks_dir[rsi].up_rows)
            return set_error(-5, "batched key switching is not available at these levels");
        R.D = &c.ks_dir[rsi];
        R.items = b->items;
        R.zn = b->n;
        R.lo = rescale && !c.windowed ? 2 : 1;
        R.hi = top;
        R.nk = b->n_keys;
        R.ns = b->n_src;
        R.wst = b->ws_step;
    } else {
        R.P = &c.ks_plan[rsi][level];
        if (!R.P->up_rows.dev) return set_error(-5, "no launch plan for this level");
        R.g.up_rows = R.P->up_rows.n, R.g.up_cols = R.P->up_cols.n;
        R.g.dn_cols = R.P->dn_cols.n, R.g.dn_rows = R.P->dn_rows.n;
        if (small_switch(c, level)) return small_keyswitch(c, R, own, extra, in, level, evk, out0, out1, s, rescale);
    }
    if (int e = modup_phase(R, own, in, b ? b->in_step : 0, b ? b->in2_step : 0, s)) return e;
    KmArgs A = km_args(c, R, in, evk, top, rescale);
    if (b) {
        A.items = b->items;
        A.in_step = b->in_step, A.in2_step = b->in2_step, A.key_step = b->key_step;
        A.ws_step = A.up_step = b->ws_step;
        if (c.windowed) A.lv = c.lv_tab;
    }
    if (int e = keymult_launch(c, own, extra, top, R.zn, A, s)) return e;
    return moddown_phase(R, level, rescale, out0, out1, b ? b->out_step : 0, s);
}

// A hoisted launch loads its keys past the caches (load_once) where they are
// more than half of the 256 MB last-level cache: a program rotates by the same
// keys again, and keys that it holds from the last call are read from there.
// 32 rotations at N = 2^12, past the caches -> through them: 25 rows in three
// digits (77 MB) 76.9 -> 70.0 us, 32 rows (100 MB) 85.9 -> 80.2, 25 rows in four
// (105 MB) 80.5 -> 74.7; N = 2^14, 8 rotations of 25 rows (79 MB) 78.6 -> 75.0;
// beyond the line 17 rows in two digits (142 MB) 125.7 -> 131.3, 25 in three
// (314 MB) 191 -> 205.5; N = 2^12, 64 rotations of 32 rows (201 MB) 130 -> 141.
constexpr size_t KEYS_ONCE_BYTES = (size_t)128 << 20;

// Hoisted HRot: one ModUp of a (materialised in the evaluation domain),
// then KeyMult with the automorphism gathered on load and ModDown for every
// rotation at once (grid.z = rotation).  Workspace: one key-switch layout
// for the shared ModUp, then one per rotation.
int launch_hrot_hoisted(const Ctx& c, const uint32_t* b_in, const uint32_t* a_in, int level, int n_rot,
                        const BatchItem* items, const uint32_t* keys, int n_keys, size_t key_step, uint32_t* outs,
                        void* ws, hipStream_t s)
{
    const int log1 = c.log_n - ROW_LOG;
    const KsPlan& P = c.ks_plan[0][level];
    if (!P.up_rows.dev || !P.up_nrows.dev || !c.ks_dir[0].dn_bc) return set_error(-5, "no launch plan for this level");
    const size_t slice = keyswitch_ws_bytes(c, level) / 4;
    KsRun U = ks_run(c, ws, level);  // shared ModUp
    U.P = &P;
    U.g.up_rows = P.up_rows.n, U.g.up_cols = P.up_cols.n;
    KsIn in;
    in.b0 = b_in;
    in.a0 = a_in;
    if (int e = modup_phase(U, Own::Plain, in, 0, 0, s)) return e;
    {  // complete the ModUp rows in the evaluation domain (row pass in place)
        LdQuads ld{U.w2, c.log_n};
        StPlain st{U.w2, nullptr, c.log_n};
        KTimer t(c, "modup_ntt_rows", s);
        CKKS_DISPATCH_LOG1(log1, (fwd_rows<L1>(c, MapByPtr{P.up_nrows.dev}, P.up_nrows.n, ld, st, s)));
        if (int e = launched("modup ntt rows")) return e;
    }
    KsRun R = ks_run(c, static_cast<uint32_t*>(ws) + slice, level);  // rotation 0's slice
    R.D = &c.ks_dir[0];
    R.items = items;
    R.zn = n_rot;
    R.lo = R.hi = level;
    R.nk = n_keys;
    R.ns = 0;  // every rotation reads the one input; item slots are not used
    R.wst = slice;
    if (!ks_grid(c, level, level, false, R.g)) return set_error(-5, "no launch plan for this level");
    KmArgs A = km_args(c, R, in, keys, level, false);
    A.up = U.w2;
    A.items = items;
    A.key_step = key_step;
    A.ws_step = slice;
    A.up_step = 0;
    A.n_rot = n_rot;
    const size_t key_bytes = (size_t)2 * c.digits(level) * (level + c.n_p) * c.n * 4;  // rows that a rotation reads
    A.once = (size_t)std::min(n_rot, n_keys) * key_bytes > KEYS_ONCE_BYTES;
    if (int e = keymult_launch(c, Own::Hoisted, Extra::HRot, level, n_rot, A, s)) return e;
    const size_t out_step = 2 * (size_t)level * c.n;
    return moddown_phase(R, level, false, outs, outs + (size_t)level * c.n, out_step, s);
}

template <int L1>
static void keymult_sum(const Ctx& c, int level, const KmArgs& A, const uint32_t* pts, size_t pt_step, int n_rot,
                        hipStream_t s)
{
    CKKS_LAUNCH((k_keymult_sum<L1>), xcd_grid(level + c.n_p, row4_tiles<L1>(), 1), dim3(NTT_THREADS), 0, s,
                tables(c, false), tables(c, true), A, pts, pt_step, n_rot);
}

// Sum of plaintext-weighted rotations: the hoisted ModUp (as above), one
// KeyMult pass over every rotation, one ModDown.  Workspace: the shared
// ModUp layout, then one key-switch layout.
int launch_hrot_sum_hoisted(const Ctx& c, const uint32_t* b_in, const uint32_t* a_in, int level, int n_rot,
                            const BatchItem* items, const uint32_t* keys, int n_keys, size_t key_step,
                            const uint32_t* pts, size_t pt_step, uint32_t* out, void* ws, hipStream_t s)
{
    const int log1 = c.log_n - ROW_LOG;
    const KsPlan& P = c.ks_plan[0][level];
    if (!P.up_rows.dev || !P.up_nrows.dev) return set_error(-5, "no launch plan for this level");
    const size_t slice = keyswitch_ws_bytes(c, level) / 4;
    KsRun U = ks_run(c, ws, level);
    U.P = &P;
    U.g.up_rows = P.up_rows.n, U.g.up_cols = P.up_cols.n;
    KsIn in;
    in.b0 = b_in;
    in.a0 = a_in;
    if (int e = modup_phase(U, Own::Plain, in, 0, 0, s)) return e;
    {
        LdQuads ld{U.w2, c.log_n};
        StPlain st{U.w2, nullptr, c.log_n};
        KTimer t(c, "modup_ntt_rows", s);
        CKKS_DISPATCH_LOG1(log1, (fwd_rows<L1>(c, MapByPtr{P.up_nrows.dev}, P.up_nrows.n, ld, st, s)));
        if (int e = launched("modup ntt rows")) return e;
    }
    KsRun R = ks_run(c, static_cast<uint32_t*>(ws) + slice, level);
    R.P = &P;
    R.g.up_rows = P.up_rows.n, R.g.up_cols = P.up_cols.n;
    R.g.dn_cols = P.dn_cols.n, R.g.dn_rows = P.dn_rows.n;
    R.nk = n_keys;
    KmArgs A = km_args(c, R, in, keys, level, false);
    A.up = U.w2;
    A.items = items;
    A.key_step = key_step;
    {
        KTimer t(c, "keymult_sum", s);
        CKKS_DISPATCH_LOG1(log1, (keymult_sum<L1>(c, level, A, pts, pt_step, n_rot, s)));
        if (int e = launched("keymult sum")) return e;
    }
    return moddown_phase(R, level, false, out, out + (size_t)level * c.n, 0, s);
}

int launch_keyswitch(const Ctx& c, Own own, Extra extra, const KsIn& in, int level, const uint32_t* evk,
                     uint32_t* out0, uint32_t* out1, void* ws, hipStream_t s, bool rescale)
{
    if (rescale && c.rs_out(level) < 1) return set_error(-1, "no level below this one to rescale to");
    return keyswitch_seq(c, own, extra, in, level, nullptr, evk, out0, out1, ws, s, rescale);
}

int launch_keyswitch_batch(const Ctx& c, Own own, Extra extra, const KsIn& in, const KsBatch& b,
                           const uint32_t* evk, uint32_t* out0, uint32_t* out1, void* ws, hipStream_t s,
                           bool rescale)
{
    if (b.n < 1 || b.n > 65535) return set_error(-1, "batch size out of range");
    return keyswitch_seq(c, own, extra, in, b.max_level, &b, evk, out0, out1, ws, s, rescale);
}

// ---------------------------------------------------------------------------
// rescale: t = lift(INTT(c_{l-1})), c'_i = (c_i - NTT([t]_{q_i})) q_{l-1}^-1
// ---------------------------------------------------------------------------
size_t rescale_ws_bytes(const Ctx& c) { return ((size_t)4 + 2 * (size_t)c.n_q) * (size_t)c.n * 4; }

int launch_rescale(const Ctx& c, const uint32_t* in, int level_in, uint32_t* out, void* ws, hipStream_t s)
{
    const int log1 = c.log_n - ROW_LOG;
    const RsPlan& P = c.rs_plan[level_in];
    if (!P.rows.dev) return set_error(-5, "no launch plan for this level");
    if (small_ring(c))
        return small_rescale(c, P.rows, P.cols, P.nrows, in, c.ninv, 1, c.rs_mat,
                             StCombine{out, out + (size_t)(level_in - 1) * c.n, in, c.rs_qinv, c.log_n},
                             static_cast<int32_t*>(ws), s);
    uint32_t* w0 = static_cast<uint32_t*>(ws);  // [2] INTT row pass of the last limbs
    uint32_t* w2 = w0 + 4 * (size_t)c.n;        // [2 (l-1)] NTT column pass of [t]_{q_i}
    {
        LdPlain ld{in, c.log_n};
        StPlain st{w0, nullptr, c.log_n};
        KTimer t(c, "rescale_intt_rows", s);
        CKKS_DISPATCH_LOG1(log1, (inv_rows<L1>(c, ptr(P.rows), 2, ld, st, s)));
        if (int e = launched("rescale intt rows")) return e;
    }
    {
        KTimer t(c, "rescale_cols", s);
        if (int e = launch_inv_bconv_list<false>(c, RS_TPW, P.cols, P.bc, w0, c.ninv, c.rs_mat, w2, BcRescale{}, s))
            return e;
    }
    {
        LdQuads ld{w2, c.log_n};
        StCombine st{out, out + (size_t)(level_in - 1) * c.n, in, c.rs_qinv, c.log_n};
        KTimer t(c, "rescale_ntt_rows_combine", s);
        CKKS_DISPATCH_LOG1(log1, (fwd_rows<L1>(c, ptr(P.nrows), P.nrows.n, ld, st, s)));
        if (int e = launched("rescale ntt rows")) return e;
    }
    return 0;
}

// ---------------------------------------------------------------------------
// launch plans: every map an internal launch needs, built once per context
// ---------------------------------------------------------------------------
namespace {

struct Blob {
    std::vector<char> bytes;
    size_t add(const void* p, size_t n)
    {
        const size_t off = (bytes.size() + 255) & ~(size_t)255;
        bytes.resize(off + n);
        std::memcpy(bytes.data() + off, p, n);
        return off;
    }
};

// offsets are stored in the pointer fields until the blob is uploaded
template <class T>
T* as_off(size_t off) { return reinterpret_cast<T*>(off); }
template <class T>
void rebase(const T*& p, char* base) { p = reinterpret_cast<const T*>(base + reinterpret_cast<size_t>(p)); }

MapRef add_map(Blob& b, LaunchMap m, int n)
{
    m.count = n;
    return MapRef{as_off<const LaunchMap>(b.add(&m, sizeof m)), n};
}

// groups of at most tpw targets sharing input rows; one BcMap per launch
struct BcBuilder {
    Blob& blob;
    int tpw;
    std::vector<BcRef>& out;
    BcMap B{};
    int groups = 0, targets = 0, n_in_max = 0;
    void flush()
    {
        if (!groups) return;
        B.groups = groups;
        out.push_back(BcRef{as_off<const BcMap>(blob.add(&B, sizeof B)), groups, n_in_max});
        B = BcMap{};
        groups = targets = n_in_max = 0;
    }
    void add(int in_off, int n_in, int n, const int32_t* mat_off, const int32_t* out_off, const int8_t* pid)
    {
        for (int i = 0; i < n; i += tpw) {
            const int cnt = n - i < tpw ? n - i : tpw;
            if (groups == MAX_BC_GROUPS || targets + cnt > MAX_LAUNCH_LIMBS) flush();
            B.in_off[groups] = in_off;
            B.n_in[groups] = n_in;
            B.first[groups] = targets;
            B.n_tg[groups] = cnt;
            for (int k = 0; k < cnt; k++) {
                B.mat_off[targets + k] = mat_off[i + k];
                B.out_off[targets + k] = out_off[i + k];
                B.pid[targets + k] = pid[i + k];
            }
            groups++;
            targets += cnt;
            n_in_max = n_in > n_in_max ? n_in : n_in_max;
        }
    }
};

void build_ks_plan(const Ctx& c, Blob& b, int level, bool rescale, KsPlan& P)
{
    const int alpha = c.n_p, beta = c.digits(level), rows = level + alpha;
    const int rs = rescale ? c.rs_drop(level) : 0, pst = alpha + rs, out_rows = rescale ? c.rs_out(level) : level;
    const int wb = c.wbase[level];  // prime id of the level's first limb
    // merged ModDown + rational rescaling (windowed context): the rows after
    // P in ks_p are the dropped window rows in row order; outputs are the
    // window below, starting at prime id ob
    const bool rr = rescale && c.windowed;
    const int ob = rr ? c.wbase[out_rows] : wb;
    int dpid[MAX_PRIMES] = {};
    for (int r = 0, k = 0; rr && r < level; r++)
        if (r < c.rr_dlo[level] || r >= c.rr_dhi[level]) dpid[k++] = wb + r;
    {  // ModUp INTT passes over the level limbs
        LaunchMap M{};
        for (int i = 0; i < level; i++) {
            M.in_off[i] = M.out_off[i] = i;
            M.pid[i] = (wb + i);
            M.cidx[i] = (level * c.n_q + wb + i);
        }
        P.up_rows = add_map(b, M, level);
        P.up_cols = add_map(b, M, level);
    }
    {  // ModUp rows other than each digit's own, for the evaluation-domain row pass (hoisted HRot)
        LaunchMap M{};
        int n = 0;
        for (int j = 0; j < beta; j++) {
            const int lo = c.digit_lo(j, level), hi = c.digit_hi(j, level);
            for (int r = 0; r < rows; r++) {
                if (r >= lo && r < hi) continue;
                if (n < MAX_LAUNCH_LIMBS) {
                    M.in_off[n] = M.out_off[n] = j * rows + r;
                    M.pid[n] = c.row_pid(r, level);
                }
                n++;
            }
        }
        if (n <= MAX_LAUNCH_LIMBS) P.up_nrows = add_map(b, M, n);
    }
    {  // ModUp BConv: digit j -> every other row
        BcBuilder bb{b, c.tpw_up, P.up_bc};
        int32_t mo[2 * MAX_PRIMES], oo[2 * MAX_PRIMES];
        int8_t pd[2 * MAX_PRIMES];
        for (int j = 0; j < beta; j++) {
            const int lo = c.digit_lo(j, level), hi = c.digit_hi(j, level);
            int n = 0;
            for (int r = 0; r < rows; r++) {
                if (r >= lo && r < hi) continue;
                const int pid = c.row_pid(r, level);
                mo[n] = ((level * c.dnum + c.key_digit(j, level)) * c.n_primes + pid) * c.n_p;
                oo[n] = j * rows + r;
                pd[n] = (int8_t)pid;
                n++;
            }
            bb.add(lo, hi - lo, n, mo, oo, pd);
        }
        bb.flush();
    }
    {  // ModDown INTT column pass (P rows, and row q_{l-1} when rescaling)
        LaunchMap M{};
        for (int poly = 0; poly < 2; poly++)
            for (int k = 0; k < pst; k++) {
                const int l = poly * pst + k;
                M.in_off[l] = M.out_off[l] = l;
                if (rr) {
                    M.pid[l] = (k < alpha ? c.n_q + k : dpid[k - alpha]);
                    M.cidx[l] = (c.rr_c_off[level] + k);
                } else {
                    M.pid[l] = (k < alpha ? c.n_q + k : level - 1);
                    M.cidx[l] = (k < alpha ? k : c.n_p + level - 1);
                }
            }
        P.dn_cols = add_map(b, M, 2 * pst);
    }
    {  // ModDown BConv P -> Q (merged: P u dropped rows -> the window below)
        BcBuilder bb{b, c.tpw_dn, P.dn_bc};
        int32_t mo[MAX_PRIMES], oo[MAX_PRIMES];
        int8_t pd[MAX_PRIMES];
        for (int poly = 0; poly < 2; poly++) {
            for (int i = 0; i < out_rows; i++) {
                mo[i] = rr ? c.rr_mat_off[level] + i * pst : (wb + i) * c.n_p;
                oo[i] = poly * out_rows + i;
                pd[i] = (int8_t)(ob + i);
            }
            bb.add(poly * pst, rr ? pst : alpha, out_rows, mo, oo, pd);
        }
        bb.flush();
    }
    {  // ModDown NTT row pass + combine: the two polynomials' limbs of a prime
        // are neighbours in the map (launch limbs 2i, 2i + 1), so the work-groups
        // that read a row's twiddles twice run together on one XCD (grid.x is a
        // multiple of 8) and the second read hits its L2
        LaunchMap M{};
        for (int poly = 0; poly < 2; poly++)
            for (int i = 0; i < out_rows; i++) {
                const int l = 2 * i + poly;
                const int r = ob + i - wb;  // the output prime's row in ks_q, if the window has it
                M.in_off[l] = poly * out_rows + i;
                M.sub_off[l] = r >= 0 && r < level ? poly * level + r : -1;
                M.out_off[l] = i;
                M.grp[l] = poly;
                M.pid[l] = (ob + i);
                M.cidx[l] = (rr ? c.rr_fin_off[level] + i : rescale ? level * c.n_q + i : wb + i);
            }
        P.dn_rows = add_map(b, M, 2 * out_rows);
    }
}

void build_rs_plan(const Ctx& c, Blob& b, int level, RsPlan& P)
{
    const int lo = level - 1;
    LaunchMap M{};
    for (int poly = 0; poly < 2; poly++) {
        M.in_off[poly] = poly * level + lo;
        M.out_off[poly] = poly;
        M.pid[poly] = lo;
        M.cidx[poly] = lo;
    }
    P.rows = add_map(b, M, 2);
    M.in_off[0] = 0, M.in_off[1] = 1;
    P.cols = add_map(b, M, 2);
    BcBuilder bb{b, RS_TPW, P.bc};
    int32_t mo[MAX_PRIMES], oo[MAX_PRIMES];
    int8_t pd[MAX_PRIMES];
    for (int poly = 0; poly < 2; poly++) {
        for (int i = 0; i < lo; i++) mo[i] = i, oo[i] = poly * lo + i, pd[i] = (int8_t)i;
        bb.add(poly, 1, lo, mo, oo, pd);
    }
    bb.flush();
    LaunchMap R{};  // the two polynomials' limbs of a prime are neighbours, as in ModDown's combine
    for (int poly = 0; poly < 2; poly++)
        for (int i = 0; i < lo; i++) {
            const int l = 2 * i + poly;
            R.in_off[l] = poly * lo + i;
            R.sub_off[l] = poly * level + i;
            R.out_off[l] = i;
            R.grp[l] = poly;
            R.pid[l] = i;
            R.cidx[l] = (level * c.n_q + i);
        }
    P.nrows = add_map(b, R, 2 * lo);
}

// stand-alone rational rescaling from the window at `level` to the window
// below: INTT of the dropped rows (both halves), BConv to the output primes +
// NTT column pass, NTT row pass + combine with the kept input rows
void build_rr_plan(const Ctx& c, Blob& b, int level, RrPlan& P)
{
    const int wb = c.wbase[level], below = c.rr_below[level], ob = c.wbase[below];
    const int nd = c.rr_drop(level);
    int dr[MAX_PRIMES] = {};
    for (int r = 0, k = 0; r < level; r++)
        if (r < c.rr_dlo[level] || r >= c.rr_dhi[level]) dr[k++] = r;
    LaunchMap M{};
    for (int poly = 0; poly < 2; poly++)
        for (int k = 0; k < nd; k++) {
            const int l = poly * nd + k;
            M.in_off[l] = poly * level + dr[k];
            M.out_off[l] = l;
            M.pid[l] = (wb + dr[k]);
            M.cidx[l] = (c.rr2_c_off[level] + k);
        }
    P.rows = add_map(b, M, 2 * nd);
    for (int l = 0; l < 2 * nd; l++) M.in_off[l] = l;
    P.cols = add_map(b, M, 2 * nd);
    BcBuilder bb{b, RS_TPW, P.bc};
    int32_t mo[MAX_PRIMES], oo[MAX_PRIMES];
    int8_t pd[MAX_PRIMES];
    for (int poly = 0; poly < 2; poly++) {
        for (int o = 0; o < below; o++) {
            mo[o] = c.rr2_mat_off[level] + o * nd;
            oo[o] = poly * below + o;
            pd[o] = (int8_t)(ob + o);
        }
        bb.add(poly * nd, nd, below, mo, oo, pd);
    }
    bb.flush();
    LaunchMap R{};
    for (int poly = 0; poly < 2; poly++)
        for (int o = 0; o < below; o++) {
            const int l = 2 * o + poly, r = ob + o - wb;
            R.in_off[l] = poly * below + o;
            R.sub_off[l] = r >= 0 && r < level ? poly * level + r : -1;
            R.out_off[l] = o;
            R.grp[l] = poly;
            R.pid[l] = (ob + o);
            R.cidx[l] = (c.rr2_fin_off[level] + o);
        }
    P.nrows = add_map(b, R, 2 * below);
}

}  // namespace

int launch_rescale_rational_window(const Ctx& c, int level, const uint32_t* ct, uint32_t* out, void* ws,
                                   hipStream_t s)
{
    const RrPlan& P = c.rr_plan[level];
    if (!P.rows.dev) return set_error(-5, "no rational rescaling plan for this level");
    const int log1 = c.log_n - ROW_LOG, nd = c.rr_drop(level), below = c.rr_below[level];
    const size_t n = c.n;
    if (small_ring(c))
        return small_rescale(c, P.rows, P.cols, P.nrows, ct, c.rr2_c, nd, c.rr2_mat + c.rr2_mat_off[level],
                             StCombine{out, out + (size_t)below * n, ct, c.rr2_fin, c.log_n},
                             static_cast<int32_t*>(ws), s);
    uint32_t* w0 = static_cast<uint32_t*>(ws);
    int32_t* w1 = reinterpret_cast<int32_t*>(w0 + 2 * (size_t)nd * n);
    uint32_t* w2 = reinterpret_cast<uint32_t*>(w1 + 2 * (size_t)nd * n);
    {
        LdPlain ld{ct, c.log_n};
        StPlain st{w0, nullptr, c.log_n};
        KTimer t(c, "rr_intt_rows", s);
        CKKS_DISPATCH_LOG1(log1, (inv_rows<L1>(c, MapByPtr{P.rows.dev}, P.rows.n, ld, st, s)));
        if (int e = launched("rational rescale intt rows")) return e;
    }
    if (nd <= RR_FUSE_MAX_IN) {
        KTimer t(c, "rr_cols", s);
        if (int e = launch_inv_bconv_list<false>(c, RS_TPW, P.cols, P.bc, w0, c.rr2_c, c.rr2_mat, w2, BcRescale{}, s))
            return e;
    } else {
        LdPlain ld{w0, c.log_n};
        StLift st{w1, c.rr2_c, c.log_n};
        {
            KTimer t(c, "rr_intt_cols", s);
            CKKS_DISPATCH_LOG1(log1, (inv_cols<L1>(c, MapByPtr{P.cols.dev}, P.cols.n, ld, st, s, 1, true)));
            if (int e = launched("rational rescale intt cols")) return e;
        }
        KTimer t(c, "rr_bconv_ntt_cols", s);
        if (int e = launch_bconv_list<false>(c, RS_TPW, P.bc, w1, c.rr2_mat, w2, BcRescale{}, s, true)) return e;
    }
    {
        LdQuads ld{w2, c.log_n};
        StCombine st{out, out + (size_t)below * n, ct, c.rr2_fin, c.log_n};
        KTimer t(c, "rr_ntt_rows_combine", s);
        CKKS_DISPATCH_LOG1(log1, (fwd_rows<L1>(c, MapByPtr{P.nrows.dev}, P.nrows.n, ld, st, s)));
        if (int e = launched("rational rescale ntt rows")) return e;
    }
    return 0;
}

// Rebuild the launch plans for new tuning knobs (the caller has drained
// every stream that uses the context).
int retune(Ctx& c, int tpw_up, int tpw_dn, int xcd_pair, int rows_ept, int rows_ept1, int col_threads, int km_ept,
           int km_ept1, int col_ept, int col_ept1)
{
    if (c.plan_block) (void)hipFree(c.plan_block);
    if (c.dir_block) (void)hipFree(c.dir_block);
    c.plan_block = c.dir_block = nullptr;
    c.tpw_up = tpw_up, c.tpw_dn = tpw_dn, c.xcd_pair = xcd_pair, c.rows_ept = rows_ept, c.rows_ept1 = rows_ept1,
    c.col_threads = col_threads, c.km_ept = km_ept, c.km_ept1 = km_ept1, c.col_ept = col_ept, c.col_ept1 = col_ept1;
    return build_plans(c);
}

int build_plans(Ctx& c)
{
    if (c.n_q > MAX_LAUNCH_LIMBS / 2 || c.n_q + c.n_p > 127)
        return set_error(-5, "too many primes for the launch maps");
    // a windowed context (levels of the 25-30 system) rescales rationally:
    // its rescaling plans merge ModDown into the rescaling to the window below
    auto planned = [&](int rs, int level) {
        return c.has_level(level) && (rs == 0 || (c.windowed ? c.rr_below[level] > 0 : level >= 2));
    };
    uint64_t q_max = 0;
    for (int i = 0; i < c.n_q; i++) q_max = std::max(q_max, c.mod[i]);
    c.up_nofix = (uint64_t)c.n_p * q_max <= (1ull << 33) ? 1 : 0;
    Blob b;
    for (int rs = 0; rs < 2; rs++) {
        c.ks_plan[rs].assign(c.n_q + 1, KsPlan{});
        for (int level = 1; level <= c.n_q; level++)
            if (planned(rs, level)) build_ks_plan(c, b, level, rs == 1, c.ks_plan[rs][level]);
    }
    c.rs_plan.assign(c.n_q + 1, RsPlan{});
    if (!c.windowed)
        for (int level = 2; level <= c.n_q; level++) build_rs_plan(c, b, level, c.rs_plan[level]);
    c.rr_plan.assign(c.n_q + 1, RrPlan{});
    for (int level = 1; level <= c.n_q && c.windowed; level++)
        if (c.has_level(level) && c.rr_below[level]) build_rr_plan(c, b, level, c.rr_plan[level]);
    if (hipMalloc(&c.plan_block, b.bytes.size()) != hipSuccess) return set_error(-4, "hipMalloc of launch plans failed");
    if (hipMemcpy(c.plan_block, b.bytes.data(), b.bytes.size(), hipMemcpyHostToDevice) != hipSuccess)
        return set_error(-4, "uploading launch plans failed");
    char* base = static_cast<char*>(c.plan_block);
    auto fix = [&](MapRef& m) { if (m.n || m.dev) rebase(m.dev, base); };
    for (int rs = 0; rs < 2; rs++)
        for (int level = 1; level <= c.n_q; level++) {
            if (!planned(rs, level)) continue;
            KsPlan& P = c.ks_plan[rs][level];
            fix(P.up_rows), fix(P.up_cols), fix(P.dn_cols), fix(P.dn_rows), fix(P.up_nrows);
            for (auto& r : P.up_bc) rebase(r.dev, base);
            for (auto& r : P.dn_bc) rebase(r.dev, base);
        }
    for (int level = 2; level <= c.n_q && !c.windowed; level++) {
        RsPlan& P = c.rs_plan[level];
        fix(P.rows), fix(P.cols), fix(P.nrows);
        for (auto& r : P.bc) rebase(r.dev, base);
    }
    for (int level = 1; level <= c.n_q && c.windowed; level++) {
        RrPlan& P = c.rr_plan[level];
        if (!P.rows.n) continue;
        fix(P.rows), fix(P.cols), fix(P.nrows);
        for (auto& r : P.bc) rebase(r.dev, base);
    }
    // per-level directories for batched launches: 6 pointer arrays per rescale flag
    const size_t per = (size_t)c.n_q + 1;
    std::vector<const void*> dir(2 * 6 * per, nullptr);
    for (int rs = 0; rs < 2; rs++)
        for (int level = 1; level <= c.n_q; level++) {
            if (!planned(rs, level)) continue;
            const KsPlan& P = c.ks_plan[rs][level];
            const void** d = dir.data() + (size_t)rs * 6 * per;
            const bool one = P.up_bc.size() == 1 && P.dn_bc.size() == 1;
            d[0 * per + level] = P.up_rows.dev;
            d[1 * per + level] = P.up_cols.dev;
            d[2 * per + level] = one ? (const void*)P.up_bc[0].dev : nullptr;
            d[3 * per + level] = P.dn_cols.dev;
            d[4 * per + level] = one ? (const void*)P.dn_bc[0].dev : nullptr;
            d[5 * per + level] = P.dn_rows.dev;
        }
    if (hipMalloc(&c.dir_block, dir.size() * sizeof(void*)) != hipSuccess)
        return set_error(-4, "hipMalloc of plan directory failed");
    if (hipMemcpy(c.dir_block, dir.data(), dir.size() * sizeof(void*), hipMemcpyHostToDevice) != hipSuccess)
        return set_error(-4, "uploading plan directory failed");
    for (int rs = 0; rs < 2; rs++) {
        const void* const* d = static_cast<const void* const*>(c.dir_block) + (size_t)rs * 6 * per;
        KsDir& D = c.ks_dir[rs];
        D.up_rows = reinterpret_cast<const LaunchMap* const*>(d + 0 * per);
        D.up_cols = reinterpret_cast<const LaunchMap* const*>(d + 1 * per);
        D.up_bc = reinterpret_cast<const BcMap* const*>(d + 2 * per);
        D.dn_cols = reinterpret_cast<const LaunchMap* const*>(d + 3 * per);
        D.dn_bc = reinterpret_cast<const BcMap* const*>(d + 4 * per);
        D.dn_rows = reinterpret_cast<const LaunchMap* const*>(d + 5 * per);
    }
    return 0;
}

}  // namespace ckks
