// The strip sweep: K steps of a strip of the lattice by one wave, the intermediate steps in
// registers.
//
// A wave takes a window of 64 C columns (C adjacent columns per lane) and moves up the rows of its
// strip.  At every row it loads the nine populations of step t once, computes step t of that row,
// step t + 1 of the row below, ... step t + K - 1 of the row K - 1 below, and stores that one.  A
// step's pull needs three rows of the step before: of the rows y - 1 and y only the populations
// that are still to be pulled are kept (three and six, in registers), and the row y + 1 has just
// been computed.  x-shifts between steps are lane shifts (DPP).  So there is no LDS tile, no barrier
// and no index arithmetic per node; what is computed more than once are K - 1 columns on either
// side of the window and K - 1 rows above and below the strip.
//
// Each value kept between steps is rounded as a store to global memory would round it, and the node
// update is node.hpp's, so the populations are bitwise those of K one-step launches.
//
// Edges.  Across a periodic edge a halo column or row is the wrapped one.  A free-slip row beyond the
// lattice is the mirror image of the row inside (its populations 2, 5, 6 are 4, 8, 7 below the first
// row, and the reverse above the last).  At the last column of a lattice with an outlet the pull of
// 3, 6, 7 takes the node's own column.  Everything about rows is uniform over the wave.
//
// Two forms: plain windows (clear of the x edges and of solid nodes), and general ones.
#pragma once

#include <type_traits>

#include "kernels.hpp"
#include "node.hpp"

namespace vplbm {

// ---- C adjacent columns of a population, as a lane holds them ------------------------------------

constexpr int kShr = 0x138, kShl = 0x130;   // DPP: the lane before / after, over the whole wave

template <int CTRL> __device__ __forceinline__ unsigned lane_shift(unsigned v)
{
    return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true);
}
template <int CTRL> __device__ __forceinline__ float lane_shift(float v) { return __uint_as_float(lane_shift<CTRL>(__float_as_uint(v))); }
template <int CTRL> __device__ __forceinline__ double lane_shift(double v)
{
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const unsigned lo = lane_shift<CTRL>((unsigned)b), hi = lane_shift<CTRL>((unsigned)(b >> 32));
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

template <typename E> __device__ __forceinline__ E buffer_elem(__amdgpu_buffer_rsrc_t r, int v, int s);
template <> __device__ __forceinline__ float buffer_elem<float>(__amdgpu_buffer_rsrc_t r, int v, int s)
{
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, v, s, 0));
}
template <> __device__ __forceinline__ double buffer_elem<double>(__amdgpu_buffer_rsrc_t r, int v, int s)
{
    const auto d = __builtin_amdgcn_raw_buffer_load_b64(r, v, s, 0);
    return __longlong_as_double((long long)(((unsigned long long)d[1] << 32) | d[0]));
}

// v is computed here: without this the compiler moves the last sums of a collision to where their
// results are used, a row later, and keeps all that they need in registers until then (binary32, two
// columns, four steps: 176 VGPRs without, 144 with).
__device__ __forceinline__ void settle_value(float &v) { asm volatile("" : "+v"(v)); }
__device__ __forceinline__ void settle_value(double &v) { asm volatile("" : "+v"(v)); }
__device__ __forceinline__ void settle_value(unsigned &v) { asm volatile("" : "+v"(v)); }

// 4- and 8-byte storage: one register (pair) per column.
template <int S, int C> struct Cols {
    using E = typename Codec<S>::elem;
    using T = typename Codec<S>::real;
    static constexpr bool shifted_loads = true;   // a window may start at any element
    E v[C];

    __device__ __forceinline__ static Cols load(__amdgpu_buffer_rsrc_t r, int voff, int soff)
    {
        Cols p;
        if constexpr (C == 2 && sizeof(E) == 4) {
            const auto d = __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0);
            p.v[0] = __uint_as_float(d[0]);
            p.v[1] = __uint_as_float(d[1]);
        } else {
#pragma unroll
            for (int c = 0; c < C; c++) p.v[c] = buffer_elem<E>(r, voff + c * (int)sizeof(E), soff);
        }
        return p;
    }
    // the first column from byte offset v0, the second from v1
    __device__ __forceinline__ static Cols gather(__amdgpu_buffer_rsrc_t r, int v0, int v1, int soff)
    {
        Cols p;
        p.v[0] = buffer_elem<E>(r, v0, soff);
        if constexpr (C == 2) p.v[1] = buffer_elem<E>(r, v1, soff);
        return p;
    }
    // the first column alone
    __device__ __forceinline__ void store1(__amdgpu_buffer_rsrc_t r, int voff, int soff) const
    {
        if constexpr (sizeof(E) == 4) {
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(float(v[0])), r, voff, soff, 0);
        } else {
            const unsigned long long b = (unsigned long long)__double_as_longlong(double(v[0]));
            using V2 = unsigned __attribute__((ext_vector_type(2)));
            __builtin_amdgcn_raw_buffer_store_b64(V2{(unsigned)b, (unsigned)(b >> 32)}, r, voff, soff, 0);
        }
    }
    __device__ __forceinline__ void store(__amdgpu_buffer_rsrc_t r, int voff, int soff) const
    {
        if constexpr (C == 2 && sizeof(E) == 4) {
            using V2 = unsigned __attribute__((ext_vector_type(2)));
            __builtin_amdgcn_raw_buffer_store_b64(V2{__float_as_uint(float(v[0])), __float_as_uint(float(v[1]))}, r, voff, soff, 0);
        } else {
#pragma unroll
            for (int c = 0; c < C; c++) Cols<S, 1>{{v[c]}}.store1(r, voff + c * (int)sizeof(E), soff);
        }
    }
    // the columns one to the left / right of each of these
    __device__ __forceinline__ Cols left() const
    {
        Cols p;
        p.v[0] = lane_shift<kShr>(v[C - 1]);
        if constexpr (C == 2) p.v[1] = v[0];
        return p;
    }
    __device__ __forceinline__ Cols right() const
    {
        Cols p;
        if constexpr (C == 2) p.v[0] = v[1];
        p.v[C - 1] = lane_shift<kShl>(v[0]);
        return p;
    }
    // the first column to element i of a plane
    __device__ __forceinline__ void put(E *plane, unsigned i) const { *at(plane, i) = v[0]; }
    __device__ __forceinline__ T get(int c, T w) const { return Codec<S>::load(&v[c], 0, w); }
    __device__ __forceinline__ void set(int c, T h, T w) { Codec<S>::store(&v[c], 0, h, w); }
    __device__ __forceinline__ void take(int c, const Cols &o) { v[c] = o.v[c]; }
    __device__ __forceinline__ void settle(int c) { settle_value(v[c]); }
};

// 2-byte storage: one column, or a pair, in the low and high halves of one register.
template <int S, int C> struct Cols16 {
    using E = typename Codec<S>::elem;
    using T = float;
    static constexpr bool shifted_loads = C == 1;   // a pair starts at an even element
    unsigned v;

    __device__ __forceinline__ void load_(__amdgpu_buffer_rsrc_t r, int voff, int soff)
    {
        if constexpr (C == 2) v = __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0);
        else v = __builtin_amdgcn_raw_buffer_load_b16(r, voff, soff, 0);
    }
    __device__ __forceinline__ void gather_(__amdgpu_buffer_rsrc_t r, int v0, int v1, int soff)
    {
        const unsigned lo = __builtin_amdgcn_raw_buffer_load_b16(r, v0, soff, 0);
        const unsigned hi = C == 2 ? __builtin_amdgcn_raw_buffer_load_b16(r, v1, soff, 0) : 0u;
        v = (lo & 0xFFFFu) | (hi << 16);
    }
    __device__ __forceinline__ void store1(__amdgpu_buffer_rsrc_t r, int voff, int soff) const
    {
        __builtin_amdgcn_raw_buffer_store_b16((unsigned short)v, r, voff, soff, 0);
    }
    __device__ __forceinline__ void store(__amdgpu_buffer_rsrc_t r, int voff, int soff) const
    {
        if constexpr (C == 2) __builtin_amdgcn_raw_buffer_store_b32(v, r, voff, soff, 0);
        else store1(r, voff, soff);
    }
    // the first column to element i of a plane
    __device__ __forceinline__ void put(E *plane, unsigned i) const { *at(plane, i) = __builtin_bit_cast(E, (unsigned short)v); }
    __device__ __forceinline__ unsigned left_() const
    {
        const unsigned n = lane_shift<kShr>(v);
        return C == 2 ? __builtin_amdgcn_alignbit(v, n, 16) : n;
    }
    __device__ __forceinline__ unsigned right_() const
    {
        const unsigned n = lane_shift<kShl>(v);
        return C == 2 ? __builtin_amdgcn_alignbit(n, v, 16) : n;
    }
    __device__ __forceinline__ float get(int c, float) const
    {
        const E e = __builtin_bit_cast(E, (unsigned short)(c ? v >> 16 : v));
        return (float)e;
    }
    // Column 0 first, then column 1 of a pair: the first is held in binary32 until both can be packed.
    __device__ __forceinline__ void set(int c, float h, float)
    {
        using F2 = float __attribute__((ext_vector_type(2)));
        using E2 = E __attribute__((ext_vector_type(2)));
        settle_value(h);   // round to binary32 first: no mixed-precision multiply-add into the conversion
        if constexpr (C == 1) {
            v = __builtin_bit_cast(unsigned short, (E)h);
        } else {
            if (c == 0) v = __float_as_uint(h);
            else v = __builtin_bit_cast(unsigned, __builtin_convertvector(F2{__uint_as_float(v), h}, E2));
        }
    }
    // The same for a binary32 value whose lower bits are to be dropped.
    __device__ __forceinline__ void set_truncated(int c, unsigned bits)
    {
        if constexpr (C == 2) {
            if (c == 0) {
                v = bits;
                return;
            }
        }
        const unsigned first = C == 2 ? v : bits;
        if constexpr (S == kBF16SR) v = C == 1 ? bits >> 16 : __builtin_amdgcn_perm(bits, first, 0x07060302u);
        else v = __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_pkrtz(__uint_as_float(first), C == 1 ? 0.0f : __uint_as_float(bits)));
    }
    __device__ __forceinline__ void take_(int c, unsigned o)
    {
        v = c ? (v & 0xFFFFu) | (o & 0xFFFF0000u) : (v & 0xFFFF0000u) | (o & 0xFFFFu);
    }
    __device__ __forceinline__ void settle(int) { settle_value(v); }
};
#define VPLBM_COLS16(S, C)                                                                                            \
    template <> struct Cols<S, C> : Cols16<S, C> {                                                                    \
        __device__ __forceinline__ static Cols of(unsigned v) { Cols p; p.v = v; return p; }                          \
        __device__ __forceinline__ static Cols load(__amdgpu_buffer_rsrc_t r, int voff, int soff) { Cols p; p.load_(r, voff, soff); return p; } \
        __device__ __forceinline__ static Cols gather(__amdgpu_buffer_rsrc_t r, int v0, int v1, int soff) { Cols p; p.gather_(r, v0, v1, soff); return p; } \
        __device__ __forceinline__ Cols left() const { return of(this->left_()); }                                     \
        __device__ __forceinline__ Cols right() const { return of(this->right_()); }                                   \
        __device__ __forceinline__ void take(int c, const Cols &o) { this->take_(c, o.v); }                            \
    }
VPLBM_COLS16(kF16S, 1);
VPLBM_COLS16(kF16S, 2);
VPLBM_COLS16(kBF16S, 1);
VPLBM_COLS16(kBF16S, 2);
VPLBM_COLS16(kF16SR, 1);
VPLBM_COLS16(kF16SR, 2);
VPLBM_COLS16(kBF16SR, 1);
VPLBM_COLS16(kBF16SR, 2);
#undef VPLBM_COLS16

// Round the updated populations of column c (0, then 1) into g as store_node would: node is the node's
// lattice index (row * pitch + column), hash the step's part of the random bits, lanes those whose
// results matter.
template <int S, int C>
__device__ __forceinline__ void round_cols(Cols<S, C> g[9], int c, const typename Codec<S>::real h[9], unsigned node,
                                           unsigned hash, unsigned long long lanes)
{
    using T = typename Codec<S>::real;
    if constexpr (!Codec<S>::stochastic) {
#pragma unroll
        for (int k = 0; k < 9; k++) g[k].set(c, h[k], weight<T>(k));
    } else {
        unsigned up[9];              // the value with random bits added under the kept mantissa
        unsigned r = mix32(node ^ hash);
        const unsigned r0 = r;
        float least = __builtin_inff(), most = 0.0f;
#pragma unroll
        for (int k = 0; k < 9; k++) {
            if (k % 2 == 0 && k > 0) r = xorshift32(r);
            const unsigned bits = (k % 2) ? (r >> 16) : r;
            up[k] = __float_as_uint(h[k]) + (bits & (S == kF16SR ? 0x1FFFu : 0xFFFFu));
            if constexpr (S == kF16SR) {
                least = __builtin_fminf(least, __builtin_fabsf(h[k]));
                most = __builtin_fmaxf(most, __builtin_fabsf(h[k]));
            }
        }
        if constexpr (S == kF16SR) {
            // Values below 2^-14 round on another quantum, and those near 2^16 to infinity.  In a wake every
            // other wave holds one, where a population changes sign: each is looked at by itself.
            if (__ballot(least < 6.103515625e-05f || most >= 65472.0f) & lanes) {
                r = r0;
#pragma unroll
                for (int k = 0; k < 9; k++) {
                    if (k % 2 == 0 && k > 0) r = xorshift32(r);
                    const float a = __builtin_fabsf(h[k]);
                    if (__any(a < 6.103515625e-05f || a >= 65472.0f))
                        up[k] = __float_as_uint((float)f16_stochastic(h[k], (k % 2) ? (r >> 16) : r));
                }
            }
        }
#pragma unroll
        for (int k = 0; k < 9; k++) g[k].set_truncated(c, up[k]);
    }
}

// ---- the sweep -----------------------------------------------------------------------------------

// Columns computed beyond the window's own on either side: K - 1 steps' worth, one more for pairs,
// whose first step may shift lanes too, rounded up to whole lanes.
template <int S, int C, int K> constexpr int strip_halo() { return C == 1 ? K - 1 : (K + 1) / 2 * 2; }
template <int S, int C, int K> constexpr int strip_width() { return 64 * C - 2 * strip_halo<S, C, K>(); }

// What a strip needs to know, uniform over the wave.
struct StripJob {
    const void *src;
    void *dst;
    const uint8_t *mask;         // the first step's; a later step's mask_step bytes further (0 unless
    size_t mask_step;            //   bodies move), its body states state_step entries further
    const BodyState *bodies;
    int state_step;
    Geom g;
    NodeParams p;
    const void *out_prev;        // convective outlet records (compute type), or null
    void *out_next;
    double out_u;
    int x0, y0, y1;              // own columns x0 .. x0 + width - 1 and rows y0 .. y1 - 1
    bool reduce;
    unsigned step;               // the first step (random bits)
};

// The populations of one step that later rows still pull: of row y - 1 those moving up, of row y
// those moving up and those moving along the row.  Already shifted to the column that pulls them
// where no row beyond the lattice needs the unshifted one.
template <typename P> struct StripRows {
    P up2, up5, up6;             // row y - 1, as pulled
    P m0, m1, m3;                // row y, as pulled
    P m2, m5, m6;                // row y, unshifted
};

// LDS of a strip: sums; per step each body's centre, velocity and angular velocity, and the outlet records
// of the last two rows, by row parity.
//
// With the sums of every step, mass and the force on every body: a lane adds to slot lane % kForceSlots, so
// that at most four lanes of a wave meet at one address; in which order they are added is the hardware's
// choice, so the last bits of a force are not fixed.
constexpr int kForceSlots = 16;
template <typename T, int K> struct StripShared {
    static constexpr bool kEveryStep = true;
    double part[K][kForceSlots][kRingWidth];
    T body[K][kMaxBodies][5];
    T record[K][2][3];
    __device__ __forceinline__ double *slot(int k, int lane) { return part[k][lane % kForceSlots]; }
};
// With the last step's alone: a slot per lane, each added to by its own lane only, row by row.
template <typename T, int K> struct StripLastShared {
    static constexpr bool kEveryStep = false;
    double part[64][kRingWidth];
    T body[K][kMaxBodies][5];
    T record[K][2][3];
    __device__ __forceinline__ double *slot(int, int lane) { return part[lane]; }
};

// K steps of one strip of windows laid out for KW.  mass: per step, this lane's sum of drho over the
// strip's own nodes.  Returns (job.reduce) whether an own node of this lane had a non-finite or
// non-positive density.  SUMS: the forces are added into shared's slots (job.reduce).
template <int S, int C, int K, bool GENERAL, int KW = K, bool SUMS = true, typename Shared>
__device__ __forceinline__ bool strip_sweep(const StripJob &job, double (&mass)[K], Shared &shared)
{
    using P = Cols<S, C>;
    using E = typename Codec<S>::elem;
    using T = typename Codec<S>::real;
    constexpr int HX = strip_halo<S, C, KW>(), ES = (int)sizeof(E);
    constexpr int mirror_y[9] = {0, 1, 4, 3, 2, 8, 7, 6, 5};
    constexpr int cx[9] = {0, 1, 0, -1, 0, 1, -1, -1, 1};
    constexpr int cy[9] = {0, 0, 1, 0, -1, 1, 1, -1, -1};
    // the first step pulls by loads from the neighbouring columns, or by lane shifts as the others do
    constexpr bool PULL = C == 1 || (!GENERAL && P::shifted_loads);
    const Geom &g = job.g;
    const Rates<T> rates(job.p);
    const T out_u = GENERAL ? uniform(T(job.out_u)) : T(0);
    const int lane = threadIdx.x & 63;
    const unsigned bytes = 9u * unsigned(g.plane) * unsigned(ES);
    const __amdgpu_buffer_rsrc_t rsrc = buffer_over(const_cast<void *>(job.src), bytes);
    const __amdgpu_buffer_rsrc_t rdst = buffer_over(job.dst, bytes);

    // Columns.  ux: the lane's first, unwrapped.  x0, x1: lattice columns of its first and last.  A lane
    // beyond a non-periodic edge takes the nearest columns inside, and nothing uses its results.
    const int ux = job.x0 - HX + C * lane;
    const bool split = GENERAL && C == 2 && g.xper && (g.nx & 1);   // a pair may straddle the wrap
    int x0 = ux, x1 = ux + C - 1;
    int off[3];                          // byte offsets of the columns before, at and after the first
    bool own0 = C * lane >= HX && C * lane < 64 * C - HX, own1 = own0;
    bool at_in = false, at_out0 = false, at_out1 = false;   // (an inlet column is a lane's first: x = 0)
    if constexpr (GENERAL) {
        auto wrapped = [&](int x) __attribute__((always_inline)) { x %= g.nx; return x < 0 ? x + g.nx : x; };
        x0 = strip_column(ux, C, g.nx, g.xper);
        if (g.xper) x1 = C == 2 ? (x0 + 1 == g.nx ? 0 : x0 + 1) : x0;
        else x1 = x0 + C - 1;
        own1 = own0 && ux + C - 1 < g.nx;
        own0 = own0 && ux < g.nx;
        at_in = g.inlet && ux == 0;
        at_out0 = !g.xper && ux == g.nx - 1;
        at_out1 = C == 2 && !g.xper && ux + 1 == g.nx - 1;
        if constexpr (PULL) {
            off[0] = (g.xper ? wrapped(ux - 1) : (x0 > 0 ? x0 - 1 : 0)) * ES;
            off[2] = (g.xper ? wrapped(ux + 1) : (x0 < g.nx - 1 ? x0 + 1 : g.nx - 1)) * ES;
        } else {
            off[0] = off[2] = 0;
        }
        off[1] = x0 * ES;
    } else {
#pragma unroll
        for (int d = 0; d < 3; d++) off[d] = (ux + d - 1) * ES;
    }
    // uniform: whether the window reaches the inlet's / the outlet's column
    const bool has_in = GENERAL && __any(at_in), has_out = GENERAL && __any(at_out0 || at_out1);

    // the populations of row y (0 <= y < ny) that step 1 pulls or, without PULL, the row's own ones of
    // the pulled rows
    auto load_row = [&](int y, P f[9], auto full) __attribute__((always_inline)) {
        constexpr bool FULL = decltype(full)::value;
        int rows[3] = {y - 1, y, y + 1};
        const bool low = !FULL && y == 0, high = !FULL && y == g.ny - 1;
        if (low) rows[0] = g.yper ? g.ny - 1 : 0;
        if (high) rows[2] = g.yper ? 0 : g.ny - 1;
#pragma unroll
        for (int a = 0; a < 9; a++) {
            const bool ghost = !g.yper && (cy[a] > 0 ? low : (cy[a] < 0 ? high : false));
            const unsigned e = unsigned(ghost ? mirror_y[a] : a) * unsigned(g.plane) + unsigned(rows[1 - cy[a]]) * unsigned(g.pitch);
            const int soff = __builtin_amdgcn_readfirstlane(int(e * unsigned(ES)));
            if (split) f[a] = P::gather(rsrc, off[1], x1 * ES, soff);
            else f[a] = P::load(rsrc, off[PULL ? 1 - cx[a] : 1], soff);
        }
    };
    auto wrap_row = [&](int y) __attribute__((always_inline)) -> int { return y < 0 ? y + g.ny : (y >= g.ny ? y - g.ny : y); };
    // ids of the lane's columns in row y of a step's mask, a byte each
    auto load_ids = [&](int k, int y) __attribute__((always_inline)) -> unsigned {
        const uint8_t *m = job.mask + k * job.mask_step + (size_t)y * g.pitch;
        if (C == 1) return m[unsigned(x0)];
        if (split) return unsigned(m[unsigned(x0)]) | unsigned(m[unsigned(x1)]) << 8;
        return *reinterpret_cast<const unsigned short *>(m + unsigned(x0));
    };
    // p seen from the left neighbour's column; the last column before an outlet sees its own
    auto from_right = [&](const P &p) __attribute__((always_inline)) -> P {
        P q = p.right();
        if (GENERAL && has_out) {
            if (at_out0) q.take(0, p);
            if (C == 2 && at_out1) q.take(1, p);
        }
        return q;
    };

    if constexpr (GENERAL) {
        for (int i = lane; i < K * kMaxBodies; i += 64) {
            const int k = i / kMaxBodies, b = i % kMaxBodies;
            const BodyState &s = job.bodies[k * job.state_step + b];
            T *o = shared.body[k][b];
            o[0] = T(s.cx);
            o[1] = T(s.cy);
            o[2] = T(s.vx);
            o[3] = T(s.vy);
            o[4] = T(s.omega);
        }
    }

    bool bad = false;
    // Step 1 + k of one row: the pulled f in, the rounded results out.
    auto relax_row = [&](int i, int k, const P f[9], int y, unsigned ids, P out[9]) __attribute__((always_inline)) {
        const bool row_own = y >= job.y0 && y < job.y1;
        const int yw = g.yper ? wrap_row(y) : y;
        T h[C][9];
#pragma unroll
        for (int c = 0; c < C; c++)
#pragma unroll
            for (int a = 0; a < 9; a++) h[c][a] = f[a].get(c, weight<T>(a));
        if (GENERAL && has_out && job.out_prev) {
            // the rule needs the values the step before recorded in this row: from global memory for
            // step 1, from the row that step did last otherwise
            constexpr int odirs[3] = {3, 6, 7};
            const bool last = k == K - 1;
            T *next = static_cast<T *>(job.out_next);
#pragma unroll
            for (int c = 0; c < C; c++) {
                if (c ? at_out1 : at_out0) {
#pragma unroll
                    for (int q = 0; q < 3; q++) {
                        const T prev = k == 0 ? static_cast<const T *>(job.out_prev)[q * g.ny + yw] : shared.record[k - 1][(i + 1) & 1][q];
                        h[c][odirs[q]] = outlet_value(prev, h[c][odirs[q]], out_u);
                        if (!last) shared.record[k][i & 1][q] = h[c][odirs[q]];
                        else if (row_own && (c ? own1 : own0)) next[q * g.ny + yw] = h[c][odirs[q]];
                    }
                }
            }
        }
        if (GENERAL && has_in) {
            if (at_in) inlet_west(h[0], rates.uin_x, rates.uin_y);
        }
        const unsigned hash = Codec<S>::stochastic ? mix32((job.step + unsigned(k)) * 0x9e3779b9u + 0x7f4a7c15u) : 0u;
        auto keep = [&](int c, const T hc[9]) __attribute__((always_inline)) {
            // lanes whose columns still count after k + 1 shifts
            const unsigned long long lanes = (~0ull << ((k + !PULL) / C)) & (~0ull >> ((k + !PULL) / C));
            round_cols<S, C>(out, c, hc, Codec<S>::stochastic ? unsigned(yw) * unsigned(g.pitch) + unsigned(c ? x1 : x0) : 0u, hash, lanes);
#pragma unroll
            for (int a = 0; a < 9; a++) out[a].settle(c);
        };
        T drho[C];
        if (GENERAL && __any(ids != 0)) {
            // every lane takes the penalized form; at a fluid node its factors make it the fluid one
#pragma unroll
            for (int c = 0; c < C; c++) {
                const int id = strip_id(ids, c, x1, g.nx);
                T usx = T(0), usy = T(0), fx, fy;
                if (id) body_velocity(shared.body[k][id - 1], c ? x1 : x0, yw, usx, usy);
                drho[c] = relax_solid(h[c], id != 0, usx, usy, rates, fx, fy);
                keep(c, h[c]);
                if (SUMS && (Shared::kEveryStep || k == K - 1) && job.reduce && row_own && id && (c ? own1 : own0)) {
                    double *slot = shared.slot(k, lane) + 2 * id;
                    unsafeAtomicAdd(slot - 1, -double(fx));   // LDS adds that nothing waits for
                    unsafeAtomicAdd(slot, -double(fy));
                }
            }
        } else {
#pragma unroll
            for (int c = 0; c < C; c++) {
                drho[c] = relax_fluid(h[c], rates);
                keep(c, h[c]);
            }
        }
        if (job.reduce && row_own) {
            bool odd = false;
#pragma unroll
            for (int c = 0; c < C; c++) {
                const T d = GENERAL ? ((c ? own1 : own0) ? drho[c] : T(0)) : drho[c];
                mass[k] += double(d);
                odd |= !(__builtin_fabs(d) < T(1));      // one compare: the exact test only where it may fail
            }
            if (__any(odd & own0)) {
#pragma unroll
                for (int c = 0; c < C; c++) {
                    const double rho = 1.0 + double(drho[c]);
                    bad |= (c ? own1 : own0) && !(rho > 0.0 && rho < 1e30);
                }
            }
        }
    };

    StripRows<P> win[K > 1 ? K - 1 : 1];
    const int yb = job.y0 - (K - 1);  // row of step 1 in iteration 0
    const int n = job.y1 - job.y0 + 2 * (K - 1);
    auto row_of = [&](int i, int k) __attribute__((always_inline)) -> int { return yb + i - k; };   // row of step 1 + k
    auto inside = [&](int y) __attribute__((always_inline)) -> bool { return g.yper || (y >= 0 && y < g.ny); };

    P next[9];
    unsigned next_ids[K];
    // full (an integral constant): every step works, on rows clear of the lattice's first and last
    auto prefetch = [&](int i, auto full) __attribute__((always_inline)) {
        constexpr bool FULL = decltype(full)::value;
        load_row(FULL ? row_of(i, 0) : strip_row(row_of(i, 0), g.ny, g.yper), next, full);
        if constexpr (GENERAL) {
#pragma unroll
            for (int k = 0; k < K; k++) {
                // A step that has not begun has no use for ids.  One column: a load of row 0 is better than a
                // branch (pool, f64, 4.9 million nodes: 45.5 against 46.2-47.4 us per step); two columns: the
                // branch (6048 x 2016: 55.5 against 56.3; 8192 x 2048: 60.7 against 60.0).
                const bool begun = FULL || strip_begun(i, k);
                if (C == 1) next_ids[k] = load_ids(k, FULL ? row_of(i, k) : begun ? strip_row(row_of(i, k), g.ny, g.yper) : 0);
                else next_ids[k] = begun ? load_ids(k, FULL ? row_of(i, k) : strip_row(row_of(i, k), g.ny, g.yper)) : 0u;
            }
        }
    };
    auto sweep_row = [&](int i, auto full) __attribute__((always_inline)) {
        constexpr bool FULL = decltype(full)::value;
        P f[9], out[9];
        unsigned ids[K];
#pragma unroll
        for (int a = 0; a < 9; a++) f[a] = next[a];
#pragma unroll
        for (int k = 0; k < K; k++) ids[k] = GENERAL ? next_ids[k] : 0u;
        if (FULL || i + 1 < n) prefetch(i + 1, full);
        if constexpr (!PULL) {
#pragma unroll
            for (int a = 0; a < 9; a++) {
                if (cx[a] > 0) f[a] = f[a].left();
                if (cx[a] < 0) f[a] = from_right(f[a]);
            }
        }
#pragma unroll
        for (int a = 0; a < 9; a++) out[a] = f[a];
#pragma unroll
        for (int k = 0; k < K; k++) {
            const int y = row_of(i, k);
            if (k > 0) {
                StripRows<P> &w = win[k - 1];
                if (!FULL && !g.yper && y + 1 == g.ny) {   // the row above is beyond the lattice
                    out[4] = w.m2;
                    out[7] = w.m6;
                    out[8] = w.m5;
                }
                f[0] = w.m0;
                f[1] = w.m1;
                f[2] = w.up2;
                f[3] = w.m3;
                f[4] = out[4];
                f[5] = w.up5;
                f[6] = w.up6;
                f[7] = from_right(out[7]);
                f[8] = out[8].left();
                w.up2 = w.m2;
                w.up5 = w.m5.left();
                w.up6 = from_right(w.m6);
                if (!FULL && !g.yper && y + 1 == 0) {      // the next row up is the lattice's first
                    w.up2 = out[4];
                    w.up5 = f[8];
                    w.up6 = f[7];
                }
                w.m0 = out[0];
                w.m1 = out[1].left();
                w.m3 = from_right(out[3]);
                w.m2 = out[2];
                w.m5 = out[5];
                w.m6 = out[6];
            }
            if (FULL || (i >= 2 * k && inside(y))) relax_row(i, k, f, y, ids[k], out);
        }
        const int y = row_of(i, K - 1);
        if (FULL || i >= 2 * (K - 1)) {              // a row of the strip: y0 <= y < y1
#pragma unroll
            for (int a = 0; a < 9; a++) {
                const unsigned e = unsigned(a) * unsigned(g.plane) + unsigned(y) * unsigned(g.pitch);
                const int soff = __builtin_amdgcn_readfirstlane(int(e * unsigned(ES)));
                if (own1) out[a].store(rdst, off[1], soff);
                else if (GENERAL && C == 2 && own0) out[a].store1(rdst, off[1], soff);
            }
        }
    };
    // Iterations full0 .. full1 - 1 are full ones: all K steps have begun, and the rows they work on,
    // the one loaded ahead and its neighbours lie inside the lattice.
    constexpr std::false_type any{};
    const int full0 = 2 * (K - 1) > 1 - yb + (K - 1) ? 2 * (K - 1) : 1 - yb + (K - 1);
    const int full1 = g.ny - 3 - yb < n - 1 ? g.ny - 3 - yb : n - 1;
    prefetch(0, any);
    int i = 0;
    for (; i < n && i < full0; i++) sweep_row(i, any);
    for (; i + 1 < full1; i += 2) {   // two rows per turn: the rows kept change places without moves
        sweep_row(i, std::true_type{});
        sweep_row(i + 1, std::true_type{});
    }
    for (; i < n; i++) sweep_row(i, any);
#pragma unroll
    for (int k = 0; k < K; k++)
        if (!own0) mass[k] = 0.0;
    return bad;
}

}  // namespace vplbm
