// HIP kernels of libhough.so (gfx950 / CDNA4, wave64).
//
// Layout shared by every kernel that votes: a theta tile of TW = 64*G columns lives in LDS
// rho-major, one row of the tile per rho bin, two 16-bit counters per dword (see Lane below).
// A wave maps 64 hits at a time, one per lane, and forms their bins in 32 columns at a time on
// the matrix cores (vote_mfma): each half of the wave then votes one hit in 32 consecutive
// columns per ds_add_u32, 32 different banks.  Elsewhere lane l owns column c = 64*q + l of group
// q, hits are wave-uniform, and the two lanes of a dword lie in different halves of the wave: no
// bank conflict, never the same address (the theta sweep of Sec. III: one column = one parallel
// task, hits streamed through it).
//
// Row n_rho of the tile is a dummy row for votes outside the grid's rows (lanes whose column
// lies outside [0, n_theta) carry C = S = 0 and B = n_rho, so their lookups land there).
//
// Floating point: the bin of a hit in a column is t = fma(u, C_j, fma(v, S_j, B)) with
// k = (int)t, exactly as the C-ABI header states.  Hits whose votes are provably all in range
// (|rho| bounded by sqrt(u^2+v^2) with slack for rounding) skip the range test; the others take
// the literal test 0 <= t < n_rho.
#include <float.h>

#include <algorithm>
#include <type_traits>

#include "hough_internal.h"

namespace hough {
namespace {

constexpr int kStageBytes = kWave * (int)sizeof(float2);
// Words of the space the waves' stages and a tile's peak words share.
template <int NW>
__host__ __device__ constexpr int stage_words(int peak_words) {
    return NW * (kStageBytes / 4) > peak_words ? NW * (kStageBytes / 4) : peak_words;
}

// ------------------------------------------------------------------ per-hit arithmetic
// Eq. (1).  Returns false for a hit whose r2 is zero, non-finite or overflowed.
__device__ __forceinline__ bool conformal(float x, float y, float &u, float &v) {
    const float y2 = y * y;
    const float r2 = __builtin_fmaf(x, x, y2);
    const bool ok = (r2 > 0.0f) && (r2 <= FLT_MAX);
    const float d = ok ? r2 : 1.0f;
    u = x / d;
    v = y / d;
    return ok;
}

// The validity part of the map alone (no division).
__device__ __forceinline__ bool valid_hit(float x, float y) {
    const float r2 = __builtin_fmaf(x, x, y * y);
    return (r2 > 0.0f) && (r2 <= FLT_MAX);
}

// True when every column's t lies strictly inside (0, n_rho).  |rho| <= sqrt(u^2 + v^2) for
// every theta, so u^2 + v^2 below safe_r2 (set on the host with slack for the rounding of this
// sum and of t) keeps every vote of the hit in range.
__device__ __forceinline__ bool all_in_range(float u, float v, const GridArgs &g) {
    return __builtin_fmaf(u, u, v * v) < g.safe_r2;
}

__device__ __forceinline__ uint32_t mbcnt(uint64_t m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// The wave's number in its workgroup, as a scalar (loops over waves' shares stay scalar).
__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)); }

// A copy of v the compiler takes for a new value: what a phase of a long kernel derives from its
// lane number is then computed in that phase, not held in registers through all the others.
__device__ __forceinline__ int opaque(int v) {
    asm volatile("" : "+v"(v));
    return v;
}

// Zero the n 16-byte words at p, NT threads together (addresses and zeros are made here: see opaque).
template <int NT>
__device__ __forceinline__ void clear_quads(uint32_t *p, int n) {
    const uint32_t z = (uint32_t)opaque(0);
#pragma unroll 1
    for (int i = opaque((int)threadIdx.x); i < n; i += NT) reinterpret_cast<uint4 *>(p)[i] = make_uint4(z, z, z, z);
}

// Element i of a wave-uniform array through a 32-bit byte offset (i below 2^30: events of at most
// kMaxBatchHits hits), which the load takes as it is: no 64-bit address per lane.
__device__ __forceinline__ float at(const float *p, uint32_t i) {
    return *reinterpret_cast<const float *>(reinterpret_cast<const char *>(p) + (i << 2));
}
__device__ __forceinline__ void put(float *p, uint32_t i, float v) {
    *reinterpret_cast<float *>(reinterpret_cast<char *>(p) + (i << 2)) = v;
}

__device__ __forceinline__ void lds_add(uint32_t *p, uint32_t v) {
    __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Per-lane constants of the columns a lane owns in the current tile.  On a theta-periodic grid
// the halo column left of column 0 is column n_theta - 1 and the one right of column
// n_theta - 1 is column 0, both with rho reversed: such a lane votes with that column's own
// constants into row n_rho - 1 - k, i.e. with a negative row stride from the top row (rs, rb:
// row stride and base in bytes, used only by the periodic kernels).
template <int G>
struct Cols {
    float C[G], S[G], B[G];
    int rs[G], rb[G];
};

template <int G, bool PER = false>
__device__ __forceinline__ Cols<G> load_cols(const GridArgs &g, int first_col, int lane, int stride,
                                             const uint32_t *col, float dummy_row = -1.0f) {
    Cols<G> cl;
#pragma unroll
    for (int q = 0; q < G; ++q) {
        const int j = first_col + 64 * q + lane;
        const bool in = (j >= 0) && (j < g.n_theta);
        const bool wrap = PER && (j == -1 || j == g.n_theta);
        const int jw = j < 0 ? g.n_theta - 1 : 0;
        cl.C[q] = in ? g.C[j] : (wrap ? g.C[jw] : 0.0f);
        cl.S[q] = in ? g.S[j] : (wrap ? g.S[jw] : 0.0f);
        // out-of-grid lanes land in the dummy row (row n_rho, or the row a windowed tile gives it)
        cl.B[q] = (in || wrap) ? g.Bf : (dummy_row >= 0.0f ? dummy_row : g.nrho_f);
        cl.rs[q] = 4 * (wrap ? -stride : stride);                                    // bytes
        cl.rb[q] = 4 * (wrap ? (g.n_rho - 1) * stride + (int)col[q] : (int)col[q]);
    }
    return cl;
}

// Where a lane's cells live in a tile row.  Unpacked: one 32-bit counter per cell, column
// 64q + l at dword 64q + l.  Packed: two 16-bit counters per dword, columns 64q + l and
// 64q + l + 32 (l < 32) share dword 32q + l; the two lanes sharing a dword sit in different
// halves of the wave, which the LDS serves in separate passes, so they never conflict.
template <int G, bool PACKED>
struct Lane {
    static constexpr int TW = 64 * G;
    static constexpr int STRIDE = PACKED ? TW / 2 : TW;    // dwords per tile row
    uint32_t col[G];
    uint32_t shift, inc, cmask;
    __device__ __forceinline__ explicit Lane(int lane) {
#pragma unroll
        for (int q = 0; q < G; ++q) col[q] = PACKED ? 32 * q + (lane & 31) : 64 * q + lane;
        shift = PACKED ? 16u * (uint32_t)(lane >> 5) : 0u;
        inc = 1u << shift;
        cmask = PACKED ? 0xffffu : ~0u;
    }
    __device__ __forceinline__ uint32_t count(uint32_t dword) const { return (dword >> shift) & cmask; }
};

// Map up to 64 hits [base, end) (one per lane) and compact the valid ones into the wave's
// stage: all-in-range hits first, then the others.  Returns (n_safe, n_total) and, through
// `bad`, whether this lane met an invalid hit, through `slot` the stage slot of the lane's hit
// (-1 if none).  `skip` hides hits the caller is done with.
struct StageCount { uint32_t safe, total; };

// Stage the lane's hit (xi, yi) when `in`.
__device__ __forceinline__ StageCount stage_values(float2 *st, float xi, float yi,
                                                   bool in, const GridArgs &g,
                                                   uint32_t &bad, int &slot) {
    float u, v;
    const bool ok = conformal(in ? xi : 0.0f, in ? yi : 0.0f, u, v);
    const bool valid = in && ok;
    if (in && !ok) bad = 1u;
    const bool safe = valid && all_in_range(u, v, g);
    const uint64_t bs = __ballot(safe);
    const uint64_t bu = __ballot(valid && !safe);
    const uint32_t ns = (uint32_t)__popcll(bs);
    const uint32_t pos = safe ? mbcnt(bs) : ns + mbcnt(bu);
    if (valid) st[pos] = make_float2(u, v);
    slot = valid ? (int)pos : -1;
    wave_sync();
    return StageCount{ns, ns + (uint32_t)__popcll(bu)};
}

__device__ __forceinline__ StageCount stage_hits(float2 *st, const float *x,
                                                 const float *y, uint32_t base, uint32_t end,
                                                 bool skip, const GridArgs &g, int lane,
                                                 uint32_t &bad, int &slot) {
    const uint32_t i = base + lane;
    const bool in = (i < end) && !skip;
    float xi = 0.0f, yi = 0.0f;
    if (in) { xi = x[i]; yi = y[i]; }
    return stage_values(st, xi, yi, in, g, bad, slot);
}

// The lane's cell of row k in group q.  Periodic kernels use the per-lane row stride (a 24-bit
// multiply-add, full rate) so that the reversed halo lanes need no other instruction.
template <int G, bool P, bool PER = false>
__device__ __forceinline__ uint32_t *cell_of(uint32_t *tile, int k, const Cols<G> &cl, const Lane<G, P> &ln,
                                             int q) {
    if (PER)
        return reinterpret_cast<uint32_t *>(reinterpret_cast<char *>(tile) + (__mul24(k, cl.rs[q]) + cl.rb[q]));
    return &tile[k * Lane<G, P>::STRIDE + (int)ln.col[q]];
}

// Steps 2-3 on the matrix cores.  The sweep of 32 hits over 32 columns is the rank-2 product
// t = [v u] [S; C] + B, and v_mfma_f32_32x32x2_f32 forms it as the chain of fused multiply-adds
// fma(u, C, fma(v, S, B)) in that order, each rounded once: bit for bit the vote's arithmetic
// (checked against fmaf on random and on denormal operands, and by every parity test).  One
// instruction replaces two FMAs per vote, which leaves a vote one conversion, one shift-add and
// its LDS atomic: the vote is then bound by the LDS atomics (14.6 lanes per clock and CU, 4.4
// clocks per 64 votes, against 2 clocks of VALU), where the VALU form bound it on issue.  Measured
// (10,000 events, 360 x 256, whole kernel): 1,075 -> 839 M VALU instructions, 11.1 -> 12.6 vote
// lanes per clock and CU during the vote phases.
//
// Operands: hits in A (lane l < 32 holds v of hit l, lane l + 32 its u), columns in B (S below
// C); both are one v_permlane32_swap away from the lane = hit and lane = column layouts.  Lane l
// of the result holds column l mod 32 for hits 8b + 4 (l / 32) + i (b, i = 0 .. 3): a vote
// instruction puts 32 different columns of a tile row range into each half of the wave, so
// the packed dwords never conflict within a half, exactly as with lane = column.
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// B in all sixteen accumulator registers, in vector registers from here to the last use (the first
// asm keeps the compiler from hoisting the copies out of a kernel's event loop and spilling them,
// the second from rebuilding them before every instruction).
__device__ __forceinline__ f32x16 bias16(float b) {
    asm volatile("" : "+v"(b));
    f32x16 r;
#pragma unroll
    for (int i = 0; i < 16; ++i) r[i] = b;
    asm volatile("" : "+v"(r));
    return r;
}

// (lo, hi) := ({x lanes 0-31, y lanes 0-31}, {x lanes 32-63, y lanes 32-63}).
__device__ __forceinline__ void swap_halves(float x, float y, float &lo, float &hi) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    lo = __uint_as_float(r[0]);
    hi = __uint_as_float(r[1]);
}

// A tile's columns in the matrix layout: B operands per 32-column half, whether the lane's
// column of each half is voted (in the grid, or a wrapped halo column), and for periodic kernels
// the lane's row stride and base in bytes (as in Cols).
template <int G>
struct VoteCols {
    float op[2 * G];
    bool in[2 * G];
    int rs[2 * G], rb[2 * G];
};

template <int G, bool PER>
__device__ __forceinline__ VoteCols<G> vote_cols(const Cols<G> &cl, const GridArgs &g, int first_col, int lane) {
    VoteCols<G> vc;
    constexpr int stride = Lane<G, true>::STRIDE;
#pragma unroll
    for (int q = 0; q < G; ++q) swap_halves(cl.S[q], cl.C[q], vc.op[2 * q], vc.op[2 * q + 1]);
#pragma unroll
    for (int h = 0; h < 2 * G; ++h) {
        const int j = first_col + 32 * h + (lane & 31), c = 32 * (h >> 1) + (lane & 31);
        const bool wrap = PER && (j == -1 || j == g.n_theta);
        vc.in[h] = (j >= 0 && j < g.n_theta) || wrap;
        vc.rs[h] = 4 * (wrap ? -stride : stride);
        vc.rb[h] = 4 * (wrap ? (g.n_rho - 1) * stride + c : c);
    }
    return vc;
}

// Votes of the first `rows` (wave-uniform) of 32 hits (operand a) in the tile's columns.  CLAMP:
// votes outside [0, n_rho) (and NaN) go to the dummy row; otherwise every vote is in range.
// Blocks of 8 hits past `rows` are skipped; the caller makes the rest of the last block harmless.
template <int G, bool PER, bool CLAMP>
__device__ __forceinline__ void vote_mfma(uint32_t *tile, float a, uint32_t rows, const VoteCols<G> &vc,
                                          const f32x16 &bf, const GridArgs &g, float dummy, int lane) {
    constexpr int ST = Lane<G, true>::STRIDE;
    char *base = reinterpret_cast<char *>(tile);
#pragma unroll
    for (int h = 0; h < 2 * G; ++h) {
        const f32x16 t = __builtin_amdgcn_mfma_f32_32x32x2f32(a, vc.op[h], bf, 0, 0, 0);
        if (vc.in[h]) {
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                if (b && (uint32_t)(8 * b) >= rows) break;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    float tt = t[4 * b + i];
                    if (CLAMP) {
                        // the literal test 0 <= t < n_rho as one unsigned compare of the bits
                        // (negative and NaN bits are above every finite positive one; the
                        // addition turns -0, which is in range, into +0)
                        tt += 0.0f;
                        tt = __float_as_uint(tt) < __float_as_uint(g.nrho_f) ? tt : dummy;
                    }
                    const int k = (int)tt;
                    uint32_t *cell = PER && !CLAMP
                        ? reinterpret_cast<uint32_t *>(base + (__mul24(k, vc.rs[h]) + vc.rb[h]))
                        : &tile[k * ST + 32 * (h >> 1) + (lane & 31)];
                    if (PER && CLAMP) {
                        // a wrapped lane reverses the rows of the grid, not the dummy row (which is row
                        // n_rho here: an event with such hits reaches every row of a periodic grid, so
                        // no window holds it)
                        const bool in = tt < g.nrho_f;
                        cell = in ? reinterpret_cast<uint32_t *>(base + (__mul24(k, vc.rs[h]) + vc.rb[h])) : cell;
                    }
                    lds_add(cell, h & 1 ? 0x10000u : 1u);
                }
            }
        }
    }
}

// A chunk with at most this many valid hits whose votes may leave the grid votes them one at a
// time with the literal range test; a chunk with more takes the clamped form for all its hits.
// (one at a time costs about 14 instructions per hit and 64 columns, clamping 3 more per vote
// instruction of the chunk, 192: they meet near 14 hits; most chunks hold none or one)
constexpr uint32_t kFewUnsafe = 8;

// Votes of hits [hb, he), 64 at a time, one per lane; returns the number of valid hits seen.
// The next 64 hits are loaded while the current ones vote.  dup (duplicate suppression, else
// null): the event's keep bytes as the duplicate pass left them; a later copy of a hit is
// counted as valid (in the sweep that maps the hits) but does not vote.
// Lanes without a vote of their own (past he, invalid, a later copy, or voting one at a time)
// take u = v = 0, which votes row (int)B of every column; their number is subtracted from that row
// at the end of the range, so the vote loop carries no masks (packed sums wrap and unwrap
// exactly, as 32-bit additions).  When B itself lies outside the grid no hit is ever
// provably in range, so such a lane votes only in clamped chunks, as NaN, into the dummy row.
// dummy_row: the tile's dummy row.
// uv (else null): room for the wave's mapped hits, u at uv[i] and v at uv[uv_stride + i], NaN for
// an invalid hit.  They are written when they are not there yet (have false) and read in place of
// x and y when they are: the map's two divisions and tests take 40 of the 55 instructions a chunk
// costs beside its votes, and an event's hits are swept once per tile (10,000 events, 360 x 256:
// 1,603 -> 1,559 us; dense 720 x 512: 1,341 -> 1,293 us).
template <int G, bool PER = false>
__device__ uint32_t vote_range(uint32_t *tile, const float *x, const float *y, uint32_t hb, uint32_t he,
                               const Cols<G> &cl, const GridArgs &g, int first_col, int lane, uint32_t &bad,
                               float dummy_row, const uint8_t *dup = nullptr, float *uv = nullptr,
                               uint32_t uv_stride = 0, bool have = false) {
    have = have && uv;
    if (have) {
        x = uv;
        y = uv + uv_stride;
    }
    const Lane<G, true> ln(lane);
    const VoteCols<G> vc = vote_cols<G, PER>(cl, g, first_col, lane);
    const f32x16 bf = bias16(g.Bf);
    uint32_t n_valid = 0, extra = 0;
    float xn = 0.0f, yn = 0.0f;
    if (hb + lane < he) { xn = at(x, hb + lane); yn = at(y, hb + lane); }
    for (uint32_t base = hb; base < he; base += 64) {
        const uint32_t i = base + lane;
        const float xi = xn, yi = yn;
        if (i + 64 < he) { xn = at(x, i + 64); yn = at(y, i + 64); }
        bool live = i < he;
        if (dup) {
            const bool copy = live && (dup[i] & kKeepDuplicate) != 0;
            if (!have) n_valid += (uint32_t)__popcll(__ballot(copy && valid_hit(xi, yi)));
            live = live && !copy;
        }
        float u = xi, v = yi;
        bool valid = live && u == u;
        if (!have) {
            valid = conformal(live ? xi : 0.0f, live ? yi : 0.0f, u, v) && live;
            if (live && !valid) bad = 1u;
            if (uv && live) {
                put(uv, i, valid ? u : __uint_as_float(0x7fc00000u));
                put(uv + uv_stride, i, v);
            }
        }
        const bool safe = valid && all_in_range(u, v, g);
        const uint64_t bs = __ballot(safe);
        uint64_t bu = __ballot(valid && !safe);
        const uint32_t nu = (uint32_t)__popcll(bu), ns = (uint32_t)__popcll(bs);
        n_valid += ns + nu;
        const uint32_t rows = min(he - base, 64u);
        float a0, a1;
        if (nu <= kFewUnsafe) {
            if (ns) {
                swap_halves(safe ? v : 0.0f, safe ? u : 0.0f, a0, a1);
#pragma unroll 1
                for (uint32_t b = 0; b < rows; b += 32, a0 = a1)
                    vote_mfma<G, PER, false>(tile, a0, rows - b, vc, bf, g, 0.0f, lane);
                extra += ((rows + 7u) & ~7u) - ns;
            }
            for (; bu; bu &= bu - 1ull) {
                const int m = __builtin_ctzll(bu);
                const float um = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(u), m));
                const float vm = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(v), m));
#pragma unroll
                for (int q = 0; q < G; ++q) {
                    const float w = __builtin_fmaf(vm, cl.S[q], cl.B[q]);
                    const float t = __builtin_fmaf(um, cl.C[q], w);
                    if (t >= 0.0f && t < g.nrho_f) lds_add(cell_of<G, true, PER>(tile, (int)t, cl, ln, q), ln.inc);
                }
            }
        } else {
            const float nan = __uint_as_float(0x7fc00000u);
            swap_halves(valid ? v : nan, valid ? u : nan, a0, a1);
#pragma unroll 1
            for (uint32_t b = 0; b < rows; b += 32, a0 = a1)
                vote_mfma<G, PER, true>(tile, a0, rows - b, vc, bf, g, dummy_row, lane);
        }
    }
    if (extra) {
#pragma unroll
        for (int q = 0; q < G; ++q) {
            const int j = first_col + 64 * q + lane;
            const bool voted = (j >= 0 && j < g.n_theta) || (PER && (j == -1 || j == g.n_theta));
            if (voted)
                lds_add(cell_of<G, true, PER>(tile, __builtin_amdgcn_readfirstlane((int)g.Bf), cl, ln, q), 0u - extra * ln.inc);
        }
    }
    return n_valid;
}

// The wave's hits [hb, he) of an event of H hits: whole blocks of 8 (the granularity of a vote
// instruction's hits), spread evenly over the NW waves.
template <int NW>
__device__ __forceinline__ void wave_hits(uint32_t H, int wave, uint32_t &hb, uint32_t &he) {
    const uint32_t blocks = (H >> 3) + ((H & 7u) != 0u), w = (uint32_t)__builtin_amdgcn_readfirstlane(wave);   // scalar
    hb = min(H, (uint32_t)((uint64_t)blocks * w / NW) * 8u);
    he = min(H, (uint32_t)((uint64_t)blocks * (w + 1u) / NW) * 8u);
}

// First and last row any vote of an event can reach, from the smallest r2 = x^2 + y^2 among its
// valid hits (the map's own float expression): |t - B| <= wA / sqrt(r2) with wA the largest
// |(C_j, S_j)|; the float map and the two fmas of t add a few 2^-24 relative, far inside the 1e-6
// and 1e-5 margins kept here.  Rows are floor(t), so the floors of the bounds are the rows.
__device__ __forceinline__ void reached_rows(const GridArgs &g, float min_r2, int &klo, int &khi) {
    const double rmax = (1.0 + 1e-6) / sqrt((double)min_r2);
    const double span = g.wA * rmax, slack = 1e-5 * (fabs(g.wB) + span) + 1e-3;
    const double lo = g.wB - span - slack, hi = g.wB + span + slack;
    const double top = (double)(g.n_rho - 1);
    klo = lo <= 0.0 ? 0 : (lo >= top ? g.n_rho - 1 : (int)lo);
    khi = hi <= 0.0 ? 0 : (hi >= top ? g.n_rho - 1 : (int)hi);
}

// The window of `win` rows that starts at the first reached row (down to a multiple of 16): whether
// it holds every row the event reaches, those of the wrapped halo columns (reversed) included.
template <bool PER>
__device__ __forceinline__ bool window_of(const GridArgs &g, float min_r2, int win, int &b0) {
    int klo, khi;
    reached_rows(g, min_r2, klo, khi);
    if (PER) {
        const int lo_r = g.n_rho - 1 - khi, hi_r = g.n_rho - 1 - klo;
        klo = min(klo, lo_r);
        khi = max(khi, hi_r);
    }
    b0 = (klo / 16) * 16;
    return khi < b0 + win;
}

// The smallest valid r2 of the wave's hits, as the bits of a float (positive floats order as
// their bits), in every lane.
__device__ __forceinline__ uint32_t wave_min(uint32_t v);
__device__ __forceinline__ uint32_t min_r2_bits(const float *x, const float *y, uint32_t hb, uint32_t he, int lane) {
    uint32_t mn = __float_as_uint(FLT_MAX);
#pragma unroll 1
    for (uint32_t i = hb + lane; i < he; i += 64) {
        const float xi = at(x, i), yi = at(y, i);
        const float r2 = __builtin_fmaf(xi, xi, yi * yi);
        if (r2 > 0.0f && r2 <= FLT_MAX) mn = min(mn, __float_as_uint(r2));
    }
    return wave_min(mn);
}

// Step 4 on rows [16*u, 16*u + 16) of the lane's columns: bit b of mask[q] is set iff cell
// (column 64q + lane, row 16*u + b) is a peak.  Raster order is (theta, rho), so the column to
// the left and the row above come first:
//   peak <=> count >= threshold, count > every earlier neighbour, count >= every later one
//        <=> count >= max(threshold, max(earlier) + 1, max(later)).
// The lane slides a three-row window down its own column, reading four rows at a time; the
// vertical maxima of the neighbouring columns come from the neighbouring lanes through DPP wave
// shifts (and across a 64-column group boundary through readlane).  Rows outside the grid count
// as 0.  The two edge columns of the tile are halo columns; the caller drops their bits.
constexpr int kPeakRows = 16;

// Count of cell (row k, column of group q) or 0 outside the grid's rows.  Row k is the same for
// every lane.  Interior units (CHECK false) never leave the grid; at the edges the address is
// clamped into the tile so that the read is unconditional and only its value is dropped.
template <bool CHECK, int G, bool P>
__device__ __forceinline__ uint32_t cell_or_zero(const uint32_t *tile, int k, int n_rho,
                                                 const Lane<G, P> &ln, int q) {
    if (!CHECK) return ln.count(tile[k * Lane<G, P>::STRIDE + ln.col[q]]);
    const int kk = min(max(k, 0), n_rho);
    const uint32_t d = tile[kk * Lane<G, P>::STRIDE + ln.col[q]];
    return (k >= 0 && k < n_rho) ? ln.count(d) : 0u;
}

// WRAP (theta-periodic grid, first and last tile): the halo column beside column 0 is column
// n_theta - 1 and follows it in raster order, the one beside column n_theta - 1 is column 0 and
// precedes it, so for those two lanes the strict and the non-strict side trade places.
// UNROLL: issue the reads of all four 4-row blocks together (for kernels with the registers).
template <bool CHECK, int G, bool P, bool WRAP = false, bool UNROLL = false>
__device__ __forceinline__ void peak_rows(const uint32_t *tile, int unit, int n_rho, uint32_t T,
                                          const Lane<G, P> &ln, int lane, uint32_t *mask,
                                          int first_col = 0, int n_theta = 0) {
    const int k0 = unit * kPeakRows;
    uint32_t Mp[G], Mc[G];
#pragma unroll
    for (int q = 0; q < G; ++q) {
        Mp[q] = cell_or_zero<CHECK, G, P>(tile, k0 - 1, n_rho, ln, q);
        Mc[q] = cell_or_zero<CHECK, G, P>(tile, k0, n_rho, ln, q);
        mask[q] = 0u;
    }
    auto block = [&](int r0) {
        uint32_t N[G][4];
#pragma unroll
        for (int d = 0; d < 4; ++d)
#pragma unroll
            for (int q = 0; q < G; ++q) N[q][d] = cell_or_zero<CHECK, G, P>(tile, k0 + r0 + d + 1, n_rho, ln, q);
        // rows r0 .. r0+3 are tested; when no lane's count there reaches the threshold none of
        // them can be a peak and only the window moves on
        uint32_t bm = 0;
#pragma unroll
        for (int q = 0; q < G; ++q) bm = max(bm, max(max(Mc[q], N[q][0]), max(N[q][1], N[q][2])));
        if (__ballot(bm >= T) == 0ull) {
#pragma unroll
            for (int q = 0; q < G; ++q) { Mp[q] = N[q][2]; Mc[q] = N[q][3]; }
            return;
        }
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            const int k = k0 + r0 + d;
            uint32_t V[G];
#pragma unroll
            for (int q = 0; q < G; ++q) V[q] = max(max(Mp[q], Mc[q]), N[q][d]);
#pragma unroll
            for (int q = 0; q < G; ++q) {
                uint32_t VL = __builtin_amdgcn_update_dpp(0u, V[q], 0x138, 0xf, 0xf, true);   // lane - 1
                uint32_t VR = __builtin_amdgcn_update_dpp(0u, V[q], 0x130, 0xf, 0xf, true);   // lane + 1
                if (q > 0) {
                    const uint32_t x = __builtin_amdgcn_readlane(V[q > 0 ? q - 1 : 0], 63);
                    VL = lane == 0 ? x : VL;
                }
                if (q + 1 < G) {
                    const uint32_t x = __builtin_amdgcn_readlane(V[q + 1 < G ? q + 1 : 0], 0);
                    VR = lane == 63 ? x : VR;
                }
                uint32_t before, after;
                if (WRAP) {
                    const int j = first_col + 64 * q + lane;
                    const bool wl = j == 0, wr = j == n_theta - 1;
                    before = max(max(wl ? 0u : VL, wr ? VR : 0u), Mp[q]);
                    after = max(max(wl ? VL : 0u, wr ? 0u : VR), N[q][d]);
                } else {
                    before = max(VL, Mp[q]);
                    after = max(VR, N[q][d]);
                }
                const uint32_t need = max(max(T, before + 1u), after);
                mask[q] |= (uint32_t)((!CHECK || k < n_rho) && Mc[q] >= need) << (r0 + d);
            }
#pragma unroll
            for (int q = 0; q < G; ++q) { Mp[q] = Mc[q]; Mc[q] = N[q][d]; }
        }
    };
    if constexpr (UNROLL) {
#pragma unroll
        for (int r0 = 0; r0 < kPeakRows; r0 += 4) block(r0);
    } else {
#pragma unroll 1
        for (int r0 = 0; r0 < kPeakRows; r0 += 4) block(r0);
    }
}

// True when no count of the 16-row unit `unit` reaches T (then it holds no peak).  The unit's
// rows are contiguous in the packed tile, so the wave reads them whole, 16 bytes per lane per
// read, and takes the maximum of each lane's 16-bit counts: a few instructions where the 3x3
// test reads and compares every row.
template <int G>
__device__ __forceinline__ bool unit_below(const uint32_t *tile, int unit, uint32_t T, int lane) {
    typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
    constexpr int ST = Lane<G, true>::STRIDE, READS = ST * kPeakRows / 4 / 64;
    const uint4 *p = reinterpret_cast<const uint4 *>(tile + unit * kPeakRows * ST) + lane;
    u16x2 m = {0, 0};
#pragma unroll
    for (int i = 0; i < READS; ++i) {
        const uint4 v = p[64 * i];
        const u16x2 a = __builtin_elementwise_max(__builtin_bit_cast(u16x2, v.x), __builtin_bit_cast(u16x2, v.y));
        const u16x2 b = __builtin_elementwise_max(__builtin_bit_cast(u16x2, v.z), __builtin_bit_cast(u16x2, v.w));
        m = __builtin_elementwise_max(m, __builtin_elementwise_max(a, b));
    }
    const uint32_t mx = max((uint32_t)m.x, (uint32_t)m.y);
    return __ballot(mx >= T) == 0ull;
}

// Inclusive prefix sum over the 64 lanes with DPP row shifts and row broadcasts (no LDS).
__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t v, int) {
    v += __builtin_amdgcn_update_dpp(0u, v, 0x111, 0xf, 0xf, true);   // row_shr:1
    v += __builtin_amdgcn_update_dpp(0u, v, 0x112, 0xf, 0xf, true);   // row_shr:2
    v += __builtin_amdgcn_update_dpp(0u, v, 0x114, 0xf, 0xf, true);   // row_shr:4
    v += __builtin_amdgcn_update_dpp(0u, v, 0x118, 0xf, 0xf, true);   // row_shr:8
    v += __builtin_amdgcn_update_dpp(0u, v, 0x142, 0xa, 0xf, false);  // row_bcast:15 -> rows 1, 3
    v += __builtin_amdgcn_update_dpp(0u, v, 0x143, 0xc, 0xf, false);  // row_bcast:31 -> rows 2, 3
    return v;
}

__device__ __forceinline__ void store_peak(hough_peak *out, uint32_t j, uint32_t k, uint32_t c) {
    uint2 *p = reinterpret_cast<uint2 *>(out);
    *p = make_uint2((j & 0xffffu) | (k << 16), c);
}

// Dwords per word row of the fused kernels' dilated words: one more than the tile's columns, so
// that the words of one column lie in different banks (lane = hit lookups) as well as one word
// of different columns (lane = column lookups).
template <int G>
constexpr uint32_t kDilPitch = 64u * G + 1u;

// Step 4 (listing) and the retention marks of step 5, shared by all waves.  pmask[wd * TW + c]
// holds the peak bits of column c, rows 32*wd ...  Every wave computes the per-column peak
// counts and their prefix over the tile's columns (raster order is column-major), then lists
// the peaks of its own words at base + (peaks in earlier columns) + (peaks above in the same
// column).  It also writes the dilated words dil[wd * kDilPitch + c]: bit b set iff a peak of column c
// lies within rho_window rows of row 32*wd + b.  For rho_window < 32 a word follows from the
// peak words above and below it; wider windows OR the row range of every peak into dil (which
// the peak phase cleared).  colcnt (optional): each column's peak count, summed by the peak
// phase (else counted here from pmask).  tpk (optional): when the tile has at most kTilePeaks peaks, all of
// them in raster order, each with its column's C and S (and its row as the bits of z), for the
// retention of tiles with few peaks.  Returns the tile's peak count.
constexpr uint32_t kTilePeaks = 64;
// Deferred retention (sparse-grid kernels): a tile with at most kDeferTilePeaks peaks, all of
// them in the caller's peak list, leaves its retention to a later pass over the event's hits
// against the peak list itself, which then covers up to kDeferPeaks peaks of several tiles.
constexpr uint32_t kDeferTilePeaks = 80;
constexpr uint32_t kDeferPeaks = 256;

template <int G, bool P>
__device__ uint32_t emit_and_dilate(const uint32_t *tile, const uint32_t *pmask, uint32_t *dil, int w0,
                                    int nwords, int first_col, const GridArgs &g, hough_peak *out,
                                    uint32_t cap, uint32_t base, const Lane<G, P> &ln, int lane,
                                    int wave, int n_waves, float4 *tpk = nullptr,
                                    const Cols<G> *cl = nullptr, const uint32_t *colcnt = nullptr,
                                    uint32_t *edge = nullptr) {
    constexpr int TW = 64 * G, DP = (int)kDilPitch<G>, ST = Lane<G, P>::STRIDE;
    const int W = g.rho_window;
    uint32_t colbase[G];
    uint32_t carry = 0;
#pragma unroll
    for (int q = 0; q < G; ++q) {
        uint32_t tot = 0;
        if (colcnt)
            tot = colcnt[64 * q + lane];
        else
            for (int w = w0; w < w0 + nwords; ++w) tot += __popc(pmask[w * TW + 64 * q + lane]);
        const uint32_t incl = wave_inclusive_scan(tot, lane);
        colbase[q] = carry + incl - tot;
        carry += __shfl(incl, 63, 64);
    }
    if (carry == 0u) return 0u;
    const bool rec = tpk != nullptr && carry <= kTilePeaks;   // then every local index fits
    const int w1 = w0 + nwords;
    for (int wd = w0 + wave; wd < w1; wd += n_waves) {
#pragma unroll
        for (int q = 0; q < G; ++q) {
            const int c = 64 * q + lane;
            uint32_t m = pmask[wd * TW + c];
            if (W < 32) {
                const uint32_t up = wd > w0 ? pmask[(wd - 1) * TW + c] : 0u;
                const uint32_t dn = wd + 1 < w1 ? pmask[(wd + 1) * TW + c] : 0u;
                uint32_t d = m;
                for (int sft = 1; sft <= W; ++sft)
                    d |= (m << sft) | (m >> sft) | (up >> (32 - sft)) | (dn << (32 - sft));
                dil[wd * DP + c] = d;
            }
            if (!m) continue;
            uint32_t idx = base + colbase[q];
            for (int w = w0; w < wd; ++w) idx += __popc(pmask[w * TW + c]);
            const uint32_t j = (uint32_t)(first_col + c);
            while (m) {
                const int b = __builtin_ctz(m);
                m &= m - 1u;
                const int k = wd * 32 + b;
                const uint32_t cv = ln.count(tile[k * ST + ln.col[q]]);
                if (idx < cap) store_peak(out + idx, j, (uint32_t)k, cv);
                if (rec) {
                    tpk[idx - base] = make_float4(cl->C[q], cl->S[q], __int_as_float(k - W), 0.0f);
                    if (edge && (k <= W || k >= g.n_rho - W)) *edge = 1u;
                }
                ++idx;
                if (W >= 32) {
                    const int lo = k - W > 0 ? k - W : 0;
                    const int hi = k + W < g.n_rho - 1 ? k + W : g.n_rho - 1;
                    // words outside [w0, w1) hold rows no hit of the event reaches
                    for (int w = max(lo >> 5, w0); w <= min(hi >> 5, w1 - 1); ++w) {
                        const int a = max(lo, w * 32) - w * 32, e = min(hi, w * 32 + 31) - w * 32;
                        const uint32_t rm = (e == 31 ? ~0u : ((1u << (e + 1)) - 1u)) & ~((1u << a) - 1u);
                        __hip_atomic_fetch_or(&dil[w * DP + c], rm, __ATOMIC_RELAXED,
                                              __HIP_MEMORY_SCOPE_WORKGROUP);
                    }
                }
            }
        }
    }
    return carry;
}

// Step 5 on the current tile: a hit is kept when its own cell in some column of the tile has
// its dil bit set.  Returns bit 0 set iff kept.  PITCH: dwords per word row of dil.
template <int G, uint32_t PITCH>
__device__ __forceinline__ uint32_t lookup1(const uint32_t *dil, float u, float v, bool checked,
                                            const Cols<G> &cl, int lane, float nrho_f) {
    uint32_t m = 0;
#pragma unroll
    for (int q = 0; q < G; ++q) {
        const float w = __builtin_fmaf(v, cl.S[q], cl.B[q]);
        const float t = __builtin_fmaf(u, cl.C[q], w);
        if (!checked || (t >= 0.0f && t < nrho_f)) {
            const uint32_t k = (uint32_t)(int)t;
            // word k / 32 of the column (a shift and one multiply- or shift-add: the empty asm
            // keeps the compiler from regrouping the pair), then bit k mod 32 (the bit-field
            // extract takes its offset modulo 32)
            uint32_t kw = k >> 5;
            asm("" : "+v"(kw));
            m |= __builtin_amdgcn_ubfe(dil[__umul24(kw, PITCH) + 64u * q + (uint32_t)lane], k, 1u);
        }
    }
    return m;
}

// OR over the 64 lanes (DPP row shifts and row broadcasts, no LDS), returned wave-uniform.
__device__ __forceinline__ uint32_t wave_or(uint32_t v) {
    v |= __builtin_amdgcn_update_dpp(0u, v, 0x111, 0xf, 0xf, true);   // row_shr:1
    v |= __builtin_amdgcn_update_dpp(0u, v, 0x112, 0xf, 0xf, true);   // row_shr:2
    v |= __builtin_amdgcn_update_dpp(0u, v, 0x114, 0xf, 0xf, true);   // row_shr:4
    v |= __builtin_amdgcn_update_dpp(0u, v, 0x118, 0xf, 0xf, true);   // row_shr:8
    v |= __builtin_amdgcn_update_dpp(0u, v, 0x142, 0xa, 0xf, false);  // row_bcast:15 -> rows 1, 3
    v |= __builtin_amdgcn_update_dpp(0u, v, 0x143, 0xc, 0xf, false);  // row_bcast:31 -> rows 2, 3
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// Look up the staged hits st[0 .. n.total) (the first n.safe need no range test), four at a
// time so that their reads are in flight together.  Each lane gathers its own column's verdicts
// as bits (hit h at bit h mod 32 of one of two words) and one OR across the wave at the end
// turns them into the mask of kept stage slots.
template <int G, uint32_t PITCH>
__device__ __forceinline__ uint64_t lookup_staged(const uint32_t *dil, const float2 *st, StageCount n,
                                                  const Cols<G> &cl, int lane, float nrho_f) {
    const float4 *st4 = reinterpret_cast<const float4 *>(st);
    uint32_t w[2] = {0u, 0u};
    uint32_t h = 0;
    // hits h .. h+3 into bits h mod 32 .. of word `half` (h is a multiple of 4, so a group
    // never straddles the two words)
    auto four = [&](uint32_t &acc, uint32_t sh) {
        const float4 a = st4[h >> 1], b = st4[(h >> 1) + 1];
        const float uu[4] = {a.x, a.z, b.x, b.z}, vv[4] = {a.y, a.w, b.y, b.w};
        uint32_t kk[4][G], wd[4][G];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int q = 0; q < G; ++q) {
                const float t = __builtin_fmaf(uu[i], cl.C[q], __builtin_fmaf(vv[i], cl.S[q], cl.B[q]));
                kk[i][q] = (uint32_t)(int)t;
                uint32_t kw = kk[i][q] >> 5;        // see lookup1
                asm("" : "+v"(kw));
                wd[i][q] = __umul24(kw, PITCH) + 64u * q + (uint32_t)lane;
            }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int q = 0; q < G; ++q) wd[i][q] = dil[wd[i][q]];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int q = 0; q < G; ++q) {
                // one shift-or per bit (the empty asm keeps the compiler from regrouping the ORs
                // into separate shifts and three-input ORs)
                acc |= __builtin_amdgcn_ubfe(wd[i][q], kk[i][q], 1u) << (sh + i);
                asm("" : "+v"(acc));
            }
    };
    for (; h + 4 <= n.safe && h < 32; h += 4) four(w[0], h);
    for (; h + 4 <= n.safe; h += 4) four(w[1], h - 32);
    for (; h < n.total; ++h) {
        const float2 p = st[h];
        const uint32_t m = lookup1<G, PITCH>(dil, p.x, p.y, h >= n.safe, cl, lane, nrho_f);
        if (h < 32) w[0] |= m << h; else w[1] |= m << (h - 32);
    }
    if (n.total == 0) return 0ull;
    const uint32_t klo = wave_or(w[0]);
    const uint32_t khi = n.total > 32 ? wave_or(w[1]) : 0u;
    return ((uint64_t)khi << 32) | klo;
}

__device__ __forceinline__ uint64_t low_bits(uint32_t n) { return n >= 64 ? ~0ull : ((1ull << n) - 1ull); }

// Lookups of up to 64 hits whose votes are all in range, lane = column: the hits of the lanes in
// `who` are compacted through the wave's stage (padded to a multiple of four with u = v = 0) and
// looked up four at a time.  Returns the lanes of `who` that are kept.
template <int G>
__device__ __forceinline__ uint64_t lookup_lanes(const uint32_t *dil, float2 *st, float u, float v, uint64_t who,
                                                 const Cols<G> &cl, const GridArgs &g, int lane) {
    if (!who) return 0ull;
    const uint32_t n = (uint32_t)__popcll(who), pos = mbcnt(who);
    const bool me = (who >> lane) & 1ull;
    if (me) st[pos] = make_float2(u, v);
    const float z = __int_as_float(opaque(0));
    if (lane < 3 && n + (uint32_t)lane < 64u) st[n + lane] = make_float2(z, z);
    wave_sync();
    const uint32_t n4 = (n + 3u) & ~3u;
    const uint64_t found = lookup_staged<G, kDilPitch<G>>(dil, st, StageCount{n4, n4}, cl, lane, g.nrho_f);
    wave_sync();
    return __ballot(me && ((found >> pos) & 1ull));
}

// The same for hits whose votes may leave the grid, one at a time with the literal range test.
template <int G>
__device__ __forceinline__ uint64_t lookup_checked(const uint32_t *dil, float u, float v, uint64_t who,
                                                   const Cols<G> &cl, const GridArgs &g, int lane) {
    uint64_t kept = 0;
    for (; who; who &= who - 1ull) {
        const int m = __builtin_ctzll(who);
        const float um = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(u), m));
        const float vm = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(v), m));
        if (__ballot(lookup1<G, kDilPitch<G>>(dil, um, vm, true, cl, lane, g.nrho_f) != 0u)) kept |= 1ull << m;
    }
    return kept;
}

// Hits of a wave's range that are valid and not yet kept, once there are at most 64 of them:
// lane l holds one entry (an event-local hit index and the mapped hit; bit 31 of idx set for a
// later copy of a hit under duplicate suppression, bit 30 when every vote is in range) while bit
// l of `live` is set.  Later tiles look up only these instead of mapping the whole range again.
struct Pending {
    uint32_t idx;
    float u, v;
    uint64_t live;   // wave-uniform
    bool on;         // wave-uniform
};
constexpr uint32_t kPendingCopy = 0x80000000u, kPendingSafe = 0x40000000u, kPendingIdx = 0x3fffffffu;

// Append the entries of the lanes in `who` after the n entries held (n + |who| <= 64): a push
// across lanes that is a permutation of all 64 (the other lanes' values are dropped).
__device__ __forceinline__ void push_pending(Pending &pd, uint32_t n, uint64_t who, uint32_t idx, float u, float v,
                                             int lane) {
    lane = opaque(lane);
    const uint32_t c = (uint32_t)__popcll(who);
    const uint32_t to = ((who >> lane) & 1ull) ? n + mbcnt(who) : n + c + mbcnt(~who);
    const int at = (int)((to & 63u) << 2);
    const uint32_t ri = (uint32_t)__builtin_amdgcn_ds_permute(at, (int)idx);
    const uint32_t ru = (uint32_t)__builtin_amdgcn_ds_permute(at, (int)__float_as_uint(u));
    const uint32_t rv = (uint32_t)__builtin_amdgcn_ds_permute(at, (int)__float_as_uint(v));
    if ((uint32_t)lane >= n && (uint32_t)lane < n + c) {
        pd.idx = ri;
        pd.u = __uint_as_float(ru);
        pd.v = __uint_as_float(rv);
    }
}

// Collect the valid unkept hits of [hb, he) into the pending list (caller: at most 64 of them).
__device__ void build_pending(Pending &pd, const float *x, const float *y, const uint8_t *ke, uint32_t hb,
                              uint32_t he, const GridArgs &g, int lane) {
    // runs once per wave and event: keep the compiler from holding its per-lane addresses in
    // registers across the whole event
    asm volatile("" : "+v"(lane));
    uint32_t n = 0;
    for (uint32_t base = hb; base < he; base += 64) {
        const uint32_t i = base + lane;
        const uint32_t kv = (i < he) ? ke[i] : 1u;
        const bool cand = (i < he) && !(kv & 1u);
        float xi = 0.0f, yi = 0.0f;
        if (cand) { xi = at(x, i); yi = at(y, i); }
        float u, v;
        const uint64_t b = __ballot(conformal(xi, yi, u, v) && cand);
        if (!b) continue;
        push_pending(pd, n, b,
                     i | ((kv & (uint32_t)kKeepDuplicate) << 30) | (all_in_range(u, v, g) ? kPendingSafe : 0u), u, v,
                     lane);
        n += (uint32_t)__popcll(b);
    }
    pd.on = true;
    pd.live = low_bits(n);
}

// The keep bytes of the pending entries in `kept`, and the list without them.
__device__ __forceinline__ uint32_t drop_pending(Pending &pd, uint64_t kept, uint8_t *ke, int lane) {
    if ((kept >> lane) & 1ull)
        ke[pd.idx & kPendingIdx] = (uint8_t)(1u | ((pd.idx & kPendingCopy) ? (uint32_t)kKeepDuplicate : 0u));
    pd.live &= ~kept;
    return (uint32_t)__popcll(kept);
}

// Step 5 for the pending list: look the live entries up, write the keep byte of each kept entry
// and drop it.
template <int G>
__device__ uint32_t retain_pending(Pending &pd, const uint32_t *dil, float2 *st, uint8_t *ke, const Cols<G> &cl,
                                   const GridArgs &g, int lane) {
    if (pd.live == 0ull) return 0u;
    const uint64_t safe = __ballot((pd.idx & kPendingSafe) != 0u) & pd.live;
    uint64_t kept = lookup_lanes<G>(dil, st, pd.u, pd.v, safe, cl, g, lane);
    kept |= lookup_checked<G>(dil, pd.u, pd.v, pd.live & ~safe, cl, g, lane);
    return drop_pending(pd, kept, ke, lane);
}

// Step 5 for 64 hits, one per lane, a few of the tile's columns at a time: lane l looks its own
// bin up in the same column as every other lane, so a column costs 7 instructions for all 64 hits
// where the lookup with lane = column costs 8 per hit.  On a tile with many peaks most hits meet
// one in a few columns: rounds of 8 columns, evenly spaced, until a round no longer pays (each
// hit it keeps spares the lookup of that hit in every column).  Returns the mask of kept lanes
// among `want` (hits whose votes are all in range; the other lanes' u and v are 0, so their bins
// are in range too).  Halo and out-of-grid columns have no dilated bits.
// (10,000 events, 360 x 256: 839 -> 739 M VALU instructions with the pending list's lookups four
// at a time; with the phases' registers kept apart, see opaque(), the batch takes 1.60 ms, 1.88
// with the VALU vote and lane = column lookups alone)
constexpr int kColumnRoundHits = 8;       // a round costs as much as the lookup of this many hits
template <int G>
__device__ __forceinline__ uint64_t kept_by_columns(const uint32_t *dil, float u, float v, uint64_t want,
                                                    int first_col, const GridArgs &g) {
    typedef const __attribute__((address_space(4))) float *cfloat;       // read by scalar loads
    const cfloat C = (cfloat)(uintptr_t)g.C, S = (cfloat)(uintptr_t)g.S;
    uint32_t m = 0;
    uint64_t kept = 0;
    for (int r = 0; r < 8 * G; ++r) {
        const int c0 = (5 * r + 2) & (8 * G - 1);                         // rounds spread over the tile too
        uint32_t word[8], k[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int c = c0 + 8 * G * i, j = min(max(first_col + c, 0), g.n_theta - 1);
            const float t = __builtin_fmaf(u, C[j], __builtin_fmaf(v, S[j], g.Bf));
            k[i] = (uint32_t)(int)t;
            uint32_t kw = k[i] >> 5;                                      // see lookup1
            asm("" : "+v"(kw));
            word[i] = dil[__umul24(kw, kDilPitch<G>) + (uint32_t)c];
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) m |= word[i] >> (k[i] & 31u);
        const uint64_t now = __ballot((m & 1u) != 0u) & want;
        const uint32_t newly = (uint32_t)__popcll(now & ~kept), left = (uint32_t)__popcll(want & ~now);
        kept = now;
        if (newly < (uint32_t)kColumnRoundHits || left < (uint32_t)kColumnRoundHits) break;
    }
    return kept;
}

// Step 5 over the whole range [hb, he): every unkept valid hit is mapped again and looked up
// (many: kept_by_columns first, then the hits it leaves with lane = column); each lane sets the
// kept bit of its own hit's keep byte (the event's keep bytes were cleared, or written by the
// duplicate pass, when it started, and only this lane touches them).  The next 64 hits and keep
// bytes are loaded while these are looked up.  When at most 64 valid hits remain unkept they
// become the pending list.  Returns the number of hits newly kept; `left` receives how many
// valid hits remain unkept.
template <int G>
__device__ uint32_t retain_range(Pending &pd, const uint32_t *dil, float2 *st, const float *x, const float *y,
                                 uint8_t *ke, uint32_t hb, uint32_t he, const Cols<G> &cl, const GridArgs &g,
                                 int first_col, bool many, int lane, uint32_t &left) {
    uint32_t newly = 0;
    left = 0;
    uint32_t kn = 1u;
    float xn = 0.0f, yn = 0.0f;
    if (hb + lane < he) { kn = ke[hb + lane]; xn = at(x, hb + lane); yn = at(y, hb + lane); }
    for (uint32_t base = hb; base < he; base += 64) {
        const uint32_t i = base + lane;
        const uint32_t kv = kn;
        const float xi = xn, yi = yn;
        if (i + 64 < he) { kn = ke[i + 64]; xn = at(x, i + 64); yn = at(y, i + 64); }
        const bool todo = (i < he) && !(kv & 1u);
        if (__ballot(todo) == 0ull) continue;                   // whole chunk already kept
        float u, v;
        const bool valid = conformal(todo ? xi : 0.0f, todo ? yi : 0.0f, u, v) && todo;
        const bool safe = valid && all_in_range(u, v, g);
        const uint64_t bs = __ballot(safe), bv = __ballot(valid);
        uint64_t kept = 0;
        if (many && __popcll(bs) >= kColumnRoundHits)
            kept = kept_by_columns<G>(dil, safe ? u : 0.0f, safe ? v : 0.0f, bs, first_col, g);
        kept |= lookup_lanes<G>(dil, st, u, v, bs & ~kept, cl, g, lane);
        kept |= lookup_checked<G>(dil, u, v, bv & ~bs, cl, g, lane);
        if ((kept >> lane) & 1ull) ke[i] = (uint8_t)(kv | 1u);
        newly += (uint32_t)__popcll(kept);
        const uint64_t rest = bv & ~kept;
        const uint32_t c = (uint32_t)__popcll(rest);
        if (c && left + c <= 64u)
            push_pending(pd, left, rest, i | ((kv & (uint32_t)kKeepDuplicate) << 30) | (safe ? kPendingSafe : 0u), u, v,
                         lane);
        left += c;
    }
    if (left <= 64u) {
        pd.on = true;
        pd.live = low_bits(left);
    }
    return newly;
}

// Step 5 on a tile with at most kTilePeaks peaks, one lane per hit: hit (u, v) is kept by
// peak (column j, row k) when its own bin in column j (the vote's arithmetic, in range) is
// within rho_window of k, which is what a lookup of the dilated words tests; here it costs
// one step per peak for 64 hits instead of one step per hit for the tile's columns.  The list
// holds k - W (as int bits in z).  For a peak with W < k < N_rho - W the range test is implied:
// a bin t outside [0, N_rho) truncates to an integer below 1 or at least N_rho, out of
// [k - W, k + W]; so unless the tile has a peak nearer an edge (`edge`) a peak costs two fmas,
// a conversion, a subtraction and one unsigned compare.  t is first clamped to [-2, N_rho + W + 2]
// (one v_med3), which keeps the conversion defined and changes no verdict: a clamped bin lies
// outside every peak's window either way.  Returns the mask of kept lanes among `valid`, and
// stops once every valid lane is kept.
__device__ __forceinline__ uint64_t kept_by_peaks(const float4 *tpk, uint32_t np, float u, float v, bool valid,
                                                  bool edge, const GridArgs &g) {
    const uint64_t want = __ballot(valid);
    const uint32_t w2 = 2u * (uint32_t)g.rho_window;
    const float hi = g.nrho_f + (float)g.rho_window + 2.0f;
    uint64_t km = 0;
    // one peak: its compares go straight into wave masks (scalar ORs and ANDs)
    auto test = [&](const float4 &P) {
        const float t = __builtin_fmaf(u, P.x, __builtin_fmaf(v, P.y, g.Bf));
        const uint32_t dd = (uint32_t)(int)__builtin_amdgcn_fmed3f(t, -2.0f, hi) - __float_as_uint(P.z);
        uint64_t m = __ballot(dd <= w2);
        if (edge) m &= __ballot(t >= 0.0f) & __ballot(t < g.nrho_f);
        km |= m;
    };
    uint32_t p = 0;
    // four peaks at a time, their list reads issued together; done once every valid lane is kept
    for (; p + 4 <= np; p += 4) {
        float4 P[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) P[q] = tpk[p + q];       // the same address in every lane
#pragma unroll
        for (int q = 0; q < 4; ++q) test(P[q]);
        if ((km & want) == want) return want;
    }
    for (; p < np; ++p) test(tpk[p]);
    return km & want;
}

// retain_pending with the tile's peak list.
__device__ uint32_t retain_pending_peaks(Pending &pd, const float4 *tpk, uint32_t np, bool edge, uint8_t *ke,
                                         const GridArgs &g, int lane) {
    if (pd.live == 0ull) return 0u;
    const bool me = (pd.live >> lane) & 1ull;
    return drop_pending(pd, kept_by_peaks(tpk, np, me ? pd.u : 0.0f, me ? pd.v : 0.0f, me, edge, g), ke, lane);
}

// retain_range with the tile's peak list: each lane maps and tests its own unkept hit.
__device__ uint32_t retain_range_peaks(const float4 *tpk, uint32_t np, bool edge, const float *x, const float *y,
                                       uint8_t *ke, uint32_t hb, uint32_t he, const GridArgs &g, int lane,
                                       uint32_t &left) {
    uint32_t newly = 0;
    left = 0;
    // the keep bytes and hits of the next 64 are loaded while these are tested
    uint32_t kn = 1u;
    float xn = 0.0f, yn = 0.0f;
    if (hb + lane < he) { kn = ke[hb + lane]; xn = at(x, hb + lane); yn = at(y, hb + lane); }
    for (uint32_t base = hb; base < he; base += 64) {
        const uint32_t i = base + lane;
        const uint32_t kv = kn;
        const float xi = xn, yi = yn;
        if (i + 64 < he) { kn = ke[i + 64]; xn = at(x, i + 64); yn = at(y, i + 64); }
        const bool cand = (i < he) && !(kv & 1u);
        if (__ballot(cand) == 0ull) continue;            // whole chunk already kept
        float u = 0.0f, v = 0.0f;
        bool valid = false;
        if (cand) valid = conformal(xi, yi, u, v);
        const uint64_t km = kept_by_peaks(tpk, np, u, v, valid, edge, g);
        if ((km >> lane) & 1ull) ke[i] = (uint8_t)(kv | 1u);
        const uint32_t nk = (uint32_t)__popcll(km);
        newly += nk;
        left += (uint32_t)__popcll(__ballot(valid)) - nk;
    }
    return newly;
}

// ------------------------------------------------------------------------ plain path
// hough_vote: workgroup (32-column group, rho slab of slab_rows rows), all of the event's hits swept
// through one 32-bit counter per cell, [rows + 1][32] in LDS (the last row a dummy).  One event
// is latency: the groups are as narrow as one matrix instruction, so that the most
// workgroups share the votes, and the tile is written out 16 bytes per lane along a column.
// (one event of 4,400 hits, 720 x 512: 33 us with 64-column groups and 4-byte stores that
// touched 64 lines each, 11 us so; 1,500 hits on 1000 x 1000: 44 and 9 us)
// SLAB: the tile holds rows [r0, r0 + nrows) only, and a vote outside goes to the dummy row.
template <bool SLAB>
__device__ __forceinline__ void vote_mfma32(uint32_t *tile, float a, uint32_t rows, float op, bool in,
                                            const f32x16 &bf, const GridArgs &g, int r0, int nrows, int lane) {
    const f32x16 t = __builtin_amdgcn_mfma_f32_32x32x2f32(a, op, bf, 0, 0, 0);
    if (!in) return;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        if (b && (uint32_t)(8 * b) >= rows) break;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float tt = t[4 * b + i];
            uint32_t k;
            if (SLAB) {
                tt += 0.0f;                                   // see vote_mfma
                tt = __float_as_uint(tt) < __float_as_uint(g.nrho_f) ? tt : -1.0f;
                k = min((uint32_t)((int)tt - r0), (uint32_t)nrows);
            } else {
                k = (uint32_t)(int)tt;
            }
            lds_add(&tile[k * 32u + (uint32_t)(lane & 31)], 1u);
        }
    }
}

// Votes of hits [hb, he) into such a tile (the whole column when r0 = 0 and nrows = n_rho); the
// same rules as vote_range.
__device__ void vote_range32(uint32_t *tile, const float *x, const float *y, uint32_t hb, uint32_t he,
                             const GridArgs &g, int first_col, int r0, int nrows, int lane) {
    const int j = first_col + (lane & 31);
    const bool in = j < g.n_theta;
    const float C = in ? g.C[j] : 0.0f, S = in ? g.S[j] : 0.0f, op = lane < 32 ? S : C;
    const bool whole = r0 == 0 && nrows == g.n_rho;
    const f32x16 bf = bias16(g.Bf);
    uint32_t extra = 0;
    float xn = 0.0f, yn = 0.0f;
    if (hb + lane < he) { xn = x[hb + lane]; yn = y[hb + lane]; }
    for (uint32_t base = hb; base < he; base += 64) {
        const uint32_t i = base + lane;
        const float xi = xn, yi = yn;
        const bool live = i < he;
        if (i + 64 < he) { xn = x[i + 64]; yn = y[i + 64]; }
        float u, v;
        const bool valid = conformal(live ? xi : 0.0f, live ? yi : 0.0f, u, v) && live;
        const bool safe = valid && all_in_range(u, v, g);
        const uint64_t bs = __ballot(safe);
        uint64_t bu = __ballot(valid && !safe);
        const uint32_t rows = min(he - base, 64u), ns = (uint32_t)__popcll(bs);
        float a0, a1;
        if (whole && (uint32_t)__popcll(bu) <= kFewUnsafe) {
            if (ns) {
                swap_halves(safe ? v : 0.0f, safe ? u : 0.0f, a0, a1);
                vote_mfma32<false>(tile, a0, rows, op, in, bf, g, r0, nrows, lane);
                if (rows > 32u) vote_mfma32<false>(tile, a1, rows - 32u, op, in, bf, g, r0, nrows, lane);
                extra += ((rows + 7u) & ~7u) - ns;
            }
            for (; bu; bu &= bu - 1ull) {
                const int m = __builtin_ctzll(bu);
                const float um = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(u), m));
                const float vm = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(v), m));
                const float t = __builtin_fmaf(um, C, __builtin_fmaf(vm, S, g.Bf));
                if (lane < 32 && in && t >= 0.0f && t < g.nrho_f) lds_add(&tile[(uint32_t)(int)t * 32u + lane], 1u);
            }
        } else {
            const float nan = __uint_as_float(0x7fc00000u);
            swap_halves(valid ? v : nan, valid ? u : nan, a0, a1);
            vote_mfma32<true>(tile, a0, rows, op, in, bf, g, r0, nrows, lane);
            if (rows > 32u) vote_mfma32<true>(tile, a1, rows - 32u, op, in, bf, g, r0, nrows, lane);
        }
    }
    if (extra && lane < 32 && in) lds_add(&tile[(uint32_t)(int)g.Bf * 32u + lane], 0u - extra);
}

// vec: rows start on a 16-byte (8-byte for 16-bit cells) boundary and hold whole quads.
template <int NW, typename T>
__global__ __launch_bounds__(NW * 64) void k_vote(GridArgs g, const float *__restrict__ x,
                                                  const float *__restrict__ y, uint32_t n_hits,
                                                  T *__restrict__ acc, int slab_rows, int vec) {
    extern __shared__ __align__(16) uint32_t tile[];                    // [(nrows + 1) * 32]
    const int r0 = (int)blockIdx.y * slab_rows, nrows = min(slab_rows, g.n_rho - r0);
    const int lane = threadIdx.x & 63, wave = wave_id(), first = (int)blockIdx.x * 32;
    for (int i = threadIdx.x; i < (nrows + 1) * 8; i += NW * 64)
        reinterpret_cast<uint4 *>(tile)[i] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    uint32_t hb, he;
    wave_hits<NW>(n_hits, wave, hb, he);
    vote_range32(tile, x, y, hb, he, g, first, r0, nrows, lane);
    __syncthreads();
    const int j = first + (lane & 31);
    if (j >= g.n_theta) return;
    T *row = acc + (size_t)j * g.n_rho + r0;
    const uint32_t *col = tile + (lane & 31);
    if (vec) {
        for (int q = 2 * wave + (lane >> 5); q < nrows / 4; q += 2 * NW) {
            const uint32_t a = col[128 * q], b = col[128 * q + 32], c = col[128 * q + 64], d = col[128 * q + 96];
            if constexpr (sizeof(T) == 4)
                reinterpret_cast<uint4 *>(row)[q] = make_uint4(a, b, c, d);
            else
                reinterpret_cast<uint2 *>(row)[q] = make_uint2(a | (b << 16), c | (d << 16));
        }
    } else {
        for (int k = 2 * wave + (lane >> 5); k < nrows; k += 2 * NW) row[k] = (T)col[32 * k];
    }
}

__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = max(v, (uint32_t)__shfl_xor((int)v, o, 64));
    return v;
}

__device__ __forceinline__ uint32_t wave_min(uint32_t v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = min(v, (uint32_t)__shfl_xor((int)v, o, 64));
    return v;
}

// The threshold of the iterative finder for a largest count mx.
__device__ __forceinline__ uint32_t iter_threshold(uint32_t mx, uint32_t frac_num, uint32_t frac_den, uint32_t floor_t) {
    const uint64_t top = (uint64_t)mx * frac_num + frac_den - 1u;
    // (a 64-bit division costs some 150 instructions, and every wave makes it)
    const uint64_t rel = top >> 32 ? top / frac_den : (uint64_t)((uint32_t)top / frac_den);
    return (uint32_t)min<uint64_t>(max<uint64_t>(rel, floor_t), 0xffffffffull);
}

// Steps 1-3 of the iterative finder's batch form: workgroup (event, 64-column tile) votes the
// event's hits into the rows they reach and hands the finder what it can need of the tile: the
// keys (count << 32 | ~raster index) of the cells that reach the threshold of the tile's own
// largest count -- never above that of the event's -- where they are few (at most kIterTileKeys),
// else every cell as 16-bit counts, [row][column of the tile].  Either goes to the tile's part of
// the event's accumulator in the workspace (64 n_rho cells, fewer in the last tile);
// head[event * tiles + tile] says which: the number of keys, or kIterDense, and the tile's
// largest count.  (Writing every accumulator and reading it back with one workgroup per event took
// 640 of the 668 us of 300 events on 1000 x 1000; the lists hold some 20 keys per tile there, and
// votes and finder take 138 and 64 us so.  Latency bounds the votes: half of the chip's VALU issue
// and a third of its LDS cycles; several tiles per workgroup or 12 waves gained nothing.)
// The LDS tile holds up to slab_rows rows (launch_batch_iterative chooses); hits that reach more go
// through it slab by slab, cells written.  Workgroup (e, 0) writes the event's status (invalid
// hits, too many hits, duplicate pass skipped); the finder ORs into it.  An event above
// kMaxBatchHits hits, or with malformed offsets, gets nothing.
constexpr uint32_t kIterTileKeys = 512;
constexpr uint32_t kIterDense = 0xffffffffu;

// A tile's keys start on the first 8-byte boundary of its part; room for how many.
__device__ __forceinline__ uint64_t *tile_keys(uint16_t *part) {
    return reinterpret_cast<uint64_t *>(((uintptr_t)part + 7u) & ~(uintptr_t)7u);
}
__device__ __forceinline__ uint32_t tile_key_room(int width, int n_rho) {
    const uint32_t bytes = 2u * (uint32_t)width * (uint32_t)n_rho;
    return min(bytes >= 8u ? (bytes - 6u) / 8u : 0u, kIterTileKeys);
}

// Votes of hits [hb, he) into rows [r0, r0 + rows) of a packed 64-column tile (tile row k - r0;
// any other vote to the dummy row after them).
__device__ void vote_range_rows(uint32_t *tile, const float *x, const float *y, uint32_t hb, uint32_t he,
                                const Cols<1> &cl, const GridArgs &g, int first_col, int lane, uint32_t &bad,
                                const uint8_t *dup, int r0, int rows) {
    const VoteCols<1> vc = vote_cols<1, false>(cl, g, first_col, lane);
    const f32x16 bf = bias16(g.Bf);
    for (uint32_t base = hb; base < he; base += 64) {
        const uint32_t i = base + lane;
        bool live = i < he;
        float xi = 0.0f, yi = 0.0f;
        if (live) { xi = x[i]; yi = y[i]; }
        if (dup && live && (dup[i] & kKeepDuplicate)) live = false;
        float u, v, a0, a1;
        const bool ok = conformal(live ? xi : 0.0f, live ? yi : 0.0f, u, v);
        if (live && !ok) bad = 1u;
        const float nan = __uint_as_float(0x7fc00000u);
        swap_halves(live && ok ? v : nan, live && ok ? u : nan, a0, a1);
#pragma unroll 1
        for (uint32_t b = base; b < he && b < base + 64u; b += 32u, a0 = a1) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const f32x16 t = __builtin_amdgcn_mfma_f32_32x32x2f32(a0, vc.op[h], bf, 0, 0, 0);
                if (vc.in[h]) {
#pragma unroll
                    for (int q = 0; q < 16; ++q) {
                        const float tt = t[q] + 0.0f;                         // see vote_mfma
                        const int k = __float_as_uint(tt) < __float_as_uint(g.nrho_f) ? (int)tt : -1;
                        lds_add(&tile[min((uint32_t)(k - r0), (uint32_t)rows) * 32u + (uint32_t)(lane & 31)],
                                h ? 0x10000u : 1u);
                    }
                }
            }
        }
    }
}

template <int NW>
__global__ __launch_bounds__(NW * 64) void k_vote_batch(GridArgs g, const float *__restrict__ x,
                                                        const float *__restrict__ y,
                                                        const uint32_t *__restrict__ offsets,
                                                        uint16_t *acc, const uint8_t *keep,
                                                        uint32_t *status, int slab_rows, uint32_t frac_num,
                                                        uint32_t frac_den, uint2 *head) {
    using L = Lane<1, true>;
    typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
    constexpr int NT = NW * 64;
    extern __shared__ __align__(16) uint32_t tile[];                       // [(slab_rows + 1) * 32]
    __shared__ uint32_t s_bad, s_minr2, s_lo, s_hi, s_max, s_cnt;
    const uint32_t e = blockIdx.x;
    const uint32_t h0 = offsets[e], h1 = offsets[e + 1];
    const bool ok = h1 >= h0 && h1 - h0 <= kMaxBatchHits;
    if (!ok) {
        if (blockIdx.y == 0 && threadIdx.x == 0) status[e] = HOUGH_EV_TOO_MANY_HITS;
        return;
    }
    const uint32_t H = h1 - h0;
    const int lane = threadIdx.x & 63, wave = wave_id();
    const uint8_t *dup = g.dedup ? keep + h0 : nullptr;
    x += h0;
    y += h0;
    uint32_t hb, he;
    wave_hits<NW>(H, wave, hb, he);
    const uint32_t mn = min_r2_bits(x, y, hb, he, lane);
    // (cleared while those hits are on their way)
    for (int i = threadIdx.x; i < (slab_rows + 1) * 8; i += NT)
        reinterpret_cast<uint4 *>(tile)[i] = make_uint4(0u, 0u, 0u, 0u);
    if (threadIdx.x == 0) { s_bad = 0u; s_max = 0u; s_cnt = 0u; s_minr2 = __float_as_uint(FLT_MAX); }
    __syncthreads();
    if (lane == 0) atomicMin(&s_minr2, mn);
    __syncthreads();
    if (threadIdx.x == 0) {
        int klo, khi;
        reached_rows(g, __uint_as_float(s_minr2), klo, khi);
        s_lo = (uint32_t)klo;
        s_hi = (uint32_t)khi;
    }
    __syncthreads();
    const int klo = __builtin_amdgcn_readfirstlane((int)s_lo), khi = __builtin_amdgcn_readfirstlane((int)s_hi);
    const bool one = khi - klo < slab_rows;                      // one slab holds every row the hits reach
    uint32_t bad = 0;
    const int tl = (int)blockIdx.y;
    const int first = tl * 64, width = min(64, g.n_theta - first);
    uint16_t *part = acc + ((size_t)e * (size_t)g.n_theta + (size_t)first) * (size_t)g.n_rho;
    const int vl = opaque(lane);
    const L ln(vl);
    const Cols<1> cl = load_cols<1>(g, first, vl, L::STRIDE, ln.col);
    uint32_t m = 0, thr = 0, count = kIterDense;
    for (int r0 = klo; r0 <= khi; r0 += slab_rows) {
        const int rows = min(slab_rows, khi + 1 - r0);
        if (r0 != klo) {
            for (int i = threadIdx.x; i < (rows + 1) * 8; i += NT)
                reinterpret_cast<uint4 *>(tile)[i] = make_uint4(0u, 0u, 0u, 0u);
            __syncthreads();
        }
        if (one)
            vote_range<1>(tile - (ptrdiff_t)r0 * L::STRIDE, x, y, hb, he, cl, g, first, lane, bad, (float)(r0 + rows), dup);
        else
            vote_range_rows(tile, x, y, hb, he, cl, g, first, lane, bad, dup, r0, rows);
        __syncthreads();
        const uint4 *q = reinterpret_cast<const uint4 *>(tile);
        u16x2 mm = {0, 0};
        for (int i = threadIdx.x; i < rows * 8; i += NT) {
            const uint4 v = q[i];
            mm = __builtin_elementwise_max(mm, __builtin_elementwise_max(
                __builtin_elementwise_max(__builtin_bit_cast(u16x2, v.x), __builtin_bit_cast(u16x2, v.y)),
                __builtin_elementwise_max(__builtin_bit_cast(u16x2, v.z), __builtin_bit_cast(u16x2, v.w))));
        }
        const uint32_t own = max((uint32_t)mm.x, (uint32_t)mm.y);      // the largest of this thread's cells
        m = wave_max(max(m, own));
        if (one) {
            if (lane == 0) atomicMax(&s_max, m);
            __syncthreads();
            thr = iter_threshold((uint32_t)__builtin_amdgcn_readfirstlane((int)s_max), frac_num, frac_den, g.threshold);
            // counted first, so that a tile of many is not half listed
            uint32_t n = 0;
            for (int i = threadIdx.x; own >= thr && i < rows * 8; i += NT) {
                const uint4 v = q[i];
                const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                for (int c = 0; c < 4; ++c) n += ((w[c] & 0xffffu) >= thr ? 1u : 0u) + ((w[c] >> 16) >= thr ? 1u : 0u);
            }
            const uint32_t incl = wave_inclusive_scan(n, lane);
            uint32_t off = 0;
            if (lane == 63 && incl) off = atomicAdd(&s_cnt, incl);
            off = (uint32_t)__builtin_amdgcn_readlane((int)off, 63) + incl - n;
            __syncthreads();
            const uint32_t total = s_cnt;
            if (total <= tile_key_room(width, g.n_rho)) {
                count = total;
                uint64_t *keys = tile_keys(part);
                if (n)
                    for (int i = threadIdx.x; i < rows * 8; i += NT) {
                        const uint4 v = q[i];
                        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                        for (int c = 0; c < 4; ++c) {
                            const int k = r0 + (i >> 3), col = 4 * (i & 7) + c;
#pragma unroll
                            for (int hi = 0; hi < 2; ++hi) {
                                const uint32_t cv = hi ? w[c] >> 16 : w[c] & 0xffffu;
                                if (cv >= thr) {
                                    const uint32_t r = (uint32_t)(first + col + 32 * hi) * (uint32_t)g.n_rho + (uint32_t)k;
                                    keys[off++] = ((uint64_t)cv << 32) | (uint64_t)(~r);
                                }
                            }
                        }
                    }
                break;
            }
        }
        if (lane < width)                       // every cell: a wave stores a row of the tile
            for (int k = r0 + wave; k < r0 + rows; k += NW)
                part[(size_t)k * width + lane] = (uint16_t)ln.count(tile[(k - r0) * L::STRIDE + ln.col[0]]);
        __syncthreads();
    }
    if (count == kIterDense) {                  // the rows no hit reaches
        for (int i = threadIdx.x; i < klo * width; i += NT) part[i] = 0;
        for (int i = (khi + 1) * width + (int)threadIdx.x; i < g.n_rho * width; i += NT) part[i] = 0;
    }
    if (!one && lane == 0) atomicMax(&s_max, m);
    if (bad) s_bad = 1u;
    __syncthreads();
    if (threadIdx.x == 0) {
        head[(size_t)e * gridDim.y + tl] = make_uint2(count, s_max);
        // every workgroup sees every hit of the event, so the first one's flags are the event's
        if (blockIdx.y == 0)
            status[e] = (s_bad ? HOUGH_EV_INVALID_HITS : 0u) |
                        (g.dedup && H > kDedupMaxHits ? HOUGH_EV_DEDUP_SKIPPED : 0u);
    }
}

// hough_peaks: workgroup b tests theta rows [NW*b, NW*b + NW), staged in LDS with one halo row
// on each side, one wave per row, lanes over rho.  Two launches: the first writes each block's
// peak count to counts[b]; the second lists each block's peaks at the sum of the earlier blocks'
// counts plus the earlier waves' (raster order), and block 0 writes the total.  Bound by latency: the
// loads of the rows, then the counts.  (Eight loads per thread whatever the rows needed, each with its
// 64-bit index and edge tests, made grids of many short columns slow: 4000 x 100 12.5 us, 8.2 so; 9000 x
// 100 20.6 and 14.5; 65535 x 8 137 and 76; 1000 x 1000 21.2 and 18.8.)
__device__ __forceinline__ uint32_t wave_sum(uint32_t v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += (uint32_t)__shfl_xor((int)v, o, 64);
    return v;
}

template <int NW, typename T, bool WRITE>
__global__ __launch_bounds__(NW * 64) void k_peaks(GridArgs g, const T *__restrict__ acc,
                                                   hough_peak *out, uint32_t cap,
                                                   uint32_t *n_peaks, uint32_t *counts) {
    extern __shared__ __align__(16) uint32_t lds[];
    // [NW][nm] each row's peaks, 64 cells a word; then [(NW + 2) * n_rho], buffer row r holds grid
    // row jb - 1 + r
    const int nm = (g.n_rho + 63) / 64;
    uint64_t *masks = reinterpret_cast<uint64_t *>(lds);
    uint32_t *rows = lds + 2 * NW * nm;
    __shared__ uint32_t s_cnt[NW];
    __shared__ uint32_t s_base;
    const int lane = threadIdx.x & 63, wave = wave_id();
    const int nr = g.n_rho;
    const int jb = (int)blockIdx.x * NW;
    // The rows are one run of acc but for the grid's edges (zero, or on a periodic grid the other
    // edge with rho reversed).  Up to eight loads in flight per thread, no more than the rows need.
    const int total = (NW + 2) * nr, from = jb == 0 ? nr : 0, to = min(NW + 2, g.n_theta - jb + 1) * nr;
    const T *src = acc + ((int64_t)jb - 1) * nr;
    auto stage = [&](auto width) {
        constexpr int U = decltype(width)::value;
        for (int i0 = threadIdx.x; i0 < total; i0 += U * NW * 64) {
            uint32_t v[U];
#pragma unroll
            for (int i = 0; i < U; ++i) {
                const int idx = i0 + i * NW * 64;
                v[i] = idx >= from && idx < to ? (uint32_t)src[idx] : 0u;
            }
#pragma unroll
            for (int i = 0; i < U; ++i)
                if (i0 + i * NW * 64 < total) rows[i0 + i * NW * 64] = v[i];
        }
    };
    if (total <= NW * 64) stage(std::integral_constant<int, 1>{});
    else if (total <= 2 * NW * 64) stage(std::integral_constant<int, 2>{});
    else if (total <= 4 * NW * 64) stage(std::integral_constant<int, 4>{});
    else stage(std::integral_constant<int, 8>{});
    if (g.periodic && (jb == 0 || to < total)) {
        __syncthreads();
        for (int k = threadIdx.x; k < nr; k += NW * 64) {
            if (jb == 0) rows[k] = (uint32_t)acc[(int64_t)g.n_theta * nr - 1 - k];
            if (to < total) rows[to + k] = (uint32_t)acc[nr - 1 - k];
        }
    }
    if (WRITE && wave == 0) {                     // peaks of the earlier blocks, and of all
        uint32_t before = 0, all = 0;
        for (uint32_t q = (uint32_t)lane; q < gridDim.x; q += 64) {
            const uint32_t c = counts[q];
            all += c;
            if (q < blockIdx.x) before += c;
        }
        before = wave_sum(before);
        all = wave_sum(all);
        if (lane == 0) {
            s_base = before;
            if (blockIdx.x == 0) *n_peaks = all;
        }
    }
    __syncthreads();
    const int j = jb + wave;
    const uint32_t *up = rows + wave * nr, *mid = up + nr, *dn = mid + nr;
    // on a periodic grid the row above column 0 is column n_theta - 1 (later in raster order)
    // and the row below column n_theta - 1 is column 0 (earlier)
    const bool up_later = g.periodic && j == 0, dn_earlier = g.periodic && j == g.n_theta - 1;
    auto is_peak = [&](int k) -> bool {
        const uint32_t c = mid[k];
        const uint32_t l = k > 0 ? 1u : 0u, r = k + 1 < nr ? 1u : 0u;
        const uint32_t u3 = max(max(l ? up[k - 1] : 0u, up[k]), r ? up[k + 1] : 0u);
        const uint32_t d3 = max(max(l ? dn[k - 1] : 0u, dn[k]), r ? dn[k + 1] : 0u);
        const uint32_t before = max(max(up_later ? 0u : u3, dn_earlier ? d3 : 0u), l ? mid[k - 1] : 0u);
        const uint32_t after = max(max(up_later ? u3 : 0u, dn_earlier ? 0u : d3), r ? mid[k + 1] : 0u);
        return c >= max(max(g.threshold, before + 1u), after);
    };
    uint32_t cnt = 0;
    if (j < g.n_theta) {
        for (int kc = 0; kc < nr; kc += 64) {
            const int k = kc + lane;
            const uint64_t m = __ballot(k < nr && is_peak(k));
            if (WRITE && lane == 0) masks[wave * nm + (kc >> 6)] = m;
            cnt += (uint32_t)__popcll(m);
        }
    }
    if (lane == 0) s_cnt[wave] = cnt;
    __syncthreads();
    if (!WRITE) {
        if (threadIdx.x == 0) {
            uint32_t t = 0;
            for (int w = 0; w < NW; ++w) t += s_cnt[w];
            counts[blockIdx.x] = t;
        }
        return;
    }
    uint32_t base = s_base;
    for (int w = 0; w < wave; ++w) base += s_cnt[w];
    if (j < g.n_theta) {
        for (int kc = 0; kc < nr; kc += 64) {
            const int k = kc + lane;
            const uint64_t m = masks[wave * nm + (kc >> 6)];
            if ((m >> lane) & 1ull) {
                const uint32_t idx = base + mbcnt(m);
                if (idx < cap) store_peak(out + idx, (uint32_t)j, (uint32_t)k, mid[k]);
            }
            base += (uint32_t)__popcll(m);
        }
    }
}

// hough_peaks_iterative: the paper's peak finder (relative threshold, then iterative extraction
// with neighbourhood suppression) for one event, in one workgroup of kIterWaves waves.
//
// A cell at or above the threshold is a candidate, keyed count << 32 | ~(raster index).  The
// step-by-step extraction takes the candidates in descending key order (larger count first, then
// earlier in raster order) and passes over those an earlier taken cell suppresses: suppression
// depends only on the cells already taken.  The kernel does exactly that in chunks.  A chunk is
// the next run of the sorted candidates that fits the LDS key buffer (K keys): its key range
// comes from a histogram of the remaining candidates' counts (and, when one count alone has more
// than K candidates, of their raster indices); it is gathered, sorted (bitonic, descending) and
// walked in order by wave 0, 64 keys at a time, against a suppression bitmap of the whole grid
// (one bit per cell, raster-indexed, set for every cell within r_theta columns and r_rho rows of
// a taken cell).  Candidates the bitmap covers are left out of later chunks.  The bitmap lives in
// LDS after the keys when it fits (GBM false), else in device memory (GBM true).
constexpr int kIterWaves = 16;
constexpr uint32_t kIterThreads = kIterWaves * 64;
constexpr uint32_t kIterMaxKeys = 16384;     // 128 KB of LDS
constexpr uint32_t kIterMinKeys = 1024;

// The suppression bitmap: every access comes from the event's own workgroup, so workgroup-scope
// atomics order the marks of wave 0 against the later reads of every wave (LDS or device memory).
__device__ __forceinline__ bool bm_test(const uint32_t *bm, uint32_t r) {
    const uint32_t w = __hip_atomic_load(bm + (r >> 5), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    return (w >> (r & 31)) & 1u;
}

// Set the bits of every cell within r_theta columns and r_rho rows of (jf, kf), clipped at the
// grid edges: per column one raster run jj * n_rho + [k0, k1], a few words each; four lanes take
// the words of a column, 16 columns at a time.
__device__ void mark_window(uint32_t *bm, int jf, int kf, int r_theta, int r_rho, int n_theta, int n_rho,
                            uint32_t lane) {
    const int j0 = max(jf - r_theta, 0), j1 = min(jf + r_theta, n_theta - 1);
    const int k0 = max(kf - r_rho, 0), k1 = min(kf + r_rho, n_rho - 1);
    for (int col = j0 + (int)(lane >> 2); col <= j1; col += 16) {
        const uint32_t a = (uint32_t)col * (uint32_t)n_rho + (uint32_t)k0, e = a + (uint32_t)(k1 - k0);
        for (uint32_t w = (a >> 5) + (lane & 3u); w <= (e >> 5); w += 4u) {
            const uint32_t lo = w == (a >> 5) ? (a & 31u) : 0u, hi = w == (e >> 5) ? (e & 31u) : 31u;
            const uint32_t bits = (hi == 31u ? ~0u : ((1u << (hi + 1u)) - 1u)) & ~((1u << lo) - 1u);
            __hip_atomic_fetch_or(bm + w, bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
    }
}

// Every cell of an accumulator of `cells` cells, eight loads in flight per lane: f(c, v, in) for
// storage index c, count v, and in = c < cells.  Every lane calls f the same number of times per
// wave, so f may use wave-wide operations.
template <typename T, typename F>
__device__ __forceinline__ void for_cells(const T *acc, uint32_t cells, F &&f) {
    constexpr int U = 8;
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (uint32_t base = wave * 64u; base < cells; base += U * kIterThreads) {
        uint32_t v[U];
#pragma unroll
        for (int r = 0; r < U; ++r) {
            const uint32_t c = base + (uint32_t)r * kIterThreads + lane;
            v[r] = c < cells ? (uint32_t)acc[c] : 0u;
        }
#pragma unroll
        for (int r = 0; r < U; ++r) {
            const uint32_t c = base + (uint32_t)r * kIterThreads + lane;
            f(c, v[r], c < cells);
        }
    }
}

// Append `key` for the lanes where p holds, at positions taken from the LDS counter *cnt (one
// atomic per wave); positions at or past `room` are counted but not stored.
__device__ __forceinline__ void append_key(uint64_t *keys, uint32_t *cnt, uint32_t room, bool p, uint64_t key,
                                           uint32_t lane) {
    const uint64_t b = __ballot(p);
    if (!b) return;
    uint32_t off = 0;
    if (lane == 0) off = atomicAdd(cnt, (uint32_t)__popcll(b));
    off = (uint32_t)__shfl((int)off, 0, 64);
    const uint32_t pos = off + mbcnt(b);
    if (p && pos < room) keys[pos] = key;
}

// Wave 0 reads hist[0 .. nb) in processing order (from bin nb - 1 down when `top`, else from bin
// 0 up) and returns, through *m, the number of leading bins whose counts sum to at most `room`
// and, through *first, the position of the first non-empty bin (nb when all are empty).  nb is a
// multiple of 64.
__device__ void hist_fit(const uint32_t *hist, uint32_t nb, bool top, uint32_t room, uint32_t lane, uint32_t *m,
                         uint32_t *first) {
    const uint32_t per = nb / 64u, q0 = lane * per;
    uint32_t s = 0, f = nb;
    for (uint32_t q = q0; q < q0 + per; ++q) {
        const uint32_t h = hist[top ? nb - 1u - q : q];
        if (h && f == nb) f = q;
        s += h;
    }
    const uint32_t incl = wave_inclusive_scan(s, (int)lane);
    const uint64_t over = __ballot(incl > room);
    uint32_t mm = nb;
    if (over) {
        const uint32_t cl = (uint32_t)__builtin_ctzll(over);
        if (lane == cl) {
            uint32_t run = incl - s;
            for (uint32_t q = q0; q < q0 + per; ++q) {
                run += hist[top ? nb - 1u - q : q];
                if (run > room) { mm = q; break; }
            }
        }
        mm = (uint32_t)__builtin_amdgcn_readlane((int)mm, (int)cl);
    }
    *m = mm;
    *first = wave_min(f);
}

// One event's accumulator read by the whole chip ahead of the finder (one workgroup reading 4 MB
// took 125 of the finder's 144 us on 1000 x 1000; this pass takes 7 and the finder 20 after it): the largest count in scan[0], and in list
// the keys of every cell that reaches the threshold (their number in scan[1]; more than kIterScanCap:
// only counted).  Each block holds its cells in registers, raises the running maximum by its own
// and lists the cells that reach the threshold of the maximum so far: that never exceeds the
// final one, so the list holds every candidate and some cells more, which the finder drops.
// The finder puts scan[0] and scan[1] back to zero.
constexpr int kScanThreads = 256, kScanCells = 16;
constexpr uint32_t kIterScanCap = kIterScanKeys;

template <typename T>
__global__ __launch_bounds__(kScanThreads) void k_iter_scan(const T *__restrict__ acc, uint32_t cells,
                                                            uint32_t floor_t, uint32_t frac_num, uint32_t frac_den,
                                                            uint64_t *__restrict__ list, uint32_t *scan) {
    __shared__ uint32_t s_max, s_cnt, s_base, s_thr;
    const uint32_t lane = threadIdx.x & 63;
    constexpr uint32_t kTile = kScanThreads * kScanCells;
    for (uint64_t b = (uint64_t)blockIdx.x * kTile; b < cells; b += (uint64_t)gridDim.x * kTile) {
        const uint32_t base = (uint32_t)b;
        if (threadIdx.x == 0) { s_max = 0u; s_cnt = 0u; }
        __syncthreads();
        uint32_t v[kScanCells], m = 0;
#pragma unroll
        for (int i = 0; i < kScanCells; ++i) {
            const uint64_t c = b + (uint64_t)(i * kScanThreads) + threadIdx.x;
            v[i] = c < cells ? (uint32_t)acc[c] : 0u;
            m = max(m, v[i]);
        }
        m = wave_max(m);
        if (lane == 0) atomicMax(&s_max, m);
        __syncthreads();
        if (threadIdx.x == 0) s_thr = iter_threshold(max(atomicMax(scan, s_max), s_max), frac_num, frac_den, floor_t);
        __syncthreads();
        const uint32_t thr = s_thr;
        uint32_t n = 0;
#pragma unroll
        for (int i = 0; i < kScanCells; ++i) n += v[i] >= thr ? 1u : 0u;
        const uint32_t incl = wave_inclusive_scan(n, (int)lane);
        uint32_t off = 0;
        if (lane == 63 && incl) off = atomicAdd(&s_cnt, incl);
        off = (uint32_t)__builtin_amdgcn_readlane((int)off, 63) + incl - n;
        __syncthreads();
        if (threadIdx.x == 0 && s_cnt) s_base = atomicAdd(scan + 1, s_cnt);
        __syncthreads();
        uint32_t pos = s_base + off;
#pragma unroll
        for (int i = 0; i < kScanCells; ++i)
            if (v[i] >= thr) {
                const uint32_t r = base + (uint32_t)(i * kScanThreads) + threadIdx.x;
                if (pos < kIterScanCap) list[pos] = ((uint64_t)v[i] << 32) | (uint64_t)(~r);
                ++pos;
            }
        __syncthreads();
    }
}

// BATCH (offsets given): workgroup e takes what k_vote_batch left of event e at acc + e * cells and
// head + e * tiles, writes its list at out + e * cap, n_peaks[e], and ORs
// HOUGH_EV_PEAKS_TRUNCATED into status[e] (which the batch vote wrote); events the vote skipped
// get no peaks.  K: keys in the LDS buffer (a power of two, kIterMinKeys .. kIterMaxKeys).
// gbm (GBM): device bitmaps of bm_words words, one per workgroup.
// list, scan (LIST: one event of more than kIterDirectCells cells): what k_iter_scan left.
template <typename T, bool GBM, bool BATCH, bool LIST>
__global__ __launch_bounds__(kIterThreads) void k_peaks_iter(GridArgs g, const T *__restrict__ acc,
                                                             uint32_t frac_num, uint32_t frac_den, int r_theta,
                                                             int r_rho, hough_peak *out, uint32_t cap,
                                                             uint32_t *n_peaks, uint32_t *status,
                                                             const uint32_t *offsets, uint32_t K, uint32_t *gbm,
                                                             const uint64_t *list, uint32_t *scan,
                                                             const uint2 *head) {
    extern __shared__ __align__(16) uint64_t keys[];       // [K]; the histograms reuse it as 2K words
    uint32_t *hist = reinterpret_cast<uint32_t *>(keys);
    __shared__ uint32_t s_red[kIterWaves];
    __shared__ uint32_t s_n, s_m, s_first, s_taken;
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t nr = (uint32_t)g.n_rho, nt = (uint32_t)g.n_theta;
    const uint32_t cells = nt * nr, bm_words = (cells + 31u) / 32u, NB = 2u * K;
    const uint32_t tiles = (nt + 63u) / 64u;
    // (batch) first listed key of each tile, [tiles + 1] after the keys and an LDS bitmap
    uint32_t *s_tile = reinterpret_cast<uint32_t *>(keys + K) + (GBM ? 0u : (bm_words + 3u) & ~3u);
    if constexpr (BATCH) {
        const uint32_t e = blockIdx.x;
        acc += (size_t)e * cells;
        out = out ? out + (size_t)e * cap : nullptr;
        n_peaks += e;
        status += e;
        const uint32_t h0 = offsets[e], h1 = offsets[e + 1];
        if (h1 < h0 || h1 - h0 > kMaxBatchHits) {              // no accumulator was written
            if (tid == 0) *n_peaks = 0u;
            return;
        }
        head += (size_t)e * tiles;
    }
    uint32_t *bm = GBM ? gbm + (BATCH ? (size_t)blockIdx.x * bm_words : (size_t)0)
                       : reinterpret_cast<uint32_t *>(keys + K);
    if constexpr (!GBM) {
        // (whole quads: the LDS bitmap ends on a 16-byte boundary)
        for (uint32_t w = tid; w < (bm_words + 3u) / 4u; w += kIterThreads)
            reinterpret_cast<uint4 *>(bm)[w] = make_uint4(0u, 0u, 0u, 0u);
    } else {
        for (uint32_t w = tid; w < bm_words; w += kIterThreads) bm[w] = 0u;
    }
    if (tid == 0) { s_n = 0u; s_taken = 0u; }
    __syncthreads();

    // every cell that can be a candidate, as f(count, raster index, valid), all lanes of a wave
    // together: the accumulator's cells; of a batch event the listed keys of its tiles and the
    // cells of those that list none
    auto each = [&](auto &&f) {
        if constexpr (!BATCH) {
            for_cells(acc, cells, [&](uint32_t c, uint32_t v, bool in) { f(v, c, in); });
        } else {
            const uint32_t listed = s_tile[tiles];
            for (uint32_t i0 = 0; i0 < listed; i0 += kIterThreads) {
                const uint32_t i = i0 + tid;
                uint64_t key = 0;
                if (i < listed) {
                    uint32_t lo = 0, hi = tiles - 1u;             // the last tile whose keys start at or before i
                    while (lo < hi) {
                        const uint32_t mid = (lo + hi + 1u) >> 1;
                        if (s_tile[mid] <= i) lo = mid; else hi = mid - 1u;
                    }
                    key = tile_keys(const_cast<uint16_t *>(acc) + (size_t)lo * 64u * nr)[i - s_tile[lo]];
                }
                f((uint32_t)(key >> 32), ~(uint32_t)key, i < listed);
            }
            for (uint32_t t = 0; t < tiles; ++t) {
                if (head[t].x != kIterDense) continue;
                const uint32_t w = min(64u, nt - 64u * t);
                for_cells(acc + (size_t)t * 64u * nr, w * nr, [&](uint32_t c, uint32_t v, bool in) {
                    const uint32_t k = c / w;
                    f(v, (64u * t + (c - k * w)) * nr + k, in);
                });
            }
        }
    };
    const uint32_t floor_t = g.threshold;
    uint32_t mx = 0, thr, n1;
    bool filtered = true;      // the keys held reach thr (else the floor)
    if constexpr (BATCH) {
        // the tiles' heads: the event's largest count, and where each tile's keys start
        uint32_t m = 0, run = 0;
        for (uint32_t t0 = 0; t0 < tiles; t0 += 64u) {            // every wave the same
            const uint32_t t = t0 + lane;
            const uint2 hd = t < tiles ? head[t] : make_uint2(0u, 0u);
            const uint32_t n = hd.x == kIterDense ? 0u : hd.x, incl = wave_inclusive_scan(n, (int)lane);
            if (wave == 0 && t < tiles) s_tile[t] = run + incl - n;
            run += (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
            m = max(m, hd.y);
        }
        if (tid == 0) s_tile[tiles] = run;
        mx = wave_max(m);
        thr = iter_threshold(mx, frac_num, frac_den, floor_t);
        __syncthreads();
        each([&](uint32_t v, uint32_t r, bool in) {
            append_key(keys, &s_n, K, in && v >= thr, ((uint64_t)v << 32) | (uint64_t)(~r), lane);
        });
        __syncthreads();
        n1 = s_n;
    } else if constexpr (LIST) {
        mx = scan[0];
        n1 = scan[1];
        thr = iter_threshold(mx, frac_num, frac_den, floor_t);
        const bool whole = n1 <= kIterScanCap;
        if (whole)
            for (uint32_t i0 = 0; i0 < n1; i0 += kIterThreads) {
                const uint32_t i = i0 + tid;
                const uint64_t key = i < n1 ? list[i] : 0ull;
                append_key(keys, &s_n, K, i < n1 && (uint32_t)(key >> 32) >= thr, key, lane);
            }
        __syncthreads();
        n1 = whole ? s_n : K + 1u;
    } else {
        // the maximum, and the candidates of the absolute floor while they fit
        uint32_t m = 0;
        each([&](uint32_t v, uint32_t r, bool in) {
            m = max(m, v);
            append_key(keys, &s_n, K, in && v >= floor_t, ((uint64_t)v << 32) | (uint64_t)(~r), lane);
        });
        m = wave_max(m);
        if (lane == 0) s_red[wave] = m;
        __syncthreads();
        for (int w = 0; w < kIterWaves; ++w) mx = max(mx, s_red[w]);
        thr = iter_threshold(mx, frac_num, frac_den, floor_t);
        n1 = s_n;
        filtered = thr == floor_t;
    }
    __syncthreads();

    bool bounded = false;      // keys below `hi` are what is left once a chunk has been walked
    uint64_t hi = 0;
    bool have_chunk = false;
    uint32_t n = 0;
    uint64_t lo = 0;           // the chunk's lowest key (0: the chunk holds every candidate left)
    if (n1 <= K) {                       // every candidate is in LDS: those that reach thr, in place
        if (!filtered) {
            if (tid == 0) s_n = 0u;
            __syncthreads();
            for (uint32_t i0 = 0; i0 < n1; i0 += kIterThreads) {
                const uint32_t i = i0 + tid;
                const uint64_t key = i < n1 ? keys[i] : 0ull;
                __syncthreads();
                append_key(keys, &s_n, K, i < n1 && (uint32_t)(key >> 32) >= thr, key, lane);
                __syncthreads();
            }
        }
        n = s_n;
        have_chunk = true;
    }
    for (;;) {
        if (!have_chunk) {
            // the next chunk: the largest remaining keys whose number fits K
            uint32_t vlo = thr, vhi = bounded ? (uint32_t)(hi >> 32) : mx;
            bool none = vhi < vlo;
            while (!none) {
                const uint32_t w = (uint32_t)(((uint64_t)vhi - vlo + 1u + NB - 1u) / NB);
                for (uint32_t b = tid; b < NB; b += kIterThreads) hist[b] = 0u;
                __syncthreads();
                each([&](uint32_t v, uint32_t r, bool in) {
                    if (!in || v < vlo || v > vhi) return;
                    const uint64_t key = ((uint64_t)v << 32) | (uint64_t)(~r);
                    if ((bounded && key >= hi) || bm_test(bm, r)) return;
                    atomicAdd(&hist[(v - vlo) / w], 1u);
                });
                __syncthreads();
                if (wave == 0) hist_fit(hist, NB, true, K, lane, &s_m, &s_first);
                __syncthreads();
                const uint32_t mb = s_m, fb = s_first;
                __syncthreads();
                if (fb == NB) { none = true; break; }                   // nothing left
                if (mb > fb) {                                          // bins NB - mb .. NB - 1 fit
                    lo = (uint64_t)(vlo + (NB - mb) * w) << 32;
                    break;
                }
                const uint32_t bt = NB - 1u - fb;                       // the top non-empty bin, too full
                if (w > 1u) {
                    vhi = (uint32_t)min<uint64_t>((uint64_t)vhi, (uint64_t)vlo + (uint64_t)bt * w + w - 1u);
                    vlo = vlo + bt * w;
                    continue;
                }
                // one count vt has more than K candidates left: split them by raster index
                const uint32_t vt = vlo + bt;
                uint32_t rlo = (bounded && vt == (uint32_t)(hi >> 32)) ? ~(uint32_t)hi + 1u : 0u, rhi = cells - 1u;
                for (;;) {
                    const uint32_t wr = (uint32_t)(((uint64_t)rhi - rlo + 1u + NB - 1u) / NB);
                    for (uint32_t b = tid; b < NB; b += kIterThreads) hist[b] = 0u;
                    __syncthreads();
                    each([&](uint32_t v, uint32_t r, bool in) {
                        if (!in || v != vt) return;
                        if (r < rlo || r > rhi || bm_test(bm, r)) return;
                        atomicAdd(&hist[(r - rlo) / wr], 1u);
                    });
                    __syncthreads();
                    if (wave == 0) hist_fit(hist, NB, false, K, lane, &s_m, &s_first);
                    __syncthreads();
                    const uint32_t mr = s_m, fr = s_first;
                    __syncthreads();
                    if (mr > fr) {                                      // raster bins 0 .. mr - 1 fit
                        const uint32_t r_end = (uint32_t)min<uint64_t>((uint64_t)rhi, (uint64_t)rlo + (uint64_t)mr * wr - 1u);
                        lo = ((uint64_t)vt << 32) | (uint64_t)(~r_end);
                        break;
                    }
                    rhi = (uint32_t)min<uint64_t>((uint64_t)rhi, (uint64_t)rlo + (uint64_t)fr * wr + wr - 1u);
                    rlo = rlo + fr * wr;
                }
                break;
            }
            if (none) break;
            if (lo == ((uint64_t)thr << 32)) lo = 0;                    // every count down to thr
            // gather the chunk: the remaining keys in [lo, hi)
            if (tid == 0) s_n = 0u;
            __syncthreads();
            each([&](uint32_t v, uint32_t r, bool in) {
                bool p = in && v >= thr;
                uint64_t key = 0;
                if (p) {
                    key = ((uint64_t)v << 32) | (uint64_t)(~r);
                    p = key >= lo && (!bounded || key < hi) && !bm_test(bm, r);
                }
                append_key(keys, &s_n, K, p, key, lane);
            });
            __syncthreads();
            n = s_n;
        }
        have_chunk = false;
        // bitonic sort, descending, over the next power of two (n <= K)
        uint32_t P = 1;
        while (P < n) P <<= 1;
        for (uint32_t i = n + tid; i < P; i += kIterThreads) keys[i] = 0ull;
        __syncthreads();
        if (P <= kIterThreads) {
            // a key per thread: partners less than a wave apart trade through the wave's lanes,
            // so that only the others need LDS and barriers (10 of 55 steps at 1,024 keys)
            uint64_t key = tid < P ? keys[tid] : 0ull;
            for (uint32_t k = 2; k <= P; k <<= 1) {
                for (uint32_t j = k >> 1; j > 0; j >>= 1) {
                    uint64_t other;
                    if (j >= 64u) {
                        if (tid < P) keys[tid] = key;
                        __syncthreads();
                        other = tid < P ? keys[tid ^ j] : 0ull;
                        __syncthreads();
                    } else {
                        const uint32_t hi32 = (uint32_t)__shfl_xor((int)(uint32_t)(key >> 32), (int)j, 64);
                        other = ((uint64_t)hi32 << 32) | (uint32_t)__shfl_xor((int)(uint32_t)key, (int)j, 64);
                    }
                    const bool larger = ((tid & k) == 0u) == ((tid & j) == 0u);       // this place takes the larger
                    key = (key > other) == larger ? key : other;
                }
            }
            if (tid < P) keys[tid] = key;
            __syncthreads();
        } else
        for (uint32_t k = 2; k <= P; k <<= 1) {
            for (uint32_t j = k >> 1; j > 0; j >>= 1) {
                for (uint32_t i = tid; i < P; i += kIterThreads) {
                    const uint32_t ixj = i ^ j;
                    if (ixj > i) {
                        const uint64_t a = keys[i], b = keys[ixj];
                        const bool desc = (i & k) == 0u;
                        if (desc ? (a < b) : (a > b)) { keys[i] = b; keys[ixj] = a; }
                    }
                }
                __syncthreads();
            }
        }
        // the walk (wave 0): a key the bitmap covers is passed over; within a group of 64 the
        // first live key is taken and suppresses the later ones in its window; the group's taken
        // cells then mark their windows for the keys after them
        if (wave == 0) {
            uint32_t taken = s_taken;
            for (uint32_t base = 0; base < n; base += 64) {
                const uint32_t i = base + lane;
                bool live = i < n;
                const uint64_t key = live ? keys[i] : 0ull;
                const uint32_t r = ~(uint32_t)key, v = (uint32_t)(key >> 32);
                const int j = live ? (int)(r / nr) : 0, k = live ? (int)(r - (uint32_t)j * nr) : 0;
                live = live && !bm_test(bm, r);
                uint64_t b = __ballot(live), took = 0;
                while (b) {
                    const int f = __builtin_ctzll(b);
                    const int jf = __builtin_amdgcn_readlane(j, f), kf = __builtin_amdgcn_readlane(k, f);
                    const uint32_t vf = (uint32_t)__builtin_amdgcn_readlane((int)v, f);
                    if (lane == 0 && taken < cap) store_peak(out + taken, (uint32_t)jf, (uint32_t)kf, vf);
                    ++taken;
                    took |= 1ull << f;
                    live = live && (int)lane != f && !(abs(j - jf) <= r_theta && abs(k - kf) <= r_rho);
                    b = __ballot(live);
                }
                if (base + 64u >= n && lo == 0) break;              // no key is left to suppress
                while (took) {
                    const int f = __builtin_ctzll(took);
                    took &= took - 1ull;
                    mark_window(bm, __builtin_amdgcn_readlane(j, f), __builtin_amdgcn_readlane(k, f), r_theta,
                                r_rho, (int)nt, (int)nr, lane);
                }
                wave_sync();
            }
            if (lane == 0) s_taken = taken;
        }
        __syncthreads();
        if (lo == 0) break;                       // the chunk reached the lowest candidate
        bounded = true;
        hi = lo;
    }
    if (tid == 0) {
        const uint32_t taken = s_taken;
        *n_peaks = taken;
        const uint32_t tr = taken > cap ? HOUGH_EV_PEAKS_TRUNCATED : 0u;
        *status = BATCH ? (*status | tr) : tr;
        if constexpr (LIST) { scan[0] = 0u; scan[1] = 0u; }
    }
}

// hough_track_params: one workgroup of kTrackWaves waves per peak.  The waves sweep the event's hits
// 64 at a time (the next 64 load meanwhile) and count, with ballots, the hits the retention rule
// associates with the peak and how many of them lie on either side of the line from the origin
// through the circle's centre; thread 0 adds the waves' counts, turns the peak into the circle
// (double precision) and writes the record.  (65 peaks over 1,500 hits: 11 us with a wave per
// peak, its 24 chunks one after the other, and 5 us so.)
constexpr int kTrackWaves = 4;

__global__ __launch_bounds__(kTrackWaves * 64) void k_track_params(GridArgs g, const float *__restrict__ x,
                                                                   const float *__restrict__ y,
                                                                   uint32_t n_hits, const hough_peak *peaks,
                                                                   const uint32_t *n_peaks, uint32_t cap,
                                                                   double rho_min, double rho_max,
                                                                   double b_tesla, hough_track *out) {
    __shared__ uint32_t s_cnt[kTrackWaves][3];
    const int lane = threadIdx.x & 63, wave = wave_id();
    const uint32_t np = min(*n_peaks, cap);
    for (uint32_t p = blockIdx.x; p < np; p += gridDim.x) {
        const uint2 rec = reinterpret_cast<const uint2 *>(peaks)[p];
        const int j = (int)(rec.x & 0xffffu), k = (int)(rec.x >> 16);
        const bool in_grid = j < g.n_theta && k < g.n_rho;
        const float Cj = in_grid ? g.C[j] : 0.0f, Sj = in_grid ? g.S[j] : 0.0f;
        const double drho = (rho_max - rho_min) / (double)g.n_rho;
        const double rho = rho_min + ((double)k + 0.5) * drho;
        uint32_t n = 0, ccw = 0, cw = 0;
        if (in_grid) {
            uint32_t i = threadIdx.x;
            float xn = 0.0f, yn = 0.0f;
            if (i < n_hits) { xn = x[i]; yn = y[i]; }
            for (uint32_t base = (uint32_t)wave * 64u; base < n_hits; base += kTrackWaves * 64u) {
                const float xi = xn, yi = yn;
                const bool live = i < n_hits;
                i += kTrackWaves * 64u;
                if (i < n_hits) { xn = x[i]; yn = y[i]; }
                float u, v;
                const bool ok = conformal(live ? xi : 0.0f, live ? yi : 0.0f, u, v) && live;
                const float w = __builtin_fmaf(v, Sj, g.Bf);
                const float t = __builtin_fmaf(u, Cj, w);
                const bool in = ok && t >= 0.0f && t < g.nrho_f;
                const int d = in ? abs((int)t - k) : 0;
                const bool mine = in && d <= g.rho_window;
                float side = __builtin_fmaf(Cj, yi, -(Sj * xi));
                if (rho < 0.0) side = -side;
                n += (uint32_t)__popcll(__ballot(mine));
                ccw += (uint32_t)__popcll(__ballot(mine && side > 0.0f));
                cw += (uint32_t)__popcll(__ballot(mine && side < 0.0f));
            }
        }
        if (lane == 0) { s_cnt[wave][0] = n; s_cnt[wave][1] = ccw; s_cnt[wave][2] = cw; }
        __syncthreads();
        if (threadIdx.x == 0) {
            for (int w = 1; w < kTrackWaves; ++w) { n += s_cnt[w][0]; ccw += s_cnt[w][1]; cw += s_cnt[w][2]; }
            const double pi = 3.14159265358979323846;
            const double theta = ((double)j * pi) / (double)g.n_theta;
            hough_track tr;
            tr.a = cos(theta) / (2.0 * rho);
            tr.b = sin(theta) / (2.0 * rho);
            tr.radius = 1.0 / (2.0 * fabs(rho));
            tr.pt = 0.299792458 * b_tesla * tr.radius * 1e-3;
            tr.phi_c = atan2(tr.b, tr.a);
            tr.charge = ccw > cw ? 1 : (ccw < cw ? -1 : 0);
            tr.n_hits = n;
            out[p] = tr;
        }
        __syncthreads();
    }
}

// hough_retain: 64 hits at a time, one per lane of each wave that works on them.
//   - Up to kRetainList peaks: they are staged once per workgroup with their columns' constants
//     (as the fused kernel's peak list) and every lane tests its own hit against them.
//   - More: the dilated peak bits (bit k of column j set iff a peak (j, k') has |k - k'| <= W) of
//     a block of columns that fits LDS are built from the list, [column][word] with an odd number
//     of words per column (different words of a column lie in different banks) and a zero one
//     after its last, beside the columns' constants, and every lane looks its own bin up in one
//     column after the other, until all 64 hits are kept.
// SHARE of the workgroup's 16 waves share each 64 hits, a part of the peaks or the columns each.  A few
// hits leave most of the chip idle otherwise; the more hits there are the fewer waves share them, down
// to one, which stops at the column that keeps the last of its hits (see launch_retain).
// A batch (offsets given, SHARE 1): workgroup
// (e, b) takes event e's chunks b * 16 + wave, + 16 * gridDim.y, ..., each wave a chunk; event
// e's peaks are at peaks + e * cap, n_peaks[e]; the keep bytes of an event the vote skipped for
// its size are zeroed (malformed offsets: nothing is touched).
// (one event of 4,400 hits and 14,000 peaks, 720 x 512: 50 us with 512 hits per workgroup looked
// up with lane = column, 16 us so; 1,500 hits and 65 peaks: 46 and 4 us; 300 events of 1,500 hits
// on 1000 x 1000: 140 us with 64 workgroups per event, most of them empty, and 21 us so)
constexpr int kRetainWaves = 16;
constexpr uint32_t kRetainList = 1024;
__host__ __device__ constexpr uint32_t retain_pitch(int n_rho) { return ((uint32_t)(n_rho + 31) / 32u + 1u) | 1u; }

// The hit's own bin in n columns (their constants at cs, their dilated bits at dil).  CHECK: the
// literal range test.  Returns the kept lanes of `want`.
template <bool CHECK>
__device__ __forceinline__ uint64_t kept_in_columns(const uint32_t *dil, const float2 *cs, uint32_t pitch, float u,
                                                    float v, uint64_t want, int n, const GridArgs &g) {
    const uint32_t zero_row = ((uint32_t)g.n_rho + 31u) & ~31u;
    uint32_t m = 0;
    uint64_t kept = 0;
    // rounds of 8 columns, evenly spaced: neighbouring columns mostly keep the same hits
    const int rounds = (n + 7) / 8;
    for (int r = 0; r < rounds; ++r) {
        uint32_t word[8], k[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int jj = min(r + i * rounds, n - 1);
            const float2 c = cs[jj];
            const float t = __builtin_fmaf(u, c.x, __builtin_fmaf(v, c.y, g.Bf));
            // a bin outside the grid looks at the column's zero word
            k[i] = !CHECK || (t >= 0.0f && t < g.nrho_f) ? (uint32_t)(int)t : zero_row;
            word[i] = dil[(uint32_t)jj * pitch + (k[i] >> 5)];
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) m |= word[i] >> (k[i] & 31u);
        kept = __ballot((m & 1u) != 0u) & want;
        if (kept == want) break;
    }
    return kept;
}

template <int SHARE>
__global__ __launch_bounds__(kRetainWaves * 64) void k_retain(GridArgs g, const float *__restrict__ x,
                                                              const float *__restrict__ y, uint32_t n_hits,
                                                              const hough_peak *__restrict__ peaks,
                                                              const uint32_t *n_peaks, uint32_t cap,
                                                              uint8_t *keep, int cols_per_block,
                                                              const uint32_t *offsets) {
    constexpr int NT = kRetainWaves * 64;
    constexpr uint32_t PER = kRetainWaves / SHARE;             // chunks of 64 hits a workgroup takes at a time
    // the block's columns: constants [cols_per_block], dilated bits [cols_per_block][pitch]
    extern __shared__ __align__(16) float2 cs[];
    uint32_t *dil = reinterpret_cast<uint32_t *>(cs + cols_per_block);
    __shared__ float4 list[kRetainList];
    __shared__ uint64_t s_kept[kRetainWaves];
    __shared__ uint32_t s_edge;
    const int lane = threadIdx.x & 63, wave = wave_id();
    if (SHARE == 1 && offsets) {
        const uint32_t e = blockIdx.x, h0 = offsets[e], h1 = offsets[e + 1];
        if (h1 < h0) return;
        if (h1 - h0 > kMaxBatchHits) {
            for (uint32_t i = h0 + blockIdx.y * NT + threadIdx.x; i < h1; i += gridDim.y * NT) keep[i] = 0u;
            return;
        }
        n_hits = h1 - h0;
        if (blockIdx.y * NT >= n_hits) return;
        x += h0;
        y += h0;
        keep += h0;
        peaks += (size_t)e * cap;
        n_peaks += e;
    }
    // the workgroup's chunks of 64 hits, this wave's among them, and its part of the work on it
    const uint32_t chunks = n_hits / 64u + (n_hits % 64u != 0u);
    const uint32_t first = blockIdx.y * PER, step = gridDim.y * PER, mine = (uint32_t)(wave / SHARE);
    const int part = wave % SHARE;
    const uint32_t np = min(*n_peaks, cap);
    const uint2 *pk = reinterpret_cast<const uint2 *>(peaks);
    const bool listed = np <= kRetainList;
    const uint32_t pitch = retain_pitch(g.n_rho);
    const int W = g.rho_window;
    if (threadIdx.x == 0) s_edge = 0u;
    // the first hits, on their way while the peaks are laid out
    float x0 = 0.0f, y0 = 0.0f;
    if (SHARE > 1 && (first + mine) * 64u + (uint32_t)lane < n_hits) {
        x0 = x[(first + mine) * 64u + lane];
        y0 = y[(first + mine) * 64u + lane];
    }
    __syncthreads();
    for (int ja = 0; ja < (listed ? 1 : g.n_theta); ja += cols_per_block) {
        const int jn = min(cols_per_block, g.n_theta - ja);
        if (listed) {
            for (uint32_t p = threadIdx.x; p < np; p += NT) {
                const uint2 r = pk[p];
                const int j = (int)(r.x & 0xffffu), k = (int)(r.x >> 16);
                const bool in = j < g.n_theta && k < g.n_rho;           // a cell outside the grid keeps nothing
                list[p] = make_float4(in ? g.C[j] : 0.0f, in ? g.S[j] : 0.0f,
                                      __int_as_float(in ? k - W : (int)0x80000000), 0.0f);
                if (in && (k <= W || k >= g.n_rho - W)) s_edge = 1u;
            }
        } else {
            if (ja) __syncthreads();                                    // the last block is still being read
            for (int t = threadIdx.x; t < jn; t += NT) cs[t] = make_float2(g.C[ja + t], g.S[ja + t]);
            for (uint32_t t = threadIdx.x; t < (uint32_t)jn * pitch; t += NT) dil[t] = 0u;
            __syncthreads();
            constexpr int U = 8;                                        // cells in flight per thread
            for (uint32_t p0 = threadIdx.x; p0 < np; p0 += U * NT) {
                uint32_t cell[U];
#pragma unroll
                for (int i = 0; i < U; ++i) cell[i] = p0 + i * NT < np ? pk[p0 + i * NT].x : 0xffffffffu;
#pragma unroll
                for (int i = 0; i < U; ++i) {
                    const int j = (int)(cell[i] & 0xffffu), k = (int)(cell[i] >> 16);
                    if (j < ja || j >= ja + jn || k >= g.n_rho) continue;
                    const int lo = max(k - W, 0), hi = min(k + W, g.n_rho - 1);
                    uint32_t *col = dil + (uint32_t)(j - ja) * pitch;
                    for (int wd = lo >> 5; wd <= (hi >> 5); ++wd) {
                        const int a = max(lo, wd * 32) - wd * 32, b = min(hi, wd * 32 + 31) - wd * 32;
                        const uint32_t m = (b == 31 ? 0xffffffffu : ((1u << (b + 1)) - 1u)) & ~((1u << a) - 1u);
                        __hip_atomic_fetch_or(&col[wd], m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    }
                }
            }
        }
        __syncthreads();
        const bool edge = s_edge != 0u;
        const uint32_t p0 = np * (uint32_t)part / SHARE, p1 = np * (uint32_t)(part + 1) / SHARE;
        const int c0 = jn * part / SHARE, c1 = jn * (part + 1) / SHARE;
        // (every wave goes round as often as the others, so the barriers below are uniform)
        for (uint32_t cb = first; cb < chunks; cb += step) {
            const uint32_t i = (cb + mine) * 64u + (uint32_t)lane;
            const bool in = cb + mine < chunks && i < n_hits;
            float xi = x0, yi = y0;
            if (!(SHARE > 1 && cb == first)) {
                xi = yi = 0.0f;
                if (in) { xi = x[i]; yi = y[i]; }
            }
            float u, v;
            const bool valid = conformal(xi, yi, u, v) && in;
            const uint64_t want = __ballot(valid);
            uint64_t kept = 0;
            if (listed) {
                if (p1 > p0) kept = kept_by_peaks(list + p0, p1 - p0, valid ? u : 0.0f, valid ? v : 0.0f, valid, edge, g);
            } else if (c1 > c0) {
                const bool safe = valid && all_in_range(u, v, g);
                const uint32_t *d = dil + (uint32_t)c0 * pitch;
                const float um = valid ? u : 0.0f, vm = valid ? v : 0.0f;
                if (__ballot(valid && !safe))
                    kept = kept_in_columns<true>(d, cs + c0, pitch, um, vm, want, c1 - c0, g);
                else if (want)
                    kept = kept_in_columns<false>(d, cs + c0, pitch, um, vm, want, c1 - c0, g);
            }
            if (SHARE > 1) {
                if (lane == 0) s_kept[wave] = kept;
                __syncthreads();
                if (part == 0) {
#pragma unroll
                    for (int w = 1; w < SHARE; ++w) kept |= s_kept[wave + w];
                }
            }
            // later blocks of columns only add to the verdicts
            if (part == 0 && in) {
                const bool k_me = (kept >> lane) & 1ull;
                if (ja == 0) keep[i] = k_me ? 1u : 0u;
                else if (k_me) keep[i] = 1u;
            }
            if (SHARE > 1) __syncthreads();
        }
    }
}

// Phase clock of the instrumented build (compiled with HOUGH_PHASE_TIMING; the product build
// compiles it away): thread 0 of a workgroup reads the constant-rate clock after each workgroup
// barrier and charges the interval to the phase that just ended; at exit it adds its totals to
// a device array that hough_debug_phase_ticks reads.
#ifdef HOUGH_PHASE_TIMING
}  // namespace
__device__ unsigned long long g_phase_ticks[kPhaseSlots];
namespace {
struct PhaseClock {
    uint64_t last = 0, t[kPhaseSlots] = {};
    __device__ __forceinline__ void start() {
        if (threadIdx.x == 0) last = (uint64_t)wall_clock64();
    }
    __device__ __forceinline__ void mark(int i) {
        if (threadIdx.x == 0) {
            const uint64_t n = (uint64_t)wall_clock64();
            t[i] += n - last;
            last = n;
        }
    }
    __device__ __forceinline__ void count(int i, uint64_t v) {
        if (threadIdx.x == 0) t[i] += v;
    }
    __device__ __forceinline__ void flush() {
        if (threadIdx.x == 0)
            for (int i = 0; i < kPhaseSlots; ++i) atomicAdd(&g_phase_ticks[i], (unsigned long long)t[i]);
    }
};
#else
struct PhaseClock {
    __device__ __forceinline__ void start() {}
    __device__ __forceinline__ void mark(int) {}
    __device__ __forceinline__ void count(int, uint64_t) {}
    __device__ __forceinline__ void flush() {}
};
#endif

// ------------------------------------------------------------------------ fused batch path
// One workgroup processes one event at a time, taken from a global work counter; the event's
// theta tiles are processed in order: vote, find peaks, list + dilate, then retain while the
// tile is cleared for the next one.  Counters are packed two per dword (an event has at most
// kMaxBatchHits hits, so a count fits 16 bits).  Wave w owns hits [hb, he) of the event for
// voting and retention and writes their keep bytes itself (each lane those of its own hits,
// the pending list aside).  Retention is skipped for the rest of the event once every valid
// hit is kept.
// queue[0] is the work counter and queue[1] counts workgroups that have left the loop; the
// last one to leave (every pop has then happened) puts both back to zero for the next launch,
// so a launch is a single kernel with no memset.
// SP: tiles with at most kTilePeaks peaks list them for the peak-list retention (the plan's
// choice for sparse grids and the relative threshold; compiled out otherwise, where it only
// costs).
// WIN: the tile holds a window of `win` rho rows (a multiple of 32) instead of the whole
// column.  The hits of an event vote only into the rows their radius lets them reach (|rho| is at
// most 1 / sqrt(x^2 + y^2) in every column), so each event is given the window [wb, wb + win)
// (wb a multiple of 16) that covers those rows; the rows outside are zero, cannot hold a peak
// and are never looked up.  Tile row r holds grid row wb - 1 + r: one zero halo row on each
// side, then the out-of-grid columns' dummy row.  The peak and dilated words stay aligned to
// the grid's 32-row words (those the window touches, plus one zero row), so retention looks
// up grid rows exactly as without a window.  An event whose hits reach beyond the window is
// left to the spill kernel (kStatusSpill).  A smaller tile lets more workgroups share a CU,
// which is what the window is for: on the paper's grid (rho range twice the reach of hits at
// 200 mm and beyond) half of the 1000 rows are enough.
// Launch bounds: a windowed tile exists to fit two or three workgroups of at most 8 waves on a
// CU, so 4 waves per SIMD are enough for it and leave it registers to spare.  The 8-wave kernel of
// dense grids fits 64 registers, so that four workgroups of a 360 x 256 tile (39.6 KB of LDS)
// share a CU: 32 waves hide the phases' latencies better than 24 (10,000 events 1,559 -> 1,478 us;
// 1,000 events, which then all run at once, 159 -> 166 us), at the price of 3 registers in scratch (12
// on theta-periodic grids, where the 10,000 events take 1,618 us).  The others keep 80.
template <int NW, int G, bool PER, bool SP, bool WIN>
__global__ __launch_bounds__(NW * 64, (NW == 16 || WIN) ? 4 : (G == 1 ? (NW == 8 && !SP ? 8 : 6) : 4)) void k_batch(GridArgs g, BatchArgs a,
                                                                                            int n_tiles, int nwords,
                                                                                            int win) {
    using L = Lane<G, true>;
    constexpr int TW = L::TW, ST = L::STRIDE, DP = (int)kDilPitch<G>, OUT = TW - 2, NT = NW * 64;
    static_assert(!WIN || G == 1, "windowed tiles: one column group");
    extern __shared__ __align__(16) uint32_t lds[];
    // tile rows (dummy row included) and peak-word rows of the LDS layout
    const int rows_t = WIN ? win + 3 : g.n_rho + 1;
    const int nwp = WIN ? win / 32 + 1 : nwords;
    uint32_t *tile = lds;                                                  // [rows_t * ST]
    // the lookups' stage takes the peak words' place, which are dead once listed (not in a windowed
    // tile, whose size sets the window's height)
    float2 *stage = reinterpret_cast<float2 *>(tile + (size_t)rows_t * ST);   // [NW * 64]
    uint32_t *pmask = reinterpret_cast<uint32_t *>(stage) + (WIN ? NW * (kStageBytes / 4) : 0);   // [nwp * TW]
    float4 *tpk = reinterpret_cast<float4 *>(pmask + (WIN ? nwp * TW : stage_words<NW>(nwp * TW)));   // [kTilePeaks] (SP)
    uint32_t *colcnt = reinterpret_cast<uint32_t *>(tpk + (SP ? kTilePeaks : 0));   // [TW] peaks per column
    uint32_t *dil = colcnt + TW;                                           // [(nwp + 1) * DP]
    __shared__ uint32_t s_event, s_npeaks, s_flags, s_nvalid, s_nkept, s_max, s_minr2, s_wb, s_fit, s_edge;
    const int lane = threadIdx.x & 63, wave = wave_id();
    const int tile_words4 = rows_t * ST / 4;
    // the launch's events: all of the batch, or those a windowed launch before it listed (none:
    // nothing to take, and the counters stay at zero)
    const uint32_t n_take = a.n_from ? (uint32_t)__builtin_amdgcn_readfirstlane((int)*a.n_from) : a.n_events;
    if (n_take == 0u) return;

    // the tile is all zero at the start of every tile; the dil row past the last word is read
    // by the out-of-grid columns' dummy row and stays zero
    for (int i = threadIdx.x; i < tile_words4; i += NT)
        reinterpret_cast<uint4 *>(tile)[i] = make_uint4(0u, 0u, 0u, 0u);
    for (int i = threadIdx.x; i < DP; i += NT) dil[nwp * DP + i] = 0u;
    for (int i = threadIdx.x; i < TW; i += NT) colcnt[i] = 0u;   // zero again after each listing
    PhaseClock pc;
    pc.start();

    for (;;) {
        if (threadIdx.x == 0) {
            const uint32_t q = atomicAdd(a.queue, 1u);
            s_event = q < n_take ? (a.order ? a.order[q] : q) : 0xffffffffu;
            s_npeaks = 0u;
            s_flags = 0u;
            s_nvalid = 0u;
            s_nkept = 0u;
            s_max = 0u;
            s_minr2 = __float_as_uint(FLT_MAX);
        }
        __syncthreads();
        pc.mark(kPhasePop);
        // wave-uniform values live in scalar registers
        const uint32_t e = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_event);
        if (e >= a.n_events) {
            pc.flush();
            if (threadIdx.x == 0 && atomicAdd(a.queue + 1, 1u) == gridDim.x - 1u) {
                __hip_atomic_store(a.queue, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(a.queue + 1, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            break;
        }
        // event e of this launch is pool event ids[e] (or e itself); its keep bytes start at
        // keep_offsets[e] (or at its first hit)
        const uint32_t pe_id = (uint32_t)__builtin_amdgcn_readfirstlane((int)(a.ids ? a.ids[e] : e));
        const uint32_t h0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)a.offsets[pe_id]);
        const uint32_t h1 = (uint32_t)__builtin_amdgcn_readfirstlane((int)a.offsets[pe_id + 1]);
        if (h1 < h0) {                       // malformed offsets: touch nothing but the counters
            if (threadIdx.x == 0) { a.n_peaks[e] = 0u; a.status[e] = HOUGH_EV_TOO_MANY_HITS; }
            __syncthreads();
            continue;
        }
        const uint32_t H = h1 - h0;
        if (H > kMaxBatchHits || H == 0u) {      // above the 16-bit counters: the spill kernel's
            uint8_t *ke = a.keep + (a.ids ? a.keep_offsets[e] : h0);
            for (uint32_t i = (uint32_t)opaque((int)threadIdx.x); i < H; i += NT) ke[i] = 0u;
            if (threadIdx.x == 0) {
                a.n_peaks[e] = 0u;
                a.status[e] = H ? kStatusSpill : 0u;
                if (H && a.spill_count) atomicAdd(a.spill_count, 1u);
            }
            __syncthreads();
            continue;
        }
        uint32_t hb, he;
        wave_hits<NW>(H, wave, hb, he);
        const float *xe = a.x + h0, *ye = a.y + h0;
        // the workgroup's room for mapped hits, where the wave's share of the event fits it
        float *uv = a.uv && he <= a.uv_hits ? a.uv + (size_t)blockIdx.x * 2u * a.uv_hits : nullptr;
        hough_peak *pe = a.peaks ? a.peaks + (size_t)e * a.max_peaks : nullptr;
        const uint32_t cap = pe ? a.max_peaks : 0u;
        uint32_t bad = 0;
        uint8_t *ke = a.keep + (a.ids ? (uint32_t)__builtin_amdgcn_readfirstlane((int)a.keep_offsets[e]) : h0);
        // with duplicate suppression the duplicate pass has written every keep byte already
        if (!g.dedup) {
#pragma unroll 1
            for (uint32_t i = hb + (uint32_t)opaque(lane); i < he; i += 64) ke[i] = 0u;
        } else if (H > kDedupMaxHits && threadIdx.x == 0) {
            atomicOr(&s_flags, HOUGH_EV_DEDUP_SKIPPED);
        }
        // the event's rho window
        int wb = 0;
        if constexpr (WIN) {
            const uint32_t mn = min_r2_bits(xe, ye, hb, he, lane);
            if (lane == 0) atomicMin(&s_minr2, mn);
            __syncthreads();
            if (threadIdx.x == 0) {
                int b0;
                s_fit = window_of<PER>(g, __uint_as_float(s_minr2), win, b0) ? 1u : 0u;
                s_wb = (uint32_t)b0;
            }
            __syncthreads();
            wb = __builtin_amdgcn_readfirstlane((int)s_wb);
            if (__builtin_amdgcn_readfirstlane((int)s_fit) == 0) {
                // list it for the launch on whole columns, or leave it to the spill kernel (its keep
                // bytes are clear, or hold the duplicate pass's marks, which the spill kernel reads)
                if (threadIdx.x == 0 && a.defer_list) {
                    a.defer_list[atomicAdd(a.defer_count, 1u)] = e;
                } else if (threadIdx.x == 0) {
                    a.n_peaks[e] = 0u;
                    a.status[e] = kStatusSpill;
                    if (a.spill_count) atomicAdd(a.spill_count, 1u);
                }
                __syncthreads();
                continue;
            }
        }
        // grid row k of the window lives in tile row k - wb + 1; grid word w of the peak and
        // dilated words in word row w - wb / 32
        uint32_t *tile_w = WIN ? tile + (ptrdiff_t)(1 - wb) * ST : tile;
        uint32_t *pmask_w = WIN ? pmask - (ptrdiff_t)(wb >> 5) * TW : pmask;
        uint32_t *dil_w = WIN ? dil - (ptrdiff_t)(wb >> 5) * DP : dil;
        const int w_lo = WIN ? (wb >> 5) : 0;
        const float dummy_row = WIN ? (float)(wb + win + 1) : -1.0f;
        uint32_t thr = g.threshold;
        // relative threshold (such launches take the SP kernels): a first round over the tiles votes
        // them only to find the event's largest count
        const bool rel = SP && a.frac_den != 0u;
        uint32_t mloc = 0;
        pc.mark(kPhaseSetup);
        pc.count(kPhaseEvents, 1u);
        Pending pd;
        pd.idx = 0u;
        pd.u = pd.v = 0.0f;
        pd.live = 0ull;
        pd.on = false;
        uint32_t unkept = he - hb;           // this wave's unkept hits after its last full pass
        // Deferred retention: peaks [def0, def0 + defn) of the event's list still have to keep
        // their hits.  flush() tests every unkept hit against them, 64 peaks at a time staged in
        // the tile's peak list (wave 0 reads the records back, then every wave tests its own
        // hits), and drops the pending lists (their entries may have been kept meanwhile).
        // (only where the launch bound leaves registers for it: windowed and 16-wave kernels)
        constexpr bool DEF = SP && (WIN || NW == 16);
        uint32_t def0 = 0, defn = 0;
        auto flush = [&]() {
            for (uint32_t b = 0; b < defn; b += kTilePeaks) {
                const uint32_t nb = min(kTilePeaks, defn - b);
                if (wave == 0) {
                    bool near = false;
                    if ((uint32_t)lane < nb) {
                        const uint64_t rec = __hip_atomic_load(
                            reinterpret_cast<const uint64_t *>(pe + def0 + b + (uint32_t)lane), __ATOMIC_RELAXED,
                            __HIP_MEMORY_SCOPE_AGENT);
                        const int j = (int)(rec & 0xffffu), k = (int)((rec >> 16) & 0xffffu);
                        tpk[lane] = make_float4(g.C[j], g.S[j], __int_as_float(k - g.rho_window), 0.0f);
                        near = k <= g.rho_window || k >= g.n_rho - g.rho_window;
                    }
                    const uint64_t nm = __ballot(near);
                    if (lane == 0) s_edge = nm ? 1u : 0u;
                }
                __syncthreads();
                uint32_t left = 0;
                const uint32_t newly = retain_range_peaks(tpk, nb, s_edge != 0u, xe, ye, ke, hb, he, g, lane, left);
                if (lane == 0 && newly) atomicAdd(&s_nkept, newly);
                unkept = left;
                __syncthreads();
            }
            defn = 0;
            pd.on = false;
            pd.live = 0ull;
        };
        // sparse event (under a quarter of the threshold per cell on average): most peak units
        // hold no count that reaches it, so each unit is first tested whole (unit_below)
        bool sparse_ev = SP && (uint64_t)H * 4u < (uint64_t)thr * (uint32_t)g.n_rho;
        const int t_first = rel ? -n_tiles : 0;
        for (int tt = t_first; tt < n_tiles; ++tt) {
            const int t = SP && tt < 0 ? tt + n_tiles : tt;
            const int first = t * OUT - 1;      // grid column of lane 0 of group 0
            const int vl = opaque(lane);
            const Cols<G> cl = load_cols<G, PER>(g, first, vl, ST, L(vl).col, dummy_row);
            // (the event's first sweep counts the valid hits and meets the invalid ones)
            const uint32_t nv = vote_range<G, PER>(tile_w, xe, ye, hb, he, cl, g, first, vl, bad,
                                                   WIN ? dummy_row : g.nrho_f, g.dedup ? ke : nullptr, uv, a.uv_hits,
                                                   tt > t_first);
            if (tt == t_first && lane == 0 && nv) atomicAdd(&s_nvalid, nv);
            __syncthreads();
            if (SP && tt < 0) {
                // every tile row but the dummy one (a window's halo rows stay zero)
#pragma unroll 1
                for (int i = opaque((int)threadIdx.x); i < (rows_t - 1) * ST / 4; i += NT) {
                    const uint4 d = reinterpret_cast<const uint4 *>(tile)[i];
                    mloc = max(mloc, max(max(max(d.x & 0xffffu, d.x >> 16), max(d.y & 0xffffu, d.y >> 16)),
                                         max(max(d.z & 0xffffu, d.z >> 16), max(d.w & 0xffffu, d.w >> 16))));
                    reinterpret_cast<uint4 *>(tile)[i] = make_uint4(0u, 0u, 0u, 0u);
                }
                for (int i = (rows_t - 1) * ST + opaque((int)threadIdx.x); i < rows_t * ST; i += NT) tile[i] = 0u;
                if (tt == -1) {
                    mloc = wave_max(mloc);
                    if (lane == 0) atomicMax(&s_max, mloc);
                }
                __syncthreads();
                if (tt == -1) {
                    const uint64_t top = (uint64_t)s_max * a.frac_num + a.frac_den - 1u;
                    thr = (uint32_t)__builtin_amdgcn_readfirstlane(
                        (int)min<uint64_t>(max<uint64_t>(top / a.frac_den, g.threshold), 0x7fffffffull));
                    sparse_ev = (uint64_t)H * 4u < (uint64_t)thr * (uint32_t)g.n_rho;
                }
                pc.mark(kPhaseSetup);
                continue;
            }
            pc.mark(kPhaseVote);
            if (t == 0) pc.count(kPhaseStagedHits, (uint64_t)s_nvalid * (uint64_t)n_tiles);
            const int pl = opaque(lane);
            const L ln(pl);
            // 16-row units of grid rows; a windowed tile tests the units inside its window (the
            // halo rows above and below are in the tile, so no unit needs bounds tests) and
            // writes zero for the other halves of the words it touches
            for (int u = 2 * w_lo + wave; u < 2 * (w_lo + nwp); u += NW) {
                uint32_t m[G];
                const bool interior = WIN || (u >= 1 && (u + 1) * kPeakRows < g.n_rho);
                constexpr bool UR = NW == 16 || WIN;     // launch bound of 4 waves per SIMD: registers to spare
                if ((WIN && (u * kPeakRows < wb || (u + 1) * kPeakRows > wb + win)) ||
                    (sparse_ev && interior && !(PER && (t == 0 || t == n_tiles - 1)) && unit_below<G>(tile_w, u, thr, pl))) {
#pragma unroll
                    for (int q = 0; q < G; ++q) m[q] = 0u;
                } else if (PER && (t == 0 || t == n_tiles - 1)) {
                    if (interior)
                        peak_rows<false, G, true, true, UR>(tile_w, u, g.n_rho, thr, ln, pl, m, first, g.n_theta);
                    else
                        peak_rows<true, G, true, true, UR>(tile_w, u, g.n_rho, thr, ln, pl, m, first, g.n_theta);
                } else if (interior) {
                    peak_rows<false, G, true, false, UR>(tile_w, u, g.n_rho, thr, ln, pl, m);
                } else {
                    peak_rows<true, G, true, false, UR>(tile_w, u, g.n_rho, thr, ln, pl, m);
                }
                uint16_t *pm16 = reinterpret_cast<uint16_t *>(pmask_w);
#pragma unroll
                for (int q = 0; q < G; ++q) {
                    const int c = 64 * q + pl;
                    const bool out_col = (c >= 1) && (c <= TW - 2) && (first + c < g.n_theta);
                    pm16[((u >> 1) * TW + c) * 2 + (u & 1)] = out_col ? (uint16_t)m[q] : (uint16_t)0;
                    if (out_col && m[q]) atomicAdd(&colcnt[c], (uint32_t)__popc(m[q]));
                }
            }
            if (g.rho_window >= 32) {
#pragma unroll 1
                for (int i = opaque((int)threadIdx.x); i < nwp * DP; i += NT) dil[i] = 0u;
            }
            if (SP && threadIdx.x == 0) s_edge = 0u;     // set by the listing for a peak near a rho edge
            __syncthreads();
            pc.mark(kPhasePeaks);
            const uint32_t base = s_npeaks;
            const int el = opaque(lane);
            uint32_t np;
            if constexpr (SP)
                np = emit_and_dilate<G, true>(tile_w, pmask_w, dil_w, w_lo, nwp, first, g, pe, cap, base, L(el), el,
                                              wave, NW, tpk, &cl, colcnt, &s_edge);
            else
                np = emit_and_dilate<G, true>(tile_w, pmask_w, dil_w, w_lo, nwp, first, g, pe, cap, base, L(el), el,
                                              wave, NW, nullptr, nullptr, colcnt);
            __syncthreads();
            pc.mark(kPhaseList);
            if (threadIdx.x == 0) s_npeaks = base + np;
            for (int i = opaque((int)threadIdx.x); i < TW; i += NT) colcnt[i] = 0u;
            // the counts are dead: clear the tile for the next one while retention reads dil
            clear_quads<NT>(tile, tile_words4);
            if (DEF && np && s_nkept < s_nvalid && pe && np <= kDeferTilePeaks && base + np <= cap &&
                defn + np <= kDeferPeaks) {
                if (defn == 0) def0 = base;          // the deferred peaks stay contiguous
                defn += np;
            } else if (np && s_nkept < s_nvalid) {
                // Few peaks: test each hit against the peak list (about 5 instructions per peak
                // for a chunk of 64 hits, kept or not; 9 when a peak lies near a rho edge) where
                // that beats looking the unkept hits up in every column's dilated words (about 7
                // per unkept hit, plus staging).  A flush of deferred peaks reuses the list's
                // storage, so after one this tile looks its hits up in the dilated words.
                const int rl = opaque(lane);
                bool few = SP && np <= kTilePeaks;
                const bool edge = SP && s_edge != 0u;
                if (DEF && defn) {
                    flush();
                    few = false;
                }
                const uint32_t cp = edge ? 9u : 5u;
                uint32_t newly;
                if (pd.on) {
                    const uint32_t n = (uint32_t)__popcll(pd.live);
                    newly = (few && np * cp < n * 7u + 10u)
                                ? retain_pending_peaks(pd, tpk, np, edge, ke, g, rl)
                                : retain_pending<G>(pd, dil_w, stage + wave * 64, ke, cl, g, rl);
                } else {
                    uint32_t left = 0;
                    const uint32_t chunks = (he - hb + 63u) >> 6;
                    if (few && np * cp * chunks < unkept * 7u + chunks * 10u) {
                        newly = retain_range_peaks(tpk, np, edge, xe, ye, ke, hb, he, g, rl, left);
                        if (left <= 64u) build_pending(pd, xe, ye, ke, hb, he, g, rl);
                    } else {
                        newly = retain_range<G>(pd, dil_w, stage + wave * 64, xe, ye, ke, hb, he, cl, g, first,
                                                np * (2u * (uint32_t)g.rho_window + 1u) >= (uint32_t)g.n_rho, rl,
                                                left);
                    }
                    if (SP) unkept = left;
                }
                if (lane == 0 && newly) atomicAdd(&s_nkept, newly);
            }
            __syncthreads();
            pc.mark(kPhaseRetain);
        }
        if (DEF && defn) {
            if (s_nkept < s_nvalid) flush();
            pc.mark(kPhaseRetain);
        }
        if (__ballot(bad != 0u) && lane == 0) atomicOr(&s_flags, HOUGH_EV_INVALID_HITS);
        if (g.dedup) {                       // drop the later-copy bit, leaving the kept bit
#pragma unroll 1
            for (uint32_t i = hb + (uint32_t)opaque(lane); i < he; i += 64) {
                const uint32_t v = ke[i];
                if (v & kKeepDuplicate) ke[i] = (uint8_t)(v & 1u);
            }
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            const uint32_t np = s_npeaks;
            a.n_peaks[e] = np;
            a.status[e] = s_flags | (np > a.max_peaks ? HOUGH_EV_PEAKS_TRUNCATED : 0u);
        }
        __syncthreads();
        pc.mark(kPhaseFinish);
    }
}

// ------------------------------------------------------------ split batch path (latency form)
// The same results as k_batch for batches small enough that latency matters more than
// throughput: the work items are the (event, theta tile) pairs, so the tiles of one event run
// on different workgroups at once.  A workgroup takes one item: it votes all of the event's hits,
// finds the tile's peaks, publishes their number in the item's slot, adds up the numbers of
// the event's earlier tiles, and lists its peaks where they belong in the event's list.  It then
// tests the event's hits that no other tile has kept yet.  Nothing is staged or merged: the
// tiles of an event share its slots and its keep bytes, and nothing else.
//
// Waiting for the earlier tiles ends: items are numbered event by event, tile by tile, and taken
// from a counter, so every earlier tile belongs to a workgroup that is already running, and a
// workgroup publishes before it waits.
//
// What the tiles share is written and read by agent-scope atomics, which pass by the L2s (one
// per XCD, not coherent with each other); a wave's stores are waited for before the barrier
// that precedes the publication.  Tile 0 clears the keep bytes before it publishes, the others
// set theirs after they have seen its slot.  No cache is written back or invalidated on the way
// (publishing with fences and merging staged lists took 11 of one event's 30 us; it takes 16
// so).  The spill kernel launched afterwards puts the slots and the counter back to zero.
// WIN: the tile holds the event's window of rows, as in k_batch (grids taller than a tile).  Each
// tile finds the window itself from all of the event's hits, so all of them agree on it, and on
// leaving an event that does not fit it to the spill kernel (1000 x 2000, one event: 183 us when
// one workgroup walked its 17 tiles, 25 so).
constexpr uint32_t kSlotReady = 0x80000000u;

__device__ __forceinline__ uint32_t keep_load(const uint8_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void keep_store(uint8_t *p, uint32_t v) {
    __hip_atomic_store(p, (uint8_t)v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Step 5 of one tile in the split form, over a wave's share of the event's hits: against the
// tile's peak list when it has one (np <= kTilePeaks), else as retain_range.  The tiles of an event
// start at different places of the share (turn of turns), so that most of the hits a tile
// comes to later have been kept by another one already.  (64 dense events, 720 x 512: 119 us per
// batch when every tile starts at the first hit)
__device__ void retain_split(const uint32_t *dil, const float4 *tpk, uint32_t np, bool edge, float2 *st,
                             const float *x, const float *y, uint8_t *ke, uint32_t hb, uint32_t he,
                             const Cols<1> &cl, const GridArgs &g, int first_col, uint32_t turn, uint32_t turns,
                             int lane) {
    const bool many = np * (2u * (uint32_t)g.rho_window + 1u) >= (uint32_t)g.n_rho;
    const uint32_t chunks = (he - hb + 63u) >> 6;
    if (chunks == 0u) return;
    uint32_t c = (uint32_t)((uint64_t)chunks * turn / turns);
    uint32_t kn = 1u;
    float xn = 0.0f, yn = 0.0f;                       // the next 64 hits load while these are tested
    auto load = [&](uint32_t cc) {
        const uint32_t i = hb + 64u * cc + (uint32_t)lane;
        kn = 1u;
        if (i < he) { kn = keep_load(ke + i); xn = x[i]; yn = y[i]; }
    };
    load(c);
    for (uint32_t n = 0; n < chunks; ++n) {
        const uint32_t i = hb + 64u * c + (uint32_t)lane, kv = kn;
        const float xi = xn, yi = yn;
        if (++c == chunks) c = 0;
        if (n + 1u < chunks) load(c);
        const bool todo = i < he && !(kv & 1u);
        if (__ballot(todo) == 0ull) continue;
        float u, v;
        const bool valid = conformal(todo ? xi : 0.0f, todo ? yi : 0.0f, u, v) && todo;
        uint64_t kept = 0;
        if (np <= kTilePeaks) {
            kept = kept_by_peaks(tpk, np, valid ? u : 0.0f, valid ? v : 0.0f, valid, edge, g);
        } else {
            const bool safe = valid && all_in_range(u, v, g);
            const uint64_t bs = __ballot(safe), bv = __ballot(valid);
            if (many && __popcll(bs) >= kColumnRoundHits)
                kept = kept_by_columns<1>(dil, safe ? u : 0.0f, safe ? v : 0.0f, bs, first_col, g);
            kept |= lookup_lanes<1>(dil, st, u, v, bs & ~kept, cl, g, lane);
            kept |= lookup_checked<1>(dil, u, v, bv & ~bs, cl, g, lane);
        }
        if ((kept >> lane) & 1ull) keep_store(ke + i, kv | 1u);
    }
}

template <int NW, bool PER, bool WIN>
__global__ __launch_bounds__(NW * 64, NW == 16 ? 4 : 6) void k_batch_split(GridArgs g, BatchArgs a, SplitArgs sp,
                                                                           int nwords, int win) {
    using L = Lane<1, true>;
    constexpr int TW = L::TW, ST = L::STRIDE, DP = (int)kDilPitch<1>, OUT = TW - 2, NT = NW * 64;
    extern __shared__ __align__(16) uint32_t lds[];
    const int rows_t = WIN ? win + 3 : g.n_rho + 1, nwp = WIN ? win / 32 + 1 : nwords;
    uint32_t *tile = lds;                                                  // [rows_t * ST]
    float2 *stage = reinterpret_cast<float2 *>(tile + (size_t)rows_t * ST);   // [NW * 64]
    uint32_t *pmask = reinterpret_cast<uint32_t *>(stage);                 // [nwp * TW], dead once listed
    float4 *tpk = reinterpret_cast<float4 *>(pmask + stage_words<NW>(nwp * TW));   // [kTilePeaks]
    uint32_t *colcnt = reinterpret_cast<uint32_t *>(tpk + kTilePeaks);     // [TW]
    uint32_t *dil = colcnt + TW;                                           // [(nwp + 1) * DP]
    __shared__ uint32_t s_item, s_bad, s_base, s_edge, s_minr2, s_wb, s_fit;
    const int lane = threadIdx.x & 63, wave = wave_id();
    if (threadIdx.x == 0) {
        s_item = atomicAdd(a.queue, 1u);
        s_bad = 0u;
        s_edge = 0u;
        s_minr2 = __float_as_uint(FLT_MAX);
    }
    for (int i = threadIdx.x; i < rows_t * ST / 4; i += NT)
        reinterpret_cast<uint4 *>(tile)[i] = make_uint4(0u, 0u, 0u, 0u);
    for (int i = threadIdx.x; i < DP; i += NT) dil[nwp * DP + i] = 0u;
    for (int i = threadIdx.x; i < TW; i += NT) colcnt[i] = 0u;
    if (g.rho_window >= 32)
        for (int i = threadIdx.x; i < nwp * DP; i += NT) dil[i] = 0u;
    __syncthreads();
    const uint32_t item = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_item), T = sp.n_tiles;
    if (item >= a.n_events * T) return;                    // (the grid holds one workgroup per item)
    const uint32_t e = item / T, t = item - e * T;
    uint32_t *slots = sp.slots + (size_t)e * T;
    const uint32_t pe_id = (uint32_t)__builtin_amdgcn_readfirstlane((int)(a.ids ? a.ids[e] : e));
    const uint32_t h0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)a.offsets[pe_id]);
    const uint32_t h1 = (uint32_t)__builtin_amdgcn_readfirstlane((int)a.offsets[pe_id + 1]);
    if (h1 <= h0 || h1 - h0 > kMaxBatchHits) {
        // malformed, empty, or left to the spill kernel (which writes everything of such an event)
        if (threadIdx.x == 0 && t == 0) {
            const bool spill = h1 > h0;
            a.n_peaks[e] = 0u;
            a.status[e] = spill ? kStatusSpill : (h1 < h0 ? HOUGH_EV_TOO_MANY_HITS : 0u);
            if (spill && a.spill_count) atomicAdd(a.spill_count, 1u);
        }
        return;                                            // every tile of the event returns here: none waits
    }
    const uint32_t H = h1 - h0;
    uint8_t *ke = a.keep + (a.ids ? (uint32_t)__builtin_amdgcn_readfirstlane((int)a.keep_offsets[e]) : h0);
    const float *xe = a.x + h0, *ye = a.y + h0;
    hough_peak *pe = a.peaks ? a.peaks + (size_t)e * a.max_peaks : nullptr;
    const uint32_t cap = pe ? a.max_peaks : 0u;
    uint32_t hb, he;
    wave_hits<NW>(H, wave, hb, he);
    if (t == 0 && !g.dedup)                                // (the duplicate pass has written every keep byte)
        for (uint32_t i = threadIdx.x; i < H; i += NT) keep_store(ke + i, 0u);
    // the event's rho window, the same in every tile of it (see k_batch)
    int wb = 0;
    if constexpr (WIN) {
        const uint32_t mn = min_r2_bits(xe, ye, hb, he, lane);
        if (lane == 0) atomicMin(&s_minr2, mn);
        __syncthreads();
        if (threadIdx.x == 0) {
            int b0;
            s_fit = window_of<PER>(g, __uint_as_float(s_minr2), win, b0) ? 1u : 0u;
            s_wb = (uint32_t)b0;
        }
        __syncthreads();
        wb = __builtin_amdgcn_readfirstlane((int)s_wb);
        if (__builtin_amdgcn_readfirstlane((int)s_fit) == 0) {   // the spill kernel's, in every tile
            if (threadIdx.x == 0 && t == 0) {
                a.n_peaks[e] = 0u;
                a.status[e] = kStatusSpill;
                if (a.spill_count) atomicAdd(a.spill_count, 1u);
            }
            return;
        }
    }
    uint32_t *tile_w = WIN ? tile + (ptrdiff_t)(1 - wb) * ST : tile;
    uint32_t *pmask_w = WIN ? pmask - (ptrdiff_t)(wb >> 5) * TW : pmask;
    uint32_t *dil_w = WIN ? dil - (ptrdiff_t)(wb >> 5) * DP : dil;
    const int w_lo = WIN ? (wb >> 5) : 0;
    const float dummy_row = WIN ? (float)(wb + win + 1) : -1.0f;
    uint32_t bad = 0;
    const int first = (int)t * OUT - 1;
    const int vl = opaque(lane);
    const Cols<1> cl = load_cols<1, PER>(g, first, vl, ST, L(vl).col, dummy_row);
    vote_range<1, PER>(tile_w, xe, ye, hb, he, cl, g, first, vl, bad, WIN ? dummy_row : g.nrho_f,
                       g.dedup ? ke : nullptr);
    __syncthreads();
    const int pl = opaque(lane);
    const L ln(pl);
    for (int u = 2 * w_lo + wave; u < 2 * (w_lo + nwp); u += NW) {
        uint32_t m[1];
        const bool interior = WIN || (u >= 1 && (u + 1) * kPeakRows < g.n_rho);
        constexpr bool UR = NW == 16;
        if (WIN && (u * kPeakRows < wb || (u + 1) * kPeakRows > wb + win)) {
            m[0] = 0u;
        } else if (PER && (t == 0 || t == T - 1)) {
            if (interior)
                peak_rows<false, 1, true, true, UR>(tile_w, u, g.n_rho, g.threshold, ln, pl, m, first, g.n_theta);
            else
                peak_rows<true, 1, true, true, UR>(tile_w, u, g.n_rho, g.threshold, ln, pl, m, first, g.n_theta);
        } else if (interior) {
            peak_rows<false, 1, true, false, UR>(tile_w, u, g.n_rho, g.threshold, ln, pl, m);
        } else {
            peak_rows<true, 1, true, false, UR>(tile_w, u, g.n_rho, g.threshold, ln, pl, m);
        }
        const bool out_col = pl >= 1 && pl <= TW - 2 && first + pl < g.n_theta;
        reinterpret_cast<uint16_t *>(pmask_w)[((u >> 1) * TW + pl) * 2 + (u & 1)] = out_col ? (uint16_t)m[0] : (uint16_t)0;
        if (out_col && m[0]) atomicAdd(&colcnt[pl], (uint32_t)__popc(m[0]));
    }
    if (t == T - 1 && __ballot(bad != 0u) && lane == 0) s_bad = 1u;
    // this wave's keep stores (tile 0) have arrived before the barrier, so before the publication
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (wave == 0) {
        const uint32_t np = (uint32_t)__builtin_amdgcn_readfirstlane((int)wave_sum(colcnt[lane]));
        if (lane == 0)
            __hip_atomic_store(slots + t, kSlotReady | np, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        uint32_t before = 0;
        for (uint32_t t0 = 0; t0 < t; t0 += 64) {
            const bool mine = t0 + (uint32_t)lane < t;
            uint32_t v;
            for (;;) {
                v = mine ? __hip_atomic_load(slots + t0 + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : kSlotReady;
                if (__ballot(!(v & kSlotReady)) == 0ull) break;
                __builtin_amdgcn_s_sleep(1);
            }
            before += v & ~kSlotReady;
        }
        before = wave_sum(before);
        if (lane == 0) {
            s_base = before;
            if (t == T - 1) {
                const uint32_t total = before + np;        // the event's true peak count
                a.n_peaks[e] = total;
                a.status[e] = (s_bad ? HOUGH_EV_INVALID_HITS : 0u) |
                              (g.dedup && H > kDedupMaxHits ? HOUGH_EV_DEDUP_SKIPPED : 0u) |
                              (total > a.max_peaks ? HOUGH_EV_PEAKS_TRUNCATED : 0u);
            }
        }
    }
    asm volatile("" ::: "memory");
    __syncthreads();
    const int el = opaque(lane);
    const uint32_t np = emit_and_dilate<1, true>(tile_w, pmask_w, dil_w, w_lo, nwp, first, g, pe, cap, s_base, L(el), el, wave,
                                                 NW, tpk, &cl, colcnt, &s_edge);
    if (np == 0u) return;
    __syncthreads();
    retain_split(dil_w, tpk, np, s_edge != 0u, stage + wave * 64, xe, ye, ke, hb, he, cl, g, first, t, T,
                 opaque(lane));
}

// ------------------------------------------------------------ spill path (rho slabs)
// Events whose accumulator the fused kernel cannot hold on chip: events whose hits reach beyond a
// windowed tile on grids taller than a whole-column one, and events above kMaxBatchHits hits on any
// grid (counts beyond 16 bits).  One workgroup processes one event at
// a time:
//   - steps 1-4 one slab at a time in LDS (62 owned columns with halo lanes by up to 1,120 owned
//     rows with halo rows; 32-bit counts and 544 rows for events above 65,535 hits): vote, then
//     the 3x3 test of every owned cell, which leaves each (column, 32-row block) its peak rows
//     as a bit mask and each peak's count in device memory; the accumulator stays on chip;
//   - a thread per column places each block's peaks within its column, a scan over the columns
//     gives raster order, and the listing pass writes the peaks and marks the dilated retention
//     bits D[w * n_theta + j] (bit b: a peak of column j within rho_window rows of row 32w + b);
//   - retention stages one 64-column group of D in LDS at a time and looks the event's hits up
//     in it, lane = column.
// Every (group, slab) maps all of the event's hits again, so this path is for what the fused
// kernel cannot take, not a fast path.
constexpr int kSpillWaves = 16;
constexpr int kSpillThreads = kSpillWaves * 64;
constexpr uint32_t kSpillBlock = 4;      // at most this many events per counter pop when only some events spill
// the slab: 143 KB of dynamic LDS, what the CU's 160 KB leave beside the kernel's static LDS
// (slabs of 1,024 rows split a 2,000-row column into three, 3.4 against 4.1 ms per 1,000
// events on 1000 x 2000 bins)
constexpr int kSpillSlabDwords = 36608;
constexpr int kSpillOwnedPacked = 1120;  // owned rows of a packed slab: 35 blocks + 2 halo rows <= 1,144
constexpr int kSpillOwnedWide = 544;     // owned rows of a 32-bit slab: 17 blocks + 2 halo rows <= 572

// A word of the dilated bits (ORed by atomics in L2) or a peak's count in the accumulator,
// read past the L1.
__device__ __forceinline__ uint32_t spill_load(const uint32_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The spill kernel's device memory belongs to one workgroup, so workgroup scope orders it: the
// release waits for this wave's stores and atomics, the barrier lines the waves up.  The waves
// of a workgroup share one L1, which their plain stores go through; the dilation's atomic ORs
// are performed beyond it (in L2), so the dilated bits, and the peak counts with them, are read
// with loads that bypass the L1 (spill_load).  (Agent-scope fences here wrote back the whole
// L2 at every barrier: with many workgroups spilling at once that took most of the kernel's
// time.)
__device__ __forceinline__ void spill_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __syncthreads();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// The spill kernel's LDS slab: one group of up to 62 owned columns with a halo lane on each
// side (lane l holds column first + l - 1; on a theta-periodic grid the halo beyond either edge
// holds the wrapped column with rho reversed, as in the fused kernel) and owned rows [ro, ro1)
// with one halo row on each side (slab row i holds grid row ro - 1 + i).  P: two 16-bit counts
// per dword (events of at most 65,535 hits), else one 32-bit count per cell.
template <bool P>
struct SpillSlab {
    const uint32_t *tile;
    static constexpr int STRIDE = Lane<1, P>::STRIDE;      // dwords per slab row
    __device__ __forceinline__ uint32_t count(int l, int i) const {
        if (P) return (tile[i * STRIDE + (l & 31)] >> (16 * (l >> 5))) & 0xffffu;
        return tile[i * STRIDE + l];
    }
};

// Steps 1-3 into the slab: votes of hits [hb, he) by the whole-grid rule (bin k of the lane's
// column, a wrapped halo lane taking row n_rho - 1 - k), kept when r0 <= k < r1, at slab row
// k - base.  dup as for vote_range.
template <bool P>
__device__ void spill_vote_slab(uint32_t *tile, float2 *st, const float *x, const float *y, uint32_t hb,
                                uint32_t he, const Cols<1> &cl, bool wrap, const GridArgs &g, int lane,
                                uint32_t &bad, const uint8_t *dup, int r0, int r1, int base) {
    const Lane<1, P> ln(lane);
    for (uint32_t b0 = hb; b0 < he; b0 += 64) {
        const uint32_t i = b0 + lane;
        bool live = i < he;
        float xi = 0.0f, yi = 0.0f;
        if (live) { xi = x[i]; yi = y[i]; }
        if (dup && live && (dup[i] & kKeepDuplicate)) live = false;
        int slot;
        const StageCount n = stage_values(st, xi, yi, live, g, bad, slot);
#pragma unroll 4
        for (uint32_t h = 0; h < n.total; ++h) {
            const float2 p = st[h];
            const float t = __builtin_fmaf(p.x, cl.C[0], __builtin_fmaf(p.y, cl.S[0], cl.B[0]));
            if (t >= 0.0f && t < g.nrho_f) {
                const int k = wrap ? g.n_rho - 1 - (int)t : (int)t;
                if (k >= r0 && k < r1) lds_add(&tile[(k - base) * Lane<1, P>::STRIDE + (int)ln.col[0]], ln.inc);
            }
        }
        wave_sync();
    }
}

// Step 4 on rows [k0, k1) of slab lane l (owned column j): bit k - k0 of the result is set iff
// cell (j, k) is a peak, and the i-th peak's count is stored to pc[i] for the listing pass (a
// block holds at most 16 peaks: of two vertically adjacent cells the later one must exceed the
// earlier, the earlier must not fall below the later, so not both are peaks).  Raster
// order: the column before (j - 1) and the row above come first, except that on a periodic
// grid the wrapped column left of column 0 comes later and the one right of the last column
// earlier; rows outside the grid are the slab's zero halo rows.
template <bool P>
__device__ uint32_t spill_slab_peaks(const SpillSlab<P> &s, int l, int j, int k0, int k1, int base,
                                     uint32_t thr, const GridArgs &g, uint32_t *pc) {
    const bool left_later = g.periodic && j == 0, right_earlier = g.periodic && j == g.n_theta - 1;
    int i = k0 - base;
    uint32_t l0 = s.count(l - 1, i - 1), c0 = s.count(l, i - 1), r0 = s.count(l + 1, i - 1);
    uint32_t l1 = s.count(l - 1, i), c1 = s.count(l, i), r1 = s.count(l + 1, i);
    uint32_t m = 0;
    for (int k = k0; k < k1; ++k, ++i) {
        const uint32_t l2 = s.count(l - 1, i + 1), c2 = s.count(l, i + 1), r2 = s.count(l + 1, i + 1);
        if (c1 >= thr) {
            const uint32_t lm = max(max(l0, l1), l2), rm = max(max(r0, r1), r2);
            const uint32_t before = max(max(left_later ? 0u : lm, right_earlier ? rm : 0u), c0);
            const uint32_t after = max(max(left_later ? lm : 0u, right_earlier ? 0u : rm), c2);
            if (c1 >= max(before + 1u, after)) {
                pc[__popc(m)] = c1;
                m |= 1u << (k - k0);
            }
        }
        l0 = l1; l1 = l2;
        c0 = c1; c1 = c2;
        r0 = r1; r1 = r2;
    }
    return m;
}

// Every (group, slab) of the grid in turn: clear the slab, vote the event's hits into it (wave
// w maps its slice of the hits), then f(slab, first owned column, ro, ro1, base) between
// barriers.
template <bool P, typename F>
__device__ void spill_for_slabs(uint32_t *tile, float2 *st, const float *x, const float *y, uint32_t H,
                                const GridArgs &g, int lane, int wave, uint32_t &bad, const uint8_t *dup, F &&f) {
    constexpr int owned = P ? kSpillOwnedPacked : kSpillOwnedWide;
    constexpr int stride = Lane<1, P>::STRIDE;
    const Lane<1, P> ln(lane);
    const uint32_t hb = (uint32_t)((uint64_t)H * wave / kSpillWaves);
    const uint32_t he = (uint32_t)((uint64_t)H * (wave + 1) / kSpillWaves);
    for (int jo = 0; jo < g.n_theta; jo += 62) {
        const int j = jo - 1 + lane;
        const bool wrap = g.periodic && (j == -1 || j == g.n_theta);
        const Cols<1> cl = g.periodic ? load_cols<1, true>(g, jo - 1, lane, stride, ln.col)
                                      : load_cols<1, false>(g, jo - 1, lane, stride, ln.col);
        for (int ro = 0; ro < g.n_rho; ro += owned) {
            const int ro1 = min(ro + owned, g.n_rho), base = ro - 1, rows = ro1 - ro + 2;
            for (int i = threadIdx.x; i < rows * stride / 4; i += kSpillThreads)
                reinterpret_cast<uint4 *>(tile)[i] = make_uint4(0u, 0u, 0u, 0u);
            __syncthreads();
            spill_vote_slab<P>(tile, st, x, y, hb, he, cl, wrap, g, lane, bad, dup, max(ro - 1, 0),
                               min(ro1 + 1, g.n_rho), base);
            __syncthreads();
            f(SpillSlab<P>{tile}, jo, ro, ro1, base);
            __syncthreads();
        }
    }
}

__global__ __launch_bounds__(kSpillThreads) void k_spill(GridArgs g, BatchArgs a, SpillArgs sp) {
    extern __shared__ __align__(16) uint32_t spill_tile[];      // [kSpillSlabDwords]
    __shared__ float2 stage[kSpillWaves][64];
    __shared__ uint32_t s_event, s_flags, s_max, s_n, s_list[kSpillThreads], s_part[kSpillThreads];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int words = (g.n_rho + 31) / 32;
    uint32_t *dil = sp.work + (size_t)blockIdx.x * sp.stride;   // [words][n_theta]
    // Work items are (column, 32-row block) pairs, item it = block it / n_theta of column
    // it mod n_theta; the per-item arrays are stored in item order
    const int n_items = g.n_theta * words;
    uint32_t *pmask = dil + (size_t)words * g.n_theta;    // [n_items] each block's peak rows
    uint32_t *colpos = pmask + n_items;                   // [n_items] its first peak's place in its column
    uint32_t *colstart = colpos + n_items;                // [n_theta + 1] each column's first peak
    uint32_t *pcount = colstart + g.n_theta + 1;          // [n_items][16] its peaks' counts

    // Every value that steers control flow around a barrier is wave-uniform (scalar), and an
    // event that is skipped passes a barrier before it returns, as a processed one does at its
    // end.  Without that barrier the compiler sends the lanes other than thread 0 straight
    // from the return to the next event's first barrier (the counter read is thread 0's alone),
    // so a wave splits: thread 0's lane waits to take the counter while the rest of the wave,
    // and the other waves, go round the barriers again on the old event index.
    auto uni = [](uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); };
    auto process = [&](uint32_t e) {
        const uint32_t pe_id = uni(a.ids ? a.ids[e] : e);
        const uint32_t h0 = uni(a.offsets[pe_id]), h1 = uni(a.offsets[pe_id + 1]);
        if (h1 <= h0) {                      // malformed offsets: touch nothing but the counters
            if (threadIdx.x == 0) { a.n_peaks[e] = 0u; a.status[e] = h1 < h0 ? HOUGH_EV_TOO_MANY_HITS : 0u; }
            __syncthreads();
            return;
        }
        const uint32_t H = h1 - h0;
        uint8_t *ke = a.keep + (a.ids ? uni(a.keep_offsets[e]) : h0);
        const float *xe = a.x + h0, *ye = a.y + h0;
        // the duplicate pass marked later copies in the keep bytes of events up to kDedupMaxHits
        const bool dup = g.dedup && H <= kDedupMaxHits;
        if (threadIdx.x == 0) {
            s_flags = (g.dedup && H > kDedupMaxHits) ? HOUGH_EV_DEDUP_SKIPPED : 0u;
            s_max = 0u;
        }
        if (!dup)
            for (uint32_t i = threadIdx.x; i < H; i += kSpillThreads) ke[i] = 0u;
        for (size_t i = threadIdx.x; i < (size_t)words * g.n_theta; i += kSpillThreads) dil[i] = 0u;
        spill_sync();

        // steps 1-4 on chip, one slab at a time: vote, then the 3x3 test of every owned cell,
        // giving each (column, 32-row block) item its peak rows as a bit mask (stored in item
        // order: neighbouring threads take neighbouring columns) and its peaks' counts.
        // Only peak cells reach device memory (writing the whole accumulator out and walking it
        // there was three quarters of the path's time).  The relative threshold needs the
        // event's largest count first: one more round of votes.
        uint32_t bad = 0;
        uint32_t thr = g.threshold;
        const uint8_t *dupk = dup ? ke : nullptr;
        auto slabs = [&](auto packed) {
            constexpr bool P = decltype(packed)::value;
            if (a.frac_den) {
                spill_for_slabs<P>(spill_tile, &stage[wave][0], xe, ye, H, g, lane, wave, bad, dupk,
                                   [&](const SpillSlab<P> &sl, int, int ro, int ro1, int) {
                    uint32_t m = 0;
                    for (int i = threadIdx.x; i < (ro1 - ro + 2) * SpillSlab<P>::STRIDE; i += kSpillThreads) {
                        const uint32_t v = sl.tile[i];
                        m = max(m, P ? max(v & 0xffffu, v >> 16) : v);
                    }
                    m = wave_max(m);
                    if (lane == 0) atomicMax(&s_max, m);
                });
                const uint64_t rel = ((uint64_t)uni(s_max) * a.frac_num + a.frac_den - 1u) / a.frac_den;
                thr = (uint32_t)min<uint64_t>(max<uint64_t>(rel, g.threshold), 0x7fffffffull);
            }
            spill_for_slabs<P>(spill_tile, &stage[wave][0], xe, ye, H, g, lane, wave, bad, dupk,
                               [&](const SpillSlab<P> &sl, int jo, int ro, int ro1, int base) {
                const int nl = min(62, g.n_theta - jo), nb = (ro1 - ro + 31) / 32;
                for (int t = threadIdx.x; t < nl * nb; t += kSpillThreads) {
                    const int bs = t / nl, l = 1 + (t - bs * nl), j = jo + l - 1;
                    const int k0 = ro + 32 * bs, k1 = min(k0 + 32, ro1);
                    const int it = (k0 >> 5) * g.n_theta + j;
                    pmask[it] = spill_slab_peaks<P>(sl, l, j, k0, k1, base, thr, g, pcount + (size_t)it * 16);
                }
            });
        };
        if (H <= 65535u) slabs(std::true_type{});
        else slabs(std::false_type{});
        if (__ballot(bad != 0u) && lane == 0) atomicOr(&s_flags, HOUGH_EV_INVALID_HITS);
        spill_sync();
        // raster order is column-major with rows in order within a column: a thread per column
        // places each block's peaks within the column (neighbouring threads, neighbouring
        // columns: coalesced), then an exclusive prefix over the columns' totals (each thread
        // sums a run of columns, the runs' totals are scanned, then each run is scanned again)
        for (int j = threadIdx.x; j < g.n_theta; j += kSpillThreads) {
            uint32_t in_col = 0;
            for (int b = 0; b < words; ++b) {
                colpos[b * g.n_theta + j] = in_col;
                in_col += (uint32_t)__popc(pmask[b * g.n_theta + j]);
            }
            colstart[j] = in_col;
        }
        spill_sync();
        const int per = (g.n_theta + kSpillThreads - 1) / kSpillThreads;
        const int c0 = min((int)threadIdx.x * per, g.n_theta), c1 = min(c0 + per, g.n_theta);
        uint32_t part = 0;
        for (int j = c0; j < c1; ++j) part += colstart[j];
        s_part[threadIdx.x] = part;
        __syncthreads();
        if (threadIdx.x == 0) {
            uint32_t run = 0;
            for (int t = 0; t < kSpillThreads; ++t) {
                const uint32_t v = s_part[t];
                s_part[t] = run;
                run += v;
            }
            s_n = run;
        }
        __syncthreads();
        uint32_t run = s_part[threadIdx.x];
        for (int j = c0; j < c1; ++j) {
            const uint32_t v = colstart[j];
            colstart[j] = run;
            run += v;
        }
        spill_sync();
        // second pass: list each block's peaks in row order at its position, and mark the rows
        // within rho_window of each peak in the column's dilated bits (words other blocks of the
        // column may mark too: atomic ORs, in L2)
        hough_peak *pe = a.peaks ? a.peaks + (size_t)e * a.max_peaks : nullptr;
        const uint32_t cap = pe ? a.max_peaks : 0u;
        for (int it = threadIdx.x; it < n_items; it += kSpillThreads) {
            const int b = it / g.n_theta, j = it - b * g.n_theta;
            uint32_t pos = colstart[j] + colpos[it];
            const uint32_t *pc = pcount + (size_t)it * 16;
            uint32_t r = 0;
            for (uint32_t m = pmask[it]; m; m &= m - 1u) {
                const int k = 32 * b + (__ffs(m) - 1);
                if (pos < cap) store_peak(pe + pos, (uint32_t)j, (uint32_t)k, spill_load(pc + r));
                ++pos;
                ++r;
                const int lo = max(k - g.rho_window, 0), hi = min(k + g.rho_window, g.n_rho - 1);
                for (int wd = lo >> 5; wd <= (hi >> 5); ++wd) {
                    const int b0 = max(lo, wd * 32) - wd * 32, b1 = min(hi, wd * 32 + 31) - wd * 32;
                    const uint32_t msk = (b1 == 31 ? 0xffffffffu : ((1u << (b1 + 1)) - 1u)) & ~((1u << b0) - 1u);
                    __hip_atomic_fetch_or(dil + (size_t)wd * g.n_theta + j, msk, __ATOMIC_RELAXED,
                                          __HIP_MEMORY_SCOPE_AGENT);
                }
            }
        }
        spill_sync();

        // step 5, one 64-column group at a time: the group's dilated words are staged in LDS
        // (the vote's slab space), then each wave looks its hits, 64 at a time, up in every
        // column of the group (lane = column, the fused kernel's lookup); a hit kept by one
        // group is not looked up again.  Bit 0 of a keep byte is the verdict; a later copy's
        // bit 1 (duplicate pass) is dropped at the end.
        const uint32_t n_peaks = uni(s_n);
        if (n_peaks > 0) {
            const Lane<1, true> ln(lane);
            uint32_t unused = 0;
            for (int j0 = 0; j0 < g.n_theta; j0 += 64) {
                // [words + 1][64]: the extra zero row is where out-of-grid lanes look
                for (int q = threadIdx.x; q < (words + 1) * 64; q += kSpillThreads) {
                    const int w = q >> 6, c = j0 + (q & 63);
                    spill_tile[q] = (w < words && c < g.n_theta) ? spill_load(dil + (size_t)w * g.n_theta + c) : 0u;
                }
                __syncthreads();
                const Cols<1> cl = load_cols<1>(g, j0, lane, Lane<1, true>::STRIDE, ln.col);
                for (uint32_t base = (uint32_t)wave * 64; base < H; base += kSpillThreads) {
                    const uint32_t i = base + lane;
                    const uint32_t kv = i < H ? ke[i] : 1u;
                    const bool done = i < H && (kv & 1u);
                    if (__ballot(i < H && !done) == 0ull) continue;
                    int slot;
                    const StageCount n = stage_hits(&stage[wave][0], xe, ye, base, H, done, g, lane, unused, slot);
                    const uint64_t kept = lookup_staged<1, 64u>(spill_tile, &stage[wave][0], n, cl, lane, g.nrho_f);
                    if (slot >= 0 && ((kept >> slot) & 1ull)) ke[i] = (uint8_t)(kv | 1u);
                    wave_sync();
                }
                __syncthreads();
            }
            for (uint32_t i = threadIdx.x; i < H; i += kSpillThreads) ke[i] = (uint8_t)(ke[i] & 1u);
        } else if (dup) {
            for (uint32_t i = threadIdx.x; i < H; i += kSpillThreads) ke[i] = 0u;
        }
        spill_sync();
        if (threadIdx.x == 0) {
            a.n_peaks[e] = n_peaks;
            a.status[e] = s_flags | (n_peaks > a.max_peaks ? HOUGH_EV_PEAKS_TRUNCATED : 0u);
        }
        __syncthreads();
    };

    // after the split form: its slots and item counter back to zero, and the later copies' marks
    // (bit 1) out of the keep bytes of the events it processed
    if (sp.n_slots) {
        for (uint32_t i = blockIdx.x * kSpillThreads + threadIdx.x; i < sp.n_slots; i += gridDim.x * kSpillThreads)
            sp.slots[i] = 0u;
        if (blockIdx.x == 0 && threadIdx.x == 0) *a.queue = 0u;
        if (g.dedup) {
            // a workgroup per event, or as few waves each as it takes to have all events in hand at once
            // (a few workgroups one event after the other: 123 events of 8 hits, whole call, 29 us)
            uint32_t group = kSpillThreads;
            while (group > 64u && gridDim.x * (kSpillThreads / group) < a.n_events) group >>= 1;
            const uint32_t groups = kSpillThreads / group, mine = threadIdx.x / group, lane0 = threadIdx.x % group;
            for (uint32_t e = blockIdx.x * groups + mine; e < a.n_events; e += gridDim.x * groups) {
                const uint32_t pe_id = a.ids ? a.ids[e] : e, h0 = a.offsets[pe_id], h1 = a.offsets[pe_id + 1];
                if (h1 <= h0 || h1 - h0 > kDedupMaxHits) continue;
                uint8_t *ke = a.keep + (a.ids ? a.keep_offsets[e] : h0);
                for (uint32_t i0 = lane0; i0 < h1 - h0; i0 += 4u * group) {
                    uint32_t v[4];
#pragma unroll
                    for (uint32_t q = 0; q < 4u; ++q) v[q] = i0 + q * group < h1 - h0 ? ke[i0 + q * group] : 0u;
#pragma unroll
                    for (uint32_t q = 0; q < 4u; ++q)
                        if (v[q] & kKeepDuplicate) ke[i0 + q * group] = (uint8_t)(v[q] & 1u);
                }
            }
        }
    }
    if (sp.defer_count && blockIdx.x == 0 && threadIdx.x == 0) *sp.defer_count = 0u;   // (see BatchArgs)
    if (sp.all) {
        for (;;) {
            if (threadIdx.x == 0) s_event = atomicAdd(sp.queue, 1u);
            __syncthreads();
            const uint32_t e = uni(s_event);
            __syncthreads();
            if (e >= a.n_events) break;
            process(e);
        }
        if (threadIdx.x == 0 && atomicAdd(sp.queue + 1, 1u) == gridDim.x - 1u) {
            __hip_atomic_store(sp.queue, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(sp.queue + 1, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        return;
    }
    // only the events the fused or split kernel left (sp.queue[0] counts them; none: nothing to
    // scan): the workgroups take blocks of up to kSpillBlock events from a counter (sp.queue[2]) and
    // process the left ones of each block, so that a batch whose events mostly spill (a window
    // its events do not fit) keeps every workgroup busy.  A batch of fewer events than that many
    // per workgroup takes smaller blocks, down to an event each (14 events on 621 x 1702, all left
    // here: 2,384 us in blocks of four, 688 so).  The last workgroup to leave clears
    // the count and both counters.
    const uint32_t left = __hip_atomic_load(sp.queue, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (uni(left) == 0u) return;               // (and the counters stay at zero)
    const uint32_t block = min(max(a.n_events / gridDim.x, 1u), kSpillBlock);
    for (;;) {
        if (threadIdx.x == 0) {
            s_event = atomicAdd(sp.queue + 2, 1u);
            s_n = 0u;
        }
        __syncthreads();
        const uint32_t b0 = uni(s_event) * block;
        if (b0 >= a.n_events) break;                   // every thread leaves together
        const uint32_t e = b0 + threadIdx.x;
        if (threadIdx.x < block && e < a.n_events) {
            const uint32_t pe_id = a.ids ? a.ids[e] : e;
            const uint32_t h0 = a.offsets[pe_id], h1 = a.offsets[pe_id + 1];
            // left here by the fused kernel or the split form
            if ((a.status[e] & kStatusSpill) || (h1 >= h0 && h1 - h0 > kMaxBatchHits)) s_list[atomicAdd(&s_n, 1u)] = e;
        }
        __syncthreads();
        const uint32_t n = uni(s_n);
        for (uint32_t p = 0; p < n; ++p) process(uni(s_list[p]));   // events are independent: any order
        __syncthreads();
    }
    if (threadIdx.x == 0 && atomicAdd(sp.queue + 1, 1u) == gridDim.x - 1u) {
        __hip_atomic_store(sp.queue, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(sp.queue + 2, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(sp.queue + 1, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// ------------------------------------------------------------ duplicate pass (HOUGH_FLAG_DEDUP)
// One workgroup per event.  Open addressing in LDS keyed by the bits of (x, y): every slot ends
// holding the smallest event-local index of its key (compare-and-swap into an empty slot, atomic
// min into a slot of the same key), so after the inserts a hit is a later copy iff the slot of
// its key holds another index.  The table has at least twice as many slots as hits, so every
// probe sequence meets its key or an empty slot; entries never empty again, so a lookup finds
// its key before any empty slot.  The probe loops are bounded by the table size all the same.
constexpr int kDedupThreads = 512;
constexpr uint32_t kEmptySlot = 0xffffffffu;

// ------------------------------------------------------------------ largest-first schedule
// Size class of an event of H hits, non-decreasing in H: H itself below 64, else the octave
// of H and its next six bits (classes of 1/64 of an octave), at most 1727.  Malformed events
// (offsets decreasing) count as empty.
__device__ __forceinline__ uint32_t size_class(const uint32_t *offsets, uint32_t e) {
    const uint32_t h0 = offsets[e], h1 = offsets[e + 1];
    const uint32_t H = h1 >= h0 ? h1 - h0 : 0u;
    if (H < 64u) return H;
    const uint32_t lg = 31u - (uint32_t)__builtin_clz(H);
    return ((lg - 5u) << 6) | ((H >> (lg - 6u)) & 63u);
}

constexpr int kOrderThreads = 1024;
constexpr int kOrderClasses = 2048;

// One workgroup: count the events of each size class, turn the counts into the first queue
// position of each class (largest class first) and scatter the event indices there.  Within a
// class the order is whatever the LDS atomics give.
__global__ __launch_bounds__(kOrderThreads) void k_order(const uint32_t *__restrict__ offsets, uint32_t n_events,
                                                          uint32_t *__restrict__ order) {
    __shared__ uint32_t cnt[kOrderClasses];
    for (int i = threadIdx.x; i < kOrderClasses; i += kOrderThreads) cnt[i] = 0u;
    __syncthreads();
    for (uint32_t e = threadIdx.x; e < n_events; e += kOrderThreads)
        atomicAdd(&cnt[kOrderClasses - 1 - size_class(offsets, e)], 1u);
    __syncthreads();
    if (threadIdx.x < 64) {
        const int lane = threadIdx.x;
        uint32_t c[kOrderClasses / 64], sum = 0;
#pragma unroll
        for (int i = 0; i < kOrderClasses / 64; ++i) { c[i] = cnt[lane * (kOrderClasses / 64) + i]; sum += c[i]; }
        uint32_t start = wave_inclusive_scan(sum, lane) - sum;
#pragma unroll
        for (int i = 0; i < kOrderClasses / 64; ++i) {
            cnt[lane * (kOrderClasses / 64) + i] = start;
            start += c[i];
        }
    }
    __syncthreads();
    for (uint32_t e = threadIdx.x; e < n_events; e += kOrderThreads)
        order[atomicAdd(&cnt[kOrderClasses - 1 - size_class(offsets, e)], 1u)] = e;
}

__device__ __forceinline__ uint32_t dedup_hash(uint32_t kx, uint32_t ky) {
    uint32_t h = kx * 0x9e3779b1u;
    h ^= ky + 0x7f4a7c15u + (h << 6) + (h >> 2);
    h *= 0x85ebca6bu;
    return h ^ (h >> 16);
}

// Slot word: the index of the first copy seen so far (low kDedupIdxBits) under 18 bits of the
// key's hash, so that a probe that meets another key's slot is settled in LDS; only equal
// fingerprints read the two hits back to compare the keys.  Among entries of one key the high
// bits are equal, so an atomic minimum over the word is one over the index.
constexpr uint32_t kDedupIdxBits = 14;
constexpr uint32_t kDedupIdxMask = (1u << kDedupIdxBits) - 1u;
static_assert(kDedupMaxHits <= kDedupIdxMask, "hit indices must fit below the fingerprint");

__global__ __launch_bounds__(kDedupThreads) void k_dedup(BatchArgs a) {
    __shared__ uint32_t tab[kDedupSlots];
    const uint32_t e = blockIdx.x;
    const uint32_t pe_id = a.ids ? a.ids[e] : e;
    const uint32_t h0 = a.offsets[pe_id], h1 = a.offsets[pe_id + 1];
    if (h1 < h0) return;                                   // malformed: the batch kernel flags it
    const uint32_t H = h1 - h0;
    if (H == 0 || H > kMaxBatchHits) return;               // too many: the batch kernel zeroes keep
    uint8_t *ke = a.keep + (a.ids ? a.keep_offsets[e] : h0);
    const uint32_t *xb = reinterpret_cast<const uint32_t *>(a.x) + h0;
    const uint32_t *yb = reinterpret_cast<const uint32_t *>(a.y) + h0;
    if (H > kDedupMaxHits) {                               // every hit votes
        for (uint32_t i = threadIdx.x; i < H; i += kDedupThreads) ke[i] = 0u;
        return;
    }
    uint32_t slots = 64;
    while (slots < 2 * H) slots <<= 1;                     // <= kDedupSlots
    const uint32_t mask = slots - 1;
    for (uint32_t q = threadIdx.x; q < slots; q += kDedupThreads) tab[q] = kEmptySlot;
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < H; i += kDedupThreads) {
        const uint32_t kx = xb[i], ky = yb[i];
        const uint32_t hsh = dedup_hash(kx, ky);
        const uint32_t fp = hsh >> kDedupIdxBits, word = (fp << kDedupIdxBits) | i;
        uint32_t q = hsh & mask;
        for (uint32_t probe = 0; probe < slots; ++probe, q = (q + 1) & mask) {
            const uint32_t cur = atomicCAS(&tab[q], kEmptySlot, word);
            if (cur == kEmptySlot) break;                  // first of its key so far
            if ((cur >> kDedupIdxBits) == fp) {
                const uint32_t j = cur & kDedupIdxMask;
                if (xb[j] == kx && yb[j] == ky) {
                    atomicMin(&tab[q], word);
                    break;
                }
            }
        }
    }
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < H; i += kDedupThreads) {
        const uint32_t kx = xb[i], ky = yb[i];
        const uint32_t hsh = dedup_hash(kx, ky);
        const uint32_t fp = hsh >> kDedupIdxBits;
        uint32_t q = hsh & mask, first = i;
        for (uint32_t probe = 0; probe < slots; ++probe, q = (q + 1) & mask) {
            const uint32_t cur = tab[q];
            if (cur == kEmptySlot) break;                  // cannot happen: every key was inserted
            if ((cur >> kDedupIdxBits) != fp) continue;
            const uint32_t j = cur & kDedupIdxMask;
            if (j == i) break;                             // its own slot: the first copy
            if (xb[j] == kx && yb[j] == ky) {
                first = j;
                break;
            }
        }
        ke[i] = first != i ? kKeepDuplicate : (uint8_t)0;
    }
}

// hough_retain's LDS: the dilated bits and constants of a block of columns, at most 60 KB of them
// beside the 16 KB peak list, so that two workgroups share a CU (808 columns of 512 rows in one
// block, 438 of 1000).
constexpr int kRetainDilBytes = 60 * 1024;
int retain_cols_per_block(const GridArgs &g) {
    const size_t cols = (size_t)kRetainDilBytes / (retain_pitch(g.n_rho) * 4 + 8);
    return (int)std::min<size_t>(cols, (size_t)g.n_theta);
}
size_t retain_lds_bytes(const GridArgs &g, int cols) { return (size_t)cols * (retain_pitch(g.n_rho) * 4 + 8); }

constexpr int kVoteWaves = 16;
constexpr int kPeakWaves = kPeakRowsPerBlock;

// The dynamic-LDS limit is a per-kernel, process-wide attribute: every kernel is allowed the
// device maximum (less room for its static LDS) so that contexts with different grids, possibly
// on different host threads, never lower each other's limit.
template <typename K>
void allow_lds(K kernel) {
    int dev = 0, lim = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&lim, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess)
        return;
    (void)hipFuncSetAttribute(reinterpret_cast<const void *>(kernel),
                              hipFuncAttributeMaxDynamicSharedMemorySize, lim - 256);
}

}  // namespace

int vote_slab_rows(int n_rho, size_t lds_limit) {
    const size_t fixed = (size_t)kVoteWaves * kStageBytes + 256 + 256;    // slack
    if (lds_limit <= fixed + 2 * 128) return 0;
    const long rows = (long)((lds_limit - fixed) / 128) - 1;
    return (int)(rows < n_rho ? rows - rows % 4 : n_rho);      // whole quads of rows per slab
}

size_t peaks_lds_bytes(int n_rho, int waves) {
    return (size_t)waves * ((n_rho + 63) / 64) * 8 + (size_t)(waves + 2) * n_rho * 4;
}

// Few rows per workgroup share one event's rows over more of the chip; every workgroup adds up all
// their counts and stages two halo rows, so grids of many columns take more (both launches, us at 4, 8
// and 16 rows: 360 x 256 8.4, 8.4, 9.2; 1000 x 1000 19.2, 18.8, 20.2; 2000 x 100 8.7, 7.5, 7.4; 4000 x
// 250 13.7, 11.4, 10.4; 4000 x 2000 72, 67, 38; 9000 x 100 22, 17, 15; 65535 x 8 273, 152, 76).
int peak_block_waves(int n_theta, int n_rho, size_t lds_limit) {
    for (int w = n_theta <= 512 ? 4 : (n_theta <= 2048 ? 8 : kPeakWaves); w >= 2; w >>= 1)
        if (peaks_lds_bytes(n_rho, w) + 512 <= lds_limit) return w;
    return 0;
}

// The fused kernel's dynamic LDS: the packed tile with its dummy row (a windowed tile: `win`
// rows, a zero halo row on each side and the dummy row), the wave stages, the peak and dilated
// words, the tile's peak list and the per-column peak counts.
size_t batch_lds_bytes(int n_rho, int waves, int groups, int win, bool sparse) {
    const size_t tw = 64u * groups;
    const size_t rows = win ? (size_t)win + 3 : (size_t)n_rho + 1;
    const size_t nwords = win ? (size_t)win / 32 + 1 : (size_t)(n_rho + 31) / 32;
    const size_t stages = (size_t)waves * kStageBytes, peak_words = nwords * tw * 4;
    return rows * (tw / 2) * 4 + (win ? stages + peak_words : std::max(stages, peak_words)) + (nwords + 1) * (tw + 1) * 4 +
           (sparse ? kTilePeaks * sizeof(float4) : 0) + tw * 4;
}

int plan_batch(int n_theta, int n_rho, int waves, int groups, size_t lds_limit, BatchPlan *out, int win) {
    if (!(waves == 4 || waves == 6 || waves == 8 || waves == 12 || waves == 16) || !(groups == 1 || groups == 2)) return -1;
    // a window is a whole number of 32-row words, one column group, shorter than the grid
    if (win != 0 && (groups != 1 || win < 32 || win % 32 != 0 || win >= n_rho)) return -1;
    BatchPlan p{};
    p.waves = waves;
    p.groups = groups;
    p.tile_cols = 64 * groups;
    p.out_cols = p.tile_cols - 2;
    p.n_tiles = (n_theta + p.out_cols - 1) / p.out_cols;
    p.win = win;
    p.sparse = n_rho >= kSparseRhoRows ? 1 : 0;
    p.lds_bytes = batch_lds_bytes(n_rho, waves, groups, win, p.sparse != 0);
    p.sp_lds_bytes = batch_lds_bytes(n_rho, waves, groups, win, true);
    if (p.sp_lds_bytes + 256 > lds_limit) return -1;     // (room for the kernel's static LDS)
    p.grid = 0;
    *out = p;
    return 0;
}

hipError_t launch_order(const uint32_t *offsets, uint32_t n_events, uint32_t *order, hipStream_t s) {
    if (n_events == 0) return hipSuccess;
    hipLaunchKernelGGL(k_order, dim3(1), dim3(kOrderThreads), 0, s, offsets, n_events, order);
    return hipGetLastError();
}

size_t spill_stride(int n_theta, int n_rho) {
    const size_t words = (size_t)(n_rho + 31) / 32;
    // dilated words, per (column, 32-row block) a peak-row mask and the place of its first peak
    // within the column, per column the place of its first peak (and the end), per (column,
    // block) the counts of its at most 16 peaks
    const size_t n = 3 * words * n_theta + n_theta + 1 + 16 * words * n_theta;
    return (n + 63) & ~(size_t)63;                  // each workgroup's slice on a 256-byte boundary
}

hipError_t launch_spill(const GridArgs &g, const BatchArgs &a, const SpillArgs &sp, int n_wg, hipStream_t s) {
    if (a.n_events == 0 || n_wg < 1) return hipSuccess;
    // the slab's dynamic LDS beside the kernel's 16 KB of static LDS (allow_lds's limit would
    // not leave room for that); the slab doubles as the retention step's [words + 1][64]
    // dilated words (at most 257 * 64 dwords)
    constexpr int kBytes = kSpillSlabDwords * (int)sizeof(uint32_t);
    static const hipError_t lds_ok = hipFuncSetAttribute(reinterpret_cast<const void *>(k_spill),
                                                         hipFuncAttributeMaxDynamicSharedMemorySize, kBytes);
    if (lds_ok != hipSuccess) return lds_ok;
    if (((size_t)(g.n_rho + 31) / 32 + 1) * 64u > (size_t)kSpillSlabDwords) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_spill, dim3(n_wg), dim3(kSpillThreads), (size_t)kBytes, s, g, a, sp);
    return hipGetLastError();
}

hipError_t launch_dedup(const BatchArgs &a, hipStream_t s) {
    if (a.n_events == 0) return hipSuccess;
    hipLaunchKernelGGL(k_dedup, dim3(a.n_events), dim3(kDedupThreads), 0, s, a);
    return hipGetLastError();
}

template <typename T>
static hipError_t launch_vote_t(const GridArgs &g, const float *x, const float *y, uint32_t n_hits, T *acc,
                                hipStream_t s) {
    static const bool lds_ok = (allow_lds(k_vote<kVoteWaves, T>), true);
    (void)lds_ok;
    const int groups = (g.n_theta + 31) / 32, slabs = (g.n_rho + g.vote_rows - 1) / g.vote_rows;
    // four cells per store where every column's (and slab's) first cell is aligned for it
    const int vec = g.n_rho % 4 == 0 && (slabs == 1 || g.vote_rows % 4 == 0) &&
                    (uintptr_t)acc % (4 * sizeof(T)) == 0;
    hipLaunchKernelGGL((k_vote<kVoteWaves, T>), dim3(groups, slabs), dim3(kVoteWaves * 64),
                       (size_t)(g.vote_rows + 1) * 128, s, g, x, y, n_hits, acc, g.vote_rows, vec);
    return hipGetLastError();
}

hipError_t launch_vote(const GridArgs &g, const float *x, const float *y, uint32_t n_hits,
                       void *acc, int acc_type, hipStream_t s) {
    if (g.vote_rows < 1) return hipErrorInvalidValue;
    return acc_type == HOUGH_ACC_U16 ? launch_vote_t(g, x, y, n_hits, static_cast<uint16_t *>(acc), s)
                                     : launch_vote_t(g, x, y, n_hits, static_cast<uint32_t *>(acc), s);
}

template <int NW, typename T>
static void launch_peaks_t(const GridArgs &g, const T *acc, hough_peak *peaks, uint32_t cap, uint32_t *n_peaks,
                           uint32_t *counts, hipStream_t s) {
    static const bool lds_ok = (allow_lds(k_peaks<NW, T, false>), allow_lds(k_peaks<NW, T, true>), true);
    (void)lds_ok;
    const size_t lds = peaks_lds_bytes(g.n_rho, NW);
    const int blocks = (g.n_theta + NW - 1) / NW;
    hipLaunchKernelGGL((k_peaks<NW, T, false>), dim3(blocks), dim3(NW * 64), lds, s, g, acc, peaks, cap, n_peaks,
                       counts);
    hipLaunchKernelGGL((k_peaks<NW, T, true>), dim3(blocks), dim3(NW * 64), lds, s, g, acc, peaks, cap, n_peaks,
                       counts);
}

template <typename T>
static hipError_t launch_peaks_w(const GridArgs &g, const T *acc, hough_peak *peaks, uint32_t cap,
                                 uint32_t *n_peaks, uint32_t *counts, hipStream_t s) {
    switch (g.peak_waves) {
        case 16: launch_peaks_t<16, T>(g, acc, peaks, cap, n_peaks, counts, s); break;
        case 8: launch_peaks_t<8, T>(g, acc, peaks, cap, n_peaks, counts, s); break;
        case 4: launch_peaks_t<4, T>(g, acc, peaks, cap, n_peaks, counts, s); break;
        case 2: launch_peaks_t<2, T>(g, acc, peaks, cap, n_peaks, counts, s); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// hough_peaks: workgroups of g.peak_waves theta rows (fewer for tall grids, whose rows take
// more LDS); counts holds one counter per workgroup.
hipError_t launch_peaks(const GridArgs &g, const void *acc, int acc_type, hough_peak *peaks,
                        uint32_t cap, uint32_t *n_peaks, uint32_t *counts, hipStream_t s) {
    if (acc_type == HOUGH_ACC_U16)
        return launch_peaks_w<uint16_t>(g, static_cast<const uint16_t *>(acc), peaks, cap, n_peaks, counts, s);
    return launch_peaks_w<uint32_t>(g, static_cast<const uint32_t *>(acc), peaks, cap, n_peaks, counts, s);
}

// Key buffer and bitmap placement of the iterative finder: the largest key buffer (a power of two
// of kIterMinKeys .. kIterMaxKeys keys) that fits beside an LDS bitmap of the grid, with room for
// `per_cu` workgroups per CU when that leaves at least 4096 keys, else one; a grid whose bitmap
// does not fit beside kIterMinKeys keys keeps it in device memory.
// The batch form also keeps a word per 64-column tile; where that does not fit beside a bitmap, the
// key buffer gives way.
static size_t iter_tile_bytes(int n_theta) { return ((size_t)((n_theta + 63) / 64 + 1) * 4 + 15) & ~(size_t)15; }

IterPlan plan_iterative_batch(int n_theta, int n_rho, size_t lds_limit, int per_cu) {
    IterPlan p = plan_iterative(n_theta, n_rho, lds_limit, per_cu);
    while (p.keys > 256 && p.lds_bytes + iter_tile_bytes(n_theta) + 512 > lds_limit) {
        p.lds_bytes -= (size_t)p.keys * 4;
        p.keys >>= 1;
    }
    return p;
}

IterPlan plan_iterative(int n_theta, int n_rho, size_t lds_limit, int per_cu) {
    IterPlan p{};
    const size_t cells = (size_t)n_theta * (size_t)n_rho;
    p.bm_bytes = (cells + 31) / 32 * 4;
    const size_t room = lds_limit > 1024 ? lds_limit - 1024 : 0;      // static LDS and slack
    const size_t bm_lds = (p.bm_bytes + 15) & ~(size_t)15;
    for (int pc = per_cu; pc >= 1; --pc) {
        const uint32_t min_keys = pc > 1 ? 4096u : kIterMinKeys;
        for (uint32_t k = kIterMaxKeys; k >= min_keys; k >>= 1) {
            if ((size_t)pc * ((size_t)k * 8 + bm_lds) <= room) {
                p.keys = k;
                p.gbm = 0;
                p.lds_bytes = (size_t)k * 8 + bm_lds;
                return p;
            }
        }
    }
    for (uint32_t k = kIterMaxKeys; k >= kIterMinKeys; k >>= 1) {
        if ((size_t)per_cu * (size_t)k * 8 <= room || k == kIterMinKeys) {
            p.keys = k;
            break;
        }
    }
    p.gbm = 1;
    p.lds_bytes = (size_t)p.keys * 8;
    return p;
}

template <typename T, bool GBM, bool BATCH, bool LIST>
static void launch_iter_t(const GridArgs &g, const T *acc, uint32_t frac_num, uint32_t frac_den, int r_theta,
                          int r_rho, hough_peak *peaks, uint32_t cap, uint32_t *n_peaks, uint32_t *status,
                          const uint32_t *offsets, uint32_t n_blocks, const IterPlan &ip, uint32_t *gbm,
                          const uint64_t *list, uint32_t *scan, const uint2 *head, hipStream_t s) {
    const size_t lds = ip.lds_bytes + (BATCH ? iter_tile_bytes(g.n_theta) : 0);
    static const bool lds_ok = (allow_lds(k_peaks_iter<T, GBM, BATCH, LIST>), true);
    (void)lds_ok;
    hipLaunchKernelGGL((k_peaks_iter<T, GBM, BATCH, LIST>), dim3(n_blocks), dim3(kIterThreads), lds, s, g, acc, frac_num,
                       frac_den, r_theta, r_rho, peaks, cap, n_peaks, status, offsets, ip.keys, GBM ? gbm : nullptr,
                       list, scan, head);
}

// The finder reads an accumulator of up to this many cells by itself: that costs less than a launch ahead
// of it (us listed / by itself, threshold of half the maximum: 10 x 12 11.4 / 8.7, 95 x 60 of a 100-hit
// event 36.5 / 33.8 and of 20,000 hits 25.4 / 24.5, 90 x 100 37.4 / 35.2 and 17.1 / 17.9, 96 x 128 33.5 / 31.9
// and 11.6 / 13.5).
constexpr uint32_t kIterDirectCells = 8192;

template <typename T>
static void launch_iter_one(const GridArgs &g, const T *acc, uint32_t frac_num, uint32_t frac_den, int r_theta,
                            int r_rho, hough_peak *peaks, uint32_t cap, uint32_t *n_peaks, uint32_t *status,
                            const IterPlan &ip, uint32_t *gbm, uint64_t *list, uint32_t *scan, hipStream_t s) {
    const uint32_t cells = (uint32_t)g.n_theta * (uint32_t)g.n_rho, tile = kScanThreads * kScanCells;
    if (cells <= kIterDirectCells && !ip.gbm) {
        launch_iter_t<T, false, false, false>(g, acc, frac_num, frac_den, r_theta, r_rho, peaks, cap, n_peaks, status,
                                              nullptr, 1u, ip, nullptr, nullptr, nullptr, nullptr, s);
        return;
    }
    hipLaunchKernelGGL(k_iter_scan<T>, dim3(std::min((cells + tile - 1u) / tile, 1024u)), dim3(kScanThreads), 0, s,
                       acc, cells, g.threshold, frac_num, frac_den, list, scan);
    const auto finder = ip.gbm ? launch_iter_t<T, true, false, true> : launch_iter_t<T, false, false, true>;
    finder(g, acc, frac_num, frac_den, r_theta, r_rho, peaks, cap, n_peaks, status, nullptr, 1u, ip, gbm, list, scan,
           nullptr, s);
}

hipError_t launch_peaks_iterative(const GridArgs &g, const void *acc, int acc_type, uint32_t frac_num,
                                  uint32_t frac_den, int r_theta, int r_rho, hough_peak *peaks,
                                  uint32_t cap, uint32_t *n_peaks, uint32_t *status, const IterPlan &ip,
                                  uint32_t *gbm, uint64_t *list, uint32_t *scan, hipStream_t s) {
    if (acc_type == HOUGH_ACC_U16)
        launch_iter_one<uint16_t>(g, static_cast<const uint16_t *>(acc), frac_num, frac_den, r_theta, r_rho, peaks,
                                  cap, n_peaks, status, ip, gbm, list, scan, s);
    else
        launch_iter_one<uint32_t>(g, static_cast<const uint32_t *>(acc), frac_num, frac_den, r_theta, r_rho, peaks,
                                  cap, n_peaks, status, ip, gbm, list, scan, s);
    return hipGetLastError();
}

hipError_t launch_track_params(const GridArgs &g, const float *x, const float *y, uint32_t n_hits,
                               const hough_peak *peaks, const uint32_t *n_peaks, uint32_t cap,
                               double rho_min, double rho_max, double b_tesla, hough_track *out,
                               hipStream_t s) {
    if (cap == 0) return hipSuccess;
    hipLaunchKernelGGL(k_track_params, dim3(std::min(cap, 2048u)), dim3(kTrackWaves * 64), 0, s, g, x, y, n_hits, peaks,
                       n_peaks, cap, rho_min, rho_max, b_tesla, out);
    return hipGetLastError();
}

template <int SHARE>
static hipError_t launch_retain_t(const GridArgs &g, const float *x, const float *y, uint32_t n_hits, uint32_t chunks,
                                  const hough_peak *peaks, const uint32_t *n_peaks, uint32_t cap, uint8_t *keep,
                                  int n_cu, hipStream_t s) {
    const int cols = retain_cols_per_block(g);
    static const hipError_t lds_ok = hipFuncSetAttribute(reinterpret_cast<const void *>(k_retain<SHARE>),
                                                         hipFuncAttributeMaxDynamicSharedMemorySize, kRetainDilBytes);
    if (lds_ok != hipSuccess) return lds_ok;
    constexpr uint32_t per = kRetainWaves / SHARE;
    const uint32_t blocks = std::min(chunks / per + (chunks % per != 0u), 2u * (uint32_t)n_cu);
    hipLaunchKernelGGL(k_retain<SHARE>, dim3(1, blocks), dim3(kRetainWaves * 64), retain_lds_bytes(g, cols), s, g, x, y,
                       n_hits, peaks, n_peaks, cap, keep, cols, nullptr);
    return hipGetLastError();
}

// As many waves share 64 hits as leave at most one workgroup per CU; where one wave each leaves more,
// two workgroups per CU take several chunks per built block.  A lookup reads LDS at random words, so
// the columns looked at cost the time, and a wave that has all of them stops early.  us at 16, 8, 4, 2
// and 1 waves per 64 hits on 256 CUs, 720 x 512 with 4,000 to 9,000 peaks: 8,000 hits 10, 13, 20, 33, 22;
// 32,000: 22, 17, 24, 35, 18; 64,000: 31, 31, 25, 36, 15; 256,000: 84, 78, 76, 74, 18; 1,000,000: 281,
// 259, 245, 234, 56.  1000 x 1000, 17,000 to 22,000 peaks (waves stop late): 26, 30, 39, 58, 94; 53, 33,
// 42, 60, 93; 71, 63, 44, 61, 96; 160, 132, 124, 119, 92; 508, 396, 374, 339, 242.  The line between two
// and one lies where the second grid still gains by sharing (128,000: 63 and 90, the first 37 and 15).
hipError_t launch_retain(const GridArgs &g, const float *x, const float *y, uint32_t n_hits,
                         const hough_peak *peaks, const uint32_t *n_peaks, uint32_t cap,
                         uint8_t *keep, int n_cu, hipStream_t s) {
    if (n_hits == 0) return hipSuccess;
    const uint32_t chunks = n_hits / 64u + (n_hits % 64u != 0u), cu = (uint32_t)n_cu;
    if (chunks <= cu) return launch_retain_t<16>(g, x, y, n_hits, chunks, peaks, n_peaks, cap, keep, n_cu, s);
    if (chunks <= 2 * cu) return launch_retain_t<8>(g, x, y, n_hits, chunks, peaks, n_peaks, cap, keep, n_cu, s);
    if (chunks <= 4 * cu) return launch_retain_t<4>(g, x, y, n_hits, chunks, peaks, n_peaks, cap, keep, n_cu, s);
    if (chunks <= 8 * cu) return launch_retain_t<2>(g, x, y, n_hits, chunks, peaks, n_peaks, cap, keep, n_cu, s);
    return launch_retain_t<1>(g, x, y, n_hits, chunks, peaks, n_peaks, cap, keep, n_cu, s);
}

// The iterative finder's batch form: (duplicate pass), votes into each tile's candidates (or
// cells), the finder, and retention with each event's first `cap` peaks; as many events at a time as
// the heads have room for.
// Rows of a tile held at a time: two workgroups per CU, or one with twice the rows where every (event,
// tile) has a CU to itself anyway, so that fewer sweeps of the hits and fewer stores of the cells are made
// (the whole call with 600 / 1,216 rows: 128 events of 1,500 hits on 63 x 1271 47 / 29 us, 40 on 360 x 2000 119 / 63,
// 16 of 100 hits that reach every row of 1000 x 1000 134 / 44, 4 on 17 x 1110 25 / 18; where 600 rows hold
// what the hits reach the two are equal).
constexpr int kIterSlabRows = 600, kIterTallRows = 1216;
constexpr int kIterVoteWaves = 8;
hipError_t launch_batch_iterative(const GridArgs &g, const BatchArgs &a, uint16_t *acc, uint32_t frac_num,
                                  uint32_t frac_den, int r_theta, int r_rho, const IterPlan &ip, uint32_t *gbm,
                                  void *head, int n_cu, hipStream_t s) {
    if (a.n_events == 0) return hipSuccess;
    hipError_t e = hipSuccess;
    if (g.dedup) {
        e = launch_dedup(a, s);
        if (e != hipSuccess) return e;
    }
    static const hipError_t vote_ok =
        hipFuncSetAttribute(reinterpret_cast<const void *>(k_vote_batch<kIterVoteWaves>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (kIterTallRows + 1) * 128);
    static const hipError_t retain_ok = hipFuncSetAttribute(reinterpret_cast<const void *>(k_retain<1>),
                                                            hipFuncAttributeMaxDynamicSharedMemorySize, kRetainDilBytes);
    if (vote_ok != hipSuccess) return vote_ok;
    if (retain_ok != hipSuccess) return retain_ok;
    const size_t cells = (size_t)g.n_theta * (size_t)g.n_rho;
    const uint32_t tiles = (uint32_t)(g.n_theta + 63) / 64u, most_events = kIterHeads / tiles;
    const int cols = retain_cols_per_block(g);
    const uint32_t most_blocks = (kMaxBatchHits + kRetainWaves * 64 - 1) / (kRetainWaves * 64);
    for (uint32_t e0 = 0; e0 < a.n_events; e0 += most_events) {
        const uint32_t n = std::min(most_events, a.n_events - e0);
        const int rows = std::min(g.n_rho, n * tiles <= (uint32_t)n_cu ? kIterTallRows : kIterSlabRows);
        const uint32_t *off = a.offsets + e0;
        hough_peak *peaks = a.peaks ? a.peaks + (size_t)e0 * a.max_peaks : nullptr;
        uint16_t *part = acc + e0 * cells;
        uint32_t *bm = gbm ? gbm + e0 * (ip.bm_bytes / 4) : nullptr;
        hipLaunchKernelGGL(k_vote_batch<kIterVoteWaves>, dim3(n, tiles), dim3(kIterVoteWaves * 64), (size_t)(rows + 1) * 128, s,
                           g, a.x, a.y, off, part, a.keep, a.status + e0, rows, frac_num, frac_den,
                           static_cast<uint2 *>(head));
        if ((e = hipGetLastError()) != hipSuccess) return e;
        const auto finder = ip.gbm ? launch_iter_t<uint16_t, true, true, false> : launch_iter_t<uint16_t, false, true, false>;
        finder(g, part, frac_num, frac_den, r_theta, r_rho, peaks, a.max_peaks, a.n_peaks + e0, a.status + e0, off, n, ip,
               bm, nullptr, nullptr, static_cast<const uint2 *>(head), s);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        // a few events: several workgroups each, up to the largest event's chunks
        const uint32_t blocks = std::max(1u, std::min(most_blocks, 512u / n));
        hipLaunchKernelGGL(k_retain<1>, dim3(n, blocks), dim3(kRetainWaves * 64), retain_lds_bytes(g, cols), s, g,
                           a.x, a.y, 0u, peaks, a.n_peaks + e0, a.max_peaks, a.keep, cols, off);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return e;
}

// Windowed tiles on theta-periodic grids: only the shapes the library picks by itself.
constexpr bool window_periodic(int waves) { return waves == 8 || waves == 16; }

template <int NW, int G, bool SP>
static void launch_batch_sp(const GridArgs &g, const BatchPlan &p, const BatchArgs &a, hipStream_t s) {
    const int nwords = (g.n_rho + 31) / 32;
    const size_t lds = SP ? p.sp_lds_bytes : p.lds_bytes;
    if constexpr (G == 1) {
        if (p.win) {
            if constexpr (window_periodic(NW))
                if (g.periodic) {
                    hipLaunchKernelGGL((k_batch<NW, G, true, SP, true>), dim3(p.grid), dim3(NW * 64), lds, s, g,
                                       a, p.n_tiles, nwords, p.win);
                    return;
                }
            hipLaunchKernelGGL((k_batch<NW, G, false, SP, true>), dim3(p.grid), dim3(NW * 64), lds, s, g, a,
                               p.n_tiles, nwords, p.win);
            return;
        }
    }
    if (g.periodic)
        hipLaunchKernelGGL((k_batch<NW, G, true, SP, false>), dim3(p.grid), dim3(NW * 64), lds, s, g, a,
                           p.n_tiles, nwords, 0);
    else
        hipLaunchKernelGGL((k_batch<NW, G, false, SP, false>), dim3(p.grid), dim3(NW * 64), lds, s, g, a,
                           p.n_tiles, nwords, 0);
}

template <int NW, int G>
static hipError_t launch_batch_t(const GridArgs &g, const BatchPlan &p, const BatchArgs &a,
                                 hipStream_t s) {
    if (p.win && (G != 1 || (g.periodic && !window_periodic(NW)))) return hipErrorInvalidValue;   // no such plan is made
    // a relative threshold leaves few peaks per tile whatever the grid
    if (p.sparse || a.frac_den != 0u)
        launch_batch_sp<NW, G, true>(g, p, a, s);
    else
        launch_batch_sp<NW, G, false>(g, p, a, s);
    return hipGetLastError();
}

hipError_t launch_batch(const GridArgs &g, const BatchPlan &p, const BatchArgs &a, hipStream_t s) {
    switch (p.waves * 10 + p.groups) {
        case 41: return launch_batch_t<4, 1>(g, p, a, s);
        case 42: return launch_batch_t<4, 2>(g, p, a, s);
        case 61: return launch_batch_t<6, 1>(g, p, a, s);
        case 62: return launch_batch_t<6, 2>(g, p, a, s);
        case 81: return launch_batch_t<8, 1>(g, p, a, s);
        case 82: return launch_batch_t<8, 2>(g, p, a, s);
        case 121: return launch_batch_t<12, 1>(g, p, a, s);
        case 122: return launch_batch_t<12, 2>(g, p, a, s);
        case 161: return launch_batch_t<16, 1>(g, p, a, s);
        case 162: return launch_batch_t<16, 2>(g, p, a, s);
        default: return hipErrorInvalidValue;
    }
}

// (a window that leaves room for one workgroup per CU wants the most waves)
constexpr int kSplitWinWaves = 16;
// LDS of the split kernel on windows of `win` rows.
static size_t split_window_lds(int waves, int win) {
    const size_t nwp = (size_t)win / 32 + 1;
    return ((size_t)win + 3) * 128 + std::max((size_t)waves * kStageBytes, nwp * 256) + kTilePeaks * sizeof(float4) + 256 +
           (nwp + 1) * kDilPitch<1> * 4;
}

template <int NW, bool WIN>
static hipError_t launch_split_t(const GridArgs &g, const BatchArgs &a, const SplitArgs &sp, uint32_t items, int win,
                                 hipStream_t s) {
    const int nwords = (g.n_rho + 31) / 32;
    const size_t lds = WIN ? split_window_lds(NW, win) : batch_lds_bytes(g.n_rho, NW, 1, 0, true);
    // one workgroup per item; a launch holds at most 2^31 threads, and the item counter runs on
    // from launch to launch
    for (uint32_t left = items; left > 0;) {
        const uint32_t n = std::min(left, 1u << 21);
        left -= n;
        if (g.periodic)
            hipLaunchKernelGGL((k_batch_split<NW, true, WIN>), dim3(n), dim3(NW * 64), lds, s, g, a, sp, nwords, win);
        else
            hipLaunchKernelGGL((k_batch_split<NW, false, WIN>), dim3(n), dim3(NW * 64), lds, s, g, a, sp, nwords, win);
    }
    return hipGetLastError();
}

uint32_t split_tiles(int n_theta) { return (uint32_t)(n_theta + 61) / 62u; }

hipError_t launch_batch_split(const GridArgs &g, const SplitPlan &p, const BatchArgs &a, const SplitArgs &sp,
                              int n_cu, hipStream_t s) {
    const uint32_t items = a.n_events * sp.n_tiles;
    // up to one item per CU the widest workgroup finishes its item first; beyond that narrower ones
    // share a CU and overlap their phases
    if (p.win) return launch_split_t<kSplitWinWaves, true>(g, a, sp, items, p.win, s);
    switch (items <= (uint32_t)n_cu ? p.wide : p.narrow) {
        case 16: return launch_split_t<16, false>(g, a, sp, items, 0, s);
        case 12: return launch_split_t<12, false>(g, a, sp, items, 0, s);
        case 8: return launch_split_t<8, false>(g, a, sp, items, 0, s);
        case 4: return launch_split_t<4, false>(g, a, sp, items, 0, s);
        default: return hipErrorInvalidValue;
    }
}

template <int NW>
static bool split_fits(int n_rho, size_t lds_limit) {
    if (batch_lds_bytes(n_rho, NW, 1, 0, true) + 256 > lds_limit) return false;
    allow_lds(k_batch_split<NW, false, false>);
    allow_lds(k_batch_split<NW, true, false>);
    return true;
}

SplitPlan plan_split_window(int win, size_t lds_limit) {
    SplitPlan p{0, 0, 0};
    if (win == 0 || split_window_lds(kSplitWinWaves, win) + 256 > lds_limit) return p;
    allow_lds(k_batch_split<kSplitWinWaves, false, true>);
    allow_lds(k_batch_split<kSplitWinWaves, true, true>);
    p.win = win;
    return p;
}

SplitPlan plan_split(int n_rho, size_t lds_limit) {
    SplitPlan p{0, 0, 0};
    if (split_fits<4>(n_rho, lds_limit)) p.wide = p.narrow = 4;
    if (split_fits<8>(n_rho, lds_limit)) p.wide = p.narrow = 8;
    // two workgroups per CU but not three: 12 waves each
    if (3 * batch_lds_bytes(n_rho, 8, 1, 0, true) > lds_limit && 2 * (batch_lds_bytes(n_rho, 12, 1, 0, true) + 256) <= lds_limit &&
        split_fits<12>(n_rho, lds_limit))
        p.narrow = 12;
    if (split_fits<16>(n_rho, lds_limit)) {
        p.wide = 16;
        if (2 * batch_lds_bytes(n_rho, 8, 1, 0, true) > lds_limit) p.narrow = 16;   // one per CU either way
    }
    return p;
}

// Workspace size of the split form.  The kernel needs one 4-byte slot per tile, at the workspace's start;
// the size, and with it the largest batch of the static form, is part of the interface and stays what it
// was when every tile's list (up to a peak in a quarter of the tile's cells), the events' keep bits and
// two words per event lay there too, each section on a 256-byte boundary.
size_t split_workspace_bytes(int n_theta, int n_rho, int groups, uint32_t n_events) {
    const size_t E = n_events, cols = 64u * (size_t)groups - 2u, tiles = ((size_t)n_theta + cols - 1u) / cols;
    const size_t list = ((cols + 1u) / 2u) * (((size_t)n_rho + 1u) / 2u) * sizeof(hough_peak);
    const size_t keep_words = (kMaxBatchHits + 31) / 32 + 1;
    auto section = [](size_t v) { return (v + 255) & ~(size_t)255; };
    return section(E * tiles * 4) + section(E * tiles * list) + section(E * keep_words * 4) + 2 * section(E * 4);
}

bool split_layout(int n_theta, int n_rho, int groups, uint32_t n_events, void *ws, size_t bytes,
                  SplitArgs *out) {
    if (!ws || bytes < split_workspace_bytes(n_theta, n_rho, groups, n_events) || ((uintptr_t)ws & 255u) != 0)
        return false;
    const uint32_t tiles = split_tiles(n_theta);
    if (bytes / 4 < (size_t)n_events * tiles) return false;
    out->n_tiles = tiles;
    out->slots = static_cast<uint32_t *>(ws);
    return true;
}

template <typename K>
static int occupancy(K kernel, int threads, size_t lds) {
    int n = 0;
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kernel, threads, lds) == hipSuccess ? n : 0;
}

template <int NW, int G>
static int prepare_t(BatchPlan *p) {
    // both grid topologies: a context's plan serves whichever kernel it launches.  The workgroups per
    // CU are those of the kernels its plain launches run; a relative launch on a grid that is
    // not sparse needs the peak list's LDS as well and may hold fewer at a time.
    allow_lds(k_batch<NW, G, false, false, false>);
    allow_lds(k_batch<NW, G, true, false, false>);
    allow_lds(k_batch<NW, G, false, true, false>);
    allow_lds(k_batch<NW, G, true, true, false>);
    const int T = NW * 64;
    if constexpr (G == 1) {
        if (p->win && p->periodic) {
            if constexpr (window_periodic(NW)) {
                allow_lds(k_batch<NW, 1, true, false, true>);
                allow_lds(k_batch<NW, 1, true, true, true>);
                return p->sparse ? occupancy(k_batch<NW, 1, true, true, true>, T, p->lds_bytes)
                                 : occupancy(k_batch<NW, 1, true, false, true>, T, p->lds_bytes);
            }
            return 0;
        }
        if (p->win) {
            allow_lds(k_batch<NW, 1, false, false, true>);
            allow_lds(k_batch<NW, 1, false, true, true>);
            return p->sparse ? occupancy(k_batch<NW, 1, false, true, true>, T, p->lds_bytes)
                             : occupancy(k_batch<NW, 1, false, false, true>, T, p->lds_bytes);
        }
    }
    if (p->sparse)
        return std::min(occupancy(k_batch<NW, G, false, true, false>, T, p->lds_bytes),
                        occupancy(k_batch<NW, G, true, true, false>, T, p->lds_bytes));
    return std::min(occupancy(k_batch<NW, G, false, false, false>, T, p->lds_bytes),
                    occupancy(k_batch<NW, G, true, false, false>, T, p->lds_bytes));
}

// Allow the plan's dynamic LDS for its kernels and return how many of the fused kernel's
// workgroups fit a CU (0 if none).  Done once when a plan is chosen, so that launches make no other runtime calls.
int prepare_batch(BatchPlan *p) {
    switch (p->waves * 10 + p->groups) {
        case 41: return prepare_t<4, 1>(p);
        case 42: return prepare_t<4, 2>(p);
        case 61: return prepare_t<6, 1>(p);
        case 62: return prepare_t<6, 2>(p);
        case 81: return prepare_t<8, 1>(p);
        case 82: return prepare_t<8, 2>(p);
        case 121: return prepare_t<12, 1>(p);
        case 122: return prepare_t<12, 2>(p);
        case 161: return prepare_t<16, 1>(p);
        case 162: return prepare_t<16, 2>(p);
        default: return 0;
    }
}

}  // namespace hough

#ifdef HOUGH_PHASE_TIMING
// include/hough_debug.h: read (and optionally clear) the phase totals of the instrumented build.
extern "C" int hough_debug_phase_ticks(uint64_t *out, int32_t n, int32_t reset, uint32_t *clock_khz) {
    if (!out || n < 1 || n > hough::kPhaseSlots) return HOUGH_EINVAL;
    unsigned long long v[hough::kPhaseSlots] = {};
    int dev = 0, khz = 0;
    if (clock_khz && (hipGetDevice(&dev) != hipSuccess ||
                      hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev) != hipSuccess))
        return HOUGH_EDEVICE;
    if (clock_khz) *clock_khz = (uint32_t)khz;
    if (hipDeviceSynchronize() != hipSuccess ||
        hipMemcpyFromSymbol(v, HIP_SYMBOL(hough::g_phase_ticks), sizeof(v)) != hipSuccess)
        return HOUGH_EDEVICE;
    for (int i = 0; i < n; ++i) out[i] = (uint64_t)v[i];
    if (reset) {
        const unsigned long long z[hough::kPhaseSlots] = {};
        if (hipMemcpyToSymbol(HIP_SYMBOL(hough::g_phase_ticks), z, sizeof(z)) != hipSuccess ||
            hipDeviceSynchronize() != hipSuccess)
            return HOUGH_EDEVICE;
    }
    return HOUGH_OK;
}
#endif
