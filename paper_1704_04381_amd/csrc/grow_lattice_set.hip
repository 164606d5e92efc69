// Long chains on the simple cubic lattice: the occupied sites as a hash set
// in LDS instead of a history (Sec. 3.3.2, Algorithm 1; weight of Eq. 3), so
// that a step costs six lookups whatever the chain's length.  Eight lanes
// per chain, up to eight chains per wave, one wave per block.
//
// Sites.  A site is one word P: bits 0-4 its place in a 4 x 4 x 2 block (two
// bits of x, two of y, one of z), bits 5-13, 14-22 and 23-31 the block's x, y
// and z.  Coordinates are kept modulo 2048, 2048 and 1024 (a torus); they are
// exact while the chain spans less than that, which is watched (below).  One
// coordinate moves by an addition with the bits between its two fields set,
// so that carries pass: three operations per candidate.
//
// Set.  Open addressing over NB buckets of 32 bytes, four entries each:
// (P | 31 of the block, bitmap of its 32 sites); 0 is an empty entry.  A
// chain has one entry per 4.6-5.3 monomers, so that the set takes 2.4-3.2 bytes
// per monomer where a history word takes 4 or 8 and its scan reads half of
// them each step.  Entries are never moved, and buckets fill in order, so a
// lookup ends at the block's entry or at the first empty one, which is also
// where a new entry goes.
//
// Step.  Lane t = 0..5 of the group looks up candidate t of the canonical
// order (-z, -y, -x, +x, +y, +z) in its home bucket, read whole (further
// buckets only behind four full entries), a ballot gives the free mask, every lane picks the same rank,
// and the lane of the chosen candidate writes the site's bit (or the new
// entry) where its own lookup ended.  Its P reaches the group by an OR over
// the eight lanes.
//
// Chains end at different steps, so groups do not share one step index: each
// takes its next chain from a queue as it ends one (a counter in the
// workspace, read in chunks), and only the step modulo 8 is common to the
// wave, which keeps one Philox block per group and eight steps.  An attempt
// that meets a dead end under the restart rule starts over the same way.
//
// Between runs of eight steps each lane follows one true coordinate and its
// extremes.  A chain that comes near the torus' period, whose lookups find
// no room, or whose |coordinate| reaches the launch's byte_box (tests) is
// grown again, from its first draw, by replay_chain: the
// same draws and tests without the set, each lane retracing an eighth of the
// moves in every step.  Both are many standard deviations away, so that this
// path is for exactness, not for speed.
//
// Sums over the placed monomers come from the bitmaps when a chain ends, in
// the pass that clears the table for the next one.
//
// Bound by the latency of a step at the number of chains whose tables fit in a
// CU's LDS.  N = 2048, 10^5 chains, six per wave and five waves per CU (counters):
// 1050 cycles, 92 vector and 4.2 LDS instructions per step of a wave, its share of
// the Philox blocks, chain ends and lookups beyond the home bucket included; the
// vector units issue 0.44 of the time.  MI355X, whole calls, scan of the history with 64 lanes or
// in LDS -> set: N = 2048, 10^5 chains, 16.9 -> 9.6 ms; N = 10000, 5000
// chains, 81.9 -> 6.7 ms, where the longest chain's 10^4 steps alone take 3 ms.
//
// 26-neighbour lattice (Z26).  The 27 sites around the tip lie in its own block
// and at most seven others: lane t = tx + 2 ty + 4 tz takes the block that is
// its own or the one next to it on the tip's side along each axis (none where
// the tip is not at that face), spreads the bitmap's rows over the code
// (dx + 1) + 3 (dy + 1) + 9 (dz + 1), and an OR over the group gives the mask.
// MI355X, growth kernel, scan -> set: N = 512, 2 10^5 chains, 10.0 -> 5.1 ms;
// N = 2048, 3 10^4, 14.5 -> 7.5; N = 8000, 1000 chains, 40 -> 4.8.
#include "lattice_common.hpp"

#include <tuple>
#include <type_traits>

namespace rsaw {

constexpr uint32_t kSetMx = 0x3u | (0x1FFu << 5);
constexpr uint32_t kSetMy = 0xCu | (0x1FFu << 14);
constexpr uint32_t kSetMz = 0x10u | (0x1FFu << 23);
constexpr uint32_t kSetCodes26 = 0x7FFFFFFu & ~(1u << 13); // 27 sites without the tip's own

__device__ __forceinline__ void set_wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// OR over an aligned group of 8 lanes (all active), every lane receiving it.
__device__ __forceinline__ uint32_t or8(uint32_t v)
{
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, false);
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, false);
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, false);
    return v;
}

// Buckets a lookup visits before it gives up.
constexpr int kSetProbes = 64;
constexpr uint32_t kSetSpare = 64 * 8; // bytes behind a block's tables: one entry per lane

// Home bucket of a block (its key P | 31): a dot product of the key's halves,
// its low 16 bits scaled to NB.  Neighbouring blocks land a fixed stride
// apart, which fills the table more evenly than a multiplicative hash: over
// grown chains, with buckets of two entries, 0.048 against 0.063 further
// buckets per lookup at N = 512 and 0.145 against 0.191 at N = 2048, in one
// full-rate operation instead of two quarter-rate ones.
__device__ __forceinline__ uint32_t set_home(uint32_t key, uint32_t NB)
{
    typedef unsigned short ushort2_t __attribute__((ext_vector_type(2)));
    const ushort2_t w = {0xC3AB, 0xE4F7};
    const uint32_t h = __builtin_amdgcn_udot2(__builtin_bit_cast(ushort2_t, key), w, 0u, false);
    return __umul24(h & 0xFFFFu, NB) >> 16;
}

// Compile-time loop: f(integral_constant<int, I>) for I = B .. E-1.
template <int B, int E, typename F>
__device__ __forceinline__ void static_for(F &&f)
{
    if constexpr (B < E) {
        f(std::integral_constant<int, B>{});
        static_for<B + 1, E>(f);
    }
}

// Outputs of one chain's final attempt.
struct SetResult {
    double lw;      // -inf for a dead chain
    int64_t nn;     // n_grown^2 Rg^2
    int32_t x, y, z;
    int32_t grown;
    bool alive;
};

template <typename CT>
__device__ __forceinline__ void set_write(const GrowArgs &a, uint64_t c, const SetResult &r)
{
    if (a.log_w) a.log_w[c] = r.lw;
    if (a.r_end) {
        CT *re = (CT *)a.r_end;
        re[c] = (CT)r.x;
        re[a.n_chains + c] = (CT)r.y;
        re[2 * a.n_chains + c] = (CT)r.z;
    }
    if (a.r2) a.r2[c] = (double)((int64_t)r.x * r.x + (int64_t)r.y * r.y + (int64_t)r.z * r.z);
    if (a.n2rg2) a.n2rg2[c] = r.nn;
    if (a.rg2) a.rg2[c] = (double)r.nn / ((double)r.grown * (double)r.grown);
    if (a.n_grown) a.n_grown[c] = (uint16_t)r.grown;
}

// log W = sum over m = 1..6, ascending, of n_m log m; n_1 log 1 = 0 and m_1 = 6.
__device__ __forceinline__ double set_log_w(const GrowArgs &a, uint32_t n2, uint32_t n3, uint32_t n4, uint32_t n5)
{
    double lw = 0.0;
    lw = lw + (double)n2 * a.logm[2];
    lw = lw + (double)n3 * a.logm[3];
    lw = lw + (double)n4 * a.logm[4];
    lw = lw + (double)n5 * a.logm[5];
    return lw + a.logm[6];
}

// Sum over the group's eight lanes.
__device__ __forceinline__ int64_t sum8(int64_t v)
{
#pragma unroll
    for (int off = 1; off < 8; off <<= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// Move of candidate j: 0..5 (-z, -y, -x, +x, +y, +z), or the code of Z26.
template <bool Z26>
__device__ __forceinline__ void set_move(int j, int &x, int &y, int &z)
{
    if constexpr (Z26) {
        x += j % 3 - 1;
        y += j / 3 % 3 - 1;
        z += j / 9 - 1;
    } else {
        x += (j == 3) - (j == 2);
        y += (j == 4) - (j == 1);
        z += (j == 5) - (j == 0);
    }
}

// log W from the group's counts: lane t holds n_m of m = t + 2 (six
// neighbours), or of m = t + 1 + 8 f in n[f] (Z26); `lane` reads one of them.
template <bool Z26, typename F>
__device__ __forceinline__ double set_sum_log_w(const GrowArgs &a, F &&lane)
{
    if constexpr (!Z26) {
        return set_log_w(a, lane(0, 0), lane(1, 0), lane(2, 0), lane(3, 0));
    } else {
        double lw = 0.0;
#pragma unroll
        for (int f = 0; f < 4; ++f)
            for (int q = 0; q < (f < 3 ? 8 : 2); ++q) lw = lw + (double)lane(q, f) * a.logm[1 + q + 8 * f];
        return lw;
    }
}

// Counts a step with m free candidates.
template <bool Z26>
__device__ __forceinline__ void set_count(uint32_t (&n)[4], uint32_t m, int t)
{
    if constexpr (Z26) {
#pragma unroll
        for (uint32_t f = 0; f < 4; ++f) n[f] += m == (uint32_t)t + 1u + 8u * f ? 1u : 0u;
    } else {
        n[0] += m == (uint32_t)t + 2u ? 1u : 0u;
    }
}

// Grows chain c of this group without a set: moves (j + 1) in `mv`, a nibble
// each (a byte in Z26); in each step lane t retraces the moves of its eighth
// of the chain.  The group's eight lanes are active; mv is left cleared.
template <bool Z26>
__device__ __forceinline__ bool replay_chain(const GrowArgs &a, uint32_t *mv, uint64_t c, SetResult *out)
{
    const int N = a.n_monomers;
    const int t = threadIdx.x & 7;
    const uint64_t g = a.chain_offset + c;
    constexpr int BITS = Z26 ? 8 : 4, PER = 32 / BITS;
    const int gbase = threadIdx.x & 56;
    const int words = (N - 2) / PER + 1;      // N - 1 moves
    const int segw = (words + 7) / 8;         // words per lane
    const int first = t * segw * PER;         // moves before this lane's
    bool failed = false;
    for (uint32_t rd = 0;; ++rd) {
        for (int w = t; w < words; w += 8) mv[w] = 0u;
        set_wave_sync();
        int x = 0, y = 0, z = 0;     // tip
        int px = 0, py = 0, pz = 0;  // site before this lane's first move
        uint32_t n[4] = {0, 0, 0, 0};
        int placed = 1;
        Philox4 blk{0, 0, 0, 0};
        const uint32_t hi = rd << 16;
        // visits the sites of this lane's part of the chain
        const auto visit = [&](auto &&f) {
            if (t == 0) f(0, 0, 0);
            int vx = px, vy = py, vz = pz;
            for (int w = t * segw; w < (t + 1) * segw && w < words; ++w) {
                uint32_t v = mv[w];
                for (; v; v >>= BITS) {
                    set_move<Z26>((int)(v & ((1u << BITS) - 1u)) - 1, vx, vy, vz);
                    f(vx, vy, vz);
                }
            }
        };
        bool dead = false;
        for (int i = 1; i < N; ++i) {
            uint32_t occ = 0;
            visit([&](int vx, int vy, int vz) {
                const int dx = vx - x, dy = vy - y, dz = vz - z;
                if constexpr (Z26) {
                    if (dx >= -1 && dx <= 1 && dy >= -1 && dy <= 1 && dz >= -1 && dz <= 1)
                        occ |= 1u << (dx + 1 + 3 * (dy + 1) + 9 * (dz + 1));
                } else {
                    const int l1 = (dx < 0 ? -dx : dx) + (dy < 0 ? -dy : dy) + (dz < 0 ? -dz : dz);
                    const int q = dx + 2 * dy + 3 * dz; // -3..3
                    if (l1 == 1) occ |= 1u << (q < 0 ? q + 3 : q + 2);
                }
            });
            occ = or8(occ);
            const uint32_t freem = ~occ & (Z26 ? kSetCodes26 : 0x3Fu), m = __builtin_popcount(freem);
            if (i == 1 || (i & 7) == 0) blk = draw(a.seed, g, (uint32_t)(i >> 3) | hi, kSlotSelect, 0);
            const uint32_t xw = half_word(blk, (uint32_t)(i & 7));
            if (m == 0) {
                dead = true;
                break;
            }
            uint32_t r = lemire_redraw16(a.seed, g, (uint32_t)i | hi, m, xw);
            if (r == kPickFailed) {
                failed = true;
                r = 0;
            }
            uint32_t f = freem;
            for (; r; --r) f &= f - 1u;
            const int j = __builtin_ctz(f);
            set_move<Z26>(j, x, y, z);
            if (t == 0) mv[(i - 1) / PER] |= (uint32_t)(j + 1) << (BITS * ((i - 1) & (PER - 1)));
            set_wave_sync();
            if (i == first) {
                px = x;
                py = y;
                pz = z;
            }
            set_count<Z26>(n, m, t);
            ++placed;
        }
        if (dead && rd + 1 < a.max_rounds) continue;
        int64_t sx = 0, sy = 0, sz = 0, s2 = 0;
        visit([&](int vx, int vy, int vz) {
            sx += vx;
            sy += vy;
            sz += vz;
            s2 += (int64_t)vx * vx + (int64_t)vy * vy + (int64_t)vz * vz;
        });
        sx = sum8(sx);
        sy = sum8(sy);
        sz = sum8(sz);
        s2 = sum8(s2);
        out->nn = (int64_t)placed * s2 - (sx * sx + sy * sy + sz * sz);
        const double lw =
            set_sum_log_w<Z26>(a, [&](int q, int f) { return (uint32_t)__shfl(n[f], gbase + q, 64); });
        out->lw = dead ? -__builtin_huge_val() : lw;
        out->x = x;
        out->y = y;
        out->z = z;
        out->grown = placed;
        out->alive = !dead;
        set_wave_sync();
        for (int w = t; w < words; w += 8) mv[w] = 0u;
        set_wave_sync();
        return failed;
    }
}

// Chains a wave takes from the queue at a time: an eighth of what each
// resident group will grow, so that the last chains still spread, and at
// most 64 (the counter's atomics complete one at a time, 11-14 ns each).
__host__ __device__ inline uint32_t set_chunk(uint64_t n_chains, uint32_t gpw, uint32_t NB)
{
    const uint64_t per_cu = 163840 / (gpw * NB * 32 + kSetSpare);
    const uint64_t c = n_chains / (256 * per_cu * gpw * 8);
    return c < 1 ? 1u : (c > 64 ? 64u : (uint32_t)c);
}

template <bool Z26, typename CT>
__device__ __forceinline__ void grow_lattice_set_body(const GrowArgs &a, uint32_t NB, uint32_t gpw)
{
    extern __shared__ uint4 set_lds[];
    const int lane = threadIdx.x & 63;
    const int t = lane & 7;
    const int gbase = lane & ~7;
    const uint32_t gi = (uint32_t)lane >> 3;
    const bool has_group = gi < gpw;
    const uint32_t TB = 2 * NB; // b128 words of a table
    uint4 *tab = set_lds + (has_group ? gi : 0u) * TB;
    const uint4 *tab_end = tab + TB;
    uint2 *spare = (uint2 *)(set_lds + gpw * TB) + lane;
    const int N = a.n_monomers;
    const uint32_t chunk = set_chunk(a.n_chains, gpw, NB);

    // this lane's candidate: the axis' field mask and the addend of its move
    const bool cand = Z26 || t < 6;
    const int axis = t == 0 || t == 5 ? 2 : (t == 1 || t == 4 ? 1 : 0);
    const uint32_t fm = axis == 0 ? kSetMx : (axis == 1 ? kSetMy : kSetMz);
    const uint32_t fn = ~fm;
    const uint32_t fd = !cand ? 0u : (t < 3 ? fm : (fm & (0u - fm)));
    const uint32_t below = (1u << t) - 1u;
    // Z26: key addends of this lane's block, and per place of the tip in its
    // block (a byte each) the shifts that take the bitmap's rows to the code
    const bool ox = t & 1, oy = (t >> 1) & 1, oz = t >> 2;
    const uint32_t px1 = ox ? 1u << 5 : 0u, mx1 = ox ? 0x1FFu << 5 : 0u;
    const uint32_t py1 = oy ? 1u << 14 : 0u, my1 = oy ? 0x1FFu << 14 : 0u;
    const uint32_t pz1 = oz ? 1u << 23 : 0u, mz1 = oz ? 0x1FFu << 23 : 0u;
    const uint32_t nowhere = (ox ? 1u : 0u) | (oy ? 4u : 0u); // of P ^ (P >> 1): not at a face
    const uint32_t shx = ox ? 0x01000006u : 0x05040302u;      // right, rows pre-shifted by 3
    const uint32_t shyl = oy ? 0x10000000u : 0x00000008u, shyr = oy ? 0x00000018u : 0x10080000u;
    const uint32_t shzl = oz ? 0x00001200u : 0x00000009u, shzr = oz ? 0x00000009u : 0u;
    uint32_t nb = NB; // in a VGPR: the step loop has scalar registers to spare for masks only
    asm volatile("" : "+v"(nb));
    // its coordinate's fields: low bits, high bits, width
    const uint32_t lo_off = axis == 0 ? 0u : (axis == 1 ? 2u : 4u), lo_w = axis == 2 ? 1u : 2u;
    const uint32_t hi_off = axis == 0 ? 5u : (axis == 1 ? 14u : 23u);
    const int wrap = 32 - 9 - (int)lo_w;
    const int period = 1 << (9 + lo_w);
    const auto field = [&](uint32_t P) {
        return (__builtin_amdgcn_ubfe(P, hi_off, 9u) << lo_w) | __builtin_amdgcn_ubfe(P, lo_off, lo_w);
    };

    for (uint32_t q = lane; q < gpw * TB; q += 64) set_lds[q] = make_uint4(0u, 0u, 0u, 0u);
    set_wave_sync();

    uint64_t next = 0, end = 0; // the wave's chunk of the queue
    bool drained = false;
    bool busy = false;          // the group has a chain
    bool alive = false;         // and it grows
    bool full = false;          // this lane found no room for a block
    bool rng_fail = false;
    uint64_t c = 0, best = 0;
    uint32_t rd = 0, i0 = 0, P = 0, n_mine[4] = {0, 0, 0, 0};
    int placed = 1, co = 0, cmin = 0, cmax = 0;
    uint32_t fprev = 0;

    const auto start = [&]() { // the chain's next attempt, on a cleared table
        alive = true;
        i0 = 0;
        P = 0;
        placed = 1;
#pragma unroll
        for (int f = 0; f < 4; ++f) n_mine[f] = 0;
        co = cmin = cmax = 0;
        fprev = 0;
        // the origin's entry
        if (t == 0) {
            *(uint2 *)(tab + 2 * set_home(31u, NB)) = make_uint2(31u, 1u);
        }
    };

    for (;;) {
        // ended groups: results, a cleared table, the next attempt
        bool fail = false;
        {
            const uint32_t f = field(P);
            co += (int)((f - fprev) << wrap) >> wrap;
            fprev = f;
            cmin = co < cmin ? co : cmin;
            cmax = co > cmax ? co : cmax;
            // extremes between the looks lie within 8 of these; the unwrapped
            // range starts on a block boundary
            bool over = cmax + 8 - ((cmin - 8) & ~3) >= period - 1;
            over = over || (a.byte_box > 0 && (cmax >= a.byte_box || -cmin >= a.byte_box));
            over = over || full;
            full = false;
            const uint64_t ob = __builtin_amdgcn_ballot_w64(busy && over);
            fail = ((ob >> gbase) & 0xFFull) != 0;
        }
        const bool ended = busy && (!alive || fail);
        const bool again = ended && !fail && placed < N && rd + 1 < a.max_rounds;
        // the whole wave takes the ended groups in turn: sums over the bitmaps
        // where the attempt counts, and a cleared table
        for (uint64_t todo = __builtin_amdgcn_ballot_w64(ended && t == 0); todo; todo &= todo - 1) {
            const int src = __builtin_ctzll(todo);
            uint4 *tb = set_lds + ((uint32_t)src >> 3) * TB;
            const int lox = (__builtin_amdgcn_readlane(cmin, src + 2) - 8) & ~3,
                      loy = (__builtin_amdgcn_readlane(cmin, src + 1) - 8) & ~3,
                      loz = (__builtin_amdgcn_readlane(cmin, src) - 8) & ~3;
            int sx = 0, sy = 0, sz = 0; // |sums| below N^2
            int64_t s2 = 0;
            const auto add = [&](uint32_t key, uint32_t bits) {
                const int X = lox + ((((int)((key >> 5) & 0x1FFu) << 2) - lox) & 2047);
                const int Y = loy + ((((int)((key >> 14) & 0x1FFu) << 2) - loy) & 2047);
                const int Z = loz + ((((int)(key >> 23) << 1) - loz) & 1023);
                const int n = __builtin_popcount(bits);
                const int x0 = __builtin_popcount(bits & 0xAAAAAAAAu), x1 = __builtin_popcount(bits & 0xCCCCCCCCu);
                const int y0 = __builtin_popcount(bits & 0xF0F0F0F0u), y1 = __builtin_popcount(bits & 0xFF00FF00u);
                const int z0 = __builtin_popcount(bits & 0xFFFF0000u);
                const int ax = x0 + 2 * x1, ay = y0 + 2 * y1;
                const int qx = x0 + 4 * x1 + 4 * __builtin_popcount(bits & 0x88888888u);
                const int qy = y0 + 4 * y1 + 4 * __builtin_popcount(bits & 0xF000F000u);
                sx += n * X + ax;
                sy += n * Y + ay;
                sz += n * Z + z0;
                s2 += (int64_t)n * (X * X + Y * Y + Z * Z) + (2 * (X * ax + Y * ay + Z * z0) + qx + qy + z0);
            };
            for (uint32_t q = lane; q < TB; q += 64) {
                const uint4 en = tb[q];
                tb[q] = make_uint4(0u, 0u, 0u, 0u);
                if (en.y) add(en.x, en.y);
                if (en.w) add(en.z, en.w);
            }
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                sx += __shfl_xor(sx, off, 64);
                sy += __shfl_xor(sy, off, 64);
                sz += __shfl_xor(sz, off, 64);
                s2 += __shfl_xor(s2, off, 64);
            }
            if (lane == src && !again && !fail) {
                SetResult r;
                r.alive = placed == N;
                r.lw = -__builtin_huge_val();
                r.nn = (int64_t)placed * s2 - ((int64_t)sx * sx + (int64_t)sy * sy + (int64_t)sz * sz);
                r.x = __builtin_amdgcn_readlane(co, src + 2);
                r.y = __builtin_amdgcn_readlane(co, src + 1);
                r.z = co;
                r.grown = placed;
                if (r.alive)
                    r.lw = set_sum_log_w<Z26>(a, [&](int q, int f) {
                        return (uint32_t)__builtin_amdgcn_readlane((int)n_mine[f], src + q);
                    });
                set_write<CT>(a, c, r);
                const uint64_t bits = r.alive ? (uint64_t)__double_as_longlong(r.lw) : 0ull;
                best = bits > best ? bits : best;
            }
        }
        set_wave_sync();
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(fail) != 0, 0)) {
            if (fail) {
                SetResult r;
                rng_fail = replay_chain<Z26>(a, (uint32_t *)tab, c, &r) || rng_fail;
                if (t == 0) {
                    set_write<CT>(a, c, r);
                    const uint64_t bits = r.alive ? (uint64_t)__double_as_longlong(r.lw) : 0ull;
                    best = bits > best ? bits : best;
                }
            }
        }
        if (ended) {
            alive = false;
            busy = again;
            if (again) {
                ++rd;
                start();
            }
        }
        set_wave_sync();
        // groups without a chain take the next ones of the queue
        for (;;) {
            const uint64_t want = __builtin_amdgcn_ballot_w64(has_group && !busy && t == 0);
            if (want == 0 || drained) break;
            if (next == end) {
                unsigned long long v = 0;
                if (lane == 0) v = atomicAdd(a.queue, (unsigned long long)chunk);
                next = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32)) << 32) |
                       (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
                end = next + chunk < a.n_chains ? next + chunk : a.n_chains;
                if (next >= a.n_chains) {
                    drained = true;
                    break;
                }
            }
            const uint64_t rank = __builtin_popcountll(want & ((1ull << gbase) - 1ull));
            const uint64_t n = (uint64_t)__builtin_popcountll(want);
            if (has_group && !busy && rank < end - next) {
                busy = true;
                c = next + rank;
                rd = 0;
                start();
            }
            next += n < end - next ? n : end - next;
        }
        set_wave_sync();
        if (__builtin_amdgcn_ballot_w64(busy) == 0) break;

        // The next eight steps i0 .. i0 + 7.  Bit e of `ticks` allows step
        // i0 + e on a candidate lane: not step 0, none past N - 1, none after
        // a dead end.  A step that is not allowed has an empty free mask.
        const uint64_t g = a.chain_offset + c;
        const uint32_t hi = rd << 16;
        const Philox4 blk = draw(a.seed, g, (i0 >> 3) | hi, kSlotSelect, 0);
        const int last = N - 1 - (int)i0;
        uint32_t ticks = last >= 7 ? 0xFFu : (2u << (last & 7)) - 1u;
        ticks &= i0 == 0 ? 0xFEu : 0xFFu;
        ticks = busy && cand ? ticks : 0u;
        static_for<0, 8>([&](auto E) {
            constexpr int e = E.value;
            const uint32_t act = 0u - ((ticks >> e) & 1u);
            uint32_t C = 0, kk, looks = act; // the candidate site, the key, whether the lookup counts
            if constexpr (Z26) {
                const auto side = [&](uint32_t bit, uint32_t up, uint32_t down) {
                    const uint32_t high = (uint32_t)((int)(P << (31 - bit)) >> 31);
                    return P + __builtin_amdgcn_bitop3_b32(high, up, down, 0xCA); // high ? up : down
                };
                kk = (side(1, px1, mx1) & (kSetMx & ~31u)) | (side(3, py1, my1) & (kSetMy & ~31u)) |
                     (side(4, pz1, mz1) & (kSetMz & ~31u)) | 31u;
                looks = ((P ^ (P >> 1)) & nowhere) ? 0u : act;
            } else {
                C = (((P | fn) + fd) & fm) | (P & fn);
                kk = C | 31u;
            }
            // a bucket's entries: (x, y), (z, w) of q0 and q1
            const uint4 *b = tab + 2 * set_home(kk, nb);
            uint4 q0, q1;
            const auto look = [&]() {
                q0 = b[0];
                q1 = b[1];
                // both whole, in flight together
                asm volatile("" : "+v"(q0.x), "+v"(q0.y), "+v"(q0.z), "+v"(q0.w), "+v"(q1.x), "+v"(q1.y),
                             "+v"(q1.z), "+v"(q1.w));
                uint32_t f = q0.x == kk ? q0.y : 0u;
                f = q0.z == kk ? q0.w : f;
                f = q1.x == kk ? q1.y : f;
                return q1.z == kk ? q1.w : f;
            };
            uint32_t bm = look();
            const uint32_t more = (bm == 0u ? q1.z : 0u) & looks; // not found, no room
            if (__builtin_expect(__builtin_amdgcn_ballot_w64(more != 0u) != 0, 0)) {
                if (more != 0u) {
                    int left = kSetProbes;
                    do {
                        b = b + 2 == tab_end ? tab : b + 2;
                        if (--left == 0) {
                            full = true; // the group's chain is grown again without a set
                            bm = 0u;
                            break;
                        }
                        bm = look();
                    } while (bm == 0u && q1.z != 0u);
                }
            }
            // free candidates: a bit per lane, or per code
            uint32_t fr = 0, mask;
            if constexpr (Z26) {
                const uint32_t ix = (P & 3u) << 3, iy = (P & 12u) << 1, iz = (P & 16u) >> 1;
                const uint32_t sx = shx >> ix, yl = shyl >> iy, yr = shyr >> iy;
                const auto plane = [&](uint32_t p) { // 16 bits, rows of 4 along x -> 9 bits of (dx, dy)
                    p = (p | (p << 8)) & 0x00FF00FFu;
                    p = (p | (p << 4)) & 0x0F0F0F0Fu;
                    p = ((p << 3) >> (sx & 31u)) & 0x07070707u;
                    p = (p << (yl & 31u)) >> (yr & 31u);
                    return __builtin_amdgcn_udot4(p, 0x00400801u, 0u, false);
                };
                uint32_t occ = plane(bm & 0xFFFFu) | (plane(bm >> 16) << 9);
                occ = (occ << ((shzl >> iz) & 31u)) >> ((shzr >> iz) & 31u);
                mask = ~or8(occ & looks) & kSetCodes26 & act;
            } else {
                fr = ~(bm >> (C & 31u)) & act & 1u;
                const uint64_t bal = __builtin_amdgcn_ballot_w64(fr != 0u);
                mask = (uint32_t)(bal >> gbase) & 0x3Fu;
            }
            const uint32_t m = __builtin_popcount(mask);
            const uint32_t x = half_word(blk, (uint32_t)e);
            const uint32_t p = x * m;
            uint32_t r = p >> 16;
            const bool redraw = (p & 0xFFFFu) < m; // never for m = 0
            if (__builtin_expect(__builtin_amdgcn_ballot_w64(redraw) != 0, 0)) {
                if (redraw) {
                    r = lemire_redraw16_inline(a.seed, g, (i0 + e) | hi, m, x);
                    if (r == kPickFailed) {
                        rng_fail = true;
                        r = 0;
                    }
                }
            }
            const bool ok = m != 0u;
            bool chosen;
            uint32_t NP = 0;
            if constexpr (Z26) {
                // the r-th free code: lane t looks among codes 4 t .. 4 t + 3
                const uint32_t four = (mask >> (4 * t)) & 15u;
                const uint32_t k = r - (uint32_t)__builtin_popcount(mask & ((1u << (4 * t)) - 1u));
                const uint32_t f1 = four & (four - 1u), f2 = f1 & (f1 - 1u), f3 = f2 & (f2 - 1u);
                const uint32_t pick = k == 0u ? four : (k == 1u ? f1 : (k == 2u ? f2 : f3));
                const bool here = k < (uint32_t)__builtin_popcount(four);
                const uint32_t code = or8(here ? 4u * t + (uint32_t)__builtin_ctz(pick | 16u) + 1u : 0u) - 1u;
                const uint32_t z = (code * 57u) >> 9, rem = code - 9u * z, y = (rem * 11u) >> 5, xx = rem - 3u * y;
                const auto moved = [&](uint32_t d, uint32_t field) {
                    const uint32_t add = d == 0u ? field : (d == 2u ? field & (0u - field) : 0u);
                    return ((P | ~field) + add) & field;
                };
                NP = moved(xx, kSetMx) | moved(y, kSetMy) | moved(z, kSetMz);
                C = NP;
                chosen = ok & (kk == (NP | 31u)); // the lane that looked its block up
            } else {
                chosen = (fr != 0u) & ((uint32_t)__builtin_popcount(mask & below) == r);
            }
            // written to its entry or the first empty one; the other lanes
            // write to their places behind the tables, which costs less than
            // a branch around the store
            uint32_t o = 3;
            o = ((q1.x == kk) | (q1.x == 0u)) ? 2u : o;
            o = ((q0.z == kk) | (q0.z == 0u)) ? 1u : o;
            o = ((q0.x == kk) | (q0.x == 0u)) ? 0u : o;
            uint2 *at = (uint2 *)b + o;
            at = chosen ? at : spare;
            *at = make_uint2(kk, bm | (1u << (C & 31u)));
            if constexpr (!Z26) NP = or8(chosen ? C : 0u);
            P = ok ? NP : P;
            placed += ok ? 1 : 0;
            set_count<Z26>(n_mine, m, t);
            // a dead end closes the run (the tick of step 0 is none)
            ticks = (e == 0 ? ok || i0 == 0 : ok) ? ticks : 0u;
            set_wave_sync();
        });
        i0 += 8;
        alive = placed == (int)i0 && placed < N; // every step of the run placed its monomer
    }
    if (rng_fail) atomicExch(a.status, 6);
    publish_log_w_max(a, best);
}

template <bool Z26, typename CT>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(Z26 ? 3 : 4, 8))) void
grow_lattice_set(GrowArgs a, uint32_t NB, uint32_t gpw)
{
    grow_lattice_set_body<Z26, CT>(a, NB, gpw);
}

// Batched launch: block b serves the ensemble whose block range holds b.
template <bool Z26, typename CT>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(Z26 ? 3 : 4, 8))) void
grow_lattice_set_batch(const GrowEntry *tab, const uint64_t *block0, int n, uint64_t base)
{
    const int e = find_segment(block0, n, base + blockIdx.x);
    grow_lattice_set_body<Z26, CT>(tab[e].a, (uint32_t)tab[e].H, (uint32_t)tab[e].S);
}

// Tables.  A chain of N monomers has N / 4.6 (N = 256) to N / 5.3 (N = 10000)
// blocks, standard deviation below 0.57 sqrt(N) (measured), with 26 neighbours
// N / 3.3 (N = 256) to N / 3.6 (N = 2048).  Its table has at least 0.30 N or
// 0.39 N entries, a load of at most 0.72, and the chains per wave and the waves
// are those that put most chains on a CU: a step's latency hardly depends on
// either, so the chains in flight set the rate.  Of equal ones, a wave per SIMD
// but no more than it takes, then the larger tables, up to 0.40 N or 0.53 N
// entries, which few chains get in any case (their rate is the latency's).  MI355X, growth kernel, 0.35 N and 0.53 N entries with
// two waves per SIMD -> this: N = 2048, 10^5 chains, 10.8 -> 9.5 ms; N = 5000,
// 2 10^4, 9.0 -> 7.7; N = 10000, 5000, 7.3 -> 6.6; 26 neighbours N = 700, 10^5,
// 4.5 -> 4.1; N = 2048, 3 10^4, 11.1 -> 7.5; N = 8000, 4000, 18.8 -> 14.8.
// Smaller tables still (0.24 N) were slower at N = 1100 and 2048 (3.9, 10.1 ms).
constexpr int kSetLds = 163840, kSetLdsUnit = 1280; // per CU, and the step in which it is given

hipError_t lattice_set_variant(int N, uint64_t n_chains, bool z26, bool i16, GrowVariant *v)
{
    const int least = N * (z26 ? 39 : 30) / 400 + 6, most = N * (z26 ? 53 : 40) / 400 + 6;
    const int waves = z26 ? 12 : 16; // that the registers allow on a CU
    const uint64_t share = (n_chains + 255) / 256;
    const int need = share < 128 ? (int)share : 128; // chains a CU gets; it holds 16 x 8 at most
    int gpw = 0, per_cu = 0, NB = 0;
    std::tuple<int, int, int, int> best(0, 0, 0, 0);
    for (int b = 1; b <= waves; ++b)
        for (int g = 1; g <= 8; ++g) {
            const int room = (kSetLds / kSetLdsUnit / b * kSetLdsUnit - (int)kSetSpare) / (32 * g);
            const int nb = room < most ? room : most;
            if (nb < least) break;
            const std::tuple<int, int, int, int> score(g * b < need ? g * b : need, b < 4 ? b : 4, -b, nb);
            if (score >= best) { // then the chains per wave, for batches of small ensembles
                best = score;
                gpw = g;
                per_cu = b;
                NB = nb;
            }
        }
    if (gpw == 0) return hipErrorInvalidValue;
    v->family = 4;
    v->p0 = 8;
    v->p1 = z26 ? 1 : 0;
    v->p2 = i16 ? 1 : 0;
    v->threads = 64;
    v->cpb = gpw;
    v->shmem = (size_t)gpw * NB * 32 + kSetSpare;
    v->H = NB;
    v->S = gpw;
    v->max_blocks = 256u * (uint32_t)per_cu;
    return hipSuccess;
}

// The byte box (rsaw_set_byte_box) that the set heeds.  A lowered one sends chains
// to replay_chain, so that tests reach it; but N^2 steps on eight lanes take long
// (2000 chains of N = 3000 at an edge of 127: 251 ms; 1.1 without), and the set
// keeps no bytes.  So it heeds only edges below every format's own (62 is the
// smallest), and none beyond N = 4096, where no kernel keeps one word per monomer.
int32_t lattice_set_box(int N, int32_t edge) { return N <= 4096 && edge < 62 ? edge : 0; }

template <bool Z26, typename CT>
static hipError_t launch_set(const GrowArgs &a, const GrowVariant &v, const GrowEntry *tab, const uint64_t *block0,
                             int n, uint64_t blocks, size_t shmem, hipStream_t s)
{
    const void *fn = tab ? (const void *)grow_lattice_set_batch<Z26, CT> : (const void *)grow_lattice_set<Z26, CT>;
    if (shmem > 65536) {
        hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shmem);
        if (e != hipSuccess) return e;
    }
    GrowArgs one = a;
    one.byte_box = lattice_set_box(a.n_monomers, a.byte_box);
    return launch_sliced(blocks, 64, [&](uint64_t b0, uint32_t nb) {
        if (tab)
            hipLaunchKernelGGL((grow_lattice_set_batch<Z26, CT>), dim3(nb), dim3(64), shmem, s, tab, block0, n, b0);
        else
            hipLaunchKernelGGL((grow_lattice_set<Z26, CT>), dim3(nb), dim3(64), shmem, s, one, (uint32_t)v.H,
                               (uint32_t)v.S);
    });
}

hipError_t launch_lattice_set(const GrowArgs &a, const GrowVariant &v, const GrowEntry *tab, const uint64_t *block0,
                              int n, uint64_t blocks, size_t shmem, hipStream_t s)
{
    if (v.p1)
        return v.p2 ? launch_set<true, int16_t>(a, v, tab, block0, n, blocks, shmem, s)
                    : launch_set<true, int32_t>(a, v, tab, block0, n, blocks, shmem, s);
    return v.p2 ? launch_set<false, int16_t>(a, v, tab, block0, n, blocks, shmem, s)
                : launch_set<false, int32_t>(a, v, tab, block0, n, blocks, shmem, s);
}

} // namespace rsaw
