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
// chain has one entry per 4.6-5.3 monomers, so that the set takes 2.8 bytes
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
// Bound by the latency of a step (about 750 cycles: one dependent LDS read,
// 40 % of it, and 62 vector instructions) at the number of chains whose tables
// fit in a CU's LDS.  MI355X, whole calls, scan of the history with 64 lanes or
// in LDS -> set: N = 2048, 10^5 chains, 16.9 -> 10.9 ms; N = 10000, 5000
// chains, 81.9 -> 7.4 ms, where the longest chain's 10^4 steps alone take 3 ms.
#include "lattice_common.hpp"

#include <type_traits>

namespace rsaw {

constexpr uint32_t kSetMx = 0x3u | (0x1FFu << 5);
constexpr uint32_t kSetMy = 0xCu | (0x1FFu << 14);
constexpr uint32_t kSetMz = 0x10u | (0x1FFu << 23);

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

// Move of canonical candidate j = 0..5 (-z, -y, -x, +x, +y, +z).
__device__ __forceinline__ void set_move(int j, int &x, int &y, int &z)
{
    x += (j == 3) - (j == 2);
    y += (j == 4) - (j == 1);
    z += (j == 5) - (j == 0);
}

// Grows chain c of this group without a set: moves as nibbles (j + 1) in
// `mv`, eight per word; in each step lane t retraces the moves of its eighth
// of the chain.  The group's eight lanes are active; mv is left cleared.
__device__ __forceinline__ bool replay_chain(const GrowArgs &a, uint32_t *mv, uint64_t c, SetResult *out)
{
    const int N = a.n_monomers;
    const int t = threadIdx.x & 7;
    const uint64_t g = a.chain_offset + c;
    const int words = (N + 6) / 8;            // N - 1 moves
    const int segw = (words + 7) / 8;         // words per lane
    const int first = t * segw * 8;           // moves before this lane's
    bool failed = false;
    for (uint32_t rd = 0;; ++rd) {
        for (int w = t; w < words; w += 8) mv[w] = 0u;
        set_wave_sync();
        int x = 0, y = 0, z = 0;     // tip
        int px = 0, py = 0, pz = 0;  // site before this lane's first move
        uint32_t n2 = 0, n3 = 0, n4 = 0, n5 = 0;
        int placed = 1;
        Philox4 blk{0, 0, 0, 0};
        const uint32_t hi = rd << 16;
        // visits the sites of this lane's part of the chain
        const auto visit = [&](auto &&f) {
            if (t == 0) f(0, 0, 0);
            int vx = px, vy = py, vz = pz;
            for (int w = t * segw; w < (t + 1) * segw && w < words; ++w) {
                uint32_t v = mv[w];
                for (; v; v >>= 4) {
                    set_move((int)(v & 15u) - 1, vx, vy, vz);
                    f(vx, vy, vz);
                }
            }
        };
        bool dead = false;
        for (int i = 1; i < N; ++i) {
            uint32_t occ = 0;
            visit([&](int vx, int vy, int vz) {
                const int dx = vx - x, dy = vy - y, dz = vz - z;
                const int l1 = (dx < 0 ? -dx : dx) + (dy < 0 ? -dy : dy) + (dz < 0 ? -dz : dz);
                const int q = dx + 2 * dy + 3 * dz; // -3..3
                if (l1 == 1) occ |= 1u << (q < 0 ? q + 3 : q + 2);
            });
            occ = or8(occ);
            const uint32_t freem = ~occ & 0x3Fu, m = __builtin_popcount(freem);
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
            set_move(j, x, y, z);
            if (t == 0) mv[(i - 1) >> 3] |= (uint32_t)(j + 1) << (4 * ((i - 1) & 7));
            set_wave_sync();
            if (i == first) {
                px = x;
                py = y;
                pz = z;
            }
            n2 += m == 2;
            n3 += m == 3;
            n4 += m == 4;
            n5 += m == 5;
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
        out->lw = dead ? -__builtin_huge_val() : set_log_w(a, n2, n3, n4, n5);
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

template <typename CT>
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
    const bool cand = t < 6;
    const int axis = t == 0 || t == 5 ? 2 : (t == 1 || t == 4 ? 1 : 0);
    const uint32_t fm = axis == 0 ? kSetMx : (axis == 1 ? kSetMy : kSetMz);
    const uint32_t fn = ~fm;
    const uint32_t fd = !cand ? 0u : (t < 3 ? fm : (fm & (0u - fm)));
    const uint32_t below = (1u << t) - 1u;
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
    uint32_t rd = 0, i0 = 0, P = 0, n_mine = 0;
    int placed = 1, co = 0, cmin = 0, cmax = 0;
    uint32_t fprev = 0;

    const auto start = [&]() { // the chain's next attempt, on a cleared table
        alive = true;
        i0 = 0;
        P = 0;
        placed = 1;
        n_mine = 0;
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
                    r.lw = set_log_w(a, n_mine, __builtin_amdgcn_readlane(n_mine, src + 1),
                                     __builtin_amdgcn_readlane(n_mine, src + 2),
                                     __builtin_amdgcn_readlane(n_mine, src + 3));
                set_write<CT>(a, c, r);
                const uint64_t bits = r.alive ? (uint64_t)__double_as_longlong(r.lw) : 0ull;
                best = bits > best ? bits : best;
            }
        }
        set_wave_sync();
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(fail) != 0, 0)) {
            if (fail) {
                SetResult r;
                rng_fail = replay_chain(a, (uint32_t *)tab, c, &r) || rng_fail;
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
            const uint32_t C = (((P | fn) + fd) & fm) | (P & fn);
            const uint32_t kk = C | 31u;
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
            const uint32_t more = (bm == 0u ? q1.z : 0u) & act; // not found, no room
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
            const uint32_t fr = ~(bm >> (C & 31u)) & act & 1u;
            const uint64_t bal = __builtin_amdgcn_ballot_w64(fr != 0u);
            const uint32_t mask = (uint32_t)(bal >> gbase) & 0x3Fu;
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
            const bool chosen = (fr != 0u) & ((uint32_t)__builtin_popcount(mask & below) == r);
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
            const uint32_t NP = or8(chosen ? C : 0u);
            const bool ok = m != 0u;
            P = ok ? NP : P;
            placed += ok ? 1 : 0;
            n_mine += m == (uint32_t)t + 2u ? 1u : 0u;
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

template <typename CT>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(4, 8))) void
grow_lattice_set(GrowArgs a, uint32_t NB, uint32_t gpw)
{
    grow_lattice_set_body<CT>(a, NB, gpw);
}

// Batched launch: block b serves the ensemble whose block range holds b.
template <typename CT>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(4, 8))) void
grow_lattice_set_batch(const GrowEntry *tab, const uint64_t *block0, int n, uint64_t base)
{
    const int e = find_segment(block0, n, base + blockIdx.x);
    grow_lattice_set_body<CT>(tab[e].a, (uint32_t)tab[e].H, (uint32_t)tab[e].S);
}

// Table of a chain of N monomers: it has N / 4.6 (N = 256) to N / 5.3
// (N = 10000) blocks, standard deviation below 0.57 sqrt(N) (measured), and
// gets 0.35 N entries, a load of 0.62 to 0.54.  Chains per wave: what a CU's
// LDS holds over eight waves (two per SIMD), at most eight; fewer chains per
// wave where the LDS holds few, since a wave waits for the slowest lookup of
// its chains.
hipError_t lattice_set_variant(int N, bool i16, GrowVariant *v)
{
    const int NB = N * 7 / 80 + 6;
    const int fit = (163840 - 8 * (int)kSetSpare) / (NB * 32); // chains per CU
    int gpw = (fit + 7) / 8;
    gpw = gpw < 1 ? 1 : (gpw > 8 ? 8 : gpw);
    v->family = 4;
    v->p0 = 8;
    v->p1 = 0;
    v->p2 = i16 ? 1 : 0;
    v->threads = 64;
    v->cpb = gpw;
    v->shmem = (size_t)gpw * NB * 32 + kSetSpare;
    v->H = NB;
    v->S = gpw;
    v->max_blocks = 256u * (uint32_t)(163840 / v->shmem);
    return hipSuccess;
}

hipError_t launch_lattice_set(const GrowArgs &a, const GrowVariant &v, const GrowEntry *tab, const uint64_t *block0,
                              int n, uint64_t blocks, size_t shmem, hipStream_t s)
{
    const void *fn = tab ? (v.p2 ? (const void *)grow_lattice_set_batch<int16_t>
                                 : (const void *)grow_lattice_set_batch<int32_t>)
                         : (v.p2 ? (const void *)grow_lattice_set<int16_t> : (const void *)grow_lattice_set<int32_t>);
    if (shmem > 65536) {
        hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shmem);
        if (e != hipSuccess) return e;
    }
    return launch_sliced(blocks, 64, [&](uint64_t b0, uint32_t nb) {
        const dim3 gr(nb), bl(64);
        if (tab) {
            if (v.p2) hipLaunchKernelGGL((grow_lattice_set_batch<int16_t>), gr, bl, shmem, s, tab, block0, n, b0);
            else hipLaunchKernelGGL((grow_lattice_set_batch<int32_t>), gr, bl, shmem, s, tab, block0, n, b0);
        } else {
            if (v.p2) hipLaunchKernelGGL((grow_lattice_set<int16_t>), gr, bl, shmem, s, a, (uint32_t)v.H, (uint32_t)v.S);
            else hipLaunchKernelGGL((grow_lattice_set<int32_t>), gr, bl, shmem, s, a, (uint32_t)v.H, (uint32_t)v.S);
        }
    });
}

} // namespace rsaw
