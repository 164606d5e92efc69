// Hard-sphere chain growth in continuous space (Sec. 3.3.3, Algorithm 2;
// weight of Eq. 3).  Trial-parallel mapping: a group of G lanes (G = 8 or the
// next power of two >= k) serves one chain, lane t of the group owns trial t.
// Bead coordinates (binary64) live in LDS as (x, y, z) triples laid out
// [bead][chain of block] with an XOR swizzle of the chain index (see
// plane_row).
//
// Per step i:
//   1. lane t obtains the Marsaglia direction of trial t (Philox slot t, the
//      first accepted attempt) and forms the candidate c_t = tip + b e.
//      Each trial lane keeps a short queue of the accepted pairs of its own
//      trial for the coming steps, drawn ahead in rounds in which every lane
//      with room tries its next attempt; a step only waits for a new round
//      when some lane's queue is empty.  (With one chain per wave and
//      G >= 4 k, the spare lanes instead try later attempts of the same
//      step at once, see `spread`.);
//   2. culling: beads i-2 and i-3 are always tested; the G lanes of the
//      chain split beads 0 .. i-4 (lane t takes every G-th bead) and flag
//      those whose squared tip distance is below (b + sigma)^2 (1 + 2^-30);
//      every other bead is farther than sigma from every candidate (see
//      below), so it cannot overlap;
//   3. each lane tests its candidate against beads i-2, i-3 and the flagged
//      beads: ((dx dx + dy dy) + dz dz) < sigma^2 means overlap (no
//      contraction).  The flag offsets are merged over the wave so that the
//      loop is uniform; re-testing a culled bead is harmless;
//   4. a ballot over the group gives the free mask; m = popcount;
//   5. Lemire's pick (16-bit word from the 8-step selection block) chooses
//      the r-th free trial; its candidate is broadcast with a lane shuffle and
//      written to LDS as bead i by its owner;
//   6. lane m - 1 of the group counts the steps with m free trials, and
//      log W = sum_m n_m log m is formed once after the last step.
//
// Culling is exact, not an approximation.  With u = 2^-53, a bead is
// dropped only when its computed squared tip distance D~^2 (three
// differences, squares and two additions of non-negative terms) is at least
// T = (b + sigma)^2 (1 + e), e = 2^-30.  Then:
//   - the exact tip distance is D >= sqrt(T) (1 + u)^-2.5;
//   - the computed direction has |e| <= 1 + 5u, so the computed candidate
//     lies within b (1 + 9u) + u |tip| of the tip;
//   - the candidate's exact distance to the bead is d >= D - b (1 + 9u) - u |tip|,
//     and its computed d~^2 >= d^2 (1 - u)^5, which is >= sigma^2 whenever
//     d >= sigma (1 - u)^-2.5.
// Putting these together, 0.49 e (b + sigma) >= 11.5 u (b + sigma) + u |tip|
// suffices, and with |tip| <= (N - 1) b that holds for N <= 4 10^6: a culled
// bead would also have passed the full test.
#include "real_skip.hpp"
#include "rsaw_device.hpp"

namespace rsaw {

// Uniform on [-1, 1) from the 53-bit integer j = (a >> 5) 2^26 + (b >> 6):
// (j - 2^52) 2^-52, built from bits rather than converted.  With m the low
// 52 bits of j, d = 1 + m 2^-52 is a double of exponent 0, and the result is
// d - 1 when bit 52 of j (bit 31 of a) is set, else d - 2; both
// subtractions are exact (Sterbenz), so the value is the same double.
__device__ __forceinline__ double uniform53(uint32_t a, uint32_t b)
{
    const uint32_t lo = __builtin_amdgcn_alignbit(a >> 5, b, 6); // m bits 0..31
    const uint32_t h = a >> 11;
    const uint32_t hi = (h & 0xFFFFFu) | 0x3FF00000u;           // m bits 32..51, exponent 0
    const uint32_t chi = 0x40000000u - (h & 0x100000u);         // 2.0, or 1.0 for bit 52
    return __hiloint2double((int)hi, (int)lo) - __hiloint2double((int)chi, 0);
}

// OR of the G-bit groups of a wave-wide ballot: bit q is set when lane q of
// any group of G lanes had its predicate set.
template <int G>
__device__ __forceinline__ uint64_t fold_groups(uint64_t v)
{
#pragma unroll
    for (int sh = 32; sh >= G; sh >>= 1) v |= v >> sh;
    return G == 64 ? v : (v & ((1ull << G) - 1ull));
}

// Orders LDS accesses of the lanes of one wave.
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// One Marsaglia attempt from a Philox block: the two 53-bit uniforms on
// [-1, 1) (always set) and whether the pair lies strictly inside the unit
// disc, off its centre.
__device__ __forceinline__ bool marsaglia_pair(const Philox4 q, double &u1, double &u2)
{
    u1 = uniform53(q.x0, q.x1);
    u2 = uniform53(q.x2, q.x3);
    const double ss = u1 * u1 + u2 * u2;
    return ss < 1.0 && ss != 0.0;
}

// Row length (in elements) of the bead array for cpb chains per block.
// Bead j of chain c is element j row + (c ^ ((j H) mod cpb)), H = 32 / G,
// an (x, y, z) triple of 24 bytes.  A wave reads binary64 words half a wave
// at a time over 64 four-byte banks; the culling pass has lane t of chain c
// read bead b0 + t (b0 a multiple of G), and with cpb = 32 (G = 8, 256
// threads) the 32 (t, c) pairs of a half wave then fall on distinct
// elements modulo 32, whose 24-byte strides cover distinct bank pairs, as
// do the other accesses, where all chains of a wave read the same bead
// index.  Smaller cpb leaves at most 2-way conflicts (4-way for G = 32 in
// 256-thread blocks).  G = 64 (one chain per wave) uses an odd row and no
// swizzle instead.
__host__ __device__ inline int plane_row(int cpb, int G) { return G == 64 ? (cpb | 1) : cpb; }

// Bead e of an (x, y, z) triple array.  LDS serves 8-byte reads over 32
// banks of 8 bytes, 32 lanes per pass; the swizzle of plane_row puts the
// lanes of a pass on distinct banks for each 8-byte read, but a 16-byte read
// of the x, y pair (which the compiler would otherwise merge the first two
// into) spans two banks per lane and meets 2-way conflicts.  The empty asm
// statements keep the three reads apart.
template <bool HBM>
__device__ __forceinline__ void load_bead(const double *P, int e, double &x, double &y, double &z)
{
    if constexpr (HBM) {
        const double *q = P + 3 * e;
        x = q[0]; y = q[1]; z = q[2];
    } else {
        typedef const double __attribute__((address_space(3))) *lds_ptr;
        lds_ptr q = (lds_ptr)(P + 3 * e);
        x = q[0];
        asm volatile("" : "+v"(q));
        y = q[1];
        asm volatile("" : "+v"(q));
        z = q[2];
    }
}

// Accepted Marsaglia pairs a trial lane keeps ahead of the current step.
constexpr int kQueue = 4;

// Lockstep kernel: the chains of a block grow step by step together.
template <int G>
__device__ __forceinline__ void grow_real_body(const GrowArgs &a, uint64_t bid)
{
    extern __shared__ double lds[]; // [N][row] (x, y, z) bead triples, swizzled

    const int cpb = blockDim.x / G;
    // wave-uniform: bead offsets of uniform bead indices stay scalar
    const int row = __builtin_amdgcn_readfirstlane(plane_row(cpb, G));
    const int swz_mul = G == 64 ? 0 : 32 / G;
    const int swz_mask = cpb - 1;
    const int N = a.n_monomers;
    double *P = lds;
    const int t = threadIdx.x & (G - 1);
    const int chb = threadIdx.x / G;
    const int lane = threadIdx.x & 63;
    const int gbase = lane & ~(G - 1);
    // element of bead j of this chain
    const auto at = [&](int j) { return j * row + (chb ^ ((j * swz_mul) & swz_mask)); };
    // bead b0 + t for b0 a multiple of G: (b0 H) mod cpb = 0 (32 divides b0 H
    // and cpb <= 32), so its element is b0 row + at(t); elements past the
    // last one are clamped to it (their results are discarded)
    const int at_lane = at(t);
    const int last_el = N * row - 1;
    const uint64_t gmask_bits = (G == 64) ? ~0ull : ((1ull << G) - 1ull);
    const uint64_t c = bid * cpb + chb;
    const bool valid = c < a.n_chains;
    const uint64_t g = a.chain_offset + c;
    const int k = a.k_trials;
    const bool has_trial = t < k;
    // Round 1 of the Marsaglia draws spreads attempts 0 .. reps-1 of the k
    // trials over the G lanes of the chain: lane t tries attempt t / k of
    // trial t mod k (G >= k).  Used when reps >= 4, where a second round is
    // rarely needed (measured 1.08-1.36x faster for k = 8, 256 <= N <= 1536);
    // otherwise each trial lane draws its own trial ahead through its queue.
    const int reps = G / k;
    bool spread = false;
    if constexpr (G >= 32) spread = reps >= 4;
    const uint32_t r1_trial = (uint32_t)(t % k), r1_att = (uint32_t)(t / k);
    const bool r1_lane = t < reps * k;
    uint64_t r1_pattern = 0; // bits 0, k, 2k, ...: the lanes of one trial
    for (int q = 0; q < reps; ++q) r1_pattern |= 1ull << (q * k);
    // a double from lane src of the wave
    const auto pull_from = [](int src, double v) {
        const int64_t bits = __double_as_longlong(v);
        const int lo = __builtin_amdgcn_ds_bpermute(src * 4, (int)(uint32_t)bits);
        const int hi = __builtin_amdgcn_ds_bpermute(src * 4, (int)(uint32_t)(bits >> 32));
        return __longlong_as_double((int64_t)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo));
    };
    const double b = a.bond_length;
    const double sigma2 = a.sigma2;
    const double cull2 = a.cull2;

    if (t == 0) {
        const int o = 3 * at(0);
        P[o] = 0.0; P[o + 1] = 0.0; P[o + 2] = 0.0;
    }
    __syncthreads();

    double tx = 0.0, ty = 0.0, tz = 0.0;
    bool alive = false;
    int grown = 1;
    uint32_t n_mine = 0; // steps with m = t + 1 (lane t counts one value of m)
    bool rng_fail = false;
    Philox4 sel{0, 0, 0, 0};
    // this lane's queue: q1[0..lvl), q2[0..lvl) hold the accepted pairs of
    // trial t for steps i, i + 1, ...; the next draw is step nstep, attempt natt
    double q1[kQueue], q2[kQueue];
#pragma unroll
    for (int q = 0; q < kQueue; ++q) { q1[q] = 0.0; q2[q] = 0.0; }
    int lvl = 0;
    uint32_t nstep = 1, natt = 0;
    // the attempt that ends the chain: the first complete one, or the last
    // allowed one (one attempt without restarts); bead 0 stays at the origin
    bool res_alive = false;
    double res_lw = -__builtin_huge_val();
    bool pending = valid;

    for (uint32_t rd = 0; rd < a.max_rounds; ++rd) {
        if (pending) {
            tx = 0.0; ty = 0.0; tz = 0.0;
            n_mine = 0;
            lvl = 0; nstep = 1; natt = 0;
        }
        alive = pending;
        grown = 1;
        const uint32_t hi = rd << 16; // attempt in the high half of the step word
        // One production round of the trial queues: each lane with room
        // tries its next attempt; an accepted pair joins the queue and the
        // lane moves on to the next step (a lane reaching the attempt cap
        // queues its last pair and reports the failure).  Every step runs one
        // round while its first bead reads are in flight, and more at its end
        // until every lane that grows a trial at the next step holds its pair.
        const auto round = [&]() {
            const bool room = alive && has_trial && lvl < kQueue && nstep < (uint32_t)N;
            double u1, u2;
            const bool ok = marsaglia_pair(draw(a.seed, g, nstep | hi, (uint32_t)t, natt), u1, u2);
            const bool capped = !ok && natt + 1u == kMaxAttempt;
            const bool put = room && (ok || capped);
            rng_fail = rng_fail || (room && capped);
#pragma unroll
            for (int q = 0; q < kQueue; ++q) {
                const bool here = put && lvl == q;
                q1[q] = here ? u1 : q1[q];
                q2[q] = here ? u2 : q2[q];
            }
            lvl += put ? 1 : 0;
            nstep += put ? 1u : 0u;
            natt = put ? 0u : natt + (room ? 1u : 0u);
        };
        // a lane starves when its queue is empty and the step it needs next
        // (nstep, when the queue is empty) exists; a starving lane always has
        // room, so every round moves it on (an acceptance, or its attempt cap)
        const auto starving = [&]() { return alive && has_trial && lvl == 0 && nstep < (uint32_t)N; };
        if (!spread)
            while (__ballot(starving()) != 0) round();

        for (int i = 1; i < N; ++i) {
            // 1. Marsaglia direction of trial t: the first accepted attempt.
            double v1 = 0.0, v2 = 0.0, s = 0.5;
            const bool need = alive && has_trial;
            if (!spread) {
                v1 = q1[0]; v2 = q2[0];
#pragma unroll
                for (int q = 0; q + 1 < kQueue; ++q) { q1[q] = q1[q + 1]; q2[q] = q2[q + 1]; }
                if (need) --lvl;
                s = v1 * v1 + v2 * v2;
            } else {
                // Round 1: the chain's G lanes try attempts 0 .. reps-1 of its
                // k trials (lane u: trial u mod k, attempt u / k) and each
                // trial takes its smallest accepted one.  Round 2 (when a
                // trial failed all of them): the 64 lanes of the wave serve
                // the failed trials, lane l taking the failed trial of rank
                // q = l mod nF at attempt reps + l / nF; each failed trial then
                // takes its first accepting helper in lane order, which is its
                // smallest accepted attempt.  Values move through the
                // cross-lane permute network (no LDS storage).  A trial whose
                // helpers all rejected continues alone after its last helped
                // attempt.
                double w1 = 0.0, w2 = 0.0;
                const bool wok = marsaglia_pair(draw(a.seed, g, (uint32_t)i | hi, r1_trial, r1_att), w1, w2) &
                                 r1_lane;
                const uint64_t B = (__ballot(wok) >> gbase) & gmask_bits;
                const uint64_t cand = has_trial ? ((B >> t) & r1_pattern) : 0ull;
                const int src = cand ? gbase + t + __builtin_ctzll(cand) : lane;
                v1 = pull_from(src, w1);
                v2 = pull_from(src, w2);
                bool acc = cand != 0;
                uint32_t att = (uint32_t)reps; // the next attempt of a trial still failing
                const uint64_t F = __ballot(need && !acc);
                if (F != 0) {
                    const uint32_t nF = (uint32_t)__popcll(F);
                    const bool failing = need && !acc;
                    const uint32_t rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(F >> 32),
                                          __builtin_amdgcn_mbcnt_lo((uint32_t)F, 0u));
                    // lane q < nF learns the lane of the failed trial of rank q
                    const int owner_of_q = __builtin_amdgcn_ds_permute((int)((failing ? rank : 63u) * 4u), lane);
                    // l / nF and l mod nF (l < 64: the float quotient is never
                    // within rounding of an integer boundary)
                    const uint32_t jh = (uint32_t)(((float)lane + 0.5f) * __builtin_amdgcn_rcpf((float)nF));
                    const uint32_t q = (uint32_t)lane - jh * nF;
                    const int owner = __builtin_amdgcn_ds_bpermute((int)(q * 4u), owner_of_q);
                    const uint64_t og = a.chain_offset + bid * cpb +
                                        (uint64_t)(((threadIdx.x & ~63) + (owner & ~(G - 1))) / G);
                    double h1 = 0.0, h2 = 0.0;
                    const bool hok = marsaglia_pair(draw(a.seed, og, (uint32_t)i | hi,
                                                         (uint32_t)(owner & (G - 1)), att + jh),
                                                    h1, h2);
                    const uint64_t H = __ballot(hok);
                    // helpers of rank r are lanes r, r + nF, r + 2 nF, ...
                    uint64_t pattern = 0;
                    for (uint32_t l = 0; l < 64u; l += nF) pattern |= 1ull << l;
                    const uint64_t mine = failing ? (H & (pattern << rank)) : 0ull;
                    const int hsrc = mine ? __builtin_ctzll(mine) : lane;
                    const double n1 = pull_from(hsrc, h1), n2 = pull_from(hsrc, h2);
                    if (failing) {
                        if (mine) {
                            v1 = n1; v2 = n2;
                            acc = true;
                        } else {
                            att = att + (64u - rank + nF - 1u) / nF;
                        }
                    }
                }
                // round 3 (rare): the remaining trials continue alone
                bool done = !need || acc;
                while (!done) {
                    double u1, u2;
                    if (marsaglia_pair(draw(a.seed, g, (uint32_t)i | hi, (uint32_t)t, att), u1, u2)) {
                        v1 = u1; v2 = u2;
                        done = true;
                    } else if (++att == kMaxAttempt) {
                        rng_fail = true;
                        done = true;
                    }
                }
                s = v1 * v1 + v2 * v2;
            }
            const double qf = 2.0 * sqrt_unit(1.0 - s); // 1 - s in [2^-53, 1)
            const double ex = v1 * qf, ey = v2 * qf, ez = 1.0 - 2.0 * s;
            const double cx = tx + b * ex, cy = ty + b * ey, cz = tz + b * ez;

            // 2-3. exact test of this lane's candidate: beads i-2 and i-3 (within
            // 2b of the tip) directly, beads 0 .. i-4 after the culling pass
            bool blocked = false; // bitwise accumulation keeps the tests branch-free
            const auto test_el = [&](int e) {
                double x, y, z;
                load_bead<false>(P, e, x, y, z);
                const double dx = cx - x, dy = cy - y, dz = cz - z;
                double d2 = dx * dx + dy * dy;
                d2 = d2 + dz * dz;
                blocked = blocked | (d2 < sigma2);
            };
            const auto is_near_el = [&](int e) {
                double x, y, z;
                load_bead<false>(P, e, x, y, z);
                const double dx = x - tx, dy = y - ty, dz = z - tz;
                double d2 = dx * dx + dy * dy;
                d2 = d2 + dz * dz;
                return !(d2 >= cull2);
            };
            {
                // beads i-2 and i-3 (masked before step 2 and 3): reads, one
                // production round while they are in flight, tests
                double x2, y2, z2, x3, y3, z3;
                load_bead<false>(P, at(i >= 2 ? i - 2 : 0), x2, y2, z2);
                load_bead<false>(P, at(i >= 3 ? i - 3 : 0), x3, y3, z3);
                if (!spread) {
                    round();
                    // keeps the round here, ahead of the tests that wait for the reads
                    asm volatile("" ::"v"(lvl), "v"(natt));
                }
                const auto overlaps = [&](double x, double y, double z) {
                    const double dx = cx - x, dy = cy - y, dz = cz - z;
                    double d2 = dx * dx + dy * dy;
                    d2 = d2 + dz * dz;
                    return d2 < sigma2;
                };
                const bool o2 = overlaps(x2, y2, z2), o3 = overlaps(x3, y3, z3);
                blocked = (i >= 2 && o2) || (i >= 3 && o3);
            }
            const int nb = __builtin_amdgcn_readfirstlane(i - 3);
            // Culling passes of two blocks of G beads, lane t taking beads
            // b0 + t and b0 + G + t; the offsets flagged by any chain of the
            // wave are re-tested exactly by every chain (a culled bead cannot
            // overlap, so testing it again changes nothing), two at a time so
            // that their reads are in flight together.  (Four blocks per pass
            // measured 4 % slower at N = 64, k = 8.)
            constexpr int PB = 2;
            const auto retest = [&](uint64_t u, int base) {
                while (u) {
                    const int qa = __builtin_ctzll(u);
                    u &= u - 1;
                    if (u) {
                        const int qb = __builtin_ctzll(u);
                        u &= u - 1;
                        double xa, ya, za, xb, yb, zb;
                        load_bead<false>(P, at(base + qa), xa, ya, za);
                        load_bead<false>(P, at(base + qb), xb, yb, zb);
                        const auto hit = [&](double x, double y, double z) {
                            const double dx = cx - x, dy = cy - y, dz = cz - z;
                            double d2 = dx * dx + dy * dy;
                            d2 = d2 + dz * dz;
                            return d2 < sigma2;
                        };
                        const bool ha = hit(xa, ya, za), hb = hit(xb, yb, zb);
                        blocked = blocked || ha || hb;
                    } else {
                        test_el(at(base + qa));
                    }
                }
            };
            for (int b0 = 0; b0 < nb; b0 += PB * G) {
                bool nearv[PB];
#pragma unroll
                for (int pb = 0; pb < PB; ++pb) {
                    const int e = min((b0 + pb * G) * row + at_lane, last_el);
                    nearv[pb] = alive & (b0 + pb * G + t < nb) & is_near_el(e);
                }
                if constexpr (PB * G <= 64) {
                    uint64_t u = 0;
#pragma unroll
                    for (int pb = 0; pb < PB; ++pb) u |= fold_groups<G>(__ballot(nearv[pb])) << (pb * G);
                    retest(u, b0);
                } else {
#pragma unroll
                    for (int pb = 0; pb < PB; ++pb) retest(fold_groups<G>(__ballot(nearv[pb])), b0 + pb * G);
                }
            }

            const bool fr = alive & has_trial & !blocked;

            // 4. free mask of the group and m
            const uint64_t bal = __ballot(fr);
            const uint64_t gm = (bal >> gbase) & gmask_bits;
            const uint32_t m = (uint32_t)__popcll(gm);

            // 5. uniform pick among the free trials (16-bit Lemire word)
            if (i == 1 || (i & 7) == 0) sel = draw(a.seed, g, (uint32_t)(i >> 3) | hi, kSlotSelect, 0);
            const uint32_t x = half_word(sel, (uint32_t)(i & 7));
            const uint32_t p = x * m;
            uint32_t r = p >> 16;
            if (__builtin_expect(alive && (p & 0xFFFFu) < m, 0)) {
                r = lemire_redraw16(a.seed, g, (uint32_t)i | hi, m, x);
                if (r == kPickFailed) {
                    rng_fail = true;
                    r = 0;
                }
            }
            const uint64_t below = (t == 0) ? 0ull : (gm & ((1ull << t) - 1ull));
            const bool chosen = fr && ((uint32_t)__popcll(below) == r);
            const uint64_t cb = __ballot(chosen);
            const uint64_t gcb = (cb >> gbase) & gmask_bits;
            const int src = gbase + (gcb ? (__ffsll((long long)gcb) - 1) : 0);
            const double nx = __shfl(cx, src, 64);
            const double ny = __shfl(cy, src, 64);
            const double nz = __shfl(cz, src, 64);

            if (alive && m == 0) {
                alive = false;
                grown = i;
            }
            if (alive) {
                if (chosen) {
                    const int o = 3 * at(i);
                    P[o] = nx; P[o + 1] = ny; P[o + 2] = nz;
                }
                tx = nx; ty = ny; tz = nz;
                n_mine += (m == (uint32_t)t + 1u) ? 1u : 0u;
            }
            if (!spread)
                while (__ballot(starving()) != 0) round();
            wave_sync();
            // long chains: once every chain of the wave has ended (most hard-sphere
            // chains beyond a few hundred beads meet a dead end), the wave leaves
            // the step loop instead of running the remaining steps on dead
            // chains (N = 1000, 2 10^4 chains: 22.9 -> 7.6 ms; N = 3000:
            // 45.9 -> 6.7 ms); at N <= 256 the test costs more than it saves
            if (N > 256 && __ballot(alive) == 0) break;
        }
        if (alive) grown = N;
        const bool ends = pending && (alive || rd + 1 >= a.max_rounds);

        // log W = sum over m = 1..k, ascending, of n_m log m (Eq. 3 grouped by
        // value); n_m is held by lane m - 1 of the group
        double lw = 0.0;
        for (int mm = 1; mm <= k; ++mm) {
            const uint32_t nm = __shfl(n_mine, gbase + mm - 1, 64);
            lw = lw + (double)nm * a.logm[mm];
        }
        if (!alive) lw = -__builtin_huge_val();

        // observables, lane 0 of the group, in bead order
        if (ends && t == 0 && valid) {
            double sx = 0.0, sy = 0.0, sz = 0.0;
            for (int j = 0; j < grown; ++j) {
                const int o = 3 * at(j);
                sx = sx + P[o]; sy = sy + P[o + 1]; sz = sz + P[o + 2];
            }
            const double gd = (double)grown;
            const double cmx = sx / gd, cmy = sy / gd, cmz = sz / gd;
            double acc = 0.0;
            for (int j = 0; j < grown; ++j) {
                const int o = 3 * at(j);
                const double dx = P[o] - cmx, dy = P[o + 1] - cmy, dz = P[o + 2] - cmz;
                double q = dx * dx + dy * dy;
                q = q + dz * dz;
                acc = acc + q;
            }
            const int oe = 3 * at(grown - 1);
            const double ex = P[oe], ey = P[oe + 1], ez = P[oe + 2];
            double r2 = ex * ex + ey * ey;
            r2 = r2 + ez * ez;
            if (a.log_w) a.log_w[c] = lw;
            if (a.r_end) {
                double *o = (double *)a.r_end;
                o[c] = ex; o[a.n_chains + c] = ey; o[2 * a.n_chains + c] = ez;
            }
            if (a.r2) a.r2[c] = r2;
            if (a.rg2) a.rg2[c] = acc / gd;
            if (a.n_grown) a.n_grown[c] = (uint16_t)grown;
        }
        if (ends) {
            res_alive = alive;
            res_lw = lw;
            pending = false;
        }
        if (__ballot(pending) == 0) break;
    }
    if (rng_fail) atomicExch(a.status, 6);
    const uint64_t bits = (res_alive && t == 0) ? (uint64_t)__double_as_longlong(res_lw) : 0ull;
    publish_log_w_max(a, bits);
}

template <int G>
__global__ __launch_bounds__(256) void grow_real_tp(GrowArgs a, uint64_t base)
{
    grow_real_body<G>(a, base + blockIdx.x);
}

// Batched launch: block b serves the ensemble whose block range holds b.
template <int G>
__global__ __launch_bounds__(256) void grow_real_tp_batch(const GrowEntry *tab, const uint64_t *block0, int n,
                                                          uint64_t base)
{
    const uint64_t bid = base + blockIdx.x;
    const int e = find_segment(block0, n, bid);
    grow_real_body<G>(tab[e].a, bid - block0[e]);
}

// ---------------------------------------------------------------------------
// Queued kernel: chains too long for eight of them to a wave's LDS, and those
// whose beads live in global memory.  G lanes per chain (16, 32 or 64), one
// wave per block; a group takes its next chain from a queue (a counter in the
// workspace) as its chain ends, so dead ends, which stop most long hard-sphere
// chains early, idle a group for at most the rest of eight steps.  i mod 8 is
// common to the wave, everything else is the group's own.
//
// Directions.  With kp = the power of two >= k, a group has PH = G / kp (at
// most 8) sets of trial lanes: lane t draws trial t mod kp of the steps
// i = t / kp (mod PH), ahead through a two-entry queue, and owns that trial's
// candidate when such a step comes.  One production round then serves up to PH
// steps of every chain (a direction takes 4 / pi attempts, so 0.32 rounds per
// step at best with PH = 4, where a round for one step's trials alone needs
// more than one).
//
// Culling as above, over all G lanes; beads i-2 and i-3 stay in registers.
// Flagged beads are tested by their own group only.  With one chain per wave
// (G = 64) a full block of 64 beads whose nearest bead is D from the tip is
// not scanned again before the tip can have come D - (b + sigma) closer, b
// per step (real_skip.hpp).
//
// Bound by VALU issue at N = 256 (0.74-0.81 of the slots, counters) and by the
// longest surviving chains' serial steps at N = 3000.  MI355X, whole calls,
// k = 8, lockstep -> queued: N = 256, 2 10^5 chains, 17.0 -> 13.4 ms; N = 3000,
// 3000 chains, 6.6 -> 3.4 ms.
// ---------------------------------------------------------------------------

// Smallest of the 64 lanes' non-negative values, in every lane (their bit
// patterns order like the values).
__device__ __forceinline__ float wave_min(float v)
{
    int x = __float_as_int(v);
    const auto least = [](int a, int b) { return a < b ? a : b; };
    x = least(x, __builtin_amdgcn_update_dpp(0, x, 0xB1, 0xF, 0xF, false));
    x = least(x, __builtin_amdgcn_update_dpp(0, x, 0x4E, 0xF, 0xF, false));
    x = least(x, __builtin_amdgcn_update_dpp(0, x, 0x141, 0xF, 0xF, false));
    x = least(x, __builtin_amdgcn_update_dpp(0, x, 0x140, 0xF, 0xF, false));
    const auto p = __builtin_amdgcn_permlane16_swap((uint32_t)x, (uint32_t)x, false, false);
    x = least((int)p[0], (int)p[1]);
    const auto q = __builtin_amdgcn_permlane32_swap((uint32_t)x, (uint32_t)x, false, false);
    return __int_as_float(least((int)q[0], (int)q[1]));
}

// A double from lane `src` (uniform) of the wave.
__device__ __forceinline__ double lane_double(double v, int src)
{
    const int64_t bits = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)(uint32_t)bits, src);
    const int hi = __builtin_amdgcn_readlane((int)(uint32_t)(bits >> 32), src);
    return __longlong_as_double((int64_t)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo));
}

// Blocks of 64 beads of the longest chain, per lane.
constexpr int kDueRegs = 4;

// Beads of a chain in global memory that LDS holds as well, the latest ones
// (a multiple of 64): the blocks scanned at every step are among them.
constexpr int kRing = 256;

// Doubles between the chains of a block: lanes G .. 2 G - 1 of a half wave
// read on from the banks of lanes 0 .. G - 1 (3 G mod 32 eight-byte banks).
__host__ __device__ inline int queue_stride(int N, int G)
{
    if (G != 16) return 3 * N;
    return (3 * N + 15) / 32 * 32 + 16;
}

template <int G, bool HBM>
__device__ __forceinline__ void grow_real_queue_body(const GrowArgs &a, uint32_t block, uint32_t blocks,
                                                     double *planes, double *ring)
{
    constexpr uint32_t CPB = 64 / G;
    static_assert(!HBM || G == 64, "global planes hold one chain per wave");
    constexpr int kAhead = 2;
    const int lane = threadIdx.x & 63;
    const int t = lane & (G - 1);
    const int gbase = lane & ~(G - 1);
    const int N = a.n_monomers;
    const int k = a.k_trials;
    int kp = 1;
    while (kp < k) kp <<= 1;
    const int PH = G / kp < 8 ? G / kp : 8;
    const int trial = t & (kp - 1), phase = t / kp;
    const bool draws = trial < k && phase < PH;
    const uint64_t kmask = kp == 64 ? ~0ull : (1ull << kp) - 1ull;
    const uint64_t lower = (1ull << trial) - 1ull;
    const int stride = queue_stride(N, G);
    double *P = planes + (lane / G) * stride;
    const double b = a.bond_length;
    const double sigma2 = a.sigma2, cull2 = a.cull2;
    const double unit = skip_unit(b);
    const float reach = skip_reach(cull2, unit);

    double tx = 0.0, ty = 0.0, tz = 0.0;                       // bead i-1
    double x2 = 0.0, y2 = 0.0, z2 = 0.0, x3 = 0.0, y3 = 0.0, z3 = 0.0; // beads i-2, i-3
    double q1[kAhead] = {0.0, 0.0}, q2[kAhead] = {0.0, 0.0};   // accepted pairs
    int lvl = 0;
    uint32_t nstep = 1, natt = 0;                              // the next draw
    int due[kDueRegs] = {0, 0, 0, 0};                          // G = 64: lane l, blocks l, l + 64, ...
    bool busy = false, alive = false, rng_fail = false;
    int placed = 1, i0 = 0;
    uint32_t n_mine = 0; // steps with m = t + 1
    uint32_t rd = 0;
    uint64_t c = 0, best = 0;
    // the wave's share of the queue: to begin with a chain for each group, its
    // own without asking; the counter holds what was taken of the others
    const uint32_t resident = blocks * CPB;
    uint64_t next = (uint64_t)block * CPB;
    uint64_t end = next + CPB < a.n_chains ? next + CPB : a.n_chains;
    uint32_t left = a.n_chains > resident ? (uint32_t)(a.n_chains - resident) : 0u; // as last seen
    bool drained = false;
    // Chains in global memory that end within a few beads (k b / sigma <= 2.25):
    // the counter would bound them, so that a wave takes half of its share, at
    // most 8 (N = 3000, sigma = 1, 10^5 chains, k = 1, 1.26 -> 0.57 ms; k = 2, 1.33
    // -> 1.06; but k = 4, sigma = 0.4, 2 10^4 chains, 32 -> 38, where many chains
    // live long and the rest should not wait for them).
    const bool brief = 16.0 * ((double)(k * k) * (b * b)) <= 81.0 * sigma2;

    const auto start = [&]() { // the chain's next attempt
        alive = N > 1;
        placed = 1;
        i0 = 0;
        n_mine = 0;
        tx = ty = tz = 0.0;
        x2 = y2 = z2 = x3 = y3 = z3 = 0.0;
        lvl = 0;
        nstep = phase == 0 ? (uint32_t)PH : (uint32_t)phase;
        natt = 0;
#pragma unroll
        for (int q = 0; q < kDueRegs; ++q) due[q] = 0;
        if (t == 0) {
            P[0] = 0.0; P[1] = 0.0; P[2] = 0.0;
            if constexpr (HBM) {
                ring[0] = 0.0; ring[1] = 0.0; ring[2] = 0.0;
            }
        }
    };

    for (;;) {
        // ended chains, the whole wave taking each in turn
        const bool ended = busy && !alive;
        const bool again = ended && placed < N && rd + 1 < a.max_rounds;
        for (uint64_t todo = __ballot(ended && !again && t == 0); todo; todo &= todo - 1) {
            const int src = __builtin_ctzll(todo);
            const double *B = planes + (src / G) * stride;
            const int n = __builtin_amdgcn_readlane(placed, src);
            const double gd = (double)n;
            // coordinate sums in bead order: lanes 0, 1, 2 take x, y, z
            double s = 0.0;
            const double *Bc = B + lane % 3;
#pragma unroll 8
            for (int j = 0; j < n; ++j) s = s + Bc[3 * j];
            const double cm = s / gd;
            const double cmx = lane_double(cm, 0), cmy = lane_double(cm, 1), cmz = lane_double(cm, 2);
            double acc = 0.0;
            for (int j0 = 0; j0 < n; j0 += 64) {
                double x, y, z;
                load_bead<HBM>(B, min(j0 + lane, n - 1), x, y, z);
                const double dx = x - cmx, dy = y - cmy, dz = z - cmz;
                double q = dx * dx + dy * dy;
                q = q + dz * dz;
                const int nj = min(64, n - j0);
                for (int j = 0; j < nj; ++j) acc = acc + lane_double(q, j);
            }
            // log W = sum over m = 1..k, ascending, of n_m log m
            double lw = 0.0;
            for (int mm = 1; mm <= k; ++mm) {
                const uint32_t nm = (uint32_t)__builtin_amdgcn_readlane((int)n_mine, src + mm - 1);
                lw = lw + (double)nm * a.logm[mm];
            }
            if (n < N) lw = -__builtin_huge_val();
            if (lane == src) {
                double r2 = tx * tx + ty * ty;
                r2 = r2 + tz * tz;
                if (a.log_w) a.log_w[c] = lw;
                if (a.r_end) {
                    double *o = (double *)a.r_end;
                    o[c] = tx; o[a.n_chains + c] = ty; o[2 * a.n_chains + c] = tz;
                }
                if (a.r2) a.r2[c] = r2;
                if (a.rg2) a.rg2[c] = acc / gd;
                if (a.n_grown) a.n_grown[c] = (uint16_t)n;
                const uint64_t bits = n == N ? (uint64_t)__double_as_longlong(lw) : 0ull;
                best = bits > best ? bits : best;
            }
        }
        wave_sync();
        if (ended) {
            busy = again;
            if (again) {
                ++rd;
                start();
            }
        }
        // groups without a chain take the next ones of the queue
        for (;;) {
            const uint64_t want = __ballot(!busy && t == 0);
            if (want == 0 || drained) break;
            if (next == end) {
                if (left == 0) {
                    drained = true;
                    break;
                }
                // A chain taken and not wanted waits for another of the wave's
                // groups to end (single chains waited 340 of a call's 620 us:
                // N = 213, k = 8, 4000 chains), so a wave takes what it wants,
                // and more (fewer atomics, 11-14 ns each on the one counter) only
                // while plenty are left.
                uint32_t take = (uint32_t)__builtin_popcountll(want);
                if constexpr (HBM) {
                    const uint32_t share = left / (2u * resident);
                    take = brief && left >= resident ? (share < 2u ? 2u : (share < 8u ? share : 8u)) : take;
                } else {
                    if (left >= resident) take = CPB;
                }
                unsigned long long v = 0;
                if (lane == 0) v = atomicAdd(a.queue, (unsigned long long)take);
                next = resident + (((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32)) << 32) |
                                   (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v));
                end = next + take < a.n_chains ? next + take : a.n_chains;
                left = (uint32_t)(a.n_chains - end);
                if (next >= a.n_chains) {
                    drained = true;
                    break;
                }
            }
            const uint64_t rank = __builtin_popcountll(want & ((1ull << gbase) - 1ull));
            const uint64_t n = (uint64_t)__builtin_popcountll(want);
            if (!busy && rank < end - next) {
                busy = true;
                c = next + rank;
                rd = 0;
                start();
            }
            next += n < end - next ? n : end - next;
        }
        wave_sync();
        if (__ballot(busy) == 0) break;

        const uint64_t g = a.chain_offset + c;
        const uint32_t hi = rd << 16;
        const Philox4 sel = draw(a.seed, g, (uint32_t)(i0 >> 3) | hi, kSlotSelect, 0);
#pragma unroll 1
        for (int e = 0; e < 8; ++e) {
            const int i = i0 + e;
            const int ph = e & (PH - 1);
            const bool act = alive && i > 0; // step 0 places nothing
            const bool owns = draws && phase == ph;
            // production rounds until every trial of this step has its pair:
            // each lane with room tries its next attempt
            while (__ballot(act && owns && lvl == 0) != 0) {
                const bool room = alive && draws && lvl < kAhead && nstep < (uint32_t)N;
                double u1, u2;
                const bool ok = marsaglia_pair(draw(a.seed, g, nstep | hi, (uint32_t)trial, natt), u1, u2);
                const bool capped = !ok && natt + 1u == kMaxAttempt;
                const bool put = room && (ok || capped);
                rng_fail = rng_fail || (room && capped);
#pragma unroll
                for (int q = 0; q < kAhead; ++q) {
                    const bool here = put && lvl == q;
                    q1[q] = here ? u1 : q1[q];
                    q2[q] = here ? u2 : q2[q];
                }
                lvl += put ? 1 : 0;
                nstep += put ? (uint32_t)PH : 0u;
                natt = put ? 0u : natt + (room ? 1u : 0u);
            }
            const double v1 = q1[0], v2 = q2[0];
            const bool takes = act && owns;
            q1[0] = takes ? q1[1] : q1[0];
            q2[0] = takes ? q2[1] : q2[0];
            lvl -= takes ? 1 : 0;
            const double s = v1 * v1 + v2 * v2;
            const double qf = 2.0 * sqrt_unit(1.0 - s); // 1 - s in [2^-53, 1]
            const double ex = v1 * qf, ey = v2 * qf, ez = 1.0 - 2.0 * s;
            const double cx = tx + b * ex, cy = ty + b * ey, cz = tz + b * ez;

            const auto overlaps = [&](double x, double y, double z) {
                const double dx = cx - x, dy = cy - y, dz = cz - z;
                double d2 = dx * dx + dy * dy;
                d2 = d2 + dz * dz;
                return d2 < sigma2;
            };
            const auto tip_dist2 = [&](double x, double y, double z) {
                const double dx = x - tx, dy = y - ty, dz = z - tz;
                double d2 = dx * dx + dy * dy;
                d2 = d2 + dz * dz;
                return d2;
            };
            bool blocked = ((i >= 2) & overlaps(x2, y2, z2)) | ((i >= 3) & overlaps(x3, y3, z3));
            const int nb = act ? i - 3 : 0; // beads 0 .. nb-1 are culled, then tested
            if constexpr (G == 64) {
                const int nbu = __builtin_amdgcn_readfirstlane(nb);
                const int iu = __builtin_amdgcn_readfirstlane(i);
                // bead base + o of a block; the block's beads, if among the
                // last kRing, come from LDS
                const auto bead = [&](int base, int o, double &x, double &y, double &z) {
                    if (HBM && base + kRing >= iu) load_bead<false>(ring, (base & (kRing - 1)) + o, x, y, z);
                    else load_bead<HBM>(P, min(base + o, N - 1), x, y, z);
                };
                const auto retest = [&](uint64_t u, int base) {
                    for (; u; u &= u - 1) {
                        double x, y, z;
                        bead(base, __builtin_ctzll(u), x, y, z);
                        blocked = blocked | overlaps(x, y, z);
                    }
                };
#pragma unroll
                for (int rg = 0; rg < kDueRegs; ++rg) {
                    if (4096 * rg >= nbu) break;
                    uint64_t todo = __ballot(due[rg] <= i && 4096 * rg + 64 * lane < nbu);
                    while (todo) { // two due blocks at a time
                        const int qa = __builtin_ctzll(todo);
                        todo &= todo - 1;
                        const bool two = todo != 0;
                        const int qb = two ? __builtin_ctzll(todo) : qa;
                        todo &= todo - 1; // 0 stays 0
                        const int ba = 4096 * rg + 64 * qa, bb = 4096 * rg + 64 * qb;
                        double xa, ya, za, xb, yb, zb;
                        bead(ba, t, xa, ya, za);
                        bead(bb, t, xb, yb, zb);
                        const double da = tip_dist2(xa, ya, za), db = tip_dist2(xb, yb, zb);
                        const uint64_t ua = __ballot(ba + t < nbu && !(da >= cull2)),
                                       ub = __ballot(two && bb + t < nbu && !(db >= cull2));
                        retest(ua, ba);
                        retest(ub, bb);
                        const auto next_due = [&](double d2, uint64_t u, int b0) {
                            if (u != 0 || b0 + 64 > nbu) return i + 1;
                            return i + 1 + skip_steps(wave_min((float)(d2 * unit)), reach);
                        };
                        const int na = next_due(da, ua, ba);
                        due[rg] = lane == qa ? na : due[rg];
                        if (two) {
                            const int n2 = next_due(db, ub, bb);
                            due[rg] = lane == qb ? n2 : due[rg];
                        }
                    }
                }
            } else {
                int nbu = __builtin_amdgcn_readlane(nb, 0);
#pragma unroll
                for (int q = G; q < 64; q += G) {
                    const int o = __builtin_amdgcn_readlane(nb, q);
                    nbu = o > nbu ? o : nbu;
                }
                const uint32_t gm32 = G == 32 ? ~0u : (1u << (G & 31)) - 1u;
                for (int b0 = 0; b0 < nbu; b0 += 2 * G) {
                    double xa, ya, za, xb, yb, zb;
                    load_bead<HBM>(P, min(b0 + t, N - 1), xa, ya, za);
                    load_bead<HBM>(P, min(b0 + G + t, N - 1), xb, yb, zb);
                    const uint64_t ua = __ballot(b0 + t < nb && !(tip_dist2(xa, ya, za) >= cull2)),
                                   ub = __ballot(b0 + G + t < nb && !(tip_dist2(xb, yb, zb) >= cull2));
                    if ((ua | ub) == 0) continue;
                    // this group's flagged beads b0 + bit, two at a time
                    uint64_t f = (uint64_t)((uint32_t)(ua >> gbase) & gm32) |
                                 (uint64_t)((uint32_t)(ub >> gbase) & gm32) << G;
                    while (__ballot(f != 0) != 0) {
                        const bool one = f != 0;
                        const int ja = one ? __builtin_ctzll(f) : 0;
                        f &= f - (one ? 1 : 0);
                        const bool two = f != 0;
                        const int jb = two ? __builtin_ctzll(f) : ja;
                        f &= f - (two ? 1 : 0);
                        double px, py, pz, qx, qy, qz;
                        load_bead<HBM>(P, b0 + ja, px, py, pz);
                        load_bead<HBM>(P, b0 + jb, qx, qy, qz);
                        const bool ha = overlaps(px, py, pz), hb = overlaps(qx, qy, qz);
                        blocked = blocked | (one & (ha | hb));
                    }
                }
            }

            const bool fr = takes & !blocked;
            const uint64_t gm = (__ballot(fr) >> (gbase + ph * kp)) & kmask;
            const uint32_t m = (uint32_t)__popcll(gm);
            const uint32_t x = half_word(sel, (uint32_t)e);
            const uint32_t p = x * m;
            uint32_t r = p >> 16;
            if (__builtin_expect(act && (p & 0xFFFFu) < m, 0)) {
                r = lemire_redraw16(a.seed, g, (uint32_t)i | hi, m, x);
                if (r == kPickFailed) {
                    rng_fail = true;
                    r = 0;
                }
            }
            const bool chosen = fr && (uint32_t)__popcll(gm & lower) == r;
            const uint64_t cb = (__ballot(chosen) >> (gbase + ph * kp)) & kmask;
            const int src = gbase + ph * kp + (cb ? __builtin_ctzll(cb) : 0);
            double nx, ny, nz;
            if constexpr (G == 64) {
                const int usrc = __builtin_amdgcn_readfirstlane(src);
                nx = lane_double(cx, usrc); ny = lane_double(cy, usrc); nz = lane_double(cz, usrc);
            } else {
                nx = __shfl(cx, src, 64); ny = __shfl(cy, src, 64); nz = __shfl(cz, src, 64);
            }
            if (chosen) {
                double *o = P + 3 * i;
                o[0] = cx; o[1] = cy; o[2] = cz;
                if constexpr (HBM) {
                    double *w = ring + 3 * (i & (kRing - 1));
                    w[0] = cx; w[1] = cy; w[2] = cz;
                }
            }
            const bool ok = act && m != 0u;
            if (ok) {
                x3 = x2; y3 = y2; z3 = z2;
                x2 = tx; y2 = ty; z2 = tz;
                tx = nx; ty = ny; tz = nz;
                n_mine += (m == (uint32_t)t + 1u) ? 1u : 0u;
                ++placed;
            }
            alive = alive && (ok || !act) && placed < N;
            wave_sync();
        }
        i0 += 8;
    }
    if (rng_fail) atomicExch(a.status, 6);
    publish_log_w_max(a, best);
}

template <int G>
__global__ __launch_bounds__(64) void grow_real_queue(GrowArgs a)
{
    extern __shared__ double lds[];
    grow_real_queue_body<G, false>(a, blockIdx.x, gridDim.x, lds, nullptr);
}

// Batched launch: block b serves the ensemble whose block range holds b.
template <int G>
__global__ __launch_bounds__(64) void grow_real_queue_batch(const GrowEntry *tab, const uint64_t *block0, int n,
                                                            uint64_t base)
{
    extern __shared__ double lds[];
    const uint64_t bid = base + blockIdx.x;
    const int e = find_segment(block0, n, bid);
    grow_real_queue_body<G, false>(tab[e].a, (uint32_t)(bid - block0[e]), (uint32_t)tab[e].H, lds, nullptr);
}

// Chains beyond the LDS limit: block s grows its chains in HBM plane region s.
__global__ __launch_bounds__(64) void grow_real_hbm(GrowArgs a)
{
    __shared__ double ring[3 * kRing];
    grow_real_queue_body<64, true>(a, blockIdx.x, gridDim.x, a.bead_slots + (size_t)blockIdx.x * 3 * a.n_monomers,
                                   ring);
}

// Largest bead count with the beads in LDS, beyond which they lie in HBM planes
// in the workspace (8 waves per CU, the latest 256 beads in LDS, the rest from
// L2).  LDS would hold N = 6826, but leaves fewer waves: MI355X, k = 8, LDS /
// HBM: N = 1024, 2 10^4 chains, 5.8 / 5.5 ms; N = 1536, 10^4, 5.0 / 4.1.  The
// line stays at 1536 all the same, since below it a call needs no bead planes in
// its workspace (72 MiB there).
constexpr int kRealLdsMax = 1536;
int real_max_monomers() { return 16384; }

// Resident blocks (and HBM plane regions) of the HBM kernel for M chains.
uint32_t real_hbm_slots(int n_monomers, uint64_t n_chains)
{
    if (n_monomers <= kRealLdsMax) return 0;
    return (uint32_t)(n_chains < 2048 ? n_chains : 2048);
}

// Queued kernel with G lanes per chain, beads in LDS.
static hipError_t queue_shape(int N, int G, GrowVariant *v)
{
    v->family = 5;
    v->p0 = G;
    v->p1 = 0;
    v->p2 = 0;
    v->threads = 64;
    v->cpb = 64 / G;
    v->shmem = (size_t)(64 / G) * queue_stride(N, G) * sizeof(double);
    if (v->shmem > 163840) return hipErrorInvalidValue;
    v->H = 0;
    v->S = 0;
    // blocks that fill the GPU: LDS, and 4 waves per SIMD (128 VGPRs)
    const uint32_t per_cu = (uint32_t)(163840 / v->shmem);
    v->max_blocks = 256u * (per_cu < 16u ? per_cu : 16u);
    return hipSuccess;
}

// Shape of the LDS kernel for N beads, G lanes per chain (8..64, G >= k: one
// trial per lane) and `threads` per block (64 or 256; G = 64 only in
// one-wave blocks).  hipErrorInvalidValue when the combination is not legal
// or the block's planes and logarithm table exceed the CU's 160 KiB.
static hipError_t real_shape(int N, int k, int G, int threads, GrowVariant *v)
{
    if (G != 8 && G != 16 && G != 32 && G != 64) return hipErrorInvalidValue;
    if (G < k) return hipErrorInvalidValue;
    if (threads != 64 && (threads != 256 || G == 64)) return hipErrorInvalidValue;
    const size_t planes = (size_t)3 * N * plane_row(threads / G, G) * sizeof(double);
    if (planes > 163840) return hipErrorInvalidValue;
    v->family = 2;
    v->p0 = G;
    v->p1 = 0;
    v->p2 = 0;
    v->threads = threads;
    v->cpb = threads / G;
    v->shmem = planes;
    v->H = 0;
    v->S = 0;
    return hipSuccess;
}

// Lanes of the queued kernel for chains of N beads and k trials, 0 where the
// lockstep kernel serves every call.  Kernel time, lockstep / queued (16, 32, 64
// lanes), MI355X, b = sigma = 1, 10^5 chains and more (fewer where N is large):
//   k = 4:  N = 64 1.35 / 1.50 1.98 3.34 ms; N = 100 1.52 / 1.15 1.32 2.06;
//           N = 160 3.77 / 1.67 1.57 2.25; N = 400 2.76 / 2.07 1.48 1.46
//   k = 8:  N = 128 2.73 / 3.02 3.28 4.69; N = 144 3.77 / 3.68 3.68 5.19;
//           N = 256 8.62 / 10.1 6.97 7.93; N = 300 7.15 / 7.51 4.88 4.58;
//           N = 1000 4.51 / - 7.17 3.40
//   k = 16: N = 300 2.94 / 4.68 3.28 2.93; N = 400 4.01 / 8.23 5.10 3.80
//   k = 32: N = 256 1.27 / - 1.71 1.64; N = 500 2.41 / - 3.25 1.97
//   k = 64: N = 256 0.98 / - - 1.13; N = 1000 2.49 / - - 2.37
static int queue_lanes(int N, int k)
{
    if (k <= 4) return N < 80 ? 0 : (N < 140 ? 16 : (N < 400 ? 32 : 64));
    if (k <= 8) return N < 144 ? 0 : (N < 280 ? 32 : 64);
    return N < (k <= 16 ? 400 : (k <= 32 ? 500 : 1000)) ? 0 : 64;
}

// Whether the queued kernel (G lanes) is the faster one for `chains` such
// chains that share the GPU.  How soon chains end goes with e = k b / sigma, the
// trials per bead diameter: k = 8, sigma = b ends like k = 4, sigma = b / 2.
//  - Chains that all fit at up to two waves per SIMD (three with one chain per
//    wave): the queued step has the shorter serial path, and ends no later.
//    Queued / lockstep time, 1000 and 4000 chains: N = 100, k = 4 0.77, 0.82;
//    N = 213, k = 6 0.78, 0.91; N = 256, k = 8 0.98, 1.01; N = 400, k = 8 (1000
//    and 3000) 0.69, 0.87.
//  - More chains than that: the queue wins by the steps that dead ends leave
//    idle in lockstep, more with shorter-lived and longer chains, against a
//    step that costs more.  `most` is the e up to which it won, by N and the
//    number of chains.  64,000 chains: N = 100, e = 3.3 0.63, e = 6.7 1.15; N =
//    180, e = 6.7 0.80, e = 10 1.03; N = 280, k = 8, e = 6.7 0.77, e = 20 1.22.
//    8000 chains: N = 213, e = 4 0.85, e = 8 1.10; N = 340, e = 8 0.80, e = 20 0.97.
//  - Beyond N = 256 the lockstep kernel's waves leave the step loop with their
//    last chain: where all end within a few beads it wins (N = 340, e = 1.3,
//    16,000 chains, 1.6; N = 500, e = 2, 1.5).
//  - N >= 500: 0.7 to 0.95 otherwise, but 1.05 where few chains live long
//    (N = 500, k = 8, sigma = 0.4, 1000 chains).
// Over 11,000 calls with k = 1..64, N = 80..1536, sigma / b = 0..1.2 and 1000 to
// 256,000 chains this is 0.6 % behind the faster of the two, the queue for every
// call 3.4 %, lockstep for every call 33 %.
static bool queue_serves(int N, int k, double e, uint64_t chains, int G)
{
    const bool few = chains <= (G == 64 ? 3072u : 2048u * (64u / (unsigned)G));
    if (k > 8) {
        if (N < 500) return k <= 12 || chains >= 6000;
        return !(N < 700 && few && e > 1.5 * k);
    }
    if (N >= 500) return e >= 3.0 && !(N < 700 && few && e > 1.5 * k);
    if (N >= 400 && e < 2.1) return false;
    if (few) return true;
    if (N > 256 && e < 2.0) return false;
    const uint64_t M = chains;
    double most = 1e300;
    if (N < 115) most = M < 24000 ? 3.0 : 4.5;
    else if (N < 140) most = 5.2;
    else if (N < 200) most = M < 12000 ? 4.2 : (M < 64000 ? 6.7 : 8.9);
    else if (N < 250) most = M < 12000 ? 4.6 : (M < 64000 ? 7.5 : 10.0);
    else if (N < 340) most = M < 8000 ? 4.5 : (M < 24000 ? 7.4 : (M < 64000 ? 8.9 : 9.3));
    else if (M < 6000) most = 7.0;
    return e <= most;
}

// Built-in rule.  Lanes per chain: at least the next power of two >= k (one
// trial per lane), and enough that the chains whose planes fit in a CU's LDS
// still fill about 8 waves (G >= 0.075 N); the extra lanes share the culling
// pass.  256-thread blocks when the bead planes fit in half a CU's LDS, else
// one wave per block (up to the whole 160 KiB).  G = 64 always runs one-wave
// blocks: four one-chain waves sharing a block's padded planes were measured
// 1.2-2.3x slower for 432 <= N <= 672 (k = 8) than four one-wave blocks.  A
// legal mapping of the tuning table replaces the rule.
hipError_t real_variant(const GrowArgs &a, GrowVariant *v, bool scan)
{
    const int N = a.n_monomers;
    if (N > kRealLdsMax) {
        // HBM planes, launched on its own (p1 = 1)
        v->family = 2;
        v->p0 = 64;
        v->p1 = 1;
        v->p2 = 0;
        v->threads = 64;
        v->cpb = 1;
        v->shmem = 0;
        v->H = 0;
        v->S = 0;
        return hipSuccess;
    }
    int tl = 0, tt = 0;
    if (tuned_mapping(1 /* hard spheres */, N, a.k_trials, &tl, &tt) &&
        real_shape(N, a.k_trials, tl, tt, v) == hipSuccess)
        return hipSuccess;
    if (!scan) {
        const int G = queue_lanes(N, a.k_trials);
        const double e = a.sigma2 > 0.0 ? a.k_trials * (a.bond_length / sqrt(a.sigma2)) : 1e300;
        if (G && queue_serves(N, a.k_trials, e, a.n_chains, G) && queue_shape(N, G, v) == hipSuccess)
            return hipSuccess;
    }
    int need = a.k_trials;
    const int occ = (3 * N + 39) / 40; // ceil(0.075 N)
    if (occ > need) need = occ;
    const int G = need <= 8 ? 8 : (need <= 16 ? 16 : (need <= 32 ? 32 : 64));
    // k = 8 or 16 with 2k lanes in 256-thread blocks whose planes leave
    // fewer than 3 blocks per CU: 4k lanes in one-wave blocks are faster
    // (the extra lanes also carry the round-1 Marsaglia attempts); measured
    // on MI355X: k = 8, 144 <= N <= 208, 1.18-1.22x; k = 16, 320 <= N <= 416,
    // 1.13-1.20x.
    const int k = a.k_trials;
    GrowVariant wide, at256;
    if ((k == 8 || k == 16) && G == 2 * k && real_shape(N, k, G, 256, &at256) == hipSuccess &&
        at256.shmem > 163840 / 3 && real_shape(N, k, 4 * k, 64, &wide) == hipSuccess) {
        *v = wide;
        return hipSuccess;
    }
    GrowVariant half_cu;
    if (G != 64 && real_shape(N, a.k_trials, G, 256, &half_cu) == hipSuccess && half_cu.shmem <= 81920) {
        *v = half_cu;
        return hipSuccess;
    }
    return real_shape(N, a.k_trials, G, 64, v);
}

template <int G>
static hipError_t launch_g(const GrowArgs &a, const GrowVariant &v, const GrowEntry *tab,
                           const uint64_t *block0, int n, uint64_t blocks, size_t shmem, hipStream_t s)
{
    const void *fn = tab ? (const void *)grow_real_tp_batch<G> : (const void *)grow_real_tp<G>;
    if (shmem > 65536) {
        hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shmem);
        if (e != hipSuccess) return e;
    }
    return launch_sliced(blocks, v.threads, [&](uint64_t b0, uint32_t nb) {
        if (tab)
            hipLaunchKernelGGL((grow_real_tp_batch<G>), dim3(nb), dim3(v.threads), shmem, s, tab, block0, n, b0);
        else
            hipLaunchKernelGGL((grow_real_tp<G>), dim3(nb), dim3(v.threads), shmem, s, a, b0);
    });
}

static hipError_t dispatch_real(const GrowArgs &a, const GrowVariant &v, const GrowEntry *tab,
                                const uint64_t *block0, int n, uint64_t blocks, size_t shmem, hipStream_t s)
{
    switch (v.p0) {
    case 8: return launch_g<8>(a, v, tab, block0, n, blocks, shmem, s);
    case 16: return launch_g<16>(a, v, tab, block0, n, blocks, shmem, s);
    case 32: return launch_g<32>(a, v, tab, block0, n, blocks, shmem, s);
    default: return launch_g<64>(a, v, tab, block0, n, blocks, shmem, s);
    }
}

template <int G>
static hipError_t launch_queue(const GrowArgs &a, const GrowEntry *tab, const uint64_t *block0, int n,
                               uint64_t blocks, size_t shmem, hipStream_t s)
{
    const void *fn = tab ? (const void *)grow_real_queue_batch<G> : (const void *)grow_real_queue<G>;
    if (shmem > 65536) {
        hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shmem);
        if (e != hipSuccess) return e;
    }
    return launch_sliced(blocks, 64, [&](uint64_t b0, uint32_t nb) {
        if (tab)
            hipLaunchKernelGGL((grow_real_queue_batch<G>), dim3(nb), dim3(64), shmem, s, tab, block0, n, b0);
        else
            hipLaunchKernelGGL((grow_real_queue<G>), dim3(nb), dim3(64), shmem, s, a);
    });
}

static hipError_t dispatch_queue(const GrowArgs &a, const GrowVariant &v, const GrowEntry *tab,
                                 const uint64_t *block0, int n, uint64_t blocks, size_t shmem, hipStream_t s)
{
    switch (v.p0) {
    case 16: return launch_queue<16>(a, tab, block0, n, blocks, shmem, s);
    case 32: return launch_queue<32>(a, tab, block0, n, blocks, shmem, s);
    default: return launch_queue<64>(a, tab, block0, n, blocks, shmem, s);
    }
}

hipError_t launch_grow_real(const GrowArgs &a, hipStream_t s)
{
    GrowVariant v;
    hipError_t e = real_variant(a, &v, false);
    if (e != hipSuccess) return e;
    if (v.family == 5)
        return dispatch_queue(a, v, nullptr, nullptr, 0, variant_blocks(v, a.n_chains), v.shmem, s);
    if (v.p1) {
        if (!a.bead_slots || a.n_slots == 0) return hipErrorInvalidValue;
        hipLaunchKernelGGL(grow_real_hbm, dim3(a.n_slots), dim3(64), 0, s, a);
        return hipGetLastError();
    }
    const uint64_t blocks = (a.n_chains + v.cpb - 1) / v.cpb;
    return dispatch_real(a, v, nullptr, nullptr, 0, blocks, v.shmem, s);
}

hipError_t launch_real_queue_batch(const GrowVariant &v, const GrowEntry *tab, const uint64_t *block0, int n,
                                   uint64_t blocks, size_t shmem, hipStream_t s)
{
    return dispatch_queue(GrowArgs{}, v, tab, block0, n, blocks, shmem, s);
}

hipError_t launch_real_batch(const GrowVariant &v, const GrowEntry *tab, const uint64_t *block0, int n,
                             uint64_t blocks, size_t shmem, hipStream_t s)
{
    return dispatch_real(GrowArgs{}, v, tab, block0, n, blocks, shmem, s);
}

} // namespace rsaw
