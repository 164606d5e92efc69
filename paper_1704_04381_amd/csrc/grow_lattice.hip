// Lattice chain growth on the simple cubic lattice (Sec. 3.3.2, Algorithm 1;
// weight of Eq. 3), one chain per lane, chain state in VGPRs: one history
// word per monomer (lattice_common.hpp), fully unrolled over NMAX.
// Coordinates of an N <= 64 chain stay in [-63, 63], so the coordinate bytes
// never wrap and never become zero.
//
// Step i (tip t = monomer i-1) tests the earlier monomers of the parity that
// can touch the tip, j = i-4, i-6, ..., two operations each; j = i-2 is the
// tip's bonded neighbour, so its direction bit is taken untested.  The free
// mask and the picked rank address one LDS table entry: the move and the
// increment of the counts n_m.  An empty mask (a dead end) has a zero entry,
// so a dead chain needs no selects: its mask is kept empty by `alive`.
//
// log W = sum over m of n_m log m (Eq. 3 grouped by value): the counts are
// 6-bit fields of one register, m = 2..5 at 0, 6, 12, 18, m = 1 at 26, and
// the one m = 6 (step 1) at bit 24; the sum is formed once after the last
// step, and the fields add up to the number of monomers placed.  Coordinate
// sums run along with the steps (of a dead chain too: its repeated last
// monomer is taken out at the end).
//
// Bound by VALU issue: 4,264 instructions per wave and N = 64 chain, where the
// four-operation test with its per-step selects took 6,888.  MI355X, N = 64,
// 10^7 chains, growth kernel: 1.83 -> 1.03 ms (with the max-log-W atomics out
// of the way).  At least 4 waves per SIMD (128 VGPRs, against the 141 the
// compiler takes by itself): 1.03 against 1.06 ms.
#include "lattice_common.hpp"

#include <type_traits>

namespace rsaw {

// Compile-time loop: f(integral_constant<int, I>) for I = B .. E-1, so that
// every index into the register-resident chain is a constant.
template <int B, int E, typename F>
__device__ __forceinline__ void static_for(F &&f)
{
    if constexpr (B < E) {
        f(std::integral_constant<int, B>{});
        static_for<B + 1, E>(f);
    }
}

template <int NMAX, bool EXACT, typename CT>
__device__ __forceinline__ void grow_lattice_reg_body(const GrowArgs &a, uint64_t bid)
{
    __shared__ uint2 lut[kByteLutSize]; // move, increment of the n_m fields
    __shared__ double logm[8];
    for (uint32_t t = threadIdx.x; t < kByteLutSize; t += blockDim.x) {
        const uint32_t m = __builtin_popcount((t >> 2) & kByteDirs);
        lut[t] = make_uint2(byte_move(t), m ? 1u << ((6u * m + 20u) & 31u) : 0u);
    }
    if (threadIdx.x < 8) logm[threadIdx.x] = a.logm[threadIdx.x];
    __syncthreads();

    const uint64_t c = bid * blockDim.x + threadIdx.x;
    const bool valid = c < a.n_chains;
    const uint64_t g = a.chain_offset + c;
    const int N = a.n_monomers;

    uint32_t pos[NMAX]; // history words
    static_for<0, NMAX>([&](auto J) { pos[J.value] = 0u; });
    pos[0] = byte_history(kByteOrigin);
    uint64_t wx = 1;
    bool rng_fail = false;
    Philox4 blk{0, 0, 0, 0};
    // outputs of the attempt that ends the chain: the first complete one, or
    // the last allowed one (one attempt without restarts)
    double res_lw = -__builtin_huge_val();
    uint64_t res_wx = 0;
    int64_t res_nn = 0;
    int32_t res_ex = 0, res_ey = 0, res_ez = 0;
    int res_grown = 1;
    bool res_alive = false;
    bool pending = valid;

    for (uint32_t rd = 0; rd < a.max_rounds; ++rd) {
        uint32_t tip = kByteOrigin;
        uint32_t alive = pending ? ~0u : 0u;
        uint32_t cnt = 0;
        // biased coordinate sums over the monomers (x and z as 16-bit halves)
        uint32_t sxz = 0x00800080u, sy = 0x00008000u, s2 = 3u * 128u * 128u;
        if (EXACT) wx = 1;
        const uint32_t hi = rd << 16; // attempt in the high half of the step word

        static_for<1, NMAX>([&](auto I) {
            constexpr int i = I.value;
            if (i >= N) return;
            // directions of the occupied neighbours; two accumulators halve
            // the dependency chain
            const uint32_t tref = tip & kByteCoords;
            uint32_t acc = 0, acc2 = 0;
            if constexpr (i >= 2) acc = pos[i - 2];
            static_for<0, (i >= 4 ? i / 2 - 1 : 0)>([&](auto Q) {
                constexpr int j = i - 4 - 2 * Q.value;
                if constexpr (Q.value & 1) acc = byte_pair(acc, pos[j], tref);
                else acc2 = byte_pair(acc2, pos[j], tref);
            });
            const uint32_t freem = byte_free(acc | acc2, tip, alive);
            const uint32_t m = __builtin_popcount(freem);

            // 16-bit selection word: half i mod 8 of one Philox block per 8 steps
            if constexpr (i == 1 || (i & 7) == 0)
                blk = draw(a.seed, g, (uint32_t)(i >> 3) | hi, kSlotSelect, 0);
            constexpr int h = i & 7;
            const uint32_t wd = (h >> 1) == 0 ? blk.x0 : ((h >> 1) == 1 ? blk.x1 : ((h >> 1) == 2 ? blk.x2 : blk.x3));
            const uint32_t x = (h & 1) ? (wd >> 16) : (wd & 0xFFFFu);
            const uint32_t p = x * m;
            uint32_t r = p >> 16;
            if (__builtin_expect((p & 0xFFFFu) < m, 0)) { // never for m = 0
                r = lemire_redraw16(a.seed, g, (uint32_t)i | hi, m, x);
                if (r == kPickFailed) {
                    rng_fail = true;
                    r = 0;
                }
            }
            const uint2 mv = lut[(freem << 2) | r]; // r < m <= 6, or 0
            tip += mv.x;
            cnt += mv.y;
            alive = m != 0 ? ~0u : 0u;
            if (EXACT) wx = wx * (uint64_t)m;
            const uint32_t co = tip & kByteCoords;
            sxz += co & 0x00FF00FFu;
            sy += co & 0x0000FF00u;
            s2 = __builtin_amdgcn_udot4(co, co, s2, false);
            if constexpr (i + 2 < NMAX) pos[i] = byte_history(tip);
        });
        const bool done = alive != 0u;
        const bool ends = pending && (done || rd + 1 >= a.max_rounds);
        if (ends) {
            const uint32_t n2 = cnt & 63u, n3 = (cnt >> 6) & 63u, n4 = (cnt >> 12) & 63u, n5 = (cnt >> 18) & 63u;
            const int grown = 1 + (int)(n2 + n3 + n4 + n5 + (cnt >> 26) + ((cnt >> 24) & 1u));
            // log W = sum over m = 1..6, ascending, of n_m log m (one rounding
            // each); n_1 log 1 = 0 and m_1 = 6 always
            double lw = 0.0;
            if (N >= 2) {
                lw = lw + (double)n2 * logm[2];
                lw = lw + (double)n3 * logm[3];
                lw = lw + (double)n4 * logm[4];
                lw = lw + (double)n5 * logm[5];
                lw = lw + logm[6];
            }
            res_ex = (int32_t)(tip & 0xFFu) - 128;
            res_ey = (int32_t)((tip >> 8) & 0xFFu) - 128;
            res_ez = (int32_t)((tip >> 16) & 0xFFu) - 128;
            // observables over the placed monomers: N terms were added, the
            // last N - grown of them the tip again
            const int32_t gg = grown, dup = N - grown;
            const int32_t Sx = (int32_t)(sxz & 0xFFFFu) - 128 * N - dup * res_ex;
            const int32_t Sy = (int32_t)(sy >> 8) - 128 * N - dup * res_ey;
            const int32_t Sz = (int32_t)(sxz >> 16) - 128 * N - dup * res_ez;
            const int32_t B = (int32_t)((sxz & 0xFFFFu) + (sy >> 8) + (sxz >> 16));
            const int32_t S2 = (int32_t)s2 - 256 * B + 3 * 16384 * N -
                               dup * (res_ex * res_ex + res_ey * res_ey + res_ez * res_ez);
            res_nn = (int64_t)gg * S2 - ((int64_t)Sx * Sx + (int64_t)Sy * Sy + (int64_t)Sz * Sz);
            res_lw = done ? lw : -__builtin_huge_val();
            res_wx = done ? wx : 0ull;
            res_grown = grown;
            res_alive = done;
            pending = false;
        }
        if (__ballot(pending) == 0) break;
    }

    if (valid) {
        if (a.log_w) a.log_w[c] = res_lw;
        if (EXACT && a.w_exact) a.w_exact[c] = res_wx;
        if (a.r_end) {
            CT *re = (CT *)a.r_end;
            re[c] = (CT)res_ex;
            re[a.n_chains + c] = (CT)res_ey;
            re[2 * a.n_chains + c] = (CT)res_ez;
        }
        if (a.r2) a.r2[c] = (double)(res_ex * res_ex + res_ey * res_ey + res_ez * res_ez);
        if (a.n2rg2) a.n2rg2[c] = res_nn;
        if (a.rg2) a.rg2[c] = (double)res_nn / ((double)res_grown * (double)res_grown);
        if (a.n_grown) a.n_grown[c] = (uint16_t)res_grown;
    }
    if (rng_fail) atomicExch(a.status, 6);
    const uint64_t bits = res_alive ? (uint64_t)__double_as_longlong(res_lw) : 0ull;
    publish_log_w_max_block(a, bits);
}

template <int NMAX, bool EXACT, typename CT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 8))) void
grow_lattice_reg(GrowArgs a, uint64_t base)
{
    grow_lattice_reg_body<NMAX, EXACT, CT>(a, base + blockIdx.x);
}

// Batched launch: block b serves the ensemble whose block range holds b.
template <int NMAX, bool EXACT, typename CT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 8))) void
grow_lattice_reg_batch(const GrowEntry *tab, const uint64_t *block0, int n,
                                                              uint64_t base)
{
    const uint64_t bid = base + blockIdx.x;
    const int e = find_segment(block0, n, bid);
    grow_lattice_reg_body<NMAX, EXACT, CT>(tab[e].a, bid - block0[e]);
}

template <int NMAX, bool EXACT, typename CT>
static hipError_t launch(const GrowArgs &a, hipStream_t s)
{
    const uint64_t blocks = (a.n_chains + 255) / 256;
    return launch_sliced(blocks, 256, [&](uint64_t b0, uint32_t nb) {
        hipLaunchKernelGGL((grow_lattice_reg<NMAX, EXACT, CT>), dim3(nb), dim3(256), 0, s, a, b0);
    });
}

// Dispatch on the N bucket, exact-weight flag and output coordinate type.
hipError_t launch_grow_lattice_lds(const GrowArgs &a, bool i16, hipStream_t s);

hipError_t launch_grow_lattice(const GrowArgs &a, bool exact, bool i16, hipStream_t s)
{
    const int N = a.n_monomers;
    if (!exact && N > 64) return launch_grow_lattice_lds(a, i16, s);
    if (exact) {
        // RSAW_EXACT_W is limited to N <= 28 by the caller
        if (N <= 16) return i16 ? launch<16, true, int16_t>(a, s) : launch<16, true, int32_t>(a, s);
        return i16 ? launch<32, true, int16_t>(a, s) : launch<32, true, int32_t>(a, s);
    }
    if (N <= 16) return i16 ? launch<16, false, int16_t>(a, s) : launch<16, false, int32_t>(a, s);
    if (N <= 32) return i16 ? launch<32, false, int16_t>(a, s) : launch<32, false, int32_t>(a, s);
    return i16 ? launch<64, false, int16_t>(a, s) : launch<64, false, int32_t>(a, s);
}

// Variant of the register kernel for one ensemble (N <= 64, or exact weights).
void lattice_reg_variant(const GrowArgs &a, bool exact, bool i16, GrowVariant *v)
{
    const int N = a.n_monomers;
    v->family = 0;
    v->p0 = exact ? (N <= 16 ? 16 : 32) : (N <= 16 ? 16 : (N <= 32 ? 32 : 64));
    v->p1 = exact ? 1 : 0;
    v->p2 = i16 ? 1 : 0;
    v->threads = 256;
    v->cpb = 256;
    v->shmem = 0;
    v->H = 0;
    v->S = 0;
}

template <int NMAX, bool EXACT, typename CT>
static hipError_t launch_batch(const GrowEntry *tab, const uint64_t *block0, int n, uint64_t blocks,
                               hipStream_t s)
{
    return launch_sliced(blocks, 256, [&](uint64_t b0, uint32_t nb) {
        hipLaunchKernelGGL((grow_lattice_reg_batch<NMAX, EXACT, CT>), dim3(nb), dim3(256), 0, s, tab, block0, n,
                           b0);
    });
}

hipError_t launch_lattice_reg_batch(const GrowVariant &v, const GrowEntry *tab, const uint64_t *block0,
                                    int n, uint64_t blocks, hipStream_t s)
{
    const bool i16 = v.p2 != 0;
    if (v.p1) {
        if (v.p0 == 16) return i16 ? launch_batch<16, true, int16_t>(tab, block0, n, blocks, s)
                                   : launch_batch<16, true, int32_t>(tab, block0, n, blocks, s);
        return i16 ? launch_batch<32, true, int16_t>(tab, block0, n, blocks, s)
                   : launch_batch<32, true, int32_t>(tab, block0, n, blocks, s);
    }
    if (v.p0 == 16) return i16 ? launch_batch<16, false, int16_t>(tab, block0, n, blocks, s)
                               : launch_batch<16, false, int32_t>(tab, block0, n, blocks, s);
    if (v.p0 == 32) return i16 ? launch_batch<32, false, int16_t>(tab, block0, n, blocks, s)
                               : launch_batch<32, false, int32_t>(tab, block0, n, blocks, s);
    return i16 ? launch_batch<64, false, int16_t>(tab, block0, n, blocks, s)
               : launch_batch<64, false, int32_t>(tab, block0, n, blocks, s);
}

} // namespace rsaw
