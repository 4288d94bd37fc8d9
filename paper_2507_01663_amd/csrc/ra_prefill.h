// gfx950 kernel of the prompt prefill: causal attention of packed prompts over themselves, and the write of
// their K and V rows into the pages of the cache that the decode steps then read (once per prompt group when
// several responses are sampled for one prompt: paper Sec. 7.1).
//
// Unlike the decode step this is a dense contraction, bound by the matrix cores.  A workgroup of eight waves
// (two per SIMD, so that one wave's vector work runs while the other's MFMAs do) takes eight (32-row tile, head) units
// of one (prompt, kv head), one per wave.  K and V stream through an LDS ring in chunks of two stages of 32
// keys (K0 K1 V0 V1 | K2 K3 V2 V3) by direct global->LDS loads; every wave
// multiplies every stage with its own query rows, held in registers:
//   S^T[key, row] = K . Q^T,   O^T[d, row] += V^T . P^T     (32x32x16 MFMA, fp32 accumulation)
// with the softmax running per query row in fp32 (base 2).  The tile layout in LDS is the decode kernel's.
// Calls of few blocks take workgroups of four waves and four units (a chunk is one stage; two or three to a compute unit), or
// of eight waves, two to a unit: one takes the even stages, the other the odd ones (prefill_shape says which calls).
#pragma once
#include "ra_device.h"

namespace ra {

constexpr int kPfWaves = 8;                  // waves of a workgroup that stays, two per SIMD
constexpr int kPfRows = 32;                  // query rows per wave: one 32x32 MFMA tile
constexpr int kPfBlock = kPfRows * kPfWaves; // rows a bound on the prompt length is rounded up to
constexpr int kPfSlots = 4;                  // ring slots of one chunk each

constexpr int kPfStageRow = 128;                    // bytes of a row in a wave's staging area: 64 bf16
constexpr int kPfStageBytes = kPfRows * kPfStageRow; // 4 KB per wave

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

// Per-lane constants of the 32x32x16 products.  A lane is (n = lane % 32, hh = lane / 32).  With the tile layout
// of lane_setup() (rows of D bf16, 16-byte units XOR-swizzled inside the row) every LDS address the step needs is
// one of two per-lane bases XOR a compile-time constant, as long as stages start at multiples of their size:
//   K operand of k-step i (key n, d = 16 i + 8 hh .. + 7):          stage + (k_base ^ 32 i)
//   V operand, d-tile dt, keys 4 hh + 8 rd .. + 3 of tile V0 / V1:  stage + 2 tiles (+ 1) + (v_base ^ 64 dt ^ kVrd rd)
// the latter through the transposing read, whose 16 lanes address a 4-key x 16-d block, lane a supplying key a / 4,
// d = 4 (a % 4) .. + 3.
template <int D> struct PfLane {
    int k_base, v_base;
};

template <int D> __device__ __forceinline__ void pf_lane_setup(PfLane<D> &pl, int lane)
{
    using G = Geo<D, 2>;
    constexpr int UM = G::kUnits - 1;
    const int n = lane & 31, hh = lane >> 5;
    const int r = n & 15;
    // unit (2 i + hh) ^ swz(r) = 2 i ^ (swz(r) ^ hh)
    pl.k_base = (n >> 4) * G::kTile + G::kRowBytes * r + 16 * ((swz(r) & UM) ^ hh);
    const int a = lane & 15, dh = (lane >> 4) & 1;
    const int vrow = 4 * hh + (a >> 2);           // + 8 rd
    const int c = 2 * dh + ((a >> 1) & 1);        // + 4 dt
    pl.v_base = G::kRowBytes * vrow + 16 * (c ^ (swz(vrow) & UM)) + 8 * (a & 1);
}
template <int D> __device__ __forceinline__ constexpr int pf_v_xor(int dt, int rd)
{
    // eight rows further on; with sixteen units per row the swizzle of those rows differs in its top bit
    return (64 * dt) ^ ((8 * Geo<D, 2>::kRowBytes + (Geo<D, 2>::kUnits == 16 ? 128 : 0)) * rd);
}

template <int D> struct PfState {
    bf16x8 qf[D / 16]; // Q^T operand of k-step i: row n, d = 16 i + 8 hh .. + 7
    f32x16 o[D / 32];  // O^T accumulators: element e of d-tile dt is d = 32 dt + 8 (e / 4) + 4 hh + e % 4, row n
    f32x16 s;          // scores of the stage whose weights are computed next: element e is key 8 (e / 4) + 4 hh + e % 4
    float m, lsum;     // reference point of the exponent (same in both lanes of a row); this lane's part of the row sum
};

// The 16-byte pieces of a staging row are XOR-swizzled by the row, so that neither the lanes of a row group that write
// the same piece of different rows nor the eight lanes that read one row meet in a bank.
__device__ __forceinline__ int pf_stage_swz(int r) { return (r + (r >> 3)) & 7; }

// The first step of a maximum over fresh MFMA results, by an instruction the compiler knows; once it has run, the
// whole accumulator (one MFMA writes all of it) is safe to read.
__device__ __forceinline__ float first_max(float a, float b) { return fmaxf(a, b); }

constexpr float kPfSlack = 8.0f;
// Least reference point of an exponent: keys that score -inf weigh nothing also while a row (or a wave's part of its keys) has
// had no others, and a row without any other has lse -inf, whatever the launch shape.
constexpr float kPfLowest = -__FLT_MAX__;

// One step of a wave's software pipeline (see the kernel): weights of stage s and scores of stage s + 1 (NEXT; MASK:
// that stage is the wave's diagonal one), then O += P V of stage s and the row maxima of the new scores.
//
// The LDS addresses: stages start at multiples of their size, so each is a stage's base plus a lane constant with a constant
// XORed in, made from that sum (opaque, or the compiler holds every lane constant in a register of its own and adds to each).
// V's serve two steps: SECOND > 0 is the step after one whose V lies that many stages before this one's, and takes va as that
// step left it.
// The vector instructions of a step, not its MFMAs, are what it can save: offsets in place of adds for V's second tiles 1244 ->
// 1226 us (16 prompts of 2048, 64 heads on eight, e4m3), the shared addresses and two additions of zero less 1236 -> 1224.
template <int D, bool MASK, bool NEXT, int SECOND = 0>
__device__ __forceinline__ void pf_step(PfState<D> &st, uint32_t k_next, uint32_t v_addr, uint32_t (&va)[D / 32][2], const PfLane<D> &pl,
                                        float scale_log2, int key_next, int row)
{
    using G = Geo<D, 2>;
    typedef s16x4 __attribute__((address_space(3))) * lds_s16x4;
    typedef bf16x8 __attribute__((address_space(3))) * lds_bf16x8;
    typedef short s16x8 __attribute__((ext_vector_type(8)));
    const int hh = (threadIdx.x & 63) >> 5;
    constexpr int KS = D / 16, DT = D / 32;
#define PF_FENCE() __builtin_amdgcn_sched_barrier(0)
    PF_FENCE();
    // K operands are read four products ahead of their use
    constexpr int KA = KS < 4 ? KS : 4;
    bf16x8 kf[KS];
    uint32_t ka = k_next + (uint32_t)pl.k_base;
    asm volatile("" : "+v"(ka));
    if (NEXT) {
#pragma unroll
        for (int i = 0; i < KA; i++) kf[i] = *(lds_bf16x8)(ka ^ (uint32_t)(32 * i));
    }
    if (!SECOND) {
        uint32_t vb = v_addr + (uint32_t)pl.v_base;
        asm volatile("" : "+v"(vb));
#pragma unroll
        for (int dt = 0; dt < DT; dt++) va[dt][0] = vb ^ (uint32_t)pf_v_xor<D>(dt, 0), va[dt][1] = vb ^ (uint32_t)pf_v_xor<D>(dt, 1);
    }
    s16x4 vr[DT][2][2];
    auto v_read = [&](int dt, int kk) {
        // (the second tile as an offset of the pointer, which the instruction takes; added to the address it would be an add each)
#pragma unroll
        for (int rd = 0; rd < 2; rd++)
            vr[dt][kk][rd] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)va[dt][rd] + (kk * G::kTile + SECOND * G::kStage) / 8);
    };
    PF_FENCE();
    // weights: item k < 16: element k (exponential, running sum, and with every second one the rounding of a pair to
    // bf16); item 16: the row sum
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    u32x4 pw[2];
    float pprev = 0.f, acc0 = 0.f, acc1 = 0.f;
    auto w_item = [&](int k) {
        if (k < 16) {
            const float pk = __builtin_amdgcn_exp2f(__builtin_fmaf(st.s[k], scale_log2, -st.m));
            if (k & 1) {
                acc1 = k == 1 ? pk : acc1 + pk;
                pw[k >> 3][(k >> 1) & 3] = __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2{pprev, pk}), bf16x2));
            } else {
                acc0 = k == 0 ? pk : acc0 + pk;
                pprev = pk;
            }
        } else {
            st.lsum += acc0 + acc1;
        }
    };
    constexpr int NW = 17;
    f32x16 sn;
    if (NEXT) {
        // the first weights cover the latency of the K reads
#pragma unroll
        for (int k = 0; k < 3; k++) w_item(k);
        PF_FENCE();
#pragma unroll
        for (int i = 0; i < KS; i++) {
            if (i == 0) {
#pragma unroll
                for (int e = 0; e < 16; e++) sn[e] = 0.f;
            }
            sn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[i], st.qf[i], sn, 0, 0, 0);
            if (i + KA < KS) kf[i + KA] = *(lds_bf16x8)(ka ^ (uint32_t)(32 * (i + KA)));
#pragma unroll
            for (int w = 3 + i * (NW - 3) / KS; w < 3 + (i + 1) * (NW - 3) / KS; w++) w_item(w);
            if (i >= KS - DT) v_read((i - (KS - DT)) / 2, (i - (KS - DT)) % 2);
            PF_FENCE();
        }
    } else {
#pragma unroll
        for (int n = 0; n < DT; n++) v_read(n / 2, n % 2);
#pragma unroll
        for (int w = 0; w < NW; w++) w_item(w);
        PF_FENCE();
    }
    // O^T += V^T P^T; in the MFMAs' shadow the mask and the maxima of the new scores.
    // item k: 0..3 the causal mask (MASK), 4..11 partial maxima, 12 the exchange, 13 the end
    float mx = 0.f, mn = 0.f;
    bool grew = false;
    auto m_item = [&](int k) {
        if (k < 4) {
            if (MASK) {
                // element e = 4 k + x is key 8 k + 4 hh + x of the stage
                const int kk = key_next + 8 * k + 4 * hh;
#pragma unroll
                for (int x = 0; x < 4; x++) {
                    if (kk + x > row) sn[4 * k + x] = -INFINITY;
                }
            }
        } else if (k == 4) {
            mx = max3(first_max(sn[0], sn[1]), sn[2], sn[2]);
        } else if (k < 11) {
            mx = max3(mx, sn[2 * k - 7], sn[2 * k - 6]); // k = 5..10: elements 3..14
        } else if (k == 11) {
            mx = max3(mx, sn[15], sn[15]);
        } else if (k == 12) {
            const u32x2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
            mx = max3(__uint_as_float(r[0]), __uint_as_float(r[1]), __uint_as_float(r[1]));
        } else {
            mn = mx * scale_log2; // the scale is positive, so the maximum may be taken before it is applied
            grew = mn > st.m + kPfSlack;
            st.s = sn;
        }
    };
    constexpr int NMI = NEXT ? 14 : 0;
    constexpr int NPV = 2 * DT;
#pragma unroll
    for (int n = 0; n < NPV; n++) {
        const int dt = n / 2, kk = n % 2;
        if (n + DT < NPV) v_read((n + DT) / 2, (n + DT) % 2); // four products ahead of its use
        const bf16x8 vf = __builtin_bit_cast(bf16x8, (s16x8)__builtin_shufflevector(vr[dt][kk][0], vr[dt][kk][1], 0, 1, 2, 3, 4, 5, 6, 7));
        st.o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, __builtin_bit_cast(bf16x8, pw[kk]), st.o[dt], 0, 0, 0);
#pragma unroll
        for (int w = n * NMI / NPV; w < (n + 1) * NMI / NPV; w++) m_item(w);
        PF_FENCE();
    }
    if (NEXT) {
        if (__any(grew)) {
            mn = mn > st.m ? mn : st.m;
            const float alpha = __builtin_amdgcn_exp2f(st.m - mn);
            st.m = mn;
            st.lsum *= alpha;
#pragma unroll
            for (int dt = 0; dt < DT; dt++) st.o[dt] *= alpha;
        }
    }
#undef PF_FENCE
}

// Scores of a stage for the wave's rows (no vector work to overlap with: used once, for the first stage).  All K
// operands are read first and the products go to two accumulators in turn, so that neither the LDS latency nor the
// MFMA latency is paid once per k-step.
template <int D>
__device__ __forceinline__ void pf_scores(uint32_t k_stage, const PfLane<D> &pl, const bf16x8 (&qf)[D / 16], f32x16 &sn)
{
    typedef bf16x8 __attribute__((address_space(3))) * lds_bf16x8;
    uint32_t ka = k_stage + (uint32_t)pl.k_base;
    asm volatile("" : "+v"(ka)); // (see pf_step)
    bf16x8 kf[D / 16];
#pragma unroll
    for (int i = 0; i < D / 16; i++) kf[i] = *(lds_bf16x8)(ka ^ (uint32_t)(32 * i));
    f32x16 s2;
#pragma unroll
    for (int e = 0; e < 16; e++) sn[e] = s2[e] = 0.f;
#pragma unroll
    for (int i = 0; i < D / 16; i += 2) {
        sn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[i], qf[i], sn, 0, 0, 0);
        s2 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[i + 1], qf[i + 1], s2, 0, 0, 0);
    }
    sn += s2;
}

// A unit of work of a wave: one head's 32 query rows of one tile, with the keys 0 .. its last row.  The units of a
// (prompt, kv head) pair are numbered from the last tile down, the G heads of a tile together, and a block is eight (or
// four) consecutive ones: under the causal mask they need the same keys but for a tile or two, so the waves of a workgroup
// have the same work and leave the block together.  (A block of 256 rows of one head streams the keys of its last row
// past all of its waves: 24 stages of 32 keys for the 512 rows of a head of a 512-token prompt, 18 this way, and half
// of the waves idle at the end of it.)
//
// Which workgroup takes which blocks is fixed by the inputs.  Workgroups are dealt to the eight dies round-robin, and
// each die has its own L2, so the blocks of a pair go to few dies: with gg = gcd(Hkv, 8), die x takes the kv heads
// congruent x mod gg, and the 8 / gg dies that take the same heads take the blocks of a pair in turn.  Every die so gets
// the same share of every prompt, however ragged the lengths are.  A die takes the prompts in groups of a.group (see
// launch_prefill), the blocks of a group ordered by length, longest first (block number from the short end of its pair,
// which is its length to within a tile, over all prompts of the group at once), and deals them to its workgroups back and
// forth, which keeps their sums within a few percent of one another.
struct PfBlock {
    int g, kvh, t0, len; // prompt, kv head; first token of the prompt, its tokens
    int u0, nst;        // first unit of the block, stages of 32 keys
    __device__ __forceinline__ int tiles() const { return (len + 31) >> 5; }
};

// A workgroup's way through its die's order of blocks.  Lane l has prompt base + l of the 64 that are in use.
struct PfCursor {
    int base, done, all; // first of those prompts; blocks (of this die) of the prompts before it and of the 64
    int round;           // blocks of this workgroup so far
    int lane0, before, blocks; // the group that the last block came from: its first lane, blocks of the 64 before it, its own
    bool turned;               // it runs from short to long
    int first, len;      // this lane's prompt: first token, tokens
    int cnt, sum;        // ... its blocks of one kv head on this die, those of the lanes up to it
    int up;              // blocks of the group from level step * lane up (see pf_next)
    int nfirst, nend;    // first token and end for the 64 prompts after these: asked for when these are taken into use
};

struct PfDeal {
    int lane, wg, wgs, gg_shift, heads, s_shift, share; // see pf_deal
};

__device__ __forceinline__ PfDeal pf_deal(const PrefillLaunch &a)
{
    PfDeal d;
    const int die = blockIdx.x & 7;
    d.lane = threadIdx.x & 63;
    d.wg = blockIdx.x >> 3;
    d.wgs = gridDim.x >> 3;
    d.gg_shift = (a.Hkv & 7) == 0 ? 3 : (a.Hkv & 3) == 0 ? 2 : (a.Hkv & 1) == 0 ? 1 : 0;
    d.heads = a.Hkv >> d.gg_shift;
    d.s_shift = 3 - d.gg_shift;
    d.share = die >> d.gg_shift;
    return d;
}

// x / n for 0 <= x < 2^31, with m = ceil(2^32 / n) (n == 1: m is not used).  The product overestimates the quotient by
// less than x / 2^32, so by one at most.
__device__ __forceinline__ int pf_div(int x, int n, uint32_t m)
{
    if (n == 1) return x;
    const int q = (int)__umulhi((uint32_t)x, m);
    return q - ((uint32_t)q * (uint32_t)n > (uint32_t)x);
}

// Asks for 64 prompts; takes them into use (and asks for the 64 after them).
__device__ __forceinline__ void pf_ask(const PrefillLaunch &a, const PfDeal &d, PfCursor &c, int base)
{
    const int g = base + d.lane;
    c.nfirst = c.nend = 0;
    if (g < a.num_prompts) c.nfirst = a.cu[g], c.nend = a.cu[g + 1];
}
__device__ __forceinline__ void pf_take(const PrefillLaunch &a, const PfDeal &d, PfCursor &c)
{
    const int len = c.nend - c.nfirst;
    c.first = c.nfirst;
    c.len = len < 0 ? 0 : (len < a.limit ? len : a.limit);
    if (c.base + 64 < a.num_prompts) pf_ask(a, d, c, c.base + 64);
    // this die's share of a pair's blocks: numbers s, s + S, ... (s moves on with the prompt, or one die would get every
    // pair's longest block)
    const int S = 1 << d.s_shift, s = (d.share + c.base + d.lane) & (S - 1);
    const int nb = (((c.len + 31) >> 5) * a.G + a.units - 1) >> a.units_shift;
    c.cnt = nb > s ? (nb - s + S - 1) >> d.s_shift : 0;
    c.sum = c.cnt + wave_scan(c.cnt, d.lane, c.all);
    c.all *= d.heads;
    c.lane0 = c.before = c.blocks = 0;
}

// The workgroup's next block (its first one when c.round is 0); false when it has no more.  The instructions on the way to
// a block count, every wave issues them: prompts are passed by 64 at a time, and a block's place is found without a walk.
// (Walked to prompt by prompt, by two cursors, 25 votes to a group of 16, against so: 876 -> 71 us for 4096 prompts of 16
// tokens, four heads on one kv head, D = 64; 421 -> 260 for 1024 of 64 and 110 -> 104 for 32 of 512, 28 on four, D = 128.
// A call of this is about 0.3 us.)
template <bool STAY, bool VOTES> __device__ __forceinline__ bool pf_next(const PrefillLaunch &a, const PfDeal &d, PfCursor &c, PfBlock &b)
{
    // back and forth: places wg, 2 wgs - 1 - wg, 2 wgs + wg, ...
    const int place = c.round * d.wgs + (c.round & 1 ? d.wgs - 1 - d.wg : d.wg);
    c.round++;
    while (place - c.done >= c.all) {
        if (c.base + 64 >= a.num_prompts) return false;
        c.done += c.all;
        c.base += 64;
        pf_take(a, d, c);
    }
    int o = place - c.done;
    // A block's level is the number of blocks left in its pair's share behind it: the highest level first.  Level j has a
    // block of every (prompt, head) with more than j, so the levels from j up hold heads * sum(max(cnt - j, 0)), and the
    // place's level is the last one for which that exceeds o: every lane tries one level, every `step`th at first.
    auto from_level = [&](int j) __attribute__((always_inline)) {
        const int left = a.num_prompts - c.base - c.lane0, prompts = left < a.group ? left : a.group;
        int n = 0;
#pragma unroll 1
        for (int i0 = 0; i0 < prompts; i0 += 8) {
#pragma unroll
            for (int i = 0; i < 8; i++) {
                const int over = __builtin_amdgcn_readlane(c.cnt, c.lane0 + i0 + i) - j;
                n += over > 0 ? over : 0;
            }
        }
        return n * d.heads;
    };
    // (A call of few blocks is so short that it counts where there is but one level to try: 0.3 us of 9.7 for 30 prompts of up to 19
    // tokens, eight heads; workgroups that stay would pay for the question.)
    const bool flat = !STAY && a.levels == 1;
    int step = (a.levels + 63) >> 6;
    if (o >= c.before + c.blocks) { // another group of prompts
        c.lane0 = (__ffsll((long long)__ballot(c.sum * d.heads > o)) - 1) & -a.group;
        c.before = c.lane0 ? __builtin_amdgcn_readlane(c.sum, c.lane0 - 1) * d.heads : 0;
        c.blocks = __builtin_amdgcn_readlane(c.sum, c.lane0 + a.group - 1) * d.heads - c.before;
        if (!VOTES && !flat) c.up = from_level(d.lane * step);
        // Every other group, if it starts in the middle of a round, runs from short to long: its first blocks go to the
        // workgroups that got the last and shortest ones of the group before.  (Turned about, a group of one round that
        // starts with a round would give its longest blocks to the workgroups that have just had the longest ones: 32
        // prompts of 512 tokens and eight heads without sharing, two rounds of 32 blocks for a die,
        // 60.1 -> 54.7 us; 58 of 792 tokens 241 -> 191.)
        const int at = c.done + c.before, phase = 4 * (at - pf_div(at, d.wgs, a.magic_wgs) * d.wgs);
        c.turned = STAY && ((c.base + c.lane0) / a.group & 1) && phase > d.wgs && phase < 3 * d.wgs;
    }
    o -= c.before;
    if (c.turned) o = c.blocks - 1 - o;
    int j = 0, up = c.up, left = c.blocks;
    const bool mine = (d.lane & -a.group) == c.lane0;
    while (VOTES) { // (left > o >= 0 blocks are of level j and up, so some are of level j)
        const int below = left - __popcll(__ballot(mine && c.cnt > j)) * d.heads;
        if (below <= o) break;
        left = below, j++;
    }
    while (!VOTES && !flat) {
        const int k = __popcll(__ballot(up > o)) - 1;
        left = __builtin_amdgcn_readlane(up, k); // blocks of level j and up
        j += k * step;
        if (step == 1) break;
        step = (step + 63) >> 6;
        up = from_level(j + d.lane * step);
    }
    const unsigned long long m = __ballot(mine && c.cnt > j);
    o -= left - __popcll(m) * d.heads; // the place inside the level
    const int nth = pf_div(o, d.heads, a.magic_heads), x = o - nth * d.heads;
    const int rank = __popcll(m & ((1ull << d.lane) - 1ull));
    const int l = __ffsll((long long)(m & __ballot(rank == nth))) - 1;
    b.g = c.base + l;
    b.t0 = __builtin_amdgcn_readlane(c.first, l);
    b.len = __builtin_amdgcn_readlane(c.len, l);
    b.kvh = ((int)blockIdx.x & ((1 << d.gg_shift) - 1)) + (x << d.gg_shift);
    b.u0 = (((d.share + b.g) & ((1 << d.s_shift) - 1)) + ((__builtin_amdgcn_readlane(c.cnt, l) - 1 - j) << d.s_shift)) << a.units_shift;
    b.nst = b.tiles() - pf_div(b.u0, a.G, a.magic_g);
    return true;
}

// The ring of a workgroup of W waves, and its LDS: kPfSlots chunks, and the waves' staging areas.
template <int D, int W> struct PfRing {
    static constexpr int kChunk = W == 8 ? 2 : 1; // stages of a chunk
    static constexpr int kBytes = kPfSlots * kChunk * Geo<D, 2>::kStage + kPfStageBytes * W;
};

// STAY: the workgroups stay: as many per die as it has compute units, each taking its blocks one after the other.  K and
// V of one block after the other stream through one ring, so the first chunks of the next block (and its query rows,
// into registers) are loaded while the last stages of the current one are being multiplied: a block starts without a
// trip to memory.  Without STAY there is a workgroup per block, which finds it by sums or (VOTES) by votes: see
// launch_prefill.  max_len is the host's upper bound of a prompt's length.
template <int D, bool STAY, int W, bool VOTES> __device__ __forceinline__ void prefill_blocks(PrefillLaunch a)
{
    constexpr int KP = W == 8 && !STAY ? 2 : 1; // parts that a unit's keys are in, each with a wave of its own
    using G = Geo<D, 2>;
    using R = PfRing<D, W>;
    constexpr int NSL = kPfSlots, CS = R::kChunk; // ring slots of one chunk; stage number s (counted over all the blocks of
                                                  // the workgroup) lives at (s % (CS * NSL)) * G::kStage
    static_assert(CS == 2 || !STAY, "V's addresses serve two steps: a block's first stage lies at an even place of the ring");
    auto chunks = [](const PfBlock &b) __attribute__((always_inline)) { return (b.nst + CS - 1) >> (CS - 1); };
    static_assert((NSL & (NSL - 1)) == 0, "slot arithmetic by masking");
    extern __shared__ __attribute__((aligned(16384))) uint8_t lds[]; // the step forms LDS addresses by XOR
    const uint32_t lds_addr = (uint32_t)(uintptr_t)lds;
    const int lane = threadIdx.x & 63, n = lane & 31, hh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);

    // the block that is being multiplied, and the ones after it: loading is two chunks ahead, so at most three blocks
    const PfDeal deal = pf_deal(a);
    PfCursor cur;
    cur.base = cur.done = cur.round = 0, cur.turned = false, cur.up = 0;
    pf_ask(a, deal, cur, 0);
    pf_take(a, deal, cur);
    PfBlock cb, n1, n2, n3;
    if (__builtin_expect(!pf_next<STAY, VOTES>(a, deal, cur, cb), 0)) return; // the whole workgroup
    int ahead = 0;      // blocks in n1, n2, n3: three until there are no more (STAY)
    bool last_known = false;
    auto look_ahead = [&](PfBlock &b) __attribute__((always_inline)) {
        if (!STAY || last_known) return;
        last_known = !pf_next<STAY, VOTES>(a, deal, cur, b);
        if (!last_known) ahead++;
    };

    LaneConst<D, 2> lc;
    lane_setup<D, 2>(lc, lane, a.Hkv * D * 2);
    PfLane<D> pl;
    pf_lane_setup<D>(pl, lane);

    // Waves 0..3 load the chunks {K0 K1 V0 V1 | K2 K3 V2 V3}: wave w brings tile w of both stages.  (Waves 4..7, the
    // second on each SIMD, are the ones that arrive last at the barriers; they issue no loads.)  With two parts waves 4..7
    // bring the second stage's.
    constexpr int LS = KP == 2 ? 1 : CS;     // stages of a chunk that a loading wave brings a tile of
    constexpr int DPW = LS * G::kDmaPerTile; // its loads per chunk
    const int tile = wave & 3, part = KP == 2 ? wave >> 2 : 0;
    const bool loader = W == 4 || KP == 2 || wave < 4;
    const int64_t tok_bytes = (int64_t)a.Hkv * D * 2;
    const uint32_t dst = lds_addr + part * G::kStage + tile * G::kTile;
    int issued = 0;  // chunks issued, counted over all blocks: chunk number c lives in ring slot c % NSL
    int lchunk = 0;  // chunks of the block being loaded that have been issued
    int tok = 0;     // first key of the wave's tile in the chunk to load next
    int l_len = 0, l_chunks = 0; // the block being loaded: tokens of its prompt, chunks
    int lb = 0;                  // which one it is: 0 cb, 1 n1, ...; past `ahead`: there is none
    const uint8_t *src = nullptr;
    auto load_from = [&](int t0, int kvh, int len, int chunks) __attribute__((always_inline)) {
        tok = kPage * (tile & 1) + 32 * part;
        src = (const uint8_t *)((tile < 2 ? a.k : a.v) + ((int64_t)(t0 + tok) * a.Hkv + kvh) * D);
        l_len = len, l_chunks = chunks;
        lchunk = 0;
    };
    auto load_chunk = [&]() __attribute__((always_inline)) { // the next chunk of the sequence
        if (loader) {
            const uint32_t d = dst + (issued & (NSL - 1)) * CS * G::kStage;
#pragma unroll
            for (int i = 0; i < LS; i++) issue_tile<D, 2>(lc, src + 32 * i * tok_bytes, l_len - tok - 32 * i, d + i * G::kStage, a.zeros); // keys past the end read zeros
        }
        src += 32 * CS * tok_bytes;
        tok += 32 * CS;
        issued++;
        lchunk++;
    };
    auto next_to_load = [&]() __attribute__((always_inline)) {
        if (lchunk < l_chunks) return;
        lb++;
        if (lb > ahead) return;
        auto of = [&](int x1, int x2, int x3) __attribute__((always_inline)) { return lb == 1 ? x1 : lb == 2 ? x2 : x3; };
        load_from(of(n1.t0, n2.t0, n3.t0), of(n1.kvh, n2.kvh, n3.kvh), of(n1.len, n2.len, n3.len), of(chunks(n1), chunks(n2), chunks(n3)));
    };
    auto issue = [&]() __attribute__((always_inline)) { // ... if there is one
        if (lb > ahead) return;
        load_chunk();
        next_to_load();
    };
    // The ring.  While a wave is in step s it reads V of stage s and K of stage s + 1.  The barrier that opens chunk
    // c (before the first step that reads its K) says that every wave's loads of the chunk have landed and that
    // every wave has left the last step that read chunk c - 2, whose slot then takes chunk c + 2 (the first two
    // chunks are loaded up front).  Chunks are numbered over all blocks, so the same holds across a block's end.
    //
    // The cache write, from the tiles that stream through the ring anyway (16 keys of a kv head: a page).  A stage's K and
    // V are written by the block that holds the first head's unit of the stage's tile, which spreads them evenly over the
    // blocks; wave w takes tile w of the chunk that has just been opened.  The stores go past the caches, like the results':
    // 64 prompts of 50 to 500 tokens, 40 heads on eight, 143.7 -> 131.3 us (with a decode step over the pages 155.5 -> 149.1),
    // 32 of 512, 28 on four, 96.1 -> 96.2 (104.3 -> 104.5), 64 of 256 75.4 -> 74.4 (84.7 -> 84.5).
    int w_lo = 1 << 30, w_hi = -1; // the block's stages to be written
    auto pages_of_block = [&]() __attribute__((always_inline)) {
        const int units = cb.tiles() * a.G, end = (cb.u0 + a.units < units ? cb.u0 + a.units : units) - 1;
        w_hi = cb.tiles() - 1 - pf_div(cb.u0 + a.G - 1, a.G, a.magic_g);
        w_lo = cb.tiles() - 1 - pf_div(end, a.G, a.magic_g);
    };
    auto write_page = [&](int c, int stage) __attribute__((always_inline)) { // chunk (counted over all blocks), stage of the block
        const int pi = 2 * stage + (wave & 1), p0 = uniform_load(a.page_off, cb.g), is_v = wave & 2;
        int rows = cb.len - kPage * pi;
        if (rows <= 0 || kPage * pi >= a.max_len || pi >= uniform_load(a.page_off, cb.g + 1) - p0) return;
        rows = rows < kPage ? rows : kPage;
        const int pid = uniform_load(a.pages, (int64_t)p0 + pi);
        if (pid < 0 || pid >= a.num_pages) return;
        int ln = lane;
        asm volatile("" : "+v"(ln)); // (nothing of this is to be kept in registers through the block)
        const uint8_t *const tile = lds + (c & (NSL - 1)) * CS * G::kStage + (wave >> 2) * G::kStage + (wave & 3) * G::kTile + 16 * ln;
        uint8_t *const page = (is_v ? a.v_pool : a.k_pool) + (int64_t)pid * a.stride_page_b + (int64_t)cb.kvh * a.stride_head_b;
        auto piece = [&](int x) __attribute__((always_inline)) { return *(const uint4 *)(tile + 1024 * x); };
        auto row_of = [&](int x) __attribute__((always_inline)) { return 64 / G::kUnits * x + ln / G::kUnits; };
        auto byte_of = [&](int x) __attribute__((always_inline)) { return 16 * (ln % G::kUnits ^ (swz(row_of(x)) & (G::kUnits - 1))); };
        if (!a.kv_fp8) {
#pragma unroll
            for (int x = 0; x < G::kDmaPerTile; x++) {
                const uint4 w = piece(x);
                if (row_of(x) < rows) __builtin_nontemporal_store(__builtin_bit_cast(u32x4, w), (u32x4 *)(page + (int64_t)row_of(x) * a.stride_token_b + byte_of(x)));
            }
            return;
        }
        // (rows past the end hold zeros: they do not change the maximum)
        uint32_t m = 0;
#pragma unroll
        for (int x = 0; x < G::kDmaPerTile; x++) m = bf16_mag_max(m, piece(x));
        m = bf16_mag_reduce(m);
        float amax = __uint_as_float(m << 16);
        if (__builtin_expect(m > 0x7f80, 0)) { // a NaN does not take part in the maximum
            amax = 0.f;
#pragma unroll 1
            for (int x = 0; x < G::kDmaPerTile; x++) {
                const uint4 w = piece(x);
                amax = fmaxf(amax, fmaxf(fmaxf(fabsf(bf16_lo(w.x)), fabsf(bf16_hi(w.x))), fmaxf(fabsf(bf16_lo(w.y)), fabsf(bf16_hi(w.y)))));
                amax = fmaxf(amax, fmaxf(fmaxf(fabsf(bf16_lo(w.z)), fabsf(bf16_hi(w.z))), fmaxf(fabsf(bf16_lo(w.w)), fabsf(bf16_hi(w.w)))));
            }
#pragma unroll 1
            for (int sh = 32; sh >= 1; sh >>= 1) amax = fmaxf(amax, __shfl_xor(amax, sh));
        }
        const float scale = amax > 0.f ? amax / 448.0f : 1.0f;
        const E4m3Scale sc = {scale, 1.0f / scale};
        const bool fast = m <= 0x7f80 && E4m3Scale::ok(amax);
#pragma unroll 1
        for (int x = 0; x < G::kDmaPerTile; x++) {
            const uint4 w = piece(x);
            const uint2 codes = fast ? e4m3_codes8(sc, w) : e4m3_codes8_any(scale, w);
            if (row_of(x) < rows) __builtin_nontemporal_store(__builtin_bit_cast(u32x2, codes), (u32x2 *)(page + (int64_t)row_of(x) * a.stride_token_b + byte_of(x) / 2));
        }
        if (ln == 0) (is_v ? a.v_scale : a.k_scale)[(int64_t)pid * a.Hkv + cb.kvh] = scale;
    };
    auto open_chunk = [&](int c, int s0) __attribute__((always_inline)) { // s0: the block's stage that the chunk starts with
        if (loader) WaitTail<NSL - 1, DPW>::run(issued - 1 - c);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        issue();
        const int stage = s0 + (wave >> 2);
        if (stage >= w_lo && stage <= w_hi) write_page(c, stage);
    };

    // The wave's unit of a block: waves w and w + 4 share a SIMD, so the longest and the shortest go together.  Past the
    // block's last unit a wave has none: it keeps the ring going and computes nothing.
    const int order = KP == 2 ? wave & 3 : wave < 4 ? wave : W + 3 - wave;
    auto unit_of = [&](const PfBlock &b, int &head, int &tile_q) -> bool {
        const int units = b.tiles() * a.G;
        int u = b.u0 + order;
        const bool own = order < a.units && u < units;
        u = own ? u : units - 1;
        const int q = pf_div(u, a.G, a.magic_g);
        tile_q = b.tiles() - 1 - q;
        head = b.kvh * a.G + (u - q * a.G);
        return own;
    };
    // A lane's part of its query row (a row past the prompt's end reads the prompt's last row instead, and is
    // zeroed by keep_q when the registers are taken into use: nothing writes the registers but the loads themselves,
    // so the compiler has no reason to wait for older loads before them).
    auto load_q = [&](const PfBlock &b, int head, int tile_q, bf16x8 (&qf)[D / 16]) {
        int row = kPfRows * tile_q + n;
        row = row < b.len ? row : b.len - 1;
#pragma unroll
        for (int i = 0; i < D / 16; i++) qf[i] = *(const bf16x8 *)(a.q + ((int64_t)(b.t0 + row) * a.Hq + head) * D + 16 * i + 8 * hh);
    };
    auto keep_q = [&](const PfBlock &b, int tile_q, bf16x8 (&qf)[D / 16]) {
        const bool ok = kPfRows * tile_q + n < b.len;
#pragma unroll
        for (int i = 0; i < D / 16; i++) {
            if (!ok) qf[i] = bf16x8{0, 0, 0, 0, 0, 0, 0, 0};
            asm volatile("" : "+v"(qf[i]));
        }
    };
    // the wave's staging area behind the ring (32 rows of 128 bytes)
    uint8_t *const stage = lds + NSL * CS * G::kStage + kPfStageBytes * wave;
    // Query rows come straight from memory, 16 bytes per lane and row.  Those of the block after the current one are
    // asked for (into qn) when the current block has its first scores, and waited for when its last step is done: qn and
    // st.qf change places there.  (The empty asm statements pin the compiler's wait for the loads to these places; left
    // to the first use it would sit inside a block and wait for younger loads as well.)
    PfState<D> st;
    bf16x8 qn[D / 16];
    int head, T;    // of the current block: the wave's head and tile
    int chunk0 = 0; // number of the current block's first chunk
    load_from(cb.t0, cb.kvh, cb.len, chunks(cb));
    load_chunk(); // (the second one follows below, the rest the barriers, one chunk at a time)
    bool own = unit_of(cb, head, T);
    load_q(cb, head, T, st.qf);
    if (STAY) {
#pragma unroll 1
        for (int i = 0; i < 3; i++) { // while they are on their way
            n1 = n2, n2 = n3;
            look_ahead(n3);
        }
    }
    next_to_load();
    issue();
    keep_q(cb, T, st.qf);

    for (;;) {
        const int nst = cb.nst;
        const int stage0 = CS * chunk0;
        const int row = kPfRows * T + n;
        st.lsum = 0.f;
#pragma unroll
        for (int dt = 0; dt < D / 32; dt++) {
#pragma unroll
            for (int e = 0; e < 16; e++) st.o[dt][e] = 0.f;
        }
        // The wave's stages of the block: number i is stage KP * i + part.  The last one is the one that holds the tile's
        // diagonal, or with two parts the one before it; earlier ones lie wholly below it.
        const int last = KP == 1 ? T : (T - part) >> 1;
        const bool works = own && (KP == 1 || T >= part);

        if (a.fused_write) pages_of_block();
        open_chunk(chunk0, 0);
        if (works) pf_scores<D>(lds_addr + ((stage0 + part) & (CS * NSL - 1)) * G::kStage, pl, st.qf, st.s);
        if (last == 0) {
#pragma unroll
            for (int e = 0; e < 16; e++) {
                if (32 * part + 8 * (e / 4) + 4 * hh + (e % 4) > row) st.s[e] = -INFINITY;
            }
        }
        {
            float mx = max3(first_max(st.s[0], st.s[1]), st.s[2], st.s[2]);
#pragma unroll
            for (int e = 3; e < 15; e += 2) mx = max3(mx, st.s[e], st.s[e + 1]);
            mx = max3(mx, st.s[15], st.s[15]);
            const u32x2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
            st.m = fmaxf(max3(__uint_as_float(r[0]), __uint_as_float(r[1]), __uint_as_float(r[1])) * a.scale_log2, kPfLowest);
            if (KP == 2 && !works) st.m = kPfLowest;
        }
        int nhead = 0, nT = 0;
        bool nown = false;
        const bool more = ahead > 0;
        if (more) {
            nown = unit_of(n1, nhead, nT);
            if (nown) load_q(n1, nhead, nT, qn);
        }
        // every wave keeps the ring going for all the stages; it computes up to its own last stage: full steps, then
        // the step whose new scores cross the diagonal, then the step without new scores
        auto ring = [&](int s) __attribute__((always_inline)) { // before step s
            if (KP == 2) {
                if (2 * (s + 1) < nst) open_chunk(chunk0 + s + 1, 2 * (s + 1));
            } else if ((CS == 1 || (s & 1)) && s + 1 < nst) open_chunk(chunk0 + ((s + 1) >> (CS - 1)), s + 1);
        };
        constexpr bool EACH = KP == 2 || CS == 1; // a chunk opens before every step
#define PF_STEP(MASK, NEXT, SECOND)                                                                                                \
    pf_step<D, MASK, NEXT, SECOND>(st, lds_addr + ((stage0 + part + KP * (s + 1)) & (CS * NSL - 1)) * G::kStage,            \
                                   lds_addr + ((stage0 + part + KP * s) & (CS * NSL - 1)) * G::kStage + 2 * G::kTile, va, pl, a.scale_log2, \
                                   32 * (KP * (s + 1) + part), row)
        int s = 0;
        if (works) {
            uint32_t va[D / 32][2];
            // Two steps at a time: the chunk opens between them, V's addresses serve both, and the scores need not change
            // registers (sixteen moves a step): 16 prompts of 2048, 64 heads on eight, e4m3, 1226 -> 1190 us, 16 of 1024, 32 on
            // two, D = 64, 112.5 -> 107.2.
#pragma unroll 1
            for (; s + 2 < last; s += 2) {
                if (EACH) ring(s);
                PF_STEP(false, true, 0);
                s++;
                ring(s);
                PF_STEP(false, true, KP);
                s--;
            }
            if (s + 1 < last) { // s is even
                if (EACH) ring(s);
                PF_STEP(false, true, 0);
                s++;
            }
            if (s + 1 == last) {
                ring(s);
                PF_STEP(true, true, 0);
                s++;
            }
            ring(s);
            PF_STEP(false, false, 0);
            s++;
        }
        for (; KP * s < nst; s++) ring(s);
#undef PF_STEP

        // the next block's query rows take their place
        const int t0 = cb.t0, len = own ? cb.len : 0, dhead = head, tile_row = kPfRows * T;
        if (more) {
            PfBlock n4;
            look_ahead(n4); // (while the query rows may still be on their way)
#pragma unroll
            for (int i = 0; i < D / 16; i++) st.qf[i] = qn[i];
            keep_q(n1, nT, st.qf);
            chunk0 += chunks(cb);
            cb = n1, n1 = n2, n2 = n3, n3 = n4;
            head = nhead, T = nT, own = nown;
            ahead--, lb--;
        }

        if (KP == 2) {
            // Half of the keys each: the waves of a unit exchange what they have.  With D = 128 each of them ends up with one
            // half of the d tiles, with D = 64 the first one with all.
            constexpr int DT = D / 32, MINE = D == 128 ? DT / 2 : DT, BYTES = 8 * 1024 + 512;
            static_assert(KP == 1 || (D == 128 ? 8 : 4) * BYTES <= NSL * CS * G::kStage, "what is exchanged fits the ring");
            auto meet = [&]() __attribute__((always_inline)) {
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
            };
            meet(); // (the ring is done with: every chunk has landed and has been read)
            if (D == 128 && part) {
#pragma unroll
                for (int dt = 0; dt < MINE; dt++) {
                    const f32x16 x = st.o[dt];
                    st.o[dt] = st.o[(dt + MINE) % DT];
                    st.o[(dt + MINE) % DT] = x;
                }
            }
            const bool gives = D == 128 || part, takes = D == 128 || !part;
            if (gives) {
                uint8_t *const at = lds + (D == 128 ? wave : wave & 3) * BYTES;
#pragma unroll
                for (int k = 0; k < 8; k++) {
                    const f32x16 &x = st.o[MINE % DT + k / 4];
                    *(f32x4 *)(at + 1024 * k + 16 * lane) = f32x4{x[4 * (k % 4)], x[4 * (k % 4) + 1], x[4 * (k % 4) + 2], x[4 * (k % 4) + 3]};
                }
                *(float *)(at + 8 * 1024 + 4 * lane) = st.m;
                *(float *)(at + 8 * 1024 + 256 + 4 * lane) = st.lsum;
            }
            meet();
            if (takes) {
                const uint8_t *const at = lds + (D == 128 ? wave ^ 4 : wave) * BYTES;
                const float m2 = *(const float *)(at + 8 * 1024 + 4 * lane), l2 = *(const float *)(at + 8 * 1024 + 256 + 4 * lane);
                const float mm = fmaxf(st.m, m2), a1 = __builtin_amdgcn_exp2f(st.m - mm), a2 = __builtin_amdgcn_exp2f(m2 - mm);
                st.m = mm;
                st.lsum = st.lsum * a1 + l2 * a2;
#pragma unroll
                for (int k = 0; k < 8; k++) {
                    const f32x4 y = *(const f32x4 *)(at + 1024 * k + 16 * lane);
#pragma unroll
                    for (int x = 0; x < 4; x++) st.o[k / 4][4 * (k % 4) + x] = st.o[k / 4][4 * (k % 4) + x] * a1 + y[x] * a2;
                }
            }
        }
        if (len > 0 && !(KP == 2 && D == 64 && part)) {
            const int col0 = KP == 2 ? 64 * part : 0; // first d of what the wave stores
            // a row's sum is spread over its two lanes
            float l;
            {
                const u32x2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(st.lsum), __float_as_uint(st.lsum), false, false);
                l = __uint_as_float(r[0]) + __uint_as_float(r[1]);
            }
            const float inv = 1.0f / l;
            const int64_t rh = (int64_t)(t0 + row) * a.Hq + dhead;
            // Results go through the wave's staging area, 64 d (128 bytes of every row) at a time: a lane holds four consecutive
            // d of its own row per accumulator quarter, and storing from there is 32 separate pieces of 16 bytes per
            // instruction, which keeps the compute unit's one memory pipeline busy for microseconds per block; read back eight
            // lanes to a row, an instruction stores whole 128-byte lines.
            int sl = lane;
            asm volatile("" : "+v"(sl));
            const int sn = sl & 31, sh = sl >> 5;
#pragma unroll
            for (int p = 0; p < (KP == 2 ? 1 : D / 64); p++) {
#pragma unroll
                for (int dtl = 0; dtl < 2; dtl++) {
#pragma unroll
                    for (int j = 0; j < 4; j++) {
                        f32x4 v;
#pragma unroll
                        for (int x = 0; x < 4; x++) v[x] = st.o[2 * p + dtl][4 * j + x] * inv; // d = 64 p + 32 dtl + 8 j + 4 hh + x
                        *(bf16x4 *)(stage + kPfStageRow * sn + 16 * ((4 * dtl + j) ^ pf_stage_swz(sn)) + 8 * sh) = __builtin_convertvector(v, bf16x4);
                    }
                }
#pragma unroll
                for (int m = 0; m < 4; m++) {
                    const int r = 8 * m + (sl >> 3), c = sl & 7; // row of the tile, 16-byte piece of its 128 bytes
                    const u32x4 v = *(const u32x4 *)(stage + kPfStageRow * r + 16 * (c ^ pf_stage_swz(r)));
                    const int orow = tile_row + r;
                    // (Past the caches: K, V and the queries are read from them meanwhile.  Same inputs call after call, in turn
                    // on one card: 32 prompts of 512 tokens, 28 heads on four, 99.8 -> 94.4 us, 64 of 256 79.8 -> 74.7, 24 of
                    // 200 to 1500 206.6 -> 195.6, 64 of 50 to 500, 40 on eight, 146.0 -> 129.7.  A matrix product over the
                    // results (their heads' width square) finds those that the last-level cache would have held no longer
                    // there; both calls: 436.4 -> 438.4, 413.7 -> 416.8, 672.3 -> 669.8, 861.6 -> 858.8, 16 of 512 219.9 ->
                    // 218.1, eight of 37 to 701 107.0 -> 106.2; a copy of them 135.6 -> 143.8, 118.3 -> 126.8, 252.7 -> 245.5,
                    // 208.1 -> 207.3.)
                    if (orow < len) __builtin_nontemporal_store(v, (u32x4 *)(a.out + ((int64_t)(t0 + orow) * a.Hq + dhead) * D + col0 + 64 * p + 8 * c));
                }
            }
            if (row < len && hh == 0 && part == 0) a.lse[rh] = (st.m + __builtin_amdgcn_logf(l)) * 0.6931471805599453f;
        }
        if (!more) break;
    }
    wait_vmcnt<0>(); // nothing may land in LDS after the workgroup has left
}

// A workgroup per block: what the first trip needs comes in arguments that are in registers when a wave starts: one prompt of 32
// tokens 6.0 -> 5.8 us.
template <int D, int W, bool VOTES = false> __global__ __launch_bounds__(64 * W, 2) void prefill_kernel(const int32_t *__restrict__ cu, int num_prompts, int limit, int G, int Hkv,
                                                                                              int units_shift, PrefillLaunch given)
{
    PrefillLaunch a = given;
    a.cu = cu, a.num_prompts = num_prompts, a.limit = limit, a.G = G, a.Hkv = Hkv, a.units_shift = units_shift, a.units = 1 << units_shift;
    prefill_blocks<D, false, W, VOTES>(a);
}

// Workgroups that stay are no faster for such arguments, and slower beside them, read or not: the compiler keeps others of the
// launch's fields in registers.  D = 64, 32 heads on two, us with them in the signature and without: 64 prompts of 200 to 210
// tokens 48.5, 48.0, 60 of 512, e4m3, 131.6, 130.9; D = 128, 32 of 512, 28 on four, 101.7, 102.2, spread 1.  (The blocks' function
// has its arguments by value.  By reference, spilling more: 48.4, 130.2, 102.4; 16 of 2048, 64 on eight, e4m3, D = 128, 1202, by
// value 1206, spread 2.)
template <int D> __global__ __launch_bounds__(64 * 8) void prefill_kernel(PrefillLaunch a)
{
    prefill_blocks<D, true, 8, false>(a);
}

} // namespace ra
