// The prompt prefill's launches (the kernel: ra_prefill.h) and the copy kernel of the cache write.
#include "ra_prefill.h"

namespace ra {

// The launch shape of a call.  Workgroups that stay load the next block's inputs under the current one, but which blocks each
// of them takes is fixed beforehand; with one per block the hardware hands them out as units become free, two or three of
// four waves to a compute unit, so that one's start and end (a block's fixed part is 4 to 5 us, its stages 0.6 each) run under
// another's stages.  Us, staying against four waves a block:
// - calls whose blocks all run side by side, about: 24 prompts of 57 to 71 tokens, 28 heads on four, 10.5, 9.1; eight of 128
//   11.9, 8.7; six of 368 (504 blocks of four units) 18.5, 15.4, but eight of 368 (702) 20.8, 21.9, ten of 256 15.8, 17.6;
// - short prompts, and any at head dim 64, up to a few rounds of such workgroups, two to a compute unit, three at D = 64: 28 of 57 to
//   71, 28 on four (1.1 rounds), 15.5, 11.9; five of 4, 64 on eight, 7.4, 5.4; 38 of up to 9, eight heads, 13.4, 5.7; 73 of 21, 40 on
//   eight (3.2), 21.0, 17.5; 42 of 37 to 49, 64 on eight (3.0), 19.1, 19.5; 127 of 18 to 24, 28 on four (4.1), 16.1, 17.3; 38 of 128 (2.5)
//   24.8, 24.4, but 24 of 97, 64 on eight (3.0), 23.2, 25.1; D = 64, 32 on two: 60 of 50 to 65 (1.7) 12.2, 10.0, 38 of 211 (3.1)
//   35.8, 27.6, twelve of 1024 (4.0) 83.2, 81.1, but 16 (5.5) 107, 117;
// - long prompts of unlike lengths, as long as a workgroup that stayed would have few blocks: 29 of 339 to 1876, four heads on
//   two, D = 64, 93.5, 45.7; 24 of 200 to 1500, 32 on two, D = 64, 146, 143.5; 50 of 200 to 1500, eight heads, 235, 219; 17 of 59
//   to 1204, 40 on eight, 170, 161; 24 of 200 to 1500, 28 on four, 227, 230 (blocks of eight waves one each: 49.9, 162, 222, 168,
//   229).  Not like ones: 16 of 860, eight heads, 63.2, 68.3; 32 of 512, 28 on four, 106, 122; 16 of 2048, 64 on eight 1182, 1320.
// - shorter ones of unlike lengths, up to fewer blocks (of eight units) to a compute unit, more at head dim 64: 24 of 16 to 300, 28
//   on four (2.1 to a unit), 33.1, 21.7; 16 of 50 to 500 (2.2) 31.4, 28.4; 20 of 150 to 480 (3.1) 50.5, 38.1; 64 of 50 to 500, eight
//   heads (2.5), 96.6, 76.8; but 14 of 124 to 413, 64 on eight (3.7), 35.1, 37.6, 32 of 50
//   to 500, 28 on four (4.3), 51.5, 54.9, 64 of 20 to 300, 64 on eight (12.8), 120, 145; D = 64:
//   32 of 30 to 400, 32 on two (3.8), 29.5, 22.8, 64 of 50 to 500 (10.1) 75.9, 69.9; nearly alike, eight of 300 to 500, 28 on four,
//   22.0, 23.1.
// The launch is sized by the tokens as well as by the bound on the lengths, which counts 256 rows for the shortest prompt.  By the
// bound alone calls of short prompts were empty workgroups mostly: 221 of 14 to 63 tokens, 32 heads on two, D = 64, 41.2 -> 29.1 us.
// (What is still empty: a prompt may have 31 tokens in a tile of its own, and the
// dies that share a pair take its blocks in turn; and as many as run side by side are launched if the bound has them: two prompts
// of 13 to 17 tokens, 64 on eight, take 5.4 us with 256 workgroups and 5.6 with the 32 that have a block, two of 231 to 367 13.0
// with 512 and 13.4 with 368.)  A bound far above the lengths leaves the call to workgroups that stay, as the levels that a
// workgroup searches are the bound's: more than eight times the blocks by the tokens, which is what the 256 rows make of prompts of
// one tile; where the choice is by unlike lengths, which a bound can feign, more than four times.
// Not many short prompts either: a workgroup passes all prompts before its own, 64 to a trip.  Trips to a round of workgroups side by
// side (rounds times prompts / 64), us, staying and four waves: with four query heads to a kv head and more 351 prompts of 22
// to 43, eight on one (28), 24.0, 21.6; 391 of 18 to 58 (36) 22.4, 24.9; 442 of 31 to 61, sixteen on one, D = 64 (52) 38.5, 35.5; 1225
// of 28 to 57, eight on two, D = 64 (231) 54.4, 72.0; with fewer, where a block of eight units is mostly empty, 1037 of 24 to 59, four
// on four, D = 64 (159) 81.0, 56.1; 964 of 32 to 57, four on two (120) 43.7, 45.0; 1032 of 9 to 294 (208) 119, 108; 1226 of 40 to 135
// (235) 77.6, 94.7; 6693 of 14 to 56, one head (1824) 139, 333.
// A call of so few blocks that each has a compute unit to itself lasts as long as its longest block: beyond 256 tokens two
// waves share a unit's keys, at head dim 64, where a chunk of one stage is little to have on the way, beyond 224.  One prompt, 28
// heads on four, four waves and eight (and before either): 256 tokens 10.8, 10.8 (10.9); 400 13.5, 12.8 (13.8); 701 20.1, 17.6
// (19.7); 593, four on two, D = 64, 15.4, 14.2 (14.8); eight on two, D = 64, 160 6.7, 7.1 (6.9), 200 7.3,
// 7.3 (7.3), 250 8.2, 7.9 (7.7); beyond a unit each, three of 600 18.4, 21.4, four of
// 368 14.4, 17.6.  (The line is by blocks, whosever they are; a lone prompt would still be faster by eight: of 1200 tokens 30.1, 25.5, of
// 1800 43.2, 36.4, but two of 900 24.6, 25.7.)
PrefillShape prefill_shape(int num_prompts, int total_tokens, int max_len, int Hkv, int G, int D, int num_cus, int stay)
{
    PrefillShape p = {0, 0, 0, 0};
    const int64_t rows = ((int64_t)max_len + kPfBlock - 1) / kPfBlock * kPfBlock;
    const int gg_shift = (Hkv & 7) == 0 ? 3 : (Hkv & 3) == 0 ? 2 : (Hkv & 1) == 0 ? 1 : 0, s_shift = 3 - gg_shift, share = 1 << s_shift, heads = Hkv >> gg_shift;
    int64_t per_die = num_cus / 8;
    per_die = per_die < 1 ? 1 : per_die;
    if (stay > 0 && stay < per_die) per_die = stay; // fewer were asked for
    // Blocks of a die at most (by the bound on the lengths, and by the tokens too) and of the batch about (by its tokens).  (Shifts
    // for divisions: with those a call's host side took 0.2 us longer.)
    int64_t by_bound, by_tokens, blocks, about;
    auto count = [&](int shift) { // ... of 2^shift units
        const int64_t n = num_prompts, tiles = ((int64_t)total_tokens + 31 * n) >> 5, most = (1 << shift) - 1, per_pair = (rows / 32 * G + most) >> shift;
        by_bound = heads * (n * (per_pair >> s_shift) + ((n + share - 1) >> s_shift) * (per_pair & (share - 1)));
        about = tiles * Hkv * G >> shift;
        p.levels = (int)((per_pair + share - 1) >> s_shift);
        // A pair's units are a multiple of G, so its last block lacks 2^shift - gcd(G, 2^shift) at most.  A die takes the numbers
        // s, s + share, ... of a pair's blocks, another s for every prompt in turn: (blocks - s + share - 1) / share of them.
        const int64_t lacks = (G & most) == 0 ? 0 : most + 1 - (G & -G), rest = n & (share - 1);
        const int64_t in_turn = (n >> s_shift) * (share * (share - 1) / 2) + rest * (share - 1) - rest * (rest - 1) / 2;
        by_tokens = heads * ((((tiles * G + n * lacks) >> shift) + in_turn) >> s_shift);
        blocks = by_bound < by_tokens ? by_bound : by_tokens;
    };
    count(3);
    const bool fit = by_bound <= per_die; // (a block for every compute unit at most: there is nothing to load ahead)
    const bool alike = 8 * (int64_t)total_tokens >= 7 * (int64_t)num_prompts * max_len;
    const bool uneven = max_len > 2 * kPfBlock ? !alike && about <= 12 * (int64_t)num_cus
                                               : 5 * (int64_t)total_tokens < 4 * (int64_t)num_prompts * max_len && 2 * about <= (D == 64 ? 24 : 7) * (int64_t)num_cus;
    const PrefillShape staying = {8, 1, p.levels, (int)per_die};
    count(2);
    const int64_t side = (D == 64 ? 3 : 2) * (int64_t)num_cus; // workgroups of four waves that run side by side
    const int rounds = D == 64 ? 8 : max_len <= 64 ? 6 : max_len <= 128 ? 5 : 0; // (halves of one)
    const bool few = 8 * about <= 9 * side || 16 * blocks <= rounds * side; // (by the tokens it is a little more than it is)
    const bool near = by_bound <= (few ? 8 : 4) * by_tokens + per_die;
    const bool many = max_len <= 2 * kPfBlock && 8.0 * (double)blocks * num_prompts > (G >= 4 ? 32 : 220) * 64.0 * (double)side;
    const bool one_each = stay == 0 ? blocks <= INT32_MAX / 16 : stay < 0 && (fit || ((few || uneven) && !many && near));
    if (!one_each) return staying;
    p.parts = about <= num_cus && 4 * by_bound <= 5 * per_die && max_len > (D == 64 ? kPfBlock - 32 : kPfBlock) ? 2 : 1;
    p.waves = 4 * p.parts;
    const int64_t fill = by_bound < side / 8 ? by_bound : side / 8; // (see above)
    p.per_die = (int)(blocks < fill ? fill : blocks);
    p.per_die = p.per_die < 1 ? 1 : p.per_die;
    return p;
}

// The attention kernel writes the cache from its ring where a block has few stages to write: with fewer than four query
// heads per kv head it would be up to eight of them per block of eight units, and the copy kernel below does it.  Not where
// blocks go one to a workgroup: those have four units, and such a call is mostly the cost of a second launch: five
// prompts of 15 to 32 tokens, four heads on two, D = 64, 7.7 -> 4.6 us; one of 600, eight heads, e4m3, 22.8 -> 20.9, 21 of 195 to 419
// 34.5 -> 22.8 (bf16 33.7 -> 17.6), 50 of 200 to 1500 219 -> 206 (bf16 219 -> 190).
static bool writes_cache(const PrefillLaunch &a, const PrefillShape &p)
{
    if (a.G >= 4) return true;
    // One query head to a kv head, D = 128: a block of four waves quantises up to four stages, 1.2 us each, and where it has a compute
    // unit to itself all of it shows.  E4m3, copied first and written by the block: one prompt of 100 tokens, eight heads, 12.3, 13.6,
    // 250 15.1, 16.5, four of 100 to 250 14.7, 15.8, eight 16.0, 16.5, but twelve 18.2, 17.2, one of 70 11.5, 11.3, of 40 10.8, 8.9.
    const int64_t about = ((int64_t)a.total_tokens + 31 * (int64_t)a.num_prompts) / 32 * a.Hkv / 4;
    if (a.G == 1 && a.D == 128 && a.kv_fp8 && p.waves == 4 && a.max_len > 96 && 16 * about <= 7 * (int64_t)a.num_cus) return false;
    return p.waves != 8 || p.parts != 1;
}

hipError_t prefill_config()
{
    hipError_t e = prefill_four_config();
#define RA_PF_CONFIG(DD)                                                                                                     \
    if (e == hipSuccess) e = hipFuncSetAttribute((const void *)prefill_kernel<DD>, hipFuncAttributeMaxDynamicSharedMemorySize, PfRing<DD, 8>::kBytes); \
    if (e == hipSuccess) e = hipFuncSetAttribute((const void *)prefill_kernel<DD, 8>, hipFuncAttributeMaxDynamicSharedMemorySize, PfRing<DD, 8>::kBytes);
    RA_PF_CONFIG(128) RA_PF_CONFIG(64)
#undef RA_PF_CONFIG
    return e;
}

static hipError_t launch_prefill_write(const PrefillLaunch &a, hipStream_t s);

hipError_t launch_prefill(const PrefillLaunch &given, hipStream_t s)
{
    const int64_t pairs = (int64_t)given.num_prompts * given.Hkv;
    const int64_t rows = ((int64_t)given.max_len + kPfBlock - 1) / kPfBlock * kPfBlock;
    if (pairs == 0 || rows == 0) return hipSuccess;
    if (rows > INT32_MAX || (pairs + 7) / 8 * (rows / kPfBlock) * given.G > INT32_MAX / 16) return hipErrorInvalidValue;
    if (given.k_pool && ((int64_t)given.max_len + kPage - 1) / kPage * pairs > INT32_MAX) return hipErrorInvalidValue;
    PrefillLaunch a = given;
    a.limit = (int32_t)rows;
    const PrefillShape p = prefill_shape(a.num_prompts, a.total_tokens, a.max_len, a.Hkv, a.G, a.D, a.num_cus, a.stay);
    a.fused_write = a.k_pool && writes_cache(a, p);
    if (a.k_pool && !a.fused_write) {
        const hipError_t e = launch_prefill_write(a, s);
        if (e != hipSuccess) return e;
    }
    const bool stays = p.waves == 8 && p.parts == 1;
    const int heads = a.Hkv / ((a.Hkv & 7) == 0 ? 8 : (a.Hkv & 3) == 0 ? 4 : (a.Hkv & 1) == 0 ? 2 : 1);
    a.units_shift = stays ? 3 : 2;
    a.units = 1 << a.units_shift;
    a.levels = p.levels;
    a.magic_g = (uint32_t)((((uint64_t)1 << 32) + a.G - 1) / a.G);
    a.magic_heads = (uint32_t)((((uint64_t)1 << 32) + heads - 1) / heads);
    a.magic_wgs = (uint32_t)((((uint64_t)1 << 32) + p.per_die - 1) / p.per_die);
    // Prompts whose blocks are dealt together.  One workgroup per block: as many as there are, so that the longest blocks
    // start first.  Else few, so that a die's workgroups share their K and V in its 4 MB L2, but enough for an even deal of
    // ragged lengths: sixteen while those fit (512 tokens, D = 128, one head a die: exactly), eight above.  Measured with 64,
    // 16 and 8: 116.5, 109.7, 122.9 us on 32 prompts of 512 tokens (28 heads on four), 198.7, 193.6, 204.3 on 256 of 64 to
    // 256; 322.5, 314.3, 309.3 on 64 of 512 (40 on eight), 1301, 1294, 1279 on 16 of 2048 (64 on eight), 1148, 1124, 1108 on 32
    // of 2048 (28 on four).
    a.group = !stays ? 64 : (int64_t)16 * a.max_len * 4 * a.D * heads <= (4 << 20) ? 16 : 8;
    // How a workgroup of four waves finds its block's level.  Few levels of many prompts, as short ones have: a vote for each from the
    // lowest up.  (The sums over a group of 64 prompts are several hundred instructions; 267 prompts of 29 to 81 tokens, 32 heads on
    // two, D = 64, 45.4 -> 39.9 us, 154 of up to 86, eight heads, 25.2 -> 23.1, 25 of 20 to 100, 40 on eight, ten levels, 16.0 -> 15.1;
    // 24 of 16 to 300, 28 on four, fourteen levels, 21.3 either way.  Of few prompts they are fewer than the votes: four of 86 to 254,
    // 64 on eight, sixteen levels, 11.4, with votes 12.1.  One kernel that does either takes 0.1 us longer over the shortest calls.)
    const bool votes = 2 * p.levels <= (a.num_prompts < 32 ? a.num_prompts : 32);
    if (p.waves == 4) return launch_prefill_four(a, votes, 8u * (unsigned)p.per_die, s);
    const dim3 grid(8u * (unsigned)p.per_die), block(64 * 8);
#define RA_PF_LAUNCH(DD)                                                                                                     \
    if (stays) hipLaunchKernelGGL((prefill_kernel<DD>), grid, block, (PfRing<DD, 8>::kBytes), s, a);                            \
    else hipLaunchKernelGGL((prefill_kernel<DD, 8>), grid, block, (PfRing<DD, 8>::kBytes), s, a.cu, a.num_prompts, a.limit, a.G, a.Hkv, a.units_shift, a)
    if (a.D == 128) {
        RA_PF_LAUNCH(128);
    } else {
        RA_PF_LAUNCH(64);
    }
#undef RA_PF_LAUNCH
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------------
// Cache write: one wave per (prompt, page of the prompt, kv head) copies the page's up to sixteen K rows and V
// rows.  bf16 pools take the bit patterns.  e4m3 pools are quantised a page at a time, in binary32: scale =
// (largest magnitude among the rows written) / 448, or 1 when that is zero; code = nearest E4M3 of x / scale.
// ------------------------------------------------------------------------------------------------------
template <int D>
__device__ __forceinline__ void write_tile(const PrefillLaunch &a, const uint16_t *src, int n, uint8_t *dst, float *scale, int lane)
{
    constexpr int kUnits = D * 2 / 16;       // 16-byte units per bf16 row
    constexpr int kIter = kPage * kUnits / 64;
    const int64_t row_elems = (int64_t)a.Hkv * D;
    bf16x8 x[kIter];
#pragma unroll
    for (int i = 0; i < kIter; i++) {
        const int u = lane + 64 * i, r = u / kUnits, c = u % kUnits;
        x[i] = bf16x8{0, 0, 0, 0, 0, 0, 0, 0};
        if (r < n) x[i] = *(const bf16x8 *)(src + r * row_elems + 8 * c);
    }
    if (!a.kv_fp8) {
#pragma unroll
        for (int i = 0; i < kIter; i++) {
            const int u = lane + 64 * i, r = u / kUnits, c = u % kUnits;
            if (r < n) *(bf16x8 *)(dst + (int64_t)r * a.stride_token_b + 16 * c) = x[i];
        }
        return;
    }
    uint32_t m = 0;
#pragma unroll
    for (int i = 0; i < kIter; i++) m = bf16_mag_max(m, __builtin_bit_cast(uint4, x[i]));
    m = bf16_mag_reduce(m);
    float amax = __uint_as_float(m << 16);
    if (m > 0x7f80) { // a NaN input does not take part in the maximum
        amax = 0.f;
#pragma unroll
        for (int i = 0; i < kIter; i++) {
#pragma unroll
            for (int e = 0; e < 8; e++) amax = fmaxf(amax, fabsf((float)x[i][e]));
        }
#pragma unroll
        for (int sh = 32; sh >= 1; sh >>= 1) amax = fmaxf(amax, __shfl_xor(amax, sh));
    }
    const E4m3Scale sc = {amax > 0.f ? amax / 448.0f : 1.0f, 1.0f / (amax > 0.f ? amax / 448.0f : 1.0f)};
    const bool fast = m <= 0x7f80 && E4m3Scale::ok(amax);
#pragma unroll
    for (int i = 0; i < kIter; i++) {
        const int u = lane + 64 * i, r = u / kUnits, c = u % kUnits;
        const uint4 w = __builtin_bit_cast(uint4, x[i]);
        const uint2 codes = fast ? e4m3_codes8(sc, w) : e4m3_codes8_any(sc.s, w);
        if (r < n) *(uint2 *)(dst + (int64_t)r * a.stride_token_b + 8 * c) = codes;
    }
    if (lane == 0) *scale = sc.s;
}

template <int D> __global__ __launch_bounds__(64) void prefill_write_kernel(PrefillLaunch a)
{
    const int lane = threadIdx.x;
    const int npg = (a.max_len + kPage - 1) / kPage;
    int bid = blockIdx.x;
    const int kvh = bid % a.Hkv;
    bid /= a.Hkv;
    const int pi = bid % npg, g = bid / npg;
    const int t0 = uniform_load(a.cu, g), len = uniform_load(a.cu, g + 1) - t0;
    int n = len - kPage * pi;
    n = n < kPage ? n : kPage;
    if (n <= 0) return;
    const int p0 = uniform_load(a.page_off, g), cnt = uniform_load(a.page_off, g + 1) - p0;
    if (pi >= cnt) return; // the caller gave fewer pages than the prompt has: the rest is not cached
    const int pid = uniform_load(a.pages, (int64_t)p0 + pi);
    if (pid < 0 || pid >= a.num_pages) return;
    const int64_t off = (int64_t)pid * a.stride_page_b + (int64_t)kvh * a.stride_head_b;
    const int64_t src = ((int64_t)(t0 + kPage * pi) * a.Hkv + kvh) * D;
    const int64_t si = (int64_t)pid * a.Hkv + kvh;
    write_tile<D>(a, a.k + src, n, a.k_pool + off, a.kv_fp8 ? a.k_scale + si : nullptr, lane);
    write_tile<D>(a, a.v + src, n, a.v_pool + off, a.kv_fp8 ? a.v_scale + si : nullptr, lane);
}

static hipError_t launch_prefill_write(const PrefillLaunch &a, hipStream_t s) // (launch_prefill has seen that its workgroups can be counted)
{
    const int64_t blocks = (int64_t)((a.max_len + kPage - 1) / kPage) * a.num_prompts * a.Hkv;
    if (a.D == 128) hipLaunchKernelGGL(prefill_write_kernel<128>, dim3((unsigned)blocks), dim3(64), 0, s, a);
    else hipLaunchKernelGGL(prefill_write_kernel<64>, dim3((unsigned)blocks), dim3(64), 0, s, a);
    return hipGetLastError();
}

} // namespace ra
