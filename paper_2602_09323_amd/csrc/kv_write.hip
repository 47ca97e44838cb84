// Quantise-on-write of new K/V rows into the paged cache (Opt-KV: Eq. 5, Alg. 1 phase 1).
//
// One wavefront owns one (token, KV head) row: the 64 lanes hold the row's d elements (d/64 per
// lane), a butterfly max gives the row's absmax, and each lane encodes and stores its own
// elements.  Both tiles are stored in matrix-core operand order (see attn_tile.hpp), so a row is
// scattered in 16-byte (K) and 1-byte (V) pieces.  Write volume is a few hundred bytes per
// row, against kilobytes per token read by attention, so for a decode step's one token per sequence
// this kernel is latency-, not bandwidth-bound and is kept simple; calls with many tokens take the
// bulk kernel further down.
#include "kv_quant.hpp"
#include "launch_grid.hpp"

namespace coopt {

// Eq. 5's SkipSet as a bitmap over the call's token indices (NULL = empty).
__device__ __forceinline__ bool in_skip_set(const uint32_t* skip_set, int tok)
{
    return skip_set != nullptr && ((skip_set[tok >> 5] >> (tok & 31)) & 1u);
}

// scale_mode (see coopt_kv_cache_write_fp8_scaled): COOPT_SCALE_TOKEN = every row's own scale;
// COOPT_SCALE_STATIC = k_static[head] / v_static[head]; COOPT_SCALE_BLOCK = one scale for all rows
// of this call that land in the row's cache block (the largest of their absmaxes): the wavefront
// scans the call's slots for the others and takes their rows' absmax itself (every row of a block
// does the same scan -- this is the comparison scheme, not the method's).
template <int HEAD_DIM, int KV>
__global__ void __launch_bounds__(256)
kv_write_fp8_kernel(const half_t* __restrict__ k, const half_t* __restrict__ v,
                    const int64_t* __restrict__ slot_mapping,
                    const uint32_t* __restrict__ skip_set, int num_rows, int H_k,
                    uint8_t* __restrict__ k_cache, uint8_t* __restrict__ v_cache,
                    float* __restrict__ k_scale, float* __restrict__ v_scale, int scale_mode,
                    const float* __restrict__ k_static, const float* __restrict__ v_static)
{
    constexpr int E = HEAD_DIM / 64;
    const int row = blockIdx.x * 4 + (threadIdx.x >> 6);        // token * H_k + head
    if (row >= num_rows) return;
    const int tok = row / H_k, head = row - tok * H_k;
    const int lane = threadIdx.x & 63;
    // the rows are asked for together with the slot, not after it: one memory round trip
    float kx[E], vx[E];
    load_row_values<HEAD_DIM>(k + (size_t)row * HEAD_DIM, lane, kx);
    load_row_values<HEAD_DIM>(v + (size_t)row * HEAD_DIM, lane, vx);
    const int64_t slot = slot_mapping[tok];
    const bool skip = in_skip_set(skip_set, tok);
    if (slot < 0 || skip) return;                               // Eq. 5: filtered token
    const int64_t blk = slot / kBlock;
    const int off = (int)(slot - blk * kBlock);
    const size_t tile = (size_t)(blk * H_k + head);
    float k_given = 0.0f, v_given = 0.0f;                       // 0: the row's own scale
    if (scale_mode == COOPT_SCALE_STATIC) {
        k_given = k_static[head];
        v_given = v_static[head];
    } else if (scale_mode == COOPT_SCALE_BLOCK) {
        float ka = row_absmax<E>(kx), va = row_absmax<E>(vx);
        const int num_tokens = num_rows / H_k;
        for (int base = 0; base < num_tokens; base += 64) {
            const int t2 = base + lane;
            bool same = false;
            if (t2 < num_tokens && t2 != tok) {
                const int64_t s2 = slot_mapping[t2];
                same = s2 >= 0 && s2 / kBlock == blk && !in_skip_set(skip_set, t2);
            }
            unsigned long long todo = __builtin_amdgcn_ballot_w64(same);
            while (todo) {                                      // wave-uniform
                const int other = base + __builtin_ctzll(todo);
                todo &= todo - 1;
                float k2[E], v2[E];
                load_row_values<HEAD_DIM>(k + ((size_t)other * H_k + head) * HEAD_DIM, lane, k2);
                load_row_values<HEAD_DIM>(v + ((size_t)other * H_k + head) * HEAD_DIM, lane, v2);
                ka = fmaxf(ka, row_absmax<E>(k2));
                va = fmaxf(va, row_absmax<E>(v2));
            }
        }
        k_given = scale_of_absmax<KV>(ka);
        v_given = scale_of_absmax<KV>(va);
    }
    quantise_values_to_cache<HEAD_DIM, KV>(kx, vx, tile, off, lane, k_cache, v_cache, k_scale, v_scale,
                                           k_given, v_given);
}

// ---- bulk form (prefill chunks, cache fills): many tokens per call.
//
// The row-per-wavefront kernel above stores a row's V codes one by one (the V tile keeps four tokens
// of one dim side by side), which is fine for one token per sequence and slow for thousands.  A cache
// fill reads and writes each byte once and is bound by HBM if its stores are whole lines, so here a
// workgroup takes a window of consecutive tokens of one KV head:
//   * one 16-byte K chunk (16 dims of a one-byte cache, 8 of fp16) belongs to a lane, which asks for
//     its rows before anything depends on a slot, and stores its K chunk as it is;
//   * the V rows meet in LDS, from where every QUAD -- four consecutive tokens in four consecutive
//     slots from a multiple of four on -- leaves as whole 16-byte pieces of the V tile, one per lane,
//     256 bytes side by side per 16-dim group set;
//   * quads are found in the slots, not by the tokens' place in the call: in a batch of ragged
//     sequences most sequences start at a token index that is no multiple of four.  The quads whose
//     first token lies among a window's first kOwn tokens are the window's own, and the three rows
//     behind those (the overhang) are there to complete the last of them.
// A token outside any quad (skipped neighbours, scattered slots, ragged ends) is stored element by
// element from the registers.  Same arithmetic as the row kernel, hence the same bytes.
//
// The window is what 256 lanes hold at one chunk each: 16 rows (fp16, d = 128) to 64 (one byte,
// d = 64).  A window of 64 rows for every type, whose lanes took two to four chunks in turn, read less
// overhang but left calls of up to a few thousand rows with few wavefronts and a long chain: 64 tokens
// x 8 heads x 128 dims 4.4 us against 3.4 (fp16: 3.7 against 2.8), and in scattered slots, as a decode
// step of 64 sequences has them, 7.1 against 4.5 (fp16: 6.3 against 3.1).
//
// The stores are non-temporal wherever they come in runs: they pass the L2, where the rows' second
// readers find theirs, and what follows the call still finds its own data there.  A LARGE call's K stores
// are plain: a window's are pieces of 128 bytes, of which the L2 makes longer runs (kLargeWriteBytes has
// both sides; V pieces are 256 bytes and stay non-temporal: both plain 108.7 us where K alone takes 107.2
// and neither 128.2).  A token whose neighbours in
// the call are not its neighbours in the cache would pass the L2 in 16-byte pieces; its K stores are
// plain (16 384 tokens in random slots, fp16, 8 heads: 102 us non-temporal, 60 us so).

template <int HEAD_DIM, int KV>
struct BulkWindow {
    static constexpr int ES = kIsFp8<KV> ? 1 : 2;           // bytes per cache element
    static constexpr int CH = HEAD_DIM * ES / 16;           // 16-byte cache chunks, and lanes, per row
    static constexpr int kRows = 256 / CH;                  // rows a workgroup holds
    static constexpr int kOwn = kRows - 3;                  // ... of which this many are its own
    static constexpr int kRowTraffic = HEAD_DIM * (4 + 2 * ES) + (kIsFp8<KV> ? 8 : 0);    // bytes read and written
};

typedef unsigned int wu32x4 __attribute__((ext_vector_type(4)));

// max over the groups of CH neighbouring lanes (CH = 4 or 8), on the vector ALU
template <int CH>
__device__ __forceinline__ float group_max(float a)
{
    static_assert(CH == 4 || CH == 8, "DPP steps below");
    auto step = [&](auto ctrl) {
        const int v = __builtin_bit_cast(int, a);
        a = fmaxf(a, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(v, v, decltype(ctrl)::value, 0xf,
                                                                           0xf, false)));
    };
    step(std::integral_constant<int, 0xb1>{});                       // quad_perm: lane ^ 1
    step(std::integral_constant<int, 0x4e>{});                       // quad_perm: lane ^ 2
    if constexpr (CH == 8) step(std::integral_constant<int, 0x141>{});   // row_half_mirror: the other quad
    return a;
}

// 16 fp16 values (two 16-byte words) -> their group's scale and 16 one-byte codes, element e in byte e.
//
// The codes are defined through the correctly rounded quotient x / scale, one division per element:
// some ten instructions each, which kept a fill busier than its memory traffic.  With r = RN(1 / scale)
// (one division per row) and q0 = RN(x * r), the corrected q0 - RN(q0 * scale - x) * r is the correctly
// rounded quotient itself (Markstein's theorem, 1990: r correctly rounded, q0 within one unit in the
// last place; nothing here leaves the normal range), in three instructions.  tests/test_quotient.py
// compares it with division over every absmax and element that fp16 has.  The signs make a zero keep
// its sign, and an infinite scale (an infinity in the row) corrects by nothing: x * 0 is what x / infinity
// is.
template <int CH, int KV>
__device__ __forceinline__ wu32x4 quantise_chunk(wu32x4 lo, wu32x4 hi, float& scale)
{
    float x[16];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        // (through scalars: a bit cast taken straight from a vector element reads element 0)
        const uint32_t wl = lo[i], wh = hi[i];
        const half2_t a = __builtin_bit_cast(half2_t, wl), b = __builtin_bit_cast(half2_t, wh);
        x[2 * i] = (float)a[0];
        x[2 * i + 1] = (float)a[1];
        x[8 + 2 * i] = (float)b[0];
        x[8 + 2 * i + 1] = (float)b[1];
    }
    float amax = 0.0f;
#pragma unroll
    for (int e = 0; e < 16; ++e) amax = fmaxf(amax, fabsf(x[e]));
    amax = group_max<CH>(amax);
    scale = scale_of_absmax<KV>(amax);
    const float r = __fdiv_rn(1.0f, scale), minus_r = -r;
    const float s = scale == INFINITY ? 0.0f : scale;
    wu32x4 codes;
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        float y[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float q0 = x[4 * d + e] * r;
            const float off = __builtin_fmaf(q0, s, -x[4 * d + e]);
            y[e] = fminf(fmaxf(__builtin_fmaf(off, minus_r, q0), -kFp8Max<KV>), kFp8Max<KV>);
        }
        int w;
        if constexpr (KV == COOPT_KV_E5M2) {
            w = __builtin_amdgcn_cvt_pk_bf8_f32(y[0], y[1], 0, false);
            w = __builtin_amdgcn_cvt_pk_bf8_f32(y[2], y[3], w, true);
        } else {
            w = __builtin_amdgcn_cvt_pk_fp8_f32(y[0], y[1], 0, false);
            w = __builtin_amdgcn_cvt_pk_fp8_f32(y[2], y[3], w, true);
        }
        codes[d] = (uint32_t)w;
    }
    return codes;
}

template <int HEAD_DIM, int KV, bool LARGE>
__global__ void __launch_bounds__(256)
kv_write_bulk_kernel(const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
                     const int64_t* __restrict__ slot_mapping, const uint32_t* __restrict__ skip_set,
                     int num_tokens, int H_k, uint8_t* __restrict__ k_cache,
                     uint8_t* __restrict__ v_cache, float* __restrict__ k_scale,
                     float* __restrict__ v_scale)
{
    using W = BulkWindow<HEAD_DIM, KV>;
    constexpr bool FP8 = kIsFp8<KV>;
    constexpr int ES = W::ES, CH = W::CH;
    constexpr int DPL = 16 / ES;                // dims per lane: one 16-byte cache chunk
    constexpr int NW = FP8 ? 2 : 1;             // 16-byte words of fp16 that those are
    constexpr int CW = CH < 8 ? CH : 8;         // chunks of a row side by side in a wavefront
    constexpr int RB = HEAD_DIM * ES + 16;      // a staged V row, skewed so that quads differ in bank
    __shared__ __attribute__((aligned(16))) unsigned char rows[W::kRows * RB];
    __shared__ int64_t slots[W::kRows + 6];     // of rows -3 .. kRows+2 (-1: no token, or filtered)

    const int tid = threadIdx.x;
    const int window = blockIdx.x / H_k, head = blockIdx.x - window * H_k;
    const int base = window * W::kOwn;
    // a wavefront's lanes cover 8 rows or more: a K chunk of 8 consecutive tokens is a whole line
    const int wave = tid >> 6;
    const int c = tid % CW + CW * (wave % (CH / CW));
    const int r = (tid & 63) / CW + (64 / CW) * (wave / (CH / CW));
    if (tid < W::kRows + 6) {
        const int tok = base - 3 + tid;
        int64_t s = -1;
        if (tid < W::kRows + 3 && tok >= 0 && tok < num_tokens && !in_skip_set(skip_set, tok))   // Eq. 5
            s = slot_mapping[tok];
        slots[tid] = s;
    }
    wu32x4 kx[NW], vx[NW];
    const size_t at = ((size_t)min(base + r, num_tokens - 1) * H_k + head) * HEAD_DIM + DPL * c;
#pragma unroll
    for (int i = 0; i < NW; ++i) {
        kx[i] = reinterpret_cast<const wu32x4*>(k + at)[i];
        vx[i] = reinterpret_cast<const wu32x4*>(v + at)[i];
    }
    __syncthreads();

    // is row r's token one of a quad?  The first token's row then is r - (its slot & 3).
    auto in_quad = [&](int r, int64_t slot) {
        const int j = (int)(slot & 3);
        bool full = slot >= 0;
#pragma unroll
        for (int m = 0; m < 4; ++m) full = full && slots[r + 3 - j + m] == slot - j + m;
        return full;
    };
    const int64_t slot = slots[r + 3];
    const bool mine = slot >= 0 && r < W::kOwn;
    const bool quad = in_quad(r, slot);
    const bool alone = slots[r + 2] != slot - 1 && slots[r + 4] != slot + 1;     // (never in a quad)
    float ks = 0.0f, vs = 0.0f;
    wu32x4 kc, vc;
    if constexpr (FP8) {
        kc = quantise_chunk<CH, KV>(kx[0], kx[1], ks);
        vc = quantise_chunk<CH, KV>(vx[0], vx[1], vs);
    } else {
        kc = kx[0];
        vc = vx[0];
    }
    *reinterpret_cast<wu32x4*>(rows + r * RB + 16 * c) = vc;
    const int64_t blk = slot / kBlock;
    const int off = (int)(slot - blk * kBlock);
    const size_t tile = (size_t)(blk * H_k + head);
    // K tile [chunks][16 tokens][16 bytes]
    wu32x4* kdst = reinterpret_cast<wu32x4*>(k_cache + tile * (kBlock * HEAD_DIM * ES) + (c * kBlock + off) * 16);
    if (mine) {
        if (FP8 && c == 0) {
            k_scale[tile * kBlock + off] = ks;
            v_scale[tile * kBlock + off] = vs;
        }
        if (!quad) {
            if (alone) *kdst = kc;
            uint8_t* vtile = v_cache + tile * (kBlock * HEAD_DIM * ES);
#pragma unroll
            for (int n = 0; n < DPL; ++n) {
                if constexpr (FP8)
                    vtile[v_tile_index<1>(off, DPL * c + n)] = (uint8_t)(vc[n >> 2] >> (8 * (n & 3)));
                else
                    reinterpret_cast<uint16_t*>(vtile)[v_tile_index<2>(off, DPL * c + n)] =
                        (uint16_t)(vc[n >> 1] >> (16 * (n & 1)));
            }
        }
    }
    __syncthreads();
    // (here, behind the barrier: in the other arm of the plain store the compiler makes one plain
    // store of the two)
    if (mine && !alone) {
        if constexpr (LARGE) *kdst = kc;
        else __builtin_nontemporal_store(kc, kdst);
    }

    // ---- V quads.  Their first tokens are at least four rows apart: at most one in rows 4b .. 4b+3.
    // Sixteen lanes (n) take one 64-byte piece (cq) per token of the quad of one b; four neighbouring
    // quads of a block are 1 KB.
    const int n = tid & 15, b = (tid >> 4) % (W::kRows / 4), cq = tid / (4 * W::kRows);
    int lead = -1;
    int64_t slot0 = 0;
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        const int rr = 4 * b + m;
        const int64_t s = slots[rr + 3];
        if ((s & 3) == 0 && rr < W::kOwn && in_quad(rr, s)) {
            lead = rr;
            slot0 = s;
        }
    }
    if (lead < 0) return;
    const int64_t vblk = slot0 / kBlock;
    const int tq = (int)(slot0 - vblk * kBlock) >> 2;
    uint8_t* vtile = v_cache + (size_t)(vblk * H_k + head) * (kBlock * HEAD_DIM * ES);
    const unsigned char* src = rows + lead * RB + (n & ~(4 / ES - 1)) * ES;
    // the element's place inside the aligned dword that holds it picks the shuffle's selector
    const uint32_t e = (uint32_t)(n & (4 / ES - 1));
    const uint32_t sel_lo = FP8 ? (0x0c0c0000u | ((4u + e) << 8) | e) : (e ? 0x07060302u : 0x05040100u);
    const uint32_t sel_hi = FP8 ? (0x00000c0cu | ((4u + e) << 24) | (e << 16)) : sel_lo;
    wu32x4 out;
#pragma unroll
    for (int cc = 0; cc < 4 / ES; ++cc) {
        const int at = 16 * ES * (cq * (4 / ES) + cc);
        uint32_t d[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) d[t] = *reinterpret_cast<const uint32_t*>(src + t * RB + at);
        const uint32_t lo = __builtin_amdgcn_perm(d[1], d[0], sel_lo);
        const uint32_t hi = __builtin_amdgcn_perm(d[3], d[2], sel_hi);
        if constexpr (FP8) {
            out[cc] = lo | hi;
        } else {
            out[2 * cc] = lo;
            out[2 * cc + 1] = hi;
        }
    }
    __builtin_nontemporal_store(out, reinterpret_cast<wu32x4*>(vtile + ((cq * 4 + tq) * 16 + n) * 16));
}

template <int HEAD_DIM>
__global__ void __launch_bounds__(256)
kv_write_fp16_kernel(const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
                     const int64_t* __restrict__ slot_mapping,
                     const uint32_t* __restrict__ skip_set, int num_rows, int H_k,
                     uint16_t* __restrict__ k_cache, uint16_t* __restrict__ v_cache)
{
    constexpr int E = HEAD_DIM / 64;
    const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= num_rows) return;
    const int tok = row / H_k, head = row - tok * H_k;
    const int64_t slot = slot_mapping[tok];
    if (slot < 0 || in_skip_set(skip_set, tok)) return;
    const int64_t blk = slot / kBlock;
    const int off = (int)(slot - blk * kBlock);
    const int lane = threadIdx.x & 63;
    const size_t tile = (size_t)(blk * H_k + head);
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int dim = lane * E + e;
        k_cache[tile * (kBlock * HEAD_DIM) + k_tile_index<2>(off, dim)] = k[(size_t)row * HEAD_DIM + dim];
        v_cache[tile * (kBlock * HEAD_DIM) + v_tile_index<2>(off, dim)] = v[(size_t)row * HEAD_DIM + dim];
    }
}

}  // namespace coopt

using namespace coopt;

// From this many bytes read and written on, a bulk call's K stores go through the L2.  us, past it / through
// it, to buffers that are new to the caches:
//              62-75 MB      83-88         100           125-134       150-167       201-268       402-536
//   E4M3 128   15.7 / 16.2   20.3 / 20.3   24.5 / 23.5   29.4 / 28.6   32.8 / 32.0   46.2 / 43.8   91.3 / 84.4
//   E4M3 64    19.6 / 20.5                 24.2 / 25.4   29.3 / 30.2   34.8 / 35.5   48.0 / 47.9   93.9 / 92.6
//   fp16 128   14.3 / 16.1   19.5 / 19.4   22.8 / 22.3   32.8 / 29.5   39.9 / 36.1   64.4 / 56.0   128.2 / 107.2
//   fp16 64    14.3 / 16.6                 23.5 / 23.4   32.8 / 30.7
template <int HEAD_DIM, int KV>
constexpr long long kLargeWriteBytes = kIsFp8<KV> && HEAD_DIM == 64 ? 200000000 : 120000000;

// The bulk kernel: from this many tokens per call on, and from as many rows (tokens times heads) as keep
// one wavefront a row from being the faster form, whatever the slots (a decode step of a large batch has
// scattered ones).  us, bulk / a wavefront per row, 8 heads x 128 dims:
//              64 tokens, run   scattered   256, run    scattered    512, run    scattered
//   E4M3       3.4 / 2.5        4.4 / 2.5   3.4 / 2.9   4.8 / 2.9    3.5 / 3.8   5.2 / 3.9
//   fp16       2.8 / 2.1        3.0 / 2.1   2.7 / 2.9   3.7 / 2.8    3.0 / 4.0   5.4 / 3.9
// and 40 heads: E4M3 64 tokens 3.5 / 3.3 and 4.9 / 3.2, 96 tokens 3.6 / 3.8 and 5.1 / 3.8; fp16 64 tokens
// 3.0 / 3.2 and 3.9 / 3.1; 128 tokens of 8 heads 2.8 / 2.3 and 3.2 / 2.3.  64 dims, whose rows are half as
// long, at both ends of the line: E4M3, 8 heads 64 tokens 3.6 / 2.7 and 4.8 / 2.7, 320 tokens 3.6 / 3.1 and 4.9 / 3.1; fp16
// 64 tokens 2.9 / 2.3 and 3.2 / 2.3, 192 tokens 2.9 / 2.5 and 3.4 / 2.5.
constexpr int kBulkWriteTokens = 64;
template <int KV> constexpr long long kRowWriteRows = kIsFp8<KV> ? 2560 : 1536;
template <int KV>
static bool takes_bulk(int32_t num_tokens, long long rows)
{
    return num_tokens >= kBulkWriteTokens && rows > kRowWriteRows<KV>;
}

template <int HEAD_DIM, int KV>
static void launch_write_bulk(const void* k, const void* v, const int64_t* slot_mapping,
                              const uint32_t* skip_set, int32_t num_tokens, int H_k, uint8_t* k_cache,
                              uint8_t* v_cache, float* k_scale, float* v_scale, hipStream_t stream)
{
    constexpr int kOwn = BulkWindow<HEAD_DIM, KV>::kOwn;
    const long long step = tokens_per_launch(num_tokens, kOwn, H_k);
    const auto kernel = (long long)num_tokens * H_k * BulkWindow<HEAD_DIM, KV>::kRowTraffic >= kLargeWriteBytes<HEAD_DIM, KV>
                            ? kv_write_bulk_kernel<HEAD_DIM, KV, true> : kv_write_bulk_kernel<HEAD_DIM, KV, false>;
    for (long long first = 0; first < num_tokens; first += step) {
        const int n = (int)(step < num_tokens - first ? step : num_tokens - first);
        const size_t at = (size_t)first * H_k * HEAD_DIM;
        // one workgroup per window and head
        hipLaunchKernelGGL(kernel, dim3((unsigned)((n - 1) / kOwn + 1) * H_k), dim3(256), 0,
                           stream, (const uint16_t*)k + at, (const uint16_t*)v + at, slot_mapping + first,
                           skip_set ? skip_set + first / 32 : nullptr, n, H_k, k_cache, v_cache, k_scale, v_scale);
    }
}

template <int HEAD_DIM, int KV>
static void launch_write_fp8(const void* k, const void* v, const int64_t* slot_mapping,
                             const uint32_t* skip_set, int32_t num_tokens, uint8_t* k_cache,
                             uint8_t* v_cache, float* k_scale, float* v_scale, int scale_mode,
                             const float* k_static, const float* v_static, int H_k,
                             hipStream_t stream)
{
    const dim3 block(256);
    const long long rows = (long long)num_tokens * H_k;
    if (takes_bulk<KV>(num_tokens, rows) && scale_mode == COOPT_SCALE_TOKEN) {
        launch_write_bulk<HEAD_DIM, KV>(k, v, slot_mapping, skip_set, num_tokens, H_k, k_cache, v_cache,
                                        k_scale, v_scale, stream);
        return;
    }
    const dim3 grid((unsigned)((rows + 3) / 4));
    hipLaunchKernelGGL((kv_write_fp8_kernel<HEAD_DIM, KV>), grid, block, 0, stream, (const half_t*)k,
                       (const half_t*)v, slot_mapping, skip_set, (int)rows, H_k, k_cache, v_cache,
                       k_scale, v_scale, scale_mode, k_static, v_static);
}

static int write_fp8(const void* k, const void* v, const int64_t* slot_mapping,
                     const uint32_t* skip_set, int32_t num_tokens, uint8_t* k_cache,
                     uint8_t* v_cache, float* k_scale, float* v_scale, int scale_mode,
                     const float* k_static, const float* v_static, const coopt_shape* shape,
                     void* hip_stream)
{
    int st = check_shape(shape);
    if (st != COOPT_OK) return st;
    if ((shape->kv_dtype != COOPT_KV_E4M3 && shape->kv_dtype != COOPT_KV_E5M2) || num_tokens < 0)
        return COOPT_ERR_SHAPE;
    if (scale_mode != COOPT_SCALE_TOKEN && scale_mode != COOPT_SCALE_BLOCK &&
        scale_mode != COOPT_SCALE_STATIC)
        return COOPT_ERR_SHAPE;
    if (num_tokens == 0) return COOPT_OK;
    if (!k || !v || !slot_mapping || !k_cache || !v_cache || !k_scale || !v_scale)
        return COOPT_ERR_NULL;
    if (scale_mode == COOPT_SCALE_STATIC && (!k_static || !v_static)) return COOPT_ERR_NULL;
    const long long rows = (long long)num_tokens * shape->num_kv_heads;
    if (rows > 0x7fffffffLL) return COOPT_ERR_SHAPE;
    hipStream_t stream = (hipStream_t)hip_stream;
    const int H_k = shape->num_kv_heads;
#define COOPT_WRITE(D, KV)                                                                          \
    launch_write_fp8<D, KV>(k, v, slot_mapping, skip_set, num_tokens, k_cache, v_cache, k_scale,    \
                            v_scale, scale_mode, k_static, v_static, H_k, stream)
    if (shape->kv_dtype == COOPT_KV_E5M2) {
        if (shape->head_dim == 128) COOPT_WRITE(128, COOPT_KV_E5M2);
        else COOPT_WRITE(64, COOPT_KV_E5M2);
    } else {
        if (shape->head_dim == 128) COOPT_WRITE(128, COOPT_KV_E4M3);
        else COOPT_WRITE(64, COOPT_KV_E4M3);
    }
#undef COOPT_WRITE
    return launch_status();
}

static int write_fp16(const void* k, const void* v, const int64_t* slot_mapping,
                      const uint32_t* skip_set, int32_t num_tokens, void* k_cache, void* v_cache,
                      const coopt_shape* shape, void* hip_stream)
{
    int st = check_shape(shape);
    if (st != COOPT_OK) return st;
    if (shape->kv_dtype != COOPT_KV_FP16 || num_tokens < 0) return COOPT_ERR_SHAPE;
    if (num_tokens == 0) return COOPT_OK;
    if (!k || !v || !slot_mapping || !k_cache || !v_cache) return COOPT_ERR_NULL;
    const long long rows = (long long)num_tokens * shape->num_kv_heads;
    if (rows > 0x7fffffffLL) return COOPT_ERR_SHAPE;
    hipStream_t stream = (hipStream_t)hip_stream;
    const dim3 block(256);
    if (takes_bulk<COOPT_KV_FP16>(num_tokens, rows)) {
        if (shape->head_dim == 128)
            launch_write_bulk<128, COOPT_KV_FP16>(k, v, slot_mapping, skip_set, num_tokens,
                                                  shape->num_kv_heads, (uint8_t*)k_cache, (uint8_t*)v_cache,
                                                  nullptr, nullptr, stream);
        else
            launch_write_bulk<64, COOPT_KV_FP16>(k, v, slot_mapping, skip_set, num_tokens,
                                                 shape->num_kv_heads, (uint8_t*)k_cache, (uint8_t*)v_cache,
                                                 nullptr, nullptr, stream);
        return launch_status();
    }
    const dim3 grid((unsigned)((rows + 3) / 4));
    if (shape->head_dim == 128)
        hipLaunchKernelGGL(kv_write_fp16_kernel<128>, grid, block, 0, stream, (const uint16_t*)k,
                           (const uint16_t*)v, slot_mapping, skip_set, (int)rows,
                           shape->num_kv_heads, (uint16_t*)k_cache, (uint16_t*)v_cache);
    else
        hipLaunchKernelGGL(kv_write_fp16_kernel<64>, grid, block, 0, stream, (const uint16_t*)k,
                           (const uint16_t*)v, slot_mapping, skip_set, (int)rows,
                           shape->num_kv_heads, (uint16_t*)k_cache, (uint16_t*)v_cache);
    return launch_status();
}

extern "C" int coopt_kv_cache_write_fp8(const void* k, const void* v, const int64_t* slot_mapping,
                                        int32_t num_tokens, uint8_t* k_cache, uint8_t* v_cache,
                                        float* k_scale, float* v_scale, const coopt_shape* shape,
                                        void* hip_stream)
{
    return write_fp8(k, v, slot_mapping, nullptr, num_tokens, k_cache, v_cache, k_scale, v_scale,
                     COOPT_SCALE_TOKEN, nullptr, nullptr, shape, hip_stream);
}

extern "C" int coopt_kv_cache_write_fp8_scaled(const void* k, const void* v,
                                               const int64_t* slot_mapping, int32_t num_tokens,
                                               uint8_t* k_cache, uint8_t* v_cache, float* k_scale,
                                               float* v_scale, int32_t scale_mode,
                                               const float* k_static, const float* v_static,
                                               const coopt_shape* shape, void* hip_stream)
{
    return write_fp8(k, v, slot_mapping, nullptr, num_tokens, k_cache, v_cache, k_scale, v_scale,
                     scale_mode, k_static, v_static, shape, hip_stream);
}

extern "C" int coopt_kv_cache_write_fp16(const void* k, const void* v, const int64_t* slot_mapping,
                                         int32_t num_tokens, void* k_cache, void* v_cache,
                                         const coopt_shape* shape, void* hip_stream)
{
    return write_fp16(k, v, slot_mapping, nullptr, num_tokens, k_cache, v_cache, shape, hip_stream);
}

extern "C" int coopt_kv_cache_write_skipset(const void* k, const void* v,
                                            const int64_t* slot_mapping, const uint32_t* skip_set,
                                            int32_t num_tokens, void* k_cache, void* v_cache,
                                            float* k_scale, float* v_scale,
                                            const coopt_shape* shape, void* hip_stream)
{
    if (shape && shape->kv_dtype == COOPT_KV_FP16)
        return write_fp16(k, v, slot_mapping, skip_set, num_tokens, k_cache, v_cache, shape, hip_stream);
    return write_fp8(k, v, slot_mapping, skip_set, num_tokens, (uint8_t*)k_cache, (uint8_t*)v_cache,
                     k_scale, v_scale, COOPT_SCALE_TOKEN, nullptr, nullptr, shape, hip_stream);
}
