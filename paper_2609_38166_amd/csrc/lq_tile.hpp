// Device code of the whole-tile kernels (quantize, commit, dequantize), shared by
// their launches and by the decode step fused with the commit.
// Whole-tile kernels: quantize a given state, commit a window, dequantize.
//
// One 256-thread workgroup (4 waves) owns one 128 x 128 tile held in registers: wave w
// owns key channels 32 w .. 32 w + 31, and lane (row j, i) of it the 8 x 8 block
// M[32 w + 8 j + a][16 b + i] of the state in paper orientation (row = key channel).  A
// sum over value channels stays inside a 16-lane row; a sum over key channels crosses
// the wave's rows in registers and the waves through LDS: one barrier per power sweep.  A
// vector over key channels never leaves its wave.  Three workgroups share a CU (168 VGPRs
// per lane, 47 KiB of LDS each; two with the BF16 state): the 128 registers of the fp64
// block leave 40 for everything else, so the code below keeps few values live across
// phases (lane coordinates re-derived where used, the next pass's records copied
// straight into LDS).
//
// Memory.  The block's 16 neighbouring lanes hold 16 value rows, and an instruction that
// loaded or stored as they hold it would touch 64 pieces of lines; states (and the BF16
// state's codes) are therefore turned in LDS, each wave its own part, and move in whole
// lines.  Codes of 8 bits and less are stored as held, 8 bytes a lane: turning them too
// costs more than it gives where memory is the bound (quantize of 8192 states without
// tokens 123 -> 129 us).
//
// What bounds it: fp64 issue, and in the sweeps the LDS transposes and the barrier
// beside it.  A sweep is 128 FMA per lane (0.25 us per tile and CU at the 2.07 GHz that
// the card holds under them); it takes 0.41 us with three workgroups per CU (quantize of
// 2048 states, 5 sweeps against 4) and 0.68 us with one (32 states).  Measured at r = 8, 4
// sweeps against a layout with a thread's block in a row of key blocks, two barriers and
// five LDS round trips a sweep: quantize 49.1 -> 36.9 us for 32 tiles, 212 -> 181 us for
// 2048; commit of 64 records (per-channel gate) 72.3 -> 51.7 us for 32 tiles, 320 -> 269 us
// for 2048, 1192 -> 1000 us for 8192 (out of cache).
//
// The rank-one terms of the reconstruction (records, Compensator Tokens) go through the
// fp64 matrix cores, v_mfma_f64_16x16x4: 77.8 TFLOP/s in a loop of nothing else (with its
// accumulators in VGPRs; copied to AGPRs and back they reach 47) against the vector
// unit's 67.8, one instruction for every 16 FMA, and ten LDS reads for a wave's 16 products
// of four records instead of nine reads for every 64 FMA of one.  Its accumulators are the
// 8 x 8 blocks (the operand rows are permuted to make them so).
//
//   commit   : reconstruct S_p = Gamma_{1:p}[C dequant(Z) + K~ U~^T]
//              + sum_j Gamma_{j+1:p} k~_j u_j^T  (Sec. 3.4 Eq. (smooth)),
//              then quantize it and reset the window (Sec. 3.3: the old
//              tokens are discarded and refitted);
//   quantize : load a given fp32 state and quantize it;
//   dequant  : reconstruct and write the fp32 state.
//
// Quantization (Sec. 3.3 Eq. (compensator-rank-r), Sec. 3.4, App. B.3): r
// Compensator Tokens fitted one after another by power iteration on the
// deflated residual (start: key-row l2 norms; each sweep y = M^T x, x = M y;
// the direction is normalised), each rounded to FP16 before it is
// subtracted; then the smoothing scales c_k = sqrt(max(mean_v |R_kv|, 1e-12)), the per-value-channel scale
// delta_v = max_k |R_kv / c_k| / qmax and the codes.
//
// Precision: the tile, the fit and the smoothing statistic are carried in
// fp64 (gfx950 runs fp64 FMA at the rate of unpacked fp32).  Each token is
// rounded to FP16 before it is deflated, so an fp32-level difference in the
// fit would flip a rounding and move every later token and the codes of whole
// rows; in fp64 the discrete decisions (FP16 tokens, fp32 scales, codes) are
// reproducible by any exact-enough implementation.  The code decision itself
// is taken in fp32 on the fp32-rounded residual.
#pragma once

#include "lq_device.hpp"
#include "lq_internal.hpp"

#include <limits.h>
#include <stddef.h>

namespace lq {

namespace {

constexpr int TCH = 8;      // records staged per pass
constexpr int TT = 256;     // threads per tile
constexpr int NW = TT / 64; // waves: each owns 32 key channels
constexpr int VPT = 8;      // value channels per thread

// The 8 codes of row v (value channel), key channels 8kb..8kb+7: 8 bytes for
// the byte formats, 4 for INT4, 6 (three 16-bit words) for INT6, 16 (eight
// BF16 values) for the BF16 state.
template <int CODE> struct Codes8 { typedef uint2 type; };
template <> struct Codes8<4> { typedef uint4 type; };

// Value a (0..7) of the 8 codes as a double (BF16 state: the value itself).
template <int CODE>
__device__ __forceinline__ double code8_value(const typename Codes8<CODE>::type &z, int a) {
    if constexpr (CODE == 4) {
        const uint32_t x = a < 2 ? z.x : a < 4 ? z.y : a < 6 ? z.z : z.w;
        return (double)bf2f((uint16_t)(x >> (16 * (a & 1))));
    } else {
        const uint32_t w[2] = {z.x, z.y};
        if (CODE == 0) return (double)sfield(w[a >> 2], 8 * (a & 3), 8);
        if (CODE == 2) return (double)sfield(w[0], 4 * a, 4);
        return (double)code_at<CODE>(w, a);
    }
}

template <int CODE>
__device__ __forceinline__ void store_codes8(uint8_t *codes, int tile, int v, int kb, uint2 w) {
    constexpr int ROW = D * CodeFmt<CODE>::BITS / 8;
    uint8_t *p = codes + ((size_t)tile * D + v) * ROW + kb * CodeFmt<CODE>::BITS;
    if (CODE <= 1) {
        *(uint2 *)p = w;
    } else if (CODE == 2) {
        *(uint32_t *)p = w.x;
    } else {
        // INT6: the row's four key blocks of a wave (lanes 16 apart) are 24 bytes, 8-byte
        // aligned: the first three lanes store 8 of them each, their own and the next
        // one's.  (Against three stores of 2 bytes from each lane: one state without tokens
        // 5.34 -> 4.63 us, 8192 states 130 -> 122.)
        const int j = kb & 3;
        const uint64_t own = w.x | ((uint64_t)w.y << 32);
        const uint64_t next = (uint32_t)__shfl_down((int)w.x, 16) | ((uint64_t)(uint32_t)__shfl_down((int)w.y, 16) << 32);
        if (j < 3) *(uint64_t *)(p + 2 * j) = (own >> (16 * j)) | (next << (48 - 16 * j));
    }
}

typedef double v4d __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

struct TileArgs {
    uint8_t *codes;
    float *scale;
    float *smooth;
    uint16_t *comp_k;
    uint16_t *comp_u;
    const uint16_t *rec_k;
    const uint16_t *rec_u;
    const uint16_t *rec_a;
    int32_t *rec_len;
    int32_t *err;
    const float *S_in;
    float *S_out;
    const int32_t *mask;
    int heads_v;
    int window;
    int n_comp;
    int power_iters;
    int smooth_on;
};

// Workgroups per CU: three (166 VGPRs, 47 KiB of LDS).  The BF16 state's 32 KiB of codes
// lie in LDS as a whole, so two.
template <int CODE> struct TileOcc { static constexpr int value = IsBF16<CODE>::value ? 2 : 3; };

template <int CODE>
struct TileShared {
    union {
        struct {                            // reconstruction
            double key[NW][TCH][32];        // a wave's record keys, decay folded in
            double val[2][TCH][D];          // record values, two passes in turn
            uint4 raw_ka[NW][64];           // copied records: a wave's keys, then decays
            uint4 raw_u[NW][32];            // two records' values of each wave
            uint4 codes[D * D * CodeFmt<CODE>::BITS / 128];    // rows rotated by v & 15 chunks
            float scale[D];
            float smooth[D];
        };
        struct {                            // fit
            double part[2][NW][D];          // per-wave partials of a sum over key channels, two in turn
            double nrm[2][NW];              // per-wave partial squared norms
            int ex[2][NW];                  // per-wave largest exponent of a squared row norm
            double vec[NW][D];              // a wave's copy of a summed vector (order below)
            double red[TT / 16][8 * 17];    // row-private transposes of a sum over value channels
        };
    };
};

// Order of a value vector in LDS: channel v = 16 (2 q + e) + i at 32 q + 2 i + e, so
// the 16 lanes of a row that read pair q of their block touch 256 consecutive
// bytes, and lane (row j, i) of a wave that holds pair j sits at 2 * lane.

// 16 value rows of a wave's part of an fp32 state (32 key channels, 128 bytes a row) in
// its own LDS, to turn them between memory's order and the block's: chunk c (16 bytes)
// of row q lies at 8 q + (c ^ (q & 7)).  Lane L of memory's order has chunk L & 7 of row
// L >> 3 (and of row 8 + (L >> 3), 64 chunks on); lane (row j, i) of the block chunks 2 j
// and 2 j + 1 of row i.  Neither order meets a bank twice in 8 lanes.
__device__ __forceinline__ constexpr int TURN_ROWS(int lane) { return (lane & 56) + ((lane & 7) ^ (lane >> 3)); }
__device__ __forceinline__ constexpr int TURN_BLOCK(int q, int c) { return 8 * q + (c ^ (q & 7)); }

// Sum over key channels of v[b] (b = 0..7: this thread's value channels, its 8
// key channels added up): over the wave's 4 rows by cross-row swaps, over the
// 4 waves through LDS.  One barrier; `buf` alternates between calls, so a
// call's writes meet only reads that the previous call's barrier has ended.
// Lane (row j, i) receives channels 32 j + i and 32 j + 16 + i (b = 2 j, 2 j + 1).
template <typename Shared>
__device__ __forceinline__ double2 sum_keys(Shared &sh, const double *v, int buf, int tid) {
    const int lane = tid & 63, w = tid >> 6;
    double s0, s1;
    rows4_reduce_scatter(v, s0, s1);
    *(double2 *)&sh.part[buf][w][2 * lane] = make_double2(s0, s1);
    __syncthreads();
    double2 p[NW];
#pragma unroll
    for (int x = 0; x < NW; ++x) p[x] = *(const double2 *)&sh.part[buf][x][2 * lane];
    return make_double2((p[0].x + p[1].x) + (p[2].x + p[3].x), (p[0].y + p[1].y) + (p[2].y + p[3].y));
}

// The lane's pair of a value vector to every lane of the wave: v[b] = channel
// 16 b + i (through the wave's own LDS copy; no barrier).
template <typename Shared>
__device__ __forceinline__ void share_pairs(Shared &sh, double2 t, double *v, int tid) {
    const int lane = tid & 63, w = tid >> 6, i = lane & 15;
    __builtin_amdgcn_wave_barrier();
    *(double2 *)&sh.vec[w][2 * lane] = t;
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const double2 y = *(const double2 *)&sh.vec[w][32 * q + 2 * i];
        v[2 * q] = y.x;
        v[2 * q + 1] = y.y;
    }
    __builtin_amdgcn_wave_barrier();
}

// Sum over value channels of part(a) (a = 0..7: this thread's key channels, its 8
// value channels added up) over the 16 lanes of its row, which lie in one
// wave: a row-private LDS transpose, no barrier.  Lane i receives key channel
// i & 7.  Channels are 17 words apart: neither the writes (16 lanes of one
// channel) nor the reads (lane (c, h): 8 lanes of channel c) share a bank.  A
// partial is stored as soon as it is made, so that the stores run beside the
// next one's arithmetic (4% off a commit and 6% off a quantization against
// storing the eight together).
template <typename Shared, typename F>
__device__ __forceinline__ double sum_values(Shared &sh, F part, int tid) {
    const int i = tid & 15, c = i & 7, h = i >> 3;
    double *r = sh.red[tid >> 4];
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int a = 0; a < 8; ++a) {
        r[17 * a + i] = part(a);
        __builtin_amdgcn_sched_barrier(0);
    }
    __builtin_amdgcn_wave_barrier();
    double s[8];
#pragma unroll
    for (int l = 0; l < 8; ++l) s[l] = r[17 * c + 8 * h + l];
    __builtin_amdgcn_wave_barrier();
    const double z = ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7]));
    return z + dpp<DPP_ROR8>(z);
}

// The value of lane a (0..7, a constant once unrolled) of the row: key channel a
// of the thread's block.
template <typename T>
__device__ __forceinline__ T row_lane(T z, int a) {
    switch (a) {
        case 0: return row_bcast<0>(z);
        case 1: return row_bcast<1>(z);
        case 2: return row_bcast<2>(z);
        case 3: return row_bcast<3>(z);
        case 4: return row_bcast<4>(z);
        case 5: return row_bcast<5>(z);
        case 6: return row_bcast<6>(z);
        default: return row_bcast<7>(z);
    }
}

// Sum over the wave of z, which lanes i and i + 8 of a row both hold.
__device__ __forceinline__ double wave_sum_half(double z) {
    z += dpp<DPP_XOR1>(z);
    z += dpp<DPP_XOR2>(z);
    z += dpp<DPP_HALF_MIRROR>(z);
    double a, b;
    swap32_d(z, z, a, b);
    z = a + b;
    swap16_d(z, z, a, b);
    return a + b;
}

template <typename Shared>
__device__ __forceinline__ double sum_nrm(const Shared &sh, int buf) {
    return (sh.nrm[buf][0] + sh.nrm[buf][1]) + (sh.nrm[buf][2] + sh.nrm[buf][3]);
}

template <int N>
__device__ __forceinline__ void wait_vm() { asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory"); }

// The whole-tile work of one workgroup.  p_given >= 0 (window commit only)
// is the number of buffered records, taken instead of the tile's rec_len and
// without the request mask: the decode step fused with the commit passes the
// count it has just made.
template <int GATE, int CODE, int MODE>
__device__ __forceinline__ void tile_body(const TileArgs &A, TileShared<CODE> &sh, int tile, int p_given) {
    // lane coordinates: column i and row j in the wave, key block kb, wave w; re-derived from
    // an opaque thread index at phase boundaries, so that the compiler recomputes
    // the addresses built from them instead of holding them across phases
    int tid = threadIdx.x, i = tid & 15, j = (tid >> 4) & 3, kb = tid >> 4;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    auto refresh = [&]() {
        int t = (int)threadIdx.x;
        asm volatile("" : "+v"(t));
        tid = t;
        i = t & 15;
        j = (t >> 4) & 3;
        kb = t >> 4;                                // key block of 8 channels (4 w + j)
    };
    const size_t tvec = (size_t)tile * D;
    const int r = A.n_comp;

    if constexpr (IsBF16<CODE>::value && MODE == TILE_QUANTIZE) {
        // the BF16 state has no tokens, scales or smoothing: every entry rounded where it is
        // (through the block and its turns one state took 4.18 us, this 2.46; 2048 states 37.3 and 34.5)
        const v4f *S = (const v4f *)(A.S_in + (size_t)tile * D * D) + 2 * tid;
        uint4 *to = (uint4 *)(A.codes + (size_t)tile * D * D * 2) + tid;
        constexpr int N = D * D / 8 / TT;
        v4f in[2 * N];
#pragma unroll
        for (int x = 0; x < 2 * N; ++x) in[x] = S[2 * TT * (x >> 1) + (x & 1)];
#pragma unroll
        for (int x = 0; x < N; ++x) {
            const v4f a = in[2 * x], b = in[2 * x + 1];
            to[TT * x] = make_uint4(f2bf(a.x) | ((uint32_t)f2bf(a.y) << 16), f2bf(a.z) | ((uint32_t)f2bf(a.w) << 16),
                                    f2bf(b.x) | ((uint32_t)f2bf(b.y) << 16), f2bf(b.z) | ((uint32_t)f2bf(b.w) << 16));
        }
        if (tid < D) {
            A.smooth[tvec + tid] = 1.0f;
            A.scale[tvec + tid] = 1.0f;
        }
        if (tid == 0) A.rec_len[tile] = 0;
        return;
    }

    // the block: M(a, b) = M[8 kb + a][16 b + i], in the accumulator layout of
    // v_mfma_f64_16x16x4 (accumulator (a >> 2, b): row j + 4 (a & 3), column i)
    v4d m4[2][VPT];
#define M(a, b) m4[(a) >> 2][b][(a) & 3]
    // holds the block in registers at a phase boundary
    auto pin = [&]() {
#pragma unroll
        for (int b = 0; b < VPT; ++b) asm volatile("" : "+v"(m4[0][b]), "+v"(m4[1][b]));
    };

    if (MODE == TILE_QUANTIZE) {
        // A wave's part of the state is 128 rows of 128 bytes.  Loaded as its lanes hold it
        // (16 value rows next to each other) an instruction touches 64 pieces of lines;
        // loaded 8 lanes to a row's 128 bytes and turned in LDS, 8 whole lines (one state
        // without tokens 5.28 -> 4.46 us, 2048 states 34.1 -> 32.5).
        const int lane = tid & 63;
        const float *S = A.S_in + (size_t)tile * D * D + (size_t)(lane >> 3) * D + 32 * w + 4 * (lane & 7);
        v4f in[2 * VPT];
#pragma unroll
        for (int x = 0; x < 2 * VPT; ++x) in[x] = *(const v4f *)(S + (size_t)(8 * x) * D);
        v4f *turn = (v4f *)sh.red[4 * w];           // (LDS that is this wave's in the fit too: no barrier ends it)
        static_assert(sizeof(sh.red) / NW >= 16 * 128 && offsetof(TileShared<CODE>, red) % 16 == 0 && sizeof(sh.red[0]) % 4 == 0);
#pragma unroll
        for (int b = 0; b < VPT; ++b) {
            turn[TURN_ROWS(lane)] = in[2 * b];
            turn[64 + TURN_ROWS(lane)] = in[2 * b + 1];
            __builtin_amdgcn_wave_barrier();
            const v4f lo = turn[TURN_BLOCK(i, 2 * j)], hi = turn[TURN_BLOCK(i, 2 * j + 1)];
            __builtin_amdgcn_wave_barrier();
            M(0, b) = lo.x; M(1, b) = lo.y; M(2, b) = lo.z; M(3, b) = lo.w;
            M(4, b) = hi.x; M(5, b) = hi.y; M(6, b) = hi.z; M(7, b) = hi.w;
        }
        asm volatile("" ::: "memory");              // (from here on the fit writes there)
    } else {
        const int p = p_given >= 0 ? p_given : A.rec_len[tile];
        // the base's codes, row v's 16-byte chunk c at chunk (c + (v & 15)) mod SEGS of
        // its row: the 16 rows that a read touches then spread over the banks
        constexpr int SEGS = D * CodeFmt<CODE>::BITS / 8 / 16, NCP = D * SEGS / TT;
        auto copy_base = [&]() {
            if constexpr (!IsBF16<CODE>::value) {
                if (tid < 32) dma16(A.scale + tvec + 4 * tid, lds_addr(sh.scale));
                if (w == 1 && (tid & 63) < 32) dma16(A.smooth + tvec + 4 * (tid & 63), lds_addr(sh.smooth));
            }
            const uint4 *zt = (const uint4 *)(A.codes + (size_t)tile * D * (SEGS * 16));
#pragma unroll
            for (int x = 0; x < NCP; ++x) {
                const int P = TT * x + (int)threadIdx.x, v = P / SEGS, c = P % SEGS;
                dma16(zt + v * SEGS + (c + 16 * SEGS - (v & 15)) % SEGS, lds_addr(sh.codes + TT * x + 64 * w));
            }
        };
        // (an export reads the base of every tile: it is on its way while rec_len is.  A
        // commit leaves tiles alone, and starts with the records, which it needs first.)
        if (MODE == TILE_DEQUANT) copy_base();
        if (p < 0 || p > A.window) {                                  // corrupt: tile untouched
            if (tid == 0) atomicOr(A.err, (int)LQ_DEVERR_BAD_REC_LEN);
            if (MODE == TILE_DEQUANT) wait_vm_all();                  // (no copy outlives its LDS)
            return;
        }
        if (MODE == TILE_COMMIT) {
            const int req = tile / A.heads_v;
            if (p == 0 || (p_given < 0 && A.mask && A.mask[req] == 0)) return;   // uniform: tile untouched
        }
        // The rank-one terms in passes of TCH: the records newest first (the
        // decay of everything newer than a pass is carried along), then the
        // Compensator Tokens, which decay like the base.  A pass's operands are
        // copied straight into LDS during the pass before: a wave copies its 32
        // key channels of all records, and all value channels of two records.
        const int nrp = (p + TCH - 1) / TCH, passes = nrp + (r + TCH - 1) / TCH;
        const size_t rbase = (size_t)tile * A.window * D, cbase = (size_t)tile * r * D;
        const uint16_t *rab = A.rec_a + (size_t)tile * A.window * (GATE ? D : 1);
        // (pinned in scalar registers: the compiler would select between the kernel's
        // arguments through memory)
        const uint16_t *rkb = A.rec_k + rbase, *rub = A.rec_u + rbase, *ckb = A.comp_k + cbase, *cub = A.comp_u + cbase;
        asm volatile("" : "+s"(rkb), "+s"(rub), "+s"(rab), "+s"(ckb), "+s"(cub));
        uint32_t ras = 0;                           // scalar gate: the decay of slot lane & 7
        auto bounds = [&](int t, int &lo, int &n) {
            if (t < nrp) {
                const int hi = p - TCH * t;
                lo = hi > TCH ? hi - TCH : 0;
                n = hi - lo;
            } else {
                lo = TCH * (t - nrp);
                n = r - lo < TCH ? r - lo : TCH;
            }
        };
        auto load_pass = [&](int t) {
            int lo, n;
            bounds(t, lo, n);
            const bool rec = t < nrp;
            const uint16_t *pk = rec ? rkb : ckb, *pu = rec ? rub : cub;
            const int l = (int)threadIdx.x & 63, c = l & 31, s = c >> 2;
            const uint32_t off = (uint32_t)(lo + s) * D + 32 * w + 8 * (c & 3);
            if (s < n && (l < 32 || (GATE && rec)))
                dma16((l < 32 ? pk : rab) + off, lds_addr(&sh.raw_ka[w][0]));
            const int su = 2 * w + (c >> 4);
            if (l < 32 && su < n) dma16(pu + (uint32_t)(lo + su) * D + 8 * (c & 15), lds_addr(&sh.raw_u[w][0]));
            if (!GATE) {
                // (out of the asm above the pointer is generic: cast back to global)
                using gh = const __attribute__((address_space(1))) uint16_t;
                ras = rec && (l & 7) < n ? (uint32_t)((gh *)rab)[lo + (l & 7)] : 0x3C00u;
            }
        };
        if (passes > 0) load_pass(0);
        if (MODE == TILE_COMMIT) copy_base();
#pragma unroll
        for (int a = 0; a < 8; ++a)
#pragma unroll
            for (int b = 0; b < VPT; ++b) M(a, b) = -0.0;      // (a sum of -0 stays -0)

        // decay of everything newer than the pass: key channel 32 w + (lane & 31)
        double carry = 1.0;
#pragma unroll 1
        for (int t = 0; t < passes; ++t) {
            refresh();
            int lo, n;
            bounds(t, lo, n);
            const bool rec = t < nrp;
            // the first pass has landed; a commit's codes may follow (with a scalar gate they
            // too are waited for: the compiler waits for its load of the decays, and cannot
            // count the copies issued after it)
            if (MODE == TILE_COMMIT && t == 0) wait_vm<NCP>();
            else wait_vm_all();
            {
                // keys: lane (c, h) folds the decay into slots 7 - 4 h - e, e = 0..3, newest first
                const int c = tid & 31, h = (tid >> 5) & 1;
                const uint16_t *raw = (const uint16_t *)sh.raw_ka[w];
                double P, av[4];
                const int s0 = 7 - 4 * h;
                uint32_t rk[4], ra[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    rk[e] = raw[32 * (s0 - e) + c];
                    if (GATE) ra[e] = raw[TCH * 32 + 32 * (s0 - e) + c];
                }
                const uint2 u = ((const uint2 *)sh.raw_u[w])[tid & 63];
                if (GATE) {
                    // (all reads issued together; a slot past the pass's records, and every
                    // token, has decay 1)
                    asm volatile("" : "+v"(ra[0]), "+v"(ra[1]), "+v"(ra[2]), "+v"(ra[3]));
                    const int last = rec ? n : 0;
#pragma unroll
                    for (int e = 0; e < 4; ++e) av[e] = (double)h2f((uint16_t)(s0 - e < last ? ra[e] : 0x3C00u));
                    const double q = (av[0] * av[1]) * (av[2] * av[3]);
                    double q0, q1;
                    swap32_d(q, q, q0, q1);         // the newer and the older half's product
                    P = h ? carry * q0 : carry;
                    carry *= q0 * q1;
                } else {
                    float f[8];
#pragma unroll
                    for (int s = 0; s < 8; ++s) f[s] = row_lane(h2f((uint16_t)ras), s);
                    double Ps[9];
                    Ps[8] = carry;
#pragma unroll
                    for (int s = 7; s >= 0; --s) Ps[s] = Ps[s + 1] * (double)f[s];
                    carry = Ps[0];
                    P = h ? Ps[4] : Ps[8];
#pragma unroll
                    for (int e = 0; e < 4; ++e) av[e] = (double)(h ? f[3 - e] : f[7 - e]);
                }
                double key[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    key[e] = P * (double)h2f((uint16_t)rk[e]);
                    P *= av[e];
                }
                // an empty slot's key is -0 whatever the decay: 0 times an infinite one is a
                // NaN, and -0 times its value +0 adds nothing, to a sum of negative zeros neither
                if (n < TCH) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        key[e] = s0 - e < n ? key[e] : -0.0;
                        asm volatile("" : "+v"(key[e]));        // (stays in its branch)
                    }
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) sh.key[w][s0 - e][c] = key[e];
                // values: lane (record, 4-channel segment) of the wave's two records
                const int s = 2 * w + h;
                double *val = &sh.val[t & 1][s][4 * c];
                const uint32_t u0 = s < n ? u.x : 0u, u1 = s < n ? u.y : 0u;
                *(double2 *)&val[0] = make_double2((double)h2f((uint16_t)u0), (double)h2f((uint16_t)(u0 >> 16)));
                *(double2 *)&val[2] = make_double2((double)h2f((uint16_t)u1), (double)h2f((uint16_t)(u1 >> 16)));
            }
            __syncthreads();
            // this wave's raw copies have been read: the next pass may land there
            if (t + 1 < passes) load_pass(t + 1);
            refresh();
            // four slots per matrix product: lane (j, i) brings slot 4 g + j of key row
            // i (channel 8 (i & 3) + 4 x + (i >> 2), so that the accumulators hold this
            // thread's block) and of value column i
            const double *krow = &sh.key[w][j][8 * (i & 3) + (i >> 2)];
            const double *vrow = &sh.val[t & 1][j][i];
#pragma unroll 1
            for (int g = 0; g < n; g += 4) {
                const double k0 = krow[32 * g], k1 = krow[32 * g + 4];
#pragma unroll
                for (int b = 0; b < VPT; ++b) {
                    const double u = vrow[D * g + 16 * b];
                    m4[0][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(k0, u, m4[0][b], 0, 0, 0);
                    m4[1][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(k1, u, m4[1][b], 0, 0, 0);
                }
            }
        }
        wait_vm_all();
        refresh();
        sh.key[w][0][tid & 31] = carry;             // Gamma_{1:p} (both half-waves hold it)
        __syncthreads();
        // + the window-start base Gamma_{1:p} C dequant(Z) (Sec. 3.4 Eq. (smooth); the
        // BF16 state has unit scales and no smoothing, its arrays are not read)
        {
            double cv[8];
#pragma unroll
            for (int a = 0; a < 8; ++a)
                cv[a] = sh.key[w][0][8 * j + a] * (IsBF16<CODE>::value ? 1.0 : (double)sh.smooth[8 * kb + a]);
            // where the 8 codes lie in a row (the 6-bit ones may cross a chunk)
            uint32_t zoff[CODE == 3 ? 3 : 1];
#pragma unroll
            for (int e = 0; e < (CODE == 3 ? 3 : 1); ++e) {
                const uint32_t y = CodeFmt<CODE>::BITS * kb + 2 * e;
                zoff[e] = 16 * ((y / 16 + i) % SEGS) + (y & 15);
            }
            // (each row's codes are read from LDS one row ahead)
            typedef typename Codes8<CODE>::type C8;
            auto read_codes = [&](int b) -> C8 {
                const uint8_t *zr = (const uint8_t *)&sh.codes[(16 * b + i) * SEGS];
                if constexpr (CODE <= 1) {
                    return *(const uint2 *)(zr + zoff[0]);
                } else if constexpr (CODE == 2) {
                    return make_uint2(*(const uint32_t *)(zr + zoff[0]), 0u);
                } else if constexpr (CODE == 3) {
                    return make_uint2(*(const uint16_t *)(zr + zoff[0]) | ((uint32_t) * (const uint16_t *)(zr + zoff[1]) << 16),
                                      *(const uint16_t *)(zr + zoff[2]));
                } else {
                    return *(const uint4 *)(zr + zoff[0]);
                }
            };
            C8 z = read_codes(0);
            float dl = IsBF16<CODE>::value ? 1.0f : sh.scale[i];
#pragma unroll
            for (int b = 0; b < VPT; ++b) {
                C8 zn = z;
                float dn = dl;
                if (b + 1 < VPT) {
                    zn = read_codes(b + 1);
                    if (!IsBF16<CODE>::value) dn = sh.scale[16 * (b + 1) + i];
                }
                const double dv = IsBF16<CODE>::value ? 1.0 : (double)dl;
#pragma unroll
                for (int a = 0; a < 8; ++a) M(a, b) = fma(cv[a], code8_value<CODE>(z, a) * dv, M(a, b));
                __builtin_amdgcn_sched_barrier(0);      // two rows' codes live at a time beside the block
                z = zn;
                dl = dn;
            }
        }

        if (MODE == TILE_DEQUANT) {
            // Turned in the wave's own LDS, like the quantized state's loads: 8 whole lines
            // per store instead of 64 pieces.  Without records 32 states 6.38 -> 5.40 us, with
            // 33 records and 6-bit codes 2048 states 83 -> 75.
            const int lane = tid & 63;
            float *S = A.S_out + (size_t)tile * D * D + (size_t)(lane >> 3) * D + 32 * w + 4 * (lane & 7);
            v4f *turn = (v4f *)sh.key[w];
            asm volatile("" ::: "memory");          // (the decays there have been read)
#pragma unroll
            for (int b = 0; b < VPT; ++b) {
                turn[TURN_BLOCK(i, 2 * j)] = v4f{(float)M(0, b), (float)M(1, b), (float)M(2, b), (float)M(3, b)};
                turn[TURN_BLOCK(i, 2 * j + 1)] = v4f{(float)M(4, b), (float)M(5, b), (float)M(6, b), (float)M(7, b)};
                __builtin_amdgcn_wave_barrier();
                const v4f lo = turn[TURN_ROWS(lane)], hi = turn[64 + TURN_ROWS(lane)];
                __builtin_amdgcn_wave_barrier();
                *(v4f *)(S + (size_t)(16 * b) * D) = lo;
                *(v4f *)(S + (size_t)(16 * b + 8) * D) = hi;
            }
            return;
        }
        __syncthreads();                            // the fit reuses this LDS
        pin();
    }

    // ------------------------------------------------------------------ quantize
    // y[b] = sum over this thread's key channels of M x, x by lane of the row.  (These
    // sums and those over value channels start from +0: a product alone would make a
    // sum of zeros -0, and with it the FP16 bits of a token and the sign of a residual.)
    auto keys_dot = [&](double x, double *y) {
        const double x0 = row_lane(x, 0);
#pragma unroll
        for (int b = 0; b < VPT; ++b) y[b] = fma(M(0, b), x0, 0.0);
#pragma unroll
        for (int a = 1; a < 8; ++a) {
            const double xa = row_lane(x, a);
#pragma unroll
            for (int b = 0; b < VPT; ++b) y[b] = fma(M(a, b), xa, y[b]);
        }
    };
    int buf = 0;
#pragma unroll 1
    for (int h = 0; h < r; ++h) {
        refresh();
        // start vector: key-row l2 norms of the current residual.  A vector over
        // key channels lives in registers: lane i of a row holds channel i & 7 of
        // the row's block.
        double x;
        {
            const double n2 = sum_values(sh, [&](int a) {
                double s = M(a, 0) * M(a, 0);
#pragma unroll
                for (int b = 1; b < VPT; ++b) s = fma(M(a, b), M(a, b), s);
                return s;
            }, tid);
            x = n2 > 0.0 ? n2 * rsqrt(n2) : 0.0;
            const int e = wave_max_i32(n2 > 0.0 ? __builtin_amdgcn_frexp_exp(n2) : INT_MIN);
            if ((tid & 63) == 0) sh.ex[buf][w] = e;     // read after the first sweep's barrier
        }
        // Sweeps without normalisation: each is scaled by one power of two (exact, so
        // only the direction matters), the first also by one near 1/|x|, and the
        // vector is normalised once after the last.  With 2^(e-1) <= n < 2^e for the
        // largest squared row norm n, n <= sigma_1^2 <= |M|_F^2 <= 128 n: a sweep scaled by
        // 2^-(e+3) grows no vector by more than 2^4, and shrinks the part along the leading
        // direction by no more than 2^-4, far from the ends of the range for every sweep
        // count.  (A start vector without such a part may shrink to 0: rows v and -v have
        // the start (1, 1) and M^T (1, 1) = 0.  The pair is then zero, as the method's.)
        double sc = 0.0;
#pragma unroll 1
        for (int it = 0; it < A.power_iters; ++it) {
            refresh();
            double y[VPT];
            keys_dot(x, y);
            double2 t = sum_keys(sh, y, buf, tid);           // y_v = sum_k M_kv x_k
            double f = sc;
            if (it == 0) {
                const int e = max(max(sh.ex[buf][0], sh.ex[buf][1]), max(sh.ex[buf][2], sh.ex[buf][3]));
                const bool any = e != INT_MIN;          // a zero residual: every vector 0
                sc = any ? ldexp(1.0, -(e + 3)) : 0.0;
                f = any ? ldexp(sc, -(e >> 1)) : 0.0;
            }
            buf ^= 1;
            t.x *= f;
            t.y *= f;
            share_pairs(sh, t, y, tid);
            x = sum_values(sh, [&](int a) {             // x_k = sum_v M_kv y_v
                double s = fma(M(a, 0), y[0], 0.0);
#pragma unroll
                for (int b = 1; b < VPT; ++b) s = fma(M(a, b), y[b], s);
                return s;
            }, tid);
        }
        refresh();
        uint32_t keep;                                  // all ones, or 0 for a zero pair (in a scalar register)
        {
            const double z = wave_sum_half(x * x);
            if ((tid & 63) == 0) sh.nrm[buf][w] = z;
            __syncthreads();
            const double n2 = sum_nrm(sh, buf);
            buf ^= 1;
            x = n2 > 0.0 ? x * rsqrt(n2) : 0.0;         // a zero or non-finite residual gives a zero pair
            keep = __builtin_amdgcn_readfirstlane(n2 > 0.0 ? 0xFFFFu : 0u);
            asm volatile("" : "+s"(keep));
        }
        // the pair, rounded to FP16 and stored as soon as it is known
        const uint16_t kh = d2h_via_f32(x);             // rounded through fp32
        if (i < 8) A.comp_k[((size_t)tile * r + h) * D + 8 * kb + i] = kh;
        double kd = (double)h2f(kh);
        double us[VPT];
        keys_dot(kd, us);
        const double2 t = sum_keys(sh, us, buf, tid);        // u~_v = fp16(sum_k M_kv k~_k)
        buf ^= 1;
        // (0 times an infinity or a NaN is no zero: u~ of a zero pair is cleared, so that
        // the entries beside a non-finite one stay what they are)
        const uint16_t u0 = (uint16_t)(d2h_via_f32(t.x) & keep), u1 = (uint16_t)(d2h_via_f32(t.y) & keep);
        if (w == (h & 3)) {
            uint16_t *cu = A.comp_u + ((size_t)tile * r + h) * D + 32 * j + i;
            cu[0] = u0;
            cu[16] = u1;
        }
        share_pairs(sh, make_double2((double)h2f(u0), (double)h2f(u1)), us, tid);
        asm volatile("" : "+v"(kd));                    // (its eight lanes are taken again, not held)
#pragma unroll
        for (int a = 0; a < 8; ++a) {
            const double ka = row_lane(kd, a);
#pragma unroll
            for (int b = 0; b < VPT; ++b) M(a, b) = fma(-ka, us[b], M(a, b));
        }
    }
    refresh();

    if constexpr (IsBF16<CODE>::value) {
        // BF16 state: every entry rounded to nearest even through fp32 (the
        // window-end rounding of the per-window BF16 variant), unit scales
        const int lane = tid & 63;
        uint4 *turn = (uint4 *)sh.key[w];
        uint8_t *to = A.codes + ((size_t)tile * D + (lane >> 2)) * (2 * D) + 64 * w + 16 * (lane & 3);
#pragma unroll
        for (int b = 0; b < VPT; ++b) {
            uint32_t o[4];
#pragma unroll
            for (int e = 0; e < 4; ++e)
                o[e] = (uint32_t)f2bf((float)M(2 * e, b)) | ((uint32_t)f2bf((float)M(2 * e + 1, b)) << 16);
            // (a wave's part of a row is 64 bytes: turned in LDS, a store covers 16 of them)
            turn[64 * (b & 1) + 4 * i + (j ^ ((i >> 1) & 3))] = make_uint4(o[0], o[1], o[2], o[3]);
            __builtin_amdgcn_wave_barrier();
            const uint4 z = turn[64 * (b & 1) + (lane & 60) + ((lane & 3) ^ ((lane >> 3) & 3))];
            __builtin_amdgcn_wave_barrier();
            *(uint4 *)(to + (size_t)(16 * b) * (2 * D)) = z;
        }
        if (tid < D) {
            A.smooth[tvec + tid] = 1.0f;
            A.scale[tvec + tid] = 1.0f;
        }
        if (tid == 0) A.rec_len[tile] = 0;
        return;
    }
    // residual smoothing over key rows: c_k = sqrt(max(mean_v |R_kv|, 1e-12)) in fp32
    float ic[8];
    {
        const double z = sum_values(sh, [&](int a) {
            double s = fabs(M(a, 0));
#pragma unroll
            for (int b = 1; b < VPT; ++b) s += fabs(M(a, b));
            return s;
        }, tid);
        float c = 1.0f;
        if (A.smooth_on) c = (float)sqrt(fmax(z * (1.0 / (double)D), (double)1e-12f));
        if (i < 8) A.smooth[tvec + 8 * kb + i] = c;
        const float rc = 1.0f / c;
#pragma unroll
        for (int a = 0; a < 8; ++a) ic[a] = row_lane(rc, a);
    }
    refresh();
    // per-value-channel scale and codes, decided in fp32.  Lane (row j, i) has the
    // largest |R^C| of channels 32 j + i, 32 j + 16 + i over its wave's keys.
    constexpr float QMAX = CodeFmt<CODE>::QMAX;
    float inv[VPT];
    float rc[8][VPT];                               // the smoothed residual
#pragma unroll
    for (int b = 0; b < VPT; ++b)
#pragma unroll
        for (int a = 0; a < 8; ++a) rc[a][b] = (float)M(a, b) * ic[a];
    {
        float am[VPT];
#pragma unroll
        for (int b = 0; b < VPT; ++b) {
            am[b] = fabsf(rc[0][b]);
#pragma unroll
            for (int a = 1; a < 8; ++a) am[b] = fmaxf(am[b], fabsf(rc[a][b]));
        }
        float a0, a1;
        rows4_max_scatter(am, a0, a1);
        const int lane = tid & 63;
        float2 *part = (float2 *)sh.part[buf];
        part[64 * w + lane] = make_float2(a0, a1);
        __syncthreads();
        float2 q[NW];
#pragma unroll
        for (int x = 0; x < NW; ++x) q[x] = part[64 * x + lane];
        a0 = fmaxf(fmaxf(q[0].x, q[1].x), fmaxf(q[2].x, q[3].x));
        a1 = fmaxf(fmaxf(q[0].y, q[1].y), fmaxf(q[2].y, q[3].y));
        if (w == 0) {
            A.scale[tvec + 32 * j + i] = a0 > 0.0f ? a0 / QMAX : 0.0f;
            A.scale[tvec + 32 * j + 16 + i] = a1 > 0.0f ? a1 / QMAX : 0.0f;
        }
        float *vec = (float *)sh.vec[w];
        __builtin_amdgcn_wave_barrier();
        *(float2 *)&vec[2 * lane] = make_float2(a0 > 0.0f ? QMAX / a0 : 0.0f, a1 > 0.0f ? QMAX / a1 : 0.0f);
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            const float2 y = *(const float2 *)&vec[32 * x + 2 * i];
            inv[2 * x] = y.x;
            inv[2 * x + 1] = y.y;
        }
    }
#pragma unroll
    for (int b = 0; b < VPT; ++b) {
        uint32_t c8[8];
#pragma unroll
        for (int a = 0; a < 8; ++a) {
            // (clamped to +-QMAX)
            if (CODE == 1) c8[a] = f_to_e4m3(__builtin_amdgcn_fmed3f(rc[a][b] * inv[b], -QMAX, QMAX));
            else c8[a] = (uint32_t)(int32_t)__builtin_amdgcn_fmed3f(rintf(rc[a][b] * inv[b]), -QMAX, QMAX);
        }
        store_codes8<CODE>(A.codes, tile, 16 * b + i, kb, encode8<CODE>(c8));
    }
    if (tid == 0) A.rec_len[tile] = 0;
}
#undef M

inline TileArgs tile_args(const lq_dims &d, const StatePtrs &s, const float *S_in, float *S_out,
                          const int32_t *mask) {
    TileArgs a;
    a.codes = (uint8_t *)s.codes;
    a.scale = s.scale;
    a.smooth = s.smooth;
    a.comp_k = s.comp_k;
    a.comp_u = s.comp_u;
    a.rec_k = s.rec_k;
    a.rec_u = s.rec_u;
    a.rec_a = s.rec_a;
    a.rec_len = s.rec_len;
    a.err = s.err;
    a.S_in = S_in;
    a.S_out = S_out;
    a.mask = mask;
    a.heads_v = d.heads_v;
    a.window = d.window;
    a.n_comp = d.n_comp;
    a.power_iters = d.power_iters;
    a.smooth_on = d.smooth;
    return a;
}

}  // namespace

}  // namespace lq
