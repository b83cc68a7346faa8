// The two-group left-to-right sweep of a layer whose first group has no
// output modes and whose second group has no input modes (the paper's TT
// layout, input cores then output cores, Sec. 4.2): W = A B with
// A [N_in][R] and B [R][N_out] through one bond of compacted rank R <= 64.
//   forward   S = X A,     Y = S B
//   backward  T = dY B^T,  dX = T A^T,  dA = X^T T,  dB = S^T dY
// Everything of size N_in, N_out or b runs at the rate of its memory traffic:
// a pass reads its input once, keeps its R-wide state in LDS between the two
// products and writes its output once, and the meets read X and dY once more.
// Launches per training step: build, pass (Y), pass (dX), meet, split sum,
// core gradients.  Sweeps of this kind outside faster_here keep the general
// route (sweep.hip).  The general sweep (one GEMM per product on tiles made for
// square operands, and one kernel per core and step of the batch-free work)
// took 17 launches and 535 us on 1024 -> 4096, r = 32, 40000 tokens in bf16
// and 205 us on 768 -> 3072, r = 30, 4096 tokens in fp32; this one 331 and
// 101 us.
//
// Batch-free side: each group is a chain of cores from its end of rank 1 to
// the bond of rank R (group 0 left to right, group 1 right to left), core j
// of the chain as C_j [c_{j-1}][s_j][c_j] with mode s_j and chain ranks c.
//   V_j[(s_1 .. s_j)][c_j] = sum_{c_{j-1}} V_{j-1}[..][c_{j-1}] C_j[c_{j-1}][s_j][c_j]
// and V_q is A, or B^T.  With E_q = dA (dB^T) the gradients are
//   E_{j-1}[x][c_{j-1}] = sum_{s, c_j} E_j[(x, s)][c_j] C_j[c_{j-1}][s][c_j]
//   dC_j[c_{j-1}][s][c_j] = sum_x V_{j-1}[x][c_{j-1}] E_j[(x, s)][c_j].
// Indices x run in the layout's own order: group 0 has s_j least significant
// (x s_j), group 1 most significant (s_j x).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>

#include "internal.h"

namespace comera {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void lds_void_t;
typedef __attribute__((address_space(3))) s16x4 lds_s16x4_t;

// two floats -> two bf16 in one dword, a low (round to nearest even)
__device__ __forceinline__ uint32_t pack2(float a, float b) {
    const f32x2 v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}
__device__ __forceinline__ void put(float *p, float v) { *p = v; }
__device__ __forceinline__ void put(uint16_t *p, float v) { *p = uint16_t(pack2(v, 0.f)); }

// acc += A B over one 64-byte k step: a lane holds the 16 bytes (8 bf16 or 4
// fp32) of its row l % 16 at 16 (l / 16); fp32 takes the four elements one
// MFMA each, the same permutation of k for both operands.  D: column l % 16,
// rows 4 (l / 16) .. + 3.
template <typename T>
__device__ __forceinline__ void mma(f32x4 &acc, u32x4 a, u32x4 b) {
    if constexpr (sizeof(T) == 2) {
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc,
                                                      0, 0, 0);
    } else {
        const f32x4 x = __builtin_bit_cast(f32x4, a), y = __builtin_bit_cast(f32x4, b);
#pragma unroll
        for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x[j], y[j], acc, 0, 0, 0);
    }
}

// 16 bytes at p, by elements when the tensor is not 16-byte aligned
template <typename T>
__device__ __forceinline__ u32x4 load16(const T *p, bool vec) {
    if (vec) return *reinterpret_cast<const u32x4 *>(p);
    constexpr int E = 16 / int(sizeof(T));
    T v[E];
#pragma unroll
    for (int e = 0; e < E; ++e) v[e] = p[e];
    u32x4 r;
    __builtin_memcpy(&r, v, 16);
    return r;
}

// orders this wave's LDS writes before its reads of other lanes' data (LDS
// operations of one wave complete in order; this keeps the compiler from
// moving them)
__device__ __forceinline__ void wave_lds_order() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---------------------------------------------------------------- pass
// state = in op1^T, out = state op2^T for tiles of 16 MT tokens: in [b][K],
// op1 [K / KE][RP][KE] (KE elements = 64 bytes, so that an MFMA operand is
// 1 KB in a row: as [RP][K], rows a power of two apart, all its lines came
// from one L2 channel, 26 against 21 us on a 3072-wide fp32 input of 4096
// tokens), op2 [N][RP], out [b][N]; the state is rounded to the
// activation dtype between the products and kept for the meets, fp32 as
// [b][RP], bf16 as [RP][spitch] (tokens contiguous, what an MFMA over tokens
// reads).  op1 and op2 are padded with zeros from R to RP.
// Bound by HBM (in read once, out written once).  The eight waves share K:
// each takes 128-byte pieces of the rows, straight from global memory in the
// MFMA's operand layout, and the partial states meet in LDS in wave order;
// then each wave takes 64-column strips of the output, which leave through
// 16 staged rows as whole lines.  MT by the token count: the largest tile
// (fewest reads of op1 and op2 from L2) that still gives every CU a
// workgroup.
struct PassArgs {
    const void *in, *op1, *op2;
    void *out, *state;
    int64_t K, N, b, spitch;
    int R;                       // state entries R .. RP are padding
    int vec_in, vec_out;
};
constexpr int kPassWaves = 8;
constexpr int kPassRounds = 2;   // rounds of loads in flight (3 and 4 measured level or slower)

template <typename T, int RP, int MT>
__global__ __launch_bounds__(64 * kPassWaves) void tt_pass_kernel(PassArgs a) {
    constexpr int ESZ = int(sizeof(T)), E = 16 / ESZ, KE = 64 / ESZ, RB = RP / 16, KK = RP / KE, NW = kPassWaves;
    constexpr int U = kPassRounds;
    constexpr int TOK = 16 * MT, RPITCH = RP + 4, SPITCH = RP * ESZ + 16, OPITCH = 64 * ESZ + 16;
    constexpr int kRed = NW * TOK * RPITCH * 4, kStage = NW * 16 * OPITCH;
    __shared__ __attribute__((aligned(16))) char buf[kRed > kStage ? kRed : kStage];
    __shared__ __attribute__((aligned(16))) char st[TOK * SPITCH];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lr = lane & 15, lg = lane >> 4;
    const int64_t t0 = int64_t(blockIdx.x) * TOK;
    const T *in = reinterpret_cast<const T *>(a.in);
    const T *op1 = reinterpret_cast<const T *>(a.op1), *op2 = reinterpret_cast<const T *>(a.op2);
    {
        f32x4 acc[MT][RB];
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int r = 0; r < RB; ++r) acc[i][r] = f32x4{0.f, 0.f, 0.f, 0.f};
        const T *row[MT];
#pragma unroll
        for (int i = 0; i < MT; ++i) row[i] = in + min(t0 + 16 * i + lr, a.b - 1) * a.K;
        const T *orow = op1 + lr * KE + lg * E;
        const int64_t pairs = (a.K + 2 * KE - 1) / (2 * KE);
        const bool vec = a.vec_in;
        // two 64-byte k steps (one line of every row) per round
        auto load = [&](int64_t p, u32x4 (&x)[2][MT], u32x4 (&o)[2][RB]) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int64_t k = (2 * p + h) * KE + lg * E;
                const bool in_k = k < a.K;   // K is a whole number of 16-byte chunks
#pragma unroll
                for (int i = 0; i < MT; ++i) x[h][i] = in_k ? load16(row[i] + k, vec) : u32x4{0, 0, 0, 0};
#pragma unroll
                for (int r = 0; r < RB; ++r)
                    o[h][r] = in_k ? *reinterpret_cast<const u32x4 *>(orow + ((2 * p + h) * RP + 16 * r) * KE)
                                   : u32x4{0, 0, 0, 0};
            }
        };
        auto madd = [&](const u32x4 (&x)[2][MT], const u32x4 (&o)[2][RB]) {
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int i = 0; i < MT; ++i)
#pragma unroll
                    for (int r = 0; r < RB; ++r) mma<T>(acc[i][r], o[h][r], x[h][i]);
        };
        u32x4 x[U][2][MT], o[U][2][RB];
        // tiles start at different columns: rows are a power of two apart on
        // many layers, and all workgroups at one column would load one
        // memory channel at a time
        const int64_t rot = int64_t(blockIdx.x % 16) * pairs / 16;
        auto place = [&](int64_t p) { return p + rot < pairs ? p + rot : p + rot - pairs; };
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (wave + u * NW < pairs) load(place(wave + u * NW), x[u], o[u]);
        for (int64_t p = wave; p < pairs; p += U * NW) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (p + u * NW < pairs) madd(x[u], o[u]);
                if (p + (u + U) * NW < pairs) load(place(p + (u + U) * NW), x[u], o[u]);
            }
        }
        // lane: token lr of its block, four consecutive state entries
        float *red = reinterpret_cast<float *>(buf) + wave * TOK * RPITCH;
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int r = 0; r < RB; ++r)
                *reinterpret_cast<f32x4 *>(red + (16 * i + lr) * RPITCH + 16 * r + 4 * lg) = acc[i][r];
    }
    __syncthreads();
    for (int id = tid; id < TOK * RP / 4; id += 64 * NW) {
        // bf16: tokens fastest (its state rows run over tokens), fp32: state entries fastest
        const int tok = sizeof(T) == 2 ? id % TOK : id / (RP / 4), r4 = sizeof(T) == 2 ? id / TOK : id % (RP / 4);
        const float *red = reinterpret_cast<const float *>(buf) + tok * RPITCH + 4 * r4;
        f32x4 v = *reinterpret_cast<const f32x4 *>(red);
#pragma unroll
        for (int w = 1; w < NW; ++w) v += *reinterpret_cast<const f32x4 *>(red + w * TOK * RPITCH);
        // an infinity times the zeros of op1 would leave NaN in the padding,
        // which the zeros of op2 carried into the whole row of out
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = 4 * r4 + e < a.R ? v[e] : 0.f;
        if constexpr (sizeof(T) == 2) {
            u32x2 h;
            h[0] = pack2(v[0], v[1]);
            h[1] = pack2(v[2], v[3]);
            *reinterpret_cast<u32x2 *>(st + tok * SPITCH + 8 * r4) = h;
            if (t0 + tok < a.b) {
                uint16_t *s = reinterpret_cast<uint16_t *>(a.state) + int64_t(4 * r4) * a.spitch + t0 + tok;
                s[0] = uint16_t(h[0]);
                s[a.spitch] = uint16_t(h[0] >> 16);
                s[2 * a.spitch] = uint16_t(h[1]);
                s[3 * a.spitch] = uint16_t(h[1] >> 16);
            }
        } else {
            *reinterpret_cast<f32x4 *>(st + tok * SPITCH + 16 * r4) = v;
            if (t0 + tok < a.b)
                *reinterpret_cast<f32x4 *>(reinterpret_cast<float *>(a.state) + (t0 + tok) * RP + 4 * r4) = v;
        }
    }
    if (!a.out) return;
    __syncthreads();
    u32x4 s[MT][KK];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int k = 0; k < KK; ++k)
            s[i][k] = *reinterpret_cast<const u32x4 *>(st + (16 * i + lr) * SPITCH + 64 * k + 16 * lg);
    char *stage = buf + wave * 16 * OPITCH;
    const int64_t strips = (a.N + 63) / 64;
    u32x4 w[4][KK];
    auto loadw = [&](int64_t c) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const T *o = op2 + min(64 * c + 16 * j + lr, a.N - 1) * RP + lg * E;
#pragma unroll
            for (int k = 0; k < KK; ++k) w[j][k] = *reinterpret_cast<const u32x4 *>(o + k * KE);
        }
    };
    if (wave < strips) loadw(wave);
    T *out = reinterpret_cast<T *>(a.out);
    for (int64_t c = wave; c < strips; c += NW) {
        f32x4 acc[MT][4];
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int k = 0; k < KK; ++k) mma<T>(acc[i][j], w[j][k], s[i][k]);
            }
        if (c + NW < strips) loadw(c + NW);
#pragma unroll
        for (int i = 0; i < MT; ++i) {
            // 16 tokens x 64 columns; a lane holds four columns of token lr
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                char *d = stage + lr * OPITCH + (16 * j + 4 * lg) * ESZ;
                if constexpr (sizeof(T) == 2) {
                    u32x2 h;
                    h[0] = pack2(acc[i][j][0], acc[i][j][1]);
                    h[1] = pack2(acc[i][j][2], acc[i][j][3]);
                    *reinterpret_cast<u32x2 *>(d) = h;
                } else {
                    *reinterpret_cast<f32x4 *>(d) = acc[i][j];
                }
            }
            wave_lds_order();
            constexpr int PPR = 64 * ESZ / 16, RPI = 64 / PPR;   // pieces per row, rows per store
#pragma unroll
            for (int q = 0; q < 16 / RPI; ++q) {
                const int r = q * RPI + lane / PPR, pc = lane % PPR;
                const u32x4 v = *reinterpret_cast<const u32x4 *>(stage + r * OPITCH + pc * 16);
                const int64_t t = t0 + 16 * i + r, col = 64 * c + pc * E;
                if (t < a.b && col < a.N) {   // N is a whole number of 16-byte pieces
                    T *o = out + t * a.N + col;
                    if (a.vec_out) {
                        *reinterpret_cast<u32x4 *>(o) = v;
                    } else {
                        T x[E];
                        __builtin_memcpy(x, &v, 16);
#pragma unroll
                        for (int e = 0; e < E; ++e) o[e] = x[e];
                    }
                }
            }
            wave_lds_order();
        }
    }
}

// ---------------------------------------------------------------- meets
// part[split][c][r] = sum over the split's tokens of V[t][c] S[t][r] for two
// problems in one launch: V = X with the dY state (rows c < C0 of a
// partial), V = dY with the X state (rows C0 ..).  Bound by HBM: V is read
// once.  No workgroup barrier: every wave owns its columns.
struct MeetArgs {
    const void *V[2], *S[2];
    int64_t C[2];
    int strips0;                 // column strips of problem 0
    int64_t b, spitch, kchunk, split_stride;
    float *part;
    int R;                       // columns R .. RP of a partial are padding: zeros, also beside infinities in V
    int vec[2];
};

// bf16: a wave takes CW columns; 32 tokens x CW columns and the state's
// [RP][32 tokens] go straight to LDS (global_load_lds), two stages per wave,
// and reach the MFMA through the transposing read (four k rows of 16
// columns per 16 lanes).  Bank conflicts: V rows are 128-byte groups of 8
// chunks; chunk pair p of row k sits at p ^ (bit 1 of k, bit 3 of k), so the
// eight rows that 32 lanes read cover all 64 banks; state chunk g of row r
// at g ^ ((r / 4) & 3).
constexpr int kMeetWaves = 4;
template <int RP>
constexpr int meet_cw() { return RP == 32 ? 128 : 64; }

template <int RP>
__global__ __launch_bounds__(64 * kMeetWaves) void tt_meet_bf16_kernel(MeetArgs a) {
    constexpr int CW = meet_cw<RP>(), NC = CW / 64, RB = RP / 16, NB = CW / 16;
    constexpr int kV = 32 * CW * 2, kSlot = kV + RP * 64, NOPS = kV / 1024 + RP * 64 / 1024;
    __shared__ __attribute__((aligned(16))) char slots0[kMeetWaves * kSlot];
    __shared__ __attribute__((aligned(16))) char slots1[kMeetWaves * kSlot];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lr = lane & 15, lg = lane >> 4;
    const int pr = int(blockIdx.x) >= a.strips0 ? 1 : 0;
    const int strip = int(blockIdx.x) - (pr ? a.strips0 : 0);
    const int64_t C = a.C[pr], c0 = (int64_t(strip) * kMeetWaves + wave) * CW;
    if (c0 >= C) return;
    const int64_t tb = int64_t(blockIdx.y) * a.kchunk, te = min(a.b, tb + a.kchunk);
    const uint16_t *V = reinterpret_cast<const uint16_t *>(a.V[pr]);
    const uint16_t *S = reinterpret_cast<const uint16_t *>(a.S[pr]);
    const int ns = te > tb ? int((te - tb + 31) / 32) : 0;
    const bool vec = a.vec[pr];
    char *slot0 = slots0 + wave * kSlot, *slot1 = slots1 + wave * kSlot;

    // instruction (column group n, i) fills rows 8 i .. 8 i + 7 of 64 columns
    auto issue = [&](char *slot, int k) {
        const int64_t t = tb + 32 * int64_t(k);
        auto chunks = [&](auto put16) {
#pragma unroll
            for (int n = 0; n < NC; ++n)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int row = 8 * i + (lane >> 3);
                    const int ch = (lane & 7) ^ ((((row >> 1) & 1) | (((row >> 3) & 1) << 1)) << 1);
                    put16(V + min(t + row, te - 1) * C + min(c0 + 64 * n + 8 * ch, C - 8), slot + (4 * n + i) * 1024);
                }
        };
        if (vec)
            chunks([&](const uint16_t *g, char *l) {
                __builtin_amdgcn_global_load_lds(reinterpret_cast<const void *>(g), (lds_void_t *)l, 16, 0, 0);
            });
        else
            chunks([&](const uint16_t *g, char *l) { *reinterpret_cast<u32x4 *>(l + 16 * lane) = load16(g, false); });
#pragma unroll
        for (int i = 0; i < RP / 16; ++i) {
            const int row = 16 * i + (lane >> 2), g = (lane & 3) ^ ((row >> 2) & 3);
            __builtin_amdgcn_global_load_lds(reinterpret_cast<const void *>(S + row * a.spitch + t + 8 * g),
                                             (lds_void_t *)(slot + kV + i * 1024), 16, 0, 0);
        }
    };
    // a last stage of rem < 32 tokens: the others are set to zero
    auto fix = [&](char *slot, int k) {
        const int rem = int(te - tb - 32 * int64_t(k));
        if (rem >= 32) return;
        const u32x4 z = {0, 0, 0, 0};
#pragma unroll
        for (int n = 0; n < NC; ++n)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (8 * i + (lane >> 3) >= rem) *reinterpret_cast<u32x4 *>(slot + (4 * n + i) * 1024 + 16 * lane) = z;
#pragma unroll
        for (int i = 0; i < RP / 16; ++i) {
            const int row = 16 * i + (lane >> 2), g = (lane & 3) ^ ((row >> 2) & 3);
            uint16_t *s = reinterpret_cast<uint16_t *>(slot + kV + i * 1024 + 16 * lane);
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (8 * g + e >= rem) s[e] = 0;
        }
        wave_lds_order();
    };
    f32x4 acc[NB][RB];
#pragma unroll
    for (int c = 0; c < NB; ++c)
#pragma unroll
        for (int r = 0; r < RB; ++r) acc[c][r] = f32x4{0.f, 0.f, 0.f, 0.f};
    // transposing reads: lane j of a 16-lane group g reads row 8 g + 4 h + j / 4,
    // columns 4 (j % 4) .. + 3 of the 16-column block
    uint32_t va[2], vf[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int row = 8 * lg + 4 * h + (lr >> 2);
        vf[h] = ((row >> 1) & 1) | (((row >> 3) & 1) << 1);
        va[h] = uint32_t(row * 128 + ((lr >> 1) & 1) * 16 + (lr & 1) * 8);
    }
    const uint32_t sa = uint32_t(kV + lr * 64 + ((lg ^ ((lr >> 2) & 3)) * 16));
    auto stage = [&](const char *slot) {
        bf16x8 sv[RB];
#pragma unroll
        for (int r = 0; r < RB; ++r) sv[r] = *reinterpret_cast<const bf16x8 *>(slot + sa + r * 1024);
#pragma unroll
        for (int c = 0; c < NB; ++c) {
            s16x4 x[2];
#pragma unroll
            for (int h = 0; h < 2; ++h)
                x[h] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                    (lds_s16x4_t *)(slot + (c / 4) * 4096 + va[h] + (((uint32_t(c) & 3) ^ vf[h]) << 5)));
            const bf16x8 vv = __builtin_bit_cast(bf16x8, __builtin_shufflevector(x[0], x[1], 0, 1, 2, 3, 4, 5, 6, 7));
#pragma unroll
            for (int r = 0; r < RB; ++r) acc[c][r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vv, sv[r], acc[c][r], 0, 0, 0);
        }
    };
    // this wave's LDS reads of a slot have returned before it is refilled
    auto reads_done = [&]() {
        __builtin_amdgcn_s_waitcnt(0xC07F);
        asm volatile("" ::: "memory");
    };
    // all but the newest stage's loads have landed (loads complete in order)
    auto landed = [&](bool newest) {
        if (newest && vec)
            __builtin_amdgcn_s_waitcnt(0x0F70 | (NOPS & 15));
        else
            __builtin_amdgcn_s_waitcnt(0x0070);
        asm volatile("" ::: "memory");
    };
    static_assert(NOPS < 16, "vmcnt immediate");
    if (ns > 0) issue(slot0, 0);
    for (int k = 0; k < ns; k += 2) {
        if (k + 1 < ns) issue(slot1, k + 1);
        landed(k + 1 < ns);
        fix(slot0, k);
        stage(slot0);
        reads_done();
        if (k + 1 >= ns) break;
        if (k + 2 < ns) issue(slot0, k + 2);
        landed(k + 2 < ns);
        fix(slot1, k + 1);
        stage(slot1);
        reads_done();
    }
    float *out = a.part + int64_t(blockIdx.y) * a.split_stride + (pr ? a.C[0] * RP : 0);
#pragma unroll
    for (int c = 0; c < NB; ++c)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int64_t col = c0 + 16 * c + 4 * lg + v;
            if (col < C)
#pragma unroll
                for (int r = 0; r < RB; ++r) out[col * RP + 16 * r + lr] = 16 * r + lr < a.R ? acc[c][r][v] : 0.f;
        }
}

// fp32: a wave takes 64 columns, straight from global memory: lane (t = l /
// 16, i = l % 16) loads columns 4 i .. 4 i + 3 of token t, whose element j is
// row i of the MFMA for columns 4 i + j; of the state, entries RB i .. of the
// same token.
template <int RP>
__global__ __launch_bounds__(64 * kMeetWaves) void tt_meet_f32_kernel(MeetArgs a) {
    constexpr int RB = RP / 16, U = 8;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lr = lane & 15, lg = lane >> 4;
    const int pr = int(blockIdx.x) >= a.strips0 ? 1 : 0;
    const int strip = int(blockIdx.x) - (pr ? a.strips0 : 0);
    const int64_t C = a.C[pr], c0 = (int64_t(strip) * kMeetWaves + wave) * 64;
    if (c0 >= C) return;
    const int64_t tb = int64_t(blockIdx.y) * a.kchunk, te = min(a.b, tb + a.kchunk);
    const bool vec = a.vec[pr];
    const float *V = reinterpret_cast<const float *>(a.V[pr]) + min(c0 + 4 * lr, C - 4);
    const float *S = reinterpret_cast<const float *>(a.S[pr]) + RB * lr;
    f32x4 acc[4][RB];
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int r = 0; r < RB; ++r) acc[j][r] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int64_t t = tb + lg; t - lg < te; t += 4 * U) {
        f32x4 v[U];
        float s[U][RB];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool in = t + 4 * u < te;
            v[u] = in ? __builtin_bit_cast(f32x4, load16(V + (t + 4 * u) * C, vec)) : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int r = 0; r < RB; ++r) s[u][r] = in ? S[(t + 4 * u) * RP + r] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int r = 0; r < RB; ++r)
                    acc[j][r] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[u][j], s[u][r], acc[j][r], 0, 0, 0);
    }
    float *out = a.part + int64_t(blockIdx.y) * a.split_stride + (pr ? a.C[0] * RP : 0);
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int64_t col = c0 + 4 * (4 * lg + v) + j;
            if (col < C)
#pragma unroll
                for (int r = 0; r < RB; ++r) out[col * RP + RB * lr + r] = RB * lr + r < a.R ? acc[j][r][v] : 0.f;
        }
}

// ---------------------------------------------------------------- batch-free
// One group as a chain from its rank-1 end; position j = 1 .. q.
struct Chain {
    int q, rev;                   // rev: right to left (group 1)
    const float *G[kMaxCores];    // raw core at position j (index j - 1)
    const float *D[kMaxCores];    // mask of that core's right bond, or null
    float *dG[kMaxCores];         // gradient of the core, or null
    float *keep[kMaxCores];       // compacted masked-core gradient for the mask gradients, or null
    int S[kMaxCores];             // mode of position j (index j - 1)
    int N[kMaxCores + 1];         // S_1 .. S_j
    int r[kMaxCores + 1];         // chain ranks (compacted), r[0] = 1, r[q] = R
    int rp[kMaxCores + 1];        // the same rounded up to 16, rp[q] = RP
    int fl[kMaxCores], fr[kMaxCores];   // full left and right ranks of the core
    int bl[kMaxCores];            // its left bond (row of the maps); the right one is the next
    float *V[kMaxCores + 1];      // V_j [N_j][rp_j], j = 1 .. q - 1
    float *C[kMaxCores + 1];      // C_j [r_{j-1}][S_j][rp_j], j = 2 .. q
    const float *E;               // E_q [N_q][RP]
    void *op, *opt;               // V_q [N_q][RP] and [N_q / KE][RP][KE] (64-byte rows over N_q), activation dtype
};
struct ChainsArgs {
    Chain ch[2];
    int blk[3];                              // first workgroup of group 1, of the folds, end
    int gblk[2 * kMaxCores + 1];             // core gradients: first workgroup of position p (both groups)
    uint8_t map[kMaxCores + 1][64];          // compacted -> full entry of every bond
};
static_assert(sizeof(ChainsArgs) <= 4096, "kernel arguments");

// What a workgroup keeps of the arguments: its group's chain, the maps, and
// per position the mask of the core's right bond (1 where there is none).
// Kernel arguments read field by field are one memory round trip each.
struct ChainLds {
    Chain h;
    uint8_t map[kMaxCores + 1][64];
    float D[kMaxCores][64];
};

// n bytes (a multiple of 4) of the kernel arguments into LDS by NT threads
template <int NT>
__device__ __forceinline__ void copy_args(void *dst, const void *src, int n, int t) {
    for (int i = t; i < n / 4; i += NT) reinterpret_cast<uint32_t *>(dst)[i] = reinterpret_cast<const uint32_t *>(src)[i];
}
template <int NT>
__device__ __forceinline__ void load_chain(ChainLds &l, const ChainsArgs &a, int g, int t) {
    static_assert(sizeof(Chain) % 4 == 0 && sizeof(a.map) % 4 == 0, "copied as dwords");
    copy_args<NT>(&l.h, &a.ch[g], int(sizeof(Chain)), t);
    copy_args<NT>(l.map, a.map, int(sizeof(a.map)), t);
    __syncthreads();
}

// C_j[cp][s][c] without the mask
__device__ __forceinline__ float core_at(const ChainLds &l, int j, int cp, int s, int c) {
    const Chain &h = l.h;
    const int i = j - 1, lt = l.map[h.bl[i]][h.rev ? c : cp], rt = l.map[h.bl[i] + 1][h.rev ? cp : c];
    return h.G[i][(lt * h.S[i] + s) * h.fr[i] + rt];
}

// Index of (x, s) at position j
__device__ __forceinline__ int chain_index(const Chain &h, int j, int x, int s) {
    return h.rev ? s * h.N[j - 1] + x : x * h.S[j - 1] + s;
}

// V_1 .. V_{q-1}, the operands A, A^T, B^T, B and the folded cores C_j: one
// workgroup per index of V_{q-1} follows the chain down to its row and
// multiplies it with the last core; the workgroups after those copy the
// cores.  Bound by latency: q - 1 dependent rounds of loads.
template <typename T>
__global__ __launch_bounds__(256) void tt_build_kernel(ChainsArgs a) {
    constexpr int KE = 64 / int(sizeof(T));
    __shared__ ChainLds l;
    __shared__ float v[64], red[4][64];
    const int t = threadIdx.x, blk = blockIdx.x;
    const bool fold = blk >= a.blk[1];
    const int g = fold ? (blk - a.blk[1]) & 1 : blk >= a.blk[0] ? 1 : 0;
    load_chain<256>(l, a, g, t);
    const Chain &h = l.h;
    const int q = h.q, rev = h.rev;
    // masks of every position's core, one round of loads
    for (int i = t; i < q * 64; i += 256) {
        const int p = i >> 6, c = i & 63, n = rev ? h.r[p] : h.r[p + 1];
        l.D[p][c] = h.D[p] && c < n ? h.D[p][l.map[h.bl[p] + 1][c]] : 1.f;
    }
    if (t < 64) v[t] = t == 0 ? 1.f : 0.f;
    __syncthreads();
    if (fold) {
        const int nb = (a.blk[2] - a.blk[1]) / 2;
        for (int j = 2; j <= q; ++j) {
            // below 2^31 entries (layout_bottleneck): unsigned, so that the
            // step past the end does not wrap
            const uint32_t rp = h.rp[j], S = h.S[j - 1], total = uint32_t(h.r[j - 1]) * S * rp;
            for (uint32_t o = ((blk - a.blk[1]) >> 1) * 256 + t; o < total; o += nb * 256) {
                const int c = o % rp, u = o / rp, cp = u / S;
                h.C[j][o] = c < h.r[j] ? core_at(l, j, cp, u - cp * int(S), c) * l.D[j - 1][rev ? cp : c] : 0.f;
            }
        }
        return;
    }
    const int xq = blk - (g ? a.blk[0] : 0);   // index of V_{q-1}
    for (int j = 1; j < q; ++j) {
        // digit and index of position j in xq: divide the later positions
        // out; when every later digit is 0 this workgroup writes V_j[y]
        int y = xq;
        bool first = true;
        for (int i = q - 1; i > j; --i) {
            const int d = rev ? h.N[i - 1] : h.S[i - 1], hi = y / d, lo = y - hi * d;
            first = first && (rev ? hi : lo) == 0;
            y = rev ? lo : hi;
        }
        const int d = rev ? h.N[j - 1] : h.S[j - 1], s = rev ? y / d : y % d;
        const int c = t & 63, part = t >> 6;
        float acc = 0.f;
        if (c < h.r[j]) {
            const float dc = rev ? 1.f : l.D[j - 1][c];
#pragma unroll 8
            for (int cp = part; cp < h.r[j - 1]; cp += 4)
                acc += v[cp] * core_at(l, j, cp, s, c) * (rev ? l.D[j - 1][cp] : dc);
        }
        red[part][c] = acc;
        __syncthreads();
        if (t < 64) {
            const float y4 = ((red[0][t] + red[1][t]) + red[2][t]) + red[3][t];
            v[t] = y4;
            if (first && t < h.rp[j]) h.V[j][int64_t(y) * h.rp[j] + t] = y4;
        }
        __syncthreads();
    }
    const int RP = h.rp[q], S = h.S[q - 1], R = h.r[q], K = h.r[q - 1];
    if (rev && t < K) v[t] *= l.D[q - 1][t];
    __syncthreads();
    T *op = reinterpret_cast<T *>(h.op), *opt = reinterpret_cast<T *>(h.opt);
    for (int o = t; o < S * RP; o += 256) {
        const int c = o % RP, s = o / RP;
        float acc = 0.f;
        if (c < R) {
#pragma unroll 16
            for (int cp = 0; cp < K; ++cp) acc += v[cp] * core_at(l, q, cp, s, c);
            if (!rev) acc *= l.D[q - 1][c];
        }
        const int64_t row = chain_index(h, q, xq, s);
        put(op + row * RP + c, acc);
        put(opt + (row / KE * RP + c) * KE + row % KE, acc);
    }
}

// Core gradients of both groups in one launch from E_q: workgroup (position
// j, mode index s) recomputes the environments E_{q-1} .. E_j it needs (only
// the rows with digit s at position j) and contracts the last of them with
// V_{j-1}, so that no partial sums are left: it writes dG of its mode index
// with the masks applied and zeros on inactive slices, and the compacted
// masked-core gradient where the mask gradients want it.  fp32 on 16 x 16 x 4
// MFMA tiles, the eight waves sharing K (summed in wave order).  Bound by
// latency (each workgroup reads at most a few hundred kilobytes from L2).
constexpr int kGradWaves = 8, kGradThreads = 64 * kGradWaves;
constexpr int kGradBuf = 8192;   // floats of one environment buffer (rows x padded rank)
__global__ __launch_bounds__(kGradThreads) void tt_grad_kernel(ChainsArgs a) {
    __shared__ __attribute__((aligned(16))) float env[2][kGradBuf];
    __shared__ __attribute__((aligned(16))) float red[kGradWaves][4][256];
    __shared__ float res[64 * 65];
    __shared__ int tab[kGradBuf / 16];
    __shared__ int16_t inv[2][256];
    __shared__ ChainLds lds;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, lr = lane & 15, lg = lane >> 4;
    int p = 0;
    const int np = a.ch[0].q + a.ch[1].q;
    while (p + 1 < np && int(blockIdx.x) >= a.gblk[p + 1]) ++p;
    const int q0 = a.ch[0].q, g = p >= q0 ? 1 : 0;
    const int j = p - (g ? q0 : 0) + 1, s = int(blockIdx.x) - a.gblk[p];
    load_chain<kGradThreads>(lds, a, g, t);
    const Chain &h = lds.h;
    const int q = h.q;
    const int RP = h.rp[q], Sj = h.S[j - 1];
    // full -> compacted entry of the core's bonds
    inv[t >> 8][t & 255] = -1;
    __syncthreads();
    const int kb = h.bl[j - 1];
    const int rcl = h.rev ? h.r[j] : h.r[j - 1], rcr = h.rev ? h.r[j - 1] : h.r[j];
    if (t < rcl) inv[0][lds.map[kb][t]] = int16_t(t);
    if (t < rcr) inv[1][lds.map[kb + 1][t]] = int16_t(t);
    // rows of E_{q-1} with digit s at position j: local row u has the digits
    // j + 1 .. q - 1 in its low part (position q - 1 least significant)
    if (j < q) {
        const int n = h.N[q - 1] / Sj;
        for (int u = t; u < n; u += kGradThreads) {
            int mul = 1;
            for (int i = j + 1; i < q; ++i) mul *= h.S[i - 1];
            int low = u % mul, x = chain_index(h, j, u / mul, s);
            for (int i = j + 1; i < q; ++i) {
                mul /= h.S[i - 1];
                x = chain_index(h, i, x, low / mul);
                low %= mul;
            }
            tab[u] = x;
        }
    }
    __syncthreads();
    auto wave_sum = [&](int i, int e) {
        float y = red[0][i][e];
#pragma unroll
        for (int w = 1; w < kGradWaves; ++w) y += red[w][i][e];
        return y;
    };
    int cur = 0;
    int n = h.N[q - 1] / Sj;   // rows at level l
    for (int l = q - 1; l >= j; --l) {
        const bool top = l == q - 1;
        const int Sn = h.S[l], rpn = h.rp[l + 1], rpl = h.rp[l], K = Sn * rpn, nb = rpl / 16;
        const float *src = env[cur ^ 1];
        float *dst = env[cur];
        const float *Cn = h.C[l + 1];
        for (int m0 = 0; m0 < n; m0 += 16) {
            const int u = min(m0 + lr, n - 1);
            const int x = top ? tab[u] : 0;
            f32x4 acc[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
            for (int k = 16 * wave; k < K; k += 16 * kGradWaves) {
                const int sn = k / rpn, c = k - sn * rpn + 4 * lg;
                const f32x4 ev = top ? *reinterpret_cast<const f32x4 *>(h.E + int64_t(chain_index(h, l + 1, x, sn)) * RP + c)
                                     : *reinterpret_cast<const f32x4 *>(src + (u * Sn + sn) * rpn + c);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if (i < nb) {
                        const f32x4 cv = *reinterpret_cast<const f32x4 *>(Cn + int64_t(min(16 * i + lr, h.r[l] - 1)) * K + k + 4 * lg);
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(ev[e], cv[e], acc[i], 0, 0, 0);
                    }
                }
            }
            __syncthreads();   // the previous block's sums have been read
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (i < nb)
#pragma unroll
                    for (int v = 0; v < 4; ++v) red[wave][i][(4 * lg + v) * 16 + lr] = acc[i][v];
            __syncthreads();
            for (int o = t; o < nb * 256; o += kGradThreads) {
                const int i = o >> 8, row = m0 + ((o >> 4) & 15), c = 16 * i + (o & 15);
                if (row < n) dst[row * rpl + c] = c < h.r[l] ? wave_sum(i, o & 255) : 0.f;
            }
        }
        __syncthreads();
        cur ^= 1;
        if (l > j) n /= h.S[l - 1];
    }
    const float *Ej = env[cur ^ 1];   // E_j rows (x, s) in x order when j < q
    const int rj = h.r[j], rpj = h.rp[j];
    if (j == 1) {
        for (int c = t; c < rj; c += kGradThreads) res[c] = q == 1 ? h.E[int64_t(s) * RP + c] : Ej[c];
        __syncthreads();
    } else {
        const int nx = h.N[j - 1], rpp = h.rp[j - 1], mb = rpp / 16, nb = rpj / 16;
        const float *V = h.V[j - 1];
        f32x4 acc[4][4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[i][c] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
        for (int x0 = 4 * wave; x0 < nx; x0 += 4 * kGradWaves) {
            const int x = x0 + lg;
            const bool in = x < nx;
            const float *vr = V + (in ? x : 0) * rpp + lr;
            const float *er = (j == q ? h.E + int64_t(in ? chain_index(h, q, x, s) : 0) * RP : Ej + (in ? x : 0) * rpj) + lr;
            float vv[4], ev[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                vv[i] = i < mb && in ? vr[16 * i] : 0.f;
                ev[i] = i < nb && in ? er[16 * i] : 0.f;
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (i < mb)
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        if (c < nb) acc[i][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(vv[i], ev[c], acc[i][c], 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (i >= mb) break;
            __syncthreads();   // the previous block's sums have been read
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (c < nb)
#pragma unroll
                    for (int v = 0; v < 4; ++v) red[wave][c][(4 * lg + v) * 16 + lr] = acc[i][c][v];
            __syncthreads();
            for (int o = t; o < nb * 256; o += kGradThreads)
                res[(16 * i + ((o >> 4) & 15)) * 65 + 16 * (o >> 8) + (o & 15)] = wave_sum(o >> 8, o & 255);
        }
        __syncthreads();
    }
    // full core entries (l, s, r): res[chain-prev][chain]
    const int fl = h.fl[j - 1], fr = h.fr[j - 1];
    float *dG = h.dG[j - 1], *keep = h.keep[j - 1];
    const float *D = h.D[j - 1];
    for (int o = t; o < fl * fr; o += kGradThreads) {
        const int l = o / fr, r = o - l * fr, cl = inv[0][l], cr = inv[1][r];
        float y = 0.f;
        if (cl >= 0 && cr >= 0) {
            y = h.rev ? res[cr * 65 + cl] : res[cl * 65 + cr];
            if (keep) keep[(int64_t(cl) * Sj + s) * rcr + cr] = y;
        }
        if (dG) dG[(int64_t(l) * Sj + s) * fr + r] = (D && cl >= 0 && cr >= 0) ? y * D[r] : y;
    }
}

inline size_t align_up(size_t x) { return (x + 255) / 256 * 256; }
inline char *at(void *ws, size_t off) { return reinterpret_cast<char *>(ws) + off; }
inline bool al16(const void *p) { return reinterpret_cast<uintptr_t>(p) % 16 == 0; }

// chain position i (0-based) of group g as core index
int core_of(const SweepLayout &L, int g, int i) { return g == 0 ? L.s[0] + i : L.e[1] - i; }

// chains of both groups with workspace pointers; G, D, dG and dD may be null
void fill_chains(const comera_ttm_plan_s *p, const float *const *G, const float *const *D, float *const *dG,
                 float *const *dD, void *ws, ChainsArgs &a) {
    const SweepLayout &L = p->sweep;
    const BottleneckLayout &B = L.bn;
    std::memset(&a, 0, sizeof(a));
    for (int k = 0; k <= p->d; ++k) {
        const bool inner = k > 0 && k < p->d;
        int n = 0;
        if (p->compacted && inner) {
            for (int x = 0; x < 256 && n < 64; ++x)
                if ((p->act[k].w[x >> 6] >> (x & 63)) & 1) a.map[k][n++] = uint8_t(x);
        } else {
            for (; n < 64; ++n) a.map[k][n] = uint8_t(n);
        }
    }
    int blk = 0;
    for (int g = 0; g < 2; ++g) {
        Chain &h = a.ch[g];
        h.q = L.e[g] - L.s[g] + 1;
        h.rev = g;
        h.N[0] = 1;
        h.r[0] = 1;
        h.rp[0] = 16;
        for (int i = 0; i < h.q; ++i) {
            const int k = core_of(L, g, i);
            h.G[i] = G ? G[k] : nullptr;
            h.D[i] = D && k < p->d - 1 ? D[k] : nullptr;
            h.dG[i] = dG ? dG[k] : nullptr;
            h.keep[i] = dD && k < p->d - 1 && dD[k] ? reinterpret_cast<float *>(at(ws, B.keep[k])) : nullptr;
            h.S[i] = int(g == 0 ? p->s.n[k] : p->s.m[k]);
            h.N[i + 1] = h.N[i] * h.S[i];
            h.r[i + 1] = int(g == 0 ? p->rho[k + 1] : p->rho[k]);
            h.rp[i + 1] = i + 1 == h.q ? B.RP : (h.r[i + 1] + 15) / 16 * 16;
            h.fl[i] = int(p->s.r[k]);
            h.fr[i] = int(p->s.r[k + 1]);
            h.bl[i] = k;
            if (i + 1 < h.q) h.V[i + 1] = reinterpret_cast<float *>(at(ws, B.v[g][i + 1]));
            if (i > 0) h.C[i + 1] = reinterpret_cast<float *>(at(ws, B.c[g][i + 1]));
        }
        h.E = reinterpret_cast<const float *>(at(ws, B.sum)) + (g ? p->N_in * B.RP : 0);
        h.op = at(ws, B.op[g]);
        h.opt = at(ws, B.opt[g]);
        blk += h.N[h.q - 1];
        a.blk[g] = blk;
    }
    a.blk[2] = a.blk[1] + 64;
    int n = 0, np = 0;
    for (int g = 0; g < 2; ++g)
        for (int i = 0; i < a.ch[g].q; ++i) {
            a.gblk[np++] = n;
            n += a.ch[g].dG[i] || a.ch[g].keep[i] ? a.ch[g].S[i] : 0;
        }
    for (; np <= 2 * kMaxCores; ++np) a.gblk[np] = n;
}

template <typename T>
int go_pass(const PassArgs &a, int RP, void *stream) {
    auto go = [&](auto kern, int MT) {
        const dim3 grid(unsigned((a.b + 16 * MT - 1) / (16 * MT)));
        COMERA_LAUNCH_NAMED("tt_pass_kernel", kern, grid, dim3(64 * kPassWaves), 0, hipStream_t(stream), a);
        return launch_status();
    };
    // the largest tile that leaves no CU without a workgroup (a step of 768 ->
    // 3072 by tokens a tile, 16 / 32 / 64: r30 fp32 8192 tokens 152 / 141 / 192
    // us, 16384 tokens 274 / 249 / 243, 65536 tokens 939 / 858 / 800; r48 bf16
    // 4096 tokens 100 / 104 / 115, 8192 tokens 130 / 113 / 123).  That is so
    // also for fp32's 64-token tile, whose 81 KiB of LDS leave one workgroup to a
    // CU (bf16 77 KiB: two).  A 64-wide state stops at 32 tokens.
    const int64_t blocks = (a.b + 15) / 16;
    if (RP == 32) {
        if (blocks >= 4 * 256) return go(tt_pass_kernel<T, 32, 4>, 4);
        if (blocks >= 2 * 256) return go(tt_pass_kernel<T, 32, 2>, 2);
        return go(tt_pass_kernel<T, 32, 1>, 1);
    }
    if (blocks >= 2 * 256) return go(tt_pass_kernel<T, 64, 2>, 2);
    return go(tt_pass_kernel<T, 64, 1>, 1);
}

int pass(const comera_ttm_plan_s *p, int64_t b, const void *in, int64_t K, size_t op1, size_t op2, void *out,
         int64_t N, size_t state, void *ws, void *stream) {
    const BottleneckLayout &B = p->sweep.bn;
    PassArgs a;
    a.in = in;
    a.op1 = at(ws, op1);
    a.op2 = at(ws, op2);
    a.out = out;
    a.state = at(ws, state);
    a.K = K;
    a.N = N;
    a.b = b;
    a.spitch = B.spitch;
    a.R = B.R;
    a.vec_in = al16(in);
    a.vec_out = al16(out);
    return p->s.act == COMERA_BF16 ? go_pass<uint16_t>(a, B.RP, stream) : go_pass<float>(a, B.RP, stream);
}

int build(const comera_ttm_plan_s *p, const float *const *G, const float *const *D, void *ws, void *stream) {
    ChainsArgs a;
    fill_chains(p, G, D, nullptr, nullptr, ws, a);
    const dim3 grid(static_cast<unsigned>(a.blk[2]));
    if (p->s.act == COMERA_BF16)
        COMERA_LAUNCH_NAMED("tt_build_kernel", tt_build_kernel<uint16_t>, grid, dim3(256), 0, hipStream_t(stream), a);
    else
        COMERA_LAUNCH_NAMED("tt_build_kernel", tt_build_kernel<float>, grid, dim3(256), 0, hipStream_t(stream), a);
    return launch_status();
}

// columns of one workgroup of the meets
int meet_strip(int act, int RP) { return kMeetWaves * (act == COMERA_BF16 ? (RP == 32 ? meet_cw<32>() : meet_cw<64>()) : 64); }

int meet(const comera_ttm_plan_s *p, int64_t b, const void *X, const void *dY, void *ws, int &splits, void *stream) {
    const BottleneckLayout &B = p->sweep.bn;
    const int sw = meet_strip(p->s.act, B.RP);
    MeetArgs a;
    a.V[0] = X;
    a.V[1] = dY;
    a.S[0] = at(ws, B.t);
    a.S[1] = at(ws, B.s);
    a.C[0] = p->N_in;
    a.C[1] = p->N_out;
    a.strips0 = int((p->N_in + sw - 1) / sw);
    a.b = b;
    a.spitch = B.spitch;
    a.R = B.R;
    a.kchunk = B.kchunk;
    splits = int((b + B.kchunk - 1) / B.kchunk);
    a.split_stride = (p->N_in + p->N_out) * B.RP;
    // a single split needs no sum
    a.part = reinterpret_cast<float *>(at(ws, splits > 1 ? B.part : B.sum));
    a.vec[0] = al16(X);
    a.vec[1] = al16(dY);
    const dim3 grid(unsigned(a.strips0 + (p->N_out + sw - 1) / sw), unsigned(splits));
    auto go = [&](auto kern) {
        COMERA_LAUNCH_NAMED("tt_meet_kernel", kern, grid, dim3(64 * kMeetWaves), 0, hipStream_t(stream), a);
        return launch_status();
    };
    if (p->s.act == COMERA_BF16) return B.RP == 32 ? go(tt_meet_bf16_kernel<32>) : go(tt_meet_bf16_kernel<64>);
    return B.RP == 32 ? go(tt_meet_f32_kernel<32>) : go(tt_meet_f32_kernel<64>);
}

comera_status status_of(int e) { return e ? COMERA_ERR_HIP : COMERA_OK; }

// Where these kernels beat the general sweep (times of a training step there
// and here):
// - Batch-free work: a workgroup of the build forms the last mode's S x RP
//   entries with 256 threads, each a sum over the K entries of the bond
//   before it, loaded 16 at a time; up to 16 such rounds one after another
//   (modes of 16 at rank 64, of 64 at rank 32) stay below the general build's
//   launches.  64 and 48 modes at rank 64, 48 rounds, bf16, 4096 tokens: 136
//   against 189 us; 1024 modes at rank 32, 256 tokens: 110 against 507 us;
//   16 rounds (64 and 64 modes at rank 32, 4096 tokens): 171 against 125 us.
// - fp32 at a padded rank of 64 is bound by the matrix units, which the
//   GEMM's larger tiles use better once there are tokens enough to fill the
//   chip with them: 768 -> 3072 r48 at 16384 tokens 502 against 451 us, at
//   32768 tokens 732 against 808 us.  Over a few tokens one workgroup's pass
//   is as long as over 16: 3840 -> 64 r64, 4 tokens, 130 against 151 us; 1024
//   -> 4096 r48, 100 tokens, level.
// - A pass gives 16 to 64 whole rows to one workgroup.  Over few tokens a few
//   CUs then walk wide rows that the GEMM splits (1536 -> 12288 r32 fp32, 10
//   tokens: 151 against 177 us), and fp32 rows or states of two padded groups
//   fall behind the GEMM's stores at any batch (384 -> 6144 r32 fp32, 19460
//   tokens: level; 128 -> 15360 r1, 17169 tokens: 989 against 1223 us; 5120 ->
//   10240 r64 bf16, 675 tokens: 174 against 255 us).  Rows of up to 4096 are
//   faster here in every form (1024 -> 4096 r64 fp32, 8192 tokens: 366 against
//   341 us); bf16 at a padded rank of 32 from 512 tokens on at every width
//   (768 -> 8000 r24, 6252 tokens: 197 against 133 us; 32768 -> 32768 r32,
//   4096 tokens: 827 against 658 us).
bool faster_here(const comera_ttm_plan_s *p, const SweepLayout &L, int RP) {
    for (int g = 0; g < 2; ++g) {
        const int q = L.e[g] - L.s[g] + 1, k = core_of(L, g, q - 1);
        const int64_t S = g == 0 ? p->s.n[k] : p->s.m[k];
        const int64_t K = q == 1 ? 1 : (g == 0 ? p->rho[k] : p->rho[k + 1]);
        if ((S * RP + 255) / 256 * ((K + 15) / 16) > 16) return false;
    }
    const int64_t esz = p->s.act == COMERA_BF16 ? 2 : 4;
    if (esz == 4 && RP == 64 && (p->batch < 64 || p->batch > 16384)) return false;
    return std::max(p->N_in, p->N_out) <= 4096 || (esz == 2 && RP == 32 && p->batch >= 512);
}

}  // namespace

bool layout_bottleneck(const comera_ttm_plan_s *p, const SweepLayout &L, size_t cap, BottleneckLayout &B) {
    B = BottleneckLayout();
    if (L.G != 2 || L.dir != COMERA_ORDER_SWEEP_LR || L.M[0] != 1 || L.N[1] != 1) return false;
    const int64_t esz = p->s.act == COMERA_BF16 ? 2 : 4;
    // rows of whole 16-byte chunks
    if (p->N_in * esz % 16 || p->N_out * esz % 16) return false;
    for (int k = 1; k < p->d; ++k)
        if (p->rho[k] > 64) return false;
    B.R = int(L.ae[0]);
    B.RP = B.R <= 32 ? 32 : 64;
    const int64_t b = std::max<int64_t>(p->batch, 1);
    B.spitch = (b + 63) / 64 * 64;
    if (!faster_here(p, L, B.RP)) return false;
    double off = 0;
    auto region = [&](double bytes) {
        const size_t o = size_t(off);
        off += double(align_up(size_t(std::min(bytes, 1e15))));
        return o;
    };
    for (int g = 0; g < 2; ++g) {
        const int q = L.e[g] - L.s[g] + 1;
        int64_t n = 1;
        for (int i = 0; i < q; ++i) {
            const int k = core_of(L, g, i);
            const int64_t S = g == 0 ? p->s.n[k] : p->s.m[k];
            const int64_t rprev = i == 0 ? 1 : (g == 0 ? p->rho[k] : p->rho[k + 1]);
            const int64_t r = g == 0 ? p->rho[k + 1] : p->rho[k], rp = i + 1 == q ? B.RP : (r + 15) / 16 * 16;
            // the folded core, at its padded rank, is indexed with 32 bits (the
            // plan bounds the unpadded core only)
            if (i > 0 && double(rprev) * double(S) * double(rp) >= 2147483648.0) return false;
            if (i > 0) B.c[g][i + 1] = region(4.0 * double(rprev * S * rp));
            n *= S;
            if (n * 64 > (int64_t(1) << 30)) return false;
            if (i + 1 < q) B.v[g][i + 1] = region(4.0 * double(n * rp));
        }
        // environment rows of a core gradient's workgroup: all rows of the
        // level above its core that share its mode index
        const int kq = core_of(L, g, q - 1);
        const int64_t nq = n / (g == 0 ? p->s.n[kq] : p->s.m[kq]);
        for (int i = 0; i + 1 < q; ++i) {
            const int k = core_of(L, g, i);
            const int64_t S = g == 0 ? p->s.n[k] : p->s.m[k];
            if (nq / S * 64 > kGradBuf) return false;
        }
        if (nq > (1 << 20)) return false;
        const int64_t ke = 64 / esz;
        B.op[g] = region(double(esz) * double(n * B.RP));
        B.opt[g] = region(double(esz) * double((n + ke - 1) / ke * ke * B.RP));
    }
    const double state = double(esz) * double(B.RP) * double(B.spitch);
    B.s = region(state);
    B.t = region(state);
    // token splits of the meets: two workgroups per CU (one at small batches,
    // where the partials would weigh as much as the activations), each over
    // at least 64 tokens
    const int sw = meet_strip(p->s.act, B.RP);
    const int64_t strips = (p->N_in + sw - 1) / sw + (p->N_out + sw - 1) / sw;
    const int64_t want = std::max<int64_t>(1, (b >= 16384 ? 512 : 256) / strips);
    B.kchunk = std::max<int64_t>(64, ((b + want - 1) / want + 31) / 32 * 32);
    const int64_t splits = (b + B.kchunk - 1) / B.kchunk;
    if (splits > 65535) return false;
    const double grads = 4.0 * double(p->N_in + p->N_out) * double(B.RP);
    B.part = region(splits > 1 ? grads * double(splits) : 0.0);
    B.sum = region(grads);
    for (int k = 0; k + 1 < p->d; ++k)
        B.keep[k] = region(4.0 * double(p->rho[k]) * double(p->s.m[k] * p->s.n[k]) * double(p->rho[k + 1]));
    if (off > double(cap)) return false;
    B.total = size_t(off);
    B.on = true;
    return true;
}

comera_status bottleneck_forward(const comera_ttm_plan_s *p, int64_t b, const void *X, const float *const *G,
                                 const float *const *D, void *Y, void *ws, void *stream) {
    const BottleneckLayout &B = p->sweep.bn;
    if (int e = build(p, G, D, ws, stream)) return status_of(note_hip(e, "group build"));
    void *ev;
    timing_begin(const_cast<comera_ttm_plan_s *>(p), COMERA_KERNEL_FWD, stream, &ev);
    const int e = note_hip(pass(p, b, X, p->N_in, B.opt[0], B.op[1], Y, p->N_out, B.s, ws, stream), "forward pass");
    timing_end(const_cast<comera_ttm_plan_s *>(p), COMERA_KERNEL_FWD, stream, ev);
    return status_of(e);
}

comera_status bottleneck_backward(const comera_ttm_plan_s *p, int64_t b, const void *X, const void *dY,
                                  const float *const *G, const float *const *D, void *dX, float *const *dG,
                                  float *const *dD, void *ws, void *stream) {
    const BottleneckLayout &B = p->sweep.bn;
    bool want = false;
    for (int k = 0; k < p->d; ++k) want = want || (dG && dG[k]) || (dD && k + 1 < p->d && dD[k]);
    if (!want && !dX) return COMERA_OK;
    if (!p->reuse) {
        if (int e = build(p, G, D, ws, stream)) return status_of(note_hip(e, "group build"));
        if (want)
            if (int e = pass(p, b, X, p->N_in, B.opt[0], B.op[1], nullptr, p->N_out, B.s, ws, stream))
                return status_of(note_hip(e, "activation state"));
    }
    void *ev;
    timing_begin(const_cast<comera_ttm_plan_s *>(p), COMERA_KERNEL_DX, stream, &ev);
    int e = note_hip(pass(p, b, dY, p->N_out, B.opt[1], B.op[0], dX, p->N_in, B.t, ws, stream), "dX pass");
    timing_end(const_cast<comera_ttm_plan_s *>(p), COMERA_KERNEL_DX, stream, ev);
    if (e || !want) return status_of(e);
    timing_begin(const_cast<comera_ttm_plan_s *>(p), COMERA_KERNEL_DW, stream, &ev);
    int splits = 1;
    e = note_hip(meet(p, b, X, dY, ws, splits, stream), "meets");
    if (!e && splits > 1)
        e = note_hip(launch_sum_splits(reinterpret_cast<const float *>(at(ws, B.part)),
                                       reinterpret_cast<float *>(at(ws, B.sum)), (p->N_in + p->N_out) * B.RP, splits,
                                       stream),
                     "split sum");
    ChainsArgs a;
    fill_chains(p, G, D, dG, dD, ws, a);
    if (!e) {
        const dim3 grid(static_cast<unsigned>(a.gblk[2 * kMaxCores]));
        COMERA_LAUNCH(tt_grad_kernel, grid, dim3(kGradThreads), 0, hipStream_t(stream), a);
        e = note_hip(launch_status(), "core gradients");
    }
    timing_end(const_cast<comera_ttm_plan_s *>(p), COMERA_KERNEL_DW, stream, ev);
    if (e || !dD) return status_of(e);
    MaskGradArgs ma;
    std::memset(&ma, 0, sizeof(ma));
    ma.d = p->d;
    ma.compacted = p->compacted ? 1 : 0;
    for (int k = 0; k < p->d; ++k) {
        ma.dD[k] = k + 1 < p->d ? dD[k] : nullptr;
        ma.sum[k] = k + 1 < p->d ? reinterpret_cast<const float *>(at(ws, B.keep[k])) : nullptr;
        ma.G[k] = G[k];
        ma.m[k] = int(p->s.m[k]);
        ma.n[k] = int(p->s.n[k]);
        ma.st[k] = core_strides(int(p->rho[k]), ma.m[k], ma.n[k], int(p->rho[k + 1]), false);
    }
    for (int k = 0; k <= p->d; ++k) {
        ma.r[k] = int(p->s.r[k]);
        ma.rc[k] = int(p->rho[k]);
        ma.act[k] = p->act[k];
    }
    return status_of(note_hip(launch_mask_grad(ma, stream), "mask gradients"));
}

}  // namespace comera
