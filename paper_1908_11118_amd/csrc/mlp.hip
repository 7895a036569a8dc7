// mlp.hip -- the learned insertion proposal network on the GPU: forward, backward,
// Adam and the training loop, bfloat16 operands on MFMA with FP32 accumulation.
//
// Network (an extension of the REGC method, not in the paper): the 16^3 occupancy
// grid of a configuration -> 128 -> 128 -> 128 -> 4096 logits over insertion
// voxels; GELU (erf form) after each hidden layer.  Layer 1 is a gather: the
// occupancy has at most n_max non-zero voxels, so its product with W1 is the sum
// of the W1 columns of the occupied voxels (one per particle, in particle order).
// Layers 2-4 and the weight/activation gradients are MFMA GEMMs
// (v_mfma_f32_16x16x16_bf16: lane l holds A row l%16 and B column l%16 at
// k = 4*(l/16)..+3; the result element D[4*(l/16)+r][l%16] sits in register r).
// Rounding points: weights and hidden activations are rounded to bfloat16
// (nearest even) before each product; pre-activations, logits, softmax, the
// gradient sums and the Adam state are FP32.
//
// Training example: a stored configuration, one particle i of it; input = the
// occupancy without i, target = the voxel of i; loss = cross-entropy.
// Parameter vector layout (FP32, also the ABI's): W1 [4096][128] (voxel-major),
// b1 [128], W2 [128][128] ([out][in]), b2, W3, b3, W4 [4096][128] ([voxel][in]), b4 [4096].
#include <algorithm>
#include <cmath>
#include <utility>
#include <vector>

#include "host_util.h"
#include "mlp_dev.h"
#include "philox_dev.h"
#include "learn_dev.h"

namespace regc {
namespace mlpk {

constexpr int NV = 4096, H = 128;
constexpr int kSplitK = 16;   // K = 4096 products split 16 ways
constexpr size_t OFF_W1 = 0, OFF_B1 = OFF_W1 + (size_t)NV * H, OFF_W2 = OFF_B1 + H, OFF_B2 = OFF_W2 + (size_t)H * H,
                 OFF_W3 = OFF_B2 + H, OFF_B3 = OFF_W3 + (size_t)H * H, OFF_W4 = OFF_B3 + H,
                 OFF_B4 = OFF_W4 + (size_t)NV * H, NPARAM = OFF_B4 + NV;

// ---- the training step ----
// Six launches: hidden_forward (the batch, layers 1-3), logits_forward, softmax_xent,
// output_backward, hidden_backward, finish (the small weight gradients, W1's gradient,
// Adam).  The step's operands fit the caches and its 0.5 GFLOP take microseconds, so what
// bounds it is launches and the dependent loads inside each: the parts that don't depend on
// each other share a launch (a block's role follows from its index) and a wave has all
// operands of 64 k in flight.  As 24 launches that was 220 us a step at a batch of 256
// (column sums with a load at a time 4 x 16, products with 2-byte operand loads 7 - 8 each, W1's
// gradient by 1.3e6 atomics 13); now 46.
constexpr int kRows = 4;           // examples per block of the hidden layers
constexpr int kPad = H + 8;        // LDS row of bfloat16 activations (16-byte aligned, off the banks' period)

struct Batch {
    int B, nmax;
    uint16_t *vox;                 // [B][nmax]
    int32_t *n, *excl, *target;    // [B]
};

// The data set a batch is drawn from (vox null: the batch is there already).
struct Source {
    int64_t n_examples, step;
    const uint16_t *vox;
    const int32_t *n;
    uint32_t k0, k1;
};

struct Acts {
    float *a1, *a2, *a3;           // pre-activations [B][H]
    bf16 *h1, *h2, *h3;
    float *da1, *da2, *da3;        // their gradients
    bf16 *g2, *g3;                 // da2, da3 in bfloat16
};

// W1's gradient gathers: for every voxel the examples that occupy it.
struct Lists {
    uint32_t *count;               // [NV]
    uint32_t *first;               // [NV + 1]
    uint32_t *cursor;              // [NV]
    uint64_t *entry;               // [B nmax]: particle << 32 | example
};

// A block's 64 x 64 tile of sum_k A(m, k) B(k, n) for k in [k0, k0 + kn), kn a multiple of
// 64, 16 k per MFMA in order; a wave (of four) has 32 x 32 of it, wave / 2 down and
// wave % 2 across.  The operands come 64 k at a time through LDS as rows of 128 bytes, the next
// two's loads in flight meanwhile (they come from beyond the XCD's cache: another kernel wrote them).  KC: stored with k contiguous, a row per m (n), a lane reads
// its four k at once; else a row per k, a lane reads two neighbouring m of each k and the
// wave's two row blocks are the even and the odd m.
constexpr int kTile = 64, kTilePad = kTile + 8;
typedef bf16 Tile[kTile][kTilePad];
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

template <bool KC>
struct Operand {
    u32x4 lo, hi;                  // rows threadIdx / 8 and 32 below, 8 elements at 8 (threadIdx % 8)
    static __device__ __forceinline__ int index(int block, int r) { return KC ? 16 * block + r : 2 * r + block; }
    __device__ __forceinline__ void load(const bf16 *p, int ld, int m0, int k)
    {
        const int row = threadIdx.x / 8, c = threadIdx.x % 8 * 8;
        const bf16 *q = KC ? p + (size_t)(m0 + row) * ld + k + c : p + (size_t)(k + row) * ld + m0 + c;
        lo = *reinterpret_cast<const u32x4 *>(q);
        hi = *reinterpret_cast<const u32x4 *>(q + (size_t)32 * ld);
    }
    __device__ __forceinline__ void store(Tile &t) const
    {
        *reinterpret_cast<u32x4 *>(&t[threadIdx.x / 8][threadIdx.x % 8 * 8]) = lo;
        *reinterpret_cast<u32x4 *>(&t[threadIdx.x / 8 + 32][threadIdx.x % 8 * 8]) = hi;
    }
    // the fragments of rows (columns) w0 .. w0 + 31 at k .. k + 3
    static __device__ __forceinline__ void read(const Tile &t, int w0, int k, bf16x4 (&f)[2])
    {
        const int r = threadIdx.x % 16;
        if (KC) {
#pragma unroll
            for (int i = 0; i < 2; ++i) f[i] = *reinterpret_cast<const bf16x4 *>(&t[w0 + 16 * i + r][k]);
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t u = *reinterpret_cast<const uint32_t *>(&t[k + q][w0 + 2 * r]);
                f[0][q] = (short)(u & 0xffffu);
                f[1][q] = (short)(u >> 16);
            }
        }
    }
};

struct Stage { __attribute__((aligned(16))) Tile a, b; };
static_assert(sizeof(Stage) >= NV * sizeof(uint32_t), "a counter per voxel takes the products' place");

// A wave's 32 x 32 results: row block i, column block j in c<i><j>.
struct Acc {
    f32x4 c00, c01, c10, c11;
    template <int E> __device__ __forceinline__ float at() const      // element E of 16: (i, j, register)
    {
        return (E < 4 ? c00 : E < 8 ? c01 : E < 12 ? c10 : c11)[E % 4];
    }
};

template <bool AK, bool BK>
__device__ __forceinline__ Acc product(Stage &st, const bf16 *A, int lda, int m0, const bf16 *B, int ldb, int n0, int k0, int kn)
{
    const int wave = threadIdx.x / 64, lk = 4 * (threadIdx.x % 64 / 16);
    Acc acc = {};
    Operand<AK> a0, a1;
    Operand<BK> b0, b1;
    auto load = [&](Operand<AK> &a, Operand<BK> &b, int k) {
        if (k >= kn) return;
        a.load(A, lda, m0, k0 + k);
        b.load(B, ldb, n0, k0 + k);
    };
    auto stage = [&](const Operand<AK> &a, const Operand<BK> &b) {
        a.store(st.a);
        b.store(st.b);
        __syncthreads();
    };
    auto multiply = [&]() {
#pragma unroll
        for (int u = 0; u < kTile / 16; ++u) {
            bf16x4 fa[2], fb[2];
            Operand<AK>::read(st.a, wave / 2 * 32, 16 * u + lk, fa);
            Operand<BK>::read(st.b, wave % 2 * 32, 16 * u + lk, fb);
            acc.c00 = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(fa[0], fb[0], acc.c00, 0, 0, 0);
            acc.c01 = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(fa[0], fb[1], acc.c01, 0, 0, 0);
            acc.c10 = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(fa[1], fb[0], acc.c10, 0, 0, 0);
            acc.c11 = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(fa[1], fb[1], acc.c11, 0, 0, 0);
        }
    };
    load(a0, b0, 0);
    load(a1, b1, kTile);
    for (int k = 0; k < kn; k += 2 * kTile) {
        if (k > 0) __syncthreads();
        stage(a0, b0);
        load(a0, b0, k + 2 * kTile);
        multiply();
        if (k + kTile >= kn) break;
        __syncthreads();
        stage(a1, b1);
        load(a1, b1, k + 3 * kTile);
        multiply();
    }
    return acc;
}

// f(E, m, n) over a lane's 16 elements of the tile at (m0, n0)
template <bool AK, bool BK, typename F, int... E>
__device__ __forceinline__ void each_element(int m0, int n0, F f, std::integer_sequence<int, E...>)
{
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
    m0 += wave / 2 * 32;
    n0 += wave % 2 * 32;
    (f(std::integral_constant<int, E>{}, m0 + Operand<AK>::index(E / 8, 4 * (lane / 16) + E % 4),
       n0 + Operand<BK>::index(E / 4 % 2, lane % 16)), ...);
}

template <bool AK, bool BK, typename F>
__device__ __forceinline__ void each_element(int m0, int n0, F f)
{
    each_element<AK, BK>(m0, n0, f, std::make_integer_sequence<int, 16>{});
}

// 16 columns of a hidden layer for the block's four examples: x from LDS, the weights'
// fragments in registers.  Rows 4 e .. 4 e + 3 of the product are all example e, so that the
// lane's first element is (example lane / 16, column lane % 16): every lane has one.
__device__ __forceinline__ float layer(const bf16 (*x)[kPad], const bf16x4 (&w)[H / 16])
{
    const int lane = threadIdx.x % 64;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int u = 0; u < H / 16; ++u) {
        const bf16x4 a = *reinterpret_cast<const bf16x4 *>(&x[lane % 16 / 4][16 * u + 4 * (lane / 16)]);
        acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, w[u], acc, 0, 0, 0);
    }
    return acc[0];
}

// Layers 1-3 of four examples: layer 1 with two waves per example (a column per lane),
// layers 2 and 3 with 16 columns per wave.  Four examples, not the matrix unit's 16, because
// the gather's loads bound the block: with 16 on a sixteenth of the CUs it took 15 us for
// 256 examples, now 12.
//
// A batch from a data set (src.vox): example e = (53-bit word) mod n_examples and left-out
// particle i = floor(U' * N_e) from Philox counter (slot, step, 0xFFFFFFFF, 5) with the
// given key.  Empty configurations are passed over for the next ones (at most 256); a
// slot left without particles gets target -1 (no loss, no gradient).
//
// Layer 1: a1[b] = b1 + sum of W1 columns of the occupied voxels (particles j != excl[b]),
// in particle order, 32 particles' loads in flight.
__global__ void __launch_bounds__(128 * kRows) hidden_forward(Batch bt, Source src, const bf16 *p16, const float *p, Acts ac,
                                                           uint32_t *count)
{
    __shared__ bf16 x[2][kRows][kPad];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64;
    const int b = blockIdx.x * kRows + wave / 2;
    // the first 64 voxels are loaded along with N
    const uint16_t *vox = bt.vox + (size_t)b * bt.nmax;
    int nb, ex, mine;
    if (src.vox) {
        const uint4 r = philox4x32_10(make_uint4((uint32_t)b, (uint32_t)src.step, 0xFFFFFFFFu, 5u), src.k0, src.k1);
        // (word mod n_examples: the quotient of 53-bit numbers in FP64 is off by one at most)
        const uint64_t word = (((uint64_t)r.x << 32) | r.y) >> 11, m = (uint64_t)src.n_examples;
        int64_t rest = (int64_t)(word - (uint64_t)((double)word / (double)m) * m);
        if (rest < 0) rest += (int64_t)m;
        else if (rest >= (int64_t)m) rest -= (int64_t)m;
        uint64_t pick = (uint64_t)rest;
        nb = src.n[pick];
        mine = lane < bt.nmax ? src.vox[pick * bt.nmax + lane] : 0;
        for (int tries = 0; nb == 0 && tries < 256; ++tries) {
            pick = pick + 1 == m ? 0 : pick + 1;
            nb = src.n[pick];
            mine = lane < bt.nmax ? src.vox[pick * bt.nmax + lane] : 0;
        }
        vox = src.vox + pick * bt.nmax;
        ex = nb > 0 ? (int)(((uint64_t)r.z * (uint64_t)nb) >> 32) : -1;
    } else {
        nb = bt.n[b];
        ex = bt.excl[b];
        mine = lane < bt.nmax ? vox[lane] : 0;
    }
    const int col = 16 * wave + lane % 16;              // of layers 2 and 3
    bf16x4 w2[H / 16], w3[H / 16];
#pragma unroll
    for (int u = 0; u < H / 16; ++u) {
        const size_t o = (size_t)col * H + 16 * u + 4 * (lane / 16);
        w2[u] = *reinterpret_cast<const bf16x4 *>(p16 + OFF_W2 + o);
        w3[u] = *reinterpret_cast<const bf16x4 *>(p16 + OFF_W3 + o);
    }
    if (count)
        for (int v = blockIdx.x * blockDim.x + threadIdx.x; v < NV; v += gridDim.x * blockDim.x) count[v] = 0u;
    nb = __builtin_amdgcn_readfirstlane(nb);
    ex = __builtin_amdgcn_readfirstlane(ex);
    const int c1 = 64 * (wave % 2) + lane;              // of layer 1
    const bf16 *W1 = p16 + OFF_W1 + c1;
    const bool keep = src.vox && wave % 2 == 0;
    const float bias2 = p[OFF_B2 + col], bias3 = p[OFF_B3 + col];
    float s = p[OFF_B1 + c1];
    for (int j0 = 0; j0 < bt.nmax; j0 += 64) {
        const int cnt = nb - j0 < 64 ? nb - j0 : 64;         // (<= 0 past the last)
        if (j0 > 0) mine = lane < cnt ? vox[j0 + lane] : 0;
        if (lane >= cnt) mine = 0;
        if (keep && j0 + lane < bt.nmax) bt.vox[(size_t)b * bt.nmax + j0 + lane] = (uint16_t)mine;
        if (keep && lane == ex - j0) bt.target[b] = mine;
        for (int j = 0; j < cnt; j += 32) {
            // (lanes past cnt hold voxel 0; selects, not branches: the loads stay together)
            bf16 u[32];
#pragma unroll
            for (int q = 0; q < 32; ++q) u[q] = W1[(size_t)__builtin_amdgcn_readlane(mine, j + q) * H];
#pragma unroll
            for (int q = 0; q < 32; ++q) {
                const float more = s + bf2f(u[q]);
                s = j + q < cnt && j0 + j + q != ex ? more : s;
            }
        }
    }
    if (keep && lane == 0) {
        bt.n[b] = nb;
        bt.excl[b] = ex;
        if (ex < 0) bt.target[b] = -1;
    }
    {
        const bf16 h = f2bf(gelu(s));
        ac.a1[(size_t)b * H + c1] = s;
        ac.h1[(size_t)b * H + c1] = h;
        x[0][wave / 2][c1] = h;
    }
    __syncthreads();
    const size_t o = (size_t)(blockIdx.x * kRows + lane / 16) * H + col;
    {
        const float v = layer(x[0], w2) + bias2;
        const bf16 h = f2bf(gelu(v));
        ac.a2[o] = v;
        ac.h2[o] = h;
        x[1][lane / 16][col] = h;
    }
    __syncthreads();
    const float v = layer(x[1], w3) + bias3;
    ac.a3[o] = v;
    ac.h3[o] = f2bf(gelu(v));
}

// The examples' entries of W1's gradient, one for every particle j != excl[b], of the part's
// share of the batch: four examples at a time (a wave each), up to 256 particles of each.  The
// block counts its entries of a voxel in LDS (`tally`, whose words are cleared by the entries
// that use them) and makes one addition to the voxel's counter in memory: an addition per entry takes
// its turn at the counter's cache line (512 examples of 150 particles in 16 voxels: 0.2 ms for
// each of the two kernels that do it).  claim(voxel, count): that addition, its result the
// voxel's first place; PLACE: then place(b, j, place) of every entry.
template <bool PLACE, typename C, typename F>
__device__ __forceinline__ void block_entries(const Batch &bt, int part, int parts, uint32_t *tally, C claim, F place)
{
    constexpr int kEach = 4;
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
    for (int b0 = part * 4; b0 < bt.B; b0 += parts * 4) {
        const int b = b0 + wave, nb = bt.n[b], ex = bt.excl[b];
        const int most = max(max(bt.n[b0], bt.n[b0 + 1]), max(bt.n[b0 + 2], bt.n[b0 + 3]));
        for (int j0 = 0; j0 < most; j0 += 64 * kEach) {
            int v[kEach];
            uint32_t old[kEach];
#pragma unroll
            for (int q = 0; q < kEach; ++q) {
                const int j = j0 + 64 * q + lane;
                v[q] = j < nb && j != ex ? (int)bt.vox[(size_t)b * bt.nmax + j] : -1;
            }
#pragma unroll
            for (int q = 0; q < kEach; ++q)
                if (v[q] >= 0) tally[v[q]] = 0u;
            __syncthreads();
#pragma unroll
            for (int q = 0; q < kEach; ++q)
                if (v[q] >= 0) old[q] = atomicAdd(tally + v[q], 1u);
            __syncthreads();
#pragma unroll
            for (int q = 0; q < kEach; ++q)
                if (v[q] >= 0 && old[q] == 0u) {
                    const uint32_t first = claim(v[q], tally[v[q]]);
                    if (PLACE) tally[v[q]] = first;
                }
            if (PLACE) {
                __syncthreads();
#pragma unroll
                for (int q = 0; q < kEach; ++q) {
                    const int j = j0 + 64 * q + lane;
                    if (v[q] >= 0) place(b, j - (j > ex), tally[v[q]] + old[q]);
                }
            }
            if (j0 + 64 * kEach < most || b0 + parts * 4 < bt.B) __syncthreads();     // the words are used again
        }
    }
}

// Blocks 0 .. (NV / 64) (B / 64) - 1: the logits, 64 x 64 each.  The others count the
// entries of every voxel.
__global__ void __launch_bounds__(256) logits_forward(Batch bt, const bf16 *p16, const float *p, const bf16 *h3,
                                                   float *logits, uint32_t *count)
{
    __shared__ Stage st;
    const int tiles = (NV / 64) * (bt.B / 64), tile = blockIdx.x;
    if (tile >= tiles) {
        block_entries<false>(bt, tile - tiles, gridDim.x - tiles, reinterpret_cast<uint32_t *>(&st),
                             [&](int v, uint32_t c) { atomicAdd(count + v, c); return 0u; }, [](int, int, uint32_t) {});
        return;
    }
    const int m0 = tile / (NV / 64) * 64, n0 = tile % (NV / 64) * 64;
    float bias[2];
    each_element<true, true>(m0, n0, [&](auto e, int, int n) { if (e < 8 && e % 4 == 0) bias[e / 4] = p[OFF_B4 + n]; });
    const Acc acc = product<true, true>(st, h3, H, m0, p16 + OFF_W4, H, n0, 0, H);
    each_element<true, true>(m0, n0, [&](auto e, int m, int n) { logits[(size_t)m * NV + n] = acc.at<e>() + bias[e / 4 % 2]; });
}

// Row-wise log-softmax cross-entropy: loss[b] = lse - logit[target]; the logit
// gradient d = (softmax - onehot) / B in FP32 and bfloat16.  A thread holds four logits; the
// sum runs over columns t, t + 256, ... by the first 256 threads, then over those.
// Block B: where each voxel's entries start.
constexpr int kSoftThreads = 1024;

__global__ void __launch_bounds__(kSoftThreads) softmax_xent(int B, const float *logits, const int32_t *target, float *loss,
                                                          float *d32, bf16 *d16, Lists ls)
{
    constexpr int kEach = NV / kSoftThreads;
    static_assert(kEach == 4, "four columns per thread");
    __shared__ __attribute__((aligned(16))) float ex[NV];
    __shared__ float sh[kSoftThreads / 64];
    const int b = blockIdx.x, tid = threadIdx.x, wave = tid / 64, lane = tid % 64;
    if (b == B) {
        uint32_t *sum = reinterpret_cast<uint32_t *>(sh);
        const uint4 c = *reinterpret_cast<const uint4 *>(ls.count + 4 * tid);
        const uint32_t mine = c.x + c.y + c.z + c.w;
        uint32_t at = mine;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t before = __shfl_up(at, o);
            if (lane >= o) at += before;
        }
        if (lane == 63) sum[wave] = at;
        __syncthreads();
        at -= mine;
        for (int w = 0; w < wave; ++w) at += sum[w];
        const uint4 f = make_uint4(at, at + c.x, at + c.x + c.y, at + c.x + c.y + c.z);
        *reinterpret_cast<uint4 *>(ls.first + 4 * tid) = f;
        *reinterpret_cast<uint4 *>(ls.cursor + 4 * tid) = f;
        if (tid == kSoftThreads - 1) ls.first[NV] = at + mine;
        return;
    }
    const float4 x = *reinterpret_cast<const float4 *>(logits + (size_t)b * NV + 4 * tid);
    const int t = target[b];          // < 0: no example in this slot (zero loss and gradient)
    const float xt = t >= 0 ? logits[(size_t)b * NV + t] : 0.f;
    float mx = fmaxf(fmaxf(x.x, x.y), fmaxf(x.z, x.w));
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
    if (lane == 0) sh[wave] = mx;
    __syncthreads();
    mx = sh[0];
    for (int w = 1; w < kSoftThreads / 64; ++w) mx = fmaxf(mx, sh[w]);
    *reinterpret_cast<float4 *>(ex + 4 * tid) = make_float4(expf(x.x - mx), expf(x.y - mx), expf(x.z - mx), expf(x.w - mx));
    __syncthreads();
    if (tid < 256) {
        float s = 0.f;
#pragma unroll
        for (int q = 0; q < NV / 256; ++q) s += ex[256 * q + tid];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
        if (lane == 0) sh[wave] = s;
    }
    __syncthreads();
    const float lse = mx + logf(((sh[0] + sh[1]) + sh[2]) + sh[3]);
    if (tid == 0) loss[b] = t >= 0 ? lse - xt : 0.0f;
    const float inv_b = t >= 0 ? 1.0f / (float)B : 0.0f;
    const int v = 4 * tid;
    const float4 g = make_float4((expf(x.x - lse) - (v == t ? 1.0f : 0.0f)) * inv_b,
                                 (expf(x.y - lse) - (v + 1 == t ? 1.0f : 0.0f)) * inv_b,
                                 (expf(x.z - lse) - (v + 2 == t ? 1.0f : 0.0f)) * inv_b,
                                 (expf(x.w - lse) - (v + 3 == t ? 1.0f : 0.0f)) * inv_b);
    *reinterpret_cast<float4 *>(d32 + (size_t)b * NV + v) = g;
    *reinterpret_cast<uint2 *>(d16 + (size_t)b * NV + v) = make_uint2((uint32_t)f2bf(g.x) | (uint32_t)f2bf(g.y) << 16,
                                                                      (uint32_t)f2bf(g.z) | (uint32_t)f2bf(g.w) << 16);
}

// out[n] = sum_m X[m][n] for 64 columns from col0 (256 threads): thread (g, c) sums rows
// g, g+4, ... of column c in order (M a multiple of 64: 16 rows' loads in flight), the four
// partial sums are added in the order g = 0..3 (deterministic).  Threads 0-63 hold it.
__device__ __forceinline__ float colsum64(int M, int N, const float *X, int col0)
{
    __shared__ float part[4][64];
    const int c = threadIdx.x % 64, g = threadIdx.x / 64;
    const float *col = X + (size_t)g * N + col0 + c;
    float s = 0.f;
    for (int m = 0; m < M; m += 64) {
        float x[16];
#pragma unroll
        for (int q = 0; q < 16; ++q) x[q] = col[(size_t)(m + 4 * q) * N];
#pragma unroll
        for (int q = 0; q < 16; ++q) s += x[q];
    }
    part[g][c] = s;
    __syncthreads();
    return ((part[0][c] + part[1][c]) + part[2][c]) + part[3][c];
}

// The output layer's gradients, by block: dh3 = d W4 as kSplitK partial products of 256 k
// each (part [kSplitK][B][H]), dW4 = d^T h3, db4 = column sums of d, and the lists of the
// voxels' examples.
constexpr int kDw4Blocks = (NV / 64) * (H / 64), kDb4Blocks = NV / 64;

__global__ void __launch_bounds__(256) output_backward(Batch bt, const bf16 *p16, const bf16 *h3, const float *d32,
                                                    const bf16 *d16, float *part, float *g, Lists ls)
{
    __shared__ Stage st;
    const int B = bt.B;
    int blk = blockIdx.x;
    const int dh = (B / 64) * (H / 64) * kSplitK;
    const int parts = gridDim.x - dh - kDw4Blocks - kDb4Blocks;
    if (blk < dh) {
        const int z = blk % kSplitK, tile = blk / kSplitK;
        const int m0 = tile / (H / 64) * 64, n0 = tile % (H / 64) * 64;
        const Acc acc = product<true, false>(st, d16, NV, m0, p16 + OFF_W4, H, n0, z * (NV / kSplitK), NV / kSplitK);
        float *out = part + (size_t)z * B * H;
        each_element<true, false>(m0, n0, [&](auto e, int m, int n) { out[(size_t)m * H + n] = acc.at<e>(); });
        return;
    }
    blk -= dh;
    if (blk < kDw4Blocks) {
        const int m0 = blk / (H / 64) * 64, n0 = blk % (H / 64) * 64;
        const Acc acc = product<false, false>(st, d16, NV, m0, h3, H, n0, 0, B);
        each_element<false, false>(m0, n0, [&](auto e, int m, int n) { g[OFF_W4 + (size_t)m * H + n] = acc.at<e>(); });
        return;
    }
    blk -= kDw4Blocks;
    if (blk < kDb4Blocks) {
        const float s = colsum64(B, NV, d32, 64 * blk);
        if (threadIdx.x < 64) g[OFF_B4 + 64 * blk + threadIdx.x] = s;
        return;
    }
    block_entries<true>(bt, blk - kDb4Blocks, parts, reinterpret_cast<uint32_t *>(&st),
                        [&](int v, uint32_t c) { return atomicAdd(ls.cursor + v, c); },
                        [&](int b, int j, uint32_t at) { ls.entry[at] = (uint64_t)j << 32 | (uint32_t)b; });
}

// Hidden layers 3, 2, 1 backwards for four examples: dh3 from the partial products (z in
// order), da = dh gelu'(a), dh of the layer below = da W.
__global__ void __launch_bounds__(128 * kRows) hidden_backward(int B, const bf16 *p16, const float *part, Acts ac)
{
    __shared__ bf16 x[2][kRows][kPad];
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64, col = 16 * wave + lane % 16;
    const size_t first = (size_t)blockIdx.x * kRows * H, i3 = first + threadIdx.x, o = first + (size_t)(lane / 16) * H + col;
    float s[kSplitK];
#pragma unroll
    for (int z = 0; z < kSplitK; ++z) s[z] = part[(size_t)z * B * H + i3];
    const float a3 = ac.a3[i3], a2 = ac.a2[o], a1 = ac.a1[o];
    bf16x4 w3[H / 16], w2[H / 16];
#pragma unroll
    for (int u = 0; u < H / 16; ++u)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const size_t k = (size_t)(16 * u + 4 * (lane / 16) + q) * H + col;
            w3[u][q] = (short)p16[OFF_W3 + k];
            w2[u][q] = (short)p16[OFF_W2 + k];
        }
#pragma unroll
    for (int z = 1; z < kSplitK; ++z) s[0] += s[z];
    const float d3 = s[0] * gelu_grad(a3);
    const bf16 q3 = f2bf(d3);
    ac.da3[i3] = d3;
    ac.g3[i3] = q3;
    x[0][threadIdx.x / H][threadIdx.x % H] = q3;
    __syncthreads();
    const float d2 = layer(x[0], w3) * gelu_grad(a2);
    const bf16 q2 = f2bf(d2);
    ac.da2[o] = d2;
    ac.g2[o] = q2;
    x[1][lane / 16][col] = q2;
    __syncthreads();
    ac.da1[o] = layer(x[1], w2) * gelu_grad(a1);
}

// Adam with bias correction (Kingma & Ba, ICLR 2015); writes the bfloat16 copy.
struct Adam {
    float *p, *m, *v;
    bf16 *p16;
    float lr, c1, c2, beta1, beta2, eps;
};

__device__ __forceinline__ void adam_one(const Adam &o, float gi, float &p, float &m, float &v)
{
    m = fmaf(1.f - o.beta1, gi, o.beta1 * m);
    v = fmaf(gi, (1.f - o.beta2) * gi, o.beta2 * v);
    p = p - o.lr * (m / o.c1) / (sqrtf(v / o.c2) + o.eps);
}

// One element: its gradient is kept (KEEP), and the parameter takes its step (UPDATE).
template <bool UPDATE, bool KEEP>
__device__ __forceinline__ void put(const Adam &o, float *g, size_t i, float gi)
{
    if (KEEP) g[i] = gi;
    if (UPDATE) {
        float p = o.p[i], m = o.m[i], v = o.v[i];
        adam_one(o, gi, p, m, v);
        o.p[i] = p; o.m[i] = m; o.v[i] = v;
        o.p16[i] = f2bf(p);
    }
}

// Two neighbouring parameters per lane.
struct AdamRow {
    float2 p, m, v;
    __device__ __forceinline__ void load(const Adam &o, size_t i)
    {
        p = *reinterpret_cast<const float2 *>(o.p + i);
        m = *reinterpret_cast<const float2 *>(o.m + i);
        v = *reinterpret_cast<const float2 *>(o.v + i);
    }
    __device__ __forceinline__ void step(const Adam &o, size_t i, float2 g)
    {
        adam_one(o, g.x, p.x, m.x, v.x);
        adam_one(o, g.y, p.y, m.y, v.y);
        *reinterpret_cast<float2 *>(o.p + i) = p;
        *reinterpret_cast<float2 *>(o.m + i) = m;
        *reinterpret_cast<float2 *>(o.v + i) = v;
        *reinterpret_cast<uint32_t *>(o.p16 + i) = (uint32_t)f2bf(p.x) | (uint32_t)f2bf(p.y) << 16;
    }
};

// What is left of the gradients, each element's Adam step with it (UPDATE), by block: dW3
// and dW2 (64 x 64 each); db3, db2, db1 (64 columns each); b4; then for a voxel per wave its
// row of W1, whose gradient is the sum of da1 over the voxel's examples, and its row of W4,
// whose gradient is there.  Both rows' loads are on their way while the list is read and
// sorted.  Adam's 24 bytes and the bfloat16 copy's 2 per parameter bound it: 28 MB.
//
// The sum runs over the list in order of the particle's index, then the example's.  That is
// how the entries arrive where every example adds its particles one after the other.  A list
// of more than kSort entries is counted by example instead (kTally examples at a time) and the
// examples' rows are added in their order, each times its count: at most one row per example,
// however many of its particles share the voxel.  (A step over 512 examples of 150 particles in
// 16 voxels, in one: 720 us and 4.9 ms with the rows of the list one by one, 520 us and 2.1 ms
// with them counted, 113 and 408 us with the lists filled by block too.)
// Both orders follow from the batch alone, so that a step is repeatable.
constexpr int kSort = 256, kTally = 512;
struct ListRoom {                  // a wave's LDS for its list
    union {
        struct { uint64_t key[kSort]; int order[kSort]; };
        struct { uint32_t tally[kTally], pick[kTally]; };
    };
};
constexpr int kSquares = 2 * (H / 64) * (H / 64), kColumns = 3 * (H / 64), kB4Blocks = NV / 256,
              kFinishBlocks = kSquares + kColumns + kB4Blocks + NV / 4;
static_assert(sizeof(Stage) >= kTile * (kTile + 1) * sizeof(float), "a tile of results takes the products' place");
static_assert(sizeof(Stage) >= 4 * sizeof(ListRoom), "the lists take the products' place");

__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// s + the rows of da1 (two columns per lane) of n <= 64 examples, each `times` (held by lane
// like `mine`, the example).
__device__ __forceinline__ void add_rows(const float *da1, int mine, float times, int n, float2 &s)
{
    const int lane = threadIdx.x % 64;
    for (int j = 0; j < n; j += 8) {
        float2 x[8];
#pragma unroll
        for (int q = 0; q < 8; ++q)
            x[q] = *reinterpret_cast<const float2 *>(da1 + (size_t)__builtin_amdgcn_readlane(mine, j + q) * H + 2 * lane);
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const float t = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(times), j + q));
            const float2 more = make_float2(fmaf(t, x[q].x, s.x), fmaf(t, x[q].y, s.y));
            s = j + q < n ? more : s;
        }
    }
}

template <bool UPDATE, bool KEEP>
__global__ void __launch_bounds__(256) finish(int B, Acts ac, Lists ls, float *g, Adam o)
{
    __shared__ Stage st;
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
    int blk = blockIdx.x;
    if (blk < kSquares) {
        const bool third = blk < kSquares / 2;
        const int tile = blk % (kSquares / 2);
        const int m0 = tile / (H / 64) * 64, n0 = tile % (H / 64) * 64;
        const size_t off = third ? OFF_W3 : OFF_W2;
        const Acc acc = product<false, false>(st, third ? ac.g3 : ac.g2, H, m0, third ? ac.h2 : ac.h1, H, n0, 0, B);
        // through LDS to whole rows: a wave two at a time, eight rounds
        float(*sq)[kTile + 1] = reinterpret_cast<float(*)[kTile + 1]>(&st);
        __syncthreads();
        each_element<false, false>(0, 0, [&](auto e, int m, int n) { sq[m][n] = acc.at<e>(); });
        __syncthreads();
        const int r = threadIdx.x / 32, c = 2 * (threadIdx.x % 32);
        AdamRow row[8];
#pragma unroll
        for (int q = 0; q < 8; ++q)
            if (UPDATE) row[q].load(o, off + (size_t)(m0 + r + 8 * q) * H + n0 + c);
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const size_t i = off + (size_t)(m0 + r + 8 * q) * H + n0 + c;
            const float2 gr = make_float2(sq[r + 8 * q][c], sq[r + 8 * q][c + 1]);
            if (KEEP) *reinterpret_cast<float2 *>(g + i) = gr;
            if (UPDATE) row[q].step(o, i, gr);
        }
        return;
    }
    blk -= kSquares;
    if (blk < kColumns) {
        const int which = blk / (H / 64), col = blk % (H / 64) * 64;
        const float s = colsum64(B, H, which == 0 ? ac.da3 : which == 1 ? ac.da2 : ac.da1, col);
        const size_t off = which == 0 ? OFF_B3 : which == 1 ? OFF_B2 : OFF_B1;
        if (threadIdx.x < 64) put<UPDATE, KEEP>(o, g, off + col + threadIdx.x, s);
        return;
    }
    blk -= kColumns;
    if (blk < kB4Blocks) {
        const size_t i = OFF_B4 + 256 * blk + threadIdx.x;
        if (UPDATE) put<true, false>(o, g, i, g[i]);
        return;
    }
    const int v = (blk - kB4Blocks) * 4 + wave;
    const size_t i1 = OFF_W1 + (size_t)v * H + 2 * lane, i4 = OFF_W4 + (size_t)v * H + 2 * lane;
    const int first = __builtin_amdgcn_readfirstlane((int)ls.first[v]);
    const int cnt = __builtin_amdgcn_readfirstlane((int)ls.first[v + 1]) - first;
    AdamRow r1, r4;
    float2 g4;
    const uint64_t *list = ls.entry + first;
    const bool sorted = cnt <= kSort;
    uint64_t k[kSort / 64];
    if (sorted) {
#pragma unroll
        for (int q = 0; q < kSort / 64; ++q)
            if (64 * q < cnt) k[q] = 64 * q + lane < cnt ? list[64 * q + lane] : ~0ull;
    }
    if (UPDATE) {
        g4 = *reinterpret_cast<const float2 *>(g + i4);
        r4.load(o, i4);
        r1.load(o, i1);
    }
    ListRoom &room = reinterpret_cast<ListRoom *>(&st)[wave];
    float2 s = make_float2(0.f, 0.f);
    if (sorted) {
#pragma unroll
        for (int q = 0; q < kSort / 64; ++q)
            if (64 * q < cnt) room.key[64 * q + lane] = k[q];
        wave_lds_sync();
#pragma unroll
        for (int q = 0; q < kSort / 64; ++q)
            if (64 * q < cnt) {
                int rank = 0;
                for (int e = 0; e < cnt; ++e) rank += room.key[e] < k[q];
                if (64 * q + lane < cnt) room.order[rank] = (int)(uint32_t)k[q];
            }
        wave_lds_sync();
        for (int e0 = 0; e0 < cnt; e0 += 64) {
            const int n = cnt - e0 < 64 ? cnt - e0 : 64;
            add_rows(ac.da1, lane < n ? room.order[e0 + lane] : 0, 1.0f, n, s);
        }
    } else {
        for (int b0 = 0; b0 < B; b0 += kTally) {
#pragma unroll
            for (int q = 0; q < kTally / 64; ++q) room.tally[64 * q + lane] = 0u;
            wave_lds_sync();
#pragma unroll 4
            for (int e = lane; e < cnt; e += 64) {
                const uint32_t b = (uint32_t)list[e] - (uint32_t)b0;
                if (b < (uint32_t)kTally) atomicAdd(&room.tally[b], 1u);
            }
            wave_lds_sync();
            int held = 0;
#pragma unroll
            for (int q = 0; q < kTally / 64; ++q) {
                const uint32_t c = room.tally[64 * q + lane];
                const uint64_t have = __ballot(c != 0u);
                if (c) room.pick[held + __popcll(have & ((1ull << lane) - 1))] = (uint32_t)(64 * q + lane) | c << 16;
                held += __popcll(have);
            }
            wave_lds_sync();
            for (int e0 = 0; e0 < held; e0 += 64) {
                const int n = held - e0 < 64 ? held - e0 : 64;
                const uint32_t u = lane < n ? room.pick[e0 + lane] : 0u;
                add_rows(ac.da1, lane < n ? b0 + (int)(u & 0xffffu) : 0, (float)(u >> 16), n, s);
            }
            wave_lds_sync();
        }
    }
    if (KEEP) *reinterpret_cast<float2 *>(g + i1) = s;
    if (UPDATE) {
        r4.step(o, i4, g4);
        r1.step(o, i1, s);
    }
}

__global__ void to_bf16(size_t count, const float *x, bf16 *y)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) y[i] = f2bf(x[i]);
}

// Flags a training set with an N outside 0..nmax or a voxel index >= NV among an
// example's first N entries (block per example, grid-stride over examples).
__global__ void check_set(int64_t n_examples, int nmax, const uint16_t *set_vox, const int32_t *set_n, int *bad)
{
    for (int64_t ex = blockIdx.x; ex < n_examples; ex += gridDim.x) {
        const int nb = set_n[ex];
        if (nb < 0 || nb > nmax) {
            if (threadIdx.x == 0) *bad = 1;
            continue;
        }
        bool out = false;
        for (int j = threadIdx.x; j < nb; j += blockDim.x) out |= set_vox[ex * nmax + j] >= NV;
        if (out) *bad = 1;
    }
}

// MFMA B-operand tiles of a [n_out][128] weight matrix (the layout of NetDev):
// P[((tile*4 + kp)*64 + lane)*8 + j] = W[16 tile + lane%16][32 kp + 16 (j/4) + 4 (lane/16) + j%4]
__global__ void pack_b_tiles(int n_out, const bf16 *W, bf16 *P)
{
    const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (size_t)n_out * H) return;
    const int j = (int)(idx % 8), lane = (int)((idx / 8) % 64), kp = (int)((idx / 512) % 4);
    const int tile = (int)(idx / 2048);
    P[idx] = W[(size_t)(16 * tile + lane % 16) * H + 32 * kp + 16 * (j / 4) + 4 * (lane / 16) + j % 4];
}

// Voxel lists of walkers: vox[w][j] = voxel of particle j of walker w (the grid of
// the learned proposal over the class's gas region), n_out[w] = N.
__global__ void capture_voxels(int n_walkers, int stride, const ClassDev *cls, const int *walker_class,
                               const int32_t *n, const double *xyz, int xyz_stride, uint16_t *vox, int32_t *n_out)
{
    const int w = blockIdx.x;
    const ClassDev &C = cls[walker_class[w]];
    const int nw = n[w];
    const double gx = (double)kNetGrid / C.lx, gy = (double)kNetGrid / C.ly, gz = (double)kNetGrid / (C.zhi - C.zlo);
    for (int j = threadIdx.x; j < stride; j += blockDim.x) {
        int v = 0;
        if (j < nw) {
            const double *p = xyz + ((size_t)w * xyz_stride + j) * 3;
            int ix = (int)floor(p[0] * gx), iy = (int)floor(p[1] * gy), iz = (int)floor((p[2] - C.zlo) * gz);
            ix = ix < 0 ? 0 : (ix > kNetGrid - 1 ? kNetGrid - 1 : ix);
            iy = iy < 0 ? 0 : (iy > kNetGrid - 1 ? kNetGrid - 1 : iy);
            iz = iz < 0 ? 0 : (iz > kNetGrid - 1 ? kNetGrid - 1 : iz);
            v = (iz * kNetGrid + iy) * kNetGrid + ix;
        }
        vox[(size_t)w * stride + j] = (uint16_t)v;
    }
    if (threadIdx.x == 0) n_out[w] = nw;
}

// k-major copy of a [n_out][128] weight matrix: T[k][o] = W[o][k]
__global__ void transpose_kmajor(int n_out, const bf16 *W, bf16 *T)
{
    const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (size_t)n_out * H) return;
    const int k = (int)(idx / n_out), o = (int)(idx % n_out);
    T[idx] = W[(size_t)o * H + k];
}

}  // namespace mlpk
}  // namespace regc

using namespace regc;
using namespace regc::mlpk;

struct regc_mlp {
    int max_batch = 0, nmax = 0;
    hipStream_t stream = nullptr;
    DevBuf<float> p, g, m, v;
    DevBuf<bf16> p16;
    DevBuf<float> a1, a2, a3, logits, d32, da1, da2, da3, loss, ksplit;
    DevBuf<bf16> h1, h2, h3, d16, g2, g3;
    DevBuf<uint16_t> bvox;
    DevBuf<int32_t> bn, bex, btgt;
    DevBuf<uint32_t> count, first, cursor;
    DevBuf<uint64_t> entry;
    DevBuf<int> bad;                  // check_set's flag
    int64_t t = 0;   // Adam steps taken
    double ms_train = 0.0;
    int64_t steps_timed = 0;
};

static int mlp_workspace(regc_mlp *h, int B, int nmax)
{
    if (B <= h->max_batch && nmax <= h->nmax) return REGC_OK;
    const int Bm = std::max(B, h->max_batch), nm = std::max(nmax, h->nmax);
    int rc;
    if ((rc = h->a1.alloc((size_t)Bm * H)) || (rc = h->a2.alloc((size_t)Bm * H)) || (rc = h->a3.alloc((size_t)Bm * H)) ||
        (rc = h->logits.alloc((size_t)Bm * NV)) || (rc = h->d32.alloc((size_t)Bm * NV)) ||
        (rc = h->da1.alloc((size_t)Bm * H)) || (rc = h->da2.alloc((size_t)Bm * H)) || (rc = h->da3.alloc((size_t)Bm * H)) ||
        (rc = h->loss.alloc(Bm)) || (rc = h->h1.alloc((size_t)Bm * H)) || (rc = h->h2.alloc((size_t)Bm * H)) ||
        (rc = h->h3.alloc((size_t)Bm * H)) || (rc = h->d16.alloc((size_t)Bm * NV)) || (rc = h->g2.alloc((size_t)Bm * H)) ||
        (rc = h->g3.alloc((size_t)Bm * H)) || (rc = h->bvox.alloc((size_t)Bm * nm)) || (rc = h->bn.alloc(Bm)) ||
        (rc = h->bex.alloc(Bm)) || (rc = h->btgt.alloc(Bm)) || (rc = h->ksplit.alloc((size_t)kSplitK * Bm * H)) ||
        (rc = h->entry.alloc((size_t)Bm * nm)) || (rc = h->count.alloc(NV)) || (rc = h->first.alloc(NV + 1)) ||
        (rc = h->cursor.alloc(NV)) || (rc = h->bad.alloc(1)))
        return rc;
    h->max_batch = Bm;
    h->nmax = nm;
    return REGC_OK;
}

static Batch batch_of(regc_mlp *h, int B, int nmax) { return {B, nmax, h->bvox.p, h->bn.p, h->bex.p, h->btgt.p}; }

static Acts acts_of(regc_mlp *h)
{
    return {h->a1.p, h->a2.p, h->a3.p, h->h1.p, h->h2.p, h->h3.p, h->da1.p, h->da2.p, h->da3.p, h->g2.p, h->g3.p};
}

// blocks over the batch's entries
static int entry_blocks(int B) { return std::min(B / 4, 1024); }

// forward of the batch in h->bvox/bn/bex, or drawn into them from src (B a multiple of 64);
// entries: count the voxels' entries for a backward pass
static int mlp_forward_dev(regc_mlp *h, int B, int nmax, const Source &src, bool entries)
{
    hipStream_t s = h->stream;
    const Batch bt = batch_of(h, B, nmax);
    hipLaunchKernelGGL(hidden_forward, dim3(B / kRows), dim3(128 * kRows), 0, s, bt, src, h->p16.p, h->p.p, acts_of(h),
                       entries ? h->count.p : nullptr);
    REGC_HIP(hipGetLastError());
    hipLaunchKernelGGL(logits_forward, dim3((NV / 64) * (B / 64) + (entries ? entry_blocks(B) : 0)), dim3(256), 0, s,
                       bt, h->p16.p, h->p.p, h->h3.p, h->logits.p, h->count.p);
    REGC_HIP(hipGetLastError());
    return REGC_OK;
}

// forward + backward of the batch; gradients into h->g (keep; W4's and b4's in any case), and
// with `adam` the update (its pointers are filled in here)
static int mlp_backward_dev(regc_mlp *h, int B, int nmax, const Source &src, const Adam *adam, bool keep)
{
    hipStream_t s = h->stream;
    int rc;
    if ((rc = mlp_forward_dev(h, B, nmax, src, true))) return rc;
    const Lists ls{h->count.p, h->first.p, h->cursor.p, h->entry.p};
    hipLaunchKernelGGL(softmax_xent, dim3(B + 1), dim3(kSoftThreads), 0, s, B, h->logits.p, h->btgt.p, h->loss.p, h->d32.p, h->d16.p,
                       ls);
    REGC_HIP(hipGetLastError());
    const int dh = (B / 64) * (H / 64) * kSplitK;
    hipLaunchKernelGGL(output_backward, dim3(dh + kDw4Blocks + kDb4Blocks + entry_blocks(B)), dim3(256), 0, s,
                       batch_of(h, B, nmax), h->p16.p, h->h3.p, h->d32.p, h->d16.p, h->ksplit.p, h->g.p, ls);
    REGC_HIP(hipGetLastError());
    hipLaunchKernelGGL(hidden_backward, dim3(B / kRows), dim3(128 * kRows), 0, s, B, h->p16.p, h->ksplit.p, acts_of(h));
    REGC_HIP(hipGetLastError());
    Adam o{};
    if (adam) o = *adam;
    o.p = h->p.p; o.m = h->m.p; o.v = h->v.p; o.p16 = h->p16.p;
    const dim3 grid(kFinishBlocks), block(256);
    if (!adam) hipLaunchKernelGGL((finish<false, true>), grid, block, 0, s, B, acts_of(h), ls, h->g.p, o);
    else if (keep) hipLaunchKernelGGL((finish<true, true>), grid, block, 0, s, B, acts_of(h), ls, h->g.p, o);
    else hipLaunchKernelGGL((finish<true, false>), grid, block, 0, s, B, acts_of(h), ls, h->g.p, o);
    REGC_HIP(hipGetLastError());
    return REGC_OK;
}

// Adam's coefficients of step h->t + 1, which it counts
static Adam next_step(regc_mlp *h, double lr)
{
    Adam o{};
    o.beta1 = 0.9f; o.beta2 = 0.999f; o.eps = 1e-8f;
    o.lr = (float)lr;
    h->t += 1;
    o.c1 = 1.0f - powf(o.beta1, (float)h->t);
    o.c2 = 1.0f - powf(o.beta2, (float)h->t);
    return o;
}

static int upload_batch(regc_mlp *h, int B, int nmax, const uint16_t *vox, const int32_t *n, const int32_t *excl,
                        const int32_t *target)
{
    hipStream_t s = h->stream;
    REGC_HIP(hipMemcpyAsync(h->bvox.p, vox, sizeof(uint16_t) * (size_t)B * nmax, hipMemcpyHostToDevice, s));
    REGC_HIP(hipMemcpyAsync(h->bn.p, n, sizeof(int32_t) * B, hipMemcpyHostToDevice, s));
    REGC_HIP(hipMemcpyAsync(h->bex.p, excl, sizeof(int32_t) * B, hipMemcpyHostToDevice, s));
    if (target) REGC_HIP(hipMemcpyAsync(h->btgt.p, target, sizeof(int32_t) * B, hipMemcpyHostToDevice, s));
    return REGC_OK;
}

static int check_batch(int B, int nmax, const uint16_t *vox, const int32_t *n, const int32_t *excl, const int32_t *target)
{
    REGC_CHECK(B > 0 && B % 64 == 0, REGC_EINVAL, "batch must be a positive multiple of 64");
    REGC_CHECK(nmax > 0 && nmax <= 65535, REGC_EINVAL, "bad nmax");
    for (int b = 0; b < B; ++b) {
        REGC_CHECK(n[b] >= 0 && n[b] <= nmax, REGC_EINVAL, "example %d: N out of range", b);
        REGC_CHECK(excl[b] >= -1 && excl[b] < std::max(n[b], 1), REGC_EINVAL, "example %d: bad left-out index", b);
        for (int j = 0; j < n[b]; ++j) REGC_CHECK(vox[(size_t)b * nmax + j] < NV, REGC_EINVAL, "voxel out of range");
        if (target) REGC_CHECK(target[b] >= 0 && target[b] < NV, REGC_EINVAL, "target voxel out of range");
    }
    return REGC_OK;
}

extern "C" int regc_mlp_create(const float *params, regc_mlp **out)
{
    REGC_CHECK(out, REGC_EINVAL, "null output pointer");
    regc_mlp *h = new regc_mlp();
    int rc;
    if ((rc = h->p.alloc(NPARAM)) || (rc = h->g.alloc(NPARAM)) || (rc = h->m.alloc(NPARAM)) ||
        (rc = h->v.alloc(NPARAM)) || (rc = h->p16.alloc(NPARAM)) || (rc = mlp_workspace(h, 64, 64))) {
        delete h;
        return rc;
    }
    if (params) {
        if (hipMemcpy(h->p.p, params, sizeof(float) * NPARAM, hipMemcpyHostToDevice) != hipSuccess) {
            delete h;
            set_error("hipMemcpy failed");
            return REGC_EHIP;
        }
    } else {
        (void)hipMemset(h->p.p, 0, sizeof(float) * NPARAM);
    }
    (void)hipMemset(h->m.p, 0, sizeof(float) * NPARAM);
    (void)hipMemset(h->v.p, 0, sizeof(float) * NPARAM);
    hipLaunchKernelGGL(to_bf16, dim3((unsigned)((NPARAM + 255) / 256)), dim3(256), 0, 0, (size_t)NPARAM, h->p.p, h->p16.p);
    if (hipDeviceSynchronize() != hipSuccess) {
        delete h;
        set_error("device synchronisation failed");
        return REGC_EHIP;
    }
    *out = h;
    return REGC_OK;
}

extern "C" int regc_mlp_param_count(int64_t *count)
{
    REGC_CHECK(count, REGC_EINVAL, "null argument");
    *count = (int64_t)NPARAM;
    return REGC_OK;
}

extern "C" int regc_mlp_set_stream(regc_mlp *h, void *stream)
{
    REGC_CHECK(h, REGC_EINVAL, "null handle");
    h->stream = (hipStream_t)stream;
    return REGC_OK;
}

extern "C" int regc_mlp_set_params(regc_mlp *h, const float *params)
{
    REGC_CHECK(h && params, REGC_EINVAL, "null argument");
    REGC_HIP(hipStreamSynchronize(h->stream));
    REGC_HIP(hipMemcpy(h->p.p, params, sizeof(float) * NPARAM, hipMemcpyHostToDevice));
    hipLaunchKernelGGL(to_bf16, dim3((unsigned)((NPARAM + 255) / 256)), dim3(256), 0, h->stream, (size_t)NPARAM, h->p.p,
                       h->p16.p);
    REGC_HIP(hipGetLastError());
    REGC_HIP(hipMemsetAsync(h->m.p, 0, sizeof(float) * NPARAM, h->stream));
    REGC_HIP(hipMemsetAsync(h->v.p, 0, sizeof(float) * NPARAM, h->stream));
    h->t = 0;
    REGC_HIP(hipStreamSynchronize(h->stream));
    return REGC_OK;
}

extern "C" int regc_mlp_get_params(regc_mlp *h, float *params)
{
    REGC_CHECK(h && params, REGC_EINVAL, "null argument");
    REGC_HIP(hipStreamSynchronize(h->stream));
    REGC_HIP(hipMemcpy(params, h->p.p, sizeof(float) * NPARAM, hipMemcpyDeviceToHost));
    return REGC_OK;
}

extern "C" int regc_mlp_forward(regc_mlp *h, int B, int nmax, const uint16_t *vox, const int32_t *n,
                                const int32_t *excl, float *logits)
{
    REGC_CHECK(h && vox && n && excl && logits, REGC_EINVAL, "null argument");
    int rc;
    if ((rc = check_batch(B, nmax, vox, n, excl, nullptr)) || (rc = mlp_workspace(h, B, nmax)) ||
        (rc = upload_batch(h, B, nmax, vox, n, excl, nullptr)) || (rc = mlp_forward_dev(h, B, nmax, Source{}, false)))
        return rc;
    REGC_HIP(hipStreamSynchronize(h->stream));
    REGC_HIP(hipMemcpy(logits, h->logits.p, sizeof(float) * (size_t)B * NV, hipMemcpyDeviceToHost));
    return REGC_OK;
}

extern "C" int regc_mlp_loss_grads(regc_mlp *h, int B, int nmax, const uint16_t *vox, const int32_t *n,
                                   const int32_t *excl, const int32_t *target, double *loss, float *grads)
{
    REGC_CHECK(h && vox && n && excl && target, REGC_EINVAL, "null argument");
    int rc;
    if ((rc = check_batch(B, nmax, vox, n, excl, target)) || (rc = mlp_workspace(h, B, nmax)) ||
        (rc = upload_batch(h, B, nmax, vox, n, excl, target)) || (rc = mlp_backward_dev(h, B, nmax, Source{}, nullptr, true)))
        return rc;
    REGC_HIP(hipStreamSynchronize(h->stream));
    if (loss) {
        std::vector<float> l(B);
        REGC_HIP(hipMemcpy(l.data(), h->loss.p, sizeof(float) * B, hipMemcpyDeviceToHost));
        double s = 0.0;
        for (float x : l) s += x;
        *loss = s / B;
    }
    if (grads) REGC_HIP(hipMemcpy(grads, h->g.p, sizeof(float) * NPARAM, hipMemcpyDeviceToHost));
    return REGC_OK;
}

extern "C" int regc_mlp_step(regc_mlp *h, int B, int nmax, const uint16_t *vox, const int32_t *n,
                             const int32_t *excl, const int32_t *target, double lr, double *loss, float *grads)
{
    REGC_CHECK(h && vox && n && excl && target, REGC_EINVAL, "null argument");
    REGC_CHECK(lr > 0, REGC_EINVAL, "learning rate must be positive");
    int rc;
    if ((rc = check_batch(B, nmax, vox, n, excl, target)) || (rc = mlp_workspace(h, B, nmax)) ||
        (rc = upload_batch(h, B, nmax, vox, n, excl, target)))
        return rc;
    const Adam adam = next_step(h, lr);
    if ((rc = mlp_backward_dev(h, B, nmax, Source{}, &adam, grads != nullptr))) {
        h->t -= 1;
        return rc;
    }
    hipStream_t s = h->stream;
    REGC_HIP(hipStreamSynchronize(s));
    if (loss) {
        std::vector<float> l(B);
        REGC_HIP(hipMemcpy(l.data(), h->loss.p, sizeof(float) * B, hipMemcpyDeviceToHost));
        double acc = 0.0;
        for (float x : l) acc += x;
        *loss = acc / B;
    }
    if (grads) REGC_HIP(hipMemcpy(grads, h->g.p, sizeof(float) * NPARAM, hipMemcpyDeviceToHost));
    return REGC_OK;
}

extern "C" int regc_mlp_train(regc_mlp *h, int64_t n_examples, int nmax, const uint16_t *vox_dev,
                              const int32_t *n_dev, int64_t steps, int batch, double lr, uint64_t seed,
                              double *mean_loss)
{
    REGC_CHECK(h && vox_dev && n_dev, REGC_EINVAL, "null argument");
    REGC_CHECK(n_examples > 0 && steps > 0 && lr > 0, REGC_EINVAL, "bad training size");
    REGC_CHECK(batch > 0 && batch % 64 == 0, REGC_EINVAL, "batch must be a positive multiple of 64");
    REGC_CHECK(nmax > 0 && nmax <= 65535, REGC_EINVAL, "bad nmax");
    int rc;
    if ((rc = mlp_workspace(h, batch, nmax))) return rc;
    hipStream_t s = h->stream;
    {
        // the batch kernels index by N and gather W1 rows by voxel: check the set first
        int h_bad = 0;
        REGC_HIP(hipMemsetAsync(h->bad.p, 0, sizeof(int), s));
        hipLaunchKernelGGL(check_set, dim3((unsigned)std::min<int64_t>(n_examples, 4096)), dim3(64), 0, s, n_examples,
                           nmax, vox_dev, n_dev, h->bad.p);
        REGC_HIP(hipGetLastError());
        REGC_HIP(hipMemcpyAsync(&h_bad, h->bad.p, sizeof(int), hipMemcpyDeviceToHost, s));
        REGC_HIP(hipStreamSynchronize(s));
        REGC_CHECK(!h_bad, REGC_EINVAL, "training set: an N outside 0..%d or a voxel index >= %d", nmax, NV);
    }
    ScopedEvent e0, e1;
    REGC_HIP(e0.create());
    REGC_HIP(e1.create());
    REGC_HIP(hipEventRecord(e0.e, s));
    double loss_acc = 0.0;
    std::vector<float> lh(batch);
    for (int64_t st = 0; st < steps; ++st) {
        const Source src{n_examples, h->t, vox_dev, n_dev, (uint32_t)seed, (uint32_t)(seed >> 32)};
        const Adam adam = next_step(h, lr);
        if ((rc = mlp_backward_dev(h, batch, nmax, src, &adam, false))) {
            h->t -= 1;
            return rc;
        }
        if (mean_loss && (st == steps - 1 || (st + 1) % 50 == 0)) {
            REGC_HIP(hipMemcpyAsync(lh.data(), h->loss.p, sizeof(float) * batch, hipMemcpyDeviceToHost, s));
            REGC_HIP(hipStreamSynchronize(s));
            double a = 0.0;
            for (float x : lh) a += x;
            loss_acc = a / batch;
        }
    }
    REGC_HIP(hipEventRecord(e1.e, s));
    REGC_HIP(hipEventSynchronize(e1.e));
    float ms = 0.f;
    REGC_HIP(hipEventElapsedTime(&ms, e0.e, e1.e));
    h->ms_train += ms;
    h->steps_timed += steps;
    if (mean_loss) *mean_loss = loss_acc;
    return REGC_OK;
}

namespace regc {
hipError_t launch_capture_voxels(int n_walkers, int stride, const ClassDev *cls, const int *walker_class,
                                 const int32_t *n, const double *xyz, int xyz_stride, uint16_t *vox, int32_t *n_out,
                                 hipStream_t s)
{
    hipLaunchKernelGGL(capture_voxels, dim3(n_walkers), dim3(64), 0, s, n_walkers, stride, cls, walker_class, n, xyz,
                       xyz_stride, vox, n_out);
    return hipGetLastError();
}

int mlp_export_sampler(regc_mlp *h, bool kmajor, uint16_t *w1, uint16_t *w2, uint16_t *w3, uint16_t *w4, float *b1,
                       float *b2, float *b3, float *b4, hipStream_t s)
{
    REGC_CHECK(h, REGC_EINVAL, "null network");
    REGC_HIP(hipStreamSynchronize(h->stream));
    REGC_HIP(hipMemcpyAsync(w1, h->p16.p + OFF_W1, sizeof(bf16) * (size_t)NV * H, hipMemcpyDeviceToDevice, s));
    const bf16 *src[3] = {h->p16.p + OFF_W2, h->p16.p + OFF_W3, h->p16.p + OFF_W4};
    uint16_t *dst[3] = {w2, w3, w4};
    const int n_out[3] = {H, H, NV};
    for (int q = 0; q < 3; ++q) {
        const unsigned blocks = (unsigned)((size_t)n_out[q] * H / 256);
        if (kmajor)
            hipLaunchKernelGGL(transpose_kmajor, dim3(blocks), dim3(256), 0, s, n_out[q], src[q], dst[q]);
        else
            hipLaunchKernelGGL(pack_b_tiles, dim3(blocks), dim3(256), 0, s, n_out[q], src[q], dst[q]);
        REGC_HIP(hipGetLastError());
    }
    REGC_HIP(hipMemcpyAsync(b1, h->p.p + OFF_B1, sizeof(float) * H, hipMemcpyDeviceToDevice, s));
    REGC_HIP(hipMemcpyAsync(b2, h->p.p + OFF_B2, sizeof(float) * H, hipMemcpyDeviceToDevice, s));
    REGC_HIP(hipMemcpyAsync(b3, h->p.p + OFF_B3, sizeof(float) * H, hipMemcpyDeviceToDevice, s));
    REGC_HIP(hipMemcpyAsync(b4, h->p.p + OFF_B4, sizeof(float) * NV, hipMemcpyDeviceToDevice, s));
    return REGC_OK;
}
}  // namespace regc

extern "C" int regc_mlp_timing(regc_mlp *h, double *ms, int64_t *steps)
{
    REGC_CHECK(h, REGC_EINVAL, "null handle");
    if (ms) *ms = h->ms_train;
    if (steps) *steps = h->steps_timed;
    return REGC_OK;
}

extern "C" void regc_mlp_destroy(regc_mlp *h) { delete h; }
