// Multi-turn session predictor (Sec. 3.3): y = W3 relu(W2 relu(W1 h + b1) + b2) + b3
// over a batch of last-token hidden states, on the matrix cores.
//
// Layer 1 (n x d) . (d x 256) is the one dense contraction of the method:
// bf16 products (exact) summed in fp32 by v_mfma_f32_32x32x16_bf16.  A
// workgroup of 8 waves (two per SIMD, so that one issues MFMAs while the other
// waits on LDS or the barrier) computes a 128 x 128 or 64 x 64 tile of one of
// four k slices.
// The sum over k is order-free, so A and B may share any permutation of k:
// lane l (row / column l mod 32, half l / 32) supplies, in a 64-wide k step,
// the 32 contiguous values of its half (64 bytes, four 16-byte pieces), and
// MFMA m of the step takes values 8m .. 8m + 7 of both operands.  Tiles are
// ordered so that the workgroups of a row tile land on the same XCD (block ids
// go round-robin over the 8 XCDs) and read the same hidden-state rows through
// one L2; giving each XCD its own part of W1 instead was slower at every size.
//
// Layers 2 and 3 are fp32: v_mfma_f32_16x16x4f32 for (16 rows x 256) . (256 x
// 64) in a workgroup of 8 waves (each a k eighth of all 16 rows, loaded once
// and fed to the four 16-column blocks, every load of a wave issued at once,
// the eighths summed in a fixed order), then the 64-term layer 3 by shuffles.  Layer 1's four k
// slices are added here, in slice order, before b1 and the ReLU.
#include <mutex>

#include "sae_internal.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
// a native vector: the HIP struct type is kept in memory when a struct of it is passed around
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int L1_THREADS = 512;  // 8 waves: a quadrant of the tile and a half of each step's k each
constexpr int KSTEP = 64;          // k per step
constexpr int KSPLIT = 4;          // k slices (workgroups per tile); their sums meet in layer 2
constexpr int LDS_ROW16 = 9;       // LDS row of a tile: 128 bytes of k + 16 bytes of padding
constexpr int L23_THREADS = 512;   // 8 waves: one k eighth each, both layer-2 column halves
constexpr int L23_ROWS = 16;

__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 v)
{
    bf16x8 r;
    __builtin_memcpy(&r, &v, sizeof(r));
    return r;
}

// One step (64 k) of a thread's share of the A and B tiles.
template <int RPT>
struct Stage {
    u32x4 a[RPT], b[RPT];
};

// A step past the end loads the last one again (in bounds; it is never
// multiplied).  Nothing may touch the loaded values here: an operation on them
// makes the compiler wait for the loads it has just issued.
template <int RPT>
__device__ __forceinline__ void load_stage(Stage<RPT> &x, const u32x4 *const (&ga)[RPT], const u32x4 *gb,
                                           long long bstride, int step, int nsteps)
{
    const int o = (step < nsteps ? step : nsteps - 1) * (KSTEP / 8);
#pragma unroll
    for (int j = 0; j < RPT; ++j) x.a[j] = ga[j][o];
#pragma unroll
    for (int j = 0; j < RPT; ++j) x.b[j] = gb[j * bstride + o];
}

template <int RPT>
__device__ __forceinline__ void put_stage(const Stage<RPT> &x, u32x4 *la, u32x4 *lb, int ls)
{
#pragma unroll
    for (int j = 0; j < RPT; ++j) {
        la[ls + j * 64 * LDS_ROW16] = x.a[j];
        lb[ls + j * 64 * LDS_ROW16] = x.b[j];
    }
}

// Layer 1, TILE x TILE tiles (128 or 64), one k slice of a tile per workgroup.
// A wave computes one quadrant of the tile over half of each step's k (the
// halves are added at the end): per step a workgroup then reads TILE / 2 rows
// of each operand 8 times from LDS, half a row each, two thirds of what 64 x 32
// blocks over the whole k read, and LDS bandwidth is what bounds a step.
template <int TILE>
__global__ void __launch_bounds__(L1_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_pred_l1(int n, int d, const uint16_t *h, const uint16_t *w1, float *part, int row_tiles)
{
    constexpr int RPT = TILE / 64;  // rows of each tile a thread moves per step
    constexpr int NB = TILE / 64;   // 32-wide MFMA blocks per side of a quadrant
    // LDS: two stages of the A tile (TILE rows) and the B tile (TILE columns),
    // 64 k each, rows padded to 144 bytes so that the 32 rows one MFMA operand
    // read touches spread over the banks
    __shared__ u32x4 lds[2][2][TILE * LDS_ROW16];
    static_assert(sizeof(lds) >= L1_THREADS * NB * NB * 8 * sizeof(float), "the k halves meet in the tile buffers");
    constexpr int CT = SAE_PRED_H1 / TILE;             // column tiles
    const int bid = blockIdx.x;
    const int xcd = bid & 7, slot = bid >> 3;
    const int ks = slot % KSPLIT;                      // k slice
    const int ct = (slot / KSPLIT) % CT;
    const int rt = (slot / KSPLIT / CT) * 8 + xcd;
    if (rt >= row_tiles) return;                      // the whole workgroup
    const int tid = threadIdx.x;
    const int lane = (int)__lane_id(), wave = tid / SAE_WAVE;
    const int wr = (wave >> 1) & 1, wc = wave & 1, kh = wave >> 2;
    const int kper = d / KSPLIT;                       // a multiple of 64
    const int kbeg = ks * kper, nsteps = kper / KSTEP;
    // global -> LDS: thread t moves 16-byte chunks of rows t / 8 + 64 j (j < RPT),
    // chunk t mod 8 of each row's 128 bytes, of both tiles
    const int lr = tid >> 3, lc = tid & 7;
    const u32x4 *ga[RPT];
#pragma unroll
    for (int j = 0; j < RPT; ++j) {
        int r = rt * TILE + lr + 64 * j;
        r = r < n ? r : n - 1;  // rows past n repeat row n - 1 (results dropped)
        ga[j] = reinterpret_cast<const u32x4 *>(h + (long long)r * d + kbeg) + lc;
    }
    const u32x4 *gb = reinterpret_cast<const u32x4 *>(w1 + (long long)(ct * TILE + lr) * d + kbeg) + lc;
    const long long bstride = 64ll * d / 8;  // 64 rows of W1, in u32x4
    const int ls = lr * LDS_ROW16 + lc;
    floatx16 acc[NB][NB];
#pragma unroll
    for (int bi = 0; bi < NB; ++bi)
#pragma unroll
        for (int bj = 0; bj < NB; ++bj)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[bi][bj][i] = 0.0f;
    // operand reads: lane (row / column l mod 32, half l / 32) takes, in MFMA
    // m of a step, the 16 bytes at k = 32 half + 8 m of its row; this wave's
    // m are 2 kh and 2 kh + 1
    const int oa = (wr * (TILE / 2) + (lane & 31)) * LDS_ROW16 + (lane >> 5) * 4 + 2 * kh;
    const int ob = (wc * (TILE / 2) + (lane & 31)) * LDS_ROW16 + (lane >> 5) * 4 + 2 * kh;
    // pipeline: step s is in LDS buffer s mod 2 while steps s + 1 and s + 2 are
    // in flight in registers.  Four steps in flight, and the next step's
    // operands read from LDS during this step's MFMAs, were no faster: what is
    // left is the rate at which a compute unit is fed from L2
    Stage<RPT> s0, s1;
    load_stage(s0, ga, gb, bstride, 0, nsteps);
    put_stage(s0, lds[0][0], lds[0][1], ls);
    load_stage(s0, ga, gb, bstride, 1, nsteps);
    load_stage(s1, ga, gb, bstride, 2, nsteps);
    __syncthreads();
    auto step = [&](Stage<RPT> &x, int b, int t) {  // step t, in LDS buffer b; x holds step t + 1
        bf16x8 va[2][NB], vb[2][NB];
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                va[m][i] = as_bf16x8(lds[b][0][oa + i * 32 * LDS_ROW16 + m]);
                vb[m][i] = as_bf16x8(lds[b][1][ob + i * 32 * LDS_ROW16 + m]);
            }
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int bi = 0; bi < NB; ++bi)
#pragma unroll
                for (int bj = 0; bj < NB; ++bj)
                    acc[bi][bj] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[m][bi], vb[m][bj], acc[bi][bj], 0, 0, 0);
        put_stage(x, lds[b ^ 1][0], lds[b ^ 1][1], ls);
        load_stage(x, ga, gb, bstride, t + 3, nsteps);
        __syncthreads();
    };
    int st = 0;
    for (; st + 2 <= nsteps; st += 2) {
        step(s0, 0, st);
        step(s1, 1, st + 1);
    }
    if (st < nsteps) step(s0, 0, st);  // uniform
    // the two k halves of a quadrant: each wave hands half of its sums to the
    // other (through the tile buffers, free since the last barrier) and
    // finishes the half it keeps, first half of k + second half
    constexpr int E = NB * NB * 16, HE = E / 2;
    float mine[HE], give[HE];
#pragma unroll
    for (int e = 0; e < HE; ++e) {
        const float lo = acc[e / 16 / NB][(e / 16) % NB][e % 16];
        const float hi = acc[(e + HE) / 16 / NB][((e + HE) / 16) % NB][(e + HE) % 16];
        mine[e] = kh ? hi : lo;
        give[e] = kh ? lo : hi;
    }
    float *xs = reinterpret_cast<float *>(lds);  // [wave][HE][64]
#pragma unroll
    for (int e = 0; e < HE; ++e) xs[(wave * HE + e) * SAE_WAVE + lane] = give[e];
    __syncthreads();
#pragma unroll
    for (int e = 0; e < HE; ++e) mine[e] = mine[e] + xs[((wave ^ 4) * HE + e) * SAE_WAVE + lane];
    // partial sums of this k slice; C layout: lane l holds column l mod 32,
    // rows 8 (i / 4) + 4 (l / 32) + i mod 4 of each 32 x 32 block
    float *out = part + (long long)ks * n * SAE_PRED_H1 + ct * TILE + wc * (TILE / 2) + (lane & 31);
    const int r0 = rt * TILE + wr * (TILE / 2) + (lane >> 5) * 4;
#pragma unroll
    for (int e = 0; e < HE; ++e) {
        // element e of the kept half: block (bi, bj), register i
        const int bi = (NB == 2) ? kh : 0, bj = (NB == 2) ? e / 16 : 0;
        const int i = (NB == 2) ? e % 16 : e + kh * HE;
        const int r = r0 + bi * 32 + (i >> 2) * 8 + (i & 3);
        if (r < n) out[(long long)r * SAE_PRED_H1 + bj * 32] = mine[e];
    }
}

__global__ void __launch_bounds__(L23_THREADS) __attribute__((amdgpu_waves_per_eu(1, 2)))
k_pred_l23(int n, const float *part, const float *b1, const float *w2, const float *b2, const float *w3,
           const float *b3, float *logit, uint8_t *pred)
{
    // 16 rows per workgroup (every compute unit busy); wave w owns k eighth w
    // (32 of the 256 layer-1 units) of all 16 rows: it loads those units once
    // (four slices) and feeds them to the MFMAs of the four 16-column blocks
    // of layer 2; the eighths meet in LDS and are added in eighth order
    constexpr int NW = L23_THREADS / SAE_WAVE;  // 8
    constexpr int KW = SAE_PRED_H1 / NW;         // 32
    constexpr int NCB = SAE_PRED_H2 / 16;        // 4 column blocks
    __shared__ float hsum[NW - 1][NCB * 4][SAE_WAVE];
    __shared__ float ysum[L23_ROWS];
    const int lane = (int)__lane_id(), wave = threadIdx.x / SAE_WAVE;
    const int r0 = blockIdx.x * L23_ROWS;
    const int row = r0 + (lane & 15);
    const int rowc = row < n ? row : n - 1;
    const int grp = lane >> 4;
    // lane group g supplies k = 32 w + 8 g + s in MFMA s, for both operands
    // (v_mfma_f32_16x16x4f32: lane l gives A[l mod 16][l / 16] and
    // B[l / 16][l mod 16]); the layer-1 value is the sum of its k slices in
    // slice order, plus b1, ReLU
    const int kb = wave * KW + grp * 8;
    const long long slice = (long long)n * SAE_PRED_H1 / 4;  // in float4
    const float4 *pa = reinterpret_cast<const float4 *>(part + (long long)rowc * SAE_PRED_H1 + kb);
    const float4 *pc = reinterpret_cast<const float4 *>(b1 + kb);
    float4 v[KSPLIT][2], bw[NCB][2], c[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {  // every load of the wave in flight together
#pragma unroll
        for (int q = 0; q < KSPLIT; ++q) v[q][u] = pa[q * slice + u];
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb)
            bw[cb][u] = reinterpret_cast<const float4 *>(w2 + (long long)(cb * 16 + (lane & 15)) * SAE_PRED_H1 + kb)[u];
        c[u] = pc[u];
    }
    // what the end needs, with the same round trip
    float bias[NCB], wt[NCB];
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
        bias[cb] = b2[cb * 16 + (lane & 15)];
        wt[cb] = w3[cb * 16 + (lane & 15)];
    }
    const float bias3 = b3[0];
    __builtin_amdgcn_sched_barrier(0);
    floatx4 acc[NCB];
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[cb][i] = 0.0f;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        float4 a = v[0][u];
#pragma unroll
        for (int q = 1; q < KSPLIT; ++q) {
            a.x = a.x + v[q][u].x;
            a.y = a.y + v[q][u].y;
            a.z = a.z + v[q][u].z;
            a.w = a.w + v[q][u].w;
        }
        a.x = a.x + c[u].x;
        a.y = a.y + c[u].y;
        a.z = a.z + c[u].z;
        a.w = a.w + c[u].w;
        a.x = a.x > 0.0f ? a.x : 0.0f;
        a.y = a.y > 0.0f ? a.y : 0.0f;
        a.z = a.z > 0.0f ? a.z : 0.0f;
        a.w = a.w > 0.0f ? a.w : 0.0f;
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) {
            acc[cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x, bw[cb][u].x, acc[cb], 0, 0, 0);
            acc[cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.y, bw[cb][u].y, acc[cb], 0, 0, 0);
            acc[cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.z, bw[cb][u].z, acc[cb], 0, 0, 0);
            acc[cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.w, bw[cb][u].w, acc[cb], 0, 0, 0);
        }
    }
    // C layout: lane l holds column 16 cb + l mod 16, rows 4 (l / 16) + i
    if (wave > 0) {
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
            for (int i = 0; i < 4; ++i) hsum[wave - 1][cb * 4 + i][lane] = acc[cb][i];
    }
    __syncthreads();
    if (wave == 0) {
        // layer 2 complete (eighths in order); layer 3: each lane's four
        // columns' weights times relu(h2) for its 4 rows, then the sum over
        // the 16 lanes that share those rows
        float t[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) t[i] = 0.0f;
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float h2 = acc[cb][i];
#pragma unroll
                for (int q = 0; q < NW - 1; ++q) h2 = h2 + hsum[q][cb * 4 + i][lane];
                h2 = h2 + bias[cb];
                t[i] = t[i] + wt[cb] * (h2 > 0.0f ? h2 : 0.0f);
            }
        }
#pragma unroll
        for (int o = 1; o < 16; o <<= 1)
#pragma unroll
            for (int i = 0; i < 4; ++i) t[i] = t[i] + __shfl_xor(t[i], o);
        if ((lane & 15) == 0) {
#pragma unroll
            for (int i = 0; i < 4; ++i) ysum[grp * 4 + i] = t[i];
        }
    }
    __syncthreads();
    if (threadIdx.x < L23_ROWS) {
        const int r = r0 + threadIdx.x;
        const float y = ysum[threadIdx.x] + bias3;
        if (r < n) {
            logit[r] = y;
            if (pred) pred[r] = y > 0.0f ? 1 : 0;
        }
    }
}

}  // namespace

// Layer 1's partial sums for sae_predict_sessions_noalloc: device memory of the
// library's own (each GPU holds its own copy of the array until the process
// ends).  Host code never passes `scratch` itself to a kernel (on the host it
// is only a stand-in for the symbol); it passes the device address that
// hipGetSymbolAddress returned for the current device.
static __device__ __align__(256) float scratch[(size_t)KSPLIT * SAE_PRED_NOALLOC_MAX_N * SAE_PRED_H1];

// The device address of `scratch` on the current device, looked up with that
// device current on its first use and kept per device.
hipError_t predict_scratch(float **out)
{
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static void *addr[kMaxDevices] = {};
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        addr[dev] = p;
    }
    *out = static_cast<float *>(addr[dev]);
    return hipSuccess;
}

// Up to 2,048 rows the 128-wide tiles are at most 128 workgroups, half of the
// compute units, and a workgroup's time is its bytes over what its unit is fed:
// 64-wide tiles halve those bytes and quadruple the workgroups.  Layer 1 at d =
// 4,096 on hidden states that no cache holds, 64- against 128-wide: 6.4 / 12.1 us at
// 1 and 256 rows, 7.8 / 12.1 at 1,024, 14.2 / 14.0 at 2,048, 30.9 / 17.8 at 4,096 (there the
// 64-wide tiles move twice the bytes).  A unit is fed 42 KB/us (512 KB in 12.1
// us) while a quarter of them work and 29 KB/us when all do: together 7.5 TB/s.
constexpr int L1_64_MAX_ROWS = 2048;

hipError_t launch_predict(int n, int d, const uint16_t *h, const uint16_t *w1, const float *b1, const float *w2,
                          const float *b2, const float *w3, const float *b3, float *work, float *logit,
                          uint8_t *pred, hipStream_t s)
{
    const int tile = n <= L1_64_MAX_ROWS ? 64 : 128;
    const int row_tiles = (n + tile - 1) / tile;
    const int groups = (row_tiles + 7) / 8;  // rounds of 8 row tiles, one per XCD
    const dim3 grid(groups * 8 * KSPLIT * (SAE_PRED_H1 / tile));
    if (tile == 64)
        hipLaunchKernelGGL(k_pred_l1<64>, grid, dim3(L1_THREADS), 0, s, n, d, h, w1, work, row_tiles);
    else
        hipLaunchKernelGGL(k_pred_l1<128>, grid, dim3(L1_THREADS), 0, s, n, d, h, w1, work, row_tiles);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_pred_l23, dim3((n + L23_ROWS - 1) / L23_ROWS), dim3(L23_THREADS), 0, s, n, work, b1, w2, b2,
                       w3, b3, logit, pred);
    return hipGetLastError();
}
