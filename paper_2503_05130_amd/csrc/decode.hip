// The decode step's kernels for gfx950: attention over the KV cache (first) and
// the skinny products that read every weight once (below).
//
// Decode-phase attention: one new query per (batch, head) against
// the keys 0 .. n_keys - 1 of a KV cache.  Memory-bound: every cached K and V
// element is read once, nothing else of size.
//
// The keys are split into chunks of CH (64 up to 2048 keys, else 256; at most
// 32 chunks); a workgroup (4 waves) takes one chunk of one (batch, head), so a
// decode step of a few sequences still has enough workgroups to keep HBM busy:
//   1. scores: a key row of K (dh bf16) is read by dh / 8 consecutive lanes,
//      16 bytes each, all of the chunk's rows issued before any is used; a
//      butterfly over those lanes sums the row.  Scores (times log2 e /
//      sqrt(dh)) go to LDS.
//   2. the chunk's max m_c, p_j = 2^(s_j - m_c) and their sum l_c.
//   3. the chunk's context: V is cached transposed, [dh, positions], so a V^T
//      row is contiguous over the chunk's keys: CH / 8 lanes read one row (8
//      keys each), multiply with p_j and reduce.  (m_c, l_c, acc_c[dh]) go to
//      the chunk's slot of a partials buffer.
//   4. a second kernel combines the chunks of each (batch, head):
//      M = max m_c, ctx = sum_c 2^(m_c - M) acc_c / sum_c 2^(m_c - M) l_c, in
//      chunk order.  (Handing the partials over at the kernel boundary keeps
//      the workgroups free of device-scope fences, which on this chip write
//      back and invalidate a whole XCD L2 each.)  A single chunk writes its
//      context directly and needs no second kernel.  The chunking depends on
//      n_keys alone, so a sequence's result depends neither on the batch nor
//      on the CUs used.
// Positions past n_keys of the cache may hold any bits: they are never
// multiplied (masked, not zeroed by arithmetic).
//
// Precision: fp32 scores, softmax and sums; q, K, V are bf16 as stored; the
// context is rounded to bf16 (the out-projection's operand).
#include "gemm_device.h"
#include "kernels.h"

namespace iefwd {
namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;
constexpr int kMaxKeys = 8192;
constexpr int kSmallChunk = 64, kLargeChunk = 256, kSmallLimit = 2048;

__device__ inline float lo_bf16(uint32_t w) { return __uint_as_float(w << 16); }
__device__ inline float hi_bf16(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

__device__ inline float dot8(u32x4 a, const float (&q)[8]) {
    float s = lo_bf16(a[0]) * q[0];
    s = fmaf(hi_bf16(a[0]), q[1], s);
    s = fmaf(lo_bf16(a[1]), q[2], s);
    s = fmaf(hi_bf16(a[1]), q[3], s);
    s = fmaf(lo_bf16(a[2]), q[4], s);
    s = fmaf(hi_bf16(a[2]), q[5], s);
    s = fmaf(lo_bf16(a[3]), q[6], s);
    s = fmaf(hi_bf16(a[3]), q[7], s);
    return s;
}

__device__ inline float wave_max(float v) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
    return v;
}

__device__ inline float wave_sum(float v) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

__device__ inline uint16_t to_bf16_bits(float f) {
    __bf16 b = (__bf16)f;
    return __builtin_bit_cast(uint16_t, b);
}

template <int DH, int CH>
__global__ __launch_bounds__(kThreads) void decode_attention_kernel(
    const bf16_t *__restrict__ Q, const bf16_t *__restrict__ K, const bf16_t *__restrict__ Vt,
    bf16_t *__restrict__ ctx, float *__restrict__ partials, int n_keys, int k_rows, int vt_stride,
    float scale_log2e) {
    constexpr int LPK = DH / 8;                  // lanes per key row of K
    constexpr int KPI = kThreads / LPK;          // key rows per workgroup load
    constexpr int NLOAD = CH / KPI;              // K loads per thread
    constexpr int LPR = CH / 8;                  // lanes per V^T row
    constexpr int RPP = kThreads / LPR;          // V^T rows per pass
    constexpr int SLOT = DH + 2;                 // floats per chunk slot: m, l, acc[DH]
    static_assert(NLOAD >= 1 && CH <= kThreads && DH % RPP == 0, "chunk shape");
    __shared__ float sc[CH];
    __shared__ float red[2 * kWaves];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int chunk = blockIdx.x, n_chunks = gridDim.x, bh = blockIdx.y;
    const int j0 = chunk * CH, nk = min(CH, n_keys - j0);     // this chunk's keys
    const bf16_t *Kh = K + (size_t)bh * k_rows * DH;
    const bf16_t *Vh = Vt + (size_t)bh * DH * vt_stride;

    // this lane's 8 elements of q
    const int part = tid % LPK;
    float q[8];
    {
        const u32x4 w = *reinterpret_cast<const u32x4 *>(Q + (size_t)bh * DH + part * 8);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            q[2 * e] = lo_bf16(w[e]);
            q[2 * e + 1] = hi_bf16(w[e]);
        }
    }

    // 1. scores: all loads first (rows past n_keys are clamped to the last key:
    // read, never used), and with them the V^T rows of step 3, which depend on
    // nothing computed here: one memory round trip for the whole chunk
    u32x4 kr[NLOAD];
#pragma unroll
    for (int i = 0; i < NLOAD; ++i) {
        const int j = min(j0 + i * KPI + tid / LPK, n_keys - 1);
        kr[i] = *reinterpret_cast<const u32x4 *>(Kh + (size_t)j * DH + part * 8);
    }
    const int r_in = tid / LPR, kk = (tid % LPR) * 8;
    const int kread = min(j0 + kk, vt_stride - 8);    // 16-byte aligned, inside the row; masked below
    u32x4 vr[DH / RPP];
#pragma unroll
    for (int i = 0; i < DH / RPP; ++i)
        vr[i] = *reinterpret_cast<const u32x4 *>(Vh + (size_t)(i * RPP + r_in) * vt_stride + kread);
    float mx = -INFINITY;
#pragma unroll
    for (int i = 0; i < NLOAD; ++i) {
        const int jl = i * KPI + tid / LPK;      // key within the chunk
        float s = dot8(kr[i], q);
#pragma unroll
        for (int o = LPK / 2; o >= 1; o >>= 1) s += __shfl_xor(s, o);
        s *= scale_log2e;
        if (jl < nk) {
            if (part == 0) sc[jl] = s;
            mx = fmaxf(mx, s);
        }
    }
    mx = wave_max(mx);
    if (lane == 0) red[wave] = mx;
    __syncthreads();
    mx = red[0];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) mx = fmaxf(mx, red[w]);

    // 2. probabilities and their sum
    float p = 0.f;
    if (tid < nk) {
        p = __builtin_amdgcn_exp2f(sc[tid] - mx);
        sc[tid] = p;
    }
    const float wsum = wave_sum(p);
    if (lane == 0) red[kWaves + wave] = wsum;
    __syncthreads();
    float l = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) l += red[kWaves + w];

    // 3. the chunk's context: RPP rows of V^T per pass, LPR lanes x 8 keys per row
    float pk[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) pk[e] = kk + e < nk ? sc[kk + e] : 0.f;
    const bool single = n_chunks == 1;
    float *slot = partials + ((size_t)bh * n_chunks + chunk) * SLOT;
    const float inv_l = 1.0f / l;
#pragma unroll
    for (int i = 0; i < DH / RPP; ++i) {
        float acc = 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (kk + 2 * e < nk) acc = fmaf(pk[2 * e], lo_bf16(vr[i][e]), acc);
            if (kk + 2 * e + 1 < nk) acc = fmaf(pk[2 * e + 1], hi_bf16(vr[i][e]), acc);
        }
#pragma unroll
        for (int o = LPR / 2; o >= 1; o >>= 1) acc += __shfl_xor(acc, o);
        if (tid % LPR == 0) {
            const int dd = i * RPP + r_in;
            if (single)
                ctx[(size_t)bh * DH + dd] = to_bf16_bits(acc * inv_l);
            else
                slot[2 + dd] = acc;
        }
    }
    if (tid == 0 && !single) {
        slot[0] = mx;
        slot[1] = l;
    }
}

// 4. one workgroup of DH threads per (batch, head): the chunks' weights from
// their maxima, then every context element summed over the chunks in order.
// Every partial this thread needs is requested before the first is used.
template <int DH>
__global__ __launch_bounds__(DH) void decode_combine_kernel(const float *__restrict__ partials,
                                                            bf16_t *__restrict__ ctx, int n_chunks) {
    constexpr int SLOT = DH + 2;
    __shared__ float wc[kDecodeMaxChunks];
    __shared__ float lsum;
    const int tid = threadIdx.x, bh = blockIdx.x;
    const float *slots = partials + (size_t)bh * n_chunks * SLOT;
    float part[kDecodeMaxChunks];
#pragma unroll
    for (int c = 0; c < kDecodeMaxChunks; ++c)
        part[c] = slots[min(c, n_chunks - 1) * SLOT + 2 + tid];   // clamped: past n_chunks never used
    if (tid < 64) {
        const bool has = tid < n_chunks;
        const float m = has ? slots[tid * SLOT] : -INFINITY;
        const float M = wave_max(m);
        const float w = has ? __builtin_amdgcn_exp2f(m - M) : 0.f;
        const float ls = wave_sum(has ? w * slots[tid * SLOT + 1] : 0.f);
        if (tid < kDecodeMaxChunks) wc[tid] = w;
        if (tid == 0) lsum = ls;
    }
    __syncthreads();
    float acc = 0.f;
#pragma unroll
    for (int c = 0; c < kDecodeMaxChunks; ++c)
        if (c < n_chunks) acc = fmaf(wc[c], part[c], acc);
    ctx[(size_t)bh * DH + tid] = to_bf16_bits(acc / lsum);
}

template <int DH>
hipError_t launch_dh(const bf16_t *q, const bf16_t *k, const bf16_t *vt, bf16_t *ctx, int bh, int n_keys,
                     int k_rows, int vt_stride, float *partials, hipStream_t stream) {
    const float scale = 1.4426950408889634f / sqrtf((float)DH);
    const int n_chunks = decode_attention_chunks(n_keys);
    const dim3 grid(n_chunks, bh), block(kThreads);
    const hipError_t e =
        n_keys <= kSmallLimit
            ? launch_kernel(decode_attention_kernel<DH, kSmallChunk>, grid, block, stream, q, k, vt, ctx, partials,
                            n_keys, k_rows, vt_stride, scale)
            : launch_kernel(decode_attention_kernel<DH, kLargeChunk>, grid, block, stream, q, k, vt, ctx, partials,
                            n_keys, k_rows, vt_stride, scale);
    if (e != hipSuccess || n_chunks == 1) return e;
    return launch_kernel(decode_combine_kernel<DH>, dim3(bh), dim3(DH), stream, (const float *)partials, ctx,
                         n_chunks);
}

}  // namespace

int decode_attention_chunks(int n_keys) {
    const int ch = n_keys <= kSmallLimit ? kSmallChunk : kLargeChunk;
    return (n_keys + ch - 1) / ch;
}

hipError_t launch_decode_attention(const bf16_t *q, const bf16_t *k, const bf16_t *vt, bf16_t *ctx, int batch,
                                   int n_heads, int n_keys, int head_dim, int k_rows, int vt_stride,
                                   float *partials, hipStream_t stream) {
    if (batch <= 0) return hipSuccess;
    if (n_keys <= 0 || n_keys > kMaxKeys || k_rows < n_keys || vt_stride < n_keys || vt_stride % 64 != 0 ||
        (long)batch * n_heads > 65535 || !partials)
        return hipErrorInvalidValue;
    if (head_dim == 64)
        return launch_dh<64>(q, k, vt, ctx, batch * n_heads, n_keys, k_rows, vt_stride, partials, stream);
    if (head_dim == 128)
        return launch_dh<128>(q, k, vt, ctx, batch * n_heads, n_keys, k_rows, vt_stride, partials, stream);
    return hipErrorInvalidValue;
}

namespace {

template <int CTRL>
__device__ inline float dpp_move(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, false));
}

// Sum over the wave's 64 lanes, the same value in every lane, in a fixed
// order: lane pairs and pairs of pairs within each quad (DPP quad permutes
// [1,0,3,2] and [2,3,0,1]), quads within each half row (row_half_mirror),
// halves within each row of 16 (row_mirror), then the four row sums as
// (r0 + r1) + (r2 + r3).  Each partner exchange adds the same two values in
// both lanes, so every lane of a group holds bitwise the same sum.
__device__ inline float row_sum(float v) {
    v += dpp_move<0xB1>(v);
    v += dpp_move<0x4E>(v);
    v += dpp_move<0x141>(v);
    v += dpp_move<0x140>(v);
    const int b = __builtin_bit_cast(int, v);
    const float r0 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 0));
    const float r1 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 16));
    const float r2 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 32));
    const float r3 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 48));
    return (r0 + r1) + (r2 + r3);
}

// ---------------------------------------------------------------- skinny GEMM (decode)
//
// M <= 16 token rows (one decode step of a batch): the product is bound by
// reading W once, so what matters is how many weight bytes are in flight on
// how many CUs.  A workgroup of 8 waves owns 16 / G output features and the
// whole of K, cut into G equal K-groups that one MFMA works on side by side:
// operand row (g, f) holds feature f's weights of K-group g, operand column
// (g, t) token t's activations of K-group g, and the diagonal blocks of the
// 16 x 16 product (row group == column group) are the per-group partial sums,
// added over g at the end (the off-diagonal blocks are discarded).  G = 1, 2
// or 4 (up to 16 / G tokens) is the largest whose N / (16 / G) workgroups all
// fit the chip at once.  The waves split the K steps (wave w takes w, w + 8,
// ...); each lane loads its weight and activation fragments straight into
// registers (16 bytes each; token columns past M repeat the last row and are
// never stored), as many K steps deep as the wave has, up to 8.  The waves' partial sums are added in wave order through
// LDS, then the K-groups in group order through lane shuffles: the summation
// order depends on K and G only.
//
// With a LayerNorm prologue the activations are LayerNorm(z) of fp32 rows z
// (a pre-LN block's input), normalised by the workgroup itself into LDS as
// bf16 while the first weight fragments are already in flight.  Needs
// M * K <= kSkinnyLnElems and K <= 4096.
//
// Weights come either row-major ([N, K]: one load instruction covers 16 rows
// x 64 bytes) or packed: a copy of W in which the 64 lanes' 16-byte pieces of
// one (workgroup, K step) fragment are one contiguous 1 KB block, in lane
// order, blocks ordered by workgroup then K step.  A load instruction then
// reads 1 KB of consecutive addresses, which streams from HBM at the rate of a
// plain copy; the fragments, the MFMAs and the summation order are the same in
// both forms, so the results are bit-identical.  The packed copy is made for
// one K-group count (skinny_pack).  A product of fewer groups, of a larger
// batch, reads it in 64-byte pieces of 4 (2) blocks that lie next to each
// other: less than its own copy would give and more than row-major weights (us
// row-major / this / own copy: 16 x 4096 -> 1024 10.5 / 9.4 / 8.4, 16 x 8192 ->
// 2048 19.0 / 17.4 / 15.5, 8 x 4096 -> 1024 6.2 / 5.7 / 5.2, 16 x 1024 -> 3072 with
// LayerNorm 6.1 / 5.9 / 6.0), without that copy's memory.  The epilogue's
// operands (bias, residual rows) and, without the LayerNorm prologue, the
// activations are requested before the weights, so that no load is left to
// start after the weight stream has ended.
constexpr int kSkinnyWaves = 8, kSkinnyUnroll = 8;
constexpr int kSkinnyLnElems = 16384;
constexpr int kSkinnyCus = 256;              // MI355X compute units

// One wave per row (rows w and w + 8 for wave w), the row held in registers
// (lane l owns the f32x4 vectors l + 64 c).  load() issues the wave's first
// row (waves past the last row load none) and this thread's share of gamma
// and beta -- before the weight fragments, so that they are not queued behind
// them; finish() stages gamma and beta in LDS,
// takes mean and rstd two-pass over the registers with a fixed reduction tree (row_sum) and
// writes y = fma(gamma, (z - mean) * rstd, beta), rounded to bf16, into the
// activation tile.  NVL = K / 256 rounded up to 8 or 16 (K <= 4096).
// finish() contains one barrier, reached by every wave.
// TWO (M > 8): the wave's second row is requested with the first, ahead of the
// weights; requested after them it would arrive when the weight stream ends.
// Rows of the activation tile are K + 8 elements apart, so that the 16 rows a
// fragment read touches lie in distinct banks (16 rows x 1024: QKV and FFN-up
// of 1024 x 3072 and 1024 x 4096 together 14.5 -> 12.9 us with the packed copy).
template <int NVL, bool TWO>
struct SkinnyLn {
    static constexpr int GBV = NVL * 64 / (64 * kSkinnyWaves);   // gamma / beta vectors per thread
    f32x4 v[NVL], v2[TWO ? NVL : 1];
    f32x4 g[GBV], b[GBV];

    // Every vector of the row is loaded (indices clamped into the row; the
    // extra vectors are never used), so that the wait for them does not wait
    // for the weights.
    __device__ static void load_row(const GemmParams &p, f32x4 (&v)[NVL], int r, int lane) {
        const f32x4 *zr = reinterpret_cast<const f32x4 *>(p.lnin.z + (size_t)r * p.K);
#pragma unroll
        for (int c = 0; c < NVL; ++c) v[c] = zr[min(c * 64 + lane, p.K / 4 - 1)];
    }

    __device__ void load(const GemmParams &p, int tid, int lane, int wave) {
#pragma unroll
        for (int j = 0; j < GBV; ++j) {
            const int i = min(tid + j * 64 * kSkinnyWaves, p.K / 4 - 1);
            g[j] = reinterpret_cast<const f32x4 *>(p.lnin.gamma)[i];
            b[j] = reinterpret_cast<const f32x4 *>(p.lnin.beta)[i];
        }
        if constexpr (TWO) {
            load_row(p, v, wave, lane);   // M > 8: every wave has a first row
            load_row(p, v2, min(wave + kSkinnyWaves, p.M - 1), lane);
        } else if (wave < p.M) {
            load_row(p, v, wave, lane);
        }
    }

    __device__ void finish(const GemmParams &p, bf16_t *a_lds, float *gb_lds, int tid, int lane, int wave) {
        const int nv = p.K / 4;
        const float inv_k = 1.0f / (float)p.K;
        f32x4 *g_l = reinterpret_cast<f32x4 *>(gb_lds), *b_l = g_l + nv;
#pragma unroll
        for (int j = 0; j < GBV; ++j) {
            const int i = tid + j * 64 * kSkinnyWaves;
            if (i < nv) {
                g_l[i] = g[j];
                b_l[i] = b[j];
            }
        }
        float mean = 0.f, rstd = 0.f;
        auto stats = [&](const f32x4 (&v)[NVL]) {
            float sum = 0.f;
#pragma unroll
            for (int c = 0; c < NVL; ++c)
                if (c * 64 + lane < nv) sum += v[c][0] + v[c][1] + v[c][2] + v[c][3];
            mean = row_sum(sum) * inv_k;
            float ss = 0.f;
#pragma unroll
            for (int c = 0; c < NVL; ++c)
                if (c * 64 + lane < nv)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float d = v[c][e] - mean;
                        ss += d * d;
                    }
            rstd = 1.0f / sqrtf(row_sum(ss) * inv_k + p.lnin.eps);
        };
        // gamma and beta of two vectors read before either is used (indices
        // clamped: unused past the row)
        auto emit = [&](const f32x4 (&v)[NVL], int r) {
#pragma unroll
            for (int c = 0; c < NVL; c += 2) {
                f32x4 gg[2], bb[2];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int i = min((c + h) * 64 + lane, nv - 1);
                    gg[h] = g_l[i];
                    bb[h] = b_l[i];
                }
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int i = (c + h) * 64 + lane;
                    if (i < nv) {
                        float y[4];
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            y[e] = __builtin_fmaf(gg[h][e], (v[c + h][e] - mean) * rstd, bb[h][e]);
                        *reinterpret_cast<u32x2 *>(a_lds + (size_t)r * (p.K + 8) + 4 * i) =
                            u32x2{pack2(y[0], y[1]), pack2(y[2], y[3])};
                    }
                }
            }
        };
        if (TWO || wave < p.M) stats(v);
        __syncthreads();                      // gamma and beta staged
        if (TWO || wave < p.M) emit(v, wave);
        if constexpr (TWO) {
            if (wave + kSkinnyWaves < p.M) {
                stats(v2);
                emit(v2, wave + kSkinnyWaves);
            }
        }
    }
};

// NVL: 0 = activations from a; 8 or 16 = LayerNorm prologue for K <= 2048 / 4096.
// Q: 0 = p.w is row-major; 1, 2, 4 = p.w is the packed copy of W (skinny_pack)
// for G Q K-groups.  U: K steps a
// wave requests at once (skinny_unroll).  TWO: 9-16 rows with the LayerNorm
// prologue.
template <Epi EPI, int G, int NVL, int Q, int U, bool TWO>
__global__ __launch_bounds__(64 * kSkinnyWaves) void skinny_kernel(GemmParams p) {
    constexpr bool LNA = NVL > 0;
    constexpr int NW = kSkinnyWaves;
    constexpr int FPW = 16 / G, TPW = 16 / G;      // features and token columns per K-group
    constexpr int kPartBytes = (NW - 1) * 64 * 16;
    // the LayerNorm prologue's bf16 activation tile, later the waves' partial
    // sums; the prologue's gamma and beta (fp32, K each) in an array of their own
    constexpr int kLnBytes = (kSkinnyLnElems + 16 * 8) * 2;
    constexpr int kLdsBytes = LNA && kLnBytes > kPartBytes ? kLnBytes : kPartBytes;
    __shared__ __attribute__((aligned(16))) char lds[kLdsBytes];
    __shared__ __attribute__((aligned(16))) float gb_lds[LNA ? 2 * NVL * 256 : 4];
    f32x4 (*part)[64] = reinterpret_cast<f32x4 (*)[64]>(lds);
    bf16_t *a_lds = reinterpret_cast<bf16_t *>(lds);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n0 = blockIdx.x * FPW;
    const int row = lane & 15, chunk = lane >> 4;               // operand row / column, 8-element K chunk
    const int kg = p.K / G;                                     // K-group length
    const int grp = row / FPW;                                  // K-group of this lane's row and column
    const int wf_row = n0 + row % FPW, a_row = min(row % TPW, p.M - 1);
    const int steps = kg / 32;
    // Step s of this lane: row-major at wrow + 32 s; in its own packed copy at
    // wrow + 512 s; in the copy for Q times the K-groups, a block of which holds
    // 16 / (G Q) features, step s is step s % (steps / Q) of that copy's K-group
    // grp Q + s / (steps / Q), whose rows lie 16 / (G Q) pieces further on
    constexpr int CPW = 16 / (G * (Q ? Q : 1));   // features of a block of the copy
    const int csteps = Q > 1 ? steps / Q : steps;
    const bf16_t *wrow = Q > 1    ? p.w + (size_t)(wf_row / CPW) * csteps * 512 +
                                     (chunk * 16 + grp * Q * CPW + wf_row % CPW) * 8
                         : Q == 1 ? p.w + (size_t)blockIdx.x * steps * 512 + lane * 8
                                  : p.w + (size_t)wf_row * p.K + grp * kg + chunk * 8;
    auto w_step = [&](int s) {
        if constexpr (Q == 0) return s * 32;
        int g = 0;
#pragma unroll
        for (int i = 1; i < Q; ++i) g += s >= i * csteps;
        return (s - g * csteps) * 512 + g * CPW * 8;
    };
    const bf16_t *arow = (LNA ? a_lds : p.a) + (size_t)a_row * (LNA ? p.K + 8 : p.K) + grp * kg + chunk * 8;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    // The epilogue's operands are fetched first.  Lane (fq, t) of wave 0
    // stores features n0 + 4 fq .. + 3 of token t (see below); every lane
    // loads (indices clamped into the operands, no branch), so that no wait
    // for these loads is placed ahead of the weights'.
    const int fq = lane / TPW, t = lane % TPW;
    const bool stores = wave == 0 && lane < (FPW / 4) * TPW && t < p.M;
    const int f_out = n0 + 4 * fq;
    const u32x2 braw = *reinterpret_cast<const u32x2 *>(p.bias + min(f_out, p.N - 4));
    f32x4 rres = {0.f, 0.f, 0.f, 0.f};
    if constexpr (EPI == Epi::BiasResidF32)
        rres = *reinterpret_cast<const f32x4 *>(p.resid + (size_t)min(t, p.M - 1) * p.N + min(f_out, p.N - 4));
    // Fragments past the wave's last K step are replaced by zeros where the
    // MFMA takes them, and every MFMA runs: a skipped step adds exactly zero.
    // (A conditional MFMA may be issued with the wave's EXEC mask empty, which
    // does not stop it from reading its operand registers.)  The selection sits
    // at the MFMA, not at the load, so that no MFMA waits for a later fragment.
    const bf16x8 zero = {};
    bf16x8 wf[U], af[U];
    // Every load is issued, steps past the wave's last one clamped to it
    // (their fragments are zeroed at the MFMA): no branch around a load, so
    // each MFMA waits for its own fragments alone
    auto load_w = [&](int s0) {
#pragma unroll
        for (int u = 0; u < U; ++u)
            wf[u] = *reinterpret_cast<const bf16x8 *>(wrow + w_step(min(s0 + u * NW, steps - 1)));
    };
    auto load_a = [&](int s0) {
#pragma unroll
        for (int u = 0; u < U; ++u)
            af[u] = *reinterpret_cast<const bf16x8 *>(arow + min(s0 + u * NW, steps - 1) * 32);
    };
    if constexpr (LNA) {
        // the LayerNorm inputs first, then the weights; the activations are
        // normalised while the weights stream in
        SkinnyLn<NVL, TWO> ln;
        ln.load(p, threadIdx.x, lane, wave);
        __builtin_amdgcn_sched_barrier(0);     // keep these loads ahead of the weights' (in-order returns)
        load_w(wave);
        ln.finish(p, a_lds, gb_lds, threadIdx.x, lane, wave);
        __syncthreads();
    } else {
        // the first round's activations (L2-resident) ahead of the weights
        load_a(wave);
        load_w(wave);
    }
    for (int s0 = wave; s0 < steps; s0 += NW * U) {
        if (LNA || s0 != wave) load_a(s0);
#pragma unroll
        for (int u = 0; u < U; ++u)
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(s0 + u * NW < steps ? wf[u] : zero,
                                                          s0 + u * NW < steps ? af[u] : zero, acc, 0, 0, 0);
        if (s0 + NW * U < steps) load_w(s0 + NW * U);
    }
    if constexpr (LNA) __syncthreads();                        // the partials reuse the activations' LDS
    if (wave > 0) part[wave - 1][lane] = acc;
    __syncthreads();
    if (wave > 0) return;
#pragma unroll
    for (int w = 0; w < NW - 1; ++w) acc += part[w][lane];
    // lane l holds product rows 4 (l / 16) + e, column l % 16.  Output lane
    // (fq, t) gathers features 4 fq .. 4 fq + 3 of token t from the diagonal
    // block of every K-group: row g FPW + 4 fq + e, column g TPW + t.
    if constexpr (G > 1) {
        f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int src = (16 * (g * FPW / 4 + fq) + g * TPW + t) & 63;
#pragma unroll
            for (int e = 0; e < 4; ++e) sum[e] += __shfl(acc[e], src);
        }
        acc = sum;
    }
    if (!stores) return;
    const int f = f_out;
    // this lane: features f .. f + 3 of token t
    float v0 = acc[0] + __uint_as_float(braw[0] << 16), v1 = acc[1] + __uint_as_float(braw[0] & 0xffff0000u);
    float v2 = acc[2] + __uint_as_float(braw[1] << 16), v3 = acc[3] + __uint_as_float(braw[1] & 0xffff0000u);
    if constexpr (EPI == Epi::BiasBf16 || EPI == Epi::BiasGeluBf16) {
        if constexpr (EPI == Epi::BiasGeluBf16) {
            v0 = gelu(v0); v1 = gelu(v1); v2 = gelu(v2); v3 = gelu(v3);
        }
        *reinterpret_cast<u32x2 *>(static_cast<bf16_t *>(p.out) + (size_t)t * p.N + f) =
            u32x2{pack2(v0, v1), pack2(v2, v3)};
    } else if constexpr (EPI == Epi::BiasResidF32) {
        const f32x4 r = rres;
        *reinterpret_cast<f32x4 *>(static_cast<float *>(p.out) + (size_t)t * p.N + f) =
            f32x4{r[0] + v0, r[1] + v1, r[2] + v2, r[3] + v3};
    } else if constexpr (EPI == Epi::Qkv) {
        const QkvDst &d = p.qkv;
        const int which = f / d.d_model, within = f - which * d.d_model;
        const int head = within / d.head_dim, jj = within - head * d.head_dim;
        const int b = t / d.seq, sp = t - b * d.seq;
        const size_t bh = (size_t)b * d.n_heads + head;
        if (which < 2) {
            bf16_t *o = which == 0 ? d.q + (bh * d.seq + sp) * d.head_dim + jj
                                   : d.k + (bh * d.k_rows + d.pos0 + sp) * d.head_dim + jj;
            *reinterpret_cast<u32x2 *>(o) = u32x2{pack2(v0, v1), pack2(v2, v3)};
        } else {
            bf16_t *o = d.vt + (bh * d.head_dim + jj) * d.vt_stride + d.pos0 + sp;
            o[0] = f32_to_bf16(v0);
            o[d.vt_stride] = f32_to_bf16(v1);
            o[2 * (size_t)d.vt_stride] = f32_to_bf16(v2);
            o[3 * (size_t)d.vt_stride] = f32_to_bf16(v3);
        }
    }
}

template <int G, int NVL, int Q, int U, bool TWO>
hipError_t launch_skinny(Epi epi, const GemmParams &p, hipStream_t stream) {
    const dim3 grid(p.N / (16 / G)), block(64 * kSkinnyWaves);
    switch (epi) {
#define EPI(E) case E: return launch_kernel(skinny_kernel<E, G, NVL, Q, U, TWO>, grid, block, stream, p);
    EPI(Epi::BiasBf16) EPI(Epi::BiasGeluBf16) EPI(Epi::BiasResidF32) EPI(Epi::Qkv)
#undef EPI
    case Epi::BiasLnResidF32:
    case Epi::F32:
    case Epi::GeluBwdBf16:
    case Epi::BiasGelu2Bf16: break;
    }
    return hipErrorInvalidValue;
}

// K steps a wave requests at once: its share of the product's steps, rounded
// up to a power of two, at most kSkinnyUnroll (more steps take more rounds).
// Not kept for narrow long products of 9-16 rows, whose few workgroups pull
// their weights alone: 16 waves (another order of sums; 16 x 4096 -> 1024 8.35 ->
// 7.96 us, but 16 x 2048 -> 2048 5.20 -> 5.50), 16 steps at once (8.35 -> 8.18, but
// 16 x 8192 -> 2048 15.4 -> 17.5).
int skinny_unroll(int K, int G) {
    const int per_wave = (K / G / 32 + kSkinnyWaves - 1) / kSkinnyWaves;
    int u = 1;
    while (u < per_wave && u < kSkinnyUnroll) u *= 2;
    return u;
}

template <int G, int NVL, int Q, bool TWO>
hipError_t launch_skinny_u(Epi epi, const GemmParams &p, hipStream_t stream) {
    switch (skinny_unroll(p.K, G)) {
    case 1: return launch_skinny<G, NVL, Q, 1, TWO>(epi, p, stream);
    case 2: return launch_skinny<G, NVL, Q, 2, TWO>(epi, p, stream);
    case 4: return launch_skinny<G, NVL, Q, 4, TWO>(epi, p, stream);
    default: return launch_skinny<G, NVL, Q, 8, TWO>(epi, p, stream);
    }
}

template <int G, int NVL, int Q>
hipError_t launch_skinny_v(Epi epi, const GemmParams &p, hipStream_t stream) {
    if constexpr (G == 1 && NVL == 8) {   // more than 8 rows have one K-group, and K <= 16384 / 9
        if (p.M > 8) return launch_skinny_u<G, NVL, Q, true>(epi, p, stream);
    }
    return launch_skinny_u<G, NVL, Q, false>(epi, p, stream);
}

template <int G, int NVL>
hipError_t launch_skinny_q(Epi epi, const GemmParams &p, int q, hipStream_t stream) {
    switch (q) {
    case 0: return launch_skinny_v<G, NVL, 0>(epi, p, stream);
    case 1: return launch_skinny_v<G, NVL, 1>(epi, p, stream);
    case 2:
        if constexpr (G <= 2) return launch_skinny_v<G, NVL, 2>(epi, p, stream);
        break;
    case 4:
        if constexpr (G == 1) return launch_skinny_v<G, NVL, 4>(epi, p, stream);
        break;
    }
    return hipErrorInvalidValue;
}

template <int NVL>
hipError_t launch_skinny_g(Epi epi, const GemmParams &p, int g, int q, hipStream_t stream) {
    switch (g) {
    case 1: return launch_skinny_q<1, NVL>(epi, p, q, stream);
    case 2: return launch_skinny_q<2, NVL>(epi, p, q, stream);
    case 4: return launch_skinny_q<4, NVL>(epi, p, q, stream);
    }
    return hipErrorInvalidValue;
}

// Packed copy for the skinny product with G K-groups: 16-byte piece i of dst
// is what lane l of workgroup b loads at K step s in the row-major form, with
// i = (b * steps + s) * 64 + l; steps = K / (32 G).
template <int G>
__global__ __launch_bounds__(256) void skinny_pack_kernel(const bf16_t *w, bf16_t *dst, int N, int K) {
    constexpr int FPW = 16 / G;
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    const int kg = K / G, steps = kg / 32;
    if (i >= (size_t)N * K / 8) return;
    const int l = (int)(i % 64);
    const size_t bs = i / 64;
    const int s = (int)(bs % steps), b = (int)(bs / steps);
    const int row = l & 15, chunk = l >> 4;
    const int f = b * FPW + row % FPW, grp = row / FPW;
    const size_t k = (size_t)grp * kg + s * 32 + chunk * 8;
    reinterpret_cast<bf16x8 *>(dst)[i] = *reinterpret_cast<const bf16x8 *>(w + (size_t)f * K + k);
}

}  // namespace

int skinny_groups(int M, int N, int K, bool ln) {
    // more K-groups while the workgroups still fit the CUs in one round (3 per
    // CU, 2 with the LayerNorm prologue's registers and LDS), so that no
    // workgroup starts streaming its weights only after another has finished
    const int limit = (ln ? 2 : 3) * kSkinnyCus;
    int g = 1;
    while (g < 4 && N / (16 / (2 * g)) <= limit && M <= 16 / (2 * g) && K % (32 * 2 * g) == 0) g *= 2;
    return g;
}

bool skinny_ln_fits(int M, int K) {
    return M >= 1 && M <= 16 && K % 32 == 0 && K <= 4096 && M * K <= kSkinnyLnElems;
}

hipError_t launch_skinny_pack(const bf16_t *w, bf16_t *dst, int N, int K, int groups, hipStream_t stream) {
    if (N <= 0 || K <= 0 || (groups != 1 && groups != 2 && groups != 4)) return hipErrorInvalidValue;
    if (N % (16 / groups) || K % (32 * groups)) return hipErrorInvalidValue;
    const size_t pieces = (size_t)N * K / 8;
    const dim3 grid((unsigned)((pieces + 255) / 256)), block(256);
    switch (groups) {
    case 1: return launch_kernel(skinny_pack_kernel<1>, grid, block, stream, w, dst, N, K);
    case 2: return launch_kernel(skinny_pack_kernel<2>, grid, block, stream, w, dst, N, K);
    default: return launch_kernel(skinny_pack_kernel<4>, grid, block, stream, w, dst, N, K);
    }
}

hipError_t launch_gemm_skinny(Epi epi, const bf16_t *a, const bf16_t *w, const bf16_t *bias, const float *resid,
                              void *out, int M, int N, int K, const QkvDst *qkv, hipStream_t stream,
                              const LnIn *ln_in, const bf16_t *w_packed, int packed_groups) {
    if (M <= 0) return hipSuccess;
    if (M > 16 || N % 16 || K % 32 || epi == Epi::BiasLnResidF32 || epi == Epi::F32 || epi == Epi::GeluBwdBf16 ||
        epi == Epi::BiasGelu2Bf16)
        return hipErrorInvalidValue;
    if (ln_in && !skinny_ln_fits(M, K)) return hipErrorInvalidValue;
    GemmParams p{};
    p.a = a; p.w = w; p.bias = bias; p.resid = resid; p.out = out;
    p.M = M; p.N = N; p.K = K;
    if (qkv) p.qkv = *qkv;
    if (ln_in) p.lnin = *ln_in;
    const int g = skinny_groups(M, N, K, ln_in != nullptr);
    // a copy for fewer groups than the product's is not read (rows wider than 2048, 5-8 of them)
    const int q = w_packed && packed_groups % g == 0 ? packed_groups / g : 0;
    if (q) p.w = w_packed;
    if (!ln_in) return launch_skinny_g<0>(epi, p, g, q, stream);
    return K <= 2048 ? launch_skinny_g<8>(epi, p, g, q, stream) : launch_skinny_g<16>(epi, p, g, q, stream);
}

}  // namespace iefwd
