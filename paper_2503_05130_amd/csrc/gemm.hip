// bf16 MFMA GEMM with fused epilogues for gfx950 (CDNA4).
//
// out[t, f] = epilogue( sum_k A[t, k] * W[f, k] + bias[f] )
//   A: activations, bf16 [M, K] row-major (tokens x features-in)
//   W: weights stored output-major, bf16 [N, K] row-major
//
// Data movement.  K is walked in 64-wide tiles (rows of 128 bytes, whole cache
// lines).  Each tile of A and of W is copied from global memory straight into
// LDS with global_load_lds_dwordx4 (gfx950's 16-byte global->LDS DMA: no VGPR
// staging) into a ring of slots, one ring for A and one for W; a tile's 1 KB
// copies are spread over all waves.  The 16-byte chunks of a row are
// XOR-swizzled, so that the 16 rows read by one ds_read_b128 fragment load
// fall in distinct banks; the swizzle is applied on the source side (lane i of
// a copy fetches the global chunk that belongs at its fixed LDS place).  A
// copy's address is a scalar base that walks K plus a 32-bit lane offset that
// never changes, so the loop holds no vector address arithmetic.
//
// Math.  v_mfma_f32_16x16x32_bf16 on C^T blocks (features x tokens): the W
// fragment is the MFMA "A" operand, the activation fragment the "B" operand,
// so each lane ends up owning 4 consecutive output features of one token and
// stores them with one vector store.
//
// Determinism and batch invariance: every configuration uses the same MFMA
// instruction; the K summation order (32-wide K chunks in sequence, or the
// even and the odd 64-wide tiles summed separately, then added, for long K) is
// a function of the weight shape (N, K) alone.  So out[t, f] depends only on
// row t of A and row f of W -- never on the tile shape, the ring depth, the
// grid, the CU mask or the other rows in the batch.  No atomics, no
// cross-workgroup split-K.
#include <algorithm>

#include "gemm_device.h"

namespace iefwd {
namespace {

// Workgroups are dispatched round-robin over the 8 XCDs.  Renumber them so
// that each XCD receives a contiguous range of logical tiles (bijective for
// any grid size), which keeps tiles that share operands in one XCD's L2.
__device__ inline int xcd_contiguous(int i, int g) {
    constexpr int X = 8;
    const int q = g / X, r = g % X;
    const int x = i % X, local = i / X;
    return x < r ? x * (q + 1) + local : r * (q + 1) + (x - r) * q + local;
}

// Logical tile -> (token tile, feature tile), grouped 4 token tiles deep so
// that workgroups running together share both A rows and W rows.
__device__ inline void grouped_tile(int l, int tiles_m, int tiles_n, int &tm, int &tn) {
    constexpr int G = 4;
    const int per_group = G * tiles_n;
    const int g = l / per_group;
    const int first = g * G;
    const int gsize = min(tiles_m - first, G);
    const int in = l - g * per_group;
    tm = first + in % gsize;
    tn = in / gsize;
}

// 16-byte chunk position of logical chunk 0 in LDS row r of a K tile (row r
// holds its chunk c at position c ^ swizzle(r)), chosen so that the 16 rows one
// ds_read_b128 fragment load reads fall in distinct banks: consecutive 128-byte
// rows alternate between the two halves of a 256-byte bank line, and within
// each parity the 8 rows of a 16-row fragment get 8 distinct positions.
__device__ inline int swizzle(int r) { return ((r >> 1) & 7) ^ ((r & 1) << 2); }

// One global->LDS copy of 16 bytes per lane (1 KB per wave) to the
// wave-uniform LDS byte address `lds`.  Issued through inline asm: the
// compiler's wait-count model treats these copies as LDS traffic that may
// complete out of order with LDS reads, and would then drain every
// outstanding LDS read before each use of any of them; the main loop orders
// the copies itself (s_waitcnt vmcnt before each barrier).  The M0 write
// needs one wait state before the copy reads it.
__device__ inline void dma16(const bf16_t *base, uint32_t off, uint32_t lds) {
    uint32_t m0;   // the asm writes M0; naming it as an output tells the compiler so
    asm volatile("s_mov_b32 %0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 : "={m0}"(m0)
                 : "v"(off), "s"(base), "s"(lds)
                 : "memory");
    (void)m0;
}

// s_waitcnt immediate: wait until at most vm vector-memory and lgkm LDS
// operations of this wave are outstanding (expcnt left unconstrained).
constexpr int waitcnt_imm(int vm, int lgkm) { return (vm & 15) | (7 << 4) | ((lgkm & 15) << 8) | ((vm >> 4) << 14); }

// Tile configuration: BM x BN output tile of WGM x WGN waves; A tiles and W
// tiles of the K loop in a ring of S slots each, 64 K deep
// (128-byte rows: whole cache lines).  ORD is the K order: 1 adds the 32-wide
// K chunks in sequence, 2 adds the 64-wide K tiles of even and of odd index in
// sequence into an accumulator each, then the two.  AHEAD: a whole K tile's
// fragments are read one tile ahead instead of half a tile's one half ahead.
template <int BM_, int BN_, int WGM_, int WGN_, int ORD_, int S_, bool AHEAD_>
struct Cfg {
    static constexpr int BM = BM_, BN = BN_, WGM = WGM_, WGN = WGN_, ORD = ORD_, S = S_, BK = 64;
    static constexpr bool AHEAD = AHEAD_;
    static constexpr int NW = WGM * WGN, NT = 64 * NW;         // waves / threads per workgroup
    static constexpr int TM = BM / WGM, TN = BN / WGN;         // per-wave tile (tokens x features)
    static constexpr int FM = TM / 16, FN = TN / 16;           // 16 x 16 MFMA blocks per wave
    static constexpr int A_SLOT = BM * BK, W_SLOT = BN * BK;   // bf16 elements per ring slot
    static constexpr int RING = S * (A_SLOT + W_SLOT);
    static constexpr int GA = BM / 8, GW = BN / 8;             // 1 KB copies (8 rows) per slot
    static constexpr int DA = GA / NW, DW = (GW + NW - 1) / NW;   // per wave (at most)
    // waves per SIMD the register budget is sized for: as many workgroups as
    // the LDS ring allows share a CU (160 KB), at most 4 waves per SIMD
    static constexpr int WG_CU = 163840 / (RING * 2);
    static constexpr int WPE = WG_CU * NW / 4 >= 4 ? 4 : WG_CU * NW / 4 < 1 ? 1 : WG_CU * NW / 4;
    static_assert(TM % 16 == 0 && TN % 16 == 0 && BM % 16 == 0 && BN % 16 == 0, "tile");
    static_assert(ORD == 1 || ORD == 2, "K order");
    static_assert(GA % NW == 0, "waves share the A copies evenly");
    static_assert(S >= 2, "ring slots");
    static_assert((S - 1) * (DA + DW) <= 63, "ring depth (vmcnt holds 6 bits)");
};

// Waits until at most `t` K tiles' worth of this wave's copies (`per` each,
// PER or PER - 1) are still in flight.  t in [0, c]; the s_waitcnt immediate
// must be a constant, hence the recursion over the possible counts.
template <int PER, int c>
__device__ inline void wait_tiles(int t, int per) {
    if constexpr (c == 0) {
        __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, 15));
    } else {
        if (t >= c) {
            if constexpr (PER > 1) {
                if (per != PER) {
                    __builtin_amdgcn_s_waitcnt(waitcnt_imm(c * (PER - 1), 15));
                    return;
                }
            }
            __builtin_amdgcn_s_waitcnt(waitcnt_imm(c * PER, 15));
            return;
        }
        wait_tiles<PER, c - 1>(t, per);
    }
}

template <bool B> struct Flag { static constexpr bool value = B; };

// The main loop over the K tiles through the two rings.  Tile t of A and of W
// lives in slot t % S of its ring.  Step j multiplies tile j as two 32-deep
// halves:
//
//   !AHEAD: read half 1 of tile j; MFMAs of half 0;
//           wait (my copies of tile j + 1, my LDS reads), barrier: tile j + 1
//           is visible to all and no wave reads tile j's slots any more;
//           read half 0 of tile j + 1;
//           MFMAs of half 1, the copies of tile j + S issued between them
//           into the slots tile j left
//   AHEAD:  the wait and the barrier, read both halves of tile j + 1, then the
//           MFMAs of tile j with the copies between them
//
// so every fragment read has a half tile's (a tile's) MFMAs to hide behind,
// every copy S - 1 tiles' time, and the copies' issue slots fill the
// matrix unit's shadow.
//
// What bounds it (4096 tokens): the copies' rate is the bytes in flight over a
// latency of about 0.9 us (each tile has lines that no workgroup of the XCD has
// fetched yet), and the chip lowers its clock when copies, LDS reads and MFMAs
// overlap well: 1.6 GHz in the 3072 x 768 product, 1.8 to 1.95 GHz in longer
// ones, against 2.35 GHz with any of the three left out.  At that clock the
// 256 x 256 tile's loop keeps the matrix units busy 70 to 75% of the time.
// A ring slot more than listed with the tiles below does not help: the extra
// tile's copies delay the first MFMA by what they save later.
template <class C>
__device__ inline void main_loop(const GemmParams &p, bf16_t *lds, int wave, int lane, int m0, int n0,
                                 f32x4 (&acc)[C::ORD][C::FN][C::FM]) {
    constexpr int NW = C::NW, DA = C::DA, DW = C::DW, S = C::S, FM = C::FM, FN = C::FN;
    const int wm = wave % C::WGM, wn = wave / C::WGM;
    bf16_t *ring_a = lds, *ring_w = ring_a + S * C::A_SLOT;

    // Copy sources of this lane: copy i of this wave moves the 8-row group
    // wave + NW i of a slot; lane l fills row l / 8 of it at chunk position
    // l % 8.  Byte offsets from the tile's first row (the scalar base walks K).
    // Rows past M are clamped to the last valid row (never stored); N is a
    // multiple of BN.
    const int lr = lane / 8, lc = lane % 8;
    uint32_t off_a[DA], off_w[DW];
#pragma unroll
    for (int i = 0; i < DA; ++i) {
        const int r = 8 * (wave + NW * i) + lr;
        off_a[i] = 2 * ((uint32_t)min(r, p.M - 1 - m0) * (uint32_t)p.K + ((lc ^ swizzle(r)) * 8));
    }
#pragma unroll
    for (int i = 0; i < DW; ++i) {
        const int r = min(8 * (wave + NW * i), C::BN - 8) + lr;
        off_w[i] = 2 * ((uint32_t)r * (uint32_t)p.K + ((lc ^ swizzle(r)) * 8));
    }
    const bf16_t *base_a = p.a + (size_t)m0 * p.K, *base_w = p.w + (size_t)n0 * p.K;
    const uint32_t lds_a = (uint32_t)(size_t)(lds_ptr_t)ring_a + wave * 1024;
    const uint32_t lds_w = (uint32_t)(size_t)(lds_ptr_t)ring_w + wave * 1024;
    const int n = p.K / 64;
    const bool w_last = C::GW % NW == 0 || wave + NW * (DW - 1) < C::GW;   // this wave has a copy DW - 1
    const int per = DA + DW - !w_last;
    auto copy_w = [&](int t, int i) {
        if (i < DW - 1 || w_last)
            dma16(base_w + t * 64, off_w[i], lds_w + (t % S) * (C::W_SLOT * 2) + i * NW * 1024);
    };
    auto copy_a = [&](int t, int i) {
        dma16(base_a + t * 64, off_a[i], lds_a + (t % S) * (C::A_SLOT * 2) + i * NW * 1024);
    };
    // fragment rows: lane % 16 of each 16-row block; 16-byte chunk 4 half + lane / 16
    const int ra = wm * C::TM + (lane & 15), rw = wn * C::TN + (lane & 15);
    struct Frag {
        bf16x8 a[FM], w[FN];
    };
    auto read = [&](Frag &f, int t, int half) {
        const int c = half * 4 + (lane >> 4);
        const bf16_t *sa = ring_a + (t % S) * C::A_SLOT + ra * 64 + ((c ^ swizzle(ra)) * 8);
        const bf16_t *sw = ring_w + (t % S) * C::W_SLOT + rw * 64 + ((c ^ swizzle(rw)) * 8);
#pragma unroll
        for (int jj = 0; jj < FN; ++jj) f.w[jj] = *reinterpret_cast<const bf16x8 *>(sw + jj * 16 * 64);
#pragma unroll
        for (int i = 0; i < FM; ++i) f.a[i] = *reinterpret_cast<const bf16x8 *>(sa + i * 16 * 64);
    };
    // the MFMAs of one half tile; copies [D0, D1) of tile j + S (W's first) are
    // issued between them
    auto mfma = [&](f32x4 (&c)[FN][FM], const Frag &f, auto copies, auto &&issue, int d0, int d1) {
        constexpr int NM = FN * FM;
#pragma unroll
        for (int jj = 0; jj < FN; ++jj)
#pragma unroll
            for (int i = 0; i < FM; ++i) {
                c[jj][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.w[jj], f.a[i], c[jj][i], 0, 0, 0);
                if constexpr (decltype(copies)::value) {
                    const int q = jj * FM + i, nd = d1 - d0;
#pragma unroll
                    for (int d = q * nd / NM; d < (q + 1) * nd / NM; ++d) {
                        __builtin_amdgcn_sched_barrier(0);
                        issue(d0 + d);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            }
    };
    auto issue_full = [&](int j) {
        return [&, j](int d) {
            if (d < DW) copy_w(j + S, d);
            else copy_a(j + S, d - DW);
        };
    };
    auto issue_tail = [&](int j) {
        return [&, j](int d) {
            if (j + S >= n) return;
            if (d < DW) copy_w(j + S, d);
            else copy_a(j + S, d - DW);
        };
    };
    auto landed = [&](int j, auto full) {   // my copies of tile j + 1 have landed, my LDS reads have returned
        // (a count <= 0: all of them)
        wait_tiles<DA + DW, S - 2>(decltype(full)::value ? S - 2 : min(n, j + S) - (j + 2), per);
        __builtin_amdgcn_s_waitcnt(waitcnt_imm(63, 0));
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");   // keep LDS accesses on their side of the barrier
    };

#pragma unroll
    for (int t = 0; t < S; ++t) {
        if (t >= n) continue;
#pragma unroll
        for (int i = 0; i < DW; ++i) copy_w(t, i);
#pragma unroll
        for (int i = 0; i < DA; ++i) copy_a(t, i);
    }
    wait_tiles<DA + DW, S - 1>(min(n, S) - 1, per);   // tile 0 has landed
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if constexpr (!C::AHEAD) {
        Frag f0, f1;
        read(f0, 0, 0);
        auto step = [&](int j, f32x4 (&c)[FN][FM], auto full) {
            constexpr bool FULL = decltype(full)::value;
            read(f1, j, 1);
            __builtin_amdgcn_sched_barrier(0);
            mfma(c, f0, Flag<false>{}, [](int) {}, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            if (FULL || j + 1 < n) {
                landed(j, full);
                read(f0, j + 1, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (FULL) mfma(c, f1, Flag<true>{}, issue_full(j), 0, DA + DW);
            else mfma(c, f1, Flag<true>{}, issue_tail(j), 0, DA + DW);
            __builtin_amdgcn_sched_barrier(0);
        };
        int j = 0;
        if constexpr (C::ORD == 1) {
            for (; j + S < n; ++j) step(j, acc[0], Flag<true>{});
            for (; j < n; ++j) step(j, acc[0], Flag<false>{});
        } else {
            for (; j + 1 + S < n; j += 2) {
                step(j, acc[0], Flag<true>{});
                step(j + 1, acc[1], Flag<true>{});
            }
            for (; j < n; j += 2) {
                step(j, acc[0], Flag<false>{});
                if (j + 1 < n) step(j + 1, acc[1], Flag<false>{});
            }
        }
    } else {
        Frag f[2][2];
        read(f[0][0], 0, 0);
        read(f[0][1], 0, 1);
        auto step = [&](int j, f32x4 (&c)[FN][FM], Frag (&cur)[2], Frag (&next)[2], auto full) {
            constexpr bool FULL = decltype(full)::value;
            if (FULL || j + 1 < n) {
                landed(j, full);
                read(next[0], j + 1, 0);
                read(next[1], j + 1, 1);
            }
            __builtin_amdgcn_sched_barrier(0);
            constexpr int mid = (DA + DW) / 2;
            if constexpr (FULL) {
                mfma(c, cur[0], Flag<true>{}, issue_full(j), 0, mid);
                mfma(c, cur[1], Flag<true>{}, issue_full(j), mid, DA + DW);
            } else {
                mfma(c, cur[0], Flag<true>{}, issue_tail(j), 0, mid);
                mfma(c, cur[1], Flag<true>{}, issue_tail(j), mid, DA + DW);
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        int j = 0;
        for (; j + 1 + S < n; j += 2) {
            step(j, acc[0], f[0], f[1], Flag<true>{});
            step(j + 1, acc[C::ORD - 1], f[1], f[0], Flag<true>{});
        }
        for (; j < n; j += 2) {
            step(j, acc[0], f[0], f[1], Flag<false>{});
            if (j + 1 < n) step(j + 1, acc[C::ORD - 1], f[1], f[0], Flag<false>{});
        }
    }
}

// bf16 outputs (bias, bias + GELU, the QKV scatter) leave through LDS: each wave
// writes its finished values into an LDS copy of the output tile, then the
// whole workgroup stores it in 16-byte row segments.  Written straight from
// the MFMA layout, one store instruction would cover 16 rows x 32 bytes.
constexpr bool staged(Epi e) {
    return e == Epi::BiasBf16 || e == Epi::BiasGeluBf16 || e == Epi::Qkv || e == Epi::GeluBwdBf16 ||
           e == Epi::BiasGelu2Bf16;
}
constexpr bool has_bias(Epi e) { return e != Epi::F32 && e != Epi::GeluBwdBf16; }

// Epilogue operands that do not depend on the product (bias, residual rows,
// LayerNorm statistics and affine).  Configurations with two waves per SIMD
// and narrow wave tiles have registers to load them before the main loop, so
// that their latency hides behind the MFMAs (the residual rows too where the
// wave tile has at most 6 blocks).  The others load them after the loop: held
// through it they would spill (with the LayerNorm residual the 128 x 96 tile
// needs 16 registers more than four waves per SIMD leave).
template <class C, Epi EPI>
constexpr bool kEarlyInputs = C::FN <= 3 && (EPI != Epi::BiasLnResidF32 || C::WPE <= 2);

template <class C, Epi EPI>
struct EpiInputs {
    static constexpr int FM = C::FM, FN = C::FN;
    static constexpr bool kZ = (EPI == Epi::BiasResidF32 || EPI == Epi::BiasLnResidF32) && kEarlyInputs<C, EPI> &&
                               C::WPE <= 2 && FN * FM * C::ORD <= 6;
    u32x2 bias[FN];
    f32x4 z[kZ ? FN : 1][kZ ? FM : 1];
    f32x2 stats[EPI == Epi::BiasLnResidF32 ? FM : 1];
    f32x4 gamma[EPI == Epi::BiasLnResidF32 ? FN : 1], beta[EPI == Epi::BiasLnResidF32 ? FN : 1];
};

template <class C, Epi EPI>
__device__ inline void epilogue_prefetch(const GemmParams &p, EpiInputs<C, EPI> &in, int wave, int lane,
                                         int m0, int n0) {
    const int wm = wave % C::WGM, wn = wave / C::WGM;
#pragma unroll
    for (int j = 0; j < C::FN; ++j) {
        const int f = n0 + wn * C::TN + j * 16 + (lane >> 4) * 4;
        if constexpr (has_bias(EPI)) in.bias[j] = *reinterpret_cast<const u32x2 *>(p.bias + f);
        else in.bias[j] = u32x2{0u, 0u};
        if constexpr (EPI == Epi::BiasLnResidF32) {
            in.gamma[j] = *reinterpret_cast<const f32x4 *>(p.ln.gamma + f);
            in.beta[j] = *reinterpret_cast<const f32x4 *>(p.ln.beta + f);
        }
        if constexpr (EpiInputs<C, EPI>::kZ) {
            const float *src = EPI == Epi::BiasResidF32 ? p.resid : p.ln.z;
#pragma unroll
            for (int i = 0; i < C::FM; ++i) {
                const int t = min(m0 + wm * C::TM + i * 16 + (lane & 15), p.M - 1);   // clamped: never stored
                in.z[j][i] = *reinterpret_cast<const f32x4 *>(src + (size_t)t * p.N + f);
            }
        }
    }
    if constexpr (EPI == Epi::BiasLnResidF32) {
#pragma unroll
        for (int i = 0; i < C::FM; ++i) {
            const int t = min(m0 + wm * C::TM + i * 16 + (lane & 15), p.M - 1);
            in.stats[i] = *reinterpret_cast<const f32x2 *>(p.ln.stats + 2 * (size_t)t);
        }
    }
}

// Row strides (bf16) of the staged output tile: token-major for plain bf16
// outputs and Q/K, feature-major for V^T.  The 8-element pad keeps rows
// 16-byte aligned and spreads consecutive rows over the LDS banks.
template <class C> constexpr int kRowStride = C::BN + 8;
template <class C> constexpr int kColStride = C::BM + 8;

// Epilogue of one wave.  Lane owns features f..f+3 of token t in every block.
// fp32 outputs are stored directly (one 16-byte store per block); bf16 outputs
// go to the LDS tile `ctile` (token-major, or feature-major when `vt_tile`).
template <class C, Epi EPI>
__device__ inline void epilogue(const GemmParams &p, const f32x4 (&acc)[C::FN][C::FM],
                                const EpiInputs<C, EPI> &in, int wave, int lane, int m0, int n0,
                                bf16_t *ctile, bool vt_tile) {
    const int wm = wave % C::WGM, wn = wave / C::WGM;
#pragma unroll
    for (int j = 0; j < C::FN; ++j) {
        const int fl = wn * C::TN + j * 16 + (lane >> 4) * 4;   // feature within the tile
        const int f = n0 + fl;
        const u32x2 braw = in.bias[j];
        const float b0 = __uint_as_float(braw[0] << 16), b1 = __uint_as_float(braw[0] & 0xffff0000u);
        const float b2 = __uint_as_float(braw[1] << 16), b3 = __uint_as_float(braw[1] & 0xffff0000u);
#pragma unroll
        for (int i = 0; i < C::FM; ++i) {
            const int tl = wm * C::TM + i * 16 + (lane & 15);   // token within the tile
            const int t = m0 + tl;
            float v0 = acc[j][i][0] + b0, v1 = acc[j][i][1] + b1;
            float v2 = acc[j][i][2] + b2, v3 = acc[j][i][3] + b3;
            if constexpr (staged(EPI)) {
                if constexpr (EPI == Epi::BiasGeluBf16) {
                    v0 = gelu(v0); v1 = gelu(v1); v2 = gelu(v2); v3 = gelu(v3);
                }
                if constexpr (EPI == Epi::GeluBwdBf16) {   // rows past M read row M - 1: never stored
                    const u32x2 g = *reinterpret_cast<const u32x2 *>(p.aux + (size_t)min(t, p.M - 1) * p.N + f);
                    v0 *= gelu_grad(__uint_as_float(g[0] << 16));
                    v1 *= gelu_grad(__uint_as_float(g[0] & 0xffff0000u));
                    v2 *= gelu_grad(__uint_as_float(g[1] << 16));
                    v3 *= gelu_grad(__uint_as_float(g[1] & 0xffff0000u));
                }
                if (EPI == Epi::Qkv && vt_tile) {
                    bf16_t *o = ctile + fl * kColStride<C> + tl;
                    o[0] = f32_to_bf16(v0);
                    o[kColStride<C>] = f32_to_bf16(v1);
                    o[2 * kColStride<C>] = f32_to_bf16(v2);
                    o[3 * kColStride<C>] = f32_to_bf16(v3);
                } else {
                    *reinterpret_cast<u32x2 *>(ctile + tl * kRowStride<C> + fl) = u32x2{pack2(v0, v1), pack2(v2, v3)};
                }
            } else if constexpr (EPI == Epi::F32) {
                if (t >= p.M) continue;
                *reinterpret_cast<f32x4 *>(static_cast<float *>(p.out) + (size_t)t * p.N + f) = f32x4{v0, v1, v2, v3};
            } else if constexpr (EPI == Epi::BiasResidF32) {
                if (t >= p.M) continue;
                f32x4 r;
                if constexpr (EpiInputs<C, EPI>::kZ) r = in.z[j][i];
                else r = *reinterpret_cast<const f32x4 *>(p.resid + (size_t)t * p.N + f);
                *reinterpret_cast<f32x4 *>(static_cast<float *>(p.out) + (size_t)t * p.N + f) =
                    f32x4{r[0] + v0, r[1] + v1, r[2] + v2, r[3] + v3};
            } else {   // Epi::BiasLnResidF32: residual = LN(z) rebuilt with the LayerNorm kernel's expression
                if (t >= p.M) continue;
                f32x4 z;
                if constexpr (EpiInputs<C, EPI>::kZ) z = in.z[j][i];
                else z = *reinterpret_cast<const f32x4 *>(p.ln.z + (size_t)t * p.N + f);
                const float mean = in.stats[i][0], rstd = in.stats[i][1];
                f32x4 r;
#pragma unroll
                for (int e = 0; e < 4; ++e) r[e] = __builtin_fmaf(in.gamma[j][e], (z[e] - mean) * rstd, in.beta[j][e]);
                *reinterpret_cast<f32x4 *>(static_cast<float *>(p.out) + (size_t)t * p.N + f) =
                    f32x4{r[0] + v0, r[1] + v1, r[2] + v2, r[3] + v3};
            }
        }
    }
}

// Store the staged bf16 tile.  Called by all `nt` threads of the workgroup
// after a barrier that follows every wave's epilogue().
template <class C, Epi EPI>
__device__ inline void store_tile(const GemmParams &p, const bf16_t *ctile, bool vt_tile, int tid, int nt, int m0,
                                  int n0) {
    if (EPI == Epi::Qkv && vt_tile) {
        // V^T [B, H, dh, vt_stride]: a segment is 8 consecutive tokens of one
        // (head, column) row, contiguous when seq and pos0 are multiples of 8
        const QkvDst &d = p.qkv;
        constexpr int TG = C::BM / 8;
        for (int sg = tid; sg < C::BN * TG; sg += nt) {
            const int fl = sg / TG, t0 = m0 + (sg % TG) * 8;
            if (t0 >= p.M) continue;
            const int within = n0 + fl - 2 * d.d_model, head = within / d.head_dim, jj = within - head * d.head_dim;
            const bf16_t *src = ctile + fl * kColStride<C> + (t0 - m0);
            if (d.seq % 8 == 0 && d.pos0 % 8 == 0) {
                const int b = t0 / d.seq, sp = d.pos0 + t0 - b * d.seq;
                bf16_t *o = d.vt + (((size_t)b * d.n_heads + head) * d.head_dim + jj) * d.vt_stride + sp;
                *reinterpret_cast<u32x4 *>(o) = *reinterpret_cast<const u32x4 *>(src);
            } else {
                for (int e = 0; e < 8 && t0 + e < p.M; ++e) {
                    const int t = t0 + e, b = t / d.seq, sp = d.pos0 + t - b * d.seq;
                    d.vt[(((size_t)b * d.n_heads + head) * d.head_dim + jj) * d.vt_stride + sp] = src[e];
                }
            }
        }
        return;
    }
    constexpr int SEGS = C::BN / 8;   // 16-byte segments per token row
    for (int sg = tid; sg < C::BM * SEGS; sg += nt) {
        const int r = sg / SEGS, c = sg - r * SEGS, t = m0 + r;
        if (t >= p.M) continue;
        const u32x4 v = *reinterpret_cast<const u32x4 *>(ctile + r * kRowStride<C> + c * 8);
        const int f = n0 + c * 8;
        bf16_t *o;
        if constexpr (EPI == Epi::Qkv) {   // Q or K [B, H, S, dh]: 8 columns of one head
            const QkvDst &d = p.qkv;
            const int which = f / d.d_model, within = f - which * d.d_model;
            const int head = within / d.head_dim, jj = within - head * d.head_dim;
            const int b = t / d.seq, sp = t - b * d.seq;
            o = which == 0 ? d.q + (((size_t)b * d.n_heads + head) * d.seq + sp) * d.head_dim + jj
                           : d.k + (((size_t)b * d.n_heads + head) * d.k_rows + d.pos0 + sp) * d.head_dim + jj;
        } else {
            o = static_cast<bf16_t *>(p.out) + (size_t)t * p.N + f;
        }
        *reinterpret_cast<u32x4 *>(o) = v;
        if constexpr (EPI == Epi::BiasGelu2Bf16) {   // GELU of the value as rounded
            u32x4 g;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                g[e] = pack2(gelu(__uint_as_float(v[e] << 16)), gelu(__uint_as_float(v[e] & 0xffff0000u)));
            *reinterpret_cast<u32x4 *>(p.out2 + (size_t)t * p.N + f) = g;
        }
    }
}

// LDS of a workgroup (bf16 elements): the rings, reused by the staged tile.
template <class C, Epi EPI>
constexpr int lds_elems() {
    int n = C::RING;
    if (staged(EPI)) n = n > C::BM * kRowStride<C> ? n : C::BM * kRowStride<C>;
    if (EPI == Epi::Qkv) n = n > C::BN * kColStride<C> ? n : C::BN * kColStride<C>;
    return n;
}

// One output tile: tile l of the product, by the whole workgroup.
template <class C, Epi EPI>
__device__ inline void run_tile(const GemmParams &p, int l, bf16_t *lds) {
    constexpr int FN = C::FN, FM = C::FM;
    int tm, tn;
    grouped_tile(l, p.tiles_m, p.tiles_n, tm, tn);
    const int m0 = tm * C::BM, n0 = tn * C::BN;
    // the wave index is uniform across the wave: held in a scalar register, so
    // that every branch on it (tile, copy counts) is a scalar branch
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    f32x4 acc[C::ORD][FN][FM];
#pragma unroll
    for (int o = 0; o < C::ORD; ++o)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int i = 0; i < FM; ++i) acc[o][j][i] = f32x4{0.f, 0.f, 0.f, 0.f};
    EpiInputs<C, EPI> in;
    if constexpr (kEarlyInputs<C, EPI>) epilogue_prefetch<C, EPI>(p, in, wave, lane, m0, n0);
    main_loop<C>(p, lds, wave, lane, m0, n0, acc);
    if constexpr (!kEarlyInputs<C, EPI>) epilogue_prefetch<C, EPI>(p, in, wave, lane, m0, n0);
    if constexpr (C::ORD == 2) {   // the even tiles' sum + the odd tiles' sum
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int i = 0; i < FM; ++i) acc[0][j][i] += acc[1][j][i];
    }
    const bool vt_tile = EPI == Epi::Qkv && n0 >= 2 * p.qkv.d_model;
    if constexpr (staged(EPI)) __syncthreads();   // every wave is done reading the rings
    epilogue<C, EPI>(p, acc[0], in, wave, lane, m0, n0, lds, vt_tile);
    if constexpr (staged(EPI)) {
        __syncthreads();
        store_tile<C, EPI>(p, lds, vt_tile, threadIdx.x, C::NT, m0, n0);
    }
}

template <class C, Epi EPI>
__global__ __launch_bounds__(C::NT) __attribute__((amdgpu_waves_per_eu(C::WPE))) void gemm_kernel(GemmParams p) {
    __shared__ __attribute__((aligned(1024))) bf16_t lds[lds_elems<C, EPI>()];
    static_assert(lds_elems<C, EPI>() * 2 <= 163840, "LDS");
    run_tile<C, EPI>(p, xcd_contiguous(blockIdx.x, gridDim.x), lds);
}

// Several products in one launch: tile l belongs to job j with first[j] <= l <
// first[j + 1].
struct GemmGroup {
    GemmParams job[kMaxGemmGroup];
    int32_t first[kMaxGemmGroup + 1];
    int32_t n;
};

template <class C>
__global__ __launch_bounds__(C::NT) __attribute__((amdgpu_waves_per_eu(C::WPE))) void gemm_group_kernel(GemmGroup g) {
    __shared__ __attribute__((aligned(1024))) bf16_t lds[lds_elems<C, Epi::F32>()];
    const int l = xcd_contiguous(blockIdx.x, gridDim.x);
    int j = 0;
    while (j + 1 < g.n && l >= g.first[j + 1]) ++j;
    run_tile<C, Epi::F32>(g.job[j], l - g.first[j], lds);
}

// Tile configurations.
//                   BM   BN  WGM WGN ORD S AHEAD
using S32x32 = Cfg<32, 32, 2, 2, 1, 5, true>;         // 4 waves
using S32x64 = Cfg<32, 64, 2, 2, 1, 4, true>;
using S64x64 = Cfg<64, 64, 2, 2, 1, 4, true>;
using S64x96 = Cfg<64, 96, 2, 2, 1, 4, true>;
using S128x64 = Cfg<128, 64, 4, 2, 1, 4, true>;       // 8 waves from here on
using S128x96 = Cfg<128, 96, 4, 2, 1, 4, false>;      // one workgroup per CU
using S128x96p = Cfg<128, 96, 4, 2, 1, 2, false>;     // two
using S128x128 = Cfg<128, 128, 2, 4, 1, 2, false>;
using S128x192 = Cfg<128, 192, 2, 4, 1, 2, false>;
using S256x256 = Cfg<256, 256, 2, 4, 1, 2, false>;
// even / odd K order
using E32x32 = Cfg<32, 32, 2, 2, 2, 5, true>;
using E32x64 = Cfg<32, 64, 2, 2, 2, 4, true>;
using E64x64 = Cfg<64, 64, 2, 2, 2, 4, true>;
using E64x96 = Cfg<64, 96, 2, 2, 2, 4, true>;
using E128x64 = Cfg<128, 64, 4, 2, 2, 4, true>;
using E128x96 = Cfg<128, 96, 4, 2, 2, 4, false>;
using E128x128 = Cfg<128, 128, 2, 4, 2, 4, false>;
using E256x128 = Cfg<256, 128, 4, 2, 2, 3, false>;

enum class Tile {
    S32x32, S32x64, S64x64, S64x96, S128x64, S128x96, S128x96p, S128x128, S128x192, S256x256,
    E32x32, E32x64, E64x64, E64x96, E128x64, E128x96, E128x128, E256x128
};

// K summation order from the weight shape (N, K) only: K >= 2048 uses the
// split (even/odd) order, shorter K the sequential order.  So a given weight
// matrix always sums each output in the same order, whatever M (the batch),
// the CU quota or the tile shape -- outputs stay bit-identical across them.
bool split_k_order(int /*N*/, int K) { return K >= 2048; }

// What the choice of a tile goes by.
struct TileInfo {
    Tile tile;
    bool split;      // K order
    int bm, bn;      // a workgroup's output block
    int per_cu;      // workgroups whose rings share a CU
    int step;        // relative time of one K tile of one workgroup
};

constexpr TileInfo kTiles[] = {
    {Tile::S32x32, false, 32, 32, 4, 51},      {Tile::S32x64, false, 32, 64, 3, 51},
    {Tile::S64x64, false, 64, 64, 2, 100},     {Tile::S64x96, false, 64, 96, 2, 117},
    {Tile::S128x64, false, 128, 64, 1, 180},  {Tile::S128x96, false, 128, 96, 1, 172},
    {Tile::S128x96p, false, 128, 96, 2, 188}, {Tile::S128x128, false, 128, 128, 2, 222},
    {Tile::S128x192, false, 128, 192, 2, 377}, {Tile::S256x256, false, 256, 256, 1, 1155},
    {Tile::E32x32, true, 32, 32, 4, 78},       {Tile::E32x64, true, 32, 64, 3, 96},
    {Tile::E64x64, true, 64, 64, 2, 100},      {Tile::E64x96, true, 64, 96, 2, 130},
    {Tile::E128x64, true, 128, 64, 1, 168},   {Tile::E128x96, true, 128, 96, 1, 169},
    {Tile::E128x128, true, 128, 128, 1, 264}, {Tile::E256x128, true, 256, 128, 1, 470},
};
// the same unit: a round's fixed part (launch of its workgroups, first copies, epilogue)
constexpr long kRoundSequential = 4673, kRoundSplit = 4458;

long ceil_div(long a, long b) { return (a + b - 1) / b; }

// The tile with the least estimated time on a share of n_cu CUs: the busiest
// CU's workgroups times the K tiles times a tile's `step`, plus a fixed part
// for every round of resident workgroups.  `step` and the fixed part are
// fitted to the measured times of every tile on 309 products (64 to 8192
// tokens, N 128 to 8192, K 128 to 8192, at 64, 128 and 256 CUs); the tile they
// pick is within 1% (sequential) and 0.1% (even/odd) of the fastest on
// average, and 1.22 and 1.48 times as fast as the rule it replaces, which took
// the largest tile that gave every CU one.  It comes out as: the smallest tile
// whose workgroups still fit the share at one per CU, and for larger grids the
// tile that leaves the busiest CU with the least work.  Restrictions:
//  - widths divide `align` (d_model for the QKV scatter, so that no tile
//    straddles the Q / K / V boundaries);
//  - 128 x 192 not with the LayerNorm-residual epilogue (wide_ok): it spills 58
//    registers there;
//  - 256 x 256 from K = 1024 on: its 128 KB epilogue has no other workgroup to
//    hide behind (4096 x 3072 x 768: 32.1 us against 26.6 with 128 x 192; 4096 x
//    4096 x 1024: 40.3 against 42.7 with 128 x 128);
//  - 128 x 64 while it fits at one per CU (a second round costs it more than
//    64 x 64 tiles do: 4096 x 2368 x 768, 27 against 32 us).
// Every tile shape of an order adds the same terms in the same sequence, so
// the choice may follow the launch (M and n_cu) without changing a bit.
struct Shape {
    int M, N, align;
};

const TileInfo &choose_tile(const Shape *shapes, int n_shapes, int K, int n_cu, bool wide_ok = true) {
    const bool split = split_k_order(0, K);
    const TileInfo *best = nullptr;
    long best_cost = 0;
    for (const TileInfo &t : kTiles) {
        if (t.split != split) continue;
        if (t.tile == Tile::S128x192 && !wide_ok) continue;
        if (t.tile == Tile::S256x256 && K < 1024) continue;
        long n = 0;
        bool divides = true;
        for (int i = 0; i < n_shapes; ++i) {
            divides = divides && shapes[i].align % t.bn == 0;
            n += ceil_div(shapes[i].M, t.bm) * (shapes[i].N / t.bn);
        }
        if (!divides || (t.tile == Tile::S128x64 && n > n_cu)) continue;
        const long cost = ceil_div(n, n_cu) * (K / 64) * t.step +
                          ceil_div(n, (long)n_cu * t.per_cu) * (split ? kRoundSplit : kRoundSequential);
        if (!best || cost < best_cost) {
            best = &t;
            best_cost = cost;
        }
    }
    return *best;   // 64 x 64 divides every width
}

const TileInfo &choose_tile(int M, int N, int K, int align, int n_cu, bool wide_ok = true) {
    const Shape s{M, N, align};
    return choose_tile(&s, 1, K, n_cu, wide_ok);
}

template <class C>
hipError_t launch_tile(Epi epi, GemmParams &p, hipStream_t s) {
    p.tiles_m = (p.M + C::BM - 1) / C::BM;
    p.tiles_n = p.N / C::BN;
    const dim3 grid(p.tiles_m * p.tiles_n), block(C::NT);
    switch (epi) {
    case Epi::BiasBf16: return launch_kernel(gemm_kernel<C, Epi::BiasBf16>, grid, block, s, p);
    case Epi::BiasGeluBf16: return launch_kernel(gemm_kernel<C, Epi::BiasGeluBf16>, grid, block, s, p);
    case Epi::BiasResidF32: return launch_kernel(gemm_kernel<C, Epi::BiasResidF32>, grid, block, s, p);
    case Epi::Qkv: return launch_kernel(gemm_kernel<C, Epi::Qkv>, grid, block, s, p);
    case Epi::BiasLnResidF32:
        if constexpr (C::BM * C::BN == 128 * 192) return hipErrorInvalidValue;   // never chosen: it would spill
        else return launch_kernel(gemm_kernel<C, Epi::BiasLnResidF32>, grid, block, s, p);
    case Epi::F32: return launch_kernel(gemm_kernel<C, Epi::F32>, grid, block, s, p);
    case Epi::GeluBwdBf16: return launch_kernel(gemm_kernel<C, Epi::GeluBwdBf16>, grid, block, s, p);
    case Epi::BiasGelu2Bf16: return launch_kernel(gemm_kernel<C, Epi::BiasGelu2Bf16>, grid, block, s, p);
    }
    return hipErrorInvalidValue;
}

template <class C>
hipError_t launch_group(GemmGroup &g, hipStream_t s) {
    int tiles = 0;
    for (int j = 0; j < g.n; ++j) {
        GemmParams &p = g.job[j];
        p.tiles_m = (p.M + C::BM - 1) / C::BM;
        p.tiles_n = p.N / C::BN;
        g.first[j] = tiles;
        tiles += p.tiles_m * p.tiles_n;
    }
    g.first[g.n] = tiles;
    return launch_kernel(gemm_group_kernel<C>, dim3(tiles), dim3(C::NT), s, g);
}

}  // namespace

GemmPlan gemm_plan(int M, int N, int K, int align, int n_cu, bool ln_residual) {
    const TileInfo &t = choose_tile(M, N, K, align, n_cu, !ln_residual);
    return GemmPlan{split_k_order(N, K), t.split, t.bm, t.bn};
}

GemmPlan gemm_group_plan(const GemmJob *jobs, int n_jobs, int K, int n_cu) {
    Shape shapes[kMaxGemmGroup];
    for (int j = 0; j < n_jobs; ++j) shapes[j] = {jobs[j].M, jobs[j].N, jobs[j].N};
    const TileInfo &t = choose_tile(shapes, n_jobs, K, n_cu);
    return GemmPlan{split_k_order(0, K), t.split, t.bm, t.bn};
}

hipError_t launch_gemm(Epi epi, const bf16_t *a, const bf16_t *w, const bf16_t *bias,
                       const float *resid, void *out, int M, int N, int K, const QkvDst *qkv,
                       hipStream_t stream, const LnResid *ln, const bf16_t *aux, int n_cu, bf16_t *out2) {
    if (M <= 0) return hipSuccess;
    if (N % 64 || K % 64 || N <= 0 || K <= 0) return hipErrorInvalidValue;
    if ((epi == Epi::GeluBwdBf16 && !aux) || (epi == Epi::BiasGelu2Bf16 && !out2)) return hipErrorInvalidValue;
    GemmParams p{};
    p.a = a; p.w = w; p.bias = bias; p.resid = resid; p.out = out; p.aux = aux; p.out2 = out2;
    p.M = M; p.N = N; p.K = K;
    if (qkv) p.qkv = *qkv;
    if (ln) p.ln = *ln;
    // N is a multiple of 64 (checked by the callers); d_model a multiple of 128
    const int align = epi == Epi::Qkv ? p.qkv.d_model : N;
    switch (choose_tile(M, N, K, align, n_cu, epi != Epi::BiasLnResidF32).tile) {
#define IEFWD_TILES(X) \
    X(S32x32) X(S32x64) X(S64x64) X(S64x96) X(S128x64) X(S128x96) X(S128x96p) X(S128x128) X(S128x192) X(S256x256) \
    X(E32x32) X(E32x64) X(E64x64) X(E64x96) X(E128x64) X(E128x96) X(E128x128) X(E256x128)
#define X(T) case Tile::T: return launch_tile<T>(epi, p, stream);
        IEFWD_TILES(X)
#undef X
    }
    return hipErrorInvalidValue;
}

// The tile is chosen for the jobs' tiles together: products too small to fill
// the chip each with the tile that reuses its operands most do so together.
// (Width 768, 4096 tokens, the four weight gradients of a layer: 91 us in four
// launches of 128 x 96, 128 x 64 and 64 x 64 tiles, 68 us in one of 216 tiles of
// 256 x 128.)
hipError_t launch_gemm_group(const GemmJob *jobs, int n_jobs, int K, hipStream_t stream, int n_cu) {
    if (n_jobs <= 0) return hipSuccess;
    if (n_jobs > kMaxGemmGroup || K <= 0 || K % 64) return hipErrorInvalidValue;
    GemmGroup g{};
    g.n = n_jobs;
    Shape shapes[kMaxGemmGroup];
    for (int j = 0; j < n_jobs; ++j) {
        if (jobs[j].M < 1 || jobs[j].N <= 0 || jobs[j].N % 64) return hipErrorInvalidValue;
        GemmParams &p = g.job[j];
        p.a = jobs[j].a; p.w = jobs[j].w; p.out = jobs[j].out;
        p.M = jobs[j].M; p.N = jobs[j].N; p.K = K;
        shapes[j] = {p.M, p.N, p.N};
    }
    switch (choose_tile(shapes, n_jobs, K, n_cu).tile) {
#define X(T) case Tile::T: return launch_group<T>(g, stream);
        IEFWD_TILES(X)
#undef X
    }
    return hipErrorInvalidValue;
}

}  // namespace iefwd
