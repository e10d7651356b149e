// conv_union.hip -- sparse convolution on a neighbour table of a 3x3x3 map or, by
// output, of a 2x2x2 one (Sec. 3.2 / 3.3) with register accumulators: the
// neighbour-table kernel described in conv.hip.
#include <algorithm>
#include <type_traits>

#include "conv_common.hpp"

namespace spv {

// f(integral_constant<int, i>) for i = B .. E-1, each i a compile-time constant
template <int B, int E, class F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (B < E) {
        f(std::integral_constant<int, B>{});
        static_for<B + 1, E>(f);
    }
}

// ---------------------------------------------------------------------------
// neighbour-table kernel (3x3x3 maps, and the 2x2x2 stride-2 maps by output)
// ---------------------------------------------------------------------------
// A workgroup of NW waves computes R = 16 RB NW output rows times NBT blocks of 16 output channels
// (NB / NBT workgroups share the rows).  A wave owns RB blocks of 16 rows; the accumulators of a
// block are D = W^T G^T fragments.  The weight fragments of a pair of channel blocks (2v, 2v + 1) are
// permuted on their way into LDS (row r16 of block 2v + u holds channel 32 v + 8 (r16 / 4) + 4 u + r16 % 4),
// so that lane (r16, g) ends with output channels 32 v + 8 g .. + 7 of row r16: a residual load and a store
// of 16 bytes each, 64 bytes of a row side by side.  An odd NBT keeps the order of the packing (channels
// nb*16 + 4g .. 4g+3, 8 bytes).
//
// What bounds it: the waits in a workgroup's chain of 27 offsets.  On one 88k-voxel sweep, 96 -> 96 (47 us), the
// matrix cores are busy 25% of the time and LDS 16%, 63% of the CUs' cycles have a wave, and a wave waits 43%
// of its life (2% for LDS); below ~50k rows the chain of one workgroup is the kernel's time, however few
// workgroups there are.  So:
// * the workgroup's rows of the neighbour table go to LDS first, in one coalesced copy: read offset by
//   offset from memory each 4-byte index cost a lane its own cache line, as much as a gathered row;
// * the weights of a group of PH offsets are copied global->LDS while the group before is multiplied
//   (two buffers, one barrier per group, instead of a stop for the copy at each group); where each of two
//   buffers would hold one offset (48 fragments an offset and more, 32 in 384-row tiles), one buffer of two
//   or three is filled between two barriers instead: 256 -> 96 on 29,789 rows 48 us, 55 with a barrier at
//   every offset;
// * the tile is chosen per call (launch_union_c below): 256 to 512 rows where the rows fill the chip, down to
//   64 rows and a slice of the output channels where they do not, and 192 rows in between at 24 to 32 fragments
//   an offset (128 -> 128 on 35,193 rows: 44 us, 49 in 256-row tiles).  256 -> 256 on 3,161 rows:
//   107 -> 31 us, 128 -> 128 on 7,697: 37 -> 17 us, 96 -> 96 on 52,357: 46 -> 33 us, on 88,119: 52 ->
//   49 us, on 356,951: 171 -> 160 us.
//
// A step is one offset's (k) slab of KS 32-channel chunks; the rows of RA steps are in flight while
// one is multiplied (a lane whose row has no neighbour reads from outside the buffer, which costs
// nothing and returns zeros, so every step issues the same loads and the compiler's waits stay exact);
// blocks with no neighbour at k skip their products.  The copies the compiler does not see are
// issued after the group's first rows have arrived and waited for by count before the barrier: the
// loads issued after them are the rows of the steps ahead.
//
// On a table of 8 each offset's products are summed by themselves and then added to the rows that have the
// offset, as the pairs' kernel sums them (the same bits): chained through one accumulator as on 27 offsets,
// the outputs differed with the kernel that a workspace's size selects, and the rows that an infinite weight
// reached had to be summed again after the loop, which held up to 160 more registers than the loop itself.

// Shape of a workgroup's tile; valid when it fits in LDS and is not another class's tile.
template <int K3, int KCH, int NB, int CLS>
struct UnionTile {
    // output-channel blocks of a workgroup: all of them (at most 8) in the classes for many rows, at
    // most half of them in the classes that spread few rows over the chip
    static constexpr int NBL = NB > 8 ? 8 : NB;
    static constexpr int NBS = NB == 2 ? 2 : NB == 4 ? 2 : NB == 6 ? (KCH == 8 ? 3 : 2) : 4;
    static constexpr int NBT = CLS < 3 || CLS == 5 ? NBL : NBS;
    static constexpr int FR = KCH * NBT;  // 1 KB weight fragments per offset
    static constexpr int RB = CLS == 0 ? 2 : 1;
    static constexpr int NW0 = FR > 32 || (K3 == 8 && FR >= 24) ? 8 : NB <= 4 && KCH == 1 ? 16 : 12;
    static constexpr int NW = CLS == 0 ? NW0 : CLS == 1 ? (FR > 32 ? 12 : 16) : CLS == 4 ? 4 : CLS == 5 ? 12 : 8;
    static constexpr int R = NW * RB * 16;
    // (a table of 8 sums an offset's products apart, so its steps are whole offsets)
    static constexpr int KS = KCH < 4 || K3 == 8 ? KCH : RB == 2 ? (NW >= 12 ? 2 : 4) : KCH;
    static constexpr int SH = KCH / KS;  // steps per offset
    static constexpr int RA = SH == 4 ? 3 : K3 == 27 && CLS == 0 && KCH == 3 && NBT <= 6 ? 2 : 1;
    static constexpr int IX = R * K3 + 32;  // table entries (and the few the last steps read past them)
    // offsets per weight group: as many as fit, in whole turns of the row ring where more than one fits
    // (two workgroups per CU in the classes of one block of rows and 8 waves or fewer, if they fit)
    static constexpr int UNIT = RA == 2 ? 3 : SH % (RA + 1) == 0 ? 1 : 2;
    static constexpr int fit(int kb) {
        const int n = (kb * 1024 - IX * 4) / (2 * FR * 1024);
        const int most = K3 == 8 ? 4 : 14;
        return RA == 1 && n == 1 ? 1 : n > most ? most / UNIT * UNIT : n / UNIT * UNIT;
    }
    static constexpr int PH2 = CLS >= 2 && fit(80) >= 2 ? fit(80) : fit(160);
    // one buffer where two would hold no more than an offset each
    static constexpr int PH1 = (160 * 1024 - IX * 4) / (FR * 1024);
    static constexpr bool TWO = K3 == 8 || PH2 >= 2 || PH1 < 2;
    static constexpr int PH = TWO ? PH2 : PH1;
    static constexpr int LDS = IX * 4 + (TWO ? 2 : 1) * PH * FR * 1024;
    static constexpr bool valid = PH >= 1 && !(CLS == 1 && FR > 48) && !(CLS == 3 && NBS == NBL) &&
                                  !(CLS == 5 && !(K3 == 27 && FR >= 24 && FR <= 32));
    // channel blocks whose products of an offset are summed at a time, on a table of 8
    static constexpr int NQ = NBT % 4 == 0 ? 4 : NBT % 3 == 0 ? 3 : 2;
    // Workgroups that share a CU, by LDS and, on a table of 8, whose small tiles leave room for up to four, by
    // the registers of a wave: accumulators, the offset's sums, two steps of rows and about 14 more per block
    // (as many as the compiler takes, or up to 20 more).  The launch bounds hold it to them.  On 27 offsets two
    // fit by LDS only in tiles of at most 8 waves, at under 128 registers each.
    static constexpr int lds_cu = 160 * 1024 / LDS;
    static constexpr int regs = (4 * RB * (NBT + NQ) + 8 * RB * KCH + 14 * RB + 7) / 8 * 8;
    static constexpr int reg_cu = 512 / regs * 4 / NW;
    static constexpr int fit_cu = K3 == 27 ? (lds_cu < 2 ? lds_cu : 2) : lds_cu < reg_cu ? lds_cu : reg_cu;
    static constexpr int per_cu = fit_cu < 1 ? 1 : fit_cu > 4 ? 4 : fit_cu;
    static constexpr bool SPREAD = K3 == 27 && RB == 2;      // spreads few live rows
    static constexpr int SLOTS = 256 / (NB / NBT);           // row tiles that give every CU one workgroup
    static constexpr int waves_eu = K3 == 8 ? per_cu * NW / 4 : 1;
};

template <int DT, int K3, int KCH, int NB, int CLS>
__global__ __launch_bounds__((64 * UnionTile<K3, KCH, NB, CLS>::NW), (UnionTile<K3, KCH, NB, CLS>::waves_eu)) void k_conv_union(
    const int32_t* __restrict__ nbr, const int64_t* __restrict__ m_out_dev, int64_t m_cap,
    const uint16_t* __restrict__ in, int64_t in_rows, const uint4* __restrict__ wpack,
    const float* __restrict__ scale, const float* __restrict__ shift, int relu, const uint16_t* __restrict__ res,
    uint16_t* __restrict__ out) {
    using T = UnionTile<K3, KCH, NB, CLS>;
    constexpr int NBT = T::NBT, FR = T::FR, RB = T::RB, NW = T::NW, R = T::R, KS = T::KS, SH = T::SH;
    constexpr int RA = T::RA, PH = T::PH, GS = PH * SH, NG = (K3 + PH - 1) / PH;  // steps per group, groups
    constexpr int Cout = NB * 16, CT = NB / NBT;
    constexpr int U = GS % (RA + 1) == 0 ? 1 : RA + 1;  // groups per turn of the loop: whole turns of the row ring
    static_assert(GS >= RA, "the rows of the steps ahead are issued after the group's weight copies");
    __shared__ __align__(16) uint4 wl[T::TWO ? 2 : 1][PH * FR * 64];
    __shared__ __align__(16) int32_t ix[T::IX];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r16 = lane & 15, g = lane >> 4;

    // Workgroups are dispatched round-robin over the 8 XCDs (workgroup b to XCD
    // b % 8).  The row tiles that exist (from the live row count, not the
    // capacity the grid was sized for) are split into 8 consecutive ranges, one
    // per XCD, so neighbouring tiles (and the channel slices of one tile) share
    // an L2 and every XCD gets work.
    const int64_t m = clamp_rows(m_out_dev, m_cap);
    const int64_t x = blockIdx.x % 8, seq = blockIdx.x / 8 / CT;
    const int ct = (int)(blockIdx.x / 8 % CT);
    // A tile of two blocks a wave was picked for a capacity.  Where the live rows, at one block for each wave, do
    // not fill the chip once, they are spread: tiles of as few blocks as that takes, a wave each (the other
    // waves and the second blocks find no rows).  128 -> 128 in buffers of 120,000 rows, 6,000 of them live:
    // 35 us, 60 in whole tiles, 41 in the one-block tiles that served it before.
    int RL = R;
    bool spread = false;
    if (T::SPREAD && m_out_dev) {
        const int64_t nb = (m + 16 * T::SLOTS - 1) / (16 * T::SLOTS);
        spread = nb <= NW;
        if (spread) RL = nb > 1 ? 16 * (int)nb : 16;
    }
    // rows of block b of a wave: wave * wave_rows + b * block_rows ..
    const int wave_rows = spread ? 16 : 16 * RB, block_rows = spread ? 16 * NW : 16;
    const int64_t ga = spread ? (uint32_t)(m + RL - 1) / (uint32_t)RL : (m + R - 1) / R, xq = ga / 8, xr = ga % 8;
    if (seq >= xq + (x < xr ? 1 : 0)) return;  // the whole workgroup
    const int64_t row0 = (x * xq + (x < xr ? x : xr) + seq) * RL;
    const int nrows = (int)(m - row0 < RL ? m - row0 : RL);

    // weights of offsets k0 .. k0 + nk - 1 (this workgroup's channel blocks) -> buffer buf
    constexpr bool PAIR = NBT % 2 == 0;
    const i32x4* wsrc = (const i32x4*)wpack + ct * NBT * 64;
    // byte offset, from the first fragment of the pair, of what this lane copies into fragment 2v + u
    uint32_t wlane[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int c = 8 * (r16 >> 2) + 4 * u + (r16 & 3);
        wlane[u] = PAIR ? (uint32_t)((c >> 4) * 64 + (lane & 48) + (c & 15)) * 16u : (uint32_t)lane * 16u;
    }
    auto load_w = [&](int k0, int nk, int buf) __attribute__((always_inline)) {
        // (a wave copies both fragments of a pair where nothing overlaps the copy: they share cache lines)
        constexpr int UF = PAIR && !T::TWO ? 2 : 1;
        for (int f0 = UF * wave; f0 < nk * FR; f0 += UF * NW) {
#pragma unroll
            for (int f = f0; f < f0 + UF; ++f) {
                const int kk = f / NBT, nb = f - kk * NBT;  // kk = (k - k0) * KCH + kc
                const int from = PAIR ? nb & ~1 : nb;
                lds_dma_x4((uint64_t)(wsrc + ((int64_t)(k0 * KCH + kk) * NB + from) * 64), wlane[nb & 1],
                           __builtin_amdgcn_readfirstlane(lds_addr(&wl[buf][f * 64])));
            }
        }
    };
    load_w(0, K3 < PH ? K3 : PH, 0);
    {
        const int32_t* src = nbr + row0 * K3;
        if (nrows == R && ((uintptr_t)src & 15) == 0) {
            for (int e = tid; e < R * K3 / 4; e += 64 * NW) ((i32x4*)ix)[e] = ((const i32x4*)src)[e];
        } else {
            for (int e = tid; e < R * K3; e += 64 * NW) ix[e] = e < nrows * K3 ? src[e] : 0;
        }
    }
    vm_wait<0>();
    __syncthreads();

    constexpr uint32_t row_bytes = KCH * 64u;
    const __amdgpu_buffer_rsrc_t in_rs = make_rsrc(in, (uint32_t)(in_rows * (int64_t)row_bytes));
    const uint32_t in_rows32 = (uint32_t)in_rows;
    const int32_t* ixw = ix + (wave * wave_rows + r16) * K3;
    const int bstep = block_rows * K3;  // table entries between a wave's blocks
    // offsets that this lane's row of each block has, and those of the block (union over its 16 rows,
    // wave-uniform)
    uint32_t rmask[RB], umask[RB];
#pragma unroll
    for (int b = 0; b < RB; ++b) {
        uint32_t bits = 0;
#pragma unroll
        for (int k = 0; k < K3; k += 4)
            if (k + g < K3) bits |= (ixw[b * bstep + k + g] > 0 ? 1u : 0u) << (k + g);
        bits |= __shfl_xor(bits, 16, 64);
        bits |= __shfl_xor(bits, 32, 64);
        rmask[b] = bits;
#pragma unroll
        for (int d = 1; d < 16; d <<= 1) bits |= __shfl_xor(bits, d, 64);
        umask[b] = __builtin_amdgcn_readfirstlane(bits);
    }
    // gathered rows of (offset k, slab h): 16-byte chunks g + 4 (h KS + kc) of row i (stored as i + 1)
    auto load_rows = [&](int k, int h, i32x4 (&dst)[RB][KS]) __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < RB; ++b) {
            const uint32_t i = (uint32_t)(ixw[b * bstep + k] - 1);
            const uint32_t base = i < in_rows32 && k < K3 ? i * row_bytes + (uint32_t)g * 16u : kOutOfRange;
#pragma unroll
            for (int kc = 0; kc < KS; ++kc)
                dst[b][kc] = __builtin_amdgcn_raw_buffer_load_b128(in_rs, base + (uint32_t)(h * KS + kc) * 64u, 0, 0);
        }
    };

    f32x4 acc[RB][NBT];
#pragma unroll
    for (int b = 0; b < RB; ++b)
#pragma unroll
        for (int nb = 0; nb < NBT; ++nb) acc[b][nb] = f32x4{0.f, 0.f, 0.f, 0.f};

    i32x4 rs[RA + 1][RB][KS];  // gathered rows of step j of a group in slot j % (RA + 1)
#pragma unroll
    for (int j = 0; j < RA; ++j) load_rows(j / SH, j % SH, rs[j]);
    // group gi of offsets, whose first step's rows are in slot R0
    auto group = [&](int gi, auto r0) __attribute__((always_inline)) {
        constexpr int R0 = decltype(r0)::value;
        const int k0 = gi * PH;
        const i32x4* wbuf = (const i32x4*)wl[T::TWO ? gi & 1 : 0] + lane;
        if (T::TWO && gi + 1 < NG) {
            // the first step's rows are here (the empty statements make the compiler wait for them), so the
            // copies of the next weights delay no row that this step needs
#pragma unroll
            for (int b = 0; b < RB; ++b)
#pragma unroll
                for (int kc = 0; kc < KS; ++kc) asm volatile("" : "+v"(rs[R0][b][kc]));
            load_w(k0 + PH, K3 - k0 - PH < PH ? K3 - k0 - PH : PH, (gi + 1) & 1);
        }
        static_for<0, GS>([&](auto jj) __attribute__((always_inline)) {
            constexpr int j = decltype(jj)::value, kp = j / SH, h = j % SH;
            const int k = k0 + kp;
            load_rows(k0 + (j + RA) / SH, (j + RA) % SH, rs[(R0 + j + RA) % (RA + 1)]);
            if (K3 % PH == 0 || k < K3) {
                uint32_t present = 0;
#pragma unroll
                for (int b = 0; b < RB; ++b) present |= ((umask[b] >> k) & 1u) << b;
                if (present) {
                    const i32x4* wk = wbuf + (kp * FR + h * KS * NBT) * 64;
                    if constexpr (K3 == 8) {
                        // an offset's products are summed by themselves and added to the rows that have it: half
                        // of a block's rows lack an offset that the block has, and an infinite weight must not
                        // reach them (the sums are those of the pairs' kernel, bit for bit)
                        constexpr int NQ = T::NQ;
#pragma unroll
                        for (int q = 0; q < NBT; q += NQ) {
                            f32x4 d[RB][NQ];
#pragma unroll
                            for (int b = 0; b < RB; ++b)
#pragma unroll
                                for (int nb = 0; nb < NQ; ++nb) d[b][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                            for (int kc = 0; kc < KS; ++kc)
#pragma unroll
                                for (int nb = 0; nb < NQ; ++nb) {
                                    const i32x4 wf = wk[(kc * NBT + q + nb) * 64];
#pragma unroll
                                    for (int b = 0; b < RB; ++b)
                                        d[b][nb] = mfma16x16x32<DT>(
                                            __builtin_bit_cast(uint4, wf),
                                            __builtin_bit_cast(uint4, rs[(R0 + j) % (RA + 1)][b][kc]), d[b][nb]);
                                }
#pragma unroll
                            for (int b = 0; b < RB; ++b)
                                if ((rmask[b] >> k) & 1u) {
#pragma unroll
                                    for (int nb = 0; nb < NQ; ++nb) acc[b][q + nb] += d[b][nb];
                                }
                        }
                    } else {
#pragma unroll
                        for (int kc = 0; kc < KS; ++kc) {
                            i32x4 wf[NBT];
#pragma unroll
                            for (int nb = 0; nb < NBT; ++nb) wf[nb] = wk[(kc * NBT + nb) * 64];
#pragma unroll
                            for (int b = 0; b < RB; ++b) {
                                if (RB == 1 || ((present >> b) & 1u)) {
#pragma unroll
                                    for (int nb = 0; nb < NBT; ++nb)
                                        acc[b][nb] = mfma16x16x32<DT>(
                                            __builtin_bit_cast(uint4, wf[nb]),
                                            __builtin_bit_cast(uint4, rs[(R0 + j) % (RA + 1)][b][kc]), acc[b][nb]);
                                }
                            }
                        }
                    }
                }
            }
        });
        if (gi + 1 < NG) {
            // of what the wave has issued since the group's weight copies, only the rows of the RA steps
            // ahead may be outstanding: the copies are complete
            if constexpr (T::TWO) vm_wait<RA * RB * KS>();
            lds_wait();
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            if constexpr (!T::TWO) {
                const int k1 = k0 + PH;
                load_w(k1, K3 - k1 < PH ? K3 - k1 : PH, 0);
                vm_wait<0>();
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
            }
        }
    };
#pragma clang loop unroll(disable)
    for (int gt = 0; gt < NG; gt += U)
        static_for<0, U>([&](auto u) __attribute__((always_inline)) {
            constexpr int uu = decltype(u)::value;
            if (U == 1 || gt + uu < NG) group(gt + uu, std::integral_constant<int, uu * GS % (RA + 1)>{});
        });

    // epilogue: act(scale * acc + shift + res), EC channels per store
    constexpr int EC = PAIR ? 8 : 4, NE = NBT * 4 / EC;  // channels of a piece, pieces
    const int c0 = ct * NBT * 16 + EC * g;
#pragma unroll
    for (int v = 0; v < NE; ++v) {
        float sc[EC], sh[EC];
#pragma unroll
        for (int e = 0; e < EC; ++e) {
            sc[e] = scale ? scale[c0 + v * 4 * EC + e] : 1.f;
            sh[e] = shift ? shift[c0 + v * 4 * EC + e] : 0.f;
        }
#pragma unroll
        for (int b = 0; b < RB; ++b) {
            const int rr = wave * wave_rows + b * block_rows + r16;
            if (rr >= nrows) continue;
            const int64_t at = (row0 + rr) * Cout + c0 + v * 4 * EC;
            uint32_t u[EC / 2], w[EC / 2];
#pragma unroll
            for (int e = 0; e < EC / 2; ++e) u[e] = 0u;
            if (res) {  // the residual input, same layout as the output
                if constexpr (PAIR) {
                    const uint4 r = *(const uint4*)(res + at);
                    u[0] = r.x;
                    u[1] = r.y;
                    u[2] = r.z;
                    u[3] = r.w;
                } else {
                    const uint2 r = *(const uint2*)(res + at);
                    u[0] = r.x;
                    u[1] = r.y;
                }
            }
#pragma unroll
            for (int e = 0; e < EC; e += 2) {
                float y[2];
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const int i = e + q;
                    const float rv = from16<DT>(q ? u[e / 2] >> 16 : u[e / 2] & 0xFFFF);
                    y[q] = acc[b][v * (EC / 4) + i / 4][i % 4] * sc[i] + sh[i] + rv;
                    if (relu) y[q] = fmaxf(y[q], 0.f);
                }
                w[e / 2] = (uint32_t)to16<DT>(y[0]) | ((uint32_t)to16<DT>(y[1]) << 16);
            }
            if constexpr (PAIR) *(uint4*)(out + at) = make_uint4(w[0], w[1], w[2], w[3]);
            else *(uint2*)(out + at) = make_uint2(w[0], w[1]);
        }
    }
}

// instantiated for C_in, C_out in {32, 64, 96, 128, 256} (the widths of the
// blocks and networks built here, square layers and the channel changes
// between stages); other shapes use the tile kernel
bool union_supported(int K3, int Cin, int Cout, int dt) {
    if ((K3 != 27 && K3 != 8) || dt == SPV_F32) return false;
    const auto width_ok = [](int c) { return c == 32 || c == 64 || c == 96 || c == 128 || c == 256; };
    return width_ok(Cin) && width_ok(Cout);
}

// Which tile: whole rounds of workgroups over the 256 CUs times what one round takes.  A round of
// workgroups of B blocks of 16 rows and FR weight fragments per offset measured about
// 4 + 0.4 FR + B (0.1 + 0.28 KCH + 0.018 FR) us on 27 offsets (96 -> 96: 21 us at 8 blocks, 31 at 16, 43 at 24;
// 32 -> 32: 8 at 8, 15 at 32; 256 -> 256 in slices of 128 channels: 87 at 16, 61 at 8, of 64: 39 at 8) and
// 1.5 + 0.13 FR + B (0.08 + 0.04 KCH + 0.016 FR) us on 8, beside the plan; so a small tile wins while it still
// fits one round and a large one when rounds are many.  The model only ranks.  On 8 offsets, every tile of the
// 25 width pairs timed at 19 sets of 354 to 188,994 coarse rows: the tile ranked first takes 1.1% longer than
// the fastest on average (27 offsets' constants, scaled, and two workgroups wherever the LDS has room: 1.9%);
// 64 -> 128 with its plan takes 26 us on 35,193 rows in 384-row tiles, 22 in 256 or 128 rows and 32 on the
// pairs, and on 69,827 rows 31, 37, 34 and 51.
// A device-side count (the block's voxels, of a capacity of all its points) is taken as 3/4 of the
// capacity, about what a LiDAR sweep has.
template <int K3, int KCH, int NB, int CLS>
static double union_cost(int64_t rows) {
    using T = UnionTile<K3, KCH, NB, CLS>;
    if constexpr (!T::valid) {
        return 1e30;
    } else {
        const int64_t wgs = (rows + T::R - 1) / T::R * (NB / T::NBT), slots = 256 * T::per_cu;
        // workgroups on one CU share its pipes: only the fixed parts overlap
        const double fixed = K3 == 8 ? 1.5 + 0.13 * T::FR : 4.0 + 0.4 * T::FR;
        const double work = T::R / 16 * (K3 == 8 ? 0.08 + 0.04 * KCH + 0.016 * T::FR : 0.1 + 0.28 * KCH + 0.018 * T::FR);
        const int64_t rest = wgs % slots, deep = (rest + 255) / 256;  // of the last round, workgroups on the fullest CU
        return (double)(wgs / slots) * (fixed + work * T::per_cu) + (rest == 0 ? 0.0 : fixed + work * (double)deep);
    }
}

template <int DT, int K3, int KCH, int NB, int CLS>
static void launch_union_tile(hipStream_t s, const ConvPlan& p, const void* in, int64_t in_rows, const void* wpack,
                              const float* scale, const float* shift, int relu, void* out) {
    using T = UnionTile<K3, KCH, NB, CLS>;
    if constexpr (T::valid) {
        // a multiple of 8 workgroups: the kernel spreads the live tiles over the 8 XCDs
        int64_t tiles = (p.m_cap + T::R - 1) / T::R;
        if (T::SPREAD && p.m_out_dev)  // few live rows are spread over up to SLOTS tiles
            tiles = std::max(tiles, std::min<int64_t>(T::SLOTS, (p.m_cap + 15) / 16));
        const unsigned grid = (unsigned)((tiles + 7) / 8 * 8 * (NB / T::NBT));
        k_conv_union<DT, K3, KCH, NB, CLS><<<grid, 64 * T::NW, 0, s>>>(p.nbr, p.m_out_dev, p.m_cap, (const uint16_t*)in,
                                                                  in_rows, (const uint4*)wpack, scale, shift, relu,
                                                                  (const uint16_t*)p.res, (uint16_t*)out);
    }
}

template <int DT, int K3, int KCH, int NB>
static void launch_union_c(hipStream_t s, const ConvPlan& p, const void* in, int64_t in_rows, const void* wpack,
                           const float* scale, const float* shift, int relu, void* out) {
    const int64_t rows = p.m_out_dev ? p.m_cap - p.m_cap / 4 : p.m_cap;
    const double cost[6] = {union_cost<K3, KCH, NB, 0>(rows), union_cost<K3, KCH, NB, 1>(rows),
                            union_cost<K3, KCH, NB, 2>(rows), union_cost<K3, KCH, NB, 3>(rows),
                            union_cost<K3, KCH, NB, 4>(rows), union_cost<K3, KCH, NB, 5>(rows)};
    int c = 0;
    for (int i = 1; i < 6; ++i)
        if (cost[i] < cost[c]) c = i;
    switch (c) {
        case 0: launch_union_tile<DT, K3, KCH, NB, 0>(s, p, in, in_rows, wpack, scale, shift, relu, out); break;
        case 1: launch_union_tile<DT, K3, KCH, NB, 1>(s, p, in, in_rows, wpack, scale, shift, relu, out); break;
        case 2: launch_union_tile<DT, K3, KCH, NB, 2>(s, p, in, in_rows, wpack, scale, shift, relu, out); break;
        case 3: launch_union_tile<DT, K3, KCH, NB, 3>(s, p, in, in_rows, wpack, scale, shift, relu, out); break;
        case 4: launch_union_tile<DT, K3, KCH, NB, 4>(s, p, in, in_rows, wpack, scale, shift, relu, out); break;
        case 5: launch_union_tile<DT, K3, KCH, NB, 5>(s, p, in, in_rows, wpack, scale, shift, relu, out); break;
    }
}

template <int DT, int K3, int KCH>
static void launch_union_cin(hipStream_t s, const ConvPlan& p, const void* in, int Cout, int64_t in_rows,
                             const void* wpack, const float* scale, const float* shift, int relu, void* out) {
    switch (Cout) {
        case 32: launch_union_c<DT, K3, KCH, 2>(s, p, in, in_rows, wpack, scale, shift, relu, out); break;
        case 64: launch_union_c<DT, K3, KCH, 4>(s, p, in, in_rows, wpack, scale, shift, relu, out); break;
        case 96: launch_union_c<DT, K3, KCH, 6>(s, p, in, in_rows, wpack, scale, shift, relu, out); break;
        case 128: launch_union_c<DT, K3, KCH, 8>(s, p, in, in_rows, wpack, scale, shift, relu, out); break;
        case 256: launch_union_c<DT, K3, KCH, 16>(s, p, in, in_rows, wpack, scale, shift, relu, out); break;
    }
}

template <int DT, int K3>
static void launch_union(hipStream_t s, const ConvPlan& p, const void* in, int Cin, int Cout, int64_t in_rows,
                         const void* wpack, const float* scale, const float* shift, int relu, void* out) {
    switch (Cin) {
        case 32: launch_union_cin<DT, K3, 1>(s, p, in, Cout, in_rows, wpack, scale, shift, relu, out); break;
        case 64: launch_union_cin<DT, K3, 2>(s, p, in, Cout, in_rows, wpack, scale, shift, relu, out); break;
        case 96: launch_union_cin<DT, K3, 3>(s, p, in, Cout, in_rows, wpack, scale, shift, relu, out); break;
        case 128: launch_union_cin<DT, K3, 4>(s, p, in, Cout, in_rows, wpack, scale, shift, relu, out); break;
        case 256: launch_union_cin<DT, K3, 8>(s, p, in, Cout, in_rows, wpack, scale, shift, relu, out); break;
    }
}

void launch_conv_union(hipStream_t s, const ConvPlan& p, const void* in, int Cin, int64_t in_rows, int Cout,
                       const void* wpack, const float* scale, const float* shift, int relu, void* out, int dt) {
    if (p.K3 == 8) {
        if (dt == SPV_BF16) launch_union<SPV_BF16, 8>(s, p, in, Cin, Cout, in_rows, wpack, scale, shift, relu, out);
        else launch_union<SPV_F16, 8>(s, p, in, Cin, Cout, in_rows, wpack, scale, shift, relu, out);
    } else {
        if (dt == SPV_BF16) launch_union<SPV_BF16, 27>(s, p, in, Cin, Cout, in_rows, wpack, scale, shift, relu, out);
        else launch_union<SPV_F16, 27>(s, p, in, Cin, Cout, in_rows, wpack, scale, shift, relu, out);
    }
}

}  // namespace spv
