// conv_up.hip -- the transposed k=2 s=2 sparse convolution (the decoder's
// upsampling, Sec. 3.2) as an output-scattered GEMM.
//
// On a stride-2 map every fine voxel has exactly one parent: fine voxel i with
// parent j at offset k receives in[j] @ W[k] and nothing else.  So instead of
// gathering, per output, the inputs of its pairs, the kernel walks the coarse
// rows.  A workgroup holds R of them in LDS; its wave k lists the rows that
// have a child at offset k, and multiplies them 16 at a time by W[k], which it
// holds in registers (NBS blocks of 16 output channels at a time), writing each
// product row, finished by act(scale * . + shift + res), straight to its
// child's row.  Every output row is written once, by one lane group; nothing
// accumulates across pairs and the waves meet only once, after the rows are in.
// children[j][k] = i + 1 (0 = none) is the stride-2 map's neighbour table.
//
// What bounds it: the scattered output rows and, before, what led up to them.
// A coarse voxel of a sweep has about two of its eight children, so blocks of
// consecutive rows multiplied at every offset did four products for each one
// used; every 128 rows waited for a copy of all weights into LDS; and a lane
// wrote four channels (8 bytes) at a time.  The lists leave only the last block
// of an offset partly empty, the weights of a workgroup are read once per R
// rows, and the fragments are permuted so that a lane holds eight consecutive
// channels: 16-byte stores, 64 bytes of a row side by side.
#include "conv_common.hpp"

namespace spv {

constexpr int kUpK = 8;

// output-channel blocks whose weights a wave holds at once: an even number that divides NB, at most 24
// fragments (96 registers)
template <int KCH, int NB>
struct UpTile {
    static constexpr int NBS = KCH == 8 ? 2 : KCH == 4 && NB != 6 ? (NB < 4 ? NB : 4) : NB > 8 ? 8 : NB;
    static constexpr int RS = KCH * 64 + 16;  // bytes of a row in LDS, so that consecutive rows lie on other banks
};

template <int DT, int KCH, int NB, int R>
__global__ __launch_bounds__(64 * kUpK) void k_conv_up(
    const int32_t* __restrict__ children, const int64_t* __restrict__ m_dev, int64_t m_cap,
    const uint16_t* __restrict__ in, const uint4* __restrict__ wpack, const float* __restrict__ scale,
    const float* __restrict__ shift, int relu, const uint16_t* __restrict__ res, uint16_t* __restrict__ out,
    int64_t out_rows) {
    constexpr int NBS = UpTile<KCH, NB>::NBS, RS = UpTile<KCH, NB>::RS, Cout = NB * 16, PC = KCH * 4;
    __shared__ __align__(16) unsigned char xs[R * RS];
    __shared__ int32_t lfine[kUpK][R];   // fine row of the list's entries
    __shared__ uint16_t lrow[kUpK][R];   // their coarse row in the tile
    const int tid = threadIdx.x, lane = tid & 63;
    const int k = __builtin_amdgcn_readfirstlane(tid >> 6);  // the wave's offset
    const int r16 = lane & 15, g = lane >> 4;
    const int64_t m = clamp_rows(m_dev, m_cap);
    const int64_t row0 = (int64_t)blockIdx.x * R;
    if (row0 >= m) return;  // the whole workgroup
    const int rows = (int)(m - row0 < R ? m - row0 : R);

    for (int e = tid; e < rows * PC; e += 64 * kUpK)
        *(i32x4*)(xs + (e / PC) * RS + (e % PC) * 16) = ((const i32x4*)(in + row0 * KCH * 32))[e];
    int cnt = 0;
    for (int b = 0; b < R; b += 64) {
        const int r = b + lane;
        const int32_t c = r < rows ? children[(row0 + r) * kUpK + k] : 0;
        const bool have = c > 0 && (int64_t)c <= out_rows;
        const uint64_t mask = __ballot(have);
        if (have) {
            const int at = cnt + __builtin_popcountll(mask & ((1ull << lane) - 1ull));
            lfine[k][at] = c - 1;
            lrow[k][at] = (uint16_t)r;
        }
        cnt += __builtin_popcountll(mask);
    }
    __syncthreads();
    if (cnt == 0) return;

    // A fragment of a pair of channel blocks (2v, 2v + 1): row r16 of block 2v + u holds output channel
    // 32 v + 8 (r16 / 4) + 4 u + r16 % 4, so that after the product lane (r16, g) holds channels
    // 32 v + 8 g .. + 7 of list entry r16
    const i32x4* wk = (const i32x4*)wpack + (int64_t)k * KCH * NB * 64;
    for (int nb0 = blockIdx.y * NBS; nb0 < NB; nb0 += gridDim.y * NBS) {
        i32x4 wf[KCH][NBS];
#pragma unroll
        for (int kc = 0; kc < KCH; ++kc)
#pragma unroll
            for (int nb = 0; nb < NBS; ++nb) {
                const int c = 8 * (r16 >> 2) + 4 * (nb & 1) + (r16 & 3);  // within the pair's 32 channels
                wf[kc][nb] = wk[(int64_t)(kc * NB + nb0 + (nb & ~1) + (c >> 4)) * 64 + (g * 16 + (c & 15))];
            }
        for (int e0 = 0; e0 < cnt; e0 += 16) {
            const int e = e0 + r16;
            const bool live = e < cnt;
            const int lr = live ? lrow[k][e] : lrow[k][e0];
            const int64_t orow = live ? lfine[k][e] : 0;
            f32x4 acc[NBS];
#pragma unroll
            for (int nb = 0; nb < NBS; ++nb) acc[nb] = f32x4{0.f, 0.f, 0.f, 0.f};
            const unsigned char* xr = xs + lr * RS + g * 16;
#pragma unroll
            for (int kc = 0; kc < KCH; ++kc) {
                const i32x4 xv = *(const i32x4*)(xr + kc * 64);
#pragma unroll
                for (int nb = 0; nb < NBS; ++nb)
                    acc[nb] = mfma16x16x32<DT>(__builtin_bit_cast(uint4, wf[kc][nb]), __builtin_bit_cast(uint4, xv),
                                               acc[nb]);
            }
            if (!live) continue;
#pragma unroll
            for (int v = 0; v < NBS / 2; ++v) {
                const int c = nb0 * 16 + v * 32 + 8 * g;
                float rv[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
                if (res) {
                    const uint4 u = *(const uint4*)(res + orow * Cout + c);
                    const uint32_t uu[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        rv[2 * j] = from16<DT>(uu[j] & 0xFFFF);
                        rv[2 * j + 1] = from16<DT>(uu[j] >> 16);
                    }
                }
                uint32_t w[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    uint32_t h[2];
#pragma unroll
                    for (int q = 0; q < 2; ++q) {
                        const int i = 2 * j + q;
                        const float sc = scale ? scale[c + i] : 1.f, sh = shift ? shift[c + i] : 0.f;
                        float y = acc[2 * v + i / 4][i % 4] * sc + sh + rv[i];
                        if (relu) y = fmaxf(y, 0.f);
                        h[q] = to16<DT>(y);
                    }
                    w[j] = h[0] | (h[1] << 16);
                }
                *(uint4*)(out + orow * Cout + c) = make_uint4(w[0], w[1], w[2], w[3]);
            }
        }
    }
}

bool up_supported(int Cin, int Cout, int dt) {
    if (dt == SPV_F32) return false;
    const auto width_ok = [](int c) { return c == 32 || c == 64 || c == 96 || c == 128 || c == 256; };
    return width_ok(Cin) && width_ok(Cout);
}

// 128 coarse rows per workgroup, 64 where 128 would leave CUs without one; the passes over the output
// channels are spread over workgroups (each with the rows in its own LDS) only while there are fewer than
// two per CU
template <int DT, int KCH, int NB>
static void launch_up_c(hipStream_t s, const UpArgs& a, const void* wpack) {
    constexpr int passes = NB / UpTile<KCH, NB>::NBS;
    const bool small = a.m_cap <= 128 * 256;
    const int64_t tiles = (a.m_cap + (small ? 63 : 127)) / (small ? 64 : 128);
    unsigned gy = 1;
    while (gy < (unsigned)passes && tiles * gy < 512) gy *= 2;
    const dim3 grid((unsigned)tiles, gy);
    if (small)
        k_conv_up<DT, KCH, NB, 64><<<grid, 64 * kUpK, 0, s>>>(
            a.children, a.m_dev, a.m_cap, (const uint16_t*)a.in, (const uint4*)wpack, a.scale, a.shift, a.relu,
            (const uint16_t*)a.res, (uint16_t*)a.out, a.out_rows);
    else
        k_conv_up<DT, KCH, NB, 128><<<grid, 64 * kUpK, 0, s>>>(
            a.children, a.m_dev, a.m_cap, (const uint16_t*)a.in, (const uint4*)wpack, a.scale, a.shift, a.relu,
            (const uint16_t*)a.res, (uint16_t*)a.out, a.out_rows);
}

template <int DT, int KCH>
static void launch_up_cin(hipStream_t s, const UpArgs& a, const void* wpack) {
    switch (a.Cout) {
        case 32: launch_up_c<DT, KCH, 2>(s, a, wpack); break;
        case 64: launch_up_c<DT, KCH, 4>(s, a, wpack); break;
        case 96: launch_up_c<DT, KCH, 6>(s, a, wpack); break;
        case 128: launch_up_c<DT, KCH, 8>(s, a, wpack); break;
        case 256: launch_up_c<DT, KCH, 16>(s, a, wpack); break;
    }
}

template <int DT>
static void launch_up_dt(hipStream_t s, const UpArgs& a, const void* wpack) {
    switch (a.Cin) {
        case 32: launch_up_cin<DT, 1>(s, a, wpack); break;
        case 64: launch_up_cin<DT, 2>(s, a, wpack); break;
        case 96: launch_up_cin<DT, 3>(s, a, wpack); break;
        case 128: launch_up_cin<DT, 4>(s, a, wpack); break;
        case 256: launch_up_cin<DT, 8>(s, a, wpack); break;
    }
}

void launch_conv_up(hipStream_t s, const UpArgs& a, const void* wpack) {
    if (a.m_cap <= 0) return;
    if (a.dt == SPV_BF16) launch_up_dt<SPV_BF16>(s, a, wpack);
    else launch_up_dt<SPV_F16>(s, a, wpack);
}

}  // namespace spv
