// patch_conv.hip -- MFMA convolution from an input patch held in LDS (gfx950).
//
// A block computes BM output channels x BN consecutive output pixels.  Per chunk of CK input
// channels it stages the input patch under its pixels once -- every input pixel any filter tap of
// the tile touches, channel-contiguous -- and then applies all R*S taps from LDS: a tap is a
// constant offset into the patch, so the im2col matrix never passes through memory, the caches or
// the LDS write port R*S times as it does in the gather GEMM.  Filters come packed in MFMA operand
// order (one coalesced 1 KiB load per operand and wave, straight into registers), so nothing but
// the patch needs barriers.
//
// Operands are bf16 in the matrix unit.  NP = 1: bf16 tensors.  NP = 3: fp32 tensors, every value
// times 2^24 written as the sum of three bf16 values x = x0 + x1 + x2 (round to nearest, then the
// remainder twice) and x*w summed from the six products of weight 2^-16 and more:
// x2 w0 + x0 w2 + x1 w1 + x1 w0 + x0 w1 + x0 w0.  24 significand bits = 3 x 8, so the split is
// exact; the factor keeps the last bit of every fp32 value, subnormal ones included (2^-149),
// above bf16's smallest normal number (without it x2 loses bits below |x| = 2^-110; it costs 0.6 %
// of a call, 45.4 -> 45.6 us on N32 64->64 56x56 3x3).  The sums are multiplied by 2^-48 at the
// end.  Where the scaled values overflow (an operand from 2^104, a sum from 2^80) or an operand is
// not finite, the fp32 matrix instruction computes the tile instead.  The three dropped products
// are together at most 2^-24 (1 + 2^-10) of |x||w| (|x1| <= 2^-8 |x|, |x2| <= 2^-17 |x|), about the
// rounding of one fp32 addition; the matrix unit does 16x the bf16 work of its fp32 work per
// cycle, i.e. 2.7x through six products.  Relative error against float64 (2-norm) on N32 64->64
// 56x56 3x3: 3.6e-7, against 4.2e-7 of the fp32 matrix instruction's sums.
//
// Measured on MI355X, us per call (filter packing included), gather GEMM -> this kernel: N32 64->64
// 56x56 3x3 fp32 72 -> 49 (103 -> 150 TFLOP/s), N32 256->512 56x56 1x1 stride 2 fp32 78 -> 68, N32
// 256->256 56x56 3x3 bf16 168 -> 132 (705 -> 897 TFLOP/s); bf16 layers whose channels the gather had
// to fetch one by one up to 11x (N16 1744->16 203x64 1x1 stride 2 NHWC 462 -> 42).  Counters of the
// first and of N32 256->256: matrix unit busy 0.54 of the kernel's cycles, other vector instructions
// 0.18 and 0.11 (at 4 cycles each), LDS bank conflicts 0.14; waves spend 0.25 of their time waiting for
// memory, LDS or barriers and 0.55 for a free issue slot, the matrix unit's above all.  x is fetched
// 2.8 times in the first (73 MB for 26): tiles that share rows run on different XCDs.
#include <type_traits>

#include "device_common.h"

namespace cv {

namespace {

// Factor of an fp32 operand before its split, and of the sum of products after it (see above).
constexpr float kSplitScale = 0x1p24f, kSplitUnscale = 0x1p-48f;

// Three bf16 planes of two fp32 values, packed (low half = lo).
struct Split2 {
    uint32_t p[3];
};
__device__ __forceinline__ uint32_t pk_bf16(float lo, float hi) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{lo, hi}, bf16x2));
}
__device__ __forceinline__ Split2 split2(float lo, float hi) {
    Split2 s;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        s.p[i] = pk_bf16(lo, hi);
        lo -= __builtin_bit_cast(float, s.p[i] << 16);
        hi -= __builtin_bit_cast(float, s.p[i] & 0xffff0000u);
    }
    return s;
}

// NP planes of 8 consecutive reduction values: planes[p] = 16 bytes of bf16.
template <int NP>
__device__ __forceinline__ void planes_of(const float (&f)[8], u32x4 (&planes)[NP]) {
    constexpr float scale = NP == 3 ? kSplitScale : 1.0f;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const Split2 s = split2(f[2 * q] * scale, f[2 * q + 1] * scale);
#pragma unroll
        for (int p = 0; p < NP; ++p) planes[p][q] = s.p[p];
    }
}

// Filters [G*Kg][Cg][RS] -> MFMA A operands: fragment ((g, mt, chunk, tap, ks), plane) is 1 KiB,
// lane l holds row mt*32 + l%32, channels chunk*CK + ks*16 + 8*(l/32) .. +7 (zero outside M and
// Cg).  One wave per fragment of the row tile (g, mt) = blockIdx.y: its 8 loads leave together, so
// the launch takes one memory round trip; filters are small next to x and the lines that the
// taps share hit in L2.
template <int NP, int KS, typename T>
__global__ __launch_bounds__(256) void pack_filters_kernel(const T* __restrict__ w, uint32_t w_bytes, void* wp,
                                                           uint32_t wp_bytes, int nfrag, int mtiles, int Kg, int Cg,
                                                           int RS, FastDiv fd_rs, FastDiv fd_mt) {
    const int f = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + (threadIdx.x >> 6)));  // of this row tile
    if (f >= nfrag) return;
    const int lane = threadIdx.x & 63;
    const __amdgpu_buffer_rsrc_t rw = make_rsrc(w, w_bytes);
    const __amdgpu_buffer_rsrc_t rp = make_rsrc(wp, wp_bytes);
    const int g = (int)fdiv(blockIdx.y, fd_mt), mt = (int)blockIdx.y - g * mtiles;
    const int st = f / KS, ks = f % KS;
    const int chunk = (int)fdiv((uint32_t)st, fd_rs), tap = st - chunk * RS;
    const int m = mt * 32 + (lane & 31);
    const int c0 = (chunk * KS + ks) * 16 + (lane >> 5) * 8;
    const uint32_t e0 = (uint32_t)(((g * Kg + m) * Cg + c0) * RS + tap);
    float v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const bool ok = (m < Kg) & (c0 + j < Cg);
        const uint32_t e = e0 + (uint32_t)(j * RS);
        if constexpr (sizeof(T) == 4) v[j] = ld_f32(rw, ok ? e * 4u : OOB_OFF);
        else v[j] = __builtin_bit_cast(float, (uint32_t)ld_u16(rw, ok ? e * 2u : OOB_OFF) << 16);
    }
    u32x4 pl[NP];
    planes_of<NP>(v, pl);
    const int at = (int)blockIdx.y * nfrag + f;
#pragma unroll
    for (int p = 0; p < NP; ++p)
        __builtin_amdgcn_raw_buffer_store_b128(pl[p], rp, (uint32_t)lane * 16u, (at * NP + p) * 1024, 0);
}

// Input element offset of output pixel (n, ho, wo) at tap (r, s) and channel 0 of the group, or
// false outside the image.
__device__ __forceinline__ bool tap_at(const PatchArgs& A, int n, int ho, int wo, int r, int s, int64_t* e) {
    const int hi = ho * A.sh - A.ph + r * A.dh, wi = wo * A.sw - A.pw + s * A.dw;
    *e = (int64_t)n * A.x_ns + (int64_t)hi * A.x_hs + (int64_t)wi * A.x_ws;
    return ((unsigned)hi < (unsigned)A.H) & ((unsigned)wi < (unsigned)A.W);
}

// RSC: 1 = 1x1 filters (patch slot = output pixel), 9 = 3x3 filters, 0 = any filter.  LD: how the
// patch is loaded.  PATCH_LD_ONE: element by element (any strides); PATCH_LD_VEC: 8 channels of a
// pixel are contiguous and 16-byte aligned (NHWC); PATCH_LD_PAIR: bf16, two neighbouring pixels of
// a channel are one aligned 4-byte word (NCHW; the 2-byte loads fetch half of what the address
// unit can pass per instruction).  UN: staging units (one patch pixel, or pair, x 8 channels) per
// thread.  NSET: register sets of filter operands (one 16-channel step each).
//
// Memory operations of a wave complete in order, so a wait for filter operands also waits for
// every staging load issued before them.  With RSC > 0 a chunk is straight-line code: the next
// chunk's staging loads leave at its start, the operands of the steps behind them are NSET - 1
// steps ahead, and every wait counts exactly what it needs.  (One loop over taps with the staging
// under a condition made the compiler wait for the staging loads at once, every chunk.)
template <int NP, int KS, int TM, int TN, int WM, int WN, int RSC, int LD, int UN, int NSET, int MINW>
__global__ __launch_bounds__(WM * WN * 64, MINW) void patch_conv_kernel(PatchArgs A) {
    constexpr int NT = WM * WN * 64;
    constexpr int BM = WM * TM * 32, BN = WN * TN * 32;
    constexpr int CK = 16 * KS, C8 = CK / 8;
    constexpr int ES = NP == 3 ? 4 : 2;
    constexpr bool PT = RSC == 1;
    constexpr bool VEC = LD == PATCH_LD_VEC, PAIR = LD == PATCH_LD_PAIR;
    static_assert(!PAIR || NP == 1, "pairs of bf16 pixels");
    constexpr int PX = PAIR ? 2 : 1;  // pixels per unit
    // bytes per patch pixel: the planes and 16 more, so that 8 neighbouring pixels fall on
    // different LDS banks (28, 20 or 52 words)
    constexpr int PITCH = NP * CK * 2 + 16;
    extern __shared__ __attribute__((aligned(16))) char lds[];

    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int lcol = lane & 31, lrow = lane >> 5;
    const int ksplit = A.ksplit > 1 ? A.ksplit : 1;
    const int gi = blockIdx.z / ksplit, sp = blockIdx.z - gi * ksplit;
    // the blocks past the whole tiles are the pieces of the tail split: chunks [cb, ce) of a tile
    const int ndp = (int)gridDim.x - A.tail_tiles * A.tail_pieces;
    const int tail = (int)blockIdx.x - ndp;
    int tile, tail_tile = -1, piece = 0, cb, ce;
    if (tail < 0) {
        tile = xcd_remap(blockIdx.x, ndp);
        cb = sp * A.split_ch;
        ce = min(cb + A.split_ch, A.nch);
    } else {
        tail_tile = tail / A.tail_pieces;
        piece = tail - tail_tile * A.tail_pieces;
        tile = ndp + tail_tile;
        cb = piece * A.tail_ch;
        ce = min(cb + A.tail_ch, A.nch);
    }
    const int tq0 = tile / A.grid_m;
    const int tile_m = tile - tq0 * A.grid_m;
    const int colb = tq0 / A.tiles_q;
    const int q0 = (tq0 - colb * A.tiles_q) * BN;
    const int qend = A.rows * A.TW;
    const int wo0 = colb * A.TW;  // first output column of this column block

    const __amdgpu_buffer_rsrc_t rx = make_rsrc(A.x, A.x_bytes);
    const __amdgpu_buffer_rsrc_t rp = make_rsrc(A.wp, A.wp_bytes);

    // first virtual input row of the patch: images follow each other with HV rows each
    int v0 = 0, vend = 0;
    if constexpr (!PT) {
        const int r0 = (int)fdiv((uint32_t)q0, A.fd_tw);
        const int r1 = (int)fdiv((uint32_t)(min(q0 + BN, qend) - 1), A.fd_tw);
        const int n0 = (int)fdiv((uint32_t)r0, A.fd_ho), n1 = (int)fdiv((uint32_t)r1, A.fd_ho);
        v0 = n0 * A.HV + (r0 - n0 * A.Ho) * A.lsh;
        vend = n1 * A.HV + (r1 - n1 * A.Ho) * A.lsh + (A.R - 1) * A.dh + 1;
    }

    // staging units of this thread: byte offset in x (channel 0 of the chunk at cb = 0) and in LDS
    uint32_t goff[UN], laddr[UN];
    const int nunits = A.nslots / PX * C8;
    const int64_t xg = (int64_t)gi * A.Cg * A.x_cs;
    // pairs start on even input columns: the patch then begins one column early where its first
    // column is odd
    const int cshift = PAIR && !PT ? (wo0 * A.lsw - A.pw) & 1 : 0;
#pragma unroll
    for (int u = 0; u < UN; ++u) {
        const int id = u * NT + t;
        int slot, c8;
        if constexpr (VEC) {
            slot = id / C8;
            c8 = id % C8;
        } else if constexpr (PT) {
            slot = id % (BN / PX) * PX;
            c8 = id / (BN / PX);
        } else {
            c8 = (int)fdiv((uint32_t)id, A.fd_ns);
            slot = (id - c8 * (A.nslots / PX)) * PX;
        }
        bool ok = id < nunits;
        laddr[u] = ok ? (uint32_t)(slot * PITCH + c8 * 16) : (uint32_t)(A.nslots * PITCH + lane * 16);
        int hi, wi, n;
        if constexpr (PT) {
            const int q = q0 + slot;
            ok &= q < qend;
            const int row = (int)fdiv((uint32_t)q, A.fd_tw);
            n = (int)fdiv((uint32_t)row, A.fd_ho);
            hi = (row - n * A.Ho) * A.sh - A.ph;
            wi = (q - row * A.TW) * A.sw - A.pw;
        } else {
            const int vr = (int)fdiv((uint32_t)slot, A.fd_pw);
            const int v = v0 + vr;
            ok &= v < vend;
            n = (int)fdiv((uint32_t)v, A.fd_hv);
            hi = (v - n * A.HV) * A.ish - A.ph;
            wi = (wo0 * A.lsw + slot - vr * A.PW - cshift) * A.isw - A.pw;
        }
        ok = ok & ((unsigned)hi < (unsigned)A.H) & ((unsigned)wi < (unsigned)A.W);
        const int64_t e = xg + (int64_t)n * A.x_ns + (int64_t)hi * A.x_hs + (int64_t)wi * A.x_ws + (int64_t)c8 * 8 * A.x_cs;
        goff[u] = ok ? (uint32_t)(e * ES) : OOB_OFF;
    }

    // this lane's pixels in the patch
    uint32_t paddr[TN];
    const int wm = wave % WM, wn = wave / WM;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int px = (wn * TN + j) * 32 + lcol;
        int slot = px;
        if constexpr (!PT) {
            const int q = q0 + px;
            const int row = (int)fdiv((uint32_t)q, A.fd_tw);
            const int n = (int)fdiv((uint32_t)row, A.fd_ho);
            slot = (n * A.HV + (row - n * A.Ho) * A.lsh - v0) * A.PW + (q - row * A.TW) * A.lsw + cshift;
            if (q >= qend) slot = 0;
        }
        paddr[j] = (uint32_t)(slot * PITCH + lrow * 16);
    }

    // ---- staging of one chunk: loads into registers, then split / pack into LDS
    constexpr int RU = VEC ? (ES == 4 ? 8 : 4) : 8;  // registers per unit
    uint32_t sreg[UN][RU];
    // (past the last chunk: the same loads from an empty buffer, so that the count of loads in
    // flight does not depend on the chunk)
    auto issue = [&](int c) __attribute__((always_inline)) {
        const bool live = c < ce;
        const __amdgpu_buffer_rsrc_t rx = make_rsrc(A.x, live ? A.x_bytes : 0u);
        const int c0 = live ? c * CK : 0;
        const bool tail = c0 + CK > A.Cg;
        if constexpr (VEC) {
            const int so = c0 * ES;
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                uint32_t off = goff[u];
                if (tail && c0 + ((u * NT + t) % C8) * 8 >= A.Cg) off = OOB_OFF;
#pragma unroll
                for (int h = 0; h < RU / 4; ++h) {
                    const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rx, off + (off == OOB_OFF ? 0u : h * 16u), so, 0);
#pragma unroll
                    for (int q = 0; q < 4; ++q) sreg[u][h * 4 + q] = v[q];
                }
            }
        } else if (!tail) {
#pragma unroll
            for (int u = 0; u < UN; ++u)
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int so = (c0 + j) * A.x_cs * ES;
                    if constexpr (ES == 4 || PAIR) sreg[u][j] = __builtin_amdgcn_raw_buffer_load_b32(rx, goff[u], so, 0);
                    else sreg[u][j] = __builtin_amdgcn_raw_buffer_load_b16(rx, goff[u], so, 0);
                }
        } else {
            // last, partial chunk: channels past C/g read as zero (the next group's values, were
            // they not finite, would survive the zero filters).  The scalar offset stays inside x.
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                const int id = u * NT + t;
                const int c8 = PT ? id / (BN / PX) : (int)fdiv((uint32_t)id, A.fd_ns);
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int so = min(c0 + j, A.Cg - 1) * A.x_cs * ES;
                    const uint32_t off = c0 + c8 * 8 + j < A.Cg ? goff[u] : OOB_OFF;
                    if constexpr (ES == 4 || PAIR) sreg[u][j] = __builtin_amdgcn_raw_buffer_load_b32(rx, off, so, 0);
                    else sreg[u][j] = __builtin_amdgcn_raw_buffer_load_b16(rx, off, so, 0);
                }
            }
        }
    };
    auto put = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            if constexpr (NP == 3) {
                float f[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) f[j] = __builtin_bit_cast(float, sreg[u][j]);
                u32x4 pl[NP];
                planes_of<NP>(f, pl);
#pragma unroll
                for (int p = 0; p < NP; ++p) *reinterpret_cast<u32x4*>(lds + laddr[u] + p * CK * 2) = pl[p];
            } else if constexpr (PAIR) {
                u32x4 v0, v1;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    v0[q] = __builtin_amdgcn_perm(sreg[u][2 * q + 1], sreg[u][2 * q], 0x05040100u);
                    v1[q] = __builtin_amdgcn_perm(sreg[u][2 * q + 1], sreg[u][2 * q], 0x07060302u);
                }
                *reinterpret_cast<u32x4*>(lds + laddr[u]) = v0;
                *reinterpret_cast<u32x4*>(lds + laddr[u] + PITCH) = v1;
            } else {
                u32x4 v;
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    v[q] = VEC ? sreg[u][q] : (sreg[u][2 * q] & 0xffffu) | (sreg[u][2 * q + 1] << 16);
                *reinterpret_cast<u32x4*>(lds + laddr[u]) = v;
            }
        }
    };

    // ---- filters: TM x NP fragments per step (chunk, tap, ks), steps consecutive in memory
    const int mt0 = tile_m * (BM / 32) + wm * TM;
    int abase[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i)
        abase[i] = (gi * A.mtiles + min(mt0 + i, A.mtiles - 1)) * (A.nch * A.RS * KS * NP * 1024);
    const uint32_t alane = (uint32_t)lane * 16u;
    const int last_step = ce * A.RS * KS - 1;
    int step = cb * A.RS * KS;  // next step to load
    bf16x8 af[NSET][TM][NP];
    auto load_a = [&](bf16x8 (&a)[TM][NP]) __attribute__((always_inline)) {
        const int so = min(step, last_step) * (NP * 1024);
        ++step;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int p = 0; p < NP; ++p)
                a[i][p] = __builtin_bit_cast(
                    bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rp, alane, abase[i] + so + p * 1024, 0));
    };

    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;

    auto compute = [&](const bf16x8 (&a)[TM][NP], int tapoff, int k) __attribute__((always_inline)) {
        if (A.loader_only) return;
        bf16x8 b[TN][NP];
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int p = 0; p < NP; ++p)
                b[j][p] = *reinterpret_cast<const bf16x8*>(lds + (paddr[j] + (uint32_t)tapoff) + p * CK * 2 + k * 32);
        auto mm = [&](int pa, int pb) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i][pa], b[j][pb], acc[i][j], 0, 0, 0);
        };
        if constexpr (NP == 3) {  // smallest products first
            mm(2, 0);
            mm(0, 2);
            mm(1, 1);
            mm(1, 0);
            mm(0, 1);
        }
        mm(0, 0);
    };
    auto swap_patch = [&](int c) __attribute__((always_inline)) {
        if (c != cb) __syncthreads();  // every wave is done with the previous patch
        put();
        __syncthreads();
        issue(c + 1);
    };

    issue(cb);
    if constexpr (RSC > 0) {
        constexpr int NSS = RSC * KS;  // steps per chunk
        // chunks per trip of the loop, so that a step's register set is a constant
        constexpr int UC = NSS % NSET == 0 ? 1 : 2 * NSS % NSET == 0 ? 2 : 3;
        static_assert(UC * NSS % NSET == 0, "register sets");
#pragma unroll
        for (int q = 0; q < NSET - 1; ++q) load_a(af[q]);
        int c = cb;
        while (true) {
#pragma unroll
            for (int uc = 0; uc < UC; ++uc) {
                swap_patch(c);
#pragma unroll
                for (int ss = 0; ss < NSS; ++ss) {
                    const int n = uc * NSS + ss;
                    load_a(af[(n + NSET - 1) % NSET]);
                    const int tap = ss / KS;
                    compute(af[n % NSET], RSC == 1 ? 0 : ((tap / 3) * A.dh * A.PW + (tap % 3) * A.dw) * PITCH, ss % KS);
                }
                if (++c == ce) break;
            }
            if (c == ce) break;
        }
    } else {
        static_assert(RSC > 0 || NSET == 2 * KS, "two taps in registers");
        int c = cb, tr = 0, ts = 0;
        auto tap_step = [&](auto par) __attribute__((always_inline)) {
            constexpr int P0 = decltype(par)::value;
            if ((tr | ts) == 0) swap_patch(c);
            const int tapoff = (tr * A.dh * A.PW + ts * A.dw) * PITCH;
#pragma unroll
            for (int k = 0; k < KS; ++k) load_a(af[(1 - P0) * KS + k]);
#pragma unroll
            for (int k = 0; k < KS; ++k) compute(af[P0 * KS + k], tapoff, k);
            if (++ts == A.S) {
                ts = 0;
                if (++tr == A.R) {
                    tr = 0;
                    ++c;
                }
            }
        };
#pragma unroll
        for (int k = 0; k < KS; ++k) load_a(af[k]);
        while (true) {
            tap_step(std::integral_constant<int, 0>{});
            if (c == ce) break;
            tap_step(std::integral_constant<int, 1>{});
            if (c == ce) break;
        }
    }
    if (A.loader_only) return;

    // pixel of each accumulator column
    int pn[TN], pho[TN], pwo[TN];
    bool pok[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int q = q0 + (wn * TN + j) * 32 + lcol;
        const int row = (int)fdiv((uint32_t)q, A.fd_tw);
        pn[j] = (int)fdiv((uint32_t)row, A.fd_ho);
        pho[j] = row - pn[j] * A.Ho;
        pwo[j] = wo0 + q - row * A.TW;
        pok[j] = (q < qend) & (pwo[j] < A.Wo);
    }

    if constexpr (NP == 3) {
        // A value that is not finite, or whose scaled form rounds past the largest bf16, splits into
        // infinities of both signs; any such operand leaves a NaN in its sums, as a sum past the
        // largest fp32 leaves an infinity.  A wave that finds one computes its tile again with the
        // fp32 matrix instruction on the operands as they are: the plain fp32 sum.  Its operands come
        // from memory for every tap (eight channels' loads leave together, each used by TM or TN
        // products): N32 64->64 56x56 3x3 with one infinity 76 us (50 without), all NaN 219 us.
        float z = 0.0f;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) z = __builtin_fmaf(acc[i][j][v], 0.0f, z);
        if (__any(z != 0.0f)) {
            const __amdgpu_buffer_rsrc_t rw = make_rsrc(A.w, A.w_bytes);
            const int ca = cb * CK, cz = min(ce * CK, A.Cg);
            constexpr int U = 4;  // steps of two channels whose loads leave together
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;
#pragma unroll 1
            for (int r = 0; r < A.R; ++r)
#pragma unroll 1
                for (int q = 0; q < A.S; ++q) {
                    int64_t e[TN];
                    bool ok[TN];
#pragma unroll
                    for (int j = 0; j < TN; ++j) ok[j] = tap_at(A, pn[j], pho[j], pwo[j], r, q, &e[j]) & pok[j];
#pragma unroll 1
                    for (int c = ca; c < cz; c += 2 * U) {
                        float xv[U][TN], wv[U][TM];
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            const int cc = c + 2 * u + lrow;
                            const bool live = cc < cz;
#pragma unroll
                            for (int j = 0; j < TN; ++j)
                                xv[u][j] = ld_f32(rx, live & ok[j] ? (uint32_t)((xg + e[j] + (int64_t)cc * A.x_cs) * 4) : OOB_OFF);
#pragma unroll
                            for (int i = 0; i < TM; ++i) {
                                const int m = (mt0 + i) * 32 + lcol;
                                const int64_t we = ((int64_t)(gi * A.Kg + m) * A.Cg + cc) * A.RS + r * A.S + q;
                                wv[u][i] = ld_f32(rw, live & (m < A.Kg) ? (uint32_t)(we * 4) : OOB_OFF);
                            }
                        }
#pragma unroll
                        for (int u = 0; u < U; ++u)
#pragma unroll
                            for (int i = 0; i < TM; ++i)
#pragma unroll
                                for (int j = 0; j < TN; ++j)
                                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(wv[u][i], xv[u][j], acc[i][j], 0, 0, 0);
                    }
                }
        } else {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int v = 0; v < 16; ++v) acc[i][j][v] *= kSplitUnscale;
        }
    }

    if (tail_tile >= 0 && !tail_reduce<TM, TN, NT>(A.tail_part, A.tail_count, A.tail_tiles, A.tail_pieces, acc,
                                                   tail_tile, piece, t))
        return;

    // ---- epilogue: accumulator v of lane l holds row 8*(v/4) + 4*(l/32) + v%4, column l%32
    const int mb = mt0 * 32;
    if (A.bias != nullptr) {
        const __amdgpu_buffer_rsrc_t rbias = make_rsrc(A.bias, (uint32_t)(A.G * A.Kg * 4));
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int m = mb + i * 32 + 8 * (v >> 2) + 4 * lrow + (v & 3);
                const float bv = ld_f32(rbias, m < A.Kg ? (uint32_t)((gi * A.Kg + m) * 4) : OOB_OFF);
#pragma unroll
                for (int j = 0; j < TN; ++j) acc[i][j][v] += bv;
            }
    }
    const __amdgpu_buffer_rsrc_t ry = make_rsrc(A.y, A.y_bytes);
    auto store = [&](auto out) __attribute__((always_inline)) {
        using TOut = decltype(out);
        constexpr int YS = sizeof(TOut);
        if (A.epi == EPI_NHWC && A.Kg % 4 == 0) {
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int64_t base = (((int64_t)pn[j] * A.Ho + pho[j]) * A.Wo + pwo[j]) * A.ldc + (int64_t)gi * A.Kg;
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int v4 = 0; v4 < 4; ++v4) {
                        const int m = mb + i * 32 + 8 * v4 + 4 * lrow;
                        const bool ok = pok[j] & (m < A.Kg);
                        const float f0 = acc[i][j][4 * v4], f1 = acc[i][j][4 * v4 + 1], f2 = acc[i][j][4 * v4 + 2],
                                    f3 = acc[i][j][4 * v4 + 3];
                        if constexpr (YS == 4)
                            store_out4<float>(ry, (uint32_t)(base + m), ok, f0, f1, f2, f3);
                        else
                            __builtin_amdgcn_raw_buffer_store_b64(u32x2{pk_bf16(f0, f1), pk_bf16(f2, f3)}, ry,
                                                                  ok ? (uint32_t)(base + m) * 2u : OOB_OFF, 0, 0);
                    }
            }
            return;
        }
        // bytes between output channels, and this lane's byte offset of its first row
        const int ms = (A.epi == EPI_NCHW ? A.HoWo : A.epi == EPI_NHWC ? 1 : A.ldc) * YS;
        const bool full = mb + TM * 32 <= A.Kg;
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            int64_t base;
            if (A.epi == EPI_NCHW)
                base = ((int64_t)pn[j] * A.G + gi) * A.Kg * A.HoWo + pho[j] * A.Wo + pwo[j];
            else if (A.epi == EPI_NHWC)
                base = (((int64_t)pn[j] * A.Ho + pho[j]) * A.Wo + pwo[j]) * A.ldc + (int64_t)gi * A.Kg;
            else
                base = (int64_t)sp * A.c_sstride + (int64_t)gi * A.Kg * A.ldc + ((int64_t)pn[j] * A.Ho + pho[j]) * A.Wo + pwo[j];
            const uint32_t lb = pok[j] ? (uint32_t)(base * YS + (int64_t)(mb + 4 * lrow) * ms) : OOB_OFF;
            if (YS == 2 && full && A.ypair) {
                // the neighbouring lane holds the next pixel of the same row: of two rows, even
                // lanes store the first and odd lanes the second, two pixels (4 bytes) each
                const bool odd = lane & 1;
                const uint32_t pb = pok[j] ? lb + (odd ? (uint32_t)ms - 2u : 0u) : OOB_OFF;
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int v = 0; v < 16; v += 2) {
                        const int r0 = i * 32 + 8 * (v >> 2) + (v & 3);
                        const float f0 = acc[i][j][v], f1 = acc[i][j][v + 1];
                        const float o = swap_adjacent_lanes(odd ? f0 : f1);
                        __builtin_amdgcn_raw_buffer_store_b32(odd ? pk_bf16(o, f1) : pk_bf16(f0, o), ry, pb, r0 * ms, 0);
                    }
            } else if (full) {  // row offsets are wave-uniform
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int v = 0; v < 16; v += 2) {
                        const int r0 = i * 32 + 8 * (v >> 2) + (v & 3);
                        const float f0 = acc[i][j][v], f1 = acc[i][j][v + 1];
                        if constexpr (YS == 4) {
                            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, f0), ry, lb, r0 * ms, 0);
                            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, f1), ry, lb, (r0 + 1) * ms, 0);
                        } else {
                            const uint32_t w2 = pk_bf16(f0, f1);
                            __builtin_amdgcn_raw_buffer_store_b16((uint16_t)w2, ry, lb, r0 * ms, 0);
                            __builtin_amdgcn_raw_buffer_store_b16((uint16_t)(w2 >> 16), ry, lb, (r0 + 1) * ms, 0);
                        }
                    }
            } else {
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const int r0 = i * 32 + 8 * (v >> 2) + (v & 3);
                        const bool ok = pok[j] & (mb + r0 + 4 * lrow < A.Kg);
                        const uint32_t off = ok ? lb + (uint32_t)(r0 * ms) : OOB_OFF;
                        const float f = acc[i][j][v];
                        if constexpr (YS == 4) st_f32(ry, off, f);
                        else st_u16(ry, off, (uint16_t)pk_bf16(f, f));
                    }
            }
        }
    };
    if constexpr (NP == 3) {
        store(0.0f);
    } else {
        if (A.y_es == 4) store(0.0f);
        else store((uint16_t)0);
    }
}

template <int NP, int KS, int TM, int TN, int WM, int WN, int MINW, bool PT, int LD, int UMAX>
hipError_t launch_ld(const PatchArgs& a, int un, unsigned lds, hipStream_t s) {
    constexpr int BM = WM * TM * 32, BN = WN * TN * 32, NT = WM * WN * 64;
    const dim3 grid((unsigned)(a.tiles_q * a.ncb * a.grid_m + a.tail_tiles * (a.tail_pieces - 1)), 1, (unsigned)(a.G * (a.ksplit > 1 ? a.ksplit : 1)));
    if ((int64_t)a.nslots * KS * 2 > (int64_t)un * NT * (LD == PATCH_LD_PAIR ? 2 : 1) || a.grid_m * BM < a.Kg)
        return hipErrorInvalidValue;
    if (a.tail_tiles != 0 &&
        (a.tail_tiles < 0 || a.tail_tiles > a.tiles_q * a.ncb * a.grid_m || a.tail_pieces < 2 || a.tail_ch < 1 || a.G != 1 ||
         a.ksplit > 1 || !a.tail_part || !a.tail_count || a.tail_pieces * a.tail_ch < a.nch ||
         (a.tail_pieces - 1) * a.tail_ch >= a.nch))
        return hipErrorInvalidValue;
#define CV_P(RSCV, UNV, NS) \
    hipLaunchKernelGGL((patch_conv_kernel<NP, KS, TM, TN, WM, WN, RSCV, LD, UNV, NS, MINW>), grid, dim3(NT), lds, s, a)
    if constexpr (PT) {
        constexpr int U = BN * KS * 2 / NT / (LD == PATCH_LD_PAIR ? 2 : 1);
        if (un != U || a.nslots != BN || a.ncb != 1) return hipErrorInvalidValue;
        CV_P(1, U, (NP == 3 ? 3 : 4));
    } else if (UMAX == 4 && un == 3) {
        if (a.R == 3 && a.S == 3) CV_P(9, 3, (NP == 3 ? 3 : 6));
        else CV_P(0, 3, 2 * KS);
    } else if (un == 4) {
        if (a.R == 3 && a.S == 3) CV_P(9, 4, (NP == 3 ? 3 : 6));
        else CV_P(0, 4, 2 * KS);
    } else if constexpr (UMAX >= 8) {
        if (un != 8) return hipErrorInvalidValue;
        if (a.R == 3 && a.S == 3) CV_P(9, 8, (NP == 3 ? 3 : 6));
        else CV_P(0, 8, 2 * KS);
    } else {
        return hipErrorInvalidValue;
    }
#undef CV_P
    return hipGetLastError();
}

template <int NP, int KS, int TM, int TN, int WM, int WN, int MINW, bool PT, int UMAX = 8>
hipError_t launch_cfg(const PatchArgs& a, const PatchPlan& p, hipStream_t s) {
    // the patch, and where staging units past its end are written
    const unsigned lds = (unsigned)patch_lds_bytes(p);
    if (lds > 160u * 1024u) return hipErrorInvalidValue;
    if (p.ld == PATCH_LD_ONE) return launch_ld<NP, KS, TM, TN, WM, WN, MINW, PT, PATCH_LD_ONE, UMAX>(a, p.un, lds, s);
    if (p.ld == PATCH_LD_VEC) {
        if (a.x_cs != 1 || a.Cg % 8 != 0 || ((uintptr_t)a.x & 15) != 0) return hipErrorInvalidValue;
        return launch_ld<NP, KS, TM, TN, WM, WN, MINW, PT, PATCH_LD_VEC, UMAX>(a, p.un, lds, s);
    }
    if constexpr (NP == 1) {
        if (a.x_ws != 1 || a.W % 2 != 0 || (PT ? a.TW % 2 != 0 || a.sw != 1 || a.pw != 0 : a.PW % 2 != 0 || a.isw != 1) ||
            ((uintptr_t)a.x & 3) != 0)
            return hipErrorInvalidValue;
        return launch_ld<NP, KS, TM, TN, WM, WN, MINW, PT, PATCH_LD_PAIR, UMAX>(a, p.un, lds, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_pack_filters(const void* w, uint32_t w_bytes, void* wp, uint32_t wp_bytes, int G, int Kg, int Cg,
                               int RS, int np, int ks, hipStream_t s) {
    const int mtiles = (Kg + 31) / 32, nch = (Cg + 16 * ks - 1) / (16 * ks);
    const int64_t nf = (int64_t)nch * RS * ks, rows = (int64_t)G * mtiles;
    if (rows * nf * np * 1024 != (int64_t)wp_bytes || rows > 65535 || (np != 1 && np != 3) || (ks != 1 && ks != 2) ||
        (np == 1 && ks == 1))
        return hipErrorInvalidValue;
    const dim3 grid((unsigned)((nf + 3) / 4), (unsigned)rows);
#define CV_W(NPV, KSV, T)                                                                                        \
    hipLaunchKernelGGL((pack_filters_kernel<NPV, KSV, T>), grid, dim3(256), 0, s, static_cast<const T*>(w), w_bytes, wp, \
                       wp_bytes, (int)nf, mtiles, Kg, Cg, RS, make_fastdiv((uint32_t)RS), make_fastdiv((uint32_t)mtiles))
    if (np == 1) CV_W(1, 2, uint16_t);
    else if (ks == 1) CV_W(3, 1, float);
    else CV_W(3, 2, float);
#undef CV_W
    return hipGetLastError();
}

int patch_threads(const PatchPlan& p) { return p.np == 1 && p.cfg == PATCH_64x128 ? 128 : 256; }
int patch_units(const PatchPlan& p) {
    if (p.pt) return kPatchShapes[p.cfg].bn * p.ks * 2 / patch_threads(p) / (p.ld == PATCH_LD_PAIR ? 2 : 1);
    return p.cfg == PATCH_256x128 || (p.np == 3 && kPatchShapes[p.cfg].bm * kPatchShapes[p.cfg].bn <= 8192) ? 4 : 8;
}
void patch_wave_tile(const PatchPlan& p, int* tm, int* tn) {
    *tm = p.cfg == PATCH_32x256 || (p.cfg == PATCH_64x128 && p.np == 3) ? 1 : 2;
    *tn = p.cfg == PATCH_256x128 ? 4 : 2;
}
int64_t patch_lds_bytes(const PatchPlan& p) {
    const int64_t pitch = p.np * p.ks * 32 + 16;
    return (int64_t)p.nslots * pitch + 1024 + 2 * pitch;
}

hipError_t launch_patch(const PatchArgs& a, const PatchPlan& p, hipStream_t s) {
#define CV_C(...) return launch_cfg<__VA_ARGS__>(a, p, s)
    if (p.np == 3 && p.pt && p.ks == 2) {
        switch (p.cfg) {
            case PATCH_64x128: CV_C(3, 2, 1, 2, 2, 2, 2, true);
            case PATCH_64x256: CV_C(3, 2, 2, 2, 1, 4, 2, true);
            case PATCH_128x128: CV_C(3, 2, 2, 2, 2, 2, 2, true);
            case PATCH_32x256: CV_C(3, 2, 1, 2, 1, 4, 2, true);
        }
    } else if (p.np == 3 && !p.pt && p.ks == 1) {
        switch (p.cfg) {
            case PATCH_64x128: CV_C(3, 1, 1, 2, 2, 2, 4, false, 4);
            case PATCH_64x256: CV_C(3, 1, 2, 2, 1, 4, 2, false);
            case PATCH_128x128: CV_C(3, 1, 2, 2, 2, 2, 2, false);
            case PATCH_32x256: CV_C(3, 1, 1, 2, 1, 4, 4, false, 4);
        }
    } else if (p.np == 1 && p.pt && p.ks == 2) {
        switch (p.cfg) {
            case PATCH_64x128: CV_C(1, 2, 2, 2, 1, 2, 2, true);
            case PATCH_64x256: CV_C(1, 2, 2, 2, 1, 4, 2, true);
            case PATCH_128x128: CV_C(1, 2, 2, 2, 2, 2, 2, true);
            case PATCH_32x256: CV_C(1, 2, 1, 2, 1, 4, 2, true);
            case PATCH_256x128: CV_C(1, 2, 2, 4, 4, 1, 2, true);
        }
    } else if (p.np == 1 && !p.pt && p.ks == 2) {
        switch (p.cfg) {
            case PATCH_64x128: CV_C(1, 2, 2, 2, 1, 2, 2, false);
            case PATCH_64x256: CV_C(1, 2, 2, 2, 1, 4, 2, false);
            case PATCH_128x128: CV_C(1, 2, 2, 2, 2, 2, 2, false);
            case PATCH_32x256: CV_C(1, 2, 1, 2, 1, 4, 2, false);
            case PATCH_256x128: CV_C(1, 2, 2, 4, 4, 1, 2, false, 4);
        }
    }
#undef CV_C
    return hipErrorInvalidValue;
}

}  // namespace cv
