// Group-wise asymmetric round-to-nearest quantization + LSB-first packing (2,
// 3 or 4 bits; the row is one bit string cut into 32-bit words), and the
// matching dequantization, for gfx950.
//
// The backbone quantizer of the paper is GPTQ (Section 5.1); without
// calibration data its error feedback vanishes and it is round-to-nearest on a
// per-group min/max grid that contains 0, defined in fp64 with IEEE division
// and round-half-to-even, the fp16 scale rounded once, directly from fp64.
// The kernels take a step of it in fp32 where the fp32 error bound shows that
// both round to the same value, and in fp64 otherwise, so the codes are
// bit-identical to the definition.
// This file is compiled with -ffp-contract=off.

#include "cl_device.h"
#include "cl_internal.h"

namespace cl {

__device__ double f16_bits_to_f64(uint16_t h) {
    return static_cast<double>(static_cast<float>(__builtin_bit_cast(f16, h)));
}

// One group's grid from its extremes (lo <= 0 <= hi): the fp16 step's bits
// and the zero point, in fp64.
__device__ void grid_exact(double lo, double hi, int qmax, uint16_t& sb, double& zf) {
    if (hi == lo) { lo = -1.0; hi = 1.0; }
    const double step = (hi - lo) / static_cast<double>(qmax);
    sb = f64_to_f16_rne(step);
    if (sb == 0) sb = 0x0001u;                 // smallest positive subnormal, 2^-24
    if (sb >= 0x7c00u) sb = 0x7bffu;           // largest finite, 65504
    zf = rint(-lo / f16_bits_to_f64(sb));
    zf = zf < 0.0 ? 0.0 : (zf > qmax ? static_cast<double>(qmax) : zf);
}

__device__ uint32_t code_exact(float w, double s16, double zf, int qmax) {
    double r = rint(static_cast<double>(w) / s16) + zf;
    r = r < 0.0 ? 0.0 : (r > qmax ? static_cast<double>(qmax) : r);
    return static_cast<uint32_t>(r);
}

// rint(r) equals the rint of the fp64 quotient that r approximates to within
// 2^-22 (a 1 ulp reciprocal and one product): r is further than 2^-21 |r|
// from the nearest half.  False for NaN and for |r| >= 2^20.
__device__ __forceinline__ bool rint_safe(float r) {
    return fabsf(r - rintf(r)) < 0.5f - fabsf(r) * 0x1p-21f;
}

struct Grid {
    float inv, zf;       // 1 / step (1 ulp), the zero point
    uint16_t sb;
};

// The same grid from fp32 arithmetic where that provably decides it, else
// from grid_exact.  hi - lo and its product with 1 / qmax are within 2^-22 of
// the fp64 step; if both ends of a 2^-21 interval round to one fp16, so does
// the step.
__device__ __forceinline__ Grid group_grid(float lo, float hi, int qmax, float rq) {
    Grid g;
    const float step = (hi - lo) * rq;
    g.sb = f32_to_f16_bits(step);
    const uint16_t up = f32_to_f16_bits(step * (1.f + 0x1p-21f)), dn = f32_to_f16_bits(step * (1.f - 0x1p-21f));
    g.inv = __builtin_amdgcn_rcpf(f16_bits_to_f32(g.sb));
    const float r = -lo * g.inv;
    g.zf = rintf(r);
    g.zf = g.zf < 0.f ? 0.f : (g.zf > qmax ? static_cast<float>(qmax) : g.zf);
    if (!(up == dn && g.sb > 0 && g.sb < 0x7bffu && rint_safe(r))) {
        double zf;
        grid_exact(static_cast<double>(lo), static_cast<double>(hi), qmax, g.sb, zf);
        g.zf = static_cast<float>(zf);          // small integer: exact
        g.inv = __builtin_amdgcn_rcpf(f16_bits_to_f32(g.sb));
    }
    return g;
}

// 8 codes as a bit string, LSB first
template <int BITS>
__device__ __forceinline__ uint32_t codes8(const float (&w)[8], const Grid& g) {
    constexpr float qmax = static_cast<float>((1 << BITS) - 1);
    uint32_t v = 0;
    bool safe = true;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const float r = w[i] * g.inv;
        safe = safe && rint_safe(r);
        const float c = fminf(fmaxf(rintf(r) + g.zf, 0.f), qmax);
        v |= static_cast<uint32_t>(c) << (BITS * i);
    }
    if (!safe) {
        const double s16 = f16_bits_to_f64(g.sb), zf = static_cast<double>(g.zf);
        v = 0;
        for (int i = 0; i < 8; ++i) v |= code_exact(w[i], s16, zf, (1 << BITS) - 1) << (BITS * i);
    }
    return v;
}

// Lanes of 8 consecutive codes each: their bit strings as whole words.  The
// lanes of a quad are all active or all idle (groups are multiples of 32
// codes).
template <int BITS>
__device__ __forceinline__ void store_codes8(uint32_t* __restrict__ q, size_t unit, uint32_t v, bool on) {
    if (BITS == 4) {
        if (on) q[unit] = v;
    } else if (BITS == 2) {
        const uint32_t next = __shfl_down(v, 1, 64);
        if (on && (unit & 1) == 0) q[unit >> 1] = v | (next << 16);
    } else {
        // word w of the quad's three: the high bytes of lane w, the low bytes of lane w + 1
        const uint32_t next = __shfl_down(v, 1, 64);
        const int l = static_cast<int>(unit & 3);
        if (on && l < 3) q[(unit >> 2) * 3 + l] = (v >> (8 * l)) | (next << (24 - 8 * l));
    }
}

template <bool VEC>
__device__ __forceinline__ void load8(const float* __restrict__ p, float (&w)[8]) {
    if (VEC) {
        const f32x4 a = *reinterpret_cast<const f32x4*>(p), b = *reinterpret_cast<const f32x4*>(p + 4);
#pragma unroll
        for (int i = 0; i < 4; ++i) { w[i] = a[i]; w[4 + i] = b[i]; }
    } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) w[i] = p[i];
    }
}

__device__ __forceinline__ void extremes8(const float (&w)[8], float& lo, float& hi) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        lo = w[i] < lo ? w[i] : lo;
        hi = w[i] > hi ? w[i] : hi;
    }
}

// min / max over blocks of L lanes.  The selects keep a +0 extreme +0, which
// decides the sign of a zero zero point.
template <int L>
__device__ __forceinline__ void extremes_across(float& lo, float& hi) {
#pragma unroll
    for (int off = 1; off < L; off *= 2) {
        const float l = __shfl_xor(lo, off, 64), h = __shfl_xor(hi, off, 64);
        lo = l < lo ? l : lo;
        hi = h > hi ? h : hi;
    }
}

// Bound by HBM: 4 bytes in and bits / 8 out per code.  A lane owns 8
// consecutive codes (32 bytes of W, coalesced) and L = G / 8 lanes a group, so
// W is read once and a lane's codes are a whole number of bytes.  Rows and
// groups are contiguous, so all indexing is flat.  The fp64 definition is
// decided in fp32 except where its error bound leaves it open: under 1 % of the
// waves at 4 bits and groups of 128, 2 % at groups of 32, mostly next to a
// rounding of the fp16 step (counted on N(0, 0.02^2) weights).
// 14336 x 4096, 4 bits: 62 us, 4.3 TB/s (one thread per group reading its codes
// one by one, with an fp64 division each: 2100 us).
template <int BITS, int L, bool VEC>
__global__ __launch_bounds__(256) void quantize_pack_kernel(const float* __restrict__ W, size_t units,
                                                            uint32_t* __restrict__ q, uint16_t* __restrict__ s,
                                                            uint16_t* __restrict__ z) {
    constexpr int qmax = (1 << BITS) - 1;
    const size_t unit = static_cast<size_t>(blockIdx.x) * 256 + threadIdx.x;
    const bool on = unit < units;               // whole groups are on or off: L divides units
    float w[8] = {};
    if (on) load8<VEC>(W + unit * 8, w);
    float lo = 0.f, hi = 0.f;
    extremes8(w, lo, hi);
    extremes_across<L>(lo, hi);
    const Grid g = group_grid(lo, hi, qmax, 1.f / qmax);
    store_codes8<BITS>(q, unit, codes8<BITS>(w, g), on);
    if (on && unit % L == 0) {
        s[unit / L] = g.sb;
        z[unit / L] = f32_to_f16_bits(g.zf);
    }
}

// Groups of any other size: one wave per group, which reads its codes twice
// (the second time from the caches).
template <int BITS>
__global__ __launch_bounds__(256) void quantize_pack_any_kernel(const float* __restrict__ W, size_t groups, int G,
                                                                uint32_t* __restrict__ q, uint16_t* __restrict__ s,
                                                                uint16_t* __restrict__ z) {
    constexpr int qmax = (1 << BITS) - 1;
    const size_t grp = static_cast<size_t>(blockIdx.x) * 4 + (threadIdx.x >> 6);
    if (grp >= groups) return;
    const int lane = threadIdx.x & 63, per = G / 8;
    const size_t unit0 = grp * per;
    float lo = 0.f, hi = 0.f, w[8];
    for (int u = lane; u < per; u += 64) {
        load8<false>(W + (unit0 + u) * 8, w);
        extremes8(w, lo, hi);
    }
    extremes_across<64>(lo, hi);
    const Grid g = group_grid(lo, hi, qmax, 1.f / qmax);
    for (int u0 = 0; u0 < per; u0 += 64) {
        const bool on = u0 + lane < per;
        if (on) load8<false>(W + (unit0 + u0 + lane) * 8, w);
        store_codes8<BITS>(q, unit0 + u0 + lane, codes8<BITS>(w, g), on);
    }
    if (lane == 0) {
        s[grp] = g.sb;
        z[grp] = f32_to_f16_bits(g.zf);
    }
}

// Bound by HBM: 4 bytes out per code.  A lane writes the 16 bytes of 4
// consecutive codes, so a wave's stores are one run of 1 KiB; kPer such runs
// per lane keep several loads in flight.  14336 x 4096, 4 bits: 39 us, 6.8 TB/s
// (one code and a 4-byte store per thread: 140 us).
template <int BITS, bool VEC>
__global__ __launch_bounds__(256) void dequantize_kernel(const uint32_t* __restrict__ q, const uint16_t* __restrict__ s,
                                                         const uint16_t* __restrict__ z, size_t units, int G4,
                                                         int shift, float* __restrict__ out) {
    constexpr int kPer = 4;
    const size_t base = static_cast<size_t>(blockIdx.x) * (256 * kPer) + threadIdx.x;
    uint32_t v[kPer];
    float sc[kPer], zp[kPer];
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        size_t u = base + 256 * k;
        u = u < units ? u : units - 1;
        if (BITS == 4) {
            v[k] = reinterpret_cast<const uint16_t*>(q)[u];
        } else if (BITS == 2) {
            v[k] = reinterpret_cast<const uint8_t*>(q)[u];
        } else {
            // 12 bits at bit 12 (u mod 8) of 3 words: bytes 3 (u / 2) + (u mod 2) and the next
            const uint8_t* b = reinterpret_cast<const uint8_t*>(q) + 3 * (u >> 1) + (u & 1);
            v[k] = (b[0] | static_cast<uint32_t>(b[1]) << 8) >> (4 * (u & 1));
        }
        const size_t gi = shift >= 0 ? u >> shift : u / static_cast<size_t>(G4);
        sc[k] = f16_bits_to_f32(s[gi]);
        zp[k] = f16_bits_to_f32(z[gi]);
    }
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const size_t u = base + 256 * k;
        if (u >= units) return;
        f32x4 o;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            o[i] = sc[k] * (static_cast<float>((v[k] >> (BITS * i)) & ((1u << BITS) - 1u)) - zp[k]);
        if (VEC) {
            *reinterpret_cast<f32x4*>(out + 4 * u) = o;
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) out[4 * u + i] = o[i];
        }
    }
}

namespace {

unsigned blocks_of(size_t n, size_t per) { return static_cast<unsigned>((n + per - 1) / per); }

bool aligned16(const void* p) { return reinterpret_cast<uintptr_t>(p) % 16 == 0; }

template <int BITS, int L>
void launch_quantize(const float* W, size_t units, uint32_t* q, uint16_t* s, uint16_t* z, hipStream_t st) {
    const dim3 grid(blocks_of(units, 256)), block(256);
    if (aligned16(W))
        hipLaunchKernelGGL((quantize_pack_kernel<BITS, L, true>), grid, block, 0, st, W, units, q, s, z);
    else
        hipLaunchKernelGGL((quantize_pack_kernel<BITS, L, false>), grid, block, 0, st, W, units, q, s, z);
}

// A group is a power-of-two number of lanes of 8 codes up to a wave (32 to
// 512 codes), or takes a wave to itself.
template <int BITS>
void launch_quantize_bits(const float* W, size_t total, int G, uint32_t* q, uint16_t* s, uint16_t* z,
                          hipStream_t st) {
    switch (G) {
        case 32: return launch_quantize<BITS, 4>(W, total / 8, q, s, z, st);
        case 64: return launch_quantize<BITS, 8>(W, total / 8, q, s, z, st);
        case 128: return launch_quantize<BITS, 16>(W, total / 8, q, s, z, st);
        case 256: return launch_quantize<BITS, 32>(W, total / 8, q, s, z, st);
        case 512: return launch_quantize<BITS, 64>(W, total / 8, q, s, z, st);
    }
    const size_t groups = total / G;
    hipLaunchKernelGGL((quantize_pack_any_kernel<BITS>), dim3(blocks_of(groups, 4)), dim3(256), 0, st, W, groups, G, q,
                       s, z);
}

template <int BITS>
void launch_dequantize_bits(const QW& w, float* out, hipStream_t st) {
    const size_t units = static_cast<size_t>(w.d_out) * w.d_in / 4;
    const int G4 = w.G / 4;
    const int shift = (G4 & (G4 - 1)) == 0 ? __builtin_ctz(G4) : -1;
    const dim3 grid(blocks_of(units, 1024)), block(256);
    if (aligned16(out))
        hipLaunchKernelGGL((dequantize_kernel<BITS, true>), grid, block, 0, st, w.q, w.s, w.z, units, G4, shift, out);
    else
        hipLaunchKernelGGL((dequantize_kernel<BITS, false>), grid, block, 0, st, w.q, w.s, w.z, units, G4, shift, out);
}

}  // namespace

hipError_t launch_quantize_pack(const float* W, int d_out, int d_in, int bits, int G, uint32_t* q,
                                uint16_t* s, uint16_t* z, hipStream_t st) {
    const size_t total = static_cast<size_t>(d_out) * d_in;
    if (bits == 4) launch_quantize_bits<4>(W, total, G, q, s, z, st);
    else if (bits == 3) launch_quantize_bits<3>(W, total, G, q, s, z, st);
    else launch_quantize_bits<2>(W, total, G, q, s, z, st);
    return hipGetLastError();
}

hipError_t launch_dequantize(const QW& w, float* out, hipStream_t st) {
    if (w.bits == 4) launch_dequantize_bits<4>(w, out, st);
    else if (w.bits == 3) launch_dequantize_bits<3>(w, out, st);
    else launch_dequantize_bits<2>(w, out, st);
    return hipGetLastError();
}

}  // namespace cl
