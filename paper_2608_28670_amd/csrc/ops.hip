// Small kernels around the block GEMMs and attention: LayerNorm + adaLN
// modulation, the skinny linear layers of the conditioning path, patch
// embedding, the final layer, sampler updates and element-wise helpers.
// All statistics and accumulations are fp32.
#include <type_traits>
#include <algorithm>
#include <cmath>

#include "ops.h"

namespace bc {

constexpr float kLnEps = 1e-6f;
constexpr int kMaxPatch = 256;

// ---------------------------------------------------------------------------
// LayerNorm + modulate: one wave per row, the row cached in registers as
// 4-element chunks (lane l holds chunks l, l + 64, ...), so every load is 16
// (fp32) or 8 (bf16) bytes and every store 8 (bf16) or 16 (fp32) bytes.
// Requires D % 4 == 0.
// ---------------------------------------------------------------------------
template <typename T> struct Vec4;
template <> struct Vec4<float> {
    __device__ static void load(const float* p, float* v) {
        const f32x4 x = *reinterpret_cast<const f32x4*>(p);
        v[0] = x[0]; v[1] = x[1]; v[2] = x[2]; v[3] = x[3];
    }
    __device__ static void store(float* p, const float* v) {
        *reinterpret_cast<f32x4*>(p) = f32x4{v[0], v[1], v[2], v[3]};
    }
};
template <> struct Vec4<bf16> {
    __device__ static void load(const bf16* p, float* v) {
        typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));
        const u32x2_t w = *reinterpret_cast<const u32x2_t*>(p);
        v[0] = __uint_as_float(w[0] << 16); v[1] = __uint_as_float(w[0] & 0xffff0000u);
        v[2] = __uint_as_float(w[1] << 16); v[3] = __uint_as_float(w[1] & 0xffff0000u);
    }
    __device__ static void store(bf16* p, const float* v) {
        typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));
        uint32_t w[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const bf16 lo = (bf16)v[2 * i], hi = (bf16)v[2 * i + 1];
            w[i] = (uint32_t)__builtin_bit_cast(uint16_t, lo) | ((uint32_t)__builtin_bit_cast(uint16_t, hi) << 16);
        }
        *reinterpret_cast<u32x2_t*>(p) = u32x2_t{w[0], w[1]};
    }
};

// Each wave takes RPW consecutive rows: the next row's chunks are loaded
// while the current one is reduced, and the modulation vectors (one pair per
// sample) are loaded once per sample instead of once per row.
template <typename Tin_, typename Tout_, int NC, int RPW>
__global__ __launch_bounds__(256) void ln_mod_kernel(const elem_t<Tin_>* __restrict__ x, int64_t rows, int D,
                                                     const float* __restrict__ shift,
                                                     const float* __restrict__ scale, int64_t ld_mod, int rps,
                                                     elem_t<Tout_>* __restrict__ h) {
    typedef elem_t<Tin_> Tin;
    typedef elem_t<Tout_> Tout;
    const int lane = threadIdx.x & 63;
    const int64_t row0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * RPW;
    if (row0 >= rows) return;
    const int nch = D >> 2;
    float v[2][NC][4], s4[NC][4], c4[NC][4];
    auto load_row = [&](int64_t row, float (&dst)[NC][4]) {
        const Tin* xr = x + row * D;
#pragma unroll
        for (int j = 0; j < NC; ++j) {
            const int c = lane + 64 * j;
            if (c < nch) Vec4<Tin>::load(xr + 4 * c, dst[j]);
            else {
#pragma unroll
                for (int e = 0; e < 4; ++e) dst[j][e] = 0.f;
            }
        }
    };
    load_row(row0, v[0]);
    int64_t cur_b = -1;
#pragma unroll
    for (int i = 0; i < RPW; ++i) {
        const int64_t row = row0 + i;
        if (row >= rows) break;
        if (i + 1 < RPW && row + 1 < rows) load_row(row + 1, v[(i + 1) & 1]);
        const int64_t b = row / rps;
        if (b != cur_b) {
            cur_b = b;
            const float* sh = shift + b * ld_mod;
            const float* sc = scale + b * ld_mod;
#pragma unroll
            for (int j = 0; j < NC; ++j) {
                const int c = lane + 64 * j;
                if (c < nch) {
                    Vec4<float>::load(sh + 4 * c, s4[j]);
                    Vec4<float>::load(sc + 4 * c, c4[j]);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) s4[j][e] = c4[j][e] = 0.f;
                }
            }
        }
        const float (&r)[NC][4] = v[i & 1];
        float sum = 0.f;
#pragma unroll
        for (int j = 0; j < NC; ++j) sum += (r[j][0] + r[j][1]) + (r[j][2] + r[j][3]);
        const float mean = wave_sum(sum) / (float)D;
        float sq = 0.f;
#pragma unroll
        for (int j = 0; j < NC; ++j) {
            if (lane + 64 * j < nch) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float d = r[j][e] - mean;
                    sq += d * d;
                }
            }
        }
        const float rstd = 1.0f / sqrtf(wave_sum(sq) / (float)D + kLnEps);
        Tout* hr = h + row * D;
#pragma unroll
        for (int j = 0; j < NC; ++j) {
            const int c = lane + 64 * j;
            if (c < nch) {
                float o[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = (r[j][e] - mean) * rstd * (1.0f + c4[j][e]) + s4[j][e];
                Vec4<Tout>::store(hr + 4 * c, o);
            }
        }
    }
}

template <typename Tin, typename Tout, int RPW>
static int run_ln_rows(const void* x, int64_t rows, int D, const float* shift, const float* scale, int64_t ld_mod,
                       int rps, void* h, hipStream_t s) {
    const int nc = (D / 4 + 63) / 64;
    dim3 g((unsigned)((rows + 4 * RPW - 1) / (4 * RPW))), b(256);
    const Tin* xi = static_cast<const Tin*>(x);
    Tout* ho = static_cast<Tout*>(h);
    if (nc <= 1) launch_k(ln_mod_kernel<tag_t<Tin>, tag_t<Tout>, 1, RPW>, g, b, s, xi, rows, D, shift, scale, ld_mod, rps, ho);
    else if (nc <= 2) launch_k(ln_mod_kernel<tag_t<Tin>, tag_t<Tout>, 2, RPW>, g, b, s, xi, rows, D, shift, scale, ld_mod, rps, ho);
    else if (nc <= 5) launch_k(ln_mod_kernel<tag_t<Tin>, tag_t<Tout>, 5, RPW>, g, b, s, xi, rows, D, shift, scale, ld_mod, rps, ho);
    else if (nc <= 8) launch_k(ln_mod_kernel<tag_t<Tin>, tag_t<Tout>, 8, RPW>, g, b, s, xi, rows, D, shift, scale, ld_mod, rps, ho);
    else if (nc <= 12) launch_k(ln_mod_kernel<tag_t<Tin>, tag_t<Tout>, 12, RPW>, g, b, s, xi, rows, D, shift, scale, ld_mod, rps, ho);
    else if (nc <= 16) launch_k(ln_mod_kernel<tag_t<Tin>, tag_t<Tout>, 16, RPW>, g, b, s, xi, rows, D, shift, scale, ld_mod, rps, ho);
    else return fail(BC_ERR_UNSUPPORTED, "LayerNorm width %d > 4096", D);
    return check_launch("ln_mod");
}

// Rows per wave: two (the second row's loads in flight while the first is
// reduced), four for rows of up to 1280 values when there are at least 8192
// of them (PixArt's 16 384 rows of 1152: 20.6 -> 18.6 us; DiT-XL/2's 4096
// rows are fastest with two: 7.7 us against 8.6 with four and 8.0 with one).
// One for up to 2048 rows, where two leave a CU fewer than four waves and the
// second row only lengthens the chain: 1020 rows of 1152 4.3 us against 5.1,
// 1846 of 3072 10.9 against 11.8, 128 of 128 3.0 against 3.5.
template <typename Tin, typename Tout>
static int run_ln(const void* x, int64_t rows, int D, const float* shift, const float* scale, int64_t ld_mod, int rps,
                  void* h, hipStream_t s) {
    if (rows <= 2048) return run_ln_rows<Tin, Tout, 1>(x, rows, D, shift, scale, ld_mod, rps, h, s);
    if (D <= 1280 && rows >= 8192) return run_ln_rows<Tin, Tout, 4>(x, rows, D, shift, scale, ld_mod, rps, h, s);
    return run_ln_rows<Tin, Tout, 2>(x, rows, D, shift, scale, ld_mod, rps, h, s);
}

int launch_ln_mod(int in_dt, const void* x, int64_t rows, int D, const float* shift, const float* scale,
                  int64_t ld_mod, int rows_per_sample, int out_dt, void* h, hipStream_t s) {
    if (rows <= 0) return BC_OK;
    if (D % 4 || ld_mod % 4 || (reinterpret_cast<uintptr_t>(shift) | reinterpret_cast<uintptr_t>(scale)) % 16)
        return fail(BC_ERR_UNSUPPORTED, "LayerNorm needs D and the modulation rows in 16-byte units");
    prof_begin(PROF_LAYERNORM, s, (double)rows * D * (dtype_size(in_dt) + dtype_size(out_dt)));
    int rc;
    if (in_dt == BC_F32 && out_dt == BC_BF16) rc = run_ln<float, bf16>(x, rows, D, shift, scale, ld_mod, rows_per_sample, h, s);
    else if (in_dt == BC_F32) rc = run_ln<float, float>(x, rows, D, shift, scale, ld_mod, rows_per_sample, h, s);
    else if (out_dt == BC_BF16) rc = run_ln<bf16, bf16>(x, rows, D, shift, scale, ld_mod, rows_per_sample, h, s);
    else rc = run_ln<bf16, float>(x, rows, D, shift, scale, ld_mod, rows_per_sample, h, s);
    prof_end(PROF_LAYERNORM, s);
    return rc;
}

// ---------------------------------------------------------------------------
// Skinny linear on MFMA.  A workgroup of 8 waves owns 16 rows of the batch
// (grid.y) and 16 TN output features; the waves deal the k-chunks among
// themselves (wave w takes chunks w, w + 8, ...) and meet in LDS once at the
// end, in a fixed order.  What bounds it is the one read of the weights, so
// enough of them have to be in flight: they go straight from memory to the
// MFMA's B operand, 16 bytes a lane, with U chunks of every tile issued before
// the first is used.  (A workgroup per 256 features with the whole of k behind
// two barriers left 27 to 72 workgroups: 33 us for DiT-XL/2's modulation, 79 us for
// the video model's.)  The activation is applied as the A operand is loaded.
// This form takes fp32 weights and k that is short or not whole 64-wide steps;
// the stream below it the rest.
// ---------------------------------------------------------------------------
template <typename T> struct SkMma;
template <> struct SkMma<bf16> {
    static constexpr int E = 8, KI = 32;      // elements per lane, k per chunk
    __device__ static f32x4 mma(const u32x4& a, const u32x4& b, const f32x4& c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    }
    __device__ static u32x4 pack(const float* v) {
        bf16x8 q;
#pragma unroll
        for (int i = 0; i < 8; ++i) q[i] = (bf16)v[i];
        return __builtin_bit_cast(u32x4, q);
    }
};
// fp32: lane group g of a chunk holds k = 4 g .. 4 g + 3, and instruction i
// takes element i of every lane; both operands permute k alike.
template <> struct SkMma<float> {
    static constexpr int E = 4, KI = 16;
    __device__ static f32x4 mma(const u32x4& a, const u32x4& b, f32x4 c) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a[i]), __uint_as_float(b[i]), c, 0, 0, 0);
        return c;
    }
    __device__ static u32x4 pack(const float* v) {
        return u32x4{__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]), __float_as_uint(v[3])};
    }
};

constexpr int kSkWaves = 8;
constexpr int kSkBatch = 4;   // chunks of weight loads issued together

template <typename T_, int TN>
__global__ __launch_bounds__(64 * kSkWaves) void skinny_kernel(SkinnyArgs a) {
    typedef elem_t<T_> T;
    typedef SkMma<T> MM;
    constexpr int E = MM::E, U = kSkBatch;
    __shared__ __attribute__((aligned(16))) f32x4 red[kSkWaves][TN][64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int r16 = lane & 15, kg = (lane >> 4) * E;
    const int n0 = blockIdx.x * 16 * TN, b0 = blockIdx.y * 16;
    const T* W = static_cast<const T*>(a.W);
    const T* wr[TN];
#pragma unroll
    for (int t = 0; t < TN; ++t) wr[t] = W + (int64_t)min(n0 + 16 * t + r16, a.N - 1) * a.K;
    const bool row_ok = b0 + r16 < a.B;
    const float* in = a.in + (int64_t)min(b0 + r16, a.B - 1) * a.ld_in;
    const bool vec = reinterpret_cast<uintptr_t>(a.in) % 16 == 0 && a.ld_in % 4 == 0;   // the caller's vectors may be unaligned
    f32x4 acc[TN];
#pragma unroll
    for (int t = 0; t < TN; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int nch = (a.K + MM::KI - 1) / MM::KI;
    for (int c0 = wave; c0 < nch; c0 += kSkWaves * U) {
        u32x4 wf[U][TN];
        float v[U][E];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = (c0 + u * kSkWaves) * MM::KI + kg;     // K % E == 0: a lane's piece is wholly in or out
            const bool ok = k < a.K;
#pragma unroll
            for (int t = 0; t < TN; ++t)
                wf[u][t] = ok ? *reinterpret_cast<const u32x4*>(wr[t] + k) : u32x4{0u, 0u, 0u, 0u};
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = (c0 + u * kSkWaves) * MM::KI + kg;
            if (row_ok && k < a.K) {
                if (vec) {
#pragma unroll
                    for (int i = 0; i < E; i += 4) {
                        const f32x4 x = *reinterpret_cast<const f32x4*>(in + k + i);
#pragma unroll
                        for (int e = 0; e < 4; ++e) v[u][i + e] = x[e];
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < E; ++i) v[u][i] = in[k + i];
                }
                if (a.act_in == 1) {
#pragma unroll
                    for (int i = 0; i < E; ++i) v[u][i] = silu(v[u][i]);
                }
            } else {
#pragma unroll
                for (int i = 0; i < E; ++i) v[u][i] = 0.f;
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const u32x4 af = MM::pack(v[u]);
#pragma unroll
            for (int t = 0; t < TN; ++t) acc[t] = MM::mma(af, wf[u][t], acc[t]);
        }
    }
#pragma unroll
    for (int t = 0; t < TN; ++t) red[wave][t][lane] = acc[t];
    __syncthreads();
    // Wave t finishes tile t: lane l holds rows 4 (l / 16) .. + 3 of column l % 16.
    if (wave >= TN) return;
    f32x4 sum = red[0][wave][lane];
#pragma unroll
    for (int w = 1; w < kSkWaves; ++w) sum += red[w][wave][lane];
    const int n = n0 + 16 * wave + r16;
    if (n >= a.N) return;
    const float bv = a.bias ? ld(static_cast<const T*>(a.bias) + n) : 0.f;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int b = b0 + 4 * (lane >> 4) + r;
        if (b >= a.B) continue;
        float v = sum[r] + bv;
        if (a.act_out == 1) v = silu(v);
        a.out[(int64_t)b * a.ld_out + n] = v;
    }
}

// The same for bf16 weights with whole 64-wide k-steps, as a stream: a
// workgroup takes column tile after column tile (16 features each), its waves
// every eighth k-step of all of them.  The activation of a wave's k-steps is
// worked out once, into registers; the weights pass through a ring of S stages
// that only this wave uses, 128 bytes of 16 rows a stage, S stages ahead across
// tile ends.  (Loaded straight into the MFMA operand, as above, 16 lanes fetch
// 16 bytes from 16 rows: a fraction of the rate of these loads.)  The partial
// tiles meet in LDS, one wave finishing each tile while the others go on.
// 18 432 x 3072 (the video model's modulation, 113 MB): 53 us with the loads
// straight into operands, 21 now (5.4 TB/s); 6912 x 1152 11.9 and 7.1.  One
// sample of 24 576 x 4096: 46.7 us with a ring that every step drained, 35.8 now
// (17 to 32 samples 92 and 75); up to k = 3072, where a CU holds two workgroups,
// the two rings cover each other and it made no difference.
// WGS: workgroups that a CU holds at once, which the launcher's grid counts on.
// Two where the activation (16 AST values a lane) leaves them 128 registers a
// wave; one at AST = 8, which takes 142 (with a grid of two there, 1 x 24 576 x
// 4096 took 35.8 us against 34.9, and with 20 samples 75 against 68).
template <int AST, int S, int WGS>
__global__ __launch_bounds__(64 * kSkWaves) __attribute__((amdgpu_waves_per_eu(2 * WGS))) void skinny_stream_kernel(
    SkinnyArgs a) {
    constexpr int STAGE = 16 * 128;
    __shared__ __attribute__((aligned(1024))) char ring[kSkWaves * S * STAGE];
    __shared__ __attribute__((aligned(16))) f32x4 red[2][kSkWaves][64];
    typedef __attribute__((address_space(3))) const char lds_char;
    typedef __attribute__((address_space(3))) const u32x4 lds_u32x4;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r16 = lane & 15, grp = lane >> 4, b0 = blockIdx.y * 16;
    const int tiles = a.N / 16, nk = a.K / 64;
    const int nt = (tiles - (int)blockIdx.x + (int)gridDim.x - 1) / (int)gridDim.x;    // this workgroup's tiles
    const int ns = nk > wave ? (nk - wave + kSkWaves - 1) / kSkWaves : 0;             // this wave's k-steps (at most AST)
    const int items = nt * ns;
    uint32_t off[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int r = 8 * q + (lane >> 3);
        off[q] = (uint32_t)r * (uint32_t)(a.K * 2) + ((lane & 7) ^ ((r >> 1) & 7)) * 16;
    }
    const uint32_t lds = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_char*)ring + wave * S * STAGE);
    // Item i is k-step wave + 8 (i % ns) of tile blockIdx.x + (i / ns) gridDim.x.
    int it = 0, is = 0;         // tile and step of the next item to load
    auto issue = [&](int stage) __attribute__((always_inline)) {
        const char* src = static_cast<const char*>(a.W) +
                          ((int64_t)(blockIdx.x + (int64_t)it * gridDim.x) * 16 * a.K + (int64_t)(wave + kSkWaves * is) * 64) * 2;
#pragma unroll
        for (int q = 0; q < 2; ++q) dma16s(src, off[q], lds + stage * STAGE + q * 1024);
        if (++is == ns) {
            is = 0;
            ++it;
        }
    };
    // The activation: row b0 + r16 of the batch (zero past the last), k = 64 step
    // + 32 kk + 8 grp ...  Its loads come back first, so that only the weights'
    // are outstanding while it is worked out.
    const bool row_ok = b0 + r16 < a.B;
    const float* in = a.in + (int64_t)min(b0 + r16, a.B - 1) * a.ld_in;
    const bool vec = reinterpret_cast<uintptr_t>(a.in) % 16 == 0 && a.ld_in % 4 == 0;   // the caller's vectors may be unaligned
    float v[AST][2][8];
#pragma unroll
    for (int j = 0; j < AST; ++j)
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            const int k = (wave + kSkWaves * j) * 64 + kk * 32 + grp * 8;
#pragma unroll
            for (int i = 0; i < 8; ++i) v[j][kk][i] = 0.f;
            if (row_ok && k < a.K) {
                if (vec) {
#pragma unroll
                    for (int i = 0; i < 8; i += 4) {
                        const f32x4 x = *reinterpret_cast<const f32x4*>(in + k + i);
#pragma unroll
                        for (int e = 0; e < 4; ++e) v[j][kk][i + e] = x[e];
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < 8; ++i) v[j][kk][i] = in[k + i];
                }
            }
        }
    wait_vmcnt<0>();
#pragma unroll
    for (int p = 0; p < S; ++p)
        if (p < items) issue(p);
    u32x4 af[AST][2];
#pragma unroll
    for (int j = 0; j < AST; ++j)
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            if (a.act_in == 1) {
                // SiLU with one native exp2 and reciprocal (rounded to bf16 next).
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    v[j][kk][i] *= __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * v[j][kk][i]));
            }
            af[j][kk] = SkMma<bf16>::pack(v[j][kk]);
        }
    lds_char* frag[2];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
        frag[kk] = (lds_char*)ring + wave * S * STAGE + r16 * 128 + ((kk * 4 + grp) ^ ((r16 >> 1) & 7)) * 16;
    int stage = 0, i = 0;
    for (int t = 0; t < nt; ++t) {
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < AST; ++j) {
            if (j < ns) {
                wait_groups<2, S - 1>(items - 1 - i);      // item i has landed
                asm volatile("" ::: "memory");
                u32x4 w[2];
#pragma unroll
                for (int kk = 0; kk < 2; ++kk) w[kk] = *(lds_u32x4*)(frag[kk] + stage * STAGE);
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");       // read before the stage is filled again
                if (i + S < items) issue(stage);
                stage = stage + 1 == S ? 0 : stage + 1;
                ++i;
#pragma unroll
                for (int kk = 0; kk < 2; ++kk) acc = SkMma<bf16>::mma(af[j][kk], w[kk], acc);
            }
        }
        // (Two sets of partial tiles: a wave may be one tile ahead of the one
        // that finishes, and the barrier of the next tile holds it there.)
        red[t & 1][wave][lane] = acc;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if (wave == t % kSkWaves) {
            f32x4 sum = red[t & 1][0][lane];
#pragma unroll
            for (int w = 1; w < kSkWaves; ++w) sum += red[t & 1][w][lane];
            const int n = (int)(blockIdx.x + (int64_t)t * gridDim.x) * 16 + r16;
            const float bv = a.bias ? ld(static_cast<const bf16*>(a.bias) + n) : 0.f;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int b = b0 + 4 * grp + r;
                if (b >= a.B) continue;
                float v = sum[r] + bv;
                if (a.act_out == 1) v = silu(v);
                a.out[(int64_t)b * a.ld_out + n] = v;
            }
        }
    }
}

template <typename T_>
static void run_skinny(const SkinnyArgs& a, hipStream_t s) {
    // Features per workgroup: as many tiles (up to four, so that the
    // activation is worked out fewer times) as leave a workgroup for every CU.
    const unsigned tiles = (unsigned)((a.N + 15) / 16), rows = (unsigned)((a.B + 15) / 16);
    const dim3 block(64 * kSkWaves);
    if (tiles * rows >= 4 * 256) skinny_kernel<T_, 4><<<dim3((tiles + 3) / 4, rows), block, 0, s>>>(a);
    else if (tiles * rows >= 2 * 256) skinny_kernel<T_, 2><<<dim3((tiles + 1) / 2, rows), block, 0, s>>>(a);
    else skinny_kernel<T_, 1><<<dim3(tiles, rows), block, 0, s>>>(a);
}

// One round of workgroups with equal shares of the column tiles.
template <int AST, int S, int WGS>
static void run_skinny_stream(const SkinnyArgs& a, hipStream_t s) {
    const int tiles = a.N / 16, per = (tiles + 256 * WGS - 1) / (256 * WGS);
    const dim3 grid((unsigned)((tiles + per - 1) / per), (unsigned)((a.B + 15) / 16)), block(64 * kSkWaves);
    skinny_stream_kernel<AST, S, WGS><<<grid, block, 0, s>>>(a);
}

int launch_skinny(int dt, const SkinnyArgs& a, hipStream_t s) {
    if (a.B <= 0) return BC_OK;
    if (a.B > 64) return fail(BC_ERR_UNSUPPORTED, "conditioning batch %d > 64", a.B);
    if (a.N % 16 || a.K % (dt == BC_BF16 ? 8 : 4)) return fail(BC_ERR_UNSUPPORTED, "skinny linear N=%d K=%d", a.N, a.K);
    if (!a.W || reinterpret_cast<uintptr_t>(a.W) % 16)
        return fail(BC_ERR_INVALID_ARG, "skinny linear weight missing or misaligned");
    if (dt == BC_BF16 && a.K % 64 == 0 && a.K >= 512 && a.K <= 4096) {
        if (a.K <= 1536) run_skinny_stream<3, 4, 2>(a, s);
        else if (a.K <= 3072) run_skinny_stream<6, 4, 2>(a, s);
        else run_skinny_stream<8, 4, 1>(a, s);
    } else if (dt == BC_BF16) {
        run_skinny<bf16_tag>(a, s);
    } else {
        run_skinny<float>(a, s);
    }
    return check_launch("skinny linear");
}

// ---------------------------------------------------------------------------
// Conditioning helpers
// ---------------------------------------------------------------------------
__global__ void step_sinusoid_kernel(int sampler, int S, int half, double shift, float* e) {
    const int k = blockIdx.y;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= half || k >= S) return;
    // Euler: 1000 sigma_k with the time shift (the device copy of flow_sigma).
    const double u = 1.0 - (double)k / S;
    const double sig = (shift == 0.0 || shift == 1.0) ? u : shift * u / (1.0 + (shift - 1.0) * u);
    const double t = sampler == BC_SAMPLER_EULER ? 1000.0 * sig : (double)(999 - (1000 * k) / S);
    const double f = exp(-log(10000.0) * (double)i / (double)half);
    const double ang = t * f;
    e[(int64_t)k * 2 * half + i] = (float)cos(ang);
    e[(int64_t)k * 2 * half + half + i] = (float)sin(ang);
}

int launch_step_sinusoid(int sampler, int S, int dim, double shift, float* e, hipStream_t s) {
    const int half = dim / 2;
    step_sinusoid_kernel<<<dim3((half + 127) / 128, S), 128, 0, s>>>(sampler, S, half, shift, e);
    return check_launch("sinusoid");
}

template <typename T_>
__global__ void build_cond_kernel(const float* temb, int S, int B, int D, const elem_t<T_>* table, const int64_t* labels,
                                  int n_rows, const float* add, float* c) {
    typedef elem_t<T_> T;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (int64_t)S * B * D) return;
    const int n = (int)(i % D);
    const int64_t kb = i / D;
    const int b = (int)(kb % B), k = (int)(kb / B);
    float v = temb[(int64_t)k * D + n];
    if (labels) {
        int64_t lab = labels[b];
        lab = lab < 0 ? 0 : (lab >= n_rows ? n_rows - 1 : lab);   // out-of-range labels are clamped
        v += ld(table + lab * D + n);
    } else if (add) {
        v += add[(int64_t)b * D + n];
    }
    c[i] = v;
}

int launch_build_cond(int dt, const float* temb, int S, int B, int D, const void* table, const int64_t* labels,
                      int n_rows, const float* add, float* c, hipStream_t s) {
    const int64_t n = (int64_t)S * B * D;
    const unsigned g = (unsigned)((n + 255) / 256);
    if (dt == BC_BF16) build_cond_kernel<bf16_tag><<<g, 256, 0, s>>>(temb, S, B, D, static_cast<const bf16*>(table), labels, n_rows, add, c);
    else build_cond_kernel<float><<<g, 256, 0, s>>>(temb, S, B, D, static_cast<const float*>(table), labels, n_rows, add, c);
    return check_launch("build_cond");
}

template <typename T_>
__global__ void gather_silu_kernel(const float* c, int B, int D, RowList rows, int n, elem_t<T_>* out) {
    typedef elem_t<T_> T;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (int64_t)n * B * D) return;
    const int d = (int)(i % D);
    const int64_t ib = i / D;
    const int b = (int)(ib % B), r = (int)(ib / B);
    st(out + i, silu(c[((int64_t)rows.row[r] * B + b) * D + d]));
}

int launch_gather_silu(int dt, const float* c, int B, int D, const RowList& rows, int n, void* out, hipStream_t s) {
    if (n <= 0) return BC_OK;
    if (n > kMaxSeg) return fail(BC_ERR_UNSUPPORTED, "gather of %d rows", n);
    const int64_t total = (int64_t)n * B * D;
    const unsigned g = (unsigned)((total + 255) / 256);
    if (dt == BC_BF16) gather_silu_kernel<bf16_tag><<<g, 256, 0, s>>>(c, B, D, rows, n, static_cast<bf16*>(out));
    else gather_silu_kernel<float><<<g, 256, 0, s>>>(c, B, D, rows, n, static_cast<float*>(out));
    return check_launch("gather_silu");
}

struct TableArgs { const void* tab[kMaxSeg]; };

template <typename T_>
__global__ void add_tables_kernel(const float* vec, int64_t ld_vec, TableArgs ta, int nseg, int N, int B, float* out,
                                  int64_t ld_out) {
    typedef elem_t<T_> T;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (int64_t)B * nseg * N) return;
    const int j = (int)(i % N);
    const int seg = (int)((i / N) % nseg);
    const int b = (int)(i / ((int64_t)N * nseg));
    out[(int64_t)b * ld_out + (int64_t)seg * N + j] = vec[(int64_t)b * ld_vec + j] + ld(static_cast<const T*>(ta.tab[seg]) + j);
}

int launch_add_tables(int dt, const float* vec, int64_t ld_vec, const void* const* tables, int nseg, int N, int B,
                      float* out, int64_t ld_out, hipStream_t s) {
    if (nseg > kMaxSeg) return fail(BC_ERR_UNSUPPORTED, "%d tables", nseg);
    TableArgs ta;
    for (int i = 0; i < nseg; ++i) ta.tab[i] = tables[i];
    const int64_t n = (int64_t)B * nseg * N;
    const unsigned g = (unsigned)((n + 255) / 256);
    if (dt == BC_BF16) add_tables_kernel<bf16_tag><<<g, 256, 0, s>>>(vec, ld_vec, ta, nseg, N, B, out, ld_out);
    else add_tables_kernel<float><<<g, 256, 0, s>>>(vec, ld_vec, ta, nseg, N, B, out, ld_out);
    return check_launch("add_tables");
}

template <typename E_>
__global__ void token_mean_kernel(const elem_t<E_>* x, int B, int T_, int D, float* out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (int64_t)B * D) return;
    const int b = (int)(i / D), n = (int)(i % D);
    float acc = 0.f;
    for (int t = 0; t < T_; ++t) acc += ld(x + ((int64_t)b * T_ + t) * D + n);
    out[i] = acc / (float)T_;
}

int launch_token_mean(int dt, const void* x, int B, int T, int D, float* out, hipStream_t s) {
    const int64_t n = (int64_t)B * D;
    const unsigned g = (unsigned)((n + 255) / 256);
    if (dt == BC_BF16) token_mean_kernel<bf16_tag><<<g, 256, 0, s>>>(static_cast<const bf16*>(x), B, T, D, out);
    else token_mean_kernel<float><<<g, 256, 0, s>>>(static_cast<const float*>(x), B, T, D, out);
    return check_launch("token_mean");
}

template <typename Tin_, typename Tout_>
__global__ void convert_kernel(const elem_t<Tin_>* in, elem_t<Tout_>* out, int64_t n) {
    typedef elem_t<Tin_> Tin;
    typedef elem_t<Tout_> Tout;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        st(out + i, ld(in + i));
}

int launch_convert(int in_dt, const void* in, int out_dt, void* out, int64_t n, hipStream_t s) {
    if (n <= 0) return BC_OK;
    int64_t blocks = (n + 255) / 256;
    if (blocks > 16384) blocks = 16384;
    const unsigned g = (unsigned)blocks;
    if (in_dt == BC_F32 && out_dt == BC_BF16) convert_kernel<float, bf16_tag><<<g, 256, 0, s>>>(static_cast<const float*>(in), static_cast<bf16*>(out), n);
    else if (in_dt == BC_BF16 && out_dt == BC_F32) convert_kernel<bf16_tag, float><<<g, 256, 0, s>>>(static_cast<const bf16*>(in), static_cast<float*>(out), n);
    else return launch_copy(in, out, n * dtype_size(in_dt), s);
    return check_launch("convert");
}

// ---------------------------------------------------------------------------
// Patch embedding and the final layer
// ---------------------------------------------------------------------------
// One workgroup per token: gather its p*p*C patch values once (LDS), then
// each thread produces output features of the row.
template <typename T_, int kPatchRows>
__global__ __launch_bounds__(256) void patch_embed_kernel(const float* __restrict__ lat, LatentShape ls,
                                                          const elem_t<T_>* __restrict__ W, const elem_t<T_>* __restrict__ bias,
                                                          const elem_t<T_>* __restrict__ pos, int D, int lat_B, int rows,
                                                          float* __restrict__ x) {
    typedef elem_t<T_> T;
    // kPatchRows tokens per workgroup: each thread reads its columns' weight
    // rows once for all of them (the weights are [D, p*p*C], one row per
    // output column), and each output still sums its patch in order q = 0, 1, ...
    // Large patches (the video model's 64 values) take 16 tokens per
    // workgroup; small ones one, which keeps enough workgroups in flight.
    __shared__ float patch[kPatchRows][kMaxPatch];
    const int Tn = ls.tokens();
    const int row0 = blockIdx.x * kPatchRows;
    const int hp = ls.H / ls.p, wp = ls.W / ls.p;
    const int PD = ls.p * ls.p * ls.C;
    for (int i = threadIdx.x; i < kPatchRows * PD; i += blockDim.x) {
        const int r = i / PD, q = i - r * PD, row = row0 + r;
        float v = 0.f;
        if (row < rows) {
            const int bm = row / Tn, tok = row - bm * Tn;
            const int b = bm % lat_B;
            const int f = tok / (hp * wp), ti = (tok / wp) % hp, tj = tok % wp;
            const int ph = q / (ls.p * ls.C), pw = (q / ls.C) % ls.p, ch = q % ls.C;
            v = lat[((((int64_t)b * ls.C + ch) * ls.F + f) * ls.H + ti * ls.p + ph) * ls.W + tj * ls.p + pw];
        }
        patch[r][q] = v;
    }
    __syncthreads();
    for (int c = threadIdx.x; c < D; c += blockDim.x) {
        const T* wr = W + (int64_t)c * PD;
        float acc[kPatchRows];
#pragma unroll
        for (int r = 0; r < kPatchRows; ++r) acc[r] = 0.f;
        for (int q = 0; q < PD; ++q) {
            const float w = ld(wr + q);
#pragma unroll
            for (int r = 0; r < kPatchRows; ++r) acc[r] = __builtin_fmaf(patch[r][q], w, acc[r]);
        }
        const float bc = ld(bias + c);
#pragma unroll
        for (int r = 0; r < kPatchRows; ++r) {
            const int row = row0 + r;
            if (row < rows) {
                const int tok = row % Tn;
                x[(int64_t)row * D + c] = acc[r] + bc + ld(pos + (int64_t)tok * D + c);
            }
        }
    }
}

int launch_patch_embed(int dt, const float* lat, LatentShape ls, int B, int lat_B, const void* W, const void* bias,
                       const void* pos, int D, float* x, hipStream_t s) {
    if (ls.p * ls.p * ls.C > kMaxPatch) return fail(BC_ERR_UNSUPPORTED, "patch of %d values", ls.p * ls.p * ls.C);
    if (lat_B < 1 || lat_B > B) return fail(BC_ERR_INVALID_ARG, "latent batch %d for a model batch of %d", lat_B, B);
    const int rows = B * ls.tokens();
    if (rows <= 0) return BC_OK;
    auto go = [&](auto tpb) {
        constexpr int TPB = decltype(tpb)::value;
        const unsigned grid = (unsigned)((rows + TPB - 1) / TPB);
        if (dt == BC_BF16)
            patch_embed_kernel<bf16_tag, TPB><<<grid, 256, 0, s>>>(lat, ls, static_cast<const bf16*>(W),
                                                               static_cast<const bf16*>(bias),
                                                               static_cast<const bf16*>(pos), D, lat_B, rows, x);
        else
            patch_embed_kernel<float, TPB><<<grid, 256, 0, s>>>(lat, ls, static_cast<const float*>(W),
                                                                static_cast<const float*>(bias),
                                                                static_cast<const float*>(pos), D, lat_B, rows, x);
    };
    if (ls.p * ls.p * ls.C >= 32) go(std::integral_constant<int, 16>{});
    else go(std::integral_constant<int, 1>{});
    return check_launch("patch_embed");
}

__global__ void cfg_labels_kernel(const int64_t* labels, int B, int64_t null_id, int64_t* out) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < B) out[i] = labels[i];
    else if (i < 2 * B) out[i] = null_id;
}

int launch_cfg_labels(const int64_t* labels, int B, int64_t null_id, int64_t* out, hipStream_t s) {
    cfg_labels_kernel<<<1, 128, 0, s>>>(labels, B, null_id, out);
    return check_launch("cfg_labels");
}

// ---------------------------------------------------------------------------
// Sampler update
// ---------------------------------------------------------------------------
// Model output arrives in token layout [B*T, p*p*C_out] (the final linear's
// output); element (b, c, f, y, x) of the latent is read from token
// (f, y/p, x/p), feature ((y%p)*p + x%p)*C_out + c, which is unpatchify.
__global__ void sampler_kernel(SamplerCoef k, float* x, const float* out_tok, float* prev, LatentShape ls, int B,
                               int C_out, float cfg, int64_t uncond_off) {
    const int64_t S = (int64_t)ls.F * ls.H * ls.W;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (int64_t)B * ls.C * S) return;
    const int xs = (int)(i % ls.W);
    const int ys = (int)((i / ls.W) % ls.H);
    const int f = (int)((i / ((int64_t)ls.W * ls.H)) % ls.F);
    const int64_t bc = i / S;
    const int c = (int)(bc % ls.C), b = (int)(bc / ls.C);
    const int hp = ls.H / ls.p, wp = ls.W / ls.p;
    const int tok = (f * hp + ys / ls.p) * wp + xs / ls.p;
    const int feat = ((ys % ls.p) * ls.p + xs % ls.p) * C_out + c;
    const int64_t o = ((int64_t)b * ls.tokens() + tok) * (ls.p * ls.p * C_out) + feat;
    float e = out_tok[o];
    if (uncond_off > 0) {
        const float u = out_tok[o + uncond_off];
        e = __builtin_fmaf(cfg, e - u, u);
    }
    sampler_update(k, x + i, e, prev ? prev + i : nullptr);
}

int launch_sampler(const SamplerCoef& k, float* x, const float* out_tok, float* prev, LatentShape ls, int B, int C_out,
                   hipStream_t s, float cfg, int64_t uncond_off) {
    const int64_t n = (int64_t)B * ls.C * ls.F * ls.H * ls.W;
    sampler_kernel<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(k, x, out_tok, prev, ls, B, C_out, cfg, uncond_off);
    return check_launch("sampler");
}

// ---------------------------------------------------------------------------
// QK RMSNorm + 3D rotary embedding: one wave per (row, head, q|k); lane i
// holds the pair (2i, 2i + 1) of the head, so the rotation is lane-local and
// the RMS is one wave reduction.
// ---------------------------------------------------------------------------
template <typename T_>
__global__ __launch_bounds__(256) void qk_norm_rope_kernel(elem_t<T_>* __restrict__ qkv, int64_t rows, int64_t ldr, int D,
                                                           int heads, int hd, const elem_t<T_>* __restrict__ wq,
                                                           const elem_t<T_>* __restrict__ wk, int L, int n_img, int gf,
                                                           int gh, int gw, float log2_theta, float q_scale) {
    typedef elem_t<T_> T;
    const int64_t wid = ((int64_t)blockIdx.x * 256 + threadIdx.x) >> 6;
    const int lane = threadIdx.x & 63;
    if (wid >= rows * heads * 2) return;   // whole waves
    const int qk = (int)(wid & 1);
    const int64_t rh = wid >> 1;
    const int h = (int)(rh % heads);
    const int64_t r = rh / heads;
    T* p = qkv + r * ldr + (int64_t)qk * D + (int64_t)h * hd;
    const bool act = 2 * lane < hd;
    float x0 = 0.f, x1 = 0.f;
    if (act) {
        x0 = ld(p + 2 * lane);
        x1 = ld(p + 2 * lane + 1);
    }
    const T* w = qk ? wk : wq;
    if (w) {
        float ss = x0 * x0 + x1 * x1;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o);
        const float inv = 1.0f / sqrtf(ss / (float)hd + 1e-6f);
        if (act) {
            x0 = x0 * inv * ld(w + 2 * lane);
            x1 = x1 * inv * ld(w + 2 * lane + 1);
        }
    }
    const int t = (int)(r % L);
    if (log2_theta > 0.f && t < n_img && act) {
        const int d_f = hd / 8, d_h = (hd - d_f) / 2, d_w = hd - d_f - d_h;
        const int e = 2 * lane;
        const int col = t % gw, row = (t / gw) % gh, fr = t / (gw * gh);
        int pos, j, da;
        if (e < d_f) { pos = fr; j = e / 2; da = d_f; }
        else if (e < d_f + d_h) { pos = row; j = (e - d_f) / 2; da = d_h; }
        else { pos = col; j = (e - d_f - d_h) / 2; da = d_w; }
        const float freq = exp2f(-(float)(2 * j) / (float)da * log2_theta);
        float sn, cs;
        sincosf((float)pos * freq, &sn, &cs);
        const float y0 = x0 * cs - x1 * sn, y1 = x0 * sn + x1 * cs;
        x0 = y0;
        x1 = y1;
    }
    if (act) {
        const float os = qk ? 1.f : q_scale;
        p[2 * lane] = (T)(x0 * os);
        p[2 * lane + 1] = (T)(x1 * os);
    }
}

// bf16 variant for head_dim = 8 * CPH with CPH a power of two (64, 128): one
// wave per (row, q|k) walks the row in 16-byte chunks, lane l taking chunks
// l, l + 64, ...  Since 64 is a multiple of CPH, lane l always holds the same
// four pairs (chunk l % CPH) of whichever head a chunk belongs to: it loads its
// eight norm scales and works out its four rotations once per row.  A head's
// RMS is a reduction over the CPH lanes that hold it.
template <int CPH, typename B_>
__global__ __launch_bounds__(256) void qk_norm_rope_row_kernel(elem_t<B_>* __restrict__ qkv, int64_t rows, int64_t ldr,
                                                               int D, const elem_t<B_>* __restrict__ wq,
                                                               const elem_t<B_>* __restrict__ wk, int L, int n_img, int gf,
                                                               int gh, int gw, float log2_theta, float q_scale) {
    constexpr int HD = 8 * CPH;
    const int64_t wid = ((int64_t)blockIdx.x * 256 + threadIdx.x) >> 6;
    const int lane = threadIdx.x & 63;
    if (wid >= rows * 2) return;   // whole waves
    const int qk = (int)(wid & 1);
    const int64_t r = wid >> 1;
    bf16* p = qkv + r * ldr + (int64_t)qk * D;
    const int nch = D / 8;
    const int e0 = (lane % CPH) * 8;   // first element of this lane's chunk within its head
    const bf16* w = qk ? wk : wq;
    float wv[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) wv[k] = w ? ld(w + e0 + k) : 1.f;
    const int t = (int)(r % L);
    const bool rot = log2_theta > 0.f && t < n_img;
    float cs[4], sn[4];
    if (rot) {
        constexpr int d_f = HD / 8, d_h = (HD - d_f) / 2, d_w = HD - d_f - d_h;
        const int col = t % gw, row = (t / gw) % gh, fr = t / (gw * gh);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int e = e0 + 2 * q;
            int pos, j, da;
            if (e < d_f) { pos = fr; j = e / 2; da = d_f; }
            else if (e < d_f + d_h) { pos = row; j = (e - d_f) / 2; da = d_h; }
            else { pos = col; j = (e - d_f - d_h) / 2; da = d_w; }
            const float freq = exp2f(-(float)(2 * j) / (float)da * log2_theta);
            sincosf((float)pos * freq, &sn[q], &cs[q]);
        }
    }
    for (int c0 = 0; c0 < nch; c0 += 64) {
        const int c = c0 + lane;
        const bool act = c < nch;
        u32x4 u = u32x4{0u, 0u, 0u, 0u};
        if (act) u = *reinterpret_cast<const u32x4*>(p + (int64_t)c * 8);
        float v[8];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            v[2 * k] = __uint_as_float(u[k] << 16);
            v[2 * k + 1] = __uint_as_float(u[k] & 0xffff0000u);
        }
        if (w) {
            float ss = 0.f;
#pragma unroll
            for (int k = 0; k < 8; ++k) ss += v[k] * v[k];
#pragma unroll
            for (int o = 1; o < CPH; o <<= 1) ss += __shfl_xor(ss, o);
            const float inv = 1.0f / sqrtf(ss / (float)HD + 1e-6f);
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = v[k] * inv * wv[k];
        }
        if (rot) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float y0 = v[2 * q] * cs[q] - v[2 * q + 1] * sn[q];
                const float y1 = v[2 * q] * sn[q] + v[2 * q + 1] * cs[q];
                v[2 * q] = y0;
                v[2 * q + 1] = y1;
            }
        }
        if (act) {
            const float os = qk ? 1.f : q_scale;
            u32x4 o;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const bf16 lo = (bf16)(v[2 * k] * os), hi = (bf16)(v[2 * k + 1] * os);
                o[k] = (uint32_t)__builtin_bit_cast(uint16_t, lo) | ((uint32_t)__builtin_bit_cast(uint16_t, hi) << 16);
            }
            *reinterpret_cast<u32x4*>(p + (int64_t)c * 8) = o;
        }
    }
}

int launch_qk_norm_rope(int dt, void* qkv, int64_t rows, int64_t ld, int D, int heads, int head_dim, const void* wq,
                        const void* wk, int rows_per_sample, int n_img, int gf, int gh, int gw, double theta,
                        float q_scale, hipStream_t s) {
    const bool rope = theta > 0.0 && n_img > 0;
    if (!wq && !wk && !rope && q_scale == 1.f) return BC_OK;
    if (head_dim < 2 || head_dim > 128 || head_dim % 2 || heads * head_dim != D || rows_per_sample < 1 ||
        (rope && (head_dim % 32 || (int64_t)gf * gh * gw != n_img)))
        return fail(BC_ERR_INVALID_ARG, "qk_norm_rope: head_dim %d, grid %d x %d x %d for %d tokens", head_dim, gf, gh,
                    gw, n_img);
    const int64_t waves = rows * heads * 2;
    if (waves < 1) return BC_OK;
    const float l2t = rope ? (float)std::log2(theta) : 0.f;
    const bool aligned = reinterpret_cast<uintptr_t>(qkv) % 16 == 0 && ld % 8 == 0 && D % 8 == 0;
    if (dt == BC_BF16 && aligned && (head_dim == 128 || head_dim == 64)) {
        const unsigned gr = (unsigned)((rows * 2 + 3) / 4);
        bf16* q = static_cast<bf16*>(qkv);
        const bf16 *a = static_cast<const bf16*>(wq), *b = static_cast<const bf16*>(wk);
        const int ni = rope ? n_img : 0;
        if (head_dim == 128)
            qk_norm_rope_row_kernel<16, bf16_tag><<<gr, 256, 0, s>>>(q, rows, ld, D, a, b, rows_per_sample, ni, gf, gh, gw, l2t, q_scale);
        else
            qk_norm_rope_row_kernel<8, bf16_tag><<<gr, 256, 0, s>>>(q, rows, ld, D, a, b, rows_per_sample, ni, gf, gh, gw, l2t, q_scale);
        return check_launch("qk_norm_rope_row");
    }
    const unsigned g = (unsigned)((waves + 3) / 4);
    if (dt == BC_BF16)
        qk_norm_rope_kernel<bf16_tag><<<g, 256, 0, s>>>(static_cast<bf16*>(qkv), rows, ld, D, heads, head_dim,
                                                    static_cast<const bf16*>(wq), static_cast<const bf16*>(wk),
                                                    rows_per_sample, rope ? n_img : 0, gf, gh, gw, l2t, q_scale);
    else
        qk_norm_rope_kernel<float><<<g, 256, 0, s>>>(static_cast<float*>(qkv), rows, ld, D, heads, head_dim,
                                                     static_cast<const float*>(wq), static_cast<const float*>(wk),
                                                     rows_per_sample, rope ? n_img : 0, gf, gh, gw, l2t, q_scale);
    return check_launch("qk_norm_rope");
}

// ---------------------------------------------------------------------------
// Blockwise mode: gated adds of module outputs into the fp32 residual stream,
// 8 consecutive elements per thread (16-byte loads of the bf16 sites).
// ---------------------------------------------------------------------------
__device__ __forceinline__ void load8(const bf16* p, float* v) {
    const u32x4 u = *reinterpret_cast<const u32x4*>(p);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        v[2 * k] = __uint_as_float(u[k] << 16);
        v[2 * k + 1] = __uint_as_float(u[k] & 0xffff0000u);
    }
}
__device__ __forceinline__ void load8(const float* p, float* v) {
    const f32x4 a = *reinterpret_cast<const f32x4*>(p), b = *reinterpret_cast<const f32x4*>(p + 4);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        v[k] = a[k];
        v[4 + k] = b[k];
    }
}

template <typename T_>
__global__ __launch_bounds__(256) void gated_add_kernel(const elem_t<T_>* __restrict__ site, int64_t n8, int D,
                                                        float* __restrict__ x, const float* __restrict__ gate,
                                                        int64_t ldg, int rows_per_gate) {
    typedef elem_t<T_> T;
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n8) return;
    const int64_t e = i * 8, r = e / D;
    const int d = (int)(e - r * D);
    float v[8], xv[8], g[8];
    load8(site + e, v);
    load8(x + e, xv);
    if (gate) load8(gate + (r / rows_per_gate) * ldg + d, g);
    else {
#pragma unroll
        for (int k = 0; k < 8; ++k) g[k] = 1.f;
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) xv[k] = fmaf(g[k], v[k], xv[k]);
    *reinterpret_cast<f32x4*>(x + e) = f32x4{xv[0], xv[1], xv[2], xv[3]};
    *reinterpret_cast<f32x4*>(x + e + 4) = f32x4{xv[4], xv[5], xv[6], xv[7]};
}

int launch_gated_add(int dt, const void* site, int64_t rows, int D, float* x, const float* gate, int64_t ldg,
                     int rows_per_gate, hipStream_t s) {
    if (D % 8 || reinterpret_cast<uintptr_t>(site) % 16 || reinterpret_cast<uintptr_t>(x) % 16 ||
        (gate && (reinterpret_cast<uintptr_t>(gate) % 16 || ldg % 4)) || rows_per_gate < 1)
        return fail(BC_ERR_INVALID_ARG, "gated_add: D %d, alignment", D);
    const int64_t n8 = rows * D / 8;
    if (n8 < 1) return BC_OK;
    const unsigned g = (unsigned)((n8 + 255) / 256);
    if (dt == BC_BF16) gated_add_kernel<bf16_tag><<<g, 256, 0, s>>>(static_cast<const bf16*>(site), n8, D, x, gate, ldg, rows_per_gate);
    else gated_add_kernel<float><<<g, 256, 0, s>>>(static_cast<const float*>(site), n8, D, x, gate, ldg, rows_per_gate);
    return check_launch("gated_add");
}

template <typename T_>
__global__ __launch_bounds__(256) void blockwise_forecast_kernel(BlockwiseArgs a) {
    typedef elem_t<T_> T;
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i * 8 >= a.numel) return;
    const int64_t e = i * 8, r = e / a.D;
    const int d = (int)(e - r * a.D);
    const T* st = static_cast<const T*>(a.storage);
    const float* mrow = a.mods + (r / a.rows_per_gate) * a.ldm + d;
    float xv[8];
    load8(a.x + e, xv);
    for (int s = 0; s < a.nsites; ++s) {
        float f[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        for (int j = 0; j < a.count; ++j) {
            float v[8];
            load8(st + ((int64_t)s * a.K + a.slot[j]) * a.numel + e, v);
#pragma unroll
            for (int k = 0; k < 8; ++k) f[k] = fmaf(a.w[j], v[k], f[k]);
        }
        float g[8];
        if (a.goff[s] >= 0) load8(mrow + a.goff[s], g);
        else {
#pragma unroll
            for (int k = 0; k < 8; ++k) g[k] = 1.f;
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) xv[k] = fmaf(g[k], f[k], xv[k]);
    }
    *reinterpret_cast<f32x4*>(a.x + e) = f32x4{xv[0], xv[1], xv[2], xv[3]};
    *reinterpret_cast<f32x4*>(a.x + e + 4) = f32x4{xv[4], xv[5], xv[6], xv[7]};
}

int launch_blockwise_forecast(int dt, const BlockwiseArgs& a, hipStream_t s) {
    if (a.D % 8 || a.numel % 8 || a.nsites < 1 || a.nsites > kMaxSites || a.count < 1 || a.count > a.K ||
        a.K > kMaxK || a.ldm % 4 || reinterpret_cast<uintptr_t>(a.storage) % 16 ||
        reinterpret_cast<uintptr_t>(a.x) % 16 || reinterpret_cast<uintptr_t>(a.mods) % 16)
        return fail(BC_ERR_INVALID_ARG, "blockwise forecast: %d sites, count %d of %d", a.nsites, a.count, a.K);
    for (int j = 0; j < a.count; ++j)
        if (a.slot[j] < 0 || a.slot[j] >= a.K) return fail(BC_ERR_INVALID_ARG, "blockwise forecast: slot %d", a.slot[j]);
    for (int q = 0; q < a.nsites; ++q)
        if (a.goff[q] >= 0 && a.goff[q] % 4)   // (negative: no gate)
            return fail(BC_ERR_INVALID_ARG, "blockwise forecast: gate offset %d", a.goff[q]);
    const int64_t n8 = a.numel / 8;
    const unsigned g = (unsigned)((n8 + 255) / 256);
    if (dt == BC_BF16) blockwise_forecast_kernel<bf16_tag><<<g, 256, 0, s>>>(a);
    else blockwise_forecast_kernel<float><<<g, 256, 0, s>>>(a);
    return check_launch("blockwise_forecast");
}

// ---------------------------------------------------------------------------
// Relative L1 change of the adaptive schedule's probe: 16-byte chunks of cur
// and prev, |cur - prev| and |prev| summed per thread, per wave (butterfly)
// and per workgroup in a fixed order; prev takes cur's bytes in the same pass.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void abs_sums(const u32x4& c, const u32x4& p, float& sd, float& sp, bf16*) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float cl = __uint_as_float(c[i] << 16), ch = __uint_as_float(c[i] & 0xffff0000u);
        const float pl = __uint_as_float(p[i] << 16), ph = __uint_as_float(p[i] & 0xffff0000u);
        sd += fabsf(cl - pl) + fabsf(ch - ph);
        sp += fabsf(pl) + fabsf(ph);
    }
}
__device__ __forceinline__ void abs_sums(const u32x4& c, const u32x4& p, float& sd, float& sp, float*) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float cf = __uint_as_float(c[i]), pf = __uint_as_float(p[i]);
        sd += fabsf(cf - pf);
        sp += fabsf(pf);
    }
}

template <typename T_>
__global__ __launch_bounds__(256) void rel_l1_kernel(const elem_t<T_>* __restrict__ cur, elem_t<T_>* __restrict__ prev, int64_t n,
                                                     float* __restrict__ part) {
    typedef elem_t<T_> T;
    constexpr int E = 16 / (int)sizeof(T);
    const int64_t nc = n / E;
    const u32x4* c4 = reinterpret_cast<const u32x4*>(cur);
    u32x4* p4 = reinterpret_cast<u32x4*>(prev);
    float sd = 0.f, sp = 0.f;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < nc; i += (int64_t)gridDim.x * 256) {
        const u32x4 c = c4[i], p = p4[i];
        abs_sums(c, p, sd, sp, (T*)nullptr);
        p4[i] = c;
    }
    if (blockIdx.x == 0) {
        for (int64_t i = nc * E + threadIdx.x; i < n; i += 256) {
            const float c = ld(cur + i), p = ld(prev + i);
            sd += fabsf(c - p);
            sp += fabsf(p);
            prev[i] = cur[i];
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        sd += __shfl_xor(sd, o);
        sp += __shfl_xor(sp, o);
    }
    __shared__ float red[2][4];
    const int wv = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        red[0][wv] = sd;
        red[1][wv] = sp;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        const float* r = red[threadIdx.x];
        part[2 * blockIdx.x + threadIdx.x] = ((r[0] + r[1]) + r[2]) + r[3];
    }
}

__global__ __launch_bounds__(256) void rel_l1_sum_kernel(const float* __restrict__ part, int nblk,
                                                         double* __restrict__ sums) {
    __shared__ double ra[256], rb[256];
    const int t = threadIdx.x;
    double a = 0.0, b = 0.0;
    for (int i = t; i < nblk; i += 256) {
        a += (double)part[2 * i];
        b += (double)part[2 * i + 1];
    }
    ra[t] = a;
    rb[t] = b;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if (t < h) {
            ra[t] += ra[t + h];
            rb[t] += rb[t + h];
        }
        __syncthreads();
    }
    if (t < 2) sums[t] = t == 0 ? ra[0] : rb[0];
}

int launch_rel_l1(int dt, const void* cur, void* prev, int64_t n, float* part, double* sums, hipStream_t s) {
    if (n < 1) return fail(BC_ERR_INVALID_ARG, "rel_l1: n=%lld", (long long)n);
    if (reinterpret_cast<uintptr_t>(cur) % 16 || reinterpret_cast<uintptr_t>(prev) % 16)
        return fail(BC_ERR_INVALID_ARG, "rel_l1: buffers must be 16-byte aligned");
    const int64_t nc = n / (16 / (int64_t)dtype_size(dt));
    const int nblk = (int)std::min<int64_t>(kRelL1Blocks, std::max<int64_t>(1, (nc + 1023) / 1024));
    if (dt == BC_BF16)
        rel_l1_kernel<bf16_tag><<<nblk, 256, 0, s>>>(static_cast<const bf16*>(cur), static_cast<bf16*>(prev), n, part);
    else
        rel_l1_kernel<float><<<nblk, 256, 0, s>>>(static_cast<const float*>(cur), static_cast<float*>(prev), n, part);
    const int rc = check_launch("rel_l1");
    if (rc != BC_OK) return rc;
    rel_l1_sum_kernel<<<1, 256, 0, s>>>(part, nblk, sums);
    return check_launch("rel_l1_sum");
}

}  // namespace bc
