// Multi-head attention softmax(Q K^T / sqrt(d)) V, flash style (online
// softmax, no T x T buffer), on MFMA.
//
// A workgroup owns 64*QG queries of one (sample, head); each of its 4 waves
// owns QG groups of 16 and keeps their Q fragments in registers.  Keys and values
// stream through LDS 64 at a time (K row-major, V transposed).  The wave
// computes the transposed scores S^T = K Q^T, so after the MFMA a lane holds
// 16 scores of a single query (its lane index mod 16).  That makes the
// softmax statistics per-lane values (plus two cross-lane reductions), and the
// probabilities are already laid out as the B operand of O^T = V^T P^T, whose
// accumulator again holds one query per lane: rescaling O by the running-max
// correction is one multiply per register.  Scores, max, sum and O are fp32.
//
// Rows of Q, K, V and O may come from two segments (the image and text
// streams of joint attention): position p of sample b is row b*T0 + p of
// segment 0 if p < T0, else row b*T1 + (p - T0) of segment 1.  Head h of a row
// is the d consecutive elements starting at column h*d.
#include <cmath>
#include <type_traits>
#include "attention.h"

namespace bc {

constexpr int kAttnThreads = 256;
constexpr int kKTile = 64;   // keys per step

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

template <typename T, int HD> struct AttnShape {
    // K dimension of Q K^T: bf16 uses 32-wide MFMA steps, the last one padded
    // with zero Q columns (a 16-wide 16x16x16 tail step was dropped: in one
    // schedule its accumulator was read back before the MFMA had written
    // it); fp32 uses 4-wide steps.
    static constexpr int n32x = sizeof(T) == 2 ? (HD + 31) / 32 : 0;   // 32-wide steps
    static constexpr int DK = sizeof(T) == 2 ? 32 * n32x : HD;
    static constexpr int DV = (HD + 15) / 16 * 16;           // rows of O^T
    static constexpr int EPC = 16 / (int)sizeof(T);          // elements per 16-byte chunk
    static constexpr int CPR = HD / EPC;                     // chunks per head row
    static constexpr int KPAD = EPC;                         // LDS row padding (elements)
};

template <typename T>
__device__ __forceinline__ const T* seg_row(const void* p0, const void* p1, int T0, int T1, int64_t ld,
                                            int b, int p) {
    return p < T0 ? static_cast<const T*>(p0) + ((int64_t)b * T0 + p) * ld
                  : static_cast<const T*>(p1) + ((int64_t)b * T1 + (p - T0)) * ld;
}

// QG groups of 16 queries per wave (64 * QG per workgroup): every K and V
// fragment read from LDS feeds QG MFMAs.
template <typename T, int HD, int QG>
__global__ __launch_bounds__(kAttnThreads) void attention_kernel(AttnArgs a) {
    typedef AttnShape<T, HD> S;
    constexpr int QT = 64 * QG;                  // queries per workgroup
    constexpr int LDK = S::DK + S::KPAD;
    constexpr int LDV = kKTile + S::KPAD;
    __shared__ __attribute__((aligned(16))) T sK[kKTile][LDK];
    __shared__ __attribute__((aligned(16))) T sVt[S::DV][LDV];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int Tq = a.Tq0 + a.Tq1, Tk = a.Tk0 + a.Tk1;
    // Workgroup order: consecutive ids go round-robin to the 8 XCDs; remap so
    // each XCD holds a contiguous range, i.e. all query tiles of a (sample,
    // head) share one L2 and its keys and values are fetched once per XCD.
    const int nqt = (Tq + QT - 1) / QT;
    const int nwg = gridDim.x;
    const int pid = xcd_contiguous(blockIdx.x, nwg);
    const int qt = pid % nqt;
    const int h = (pid / nqt) % a.H;
    const int b = pid / (nqt * a.H);
    const int col0 = h * HD;
    const int ql = lane & 15, grp = lane >> 4;

    // Zero the padding columns of K and the padding rows of V^T once.
    for (int i = tid; i < kKTile * (LDK - HD); i += kAttnThreads)
        sK[i / (LDK - HD)][HD + i % (LDK - HD)] = (T)0.f;
    for (int i = tid; i < (S::DV - HD) * LDV; i += kAttnThreads)
        sVt[HD + i / LDV][i % LDV] = (T)0.f;

    // Q fragments (B operand of S^T = K Q^T): in group g, lane holds query
    // qt*QT + wave*16*QG + 16g + ql.
    bf16x8 qf[QG][S::n32x > 0 ? S::n32x : 1];
    float qf32[QG][sizeof(T) == 4 ? HD / 4 : 1];
    int myq[QG];
#pragma unroll
    for (int g = 0; g < QG; ++g) {
        myq[g] = qt * QT + wave * 16 * QG + 16 * g + ql;
        const T* qrow = myq[g] < Tq ? seg_row<T>(a.q0, a.q1, a.Tq0, a.Tq1, a.ldq, b, myq[g]) + col0 : nullptr;
        if constexpr (sizeof(T) == 2) {
#pragma unroll
            for (int c = 0; c < S::n32x; ++c)
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const int d = 32 * c + grp * 8 + i;
                    qf[g][c][i] = (qrow && d < HD) ? (bf16)qrow[d] : (bf16)0.f;
                }
        } else {
#pragma unroll
            for (int c = 0; c < HD / 4; ++c) qf32[g][c] = qrow ? (float)qrow[4 * c + grp] : 0.f;
        }
    }

    f32x4 o[QG][S::DV / 16];
    float m_run[QG], l_run[QG];
#pragma unroll
    for (int g = 0; g < QG; ++g) {
        m_run[g] = -INFINITY;
        l_run[g] = 0.f;
#pragma unroll
        for (int i = 0; i < S::DV / 16; ++i) o[g][i] = f32x4{0.f, 0.f, 0.f, 0.f};
    }

    // Staging of one K/V tile (64 keys x CPR 16-byte chunks).  K chunks are
    // assigned row-major (coalesced global reads, 16-byte LDS stores); V chunks
    // key-major, so a wave's transposed 2-byte LDS stores cover 64 consecutive
    // keys of one row of V^T.
    constexpr int NCH = kKTile * S::CPR;
    constexpr int PER = (NCH + kAttnThreads - 1) / kAttnThreads;
    u32x4 rk[PER], rv[PER];
    auto load_tile = [&](int k0) {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int c = tid + i * kAttnThreads;
            rk[i] = u32x4{0, 0, 0, 0};
            rv[i] = u32x4{0, 0, 0, 0};
            if (c < NCH) {
                const int krow = c / S::CPR, kch = c % S::CPR;
                if (k0 + krow < Tk)
                    rk[i] = *reinterpret_cast<const u32x4*>(
                        seg_row<T>(a.k0, a.k1, a.Tk0, a.Tk1, a.ldk, b, k0 + krow) + col0 + kch * S::EPC);
                const int vrow = c % kKTile, vch = c / kKTile;
                if (k0 + vrow < Tk)
                    rv[i] = *reinterpret_cast<const u32x4*>(
                        seg_row<T>(a.v0, a.v1, a.Tk0, a.Tk1, a.ldv, b, k0 + vrow) + col0 + vch * S::EPC);
            }
        }
    };
    auto store_tile = [&]() {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int c = tid + i * kAttnThreads;
            if (c < NCH) {
                *reinterpret_cast<u32x4*>(&sK[c / S::CPR][(c % S::CPR) * S::EPC]) = rk[i];
                const int vrow = c % kKTile, vch = c / kKTile;
                if constexpr (sizeof(T) == 2) {
                    const uint32_t w4[4] = {rv[i].x, rv[i].y, rv[i].z, rv[i].w};
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        sVt[vch * 8 + 2 * e][vrow] = __builtin_bit_cast(bf16, (unsigned short)(w4[e] & 0xffffu));
                        sVt[vch * 8 + 2 * e + 1][vrow] = __builtin_bit_cast(bf16, (unsigned short)(w4[e] >> 16));
                    }
                } else {
                    sVt[vch * 4 + 0][vrow] = __uint_as_float(rv[i].x);
                    sVt[vch * 4 + 1][vrow] = __uint_as_float(rv[i].y);
                    sVt[vch * 4 + 2][vrow] = __uint_as_float(rv[i].z);
                    sVt[vch * 4 + 3][vrow] = __uint_as_float(rv[i].w);
                }
            }
        }
    };

    const int ntiles = (Tk + kKTile - 1) / kKTile;
    load_tile(0);
    __syncthreads();   // padding zeroed before the first tile lands
    store_tile();
    __syncthreads();

    for (int t = 0; t < ntiles; ++t) {
        const int k0 = t * kKTile;
        if (t + 1 < ntiles) load_tile(k0 + kKTile);

        // S^T tiles: s[g][j] covers keys k0 + 16j .. +16; lane holds keys
        // 16j + 4grp + r of its query in group g.
        f32x4 s[QG][4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
#pragma unroll
            for (int g = 0; g < QG; ++g) s[g][j] = f32x4{0.f, 0.f, 0.f, 0.f};
            const int krow = 16 * j + ql;
            if constexpr (sizeof(T) == 2) {
#pragma unroll
                for (int c = 0; c < S::n32x; ++c) {
                    const bf16x8 kf = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(&sK[krow][32 * c + grp * 8]));
#pragma unroll
                    for (int g = 0; g < QG; ++g) s[g][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf, qf[g][c], s[g][j], 0, 0, 0);
                }
            } else {
#pragma unroll
                for (int c = 0; c < HD / 4; ++c) {
                    const float kv = (float)sK[krow][4 * c + grp];
#pragma unroll
                    for (int g = 0; g < QG; ++g) s[g][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(kv, qf32[g][c], s[g][j], 0, 0, 0);
                }
            }
        }

        // Online softmax (base 2, scores pre-scaled by log2(e)/sqrt(d)).
#pragma unroll
        for (int g = 0; g < QG; ++g) {
            float mloc = -INFINITY;
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int key = k0 + 16 * j + 4 * grp + r;
                    const float v = key < Tk ? s[g][j][r] * a.scale_log2 : -INFINITY;
                    s[g][j][r] = v;
                    mloc = fmaxf(mloc, v);
                }
            mloc = fmaxf(mloc, __shfl_xor(mloc, 16, 64));
            mloc = fmaxf(mloc, __shfl_xor(mloc, 32, 64));
            const float m_new = fmaxf(m_run[g], mloc);
            const float alpha = exp2f(m_run[g] - m_new);
            float lsum = 0.f;
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float p = exp2f(s[g][j][r] - m_new);
                    s[g][j][r] = p;
                    lsum += p;
                }
            lsum += __shfl_xor(lsum, 16, 64);
            lsum += __shfl_xor(lsum, 32, 64);
            l_run[g] = l_run[g] * alpha + lsum;
            m_run[g] = m_new;
#pragma unroll
            for (int i = 0; i < S::DV / 16; ++i) o[g][i] *= alpha;
        }

        // O^T += V^T P^T.
        if constexpr (sizeof(T) == 2) {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                bf16x8 pf[QG];
#pragma unroll
                for (int g = 0; g < QG; ++g)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        pf[g][r] = (bf16)s[g][2 * u][r];
                        pf[g][4 + r] = (bf16)s[g][2 * u + 1][r];
                    }
#pragma unroll
                for (int i = 0; i < S::DV / 16; ++i) {
                    // keys 32u + 4grp + 0..3 and 32u + 16 + 4grp + 0..3, matching pf
                    const T* vrow = &sVt[16 * i + ql][32 * u + 4 * grp];
                    const u32x2 lo = *reinterpret_cast<const u32x2*>(vrow);
                    const u32x2 hi = *reinterpret_cast<const u32x2*>(vrow + 16);
                    const bf16x8 vf = __builtin_bit_cast(bf16x8, u32x4{lo.x, lo.y, hi.x, hi.y});
#pragma unroll
                    for (int g = 0; g < QG; ++g) o[g][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, pf[g], o[g][i], 0, 0, 0);
                }
            }
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int i = 0; i < S::DV / 16; ++i) {
                        const float vv = (float)sVt[16 * i + ql][16 * j + 4 * grp + r];
#pragma unroll
                        for (int g = 0; g < QG; ++g) o[g][i] = __builtin_amdgcn_mfma_f32_16x16x4f32(vv, s[g][j][r], o[g][i], 0, 0, 0);
                    }
        }

        __syncthreads();
        if (t + 1 < ntiles) {
            store_tile();
            __syncthreads();
        }
    }

#pragma unroll
    for (int g = 0; g < QG; ++g) {
        if (myq[g] < Tq) {
            const float inv = 1.f / l_run[g];
            T* orow = const_cast<T*>(seg_row<T>(a.o0, a.o1, a.Tq0, a.Tq1, a.ldo, b, myq[g])) + col0;
#pragma unroll
            for (int i = 0; i < S::DV / 16; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int d = 16 * i + 4 * grp + r;
                    if (d < HD) st(orow + d, o[g][i][r] * inv);
                }
        }
    }
}

// ---------------------------------------------------------------------------
// bf16 kernel with direct-to-LDS K/V tiles.
//
// K and V tiles are both kept row-major (key rows, head_dim contiguous) and
// stream HBM -> LDS with global_load_lds_dwordx4 (no register staging), double
// buffered with one barrier per 64-key step.  The V^T operand of O^T = V^T P^T
// is read with ds_read_b64_tr_b16: within a 16-lane group, lane L receives
// element L % 4 of the 8-byte reads of lanes L/4 + 4i (i = 0..3), so if lane s
// reads V[k0 + s/4][d0 + 4 (s % 4)], lane L gets V[k0 + i][d0 + L], i = 0..3:
// four consecutive keys of one head-dim column, the operand layout.  Rows of
// 128 or 256 bytes are XOR-swizzled by 16-byte chunk so the 16-row fragment
// reads hit distinct banks (a 144-byte row of d = 72 already does).
// ---------------------------------------------------------------------------
template <int HD> struct KvLayout {
    static constexpr int CPR = HD / 8;                       // 16-byte chunks per row
    static constexpr int RPB = (HD * 2) >= 256 ? 1 : 256 / (HD * 2);   // rows per 256 bytes
    static constexpr bool SWZ = (CPR & (CPR - 1)) == 0;      // power-of-two rows are swizzled
    __device__ static int slot(int row, int chunk) { return SWZ ? chunk ^ ((row / RPB) % CPR) : chunk; }
    // element offset of (row, column d) in a tile
    __device__ static int at(int row, int d) { return row * HD + slot(row, d >> 3) * 8 + (d & 7); }
};

// NWV waves of 16 QG queries each per workgroup; NB K/V tile buffers.  STREAM
// false: all key tiles fit in the NB buffers (the launcher sees to it); they
// are loaded once, up front, and the key loop runs without further barriers.
// STREAM: the NB = 2 buffers are a double buffer.
// Reductions over the four lanes l, l ^ 16, l ^ 32, l ^ 48 that hold one
// query's scores: with both operands equal, v_permlane16_swap returns the
// value of lane l in one result and of lane l ^ 16 in the other (likewise
// v_permlane32_swap for l ^ 32), so no LDS round trip is needed.
// Maximum without the NaN-quieting canonicalisation that fmaxf's IEEE
// semantics add per operand (gfx950 has a native three-input form); scores
// are finite or -inf.
__device__ __forceinline__ float vmax(float a, float b) { return __builtin_elementwise_maximum(a, b); }
__device__ __forceinline__ float group_max(float v) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = vmax(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return vmax(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float group_sum(float v) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// The QKV projection of one (sample, head) for the fused kernel below: the
// sample's T <= 256 rows of x times the head's q, k and v rows of W_qkv (3 HD
// of them, padded to whole 16-row MFMA blocks with repeats of the last), plus
// the bias, with the q columns times q_scale, rounded to bf16 -- the same
// operands, k order, MFMA and roundings as the separate QKV GEMM when its
// tiles keep K in one wave group (DiT-XL/2's 4096 rows), so there the same
// bits.  64-wide k-steps through two LDS stages of direct-to-LDS loads, in the
// phases of the large GEMM tiles: the stage's 256 rows of x are two halves, its
// weight rows two parts, each loaded again for the step after the next as soon as
// every wave has read it, and the next pair's fragments are read under the
// present one's MFMAs; 8 waves as 4 x 2.  (One burst of loads and one barrier a
// step: 47.2 us against 43.5 for the whole kernel at DiT-XL/2's 16 x 256 tokens.)
// The results go to LDS in the attention's layouts: Q row-major [256, HD],
// K and V as the four 64-key tiles.  Rows past T repeat row T - 1 (finite;
// their keys are masked and their queries not stored).
template <int HD, int TILE>
__device__ __forceinline__ void qkv_head_to_lds(const AttnArgs& a, int b, int h, bf16* smem, bf16 (*sK)[TILE],
                                                bf16 (*sV)[TILE], bf16* sQ) {
    typedef KvLayout<HD> LY;
    typedef __attribute__((address_space(3))) const char lds_char;
    typedef __attribute__((address_space(3))) const u32x4 lds_u32x4;
    constexpr int WAVES_N = 2, TM = 2;                     // 4 x 2 waves; 16-row blocks of a wave in one half
    constexpr int NBLK = (3 * HD + 15) / 16, TN = NBLK / WAVES_N;   // 16-row blocks of the weights (the last padded)
    static_assert(NBLK % WAVES_N == 0, "column blocks per wave");
    constexpr int TN0 = (TN + 1) / 2, TN1 = TN / 2;        // a wave's blocks in the two weight parts
    constexpr int ABYTES = 128 * 128, W0BYTES = 32 * TN0 * 128, W1BYTES = 32 * TN1 * 128;
    constexpr int W0AT = 4 * ABYTES, W1AT = W0AT + 2 * W0BYTES;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WAVES_N, wn = wave % WAVES_N;
    const int frow = lane & 15, grp = lane >> 4;
    const int T = a.Tk0, D = a.dmodel;
    const char* x = reinterpret_cast<const char*>(static_cast<const bf16*>(a.x) + (int64_t)b * T * a.ldx);
    const char* W = static_cast<const char*>(a.w_qkv);
    // Wave-wide loads of 8 rows: wave w takes loads w and w + 8 of every half and
    // part; a part has 4 TN0 or 4 TN1 of them, so waves 4-7 may make one fewer.
    constexpr int N0 = (4 * TN0 + 7) / 8, N1 = (4 * TN1 + 7) / 8;                 // by waves 0-3
    constexpr int M0 = 4 * TN0 / 8, M1 = 4 * TN1 / 8;                             // by waves 4-7
    static_assert(4 * TN0 - 8 * M0 <= 4 && 4 * TN1 - 8 * M1 <= 4, "loads per wave");
    const bool low = wave < 4;
    uint32_t offA[2][2], off0[N0], off1[N1];
    auto chunk_of = [&](int r) __attribute__((always_inline)) { return (uint32_t)((lane & 7) ^ ((r >> 1) & 7)) * 16; };
    auto weight_row = [&](int r) __attribute__((always_inline)) {
        const int rr = min(r, 3 * HD - 1), sec = rr / HD;
        return (uint32_t)(sec * D + h * HD + (rr - sec * HD)) * (uint32_t)(D * 2);
    };
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int r = 64 * q + 8 * wave + (lane >> 3);
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) offA[hf][q] = (uint32_t)min(128 * hf + r, T - 1) * (uint32_t)(a.ldx * 2) + chunk_of(r);
        if (q < N0) off0[q] = weight_row(r) + chunk_of(r);
        if (q < N1) off1[q] = weight_row(32 * TN0 + r) + chunk_of(r);
    }
    const uint32_t ldsw = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_char*)smem + wave * 1024);
    auto loadA = [&](int hf, int par, int k) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < 2; ++q) dma16s(x + (int64_t)k * 128, offA[hf][q], ldsw + (2 * hf + par) * ABYTES + q * 8192);
    };
    auto loadW0 = [&](int par, int k) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < N0; ++q)
            if (q < M0 || low) dma16s(W + (int64_t)k * 128, off0[q], ldsw + W0AT + par * W0BYTES + q * 8192);
    };
    auto loadW1 = [&](int par, int k) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < N1; ++q)
            if (q < M1 || low) dma16s(W + (int64_t)k * 128, off1[q], ldsw + W1AT + par * W1BYTES + q * 8192);
    };
    // Waits until at most A halves', B first parts' and C second parts' loads,
    // issued after the ones needed, are outstanding.
    auto wait = [&](auto ac, auto bc, auto cc) __attribute__((always_inline)) {
        constexpr int A = decltype(ac)::value, B = decltype(bc)::value, C = decltype(cc)::value;
        if (low) wait_vmcnt<2 * A + N0 * B + N1 * C>();
        else wait_vmcnt<2 * A + M0 * B + M1 * C>();
    };
#define QP_WAIT(A, B, C) wait(std::integral_constant<int, A>{}, std::integral_constant<int, B>{}, std::integral_constant<int, C>{})
    lds_char *pA[2], *pW0[2], *pW1[2];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
        const uint32_t c = (uint32_t)((kk * 4 + grp) ^ ((frow >> 1) & 7)) * 16;
        pA[kk] = (lds_char*)smem + (wm * 32 + frow) * 128 + c;
        pW0[kk] = (lds_char*)smem + W0AT + (wn * 16 * TN0 + frow) * 128 + c;
        pW1[kk] = (lds_char*)smem + W1AT + (wn * 16 * TN1 + frow) * 128 + c;
    }
    u32x4 fa[2][TM][2], fw[2][TN0][2];     // [half][block][kk]; [register set][block][kk]
    auto readA = [&](int hf, int par) __attribute__((always_inline)) {
#pragma unroll
        for (int kk = 0; kk < 2; ++kk)
#pragma unroll
            for (int i = 0; i < TM; ++i) fa[hf][i][kk] = *(lds_u32x4*)(pA[kk] + (2 * hf + par) * ABYTES + i * 2048);
    };
    auto readW0 = [&](int par, int set) __attribute__((always_inline)) {
#pragma unroll
        for (int kk = 0; kk < 2; ++kk)
#pragma unroll
            for (int j = 0; j < TN0; ++j) fw[set][j][kk] = *(lds_u32x4*)(pW0[kk] + par * W0BYTES + j * 2048);
    };
    auto readW1 = [&](int par, int set) __attribute__((always_inline)) {
#pragma unroll
        for (int kk = 0; kk < 2; ++kk)
#pragma unroll
            for (int j = 0; j < TN1; ++j) fw[set][j][kk] = *(lds_u32x4*)(pW1[kk] + par * W1BYTES + j * 2048);
    };
    f32x4 acc[2][TM][TN];      // blocks j < TN0 of the first part, the rest of the second
#pragma unroll
    for (int hf = 0; hf < 2; ++hf)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[hf][i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto mma = [&](int hf, auto partc, int set) __attribute__((always_inline)) {
        constexpr int P = decltype(partc)::value;
#pragma unroll
        for (int kk = 0; kk < 2; ++kk)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < (P ? TN1 : TN0); ++j)
                    acc[hf][i][P * TN0 + j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                        __builtin_bit_cast(bf16x8, fw[set][j][kk]), __builtin_bit_cast(bf16x8, fa[hf][i][kk]), acc[hf][i][P * TN0 + j], 0, 0, 0);
    };
    auto barrier = [&]() __attribute__((always_inline)) {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    auto reads_done = [&]() __attribute__((always_inline)) { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); };
    // A phase's order: its NR fragment reads, each ahead of one MFMA (two reads where there are fewer MFMAs), then the other MFMAs.
#define QP_ORDER(NR, NM) do { constexpr int RPM = (NR + NM - 1) / NM; \
        _Pragma("unroll") for (int z = 0; z < NR; z += RPM) { __builtin_amdgcn_sched_group_barrier(0x100, RPM, 0); __builtin_amdgcn_sched_group_barrier(0x008, 1, 0); } \
        __builtin_amdgcn_sched_group_barrier(0x008, NM - (NR + RPM - 1) / RPM, 0); __builtin_amdgcn_sched_barrier(0); } while (0)
    typedef std::integral_constant<int, 0> C0;
    typedef std::integral_constant<int, 1> C1;
    typedef std::integral_constant<int, 2> C2;
    const int nk = D / 64;
    // One k-step on the buffers of parity PAR (also the register set of its first
    // weight part): x0 W0, x0 W1, x1 W1, x1 W0.  MODE 0: the loads of step k + 2
    // go out; 1: the last step but one; 2: the last.
    auto step = [&](int k, auto parc, auto modec) __attribute__((always_inline)) {
        constexpr int PAR = decltype(parc)::value, MODE = decltype(modec)::value;
        if (MODE == 0) loadA(0, PAR, k + 2);
        readW1(PAR, PAR ^ 1);
        mma(0, C0{}, PAR);
        QP_ORDER(2 * TN1, 2 * TM * TN0);
        if (MODE == 0) QP_WAIT(3, 1, 1); else if (MODE == 1) QP_WAIT(2, 1, 1); else QP_WAIT(0, 0, 0);
        barrier();
        if (MODE == 0) loadW0(PAR, k + 2);
        readA(1, PAR);
        mma(0, C1{}, PAR ^ 1);
        QP_ORDER(2 * TM, 2 * TM * TN1);
        barrier();
        if (MODE == 0) loadW1(PAR, k + 2);
        mma(1, C1{}, PAR ^ 1);
        if (MODE == 2) {
            mma(1, C0{}, PAR);
            return;
        }
        __builtin_amdgcn_sched_barrier(0);
        if (MODE == 0) QP_WAIT(2, 1, 2); else QP_WAIT(1, 0, 1);
        barrier();
        if (MODE == 0) loadA(1, PAR, k + 2);
        readW0(PAR ^ 1, PAR ^ 1);
        readA(0, PAR ^ 1);
        mma(1, C0{}, PAR);
        QP_ORDER(2 * (TN0 + TM), 2 * TM * TN0);
        if (MODE == 0) QP_WAIT(3, 1, 1); else QP_WAIT(1, 0, 0);
        reads_done();
        barrier();
    };
    auto first = [&](auto parc) __attribute__((always_inline)) {
        constexpr int PAR = decltype(parc)::value;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            loadA(0, PAR ^ k, k);
            loadW0(PAR ^ k, k);
            loadW1(PAR ^ k, k);
            loadA(1, PAR ^ k, k);
        }
        QP_WAIT(3, 1, 1);
        barrier();
        readA(0, PAR);
        readW0(PAR, PAR);
        reads_done();
        barrier();
    };
    const int odd = nk & 1;      // an odd number of steps starts on the odd buffers
    if (odd) {
        first(C1{});
        step(0, C1{}, C0{});
    } else {
        first(C0{});
    }
    int k = odd;
    for (; k + 2 < nk; k += 2) {
        step(k, C0{}, C0{});
        step(k + 1, C1{}, C0{});
    }
    step(k, C0{}, C1{});
    step(k + 1, C1{}, C2{});
#undef QP_WAIT
#undef QP_ORDER
    __syncthreads();   // every wave is done with the stages, which Q, K and V now overwrite
    // A lane holds four consecutive columns of one row per block.
    const bf16* bias = static_cast<const bf16*>(a.b_qkv);
    const float qs = a.proj_q_scale;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int col = (j < TN0 ? wn * 16 * TN0 + j * 16 : 32 * TN0 + wn * 16 * TN1 + (j - TN0) * 16) + 4 * grp;
        if (col >= 3 * HD) continue;
        const int sec = col / HD, e = col - sec * HD;   // HD % 4 == 0: the four columns share a section
        float bv[4] = {0.f, 0.f, 0.f, 0.f};
        if (bias) {
            const bf16x4 b4 = *reinterpret_cast<const bf16x4*>(bias + (int64_t)sec * D + h * HD + e);
#pragma unroll
            for (int r = 0; r < 4; ++r) bv[r] = (float)b4[r];
        }
        const float sc = sec == 0 ? qs : 1.f;
#pragma unroll
        for (int hf = 0; hf < 2; ++hf)
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const int row = 128 * hf + wm * 32 + i * 16 + frow;
                bf16x4 q;
#pragma unroll
                for (int r = 0; r < 4; ++r) q[r] = (bf16)((acc[hf][i][j][r] + bv[r]) * sc);
                bf16* dst = sec == 0 ? sQ + row * HD + e
                                     : (sec == 1 ? sK[row / 64] : sV[row / 64]) + LY::at(row % 64, e);
                *reinterpret_cast<bf16x4*>(dst) = q;
            }
    }
    // The slack past each tile's last row is read (for d >= HD operand rows,
    // whose outputs are discarded): keep it finite.
    if (tid < 32) {
#pragma unroll
        for (int nb = 0; nb < 4; ++nb) {
            sK[nb][kKTile * HD + tid] = (bf16)0.f;
            sV[nb][kKTile * HD + tid] = (bf16)0.f;
        }
    }
    __syncthreads();
}

// Four-wave workgroups are held to two waves per SIMD (256 registers), so two
// workgroups share a CU and their barriers do not line up.
// QKV: the block's QKV projection for this (sample, head) runs first, into
// LDS (qkv_head_to_lds), and the attention reads Q, K and V from there: one
// workgroup per (sample, head) of up to 256 tokens.
template <int HD, int QG, int NWV, int NB, bool STREAM, bool QS, bool QKV = false>
__global__ __launch_bounds__(64 * NWV) __attribute__((amdgpu_waves_per_eu(NWV == 4 ? 2 : 1))) void attention_dma_kernel(
    AttnArgs a) {
    static_assert(!QKV || (!STREAM && QS && QG == 2 && NWV == 8 && NB == 4 && HD <= 72), "fused QKV shape");
    typedef AttnShape<bf16, HD> S;
    typedef KvLayout<HD> LY;
    constexpr int QT = 16 * QG * NWV;
    static_assert(NB >= 2, "buffers");
    constexpr int TILE = kKTile * HD + 32;     // elements per K or V tile (+ slack for d >= HD operand reads)
    // The softmax row sums come from the MFMAs, as P times a V column of
    // ones (no per-score adds): when HD is not a multiple of 16 the padding
    // rows of the last output block carry them (the deferred rescale of O
    // covers them); otherwise one more 16-row block of ones, osum.
    constexpr bool PADSUM = HD % 16 != 0;
    // QKV: one buffer holds the projection's stages, then K, V and Q.
    constexpr int QKV_ELEMS = QKV ? (2 * (256 + (3 * HD + 15) / 16 * 16) * 64 > 2 * NB * TILE + 256 * HD
                                         ? 2 * (256 + (3 * HD + 15) / 16 * 16) * 64
                                         : 2 * NB * TILE + 256 * HD)
                                  : 8;
    __shared__ __attribute__((aligned(1024))) bf16 sK_[QKV ? 8 : NB * TILE];
    __shared__ __attribute__((aligned(1024))) bf16 sV_[QKV ? 8 : NB * TILE];
    __shared__ __attribute__((aligned(1024))) bf16 sX_[QKV_ELEMS];
    typedef bf16 TileArr[TILE];
    TileArr* sK = reinterpret_cast<TileArr*>(QKV ? sX_ : sK_);
    TileArr* sV = reinterpret_cast<TileArr*>(QKV ? sX_ + NB * TILE : sV_);
    bf16* sQ = sX_ + 2 * NB * TILE;     // QKV only

    // The small resident grids are one chain of latencies: all the arguments in
    // one round of scalar loads (3 x 65 x 256 at d = 128: 8.4 us without, 8.2 with).
    if constexpr (!STREAM && !QKV && NWV == 4) {
        const unsigned nblk = gridDim.x;
        asm volatile("" : : "s"(nblk), "s"(a.Tq0), "s"(a.Tk0), "s"(a.k0), "s"(a.k1), "s"(a.v0), "s"(a.v1), "s"(a.ldk),
                     "s"(a.ldv), "s"(a.q0), "s"(a.ldq), "s"(a.H), "s"(a.o0), "s"(a.ldo), "s"(a.scale_log2));
    }
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int Tq = a.Tq0 + a.Tq1, Tk = a.Tk0 + a.Tk1;
    const int nqt = (Tq + QT - 1) / QT;
    const int nwg = gridDim.x;
    const int pid = xcd_contiguous(blockIdx.x, nwg);
    const int qt = pid % nqt;
    const int h = (pid / nqt) % a.H;
    const int b = pid / (nqt * a.H);
    const int col0 = h * HD;
    const int ql = lane & 15, grp = lane >> 4;

    // The slack past the last row is read (for d >= HD operand rows, whose
    // outputs are discarded) but never loaded: keep it finite.  (QKV: written
    // after the projection, whose stages share the buffer.)
    if constexpr (QKV) qkv_head_to_lds<HD, TILE>(a, b, h, sX_, sK, sV, sQ);
    else if (tid < 32) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            sK[nb][kKTile * HD + tid] = (bf16)0.f;
            sV[nb][kKTile * HD + tid] = (bf16)0.f;
        }
    }

    // One tile = 64 keys x CPR chunks = CPR wave-wide DMA instructions per
    // operand; wave w issues instructions w, w + 4, ...  Lane L of instruction j
    // fills LDS chunk 64 j + L = (row, slot) and fetches the global chunk that
    // belongs there.  Keys past the end are clamped to the last key (finite
    // data; their scores are masked).
    // This wave's instructions and its lane's (row, chunk) in each are fixed:
    // worked out once, so a tile's issue only offsets the key.
    constexpr int NJ = (LY::CPR + NWV - 1) / NWV;
    // (row, global column) of this lane's chunk in instruction q, recomputed
    // where needed rather than held in registers.
    auto irow = [&](int q) { return (64 * (wave + NWV * q) + lane) / LY::CPR; };
    auto icol = [&](int q) {
        const int c = 64 * (wave + NWV * q) + lane;
        const int row = c / LY::CPR, slot = c % LY::CPR;
        return col0 + 8 * (LY::SWZ ? slot ^ ((row / LY::RPB) % LY::CPR) : slot);
    };
    // With four query groups per wave the value offsets are derived from the
    // key offsets (one register per instruction fewer).
    constexpr bool VFROMK = QG >= 4;
    // STREAM (the instantiations for long key sequences, whose tiles stream
    // through the buffers): a tile that lies wholly inside one key segment
    // is addressed from one row pointer, common to the workgroup, plus each
    // lane's fixed offset (when offsets within a tile fit 32 bits).  The tile
    // that crosses the segment boundary or runs past the last key, and every
    // tile of the other instantiations, take the per-row path.
    const bool off32 = STREAM && (int64_t)kKTile * (a.ldk > a.ldv ? a.ldk : a.ldv) < ((int64_t)1 << 31);
    int koff[NJ], voff[VFROMK ? 1 : NJ];
    if constexpr (STREAM) {
#pragma unroll
        for (int q = 0; q < NJ; ++q) {
            koff[q] = (int)(irow(q) * a.ldk + icol(q));     // used only when off32
            if constexpr (!VFROMK) voff[q] = (int)(irow(q) * a.ldv + icol(q));
        }
    }
    auto issue_rows = [&](int k0, int buf) {
#pragma unroll
        for (int q = 0; q < NJ; ++q) {
            const int j = wave + NWV * q;
            if (j >= LY::CPR) break;
            const int key = min(k0 + irow(q), Tk - 1);
            const int ic = icol(q);
            const bf16* kr = seg_row<bf16>(a.k0, a.k1, a.Tk0, a.Tk1, a.ldk, b, key) + ic;
            const bf16* vr = seg_row<bf16>(a.v0, a.v1, a.Tk0, a.Tk1, a.ldv, b, key) + ic;
            dma16(kr, &sK[buf][64 * j * 8]);
            dma16(vr, &sV[buf][64 * j * 8]);
        }
    };
    auto issue = [&](int k0, int buf) {
        if constexpr (!STREAM) {
            issue_rows(k0, buf);
            return;
        }
        const bf16 *kb = nullptr, *vb = nullptr;
        if (off32 && k0 + kKTile <= a.Tk0) {
            kb = static_cast<const bf16*>(a.k0) + ((int64_t)b * a.Tk0 + k0) * a.ldk;
            vb = static_cast<const bf16*>(a.v0) + ((int64_t)b * a.Tk0 + k0) * a.ldv;
        } else if (off32 && k0 >= a.Tk0 && k0 + kKTile <= Tk) {
            kb = static_cast<const bf16*>(a.k1) + ((int64_t)b * a.Tk1 + (k0 - a.Tk0)) * a.ldk;
            vb = static_cast<const bf16*>(a.v1) + ((int64_t)b * a.Tk1 + (k0 - a.Tk0)) * a.ldv;
        }
        if (kb) {
#pragma unroll
            for (int q = 0; q < NJ; ++q) {
                const int j = wave + NWV * q;
                if (j >= LY::CPR) break;
                dma16(kb + koff[q], &sK[buf][64 * j * 8]);
                dma16(vb + (VFROMK ? koff[q] + irow(q) * (int)(a.ldv - a.ldk) : voff[VFROMK ? 0 : q]), &sV[buf][64 * j * 8]);
            }
        } else {
            issue_rows(k0, buf);
        }
    };
    const int ntiles = (Tk + kKTile - 1) / kKTile;
    // K/V loads go out first so that their latency overlaps the Q loads.
    if constexpr (QKV) {
        // (K and V are in LDS already.)
    } else if (!STREAM) {
        for (int t = 0; t < ntiles; ++t) issue_rows(t * kKTile, t);
    } else {
        issue(0, 0);
    }

    bf16x8 qf[QG][S::n32x > 0 ? S::n32x : 1];
    int myq[QG];
#pragma unroll
    for (int g = 0; g < QG; ++g) {
        myq[g] = qt * QT + wave * 16 * QG + 16 * g + ql;
        const bf16* qrow = QKV ? sQ + myq[g] * HD
                         : myq[g] < Tq ? seg_row<bf16>(a.q0, a.q1, a.Tq0, a.Tq1, a.ldq, b, myq[g]) + col0 : nullptr;
#pragma unroll
        for (int c = 0; c < S::n32x; ++c) {
            const int d = 32 * c + grp * 8;       // HD % 8 == 0: a chunk is wholly in or out
            qf[g][c] = (qrow && d < HD) ? __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(qrow + d))
                                        : __builtin_bit_cast(bf16x8, u32x4{0u, 0u, 0u, 0u});
        }
    }

    f32x4 o[QG][S::DV / 16], osum[QG];
    float m_run[QG];
    const bool o8 = (a.ldo & 3) == 0 && ((reinterpret_cast<uintptr_t>(a.o0) | reinterpret_cast<uintptr_t>(a.o1)) & 7) == 0;
#pragma unroll
    for (int g = 0; g < QG; ++g) {
        m_run[g] = STREAM ? 0.f : -INFINITY;     // the streaming tile's reference is set by its first tile
        osum[g] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < S::DV / 16; ++i) o[g][i] = f32x4{0.f, 0.f, 0.f, 0.f};
    }


    // Operand addresses: per-lane byte offsets within a tile, worked out once.
    // A row's swizzle depends only on the row mod 16, so the fragments 16 and
    // 32 rows further on sit at constant distances, and with the buffer fixed
    // at compile time every read is a lane offset plus an immediate.
    typedef __attribute__((address_space(3))) const char lds_char;
    uint32_t kofs[S::n32x], vofs[S::DV / 16];
#pragma unroll
    for (int c = 0; c < S::n32x; ++c) kofs[c] = 2u * (uint32_t)LY::at(ql, 32 * c + grp * 8);
#pragma unroll
    for (int i = 0; i < S::DV / 16; ++i) vofs[i] = 2u * (uint32_t)LY::at(4 * grp + (ql >> 2), 16 * i + 4 * (ql & 3));
    constexpr uint32_t ROWB = 2u * HD;    // bytes per tile row
    // O^T += V^T P^T for one tile's probabilities (and the row sums, see
    // above) from the V tile at Vb.
    auto pv = [&](lds_char* Vb, f32x4 (&s)[QG][4]) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            bf16x8 pf[QG];
#pragma unroll
            for (int g = 0; g < QG; ++g)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    pf[g][r] = (bf16)s[g][2 * u][r];
                    pf[g][4 + r] = (bf16)s[g][2 * u + 1][r];
                }
#pragma unroll
            for (int i = 0; i < S::DV / 16; ++i) {
                lds_char* p = Vb + vofs[i] + 32u * u * ROWB;
                const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)p);
                const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(p + 16 * ROWB));
                bf16x8 vf = __builtin_bit_cast(bf16x8, u32x4{__builtin_bit_cast(u32x2, lo).x, __builtin_bit_cast(u32x2, lo).y,
                                                            __builtin_bit_cast(u32x2, hi).x, __builtin_bit_cast(u32x2, hi).y});
                // Padding rows d >= HD of the last block take ones: their
                // output rows become the row sums of P (as rounded for the MFMA).
                if (PADSUM && i == S::DV / 16 - 1 && (lane & 15) >= HD - 16 * i)
                    vf = __builtin_bit_cast(bf16x8, u32x4{0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u});
#pragma unroll
                for (int g = 0; g < QG; ++g) o[g][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, pf[g], o[g][i], 0, 0, 0);
            }
            if constexpr (!PADSUM) {
                const bf16x8 ones = __builtin_bit_cast(bf16x8, u32x4{0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u});
#pragma unroll
                for (int g = 0; g < QG; ++g) osum[g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, pf[g], osum[g], 0, 0, 0);
            }
        }
    };

    // Scores, online softmax and the P V update of one resident 64-key tile at
    // k0 (scores times c in one FMA with the max; c is 1 for pre-scaled
    // queries).  Keys past Tk occur in the last tile only; their score
    // accumulators start at -inf, one select per score slot shared by the query
    // groups, which keeps the tile one basic block for the scheduler.
    auto tile = [&](int k0, lds_char* Kb, lds_char* Vb, float c) __attribute__((always_inline)) {
        f32x4 init[4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) init[j][r] = k0 + 16 * j + 4 * grp + r < Tk ? 0.f : -INFINITY;

        f32x4 s[QG][4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
#pragma unroll
            for (int g = 0; g < QG; ++g) s[g][j] = init[j];
#pragma unroll
            for (int i = 0; i < S::n32x; ++i) {
                const bf16x8 kf = __builtin_bit_cast(
                    bf16x8, *(__attribute__((address_space(3))) const u32x4*)(Kb + kofs[i] + 16u * j * ROWB));
#pragma unroll
                for (int g = 0; g < QG; ++g) s[g][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf, qf[g][i], s[g][j], 0, 0, 0);
            }
        }
        // Softmax in the log2 domain on raw scores (the scale is positive, so
        // the row max can be taken before scaling and folded into one FMA).
        // The reference max m_run moves only when some lane's row max exceeds
        // it by more than 8 (log2 units), so the rescale of O and l is rare
        // after the first tiles; until then p = 2^(s c - m c) stays below 2^8.
#pragma unroll
        for (int g = 0; g < QG; ++g) {
            float mloc = -INFINITY;
#pragma unroll
            for (int j = 0; j < 4; ++j)
                mloc = vmax(vmax(mloc, vmax(s[g][j][0], s[g][j][1])), vmax(s[g][j][2], s[g][j][3]));
            mloc = group_max(mloc);
            const float m_cand = vmax(m_run[g], mloc);
            if (__any((m_cand - m_run[g]) * c > 8.0f)) {     // true on the first tile (m_run = -inf)
                const float alpha = __builtin_amdgcn_exp2f((m_run[g] - m_cand) * c);
                if constexpr (!PADSUM) osum[g] *= alpha;
#pragma unroll
                for (int i = 0; i < S::DV / 16; ++i) o[g][i] *= alpha;
                m_run[g] = m_cand;
            }
            const float mc = m_run[g] * c;
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s[g][j][r], c, -mc));
                    s[g][j][r] = p;
                }
        }

        pv(Vb, s);
    };

    // Streaming tile.  The reference max m of a query moves (with O and the row
    // sums rescaled) on the first tile and whenever one of a lane's scores
    // exceeds it by more than 8 (log2 units), which keeps p < 2^8.  Keys past
    // Tk occur only in the last tile; their scores are set to -inf under a
    // branch.  The row max takes 8 three-input maxima for the 16 scores of a
    // lane.
    // Pre-scaled queries (QS: q already carries the factor c = log2(e) /
    // sqrt(d)): the MFMA yields scores in log2 units, and each group's score
    // accumulators start at -m, so its output is already s c - m and
    // p = 2^(output), no per-score FMA.  Otherwise they start at 0 and
    // p = 2^(s c - m c), one FMA per score.
    f32x4 negm[QG];
#pragma unroll
    for (int g = 0; g < QG; ++g) negm[g] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto tile_stream = [&](int k0, auto bufc, bool first) __attribute__((always_inline)) {
        constexpr int BUF = decltype(bufc)::value;
        lds_char* Kb = (lds_char*)&sK[BUF][0];
        lds_char* Vb = (lds_char*)&sV[BUF][0];
        f32x4 s[QG][4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
#pragma unroll
            for (int c = 0; c < S::n32x; ++c) {
                const bf16x8 kf = __builtin_bit_cast(
                    bf16x8, *(__attribute__((address_space(3))) const u32x4*)(Kb + kofs[c] + 16u * j * ROWB));
#pragma unroll
                for (int g = 0; g < QG; ++g)
                    s[g][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf, qf[g][c], c == 0 ? negm[g] : s[g][j], 0, 0, 0);
            }
        }
        if (k0 + kKTile > Tk) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (k0 + 16 * j + 4 * grp + r >= Tk) {
#pragma unroll
                        for (int g = 0; g < QG; ++g) s[g][j][r] = -INFINITY;
                    }
        }
        float mloc[QG];
#pragma unroll
        for (int g = 0; g < QG; ++g) {
            const f32x4* v = s[g];
            float m1 = vmax(vmax(v[0][0], v[0][1]), v[0][2]);
            float m2 = vmax(vmax(v[0][3], v[1][0]), v[1][1]);
            float m3 = vmax(vmax(v[1][2], v[1][3]), v[2][0]);
            float m4 = vmax(vmax(v[2][1], v[2][2]), v[2][3]);
            float m5 = vmax(vmax(v[3][0], v[3][1]), v[3][2]);
            float m6 = vmax(vmax(m1, m2), v[3][3]);
            float m7 = vmax(vmax(m3, m4), m5);
            mloc[g] = vmax(m6, m7);     // this lane's 16 scores; the query's max needs its 4 lanes
        }
        // The test needs no cross-lane max: some lane over the threshold is
        // enough, and only the (rare) rescale reduces over a query's lanes.
        const float sc = QS ? 1.f : a.scale_log2;
        float lane_top = QS ? mloc[0] : (mloc[0] - m_run[0]) * sc;      // excess over the reference, log2 units
#pragma unroll
        for (int g = 1; g < QG; ++g) lane_top = vmax(lane_top, QS ? mloc[g] : (mloc[g] - m_run[g]) * sc);
        if (__any(first || lane_top > 8.0f)) {
#pragma unroll
            for (int g = 0; g < QG; ++g) {
                const float qmax = QS ? group_max(mloc[g]) : group_max(mloc[g]) - m_run[g];
                const float shift = first ? qmax : vmax(qmax, 0.f);
                m_run[g] += shift;
                if constexpr (QS) negm[g] = f32x4{-m_run[g], -m_run[g], -m_run[g], -m_run[g]};
                if (!first) {
                    const float alpha = __builtin_amdgcn_exp2f(-shift * sc);
                    if constexpr (!PADSUM) osum[g] *= alpha;
#pragma unroll
                    for (int i = 0; i < S::DV / 16; ++i) o[g][i] *= alpha;
                }
                if constexpr (QS) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) s[g][j] -= shift;
                }
            }
        }
#pragma unroll
        for (int g = 0; g < QG; ++g) {
            const float mc = m_run[g] * sc;
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    s[g][j][r] = __builtin_amdgcn_exp2f(QS ? s[g][j][r] : __builtin_fmaf(s[g][j][r], sc, -mc));
        }
        pv(Vb, s);
    };

    if constexpr (!STREAM) {
        // What needs no K or V (accumulators, operand addresses, the scale) is
        // worked out while they are on their way; the compiler puts it behind the
        // wait, where every wave of the workgroup does it at once: 2 x 19 x 2624 x
        // 207 at d = 64 19.1 us so and 18.8 now, 18 x 1178 x 137 at d = 128 9.26 and
        // 9.10.  d = 72 keeps its order: addresses held over the wait are ten
        // registers, and with two query groups the key loop came out slower.
        float c = a.scale_log2;
        if constexpr (!QKV && !(HD == 72 && QG == 2)) {
#pragma unroll
            for (int g = 0; g < QG; ++g) {
                asm volatile("" : "+v"(m_run[g]));
                if constexpr (!PADSUM) asm volatile("" : "+v"(osum[g]));
#pragma unroll
                for (int i = 0; i < S::DV / 16; ++i) asm volatile("" : "+v"(o[g][i]));
            }
        }
        if constexpr (!QKV && HD != 72) {
            asm volatile("" : "+s"(c));
#pragma unroll
            for (int i = 0; i < S::n32x; ++i) asm volatile("" : "+v"(kofs[i]));
#pragma unroll
            for (int i = 0; i < S::DV / 16; ++i) asm volatile("" : "+v"(vofs[i]));
        }
        __builtin_amdgcn_s_waitcnt((0 & 15) | (7 << 4) | (15 << 8));   // vmcnt(0): this wave's loads
        __syncthreads();
        for (int t = 0; t < ntiles; ++t) tile(t * kKTile, (lds_char*)sK[t], (lds_char*)sV[t], c);
    } else {
        // Unrolled by two so that each step's buffer is a compile-time constant.
        auto step = [&](int t, auto bufc) __attribute__((always_inline)) {
            constexpr int BUF = decltype(bufc)::value;
            __builtin_amdgcn_s_waitcnt((0 & 15) | (7 << 4) | (15 << 8));   // vmcnt(0): this wave's loads of tile t
            __syncthreads();
            if (t + 1 < ntiles) issue((t + 1) * kKTile, BUF ^ 1);
            tile_stream(t * kKTile, bufc, t == 0);
        };
        for (int t = 0; t < ntiles; t += 2) {
            step(t, std::integral_constant<int, 0>{});
            if (t + 1 < ntiles) step(t + 1, std::integral_constant<int, 1>{});
        }
    }

#pragma unroll
    for (int g = 0; g < QG; ++g) {
        float lsum;
        if constexpr (PADSUM) {
            // Output rows 4 (l / 16) + r of the last block: lanes 32-63 hold the
            // padding rows (the row sums), lanes 0-31 take them from l ^ 32.
            const float mine = o[g][S::DV / 16 - 1][0];
            const float other = __shfl_xor(mine, 32);
            lsum = lane < 32 ? other : mine;
        } else {
            lsum = osum[g][0];     // every row of the ones block is the sum
        }
        const float inv = 1.f / lsum;
        if (myq[g] < Tq) {
            bf16* orow = const_cast<bf16*>(seg_row<bf16>(a.o0, a.o1, a.Tq0, a.Tq1, a.ldo, b, myq[g])) + col0;
            // A lane holds four consecutive d of each 16-row block: one 8-byte
            // store each, at any alignment of the output.  The streaming kernels
            // are given an aligned and an unaligned path, which compile to the
            // same stores, in an order that is 1 % faster there (3 x 14 heads of
            // 517 x 600 at d = 64 11.55 us against 11.67); the resident ones lost
            // as much by the branches.
#pragma unroll
            for (int i = 0; i < S::DV / 16; ++i) {
                const int d = 16 * i + 4 * grp;     // HD % 4 == 0: all four in or all out
                if (d >= HD) continue;
                if (!STREAM || o8) {
                    bf16x4 w;
#pragma unroll
                    for (int r = 0; r < 4; ++r) w[r] = (bf16)(o[g][i][r] * inv);
                    if constexpr (STREAM) *reinterpret_cast<bf16x4*>(orow + d) = w;
                    else __builtin_memcpy(orow + d, &w, sizeof w);
                } else {
#pragma unroll
                    for (int r = 0; r < 4; ++r) st(orow + d + r, o[g][i][r] * inv);
                }
            }
        }
    }
}

template <int QG, int NWV, int NB, bool STREAM = true, bool QS = false>
static int run_attention_dma(const AttnArgs& a, int hd, hipStream_t s) {
    const int Tq = a.Tq0 + a.Tq1;
    const int64_t nwg = (int64_t)((Tq + 16 * QG * NWV - 1) / (16 * QG * NWV)) * a.H * a.B;
    if (nwg > 0x7fffffff) return fail(BC_ERR_UNSUPPORTED, "attention grid too large");
    dim3 grid((unsigned)nwg), block(64 * NWV);
    switch (hd) {
#define BC_ATT_CASE(HD) case HD: launch_k(attention_dma_kernel<HD, QG, NWV, NB, STREAM, QS>, grid, block, s, a); break;
        BC_ATT_CASE(32) BC_ATT_CASE(64) BC_ATT_CASE(72)
#undef BC_ATT_CASE
        case 128:
            // 64 queries per wave at d = 128 would spill: only up to 32.
            if constexpr (QG <= 2) {
                launch_k(attention_dma_kernel<128, QG, NWV, NB, STREAM, QS>, grid, block, s, a);
                break;
            } else {
                return fail(BC_ERR_UNSUPPORTED, "head_dim 128 with %d query groups per wave", QG);
            }
        default: return fail(BC_ERR_UNSUPPORTED, "head_dim %d (supported: 32, 64, 72, 128)", hd);
    }
    return check_launch("attention");
}

template <typename T, int QG>
static int run_attention(const AttnArgs& a, int hd, hipStream_t s) {
    const int Tq = a.Tq0 + a.Tq1;
    const int64_t nwg = (int64_t)((Tq + 64 * QG - 1) / (64 * QG)) * a.H * a.B;
    if (nwg > 0x7fffffff) return fail(BC_ERR_UNSUPPORTED, "attention grid too large");
    dim3 grid((unsigned)nwg), block(kAttnThreads);
    switch (hd) {
#define BC_ATT_CASE(HD) case HD: launch_k(attention_kernel<T, HD, QG>, grid, block, s, a); break;
        BC_ATT_CASE(32) BC_ATT_CASE(64) BC_ATT_CASE(72) BC_ATT_CASE(128)
#undef BC_ATT_CASE
        default: return fail(BC_ERR_UNSUPPORTED, "head_dim %d (supported: 32, 64, 72, 128)", hd);
    }
    return check_launch("attention");
}

bool attention_supported(int hd) { return hd == 32 || hd == 64 || hd == 72 || hd == 128; }

// The workgroup's shape for a call.  Up to 256 keys, every key tile is resident
// in LDS (one load, no barriers in the key loop): 8 waves of 32 queries when
// that still leaves two rounds of 256-query workgroups (PixArt's
// cross-attention to 120 keys at batch 4: 35.1 -> 28.7 us in a probe, 59.6 ->
// 58.5 ms of attention per sampling run), 4 waves of 16 when those make at most
// one round (one DiT-XL/2 sample: 6.5 us against 7.4 with 8 waves), else 8
// waves of 16 (DiT-XL/2's self-attention at batch 16: 13.9 us against 17.6 with
// 4 waves).
// Longer sequences, waves over a double buffer: 8 waves of 64 queries (d <= 72:
// every K/V fragment read from LDS feeds four MFMAs; at d = 128 they would
// spill), 4 waves of 32, or 4 of 16; the one whose fullest CU (rounds of 256
// workgroups times queries each) finishes first at the rate that it reaches on
// a full grid (4 x 16 x 4096^2 x 72: 1014, 965 and 733 TFLOP/s; 550 for 4 x 16
// at d = 128, where two workgroups fill a CU's LDS: 24 heads of 1846^2 71 us
// against 56 with 4 x 32).  2 x 16 x 2050^2 x 64, unscaled: 4 x 32 queries in 63
// us, 4 x 16 in 65, 8 x 32 in 99; 1 x 16 x 1020^2 x 72: 4 x 16 in 16.4 us, 4 x 32
// in 20.1; at d = 128 two 4-wave workgroups a CU, whose barriers do not line up,
// ran 24 x 14 566 tokens 6 % faster than one of 8 waves.
// Where the 128-query workgroups make at most one round, 8 waves of 16 queries
// instead of 4 of 32, which would leave one wave on each SIMD (3 x 15 heads of
// 337^2 x 64: 8.9 us against 10.4; 18 of 1126 x 558 x 72: 13.6 against 15.1; 2 x
// 19 of 432^2 x 128: 15.7 against 17.3).
static AttnVariant attention_variant(int B, int H, int Tq, int Tk, int d) {
    const int64_t bh = (int64_t)B * H;
    auto wgs = [&](int queries) { return (Tq + queries - 1) / queries * bh; };
    if (Tk <= 4 * kKTile) {
        if (wgs(256) >= 512) return {2, 8, false};
        return {1, wgs(64) <= 256 ? 4 : 8, false};
    }
    auto cost = [&](int queries, double rate) { return (double)((wgs(queries) + 255) / 256 * queries) / rate; };
    const double c64 = d <= 72 ? cost(512, 1014) : INFINITY, c32 = cost(128, 965), c16 = cost(64, d <= 72 ? 733 : 550);
    if (c64 <= c32 && c64 <= c16) return {4, 8, true};
    if (c32 > c16) return {1, 4, true};
    return wgs(128) <= 256 ? AttnVariant{1, 8, true} : AttnVariant{2, 4, true};
}

int launch_attention(int dtype, AttnArgs a, hipStream_t s) {
    if (a.B <= 0 || a.H <= 0 || a.Tq0 + a.Tq1 <= 0) return BC_OK;
    if (a.Tk0 + a.Tk1 <= 0) return fail(BC_ERR_INVALID_ARG, "attention over zero keys");
    if (!attention_supported(a.d)) return fail(BC_ERR_UNSUPPORTED, "head_dim %d (supported: 32, 64, 72, 128)", a.d);
    const uintptr_t kv = reinterpret_cast<uintptr_t>(a.k0) | reinterpret_cast<uintptr_t>(a.v0) |
                         reinterpret_cast<uintptr_t>(a.k1) | reinterpret_cast<uintptr_t>(a.v1);
    const uintptr_t qa = reinterpret_cast<uintptr_t>(a.q0) | reinterpret_cast<uintptr_t>(a.q1);
    if ((a.ldk | a.ldv) % 8 || kv % 16 || (dtype == BC_BF16 && (a.ldq % 8 || qa % 16)))
        return fail(BC_ERR_UNSUPPORTED, "attention rows must be 16-byte aligned");
    if (dtype == BC_F32 && a.d > 64) return fail(BC_ERR_UNSUPPORTED, "fp32 attention supports head_dim <= 64");
    // Pre-scaled queries (q_scaled) already carry the factor log2(e) / sqrt(d).
    a.scale_log2 = a.q_scaled ? 1.0f : attn_q_scale(a.d);
    prof_begin(PROF_ATTENTION, s, 4.0 * a.B * a.H * (double)(a.Tq0 + a.Tq1) * (double)(a.Tk0 + a.Tk1) * a.d);
    // The direct-to-LDS kernel needs 16-byte aligned Q/K/V rows (checked above).
    int rc;
    if (dtype == BC_BF16) {
        const AttnVariant v = attention_variant(a.B, a.H, a.Tq0 + a.Tq1, a.Tk0 + a.Tk1, a.d);
        if (!v.stream) {
            if (v.qg == 2) rc = run_attention_dma<2, 8, 4, false>(a, a.d, s);
            else if (v.waves == 4) rc = run_attention_dma<1, 4, 4, false>(a, a.d, s);
            else rc = run_attention_dma<1, 8, 4, false>(a, a.d, s);
        } else if (v.qg == 4) {
            rc = a.q_scaled ? run_attention_dma<4, 8, 2, true, true>(a, a.d, s) : run_attention_dma<4, 8, 2>(a, a.d, s);
        } else if (v.qg == 2) {
            rc = a.q_scaled ? run_attention_dma<2, 4, 2, true, true>(a, a.d, s) : run_attention_dma<2, 4, 2>(a, a.d, s);
        } else if (v.waves == 8) {
            rc = a.q_scaled ? run_attention_dma<1, 8, 2, true, true>(a, a.d, s) : run_attention_dma<1, 8, 2>(a, a.d, s);
        } else {
            rc = a.q_scaled ? run_attention_dma<1, 4, 2, true, true>(a, a.d, s) : run_attention_dma<1, 4, 2>(a, a.d, s);
        }
    } else {
        rc = run_attention<float, 1>(a, a.d, s);
    }
    prof_end(PROF_ATTENTION, s);
    return rc;
}

bool qkv_attention_supported(int dtype, int T, int head_dim, int dmodel) {
    return dtype == BC_BF16 && T >= 1 && T <= 4 * kKTile && (head_dim == 32 || head_dim == 64 || head_dim == 72) &&
           dmodel >= 128 && dmodel <= 16384 && dmodel % 64 == 0;
}

int launch_qkv_attention(int dtype, AttnArgs a, hipStream_t s) {
    auto al = [](const void* p, int n) { return reinterpret_cast<uintptr_t>(p) % n == 0; };
    if (!qkv_attention_supported(dtype, a.Tk0, a.d, a.dmodel) || a.Tq0 != a.Tk0 || a.Tq1 || a.Tk1 || a.H * a.d != a.dmodel)
        return fail(BC_ERR_UNSUPPORTED, "fused QKV attention: T=%d, d=%d, D=%d, H=%d", a.Tk0, a.d, a.dmodel, a.H);
    if (!a.x || !a.w_qkv || !a.o0 || !al(a.x, 16) || !al(a.w_qkv, 16) || a.ldx % 8 || !al(a.b_qkv, 8))
        return fail(BC_ERR_UNSUPPORTED, "fused QKV attention: 16-byte aligned x and weights, 8-byte aligned bias");
    if (a.B < 1 || a.H < 1) return BC_OK;
    a.o1 = a.o0;
    a.q_scaled = 1;
    a.scale_log2 = 1.0f;
    a.proj_q_scale = attn_q_scale(a.d);
    const double T = a.Tk0;
    prof_begin(PROF_ATTENTION, s, 2.0 * a.B * T * 3.0 * a.dmodel * a.dmodel + 4.0 * a.B * a.H * T * T * a.d);
    const dim3 grid((unsigned)(a.B * a.H)), block(512);
    switch (a.d) {
        case 32: launch_k(attention_dma_kernel<32, 2, 8, 4, false, true, true>, grid, block, s, a); break;
        case 64: launch_k(attention_dma_kernel<64, 2, 8, 4, false, true, true>, grid, block, s, a); break;
        default: launch_k(attention_dma_kernel<72, 2, 8, 4, false, true, true>, grid, block, s, a); break;
    }
    prof_end(PROF_ATTENTION, s);
    return check_launch("qkv attention");
}

}  // namespace bc

using namespace bc;

extern "C" {

int bc_attention_workspace_size(int B, int H, int Tq, int Tk, int d, int dtype, size_t* bytes) {
    clear_error();
    if (!bytes) return fail(BC_ERR_INVALID_ARG, "NULL pointer");
    (void)B; (void)H; (void)Tq; (void)Tk; (void)d; (void)dtype;
    *bytes = 0;   // the kernel reads the [B, T, H, d] layout directly
    return BC_OK;
}

int bc_attention_variant(int B, int H, int Tq, int Tk, int d, int* qg, int* waves, int* stream) {
    clear_error();
    if (!qg || !waves || !stream) return fail(BC_ERR_INVALID_ARG, "NULL pointer");
    if (B < 1 || H < 1 || Tq < 1 || Tk < 1 || !attention_supported(d)) return fail(BC_ERR_INVALID_ARG, "attention shape");
    const AttnVariant v = attention_variant(B, H, Tq, Tk, d);
    *qg = v.qg;
    *waves = v.waves;
    *stream = v.stream ? 1 : 0;
    return BC_OK;
}

static int attention_entry(int B, int H, int Tq, int Tk, int d, const void* q, const void* k, const void* v, void* out,
                           int dtype, int q_scaled, void* stream) {
    if (!q || !k || !v || !out) return fail(BC_ERR_INVALID_ARG, "NULL pointer");
    if (B < 1 || H < 1 || Tq < 1 || Tk < 1 || d < 1) return fail(BC_ERR_INVALID_ARG, "empty attention");
    if (dtype != BC_F32 && dtype != BC_BF16) return fail(BC_ERR_INVALID_ARG, "dtype %d", dtype);
    if (q_scaled && dtype != BC_BF16) return fail(BC_ERR_UNSUPPORTED, "pre-scaled queries are bf16 only");
    AttnArgs a = {};
    a.q_scaled = q_scaled;
    a.q0 = q; a.q1 = q; a.Tq0 = Tq; a.Tq1 = 0; a.ldq = (int64_t)H * d;
    a.k0 = k; a.k1 = k; a.Tk0 = Tk; a.Tk1 = 0; a.ldk = (int64_t)H * d;
    a.v0 = v; a.v1 = v; a.ldv = (int64_t)H * d;
    a.o0 = out; a.o1 = out; a.ldo = (int64_t)H * d;
    a.B = B; a.H = H; a.d = d;
    return launch_attention(dtype, a, static_cast<hipStream_t>(stream));
}

int bc_attention(int B, int H, int Tq, int Tk, int d, const void* q, const void* k, const void* v, void* out,
                 int dtype, void* ws, size_t ws_bytes, void* stream) {
    clear_error();
    (void)ws; (void)ws_bytes;
    return attention_entry(B, H, Tq, Tk, d, q, k, v, out, dtype, 0, stream);
}

int bc_attention_prescaled(int B, int H, int Tq, int Tk, int d, const void* q, const void* k, const void* v,
                           void* out, int dtype, void* ws, size_t ws_bytes, void* stream) {
    clear_error();
    (void)ws; (void)ws_bytes;
    return attention_entry(B, H, Tq, Tk, d, q, k, v, out, dtype, 1, stream);
}

}  // extern "C"
