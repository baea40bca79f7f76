// Dense linear layers of the DiT block, y = epilogue(A W^T), on MFMA.
//
// A [M, K] and W [N, K] are both K-contiguous (the nn.Linear layout), so both
// operands stream into LDS the same way.  A workgroup of 4 waves owns a
// BM x BN output tile and walks K in steps of 128 bytes (64 bf16 / 32 fp32):
// global -> registers (prefetch of the next step) -> LDS (double buffered,
// rows padded by 16 bytes so the 16-byte fragment reads of 16 lanes hit 16
// distinct bank groups) -> MFMA operands.  Each wave computes a
// (BM/2) x (BN/2) sub-tile as a grid of 16x16 MFMA tiles:
//   bf16: v_mfma_f32_16x16x32_bf16, lane l holds row l%16, k = 8(l/16)..+8;
//   fp32: v_mfma_f32_16x16x4_f32,   lane l holds row l%16, k = l/16;
// and accumulates in fp32; lane l ends with rows 4(l/16)..+4 of column l%16.
// The epilogue applies the bias and then one of: nothing, GELU (tanh form),
// or the gated residual x + g * y of the adaLN blocks.
#include <type_traits>

#include "gemm.h"

namespace bc {

// GELU, tanh form: 0.5 x (1 + tanh(y)), y = sqrt(2/pi) (x + 0.044715 x^3).
// Since 0.5 (1 + tanh(y)) = 1 / (1 + exp(-2 y)), this is x / (1 + 2^z) with
// z = -2 log2(e) y = x (A + B x^2): one native exp2 and one reciprocal per
// element (2^z overflows to +inf for very negative x, giving 0 as it should).
__device__ __forceinline__ float gelu_tanh(float x) {
    constexpr float A = -2.0f * 0.7978845608028654f * 1.4426950408889634f;
    constexpr float B = A * 0.044715f;
    const float z = x * __builtin_fmaf(B, x * x, A);
    return x * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(z));
}

template <typename T> struct Mma;
template <> struct Mma<bf16> {
    static constexpr int E = 8;    // operand elements per lane
    static constexpr int KI = 32;  // k per instruction
    typedef bf16x8 frag;
    __device__ static __forceinline__ f32x4 mma(const frag& a, const frag& b, const f32x4& c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
    }
    __device__ static __forceinline__ frag load(const bf16* p) {
        return __builtin_bit_cast(frag, *reinterpret_cast<const u32x4*>(p));
    }
};
template <> struct Mma<float> {
    static constexpr int E = 1;
    static constexpr int KI = 4;
    typedef float frag;
    __device__ static __forceinline__ f32x4 mma(frag a, frag b, const f32x4& c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    __device__ static __forceinline__ frag load(const float* p) { return *p; }
};

// Bias + GELU / gated-residual epilogue for a wave's TM x TN block of 16x16
// accumulators whose top-left output element is (row0, col0).
template <typename T, int EPI, int TM, int TN>
__device__ __forceinline__ void epilogue(const GemmArgs& g, const f32x4 (&acc)[TM][TN], int row0, int col0, int lane) {
    const GemmEpi& e = g.e;
    const T* __restrict__ bias = static_cast<const T*>(e.bias);
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int col = col0 + j * 16 + (lane & 15);
        if (col >= g.N) continue;
        const float bv = bias ? ld(bias + col) : 0.f;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = row0 + i * 16 + 4 * (lane >> 4) + r;
                if (row >= g.M) continue;
                float v = acc[i][j][r] + bv;
                if constexpr (EPI == BC_EPI_GATE_RES) {
                    const float gv = e.gate ? e.gate[(int64_t)(row / e.rows_per_gate) * e.ldg + col] : 1.f;
                    v = e.res[(int64_t)row * e.ldr + col] + gv * v;
                    const int b = row / e.seg, s = row - b * e.seg;
                    if (s < e.keep) {
                        const int64_t o = (int64_t)(b * e.keep + s) * e.ldo + col;
                        if (e.out_f32) static_cast<float*>(e.out)[o] = v;
                        else st(static_cast<T*>(e.out) + o, v);
                    }
                } else {
                    if (col < e.q_scale_to) v *= e.q_scale;
                    if (col >= e.gelu_from) v = gelu_tanh(v);
                    if (col >= e.split) st(static_cast<T*>(e.out2) + (int64_t)row * e.ldo2 + (col - e.split + e.off2), v);
                    else if (e.out_f32) static_cast<float*>(e.out)[(int64_t)row * e.ldo + col] = v;
                    else st(static_cast<T*>(e.out) + (int64_t)row * e.ldo + col, v);
                }
            }
        }
    }
}

// Tile shape: BM x BN per workgroup, a WAVES_M x WAVES_N grid of waves, each
// wave owning a (BM/WAVES_M) x (BN/WAVES_N) block of 16x16 MFMA tiles.
template <typename T_, int EPI, int BM, int BN, int WAVES_M, int WAVES_N>
__global__ __launch_bounds__(64 * WAVES_M * WAVES_N) void gemm_kernel(GemmArgs g) {
    typedef elem_t<T_> T;
    constexpr int NT = 64 * WAVES_M * WAVES_N;       // threads
    constexpr int EPC = 16 / (int)sizeof(T);        // elements per 16-byte chunk
    constexpr int BK = 8 * EPC;                      // 128 bytes of K per step
    constexpr int LDK = BK + EPC;                    // padded LDS row (elements)
    constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;
    constexpr int TM = WM / 16, TN = WN / 16;
    constexpr int CA = BM * 8 / NT;                  // 16-byte chunks per thread per step
    constexpr int CB = BN * 8 / NT;
    static_assert(CA * NT == BM * 8 && CB * NT == BN * 8, "tile must split evenly over threads");
    typedef Mma<T> MM;

    __shared__ __attribute__((aligned(16))) T sA[2][BM][LDK];
    __shared__ __attribute__((aligned(16))) T sB[2][BN][LDK];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int wm = wave / WAVES_N, wn = wave % WAVES_N;

    // Tile order: consecutive workgroup ids go round-robin to the 8 XCDs; give
    // each XCD a contiguous range of tiles, then raster in groups of 8 row
    // tiles so neighbouring workgroups share A rows and W rows in L2.
    const int tiles_m = (g.M + BM - 1) / BM;
    const int tiles_n = (g.N + BN - 1) / BN;
    const int nwg = gridDim.x;
    const int pid = xcd_contiguous(blockIdx.x, nwg);
    constexpr int GROUP_M = 8;
    const int group = GROUP_M * tiles_n;
    const int first_m = (pid / group) * GROUP_M;
    const int gm = min(tiles_m - first_m, GROUP_M);
    const int tm = first_m + (pid % group) % gm;
    const int tn = (pid % group) / gm;
    const int bm = tm * BM, bn = tn * BN;

    const T* __restrict__ A = static_cast<const T*>(g.A);
    const T* __restrict__ W = static_cast<const T*>(g.W);

    u32x4 ra[CA], rb[CB];
    auto load_global = [&](int k0) {
#pragma unroll
        for (int i = 0; i < CA; ++i) {
            const int c = tid + i * NT;
            const int row = c >> 3, kc = k0 + (c & 7) * EPC;
            const int grow = bm + row;
            if (grow < g.M && kc < g.K)
                ra[i] = *reinterpret_cast<const u32x4*>(A + (int64_t)grow * g.lda + kc);
            else
                ra[i] = u32x4{0, 0, 0, 0};
        }
#pragma unroll
        for (int i = 0; i < CB; ++i) {
            const int c = tid + i * NT;
            const int row = c >> 3, kc = k0 + (c & 7) * EPC;
            const int grow = bn + row;
            if (grow < g.N && kc < g.K)
                rb[i] = *reinterpret_cast<const u32x4*>(W + (int64_t)grow * g.ldw + kc);
            else
                rb[i] = u32x4{0, 0, 0, 0};
        }
    };
    auto store_lds = [&](int buf) {
#pragma unroll
        for (int i = 0; i < CA; ++i) {
            const int c = tid + i * NT;
            *reinterpret_cast<u32x4*>(&sA[buf][c >> 3][(c & 7) * EPC]) = ra[i];
        }
#pragma unroll
        for (int i = 0; i < CB; ++i) {
            const int c = tid + i * NT;
            *reinterpret_cast<u32x4*>(&sB[buf][c >> 3][(c & 7) * EPC]) = rb[i];
        }
    };

    f32x4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    const int nk = (g.K + BK - 1) / BK;
    load_global(0);
    store_lds(0);
    __syncthreads();

    const int frow = lane & 15;
    const int fk = (lane >> 4) * MM::E;
    for (int kt = 0; kt < nk; ++kt) {
        const int cur = kt & 1;
        if (kt + 1 < nk) load_global((kt + 1) * BK);
#pragma unroll
        for (int kk = 0; kk < BK / MM::KI; ++kk) {
            typename MM::frag af[TM], bfr[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i) af[i] = MM::load(&sA[cur][wm * WM + i * 16 + frow][kk * MM::KI + fk]);
#pragma unroll
            for (int j = 0; j < TN; ++j) bfr[j] = MM::load(&sB[cur][wn * WN + j * 16 + frow][kk * MM::KI + fk]);
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) acc[i][j] = MM::mma(af[i], bfr[j], acc[i][j]);
        }
        if (kt + 1 < nk) store_lds(cur ^ 1);
        __syncthreads();
    }

    epilogue<T, EPI, TM, TN>(g, acc, bm + wm * WM, bn + wn * WN, lane);
}

// ---------------------------------------------------------------------------
// bf16 main loop with direct-to-LDS loads.
//
// Operand tiles go from HBM straight into LDS with global_load_lds_dwordx4:
// one wave-wide instruction moves 8 rows x 128 bytes (each lane 16 bytes,
// lane i landing at M0 + 16 i), so no registers or ds_write instructions are
// spent on staging.  LDS rows are 128 bytes (64 k) with no padding; to keep
// the 16-byte fragment reads of 16 consecutive rows conflict-free, the 16-byte
// chunk c of row r is stored in slot c ^ ((r >> 1) & 7), which the loading
// lane realises by choosing which global chunk it fetches.  STAGES k-steps are
// in flight: after the barrier of step kt the loads of step kt + STAGES - 1
// are issued into the buffer step kt - 1 used, and the wait before each
// barrier only drains the loads of the step about to be consumed.
// Requires K % 64 == 0 (whole k-steps); rows past M or N are clamped to the
// last row, so they load valid memory and only feed outputs never stored.
// ---------------------------------------------------------------------------
// LDS slot permutation of row r (see above).
__device__ __forceinline__ int swz(int row) { return (row >> 1) & 7; }

template <int EPI, int BM, int BN, int WAVES_M, int WAVES_N, int STAGES, bool SEG>
__device__ __forceinline__ void gemm_dma_body(GemmArgs g, const GemmSeg* sg) {
    typedef bf16 T;
    typedef Mma<bf16> MM;
    constexpr int NW = WAVES_M * WAVES_N;
    constexpr int BK = 64;
    constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;
    constexpr int TM = WM / 16, TN = WN / 16;
    constexpr int OA = BM / 8 / NW, OB = BN / 8 / NW;     // row octets per wave per step
    constexpr int L = OA + OB;                             // loads per wave per step
    static_assert(OA * 8 * NW == BM && OB * 8 * NW == BN, "octets must split over waves");

    __shared__ __attribute__((aligned(1024))) T sA[STAGES][BM * BK];
    __shared__ __attribute__((aligned(1024))) T sB[STAGES][BN * BK];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WAVES_N, wn = wave % WAVES_N;

    const int tiles_m = (g.M + BM - 1) / BM;
    const int tiles_n = (g.N + BN - 1) / BN;
    const int nwg = gridDim.x;
    const int pid = xcd_contiguous(blockIdx.x, nwg);
    constexpr int GROUP_M = 8;
    const int group = GROUP_M * tiles_n;
    const int first_m = (pid / group) * GROUP_M;
    const int gm = min(tiles_m - first_m, GROUP_M);
    const int tm = first_m + (pid % group) % gm;
    const int tn = (pid % group) / gm;
    const int bm = tm * BM, bn = tn * BN;
    if constexpr (SEG) {
        // Grouped GEMM: column block bn lies in segment bn / Nseg, whose own
        // weight matrix [Nseg, K] and bias hold its rows.
        const int seg = bn / sg->Nseg;
        const int off = seg * sg->Nseg;
        g.W = static_cast<const bf16*>(sg->W[seg]) - (int64_t)off * g.ldw;
        g.e.bias = sg->bias[seg] ? static_cast<const bf16*>(sg->bias[seg]) - off : nullptr;
    }

    // Per-lane global source of each of this wave's octets (k offset added per step).
    const T* srcA[OA];
    const T* srcB[OB];
    const int lrow = lane >> 3, lslot = lane & 7;
#pragma unroll
    for (int o = 0; o < OA; ++o) {
        const int r = (wave * OA + o) * 8 + lrow;
        const int grow = min(bm + r, g.M - 1);
        srcA[o] = static_cast<const T*>(g.A) + (int64_t)grow * g.lda + ((lslot ^ swz(r)) * 8);
    }
#pragma unroll
    for (int o = 0; o < OB; ++o) {
        const int r = (wave * OB + o) * 8 + lrow;
        const int grow = min(bn + r, g.N - 1);
        srcB[o] = static_cast<const T*>(g.W) + (int64_t)grow * g.ldw + ((lslot ^ swz(r)) * 8);
    }
    auto issue = [&](int kt, int buf) {
        const int k0 = kt * BK;
#pragma unroll
        for (int o = 0; o < OA; ++o)
            dma16(srcA[o] + k0, &sA[buf][(wave * OA + o) * 8 * BK]);
#pragma unroll
        for (int o = 0; o < OB; ++o)
            dma16(srcB[o] + k0, &sB[buf][(wave * OB + o) * 8 * BK]);
    };

    f32x4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    const int nk = g.K / BK;
#pragma unroll
    for (int p = 0; p < STAGES - 1; ++p)
        if (p < nk) issue(p, p);

    const int frow = lane & 15, grp = lane >> 4;
    for (int kt = 0; kt < nk; ++kt) {
        if (kt + STAGES - 2 < nk) wait_vmcnt<(STAGES - 2) * L>();
        else wait_vmcnt<0>();
        __syncthreads();
        if (kt + STAGES - 1 < nk) issue(kt + STAGES - 1, (kt + STAGES - 1) % STAGES);
        const T* a = sA[kt % STAGES];
        const T* b = sB[kt % STAGES];
#pragma unroll
        for (int kk = 0; kk < BK / 32; ++kk) {
            const int c = kk * 4 + grp;
            MM::frag af[TM], bfr[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const int r = wm * WM + i * 16 + frow;
                af[i] = MM::load(a + r * BK + ((c ^ swz(r)) * 8));
            }
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int r = wn * WN + j * 16 + frow;
                bfr[j] = MM::load(b + r * BK + ((c ^ swz(r)) * 8));
            }
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) acc[i][j] = MM::mma(af[i], bfr[j], acc[i][j]);
        }
    }

    epilogue<T, EPI, TM, TN>(g, acc, bm + wm * WM, bn + wn * WN, lane);
}

// ---------------------------------------------------------------------------
// Wide-tile bf16 kernel (128 x 432 and 128 x 128 tiles).
//
// Same direct-to-LDS staging and swizzle as above, two stages, with two
// changes:
//  * tiles need not be powers of two (128 x 432); the (BM + BN) / 8 row octets
//    of a k-step are dealt round-robin to the waves;
//  * the MFMA operands are swapped (W rows as the instruction's A), so lane l
//    accumulates out[row][col..col+3] with row = l % 16 and
//    col = 4 (l / 16): the epilogue reads and writes four consecutive
//    columns per lane with one vector access.
// Host-side conditions: K % 64 == 0; lda, ldw % 8 == 0; every epilogue
// column index, stride and boundary (N, split, gelu_from, off2, ldo, ldo2,
// ldr, ldg) a multiple of 4 and the epilogue pointers 16-byte aligned.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void st4(bf16* p, const float (&v)[4]) {
    bf16x4 q;
    q[0] = (bf16)v[0]; q[1] = (bf16)v[1]; q[2] = (bf16)v[2]; q[3] = (bf16)v[3];
    *reinterpret_cast<bf16x4*>(p) = q;
}
__device__ __forceinline__ void st4(float* p, const float (&v)[4]) {
    *reinterpret_cast<f32x4*>(p) = f32x4{v[0], v[1], v[2], v[3]};
}

// The gated residual of four consecutive columns of one row (bf16 operands).
__device__ __forceinline__ void gate_res4(const GemmArgs& g, int row, int col, const f32x4& acc, const f32x4& res) {
    const GemmEpi& e = g.e;
    const int b = row / e.seg, sidx = row - b * e.seg;
    if (sidx >= e.keep) return;
    const f32x4 gv = e.gate ? *reinterpret_cast<const f32x4*>(e.gate + (int64_t)(row / e.rows_per_gate) * e.ldg + col)
                            : f32x4{1.f, 1.f, 1.f, 1.f};
    float bv[4] = {0.f, 0.f, 0.f, 0.f}, v[4];
    if (e.bias) {
        const bf16x4 b4 = *reinterpret_cast<const bf16x4*>(static_cast<const bf16*>(e.bias) + col);
#pragma unroll
        for (int r = 0; r < 4; ++r) bv[r] = (float)b4[r];
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = res[r] + gv[r] * (acc[r] + bv[r]);
    const int64_t o = (int64_t)(b * e.keep + sidx) * e.ldo + col;
    if (e.out_f32) st4(static_cast<float*>(e.out) + o, v);
    else st4(static_cast<bf16*>(e.out) + o, v);
}

// Epilogue straight from the accumulators (gated residual; fp32 outputs of
// the plain epilogue).
template <int EPI, int TM, int TN>
__device__ __forceinline__ void epilogue_t(const GemmArgs& g, const f32x4 (&acc)[TM][TN], int row0, int col0, int lane) {
    const GemmEpi& e = g.e;
    if constexpr (EPI == BC_EPI_GATE_RES) {
        // Rows outer: the row's destination (ring-slot remap) is worked out once.
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int row = row0 + i * 16 + (lane & 15);
            if (row >= g.M) continue;
            const int b = row / e.seg, sidx = row - b * e.seg;
            if (sidx >= e.keep) continue;
            const int64_t orow = (int64_t)(b * e.keep + sidx) * e.ldo;
            const float* grow = e.gate ? e.gate + (int64_t)(row / e.rows_per_gate) * e.ldg : nullptr;
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int col = col0 + j * 16 + 4 * (lane >> 4);
                if (col >= g.N) continue;
                float v[4];
                const bf16* __restrict__ bias = static_cast<const bf16*>(e.bias);
                float bv[4] = {0.f, 0.f, 0.f, 0.f};
                if (bias) {
                    const bf16x4 b4 = *reinterpret_cast<const bf16x4*>(bias + col);
#pragma unroll
                    for (int r = 0; r < 4; ++r) bv[r] = (float)b4[r];
                }
                const f32x4 gv = grow ? *reinterpret_cast<const f32x4*>(grow + col) : f32x4{1.f, 1.f, 1.f, 1.f};
                const f32x4 rv = *reinterpret_cast<const f32x4*>(e.res + (int64_t)row * e.ldr + col);
#pragma unroll
                for (int r = 0; r < 4; ++r) v[r] = rv[r] + gv[r] * (acc[i][j][r] + bv[r]);
                if (e.out_f32) st4(static_cast<float*>(e.out) + orow + col, v);
                else st4(static_cast<bf16*>(e.out) + orow + col, v);
            }
        }
        return;
    }
    const bf16* __restrict__ bias = static_cast<const bf16*>(e.bias);
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int col = col0 + j * 16 + 4 * (lane >> 4);
        const bool col_ok = col < g.N;
        float bv[4] = {0.f, 0.f, 0.f, 0.f};
        if (bias && col_ok) {
            const bf16x4 b4 = *reinterpret_cast<const bf16x4*>(bias + col);
#pragma unroll
            for (int r = 0; r < 4; ++r) bv[r] = (float)b4[r];
        }
        if (!col_ok) continue;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int row = row0 + i * 16 + (lane & 15);
            if (row >= g.M) continue;
            float v[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = acc[i][j][r] + bv[r];
            if (col < e.q_scale_to) {
#pragma unroll
                for (int r = 0; r < 4; ++r) v[r] *= e.q_scale;
            }
            if (col >= e.gelu_from) {
#pragma unroll
                for (int r = 0; r < 4; ++r) v[r] = gelu_tanh(v[r]);
            }
            if (col >= e.split) st4(static_cast<bf16*>(e.out2) + (int64_t)row * e.ldo2 + (col - e.split + e.off2), v);
            else if (e.out_f32) st4(static_cast<float*>(e.out) + (int64_t)row * e.ldo + col, v);
            else st4(static_cast<bf16*>(e.out) + (int64_t)row * e.ldo + col, v);
        }
    }
}

// AHEAD (gated epilogue through LDS): when the residual is read, see there.
template <int EPI, int BM, int BN, int WAVES_M, int WAVES_N, bool AHEAD = false>
__global__ __launch_bounds__(64 * WAVES_M * WAVES_N) void gemm_wide_kernel(GemmArgs g) {
    typedef bf16 T;
    typedef Mma<bf16> MM;
    constexpr int NW = WAVES_M * WAVES_N, NT = 64 * NW, BK = 64;
    constexpr int TM = BM / WAVES_M / 16, TN = BN / WAVES_N / 16;
    constexpr int NOCT = (BM + BN) / 8;                    // wave-wide loads per stage (8 rows of 128 bytes each)
    constexpr int QMAX = (NOCT + NW - 1) / NW;             // of them per wave (at most)
    static_assert(TM * 16 * WAVES_M == BM && TN * 16 * WAVES_N == BN, "tile shape");
    constexpr int STAGE = (BM + BN) * BK;                  // BM rows of A, then BN rows of W
    constexpr int OPITCH = BN + 8;                         // staged bf16 output row (16-byte pad)
    constexpr int SMEM0 = 2 * STAGE > BM * OPITCH ? 2 * STAGE : BM * OPITCH;
    // Gated epilogue through LDS (small tiles): an fp32 row-major copy of the
    // tile, FPITCH floats per row.
    constexpr int FPITCH = BN + 4;
    constexpr bool STAGE_GATED = EPI == BC_EPI_GATE_RES && BM * FPITCH * 4 <= 96 * 1024;
    constexpr int SMEM = STAGE_GATED && BM * FPITCH * 2 > SMEM0 ? BM * FPITCH * 2 : SMEM0;   // in bf16 units
    __shared__ __attribute__((aligned(1024))) T sm[SMEM];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WAVES_N, wn = wave % WAVES_N;
    const int tile = xcd_contiguous(blockIdx.x, gridDim.x);

    const int tiles_m = (g.M + BM - 1) / BM;
    const int tiles_n = (g.N + BN - 1) / BN;
    constexpr int GROUP_M = 8;
    const int group = GROUP_M * tiles_n;
    const int first_m = (tile / group) * GROUP_M;
    const int gm = min(tiles_m - first_m, GROUP_M);
    const int tm = first_m + (tile % group) % gm;
    const int tn = (tile % group) / gm;
    const int bm = tm * BM, bn = tn * BN;

    // Load o = wave + NW q of a stage fills rows 8 o .. 8 o + 7 (A rows first,
    // then W rows); lane L loads row 8 o + L / 8 into slot L % 8, fetching the
    // global chunk that the swizzle puts there.
    const T* src[QMAX];
#pragma unroll
    for (int q = 0; q < QMAX; ++q) {
        const int r = 8 * min(wave + NW * q, NOCT - 1) + (lane >> 3);
        const T* p;
        if (r < BM) p = static_cast<const T*>(g.A) + (int64_t)min(bm + r, g.M - 1) * g.lda;
        else p = static_cast<const T*>(g.W) + (int64_t)min(bn + r - BM, g.N - 1) * g.ldw;
        src[q] = p + ((lane & 7) ^ swz(r)) * 8;
    }
    const int nk = g.K / BK;
    auto issue = [&](int kt, int buf) {
#pragma unroll
        for (int q = 0; q < QMAX; ++q) {
            const int o = wave + NW * q;
            if (NOCT % NW == 0 || o < NOCT) dma16(src[q] + kt * BK, &sm[buf * STAGE + o * 8 * BK]);
        }
    };

    f32x4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    issue(0, 0);
    const int frow = lane & 15, grp = lane >> 4;
    for (int kt = 0; kt < nk; ++kt) {
        wait_vmcnt<0>();
        __syncthreads();
        if (kt + 1 < nk) issue(kt + 1, (kt + 1) & 1);
        const T* st = sm + (kt & 1) * STAGE;
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            const int c = kk * 4 + grp;
            MM::frag af[TM], bfr[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const int r = (wm * TM + i) * 16 + frow;
                af[i] = MM::load(st + r * BK + (c ^ swz(r)) * 8);
            }
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int r = BM + (wn * TN + j) * 16 + frow;
                bfr[j] = MM::load(st + r * BK + (c ^ swz(r)) * 8);
            }
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) acc[i][j] = MM::mma(bfr[j], af[i], acc[i][j]);
        }
    }

    const GemmEpi& e = g.e;
    const bf16* __restrict__ bias = static_cast<const bf16*>(e.bias);
    if constexpr (STAGE_GATED) {
        // The tile goes through LDS as fp32 rows, and all waves then apply the
        // gated residual to whole rows, reading the residual and gate and
        // writing the stream as consecutive 16-byte chunks.  The residual is read
        // where it is added; AHEAD: all of a thread's before the LDS passes (the
        // stream is updated in place, so no load is moved over a store by itself).
        constexpr int C4 = BN / 4, IT = BM * C4 / NT;         // 4-column chunks per tile row, and per thread
        static_assert(IT * NT == BM * C4, "chunks per thread");
        f32x4 rv[AHEAD ? IT : 1];
        if constexpr (AHEAD) {
#pragma unroll
            for (int t = 0; t < IT; ++t) {
                const int q = tid + NT * t, row = min(bm + q / C4, g.M - 1), col = min(bn + q % C4 * 4, g.N - 4);
                rv[t] = *reinterpret_cast<const f32x4*>(e.res + (int64_t)row * e.ldr + col);
            }
        }
        float* ft = reinterpret_cast<float*>(sm);
        __syncthreads();   // every wave is done with the stage buffers
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int i = 0; i < TM; ++i)
                *reinterpret_cast<f32x4*>(ft + ((wm * TM + i) * 16 + frow) * FPITCH + (wn * TN + j) * 16 + 4 * grp) = acc[i][j];
        __syncthreads();
#pragma unroll
        for (int t = 0; t < IT; ++t) {
            const int q = tid + NT * t, lr = q / C4, lc = q % C4 * 4;
            const int row = bm + lr, col = bn + lc;
            if (row >= g.M || col >= g.N) continue;
            if constexpr (!AHEAD) rv[0] = *reinterpret_cast<const f32x4*>(e.res + (int64_t)row * e.ldr + col);
            gate_res4(g, row, col, *reinterpret_cast<const f32x4*>(ft + lr * FPITCH + lc), rv[AHEAD ? t : 0]);
        }
        return;
    }
    if constexpr (EPI == BC_EPI_BIAS) {
        if (!e.out_f32) {
            // bf16 outputs leave through LDS: the waves write their finished
            // values into a row-major copy of the tile, then the workgroup stores
            // it as consecutive 16-byte chunks of each row, so every store
            // instruction covers whole cache lines.  (Written straight from the
            // accumulators, 32-byte pieces of lines from all 256 one-round tiles
            // at once came back as about 1.5x the output bytes in HBM writes.)
            __syncthreads();   // every wave is done with the stage buffers
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int lc = (wn * TN + j) * 16 + 4 * grp;
                const int col = bn + lc;
                float bv[4] = {0.f, 0.f, 0.f, 0.f};
                if (bias && col < g.N) {
                    const bf16x4 b4 = *reinterpret_cast<const bf16x4*>(bias + col);
#pragma unroll
                    for (int r = 0; r < 4; ++r) bv[r] = (float)b4[r];
                }
                const bool act = col >= e.gelu_from;
                const float qs = col < e.q_scale_to ? e.q_scale : 1.f;
#pragma unroll
                for (int i = 0; i < TM; ++i) {
                    bf16x4 q;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        float v = (acc[i][j][r] + bv[r]) * qs;
                        if (act) v = gelu_tanh(v);
                        q[r] = (bf16)v;
                    }
                    *reinterpret_cast<bf16x4*>(sm + ((wm * TM + i) * 16 + frow) * OPITCH + lc) = q;
                }
            }
            __syncthreads();
            constexpr int CPRO = BN / 8;    // 16-byte chunks per tile row
            for (int q = tid; q < BM * CPRO; q += NT) {
                const int lr = q / CPRO, c8 = q - lr * CPRO;
                const int row = bm + lr, col = bn + c8 * 8;
                if (row >= g.M || col >= g.N) continue;
                const u32x4 val = *reinterpret_cast<const u32x4*>(sm + lr * OPITCH + c8 * 8);
                bf16* dst = col >= e.split ? static_cast<bf16*>(e.out2) + (int64_t)row * e.ldo2 + (col - e.split + e.off2)
                                           : static_cast<bf16*>(e.out) + (int64_t)row * e.ldo + col;
                *reinterpret_cast<u32x4*>(dst) = val;
            }
            return;
        }
    }
    epilogue_t<EPI, TM, TN>(g, acc, bm + wm * TM * 16, bn + wn * TN * 16, lane);
}

// ---------------------------------------------------------------------------
// Phased bf16 kernel: the large tiles, whose loads are spread over the whole
// k-step.
//
// With two whole stages and one barrier per k-step (the wide kernel above) all
// loads of a stage go out at once and must all be back one step later, and the
// fragment reads of a step cannot start before its barrier: on 14 566 x 3072 x
// 15 360 the loads alone took 1058 us of the kernel's 1187.  Here a stage is
// cut into A halves of 128 rows and W parts of 128 or 96 rows, a wave's output
// is its share of every (half, part), and a step runs through these pairs in
// an order in which each keeps one of the last pair's operands in registers.
// The fragments of the next pair are read under the MFMAs of the present one,
// and a half or part is loaded again, for the step after the next, as soon as
// every wave has read it: 1.5 to 1.75 steps of loads are always on their way,
// and no wait drains them.  Eight waves (two per SIMD) of 128 x 64 (256 x 256
// tiles: A0 W0, A0 W1, A1 W1, A1 W0) or 64 x 144 (256 x 288: A0 W0, A1 W0,
// A1 W1, A0 W1, A0 W2, A1 W2), 24 or 26 fragment reads per 64 or 72 MFMAs.
// Same k order per output as the wide kernel, so the same bits.
// Measured against it (us): 14 566 x 21 504 x 3072 GELU 1800 -> 1495, 14 310 x
// 12 288 x 3072 GELU 921 -> 825, 14 566 x 3072 x 15 360 gated 1266 -> 1070,
// 14 310 x 3072 x 3072 gated 307 -> 276; with 256 x 288 tiles 16 384 x 1152 x
// 4608 gated 172 -> 155, 16 384 x 4608 x 1152 GELU 172 -> 169.  What bounds it
// now: the MFMAs are busy 0.65 to 0.67 of a video GEMM's cycles (counters, with
// prologue and epilogue), at the 1.8 to 1.9 GHz that the card's power leaves
// them; at K = 1152, where every round has 18 steps, 0.35 to 0.42.
// (32 x 32 x 16 MFMAs in the same phases: 10 % slower, two accumulators per
// phase being too short a chain; s_setprio around the MFMAs, or the reads all
// ahead of them: 3 to 8 % slower.)
// Needs at least two k-steps, and offsets within a tile below 4 GB.
// ---------------------------------------------------------------------------
enum PhaseStep { PH_MAIN = 0, PH_LAST2 = 1, PH_LAST = 2 };

// NP column parts per tile: 2 for 256 x 256, 3 for 256 x 288.
template <int NP> struct PhaseTile;
template <> struct PhaseTile<2> { static constexpr int BN = 256, WAVES_M = 2, WAVES_N = 4; };
template <> struct PhaseTile<3> { static constexpr int BN = 288, WAVES_M = 4, WAVES_N = 2; };

template <int EPI, int NP>
__device__ __forceinline__ void gemm_phase_body(const GemmArgs& g, int tile) {
    typedef PhaseTile<NP> PT;
    typedef Mma<bf16> MM;
    constexpr int BM = 256, BN = PT::BN, BK = 64;
    constexpr int WAVES_M = PT::WAVES_M, WAVES_N = PT::WAVES_N;
    constexpr int AH = 128, BP = BN / NP;                      // rows of an A half, of a W part
    constexpr int TM = AH / WAVES_M / 16, TN = BP / WAVES_N / 16;   // a wave's 16 x 16 blocks in one (half, part)
    static_assert(TM * WAVES_M * 16 == AH && TN * WAVES_N * 16 == BP, "tile split");
    constexpr int ABYTES = AH * 128, BBYTES = BP * 128;
    constexpr int OPITCH = BN + 8, STAGES = 2 * (2 * ABYTES + NP * BBYTES);
    constexpr int SMEM = BM * OPITCH * 2 > STAGES ? BM * OPITCH * 2 : STAGES;
    __shared__ __attribute__((aligned(1024))) char sm[SMEM];
    typedef __attribute__((address_space(3))) const char lds_char;
    typedef __attribute__((address_space(3))) const u32x4 lds_u32x4;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WAVES_N, wn = wave % WAVES_N;
    const int frow = lane % 16, grp = lane / 16;

    const int tiles_m = (g.M + BM - 1) / BM;
    const int tiles_n = (g.N + BN - 1) / BN;
    constexpr int GROUP_M = 8;
    const int group = GROUP_M * tiles_n;
    const int first_m = (tile / group) * GROUP_M;
    const int gm = min(tiles_m - first_m, GROUP_M);
    const int tm = first_m + (tile % group) % gm;
    const int tn = (tile % group) / gm;
    const int bm = tm * BM, bn = tn * BN;

    // LDS: the A halves, then the W parts, each for even and odd k-steps side
    // by side; rows of 128 bytes, 16-byte chunk c of row r in slot
    // c ^ ((r >> 1) & 7).  A wave-wide load fills 8 rows: wave w takes loads w
    // and w + 8 of every half and part (the last four of a 288-column tile's
    // twelve go to waves 0-3).
    constexpr int AL = AH / 64, BL = (BP / 8 + 7) / 8;          // loads per wave: of a half, of a part (at most)
    constexpr bool EVEN = BP / 8 % 8 == 0;
    const bool more = EVEN || wave < BP / 8 % 8;                // this wave makes BL loads of a part, not BL - 1
    const uint32_t ldsw = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_char*)sm + wave * 1024);
    const char* baseA = reinterpret_cast<const char*>(static_cast<const bf16*>(g.A) + (int64_t)bm * g.lda);
    const char* baseW = reinterpret_cast<const char*>(static_cast<const bf16*>(g.W) + (int64_t)bn * g.ldw);
    uint32_t offA[2][AL], offW[NP][BL];
#pragma unroll
    for (int q = 0; q < (AL > BL ? AL : BL); ++q) {
        const int r = 64 * q + 8 * wave + (lane >> 3);
        const uint32_t ch = ((lane & 7) ^ ((r >> 1) & 7)) * 16;
#pragma unroll
        for (int h = 0; h < 2; ++h)
            if (q < AL) offA[h][q] = (uint32_t)(min(bm + AH * h + r, g.M - 1) - bm) * (uint32_t)(g.lda * 2) + ch;
#pragma unroll
        for (int p = 0; p < NP; ++p)
            if (q < BL) offW[p][q] = (uint32_t)(min(bn + BP * p + r, g.N - 1) - bn) * (uint32_t)(g.ldw * 2) + ch;
    }
    auto loadA = [&](int h, int par, int k) __attribute__((always_inline)) {
        const char* b = baseA + (int64_t)k * 128;
#pragma unroll
        for (int q = 0; q < AL; ++q) dma16s(b, offA[h][q], ldsw + (2 * h + par) * ABYTES + q * 8192);
    };
    auto loadW = [&](int p, int par, int k) __attribute__((always_inline)) {
        const char* b = baseW + (int64_t)k * 128;
#pragma unroll
        for (int q = 0; q < BL; ++q)
            if (EVEN || q + 1 < BL || more) dma16s(b, offW[p][q], ldsw + 4 * ABYTES + (2 * p + par) * BBYTES + q * 8192);
    };
    // Waits until at most A loads of A halves and B W parts (counted in loads
    // of parts) issued after the ones needed are outstanding.
    auto wait = [&](auto ac, auto bc) __attribute__((always_inline)) {
        constexpr int A = decltype(ac)::value * AL, B = decltype(bc)::value;
        if (more) wait_vmcnt<A + B * BL>();
        else wait_vmcnt<A + B * (EVEN ? BL : BL - 1)>();
    };
#define PH_WAIT(A, B) wait(std::integral_constant<int, A>{}, std::integral_constant<int, B>{})
    // Fragment addresses: a row's swizzle depends only on the row mod 16.
    lds_char *pA[2], *pW[2];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
        const uint32_t c = (uint32_t)((kk * 4 + grp) ^ ((frow >> 1) & 7)) * 16;
        pA[kk] = (lds_char*)sm + (wm * TM * 16 + frow) * 128 + c;
        pW[kk] = (lds_char*)sm + 4 * ABYTES + (wn * TN * 16 + frow) * 128 + c;
    }
    u32x4 fa[2][TM][2], fw[2][TN][2];     // [half][block][kk]; [register set][block][kk]
    auto readA = [&](int h, int par) __attribute__((always_inline)) {
#pragma unroll
        for (int kk = 0; kk < 2; ++kk)
#pragma unroll
            for (int i = 0; i < TM; ++i) fa[h][i][kk] = *(lds_u32x4*)(pA[kk] + (2 * h + par) * ABYTES + i * 16 * 128);
    };
    auto readW = [&](int p, int par, int set) __attribute__((always_inline)) {
#pragma unroll
        for (int kk = 0; kk < 2; ++kk)
#pragma unroll
            for (int j = 0; j < TN; ++j) fw[set][j][kk] = *(lds_u32x4*)(pW[kk] + (2 * p + par) * BBYTES + j * 16 * 128);
    };
    f32x4 acc[2][NP][TM][TN];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) acc[h][p][i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto mma = [&](int h, int p, int set) __attribute__((always_inline)) {
#pragma unroll
        for (int kk = 0; kk < 2; ++kk)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[h][p][i][j] = MM::mma(__builtin_bit_cast(MM::frag, fw[set][j][kk]),
                                              __builtin_bit_cast(MM::frag, fa[h][i][kk]), acc[h][p][i][j]);
    };
    auto barrier = [&]() __attribute__((always_inline)) {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    auto reads_done = [&]() __attribute__((always_inline)) { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); };
    // A phase's order: its NR fragment reads, each ahead of one MFMA, then the other MFMAs.
    constexpr int NM = 2 * TM * TN;
#define PH_ORDER(NR) do { \
        _Pragma("unroll") for (int z = 0; z < NR; ++z) { __builtin_amdgcn_sched_group_barrier(0x100, 1, 0); __builtin_amdgcn_sched_group_barrier(0x008, 1, 0); } \
        __builtin_amdgcn_sched_group_barrier(0x008, NM - NR, 0); __builtin_amdgcn_sched_barrier(0); } while (0)

    const int nk = g.K / BK;
    // One k-step on the buffers of parity PAR, which is also the register set
    // that holds the step's first W part.
    auto step = [&](int k, auto parc, auto modec) __attribute__((always_inline)) {
        constexpr int PAR = decltype(parc)::value, MODE = decltype(modec)::value;
        constexpr bool MAIN = MODE == PH_MAIN;
        if constexpr (NP == 2) {
            if (MAIN) loadA(0, PAR, k + 2);
            readW(1, PAR, PAR ^ 1);
            mma(0, 0, PAR);
            PH_ORDER(2 * TN);
            if (MAIN) PH_WAIT(3, 2); else if (MODE == PH_LAST2) PH_WAIT(2, 2); else PH_WAIT(0, 0);
            barrier();
            if (MAIN) loadW(0, PAR, k + 2);
            readA(1, PAR);
            mma(0, 1, PAR ^ 1);
            PH_ORDER(2 * TM);
            barrier();
            if (MAIN) loadW(1, PAR, k + 2);
            mma(1, 1, PAR ^ 1);
            if (MODE == PH_LAST) {
                mma(1, 0, PAR);
                return;
            }
            __builtin_amdgcn_sched_barrier(0);
            if (MAIN) PH_WAIT(2, 3); else PH_WAIT(1, 1);
            barrier();
            if (MAIN) loadA(1, PAR, k + 2);
            readW(0, PAR ^ 1, PAR ^ 1);
            readA(0, PAR ^ 1);
            mma(1, 0, PAR);
            PH_ORDER(2 * (TM + TN));
            if (MAIN) PH_WAIT(3, 2); else PH_WAIT(1, 0);
            reads_done();
            barrier();
        } else {
            if (MAIN) loadA(0, PAR, k + 2);
            readA(1, PAR);
            mma(0, 0, PAR);
            PH_ORDER(2 * TM);
            if (MAIN) PH_WAIT(3, 4); else if (MODE == PH_LAST2) PH_WAIT(2, 4); else PH_WAIT(0, 1);
            reads_done();
            barrier();
            if (MAIN) loadW(0, PAR, k + 2);
            readW(1, PAR, PAR ^ 1);
            mma(1, 0, PAR);
            PH_ORDER(2 * TN);
            if (MAIN) loadA(1, PAR, k + 2);
            mma(1, 1, PAR ^ 1);
            __builtin_amdgcn_sched_barrier(0);
            if (MAIN) PH_WAIT(4, 4); else if (MODE == PH_LAST2) PH_WAIT(2, 3); else PH_WAIT(0, 0);
            barrier();
            if (MAIN) loadW(1, PAR, k + 2);
            readW(2, PAR, PAR);
            mma(0, 1, PAR ^ 1);
            PH_ORDER(2 * TN);
            mma(0, 2, PAR);
            if (MODE == PH_LAST) {
                mma(1, 2, PAR);
                return;
            }
            __builtin_amdgcn_sched_barrier(0);
            if (MAIN) PH_WAIT(3, 4); else PH_WAIT(1, 2);
            barrier();
            if (MAIN) loadW(2, PAR, k + 2);
            readW(0, PAR ^ 1, PAR ^ 1);
            readA(0, PAR ^ 1);
            mma(1, 2, PAR);
            PH_ORDER(2 * (TM + TN));
            if (MAIN) PH_WAIT(2, 5); else PH_WAIT(0, 2);
            reads_done();
            barrier();
        }
    };
    typedef std::integral_constant<int, 0> C0;
    typedef std::integral_constant<int, 1> C1;
    typedef std::integral_constant<int, 2> C2;
    auto load_step = [&](auto parc, int k) __attribute__((always_inline)) {
        constexpr int PAR = decltype(parc)::value;
        loadA(0, PAR, k);
        loadW(0, PAR, k);
        if constexpr (NP == 2) {
            loadW(1, PAR, k);
            loadA(1, PAR, k);
        } else {
            loadA(1, PAR, k);
            loadW(1, PAR, k);
            loadW(2, PAR, k);
        }
    };
    auto first = [&](auto parc) __attribute__((always_inline)) {
        constexpr int PAR = decltype(parc)::value;
        load_step(parc, 0);
        load_step(std::integral_constant<int, PAR ^ 1>{}, 1);
        if constexpr (NP == 2) PH_WAIT(3, 2); else PH_WAIT(2, 5);
        barrier();
        readA(0, PAR);
        readW(0, PAR, PAR);
        reads_done();
        barrier();
    };
    // An odd number of steps starts on the odd buffers, so that the last two
    // steps always run on the even, then the odd ones.
    const int odd = nk & 1;
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
#undef PH_ORDER
#undef PH_WAIT

    // A lane holds, of each block, four consecutive columns of one row.
    const GemmEpi& e = g.e;
    const bf16* __restrict__ bias = static_cast<const bf16*>(e.bias);
    auto lrow_of = [&](int h, int i) __attribute__((always_inline)) { return AH * h + (wm * TM + i) * 16 + frow; };
    auto lcol_of = [&](int p, int j) __attribute__((always_inline)) { return BP * p + (wn * TN + j) * 16 + 4 * grp; };
    auto bias4 = [&](int col, float (&bv)[4]) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < 4; ++r) bv[r] = 0.f;
        if (bias && col < g.N) {
            const bf16x4 b4 = *reinterpret_cast<const bf16x4*>(bias + col);
#pragma unroll
            for (int r = 0; r < 4; ++r) bv[r] = (float)b4[r];
        }
    };
    if constexpr (EPI == BC_EPI_GATE_RES) {
        // Straight from the accumulators, one (half, part) after the other,
        // the residual of the next one requested before the present one is
        // stored: the stream is updated in place, so no load is moved
        // over a store by itself.
        f32x4 rv[2][TM][TN], gv[TN];
        // One sample's gate for the whole tile (else read row by row).
        const bool one_gate = e.gate && bm / e.rows_per_gate == min(bm + BM - 1, g.M - 1) / e.rows_per_gate;
        auto fetch = [&](int u) __attribute__((always_inline)) {
            const int h = u / NP, p = u % NP;
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int col = min(bn + lcol_of(p, j), g.N - 4);
#pragma unroll
                for (int i = 0; i < TM; ++i)
                    rv[u & 1][i][j] = *reinterpret_cast<const f32x4*>(e.res + (int64_t)min(bm + lrow_of(h, i), g.M - 1) * e.ldr + col);
            }
        };
        fetch(0);
#pragma unroll
        for (int u = 0; u < 2 * NP; ++u) {
            const int h = u / NP, p = u % NP;
            if (u + 1 < 2 * NP) fetch(u + 1);
            if (one_gate) {
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    gv[j] = *reinterpret_cast<const f32x4*>(e.gate + (int64_t)(bm / e.rows_per_gate) * e.ldg + min(bn + lcol_of(p, j), g.N - 4));
            }
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const int row = bm + lrow_of(h, i);
                const int b = row / e.seg, sidx = row - b * e.seg;
                const bool row_ok = row < g.M && sidx < e.keep;
                const int64_t orow = (int64_t)(b * e.keep + sidx) * e.ldo;
                const float* grow = e.gate && !one_gate && row_ok ? e.gate + (int64_t)(row / e.rows_per_gate) * e.ldg : nullptr;
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    const int col = bn + lcol_of(p, j);
                    if (!row_ok || col >= g.N) continue;
                    float bv[4], v[4];
                    bias4(col, bv);
                    const f32x4 gt = one_gate ? gv[j] : grow ? *reinterpret_cast<const f32x4*>(grow + col)
                                                                    : f32x4{1.f, 1.f, 1.f, 1.f};
#pragma unroll
                    for (int r = 0; r < 4; ++r) v[r] = rv[u & 1][i][j][r] + gt[r] * (acc[h][p][i][j][r] + bv[r]);
                    if (e.out_f32) st4(static_cast<float*>(e.out) + orow + col, v);
                    else st4(static_cast<bf16*>(e.out) + orow + col, v);
                }
            }
        }
    } else {
        // The bias kind.  bf16: as in gemm_wide_kernel the finished tile goes
        // through LDS, row-major, and leaves as consecutive 16-byte chunks of
        // its rows.  fp32: straight from the accumulators.
        bf16* so = reinterpret_cast<bf16*>(sm);
        __syncthreads();   // every wave is done with the stage buffers
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int lc = lcol_of(p, j), col = bn + lc;
                float bv[4];
                bias4(col, bv);
                const bool act = col >= e.gelu_from;
                const float qs = col < e.q_scale_to ? e.q_scale : 1.f;
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int i = 0; i < TM; ++i) {
                        float v[4];
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            v[r] = (acc[h][p][i][j][r] + bv[r]) * qs;
                            if (act) v[r] = gelu_tanh(v[r]);
                        }
                        const int lr = lrow_of(h, i);
                        if (!e.out_f32) st4(so + lr * OPITCH + lc, v);
                        else if (bm + lr < g.M && col < g.N) {     // (the split part is in the operand dtype)
                            if (col >= e.split) st4(static_cast<bf16*>(e.out2) + (int64_t)(bm + lr) * e.ldo2 + (col - e.split + e.off2), v);
                            else st4(static_cast<float*>(e.out) + (int64_t)(bm + lr) * e.ldo + col, v);
                        }
                    }
            }
        if (e.out_f32) return;
        __syncthreads();
        constexpr int CPRO = BN / 8;
#pragma unroll 4
        for (int q = tid; q < BM * CPRO; q += 512) {
            const int lr = q / CPRO, c8 = q - lr * CPRO;
            const int row = bm + lr, col = bn + c8 * 8;
            if (row >= g.M || col >= g.N) continue;
            const u32x4 val = *reinterpret_cast<const u32x4*>(so + lr * OPITCH + c8 * 8);
            bf16* dst = col >= e.split ? static_cast<bf16*>(e.out2) + (int64_t)row * e.ldo2 + (col - e.split + e.off2)
                                       : static_cast<bf16*>(e.out) + (int64_t)row * e.ldo + col;
            *reinterpret_cast<u32x4*>(dst) = val;
        }
    }
}

template <int EPI, int NP>
__global__ __launch_bounds__(512) void gemm_phase_kernel(GemmArgs g) {
    gemm_phase_body<EPI, NP>(g, xcd_contiguous(blockIdx.x, gridDim.x));
}

// Two GEMMs in one grid: workgroups [0, tiles0) take the first (in the
// XCD-contiguous order over its own tiles), the rest the second, whose
// workgroups come last and are dealt round-robin to the XCDs, so its tiles
// fill the first one's last round.
template <int EPI>
__global__ __launch_bounds__(512) void gemm_phase_pair_kernel(GemmArgs g0, GemmArgs g1, int tiles0) {
    const int b = blockIdx.x;
    const bool second = b >= tiles0;
    gemm_phase_body<EPI, 2>(second ? g1 : g0, second ? b - tiles0 : xcd_contiguous(b, tiles0));
}

template <int EPI, int NP>
static void launch_phase(const GemmArgs& g, hipStream_t s) {
    constexpr int BN = PhaseTile<NP>::BN;
    launch_k(gemm_phase_kernel<EPI, NP>, dim3((unsigned)(((g.M + 255) / 256) * ((g.N + BN - 1) / BN))), dim3(512), s, g);
}

template <int EPI, int BM, int BN, int WAVES_M, int WAVES_N, bool AHEAD = false>
static void launch_wide(const GemmArgs& g, hipStream_t s) {
    const unsigned tiles = (unsigned)(((g.M + BM - 1) / BM) * ((g.N + BN - 1) / BN));
    launch_k(gemm_wide_kernel<EPI, BM, BN, WAVES_M, WAVES_N, AHEAD>, dim3(tiles), dim3(64 * WAVES_M * WAVES_N), s, g);
}

template <int EPI, int BM, int BN, int WAVES_M, int WAVES_N, int STAGES>
__global__ __launch_bounds__(64 * WAVES_M * WAVES_N) void gemm_dma_kernel(GemmArgs g) {
    gemm_dma_body<EPI, BM, BN, WAVES_M, WAVES_N, STAGES, false>(g, nullptr);
}

template <int EPI, int BM, int BN, int WAVES_M, int WAVES_N, int STAGES>
__global__ __launch_bounds__(64 * WAVES_M * WAVES_N) void gemm_dma_seg_kernel(GemmArgs g, GemmSeg sg) {
    gemm_dma_body<EPI, BM, BN, WAVES_M, WAVES_N, STAGES, true>(g, &sg);
}

template <int EPI, int BM, int BN, int WAVES_M, int WAVES_N, int STAGES>
static void launch_dma(const GemmArgs& g, hipStream_t s) {
    const unsigned tiles = (unsigned)(((g.M + BM - 1) / BM) * ((g.N + BN - 1) / BN));
    launch_k(gemm_dma_kernel<EPI, BM, BN, WAVES_M, WAVES_N, STAGES>, dim3(tiles), dim3(64 * WAVES_M * WAVES_N), s, g);
}

// ---------------------------------------------------------------------------
// Small grids: K split over the waves of a workgroup.
//
// With few rows the tiles above leave most CUs idle and walk all of K as one
// serial chain of loads, barrier and MFMAs (M = 256, N = 1152, K = 4608: 16
// workgroups, 72 steps, 46 us).  Here a tile is small, and each of the 8 waves
// accumulates all of it over k-steps of its own (wave w takes steps w, w + 8,
// ...; a step is 128 bytes of every operand row), loaded straight into a stage
// that only this wave uses and loaded again as soon as it has been read: the
// loads of the waves keep each other company, and no barrier stops them until
// the partial tiles meet in LDS, in a fixed order, for the epilogue.  What
// bounds it is what a CU's loads deliver, about 64 GB/s, so the time is close to
// (rounds of workgroups) (BM + BN) K bytes over that: 10.6 us for the shape
// above.  (Fragments loaded from global memory straight into registers, without
// the trip through LDS, ran at a third of that: the 16 lanes of a fragment row
// fetch from 16 rows, 16 bytes each.)
// Any N and alignment of the outputs (vec: 4-column accesses are possible).
// ---------------------------------------------------------------------------
constexpr int kKsWaves = 8;

template <typename T> struct KsMma;
template <> struct KsMma<bf16> {
    __device__ static __forceinline__ f32x4 mma(const u32x4& w, const u32x4& a, const f32x4& c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w), __builtin_bit_cast(bf16x8, a), c, 0, 0, 0);
    }
};
// fp32: instruction i takes element i of every lane, k = 4 (l / 16) + i.
template <> struct KsMma<float> {
    __device__ static __forceinline__ f32x4 mma(const u32x4& w, const u32x4& a, f32x4 c) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(w[i]), __uint_as_float(a[i]), c, 0, 0, 0);
        return c;
    }
};

// The epilogue of four consecutive columns of one row (see GemmEpi); columns
// past N are dropped.
template <typename T, int EPI>
__device__ __forceinline__ void finish4(const GemmArgs& g, int row, int col, const f32x4& acc, bool vec) {
    const GemmEpi& e = g.e;
    const T* bias = static_cast<const T*>(e.bias);
    if constexpr (EPI == BC_EPI_GATE_RES) {
        const int b = row / e.seg, sidx = row - b * e.seg;
        if (sidx >= e.keep) return;
        const int64_t o = (int64_t)(b * e.keep + sidx) * e.ldo + col;
        const float* res = e.res + (int64_t)row * e.ldr + col;
        const float* gate = e.gate ? e.gate + (int64_t)(row / e.rows_per_gate) * e.ldg + col : nullptr;
        float v[4];
        if (vec) {
            const f32x4 rv = *reinterpret_cast<const f32x4*>(res);
            const f32x4 gv = gate ? *reinterpret_cast<const f32x4*>(gate) : f32x4{1.f, 1.f, 1.f, 1.f};
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = rv[r] + gv[r] * (acc[r] + (bias ? ld(bias + col + r) : 0.f));
            if (e.out_f32) st4(static_cast<float*>(e.out) + o, v);
            else if constexpr (sizeof(T) == 2) st4(static_cast<bf16*>(e.out) + o, v);
            return;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if (col + r >= g.N) break;
            const float y = res[r] + (gate ? gate[r] : 1.f) * (acc[r] + (bias ? ld(bias + col + r) : 0.f));
            if (e.out_f32) static_cast<float*>(e.out)[o + r] = y;
            else st(static_cast<T*>(e.out) + o + r, y);
        }
    } else {
        float v[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            v[r] = acc[r] + (bias && col + r < g.N ? ld(bias + col + r) : 0.f);
            if (col + r < e.q_scale_to) v[r] *= e.q_scale;
            if (col + r >= e.gelu_from) v[r] = gelu_tanh(v[r]);
        }
        if (vec) {     // the boundaries are multiples of 4: all four columns go one way
            if (col >= e.split) st4(static_cast<T*>(e.out2) + (int64_t)row * e.ldo2 + (col - e.split + e.off2), v);
            else if (e.out_f32) st4(static_cast<float*>(e.out) + (int64_t)row * e.ldo + col, v);
            else st4(static_cast<T*>(e.out) + (int64_t)row * e.ldo + col, v);
            return;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int c = col + r;
            if (c >= g.N) break;
            if (c >= e.split) st(static_cast<T*>(e.out2) + (int64_t)row * e.ldo2 + (c - e.split + e.off2), v[r]);
            else if (e.out_f32) static_cast<float*>(e.out)[(int64_t)row * e.ldo + c] = v[r];
            else st(static_cast<T*>(e.out) + (int64_t)row * e.ldo + c, v[r]);
        }
    }
}

template <typename T_, int EPI, int TM, int TN>
__global__ __launch_bounds__(64 * kKsWaves) void gemm_ksplit_kernel(GemmArgs g, int vec) {
    typedef elem_t<T_> T;
    typedef KsMma<T> MM;
    constexpr int WK = kKsWaves, BM = 16 * TM, BN = 16 * TN, PITCH = BN + 4;
    constexpr int BK = 128 / (int)sizeof(T);               // k per step: 128 bytes of every row
    constexpr int Q = (BM + BN) / 8;                       // wave-wide loads per step
    constexpr int STAGE = (BM + BN) * 128;
    // Partial tiles held in LDS at once: all of them, or half of them.
    constexpr int SLOT = BM * PITCH;
    constexpr int NS = SLOT * 4 <= STAGE ? WK : WK / 2;
    static_assert(NS * SLOT * 4 <= WK * STAGE && WK * STAGE <= 160 * 1024, "LDS");
    __shared__ __attribute__((aligned(1024))) char sm[WK * STAGE];
    typedef __attribute__((address_space(3))) const char lds_char;
    typedef __attribute__((address_space(3))) const u32x4 lds_u32x4;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r16 = lane & 15, grp = lane >> 4;
    // Row tiles fastest: the workgroups that share a column tile's weights are neighbours on one XCD.
    const int tiles_m = (g.M + BM - 1) / BM;
    const int pid = xcd_contiguous(blockIdx.x, gridDim.x);
    const int bm = pid % tiles_m * BM, bn = pid / tiles_m * BN;
    const char* baseA = reinterpret_cast<const char*>(static_cast<const T*>(g.A) + (int64_t)bm * g.lda);
    const char* baseW = reinterpret_cast<const char*>(static_cast<const T*>(g.W) + (int64_t)bn * g.ldw);
    uint32_t voff[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int r = 8 * q + (lane >> 3);
        const uint32_t ch = ((lane & 7) ^ ((r >> 1) & 7)) * 16;
        voff[q] = r < BM ? (uint32_t)(min(bm + r, g.M - 1) - bm) * (uint32_t)(g.lda * sizeof(T)) + ch
                         : (uint32_t)(min(bn + r - BM, g.N - 1) - bn) * (uint32_t)(g.ldw * sizeof(T)) + ch;
    }
    const uint32_t stage = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_char*)sm + wave * STAGE);
    // Step i of this wave is k-step wave + WK i.
    const int nk = g.K / BK;
    const int n = nk > wave ? (nk - wave + WK - 1) / WK : 0;
    auto issue = [&](int i) __attribute__((always_inline)) {
        const int64_t k = (int64_t)(wave + WK * i) * 128;
#pragma unroll
        for (int q = 0; q < Q; ++q) dma16s((8 * q < BM ? baseA : baseW) + k, voff[q], stage + q * 1024);
    };
    lds_char* frag[2];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
        frag[kk] = (lds_char*)sm + wave * STAGE + r16 * 128 + ((kk * 4 + grp) ^ ((r16 >> 1) & 7)) * 16;
    f32x4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (n > 0) issue(0);
    for (int i = 0; i < n; ++i) {
        wait_vmcnt<0>();       // step i has landed
        asm volatile("" ::: "memory");
        u32x4 fa[2][TM], fw[2][TN];
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
#pragma unroll
            for (int j = 0; j < TN; ++j) fw[kk][j] = *(lds_u32x4*)(frag[kk] + (BM + 16 * j) * 128);
#pragma unroll
            for (int m = 0; m < TM; ++m) fa[kk][m] = *(lds_u32x4*)(frag[kk] + 16 * m * 128);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // read before the stage is filled again
        if (i + 1 < n) issue(i + 1);
#pragma unroll
        for (int kk = 0; kk < 2; ++kk)
#pragma unroll
            for (int m = 0; m < TM; ++m)
#pragma unroll
                for (int j = 0; j < TN; ++j) acc[m][j] = MM::mma(fw[kk][j], fa[kk][m], acc[m][j]);
    }
    __syncthreads();      // the partial tiles take the stages' place
    float* red = reinterpret_cast<float*>(sm);
    // Partial tiles to LDS: the last NS waves store, the NS before them (if any) add.
#pragma unroll
    for (int r = WK / NS - 1; r >= 0; --r) {
        if (wave / NS == r) {
            float* slot = red + (wave % NS) * SLOT;
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    f32x4* d = reinterpret_cast<f32x4*>(slot + (16 * i + r16) * PITCH + 16 * j + 4 * grp);
                    *d = r == WK / NS - 1 ? acc[i][j] : *d + acc[i][j];
                }
        }
        __syncthreads();
    }
    constexpr int C4 = BN / 4;
    for (int q = tid; q < BM * C4; q += 64 * WK) {
        const int lr = q / C4, lc = (q - lr * C4) * 4;
        const int row = bm + lr, col = bn + lc;
        if (row >= g.M || col >= g.N) continue;
        f32x4 sum = *reinterpret_cast<const f32x4*>(red + lr * PITCH + lc);
#pragma unroll
        for (int w = 1; w < NS; ++w) sum += *reinterpret_cast<const f32x4*>(red + w * SLOT + lr * PITCH + lc);
        finish4<T, EPI>(g, row, col, sum, vec != 0);
    }
}

template <typename T, int EPI, int TM, int TN>
static void launch_ksplit(const GemmArgs& g, bool vec, hipStream_t s) {
    const unsigned tiles = (unsigned)(((g.M + 16 * TM - 1) / (16 * TM)) * ((g.N + 16 * TN - 1) / (16 * TN)));
    launch_k(gemm_ksplit_kernel<tag_t<T>, EPI, TM, TN>, dim3(tiles), dim3(64 * kKsWaves), s, g, vec ? 1 : 0);
}

// Whether every column index, stride and boundary of the epilogue is a
// multiple of 4 elements and its pointers allow accesses of that width.
static bool vec4_ok(const GemmArgs& g, int epi) {
    const GemmEpi& e = g.e;
    auto al = [](const void* p) { return reinterpret_cast<uintptr_t>(p) % 16 == 0; };
    if (g.N % 4 || e.ldo % 4 || !al(e.out)) return false;
    if (epi == BC_EPI_GATE_RES) return e.ldr % 4 == 0 && al(e.res) && (!e.gate || (e.ldg % 4 == 0 && al(e.gate)));
    return e.split >= g.N || (e.split % 4 == 0 && e.off2 % 4 == 0 && e.ldo2 % 4 == 0 && al(e.out2));
}

// ---------------------------------------------------------------------------
// 128 x 144 and 128 x 192 tiles for grids of at most one round (the N = 1152
// projections at M = 4096; the video model's N = 3072 at one frame).
//
// What bounds these shapes is what a CU can load (35 KB a k-step at about 64
// GB/s) and read back from LDS: 16 waves of 32 x 48 and 32 x 32 read 139 KB of
// fragments a step for 576 cycles of MFMAs.  Here twelve (sixteen) waves, three
// (four) per SIMD, are two groups of 2 x 3 (2 x 4) waves of 64 x 48, each group
// taking one half of every k-step: 86 KB of fragments a step, read one step ahead of their MFMAs, four
// stages of loads, one barrier a step; the groups' halves meet in LDS at the
// end.  M = 4096, N = 1152, K = 4608, gated: 58.1 us with the sixteen waves,
// 48.9 now (M = 2048: 49.6 and 39.1); K = 1152: 21.1 and 20.0.  128 x 192:
// M = 1846, N = 3072, K = 15 360, gated: 171 us against 217 with
// 128 x 128 (two rounds of loads on the CUs that get two); K = 3072: 43 and 50.
// ---------------------------------------------------------------------------
template <int EPI, int BN>
__global__ __launch_bounds__(64 * (BN / 12)) void gemm_mid_kernel(GemmArgs g) {
    typedef Mma<bf16> MM;
    constexpr int BM = 128, STAGE = (BM + BN) * 128, S = 4;
    constexpr int TM = 4, TN = 3, WN = BN / 48, NW = 4 * WN, NT = 64 * NW, NOCT = (BM + BN) / 8, Q = (NOCT + NW - 1) / NW;   // Q: loads per wave and step (at most)
    constexpr int PITCH = BN + 4;
    static_assert(BM * PITCH * 4 <= S * STAGE, "the reduced tile fits the stages");
    __shared__ __attribute__((aligned(1024))) char sm[S * STAGE];
    typedef __attribute__((address_space(3))) const char lds_char;
    typedef __attribute__((address_space(3))) const u32x4 lds_u32x4;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kg = wave / (2 * WN), wig = wave % (2 * WN), wm = wig / WN, wn = wig % WN;
    const int frow = lane & 15, grp = lane >> 4;
    const int tiles_m = (g.M + BM - 1) / BM, tiles_n = (g.N + BN - 1) / BN;
    const int tile = xcd_contiguous(blockIdx.x, gridDim.x);
    constexpr int GROUP_M = 8;
    const int group = GROUP_M * tiles_n;
    const int first_m = (tile / group) * GROUP_M;
    const int gm = min(tiles_m - first_m, GROUP_M);
    const int bm = (first_m + (tile % group) % gm) * BM, bn = (tile % group) / gm * BN;

    const char* baseA = reinterpret_cast<const char*>(static_cast<const bf16*>(g.A) + (int64_t)bm * g.lda);
    const char* baseW = reinterpret_cast<const char*>(static_cast<const bf16*>(g.W) + (int64_t)bn * g.ldw);
    // Load o = wave + NW q of a step fills rows 8 o .. 8 o + 7 of the stage (A rows, then W rows).
    const bool more = NOCT % NW == 0 || wave < NOCT % NW;
    uint32_t off[Q];
    const char* base[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int o = min(wave + NW * q, NOCT - 1), r = 8 * o + (lane >> 3);
        const uint32_t ch = ((lane & 7) ^ ((r >> 1) & 7)) * 16;
        base[q] = 8 * o < BM ? baseA : baseW;
        off[q] = 8 * o < BM ? (uint32_t)(min(bm + r, g.M - 1) - bm) * (uint32_t)(g.lda * 2) + ch
                            : (uint32_t)(min(bn + r - BM, g.N - 1) - bn) * (uint32_t)(g.ldw * 2) + ch;
    }
    const uint32_t ldsw = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_char*)sm + wave * 1024);
    auto issue = [&](int k, int st) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < Q; ++q)
            if (q + 1 < Q || more) dma16s(base[q] + (int64_t)k * 128, off[q], ldsw + st * STAGE + q * NW * 1024);
    };
    auto wait_steps = [&](int later) __attribute__((always_inline)) {      // at most `later` (0 to 2) steps' loads outstanding
        if (more) wait_groups<Q, 2>(later);
        else wait_groups<Q - 1, 2>(later);
    };
    const uint32_t c = (uint32_t)((kg * 4 + grp) ^ ((frow >> 1) & 7)) * 16;
    lds_char* pA = (lds_char*)sm + (wm * 64 + frow) * 128 + c;
    lds_char* pW = (lds_char*)sm + (BM + wn * 48 + frow) * 128 + c;
    // Fragments one step ahead of their MFMAs where the registers allow it (three
    // waves per SIMD; four hide the reads by themselves).
    constexpr bool AHEAD = NW == 12;
    u32x4 fa[AHEAD ? 2 : 1][TM], fw[AHEAD ? 2 : 1][TN];
    auto read = [&](int st, int set) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < TN; ++j) fw[set][j] = *(lds_u32x4*)(pW + st * STAGE + j * 2048);
#pragma unroll
        for (int i = 0; i < TM; ++i) fa[set][i] = *(lds_u32x4*)(pA + st * STAGE + i * 2048);
    };
    f32x4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto mma = [&](int set) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
                acc[i][j] = MM::mma(__builtin_bit_cast(MM::frag, fw[set][j]), __builtin_bit_cast(MM::frag, fa[set][i]), acc[i][j]);
    };
    auto barrier = [&]() __attribute__((always_inline)) {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    const int nk = g.K / 64;
    // Step k, in stage ST.  After the barrier the step that is read next (k, or k
    // + 1 when reading ahead) has landed for every wave, and every wave is done
    // with the fragments of step k - 1, whose stage step k + 3 takes.
    auto step = [&](int k, auto stc) __attribute__((always_inline)) {
        constexpr int ST = decltype(stc)::value;
        if constexpr (AHEAD) {
            if (k + 1 >= nk) {
                mma(ST & 1);
                return;
            }
            wait_steps(min(1, nk - 2 - k));
            barrier();
            if (k + 3 < nk) issue(k + 3, (ST + 3) % 4);
            read((ST + 1) % 4, (ST + 1) & 1);
            mma(ST & 1);
#pragma unroll
            for (int z = 0; z < TM + TN; ++z) {
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            }
            __builtin_amdgcn_sched_group_barrier(0x008, TM * TN - TM - TN, 0);
            __builtin_amdgcn_sched_barrier(0);
        } else {
            wait_steps(min(2, nk - 1 - k));
            barrier();
            if (k + 3 < nk) issue(k + 3, (ST + 3) % 4);
            read(ST, 0);
            mma(0);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
#pragma unroll
    for (int p = 0; p < 3; ++p)
        if (p < nk) issue(p, p);
    if constexpr (AHEAD) {
        wait_steps(min(2, nk - 1));
        barrier();
        read(0, 0);
    }
    int k = 0;
    for (; k + 4 <= nk; k += 4) {
        step(k, std::integral_constant<int, 0>{});
        step(k + 1, std::integral_constant<int, 1>{});
        step(k + 2, std::integral_constant<int, 2>{});
        step(k + 3, std::integral_constant<int, 3>{});
    }
    if (k < nk) step(k, std::integral_constant<int, 0>{});
    if (k + 1 < nk) step(k + 1, std::integral_constant<int, 1>{});
    if (k + 2 < nk) step(k + 2, std::integral_constant<int, 2>{});

    // The residual is on its way while the two groups' halves meet in LDS (group
    // 1's first, then group 0 adds its own); all waves then finish whole rows.
    constexpr int C4 = BN / 4, IT = BM * C4 / NT;
    static_assert(IT * NT == BM * C4, "chunks per thread");
    f32x4 rv[EPI == BC_EPI_GATE_RES ? IT : 1];
    if constexpr (EPI == BC_EPI_GATE_RES) {
#pragma unroll
        for (int t = 0; t < IT; ++t) {
            const int q = tid + NT * t, row = min(bm + q / C4, g.M - 1), col = min(bn + q % C4 * 4, g.N - 4);
            rv[t] = *reinterpret_cast<const f32x4*>(g.e.res + (int64_t)row * g.e.ldr + col);
        }
    }
    float* ft = reinterpret_cast<float*>(sm);
    __syncthreads();
#pragma unroll
    for (int pass = 1; pass >= 0; --pass) {
        if (kg == pass) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    f32x4* d = reinterpret_cast<f32x4*>(ft + (wm * 64 + i * 16 + frow) * PITCH + wn * 48 + j * 16 + 4 * grp);
                    *d = pass == 1 ? acc[i][j] : *d + acc[i][j];
                }
        }
        __syncthreads();
    }
#pragma unroll
    for (int t = 0; t < IT; ++t) {
        const int q = tid + NT * t, lr = q / C4, lc = q % C4 * 4;
        const int row = bm + lr, col = bn + lc;
        if (row >= g.M || col >= g.N) continue;
        const f32x4 y = *reinterpret_cast<const f32x4*>(ft + lr * PITCH + lc);
        if constexpr (EPI == BC_EPI_GATE_RES) {
            gate_res4(g, row, col, y, rv[t]);
        } else {
            finish4<bf16, EPI>(g, row, col, y, true);
        }
    }
}

template <int EPI, int BN>
static void launch_mid(const GemmArgs& g, hipStream_t s) {
    launch_k(gemm_mid_kernel<EPI, BN>, dim3((unsigned)(((g.M + 127) / 128) * ((g.N + BN - 1) / BN))), dim3(64 * (BN / 12)), s, g);
}

template <typename T, int EPI, int BM, int BN, int WAVES_M, int WAVES_N>
static void launch_tile(const GemmArgs& g, hipStream_t s) {
    const unsigned tiles = (unsigned)(((g.M + BM - 1) / BM) * ((g.N + BN - 1) / BN));
    launch_k(gemm_kernel<tag_t<T>, EPI, BM, BN, WAVES_M, WAVES_N>, dim3(tiles), dim3(64 * WAVES_M * WAVES_N), s, g);
}

// The wide kernel's vector epilogue needs every column index and stride it
// touches to be a multiple of 4 and its pointers 16-byte aligned.
static bool wide_ok(const GemmArgs& g, int epi) {
    const GemmEpi& e = g.e;
    auto al = [](const void* p) { return reinterpret_cast<uintptr_t>(p) % 16 == 0; };
    if (g.K % 64 || g.lda % 8 || g.ldw % 8 || g.N % 4 || e.ldo % 4 || !al(e.out)) return false;
    if (e.bias && reinterpret_cast<uintptr_t>(e.bias) % 8) return false;
    if (epi == BC_EPI_GATE_RES) return e.ldr % 4 == 0 && al(e.res) && (!e.gate || (e.ldg % 4 == 0 && al(e.gate)));
    // The plain epilogue pairs lanes into 8-column groups: N, the split and
    // GELU boundaries and the bf16 row strides and offsets are multiples of 8.
    if (g.N % 8 || e.ldo % 8) return false;
    if (e.gelu_from < g.N && e.gelu_from % 8) return false;
    if (e.q_scale_to > 0 && e.q_scale_to % 8) return false;
    if (e.split < g.N && (e.split % 8 || e.off2 % 8 || e.ldo2 % 8 || !al(e.out2))) return false;
    return true;
}

// Column parts of the phased kernel's tile (2: 256 x 256, 3: 256 x 288), or 0
// where its tiles do not make a round over the 256 CUs (see the choice below).
// A round of 256 x 256 tiles takes about 1.34 us per k-step and 11 us for the
// prologue and epilogue, one of 256 x 288 tiles 1.58 and 14 (from K = 1152 and
// 3072 at 14 310 and 16 384 rows); the tile with the least rounds times that:
// 16 384 x 4608 x 1152 177 against 169 us (5 against 4 rounds), 5000 x 4608 x
// 1152 66 against 77 (2 rounds each).
static int phase_parts(const GemmArgs& g) {
    const int64_t tm = (g.M + 255) / 256, t256 = tm * ((g.N + 255) / 256), t288 = tm * ((g.N + 287) / 288);
    const int nk = g.K / 64;
    if (t288 < 256 || nk < 2 || (g.lda > g.ldw ? g.lda : g.ldw) > (1 << 22)) return 0;
    const double c2 = (double)((t256 + 255) / 256) * (1.34 * nk + 11), c3 = (double)((t288 + 255) / 256) * (1.58 * nk + 14);
    return c2 <= c3 ? 2 : 3;
}

// Tile choice (measured on MI355X over the DiT-XL/2, PixArt and HunyuanVideo
// block shapes), for bf16 operands with whole 64-wide
// k-steps and an epilogue the wide kernel can vectorise:
//   * at least one full round of 256 x 288 tiles over the 256 CUs: the phased
//     kernel;
//   * N a multiple of 432 with at least one round of 128 x 432 tiles (the
//     DiT-XL/2 QKV projection: exactly 256): 4 x 3 waves of 32 x 144;
//   * at most 256 tiles of 128 x 144 (the N = 1152 projections at M = 4096) and
//     K >= 1024: those (M = 4096, N = 1152, K = 1152: 20.0 us against 24.8 with
//     128 x 128 tiles; M = 3000, K = 768: 15.0 against 12.6);
//   * at most 256 tiles of 128 x 192 and K >= 1152: those (M = 2048, N = 3072, K =
//     1536: 28.5 us against 31.3; equal at K = 1152, 21.4 against 20.6 at 1024);
//   * otherwise 128 x 128 (16 waves of 32 x 32, two workgroups per CU).  Gated: the
//     two cover each other's epilogue, and a residual requested ahead of it cost
//     up to a tenth (16 000 x 384 x 384 16.4 us against 14.9, 8192 x 768 x 768 20.9
//     against 20.0, 3500 x 2304 x 768 24.3 against 22.6); only where few workgroups
//     are left for a last round, alone on their CUs, is it read ahead (528 tiles,
//     4100 x 2048 x 2048, 59.2 us against 62.1; 564, 12 000 x 768 x 768, 35.2
//     against 37.7; 624, 9900 x 1000 x 640, 33.9 against 36.7; 768 of them 44.2
//     against 43.7; and at K = 256, 549 tiles, 22.5 against 21.5).
// Other bf16 operands take the direct-to-LDS kernel with the scalar
// epilogue, or the register-staged kernel, as does fp32 with K % 32 != 0.
// Before all of these, grids too small for them go to the k-split kernel.
//
// bf16: the k-split kernel's tile is the one with the least work per CU, rounds
// of 256 workgroups times operand rows per tile (the rows are what a CU loads).
// It is taken up to 240 such rows, when 128 x 144 tiles would not fill a round:
// measured against those tiles (us, K = 1152 / 4608) 4.8 against 16.3 / 10.6
// against 45.8 at 80 rows (M = 256, N = 1152), 9.7 against 16.6 / 23.2 against
// 48.0 at 144 (M = 1020, N = 1152); at 288 rows it is 22 against 17 / 54 against
// 51 (M = 2048).
// fp32: always (the MFMA is a sixteenth as fast, so the loads hardly matter):
// 16 x 16 tiles where they make at most four rounds (M = N = 128, K = 512: 3.2 us
// against 6.3 with 32 x 48 tiles and 53 with the register-staged 128 x 128
// tile), else 32 x 48 (M = 2048, N = 1500, K = 6144: 275 us, 138 TFLOP/s, against
// 626 and 464).
template <typename T, int EPI>
static bool run_ksplit(const GemmArgs& g, hipStream_t s) {
    constexpr int BK = 128 / (int)sizeof(T);
    // Offsets within a tile are 32-bit.
    if (g.K % BK || (g.lda > g.ldw ? g.lda : g.ldw) > (1 << 20)) return false;
    auto tiles = [&](int bm, int bn) { return (int64_t)((g.M + bm - 1) / bm) * ((g.N + bn - 1) / bn); };
    const bool vec = vec4_ok(g, EPI);
    if constexpr (sizeof(T) == 4) {
        if (tiles(32, 48) > 0x7fffffff) return false;
        if (tiles(16, 16) <= 4 * 256) launch_ksplit<T, EPI, 1, 1>(g, vec, s);
        else launch_ksplit<T, EPI, 2, 3>(g, vec, s);
        return true;
    } else {
        auto rows = [&](int bm, int bn) { return (tiles(bm, bn) + 255) / 256 * (bm + bn); };
        const int64_t r[4] = {rows(32, 48), rows(64, 48), rows(64, 64), rows(64, 80)};
        int best = 0;
        for (int i = 1; i < 4; ++i)
            if (r[i] < r[best]) best = i;
        if (r[best] > 240 || tiles(128, 144) > 256) return false;
        switch (best) {
            case 0: launch_ksplit<T, EPI, 2, 3>(g, vec, s); break;
            case 1: launch_ksplit<T, EPI, 4, 3>(g, vec, s); break;
            case 2: launch_ksplit<T, EPI, 4, 4>(g, vec, s); break;
            default: launch_ksplit<T, EPI, 4, 5>(g, vec, s); break;
        }
        return true;
    }
}

template <typename T, int EPI>
static int run_gemm(const GemmArgs& g, hipStream_t s) {
    const int64_t tiles128 = (int64_t)((g.M + 127) / 128) * ((g.N + 127) / 128);
    if (tiles128 > 0x7fffffff) return fail(BC_ERR_UNSUPPORTED, "GEMM grid too large");
    if (run_ksplit<T, EPI>(g, s)) return check_launch("gemm");
    if constexpr (sizeof(T) == 2) {
        const int64_t tiles144 = (int64_t)((g.M + 127) / 128) * ((g.N + 143) / 144);
        const int64_t tiles192 = (int64_t)((g.M + 127) / 128) * ((g.N + 191) / 192);
        const bool mid = g.K >= 1024 && (g.lda > g.ldw ? g.lda : g.ldw) <= (1 << 22);
        const bool dma = g.K % 64 == 0 && g.lda % 8 == 0 && g.ldw % 8 == 0;
        if (dma && wide_ok(g, EPI)) {
            const int parts = phase_parts(g);
            if (parts == 2) {
                launch_phase<EPI, 2>(g, s);
            } else if (parts == 3) {
                launch_phase<EPI, 3>(g, s);
            } else if (g.N % 432 == 0 && (int64_t)((g.M + 127) / 128) * (g.N / 432) >= 256) {
                launch_wide<EPI, 128, 432, 4, 3>(g, s);
            } else if (tiles144 <= 256 && mid) {
                launch_mid<EPI, 144>(g, s);
            } else if (tiles192 <= 256 && mid && g.K >= 1152) {
                launch_mid<EPI, 192>(g, s);
            } else if (EPI == BC_EPI_GATE_RES && g.K >= 512 && tiles128 > 512 && (tiles128 - 1) % 512 < 128) {
                launch_wide<EPI, 128, 128, 4, 4, EPI == BC_EPI_GATE_RES>(g, s);
            } else {
                launch_wide<EPI, 128, 128, 4, 4>(g, s);
            }
        } else if (dma) {
            launch_dma<EPI, 128, 128, 4, 2, 2>(g, s);
        } else {
            launch_tile<T, EPI, 128, 128, 4, 2>(g, s);
        }
    } else {
        launch_tile<T, EPI, 128, 128, 2, 2>(g, s);
    }
    return check_launch("gemm");
}

int launch_gemm_grouped(int dtype, const GemmArgs& g0, const GemmSeg& sg, int nseg, hipStream_t s) {
    // Column segment i of the output uses weights sg.W[i] ([Nseg, K]) and bias sg.bias[i].
    if (g0.M <= 0 || nseg <= 0) return BC_OK;
    if (nseg > kMaxGemmSeg) return fail(BC_ERR_UNSUPPORTED, "%d GEMM segments", nseg);
    GemmArgs g = g0;
    g.N = nseg * sg.Nseg;
    const bool dma = dtype == BC_BF16 && g.K % 64 == 0 && g.ldw % 8 == 0 && g.lda % 8 == 0 && sg.Nseg % 128 == 0 &&
                     reinterpret_cast<uintptr_t>(g.A) % 16 == 0;
    if (dma) {
        for (int i = 0; i < nseg; ++i)
            if (reinterpret_cast<uintptr_t>(sg.W[i]) % 16) return fail(BC_ERR_UNSUPPORTED, "misaligned segment weight");
        prof_begin(PROF_GEMM_BIAS, s, 2.0 * g.M * (double)g.N * g.K);
        const unsigned tiles = (unsigned)(((g.M + 127) / 128) * (g.N / 128));
        launch_k(gemm_dma_seg_kernel<BC_EPI_BIAS, 128, 128, 4, 2, 2>, dim3(tiles), dim3(512), s, g, sg);
        prof_end(PROF_GEMM_BIAS, s);
        return check_launch("grouped gemm");
    }
    // One launch per segment, writing its column block of the output.
    for (int i = 0; i < nseg; ++i) {
        GemmArgs gi = g0;
        gi.N = sg.Nseg;
        gi.W = sg.W[i];
        gi.e.bias = sg.bias[i];
        gi.e.out = static_cast<char*>(g0.e.out) + (size_t)i * sg.Nseg * (g0.e.out_f32 ? 4 : dtype_size(dtype));
        const int rc = launch_gemm(dtype, BC_EPI_BIAS, gi, s);
        if (rc != BC_OK) return rc;
    }
    return BC_OK;
}

int launch_gemm(int dtype, int epi, const GemmArgs& g, hipStream_t s) {
    if (g.M <= 0 || g.N <= 0) return BC_OK;
    const int epc = dtype == BC_BF16 ? 8 : 4;
    if (g.K <= 0 || g.K % epc || g.lda % epc || g.ldw % epc)
        return fail(BC_ERR_UNSUPPORTED, "GEMM K=%d, lda=%lld, ldw=%lld must be multiples of %d", g.K,
                    (long long)g.lda, (long long)g.ldw, epc);
    if ((reinterpret_cast<uintptr_t>(g.A) | reinterpret_cast<uintptr_t>(g.W)) % 16)
        return fail(BC_ERR_UNSUPPORTED, "GEMM operands must be 16-byte aligned");
    const int cls = epi == BC_EPI_GATE_RES ? (g.K > g.N ? PROF_GEMM_DOWN : PROF_GEMM_GATE)
                    : g.e.gelu_from < g.N ? PROF_GEMM_GELU : PROF_GEMM_BIAS;
    prof_begin(cls, s, 2.0 * g.M * (double)g.N * g.K);
    int rc;
    if (dtype == BC_BF16) {
        rc = epi == BC_EPI_GATE_RES ? run_gemm<bf16, BC_EPI_GATE_RES>(g, s) : run_gemm<bf16, BC_EPI_BIAS>(g, s);
    } else {
        rc = epi == BC_EPI_GATE_RES ? run_gemm<float, BC_EPI_GATE_RES>(g, s) : run_gemm<float, BC_EPI_BIAS>(g, s);
    }
    prof_end(cls, s);
    return rc;
}

// The first GEMM's tile choice must be the phased kernel's 256 x 256 (as
// run_gemm picks it), the second one must suit that kernel, and its tiles must fit the idle part of the first one's last
// round; otherwise two launches.
int launch_gemm_pair(int dtype, int epi, const GemmArgs& g0, const GemmArgs& g1, hipStream_t s) {
    if (g1.M <= 0 || g1.N <= 0) return launch_gemm(dtype, epi, g0, s);
    if (g0.M <= 0 || g0.N <= 0) return launch_gemm(dtype, epi, g1, s);
    auto wide = [&](const GemmArgs& g) {
        return dtype == BC_BF16 && g.K > 0 && g.K % 64 == 0 && g.lda % 8 == 0 && g.ldw % 8 == 0 &&
               (reinterpret_cast<uintptr_t>(g.A) | reinterpret_cast<uintptr_t>(g.W)) % 16 == 0 && wide_ok(g, epi);
    };
    const int64_t t0 = (int64_t)((g0.M + 255) / 256) * ((g0.N + 255) / 256);
    const int64_t t1 = (int64_t)((g1.M + 255) / 256) * ((g1.N + 255) / 256);
    const int64_t idle = (t0 + 255) / 256 * 256 - t0;
    const bool fits = g1.K >= 128 && (g1.lda > g1.ldw ? g1.lda : g1.ldw) <= (1 << 22);
    if (!(wide(g0) && wide(g1) && phase_parts(g0) == 2 && fits && t1 <= idle && t0 + t1 <= 0x7fffffff)) {
        const int rc = launch_gemm(dtype, epi, g0, s);
        return rc != BC_OK ? rc : launch_gemm(dtype, epi, g1, s);
    }
    const int cls = epi == BC_EPI_GATE_RES ? (g0.K > g0.N ? PROF_GEMM_DOWN : PROF_GEMM_GATE)
                    : g0.e.gelu_from < g0.N ? PROF_GEMM_GELU : PROF_GEMM_BIAS;
    prof_begin(cls, s, 2.0 * g0.M * (double)g0.N * g0.K + 2.0 * g1.M * (double)g1.N * g1.K);
    const dim3 grid((unsigned)(t0 + t1)), block(512);
    if (epi == BC_EPI_GATE_RES)
        launch_k(gemm_phase_pair_kernel<BC_EPI_GATE_RES>, grid, block, s, g0, g1, (int)t0);
    else
        launch_k(gemm_phase_pair_kernel<BC_EPI_BIAS>, grid, block, s, g0, g1, (int)t0);
    prof_end(cls, s);
    return check_launch("gemm pair");
}

GemmArgs gemm_args(const void* A, int64_t lda, const void* W, int64_t ldw, int M, int N, int K) {
    GemmArgs g;
    g.A = A; g.lda = lda; g.W = W; g.ldw = ldw;
    g.M = M; g.N = N; g.K = K;
    GemmEpi& e = g.e;
    e.bias = nullptr;
    e.out = nullptr; e.ldo = N; e.out_f32 = 0;
    e.out2 = nullptr; e.ldo2 = 0; e.split = N; e.off2 = 0;
    e.gelu_from = N;
    e.q_scale_to = 0; e.q_scale = 1.f;
    e.res = nullptr; e.ldr = N;
    e.gate = nullptr; e.ldg = N; e.rows_per_gate = 1;
    e.seg = M > 0 ? M : 1; e.keep = e.seg;
    return g;
}

}  // namespace bc

using namespace bc;

extern "C" int bc_linear(int M, int N, int K, const void* A, const void* W, const void* bias, void* out,
                         int epilogue, const float* res, const float* gate, int rows_per_gate, int dtype,
                         void* stream) {
    clear_error();
    if (!A || !W || !out) return fail(BC_ERR_INVALID_ARG, "NULL operand");
    if (M < 0 || N < 1 || K < 1) return fail(BC_ERR_INVALID_ARG, "M=%d N=%d K=%d", M, N, K);
    if (dtype != BC_F32 && dtype != BC_BF16) return fail(BC_ERR_INVALID_ARG, "dtype %d", dtype);
    if (epilogue < BC_EPI_BIAS || epilogue > BC_EPI_GATE_RES) return fail(BC_ERR_INVALID_ARG, "epilogue %d", epilogue);
    GemmArgs g = gemm_args(A, K, W, K, M, N, K);
    g.e.bias = bias;
    g.e.out = out;
    if (epilogue == BC_EPI_BIAS_GELU) g.e.gelu_from = 0;
    if (epilogue == BC_EPI_GATE_RES) {
        if (!res || !gate || rows_per_gate < 1) return fail(BC_ERR_INVALID_ARG, "gated residual needs res, gate, rows_per_gate");
        g.e.res = res;
        g.e.gate = gate;
        g.e.rows_per_gate = rows_per_gate;
        g.e.out_f32 = 1;
    }
    return launch_gemm(dtype, epilogue == BC_EPI_GATE_RES ? BC_EPI_GATE_RES : BC_EPI_BIAS, g,
                       static_cast<hipStream_t>(stream));
}
