// HIP kernels for gfx950 (CDNA4): fused gate passes, encoding, measurement, sampling, gradient
// assembly.  64-wide wavefronts throughout.  No code is shared with the CPU oracle.
#include "qsv_kernels.h"
#include "qsv_gate_asm.h"

#include <mutex>

namespace qsv {

namespace {

constexpr int R = kRegBits;
constexpr int NR = 1 << R;
constexpr int CHUNK_BITS = 12;            // reduction kernels: 256 threads x 16 elements
constexpr int CHUNK = 1 << CHUNK_BITS;

typedef unsigned long long u64;

__device__ __forceinline__ float prob32(float2 a) {
    // one fixed rounding sequence so that every kernel that needs p32 gets the same bits: re * re
    // rounded, then one fused multiply-add (written out: a plain sum of two products leaves the
    // compiler free to fuse either product, differently from kernel to kernel)
    return __builtin_fmaf(a.y, a.y, a.x * a.x);
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Reduction kernels run one block per (chunk of a row, row): the chunk in grid.x, the row spread over
// grid.y and grid.z (a grid dimension other than x holds at most 65535 blocks).
__device__ __forceinline__ unsigned long long grid_row() {
    return (unsigned long long)blockIdx.z * gridDim.y + blockIdx.y;
}

// Sum over a 256-thread block; result valid in thread 0.  sm: 4 doubles.
__device__ __forceinline__ double block_sum256(double v, double* sm) {
    v = wave_sum(v);
    const int w = threadIdx.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sm[w] = v;
    __syncthreads();
    return sm[0] + sm[1] + sm[2] + sm[3];
}

// ------------------------------------------------------------------------------------------
// Row mapping (plain: row = sample; gradient: row -> (sample, shifted parameter)).
struct RowCtx {
    u64 sample;
    int ovr_id;     // matrix id replaced by the shifted matrix, or -1
    u64 ovr_off;    // float offset of that matrix inside the shifted table (per-sample part added by caller)
};

__device__ __forceinline__ RowCtx row_ctx(const RowMap& rm, u64 row) {
    RowCtx rc;
    rc.sample = row;
    rc.ovr_id = -1;
    rc.ovr_off = 0;
    if (rm.grad) {
        const u64 gid = (u64)rm.row0 + row;
        const u64 per = (u64)rm.per;
        rc.sample = gid / per;
        const int v = (int)(gid % per);
        if (v < rm.two_p) {
            const int p = v >> 1;
            const int l = p / rm.slots_n;
            const int q = p % rm.n;
            rc.ovr_id = l * rm.n + q;
            rc.ovr_off = (u64)v * 8;
        }
    }
    return rc;
}

// ------------------------------------------------------------------------------------------
// Fused pass kernel.
//
// Tile-local index tau (T bits) <-> extended index e: e = tile_base | (tau & (2^c-1)) |
// ((tau >> c) << w).  In layout s a lane holds the 16 amplitudes tau = thr_part | (i << s),
// i = 0..15, where thr_part spreads the thread index over the other T-4 bits.


// One 2x2 complex matrix times one amplitude pair, in place.  (a,b) = (re,im) of the amplitude
// whose target bit is 0, (c,d) of the one whose bit is 1; m = (m00r,m00i,m01r,m01i,m10r,m10i,m11r,
// m11i).  Written as one asm block with tied operands so that the 32 amplitude registers never
// move: four interleaved accumulation chains whose last step overwrites an input that is dead by
// then.  16 VALU instructions per pair, none of them a copy.  Used where the matrix differs per lane;
// matrices shared by a wavefront are applied inside the interpreter.
#define QSV_U_PAIR_BODY                      \
    "v_mul_f32 %4, %8, %0\n\t"               \
    "v_mul_f32 %5, %9, %0\n\t"               \
    "v_mul_f32 %6, %12, %0\n\t"              \
    "v_mul_f32 %7, %13, %0\n\t"              \
    "v_fma_f32 %4, -%9, %1, %4\n\t"          \
    "v_fma_f32 %5, %8, %1, %5\n\t"           \
    "v_fma_f32 %6, -%13, %1, %6\n\t"         \
    "v_fma_f32 %7, %12, %1, %7\n\t"          \
    "v_fma_f32 %4, %10, %2, %4\n\t"          \
    "v_fma_f32 %5, %11, %2, %5\n\t"          \
    "v_fma_f32 %6, %14, %2, %6\n\t"          \
    "v_fma_f32 %7, %15, %2, %7\n\t"          \
    "v_fma_f32 %0, -%11, %3, %4\n\t"         \
    "v_fma_f32 %1, %10, %3, %5\n\t"          \
    "v_fma_f32 %2, -%15, %3, %6\n\t"         \
    "v_fma_f32 %3, %14, %3, %7\n\t"

// matrix in vector registers (differs per lane: several state rows share a tile)
__device__ __forceinline__ void u_pair_v(float& a, float& b, float& c, float& d, const float (&m)[8]) {
    float t0, t1, t2, t3;
    asm volatile(QSV_U_PAIR_BODY
                 : "+v"(a), "+v"(b), "+v"(c), "+v"(d), "=&v"(t0), "=&v"(t1), "=&v"(t2), "=&v"(t3)
                 : "v"(m[0]), "v"(m[1]), "v"(m[2]), "v"(m[3]), "v"(m[4]), "v"(m[5]), "v"(m[6]), "v"(m[7]));
}

template <int J>
__device__ __forceinline__ void apply_u(float (&vr)[NR], float (&vi)[NR], const float (&m)[8]) {
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        if (i & (1 << J)) continue;
        const int i1 = i | (1 << J);
        u_pair_v(vr[i], vi[i], vr[i1], vi[i1], m);
    }
}

__device__ __forceinline__ void apply_u_any(int j, float (&vr)[NR], float (&vi)[NR], const float (&m)[8]) {
    switch (j) {
        case 0: apply_u<0>(vr, vi, m); break;
        case 1: apply_u<1>(vr, vi, m); break;
        case 2: apply_u<2>(vr, vi, m); break;
        default: apply_u<3>(vr, vi, m); break;
    }
}

// constant-address-space views: uniform loads through them become scalar loads
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef const __attribute__((address_space(4))) u32x2* cuint2_p;
typedef const __attribute__((address_space(4))) f32x4* cfloat4_p;

// A value that is certainly held in a scalar register (an "s" input constraint alone is not
// enough: the compiler may hand a vector register to the asm).
__device__ __forceinline__ unsigned to_sgpr(unsigned v) {
    unsigned r;
    // The compiler cannot see into the asm, so it does not pad the one wait state this chip needs
    // between a vector write of a register and a readfirstlane of it; s_nop covers it.
    asm volatile("s_nop 4\n\tv_readfirstlane_b32 %0, %1\n\ts_nop 1" : "=s"(r) : "v"(v));
    return r;
}

__device__ __forceinline__ u64 uni64(u64 v) {
    return ((u64)to_sgpr((unsigned)(v >> 32)) << 32) | to_sgpr((unsigned)v);
}

// The 16 amplitudes of a lane live in 32 separately named scalars (vr0..vr15, vi0..vi15): as an
// array the compiler turns them into one 16-wide vector value and copies the whole tuple around
// the asm block.  QSV_16 applies a statement macro to every index.
#define QSV_16(X) X(0) X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15)
// The same 16 indices in Gray-code order, with the register bit that changes on the way in and the
// direction (+: the bit turns on): X(k, bit, sign).  The address of element k of a tile then follows
// from the previous one by adding or subtracting one of four strides, two scalar instructions
// instead of the nine it takes to build it from k (scalar instructions compete with the vector
// ones for issue slots).  The walk starts from "element 0 minus stride 0".
#define QSV_8G(X) X(0, 0, +) X(1, 0, +) X(3, 1, +) X(2, 0, -) X(6, 2, +) X(7, 0, +) X(5, 1, -) X(4, 0, -)
#define QSV_8G2(X) X(12, 3, +) X(13, 0, +) X(15, 1, +) X(14, 0, -) X(10, 2, -) X(11, 0, +) X(9, 1, -) X(8, 0, -)
#define QSV_16G(X) QSV_8G(X) QSV_8G2(X)
#define QSV_DECL(k) float vr##k, vi##k;
#define QSV_RV(k) [r##k] "+v"(vr##k), [i##k] "+v"(vi##k),
#define QSV_DECL2(k) float lr##k, li##k;
#define QSV_RV2(k) [p##k] "+v"(lr##k), [q##k] "+v"(li##k),

// Byte offsets of register elements 1, 2, 4, 8 in layout s inside an LDS plane, as XORed onto the
// lane's own address part: swz(k << s) * 4 with swz(x) = x ^ ((x >> 4) & 31).  swz is linear over
// XOR, so the offset of any element is the XOR of the offsets of its set bits.  One 16-byte row per
// layout.
struct XpOffsets {
    unsigned v[12][4];
    constexpr XpOffsets() : v() {
        for (int s = 0; s < 12; ++s)
            for (int j = 0; j < 4; ++j) {
                const unsigned x = (1u << j) << s;
                v[s][j] = (x ^ ((x >> 4) & 31u)) * 4u;
            }
    }
};
__device__ __attribute__((aligned(64))) const XpOffsets k_xp_tab = XpOffsets();
#define k_xp_off k_xp_tab.v

// PERLANE = true is the variant for tiles that hold several state rows (n < T): it adds the
// per-lane-matrix path; the main variant keeps its operation loop minimal.
//
// Structure of a pass: the first operation loads the tile; the assembly interpreter then runs
// gates, sign flips and LDS transposes in place until it meets an operation it does not handle
// (a per-lane unitary, or the end), which the C++ loop handles before re-entering it.
template <int T, bool PERLANE, int PLANES>
// 96 scalar registers (the interpreter pins 37 of them) allow eight wavefronts per SIMD; the main
// variant needs no scalar spills for that (the per-lane-matrix variant has some, and is limited by
// its vector registers anyway).
__global__ __launch_bounds__(1 << (T - R)) __attribute__((amdgpu_num_sgpr(96)))
void k_pass(const PassArgs a) {
    // PLANES XOR-swizzled planes of 2^T floats each (real and imaginary parts at once, or one
    // after the other through a single plane, which halves the LDS a workgroup holds); see the
    // interpreter's generator.  The segment must start at LDS byte 0 (no static LDS here).
    extern __shared__ float lds[];
    // A workgroup that has just started shares its SIMDs with up to seven older ones in the middle of
    // their gates; the sooner its loads are on their way, the more of their latency those gates hide.
    if (a.prio) __builtin_amdgcn_s_setprio(3);
    constexpr unsigned PLANE = 1u << T;
    static_assert(PLANES == 1 || (PLANE * 4u < 65536u && PLANE / 64u < 256u),
                  "with two planes the second plane is reached through the LDS offset fields");
    const unsigned lds_byte0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) float*)lds;
    const unsigned thr = threadIdx.x;
    const u64 tb = a.rev ? (u64)reversed_tile(blockIdx.x, gridDim.x, a.rev) : (u64)blockIdx.x;
    const int c = a.c, w = a.w;
    const unsigned cmask = (1u << c) - 1u;
    const int wc = w - c;
    const u64 tile_base = ((tb & ((1ull << wc) - 1ull)) << c) | ((tb >> wc) << (w + T - c));
    auto expand = [&](unsigned tau) -> u64 {
        return (u64)(tau & cmask) | ((u64)(tau >> c) << w);
    };
    if (tile_base >= a.total) return;  // padding tile (batch not a power of two): nothing to do
    if (lds_byte0 != 0) return;        // cannot happen; the swizzled addressing relies on it
    // every element of the tile in range? (false only for the last tile of a ragged batch)
    const bool full = (tile_base | expand((1u << T) - 1u)) < a.total;
    // tiles never straddle a state row unless T > n, in which case rows are per lane
    const bool rows_uniform = !PERLANE;
    const RowCtx urc = row_ctx(a.rm, tile_base >> a.n);
    // scalar operands of the interpreter
    const u64 mbase = (u64)(uintptr_t)(a.mats + (a.rowdep && rows_uniform ? urc.sample * (u64)a.n_mats * 8 : 0));
    const u64 ovrp = (u64)(uintptr_t)(a.ovr + (a.rowdep && rows_uniform ? urc.sample * (u64)a.rm.two_p * 8 : 0) + urc.ovr_off);
    const unsigned mlo = to_sgpr((unsigned)mbase), mhi = to_sgpr((unsigned)(mbase >> 32));
    const unsigned olo = to_sgpr((unsigned)ovrp), ohi = to_sgpr((unsigned)(ovrp >> 32));
    // unitaries are numbered in execution order; exec_of maps (layer, qubit) ids to that order
    const unsigned ovr_id = to_sgpr((unsigned)((rows_uniform && urc.ovr_id >= 0) ? a.exec_of[urc.ovr_id] : -1));
    const unsigned nonuni = to_sgpr(rows_uniform ? 0u : 1u);
    const unsigned sc_c = to_sgpr((unsigned)c), sc_w = to_sgpr((unsigned)w), sc_cmask = to_sgpr(cmask);
    const unsigned tblo = to_sgpr((unsigned)tile_base), tbhi = to_sgpr((unsigned)(tile_base >> 32));
    const u64 tab = (u64)(uintptr_t)&k_xp_off[0][0];
    const unsigned tablo = to_sgpr((unsigned)tab), tabhi = to_sgpr((unsigned)(tab >> 32));
    unsigned opslo = to_sgpr((unsigned)(uintptr_t)a.ops), opshi = to_sgpr((unsigned)((u64)(uintptr_t)a.ops >> 32));

    QSV_16(QSV_DECL)
    // ---- first operation: load the tile in layout s (register run at tile bits s..s+3)
    const u32x2 first = *(cuint2_p)(uintptr_t)a.ops;
    unsigned scur = to_sgpr((first.x >> 8) & 0xffu);
    const unsigned tau0 = ((thr >> scur) << (scur + R)) | (thr & ((1u << scur) - 1u));
    u64 e0 = tile_base | expand(tau0);
    // A tile's index bits span less than 2^29 elements unless n > 28: then an element's address is
    // a scalar base (tile and register part) plus one 32-bit per-lane byte offset, which costs no
    // vector arithmetic per element.
    const bool off32 = (expand((1u << T) - 1u) >> 29) == 0;
    // Where the tile is read from: the state itself, or (first pass of a gradient chunk, rows
    // uniform per tile) the kept start state of the row's sample, so that no copy pass is needed.
    const float2* ld = a.in;
    if (a.src && rows_uniform) {
        const u64 d = (u64)(((long long)urc.sample - (long long)(tile_base >> a.n)) << a.n);
        const long long ds = (long long)(((u64)to_sgpr((unsigned)(d >> 32)) << 32) | to_sgpr((unsigned)d));
        ld = a.src + ds;
    }
    if (full && off32 && ld == a.in) {
        // the common case, written against the kernel argument itself: the compiler then keeps the
        // per-element base in scalar registers and spends no vector arithmetic on addresses
        const unsigned lane_byte = (unsigned)expand(tau0) * 8u;
        const u64 st0 = expand(1u << scur) * 8u, st1 = expand(2u << scur) * 8u, st2 = expand(4u << scur) * 8u,
                  st3 = expand(8u << scur) * 8u;
        const char* bp = (const char*)(a.in + tile_base) - st0;
#define QSV_LD(k, bit, sign) { bp = bp sign st##bit; \
                    const float2 v = *(const float2*)(bp + lane_byte); vr##k = v.x; vi##k = v.y; }
        QSV_16G(QSV_LD)
#undef QSV_LD
    } else if (full && off32) {
        const unsigned lane_byte = (unsigned)expand(tau0) * 8u;
#define QSV_LD(k) { const char* bp = (const char*)(ld + (tile_base | expand((unsigned)k << scur))); \
                    const float2 v = *(const float2*)(bp + lane_byte); vr##k = v.x; vi##k = v.y; }
        QSV_16(QSV_LD)
#undef QSV_LD
    } else if (full) {
#define QSV_LD(k) { const float2 v = ld[e0 | expand((unsigned)k << scur)]; vr##k = v.x; vi##k = v.y; }
        QSV_16(QSV_LD)
#undef QSV_LD
    } else {
#define QSV_LD(k) { const u64 e = e0 | expand((unsigned)k << scur); const float2 v = ld[e < a.total ? e : tile_base]; \
                    vr##k = e < a.total ? v.x : 0.f; vi##k = e < a.total ? v.y : 0.f; }
        QSV_16(QSV_LD)
#undef QSV_LD
    }
    { const u64 nx = (u64)(uintptr_t)a.ops + 8; opslo = to_sgpr((unsigned)nx); opshi = to_sgpr((unsigned)(nx >> 32)); }
    if (a.prio) __builtin_amdgcn_s_setprio(0);
    unsigned e0lo = (unsigned)e0, e0hi = (unsigned)(e0 >> 32);
    unsigned ldsb = (tau0 ^ ((tau0 >> 4) & 31u)) * 4u;

    for (;;) {
        {
            float t0, t1, t2, t3, tc, m0, m1, m2, m3, m4, m5, m6, m7;
            unsigned ba0, ba1, ba2, ba3, bb0, bb1, bb2, bb3;
#define QSV_LOOP_OUT QSV_16(QSV_RV) [t0] "=&v"(t0), [t1] "=&v"(t1), [t2] "=&v"(t2),                 \
                     [t3] "=&v"(t3), [tc] "=&v"(tc), [m0] "=&v"(m0), [m1] "=&v"(m1), [m2] "=&v"(m2), \
                     [m3] "=&v"(m3), [m4] "=&v"(m4), [m5] "=&v"(m5), [m6] "=&v"(m6), [m7] "=&v"(m7), \
                     [ba0] "=&v"(ba0), [ba1] "=&v"(ba1), [ba2] "=&v"(ba2), [ba3] "=&v"(ba3),       \
                     [bb0] "=&v"(bb0), [bb1] "=&v"(bb1), [bb2] "=&v"(bb2), [bb3] "=&v"(bb3),       \
                     [opslo] "+s"(opslo), [opshi] "+s"(opshi),                                     \
                     [scur] "+s"(scur), [ldsb] "+v"(ldsb), [e0lo] "+v"(e0lo), [e0hi] "+v"(e0hi)
#define QSV_LOOP_IN [mlo] "s"(mlo), [mhi] "s"(mhi), [olo] "s"(olo), [ohi] "s"(ohi),                 \
                    [ovrid] "s"(ovr_id), [nonuni] "s"(nonuni), [thr] "v"(thr), [c] "s"(sc_c),       \
                    [w] "s"(sc_w), [cmask] "s"(sc_cmask), [tblo] "s"(tblo), [tbhi] "s"(tbhi),       \
                    [tablo] "s"(tablo), [tabhi] "s"(tabhi)
            // four texts: two or one LDS plane, and whether a unitary may have to be left to the C++
            // code below (several state rows per tile with row-dependent matrices)
            if constexpr (PLANES == 2 && PERLANE) {
                asm volatile(QSV_GATE_LOOP_ASM_2P_ROWS
                             : QSV_LOOP_OUT
                             : QSV_LOOP_IN, [plane4] "n"(PLANE * 4u), [pl64] "n"(PLANE / 64u)
                             : QSV_GATE_LOOP_CLOBBERS);
            } else if constexpr (PLANES == 2) {
                asm volatile(QSV_GATE_LOOP_ASM_2P
                             : QSV_LOOP_OUT
                             : QSV_LOOP_IN, [plane4] "n"(PLANE * 4u), [pl64] "n"(PLANE / 64u)
                             : QSV_GATE_LOOP_CLOBBERS);
            } else if constexpr (PERLANE) {
                unsigned ldsn;
                asm volatile(QSV_GATE_LOOP_ASM_1P_ROWS
                             : QSV_LOOP_OUT, [ldsn] "=&v"(ldsn)
                             : QSV_LOOP_IN
                             : QSV_GATE_LOOP_CLOBBERS);
            } else {
                unsigned ldsn;
                asm volatile(QSV_GATE_LOOP_ASM_1P
                             : QSV_LOOP_OUT, [ldsn] "=&v"(ldsn)
                             : QSV_LOOP_IN
                             : QSV_GATE_LOOP_CLOBBERS);
            }
#undef QSV_LOOP_OUT
#undef QSV_LOOP_IN
        }
        // Operations are read as one aligned 64-bit word each and decoded with shifts.
        const u64 opp = ((u64)opshi << 32) | opslo;
        const u32x2 word = *(cuint2_p)(uintptr_t)opp;
        const unsigned kind = word.x & 0xffu;
        const int arg = (int)word.y;
        e0 = ((u64)e0hi << 32) | e0lo;
        if (PERLANE && kind == OP_U) {
            // several rows per tile and row-dependent matrices: per-lane matrix.  The run lies
            // inside the qubit bits (planner rule), so a lane's 16 amplitudes share one row.
            float m[8], xr[NR], xi[NR];
            const u64 ee = e0 < a.total ? e0 : 0;
            const RowCtx rc = row_ctx(a.rm, ee >> a.n);
            const int lane_ovr = rc.ovr_id >= 0 ? a.exec_of[rc.ovr_id] : -1;
            const float* p = (arg == lane_ovr)
                ? a.ovr + (a.rowdep ? rc.sample * (u64)a.rm.two_p * 8 : 0) + rc.ovr_off
                : a.mats + ((a.rowdep ? rc.sample * (u64)a.n_mats : 0) + (u64)arg) * 8;
            const float4 lo = *reinterpret_cast<const float4*>(p);
            const float4 hi = *reinterpret_cast<const float4*>(p + 4);
            m[0] = lo.x; m[1] = lo.y; m[2] = lo.z; m[3] = lo.w;
            m[4] = hi.x; m[5] = hi.y; m[6] = hi.z; m[7] = hi.w;
#define QSV_IN(k) xr[k] = vr##k; xi[k] = vi##k;
            QSV_16(QSV_IN)
#undef QSV_IN
            apply_u_any((int)((word.x >> 8) & 0xffu), xr, xi, m);
#define QSV_OUT(k) vr##k = xr[k]; vi##k = xi[k];
            QSV_16(QSV_OUT)
#undef QSV_OUT
        } else {
            break;  // OP_END (the interpreter never stops on anything else)
        }
        { const u64 nx = opp + 8; opslo = (unsigned)nx; opshi = (unsigned)(nx >> 32); }
    }
    if (a.zout) {
        // Last pass of a gradient row: <Z_q> of the tile instead of (or besides) the stored state.
        // A lane sums its 16 probabilities with the sign of bit q (register part: per element,
        // uniform; the rest: from the lane's index), a wavefront adds its lanes in double, and each
        // wavefront writes one partial: [tile][wavefront], summed per row in a fixed order later.
        const int zq = a.zq;
        float acc = 0.f;
#define QSV_Z(k) { const float p = vr##k * vr##k + vi##k * vi##k; \
                   acc += ((expand((unsigned)k << scur) >> zq) & 1ull) ? -p : p; }
        QSV_16(QSV_Z)
#undef QSV_Z
        if ((e0 >> zq) & 1ull) acc = -acc;
        const double tot = wave_sum((double)acc);
        if ((thr & 63u) == 0) a.zout[tb * (blockDim.x >> 6) + (thr >> 6)] = tot;
        if (a.nostore) return;
    }
    if (a.prio) __builtin_amdgcn_s_setprio(3);
    if (a.imap) {
        // Deferred CNOTs: every amplitude goes to the index its position maps to.  The map is linear
        // over XOR, so the destination is (tile's part) ^ (lane's part) ^ (register element's part);
        // bits at and above n (the state row) stay.  The host only sets imap when every tile is full and
        // byte offsets inside a row fit 32 bits.
        const unsigned nmask = (1u << a.n) - 1u;
        const unsigned* im = a.imap;
        unsigned et = 0;
        for (unsigned rem = to_sgpr((unsigned)tile_base & nmask); rem; rem &= rem - 1u) et ^= im[__builtin_ctz(rem)];
        const unsigned pos_lane = (unsigned)(e0 ^ tile_base);      // the lane's own index bits (register bits zero)
        unsigned el = et;
        for (int b = 0; b < T; ++b) {
            if (b >= (int)scur && b < (int)scur + R) continue;       // register bits follow below
            const int q = b < c ? b : b - c + w;                     // index bit behind tile bit b
            if (q >= a.n) continue;
            el ^= ((pos_lane >> q) & 1u) ? im[q] : 0u;
        }
        auto reg_part = [&](int j) -> unsigned {
            const int b = (int)scur + j;
            const int q = b < c ? b : b - c + w;
            return im[q];
        };
        const unsigned x0 = reg_part(0), x1 = reg_part(1), x2 = reg_part(2), x3 = reg_part(3);
        char* bp = (char*)(a.state + (tile_base & ~(u64)nmask));
        unsigned idx = el ^ x0;                                      // the walk starts from "element 0 minus bit 0"
        if (a.nt_store) {
#define QSV_ST(k, bit, sign) { idx ^= x##bit; \
                    f32x2 v; v.x = vr##k; v.y = vi##k; __builtin_nontemporal_store(v, (f32x2*)(bp + (u64)idx * 8u)); }
            QSV_16G(QSV_ST)
#undef QSV_ST
        } else {
#define QSV_ST(k, bit, sign) { idx ^= x##bit; *(float2*)(bp + (u64)idx * 8u) = make_float2(vr##k, vi##k); }
            QSV_16G(QSV_ST)
#undef QSV_ST
        }
    } else if (full && off32 && a.nt_store) {
        // States much larger than the last-level cache: nontemporal stores, so that the lines written
        // now (read again only a whole pass later) do not displace what the pass still has to read.
        const unsigned lane_byte = (unsigned)(e0 ^ tile_base) * 8u;   // the lane's own index bits
        const u64 st0 = expand(1u << scur) * 8u, st1 = expand(2u << scur) * 8u, st2 = expand(4u << scur) * 8u,
                  st3 = expand(8u << scur) * 8u;
        char* bp = (char*)(a.state + tile_base) - st0;
#define QSV_ST(k, bit, sign) { bp = bp sign st##bit; \
                    f32x2 v; v.x = vr##k; v.y = vi##k; __builtin_nontemporal_store(v, (f32x2*)(bp + lane_byte)); }
        QSV_16G(QSV_ST)
#undef QSV_ST
    } else if (full && off32) {
        const unsigned lane_byte = (unsigned)(e0 ^ tile_base) * 8u;
        const u64 st0 = expand(1u << scur) * 8u, st1 = expand(2u << scur) * 8u, st2 = expand(4u << scur) * 8u,
                  st3 = expand(8u << scur) * 8u;
        char* bp = (char*)(a.state + tile_base) - st0;
#define QSV_ST(k, bit, sign) { bp = bp sign st##bit; *(float2*)(bp + lane_byte) = make_float2(vr##k, vi##k); }
        QSV_16G(QSV_ST)
#undef QSV_ST
    } else if (full) {
#define QSV_ST(k) a.state[e0 | expand((unsigned)k << scur)] = make_float2(vr##k, vi##k);
        QSV_16(QSV_ST)
#undef QSV_ST
    } else {
#define QSV_ST(k) { const u64 e = e0 | expand((unsigned)k << scur); if (e < a.total) a.state[e] = make_float2(vr##k, vi##k); }
        QSV_16(QSV_ST)
#undef QSV_ST
    }
}

// Fetches what the interpreter will read, `bytes` from p on, into the scalar cache, every wavefront its share of the lines, all
// at once.  The interpreter itself looks one operation ahead, and a line that it finds missing costs it an L2's latency: on
// one 19-qubit state a pass of 80 operations found 46 lines missing, one after the other, in the 15 us that it took (58 % of
// the wavefronts' cycles were waits); 8 layers and back 84.6 -> 75.6 us.  The caller's rule has both sides.
__device__ __forceinline__ void warm_scalar_cache(u64 p, unsigned bytes) {
    unsigned at = to_sgpr(threadIdx.x >> 6) * 64u;
    const unsigned step = to_sgpr(blockDim.x >> 6) * 64u;
    if (at >= bytes) return;
    asm volatile("L_warm_%=:\n\t"
                 "s_load_dword s36, %[p], %[at]\n\t"
                 "s_add_u32 %[at], %[at], %[step]\n\t"
                 "s_cmp_lt_u32 %[at], %[n]\n\t"
                 "s_cbranch_scc1 L_warm_%=\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : [at] "+s"(at)
                 : [p] "s"(uni64(p)), [step] "s"(step), [n] "s"(to_sgpr(bytes))
                 : "s36", "scc", "memory");
}

// ------------------------------------------------------------------------------------------
// The same pass for tiles of one state row (n >= T, n <= 28): the form that almost every launch takes.
// What a row's tiles have in common (register layouts of the load and the store, the row's sample, the
// first table entry) comes from the host or is worked out once per wavefront with 32-bit numbers; a row is
// one buffer of at most 2^31 bytes, so an element's address is the lane's byte offset plus one scalar
// offset; and the gates run in the direct interpreter (see gen_gate_asm.py).
// Bound by the issue of vector and scalar instructions together with memory.  Measured against k_pass on the
// same plans, alternating the two: 16 qubits x 256 shift-rule gradient 120 -> 102 ms, 26 qubits x 30 layers
// 12.1 -> 11.4 ms, 20 qubits x 32 autoencoder 5.95 -> 5.83 ms, one 19-qubit state 114 -> 88 us.
// Eight wavefronts per SIMD: at most 64 vector registers (a workgroup of a 2^13 tile is eight wavefronts, and
// a CU that holds three of them instead of four took 6 % longer).
// GATHER: the variant for passes that read through an index map.  Such a map may leave the two halves of a
// 128-byte line to two tiles, t and t ^ mate, and both fetch the line: mate_order lets them start eight
// workgroups apart, that is on the same XCD and at nearly the same time, so that its L2 serves the second.
// 20 qubits x 32, 20 layers and back: reads of the mirrored passes 1.31 -> 1.00 times their bytes (2.00 in the worst),
// 4416 -> 4365 us.
// TURNED: the variant for the last pass of turned gradient rows, which stores three sums and no state.
// WARM: the variant that fetches ahead (see warm_scalar_cache): as a branch it costs launches that don't 0.5 % (26 qubits).
template <int T, bool GATHER, bool TURNED = false, bool WARM = false>
__global__ __launch_bounds__(1 << (T - R)) __attribute__((amdgpu_num_sgpr(96), amdgpu_waves_per_eu(8, 8)))
void k_pass_direct(const PassArgs a) {
    extern __shared__ float lds[];
    if (a.prio) __builtin_amdgcn_s_setprio(3);
    if ((unsigned)(uintptr_t)(__attribute__((address_space(3))) float*)lds != 0) return;   // cannot happen; LDS addresses rely on it
    const unsigned thr = threadIdx.x;
    const unsigned tile = a.rev ? reversed_tile(blockIdx.x, gridDim.x, a.rev) : blockIdx.x;
    const unsigned nb = (unsigned)(a.n - T), row = tile >> nb;
    unsigned tr = tile & ((1u << nb) - 1u);
    if constexpr (GATHER) tr = mate_order(tr, a.mate);
    const unsigned c = (unsigned)a.c, w = (unsigned)a.w, cmask = (1u << c) - 1u;
    const unsigned base = ((tr & ((1u << (w - c)) - 1u)) << c) | ((tr >> (w - c)) << (w + T - c));
    auto expand = [&](unsigned tau) -> unsigned { return (tau & cmask) | ((tau >> c) << w); };
    auto lane_tau = [&](unsigned s) -> unsigned { return ((thr >> s) << (s + R)) | (thr & ((1u << s) - 1u)); };
    unsigned sample = row;
    const float* ovr = a.ovr;
    int ovr_at = -1;                               // table position of the row's shifted matrix
    if (a.rm.grad) {
        const unsigned local = a.g_rem0 + row;
        sample = a.g_sample0 + local / (unsigned)a.rm.per;
        const unsigned v = local % (unsigned)a.rm.per;
        if (v < (unsigned)a.rm.two_p) {
            const unsigned p = a.turns ? v : v >> 1;
            ovr_at = a.exec_of[p / (unsigned)a.rm.slots_n * (unsigned)a.n + p % (unsigned)a.n];
            ovr += ((a.rowdep ? (u64)sample * (unsigned)a.rm.two_p : 0) + v) * 8;
        }
    }
    const float* mats = a.mats + (a.rowdep ? (u64)sample * (unsigned)a.n_mats * 8 : 0);
    const int row_bytes = (int)(8u << a.n);        // the resource's size (unsigned to the hardware): one row
    typedef unsigned u32x2v __attribute__((ext_vector_type(2)));
    // deferred CNOTs: lane j of every half wavefront holds the map's entry of index bit j
    unsigned im = 0;
    if (a.imap && (thr & 31u) < (unsigned)a.n) im = a.imap[thr & 31u];
    QSV_16(QSV_DECL)
    const unsigned s_in = (unsigned)a.s_in, s_out = (unsigned)a.s_out;
    const unsigned tau0 = lane_tau(s_in);
    unsigned e0 = expand(tau0);
    // Deferred CNOTs: position p of a tile belongs at the index that is the XOR of the map's entries over p's
    // set bits, (tile's part) ^ (lane's part) ^ (register element's part).  Byte offset of the lane's element 0
    // in its row in layout s, and what the register bits flip in it.
    unsigned map_off = 0, x0 = 0, x1 = 0, x2 = 0, x3 = 0;
    auto follow_map = [&](unsigned s) {
        unsigned et = (base >> (thr & 31u)) & 1u ? im : 0u;
#pragma unroll
        for (int d = 16; d > 0; d >>= 1) et ^= __shfl_xor(et, d, 32);
        auto entry = [&](unsigned b) -> unsigned {   // of the index bit behind tile bit b
            return (unsigned)__builtin_amdgcn_readlane((int)im, (int)(b < c ? b : b - c + w));
        };
#pragma unroll
        for (unsigned i = 0; i < T - R; ++i) {       // thread bit i is tile bit i or i + 4
            const unsigned m = entry(i < s ? i : i + R);
            et ^= (thr >> i) & 1u ? m : 0u;
        }
        map_off = et * 8u;
        x0 = entry(s) * 8u; x1 = entry(s + 1) * 8u; x2 = entry(s + 2) * 8u; x3 = entry(s + 3) * 8u;
    };
    {
        const float2* in = a.src ? a.src + ((u64)sample << a.n) : a.in + ((u64)row << a.n);
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)in, 0, row_bytes, 0x00020000);
#define QSV_GET(k, off, so) { const u32x2v v = __builtin_bit_cast(u32x2v, __builtin_amdgcn_raw_buffer_load_b64(rs, (int)(off), (int)(so), 0)); \
            vr##k = __uint_as_float(v.x); vi##k = __uint_as_float(v.y); }
        if constexpr (GATHER) {
            follow_map(s_in);
            unsigned off = map_off ^ x0;
            // the empty asm keeps the offsets in one register, one after the other
#define QSV_LD(k, bit, sign) { off ^= x##bit; asm volatile("" : "+v"(off)); QSV_GET(k, off, 0) }
            QSV_16G(QSV_LD)
#undef QSV_LD
        } else {
            const unsigned st0 = expand(1u << s_in) * 8u, st1 = expand(2u << s_in) * 8u, st2 = expand(4u << s_in) * 8u,
                           st3 = expand(8u << s_in) * 8u;
            const unsigned voff = e0 * 8u;
            unsigned so = base * 8u - st0;
#define QSV_LD(k, bit, sign) { so = so sign st##bit; QSV_GET(k, voff, so) }
            QSV_16G(QSV_LD)
#undef QSV_LD
        }
#undef QSV_GET
    }
    if (a.prio) __builtin_amdgcn_s_setprio(0);
    if constexpr (WARM) {                            // while the tile is on its way
        warm_scalar_cache((u64)(uintptr_t)a.ops, (unsigned)a.warm_ops);
        warm_scalar_cache((u64)(uintptr_t)(mats + (u64)a.first_mat * 8), (unsigned)a.warm_mats);
    }
    const bool scatter = !GATHER && !TURNED && a.imap;
    if (scatter) follow_map(s_out);                  // while the tile is on its way
    {
        unsigned ldsb = (tau0 + 2u * (tau0 >> 5)) * 4u, ldsn;
        e0 |= base;
        float t0, t1, t2, t3, tc, m0, m1, m2, m3, m4, m5, m6, m7;
        const u64 ops = (u64)(uintptr_t)a.ops, mat = (u64)(uintptr_t)mats, ov = (u64)(uintptr_t)ovr;
        asm volatile(QSV_GATE_DIRECT_ASM
                     : QSV_16(QSV_RV)[t0] "=&v"(t0), [t1] "=&v"(t1), [t2] "=&v"(t2), [t3] "=&v"(t3), [tc] "=&v"(tc),
                       [m0] "=&v"(m0), [m1] "=&v"(m1), [m2] "=&v"(m2), [m3] "=&v"(m3), [m4] "=&v"(m4), [m5] "=&v"(m5),
                       [m6] "=&v"(m6), [m7] "=&v"(m7), [ldsb] "+v"(ldsb), [ldsn] "=&v"(ldsn), [e0] "+v"(e0)
                     : [thr] "v"(thr), [ops] "s"(uni64(ops)), [mats] "s"(uni64(mat)), [ovr] "s"(uni64(ov)),
                       [ovrid] "s"(to_sgpr((unsigned)ovr_at)), [first] "s"(to_sgpr((unsigned)a.first_mat * 32u)),
                       [c] "s"(to_sgpr(c)), [w] "s"(to_sgpr(w)), [cmask] "s"(to_sgpr(cmask)), [tb] "s"(to_sgpr(base))
                     : QSV_GATE_DIRECT_CLOBBERS);
    }
    const unsigned lane_out = expand(lane_tau(s_out));
    if (TURNED || a.zout) {
        // last pass of a gradient row: see k_pass
        const int zq = a.zq;
        const u64 at = (u64)tile * (blockDim.x >> 6) + (thr >> 6);
        const bool flip = ((base | lane_out) >> zq) & 1u;
        if constexpr (TURNED) {
            // The row's angle is turned by pi: its state b and the unturned a make the two shifted ones.  a's amplitudes come
            // eight at a time: what is free of 64 registers does not hold all 16.
            const __amdgpu_buffer_rsrc_t ru =
                __builtin_amdgcn_make_buffer_rsrc((void*)(a.unturned + ((u64)sample << a.n)), 0, row_bytes, 0x00020000);
            float zb = 0.f, cr = 0.f, ci = 0.f;
            unsigned off = lane_out * 8u;
            // Gray-code walk over the register elements: strides of their bits, and the sign bit where bit zq is among them
            const unsigned st0 = expand(1u << s_out), st1 = expand(2u << s_out), st2 = expand(4u << s_out), st3 = expand(8u << s_out);
            const unsigned zm = 1u << zq, f0 = st0 & zm ? 1u << 31 : 0u, f1 = st1 & zm ? 1u << 31 : 0u, f2 = st2 & zm ? 1u << 31 : 0u,
                           f3 = st3 & zm ? 1u << 31 : 0u;
            unsigned so = base - st0, sg = f0;
#define QSV_ZP(k, bit, sign) { so = so sign st##bit; sg ^= f##bit; \
                    const u32x2v g = __builtin_bit_cast(u32x2v, __builtin_amdgcn_raw_buffer_load_b64(ru, (int)off, (int)(so * 8u), 0)); \
                    const float ur = __uint_as_float(g.x), ui = __uint_as_float(g.y), pb = vr##k * vr##k + vi##k * vi##k, \
                                pr = ur * vr##k + ui * vi##k, pi = ur * vi##k - ui * vr##k; \
                    zb += __uint_as_float(__float_as_uint(pb) ^ sg); cr += __uint_as_float(__float_as_uint(pr) ^ sg); \
                    ci += __uint_as_float(__float_as_uint(pi) ^ sg); }
            QSV_8G(QSV_ZP)
            asm volatile("" : "+v"(off), "+v"(zb), "+v"(cr), "+v"(ci));      // the second half's loads wait for these sums
            QSV_8G2(QSV_ZP)
#undef QSV_ZP
            const double sign = flip ? -1.0 : 1.0;
            const double tb = wave_sum(sign * zb), tr = wave_sum(sign * cr), ti = wave_sum(sign * ci);
            if ((thr & 63u) == 0) {
                a.zout[3 * at] = tb;
                a.zout[3 * at + 1] = tr;
                a.zout[3 * at + 2] = ti;
            }
            return;
        } else {
            float acc = 0.f;
#define QSV_Z(k) { const float p = vr##k * vr##k + vi##k * vi##k; \
                   acc += (expand((unsigned)k << s_out) >> zq) & 1u ? -p : p; }
            QSV_16(QSV_Z)
#undef QSV_Z
            const double tot = wave_sum((double)(flip ? -acc : acc));
            if ((thr & 63u) == 0) a.zout[at] = tot;
        }
        if (a.nostore) return;
    }
    if (a.prio) __builtin_amdgcn_s_setprio(3);
    const __amdgpu_buffer_rsrc_t ro =
        __builtin_amdgcn_make_buffer_rsrc((void*)(a.state + ((u64)row << a.n)), 0, row_bytes, 0x00020000);
#define QSV_PUT(k, off, so, aux) { u32x2v v; v.x = __float_as_uint(vr##k); v.y = __float_as_uint(vi##k); \
            __builtin_amdgcn_raw_buffer_store_b64(v, ro, (int)(off), (int)(so), aux); }
    if (scatter) {
        unsigned off = map_off ^ x0;
#define QSV_ST(k, bit, sign) { off ^= x##bit; QSV_PUT(k, off, 0, AUX) }
        if (a.nt_store) {
#define AUX 2
            QSV_16G(QSV_ST)
#undef AUX
        } else {
#define AUX 0
            QSV_16G(QSV_ST)
#undef AUX
        }
#undef QSV_ST
    } else {
        const unsigned st0 = expand(1u << s_out) * 8u, st1 = expand(2u << s_out) * 8u, st2 = expand(4u << s_out) * 8u,
                       st3 = expand(8u << s_out) * 8u;
        unsigned so = base * 8u - st0;
#define QSV_ST(k, bit, sign) { so = so sign st##bit; QSV_PUT(k, lane_out * 8u, so, AUX) }
        if (a.nt_store) {
#define AUX 2
            QSV_16G(QSV_ST)
#undef AUX
        } else {
#define AUX 0
            QSV_16G(QSV_ST)
#undef AUX
        }
#undef QSV_ST
    }
#undef QSV_PUT
}

// ------------------------------------------------------------------------------------------
// A diagonal observable O, given by its weight w(k):
//   kind 0: Z_q,             w = +1 / -1 by bit q
//   kind 1: -P0(mask),       w = -1 where no bit of mask is set, else 0  (loss 1 - P0)
//   kind 2: sum_q c[r][q] Z_q, w = sum_q c[r][q] (1 - 2 bit_q(k))        (chain rule of the squared error)
struct AdjObs { int kind; int q; u64 mask; const double* coef; };

__device__ __forceinline__ float adj_weight(const AdjObs& o, u64 r, u64 k, int n) {
    if (o.kind == 0) return ((k >> o.q) & 1ull) ? -1.f : 1.f;
    if (o.kind == 1) return (k & o.mask) ? 0.f : -1.f;
    double w = 0.0;
    const double* c = o.coef + r * n;
#pragma unroll 1
    for (int q = 0; q < n; ++q) w += ((k >> q) & 1ull) ? -c[q] : c[q];
    return (float)w;
}

// A mirrored pass on two states at once: psi (read only) and lambda, in the paired interpreter, which takes the
// transition sums of every unitary off the registers.  GATHER: through an index map, as in k_pass_direct.
// Bound by vector issue (the sums and two unitaries take 3.3 times the instructions of one) and by how much of the
// transposes and loads other wavefronts cover: a wavefront holds both tiles' parts, 64 registers of amplitudes in 77, so
// that six fit a SIMD, and a workgroup one LDS plane.  With 84 registers and two planes (four wavefronts, half the
// barriers of a transpose) 20 qubits x 32, 20 layers took 7.88 instead of 7.12 ms, 16 x 256, 10 layers 1.12 instead of 1.05.
// Against layer by layer (psi of every layer kept, lambda taken back by k_pass_direct, the sums by two or three launches
// that read both): 11.8 -> 7.1 ms and 2.83 -> 1.05 ms; 13 x 37, 5 re-uploading layers 500 -> 160 us, 18 x 4, 6 layers 584 ->
// 300, 22 x 2, 6 layers 1428 -> 840.
// WARM: as in k_pass_direct.
template <int T, bool GATHER, bool WARM>
__global__ __launch_bounds__(1 << (T - R)) __attribute__((amdgpu_num_sgpr(100), amdgpu_waves_per_eu(6, 6)))
void k_pair_pass(const PairArgs a) {
    extern __shared__ float lds[];
    if ((unsigned)(uintptr_t)(__attribute__((address_space(3))) float*)lds != 0) return;   // cannot happen; LDS addresses rely on it
    const unsigned thr = threadIdx.x;
    const unsigned tile = a.rev ? reversed_tile(blockIdx.x, gridDim.x, a.rev) : blockIdx.x;
    const unsigned nb = (unsigned)(a.n - T), row = tile >> nb;
    unsigned tr = tile & ((1u << nb) - 1u);
    if constexpr (GATHER) tr = mate_order(tr, a.mate);
    const unsigned c = (unsigned)a.c, w = (unsigned)a.w, cmask = (1u << c) - 1u;
    const unsigned base = ((tr & ((1u << (w - c)) - 1u)) << c) | ((tr >> (w - c)) << (w + T - c));
    auto expand = [&](unsigned tau) -> unsigned { return (tau & cmask) | ((tau >> c) << w); };
    auto lane_tau = [&](unsigned s) -> unsigned { return ((thr >> s) << (s + R)) | (thr & ((1u << s) - 1u)); };
    const float* mats = a.mats + (a.rowdep ? ((u64)a.sample0 + row) * (unsigned)a.n_mats * 8 : 0);
    const int row_bytes = (int)(8u << a.n);        // the resources' size (unsigned to the hardware): one row
    typedef unsigned u32x2v __attribute__((ext_vector_type(2)));
    unsigned im = 0;
    if constexpr (GATHER) { if ((thr & 31u) < (unsigned)a.n) im = a.imap[thr & 31u]; }
    QSV_16(QSV_DECL)
    QSV_16(QSV_DECL2)
    const unsigned s_in = (unsigned)a.s_in, s_out = (unsigned)a.s_out;
    const unsigned tau0 = lane_tau(s_in);
    unsigned e0 = expand(tau0);
    unsigned map_off = 0, x0 = 0, x1 = 0, x2 = 0, x3 = 0;
    const float2* psi = a.psi + ((u64)row << a.n);
    const float2* lam = a.lam_in ? a.lam_in + ((u64)row << a.n) : psi;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)psi, 0, row_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rl = __builtin_amdgcn_make_buffer_rsrc((void*)lam, 0, row_bytes, 0x00020000);
#define QSV_GETV(S, rsrc, k, off, so) { const u32x2v got = __builtin_bit_cast(u32x2v, __builtin_amdgcn_raw_buffer_load_b64(rsrc, (int)(off), (int)(so), 0)); \
        S##r##k = __uint_as_float(got.x); S##i##k = __uint_as_float(got.y); }
    if constexpr (GATHER) {
        unsigned et = (base >> (thr & 31u)) & 1u ? im : 0u;
#pragma unroll
        for (int d = 16; d > 0; d >>= 1) et ^= __shfl_xor(et, d, 32);
        auto entry = [&](unsigned b) -> unsigned {   // of the index bit behind tile bit b
            return (unsigned)__builtin_amdgcn_readlane((int)im, (int)(b < c ? b : b - c + w));
        };
#pragma unroll
        for (unsigned i = 0; i < T - R; ++i) {       // thread bit i is tile bit i or i + 4
            const unsigned m = entry(i < s_in ? i : i + R);
            et ^= (thr >> i) & 1u ? m : 0u;
        }
        map_off = et * 8u;
        x0 = entry(s_in) * 8u; x1 = entry(s_in + 1) * 8u; x2 = entry(s_in + 2) * 8u; x3 = entry(s_in + 3) * 8u;
        unsigned off = map_off ^ x0;
        // the empty asm keeps the offsets in one register, one after the other
#define QSV_LD(k, bit, sign) { off ^= x##bit; asm volatile("" : "+v"(off)); QSV_GETV(v, rs, k, off, 0) QSV_GETV(l, rl, k, off, 0) }
        QSV_16G(QSV_LD)
#undef QSV_LD
    } else {
        x0 = expand(1u << s_in) * 8u; x1 = expand(2u << s_in) * 8u; x2 = expand(4u << s_in) * 8u; x3 = expand(8u << s_in) * 8u;
        const unsigned voff = e0 * 8u;
        unsigned so = base * 8u - x0;
#define QSV_LD(k, bit, sign) { so = so sign x##bit; QSV_GETV(v, rs, k, voff, so) QSV_GETV(l, rl, k, voff, so) }
        QSV_16G(QSV_LD)
#undef QSV_LD
        map_off = voff | base * 8u;
    }
#undef QSV_GETV
    if constexpr (WARM) {                            // while the tiles are on their way
        warm_scalar_cache((u64)(uintptr_t)a.ops, (unsigned)a.warm_ops);
        warm_scalar_cache((u64)(uintptr_t)(mats + (u64)a.first_mat * 8), (unsigned)a.warm_mats);
    }
    if (!a.lam_in) {                                 // lambda = O psi, at the indices the amplitudes were read from
        const AdjObs o{a.kind, a.q, a.mask, a.coef};
        unsigned off = map_off ^ x0;
#define QSV_OBS(k, bit, sign) { off ^= x##bit; const float wk = adj_weight(o, row, off >> 3, a.n); lr##k = wk * vr##k; li##k = wk * vi##k; }
        QSV_16G(QSV_OBS)
#undef QSV_OBS
    }
    {
        unsigned ldsb = (tau0 + 2u * (tau0 >> 5)) * 4u, ldsn;
        e0 |= base;
        float t0, t1, m0, m1, m2, m3, m4, m5, kept;
        const u64 ops = (u64)(uintptr_t)a.ops, mat = (u64)(uintptr_t)mats;
        // the pass's records: of a unitary, 16 bytes per wavefront in the order of the rows and tiles
        const u64 waves = (u64)a.rows << (a.n - 10);
        const u64 sums = (u64)(uintptr_t)(a.sums + ((u64)(unsigned)a.first_u * waves + (((u64)row << nb) + tr) * (blockDim.x >> 6)) * 4);
        asm volatile(QSV_GATE_PAIRED_ASM
                     : QSV_16(QSV_RV) QSV_16(QSV_RV2)[t0] "=&v"(t0), [t1] "=&v"(t1), [m0] "=&v"(m0), [m1] "=&v"(m1), [m2] "=&v"(m2),
                       [m3] "=&v"(m3), [m4] "=&v"(m4), [m5] "=&v"(m5), [kept] "=&v"(kept), [ldsb] "+v"(ldsb), [ldsn] "=&v"(ldsn),
                       [e0] "+v"(e0)
                     : [thr] "v"(thr), [ops] "s"(uni64(ops)), [mats] "s"(uni64(mat)), [sums] "s"(uni64(sums)),
                       [sstep] "s"(to_sgpr((unsigned)(waves * 16u))), [first] "s"(to_sgpr((unsigned)a.first_mat * 32u)),
                       [c] "s"(to_sgpr(c)), [w] "s"(to_sgpr(w)), [cmask] "s"(to_sgpr(cmask)), [tb] "s"(to_sgpr(base))
                     : QSV_GATE_PAIRED_CLOBBERS);
    }
    if (!a.lam_out) return;
    const unsigned lane_out = expand(lane_tau(s_out));
    const __amdgpu_buffer_rsrc_t ro =
        __builtin_amdgcn_make_buffer_rsrc((void*)(a.lam_out + ((u64)row << a.n)), 0, row_bytes, 0x00020000);
    const unsigned st0 = expand(1u << s_out) * 8u, st1 = expand(2u << s_out) * 8u, st2 = expand(4u << s_out) * 8u,
                   st3 = expand(8u << s_out) * 8u;
    unsigned so = base * 8u - st0;
#define QSV_ST(k, bit, sign) { so = so sign st##bit; u32x2v v; v.x = __float_as_uint(lr##k); v.y = __float_as_uint(li##k); \
            __builtin_amdgcn_raw_buffer_store_b64(v, ro, (int)(lane_out * 8u), (int)so, AUX); }
    if (a.nt_store) {
#define AUX 2
        QSV_16G(QSV_ST)
#undef AUX
    } else {
#define AUX 0
        QSV_16G(QSV_ST)
#undef AUX
    }
#undef QSV_ST
}

// ------------------------------------------------------------------------------------------
// One-gate-per-launch kernels.
__global__ __launch_bounds__(256) void k_naive_u(float2* state, u64 pairs, int n, int q,
                                                 const float* mats, const float* ovr, int mat_id,
                                                 int n_mats, int rowdep, RowMap rm) {
    const u64 i = (u64)blockIdx.x * 256 + threadIdx.x;
    if (i >= pairs) return;
    const u64 bit = 1ull << q;
    const u64 k0 = ((i >> q) << (q + 1)) | (i & (bit - 1));  // extended index, bit q clear
    const u64 k1 = k0 | bit;
    const RowCtx rc = row_ctx(rm, k0 >> n);
    const float* m = (mat_id == rc.ovr_id)
        ? ovr + (rowdep ? rc.sample * (u64)rm.two_p * 8 : 0) + rc.ovr_off
        : mats + ((rowdep ? rc.sample * (u64)n_mats : 0) + (u64)mat_id) * 8;
    const float2 x0 = state[k0], x1 = state[k1];
    float2 y0, y1;
    y0.x = m[0] * x0.x - m[1] * x0.y + m[2] * x1.x - m[3] * x1.y;
    y0.y = m[0] * x0.y + m[1] * x0.x + m[2] * x1.y + m[3] * x1.x;
    y1.x = m[4] * x0.x - m[5] * x0.y + m[6] * x1.x - m[7] * x1.y;
    y1.y = m[4] * x0.y + m[5] * x0.x + m[6] * x1.y + m[7] * x1.x;
    state[k0] = y0;
    state[k1] = y1;
}

__global__ __launch_bounds__(256) void k_naive_cnot(float2* state, u64 total, int ctrl, int tgt) {
    const u64 k = (u64)blockIdx.x * 256 + threadIdx.x;
    if (k >= total) return;
    if (((k >> ctrl) & 1) && !((k >> tgt) & 1)) {
        const u64 k1 = k | (1ull << tgt);
        const float2 t = state[k];
        state[k] = state[k1];
        state[k1] = t;
    }
}

__global__ __launch_bounds__(256) void k_naive_cz_ladder(float2* state, u64 total, int n) {
    const u64 e = (u64)blockIdx.x * 256 + threadIdx.x;
    if (e >= total) return;
    const u64 k = e & ((1ull << n) - 1);
    if (__popcll(k & (k >> 1)) & 1) {
        float2 v = state[e];
        v.x = -v.x; v.y = -v.y;
        state[e] = v;
    }
}

// ------------------------------------------------------------------------------------------
// Fused per-(layer, qubit) matrices, computed in double and rounded once to float.
struct M2 { double r[4], i[4]; };  // row-major 2x2: [0]=m00 [1]=m01 [2]=m10 [3]=m11

__device__ __forceinline__ int axis_of(const CircDev& c, int sl) {
    return c.reupload && sl == 0 ? (int)QSV_RX : c.rot[sl - c.reupload];
}

__device__ __forceinline__ M2 rot_m(int axis, double t) {
    double s, c;
    sincos(0.5 * t, &s, &c);
    M2 m;
    for (int k = 0; k < 4; ++k) { m.r[k] = 0.0; m.i[k] = 0.0; }
    if (axis == QSV_RX) { m.r[0] = c; m.i[1] = -s; m.i[2] = -s; m.r[3] = c; }
    else if (axis == QSV_RY) { m.r[0] = c; m.r[1] = -s; m.r[2] = s; m.r[3] = c; }
    else { m.r[0] = c; m.i[0] = -s; m.r[3] = c; m.i[3] = s; }
    return m;
}

__device__ __forceinline__ M2 mul_m(const M2& a, const M2& b) {  // a * b
    M2 o;
    for (int r = 0; r < 2; ++r)
        for (int cc = 0; cc < 2; ++cc) {
            double sr = 0.0, si = 0.0;
            for (int k = 0; k < 2; ++k) {
                const double ar = a.r[r * 2 + k], ai = a.i[r * 2 + k];
                const double br = b.r[k * 2 + cc], bi = b.i[k * 2 + cc];
                sr += ar * br - ai * bi;
                si += ar * bi + ai * br;
            }
            o.r[r * 2 + cc] = sr; o.i[r * 2 + cc] = si;
        }
    return o;
}

// (a, b) = first column of R(axis, t) U from that of U; s, co = sin, cos of t / 2
__device__ __forceinline__ void rotate_column(int axis, double s, double co, double& ar, double& ai, double& br,
                                              double& bi) {
    const double a0 = ar, a1 = ai, b0 = br, b1 = bi;
    if (axis == QSV_RX) {
        ar = co * a0 + s * b1; ai = co * a1 - s * b0;
        br = co * b0 + s * a1; bi = co * b1 - s * a0;
    } else if (axis == QSV_RY) {
        ar = co * a0 - s * b0; ai = co * a1 - s * b1;
        br = co * b0 + s * a0; bi = co * b1 + s * a1;
    } else {
        ar = co * a0 + s * a1; ai = co * a1 - s * a0;
        br = co * b0 - s * b1; bi = co * b1 + s * b0;
    }
}

// U(l,q) for one sample: slots applied in order (re-upload RX first), i.e. U = R_last ... R_first.
// shift_slot >= 0 adds shift to that slot's angle.  All factors have the form [[a, -conj b], [b, conj a]], so
// only the first column is multiplied up.
__device__ __forceinline__ M2 fused_raw(const CircDev& c, const float* params, const float* feats, u64 sample, int l,
                                        int q, int shift_slot, double shift, int inverse) {
    double ar = 1.0, ai = 0.0, br = 0.0, bi = 0.0;
    const int slots = c.reupload + c.n_rot;
    for (int sl = 0; sl < slots; ++sl) {
        double t = (double)params[((u64)l * slots + sl) * c.n + q];
        int axis;
        if (c.reupload && sl == 0) { t *= (double)feats[sample * c.n + q]; axis = QSV_RX; }
        else axis = c.rot[sl - c.reupload];
        if (sl == shift_slot) t += shift;
        double s, co;
        sincos(0.5 * t, &s, &co);
        rotate_column(axis, s, co, ar, ai, br, bi);
    }
    if (inverse) { ai = -ai; br = -br; bi = -bi; }   // conjugate transpose
    M2 u;
    u.r[0] = ar; u.i[0] = ai; u.r[1] = -br; u.i[1] = bi;
    u.r[2] = br; u.i[2] = bi; u.r[3] = ar; u.i[3] = -ai;
    return u;
}

struct Cx { double r, i; };

__device__ __forceinline__ Cx mul_c(Cx a, Cx b) { return {a.r * b.r - a.i * b.i, a.r * b.i + a.i * b.r}; }

__device__ __forceinline__ void scale_m(M2& u, Cx f) {  // u *= f
    for (int k = 0; k < 4; ++k) {
        const Cx v = mul_c({u.r[k], u.i[k]}, f);
        u.r[k] = v.r;
        u.i[k] = v.i;
    }
}

__device__ __forceinline__ void store_m(const M2& u, float* out8) {
    float4* o = reinterpret_cast<float4*>(out8);
    o[0] = make_float4((float)u.r[0], (float)u.i[0], (float)u.r[1], (float)u.i[1]);
    o[1] = make_float4((float)u.r[2], (float)u.i[2], (float)u.r[3], (float)u.i[3]);
}

// The turn by the unit number p = i^quarter sigma e^(i angle) as three shears, t = -tan(angle/2), s = sin(angle):
// |angle| <= pi/2, or <= pi/4 where a quarter turn may be taken out.  A phase that vanishes by structure comes out as
// rounding noise of a few 1e-17 and is dropped.
// The shears of a rounded pair (t, s) multiply to a turn by a slightly different angle and a small
// stretch, about 1e-8 each; s is the one that belongs to the rounded t, which keeps the stretch to its rounding.
__device__ __forceinline__ bool has_phase(Cx p) { return !(fabs(p.i) < 1e-14); }

__device__ __forceinline__ void shears(Cx p, bool quarters, double* sigma, bool* quarter, float* t, float* s) {
    *quarter = quarters && fabs(p.i) > fabs(p.r);
    if (*quarter) p = {p.i, -p.r};
    *sigma = 1.0;
    if (p.r < 0.0) { *sigma = -1.0; p.r = -p.r; p.i = -p.i; }
    *t = 0.f;
    *s = 0.f;
    if (!has_phase(p)) return;
    *t = (float)(-p.i / (1.0 + p.r));
    const double td = (double)*t;
    *s = (float)(-2.0 * td / (1.0 + td * td));
}

// What the three shears and the quarter turn multiply q by (as far as it is a number: see shears).
__device__ __forceinline__ Cx turned(float t, float s, bool quarter) {
    const double td = (double)t, sd = (double)s;
    const Cx z = {1.0 + td * sd, 0.5 * (sd - 2.0 * td - td * td * sd)};
    return quarter ? Cx{-z.i, z.r} : z;
}

// u (unitary with determinant 1) = g * diag(1, zB) core diag(1, zA), the core being the real rotation
// divided by its larger entry: see rot_pair in gen_gate_asm.py, which lists the entry's fields and
// applies it.  inverse: the entry of the conjugate transpose, with the same rounded
// numbers: a reverse-mode gradient compares states taken forward and back, and an angle that differs
// between the two by its rounding shows in it undiminished (measured: 1e-5 instead of 3e-6).
// g brings the rounded entry nearest to u: the angles of zA and zB are off by about 2e-8, and half of such an angle
// is a factor of the whole entry, which g takes back; the other half acts on p and q in opposite directions and is
// less of an error by sqrt 2 than the whole angle on q.
__device__ __forceinline__ Cx factor_m(const M2& u, int inverse, int seq0, int seq_stride, float* out8) {
    const double a = sqrt(u.r[0] * u.r[0] + u.i[0] * u.i[0]), b = sqrt(u.r[2] * u.r[2] + u.i[2] * u.i[2]);
    Cx ea = {1.0, 0.0}, eb = {1.0, 0.0};              // phases of the first column
    if (a != 0.0) ea = {u.r[0] / a, u.i[0] / a};
    if (b != 0.0) eb = {u.r[2] / b, u.i[2] / b};
    if (a == 0.0) ea = {eb.r, -eb.i};                 // free: leave no phase in front
    if (b == 0.0) eb = {ea.r, -ea.i};
    const Cx ab = mul_c(ea, eb), za = {ab.r, -ab.i}, zb = mul_c(eb, {ea.r, -ea.i});
    bool before = has_phase(za), after = has_phase(zb);
    const bool both = before && after;
    double sa, sb;
    bool qa, qb;
    float ta, na, tb, nb;
    shears(za, both, &sa, &qa, &ta, &na);
    shears(zb, both, &sb, &qb, &tb, &nb);
    float e[6] = {ta, na, 0.f, 0.f, tb, nb};
    double turn = 1.0;                                // sign of the rotation's lower left entry
    if (inverse) {                                    // the phases change places and signs: conj(i) = -i
        e[0] = -tb; e[1] = -nb; e[4] = -ta; e[5] = -na;
        const double other = qa ? -sa : sa;
        sa = qb ? -sb : sb;
        sb = other;
        bool keep = qa; qa = qb; qb = keep;
        keep = before; before = after; after = keep;
        turn = -1.0;
    }
    const bool c_core = !(a < b);                     // also the way of a NaN
    const float q = (float)(c_core ? b / a : a / b);
    // rotation (1, -turn q; turn q, 1) or (q, -turn; turn, q), with the signs of the phases, divided by the entry that is
    // to be 1: 1 or sb turn
    e[2] = (float)(c_core ? -sa * turn : sb * turn) * q;
    e[3] = (float)(c_core ? sb * turn : sa * turn) * q;
    const int form = both ? 3 + (qa ? 1 : 0) + (qb ? 2 : 0) : (after ? 2 : 0) + (before ? 1 : 0);
    const int seq = form * 4 + (c_core ? 0 : 2) + (sa * sb < 0.0 ? 1 : 0);
    float4* o = reinterpret_cast<float4*>(out8);
    o[0] = make_float4(e[0], e[1], e[2], e[3]);
    o[1] = make_float4(e[4], e[5], __int_as_float(seq0 + seq * seq_stride), 0.f);
    // Of the entries that are to be u's (or its conjugate transpose's), two belong to the core's ones: x, and conj(x) or
    // -conj(x).  Divided by their phases in the rounded entry they agree but for the errors of those: their mean, with
    // the length that gives the entry columns of length 1.
    const Cx z1 = turned(e[0], e[1], qa), z2 = turned(e[4], e[5], qb), z12 = mul_c(z1, z2);
    const Cx x = c_core ? Cx{u.r[0], turn * u.i[0]} : Cx{turn * u.r[2], turn * u.i[2]};
    const double sigma = sa * sb;
    const Cx x1 = c_core ? x : mul_c({z2.r, -z2.i}, x), x2 = mul_c(c_core ? z12 : z1, x);   // the second's conjugate
    const double big = c_core ? a : b, len = 0.5 * rsqrt((1.0 + (double)q * (double)q) * big * big);
    return {len * (x1.r + sigma * x2.r), len * (x1.i - sigma * x2.i)};
}

// The matrix of a table entry as the interpreter applies it, scaled to columns of length 1.
__device__ __forceinline__ M2 entry_m(const float* e, bool whole, int seq0, int seq_stride) {
    M2 u;
    if (whole) {
        for (int k = 0; k < 4; ++k) { u.r[k] = (double)e[2 * k]; u.i[k] = (double)e[2 * k + 1]; }
    } else {
        const int seq = (__float_as_int(e[6]) - seq0) / seq_stride, core = seq & 3, form = seq >> 2;
        const double sigma = (core & 1) ? -1.0 : 1.0, x = (double)e[2], y = (double)e[3];
        const Cx z1 = turned(e[0], e[1], form == 4 || form == 6), z2 = turned(e[4], e[5], form == 5 || form == 6);
        const bool c_core = core < 2;
        const double m00 = c_core ? 1.0 : x, m01 = c_core ? x : -sigma, m10 = c_core ? y : 1.0, m11 = c_core ? sigma : y;
        const Cx z12 = mul_c(z1, z2);
        u.r[0] = m00; u.i[0] = 0.0;
        u.r[1] = m01 * z1.r; u.i[1] = m01 * z1.i;
        u.r[2] = m10 * z2.r; u.i[2] = m10 * z2.i;
        u.r[3] = m11 * z12.r; u.i[3] = m11 * z12.i;
    }
    const double len = rsqrt(u.r[0] * u.r[0] + u.i[0] * u.i[0] + u.r[2] * u.r[2] + u.i[2] * u.i[2]);
    for (int k = 0; k < 4; ++k) { u.r[k] *= len; u.i[k] *= len; }
    return u;
}

// Entry pos of an order table.  period > 0: the table has `period` entries and describes one layer;
// it repeats for every layer (entry pos of layer pos / period is that layer's entry pos % period).
__device__ __forceinline__ int ordered(const int* table, int period, int pos) {
    return period > 0 ? (pos / period) * period + table[pos % period] : table[pos];
}

// One thread per unitary, one wavefront per group of kMatGroup consecutive ones (a layer's unitaries when
// period > 0): all but the one with the highest id are stored factored, and their scalars, multiplied up
// across the wavefront, go into that one, which is stored as a matrix.  kind = plain: every entry is the matrix
// itself (tables that are read per lane, and the one-gate-per-launch path).  kind = phaseless: matrices in the factored
// ones' place too, without the phase of their upper left entry; products with its imaginary part, an exact zero, round
// nothing (gradients of the small sweep 2 to 4 % nearer to 64 bits).
// scale (may be NULL): what a matrix that replaces entry pos has to be multiplied by.
// starts: groups of their own sizes, whose scalars are an entry behind each (see Plan::groups).  kind = paired: scale
// receives what sums over two states, both taken through the entries up to this one, are to be multiplied by (they lack
// the scalars of the group's unitaries so far), and the same without this entry.
// One launch where the factors used to be collected by a second one (10 us to 5 us before a circuit).
// GROUPED: starts is given.  As a branch at run time it cost launches without groups 0.3 to 0.8 us (reverse mode of 8 qubits x 110, 1
// layer 17.2 -> 16.4 us, 5 x 275, 3 layers 20.2 -> 19.6).
template <bool GROUPED>
__global__ __launch_bounds__(256) void k_build_mats(CircDev c, const float* params, const float* feats,
                                                    u64 groups, int inverse, const int* order, int period,
                                                    const int* starts, int n_starts,
                                                    MatForm kind, int seq0, int seq_stride, float* out, double* scale) {
    static_assert(kMatGroup == 64, "a wavefront is a group");
    const u64 gi = (u64)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (gi >= groups) return;
    const int lane = threadIdx.x & 63;
    const int per = c.n_layers * c.n, seg = period > 0 ? period : per;
    const int per_seg = GROUPED ? n_starts : (seg + kMatGroup - 1) / kMatGroup, per_table = per_seg * (per / seg);
    const u64 sample = gi / (u64)per_table;
    const int gt = (int)(gi % (u64)per_table);
    const int in_seg = (GROUPED ? starts[gt % per_seg] : (gt % per_seg) * kMatGroup) + lane;
    const int seg_end = GROUPED ? starts[gt % per_seg + 1] : seg;
    const int pos = (gt / per_seg) * seg + in_seg;
    const bool live = in_seg < seg_end;
    const int lq = !live ? -1 : order ? ordered(order, period, pos) : pos;
    int top = lq;
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) top = max(top, __shfl_xor(top, d, 64));
    const bool whole = !GROUPED && (kind == MatForm::plain || lq == top), matrix = whole || kind == MatForm::phaseless;
    Cx g = {1.0, 0.0};
    M2 u;
    float* o = out + (sample * (u64)(per + (GROUPED ? per_table : 0)) + (u64)(pos + (GROUPED ? gt : 0))) * 8;
    if (live) {
        u = fused_raw(c, params, feats, sample, lq / c.n, lq % c.n, -1, 0.0, matrix ? inverse : 0);
        if (!matrix) g = factor_m(u, inverse, seq0, seq_stride, o);
        else if (!whole) {
            const double a = sqrt(u.r[0] * u.r[0] + u.i[0] * u.i[0]);
            if (a != 0.0) g = {u.r[0] / a, u.i[0] / a};
            scale_m(u, {g.r, -g.i});
            u.r[0] = a;
            u.i[0] = 0.0;
            store_m(u, o);
        }
    }
    Cx f = g;
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) {
        const Cx other = {__shfl_xor(f.r, d, 64), __shfl_xor(f.i, d, 64)};
        f = (lane & d) ? mul_c(other, f) : mul_c(f, other);   // the same product in every lane
    }
    if constexpr (GROUPED) {
        if (live && in_seg + 1 == seg_end) {
            float4* own = reinterpret_cast<float4*>(o + 8);
            own[0] = make_float4((float)f.r, (float)f.i, 0.f, 0.f);
            own[1] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (scale && kind == MatForm::direct) {      // what rounding the scalar has changed it by
                const double m2 = f.r * f.r + f.i * f.i;
                const Cx x = mul_c({(double)(float)f.r, (double)(float)f.i}, {f.r / m2, -f.i / m2});
                double* to = scale + (sample * (u64)per_table + (u64)gt) * 2;
                to[0] = x.r;
                to[1] = x.i;
            }
        }
        if (kind != MatForm::paired) return;
        const double own = g.r * g.r + g.i * g.i;
        double up = own;                                 // of the entries up to this one
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const double before = __shfl_up(up, d, 64);
            if (lane >= d) up *= before;
        }
        if (live) {
            double* to = scale + (sample * (u64)per + (u64)pos) * 2;
            to[0] = up;
            to[1] = up / own;
        }
        return;
    }
    if (!live) return;
    if (whole) {
        scale_m(u, f);
        store_m(u, o);
    } else {
        const double m2 = g.r * g.r + g.i * g.i;
        f = {g.r / m2, -g.i / m2};
    }
    if (scale) {
        scale[(sample * (u64)per + (u64)pos) * 2] = f.r;
        scale[(sample * (u64)per + (u64)pos) * 2 + 1] = f.i;
    }
}

// Matrices with one angle shifted by +-pi/2 (parameter-shift rule), each multiplied by what the entry it
// replaces asks for (scale: [tables][per] as k_build_mats wrote it, NULL with a plain table).
__global__ __launch_bounds__(256) void k_build_shifted(CircDev c, const float* params, const float* feats, u64 count,
                                                       const int* exec_of, const double* scale, int per, float* out) {
    const u64 idx = (u64)blockIdx.x * 256 + threadIdx.x;
    if (idx >= count) return;
    const int slots = c.reupload + c.n_rot;
    const u64 two_p = 2ull * c.n_layers * slots * c.n;
    const u64 sample = idx / two_p;
    const int v = (int)(idx % two_p);
    const int p = v >> 1;
    const int q = p % c.n;
    const int sl = (p / c.n) % slots;
    const int l = p / (c.n * slots);
    const double shift = (v & 1) ? -1.57079632679489661923 : 1.57079632679489661923;
    M2 u = fused_raw(c, params, feats, sample, l, q, sl, shift, 0);
    if (scale) {
        const double* f = scale + (sample * (u64)per + (u64)exec_of[l * c.n + q]) * 2;
        scale_m(u, {f[0], f[1]});
    }
    store_m(u, out + idx * 8);
}

// Turns of a layer's angles by pi: R_last .. R_s(t + pi) .. R_0 = U S with S = W^dagger R_s(pi) W, W the slots before s, or
// (behind) S U with S = V R_s(pi) V^dagger, V the slots after s.  S = -i (x X + y Y + z Z), whose float32 numbers have
// columns of exactly equal length at right angles.
__global__ __launch_bounds__(256) void k_build_turns(CircDev c, const float* params, const float* feats, u64 count, int behind,
                                                     float* out) {
    const u64 idx = (u64)blockIdx.x * 256 + threadIdx.x;
    if (idx >= count) return;
    const int slots = c.reupload + c.n_rot, per = slots * c.n, p = (int)(idx % (u64)per), q = p % c.n, s = p / c.n;
    auto rot = [&](int sl, double sign) {
        double t = (double)params[(u64)sl * c.n + q];
        if (c.reupload && sl == 0) t *= (double)feats[idx / (u64)per * c.n + q];
        return rot_m(axis_of(c, sl), sign * t);
    };
    M2 m = rot_m(axis_of(c, s), 3.14159265358979323846);
    if (behind)
        for (int sl = s + 1; sl < slots; ++sl) m = mul_m(mul_m(rot(sl, 1.0), m), rot(sl, -1.0));
    else
        for (int sl = s - 1; sl >= 0; --sl) m = mul_m(mul_m(rot(sl, -1.0), m), rot(sl, 1.0));
    M2 o;                                            // equal and vanishing entries exactly so
    const double x = -m.i[1], y = m.r[2], z = m.i[3];
    o.r[0] = 0.0; o.i[0] = -z; o.r[1] = -y; o.i[1] = -x;
    o.r[2] = y; o.i[2] = -x; o.r[3] = 0.0; o.i[3] = z;
    store_m(o, out + idx * 8);
}

// ------------------------------------------------------------------------------------------
// Amplitude encoding.
// inv_norm != NULL (only with nblk = 1): the block is the whole sample and finishes the norm itself.
__global__ __launch_bounds__(256) void k_sumsq(const float* x, u64 rows, u64 dim, double* partial, int nblk,
                                               double* inv_norm, float* norm_out) {
    __shared__ double sm[4];
    const u64 b = grid_row();
    if (b >= rows) return;
    const float* xb = x + b * dim;
    double acc = 0.0;
    if ((dim & 3) == 0 && ((uintptr_t)x & 15) == 0) {
        // rows are 16-byte aligned: four floats per load (the one-float form reaches 2 TB/s only)
        const float4* xv = reinterpret_cast<const float4*>(xb);
        const u64 dimv = dim >> 2;
        for (u64 base = (u64)blockIdx.x * (CHUNK / 4); base < dimv; base += (u64)nblk * (CHUNK / 4)) {
            float4 v[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const u64 k = base + (u64)i * 256 + threadIdx.x;
                v[i] = k < dimv ? xv[k] : make_float4(0.f, 0.f, 0.f, 0.f);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)
                acc += (double)v[i].x * v[i].x + (double)v[i].y * v[i].y + (double)v[i].z * v[i].z +
                       (double)v[i].w * v[i].w;
        }
    } else {
        for (u64 base = (u64)blockIdx.x * CHUNK; base < dim; base += (u64)nblk * CHUNK) {
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const u64 k = base + (u64)i * 256 + threadIdx.x;
                if (k < dim) { const double v = (double)xb[k]; acc += v * v; }
            }
        }
    }
    const double tot = block_sum256(acc, sm);
    if (threadIdx.x == 0) {
        partial[b * nblk + blockIdx.x] = tot;
        if (inv_norm) {
            const double nrm = sqrt(tot);
            inv_norm[b] = nrm > 0.0 ? 1.0 / nrm : 0.0;
            if (norm_out) norm_out[b] = (float)nrm;
        }
    }
}

__global__ __launch_bounds__(256) void k_norm_finish(const double* partial, int nblk, double* inv_norm,
                                                     float* norm_out) {
    __shared__ double sm[4];
    const u64 b = blockIdx.x;
    double acc = 0.0;
    for (int i = threadIdx.x; i < nblk; i += 256) acc += partial[b * nblk + i];
    const double tot = block_sum256(acc, sm);
    if (threadIdx.x == 0) {
        const double nrm = sqrt(tot);
        inv_norm[b] = nrm > 0.0 ? 1.0 / nrm : 0.0;
        if (norm_out) norm_out[b] = (float)nrm;
    }
}

// FOLDED: every block adds up the sums of k_sumsq ([samples][nblk]) of its row again, in one order, and the row's first
// block writes the norm.  It saves k_norm_finish, a launch between two that wait for it: 19 qubits 7.2 -> 6.5 us, 16 x 4
// 7.1 -> 6.1, 20 qubits 8.5 -> 7.9.  From 2^22 amplitudes the wait in every block costs more than the launch (16 x 64
// 17.5 -> 17.9, 16 x 1024 224 -> 272): inv_norm is then read.
template <bool FOLDED>
__global__ __launch_bounds__(256) void k_encode_write(const float* x, u64 dim, int n, u64 total, const double* partial,
                                                      int nblk, double* inv_norm, float* norm_out, RowMap rm, float2* state) {
    __shared__ double sm[4];
    const u64 e2 = ((u64)blockIdx.x * 256 + threadIdx.x) * 2;
    if constexpr (FOLDED) {                                 // rows of 512 amplitudes and more: a block lies in one row
        const u64 first = (u64)blockIdx.x * 512, sample = row_ctx(rm, first >> n).sample;
        double acc = 0.0;
        for (int i = threadIdx.x; i < nblk; i += 256) acc += partial[sample * (u64)nblk + i];
        const double nrm = sqrt(block_sum256(acc, sm)), inv = nrm > 0.0 ? 1.0 / nrm : 0.0;
        __syncthreads();
        if (threadIdx.x == 0) {
            sm[0] = inv;
            if ((first & ((1ull << n) - 1)) == 0) {
                inv_norm[sample] = inv;
                if (norm_out) norm_out[sample] = (float)nrm;
            }
        }
        __syncthreads();
    }
    if (e2 >= total) return;
    const u64 row = e2 >> n;
    const u64 sample = row_ctx(rm, row).sample;
    const double inv = FOLDED ? sm[0] : inv_norm[sample];
    const u64 k = e2 & ((1ull << n) - 1);
    const float* xb = x + sample * dim;
    float4 o;
    o.x = k < dim ? (float)((double)xb[k] * inv) : 0.f;
    o.y = 0.f;
    o.z = (k + 1) < dim ? (float)((double)xb[k + 1] * inv) : 0.f;
    o.w = 0.f;
    *reinterpret_cast<float4*>(state + e2) = o;
}

// Samples of up to 2^7 entries: norm and state row in one launch.
__global__ __launch_bounds__(256) void k_encode_small(const float* x, u64 rows, u64 dim, int n, double* inv_norm,
                                                      float* norm_out, float2* state) {
    __shared__ double sm[4];
    const u64 b = grid_row();
    if (b >= rows) return;
    const float* xb = x + b * dim;
    double acc = 0.0;
    for (u64 k = threadIdx.x; k < dim; k += 256) { const double v = (double)xb[k]; acc += v * v; }
    const double tot = block_sum256(acc, sm);
    const double nrm = sqrt(tot);
    const double inv = nrm > 0.0 ? 1.0 / nrm : 0.0;
    if (threadIdx.x == 0) {
        inv_norm[b] = inv;
        if (norm_out) norm_out[b] = (float)nrm;
    }
    float2* row = state + (b << n);
    for (u64 k = threadIdx.x; k < (1ull << n); k += 256)
        row[k] = make_float2(k < dim ? (float)((double)xb[k] * inv) : 0.f, 0.f);
}

// A workgroup per sample of 4 THREADS V = 2^n entries, which stay in registers between the sum of their squares and the
// state row: one read of x and one launch instead of two or three.  Bound by the latency of a load, a reduction and a store
// where samples are few, by memory where they are many (15 x 4096: 310 us, 5.2 TB/s).  Before and after: 12 qubits 6.2 -> 2.9
// us, 12 x 4096 41.7 -> 33.0, 13 6.1 -> 3.5, 13 x 256 11.0 -> 6.9, 14 6.2 -> 4.6, 14 x 1024 47 -> 34.  15 qubits: 32
// samples 8.8 -> 8.3, 256 27 -> 19, but 1 sample 6.2 -> 7.1, so few samples are spread over more blocks.  A form for 16
// qubits gained at 256 samples (46 -> 41) and lost at 512 (93 -> 100).
template <int THREADS, int V>
__global__ __launch_bounds__(THREADS) void k_encode_row(const float* x, u64 rows, u64 dim, int n, double* inv_norm,
                                                        float* norm_out, float2* state) {
    __shared__ double sm[THREADS / 64];
    const u64 b = grid_row();
    if (b >= rows) return;
    const float* xb = x + b * dim;
    const unsigned t = threadIdx.x;
    float4 v[V];
    if ((dim & 3) == 0 && ((uintptr_t)x & 15) == 0) {
        const float4* xv = reinterpret_cast<const float4*>(xb);
        const u64 dimv = dim >> 2;
#pragma unroll
        for (int i = 0; i < V; ++i) {
            const u64 k = (u64)i * THREADS + t;
            v[i] = k < dimv ? xv[k] : make_float4(0.f, 0.f, 0.f, 0.f);
        }
    } else {
#pragma unroll
        for (int i = 0; i < V; ++i) {
            const u64 k = ((u64)i * THREADS + t) * 4;
            v[i] = make_float4(k < dim ? xb[k] : 0.f, k + 1 < dim ? xb[k + 1] : 0.f, k + 2 < dim ? xb[k + 2] : 0.f,
                               k + 3 < dim ? xb[k + 3] : 0.f);
        }
    }
    double acc = 0.0;
#pragma unroll
    for (int i = 0; i < V; ++i)
        acc += (double)v[i].x * v[i].x + (double)v[i].y * v[i].y + (double)v[i].z * v[i].z + (double)v[i].w * v[i].w;
    double tot = wave_sum(acc);
    if constexpr (THREADS > 64) {
        if ((t & 63u) == 0) sm[t >> 6] = tot;
        __syncthreads();
        tot = 0.0;
#pragma unroll
        for (int w = 0; w < THREADS / 64; ++w) tot += sm[w];
    }
    const double nrm = sqrt(tot), inv = nrm > 0.0 ? 1.0 / nrm : 0.0;
    if (t == 0) {
        inv_norm[b] = inv;
        if (norm_out) norm_out[b] = (float)nrm;
    }
    float4* row = reinterpret_cast<float4*>(state + (b << n));
#pragma unroll
    for (int i = 0; i < V; ++i) {
        const u64 k = ((u64)i * THREADS + t) * 2;
        row[k] = make_float4((float)((double)v[i].x * inv), 0.f, (float)((double)v[i].y * inv), 0.f);
        row[k + 1] = make_float4((float)((double)v[i].z * inv), 0.f, (float)((double)v[i].w * inv), 0.f);
    }
}

// ------------------------------------------------------------------------------------------
// Measurement.
__global__ __launch_bounds__(256) void k_probs(const float2* state, u64 total, float* out) {
    const u64 e2 = ((u64)blockIdx.x * 256 + threadIdx.x) * 2;
    if (e2 >= total) return;
    const float4 v = *reinterpret_cast<const float4*>(state + e2);
    float2 o;
    o.x = prob32(make_float2(v.x, v.y));
    o.y = prob32(make_float2(v.z, v.w));
    *reinterpret_cast<float2*>(out + e2) = o;
}

// <Z_q> of every qubit: signed sums of the probabilities, in double.  Where index bits are register bits
// their sums come out of a tree (sums and differences of neighbours), behind lane bits out of the
// butterfly that adds up the lanes.
//
// The lanes' part: T (total) and the NR plain sums in z are added over the wavefront, zl[b] becomes the sum signed
// by lane bit b.
template <int NR_>
__device__ __forceinline__ void expz_lanes(double& T, double (&z)[NR_], double (&zl)[6]) {
    const int lane = threadIdx.x & 63;
    auto flip = [&](double v, int b) -> double { return __shfl_xor(v, 1 << b, 64); };
#pragma unroll
    for (int b = 0; b < 6; ++b) {
        const double Tp = flip(T, b);
#pragma unroll
        for (int j = 0; j < NR_; ++j) z[j] += flip(z[j], b);
#pragma unroll
        for (int j = 0; j < 6; ++j)
            if (j < b) zl[j] += flip(zl[j], b);
        zl[b] = ((lane >> b) & 1) ? Tp - T : T - Tp;
        T += Tp;
    }
}

// 8 pairs of neighbouring amplitudes per thread: index = step * 512 + thread * 2 + {0, 1}, so bit 0 and the
// three step bits are register bits: T and z[0..3] (bits 0, 9, 10, 11) of one chunk of 4096.
__device__ __forceinline__ void expz_tree(const double (&p)[16], double& T, double (&z)[4]) {
    double s[8];
    double d = 0.0;
#pragma unroll
    for (int i = 0; i < 8; ++i) { s[i] = p[2 * i] + p[2 * i + 1]; d += p[2 * i] - p[2 * i + 1]; }
    z[0] += d;
#pragma unroll
    for (int j = 0; j < 3; ++j) {                  // step bit j pairs s[2k], s[2k + 1] of what is left
        double e = 0.0;
#pragma unroll
        for (int k = 0; k < (4 >> j); ++k) { e += s[2 * k] - s[2 * k + 1]; s[k] = s[2 * k] + s[2 * k + 1]; }
        z[1 + j] += e;
    }
    T += s[0];
}

// A block takes 2^g consecutive chunks of 4096 amplitudes of a row, whose numbers' bits (index bits 12..12+g-1)
// are signs of the chunks' totals.  partial: [row][13 + g][nblk] doubles: T, index bits 0..11, then those.
// One chunk per block and one reduction per chunk: 40 us on 24 qubits and 21 us for the finishing kernel,
// which walked over 104-byte records; with 2048 blocks left and the entries side by side 24 + 10 us.
// out (NULL: partials): the block has the whole row (nblk = 1) and writes <Z_q> itself, of every qubit or of q_only.  Rows
// of 13 and 14 qubits, one launch instead of two: 13 qubits 6.0 -> 4.1 us, 13 x 256 8.6 -> 4.9, 14 6.0 -> 4.7, 14 x 1024
// 28.7 -> 22.9.  15 and 16 qubits from 64 rows: 15 x 64 8.4 -> 6.4, 15 x 256 19.7 -> 13.0, 16 x 64 11.9 -> 9.8; with fewer
// rows too few blocks work (16 x 16: 6.6 -> 8.9, 15 qubits 6.1 -> 6.2).
__global__ __launch_bounds__(256) void k_expz_block(const float2* state, u64 rows, int n, int g, int nblk,
                                                    double* partial, float* out, int q_only) {
    __shared__ double sm[4][15];
    const u64 row = grid_row();
    if (row >= rows) return;
    const float4* a = reinterpret_cast<const float4*>(state + (row << n)) + (((u64)blockIdx.x << g) * (CHUNK / 2));
    double T = 0.0, z[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};   // bits 0, 9, 10, 11; 12..15
    for (int c = 0; c < (1 << g); ++c) {
        float4 v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = a[(u64)c * (CHUNK / 2) + i * 256 + threadIdx.x];
        double p[16];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            p[2 * i] = (double)prob32(make_float2(v[i].x, v[i].y));
            p[2 * i + 1] = (double)prob32(make_float2(v[i].z, v[i].w));
        }
        double Tc = 0.0, zc[4] = {z[0], z[1], z[2], z[3]};
        expz_tree(p, Tc, zc);
        T += Tc;
#pragma unroll
        for (int j = 0; j < 4; ++j) { z[j] = zc[j]; z[4 + j] += ((c >> j) & 1) ? -Tc : Tc; }
    }
    double zl[6];
    expz_lanes(T, z, zl);                          // lane bits are index bits 1..6
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (lane == 0) {
        sm[wv][0] = T;
#pragma unroll
        for (int j = 0; j < 8; ++j) sm[wv][1 + j] = z[j];
#pragma unroll
        for (int j = 0; j < 6; ++j) sm[wv][9 + j] = zl[j];
    }
    __syncthreads();
    const int e = threadIdx.x;                     // thread e writes entry e
    if (e >= 13 + g) return;
    int from = 0, sign = 0;                        // sm column; 1, 2: signed by that bit of the wavefront's number
    if (e == 1) from = 1;
    else if (e >= 2 && e <= 7) from = 9 + e - 2;
    else if (e == 8 || e == 9) sign = e - 7;
    else if (e >= 10 && e <= 12) from = 2 + e - 10;
    else if (e >= 13) from = 5 + e - 13;
    const double w0 = sm[0][from], w1 = sm[1][from], w2 = sm[2][from], w3 = sm[3][from];
    const double tot = sign == 1 ? (w0 - w1) + (w2 - w3) : sign == 2 ? (w0 + w1) - (w2 + w3) : (w0 + w1) + (w2 + w3);
    if (!out) partial[(row * (u64)(13 + g) + e) * (u64)nblk + blockIdx.x] = tot;
    else if (e > 0 && (q_only < 0 || e - 1 == q_only)) out[q_only < 0 ? row * (u64)n + (e - 1) : row] = (float)tot;
}

// Rows of at most 4096 amplitudes: a wavefront per row, index = step * 128 + lane * 2 + {0, 1}, which writes the
// row's <Z_q> itself (for every qubit, or for q_only alone) or, out = NULL, a record of 13 doubles as
// k_expz_block does with one block per row.  Replaces a block per row, of which a 10-qubit
// row used a quarter: 14 -> 5 us for 1024 rows.
__global__ __launch_bounds__(256) void k_expz_row(const float2* state, u64 rows, int n, int q_only, float* out,
                                                  double* partial) {
    const u64 row = (u64)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    if (row >= rows) return;
    const int lane = threadIdx.x & 63;
    const int pairs = 1 << (n - 1), steps = pairs > 64 ? pairs >> 6 : 1;
    const float4* a = reinterpret_cast<const float4*>(state + (row << n));
    double T = 0.0, z[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};       // bit 0, bits 7..11
#pragma unroll 8
    for (int i = 0; i < steps; ++i) {
        const int k = i * 64 + lane;
        const float4 v = k < pairs ? a[k] : make_float4(0.f, 0.f, 0.f, 0.f);
        const double p0 = (double)prob32(make_float2(v.x, v.y)), p1 = (double)prob32(make_float2(v.z, v.w));
        const double s = p0 + p1;
        T += s;
        z[0] += p0 - p1;
#pragma unroll
        for (int j = 0; j < 5; ++j) z[1 + j] += ((i >> j) & 1) ? -s : s;
    }
    double zl[6];
    expz_lanes(T, z, zl);
    if (lane != 0) return;
    if (!out) partial[row * 13] = T;
    const double all[12] = {z[0], zl[0], zl[1], zl[2], zl[3], zl[4], zl[5], z[1], z[2], z[3], z[4], z[5]};
#pragma unroll
    for (int q = 0; q < 12; ++q) {
        if (!out) partial[row * 13 + 1 + q] = all[q];
        else if (q_only < 0 ? q < n : q == q_only) out[q_only < 0 ? row * (u64)n + q : row] = (float)all[q];
    }
}

// The first of a sample's entries.
__device__ __forceinline__ const double* residues_of(const Residues& res, int rowdep, u64 sample) {
    return res.table + ((rowdep ? sample * (u64)res.stride : 0) + (u64)res.first) * 2;
}

// One wavefront per (row, qubit): combine block partials.  Bits up to 12 + g - 1 use the blocks' signed
// sums; higher bits are constant inside a block, so they sign the block totals.
// WHOLE: a workgroup per (row, qubit), four loads of a thread in flight.  From 1024 partials on, of which there are few sums
// (a wavefront takes 32 of them one after the other, latencies that nothing covers): 24 qubits 9.9 -> 4.6 us.
// SCALED: rows that have come through tables with groups, whose rounded scalars make a row longer or shorter by what res has of
// its sample: that is divided out.  Left in, it makes every <Z> of a row wrong by the same 3e-8 a group (shift rule, 16
// qubits x 16, 10 layers in two passes each, 60 seeds: losses 8.7e-7 from 64 bits, without it 8.5e-7; reverse mode,
// forty shapes, 16 seeds: trash losses 1.03 times as far as layer by layer with it, 0.69 times without, losses of <Z> 1.01 and 1.00).
template <bool WHOLE, bool SCALED = false>
__global__ __launch_bounds__(256) void k_expz_finish(const double* partial, u64 rows, int n, int g, int nblk,
                                                     int q_only, float* out_f, double* out_d,
                                                     Scatter sc, Residues res, int rowdep) {
    __shared__ double sm[WHOLE ? 4 : 1];
    const int lane = WHOLE ? threadIdx.x : threadIdx.x & 63;
    const u64 job = WHOLE ? (u64)blockIdx.x : (u64)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int nq = q_only >= 0 ? 1 : n;
    if (job >= rows * nq) return;
    const u64 row = job / nq;
    const int q = q_only >= 0 ? q_only : (int)(job % nq);
    const double* p = partial + row * (u64)(13 + g) * (u64)nblk;
    double acc = 0.0;
    if constexpr (WHOLE) {                           // nblk is a multiple of 1024
        const bool total = q >= CHUNK_BITS + g;
        const int bit = total ? q - CHUNK_BITS - g : 31;
        if (!total) p += (u64)(1 + q) * (u64)nblk;
        for (int b = lane; b < nblk; b += 1024) {
            double t[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) t[i] = p[b + 256 * i];
#pragma unroll
            for (int i = 0; i < 4; ++i) acc += (((unsigned)(b + 256 * i) >> bit) & 1u) ? -t[i] : t[i];
        }
        acc = block_sum256(acc, sm);
    } else {
        if (q < CHUNK_BITS + g) {
            p += (u64)(1 + q) * (u64)nblk;
            for (int b = lane; b < nblk; b += 64) acc += p[b];
        } else {
            for (int b = lane; b < nblk; b += 64) {
                const double t = p[b];
                acc += ((b >> (q - CHUNK_BITS - g)) & 1) ? -t : t;
            }
        }
        acc = wave_sum(acc);
    }
    if constexpr (SCALED) {
        const double* e = residues_of(res, rowdep, row);
        double m = 1.0;
        for (int k = (int)(threadIdx.x & 63u); k < res.count; k += 64) m *= e[2 * k] * e[2 * k] + e[2 * k + 1] * e[2 * k + 1];
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) m *= __shfl_xor(m, d, 64);
        acc /= m;
    }
    if (lane == 0) {
        u64 o = job;
        if (sc.per > 0) {  // one qubit per row (q_only >= 0): job = row of the chunk
            const u64 gid = (u64)sc.row0 + job;
            o = (gid / (u64)sc.per) * (u64)sc.stride + (u64)sc.offset + gid % (u64)sc.per;
        }
        if (out_f) out_f[o] = (float)acc;
        if (out_d) out_d[o] = acc;
    }
}

// Sums the per-wavefront <Z> partials the last pass wrote, one thread per row, in index order.
__global__ __launch_bounds__(256) void k_zsum_finish(const double* partial, u64 rows, u64 per_row,
                                                     double* out, Scatter sc) {
    const u64 r = (u64)blockIdx.x * 256 + threadIdx.x;
    if (r >= rows) return;
    const double* p = partial + r * per_row;
    double acc = 0.0;
    for (u64 i = 0; i < per_row; ++i) acc += p[i];
    const u64 gid = (u64)sc.row0 + r;
    out[(gid / (u64)sc.per) * (u64)sc.stride + (u64)sc.offset + gid % (u64)sc.per] = acc;
}

// ... of turned rows (see launch_turned_finish), two results a row: a wavefront per row.
struct TurnedArgs { Scatter sc; u64 unturned_at; Residues ra, rb1, rb2; int rowdep; };

__global__ __launch_bounds__(256) void k_turned_finish(const double* partial, u64 rows, u64 per_row, double* out, TurnedArgs t) {
    const u64 r = (u64)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (r >= rows) return;
    const double* p = partial + r * per_row * 3;
    double zb = 0.0, cr = 0.0, ci = 0.0;
    for (u64 i = threadIdx.x & 63u; i < per_row; i += 64) { zb += p[3 * i]; cr += p[3 * i + 1]; ci += p[3 * i + 2]; }
    zb = wave_sum(zb);
    cr = wave_sum(cr);
    ci = wave_sum(ci);
    const u64 gid = (u64)t.sc.row0 + r, sample = gid / (u64)t.sc.per;
    // conj(a) b of the exact states is c / d, d = conj(ra) rb: a lane multiplies every 64th entry
    Cx d = {1.0, 0.0};
    auto take = [&](const Residues& res, double sign) {
        const double* e = residues_of(res, t.rowdep, sample);
        for (int k = (int)(threadIdx.x & 63u); k < res.count; k += 64) d = mul_c(d, {e[2 * k], sign * e[2 * k + 1]});
    };
    take(t.ra, -1.0);
    take(t.rb1, 1.0);
    take(t.rb2, 1.0);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) d = mul_c(d, {__shfl_xor(d.r, o, 64), __shfl_xor(d.i, o, 64)});
    if (threadIdx.x & 63u) return;
    const double cross = (cr * d.r + ci * d.i) / (d.r * d.r + d.i * d.i);
    double* o = out + sample * (u64)t.sc.stride;
    const double half = 0.5 * (o[t.unturned_at] + zb);
    o += (u64)t.sc.offset + gid % (u64)t.sc.per * 2;
    o[0] = half + cross;
    o[1] = half - cross;
}

// Copies each row's starting state from the per-sample source (16 bytes per lane and step).
__global__ __launch_bounds__(256) void k_gather_rows(const float2* src, int n, u64 total, RowMap rm,
                                                     float2* states) {
    const u64 e2 = ((u64)blockIdx.x * 256 + threadIdx.x) * 2;
    if (e2 >= total) return;
    const u64 row = e2 >> n;
    const u64 k = e2 & ((1ull << n) - 1);
    const u64 sample = row_ctx(rm, row).sample;
    *reinterpret_cast<float4*>(states + e2) = *reinterpret_cast<const float4*>(src + ((sample << n) | k));
}

__device__ __forceinline__ u64 deposit(u64 v, u64 mask, int n) {  // spread the bits of v over mask
    u64 o = 0;
    int j = 0;
    for (int q = 0; q < n; ++q)
        if ((mask >> q) & 1) { o |= ((v >> j) & 1ull) << q; ++j; }
    return o;
}

// Block (row, v, blk): sum of p over the indices whose mask bits read v, 4096 of them per block.
__global__ __launch_bounds__(256) void k_marginal_block(const float2* state, int n, u64 mask, u64 n_v,
                                                        u64 nblk, u64 sub, double* partial) {
    __shared__ double sm[4];
    const u64 id = blockIdx.x;
    const u64 blk = id % nblk;
    const u64 v = (id / nblk) % n_v;
    const u64 row = id / (nblk * n_v);
    const u64 fixed = deposit(v, mask, n);
    const u64 free_mask = ((1ull << n) - 1) & ~mask;
    const float2* a = state + (row << n);
    double acc = 0.0;
    if ((free_mask & (CHUNK - 1)) == (u64)(CHUNK - 1)) {
        // no mask bit among the low 12 index bits: a block's elements are contiguous
        // (and so sub >= 4096: every block is full)
        const float4* ab = reinterpret_cast<const float4*>(a + (fixed | deposit(blk * CHUNK, free_mask, n)));
        float4 v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = ab[i * 256 + threadIdx.x];
#pragma unroll
        for (int i = 0; i < 8; ++i)
            acc += (double)prob32(make_float2(v[i].x, v[i].y)) + (double)prob32(make_float2(v[i].z, v[i].w));
    } else {
#pragma unroll 4
        for (int i = 0; i < 16; ++i) {
            const u64 j = blk * CHUNK + (u64)i * 256 + threadIdx.x;
            if (j < sub) acc += (double)prob32(a[fixed | deposit(j, free_mask, n)]);
        }
    }
    const double tot = block_sum256(acc, sm);
    if (threadIdx.x == 0) partial[id] = tot;
}

// One wavefront per (row, v).  renorm_mode: 0 plain marginal; 1 also scale = 1; 2 also
// scale = 1/sqrt(P) (0 when P = 0).
__global__ __launch_bounds__(256) void k_marginal_finish(const double* partial, u64 jobs, u64 nblk,
                                                         float* out, int renorm_mode, double* scale) {
    const int lane = threadIdx.x & 63;
    const u64 job = (u64)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (job >= jobs) return;
    double acc = 0.0;
    for (u64 b = lane; b < nblk; b += 64) acc += partial[job * nblk + b];
    acc = wave_sum(acc);
    if (lane == 0) {
        out[job] = (float)acc;
        if (renorm_mode == 1) scale[job] = 1.0;
        if (renorm_mode == 2) scale[job] = acc > 0.0 ? 1.0 / sqrt(acc) : 0.0;
    }
}

__global__ __launch_bounds__(256) void k_project(float2* state, u64 total, int n, u64 mask,
                                                 const double* scale) {
    const u64 e = (u64)blockIdx.x * 256 + threadIdx.x;
    if (e >= total) return;
    float2 v = state[e];
    if (e & mask) {  // mask has no bits at or above n
        v.x = 0.f; v.y = 0.f;
    } else {
        const double sc = scale[e >> n];
        v.x = (float)((double)v.x * sc);
        v.y = (float)((double)v.y * sc);
    }
    state[e] = v;
}

// Pauli string: T = sum_k conj(a[k ^ f]) (-1)^popcount(k & s) a[k], f = X and Y bits, s = Y and Z
// bits; <P> = Re(i^nY T).  The terms of k and k ^ f are conjugates of each other up to the sign
// (-1)^nY, so for f != 0 only the k whose highest flip bit is clear are visited, each amplitude is
// read once, and a pair adds 2 Re t (nY even) or 2 i Im t (nY odd) with t = conj(a[k ^ f]) sign(k) a[k].
// One block per 4096 visited indices and row; partial: [row][blk][2].
__global__ __launch_bounds__(256) void k_pauli_block(const float2* state, u64 rows, int n, u64 f, u64 s, int ny,
                                                     int nblk, double* partial) {
    __shared__ double sm[4];
    const u64 row = grid_row();
    if (row >= rows) return;
    const float2* a = state + (row << n);
    float tr = 0.f, ti = 0.f;
    if (f == 0) {
        const u64 N = 1ull << n;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const u64 k = (u64)blockIdx.x * CHUNK + (u64)i * 256 + threadIdx.x;
            if (k < N) {
                const float2 v = a[k];
                const float p = v.x * v.x + v.y * v.y;
                tr += (__popcll(k & s) & 1) ? -p : p;
            }
        }
    } else {
        const int hb = 63 - __clzll(f);               // pairs differ in this bit (and the lower bits of f)
        const u64 half = 1ull << (n - 1), low = (1ull << hb) - 1ull;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const u64 j = (u64)blockIdx.x * CHUNK + (u64)i * 256 + threadIdx.x;
            if (j < half) {
                const u64 k = ((j & ~low) << 1) | (j & low);        // bit hb clear
                const float2 v = a[k], u = a[k ^ f];
                float cr = u.x * v.x + u.y * v.y, ci = u.x * v.y - u.y * v.x;   // conj(u) v
                if (__popcll(k & s) & 1) { cr = -cr; ci = -ci; }
                if (ny & 1) ti += 2.f * ci; else tr += 2.f * cr;
            }
        }
    }
    const double t0 = block_sum256((double)tr, sm);
    const double t1 = block_sum256((double)ti, sm);
    if (threadIdx.x == 0) { double* o = partial + (row * nblk + blockIdx.x) * 2; o[0] = t0; o[1] = t1; }
}

__global__ __launch_bounds__(256) void k_pauli_finish(const double* partial, int nblk, int ny, float* out) {
    __shared__ double sm[4];
    const u64 row = blockIdx.x;
    double tr = 0.0, ti = 0.0;
    for (int i = threadIdx.x; i < nblk; i += 256) {
        const double* p = partial + (row * nblk + i) * 2;
        tr += p[0]; ti += p[1];
    }
    const double t0 = block_sum256(tr, sm);
    const double t1 = block_sum256(ti, sm);
    // Re(i^ny (t0 + i t1)): ny mod 4 = 0: t0; 1: -t1; 2: -t0; 3: t1
    if (threadIdx.x == 0) out[row] = (float)((ny & 3) == 0 ? t0 : (ny & 3) == 1 ? -t1 : (ny & 3) == 2 ? -t0 : t1);
}

__global__ __launch_bounds__(256) void k_fidelity_block(const float2* state, u64 rows, int n, const float* x,
                                                        u64 dim, int nblk, RowMap rm, double* partial) {
    __shared__ double sm[4];
    const u64 row = grid_row();
    if (row >= rows) return;
    const float2* a = state + (row << n);
    const float* xb = x + row_ctx(rm, row).sample * dim;
    double sxx = 0.0, sr = 0.0, si = 0.0;
    auto add = [&](float xf, float re, float im) {
        const double xv = (double)xf;
        sxx += xv * xv;
        sr += xv * (double)re;
        si += xv * (double)im;
    };
    // full chunks of x rows that start on 8 bytes: two entries per load (24 qubits 47 -> 30 us)
    const bool pairs = ((u64)(uintptr_t)xb & 7) == 0;
    for (u64 base = (u64)blockIdx.x * CHUNK; base < dim; base += (u64)nblk * CHUNK) {
        if (pairs && base + CHUNK <= dim) {
            const float2* x2 = reinterpret_cast<const float2*>(xb + base);
            const float4* a2 = reinterpret_cast<const float4*>(a + base);
            float2 xv[8];
            float4 av[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) { xv[i] = x2[i * 256 + threadIdx.x]; av[i] = a2[i * 256 + threadIdx.x]; }
#pragma unroll
            for (int i = 0; i < 8; ++i) { add(xv[i].x, av[i].x, av[i].y); add(xv[i].y, av[i].z, av[i].w); }
        } else {
#pragma unroll 4
            for (int i = 0; i < 16; ++i) {
                const u64 k = base + (u64)i * 256 + threadIdx.x;
                if (k < dim) { const float2 av = a[k]; add(xb[k], av.x, av.y); }
            }
        }
    }
    const double t0 = block_sum256(sxx, sm);
    const double t1 = block_sum256(sr, sm);
    const double t2 = block_sum256(si, sm);
    if (threadIdx.x == 0) {
        double* o = partial + (row * nblk + blockIdx.x) * 3;
        o[0] = t0; o[1] = t1; o[2] = t2;
    }
}

__global__ __launch_bounds__(256) void k_fidelity_finish(const double* partial, int nblk, float* out,
                                                         double* out_d) {
    __shared__ double sm[4];
    const u64 row = blockIdx.x;
    double sxx = 0.0, sr = 0.0, si = 0.0;
    for (int i = threadIdx.x; i < nblk; i += 256) {
        const double* p = partial + (row * nblk + i) * 3;
        sxx += p[0]; sr += p[1]; si += p[2];
    }
    const double t0 = block_sum256(sxx, sm);
    const double t1 = block_sum256(sr, sm);
    const double t2 = block_sum256(si, sm);
    if (threadIdx.x == 0) {
        const double F = t0 > 0.0 ? (t1 * t1 + t2 * t2) / t0 : 0.0;
        if (out) out[row] = (float)F;
        if (out_d) out_d[row] = F;
    }
}

// Trash reset: row gid = row0 + r stands for (sample, outcome t) = (gid / per, gid % per), per = 2^m.
// work[r][k] = state[sample][k | bits of t spread over mask] where k has no mask bit, else 0.
__global__ __launch_bounds__(256) void k_reset_rows(const float2* state, int n, u64 mask, u64 total,
                                                    RowMap rm, float2* work) {
    const u64 e2 = ((u64)blockIdx.x * 256 + threadIdx.x) * 2;
    if (e2 >= total) return;
    const u64 r = e2 >> n, k = e2 & ((1ull << n) - 1);
    const u64 gid = (u64)rm.row0 + r;
    const u64 sample = gid / (u64)rm.per, t = gid % (u64)rm.per;
    const u64 tb = deposit(t, mask, n);
    const float2* src = state + (sample << n);
    float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
    if ((k & mask) == 0) { const float2 v = src[k | tb]; o.x = v.x; o.y = v.y; }
    if (((k + 1) & mask) == 0) { const float2 v = src[(k + 1) | tb]; o.z = v.x; o.w = v.y; }
    *reinterpret_cast<float4*>(work + e2) = o;
}

// out[b] = sum over the per outcomes of Frow[b * per + t], in order.
__global__ __launch_bounds__(256) void k_reset_sum(const double* Frow, u64 per, u64 B, float* out) {
    const u64 b = (u64)blockIdx.x * 256 + threadIdx.x;
    if (b >= B) return;
    double acc = 0.0;
    for (u64 t = 0; t < per; ++t) acc += Frow[b * per + t];
    out[b] = (float)acc;
}

// <Z_q> of every qubit from the samples of a row: one block per row.  A wavefront takes 64 samples at a time and
// counts the set bits of every qubit by a ballot, so that a sample is read once and not once per qubit;
// whole numbers, so the mean is the same (24 qubits, 4096 shots: 22 -> 9 us).
__global__ __launch_bounds__(1024) void k_shot_expz(const long long* samples, u64 shots, int n, float* out) {
    __shared__ unsigned long long ones[31];        // per qubit, and the valid samples behind them
    const u64 row = blockIdx.x;
    for (int q = threadIdx.x; q <= n; q += blockDim.x) ones[q] = 0;
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const long long* s = samples + row * shots;
    u64 mine = 0;                                   // lane q: the count of qubit q; lane n: the valid ones
    for (u64 i0 = (u64)(threadIdx.x & ~63u); i0 < shots; i0 += blockDim.x) {
        const u64 i = i0 + lane;
        const long long v = i < shots ? s[i] : -1;
        const u64 valid = __ballot(v >= 0);
        if (lane == n) mine += __popcll(valid);
        for (int q = 0; q < n; ++q) {
            const u64 set = __ballot((v >> q) & 1) & valid;
            if (lane == q) mine += __popcll(set);
        }
    }
    if (lane <= n && mine) atomicAdd(&ones[lane], (unsigned long long)mine);
    __syncthreads();
    if ((int)threadIdx.x < n) {
        const double cnt = (double)ones[n], acc = cnt - 2.0 * (double)ones[threadIdx.x];
        out[row * n + threadIdx.x] = cnt > 0.0 ? (float)(acc / cnt) : 0.f;
    }
}

// ------------------------------------------------------------------------------------------
// Sampling: integer inverse CDF (see qsv.h).  All sums are uint64, hence order-independent.
__device__ __forceinline__ u64 weight60(float2 a) {
    const double p = (double)prob32(a);
    return p > 0.0 ? (u64)(p * 1152921504606846976.0) : 0ull;  // 2^60, truncation = floor
}

__device__ __forceinline__ u64 wave_sum_u64(u64 v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// sub (may be NULL): [row][nblk][16] sums of 256 consecutive amplitudes each.
__global__ __launch_bounds__(256) void k_sample_blocksum(const float2* state, u64 rows, int n, int nblk, u64* bsum,
                                                         u64* sub) {
    __shared__ u64 sm[16];
    const u64 row = grid_row();
    if (row >= rows) return;
    const u64 dimn = 1ull << n;
    const float2* a = state + (row << n);
    const int grp = threadIdx.x >> 4, in = threadIdx.x & 15;     // 16 lanes take 256 amplitudes
    u64 acc = 0;
    if (dimn >= 2) {
        // two amplitudes per 16-byte load; integer sums do not care about the order
        const float4* a2 = reinterpret_cast<const float4*>(a);
        float4 v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const u64 k2 = (u64)blockIdx.x * (CHUNK / 2) + (u64)grp * 128 + (u64)i * 16 + in;
            v[i] = k2 * 2 < dimn ? a2[k2] : make_float4(0.f, 0.f, 0.f, 0.f);
        }
#pragma unroll
        for (int i = 0; i < 8; ++i)
            acc += weight60(make_float2(v[i].x, v[i].y)) + weight60(make_float2(v[i].z, v[i].w));
    } else if (blockIdx.x == 0 && threadIdx.x == 0) {
        acc = weight60(a[0]);
    }
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
    if (in == 0) {
        sm[grp] = acc;
        if (sub) sub[(row * nblk + blockIdx.x) * 16 + grp] = acc;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        u64 tot = 0;
        for (int g = 0; g < 16; ++g) tot += sm[g];
        bsum[row * nblk + blockIdx.x] = tot;
    }
}

// In-place inclusive prefix sum of each row's block sums (one 1024-thread block per row).
__global__ __launch_bounds__(1024) void k_sample_scan(u64* cum, int nblk) {
    __shared__ u64 sm[1024];
    u64* c = cum + (u64)blockIdx.x * nblk;
    const int per = (nblk + 1023) / 1024;
    const int lo = threadIdx.x * per;
    const int hi = min(lo + per, nblk);
    u64 loc = 0;
    for (int i = lo; i < hi; ++i) loc += c[i];
    sm[threadIdx.x] = loc;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {
        u64 add = 0;
        if ((int)threadIdx.x >= o) add = sm[threadIdx.x - o];
        __syncthreads();
        sm[threadIdx.x] += add;
        __syncthreads();
    }
    u64 run = sm[threadIdx.x] - loc;  // exclusive prefix of this thread's span
    for (int i = lo; i < hi; ++i) { run += c[i]; c[i] = run; }
}

// Inclusive sums over the first `width` lanes.
__device__ __forceinline__ u64 scan_u64(u64 v, int width, int lane) {
    for (int o = 1; o < width; o <<= 1) {
        const u64 up = __shfl_up(v, o, 64);
        if (lane >= o) v += up;
    }
    return v;
}

// One wavefront per shot.  The block is found by a search with 64 probes at a time (two loads in turn for 4096 blocks instead of 12);
// with sub the 256 amplitudes in question by its 16 sums, without it by scanning the block's 4096 (24 qubits,
// 4096 shots: 51 -> 6 us).
__global__ __launch_bounds__(256) void k_sample_draw(const float2* state, int n, int nblk, const u64* cum,
                                                     const u64* sub, const double* uniforms, u64 shots, u64 jobs,
                                                     long long* out) {
    const int lane = threadIdx.x & 63;
    const u64 job = (u64)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (job >= jobs) return;
    const u64 row = job / shots;
    const u64* c = cum + row * nblk;
    const u64 W = c[nblk - 1];
    if (W == 0) { if (lane == 0) out[job] = -1; return; }
    const u64 r = (u64)(uniforms[job] * 9007199254740992.0);  // floor(u * 2^53)
    const u64 t = (__umul64hi(r, W) << 11) | ((r * W) >> 53);   // floor(r * W / 2^53)
    int lo = 0, len = nblk;                                     // smallest block with cum > t is in lo..lo+len-1
    while (len > 1) {
        const int stride = (len + 63) >> 6;
        const int probe = min((lane + 1) * stride, len) - 1;    // the last block of the lane's part
        const u64 hit = __ballot(c[lo + probe] > t);            // never empty for t < W
        const int f = hit ? __ffsll((long long)hit) - 1 : 63;
        const int off = min(f * stride, len - 1);
        lo += off;
        len = min(stride, len - off);
    }
    u64 base = lo > 0 ? c[lo - 1] : 0;
    const u64 dimn = 1ull << n;
    const float2* a = state + (row << n);
    u64 k0 = (u64)lo * CHUNK;
    long long found = -1;
    if (sub) {
        const u64 own = lane < 16 ? sub[(row * nblk + lo) * 16 + lane] : 0ull;
        const u64 incl = scan_u64(own, 16, lane);
        const u64 hit = __ballot(lane < 16 && base + incl > t);
        if (hit) {
            const int g = __ffsll((long long)hit) - 1;
            base += __shfl(incl - own, g, 64);
            k0 += (u64)g * 256 + (u64)lane * 4;                 // four amplitudes per lane
            u64 w[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) w[i] = k0 + i < dimn ? weight60(a[k0 + i]) : 0ull;
            const u64 four = w[0] + w[1] + w[2] + w[3];
            u64 run = base + scan_u64(four, 64, lane) - four;
            int at = 4;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                run += w[i];
                if (at == 4 && run > t) at = i;
            }
            const u64 who = __ballot(at < 4);
            if (who) found = __shfl((long long)(k0 + at), __ffsll((long long)who) - 1, 64);
        }
    } else {
        for (int it = 0; it < CHUNK / 64; ++it) {
            const u64 k = k0 + (u64)it * 64 + lane;
            const u64 incl = scan_u64(k < dimn ? weight60(a[k]) : 0ull, 64, lane);
            const u64 hit = __ballot(base + incl > t);
            if (hit) { found = (long long)(k0 + (u64)it * 64 + (u64)(__ffsll((long long)hit) - 1)); break; }
            base += __shfl(incl, 63, 64);
        }
    }
    if (lane == 0) out[job] = found;
}

// ------------------------------------------------------------------------------------------
// Gradient assembly.
__global__ __launch_bounds__(256) void k_grad_finish(const double* f, u64 B, u64 P, CircDev c,
                                                     const float* feats, float* loss, float* grad) {
    const u64 idx = (u64)blockIdx.x * 256 + threadIdx.x;
    if (idx >= B * (P + 1)) return;
    const u64 b = idx / (P + 1), p = idx % (P + 1);
    const double* fb = f + b * (2 * P + 1);
    if (p == P) { if (loss) loss[b] = (float)fb[2 * P]; return; }
    double g = 0.5 * (fb[2 * p] - fb[2 * p + 1]);
    const int slots = c.reupload + c.n_rot;
    if (c.reupload && ((p / c.n) % slots) == 0) g *= (double)feats[b * c.n + (p % c.n)];
    grad[b * P + p] = (float)g;
}

// Batch means in a fixed order: one block per parameter (block P does the loss); thread t adds the
// samples t, t + 256, ... and the block adds its threads.
__global__ __launch_bounds__(256) void k_grad_mean(const double* f, u64 B, u64 P, CircDev c,
                                                   const float* feats, float* mean_loss,
                                                   float* mean_grad) {
    __shared__ double sm[4];
    const u64 p = blockIdx.x;
    const int slots = c.reupload + c.n_rot;
    double acc = 0.0;
    if (p == P) {
        if (!mean_loss) return;
        for (u64 b = threadIdx.x; b < B; b += 256) acc += f[b * (2 * P + 1) + 2 * P];
        const double tot = block_sum256(acc, sm);
        if (threadIdx.x == 0) mean_loss[0] = (float)(tot / (double)B);
        return;
    }
    if (!mean_grad) return;
    const bool isw = c.reupload && ((p / c.n) % slots) == 0;
    for (u64 b = threadIdx.x; b < B; b += 256) {
        const double* fb = f + b * (2 * P + 1);
        double g = 0.5 * (fb[2 * p] - fb[2 * p + 1]);
        if (isw) g *= (double)feats[b * c.n + (p % c.n)];
        acc += g;
    }
    const double tot = block_sum256(acc, sm);
    if (threadIdx.x == 0) mean_grad[p] = (float)(tot / (double)B);
}

// ------------------------------------------------------------------------------------------
// Reverse-mode (adjoint) gradient of <Z_obs>.  Rows come in pairs: 2r holds psi, 2r+1 holds lambda.

// S[2r] = A[r], S[2r+1] = O A[r].
__global__ __launch_bounds__(256) void k_adj_init(const float2* A, int n, AdjObs o, u64 total, float2* S,
                                                  int paired) {
    const u64 e2 = ((u64)blockIdx.x * 256 + threadIdx.x) * 2;
    if (e2 >= total) return;
    const u64 r = e2 >> n, k = e2 & ((1ull << n) - 1);
    const float4 v = *reinterpret_cast<const float4*>(A + e2);
    const float w0 = adj_weight(o, r, k, n), w1 = adj_weight(o, r, k + 1, n);
    float4 z;
    z.x = w0 * v.x; z.y = w0 * v.y; z.z = w1 * v.z; z.w = w1 * v.w;
    if (paired) {
        *reinterpret_cast<float4*>(S + (((2 * r) << n) | k)) = v;
        *reinterpret_cast<float4*>(S + (((2 * r + 1) << n) | k)) = z;
    } else {
        *reinterpret_cast<float4*>(S + e2) = z;
    }
}

// P0(mask) of every row: block partials, then one thread per row; f[sample][2P] = 1 - P0.
__global__ __launch_bounds__(256) void k_p0_block(const float2* A, u64 rows, int n, u64 mask, int nblk, double* partial) {
    __shared__ double sm[4];
    const u64 r = grid_row(), N = 1ull << n;
    if (r >= rows) return;
    const float2* a = A + (r << n);
    float acc = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const u64 k = (u64)blockIdx.x * 4096 + (u64)i * 256 + threadIdx.x;
        if (k < N && (k & mask) == 0) { const float2 v = a[k]; acc += v.x * v.x + v.y * v.y; }
    }
    const double t = block_sum256((double)acc, sm);
    if (threadIdx.x == 0) partial[r * nblk + blockIdx.x] = t;
}

// SCALED: see k_expz_finish.
template <bool SCALED>
__global__ __launch_bounds__(256) void k_trash_loss(const double* partial, int nblk, u64 rows, u64 sample0,
                                                    u64 P, double* f, Residues res, int rowdep) {
    const u64 r = (u64)blockIdx.x * 256 + threadIdx.x;
    if (r >= rows) return;
    double acc = 0.0;
    for (int b = 0; b < nblk; ++b) acc += partial[r * nblk + b];
    if constexpr (SCALED) {
        const double* e = residues_of(res, rowdep, r);
        double m = 1.0;
        for (int k = 0; k < res.count; ++k) m *= e[2 * k] * e[2 * k] + e[2 * k + 1] * e[2 * k + 1];
        acc /= m;
    }
    f[(sample0 + r) * (2 * P + 1) + 2 * P] = 1.0 - acc;
}

// Squared-error loss on <Z_q>: z [rows][n] (double), y [samples][n] (float):
// f[sample][2P] = 1/n sum (z - y)^2 and coef[r][q] = 2/n (z - y), the weights of the Z_q in lambda.
__global__ __launch_bounds__(256) void k_mse_coef(const double* z, const float* y, int n, u64 rows,
                                                  u64 sample0, u64 P, double* coef, double* f) {
    const u64 r = (u64)blockIdx.x * 256 + threadIdx.x;
    if (r >= rows) return;
    double acc = 0.0;
    for (int q = 0; q < n; ++q) {
        const double d = z[r * n + q] - (double)y[(sample0 + r) * n + q];
        acc += d * d;
        coef[r * n + q] = 2.0 * d / n;
    }
    f[(sample0 + r) * (2 * P + 1) + 2 * P] = acc / n;
}

// M_q[a][b] = sum over the other qubits of conj(lambda[a, rest]) psi[b, rest], for one row pair
// (blockIdx.z) and one qubit (blockIdx.y); a block covers 4096 index pairs and writes 8 doubles in
// the layout (re, im of M00, M01, M10, M11).  The derivative is 2 Re sum_ab Bt[a][b] M[a][b] with an
// anti-Hermitian Bt (Bt00, Bt11 imaginary, Bt10 = -conj(Bt01)), which equals
// -2 (Im Bt00 Im M00 + Im Bt11 Im M11) + 2 Re(Bt01 K) with K = M01 - conj(M10).  So only Im M00,
// Im M11 and K are summed; K is stored in the place of M01 and the other entries are zero, which lets
// k_adj_layers use the plain formula.  Pair r is (psi0 + rstride r 2^n, lam0 + rstride r 2^n): the two
// states interleaved in one buffer (lam0 = psi0 + 2^n, rstride 2) or in buffers of their own (rstride 1).
__global__ __launch_bounds__(256) void k_trans_block(const float2* psi0, const float2* lam0, int rstride, int n,
                                                     u64 pairs, int nblk, double* partial) {
    __shared__ double sm[4];
    const int q = blockIdx.y;
    const u64 r = blockIdx.z;
    const float2* psi = psi0 + ((rstride * r) << n);
    const float2* lam = lam0 + ((rstride * r) << n);
    const u64 bit = 1ull << q;
    float acc[4];   // Im M00, Re K, Im K, Im M11
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[j] = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const u64 p = (u64)blockIdx.x * 4096 + (u64)i * 256 + threadIdx.x;
        if (p < pairs) {
            const u64 k0 = ((p >> q) << (q + 1)) | (p & (bit - 1));
            const u64 k1 = k0 | bit;
            const float2 l0 = lam[k0], l1 = lam[k1], s0 = psi[k0], s1 = psi[k1];
            acc[0] += l0.x * s0.y - l0.y * s0.x;
            acc[3] += l1.x * s1.y - l1.y * s1.x;
            acc[1] += (l0.x * s1.x + l0.y * s1.y) - (l1.x * s0.x + l1.y * s0.y);
            acc[2] += (l0.x * s1.y - l0.y * s1.x) + (l1.x * s0.y - l1.y * s0.x);
        }
    }
    double* out = partial + ((r * n + q) * (u64)nblk + blockIdx.x) * 8;
    const double m00 = block_sum256((double)acc[0], sm), kre = block_sum256((double)acc[1], sm);
    const double kim = block_sum256((double)acc[2], sm), m11 = block_sum256((double)acc[3], sm);
    if (threadIdx.x == 0) {
        out[0] = 0.0; out[1] = m00; out[2] = kre; out[3] = kim;
        out[4] = 0.0; out[5] = 0.0; out[6] = 0.0; out[7] = m11;
    }
}

// The same sums for n >= 12, several qubits per read of the two states: a workgroup takes a tile of
// 2^12 amplitudes of psi and of lambda (tile = the c lowest index bits plus 12 - c bits from bit w,
// as in the pass kernel) and forms the index pairs of a qubit in registers: a lane holds, of each
// state, a run of amplitudes that differ in a few tile bits.
// Arithmetic per amplitude and qubit (only Im M00, Im M11 and K = M01 - conj(M10) are needed, see
// k_trans_block): d = Im conj(lambda[k]) psi[k] does not depend on the qubit, Im M00 sums it over the
// indices with the bit clear, and Im (M00 + M11) = sum of all d is the same for every qubit, so it is
// kept once (tsum) and Im M11 comes out as a difference at the end; K takes 8 FMAs per index pair.
// A workgroup covers `per_group` consecutive tiles of one row pair before it reduces its
// accumulators, so the reduction is amortised.
// partial: [(pair * n + qubit) * nblk + group * 4 + wavefront][8] (nblk = 4 * groups), the layout
// k_trans_finish reads.

// A pointer to global memory that is the same in every lane, moved to scalar registers so that loads
// through it take the scalar-base + 32-bit lane offset form (no 64-bit address per lane).
typedef const __attribute__((address_space(1))) char* global_bytes;
__device__ __forceinline__ global_bytes uniform_ptr(const void* p) {
    const u64 v = (u64)p;
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)v);
    const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(v >> 32));
    return (global_bytes)(((u64)hi << 32) | lo);
}
__device__ __forceinline__ float2 load_f2(global_bytes base, unsigned byte_offset) {
    const f32x2 v = *(const __attribute__((address_space(1))) f32x2*)(base + byte_offset);
    return make_float2(v.x, v.y);
}

template <int N>
__device__ __forceinline__ void trans_diag(const float2 (&s)[N], const float2 (&l)[N], float (&d)[N],
                                           float& tsum) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
        d[i] = fmaf(-l[i].y, s[i].x, l[i].x * s[i].y);      // Im conj(lambda) psi
        tsum += d[i];
    }
}

// acc: Im M00, Re K, Im K of the qubit behind run bit BIT (K = M01 - conj(M10))
template <int N, int BIT>
__device__ __forceinline__ void trans_acc(const float2 (&s)[N], const float2 (&l)[N], const float (&d)[N],
                                          float (&acc)[3]) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
        if (i & (1 << BIT)) continue;
        constexpr int B = 1 << BIT;
        acc[0] += d[i];
        acc[1] = fmaf(-l[i | B].y, s[i].y, fmaf(-l[i | B].x, s[i].x,
                 fmaf(l[i].y, s[i | B].y, fmaf(l[i].x, s[i | B].x, acc[1]))));
        acc[2] = fmaf(-l[i | B].y, s[i].x, fmaf(l[i | B].x, s[i].y,
                 fmaf(-l[i].y, s[i | B].x, fmaf(l[i].x, s[i | B].y, acc[2]))));
    }
}

// What a wavefront writes for one qubit: the 8-double layout of k_trans_block.
__device__ __forceinline__ void trans_store(double* out, double m00, double kre, double kim, double tsum) {
    out[0] = 0.0; out[1] = m00; out[2] = kre; out[3] = kim;
    out[4] = 0.0; out[5] = 0.0; out[6] = 0.0; out[7] = tsum - m00;
}

// Tile bits J0..11, J0 >= 8 (a window of which only the top bits are still wanted): they are the run
// of the 16 amplitudes a lane loads from memory (tau = i * 256 + lane index, coalesced), so nothing
// goes through LDS.
template <int J0>
__global__ __launch_bounds__(256) void k_trans_tile(const float2* psi0, const float2* lam0, int rstride, int n,
                                                    int c, int w, int per_group, int nblk, double* partial) {
    static_assert(J0 >= 8 && J0 < 12, "lower tile bits are served by k_trans_wave");
    constexpr int NJ = 12 - J0;                      // acc[a] belongs to tile bit J0 + a
    const u64 r = blockIdx.y;
    const float2* psi = psi0 + ((rstride * r) << n);
    const float2* lam = lam0 + ((rstride * r) << n);
    const unsigned t = threadIdx.x;
    const unsigned cmask = (1u << c) - 1u;
    const int wc = w - c;
    float acc[NJ][3];
    float tsum = 0.f;
#pragma unroll
    for (int a = 0; a < NJ; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) acc[a][b] = 0.f;
    // tau = i * 256 + t sits at index base | (tau & cmask) | (tau >> c) << w = base + i * stride + kt, both
    // for contiguous tiles (c = 12) and for c = 4 (tau >> 4 = i * 16 + (t >> 4)); base + i * stride is the
    // same for all lanes (scalar registers), kt a 32-bit lane offset
    const u64 stride = c == 12 ? 256ull : (16ull << w);
    const unsigned kt8 = ((t & cmask) | ((t >> c) << w)) * 8u;   // in bytes: below 2^(n-1)
    for (int g = 0; g < per_group; ++g) {
        const u64 tb = (u64)blockIdx.x * per_group + g;      // tile of the row
        const u64 base = ((tb & ((1ull << wc) - 1ull)) << c) | ((tb >> wc) << (w + 12 - c));
        float2 s[16], l[16];
        float d[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            s[i] = load_f2(uniform_ptr(psi + (base + (u64)i * stride)), kt8);
            l[i] = load_f2(uniform_ptr(lam + (base + (u64)i * stride)), kt8);
        }
        trans_diag<16>(s, l, d, tsum);
        if constexpr (J0 <= 8) trans_acc<16, 0>(s, l, d, acc[J0 <= 8 ? 8 - J0 : 0]);
        if constexpr (J0 <= 9) trans_acc<16, 1>(s, l, d, acc[J0 <= 9 ? 9 - J0 : 0]);
        if constexpr (J0 <= 10) trans_acc<16, 2>(s, l, d, acc[J0 <= 10 ? 10 - J0 : 0]);
        trans_acc<16, 3>(s, l, d, acc[11 - J0]);
    }
    // every wavefront writes its own partial: index (group, wavefront)
    const double t1 = wave_sum((double)tsum);
#pragma unroll
    for (int a = 0; a < NJ; ++a) {
        const int j = J0 + a;
        const int q = j < c ? j : j - c + w;                 // the qubit behind tile bit j
        double* out = partial + ((r * n + q) * (u64)nblk + (u64)blockIdx.x * 4 + (t >> 6)) * 8;
        double tot[3];
#pragma unroll
        for (int b = 0; b < 3; ++b) tot[b] = wave_sum((double)acc[a][b]);
        if ((t & 63u) == 0) trans_store(out, tot[0], tot[1], tot[2], t1);
    }
}

// Where the 12 bits of a tile index come from when a wavefront reads the tile from LDS in runs of RB
// bits starting at tile bit R0: pos[0..RB) = the run, pos[RB..RB+6) = the lane bits, the rest = the
// step counter h.  The four low lane bits are placed so that, after the swizzle tau ^ ((tau >> 4) & 15),
// 16 consecutive lanes fall on 16 different 8-byte slots of a 128-byte row: into the free bits of the
// low nibble, and, for every low-nibble bit p the run occupies, into bit p + 4 (which the swizzle
// folds onto p).
template <int RB, int R0>
struct TransMap {
    int pos[12];
    constexpr TransMap() : pos{} {
        bool used[12] = {};
        int k = 0;
        for (int j = 0; j < RB; ++j) { pos[k++] = R0 + j; used[R0 + j] = true; }
        for (int p = 0; p < 4; ++p)
            if (!used[p]) { pos[k++] = p; used[p] = true; }
        for (int j = 0; j < RB; ++j)
            if (R0 + j < 4) { pos[k++] = R0 + j + 4; used[R0 + j + 4] = true; }
        for (int p = 0; p < 12; ++p)
            if (!used[p]) { pos[k++] = p; used[p] = true; }
    }
    // bits [first, first + count) of the source list take the low bits of v
    constexpr unsigned deposit(int first, int count, unsigned v) const {
        unsigned a = 0;
        for (int j = 0; j < count; ++j) a |= ((v >> j) & 1u) << pos[first + j];
        return a;
    }
};
__device__ constexpr unsigned trans_swz(unsigned tau) { return tau ^ ((tau >> 4) & 15u); }

// One wavefront, the whole tile in LDS, the qubits behind tile bits R0..R0+RB-1: 2^(6-RB) steps of one
// run per lane; the reads of a step are issued before the sums of the step before it.
template <int RB, int R0>
__device__ __forceinline__ void trans_wave(const float2* ps, const float2* lm, unsigned lane,
                                           float (&acc)[RB][3], float& tsum) {
    constexpr TransMap<RB, R0> map{};
    constexpr int NR = 1 << RB, HB = 6 - RB, NH = 1 << HB;
    unsigned lp = 0;
#pragma unroll
    for (int j = 0; j < 6; ++j) lp |= ((lane >> j) & 1u) << map.pos[RB + j];
    lp = trans_swz(lp);                              // the swizzle is linear over XOR
    float2 rs[2][NR], rl[2][NR];
    auto read_step = [&](int h, float2 (&a)[NR], float2 (&b)[NR]) __attribute__((always_inline)) {
        unsigned hp = 0;
#pragma unroll
        for (int j = 0; j < HB; ++j) hp |= (((unsigned)h >> j) & 1u) << map.pos[RB + 6 + j];
        const unsigned base = lp ^ trans_swz(hp);
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            const unsigned ip = trans_swz(map.deposit(0, RB, (unsigned)i));
            a[i] = ps[base ^ ip];
            b[i] = lm[base ^ ip];
        }
    };
    auto sums = [&](const float2 (&a)[NR], const float2 (&b)[NR]) __attribute__((always_inline)) {
        float d[NR];
        trans_diag<NR>(a, b, d, tsum);
        trans_acc<NR, 0>(a, b, d, acc[0]);
        trans_acc<NR, 1>(a, b, d, acc[1]);
        if constexpr (RB > 2) trans_acc<NR, 2>(a, b, d, acc[RB > 2 ? 2 : 0]);
    };
    read_step(0, rs[0], rl[0]);
#pragma unroll 1
    for (int h = 0; h < NH; h += 2) {
        read_step(h + 1, rs[1], rl[1]);
        sums(rs[0], rl[0]);
        if (h + 2 < NH) read_step(h + 2, rs[0], rl[0]);
        sums(rs[1], rl[1]);
    }
}

// The sums for tile bits JB..11 (JB = 0 with RB = 3: contiguous tiles; JB = 4 with RB = 2: tiles with
// a window), of which bits >= j0 are wanted.  The tile of psi and of lambda goes from memory through
// registers into LDS (64 KiB); then every wavefront reads the whole tile in runs of its own RB bits
// (wavefront v: tile bits JB + RB v ...), so a lane carries accumulators for RB qubits only and the
// loads of the workgroup's next tile stay in flight meanwhile (the loop is rotated for that: load
// tile g, sums of tile g - 1, tile g into LDS).  Every wavefront sums d over the whole tile, so
// Im M11 = tsum - Im M00 holds per wavefront.  Output layout as k_trans_tile; the wavefronts that do not own
// a qubit write zeros for it.
template <int RB>
__global__ __launch_bounds__(256, 2) void k_trans_wave(const float2* psi0, const float2* lam0, int rstride,
                                                       int n, int c, int w, int j0, int per_group, int nblk,
                                                       double* partial) {
    __shared__ float2 ps[4096];
    __shared__ float2 lm[4096];                      // 64 KiB in all
    constexpr int JB = RB == 3 ? 0 : 4;
    const u64 r = blockIdx.y;
    const float2* psi = psi0 + ((rstride * r) << n);
    const float2* lam = lam0 + ((rstride * r) << n);
    const unsigned t = threadIdx.x, lane = t & 63u;
    const int wv = (int)(t >> 6);
    const unsigned cmask = (1u << c) - 1u;
    const int wc = w - c;
    float acc[RB][3];
    float tsum = 0.f;
#pragma unroll
    for (int a = 0; a < RB; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) acc[a][b] = 0.f;
    const unsigned tc = t ^ ((t >> 4) & 15u);        // swizzled lane part of the layout loaded from memory
    float2 s[16], l[16];                             // tau = i * 256 + t
    const u64 stride = c == 12 ? 256ull : (16ull << w);          // addressing as in k_trans_tile
    const unsigned kt8 = ((t & cmask) | ((t >> c) << w)) * 8u;
    const bool active = JB + RB * wv + RB - 1 >= j0;             // the wavefront owns a wanted bit
    for (int g = 0; g <= per_group; ++g) {
        if (g < per_group) {
            const u64 tb = (u64)blockIdx.x * per_group + g;      // tile of the row
            const u64 base = ((tb & ((1ull << wc) - 1ull)) << c) | ((tb >> wc) << (w + 12 - c));
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                s[i] = load_f2(uniform_ptr(psi + (base + (u64)i * stride)), kt8);
                l[i] = load_f2(uniform_ptr(lam + (base + (u64)i * stride)), kt8);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        if (g > 0 && active) {
            switch (wv) {
                case 0: trans_wave<RB, JB>(ps, lm, lane, acc, tsum); break;
                case 1: trans_wave<RB, JB + RB>(ps, lm, lane, acc, tsum); break;
                case 2: trans_wave<RB, JB + 2 * RB>(ps, lm, lane, acc, tsum); break;
                default: trans_wave<RB, JB + 3 * RB>(ps, lm, lane, acc, tsum); break;
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        if (g < per_group) {
            if (g) __syncthreads();                  // the previous tile has been read by everyone
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                ps[(unsigned)i * 256u + tc] = s[i];
                lm[(unsigned)i * 256u + tc] = l[i];
            }
            __syncthreads();
        }
    }
    const double t1 = wave_sum((double)tsum);
    double tot[RB][3];
#pragma unroll
    for (int a = 0; a < RB; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) tot[a][b] = wave_sum((double)acc[a][b]);
    if (lane != 0) return;
    for (int j = j0 > JB ? j0 : JB; j < 12; ++j) {
        const int q = j < c ? j : j - c + w;                 // the qubit behind tile bit j
        double* out = partial + ((r * n + q) * (u64)nblk + (u64)blockIdx.x * 4 + wv) * 8;
        if ((j - JB) / RB != wv) {
            for (int b = 0; b < 8; ++b) out[b] = 0.0;
            continue;
        }
#pragma unroll
        for (int a = 0; a < RB; ++a)
            if ((j - JB) % RB == a) trans_store(out, tot[a][0], tot[a][1], tot[a][2], t1);
    }
}

// Adds the nblk partials of every (row pair, qubit): one wavefront per job, lanes stride over the
// partials, fixed order.  out: [jobs][8].
__global__ __launch_bounds__(256) void k_trans_finish(const double* partial, int nblk, u64 jobs, double* out) {
    const u64 job = (u64)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (job >= jobs) return;
    const int lane = threadIdx.x & 63;
    double acc[8];
    for (int j = 0; j < 8; ++j) acc[j] = 0.0;
    const double* p = partial + job * (u64)nblk * 8;
    for (int b = lane; b < nblk; b += 64)
        for (int j = 0; j < 8; ++j) acc[j] += p[(u64)b * 8 + j];
    for (int j = 0; j < 8; ++j) {
        const double t = wave_sum(acc[j]);
        if (lane == 0) out[job * 8 + j] = t;
    }
}

// The RZ rotations that end the last layer are followed by an entangler, which permutes or signs basis
// states, and a diagonal observable: their derivative is exactly zero (what was summed is rounding, about
// 1e-9 a sample, and an optimiser that divides by a gradient's size makes steps of it).
__device__ __forceinline__ bool vanishing(const CircDev& c, int layer, int s) {
    bool all = layer + 1 == c.n_layers;
    for (int sl = s; sl < c.reupload + c.n_rot; ++sl) all = all && axis_of(c, sl) == QSV_RZ;
    return all;
}

// Derivative with respect to the angle of slot s on qubit q of a layer, from the qubit's transition sums M at the
// layer's start.  With U the qubit's unitary and V = R_last ... R_{s+1} its slots after s it is
// 2 Re sum_ab Bt[a][b] M[a][b], Bt = U^dagger V (-i/2 P_s) V^dagger U.  U^dagger (ud) is taken from the
// table that lambda came back through, as rounded as it is there: a derivative that vanishes because the
// rest of the circuit commutes with P_s then vanishes here too, up to the sums' rounding.
__device__ __forceinline__ double adj_derivative(const double (&M)[8], const M2& ud, const CircDev& c, int layer, int s, int q,
                                                 const float* params) {
    const int slots = c.reupload + c.n_rot;
    M2 w = ud;                                       // then times V
    for (int sl = slots - 1; sl > s; --sl)          // never the re-upload slot
        w = mul_m(w, rot_m(axis_of(c, sl), (double)params[((u64)layer * slots + sl) * c.n + q]));
    const int axis = axis_of(c, s);
    // G = -i/2 P for the axis of slot s
    M2 g;
    for (int k = 0; k < 4; ++k) { g.r[k] = 0.0; g.i[k] = 0.0; }
    if (axis == QSV_RX) { g.i[1] = -0.5; g.i[2] = -0.5; }
    else if (axis == QSV_RY) { g.r[1] = -0.5; g.r[2] = 0.5; }
    else { g.i[0] = -0.5; g.i[3] = 0.5; }
    M2 wd;   // its conjugate transpose
    wd.r[0] = w.r[0]; wd.i[0] = -w.i[0]; wd.r[1] = w.r[2]; wd.i[1] = -w.i[2];
    wd.r[2] = w.r[1]; wd.i[2] = -w.i[1]; wd.r[3] = w.r[3]; wd.i[3] = -w.i[3];
    const M2 bt = mul_m(w, mul_m(g, wd));
    double acc = 0.0;
    for (int k = 0; k < 4; ++k) acc += bt.r[k] * M[2 * k] - bt.i[k] * M[2 * k + 1];
    if (vanishing(c, layer, s)) acc *= 0.0;
    return 2.0 * acc;
}

// Gradients of the layers layer0 .. layer0 + n_layers - 1: thread = (layer, row pair, slot, qubit), sums in the order
// [layer][row pair][qubit].  Written as f+ = g, f- = -g so that the same finishing kernels as for the shift rule apply
// (they halve the difference and multiply re-upload weights by the feature).
__global__ __launch_bounds__(256) void k_adj_layers(const double* sums, CircDev c, int layer0, int n_layers,
                                                    const float* params, u64 sample0, u64 pairs_rows, u64 P,
                                                    const float* back, const int* exec_of, int plain, int seq0,
                                                    int seq_stride, double* f) {
    const u64 idx = (u64)blockIdx.x * 256 + threadIdx.x;
    const int slots = c.reupload + c.n_rot;
    const u64 per = (u64)slots * c.n;
    if (idx >= (u64)n_layers * pairs_rows * per) return;
    const u64 lr = idx / per, r = lr % pairs_rows;      // lr: row of the sums
    const int s = (int)((idx % per) / c.n), q = (int)(idx % c.n);
    const int layer = layer0 + (int)(lr / pairs_rows);
    const u64 sample = sample0 + r;
    double M[8];
    for (int j = 0; j < 8; ++j) M[j] = sums[(lr * c.n + q) * 8 + j];
    const u64 entry = (c.reupload ? sample * (u64)c.n_layers * c.n : 0) + (u64)layer * c.n + (exec_of ? exec_of[q] : q);
    const double g = adj_derivative(M, entry_m(back + entry * 8, plain || q + 1 == c.n, seq0, seq_stride), c, layer, s, q,
                                    params);
    const u64 p = ((u64)layer * slots + s) * c.n + q;
    double* fb = f + sample * (2 * P + 1);
    fb[2 * p] = g;
    fb[2 * p + 1] = -g;
}

// The same for all layers of the samples that k_sweep_small took: thread = (sample, parameter); sums as that kernel
// writes them.  back: the phaseless table of the inverse circuit in natural order.
__global__ __launch_bounds__(256) void k_adj_all(const double* sums, int waves, CircDev c, const float* params, u64 rows,
                                                 const float* back, double* f) {
    const u64 idx = (u64)blockIdx.x * 256 + threadIdx.x;
    const int slots = c.reupload + c.n_rot;
    const u64 P = (u64)c.n_layers * slots * c.n;
    if (idx >= rows * P) return;
    const u64 sample = idx / P, p = idx % P;
    const int q = (int)(p % c.n), s = (int)(p / c.n % slots), l = (int)(p / ((u64)c.n * slots));
    const double* rec = sums + (sample * c.n_layers + l) * (u64)waves * 32;
    double t = 0.0, m00 = 0.0, kre = 0.0, kim = 0.0;
    for (int w = 0; w < waves; ++w) {
        t += rec[w * 32];
        m00 += rec[w * 32 + 1 + 3 * q];
        kre += rec[w * 32 + 2 + 3 * q];
        kim += rec[w * 32 + 3 + 3 * q];
    }
    const double M[8] = {0.0, m00, kre, kim, 0.0, 0.0, 0.0, t - m00};
    const u64 entry = (c.reupload ? sample * (u64)c.n_layers * c.n : 0) + (u64)l * c.n + q;
    const double g = adj_derivative(M, entry_m(back + entry * 8, true, 0, 1), c, l, s, q, params);
    double* fb = f + sample * (2 * P + 1);
    fb[2 * p] = g;
    fb[2 * p + 1] = -g;
}

// The same from the records of k_pair_pass: `lanes` lanes per (unitary by position, row) add its records up in a
// fixed order, and lane s of them takes the derivative of slot s.  corr: the scale table of k_build_mats.
__global__ __launch_bounds__(256) void k_pair_finish(const float4* sums, int waves, int lanes, CircDev c, const float* params,
                                                     u64 rows, u64 sample0, u64 P, const int* order,
                                                     const int* entry_of, const float* back, int n_mats,
                                                     const double* corr, int seq0, int seq_stride, double* f) {
    const u64 job = ((u64)blockIdx.x * 256 + threadIdx.x) / (unsigned)lanes;
    const int lane = (int)(threadIdx.x & (unsigned)(lanes - 1));
    const int per = c.n_layers * c.n, slots = c.reupload + c.n_rot;
    const bool live = job < (u64)per * rows;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    const u64 pos = live ? job / rows : 0, r = live ? job % rows : 0;
    if (live) {
        const float4* rec = sums + job * (u64)waves;
        for (int i = lane; i < waves; i += lanes) {
            const float4 v = rec[i];
            acc[0] += (double)v.x; acc[1] += (double)v.y; acc[2] += (double)v.z; acc[3] += (double)v.w;
        }
    }
    for (int d = lanes >> 1; d > 0; d >>= 1)
        for (int j = 0; j < 4; ++j) acc[j] += __shfl_xor(acc[j], d, 64);
    if (!live || lane >= slots) return;
    const int lq = order[pos], layer = lq / c.n, q = lq % c.n, s = lane;
    const u64 sample = sample0 + r, table = c.reupload ? sample : 0;
    const double up = corr[(table * (u64)per + pos) * 2], up_before = corr[(table * (u64)per + pos) * 2 + 1];
    double g;
    if (slots >= 3) {
        const double x = acc[0] * up, z = acc[1] * up, y = acc[2] * up;
        const double M[8] = {0.0, 0.5 * z, -y, x, 0.0, 0.0, 0.0, -0.5 * z};
        const float* entry = back + (table * (u64)n_mats + (u64)entry_of[pos]) * 8;
        g = adj_derivative(M, entry_m(entry, false, seq0, seq_stride), c, layer, s, q, params);
    } else {
        g = s == 0 ? acc[0] * up : acc[2] * up_before;
        if (vanishing(c, layer, s)) g *= 0.0;
    }
    const u64 p = ((u64)layer * slots + s) * c.n + q;
    double* fb = f + sample * (2 * P + 1);
    fb[2 * p] = g;
    fb[2 * p + 1] = -g;
}

// ------------------------------------------------------------------------------------------
// Optimiser steps on the parameter vector, in double, stored as float.
__global__ __launch_bounds__(256) void k_sgd(float* p, const float* g, u64 count, double lr) {
    const u64 i = (u64)blockIdx.x * 256 + threadIdx.x;
    if (i < count) p[i] = (float)((double)p[i] - lr * (double)g[i]);
}

__global__ __launch_bounds__(256) void k_adam(float* p, const float* g, float* m, float* v, u64 count,
                                              double lr, double b1, double b2, double eps, double c1,
                                              double c2) {
    const u64 i = (u64)blockIdx.x * 256 + threadIdx.x;
    if (i >= count) return;
    const double gi = (double)g[i];
    const double mi = b1 * (double)m[i] + (1.0 - b1) * gi;
    const double vi = b2 * (double)v[i] + (1.0 - b2) * gi * gi;
    p[i] = (float)((double)p[i] - lr * (mi / c1) / (sqrt(vi / c2) + eps));
    m[i] = (float)mi;
    v[i] = (float)vi;
}

// ------------------------------------------------------------------------------------------
// A whole small workload in one launch (at most 10 qubits): amplitude encoding, the circuit (and,
// as decoder, its exact inverse), the final state and one measurement.  A thread keeps 2^R
// amplitudes in registers (index bits 0..R-1), the index bits above are bits of the thread number:
// up to six inside the wavefront, the rest across the wavefronts of the workgroup; with fewer than
// six the spare lane bits number the samples that share the wavefront.  A gate on a register bit
// pairs registers; on a lane bit it exchanges with the partner lane (DPP, the LDS crossbar);
// on a bit across wavefronts it exchanges through LDS.  Nothing goes to device memory between the
// gates.  R = 2, 3 or 4 is chosen so that the batch gives the chip enough wavefronts (a lone
// wavefront on a SIMD issues one vector instruction in about eight cycles, four of them one every
// three).  The matrices are built once per workgroup, one per thread at a time, and kept in LDS.
template <int R> struct Amps { float re[1 << R], im[1 << R]; };  // every index is a compile-time constant after unrolling

__device__ __forceinline__ float lane_xchg(int addr, float v) {
    return __int_as_float(__builtin_amdgcn_ds_bpermute(addr, __float_as_int(v)));
}

// The value that the lane whose number differs in bit B holds.  Bits 0..3: DPP moves (inside a row
// of 16 lanes; XOR 4 = reversal of 8 then of 4, XOR 8 = reversal of 16 then of 8); bit 4: the
// swizzle of the LDS crossbar; bit 5: ds_bpermute (addr = 4 * partner lane).
template <int B>
__device__ __forceinline__ float lane_flip(float v, int addr) {
    const int x = __float_as_int(v);
    if constexpr (B == 0) return __int_as_float(__builtin_amdgcn_mov_dpp(x, 0xB1, 0xf, 0xf, true));   // quad_perm [1,0,3,2]
    else if constexpr (B == 1) return __int_as_float(__builtin_amdgcn_mov_dpp(x, 0x4E, 0xf, 0xf, true));   // [2,3,0,1]
    else if constexpr (B == 2)
        return __int_as_float(__builtin_amdgcn_mov_dpp(__builtin_amdgcn_mov_dpp(x, 0x141, 0xf, 0xf, true), 0x1B, 0xf, 0xf, true));
    else if constexpr (B == 3)
        return __int_as_float(__builtin_amdgcn_mov_dpp(__builtin_amdgcn_mov_dpp(x, 0x140, 0xf, 0xf, true), 0x141, 0xf, 0xf, true));
    else if constexpr (B == 4) return __int_as_float(__builtin_amdgcn_ds_swizzle(x, 0x401F));           // xor 16 within 32 lanes
    else return lane_xchg(addr, v);
}

// Exchange between the wavefronts of a workgroup: every thread puts its registers into the current
// one of two buffers [2 * 2^R][threads], and after the barrier reads another thread's.  The
// buffers alternate, so one barrier per exchange is enough (whoever writes a buffer again has
// passed the barrier of the exchange in between, which every reader of the old contents reaches
// only after reading).
struct Xchg { float* buf; int threads, cur; };

template <int R>
__device__ __forceinline__ void xchg_through_lds(const Amps<R>& a, float* pr, float* pi, Xchg& x, int tid, int src) {
    float* b = x.buf + (size_t)x.cur * (2 << R) * x.threads;
#pragma unroll
    for (int k = 0; k < (1 << R); ++k) {
        b[(2 * k) * x.threads + tid] = a.re[k];
        b[(2 * k + 1) * x.threads + tid] = a.im[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < (1 << R); ++k) {
        pr[k] = b[(2 * k) * x.threads + src];
        pi[k] = b[(2 * k + 1) * x.threads + src];
    }
    x.cur ^= 1;
}

// m = (m00r, m00i, m01r, m01i, m10r, m10i, m11r, m11i)
template <int R, int J>
__device__ __forceinline__ void small_u_reg(Amps<R>& a, const float* m) {
#pragma unroll
    for (int k = 0; k < (1 << R); ++k) {
        if (k & (1 << J)) continue;
        const int k1 = k | (1 << J);
        const float ar = a.re[k], ai = a.im[k], br = a.re[k1], bi = a.im[k1];
        a.re[k] = m[0] * ar - m[1] * ai + m[2] * br - m[3] * bi;
        a.im[k] = m[0] * ai + m[1] * ar + m[2] * bi + m[3] * br;
        a.re[k1] = m[4] * ar - m[5] * ai + m[6] * br - m[7] * bi;
        a.im[k1] = m[4] * ai + m[5] * ar + m[6] * bi + m[7] * br;
    }
}

// The qubit is bit B of the thread number: this thread holds the amplitudes with the bit equal to
// its own, the partner thread the ones with the other value.
template <int R, int B>
__device__ __forceinline__ void small_u_thr(Amps<R>& a, const float* m, int tid, Xchg& x) {
    constexpr int NR = 1 << R;
    const bool bit = (tid >> B) & 1;
    const float sr = bit ? m[6] : m[0], si = bit ? m[7] : m[1];   // row `bit`, own column
    const float qr = bit ? m[4] : m[2], qi = bit ? m[5] : m[3];   // row `bit`, the partner's column
    float pr[NR], pi[NR];                    // all exchanges first: their latencies overlap
    if constexpr (B < 6) {
        const int addr = ((tid & 63) ^ (1 << B)) << 2;
#pragma unroll
        for (int k = 0; k < NR; ++k) { pr[k] = lane_flip<B>(a.re[k], addr); pi[k] = lane_flip<B>(a.im[k], addr); }
    } else {
        xchg_through_lds<R>(a, pr, pi, x, tid, tid ^ (1 << B));
    }
#pragma unroll
    for (int k = 0; k < NR; ++k) {
        const float ar = a.re[k], ai = a.im[k];
        a.re[k] = sr * ar - si * ai + qr * pr[k] - qi * pi[k];
        a.im[k] = sr * ai + si * ar + qr * pi[k] + qi * pr[k];
    }
}

template <int R, int C, int T>
__device__ __forceinline__ void small_cx_rr(Amps<R>& a) {
    if constexpr (C < R && T < R) {
#pragma unroll
        for (int k = 0; k < (1 << R); ++k) {
            if (!(k & (1 << C)) || (k & (1 << T))) continue;
            const int k1 = k | (1 << T);
            const float r = a.re[k], i = a.im[k];
            a.re[k] = a.re[k1]; a.im[k] = a.im[k1];
            a.re[k1] = r; a.im[k1] = i;
        }
    }
}

template <int R>
__device__ __forceinline__ void small_cx_to_reg0(Amps<R>& a, bool ctrl) {  // control on a thread bit, target register bit 0
#pragma unroll
    for (int k = 0; k < (1 << R); k += 2) {
        const float r0 = a.re[k], i0 = a.im[k], r1 = a.re[k + 1], i1 = a.im[k + 1];
        a.re[k] = ctrl ? r1 : r0; a.im[k] = ctrl ? i1 : i0;
        a.re[k + 1] = ctrl ? r0 : r1; a.im[k + 1] = ctrl ? i0 : i1;
    }
}

// The CNOT ring on n qubits, control q, target q + 1 (the last one's target is qubit 0), in order,
// or with reverse = true in the opposite order (the ring's inverse).  The CNOTs between register
// bits rename registers; the one from the top register bit to thread bit 0 exchanges half of the
// registers with the neighbouring lane; the CNOTs between thread bits are together one
// permutation of the threads (src_f / src_r: the thread each one reads from), done by
// ds_bpermute inside a wavefront and through LDS across wavefronts; the closing one swaps register
// pairs in the threads whose top index bit is set.
template <int R, int N>
__device__ __forceinline__ void small_ring(Amps<R>& a, int tid, bool reverse, int src_f, int src_r, Xchg& x) {
    constexpr int NR = 1 << R, n = N, tb = N > R ? N - R : 0;
    auto wrap = [&]() {
        if (n > R) small_cx_to_reg0<R>(a, (tid >> (tb - 1)) & 1);
        else if (n == 2) small_cx_rr<R, 1, 0>(a);
        else if (n == 3) small_cx_rr<R, 2, 0>(a);
        else if (n == 4) small_cx_rr<R, 3, 0>(a);
    };
    auto bridge = [&]() {                          // control register bit R - 1, target thread bit 0
        if (n > R) {
#pragma unroll
            for (int k = NR / 2; k < NR; ++k) { a.re[k] = lane_flip<0>(a.re[k], 0); a.im[k] = lane_flip<0>(a.im[k], 0); }
        }
    };
    auto chain = [&](int src) {
        if (tb < 2) return;
        float pr[NR], pi[NR];
        if (tb <= 6) {
            const int addr = src << 2;             // src differs from tid in lane bits only
#pragma unroll
            for (int k = 0; k < NR; ++k) { pr[k] = lane_xchg(addr, a.re[k]); pi[k] = lane_xchg(addr, a.im[k]); }
        } else {
            xchg_through_lds<R>(a, pr, pi, x, tid, src);
        }
#pragma unroll
        for (int k = 0; k < NR; ++k) { a.re[k] = pr[k]; a.im[k] = pi[k]; }
    };
    if (!reverse) {
        if (n >= 2) small_cx_rr<R, 0, 1>(a);
        if (n >= 3) small_cx_rr<R, 1, 2>(a);
        if (n >= 4) small_cx_rr<R, 2, 3>(a);
        bridge();
        chain(src_f);
        wrap();
    } else {
        wrap();
        chain(src_r);
        bridge();
        if (n >= 4) small_cx_rr<R, 2, 3>(a);
        if (n >= 3) small_cx_rr<R, 1, 2>(a);
        if (n >= 2) small_cx_rr<R, 0, 1>(a);
    }
}

// CZ on qubits q and q + 1 for q = 0..n-2 (the gates commute, so the order does not matter): the
// sign of an amplitude changes once for every pair of neighbouring set bits of its index.
template <int R, int N>
__device__ __forceinline__ void small_cz_ladder(Amps<R>& a, int ti) {
    constexpr int mask = (1 << (N - 1)) - 1;           // pairs (q, q + 1) for q = 0..n-2
#pragma unroll
    for (int k = 0; k < (1 << R); ++k) {
        const int idx = (ti << R) | k;
        const bool f = __builtin_popcount(idx & (idx >> 1) & mask) & 1;
        a.re[k] = f ? -a.re[k] : a.re[k];
        a.im[k] = f ? -a.im[k] : a.im[k];
    }
}

struct SmallArgs {
    const float* x;        // [batch][dim]
    int64_t dim, batch;
    CircDev c;
    int entangler;         // qsv_ent
    const float* params;
    const float* feats;
    int pass_first, pass_last;  // 0 = the circuit, 1 = its inverse: (0,0) circuit, (0,1) circuit then inverse, (1,1) inverse
    int from_state;        // 1: start from the amplitudes in `state` instead of encoding x
    int kind;              // QSV_M_PROBS, QSV_M_EXPZ_ALL, or 0: no measurement
    float2* state;         // [batch][2^n], receives the final state
    float* out;            // probabilities [batch][2^n] or expectations [batch][n]
    float* norm_out;       // [batch] or NULL
    int mat_floats;        // LDS floats set aside for the workgroup's matrices (a multiple of 8)
    int rows;              // samples per workgroup: at most what its lanes have room for
};

// Fused matrices of the samples first..first+rows_m-1 into LDS.  The angles and features come to LDS first, all
// loads at once (read where they were needed, every matrix waited for them).  Neighbouring threads take the rotations of one matrix, a sine and cosine in double each, and
// multiply up what they found.
template <int N>
__device__ __forceinline__ void small_build(const CircDev& c, const float* params, const float* feats, int64_t first,
                                            int64_t batch, int rows_m, int tid, float* mats, float* stage) {
    const int slots = c.reupload + c.n_rot, L = c.n_layers, n_par = small_staged_angles(c), n_feat = small_staged_features(c, rows_m);
    const int64_t feat0 = first * N, feat_end = batch * N;
    for (int i = tid; i < n_par; i += (int)blockDim.x) stage[i] = params[i];
    for (int i = tid; i < n_feat; i += (int)blockDim.x) stage[n_par + i] = feat0 + i < feat_end ? feats[feat0 + i] : 0.f;
    __syncthreads();
    const int lg = slots > 2 ? 2 : slots - 1, count = (rows_m * L * N) << lg;
    const int end = (count + (int)blockDim.x - 1) / (int)blockDim.x * (int)blockDim.x;
    const float inv_l = 1.f / (float)L;
    for (int i = tid; i < end; i += (int)blockDim.x) {       // every lane takes part in the exchanges
        const int m = (i < count ? i : 0) >> lg, sl = i & ((1 << lg) - 1);
        const int rl = m / N, q = m % N;
        const int r = (int)(((float)rl + 0.5f) * inv_l), l = rl - r * L;      // rl < 2^9: exact
        double sn = 0.0, co = 1.0;
        if (sl < slots) {
            double t = (double)stage[(l * slots + sl) * N + q];
            if (c.reupload && sl == 0) t *= (double)stage[n_par + r * N + q];
            sincos(0.5 * t, &sn, &co);
        }
        double ar = 1.0, ai = 0.0, br = 0.0, bi = 0.0;
        const int lane0 = (tid & 63) & ~((1 << lg) - 1);
        for (int k = 0; k < slots; ++k) {
            const double ks = __shfl(sn, lane0 + k, 64), kc = __shfl(co, lane0 + k, 64);
            rotate_column(c.reupload && k == 0 ? (int)QSV_RX : c.rot[k - c.reupload], ks, kc, ar, ai, br, bi);
        }
        if (sl == 0 && i < count) {
            float4* o = reinterpret_cast<float4*>(mats + (size_t)m * 8);
            o[0] = make_float4((float)ar, (float)ai, (float)-br, (float)bi);
            o[1] = make_float4((float)br, (float)bi, (float)ar, (float)-ai);
        }
    }
}

// dynamic LDS: [64] doubles for sums across wavefronts, the workgroup's matrices, then the exchange buffers (which
// hold the angles and features while the matrices are built)
// The number of qubits is a template argument: with it at run time every gate stood behind a branch, which kept
// the matrices' loads and the exchanges of neighbouring gates from overlapping.
template <int R, int N>
__global__ __launch_bounds__(256) void k_forward_small(SmallArgs a) {
    constexpr int NR = 1 << R;
    extern __shared__ __align__(16) unsigned char small_lds[];
    double* red = reinterpret_cast<double*>(small_lds);
    float* mats = reinterpret_cast<float*>(small_lds + 64 * sizeof(double));
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    constexpr int n = N;
    const int L = a.c.n_layers;
    constexpr int tb = n > R ? n - R : 0;        // index bits held by the thread number
    constexpr int lb = tb < 6 ? tb : 6;          // of which inside the wavefront
    constexpr int n_waves = tb > 6 ? 1 << (tb - 6) : 1;
    constexpr int rows_g = 64 >> lb;             // samples per workgroup (1 when tb >= 6)
    const int r_in = tb < 6 ? lane >> tb : 0;
    const int ti = tid & ((1 << tb) - 1);
    Xchg xc;
    xc.buf = mats + a.mat_floats;
    xc.threads = (int)blockDim.x;
    xc.cur = 0;
    const int64_t first = (int64_t)blockIdx.x * a.rows;
    const int64_t sample = first + r_in;
    const bool live = r_in < a.rows && sample < a.batch;
    const int per = L * n;
    const bool has_u = small_has_unitaries(a.c);
    // what the circuit starts from is on its way while the matrices are built
    Amps<R> A;
    const bool inside = live && ((int64_t)ti << R) < ((int64_t)1 << n);
    if (a.from_state) {
        const float2* srow = a.state + ((live ? sample : 0) << n) + ((int64_t)ti << R);
#pragma unroll
        for (int k = 0; k < NR; ++k) {
            const int64_t idx = ((int64_t)ti << R) | k;
            const float2 v = (inside && idx < ((int64_t)1 << n)) ? srow[k] : make_float2(0.f, 0.f);
            A.re[k] = v.x; A.im[k] = v.y;
        }
    } else {
        const float* xb = a.x + (live ? sample : 0) * a.dim;
#pragma unroll
        for (int k = 0; k < NR; ++k) {
            const int64_t idx = ((int64_t)ti << R) | k;
            A.re[k] = (live && idx < a.dim) ? xb[idx] : 0.f;
            A.im[k] = 0.f;
        }
    }
    if (has_u)
        small_build<N>(a.c, a.params, a.feats, first, a.batch, a.c.reupload ? a.rows : 1, tid, mats, xc.buf);
    // amplitude encoding: x / ||x||, the norm in double
    if (!a.from_state) {
        double ss = 0.0;
#pragma unroll
        for (int k = 0; k < NR; ++k) ss += (double)A.re[k] * (double)A.re[k];
#pragma unroll
        for (int b = 0; b < 6; ++b)
            if (b < lb) ss += __shfl_xor(ss, 1 << b, 64);
        if (n_waves > 1) {
            if (lane == 0) red[wave] = ss;
            __syncthreads();
            ss = 0.0;
            for (int w = 0; w < n_waves; ++w) ss += red[w];
        }
        const double nrm = sqrt(ss);
        const double inv = nrm > 0.0 ? 1.0 / nrm : 0.0;
#pragma unroll
        for (int k = 0; k < NR; ++k) A.re[k] = (float)((double)A.re[k] * inv);
        if (a.norm_out && live && ti == 0) a.norm_out[sample] = (float)nrm;
    }
    __syncthreads();                             // the matrices are in LDS; red[] may be written again
    const float* mrow = mats + (size_t)(a.c.reupload && live ? r_in * per : 0) * 8;
    // Thread permutations of the ring's CNOTs between thread bits (qubits R..n-1): an amplitude in
    // thread j moves to C(j), so afterwards thread j holds what thread C_first(...C_last(j)) held.
    int src_f = tid, src_r = tid;
    for (int b = tb - 2; b >= 0; --b) src_f ^= ((src_f >> b) & 1) << (b + 1);
    for (int b = 0; b + 1 < tb; ++b) src_r ^= ((src_r >> b) & 1) << (b + 1);
    // the gates: per layer the unitaries then the entangler; in the decoder layers last to first,
    // the entangler's gates in reverse order first, then the conjugate-transposed unitaries
    for (int pass = a.pass_first; pass <= a.pass_last; ++pass) {
        for (int ll = 0; ll < L; ++ll) {
            const int l = pass ? L - 1 - ll : ll;
            for (int stage = 0; stage < 2; ++stage) {
                if ((stage == 0) == (pass == 1)) {
                    if (a.entangler == QSV_ENT_CNOT_RING) small_ring<R, N>(A, tid, pass != 0, src_f, src_r, xc);
                    else if (a.entangler == QSV_ENT_CZ_LADDER) small_cz_ladder<R, N>(A, ti);
                } else if (has_u) {
                    const float* ml = mrow + (size_t)l * n * 8;
                    auto load_m = [&](int q, float* m) {
                        const float4 lo = *reinterpret_cast<const float4*>(ml + q * 8);
                        const float4 hi = *reinterpret_cast<const float4*>(ml + q * 8 + 4);
                        if (!pass) {
                            m[0] = lo.x; m[1] = lo.y; m[2] = lo.z; m[3] = lo.w;
                            m[4] = hi.x; m[5] = hi.y; m[6] = hi.z; m[7] = hi.w;
                        } else {                 // conjugate transpose
                            m[0] = lo.x; m[1] = -lo.y; m[2] = hi.x; m[3] = -hi.y;
                            m[4] = lo.z; m[5] = -lo.w; m[6] = hi.z; m[7] = -hi.w;
                        }
                    };
                    float m[8];
#define QSV_SMALL_U(Q)                                                      \
    if constexpr (n > Q) {                                                  \
        load_m(Q, m);                                                       \
        if constexpr (Q < R) small_u_reg<R, Q>(A, m);                       \
        else if constexpr (Q - R < 8) small_u_thr<R, Q - R>(A, m, tid, xc); \
    }
                    QSV_SMALL_U(0) QSV_SMALL_U(1) QSV_SMALL_U(2) QSV_SMALL_U(3) QSV_SMALL_U(4)
                    QSV_SMALL_U(5) QSV_SMALL_U(6) QSV_SMALL_U(7) QSV_SMALL_U(8) QSV_SMALL_U(9)
#undef QSV_SMALL_U
                }
            }
        }
    }
    // final state and the measurement
    const int dimn = 1 << n;
    if (live) {
        float2* srow = a.state + (sample << n) + ((int64_t)ti << R);
        if (n >= R) {
#pragma unroll
            for (int k = 0; k < NR; k += 2)
                *reinterpret_cast<float4*>(srow + k) = make_float4(A.re[k], A.im[k], A.re[k + 1], A.im[k + 1]);
        } else {
#pragma unroll
            for (int k = 0; k < NR; ++k)
                if (k < dimn) srow[k] = make_float2(A.re[k], A.im[k]);
        }
    }
    if (a.kind == 0) return;
    float p[NR];
#pragma unroll
    for (int k = 0; k < NR; ++k) p[k] = prob32(make_float2(A.re[k], A.im[k]));
    if (a.kind == QSV_M_PROBS) {
        if (live) {
            float* prow = a.out + (sample << n) + ((int64_t)ti << R);
            if (n >= R) {
#pragma unroll
                for (int k = 0; k < NR; k += 4)
                    *reinterpret_cast<float4*>(prow + k) = make_float4(p[k], p[k + 1], p[k + 2], p[k + 3]);
            } else {
#pragma unroll
                for (int k = 0; k < NR; ++k)
                    if (k < dimn) prow[k] = p[k];
            }
        }
        return;
    }
    // <Z_q> for every qubit: signed sums in double, combined over the threads of the sample
    double T = 0.0, zr[R], zl[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int j = 0; j < R; ++j) zr[j] = 0.0;
#pragma unroll
    for (int k = 0; k < NR; ++k) {
        const double pk = (double)p[k];
        T += pk;
#pragma unroll
        for (int j = 0; j < R; ++j) zr[j] += ((k >> j) & 1) ? -pk : pk;
    }
#pragma unroll
    for (int b = 0; b < 6; ++b) {
        if (b < lb) {
            const double Tp = __shfl_xor(T, 1 << b, 64);
#pragma unroll
            for (int j = 0; j < R; ++j) zr[j] += __shfl_xor(zr[j], 1 << b, 64);
#pragma unroll
            for (int j = 0; j < 6; ++j)
                if (j < b) zl[j] += __shfl_xor(zl[j], 1 << b, 64);
            zl[b] = ((lane >> b) & 1) ? Tp - T : T - Tp;
            T += Tp;
        }
    }
    if (n_waves == 1) {
        if (live && ti == 0) {
            float* orow = a.out + sample * n;
#pragma unroll
            for (int q = 0; q < R; ++q)            // qubits behind register bits
                if (q < n) orow[q] = (float)zr[q];
#pragma unroll
            for (int b = 0; b < 6; ++b)            // qubits behind lane bits
                if (R + b < n) orow[R + b] = (float)zl[b];
        }
        return;
    }
    // several wavefronts hold the sample: totals per wavefront through LDS, thread q adds up qubit q
    // (qubits beyond the lane bits take the wavefront totals signed by the wavefront's number)
    if (lane == 0) {
        double* o = red + wave * 16;
        o[0] = T;
#pragma unroll
        for (int j = 0; j < R; ++j) o[1 + j] = zr[j];
#pragma unroll
        for (int j = 0; j < 6; ++j) o[1 + R + j] = zl[j];
    }
    __syncthreads();
    if (tid < n && live) {
        const int q = tid;
        double acc = 0.0;
        for (int w = 0; w < n_waves; ++w) {
            const double* o = red + w * 16;
            if (q < R + 6) acc += o[1 + q];
            else acc += ((w >> (q - R - 6)) & 1) ? -o[0] : o[0];
        }
        a.out[sample * n + q] = (float)acc;
    }
}

// Reverse-mode sweep of small states (at most 10 qubits) in one launch: encoding, circuit, loss, lambda = O psi, then
// lambda back through the layers, and at every layer's start the transition sums of all qubits, which are
// what leaves the chip.  The layout is that of k_forward_small.  KEEP: psi is written at every layer's start on the way
// forward and read on the way back (each thread its own amplitudes, while lambda's gates run); without room for that it
// is taken back beside lambda, with a third more gates and the roundings of those (gradients 1.3 to 1.8 times as far from
// 64 bits).  Bound by vector issue.  Through the fused passes the same takes six launches per layer, each of which reads
// and writes the states.  Passes / taken back / kept: 10 qubits x 1024 re-uploading 6 layers 391 / 102 / 85 us, 8 x 64 319 / 39 /
// 35 us, 4 x 1 176 / 23.4 / 21.5 us.
struct SweepArgs {
    const float* x;          // [batch][dim]
    int64_t dim, batch;
    CircDev c;
    int entangler;
    const float* back;       // phaseless table of the inverse circuit in natural order
    int rows;                // samples per workgroup
    int mat_floats;          // LDS floats of the workgroup's matrices
    int kind, obs_qubit;     // as launch_adj_init
    u64 mask;
    const float* targets;    // kind 2: [batch][n]
    double* f;               // [batch][2P + 1]: the loss goes to entry 2P
    float2* kept;            // KEEP: [L][batch][2^n], psi at the start of every layer
    double* sums;            // [batch][L][wavefronts of a sample][32]: sum of d, then 3 per qubit (see k_adj_all)
};

// Sums 32 values over the lanes of a sample (2^LB of them, LB <= 6): in step b lanes that differ in bit b split the
// values between them, so that a lane ends with 32 >> LB of them (at least one), number first..first + that - 1.
template <int H>
__device__ __forceinline__ void reduce_step(double (&v)[32], int mask) {   // H: half of the values still held
    const bool up = threadIdx.x & mask;
#pragma unroll
    for (int i = 0; i < H; ++i) {
        const double lo = v[i], hi = v[i + H];
        const double keep = up ? hi : lo, give = up ? lo : hi;
        v[i] = keep + __shfl_xor(give, mask, 64);
    }
}

template <int LB>
__device__ __forceinline__ int reduce32(double (&v)[32]) {
    const int lane = threadIdx.x & 63;
    if constexpr (LB > 0) reduce_step<16>(v, 1);
    if constexpr (LB > 1) reduce_step<8>(v, 2);
    if constexpr (LB > 2) reduce_step<4>(v, 4);
    if constexpr (LB > 3) reduce_step<2>(v, 8);
    if constexpr (LB > 4) reduce_step<1>(v, 16);
    if constexpr (LB > 5) v[0] += __shfl_xor(v[0], 32, 64);
    int first = 0;
#pragma unroll
    for (int b = 0; b < (LB < 5 ? LB : 5); ++b) first += (lane >> b) & 1 ? 16 >> b : 0;
    return first;
}

// the values that another thread of the sample holds for thread bit B
template <int R, int B>
__device__ __forceinline__ void small_partner(const Amps<R>& a, float* pr, float* pi, int tid, Xchg& x) {
    if constexpr (B < 6) {
        const int addr = ((tid & 63) ^ (1 << B)) << 2;
#pragma unroll
        for (int k = 0; k < (1 << R); ++k) { pr[k] = lane_flip<B>(a.re[k], addr); pi[k] = lane_flip<B>(a.im[k], addr); }
    } else {
        xchg_through_lds<R>(a, pr, pi, x, tid, tid ^ (1 << B));
    }
}

// Im M00, Re K, Im K of qubit Q (see trans_acc) from this thread's amplitudes; d = Im conj(lambda) psi, dsum its sum
template <int R, int Q>
__device__ __forceinline__ void small_trans(const Amps<R>& s, const Amps<R>& l, const float (&d)[1 << R], float dsum, int tid,
                                            Xchg& x, float (&acc)[3]) {
    acc[0] = acc[1] = acc[2] = 0.f;
    if constexpr (Q < R) {
#pragma unroll
        for (int k = 0; k < (1 << R); ++k) {
            if (k & (1 << Q)) continue;
            const int k1 = k | (1 << Q);
            acc[0] += d[k];
            acc[1] += (l.re[k] * s.re[k1] + l.im[k] * s.im[k1]) - (l.re[k1] * s.re[k] + l.im[k1] * s.im[k]);
            acc[2] += (l.re[k] * s.im[k1] - l.im[k] * s.re[k1]) + (l.re[k1] * s.im[k] - l.im[k1] * s.re[k]);
        }
    } else {
        float pr[1 << R], pi[1 << R];
        small_partner<R, Q - R>(s, pr, pi, tid, x);
        const bool bit = (tid >> (Q - R)) & 1;
        float re = 0.f;
#pragma unroll
        for (int k = 0; k < (1 << R); ++k) {
            re += l.re[k] * pr[k] + l.im[k] * pi[k];
            acc[2] += l.re[k] * pi[k] - l.im[k] * pr[k];
        }
        acc[0] = bit ? 0.f : dsum;
        acc[1] = bit ? -re : re;
    }
}

template <int R, int N, bool KEEP>
__global__ __launch_bounds__(256) void k_sweep_small(SweepArgs a) {
    constexpr int NR = 1 << R, n = N, NV = N < R ? 1 << N : NR;     // NV of a thread's amplitudes exist
    constexpr int tb = n > R ? n - R : 0, lb = tb < 6 ? tb : 6, n_waves = tb > 6 ? 1 << (tb - 6) : 1;
    extern __shared__ __align__(16) unsigned char small_lds[];
    double* red = reinterpret_cast<double*>(small_lds);
    float* mats = reinterpret_cast<float*>(small_lds + 64 * sizeof(double));
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int L = a.c.n_layers, per = L * n;
    const int r_in = tb < 6 ? lane >> tb : 0;
    const int ti = tid & ((1 << tb) - 1);
    Xchg xc;
    xc.buf = mats + a.mat_floats;
    xc.threads = (int)blockDim.x;
    xc.cur = 0;
    const int64_t first = (int64_t)blockIdx.x * a.rows;
    const int64_t sample = first + r_in;
    const bool live = r_in < a.rows && sample < a.batch;
    const u64 P = (u64)per * (a.c.reupload + a.c.n_rot);
    Amps<R> S, La;
    const float* xb = a.x + (live ? sample : 0) * a.dim;
#pragma unroll
    for (int k = 0; k < NR; ++k) {
        const int64_t idx = ((int64_t)ti << R) | k;
        S.re[k] = (live && idx < a.dim) ? xb[idx] : 0.f;
        S.im[k] = 0.f;
    }
    {
        const int64_t rows_m = a.c.reupload ? (a.batch - first < a.rows ? a.batch - first : a.rows) : 1;
        const float4* src = reinterpret_cast<const float4*>(a.back + (a.c.reupload ? first * per * 8 : 0));
        float4* dst = reinterpret_cast<float4*>(mats);
        for (int i = tid; i < (int)rows_m * per * 2; i += (int)blockDim.x) dst[i] = src[i];
    }
    auto sample_sum = [&](double v) -> double {      // over the threads of the sample
#pragma unroll
        for (int b = 0; b < 6; ++b)
            if (b < lb) v += __shfl_xor(v, 1 << b, 64);
        if constexpr (n_waves > 1) {
            __syncthreads();
            if (lane == 0) red[wave] = v;
            __syncthreads();
            v = 0.0;
            for (int w = 0; w < n_waves; ++w) v += red[w];
        }
        return v;
    };
    {
        double ss = 0.0;
#pragma unroll
        for (int k = 0; k < NR; ++k) ss += (double)S.re[k] * (double)S.re[k];
        const double nrm = sqrt(sample_sum(ss)), inv = nrm > 0.0 ? 1.0 / nrm : 0.0;
#pragma unroll
        for (int k = 0; k < NR; ++k) S.re[k] = (float)((double)S.re[k] * inv);
    }
    __syncthreads();                                 // the matrices are in LDS
    const float* mrow = mats + (size_t)(a.c.reupload && live ? r_in * per : 0) * 8;
    int src_f = tid, src_r = tid;
    for (int b = tb - 2; b >= 0; --b) src_f ^= ((src_f >> b) & 1) << (b + 1);
    for (int b = 0; b + 1 < tb; ++b) src_r ^= ((src_r >> b) & 1) << (b + 1);
    auto entangle = [&](Amps<R>& A, bool reverse) {
        if (a.entangler == QSV_ENT_CNOT_RING) small_ring<R, N>(A, tid, reverse, src_f, src_r, xc);
        else if (a.entangler == QSV_ENT_CZ_LADDER) small_cz_ladder<R, N>(A, ti);
    };
#define QSV_ALL_Q(X) X(0) X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9)
    auto kept = [&](int l) -> float4* {
        return reinterpret_cast<float4*>(a.kept + (((int64_t)l * a.batch + (live ? sample : 0)) << n) + ti * NV);
    };
    for (int l = 0; l < L; ++l) {
        if constexpr (KEEP) {
            if (live) {
#pragma unroll
                for (int k = 0; k < NV; k += 2) kept(l)[k / 2] = make_float4(S.re[k], S.im[k], S.re[k + 1], S.im[k + 1]);
            }
        }
        const float* ml = mrow + (size_t)l * n * 8;
        float m[8];
#define QSV_FWD(Q)                                                                          \
    if constexpr (n > Q) {                                                                  \
        const float4 lo = *reinterpret_cast<const float4*>(ml + Q * 8);                     \
        const float4 hi = *reinterpret_cast<const float4*>(ml + Q * 8 + 4);                 \
        m[0] = lo.x; m[1] = -lo.y; m[2] = hi.x; m[3] = -hi.y;                               \
        m[4] = lo.z; m[5] = -lo.w; m[6] = hi.z; m[7] = -hi.w;                               \
        if constexpr (Q < R) small_u_reg<R, Q>(S, m);                                       \
        else if constexpr (Q - R < 8) small_u_thr<R, Q - R>(S, m, tid, xc);                 \
    }
        QSV_ALL_Q(QSV_FWD)
#undef QSV_FWD
        entangle(S, false);
    }
    // the loss, and lambda = (diagonal weight) psi
    double loss = 0.0, coef[N];
    if (a.kind == 2) {
#pragma unroll
        for (int q = 0; q < N; ++q) {
            double z = 0.0;
#pragma unroll
            for (int k = 0; k < NR; ++k) {
                const double p = (double)prob32(make_float2(S.re[k], S.im[k]));
                z += ((((ti << R) | k) >> q) & 1) ? -p : p;
            }
            const double off = sample_sum(z) - (double)a.targets[(live ? sample : 0) * n + q];
            loss += off * off;
            coef[q] = 2.0 * off / n;
        }
        loss /= n;
    } else {
        double v = 0.0;
#pragma unroll
        for (int k = 0; k < NR; ++k) {
            const unsigned idx = ((unsigned)ti << R) | k;
            const double p = (double)prob32(make_float2(S.re[k], S.im[k]));
            if (a.kind == 0) v += ((idx >> a.obs_qubit) & 1u) ? -p : p;
            else v += (idx & (unsigned)a.mask) ? 0.0 : p;
        }
        v = sample_sum(v);
        loss = a.kind == 0 ? v : 1.0 - v;
    }
    if (live && ti == 0) a.f[sample * (2 * P + 1) + 2 * P] = loss;
#pragma unroll
    for (int k = 0; k < NR; ++k) {
        const unsigned idx = ((unsigned)ti << R) | k;
        float w;
        if (a.kind == 0) w = ((idx >> a.obs_qubit) & 1u) ? -1.f : 1.f;
        else if (a.kind == 1) w = (idx & (unsigned)a.mask) ? 0.f : -1.f;
        else {
            double wd = 0.0;
#pragma unroll
            for (int q = 0; q < N; ++q) wd += ((idx >> q) & 1u) ? -coef[q] : coef[q];
            w = (float)wd;
        }
        La.re[k] = w * S.re[k];
        La.im[k] = w * S.im[k];
    }
    for (int l = L - 1; l >= 0; --l) {
        if constexpr (KEEP) {
#pragma unroll
            for (int k = 0; k < NV; k += 2) {
                const float4 v = kept(l)[k / 2];
                S.re[k] = v.x; S.im[k] = v.y; S.re[k + 1] = v.z; S.im[k + 1] = v.w;
            }
        } else {
            entangle(S, true);
        }
        entangle(La, true);
        const float* ml = mrow + (size_t)l * n * 8;
        float m[8];
#define QSV_BACK(Q)                                                                         \
    if constexpr (n > Q) {                                                                  \
        const float4 lo = *reinterpret_cast<const float4*>(ml + Q * 8);                     \
        const float4 hi = *reinterpret_cast<const float4*>(ml + Q * 8 + 4);                 \
        m[0] = lo.x; m[1] = lo.y; m[2] = lo.z; m[3] = lo.w;                                 \
        m[4] = hi.x; m[5] = hi.y; m[6] = hi.z; m[7] = hi.w;                                 \
        if constexpr (Q < R) { if constexpr (!KEEP) small_u_reg<R, Q>(S, m); small_u_reg<R, Q>(La, m); } \
        else if constexpr (Q - R < 8) {                                                     \
            if constexpr (!KEEP) small_u_thr<R, Q - R>(S, m, tid, xc);                      \
            small_u_thr<R, Q - R>(La, m, tid, xc);                                          \
        }                                                                                   \
    }
        QSV_ALL_Q(QSV_BACK)
#undef QSV_BACK
        float d[NR], dsum = 0.f;
#pragma unroll
        for (int k = 0; k < NR; ++k) {
            d[k] = La.re[k] * S.im[k] - La.im[k] * S.re[k];
            dsum += d[k];
        }
        double v[32];
#pragma unroll
        for (int i = 0; i < 32; ++i) v[i] = 0.0;
        v[0] = (double)dsum;
#define QSV_SUMS(Q)                                                                         \
    if constexpr (n > Q) {                                                                  \
        float acc[3];                                                                       \
        small_trans<R, Q>(S, La, d, dsum, tid, xc, acc);                                    \
        v[1 + 3 * Q] = (double)acc[0]; v[2 + 3 * Q] = (double)acc[1]; v[3 + 3 * Q] = (double)acc[2]; \
    }
        QSV_ALL_Q(QSV_SUMS)
#undef QSV_SUMS
        const int v0 = reduce32<lb>(v);
        if (live && (lb < 6 || lane < 32)) {
            double* rec = a.sums + ((sample * L + l) * n_waves + wave) * 32 + v0;
#pragma unroll
            for (int i = 0; i < (lb < 5 ? 32 >> lb : 1); ++i) rec[i] = v[i];
        }
    }
#undef QSV_ALL_Q
}

inline unsigned blocks_for(u64 items, unsigned per) { return (unsigned)((items + per - 1) / per); }

// grid of the reduction kernels: chunks in x, rows over y and z (see grid_row)
inline dim3 rows_grid(unsigned nblk, u64 rows) {
    const unsigned gy = (unsigned)(rows < 32768 ? rows : 32768);
    return dim3(nblk, gy, (unsigned)((rows + gy - 1) / gy));
}

}  // namespace

// ============================================================================================
// Launchers.
template <int T, int PLANES>
static hipError_t set_attr_for() {
    const int bytes = PLANES * (1 << T) * 4;
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_pass<T, false, PLANES>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e != hipSuccess) return e;
    return hipFuncSetAttribute(reinterpret_cast<const void*>(k_pass<T, true, PLANES>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
}

constexpr int direct_lds_bytes(int tile) { return ((1 << tile) + (1 << (tile - 4))) * 4; }   // two words of padding per 32

// the variants that use 64 KiB of dynamic LDS and more; once per device
hipError_t set_pass_attributes(int device) {
    static std::mutex mu;
    static bool done[64] = {};
    std::lock_guard<std::mutex> lock(mu);
    if (device >= 0 && device < 64 && done[device]) return hipSuccess;
    hipError_t e = set_attr_for<13, 2>();
    if (e == hipSuccess) e = set_attr_for<14, 1>();
    if (e == hipSuccess)
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_pass_direct<14, false>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, direct_lds_bytes(14));
    if (e == hipSuccess)
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_pass_direct<14, false, true>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, direct_lds_bytes(14));
    if (e == hipSuccess)
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_pass_direct<14, true>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, direct_lds_bytes(14));
    if (e == hipSuccess && device >= 0 && device < 64) done[device] = true;
    return e;
}

template <int T, int PLANES>
static void launch_pass_t(const PassArgs& a, dim3 grid, hipStream_t st) {
    const size_t lds = (size_t)PLANES * ((size_t)1 << T) * sizeof(float);
    if (a.n >= T) hipLaunchKernelGGL((k_pass<T, false, PLANES>), grid, dim3(1 << (T - R)), lds, st, a);
    else hipLaunchKernelGGL((k_pass<T, true, PLANES>), grid, dim3(1 << (T - R)), lds, st, a);
}

hipError_t launch_pass(int tile, int planes, const PassArgs& a, uint64_t n_tiles, hipStream_t st) {
    if (n_tiles == 0 || n_tiles > 0x7fffffffull) return hipErrorInvalidValue;
    if (planes != 1 && planes != 2) return hipErrorInvalidValue;
    if (tile == 14) planes = 1;   // the largest tile exists with one plane only
    const dim3 grid((unsigned)n_tiles);
    if (!a.direct && (a.gather || a.unturned || a.turns)) return hipErrorInvalidValue;
    if (a.unturned && (!a.zout || !a.nostore || a.imap)) return hipErrorInvalidValue;
    if (a.direct) {
        if (a.n < tile || a.n > kDirectMaxQubits || planes != 1 || a.w + tile - a.c > a.n || a.s_in < 0 || a.s_out < 0 ||
            a.s_in > tile - R || a.s_out > tile - R)
            return hipErrorInvalidValue;
        const dim3 block(1u << (tile - R));
        const size_t bytes = (size_t)direct_lds_bytes(tile);
        switch (a.imap && a.gather ? -tile : tile) {
#define QSV_DIRECT(T)                                                                         \
    case T: if (a.unturned) hipLaunchKernelGGL((k_pass_direct<T, false, true>), grid, block, bytes, st, a);             \
            else if (a.warm_ops) hipLaunchKernelGGL((k_pass_direct<T, false, false, (T < 14)>), grid, block, bytes, st, a); \
            else hipLaunchKernelGGL((k_pass_direct<T, false>), grid, block, bytes, st, a);                          \
            break;                                                                                                  \
    case -T: if (a.warm_ops) hipLaunchKernelGGL((k_pass_direct<T, true, false, (T < 14)>), grid, block, bytes, st, a);   \
             else hipLaunchKernelGGL((k_pass_direct<T, true>), grid, block, bytes, st, a);                           \
             break;
            QSV_DIRECT(10) QSV_DIRECT(11) QSV_DIRECT(12) QSV_DIRECT(13) QSV_DIRECT(14)
#undef QSV_DIRECT
            default: return hipErrorInvalidValue;
        }
        return hipGetLastError();
    }
    switch (tile * 2 + planes - 1) {
        case 20: launch_pass_t<10, 1>(a, grid, st); break;
        case 21: launch_pass_t<10, 2>(a, grid, st); break;
        case 22: launch_pass_t<11, 1>(a, grid, st); break;
        case 23: launch_pass_t<11, 2>(a, grid, st); break;
        case 24: launch_pass_t<12, 1>(a, grid, st); break;
        case 25: launch_pass_t<12, 2>(a, grid, st); break;
        case 26: launch_pass_t<13, 1>(a, grid, st); break;
        case 27: launch_pass_t<13, 2>(a, grid, st); break;
        case 28: launch_pass_t<14, 1>(a, grid, st); break;   // two planes of 2^14 floats do not fit the offset fields
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_pair_pass(int tile, const PairArgs& a, hipStream_t st) {
    if (tile < kMinTile || tile > kPairMaxTile || a.n < tile || a.n > kDirectMaxQubits || a.w + tile - a.c > a.n || a.s_in < 0 ||
        a.s_out < 0 || a.s_in > tile - R || a.s_out > tile - R || a.rows < 1 || !a.psi || !a.sums ||
        (a.imap && a.lam_in && a.lam_in == a.lam_out) || a.psi == a.lam_out)
        return hipErrorInvalidValue;
    const u64 tiles = (u64)a.rows << (a.n - tile);
    if (tiles > 0x7fffffffull || ((u64)a.rows << (a.n - 10)) * 16 > 0xffffffffull) return hipErrorInvalidValue;
    const dim3 grid((unsigned)tiles), block(1u << (tile - R));
    const size_t bytes = (size_t)direct_lds_bytes(tile);
    switch (a.imap ? -tile : tile) {
#define QSV_PAIR(T)                                                                         \
    case T: if (a.warm_ops) hipLaunchKernelGGL((k_pair_pass<T, false, true>), grid, block, bytes, st, a);  \
            else hipLaunchKernelGGL((k_pair_pass<T, false, false>), grid, block, bytes, st, a);           \
            break;                                                                                    \
    case -T: if (a.warm_ops) hipLaunchKernelGGL((k_pair_pass<T, true, true>), grid, block, bytes, st, a);  \
             else hipLaunchKernelGGL((k_pair_pass<T, true, false>), grid, block, bytes, st, a);           \
             break;
        QSV_PAIR(10) QSV_PAIR(11) QSV_PAIR(12) QSV_PAIR(13)
#undef QSV_PAIR
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_naive_u(float2* state, int64_t rows, int n, int q, const float* mats,
                          const float* ovr, int mat_id, int n_mats, int rowdep, const RowMap& rm,
                          hipStream_t st) {
    const u64 pairs = ((u64)rows << n) >> 1;
    hipLaunchKernelGGL(k_naive_u, dim3(blocks_for(pairs, 256)), dim3(256), 0, st, state, pairs, n, q,
                       mats, ovr, mat_id, n_mats, rowdep, rm);
    return hipGetLastError();
}

hipError_t launch_naive_cnot(float2* state, int64_t rows, int n, int ctrl, int tgt, hipStream_t st) {
    const u64 total = (u64)rows << n;
    hipLaunchKernelGGL(k_naive_cnot, dim3(blocks_for(total, 256)), dim3(256), 0, st, state, total, ctrl,
                       tgt);
    return hipGetLastError();
}

hipError_t launch_naive_cz_ladder(float2* state, int64_t rows, int n, hipStream_t st) {
    const u64 total = (u64)rows << n;
    hipLaunchKernelGGL(k_naive_cz_ladder, dim3(blocks_for(total, 256)), dim3(256), 0, st, state, total,
                       n);
    return hipGetLastError();
}

// how a factored entry names its instruction sequence
inline int seq_first(MatForm f) {
    return f == MatForm::direct ? (int)direct::kSeq0 : f == MatForm::paired ? (int)paired::kSeq0 : 0;
}
inline int seq_step(MatForm f) {
    return f == MatForm::direct ? (int)direct::kSeqStride : f == MatForm::paired ? (int)paired::kSeqStride : 16;
}

hipError_t launch_build_mats(const CircDev& c, const float* params, const float* feats, int64_t samples, int inverse,
                             const int* order, int period, const int* starts, int n_starts, MatForm form, float* out,
                             double* scale, hipStream_t st) {
    if (period < 0 || (period > 0 && period != c.n) || (starts && (n_starts < 1 || !order)) ||
        (form == MatForm::paired && !(scale && starts)))
        return hipErrorInvalidValue;
    const u64 tables = (u64)(c.reupload ? samples : 1);
    const u64 per = (u64)c.n_layers * c.n;
    if (tables * per == 0) return hipSuccess;
    const u64 seg = period > 0 ? (u64)period : per;
    const u64 groups = tables * (per / seg) * (starts ? (u64)n_starts : (seg + kMatGroup - 1) / kMatGroup);
    hipLaunchKernelGGL(starts ? k_build_mats<true> : k_build_mats<false>, dim3(blocks_for(groups, 4)), dim3(256), 0, st, c, params,
                       feats, groups, inverse, order, period, starts, n_starts, form, seq_first(form), seq_step(form), out, scale);
    return hipGetLastError();
}

hipError_t launch_build_shifted(const CircDev& c, const float* params, const float* feats, int64_t samples,
                                const int* exec_of, const double* scale, int per, float* out, hipStream_t st) {
    const u64 two_p = 2ull * c.n_layers * c.slots() * c.n;
    const u64 count = (u64)(c.reupload ? samples : 1) * two_p;
    if (count == 0) return hipSuccess;
    if (scale && !exec_of) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_build_shifted, dim3(blocks_for(count, 256)), dim3(256), 0, st, c, params, feats, count,
                       exec_of, scale, per, out);
    return hipGetLastError();
}

hipError_t launch_build_turns(const CircDev& c, const float* params, const float* feats, int64_t samples, int behind,
                              float* out, hipStream_t st) {
    const u64 count = (u64)(c.reupload ? samples : 1) * c.slots() * c.n;
    if (c.n_layers != 1) return hipErrorInvalidValue;
    if (count == 0) return hipSuccess;
    hipLaunchKernelGGL(k_build_turns, dim3(blocks_for(count, 256)), dim3(256), 0, st, c, params, feats, count, behind, out);
    return hipGetLastError();
}

// ||x_b|| of every sample: inv_norm [samples] (0 for a zero vector), norm_out optional.  One launch
// when a sample fits one block, else block partials and a finishing launch.
hipError_t launch_norms(const float* x, int64_t samples, int64_t dim, double* partial, int nblk,
                        double* inv_norm, float* norm_out, hipStream_t st) {
    const bool one = nblk == 1;
    hipLaunchKernelGGL(k_sumsq, rows_grid(nblk, (u64)samples), dim3(256), 0, st, x, (u64)samples, (u64)dim, partial, nblk,
                       one ? inv_norm : (double*)nullptr, one ? norm_out : (float*)nullptr);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || one) return e;
    hipLaunchKernelGGL(k_norm_finish, dim3((unsigned)samples), dim3(256), 0, st, partial, nblk,
                       inv_norm, norm_out);
    return hipGetLastError();
}

hipError_t launch_encode(const float* x, int64_t samples, int64_t dim, int n, double* partial, int nblk, double* inv_norm,
                         float* norm_out, float2* state, hipStream_t st) {
    if (dim < 1 || dim > (int64_t)1 << n) return hipErrorInvalidValue;
    const dim3 grid = rows_grid(1, (u64)samples);
    switch (n) {
#define QSV_ROW(THREADS, V) { hipLaunchKernelGGL((k_encode_row<THREADS, V>), grid, dim3(THREADS), 0, st, x, (u64)samples, (u64)dim, n, inv_norm, norm_out, state); return hipGetLastError(); }
        case 8: QSV_ROW(64, 1);
        case 9: QSV_ROW(128, 1);
        case 10: QSV_ROW(256, 1);
        case 11: QSV_ROW(256, 2);
        case 12: QSV_ROW(256, 4);
        case 13: QSV_ROW(1024, 2);
        case 14: QSV_ROW(1024, 4);
        case 15: if (samples >= 32) QSV_ROW(1024, 8); break;
#undef QSV_ROW
        default: break;
    }
    if (n < 8) {
        hipLaunchKernelGGL(k_encode_small, grid, dim3(256), 0, st, x, (u64)samples, (u64)dim, n, inv_norm, norm_out, state);
        return hipGetLastError();
    }
    const RowMap rm{0, 0, 1, 0, 1, n};
    if (nblk == 1 || (u64)samples << n > kEncodeFolded) {
        hipError_t e = launch_norms(x, samples, dim, partial, nblk, inv_norm, norm_out, st);
        return e != hipSuccess ? e : launch_encode_write(x, dim, n, samples, inv_norm, rm, state, st);
    }
    hipLaunchKernelGGL(k_sumsq, rows_grid(nblk, (u64)samples), dim3(256), 0, st, x, (u64)samples, (u64)dim, partial, nblk,
                       (double*)nullptr, (float*)nullptr);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const u64 total = (u64)samples << n;
    hipLaunchKernelGGL((k_encode_write<true>), dim3(blocks_for(total / 2, 256)), dim3(256), 0, st, x, (u64)dim, n, total, partial, nblk,
                       inv_norm, norm_out, rm, state);
    return hipGetLastError();
}

hipError_t launch_forward_small(int regs, const float* x, int64_t dim, int64_t batch, const CircDev& c, int entangler,
                                const float* params, const float* feats, int pass_first, int pass_last, int kind,
                                float2* state, float* out, float* norm_out, hipStream_t st) {
    if (c.n < 1 || c.n > kSmallMaxQubits || batch < 1) return hipErrorInvalidValue;
    if (x && (dim < 1 || dim > ((int64_t)1 << c.n))) return hipErrorInvalidValue;
    if (pass_first < 0 || pass_last > 1 || pass_first > pass_last || (kind != 0 && !out)) return hipErrorInvalidValue;
    if (regs < 2 || regs > 4 || c.n - regs > 8) return hipErrorInvalidValue;
    if (small_mats_per_group(c, regs) > kSmallMats) return hipErrorInvalidValue;
    const SmallShape shape = small_shape(c, regs, batch);
    SmallArgs a;
    a.x = x; a.dim = dim; a.batch = batch; a.c = c; a.entangler = entangler; a.params = params; a.feats = feats;
    a.pass_first = pass_first; a.pass_last = pass_last; a.from_state = x ? 0 : 1; a.kind = kind;
    a.state = state; a.out = out; a.norm_out = norm_out;
    a.rows = shape.rows;
    a.mat_floats = shape.mat_floats;
    const int64_t blocks = (batch + a.rows - 1) / a.rows;
    if (blocks > 0x7fffffff) return hipErrorInvalidValue;
    const dim3 grid((unsigned)blocks), block(shape.threads);
    switch (regs * 16 + c.n) {
#define QSV_SMALL(R, N) \
    case R * 16 + N: hipLaunchKernelGGL((k_forward_small<R, N>), grid, block, shape.lds, st, a); break;
#define QSV_SMALL_ALL(R) QSV_SMALL(R, 1) QSV_SMALL(R, 2) QSV_SMALL(R, 3) QSV_SMALL(R, 4) QSV_SMALL(R, 5) QSV_SMALL(R, 6) \
                         QSV_SMALL(R, 7) QSV_SMALL(R, 8) QSV_SMALL(R, 9) QSV_SMALL(R, 10)
        QSV_SMALL_ALL(2) QSV_SMALL_ALL(3) QSV_SMALL_ALL(4)
#undef QSV_SMALL_ALL
#undef QSV_SMALL
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_sweep_small(const float* x, int64_t dim, int64_t batch, const CircDev& c, int entangler,
                              const float* params, const float* back, int kind, int q, uint64_t mask, const float* targets,
                              float2* kept, double* sums, double* f, hipStream_t st) {
    if (c.n < 1 || c.n > kSmallMaxQubits || batch < 1 || dim < 1 || dim > ((int64_t)1 << c.n)) return hipErrorInvalidValue;
    if (c.slots() < 1 || c.n_layers < 1 || (int64_t)c.n_layers * c.n > kSmallMats) return hipErrorInvalidValue;
    // four amplitudes per thread: eight and sixteen measured slower or the same at every batch (9 qubits x 64 47 / 59 /
    // 89 us, 10 x 1024 102 / 101 / 108 us)
    constexpr int regs = 2;
    const int rows_g = small_rows_per_group(c.n, regs), per = c.n_layers * c.n;
    const int tb = c.n > regs ? c.n - regs : 0;
    const unsigned threads = tb > 6 ? 64u << (tb - 6) : 64u;
    SweepArgs a;
    a.x = x; a.dim = dim; a.batch = batch; a.c = c; a.entangler = entangler; a.back = back;
    a.kind = kind; a.obs_qubit = q; a.mask = mask; a.targets = targets; a.f = f; a.kept = kept; a.sums = sums;
    a.rows = rows_g;
    if (c.reupload && a.rows > kSmallMats / per) a.rows = kSmallMats / per;
    a.mat_floats = (c.reupload ? a.rows : 1) * per * 8;
    const int64_t blocks = (batch + a.rows - 1) / a.rows;
    if (blocks > 0x7fffffff) return hipErrorInvalidValue;
    size_t lds = 64 * sizeof(double) + (size_t)a.mat_floats * sizeof(float);
    if (threads > 64) lds += 2 * (size_t)(2 << regs) * threads * sizeof(float);
    const dim3 grid((unsigned)blocks), block(threads);
    switch (kept ? -c.n : c.n) {
#define QSV_SWEEP(N)                                                                                   \
    case N: hipLaunchKernelGGL((k_sweep_small<regs, N, false>), grid, block, lds, st, a); break;       \
    case -N: hipLaunchKernelGGL((k_sweep_small<regs, N, true>), grid, block, lds, st, a); break;
        QSV_SWEEP(1) QSV_SWEEP(2) QSV_SWEEP(3) QSV_SWEEP(4) QSV_SWEEP(5) QSV_SWEEP(6) QSV_SWEEP(7) QSV_SWEEP(8) QSV_SWEEP(9)
        QSV_SWEEP(10)
#undef QSV_SWEEP
        default: return hipErrorInvalidValue;
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const u64 jobs = (u64)batch * per * c.slots();
    hipLaunchKernelGGL(k_adj_all, dim3(blocks_for(jobs, 256)), dim3(256), 0, st, sums, (int)(threads / 64), c, params, (u64)batch,
                       back, f);
    return hipGetLastError();
}

hipError_t launch_encode_write(const float* x, int64_t dim, int n, int64_t rows, const double* inv_norm,
                               const RowMap& rm, float2* state, hipStream_t st) {
    const u64 total = (u64)rows << n;
    hipLaunchKernelGGL((k_encode_write<false>), dim3(blocks_for(total / 2, 256)), dim3(256), 0, st, x, (u64)dim, n, total,
                       (const double*)nullptr, 0, const_cast<double*>(inv_norm), (float*)nullptr, rm, state);
    return hipGetLastError();
}

hipError_t launch_probs(const float2* state, uint64_t total, float* out, hipStream_t st) {
    hipLaunchKernelGGL(k_probs, dim3(blocks_for(total / 2, 256)), dim3(256), 0, st, state, (u64)total,
                       out);
    return hipGetLastError();
}

static inline int chunk_blocks(int bits) { return bits > CHUNK_BITS ? 1 << (bits - CHUNK_BITS) : 1; }

// Chunks a block of k_expz_block takes, as a power of two: as many as leave the chip eight blocks per CU.
static int expz_group(int n, int64_t rows) {
    const int chunks = n > CHUNK_BITS ? n - CHUNK_BITS : 0;
    int g = 0;
    while (g < 4 && g < chunks && (rows << (chunks - g - 1)) >= 2048) ++g;
    return g;
}

// Few rows: a workgroup each, which spreads them over the CUs (12 qubits x 64: 6.3 -> 5.6 us).
static hipError_t launch_expz_row(const float2* state, int64_t rows, int n, int q_only, float* out, double* partial,
                                  hipStream_t st) {
    const unsigned waves = rows <= 1024 ? 1 : 4;
    hipLaunchKernelGGL(k_expz_row, dim3(blocks_for((u64)rows, waves)), dim3(64 * waves), 0, st, state, (u64)rows, n, q_only,
                       out, partial);
    return hipGetLastError();
}

hipError_t launch_expz_block(const float2* state, int64_t rows, int n, double* partial, hipStream_t st) {
    if (n < CHUNK_BITS) return launch_expz_row(state, rows, n, -1, nullptr, partial, st);
    const int g = expz_group(n, rows), nblk = chunk_blocks(n) >> g;
    hipLaunchKernelGGL(k_expz_block, rows_grid(nblk, (u64)rows), dim3(256), 0, st, state, (u64)rows, n, g, nblk, partial,
                       (float*)nullptr, -1);
    return hipGetLastError();
}
bool expz_in_one_launch(int n, int64_t rows) { return n <= 14 || (n <= 16 && rows >= 64); }
hipError_t launch_expz_small(const float2* state, int64_t rows, int n, int q_only, float* out_f, hipStream_t st) {
    if (!expz_in_one_launch(n, rows) || !out_f || q_only >= n) return hipErrorInvalidValue;
    if (n > CHUNK_BITS) {
        hipLaunchKernelGGL(k_expz_block, rows_grid(1, (u64)rows), dim3(256), 0, st, state, (u64)rows, n, n - CHUNK_BITS, 1,
                           (double*)nullptr, out_f, q_only);
        return hipGetLastError();
    }
    return launch_expz_row(state, rows, n, q_only, out_f, nullptr, st);
}
static hipError_t expz_finish(const double* partial, int64_t rows, int n, int q_only, float* out_f, double* out_d,
                              const Scatter& sc, const Residues* res, int rowdep, hipStream_t st) {
    const u64 jobs = (u64)rows * (q_only >= 0 ? 1 : n);
    const int g = expz_group(n, rows), nblk = chunk_blocks(n) >> g;
    const bool whole = nblk >= 1024 && jobs <= 4096;
    const auto kernel = whole ? (res ? k_expz_finish<true, true> : k_expz_finish<true>)
                              : (res ? k_expz_finish<false, true> : k_expz_finish<false>);
    hipLaunchKernelGGL(kernel, dim3(whole ? (unsigned)jobs : blocks_for(jobs, 4)), dim3(256), 0, st, partial, (u64)rows, n, g, nblk,
                       q_only, out_f, out_d, sc, res ? *res : Residues{nullptr, 0, 0, 0}, rowdep);
    return hipGetLastError();
}
hipError_t launch_expz_finish(const double* partial, int64_t rows, int n, int q_only, float* out_f,
                              double* out_d, hipStream_t st, const Residues* res, int rowdep) {
    if (res && !res->table) return hipErrorInvalidValue;
    return expz_finish(partial, rows, n, q_only, out_f, out_d, Scatter{0, 0, 0, 0}, res, rowdep, st);
}
hipError_t launch_expz_finish_scatter(const double* partial, int64_t rows, int n, int q, double* out,
                                      const Scatter& sc, hipStream_t st, const Residues* res, int rowdep) {
    if (q < 0 || sc.per < 1 || (res && !res->table)) return hipErrorInvalidValue;
    return expz_finish(partial, rows, n, q, nullptr, out, sc, res, rowdep, st);
}
hipError_t launch_zsum_finish(const double* partial, int64_t rows, int64_t per_row, double* out,
                              const Scatter& sc, hipStream_t st) {
    if (rows < 1 || per_row < 1 || sc.per < 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_zsum_finish, dim3(blocks_for((u64)rows, 256)), dim3(256), 0, st, partial, (u64)rows,
                       (u64)per_row, out, sc);
    return hipGetLastError();
}

hipError_t launch_turned_finish(const double* partial, int64_t rows, int64_t per_row, double* out, const Scatter& sc,
                                int64_t unturned_at, const Residues& ra, const Residues& rb1, const Residues& rb2, int rowdep,
                                hipStream_t st) {
    if (rows < 1 || per_row < 1 || sc.per < 1) return hipErrorInvalidValue;
    const TurnedArgs t{sc, (u64)unturned_at, ra, rb1, rb2, rowdep};
    hipLaunchKernelGGL(k_turned_finish, dim3(blocks_for((u64)rows, 4)), dim3(256), 0, st, partial, (u64)rows,
                       (u64)per_row, out, t);
    return hipGetLastError();
}

hipError_t launch_gather_rows(const float2* src, int n, int64_t rows, const RowMap& rm, float2* states,
                              hipStream_t st) {
    if (n < 1) return hipErrorInvalidValue;   // rows of one amplitude cannot be copied in pairs
    const u64 total = (u64)rows << n;
    hipLaunchKernelGGL(k_gather_rows, dim3(blocks_for(total / 2, 256)), dim3(256), 0, st, src, n, total, rm,
                       states);
    return hipGetLastError();
}

hipError_t launch_marginal_block(const float2* state, int64_t rows, int n, uint64_t mask, int64_t n_v,
                                 double* partial, hipStream_t st) {
    const int m = __builtin_popcountll(mask);
    const u64 sub = 1ull << (n - m);
    const u64 nblk = (u64)chunk_blocks(n - m);
    const u64 blocks = (u64)rows * (u64)n_v * nblk;
    if (blocks > 0x7fffffffull) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_marginal_block, dim3((unsigned)blocks), dim3(256), 0, st, state, n, (u64)mask,
                       (u64)n_v, nblk, sub, partial);
    return hipGetLastError();
}

hipError_t launch_marginal_finish(const double* partial, int64_t jobs, int64_t nblk, float* out,
                                  int renorm_mode, double* scale, hipStream_t st) {
    hipLaunchKernelGGL(k_marginal_finish, dim3(blocks_for((u64)jobs, 4)), dim3(256), 0, st, partial,
                       (u64)jobs, (u64)nblk, out, renorm_mode, scale);
    return hipGetLastError();
}

hipError_t launch_project(float2* state, int64_t rows, int n, uint64_t mask, const double* scale,
                          hipStream_t st) {
    const u64 total = (u64)rows << n;
    hipLaunchKernelGGL(k_project, dim3(blocks_for(total, 256)), dim3(256), 0, st, state, total, n,
                       (u64)mask, scale);
    return hipGetLastError();
}

hipError_t launch_fidelity_block(const float2* state, int64_t rows, int n, const float* x, int64_t dim,
                                 double* partial, int nblk, const RowMap& rm, hipStream_t st) {
    hipLaunchKernelGGL(k_fidelity_block, rows_grid(nblk, (u64)rows), dim3(256), 0, st, state, (u64)rows, n, x,
                       (u64)dim, nblk, rm, partial);
    return hipGetLastError();
}

hipError_t launch_fidelity_finish(const double* partial, int nblk, int64_t rows, float* out, double* out_d,
                                  hipStream_t st) {
    hipLaunchKernelGGL(k_fidelity_finish, dim3((unsigned)rows), dim3(256), 0, st, partial, nblk, out, out_d);
    return hipGetLastError();
}

hipError_t launch_reset_rows(const float2* state, int n, uint64_t mask, int64_t rows, const RowMap& rm,
                             float2* work, hipStream_t st) {
    const u64 total = (u64)rows << n;
    hipLaunchKernelGGL(k_reset_rows, dim3(blocks_for(total / 2, 256)), dim3(256), 0, st, state, n, (u64)mask,
                       total, rm, work);
    return hipGetLastError();
}

hipError_t launch_reset_sum(const double* Frow, int64_t per, int64_t B, float* out, hipStream_t st) {
    hipLaunchKernelGGL(k_reset_sum, dim3(blocks_for((u64)B, 256)), dim3(256), 0, st, Frow, (u64)per, (u64)B, out);
    return hipGetLastError();
}

hipError_t launch_shot_expz(const long long* samples, int64_t shots, int64_t rows, int n, float* out,
                            hipStream_t st) {
    // a wavefront per 64 samples, at most 16 of them
    const unsigned threads = shots > 512 ? 1024u : shots > 128 ? 256u : 64u;
    hipLaunchKernelGGL(k_shot_expz, dim3((unsigned)rows), dim3(threads), 0, st, samples, (u64)shots, n, out);
    return hipGetLastError();
}

hipError_t launch_pauli(const float2* state, int64_t rows, int n, uint64_t xmask, uint64_t ymask,
                        uint64_t zmask, double* partial, float* out, hipStream_t st) {
    const u64 f = (u64)(xmask | ymask);
    const int nblk = chunk_blocks(f ? n - 1 : n);    // with flips, half the indices are visited
    hipLaunchKernelGGL(k_pauli_block, rows_grid(nblk, (u64)rows), dim3(256), 0, st, state, (u64)rows, n,
                       f, (u64)(ymask | zmask), __builtin_popcountll(ymask), nblk, partial);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_pauli_finish, dim3((unsigned)rows), dim3(256), 0, st, partial, nblk,
                       __builtin_popcountll(ymask), out);
    return hipGetLastError();
}

hipError_t launch_sample(const float2* state, int64_t rows, int n, const double* uniforms, int64_t shots,
                         unsigned long long* cum, unsigned long long* sub, long long* out, hipStream_t st) {
    const int nblk = chunk_blocks(n);
    hipLaunchKernelGGL(k_sample_blocksum, rows_grid(nblk, (u64)rows), dim3(256), 0, st, state, (u64)rows, n, nblk,
                       cum, sub);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_sample_scan, dim3((unsigned)rows), dim3(1024), 0, st, cum, nblk);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    const u64 jobs = (u64)rows * (u64)shots;
    if (jobs == 0) return hipSuccess;
    hipLaunchKernelGGL(k_sample_draw, dim3(blocks_for(jobs, 4)), dim3(256), 0, st, state, n, nblk, cum, sub,
                       uniforms, (u64)shots, jobs, out);
    return hipGetLastError();
}

hipError_t launch_adj_init(const float2* A, int n, int kind, int q, uint64_t mask, const double* coef,
                           int64_t rows, float2* S, int paired, hipStream_t st) {
    if (n < 1 || rows < 1 || kind < 0 || kind > 2 || (kind == 2 && !coef)) return hipErrorInvalidValue;
    const u64 total = (u64)rows << n;
    const AdjObs o{kind, q, (u64)mask, coef};
    hipLaunchKernelGGL(k_adj_init, dim3(blocks_for(total / 2, 256)), dim3(256), 0, st, A, n, o, total, S, paired);
    return hipGetLastError();
}

hipError_t launch_trash_loss(const float2* A, int n, uint64_t mask, int64_t rows, int64_t sample0, int64_t P,
                             double* partial, double* f, hipStream_t st, const Residues* res, int rowdep) {
    if (rows < 1 || (res && !res->table)) return hipErrorInvalidValue;
    const int nblk = chunk_blocks(n);
    hipLaunchKernelGGL(k_p0_block, rows_grid(nblk, (u64)rows), dim3(256), 0, st, A, (u64)rows, n, (u64)mask, nblk, partial);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(res ? k_trash_loss<true> : k_trash_loss<false>, dim3(blocks_for((u64)rows, 256)), dim3(256), 0, st, partial,
                       nblk, (u64)rows, (u64)sample0, (u64)P, f, res ? *res : Residues{nullptr, 0, 0, 0}, rowdep);
    return hipGetLastError();
}

hipError_t launch_mse_coef(const double* z, const float* y, int n, int64_t rows, int64_t sample0, int64_t P,
                           double* coef, double* f, hipStream_t st) {
    hipLaunchKernelGGL(k_mse_coef, dim3(blocks_for((u64)rows, 256)), dim3(256), 0, st, z, y, n, (u64)rows,
                       (u64)sample0, (u64)P, coef, f);
    return hipGetLastError();
}

hipError_t launch_sgd(float* p, const float* g, int64_t count, double lr, hipStream_t st) {
    if (count < 1) return hipSuccess;
    hipLaunchKernelGGL(k_sgd, dim3(blocks_for((u64)count, 256)), dim3(256), 0, st, p, g, (u64)count, lr);
    return hipGetLastError();
}

hipError_t launch_adam(float* p, const float* g, float* m, float* v, int64_t count, int64_t t, double lr,
                       double b1, double b2, double eps, hipStream_t st) {
    if (count < 1) return hipSuccess;
    const double c1 = 1.0 - pow(b1, (double)t), c2 = 1.0 - pow(b2, (double)t);
    hipLaunchKernelGGL(k_adam, dim3(blocks_for((u64)count, 256)), dim3(256), 0, st, p, g, m, v, (u64)count,
                       lr, b1, b2, eps, c1, c2);
    return hipGetLastError();
}



// The fewest tiles of a row one workgroup of the tile kernels takes, and the resulting (largest
// number of) groups per row.
static inline int trans_tiles_per_group(int n) { const int tiles = 1 << (n - 12); return tiles < 4 ? tiles : 4; }
static inline int trans_groups(int n) { return (1 << (n - 12)) / trans_tiles_per_group(n); }

// upper bound of the partial entries per (row pair, qubit) of the transition sums
int adj_trans_blocks(int n) { return n < 12 ? 1 : 4 * trans_groups(n); }

// A workgroup's first load and last sums overlap with nothing, so it takes as many tiles as still leaves two
// workgroups per compute unit (never fewer than the buffer was sized for).
static inline int trans_per_group(int n, int64_t row_pairs) {
    const int tiles = 1 << (n - 12);
    int per_group = trans_tiles_per_group(n);
    while (per_group * 2 <= tiles && per_group < 32 && (int64_t)(tiles / (per_group * 2)) * row_pairs >= 512)
        per_group *= 2;
    return per_group;
}
// partial entries per (row pair, qubit): one per wavefront of a group of tiles
int adj_trans_count(int n, int64_t row_pairs) {
    return n < 12 ? adj_trans_blocks(n) : 4 * ((1 << (n - 12)) / trans_per_group(n, row_pairs));
}

hipError_t launch_trans(const float2* psi0, const float2* lam0, int rstride, int n, int64_t row_pairs, double* partial,
                        hipStream_t st) {
    if (row_pairs < 1 || row_pairs > 65535) return hipErrorInvalidValue;
    const int nblk = adj_trans_count(n, row_pairs);
    if (n < 12) {
        hipLaunchKernelGGL(k_trans_block, dim3(nblk, n, (unsigned)row_pairs), dim3(256), 0, st, psi0, lam0, rstride,
                           n, (u64)1 << (n - 1), nblk, partial);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    } else {
        // qubits 0..11 from contiguous tiles, then 8 more per read from tiles whose window sits higher
        // (the last window ends at bit n and only its not yet covered qubits are taken)
        const int per_group = trans_per_group(n, row_pairs), groups = (1 << (n - 12)) / per_group;
        const dim3 grid(groups, (unsigned)row_pairs);
        hipLaunchKernelGGL((k_trans_wave<3>), grid, dim3(256), 0, st, psi0, lam0, rstride, n, 12, 12, 0, per_group,
                           nblk, partial);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        for (int done = 12; done < n;) {
            int w = done, j0 = 4;
            if (w + 8 > n) { w = n - 8; j0 = 4 + (done - w); }
            switch (j0) {
#define QSV_TRANS_CASE(J) case J: hipLaunchKernelGGL((k_trans_tile<J>), grid, dim3(256), 0, st, psi0, lam0, rstride, n, 4, w, per_group, nblk, partial); break;
                case 4: case 5: case 6: case 7:
                    hipLaunchKernelGGL((k_trans_wave<2>), grid, dim3(256), 0, st, psi0, lam0, rstride, n, 4, w, j0, per_group,
                                       nblk, partial);
                    break;
                QSV_TRANS_CASE(8) QSV_TRANS_CASE(9) QSV_TRANS_CASE(10) QSV_TRANS_CASE(11)
#undef QSV_TRANS_CASE
                default: return hipErrorInvalidValue;
            }
            e = hipGetLastError();
            if (e != hipSuccess) return e;
            done = w + 8;
        }
    }
    return hipSuccess;
}

hipError_t launch_adj_layers(double* partial, int64_t row_pairs, const CircDev& c, int layer0, int n_layers,
                             const float* params, int64_t sample0, int64_t P, const float* back, const int* exec_of,
                             MatForm form, double* f, hipStream_t st) {
    const u64 jobs = (u64)n_layers * row_pairs * c.slots() * c.n, sums_n = (u64)n_layers * row_pairs * c.n;
    if (jobs == 0) return hipSuccess;
    const int nblk = adj_trans_count(c.n, row_pairs);
    const double* sums = partial;
    if (nblk > 1) {   // the summed matrices go behind the partials
        double* M = partial + sums_n * nblk * 8;
        hipLaunchKernelGGL(k_trans_finish, dim3(blocks_for(sums_n, 4)), dim3(256), 0, st, partial, nblk, sums_n, M);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        sums = M;
    }
    hipLaunchKernelGGL(k_adj_layers, dim3(blocks_for(jobs, 256)), dim3(256), 0, st, sums, c, layer0, n_layers, params,
                       (u64)sample0, (u64)row_pairs, (u64)P, back, exec_of, form == MatForm::plain ? 1 : 0,
                       seq_first(form), seq_step(form), f);
    return hipGetLastError();
}

hipError_t launch_pair_finish(const float* sums, int64_t rows, const CircDev& c, const float* params, int64_t sample0,
                              int64_t P, const int* order, const int* entry_of, const float* back, int n_mats,
                              const double* corr, double* f, hipStream_t st) {
    const u64 jobs = (u64)rows * c.n_layers * c.n;
    if (jobs == 0 || c.slots() < 1) return hipSuccess;
    const int waves = 1 << (c.n - 10);
    const int lanes = waves < 4 ? 4 : waves > 64 ? 64 : waves;     // a lane per slot at least
    hipLaunchKernelGGL(k_pair_finish, dim3(blocks_for(jobs * lanes, 256)), dim3(256), 0, st,
                       reinterpret_cast<const float4*>(sums), waves, lanes, c, params, (u64)rows, (u64)sample0, (u64)P,
                       order, entry_of, back, n_mats, corr, seq_first(MatForm::paired), seq_step(MatForm::paired), f);
    return hipGetLastError();
}

hipError_t launch_grad_finish(const double* f, int64_t B, int64_t P, const CircDev& c, const float* feats,
                              float* loss, float* grad, float* mean_loss, float* mean_grad,
                              hipStream_t st) {
    hipLaunchKernelGGL(k_grad_finish, dim3(blocks_for((u64)B * (P + 1), 256)), dim3(256), 0, st, f,
                       (u64)B, (u64)P, c, feats, loss, grad);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (mean_loss || mean_grad) {
        hipLaunchKernelGGL(k_grad_mean, dim3((unsigned)(P + 1)), dim3(256), 0, st, f, (u64)B,
                           (u64)P, c, feats, mean_loss, mean_grad);
        e = hipGetLastError();
    }
    return e;
}

}  // namespace qsv

// ============================================================================================
// Scratch memory for callers that cannot allocate (code under HIP graph capture, serving loops,
// harnesses that forbid hipMalloc): a fixed array in the code object, one copy per GPU that loads
// the library, held until the process ends.  Its name is a host-side stand-in, not a device
// address: host code asks the runtime for the address once per device and uses that pointer.
static __device__ __align__(256) unsigned char scratch[qsv::kStaticScratchBytes];

namespace qsv {

hipError_t static_scratch(int device, void** ptr) {
    constexpr int kMaxDevices = 64;
    static void* ptrs[kMaxDevices] = {};
    static std::mutex mu;
    if (device < 0 || device >= kMaxDevices || !ptr) return hipErrorInvalidValue;
    std::lock_guard<std::mutex> lock(mu);
    if (!ptrs[device]) {
        // the caller has made `device` current: the address is that device's copy of the array
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        ptrs[device] = p;
    }
    *ptr = ptrs[device];
    return hipSuccess;
}

}  // namespace qsv
