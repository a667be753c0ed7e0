// HIP kernels of the docking hot path for gfx950 (MI355X, CDNA4, wave64).
//
// One wave owns one individual, but for the layouts below. The per-evaluation
// pipeline (Sec. 2.1 of the paper: pose from the genotype, pairwise free-energy
// terms, gradient and torque sums, ADADELTA step) runs entirely inside the wave:
//
//   genotype (lane c holds gene c)
//   -> torsion transforms (lane k: Rodrigues rotation about bond k)
//   -> atom positions (lane a: atom a in depth-first order, a second slot
//      holds atom a + 64 for ligands of 65..128 atoms): the torsions that
//      enclose the atom's fragment, innermost first, then the rigid rotation
//   -> grid term: trilinear interpolation of three maps per atom
//   -> pair terms: host-built batches of 64 kept pairs, one pair per lane,
//      forces added to per-copy LDS accumulators of both atoms
//   -> block sum of {E, gx, gy, gz} (Sec. 3/4.2; selectable shuffle or MFMA
//      variants); torque and torsion torques by a wave prefix scan
//   -> gradient with respect to the genotype, ADADELTA update.
//
// Two waves or four may hold an individual (ls_kernel_mw), two individuals a wave
// (ls_kernel_two, score_kernel_two), and the waves of a block may share the pair
// terms of one individual (ls_kernel_coop, the same results as a wave each). Only
// kernels with several waves per individual have block barriers, no LDS or global
// float atomics are used, and every sum runs in a fixed order, so results are
// deterministic run to run and independent of what else shares the launch.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <atomic>

#include "dock.h"
#include "dock_blob.h"
#include "dock_launch.h"

// No fused operation but those written out (fmaf), so that a kernel's rounding
// does not hang on what else the compiler finds to share there: searches amplify a
// last-bit difference within a few steps. The kernels do not all round alike:
// which square of a separation (pair_term's xfirst) or of an outside distance
// (grid_term's XFIRST) is added first is what each kernel's results have always
// been formed with, by batch and by kernel, and is kept for their sake. The trial
// energies of a random search can so differ from dock_score_batch's in last bits.
#pragma clang fp contract(off)

namespace {

using dockblob::Header;
using dockblob::Torsion;
using docklaunch::DevItem;
using docklaunch::GridParams;
using docklaunch::LsParams;

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

constexpr int kWave = 64;
// Fourth word of a raw buffer resource on CDNA (32-bit data format, no
// swizzle, no stride): loads address bytes [0, num_records).
constexpr int kBufferWord3 = 0x00020000;
constexpr int kMaxTors = dockblob::kMaxTorsions;
constexpr int kMaxFrag = dockblob::kMaxFrag;
constexpr int kChain = dockblob::kChainStride;

// Force-field constants (AutoDock4 forms, Mehler-Solmajer dielectric).
constexpr float kR2Min = 1.0e-4f;        // A^2 lower clamp on r^2
constexpr float kCap = 1.0e5f;           // cap of the 12-6 / 12-10 term
constexpr float kOut = 100.0f;           // outside-the-box penalty constant
constexpr float kDielA = -8.5525f;
constexpr float kDielB = 86.9525f;       // eps0 - A with eps0 = 78.4
constexpr float kDielK = 7.7839f;
constexpr float kDielLB = 0.003627f * 86.9525f;            // lambda * B
constexpr float kDielBKLB = 86.9525f * 7.7839f * 0.003627f * 86.9525f;
constexpr float kDsInv2S2 = 1.0f / (2.0f * 3.5f * 3.5f);   // 1 / (2 sigma^2)
constexpr float kDsInvS2 = 1.0f / (3.5f * 3.5f);
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kSqrtElec = 18.222613f;      // sqrt(332.06363 kcal A / (mol e^2)): charges in LDS carry it

// ---------------------------------------------------------------------------
// Cross-lane primitives (wave64).
// ---------------------------------------------------------------------------

template <int CTRL, int ROW_MASK = 0xf, int BANK_MASK = 0xf>
__device__ __forceinline__ float dpp(float v) {
    // lanes whose source is outside the row, or whose row is masked off, read 0
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(
        0, __builtin_bit_cast(int, v), CTRL, ROW_MASK, BANK_MASK, true));
}

__device__ __forceinline__ float readlane(float v, int l) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l));
}

__device__ __forceinline__ int lane_id() { return (int)__lane_id(); }

// Value of lane `l` mod 64 (the permute reads bits 2 to 7 of its byte address).
__device__ __forceinline__ float lane_at(float v, uint32_t l) {
    return __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute((int)(l << 2), __builtin_bit_cast(int, v)));
}

// Ordering of LDS accesses between the lanes of one wave, where one wave is
// everything that shares the data: a wave's LDS instructions execute in
// program order, so it only has to keep the compiler from moving LDS
// accesses across this point (a wavefront-scope fence orders them in the
// compiler; the wave barrier keeps the instruction scheduler from moving
// them). No block barrier: another wave of the block may be working on
// something else, at another point of its code.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// The LDS ordering an evaluation needs: the wave's own when it holds the
// whole individual, the block's when WAVES waves share it.
template <int WAVES>
__device__ __forceinline__ void lds_sync() {
    if constexpr (WAVES == 1) wave_sync();
    else __syncthreads();
}

// Block barrier that orders LDS accesses only: __syncthreads also waits for the
// wave's global loads, which the shared evaluation keeps in flight across it.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Wave-uniform value: lets the compiler keep it (and what is derived from it,
// such as loop bounds and addresses) in scalar registers.
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
template <class T>
__device__ __forceinline__ T* uniform_ptr(T* p) {
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return reinterpret_cast<T*>(((uint64_t)hi << 32) | lo);
}

// Global-memory view of a pointer, so that loads are issued as global (not
// flat) instructions and do not count against the LDS wait counter.
template <class T>
__device__ __forceinline__ const __attribute__((address_space(1))) T* gmem(const T* p) {
    return (const __attribute__((address_space(1))) T*)(p);
}

// Broadcast of lane `c` of each 16-lane row to that row.
template <int C>
__device__ __forceinline__ float row_lane(float v) { return dpp<0x150 + C>(v); }

// The DPP steps of the sums and scans below, one instruction per step. They
// are written out because the compiler does not fold a masked row broadcast
// into the addition (a zero, a move and an addition instead of one v_add).
// Lanes whose source lies outside their row add 0; rows a broadcast masks off
// keep their value. A DPP operand must have been written at least two
// instructions before: N independent values are stepped side by side, with
// waits only where fewer than three are. Every block ends with two wait states:
// the compiler does not see what a block wrote last, and a lane read of it needs
// one, a DPP instruction of its own two (tests/test_asm_waits_cpu.py).
#define DPP_STEP(r, how) "v_add_f32_dpp " r ", " r ", " r " " how "\n\t"
#define DPP_ROW "row_mask:0xf bank_mask:0xf bound_ctrl:1"
#define DPP_STEP1(how) DPP_STEP("%0", how) "s_nop 1\n\t"
#define DPP_STEP4(how) DPP_STEP("%0", how) DPP_STEP("%1", how) DPP_STEP("%2", how) DPP_STEP("%3", how)
#define DPP_STEP6(how) DPP_STEP4(how) DPP_STEP("%4", how) DPP_STEP("%5", how)
#define DPP_END "s_nop 1"
#define DPP_ROW_SUM(STEP) \
    STEP("quad_perm:[1,0,3,2] " DPP_ROW) STEP("quad_perm:[2,3,0,1] " DPP_ROW) \
    STEP("row_half_mirror " DPP_ROW) STEP("row_mirror " DPP_ROW)
#define DPP_ROW_SCAN(STEP) \
    STEP("row_shr:1 " DPP_ROW) STEP("row_shr:2 " DPP_ROW) STEP("row_shr:4 " DPP_ROW) STEP("row_shr:8 " DPP_ROW)
#define DPP_HALF(STEP) STEP("row_bcast:15 row_mask:0xa bank_mask:0xf")
#define DPP_WAVE(STEP) DPP_HALF(STEP) STEP("row_bcast:31 row_mask:0xc bank_mask:0xf")

// Sum over the wave, every lane receives the same value. Butterfly inside
// each 16-lane row with DPP (quad swaps, half-row and row mirrors), then the
// row sums S0..S3 are combined by row broadcasts as (S3 + S2) + (S1 + S0)
// in the last lane, which is read as a scalar.
__device__ __forceinline__ float wave_sum(float v) {
    asm("s_nop 1\n\t" DPP_ROW_SUM(DPP_STEP1) DPP_WAVE(DPP_STEP1) : "+v"(v));
    return readlane(v, 63);
}
__device__ __forceinline__ float4 wave_sum4(float4 v) {
    asm("s_nop 1\n\t" DPP_ROW_SUM(DPP_STEP4) DPP_WAVE(DPP_STEP4) DPP_END : "+v"(v.x), "+v"(v.y), "+v"(v.z), "+v"(v.w));
    return make_float4(readlane(v.x, 63), readlane(v.y, 63), readlane(v.z, 63), readlane(v.w, 63));
}

__device__ __forceinline__ float wave_max(float v) {
    v = fmaxf(v, dpp<0xB1>(v));
    v = fmaxf(v, dpp<0x4E>(v));
    v = fmaxf(v, dpp<0x141>(v));
    v = fmaxf(v, dpp<0x140>(v));
    return fmaxf(fmaxf(readlane(v, 0), readlane(v, 16)), fmaxf(readlane(v, 32), readlane(v, 48)));
}

// Inclusive prefix sums of six values over the 64 lanes.
__device__ __forceinline__ void wave_scan6(float v[6]) {
    asm("s_nop 1\n\t" DPP_ROW_SCAN(DPP_STEP6) DPP_WAVE(DPP_STEP6) DPP_END
        : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "+v"(v[4]), "+v"(v[5]));
}

// ---------------------------------------------------------------------------
// Block sum of 4-vectors over one wave: the variants of the paper's step.
// ---------------------------------------------------------------------------

// R0: plain wavefront shuffle (the Sec. 3 baseline without its atomics and
// barriers: one wave needs neither).
__device__ __forceinline__ float4 sum4_shuffle(float4 v) {
    return wave_sum4(v);
}

// Tail shared by the MFMA variants. The 16x16 result holds, in column n,
// partial sums of component n % 4; lane l owns rows 4(l/16)..4(l/16)+3 of
// column l % 16. Adding its four rows and the matching lanes of the other
// three lane groups gives every lane the total of component l % 4.
__device__ __forceinline__ float4 mfma_tail(f32x4 acc) {
    float s = (acc[0] + acc[1]) + (acc[2] + acc[3]);
    s += __shfl_xor(s, 16);
    s += __shfl_xor(s, 32);
    return make_float4(readlane(s, 0), readlane(s, 1), readlane(s, 2), readlane(s, 3));
}

// R1: FP32 MFMA 16x16x4. The analogue of the paper's V = A P: each lane's
// component c enters A (row l % 16, k = l / 16); B is a 0/1 selection matrix
// that routes component c to the columns n with n % 4 == c, so four
// accumulating products leave, in each column, the sums over k (lanes l,
// l+16, l+32, l+48) of one component. The second product of the paper (Q V)
// is replaced by the in-register tail.
__device__ __forceinline__ float4 sum4_mfma_f32(float4 v) {
    const int c = lane_id() & 3;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(v.x, c == 0 ? 1.f : 0.f, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(v.y, c == 1 ? 1.f : 0.f, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(v.z, c == 2 ? 1.f : 0.f, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(v.w, c == 3 ? 1.f : 0.f, acc, 0, 0, 0);
    return mfma_tail(acc);
}

// R2: half-width MFMA 16x16x32 with split operands (precision refinement):
// each lane supplies 8 narrow values, hi and lo parts of its 4 components,
// B[k][n] = [k % 4 == n % 4], and the matrix unit adds hi + lo of 4 lanes per
// output element in FP32. The selection is invariant to how the unit maps
// (lane, slot) to k, since A and B share that mapping and k % 4 = slot % 4.
__device__ __forceinline__ bf16x8 sel_bf16() {
    const int c = lane_id() & 3;
    bf16x8 b;
#pragma unroll
    for (int i = 0; i < 8; ++i) b[i] = (__bf16)(((i & 3) == c) ? 1.0f : 0.0f);
    return b;
}

template <int TERMS>
__device__ __forceinline__ float4 sum4_mfma_bf16(float4 v) {
    const float vv[4] = {v.x, v.y, v.z, v.w};
    bf16x8 a;
    bf16x8 a2;
    float rem[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        __bf16 h = (__bf16)vv[i];
        a[i] = h;
        rem[i] = vv[i] - (float)h;
        __bf16 m = (__bf16)rem[i];
        a[4 + i] = m;
        rem[i] = rem[i] - (float)m;
        a2[i] = (__bf16)rem[i];
        a2[4 + i] = (__bf16)0.0f;
    }
    const bf16x8 b = sel_bf16();
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc, 0, 0, 0);
    if (TERMS == 3) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a2, b, acc, 0, 0, 0);
    return mfma_tail(acc);
}

// FP16 has 5 exponent bits, so each component is first scaled by a power of
// two that brings the wave's largest magnitude just below 2^14 (exact), and
// the sum is scaled back (exact).
__device__ __forceinline__ float4 sum4_mfma_f16(float4 v) {
    const float vv[4] = {v.x, v.y, v.z, v.w};
    float mx[4] = {wave_max(fabsf(v.x)), wave_max(fabsf(v.y)), wave_max(fabsf(v.z)),
                   wave_max(fabsf(v.w))};
    int k[4];
    f16x8 a;
    f16x8 b;
    const int c = lane_id() & 3;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        k[i] = (mx[i] > 0.f && mx[i] <= 3.0e38f) ? 13 - ilogbf(mx[i]) : 0;
        k[i] = k[i] < -120 ? -120 : (k[i] > 120 ? 120 : k[i]);
        float s = ldexpf(vv[i], k[i]);
        _Float16 h = (_Float16)s;
        a[i] = h;
        a[4 + i] = (_Float16)(s - (float)h);
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) b[i] = (_Float16)(((i & 3) == c) ? 1.0f : 0.0f);
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, acc, 0, 0, 0);
    float4 t = mfma_tail(acc);
    return make_float4(ldexpf(t.x, -k[0]), ldexpf(t.y, -k[1]), ldexpf(t.z, -k[2]),
                       ldexpf(t.w, -k[3]));
}

template <int VAR>
__device__ __forceinline__ float4 sum4(float4 v) {
    if constexpr (VAR == DOCK_REDUCE_SHUFFLE) return sum4_shuffle(v);
    else if constexpr (VAR == DOCK_REDUCE_MFMA_F32) return sum4_mfma_f32(v);
    else if constexpr (VAR == DOCK_REDUCE_MFMA_BF16) return sum4_mfma_bf16<2>(v);
    else if constexpr (VAR == DOCK_REDUCE_MFMA_F16) return sum4_mfma_f16(v);
    else return sum4_mfma_bf16<3>(v);
}

// A variant known at run time only. The kernels that serve several hold one
// evaluation that chooses here: with one evaluation per variant side by side
// the ligand lived in scratch memory (328 bytes a lane), and searches on plain
// maps, 3000 individuals and 41 evaluations, took 505 us instead of 240 (24
// atoms), 973 instead of 424 (48) and 4,490 instead of 1,857 (112).
__device__ __forceinline__ float4 sum4_of(int var, float4 v) {
    switch (var) {
        case DOCK_REDUCE_MFMA_F32: return sum4<DOCK_REDUCE_MFMA_F32>(v);
        case DOCK_REDUCE_MFMA_BF16: return sum4<DOCK_REDUCE_MFMA_BF16>(v);
        case DOCK_REDUCE_MFMA_F16: return sum4<DOCK_REDUCE_MFMA_F16>(v);
        case DOCK_REDUCE_MFMA_BF16X3: return sum4<DOCK_REDUCE_MFMA_BF16X3>(v);
        default: return sum4<DOCK_REDUCE_SHUFFLE>(v);
    }
}

// The sum of one value, as the first component of sum4<VAR>.
template <int VAR>
__device__ __forceinline__ float sum1(float v) {
    if constexpr (VAR == DOCK_REDUCE_SHUFFLE) return wave_sum(v);
    else if constexpr (VAR == DOCK_REDUCE_MFMA_F32) {
        const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
        return mfma_tail(__builtin_amdgcn_mfma_f32_16x16x4f32(v, (lane_id() & 3) == 0 ? 1.f : 0.f, zero, 0, 0, 0)).x;
    } else return sum4<VAR>(make_float4(v, 0.f, 0.f, 0.f)).x;
}

// ---------------------------------------------------------------------------
// Ligand data held by a wave.
// ---------------------------------------------------------------------------

// Torsion transforms (3x4, row-major) and pair-force accumulators of one
// individual share memory: transform k lives until the atom positions are
// written, the accumulators from then on. The identity (transform kMaxTors)
// lies past the accumulators, so that it is written once per ligand.
template <int SLOTS>
struct __align__(16) TorsionAcc {
    static constexpr int kFirst = SLOTS > 3 * kMaxTors ? SLOTS - 3 * kMaxTors : 0;
    float4 acc[kFirst + 3 * kMaxTors];
    float4 identity[3];
    __device__ __forceinline__ float4* transforms() { return acc + kFirst; }
    __device__ __forceinline__ void write_identity(int row) {
        identity[row] = make_float4(row == 0 ? 1.f : 0.f, row == 1 ? 1.f : 0.f, row == 2 ? 1.f : 0.f, 0.f);
    }
};

// LDS of one individual. Sized per layout: SLOTS atoms per lane and WAVES
// waves per individual (a wave of the two- and four-wave layouts owns 64
// atom positions, of which past the ligand's last atom none is used, and its
// own range of accumulator copies). A ligand of at most 64 atoms has at most
// 320 accumulator slots (n_copies * stride, n_copies <= 128/N + 2).
template <int SLOTS, int WAVES = 1>
struct __align__(16) Smem {
    static constexpr int kAtoms = kWave * SLOTS * WAVES;
    static constexpr int kSlots =
        (SLOTS == 1 && WAVES == 1) ? dockblob::kMaxSlotsSmall : dockblob::kMaxSlots * WAVES;
    float4 dyn[kAtoms];             // x, y, z relative to t, and sqrt(kElec) q (depth-first
                                    // order); atom 0's place and no charge past the last atom
    TorsionAcc<kSlots> u;           // accumulator slot = (range * C + copy) * stride + atom, one
                                    // range per wave
    float4 tor[kMaxTors][2];        // torsion k: axis point p, unit axis u
    uint32_t chain[kMaxFrag][kChain / 4];  // per fragment: enclosing torsions, innermost
                                           // first, 4 per word, padded with the identity
    // several waves per individual: each wave's prefix sums of (g, x cross g)
    // at its atoms, and its {E, g} partial
    float pre[WAVES > 1 ? 6 : 1][WAVES > 1 ? kAtoms : 1];
    float4 xchg[WAVES][2];
    int unit;                       // several waves per individual: the block's work unit
};

template <int SLOTS>
struct Lig {
    // uniform
    int N, T, NF, G, n_batches, n_copies, max_depth;
    int stride;                     // accumulator stride (power of two >= N)
    int pmask;                      // stride * 16 - 1: slot byte offset -> position byte offset
    int pbits;                      // its number of bits
    int wv;                         // wave of the individual (several waves per individual), else 0
    const u32x4* plist;             // pair records (dockblob::PairRec), n_batches x 64
    // per lane, per slot: atom a = lane + 64 * (slot + wv)
    float y0[SLOTS][3];
    float chg[SLOTS][3];            // 332.06363 q, q, |q|
    int cls[SLOTS];
    int frag[SLOTS];
    int orig[SLOTS];                // original atom index
    uint32_t chain[SLOTS];          // the fragment's first four enclosing torsions
    // the torsion of this lane's gene (gene 7 + k is torsion k's angle): depth-first
    // positions of the bond atoms a, b, and of the atoms before the first and
    // at the end of the moving range, a | b << 8 | (first - 1) << 16 | (end - 1) << 24
    uint32_t torsion;
};
constexpr int kFirstTorsion = 7;    // its gene

// The packed torsion word of Lig; lanes without a torsion get harmless positions.
__device__ __forceinline__ uint32_t torsion_word(const uint8_t* blob, int T, int k) {
    if (k < 0 || k >= T) return 0;
    const Torsion& t = reinterpret_cast<const Torsion*>(blob + reinterpret_cast<const Header*>(blob)->off_tors)[k];
    return (uint32_t)t.a_pos | (uint32_t)t.b_pos << 8 | (uint32_t)(t.first - 1) << 16 | (uint32_t)(t.end - 1) << 24;
}

// First word of a fragment's chain (the rest is read from LDS where it is needed).
__device__ __forceinline__ uint32_t chain_word(const uint8_t* blob, int frag) {
    const int off = reinterpret_cast<const Header*>(blob)->off_chain;
    return reinterpret_cast<const uint32_t*>(blob + off)[frag * (kChain / 4)];
}

// Header fields and this wave's atoms (`wv`: which 64 x SLOTS of them).
template <int SLOTS, bool FOLLOW = true>
__device__ __forceinline__ void load_atoms(const uint8_t* __restrict__ blob, int wv, Lig<SLOTS>& L) {
    const Header* h = reinterpret_cast<const Header*>(blob);
    const int lane = lane_id();
    L.wv = wv;
    L.N = uniform(h->n_atoms);
    L.T = uniform(h->n_torsions);
    L.NF = uniform(h->n_frag);
    L.G = uniform(h->n_genes);
    L.n_batches = uniform(h->n_batches);
    L.n_copies = uniform(h->n_copies);
    L.max_depth = uniform(h->max_depth);
    L.stride = uniform(h->slot_stride);
    L.pmask = L.stride * 16 - 1;
    L.pbits = 31 - __builtin_clz(L.stride * 16);
    L.plist = uniform_ptr(reinterpret_cast<const u32x4*>(blob + h->off_plist));
    const float4* ref = reinterpret_cast<const float4*>(blob + h->off_ref);
    const float4* chg = reinterpret_cast<const float4*>(blob + h->off_chg);
    const int4* iv = reinterpret_cast<const int4*>(blob + h->off_int);
#pragma unroll
    for (int s = 0; s < SLOTS; ++s) {
        const int a = lane + kWave * (s + L.wv);
        const bool ok = a < L.N;
        const int ai = ok ? a : 0;
        float4 r = ref[ai], c = chg[ai];
        int4 ii = iv[ai];
        // lanes past the last atom follow atom 0 without its charge: they read
        // the map cells that it reads (at a place of their own, on plain maps,
        // a random search over 24 atoms took 155 us instead of 150), and no
        // torsion moves the root (unused pair lanes may read their positions).
        // Without FOLLOW they sit at the rotation centre: the shared evaluation,
        // on corner-expanded maps only, is faster so (500 individuals of 64 atoms
        // 6.5 us per evaluation, else 6.9; 150 of 48 2.30 and 2.32)
        const bool real = FOLLOW || ok;
        L.y0[s][0] = real ? r.x : 0.f; L.y0[s][1] = real ? r.y : 0.f; L.y0[s][2] = real ? r.z : 0.f;
        L.chg[s][0] = ok ? c.x : 0.f; L.chg[s][1] = ok ? c.y : 0.f; L.chg[s][2] = ok ? c.z : 0.f;
        L.cls[s] = ii.x;
        L.frag[s] = real ? ii.y : 0;
        L.orig[s] = ii.z;
        L.chain[s] = chain_word(blob, L.frag[s]);
    }
    L.torsion = torsion_word(blob, L.T, lane - kFirstTorsion);
}

// The LDS tables of a ligand: torsions and the identity (by the threads of the first wave) and
// fragment chains (by `threads` threads).
template <class SM>
__device__ __forceinline__ void fill_tables(const uint8_t* __restrict__ blob, SM& sm, int T, int NF, int thread,
                                            int threads) {
    const Header* h = reinterpret_cast<const Header*>(blob);
    const Torsion* tr = reinterpret_cast<const Torsion*>(blob + h->off_tors);
    if (thread < T) {
        const Torsion t = tr[thread];
        sm.tor[thread][0] = make_float4(t.p[0], t.p[1], t.p[2], 0.f);
        sm.tor[thread][1] = make_float4(t.u[0], t.u[1], t.u[2], 0.f);
    }
    if (thread < 3) sm.u.write_identity(thread);
    const uint32_t* ch = reinterpret_cast<const uint32_t*>(blob + h->off_chain);
    uint32_t* dst = &sm.chain[0][0];
    for (int i = thread; i < NF * (kChain / 4); i += threads) dst[i] = ch[i];
}

template <int SLOTS, int WAVES = 1>
__device__ void load_ligand(const uint8_t* __restrict__ blob, Smem<SLOTS, WAVES>& sm, Lig<SLOTS>& L,
                            bool fill_lds = true) {
    if (fill_lds) lds_sync<WAVES>();  // previous users of the LDS tables are done
    load_atoms<SLOTS>(blob, WAVES == 1 ? 0 : uniform((int)threadIdx.x >> 6), L);
    if (fill_lds) fill_tables(blob, sm, L.T, L.NF, WAVES == 1 ? lane_id() : (int)threadIdx.x, kWave * WAVES);
    lds_sync<WAVES>();
}

// ---------------------------------------------------------------------------
// Intermolecular grid term of one atom.
//
// The atom's world position is t + xl, with xl its position relative to the
// ligand's rotation centre. The cell is chosen from the rounded world
// coordinate, but the fraction inside the cell is taken from the exact
// difference to the cell's lower node, (t - node) + xl, summed with error
// compensation: a fraction derived from u = (x - origin)/h would carry the
// rounding of |u| (up to the grid size) into every interpolation weight.
// ---------------------------------------------------------------------------
__device__ __forceinline__ float two_sum_fraction(float t, float node, float xl) {
    const float s = t - node;
    const float bp = s - t;
    const float e1 = (t - (s - bp)) + (-node - bp);
    const float s2 = s + xl;
    const float bq = s2 - s;
    const float e2 = (s - (s2 - bq)) + (xl - bq);
    return s2 + (e1 + e2);
}

// Corner values an atom reads: v[m][4 dz + 2 dy + dx] for the atom's type map
// (m = 0), the electrostatic map (1) and the desolvation map (2). The loads
// are issued early (grid_load) and consumed later (grid_term), so that their
// latency overlaps other work.
struct GridTaps {
    float v[3][8];
    int cell[3];
};

__device__ __forceinline__ int axis_index(float t, float xl, float lo, float hi, float ih, int n) {
    // the clamped point is not below lo, so truncation is the floor (a NaN
    // converts to cell 0)
    const float xc = __builtin_amdgcn_fmed3f(t + xl, lo, hi);
    return (int)min((unsigned)((xc - lo) * ih), (unsigned)(n - 2));
}

// ANY_LAYOUT: the maps may be plain or corner-expanded (checked at run time);
// otherwise the corner-expanded copy is bound (the host makes sure), and the
// plain path is not compiled in (it costs registers).
template <bool ANY_LAYOUT>
__device__ __forceinline__ void grid_load(const GridParams& G, int cls, const float xl[3],
                                          const float t[3], GridTaps& tp) {
    const float ih = G.inv_spacing;
    const int cx = axis_index(t[0], xl[0], G.origin[0], G.hi[0], ih, G.nx);
    const int cy = axis_index(t[1], xl[1], G.origin[1], G.hi[1], ih, G.ny);
    const int cz = axis_index(t[2], xl[2], G.origin[2], G.hi[2], ih, G.nz);
    tp.cell[0] = cx;
    tp.cell[1] = cy;
    tp.cell[2] = cz;
    if (!ANY_LAYOUT || G.corners) {
        // corner-expanded maps: for the atom's type and cell, the 8 corners of
        // its type map, of the electrostatic and of the desolvation map are 96
        // contiguous bytes of a 128-byte block (one cache line), six 16-byte
        // loads instead of twelve rows (same values)
        const int ncx = G.nx - 1, ncy = G.ny - 1;
        const size_t ncell = (size_t)ncx * ncy * (G.nz - 1);
        const size_t cell = (size_t)((cz * ncy + cy) * ncx + cx);
        const auto base = gmem(reinterpret_cast<const f32x4*>(G.corners)) + ((size_t)cls * ncell + cell) * 8;
#pragma unroll
        for (int m = 0; m < 3; ++m) {
            const f32x4 a = base[2 * m], b = base[2 * m + 1];
            tp.v[m][0] = a.x; tp.v[m][1] = a.y; tp.v[m][2] = a.z; tp.v[m][3] = a.w;
            tp.v[m][4] = b.x; tp.v[m][5] = b.y; tp.v[m][6] = b.z; tp.v[m][7] = b.w;
        }
        return;
    }
    if constexpr (!ANY_LAYOUT) return;
    const int plane = G.nx * G.ny;
    const int vol = plane * G.nz;
    const int base = (cz * G.ny + cy) * G.nx + cx;
    const auto mc = gmem(G.maps + (size_t)cls * vol + base);
    const auto me = gmem(G.maps + (size_t)(G.n_maps - 2) * vol + base);
    const auto md = gmem(G.maps + (size_t)(G.n_maps - 1) * vol + base);
    const int off[8] = {0, 1, G.nx, G.nx + 1, plane, plane + 1, plane + G.nx, plane + G.nx + 1};
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        tp.v[0][i] = mc[off[i]];
        tp.v[1][i] = me[off[i]];
        tp.v[2][i] = md[off[i]];
    }
}

// Corner expansion of a grid set: eight threads per cell, thread k of a cell
// writing 16-byte word k of the cell's 128-byte block: words 2m and 2m + 1 are
// the lower and upper z corners of map m (the type map, the electrostatic, the
// desolvation map), words 6 and 7 the zero padding. A wave's store is then
// 1 KB of consecutive bytes. Each thread serves its cell for every atom type,
// so that the words of the two shared maps are read once. Bound by the writes
// (24 times the bytes read): one thread per cell, whose wave stores touch 64
// lines each, ran at 3.1 TB/s (85 us for 64^3 x 10 maps, 425 us for 96^3 x
// 12); this split takes 55 and 217 us (4.7 and 5.1 TB/s), what a plain fill of
// the same buffers takes (55 and 265 us). The stores are non-temporal: with
// plain ones the larger set, four times the memory-side cache, took 303 us.
// Every corner index stays inside the maps (cells stop one node before each
// upper face).
__global__ __launch_bounds__(256) void expand_corners_kernel(GridParams G, f32x4* __restrict__ out, int ncell) {
    const int k = threadIdx.x & 7;
    const int cell = blockIdx.x * 32 + (threadIdx.x >> 3);
    if (cell >= ncell) return;
    const int ncx = G.nx - 1, ncy = G.ny - 1;
    const int rest = cell / ncx, cx = cell - rest * ncx;
    const int cz = rest / ncy, cy = rest - cz * ncy;
    const size_t plane = (size_t)G.nx * G.ny, vol = plane * G.nz;
    const float* at = G.maps + ((size_t)(cz + (k & 1)) * G.ny + cy) * G.nx + cx;
    const int m = k >> 1;                    // 0 the type map, 1 and 2 the shared ones, 3 the padding
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if (m == 1 || m == 2) {
        const float* p = at + (size_t)(G.n_maps - 3 + m) * vol;
        v = f32x4{p[0], p[1], p[G.nx], p[G.nx + 1]};
    }
    f32x4* o = out + (size_t)cell * 8 + k;
    for (int type = 0; type < G.n_maps - 2; ++type, at += vol, o += (size_t)ncell * 8) {
        if (m == 0) v = f32x4{at[0], at[1], at[G.nx], at[G.nx + 1]};
        __builtin_nontemporal_store(v, o);
    }
}

// The atom's energy and gradient from its corner values. Poses mostly lie
// inside the box: what only atoms outside it need (the fraction of the clamped
// point, the penalty and the cut gradient) is skipped when the wave has none.
template <bool XFIRST = false>
__device__ __forceinline__ void grid_term(const GridParams& G, const GridTaps& tp, float q, float aq,
                                          const float xl[3], const float t[3],
                                          float& e, float& gx, float& gy, float& gz) {
    const float ih = G.inv_spacing;
    float f[3], out[3];
    bool in[3];
    bool all_in = true;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const float node = fmaf((float)tp.cell[c], G.spacing, G.origin[c]);
        f[c] = two_sum_fraction(t[c], node, xl[c]);
        const float xw = t[c] + xl[c];
        const float xc = __builtin_amdgcn_fmed3f(xw, G.origin[c], G.hi[c]);
        in[c] = xw == xc;
        all_in = all_in && in[c];
    }
    const bool any_out = __any(!all_in);
    if (any_out) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const float node = fmaf((float)tp.cell[c], G.spacing, G.origin[c]);
            const float xw = t[c] + xl[c];
            const float xc = __builtin_amdgcn_fmed3f(xw, G.origin[c], G.hi[c]);
            f[c] = in[c] ? f[c] : xc - node;
            out[c] = xw - xc;
        }
    }
    const float fx = f[0] * ih, fy = f[1] * ih, fz = f[2] * ih;
    float v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = fmaf(aq, tp.v[2][i], fmaf(q, tp.v[1][i], tp.v[0][i]));
    // v index = 4 dz + 2 dy + dx
    const float d00 = v[1] - v[0], d01 = v[3] - v[2], d10 = v[5] - v[4], d11 = v[7] - v[6];
    const float a00 = fmaf(d00, fx, v[0]), a01 = fmaf(d01, fx, v[2]);
    const float a10 = fmaf(d10, fx, v[4]), a11 = fmaf(d11, fx, v[6]);
    const float ey0 = a01 - a00, ey1 = a11 - a10;
    const float b0 = fmaf(fy, ey0, a00), b1 = fmaf(fy, ey1, a10);
    const float dfz = b1 - b0;
    const float dfy = fmaf(fz, ey1 - ey0, ey0);
    const float dx0 = fmaf(d01 - d00, fy, d00), dx1 = fmaf(d11 - d10, fy, d10);
    const float dfx = fmaf(fz, dx1 - dx0, dx0);
    e = fmaf(fz, dfz, b0);
    gx = dfx * ih;
    gy = dfy * ih;
    gz = dfz * ih;
    if (any_out) {
        const float o2 = XFIRST ? fmaf(out[1], out[1], out[0] * out[0]) : fmaf(out[0], out[0], out[1] * out[1]);
        e = fmaf(kOut, fmaf(out[2], out[2], o2), e);
        gx = fmaf(2.f * kOut, out[0], in[0] ? gx : 0.f);
        gy = fmaf(2.f * kOut, out[1], in[1] ? gy : 0.f);
        gz = fmaf(2.f * kOut, out[2], in[2] ? gz : 0.f);
    }
}

// ---------------------------------------------------------------------------
// One pair: energy e and w = (dE/dr)/r from the separation d = x_b - x_a.
// Both dispersion-repulsion forms are A / r^12 + B / r^m, with A = eps a
// r0^12 and B = eps b r0^m taken from the pair record: 12-6
// (a, b, m) = (1, -2, 6), 12-10 hydrogen bond (5, -6, 10); r dE/dr is
// -12 A / r^12 - m B / r^m. `live` masks pairs that are not kept (e = w = 0)
// and `slope` masks the slope where r^2 is clamped (selects, so a masked
// NaN or infinity gives 0 too). xfirst: the order in which the squares of the
// separation are added, dy^2 before dx^2 or the other way round; the callers
// fix it per pipeline step, since a different order rounds differently.
// ---------------------------------------------------------------------------

__device__ __forceinline__ void pair_term(bool xfirst, float dx, float dy, float dz, float A, float B, bool hb,
                                          float qq, float ds, bool live, float& e, float& w) {
    const float r2raw = fmaf(dz, dz, xfirst ? fmaf(dy, dy, dx * dx) : fmaf(dx, dx, dy * dy));
    const bool slope = live && (r2raw >= kR2Min);
    const float r2 = fmaxf(r2raw, kR2Min);
    const float rinv = __builtin_amdgcn_rsqf(r2);
    const float ir2 = rinv * rinv;
    const float r = r2 * rinv;
    const float i4 = ir2 * ir2;
    const float i6 = i4 * ir2;
    const float i12 = i6 * i6;
    const float im = hb ? i6 * i4 : i6;
    const float t12 = A * i12;
    const float tm = B * im;
    float elj = fmaf(i12, A, tm);
    float dlj = fmaf(hb ? -10.f : -6.f, tm, -(12.f * t12));                   // r dE/dr
    const bool capped = elj > kCap;
    elj = capped ? kCap : elj;
    dlj = capped ? 0.f : dlj;
    // Mehler-Solmajer dielectric eps(r) = A' + B' / D, D = 1 + K exp(-lambda B' r),
    // d eps / dr = lambda B'^2 K exp(-lambda B' r) / D^2. With M = D eps =
    // A' D + B' (> 0 for every r) one reciprocal q = 1 / (r D M) gives both
    // 1 / (r eps) = D^2 q and r eps' / eps = lambda B'^2 K exp(..) r^2 q.
    const float ex = __builtin_amdgcn_exp2f(-kDielLB * kLog2e * r);
    const float D = fmaf(kDielK, ex, 1.f);
    const float M = fmaf(kDielA, D, kDielB);
    const float q = __builtin_amdgcn_rcpf((r * D) * M);
    const float ired = (D * D) * q;
    const float eel = qq * ired;
    // r dE/dr = -E (1 + r eps' / eps), with this factor
    const float rel = fmaf((r2 * ex) * q, kDielBKLB, 1.f);
    // desolvation ds exp(-r^2 / (2 sigma^2)), r dE/dr = -E r^2 / sigma^2
    const float eds0 = __builtin_amdgcn_exp2f(-kDsInv2S2 * kLog2e * r2);
    const float eds = ds * eds0;
    e = live ? fmaf(ds, eds0, fmaf(qq, ired, elj)) : 0.f;
    w = slope ? fmaf(eds, r2 * -kDsInvS2, fmaf(-rel, eel, dlj)) * ir2 : 0.f;
}

// ---------------------------------------------------------------------------
// One listed pair (a packed record, see the blob layout) evaluated from the
// atom positions in LDS; the caller adds its force to the two slots.
// ---------------------------------------------------------------------------
struct PairForce {
    float w, dx, dy, dz, e;         // force on atom j is w * d, on atom i -w * d
    int si, sj;                     // byte offsets of the two accumulator slots
};

// Ends a scheduling region of two pipeline steps: their pairs are independent, so
// one's transcendentals (eight in all, whose results a lone wave would wait for) are
// set among the other's instructions, some eight apart. 600 individuals of 64 atoms
// take 7.4 us per evaluation so and 7.7 us with a region per step; 50,001 energies of
// 48 atoms 80.5 and 82.5. On two atoms per lane, which has the registers of two waves
// per SIMD, 110.0 and 108.3 (8191 genotypes of 112 atoms with gradients).
__device__ __forceinline__ void two_steps_end() {
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        __builtin_amdgcn_sched_group_barrier(0x400, 1, 0);   // a transcendental
        __builtin_amdgcn_sched_group_barrier(0x002, 8, 0);   // VALU instructions
    }
    __builtin_amdgcn_sched_barrier(0);
}

// Compile-time integer argument for the unrolled pipeline steps.
template <int V>
struct IntC { static constexpr int value = V; };

// Unused lanes (A = -0.0f) carry two slots no pair of their batch uses and
// get zero energy and force, so every lane updates its slots.
__device__ __forceinline__ PairForce pair_force(u32x4 pr, float4 pi, float4 pj, bool xfirst = false) {
    PairForce o;
    const uint32_t rec = pr.x;
    const bool valid = pr.y != dockblob::kPadC12;
    const bool hb = (int)rec < 0;
    const float dx = pj.x - pi.x, dy = pj.y - pi.y, dz = pj.z - pi.z;
    const float qq = pi.w * pj.w;           // charges pre-scaled by sqrt(kElec)
    float e, w;
    pair_term(xfirst, dx, dy, dz, __uint_as_float(pr.y), __uint_as_float(pr.z), hb, qq,
              __uint_as_float(pr.w), valid, e, w);
    o.e = e;
    o.w = w;
    o.dx = dx;
    o.dy = dy;
    o.dz = dz;
    o.si = rec & dockblob::kSlotMask;
    o.sj = (rec >> dockblob::kSlotShift) & dockblob::kSlotMask;
    return o;
}

// The pair records of a wave's batches, LANES to a row, through a buffer resource:
// a load past the last row gives zeros, whose positions may be read, so prefetches
// need no clamp. Rows are loaded in groups of four from a scalar row offset, which
// must not exceed the end (the resource's bound is checked against the rest).
template <int LANES>
struct PairRecords {
    static constexpr int kRow = LANES * (int)sizeof(u32x4);
    __amdgpu_buffer_rsrc_t rsrc;
    int lane_off;
    __device__ __forceinline__ PairRecords(const u32x4* first, int rows, int lane)
        : rsrc(__builtin_amdgcn_make_buffer_rsrc(const_cast<u32x4*>(first), 0, rows * kRow, kBufferWord3)),
          lane_off(lane * (int)sizeof(u32x4)) {}
    // row `q` (0 to 3) of the group that starts at byte `group`
    __device__ __forceinline__ u32x4 load(int group, int q) const {
        return __builtin_amdgcn_raw_buffer_load_b128(rsrc, lane_off + q * kRow, group, 0);
    }
};

// Accumulator slot at a byte offset (a multiple of 16) from `base`.
__device__ __forceinline__ float4* slot(float4* base, int byte_offset) {
    return reinterpret_cast<float4*>(
        __builtin_assume_aligned(reinterpret_cast<char*>(base) + byte_offset, 16));
}

// Adds -w d to slot si and +w d to slot sj, from their values read earlier.
// Slots are read and written whole (the fourth word passes through): 16-byte
// LDS accesses are served 16 lanes at a time, 12-byte ones take longer.
__device__ __forceinline__ void store_force(float4* base, const PairForce& f, float4 ai, float4 aj) {
    *slot(base, f.si) = make_float4(fmaf(-f.w, f.dx, ai.x), fmaf(-f.w, f.dy, ai.y), fmaf(-f.w, f.dz, ai.z), ai.w);
    *slot(base, f.sj) = make_float4(fmaf(f.w, f.dx, aj.x), fmaf(f.w, f.dy, aj.y), fmaf(f.w, f.dz, aj.z), aj.w);
}

// ---------------------------------------------------------------------------
// Rigid-body and torsion arithmetic shared by the evaluations.
// ---------------------------------------------------------------------------

// Unit quaternion of the orientation genes and its rotation matrix.
struct Rot {
    float inv;                       // 1 / |q|
    float w, x, y, z;
    float m[9];
};
__device__ __forceinline__ Rot rotation(float w0, float x0, float y0, float z0) {
    Rot r;
    r.inv = __builtin_amdgcn_rsqf(fmaf(z0, z0, fmaf(y0, y0, fmaf(w0, w0, x0 * x0))));
    r.w = w0 * r.inv; r.x = x0 * r.inv; r.y = y0 * r.inv; r.z = z0 * r.inv;
    r.m[0] = fmaf(fmaf(r.y, r.y, r.z * r.z), -2.f, 1.f);
    r.m[1] = 2.f * fmaf(r.x, r.y, -(r.w * r.z));
    r.m[2] = 2.f * fmaf(r.x, r.z, r.w * r.y);
    r.m[3] = 2.f * fmaf(r.x, r.y, r.w * r.z);
    r.m[4] = fmaf(fmaf(r.x, r.x, r.z * r.z), -2.f, 1.f);
    r.m[5] = 2.f * fmaf(r.y, r.z, -(r.w * r.x));
    r.m[6] = 2.f * fmaf(r.x, r.z, -(r.w * r.y));
    r.m[7] = 2.f * fmaf(r.y, r.z, r.w * r.x);
    r.m[8] = fmaf(fmaf(r.x, r.x, r.y * r.y), -2.f, 1.f);
    return r;
}
__device__ __forceinline__ void rotate(const Rot& R, float y0, float y1, float y2, float x[3]) {
#pragma unroll
    for (int r = 0; r < 3; ++r) x[r] = fmaf(R.m[3 * r + 2], y2, fmaf(R.m[3 * r + 1], y1, R.m[3 * r] * y0));
}

// Transform of one torsion, T(y) = R (y - p) + p about the unit axis u, as
// three rows of a 3x4 matrix.
__device__ __forceinline__ void torsion_transform(float psi, float4 p, float4 u, float4* rows) {
    float sn, cs;
    sincosf(psi, &sn, &cs);
    const float oc = 1.f - cs;
    const float ox = oc * u.x, oy = oc * u.y, oz = oc * u.z;
    const float sx = sn * u.x, sy = sn * u.y, sz = sn * u.z;
    const float R[9] = {fmaf(u.x, ox, cs), fmaf(u.y, ox, -sz), fmaf(u.z, ox, sy),
                        fmaf(u.x, oy, sz), fmaf(u.y, oy, cs), fmaf(u.z, oy, -sx),
                        fmaf(u.x, oz, -sy), fmaf(u.y, oz, sx), fmaf(u.z, oz, cs)};
    const float at[3] = {p.x, p.y, p.z};
#pragma unroll
    for (int r = 0; r < 3; ++r)
        rows[r] = make_float4(R[3 * r], R[3 * r + 1], R[3 * r + 2],
                              at[r] - fmaf(R[3 * r + 2], p.z, fmaf(R[3 * r], p.x, R[3 * r + 1] * p.y)));
}
// y <- T(y): one row is three FMAs, starting from the translation column.
__device__ __forceinline__ void apply_transform(const float4 T[3], float& y0, float& y1, float& y2) {
    const float z0 = fmaf(T[0].x, y0, fmaf(T[0].y, y1, fmaf(T[0].z, y2, T[0].w)));
    const float z1 = fmaf(T[1].x, y0, fmaf(T[1].y, y1, fmaf(T[1].z, y2, T[1].w)));
    const float z2 = fmaf(T[2].x, y0, fmaf(T[2].y, y1, fmaf(T[2].z, y2, T[2].w)));
    y0 = z0; y1 = z1; y2 = z2;
}

// Gradient with respect to a torsion angle: the axis (from atom a to atom b)
// times the torque about it, S_xg - x_a cross S_g, with S the sums of
// (g, x cross g) over the atoms the torsion moves.
__device__ __forceinline__ float torsion_gradient(const float S[6], float4 a, float4 b) {
    float ux = b.x - a.x, uy = b.y - a.y, uz = b.z - a.z;
    const float il = __builtin_amdgcn_rsqf(fmaf(uz, uz, fmaf(ux, ux, uy * uy)));
    ux *= il; uy *= il; uz *= il;
    const float mx = S[3] - fmaf(a.y, S[2], -(a.z * S[1]));
    const float my = S[4] - fmaf(a.z, S[0], -(a.x * S[2]));
    const float mz = S[5] - fmaf(a.x, S[1], -(a.y * S[0]));
    return fmaf(uz, mz, fmaf(ux, mx, uy * my));
}

// This lane's gradient component from the totals: the force E/x (EG.y .. w)
// for genes 0..2, (2/|q|) (0, tau) (x) q_hat with the torque tau for genes
// 3..6, `gt` (the torsion gradient) from gene 7 on.
__device__ __forceinline__ float gene_gradient(int gene, float4 EG, float4 TQ, const Rot& q, float gt) {
    const float k2 = 2.0f * q.inv;
    const float gw = -fmaf(TQ.z, q.z, fmaf(TQ.x, q.x, TQ.y * q.y));
    const float gx = fmaf(q.w, TQ.x, fmaf(TQ.y, q.z, -(TQ.z * q.y)));
    const float gy = fmaf(q.w, TQ.y, fmaf(TQ.z, q.x, -(TQ.x * q.z)));
    const float gz = fmaf(q.w, TQ.z, fmaf(TQ.x, q.y, -(TQ.y * q.x)));
    float gr = gt;
    gr = gene == 0 ? EG.y : gr;
    gr = gene == 1 ? EG.z : gr;
    gr = gene == 2 ? EG.w : gr;
    gr = gene == 3 ? k2 * gw : gr;
    gr = gene == 4 ? k2 * gx : gr;
    gr = gene == 5 ? k2 * gy : gr;
    gr = gene == 6 ? k2 * gz : gr;
    return gr;
}

// One ADADELTA step of a gene: running means of g^2 and dx^2, and the new
// position (Zeiler 2012, Alg. 1).
__device__ __forceinline__ float adadelta(float x, float gr, float rho, float eps, float& ag, float& ad) {
    const float keep = 1.f - rho;
    ag = fmaf(rho, ag, (keep * gr) * gr);
    const float rate = -(__builtin_amdgcn_sqrtf(ad + eps) * __builtin_amdgcn_rsqf(ag + eps));
    const float dx = rate * gr;
    ad = fmaf(rho, ad, (keep * dx) * dx);
    return fmaf(rate, gr, x);
}

// Applies the torsions that enclose an atom, innermost first: `first` holds the
// four innermost, `row` all, four to a word; the transforms are read LEVELS at a
// time. Levels past the atom's depth apply the identity, so every lane takes the
// same (uniform) number of LDS round trips. Up to four levels need no read of the
// row, which a lone wave would wait for.
template <int LEVELS>
__device__ __forceinline__ void apply_chain(uint32_t first, const uint32_t* row, const float4* transforms, int max_depth,
                                            float& y0, float& y1, float& y2) {
    static_assert(LEVELS == 2 || LEVELS == 4, "a chain word holds four levels");
    uint32_t w = first;
    for (int d = 0; d < max_depth; d += LEVELS) {
        if (d >= 4 && d % 4 == 0) w = row[d >> 2];
        float4 T[LEVELS][3];
#pragma unroll
        for (int q = 0; q < LEVELS; ++q) {
            const unsigned k = (w >> (8 * q)) & 255u;
            const float4* t = reinterpret_cast<const float4*>(__builtin_assume_aligned(
                reinterpret_cast<const char*>(transforms) + __umul24(k, 48u), 16));
            T[q][0] = t[0]; T[q][1] = t[1]; T[q][2] = t[2];
        }
#pragma unroll
        for (int q = 0; q < LEVELS; ++q) apply_transform(T[q], y0, y1, y2);
        if constexpr (LEVELS == 2) w >>= 16;
    }
}

// Rigid body (rotation and translation) and torsion transforms of the individual
// whose genes this wave holds; the transforms are left in LDS.
template <int WAVES, class SM, class LIG>
__device__ __forceinline__ void transforms_of(SM& sm, const LIG& L, float gene, Rot& Rq, float tv[3]) {
    const bool lead = WAVES == 1 || L.wv == 0;  // the wave that writes shared tables
    // rigid-body genes (uniform)
    const float tx = readlane(gene, 0), ty = readlane(gene, 1), tz = readlane(gene, 2);
    const float qw0 = readlane(gene, 3), qx0 = readlane(gene, 4), qy0 = readlane(gene, 5),
                qz0 = readlane(gene, 6);
    Rq = rotation(qw0, qx0, qy0, qz0);

    // torsion transforms: T_k(y) = R_k (y - p) + p, about the reference axis, by
    // the lane that holds the angle
    const int k = lane_id() - kFirstTorsion;
    if (lead && k >= 0 && k < L.T) {
        torsion_transform(gene, sm.tor[k][0], sm.tor[k][1], sm.u.transforms() + 3 * k);
    }
    tv[0] = tx; tv[1] = ty; tv[2] = tz;
    lds_sync<WAVES>();
}

// Atom positions from the rigid body and the transforms in LDS: relative to the
// translation, in registers (x) and in the LDS position table.
template <int SLOTS, int WAVES, int LEVELS = 2, class SM>
__device__ __forceinline__ void place_atoms(SM& sm, const Lig<SLOTS>& L, const Rot& Rq, float x[SLOTS][3]) {
    const int lane = lane_id();
    // atom positions relative to the rotation centre: the torsions enclosing
    // the atom's fragment, innermost first (each about its reference axis,
    // which no inner torsion moves), then the rotation Rq. The translation t
    // is added only where world coordinates are needed (the grid term): pair
    // separations, torques and torsion axes are translation invariant and
    // keep the precision of the small local coordinates.
#pragma unroll
    for (int s = 0; s < SLOTS; ++s) {
        const int a = lane + kWave * (s + L.wv);
        float y0 = L.y0[s][0], y1 = L.y0[s][1], y2 = L.y0[s][2];
        apply_chain<LEVELS>(L.chain[s], sm.chain[L.frag[s]], sm.u.transforms(), L.max_depth, y0, y1, y2);
        rotate(Rq, y0, y1, y2, x[s]);
        sm.dyn[a] = make_float4(x[s][0], x[s][1], x[s][2], kSqrtElec * L.chg[s][1]);
    }
    lds_sync<WAVES>();
}

// The rigid bodies and torsion transforms of several genotypes, made at once: a
// genotype takes T + 1 of the lanes, one per torsion and one for the rigid body,
// and holds them until its turn. A wave whose next genotypes are known so spends
// the 140 instructions, of which a genotype alone uses a few lanes, once for
// 64 / (T + 1) of them. Used where instructions bound the kernel: energies of 50,001
// genotypes take 85.1 us with a pose each, 82.6 so (48 atoms), 40.0 and 36.3 (24
// atoms). With gradients, or two genotypes per wave, the LDS unit is as busy as the
// VALU, and the reads of the rigid body cost what the instructions save (24 atoms
// two per wave 57.2 and 57.0 us, 112 atoms 108.2 and 109.7).
struct PoseGroup {
    static constexpr int kRigid = 5;   // float4s of a rigid body in LDS
    int size;                   // genotypes
    int mine, part;             // this lane's genotype, and its torsion or (T) the rigid body
    int T;
    float4 row[3], more;        // transform; or rotation rows with 1/|q|, w, x and y, z, t.x, t.y
    float last;                 // t.z

    __device__ __forceinline__ PoseGroup(int torsions, int lane) : T(torsions) {
        size = kWave / (torsions + 1);
        mine = lane / (torsions + 1);
        part = lane - mine * (torsions + 1);
    }
    // `genes`: this lane's genotype; not read unless `live`
    __device__ __forceinline__ void make(const float4 (*tor)[2], const float* genes, bool live) {
        if (!live) return;
        if (part < T) {
            torsion_transform(genes[kFirstTorsion + part], tor[part][0], tor[part][1], row);
        } else {
            const Rot R = rotation(genes[3], genes[4], genes[5], genes[6]);
            row[0] = make_float4(R.m[0], R.m[1], R.m[2], R.inv);
            row[1] = make_float4(R.m[3], R.m[4], R.m[5], R.w);
            row[2] = make_float4(R.m[6], R.m[7], R.m[8], R.x);
            more = make_float4(R.y, R.z, genes[0], genes[1]);
            last = genes[2];
        }
    }
    // genotype q's transforms and rigid body to their places in LDS
    __device__ __forceinline__ void store(int q, float4* transforms, float4* rigid) const {
        if (mine != q) return;
        float4* const to = part < T ? transforms + 3 * part : rigid;
        to[0] = row[0]; to[1] = row[1]; to[2] = row[2];
        if (part == T) {
            rigid[3] = more;
            rigid[4].x = last;
        }
    }
    static __device__ __forceinline__ void load(const float4* rigid, Rot& R, float tv[3]) {
        const float4 a = rigid[0], b = rigid[1], c = rigid[2], d = rigid[3];
        R.m[0] = a.x; R.m[1] = a.y; R.m[2] = a.z;
        R.m[3] = b.x; R.m[4] = b.y; R.m[5] = b.z;
        R.m[6] = c.x; R.m[7] = c.y; R.m[8] = c.z;
        R.inv = a.w; R.w = b.w; R.x = c.w; R.y = d.x; R.z = d.y;
        tv[0] = d.z; tv[1] = d.w; tv[2] = rigid[4].x;
    }
};

// Sum of an atom's `n` accumulator copies, `stride` slots apart, in copy order;
// four reads in flight at a time.
__device__ __forceinline__ void sum_copies(const float4* acc, int n, int stride, float g[3]) {
    g[0] = g[1] = g[2] = 0.f;
    int c = 0;
    for (; c + 4 <= n; c += 4, acc += 4 * stride) {
        float4 v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = acc[k * stride];
#pragma unroll
        for (int k = 0; k < 4; ++k) { g[0] += v[k].x; g[1] += v[k].y; g[2] += v[k].z; }
    }
    for (; c < n; ++c, acc += stride) {
        const float4 v = *acc;
        g[0] += v.x; g[1] += v.y; g[2] += v.z;
    }
}

// Energy and this lane's gradient component from the per-atom gradients `g`
// and the lane energies; `sum` is the block sum of 4-vectors.
template <int SLOTS, int WAVES, class SM, class SUM>
__device__ __forceinline__ float finish(SM& sm, const Lig<SLOTS>& L, const Rot& Rq, const float x[SLOTS][3],
                                        const float g[SLOTS][3], float e_lane, SUM&& sum, float& grad) {
    const int lane = lane_id();
    // this lane's torsion: positions of its bond atoms, read ahead of the sums
    const float4 bond_a = sm.dyn[L.torsion & 255], bond_b = sm.dyn[(L.torsion >> 8) & 255];
    // block sum of {E, gx, gy, gz}: the paper's reduction, in the chosen variant
    float4 eg = make_float4(e_lane, g[0][0], g[0][1], g[0][2]);
    if constexpr (SLOTS == 2) { eg.y += g[1][0]; eg.z += g[1][1]; eg.w += g[1][2]; }
    float4 EG = sum(eg);

    // torsion torques: prefix sums of (g, x cross g) in depth-first order;
    // the last lane's x cross g sums give the torque about t (FP32 always)
    float P[SLOTS][6];
#pragma unroll
    for (int s = 0; s < SLOTS; ++s) {
        P[s][0] = g[s][0]; P[s][1] = g[s][1]; P[s][2] = g[s][2];
        P[s][3] = fmaf(x[s][1], g[s][2], -(x[s][2] * g[s][1]));
        P[s][4] = fmaf(x[s][2], g[s][0], -(x[s][0] * g[s][2]));
        P[s][5] = fmaf(x[s][0], g[s][1], -(x[s][1] * g[s][0]));
    }
    wave_scan6(P[0]);
    if constexpr (SLOTS == 2) {
        wave_scan6(P[1]);
#pragma unroll
        for (int c = 0; c < 6; ++c) P[1][c] += readlane(P[0][c], 63);
    }
    float4 TQ = make_float4(readlane(P[SLOTS - 1][3], 63), readlane(P[SLOTS - 1][4], 63),
                            readlane(P[SLOTS - 1][5], 63), 0.f);
    if constexpr (WAVES > 1) {
        // the waves' partials and prefix sums meet in LDS; every wave then
        // holds the same totals (added in wave order) and steps identically
        const int a = lane + kWave * L.wv;
#pragma unroll
        for (int c = 0; c < 6; ++c) sm.pre[c][a] = P[0][c];
        if (lane == 0) sm.xchg[L.wv][0] = EG;
        lds_sync<WAVES>();
        EG = sm.xchg[0][0];
        TQ = make_float4(sm.pre[3][kWave - 1], sm.pre[4][kWave - 1], sm.pre[5][kWave - 1], 0.f);
#pragma unroll
        for (int w = 1; w < WAVES; ++w) {
            const float4 ew = sm.xchg[w][0];
            EG = make_float4(EG.x + ew.x, EG.y + ew.y, EG.z + ew.z, EG.w + ew.w);
            TQ = make_float4(TQ.x + sm.pre[3][(w + 1) * kWave - 1], TQ.y + sm.pre[4][(w + 1) * kWave - 1],
                             TQ.z + sm.pre[5][(w + 1) * kWave - 1], 0.f);
        }
    }
    // sums over the atoms this lane's torsion moves: differences of the prefix
    // sums at the end of the range and before its start
    float S[6];
#pragma unroll
    for (int c = 0; c < 6; ++c) {
        if constexpr (WAVES > 1) {
            // global prefix: a wave's local prefix plus the totals of the
            // waves before it (added in wave order)
            const int hi = L.torsion >> 24, lo = (L.torsion >> 16) & 255;
            const float bh = sm.pre[c][hi], bl = sm.pre[c][lo];
            float ph = bh, pl = bl, off = 0.f;
#pragma unroll
            for (int w = 1; w < WAVES; ++w) {
                off = w == 1 ? sm.pre[c][kWave - 1] : off + sm.pre[c][w * kWave - 1];
                ph = hi >= w * kWave ? bh + off : ph;
                pl = lo >= w * kWave ? bl + off : pl;
            }
            S[c] = ph - pl;
        } else {
            float ph = lane_at(P[0][c], L.torsion >> 24), pl = lane_at(P[0][c], L.torsion >> 16);
            if constexpr (SLOTS == 2) {
                const float ph1 = lane_at(P[1][c], L.torsion >> 24), pl1 = lane_at(P[1][c], L.torsion >> 16);
                ph = (L.torsion >> 24) >= kWave ? ph1 : ph;
                pl = ((L.torsion >> 16) & 255) >= kWave ? pl1 : pl;
            }
            S[c] = ph - pl;
        }
    }
    grad = gene_gradient(lane, EG, TQ, Rq, torsion_gradient(S, bond_a, bond_b));
    return EG.x;
}

// ---------------------------------------------------------------------------
// One evaluation of E and dE/dgenotype by this wave, of the individual whose
// transforms `prepare` leaves in LDS and whose rigid body it gives; returns E
// (uniform) and writes this lane's gradient component to `grad`.
// ---------------------------------------------------------------------------
template <int SLOTS, int VAR, int WAVES, bool ANY_LAYOUT, bool GRAD, bool TRIAL, class PREPARE>
__device__ __forceinline__ float evaluate_prepared(const GridParams& G, Smem<SLOTS, WAVES>& sm, const Lig<SLOTS>& L,
                                                   PREPARE&& prepare, float& grad, float* atom_out,
                                                   int var = VAR) {
    const int lane = lane_id();
    const int N = L.N;
    // this wave's batches, the first four of which are loaded ahead of the pose (a
    // lone wave waited 500 of 11,600 cycles for them: with that, the chain words in
    // registers and no clamps 3000 individuals of 48 atoms take 2,323 us for 301
    // evaluations instead of 2,385, 50,001 energies 84.8 instead of 89.0; with several waves per
    // individual, wave w takes the w-th of WAVES consecutive runs of
    // ceil(n_batches / WAVES) batches, the last of which may be short or empty)
    const int run = (L.n_batches + WAVES - 1) / WAVES;
    const int b0 = WAVES == 1 ? 0 : min(L.wv * run, L.n_batches);
    const int nb = WAVES == 1 ? L.n_batches : min(L.n_batches - b0, run);
    using Records = PairRecords<kWave>;
    const Records records(L.plist + b0 * kWave, nb, lane);
    u32x4 R[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) R[q] = records.load(0, q);

    Rot Rq;
    float tv[3], x[SLOTS][3];
    prepare(Rq, tv);
    place_atoms<SLOTS, WAVES>(sm, L, Rq, x);

    float g[SLOTS][3];
    float e_lane = 0.f;
    GridTaps tap[SLOTS];

    // pair terms: batches of 64 listed pairs, one per lane. Each lane adds
    // its pair's force to both atoms' accumulator slots; the host schedule
    // makes the slots of one batch distinct, so no two lanes of an
    // instruction touch one address and the order of additions is fixed.
    // (LDS float atomics would serialise in the LDS unit: they made this
    // phase several times slower.)
    if constexpr (!GRAD) {
        // energies only (a search that needs no gradient): each lane sums its
        // pairs' energies from the positions, in batch order; no
        // accumulators, no force. Software pipeline: step k reads the
        // positions of batch k + 1 from LDS before computing batch k, and
        // loads the record of batch k + 4 (records live four steps, positions
        // two; register sets indexed by k mod 4 and mod 2, steps unrolled by
        // four).
        static_assert(WAVES == 1, "the energy-only evaluation is one wave per individual");
        const int pmask = L.pmask;
        auto pos_i = [&](uint32_t w) { return *slot(sm.dyn, w & pmask); };
        auto pos_j = [&](uint32_t w) { return *slot(sm.dyn, __builtin_amdgcn_ubfe(w, dockblob::kSlotShift, L.pbits)); };
        if (nb > 0) {
            float4 Pi[2], Pj[2];
            Pi[0] = pos_i(R[0].x);
            Pj[0] = pos_j(R[0].x);
            int k = 0;
            int group = 4 * Records::kRow;    // the rows of batches k + 4 to k + 7, k mod 4 = 0
            auto step = [&](auto residue, auto load) {
                constexpr int r = decltype(residue)::value;  // k mod 4
                constexpr int c = r & 1, n = (r + 1) & 1;
                const u32x4 rn = R[(r + 1) & 3];
                Pi[n] = pos_i(rn.x);
                Pj[n] = pos_j(rn.x);
                if constexpr (r % 2 == 0) __builtin_amdgcn_sched_barrier(0);   // keep the reads at the start
                constexpr bool last = decltype(load)::value == 0;
                constexpr bool xfirst = (TRIAL && r == 0) || (last && r == 2);
                e_lane += pair_force(R[r], Pi[c], Pj[c], xfirst).e;
                if constexpr (decltype(load)::value != 0) R[r] = records.load(group, r);
                if constexpr (r % 2 == 1) two_steps_end();
                ++k;
            };
            using I0 = IntC<0>;
            using I1 = IntC<1>;
            using I2 = IntC<2>;
            using I3 = IntC<3>;
            using Load = IntC<1>;
            using NoLoad = IntC<0>;
            for (; k + (TRIAL ? 4 : 5) <= nb; group += 4 * Records::kRow) {
                step(I0(), Load()); step(I1(), Load()); step(I2(), Load()); step(I3(), Load());
            }
            // the grid-map loads follow the last record load (global loads
            // complete in order)
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int s = 0; s < SLOTS; ++s) grid_load<ANY_LAYOUT>(G, L.cls[s], x[s], tv, tap[s]);
            __builtin_amdgcn_sched_barrier(0);
            if (k < nb) step(I0(), NoLoad());
            if (k < nb) step(I1(), NoLoad());
            if (k < nb) step(I2(), NoLoad());
            if constexpr (!TRIAL) if (k < nb) step(I3(), NoLoad());
        } else {
#pragma unroll
            for (int s = 0; s < SLOTS; ++s) grid_load<ANY_LAYOUT>(G, L.cls[s], x[s], tv, tap[s]);
        }
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) g[s][0] = g[s][1] = g[s][2] = 0.f;
    } else {
        // each wave adds into its own range of copies
        const int nslot = L.n_copies * L.stride;
        float4* const accw = sm.u.acc + (WAVES == 1 ? 0 : L.wv * nslot);
        // cleared by whole waves of slots (the array holds a multiple of 64;
        // a wave's last store may clear slots of the next wave's range, which
        // nobody has added to yet)
        static_assert(Smem<SLOTS, WAVES>::kSlots % kWave == 0, "clearing stays inside the accumulators");
        for (int k = 0; k < nslot; k += kWave) accw[k + lane] = make_float4(0.f, 0.f, 0.f, 0.f);
        lds_sync<WAVES>();
        const int pmask = L.pmask;
        // an atom's position sits at its slot's byte offset masked to one stride
        auto pos_i = [&](uint32_t w) { return *slot(sm.dyn, w & pmask); };
        auto pos_j = [&](uint32_t w) { return *slot(sm.dyn, __builtin_amdgcn_ubfe(w, dockblob::kSlotShift, L.pbits)); };
        // Software pipeline over batches with no branch inside. Step k
        // stores batch k (its slot values were read in step k - 1) and
        // computes batch k + 1 while reading the positions of batch k + 2
        // and loading the record of batch k + 4. A record lives four steps
        // and positions, forces and slot values two, so the steps are
        // unrolled by four with register sets indexed by the batch number
        // mod 4 and mod 2: no loaded value is copied between steps. Slot
        // updates stay in batch order (LDS executes a wave's accesses in
        // order: batch k's stores precede batch k + 1's loads).
        if (nb > 0) {
            // steps scheduled two by two, but for the layouts that gain nothing from it
            constexpr bool kPairs = SLOTS == 1 && WAVES == 1;
            float4 Pi[2], Pj[2], Ai[2], Aj[2];
            PairForce F[2];
            // the prologue issues its LDS reads in the loop's order (positions
            // of the next batch before the slots of this one), so that at the
            // loop head the slot reads may still be in flight
            Pi[0] = pos_i(R[0].x);
            Pj[0] = pos_j(R[0].x);
            Pi[1] = pos_i(R[1].x);
            Pj[1] = pos_j(R[1].x);
            F[0] = pair_force(R[0], Pi[0], Pj[0]);
            Ai[0] = *slot(accw, F[0].si);
            Aj[0] = *slot(accw, F[0].sj);
            int k = 0;
            int group = 4 * Records::kRow;
            auto step = [&](auto residue, auto load) {
                constexpr int r = decltype(residue)::value;  // k mod 4
                constexpr int c = r & 1, n = (r + 1) & 1;
                const u32x4 rf = R[(r + 2) & 3];
                Pi[c] = pos_i(rf.x);
                Pj[c] = pos_j(rf.x);
                if constexpr (decltype(load)::value != 0) R[r] = records.load(group, r);
                if constexpr (!kPairs || r % 2 == 0) __builtin_amdgcn_sched_barrier(0);   // keep the loads at the start
                F[n] = pair_force(R[(r + 1) & 3], Pi[n], Pj[n], r == 1 && decltype(load)::value == 0);
                store_force(accw, F[c], Ai[c], Aj[c]);
                e_lane += F[c].e;
                Ai[n] = *slot(accw, F[n].si);
                Aj[n] = *slot(accw, F[n].sj);
                if constexpr (!kPairs) __builtin_amdgcn_sched_barrier(0);
                else if constexpr (r % 2 == 1) two_steps_end();
                ++k;
            };
            using I0 = IntC<0>;
            using I1 = IntC<1>;
            using I2 = IntC<2>;
            using I3 = IntC<3>;
            using Load = IntC<1>;
            using NoLoad = IntC<0>;
            for (; k + 4 < nb; group += 4 * Records::kRow) {
                step(I0(), Load()); step(I1(), Load()); step(I2(), Load()); step(I3(), Load());
            }
            // Every record the remaining steps need is loaded. The grid-map
            // loads go here, after the last record load: global loads
            // complete in order, so a record load issued after them would
            // wait for them. They are consumed after the pair phase.
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int s = 0; s < SLOTS; ++s) grid_load<ANY_LAYOUT>(G, L.cls[s], x[s], tv, tap[s]);
            __builtin_amdgcn_sched_barrier(0);
            if (k < nb - 1) step(I0(), NoLoad());
            if (k < nb - 1) step(I1(), NoLoad());
            if (k < nb - 1) step(I2(), NoLoad());
            // k == nb - 1: the last batch is computed and its slots read
            if (k & 1) {
                store_force(accw, F[1], Ai[1], Aj[1]);
                e_lane += F[1].e;
            } else {
                store_force(accw, F[0], Ai[0], Aj[0]);
                e_lane += F[0].e;
            }
        } else {
#pragma unroll
            for (int s = 0; s < SLOTS; ++s) grid_load<ANY_LAYOUT>(G, L.cls[s], x[s], tv, tap[s]);
        }
        lds_sync<WAVES>();
        // each atom adds its copies in copy order (range by range)
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
            const int a = lane + kWave * (s + L.wv);
            g[s][0] = g[s][1] = g[s][2] = 0.f;
            if (a < N) sum_copies(sm.u.acc + a, L.n_copies * WAVES, L.stride, g[s]);
        }
    }
    // grid term, from the corner values loaded before the pair phase
    float e_atom[SLOTS];
#pragma unroll
    for (int s = 0; s < SLOTS; ++s) {
        const int a = lane + kWave * (s + L.wv);
        float e, gx, gy, gz;
        grid_term<TRIAL>(G, tap[s], L.chg[s][1], L.chg[s][2], x[s], tv, e, gx, gy, gz);
        const bool ok = a < N;
        e_atom[s] = ok ? e : 0.f;
        g[s][0] += ok ? gx : 0.f;
        g[s][1] += ok ? gy : 0.f;
        g[s][2] += ok ? gz : 0.f;
        e_lane += e_atom[s];
    }
    if constexpr (!GRAD) {
        // the block sum of E alone, in the chosen variant
        grad = 0.f;
        lds_sync<WAVES>();   // the next evaluation rewrites the position table
        return sum1<VAR>(e_lane);
    }

    const float E = finish<SLOTS, WAVES>(sm, L, Rq, x, g, e_lane, [var](float4 v) {
        if constexpr (VAR >= 0) return sum4<VAR>(v);
        else return sum4_of(var, v);
    }, grad);
    if (atom_out) {
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
            const int a = lane + kWave * (s + L.wv);
            if (a < N) {
                float4* o = reinterpret_cast<float4*>(atom_out) + 2 * L.orig[s];
                // position relative to t, as held (t + it is the world position)
                o[0] = make_float4(x[s][0], x[s][1], x[s][2], e_atom[s]);
                o[1] = make_float4(g[s][0], g[s][1], g[s][2], 0.f);
            }
        }
    }
    return E;
}

// The same for the individual whose gene `lane` is `gene` (lanes >= G ignored).
template <int SLOTS, int VAR, int WAVES = 1, bool ANY_LAYOUT = true, bool GRAD = true, bool TRIAL = false>
__device__ float evaluate(const GridParams& G, Smem<SLOTS, WAVES>& sm, const Lig<SLOTS>& L, float gene,
                          float& grad, float* atom_out, int var = VAR) {
    return evaluate_prepared<SLOTS, VAR, WAVES, ANY_LAYOUT, GRAD, TRIAL>(
        G, sm, L, [&](Rot& Rq, float tv[3]) { transforms_of<WAVES>(sm, L, gene, Rq, tv); }, grad, atom_out, var);
}

// ---------------------------------------------------------------------------
// Kernels.
// ---------------------------------------------------------------------------

// Persistent scoring kernel: each wave loads the ligand once (LDS tables and
// per-lane registers) and evaluates genotypes ind = blockIdx.x,
// blockIdx.x + gridDim.x, ... (independent evaluations, so a static stride
// gives the same results as any other assignment). ANY_LAYOUT: the maps may
// be plain or corner-expanded; otherwise the corner-expanded copy is bound.
// GRAD = false, for calls that ask for neither a gradient nor the per-atom
// output: the energy-only evaluation, same energies bit for bit. It is bound
// by VALU issue like the full one but issues 0.6 of its instructions, and within
// 128 registers four waves fit a SIMD instead of three: 50,001 genotypes
// of a 48-atom ligand took 139 us with the gradient made and dropped, 90 us so
// (80 with what came since); 65,536 of a 24-atom one 100 and 52 us, two per wave
// 65 and 40 us.
template <int SLOTS, int VAR, bool ANY_LAYOUT, bool GRAD>
__global__ __launch_bounds__(64, (SLOTS == 1 ? 3 : 2) + (GRAD ? 0 : 1)) void score_kernel(
    GridParams G, const uint8_t* __restrict__ blob, int n, const float* __restrict__ gen, float* __restrict__ energy,
    float* __restrict__ grad, float* __restrict__ atom_out) {
    __shared__ Smem<SLOTS> sm;
    Lig<SLOTS> L;
    load_ligand<SLOTS>(blob, sm, L);
    const int lane = lane_id();
    const int G_ = L.G;
    if constexpr (SLOTS == 1 && !GRAD) {
        // the poses of as many of the wave's genotypes as its lanes hold, made at once
        __shared__ float4 rigid[PoseGroup::kRigid];
        PoseGroup group(L.T, lane);
        int q = group.size;
        for (long long ind = blockIdx.x; ind < n; ind += gridDim.x, ++q) {
            if (q == group.size) {
                q = 0;
                const long long row = ind + (long long)group.mine * gridDim.x;
                group.make(sm.tor, gen + row * G_, group.mine < group.size && row < n);
            }
            float gr;
            const float E = evaluate_prepared<SLOTS, VAR, 1, ANY_LAYOUT, GRAD, false>(
                G, sm, L,
                [&](Rot& Rq, float tv[3]) {
                    group.store(q, sm.u.transforms(), rigid);
                    wave_sync();
                    group.load(rigid, Rq, tv);
                },
                gr, nullptr);
            if (lane == 0) energy[ind] = E;
        }
    } else {
        for (int ind = blockIdx.x; ind < n; ind += gridDim.x) {
            const float gene = lane < G_ ? gen[(size_t)ind * G_ + lane] : 0.f;
            float gr;
            float* ao = GRAD && atom_out ? atom_out + (size_t)ind * L.N * 8 : nullptr;
            const float E = evaluate<SLOTS, VAR, 1, ANY_LAYOUT, GRAD>(G, sm, L, gene, gr, ao);
            if (lane == 0) energy[ind] = E;
            if (GRAD && grad && lane < G_) grad[(size_t)ind * G_ + lane] = gr;
        }
    }
}

// Solis-Wets random search (Sec. 2.1: the LGA's second local search; the
// steps are those of Solis and Wets as AutoDock uses them): per iteration the
// trial x + bias + dev, else x - bias - dev, accepted when its energy is lower;
// bias and the step scale rho follow the outcome. One wave per individual,
// gene `lane`; energies only.
// State updates are float32 in a fixed order with no fused operations. Bound by
// VALU issue (1,540 instructions per iteration of a 48-atom ligand), which fills 80 %
// of the launch: of the 2.9 waves that each SIMD gets, 2.1 are there on average
// (trials per individual differ by 6 % at most, so it is not their number): 3000
// individuals, 100 iterations 1,023 us with the full evaluation's layout checks
// and normals read where they are used, 977 once the evaluation waited less, 963
// with a kernel for the corner-expanded maps and the normals an iteration ahead.
template <int SLOTS, int VAR, bool ANY_LAYOUT>
__global__ __launch_bounds__(64, (SLOTS == 1 ? 3 : 2)) void sw_kernel(GridParams G, const uint8_t* __restrict__ blob,
                                                docklaunch::SwParams p) {
    __shared__ Smem<SLOTS> sm;
    Lig<SLOTS> L;
    load_ligand<SLOTS>(blob, sm, L);
    const int lane = lane_id();
    const int ind = blockIdx.x;
    if (ind >= p.n) return;
    const int Gn = L.G;
    const bool on = lane < Gn;
    const size_t row = (size_t)ind * Gn + lane;
    float x = on ? p.genotype[row] : 0.f;
    float b = on ? p.bias[row] : 0.f;
    const float sc = on ? p.scale[lane] : 0.f;
    float E = p.energy[ind];
    float rho = p.rho[ind];
    int succ = p.counts[2 * ind], fail = p.counts[2 * ind + 1];
    // the next iteration's normals are read an iteration ahead
    auto normal = [&](int it) {
        return on && it < p.iterations ? p.normals[((size_t)it * p.n + ind) * Gn + lane] : 0.f;
    };
    float z_next = normal(0);
    for (int it = 0; it < p.iterations; ++it) {
        const float z = z_next;
        z_next = normal(it + 1);
        const float dev = rho * (sc * z);
        float e_try0 = __builtin_nanf(""), e_try1 = __builtin_nanf("");
        int accepted = -1;
        for (int t = 0; t < 2; ++t) {      // uniform: E and the trial energies are wave-uniform
            const float c = t == 0 ? (x + b) + dev : (x - b) - dev;
            float gr;
            const float Et = evaluate<SLOTS, VAR, 1, ANY_LAYOUT, false, true>(G, sm, L, c, gr, nullptr);
            if (t == 0) e_try0 = Et; else e_try1 = Et;
            if (Et < E) {
                x = c;
                E = Et;
                accepted = t;
                break;
            }
        }
        if (accepted == 0) {
            b = 0.2f * b + 0.4f * dev;
            ++succ;
            fail = 0;
        } else if (accepted == 1) {
            b = b - 0.4f * dev;
            ++succ;
            fail = 0;
        } else {
            b = 0.5f * b;
            ++fail;
            succ = 0;
        }
        if (succ >= p.n_success) {
            rho = 2.f * rho;
            succ = 0;
        } else if (fail >= p.n_failure) {
            rho = 0.5f * rho;
            fail = 0;
        }
        if (p.log && lane == 0) {
            p.log[((size_t)ind * p.iterations + it) * 2] = e_try0;
            p.log[((size_t)ind * p.iterations + it) * 2 + 1] = e_try1;
        }
    }
    if (on) {
        p.genotype[row] = x;
        p.bias[row] = b;
    }
    if (lane == 0) {
        p.energy[ind] = E;
        p.rho[ind] = rho;
        p.counts[2 * ind] = succ;
        p.counts[2 * ind + 1] = fail;
    }
}

// ADADELTA search of individual `ind` by one wave, gene `lane`; `eval` returns
// E and the gradient component at the current point. With several waves per
// individual that hold the genotype all take the same steps on the same
// totals, and the `writer` writes the results.
template <class EVAL>
__device__ __forceinline__ void search(const DevItem& it, int ind, int G, int iterations, float rho, float eps,
                                       bool final_eval, bool writer, EVAL&& eval) {
    const int lane = lane_id();
    const bool act = lane < G;
    const size_t o = (size_t)ind * G + lane;
    float x = act ? it.genotype[o] : 0.f;
    float ag = act ? it.acc_g2[o] : 0.f;
    float ad = act ? it.acc_dx2[o] : 0.f;
    float bx = act ? it.best_genotype[o] : 0.f;
    float bestE = it.best_energy[ind];
    float lastE = it.energy[ind];
    float lastG = 0.f;
    // the final evaluation, if asked for, is one more pass without a step
    const int passes = iterations + (final_eval ? 1 : 0);
    for (int pass = 0; pass < passes; ++pass) {
        float gr;
        const float E = eval(x, gr);
        lastE = E;
        lastG = gr;
        if (E < bestE) { bestE = E; bx = x; }
        if (pass == iterations) break;
        gr = act ? gr : 0.f;
        float xn = adadelta(x, gr, rho, eps, ag, ad);
        const bool isq = lane >= 3 && lane < 7;
        const float q2 = isq ? xn * xn : 0.f;
        // genes 3..6 share the first row; the other rows' lanes discard it
        const float nq2 = (row_lane<3>(q2) + row_lane<4>(q2)) + (row_lane<5>(q2) + row_lane<6>(q2));
        if (isq) xn = (nq2 >= 1e-12f) ? xn * __builtin_amdgcn_rsqf(nq2) : x;
        x = act ? xn : 0.f;
    }
    if (!writer) return;
    if (act && it.grad && (iterations > 0 || final_eval)) it.grad[o] = lastG;
    if (act) {
        it.genotype[o] = x;
        it.acc_g2[o] = ag;
        it.acc_dx2[o] = ad;
        it.best_genotype[o] = bx;
    }
    if (lane == 0) {
        it.best_energy[ind] = bestE;
        it.energy[ind] = lastE;
        it.iters_done[ind] += iterations;
    }
}

template <int SLOTS, int VAR, int WAVES = 1, bool ANY_LAYOUT = true>
__device__ void local_search_one(const DevItem& it, int ind, Smem<SLOTS, WAVES>& sm, const Lig<SLOTS>& L,
                                 int iterations, float rho, float eps, bool final_eval) {
    search(it, ind, L.G, iterations, rho, eps, final_eval, WAVES == 1 || L.wv == 0, [&](float x, float& gr) {
        return evaluate<SLOTS, VAR, WAVES, ANY_LAYOUT>(it.grid, sm, L, x, gr, nullptr, VAR >= 0 ? VAR : it.variant);
    });
}

template <int SLOTS, int VAR, int WAVES = 1>
__device__ void ls_run(const DevItem& it, int ind, Smem<SLOTS, WAVES>& sm, const Lig<SLOTS>& L,
                       const LsParams& p) {
    // a kernel specialised for one variant runs only items whose grids have
    // the corner-expanded copy bound; the dispatching kernel takes any
    local_search_one<SLOTS, VAR, WAVES, (VAR < 0)>(it, ind, sm, L, it.iterations, p.rho, p.eps, it.final_eval != 0);
}

// The item of work unit u: the last item with unit_begin <= u (items are
// in unit order).
__device__ __forceinline__ int item_of_unit(const LsParams& p, int u) {
    int lo = 0, hi = p.n_items - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (uniform(gmem(&p.items[mid].unit_begin)[0]) <= u) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// The item record, read once per work unit, with every word made
// wave-uniform (scalar registers).
__device__ __forceinline__ DevItem load_item(const DevItem* items, int k) {
    static_assert(sizeof(DevItem) % 4 == 0, "item record is made of 32-bit words");
    constexpr int kWords = sizeof(DevItem) / 4;
    const auto src = gmem(reinterpret_cast<const uint32_t*>(items + k));
    DevItem out;
    uint32_t* dst = reinterpret_cast<uint32_t*>(&out);
#pragma unroll
    for (int w = 0; w < kWords; ++w) dst[w] = __builtin_amdgcn_readfirstlane(src[w]);
    return out;
}

// Persistent local-search kernel. Work units are individuals, numbered item by
// item in the order the host gives (longest items first); each wave takes the
// next unit from a global counter until none is left, reloading the ligand
// only when the item changes. Every wave exits once the counter passes the
// last unit.
template <int MODE, int VAR>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(MODE == docklaunch::kSlots1 ? 3 : 2, MODE == docklaunch::kSlots1 ? 3 : 2))) void ls_kernel(LsParams p) {
    // LDS sized for the layouts the launch can meet
    constexpr size_t kBytes = MODE == docklaunch::kSlots1 ? sizeof(Smem<1>) : sizeof(Smem<2>);
    __shared__ __align__(16) unsigned char smem[kBytes];
    int cur_item = -1;
    while (true) {
        int u = 0;
        if (lane_id() == 0) u = atomicAdd(p.counter, 1);
        u = uniform(u);
        if (u >= p.total_units) break;
        const int lo = item_of_unit(p, u);
        const DevItem it = load_item(p.items, lo);
        const int ind = u - it.unit_begin;
        // the ligand's LDS tables are refilled only when the item changes;
        // its per-lane registers are rebuilt for every individual, so that no
        // ligand state stays live across units (the two atom-slot layouts of
        // a mixed launch would otherwise both hold registers)
        const bool reload = lo != cur_item;
        cur_item = lo;
        const bool one = MODE == docklaunch::kSlots1 || (MODE == docklaunch::kSlotsAny && it.slots == 1);
        if (one) {
            Smem<1>& sm = *reinterpret_cast<Smem<1>*>(smem);
            Lig<1> L;
            load_ligand<1>(it.blob, sm, L, reload);
            ls_run<1, VAR>(it, ind, sm, L, p);
        } else if constexpr (MODE != docklaunch::kSlots1) {
            Smem<2>& sm = *reinterpret_cast<Smem<2>*>(smem);
            Lig<2> L;
            load_ligand<2>(it.blob, sm, L, reload);
            ls_run<2, VAR>(it, ind, sm, L, p);
        }
    }
}

// Persistent local-search kernel with WAVES (2 or 4) waves per individual:
// one individual per block of 64 WAVES threads, wave w owning atom positions
// 64 w .. 64 w + 63 and the w-th run of the pair batches. The first thread
// takes the next unit and hands it to every wave through LDS; every wave
// exits once the counter passes the last unit.
template <int VAR, int WAVES>
__global__ __launch_bounds__(64 * WAVES) __attribute__((amdgpu_waves_per_eu(3, 3))) void ls_kernel_mw(LsParams p) {
    __shared__ Smem<1, WAVES> sm;
    int cur_item = -1;
    while (true) {
        __syncthreads();                       // the previous unit is read by every wave
        if (threadIdx.x == 0) sm.unit = atomicAdd(p.counter, 1);
        __syncthreads();
        const int u = uniform(sm.unit);
        if (u >= p.total_units) break;
        const int lo = item_of_unit(p, u);
        const DevItem it = load_item(p.items, lo);
        const int ind = u - it.unit_begin;
        const bool reload = lo != cur_item;
        cur_item = lo;
        Lig<1> L;
        load_ligand<1, WAVES>(it.blob, sm, L, reload);
        ls_run<1, VAR, WAVES>(it, ind, sm, L, p);
    }
}

// ---------------------------------------------------------------------------
// One individual per block, for populations too small to fill the GPU with a
// wave each: the waves of a block share the pair terms of one individual and
// give the result of the one-wave evaluation bit for bit. A lone wave needs
// some 10,500 cycles per evaluation (48 atoms, 886 pairs), 6,000 of them in the
// pair batches, whose accumulator slots chain one batch to the next, and the
// rest of the GPU idles.
//
// Wave role 0 leads: it holds the genotype and does what the one-wave kernel
// does outside the pair terms. Per evaluation the waves meet three times:
//   positions written (role 0) | pair terms, batches dealt out to the waves,
//   each pair's (d, w) and energy left in LDS | accumulator slots summed by
//   all threads, a thread per slot, from the pairs that the ligand's gather
//   table names in batch order (the order the one-wave kernel adds them in),
//   the lane energies and the grid term by the last two roles | totals,
//   genotype gradient and step (role 0).
// More batches than a buffer holds go in chunks through two buffers in turn:
// while one is summed the other is filled, one barrier per chunk.
//
// Bound by the leader's serial part, 3,500 of 5,800 cycles (150 individuals of 48
// atoms: pose 1,480, shared part 2,280, copy sums 390, totals and gradient 1,230,
// step 390), for long pair lists by the shared one (112 atoms, 89 batches: 17,500 of
// 22,700). Four waves on more than sixteen batches spill 49 registers. us per evaluation at
// 256 individuals, a wave each against this: 24 atoms 2.48 and 2.27, 48 atoms 4.58
// and 2.58, 64 atoms (28 batches) 6.75 and 4.15, 112 atoms (90 batches) 18.6 and
// 10.0; with four waves at 512 individuals 48 atoms 4.87 and 3.65, 64 atoms 7.14
// and 6.38.
// ---------------------------------------------------------------------------
constexpr int kPairRow = dockblob::kGatherRow / 16;   // float4s per batch: 64 pairs and a zero
constexpr int kCoopRows = docklaunch::kCoopKeep;        // batches a buffer holds

template <int SLOTS>
struct __align__(16) SmemC {
    static constexpr int kSlots = SLOTS == 1 ? dockblob::kMaxSlotsSmall : dockblob::kMaxSlots;
    float4 dyn[kWave * SLOTS];                  // as in Smem
    TorsionAcc<0> u;                            // the transforms alone
    float4 tor[kMaxTors][2];
    uint32_t chain[kMaxFrag][kChain / 4];
    float4 acc[kSlots];                         // summed accumulator slots
    float4 grid[kWave * SLOTS];                 // per atom: grid energy and gradient
    float esum[kWave];                          // lane energies of the pairs
    float t[4];                                 // translation genes
    int unit, go;                               // work unit; another evaluation follows
};

// What a wave needs of the shared pair terms.
struct CoopPairs {
    const u32x4* table;     // gather table: [octet of batches][slot], eight entries each
    float4* pair;           // one or two buffers of kCoopRows x kPairRow
    float* energy;          // and of kCoopRows x 64
    int nslot, role;
};

// Two unused gather table entries.
constexpr uint32_t kGatherPad = dockblob::kGatherNone | (uint32_t)dockblob::kGatherNone << 16;

// A wave's share of one chunk of batches, in registers: its records, and the
// gather table entries of its threads' accumulator slots.
template <int SLOTS, int W>
struct CoopShare {
    static constexpr int kOctets = kCoopRows / dockblob::kGatherRows;
    static constexpr int kMine = kCoopRows / W;                                                      // batches
    static constexpr int kOwn = (SmemC<SLOTS>::kSlots + W * kWave - 1) / (W * kWave);              // slots
    static_assert(kCoopRows % W == 0 && kCoopRows % dockblob::kGatherRows == 0, "whole octets, dealt out evenly");
    u32x4 rec[kMine];
    u32x4 tab[kOwn][kOctets];
    int words[kOwn][kOctets];           // of the entries (two to a word), how many any lane needs

    // `chunk` exists; indices past the last batch or slot are clamped, so that
    // the loads need no branch
    __device__ __forceinline__ void load(const Lig<SLOTS>& L, const CoopPairs& c, int chunk) {
        const auto at = gmem(L.plist) + lane_id();
#pragma unroll
        for (int q = 0; q < kMine; ++q)
            rec[q] = at[(size_t)min(kCoopRows * chunk + c.role + W * q, L.n_batches - 1) * kWave];
#pragma unroll
        for (int s = 0; s < kOwn; ++s) {
            const int k = c.role * kWave + lane_id() + s * W * kWave;
#pragma unroll
            for (int h = 0; h < kOctets; ++h) {
                const int octet = kOctets * chunk + h;
                tab[s][h] = gmem(c.table)[(size_t)min(octet, (L.n_batches - 1) >> 3) * c.nslot + min(k, c.nslot - 1)];
                if (k >= c.nslot || 8 * octet >= L.n_batches) tab[s][h] = u32x4{kGatherPad, kGatherPad, kGatherPad, kGatherPad};
            }
        }
    }
    __device__ __forceinline__ void count() {
#pragma unroll
        for (int s = 0; s < kOwn; ++s)
#pragma unroll
            for (int h = 0; h < kOctets; ++h) {
                words[s][h] = 0;
#pragma unroll
                for (int w = 0; w < 4; ++w)
                    if (__any(tab[s][h][w] != kGatherPad)) words[s][h] = w + 1;   // a slot's entries lie at the front
            }
    }
};

// The shared part of one evaluation, entered by every wave of the block with
// its shares of the first chunks. KEEP: the ligand has one chunk, whose share
// stays in registers; else a share is replaced by that of the chunk after next
// once used, and those of the first two are back at the end. GRID: the wave
// that has the grid term (role W - 1), code of its own so that its gathers
// stay in flight until the pair terms are done.
template <int SLOTS, int W, bool KEEP, bool GRID>
__device__ __forceinline__ void coop_pairs(const GridParams& G, SmemC<SLOTS>& sm, const Lig<SLOTS>& L,
                                           const CoopPairs& c, CoopShare<SLOTS, W> (&share)[KEEP ? 1 : 2]) {
    using Share = CoopShare<SLOTS, W>;
    const int lane = lane_id();
    const int nb = L.n_batches;
    const int chunks = (nb + kCoopRows - 1) / kCoopRows;
    const int y_batch = 4 * ((nb - 1) >> 2) + 2;      // the batch whose squares are added x first
    float x[SLOTS][3], tv[3] = {sm.t[0], sm.t[1], sm.t[2]};
    GridTaps tap[SLOTS];
    if constexpr (GRID) {
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
            const float4 p = sm.dyn[lane + kWave * s];
            x[s][0] = p.x; x[s][1] = p.y; x[s][2] = p.z;
            grid_load<false>(G, L.cls[s], x[s], tv, tap[s]);
        }
    }
    float4 acc[Share::kOwn];
#pragma unroll
    for (int s = 0; s < Share::kOwn; ++s) acc[s] = make_float4(0.f, 0.f, 0.f, 0.f);
    float e_lane = 0.f;
    auto pairs = [&](int chunk, auto set) {
        constexpr int b = decltype(set)::value;
        float4* const pair = c.pair + b * kCoopRows * kPairRow;
        float* const energy = c.energy + b * kCoopRows * kWave;
#pragma unroll
        for (int q = 0; q < Share::kMine; ++q) {
            const int r = c.role + W * q, batch = kCoopRows * chunk + r;
            if (q % 2 == 0) __builtin_amdgcn_sched_barrier(0);    // two batches in flight
            if (batch < nb) {
                const u32x4 rec = share[b].rec[q];
                const float4 pi = *slot(sm.dyn, rec.x & L.pmask);
                const float4 pj = *slot(sm.dyn, __builtin_amdgcn_ubfe(rec.x, dockblob::kSlotShift, L.pbits));
                const PairForce F = pair_force(rec, pi, pj, batch == y_batch);
                pair[r * kPairRow + lane] = make_float4(F.dx, F.dy, F.dz, F.w);
                energy[r * kWave + lane] = F.e;
            }
        }
    };
    auto gather = [&](int chunk, auto set) {
        constexpr int b = decltype(set)::value;
        float4* const pair = c.pair + b * kCoopRows * kPairRow;
        const float* const energy = c.energy + b * kCoopRows * kWave;
        if constexpr (!KEEP) share[b].count();
#pragma unroll
        for (int s = 0; s < Share::kOwn; ++s)
#pragma unroll
            for (int h = 0; h < Share::kOctets; ++h) {
                // four entries at a time, all of an octet's reads ahead of the
                // sums; an entry is the byte offset of a pair in the octet's
                // rows, with its sign in bit 15
                const float4* const rows = pair + h * dockblob::kGatherRows * kPairRow;
                const u32x4 tab = share[b].tab[s][h];
                const bool some = share[b].words[s][h] > 0, more = share[b].words[s][h] > 2;
                float4 f[8];
                auto read = [&](int k) {
                    const uint32_t word = tab[k];
                    f[2 * k] = *slot(const_cast<float4*>(rows), (int)(word & 0x7fffu));
                    f[2 * k + 1] = *slot(const_cast<float4*>(rows), (int)__builtin_amdgcn_ubfe(word, 16, 15));
                };
                auto add = [&](int k) {
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        const float4 v = f[2 * k + e];
                        const uint32_t flip = (e ? tab[k] : tab[k] << 16) & 0x80000000u;
                        const float w = __uint_as_float(__float_as_uint(v.w) ^ flip);
                        acc[s].x = fmaf(w, v.x, acc[s].x);
                        acc[s].y = fmaf(w, v.y, acc[s].y);
                        acc[s].z = fmaf(w, v.z, acc[s].z);
                    }
                };
                if (some) { read(0); read(1); }
                if (more) { read(2); read(3); }
                __builtin_amdgcn_sched_barrier(0);
                if (some) { add(0); add(1); }
                if (more) { add(2); add(3); }
            }
        if (c.role == W - 2) {
            float e[kCoopRows];                       // rows no batch filled are read, not used
#pragma unroll
            for (int r = 0; r < kCoopRows; ++r) e[r] = energy[r * kWave + lane];
#pragma unroll
            for (int r = 0; r < kCoopRows; ++r)
                if (kCoopRows * chunk + r < nb) e_lane += e[r];
        }
        if constexpr (!KEEP) share[b].load(L, c, chunk + 2 < chunks ? chunk + 2 : min(chunk & 1, chunks - 1));
    };
    using Set0 = IntC<0>;
    using Set1 = IntC<KEEP ? 0 : 1>;
    if (chunks > 0) {
        pairs(0, Set0());
        lds_barrier();
        if constexpr (KEEP) {
            gather(0, Set0());
        } else {
            // one buffer is filled while the other is summed
            for (int chunk = 0;; chunk += 2) {
                if (chunk + 1 < chunks) pairs(chunk + 1, Set1());
                gather(chunk, Set0());
                if (chunk + 1 >= chunks) break;
                lds_barrier();
                if (chunk + 2 < chunks) pairs(chunk + 2, Set0());
                gather(chunk + 1, Set1());
                if (chunk + 2 >= chunks) break;
                lds_barrier();
            }
        }
    }
#pragma unroll
    for (int s = 0; s < Share::kOwn; ++s) {
        const int k = c.role * kWave + lane + s * W * kWave;
        if (k < c.nslot) sm.acc[k] = acc[s];
    }
    if (c.role == W - 2) sm.esum[lane] = e_lane;
    if constexpr (GRID) {
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
            float4 e;
            grid_term(G, tap[s], L.chg[s][1], L.chg[s][2], x[s], tv, e.x, e.y, e.z, e.w);
            sm.grid[lane + kWave * s] = e;
        }
    }
    lds_barrier();
}

// One individual's search by the block (the code of one work unit).
template <int SLOTS, int W, bool KEEP>
__device__ __forceinline__ void coop_search(const DevItem& it, int ind, SmemC<SLOTS>& sm, float4* dyn_lds, bool reload,
                                            const LsParams& p) {
    constexpr int kBuffers = KEEP ? 1 : 2;
    const int lane = lane_id();
    const int wave = uniform((int)threadIdx.x >> 6);
    // the leaders of the two blocks that share a CU (of 256) sit on different SIMDs;
    // on another number of CUs only that placement is lost
    const int role = uniform((wave + ((int)blockIdx.x >> 8)) & (W - 1));
    Lig<SLOTS> L;
    load_atoms<SLOTS, false>(it.blob, 0, L);
    const Header* h = reinterpret_cast<const Header*>(it.blob);
    CoopPairs c;
    c.table = uniform_ptr(reinterpret_cast<const u32x4*>(it.blob + h->off_gather));
    c.pair = dyn_lds;
    c.energy = reinterpret_cast<float*>(dyn_lds + kBuffers * kCoopRows * kPairRow);
    c.nslot = L.n_copies * L.stride;
    c.role = role;
    if (reload) {
        fill_tables(it.blob, sm, L.T, L.NF, (int)threadIdx.x, kWave * W);
        // the zeros that unused gather entries name, one per octet
        if (threadIdx.x < kBuffers * kCoopRows / dockblob::kGatherRows)
            c.pair[threadIdx.x * dockblob::kGatherRows * kPairRow + kWave] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    CoopShare<SLOTS, W> share[kBuffers];
    if (L.n_batches > 0) {
#pragma unroll
        for (int k = 0; k < kBuffers; ++k) {
            share[k].load(L, c, min(k, (L.n_batches - 1) / kCoopRows));
            share[k].count();
        }
    }
    lds_barrier();
    if (role != 0) {
        while (true) {
            lds_barrier();
            if (!uniform(sm.go)) return;
            if (role == W - 1) coop_pairs<SLOTS, W, KEEP, true>(it.grid, sm, L, c, share);
            else coop_pairs<SLOTS, W, KEEP, false>(it.grid, sm, L, c, share);
        }
    }
    search(it, ind, L.G, it.iterations, p.rho, p.eps, it.final_eval != 0, true, [&](float gene, float& gr) {
        Rot Rq;
        float tv[3], x[SLOTS][3], g[SLOTS][3];
        transforms_of<1>(sm, L, gene, Rq, tv);
        place_atoms<SLOTS, 1, 4>(sm, L, Rq, x);
        if (lane < 3) sm.t[lane] = gene;
        if (lane == 0) sm.go = 1;
        lds_barrier();
        coop_pairs<SLOTS, W, KEEP, false>(it.grid, sm, L, c, share);
        float e_lane = sm.esum[lane];
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
            const int a = lane + kWave * s;
            const float4 e = sm.grid[a];
            g[s][0] = g[s][1] = g[s][2] = 0.f;
            const bool ok = a < L.N;
            if (ok) sum_copies(sm.acc + a, L.n_copies, L.stride, g[s]);
            g[s][0] += ok ? e.y : 0.f;
            g[s][1] += ok ? e.z : 0.f;
            g[s][2] += ok ? e.w : 0.f;
            e_lane += ok ? e.x : 0.f;
        }
        const int var = it.variant;
        return finish<SLOTS, 1>(sm, L, Rq, x, g, e_lane, [var](float4 v) { return sum4_of(var, v); }, gr);
    });
    if (lane == 0) sm.go = 0;
    lds_barrier();
}

// Persistent kernel of 64 W threads per individual; units and items as in
// ls_kernel. Every wave of a block takes the same unit and exits once the
// counter passes the last.
template <int SLOTS, int W, bool KEEP>
__global__ __launch_bounds__(64 * W, 2) void ls_kernel_coop(LsParams p) {
    __shared__ SmemC<SLOTS> sm;
    extern __shared__ float4 dyn_lds[];
    int cur_item = -1;
    while (true) {
        lds_barrier();                         // the previous unit is done with the LDS
        if (threadIdx.x == 0) sm.unit = atomicAdd(p.counter, 1);
        lds_barrier();
        const int u = uniform(sm.unit);
        if (u >= p.total_units) break;
        const int k = item_of_unit(p, u);
        const DevItem it = load_item(p.items, k);
        const bool reload = k != cur_item;
        cur_item = k;
        coop_search<SLOTS, W, KEEP>(it, u - it.unit_begin, sm, dyn_lds, reload, p);
    }
}

// ---------------------------------------------------------------------------
// Two individuals per wave, for ligands of at most 32 atoms and 25 torsions
// (G = 7 + T <= 32 genes): each 32-lane half of the wave holds one
// individual, lane j of half h holding atom j and gene j of individual h.
// The per-atom stages then fill twice as many lanes as with one individual
// per wave, and the per-evaluation tail (block sum, prefix scans, gradient
// assembly, update) serves two individuals. The pair phase walks the same
// 64-record batches in two steps of 32 records, each half adding forces to
// its own accumulator slots (the slots of a batch are distinct, so those of
// a half-batch are too). The block sum is the wavefront shuffle over each
// half; the halves never exchange values, so an individual's result does
// not depend on the other half.
// ---------------------------------------------------------------------------
constexpr int kHalf = 32;

// LDS of a two-individual wave. Twelve such blocks (three waves per SIMD) must
// fit in the CU's 160 KB after each block's LDS is rounded up to the
// allocation granularity: 12,800 bytes per block fit, while the 13,344 bytes
// of accumulators sized for 320 slots per half left room for eleven blocks
// per CU. A ligand of <= 32 atoms needs at most 288 slots; an energy-only
// evaluation none (FORCES = false: sixteen blocks, four waves per SIMD).
template <bool FORCES>
struct __align__(16) Smem2T {
    float4 dyn[2][kHalf];               // per half: positions relative to t, sqrt(kElec) q
    TorsionAcc<FORCES ? dockblob::kMaxSlotsTiny : 0> u[2];   // per half
    float4 tor[kMaxTors][2];
    uint32_t chain[kMaxFrag][kChain / 4];
};
using Smem2 = Smem2T<true>;
static_assert(sizeof(Smem2) <= 12800, "twelve two-individual blocks per CU");

// Exchanges the second and fourth row of `lo` with the first and third of
// `hi`: from two copies of a value, `lo` then holds each half's first row in
// both of the half's rows, `hi` its second.
#define SWAP_ROWS(lo, hi) "v_permlane16_swap_b32 " lo ", " hi "\n\t"
__device__ __forceinline__ void half_rows(float v, float& lo, float& hi) {
    lo = hi = v;
    asm("s_nop 1\n\t" SWAP_ROWS("%0", "%1") "s_nop 1" : "+v"(lo), "+v"(hi));
}

// Sums over this lane's half, every lane of the half receives them: row sums
// by a DPP butterfly, then the half's two rows.
__device__ __forceinline__ float half_sum(float v) {
    asm("s_nop 1\n\t" DPP_ROW_SUM(DPP_STEP1) : "+v"(v));
    float lo, hi;
    half_rows(v, lo, hi);
    return lo + hi;
}
__device__ __forceinline__ float4 half_sum4(float4 v) {
    asm("s_nop 1\n\t" DPP_ROW_SUM(DPP_STEP4) DPP_END : "+v"(v.x), "+v"(v.y), "+v"(v.z), "+v"(v.w));
    float4 w = v;
    asm("s_nop 1\n\t" SWAP_ROWS("%0", "%4") SWAP_ROWS("%1", "%5") SWAP_ROWS("%2", "%6") SWAP_ROWS("%3", "%7") "s_nop 1"
        : "+v"(v.x), "+v"(v.y), "+v"(v.z), "+v"(v.w), "+v"(w.x), "+v"(w.y), "+v"(w.z), "+v"(w.w));
    return make_float4(v.x + w.x, v.y + w.y, v.z + w.z, v.w + w.w);
}

// Inclusive prefix sums of six values within each half.
__device__ __forceinline__ void half_scan6(float v[6]) {
    asm("s_nop 1\n\t" DPP_ROW_SCAN(DPP_STEP6) DPP_HALF(DPP_STEP6) DPP_END
        : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "+v"(v[4]), "+v"(v[5]));
}

// The ligand as a two-individual wave holds it: lane j of either half the
// atom j (per-lane registers), the shared torsion and fragment tables in LDS.
template <bool FORCES>
__device__ void load_ligand2(const uint8_t* __restrict__ blob, Smem2T<FORCES>& sm, Lig<1>& L, bool fill_lds = true) {
    if (fill_lds) wave_sync();  // previous users of the LDS tables are done
    const Header* h = reinterpret_cast<const Header*>(blob);
    const int lane = lane_id();
    L.wv = 0;
    L.N = uniform(h->n_atoms);
    L.T = uniform(h->n_torsions);
    L.NF = uniform(h->n_frag);
    L.G = uniform(h->n_genes);
    L.n_batches = uniform(h->n_batches);
    L.n_copies = uniform(h->n_copies);
    L.max_depth = uniform(h->max_depth);
    L.stride = uniform(h->slot_stride);
    L.pmask = L.stride * 16 - 1;
    L.pbits = 31 - __builtin_clz(L.stride * 16);
    L.plist = uniform_ptr(reinterpret_cast<const u32x4*>(blob + h->off_plist));
    const float4* ref = reinterpret_cast<const float4*>(blob + h->off_ref);
    const float4* chg = reinterpret_cast<const float4*>(blob + h->off_chg);
    const int4* iv = reinterpret_cast<const int4*>(blob + h->off_int);
    const int a = lane & (kHalf - 1);
    const bool ok = a < L.N;
    const int ai = ok ? a : 0;
    const float4 r = ref[ai], c = chg[ai];
    const int4 ii = iv[ai];
    L.y0[0][0] = r.x; L.y0[0][1] = r.y; L.y0[0][2] = r.z;
    L.chg[0][0] = ok ? c.x : 0.f; L.chg[0][1] = ok ? c.y : 0.f; L.chg[0][2] = ok ? c.z : 0.f;
    L.cls[0] = ii.x;
    L.frag[0] = ii.y;
    L.orig[0] = ii.z;
    L.chain[0] = chain_word(blob, L.frag[0]);
    // the prefix sums' positions are lanes of this half
    L.torsion = torsion_word(blob, L.T, a - kFirstTorsion) + (uint32_t)(lane & kHalf) * 0x01010000u;
    const Torsion* tr = reinterpret_cast<const Torsion*>(blob + h->off_tors);
    if (fill_lds && lane < L.T) {
        const Torsion t = tr[lane];
        sm.tor[lane][0] = make_float4(t.p[0], t.p[1], t.p[2], 0.f);
        sm.tor[lane][1] = make_float4(t.u[0], t.u[1], t.u[2], 0.f);
    }
    if (fill_lds && a < 3) sm.u[lane >> 5].write_identity(a);
    const uint32_t* ch = reinterpret_cast<const uint32_t*>(blob + h->off_chain);
    const int n_chain_words = L.NF * (kChain / 4);
    uint32_t* dst = &sm.chain[0][0];
    if (fill_lds)
        for (int i = lane; i < n_chain_words; i += kWave) dst[i] = ch[i];
    wave_sync();
}

// One evaluation of E and dE/dgenotype for the two individuals of the wave.
// `gene` is gene j of this lane's individual (j = lane % 32; j >= G
// ignored); returns this half's E and writes this lane's gradient component
// to `grad`. atom_out: this half's per-atom output (or nullptr).
template <bool ANY_LAYOUT, bool GRAD = true>
__device__ float evaluate2(const GridParams& G, Smem2T<GRAD>& sm, const Lig<1>& L, float gene, float& grad,
                           float* atom_out) {
    const int lane = lane_id();
    const int j = lane & (kHalf - 1);
    const int h = lane >> 5;
    const int N = L.N;
    const int ns = 2 * L.n_batches;              // steps of the pair terms, the first four's records loaded here
    using Records = PairRecords<kHalf>;
    const Records records(L.plist, ns, j);
    u32x4 R[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) R[q] = records.load(0, q);
    float body, rest;                            // the rigid-body genes lie in the half's first row
    half_rows(gene, body, rest);
    const float tx = row_lane<0>(body), ty = row_lane<1>(body), tz = row_lane<2>(body);
    const Rot Rq = rotation(row_lane<3>(body), row_lane<4>(body), row_lane<5>(body), row_lane<6>(body));

    // torsion transforms of this half's individual
    const int k = j - kFirstTorsion;
    if (k >= 0 && k < L.T) {
        torsion_transform(gene, sm.tor[k][0], sm.tor[k][1], sm.u[h].transforms() + 3 * k);
    }
    wave_sync();
    // atom positions relative to the rotation centre, as in `evaluate`
    const float tv[3] = {tx, ty, tz};
    float x[3];
    {
        float y0 = L.y0[0][0], y1 = L.y0[0][1], y2 = L.y0[0][2];
        apply_chain<2>(L.chain[0], sm.chain[L.frag[0]], sm.u[h].transforms(), L.max_depth, y0, y1, y2);
        rotate(Rq, y0, y1, y2, x);
        sm.dyn[h][j] = make_float4(x[0], x[1], x[2], kSqrtElec * L.chg[0][1]);
    }
    wave_sync();

    float g[3] = {0.f, 0.f, 0.f};
    float e_lane = 0.f;
    GridTaps tap;
    float4* const dynh = sm.dyn[h];
    float4* const acch = sm.u[h].acc;
    const int pmask = L.pmask;
    auto pos_i = [&](uint32_t w) { return *slot(dynh, w & pmask); };
    auto pos_j = [&](uint32_t w) { return *slot(dynh, __builtin_amdgcn_ubfe(w, dockblob::kSlotShift, L.pbits)); };
    if constexpr (GRAD) {
        const int nslot = L.n_copies * L.stride;
        static_assert(dockblob::kMaxSlotsTiny % kHalf == 0, "clearing stays inside the half's accumulators");
        for (int k = 0; k < nslot; k += kHalf) acch[k + j] = make_float4(0.f, 0.f, 0.f, 0.f);
        wave_sync();
    }
    // pair terms: step s takes records 32 (s % 2) .. 32 (s % 2) + 31 of
    // batch s / 2, record j for lane j of either half. Software pipeline:
    // step s reads the positions of step s + 1 before computing its own pair
    // and loads the record of step s + 4 (register sets indexed by s mod 4
    // and mod 2, steps unrolled by four, no loaded value copied between
    // steps).
    if (ns > 0) {
        float4 Pi[2], Pj[2];
        Pi[0] = pos_i(R[0].x);
        Pj[0] = pos_j(R[0].x);
        int s = 0, group = 4 * Records::kRow;        // group: the rows of steps s + 4 to s + 7, s mod 4 = 0
        auto step = [&](auto residue, auto load) {
            constexpr int r = decltype(residue)::value;  // s mod 4
            constexpr int c = r & 1, n = (r + 1) & 1;
            const u32x4 rn = R[(r + 1) & 3];
            Pi[n] = pos_i(rn.x);
            Pj[n] = pos_j(rn.x);
            __builtin_amdgcn_sched_barrier(0);
            const PairForce F = pair_force(R[r], Pi[c], Pj[c], r == 0 || (decltype(load)::value == 0 && r == 2));
            if constexpr (GRAD) {
                const float4 ai = *slot(acch, F.si);
                const float4 aj = *slot(acch, F.sj);
                store_force(acch, F, ai, aj);
            }
            e_lane += F.e;
            if constexpr (decltype(load)::value != 0) R[r] = records.load(group, r);
            __builtin_amdgcn_sched_barrier(0);
            ++s;
        };
        using I0 = IntC<0>;
        using I1 = IntC<1>;
        using I2 = IntC<2>;
        using I3 = IntC<3>;
        using Load = IntC<1>;
        using NoLoad = IntC<0>;
        for (; s + 4 <= ns; group += 4 * Records::kRow) {
            step(I0(), Load()); step(I1(), Load()); step(I2(), Load()); step(I3(), Load());
        }
        __builtin_amdgcn_sched_barrier(0);
        grid_load<ANY_LAYOUT>(G, L.cls[0], x, tv, tap);
        __builtin_amdgcn_sched_barrier(0);
        if (s < ns) step(I0(), NoLoad());
        if (s < ns) step(I1(), NoLoad());
        if (s < ns) step(I2(), NoLoad());
    } else {
        grid_load<ANY_LAYOUT>(G, L.cls[0], x, tv, tap);
    }
    if constexpr (GRAD) {
        wave_sync();
        // each atom adds its copies in copy order
        if (j < N) sum_copies(acch + j, L.n_copies, L.stride, g);
    }
    // grid term
    float e_atom;
    {
        float e, gx, gy, gz;
        grid_term(G, tap, L.chg[0][1], L.chg[0][2], x, tv, e, gx, gy, gz);
        const bool ok = j < N;
        e_atom = ok ? e : 0.f;
        g[0] = ok ? g[0] + gx : 0.f;
        g[1] = ok ? g[1] + gy : 0.f;
        g[2] = ok ? g[2] + gz : 0.f;
        e_lane += e_atom;
    }
    if constexpr (!GRAD) {
        grad = 0.f;
        wave_sync();   // the next evaluation rewrites the position table
        return half_sum(e_lane);
    }
    const float4 bond_a = dynh[L.torsion & 255], bond_b = dynh[(L.torsion >> 8) & 255];
    // block sum of {E, gx, gy, gz} over each half (wavefront shuffle)
    const float4 EG = half_sum4(make_float4(e_lane, g[0], g[1], g[2]));
    // torsion torques: prefix sums of (g, x cross g) within each half; the
    // half's last lane gives the torque about t
    float P[6];
    P[0] = g[0]; P[1] = g[1]; P[2] = g[2];
    P[3] = fmaf(x[1], g[2], -(x[2] * g[1]));
    P[4] = fmaf(x[2], g[0], -(x[0] * g[2]));
    P[5] = fmaf(x[0], g[1], -(x[1] * g[0]));
    half_scan6(P);
    float lo, tq[3];                             // the half's last lane lies in its second row
#pragma unroll
    for (int c = 0; c < 3; ++c) half_rows(P[3 + c], lo, tq[c]);
    const float4 TQ = make_float4(row_lane<15>(tq[0]), row_lane<15>(tq[1]), row_lane<15>(tq[2]), 0.f);
    float S[6];
#pragma unroll
    for (int c = 0; c < 6; ++c) S[c] = lane_at(P[c], L.torsion >> 24) - lane_at(P[c], L.torsion >> 16);
    grad = gene_gradient(j, EG, TQ, Rq, torsion_gradient(S, bond_a, bond_b));
    if (atom_out && j < N) {
        float4* o = reinterpret_cast<float4*>(atom_out) + 2 * L.orig[0];
        o[0] = make_float4(x[0], x[1], x[2], e_atom);
        o[1] = make_float4(g[0], g[1], g[2], 0.f);
    }
    return EG.x;
}

// ADADELTA local search of the two individuals ind0 and ind0 + 1 of an item
// (count = 1: only the first; the second half then mirrors the first and
// writes nothing). The steps are those of local_search_one.
template <bool ANY_LAYOUT>
__device__ void local_search_two(const DevItem& it, int ind0, int count, Smem2& sm, const Lig<1>& L,
                                 int iterations, float rho, float eps, bool final_eval) {
    const int lane = lane_id();
    const int j = lane & (kHalf - 1);
    const int h = lane >> 5;
    const bool live = h < count;
    const int ind = ind0 + (live ? h : 0);
    const int G = L.G;
    const bool act = j < G;
    const size_t o = (size_t)ind * G + j;
    float x = act ? it.genotype[o] : 0.f;
    float ag = act ? it.acc_g2[o] : 0.f;
    float ad = act ? it.acc_dx2[o] : 0.f;
    float bx = act ? it.best_genotype[o] : 0.f;
    float bestE = it.best_energy[ind];
    float lastE = it.energy[ind];
    float lastG = 0.f;
    const int passes = iterations + (final_eval ? 1 : 0);
    for (int pass = 0; pass < passes; ++pass) {
        float gr;
        const float E = evaluate2<ANY_LAYOUT>(it.grid, sm, L, x, gr, nullptr);
        lastE = E;
        lastG = gr;
        if (E < bestE) { bestE = E; bx = x; }
        if (pass == iterations) break;
        gr = act ? gr : 0.f;
        float xn = adadelta(x, gr, rho, eps, ag, ad);
        const bool isq = j >= 3 && j < 7;
        const float q2 = isq ? xn * xn : 0.f;
        const float nq2 = (row_lane<3>(q2) + row_lane<4>(q2)) + (row_lane<5>(q2) + row_lane<6>(q2));
        if (isq) xn = (nq2 >= 1e-12f) ? xn * __builtin_amdgcn_rsqf(nq2) : x;
        x = act ? xn : 0.f;
    }
    if (!live) return;
    if (act && it.grad && (iterations > 0 || final_eval)) it.grad[o] = lastG;
    if (act) {
        it.genotype[o] = x;
        it.acc_g2[o] = ag;
        it.acc_dx2[o] = ad;
        it.best_genotype[o] = bx;
    }
    if (j == 0) {
        it.best_energy[ind] = bestE;
        it.energy[ind] = lastE;
        it.iters_done[ind] += iterations;
    }
}

// Persistent local-search kernel, two individuals per wave: work units are
// pairs of individuals of one item ((n + 1) / 2 per item), pulled from the
// counter as in ls_kernel.
template <bool ANY_LAYOUT>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(3, 3))) void ls_kernel_two(LsParams p) {
    __shared__ Smem2 sm;
    int cur_item = -1;
    while (true) {
        int u = 0;
        if (lane_id() == 0) u = atomicAdd(p.counter, 1);
        u = uniform(u);
        if (u >= p.total_units) break;
        const int lo = item_of_unit(p, u);
        const DevItem it = load_item(p.items, lo);
        const int ind0 = 2 * (u - it.unit_begin);
        const int count = min(2, it.n - ind0);
        const bool reload = lo != cur_item;
        cur_item = lo;
        Lig<1> L;
        load_ligand2(it.blob, sm, L, reload);
        local_search_two<ANY_LAYOUT>(it, ind0, count, sm, L, it.iterations, p.rho, p.eps, it.final_eval != 0);
    }
}

// One persistent launch for a batch that mixes two-wave individuals with
// one-wave units (an individual of a ligand of <= 64 atoms, or a pair of
// individuals two per wave): 128-thread blocks, two work counters. Units
// [0, block_units) are the two-wave individuals (their items come first):
// a block takes them from the first counter as ls_kernel_mw does. Once that
// counter passes them, or from the start for the last wave_blocks blocks of
// the grid, each wave takes the remaining units from the second counter on
// its own, in its own half of the block's LDS, ordering its LDS accesses at
// wave scope only (the other wave may be anywhere in its own unit). Every
// wave exits once the second counter passes the last unit.
constexpr size_t kWaveLds =
    ((sizeof(Smem2) > sizeof(Smem<1>) ? sizeof(Smem2) : sizeof(Smem<1>)) + 15) / 16 * 16;

struct __align__(16) SmemUni {
    union {
        Smem<1, 2> two;                       // a two-wave individual
        unsigned char wave[2][kWaveLds];      // per wave: Smem<1> or Smem2
    } u;
    int unit;                                 // outside the union: read after the
                                              // waves start writing their halves
};
static_assert(sizeof(SmemUni) <= 20 * 1280, "six 128-thread blocks per CU");

template <int VAR>
__global__ __launch_bounds__(128) __attribute__((amdgpu_waves_per_eu(3, 3))) void ls_kernel_uni(LsParams p) {
    __shared__ SmemUni sm;
    int cur_item = -1;
    if ((int)blockIdx.x < (int)gridDim.x - p.wave_blocks) {
        while (true) {
            __syncthreads();                   // the previous unit is read by both waves
            if (threadIdx.x == 0) sm.unit = atomicAdd(p.counter, 1);
            __syncthreads();
            const int u = uniform(sm.unit);
            if (u >= p.block_units) break;
            const int lo = item_of_unit(p, u);
            const DevItem it = load_item(p.items, lo);
            const bool reload = lo != cur_item;
            cur_item = lo;
            Lig<1> L;
            load_ligand<1, 2>(it.blob, sm.u.two, L, reload);
            ls_run<1, VAR, 2>(it, u - it.unit_begin, sm.u.two, L, p);
        }
    }
    const int w = uniform((int)threadIdx.x >> 6);
    unsigned char* const lds = sm.u.wave[w];
    cur_item = -1;                             // the two-wave tables are gone
    while (true) {
        int v = 0;
        if (lane_id() == 0) v = atomicAdd(p.counter2, 1);
        const int next = p.block_units + uniform(v);
        if (next >= p.total_units) break;
        const int lo = item_of_unit(p, next);
        const DevItem it = load_item(p.items, lo);
        const bool reload = lo != cur_item;
        cur_item = lo;
        Lig<1> L;
        if (it.pack == 2) {
            Smem2& s2 = *reinterpret_cast<Smem2*>(lds);
            const int ind0 = 2 * (next - it.unit_begin);
            load_ligand2(it.blob, s2, L, reload);
            local_search_two<false>(it, ind0, min(2, it.n - ind0), s2, L, it.iterations, p.rho, p.eps,
                                    it.final_eval != 0);
        } else {
            Smem<1>& s1 = *reinterpret_cast<Smem<1>*>(lds);
            load_ligand<1, 1>(it.blob, s1, L, reload);
            ls_run<1, VAR, 1>(it, next - it.unit_begin, s1, L, p);
        }
    }
}

// Persistent scoring kernel, two genotypes per wave (ind = 2 k + half).
template <bool ANY_LAYOUT, bool GRAD>
__global__ __launch_bounds__(64, GRAD ? 3 : 4) void score_kernel_two(GridParams G, const uint8_t* __restrict__ blob, int n,
                                                          const float* __restrict__ gen,
                                                          float* __restrict__ energy,
                                                          float* __restrict__ grad,
                                                          float* __restrict__ atom_out) {
    __shared__ Smem2T<GRAD> sm;
    Lig<1> L;
    load_ligand2(blob, sm, L);
    const int lane = lane_id();
    const int j = lane & (kHalf - 1);
    const int h = lane >> 5;
    const int G_ = L.G;
    const int n_pairs = (n + 1) >> 1;
    for (int k = blockIdx.x; k < n_pairs; k += gridDim.x) {
        const bool live = 2 * k + h < n;
        const int ind = live ? 2 * k + h : 2 * k;
        const float gene = j < G_ ? gen[(size_t)ind * G_ + j] : 0.f;
        float gr;
        float* ao = (GRAD && atom_out && live) ? atom_out + (size_t)ind * L.N * 8 : nullptr;
        const float E = evaluate2<ANY_LAYOUT, GRAD>(G, sm, L, gene, gr, ao);
        if (live && j == 0) energy[ind] = E;
        if (GRAD && live && grad && j < G_) grad[(size_t)ind * G_ + j] = gr;
    }
}

// Sum over the first 16-lane row (lanes 16..63 ignored), every lane receives it.
__device__ __forceinline__ float row0_sum(float v) {
    v += dpp<0xB1>(v);    // quad_perm [1,0,3,2]
    v += dpp<0x4E>(v);    // quad_perm [2,3,0,1]
    v += dpp<0x141>(v);   // row_half_mirror
    v += dpp<0x140>(v);   // row_mirror
    return readlane(v, 0);
}

// Isolated block sum (reduction test kernel): every thread holds a float4;
// each wave reduces with the chosen variant, the per-wave totals (at most 16)
// meet in LDS after one barrier, and every wave adds them with a butterfly
// over its first row (lane l holds wave l's total), so every thread gets the
// block total in a fixed order.
template <int VAR>
__global__ __launch_bounds__(1024) void block_sum4_kernel(const float4* __restrict__ in,
                                                          float4* __restrict__ out, int repeat,
                                                          float chain) {
    __shared__ float4 part[2][16];
    const int t = threadIdx.x;
    const int nw = blockDim.x >> 6;
    const int w = t >> 6;
    const int lane = t & 63;
    const size_t idx = (size_t)blockIdx.x * blockDim.x + t;
    const float4 v0 = in[idx];
    float4 v = v0;
    float4 tot = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int r = 0; r < repeat; ++r) {
        const float4 ws = sum4<VAR>(v);
        if (nw == 1) {
            tot = ws;
        } else {
            if (lane == 0) part[r & 1][w] = ws;
            __syncthreads();
            const float4 p = lane < nw ? part[r & 1][lane & 15] : make_float4(0.f, 0.f, 0.f, 0.f);
            tot = make_float4(row0_sum(p.x), row0_sum(p.y), row0_sum(p.z), row0_sum(p.w));
        }
        v = make_float4(v0.x + chain * tot.x, v0.y + chain * tot.y, v0.z + chain * tot.z,
                        v0.w + chain * tot.w);
    }
    out[idx] = tot;
}

// The Sec. 3 baseline, for the reduction test only: per component, a wave
// shuffle tree, then the first lane of each wave adds its value into a
// shared accumulator with an atomic, a barrier, and every thread reads the
// accumulator back (three barriers per component, as described there).
__global__ __launch_bounds__(1024) void block_sum4_atomic_kernel(const float4* __restrict__ in,
                                                                 float4* __restrict__ out,
                                                                 int repeat, float chain) {
    __shared__ float acc[4];
    const int t = threadIdx.x;
    const size_t idx = (size_t)blockIdx.x * blockDim.x + t;
    const float4 v0 = in[idx];
    float4 v = v0;
    float4 tot = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int r = 0; r < repeat; ++r) {
        float vc[4] = {v.x, v.y, v.z, v.w};
        float res[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            if (t == 0) acc[c] = 0.f;
            __syncthreads();
            float s = vc[c];
#pragma unroll
            for (int o = 32; o >= 1; o >>= 1) s += __shfl_xor(s, o);
            if ((t & 63) == 0) atomicAdd(&acc[c], s);
            __syncthreads();
            res[c] = acc[c];
            __syncthreads();
        }
        tot = make_float4(res[0], res[1], res[2], res[3]);
        v = make_float4(v0.x + chain * tot.x, v0.y + chain * tot.y, v0.z + chain * tot.z,
                        v0.w + chain * tot.w);
    }
    out[idx] = tot;
}

// Blocks of a kernel that a CU holds at once. The runtime's count divides the
// LDS by the size asked for, but LDS is given out in granules of 1,280 bytes: 13
// blocks of 12,416 bytes were launched per CU where 12 fit, and the last one ran
// as a round of its own (65,536 genotypes of 24 atoms: 80 us instead of 63).
constexpr size_t kLdsGranule = 1280, kLdsPerCu = 160 * 1024;

bool resident_blocks(int* per_cu, const void* k, int threads, size_t dynamic_lds) {
    hipFuncAttributes a;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(per_cu, k, threads, dynamic_lds) != hipSuccess ||
        *per_cu <= 0 || hipFuncGetAttributes(&a, k) != hipSuccess)
        return false;
    const size_t granules = (a.sharedSizeBytes + dynamic_lds + kLdsGranule - 1) / kLdsGranule;
    if (granules) *per_cu = std::min(*per_cu, (int)std::max<size_t>(1, kLdsPerCu / (granules * kLdsGranule)));
    return true;
}

template <int SLOTS, int VAR, bool ANY, bool GRAD>
hipError_t launch_score_k(const GridParams& g, const uint8_t* blob, int n, const float* gen, float* energy,
                          float* grad, float* atom_out, int n_cu, hipStream_t st) {
    auto k = score_kernel<SLOTS, VAR, ANY, GRAD>;
    // resident blocks per CU, queried once per kernel (the query costs tens
    // of microseconds of host time, as much as a small call's kernel)
    static std::atomic<int> cached{0};
    int per_cu = cached.load(std::memory_order_relaxed);
    if (per_cu <= 0) {
        if (!resident_blocks(&per_cu, reinterpret_cast<const void*>(k), 64, 0)) per_cu = 2;
        cached.store(per_cu, std::memory_order_relaxed);
    }
    const long long resident = (long long)per_cu * (n_cu > 0 ? n_cu : 256);
    const int blocks = (int)(n < resident ? n : resident);
    hipLaunchKernelGGL(k, dim3(blocks), dim3(64), 0, st, g, blob, n, gen, energy, grad, atom_out);
    return hipGetLastError();
}

template <int VAR>
hipError_t launch_score_v(const GridParams& g, const uint8_t* blob, int slots, int n,
                          const float* gen, float* energy, float* grad, float* atom_out, int n_cu,
                          hipStream_t st) {
    // no gradient and no per-atom output asked for: the energy-only evaluation
    const bool any = g.corners == nullptr, forces = grad || atom_out;
    auto go = [&](auto launch) { return launch(g, blob, n, gen, energy, grad, atom_out, n_cu, st); };
    if (slots == 1) {
        if (forces) return any ? go(launch_score_k<1, VAR, true, true>) : go(launch_score_k<1, VAR, false, true>);
        return any ? go(launch_score_k<1, VAR, true, false>) : go(launch_score_k<1, VAR, false, false>);
    }
    if (forces) return any ? go(launch_score_k<2, VAR, true, true>) : go(launch_score_k<2, VAR, false, true>);
    return any ? go(launch_score_k<2, VAR, true, false>) : go(launch_score_k<2, VAR, false, false>);
}

template <int VAR>
hipError_t launch_sw_v(const GridParams& g, const uint8_t* blob, int slots, const docklaunch::SwParams& p,
                       hipStream_t st) {
    if (slots == 1 && g.corners)
        hipLaunchKernelGGL((sw_kernel<1, VAR, false>), dim3(p.n), dim3(64), 0, st, g, blob, p);
    else if (slots == 1)
        hipLaunchKernelGGL((sw_kernel<1, VAR, true>), dim3(p.n), dim3(64), 0, st, g, blob, p);
    else if (g.corners)
        hipLaunchKernelGGL((sw_kernel<2, VAR, false>), dim3(p.n), dim3(64), 0, st, g, blob, p);
    else
        hipLaunchKernelGGL((sw_kernel<2, VAR, true>), dim3(p.n), dim3(64), 0, st, g, blob, p);
    return hipGetLastError();
}

template <int MODE>
const void* ls_kernel_ptr(int var) {
    switch (var) {
        case 0: return reinterpret_cast<const void*>(&ls_kernel<MODE, 0>);
        case 1: return reinterpret_cast<const void*>(&ls_kernel<MODE, 1>);
        case 2: return reinterpret_cast<const void*>(&ls_kernel<MODE, 2>);
        case 3: return reinterpret_cast<const void*>(&ls_kernel<MODE, 3>);
        case 4: return reinterpret_cast<const void*>(&ls_kernel<MODE, 4>);
        default: return reinterpret_cast<const void*>(&ls_kernel<MODE, -1>);
    }
}

template <int WAVES>
const void* ls_kernel_mw_ptr(int var) {
    switch (var) {
        case 0: return reinterpret_cast<const void*>(&ls_kernel_mw<0, WAVES>);
        case 1: return reinterpret_cast<const void*>(&ls_kernel_mw<1, WAVES>);
        case 2: return reinterpret_cast<const void*>(&ls_kernel_mw<2, WAVES>);
        case 3: return reinterpret_cast<const void*>(&ls_kernel_mw<3, WAVES>);
        case 4: return reinterpret_cast<const void*>(&ls_kernel_mw<4, WAVES>);
        default: return reinterpret_cast<const void*>(&ls_kernel_mw<-1, WAVES>);
    }
}

const void* ls_kernel_uni_ptr(int var) {
    switch (var) {
        case 0: return reinterpret_cast<const void*>(&ls_kernel_uni<0>);
        case 1: return reinterpret_cast<const void*>(&ls_kernel_uni<1>);
        case 2: return reinterpret_cast<const void*>(&ls_kernel_uni<2>);
        case 3: return reinterpret_cast<const void*>(&ls_kernel_uni<3>);
        case 4: return reinterpret_cast<const void*>(&ls_kernel_uni<4>);
        default: return nullptr;             // the plan gives this launch one variant
    }
}

const void* ls_kernel_for(int mode, int var) {
    if (mode == docklaunch::kTwoPerWave)
        return var == DOCK_REDUCE_SHUFFLE ? reinterpret_cast<const void*>(&ls_kernel_two<false>)
                                          : reinterpret_cast<const void*>(&ls_kernel_two<true>);
    if (mode == docklaunch::kTwoWave) return ls_kernel_mw_ptr<2>(var);
    if (mode == docklaunch::kFourWave) return ls_kernel_mw_ptr<4>(var);
    if (mode == docklaunch::kUnified) return ls_kernel_uni_ptr(var);
    if (mode == docklaunch::kSlots1) return ls_kernel_ptr<docklaunch::kSlots1>(var);
    if (mode == docklaunch::kSlots2) return ls_kernel_ptr<docklaunch::kSlots2>(var);
    return ls_kernel_ptr<docklaunch::kSlotsAny>(var);
}

}  // namespace

namespace docklaunch {

hipError_t launch_score(const GridParams& g, const uint8_t* blob, int slots, int n,
                        const float* genotypes, float* energy, float* grad, float* atom_out,
                        int variant, int n_cu, hipStream_t stream) {
    switch (variant) {
        case DOCK_REDUCE_SHUFFLE: return launch_score_v<0>(g, blob, slots, n, genotypes, energy, grad, atom_out, n_cu, stream);
        case DOCK_REDUCE_MFMA_F32: return launch_score_v<1>(g, blob, slots, n, genotypes, energy, grad, atom_out, n_cu, stream);
        case DOCK_REDUCE_MFMA_BF16: return launch_score_v<2>(g, blob, slots, n, genotypes, energy, grad, atom_out, n_cu, stream);
        case DOCK_REDUCE_MFMA_F16: return launch_score_v<3>(g, blob, slots, n, genotypes, energy, grad, atom_out, n_cu, stream);
        case DOCK_REDUCE_MFMA_BF16X3: return launch_score_v<4>(g, blob, slots, n, genotypes, energy, grad, atom_out, n_cu, stream);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_score_two(const GridParams& g, const uint8_t* blob, int n, const float* genotypes,
                            float* energy, float* grad, float* atom_out, int n_cu, hipStream_t stream) {
    const bool any = g.corners == nullptr, forces = grad || atom_out;
    const void* k = forces ? (any ? reinterpret_cast<const void*>(&score_kernel_two<true, true>)
                                  : reinterpret_cast<const void*>(&score_kernel_two<false, true>))
                           : (any ? reinterpret_cast<const void*>(&score_kernel_two<true, false>)
                                  : reinterpret_cast<const void*>(&score_kernel_two<false, false>));
    static std::atomic<int> cached[4];
    std::atomic<int>& slot = cached[2 * any + forces];
    int per_cu = slot.load(std::memory_order_relaxed);
    if (per_cu <= 0) {
        if (!resident_blocks(&per_cu, k, 64, 0)) per_cu = 2;
        slot.store(per_cu, std::memory_order_relaxed);
    }
    const long long pairs = ((long long)n + 1) / 2;
    const long long resident = (long long)per_cu * (n_cu > 0 ? n_cu : 256);
    const int blocks = (int)(pairs < resident ? pairs : resident);
    GridParams gg = g;
    const uint8_t* bb = blob;
    int nn = n;
    const float* gen = genotypes;
    float* e = energy;
    float* gr = grad;
    float* ao = atom_out;
    void* args[] = {&gg, &bb, &nn, &gen, &e, &gr, &ao};
    return hipLaunchKernel(k, dim3(blocks), dim3(64), args, 0, stream);
}

hipError_t launch_sw(const GridParams& g, const uint8_t* blob, int slots, int variant, const SwParams& p,
                     hipStream_t stream) {
    switch (variant) {
        case DOCK_REDUCE_SHUFFLE: return launch_sw_v<0>(g, blob, slots, p, stream);
        case DOCK_REDUCE_MFMA_F32: return launch_sw_v<1>(g, blob, slots, p, stream);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_expand_corners(const GridParams& g, float* corners, hipStream_t stream) {
    // nodes of all maps together stay below 2^31, so a map's cells do
    const int ncell = (g.nx - 1) * (g.ny - 1) * (g.nz - 1);
    hipLaunchKernelGGL(expand_corners_kernel, dim3((unsigned)(ncell + 31) / 32), dim3(256), 0, stream, g,
                       reinterpret_cast<f32x4*>(corners), ncell);
    return hipGetLastError();
}

hipError_t launch_ls(const LsParams& p, int mode, int variant_uniform, int grid_blocks,
                     hipStream_t stream) {
    const void* k = ls_kernel_for(mode, variant_uniform);
    if (!k) return hipErrorInvalidValue;
    LsParams pp = p;
    void* args[] = {&pp};
    return hipLaunchKernel(k, dim3(grid_blocks), dim3(ls_block_threads(mode)), args, 0, stream);
}

int ls_blocks_per_cu(int mode, int variant_uniform) {
    // cached per (mode, variant): the occupancy query costs host time on
    // every call otherwise
    static std::atomic<int> cache[docklaunch::kLsModes][DOCK_REDUCE_COUNT + 1];
    const int m = mode >= 0 && mode < docklaunch::kLsModes ? mode : 0;
    const int v = variant_uniform >= 0 && variant_uniform < DOCK_REDUCE_COUNT ? variant_uniform : DOCK_REDUCE_COUNT;
    int nb = cache[m][v].load(std::memory_order_relaxed);
    if (nb > 0) return nb;
    const void* k = ls_kernel_for(mode, variant_uniform);
    if (!k || !resident_blocks(&nb, k, ls_block_threads(mode), 0)) return 0;
    cache[m][v].store(nb, std::memory_order_relaxed);
    return nb;
}

namespace {
const void* coop_kernel(int mode, int waves, bool keep) {
    if (mode == kSlots2 && waves == 8)
        return reinterpret_cast<const void*>(keep ? &ls_kernel_coop<2, 8, true> : &ls_kernel_coop<2, 8, false>);
    if (mode == kSlots1 && waves == 8)
        return reinterpret_cast<const void*>(keep ? &ls_kernel_coop<1, 8, true> : &ls_kernel_coop<1, 8, false>);
    if (mode == kSlots1 && waves == 4)
        return reinterpret_cast<const void*>(keep ? &ls_kernel_coop<1, 4, true> : &ls_kernel_coop<1, 4, false>);
    return nullptr;
}
size_t coop_lds(bool keep) { return (size_t)kCoopRows * (keep ? 1 : 2) * (kPairRow * sizeof(float4) + kWave * sizeof(float)); }
}  // namespace

int coop_blocks_per_cu(int mode, int waves, bool keep) {
    // cached per kernel, as in ls_blocks_per_cu
    static std::atomic<int> cache[2][2][2];
    const void* k = coop_kernel(mode, waves, keep);
    if (!k) return 0;
    std::atomic<int>& slot = cache[mode == kSlots1][waves == 8][keep];
    int nb = slot.load(std::memory_order_relaxed);
    if (nb > 0) return nb;
    if (!resident_blocks(&nb, k, 64 * waves, coop_lds(keep))) return 0;
    slot.store(nb, std::memory_order_relaxed);
    return nb;
}

hipError_t launch_ls_coop(const LsParams& p, int mode, int waves, bool keep, int grid_blocks, hipStream_t stream) {
    const void* k = coop_kernel(mode, waves, keep);
    if (!k) return hipErrorInvalidValue;
    LsParams pp = p;
    void* args[] = {&pp};
    return hipLaunchKernel(k, dim3(grid_blocks), dim3(64 * waves), args, coop_lds(keep), stream);
}

hipError_t launch_block_sum4(const float* in, float* out, int n_blocks, int threads, int variant,
                             int repeat, hipStream_t stream) {
    const float4* i4 = reinterpret_cast<const float4*>(in);
    float4* o4 = reinterpret_cast<float4*>(out);
    const float chain = 0.0f;
    switch (variant) {
        case 0: hipLaunchKernelGGL((block_sum4_kernel<0>), dim3(n_blocks), dim3(threads), 0, stream, i4, o4, repeat, chain); break;
        case 1: hipLaunchKernelGGL((block_sum4_kernel<1>), dim3(n_blocks), dim3(threads), 0, stream, i4, o4, repeat, chain); break;
        case 2: hipLaunchKernelGGL((block_sum4_kernel<2>), dim3(n_blocks), dim3(threads), 0, stream, i4, o4, repeat, chain); break;
        case 3: hipLaunchKernelGGL((block_sum4_kernel<3>), dim3(n_blocks), dim3(threads), 0, stream, i4, o4, repeat, chain); break;
        case 4: hipLaunchKernelGGL((block_sum4_kernel<4>), dim3(n_blocks), dim3(threads), 0, stream, i4, o4, repeat, chain); break;
        case 5: hipLaunchKernelGGL(block_sum4_atomic_kernel, dim3(n_blocks), dim3(threads), 0, stream, i4, o4, repeat, chain); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace docklaunch
