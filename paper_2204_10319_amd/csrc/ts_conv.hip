// Feature computation of the sparse-convolution layer (paper Sec. 2.2, Alg. 2; Eq. 1).
//
// Two dataflows over the same kernel map:
//
//  explicit  - Alg. 2 in three launches for all offsets at once ("fused" gather / scatter of
//              Sec. 4.3.2): gather rows into the offset-major buffer F, grouped matmul
//              G = F_n * W_n scheduled as tiles over (offset, row block) without padding,
//              output-stationary reduction of G into X_out (each row reduced in registers,
//              written once).
//  fused     - one output-stationary kernel.  A workgroup owns 128 outputs (sorted by
//              neighbour bitmask so that they share offsets), walks the offsets present in
//              the tile, brings the neighbours' feature rows into LDS or straight into the MFMA
//              operand registers and keeps the sum over offsets in the accumulators.
//              Neither F nor G exists; every output row is written once.
//
// MFMA orientation: D[co][m] += Wt[co][ci] * X[m][ci]  ("A" = transposed weights, "B" = gathered
// feature rows).  A lane then owns 4 consecutive output channels of
// one row per accumulator quad, which makes the stores 8-16 bytes wide.
#include "ts_internal.h"

#include <new>
#include <type_traits>
#include <utility>

using namespace ts;

namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;
constexpr int kWaveRows = 32;                 // rows (MFMA columns) per wave
static_assert(kWaves * kWaveRows == kTileRows, "tile = 4 waves x 32 rows");

// Per-dtype constants.  A lane moves 16-byte vectors of VEC elements.  One operand step covers
// KSTEP = 2*VEC input channels (lane halves h = 0/1 take VEC each).
template <class T> struct Elem;
template <> struct Elem<_Float16> {
    typedef half8 vec;
    static constexpr int VEC = 8, KSTEP = 16;
};
template <> struct Elem<float> {
    typedef floatx4 vec;
    static constexpr int VEC = 4, KSTEP = 8;
};

// Kernel shape: NCB blocks of 32 output channels per workgroup, input channels consumed in
// chunks of KC (KC divides C_in, so every chunk is full and the inner code is branch-free).
// LDS holds a [NCB*32][KC + VEC] slab of transposed weights; the VEC-element row padding
// makes the 16 lanes of a ds_read_b128 phase hit distinct bank groups.
template <class T, int NCB, int KC_>
struct Shape {
    typedef typename Elem<T>::vec vec;
    static constexpr int VEC = Elem<T>::VEC, KSTEP = Elem<T>::KSTEP, KC = KC_;
    static constexpr int NKB = KC / KSTEP;            // operand steps per chunk
    static constexpr int STRIDE = KC + VEC;           // LDS row stride in elements
    static constexpr int VPR = KC / VEC;              // 16-byte vectors per slab row
    static constexpr int ROWS = NCB * 32;
    static constexpr int TOTAL = ROWS * VPR;          // vectors per slab
    static constexpr int WV = (TOTAL + kThreads - 1) / kThreads;   // vectors per thread
    static constexpr int SLAB = ROWS * STRIDE;        // elements per slab
};

__device__ __forceinline__ void mma_step(const half8 &a, const half8 &b, floatx16 &acc) {
    acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, acc, 0, 0, 0);
}
__device__ __forceinline__ void mma_step(const floatx4 &a, const floatx4 &b, floatx16 &acc) {
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[0], b[0], acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[1], b[1], acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[2], b[2], acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[3], b[3], acc, 0, 0, 0);
}

// Global -> registers: this thread's share of the weight slab of (offset n, channels k0..k0+KC).
// Threads past the end of a small slab repeat its last vector (same value to the same place).
template <class S, class T>
__device__ __forceinline__ void load_w_regs(typename S::vec (&wreg)[S::WV], const T *__restrict__ Wt, int n, int co0,
                                            int k0, int cin, int cout) {
    const T *src = Wt + ((int64_t)n * cout + co0) * cin + k0;
#pragma unroll
    for (int i = 0; i < S::WV; ++i) {
        int v = threadIdx.x + i * kThreads;
        v = v < S::TOTAL ? v : S::TOTAL - 1;
        int row = v / S::VPR, col = v % S::VPR;
        wreg[i] = *reinterpret_cast<const typename S::vec *>(src + (int64_t)row * cin + col * S::VEC);
    }
}

// Registers -> LDS, same mapping.
template <class S, class T>
__device__ __forceinline__ void store_w_regs(const typename S::vec (&wreg)[S::WV], T *lds) {
#pragma unroll
    for (int i = 0; i < S::WV; ++i) {
        int v = threadIdx.x + i * kThreads;
        v = v < S::TOTAL ? v : S::TOTAL - 1;
        int row = v / S::VPR, col = v % S::VPR;
        *reinterpret_cast<typename S::vec *>(lds + row * S::STRIDE + col * S::VEC) = wreg[i];
    }
}

// Global -> registers: the lane's operand vectors for channels [k0, k0+KC) of the row at `row`
// (already offset to the lane's half).  No predication: absent neighbours point at a zero row.
template <class S, class T>
__device__ __forceinline__ void load_x_regs(typename S::vec (&b)[S::NKB], const T *row) {
#pragma unroll
    for (int kb = 0; kb < S::NKB; ++kb) b[kb] = *reinterpret_cast<const typename S::vec *>(row + kb * S::KSTEP);
}

// acc[cb] += slab[cb*32 .. +32][0 .. KC) * b^T.
template <class S, class T, int NCB>
__device__ __forceinline__ void mma_stage(const T *lds, const typename S::vec (&b)[S::NKB], floatx16 (&acc)[NCB]) {
    const int lane = threadIdx.x & 63, m = lane & 31, h = lane >> 5;
    const T *base = lds + m * S::STRIDE + h * S::VEC;
#pragma unroll
    for (int kb = 0; kb < S::NKB; ++kb) {
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) {
            typename S::vec a = *reinterpret_cast<const typename S::vec *>(base + cb * 32 * S::STRIDE + kb * S::KSTEP);
            mma_step(a, b[kb], acc[cb]);
        }
    }
}

// Store the wave's accumulators: lane (m, h) holds, for block cb and quad g, the channels
// co0 + cb*32 + g*8 + h*4 + {0..3} of row m.
template <class TO, int NCB>
__device__ __forceinline__ void store_rows(TO *out, int64_t row, int cout, int co0, const floatx16 (&acc)[NCB]) {
    const int lane = threadIdx.x & 63, h = lane >> 5;
    if (row < 0) return;
    TO *dst = out + row * cout + co0 + h * 4;
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            if constexpr (sizeof(TO) == 2) {
                half4 v = {(_Float16)acc[cb][g * 4 + 0], (_Float16)acc[cb][g * 4 + 1], (_Float16)acc[cb][g * 4 + 2],
                           (_Float16)acc[cb][g * 4 + 3]};
                *reinterpret_cast<half4 *>(dst + cb * 32 + g * 8) = v;
            } else {
                floatx4 v = {acc[cb][g * 4 + 0], acc[cb][g * 4 + 1], acc[cb][g * 4 + 2], acc[cb][g * 4 + 3]};
                *reinterpret_cast<floatx4 *>(dst + cb * 32 + g * 8) = v;
            }
        }
    }
}

// ---- fused output-stationary kernel ---------------------------------------------------------
// grid = (tiles, cout / (NCB*32)); cin is a multiple of KC.  A "stage" is one (offset n,
// channel chunk k0) pair of the tile.  Software pipeline with one barrier per stage: while the
// MFMAs of stage s read LDS slab `cur` and the operand registers loaded one stage earlier,
// the global loads of stage s+1 (weight slab, neighbour rows) are in flight; the slab goes to
// the other LDS buffer after the MFMAs.  All loads are unconditional so that the compiler can
// count them: rows without a neighbour read `zero_row` instead.
template <class T, int NCB, int KC, int G>
__global__ void __launch_bounds__(kThreads) k_fused(const T *__restrict__ X, const T *__restrict__ Wt,
                                                    const int32_t *__restrict__ nbr, int stride,
                                                    const int32_t *__restrict__ perm, int64_t n_out,
                                                    T *__restrict__ out, const T *__restrict__ zero_row, int cin,
                                                    int cout, int K3, int centre) {
    typedef Shape<T, NCB, KC> S;
    typedef typename S::vec vec;
    __shared__ __attribute__((aligned(16))) T lds_w[2][G][S::SLAB];
    __shared__ int32_t lds_j[kMaxK3][kTileRows];
    __shared__ uint32_t s_mask;
    const int64_t tile = blockIdx.x;
    const int co0 = blockIdx.y * NCB * 32;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, m = lane & 31, h = lane >> 5;
    const int slot = wave * kWaveRows + m;
    floatx16 acc[NCB];
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb)
        for (int r = 0; r < 16; ++r) acc[cb][r] = 0.f;

    // Neighbour rows of the tile's outputs -> LDS (offset-major), and the OR of their offset
    // bitmasks.  Two threads share an output row and read half of its table row each, all
    // loads issued before the first is used.
    if (threadIdx.x == 0) s_mask = 0;
    __syncthreads();
    {
        const int half = threadIdx.x >> 7, col = threadIdx.x & 127;
        const int64_t pos = tile * kTileRows + col;
        const int32_t k = perm ? perm[pos] : (pos < n_out ? (int32_t)pos : -1);
        const int chunks = stride / 4, cph = chunks >= 2 ? chunks / 2 : 1;
        const int4 *src = reinterpret_cast<const int4 *>(nbr + (int64_t)(k >= 0 ? k : 0) * stride);
        int4 v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int ch = half * cph + i;
            v[i] = make_int4(-1, -1, -1, -1);
            if (k >= 0 && i < cph && ch < chunks) v[i] = src[ch];
        }
        uint32_t mm = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int ch = half * cph + i;
            if (i < cph && ch < chunks) {
                const int32_t e[4] = {v[i].x, v[i].y, v[i].z, v[i].w};
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int idx = ch * 4 + q;
                    // the row's offsets are read off its entries (the bitmask word of the table and
                    // the centre entry may not have been written yet: a map's row pass runs on demand)
                    if (idx < K3) {
                        const int32_t j = idx == centre ? k : (k >= 0 ? e[q] : -1);
                        lds_j[idx][col] = j;
                        if (j >= 0) mm |= 1u << idx;
                    }
                }
            }
        }
        for (int d = 32; d >= 1; d >>= 1) mm |= (uint32_t)__shfl_xor((int)mm, d, 64);
        if (lane == 0 && mm) atomicOr(&s_mask, mm);
    }
    __syncthreads();   // lds_j and s_mask complete
    const uint32_t mask = s_mask;

    if (mask) {
        // Iterator over the tile's (offset, chunk) pairs; a stage takes the next G of them.
        // Past the end it keeps returning the last pair with live = false (loads stay
        // unconditional and in bounds, the MFMAs are skipped).
        uint32_t rem = mask;
        int it_n = __builtin_ctz(rem), it_k = 0;
        bool it_live = true;
        rem &= rem - 1;
        auto next_pair = [&](int &n, int &k0, bool &live) {
            n = it_n;
            k0 = it_k;
            live = it_live;
            if (it_k + KC < cin) {
                it_k += KC;
            } else if (rem) {
                it_k = 0;
                it_n = __builtin_ctz(rem);
                rem &= rem - 1;
            } else {
                it_live = false;
            }
        };
        vec wreg[G][S::WV], bx_a[G][S::NKB], bx_b[G][S::NKB];
        int32_t j_a[G], j_b[G];
        bool live_a[G], live_b[G];
        auto issue_loads = [&](vec(&b)[G][S::NKB], int32_t(&j)[G], bool(&live)[G]) {
#pragma unroll
            for (int g = 0; g < G; ++g) {
                int n, k0;
                next_pair(n, k0, live[g]);
                load_w_regs<S, T>(wreg[g], Wt, n, co0, k0, cin, cout);
                j[g] = live[g] ? lds_j[n][slot] : -1;
                load_x_regs<S, T>(b[g], (j[g] >= 0 ? X + (int64_t)j[g] * cin + k0 : zero_row) + h * S::VEC);
            }
        };
        issue_loads(bx_a, j_a, live_a);
#pragma unroll
        for (int g = 0; g < G; ++g) store_w_regs<S, T>(wreg[g], lds_w[0][g]);
        int cur = 0;
        // One stage.  The two operand register sets swap roles between calls, so prefetched
        // registers are never copied (a copy would wait for the loads at once).
        auto stage = [&](vec(&b_now)[G][S::NKB], int32_t(&j_now)[G], bool(&live_now)[G], vec(&b_next)[G][S::NKB],
                         int32_t(&j_next)[G], bool(&live_next)[G]) -> bool {
            __syncthreads();   // slabs `cur` are complete; nobody still reads the other buffer
            const bool more = it_live;
            issue_loads(b_next, j_next, live_next);
#pragma unroll
            for (int g = 0; g < G; ++g)
                if (live_now[g] && __ballot(j_now[g] >= 0) != 0) mma_stage<S, T, NCB>(lds_w[cur][g], b_now[g], acc);
#pragma unroll
            for (int g = 0; g < G; ++g) store_w_regs<S, T>(wreg[g], lds_w[cur ^ 1][g]);
            cur ^= 1;
            return more;
        };
        for (;;) {
            if (!stage(bx_a, j_a, live_a, bx_b, j_b, live_b)) break;
            if (!stage(bx_b, j_b, live_b, bx_a, j_a, live_a)) break;
        }
    }
    {
        const int64_t pos = tile * kTileRows + slot;
        store_rows<T, NCB>(out, perm ? perm[pos] : (pos < n_out ? pos : -1), cout, co0, acc);
    }
}

typedef _Float16 half8v __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));   // native vector: arrays of it stay in registers

// Calls fn(std::integral_constant<int, 0>{}) ... fn(std::integral_constant<int, N-1>{}): the index
// is a constant expression inside fn, so arrays indexed with it stay in registers.
template <class Fn, int... I>
__device__ __forceinline__ void static_for_impl(Fn &&fn, std::integer_sequence<int, I...>) {
    (fn(std::integral_constant<int, I>{}), ...);
}
template <int N, class Fn>
__device__ __forceinline__ void static_for(Fn &&fn) {
    static_for_impl(fn, std::make_integer_sequence<int, N>{});
}

// Epilogue of k_conv_res and k_conv_direct.  A lane holds, per block of 16 output channels, channels 4 (l / 16) .. +3 of
// rows l % 16 and 16 + l % 16 of the wave's 32: stored from there, an instruction writes 32 bytes each of 16 rows, in
// 64 separate accesses.  Through LDS (16 rows at a time, `buf`: NCO KiB / 2 that only this wave touches, in k_conv_direct a part
// of the weight slabs, which are free by then; 16-byte units swizzled by row) rows leave, and the residual's come in, as
// whole lines.
template <int NCO>
struct RowStore {
    static constexpr int UPR = NCO * 2, PER = NCO / 2;   // 16-byte units per row; units per lane and half of the rows
    typedef _Float16 half8u __attribute__((ext_vector_type(8)));
    half4 sum[2][NCO];
    int32_t row[2][PER];
    half8u res[2][PER];
    __device__ __forceinline__ static int swizzle(int r) { return NCO % 4 == 0 ? r & 7 : r & 3; }
    // rows: the lane's two output rows (-1: none).  Takes the layer's own result, rounded once to fp16, and asks for
    // the residual.
    __device__ __forceinline__ void open(const floatx4 (&acc)[NCO][2], const int32_t (&rows)[2], const _Float16 *residual, int cout, int co0) {
#pragma unroll
        for (int c2 = 0; c2 < 2; ++c2)
#pragma unroll
            for (int cb = 0; cb < NCO; ++cb)
                sum[c2][cb] = half4{(_Float16)acc[cb][c2][0], (_Float16)acc[cb][c2][1], (_Float16)acc[cb][c2][2], (_Float16)acc[cb][c2][3]};
        int lane = threadIdx.x & 63;
        asm volatile("" : "+v"(lane));   // what follows from the lane number is worked out here, not kept through the stage loop
#pragma unroll
        for (int c2 = 0; c2 < 2; ++c2)
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                row[c2][i] = __shfl(rows[c2], (i * 64 + lane) / UPR, 64);
                if (residual && row[c2][i] >= 0)
                    res[c2][i] = *reinterpret_cast<const half8u *>(residual + (int64_t)row[c2][i] * cout + co0 + (i * 64 + lane) % UPR * 8);
            }
    }
    __device__ __forceinline__ void store(u32x4 *buf, _Float16 *out, const _Float16 *bias, bool residual,
                                          int relu, int cout, int co0) const {
        int lane = threadIdx.x & 63;
        asm volatile("" : "+v"(lane));
        const int m16 = lane & 15, g = lane >> 4;
#pragma unroll
        for (int c2 = 0; c2 < 2; ++c2) {
#pragma unroll
            for (int cb = 0; cb < NCO; ++cb)
                reinterpret_cast<half4 *>(buf + m16 * UPR + ((cb * 2 + (g >> 1)) ^ swizzle(m16)))[g & 1] = sum[c2][cb];
            __builtin_amdgcn_wave_barrier();   // LDS serves a wave's accesses in order
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                const int r = (i * 64 + lane) / UPR, c = (i * 64 + lane) % UPR;
                half8u v;
                const u32x4 raw = buf[r * UPR + (c ^ swizzle(r))];
                __builtin_memcpy(&v, &raw, 16);
                if (row[c2][i] < 0) continue;
                // if asked for, what ts_bias_act would do with it: fp32 sum, ReLU, one rounding
                if (bias || residual || relu) {
                    half8u bv;
                    if (bias) bv = *reinterpret_cast<const half8u *>(bias + co0 + c * 8);
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        float f = (float)v[e];
                        if (bias) f += (float)bv[e];
                        if (residual) f += (float)res[c2][i][e];
                        v[e] = (_Float16)(relu && f < 0.f ? 0.f : f);
                    }
                }
                *reinterpret_cast<half8u *>(out + (int64_t)row[c2][i] * cout + co0 + c * 8) = v;
            }
            __builtin_amdgcn_wave_barrier();
        }
    }
};

// ---- fused output-stationary kernel, fp16 -----------------------------------------------------------------
// D[co][m] += Wt[co][ci] * X[m][ci] with v_mfma_f32_16x16x32_f16.  A workgroup of four waves owns 128 output rows and
// 16 NCO output channels, a wave RB blocks of 16 rows and CB of 16 channels of them; a stage is one (offset, 32 KS
// channels), with HALF also the 32 channels that are left over at the end of a row.  The accumulators stay in registers
// across all stages; rows of an output are added in offset order whatever the tile holds, so results do not depend on how
// rows are grouped.
//
// What bounds it, and the layout that follows (MI355X, measured):
//  - A vector load costs the address unit 16 cycles per KiB when neighbouring lanes read neighbouring bytes, 40 to 48 when 16
//    neighbouring lanes are 16 rows, as an MFMA operand wants them (loads alone: 31 and 13 TB/s out of L2 over the chip; counted,
//    TA_BUSY by loads: 16 to 18 in this kernel, 25 in one whose rows are operands and whose weights are whole lines).  So the
//    rows of a stage go from memory straight into LDS, whole lines at a time (eight lanes a row of 64 channels), and operands
//    are read from there, 16-byte units being swizzled so that 16 lanes meet 16 different banks.  Rows for the next stage are
//    under way while this one is multiplied.  Only blocks of 16 rows that meet the offset are fetched, read and multiplied.
//  - Weights are not shared through LDS: in operand order a wave reads its own channels' as whole KiB, a stage ahead.
//  - The neighbour table's rows of a tile are brought into LDS the same way while the tile before is stored.
//  - A stage has one barrier and some 150 instructions around 16 to 32 MFMAs; three workgroups per CU are what hides that
//    (two: 15 to 20 % slower), so registers are held to 168.
//  - The next tile is asked for shortly before this one ends: asked for at its start, the workgroups with the longest
//    tiles took as many more as the others.
// Layers with their tail on kept maps, against a kernel that loaded rows as operands and weights through LDS (us; 64 -> 64,
// 128 -> 128, 96 -> 96): 153 k points of a scan 40 -> 28, 69 -> 51, 58 -> 49; 98 k of surfaces 32 -> 26, 63 -> 51, 47 -> 40;
// 1.53 M of scans 279 -> 249, 624 -> 516, 472 -> 454; 65 k after one halving 23 -> 20, 46 -> 41, 38 -> 31; 150 k scattered
// 33 -> 31, 73 -> 58, 59 -> 52.
// What is left at 64 channels on a map's first layer, 38 us: 1.6 times the matrix work there is (15 % of the cycles), the address
// unit busy 41 %, LDS 17 %, and 10 k instructions a SIMD, as many scalar ones as vector ones.  Stages of 96 channels also meet
// bank conflicts (44 % of their LDS cycles).

// A raw buffer descriptor for load_to_lds, in scalar registers.
__device__ __forceinline__ u32x4 lds_source(const void *p, int bytes) {
    const uint64_t a = reinterpret_cast<uint64_t>(p);
    return u32x4{(uint32_t)a, (uint32_t)(a >> 32) & 0xffffu, (uint32_t)bytes, 0x00020000u};
}

// 16 bytes per lane from a buffer straight into LDS, lane l's to dst + l (dst: the same in all lanes); an offset beyond the
// buffer gives zeros.  The compiler does not count this load: whoever reads dst has waited for it (vmcnt) himself.  (With
// the builtin, which it counts, it waits for all of them wherever one of them is issued under a condition.)
__device__ __forceinline__ void load_to_lds(const u32x4 &src, u32x4 *dst, int lane_offset, int offset) {
#ifdef __HIP_DEVICE_COMPILE__
    const uint32_t at = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void *)dst;
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" : : "s"(at), "v"(lane_offset), "s"(src), "s"(offset) : "memory", "m0");
#endif
}

// The same from an address of its own per lane.
__device__ __forceinline__ void load_to_lds(const void *src, u32x4 *dst) {
#ifdef __HIP_DEVICE_COMPILE__
    const uint32_t at = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void *)dst;
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(at), "v"(src) : "memory", "m0");
#endif
}

// A value whose origin the compiler does not see: what follows from it is worked out where it stands, and not kept in
// registers through the loops before.
__device__ __forceinline__ int fresh(int v) {
    asm volatile("" : "+v"(v));
    return v;
}

// Bitwise or over the 16 lanes of a row: rotations by 1, 2, 4 and 8 lanes.
__device__ __forceinline__ uint32_t or_row16(uint32_t v) {
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x121, 0xf, 0xf, false);
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x122, 0xf, 0xf, false);
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x124, 0xf, 0xf, false);
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x128, 0xf, 0xf, false);
    return v;
}

// Waits for this wave's vector memory, and for its LDS accesses too, in a form that the compiler counts with.
constexpr int kWaitVm0 = 0x0F70, kWaitAll = 0x0070;

// Waves that share the columns: with 8 blocks of output channels every wave takes all rows and 2 blocks; with fewer, two
// waves share rows, so that operands are read twice, not four times, and weights loaded twice.
template <int NCO, int KS, int GR = 1>
struct TileShape {
    static constexpr int WC = NCO == 8 ? 4 : 2, WR = kWaves / WC;
    static constexpr int RB = kTileRows / 16 / WR, CB = NCO / WC;
    static constexpr int GB = KS == 1 || (KS == 3 && NCO >= 6) ? 2 : 4;      // row blocks whose operands are read together
    static constexpr int UN = KS * 4;                            // 16-byte units of a row in a stage
    static constexpr int ROWS = kTileRows * UN;                  // units of a stage's rows
    static constexpr int UPR = NCO * 2;                          // units of a result row
    static constexpr int RESULT = kTileRows * UPR * (GR > 1 ? 2 : 1);   // units of a tile's results, or of its sums
    static constexpr int XROW = 2 * GR * ROWS > RESULT ? 2 * GR * ROWS : RESULT;
    static constexpr int WAVES_PER_EU = KS == 3 ? 2 : 3;
};

// GR > 1, for launches of hardly more than a workgroup a CU: GR groups of four waves have the tile together, each a share of the
// offsets, whose stages it walks with rows, weights and sums of its own; at the end the groups' sums are added through LDS, in
// the groups' order.  What binds such a launch is the chain of a tile's stages, in each of which four waves ask for rows and
// weights, read LDS and multiply one after the other, 1.0 to 2.1 us a stage whatever is in flight; three groups take three
// stages in hardly more than that, the work of one behind the loads of another.  (More stages in flight for the same four
// waves gained nothing: 128 channels a stage 32.6 us where the groups take 26.5.)  Which group has an offset does not hang on
// the tile, so that a row's sum does not.  Four groups gain another 3 % at up to 4 blocks of output channels and spill
// registers beyond; stages of 96 channels leave LDS for two.
// Layers on kept maps, rows from memory, one group or k_conv_direct -> groups (us; a scan after one halving | scattered):
// 64 -> 64 on 8 k rows 14.7 -> 11.4 | 15.0 -> 12.4, on 32 k 18.2 -> 15.1 | 20.1 -> 17.2; 96 -> 96 on 32 k 34.3 -> 23.9 | 32.0 -> 25.7;
// 128 -> 128 on 8 k 23.3 -> 18.0 | 23.7 -> 19.2, on 32 k 36.0 -> 29.0 | 37.5 -> 30.4; (96, 64) -> 96 on 8 k 40.0 -> 24.6 |
// 43.7 -> 26.7.

// Offsets of a 3x3x3 map by the sum of their steps modulo 3: a plane of nine has three in each share.
constexpr uint32_t share27(int q) {
    uint32_t m = 0;
    for (int n = 0; n < 27; ++n)
        if ((n / 9 + n / 3 % 3 + n % 3) % 3 == q) m |= 1u << n;
    return m;
}
constexpr uint32_t kShare0 = share27(0), kShare1 = share27(1), kShare2 = share27(2);

template <int NCO, int KS, bool TWO, bool HALF, int GR>
__global__ void __launch_bounds__(kThreads * GR) __attribute__((amdgpu_waves_per_eu(TileShape<NCO, KS, GR>::WAVES_PER_EU))) k_conv_tile(
    const _Float16 *__restrict__ X, const u32x4 *__restrict__ Wf, const int32_t *__restrict__ nbr, int row_shift,
    const int32_t *__restrict__ perm, int from_end, const int32_t *__restrict__ tile_order, int64_t n_out,
    _Float16 *__restrict__ out, int *__restrict__ sched, int cin, int cout, int K3, const _Float16 *__restrict__ bias,
    const _Float16 *__restrict__ residual, int relu, int x_bytes, int w_bytes, int centre, const _Float16 *__restrict__ X2,
    int x2_bytes, int cin1) {
    // TWO: the layer's input is the channel concatenation [X | X2], which is never formed: input channels below cin1 are
    // read from X (rows of cin1 channels), the others from X2 (rows of cin - cin1 channels); cin1 is a multiple of 32.
    // Otherwise X2, x2_bytes are unused and cin1 = cin.
    typedef TileShape<NCO, KS, GR> S;
    constexpr int TH = kThreads * GR, TABLE = (kTileRows * 8 + TH - 1) / TH;   // threads; table units of each
    constexpr int TR = kTileRows, WC = S::WC, RB = S::RB, CB = S::CB, GB = S::GB, UN = S::UN, UPR = S::UPR;
    constexpr int kAskAhead = 10;          // stages before the end of a tile that the next one is asked for
    constexpr int kNoRow = (int)0x80000000u;   // beyond any buffer this kernel is launched with
    __shared__ u32x4 xrow[S::XROW], tab[TR * 8];
    __shared__ int32_t s_row[2 * TR];
    __shared__ uint32_t s_m16[TR / 16];
    __shared__ int s_tile;
    // The launch holds as many workgroups as stay resident at once.  Workgroup b starts with tile b; the tiles beyond the
    // grid are handed out through counters, so nobody waits for a second round of workgroups.  One counter per XCD
    // (blockIdx % 8), on cache lines of their own: atomics on one address are served one after the other.  Longest tiles
    // come first, so that they do not start when everything else is done: by the order that the map build prepared (tiles
    // of rows in input order by descending number of offsets); rows sorted by bitmask put the tiles with the most offsets
    // last, so those are taken from the end.
    const int n_tiles = (int)((n_out + TR - 1) / TR);
    sched += kSchedWords * blockIdx.y;
    const int xcd = blockIdx.x & 7;
    const int wave_of_all = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), group = GR == 1 ? 0 : wave_of_all / kWaves, wave = wave_of_all - group * kWaves;
    const int lane = threadIdx.x & 63, m16 = lane & 15, g = lane >> 4;
    const int rows0 = GR == 1 ? 0 : group * (2 * S::ROWS);   // where the group's rows lie
    const int wr = wave / WC, wc = wave % WC;
    const int cblocks = cout / 16, nk = cin / 32, cb0 = blockIdx.y * NCO + wc * CB, co0 = blockIdx.y * (NCO * 16);
    const u32x4 xrsrc = lds_source(X, x_bytes), xrsrc2 = lds_source(TWO ? X2 : X, TWO ? x2_bytes : x_bytes);
    const __amdgpu_buffer_rsrc_t wrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<u32x4 *>(Wf), 0, w_bytes, 0x00020000);
    const int row_bytes = cin1 * 2, row_bytes2 = (cin - cin1) * 2;
    constexpr bool BY_STEP = KS != 2 || HALF;   // weights: 32 channels of every output block together, else 64
    const int nch1 = (cin1 + 63) / 64, nch = HALF ? nch1 + (cin - cin1 + 63) / 64 : nk / KS;   // stages per offset, with HALF those of X first

    // The neighbour table's rows of a tile lie in LDS as they do in memory, 1 << row_shift units of 16 bytes each, unit c of
    // row r at place c ^ (r % their number).  The lanes' rows are known a stage or more before they are needed.
    const int table_units = TR << row_shift, unit_mask = (1 << row_shift) - 1;
    int32_t kk[TABLE];
    auto rows_of = [&](int t) __attribute__((always_inline)) {
        const int l = fresh(threadIdx.x & 63);
        const int tile = from_end ? n_tiles - 1 - t : (tile_order ? tile_order[t] : t);
#pragma unroll
        for (int i = 0; i < TABLE; ++i) {
            const int u = (i * kWaves * GR + wave_of_all) * 64;
            kk[i] = -1;
            if (u < table_units) {
                const int64_t pos = (int64_t)tile * TR + ((u + l) >> row_shift);
                kk[i] = perm ? perm[pos] : (pos < n_out ? (int32_t)pos : -1);
            }
        }
    };
    auto fetch_table = [&](int rows) __attribute__((always_inline)) {
        const int l = fresh(threadIdx.x & 63);
#pragma unroll
        for (int i = 0; i < TABLE; ++i) {
            const int u = (i * kWaves * GR + wave_of_all) * 64;
            if (u < table_units) {
                const int r = (u + l) >> row_shift, c = (l ^ r) & unit_mask;
                if (kk[i] >= 0) load_to_lds(nbr + (((int64_t)kk[i] << row_shift) + c) * 4, tab + u);
                if ((l & unit_mask) == 0) s_row[rows + r] = kk[i];
            }
        }
    };
    int turn = blockIdx.x, then = n_tiles;
    if (turn < n_tiles) {
        rows_of(turn);
        fetch_table(0);
        __builtin_amdgcn_s_waitcnt(kWaitVm0);
        __syncthreads();
    }
    // A wave fetches the rows of two blocks of 16 (2 wave, 2 wave + 1), KS loads each: 16-byte unit v = 64 i + lane of load i
    // is place v % UN of row v / UN, and holds unit place ^ key(row) of the row.
    auto key = [](int r) __attribute__((always_inline)) { return KS == 2 ? r >> 1 & 7 : r >> 2 & 3; };
    int fetch_row[KS], fetch_at[KS];
#pragma unroll
    for (int i = 0; i < KS; ++i) {
        const int v = i * 64 + lane, r = v / UN;
        fetch_row[i] = wave * 32 + r;
        fetch_at[i] = ((v % UN) ^ key(r)) * 16;
    }
    // HALF: lanes that bring the second 32 channels of a stage
    int second[KS];
#pragma unroll
    for (int i = 0; i < KS; ++i) second[i] = HALF && fetch_at[i] >= 64 ? kNoRow : 0;
    // where the lane's operands lie: step ks of row block rb at read_at[ks] + rb * 16 * UN
    int read_at[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) read_at[ks] = (wr * RB * 16 + m16) * UN + ((ks * 4 + g) ^ key(m16));

    // Groups: an offset is the same group's in every tile, so that a row's sum does not hang on the tile it is in.
    auto share = [&](int q) __attribute__((always_inline)) -> uint32_t {
        if (GR == 1) return ~0u;
        if (GR == 2) return 0x55555555u << q;
        return K3 == 27 ? (q == 0 ? kShare0 : q == 1 ? kShare1 : kShare2) : 0x49249249u << q;
    };
    int rows_now = 0;   // where the tile's rows stand in s_row
    while (turn < n_tiles) {
        int ticket = 0;
        // The offsets that each block of 16 rows meets, read off the entries: two threads a row (the row's bitmask word and its
        // centre entry may not have been written yet, a map's row pass runs on demand).  What stays in LDS is where the input rows
        // begin, in bytes, or, of a two-part input, their numbers.
        if (GR == 1 || group == 0) {
            const int t = fresh(threadIdx.x), r = t >> 1, h = t & 1;
            const int32_t k = s_row[rows_now + r];
            uint32_t have = 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int c = 2 * i + h;
                if (c <= unit_mask) {
                    u32x4 &unit = tab[(r << row_shift) + (c ^ (r & unit_mask))];
                    u32x4 e = unit;
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int idx = c * 4 + q;
                        const int32_t j = k < 0 || idx >= K3 ? -1 : idx == centre ? k : (int32_t)e[q];
                        if (j >= 0) have |= 1u << idx;
                        e[q] = (uint32_t)(TWO ? j : j * row_bytes);   // (no row: -1, and a place beyond any buffer)
                    }
                    unit = e;
                }
            }
            have = or_row16(have);
            const uint32_t first = (uint32_t)__builtin_amdgcn_readlane((int)have, 0) | (uint32_t)__builtin_amdgcn_readlane((int)have, 16);
            const uint32_t second = (uint32_t)__builtin_amdgcn_readlane((int)have, 32) | (uint32_t)__builtin_amdgcn_readlane((int)have, 48);
            if (lane < 2) s_m16[wave * 2 + lane] = lane ? second : first;
        }
        __syncthreads();
        // Lane n: the row blocks that meet offset n, a bit each.
        uint32_t blocks = 0;
#pragma unroll
        for (int i = 0; i < TR / 16; ++i) blocks |= (s_m16[i] >> (lane & 31) & 1u) << i;
        const uint32_t mask = (uint32_t)__ballot(blocks != 0) & share(group);   // the offsets that the tile meets
        floatx4 acc[CB][RB];
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) acc[cb][rb] = floatx4{0.f, 0.f, 0.f, 0.f};
        const int own = __builtin_popcount(mask) * nch;   // stages of this group
        int nstage = own;                                 // and of the longest
        if constexpr (GR > 1) {
            const uint32_t all = (uint32_t)__ballot(blocks != 0);
#pragma unroll
            for (int q = 0; q < GR; ++q) nstage = max(nstage, __builtin_popcount(all & share(q)) * nch);
        }
        uint32_t rem = mask;
        int in = mask ? __builtin_ctz(mask) : 0, ich = 0;   // the stage whose loads are issued next
        auto advance = [&]() __attribute__((always_inline)) {
            if (++ich == nch) {
                ich = 0;
                if (rem & (rem - 1)) rem &= rem - 1;
                in = __builtin_ctz(rem | 0x80000000u);
            }
        };
        int32_t jn[2][KS];   // the input rows of that stage
        auto load_j = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < KS; ++i) {   // (16 rows on, a row's units stand in the same order)
                const int at = ((fetch_row[i] << row_shift) + ((in >> 2) ^ (fetch_row[i] & unit_mask))) * 4 + (in & 3);
                jn[0][i] = reinterpret_cast<const int32_t *>(tab)[at];
                jn[1][i] = reinterpret_cast<const int32_t *>(tab)[at + (64 << row_shift)];
            }
        };
        uint32_t met = 0;    // the row blocks of the stage being multiplied
        bool half = false;   // HALF: it is the last 32 channels of a row
        auto issue = [&](u32x4 (&a)[CB][KS], int rows) __attribute__((always_inline)) {
            met = (uint32_t)__builtin_amdgcn_readlane((int)blocks, in);
            // Which part the stage lies in, and where there, is settled once for all its loads, in scalar registers: asked load
            // by load, a lone workgroup's stage took 0.09 us longer ((64, 64) -> 64 on 4 k scattered points 32.4 -> 28.6 us).
            const int stage0 = ich * (KS * 32);
            const bool of_x2 = TWO && (HALF ? ich >= nch1 : stage0 >= cin1);
            const int c0 = HALF ? (of_x2 ? ich - nch1 : ich) * 64 : of_x2 ? stage0 - cin1 : stage0;   // its first channel, within the part
            const u32x4 src = of_x2 ? xrsrc2 : xrsrc;
            const int src_row = of_x2 ? row_bytes2 : row_bytes;
            // The last 32 channels of a row: of the other half of the stage there are neither weights nor rows, and what is
            // read beyond a buffer is zero.
            half = HALF && c0 * 2 + 64 == src_row;
            const int beyond = half ? kNoRow : 0;
            const int step = ((of_x2 ? cin1 : 0) + c0) >> 5;
            const int base = BY_STEP ? ((in * nk + step) * cblocks + cb0) * 1024 : ((in * nch + ich) * cblocks + cb0) * (KS * 1024);
            const int next_cb = BY_STEP ? 1024 : KS * 1024, next_ks = BY_STEP ? cblocks * 1024 : 1024;
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                for (int ks = 0; ks < KS; ++ks)
                    a[cb][ks] = __builtin_amdgcn_raw_buffer_load_b128(wrsrc, HALF && ks ? lane * 16 | beyond : lane * 16, base + cb * next_cb + ks * next_ks, 0);
            if (TWO && !HALF && !of_x2 && stage0 + KS * 32 > cin1) {   // the first channels of the stage from X, the others from X2
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    if (met >> (wave * 2 + h) & 1u) {
#pragma unroll
                        for (int i = 0; i < KS; ++i) {
                            u32x4 *dst = xrow + rows + (wave * 2 + h) * (16 * UN) + i * 64;
                            const int32_t j = jn[h][i];
                            if (c0 * 2 + fetch_at[i] < row_bytes) load_to_lds(xrsrc, dst, j * row_bytes + fetch_at[i], c0 * 2);
                            else load_to_lds(xrsrc2, dst, j * row_bytes2 + (c0 * 2 + fetch_at[i] - row_bytes), 0);
                        }
                    }
                return;
            }
#pragma unroll
            for (int h = 0; h < 2; ++h)
                if (met >> (wave * 2 + h) & 1u) {
#pragma unroll
                    for (int i = 0; i < KS; ++i)
                        load_to_lds(src, xrow + rows + (wave * 2 + h) * (16 * UN) + i * 64,
                                    ((TWO ? jn[h][i] * src_row : jn[h][i]) + fetch_at[i]) | (HALF ? second[i] & beyond : 0), c0 * 2);
                }
        };
        u32x4 a0[CB][KS], a1[CB][KS];
        auto stage = [&](int s, const u32x4 (&a)[CB][KS], u32x4 (&a_next)[CB][KS], int rows, int rows_next) __attribute__((always_inline)) {
            __builtin_amdgcn_s_waitcnt(kWaitAll);   // rows and weights of this stage
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_barrier();           // everybody's; and everybody has read the rows of the stage before
            asm volatile("" ::: "memory");
            const uint32_t now = GR == 1 || s < own ? met >> (wr * RB) : 0;
            const bool one_step = half;
            if (s + 1 < own) {
                issue(a_next, rows_next);
                advance();
                load_j();
            }
#pragma unroll
            for (int r0 = 0; r0 < RB; r0 += GB) {
                asm volatile("" ::: "memory");   // (one group's operands at a time)
                if ((now >> r0 & ((1u << GB) - 1)) == 0) continue;
                u32x4 b[GB][KS];
#pragma unroll
                for (int q = 0; q < GB; ++q)
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) b[q][ks] = xrow[rows + read_at[ks] + (r0 + q) * (16 * UN)];
                __builtin_amdgcn_s_setprio(1);
#pragma unroll
                for (int q = 0; q < GB; ++q)
                    if (now >> (r0 + q) & 1u) {
#pragma unroll
                        for (int ks = 0; ks < KS; ++ks) {
                            if (HALF && ks && one_step) continue;
                            half8v bv;
                            __builtin_memcpy(&bv, &b[q][ks], 16);
#pragma unroll
                            for (int cb = 0; cb < CB; ++cb) {
                                half8v av;
                                __builtin_memcpy(&av, &a[cb][ks], 16);
                                acc[cb][r0 + q] = __builtin_amdgcn_mfma_f32_16x16x32_f16(av, bv, acc[cb][r0 + q], 0, 0, 0);
                            }
                        }
                    }
                __builtin_amdgcn_s_setprio(0);
            }
        };
        if (own > 0) {
            load_j();
            issue(a0, rows0);
            advance();
            load_j();
        }
        int s = 0, until = nstage > kAskAhead ? (nstage - kAskAhead) & ~1 : 0;
#pragma nounroll
        for (int phase = 0; phase < 3; ++phase) {
#pragma nounroll
            for (; s < until && s < nstage; s += 2) {
                stage(s, a0, a1, rows0, rows0 + S::ROWS);
                if (s + 1 < nstage) stage(s + 1, a1, a0, rows0 + S::ROWS, rows0);
            }
            if (phase == 0) {
                if (threadIdx.x == 0) ticket = atomicAdd(&sched[xcd * 32], 1);
                until += 4;
            } else if (phase == 1) {
                if (threadIdx.x == 0) s_tile = ticket;
                __syncthreads();
                then = (int)gridDim.x + xcd + 8 * __builtin_amdgcn_readfirstlane(s_tile);
                if (then < n_tiles) rows_of(then);
                until = nstage;
            }
        }
        if (then < n_tiles) fetch_table(TR - rows_now);   // everybody has read the last of this tile's table

        if constexpr (GR > 1) {
            // the groups' sums, added in the groups' order
#pragma nounroll
            for (int q = 1; q < GR; ++q) {
                __syncthreads();   // everybody has read the last rows, or the sums before
                u32x4 *part = xrow + wave * (CB * RB * 64) + lane;
                if (group == q) {
#pragma unroll
                    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                        for (int rb = 0; rb < RB; ++rb) __builtin_memcpy(&part[(cb * RB + rb) * 64], &acc[cb][rb], 16);
                }
                __syncthreads();
                if (group == 0) {
#pragma unroll
                    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                        for (int rb = 0; rb < RB; ++rb) {
                            floatx4 v;
                            __builtin_memcpy(&v, &part[(cb * RB + rb) * 64], 16);
                            acc[cb][rb] += v;
                        }
                }
            }
        }
        // The sums, rounded once to fp16, go through LDS, so that rows leave, and the residual's come in, as whole lines.
        typedef _Float16 half8u __attribute__((ext_vector_type(8)));
        half4 sum[CB][RB];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) {
                sum[cb][rb] = half4{(_Float16)acc[cb][rb][0], (_Float16)acc[cb][rb][1], (_Float16)acc[cb][rb][2], (_Float16)acc[cb][rb][3]};
                asm volatile("" : "+v"(sum[cb][rb]));
            }
        // a thread stores unit c of rows r0, r0 + STEP, ...
        constexpr int STEP = TH / UPR, PER = (TR + STEP - 1) / STEP;
        const int tid = fresh(threadIdx.x), c = tid % UPR, r0 = tid / UPR;
        const uint32_t out_bytes = (uint32_t)cout * 2;
        const int col = (co0 + c * 8) * 2;
        int32_t row[PER];
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int r = r0 + i * STEP;
            row[i] = (STEP * UPR == TH || r0 < STEP) && (TR % STEP == 0 || r < TR) ? s_row[rows_now + r] : -1;
        }
        half8u res[PER];
#pragma unroll
        for (int i = 0; i < PER; ++i) res[i] = half8u{0, 0, 0, 0, 0, 0, 0, 0};   // (else their registers stay taken through the tile)
        if (residual) {
#pragma unroll
            for (int i = 0; i < PER; ++i)
                if (row[i] >= 0) res[i] = *reinterpret_cast<const half8u *>(reinterpret_cast<const char *>(residual) + (uint64_t)(uint32_t)row[i] * out_bytes + col);
        }
        __syncthreads();   // everybody has read the last rows
        auto swizzle = [](int r) __attribute__((always_inline)) { return NCO % 4 == 0 ? r & 7 : r & 3; };
        if (GR == 1 || group == 0) {
            const int m = tid & 15, q = tid >> 4 & 3;
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                for (int cb = 0; cb < CB; ++cb) {
                    const int r = (wr * RB + rb) * 16 + m;
                    reinterpret_cast<half4 *>(xrow + r * UPR + (((wc * CB + cb) * 2 + (q >> 1)) ^ swizzle(r)))[q & 1] = sum[cb][rb];
                }
        }
        __builtin_amdgcn_s_waitcnt(kWaitVm0);   // the next tile's table is there
        __syncthreads();
        half8u bv = {0, 0, 0, 0, 0, 0, 0, 0};
        if (bias) bv = *reinterpret_cast<const half8u *>(reinterpret_cast<const char *>(bias) + col);
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            if (row[i] < 0) continue;
            const int r = r0 + i * STEP;
            half8u v;
            const u32x4 raw = xrow[r * UPR + (c ^ swizzle(r))];
            __builtin_memcpy(&v, &raw, 16);
            // if asked for, what ts_bias_act would do with it: fp32 sum, ReLU, one rounding
            if (bias || residual || relu) {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    float f = (float)v[e];
                    if (bias) f += (float)bv[e];
                    if (residual) f += (float)res[i][e];
                    v[e] = (_Float16)(relu && f < 0.f ? 0.f : f);
                }
            }
            *reinterpret_cast<half8u *>(reinterpret_cast<char *>(out) + (uint64_t)(uint32_t)row[i] * out_bytes + col) = v;
        }
        turn = then;
        rows_now = TR - rows_now;
    }
    // the last workgroup to leave rearms the counters for the next launch on this map
    if (threadIdx.x == 0 && atomicAdd(&sched[8 * 32], 1) == (int)gridDim.x - 1) {
        for (int i = 0; i <= 8; ++i) sched[i * 32] = 0;
    }
}

// ---- the same layer with rows as operands, for launches of one to three workgroups a CU ------------------------------------
// D[co][m] as above, but a wave owns 32 rows and all 16 NCO channels, gathered rows go from memory straight into operand
// registers (4 lanes per 64 bytes of a row) two stages ahead, and the weights of a stage (one offset, 32 KSTEPS channels)
// through registers into LDS for the four waves.  Same bits as k_conv_tile.  Each load costs the address unit more, which
// decides nothing while a CU has one or two workgroups: those wait out every stage's loads, and two stages in flight with
// one short barrier each beat one stage ahead.  (Three groups of waves in a workgroup beat both while it has a CU to itself.)
// run_fused_f16 says which launches come here.
template <int NCO, int KSTEPS, int DEPTH, bool TWO>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(NCO * KSTEPS <= 8 && NCO < 8 ? 3 : 2))) k_conv_direct(const _Float16 *__restrict__ X, const u32x4 *__restrict__ Wf,
                                                        const int32_t *__restrict__ nbr, int stride,
                                                        const int32_t *__restrict__ perm, int from_end,
                                                        const int32_t *__restrict__ tile_order, int64_t n_out,
                                                        _Float16 *__restrict__ out, int *__restrict__ sched,
                                                        int cin, int cout, int K3, const _Float16 *__restrict__ bias,
                                                        const _Float16 *__restrict__ residual, int relu, int x_bytes,
                                                        int w_bytes, int centre, const _Float16 *__restrict__ X2,
                                                        int x2_bytes, int cin1) {
    // TWO: the layer's input is the channel concatenation [X | X2], which is never formed: input channels
    // below cin1 are read from X (rows of cin1 channels), the others from X2 (rows of cin - cin1 channels);
    // cin1 is a multiple of 32, so each 32-channel operand step lies in one of the two.  Otherwise X2,
    // x2_bytes are unused and cin1 = cin.
    constexpr int KC = KSTEPS * 32, FRAGS = NCO * KSTEPS, SLAB = FRAGS * 64;   // slab in 16-byte vectors
    constexpr int WV = (SLAB + kThreads - 1) / kThreads;
    __shared__ u32x4 lds_w[2][SLAB];
    __shared__ int32_t lds_j[kMaxK3][kTileRows], s_row[kTileRows];
    __shared__ uint32_t s_mask;
    __shared__ int s_tile;
    // The launch holds as many workgroups as stay resident at once.  Workgroup b starts with tile b;
    // the tiles beyond the grid are handed out through counters, so nobody waits for a second
    // round of workgroups.  One counter per XCD (blockIdx % 8), on cache lines of their own:
    // atomics on one address are served one after the other.
    const int64_t n_tiles = (n_out + kTileRows - 1) / kTileRows;
    sched += kSchedWords * blockIdx.y;
    const int xcd = blockIdx.x & 7;
    const int cb0 = blockIdx.y * NCO;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, m16 = lane & 15, g = lane >> 4;
    const int r0 = wave * kWaveRows + m16, r1 = r0 + 16;   // the lane's two output rows (tile slots)
    // Longest tiles first, so that they do not start when everything else is done: by the order
    // the map build prepared (tiles of rows in input order by descending number of offsets); rows
    // sorted by bitmask put the tiles with the most offsets last, so those are taken from the end.
    int64_t turn = blockIdx.x;
    // The rows of a tile, known one tile ahead (where they go through perm, that is a memory latency less per tile):
    // in the prologue, the 16-byte chunks of a table row go to neighbouring lanes, so that one load instruction
    // covers whole rows (a row touched by several instructions costs a request each).
    const int row_chunks = stride / 4;                                           // 8, 4 or 1 lanes per row
    const int row_ch = threadIdx.x % row_chunks, row_sub = threadIdx.x / row_chunks;
    const int rows_per_pass = kThreads / row_chunks;                             // 32, 64 or 256
    int32_t kk[4];                                                               // -2: no row of the tile in this pass
    auto rows_of = [&](int64_t t) __attribute__((always_inline)) {
        const int64_t tile = from_end ? n_tiles - 1 - t : (tile_order ? tile_order[t] : t);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int col = i * rows_per_pass + row_sub;
            const int64_t pos = tile * kTileRows + col;
            kk[i] = -2;
            if (col < kTileRows) kk[i] = perm ? perm[pos] : (pos < n_out ? (int32_t)pos : -1);
        }
    };
    if (turn < n_tiles) rows_of(turn);
    while (turn < n_tiles) {
    // ask for the next tile now; the answer is needed when this one is done
    int ticket = 0;
    if (threadIdx.x == 0) ticket = atomicAdd(&sched[xcd * 32], 1);

    // Neighbour rows of the tile's outputs -> LDS (offset-major), and the OR of their offset bitmasks.
    if (threadIdx.x == 0) s_mask = 0;
    __syncthreads();
    {
        int4 v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            v[i] = make_int4(-1, -1, -1, -1);
            if (kk[i] >= 0) v[i] = reinterpret_cast<const int4 *>(nbr + (int64_t)kk[i] * stride)[row_ch];
        }
        uint32_t mm = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (kk[i] == -2) continue;
            const int col = i * rows_per_pass + row_sub;
            const int32_t k = kk[i];
            if (row_ch == 0) s_row[col] = k;
            const int32_t e[4] = {v[i].x, v[i].y, v[i].z, v[i].w};
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int idx = row_ch * 4 + q;
                if (idx < K3) {
                    const int32_t j = idx == centre ? k : (k >= 0 ? e[q] : -1);
                    lds_j[idx][col] = j;
                    if (j >= 0) mm |= 1u << idx;
                }
            }
        }
        for (int d = 32; d >= 1; d >>= 1) mm |= (uint32_t)__shfl_xor((int)mm, d, 64);
        if (lane == 0 && mm) atomicOr(&s_mask, mm);
    }
    __syncthreads();
    // the offsets present in the tile, as a bitmask in a scalar register: the stages walk its set bits
    const uint32_t mask = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_mask);
    const int nchunks = cin / KC;
    const int nstage = __builtin_popcount(mask) * nchunks;
    const int cblocks = cout / 16;

    floatx4 acc[NCO][2];
#pragma unroll
    for (int cb = 0; cb < NCO; ++cb)
#pragma unroll
        for (int c2 = 0; c2 < 2; ++c2) acc[cb][c2] = floatx4{0.f, 0.f, 0.f, 0.f};

    u32x4 wreg[DEPTH][WV];
    half8v xreg[DEPTH][2][KSTEPS];
    bool xlive[DEPTH];
    // Issue the loads of stage s into register set d (d is a compile-time constant at every call).
    // Every call issues the same number of loads, unconditionally (past the last stage it repeats
    // that stage; rows without the offset read the zero row): the compiler counts outstanding
    // loads to place its waits, and a load it cannot count would make every wait a full drain.
    // Loads go through buffer descriptors: a 32-bit byte offset per lane plus a wave-uniform one, no
    // 64-bit address arithmetic in the loop, and an offset beyond the buffer reads as zero without
    // touching memory, which is what a row without the offset must contribute.  The loop body is
    // short on purpose: with ~200 vector instructions per stage around 16 MFMAs this kernel was
    // bound by instruction issue.
    const __amdgpu_buffer_rsrc_t xrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<_Float16 *>(X), 0, x_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t xrsrc2 = __builtin_amdgcn_make_buffer_rsrc(const_cast<_Float16 *>(TWO ? X2 : X), 0, TWO ? x2_bytes : x_bytes, 0x00020000);
    const int row_bytes2 = (cin - cin1) * 2;
    const __amdgpu_buffer_rsrc_t wrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<u32x4 *>(Wf), 0, w_bytes, 0x00020000);
    constexpr int kNoRow = (int)0x80000000u;   // beyond any buffer this kernel is launched with
    const int row_bytes = cin1 * 2, xlane = g * 16;
    // A fragment of the slab (16 output channels, 32 input channels) is 1 KiB; in memory the steps of a stage follow each
    // other, block by block of output channels.
    int wlane[WV], wslot[WV];
#pragma unroll
    for (int v = 0; v < WV; ++v) {
        int idx = threadIdx.x + v * kThreads;
        if (SLAB % kThreads != 0) idx = idx < SLAB ? idx : SLAB - 1;   // surplus threads repeat the last vector
        wslot[v] = idx;
        wlane[v] = KSTEPS == 3 ? (((idx >> 6) % KSTEPS * cblocks + (idx >> 6) / KSTEPS) * 64 + (idx & 63)) * 16 : idx * 16;
    }
    uint32_t it_rem = mask ? mask : 1u;   // offsets not issued yet; the lowest set bit is the one being issued
    int it_ch = 0;                        // its chunk
    // neighbour rows of the lane's two outputs for the stage issued next: read out of LDS one stage
    // ahead, so that no stage waits for them
    int32_t pj0 = lds_j[__builtin_ctz(it_rem)][r0], pj1 = lds_j[__builtin_ctz(it_rem)][r1];
    // Issue the loads of stage s into register set d (a compile-time constant at every call).
    // Every call issues the same loads, unconditionally (past the last stage it repeats that
    // stage): the compiler counts outstanding loads to place its waits, and a load it cannot count
    // makes every wait a full drain.
    auto issue = [&](int s, auto dc) __attribute__((always_inline)) {
        constexpr int d = decltype(dc)::value;
        const bool real = s < nstage;
        const int ch = it_ch, n = __builtin_ctz(it_rem);   // scalar: the weight slab's address stays in scalar registers
        const int32_t j0 = pj0, j1 = pj1;
        if (s + 1 < nstage) {   // stages are issued in order: step the pair, stay on the last one past the end
            if (++it_ch == nchunks) {
                it_ch = 0;
                it_rem &= it_rem - 1;
            }
        }
        pj0 = lds_j[__builtin_ctz(it_rem)][r0];
        pj1 = lds_j[__builtin_ctz(it_rem)][r1];
        const int wsoff = KSTEPS == 3 ? ((n * nchunks + ch) * KSTEPS * cblocks + cb0) * 1024 : ((n * nchunks + ch) * cblocks + cb0) * (KSTEPS * 1024);
#pragma unroll
        for (int v = 0; v < WV; ++v) wreg[d][v] = __builtin_amdgcn_raw_buffer_load_b128(wrsrc, wlane[v], wsoff, 0);
        xlive[d] = real && __ballot(j0 >= 0 || j1 >= 0) != 0;   // false: none of the wave's rows has this offset
        const int off0 = j0 >= 0 ? j0 * row_bytes + xlane : kNoRow;
        const int off1 = j1 >= 0 ? j1 * row_bytes + xlane : kNoRow;
        const int xsoff = ch * (KC * 2);
        int offb0 = 0, offb1 = 0;
        if constexpr (TWO) {
            offb0 = j0 >= 0 ? j0 * row_bytes2 + xlane : kNoRow;
            offb1 = j1 >= 0 ? j1 * row_bytes2 + xlane : kNoRow;
        }
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks) {
            u32x4 v0, v1;
            if constexpr (TWO) {
                const int c0 = ch * KC + ks * 32;        // first input channel of this operand step
                const bool second = c0 >= cin1;          // wave-uniform: the step lies in X2
                const int so = second ? (c0 - cin1) * 2 : c0 * 2;
                v0 = __builtin_amdgcn_raw_buffer_load_b128(second ? xrsrc2 : xrsrc, second ? offb0 : off0, so, 0);
                v1 = __builtin_amdgcn_raw_buffer_load_b128(second ? xrsrc2 : xrsrc, second ? offb1 : off1, so, 0);
            } else {
                v0 = __builtin_amdgcn_raw_buffer_load_b128(xrsrc, off0, xsoff + ks * 64, 0);
                v1 = __builtin_amdgcn_raw_buffer_load_b128(xrsrc, off1, xsoff + ks * 64, 0);
            }
            __builtin_memcpy(&xreg[d][0][ks], &v0, 16);
            __builtin_memcpy(&xreg[d][1][ks], &v1, 16);
        }
    };
    auto run = [&](int s, auto dc) __attribute__((always_inline)) {
        constexpr int d = decltype(dc)::value;
        u32x4 *slab = lds_w[s & 1];
#pragma unroll
        for (int v = 0; v < WV; ++v) slab[wslot[v]] = wreg[d][v];
        __syncthreads();   // slab complete; everybody is done with the other slab
        if (xlive[d]) {
#pragma unroll
            for (int ks = 0; ks < KSTEPS; ++ks) {
                // all weight fragments of the step out of LDS first, then the MFMAs: a read placed
                // right before its MFMA costs one LDS latency per fragment
                u32x4 raw[NCO];
#pragma unroll
                for (int cb = 0; cb < NCO; ++cb) raw[cb] = slab[(cb * KSTEPS + ks) * 64 + lane];
                __builtin_amdgcn_s_setprio(1);
#pragma unroll
                for (int cb = 0; cb < NCO; ++cb) {
                    half8v a;
                    __builtin_memcpy(&a, &raw[cb], 16);
                    acc[cb][0] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, xreg[d][0][ks], acc[cb][0], 0, 0, 0);
                    acc[cb][1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, xreg[d][1][ks], acc[cb][1], 0, 0, 0);
                }
                __builtin_amdgcn_s_setprio(0);
            }
        }
        issue(s + DEPTH, dc);
    };
    if (nstage > 0) {
        static_for<DEPTH>([&](auto dc) __attribute__((always_inline)) { issue(decltype(dc)::value, dc); });
        // whole rounds of DEPTH stages; stages past the end only repeat loads and skip the MFMAs
        for (int s0 = 0; s0 < nstage; s0 += DEPTH) static_for<DEPTH>([&](auto dc) __attribute__((always_inline)) { run(s0 + decltype(dc)::value, dc); });
    }

    const int32_t out_row[2] = {s_row[r0], s_row[r1]};
    RowStore<NCO> rows;
    rows.open(acc, out_row, residual, cout, cb0 * 16);
    if (threadIdx.x == 0) s_tile = ticket;
    __syncthreads();   // the tile's LDS is free; s_tile is set
    turn = (int64_t)gridDim.x + xcd + 8 * (int64_t)s_tile;
    if (turn < n_tiles) rows_of(turn);
    // (the pointer is made opaque per tile: loads the compiler can prove the same for every tile move to the
    // top of the kernel and hold registers through the stage loop, which has none to spare)
    const _Float16 *bp = bias;
    asm volatile("" : "+s"(bp));
    rows.store(&lds_w[0][0] + wave * (NCO * 32), out, bp, residual != nullptr, relu, cout, cb0 * 16);
    }
    // the last workgroup to leave rearms the counters for the next launch on this map
    if (threadIdx.x == 0 && atomicAdd(&sched[8 * 32], 1) == (int)gridDim.x - 1) {
        for (int i = 0; i <= 8; ++i) sched[i * 32] = 0;
    }
}

// ---- fused kernel for narrow layers: all weights resident in LDS -----------------------------------
// With C_in = 32 KSTEPS and a slice of 16 NCO output channels the weights, in operand order, are
// K^3 NCO KSTEPS KiB (used with C_in <= 32 and C_out = 32 or 64: 54 or 108 KiB):
// it is loaded into LDS once per workgroup and stays.  Nothing is shared between waves after that,
// so there is no barrier in the loop and the unit of work is a wave's own 32 output rows: its
// neighbour rows sit in a slice of LDS that only this wave touches, the offsets it walks are the
// ones its own 32 rows have (fewer than a 128-row tile has), and units are handed to waves, not to
// workgroups.  Operand layout, accumulation order (offsets ascending per output) and epilogue are
// those of k_conv_tile: the two kernels give the same bits.
// (8 to 16 waves per workgroup and 2 to 8 stages of loads in flight all land within 10 % of each other on
// 153 k points; 12 waves with 3 stages was the fastest.)
constexpr int kResWaves = 12, kResDepth = 3, kResThreads = kResWaves * 64, kResRows = 32;
template <int FRAGS>
constexpr size_t res_lds_bytes() {
    return (size_t)kMaxK3 * FRAGS * 64 * 16 + (size_t)kResWaves * kMaxK3 * kResRows * 4;
}

template <int NCO, int KSTEPS, int DEPTH>
__global__ void __launch_bounds__(kResThreads) k_conv_res(const _Float16 *__restrict__ X, const u32x4 *__restrict__ Wf,
                                                          const int32_t *__restrict__ nbr, int stride,
                                                          const int32_t *__restrict__ perm, int64_t n_out,
                                                          _Float16 *__restrict__ out, int *__restrict__ sched, int K3, int cout,
                                                          const _Float16 *__restrict__ bias,
                                                          const _Float16 *__restrict__ residual, int relu, int x_bytes,
                                                          int centre) {
    extern __shared__ u32x4 lds_res[];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, m16 = lane & 15, g = lane >> 4;
    constexpr int FRAGS = NCO * KSTEPS;
    const int cb0 = blockIdx.y * NCO, cblocks = cout / 16;
    sched += kSchedWords * blockIdx.y;
    u32x4 *lds_w = lds_res;                                                         // [K3][NCO][KSTEPS][64]
    int32_t *lds_j = reinterpret_cast<int32_t *>(lds_res + kMaxK3 * FRAGS * 64) + wave * (kMaxK3 * kResRows);   // [K3][32], this wave's
    // the fragments of this slice of output channels are contiguous within an offset
    for (int i = threadIdx.x; i < K3 * FRAGS * 64; i += kResThreads) {
        const int n = i / (FRAGS * 64), rem = i % (FRAGS * 64);
        lds_w[i] = Wf[(n * cblocks + cb0) * KSTEPS * 64 + rem];
    }
    __syncthreads();

    constexpr int row_bytes = KSTEPS * 64;
    const int64_t n_units = (n_out + kResRows - 1) / kResRows;
    const int64_t n_waves = (int64_t)gridDim.x * kResWaves;
    const int xcd = blockIdx.x & 7;
    const int r0 = m16, r1 = m16 + 16;
    const __amdgpu_buffer_rsrc_t xrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<_Float16 *>(X), 0, x_bytes, 0x00020000);
    constexpr int kNoRow = (int)0x80000000u;
    const int xlane = g * 16;
    // A wave starts with unit (its index in the launch); the units beyond the launch come from the
    // per-XCD counters, as tiles do in k_conv_tile.
    int64_t turn = (int64_t)blockIdx.x * kResWaves + wave;
    while (turn < n_units) {
        const int64_t unit = perm ? n_units - 1 - turn : turn;
        int ticket = 0;
        if (lane == 0) ticket = atomicAdd(&sched[xcd * 32], 1);
        uint32_t mm = 0;
        {
            const int chunks = stride / 4;                       // 8, 4 or 1 lanes per table row
            const int ch = lane % chunks, sub = lane / chunks;
            const int rows_per_pass = 64 / chunks;               // 8, 16 or 64
            int4 v[4];
            int32_t kk[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int col = i * rows_per_pass + sub;
                const int64_t pos = unit * kResRows + col;
                kk[i] = -2;                                      // -2: no row of the unit in this pass
                if (col < kResRows) kk[i] = perm ? perm[pos] : (pos < n_out ? (int32_t)pos : -1);
                v[i] = make_int4(-1, -1, -1, -1);
                if (kk[i] >= 0) v[i] = reinterpret_cast<const int4 *>(nbr + (int64_t)kk[i] * stride)[ch];
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (kk[i] == -2) continue;
                const int col = i * rows_per_pass + sub;
                const int32_t k = kk[i];
                const int32_t e[4] = {v[i].x, v[i].y, v[i].z, v[i].w};
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int idx = ch * 4 + q;
                    if (idx < K3) {
                        const int32_t j = idx == centre ? k : (k >= 0 ? e[q] : -1);
                        lds_j[idx * kResRows + col] = j;
                        if (j >= 0) mm |= 1u << idx;
                    }
                }
            }
            for (int d = 32; d >= 1; d >>= 1) mm |= (uint32_t)__shfl_xor((int)mm, d, 64);
        }
        // LDS serves a wave's accesses in order: what its lanes wrote above is what they read below
        __builtin_amdgcn_wave_barrier();
        const uint32_t mask = (uint32_t)__builtin_amdgcn_readfirstlane((int)mm);
        const int nstage = __builtin_popcount(mask);

        floatx4 acc[NCO][2];
#pragma unroll
        for (int cb = 0; cb < NCO; ++cb)
#pragma unroll
            for (int c2 = 0; c2 < 2; ++c2) acc[cb][c2] = floatx4{0.f, 0.f, 0.f, 0.f};
        half8v xreg[DEPTH][2][KSTEPS];
        int nn[DEPTH];
        bool xlive[DEPTH];
        uint32_t it_rem = mask ? mask : 1u;
        int32_t pj0 = lds_j[__builtin_ctz(it_rem) * kResRows + r0], pj1 = lds_j[__builtin_ctz(it_rem) * kResRows + r1];
        // the same loads at every call (past the last stage they repeat it), so the compiler can count them
        auto issue = [&](int s, auto dc) __attribute__((always_inline)) {
            constexpr int d = decltype(dc)::value;
            xlive[d] = s < nstage;
            nn[d] = __builtin_ctz(it_rem);
            const int32_t j0 = pj0, j1 = pj1;
            if (s + 1 < nstage) it_rem &= it_rem - 1;
            pj0 = lds_j[__builtin_ctz(it_rem) * kResRows + r0];
            pj1 = lds_j[__builtin_ctz(it_rem) * kResRows + r1];
            const int off0 = j0 >= 0 ? j0 * row_bytes + xlane : kNoRow;
            const int off1 = j1 >= 0 ? j1 * row_bytes + xlane : kNoRow;
#pragma unroll
            for (int ks = 0; ks < KSTEPS; ++ks) {
                const u32x4 v0 = __builtin_amdgcn_raw_buffer_load_b128(xrsrc, off0, ks * 64, 0);
                const u32x4 v1 = __builtin_amdgcn_raw_buffer_load_b128(xrsrc, off1, ks * 64, 0);
                __builtin_memcpy(&xreg[d][0][ks], &v0, 16);
                __builtin_memcpy(&xreg[d][1][ks], &v1, 16);
            }
        };
        auto run = [&](int s, auto dc) __attribute__((always_inline)) {
            constexpr int d = decltype(dc)::value;
            if (xlive[d]) {
                u32x4 raw[NCO][KSTEPS];
#pragma unroll
                for (int cb = 0; cb < NCO; ++cb)
#pragma unroll
                    for (int ks = 0; ks < KSTEPS; ++ks) raw[cb][ks] = lds_w[((nn[d] * NCO + cb) * KSTEPS + ks) * 64 + lane];
#pragma unroll
                for (int ks = 0; ks < KSTEPS; ++ks)
#pragma unroll
                    for (int cb = 0; cb < NCO; ++cb) {
                        half8v a;
                        __builtin_memcpy(&a, &raw[cb][ks], 16);
                        acc[cb][0] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, xreg[d][0][ks], acc[cb][0], 0, 0, 0);
                        acc[cb][1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, xreg[d][1][ks], acc[cb][1], 0, 0, 0);
                    }
            }
            issue(s + DEPTH, dc);
        };
        if (nstage > 0) {
            static_for<DEPTH>([&](auto dc) __attribute__((always_inline)) { issue(decltype(dc)::value, dc); });
            for (int s0 = 0; s0 < nstage; s0 += DEPTH) static_for<DEPTH>([&](auto dc) __attribute__((always_inline)) { run(s0 + decltype(dc)::value, dc); });
        }
        // the reads of lds_j issued last belong to no stage: they must have returned before the next unit overwrites it
        __builtin_amdgcn_wave_barrier();

        int32_t out_row[2];
#pragma unroll
        for (int c2 = 0; c2 < 2; ++c2) {
            const int64_t pos = unit * kResRows + (c2 ? r1 : r0);
            out_row[c2] = perm ? perm[pos] : (pos < n_out ? (int32_t)pos : -1);
        }
        RowStore<NCO> rows;
        rows.open(acc, out_row, residual, cout, cb0 * 16);
        rows.store(reinterpret_cast<u32x4 *>(lds_j), out, bias, residual != nullptr, relu, cout, cb0 * 16);
        ticket = __builtin_amdgcn_readfirstlane(ticket);
        turn = n_waves + xcd + 8 * (int64_t)ticket;
    }
    __syncthreads();   // all waves of the workgroup are done
    // the last workgroup to leave rearms the counters for the next launch on this map
    if (threadIdx.x == 0 && atomicAdd(&sched[8 * 32], 1) == (int)gridDim.x - 1) {
        for (int i = 0; i <= 8; ++i) sched[i * 32] = 0;
    }
}

// Weights in the operand order of k_conv_tile:
// Wf[n][chunk][cb][ks][lane][e] = W[n][ci][co], co = cb*16 + lane%16, ci = chunk*KC + ks*32 + 8*(lane/16) + e
// (0 for ci >= cin).  One (n, chunk, cb, ks) fragment is 64 lanes x 16 bytes, contiguous.
__global__ void k_pack_weights_tile(const _Float16 *__restrict__ W, _Float16 *__restrict__ Wf, int K3, int cin,
                                    int cin_pad, int cout, int ksteps) {
    const int64_t gidx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t total = (int64_t)K3 * cout * cin_pad;
    if (gidx >= total) return;
    const int kc = ksteps * 32, nchunks = cin_pad / kc, cblocks = cout / 16;
    int64_t r = gidx;
    const int e = (int)(r % 8); r /= 8;
    const int lane = (int)(r % 64); r /= 64;
    const int ks = (int)(r % ksteps); r /= ksteps;
    const int cb = (int)(r % cblocks); r /= cblocks;
    const int chunk = (int)(r % nchunks); r /= nchunks;
    const int n = (int)r;
    const int co = cb * 16 + (lane & 15);
    const int ci = chunk * kc + ks * 32 + 8 * (lane >> 4) + e;
    Wf[gidx] = ci < cin ? W[((int64_t)n * cin + ci) * cout + co] : (_Float16)0;
}

// ---- explicit dataflow ------------------------------------------------------------------------
// Gather (Alg. 2, "F[m] <- X_in[j]") for all offsets: a thread moves kGatherPer 16-byte vectors,
// one each of rows a workgroup-stride apart, all loaded before the first store.  F is written
// once and read once by the matmul, so its stores bypass the caches and leave them to X, every row
// of which is gathered several times.
constexpr int kGatherPer = 2;
__global__ void __launch_bounds__(kThreads) k_gather(const u32x4 *__restrict__ X, const int32_t *__restrict__ in_idx,
                                                     u32x4 *__restrict__ F, int64_t M, int vec_per_row, int64_t skip_lo,
                                                     int64_t skip_hi) {
    const int64_t base = (int64_t)blockIdx.x * (kThreads * kGatherPer) + threadIdx.x;
    u32x4 v[kGatherPer];
    int64_t at[kGatherPer];
#pragma unroll
    for (int u = 0; u < kGatherPer; ++u) {
        const int64_t g = base + (int64_t)u * kThreads;
        const int64_t p = g / vec_per_row;
        const int c = (int)(g - p * vec_per_row);
        at[u] = (p < M && !(p >= skip_lo && p < skip_hi)) ? g : -1;
        if (at[u] >= 0) v[u] = X[(int64_t)in_idx[p] * vec_per_row + c];
    }
#pragma unroll
    for (int u = 0; u < kGatherPer; ++u)
        if (at[u] >= 0) __builtin_nontemporal_store(v[u], &F[at[u]]);
}

// The same gather in input-stationary order (the locality-aware order of Sec. 4.3.2: an input row is read
// once and written to every place it is needed), for 3x3x3 stride-1 maps.  VPR lanes share an input row j
// and hold 16 bytes of it each.  By the symmetry of Sec. 4.2.1 row j of the out-major table also lists
// where j is an input: nbr[j][n'] = k means input j feeds output k through offset n = 26 - n', and that
// pair's row in F is offs[n] + (rank of k among the outputs with offset n), read off the rank bitmaps.
// The lanes of a group first work out those rows for the offsets they own (n' = c, c + VPR, ...), all
// lookups in flight together, then the group walks the 27 offsets and stores.  Reads X sequentially and
// once; F's rows are written whole but scattered.  Centre rows are left out, as in k_gather.
template <int VPR>
__global__ void __launch_bounds__(kThreads) k_gather_in(const u32x4 *__restrict__ X, const int32_t *__restrict__ nbr,
                                                        const uint64_t *__restrict__ colbits,
                                                        const int32_t *__restrict__ colbase, Offs offs, int64_t n_blocks,
                                                        u32x4 *__restrict__ F, int64_t n_in) {
    constexpr int K3 = 27, STRIDE = 32, PER = (K3 + VPR - 1) / VPR;
    const int64_t t = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    const int64_t j = t / VPR;
    const int c = (int)(t % VPR), lane = threadIdx.x & 63, first = lane - c;   // first: the group's lane 0
    const bool ok = j < n_in;
    u32x4 v = {0u, 0u, 0u, 0u};
    if (ok) v = X[j * VPR + c];
    int32_t pos[PER];
#pragma unroll
    for (int r = 0; r < PER; ++r) {
        const int np = c + r * VPR;     // this lane's offset n' of row j
        pos[r] = -1;
        if (ok && np < K3 && np != K3 / 2) {
            const int32_t k = nbr[j * STRIDE + np];
            if (k >= 0) {
                const int n = K3 - 1 - np;
                const int64_t b = (int64_t)n * n_blocks + (k >> 6);
                pos[r] = offs.v[n] + colbase[b] + __popcll(colbits[b] & ((1ull << (k & 63)) - 1ull));
            }
        }
    }
#pragma unroll
    for (int np = 0; np < K3; ++np) {
        const int32_t p = __shfl(pos[np / VPR], first + np % VPR, 64);
        if (p >= 0) __builtin_nontemporal_store(v, &F[(int64_t)p * VPR + c]);
    }
}

// One launch of the grouped matmul: the offsets it covers and how many 128-row blocks each gets.
// An offset given more blocks than its list fills stands for a list padded to a longer one
// (the batched matmul of Appendix B, Alg. 4): the surplus blocks multiply zero rows and store nothing.
struct MmPlan {
    int32_t count;
    int32_t n[kMaxK3];
    int32_t tiles[kMaxK3];
};

// Grouped matmul: block -> (offset n, 128-row block) by walking the plan's block counts.
// Rows of the centre offset of an identity map come from X itself.  Rows past the end of an
// offset's list read `zero_row` and are not stored.
template <class T, int NCB, int KC>
__global__ void __launch_bounds__(kThreads) k_grouped_mm(const T *__restrict__ F, const T *__restrict__ X,
                                                         const T *__restrict__ Wt, Offs offs, MmPlan plan,
                                                         float *__restrict__ G, const T *__restrict__ zero_row,
                                                         int cin, int cout, int centre,
                                                         const int32_t *__restrict__ in_idx,
                                                         const T *__restrict__ X2, int cin1) {
    // X2 != nullptr (rows fetched through the map only: F is not used then): the input is the channel
    // concatenation [X | X2], never formed; channels below cin1 come from X, the others from X2.
    typedef Shape<T, NCB, KC> S;
    typedef typename S::vec vec;
    __shared__ __attribute__((aligned(16))) T lds_w[S::SLAB];
    int t = blockIdx.x, i = 0;
    for (; i < plan.count; ++i) {
        if (t < plan.tiles[i]) break;
        t -= plan.tiles[i];
    }
    if (i >= plan.count) return;
    const int n = plan.n[i];
    const int lo = offs.v[n], hi = offs.v[n + 1];
    const int co0 = blockIdx.y * NCB * 32;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, m = lane & 31, h = lane >> 5;
    const int64_t p = (int64_t)lo + (int64_t)t * kTileRows + wave * kWaveRows + m;   // row of F and G
    const bool valid = p < hi;
    const int64_t j = !valid ? 0 : (n == centre ? p - lo : (in_idx ? (int64_t)in_idx[p] : p));
    const T *src = !valid ? zero_row : ((n == centre || in_idx) ? X + j * cin1 : F + p * cin);
    const T *src2 = (!valid || !X2) ? zero_row : X2 + j * (cin - cin1) - cin1;   // indexed with k0 >= cin1
    const int kstride = valid ? 1 : 0;   // the zero row is one chunk long
    floatx16 acc[NCB];
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb)
        for (int r = 0; r < 16; ++r) acc[cb][r] = 0.f;
    vec wreg[S::WV], bx[S::NKB];
    for (int k0 = 0; k0 < cin; k0 += KC) {
        load_w_regs<S, T>(wreg, Wt, n, co0, k0, cin, cout);
        load_x_regs<S, T>(bx, (k0 < cin1 ? src : src2) + k0 * kstride + h * S::VEC);
        __syncthreads();
        store_w_regs<S, T>(wreg, lds_w);
        __syncthreads();
        mma_stage<S, T, NCB>(lds_w, bx, acc);
    }
    store_rows<float, NCB>(G, valid ? p : -1, cout, co0, acc);
}

// The same matmul for fp16 rows of a multiple of 64 channels, the way k_conv_tile reads its operands: rows as whole lines
// into LDS, a stage of 64 channels ahead, weights in operand order as whole KiB per wave.  The kernel above asks for 32
// rows an instruction, which costs the address unit four times what whole lines cost, and waits for every stage's loads.
// Blocks of 16 rows past the end of a list are not multiplied; the sums leave as whole lines through the LDS that only
// their wave touches.  What bounds it now: the fp32 sums on their way to memory and back (64 MB each way for 62 k pairs
// of 256 channels).  Layers, before -> after, us: 256 -> 256 on 8 k points 40.1 -> 33.5, (256, 256) -> 256 51.9 -> 42.1,
// (128, 128) -> 128 on 22 k points 51.1 -> 45.3, 256 -> 256 on 2.7 k points 24.0 -> 22.0, 2x2x2 of 256 -> 256 channels
// from 8 k points 16.0 -> 15.4.
template <int NCO, bool TWO>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(3))) k_grouped_lines(
    const _Float16 *__restrict__ F, const _Float16 *__restrict__ X, const u32x4 *__restrict__ Wf, Offs offs, MmPlan plan,
    float *__restrict__ G, int cin, int cout, int centre, const int32_t *__restrict__ in_idx, int x_bytes, int w_bytes,
    const _Float16 *__restrict__ X2, int x2_bytes, int cin1, int slices_first) {
    typedef TileShape<NCO, 2> S;
    constexpr int WC = S::WC, RB = S::RB, CB = S::CB, GB = S::GB, ROWS = S::ROWS;
    __shared__ u32x4 xrow[2 * ROWS];
    const int slice = slices_first ? blockIdx.x : blockIdx.y;
    int t = slices_first ? blockIdx.y : blockIdx.x, i = 0;
    for (; i < plan.count; ++i) {
        if (t < plan.tiles[i]) break;
        t -= plan.tiles[i];
    }
    if (i >= plan.count) return;
    const int n = plan.n[i];
    const int lo = offs.v[n], hi = offs.v[n + 1], p0 = lo + t * kTileRows, rows = hi - p0;   // rows of the list in this tile, if positive
    if (rows <= 0) return;   // a batched launch pads lists to the longest: nothing to store, and F may end before p0
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, m16 = lane & 15, g = lane >> 4;
    const int wr = wave / WC, wc = wave % WC;
    const int cblocks = cout / 16, nch = cin / 64, cb0 = slice * NCO + wc * CB;
    const bool whole = n == centre || in_idx;   // rows of X, wherever they are; else F's own, one after the other
    const int valid = rows < kTileRows ? rows : kTileRows;
    const u32x4 xrsrc = whole ? lds_source(X, x_bytes) : lds_source(F + (int64_t)p0 * cin, valid * cin * 2);
    const u32x4 xrsrc2 = lds_source(TWO ? X2 : X, TWO ? x2_bytes : 0);
    const __amdgpu_buffer_rsrc_t wrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<u32x4 *>(Wf), 0, w_bytes, 0x00020000);
    const int row_bytes = cin1 * 2, row_bytes2 = (cin - cin1) * 2;
    int at[4], at2[4];   // where in X, and X2, the lane's 16 bytes of its four rows begin; no row: beyond any buffer
#pragma unroll
    for (int l = 0; l < 4; ++l) {
        const int r = wave * 32 + l * 8 + (lane >> 3), unit = ((lane & 7) ^ (lane >> 4) ^ (l & 1) * 4) * 16;
        const int j = r >= valid ? -1 : n == centre ? p0 - lo + r : in_idx ? in_idx[p0 + r] : r;
        at[l] = j * row_bytes + unit;
        at2[l] = j * row_bytes2 + unit;
    }
    const int read_at[2] = {(wr * RB * 16 + m16) * 8 + (g ^ (m16 >> 1)), (wr * RB * 16 + m16) * 8 + (g ^ (m16 >> 1) ^ 4)};
    floatx4 acc[CB][RB];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) acc[cb][rb] = floatx4{0.f, 0.f, 0.f, 0.f};
    auto issue = [&](int ch, u32x4 (&a)[CB][2], int into) __attribute__((always_inline)) {
        const int base = ((n * nch + ch) * cblocks + cb0) * 2048, c0 = ch * 64;
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) a[cb][ks] = __builtin_amdgcn_raw_buffer_load_b128(wrsrc, lane * 16, base + (cb * 2 + ks) * 1024, 0);
#pragma unroll
        for (int l = 0; l < 4; ++l) {
            u32x4 *dst = xrow + into + wave * 256 + l * 64;
            if (!TWO || c0 < cin1) load_to_lds(xrsrc, dst, at[l], c0 * 2);
            else load_to_lds(xrsrc2, dst, at2[l], (c0 - cin1) * 2);
        }
    };
    const int blocks = (valid + 15) / 16 - wr * RB;   // blocks of 16 rows that are this wave's, counted from its first
    auto stage = [&](int ch, const u32x4 (&a)[CB][2], u32x4 (&a_next)[CB][2], int from, int into) __attribute__((always_inline)) {
        __builtin_amdgcn_s_waitcnt(kWaitAll);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if (ch + 1 < nch) issue(ch + 1, a_next, into);
#pragma unroll
        for (int r0 = 0; r0 < RB; r0 += GB) {
            asm volatile("" ::: "memory");
            if (blocks <= r0) continue;
            u32x4 b[GB][2];
#pragma unroll
            for (int q = 0; q < GB; ++q)
#pragma unroll
                for (int ks = 0; ks < 2; ++ks) b[q][ks] = xrow[from + read_at[ks] + (r0 + q) * 128];
#pragma unroll
            for (int q = 0; q < GB; ++q)
                if (r0 + q < blocks) {
#pragma unroll
                    for (int ks = 0; ks < 2; ++ks) {
                        half8v bv;
                        __builtin_memcpy(&bv, &b[q][ks], 16);
#pragma unroll
                        for (int cb = 0; cb < CB; ++cb) {
                            half8v av;
                            __builtin_memcpy(&av, &a[cb][ks], 16);
                            acc[cb][r0 + q] = __builtin_amdgcn_mfma_f32_16x16x32_f16(av, bv, acc[cb][r0 + q], 0, 0, 0);
                        }
                    }
                }
        }
    };
    u32x4 a0[CB][2], a1[CB][2];
    issue(0, a0, 0);
    for (int ch = 0; ch < nch; ch += 2) {
        stage(ch, a0, a1, 0, ROWS);
        if (ch + 1 < nch) stage(ch + 1, a1, a0, ROWS, 0);
    }
    __syncthreads();   // everybody has read the last rows
    // 16 rows of the wave's CB blocks at a time: written as the accumulators lie, read as lines
    u32x4 *buf = xrow + wave * (CB * 64);
    constexpr int UPR = CB * 4;                       // 16-byte units of a row
    const int col = cb0 * 16;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        if (rb >= blocks) break;
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
            u32x4 v;
            __builtin_memcpy(&v, &acc[cb][rb], 16);
            buf[m16 * UPR + ((cb * 4 + g) ^ (m16 & 3))] = v;
        }
        __builtin_amdgcn_wave_barrier();   // LDS serves a wave's accesses in order
#pragma unroll
        for (int l = 0; l < CB; ++l) {
            const int u = l * 64 + lane, r = u / UPR, c = u % UPR, row = (wr * RB + rb) * 16 + r;
            const u32x4 v = buf[r * UPR + (c ^ (r & 3))];
            if (row < valid) *reinterpret_cast<u32x4 *>(G + (int64_t)(p0 + row) * cout + col + c * 4) = v;
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// Scatter-accumulate, output-stationary: thread = (output row, 4 channels); partial sums are
// added in offset order in fp32 registers and the row is written once.  The row of G that holds
// the pair (k, n) follows from the offset's start, the base of k's 64-row block and the block's
// presence bitmap.
// LANES (rows of a multiple of 4 * LANES channels; else 0): so many lanes share a row, and work out its up to 27 positions
// side by side while the row's bitmask is still on its way; the rows of G are asked for eight at a time.  Without, a thread
// pays three dependent loads for every four offsets.  Layers on 3x3x3 maps, without -> with, us: 256 -> 256 on 2.7 k points
// 22.0 -> 19.8, on 8 k 32.6 -> 30.8, (128, 128) -> 128 on 22 k 45.3 -> 42.2.
template <class T, int LANES>
__global__ void __launch_bounds__(kThreads) k_scatter_reduce(const float *__restrict__ G, const int32_t *__restrict__ nbr,
                                                             int stride, const uint64_t *__restrict__ colbits,
                                                             const int32_t *__restrict__ colbase, Offs offs,
                                                             int64_t n_blocks,
                                                             T *__restrict__ out, int64_t n_out, int cout, int K3,
                                                             const T *__restrict__ bias, const T *__restrict__ residual,
                                                             int relu) {
    const int quads = cout / 4;
    int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t k = g / quads;
    int q = (int)(g - k * quads);
    if (k >= n_out) return;
    uint32_t mask = (uint32_t)nbr[k * stride + K3];
    const int64_t b = k >> 6;
    const uint64_t before = (1ull << (k & 63)) - 1ull;
    floatx4 acc = {0.f, 0.f, 0.f, 0.f};
    if constexpr (LANES != 0) {
        int32_t at[32 / LANES];
#pragma unroll
        for (int i = 0; i < 32 / LANES; ++i) {
            const int n = i * LANES + (threadIdx.x & (LANES - 1));
            at[i] = n < K3 ? offs.v[n] + colbase[n * n_blocks + b] + __popcll(colbits[n * n_blocks + b] & before) : 0;
        }
        while (mask) {
            int32_t p[8];
            floatx4 v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                p[u] = -1;
                if (mask) {
                    const int n = __builtin_ctz(mask);
                    p[u] = __shfl(n < LANES ? at[0] : at[32 / LANES - 1], n & (LANES - 1), LANES);
                    mask &= mask - 1;
                }
            }
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (p[u] >= 0) v[u] = __builtin_nontemporal_load(reinterpret_cast<const floatx4 *>(G + (int64_t)p[u] * cout + q * 4));
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (p[u] >= 0) acc += v[u];
        }
    }
    // four offsets at a time: their positions first, then their rows of G (read once: streamed
    // past the caches), then the adds in offset order
    while (LANES == 0 && mask) {
        int64_t p[4];
        floatx4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            p[u] = -1;
            if (mask) {
                const int n = __builtin_ctz(mask);
                mask &= mask - 1;
                p[u] = offs.v[n] + colbase[n * n_blocks + b] + __popcll(colbits[n * n_blocks + b] & before);
            }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (p[u] >= 0) v[u] = __builtin_nontemporal_load(reinterpret_cast<const floatx4 *>(G + p[u] * cout + q * 4));
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (p[u] >= 0) acc += v[u];
    }
    // the layer's own result in T, then, if asked for, what ts_bias_act would do with it: fp32 sum
    // (bias first, then the residual), ReLU, one rounding
    const int64_t at = k * cout + q * 4;
    const bool tail = bias || residual || relu;
    if constexpr (sizeof(T) == 2) {
        half4 v = {(_Float16)acc[0], (_Float16)acc[1], (_Float16)acc[2], (_Float16)acc[3]};
        if (tail) {
            float f[4] = {(float)v[0], (float)v[1], (float)v[2], (float)v[3]};
            if (bias) {
                const half4 b = *reinterpret_cast<const half4 *>(bias + q * 4);
#pragma unroll
                for (int e = 0; e < 4; ++e) f[e] += (float)b[e];
            }
            if (residual) {
                const half4 r = *reinterpret_cast<const half4 *>(residual + at);
#pragma unroll
                for (int e = 0; e < 4; ++e) f[e] += (float)r[e];
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = (_Float16)(relu && f[e] < 0.f ? 0.f : f[e]);
        }
        *reinterpret_cast<half4 *>(out + at) = v;
    } else {
        if (tail) {
            if (bias) acc += *reinterpret_cast<const floatx4 *>(bias + q * 4);
            if (residual) acc += *reinterpret_cast<const floatx4 *>(residual + at);
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[e] = relu && acc[e] < 0.f ? 0.f : acc[e];
        }
        *reinterpret_cast<floatx4 *>(out + at) = acc;
    }
}

// ---- operand preparation ----------------------------------------------------------------------
// Wt[n][co][ci'] = W[n][ci'][co] for ci' < cin, 0 for cin <= ci' < cin_pad.
template <class T>
__global__ void k_pack_weights(const T *__restrict__ W, T *__restrict__ Wt, int K3, int cin, int cin_pad, int cout) {
    int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t total = (int64_t)K3 * cout * cin_pad;
    if (g >= total) return;
    int ci = (int)(g % cin_pad);
    int co = (int)((g / cin_pad) % cout);
    int n = (int)(g / ((int64_t)cin_pad * cout));
    Wt[g] = ci < cin ? W[((int64_t)n * cin + ci) * cout + co] : (T)0;
}

// Xp[row][c] = X[row][c] for c < cin, 0 up to cin_pad.
// A thread writes 8 consecutive elements of a padded row (cin_pad is a multiple of 8) with 16-byte stores.
template <class T>
__global__ void k_pad_rows(const T *__restrict__ X, T *__restrict__ Xp, int64_t rows, int cin, int cin_pad) {
    const int per_row = cin_pad / 8;
    int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= rows * per_row) return;
    int64_t r = g / per_row;
    const int c0 = (int)(g - r * per_row) * 8;
    T v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = c0 + e < cin ? X[r * cin + c0 + e] : (T)0;
    u32x4 raw[sizeof(T) / 2];
    __builtin_memcpy(raw, v, sizeof(v));
    u32x4 *dst = reinterpret_cast<u32x4 *>(Xp + r * cin_pad + c0);
#pragma unroll
    for (unsigned i = 0; i < sizeof(T) / 2; ++i) dst[i] = raw[i];
}

inline unsigned blocks_for(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }
inline size_t elem_size(int dtype) { return dtype == TS_F16 ? 2 : 4; }
inline int kstep(int dtype) { return dtype == TS_F16 ? Elem<_Float16>::KSTEP : Elem<float>::KSTEP; }

// Output-channel blocks of 32 handled by one workgroup: the largest of 4,3,2,1 dividing cout/32.
inline int pick_ncb(int cout) {
    int blocks = cout / 32;
    for (int ncb = 4; ncb >= 1; --ncb)
        if (blocks % ncb == 0) return ncb;
    return 1;
}

}  // namespace

// Weights of one layer in the layouts the kernels read (ts_weights_prepare); device memory owned
// by the object.
struct ts_weights {
    int K3 = 0, cin = 0, cout = 0, dtype = 0;
    void *wt = nullptr;     // [K3][cout][cin rounded up to the operand step], for k_fused / k_grouped_mm
    void *tile = nullptr;   // fp16: operand order of k_conv_tile (see k_pack_weights_tile)
};

namespace {

// 32-channel operand steps that stand together in the weights of k_conv_tile: the whole stage where every stage takes 64
// channels, else one, from which stages of any length are put together.
inline int tile_ksteps(int cin_pad) { return cin_pad % 64 == 0 ? 2 : 1; }

struct Prepared {
    const void *x;    // features, rows padded to cin_pad channels
    const void *wt;   // transposed, padded weights, or, for k_grouped_lines, weights in operand order
    int cin_pad;
};

// Whether the grouped matmul of a layer is k_grouped_lines: the same for every way of asking for it, for the two kernels'
// sums need not agree in their last bits.
inline bool mm_by_lines(size_t elem, const ts_kmap *kmap, int cin_pad, int cin1, int cout) {
    return elem == 2 && cin_pad % 64 == 0 && cin1 % 64 == 0 && (size_t)kmap->n_in * cin_pad * 2 < (1ull << 31) &&
           (size_t)kmap->K3 * cin_pad * cout * 2 < (1ull << 31);   // 31-bit offsets
}

int check_tensor(const ts_tensor *t, const char *name) {
    if (!t) return fail(TS_ERR_INVALID_ARG, "%s is NULL", name);
    if (t->dtype != TS_F32 && t->dtype != TS_F16) return fail(TS_ERR_INVALID_ARG, "%s: unknown dtype %d", name, t->dtype);
    if (t->rows < 0 || t->cols <= 0) return fail(TS_ERR_SHAPE, "%s: bad shape [%lld, %d]", name, (long long)t->rows, t->cols);
    if (t->rows > 0 && !t->data) return fail(TS_ERR_INVALID_ARG, "%s: data is NULL", name);
    if (reinterpret_cast<uintptr_t>(t->data) & 15) return fail(TS_ERR_INVALID_ARG, "%s: data must be 16-byte aligned", name);
    return TS_OK;
}

int check_layer(const ts_tensor *feats, const ts_tensor *weights, const ts_kmap *kmap, const ts_tensor *out) {
    if (!kmap) return fail(TS_ERR_INVALID_ARG, "kmap is NULL");
    if (kmap->pending_slot < 0 && kmap->error != TS_OK) return resolve(kmap);   // a map whose build found bad input
    TS_TRY(check_tensor(feats, "feats"));
    TS_TRY(check_tensor(weights, "weights"));
    TS_TRY(check_tensor(out, "out"));
    if (feats->dtype != weights->dtype || feats->dtype != out->dtype)
        return fail(TS_ERR_SHAPE, "feats, weights and out must share one dtype");
    TS_TRY(resolve_count(kmap));
    TS_TRY(settle(kmap));
    if (feats->rows != kmap->n_in) return fail(TS_ERR_SHAPE, "feats has %lld rows, the map expects %lld", (long long)feats->rows, (long long)kmap->n_in);
    if (out->rows != kmap->n_out) return fail(TS_ERR_SHAPE, "out has %lld rows, the map produces %lld", (long long)out->rows, (long long)kmap->n_out);
    if (weights->rows != (int64_t)kmap->K3 * feats->cols)
        return fail(TS_ERR_SHAPE, "weights must be [K^3*C_in, C_out] = [%lld, .], got %lld rows", (long long)kmap->K3 * feats->cols, (long long)weights->rows);
    if (weights->cols != out->cols) return fail(TS_ERR_SHAPE, "weights has %d columns, out has %d", weights->cols, out->cols);
    if (out->cols % 32 != 0 || out->cols > 1024) return fail(TS_ERR_UNSUPPORTED, "C_out must be a multiple of 32 (<= 1024), got %d", out->cols);
    if (feats->cols > 1024) return fail(TS_ERR_UNSUPPORTED, "C_in must be <= 1024, got %d", feats->cols);
    return TS_OK;
}

// Transpose/pad the weights into scratch, and pad the features when C_in is not a multiple of
// the operand step.
template <class T>
int prepare(const ts_tensor *feats, const ts_tensor *weights, const ts_kmap *kmap, Prepared *pr,
            const ts_weights *pw = nullptr, void *wbuf = nullptr, bool lines = false) {
    const int cin = feats->cols, cout = weights->cols, ks = Elem<T>::KSTEP;
    const int cin_pad = (cin + ks - 1) / ks * ks;
    pr->cin_pad = cin_pad;
    if (wbuf && cin_pad != cin) return fail(TS_ERR_UNSUPPORTED, "C_in must be a multiple of %d here", ks);
    if (pw) {
        pr->wt = lines ? pw->tile : pw->wt;
    } else {
        size_t wn = (size_t)kmap->K3 * cout * cin_pad;
        T *wt = static_cast<T *>(wbuf ? wbuf : scratch(2, wn * sizeof(T)));
        if (!wt) return last_fail_code();
        if (lines)
            TS_LAUNCH("k_pack_weights", k_pack_weights_tile, dim3(blocks_for((int64_t)wn, kThreads)), dim3(kThreads), static_cast<const _Float16 *>(weights->data), reinterpret_cast<_Float16 *>(wt), kmap->K3, cin, cin_pad, cout, tile_ksteps(cin_pad));
        else
            TS_LAUNCH("k_pack_weights", k_pack_weights<T>, dim3(blocks_for((int64_t)wn, kThreads)), dim3(kThreads), static_cast<const T *>(weights->data), wt, kmap->K3, cin, cin_pad, cout);
        pr->wt = wt;
    }
    pr->x = feats->data;
    if (cin_pad != cin && feats->rows > 0) {
        size_t xn = (size_t)feats->rows * cin_pad;
        T *xp = static_cast<T *>(scratch(3, xn * sizeof(T)));
        if (!xp) return last_fail_code();
        TS_LAUNCH("k_pad_rows", k_pad_rows<T>, dim3(blocks_for((int64_t)xn / 8, kThreads)), dim3(kThreads), static_cast<const T *>(feats->data), xp, feats->rows, cin, cin_pad);
        pr->x = xp;
    }
    return TS_OK;
}

// Largest chunk of {8,4,2} operand steps (KC = 64/32/16 for fp16, 32/16/8 for fp32) that divides cin.
inline int pick_ksteps(int cin, int kstep_elems) {
    int steps = cin / kstep_elems;
    if (steps % 4 == 0) return 4;
    if (steps % 2 == 0) return 2;
    return 1;
}

// Run `fn.template operator()<NCB, KSTEPS>()` for the runtime pair (ncb, ksteps).
template <class Fn>
void dispatch_shape(int ncb, int ksteps, Fn &&fn) {
#define TS_CASE(N, K)                     \
    if (ncb == N && ksteps == K) {        \
        fn.template operator()<N, K>();   \
        return;                           \
    }
    TS_CASE(1, 1) TS_CASE(1, 2) TS_CASE(1, 4) TS_CASE(2, 1) TS_CASE(2, 2) TS_CASE(2, 4)
    TS_CASE(3, 1) TS_CASE(3, 2) TS_CASE(3, 4) TS_CASE(4, 1) TS_CASE(4, 2) TS_CASE(4, 4)
#undef TS_CASE
}

// (offset, chunk) pairs per pipeline stage of k_fused: narrow shapes have little MFMA work
// per pair, so several are batched between barriers to shorten the chain of memory latencies.
constexpr int fused_group(int ncb, int ksteps) {
    return ncb * ksteps <= 2 ? 4 : (ncb * ksteps <= 8 ? 3 : 1);
}

inline int compute_units() {
    static int n = 0;
    if (n == 0) {
        int dev = 0;
        hipDeviceProp_t prop;
        if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess) n = prop.multiProcessorCount;
        if (n <= 0) n = 256;
    }
    return n;
}

// Rows ordered by the offsets they meet (5 to 9 us, once per map) make a layer 7 to 20 % faster on scans and
// surfaces of more than about a tile per compute unit and 25 to 45 % faster on scattered points (153 k LiDAR
// points: 64 channels 43.9 -> 40.9 us, 96: 62 -> 55, 128: 92 -> 73); below that the longest tile decides.
// Single precision gains more, a pair's work there takes some ten times as long: 153 k LiDAR points, 32 -> 32 channels
// 63 -> 47 us, 64 -> 64 192 -> 127; 200 k scattered points 120 -> 64, 403 -> 195; 40 k LiDAR points 29 -> 27, 80 -> 71.
// A map that has served a layer will serve more; one that has not is ordered only for a layer that gains more than
// the ordering takes (at_once).  2x2x2 maps that go up gain at every size (the order takes 4 to 6 us; 64 -> 64 on 4 k rows
// 8.0 -> 6.2, 128 -> 64 on 16 k 10.4 -> 8.5, 128 -> 128 14.6 -> 9.0, on 150 k of a scan 35 -> 26).
inline void order_for_layer(const ts_kmap *kmap, bool at_once) {
    if ((kmap->n_tiles > compute_units() || (goes_up_by_two(kmap) && kmap->n_tiles > 1)) && (kmap->uses > 0 || at_once)) order_windows(kmap);
}
// Single precision, map and first layer together, with the order and without it (us), by tiles * C_in * C_out, which the
// gain follows; the ordering itself takes 5 to 9:
//   0.8 M (100 k points, 32 -> 32)    LiDAR  66, 65    surfaces 66, 65    scattered  77, 101
//   1.0 M (125 k points, 32 -> 32)           73, 79             75, 78               83, 105
//   1.2 M (153 k points, 32 -> 32)           79, 88             86, 97               98, 123
//   1.4 M ( 45 k points, 64 -> 64)           94, 105           106, 107             111, 138
// With hardly more than a tile per compute unit the longest tile decides once more: 258 tiles, 64 -> 64, 84 and 77 us
// on a scan, 98 and 83 on surfaces; from 282 on every layer gains.
// fp16 the same way (the ordering takes 8; without it and with it; a scan, surfaces, scattered points):
//   3.2 M (100 k points, 64 -> 64)    46 53, 51 52, 71 61       4.9 M (153 k, 64 -> 64)    59 60, 60 58, 81 74
//   6.4 M (100 k, 64 -> 128)          49 56, 58 56, 76 64       7.2 M (100 k, 96 -> 96)    64 59, 68 60, 90 71
//   7.7 M ( 80 k, 128 -> 96)          62 67, 61 66, 84 73       9.6 M (300 k, 64 -> 64)    89 88, 91 86, 138 120
//   9.8 M (153 k, 64 -> 128)          66 65, 72 67, 90 78       9.8 M (153 k, 128 -> 64)   81 73, 87 74, 110 89
//   14.7 M (153 k, 128 -> 96)         92 82, 106 87, 124 98     48 M (1.5 M, 64 -> 64)     446 434, 487 455, 694 567
// From 9 M on every scene gains; below, scattered points do and scans and surfaces mostly lose, but for 96 -> 96.  Layers on 513 to
// 549 tiles of 128 -> 128 lie just below: 64 57, 68 59, 71 80 (66 k points, with the order and without it).
inline bool order_at_once(const ts_kmap *kmap, int cin, int cout, size_t elem) {
    if (elem == 4) return kmap->n_tiles > compute_units() * 17 / 16 && kmap->n_tiles * cin * cout >= 1000000;
    if (goes_up_by_two(kmap)) return cin * cout >= 128 * 128;
    return kmap->n_tiles > 2 * compute_units() && kmap->n_tiles * cin * cout >= 9000000;
}

template <class T>
struct FusedLaunch {
    const Prepared &pr;
    const ts_kmap *kmap;
    ts_tensor *out;
    const T *zero;
    template <int NCB, int KSTEPS>
    void operator()() const {
        constexpr int KC = KSTEPS * Elem<T>::KSTEP;
        constexpr int G = fused_group(NCB, KSTEPS);
        dim3 grid((unsigned)kmap->n_tiles, out->cols / (NCB * 32));
        TS_LAUNCH("k_fused", (k_fused<T, NCB, KC, G>), grid, dim3(kThreads), static_cast<const T *>(pr.x),
                  static_cast<const T *>(pr.wt), kmap->d_nbr, kmap->stride, row_order(kmap), kmap->n_out,
                  static_cast<T *>(out->data), zero, pr.cin_pad, out->cols, kmap->K3, kmap->centre);
    }
};

template <class T>
int run_fused_staged(const ts_tensor *feats, const ts_tensor *weights, const ts_kmap *kmap, ts_tensor *out,
                     const ts_weights *pw = nullptr, void *wbuf = nullptr, const void *zeros = nullptr) {
    Prepared pr;
    TS_TRY(prepare<T>(feats, weights, kmap, &pr, pw, wbuf));
    const T *zero = static_cast<const T *>(zeros ? zeros : zero_row());
    if (!zero) return last_fail_code();
    if (!wbuf) order_for_layer(kmap, order_at_once(kmap, pr.cin_pad, out->cols, sizeof(T)));
    ++const_cast<ts_kmap *>(kmap)->uses;
    dispatch_shape(pick_ncb(out->cols), pick_ksteps(pr.cin_pad, Elem<T>::KSTEP), FusedLaunch<T>{pr, kmap, out, zero});
    TS_HIP(hipGetLastError());
    return TS_OK;
}

// What follows the layer's sum, if anything: y = act(conv + bias + residual) (see ts_sparse_conv_act).
struct Epilogue {
    const void *bias = nullptr;
    const void *residual = nullptr;
    int relu = 0;
    bool any() const { return bias || residual || relu; }
};

// The second half of a layer input that is the channel concatenation [x | x2] of two tensors (never
// formed): x has cin1 channels per row, x2 the rest.  x2 == nullptr: one tensor, as usual.
struct Second {
    const void *x2 = nullptr;
    int cin1 = 0;
};

template <int NCO, int KS, bool TWO, bool HALF = false, int GR = 1>
void launch_conv_tile(const _Float16 *x, const _Float16 *wf, const ts_kmap *kmap, ts_tensor *out, int cin_pad,
                      const Epilogue &ep, const Second &sec) {
    // as many workgroups as stay resident at once, fewer for small maps
    static int per_cu = 0;   // per instantiation
    if (per_cu == 0) {
        int n = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_conv_tile<NCO, KS, TWO, HALF, GR>, kThreads * GR, 0) != hipSuccess || n <= 0) {
            (void)hipGetLastError();
            n = 2;
        }
        per_cu = n;
    }
    const int64_t resident = (int64_t)compute_units() * per_cu;
    dim3 grid((unsigned)(kmap->n_tiles < resident ? kmap->n_tiles : resident), out->cols / (NCO * 16));
    const int cin1 = TWO ? sec.cin1 : cin_pad;
    const int32_t *perm = row_order(kmap);
    const int row_shift = kmap->stride == 32 ? 3 : kmap->stride == 16 ? 2 : 0;   // 16-byte units of a table row
    TS_LAUNCH(GR > 1 ? "k_conv_tile_groups" : "k_conv_tile", (k_conv_tile<NCO, KS, TWO, HALF, GR>), grid, dim3(kThreads * GR), x, reinterpret_cast<const u32x4 *>(wf), kmap->d_nbr,
              row_shift, perm, kmap->d_perm != nullptr,
              !perm && (kmap->scan_done || (kmap->scan_enqueued && kmap->stream == stream())) ? kmap->d_tile_order : nullptr,
              kmap->n_out, static_cast<_Float16 *>(out->data), kmap->d_sched, cin_pad, out->cols, kmap->K3,
              static_cast<const _Float16 *>(ep.bias), static_cast<const _Float16 *>(ep.residual), ep.relu,
              (int)((size_t)kmap->n_in * cin1 * 2), (int)((size_t)kmap->K3 * cin_pad * out->cols * 2), kmap->centre,
              static_cast<const _Float16 *>(sec.x2), (int)((size_t)kmap->n_in * (cin_pad - cin1) * 2), cin1);
}

constexpr int kDirectDepth = 2;   // (3 took registers that two more waves can have: 2 to 4 % slower)

template <int NCO, int KSTEPS, bool TWO>
void launch_conv_direct(const _Float16 *x, const _Float16 *wf, const ts_kmap *kmap, ts_tensor *out, int cin_pad,
                        const Epilogue &ep, const Second &sec) {
    // as many workgroups as stay resident at once, fewer for small maps
    static int per_cu = 0;   // per instantiation
    if (per_cu == 0) {
        int n = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_conv_direct<NCO, KSTEPS, kDirectDepth, TWO>, kThreads, 0) != hipSuccess || n <= 0) {
            (void)hipGetLastError();
            n = 2;
        }
        per_cu = n;
    }
    const int64_t resident = (int64_t)compute_units() * per_cu;
    dim3 grid((unsigned)(kmap->n_tiles < resident ? kmap->n_tiles : resident), out->cols / (NCO * 16));
    const int cin1 = TWO ? sec.cin1 : cin_pad;
    const int32_t *perm = row_order(kmap);
    TS_LAUNCH("k_conv_direct", (k_conv_direct<NCO, KSTEPS, kDirectDepth, TWO>), grid, dim3(kThreads), x,
              reinterpret_cast<const u32x4 *>(wf), kmap->d_nbr, kmap->stride, perm, kmap->d_perm != nullptr,
              !perm && (kmap->scan_done || (kmap->scan_enqueued && kmap->stream == stream())) ? kmap->d_tile_order : nullptr,
              kmap->n_out, static_cast<_Float16 *>(out->data), kmap->d_sched, cin_pad, out->cols, kmap->K3,
              static_cast<const _Float16 *>(ep.bias), static_cast<const _Float16 *>(ep.residual), ep.relu,
              (int)((size_t)kmap->n_in * cin1 * 2), (int)((size_t)kmap->K3 * cin_pad * out->cols * 2), kmap->centre,
              static_cast<const _Float16 *>(sec.x2), (int)((size_t)kmap->n_in * (cin_pad - cin1) * 2), cin1);
}

// Narrow layers (C_in <= 32, C_out = 32): the kernel that keeps all weights in LDS.  False if this
// device does not give a workgroup that much LDS: the caller then takes k_conv_tile.
template <int NCO, int KSTEPS>
bool launch_conv_res(const _Float16 *x, const _Float16 *wf, const ts_kmap *kmap, ts_tensor *out, const Epilogue &ep) {
    static int usable = -1;   // per instantiation
    constexpr size_t lds = res_lds_bytes<NCO * KSTEPS>();
    if (usable < 0) {
        usable = hipFuncSetAttribute(reinterpret_cast<const void *>(k_conv_res<NCO, KSTEPS, kResDepth>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) == hipSuccess;
        if (!usable) (void)hipGetLastError();
    }
    if (!usable) return false;
    const int64_t n_units = (kmap->n_out + kResRows - 1) / kResRows;
    const int64_t wgs = (n_units + kResWaves - 1) / kResWaves;
    const int64_t cus = compute_units();
    TS_LAUNCH_SHM("k_conv_res", (k_conv_res<NCO, KSTEPS, kResDepth>), dim3((unsigned)(wgs < cus ? wgs : cus), out->cols / (NCO * 16)), dim3(kResThreads), lds,
                       x, reinterpret_cast<const u32x4 *>(wf), kmap->d_nbr, kmap->stride, kmap->d_perm, kmap->n_out,
                       static_cast<_Float16 *>(out->data), kmap->d_sched, kmap->K3, out->cols, static_cast<const _Float16 *>(ep.bias),
                       static_cast<const _Float16 *>(ep.residual), ep.relu, (int)((size_t)kmap->n_in * KSTEPS * 64), kmap->centre);
    return true;
}

// fp16: input channels padded to a multiple of 32 (one MFMA step), chunks of 64 where possible.
// feats->cols is the layer's C_in; with sec.x2 set, feats->data holds only the first sec.cin1 channels of
// every row (both parts multiples of 32 channels: nothing is padded then).
int run_fused_f16(const ts_tensor *feats, const ts_tensor *weights, const ts_kmap *kmap, ts_tensor *out,
                  const Epilogue &ep, const ts_weights *pw = nullptr, void *wbuf = nullptr, const Second &sec = Second()) {
    typedef _Float16 T;
    const int cin = feats->cols, cout = out->cols;
    const int cin_pad = (cin + 31) / 32 * 32;
    const int wsteps = tile_ksteps(cin_pad), ksteps = cin_pad % 64 != 0 && cin_pad % 96 == 0 ? 3 : wsteps;
    // the kernel addresses features and weights with 31-bit byte offsets
    if ((size_t)kmap->n_in * cin_pad * 2 >= (1ull << 31) || (size_t)kmap->K3 * cin_pad * cout * 2 >= (1ull << 31)) {
        if (ep.any()) return fail(TS_ERR_UNSUPPORTED, "feature matrix of 2 GiB or more: call ts_sparse_conv and ts_bias_act");
        if (wbuf) return fail(TS_ERR_UNSUPPORTED, "feature matrix of 2 GiB or more");
        return run_fused_staged<_Float16>(feats, weights, kmap, out, pw);
    }
    if (wbuf && cin_pad != cin) return fail(TS_ERR_UNSUPPORTED, "C_in must be a multiple of 32 here");
    const T *wf = pw ? static_cast<const T *>(pw->tile) : nullptr;
    if (!wf) {
        const size_t wn = (size_t)kmap->K3 * cout * cin_pad;
        T *buf = static_cast<T *>(wbuf ? wbuf : scratch(2, wn * sizeof(T)));
        if (!buf) return last_fail_code();
        TS_LAUNCH("k_pack_weights", k_pack_weights_tile, dim3(blocks_for((int64_t)wn, kThreads)), dim3(kThreads),
                  static_cast<const T *>(weights->data), buf, kmap->K3, cin, cin_pad, cout, wsteps);
        wf = buf;
    }
    const T *x = static_cast<const T *>(feats->data);
    if (cin_pad != cin) {
        const size_t xn = (size_t)feats->rows * cin_pad;
        T *xp = static_cast<T *>(scratch(3, xn * sizeof(T)));
        if (!xp) return last_fail_code();
        TS_LAUNCH("k_pad_rows", k_pad_rows<T>, dim3(blocks_for((int64_t)xn / 8, kThreads)), dim3(kThreads), x, xp, feats->rows, cin, cin_pad);
        x = xp;
    }
    const int cblocks = cout / 16;
    // Launches of hardly more than a workgroup a CU: several groups of waves to a tile (k_conv_tile<..., GR>), and the fewest
    // output blocks a workgroup with which each still has a CU (64 -> 64 on 8 k rows of a scan, by 2 and 4 blocks, 11.4 and
    // 13.8 us, on 26 k, where 2 blocks make 408 workgroups, 18.4 and 14.5).  With 128 input channels and more the groups stay ahead
    // on kept maps until a CU has two, or two and a half, workgroups, if those take all output channels (one group and three; a
    // scan, scattered points): 128 -> 128 on 65 k rows 40.1 38.0, 41.1 36.1, on 80 k 42.8 44.1, 46.9 47.3; 192 -> 64 on 80 k
    // 50.6 43.8, 53.3 51.2, on 110 k 60.3 61.8, 57.4 70.6; in five slices 128 -> 160 on 12 k 30.5 32.7; 64 -> 64 on 40 k 20.1 20.3,
    // 21.0 19.5, on 65 k 20.3 21.4, 22.2 23.2.  Not on maps with a stride, whose rows are never sorted by the library (down to
    // 44 k rows of a scan after one halving, 128 -> 64 32.4 38.2, 192 -> 96 51.6 62.8, of scattered points 32.2 41.8, 57.9 68.6).
    // Going up, and on 1x1x1 maps, a tile has a stage or two: nothing to share.
    // Which layers these are goes by sizes alone, not by the parts of an input or the order of the rows: the sums of groups are
    // not those of one.
    const int64_t cus = compute_units();
    int group_nco = 0;
    if (kmap->K3 > 1 && !goes_up_by_two(kmap)) {
        int most = 2;
        for (int c : {8, 6, 4, 2}) {
            if (cblocks % c != 0) continue;
            if (most < c) most = c;
            // 96 output channels in one slice, of at most 96: no faster than three slices of one group before nearly half of the CUs
            // have a tile (us, one group and three; a scan, a scan after one halving, surfaces, scattered points): 96 -> 96 on 11 k
            // rows 18.9 20.8, 22.1 24.4, 20.0 20.3, 23.6 24.8, on 14 k 20.0 21.6, 25.0 24.9, 19.9 20.3, 24.3 25.1, on 16 k 23.5 21.1,
            // 25.8 25.0, 23.3 21.2, 25.2 25.2; 32 -> 96 down to 12 k rows 10.6 11.7, 10.9 11.4, 11.0 11.6, 10.4 11.6
            if (c == 6 && cblocks == 6 && cin_pad <= 96 && 20 * kmap->n_tiles <= 9 * cus) continue;
            if (kmap->n_tiles * (cblocks / c) <= cus) group_nco = c;
        }
        if (!group_nco && kmap->K3 == 27 && kmap->s == 1 && cin_pad >= 128 && cblocks == most && 2 * kmap->n_tiles <= (cin_pad > 128 ? 5 : 4) * cus) group_nco = most;
    }
    // 32 input channels and 27 offsets: the kernel with resident weights (for 2x2x2 maps and for 64 -> 32 it
    // measured no faster than k_conv_tile, and 64 -> 64 in two slices of output channels much slower: every
    // slice gathers all rows again)
    // (In groups instead while every tile has a CU: 32 -> 32 on 1 k rows 9.3 -> 7.1 us, on 32 k 12.6 -> 9.9, 4 -> 32 12.4 -> 9.4,
    // 15.8 -> 13.1.)
    if (!group_nco && cin_pad == 32 && kmap->K3 > 8 && kmap->n_out > 0 && (cout == 32 || cout == 64) && !sec.x2) {
        const bool done = cout == 32 ? launch_conv_res<2, 1>(x, wf, kmap, out, ep) : launch_conv_res<4, 1>(x, wf, kmap, out, ep);
        if (done) {
            TS_HIP(hipGetLastError());
            return TS_OK;
        }
    }
    // With more tiles than CUs the groups are ahead in sorted rows alone: in natural order a workgroup, which has its CU to
    // itself, has tiles of nearly all offsets, and one round too many of them.  So a new map's rows are sorted for its first
    // such layer; in time with the map (us, one group in natural order, groups in natural order, sorting and groups; a scan, a scan
    // after one halving, surfaces, scattered points): 128 -> 64 on 46 k rows 50 48 49, 54 55 50, 52 50 48, 54 63 53; 128 -> 128 on 64 k
    // 55 59 59, 61 67 62, 58 61 64, 70 75 65; 192 -> 96 on 52 k 68 69 60, 74 80 60, 74 71 60, 79 89 67; 192 -> 64 on 76 k 66 70 67,
    // 70 85 68, 73 82 67, 92 111 79.  With hardly more than a tile a CU the longest tile decides, as elsewhere (192 -> 64 on 34 k
    // 56 51 52, 55 48 54, 56 45 53, 64 77 57), and 128 -> 32 gains too little (46 k 47 42 45, 50 48 46, 48 43 44, 48 56 49; 192 -> 32
    // 57 48 48, 62 60 51, 61 53 47, 58 69 55).
    const bool groups_at_once = group_nco && 16 * kmap->n_tiles > 17 * cus && cin_pad * cout > 128 * 32;
    if (!wbuf) order_for_layer(kmap, groups_at_once || order_at_once(kmap, cin_pad, cout, sizeof(T)));
    ++const_cast<ts_kmap *>(kmap)->uses;
    if (group_nco) {
#define TS_GROUPS_CASE(N)                                                                                      \
    if (group_nco == N) {                                                                                      \
        if (sec.x2) {                                                                                          \
            if (ksteps == 2) launch_conv_tile<N, 2, true, false, 3>(x, wf, kmap, out, cin_pad, ep, sec);       \
            else if (ksteps == 3) launch_conv_tile<N, 2, true, true, 2>(x, wf, kmap, out, cin_pad, ep, sec);   \
            else launch_conv_tile<N, 2, true, true, 3>(x, wf, kmap, out, cin_pad, ep, sec);                    \
        } else if (ksteps == 2) launch_conv_tile<N, 2, false, false, 3>(x, wf, kmap, out, cin_pad, ep, sec);   \
        else if (ksteps == 3) launch_conv_tile<N, 3, false, false, 2>(x, wf, kmap, out, cin_pad, ep, sec);     \
        else if (cin_pad == 32) launch_conv_tile<N, 1, false, false, 3>(x, wf, kmap, out, cin_pad, ep, sec);   \
        else launch_conv_tile<N, 2, false, true, 3>(x, wf, kmap, out, cin_pad, ep, sec);                       \
    }
        TS_GROUPS_CASE(8) TS_GROUPS_CASE(6) TS_GROUPS_CASE(4) TS_GROUPS_CASE(2)
#undef TS_GROUPS_CASE
        TS_HIP(hipGetLastError());
        return TS_OK;
    }
    // Output channels per workgroup: as many as divide C_out (every slice gathers the rows again), fewer
    // when the launch would leave most of the chip idle: a lone workgroup per CU walks its stages one
    // after the other, and a stage of eight output blocks takes twice as long as one of four.
    int nco = 2, cap = 8;
    const int64_t wgs8 = kmap->n_tiles * ((cblocks + 7) / 8);
    if (wgs8 <= cus / 2 || (wgs8 <= cus && kmap->K3 > 8)) cap = 4;
    if (cap == 4 && kmap->n_tiles * ((cblocks + 3) / 4) <= cus / 2) cap = 2;
    for (int c : {8, 6, 4, 2})
        if (c <= cap && cblocks % c == 0) {
            nco = c;
            break;
        }
    // Layers that k_conv_direct does faster than one group.  It keeps two stages in flight and issues less for each, which
    // decides while a CU has a workgroup or two, the more the further rows have to come; k_conv_tile skips the blocks that do not
    // meet an offset.  The lines lie where most scenes change sides (us, k_conv_tile and k_conv_direct, on kept maps whose rows
    // come new from memory every time, as a network's do: scattered points, surfaces, a scan, a scan after one halving).
    //  - stages of two sources, a part of the input being no multiple of 64 channels: up to two tiles a CU, (96, 32) -> 192 on 33 k
    //    rows 51 42, 48 41, 41 34, 48 42, on 65 k 61 52, 62 56, 52 49, 58 51, on 97 k 74 77, 77 77, 69 71, 76 74; with one stage an
    //    offset up to three, (32, 32) -> 32 on 33 k 23 16, 21 16, 18 14, 21 15, on 97 k 26 22, 28 23, 25 22, 25 22
    //  - maps that go up, and 1x1x1 ones, leave a tile a stage or two: k_conv_tile at every size
    //  - 2x2x2 maps that go down: while one workgroup has at most 64 output channels (32 input channels: up to two tiles a CU; 96:
    //    while there is one slice), 128 -> 64 from 160 k points 39 32, 21 22, 26 26, 23 22, from 300 k 52 46, 27 29, 34 33, 33 30,
    //    64 -> 64 from 300 k 38 34, 21 22, 26 26, 27 25, 96 -> 96 from 80 k 23 22, 14 14, 18 18, 17 17
    //  - stages of 96 channels on 27 offsets: in two parts up to two tiles a CU, (64, 32) -> 96 on 33 k rows 39 28, 35 28, 30 24,
    //    35 27, on 65 k 40 31, 38 33, 36 29, 36 31, on 97 k 43 41, 43 45, 41 40, 39 42; in one part never, 96 -> 96 on 14 k 26 25,
    //    20 20, 20 21, 26 26, 96 -> 192 on 20 k 37 39, 30 31, 27 28, 33 35, 96 -> 256 on 32 k 43 49, 38 42, 32 39, 44 49
    //  - stages of 32: up to two tiles a CU, 32 -> 96 on 33 k rows 20 18, 20 18, 17 17, 19 18, on 65 k 23 21, 23 23, 21 20, 21 21, on
    //    97 k 25 25, 27 27, 26 26, 25 26
    //  - stages of 64 and a half empty one, in slices of at most 64 output channels: from a few tiles to 1.6 a CU, 160 -> 160 on
    //    11 k rows 51 47, 40 38, 41 39, 49 45, on 50 k 95 84, 98 104, 76 75, 92 96, 160 -> 320 on 20 k 108 97, 72 69, 53 50, 72 65, on
    //    50 k 111 97, 113 112, 88 85, 109 105; not in two parts, where the kernel with stages of 32 walks twice as many
    //  - whole stages of 64 in one part on 27 offsets: what it was ahead in goes to the groups, but for maps with a stride and several
    //    stages an offset, one slice of at most 96 output channels: up to 1.6 tiles a CU, up to 40 k rows of scattered points, a scan, a
    //    scan after one halving 128 -> 64 37 33, 32 28, 32 29, of surfaces, a scan, a scan after one halving 192 -> 96 42 40, 51 46, 51 48
    const bool split = sec.x2 && ksteps == 2 && sec.cin1 % 64 != 0, half_empty = ksteps == 1 && cin_pad != 32, up = goes_up_by_two(kmap);
    bool direct;
    if (split) direct = kmap->K3 > 1 && kmap->n_tiles <= (cin_pad == 64 ? 3 : 2) * cus;
    else if (kmap->K3 == 1 || up) direct = false;
    else if (ksteps == 3) direct = kmap->K3 == 8 ? nco == cblocks : sec.x2 && kmap->n_tiles <= 2 * cus;
    else if (cin_pad == 32) direct = kmap->n_tiles <= 2 * cus && (kmap->K3 > 8 || nco <= 4);
    else if (half_empty && sec.x2) direct = false;
    else if (kmap->K3 == 8) direct = nco <= 4;
    else if (half_empty) direct = nco <= 4 && 16 * kmap->n_tiles > cus && 5 * kmap->n_tiles <= 8 * cus;
    else direct = cin_pad >= 128 && nco == cblocks && nco <= 6 && 5 * kmap->n_tiles <= 8 * cus;
    // Maps that go up, their rows in order of their offset, and 1x1x1 ones leave a tile few stages, for which three workgroups a CU
    // beat the two that stages of 96 channels leave room for, beyond four tiles a CU: 96 -> 96 up to 130 k scattered points 25 and,
    // by 32 channels a stage, 27, to 200 k 36.9 and 35.5, to 300 k 44 and 39; 1x1x1 on 200 k, by 64 and 32, 31.4 and 29.1, on
    // 300 k 41.7 and 35.5.
    const bool by_32 = ksteps == 3 && !sec.x2 && up && kmap->n_tiles > 4 * cus;
    const bool by_64 = ksteps == 3 && !sec.x2 && kmap->K3 == 1 && kmap->n_tiles > 4 * cus;
#define TS_DIRECT_CASE(N)                                                                          \
    if (direct && nco == N) {                                                                      \
        if (sec.x2) {                                                                              \
            if (ksteps == 2) launch_conv_direct<N, 2, true>(x, wf, kmap, out, cin_pad, ep, sec);   \
            else launch_conv_direct<N, 3, true>(x, wf, kmap, out, cin_pad, ep, sec);               \
        } else if (ksteps == 2) {                                                                  \
            if constexpr (N <= 6) launch_conv_direct<N, 2, false>(x, wf, kmap, out, cin_pad, ep, sec); \
            else return fail(TS_ERR_UNSUPPORTED, "no k_conv_direct for %d blocks of output channels in stages of 64", N); \
        } else if (ksteps == 3) launch_conv_direct<N, 3, false>(x, wf, kmap, out, cin_pad, ep, sec); \
        else launch_conv_direct<N, 1, false>(x, wf, kmap, out, cin_pad, ep, sec);                  \
    }
    TS_DIRECT_CASE(8) TS_DIRECT_CASE(6) TS_DIRECT_CASE(4) TS_DIRECT_CASE(2)   // (one part, stages of 64: never 8 blocks)
#undef TS_DIRECT_CASE
#define TS_TILE_CASE(N)                                                                            \
    if (!direct && nco == N) {                                                                     \
        if (sec.x2) {                                                                              \
            if (ksteps == 2) launch_conv_tile<N, 2, true>(x, wf, kmap, out, cin_pad, ep, sec);     \
            else launch_conv_tile<N, 2, true, true>(x, wf, kmap, out, cin_pad, ep, sec);          \
        } else if (ksteps == 2) launch_conv_tile<N, 2, false>(x, wf, kmap, out, cin_pad, ep, sec); \
        else if (ksteps == 3 && !by_32 && !by_64) launch_conv_tile<N, 3, false>(x, wf, kmap, out, cin_pad, ep, sec); \
        else if (cin_pad == 32 || by_32) launch_conv_tile<N, 1, false>(x, wf, kmap, out, cin_pad, ep, sec); \
        else launch_conv_tile<N, 2, false, true>(x, wf, kmap, out, cin_pad, ep, sec);             \
    }
    TS_TILE_CASE(8) TS_TILE_CASE(6) TS_TILE_CASE(4) TS_TILE_CASE(2)
#undef TS_TILE_CASE
    static_assert(1024 / 32 <= kMaxSchedSlices, "C_out <= 1024 in slices of at least 32 channels");
    TS_HIP(hipGetLastError());
    return TS_OK;
}

template <class T>
int run_fused(const ts_tensor *feats, const ts_tensor *weights, const ts_kmap *kmap, ts_tensor *out,
              const ts_weights *pw = nullptr) {
    if constexpr (sizeof(T) == 2) return run_fused_f16(feats, weights, kmap, out, Epilogue(), pw);
    return run_fused_staged<T>(feats, weights, kmap, out, pw);
}

int64_t mm_tiles(int64_t rows) { return (rows + kTileRows - 1) / kTileRows; }

// Every offset with the blocks its own list needs: no padding, one launch.
MmPlan whole_plan(const ts_kmap *kmap) {
    MmPlan plan;
    plan.count = 0;
    for (int n = 0; n < kmap->K3; ++n) {
        if (kmap->sizes[n] == 0) continue;
        plan.n[plan.count] = n;
        plan.tiles[plan.count++] = (int32_t)mm_tiles(kmap->sizes[n]);
    }
    return plan;
}

int64_t plan_tiles(const MmPlan &plan) {
    int64_t t = 0;
    for (int i = 0; i < plan.count; ++i) t += plan.tiles[i];
    return t;
}

template <class T>
struct GroupedLaunch {
    const T *F, *X, *wt;
    const ts_kmap *kmap;
    MmPlan plan;
    float *G;
    const T *zero;
    int cin_pad, cout;
    const int32_t *in_idx;
    const T *X2;
    int cin1;
    template <int NCB, int KSTEPS>
    void operator()() const {
        constexpr int KC = KSTEPS * Elem<T>::KSTEP;
        dim3 grid((unsigned)plan_tiles(plan), cout / (NCB * 32));
        TS_LAUNCH("k_grouped_mm", (k_grouped_mm<T, NCB, KC>), grid, dim3(kThreads), F, X, wt, offs_of(kmap), plan, G, zero,
                  cin_pad, cout, kmap->centre, in_idx, X2, cin1);
    }
};

// order: 0 = the library's choice, 1 = output order (k_gather), 2 = input-stationary (k_gather_in) where it applies.
int gather_impl(const void *x, int64_t /*rows*/, int cin_pad, int dtype, const ts_kmap *kmap, void *F, int order = 0) {
    if (kmap->M == 0) return TS_OK;
    const int vec_per_row = (int)(cin_pad * elem_size(dtype) / 16);
    // Input-stationary order reads every input row once instead of once per pair, and writes whole rows of F
    // at scattered places.  Measured on the LiDAR-like scene at 153 k, 1.5 M and 15 M points: with rows of 128
    // bytes or more it wins at every size (C = 64: 31 against 35 us at 153 k, 3.0 against 4.4 ms at 15 M;
    // C = 128: 51 against 67 us, 5.4 against 8.8 ms); with 64-byte rows (half a cache line per scattered
    // write) only once the feature matrix no longer fits the 256 MB last-level cache.
    const bool can_in = kmap->K3 == 27 && kmap->centre >= 0 && kmap->stride == 32 &&
                        (vec_per_row == 4 || vec_per_row == 8 || vec_per_row == 16 || vec_per_row == 32) &&
                        kmap->M < (int64_t)1 << 31;
    const size_t x_bytes = (size_t)kmap->n_in * vec_per_row * 16;
    if (can_in && (order == 2 || (order == 0 && (vec_per_row >= 8 || x_bytes > ((size_t)256 << 20))))) {
        TS_TRY(resolve(kmap));
        const int64_t threads = kmap->n_in * vec_per_row;
        const dim3 grid(blocks_for(threads, kThreads)), block(kThreads);
        const u32x4 *xs = static_cast<const u32x4 *>(x);
        u32x4 *fs = static_cast<u32x4 *>(F);
#define TS_GATHER_IN(V) TS_LAUNCH("k_gather_in", k_gather_in<V>, grid, block, xs, kmap->d_nbr, kmap->d_colbits, kmap->d_colbase, offs_of(kmap), kmap->n_blocks, fs, kmap->n_in)
        if (vec_per_row == 4) TS_GATHER_IN(4);
        else if (vec_per_row == 8) TS_GATHER_IN(8);
        else if (vec_per_row == 16) TS_GATHER_IN(16);
        else TS_GATHER_IN(32);
#undef TS_GATHER_IN
        TS_HIP(hipGetLastError());
        return TS_OK;
    }
    TS_TRY(ensure_pairs(kmap));
    int64_t lo = 0, hi = 0;
    if (kmap->centre >= 0) {
        lo = kmap->offs[kmap->centre];
        hi = kmap->offs[kmap->centre + 1];
    }
    TS_LAUNCH("k_gather", k_gather, dim3(blocks_for(kmap->M * vec_per_row, kThreads * kGatherPer)), dim3(kThreads), static_cast<const u32x4 *>(x), kmap->d_in_idx, static_cast<u32x4 *>(F), kmap->M, vec_per_row, lo, hi);
    TS_HIP(hipGetLastError());
    return TS_OK;
}

template <int NCO>
void launch_grouped_lines(const void *F, const void *X, const void *wf, const ts_kmap *kmap, const MmPlan &plan, float *G, int cin,
                          int cout, const int32_t *in_idx, const Second &sec) {
    const int cin1 = sec.x2 ? sec.cin1 : cin;
    // Where there are two slices, and more tiles than CUs, a tile's slices start together, while its rows are on their way.  Slice
    // after slice and tile after tile (us; a scan after three halvings | scattered points): 256 -> 256 on 2.7 k points 19.7 20.2 |
    // 14.8 14.8, on 7.5 k 30.3 30.3 | 20.2 20.3, on 16 k 55.8 55.1 | 30.1 29.5; (256, 256) -> 256 on 4.5 k 25.3 25.0 | 18.4 18.8, on
    // 7.5 k 38.5 37.2 | 24.7 24.3, on 16 k 74.6 72.4 | 39.1 36.4; with five slices 192 -> 160 on 13 k points 38.5 39.6.  Not on
    // 2x2x2 maps, whose pairs share few input rows (256 -> 256 from 60 k points of a scan 46.9 52.2).
    dim3 grid((unsigned)plan_tiles(plan), cout / (NCO * 16));
    const int slices_first = kmap->K3 == 27 && grid.x > (unsigned)compute_units() && grid.x < 65536 && grid.y == 2;
    if (slices_first) grid = dim3(grid.y, grid.x);
    const int x_bytes = (int)((size_t)kmap->n_in * cin1 * 2), x2_bytes = (int)((size_t)kmap->n_in * (cin - cin1) * 2);
    const int w_bytes = (int)((size_t)kmap->K3 * cin * cout * 2);
// (under the name of the stage, which k_grouped_mm computes for other rows)
#define TS_GROUPED_LINES(TWO) \
    TS_LAUNCH("k_grouped_mm", (k_grouped_lines<NCO, TWO>), grid, dim3(kThreads), static_cast<const _Float16 *>(F), static_cast<const _Float16 *>(X), \
              static_cast<const u32x4 *>(wf), offs_of(kmap), plan, G, cin, cout, kmap->centre, in_idx, x_bytes, w_bytes,                      \
              static_cast<const _Float16 *>(sec.x2), x2_bytes, cin1, slices_first)
    if (sec.x2) TS_GROUPED_LINES(true);
    else TS_GROUPED_LINES(false);
#undef TS_GROUPED_LINES
}

template <class T>
int grouped_mm_launch(const void *F, const void *X, const void *wt, const ts_kmap *kmap, const MmPlan &plan, float *G,
                      int cin_pad, int cout, const int32_t *in_idx = nullptr, const Second &sec = Second()) {
    if (plan_tiles(plan) == 0) return TS_OK;
    if (mm_by_lines(sizeof(T), kmap, cin_pad, sec.x2 ? sec.cin1 : cin_pad, cout)) {
        const int cblocks = cout / 16;
        if (cblocks % 8 == 0) launch_grouped_lines<8>(F, X, wt, kmap, plan, G, cin_pad, cout, in_idx, sec);
        else if (cblocks % 6 == 0) launch_grouped_lines<6>(F, X, wt, kmap, plan, G, cin_pad, cout, in_idx, sec);
        else if (cblocks % 4 == 0) launch_grouped_lines<4>(F, X, wt, kmap, plan, G, cin_pad, cout, in_idx, sec);
        else launch_grouped_lines<2>(F, X, wt, kmap, plan, G, cin_pad, cout, in_idx, sec);
        TS_HIP(hipGetLastError());
        return TS_OK;
    }
    const T *zero = static_cast<const T *>(zero_row());
    if (!zero) return last_fail_code();
    // the chunk of input channels a step takes must divide both parts of a two-part input
    int ksteps = pick_ksteps(cin_pad, Elem<T>::KSTEP);
    const int cin1 = sec.x2 ? sec.cin1 : cin_pad;
    if (sec.x2) {
        const int k1 = pick_ksteps(cin1, Elem<T>::KSTEP), k2 = pick_ksteps(cin_pad - cin1, Elem<T>::KSTEP);
        ksteps = k1 < k2 ? k1 : k2;
    }
    dispatch_shape(pick_ncb(cout), ksteps,
                   GroupedLaunch<T>{static_cast<const T *>(F), static_cast<const T *>(X), static_cast<const T *>(wt),
                                    kmap, plan, G, zero, cin_pad, cout, in_idx, static_cast<const T *>(sec.x2), cin1});
    TS_HIP(hipGetLastError());
    return TS_OK;
}

template <class T>
int grouped_mm_impl(const void *F, const void *X, const void *wt, const ts_kmap *kmap, float *G, int cin_pad,
                    int cout) {
    return grouped_mm_launch<T>(F, X, wt, kmap, whole_plan(kmap), G, cin_pad, cout);
}

// Consecutive indices are grouped while the padded share of the group, 1 - n_min / n_max, stays within
// epsilon (Appendix B, Alg. 4, first loop).  group_of[i] = number of the group index i falls in.
int partition_by_size(const int64_t *sizes, int count, double epsilon, int32_t *group_of) {
    int groups = 0;
    for (int first = 0; first < count;) {
        int64_t lo = sizes[first], hi = sizes[first];
        int next = first + 1;
        for (; next < count; ++next) {
            const int64_t l = sizes[next] < lo ? sizes[next] : lo, h = sizes[next] > hi ? sizes[next] : hi;
            const double padded = h == 0 ? 0.0 : 1.0 - (double)l / (double)h;
            if (padded > epsilon) break;
            lo = l;
            hi = h;
        }
        for (int i = first; i < next; ++i) group_of[i] = groups;
        ++groups;
        first = next;
    }
    return groups;
}

// The grouped matmul the way Appendix B, Alg. 4 schedules it: per group one batched launch with every
// member padded to the longest when that length is below S, else one launch per member.  With an odd
// kernel at stride 1 index i and its mirror K^3-1-i have maps of one size and always share a launch
// (symmetric grouping, Sec. 4.2.3), the groups are formed over the first half of the indices, and the
// centre is a launch of its own.  epsilon < 0: no grouping at all, one launch per offset.
template <class T>
int grouped_mm_adaptive(const void *F, const void *X, const void *wt, const ts_kmap *kmap, float *G, int cin_pad, int cout,
                        double epsilon, int64_t S, int64_t *stats) {
    const int K3 = kmap->K3;
    const bool mirrored = kmap->centre >= 0 && epsilon >= 0;
    const int count = mirrored ? K3 / 2 : K3;
    int32_t group_of[kMaxK3];
    int groups;
    if (epsilon < 0) {
        for (int i = 0; i < count; ++i) group_of[i] = i;
        groups = count;
    } else {
        groups = partition_by_size(kmap->sizes, count, epsilon, group_of);
    }
    int64_t launches = 0, padded_rows = 0;
    auto launch = [&](const MmPlan &plan) -> int {
        if (plan_tiles(plan) == 0) return TS_OK;
        ++launches;
        return grouped_mm_launch<T>(F, X, wt, kmap, plan, G, cin_pad, cout);
    };
    auto add = [&](MmPlan &plan, int n, int64_t rows) {
        plan.n[plan.count] = n;
        plan.tiles[plan.count++] = (int32_t)mm_tiles(rows);
        padded_rows += rows;
    };
    for (int g = 0, first = 0; g < groups; ++g) {
        int next = first;
        int64_t n_max = 0;
        for (; next < count && group_of[next] == g; ++next) n_max = kmap->sizes[next] > n_max ? kmap->sizes[next] : n_max;
        const bool batched = n_max < S;
        MmPlan plan;
        plan.count = 0;
        for (int i = first; i < next; ++i) {
            if (!batched) plan.count = 0;
            const int64_t rows = batched ? n_max : kmap->sizes[i];
            add(plan, i, rows);
            if (mirrored) add(plan, K3 - 1 - i, rows);
            if (!batched) TS_TRY(launch(plan));
        }
        if (batched) TS_TRY(launch(plan));
        first = next;
    }
    if (mirrored) {
        MmPlan plan;
        plan.count = 0;
        add(plan, kmap->centre, kmap->sizes[kmap->centre]);
        TS_TRY(launch(plan));
    }
    if (stats) {
        stats[0] = launches;
        stats[1] = groups;
        stats[2] = padded_rows;
        stats[3] = kmap->M;
    }
    return TS_OK;
}

template <class T>
int reduce_impl(const float *G, const ts_kmap *kmap, ts_tensor *out, const Epilogue &ep = Epilogue()) {
    if (kmap->n_out == 0) return TS_OK;
    const int64_t threads = kmap->n_out * (out->cols / 4);
    if (out->cols % 128 == 0)
        TS_LAUNCH("k_scatter_reduce", (k_scatter_reduce<T, 32>), dim3(blocks_for(threads, kThreads)), dim3(kThreads), G, kmap->d_nbr, kmap->stride, kmap->d_colbits, kmap->d_colbase, offs_of(kmap), kmap->n_blocks, static_cast<T *>(out->data), kmap->n_out, out->cols, kmap->K3, static_cast<const T *>(ep.bias), static_cast<const T *>(ep.residual), ep.relu);
    else if (out->cols % 64 == 0)
        TS_LAUNCH("k_scatter_reduce", (k_scatter_reduce<T, 16>), dim3(blocks_for(threads, kThreads)), dim3(kThreads), G, kmap->d_nbr, kmap->stride, kmap->d_colbits, kmap->d_colbase, offs_of(kmap), kmap->n_blocks, static_cast<T *>(out->data), kmap->n_out, out->cols, kmap->K3, static_cast<const T *>(ep.bias), static_cast<const T *>(ep.residual), ep.relu);
    else
        TS_LAUNCH("k_scatter_reduce", (k_scatter_reduce<T, 0>), dim3(blocks_for(threads, kThreads)), dim3(kThreads), G, kmap->d_nbr, kmap->stride, kmap->d_colbits, kmap->d_colbase, offs_of(kmap), kmap->n_blocks, static_cast<T *>(out->data), kmap->n_out, out->cols, kmap->K3, static_cast<const T *>(ep.bias), static_cast<const T *>(ep.residual), ep.relu);
    TS_HIP(hipGetLastError());
    return TS_OK;
}

template <class T>
int run_explicit(const ts_tensor *feats, const ts_tensor *weights, const ts_kmap *kmap, ts_tensor *out,
                 const ts_weights *pw = nullptr, bool fetch = false, const Epilogue &ep = Epilogue(),
                 const Second &sec = Second()) {
    TS_TRY(resolve(kmap));
    Prepared pr;
    const int cin_step = (feats->cols + Elem<T>::KSTEP - 1) / Elem<T>::KSTEP * Elem<T>::KSTEP;
    TS_TRY(prepare<T>(feats, weights, kmap, &pr, pw, nullptr, mm_by_lines(sizeof(T), kmap, cin_step, sec.x2 ? sec.cin1 : cin_step, out->cols)));
    if (sec.x2 && (!fetch || pr.cin_pad != feats->cols)) return fail(TS_ERR_UNSUPPORTED, "a two-part input needs the fetch-on-demand dataflow and unpadded rows");
    const int64_t M = kmap->M;
    float *G = static_cast<float *>(scratch(1, (size_t)(M ? M : 1) * out->cols * sizeof(float)));
    if (!G) return last_fail_code();
    if (fetch) {   // the matmul reads X_in[j] through the pair lists: no buffer F, no gather launch
        if (M == 0) return reduce_impl<T>(G, kmap, out, ep);
        TS_TRY(ensure_pairs(kmap));
        TS_TRY(grouped_mm_launch<T>(nullptr, pr.x, pr.wt, kmap, whole_plan(kmap), G, pr.cin_pad, out->cols, kmap->d_in_idx, sec));
        return reduce_impl<T>(G, kmap, out, ep);
    }
    void *F = scratch(0, (size_t)(M ? M : 1) * pr.cin_pad * sizeof(T));
    if (!F) return last_fail_code();
    TS_TRY(gather_impl(pr.x, feats->rows, pr.cin_pad, feats->dtype, kmap, F));
    TS_TRY(grouped_mm_impl<T>(F, pr.x, pr.wt, kmap, G, pr.cin_pad, out->cols));
    return reduce_impl<T>(G, kmap, out, ep);
}

}  // namespace

// TS_DATAFLOW_AUTO.  The fused kernel re-reads a layer's weights for every tile of 128 outputs
// (about 20 of the 27 offsets meet an input somewhere in a tile); the explicit dataflow reads
// them once but moves every pair's rows through the buffer G (and F, unless the matmul fetches
// the rows itself, which is the form taken here).  Wide layers on point sets too
// small to fill the machine with tiles (the coarse levels of a U-Net) are cheaper explicit,
// everything else fused; the factor and the size limit come from timing both on the layers of
// the MinkUNet-style benchmark network.
// What the line is drawn by is the number of pairs.  An asynchronous build that nobody has asked does not know its own yet,
// and waiting for it costs a step of a small map and one layer 6 to 20 us.  Whether somebody has asked must not decide, the
// dataflows differ in bits.  So:
//   - fp16 goes by the typical number of surface-like scenes, or the map's own where that is larger: a solid has up to 27 a
//     point where scans and surfaces have 7 to 9, and fetching them costs three times the fused kernel (192 -> 192 on 32 k points
//     of a solid 292 us and 77, 256 -> 256 on 20 k 238 and 97).  Where the layer comes out fused by the typical number it
//     does so by any larger one, and nothing is waited for; where it does not, the explicit dataflow waits in any case.
//     On so few points that the pairs' bytes are less than 40 times the weights that one workgroup goes through, fetching stays
//     ahead however dense they are (192 -> 192, fused and fetched, surfaces 1 k 18 us and 18, 3 k (41 times) 18 and 24, a solid of
//     1 k 33 and 25, of 8 k (300 times) 39 and 68).
//     A smaller number does not count, though fetching gains on scattered points, which have 3 (96 -> 96 on 1 k points 18 us
//     fused and 13 fetched, 128 -> 128 on 8 k 23 and 20; nothing on 32 k or on a thinned-out scan): the wait would take more
//     from a step.
//     The factor was drawn before groups of waves shared a tile (k_conv_tile<..., GR>), and is the same since, so that it is on the
//     safe side for scans and surfaces: fused and fetched, 256 -> 256 on a scan after two halvings, 7.5 k points 42 and 36, 16 k
//     50 and 58, 30 k 75 and 104, 192 -> 192 33 and 30, 39 and 45, 56 and 78, and all of these are fetched; on 30 k scattered
//     points 90 and 55, 62 and 44.
//   - Single precision with weights of 16 KiB an offset and more goes by its own number, and waits for it: the fused kernel
//     walks a tile's offsets at 2.3 us each (64 -> 64; 8.6 at 128 -> 128), however few tiles there are, so that what decides is
//     the pairs' bytes against the weights that one workgroup goes through, a thousand to one by the rates measured: 64 -> 64,
//     fused and fetched, scattered 1 k 67 us and 14, scan 8 k 58 and 20, surfaces 32 k (0.92 of the line) 69 and 55, a solid
//     of 32 k (2.6) 74 and 122; 128 -> 128, surfaces 16 k 199 and 78.  Narrower ones gain less than the wait takes.
//     (Recorded on a map without pair lists, which need memory, such a layer goes by the typical number.)
// (A build that found bad input, or whose sizes cannot be had now, leaves the fused kernel, which needs none.)
// 2x2x2 maps that go up, in fp16 (us, fused and fetched): rows of one offset stand together, so that a tile walks little more
// than one offset, and the two dataflows give the same bits: 64 -> 64 on 300 rows 8.4, 11.1, on 20 k 9.4, 12.3; 256 -> 256 on
// 1 k 13.0, 14.1, on 20 k 16.8, 24.1, but on 300, where three tiles walk 32 stages each, 14.8, 12.4; 160 -> 64 11.7, 10.9.
// Maps that go down share the line of the others.  Drawn at 0.9 times the pairs' bytes it gains on wide outputs (64 -> 128
// from 16 k scattered points 11.8, 15.8, 256 -> 256 from 60 k points of surfaces 26.6, 39.0) but costs more where C_in is the
// larger one, whose stages a tile walks one after the other: 256 -> 64 from 24 k points of a scan 17.2, 14.9, 256 -> 128 from
// 11 k after one halving 17.3, 16.3.  And the two dataflows differ in bits.
bool prefer_explicit(const ts_kmap *kmap, int cin, int cout, size_t elem) {
    if (kmap->n_tiles > compute_units()) return false;
    if (elem == 2 && goes_up_by_two(kmap) && (cin <= 128 || kmap->n_out >= 4 * kTileRows)) return false;
    const double tile_offsets = kmap->K3 < 20 ? kmap->K3 : 20;
    const double fine = kmap->transposed ? kmap->n_out : kmap->n_in;
    const double typical = kmap->s == 1 ? (kmap->K3 > 1 ? 7.5 : 1.0) * fine : fine * kmap->K3 / 8.0;
    const double slabs = tile_offsets * cin * cout * elem, fused_weight_bytes = (double)kmap->n_tiles * slabs;
    const double bytes_per_pair = 2.0 * cin * elem + 2.0 * cout * sizeof(float);
    const bool wide_f32 = elem == 4 && kmap->s == 1 && kmap->K3 == 27 && cin * cout >= 4096 && (kmap->d_in_idx || !stream_capturing(stream()));
    if (!wide_f32 && fused_weight_bytes <= 0.6 * typical * bytes_per_pair) return false;
    if (resolve(kmap) != TS_OK) return false;
    const double pair_bytes = (double)kmap->M * bytes_per_pair;
    if (wide_f32) return pair_bytes < 1000 * slabs;
    return (double)kmap->M <= typical || fused_weight_bytes > 0.6 * pair_bytes || pair_bytes < 40 * slabs;
}

// ---- the layer for callers that cannot allocate -----------------------------------------------------------
// ts_sparse_conv's kernels take two pieces of memory beyond their inputs and outputs: the weights repacked
// into operand order (a staging buffer written by k_pack_weights* and read by the layer kernel) and, for
// TS_F32, a row of zeros that stands in for absent neighbours.  Here both live in one array that is part of
// the library's code object, so that a call reaches no allocator: [0, 4 KiB) zeros, then the packed weights.
constexpr size_t kStaticZeroBytes = 4096;
constexpr size_t kStaticWeightBytes = size_t(4) << 20;
static __device__ __align__(256) unsigned char g_static_scratch[kStaticZeroBytes + kStaticWeightBytes];

namespace {
constexpr int kMaxDevices = 64;
unsigned char *g_static_ptr[kMaxDevices] = {nullptr};   // per device: where that device holds its copy of the array

__global__ void k_clear_words(uint32_t *p, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0u;
}

// The device address of the array on the current device (looked up once per device).
int static_scratch(unsigned char **ptr) {
    int dev = -1;
    TS_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return fail(TS_ERR_UNSUPPORTED, "device ordinal %d is beyond %d", dev, kMaxDevices - 1);
    if (!g_static_ptr[dev]) {
        void *p = nullptr;
        TS_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(g_static_scratch)));
        if (!p) return fail(TS_ERR_HIP, "hipGetSymbolAddress gave no address");
        g_static_ptr[dev] = static_cast<unsigned char *>(p);
    }
    *ptr = g_static_ptr[dev];
    return TS_OK;
}
}  // namespace

extern "C" {

int ts_sparse_conv_static(const ts_tensor *feats, const ts_tensor *weights, const ts_kmap *kmap, ts_tensor *out) {
    if (kmap) TS_TRY(resolve_count(kmap, false));
    TS_TRY(check_layer(feats, weights, kmap, out));
    const bool f16 = feats->dtype == TS_F16;
    const int cin = feats->cols, cout = out->cols, step = f16 ? 32 : Elem<float>::KSTEP;
    if (cin % step != 0) return fail(TS_ERR_UNSUPPORTED, "ts_sparse_conv_static: C_in must be a multiple of %d, got %d (ts_sparse_conv pads narrower rows, in memory it allocates)", step, cin);
    const size_t wbytes = (size_t)kmap->K3 * cin * cout * (f16 ? 2 : 4);
    if (wbytes > kStaticWeightBytes)
        return fail(TS_ERR_UNSUPPORTED, "ts_sparse_conv_static: the weights take %zu bytes, the static area holds %zu (K^3 * C_in * C_out * element size)", wbytes, kStaticWeightBytes);
    if (kmap->n_out == 0) return TS_OK;
    unsigned char *base = nullptr;
    TS_TRY(static_scratch(&base));
    void *wbuf = base + kStaticZeroBytes;
    if (f16) return run_fused_f16(feats, weights, kmap, out, Epilogue(), nullptr, wbuf);
    // the zeros are never written by a layer kernel; they are cleared all the same, so that nothing rests on
    // what an earlier user of the array left there (a fill kernel, not a memset: a caller may be capturing)
    TS_LAUNCH("k_clear_words", k_clear_words, dim3((unsigned)(kStaticZeroBytes / 4 / kThreads)), dim3(kThreads), reinterpret_cast<uint32_t *>(base), (int)(kStaticZeroBytes / 4));
    return run_fused_staged<float>(feats, weights, kmap, out, nullptr, wbuf, base);
}

int ts_sparse_conv_ex(const ts_tensor *feats, const ts_tensor *weights, const ts_kmap *kmap, ts_tensor *out,
                      int dataflow) {
    TS_TRY(check_layer(feats, weights, kmap, out));
    if (dataflow != TS_DATAFLOW_AUTO && dataflow != TS_DATAFLOW_EXPLICIT && dataflow != TS_DATAFLOW_FUSED &&
        dataflow != TS_DATAFLOW_FUSED_STAGED && dataflow != TS_DATAFLOW_FETCH)
        return fail(TS_ERR_INVALID_ARG, "unknown dataflow %d", dataflow);
    if (kmap->n_out == 0) return TS_OK;
    const bool f16 = feats->dtype == TS_F16;
    if (dataflow == TS_DATAFLOW_AUTO && prefer_explicit(kmap, feats->cols, out->cols, f16 ? 2 : 4)) dataflow = TS_DATAFLOW_FETCH;
    if (dataflow == TS_DATAFLOW_EXPLICIT || dataflow == TS_DATAFLOW_FETCH) {
        const bool fetch = dataflow == TS_DATAFLOW_FETCH;
        return f16 ? run_explicit<_Float16>(feats, weights, kmap, out, nullptr, fetch)
                   : run_explicit<float>(feats, weights, kmap, out, nullptr, fetch);
    }
    if (dataflow == TS_DATAFLOW_FUSED_STAGED)
        return f16 ? run_fused_staged<_Float16>(feats, weights, kmap, out) : run_fused_staged<float>(feats, weights, kmap, out);
    return f16 ? run_fused<_Float16>(feats, weights, kmap, out) : run_fused<float>(feats, weights, kmap, out);
}

int ts_sparse_conv(const ts_tensor *feats, const ts_tensor *weights, const ts_kmap *kmap, ts_tensor *out) {
    return ts_sparse_conv_ex(feats, weights, kmap, out, TS_DATAFLOW_AUTO);
}

// The layer with its optional elementwise tail; pw, when given, holds the weights already packed.
static int conv_act(const ts_tensor *feats_in, const ts_tensor *weights, const ts_weights *pw, const ts_kmap *kmap,
                    const void *bias, const ts_tensor *residual, int relu, ts_tensor *out,
                    const ts_tensor *feats2 = nullptr) {
    // With feats2 the layer's input is [feats_in | feats2] along the channels.  Where the kernels can read
    // the two parts in place (fp16 fused: both parts multiples of 32 channels; fetch-on-demand: multiples of
    // the operand step) the concatenation is never formed; otherwise it is formed in scratch memory first.
    ts_tensor cat;
    const ts_tensor *feats = feats_in;
    Second sec;
    if (feats2) {
        TS_TRY(check_tensor(feats_in, "feats"));
        TS_TRY(check_tensor(feats2, "feats2"));
        if (feats2->rows != feats_in->rows || feats2->dtype != feats_in->dtype)
            return fail(TS_ERR_SHAPE, "feats2 must have the rows and dtype of feats");
        cat = *feats_in;
        cat.cols = feats_in->cols + feats2->cols;
        feats = &cat;
        sec.x2 = feats2->data;
        sec.cin1 = feats_in->cols;
    }
    TS_TRY(check_layer(feats, weights, kmap, out));
    if (residual) {
        TS_TRY(check_tensor(residual, "residual"));
        if (residual->rows != out->rows || residual->cols != out->cols || residual->dtype != out->dtype)
            return fail(TS_ERR_SHAPE, "residual must have the shape and dtype of out");
        if (residual->data == out->data) return fail(TS_ERR_INVALID_ARG, "residual must not alias out");
    }
    if (bias && (reinterpret_cast<uintptr_t>(bias) & 15)) return fail(TS_ERR_INVALID_ARG, "bias must be 16-byte aligned");
    if (kmap->n_out == 0) return TS_OK;
    const bool f16 = feats->dtype == TS_F16;
    const bool go_explicit = prefer_explicit(kmap, feats->cols, out->cols, f16 ? 2 : 4);
    if (feats2) {
        const int step = go_explicit ? kstep(feats->dtype) : 32;
        const bool in_place = (f16 || go_explicit) && feats_in->cols % step == 0 && feats2->cols % step == 0 &&
                              (go_explicit || ((size_t)kmap->n_in * feats->cols * 2 < (1ull << 31)));
        if (!in_place) {
            void *buf = scratch(4, (size_t)(feats->rows ? feats->rows : 1) * feats->cols * (f16 ? 2 : 4));
            if (!buf) return last_fail_code();
            cat.data = buf;
            TS_TRY(ts_concat_cols(feats_in, feats2, &cat));
            sec = Second();
        }
    }
    Epilogue ep;
    ep.bias = bias;
    ep.residual = residual ? residual->data : nullptr;
    ep.relu = relu != 0;
    if (f16 && !go_explicit) return run_fused_f16(feats, weights, kmap, out, ep, pw, nullptr, sec);
    // fetch-on-demand: the tail runs in the scatter-accumulate kernel
    if (go_explicit)
        return f16 ? run_explicit<_Float16>(feats, weights, kmap, out, pw, true, ep, sec) : run_explicit<float>(feats, weights, kmap, out, pw, true, ep, sec);
    // otherwise (fp32, fused): the layer, then the elementwise step on its output
    TS_TRY(run_fused<float>(feats, weights, kmap, out, pw));
    if (!bias && !residual && !relu) return TS_OK;
    return ts_bias_act(out, bias, residual, relu, out);
}

int ts_sparse_conv_act(const ts_tensor *feats, const ts_tensor *weights, const ts_kmap *kmap, const void *bias,
                       const ts_tensor *residual, int relu, ts_tensor *out) {
    return conv_act(feats, weights, nullptr, kmap, bias, residual, relu, out);
}

int ts_weights_prepare(const ts_tensor *weights, int kernel_volume, ts_weights **out_weights) {
    if (!out_weights) return fail(TS_ERR_INVALID_ARG, "out_weights is NULL");
    *out_weights = nullptr;
    TS_TRY(check_tensor(weights, "weights"));
    if (kernel_volume != 1 && kernel_volume != 8 && kernel_volume != 27) return fail(TS_ERR_INVALID_ARG, "kernel_volume must be 1, 8 or 27");
    if (weights->rows <= 0 || weights->rows % kernel_volume != 0) return fail(TS_ERR_SHAPE, "weights must be [K^3*C_in, C_out]");
    const int cin = (int)(weights->rows / kernel_volume), cout = weights->cols;
    if (cout % 32 != 0 || cout > 1024 || cin > 1024) return fail(TS_ERR_UNSUPPORTED, "C_out must be a multiple of 32, C_in and C_out at most 1024");
    ts_weights *w = new (std::nothrow) ts_weights();
    if (!w) return fail(TS_ERR_OOM, "host allocation failed");
    w->K3 = kernel_volume;
    w->cin = cin;
    w->cout = cout;
    w->dtype = weights->dtype;
    const bool f16 = weights->dtype == TS_F16;
    const int ks = f16 ? Elem<_Float16>::KSTEP : Elem<float>::KSTEP;
    const int cin_wt = (cin + ks - 1) / ks * ks;
    const size_t n_wt = (size_t)kernel_volume * cout * cin_wt;
    w->wt = dev_alloc(n_wt * elem_size(weights->dtype));
    if (!w->wt) {
        delete w;
        return TS_ERR_OOM;
    }
    if (f16)
        TS_LAUNCH("k_pack_weights", k_pack_weights<_Float16>, dim3(blocks_for((int64_t)n_wt, kThreads)), dim3(kThreads), static_cast<const _Float16 *>(weights->data), static_cast<_Float16 *>(w->wt), kernel_volume, cin, cin_wt, cout);
    else
        TS_LAUNCH("k_pack_weights", k_pack_weights<float>, dim3(blocks_for((int64_t)n_wt, kThreads)), dim3(kThreads), static_cast<const float *>(weights->data), static_cast<float *>(w->wt), kernel_volume, cin, cin_wt, cout);
    if (f16) {
        const int cin_tile = (cin + 31) / 32 * 32, ksteps = tile_ksteps(cin_tile);
        const size_t n_tile = (size_t)kernel_volume * cout * cin_tile;
        w->tile = dev_alloc(n_tile * 2);
        if (!w->tile) {
            dev_free(w->wt);
            delete w;
            return TS_ERR_OOM;
        }
        TS_LAUNCH("k_pack_weights", k_pack_weights_tile, dim3(blocks_for((int64_t)n_tile, kThreads)), dim3(kThreads), static_cast<const _Float16 *>(weights->data), static_cast<_Float16 *>(w->tile), kernel_volume, cin, cin_tile, cout, ksteps);
    }
    TS_HIP(hipGetLastError());
    *out_weights = w;
    return TS_OK;
}

void ts_weights_free(ts_weights *w) {
    if (!w) return;
    dev_free(w->wt);
    dev_free(w->tile);
    delete w;
}

int ts_sparse_conv_prepared(const ts_tensor *feats, const ts_weights *w, const ts_kmap *kmap, const void *bias,
                            const ts_tensor *residual, int relu, ts_tensor *out) {
    if (!w) return fail(TS_ERR_INVALID_ARG, "weights is NULL");
    if (kmap && w->K3 != kmap->K3) return fail(TS_ERR_SHAPE, "weights were prepared for kernel volume %d, the map has %d", w->K3, kmap->K3);
    const ts_tensor desc = {w->wt, (int64_t)w->K3 * w->cin, w->cout, w->dtype};   // shape and dtype for the checks
    return conv_act(feats, &desc, w, kmap, bias, residual, relu, out);
}

int ts_sparse_conv_prepared2(const ts_tensor *feats, const ts_tensor *feats2, const ts_weights *w, const ts_kmap *kmap,
                             const void *bias, const ts_tensor *residual, int relu, ts_tensor *out) {
    if (!w) return fail(TS_ERR_INVALID_ARG, "weights is NULL");
    if (kmap && w->K3 != kmap->K3) return fail(TS_ERR_SHAPE, "weights were prepared for kernel volume %d, the map has %d", w->K3, kmap->K3);
    const ts_tensor desc = {w->wt, (int64_t)w->K3 * w->cin, w->cout, w->dtype};
    return conv_act(feats, &desc, w, kmap, bias, residual, relu, out, feats2);
}

int ts_gather_ex(const ts_tensor *feats, const ts_kmap *kmap, ts_tensor *F, int order) {
    if (!kmap) return fail(TS_ERR_INVALID_ARG, "kmap is NULL");
    if (order != TS_GATHER_AUTO && order != TS_GATHER_OUTPUT_ORDER && order != TS_GATHER_INPUT_STATIONARY)
        return fail(TS_ERR_INVALID_ARG, "unknown gather order %d", order);
    TS_TRY(resolve(kmap));
    TS_TRY(check_tensor(feats, "feats"));
    TS_TRY(check_tensor(F, "F"));
    if (feats->rows != kmap->n_in) return fail(TS_ERR_SHAPE, "feats has %lld rows, the map expects %lld", (long long)feats->rows, (long long)kmap->n_in);
    if (F->rows != kmap->M || F->cols != feats->cols || F->dtype != feats->dtype)
        return fail(TS_ERR_SHAPE, "F must be [num_pairs, C_in] of the dtype of feats");
    if ((feats->cols * elem_size(feats->dtype)) % 16 != 0)
        return fail(TS_ERR_UNSUPPORTED, "rows must be a multiple of 16 bytes");
    return gather_impl(feats->data, feats->rows, feats->cols, feats->dtype, kmap, F->data, order);
}

int ts_gather(const ts_tensor *feats, const ts_kmap *kmap, ts_tensor *F) { return ts_gather_ex(feats, kmap, F, TS_GATHER_AUTO); }

int ts_adaptive_groups(const int64_t *sizes, int32_t count, double epsilon, int32_t *group_of, int32_t *num_groups) {
    if (!sizes || !group_of || !num_groups) return fail(TS_ERR_INVALID_ARG, "sizes, group_of and num_groups must not be NULL");
    if (count < 0 || count > kMaxK3) return fail(TS_ERR_INVALID_ARG, "count must be in [0, %d]", kMaxK3);
    if (!(epsilon >= 0.0 && epsilon <= 1.0)) return fail(TS_ERR_INVALID_ARG, "epsilon must be in [0, 1]");
    for (int i = 0; i < count; ++i)
        if (sizes[i] < 0) return fail(TS_ERR_INVALID_ARG, "sizes[%d] is negative", i);
    *num_groups = partition_by_size(sizes, count, epsilon, group_of);
    return TS_OK;
}

static int grouped_matmul_checked(const ts_tensor *F, const ts_tensor *feats, const ts_tensor *weights, const ts_kmap *kmap,
                                  ts_tensor *G, bool adaptive, double epsilon, int64_t S, int64_t *stats) {
    if (!kmap) return fail(TS_ERR_INVALID_ARG, "kmap is NULL");
    TS_TRY(resolve(kmap));
    TS_TRY(check_tensor(F, "F"));
    TS_TRY(check_tensor(weights, "weights"));
    TS_TRY(check_tensor(G, "G"));
    if (kmap->centre >= 0) {
        TS_TRY(check_tensor(feats, "feats"));
        if (feats->rows != kmap->n_in || feats->cols != F->cols || feats->dtype != F->dtype)
            return fail(TS_ERR_SHAPE, "feats must be [num_in, C_in] of the dtype of F");
    }
    if (F->rows != kmap->M || G->rows != kmap->M) return fail(TS_ERR_SHAPE, "F and G must have num_pairs rows");
    if (weights->dtype != F->dtype || G->dtype != TS_F32) return fail(TS_ERR_SHAPE, "weights must match F; G must be TS_F32");
    if (weights->rows != (int64_t)kmap->K3 * F->cols || weights->cols != G->cols)
        return fail(TS_ERR_SHAPE, "weights must be [K^3*C_in, C_out]");
    if (G->cols % 32 != 0 || F->cols % kstep(F->dtype) != 0)
        return fail(TS_ERR_UNSUPPORTED, "C_out must be a multiple of 32 and C_in of %d", kstep(F->dtype));
    // weights only: the rows of F are already in the operand layout
    ts_tensor none = {nullptr, 0, F->cols, F->dtype};
    Prepared pr;
    const void *X = feats ? feats->data : nullptr;
    float *g = static_cast<float *>(G->data);
    if (F->dtype == TS_F16) {
        TS_TRY(prepare<_Float16>(&none, weights, kmap, &pr, nullptr, nullptr, mm_by_lines(2, kmap, F->cols, F->cols, G->cols)));
        return adaptive ? grouped_mm_adaptive<_Float16>(F->data, X, pr.wt, kmap, g, F->cols, G->cols, epsilon, S, stats)
                        : grouped_mm_impl<_Float16>(F->data, X, pr.wt, kmap, g, F->cols, G->cols);
    }
    TS_TRY(prepare<float>(&none, weights, kmap, &pr));
    return adaptive ? grouped_mm_adaptive<float>(F->data, X, pr.wt, kmap, g, F->cols, G->cols, epsilon, S, stats)
                    : grouped_mm_impl<float>(F->data, X, pr.wt, kmap, g, F->cols, G->cols);
}

int ts_grouped_matmul(const ts_tensor *F, const ts_tensor *feats, const ts_tensor *weights, const ts_kmap *kmap,
                      ts_tensor *G) {
    return grouped_matmul_checked(F, feats, weights, kmap, G, false, 0.0, 0, nullptr);
}

int ts_grouped_matmul_adaptive(const ts_tensor *F, const ts_tensor *feats, const ts_tensor *weights, const ts_kmap *kmap,
                               double epsilon, int64_t S, ts_tensor *G, int64_t *stats) {
    if (!(epsilon <= 1.0)) return fail(TS_ERR_INVALID_ARG, "epsilon must be at most 1 (negative: no grouping)");
    if (S < 0) return fail(TS_ERR_INVALID_ARG, "S must not be negative");
    return grouped_matmul_checked(F, feats, weights, kmap, G, true, epsilon, S, stats);
}

int ts_scatter_reduce(const ts_tensor *G, const ts_kmap *kmap, ts_tensor *out) {
    if (!kmap) return fail(TS_ERR_INVALID_ARG, "kmap is NULL");
    TS_TRY(resolve(kmap));
    TS_TRY(check_tensor(G, "G"));
    TS_TRY(check_tensor(out, "out"));
    if (G->dtype != TS_F32 || G->rows != kmap->M) return fail(TS_ERR_SHAPE, "G must be TS_F32 [num_pairs, C_out]");
    if (out->rows != kmap->n_out || out->cols != G->cols) return fail(TS_ERR_SHAPE, "out must be [num_out, C_out]");
    if (out->cols % 4 != 0) return fail(TS_ERR_UNSUPPORTED, "C_out must be a multiple of 4");
    return out->dtype == TS_F16 ? reduce_impl<_Float16>(static_cast<const float *>(G->data), kmap, out)
                                : reduce_impl<float>(static_cast<const float *>(G->data), kmap, out);
}

}  // extern "C"
