// LM head with the vocabulary reduction as its epilogue: the last layer of
// the forward f_theta of Alg. 1, Z = H W^T, reduced per row to the symbols of
// Eq. 1 (max, lowest index of the max, sum of exponentials) without the
// logits ever reaching memory.
//
// lmhead_kernel   one workgroup of 8 waves per (256-row token tile, vocabulary
//                 partition).  It walks the partition's 256-id vocabulary
//                 tiles; for each, Z^T tile = W_tile . H_tile^T on
//                 v_mfma_f32_32x32x16_bf16 over K = D in 64-wide stages
//                 (double-buffered LDS, filled by direct global->LDS loads
//                 with a scalar base and a per-lane offset fixed for the
//                 whole kernel), then folds the tile into a running
//                 (max, index, scaled sum) per token.  Wave (wv, wt) owns
//                 vocabulary rows wv*128.. and tokens wt*64.. of the tile.
//                 With Z^T in the accumulators each lane holds one token and
//                 16 vocabulary ids per MFMA tile, so the per-token reduction
//                 is mostly in-lane.  Up to 128 rows: lm_few_rows.
// lm_merge_kernel one wave per row: merges the row's partition partials in a
//                 fixed order into the first partial of the update workspace
//                 (the rest are set empty), the input of the update kernel.
#include <climits>
#include <map>
#include <mutex>
#include <tuple>

#include "internal.h"
#include "top.h"

namespace fb {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr int kLmThreads = 512;                   // 8 waves
constexpr int kTileV = 256;                       // vocabulary ids per tile
constexpr int kTileT = 256;                       // tokens per tile
constexpr int kBK = 64;                           // K per stage
constexpr int kRowBytes = kBK * 2;                // 128 B: one row of a stage
constexpr int kHalfBytes = kTileV * kRowBytes;    // 32 KB: W part of a stage
constexpr int kStageBytes = 2 * kHalfBytes;       // W part, then H part
constexpr int kStages = 2;
constexpr int kFewRows = 128;                     // rows the weight-streaming form takes
constexpr int kFewStages = 3;
constexpr int kMergeThreads = 256;

// LDS reads drained, then a workgroup barrier.  The wait is the builtin, not
// inline asm, so the compiler knows the reads issued before it are complete
// and does not wait for them again after the barrier (behind newer reads).
__device__ inline void lds_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0); vmcnt and expcnt not waited
    asm volatile("s_barrier" ::: "memory");
}
__device__ inline void wait_vm0() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Vocabulary partitions for n_lt token tiles.  One workgroup runs per CU at
// a time, so the kernel takes about (rounds of workgroups over the CUs) x
// (tiles of the largest partition + a workgroup's fixed start and end,
// about 1/8 of a tile); the partition count P minimizes that (the smallest
// such P), with P <= kMaxParts.  Host and device evaluate the same integer
// expression, so both sides agree on P.
constexpr int kMaxParts = 1024;
__host__ __device__ inline long long lm_cost(int n_lt, int nv, int cu, int P) {
    return (long long)((n_lt * P + cu - 1) / cu) * (((nv + P - 1) / P) * 8 + 1);
}
inline int lm_parts_host(int n_lt, int nv, int cu) {
    const int pmax = nv < kMaxParts ? nv : kMaxParts;
    int best = 1;
    long long best_c = lm_cost(n_lt, nv, cu, 1);
    for (int P = 2; P <= pmax; ++P) {
        const long long c = lm_cost(n_lt, nv, cu, P);
        if (c < best_c) best_c = c, best = P;
    }
    return best;
}
// the same choice by one wave (lane i tries P = i + 1, i + 65, ...); every
// lane returns it
__device__ inline int lm_parts_dev(int n_lt, int nv, int cu) {
    const int lane = threadIdx.x & 63;
    const int pmax = nv < kMaxParts ? nv : kMaxParts;
    long long key = LLONG_MAX;   // cost * 2048 + P: the minimum is the smallest P of least cost
    for (int P = lane + 1; P <= pmax; P += 64) {
        const long long k = lm_cost(n_lt, nv, cu, P) * 2048 + P;
        key = k < key ? k : key;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const long long o = __shfl_xor(key, off, 64);
        key = o < key ? o : key;
    }
    return __builtin_amdgcn_readfirstlane((int)(key & 2047));   // uniform: keeps it scalar
}

// ---- few rows: the weight streamed once -----------------------------------
// With at most 128 rows the MFMAs of a 256-token tile are mostly padding, so
// the tile is 64 or 128 tokens wide and the kernel is bound by reading W.  The
// vocabulary goes to the CUs in equal contiguous ranges of 32-id groups; a
// wave owns one group of a tile of eight and all tokens, so the W rows it
// loads are its own, and a wave past the range's end loads and multiplies
// nothing.  Three 64-wide stages in LDS keep two stages of loads in flight.
//
// K is summed as two halves, (first) + (second), and every other workgroup
// takes the second half first: with every CU at the same K offset the 128-byte
// pieces read at one time fall on few memory channels where D is a power of
// two.  The sum of two is the same in either order, so a row of W gives the
// same logit in any workgroup (equal rows tie exactly).  It is not the sum of
// the 256-token form, which takes K in one chain: a row's logits may differ by
// float32 rounding with the form that its pack gets.
//
// Measured (96 rows, V = 157184, D = 2048: 644 MB of W, 92 us at the read
// probe's 7.06 TB/s): 180-198 us with the 256-token
// tile, 106-111 us here (64 rows: 190 -> 111 us for the whole call; all workgroups
// starting K together and without the nontemporal hint: 145-150 us).  From 129
// rows on it is the 256-token tile again (160 rows 198 us, 256 rows 205): here 256
// tokens would take 128 accumulators and as many for the second sum of K, all
// of a wave's registers.
__host__ __device__ inline int lm_few_parts(int V, int cu) {
    const int groups = (V + 31) / 32;
    return groups < cu ? groups : cu;
}

__device__ inline void wait_vm_n(bool more, int n_more, int n_less) {
    // n_more or n_less loads may stay in flight (both among 1, 2, 5, 6)
    const int n = more ? n_more : n_less;
    if (n == 1) asm volatile("s_waitcnt vmcnt(1)" ::: "memory");
    else if (n == 2) asm volatile("s_waitcnt vmcnt(2)" ::: "memory");
    else if (n == 5) asm volatile("s_waitcnt vmcnt(5)" ::: "memory");
    else if (n == 6) asm volatile("s_waitcnt vmcnt(6)" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

template <int NT>   // 32-token groups: 2 or 4
__device__ __attribute__((always_inline)) inline void
lm_few_rows(const uint16_t* __restrict__ H, const uint16_t* __restrict__ W, int D, int V,
            int row_cap, int cu, const PackView& pv, float4* __restrict__ part,
            unsigned char* lds) {
    constexpr int NH = NT / 2;                       // H loads of a wave per stage
    constexpr int kStage = kHalfBytes + NT * 32 * kRowBytes;
    const int P = lm_few_parts(V, cu);
    const int blk = blockIdx.x;
    if (blk >= P) return;
    const int groups = (V + 31) / 32;
    const int g0 = (int)((long long)blk * groups / P);
    const int g1 = (int)((long long)(blk + 1) * groups / P);

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // scalar: so is its group
    const int lane = tid & 63;
    const int n = lane & 31;
    const int h = lane >> 5;
    const int lrow = lane >> 3;

    // loads: 8 rows of 128 bytes per instruction, chunks swizzled with
    // (row/2)%8 as in the 256-token form
    uint32_t w_off[4], h_off[NH];
    auto chunk = [&](int r) { return (lane & 7) ^ ((r >> 1) & 7); };
#pragma unroll
    for (int j = 0; j < NH; ++j) {
        const int r = (wave * NH + j) * 8 + lrow;
        h_off[j] = (uint32_t)(((size_t)min(r, row_cap - 1) * D + chunk(r) * 8) * 2);
    }
    auto set_group = [&](int grp) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int r = j * 8 + lrow;
            const int id = min(grp * 32 + r, V - 1);
            w_off[j] = (uint32_t)(((size_t)id * D + chunk(r) * 8) * 2);
        }
    };
    const uint32_t lds0 = (uint32_t)(uintptr_t)lds;
    const uint32_t m0_w = __builtin_amdgcn_readfirstlane(lds0 + wave * 4096);
    const uint32_t m0_h = __builtin_amdgcn_readfirstlane(lds0 + kHalfBytes + wave * NH * 1024);

    const int KS = D / kBK;
    const int tiles = (g1 - g0 + 7) / 8;
    const int T = tiles * KS;
    // K stages in the order taken: from k_start to the end, then from 0
    const int half = (KS + 1) / 2;
    const int k_start = (blk & 1) && KS > 1 ? half : 0;
    const int n_first = (blk & 1) && KS > 1 ? KS - half : half;   // stages before the turn
    int ld_ks = 0, ld_grp = g0 + wave, ld_slot = 0;   // the next stage to load
    bool ld_live = ld_grp < g1;
    set_group(ld_grp);
    auto issue = [&]() {
        const uint32_t so = ld_slot * kStage;
        const int kz = ld_ks + k_start < KS ? ld_ks + k_start : ld_ks + k_start - KS;
        const uint16_t* wb = W + kz * kBK;
        const uint16_t* hb = H + kz * kBK;
        if (ld_live) {
#pragma unroll
            for (int j = 0; j < 4; ++j)   // read once: nontemporal
                asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2 nt"
                             :: "s"(m0_w + so + j * 1024), "v"(w_off[j]), "s"(wb) : "memory");
        }
#pragma unroll
        for (int j = 0; j < NH; ++j)
            asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2"
                         :: "s"(m0_h + so + j * 1024), "v"(h_off[j]), "s"(hb) : "memory");
        ld_slot = ld_slot == kFewStages - 1 ? 0 : ld_slot + 1;
        if (++ld_ks == KS) {
            ld_ks = 0;
            ld_grp += 8;
            ld_live = ld_grp < g1;
            set_group(ld_grp);
        }
    };

    const uint32_t swz = (uint32_t)((h ^ ((n >> 1) & 7)) * 16);
    const uint32_t a_row = (uint32_t)((wave * 32 + n) * kRowBytes);
    const uint32_t b_row = (uint32_t)(kHalfBytes + n * kRowBytes);
    floatx16 acc[NT], done[NT];   // the half being summed, the half before it
    Top top[NT];
#pragma unroll
    for (int ti = 0; ti < NT; ++ti) {
        acc[ti] = done[ti] = floatx16{};
        top[ti] = top_empty();
    }

    issue();
    bool next_live = ld_live;   // whether stage s + 1 holds loads of W for this wave
    if (T > 1) issue();
    int s = 0, slot = 0;
    // One stage: it has landed (stage s + 1 may be in flight), and every wave
    // is done with stage s - 1, whose slot takes stage s + 2.  The fragments
    // of K step kk + 1 are read under the MFMAs of kk.
    auto stage = [&](bool live) __attribute__((always_inline)) {
        if (s + 1 < T) wait_vm_n(next_live, 4 + NH, NH);
        else wait_vm0();
        lds_barrier();
        if (s + 2 < T) {
            next_live = ld_live;
            issue();
        }
        if (live) {
            const unsigned char* st = lds + slot * kStage;
            bf16x8 a[2], b[2][NT];
            auto read = [&](int kk) __attribute__((always_inline)) {
                const uint32_t ko = swz ^ (uint32_t)(kk << 5);
                a[kk & 1] = *reinterpret_cast<const bf16x8*>(st + a_row + ko);
#pragma unroll
                for (int ti = 0; ti < NT; ++ti)
                    b[kk & 1][ti] = *reinterpret_cast<const bf16x8*>(
                        st + b_row + ti * 32 * kRowBytes + ko);
            };
            read(0);
#pragma unroll
            for (int kk = 0; kk < kBK / 16; ++kk) {
                if (kk + 1 < kBK / 16) read(kk + 1);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int ti = 0; ti < NT; ++ti)
                    acc[ti] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[kk & 1], b[kk & 1][ti],
                                                                      acc[ti], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        slot = slot == kFewStages - 1 ? 0 : slot + 1;
        ++s;
    };
    for (int grp = g0 + wave, tile = 0; tile < tiles; ++tile, grp += 8) {
        const bool live = grp < g1;
        for (int ks = 0; ks < n_first; ++ks) stage(live);
#pragma unroll
        for (int ti = 0; ti < NT; ++ti) {
            done[ti] = acc[ti];
            acc[ti] = floatx16{};
        }
        for (int ks = n_first; ks < KS; ++ks) stage(live);
        if (!live) continue;
        // lane value r is id grp*32 + (r/4)*8 + h*4 + r%4: increasing in r
        const int vbase = grp * 32 + h * 4;
#pragma unroll
        for (int ti = 0; ti < NT; ++ti) {
            float f[16];
#pragma unroll
            for (int r = 0; r < 16; ++r)
                f[r] = vbase + (r >> 2) * 8 + (r & 3) < V ? acc[ti][r] + done[ti][r] : -INFINITY;
            float vmax = f[0];
#pragma unroll
            for (int r = 1; r < 16; ++r) vmax = fmaxf(vmax, f[r]);
            Top& t = top[ti];
            if (vmax > t.m) {
#pragma clang fp contract(off)
                int r0 = 15;
#pragma unroll
                for (int r = 15; r >= 0; --r)
                    if (f[r] == vmax) r0 = r;
                const float nmL = scaled_ref(vmax);
                t.s *= __builtin_amdgcn_exp2f(t.mL - nmL);
                t.m = vmax;
                t.mL = nmL;
                t.idx = vbase + (r0 >> 2) * 8 + (r0 & 3);
            }
            if (t.m != -INFINITY) {
                float e[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    e[r & 3] += __builtin_amdgcn_exp2f(fmaf(f[r], kLog2e, -t.mL));
                t.s += (e[0] + e[1]) + (e[2] + e[3]);
            }
            acc[ti] = floatx16{};
        }
    }

    // lane halves, then the eight waves of each token in order
    __syncthreads();   // the stages' LDS is reused
    Top* s_w = reinterpret_cast<Top*>(lds);   // [8][NT * 32]
#pragma unroll
    for (int ti = 0; ti < NT; ++ti) {
        Top o;
        o.m = __shfl_xor(top[ti].m, 32, 64);
        o.mL = __shfl_xor(top[ti].mL, 32, 64);
        o.s = __shfl_xor(top[ti].s, 32, 64);
        o.idx = __shfl_xor(top[ti].idx, 32, 64);
        const Top t = top_merge(top[ti], o);
        if (h == 0) s_w[wave * NT * 32 + ti * 32 + n] = t;
    }
    __syncthreads();
    if (tid < NT * 32 && tid < row_cap && pv.row_req[tid] >= 0) {
        Top t = s_w[tid];
        for (int w = 1; w < 8; ++w) t = top_merge(t, s_w[w * NT * 32 + tid]);
        part[(size_t)blk * kTileT + tid] = top_pack(t);
    }
}

__global__ void __launch_bounds__(kLmThreads, 1)
lm_few_kernel(const uint16_t* __restrict__ H, const uint16_t* __restrict__ W, int D, int V,
              int row_cap, int padded, int cu, PackView pv, float4* __restrict__ part) {
    __shared__ __attribute__((aligned(16))) unsigned char
        lds[kFewStages * (kHalfBytes + kFewRows * kRowBytes)];
    const int n_rows = padded ? row_cap : pv.hdr[kHdrRows];
    if (n_rows < 1 || n_rows > kFewRows) return;
    if (n_rows > 64) lm_few_rows<4>(H, W, D, V, row_cap, cu, pv, part, lds);
    else lm_few_rows<2>(H, W, D, V, row_cap, cu, pv, part, lds);
}

// FEW: calls of at most few_rows live rows, which only the device knows, take
// the few-rows form here (a launch of its own that returns at once when they
// are more cost 2 us).  An instance of its own, as the argument and the test
// alone cost the large calls 2% (20416 rows, V = 157184, D = 2048: 11.21 ->
// 11.45 ms).
template <bool FEW>
__global__ void __launch_bounds__(kLmThreads, 1)
lmhead_kernel(const uint16_t* __restrict__ H, const uint16_t* __restrict__ W, int D, int V,
              int row_cap, int padded, int n_vtiles, int cu, int few_rows, PackView pv,
              float4* __restrict__ part) {
    constexpr int kFewLds = kFewStages * (kHalfBytes + kFewRows * kRowBytes);
    __shared__ __attribute__((aligned(16))) unsigned char
        lds[FEW && kFewLds > kStages * kStageBytes ? kFewLds : kStages * kStageBytes];
    __shared__ Top s_top[kTileT];
    __shared__ int s_live;

    const int tid = threadIdx.x;
    // token tiles that can hold live rows (ragged rows are the first
    // header-count rows; padded rows sit anywhere below row_cap), and the
    // partitions for them; block b is token tile b mod n_lt of partition
    // b / n_lt, and workgroup i takes blocks i, i + gridDim.x, ...
    const int n_rows = padded ? row_cap : pv.hdr[kHdrRows];
    if (FEW && n_rows <= few_rows) {
        if (n_rows > 64) lm_few_rows<4>(H, W, D, V, row_cap, cu, pv, part, lds);
        else if (n_rows > 0) lm_few_rows<2>(H, W, D, V, row_cap, cu, pv, part, lds);
        return;
    }
    const int n_lt = (n_rows + kTileT - 1) / kTileT;
    const int P = n_lt > 0 ? lm_parts_dev(n_lt, n_vtiles, cu) : 0;
    for (int blk = blockIdx.x; blk < n_lt * P; blk += gridDim.x) {
    const int rt = blk % n_lt;
    const int pidx = blk / n_lt;
    const int row0 = rt * kTileT;
    // partitions of floor or ceil(n_vtiles / P) tiles
    const int vt0 = (int)((long long)pidx * n_vtiles / P);
    const int vt1 = (int)((long long)(pidx + 1) * n_vtiles / P);
    if (vt0 >= vt1) continue;
    // skip token tiles without a live row (the first barrier also keeps the
    // previous block's last reads of s_live and s_top before these writes)
    __syncthreads();
    if (tid == 0) s_live = 0;
    __syncthreads();
    if (tid < kTileT && row0 + tid < row_cap && pv.row_req[row0 + tid] >= 0) s_live = 1;
    __syncthreads();
    if (!s_live) continue;

    const int wave = tid >> 6;
    const int lane = tid & 63;
    const int n = lane & 31;
    const int h = lane >> 5;
    const int wv = wave & 1;          // vocabulary half of the tile
    const int wt = wave >> 1;         // token quarter of the tile

    // ---- DMA assignment: wave w fills W rows [32w, 32w+32) and H rows
    // [32w, 32w+32) of each stage, 8 rows (1 KB) per instruction; lane L
    // writes LDS chunk L%8 of row r = 32w + 8j + L/8, which holds logical K
    // chunk (L%8) ^ ((r/2)%8).  With 128-byte rows, 16 consecutive rows then
    // cover all 16 bank groups of 16 bytes at any logical chunk, so the
    // operand reads (16 lanes = 16 rows per access) are conflict-free.
    const int lrow = lane >> 3;
    uint32_t h_off[4];
    int w_row[4], w_chunk[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int r = wave * 32 + j * 8 + lrow;
        const int c = (lane & 7) ^ ((r >> 1) & 7);
        const int tr = min(row0 + r, row_cap - 1);
        h_off[j] = (uint32_t)(((size_t)tr * D + c * 8) * 2);
        w_row[j] = r;
        w_chunk[j] = c;
    }
    uint32_t m0_w[4], m0_h[4];
    const uint32_t lds_base = (uint32_t)(uintptr_t)&lds[0];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        m0_w[j] = __builtin_amdgcn_readfirstlane(lds_base + (wave * 4 + j) * 1024);
        m0_h[j] = __builtin_amdgcn_readfirstlane(lds_base + kHalfBytes + (wave * 4 + j) * 1024);
    }
    uint32_t w_off[4];
    auto set_vtile = [&](int vt) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int vr = min(vt * kTileV + w_row[j], V - 1);
            w_off[j] = (uint32_t)(((size_t)vr * D + w_chunk[j] * 8) * 2);
        }
    };
    const int KS = D / kBK;
    // issue K step ks of the current DMA tile into `stage`
    auto issue = [&](int ks, int stage) {
        const int k0 = ks * kBK;
        const uint16_t* wb = W + k0;
        const uint16_t* hb = H + k0;
        const uint32_t so = stage * kStageBytes;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2"
                         :: "s"(m0_w[j] + so), "v"(w_off[j]), "s"(wb) : "memory");
#pragma unroll
        for (int j = 0; j < 4; ++j)
            asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2"
                         :: "s"(m0_h[j] + so), "v"(h_off[j]), "s"(hb) : "memory");
    };

    // operand reads: row r of a stage part, logical chunk 2kk + h, stored at
    // chunk (2kk + h) ^ ((r/2)%8); every row read here has (r/2)%8 == (n/2)%8
    const uint32_t swz = (uint32_t)((h ^ ((n >> 1) & 7)) * 16);
    const uint32_t a_row = (uint32_t)((wv * 128 + n) * kRowBytes);
    const uint32_t b_row = (uint32_t)(kHalfBytes + (wt * 64 + n) * kRowBytes);

    floatx16 acc[4][2];
#pragma unroll
    for (int vi = 0; vi < 4; ++vi)
#pragma unroll
        for (int ti = 0; ti < 2; ++ti) acc[vi][ti] = floatx16{};
    Top top[2] = {top_empty(), top_empty()};

    // Operand fragments of one k step (16 of K): four of W, two of H, in two
    // register sets so the reads of k step kk + 1 overlap the eight MFMAs of
    // k step kk.
    constexpr int KK = kBK / 16;
    bf16x8 a[2][4], b[2][2];
    auto read = [&](int stage, int kk, int buf) {
        const unsigned char* st = lds + stage * kStageBytes;
        const uint32_t ko = swz ^ (uint32_t)(kk << 5);
#pragma unroll
        for (int vi = 0; vi < 4; ++vi)
            a[buf][vi] = *reinterpret_cast<const bf16x8*>(st + a_row + vi * 32 * kRowBytes + ko);
#pragma unroll
        for (int ti = 0; ti < 2; ++ti)
            b[buf][ti] = *reinterpret_cast<const bf16x8*>(st + b_row + ti * 32 * kRowBytes + ko);
    };
    // MFMAs x0 .. x1-1 of a k step (x = 2 vi + ti)
    auto mfmas = [&](int buf, int x0 = 0, int x1 = 8) {
#pragma unroll
        for (int x = x0; x < x1; ++x)
            acc[x >> 1][x & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                a[buf][x >> 1], b[buf][x & 1], acc[x >> 1][x & 1], 0, 0, 0);
    };

    // fold the finished tile vt into the running tops; lane value (vi, r)
    // is vocabulary id vt*256 + wv*128 + vi*32 + (r/4)*8 + h*4 + r%4 --
    // increasing in (vi, r), so the first maximum in that order is the
    // lowest id.
    auto fold = [&](int vt, auto partial) {
        const int vbase = vt * kTileV + wv * 128 + h * 4;
#pragma unroll
        for (int ti = 0; ti < 2; ++ti) {
            float f[64];
#pragma unroll
            for (int vi = 0; vi < 4; ++vi)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int v = vbase + vi * 32 + (r >> 2) * 8 + (r & 3);
                    f[vi * 16 + r] = (!partial || v < V) ? acc[vi][ti][r] : -INFINITY;
                }
            // maxima of the four 16-id groups (one MFMA tile each), then the
            // tile maximum
            float g[4];
#pragma unroll
            for (int vi = 0; vi < 4; ++vi) {
                g[vi] = f[vi * 16];
#pragma unroll
                for (int r = 1; r < 16; ++r) g[vi] = fmaxf(g[vi], f[vi * 16 + r]);
            }
            const float vmax = fmaxf(fmaxf(g[0], g[1]), fmaxf(g[2], g[3]));
            Top& t = top[ti];
            if (vmax > t.m) {
#pragma clang fp contract(off)
                // lowest position of the maximum: the first group that holds
                // it (every earlier group is below it), then the first
                // position inside that group
                int gs = 3;
#pragma unroll
                for (int vi = 2; vi >= 0; --vi)
                    if (g[vi] == vmax) gs = vi;
                // the group's values by bit masks (v_bfi: (m & a) | (~m & b)),
                // so the selection stays free of branches
                const uint32_t m1 = gs >= 1 ? ~0u : 0u, m2 = gs >= 2 ? ~0u : 0u,
                               m3 = gs >= 3 ? ~0u : 0u;
                auto bfi = [](uint32_t m, float a, float b) -> float {
                    uint32_t r;
                    asm("v_bfi_b32 %0, %1, %2, %3"
                        : "=v"(r) : "v"(m), "v"(__float_as_uint(a)), "v"(__float_as_uint(b)));
                    return __uint_as_float(r);
                };
                int r0 = 15;
#pragma unroll
                for (int r = 15; r >= 0; --r) {
                    const float x = bfi(m3, f[48 + r], bfi(m2, f[32 + r], bfi(m1, f[16 + r], f[r])));
                    if (x == vmax) r0 = r;
                }
                const int j0 = gs * 16 + r0;
                const float nmL = scaled_ref(vmax);
                t.s *= __builtin_amdgcn_exp2f(t.mL - nmL);
                t.m = vmax;
                t.mL = nmL;
                t.idx = vbase + (j0 >> 4) * 32 + ((j0 & 15) >> 2) * 8 + (j0 & 3);
            }
            if (t.m != -INFINITY) {
                float e[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int j = 0; j < 64; ++j)
                    e[j & 3] += __builtin_amdgcn_exp2f(fmaf(f[j], kLog2e, -t.mL));
                t.s += (e[0] + e[1]) + (e[2] + e[3]);
            }
        }
#pragma unroll
        for (int vi = 0; vi < 4; ++vi)
#pragma unroll
            for (int ti = 0; ti < 2; ++ti) acc[vi][ti] = floatx16{};
    };

    // ---- main loop over the partition's stages k (vocabulary tile
    // vt0 + k / KS, K step k % KS) in two LDS slots; stage k + 1 is loaded
    // while stage k is computed.  The last k step's fragments of a stage are
    // read before the barrier that hands its slot back to the loader, and
    // their MFMAs issue right after it, so the next stage's first reads
    // overlap eight MFMAs instead of stalling the matrix core.
    const int T = (vt1 - vt0) * KS;
    int ld_vt = vt0, ld_ks = 0;      // next stage to load
    set_vtile(vt0);
    auto issue_next = [&](int k) {
        issue(ld_ks, k & 1);
        if (++ld_ks == KS) {
            ld_ks = 0;
            if (++ld_vt < vt1) set_vtile(ld_vt);
        }
    };
    issue_next(0);
    wait_vm0();
    lds_barrier();
    if (T > 1) issue_next(1);
    read(0, 0, 0);
    // k steps 0 .. KK-2 of stage k: reads of step kk + 1 under the MFMAs of kk
    auto body = [&](int slot) {
#pragma unroll
        for (int kk = 0; kk + 1 < KK; ++kk) {
            read(slot, kk + 1, (kk + 1) & 1);
            __builtin_amdgcn_sched_barrier(0);
            mfmas(kk & 1);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    int k = 0;
    for (int vt = vt0; vt < vt1; ++vt) {
        for (int ks = 0; ks + 1 < KS; ++ks, ++k) {
            const int slot = k & 1;
            body(slot);
            wait_vm0();
            lds_barrier();         // stage k + 1 landed; slot k & 1 is free
            read(slot ^ 1, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            mfmas((KK - 1) & 1, 0, 2);
            __builtin_amdgcn_sched_barrier(0);
            if (k + 2 < T) issue_next(k + 2);   // under the MFMAs in flight
            __builtin_amdgcn_sched_barrier(0);
            mfmas((KK - 1) & 1, 2, 8);
            __builtin_amdgcn_sched_barrier(0);
        }
        // the tile's last stage: its last MFMAs, then the fold (no fragments
        // live across it), then the hand-over to the next stage
        const int slot = k & 1;
        body(slot);
        mfmas((KK - 1) & 1);
        if ((vt + 1) * kTileV > V)
            fold(vt, std::true_type{});
        else
            fold(vt, std::false_type{});
        if (k + 1 < T) {
            wait_vm0();
            lds_barrier();
            if (k + 2 < T) issue_next(k + 2);
            read(slot ^ 1, 0, 0);
        }
        ++k;
    }

    // ---- merge: lane halves, then the two vocabulary halves of each token
#pragma unroll
    for (int ti = 0; ti < 2; ++ti) {
        Top o;
        o.m = __shfl_xor(top[ti].m, 32, 64);
        o.mL = __shfl_xor(top[ti].mL, 32, 64);
        o.s = __shfl_xor(top[ti].s, 32, 64);
        o.idx = __shfl_xor(top[ti].idx, 32, 64);
        top[ti] = top_merge(top[ti], o);
    }
    __syncthreads();
    if (wv == 1 && h == 0) {
#pragma unroll
        for (int ti = 0; ti < 2; ++ti) s_top[wt * 64 + ti * 32 + n] = top[ti];
    }
    __syncthreads();
    if (wv == 0 && h == 0) {
#pragma unroll
        for (int ti = 0; ti < 2; ++ti) {
            const int tok = wt * 64 + ti * 32 + n;
            const int row = row0 + tok;
            const Top t = top_merge(top[ti], s_top[tok]);
            if (row < row_cap && pv.row_req[row] >= 0)
                part[(size_t)blk * kTileT + tok] = top_pack(t);
        }
    }
    }
}

// One wave per row: partials k = lane, lane + 64, ... (partition k of the
// row's token tile, written by block k * n_lt + tile) merged per lane in
// increasing k, then across lanes by a fixed butterfly.
__global__ void __launch_bounds__(kMergeThreads)
lm_merge_kernel(const float4* __restrict__ lm_part, int V, int n_vtiles, int cu, int few_rows,
                PackView pv, int row_cap, int padded, float4* __restrict__ upd_part, int nsplit) {
    const int row = blockIdx.x * (kMergeThreads / 64) + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (row >= row_cap || pv.row_req[row] < 0) return;
    const int n_rows = padded ? row_cap : pv.hdr[kHdrRows];
    const int n_lt = (n_rows + kTileT - 1) / kTileT;
    const int P = n_rows <= few_rows ? lm_few_parts(V, cu) : lm_parts_dev(n_lt, n_vtiles, cu);
    const size_t base = (size_t)(row / kTileT) * kTileT + row % kTileT;
    const size_t stride = (size_t)n_lt * kTileT;
    Top t = top_empty();
    for (int k = lane; k < P; k += 64) t = top_merge(t, top_unpack(lm_part[base + k * stride]));
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        Top o;
        o.m = __shfl_xor(t.m, off, 64);
        o.mL = __shfl_xor(t.mL, off, 64);
        o.s = __shfl_xor(t.s, off, 64);
        o.idx = __shfl_xor(t.idx, off, 64);
        t = top_merge(t, o);
    }
    for (int k = lane; k < nsplit; k += 64)
        upd_part[(size_t)row * nsplit + k] = top_pack(k == 0 ? t : top_empty());
}

}  // namespace

LmSizes lm_sizes(const fb_pack* pack, int V, int D, int cu_count) {
    LmSizes z{};
    z.n_rtiles = (pack->row_cap + kTileT - 1) / kTileT;
    z.n_vtiles = (V + kTileV - 1) / kTileV;
    z.cu = cu_count > 0 ? cu_count : 256;
    // the grid: the largest n_lt * P over every count of token tiles the
    // rows can fill (memoized: the search is over n_rtiles x kMaxParts)
    static std::mutex mu;
    static std::map<std::tuple<int, int, int>, int> memo;
    const auto key = std::make_tuple(z.n_rtiles, z.n_vtiles, z.cu);
    int grid = 0;
    {
        std::lock_guard<std::mutex> lock(mu);
        auto it = memo.find(key);
        if (it != memo.end()) {
            grid = it->second;
        } else {
            for (int n = 1; n <= z.n_rtiles; ++n) {
                const int g = n * lm_parts_host(n, z.n_vtiles, z.cu);
                grid = g > grid ? g : grid;
            }
            memo.emplace(key, grid);
        }
    }
    // The few-rows form has a block per vocabulary range.  The live rows are
    // known on the device only; where the capacity allows more, the kernel
    // chooses by them, if the weight is large (from 256 MB the few-rows form is
    // 1.4-1.7x as fast where it applies) and the capacity at most 1024 rows,
    // above which so few live ones are unlikely.  A padded pack's rows may lie
    // anywhere in its capacity, so that alone decides.
    const bool few = pack->row_cap <= kFewRows ||
                     (pack->layout != FB_PADDED && pack->row_cap <= 8 * kFewRows &&
                      (long long)V * D >= (1LL << 27));
    z.few_rows = few ? kFewRows : 0;
    z.few_grid = few ? lm_few_parts(V, z.cu) : 0;
    const int blocks = grid > z.few_grid ? grid : z.few_grid;
    // partials: one per block; workgroups: at most eight per CU, each taking
    // blocks in turn (blocks past n_lt * P end at once, but each still holds
    // its CU for a moment)
    z.total = (size_t)blocks * kTileT * sizeof(float4);
    z.grid = grid < 8 * z.cu ? grid : 8 * z.cu;
    return z;
}

hipError_t launch_lmhead(const void* hidden, const void* weight, int D, int V,
                         const fb_pack* pack, void* lm_ws, const LmSizes& z, void* upd_ws,
                         const UpdateSizes& uz, hipStream_t stream) {
    PackView pv = pack_view(pack);
    float4* lm_part = static_cast<float4*>(lm_ws);
    const uint16_t* hp = static_cast<const uint16_t*>(hidden);
    const uint16_t* wp = static_cast<const uint16_t*>(weight);
    const int padded = pack->layout == FB_PADDED ? 1 : 0;
    auto tiles = [&](auto kernel, int wgs) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)wgs), dim3(kLmThreads), 0, stream, hp, wp, D, V,
                           pack->row_cap, padded, z.n_vtiles, z.cu, z.few_rows, pv, lm_part);
    };
    if (pack->row_cap <= kFewRows)
        hipLaunchKernelGGL(lm_few_kernel, dim3((unsigned)z.few_grid), dim3(kLmThreads), 0, stream,
                           hp, wp, D, V, pack->row_cap, padded, z.cu, pv, lm_part);
    else if (z.few_grid > 0)
        tiles(lmhead_kernel<true>, z.grid > z.few_grid ? z.grid : z.few_grid);
    else
        tiles(lmhead_kernel<false>, z.grid);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int rows_per_wg = kMergeThreads / 64;
    hipLaunchKernelGGL(lm_merge_kernel,
                       dim3((unsigned)((pack->row_cap + rows_per_wg - 1) / rows_per_wg)),
                       dim3(kMergeThreads), 0, stream, lm_part, V, z.n_vtiles, z.cu, z.few_rows, pv,
                       pack->row_cap, padded, static_cast<float4*>(upd_ws), uz.nsplit);
    return hipGetLastError();
}

}  // namespace fb
