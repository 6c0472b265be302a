// Window prologue: rotary position embedding at absolute positions on the
// live rows' queries and keys (the "absolute RoPE position ids" of Sec. 4.2),
// fused with the Eq. 6 window KV write, so the fresh keys are rotated and
// land in the paged cache in one pass.
//
// rope_kv_kernel  one workgroup per (live block of bl rows, KV head c): the
//                 g = Hq/Hkv query heads of c, key head c and value head c;
//                 the block's cos/sin table (positions x d/2 pairs, angles
//                 formed and reduced to [-pi, pi] in float64, sin/cos in
//                 float) in LDS; queries
//                 rotated in place or into q_out; keys rotated and written to
//                 their absolute slots of the K cache; values staged in LDS
//                 and written key-innermost to the V cache.  Pair j of a head
//                 vector is (x_j, x_{j+d/2}) (rotate-half arrangement), angle
//                 p * base^(-2j/d).
#include "internal.h"

namespace fb {
namespace {

constexpr int kRopeThreads = 256;
constexpr size_t kCacheBytes = 256u << 20;   // the memory-side cache
constexpr double k2Pi = 6.283185307179586;
constexpr double kInv2Pi = 0.15915494309189535;

struct ThetaTable {
    double t[64];   // base^(-2j/d), j < d/2 <= 64
};

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

template <bool NT>
__device__ inline u32x4 load16(const void* p) {
    if constexpr (NT) return __builtin_nontemporal_load(static_cast<const u32x4*>(p));
    else return *static_cast<const u32x4*>(p);
}

// Eight consecutive elements as loaded (one 16-byte word in bf16, two in fp32).
template <typename T, bool NT>
struct Raw8 {
    static constexpr int N = sizeof(T) * 8 / 16;
    u32x4 w[N];
    __device__ inline void load(const T* p) {
#pragma unroll
        for (int i = 0; i < N; ++i) w[i] = load16<NT>(p + i * (16 / sizeof(T)));
    }
    // the words are wanted here: a use that the compiler cannot move
    __device__ inline void settle() {
#pragma unroll
        for (int i = 0; i < N; ++i) asm volatile("" : "+v"(w[i]));
    }
    __device__ inline void get(float (&f)[8]) const {
        if constexpr (sizeof(T) == 2) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                f[2 * j] = __uint_as_float(w[0][j] << 16);
                f[2 * j + 1] = __uint_as_float(w[0][j] & 0xffff0000u);
            }
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) f[j] = __uint_as_float(w[j >> 2][j & 3]);
        }
    }
};

__device__ inline void store8(uint16_t* p, const float (&f)[8]) {
    u32x4 w;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const __bf16 a = (__bf16)f[2 * j], b = (__bf16)f[2 * j + 1];
        w[j] = (uint32_t)__builtin_bit_cast(uint16_t, a) |
               ((uint32_t)__builtin_bit_cast(uint16_t, b) << 16);
    }
    *reinterpret_cast<u32x4*>(p) = w;
}
__device__ inline void store8(float* p, const float (&f)[8]) {
    *reinterpret_cast<float4*>(p) = make_float4(f[0], f[1], f[2], f[3]);
    *reinterpret_cast<float4*>(p + 4) = make_float4(f[4], f[5], f[6], f[7]);
}

// Rotate the 8 pairs (lo[k], hi[k]) of group g of row i with the table.
__device__ inline void rotate8(float (&lo)[8], float (&hi)[8], const float2* cs) {
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const float c = cs[k].x, s = cs[k].y;
        const float a = lo[k], b = hi[k];
        lo[k] = fmaf(a, c, -b * s);
        hi[k] = fmaf(b, c, a * s);
    }
}

// Bound by HBM (every byte of q, k and v is read and written once).  What it
// needs: the first round's loads in flight while the table is worked out; the
// KV heads of one block side by side in the grid, so that the workgroups at
// work together walk whole rows instead of one head's 1 KB in every 8; and, NT,
// the nontemporal hint where the inputs are larger than the 256 MB memory-side
// cache.  256 requests, 20416 live rows of 32 + 2 x 8 heads of 128 in bf16 (502
// MB): 111 us before, 100 now on inputs that change from call to call, 80 =
// 6.2 TB/s on the same ones again.  The hint is for inputs that come from
// memory: the first call on new ones takes 125 us with it and 148 without.
// Calls back to back on changing inputs lose 2.5% by it (97 us without), and
// smaller inputs, served from the cache, up to a fifth (16384 rows of 16 + 2 x 2
// heads: 26.6 us, with the hint 31.5).
template <typename T, bool NT>
__global__ void __launch_bounds__(kRopeThreads)
rope_kv_kernel(const T* __restrict__ q_in, T* __restrict__ q_out, const T* __restrict__ k_new,
               const T* __restrict__ v_new, T* __restrict__ k_cache, T* __restrict__ v_cache,
               const int32_t* __restrict__ page_table, PackView pv, int Hq, int Hkv, int D,
               int bl, int ps, int max_pages, int num_pages, int pitch, ThetaTable theta) {
    extern __shared__ __attribute__((aligned(16))) unsigned char rope_smem[];
    float2* tab = reinterpret_cast<float2*>(rope_smem);   // [bl][D/2] (cos, sin)
    T* vs = reinterpret_cast<T*>(rope_smem);              // later: [bl][pitch]
    const bool heads_first = gridDim.x == (unsigned)Hkv;   // else tiles first (see the launch)
    const int t = heads_first ? blockIdx.y : blockIdx.x;
    const int c = heads_first ? blockIdx.x : blockIdx.y;
    // d / 2 divides the workgroup, so a thread works on one pair of every row;
    // its angle step comes first, ahead of the loads that the table covers
    const double step = theta.t[threadIdx.x % (D / 2)];
    if (t >= pv.hdr[kHdrTiles]) return;
    const int g = Hq / Hkv;
    const int32_t* tile = pv.tiles + (size_t)t * kTileInts;
    const int b = tile[kTB];
    const int row0 = tile[kTRow0];
    const int pos0 = tile[kTPos0];
    const int32_t* pt = page_table + (size_t)b * max_pages;
    const int half = D / 2;
    const int ng = half / 8;                              // 8-pair groups per head (2^k)
    const int ng_sh = __builtin_ctz(ng);
    constexpr int VEC = 16 / sizeof(T);
    const int dch = D / VEC;

    // Q pair groups of the heads that read KV head c, kQ per thread and round;
    // K pair groups one per thread and round; V words kV.
    constexpr int kQ = sizeof(T) == 2 ? 4 : 2;
    constexpr int kV = 2;
    const int n_q = bl * g * ng, n_k = bl * ng, n_v = bl * dch;
    Raw8<T, NT> ql[kQ], qh[kQ], kl, kh;
    size_t q_at[kQ];   // element offset of the group's first half
    int q_cs[kQ];      // its place in the table
    u32x4 vw[kV];
    int k_page;
    // past the last group a thread reloads it (an address inside the block)
    // and stores nothing
    auto load_q = [&](int e0) {
#pragma unroll
        for (int j = 0; j < kQ; ++j) {
            if (e0 + j * kRopeThreads >= n_q) break;
            const unsigned e = min(e0 + j * kRopeThreads + (int)threadIdx.x, n_q - 1);
            const unsigned rh = e >> ng_sh, gi = e & (ng - 1);   // (row, head of the group)
            const unsigned i = rh / (unsigned)g, hh = rh - i * g;
            q_at[j] = ((size_t)(row0 + i) * Hq + c * g + hh) * D + gi * 8;
            q_cs[j] = i * half + gi * 8;
            ql[j].load(q_in + q_at[j]);
            qh[j].load(q_in + q_at[j] + half);
        }
    };
    auto load_k = [&](int e0) {
        const int e = min(e0 + (int)threadIdx.x, n_k - 1);
        const int i = e >> ng_sh;
        const T* src = k_new + ((size_t)(row0 + i) * Hkv + c) * D + (e & (ng - 1)) * 8;
        kl.load(src);
        kh.load(src + half);
        const int pidx = (pos0 + i) / ps;
        const int p = pt[min(pidx, max_pages - 1)];
        k_page = pidx < max_pages ? p : -1;
    };
    auto load_v = [&](int e0) {
#pragma unroll
        for (int j = 0; j < kV; ++j) {
            if (e0 + j * kRopeThreads >= n_v) break;
            const int e = min(e0 + j * kRopeThreads + (int)threadIdx.x, n_v - 1);
            vw[j] = load16<NT>(
                v_new + ((size_t)(row0 + e / dch) * Hkv + c) * D + (size_t)(e % dch) * VEC);
        }
    };
    // The first round's loads go out before the table is worked out.
    load_q(0);
    load_k(0);
    load_v(0);

    for (int i = threadIdx.x / half; i < bl; i += kRopeThreads / half) {
        // angle in float64, reduced to [-pi, pi] in float64, then float sin/cos
        const double a = (double)(pos0 + i) * step;
        const double r = a - rint(a * kInv2Pi) * k2Pi;
        float s, c;
        sincosf((float)r, &s, &c);
        tab[i * half + threadIdx.x % half] = make_float2(c, s);
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kQ; ++j) ql[j].settle(), qh[j].settle();
    kl.settle();
    kh.settle();
    asm volatile("" : "+v"(k_page));
#pragma unroll
    for (int j = 0; j < kV; ++j) asm volatile("" : "+v"(vw[j]));

    for (int e0 = 0; e0 < n_q; e0 += kQ * kRopeThreads) {
        if (e0 > 0) load_q(e0);
#pragma unroll
        for (int j = 0; j < kQ; ++j) {
            const int e = e0 + j * kRopeThreads + threadIdx.x;
            if (e >= n_q) continue;
            float lo[8], hi[8];
            ql[j].get(lo);
            qh[j].get(hi);
            rotate8(lo, hi, tab + q_cs[j]);
            T* dst = q_out + q_at[j];
            store8(dst, lo);
            store8(dst + half, hi);
        }
    }
    // keys: rotated straight into their absolute slots
    for (int e0 = 0; e0 < n_k; e0 += kRopeThreads) {
        if (e0 > 0) load_k(e0);
        const int e = e0 + threadIdx.x;
        if (e >= n_k) continue;
        const int gi = e & (ng - 1);
        const int i = e >> ng_sh;
        if (k_page < 0 || k_page >= num_pages) {
            if (gi == 0) record_error(pv.hdr, b, FB_DERR_PAGE);
            continue;
        }
        float lo[8], hi[8];
        kl.get(lo);
        kh.get(hi);
        rotate8(lo, hi, tab + i * half + gi * 8);
        T* dst = k_cache + (((size_t)k_page * Hkv + c) * ps + ((pos0 + i) % ps)) * D + gi * 8;
        store8(dst, lo);
        store8(dst + half, hi);
    }
    __syncthreads();   // the table's LDS is reused for the values below

    // values of head c: key-innermost rows of the V cache
    {
        for (int e0 = 0; e0 < n_v; e0 += kV * kRopeThreads) {
            if (e0 > 0) load_v(e0);
#pragma unroll
            for (int j = 0; j < kV; ++j) {
                const int e = e0 + j * kRopeThreads + threadIdx.x;
                if (e < n_v)
                    *reinterpret_cast<u32x4*>(vs + (size_t)(e / dch) * pitch + (e % dch) * VEC) =
                        vw[j];
            }
        }
        __syncthreads();
        if (pos0 % VEC == 0 && ps % VEC == 0 && bl % VEC == 0) {
            const int nrun = bl / VEC;
            for (int e = threadIdx.x; e < D * nrun; e += kRopeThreads) {
                const int ic = e % nrun;
                const int d = e / nrun;
                const int pos = pos0 + ic * VEC;
                const int pidx = pos / ps;
                const int page = pidx < max_pages ? pt[pidx] : -1;
                if (page < 0 || page >= num_pages) continue;   // recorded with the keys
                union {
                    uint4 v;
                    T x[VEC];
                } run;
#pragma unroll
                for (int k = 0; k < VEC; ++k) run.x[k] = vs[(size_t)(ic * VEC + k) * pitch + d];
                *reinterpret_cast<uint4*>(v_cache + (((size_t)page * Hkv + c) * D + d) * ps +
                                          (pos % ps)) = run.v;
            }
        } else {
            for (int e = threadIdx.x; e < bl * D; e += kRopeThreads) {
                const int d = e / bl;
                const int i = e % bl;
                const int pos = pos0 + i;
                const int pidx = pos / ps;
                const int page = pidx < max_pages ? pt[pidx] : -1;
                if (page < 0 || page >= num_pages) continue;
                v_cache[(((size_t)page * Hkv + c) * D + d) * ps + (pos % ps)] =
                    vs[(size_t)i * pitch + d];
            }
        }
        __syncthreads();
    }
}

}  // namespace

size_t prologue_smem_bytes(const fb_pack* pack, const fb_attn_shape* sh, int* pitch_out) {
    const size_t elt = sh->dtype == FB_BF16 ? 2 : 4;
    int pitch = sh->head_dim + (int)(16 / elt);
    if ((size_t)pack->bl * pitch * elt > 65536) pitch = sh->head_dim;
    if (pitch_out) *pitch_out = pitch;
    const size_t table = (size_t)pack->bl * (sh->head_dim / 2) * sizeof(float2);
    const size_t vstage = (size_t)pack->bl * pitch * elt;
    return table > vstage ? table : vstage;
}

hipError_t launch_window_prologue(const void* q_in, void* q_out, const void* k_new,
                                  const void* v_new, void* k_cache, void* v_cache,
                                  const int32_t* page_table, const fb_pack* pack,
                                  const fb_attn_shape* sh, double rope_base,
                                  hipStream_t stream) {
    PackView pv = pack_view(pack);
    ThetaTable th{};
    const int D = sh->head_dim;
    for (int j = 0; j < D / 2; ++j) th.t[j] = pow(rope_base, -2.0 * j / D);
    int pitch = 0;
    const size_t smem = prologue_smem_bytes(pack, sh, &pitch);
    // a grid's second extent ends at 65535: packs of more tiles go tiles first
    const dim3 grid = pack->tile_cap <= 65535 ? dim3(sh->Hkv, pack->tile_cap)
                                              : dim3(pack->tile_cap, sh->Hkv);
    // NT goes by the capacity, as the live rows are known on the device only.  A
    // capacity of 32768 rows (403 MB of inputs) with few of them live, us with the
    // hint and without: 512 rows 7.7 / 7.6, 2048 13.2 / 12.7, 8192 38 / 44, 16384
    // 81 / 79; on new inputs 33 / 30, 38 / 36, 59 / 84, 93 / 118; right behind the
    // kernels that write them it costs 0-2.5.
    const size_t elt = sh->dtype == FB_BF16 ? 2 : 4;
    const bool nt = (size_t)pack->row_cap * (sh->Hq + 2 * sh->Hkv) * D * elt > kCacheBytes;
    auto go = [&](auto kernel, auto zero) {
        using T = decltype(zero);
        hipLaunchKernelGGL(kernel, grid, dim3(kRopeThreads), smem, stream,
                           static_cast<const T*>(q_in), static_cast<T*>(q_out),
                           static_cast<const T*>(k_new), static_cast<const T*>(v_new),
                           static_cast<T*>(k_cache), static_cast<T*>(v_cache), page_table, pv,
                           sh->Hq, sh->Hkv, D, pack->bl, sh->page_size, sh->max_pages,
                           sh->num_pages, pitch, th);
    };
    if (sh->dtype == FB_BF16) {
        if (nt) go(rope_kv_kernel<uint16_t, true>, uint16_t());
        else go(rope_kv_kernel<uint16_t, false>, uint16_t());
    } else {
        if (nt) go(rope_kv_kernel<float, true>, float());
        else go(rope_kv_kernel<float, false>, float());
    }
    return hipGetLastError();
}

}  // namespace fb
