// Skinny-M projection kernels and the one-time weight re-tiling.
//
// Work decomposition: workgroup (grp, mb) owns NT consecutive 16-feature tiles ("group" grp) for the
// MT*16 rows of row block mb.  Its NW waves split the K range round-robin; wave w streams the weight
// fragments of k-tiles w, w + NW, ... — NT contiguous KiB per k-tile in the re-tiled layout — and
// multiplies them with the activation fragments of the same k-tiles (read through L2).
// Partial 16x16 tiles are summed across waves through LDS, then the epilogue runs on the reduced tile.
//
// Operand roles: A = weights (rows = output features), B = activations (rows = segment rows), so the
// result tile is Y^T: lane l holds features n = (l/16)*4 + v, v = 0..3, of row m = l % 16 — four
// consecutive features of one row per lane: vector stores, and per-row scalars (RMSNorm scale) are
// per-lane.
//
// RMSNorm is split algebraically: norm(x) . w = rs(x) * sum_k x_k g_k w_k.  The gain g is folded into the
// re-tiled weights once; rs(x) = rsqrt(mean(x^2) + eps) is computed from the activation fragments the
// workgroup reads anyway (it covers the whole K range) and applied in the epilogue.
#include "gemm.hpp"

#include <algorithm>


typedef __attribute__((ext_vector_type(2))) bf16_t bf16x2;
struct bf16x2x4 {
    bf16x2 v[4];
};

template <typename T>
static __device__ __forceinline__ typename Elem<T>::frag_t load_w(const void* p) {
    using frag_t = typename Elem<T>::frag_t;
    return __builtin_nontemporal_load((const frag_t*)p);
}

// Residual-stream values [m][n .. n+3] (fp32 stream, or the T-typed stage input at the first layer).
template <typename T>
static __device__ __forceinline__ f32x4 load_resid(const GemmArgs& a, int m, int n) {
    using E = Elem<T>;
    if (a.resid_is_T) {
        const T* p = (const T*)a.resid + (size_t)m * a.N + n;
        return f32x4{E::to_f(p[0]), E::to_f(p[1]), E::to_f(p[2]), E::to_f(p[3])};
    }
    return *(const f32x4*)((const float*)a.resid + (size_t)m * a.N + n);
}

// The residual values of the item a wave will finish first (item w), fetched before the K loop so that the epilogue does
// not start with a dependent global load.  Only this workgroup ever writes those elements, so reading them early is safe
// even when the projection updates the residual stream in place.
template <typename T, int MT, int NT, int EPI>
static __device__ __forceinline__ f32x4 prefetch_resid(const GemmArgs& a, int w, int grp, int row0, int r16, int g) {
    f32x4 v{0.f, 0.f, 0.f, 0.f};
    if constexpr (EPI == EPI_RESID) {
        if (w < MT * NT) {
            const int m = row0 + (w / NT) * 16 + r16, n = (grp * NT + w % NT) * 16 + g * 4;
            if (m < a.M && n < a.N) v = load_resid<T>(a, m, n);
        }
    }
    return v;
}

// What the QKV epilogue reads for a row and a pair of tiles, fetched before the K loop: behind it, the rotary table and the cache row's
// address are two rounds of memory latency in front of the stores (4096-wide layer, 16 rows 21.0 -> 20.6 us).
struct QkvPre {
    float2 cs[4];             // rotary table of the lane's features
    unsigned long long krow;  // cache row (K and V heads)
};
static __device__ __forceinline__ QkvPre prefetch_qkv(const GemmArgs& a, int m, int ptile, int g) {
    QkvPre p;
    const int tph = a.hd >> 4, mc = min(m, a.M - 1);
    const float2* cs = a.rope + (size_t)mc * (a.hd >> 1) + ((ptile % tph) >> 1) * 16 + g * 4;
#pragma unroll
    for (int v = 0; v < 4; ++v) p.cs[v] = cs[v];
    p.krow = a.krow[mc];
    return p;
}

// Fused epilogue for one "item": one 16x16 result tile (RESID, LOGITS) or a pair of tiles (QKV, SWIGLU) in the
// MFMA result layout — this lane holds features g*4 + v of row m; rs is the row's RMSNorm scale.
// Returns this lane's share of the sum of squares of the new residual-stream values (RESID), else 0.
template <typename T, int EPI>
static __device__ __forceinline__ float epilogue_item(const GemmArgs& a, const float (&y)[(EPI == EPI_QKV || EPI == EPI_SWIGLU) ? 2 : 1][4],
                                                      float rs, int m, int ptile, int g, const f32x4* resid_pre = nullptr,
                                                      const QkvPre* qkv_pre = nullptr) {
    using E = Elem<T>;
    float hsq = 0.f;
    if constexpr (EPI != EPI_RESID) {
        if (m >= a.M) return 0.f;
    }
    if constexpr (EPI == EPI_RESID) {
        const int n = ptile * 16 + g * 4;
        if (m < a.M && n < a.N) {
            const f32x4 rv = resid_pre ? *resid_pre : load_resid<T>(a, m, n);
            const float r[4] = {rv[0], rv[1], rv[2], rv[3]};
            f32x4 h{r[0] + y[0][0], r[1] + y[0][1], r[2] + y[0][2], r[3] + y[0][3]};
            *(f32x4*)(a.h_out + (size_t)m * a.N + n) = h;
            hsq = h[0] * h[0] + h[1] * h[1] + h[2] * h[2] + h[3] * h[3];
            if (a.gain_next) {
#pragma unroll
                for (int v = 0; v < 4; ++v) h[v] *= E::to_f(((const T*)a.gain_next)[n + v]);
            }
            const size_t hi = a.hb_frag ? frag_major_index<T>(m, n, a.N / E::KT) : (size_t)m * a.N + n;
            *(typename E::out4_t*)((T*)a.hb_out + hi) = E::pack4(h[0], h[1], h[2], h[3]);
        }
    } else if constexpr (EPI == EPI_LOGITS) {
        const int n = ptile * 16 + g * 4;
        float* dst = a.logits + (size_t)m * a.N + n;
        // Four stores of a float each, every one into 64 pieces of memory, held up the ends of the launches (us, one by one -> together: 16 rows x
        // 32000 48.0 -> 46.3, 128 rows 61.8 -> 56.2, with K 1024 28.9 -> 22.9; 128 rows x 152064 275 -> 250; 4-bit, 128 rows x 32000 101 -> 89).
        if (a.logits_vec) {
            if (n < a.N) *(f32x4*)dst = f32x4{rs * y[0][0], rs * y[0][1], rs * y[0][2], rs * y[0][3]};
        } else {
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (n + v < a.N) dst[v] = rs * y[0][v];
        }
    } else if constexpr (EPI == EPI_SWIGLU) {
        const int f = (ptile >> 1) * 16 + g * 4;
        if (f < a.F) {
            float o[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                float gt = rs * y[0][v], up = rs * y[1][v];
                o[v] = gt / (1.0f + expf(-gt)) * up;
            }
            *(typename E::out4_t*)((T*)a.act_out + frag_major_index<T>(m, f, a.F / E::KT)) = E::pack4(o[0], o[1], o[2], o[3]);
        }
    } else {  // EPI_QKV
        const int tph = a.hd >> 4;  // tiles per head
        const int head = ptile / tph, tih = ptile % tph;
        if (head >= a.Hq + 2 * a.Hkv) return 0.f;  // padding tiles of the last group
        float lo[4], hi[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            lo[v] = rs * y[0][v];
            hi[v] = rs * y[1][v];
            if (a.bias) {
                lo[v] += a.bias[ptile * 16 + g * 4 + v];
                hi[v] += a.bias[(ptile + 1) * 16 + g * 4 + v];
            }
        }
        if (head < a.Hq + a.Hkv) {
            // q / k head: the pair holds features t and t + hd/2, t = (tih/2)*16 + g*4 + v
            const int t = (tih >> 1) * 16 + g * 4, half = a.hd >> 1;
            const float2* cs = a.rope + (size_t)m * half + t;
            float olo[4], ohi[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const float2 c = qkv_pre ? qkv_pre->cs[v] : cs[v];
                olo[v] = lo[v] * c.x - hi[v] * c.y;
                ohi[v] = hi[v] * c.x + lo[v] * c.y;
            }
            T* dst;
            if (head < a.Hq)
                dst = (T*)a.q_out + (size_t)m * (a.Hq * a.hd) + (size_t)head * a.hd;
            else
                dst = (T*)(qkv_pre ? qkv_pre->krow : a.krow[m]) + a.layer_off + (size_t)(head - a.Hq) * a.stride_head;
            *(typename E::out4_t*)(dst + t) = E::pack4(olo[0], olo[1], olo[2], olo[3]);
            *(typename E::out4_t*)(dst + t + half) = E::pack4(ohi[0], ohi[1], ohi[2], ohi[3]);
        } else if (head < a.Hq + 2 * a.Hkv) {
            // v head: natural tile order, no rotation
            T* dst = (T*)a.krow[m] + a.layer_off + a.stride_kv + (size_t)(head - a.Hq - a.Hkv) * a.stride_head;
            const int t = tih * 16 + g * 4;
            *(typename E::out4_t*)(dst + t) = E::pack4(lo[0], lo[1], lo[2], lo[3]);
            *(typename E::out4_t*)(dst + t + 16) = E::pack4(hi[0], hi[1], hi[2], hi[3]);
        }
    }
    return hsq;
}

// Two neighbouring items of a wave at once (bf16; ptile a multiple of 4, so that both belong to one head or one k-tile of the activations): lanes
// g and g ^ 1 trade four features of one item against four of the other, and every lane stores 16 bytes of one item, features
// (g >> 1) * 8 .. + 7, where epilogue_item stores 8 of each.  permlane16_swap trades the second 16 lanes of its first operand against the first 16
// of its second one, the fourth against the third: exactly that.
static __device__ __forceinline__ u32x4 trade_halves(const float (&p)[4], const float (&q)[4]) {
    typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
    const u32x2 u = __builtin_bit_cast(u32x2, Elem<bf16_t>::pack4(p[0], p[1], p[2], p[3]));
    const u32x2 v = __builtin_bit_cast(u32x2, Elem<bf16_t>::pack4(q[0], q[1], q[2], q[3]));
    const auto x = __builtin_amdgcn_permlane16_swap(u[0], v[0], false, false), y = __builtin_amdgcn_permlane16_swap(u[1], v[1], false, false);
    return u32x4{x[0], y[0], x[1], y[1]};
}
template <int EPI>
static __device__ __forceinline__ void epilogue_two(const GemmArgs& a, const float (&y0)[2][4], const float (&y1)[2][4], float rs, int m, int ptile, int g) {
    using T = bf16_t;
    static_assert(EPI == EPI_QKV || EPI == EPI_SWIGLU, "paired epilogues");
    const int odd = g & 1, k8 = (g >> 1) * 8;  // which item, and which half of its features, this lane stores
    if (m >= a.M) return;  // the four lanes of a row together
    if constexpr (EPI == EPI_SWIGLU) {
        float o0[4], o1[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const float g0 = rs * y0[0][v], g1 = rs * y1[0][v];
            o0[v] = g0 / (1.0f + expf(-g0)) * (rs * y0[1][v]);
            o1[v] = g1 / (1.0f + expf(-g1)) * (rs * y1[1][v]);
        }
        const u32x4 o = trade_halves(o0, o1);
        const int f = (ptile >> 1) * 16 + odd * 16 + k8;
        if (f < a.F) *(u32x4*)((T*)a.act_out + frag_major_index<T>(m, f, a.F / 32)) = o;
    } else {
        const int tph = a.hd >> 4, head = ptile / tph, tih = ptile % tph;
        if (head >= a.Hq + 2 * a.Hkv) return;  // padding tiles of the last group
        float lo0[4], hi0[4], lo1[4], hi1[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            lo0[v] = rs * y0[0][v], hi0[v] = rs * y0[1][v], lo1[v] = rs * y1[0][v], hi1[v] = rs * y1[1][v];
            if (a.bias) {
                const float* b = a.bias + ptile * 16 + g * 4 + v;
                lo0[v] += b[0], hi0[v] += b[16], lo1[v] += b[32], hi1[v] += b[48];
            }
        }
        if (head < a.Hq + a.Hkv) {  // features t and t + hd/2 per item, t = (tih / 2) * 16 + g * 4 + v, and 16 on
            const int t = (tih >> 1) * 16, half = a.hd >> 1;
            const float2* cs = a.rope + (size_t)m * half + t + g * 4;
            float p0[4], q0[4], p1[4], q1[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const float2 c = cs[v], d = cs[16 + v];
                p0[v] = lo0[v] * c.x - hi0[v] * c.y;
                q0[v] = hi0[v] * c.x + lo0[v] * c.y;
                p1[v] = lo1[v] * d.x - hi1[v] * d.y;
                q1[v] = hi1[v] * d.x + lo1[v] * d.y;
            }
            T* dst = head < a.Hq ? (T*)a.q_out + (size_t)m * (a.Hq * a.hd) + (size_t)head * a.hd
                                 : (T*)a.krow[m] + a.layer_off + (size_t)(head - a.Hq) * a.stride_head;
            dst += t + odd * 16 + k8;
            *(u32x4*)dst = trade_halves(p0, p1);
            *(u32x4*)(dst + half) = trade_halves(q0, q1);
        } else {  // natural tile order, no rotation
            T* dst = (T*)a.krow[m] + a.layer_off + a.stride_kv + (size_t)(head - a.Hq - a.Hkv) * a.stride_head + tih * 16 + odd * 16 + k8;
            *(u32x4*)dst = trade_halves(lo0, hi0);
            *(u32x4*)(dst + 32) = trade_halves(lo1, hi1);
        }
    }
}

// The items of a wave's NT tiles of one row tile, two at a time where they begin on a multiple of four tiles; returns as epilogue_item.  Us of
// launches of 1024 rows, one at a time -> so: QKV 28.0 -> 24.7 (1024 wide), 67.5 -> 64.0 (3584), 101.1 -> 99.6 (4096), 146.8 -> 145.2 (5120);
// gate/up 172.9 -> 172.1 (4096).
template <int EPI, int NT>
static __device__ __forceinline__ float epilogue_row(const GemmArgs& a, const f32x4 (&acc)[NT], float rs, int m, int ptile, int g) {
    constexpr int TPI = (EPI == EPI_QKV || EPI == EPI_SWIGLU) ? 2 : 1;
    float hsq = 0.f;
    auto one = [&](int i) __attribute__((always_inline)) {
        float y[TPI][4];
#pragma unroll
        for (int tt = 0; tt < TPI; ++tt)
#pragma unroll
            for (int v = 0; v < 4; ++v) y[tt][v] = acc[i * TPI + tt][v];
        hsq += epilogue_item<bf16_t, EPI>(a, y, rs, m, ptile + i * TPI, g);
    };
    if constexpr (TPI == 2 && NT >= 4) {
        auto two = [&](int i) __attribute__((always_inline)) {
            float y0[2][4], y1[2][4];
#pragma unroll
            for (int tt = 0; tt < 2; ++tt)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    y0[tt][v] = acc[i * 2 + tt][v];
                    y1[tt][v] = acc[i * 2 + 2 + tt][v];
                }
            epilogue_two<EPI>(a, y0, y1, rs, m, ptile + i * 2, g);
        };
        static_assert(NT == 4 || NT == 6, "a wave's first tile is a multiple of NT");
        if (NT == 4 || (ptile & 3) == 0) {  // uniform
            two(0);
            if constexpr (NT == 6) one(2);
        } else if constexpr (NT == 6) {
            one(0);
            two(1);
        }
    } else {
#pragma unroll
        for (int i = 0; i < NT / TPI; ++i) one(i);
    }
    return hsq;
}

// Cross-wave reduction through LDS and the fused epilogue, shared by the dense and the 4-bit kernels.
template <typename T, int MT, int NT, int EPI>
static __device__ __forceinline__ void reduce_and_store(const GemmArgs& a, f32x4 (&acc)[MT][NT], float (&ss)[MT], unsigned char* smem,
                                                        int lane, int w, int NW, int grp, int row0, const f32x4& resid_first) {
    constexpr bool NORM = (EPI != EPI_RESID);
    const int r16 = lane & 15, g = lane >> 4;
    // ---- cross-wave reduction through LDS ---------------------------------------------------------
    // LDS holds NC = a.red_copies copies of the workgroup's tiles.  With more waves than copies, the last (up to NC) active
    // waves hand their tiles to the first ones, round by round, until NC waves are left; those write their copies and the
    // epilogue items add them up.  (Many-row tile shapes would otherwise have to run with fewer waves.)
    constexpr bool ROUNDS = (MT * NT > 6);  // only then can the launcher pick fewer copies than waves (48 KiB / (MT*NT) KiB < 8)
    const int NC = ROUNDS ? a.red_copies : NW;
    float* red = (float*)smem;                       // [NC][MT*NT][4][64]
    float* ssr = red + (size_t)NC * MT * NT * 256;   // [NW][MT][16]
    auto put = [&](int slot) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int v = 0; v < 4; ++v) red[(((size_t)slot * MT * NT + mt * NT + nt) * 4 + v) * 64 + lane] = acc[mt][nt][v];
    };
    for (int active = NW; ROUNDS && active > NC;) {  // uniform
        const int k = min(NC, active - NC);  // the top k active waves hand over to waves 0 .. k-1
        if (w >= active - k && w < active) put(w - (active - k));
        __syncthreads();
        if (w < k) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                    for (int v = 0; v < 4; ++v) acc[mt][nt][v] += red[(((size_t)w * MT * NT + mt * NT + nt) * 4 + v) * 64 + lane];
        }
        __syncthreads();
        active -= k;
    }
    const int copies = ROUNDS ? (NW < NC ? NW : NC) : NW;
    if (!ROUNDS || w < copies) put(w);
    if (NORM) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            float t = wave_xor_add(wave_xor_add(ss[mt], 16), 32);
            if (lane < 16) ssr[(w * MT + mt) * 16 + lane] = t;
        }
    }
    __syncthreads();

    // ---- epilogue: an "item" is one 16x16 tile (RESID, LOGITS) or a pair of tiles (QKV, SWIGLU) ---
    constexpr bool PAIR = (EPI == EPI_QKV || EPI == EPI_SWIGLU);
    constexpr int TPI = PAIR ? 2 : 1;  // tiles per item
    constexpr int ITEMS = MT * NT / TPI;
    static_assert(!PAIR || NT % 2 == 0, "paired epilogues need an even NT");
    for (int item = w; item < ITEMS; item += NW) {
        const int mt = item / (NT / TPI), ntp = item % (NT / TPI);
        const int m = row0 + mt * 16 + r16;
        float y[TPI][4];
#pragma unroll
        for (int t = 0; t < TPI; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                float s = 0.f;
                for (int ww = 0; ww < copies; ++ww) s += red[(((size_t)ww * MT * NT + mt * NT + ntp * TPI + t) * 4 + v) * 64 + lane];
                y[t][v] = s;
            }
        float rs = 1.f;
        if (NORM) {
            float s = 0.f;
            for (int ww = 0; ww < NW; ++ww) s += ssr[(ww * MT + mt) * 16 + r16];
            rs = 1.0f / sqrtf(s / (float)a.K + a.eps);
        }
        const int ptile = grp * NT + ntp * TPI;  // first packed tile of the item
        float hsq = epilogue_item<T, EPI>(a, y, rs, m, ptile, g, item == w ? &resid_first : nullptr);
        if constexpr (EPI == EPI_RESID) {
            if (a.ssp_out) {  // uniform over the workgroup; every lane of the wave is here
                hsq = wave_xor_add(wave_xor_add(hsq, 16), 32);
                if (g == 0 && ptile * 16 < a.N && m < a.ssp_stride) a.ssp_out[(size_t)ptile * a.ssp_stride + m] = hsq;
            }
        }
    }
}

// The values the first loads depend on travel as leading scalar kernel arguments: those can be preloaded into SGPRs with
// the wave (compiler option -amdgpu-kernarg-preload-count), whereas the fields of the by-value struct are fetched from
// the kernarg segment by a scalar load the whole prologue would have to wait for.
template <typename T, int MT, int NT, int EPI>
__global__ void __launch_bounds__(512) skinny_gemm_kernel(const void* Wp, const void* X, int nkt_, int ldx_, int M_, int x_frag_, const GemmArgs a) {
    using E = Elem<T>;
    using frag_t = typename E::frag_t;
    constexpr bool NORM = (EPI != EPI_RESID);
    constexpr int PF = (MT + NT <= 3) ? 8 : 4;  // k-steps of loads kept in flight per wave
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, NW = blockDim.x >> 6;
    const int r16 = lane & 15, g = lane >> 4;
    const int grp = blockIdx.x, mb = blockIdx.y;
    const int row0 = mb * MT * 16;

    // k-tiles are dealt to the waves round-robin (wave w takes w, w + NW, ...): at any moment the workgroup's
    // waves read neighbouring KiBs, so the group's weight block is swept front to back as one stream.
    const int nsteps = (nkt_ - w + NW - 1) / NW;  // >= 1: the host never launches more waves than k-tiles
    const unsigned char* wbase = (const unsigned char*)Wp + ((size_t)grp * nkt_) * (size_t)(NT * 1024) + (size_t)lane * 16;
    // Rows beyond M read row M-1 instead: their results are never stored, and the loop stays free of branches.
    // Fragment-major activations (padded to whole 16-row tiles) are addressed like the weights.
    const T* xrow[MT];
    const size_t xstep = x_frag_ ? (size_t)64 * E::EPF : (size_t)E::KT;  // elements between consecutive k-tiles
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        if (x_frag_) {
            xrow[mt] = (const T*)X + (((size_t)(mb * MT + mt) * nkt_) * 64 + lane) * E::EPF;
        } else {
            const int m = min(row0 + mt * 16 + r16, M_ - 1);
            xrow[mt] = (const T*)X + (size_t)m * ldx_ + g * E::EPF;
        }
    }

    const f32x4 resid_first = prefetch_resid<T, MT, NT, EPI>(a, w, grp, row0, r16, g);
    f32x4 acc[MT][NT];
    float ss[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        ss[mt] = 0.f;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
    }

    // Software pipeline of PF k-steps.  The loads are unconditional (step indices are clamped to the wave's last k-tile) so that
    // those of later steps stay in flight while earlier ones are consumed.
    // f32 with two and four row tiles: a step's rows are asked for before its weights (33 rows x 32000 x 4096 177 -> 167 us, 400 rows QKV 289 -> 278;
    // one row tile the other way round: 16 rows, output projection 17.3 / 17.9)
    constexpr bool ROWS_FIRST = sizeof(T) == 4 && MT > 1;
    frag_t bq[PF][NT], aq[PF][MT];
    auto issue = [&](int s, int step) {
        const int kt = w + min(step, nsteps - 1) * NW;
        const unsigned char* wp = wbase + (size_t)kt * (NT * 1024);
        auto load_rows = [&] {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) aq[s][mt] = *(const frag_t*)(xrow[mt] + (size_t)kt * xstep);
        };
        if (ROWS_FIRST) load_rows();
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) bq[s][nt] = load_w<T>(wp + nt * 1024);
        if (!ROWS_FIRST) load_rows();
    };
    // f32 residual projections, one feature tile to a group: the four dependent matrix instructions of a row tile alternate with the other row
    // tiles' (one after another, launches that fill the matrix cores are 30 % longer: 1000 rows x 4096 x 11008 982 / 1282 us).  QKV and gate/up have
    // two tiles and more to alternate between and are 1 to 3 % longer so.
    auto consume = [&](int s) {
#pragma unroll
        for (int e = 0; e < (NORM ? 1 : E::STEPS); ++e)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                const frag_t av = aq[s][mt];
                if (NORM) ss[mt] += E::sumsq(av);
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = NORM ? E::mma(bq[s][nt], av, acc[mt][nt]) : E::mma_step(e, bq[s][nt], av, acc[mt][nt]);
            }
    };
#pragma unroll
    for (int s = 0; s < PF; ++s) issue(s, s);
    const int nrounds = (nsteps + PF - 1) / PF;
    for (int rd = 0; rd + 1 < nrounds; ++rd) {
#pragma unroll
        for (int s = 0; s < PF; ++s) {
            consume(s);
            issue(s, (rd + 1) * PF + s);
            __builtin_amdgcn_sched_barrier(0);  // keep the refill right behind its consumer: PF-1 stages stay in flight
        }
    }
    // (no loads in here: a step that the wave does not have is skipped.  Multiplied by zero instead, the six of eight steps that 256 columns
    // in f32 leave over were 0.7 - 1.4 us of a launch.)
#pragma unroll
    for (int s = 0; s < PF; ++s)
        if ((nrounds - 1) * PF + s < nsteps) consume(s);

    reduce_and_store<T, MT, NT, EPI>(a, acc, ss, smem, lane, w, NW, grp, row0, resid_first);
}

// QKV of up to 16 rows where every rotary pair of query / key tiles has a value tile to go with it (as many KV heads as query heads): the
// workgroup takes pair i and value tile i.  Bound by the weight stream, and a launch lasts as long as its most loaded compute unit: 768 tiles
// of a 4096-wide layer are 384 pairs on 256 compute units, four tiles on half of them, where this is three on each.  16 rows, us, groups
// of two (four) tiles -> this: 2816 wide 19.8 -> 16.1, 3072 20.4 -> 16.7, 4096 23.6 -> 20.6 (4.9 TB/s), 4096 in f32 45.6 -> 40.6, 8192 columns x
// 12288 46.8 -> 39.6; groups of four: 5632 50.0 -> 43.1, 6144 52.8 -> 46.5, 7168 61.5 -> 58.
template <typename T>
__global__ void __launch_bounds__(512) skinny_qkv_kernel(const void* Wp, const void* X, int nkt_, int ldx_, int M_, int flags, const GemmArgs a) {
    using E = Elem<T>;
    using frag_t = typename E::frag_t;
    constexpr int NT = 3, PF = 8;
    __shared__ __align__(16) float red[8 * NT * 256];
    __shared__ float ssr[8 * 16];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, NW = blockDim.x >> 6;
    const int r16 = lane & 15, g = lane >> 4;
    const int x_frag = flags & 1, lsh = flags >> 1;  // log2 of the weights' tiles per group
    const int nsteps = (nkt_ - w + NW - 1) / NW;  // >= 1: the host never launches more waves than k-tiles
    const int pair = blockIdx.x, vtile = 2 * gridDim.x + blockIdx.x;  // gridDim.x pairs, then as many value tiles
    auto first = [&](int pt) {
        return (const unsigned char*)Wp + ((((size_t)(pt >> lsh) * nkt_) << lsh) + (pt & ((1 << lsh) - 1))) * 1024 + (size_t)lane * 16;
    };
    const unsigned char* const wb[NT] = {first(2 * pair), first(2 * pair + 1), first(vtile)};
    const T* xrow;
    const size_t xstep = x_frag ? (size_t)64 * E::EPF : (size_t)E::KT;
    if (x_frag)
        xrow = (const T*)X + (size_t)lane * E::EPF;
    else
        xrow = (const T*)X + (size_t)min(r16, M_ - 1) * ldx_ + g * E::EPF;

    const QkvPre pre = prefetch_qkv(a, r16, 2 * pair, g);
    f32x4 acc[NT];
    float ss = 0.f;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[nt] = f32x4{0.f, 0.f, 0.f, 0.f};
    frag_t bq[PF][NT], aq[PF];
    auto issue = [&](int s, int step) {
        const int kt = w + min(step, nsteps - 1) * NW;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) bq[s][nt] = load_w<T>(wb[nt] + ((size_t)kt << (10 + lsh)));
        aq[s] = *(const frag_t*)(xrow + (size_t)kt * xstep);
    };
    auto consume = [&](int s) {
        ss += E::sumsq(aq[s]);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[nt] = E::mma(bq[s][nt], aq[s], acc[nt]);
    };
#pragma unroll
    for (int s = 0; s < PF; ++s) issue(s, s);
    const int nrounds = (nsteps + PF - 1) / PF;
    for (int rd = 0; rd + 1 < nrounds; ++rd) {
#pragma unroll
        for (int s = 0; s < PF; ++s) {
            consume(s);
            issue(s, (rd + 1) * PF + s);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int s = 0; s < PF; ++s)
        if ((nrounds - 1) * PF + s < nsteps) consume(s);

#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int v = 0; v < 4; ++v) red[((w * NT + nt) * 4 + v) * 64 + lane] = acc[nt][v];
    ss = wave_xor_add(wave_xor_add(ss, 16), 32);
    if (lane < 16) ssr[w * 16 + lane] = ss;
    __syncthreads();
    if (w > 1 && NW > 1) return;
    float s = 0.f;
    for (int k = 0; k < NW; ++k) s += ssr[k * 16 + r16];
    const float rs = 1.0f / sqrtf(s / (float)a.K + a.eps);
    auto tile_sum = [&](int nt, float (&y)[4]) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            y[v] = 0.f;
            for (int k = 0; k < NW; ++k) y[v] += red[((k * NT + nt) * 4 + v) * 64 + lane];
        }
    };
    // wave 0 finishes the pair, wave 1 the value tile
    if (w == 0) {
        float y[2][4];
        tile_sum(0, y[0]);
        tile_sum(1, y[1]);
        epilogue_item<T, EPI_QKV>(a, y, rs, r16, 2 * pair, g, nullptr, &pre);
    }
    if ((w == 1 || NW == 1) && r16 < a.M) {
        float y[4];
        tile_sum(2, y);
        const int tph = a.hd >> 4, head = vtile / tph, t = vtile % tph * 16 + g * 4;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            y[v] *= rs;
            if (a.bias) y[v] += a.bias[vtile * 16 + g * 4 + v];
        }
        T* dst = (T*)pre.krow + a.layer_off + a.stride_kv + (size_t)(head - a.Hq - a.Hkv) * a.stride_head;
        *(typename E::out4_t*)(dst + t) = E::pack4(y[0], y[1], y[2], y[3]);
    }
}

// copies of the workgroup's tiles the cross-wave reduction keeps in LDS: as many as there are waves, within about 48 KiB
static int reduction_copies(int nw, int mt, int nt) {
    const int fit = 48 / (mt * nt);  // 1 KiB per tile and copy
    return nw < fit ? nw : (fit < 1 ? 1 : fit);
}

template <typename T, int MT, int NT, int EPI>
static hipError_t launch_one(int NW, int n_groups, const GemmArgs& a0, hipStream_t s) {
    GemmArgs a = a0;
    const int mblocks = (a.M + MT * 16 - 1) / (MT * 16);
    if (NW > 8) NW = 8;
    a.red_copies = reduction_copies(NW, MT, NT);
    const size_t lds = (size_t)a.red_copies * MT * NT * 1024 + (size_t)NW * MT * 16 * sizeof(float);
    hipLaunchKernelGGL((skinny_gemm_kernel<T, MT, NT, EPI>), dim3(n_groups, mblocks), dim3(NW * 64), lds, s, a.Wp, a.X, a.nkt, a.ldx, a.M, a.x_frag, a);
    return hipGetLastError();
}

template <typename T, int EPI>
static hipError_t launch_mt_nt(int MT, int NT, int NW, int n_groups, const GemmArgs& a, hipStream_t s) {
    constexpr bool PAIR = (EPI == EPI_QKV || EPI == EPI_SWIGLU);
#define FS_CASE(mt, nt) \
    if (MT == mt && NT == nt) return launch_one<T, mt, nt, EPI>(NW, n_groups, a, s);
    if constexpr (!PAIR) {
        FS_CASE(1, 1) FS_CASE(2, 1) FS_CASE(4, 1)
    }
    FS_CASE(1, 2) FS_CASE(2, 2) FS_CASE(4, 2) FS_CASE(1, 4) FS_CASE(2, 4) FS_CASE(4, 4)
#undef FS_CASE
    return hipErrorInvalidValue;
}

hipError_t launch_gemm(int dtype, int epi, int NT, int NW, int n_groups, const GemmArgs& a, hipStream_t s) {
    // 33 to 64 rows per block: 4 row tiles and at most 4 waves (several smaller workgroups per compute unit overlap each
    // other's start-up and epilogue; 8 waves: QKV 42 -> 44 us, gate/up 50 -> 53 us at 64 rows).  Two 32-row blocks per
    // group instead were slower as well (gate/up 54 -> 61 us).
    const int MT = a.M <= 16 ? 1 : (a.M <= 32 ? 2 : 4);
    if (epi == EPI_QKV && MT == 1 && a.Hq == a.Hkv) {
        // pairs with a value tile where that leaves fewer tiles on the most loaded compute unit; with two full rounds of them (its 8 waves
        // leave no registers for a second workgroup on the unit) groups of four are the faster ones all the same (512 pairs 76.0 / 70.3 us)
        const int pairs = a.Hq * a.hd / 16;
        if (pairs < 480 && (pairs + 255) / 256 * 3 < (n_groups + 255) / 256 * NT) {
            const int flags = a.x_frag | (NT == 4 ? 4 : 2);
            const dim3 grid(pairs), block(std::min(NW, 8) * 64);
            if (dtype == 0)
                hipLaunchKernelGGL(skinny_qkv_kernel<float>, grid, block, 0, s, a.Wp, a.X, a.nkt, a.ldx, a.M, flags, a);
            else
                hipLaunchKernelGGL(skinny_qkv_kernel<bf16_t>, grid, block, 0, s, a.Wp, a.X, a.nkt, a.ldx, a.M, flags, a);
            return hipGetLastError();
        }
    }
    if (MT == 4 && NW > 4) NW = 4;
    if (MT * NT >= 8 && NW > 4) NW = 4;  // 8 tiles per workgroup: 4 waves keep a copy each in LDS without reduction rounds
#define FS_EPI(e)                                                                      \
    if (epi == e) {                                                                    \
        if (dtype == 0) return launch_mt_nt<float, e>(MT, NT, NW, n_groups, a, s);     \
        return launch_mt_nt<bf16_t, e>(MT, NT, NW, n_groups, a, s);                    \
    }
    FS_EPI(EPI_QKV) FS_EPI(EPI_RESID) FS_EPI(EPI_SWIGLU) FS_EPI(EPI_LOGITS)
#undef FS_EPI
    return hipErrorInvalidValue;
}

// ---- many-row segments (chunked prefill, stacked requests): projection as a matrix product -------------------
// With more than a row tile or two the projections stop being a pure weight stream: the few-row kernel re-reads the
// activations once per workgroup and ends up bound by the path from L2 into the compute units.  This kernel shares the
// activations between the waves instead.  Workgroup = 4 waves; block = 128 rows x 256 features (from 384 rows), 128 rows
// x 128 features (up to 383 rows) or 64 rows x 128 features (LM head and gate/up of up to 64 rows); wave w owns a quarter of the features for
// all rows of the block (8 x 4, 8 x 2 or 4 x 2 accumulator tiles).
//   * Weights are private to a wave, so they skip LDS: each wave streams its tiles per k-tile straight from the re-tiled
//     copy into registers, a ring of PFW k-tiles deep (the same coalesced 1 KiB fragment loads as the few-row kernel).
//   * Activations are shared by the four waves: the block's fragments per k-tile (fragment-major in memory, so a plain
//     copy of 8 or 4 KiB) go through a double-buffered LDS stage, one barrier per k-tile.
//   Per k-tile and wave of the largest block: 8 LDS fragment reads + 4 global fragment loads feed 32 MFMAs — half of the
//   LDS and of the vector-memory bandwidth at full MFMA rate.  What binds it there is the L2: every k-tile of a block
//   asks it for 24 KiB (16 KiB of weights, 8 KiB of activations) per 2.1 MFLOP.
//   * RMSNorm: the 256-feature blocks take the row scale from partial sums of squares left by the producer of the
//     activations (GemmArgs::ssp_in), so their loop contains no per-element arithmetic; the 128-feature blocks have
//     registers to spare and add the squares up while they stage the activations.
//   * Workgroups that share weights (the row blocks of one feature block) get consecutive slots on one XCD, so the
//     weights are fetched from HBM once and hit in that XCD's L2 afterwards.
//   * Projections too narrow to fill the chip (d_model outputs, a few row blocks) split K over `k_splits` workgroups;
//     each writes its raw accumulator tiles (MFMA lane order, so 16 bytes per lane, contiguous per wave) to a scratch
//     array and wide_fixup_kernel adds them up and runs the residual epilogue.
//   * Below 129 rows only what mid_kernel sends here.
template <int EPI, bool PARTIAL, int BMT, int WNT, int WAVES, bool STREAMW>
__global__ void __launch_bounds__(WAVES * 64, BMT == 8 ? 2 : 3) wide_gemm_kernel(const GemmArgs a, int layout_nt, int n_tiles, int n_cols, int m_blocks, int k_splits,
                                                           float* part) {
    using T = bf16_t;
    using E = Elem<T>;
    using frag_t = E::frag_t;
    constexpr bool NORM = (EPI != EPI_RESID);
    // Weight fragments are fetched PFW k-tiles ahead and activation pieces XD k-tiles ahead.  Loads retire in order, so
    // waiting for an activation piece also waits for every weight fetch issued before it: XD, not PFW, is the latency
    // budget of a weight fetch, and PFW > XD + 1 only adds loads in flight.  (With XD = 2 a k-tile took 0.7 us whenever
    // the weights came from HBM — one row block — i.e. about a third of the memory latency.)
    constexpr int PFW = (BMT == 8 && WNT == 4) ? 4 : 8;
    constexpr int XD = (BMT == 8 && WNT == 4) ? 4 : 8;
    constexpr int XL = BMT / WAVES;        // 16-byte pieces of the activation stage per thread
    static_assert(BMT % WAVES == 0 && BMT % 4 == 0, "row tiles must split over the waves and over groups of 4");
    __shared__ __align__(16) unsigned char xs[2][BMT * 1024];
    __shared__ float rs_s[BMT * 16];

    // XCD-aware placement (workgroup id = slot * 8 + XCD): the row blocks of a feature block are neighbours on one XCD, which shares its weights.
    // Without K slices, or with a multiple of 8 feature blocks, XCD x takes the feature blocks x, x + 8, ...; K slices of other numbers go by
    // units = (K slice, feature block), neighbours on one XCD, so that none gets more than its share.  (By units also there, us: 1024 x 1024 in
    // 8 feature blocks and 4 slices, 200 rows 11.9 -> 12.8, 383 rows 13.0 -> 14.6.)
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    int col, mb, ks;
    if (k_splits == 1 || (n_cols & 7) == 0) {
        const int per_col = m_blocks * k_splits;
        col = (slot / per_col) * 8 + xcd, mb = (slot % per_col) / k_splits, ks = slot % k_splits;
        if (col >= n_cols) return;
    } else {
        const int units = n_cols * k_splits, unit = (units * xcd >> 3) + slot / m_blocks;
        mb = slot % m_blocks, ks = unit / n_cols, col = unit % n_cols;
        if (unit >= units * (xcd + 1) >> 3) return;
    }
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int r16 = lane & 15, g = lane >> 4;
    const int kt_lo = (int)((long long)a.nkt * ks / k_splits), nkt = (int)((long long)a.nkt * (ks + 1) / k_splits) - kt_lo;  // >= 1 (host)
    const int mt0 = mb * BMT, m_tiles = (a.M + 15) >> 4;

    // RMSNorm scale of the rows.  The 256-feature blocks have no registers to spare and take it from the partial sums of
    // squares their producer left (one per workgroup column of that producer: a few dozen independent loads per row); the
    // 128-feature blocks add the squares up themselves while they stage the activations (see store_x), so that they can
    // also follow a producer that leaves no such sums.
    constexpr bool SELF_NORM = NORM && WNT == 2;
    if (NORM && !SELF_NORM && t < BMT * 16) {
        const int m = min(mt0 * 16 + t, a.M - 1);
        float s0 = 0.f, s1 = 0.f;
        int j = 0;
#pragma unroll 4
        for (; j + 1 < a.ssp_n; j += 2) {
            s0 += a.ssp_in[(size_t)j * a.ssp_stride + m];
            s1 += a.ssp_in[(size_t)(j + 1) * a.ssp_stride + m];
        }
        if (j < a.ssp_n) s0 += a.ssp_in[(size_t)j * a.ssp_stride + m];
        rs_s[t] = 1.0f / sqrtf((s0 + s1) / (float)a.K + a.eps);
    }

    // this wave's weight tiles; tiles beyond the matrix re-read the last one (their results are never stored).
    // Addresses are a uniform base plus a 32-bit byte offset per lane (one matrix is far below 4 GiB), advanced by one
    // k-tile per fetch until the last k-tile of the slice is reached.
    const int pt0 = (col * WAVES + w) * WNT;
    const unsigned char* wbase = (const unsigned char*)a.Wp;
    const unsigned char* xbase = (const unsigned char*)a.X;
    unsigned woff[WNT], xoff[XL];
#pragma unroll
    for (int nt = 0; nt < WNT; ++nt) {
        const int pc = min(pt0 + nt, n_tiles - 1);
        woff[nt] = (unsigned)((((size_t)(pc / layout_nt) * a.nkt + kt_lo) * layout_nt + pc % layout_nt) * 1024 + (size_t)lane * 16);
    }
    const unsigned wstep = (unsigned)layout_nt * 1024;
    // this thread's 16-byte pieces of the activation stage: fragments w, w + WAVES, ... of the block's BMT
#pragma unroll
    for (int i = 0; i < XL; ++i) {
        const int mt = min(mt0 + w + WAVES * i, m_tiles - 1);
        xoff[i] = (unsigned)((((size_t)mt * a.nkt + kt_lo) * 64 + lane) * 16);
    }
    const unsigned xstep = 1024;
    int wk = 0, xk = 0;  // k-tiles already fetched (weights / activations)

    f32x4 acc[BMT][WNT];
#pragma unroll
    for (int mt = 0; mt < BMT; ++mt)
#pragma unroll
        for (int nt = 0; nt < WNT; ++nt) acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};

    frag_t wq[PFW][WNT], xr[XD][XL];
    auto fetch_w = [&](int j, int) {
#pragma unroll
        for (int nt = 0; nt < WNT; ++nt)  // weights that other row blocks read again stay in L2; with one row block they stream past it
            wq[j][nt] = STREAMW ? load_w<T>(wbase + woff[nt]) : *(const frag_t*)(wbase + woff[nt]);
        const unsigned adv = (++wk < nkt) ? wstep : 0u;  // past the slice's end the last k-tile is re-read (and never used)
#pragma unroll
        for (int nt = 0; nt < WNT; ++nt) woff[nt] += adv;
    };
    auto load_x = [&](int j, int) {
#pragma unroll
        for (int i = 0; i < XL; ++i) xr[j][i] = *(const frag_t*)(xbase + xoff[i]);
        const unsigned adv = (++xk < nkt) ? xstep : 0u;
#pragma unroll
        for (int i = 0; i < XL; ++i) xoff[i] += adv;
    };
    // Self-computed RMSNorm scale: every 16-byte piece of the activations passes through exactly one thread on its way to
    // LDS (lane (r16, g) carries 8 consecutive k of row r16), which adds its squares up; pieces fetched past the end of the
    // K range (the ring runs ahead of the loop) are not counted.
    float ssq[XL];
#pragma unroll
    for (int i = 0; i < XL; ++i) ssq[i] = 0.f;
    int xstored = 0;  // k-tiles handed to LDS so far
    auto store_x = [&](int j, int buf) {
#pragma unroll
        for (int i = 0; i < XL; ++i) *(frag_t*)(xs[buf] + (size_t)(w + WAVES * i) * 1024 + (size_t)lane * 16) = xr[j][i];
        if constexpr (SELF_NORM) {
            const bool counts = xstored < nkt;  // uniform
#pragma unroll
            for (int i = 0; i < XL; ++i) {
                const bf16x2x4 pr = __builtin_bit_cast(bf16x2x4, xr[j][i]);
                float sq = 0.f;
#pragma unroll
                for (int e = 0; e < 4; ++e) sq = __builtin_amdgcn_fdot2_f32_bf16(pr.v[e], pr.v[e], sq, false);
                ssq[i] += counts ? sq : 0.f;
            }
            ++xstored;
        }
    };
    // Pipeline, k-tile kt: weights in wq[kt % PFW], activations in LDS buffer kt & 1; xr[n % XD] carries k-tile n from
    // memory to LDS (n = kt + 1 .. kt + XD are in registers or in flight when the iteration starts).  One barrier per
    // k-tile: it publishes buffer kt & 1 (filled during k-tile kt - 1) and tells that nobody still reads the other buffer,
    // which the refill at the end of the iteration overwrites.
#pragma unroll
    for (int j = 0; j < PFW; ++j) fetch_w(j, j);
#pragma unroll
    for (int j = 0; j < XD; ++j) load_x(j, j);
    store_x(0, 0);
    load_x(0, XD);
    constexpr int U = (PFW % XD == 0) ? PFW : ((XD % PFW == 0) ? XD : PFW * XD);  // kt % PFW, kt % XD and kt & 1 compile-time
    static_assert(U % 2 == 0 && U % PFW == 0 && U % XD == 0, "unroll factor must cover both rings and the buffer parity");
    auto ktile = [&](int ju) {  // k-tile kt0 + ju of a group of U: ring slots and buffer parity are compile-time
        const int j = ju % PFW;
        __syncthreads();
        const unsigned char* xb = xs[ju & 1] + (size_t)lane * 16;
#pragma unroll
        for (int h = 0; h < BMT / 4; ++h) {
            frag_t bf[4];
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) bf[mt] = *(const frag_t*)(xb + (size_t)(h * 4 + mt) * 1024);
#pragma unroll
            for (int nt = 0; nt < WNT; ++nt)
#pragma unroll
                for (int mt = 0; mt < 4; ++mt) acc[h * 4 + mt][nt] = E::mma(wq[j][nt], bf[mt], acc[h * 4 + mt][nt]);
        }
        store_x((ju + 1) % XD, (ju + 1) & 1);
        load_x((ju + 1) % XD, 0);
        fetch_w(j, 0);
    };
    // Whole groups of U k-tiles run as straight-line code: a k-tile that could be skipped inside the loop would make the
    // compiler assume that the fetch it is about to wait for might be the newest one in flight, and wait for all of them
    // (the weight ring would then drain once per group).  The last, partial group takes the guarded form.
    int kt0 = 0;
    for (; kt0 + U <= nkt; kt0 += U) {
#pragma unroll
        for (int ju = 0; ju < U; ++ju) ktile(ju);
    }
#pragma unroll
    for (int ju = 0; ju < U; ++ju)
        if (kt0 + ju < nkt) ktile(ju);  // uniform over the workgroup

    if constexpr (PARTIAL) {
        // raw tiles: part[ks][m tile][n tile][lane] (f32x4); tiles beyond the matrix are dropped
        const int nt_all = n_cols * WAVES * WNT;
#pragma unroll
        for (int mt = 0; mt < BMT; ++mt) {
            if (mt0 + mt >= m_tiles) break;
#pragma unroll
            for (int nt = 0; nt < WNT; ++nt)
                ((f32x4*)part)[(((size_t)ks * m_tiles + mt0 + mt) * nt_all + pt0 + nt) * 64 + lane] = acc[mt][nt];
        }
        return;
    }
    if constexpr (SELF_NORM) {
#pragma unroll
        for (int i = 0; i < XL; ++i) {
            const float tot = wave_xor_add(wave_xor_add(ssq[i], 16), 32);
            if (g == 0) rs_s[(w + WAVES * i) * 16 + r16] = 1.0f / sqrtf(tot / (float)a.K + a.eps);
        }
        __syncthreads();
    }
    // ---- epilogue straight from the accumulators -------------------------------------------------------------
    // (residual projections also leave one partial sum of squares per row and workgroup: the waves' shares meet in LDS,
    //  where the activation stage is free once every wave has left the loop)
    float* hs = (float*)xs[0];  // [WAVES][BMT * 16]
    if constexpr (EPI == EPI_RESID) {
        if (a.ssp_out) __syncthreads();
    }
#pragma unroll
    for (int mt = 0; mt < BMT; ++mt) {
        const int m = (mt0 + mt) * 16 + r16;
        const float rs = NORM ? rs_s[mt * 16 + r16] : 1.f;
        float hsq = epilogue_row<EPI, WNT>(a, acc[mt], rs, m, pt0, g);
        if constexpr (EPI == EPI_RESID) {
            if (a.ssp_out) {
                hsq = wave_xor_add(wave_xor_add(hsq, 16), 32);
                if (g == 0) hs[w * (BMT * 16) + mt * 16 + r16] = hsq;
            }
        }
    }
    if constexpr (EPI == EPI_RESID) {
        if (a.ssp_out) {
            __syncthreads();
            if (t < BMT * 16) {
                float sum = 0.f;
#pragma unroll
                for (int ww = 0; ww < WAVES; ++ww) sum += hs[ww * (BMT * 16) + t];
                const int m = mt0 * 16 + t;
                if (m < a.ssp_stride) a.ssp_out[(size_t)col * a.ssp_stride + m] = sum;
            }
        }
    }
}

// Sum of the K slices' raw tiles + residual epilogue.  One wave per (row tile, group of WNT feature tiles): the same lane layout as
// the accumulators; a workgroup's 4 waves leave one partial sum of squares per row.  All loads of a wave go out together (a loop
// of load - add per slice before: 512 rows x 4096 features, 4 slices 10.5 - 12.7 -> 9.8 - 10.9 us; 1024 rows, 2 slices 13.4 -> 12.6).
template <int KS, int WNT>
__global__ void __launch_bounds__(256) wide_fixup_kernel(const GemmArgs a, int nt_all, const float* part) {
    const int lane = threadIdx.x & 63, r16 = lane & 15, g = lane >> 4;
    const int m_tiles = (a.M + 15) >> 4, groups = nt_all / WNT;
    __shared__ float hs[4][16];
    const int wv = threadIdx.x >> 6;
    const int unit = blockIdx.x * 4 + wv;  // groups is a multiple of 4: the workgroup's 4 units are neighbours of one row tile
    if (unit >= m_tiles * groups) return;  // whole workgroup
    const int mt = unit / groups, grp = unit % groups;
    const int m = mt * 16 + r16;
    f32x4 v[WNT][KS], pre[WNT];
#pragma unroll
    for (int nt = 0; nt < WNT; ++nt) {
        const int ptile = grp * WNT + nt;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) v[nt][ks] = ((const f32x4*)part)[(((size_t)ks * m_tiles + mt) * nt_all + ptile) * 64 + lane];
        pre[nt] = f32x4{0.f, 0.f, 0.f, 0.f};
        const int n = ptile * 16 + g * 4;
        if (m < a.M && n < a.N) pre[nt] = load_resid<bf16_t>(a, m, n);
    }
    float hsq = 0.f;
#pragma unroll
    for (int nt = 0; nt < WNT; ++nt) {
        f32x4 sum = v[nt][0];
#pragma unroll
        for (int ks = 1; ks < KS; ++ks) sum += v[nt][ks];
        const float y[1][4] = {{sum[0], sum[1], sum[2], sum[3]}};
        hsq += epilogue_item<bf16_t, EPI_RESID>(a, y, 1.f, m, grp * WNT + nt, g, &pre[nt]);
    }
    if (a.ssp_out) {
        hsq = wave_xor_add(wave_xor_add(hsq, 16), 32);
        if (g == 0) hs[wv][r16] = hsq;
        __syncthreads();
        if (threadIdx.x < 16 && mt * 16 + (int)threadIdx.x < a.ssp_stride && (grp >> 2) * (64 * WNT) < a.N)  // not for padding blocks
            a.ssp_out[(size_t)(grp >> 2) * a.ssp_stride + mt * 16 + threadIdx.x] = hs[0][threadIdx.x] + hs[1][threadIdx.x] + hs[2][threadIdx.x] + hs[3][threadIdx.x];
    }
}

template <int WNT>
static hipError_t launch_fixup(const GemmArgs& a, int nt_all, int k_splits, const float* part, hipStream_t s) {
    const int units = ((a.M + 15) / 16) * (nt_all / WNT);
#define FS_FIX(k) \
    case k: hipLaunchKernelGGL((wide_fixup_kernel<k, WNT>), dim3((units + 3) / 4), dim3(256), 0, s, a, nt_all, part); break;
    switch (k_splits) { FS_FIX(1) FS_FIX(2) FS_FIX(3) FS_FIX(4) FS_FIX(5) FS_FIX(6) FS_FIX(7) FS_FIX(8) default: return hipErrorInvalidValue; }
#undef FS_FIX
    return hipGetLastError();
}

// ---- many-row segments: 256-row blocks, both operands through LDS ------------------------------------------------------
// The 128-row kernel above moves 24 KiB from L2 per k-tile and block for 2.1 MFLOP and is bound by the path from L2 into a
// compute unit (about 50 GB/s per unit, whatever the kernel does).  This kernel gives a compute unit one block of 256 rows x
// 16 * BNT features at a time and brings both operands in through LDS, so that every byte that arrives serves the whole block:
// 256 x 256 features take 32 KiB per k-tile for 4.2 MFLOP.  WM x WN waves, each with MT x NT accumulator tiles (WM * MT = 16
// row tiles, WN * NT = BNT feature tiles); the shape in use is 2 x 4 waves of 8 x 4 tiles (two waves per SIMD, 128 accumulator
// registers each).
//   * Both operands are fragment-major in memory (one fragment = one contiguous KiB in MFMA operand order), so a fragment goes
//     from global memory straight into LDS with one 16-byte-per-lane direct-to-LDS load per wave: no staging registers.
//     A stage is the block's 16 activation fragments and BNT weight fragments of one k-tile; the waves share its loads.
//   * STAGES stage buffers; the loads of a stage are issued STAGES - 1 k-tiles before its MFMAs, into the buffer whose
//     fragments were read two k-tiles ago.
//   * Fragments travel LDS -> registers one k-tile ahead, without a second register set: an activation fragment is replaced
//     by the next k-tile's as soon as the MFMAs of its row tile are issued, a weight fragment during the last row tile.
//   * One barrier per k-tile.  It is the bare s_barrier with explicit wait counts: the workgroup fence of __syncthreads would
//     wait for every direct-to-LDS load in flight, i.e. drain the prefetch, and for the fragment reads of the k-tile about to
//     start.  Before the barrier of k-tile kt a wave waits for its own loads of stage kt + 1 (those of stage kt + 2 stay in
//     flight) and for all its LDS reads but the newest ones (reads return in order: everything read two k-tiles ago is then
//     done).  Behind the barrier stage kt + 1 is complete for every wave and the buffer of stage kt - 1 is free.
//   * Epilogues, RMSNorm hand-over (partial sums of squares from the producer) and XCD-aware placement are those of the
//     128-row kernel; K slices (PARTIAL) write the same raw tiles for the same fix-up kernel.

template <int EPI, bool PARTIAL, int WM, int WN, int MT, int NT, int STAGES>
__global__ void __launch_bounds__(WM * WN * 64) block_gemm_kernel(const GemmArgs a, int layout_nt, int n_tiles, int n_cols, int m_blocks, int k_splits,
                                                                  float* part) {
    using T = bf16_t;
    using E = Elem<T>;
    using frag_t = E::frag_t;
    constexpr bool NORM = (EPI != EPI_RESID);
    constexpr bool PAIR = (EPI == EPI_QKV || EPI == EPI_SWIGLU);
    constexpr int NWAVES = WM * WN;
    constexpr int BMT = WM * MT, BNT = WN * NT, FR = BMT + BNT;  // row tiles, feature tiles, fragments (KiB) per stage
    constexpr int DIST = STAGES - 1;                             // k-tiles between a stage's loads and its MFMAs
    constexpr int LPW = (FR + NWAVES - 1) / NWAVES;              // direct-to-LDS loads per wave and stage
    constexpr int RPT = MT + NT;                                 // LDS fragment reads per wave and k-tile
    static_assert(BMT == 16, "blocks are 256 rows");
    static_assert(!PAIR || NT % 2 == 0, "paired epilogues need both tiles of a pair in one wave");
    static_assert(STAGES == 3 || STAGES == 4, "3 or 4 stage buffers");
    static_assert((STAGES * FR + 1) * 1024 <= 160 * 1024, "stage buffers must fit the 160 KiB of LDS");
    static_assert((DIST - 1) * LPW < 64, "vmcnt is a 6-bit counter");
    // one array per stage: distinct objects, so that the compiler's own wait-count tracking of the direct-to-LDS loads never
    // ties a read of one stage to a load into another
    __shared__ __align__(1024) unsigned char sb0[FR * 1024];
    __shared__ __align__(1024) unsigned char sb1[FR * 1024];
    __shared__ __align__(1024) unsigned char sb2[FR * 1024];
    __shared__ __align__(1024) unsigned char sb3[STAGES == 4 ? FR * 1024 : 16];
    __shared__ float rs_s[BMT * 16];
    auto stage_buf = [&](int j) -> unsigned char* { return j == 0 ? sb0 : (j == 1 ? sb1 : (j == 2 ? sb2 : sb3)); };

    const int id = blockIdx.x, xcd = id & 7, slot = id >> 3;
    int col, mb, ks;
    if constexpr (PARTIAL) {  // units (K slice, feature block), neighbours on one XCD: none gets more than its share
        const int units = n_cols * k_splits, unit = (units * xcd >> 3) + slot / m_blocks;
        mb = slot % m_blocks, ks = unit / n_cols, col = unit % n_cols;
        if (unit >= units * (xcd + 1) >> 3) return;
    } else {
        col = (slot / m_blocks) * 8 + xcd, mb = slot % m_blocks, ks = 0;
        if (col >= n_cols) return;
    }
    const int t = threadIdx.x, lane = t & 63;
    const int w = __builtin_amdgcn_readfirstlane(t >> 6), wm = w / WN, wn = w % WN;  // wave-uniform: scalar address arithmetic below
    const int r16 = lane & 15, g = lane >> 4;
    const int kt_lo = (int)((long long)a.nkt * ks / k_splits), nkt = (int)((long long)a.nkt * (ks + 1) / k_splits) - kt_lo;  // >= 1 (host)
    const int mt0 = mb * BMT, m_tiles = (a.M + 15) >> 4;

    if (NORM) {  // RMSNorm scale of the block's rows from the producer's partial sums of squares
        for (int r = t; r < BMT * 16; r += NWAVES * 64) {
            const int m = min(mt0 * 16 + r, a.M - 1);
            float s0 = 0.f, s1 = 0.f;
            int j = 0;
#pragma unroll 4
            for (; j + 1 < a.ssp_n; j += 2) {
                s0 += a.ssp_in[(size_t)j * a.ssp_stride + m];
                s1 += a.ssp_in[(size_t)(j + 1) * a.ssp_stride + m];
            }
            if (j < a.ssp_n) s0 += a.ssp_in[(size_t)j * a.ssp_stride + m];
            rs_s[r] = 1.0f / sqrtf((s0 + s1) / (float)a.K + a.eps);
        }
    }

    // this wave's share of a stage: fragments w * LPW .. + LPW - 1 (activation row tiles first, then weight tiles; a share that
    // runs past the stage's end loads its last fragment again); tiles beyond the matrix re-read the last one (their results
    // are never stored).  Wave-uniform 64-bit base + this lane's 16 bytes.
    const unsigned char* src[LPW];
    unsigned step[LPW], dst_off[LPW];
#pragma unroll
    for (int i = 0; i < LPW; ++i) {
        const int f = min(w * LPW + i, FR - 1);
        const int mt = min(mt0 + f, m_tiles - 1);
        const int pc = min(col * BNT + max(f - BMT, 0), n_tiles - 1);
        const size_t xo = ((size_t)mt * a.nkt + kt_lo) * 1024;
        const size_t wo = (((size_t)(pc / layout_nt) * a.nkt + kt_lo) * layout_nt + pc % layout_nt) * 1024;
        src[i] = (f < BMT) ? (const unsigned char*)a.X + xo : (const unsigned char*)a.Wp + wo;
        step[i] = (f < BMT) ? 1024u : (unsigned)layout_nt * 1024u;
        dst_off[i] = (unsigned)f * 1024u;
    }
    const unsigned lane_off = (unsigned)lane * 16u;
    int issued = 0;
    auto issue = [&](int j) {  // next k-tile of this wave's fragments -> stage buffer j (past the slice's end: the last k-tile again)
        unsigned char* dst = stage_buf(j);
#pragma unroll
        for (int i = 0; i < LPW; ++i) __builtin_amdgcn_global_load_lds(FS_GLB_PTR(src[i] + lane_off), FS_LDS_PTR(dst + dst_off[i]), 16, 0, 0);
        const bool more = ++issued < nkt;
#pragma unroll
        for (int i = 0; i < LPW; ++i) src[i] += more ? step[i] : 0u;
    };
    f32x4 acc[MT][NT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
    frag_t xf[MT], wf[NT];
    auto frag_at = [&](int j, int f) { return *(const frag_t*)(stage_buf(j) + (size_t)f * 1024 + lane_off); };

#pragma unroll
    for (int j = 0; j < DIST; ++j) issue(j);
    FS_WAIT_VM_LGKM((DIST - 1) * LPW, 0);
    __builtin_amdgcn_s_barrier();
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) wf[nt] = frag_at(0, BMT + wn * NT + nt);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) xf[mt] = frag_at(0, wm * MT + mt);
    auto ktile = [&](int ju) {  // k-tile kt0 + ju of a group of STAGES: the buffers are compile-time
        const int jn = (ju + 1) % STAGES;
        FS_WAIT_VM_LGKM((DIST - 2) * LPW, RPT < 15 ? RPT : 15);
        __builtin_amdgcn_s_barrier();
        issue((ju + DIST) % STAGES);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                acc[mt][nt] = E::mma(wf[nt], xf[mt], acc[mt][nt]);
                if (mt == MT - 1) wf[nt] = frag_at(jn, BMT + wn * NT + nt);
            }
            xf[mt] = frag_at(jn, wm * MT + mt);
        }
    };
    int kt0 = 0;
    for (; kt0 + STAGES <= nkt; kt0 += STAGES) {
#pragma unroll
        for (int ju = 0; ju < STAGES; ++ju) ktile(ju);
    }
#pragma unroll
    for (int ju = 0; ju < STAGES; ++ju)
        if (kt0 + ju < nkt) ktile(ju);  // uniform over the workgroup
    // every direct-to-LDS load has landed and every wave has left the loop before LDS is reused below
    FS_WAIT_VM_LGKM(0, 0);
    __builtin_amdgcn_s_barrier();

    if constexpr (PARTIAL) {
        const int nt_all = n_cols * BNT;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            const int mtile = mt0 + wm * MT + mt;
            if (mtile >= m_tiles) break;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
                ((f32x4*)part)[(((size_t)ks * m_tiles + mtile) * nt_all + col * BNT + wn * NT + nt) * 64 + lane] = acc[mt][nt];
        }
        return;
    }
    const int pt0 = col * BNT + wn * NT;
    float* hs = (float*)sb0;  // [WN feature waves][256 rows]
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        const int lr = (wm * MT + mt) * 16 + r16;  // row within the block
        const int m = mt0 * 16 + lr;
        const float rs = NORM ? rs_s[lr] : 1.f;
        float hsq = epilogue_row<EPI, NT>(a, acc[mt], rs, m, pt0, g);
        if constexpr (EPI == EPI_RESID) {
            if (a.ssp_out) {
                hsq = wave_xor_add(wave_xor_add(hsq, 16), 32);
                if (g == 0) hs[wn * (BMT * 16) + lr] = hsq;
            }
        }
    }
    if constexpr (EPI == EPI_RESID) {
        if (a.ssp_out) {
            __syncthreads();
            for (int r = t; r < BMT * 16; r += NWAVES * 64) {
                float sum = 0.f;
#pragma unroll
                for (int x = 0; x < WN; ++x) sum += hs[x * (BMT * 16) + r];
                const int m = mt0 * 16 + r;
                if (m < a.ssp_stride) a.ssp_out[(size_t)col * a.ssp_stride + m] = sum;
            }
        }
    }
}

// ---- 17 to 128 rows: one pass over the weights, both operands through LDS ------------------------------------------------
// A weight byte is used by at most 128 rows, so the launch is bound by what a compute unit can draw: its share of the weights from
// memory and the whole activation block from L2.  A workgroup that streams through registers has too little in flight for that
// (96 workgroups of 4 waves: 2.5 TB/s, through direct-to-LDS loads 4.5 TB/s).  Workgroup = WM x WN x KG waves on a block of
// all rows (16 * WM * MT) x 16 * WN * NT features; the KG wave groups take alternate k-tiles of the block (larger wave tiles, hence
// fewer LDS reads per MFMA, than dividing it further) and add their tiles up through LDS at the end.
//   * A stage is the block's fragments of KG k-tiles; R stage buffers, all but one of them in flight.  Loads are 16 bytes per
//     lane straight into LDS, a fixed number per wave and stage, so the explicit wait counts are exact; stages beyond the K
//     range are still "loaded" (one cache line, into a buffer nobody reads).
//   * Per stage one bare barrier: before it a wave waits for its own loads of stage s + 1 and for its LDS reads of stage s;
//     behind it stage s + 1 is complete and the buffer of stage s free.  Fragments travel LDS -> registers one stage ahead.
//   * RMSNorm: every wave adds up the squares of the activation fragments it multiplies anyway (the row scale is wanted per lane
//     in exactly that layout), so no producer has to leave sums behind.
// Before (few-row kernel, or 64 / 128-row blocks streamed through registers) -> now, 7B shapes, us: 32 rows QKV 25.5 -> 22.7, gate/up
// 38.3 -> 32.4, down 28.5 -> 21.1; 64 rows QKV 34.7 -> 27.2, gate/up 41 -> 33.9, down 30.1 -> 24.3; 128 rows QKV 47.9 -> 35.7, output
// 25.5 -> 19.3, gate/up 53.9 -> 47.7, down 34.7 -> 31.2.  MFMAs, LDS reads and RMSNorm sums are hidden (128 rows QKV: 1.3 us without
// them, the epilogue another 4); above the 19 us in which the same loads run alone it is the activations, first read beyond L2.
template <int EPI, bool PARTIAL, int WM, int WN, int KG, int MT, int NT, int R>
__global__ void __launch_bounds__(WM * WN * KG * 64) stream_gemm_kernel(const void* Wp, const void* X, int nkt, int ldx, int M, int flags, int n_tiles,
                                                                        int kt_per, const GemmArgs a, float* part) {
    using T = bf16_t;
    using E = Elem<T>;
    using frag_t = E::frag_t;
    constexpr bool NORM = (EPI != EPI_RESID);
    constexpr int S = KG;  // k-tiles per stage: one per wave and stage
    constexpr int NW = WM * WN * KG, BMT = WM * MT, BNT = WN * NT, H = MT / KG;
    constexpr int AF = S * BMT, WF = S * BNT, LA = AF / NW, LW = WF / NW, LPS = LA + LW;  // fragments per stage, loads per wave and stage
    static_assert(AF % NW == 0 && WF % NW == 0, "every wave issues the same loads");
    static_assert(KG == 1 || (KG == 2 && MT % 2 == 0), "two wave groups take one k-tile of a stage each");
    static_assert(R % 2 == 0 && R >= 4 && R <= 8, "register sets alternate with the stages; at most 8 buffers");
    static_assert(R * (AF + WF) <= 158 && LPS * (R - 1) < 64, "160 KiB of LDS, 6-bit wait counter");
    static_assert(KG == 1 || H * NT * WM * WN <= AF + WF, "exchange of half the tiles fits a stage buffer");
    // one array per buffer: distinct objects, see block_gemm_kernel
    __shared__ __align__(1024) unsigned char sb0[(AF + WF) * 1024];
    __shared__ __align__(1024) unsigned char sb1[(AF + WF) * 1024];
    __shared__ __align__(1024) unsigned char sb2[(AF + WF) * 1024];
    __shared__ __align__(1024) unsigned char sb3[(AF + WF) * 1024];
    __shared__ __align__(1024) unsigned char sb4[R > 4 ? (AF + WF) * 1024 : 16];
    __shared__ __align__(1024) unsigned char sb5[R > 4 ? (AF + WF) * 1024 : 16];
    __shared__ __align__(1024) unsigned char sb6[R > 6 ? (AF + WF) * 1024 : 16];
    __shared__ __align__(1024) unsigned char sb7[R > 6 ? (AF + WF) * 1024 : 16];
    __shared__ float ssx[KG == 2 ? 2 * BMT * 16 : 1];
    auto buf_at = [&](int j) -> unsigned char* {
        return j == 0 ? sb0 : (j == 1 ? sb1 : (j == 2 ? sb2 : (j == 3 ? sb3 : (j == 4 ? sb4 : (j == 5 ? sb5 : (j == 6 ? sb6 : sb7))))));
    };

    // grid (feature block, K slice); all rows are in one block.
    // What the first loads depend on arrives in SGPRs, and the prologue is kept free of divisions: a launch of a few dozen stages
    // feels every microsecond in front of its first load.
    const int col = blockIdx.x, ks = blockIdx.y;
    const int x_frag = flags & 1, lsh = flags >> 1;  // log2 of the weights' tiles per group
    const int t = threadIdx.x, lane = t & 63;
    const int w = __builtin_amdgcn_readfirstlane(t >> 6), kg = w / (WM * WN), wm = (w / WN) % WM, wn = w % WN;
    const int r16 = lane & 15, g = lane >> 4;
    const int kt_lo = ks * kt_per, n = min(kt_per, nkt - kt_lo);  // >= 1 (host)
    const int ns = (n + S - 1) / S;
    const int m_tiles = (M + 15) >> 4;

    // This wave's fragments of a stage: i * NW + w of the activations (k-tile, row tile), then of the weights (k-tile, feature tile).
    // A 32-bit offset per lane and load, advanced by one stage per issue; tiles beyond the matrix re-read the last one.  The issue
    // path is kept to a handful of instructions per load: with one wave per SIMD it is not hidden by anything.
    const unsigned char* const xb = (const unsigned char*)X;
    const unsigned char* const wb = (const unsigned char*)Wp;
    const unsigned xkt = x_frag ? 1024u : 64u, wkt = 1024u << lsh;  // bytes from one k-tile to the next
    unsigned xo[LA], wo[LW];
    int xn[LA], wn_[LW];  // stages in which the load's k-tile exists
#pragma unroll
    for (int i = 0; i < LA; ++i) {
        const int f = i * NW + w, j = f / BMT, mt = min(f % BMT, m_tiles - 1);
        const unsigned o = x_frag ? (unsigned)mt * (unsigned)nkt * 1024u + (unsigned)lane * 16u
                                  : (unsigned)min(mt * 16 + r16, M - 1) * (unsigned)ldx * 2u + (unsigned)g * 16u;
        xo[i] = o + (unsigned)(kt_lo + j) * xkt;
        xn[i] = (n - j + S - 1) / S;
    }
#pragma unroll
    for (int i = 0; i < LW; ++i) {
        const int f = i * NW + w, j = f / BNT, pc = min(col * BNT + f % BNT, n_tiles - 1);
        wo[i] = ((((unsigned)(pc >> lsh) * (unsigned)nkt + (unsigned)(kt_lo + j)) << lsh) + (unsigned)(pc & ((1 << lsh) - 1))) * 1024u + (unsigned)lane * 16u;
        wn_[i] = (n - j + S - 1) / S;
    }
    const unsigned lane16 = (unsigned)lane * 16u;
    int st = 0;  // next stage to issue
    auto issue = [&](int j) {  // next stage -> buffer j; k-tiles beyond the range fetch the first line of the operand (no branch around a load)
        unsigned char* dst = buf_at(j);
#pragma unroll
        for (int i = 0; i < LA; ++i) {
            const unsigned live = (unsigned)((st - xn[i]) >> 31);  // uniform, all ones or zero
            __builtin_amdgcn_global_load_lds(FS_GLB_PTR(xb + (xo[i] & live)), FS_LDS_PTR(dst + (i * NW + w) * 1024), 16, 0, 0);
            xo[i] += S * xkt;
        }
#pragma unroll
        for (int i = 0; i < LW; ++i) {
            const unsigned live = (unsigned)((st - wn_[i]) >> 31);
            __builtin_amdgcn_global_load_lds(FS_GLB_PTR(wb + (wo[i] & live)), FS_LDS_PTR(dst + (AF + i * NW + w) * 1024), 16, 0, 2);
            wo[i] += S * wkt;
        }
        ++st;
    };

    f32x4 acc[MT][NT];
    float ss[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        ss[mt] = 0.f;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    frag_t xf[2][MT], wf[2][NT];
    auto read = [&](int set, int j) {  // this group's k-tile of the stage in buffer j
        const unsigned char* b = buf_at(j) + lane16;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) wf[set][nt] = *(const frag_t*)(b + (AF + kg * BNT + wn * NT + nt) * 1024);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) xf[set][mt] = *(const frag_t*)(b + (kg * BMT + wm * MT + mt) * 1024);
    };
#pragma unroll
    for (int j = 0; j < R; ++j) issue(j);
    FS_WAIT_VM_LGKM((R - 1) * LPS, 0);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    read(0, 0);
    int cur = 0;  // stage being multiplied
    auto stage = [&](int ju) {  // the next stage, in buffer ju, its fragments in register set ju & 1
        const int set = ju & 1;
        asm volatile("" ::: "memory");
        FS_WAIT_VM_LGKM((R - 2) * LPS, 0);
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        issue(ju);
        read(set ^ 1, (ju + 1) % R);
        if (cur++ * S + kg < n) {  // uniform; the last stage may hold one k-tile only
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                if constexpr (NORM) {
                    const bf16x2x4 pr = __builtin_bit_cast(bf16x2x4, xf[set][mt]);
#pragma unroll
                    for (int e = 0; e < 4; ++e) ss[mt] = __builtin_amdgcn_fdot2_f32_bf16(pr.v[e], pr.v[e], ss[mt], false);
                }
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = E::mma(wf[set][nt], xf[set][mt], acc[mt][nt]);
            }
        }
    };
    int s0 = 0;
    for (; s0 + R <= ns; s0 += R) {
#pragma unroll
        for (int ju = 0; ju < R; ++ju) stage(ju);
    }
#pragma unroll
    for (int ju = 0; ju < R; ++ju) {
        if (s0 + ju >= ns) break;
        stage(ju);
    }
    // every load has landed and every wave has left the loop before LDS is reused or given back
    FS_WAIT_VM_LGKM(0, 0);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");

    // ---- the groups' tiles: each group finishes half of the row tiles ----
    f32x4 own[H][NT];
    float so[H];
    if constexpr (KG == 2) {
        f32x4* give = (f32x4*)(kg == 0 ? sb0 : sb1) + (size_t)(wm * WN + wn) * H * NT * 64 + lane;
        const f32x4* take = (const f32x4*)(kg == 0 ? sb1 : sb0) + (size_t)(wm * WN + wn) * H * NT * 64 + lane;
#pragma unroll
        for (int h = 0; h < H; ++h)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                own[h][nt] = kg == 0 ? acc[h][nt] : acc[H + h][nt];
                give[(h * NT + nt) * 64] = kg == 0 ? acc[H + h][nt] : acc[h][nt];
            }
        if constexpr (NORM) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                const float tot = wave_xor_add(wave_xor_add(ss[mt], 16), 32);
                if (wn == 0 && g == 0) ssx[(kg * BMT + wm * MT + mt) * 16 + r16] = tot;
            }
        }
        __syncthreads();
#pragma unroll
        for (int h = 0; h < H; ++h) {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) own[h][nt] += take[(h * NT + nt) * 64];
            const int rt = (wm * MT + kg * H + h) * 16 + r16;
            so[h] = NORM ? ssx[rt] + ssx[BMT * 16 + rt] : 0.f;
        }
    } else {
#pragma unroll
        for (int h = 0; h < H; ++h) {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) own[h][nt] = acc[h][nt];
            so[h] = NORM ? wave_xor_add(wave_xor_add(ss[h], 16), 32) : 0.f;
        }
    }
    const int pt0 = col * BNT + wn * NT;
#pragma unroll
    for (int h = 0; h < H; ++h) {
        const int mt = wm * MT + kg * H + h;
        if (mt >= m_tiles) break;
        if constexpr (PARTIAL) {  // raw tiles: part[ks][m tile][n tile][lane]
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) ((f32x4*)part)[(((size_t)ks * m_tiles + mt) * (gridDim.x * BNT) + pt0 + nt) * 64 + lane] = own[h][nt];
        } else {
            const float rs = NORM ? 1.0f / sqrtf(so[h] / (float)a.K + a.eps) : 1.f;
            epilogue_row<EPI, NT>(a, own[h], rs, mt * 16 + r16, pt0, g);
        }
    }
}

// Sum of the K slices' raw tiles + residual epilogue, one wave per 16 x 16 tile; a workgroup's four tiles (neighbours of one row tile:
// nt_all is a multiple of 4) leave one partial sum of squares per row where the consumer wants them.
template <int KS>
__global__ void __launch_bounds__(256) stream_fixup_kernel(const GemmArgs a, int nt_all, const float* part) {
    __shared__ float hs[4][16];
    const int lane = threadIdx.x & 63, r16 = lane & 15, g = lane >> 4, wv = threadIdx.x >> 6;
    const int m_tiles = (a.M + 15) >> 4;
    const int unit = blockIdx.x * 4 + wv;
    const int mt = unit / nt_all, ptile = unit % nt_all, m = mt * 16 + r16, n = ptile * 16 + g * 4;
    f32x4 v[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) v[ks] = ((const f32x4*)part)[(((size_t)ks * m_tiles + mt) * nt_all + ptile) * 64 + lane];
    f32x4 pre{0.f, 0.f, 0.f, 0.f};
    if (m < a.M && n < a.N) pre = load_resid<bf16_t>(a, m, n);
    f32x4 sum = v[0];
#pragma unroll
    for (int ks = 1; ks < KS; ++ks) sum += v[ks];
    const float y[1][4] = {{sum[0], sum[1], sum[2], sum[3]}};
    float hsq = epilogue_item<bf16_t, EPI_RESID>(a, y, 1.f, m, ptile, g, &pre);
    if (a.ssp_out) {
        hsq = wave_xor_add(wave_xor_add(hsq, 16), 32);
        if (g == 0) hs[wv][r16] = hsq;
        __syncthreads();
        if (wv == 0 && g == 0 && m < a.ssp_stride && ptile * 16 < a.N)  // not for padding tiles
            a.ssp_out[(size_t)(ptile >> 2) * a.ssp_stride + m] = hs[0][r16] + hs[1][r16] + hs[2][r16] + hs[3][r16];
    }
}

static hipError_t launch_stream_fixup(const GemmArgs& a, int nt_all, int k_splits, const float* part, hipStream_t s) {
    const dim3 grid(((a.M + 15) / 16 * nt_all + 3) / 4);
#define FS_FIX(k) \
    case k: hipLaunchKernelGGL((stream_fixup_kernel<k>), grid, dim3(256), 0, s, a, nt_all, part); break;
    switch (k_splits) { FS_FIX(1) FS_FIX(2) FS_FIX(3) FS_FIX(4) FS_FIX(5) FS_FIX(6) FS_FIX(7) FS_FIX(8) default: return hipErrorInvalidValue; }
#undef FS_FIX
    return hipGetLastError();
}

// Block geometry by projection kind and row count (see the kernel's header comment).
struct WideShape {
    int bmt, wnt, waves;
};
// Up to a few row blocks there are too few 256-feature blocks to fill the chip: 128-feature blocks (2 tiles per wave) then.
static int wide_narrow_rows() {
    static const int v = [] { const char* e = getenv("FLOWSPEC_WIDE_NARROW_ROWS"); return e ? atoi(e) : 384; }();
    return v;
}
static int env_int(const char* name, int dflt) { const char* e = getenv(name); return e ? atoi(e) : dflt; }
static WideShape wide_shape(int epi, int M) {
    if (M <= 64 && (epi == EPI_LOGITS || epi == EPI_SWIGLU)) return WideShape{4, 2, 4};  // one 64-row block
    return M < wide_narrow_rows() ? WideShape{8, 2, 4} : WideShape{8, 4, 4};
}

struct WideGrid {
    int n_cols, m_blocks, k_splits;
    double us;  // residual projections: estimate
};
// K slices for the d_model-wide residual projections: the number that costs least in rounds of one block per compute unit (0.43 us per
// k-tile of a 128 x 256 block, 0.3 of a 128 x 128 one, 4 us into and out of it, 15 with the residual epilogue), partial results (0.5 us a MiB
// to write and sum) and the launch that sums them; at least 8 k-tiles per slice, and no more than the scratch array holds.  512 rows x
// 4096: 4 slices -> 256 workgroups 36 / 60 us for the attention-output / down projection, 8 slices 52 / 80; 13824 x 5120: 2 slices 117 us,
// 3 slices 95; 700 rows 1 slice 172, 3 slices 129; 1024 rows x 1024 x 1024: 1 slice 31.7, 4 slices 20.3.
static WideGrid wide_grid(const WideShape& sh, int epi, int M, int n_tiles, int nkt, size_t part_bytes) {
    WideGrid g;
    const int col_tiles = sh.waves * sh.wnt;
    g.n_cols = (n_tiles + col_tiles - 1) / col_tiles;
    g.m_blocks = (M + sh.bmt * 16 - 1) / (sh.bmt * 16);
    g.k_splits = 1;
    g.us = 0;
    if (epi == EPI_RESID) {
        const size_t per_split = (size_t)((M + 15) / 16) * g.n_cols * col_tiles * 1024;
        const double kt = sh.wnt == 4 ? 0.43 : 0.3;
        g.us = 1e30;
        for (int k = 1; k <= 8 && (k == 1 || (nkt / k >= 8 && per_split * k <= part_bytes)); ++k) {
            const int rounds = ((g.n_cols * k + 7) / 8 * g.m_blocks + 31) / 32;
            const double cost = rounds * (nkt * kt / k + (k > 1 ? 4 : 15)) + (k > 1 ? 4 + per_split * k * 0.5e-6 : 0);
            if (cost < g.us) {
                g.us = cost;
                g.k_splits = k;
            }
        }
    }
    return g;
}

int wide_ssp_parts(int M, int n_tiles) {  // one per workgroup column of the residual projection
    const WideShape sh = wide_shape(EPI_RESID, M);
    const int col_tiles = sh.waves * sh.wnt;
    return (n_tiles + col_tiles - 1) / col_tiles;
}

size_t wide_partial_bytes(int max_rows, int n_tiles) {
    // slices * row tiles * feature tiles KiB: 8 slices of the whole result, and at most 64 MiB; the launches take fewer slices where those do
    // not fit
    const size_t whole = (size_t)8 * ((max_rows + 15) / 16) * (size_t)(n_tiles + 15) * 1024;
    const size_t cap = (size_t)64 << 20;
    return whole < cap ? whole : cap;
}

template <int EPI, int BMT, int WNT, int WAVES>
static hipError_t launch_wide_shape(int layout_nt, int n_tiles, const GemmArgs& a, float* part, size_t part_bytes, hipStream_t s) {
    const WideShape sh{BMT, WNT, WAVES};
    const WideGrid g = wide_grid(sh, EPI, a.M, n_tiles, a.nkt, part ? part_bytes : 0);
    const int grid = (g.n_cols * g.k_splits + 7) / 8 * 8 * g.m_blocks;
    // one row block (only the narrow shape has that few rows): every weight byte is read once
    const bool stream = (WNT == 2) && g.m_blocks == 1;
    if constexpr (EPI == EPI_RESID) {
        if (g.k_splits > 1) {
            if (stream)
                hipLaunchKernelGGL((wide_gemm_kernel<EPI, true, BMT, WNT, WAVES, WNT == 2>), dim3(grid), dim3(WAVES * 64), 0, s, a, layout_nt, n_tiles,
                                   g.n_cols, g.m_blocks, g.k_splits, part);
            else
                hipLaunchKernelGGL((wide_gemm_kernel<EPI, true, BMT, WNT, WAVES, false>), dim3(grid), dim3(WAVES * 64), 0, s, a, layout_nt, n_tiles,
                                   g.n_cols, g.m_blocks, g.k_splits, part);
            return launch_fixup<WNT>(a, g.n_cols * WAVES * WNT, g.k_splits, part, s);
        }
    }
    if (stream)
        hipLaunchKernelGGL((wide_gemm_kernel<EPI, false, BMT, WNT, WAVES, WNT == 2>), dim3(grid), dim3(WAVES * 64), 0, s, a, layout_nt, n_tiles, g.n_cols,
                           g.m_blocks, 1, nullptr);
    else
        hipLaunchKernelGGL((wide_gemm_kernel<EPI, false, BMT, WNT, WAVES, false>), dim3(grid), dim3(WAVES * 64), 0, s, a, layout_nt, n_tiles, g.n_cols,
                           g.m_blocks, 1, nullptr);
    return hipGetLastError();
}

// 256-row blocks of 256 or 192 features, both operands through LDS (block_gemm_kernel): 2 x 4 waves of 8 x 4 accumulator tiles, or
// 4 x 2 waves of 4 x 6.
template <int EPI, int WM, int WN, int MT, int NT>
static hipError_t launch_block(int layout_nt, int n_tiles, const GemmArgs& a, hipStream_t s) {
    constexpr int BNT = WN * NT;
    const int n_cols = (n_tiles + BNT - 1) / BNT, m_blocks = (a.M + 255) / 256;
    const int grid = (n_cols + 7) / 8 * 8 * m_blocks;
    hipLaunchKernelGGL((block_gemm_kernel<EPI, false, WM, WN, MT, NT, 4>), dim3(grid), dim3(WM * WN * 64), 0, s, a, layout_nt, n_tiles, n_cols, m_blocks, 1,
                       nullptr);
    return hipGetLastError();
}

// Which many-row kernel takes a projection: 0 = the 128-row kernel, 16 / 12 = the 256-row kernel with blocks of 16 / 12 feature
// tiles.  The 256-row block needs two thirds of the 128-row blocks' operand bytes per flop (a compute unit draws about 50 GB/s in
// either kernel; a fifth of the requests go beyond the XCD's L2 and a request takes 400 cycles and more on average), but the
// compute units take its blocks one at a time, so a launch costs whole rounds of blocks and what counts is how many of the 256
// units its one round keeps busy: the width whose blocks number at most 256 and come closest to it (1024 rows x 12288 features:
// 192 blocks of 256 features or 256 blocks of 192).  It wins when that is most of the chip while the 128-row kernel would have to
// give some compute units a second pair of blocks (measured, 1024 rows: QKV 111 -> 97 us; 512 rows: gate/up 108 -> 92 us); with
// more than 256 blocks its second round costs more than it saves (1024 rows: gate/up 159 -> 187 us), with few blocks the 128-row
// kernel's finer grain fills more compute units (512 rows: QKV 66 -> 92 us).  The d_model-wide residual
// projections come by a rule of their own (launch_gemm_wide).
static int block_gemm_width(int mode, int epi, int M, int n_tiles) {  // mode 0 / 1 / 2: never / always 16 tiles / always 12 tiles (tuning knob)
    if (epi == EPI_RESID || mode == 0) return 0;
    if (mode == 1) return 16;
    if (mode == 2) return 12;
    const int m_blocks = (M + 255) / 256;
    const int b16 = (n_tiles + 15) / 16 * m_blocks, b12 = (n_tiles + 11) / 12 * m_blocks, blocks128 = (n_tiles + 15) / 16 * ((M + 127) / 128);
    if (blocks128 <= 256) return 0;
    if (b12 <= 256 && b12 >= 144) return 12;  // the narrower block has more blocks: closer to one per compute unit
    if (b16 <= 256 && b16 >= 144) return 16;
    return 0;
}

// K slices of a residual projection in 256-row blocks of 16 feature tiles, one round of them (32 blocks on an XCD's compute units) and at least 24
// k-tiles per slice; 0 if none is estimated below `other` us: 0.8 us per k-tile, 0.45 us a MiB of partial results to write and sum, 4 us.
static int block_slices(int n_cols, int M, int nkt, size_t part_bytes, double other) {
    const int m_blocks = (M + 255) / 256;
    const size_t per_split = (size_t)((M + 15) / 16) * n_cols * 16 * 1024;
    int best = 0;
    for (int k = 2; k <= 8 && (n_cols * k + 7) / 8 * m_blocks <= 32 && nkt / k >= 24 && per_split * k <= part_bytes; ++k) {
        const double us = 4 + per_split * k * 0.45e-6 + 0.8 * ((nkt + k - 1) / k);
        if (us < other) {
            other = us;
            best = k;
        }
    }
    return best;
}

// the kernels address weights and activations with 32-bit byte offsets from their bases
static bool wide_fits(int layout_nt, int n_tiles, int M, int nkt) {
    return (unsigned long long)(n_tiles + layout_nt) * nkt * 1024ull < (1ull << 32) && (unsigned long long)(M + 16) * nkt * 64ull < (1ull << 32);
}

hipError_t launch_gemm_wide(int epi, int layout_nt, int n_tiles, const GemmArgs& a, float* part, size_t part_bytes, int block_mode, hipStream_t s) {
    if (!a.x_frag || !wide_fits(layout_nt, n_tiles, a.M, a.nkt)) return hipErrorInvalidValue;
    const WideShape sh = wide_shape(epi, a.M);
    const bool narrow = sh.wnt == 2, half = sh.bmt == 4;
    const int bw = (!narrow && !half) ? block_gemm_width(block_mode, epi, a.M, n_tiles) : 0;
    if (bw == 16) {
        switch (epi) {
            case EPI_QKV: return launch_block<EPI_QKV, 2, 4, 8, 4>(layout_nt, n_tiles, a, s);
            case EPI_SWIGLU: return launch_block<EPI_SWIGLU, 2, 4, 8, 4>(layout_nt, n_tiles, a, s);
            case EPI_LOGITS: return launch_block<EPI_LOGITS, 2, 4, 8, 4>(layout_nt, n_tiles, a, s);
        }
    } else if (bw == 12) {
        switch (epi) {
            case EPI_QKV: return launch_block<EPI_QKV, 4, 2, 4, 6>(layout_nt, n_tiles, a, s);
            case EPI_SWIGLU: return launch_block<EPI_SWIGLU, 4, 2, 4, 6>(layout_nt, n_tiles, a, s);
            case EPI_LOGITS: return launch_block<EPI_LOGITS, 4, 2, 4, 6>(layout_nt, n_tiles, a, s);
        }
    }
    if (epi == EPI_RESID && !narrow && part && block_mode != 0) {
        // 256-row blocks where their estimate is 3 % below the 128-row kernel's: with up to 216 of its blocks 6 to 20 % faster in all of 30 launches
        // (us, 128-row blocks -> 256-row blocks: 5120 x 5120, 1024 rows 91.0 -> 75.8; 14336 x 4096, 700 rows 114 -> 97.5; 16384 x 6144, 512 rows
        // 137 -> 109).  217 to 256 blocks, nearly every compute unit at once, take up to 18 % more than estimated behind a long K: up to 2 % above it
        // the 256-row blocks are still 2 to 11 % faster in all of 26 (22016 x 8192, 900 rows 364 -> 332, estimates 311 and 306; 14336 x 4096, 960 rows
        // 132 -> 121; from 2 to 4 % above 0.95 .. 1.02, further up mostly slower).  Two rounds of short slices overlap, which the estimate does not
        // know: 4608 x 4608 in slices of 36 k-tiles, 769 rows 58.2 / 59.9, 850 rows 60.7 / 62.6; of 100 and more 11 % faster to 1 %
        // (12288 x 4608, 1024 rows 138.6 -> 131.3).  A short K, or a second round on some XCD, is worse: 2048 x 2048, 512 rows 21.9 / 32.1;
        // 18944 x 3584, 850 rows 128.8 / 137.5.
        const WideGrid g = wide_grid(sh, epi, a.M, n_tiles, a.nkt, part_bytes);
        const int blocks = g.n_cols * g.k_splits * g.m_blocks;
        const bool full = blocks > 216 && blocks <= 256, overlap = blocks > 256 && a.nkt / g.k_splits < 64;
        const int ks = block_slices(g.n_cols, a.M, a.nkt, part_bytes, block_mode > 0 ? 1e30 : overlap ? 0 : g.us * (full ? 1.02 : 0.97));
        if (ks > 1) {
            const int m_blocks = (a.M + 255) / 256, grid = (g.n_cols * ks + 7) / 8 * 8 * m_blocks;
            hipLaunchKernelGGL((block_gemm_kernel<EPI_RESID, true, 2, 4, 8, 4, 4>), dim3(grid), dim3(512), 0, s, a, layout_nt, n_tiles, g.n_cols, m_blocks, ks,
                               part);
            return launch_fixup<4>(a, g.n_cols * 16, ks, part, s);
        }
    }
    switch (epi) {
        case EPI_QKV:
            return narrow ? launch_wide_shape<EPI_QKV, 8, 2, 4>(layout_nt, n_tiles, a, part, part_bytes, s)
                          : launch_wide_shape<EPI_QKV, 8, 4, 4>(layout_nt, n_tiles, a, part, part_bytes, s);
        case EPI_SWIGLU:
            if (half) return launch_wide_shape<EPI_SWIGLU, 4, 2, 4>(layout_nt, n_tiles, a, part, part_bytes, s);
            return narrow ? launch_wide_shape<EPI_SWIGLU, 8, 2, 4>(layout_nt, n_tiles, a, part, part_bytes, s)
                          : launch_wide_shape<EPI_SWIGLU, 8, 4, 4>(layout_nt, n_tiles, a, part, part_bytes, s);
        case EPI_RESID:
            return narrow ? launch_wide_shape<EPI_RESID, 8, 2, 4>(layout_nt, n_tiles, a, part, part_bytes, s)
                          : launch_wide_shape<EPI_RESID, 8, 4, 4>(layout_nt, n_tiles, a, part, part_bytes, s);
        case EPI_LOGITS:
            if (half) return launch_wide_shape<EPI_LOGITS, 4, 2, 4>(layout_nt, n_tiles, a, part, part_bytes, s);
            return narrow ? launch_wide_shape<EPI_LOGITS, 8, 2, 4>(layout_nt, n_tiles, a, part, part_bytes, s)
                          : launch_wide_shape<EPI_LOGITS, 8, 4, 4>(layout_nt, n_tiles, a, part, part_bytes, s);
    }
    return hipErrorInvalidValue;
}

// ---- launch of the 17 to 128 row kernel -----------------------------------------------------------------------------------
template <int EPI, int WM, int WN, int KG, int MT, int NT, int R>
static hipError_t launch_stream_shape(int layout_nt, int n_tiles, const GemmArgs& a, float* part, size_t part_bytes, hipStream_t s) {
    constexpr int BNT = WN * NT, S = KG;
    const int n_cols = (n_tiles + BNT - 1) / BNT, m_tiles = (a.M + 15) / 16;
    const int flags = a.x_frag | (layout_nt == 4 ? 4 : layout_nt == 2 ? 2 : 0);
    const dim3 block(WM * WN * KG * 64);
    if constexpr (EPI == EPI_RESID) {  // K slices until there is about one workgroup per compute unit
        int ks = std::min(std::min(256 / n_cols, 8), a.nkt / 8);
        while (ks > 1 && (size_t)ks * m_tiles * n_cols * BNT * 1024 > part_bytes) --ks;
        if (ks > 1) {
            const int per = ((a.nkt + ks - 1) / ks + S - 1) / S * S;
            ks = (a.nkt + per - 1) / per;
            hipLaunchKernelGGL((stream_gemm_kernel<EPI, true, WM, WN, KG, MT, NT, R>), dim3(n_cols, ks), block, 0, s, a.Wp, a.X, a.nkt, a.ldx, a.M, flags,
                               n_tiles, per, a, part);
            return launch_stream_fixup(a, n_cols * BNT, ks, part, s);
        }
    }
    hipLaunchKernelGGL((stream_gemm_kernel<EPI, false, WM, WN, KG, MT, NT, R>), dim3(n_cols), block, 0, s, a.Wp, a.X, a.nkt, a.ldx, a.M, flags, n_tiles,
                       (a.nkt + S - 1) / S * S, a, nullptr);
    return hipGetLastError();
}

// Feature tiles per block: a compute unit holds one block at a time and draws its weights and the activations for it, so a launch
// costs rounds x (feature tiles + row tiles); the residual projections fill the chip with K slices instead, where wider blocks
// only pay by reading a long activation block less often (128 rows x 11008: 33.5 -> 31.2 us; 64 rows x 28672, 8192 features: 86.6 -> 84.3).
static int stream_width(int epi, int M, int n_tiles, int nkt) {
    const int bmt = M <= 64 ? 4 : 8;
    if (epi == EPI_RESID) return (M > 64 && nkt > 256) || (M > 32 && nkt > 512) ? 8 : 4;
    int best = 4, cost = 1 << 30;
    for (int bn = 4; bn <= 8; bn += 2) {
        const int blocks = (n_tiles + bn - 1) / bn, c = (blocks + 255) / 256 * (bn + bmt);
        if (c < cost) {
            cost = c;
            best = bn;
        }
    }
    return best;
}

// Which kernel takes a projection of 17 to 128 rows.  The streaming kernel's offsets from the operands' bases have 32 bits: matrices of
// 4 GiB and more stay with the few-row kernel.  Measured, us, the streaming kernel / the other one unless said otherwise:
//   * LM head: streaming while its blocks run in one round (32000 rows x 4096: 64 rows 50 / 49 + 5 for the conversion pass the other one
//     needs); with many rounds several workgroups per compute unit hide each other's ends (152064 x 3584, 64 rows: 242 / 220 + 5).
//     That other kernel, with blocks in registers, has one 64-row block per 128 features, a good launch if they all run at once or in
//     many rounds, not if a few compute units get a second one.  Few-row kernel then (blocks in registers / few-row) for 257 to 384
//     blocks up to 40 rows (33024 x 4096: 17 rows 74.7 / 60.9, 32 rows 75.6 / 67.3, 40 rows 2 % more, 48 rows 3 % less) and for 385 to
//     511 up to 24, with a short K up to 32 (50257 x 4096: 17 rows 85.7 / 84.6, 32 rows 85 / 93; x 1024: 17 rows 33.2 / 29.8, 32 rows
//     35.5 / 35.8; 61440 x 1024, 28 rows 38.2 / 36.3).
//   * QKV up to 64 rows: not of few heads (288 tiles, 72 blocks: 48 rows 23.4 / 21.6; from 65 rows on 80 rows 34 / 43), and up to 32 rows
//     not from about a round of blocks on (2016 tiles x 2048 29 / 27, 3264 tiles 48.7 / 42.8, x 5120 alike).
//   * gate/up up to 64 rows: streaming (2368 tiles, 48 rows 54.7 / 62.2) but where 64-row blocks in registers make a nearly full first or
//     second round (4096 tiles x 4096, 33 rows 91.6 / 88.9, x 2048 51.7 / 49.2; 1792 tiles x 4096, 32 rows 45.0 / 42.7, but 1728 x 5120 48.1 /
//     49.2); up to 32 rows the few-row kernel from a full round of blocks on (2048 tiles x 4096 50.5 / 46.7; 2368 tiles 53.4 / 52.4)
//     and with a short K (1728 tiles x 2048 27.8 / 26.6).
//   * QKV and gate/up from 65 rows on: the kernel with blocks in registers runs two of the same 128-feature blocks per compute unit and
//     wins where this one pays a whole further round for it (65 rows, gate/up of 3584 tiles x 4096 105 / 88, 4096 x 8192 215 / 174, QKV of
//     3072 x 5120 110 / 104), or has its first one nearly full (gate/up of 1728 tiles x 8192 97 / 91); not with few blocks in the second
//     round (gate/up x 4096, 65 rows: 2368 tiles 5 % less, 3072 tiles 3 % less).
//   * residual projections: the second launch that adds the K slices costs more than it gives while K is short: up to 32 rows to K 2048
//     (5120 .. 7168 features x 1024 9.6 .. 9.8 / 7.9 .. 8.7), to 4096 where the few-row kernel has at most one workgroup per compute unit or
//     a nearly full round of them (4096 x 4096 15 / 13; 8192 x 4096 18.9 / 17.1; but 5120 x 5120 with its 320 tiles 15.4 / 18.4, and
//     4096 x 11008 21.1 / 28); up to 64 rows to K 1024 (512 .. 8192 features: K 512 8.8 / 6.5 .. 11.2 / 9.8, K 1024 9.0 / 8.2 .. 11.8 / 11.0,
//     K 2048 10 % less).
static bool stream_fits(int n_tiles, int nkt) { return (unsigned long long)(n_tiles + 8) * nkt * 1024ull < (1ull << 32); }
MidKernel mid_kernel(int epi, int layout_nt, int M, int n_tiles, int nkt) {
    if (!stream_fits(n_tiles, nkt) || !wide_fits(layout_nt, n_tiles, M, nkt)) return MID_FEW;
    const int blocks = (n_tiles + 7) / 8;  // of 128 features
    switch (epi) {
        case EPI_LOGITS:
            if (M <= 64 && blocks <= 256) return MID_STREAM;
            return blocks > 256 && blocks < 512 && M <= (blocks <= 384 ? 40 : nkt <= 64 ? 32 : 24) ? MID_FEW : MID_WIDE;
        case EPI_RESID:
            if (M <= 32) return nkt <= 64 || (nkt <= 128 && (n_tiles <= 256 || n_tiles >= 448)) ? MID_FEW : MID_STREAM;
            return M <= 64 && nkt <= 32 ? MID_FEW : MID_STREAM;
        case EPI_QKV:
            if (M <= 64) return n_tiles < 512 || (M <= 32 && blocks >= 250) ? MID_FEW : MID_STREAM;
            break;
        case EPI_SWIGLU:
            if (M <= 32 && (blocks >= 256 || (blocks > 192 && nkt <= 64))) return MID_FEW;
            if (M <= 64) return (blocks > 464 && blocks <= 512) || (blocks >= 220 && blocks <= 256 && nkt <= 128) ? MID_WIDE : MID_STREAM;
            break;
    }
    // (the producers leave no sums of squares here: only the 128-feature blocks in registers, which work them out themselves)
    return M < wide_narrow_rows() && (blocks >= (epi == EPI_QKV ? 384 : 400) || (blocks > 192 && blocks <= 256)) ? MID_WIDE : MID_STREAM;
}

template <int EPI>
static hipError_t launch_stream_epi(int layout_nt, int n_tiles, const GemmArgs& a, float* part, size_t part_bytes, hipStream_t s) {
    const int bn = stream_width(EPI, a.M, n_tiles, a.nkt);
    if (a.M <= 32 && bn == 4) return launch_stream_shape<EPI, 1, 2, 2, 2, 2, 6>(layout_nt, n_tiles, a, part, part_bytes, s);
    if (a.M <= 64) {
        if (bn == 4) return launch_stream_shape<EPI, 2, 2, 2, 2, 2, 6>(layout_nt, n_tiles, a, part, part_bytes, s);
        if constexpr (EPI != EPI_RESID) {
            if (bn == 6) return launch_stream_shape<EPI, 2, 1, 2, 2, 6, 6>(layout_nt, n_tiles, a, part, part_bytes, s);
            return launch_stream_shape<EPI, 1, 2, 2, 4, 4, 6>(layout_nt, n_tiles, a, part, part_bytes, s);
        }
    }
    if constexpr (EPI != EPI_LOGITS) {
        if (bn == 4) return launch_stream_shape<EPI, 4, 1, 2, 2, 4, 6>(layout_nt, n_tiles, a, part, part_bytes, s);
        if constexpr (EPI != EPI_RESID) {
            if (bn == 6) return launch_stream_shape<EPI, 2, 1, 2, 4, 6, 4>(layout_nt, n_tiles, a, part, part_bytes, s);
        }
        return launch_stream_shape<EPI, 2, 2, 1, 4, 4, 8>(layout_nt, n_tiles, a, part, part_bytes, s);
    }
    return hipErrorInvalidValue;  // an LM head of more rows has another kernel
}

hipError_t launch_gemm_stream(int epi, int layout_nt, int n_tiles, const GemmArgs& a, float* part, size_t part_bytes, hipStream_t s) {
    if (!stream_fits(n_tiles, a.nkt) || a.M > 128) return hipErrorInvalidValue;
    switch (epi) {
        case EPI_QKV: return launch_stream_epi<EPI_QKV>(layout_nt, n_tiles, a, part, part_bytes, s);
        case EPI_RESID: return launch_stream_epi<EPI_RESID>(layout_nt, n_tiles, a, part, part_bytes, s);
        case EPI_SWIGLU: return launch_stream_epi<EPI_SWIGLU>(layout_nt, n_tiles, a, part, part_bytes, s);
        case EPI_LOGITS: return launch_stream_epi<EPI_LOGITS>(layout_nt, n_tiles, a, part, part_bytes, s);
    }
    return hipErrorInvalidValue;
}

// ---- 4-bit weights (W4A16) ------------------------------------------------------------------------
// w[n][k] = scale[n][k/128] * (code[n][k] - 8), codes 0..15, scales bf16 per 128-column group.  The stream from HBM
// is a quarter of the bf16 one, so the unpacking has to stay cheap:
//   * a lane's 16 bytes hold its 8 codes for each of the 4 k-tiles of one 128-column chunk; inside a dword the
//     nibbles are ordered so that ((d >> 4j) & 0x000F000F) | 0x43004300 is the bf16 pair (128 + code[2j], 128 +
//     code[2j+1]) — two integer instructions per pair, no conversion;
//   * the constant 128 + 8 is taken out by one extra MFMA per k-tile whose weight operand is the constant -136
//     (it adds -136 * sum_k x_k to every row, exactly what the offset contributes);
//   * the group's partial result is scaled once per chunk: acc += scale[n] * acc_chunk.
// RMSNorm: the gain cannot be folded into integer codes; a normed projection gets activations that already carry
// the gain, and the rows' sums of squares as partial sums left by the kernel that produced them.
template <int MT, int NT, int EPI, int SH>
__global__ void __launch_bounds__(512) skinny_gemm_w4_kernel(const GemmArgs a) {
    using T = bf16_t;
    using E = Elem<T>;
    using frag_t = E::frag_t;
    constexpr bool NORM = (EPI != EPI_RESID);
    constexpr int PF = 2;  // 128-column chunks of loads kept in flight per wave (4 was measured slower: qkv 14.5 -> 16.9 us at 16 rows)
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, NW = blockDim.x >> 6;
    const int r16 = lane & 15, g = lane >> 4;
    const int grp = blockIdx.x, mb = blockIdx.y;
    const int row0 = mb * MT * 16;
    const int nkc = a.nkt >> 2;                       // chunks of 4 k-tiles
    const int nsteps = (nkc - w + NW - 1) / NW;       // >= 1: the host never launches more waves than chunks
    // the workgroup's tiles: a whole group of the re-tiled weights, or half of one (SH: log2 of the tiles per group; a launch argument
    // in its place costs 0.2 - 0.3 us)
    constexpr int sh = SH;
    const int tile0 = grp * NT;
    const size_t first = (((size_t)(tile0 >> sh) * nkc) << sh) + (tile0 & ((1 << sh) - 1));
    const unsigned char* wbase = (const unsigned char*)a.Wp + first * 1024 + (size_t)lane * 16;
    const bf16_t* sbase = (const bf16_t*)a.Sp + first * 16 + g * 4;
    const T* xrow[MT];
    const size_t xstep = a.x_frag ? (size_t)64 * E::EPF : (size_t)E::KT;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        if (a.x_frag) {
            xrow[mt] = (const T*)a.X + (((size_t)(mb * MT + mt) * a.nkt) * 64 + lane) * E::EPF;
        } else {
            const int m = min(row0 + mt * 16 + r16, a.M - 1);
            xrow[mt] = (const T*)a.X + (size_t)m * a.ldx + g * E::EPF;
        }
    }

    const f32x4 resid_first = prefetch_resid<T, MT, NT, EPI>(a, w, grp, row0, r16, g);
    f32x4 acc[MT][NT];
    float ss[MT];
    constexpr int SSP_LOADS = 12;  // 8 waves x 4 lane groups x 12 = 384 partial sums: d_model up to 6144 without the tail loop
    float sp[MT][SSP_LOADS];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        ss[mt] = 0.f;
        if (NORM) {
            // This lane's share of the row's partial sums of squares; the cross-wave reduction adds the shares up.  The
            // loads go out together here (a loop of load-wait-add would put several memory round trips in front of the
            // first weight fetch); they are added up after the K loop.
            const int m = min(row0 + mt * 16 + r16, a.M - 1);
#pragma unroll
            for (int i = 0; i < SSP_LOADS; ++i) {
                const int j = w * 4 + g + i * 4 * NW;
                sp[mt][i] = j < a.ssp_n ? a.ssp_in[(size_t)j * a.ssp_stride + m] : 0.f;
            }
            for (int j = w * 4 + g + SSP_LOADS * 4 * NW; j < a.ssp_n; j += 4 * NW) ss[mt] += a.ssp_in[(size_t)j * a.ssp_stride + m];  // very wide models
        }
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    frag_t koff;
#pragma unroll
    for (int e = 0; e < 8; ++e) koff[e] = (bf16_t)(-136.0f);

    u32x4 cq[PF][NT];
    bf16x4 sq[PF][NT];
    frag_t xq[PF][4][MT];
    auto issue = [&](int s, int step) {
        const int c = w + min(step, nsteps - 1) * NW;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            cq[s][nt] = __builtin_nontemporal_load((const u32x4*)(wbase + (((size_t)c << sh) + nt) * 1024));
            sq[s][nt] = *(const bf16x4*)(sbase + (((size_t)c << sh) + nt) * 16);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) xq[s][q][mt] = *(const frag_t*)(xrow[mt] + (size_t)(c * 4 + q) * xstep);
        }
    };
    auto consume = [&](int s, int step) {
        const bool live = step < nsteps;
        f32x4 accg[MT][NT], acco[MT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            acco[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) accg[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            frag_t wf[NT];
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const unsigned d = cq[s][nt][q];
                unsigned pr[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) pr[j] = ((d >> (4 * j)) & 0x000F000Fu) | 0x43004300u;
                wf[nt] = __builtin_bit_cast(frag_t, u32x4{pr[0], pr[1], pr[2], pr[3]});
            }
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                const frag_t av = xq[s][q][mt];
                acco[mt] = E::mma(koff, av, acco[mt]);
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) accg[mt][nt] = E::mma(wf[nt], av, accg[mt][nt]);
            }
        }
        if (live) {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const float sc = (float)sq[s][nt][v];
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) acc[mt][nt][v] += sc * (accg[mt][nt][v] + acco[mt][v]);
                }
        }
    };
#pragma unroll
    for (int s = 0; s < PF; ++s) issue(s, s);
    const int nrounds = (nsteps + PF - 1) / PF;
    for (int rd = 0; rd + 1 < nrounds; ++rd) {
#pragma unroll
        for (int s = 0; s < PF; ++s) {
            consume(s, rd * PF + s);
            issue(s, (rd + 1) * PF + s);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int s = 0; s < PF; ++s) consume(s, (nrounds - 1) * PF + s);

    if (NORM) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int i = 0; i < SSP_LOADS; ++i) ss[mt] += sp[mt][i];
    }
    reduce_and_store<T, MT, NT, EPI>(a, acc, ss, smem, lane, w, NW, grp, row0, resid_first);
}

template <int MT, int NT, int EPI, int SH>
static hipError_t launch_one_w4(int NW, int n_groups, const GemmArgs& a0, hipStream_t s) {
    GemmArgs a = a0;
    const int mblocks = (a.M + MT * 16 - 1) / (MT * 16);
    a.red_copies = reduction_copies(NW, MT, NT);
    const size_t lds = (size_t)a.red_copies * MT * NT * 1024 + (size_t)NW * MT * 16 * sizeof(float);
    hipLaunchKernelGGL((skinny_gemm_w4_kernel<MT, NT, EPI, SH>), dim3(n_groups, mblocks), dim3(NW * 64), lds, s, a);
    return hipGetLastError();
}

template <int EPI>
static hipError_t launch_mt_nt_w4(int MT, int NT, bool half, int NW, int n_groups, const GemmArgs& a, hipStream_t s) {
    constexpr bool PAIR = (EPI == EPI_QKV || EPI == EPI_SWIGLU);
    if (half) return launch_one_w4<1, 2, EPI, 2>(NW, n_groups, a, s);
#define FS_CASE(mt, nt, sh) \
    if (MT == mt && NT == nt) return launch_one_w4<mt, nt, EPI, sh>(NW, n_groups, a, s);
    if constexpr (!PAIR) {
        FS_CASE(1, 1, 0) FS_CASE(2, 1, 0)
    }
    FS_CASE(1, 2, 1) FS_CASE(2, 2, 1) FS_CASE(1, 4, 2) FS_CASE(2, 4, 2)
#undef FS_CASE
    return hipErrorInvalidValue;
}

// ---- 4-bit weights, many rows (prompt chunks, stacked requests) ------------------------------------------------------------
// The few-row kernel above unpacks its weights again for every 32 rows and reads the activations once per workgroup of 32 or 64
// features: at a few hundred rows it is bound by both (13B layer, 389 rows: 1048 us, now 395).  Here a workgroup of WM x WN waves owns
// 16 * WM * MT rows x 16 * WN * NT features; a stage is one 128-column chunk: the rows' fragments of its four k-tiles, the feature
// tiles' codes (a KiB each) and scales, all by direct-to-LDS loads, R buffers.  A wave unpacks its NT code tiles once per chunk
// into 16 operand registers each (2 VALU operations per pair of weights) and multiplies them with MT row tiles; the chunk's products start
// at -136 * sum of the activations, which the waves work out for one row tile each, a stage ahead, and share through LDS (each for its own
// row tiles, added behind the products, before: 389 rows x 27648 features x 5120 188 -> 182 us), and enter the accumulators times the
// scale.  Per chunk and wave of 4 x 4 tiles: 68 MFMAs (64 of them products), about 200 VALU operations, 24 KB of LDS reads.  A 128 x 256
// block takes 2.2 us per chunk; 1.3 its MFMAs alone, 1.1 its loads alone, 1.9 everything but the loads, and none of the LDS reads, the
// unpacking or the scaling more than 0.15 when it is left out (1024 rows x 27648 features x 5120: 0.8 PFLOP/s).  Same arithmetic as the
// few-row kernel: exact codes, f32 sums per chunk, f32 scaling.
template <int EPI, bool PARTIAL, int WM, int WN, int MT, int NT, int R>
__global__ void __launch_bounds__(WM * WN * 64) block_gemm_w4_kernel(const void* Wp, const void* X, const void* Sp, int nkc, int M, int lsh, int n_tiles,
                                                                     int kc_per, int bt, const GemmArgs a, float* part) {
    using T = bf16_t;
    using E = Elem<T>;
    using frag_t = E::frag_t;
    constexpr bool NORM = (EPI != EPI_RESID);
    constexpr int NW = WM * WN, BMT = WM * MT, BNT = WN * NT, ROWS = BMT * 16, THREADS = NW * 64;
    constexpr int AF = 4 * BMT, LA = AF / NW, LW = BNT / NW, LPS = LA + LW + 1;
    constexpr int SCALES = (AF + BNT) * 1024, STAGE = SCALES + NW * 256;
    static_assert(AF % NW == 0 && BNT % NW == 0 && BMT <= NW, "every wave issues the same loads");
    static_assert((R == 3 || R == 4) && LPS * (R - 1) < 64 && R * STAGE + ROWS * 12 <= 160 * 1024, "6-bit wait counter, 160 KiB of LDS");
    static_assert(NT <= 8 && THREADS % ROWS == 0, "a wave's scales fit one load; whole rows per pass of the row-scale sums");
    __shared__ __align__(1024) unsigned char sb0[STAGE];
    __shared__ __align__(1024) unsigned char sb1[STAGE];
    __shared__ __align__(1024) unsigned char sb2[STAGE];
    __shared__ __align__(1024) unsigned char sb3[R > 3 ? STAGE : 16];
    __shared__ float rs_s[ROWS];
    __shared__ float off_s[2][ROWS];
    auto buf_at = [&](int j) -> unsigned char* { return j == 0 ? sb0 : (j == 1 ? sb1 : (j == 2 ? sb2 : sb3)); };

    // grid (8 * row blocks, units / 8), unit = (K slice, feature block): an XCD takes neighbouring units, most of one slice, and all their
    // row blocks, and no XCD more than its share (slices of 20 feature blocks padded to 24 instead left half the XCDs with 36 blocks for
    // 32 compute units: 389 rows, 13824 x 5120 163 -> 93 us, 5120 x 5120 70 -> 48)
    const int n_cols = (n_tiles + BNT - 1) / BNT, units = PARTIAL ? n_cols * ((nkc + kc_per - 1) / kc_per) : n_cols;
    const int xcd = blockIdx.x & 7, unit = (units * xcd >> 3) + (int)blockIdx.y;
    const int mb = blockIdx.x >> 3, ks = unit / n_cols, col = unit - ks * n_cols;
    if (unit >= units * (xcd + 1) >> 3) return;
    const int t = threadIdx.x, lane = t & 63;
    const int w = __builtin_amdgcn_readfirstlane(t >> 6), wm = w / WN, wn = w % WN;
    const int r16 = lane & 15, g = lane >> 4;
    const int kc_lo = ks * kc_per, ns = min(kc_per, nkc - kc_lo);  // >= 1 (host)
    const int mt0 = mb * bt, m_tiles = (M + 15) >> 4;
    // the block's bt row tiles (at most BMT), half of them for each row of waves: a block of 7 rather than 8 row tiles (389 rows in four
    // blocks) 182 -> 173 us, of 5 (140 rows in two) 91 -> 63
    const int tb = wm * (bt - bt / 2), my = WM == 1 ? bt : wm ? bt / 2 : bt - bt / 2;
    static_assert(WM <= 2, "");

    // RMSNorm: this thread's share of its row's partial sums of squares (the loads go out in front of the ring's)
    constexpr int TPR = THREADS / ROWS, SL = 8;
    float sp[SL], s_more = 0.f;
    const int row = t % ROWS, sub = t / ROWS;
    if (NORM) {
        const int m = min(mt0 * 16 + row, M - 1);
#pragma unroll
        for (int i = 0; i < SL; ++i) sp[i] = a.ssp_in[(size_t)min(sub + i * TPR, a.ssp_n - 1) * a.ssp_stride + m];
#pragma unroll 8
        for (int j = sub + SL * TPR; j < a.ssp_n; j += TPR) s_more += a.ssp_in[(size_t)j * a.ssp_stride + m];
    }

    // this wave's loads of a stage: fragments i * NW + w of the activations (k-tile, row tile), code tiles i * NW + w, its own scales
    const unsigned char* const xb = (const unsigned char*)X;
    const unsigned char* const wb = (const unsigned char*)Wp;
    const unsigned char* const sb = (const unsigned char*)Sp;
    const unsigned wkc = 1024u << lsh, skc = 32u << lsh;  // bytes from one chunk to the next
    unsigned xo[LA], wo[LW], so;
#pragma unroll
    for (int i = 0; i < LA; ++i) {
        const int f = i * NW + w, mt = min(mt0 + min(f % BMT, bt - 1), m_tiles - 1);
        xo[i] = ((unsigned)mt * (unsigned)nkc * 4u + (unsigned)kc_lo * 4u + (unsigned)(f / BMT)) * 1024u + (unsigned)lane * 16u;
    }
#pragma unroll
    for (int i = 0; i < LW; ++i) {
        const int pc = min(col * BNT + i * NW + w, n_tiles - 1);
        wo[i] = ((((unsigned)(pc >> lsh) * (unsigned)nkc + (unsigned)kc_lo) << lsh) + (unsigned)(pc & ((1 << lsh) - 1))) * 1024u + (unsigned)lane * 16u;
    }
    {  // 4 bytes per lane: lane = (tile of the wave, pair of rows); lanes beyond the wave's tiles repeat its last one
        const int pc = min(col * BNT + wn * NT + min(lane >> 3, NT - 1), n_tiles - 1);
        so = ((((unsigned)(pc >> lsh) * (unsigned)nkc + (unsigned)kc_lo) << lsh) + (unsigned)(pc & ((1 << lsh) - 1))) * 32u + (unsigned)(lane & 7) * 4u;
    }
    const unsigned lane16 = (unsigned)lane * 16u;
    int st = 0;
    auto issue = [&](int j) {  // next stage -> buffer j; stages beyond the range fetch the operands' first line (no branch around a load)
        unsigned char* dst = buf_at(j);
        const unsigned live = (unsigned)((st - ns) >> 31);  // uniform, all ones or zero
#pragma unroll
        for (int i = 0; i < LA; ++i) {
            __builtin_amdgcn_global_load_lds(FS_GLB_PTR(xb + (xo[i] & live)), FS_LDS_PTR(dst + (i * NW + w) * 1024), 16, 0, 0);
            xo[i] += 4096u;
        }
#pragma unroll
        for (int i = 0; i < LW; ++i) {
            __builtin_amdgcn_global_load_lds(FS_GLB_PTR(wb + (wo[i] & live)), FS_LDS_PTR(dst + (AF + i * NW + w) * 1024), 16, 0, 0);
            wo[i] += wkc;
        }
        __builtin_amdgcn_global_load_lds(FS_GLB_PTR(sb + (so & live)), FS_LDS_PTR(dst + SCALES + w * 256), 4, 0, 0);
        so += skc;
        ++st;
    };
    f32x4 acc[MT][NT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
    frag_t koff;
#pragma unroll
    for (int e = 0; e < 8; ++e) koff[e] = (bf16_t)(-136.0f);
    const f32x4 zero{0.f, 0.f, 0.f, 0.f};
    // mask and exponent of the unpacking, one in a scalar and one in a vector register: a single and-or instruction takes both
    unsigned nib = 0x000F000Fu, one28 = 0x43004300u;
    asm volatile("" : "+s"(nib));
    asm volatile("" : "+v"(one28));
    const bool works = (mt0 + tb) * 16 < M;  // uniform: a wave whose rows all lie beyond the matrix only loads

#pragma unroll
    for (int j = 0; j + 1 < R; ++j) issue(j);
    if (NORM) {  // partial row sums meet in rs_s (one thread per row and pass of the loop below)
        float tot = s_more;
#pragma unroll
        for (int i = 0; i < SL; ++i) tot += sub + i * TPR < a.ssp_n ? sp[i] : 0.f;
        for (int k = 0; k < TPR; ++k) {  // uniform; TPR is 8 (64-row blocks) or 4
            if (sub == k) rs_s[row] = k == 0 ? tot : rs_s[row] + tot;
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
        }
    }
    // -136 * sum of the activations, per row, of the chunk in buffer j: a row tile per wave, for everybody
    auto offsets = [&](int j, int set) {
        if (BMT < NW && w >= BMT) return;
        const unsigned char* b = buf_at(j);
        f32x4 o = zero;
#pragma unroll
        for (int q = 0; q < 4; ++q) o = E::mma(koff, *(const frag_t*)(b + (q * BMT + w) * 1024 + lane16), o);
        if (g == 0) off_s[set][w * 16 + r16] = o[0];
    };
    asm volatile("" ::: "memory");
    FS_WAIT_VM_LGKM((R - 2) * LPS, 0);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    offsets(0, 0);
    int par = 0;
    auto run = [&](auto tiles) {  // tiles: the wave's row tiles
        constexpr int MX = decltype(tiles)::value;
        auto stage = [&](int ju) {  // the next stage, in buffer ju
            asm volatile("" ::: "memory");
            FS_WAIT_VM_LGKM((R - 3) * LPS, 0);
            __builtin_amdgcn_s_barrier();  // the stage behind this one is complete for every wave, and everybody is done with the one before
            asm volatile("" ::: "memory");
            issue((ju + R - 1) % R);
            const int set = par;
            par ^= 1;
            if (!works) return offsets((ju + 1) % R, par);
            const unsigned char* b = buf_at(ju);
            u32x4 c[NT];
            bf16x4 s4[NT];
            frag_t wf[2][NT], x[2][MX];
            f32x4 tq[MX][NT];
            auto unpack = [&](int set, int q) {
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    unsigned pr[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) pr[j] = ((c[nt][q] >> (4 * j)) & nib) | one28;
                    wf[set][nt] = __builtin_bit_cast(frag_t, u32x4{pr[0], pr[1], pr[2], pr[3]});
                }
            };
            auto read_x = [&](int set, int q) {
#pragma unroll
                for (int mt = 0; mt < MX; ++mt) x[set][mt] = *(const frag_t*)(b + (q * BMT + tb + mt) * 1024 + lane16);
            };
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) c[nt] = *(const u32x4*)(b + (AF + wn * NT + nt) * 1024 + lane16);
            read_x(0, 0);
            float off[MX];
#pragma unroll
            for (int mt = 0; mt < MX; ++mt) off[mt] = off_s[set][(tb + mt) * 16 + r16];
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) s4[nt] = *(const bf16x4*)(b + SCALES + w * 256 + nt * 32 + g * 8);
            unpack(0, 0);
            // k-tile by k-tile: the next one's operands are read and unpacked while this one's MFMAs run; the products start at the offsets
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int cu = q & 1, nx = cu ^ 1;
                if (q < 3) {
                    read_x(nx, q + 1);
                    unpack(nx, q + 1);
                }
#pragma unroll
                for (int mt = 0; mt < MX; ++mt) {
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) tq[mt][nt] = E::mma(wf[cu][nt], x[cu][mt], q ? tq[mt][nt] : f32x4{off[mt], off[mt], off[mt], off[mt]});
                }
                if (q < 3) {
                    __builtin_amdgcn_sched_group_barrier(0x100, MX, 0);  // the next k-tile's LDS reads first
#pragma unroll
                    for (int k = 0; k < MX * NT; ++k) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                                  // one MFMA
                        __builtin_amdgcn_sched_group_barrier(0x002, (7 * NT + MX * NT - 1) / (MX * NT), 0);  // its share of the unpacking
                    }
                }
            }
            offsets((ju + 1) % R, par);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const float sc = (float)s4[nt][v];
#pragma unroll
                    for (int mt = 0; mt < MX; ++mt) acc[mt][nt][v] += sc * tq[mt][nt][v];
                }
        };
        int s0 = 0;
        for (; s0 + R <= ns; s0 += R) {
#pragma unroll
            for (int ju = 0; ju < R; ++ju) stage(ju);
        }
#pragma unroll
        for (int ju = 0; ju < R; ++ju) {
            if (s0 + ju >= ns) break;
            stage(ju);
        }
    };
    if (my == MT)
        run(std::integral_constant<int, MT>());
    else
        run(std::integral_constant<int, MT - 1>());
    // every load has landed and every wave has left the loop before LDS is reused or given back
    FS_WAIT_VM_LGKM(0, 0);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");

    const int pt0 = col * BNT + wn * NT;
    if constexpr (PARTIAL) {  // raw tiles: part[ks][m tile][n tile][lane]
        const int nt_all = n_cols * BNT;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            const int mtile = mt0 + tb + mt;
            if (mt >= my || mtile >= m_tiles) break;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) ((f32x4*)part)[(((size_t)ks * m_tiles + mtile) * nt_all + pt0 + nt) * 64 + lane] = acc[mt][nt];
        }
        return;
    }
    float* hs = (float*)sb0;  // residual projections: [WN feature waves][ROWS] sums of squares
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        if (mt >= my) break;
        const int lr = (tb + mt) * 16 + r16, m = mt0 * 16 + lr;
        const float rs = NORM ? 1.0f / sqrtf(rs_s[lr] / (float)a.K + a.eps) : 1.f;
        float hsq = epilogue_row<EPI, NT>(a, acc[mt], rs, m, pt0, g);
        if constexpr (EPI == EPI_RESID) {
            hsq = wave_xor_add(wave_xor_add(hsq, 16), 32);
            if (g == 0) hs[wn * ROWS + lr] = hsq;
        }
    }
    if constexpr (EPI == EPI_RESID) {
        if (a.ssp_out) {
            __syncthreads();
            for (int r = t; r < bt * 16; r += THREADS) {
                float sum = 0.f;
#pragma unroll
                for (int k = 0; k < WN; ++k) sum += hs[k * ROWS + r];
                if (mt0 * 16 + r < a.ssp_stride) a.ssp_out[(size_t)col * a.ssp_stride + mt0 * 16 + r] = sum;
            }
        }
    }
}

// ---- 4-bit weights, up to 64 rows: one pass over the codes, both operands through LDS --------------------------------------
// At these row counts a workgroup of the few-row kernel above reads the whole activation block from L2 for its two or four feature
// tiles, a larger operand than its codes (24 rows x 5120: 320 KiB against 170), in loads that are each waited for after two
// 128-column chunks.  Here a block of WN * NT feature tiles and all rows goes through a ring of R direct-to-LDS stages, as in the dense
// streaming kernel: KG wave groups take alternate chunks (the waves of a SIMD then unpack and multiply in turn), a stage is the
// activations of KG chunks, the blocks' codes (a KiB per tile and chunk) and, per wave, the scales of its own tiles.
//   * -136 * sum of the activations (the codes' offset) is formed first and is where the products' accumulators start; the chunk's
//     result enters the sums times the scale.  f32 sums per chunk and f32 scaling as in the kernels beside it.
//   * RMSNorm: a row's partial sums of squares are spread over the workgroup's threads in front of the ring's first load.
//   * The groups' tiles meet in LDS; the items of the epilogue are dealt to the groups.  Residual projections are cut along K and
//     summed by stream_fixup_kernel.
// 5120-wide layer, 24 rows, before -> now, us: QKV 22.3 -> 18.5, output 14.7 -> 13.0, gate/up 32.2 -> 25.5, down 24.7 -> 18.4.  Gate/up without
// unpacking and products takes 20.1: a compute unit draws 36 GB/s of codes and activations together.  What is above that is left over with
// fragments read a stage ahead, with groups half a chunk apart and with raised wave priorities alike.
template <int EPI, int WN, int KG, int MT, int NT, int R>
__global__ void __launch_bounds__(WN * KG * 64) stream_gemm_w4_kernel(const void* Wp, const void* X, const void* Sp, int nkc, int M, int lsh, int n_tiles,
                                                                      int kc_per, const GemmArgs a, float* part) {
    using T = bf16_t;
    using E = Elem<T>;
    using frag_t = E::frag_t;
    constexpr bool NORM = (EPI != EPI_RESID);
    constexpr bool PAIR = (EPI == EPI_QKV || EPI == EPI_SWIGLU);
    constexpr int TPI = PAIR ? 2 : 1;
    constexpr int NW = WN * KG, BNT = WN * NT, ROWS = MT * 16, THREADS = NW * 64;
    constexpr int AF = KG * 4 * MT, WF = KG * BNT, LA = AF / NW, LW = WF / NW, LPS = LA + LW + 1;
    constexpr int SCALES = (AF + WF) * 1024, STAGE = SCALES + NW * 256;
    constexpr int ITEMS = MT * NT / TPI;
    static_assert(AF % NW == 0 && WF % NW == 0 && KG > 1 && NT % TPI == 0 && NT <= 8, "every wave issues the same loads; its scales fit one of them");
    static_assert(R >= 3 && R <= 6 && LPS * (R - 1) < 64 && R * STAGE + NW * ROWS * 4 <= 160 * 1024, "6-bit wait counter, 160 KiB of LDS");
    static_assert((NW + 1) / 2 * MT * NT * 1024 <= STAGE, "the groups' tiles fit two stage buffers");
    // one array per buffer: distinct objects, see block_gemm_kernel
    __shared__ __align__(1024) unsigned char sb0[STAGE];
    __shared__ __align__(1024) unsigned char sb1[STAGE];
    __shared__ __align__(1024) unsigned char sb2[STAGE];
    __shared__ __align__(1024) unsigned char sb3[R > 3 ? STAGE : 16];
    __shared__ __align__(1024) unsigned char sb4[R > 4 ? STAGE : 16];
    __shared__ __align__(1024) unsigned char sb5[R > 5 ? STAGE : 16];
    __shared__ float rs_s[NORM ? NW * ROWS : 1];
    auto buf_at = [&](int j) -> unsigned char* { return j == 0 ? sb0 : (j == 1 ? sb1 : (j == 2 ? sb2 : (j == 3 ? sb3 : (j == 4 ? sb4 : sb5)))); };

    // grid (feature block, K slice); all rows are in one block
    const int col = blockIdx.x, ks = blockIdx.y;
    const int t = threadIdx.x, lane = t & 63;
    const int w = __builtin_amdgcn_readfirstlane(t >> 6), kg = w / WN, wn = w % WN;
    const int r16 = lane & 15, g = lane >> 4;
    const int kc_lo = ks * kc_per, n = min(kc_per, nkc - kc_lo);  // >= 1 (host)
    const int ns = (n + KG - 1) / KG;
    const int m_tiles = (M + 15) >> 4;

    // RMSNorm: this lane's share of its row's partial sums of squares (the loads go out in front of the ring's)
    constexpr int TPR = THREADS / ROWS, SL = MT == 1 ? 12 : 20;
    // (TPR * SL partial sums without the loop below, which waits: 384 up to 16 rows, 320 up to 32, 160 or 80 up to 64)
    float sp[SL], s_more = 0.f;
    const int row = t % ROWS, sub = t / ROWS;
    if (NORM) {
        const int m = min(row, M - 1);
#pragma unroll
        for (int i = 0; i < SL; ++i) sp[i] = a.ssp_in[(size_t)min(sub + i * TPR, a.ssp_n - 1) * a.ssp_stride + m];
#pragma unroll 8
        for (int j = sub + SL * TPR; j < a.ssp_n; j += TPR) s_more += a.ssp_in[(size_t)j * a.ssp_stride + m];
    }

    // this wave's loads of a stage: fragments i * NW + w of the activations (chunk, k-tile, row tile), code tiles i * NW + w (chunk, feature
    // tile), the scales of its own tiles.  A 32-bit offset per lane and load; tiles and rows beyond the matrix re-read the last one
    const unsigned char* const xb = (const unsigned char*)X;
    const unsigned char* const wb = (const unsigned char*)Wp;
    const unsigned char* const sb = (const unsigned char*)Sp;
    const unsigned wkc = 1024u << lsh, skc = 32u << lsh;  // bytes from one chunk to the next
    unsigned xo[LA], wo[LW], so;
    int xn[LA], wn_[LW];  // stages in which the load's chunk exists
#pragma unroll
    for (int i = 0; i < LA; ++i) {
        const int f = i * NW + w, j = f / (4 * MT), mt = min(f % MT, m_tiles - 1);
        xo[i] = ((unsigned)mt * (unsigned)nkc * 4u + (unsigned)(kc_lo + j) * 4u + (unsigned)(f / MT % 4)) * 1024u + (unsigned)(lane - r16 + min(r16, M - 1 - mt * 16)) * 16u;
        xn[i] = (n - j + KG - 1) / KG;
    }
#pragma unroll
    for (int i = 0; i < LW; ++i) {
        const int f = i * NW + w, j = f / BNT, pc = min(col * BNT + f % BNT, n_tiles - 1);
        wo[i] = ((((unsigned)(pc >> lsh) * (unsigned)nkc + (unsigned)(kc_lo + j)) << lsh) + (unsigned)(pc & ((1 << lsh) - 1))) * 1024u + (unsigned)lane * 16u;
        wn_[i] = (n - j + KG - 1) / KG;
    }
    const int sn = (n - kg + KG - 1) / KG;
    {  // 4 bytes per lane: lane = (tile of the wave, pair of rows); lanes beyond the wave's tiles repeat its last one
        const int pc = min(col * BNT + wn * NT + min(lane >> 3, NT - 1), n_tiles - 1);
        so = ((((unsigned)(pc >> lsh) * (unsigned)nkc + (unsigned)(kc_lo + kg)) << lsh) + (unsigned)(pc & ((1 << lsh) - 1))) * 32u + (unsigned)(lane & 7) * 4u;
    }
    const unsigned lane16 = (unsigned)lane * 16u;
    int st = 0;
    auto issue = [&](int j) {  // next stage -> buffer j; chunks beyond the range fetch the operands' first line (no branch around a load)
        unsigned char* dst = buf_at(j);
#pragma unroll
        for (int i = 0; i < LW; ++i) {
            const unsigned live = (unsigned)((st - wn_[i]) >> 31);  // uniform, all ones or zero
            __builtin_amdgcn_global_load_lds(FS_GLB_PTR(wb + (wo[i] & live)), FS_LDS_PTR(dst + (AF + i * NW + w) * 1024), 16, 0, 2);
            wo[i] += KG * wkc;
        }
        __builtin_amdgcn_global_load_lds(FS_GLB_PTR(sb + (so & (unsigned)((st - sn) >> 31))), FS_LDS_PTR(dst + SCALES + w * 256), 4, 0, 0);
        so += KG * skc;
#pragma unroll
        for (int i = 0; i < LA; ++i) {
            const unsigned live = (unsigned)((st - xn[i]) >> 31);
            __builtin_amdgcn_global_load_lds(FS_GLB_PTR(xb + (xo[i] & live)), FS_LDS_PTR(dst + (i * NW + w) * 1024), 16, 0, 0);
            xo[i] += KG * 4096u;
        }
        ++st;
    };
    f32x4 acc[MT][NT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
    frag_t koff;
#pragma unroll
    for (int e = 0; e < 8; ++e) koff[e] = (bf16_t)(-136.0f);
    // mask and exponent of the unpacking, one in a scalar and one in a vector register: a single and-or instruction takes both
    unsigned nib = 0x000F000Fu, one28 = 0x43004300u;
    asm volatile("" : "+s"(nib));
    asm volatile("" : "+v"(one28));

#pragma unroll
    for (int j = 0; j + 1 < R; ++j) issue(j);
    if (NORM) {  // a wave's share of every row's sum; the waves' shares are added up in the epilogue
        __builtin_amdgcn_sched_barrier(0);  // their first use stays behind the ring's loads
        float tot = s_more;
#pragma unroll
        for (int i = 0; i < SL; ++i) tot += sub + i * TPR < a.ssp_n ? sp[i] : 0.f;
#pragma unroll
        for (int sh = ROWS; sh < 64; sh *= 2) tot = wave_xor_add(tot, sh);
        if (lane < ROWS) rs_s[w * ROWS + lane] = tot;
    }
    int cur = 0;  // stage being multiplied
    auto stage = [&](int ju) {  // the next stage, in buffer ju
        asm volatile("" ::: "memory");
        FS_WAIT_VM_LGKM((R - 2) * LPS, 0);
        __builtin_amdgcn_s_barrier();  // the stage is complete for every wave, and everybody is done with the one before
        asm volatile("" ::: "memory");
        issue((ju + R - 1) % R);
        if (cur++ * KG + kg >= n) return;  // uniform; the last stage may hold fewer chunks
        const unsigned char* b = buf_at(ju);
        u32x4 c[NT];
        bf16x4 s4[NT];
        frag_t x[4][MT];
        f32x4 tq[MT][NT];
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) x[q][mt] = *(const frag_t*)(b + ((kg * 4 + q) * MT + mt) * 1024 + lane16);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) c[nt] = *(const u32x4*)(b + (AF + kg * BNT + wn * NT + nt) * 1024 + lane16);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) s4[nt] = *(const bf16x4*)(b + SCALES + w * 256 + nt * 32 + g * 8);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            f32x4 off{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int q = 0; q < 4; ++q) off = E::mma(koff, x[q][mt], off);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) tq[mt][nt] = off;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                unsigned pr[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) pr[j] = ((c[nt][q] >> (4 * j)) & nib) | one28;
                const frag_t wf = __builtin_bit_cast(frag_t, u32x4{pr[0], pr[1], pr[2], pr[3]});
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) tq[mt][nt] = E::mma(wf, x[q][mt], tq[mt][nt]);
            }
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const float sc = (float)s4[nt][v];
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) acc[mt][nt][v] += sc * tq[mt][nt][v];
            }
    };
    int s0 = 0;
    for (; s0 + R <= ns; s0 += R) {
#pragma unroll
        for (int ju = 0; ju < R; ++ju) stage(ju);
    }
#pragma unroll
    for (int ju = 0; ju < R; ++ju) {
        if (s0 + ju >= ns) break;
        stage(ju);
    }
    // every load has landed and every wave has left the loop before LDS is reused or given back
    FS_WAIT_VM_LGKM(0, 0);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");

    // ---- the groups' tiles meet in two stage buffers; item i belongs to group i % KG ----
    auto slot = [&](int ww) -> f32x4* { return (f32x4*)((ww & 1) ? sb1 : sb0) + (size_t)(ww >> 1) * MT * NT * 64 + lane; };
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) slot(w)[(mt * NT + nt) * 64] = acc[mt][nt];
    __syncthreads();
    const int pt0 = col * BNT + wn * NT;
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        if (it % KG != kg) continue;
        const int mt = it / (NT / TPI), ntp = it % (NT / TPI);
        if (mt >= m_tiles) break;
        f32x4 y4[TPI];
#pragma unroll
        for (int tt = 0; tt < TPI; ++tt) {
            const int nt = ntp * TPI + tt;
            y4[tt] = slot(wn)[(mt * NT + nt) * 64];
#pragma unroll
            for (int k = 1; k < KG; ++k) y4[tt] += slot(k * WN + wn)[(mt * NT + nt) * 64];
        }
        if constexpr (EPI == EPI_RESID) {  // raw tiles: part[ks][m tile][n tile][lane]
            ((f32x4*)part)[(((size_t)ks * m_tiles + mt) * (gridDim.x * BNT) + pt0 + ntp) * 64 + lane] = y4[0];
        } else {
            float sum = 0.f;
#pragma unroll
            for (int ww = 0; ww < NW; ++ww) sum += rs_s[ww * ROWS + mt * 16 + r16];
            const float rs = 1.0f / sqrtf(sum / (float)a.K + a.eps);
            float y[TPI][4];
#pragma unroll
            for (int tt = 0; tt < TPI; ++tt)
#pragma unroll
                for (int v = 0; v < 4; ++v) y[tt][v] = y4[tt][v];
            epilogue_item<T, EPI>(a, y, rs, mt * 16 + r16, pt0 + ntp * TPI, g);
        }
    }
}

// K slices of a residual projection: until there is about one workgroup per compute unit
static int stream_w4_slices(int KG, int n_cols, int nkc) { return std::max(1, std::min(std::min(256 / n_cols, 8), nkc / (2 * KG))); }

// Four or eight feature tiles per block: a compute unit holds one block at a time and draws its codes and the activations for it (24
// rows x 5120, four / eight: 960 tiles 18.5 / 24.3 us, 1728 tiles 31.3 / 25.5); residual projections fill the chip with K slices,
// where few tiles per block mean fewer slices to sum (11008 x 4096, 32 rows 15.7 / 16.9; but 13824 x 5120, 64 rows 27.3 / 25.3)
static bool stream_w4_narrow(int epi, int M, int n_tiles) {
    const int mt = M <= 16 ? 1 : M <= 32 ? 2 : 4, b4 = (n_tiles + 3) / 4, b8 = (n_tiles + 7) / 8;
    return epi == EPI_RESID ? mt < 4 : (b4 + 255) / 256 * (4 + 4 * mt) < (b8 + 255) / 256 * (8 + 4 * mt);
}

template <int EPI, int WN, int KG, int MT, int NT, int R>
static hipError_t launch_stream_w4_shape(int layout_nt, int n_tiles, const GemmArgs& a, float* part, size_t part_bytes, hipStream_t s) {
    constexpr int BNT = WN * NT;
    const int n_cols = (n_tiles + BNT - 1) / BNT, m_tiles = (a.M + 15) / 16, nkc = a.nkt / 4;
    const int lsh = layout_nt == 4 ? 2 : layout_nt == 2 ? 1 : 0;
    int ks = 1;
    if constexpr (EPI == EPI_RESID) {
        ks = stream_w4_slices(KG, n_cols, nkc);
        while (ks > 1 && (size_t)ks * m_tiles * n_cols * BNT * 1024 > part_bytes) --ks;
        if ((size_t)ks * m_tiles * n_cols * BNT * 1024 > part_bytes) return hipErrorInvalidValue;
    }
    const int per = ((nkc + ks - 1) / ks + KG - 1) / KG * KG;
    ks = (nkc + per - 1) / per;
    hipLaunchKernelGGL((stream_gemm_w4_kernel<EPI, WN, KG, MT, NT, R>), dim3(n_cols, ks), dim3(WN * KG * 64), 0, s, a.Wp, a.X, a.Sp, nkc, a.M, lsh, n_tiles,
                       per, a, part);
    if (EPI == EPI_RESID) return launch_stream_fixup(a, n_cols * BNT, ks, part, s);
    return hipGetLastError();
}

template <int EPI>
static hipError_t launch_stream_w4_epi(int layout_nt, int n_tiles, const GemmArgs& a, float* part, size_t part_bytes, hipStream_t s) {
    const int mt = a.M <= 16 ? 1 : a.M <= 32 ? 2 : 4;
    const bool narrow = stream_w4_narrow(EPI, a.M, n_tiles);
#define FS_S(wn, kg, mt, r) return launch_stream_w4_shape<EPI, wn, kg, mt, 2, r>(layout_nt, n_tiles, a, part, part_bytes, s)
    if (mt == 1) {
        if (narrow) FS_S(2, 4, 1, 4);
        FS_S(4, 2, 1, 6);
    }
    if (mt == 2) {
        if (narrow) FS_S(2, 4, 2, 3);
        FS_S(4, 2, 2, 4);
    }
    if constexpr (EPI != EPI_RESID) if (narrow) FS_S(2, 2, 4, 3);
    FS_S(4, 2, 4, 3);
#undef FS_S
}

static hipError_t launch_stream_w4(int epi, int layout_nt, int n_tiles, const GemmArgs& a, float* part, size_t part_bytes, hipStream_t s) {
    switch (epi) {
        case EPI_QKV: return launch_stream_w4_epi<EPI_QKV>(layout_nt, n_tiles, a, part, part_bytes, s);
        case EPI_RESID: return launch_stream_w4_epi<EPI_RESID>(layout_nt, n_tiles, a, part, part_bytes, s);
        case EPI_SWIGLU: return launch_stream_w4_epi<EPI_SWIGLU>(layout_nt, n_tiles, a, part, part_bytes, s);
        case EPI_LOGITS: return launch_stream_w4_epi<EPI_LOGITS>(layout_nt, n_tiles, a, part, part_bytes, s);
    }
    return hipErrorInvalidValue;
}

// K slices of a residual projection in the block kernel, and its time in us: whole rounds of blocks (bt row tiles of at most 4 or 8), a
// slice's partial results, 0.4 us a MiB to write and sum, and the launch that sums them against the residual epilogue in the blocks
// themselves (13824 x 5120, 1024 rows: 160 blocks on 256 compute units 235 us, 3 slices 188).  A block's time grows with its rows only in
// part, the codes are unpacked anyway: taken as proportional, and with no cost for the epilogue, short K got too few slices (1024 x 4096,
// 300 rows: 1 slice 31, 2 slices 22; 2048 x 8192, 389 rows: 1 slice 47.6, 2 slices 37.6).  Fitted to 5000 launches of 160 shapes, rms 4 %.
struct W4Slices {
    int ks;
    double us;
};
static W4Slices block_w4_slices(int M, int n_tiles, int nkc, size_t part_bytes) {
    const bool small = M <= 64;
    const int m_tiles = (M + 15) / 16, m_blocks = small ? 1 : (m_tiles + 7) / 8, bt = (m_tiles + m_blocks - 1) / m_blocks, n_cols = (n_tiles + 15) / 16;
    const double chunk = small ? 0.15 + 0.27 * bt : 0.8 + 0.17 * bt;
    W4Slices best{1, 1e30};
    for (int k = 1; k <= std::min(8, std::max(1, nkc / 4)); ++k) {
        const int per = (nkc + k - 1) / k, ks = (nkc + per - 1) / per, rounds = ((n_cols * ks + 7) / 8 * m_blocks + 31) / 32;
        const size_t bytes = (size_t)ks * m_tiles * n_cols * 16 * 1024;
        if (ks > 1 && bytes > part_bytes) break;
        const double us = ks > 1 ? (small ? 8.2 : 10) + rounds * (1.5 + per * chunk) + bytes * 0.4e-6 : 7 + rounds * ((small ? 2 : 6.5) + nkc * chunk);
        if (us < best.us) best = W4Slices{ks, us};
    }
    return best;
}

// One row tile: half a group of four tiles per workgroup where whole groups would leave a last round of few workgroups (592 of them, three
// rounds of 256 compute units, a fill of 0.77 against 0.925: gate/up 28.3 -> 26.5 us; but 896, 0.875 against 1: 64 -> 70)
static bool few_w4_half(int NT, int M, int n_groups) {
    auto fill = [](int n) { return (double)n / ((n + 255) / 256 * 256); };
    return NT == 4 && M <= 16 && fill(2 * n_groups) > 1.18 * fill(n_groups);
}

// Time of the few-row kernel in us: whole rounds of workgroups, each one group of NT feature tiles and up to 32 rows, a wave's chunks one
// after another.  Fitted to 2500 launches of up to 64 rows and 300 of more, rms 5 % (residual projections of one tile per group 8 %: two of
// their workgroups share a compute unit).
static double few_w4_us(int epi, int NT, int M, int n_tiles, int nkc) {
    int groups = (n_tiles + NT - 1) / NT;
    if (few_w4_half(NT, M, groups)) {
        NT = 2;
        groups *= 2;
    }
    const int rounds = (groups * ((M + 31) / 32) + 255) / 256;
    const bool one = M <= 16, r = epi == EPI_RESID;
    if (NT == 4) return 5 + rounds * (one ? 1.6 + 0.213 * nkc : 3 + 0.235 * nkc);
    if (NT == 2) return 5 + rounds * (one ? 1 + 0.119 * nkc : (r ? 2 : 2.8) + (r ? 0.165 : 0.172) * nkc);
    return 5 + rounds * (one ? (r ? 1.2 + 0.06 * nkc : 1.7 + 0.1 * nkc) : r ? 1.5 + 0.115 * nkc : 2 + 0.13 * nkc);
}

// Which 4-bit kernel: a round of the block kernel takes 1.45 (64 rows) or 2.2 us (128 rows) per 128-column chunk, the few-row kernel
// with four tiles per workgroup 0.37 ns per chunk, feature tile and 32-row block.  Both sides, us (few / block): 4096 x 12288, 128
// rows 36 / 74, 200 rows 63 / 74, 389 rows 181 / 75; 5120 x 15360, 65 rows 42 / 87; 5120 x 27648, 128 rows 101 / 89.  Residual
// projections (two tiles per workgroup there, K slices here): 4096 x 4096, 128 rows 18.7 / 24.2, 160 rows 24.2 / 24.5; 5120 x 5120, 65 rows
// 23.3 / 24.2; 11008 x 4096, 65 rows 37.6 / 32.5; 13824 x 5120, 65 rows 43.9 / 39.2; 18944 x 3584, 65 rows 65 / 46, 128 rows 85 / 52; 5632 x
// 2048, 128 rows 18.3 / 25.6, 160 rows 24.2 / 24.9; with a short K there are too few slices to fill the chip: 1024 x 1024, 640 rows 17.9 /
// 22.6, 1024 rows 24.5 / 25; 1536 x 1536, 512 rows 19.8 / 22.2, 640 rows less; 2048 x 2048, 300 rows 18.7 / 21.2.
// Between the line of a long K and the one before it the two times decide, since the few-row kernel's come in whole rounds: 4096 features, 65 to
// 128 rows are two of them, 5632 columns, 128 rows 23.4 / 27.1, 9216 columns, 80 rows 32.8 / 28.7, 128 rows 33.6 / 33.0.
// Its offsets from the operands' bases have 32 bits: 4 GiB of codes and more stay with the few-row kernel.
static bool block_w4_fits(int M, int n_tiles, int nkt) {
    return (unsigned long long)(n_tiles + 16) * nkt * 256ull < (1ull << 32) && (unsigned long long)(M + 16) * nkt * 64ull < (1ull << 32);
}
static bool block_w4_pays(int epi, int layout_nt, int M, int n_tiles, int nkt) {
    if (M <= 32 || !block_w4_fits(M, n_tiles, nkt)) return false;
    const int work = n_tiles * ((M + 31) / 32), rounds = ((n_tiles + 15) / 16 * ((M + 127) / 128) + 255) / 256;
    if (epi == EPI_RESID) {
        if (M <= 64) return work > 600;
        if (work > std::max(1100, 800 + 44000 / nkt)) return true;
        return work > std::min(400 + 90000 / nkt, 800 + 44000 / nkt) &&
               block_w4_slices(M, n_tiles, nkt / 4, (size_t)64 << 20).us < 0.97 * few_w4_us(epi, layout_nt, M, n_tiles, nkt / 4);
    }
    return work > (M <= 64 ? 4200 : 6000) * rounds;
}

// The streaming kernel, up to 64 rows.  It runs one block per compute unit and time, so a launch costs whole rounds of blocks, and a residual
// projection a second launch; the few-row kernel costs whole rounds of its own workgroups, which end elsewhere (256 groups of two tiles are
// one round, 257 two).  So from a least number of tiles or chunks on the two times are worked out and compared.  With that least number
// alone calls of a full round lost, us, few-row / this: QKV of 512 tiles x 4096, 16 rows 10.6 / 12.7, 32 rows 13.3 / 15.4, 64 rows 22.6 / 23.8, x
// 8192 14.6 / 18.0, 18.7 / 22.7, 33.3 / 38.8; gate/up of 256 x 4096, 32 rows 12.4 / 14.8, 64 rows 12.7 / 22.5; head of 512 x 8192, 32 rows 18.5 /
// 23.4; output projection 6144 x 6144, 32 rows 14.7 / 15.9; block kernel / this: 9216 x 6144, 40 rows 21.4 / 23.2.  Where it pays: QKV of 768 x
// 4096, 24 rows 19.1 / 15.2; gate/up of 1728 x 5120, 16 rows 27.7 / 22.6, 24 rows 34.1 / 26.3, 64 rows 50.9 / 37.1; 11008 x 4096, 16 rows 16.1 /
// 13.5.  The least numbers: below them both kernels are short and the estimates (fitted to 4500 launches of 70 shapes, rms 4 - 7 %) say too
// little: head of 640 x 2048, 16 rows 9.5 / 10.2; 4096 x 1024, 24 rows 9.3 / 9.8.
// (Near a tie the estimates still choose well, and a margin for the few-row kernel gives calls away: QKV of 960 x 5120, 24 rows 15.3 / 17.3.)
static bool stream_w4_pays(int epi, int layout_nt, int M, int n_tiles, int nkt) {
    // (16000 tiles: one slice's partial results of a residual projection then fit 64 MiB; a head that wide has not been measured)
    if (M > 64 || n_tiles > 16000 || !block_w4_fits(M, n_tiles, nkt)) return false;
    const int nkc = nkt / 4, m = M <= 16 ? 0 : M <= 32 ? 1 : 2, m_tiles = (M + 15) / 16;
    const bool narrow = stream_w4_narrow(epi, M, n_tiles);
    const int tiles = narrow ? 4 : 8, n_cols = (n_tiles + tiles - 1) / tiles;
    static const double chunk_us[2][3] = {{0.34, 0.45, 0.68}, {0.185, 0.25, 0.488}};  // a block's time per chunk, eight / four tiles
    double us;
    if (epi == EPI_RESID) {
        if (nkc < (m == 0 ? 65 : m == 1 ? 40 : 24)) return false;
        const int kg = narrow ? 4 : 2, k = stream_w4_slices(kg, n_cols, nkc), per = ((nkc + k - 1) / k + kg - 1) / kg * kg, ks = (nkc + per - 1) / per;
        const double in_out = m < 2 ? 3.7 : 3.95, mib_us = m == 0 ? 1 : m == 1 ? 0.8 : 0.67;
        us = in_out + (n_cols * ks + 255) / 256 * (in_out + 0.93 * chunk_us[narrow][m] * per) + mib_us * ks * m_tiles * n_cols * tiles / 1024;
    } else {
        if (n_tiles < (epi == EPI_QKV ? 512 : m == 0 ? 704 : 256) || (m == 2 && n_cols > 256)) return false;
        static const double round_us[2][3] = {{4.4, 6, 8}, {4.2, 4.7, 5.6}};
        us = 2 + (n_cols + 255) / 256 * (round_us[narrow][m] + chunk_us[narrow][m] * nkc);
    }
    double other;
    if (!block_w4_pays(epi, layout_nt, M, n_tiles, nkt))
        other = few_w4_us(epi, layout_nt, M, n_tiles, nkc);
    else if (epi == EPI_RESID)
        other = block_w4_slices(M, n_tiles, nkc, (size_t)64 << 20).us;
    else
        other = (((n_tiles + 15) / 16 + 7) / 8 + 31) / 32 * (10 + (0.15 + 0.27 * m_tiles) * nkc);
    return us < other;
}

int w4_ssp_parts(int layout_nt, int M, int n_tiles, int nkt) {
    if (stream_w4_pays(EPI_RESID, layout_nt, M, n_tiles, nkt)) return (n_tiles + 3) / 4;
    return block_w4_pays(EPI_RESID, layout_nt, M, n_tiles, nkt) ? (n_tiles + 15) / 16 : n_tiles;
}

// Row tiles per block.  Equal heights, since a round lasts as long as its tallest block (5 tiles against 8: 0.9 of the time).  But where an
// odd number of row blocks would leave at most 7 blocks to an XCD's last round (32 compute units) and the last row block of full height has at
// most four tiles, so that half its waves only load, what would be the last round starts behind such blocks and runs beside the others.  us,
// equal / full heights: 4096 x 22016, 257 rows 129.6 / 110.2, 300 rows 136 / 112.7; 7168 x 21504, 300 rows 230 / 188; 8192 x 25600 (39 blocks an
// XCD) 262 / 240; 2048 x 11264 (66) 119 / 108, 5120 x 11008 263 / 237; 5120 x 6400, 530 rows (65 blocks in five row blocks) 263 / 235; 129 blocks
// 199 / 180, 161 in seven row blocks 245 / 225.  With more in the last round the difference goes: 40 blocks 80.3 / 84.8, 42 160 / 179.  With an even
// number the short blocks all fall to the same part of an XCD and make no room elsewhere: 7168 x 33024, 129 rows 214 / 238; 4096 x 18432, 389 rows
// 138 / 147.
static int block_w4_height(bool resid, int m_tiles, int m_blocks, int n_cols) {
    const int equal = (m_tiles + m_blocks - 1) / m_blocks, blocks = (n_cols + 7) / 8 * m_blocks, over = blocks % 32;
    if (!resid && m_blocks % 2 && m_tiles - 8 * (m_blocks - 1) <= 4 && m_blocks > 1 && blocks > 32 && over > 0 && over < 8) return 8;
    return equal;
}

template <int EPI, int WM, int WN, int MT, int NT, int R>
static hipError_t launch_w4_shape(int layout_nt, int n_tiles, const GemmArgs& a, float* part, size_t part_bytes, hipStream_t s) {
    constexpr int BMT = WM * MT, BNT = WN * NT;
    static_assert(BNT == 16, "the residual projections' sums of squares come per 16 feature tiles");
    const int m_tiles = (a.M + 15) / 16, m_blocks = (m_tiles + BMT - 1) / BMT, n_cols = (n_tiles + BNT - 1) / BNT, nkc = a.nkt / 4;
    const int bt = block_w4_height(EPI == EPI_RESID, m_tiles, m_blocks, n_cols);
    const int lsh = layout_nt == 4 ? 2 : layout_nt == 2 ? 1 : 0;
    const dim3 block(WM * WN * 64);
    if constexpr (EPI == EPI_RESID) {
        const int ks = block_w4_slices(a.M, n_tiles, nkc, part_bytes).ks;
        if (ks > 1) {
            const int per = (nkc + ks - 1) / ks;
            hipLaunchKernelGGL((block_gemm_w4_kernel<EPI, true, WM, WN, MT, NT, R>), dim3(8 * m_blocks, (n_cols * ks + 7) / 8), block, 0, s, a.Wp, a.X, a.Sp, nkc, a.M, lsh,
                               n_tiles, per, bt, a, part);
            return launch_fixup<4>(a, n_cols * BNT, ks, part, s);
        }
    }
    hipLaunchKernelGGL((block_gemm_w4_kernel<EPI, false, WM, WN, MT, NT, R>), dim3(8 * m_blocks, (n_cols + 7) / 8), block, 0, s, a.Wp, a.X, a.Sp, nkc, a.M, lsh, n_tiles,
                       nkc, bt, a, nullptr);
    return hipGetLastError();
}

static hipError_t launch_block_w4(int epi, int layout_nt, int n_tiles, const GemmArgs& a, float* part, size_t part_bytes, hipStream_t s) {
    if (!a.x_frag || !block_w4_fits(a.M, n_tiles, a.nkt)) return hipErrorInvalidValue;
#define FS_W4(e)                                                                                              \
    if (epi == e) {                                                                                           \
        if (a.M <= 64) return launch_w4_shape<e, 1, 8, 4, 2, 4>(layout_nt, n_tiles, a, part, part_bytes, s);  \
        return launch_w4_shape<e, 2, 4, 4, 4, 3>(layout_nt, n_tiles, a, part, part_bytes, s);                 \
    }
    FS_W4(EPI_QKV) FS_W4(EPI_RESID) FS_W4(EPI_SWIGLU) FS_W4(EPI_LOGITS)
#undef FS_W4
    return hipErrorInvalidValue;
}

hipError_t launch_gemm_w4(int epi, int NT, int NW, int n_groups, const GemmArgs& a, float* part, size_t part_bytes, hipStream_t s) {
    if (stream_w4_pays(epi, NT, a.M, n_groups * NT, a.nkt)) return launch_stream_w4(epi, NT, n_groups * NT, a, part, part_bytes, s);
    if (block_w4_pays(epi, NT, a.M, n_groups * NT, a.nkt)) return launch_block_w4(epi, NT, n_groups * NT, a, part, part_bytes, s);
    // at most 32 rows per workgroup (register budget); longer segments take further row blocks, whose passes over
    // the quarter-size weights mostly hit in L2
    const int MT = a.M <= 16 ? 1 : 2;
    const bool half = few_w4_half(NT, a.M, n_groups);
    if (half) {
        NT = 2;
        n_groups *= 2;
    }
    if (NW > 8) NW = 8;
    if (MT * NT >= 8 && NW > 4) NW = 4;  // as in the dense launcher
    if (epi == EPI_QKV) return launch_mt_nt_w4<EPI_QKV>(MT, NT, half, NW, n_groups, a, s);
    if (epi == EPI_RESID) return launch_mt_nt_w4<EPI_RESID>(MT, NT, half, NW, n_groups, a, s);
    if (epi == EPI_SWIGLU) return launch_mt_nt_w4<EPI_SWIGLU>(MT, NT, half, NW, n_groups, a, s);
    if (epi == EPI_LOGITS) return launch_mt_nt_w4<EPI_LOGITS>(MT, NT, half, NW, n_groups, a, s);
    return hipErrorInvalidValue;
}

// Entry of a stage whose projections take fragment-major activations and the rows' sums of squares from their producer
// (4-bit weights, many-row segments; see GemmArgs::gain_next): row-major rows -> fragment-major copy (times the gain, if
// given) + partial sums of squares per 512-column slice.  Workgroup (row tile, slice); thread (r, g, j) converts the
// 8-element fragment pieces of k-tiles j, j + 4, ... of its slice.
__global__ void __launch_bounds__(256) prenorm_kernel(const bf16_t* X, int ldx, int M, int K, const bf16_t* gain, bf16_t* xg, float* ssp,
                                                         int ssp_stride) {
    __shared__ float red[16][17];
    const int t = threadIdx.x, r = t & 15, g = (t >> 4) & 3, j = t >> 6;
    const int mt = blockIdx.x, slice = blockIdx.y, nkt = K >> 5;
    const int m = mt * 16 + r, mc = min(m, M - 1);
    float ss = 0.f;
    const int kt_end = min(nkt, slice * 16 + 16);
    for (int kt = slice * 16 + j; kt < kt_end; kt += 4) {
        const int k = kt * 32 + g * 8;
        const bf16x8 x = *(const bf16x8*)(X + (size_t)mc * ldx + k);
        bf16x8 y = x;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float f = (float)x[e];
            ss += f * f;
        }
        if (gain) {
            const bf16x8 gn = *(const bf16x8*)(gain + k);
#pragma unroll
            for (int e = 0; e < 8; ++e) y[e] = (bf16_t)((float)x[e] * (float)gn[e]);
        }
        *(bf16x8*)(xg + frag_major_index<bf16_t>(m, k, nkt)) = y;
    }
    red[t >> 4][r] = ss;
    __syncthreads();
    if (t < 16) {
        float s = 0.f;
        for (int i = 0; i < 16; ++i) s += red[i][t];
        if (mt * 16 + t < ssp_stride) ssp[(size_t)slice * ssp_stride + mt * 16 + t] = s;
    }
}

hipError_t launch_prenorm(const void* X, int ldx, int M, int K, const void* gain, void* xg, float* ssp, int ssp_stride, int* n_slices,
                             hipStream_t s) {
    const int slices = (K + 511) / 512;
    *n_slices = slices;
    hipLaunchKernelGGL(prenorm_kernel, dim3((M + 15) / 16, slices), dim3(256), 0, s, (const bf16_t*)X, ldx, M, K, (const bf16_t*)gain,
                       (bf16_t*)xg, ssp, ssp_stride);
    return hipGetLastError();
}

// Source row of packed row (ptile, r) for the three matrix kinds; -1 if beyond the matrix.  `which` selects the source slot.
static __device__ __forceinline__ long long packed_source_row(int kind, int ptile, int r, int N, int Hq, int Hkv, int hd, int* which) {
    *which = 0;
    if (kind == PACK_PLAIN) {
        const long long row = (long long)ptile * 16 + r;
        return row < N ? row : -1;
    }
    if (kind == PACK_GATEUP) {
        *which = ptile & 1;
        const long long row = (long long)(ptile >> 1) * 16 + r;
        return row < N ? row : -1;
    }
    const int tph = hd >> 4, head = ptile / tph, tih = ptile % tph;
    if (head < Hq + Hkv) {
        const int orig = (tih >> 1) + (tih & 1) * (tph >> 1);
        *which = head < Hq ? 0 : 1;
        return (long long)(head < Hq ? head : head - Hq) * hd + orig * 16 + r;
    }
    if (head < Hq + 2 * Hkv) {
        *which = 2;
        return (long long)(head - Hq - Hkv) * hd + tih * 16 + r;
    }
    return -1;
}

__global__ void pack_w4_kernel(const PackW4Args a) {
    const int nkc = a.K / 128;
    const size_t total = (size_t)a.n_groups * nkc * a.NT * 64;
    for (size_t c = (size_t)blockIdx.x * blockDim.x + threadIdx.x; c < total; c += (size_t)gridDim.x * blockDim.x) {
        const int lane = (int)(c & 63);
        size_t t = c >> 6;
        const int nt = (int)(t % a.NT);
        t /= a.NT;
        const int chunk = (int)(t % nkc), grp = (int)(t / nkc);
        const int r = lane & 15, g = lane >> 4;
        const int ptile = grp * a.NT + nt;
        int which;
        const long long row = packed_source_row(a.kind, ptile, r, a.N, a.Hq, a.Hkv, a.hd, &which);
        const unsigned char* codes = (const unsigned char*)(which == 0 ? a.c0 : (which == 1 ? a.c1 : a.c2));
        unsigned d[4];
        for (int q = 0; q < 4; ++q) {
            unsigned v = 0;
            for (int e = 0; e < 8; ++e) {
                unsigned code = 8;  // rows beyond the matrix: zero weight
                if (row >= 0) {
                    const int k = chunk * 128 + q * 32 + g * 8 + e;
                    const unsigned char b = codes[(size_t)row * (a.K / 2) + (k >> 1)];
                    code = (k & 1) ? (b >> 4) : (b & 15);
                }
                v |= code << (4 * ((e & 1) * 4 + (e >> 1)));
            }
            d[q] = v;
        }
        ((u32x4*)a.dst)[c] = u32x4{d[0], d[1], d[2], d[3]};
        if (g == 0) {
            const bf16_t* sc = (const bf16_t*)(which == 0 ? a.s0 : (which == 1 ? a.s1 : a.s2));
            ((bf16_t*)a.sdst)[(((size_t)grp * nkc + chunk) * a.NT + nt) * 16 + r] = row >= 0 ? sc[(size_t)row * nkc + chunk] : (bf16_t)0.f;
        }
    }
    if (a.kind == PACK_QKV && a.bias_dst) {
        const int np = a.n_groups * a.NT * 16;
        for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < np; i += gridDim.x * blockDim.x) {
            int which;
            const long long row = packed_source_row(PACK_QKV, i >> 4, i & 15, a.N, a.Hq, a.Hkv, a.hd, &which);
            const bf16_t* b = (const bf16_t*)(which == 0 ? a.b0 : (which == 1 ? a.b1 : a.b2));
            a.bias_dst[i] = (row >= 0 && b) ? (float)b[row] : 0.f;
        }
    }
}

void launch_pack_w4(const PackW4Args& a, hipStream_t s) {
    const size_t total = (size_t)a.n_groups * (a.K / 128) * a.NT * 64;
    int blocks = (int)((total + 255) / 256);
    if (blocks > 65536) blocks = 65536;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(pack_w4_kernel, dim3(blocks), dim3(256), 0, s, a);
}

// ---- one-time weight re-tiling ------------------------------------------------------------------
// One thread per 16-byte fragment slot of the destination.  Rows of Q and K heads are re-ordered so that
// tiles (2i, 2i+1) of a head hold features [16i, 16i+16) and [hd/2 + 16i, hd/2 + 16i + 16): the two halves
// of the rotary pairs land in one workgroup.  Gate and up rows alternate tile by tile so that silu(gate)*up
// is formed in the epilogue.  Rows / columns beyond N / K are zero.
template <typename T>
__global__ void pack_kernel(const PackArgs a) {
    using E = Elem<T>;
    const size_t total = (size_t)a.n_groups * a.nkt * a.NT * 64;
    for (size_t c = (size_t)blockIdx.x * blockDim.x + threadIdx.x; c < total; c += (size_t)gridDim.x * blockDim.x) {
        const int lane = (int)(c & 63);
        size_t t = c >> 6;
        const int nt = (int)(t % a.NT);
        t /= a.NT;
        const int kt = (int)(t % a.nkt);
        const int grp = (int)(t / a.nkt);
        const int r = lane & 15, g = lane >> 4;
        const int ptile = grp * a.NT + nt;
        const int k = kt * E::KT + g * E::EPF;
        const T* src = nullptr;
        long long row = -1;
        if (a.kind == PACK_PLAIN) {
            row = (long long)ptile * 16 + r;
            src = (const T*)a.src0;
            if (row >= a.N) row = -1;
        } else if (a.kind == PACK_GATEUP) {
            row = (long long)(ptile >> 1) * 16 + r;
            src = (const T*)((ptile & 1) ? a.src1 : a.src0);
            if (row >= a.N) row = -1;  // N = d_ffn here
        } else {
            const int tph = a.hd >> 4;
            const int head = ptile / tph, tih = ptile % tph;
            if (head < a.Hq + a.Hkv) {
                const int orig = (tih >> 1) + (tih & 1) * (tph >> 1);
                const int hh = head < a.Hq ? head : head - a.Hq;
                src = (const T*)(head < a.Hq ? a.src0 : a.src1);
                row = (long long)hh * a.hd + orig * 16 + r;
            } else if (head < a.Hq + 2 * a.Hkv) {
                src = (const T*)a.src2;
                row = (long long)(head - a.Hq - a.Hkv) * a.hd + tih * 16 + r;
            }
        }
        typename E::frag_t f = E::zero();
        if (row >= 0 && k < a.K) {
#pragma unroll
            for (int e = 0; e < E::EPF; ++e) {
                float v = E::to_f(src[(size_t)row * a.K + k + e]);
                if (a.gain) v *= E::to_f(((const T*)a.gain)[k + e]);
                f[e] = E::from_f(v);
            }
        }
        ((typename E::frag_t*)a.dst)[c] = f;
    }
    // packed-order bias (QKV only)
    if (a.kind == PACK_QKV && a.bias_dst) {
        const int np = a.n_groups * a.NT * 16;
        for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < np; i += gridDim.x * blockDim.x) {
            const int ptile = i >> 4, r = i & 15;
            const int tph = a.hd >> 4;
            const int head = ptile / tph, tih = ptile % tph;
            float v = 0.f;
            if (head < a.Hq + a.Hkv) {
                const int orig = (tih >> 1) + (tih & 1) * (tph >> 1);
                const int hh = head < a.Hq ? head : head - a.Hq;
                const T* b = (const T*)(head < a.Hq ? a.b0 : a.b1);
                if (b) v = E::to_f(b[hh * a.hd + orig * 16 + r]);
            } else if (head < a.Hq + 2 * a.Hkv) {
                const T* b = (const T*)a.b2;
                if (b) v = E::to_f(b[(head - a.Hq - a.Hkv) * a.hd + tih * 16 + r]);
            }
            a.bias_dst[i] = v;
        }
    }
}

void launch_pack(int dtype, const PackArgs& a, hipStream_t s) {
    const size_t total = (size_t)a.n_groups * a.nkt * a.NT * 64;
    int blocks = (int)((total + 255) / 256);
    if (blocks > 65536) blocks = 65536;
    if (blocks < 1) blocks = 1;
    if (dtype == 0)
        hipLaunchKernelGGL(pack_kernel<float>, dim3(blocks), dim3(256), 0, s, a);
    else
        hipLaunchKernelGGL(pack_kernel<bf16_t>, dim3(blocks), dim3(256), 0, s, a);
}
