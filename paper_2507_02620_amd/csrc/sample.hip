// Stochastic acceptance (temperature > 0): sequential candidate test along the tree with integer probability
// weights, so that every decision is an integer comparison and reproducible bit for bit.
//
//   z_v = logits_v * inv_temp;  m = max_v z_v;  e_v = exp2_spec((z_v - m) * log2 e);  E_v = (uint64)(e_v * 2^32);  Z = sum E_v
//   at accepted node u (remaining mass R = Z_u): children in S order; child c accepted iff r24 * R < E_c * 2^24, else
//   R -= E_c and the token is struck; no child accepted -> x_new = first v with running sum of unstruck E > u48*R/2^48.
//   Uniform numbers: counter-based generator keyed by (seed, step, draw index).
//
// exp2_spec is a fixed sequence of IEEE fp32 operations (no contraction), so any implementation produces the same bits.
#include "tree.hpp"

#include <algorithm>

#pragma clang fp contract(off)

static __device__ __forceinline__ uint64_t rng64(uint64_t seed, uint64_t step, uint64_t k) {
    uint64_t z = seed ^ (step * 0x9E3779B97F4A7C15ull) ^ (k * 0xBF58476D1CE4E5B9ull);
    z ^= z >> 30; z *= 0xBF58476D1CE4E5B9ull;
    z ^= z >> 27; z *= 0x94D049BB133111EBull;
    z ^= z >> 31;
    return z;
}

// E = (uint64)(exp2_spec * 2^32).  The polynomial's value p lies in [1, 2]; scaling it by 2^(n + 32), n <= 0, and truncating is a
// shift of its 24-bit significand, exact and without the conversion sequence a float -> uint64 cast takes.
static __device__ __forceinline__ uint64_t exp_weight(float z, float m) {
    const float t = __fmul_rn(__fsub_rn(z, m), 1.44269504088896341f);  // <= 0: m is the row's maximum
    if (!(t >= -64.0f)) return 0;
    const float n = floorf(t), f = __fsub_rn(t, n);
    float p = 1.52527338e-5f;
    p = fmaf(p, f, 1.54035304e-4f);
    p = fmaf(p, f, 1.33335581e-3f);
    p = fmaf(p, f, 9.61812911e-3f);
    p = fmaf(p, f, 5.55041087e-2f);
    p = fmaf(p, f, 2.40226507e-1f);
    p = fmaf(p, f, 6.93147181e-1f);
    p = fmaf(p, f, 1.0f);
    const unsigned bits = __float_as_uint(p);
    const int sh = 127 - (int)(bits >> 23) - (int)n;  // 0 .. 64 places below 2^32 (p = 2 only with n <= -1)
    // (the shift in 32 bits, with the cases of no and of more than 32 places apart, makes the sums' launch 12.8 -> 14.2 us)
    return ((uint64_t)((bits & 0x7FFFFFu) | 0x800000u) << 9) >> min(sh, 63);
}

// Row maxima are kept as unsigned keys that order like the floats do (0: below every float), so that the chunks of a row can
// meet in an atomic maximum.
static __device__ __forceinline__ unsigned max_key(float m) {
    const unsigned b = __float_as_uint(m);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
static __device__ __forceinline__ float key_max(unsigned k) { return __uint_as_float((k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k); }

// Visits n pieces of E floats with all threads of the group, adjacent threads on adjacent pieces, U loads in flight per thread.  fn(x, live).
// CLAMP: what a thread has left behind its full rounds goes out together too and repeats the last piece (live is false for repeats) instead of
// one load at a time: shorter where a round is most of the work, longer where it is little of it.
template <int U, bool CLAMP, int E, typename F>
static __device__ __forceinline__ void for_pieces(const float* __restrict__ p, int n, int t, int nt, F&& fn) {
    auto load = [&](int i, float (&x)[E]) __attribute__((always_inline)) {
        if constexpr (E == 4) {
            const f32x4 q = *(const f32x4*)(p + (size_t)i * 4);
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = q[e];
        } else {
            x[0] = p[i];
        }
    };
    int i = t;
    for (; i + (U - 1) * nt < n; i += U * nt) {
        float x[U][E];
#pragma unroll
        for (int k = 0; k < U; ++k) load(i + k * nt, x[k]);
#pragma unroll
        for (int k = 0; k < U; ++k)
#pragma unroll
            for (int e = 0; e < E; ++e) fn(x[k][e], true);
    }
    if constexpr (CLAMP) {
        if (i < n) {
            float x[U][E];
#pragma unroll
            for (int k = 0; k < U; ++k) load(min(i + k * nt, n - 1), x[k]);
#pragma unroll
            for (int k = 0; k < U; ++k)
#pragma unroll
                for (int e = 0; e < E; ++e) fn(x[k][e], i + k * nt < n);
        }
    } else {
        for (; i < n; i += nt) {
            float x[E];
            load(i, x);
#pragma unroll
            for (int e = 0; e < E; ++e) fn(x[e], true);
        }
    }
}

// The elements [lo, hi) of a row: by 16 bytes where the row allows it (lo a multiple of 4), the rest by elements.
template <int U, bool CLAMP, typename F>
static __device__ __forceinline__ void for_row(const float* __restrict__ p, int lo, int hi, int t, int nt, bool vec, F&& fn) {
    int v = lo;
    if (vec) {
        for_pieces<U, CLAMP, 4>(p + lo, (hi - lo) >> 2, t, nt, fn);
        v = lo + ((hi - lo) & ~3);
    }
    for_pieces<U, CLAMP, 1>(p + v, hi - v, t, nt, fn);
}

static __device__ __forceinline__ uint64_t wave_sum_u64(uint64_t v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, FS_WAVE);
    return v;
}

#define SMP_STAT_THREADS 256
// Row statistics of the verified rows: m = max z and Z = sum of the integer weights, which needs m first.  A compute unit draws 25 - 45 GB/s
// from memory, so one workgroup per row leaves most of the chip idle (80 rows x 152064: 351 us in one launch with scalar loads);
// here every row is cut into gridDim.x chunks and the chunks of a row meet in an atomic maximum and an atomic (integer: order does
// not matter) sum: 1.6 + 11 + 13 us, 48.7 MB read twice at 4.4 and 3.7 TB/s (the weights' arithmetic alone is about 9 us of the second pass).
__global__ void __launch_bounds__(256) sample_clear_kernel(unsigned* __restrict__ rowm, unsigned long long* __restrict__ rowZ, int rows) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < rows) {
        rowm[i] = 0u;
        rowZ[i] = 0ull;
    }
}

__global__ void __launch_bounds__(SMP_STAT_THREADS) sample_max_kernel(const float* __restrict__ logits, int vocab, float inv_temp, int chunk, bool vec,
                                                                      unsigned* __restrict__ rowm) {
    __shared__ float shm[SMP_STAT_THREADS / 64];
    const float* p = logits + (size_t)blockIdx.y * vocab;
    const int lo = blockIdx.x * chunk, hi = min(vocab, lo + chunk);
    float m = -INFINITY;
    for_row<4, true>(p, lo, hi, threadIdx.x, SMP_STAT_THREADS, vec, [&](float x, bool) { m = fmaxf(m, __fmul_rn(x, inv_temp)); });
    for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, FS_WAVE));
    if ((threadIdx.x & 63) == 0) shm[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < SMP_STAT_THREADS / 64; ++w) m = fmaxf(m, shm[w]);
        atomicMax(&rowm[blockIdx.y], max_key(m));
    }
}

__global__ void __launch_bounds__(SMP_STAT_THREADS) sample_sum_kernel(const float* __restrict__ logits, int vocab, float inv_temp, int chunk, bool vec,
                                                                      const unsigned* __restrict__ rowm, unsigned long long* __restrict__ rowZ) {
    __shared__ uint64_t shz[SMP_STAT_THREADS / 64];
    const float* p = logits + (size_t)blockIdx.y * vocab;
    const int lo = blockIdx.x * chunk, hi = min(vocab, lo + chunk);
    const float m = key_max(rowm[blockIdx.y]);
    uint64_t z = 0;
    for_row<4, true>(p, lo, hi, threadIdx.x, SMP_STAT_THREADS, vec, [&](float x, bool live) { z += live ? exp_weight(__fmul_rn(x, inv_temp), m) : 0; });
    z = wave_sum_u64(z);
    if ((threadIdx.x & 63) == 0) shz[threadIdx.x >> 6] = z;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < SMP_STAT_THREADS / 64; ++w) z += shz[w];
        atomicAdd(&rowZ[blockIdx.y], (unsigned long long)z);
    }
}

// The same with one workgroup per row, in one launch: small vocabularies, where the three launches are the time, and rows enough
// to fill the chip.
__global__ void __launch_bounds__(SMP_STAT_THREADS) sample_rowstats_kernel(const float* __restrict__ logits, int vocab, float inv_temp, bool vec,
                                                                           unsigned* __restrict__ rowm, unsigned long long* __restrict__ rowZ) {
    __shared__ float shm[SMP_STAT_THREADS / 64];
    __shared__ uint64_t shz[SMP_STAT_THREADS / 64];
    const float* p = logits + (size_t)blockIdx.x * vocab;
    float m = -INFINITY;
    for_row<4, false>(p, 0, vocab, threadIdx.x, SMP_STAT_THREADS, vec, [&](float x, bool) { m = fmaxf(m, __fmul_rn(x, inv_temp)); });
    for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, FS_WAVE));
    if ((threadIdx.x & 63) == 0) shm[threadIdx.x >> 6] = m;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < SMP_STAT_THREADS / 64; ++w) m = fmaxf(m, shm[w]);
    uint64_t z = 0;
    for_row<4, false>(p, 0, vocab, threadIdx.x, SMP_STAT_THREADS, vec, [&](float x, bool live) { z += live ? exp_weight(__fmul_rn(x, inv_temp), m) : 0; });
    z = wave_sum_u64(z);
    if ((threadIdx.x & 63) == 0) shz[threadIdx.x >> 6] = z;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < SMP_STAT_THREADS / 64; ++w) z += shz[w];
        rowm[blockIdx.x] = max_key(m);
        rowZ[blockIdx.x] = z;
    }
}

#define SMP_THREADS 1024 /* one node of the tree per thread */
#define SMP_WAVES (SMP_THREADS / 64)
#define SMP_PENDING (-2)  /* x_new = SMP_PENDING - u while the residual draw at node u is still to come */

// Rank of this thread among the threads whose flag is set, and their number (two barriers).
static __device__ __forceinline__ int block_rank(bool flag, int* sh, int* total) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const unsigned long long b = __ballot(flag);
    __syncthreads();
    if (lane == 0) sh[w] = __popcll(b);
    __syncthreads();
    int before = 0, all = 0;
#pragma unroll
    for (int k = 0; k < SMP_WAVES; ++k) {
        const int c = sh[k];
        before += k < w ? c : 0;
        all += c;
    }
    *total = all;
    return before + __popcll(b & ((1ull << lane) - 1));
}

// One workgroup walks the tree.  Latency is what it costs, so everything that can be parallel is: every node's weight under its parent's
// row and every row's sum are fetched before the walk (one round of memory latency for the whole tree instead of two per accepted
// node), the children of a node are gathered by ballots and their duplicate tests run side by side; one lane then only takes
// the decisions from LDS.  The residual draw narrows the vocabulary down in up to three coalesced passes (a sixteenth per wave, a
// sixteenth of that per wave, then 64 elements at a time) with the rejected tokens' weights taken off the sums; what is down to
// 256 elements (64 behind many rejected tokens, which every step of the last pass looks through) goes to the last one at once: two
// barriers of 16 waves cost more than its three further steps (one node, 200 entries, whole call 11.0 -> 6.9 us).
// (16 rows x 32000 below a star of 16 nodes, whole call: 338 -> 35 us.)  Where sample_draw_kernel follows (`pending`), the draw's target is
// left to it: three accepted nodes and a draw over 152064 entries 40 us in here, of which the 608 KB row through one compute unit was the
// larger part, now 8 here and 10 there.
__global__ void __launch_bounds__(SMP_THREADS) accept_sample_kernel(const float* __restrict__ logits, int vocab, float inv_temp, bool vec,
                                                                    const unsigned* __restrict__ rowm, const unsigned long long* rowZ,
                                                                    const int32_t* __restrict__ token, const int32_t* __restrict__ parent, int T,
                                                                    int n_ver, uint64_t seed, uint64_t step, AcceptResultDev* __restrict__ res,
                                                                    int32_t* __restrict__ retain, unsigned long long* pending) {
    __shared__ short child[1024], jump[2][1024];
    __shared__ unsigned char keep[1024], reach[2][1024], skip[1024];
    __shared__ __align__(16) int ctok[1024];
    __shared__ int rej[1024], sh[SMP_WAVES];
    __shared__ uint64_t cw[1024], rejw[1024], zrow[1024], sums[SMP_WAVES];
    __shared__ int s_next, s_nrej;
    __shared__ uint64_t s_draw, s_target;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;

    const int par = tid < T ? parent[tid] : -1;
    const int tok = tid < T ? token[tid] : 0;
    const int bad_topo = tid < T && (par < -1 || par >= tid || (tid == 0 && par != -1));
    keep[tid] = 0;
    if (tid == 0) s_draw = 0;
    if (__syncthreads_or(bad_topo)) {
        if (tid == 0) res->n_acc = -1;
        return;
    }
    if (n_ver == 0) {
        if (tid < T) retain[tid] = tid;
        if (tid == 0) *res = AcceptResultDev{0, -1, 0, 1, T, 0};
        return;
    }

    const bool in_vocab = tid < T && tok >= 0 && tok < vocab;
    const uint64_t wt = in_vocab && par >= 0 && par < n_ver ? exp_weight(__fmul_rn(logits[(size_t)par * vocab + tok], inv_temp), key_max(rowm[par])) : 0;
    if (tid < n_ver) zrow[tid] = rowZ[tid];

    int u = 0, n_acc = 0, x_new = -1, n_new = -1;  // uniform over the workgroup
    for (;;) {  // one iteration per accepted node: at most T of them
        // children of u in ascending order, their tokens and weights
        const bool is_child = tid < T && par == u;
        int n_child;
        const int rank = block_rank(is_child, sh, &n_child);
        if (is_child) {
            child[rank] = (short)tid;
            ctok[rank] = in_vocab ? tok : -1;
            cw[rank] = wt;
        }
        if (tid == 0) keep[u] = 1;
        ++n_acc;
        __syncthreads();
        // A child whose token an earlier sibling carries is passed over: whenever it is reached, that sibling was rejected.
        if (tid < n_child) {
            const int t = ctok[tid];
            bool dup = t < 0;
#pragma unroll 1  // unrolled it is only more code to fetch by a cold launch
            for (int j = 0; j < tid && !dup; j += 4) {
                const int4 c = *(const int4*)(ctok + j);
                dup = c.x == t || (c.y == t && j + 1 < tid) || (c.z == t && j + 2 < tid) || (c.w == t && j + 3 < tid);
            }
            skip[tid] = dup;
        }
        __syncthreads();
        if (tid == 0) {
            uint64_t R = zrow[u], draw = s_draw;
            int n_rej = 0, next = -1;
            for (int k = 0; k < n_child && next < 0; ++k) {
                if (skip[k]) continue;
                const uint64_t Ec = cw[k];
                const uint64_t r24 = rng64(seed, step, draw++) >> 40;
                const uint64_t hi = __umul64hi(r24, R), lo = r24 * R;
                if (hi == 0 && lo < (Ec << 24)) {
                    next = child[k];
                } else {
                    R -= Ec;
                    rej[n_rej] = ctok[k];
                    rejw[n_rej++] = Ec;
                }
            }
            s_next = next; s_nrej = n_rej;
            if (next < 0) {
                const uint64_t u48 = ((rng64(seed, step, draw) >> 40) << 24) | (rng64(seed, step, draw + 1) >> 40);
                draw += 2;
                s_target = (__umul64hi(u48, R) << 16) | ((u48 * R) >> 48);
            }
            s_draw = draw;
        }
        __syncthreads();
        const int next = s_next;
        if (next >= 0 && next < n_ver) {  // accepted and verified: descend
            u = next;
            continue;
        }
        if (next >= 0) {  // accepted, not verified yet: the node n_new of the continuous condition
            for (int k = 0; k < n_child; ++k)
                if (child[k] == next) x_new = ctok[k];
            n_new = next;
            break;
        }
        // Residual draw: the first v whose running sum of unstruck weights exceeds the target.  Integer sums: any grouping gives
        // the same token.
        if (pending) {  // left to the launches behind this one
            if (tid == 0) {
                pending[0] = s_target;
                pending[1] = 0;
            }
            x_new = SMP_PENDING - u;
            break;
        }
        const float* row = logits + (size_t)u * vocab;
        const float m = key_max(rowm[u]);
        const uint64_t target = s_target;
        const int n_rej = s_nrej;
        int lo = 0, hi = vocab;
        uint64_t base = 0;  // running sum below lo
        bool found = true;
        const int scan = n_rej < 8 ? 256 : 64;
        for (int pass = vocab > scan ? 0 : 2; pass < 2 && found; ++pass) {
            const int part = ((hi - lo + SMP_WAVES - 1) / SMP_WAVES + 3) & ~3;  // a multiple of 4 elements per wave
            const int wlo = min(hi, lo + w * part), whi = min(hi, wlo + part);
            uint64_t z = 0;
            for_row<4, false>(row, wlo, whi, lane, 64, vec, [&](float x, bool live) { z += live ? exp_weight(__fmul_rn(x, inv_temp), m) : 0; });
            for (int j = lane; j < n_rej; j += 64)
                if (rej[j] >= wlo && rej[j] < whi) z -= rejw[j];
            z = wave_sum_u64(z);
            __syncthreads();
            if (lane == 0) sums[w] = z;
            __syncthreads();
            found = false;
            const int lo0 = lo, hi0 = hi;
            uint64_t before = base;
            for (int k = 0; k < SMP_WAVES; ++k) {
                const uint64_t s = sums[k];
                if (!found && target < before + s) {  // the first part that reaches beyond the target
                    found = true;
                    lo = min(hi0, lo0 + k * part);
                    hi = min(hi0, lo + part);
                    base = before;
                }
                before += s;
            }
            if (hi - lo <= scan) break;
        }
        x_new = vocab - 1;  // the definition's default (no weight left)
        for (int v0 = lo; found && v0 < hi; v0 += 64) {  // every wave does the same
            const int v = v0 + lane;
            uint64_t run = 0;
            if (v < hi) {
                run = exp_weight(__fmul_rn(row[v], inv_temp), m);
                for (int j = 0; j < n_rej; ++j)
                    if (rej[j] == v) run = 0;
            }
            for (int o = 1; o < 64; o <<= 1) {
                const uint64_t below = __shfl_up(run, o, FS_WAVE);
                if (lane >= o) run += below;
            }
            const unsigned long long hit = __ballot(v < hi && base + run > target);
            if (hit) {
                x_new = v0 + __ffsll(hit) - 1;
                break;
            }
            base += __shfl(run, 63, FS_WAVE);
        }
        break;
    }

    // n_new and its descendants: pointer doubling over the parent links (ceil(log2 T) rounds)
    int cur = 0;
    if (n_new >= 0) {
        jump[0][tid] = (short)(tid < T ? par : -1);
        reach[0][tid] = tid == n_new;
        for (int span = 1; span < T; span <<= 1) {
            __syncthreads();
            const int j = jump[cur][tid];
            reach[cur ^ 1][tid] = reach[cur][tid] | (j >= 0 ? reach[cur][j] : 0);
            jump[cur ^ 1][tid] = j >= 0 ? jump[cur][j] : (short)-1;
            cur ^= 1;
        }
    }
    __syncthreads();
    const bool on_path = tid < T && keep[tid] == 1, below = n_new >= 0 && tid < T && reach[cur][tid];
    int total, prv;
    const int pos = block_rank(on_path || below, sh, &total);
    if (on_path || below) retain[pos] = tid;
    (void)block_rank(below && tid < n_ver, sh, &prv);
    if (tid == 0) *res = AcceptResultDev{n_acc, x_new, n_new, n_new >= 0, total, prv};
}

// ---- residual draw of a large vocabulary -----------------------------------------------------------------------------------
// One compute unit takes 24 us for a row of 152064 logits.  Spread over the chip every workgroup sums one chunk of the row, and the one that
// arrives last finds the token in the chunk that holds the target: about 10 us (two launches instead: 5.4 + 5.6, but a call whose
// walk ends without a draw then pays for two that do nothing, 2.3 us each).  Nobody waits for anybody: the last to arrive is told by a
// counter.  All children of the last accepted node were rejected, so the struck tokens are read off the tree again.
#define DRAW_THREADS 256
#define DRAW_EACH 16  /* consecutive logits per thread */
#define DRAW_BLOCK (DRAW_THREADS * DRAW_EACH)

// Bit e of word t: entry lo + 16 t + e is struck: tok[] are the tokens of this thread's nodes that are children of u, -1 else.  Ends with a barrier.
#define DRAW_NODES (1024 / DRAW_THREADS) /* nodes per thread */
static __device__ __forceinline__ void struck_bits(unsigned* bits, const int (&tok)[DRAW_NODES], int lo, int hi) {
    const int tid = threadIdx.x;
    __syncthreads();
    bits[tid] = 0;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < DRAW_NODES; ++k)
        if (tok[k] >= lo && tok[k] < hi) atomicOr(&bits[(tok[k] - lo) / DRAW_EACH], 1u << ((tok[k] - lo) % DRAW_EACH));
    __syncthreads();
}

// This thread's 16 logits of the block at lo (those at hi and beyond come as -inf: no weight).
static __device__ __forceinline__ void draw_load(const float* __restrict__ row, int lo, int hi, bool vec, float (&x)[DRAW_EACH]) {
    const int v = lo + threadIdx.x * DRAW_EACH;
    if (vec && v + DRAW_EACH <= hi) {
#pragma unroll
        for (int k = 0; k < DRAW_EACH / 4; ++k) {
            const f32x4 q = *(const f32x4*)(row + v + 4 * k);
#pragma unroll
            for (int e = 0; e < 4; ++e) x[4 * k + e] = q[e];
        }
    } else {
#pragma unroll
        for (int e = 0; e < DRAW_EACH; ++e) x[e] = v + e < hi ? row[v + e] : -INFINITY;
    }
}

// Running sum of v over the lanes, this lane's included.
static __device__ __forceinline__ uint64_t wave_scan_u64(uint64_t v) {
    const int lane = threadIdx.x & 63;
    for (int o = 1; o < 64; o <<= 1) {
        const uint64_t below = __shfl_up(v, o, FS_WAVE);
        if (lane >= o) v += below;
    }
    return v;
}

// draw: {target, workgroups that are done (0 before the launch), sums of the chunks}
__global__ void __launch_bounds__(DRAW_THREADS) sample_draw_kernel(const float* __restrict__ logits, int vocab, float inv_temp, bool vec, int chunk,
                                                                   const unsigned* __restrict__ rowm, const int32_t* __restrict__ token,
                                                                   const int32_t* __restrict__ parent, int T, AcceptResultDev* res,
                                                                   unsigned long long* draw) {
    __shared__ unsigned bits[DRAW_THREADS];
    __shared__ uint64_t shz[DRAW_THREADS / 64];
    __shared__ int s_last, s_x;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, chunks = gridDim.x;
    int par[DRAW_NODES], tok[DRAW_NODES];  // before anything is known of u: one round of memory latency less
#pragma unroll
    for (int k = 0; k < DRAW_NODES; ++k) {
        const int i = min(tid + k * DRAW_THREADS, T - 1);
        par[k] = parent[i];
        tok[k] = token[i];
    }
    const int n_acc = res->n_acc, u = SMP_PENDING - res->x_new;
    if (n_acc < 1 || u < 0) return;
#pragma unroll
    for (int k = 0; k < DRAW_NODES; ++k) tok[k] = par[k] == u && tid + k * DRAW_THREADS < T ? tok[k] : -1;
    const float* row = logits + (size_t)u * vocab;
    const float m = key_max(rowm[u]);
    auto weights = [&](int lo, int hi, float (&x)[DRAW_EACH], unsigned& b) {  // this thread's sum of the block at lo
        draw_load(row, lo, hi, vec, x);
        struck_bits(bits, tok, lo, hi);
        b = bits[tid];
        uint64_t z = 0;
#pragma unroll
        for (int e = 0; e < DRAW_EACH; ++e) z += (b >> e) & 1 ? 0 : exp_weight(__fmul_rn(x[e], inv_temp), m);
        return z;
    };
    float x[DRAW_EACH];
    unsigned b;
    uint64_t z = 0;
    for (int lo = blockIdx.x * chunk, c_hi = min(vocab, lo + chunk); lo < c_hi; lo += DRAW_BLOCK) z += weights(lo, min(c_hi, lo + DRAW_BLOCK), x, b);
    z = wave_sum_u64(z);
    if (lane == 0) shz[w] = z;
    __syncthreads();
    if (tid == 0) {
        for (int k = 1; k < DRAW_THREADS / 64; ++k) z += shz[k];
        __hip_atomic_store(&draw[2 + blockIdx.x], z, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        s_last = __hip_atomic_fetch_add(&draw[1], 1ull, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == (unsigned long long)(chunks - 1);
    }
    __syncthreads();
    if (!s_last) return;
    // the first chunk whose running sum exceeds the target (at most 64 chunks; every wave does the same)
    const uint64_t target = draw[0], own = lane < chunks ? __hip_atomic_load(&draw[2 + lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
    const uint64_t upto = wave_scan_u64(own);
    const unsigned long long hit = __ballot(lane < chunks && upto > target);
    int x_new = vocab - 1;  // the definition's default (no weight left)
    if (hit) {
        const int c = __ffsll(hit) - 1;
        uint64_t base = __shfl(upto - own, c, FS_WAVE);
        for (int lo = c * chunk, c_hi = min(vocab, lo + chunk); lo < c_hi; lo += DRAW_BLOCK) {
            if (tid == 0) s_x = -1;
            z = weights(lo, min(c_hi, lo + DRAW_BLOCK), x, b);
            const uint64_t run = wave_scan_u64(z);
            if (lane == 63) shz[w] = run;
            __syncthreads();
            uint64_t before = base;
#pragma unroll
            for (int k = 0; k < DRAW_THREADS / 64; ++k) {
                before += k < w ? shz[k] : 0;
                base += shz[k];
            }
            before += run - z;
            if (before <= target && target < before + z) {  // at most one thread
                int at = -1;
#pragma unroll
                for (int e = 0; e < DRAW_EACH; ++e) {
                    before += (b >> e) & 1 ? 0 : exp_weight(__fmul_rn(x[e], inv_temp), m);
                    if (at < 0 && before > target) at = e;
                }
                s_x = lo + tid * DRAW_EACH + at;
            }
            __syncthreads();
            if (s_x >= 0) {
                x_new = s_x;
                break;
            }
        }
    }
    if (tid == 0) res->x_new = x_new;
}

// Workgroups that share a row's statistics.  Up to 256 rows: about 512 in all, up to 1024 while they have 12288 elements each, at least 4096
// elements each and four to a row; twice to four times as many, smaller ones cost more to start than their loads take (us of a call without a
// draw, 2048 in all / so: x 152064 40 rows 38.0 / 28.1, 80 rows 41.1 / 36.5, 120 rows 44.8 / 42.6; x 152065, off 16 bytes, 40 rows 37.8 / 29.1,
// 120 rows 49.3 / 45.8).  More rows: about 2048 (1024 / 2048: 400 rows x 152064 98.3 / 96.2, x 100000 71.5 / 70.0, x 32000 38.0 / 35.4).  From
// four chunks on the three launches beat one workgroup per row (256 x 32000 30.0 / 30.8, 80 x 32000 22.7 / 25.1, 80 x 152064 36.5 / 81.3), with
// fewer they do not (600 x 32000, five chunks 44.1 / 42.3).
extern "C" int sample_chunks(int vocab, int n_ver) {
    const int smallest = (vocab + 4095) / 4096;
    if (n_ver > 256) return std::min(smallest, std::max(1, 2048 / n_ver));
    return std::min(smallest, std::max(std::max(512 / n_ver, std::min(1024 / n_ver, (vocab + 12287) / 12288)), 4));
}

hipError_t launch_accept_sample(const float* logits, int vocab, float inv_temp, const int32_t* token, const int32_t* parent, int T, int n_ver,
                                uint64_t seed, uint64_t step, AcceptResultDev* res, int32_t* retain, void* work, hipStream_t s) {
    unsigned* rowm = (unsigned*)work;
    unsigned long long* rowZ = (unsigned long long*)((char*)work + (((size_t)n_ver * sizeof(float) + 15) / 16) * 16);
    const bool vec = (vocab & 3) == 0 && ((uintptr_t)logits & 15) == 0;  // every row starts on 16 bytes
    if (n_ver > 0) {
        int chunks = sample_chunks(vocab, n_ver);
        if (chunks >= 4) {
            const int chunk = ((vocab + chunks - 1) / chunks + 3) & ~3;
            chunks = (vocab + chunk - 1) / chunk;
            hipLaunchKernelGGL(sample_clear_kernel, dim3((n_ver + 255) / 256), dim3(256), 0, s, rowm, rowZ, n_ver);
            const dim3 grid(chunks, n_ver), block(SMP_STAT_THREADS);
            hipLaunchKernelGGL(sample_max_kernel, grid, block, 0, s, logits, vocab, inv_temp, chunk, vec, rowm);
            hipLaunchKernelGGL(sample_sum_kernel, grid, block, 0, s, logits, vocab, inv_temp, chunk, vec, rowm, rowZ);
        } else {
            hipLaunchKernelGGL(sample_rowstats_kernel, dim3(n_ver), dim3(SMP_STAT_THREADS), 0, s, logits, vocab, inv_temp, vec, rowm, rowZ);
        }
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    // Residual draw in a launch of its own: its target, counter and the chunks' sums take the places of the row sums, which nobody needs
    // behind the walk.  From 12 chunks on, us of the whole call with the draw inside / outside of the walk: 16 rows x 50257 35.1 / 31.2, 40 rows x
    // 100000 47 / 36, 80 rows x 152064 66 / 48; a call without a draw pays 2 us for the empty launch.  A row sum's place holds one chunk's sum, so
    // 12 chunks also need 14 rows: that line is the scratch's, not a measured one, and with fewer rows the draw stays in the walk (24 us of
    // one compute unit for 152064 logits).
    const int draw_chunks = std::min(std::min((vocab + DRAW_BLOCK - 1) / DRAW_BLOCK, 64), n_ver - 2);
    const bool draw = draw_chunks >= 12;
    hipLaunchKernelGGL(accept_sample_kernel, dim3(1), dim3(SMP_THREADS), 0, s, logits, vocab, inv_temp, vec, rowm, rowZ, token, parent, T, n_ver, seed,
                       step, res, retain, draw ? rowZ : nullptr);
    if (draw) {
        const int chunk = ((vocab + draw_chunks - 1) / draw_chunks + DRAW_BLOCK - 1) / DRAW_BLOCK * DRAW_BLOCK, chunks = (vocab + chunk - 1) / chunk;
        hipLaunchKernelGGL(sample_draw_kernel, dim3(chunks), dim3(DRAW_THREADS), 0, s, logits, vocab, inv_temp, vec, chunk, rowm, token, parent, T, res, rowZ);
    }
    return hipGetLastError();
}
