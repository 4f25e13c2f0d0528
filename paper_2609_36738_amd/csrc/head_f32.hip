// fp32 head products on the matrix cores (v_mfma_f32_32x32x2_f32: exact fp32 products, fp32 sums):
//   dW = H^T G (+ beta dW),  dH = G W^T  with G_ij = [i in I] (alpha R_ij + cq_j) formed as R is staged,
//   Z = H W (+ b).
// Both VJP products run in one grid of 64 x 64 (or 32 x 32) output tiles, four waves each, k tiles of 32 through two LDS
// buffers with the next two tiles' words in registers. What bounds it: staging beside the matrix instructions. At N = 4096,
// d = 1024, V = 2000 it runs at 101 TFLOP/s; without the loads 110, without the LDS writes too 128, and the same
// fragment reads and products alone reach 153 of the 157 peak. At small sizes it is the waits of few tiles for their
// loads. Any size, leading dimension and alignment takes this path.
// Head VJP of a 1000-class head (N = 1024, d = 768): 51 us; the SIMT tiles that it replaces took 428 us there (two LDS
// words read per product, 7-15 TFLOP/s). Of small heads, in one launch: N = 256, d = 128, V = 10 23.1 -> 8.3 us in the trace;
// N = 64, d = 64, V = 4000 419 -> 15 us.
#include <algorithm>
#include <type_traits>

#include "common.hpp"
#include "kernels.hpp"

namespace bom {
namespace {

constexpr int TK = 32;          // k tile
constexpr int LDC = TK + 4;     // LDS pitch of a k-contiguous operand tile [TB][32]
constexpr int kF32MaxSplits = 64;

enum { kDH = 0, kDW = 1, kFWD = 2 };

struct F32Args {
    const float* H; int64_t ldh;
    const float* W; int64_t ldw;
    const float* R; int64_t ldr;      // the VJP's R, or the logits with row_lse
    const float* row_lse;
    const int32_t* labels; int32_t ig;
    const float* q_hat; const float* s; const int32_t* n_valid; float lambda;
    int N, d, V;
    float* dW; int64_t lddw; float beta;
    float* db;
    void* dH; int64_t lddh;
    const float* bias; float* Z; int64_t ldz;   // forward
    int tiles_w, splits_w, kps_w, tiles_h, splits_h, kps_h;   // tiles, k splits, k per split of dW (forward) and dH
    int flush_w;   // dW: products per partial sum (a multiple of 16)
    float* part_w; float* part_h;               // [splits][rows][columns] sums of a product that splits k
};

// TB x TB output tiles: 64, or 32 for products of few tiles (128, with waves of 64 x 64, measured no faster than 64:
// 331 against 332 us for N = 4096, d = 1024, V = 2000, and it fills the chip later).
template <int TB>
struct Stage {
    float a[2][TB * LDC];
    float b[2][TB * LDC];
};

// A chunk of four (from a multiple of four) across the end n >= 4 of its direction is read from n - 4 on: what its place x
// then holds (-1: nothing that an earlier chunk does not hold). Along k both operands place their words alike and the
// repeated ones are zeroed; along the output the epilogue stores a place's sum to the row or column that it came from.
__device__ __forceinline__ int moved(int x, int n) {
    const int c = x & ~3;
    if (c + 4 <= n) return x;
    const int r = n - 4 + (x & 3);
    return c < n && r >= c ? r : -1;
}

// One TB x TB tile over k in [kb, ke), each wave a quarter of it in one accumulator block: 32 x 32 with a step of the
// matrix instruction adding two k, or 16 x 16 with a step adding four (a quarter of the time per k that one tile takes
// alone). The G = 2 or 4 lane groups of a wave hold one k of a step each. With a k-contiguous operand these are k,
// k + 4, ... of a block of 4 G, so that a lane's four fragments are one 16-byte LDS read; dW takes them in the order of k.
// A k-outer tile [32][TB] has the columns of some rows rotated so that a wave's groups read all 64 banks.
// Sums of `flush` products at a time are added to the tile's total. dH: 512, so that the rounding error grows like the
// root of 512 and of K / 512 instead of the root of K. dW: see F32Plan.
template <int TB, int MODE, typename TO, bool ZR = false>
__device__ __forceinline__ void f32_tile(const F32Args& g, int tile, int z, Stage<TB>& sh) {
    static_assert(TB == 64 || (TB == 32 && MODE != kFWD), "tile sizes");
    constexpr int WB = TB / 2, G = kWave / WB, BK = 4 * G;   // block edge of a wave, lane groups, k per four steps
    constexpr int OCT = TB / 4, ORS = 256 / OCT;             // k-outer chunks per row, rows per pass of the workgroup
    typedef __attribute__((ext_vector_type(WB == 32 ? 16 : 4))) float acc_t;
    constexpr int NR = WB == 32 ? 16 : 4;
    constexpr bool KA = MODE != kDW;   // operand A k-contiguous (dH: G rows, forward: H rows); dW: H^T
    constexpr bool KB = MODE == kDH;   // operand B k-contiguous (W rows); else k-outer
    const int M = MODE == kDW ? g.d : g.N, Nn = MODE == kDH ? g.d : g.V, K = MODE == kDW ? g.N : MODE == kDH ? g.V : g.d;
    const float* A = MODE == kDH ? g.R : g.H;
    const float* B = MODE == kDW ? g.R : g.W;
    const int64_t lda = MODE == kDH ? g.ldr : g.ldh, ldb = MODE == kDW ? g.ldr : g.ldw;
    const int kps = MODE == kDW ? g.kps_w : MODE == kDH ? g.kps_h : K;
    const int tn = (Nn + TB - 1) / TB;
    const int m0 = (tile / tn) * TB, n0 = (tile % tn) * TB;
    const int kb = z * kps, ke = min(K, kb + kps);
    const int t = threadIdx.x, l = t % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(t / kWave);
    const int wm = wave / 2, wn = wave % 2;

    float alpha = 0.f;
    double cs = 0.0;
    if constexpr (MODE != kFWD) {
        const int nt = *g.n_valid;
        alpha = nt > 0 ? (float)((1.0 - (double)g.lambda) / (double)nt) : 0.f;
        cs = nt > 0 ? (double)g.lambda / (double)nt : 0.0;
    }
    // Each thread stages chunks of four elements along the contiguous direction: k-contiguous k = 4 (t % 8) .. + 3 of
    // rows t / 8 + 32 e, k-outer columns 4 (t % OCT) .. + 3 of rows k = t / OCT + ORS e. A chunk is one 16-byte load at any
    // 4-byte address inside the operand: see moved() for a chunk across an end. Rows past an end are clamped; they reach
    // only outputs that are not stored.
    const int ck = 4 * (t % 8), cr = t / 8, oc = 4 * (t % OCT), ok = t / OCT;
    constexpr int CH = TB * TK / 1024;   // chunks per thread and operand
    // chunk e of an operand whose rows (columns) start at x0 and end at `rows`; a product with an extent below four
    // loads words one by one
    const bool fast = min(min(M, Nn), K) >= 4;
    auto slot = [&](int x, int n) { return fast ? moved(x, n) : x < n ? x : -1; };
    auto load4 = [&](const float* X, int64_t ld, bool kcontig, int x0, int rows, int k0, int e) -> f32x4 {
        const int r = kcontig ? min(x0 + cr + 32 * e, rows - 1) : max(moved(k0 + ok + ORS * e, K), 0);
        const int c = kcontig ? min(k0 + ck, K - 4) : min(x0 + oc, rows - 4);
        return *reinterpret_cast<const f32x4_any_t*>(X + (int64_t)r * ld + c);
    };
    auto load1 = [&](const float* X, int64_t ld, bool kcontig, int x0, int rows, int k0, int e) {
        const int r = kcontig ? min(x0 + cr + 32 * e, rows - 1) : min(k0 + ok + ORS * e, K - 1);
        const int c = kcontig ? k0 + ck : x0 + oc, last = (kcontig ? K : rows) - 1;
        const float* p = X + (int64_t)r * ld;
        return f32x4{p[min(c, last)], p[min(c + 1, last)], p[min(c + 2, last)], p[min(c + 3, last)]};
    };
    // rows of G: label and lse. dH: this thread's rows, fixed over k; dW: lane i of every wave holds row k0 + i
    float lse_h[CH];
    int y_h[CH];
    f32x4 cq_w = {0.f, 0.f, 0.f, 0.f};
    auto valid = [&](int y) {
        bool bad = false;
        return label_valid(y, g.V, g.ig, &bad);
    };
    if constexpr (MODE == kDH) {
#pragma unroll
        for (int e = 0; e < CH; ++e) {
            const int i = min(m0 + cr + 32 * e, M - 1);
            y_h[e] = g.labels[i];
            lse_h[e] = ZR ? g.row_lse[i] : 0.f;
        }
    }
    if constexpr (MODE == kDW)
#pragma unroll
        for (int i = 0; i < 4; ++i) cq_w[i] = (float)(cs * (double)g.q_hat[max(slot(n0 + oc + i, Nn), 0)]);

    struct Set {   // one k tile in registers
        f32x4 xa[CH], xb[CH], q_k;
        float lse_k;
        int y_k;
    };
    auto load = [&](Set& x, int k0) {
        f32x4 (&xa)[CH] = x.xa, (&xb)[CH] = x.xb, &q_k = x.q_k;
        if constexpr (MODE == kDW) {
            const int k = max(slot(k0 + l % TK, K), 0);
            x.y_k = g.labels[k];
            if (ZR) x.lse_k = g.row_lse[k];
        }
        // one branch around all of the tile's loads, so that they are in flight together
        if (fast) {
#pragma unroll
            for (int e = 0; e < CH; ++e) {
                xa[e] = load4(A, lda, KA, m0, M, k0, e);
                xb[e] = load4(B, ldb, KB, n0, Nn, k0, e);
            }
            if constexpr (MODE == kDH) q_k = *reinterpret_cast<const f32x4_any_t*>(g.q_hat + min(k0 + ck, K - 4));
        } else {
#pragma unroll
            for (int e = 0; e < CH; ++e) {
                xa[e] = load1(A, lda, KA, m0, M, k0, e);
                xb[e] = load1(B, ldb, KB, n0, Nn, k0, e);
            }
            if constexpr (MODE == kDH)
#pragma unroll
                for (int i = 0; i < 4; ++i) q_k[i] = g.q_hat[min(k0 + ck + i, K - 1)];
        }
    };
    // four elements of G from R (or Z) of one row: row mask, label, lse, and cq of the four places from column j on
    auto g_of = [&](f32x4 r, bool row_valid, int y, float lse, f32x4 cq, int j) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float x = ZR ? r_from_z(r[i], lse * kLog2e, slot(j + i, g.V) == y) : r[i];
            r[i] = row_valid ? fmaf(alpha, x, cq[i]) : 0.f;
        }
        return r;
    };
    // row k and column c of a k-outer tile
    auto outer = [](int k, int c) {
        const int rot = MODE != kDW ? (k >> 2) & 1 : TB == 64 ? k & 1 : (k >> 1) & 1;
        return k * TB + (c ^ (rot * WB));
    };
    auto store = [&](const Set& x, int buf, int k0) {
        f32x4 cq_k = {0.f, 0.f, 0.f, 0.f};
        if constexpr (MODE == kDH)
#pragma unroll
            for (int i = 0; i < 4; ++i) cq_k[i] = (float)(cs * (double)x.q_k[i]);
        const bool tail = k0 + TK > ke;   // places past the end of k: zeros in both operands
#pragma unroll
        for (int e = 0; e < CH; ++e) {
            f32x4 a = x.xa[e], b = x.xb[e];
            if constexpr (MODE == kDH) a = g_of(a, valid(y_h[e]), y_h[e], lse_h[e], cq_k, k0 + ck);
            if constexpr (MODE == kDW) {   // this thread's row of G: ok + ORS e, held by that lane
                const int y = __shfl(x.y_k, ok + ORS * e, kWave);
                b = g_of(b, valid(y), y, ZR ? __shfl(x.lse_k, ok + ORS * e, kWave) : 0.f, cq_w, n0 + oc);
            }
            if (tail) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int ka = KA ? k0 + ck + i : k0 + ok + ORS * e, kk = KB ? k0 + ck + i : k0 + ok + ORS * e;
                    if (slot(ka, K) < 0 || (ka >= ke && ke < K)) a[i] = 0.f;
                    if (slot(kk, K) < 0 || (kk >= ke && ke < K)) b[i] = 0.f;
                }
            }
            *reinterpret_cast<f32x4*>(&sh.a[buf][KA ? (cr + 32 * e) * LDC + ck : outer(ok + ORS * e, oc)]) = a;
            *reinterpret_cast<f32x4*>(&sh.b[buf][KB ? (cr + 32 * e) * LDC + ck : outer(ok + ORS * e, oc)]) = b;
        }
    };
    auto frag = [&](const float* s, bool kcontig, int base, int blk, float (&f)[4]) {
        const int r = base + l % WB, h = l / WB;
        if (kcontig) {
            const f32x4 v = *reinterpret_cast<const f32x4*>(s + r * LDC + blk * BK + h * 4);
#pragma unroll
            for (int i = 0; i < 4; ++i) f[i] = v[i];
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) f[i] = s[outer(blk * BK + (MODE == kDW ? G * i + h : 4 * h + i), r)];
        }
    };
    const int flush = MODE == kDW ? g.flush_w : 512;
    acc_t acc, total;
#pragma unroll
    for (int r = 0; r < NR; ++r) acc[r] = total[r] = 0.f;
    // two k tiles in registers: tile j + 1 goes to the other LDS buffer after tile j's products, and tile j + 3 is loaded
    // into its registers
    Set sets[2];
    load(sets[0], kb);
    if (kb + TK < ke) load(sets[1], kb + TK);
    store(sets[0], 0, kb);
    if (kb + 2 * TK < ke) load(sets[0], kb + 2 * TK);
    __syncthreads();
    int since = 0;
    auto step = [&](int k0, int buf, Set& next) {
        const bool more = k0 + TK < ke;
#pragma unroll
        for (int blk = 0; blk < TK / BK; ++blk) {
            float fa[4], fb[4];
            frag(sh.a[buf], KA, wm * WB, blk, fa);
            frag(sh.b[buf], KB, wn * WB, blk, fb);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if constexpr (WB == 32) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[q], fb[q], acc, 0, 0, 0);
                else acc = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[q], fb[q], acc, 0, 0, 0);
            }
            if ((blk + 1) * BK % 16 == 0) {
                since += 16;
                if (since == flush || (blk == TK / BK - 1 && !more)) {
#pragma unroll
                    for (int r = 0; r < NR; ++r) {
                        total[r] += acc[r];
                        acc[r] = 0.f;
                    }
                    since = 0;
                }
            }
        }
        if (more) {
            store(next, buf ^ 1, k0 + TK);
            if (k0 + 3 * TK < ke) load(next, k0 + 3 * TK);
        }
        __syncthreads();
    };
    for (int k0 = kb; k0 < ke; k0 += 2 * TK) {
        step(k0, 0, sets[1]);
        if (k0 + TK < ke) step(k0 + TK, 1, sets[0]);
    }
    // accumulator element r of lane l: block row (r/4) 4G + (l/WB) 4 + r%4, block column l % WB
    const int splits = MODE == kDW ? g.splits_w : MODE == kDH ? g.splits_h : 1;
    const int nt = n0 + wn * WB + l % WB;
    const int n = KB ? (nt < Nn ? nt : -1) : slot(nt, Nn);
    if (n >= 0) {
        const float bn = MODE == kFWD && g.bias != nullptr ? g.bias[n] : 0.f;
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const int mt = m0 + wm * WB + (r / 4) * BK + (l / WB) * 4 + r % 4;
            const int m = KA ? (mt < M ? mt : -1) : slot(mt, M);
            if (m < 0) continue;
            if constexpr (MODE == kFWD) {
                g.Z[(int64_t)m * g.ldz + n] = total[r] + bn;
            } else if (splits > 1) {
                (MODE == kDW ? g.part_w : g.part_h)[((int64_t)z * M + m) * Nn + n] = total[r];
            } else if constexpr (MODE == kDW) {
                float* p = g.dW + (int64_t)m * g.lddw + n;
                *p = g.beta != 0.f ? total[r] + g.beta * *p : total[r];
            } else {
                TO* p = static_cast<TO*>(g.dH) + (int64_t)m * g.lddh + n;
                if constexpr (sizeof(TO) == 2) *p = f32_to_bf16(total[r]);
                else *p = total[r];
            }
        }
    }
    if constexpr (MODE == kDW) {   // the first row of tiles also writes db
        if (m0 == 0 && z == 0 && g.db != nullptr && t < TB && n0 + t < g.V) {
            const int j = n0 + t;
            g.db[j] = *g.n_valid > 0 ? (1.0f - g.lambda) * g.s[j] + g.lambda * g.q_hat[j] : 0.f;
        }
    }
}

// Unit of block `id` among n (workgroups go to the 8 XCDs in turn): each XCD takes a run of consecutive units, whose
// tiles share operand rows in its L2. Parts of a grid are padded to multiples of 8 blocks; n or more: no unit.
__device__ __forceinline__ int xcd_unit(int id, int n) { return (id % 8) * ((n + 7) / 8) + id / 8; }

// Blocks [0, tiles_w * splits_w), padded: dW's units; the rest dH's. A unit is (split, tile), tiles varying fastest.
template <int TB, typename TO, bool ZR>
__global__ __launch_bounds__(256) void vjp_f32_mfma_kernel(F32Args g) {
    __shared__ __attribute__((aligned(16))) Stage<TB> sh;
    const int uw = g.tiles_w * g.splits_w, bw = (uw + 7) / 8 * 8, uh = g.tiles_h * g.splits_h;
    if ((int)blockIdx.x < bw) {
        const int u = xcd_unit(blockIdx.x, uw);
        if (u < uw) f32_tile<TB, kDW, float, ZR>(g, u % g.tiles_w, u / g.tiles_w, sh);
    } else {
        const int u = xcd_unit((int)blockIdx.x - bw, uh);
        if (u < uh) f32_tile<TB, kDH, TO, ZR>(g, u % g.tiles_h, u / g.tiles_h, sh);
    }
}

__global__ __launch_bounds__(256) void forward_f32_mfma_kernel(F32Args g) {
    __shared__ __attribute__((aligned(16))) Stage<64> sh;
    const int u = xcd_unit(blockIdx.x, g.tiles_w);
    if (u < g.tiles_w) f32_tile<64, kFWD, float>(g, u, 0, sh);
}

// Sums of the k splits in split order, both products' in one launch: dW = sum_z part_w[z] (+ beta dW), dH = sum_z
// part_h[z]. A product that does not split k has no elements here.
template <typename TO>
__global__ __launch_bounds__(256) void f32_splits_kernel(F32Args g, int64_t nw, int64_t nh) {
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    float a = 0.f;
    if (idx < nw) {
        for (int z = 0; z < g.splits_w; ++z) a += g.part_w[z * nw + idx];
        float* p = g.dW + (idx / g.V) * g.lddw + idx % g.V;
        *p = g.beta != 0.f ? a + g.beta * *p : a;
    } else if (idx - nw < nh) {
        const int64_t k = idx - nw;
        for (int z = 0; z < g.splits_h; ++z) a += g.part_h[z * nh + k];
        TO* p = static_cast<TO*>(g.dH) + (k / g.d) * g.lddh + k % g.d;
        if constexpr (sizeof(TO) == 2) *p = f32_to_bf16(a);
        else *p = a;
    }
}

int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Tile size, the length of dH's k ranges (a power of two) and dW's split or not: those of the least modelled time. A CU
// takes its units at 20 ns per k of a 64 x 64 tile and 7.5 ns of a 32 x 32 one (the rates with several resident); a unit
// alone on its CU waits for its loads and its own steps, 30 and 15 ns per k; a unit's start and end take 0.6 us; splits
// add the partial sums' traffic and the reduction launch. Measured (N x d x V, tiles of 64 and of 32): 4096 x 1024 x 2000 336 and 483 us, 256 x 1024 x 1000
// 21.0 and 25.6, 1024 x 768 x 1000 50.7 and 50.5, 1024 x 128 x 10 36.5 and 20.3, 4096 x 64 x 10 23.9 and 15.9.
// dW's sums keep one order whatever the plan: `sums` partial sums of equal k ranges, each in the order of k, added in that
// order, either as that many units or as one unit that adds them itself. (The update divides by the gradient's own size
// plus 1e-8 in its first steps, so there the last bits of a small sum reach theta.)
struct F32Plan {
    int tb, splits_w = 1, kps_w, splits_h = 1, kps_h, flush_w;
};
F32Plan plan_f32(int64_t N, int64_t d, int64_t V, int sums) {
    const int64_t per = cdiv(cdiv(N, sums), 16) * 16;
    F32Plan best;
    double best_t = 1e300;
    for (int tb : {64, 32}) {
        const int64_t tw = cdiv(d, tb) * cdiv(V, tb), th = cdiv(N, tb) * cdiv(d, tb);
        for (int cut_w = 0; cut_w < (sums > 1 ? 2 : 1); ++cut_w) {
            for (int64_t len = (int64_t)1 << 31; len >= 128; len /= 2) {
                F32Plan p;
                p.tb = tb;
                p.flush_w = (int)per;
                p.splits_w = cut_w ? (int)cdiv(N, per) : 1;
                p.kps_w = cut_w ? (int)per : (int)N;
                p.splits_h = (int)std::min<int64_t>(kF32MaxSplits, cdiv(V, len));
                p.kps_h = (int)std::min<int64_t>(cdiv(cdiv(V, p.splits_h), TK) * TK, 0x7fffffff / TK * TK);
                p.splits_h = (int)cdiv(V, p.kps_h);
                const double work = (double)tw * N + (double)th * V;   // tile k steps
                const int64_t units = tw * p.splits_w + th * p.splits_h;
                const double per_cu = units < 1024 ? (double)cdiv(units, 256) * work / units : work / 256;
                const double longest = (double)std::max<int64_t>(p.kps_w, std::min<int64_t>(p.kps_h, V));
                double t = std::max(per_cu * (tb == 64 ? 20e-9 : 7.5e-9), longest * (tb == 64 ? 30e-9 : 15e-9));
                const double pw = p.splits_w > 1 ? (2.0 * p.splits_w + 1) * 4.0 * d * V : 0.0;
                const double ph = p.splits_h > 1 ? (2.0 * p.splits_h + 1) * 4.0 * N * d : 0.0;
                t += 0.6e-6 * (double)cdiv(units, 256);
                if (pw + ph > 0.0) t += (pw + ph) / 4e12 + 4e-6;
                if (t < best_t * 0.98) {
                    best_t = t;
                    best = p;
                }
            }
        }
    }
    return best;
}

}  // namespace

size_t vjp_f32_workspace_bytes(int64_t N, int64_t d, int64_t V, int sums) {
    const F32Plan p = plan_f32(N, d, V, sums);
    return align256(p.splits_w > 1 ? (size_t)p.splits_w * d * V * 4 : 0) +
           align256(p.splits_h > 1 ? (size_t)p.splits_h * N * d * 4 : 0);
}

hipError_t launch_vjp_f32_products(const HeadVjpArgs& a, int sums, void* part, hipStream_t st) {
    const F32Plan p = plan_f32(a.N, a.d, a.V, sums);
    F32Args g{};
    g.H = static_cast<const float*>(a.H);
    g.ldh = a.ldh;
    g.W = static_cast<const float*>(a.W);
    g.ldw = a.ldw;
    g.R = static_cast<const float*>(a.R);
    g.ldr = a.ldr;
    g.row_lse = a.is_residual ? nullptr : a.row_lse;
    g.labels = a.labels;
    g.ig = a.ignore_index;
    g.q_hat = a.q_hat;
    g.s = a.s;
    g.n_valid = a.n_valid;
    g.lambda = a.lambda;
    g.N = a.N;
    g.d = a.d;
    g.V = a.V;
    g.dW = static_cast<float*>(a.dW);
    g.lddw = a.lddw;
    g.beta = a.dW_beta;
    g.db = static_cast<float*>(a.db);
    g.dH = a.dH;
    g.lddh = a.lddh;
    const int64_t tw = cdiv(a.d, p.tb) * cdiv(a.V, p.tb), th = a.dH ? cdiv(a.N, p.tb) * cdiv(a.d, p.tb) : 0;
    g.tiles_w = (int)tw;
    g.splits_w = p.splits_w;
    g.kps_w = p.kps_w;
    g.flush_w = p.flush_w;
    g.tiles_h = (int)th;
    g.splits_h = p.splits_h;
    g.kps_h = p.kps_h;
    g.part_w = static_cast<float*>(part);
    g.part_h = reinterpret_cast<float*>(static_cast<char*>(part) +
                                        align256(p.splits_w > 1 ? (size_t)p.splits_w * a.d * a.V * 4 : 0));
    const int64_t units = cdiv(tw * p.splits_w, 8) * 8 + cdiv(th * p.splits_h, 8) * 8;
    if (units >= ((int64_t)1 << 31)) return hipErrorInvalidValue;
    const bool h16 = a.dH != nullptr && a.dh_dt == BOM_BF16;
    auto pick = [&](auto tb) {
        constexpr int TB = decltype(tb)::value;
        return a.is_residual ? (h16 ? vjp_f32_mfma_kernel<TB, uint16_t, false> : vjp_f32_mfma_kernel<TB, float, false>)
                             : (h16 ? vjp_f32_mfma_kernel<TB, uint16_t, true> : vjp_f32_mfma_kernel<TB, float, true>);
    };
    const auto kern = p.tb == 32 ? pick(std::integral_constant<int, 32>{}) : pick(std::integral_constant<int, 64>{});
    hipLaunchKernelGGL(kern, dim3((unsigned)units), dim3(256), 0, st, g);
    hipError_t e = hipGetLastError();
    const int64_t nw = p.splits_w > 1 ? (int64_t)a.d * a.V : 0, nh = a.dH && p.splits_h > 1 ? (int64_t)a.N * a.d : 0;
    if (e == hipSuccess && nw + nh > 0) {
        const auto red = h16 ? f32_splits_kernel<uint16_t> : f32_splits_kernel<float>;
        hipLaunchKernelGGL(red, dim3((unsigned)cdiv(nw + nh, 256)), dim3(256), 0, st, g, nw, nh);
        e = hipGetLastError();
    }
    return e;
}

hipError_t launch_forward_f32(const float* H, int64_t ldh, const float* W, int64_t ldw, const float* b, int N, int d,
                              int V, float* Z, int64_t ldz, hipStream_t st) {
    F32Args g{};
    g.H = H;
    g.ldh = ldh;
    g.W = W;
    g.ldw = ldw;
    g.bias = b;
    g.Z = Z;
    g.ldz = ldz;
    g.N = N;
    g.d = d;
    g.V = V;
    const int64_t tiles = cdiv(N, 64) * cdiv(V, 64);
    if (tiles >= ((int64_t)1 << 31)) return hipErrorInvalidValue;
    g.tiles_w = (int)tiles;
    hipLaunchKernelGGL(forward_f32_mfma_kernel, dim3((unsigned)(cdiv(tiles, 8) * 8)), dim3(256), 0, st, g);
    return hipGetLastError();
}

}  // namespace bom
