// Tile-grid products: the single-tile entry point and the tensor-level nnt_gemm,
// which turns a contraction of tiled tensors into a cached plan (tables of tasks,
// chunks and workgroups in device memory) and submits it to the executor.
#include "gemm_common.hpp"
#include "internal.hpp"

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <sstream>

namespace nnt {

// One macro-tile of C whose contraction was cut into k-slices: where the slices lie and where
// the sum goes.
struct SplitReduce {
    void* C;                // base of the C tile
    const float* bias;      // bias of the C tile (length m of the tile), or nullptr
    const float* ws;        // slice s of element (i, j) of the macro-tile at ws[s * slice + j * ldw + i]
    int64_t ldc, slice;
    int32_t m0, n0, rows, cols, ldw, nsplit;
    int64_t cin_off;        // the beta term is read at C + cin_off elements (0: C itself; else a residual input's tile)
};

typedef float f4_any __attribute__((ext_vector_type(4), aligned(4)));           // at any address of a float
typedef uint32_t u2_any __attribute__((ext_vector_type(2), aligned(2)));         // at any address of a bf16 element

template <typename TO>
__global__ void __launch_bounds__(256) splitk_reduce(const SplitReduce* tab, float alpha, float beta) {
    SplitReduce t = tab[blockIdx.y];
    t.ws = in_global(t.ws);
    t.bias = in_global(t.bias);
    const int q = t.ldw >> 2;
    const int idx = blockIdx.x * 256 + threadIdx.x;
    const int i = (idx % q) << 2, j = idx / q;
    if (j >= t.cols || i >= t.rows) return;
    const int n = t.rows - i < 4 ? t.rows - i : 4;
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    const float* p = t.ws + (int64_t)j * t.ldw + i;       // (16-byte aligned unless the macro-tile crosses an edge of C's tiles)
    // slices are added in their fixed order; four loads are started before the first of them is used
    int sl = 0;
    for (; sl + 4 <= t.nsplit; sl += 4) {
        f4_any v[4];
#pragma unroll
        for (int u = 0; u < 4; u++) v[u] = *reinterpret_cast<const f4_any*>(p + (int64_t)(sl + u) * t.slice);
#pragma unroll
        for (int u = 0; u < 4; u++) {
            acc[0] += v[u][0]; acc[1] += v[u][1]; acc[2] += v[u][2]; acc[3] += v[u][3];
        }
    }
    for (; sl < t.nsplit; sl++) {
        const f4_any v = *reinterpret_cast<const f4_any*>(p + (int64_t)sl * t.slice);
        acc[0] += v[0]; acc[1] += v[1]; acc[2] += v[2]; acc[3] += v[3];
    }
    TO* c = global_as<TO>(t.C) + (t.m0 + i) + (int64_t)(t.n0 + j) * t.ldc;
    if constexpr (sizeof(TO) == 4) {
        // four whole rows: one vector access instead of four, at any alignment
        if (n == 4) {
            f4_any o = {alpha * acc[0], alpha * acc[1], alpha * acc[2], alpha * acc[3]};
            if (t.bias) {
                const float* bp = t.bias + t.m0 + i;
                o[0] += bp[0]; o[1] += bp[1]; o[2] += bp[2]; o[3] += bp[3];
            }
            if (beta != 0.f) {
                const f4_any old = *reinterpret_cast<const f4_any*>(c + t.cin_off);
                o[0] += beta * old[0]; o[1] += beta * old[1]; o[2] += beta * old[2]; o[3] += beta * old[3];
            }
            *reinterpret_cast<f4_any*>(c) = o;
            return;
        }
    } else {
        if (n == 4) {
            float o[4];
            u2_any ow = {0u, 0u};
            if (beta != 0.f) ow = *reinterpret_cast<const u2_any*>(c + t.cin_off);
#pragma unroll
            for (int jj = 0; jj < 4; jj++) {
                o[jj] = alpha * acc[jj];
                if (t.bias) o[jj] += t.bias[t.m0 + i + jj];
                if (beta != 0.f) o[jj] += beta * __uint_as_float((jj & 1) ? (ow[jj >> 1] & 0xffff0000u) : (ow[jj >> 1] << 16));
            }
            uint32_t h[4];
#pragma unroll
            for (int jj = 0; jj < 4; jj++) {
                const __bf16 b = (__bf16)o[jj];
                h[jj] = (uint32_t)__builtin_bit_cast(uint16_t, b);
            }
            *reinterpret_cast<u2_any*>(c) = u2_any{h[0] | (h[1] << 16), h[2] | (h[3] << 16)};
            return;
        }
    }
    for (int jj = 0; jj < n; jj++) {
        float v = alpha * acc[jj];
        if (t.bias) v += t.bias[t.m0 + i + jj];
        if (beta != 0.f) {
            if constexpr (sizeof(TO) == 4) v += beta * (float)c[t.cin_off + jj];
            else v += beta * __uint_as_float((uint32_t)c[t.cin_off + jj] << 16);
        }
        if constexpr (sizeof(TO) == 4) c[jj] = v;
        else { const __bf16 h = (__bf16)v; c[jj] = __builtin_bit_cast(uint16_t, h); }
    }
}

struct GemmPlan {
    nnt_ctx* ctx = nullptr;
    uint64_t ids[5] = {0, 0, 0, 0, 0};         // tensors the tables point into (A, B, C, bias, residual input)
    int dtype_in = NNT_F32, dtype_out = NNT_F32;
    int akf = 0, bkf = 0, cfg = kCfgSquare;
    double flops = 0.0;                        // 2 m n k summed over tasks, chunks and batch members
    std::string label;                         // the kernel instance that runs the plan
    std::vector<GemmTask> tasks;
    std::vector<GemmChunk> chunks;
    std::vector<GemmWg> wgs, wgs_op;
    std::vector<int64_t> task_wg0;             // first workgroup of each task (+ total at the end)
    std::vector<int64_t> task_nfast;           // leading workgroups of each task that qualify for the direct-load kernel
    int64_t op_nfast = 0;                      // the same for the whole-operation order
    int64_t table_bytes = 0, ws_bytes = 0;     // device memory of the descriptor tables / the k-slice workspaces
    int epi_mode = 0;                          // GemmEpi mode of a product with an activation on its result path
    bool epi_ok = false;                       // every workgroup runs in a direct-load kernel that has that form
    bool dl_ragged = false;                    // they need the direct-load kernel's variant for ragged macro-tiles and short k-steps
    std::vector<int64_t> task_ctile;           // C tile index per task
    std::vector<std::vector<int64_t>> task_atiles, task_btiles;   // operand tiles per task (dependencies)
    std::vector<int64_t> task_bias_tile;
    GemmTask* d_tasks = nullptr;
    GemmChunk* d_chunks = nullptr;
    GemmWg* d_wgs = nullptr;
    GemmWg* d_wgs_op = nullptr;
    // Whole-operation launches may cut the contraction of some macro-tiles (the last `n_split`
    // of the launch order) into `splits` k-slices: each slice is a workgroup of its own that
    // writes raw fp32 sums to scratch memory, and a second kernel adds the slices in a fixed
    // order and applies alpha, beta and the bias.  The extra tasks and chunks of the slices
    // follow the regular ones in the same device tables.
    int splits = 1;
    int64_t n_split = 0, op_nwg = 0;
    int red_blocks = 0;
    int64_t slice_elems = 0;                   // elements of one slice of one cut macro-tile
    SplitReduce* d_red = nullptr;
    float* d_ws = nullptr;
    TileDep ws_dep;
    // Per-tile launches: a task that has only a few macro-tiles but a long contraction (a tile of a
    // weight gradient: 256 x 256 over all tokens) would leave the chip idle, so its contraction is cut
    // the same way, into its own scratch block (tasks of one operation run concurrently on several
    // streams), followed by the slice sum over just that task's macro-tiles.
    struct TileSplit { int64_t wg0 = 0, nwg = 0, nfast = 0, red0 = 0, nred = 0; };
    std::vector<TileSplit> tile_split;         // per task; nwg == 0: launched whole
    std::vector<GemmWg> wgs_ts;
    int64_t slice_elems_ts = 0;
    // Whole-operation launches of operands that only the register-staged kernels could read as they are: the operands are
    // laid out afresh in the context's pack space first and the macro-tiles lie on one grid over all of C, with tables of its own.  Such a plan has
    // nothing else: launches tile by tile of the same product have a plan to themselves.
    bool packed = false;
    PackOperand pack[2] = {};
    int pack_cfg = 0;
    std::shared_ptr<PackSpace> pack_space;
    char* d_pack_tables = nullptr;
    GemmArgs pack_args = {};
    const SplitReduce* pack_red = nullptr;
    int64_t pack_nwg = 0;
    GemmWg* d_wgs_ts = nullptr;
    SplitReduce* d_red_ts = nullptr;
    float* d_ws_ts = nullptr;
    ~GemmPlan() {
        for (void* p : {(void*)d_tasks, (void*)d_chunks, (void*)d_wgs, (void*)d_wgs_op, (void*)d_red, (void*)d_ws, (void*)d_wgs_ts,
                        (void*)d_red_ts, (void*)d_ws_ts, (void*)d_pack_tables})
            if (p) (void)hipFree(p);
    }
};

void plan_device_bytes(nnt_ctx* ctx, int64_t* tables, int64_t* workspaces) {
    for (const auto& kv : ctx->gemm_plans) {
        *tables += kv.second->table_bytes;
        *workspaces += kv.second->ws_bytes;
    }
}

void drop_plans_of(nnt_ctx* ctx, uint64_t id) {
    for (auto it = ctx->gemm_plans.begin(); it != ctx->gemm_plans.end();) {
        const uint64_t* ids = it->second->ids;
        if (ids[0] == id || ids[1] == id || ids[2] == id || ids[3] == id || ids[4] == id) it = ctx->gemm_plans.erase(it);
        else ++it;
    }
}

// The first `nfast` workgroups of the table qualify for the direct-load kernel of the type.
static int32_t launch_any(hipStream_t st, int dtype_in, int dtype_out, int akf, int bkf, int cfg,
                          const GemmArgs& g, int64_t nwg, int64_t nfast = 0, bool ragged = false, int epi_mode = 0) {
    const bool f32 = dtype_in == NNT_F32;
    if (epi_mode) {     // (plans with an activation form are only run when all their workgroups qualify: GemmPlan::epi_ok)
        if (nfast != nwg) return NNT_EINVAL;
        return f32 ? launch_gemm_f32_dl(st, akf, bkf, cfg, false, g, nwg, epi_mode) : NNT_EINVAL;
    }
    auto general = [&](const GemmArgs& ga, int64_t n) {
        return f32 ? launch_gemm_f32(st, akf, bkf, cfg, ga, n) : launch_gemm_bf16(st, dtype_out == NNT_F32, akf, bkf, cfg, ga, n);
    };
    // debugging aid: NNT_GEMM_NO_DL=1 sends every workgroup to the general kernels
    static const bool no_dl = getenv("NNT_GEMM_NO_DL") != nullptr;
    if (nfast <= 0 || no_dl) return general(g, nwg);
    int32_t rc = f32 ? launch_gemm_f32_dl(st, akf, bkf, cfg, ragged, g, nfast) : launch_gemm_bf16_dl(st, dtype_out == NNT_F32, akf, bkf, cfg, ragged, g, nfast);
    if (rc != NNT_OK || nfast == nwg) return rc;
    GemmArgs rest = g;
    if (rest.wgs) rest.wgs += nfast;
    return general(rest, nwg - nfast);
}

// Whether the direct-load kernels may read an operand: 16-byte aligned lines, and, as their lanes' byte offsets from the first
// element of a macro-tile have 32 bits, lines that lie close enough together: up to 128 fp32 (256 bf16) rows where k is the
// contiguous index, 32 k where it is not.  (The register-staged kernels address with 64 bits.)
static int vec_flag(const void* p, int64_t ld, int64_t stride, int elem, bool k_contiguous) {
    const int per = 16 / elem;
    return ((uintptr_t)p % 16 == 0) && (ld % per == 0) && (stride % per == 0) && ld <= (k_contiguous ? (int64_t)1 << 23 : ((int64_t)1 << 27) / elem);
}

// Workgroups are handed to the 8 XCDs (each with its own L2) in turn by their linear id, so the
// workgroups with id = x (mod 8) run on XCD x, about one per CU at a time.  The list arrives in
// tile order (rows fastest, then columns, batch members, tasks).  Each macro-tile grid is cut into
// blocks of 16 x 16 tiles; inside a block XCD x owns a sub-block of 8 x 4 tiles, so the workgroups
// that an XCD runs together need 8 + 4 operand panels instead of up to 33, and the eight XCDs
// together work on one compact 16 x 16 region whose panels meet in the last-level cache.  Small
// grids (batched attention products) go to one XCD each.  The per-XCD queues are then dealt out
// in turn; a queue that runs dry takes work from the longest one.
static void xcd_interleave(std::vector<GemmWg>& wgs, int bm, int bn) {
    const size_t n = wgs.size();
    if (n < 64) return;
    std::vector<GemmWg> q[8];
    int small_turn = 0;
    size_t a = 0;
    while (a < n) {
        size_t b = a;
        int gm = 0, gn = 0;
        while (b < n && wgs[b].task == wgs[a].task && wgs[b].batch == wgs[a].batch) {
            gm = std::max(gm, wgs[b].m0 / bm + 1);
            gn = std::max(gn, wgs[b].n0 / bn + 1);
            b++;
        }
        if ((size_t)gm * gn != b - a || gm * gn < 64) {
            // small or irregular grid: keep it together on one XCD
            std::vector<GemmWg>& dst = q[small_turn++ & 7];
            dst.insert(dst.end(), wgs.begin() + a, wgs.begin() + b);
        } else {
            for (int J = 0; J < gn; J += 16)
                for (int I = 0; I < gm; I += 16)
                    for (int x = 0; x < 8; x++)
                        for (int j = 0; j < 4; j++)
                            for (int i = 0; i < 8; i++) {
                                const int ii = I + (x & 1) * 8 + i, jj = J + (x >> 1) * 4 + j;
                                if (ii < gm && jj < gn) q[x].push_back(wgs[a + (size_t)jj * gm + ii]);
                            }
        }
        a = b;
    }
    std::vector<GemmWg> out;
    out.reserve(n);
    size_t head[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    while (out.size() < n) {
        for (int x = 0; x < 8 && out.size() < n; x++) {
            if (head[x] < q[x].size()) {
                out.push_back(q[x][head[x]++]);
            } else {
                int longest = 0;
                for (int y = 1; y < 8; y++)
                    if (q[y].size() - head[y] > q[longest].size() - head[longest]) longest = y;
                out.push_back(q[longest].back());
                q[longest].pop_back();
            }
        }
    }
    wgs.swap(out);
}

// Cost model for a product of whole matrices (no batch axes): picks the macro-tile shape, how many macro-tiles get
// their contraction cut into k-slices, and into how many.  A launch spreads its equal workgroups evenly over the 256
// compute units; `occ` of them fit on a unit at a time, and `us_k[c - 1]` is what a unit that holds c of them takes per
// unit of k, `t0` what a set of them takes besides (first loads, result stores), all in us as measured with
// nnt_tile_gemm on 16 to 1024 macro-tiles of k = 256, 1024 and 4096 (N N, T N and N T agree within 10 % in fp32 and in the
// direct-load bf16 kernels).  `occ` follows from each kernel's registers and LDS and has to be changed with them.  Large
// macro-tiles have the better rate on a full chip (fp32 128 x 128: 0.56 TFLOP/s per unit against 0.49 for 64 x 64; bf16
// 256 x 256: 4.6, 256 x 128: 4.2, 128 x 128: 3.1), small ones the shorter time where
// there are fewer macro-tiles than places: a unit with one 128 x 128 fp32 workgroup takes 62 ns per k, with one 64 x 64
// workgroup 24.  Cutting the contraction into s slices turns a launch (or its last, partial set) into 1/s of its length and adds
// a second pass over the fp32 partial sums: one more launch, about 6 us, and their bytes at 3.5 TB/s.
constexpr int kSplitStep = 64;
constexpr int64_t kMinSliceK = 128;
struct ShapeChoice { int cfg; int64_t n_split; int s; double us; };
struct ShapeCost { int cfg, occ; double us_k[4], t0; };
// `whole`: every macro-tile takes the direct-load kernels; `ragged`: their forms for edges and short k-steps; `general`:
// operands that only the register-staged kernels take (figures of odd leading dimensions).
enum ShapeKind { kShapeWhole = 0, kShapeRagged = 1, kShapeGeneral = 2 };
static const ShapeCost kCostF32[2][3] = {
    {{kCfgSquare, 2, {0.0625, 0.1180}, 5.0}, {kCfgMid, 2, {0.0345, 0.0630}, 3.0}, {kCfgSkinny64n64, 4, {0.0235, 0.0385, 0.0525, 0.0665}, 1.5}},
    {{kCfgSquare, 2, {0.130, 0.183}, 5.0}, {kCfgMid, 4, {0.0885, 0.112, 0.140, 0.170}, 3.0}, {kCfgSkinny64n64, 4, {0.046, 0.063, 0.079, 0.094}, 2.0}}};
static const ShapeCost kCostBf16[3][3] = {
    {{kCfgSquare, 1, {0.0285}, 15.0}, {kCfgTall, 2, {0.0195, 0.0312}, 5.0}, {kCfgWide, 2, {0.0130, 0.0212}, 4.0}},
    {{kCfgTall, 2, {0.0225, 0.0335}, 6.0}, {kCfgWide, 2, {0.0131, 0.0225}, 4.0}, {kCfgWide, 0, {}, 0.0}},       // (two shapes)
    {{kCfgTall, 1, {0.043}, 8.0}, {kCfgMid, 2, {0.035, 0.043}, 4.0}, {kCfgSkinny64n64, 4, {0.028, 0.030, 0.034, 0.037}, 1.5}}};
// A launch of X equal workgroups with a contraction of k: whole resident sets, then a last set spread over the units.
static double launch_us(const ShapeCost& cd, int64_t X, int64_t k) {
    const int64_t G = 256 * (int64_t)cd.occ, last = (X % G + 255) / 256;      // G: workgroups resident at a time
    return (double)(X / G) * (cd.us_k[cd.occ - 1] * (double)k + cd.t0) + (last ? cd.us_k[last - 1] * (double)k + cd.t0 : 0.0);
}
// What the register-staged kernel of a shape takes (bf16 128 x 128: one kernel for both wave layouts; 256 x 256: 60 ns per k
// where the operands reach it, 704 x 3192 over 1515, 24 of them).
static const ShapeCost& staged_cost(bool bf16, int cfg) {
    static const ShapeCost square = {kCfgSquare, 1, {0.060}, 8.0};
    const int shape = bf16 ? (cfg == kCfgWide ? kCfgMid : cfg) : (cfg == kCfgSkinny64n128 || cfg == kCfgResident ? kCfgMid : cfg);
    const ShapeCost* c = bf16 ? kCostBf16[kShapeGeneral] : kCostF32[1];
    for (int i = 0; i < 3; i++)
        if (c[i].cfg == shape) return c[i];
    return square;
}
// Whether a plan of which only some workgroups can take the direct-load kernel should run as two launches, one behind the
// other, or all on the register-staged kernel in one: by the longest contraction on either side.  Where neither fills
// the chip, the second launch costs its whole length again (fp32, 16 pairs of 128 x 261 over 261 on tiles of 128:
// 59 us in two launches, 34 in one).
static bool two_launches_pay(bool bf16, int cfg, bool ragged, int64_t n_fast, int64_t k_fast, int64_t n_rest, int64_t k_rest) {
    const int shape = !bf16 && (cfg == kCfgSkinny64n128 || cfg == kCfgResident) ? kCfgMid : cfg;
    const ShapeCost& staged = staged_cost(bf16, cfg);
    for (int i = 0; i < 3; i++) {
        const ShapeCost& fast = bf16 ? kCostBf16[ragged ? kShapeRagged : kShapeWhole][i] : kCostF32[0][i];
        if (fast.cfg == shape) return launch_us(fast, n_fast, k_fast) + launch_us(staged, n_rest, k_rest) < launch_us(staged, n_fast + n_rest, std::max(k_fast, k_rest));
    }
    return true;
}
// `act`: products with an activation on their result path, whose kernels exist for the two larger fp32 shapes.
static ShapeChoice choose_shape(bool bf16, ShapeKind kind, const std::vector<int64_t>& tm, const std::vector<int64_t>& tn,
                                const std::vector<int64_t>& ktot, bool may_split, bool act = false) {
    const ShapeCost* cands = bf16 ? kCostBf16[kind] : kCostF32[kind == kShapeGeneral];
    const int ncand = act ? 2 : 3;
    ShapeChoice best = {cands[0].cfg, 0, 1, 1e30};
    int64_t kmax = 0, kmin = INT64_MAX;
    for (int64_t kq : ktot) { kmax = std::max(kmax, kq); kmin = std::min(kmin, kq); }
    int64_t w_tall = 0, m_max = 0;
    for (int64_t mq : tm) m_max = std::max(m_max, mq);
    for (int ci = 0; ci < ncand; ci++) {
        const ShapeCost& cd = cands[ci];
        if (cd.occ == 0) continue;
        int bm, bn;
        gemm_cfg_tile(bf16, cd.cfg, &bm, &bn);
        const int64_t G = 256 * (int64_t)cd.occ;      // workgroups resident at a time
        int64_t W = 0;
        for (size_t i = 0; i < tm.size(); i++) W += ((tm[i] + bm - 1) / bm) * ((tn[i] + bn - 1) / bn);
        // Ragged bf16 products of tiles of more than 128 rows change to the 128 x 128 shape only below 40 macro-tiles of 256 x 128.
        // Alone it is often the faster one beyond that too (1200 x 2496 over 800: 24 us, 28; over 1165 random ones of 256 to 9000
        // rows and columns on tiles of 200 to 1000 by a tenth, with 16 to 17 ns per k and 6 us for it, which chunks of odd
        // lengths take), but twice the workgroups leave the products of the other stream no units: linear layers and
        // MLPs, forward and backward on two streams, 203 -> 184 us (872 wide), 86 -> 98 (1696 x 5952, 896 tokens),
        // 190 -> 205 (1280 wide, 1152 tokens).
        if (bf16 && kind == kShapeRagged) {
            if (ci == 0) w_tall = W;
            else if (m_max > 128 && w_tall >= 40) continue;
        }
        auto group_time = [&](int64_t X, int64_t k) { return launch_us(cd, X, k); };
        const double t_plain = group_time(W, kmax);
        if (t_plain < best.us) best = {cd.cfg, 0, 1, t_plain};
        if (!may_split) continue;
        const int64_t R = W % G;
        const int64_t ns_cands[2] = {W, (W > G && R > 0) ? R : 0};
        for (int64_t ns : ns_cands) {
            if (ns <= 0) continue;
            for (int sp = 2; sp <= 32; sp++) {
                const int64_t part = ((kmax + sp - 1) / sp + kSplitStep - 1) / kSplitStep * kSplitStep;
                if (part < kMinSliceK || part * (sp - 1) >= kmin) break;
                const double t = (ns < W ? group_time(W - ns, kmax) : 0.0) + group_time(ns * sp, part) + 6.0 +
                                 (double)ns * bm * bn * 4.0 * (sp + 1) / 3.5e6;
                if (t < best.us) best = {cd.cfg, ns, sp, t};
            }
        }
    }
    return best;
}

// Which configurations have a direct-load kernel, and which of those a form for macro-tiles that end inside their C
// tile and for chunks of any length (whether a chunk's length fits that form: whole vectors along k where an
// operand is k-contiguous; the bf16 form wants multiples of 8 throughout).
static bool has_direct_load(bool bf, int cfg) {
    if (bf) return cfg == kCfgSquare || cfg == kCfgTall || cfg == kCfgWide;
    return cfg == kCfgSquare || cfg == kCfgMid || cfg == kCfgSkinny64n128 || cfg == kCfgSkinny64n64 || cfg == kCfgResident;
}
static bool has_ragged(bool bf, int cfg) { return has_direct_load(bf, cfg) && !(bf && cfg == kCfgSquare); }
static bool ragged_k_ok(bool bf, bool akf, bool bkf, int64_t k) { return bf ? k % 8 == 0 : (k % 4 == 0 || (!akf && !bkf)); }
// What an m x n tile with a chunk of k needs (as if its macro-tiles were the largest of the type).
static ShapeKind shape_kind(bool bf, bool akf, bool bkf, int64_t m, int64_t n, int64_t k, bool aligned) {
    const int64_t t = bf ? 256 : 128, v = bf ? 8 : 4;
    if (aligned && m % t == 0 && n % t == 0 && k % (bf ? 64 : 32) == 0) return kShapeWhole;
    return aligned && ragged_k_ok(bf, akf, bkf, k) && (akf || m % v == 0) && (bkf || n % v == 0) ? kShapeRagged : kShapeGeneral;
}

// Products with batch axes (attention).  `kk`: both operands are k-contiguous (A read transposed, B as [k, n]).
// `kind`: what most of the work needs.
static int pick_cfg(int bf16, int64_t m_max, int64_t n_max, int64_t n_tiles_big, int64_t k_max, bool kk, ShapeKind kind) {
    // fp32 products whose whole contraction is a head size and whose result is score-shaped: bound by their result
    // stores, which a workgroup waits out before it ends, so the shape of which a compute unit holds three
    if (!bf16 && kk && k_max <= 64 && m_max >= 64 && n_max >= 128) return kCfgResident;
    // bf16 products with few rows (m = head size) read a score-shaped operand and are bound by that traffic: the
    // 128-row direct-load shape streams it four k-steps ahead
    if (bf16 && m_max <= 128) return kCfgWide;
    if (m_max <= 64) return kCfgSkinny64n128;
    if (bf16 && (n_max <= 128 || n_tiles_big < 256)) return kCfgWide;
    // short contractions are bound by the result stores: several small workgroups per compute
    // unit overlap one's stores with another's loads, one large workgroup cannot
    // (tiles that are not whole macro-tiles go to the ragged variant of that kernel: C4's tiles of 400 are 256 + 144 by 3 x 128 + 16)
    if (bf16 && k_max <= 128) return (m_max >= 256 && n_max >= 128) ? kCfgTall : kCfgWide;
    // the 256 x 256 shape has no direct-load form for edges (160 x 1152 over 1152, 64 of them: 163 us on its register-staged
    // kernel, 61 on the 256 x 128 one); of the register-staged kernels it is the better one (704 x 3192 over 1515, 24: 374 us, 473)
    if (bf16 && kind == kShapeRagged) return kCfgTall;
    return kCfgSquare;
}

}  // namespace nnt

using namespace nnt;

extern "C" int32_t nnt_tile_gemm(void* stream, int32_t dtype_in, int32_t dtype_out, int32_t opA, int32_t opB,
                                 int64_t m, int64_t n, int64_t k, int64_t batch, float alpha,
                                 const void* A, int64_t lda, int64_t strideA,
                                 const void* B, int64_t ldb, int64_t strideB,
                                 float beta, void* C, int64_t ldc, int64_t strideC) {
    if (dtype_in != NNT_F32 && dtype_in != NNT_BF16) return NNT_EDTYPE;
    if (dtype_out != NNT_F32 && dtype_out != NNT_BF16) return NNT_EDTYPE;
    if (dtype_in == NNT_F32 && dtype_out != NNT_F32) return NNT_EDTYPE;
    if ((opA != NNT_OP_N && opA != NNT_OP_T) || (opB != NNT_OP_N && opB != NNT_OP_T)) return NNT_EINVAL;
    if (m < 0 || n < 0 || k < 0 || batch < 0 || m > INT32_MAX || n > INT32_MAX || k > INT32_MAX) return NNT_EINVAL;
    if (m == 0 || n == 0 || batch == 0) return NNT_OK;
    if (!C || (k > 0 && (!A || !B))) return NNT_EINVAL;
    const int64_t a_rows = opA == NNT_OP_N ? m : k, b_rows = opB == NNT_OP_N ? k : n;
    if (ldc < m || (k > 0 && (lda < a_rows || ldb < b_rows))) return NNT_EINVAL;
    const int bf = dtype_in == NNT_BF16;
    const int elem = bf ? 2 : 4;
    GemmArgs g = {};
    g.wgs = nullptr;
    g.one_task = GemmTask{};
    g.one_task.C = C;
    g.one_task.bias = nullptr;
    g.one_task.ldc = ldc;
    g.one_task.strideC = strideC;
    g.one_task.m = (int32_t)m;
    g.one_task.n = (int32_t)n;
    g.one_task.chunk0 = 0;
    g.one_task.nchunk = k > 0 ? 1 : 0;
    g.one_chunk.A = A;
    g.one_chunk.B = B;
    g.one_chunk.lda = lda;
    g.one_chunk.ldb = ldb;
    g.one_chunk.strideA = strideA;
    g.one_chunk.strideB = strideB;
    g.one_chunk.k = (int32_t)k;
    g.one_chunk.vec_ok = vec_flag(A, lda, strideA, elem, opA == NNT_OP_T) | (vec_flag(B, ldb, strideB, elem, opB == NNT_OP_N) << 1);
    g.alpha = alpha;
    g.beta = beta;
    int bm, bn;
    const ShapeKind kind = shape_kind(bf, opA == NNT_OP_T, opB == NNT_OP_N, m, n, k, g.one_chunk.vec_ok == 3);
    int cfg = pick_cfg(bf, m, n, ((m + 255) / 256) * ((n + 255) / 256) * batch, k, opA == NNT_OP_T && opB == NNT_OP_N, kind);
    if (batch == 1 && cfg != kCfgResident) cfg = choose_shape(bf, kind, {m}, {n}, {k}, false).cfg;
    // debugging aid: NNT_TILE_GEMM_CFG=<number of a macro-tile configuration> overrides the choice for this entry point
    static const char* const force = getenv("NNT_TILE_GEMM_CFG");
    if (force) {      // (not kCfgResident: it exists for one operand form)
        const int f = atoi(force);
        if (f == kCfgSquare || f == kCfgMid || f == kCfgSkinny64n64 || (bf ? (f == kCfgTall || f == kCfgWide) : f == kCfgSkinny64n128)) cfg = f;
    }
    gemm_cfg_tile(bf, cfg, &bm, &bn);
    g.grid_m = (int32_t)((m + bm - 1) / bm);
    g.grid_n = (int32_t)((n + bn - 1) / bn);
    const int64_t nwg = (int64_t)g.grid_m * g.grid_n * batch;
    if (nwg > INT32_MAX) return NNT_EINVAL;
    const bool akf = opA == NNT_OP_T, bkf = opB == NNT_OP_N;
    bool ragged = !(m % bm == 0 && n % bn == 0 && k % ((bf && cfg == kCfgSquare) ? 64 : 32) == 0);
    const bool fast = k > 0 && has_direct_load(bf, cfg) && g.one_chunk.vec_ok == 3 &&
                      (!ragged || (has_ragged(bf, cfg) && (cfg != kCfgResident || k % 32 == 0) && ragged_k_ok(bf, akf, bkf, k) &&
                                   (akf || (m % bm) % (bf ? 8 : 4) == 0) && (bkf || (n % bn) % (bf ? 8 : 4) == 0)));
    return launch_any((hipStream_t)stream, dtype_in, dtype_out, opA == NNT_OP_T, opB == NNT_OP_N, cfg, g, nwg, fast ? nwg : 0, ragged);
}

// ---------------------------------------------------------------- tensor-level product
namespace {

struct AxisMap {
    std::vector<int> a_free, a_con, b_con, b_free, a_bat, b_bat;
};

int64_t prod_extent(const nnt_tensor* t, const int64_t* tc, const std::vector<int>& axes) {
    int64_t p = 1;
    for (int a : axes) p *= t->tile_extent(a, tc[a]);
    return p;
}

// Appends to P->chunks the chunks of `S` consecutive k-slices of task `t0` (slice lengths in multiples
// of the step the kernels want) and returns (first chunk, chunk count) per slice.
std::vector<std::pair<int32_t, int32_t>> cut_into_slices(GemmPlan* P, const GemmTask& t0, int64_t ktot, int S, int elem) {
    std::vector<std::pair<int32_t, int32_t>> ranges;
    const int64_t part = ((ktot + S - 1) / S + kSplitStep - 1) / kSplitStep * kSplitStep;
    int32_t q = t0.chunk0;
    int64_t used = 0;                       // k already consumed of chunk q
    for (int sidx = 0; sidx < S; sidx++) {
        const int32_t c0i = (int32_t)P->chunks.size();
        int64_t want = part;
        while (want > 0 && q < t0.chunk0 + t0.nchunk) {
            const GemmChunk c0 = P->chunks[q];
            const int64_t take = std::min<int64_t>(want, c0.k - used);
            GemmChunk c = c0;
            c.A = static_cast<const char*>(c0.A) + used * (P->akf ? 1 : c0.lda) * elem;
            c.B = static_cast<const char*>(c0.B) + used * (P->bkf ? 1 : c0.ldb) * elem;
            c.k = (int32_t)take;
            c.vec_ok = vec_flag(c.A, c.lda, c.strideA, elem, P->akf) | (vec_flag(c.B, c.ldb, c.strideB, elem, P->bkf) << 1);
            P->chunks.push_back(c);
            want -= take;
            used += take;
            if (used == c0.k) { q++; used = 0; }
        }
        ranges.push_back({c0i, (int32_t)P->chunks.size() - c0i});
    }
    return ranges;
}

// The slices of macro-tile `mw` of task `t0`: one partial task per slice, writing raw fp32 sums into
// `block` (slice after slice, bm x bn each), appended to P->tasks; their workgroups go to `by_slice`.
// Returns the record from which the slice-sum kernel finishes the macro-tile.
SplitReduce add_slice_tasks(GemmPlan* P, const GemmTask& t0, const GemmWg& mw, const std::vector<std::pair<int32_t, int32_t>>& ranges,
                            float* block, int bm, int bn, std::vector<std::vector<GemmWg>>& by_slice) {
    const int S = (int)ranges.size();
    const int64_t slice = (int64_t)bm * bn;
    SplitReduce r;
    r.C = t0.C; r.bias = t0.bias; r.ws = block; r.ldc = t0.ldc; r.slice = slice; r.cin_off = t0.cin_off;
    r.m0 = mw.m0; r.n0 = mw.n0;
    r.rows = std::min<int32_t>(bm, t0.m - mw.m0);
    r.cols = std::min<int32_t>(bn, t0.n - mw.n0);
    r.ldw = bm; r.nsplit = S;
    for (int sidx = 0; sidx < S; sidx++) {
        GemmTask t = t0;
        // element (m0 + i, n0 + j) of the "tile" lands on block[i + j * bm] of this slice
        t.C = block + (int64_t)sidx * slice - (mw.m0 + (int64_t)mw.n0 * bm);
        t.ldc = bm;
        t.strideC = 0;
        t.bias = nullptr;
        t.cin_off = 0;
        t.epi = 0;
        t.partial = 1;
        t.chunk0 = ranges[sidx].first;
        t.nchunk = ranges[sidx].second;
        by_slice[sidx].push_back(GemmWg{(int32_t)P->tasks.size(), mw.m0, mw.n0, 0});
        P->tasks.push_back(t);
    }
    return r;
}

// Launch order of k-slices: workgroup p runs on XCD p mod 8, and the workgroups of one k-slice read
// one k-range of both operands, so each slice is dealt to one XCD (slice s to XCD s mod 8): that XCD's
// L2 then fetches the range once for all macro-tiles.  An XCD whose queue runs dry takes from the
// longest one.
void deal_slices(const std::vector<std::vector<GemmWg>>& by_slice, std::vector<GemmWg>& out) {
    std::vector<GemmWg> q[8];
    for (size_t sidx = 0; sidx < by_slice.size(); sidx++) q[sidx & 7].insert(q[sidx & 7].end(), by_slice[sidx].begin(), by_slice[sidx].end());
    size_t head[8] = {0, 0, 0, 0, 0, 0, 0, 0}, left = 0;
    for (int x = 0; x < 8; x++) left += q[x].size();
    while (left > 0) {
        const int x = (int)(out.size() & 7);
        if (head[x] < q[x].size()) {
            out.push_back(q[x][head[x]++]);
        } else {
            int longest = 0;
            for (int y = 1; y < 8; y++)
                if (q[y].size() - head[y] > q[longest].size() - head[longest]) longest = y;
            out.push_back(q[longest].back());
            q[longest].pop_back();
        }
        left--;
    }
}

// Extents of the groups of tiles along `axes` of `t` taken together (first axis fastest), as first elements of the groups with the total
// at the end.
std::vector<int64_t> group_starts(const nnt_tensor* t, const std::vector<int>& axes) {
    int64_t n = 1;
    for (int a : axes) n *= t->grid[a];
    std::vector<int64_t> out(1, 0);
    for (int64_t i = 0; i < n; i++) {
        int64_t tc[kMaxDim] = {0, 0, 0, 0}, rem = i;
        for (int a : axes) { tc[a] = rem % t->grid[a]; rem /= t->grid[a]; }
        out.push_back(out.back() + prod_extent(t, tc, axes));
    }
    return out;
}

// The form of a product that lays its operands out afresh (GemmPlan::packed), if it can take the product and promises to take less than
// nine tenths of what the model says of them as they are (`as_is`, of `as_is_wgs` macro-tiles).  The copy, and a result path that sorts, are priced at
// 10 us (fp32) or 15 us (bf16) and 3 TB/s.  1217 random products of 128 to 5000 rows, columns and contraction on tiles of 256 to 1024, both forms
// of each timed: fp32 80 of 640 take the copy, 1.29 times faster, none slower (at 7 us 3 of 104 by up to 9 %; at 3.5 us 37 of 173 by up to
// 29 %, 1538 x 359 over 469 20 -> 24 us); bf16 57 of 577, 1.59 times (3204 x 3811 over 808 135 -> 45 us), none slower (at 10 us 7 of 73, by up to
// 42 %).  Layers of odd sizes, whose products overlap on two streams: 66 in fp32 the same within 0.5 % at any price from 6 us on, with the copy or without
// (1153 x 1337 over 648 tokens 113 -> 100 us at 8, others slower), 41 in bf16 6 % faster.
int32_t try_packed(nnt_ctx* ctx, const AxisMap& ax, nnt_tensor* A, nnt_tensor* B, nnt_tensor* C, nnt_tensor* bias, nnt_tensor* R, GemmPlan* P, const ShapeChoice& as_is,
                   int64_t as_is_wgs) {
    const bool bf = A->dtype == NNT_BF16;
    const int64_t elem = A->elem_size(), pad = bf ? 256 : 128;      // (pad: the most rows of a macro-tile)
    const std::vector<int>*contig[2] = {P->akf ? &ax.a_con : &ax.a_free, P->bkf ? &ax.b_con : &ax.b_free};
    if ((P->akf && !P->bkf) || contig[0]->size() != 1 || contig[1]->size() != 1) return NNT_OK;
    for (const nnt_tensor* t : {A, B, C})
        for (void* p : t->tiles) if (!p) return NNT_OK;
    const std::vector<int64_t> rows = group_starts(A, ax.a_free), cols = group_starts(B, ax.b_free), ks = group_starts(A, ax.a_con);
    const int64_t M = rows.back(), N = cols.back(), K = ks.back(), Kp = (K + 63) / 64 * 64;
    const int64_t Mp = (M + pad - 1) / pad * pad, Np = (N + pad - 1) / pad * pad;
    const int64_t a_elems = Mp * Kp, b_elems = Np * Kp;
    // (byte offsets of a macro-tile's lines and vector numbers have 32 bits)
    if (Kp > (1 << 23) || Mp > (1 << 23) || Np > (1 << 23) || a_elems > INT32_MAX || b_elems > INT32_MAX || (a_elems + b_elems) * elem > ((int64_t)2 << 30)) return NNT_OK;
    ShapeChoice sc = choose_shape(bf, kShapeWhole, {M}, {N}, {Kp}, true);
    int bm, bn;
    gemm_cfg_tile(bf, sc.cfg, &bm, &bn);
    const int64_t gm = (M + bm - 1) / bm, gn = (N + bn - 1) / bn;
    if (bf && C->dtype == NNT_F32 && sc.cfg != kCfgWide) {
        // The larger bf16 shapes have no registers to move partial sums to, so their fp32 results are cut into slices at least as the operands as
        // they are would have been (whole contractions in one chain instead: up to 1.8 times less exact, 4065 x 1211 over 2832 1.8e-7 -> 3.2e-7).
        const double cut0 = (double)as_is.n_split / (double)std::max<int64_t>(as_is_wgs, 1), cut1 = (double)sc.n_split / (double)(gm * gn);
        if (1.0 - cut1 + cut1 / sc.s > 1.0 - cut0 + cut0 / as_is.s) {
            const ShapeCost* cd = kCostBf16[kShapeWhole];
            while (cd->cfg != sc.cfg) cd++;
            sc.s = as_is.s;
            sc.n_split = std::min<int64_t>(gm * gn, (int64_t)std::ceil(cut0 * (double)(gm * gn)));
            const int64_t part = ((Kp + sc.s - 1) / sc.s + 63) / 64 * 64, uncut = gm * gn - sc.n_split;
            sc.us = (uncut > 0 ? launch_us(*cd, uncut, Kp) : 0.0) + launch_us(*cd, sc.n_split * sc.s, part) + 6.0 + (double)sc.n_split * bm * bn * 4.0 * (sc.s + 1) / 3.5e6;
        }
    }
    if (sc.us + (bf ? 15.0 : 10.0) + (double)(M + N) * K * 2.0 * elem / 3.0e6 >= 0.9 * as_is.us) return NNT_OK;
    if (sc.s > 1 && (sc.n_split * sc.s * bm * bn * (int64_t)sizeof(float) > ((int64_t)2 << 30) || sc.n_split > 65535 / 4)) return NNT_OK;

    // where the results of every macro-tile go: at most two tiles of C along either axis
    const int64_t NR = (int64_t)rows.size() - 1;
    const int64_t esize = C->elem_size();
    std::vector<GemmSpan> spans((size_t)(gm * gn));
    for (int64_t j = 0, cb = 0; j < gn; j++) {
        while (j * bn >= cols[cb + 1]) cb++;
        const int64_t j1 = std::min(N, (j + 1) * bn);
        if (j1 > cols[cb + 1] && j1 > cols[cb + 2]) return NNT_OK;
        for (int64_t i = 0, ra = 0; i < gm; i++) {
            while (i * bm >= rows[ra + 1]) ra++;
            const int64_t i1 = std::min(M, (i + 1) * bm);
            if (i1 > rows[ra + 1] && i1 > rows[ra + 2]) return NNT_OK;
            GemmSpan& s = spans[(size_t)(i + j * gm)];
            s = GemmSpan{};
            s.rows = (int32_t)(i1 - i * bm);
            s.cols = (int32_t)(j1 - j * bn);
            s.sm = i1 > rows[ra + 1] ? (int32_t)(rows[ra + 1] - i * bm) : INT32_MAX;
            s.sn = j1 > cols[cb + 1] ? (int32_t)(cols[cb + 1] - j * bn) : INT32_MAX;
            for (int a = 0; a < 2; a++) {
                const int64_t r = ra + (a && s.sm != INT32_MAX);
                s.ldc[a] = rows[r + 1] - rows[r];
                if (bias) s.bias[a] = static_cast<const float*>(bias->tiles[r]) + (i * bm - rows[r]);
                if (bias && !bias->tiles[r]) return NNT_OK;
                for (int b = 0; b < 2; b++) {
                    const int64_t c = cb + (b && s.sn != INT32_MAX), t = r + NR * c;
                    s.C[a + 2 * b] = static_cast<char*>(C->tiles[t]) + ((i * bm - rows[r]) + (j * bn - cols[c]) * s.ldc[a]) * esize;
                    if (R) {
                        const ptrdiff_t delta = static_cast<const char*>(R->tiles[t]) - static_cast<const char*>(C->tiles[t]);
                        if (!R->tiles[t] || delta % esize != 0) return NNT_OK;
                        s.cin[a + 2 * b] = delta / esize;
                    }
                }
            }
        }
    }

    // the operands
    std::vector<int32_t> line0;
    const std::vector<int64_t>* lines[2] = {P->akf ? &rows : &ks, P->bkf ? &cols : &ks};
    for (const std::vector<int64_t>* l : lines) line0.insert(line0.end(), l->begin(), l->end());
    const int64_t cut_part = ((Kp + sc.s - 1) / sc.s + 63) / 64 * 64, n_cut = sc.s > 1 ? std::min<int64_t>(sc.n_split, gm * gn) : 0;
    const int S = n_cut > 0 ? (int)((Kp + cut_part - 1) / cut_part) : 1;
    const int64_t slice = (int64_t)bm * bn;
    // (where there is no memory for them the product runs on the operands as they are; four floats more: the sum reads whole vectors, also of
    // parts that do not begin at one)
    const size_t cut_bytes = n_cut > 0 ? ((size_t)n_cut * S * slice + 4) * sizeof(float) : 0;
    auto none = [&]() {
        (void)hipGetLastError();
        for (void* p : {(void*)P->d_ws, (void*)P->d_pack_tables}) if (p) (void)hipFree(p);
        P->d_ws = nullptr;
        P->d_pack_tables = nullptr;
        P->pack_space.reset();
        return (int32_t)NNT_OK;
    };
    const int32_t src = share_pack_space(ctx, (a_elems + b_elems) * elem, &P->pack_space);
    if (src != NNT_OK) return src;
    if (!P->pack_space || (cut_bytes && hipMalloc((void**)&P->d_ws, cut_bytes) != hipSuccess)) return none();
    for (int o = 0; o < 2; o++) {
        nnt_tensor* const t = o ? B : A;
        const bool kf = o ? P->bkf : P->akf;
        const int64_t free_pad = o ? Np : Mp;
        const int cx = (*contig[o])[0];
        PackOperand& p = P->pack[o];
        p.tiles = t->d_tiles;
        p.dst = (void*)(o ? a_elems * elem : 0);      // (an offset, as the chunks' are: which stream's part it is, a launch knows)
        p.ntc = (int32_t)t->grid[cx];
        p.ntl = (int32_t)lines[o]->size() - 1;
        p.base = (int32_t)t->base[cx];
        p.contig = (int32_t)t->shape[cx];
        p.pitch = (int32_t)(kf ? Kp : free_pad);
        p.lines = (int32_t)lines[o]->back();
        p.all_lines = kf ? p.lines : (int32_t)Kp;      // (lines of rows that do not exist are read, but only reach results that are not stored)
    }

    // tasks: the product, and one per k-slice of every macro-tile that is cut
    GemmChunk whole = {};
    whole.A = P->pack[0].dst;
    whole.B = P->pack[1].dst;
    whole.lda = P->pack[0].pitch;
    whole.ldb = P->pack[1].pitch;
    whole.k = (int32_t)Kp;
    whole.vec_ok = 3;
    std::vector<GemmChunk> chunks(1, whole);
    GemmTask main = {};
    main.m = (int32_t)M;
    main.n = (int32_t)N;
    main.nchunk = 1;
    std::vector<GemmTask> tasks(1, main);
    std::vector<GemmWg> wgs;
    std::vector<SplitReduce> red;
    for (int64_t j = 0; j < gn; j++)
        for (int64_t i = 0; i < gm; i++) wgs.push_back(GemmWg{0, (int32_t)(i * bm), (int32_t)(j * bn), 0});
    xcd_interleave(wgs, bm, bn);
    if (n_cut > 0) {
        const int64_t part = cut_part;
        for (int q = 0; q < S; q++) {
            GemmChunk c = whole;
            c.A = (const void*)((intptr_t)whole.A + q * part * (P->akf ? 1 : whole.lda) * elem);
            c.B = (const void*)((intptr_t)whole.B + q * part * (P->bkf ? 1 : whole.ldb) * elem);
            c.k = (int32_t)std::min(part, Kp - q * part);
            chunks.push_back(c);
        }
        const std::vector<GemmWg> cut(wgs.end() - n_cut, wgs.end());
        wgs.resize(wgs.size() - (size_t)n_cut);
        std::vector<std::vector<GemmWg>> by_slice(S);
        for (int64_t w = 0; w < n_cut; w++) {
            const GemmWg& mw = cut[(size_t)w];
            float* const block = P->d_ws + w * S * slice;
            for (int q = 0; q < S; q++) {
                GemmTask t = main;
                t.C = block + q * slice - (mw.m0 + (int64_t)mw.n0 * bm);
                t.ldc = bm;
                t.partial = 1;
                t.chunk0 = 1 + q;
                by_slice[q].push_back(GemmWg{(int32_t)tasks.size(), mw.m0, mw.n0, 0});
                tasks.push_back(t);
            }
            const GemmSpan& s = spans[(size_t)(mw.m0 / bm + (mw.n0 / bn) * gm)];
            const int32_t ie[3] = {0, std::min(s.sm, s.rows), s.rows}, je[3] = {0, std::min(s.sn, s.cols), s.cols};
            for (int b = 0; b < 2; b++)
                for (int a = 0; a < 2; a++) {
                    if (ie[a + 1] == ie[a] || je[b + 1] == je[b]) continue;
                    SplitReduce r = {};
                    r.C = s.C[a + 2 * b];
                    r.bias = s.bias[a];
                    r.ws = block + ie[a] + (int64_t)je[b] * bm;
                    r.ldc = s.ldc[a];
                    r.slice = slice;
                    r.m0 = ie[a];
                    r.n0 = je[b];
                    r.rows = ie[a + 1] - ie[a];
                    r.cols = je[b + 1] - je[b];
                    r.ldw = bm;
                    r.nsplit = S;
                    r.cin_off = s.cin[a + 2 * b];
                    red.push_back(r);
                }
        }
        deal_slices(by_slice, wgs);
    }
    // all tables in one piece: an allocation and a copy cost some 15 us each in the first call on new tensors
    std::vector<char> blob;
    auto put = [&](const void* h, size_t bytes) {
        const size_t at = (blob.size() + 15) / 16 * 16;
        blob.resize(at + bytes);
        if (bytes) memcpy(blob.data() + at, h, bytes);
        return at;
    };
    const size_t at_lines = put(line0.data(), line0.size() * sizeof(int32_t)), at_red = put(red.data(), red.size() * sizeof(SplitReduce)),
                 at_spans = put(spans.data(), spans.size() * sizeof(GemmSpan)), at_tasks = put(tasks.data(), tasks.size() * sizeof(GemmTask)),
                 at_chunks = put(chunks.data(), chunks.size() * sizeof(GemmChunk)), at_wgs = put(wgs.data(), wgs.size() * sizeof(GemmWg));
    if (hipMalloc((void**)&P->d_pack_tables, blob.size()) != hipSuccess) return none();
    NNT_HIP(ctx, hipMemcpy(P->d_pack_tables, blob.data(), blob.size(), hipMemcpyHostToDevice));
    P->table_bytes += (int64_t)blob.size();
    P->ws_bytes += (int64_t)cut_bytes;
    if (n_cut > 0) {
        P->splits = S;
        P->n_split = (int64_t)red.size();
        P->slice_elems = slice * n_cut / (int64_t)red.size();
        P->red_blocks = (int)((slice / 4 + 255) / 256);
    }
    const int32_t* const d_lines = reinterpret_cast<const int32_t*>(P->d_pack_tables + at_lines);
    P->pack[0].line0 = d_lines;
    P->pack[1].line0 = d_lines + lines[0]->size();
    P->pack_red = reinterpret_cast<const SplitReduce*>(P->d_pack_tables + at_red);
    P->pack_args.spans = reinterpret_cast<const GemmSpan*>(P->d_pack_tables + at_spans);
    P->pack_args.tasks = reinterpret_cast<const GemmTask*>(P->d_pack_tables + at_tasks);
    P->pack_args.chunks = reinterpret_cast<const GemmChunk*>(P->d_pack_tables + at_chunks);
    P->pack_args.wgs = reinterpret_cast<const GemmWg*>(P->d_pack_tables + at_wgs);
    P->pack_args.grid_m = (int32_t)gm;
    P->pack_cfg = sc.cfg;
    P->pack_nwg = (int64_t)wgs.size();
    P->packed = true;
    return NNT_OK;
}

// `view_ld` (or nullptr): per operand (A, B, C) the leading dimension of a tensor that is a window on a tensor
// with the heads side by side along its first axis (see nnt_gemm_heads), or 0 for an ordinary tensor.  With it
// the two batch axes stay apart (batch member, head): GemmTask::nb1 and the second strides.
int32_t build_plan(nnt_ctx* ctx, int opA, nnt_tensor* A, int opB, nnt_tensor* B, nnt_tensor* C, int ncon, int nbat,
                   nnt_tensor* bias, nnt_tensor* R, GemmPlan* P, const int64_t* view_ld = nullptr, int epi = 0) {
    const bool pairs = view_ld != nullptr;
    if (epi && (nbat != 0 || !R || pairs)) return fail(ctx, NNT_EINVAL, "nnt_gemm_gelu: unsupported form");
    if (pairs && (nbat != 2 || ncon != 1 || bias || R)) return fail(ctx, NNT_EINVAL, "nnt_gemm_heads: unsupported form");
    const int na = A->ndim - nbat, nb = B->ndim - nbat;
    if (ncon < 1 || nbat < 0 || na < ncon || nb < ncon)
        return fail(ctx, NNT_EINVAL, "nnt_gemm: axis counts do not fit the operands");
    AxisMap ax;
    if (opA == NNT_OP_N) { for (int i = 0; i < na - ncon; i++) ax.a_free.push_back(i); for (int i = na - ncon; i < na; i++) ax.a_con.push_back(i); }
    else { for (int i = 0; i < ncon; i++) ax.a_con.push_back(i); for (int i = ncon; i < na; i++) ax.a_free.push_back(i); }
    if (opB == NNT_OP_N) { for (int i = 0; i < ncon; i++) ax.b_con.push_back(i); for (int i = ncon; i < nb; i++) ax.b_free.push_back(i); }
    else { for (int i = 0; i < nb - ncon; i++) ax.b_free.push_back(i); for (int i = nb - ncon; i < nb; i++) ax.b_con.push_back(i); }
    for (int i = 0; i < nbat; i++) { ax.a_bat.push_back(na + i); ax.b_bat.push_back(nb + i); }
    const int nfa = (int)ax.a_free.size(), nfb = (int)ax.b_free.size();
    if (C->ndim != nfa + nfb + nbat) return fail(ctx, NNT_EINVAL, "nnt_gemm: C has the wrong number of axes");
    for (int i = 0; i < ncon; i++)
        if (A->shape[ax.a_con[i]] != B->shape[ax.b_con[i]] || A->base[ax.a_con[i]] != B->base[ax.b_con[i]])
            return fail(ctx, NNT_EINVAL, "nnt_gemm: contracted axes differ in extent or tiling");
    for (int i = 0; i < nfa; i++)
        if (A->shape[ax.a_free[i]] != C->shape[i] || A->base[ax.a_free[i]] != C->base[i])
            return fail(ctx, NNT_EINVAL, "nnt_gemm: free axes of A and C differ in extent or tiling");
    for (int i = 0; i < nfb; i++)
        if (B->shape[ax.b_free[i]] != C->shape[nfa + i] || B->base[ax.b_free[i]] != C->base[nfa + i])
            return fail(ctx, NNT_EINVAL, "nnt_gemm: free axes of B and C differ in extent or tiling");
    for (int i = 0; i < nbat; i++) {
        const int ca = nfa + nfb + i;
        if (A->shape[ax.a_bat[i]] != C->shape[ca] || A->base[ax.a_bat[i]] != C->base[ca] ||
            B->shape[ax.b_bat[i]] != C->shape[ca] || B->base[ax.b_bat[i]] != C->base[ca])
            return fail(ctx, NNT_EINVAL, "nnt_gemm: batch axes differ in extent or tiling");
    }
    if (A->dtype != B->dtype) return fail(ctx, NNT_EDTYPE, "nnt_gemm: A and B must have one element type");
    if (A->dtype == NNT_F32 && C->dtype != NNT_F32) return fail(ctx, NNT_EDTYPE, "nnt_gemm: fp32 operands need an fp32 result");
    if (bias) {
        if (bias->dtype != NNT_F32 || bias->ndim != 1 || nfa != 1 || bias->shape[0] != C->shape[0] || bias->base[0] != C->base[0])
            return fail(ctx, NNT_EINVAL, "nnt_gemm: bias must be an fp32 vector tiled like C's first axis");
    }

    P->ctx = ctx;
    P->ids[0] = A->id; P->ids[1] = B->id; P->ids[2] = C->id; P->ids[3] = bias ? bias->id : 0; P->ids[4] = R ? R->id : 0;
    P->dtype_in = A->dtype;
    P->dtype_out = C->dtype;
    P->akf = opA == NNT_OP_T;
    P->bkf = opB == NNT_OP_N;
    const int elem = A->dtype == NNT_BF16 ? 2 : 4;

    // contracted tile grid
    int64_t ncon_tiles = 1;
    for (int i = 0; i < ncon; i++) ncon_tiles *= A->grid[ax.a_con[i]];
    int64_t m_max = 0, n_max = 0, big = 0;

    struct TaskGeom { int64_t m, n, batch; };
    std::vector<TaskGeom> geom;
    for (int64_t ci = 0; ci < C->ntiles; ci++) {
        if (!C->tiles[ci]) continue;
        int64_t cc[kMaxDim], ac[kMaxDim] = {0, 0, 0, 0}, bc[kMaxDim] = {0, 0, 0, 0};
        C->tile_coords(ci, cc);
        for (int i = 0; i < nfa; i++) ac[ax.a_free[i]] = cc[i];
        for (int i = 0; i < nfb; i++) bc[ax.b_free[i]] = cc[nfa + i];
        for (int i = 0; i < nbat; i++) { ac[ax.a_bat[i]] = cc[nfa + nfb + i]; bc[ax.b_bat[i]] = cc[nfa + nfb + i]; }
        const int64_t m = prod_extent(A, ac, ax.a_free), n = prod_extent(B, bc, ax.b_free);
        const int64_t batch = prod_extent(A, ac, ax.a_bat);
        if (m > INT32_MAX || n > INT32_MAX) return fail(ctx, NNT_EINVAL, "nnt_gemm: tile too large");
        GemmTask t = {};
        t.C = C->tiles[ci];
        t.bias = bias ? static_cast<const float*>(bias->tiles[cc[0]]) : nullptr;
        if (bias && !t.bias) return fail(ctx, NNT_EINVAL, "nnt_gemm: bias tile missing");
        if (R) {
            // the beta term of this tile comes from the residual input's tile: same geometry, so one offset does
            const ptrdiff_t delta = static_cast<const char*>(R->tiles[ci]) - static_cast<const char*>(C->tiles[ci]);
            if (delta % (ptrdiff_t)C->elem_size() != 0) return fail(ctx, NNT_EINVAL, "nnt_gemm_res: residual tile not aligned to the element size");
            t.cin_off = delta / (ptrdiff_t)C->elem_size();
            t.epi = epi;
        }
        t.ldc = (pairs && view_ld[2]) ? view_ld[2] : m;
        t.strideC = t.ldc * n;
        int64_t nb1 = 0;
        if (pairs) {
            nb1 = C->tile_extent(nfa + nfb, cc[nfa + nfb]);         // batch members of the tile; the heads follow
            t.nb1 = (int32_t)nb1;
            t.strideC2 = view_ld[2] ? m : t.strideC * nb1;           // a window keeps head hl at rows hl * h .. of its tile
        }
        t.m = (int32_t)m;
        t.n = (int32_t)n;
        t.chunk0 = (int32_t)P->chunks.size();
        std::vector<int64_t> atl, btl;
        for (int64_t l = 0; l < ncon_tiles; l++) {
            int64_t rem = l;
            for (int i = 0; i < ncon; i++) {
                const int64_t gi = A->grid[ax.a_con[i]];
                ac[ax.a_con[i]] = rem % gi;
                bc[ax.b_con[i]] = rem % gi;
                rem /= gi;
            }
            const int64_t ai = A->tile_index(ac), bi = B->tile_index(bc);
            if (!A->tiles[ai] || !B->tiles[bi]) continue;      // structural zeros: no contribution
            const int64_t k = prod_extent(A, ac, ax.a_con);
            GemmChunk ch = {};
            ch.A = A->tiles[ai];
            ch.B = B->tiles[bi];
            ch.lda = (pairs && view_ld[0]) ? view_ld[0] : (P->akf ? k : m);
            ch.ldb = (pairs && view_ld[1]) ? view_ld[1] : (P->bkf ? k : n);
            ch.strideA = ch.lda * (P->akf ? m : k);
            ch.strideB = ch.ldb * (P->bkf ? n : k);
            ch.k = (int32_t)k;
            if (pairs) {
                // the first axis of a window is the head size: m of A (k when A is read transposed), k of B (n when transposed)
                ch.strideA2 = view_ld[0] ? (P->akf ? k : m) : ch.strideA * nb1;
                ch.strideB2 = view_ld[1] ? (P->bkf ? k : n) : ch.strideB * nb1;
            }
            ch.vec_ok = (vec_flag(ch.A, ch.lda, ch.strideA, elem, P->akf) && ch.strideA2 % (16 / elem) == 0 ? 1 : 0) |
                        (vec_flag(ch.B, ch.ldb, ch.strideB, elem, P->bkf) && ch.strideB2 % (16 / elem) == 0 ? 2 : 0);
            P->chunks.push_back(ch);
            atl.push_back(ai);
            btl.push_back(bi);
        }
        t.nchunk = (int32_t)P->chunks.size() - t.chunk0;
        for (int32_t q = t.chunk0; q < t.chunk0 + t.nchunk; q++) P->flops += 2.0 * m * n * P->chunks[q].k * batch;
        P->tasks.push_back(t);
        P->task_ctile.push_back(ci);
        P->task_atiles.push_back(atl);
        P->task_btiles.push_back(btl);
        P->task_bias_tile.push_back(bias ? cc[0] : -1);
        geom.push_back({m, n, batch});
        m_max = std::max(m_max, m);
        n_max = std::max(n_max, n);
        big += ((m + 255) / 256) * ((n + 255) / 256) * batch;
    }
    const bool bf = A->dtype == NNT_BF16;
    std::vector<int64_t> ktot(P->tasks.size(), 0);
    for (size_t ti = 0; ti < P->tasks.size(); ti++)
        for (int32_t q = P->tasks[ti].chunk0; q < P->tasks[ti].chunk0 + P->tasks[ti].nchunk; q++) ktot[ti] += P->chunks[q].k;
    int64_t k_max = 0;
    for (int64_t kq : ktot) k_max = std::max(k_max, kq);
    // what the operands need: by the most demanding task, and by most of the work
    ShapeKind kind = kShapeWhole;
    double work_of[3] = {0.0, 0.0, 0.0};
    std::vector<char> staged(P->tasks.size(), 0);       // tasks that only the register-staged kernels take
    for (size_t ti = 0; ti < P->tasks.size(); ti++)
        for (int32_t q = P->tasks[ti].chunk0; q < P->tasks[ti].chunk0 + P->tasks[ti].nchunk; q++) {
            const ShapeKind kq = shape_kind(bf, P->akf, P->bkf, geom[ti].m, geom[ti].n, P->chunks[q].k, P->chunks[q].vec_ok == 3);
            kind = std::max(kind, kq);
            if (kq == kShapeGeneral) staged[ti] = 1;
            work_of[kq] += (double)geom[ti].batch * geom[ti].m * geom[ti].n * P->chunks[q].k;
        }
    const ShapeKind most = work_of[kShapeGeneral] > work_of[kShapeWhole] + work_of[kShapeRagged] ? kShapeGeneral : std::min(kind, kShapeRagged);
    P->cfg = pick_cfg(bf, m_max, n_max, big, k_max, P->akf && P->bkf, most);
    int S = 1;
    int64_t n_split = 0;
    if (nbat == 0 && !P->tasks.empty() && (P->cfg != kCfgResident || epi)) {
        // products of whole matrices: macro-tile shape and k-slices by the cost model (with an activation on the result path also
        // where the contraction is short: the kernels with the whole contraction in LDS have no such form)
        std::vector<int64_t> tm, tn;
        for (size_t ti = 0; ti < P->tasks.size(); ti++) {
            tm.push_back(geom[ti].m);
            tn.push_back(geom[ti].n);
        }
        // (the activation forms keep the whole contraction in one workgroup: the slice sum does not know them)
        ShapeChoice sc = choose_shape(bf, kind, tm, tn, ktot, epi == 0, epi != 0);
        if (kind == kShapeGeneral && most != kShapeGeneral) {
            // a few tiles keep the product off the direct-load kernels as a whole (5208 x 5585 over 576 on tiles of 400, bf16: the last
            // column of tiles has odd lines): the shape for the others, and these in a launch of their own (176 -> 120 us), where that
            // is clearly less (the cost of two launches is less certain than that of one)
            ShapeChoice two = choose_shape(bf, most, tm, tn, ktot, epi == 0, epi != 0);
            int bm2, bn2;
            gemm_cfg_tile(bf, two.cfg, &bm2, &bn2);
            int64_t n[2] = {0, 0};          // macro-tiles, of the others and of these
            for (size_t ti = 0; ti < P->tasks.size(); ti++) n[staged[ti]] += ((tm[ti] + bm2 - 1) / bm2) * ((tn[ti] + bn2 - 1) / bn2);
            const int s = two.n_split == n[0] + n[1] ? two.s : 1;         // (slices of only the last macro-tiles need not be theirs)
            two.us += launch_us(staged_cost(bf, two.cfg), n[1] * s, k_max / s);
            if (two.us < 0.85 * sc.us) sc = two;
        }
        P->cfg = sc.cfg;
        S = sc.s;
        n_split = sc.n_split;
        static const bool no_pack = getenv("NNT_GEMM_NO_PACK") != nullptr;      // debugging aid: operands are read as they are
        if (kind == kShapeGeneral && epi == 0 && ctx->granularity == NNT_GRAN_OP && !no_pack) {
            int bm0, bn0;
            gemm_cfg_tile(bf, sc.cfg, &bm0, &bn0);
            int64_t wgs = 0;
            for (size_t ti = 0; ti < P->tasks.size(); ti++) wgs += ((tm[ti] + bm0 - 1) / bm0) * ((tn[ti] + bn0 - 1) / bn0);
            const int32_t rc = try_packed(ctx, ax, A, B, C, bias, R, P, sc, wgs);
            if (rc != NNT_OK) return rc;
        }
    }
    int bm, bn;
    gemm_cfg_tile(bf, P->cfg, &bm, &bn);
    {
        // spelled like the demangled kernel name, so that profiler output can be matched against it
        static const char* const shape[9] = {"2, 2, 4, 4", "2, 2, 2, 2", "", "", "1, 4, 2, 1", "2, 2, 1, 1", "2, 2, 4, 2", "2, 2, 2, 2", "2, 2, 1, 2"};
        std::ostringstream l;
        const char* tf[2] = {"false", "true"};
        if (A->dtype == NNT_F32) l << "gemm_f32_kernel<" << tf[P->akf] << ", " << tf[P->bkf] << ", " << (P->cfg == kCfgSquare ? "2, 2, 2, 2" : P->cfg == kCfgMid ? "2, 2, 1, 2" : shape[P->cfg]) << ">";
        else l << "gemm_bf16_kernel<" << (C->dtype == NNT_F32 ? "float" : "unsigned short") << ", " << tf[P->akf] << ", " << tf[P->bkf]
               << ", " << shape[P->cfg] << ", 32>";
        if (nbat > 0) l << " batched";     // per-head attention products: short contractions, memory-leaning
        if (getenv("NNT_LABEL_SHAPES")) {  // one profile line per product shape instead of per kernel instance
            int64_t kmax = 0;
            for (int64_t kq : ktot) kmax = std::max(kmax, kq);
            int64_t rows = 1, cols = 1;
            for (int i = 0; i < nfa; i++) rows *= C->shape[i];
            for (int i = nfa; i < nfa + nfb; i++) cols *= C->shape[i];
            l << " [" << rows << " x " << cols << ", k/tile " << kmax << ", " << n_split << " macro-tiles in " << S << " slices]";
        }
        P->label = l.str();
    }
    if (P->packed) {
        const std::string old_name = P->label.substr(0, P->label.find('>') + 1);
        const char* tf[2] = {"false", "true"};
        if (!bf) P->label = std::string("gemm_f32_span_kernel<") + tf[P->akf] + ", " + tf[P->bkf] +
                            (P->pack_cfg == kCfgSquare ? ", 2, 2>" : P->pack_cfg == kCfgMid ? ", 1, 2>" : ", 1, 1>") + P->label.substr(old_name.size());
        else P->label = std::string(P->pack_cfg == kCfgSquare ? "gemm_bf16_span_kernel<" : P->pack_cfg == kCfgTall ? "gemm_bf16_span_tall_kernel<" : "gemm_bf16_span_wide_kernel<") +
                   (C->dtype == NNT_F32 ? "float, " : "unsigned short, ") + tf[P->akf] + ", " + tf[P->bkf] + ">" + P->label.substr(old_name.size());
        return NNT_OK;
    }
    // Workgroup order inside a task: m index fastest, so that workgroups in flight
    // together share a column panel of B.
    for (size_t ti = 0; ti < P->tasks.size(); ti++) {
        P->task_wg0.push_back((int64_t)P->wgs.size());
        const int64_t gm = (geom[ti].m + bm - 1) / bm, gn = (geom[ti].n + bn - 1) / bn;
        for (int64_t b = 0; b < geom[ti].batch; b++)
            for (int64_t j = 0; j < gn; j++)
                for (int64_t i = 0; i < gm; i++)
                    P->wgs.push_back(GemmWg{(int32_t)ti, (int32_t)(i * bm), (int32_t)(j * bn), (int32_t)b});
    }
    P->task_wg0.push_back((int64_t)P->wgs.size());
    if (P->wgs.size() > (size_t)INT32_MAX) return fail(ctx, NNT_EINVAL, "nnt_gemm: too many workgroups");
    // whole-operation launches use the XCD-aware order; per-task launches keep the order by task
    P->wgs_op = P->wgs;
    {
        // tasks of unequal length (causal attention: one to N_s / tile chunks): longest first, so that
        // the short ones fill the end of the launch instead of the long ones making its tail
        int64_t kmx = 0, kmn = INT64_MAX;
        for (int64_t kq : ktot) { kmx = std::max(kmx, kq); kmn = std::min(kmn, kq); }
        if (kmx > kmn)
            std::stable_sort(P->wgs_op.begin(), P->wgs_op.end(),
                             [&](const GemmWg& a, const GemmWg& b) { return ktot[a.task] > ktot[b.task]; });
    }
    xcd_interleave(P->wgs_op, bm, bn);

    // ---- k-slices for the last n_split macro-tiles of the whole-operation order
    // (a workspace above 2 GiB is not worth its memory: such a product runs without slices)
    if (S > 1 && (int64_t)std::min<int64_t>(n_split, (int64_t)P->wgs_op.size()) * S * bm * bn * (int64_t)sizeof(float) > ((int64_t)2 << 30)) {
        S = 1;
        n_split = 0;
    }
    P->splits = S;
    P->n_split = n_split = std::min<int64_t>(n_split, (int64_t)P->wgs_op.size());
    if (S > 1 && n_split > 0) {
        const size_t keep = P->wgs_op.size() - (size_t)n_split;
        const std::vector<GemmWg> cut(P->wgs_op.begin() + keep, P->wgs_op.end());
        P->wgs_op.resize(keep);
        const int64_t slice = (int64_t)bm * bn;
        NNT_HIP(ctx, hipMalloc((void**)&P->d_ws, (size_t)n_split * S * slice * sizeof(float)));
        P->ws_bytes += (int64_t)n_split * S * slice * (int64_t)sizeof(float);
        // chunk ranges of the slices, built once per C tile
        std::vector<std::vector<std::pair<int32_t, int32_t>>> ranges(P->tasks.size());
        std::vector<SplitReduce> red;
        std::vector<std::vector<GemmWg>> by_slice(S);
        for (size_t w = 0; w < cut.size(); w++) {
            const GemmWg& mw = cut[w];
            const GemmTask t0 = P->tasks[mw.task];
            if (ranges[mw.task].empty()) ranges[mw.task] = cut_into_slices(P, t0, ktot[mw.task], S, elem);
            red.push_back(add_slice_tasks(P, t0, mw, ranges[mw.task], P->d_ws + (int64_t)w * S * slice, bm, bn, by_slice));
        }
        deal_slices(by_slice, P->wgs_op);
        P->red_blocks = (int)((slice / 4 + 255) / 256);
        P->slice_elems = slice;
        NNT_HIP(ctx, hipMalloc((void**)&P->d_red, red.size() * sizeof(SplitReduce)));
        P->table_bytes += (int64_t)(red.size() * sizeof(SplitReduce));
        NNT_HIP(ctx, hipMemcpy(P->d_red, red.data(), red.size() * sizeof(SplitReduce), hipMemcpyHostToDevice));
    } else {
        P->splits = 1;
        P->n_split = 0;
    }
    P->op_nwg = (int64_t)P->wgs_op.size();

    // ---- k-slices per task for tile-granular launches
    const size_t n_tile_tasks = P->task_ctile.size();
    P->tile_split.assign(n_tile_tasks, GemmPlan::TileSplit{});
    std::vector<SplitReduce> red_ts;
    if (nbat == 0 && epi == 0 && ctx->granularity == NNT_GRAN_TILE) {      // (a plan first built for whole-operation launches has none)
        constexpr int64_t kTargetWgs = 64, kMinSlice = 512;
        constexpr int64_t kScratchCap = (int64_t)2 << 30;      // bytes of slice scratch per plan
        const int64_t slice = (int64_t)bm * bn;
        int64_t ws_blocks = 0;
        std::vector<int> st(n_tile_tasks, 1);
        for (int64_t max_slices = 8; max_slices >= 2; max_slices /= 2) {
            ws_blocks = 0;
            for (size_t ti = 0; ti < n_tile_tasks; ti++) {
                st[ti] = 1;
                const int64_t nwg = P->task_wg0[ti + 1] - P->task_wg0[ti];
                if (nwg == 0 || nwg >= kTargetWgs) continue;
                const int64_t want = std::min<int64_t>({max_slices, (kTargetWgs + nwg - 1) / nwg, ktot[ti] / kMinSlice});
                if (want < 2) continue;
                st[ti] = (int)want;
                ws_blocks += nwg * want;
            }
            if (ws_blocks * slice * (int64_t)sizeof(float) <= kScratchCap) break;
            ws_blocks = 0;
            std::fill(st.begin(), st.end(), 1);
        }
        if (ws_blocks > 0) {
            NNT_HIP(ctx, hipMalloc((void**)&P->d_ws_ts, (size_t)ws_blocks * slice * sizeof(float)));
            P->ws_bytes += (int64_t)ws_blocks * slice * (int64_t)sizeof(float);
            float* next_block = P->d_ws_ts;
            for (size_t ti = 0; ti < n_tile_tasks; ti++) {
                const int St = st[ti];
                if (St < 2) continue;
                const GemmTask t0 = P->tasks[ti];
                const std::vector<std::pair<int32_t, int32_t>> ranges = cut_into_slices(P, t0, ktot[ti], St, elem);
                GemmPlan::TileSplit& ts = P->tile_split[ti];
                ts.wg0 = (int64_t)P->wgs_ts.size();
                ts.red0 = (int64_t)red_ts.size();
                std::vector<std::vector<GemmWg>> by_slice(St);
                for (int64_t w = P->task_wg0[ti]; w < P->task_wg0[ti + 1]; w++) {
                    red_ts.push_back(add_slice_tasks(P, t0, P->wgs[w], ranges, next_block, bm, bn, by_slice));
                    next_block += (int64_t)St * slice;
                }
                for (int sidx = 0; sidx < St; sidx++) P->wgs_ts.insert(P->wgs_ts.end(), by_slice[sidx].begin(), by_slice[sidx].end());
                ts.nwg = (int64_t)P->wgs_ts.size() - ts.wg0;
                ts.nred = (int64_t)red_ts.size() - ts.red0;
            }
            P->red_blocks = (int)((slice / 4 + 255) / 256);    // (the same value the whole-operation slices set)
            P->slice_elems_ts = slice;
            NNT_HIP(ctx, hipMalloc((void**)&P->d_red_ts, red_ts.size() * sizeof(SplitReduce)));
            P->table_bytes += (int64_t)(red_ts.size() * sizeof(SplitReduce));
            NNT_HIP(ctx, hipMemcpy(P->d_red_ts, red_ts.data(), red_ts.size() * sizeof(SplitReduce), hipMemcpyHostToDevice));
        }
    }

    // workgroups that qualify for the direct-load kernel go first in every launch range
    P->task_nfast.assign(P->task_ctile.size(), 0);
    if (has_direct_load(bf, P->cfg)) {
        const int kmul = (bf && P->cfg == kCfgSquare) ? 64 : 32;   // loads are started two k-steps at a time
        // whether the kernel has a form for macro-tiles that end inside their C tile (at a whole vector of rows of an
        // operand whose row index is the contiguous one) and for chunks that are not whole k-steps
        const bool rag_ok = has_ragged(bf, P->cfg);
        const int vec = bf ? 8 : 4;
        std::vector<char> task_ok(P->tasks.size(), 1), task_rag(P->tasks.size(), 0);
        if (P->cfg == kCfgResident)      // the whole contraction, one chunk of at most 64, sits in LDS at once
            for (size_t ti = 0; ti < P->tasks.size(); ti++)
                if (P->tasks[ti].nchunk != 1 || P->chunks[P->tasks[ti].chunk0].k > 64 || P->chunks[P->tasks[ti].chunk0].k % 32 != 0) task_ok[ti] = 0;
        for (size_t ti = 0; ti < P->tasks.size(); ti++)
            for (int32_t q = P->tasks[ti].chunk0; q < P->tasks[ti].chunk0 + P->tasks[ti].nchunk; q++) {
                const GemmChunk& c = P->chunks[q];
                if (c.vec_ok != 3 || c.k <= 0 || (c.k % kmul != 0 && !(rag_ok && ragged_k_ok(bf, P->akf, P->bkf, c.k)))) task_ok[ti] = 0;
                else if (c.k % kmul != 0) task_rag[ti] = 1;
            }
        auto edge_ok = [&](const GemmWg& w) {
            const GemmTask& t = P->tasks[w.task];
            const int mv = std::min(bm, t.m - w.m0), nv = std::min(bn, t.n - w.n0);
            return rag_ok && (P->akf || mv % vec == 0) && (P->bkf || nv % vec == 0);
        };
        auto whole = [&](const GemmWg& w) {
            const GemmTask& t = P->tasks[w.task];
            return w.m0 + bm <= t.m && w.n0 + bn <= t.n;
        };
        auto qualifies = [&](const GemmWg& w) { return task_ok[w.task] && (whole(w) || edge_ok(w)); };
        for (const std::vector<GemmWg>* list : {&P->wgs, &P->wgs_op, &P->wgs_ts})
            for (const GemmWg& w : *list)
                if (qualifies(w) && (task_rag[w.task] || !whole(w))) P->dl_ragged = true;
        P->op_nfast = std::stable_partition(P->wgs_op.begin(), P->wgs_op.end(), qualifies) - P->wgs_op.begin();
        if (P->op_nfast > 0 && P->op_nfast < P->op_nwg) {
            int64_t k[2] = {0, 0};
            for (int64_t w = 0; w < P->op_nwg; w++) {
                const GemmTask& t = P->tasks[P->wgs_op[w].task];
                int64_t kw = 0;
                for (int32_t q = t.chunk0; q < t.chunk0 + t.nchunk; q++) kw += P->chunks[q].k;
                k[w >= P->op_nfast] = std::max(k[w >= P->op_nfast], kw);
            }
            if (!two_launches_pay(bf, P->cfg, P->dl_ragged, P->op_nfast, k[0], P->op_nwg - P->op_nfast, k[1])) P->op_nfast = 0;
        }
        for (size_t ti = 0; ti + 1 < P->task_wg0.size(); ti++)
            P->task_nfast[ti] = std::stable_partition(P->wgs.begin() + P->task_wg0[ti], P->wgs.begin() + P->task_wg0[ti + 1], qualifies) -
                                (P->wgs.begin() + P->task_wg0[ti]);
        for (GemmPlan::TileSplit& ts : P->tile_split)
            if (ts.nwg > 0)
                ts.nfast = std::stable_partition(P->wgs_ts.begin() + ts.wg0, P->wgs_ts.begin() + ts.wg0 + ts.nwg, qualifies) -
                           (P->wgs_ts.begin() + ts.wg0);
        if (2 * P->op_nfast >= P->op_nwg && P->op_nwg > 0) {
            // most of the work runs in the direct-load kernel: profile lines carry its name
            const std::string old_name = P->label.substr(0, P->label.find('>') + 1);
            const char* tf[2] = {"false", "true"};
            std::ostringstream l;
            if (bf)
                l << (P->cfg == kCfgTall ? "gemm_bf16_dl_tall_kernel<" : P->cfg == kCfgWide ? "gemm_bf16_dl_wide_kernel<" : "gemm_bf16_dl_kernel<")
                  << (C->dtype == NNT_F32 ? "float" : "unsigned short")
                  << ", " << tf[P->akf] << ", " << tf[P->bkf] << (P->cfg == kCfgTall ? (P->dl_ragged ? ", true>" : ", false>") : ">");
            else if (P->cfg == kCfgResident)
                l << (P->dl_ragged ? "gemm_f32_dl_rk_rag_kernel" : "gemm_f32_dl_rk_kernel");
            else
                l << (P->dl_ragged || P->cfg == kCfgSkinny64n64 ? "gemm_f32_dl_rag_kernel<" : "gemm_f32_dl_kernel<") << tf[P->akf] << ", " << tf[P->bkf]
                  << (P->cfg == kCfgSquare ? ", 2, 2>" : P->cfg == kCfgSkinny64n64 ? ", 1, 1>" : ", 1, 2>");
            P->label = l.str() + P->label.substr(old_name.size());
        }
    }

    if (epi) {
        P->epi_mode = epi & 15;
        bool all_fast = P->op_nwg > 0 && P->op_nfast == P->op_nwg && getenv("NNT_GEMM_NO_DL") == nullptr;
        for (size_t ti = 0; ti + 1 < P->task_wg0.size(); ti++) all_fast = all_fast && P->task_nfast[ti] == P->task_wg0[ti + 1] - P->task_wg0[ti];
        P->epi_ok = all_fast && !bf && !P->dl_ragged && P->cfg != kCfgSkinny64n64 && gemm_f32_dl_has_act(P->akf, P->bkf, P->epi_mode);
        if (P->epi_ok) {
            const std::string old_name = P->label.substr(0, P->label.find('>') + 1);
            const char* tf[2] = {"false", "true"};
            std::ostringstream l;
            l << "gemm_f32_dl_act_kernel<" << tf[P->akf] << (P->cfg == kCfgSquare ? ", 2, 2, " : ", 1, 2, ") << P->epi_mode << ">";
            P->label = l.str() + P->label.substr(old_name.size());
        }
    }

    auto up = [&](void** d, const void* h, size_t bytes) -> hipError_t {
        if (bytes == 0) return hipSuccess;
        hipError_t e = hipMalloc(d, bytes);
        if (e != hipSuccess) return e;
        P->table_bytes += (int64_t)bytes;
        return hipMemcpy(*d, h, bytes, hipMemcpyHostToDevice);
    };
    NNT_HIP(ctx, up((void**)&P->d_tasks, P->tasks.data(), P->tasks.size() * sizeof(GemmTask)));
    NNT_HIP(ctx, up((void**)&P->d_chunks, P->chunks.data(), P->chunks.size() * sizeof(GemmChunk)));
    NNT_HIP(ctx, up((void**)&P->d_wgs, P->wgs.data(), P->wgs.size() * sizeof(GemmWg)));
    NNT_HIP(ctx, up((void**)&P->d_wgs_op, P->wgs_op.data(), P->wgs_op.size() * sizeof(GemmWg)));
    NNT_HIP(ctx, up((void**)&P->d_wgs_ts, P->wgs_ts.data(), P->wgs_ts.size() * sizeof(GemmWg)));
    return NNT_OK;
}

}  // namespace

extern "C" int32_t nnt_gemm(nnt_ctx* ctx, float alpha, int32_t opA, nnt_tensor* A, int32_t opB, nnt_tensor* B,
                            float beta, nnt_tensor* C, int32_t ncon, int32_t nbat, nnt_tensor* bias) {
    return nnt_gemm_res(ctx, alpha, opA, A, opB, B, beta, C, ncon, nbat, bias, nullptr);
}

namespace {

void launch_splitk_reduce(hipStream_t st, const GemmPlan* P, const SplitReduce* red, float alpha, float beta) {
    const dim3 grid((unsigned)P->red_blocks, (unsigned)P->n_split), block(256);
    if (P->dtype_out == NNT_F32) hipLaunchKernelGGL((splitk_reduce<float>), grid, block, 0, st, red, alpha, beta);
    else hipLaunchKernelGGL((splitk_reduce<uint16_t>), grid, block, 0, st, red, alpha, beta);
}

// what gemm_core answers when the plan of a product with an activation form has workgroups that no kernel with that
// form takes (never leaves the library: the callers then run the product and the activation as two passes)
constexpr int32_t kNoActKernel = 1 << 20;

// The product proper.  A, B, C give the geometry (ordinary tensors, or the windows of nnt_gemm_heads: then `view_ld`
// and `key_extra` are set); `dep` are the tensors whose tiles order the tasks (the operands themselves, or what
// the windows look at).
int32_t gemm_core(nnt_ctx* ctx, float alpha, int32_t opA, nnt_tensor* A, int32_t opB, nnt_tensor* B, float beta, nnt_tensor* C,
                  int32_t ncon, int32_t nbat, nnt_tensor* bias, nnt_tensor* R, nnt_tensor* const* dep, const int64_t* view_ld,
                  const std::string& key_extra, int32_t part_c = 0, int epi = 0) {
    std::ostringstream key;
    key << opA << opB << ':' << A->id << ':' << B->id << ':' << C->id << ':' << (bias ? bias->id : 0) << ':' << ncon << ':' << nbat
        << ':' << (R ? R->id : 0) << key_extra;
    GemmPlan* P = nullptr;
    const bool by_tile = ctx->granularity == NNT_GRAN_TILE && !view_ld;
    for (const char* which : {"", ":t"}) {
        const std::string k = key.str() + which;
        auto it = ctx->gemm_plans.find(k);
        if (it == ctx->gemm_plans.end()) {
            if (ctx->capturing && P) break;      // (inside a capture, where none can be built, the one that is there runs as a whole)
            if (ctx->capturing) return fail(ctx, NNT_ESTATE, "nnt_gemm: plan must exist before capture (run the call once first)");
            std::shared_ptr<GemmPlan> np(new GemmPlan());
            int32_t rc = build_plan(ctx, opA, A, opB, B, C, ncon, nbat, bias, R, np.get(), view_ld, epi);
            if (rc != NNT_OK) return rc;
            P = np.get();
            ctx->gemm_plans[k] = np;
        } else {
            P = it->second.get();
        }
        if (!(by_tile && P->packed)) break;      // (a plan that lays the operands out afresh has no tasks per tile: another one is built)
    }
    if (epi && !P->epi_ok) return kNoActKernel;
    const int epi_mode = P->epi_mode;
    nnt_tensor* const dA = dep[0];
    nnt_tensor* const dB = dep[1];
    nnt_tensor* const dC = dep[2];
    OpTag tag(ctx, P->label.c_str(), P->flops, false);
    GemmArgs g = {};
    g.tasks = P->d_tasks;
    g.chunks = P->d_chunks;
    g.alpha = alpha;
    g.beta = beta;
    const int cmode = beta != 0.f ? kReadWrite : kWrite;
    if (!by_tile || P->packed) {
        // (a window writes the rows of its part in every tile it touches and leaves the others)
        std::vector<Access> acc = {dA->all(kRead), dB->all(kRead), dC->all((view_ld && view_ld[2]) ? kWritePart : (R ? kWrite : cmode))};
        acc[2].part = part_c;
        if (bias) acc.push_back(bias->all(kRead));
        if (R && (beta != 0.f || epi)) acc.push_back(R->all((epi & 15) == kEpiGeluOut ? kWrite : kRead));
        g.wgs = P->d_wgs_op;
        if (P->packed) {
            g = P->pack_args;
            g.alpha = alpha;
            g.beta = beta;
            if (P->n_split > 0) acc.push_back(Access{&P->ws_dep, 1, kReadWrite});
            const double red_bytes = (double)P->n_split * P->slice_elems * 4.0 * (P->splits + 1);
            return submit(ctx, acc, [=](hipStream_t st) {
                const bool bf16 = P->dtype_in == NNT_BF16;
                GemmArgs ga = g;
                ga.pack_base = reinterpret_cast<char*>(P->pack_space->mem->p) + ctx->cur_stream * P->pack_space->part;
                PackOperand o[2] = {P->pack[0], P->pack[1]};
                for (PackOperand& p : o) p.dst = ga.pack_base + (intptr_t)p.dst;
                int32_t rc = pack_operands(st, bf16, o[0], o[1]);
                if (rc != NNT_OK) return rc;
                rc = bf16 ? launch_gemm_bf16_span(st, P->dtype_out == NNT_F32, P->akf, P->bkf, P->pack_cfg, ga, P->pack_nwg)
                          : launch_gemm_f32_span(st, P->akf, P->bkf, P->pack_cfg, ga, P->pack_nwg);
                if (rc != NNT_OK || P->n_split == 0) return rc;
                profile_mark(ctx, st, "splitk_reduce", red_bytes, true);
                launch_splitk_reduce(st, P, P->pack_red, alpha, beta);
                return hipGetLastError() == hipSuccess ? (int32_t)NNT_OK : (int32_t)NNT_EHIP;
            }, P->n_split > 0 ? 3 : 2);
        }
        const int64_t nwg = P->op_nwg;
        if (nwg == 0) return NNT_OK;
        if (P->n_split > 0) {
            acc.push_back(Access{&P->ws_dep, 1, kReadWrite});
            const double red_bytes = (double)P->n_split * P->slice_elems * 4.0 * (P->splits + 1);
            return submit(ctx, acc, [=](hipStream_t st) {
                int32_t rc = launch_any(st, P->dtype_in, P->dtype_out, P->akf, P->bkf, P->cfg, g, nwg, P->op_nfast, P->dl_ragged);
                if (rc != NNT_OK) return rc;
                profile_mark(ctx, st, "splitk_reduce", red_bytes, true);
                launch_splitk_reduce(st, P, P->d_red, alpha, beta);
                return hipGetLastError() == hipSuccess ? (int32_t)NNT_OK : (int32_t)NNT_EHIP;
            }, 2);
        }
        return submit(ctx, acc, [=](hipStream_t st) {
            return launch_any(st, P->dtype_in, P->dtype_out, P->akf, P->bkf, P->cfg, g, nwg, P->op_nfast, P->dl_ragged, epi_mode);
        });
    }
    const size_t n_tile_tasks = P->task_ctile.size();
    for (size_t ti = 0; ti < n_tile_tasks; ti++) {
        std::vector<Access> acc;
        acc.push_back(C->one(P->task_ctile[ti], R ? kWrite : cmode));
        if (R && (beta != 0.f || epi)) acc.push_back(R->one(P->task_ctile[ti], (epi & 15) == kEpiGeluOut ? kWrite : kRead));
        for (int64_t a : P->task_atiles[ti]) acc.push_back(A->one(a, kRead));
        for (int64_t b : P->task_btiles[ti]) acc.push_back(B->one(b, kRead));
        if (bias) acc.push_back(bias->one(P->task_bias_tile[ti], kRead));
        GemmArgs gt = g;
        const GemmPlan::TileSplit ts = P->tile_split[ti];
        int32_t rc;
        if (ts.nwg > 0) {
            // few macro-tiles, long contraction: k-slices into this task's scratch block, then their sum
            gt.wgs = P->d_wgs_ts + ts.wg0;
            const double red_bytes = (double)ts.nred * P->slice_elems_ts * 4.0 * (ts.nwg / ts.nred + 1);
            rc = submit(ctx, acc, [=](hipStream_t st) {
                int32_t r = launch_any(st, P->dtype_in, P->dtype_out, P->akf, P->bkf, P->cfg, gt, ts.nwg, ts.nfast, P->dl_ragged);
                if (r != NNT_OK) return r;
                profile_mark(ctx, st, "splitk_reduce", red_bytes, true);
                const dim3 grid((unsigned)P->red_blocks, (unsigned)ts.nred), block(256);
                if (P->dtype_out == NNT_F32) hipLaunchKernelGGL((splitk_reduce<float>), grid, block, 0, st, P->d_red_ts + ts.red0, alpha, beta);
                else hipLaunchKernelGGL((splitk_reduce<uint16_t>), grid, block, 0, st, P->d_red_ts + ts.red0, alpha, beta);
                return hipGetLastError() == hipSuccess ? (int32_t)NNT_OK : (int32_t)NNT_EHIP;
            }, 2);
        } else {
            gt.wgs = P->d_wgs + P->task_wg0[ti];
            const int64_t nwg = P->task_wg0[ti + 1] - P->task_wg0[ti];
            const int64_t nfast = P->task_nfast[ti];
            rc = submit(ctx, acc, [=](hipStream_t st) {
                return launch_any(st, P->dtype_in, P->dtype_out, P->akf, P->bkf, P->cfg, gt, nwg, nfast, P->dl_ragged, epi_mode);
            });
        }

        if (rc != NNT_OK) return rc;
    }
    return NNT_OK;
}

// A window on `T` ([n_parts * N_h * h, N_s, N_b], the heads side by side along the first axis): rows
// [part * N_h * h, (part + 1) * N_h * h) seen as [h, N_s, N_b, N_h].  Its tiles are T's own (one per group of
// base[0] / h heads), addressed with T's leading dimension; nothing is copied.  Parts and groups of heads must
// coincide with T's row tiles.
int32_t make_window(nnt_ctx* ctx, nnt_tensor* T, int32_t part, int64_t h, int64_t N_h, nnt_tensor* W, int64_t* ld) {
    const int64_t N_e = h * N_h, t0 = T->base[0];
    if (T->ndim != 3 || part < 0 || T->shape[0] % N_e != 0 || (int64_t)(part + 1) * N_e > T->shape[0])
        return fail(ctx, NNT_EINVAL, "nnt_gemm_heads: a window needs a 3-axis tensor of whole parts of N_h * h rows and a part inside it");
    if (t0 % h != 0 || N_e % t0 != 0)
        return fail(ctx, NNT_EINVAL, "nnt_gemm_heads: row tiles must hold whole heads and a part whole row tiles");
    const int64_t hp = t0 / h;
    W->ctx = ctx;
    W->dtype = T->dtype;
    W->ndim = 4;
    const int64_t shape[4] = {h, T->shape[1], T->shape[2], N_h}, base[4] = {h, T->base[1], T->base[2], hp};
    W->ntiles = 1;
    for (int a = 0; a < 4; a++) {
        W->shape[a] = shape[a];
        W->base[a] = base[a];
        W->grid[a] = (shape[a] + base[a] - 1) / base[a];
        W->ntiles *= W->grid[a];
    }
    W->tiles.assign((size_t)W->ntiles, nullptr);
    W->d_tiles = nullptr;
    W->id = T->id;
    for (int64_t i = 0; i < W->ntiles; i++) {
        int64_t wc[kMaxDim], tc[kMaxDim] = {0, 0, 0, 0};
        W->tile_coords(i, wc);
        tc[0] = (int64_t)part * (N_e / t0) + wc[3];
        tc[1] = wc[1];
        tc[2] = wc[2];
        W->tiles[(size_t)i] = T->tiles[(size_t)T->tile_index(tc)];
        if (!W->tiles[(size_t)i]) return fail(ctx, NNT_EINVAL, "nnt_gemm_heads: a tensor with the heads side by side must hold all its tiles");
    }
    *ld = t0;
    return NNT_OK;
}

// An ordinary tensor [., ., N_b, N_h] seen with `hp` heads per tile along its last axis (what the windows on the
// other operands have): a tile of the coarser tiling is cut along its slowest axis, so the pieces are contiguous
// and keep its strides.  Absent tiles stay absent.
int32_t make_retiled(nnt_ctx* ctx, nnt_tensor* T, int64_t hp, nnt_tensor* W) {
    if (T->ndim != 4 || T->base[3] % hp != 0)
        return fail(ctx, NNT_EINVAL, "nnt_gemm_heads: the head axis of an ordinary operand must be tiled in multiples of the heads per row tile");
    *W = *T;                           // geometry, type, id
    W->deps.clear();
    W->d_tiles = nullptr;
    W->base[3] = hp;
    W->grid[3] = (T->shape[3] + hp - 1) / hp;
    W->ntiles = W->grid[0] * W->grid[1] * W->grid[2] * W->grid[3];
    W->tiles.assign((size_t)W->ntiles, nullptr);
    for (int64_t i = 0; i < W->ntiles; i++) {
        int64_t wc[kMaxDim], tc[kMaxDim];
        W->tile_coords(i, wc);
        for (int a = 0; a < 3; a++) tc[a] = wc[a];
        tc[3] = wc[3] * hp / T->base[3];
        char* basep = static_cast<char*>(T->tiles[(size_t)T->tile_index(tc)]);
        if (!basep) continue;
        const int64_t first = wc[3] * hp - tc[3] * T->base[3];           // heads of the coarse tile before this piece
        const int64_t per_head = T->tile_extent(0, tc[0]) * T->tile_extent(1, tc[1]) * T->tile_extent(2, tc[2]);
        W->tiles[(size_t)i] = basep + first * per_head * T->elem_size();
    }
    return NNT_OK;
}

}  // namespace

extern "C" int32_t nnt_gemm_res(nnt_ctx* ctx, float alpha, int32_t opA, nnt_tensor* A, int32_t opB, nnt_tensor* B,
                                float beta, nnt_tensor* C, int32_t ncon, int32_t nbat, nnt_tensor* bias, nnt_tensor* R) {
    NNT_CHECK_CTX(ctx);
    if (!A || !B || !C) return fail(ctx, NNT_EINVAL, "nnt_gemm: null tensor");
    if ((opA != NNT_OP_N && opA != NNT_OP_T) || (opB != NNT_OP_N && opB != NNT_OP_T))
        return fail(ctx, NNT_EINVAL, "nnt_gemm: bad op");
    if (R == C) R = nullptr;
    if (R) {
        if (R->dtype != C->dtype || !same_tiling(R, C)) return fail(ctx, NNT_EINVAL, "nnt_gemm_res: the residual input must have C's type, shape and tiling");
        for (int64_t t = 0; t < C->ntiles; t++)
            if (C->tiles[t] && !R->tiles[t]) return fail(ctx, NNT_EINVAL, "nnt_gemm_res: the residual input lacks a tile that C has");
        if (R == A || R == B) return fail(ctx, NNT_EINVAL, "nnt_gemm_res: the residual input must not be an operand");
    }
    nnt_tensor* const dep[3] = {A, B, C};
    return gemm_core(ctx, alpha, opA, A, opB, B, beta, C, ncon, nbat, bias, R, dep, nullptr, std::string());
}

namespace {

int32_t gemm_gelu(nnt_ctx* ctx, const char* who, int mode, float alpha, int32_t opA, nnt_tensor* A, int32_t opB, nnt_tensor* B, nnt_tensor* C,
                  int32_t ncon, nnt_tensor* bias, int32_t variant, nnt_tensor* X) {
    NNT_CHECK_CTX(ctx);
    if (!A || !B || !C || !X) return fail(ctx, NNT_EINVAL, std::string(who) + ": null tensor");
    if ((opA != NNT_OP_N && opA != NNT_OP_T) || (opB != NNT_OP_N && opB != NNT_OP_T) || (variant != NNT_GELU_TANH && variant != NNT_GELU_ERF))
        return fail(ctx, NNT_EINVAL, std::string(who) + ": bad op or GELU variant");
    if (X == C || X == A || X == B || X->dtype != C->dtype || !same_tiling(X, C))
        return fail(ctx, NNT_EINVAL, std::string(who) + ": the second tensor must be distinct from A, B and C and have C's type, shape and tiling");
    for (int64_t t = 0; t < C->ntiles; t++)
        if (C->tiles[t] && !X->tiles[t]) return fail(ctx, NNT_EINVAL, std::string(who) + ": the second tensor lacks a tile that C has");
    nnt_tensor* const dep[3] = {A, B, C};
    std::ostringstream extra;
    extra << ":gelu" << mode << variant;
    if (A->dtype == NNT_F32 && gemm_f32_dl_has_act(opA == NNT_OP_T, opB == NNT_OP_N, mode)) {
        const int32_t rc = gemm_core(ctx, alpha, opA, A, opB, B, 0.f, C, ncon, 0, bias, X, dep, nullptr, extra.str(), 0, mode | (variant << 4));
        if (rc != kNoActKernel) return rc;
    }
    // bf16, or ragged macro-tiles, operand forms or alignments that only the general kernels take: product, then activation
    int32_t r2 = gemm_core(ctx, alpha, opA, A, opB, B, 0.f, C, ncon, 0, bias, nullptr, dep, nullptr, std::string());
    if (r2 != NNT_OK) return r2;
    return mode == kEpiGeluOut ? nnt_gelu(ctx, variant, C, X) : nnt_gelu_bwd(ctx, variant, X, C, C);
}

}  // namespace

extern "C" int32_t nnt_gemm_gelu(nnt_ctx* ctx, float alpha, int32_t opA, nnt_tensor* A, int32_t opB, nnt_tensor* B, nnt_tensor* C,
                                 int32_t ncon, nnt_tensor* bias, int32_t variant, nnt_tensor* G) {
    return gemm_gelu(ctx, "nnt_gemm_gelu", kEpiGeluOut, alpha, opA, A, opB, B, C, ncon, bias, variant, G);
}

extern "C" int32_t nnt_gemm_gelu_bwd(nnt_ctx* ctx, float alpha, int32_t opA, nnt_tensor* A, int32_t opB, nnt_tensor* B, nnt_tensor* C,
                                     int32_t ncon, int32_t variant, nnt_tensor* X) {
    return gemm_gelu(ctx, "nnt_gemm_gelu_bwd", kEpiGeluGradMul, alpha, opA, A, opB, B, C, ncon, nullptr, variant, X);
}

extern "C" int32_t nnt_gemm_heads(nnt_ctx* ctx, float alpha, int32_t opA, nnt_tensor* A, int32_t partA, int32_t opB, nnt_tensor* B,
                                  int32_t partB, nnt_tensor* C, int32_t partC, int32_t h, int32_t N_h) {
    NNT_CHECK_CTX(ctx);
    if (!A || !B || !C) return fail(ctx, NNT_EINVAL, "nnt_gemm_heads: null tensor");
    if ((opA != NNT_OP_N && opA != NNT_OP_T) || (opB != NNT_OP_N && opB != NNT_OP_T) || h < 1 || N_h < 1)
        return fail(ctx, NNT_EINVAL, "nnt_gemm_heads: bad argument");
    nnt_tensor win[3];
    nnt_tensor* geo[3] = {A, B, C};
    nnt_tensor* const dep[3] = {A, B, C};
    const int32_t part[3] = {partA, partB, partC};
    int64_t view_ld[3] = {0, 0, 0};
    std::ostringstream extra;
    extra << ":heads" << h << 'x' << N_h;
    int64_t hp = 0;
    for (int i = 0; i < 3; i++) {
        extra << ':' << part[i];
        if (part[i] < 0) continue;
        int32_t rc = make_window(ctx, dep[i], part[i], h, N_h, &win[i], &view_ld[i]);
        if (rc != NNT_OK) return rc;
        geo[i] = &win[i];
        if (hp && hp != win[i].base[3]) return fail(ctx, NNT_EINVAL, "nnt_gemm_heads: the tensors with parts must have one row tiling");
        hp = win[i].base[3];
    }
    if (!hp) return fail(ctx, NNT_EINVAL, "nnt_gemm_heads: no operand has a part (use nnt_gemm)");
    for (int i = 0; i < 3; i++) {
        if (part[i] >= 0) continue;
        if (dep[i]->ndim != 4 || dep[i]->shape[3] != N_h)
            return fail(ctx, NNT_EINVAL, "nnt_gemm_heads: tensors without a part must have the axes [., ., N_b, N_h]");
        if (dep[i]->base[3] == hp) continue;
        int32_t rc = make_retiled(ctx, dep[i], hp, &win[i]);
        if (rc != NNT_OK) return rc;
        geo[i] = &win[i];
    }
    return gemm_core(ctx, alpha, opA, geo[0], opB, geo[1], 0.f, geo[2], 1, 2, nullptr, nullptr, dep, view_ld, extra.str(), partC > 0 ? partC : 0);
}
