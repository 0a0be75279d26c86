// Host side of the sampling-verification library (gfx950): validation of a problem, the choice
// of a kernel family (spechub_resident.hip, rrs_resident.hip, verify_generic_*.hip,
// draft_*.hip; the device code they share is in node_common.h), the tree walk and Philox
// kernels, and the C entry points.
#include "launch.h"
#include "launch_group.h"
#include "launch_half.h"
#include "launch_small.h"
#include "launch_wide.h"

#include <atomic>

namespace mdsd {

// ---------------------------------------------------------------- tree walk
// The walk as a launch of its own (see group_walk and wave_walk in node_common.h).  Trees of at most
// 64 nodes: a group of W lanes per tree (W = the power of two from N up), 64 / W trees per wavefront.
// Larger trees (W = 0): one wavefront per tree.
__global__ __launch_bounds__(256) void tree_walk_kernel(const int32_t* outcome, const int32_t* token, int B, int N,
                                                        int W, int k, int depth, const int32_t* first_child,
                                                        int32_t* accept_depth, int32_t* emitted)
{
    const int wave = blockIdx.x * (blockDim.x / 64) + (int)(threadIdx.x / 64);
    if (W == 0) {
        if (wave < B) wave_walk<false>(outcome, token, wave, N, k, depth, first_child, accept_depth, emitted);
        return;
    }
    const int per_wave = 64 / W;
    if ((int64_t)wave * per_wave >= B) return;  // the whole wavefront: the shuffles below need every lane of the others
    const int b = wave * per_wave + (int)(threadIdx.x & 63) / W;
    group_walk<false>(outcome, token, b < B ? b : 0, b < B, W, N, k, depth, first_child, accept_depth, emitted);
}

// ---------------------------------------------------------------- Philox4x32-10
// Salmon, Moraes, Dror, Shaw, SC'11: ten rounds of two 32x32->64 multiplies,
// swap and xor with the key; the key advances by the two Weyl constants.
__global__ void philox_uniform_kernel(uint32_t k0, uint32_t k1, uint32_t stream_id, int64_t rows,
                                      int slots, float* out, uint32_t* words)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int blocks_per_row = (slots + 3) >> 2;
    if (i >= rows * blocks_per_row) return;
    const int64_t row = i / blocks_per_row;
    const int blk = (int)(i - row * blocks_per_row);
    uint32_t c0 = (uint32_t)row, c1 = (uint32_t)((uint64_t)row >> 32), c2 = (uint32_t)blk, c3 = stream_id;
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint32_t h0 = __umulhi(0xD2511F53u, c0), l0 = 0xD2511F53u * c0;
        const uint32_t h1 = __umulhi(0xCD9E8D57u, c2), l1 = 0xCD9E8D57u * c2;
        const uint32_t n0 = h1 ^ c1 ^ k0, n2 = h0 ^ c3 ^ k1;
        c0 = n0;
        c1 = l1;
        c2 = n2;
        c3 = l0;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    const uint32_t w[4] = {c0, c1, c2, c3};
    for (int j = 0; j < 4; ++j) {
        const int s = blk * 4 + j;
        if (s < slots) {
            if (out) out[row * slots + s] = (float)(w[j] >> 8) * (1.0f / 16777216.0f);
            if (words) words[row * slots + s] = w[j];
        }
    }
}
// ---------------------------------------------------------------- host side
static int complete_tree_nodes(int k, int depth, int64_t* n_internal)
{
    int64_t n = 0, level = 1, internal = 0;
    for (int d = 0; d < depth; ++d) {
        if (d == depth - 1) internal = n;
        n += level;
        level *= k;
        if (n > INT_MAX) return -1;
    }
    *n_internal = internal;
    return (int)n;
}

// what validate returns for a batch of no trees: the entry points then return MDSD_OK at once
static constexpr int kEmptyBatch = 1;

static int validate(const mdsd_problem* pb, int method, bool need_target, Params* P)
{
    if (!pb) return MDSD_E_NULL;
    if (pb->B == 0) return kEmptyBatch;
    if (!pb->draft || (need_target && !pb->target)) return MDSD_E_NULL;
    if (pb->dtype != MDSD_FP32 && pb->dtype != MDSD_BF16) return MDSD_E_DTYPE;
    if (pb->kind != MDSD_PROBS && pb->kind != MDSD_LOGITS) return MDSD_E_DTYPE;
    if (pb->B < 1 || pb->N < 1 || pb->V < 2 || pb->depth < 1) return MDSD_E_SHAPE;
    if (pb->ld_d < pb->V || (need_target && pb->ld_t < pb->V)) return MDSD_E_SHAPE;
    if (pb->k < 1 || pb->k > MDSD_MAX_K) return MDSD_E_K;
    if (method == kSpecHub && pb->k != 2) return MDSD_E_K;
    if (pb->kind == MDSD_LOGITS) {
        if (!(pb->temp_draft > 0.f)) return MDSD_E_TEMP;
        if (need_target && !(pb->temp_target > 0.f)) return MDSD_E_TEMP;
    }
    const int es = pb->dtype == MDSD_FP32 ? 4 : 2;
    const int per_chunk = 16 / es;
    // vocabulary bound of the per-slab partial sums kept in LDS
    if ((int64_t)pb->V + per_chunk > (int64_t)kMaxSlabs * 64 * per_chunk) return MDSD_E_SHAPE;
    if ((int64_t)pb->B * pb->N > INT_MAX) return MDSD_E_SHAPE;
    const uintptr_t at = (uintptr_t)pb->target, ad = (uintptr_t)pb->draft;
    if ((ad % es) != 0 || (need_target && (at % es) != 0)) return MDSD_E_ALIGN;
    if (need_target) {
        // every pair of rows must share its offset modulo 16 bytes
        if ((at & 15) != (ad & 15)) return MDSD_E_ALIGN;
        if (pb->B * (int64_t)pb->N > 1 && ((pb->ld_t * es) & 15) != ((pb->ld_d * es) & 15)) return MDSD_E_ALIGN;
    }
    int64_t n_internal = 0;
    if (!pb->first_child) {
        const int n = complete_tree_nodes(pb->k, pb->depth, &n_internal);
        if (n != pb->N) return MDSD_E_SHAPE;
    }
    P->target = pb->target;
    P->draft = pb->draft;
    P->ld_t = pb->ld_t;
    P->ld_d = pb->ld_d;
    P->temp_target = pb->temp_target;
    P->temp_draft = pb->temp_draft;
    P->scale_t = pb->kind == MDSD_LOGITS && need_target ? kLog2e / pb->temp_target : 0.f;
    P->scale_d = pb->kind == MDSD_LOGITS ? kLog2e / pb->temp_draft : 0.f;
    P->B = pb->B;
    P->N = pb->N;
    P->V = pb->V;
    P->k = pb->k;
    P->depth = pb->depth;
    P->n_internal = (int)n_internal;
    P->first_child = pb->first_child;
    P->masked = (ad & 15) || ((pb->ld_d * es) & 15) || (pb->V % per_chunk) ||
                (need_target && ((at & 15) || ((pb->ld_t * es) & 15)));
    // rows that start anywhere: up to per_chunk - 1 masked elements in front
    P->row_chunks = (int)(((int64_t)pb->V + (P->masked ? 2 * per_chunk - 2 : 0)) / per_chunk);
    return MDSD_OK;
}

// chunks per lane that hold a whole row in registers; 0 = stream the row in every pass
static int resident_chunks(const mdsd_problem* pb)
{
    const int per_chunk = pb->dtype == MDSD_FP32 ? 4 : 8;
    // worst case head of per_chunk - 1 masked elements in front of the row
    const int64_t nchunk = ((int64_t)pb->V + 2 * per_chunk - 2) / per_chunk;
    const int64_t per_lane = (nchunk + kWG - 1) / kWG;
    if (per_lane <= 4) return 4;
    if (per_lane <= 8) return 8;
    if (per_lane <= 16) return 16;
    return 0;
}
// Rows too long for a group of lanes (and SpecHub nodes in large batches, see verify_lanes()) but short
// go to a build of the generic kernels with fewer threads per node (1, 2 or 4 wavefronts: four chunks per
// lane) instead of one 512-thread workgroup most of whose wavefronts would hold no part of the row; 0 =
// the main build
static int small_build(const mdsd_problem* pb)
{
    const int per_chunk = pb->dtype == MDSD_FP32 ? 4 : 8;
    const int64_t nchunk = ((int64_t)pb->V + 2 * per_chunk - 2) / per_chunk;
    if (nchunk <= mdsd_wave::kMaxChunks) return 1;
    if (nchunk <= mdsd_pair::kMaxChunks) return 2;
    if (nchunk <= mdsd_quad::kMaxChunks) return 4;
    return 0;
}
// true when some element of some row may need masking: a row that does not start on a
// 16-byte boundary, or a vocabulary that is not a whole number of 16-byte chunks
static bool rows_need_mask(const mdsd_problem* pb)
{
    const int es = pb->dtype == MDSD_FP32 ? 4 : 2;
    const uintptr_t at = (uintptr_t)pb->target, ad = (uintptr_t)pb->draft;
    return (at & 15) || (ad & 15) || ((pb->ld_t * es) & 15) || ((pb->ld_d * es) & 15) || (pb->V % (16 / es));
}
// One workgroup per node.  Complete trees with more than one node: (trees, nodes), which
// node_of_block() reads without a division (a one-node tree keeps gridDim.y == 1, which is how the
// kernels tell the two numberings apart; there the single node is node 0 of tree blockIdx.x
// either way).  Explicit topologies, and trees of more nodes than a grid's second dimension
// holds: one dimension.
// Rows too long for registers (nit == 0) keep the one-dimensional numbering as well: there
// the workgroups that run side by side would read rows a whole tree apart, which measured 4 %
// slower than rows next to each other (config 4).
static dim3 node_grid(const Params& P, int nit)
{
    if (P.first_child == nullptr && P.N > 1 && P.N <= 65535 && nit > 0) return dim3((unsigned)P.B, (unsigned)P.N);
    return dim3((unsigned)(P.B * P.N));
}

// Trees given by a table, a workgroup per node: node by node over the batch (SpecHub and RRSw steps of 9- and 31-node trees,
// tree by tree -> node by node: bf16 rows of 32000, 1800 nodes 54.9 -> 50.4 and 63.8 -> 57.2 us, 56.7 -> 55.4 and 66.0 ->
// 64.3; of 128256, 900 nodes 117 -> 115, 133 -> 115, 126 -> 117, 143 -> 131, 3600 312 -> 292, 383 -> 342, 322 -> 318, 401 ->
// 393), but tree by tree where the rows are held in registers and so many that the launch's end weighs less than the
// place of neighbouring rows in memory: SpecHub from 400 MB of rows per call on (fp32 rows of 8000, 432 MB 137 against 141
// and 141 against 148; bf16 of 32000, 864 MB 256 against 264, 265 against 272; of 50304, 270 MB 112 against 105, 720 MB 243
// against 239, 250 against 256), the RRS methods from 800 MB on (432 MB RRSw 165 against 164, 170 against 174, bf16 of
// 8000, 576 MB 343 against 330, 357 against 353; of 32000, 864 MB 276 against 281, 285 against 287).  Handing a node's trees
// round among the XCDs, as node_of_block() does for complete trees, makes no difference here (1800 nodes of 32000 50.6,
// 57.6).
static int table_by_tree(int method, const mdsd_problem* pb)
{
    if (pb->kind != MDSD_LOGITS || resident_chunks(pb) == 0) return 0;
    const int64_t bytes = (int64_t)pb->B * pb->N * pb->V * (pb->dtype == MDSD_FP32 ? 4 : 2);
    return bytes >= (method == kSpecHub ? 400000000 : 800000000);
}

// tree nodes per batch from which the 256-thread verify kernels take over from the 512-thread ones
constexpr int64_t kHalfWidthMinNodes = 2300;

// ---- 1024 threads per node, logit rows in registers
// chunks per lane of such a workgroup; 0: the row is too long
static int wide_chunks(const Params& P)
{
    const int per_lane = (P.row_chunks + mdsd_wide::kThreads - 1) / mdsd_wide::kThreads;
    return per_lane <= 4 ? 4 : per_lane <= 8 ? 8 : per_lane <= 16 ? 16 : per_lane <= 20 ? 20 : 0;
}
// a batch that leaves CUs without a node
constexpr int64_t kWideMaxNodes = 256;
// Verify.  SpecHub, which reads its rows once or twice, up to 256 nodes (512 against 1024 threads, 60 nodes).
// Rows that 512 threads stream (more than 16 chunks per lane): 66048 bf16 19.3 -> 18.0 us, 100000 28.0 -> 23.0.
// Rows that they hold too: with the draft call's records aligned ones lose (fp32 17000 8.8 -> 9.2, 32000 11.0 ->
// 11.0; bf16 33000 11.7 -> 12.0, 50304 14.2 -> 14.4), unaligned ones gain (fp32 32001 12.9 -> 12.3; bf16 33001 12.7
// -> 12.8, 65001 18.3 -> 17.6), and so do calls without records, which hold both rows (fp32 16400 11.3 -> 11.3,
// 32000 15.5 -> 14.5, 32001 19.7 -> 17.3; bf16 50304 19.8 -> 18.8).
// Path-only, where a tree's nodes pass their barriers one after another: resident rows lose with records (8 trees,
// fp32 17000 18.6 -> 21.3, bf16 50304 28.7 -> 31.2) and without if aligned (fp32 17000 28.8 -> 30.9); without records
// and unaligned they gain (fp32 32001 51.9 -> 46.8).  Streamed ones gain from 32 trees on (66048 54.5 -> 48.9, 70001
// 58.7 -> 54.7; up to 16 trees between -9 and +9 % by the paths drawn), rows of more than 20 chunks per lane
// always (100000, 4 trees 35.8 -> 35.1, 8 trees 45.4 -> 44.0).
static int wide_spechub_chunks(const mdsd_problem* pb, const Params& P, bool path)
{
    const int nit = wide_chunks(P);
    const int64_t nodes = (int64_t)P.B * (path ? 1 : P.N);
    if (nodes > kWideMaxNodes || P.row_chunks <= 8 * kWG) return 0;
    if (resident_chunks(pb) == 0) {
        if (!P.stats_in || nit > 16) return 0;
        return !path || (nit == 16 && (P.B >= 32 || P.row_chunks > 20 * kWG)) ? nit : 0;
    }
    return P.masked ? (path && P.stats_in ? 0 : nit) : path || P.stats_in ? 0 : nit;
}
// Verify, RRS methods: up to how many nodes (512 against 1024 threads, us).  One node per CU gains on the nodes
// that reject and loses on leaves, which are loaded and worked on in turns.
// Rows that the 512-thread kernels would stream again in every rejected round: k = 4 up to 1536 nodes (bf16 rows of
// 100 thousand, 672 nodes 100 -> 60, 1533 145 -> 109), k = 3, where leaves are a larger part, to 1440 (1391 113 -> 101,
// 1495 of 100001 115 -> 116), k = 2 to 1024 (620 75 -> 51, 1023 84 -> 76, 1920 124 -> 140).  Rows that use little more
// than half of their registers (66048: nine of sixteen chunks per lane) or spill them (152064: twenty) sooner
// meet their end: k = 3 1280 (152064, 1235 167 -> 155, 1495 171 -> 182), k = 2 896 (66048, 868 56.7 -> 51.8, 961 58.6 ->
// 59.1) and, unaligned or spilling, 832 (70001, 775 57.8 -> 57.5, 868 59.8 -> 60.8; 152064, 775 119 -> 114, 961 121 ->
// 131; 140001 RRSw, 868 120 -> 123).  Without the draft call's records, whose 512-thread form reads more, always up to
// 1024 and 1536 (152064, 1023 195 -> 168).
// Rows of which a CU holds two 512-thread nodes (more than eight chunks per lane): some way into the second round
// of one node per CU.  k > 2 up to 512 nodes (504 of 50257 39.7 -> 34.6), k = 2 to 384 (372 of 34000 18.0 -> 17.1, 434
// 18.7 -> 20.6; fp32 17000, 372 14.1 -> 14.1, 420 14.6 -> 15.1), unaligned to 448 (434 of 50257 26.1 -> 25.5).  Aligned
// rows without records from 257 nodes on only (248 of 34000 21.0 -> 21.2, 372 21.8 -> 21.6, 504 31.7 -> 30.2).
// Shorter rows: unaligned bf16 ones up to 256 nodes (248 of 32001 18.2 -> 17.2; aligned 24000 13.7 -> 13.8, RRSw 15.0 ->
// 15.5; fp32 12001 RRSw 13.3 -> 13.6; without records aligned ones 7 to 18 % slower).
// Nodes with children here and leaves streamed, in two launches, was slower than either (k = 4, 2688 nodes
// of 152064: 216 + 133 against 268).
static int64_t wide_rrs_nodes(const mdsd_problem* pb, const Params& P)
{
    const bool records = P.stats_in != nullptr;
    switch (resident_chunks(pb)) {
    case 4: return 0;
    case 8: return pb->dtype == MDSD_BF16 && P.masked ? kWideMaxNodes : 0;
    case 16: return P.k > 2 ? 512 : P.masked ? 448 : 384;
    default: break;
    }
    if (P.k > 3) return 1536;
    const bool spills = wide_chunks(P) == 20;
    if (!records || !(spills || P.row_chunks <= 9 * mdsd_wide::kThreads)) return P.k < 3 ? 1024 : records ? 1440 : 1536;
    return P.k == 3 ? 1280 : P.masked || spills ? 832 : 896;
}
static int wide_verify_chunks(int method, const mdsd_problem* pb, const Params& P, bool path)
{
    if (pb->kind != MDSD_LOGITS) return 0;
    if (method == kSpecHub) return wide_spechub_chunks(pb, P, path);
    const int64_t nodes = (int64_t)P.B * P.N;
    if (path || nodes > wide_rrs_nodes(pb, P)) return 0;
    if (resident_chunks(pb) == 16 && !P.stats_in && !P.masked && nodes <= kWideMaxNodes) return 0;
    return wide_chunks(P);
}
// Draft, up to 128 nodes with children (12 and 120 nodes, 512 against 1024 threads): SpecHub on bf16 rows that are
// resident either way, from 2400 chunks on (rows of 20000 5.62 -> 5.52 and 5.81 -> 5.70 us, 24001 6.62 -> 6.24 and 6.81 ->
// 6.57, 32000 6.37 -> 6.14 and 6.73 -> 6.63; 16640 5.45 -> 5.40 and 5.59 -> 5.72; fp32 rows of 12000 4.84 -> 4.86 and 4.96 ->
// 5.05), and RRS on aligned fp32 rows that 512 threads would stream (k = 2, 16500 5.29 -> 4.59 and 6.22 -> 5.04, 32000 6.86 ->
// 5.49 and 8.84 -> 7.11; k = 4, 20000 5.85 -> 4.99 and 6.67 -> 5.58).  Other resident rows of the RRS methods lose up to 6 %
// (fp32 9000, bf16 16640 to 32000: -0.3 to +6).  Since every draw crosses one barrier, more of the rows that 512 threads stream
// would gain, for which there is no kernel of 1024: k = 4 below 4608 chunks (16500 5.42 -> 4.77), fp32 32001 6.84 -> 5.95, RRSw
// 32000 7.94 -> 6.58, SpecHub 32000 7.08 -> 6.51, bf16 50304 RRS 7.12 -> 6.28, RRSw 8.33 -> 7.42, SpecHub 7.94 -> 7.48.
static bool wide_draft(int method, const mdsd_problem* pb, const Params& P)
{
    const int64_t nodes = (int64_t)P.B * (P.first_child ? P.N : P.n_internal);
    if (pb->kind != MDSD_LOGITS || nodes > kWideMaxNodes / 2) return false;
    if (method == kSpecHub) return pb->dtype == MDSD_BF16 && P.row_chunks > 2400 && P.row_chunks <= 8 * kWG;
    return method == kRRS && pb->dtype == MDSD_FP32 && !P.masked &&
           P.row_chunks > (P.k > 2 ? 9 : 8) * kWG && P.row_chunks <= 16 * kWG;
}

// SpecHub nodes of more than 64 chunks per row, from this many on: one wavefront per node with the rows
// in registers and more wavefronts on a SIMD (60000 nodes of 1000 bf16 elements 68 -> 55 us, of 2000 90 ->
// 77; 8000 nodes 11.3 against 11.8 us); bf16 rows of more than 128 chunks sooner (1500 elements, 9000 nodes 16.2 ->
// 16.2, 15000 23.2 -> 20.6; fp32 rows of 250 chunks 17.4 and 20.1).  The RRS methods gain from their groups
// at every size (119 -> 80, 146 -> 100 us).
// Path-only from 2048 trees on (4000 trees, 1000 elements 25.4 -> 22.6 us, 2000 elements 33.5 -> 29.7).
constexpr int64_t kWaveSpecHubMinNodes = 16384, kWaveSpecHubMinNodesLong = 10240, kWaveSpecHubMinPathTrees = 2048;

// lanes per node of the verify kernels for short rows; 0: another build takes the call
static int verify_lanes(int method, int dtype, const Params& P, bool path)
{
    const int64_t nodes = (int64_t)P.B * (path ? 1 : P.N);
    const int64_t wave_from = path ? kWaveSpecHubMinPathTrees
                              : dtype == MDSD_BF16 && P.row_chunks > 128 ? kWaveSpecHubMinNodesLong
                                                                         : kWaveSpecHubMinNodes;
    if (method == kSpecHub && P.row_chunks > 64 && nodes >= wave_from) return 0;
    return group_lanes(P.row_chunks, nodes, !path && P.accept_depth ? P.N : 1, path);
}

// path == false: one workgroup per node.  path == true: one workgroup per tree.
static void launch_verify(int method, const mdsd_problem* pb, const Params& P, bool path, hipStream_t st)
{
    const bool lg = pb->kind == MDSD_LOGITS;
    if (const int lanes = verify_lanes(method, pb->dtype, P, path)) {
        (method == kSpecHub ? launch_group_spechub : method == kRRS ? launch_group_rrs : launch_group_rrsw)(
            lanes, pb->dtype, lg, path, st, P);
        return;
    }
    int nit = resident_chunks(pb);
    const dim3 grid = path ? dim3((unsigned)P.B) : node_grid(P, nit), block(kWG);
    switch (small_build(pb)) {
    case 1: mdsd_wave::launch_spechub(pb->dtype, lg, path, grid, st, P); return;  // verify_lanes() left it SpecHub nodes
    case 2: mdsd_pair::launch_verify(method, pb->dtype, lg, path, grid, st, P); return;
    case 4: mdsd_quad::launch_verify(method, pb->dtype, lg, path, grid, st, P); return;
    default: break;
    }
    if (const int wide = wide_verify_chunks(method, pb, P, path)) {
        if (method == kSpecHub)
            mdsd_wide::launch_spechub(pb->dtype, wide, path, path ? grid : node_grid(P, wide), st, P);
        else
            (method == kRRS ? mdsd_wide::launch_rrs : mdsd_wide::launch_rrsw)(pb->dtype, wide, node_grid(P, wide), st, P);
        return;
    }
    // Rows of eight chunks per lane, the draft call's records at hand, and a batch that fills the chip
    // several times over: 256 threads per node with sixteen chunks per lane, four nodes per CU
    // instead of three (config-3 rows, 31 nodes per tree: B = 80 41.8 -> 41.1 us, B = 128 58.7 -> 56.6 us,
    // B = 1024 437 -> 410 us; B = 64 33.3 -> 34.3 us and B = 32 21.5 -> 23.5 us, hence the bound)
    const bool half_width = lg && nit == 8 && !path && P.stats_in != nullptr &&
                            (int64_t)P.B * P.N >= kHalfWidthMinNodes;
    if (half_width && method == kSpecHub) {
        mdsd_half::launch_spechub(pb->dtype, rows_need_mask(pb), grid, st, P);
        return;
    }
    if (half_width) {
        mdsd_half::launch_rrs(method == kRRSw, pb->dtype, rows_need_mask(pb), grid, st, P);
        return;
    }
    if (method == kSpecHub && lg && nit > 0) {
        launch_spechub_resident(pb->dtype, nit, rows_need_mask(pb), path, grid, block, st, P);
        return;
    }
    if (method != kSpecHub && lg && nit > 0) {
        (method == kRRSw ? launch_rrsw_resident : launch_rrs_resident)(pb->dtype, nit, rows_need_mask(pb), path, grid, block, st,
                                                                       P);
        return;
    }
    // The generic RRS rounds hold many registers beside two resident rows (8 chunks per lane and
    // row: more than 200, one workgroup per CU): from that size on the rows are streamed, which
    // measures faster (config 3, rrsw_verify: 117 -> 82 us).
    if (method != kSpecHub && nit >= 8) nit = 0;
    if (method == kSpecHub)
        launch_verify_generic_spechub(pb->dtype, lg, nit, path, grid, block, st, P);
    else if (method == kRRS)
        launch_verify_generic_rrs(pb->dtype, lg, nit, path, grid, block, st, P);
    else
        launch_verify_generic_rrsw(pb->dtype, lg, nit, path, grid, block, st, P);
}

// Draft, 256 threads per node: chunks per lane, 0 = not.  Half the reductions per element, worth more than the longer chain of
// a node once the nodes with children do not fit the chip at once (512 -> 256 threads, us a call, 31-node trees; the same
// bits).  Rows of four chunks per lane at 512 threads: bf16 12000, 960 nodes with children SpecHub 10.0 -> 10.4, 1920 16.1 -> 14.8,
// RRS 14.0 -> 13.2, RRSw 16.5 -> 14.5; fp32 7000, 1920 14.6 -> 13.0.  Eight chunks, RRSw: 32000, 960 17.1 -> 18.1, 1920 30.3 ->
// 29.1, 3840 51.7 -> 50.6; the others lose (SpecHub 1920 28.7 -> 31.8, RRS 26.8 -> 27.1).
static int half_draft_chunks(int method, const mdsd_problem* pb, const Params& P, int nit)
{
    const int64_t nodes = (int64_t)P.B * (P.first_child ? P.N : P.n_internal);
    if (pb->kind != MDSD_LOGITS || nodes < 1536) return 0;
    return nit == 4 ? 8 : nit == 8 && method == kRRSw && nodes >= 1920 ? 16 : 0;
}

static void launch_draft(int method, const mdsd_problem* pb, const Params& P, hipStream_t st)
{
    const bool lg = pb->kind == MDSD_LOGITS;
    if (const int lanes = group_lanes(P.row_chunks, (int64_t)P.B * (P.first_child ? P.N : P.n_internal), 1, false)) {
        launch_group_draft(method, lanes, pb->dtype, lg, st, P);
        return;
    }
    int nit = resident_chunks(pb);
    // Rows of sixteen chunks per lane are streamed: the draft kernel with such a row in registers
    // fits two workgroups on a CU, the streaming one four, and its one-sweep statistics are the
    // cheaper (V = 50304, B = 64: spechub_draft 33.7 -> 24.7 us, rrsw_draft 47.2 -> 26.8 us).  At
    // eight chunks per lane the row in registers wins (V = 32000: 18.8 against 19.4 us).
    // SpecHub on probabilities the same, in one sweep without exponentials (fp32 32000, 480 nodes with and without
    // children 11.2 -> 8.9 us, 15 8.1 -> 6.1, 4000 47.3 -> 45.4; bf16 60000 12.2 -> 9.3, 9.1 -> 7.1, 55.3 -> 53.0; eight chunks
    // per lane lose in large batches: bf16 32000, 4000 nodes 23.0 -> 30.5); the RRS methods, which need no maximum, gain
    // nothing (8.3 and 8.3) and stay in registers.
    if (nit == 16 && (lg || method == kSpecHub)) nit = 0;
    const dim3 grid = node_grid(P, nit), block(kWG);
    switch (small_build(pb)) {
    case 2: mdsd_pair::launch_draft(method, pb->dtype, lg, st, P); return;
    case 4: mdsd_quad::launch_draft(method, pb->dtype, lg, st, P); return;
    default: break;
    }
    if (wide_draft(method, pb, P)) {
        mdsd_wide::launch_draft(method, node_grid(P, 4), st, P);
        return;
    }
    const int es = pb->dtype == MDSD_FP32 ? 4 : 2;
    const bool masked = ((uintptr_t)pb->draft & 15) || ((pb->ld_d * es) & 15) || (pb->V % (16 / es));
    if (const int half = half_draft_chunks(method, pb, P, nit)) {
        mdsd_half::launch_draft(method, pb->dtype, half, masked, grid, st, P);
        return;
    }
    if (method == kSpecHub)
        launch_draft_spechub(pb->dtype, lg, nit, masked, grid, block, st, P);
    else if (method == kRRS)
        launch_draft_rrs(pb->dtype, lg, nit, masked, grid, block, st, P);
    else
        launch_draft_rrsw(pb->dtype, lg, nit, masked, grid, block, st, P);
}

static int walk(const mdsd_problem* pb, const int32_t* outcome, const int32_t* token,
                int32_t* accept_depth, int32_t* emitted, hipStream_t st)
{
    int W = 0;  // lanes per tree
    if (pb->N <= 64) {
        W = 1;
        while (W < pb->N) W *= 2;
    }
    const int64_t waves = W ? ((int64_t)pb->B * W + 63) / 64 : (int64_t)pb->B;
    const int waves_per_block = 4;
    hipLaunchKernelGGL(tree_walk_kernel, dim3((unsigned)((waves + waves_per_block - 1) / waves_per_block)),
                       dim3(64 * waves_per_block), 0, st, outcome, token, pb->B, pb->N, W, pb->k, pb->depth,
                       pb->first_child, accept_depth, emitted);
    return hipGetLastError() == hipSuccess ? MDSD_OK : MDSD_E_LAUNCH;
}

// bytes of workspace the full verify calls take when they walk the trees themselves
static size_t walk_workspace_bytes(int B) { return B > 0 ? (size_t)B * sizeof(int32_t) : 0; }

// tree_count: per-tree arrival counters (zero on entry) when the kernel is to walk the trees
// itself, nullptr when the walk is a launch of its own
static int verify_entry(int method, const mdsd_problem* pb, const int32_t* tokens, const float* u,
                        const mdsd_result* out, bool path, int32_t* tree_count, void* stream)
{
    Params P = {};
    const int rc = validate(pb, method, true, &P);
    if (rc == kEmptyBatch) return MDSD_OK;
    if (rc != MDSD_OK) return rc;
    if (!tokens || !u || !out || !out->outcome || !out->token) return MDSD_E_NULL;
    if ((out->accept_depth == nullptr) != (out->emitted == nullptr)) return MDSD_E_NULL;
    if (path && !out->accept_depth) return MDSD_E_NULL;
    if (path && out->resid_prob) return MDSD_E_UNSUPPORTED;
    P.accept_depth = out->accept_depth;
    P.emitted = out->emitted;
    // short rows: where a workgroup holds whole trees it walks them without counting arrivals
    const int lanes = path ? 0 : verify_lanes(method, pb->dtype, P, false);
    const int64_t nodes = (int64_t)P.B * P.N;
    const bool trees_whole = lanes && out->accept_depth && walks_in_workgroups(lanes, P.N, P.k, nodes);
    const bool walk_inside = !path && out->accept_depth && (tree_count || trees_whole);
    P.tree_count = walk_inside && !trees_whole ? tree_count : nullptr;
    if (pb->first_child && !lanes) P.n_internal = table_by_tree(method, pb);
    P.tokens = tokens;
    P.u = u;
    P.outcome = out->outcome;
    P.token = out->token;
    P.resid_mass = out->resid_mass;
    P.flags = out->flags;
    P.resid_prob = out->resid_prob;
    P.stats_in = pb->draft_stats;
    hipStream_t st = (hipStream_t)stream;
    (void)hipGetLastError();
    launch_verify(method, pb, P, path, st);
    if (hipGetLastError() != hipSuccess) return MDSD_E_LAUNCH;
    if (path || walk_inside) return MDSD_OK;  // the walk is part of the kernel
    if (out->accept_depth) return walk(pb, out->outcome, out->token, out->accept_depth, out->emitted, st);
    return MDSD_OK;
}

// the full verify calls: a workspace, when given, holds the trees' arrival counters
static int verify_with_workspace(int method, const mdsd_problem* pb, const int32_t* tokens, const float* u,
                                 const mdsd_result* out, void* ws, size_t ws_bytes, void* stream)
{
    if (ws && pb && ws_bytes < walk_workspace_bytes(pb->B)) return MDSD_E_WORKSPACE;
    if (ws && ((uintptr_t)ws & 3)) return MDSD_E_ALIGN;
    return verify_entry(method, pb, tokens, u, out, false, (int32_t*)ws, stream);
}

// ---------------------------------------------------------------- arrival counters owned by the library
// For callers that cannot allocate a workspace (code under HIP graph capture, serving loops that
// must not call hipMalloc): the arrival counters of up to MDSD_STATIC_MAX_TREES trees in a
// file-scope device array, zero when the code object is loaded and left zero by every call.  Each
// GPU holds its own copy at its own address; the array's name is a host-side stand-in, so the
// address on the current device is asked for once per device and used from then on.
static __device__ __align__(256) int32_t scratch[MDSD_STATIC_MAX_TREES];

static constexpr int kMaxDevices = 64;
static std::atomic<int32_t*> scratch_on_device[kMaxDevices];

static int static_tree_counters(int32_t** out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return MDSD_E_LAUNCH;
    int32_t* ptr = scratch_on_device[dev].load(std::memory_order_acquire);
    if (ptr == nullptr) {
        // two threads asking at once get the same answer
        if (hipGetSymbolAddress((void**)&ptr, HIP_SYMBOL(scratch)) != hipSuccess || ptr == nullptr) {
            (void)hipGetLastError();
            return MDSD_E_LAUNCH;
        }
        scratch_on_device[dev].store(ptr, std::memory_order_release);
    }
    *out = ptr;
    return MDSD_OK;
}

static int draft_entry(int method, const mdsd_problem* pb, const float* u, int32_t* tokens,
                       int32_t* hub, int32_t* flags, void* stream)
{
    Params P = {};
    const int rc = validate(pb, method, false, &P);
    if (rc == kEmptyBatch) return MDSD_OK;
    if (rc != MDSD_OK) return rc;
    if (!u || !tokens) return MDSD_E_NULL;
    if (pb->first_child) P.n_internal = table_by_tree(method, pb);
    P.u = u;
    P.tokens_out = tokens;
    P.hub_out = hub;
    P.flags = flags;
    P.stats_out = pb->draft_stats;
    hipStream_t st = (hipStream_t)stream;
    (void)hipGetLastError();
    launch_draft(method, pb, P, st);
    return hipGetLastError() == hipSuccess ? MDSD_OK : MDSD_E_LAUNCH;
}

// Steps, 256 threads per node instead of 512 (half the reductions and barriers per element, all nodes with children of the
// serving batch on the chip at once, but twice the chain per node): from how many nodes on (512 -> 256 threads, us a
// step, 31-node trees unless noted).  Rows of four chunks per lane at 512 threads, k = 2: bf16 12000, 1488 nodes
// SpecHub 21.3 -> 21.0, RRS 22.3 -> 22.5, 1736 24.2 -> 23.2, 26.9 -> 25.4, 3968 47.1 -> 39.0, 49.6 -> 43.7; fp32 7001,
// 1240 18.0 -> 20.3, 1736 23.7 -> 22.4, RRSw 29.0 -> 26.5.  Eight chunks, SpecHub on aligned rows: bf16 32000, 1736 44.4
// -> 45.2, 1984 48.7 -> 46.9, 26000 42.4 -> 39.8.  The others of eight chunks: SpecHub 28001, 1984 46.5 -> 47.7, 2480 56.5
// -> 59.8, 2976 65.7 -> 65.0; RRS 32000, 2480 60.5 -> 62.1, 2976 69.1 -> 67.9, 3968 87.9 -> 83.9, RRSw 64.7 -> 65.6, 73.4 ->
// 71.5.  k = 4, whose nodes wait longest for one another, as those (12000, 1680 24.0 -> 25.8; 30000, 2310 53.4 -> 56.7).
static bool half_width_step(int method, const Params& P, int nit)
{
    const int64_t nodes = (int64_t)P.B * P.N;
    if (nit == 0 || nit > 8) return false;
    if (P.k > 2) return nodes >= 2900;
    return nodes >= (nit == 4 ? 1600 : method == kSpecHub && !P.masked ? 1900 : 2900);
}

// Steps, 1024 threads per node: chunks per lane, 0 = another build takes the call.  Later than in the verify calls, since
// the draft gains from them too (512 -> 1024 threads, us a step, 31-node trees unless noted).  256 nodes run at once, so
// that the gain ends a little before a multiple of that.
// Rows of eight chunks per lane at 512 threads, up to 384 nodes where unaligned or long: bf16 20001, 372 nodes SpecHub 17.4
// -> 16.6, RRSw 20.9 -> 19.4, 32000 19.5 -> 19.0, 23.0 -> 22.1, 496 23.9 -> 24.3, 25.9 -> 26.1; 20000 15.6 -> 15.6.  Sixteen: SpecHub
// to 384 (50304, 372 27.4 -> 25.5, 434 29.1 -> 30.6); RRS methods, k = 2, to 640 (50304, 558 45.2 -> 43.9), fp32 rows and those of
// less than 5000 chunks to 448 (34000, 403 26.3 -> 24.3, 496 28.7 -> 30.2; fp32 24000 RRSw, 496 31.2 -> 30.8, 620 36.1 -> 39.8); k = 1
// to 256 (50304, 250 24.8 -> 23.9, 400 34.9 -> 41.8); k = 3 to 768 (13-node trees, 50304, 650 42.0 -> 40.7, 780 43.9 -> 46.3), k = 4
// to 870 (21-node trees, 819 48.8 -> 45.9, 861 49.1 -> 47.6, 966 49.8 -> 51.8).
// Streamed rows: SpecHub to 640 (128256, 372 60.2 -> 50.9, 620 85.5 -> 78.6, 744 90.7 -> 91.1; 152064, 558 96.6 -> 85.3).  RRS
// methods, by k and by length (more than 9216 chunks; 16384), unaligned rows less far:
//   1  256 (70001, 250 39.2 -> 32.9, 400 48.6 -> 56.4; 152064, 400 90.4 -> 94.8)
//   2  as far as the verify call takes 1024 threads (70001, 868 75.2 -> 79.5), long rows 1300 (128256, 1240 159 -> 147, 1364 161 ->
//      160), longest 1100 (152064 RRSw, 1054 160 -> 159, 1240 190 -> 189); unaligned 1024 (100001, 1054 108 -> 115, 1240 126 -> 134;
//      128257, 1147 150 -> 149), longest 780 (152065 RRSw, 713 144 -> 140, 806 148 -> 155)
//   3  1280 (70001, 1300 97.5 -> 99.1), longer 1950 (100000, 1898 162 -> 163; 152064, 1300 192 -> 165, 2054 239 -> 247), unaligned 1400
//      (100001, 1300 133 -> 127, 1495 136 -> 143; 152065, 1495 200 -> 206)
//   4  1536 (70001, 1491 120 -> 108, 1701 121 -> 126), longer 2500 (100000, 2394 205 -> 190, 2793 210 -> 217; 128256, 2394 255 -> 228;
//      152064, 2205 254 -> 253, 2394 305 -> 274, 2793 310 -> 317, 2688 with a quarter of them nearly uniform 312 -> 330), unaligned
//      1800 or 1950 (100001, 1701 165 -> 153, 1890 168 -> 173; 128257, 1890 211 -> 196, 2058 215 -> 214; 152065, 2058 254 -> 260).
static int wide_step_chunks(int method, const mdsd_problem* pb, const Params& P)
{
    const int nit = resident_chunks(pb), wide = wide_chunks(P);
    const bool longer = P.row_chunks > 9 * mdsd_wide::kThreads;
    const int64_t nodes = (int64_t)P.B * P.N;
    // Up to 256 nodes SpecHub stays where its verify call would run (aligned rows of sixteen chunks, streamed ones of more than
    // sixteen at 1024 threads): the same sums in the same order, and the step gives what the two calls give bit for bit.  Rows of
    // eight chunks are not kept back: their draft is the same at any width, only the sums over the target row change their order.
    if (method == kSpecHub && nodes <= kWideMaxNodes && nit != 8 && !(nit == 16 ? P.masked : wide == 16)) return 0;
    int64_t most = 0;
    if (nit == 8)
        most = P.masked || P.row_chunks > 3072 ? 384 : 0;
    else if (nit == 16 && method == kSpecHub)
        most = 384;
    else if (nit == 16)
        most = P.k > 3 ? 870 : P.k == 3 ? 768 : P.k == 1 ? 256 : pb->dtype == MDSD_FP32 || P.row_chunks < 5000 ? 448 : 640;
    else if (nit == 0 && method == kSpecHub)
        most = 640;
    else if (nit == 0 && P.k == 1)
        most = 256;
    else if (nit == 0 && P.k == 2)
        most = !longer    ? wide_rrs_nodes(pb, P)
               : P.masked ? (wide == 20 ? 780 : 1024)
                          : (wide == 20 ? 1100 : 1300);
    else if (nit == 0 && P.k == 3)
        most = !longer ? 1280 : P.masked ? 1400 : 1950;
    else if (nit == 0)
        most = !longer ? 1536 : !P.masked ? 2500 : P.row_chunks > 14000 ? 1950 : 1800;
    return nodes <= most ? wide : 0;
}

// Steps whose two calls one after the other are faster than one launch.  A draft kernel runs four nodes on a CU, 1024 at once,
// but the step kernels of long rows run three (streamed rows, 768), two (sixteen chunks per lane, 512) or one (1024 threads,
// 256): where the nodes with children fill a little more than the chip holds, what is left of them drafts by itself.  By
// `inner`, the number of nodes with children (two launches -> one, us a step, 31-node trees, k = 2, unless noted):
// Streamed rows, 769 to 1024 of them, RRS 70001, 750 99.1 -> 94.1, 795 109 -> 110, 900 116 -> 118, 945 118 -> 121, 1065 136 -> 127;
// RRSw 115 -> 117, 121 -> 124, 123 -> 127, 142 -> 133; RRS 152064, 795 216 -> 222, 1065 279 -> 263; k = 1 100000, 800 112 -> 116; RRSw, k =
// 3, to 840 only (13-node trees, 128256, 800 248 -> 252, 860 259 -> 257); SpecHub never (100000, 820 147 -> 140).  RRS, k = 4, up to
// 2450 nodes on unaligned rows (152065, 2058 247 -> 254, 2394 303 -> 307, 2604 307 -> 308).
// Sixteen chunks per lane, RRS 50304, 480 51.3 -> 49.0, 525 54.7 -> 58.1, 720 68.2 -> 71.0, 870 80.3 -> 79.7, 1065 98.4 ->
// 93.9, 1215 109 -> 106, 1455 122 -> 123, 1785 145 -> 148, 2910 230 -> 235; RRSw 54.1 -> 51.3, 56.8 -> 61.5, 71.4 -> 75.6,
// 83.1 -> 83.9, 102 -> 98.4, 114 -> 111, 128 -> 129, 152 -> 156, 237 -> 245; fp32 24000 RRS 675 53.2 -> 53.9, 840 63.1 ->
// 62.4; k = 1 50304, 416 39.0 -> 37.2, 560 44.8 -> 49.4, 1200 80.4 -> 82.8; k = 3 (42001, RRSw, 13-node trees, 400 62.0 ->
// 57.2, 528 69.8 -> 71.4, 584 76.9 -> 75.4, 952 109 -> 111, 1200 138 -> 137, 1848 196 -> 203); SpecHub 33000, 1455 87.2 ->
// 86.9, 1785 99.1 -> 101, 4350 221 -> 232.
// Between the sizes that 1024 threads gain at and those that 512 do: bf16, k = 2, from the third node of every CU on while
// the verify call still takes 1024 threads (100000, 496 nodes 64.1 -> 57.8, 558 68.8 -> 69.8, 744 79.9 -> 81.6, 806 85.5 ->
// 89.6, 1147 125 -> 116; 138048, 675 110 -> 116; fp32 40000, 713 56.6 -> 56.0, unaligned 45445, 720 68.9 -> 71.6); RRS on
// longer rows from 1024 nodes on (152064, 961 149 -> 150, 1054 154 -> 163), unaligned from 512 on (152065, 558 109 -> 112,
// 713 133 -> 135; 868 at 512 threads 149 -> 146); k = 1, long rows, from 256 nodes on (128256, 400 69.8 -> 77.8, 700 96.4 ->
// 103, 850 of 100000 94.8 -> 90.8), the longest for a little (138886, 272 64.7 -> 69.0; 152064, 400 97.1 -> 90.4).  Sixteen
// chunks, k > 2, fewer than 256 of them but too many nodes for 1024 threads (65500, 819 61.7 -> 65.0, 1050 66.0 -> 67.5;
// 38000 41.6 -> 41.1, unaligned 38156 39.4 -> 40.2).
static bool step_in_two(int method, const mdsd_problem* pb, const Params& P, int nit, int wide)
{
    const int64_t nodes = (int64_t)P.B * P.N, inner = (int64_t)P.B * ((P.N - 1) / P.k);
    const bool bf16 = pb->dtype == MDSD_BF16;
    if (nit == 16) {
        if (wide) return false;
        if (method == kSpecHub) return inner > 1550;
        if (P.k > 2 && inner <= 256) return P.row_chunks > (P.masked ? 4500 : 5000);
        if (inner > 1350) return true;
        if (P.k > 2) return inner <= 1024 && (inner > 900 || (method == kRRSw && inner > 512 && inner <= 545));
        return inner > 512 && (P.k == 1 || inner <= (bf16 || method == kRRSw ? 1024 : 750));
    }
    if (nit != 0 || method == kSpecHub) return false;
    const int chunks = wide_chunks(P);  // 0: too long for 1024 threads
    const bool longer = P.row_chunks > 9 * mdsd_wide::kThreads;
    if (P.k == 2 && (bf16 || P.masked) && chunks && nodes > 2 * kWideMaxNodes) {
        if (P.row_chunks < 18 * mdsd_wide::kThreads && nodes <= wide_rrs_nodes(pb, P)) return true;
        if (chunks == 20 && method == kRRS && (P.masked ? nodes <= wide_rrs_nodes(pb, P) : wide && nodes > 4 * kWideMaxNodes))
            return true;
    }
    if (wide) return false;
    if (P.k == 1 && longer && chunks && (chunks < 20 ? inner <= 600 : nodes <= 320)) return true;
    if (P.k > 3) return method == kRRS && longer && chunks && nodes <= 2450;
    return inner > 768 && (P.k < 3 ? inner <= 1024 : method == kRRSw && inner <= 840);
}

// Lanes per node of the step kernels for short rows; 0: another build takes the call.  As in the verify calls, by the number
// of all nodes; a draft call goes by those with children and may take more lanes, whose sums have another order.  SpecHub in
// large batches of more than 64 chunks, whose verify calls take a wavefront per node, as well (4000 trees of 15 nodes, two
// launches -> one: bf16 1000 73.6 -> 64.3 us, fp32 1000 95.2 -> 79.3), but bf16 rows of more than 128 chunks up to 24576
// nodes only (1900, 18000 nodes 44.5 -> 41.9; 1300, 27000 50.2 -> 50.9; 1100, 60000 91 -> 102).
static int step_lanes(int method, int dtype, const Params& P)
{
    const int64_t nodes = (int64_t)P.B * P.N;
    if (method == kSpecHub && dtype == MDSD_BF16 && P.row_chunks > 128 && nodes > 24576) return 0;
    return group_lanes(P.row_chunks, nodes, P.accept_depth ? P.N : 1, false);
}

// A step's kernel that drafts and verifies every node in one launch; false: there is none for this call.
static bool launch_step(int method, const mdsd_problem* pb, const Params& P, hipStream_t st)
{
    if (pb->kind != MDSD_LOGITS || P.stats_out == nullptr || P.resid_mass || P.resid_prob) return false;
    if (const int lanes = step_lanes(method, pb->dtype, P)) {
        (method == kSpecHub ? launch_group_step_spechub
         : method == kRRS   ? launch_group_step_rrs
                            : launch_group_step_rrsw)(lanes, pb->dtype, st, P);
        return true;
    }
    const bool masked = rows_need_mask(pb);
    const int nit = resident_chunks(pb), wide = wide_step_chunks(method, pb, P), small = small_build(pb);
    const dim3 grid = node_grid(P, wide ? wide : nit);
    if (small == 1) return false;  // SpecHub in large batches
    if (small == 0 && step_in_two(method, pb, P, nit, wide)) return false;
    if (small == 2)
        mdsd_pair::launch_step(method, pb->dtype, masked, grid, st, P);
    else if (small == 4)
        mdsd_half::launch_step(method, pb->dtype, 4, masked, grid, st, P);
    else if (wide)
        (method == kSpecHub ? mdsd_wide::launch_step_spechub
         : method == kRRS   ? mdsd_wide::launch_step_rrs
                            : mdsd_wide::launch_step_rrsw)(pb->dtype, wide, masked, grid, st, P);
    else if (half_width_step(method, P, nit))
        mdsd_half::launch_step(method, pb->dtype, 2 * nit, masked, grid, st, P);
    else
        (method == kSpecHub ? launch_step_spechub : method == kRRS ? launch_step_rrs : launch_step_rrsw)(pb->dtype, nit, masked,
                                                                                                        grid, st, P);
    return true;
}

// draft and verification in one call, in one launch where there is a kernel for it
static int step_entry(int method, const mdsd_problem* pb, const float* u_draft, const float* u_verify, int32_t* tokens,
                      int32_t* hub, int32_t* draft_flags, const mdsd_result* out, int32_t* tree_count, void* stream)
{
    Params P = {};
    const int rc = validate(pb, method, true, &P);
    if (rc == kEmptyBatch) return MDSD_OK;
    if (rc != MDSD_OK) return rc;
    if (!u_draft || !u_verify || !tokens || !out || !out->outcome || !out->token) return MDSD_E_NULL;
    if ((out->accept_depth == nullptr) != (out->emitted == nullptr)) return MDSD_E_NULL;
    P.accept_depth = out->accept_depth;
    P.emitted = out->emitted;
    const int lanes = step_lanes(method, pb->dtype, P);
    const bool trees_whole = lanes && out->accept_depth && walks_in_workgroups(lanes, P.N, P.k, (int64_t)P.B * P.N);
    P.tree_count = out->accept_depth && !trees_whole ? tree_count : nullptr;
    if (pb->first_child && !lanes) P.n_internal = table_by_tree(method, pb);
    P.u_draft = u_draft;
    P.u = u_verify;
    P.tokens = P.tokens_out = tokens;
    P.hub_out = hub;
    P.draft_flags = draft_flags;
    P.outcome = out->outcome;
    P.token = out->token;
    P.resid_mass = out->resid_mass;
    P.flags = out->flags;
    P.resid_prob = out->resid_prob;
    P.stats_in = P.stats_out = pb->draft_stats;
    hipStream_t st = (hipStream_t)stream;
    (void)hipGetLastError();
    if (launch_step(method, pb, P, st)) {
        if (hipGetLastError() != hipSuccess) return MDSD_E_LAUNCH;
        if (P.accept_depth && !P.tree_count && !trees_whole) return walk(pb, P.outcome, P.token, P.accept_depth, P.emitted, st);
        return MDSD_OK;
    }
    const int drafted = draft_entry(method, pb, u_draft, tokens, hub, draft_flags, stream);
    return drafted != MDSD_OK ? drafted : verify_entry(method, pb, tokens, u_verify, out, false, tree_count, stream);
}

static int step_with_workspace(int method, const mdsd_problem* pb, const float* u_draft, const float* u_verify,
                               int32_t* tokens, int32_t* hub, int32_t* draft_flags, const mdsd_result* out, void* ws,
                               size_t ws_bytes, void* stream)
{
    if (ws && pb && ws_bytes < walk_workspace_bytes(pb->B)) return MDSD_E_WORKSPACE;
    if (ws && ((uintptr_t)ws & 3)) return MDSD_E_ALIGN;
    return step_entry(method, pb, u_draft, u_verify, tokens, hub, draft_flags, out, (int32_t*)ws, stream);
}

}  // namespace mdsd

// ---------------------------------------------------------------- C ABI
extern "C" {

size_t mdsd_workspace_bytes(const mdsd_problem* pb)
{
    // every intermediate of a node lives in registers and LDS; the workspace holds one arrival
    // counter per tree for the verify calls that walk the trees inside their kernel
    return pb ? mdsd::walk_workspace_bytes(pb->B) : 0;
}

int spechub_draft(const mdsd_problem* pb, const float* u, int32_t* tokens, int32_t* hub, int32_t* flags,
                  void* ws, size_t ws_bytes, void* stream)
{
    (void)ws;
    (void)ws_bytes;
    return mdsd::draft_entry(mdsd::kSpecHub, pb, u, tokens, hub, flags, stream);
}

int rrs_draft(const mdsd_problem* pb, const float* u, int32_t* tokens, int32_t* flags, void* ws,
              size_t ws_bytes, void* stream)
{
    (void)ws;
    (void)ws_bytes;
    return mdsd::draft_entry(mdsd::kRRS, pb, u, tokens, nullptr, flags, stream);
}

int rrsw_draft(const mdsd_problem* pb, const float* u, int32_t* tokens, int32_t* flags, void* ws,
               size_t ws_bytes, void* stream)
{
    (void)ws;
    (void)ws_bytes;
    return mdsd::draft_entry(mdsd::kRRSw, pb, u, tokens, nullptr, flags, stream);
}

int spechub_verify(const mdsd_problem* pb, const int32_t* tokens, const float* u, const mdsd_result* out,
                   void* ws, size_t ws_bytes, void* stream)
{
    return mdsd::verify_with_workspace(mdsd::kSpecHub, pb, tokens, u, out, ws, ws_bytes, stream);
}

int spechub_verify_static(const mdsd_problem* pb, const int32_t* tokens, const float* u, const mdsd_result* out,
                          void* stream)
{
    if (!pb) return MDSD_E_NULL;
    if (pb->B > MDSD_STATIC_MAX_TREES) return MDSD_E_WORKSPACE;
    if (!out || !out->accept_depth || !out->emitted) return MDSD_E_NULL;
    int32_t* counters = nullptr;
    const int rc = mdsd::static_tree_counters(&counters);
    if (rc != MDSD_OK) return rc;
    return mdsd::verify_entry(mdsd::kSpecHub, pb, tokens, u, out, false, counters, stream);
}

int rrs_verify(const mdsd_problem* pb, const int32_t* tokens, const float* u, const mdsd_result* out,
               void* ws, size_t ws_bytes, void* stream)
{
    return mdsd::verify_with_workspace(mdsd::kRRS, pb, tokens, u, out, ws, ws_bytes, stream);
}

int rrsw_verify(const mdsd_problem* pb, const int32_t* tokens, const float* u, const mdsd_result* out,
                void* ws, size_t ws_bytes, void* stream)
{
    return mdsd::verify_with_workspace(mdsd::kRRSw, pb, tokens, u, out, ws, ws_bytes, stream);
}

int spechub_step(const mdsd_problem* pb, const float* u_draft, const float* u_verify, int32_t* tokens, int32_t* hub,
                 int32_t* draft_flags, const mdsd_result* out, void* ws, size_t ws_bytes, void* stream)
{
    return mdsd::step_with_workspace(mdsd::kSpecHub, pb, u_draft, u_verify, tokens, hub, draft_flags, out, ws, ws_bytes,
                                     stream);
}

int rrs_step(const mdsd_problem* pb, const float* u_draft, const float* u_verify, int32_t* tokens, int32_t* draft_flags,
             const mdsd_result* out, void* ws, size_t ws_bytes, void* stream)
{
    return mdsd::step_with_workspace(mdsd::kRRS, pb, u_draft, u_verify, tokens, nullptr, draft_flags, out, ws, ws_bytes,
                                     stream);
}

int rrsw_step(const mdsd_problem* pb, const float* u_draft, const float* u_verify, int32_t* tokens, int32_t* draft_flags,
              const mdsd_result* out, void* ws, size_t ws_bytes, void* stream)
{
    return mdsd::step_with_workspace(mdsd::kRRSw, pb, u_draft, u_verify, tokens, nullptr, draft_flags, out, ws, ws_bytes,
                                     stream);
}

int spechub_verify_path(const mdsd_problem* pb, const int32_t* tokens, const float* u, const mdsd_result* out,
                        void* ws, size_t ws_bytes, void* stream)
{
    (void)ws;
    (void)ws_bytes;
    return mdsd::verify_entry(mdsd::kSpecHub, pb, tokens, u, out, true, nullptr, stream);
}

int rrs_verify_path(const mdsd_problem* pb, const int32_t* tokens, const float* u, const mdsd_result* out,
                    void* ws, size_t ws_bytes, void* stream)
{
    (void)ws;
    (void)ws_bytes;
    return mdsd::verify_entry(mdsd::kRRS, pb, tokens, u, out, true, nullptr, stream);
}

int rrsw_verify_path(const mdsd_problem* pb, const int32_t* tokens, const float* u, const mdsd_result* out,
                     void* ws, size_t ws_bytes, void* stream)
{
    (void)ws;
    (void)ws_bytes;
    return mdsd::verify_entry(mdsd::kRRSw, pb, tokens, u, out, true, nullptr, stream);
}

int mdsd_tree_walk(const mdsd_problem* pb, const int32_t* outcome, const int32_t* token,
                   int32_t* accept_depth, int32_t* emitted, void* stream)
{
    if (!pb) return MDSD_E_NULL;
    if (pb->B == 0) return MDSD_OK;
    if (!outcome || !token || !accept_depth || !emitted) return MDSD_E_NULL;
    if (pb->B < 1 || pb->N < 1 || pb->depth < 1) return MDSD_E_SHAPE;
    if (pb->k < 1 || pb->k > MDSD_MAX_K) return MDSD_E_K;
    (void)hipGetLastError();
    return mdsd::walk(pb, outcome, token, accept_depth, emitted, (hipStream_t)stream);
}

int mdsd_philox_uniform(uint64_t seed, uint32_t stream_id, int64_t rows, int32_t slots, float* out,
                        uint32_t* words, void* stream)
{
    if (rows < 0 || slots < 1) return MDSD_E_SHAPE;
    if (rows == 0) return MDSD_OK;
    if (!out && !words) return MDSD_E_NULL;
    const int64_t n = rows * ((slots + 3) >> 2);
    const int threads = 256;
    const int64_t blocks = (n + threads - 1) / threads;
    if (blocks > INT_MAX) return MDSD_E_SHAPE;
    (void)hipGetLastError();
    hipLaunchKernelGGL(mdsd::philox_uniform_kernel, dim3((unsigned)blocks), dim3(threads), 0,
                       (hipStream_t)stream, (uint32_t)seed, (uint32_t)(seed >> 32), stream_id, rows,
                       (int)slots, out, words);
    return hipGetLastError() == hipSuccess ? MDSD_OK : MDSD_E_LAUNCH;
}

const char* mdsd_strerror(int code)
{
    switch (code) {
    case MDSD_OK: return "ok";
    case MDSD_E_NULL: return "a required pointer is NULL";
    case MDSD_E_SHAPE: return "bad shape: B, N, V, ld, depth or tree/N mismatch";
    case MDSD_E_K: return "k out of range (SpecHub needs k == 2)";
    case MDSD_E_TEMP: return "temperature must be > 0";
    case MDSD_E_DTYPE: return "unknown dtype or kind";
    case MDSD_E_ALIGN: return "pointer not element-aligned, or target/draft rows differ modulo 16 bytes";
    case MDSD_E_WORKSPACE: return "workspace smaller than mdsd_workspace_bytes()";
    case MDSD_E_LAUNCH: return "HIP launch failed";
    case MDSD_E_UNSUPPORTED: return "output not available from this entry point";
    default: return "unknown status";
    }
}

int mdsd_version(void) { return 104; }

}  // extern "C"
