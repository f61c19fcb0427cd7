// Host-side launch planning of the layer sweep: GEMM tile choice, split-K factors and the
// layout of the per-chunk workspaces of one Block-GD step.  Pure C++ (no HIP types), so the
// CPU test suite compiles this unit on its own with AddressSanitizer and checks the sizing
// arithmetic against the launches it describes.
#pragma once
#include <stdint.h>

#include <vector>

namespace realq {
namespace plan {

// Tile shapes of the bf16 MFMA GEMM (the kernel asserts that its configurations match).
constexpr int64_t kBK = 32;                          // K slice
constexpr int64_t kLargeBM = 256, kLargeBN = 256;    // 8 waves
constexpr int64_t kSmallBM = 128, kSmallBN = 128;    // 4 waves
constexpr int64_t kLargeMinTiles = 256;              // the large tile once a launch has this many

int64_t tiles(int64_t M, int64_t N, bool large);
// tile: 0 = chosen from the shape, 1 = large, 2 = small
bool pick_large(int64_t M, int64_t N, int tile);
int64_t num_blocks(int64_t M, int64_t N, int tile);
// K range per split (a multiple of kBK) and the number of non-empty splits it gives.
int64_t k_per_split(int64_t K, int64_t splits);
int64_t effective_splits(int64_t K, int64_t splits);
// Split-K factor of the gradient GEMM (always the large tile): the smallest factor up to 16
// whose launch fills at least 97% of its last round of `cus` blocks, else the fullest one;
// every split keeps at least 256 tokens.
int64_t choose_splits(int64_t M, int64_t N, int64_t K, int cus);

// Row stride (elements) of a bf16 operand over the columns or rows of a module (activations, weight
// splits, Gram matrices, metrics): whole 128-byte lines.  Rows that start inside a line cost the residual products 5 to 25% (2048 x
// 4104 at 65664 tokens 33.2 ms on whole lines, 38.4 at 4104 elements; of an increment 20.1 and
// 25.6).  An odd number of lines gains nothing here, where K is a few thousand: 1024 x 8192 at 131072
// tokens 105 ms at 8192 elements, 112 at 8256 (and a copy of the activations to get there); Gram steps
// of 1024 x 8192 87 and 95 ms.
int64_t row_stride(int64_t n);

// Row stride (elements) of a bf16 GEMM operand over the tokens: whole 128-byte lines, an odd
// number of them.  A tile's loads walk 256 rows at one K offset; with a power-of-two stride those
// lines fall on a few memory channels (gradient product of 2048 x 4096 over 65536 tokens: 1.11 to
// 1.46 ms from run to run at a stride of 65536 elements, 0.93 ms at 65600).
int64_t operand_stride(int64_t n);

// Split-K factor of a product accumulated in float64 over `tiles` 256x256 tiles and K tokens with
// `passes` MFMA passes per tile: the cheapest by the time its rounds of `cus` tiles take at the GEMM's
// rate (about 30 ns per token, tile and pass) plus the write and read of its float32 slices (about 0.11
// us per tile and slice), from 1 or, with max_k > 0, from ceil(K / max_k), so that no split sums more
// than max_k tokens, up to 256 splits of at least 256 tokens (or that least number, where it is more:
// 2048 for 2^21 tokens at 1024 a sum).
int64_t choose_acc_splits(int64_t tiles, int64_t K, int passes, int cus, int64_t max_k);

// Whether such a symmetric product in one slice is as well formed in full, straight into its matrix
// (the same float32 sums): the other triangle's tiles against the slice's write and read and a launch
// (about 0.21 us per tile).  Unweighted Hessians, straight and in a slice: 4096 columns over 1024 tokens
// 103 and 146 us, 14336 over 1024 1.22 and 1.29 ms, over 2048 1.55 and 1.47; 512 over 16 (small
// tiles, whose launch takes as long as both of the slice's) 37 and 34 us.
bool straight_acc(int64_t M, int64_t K, int cus);

// Whether the pulled-back metric of m columns through m_next rows (and a dense metric) is small enough
// for float64 products straight from the float32 operands (one or two launches, bound by latency) rather
// than term splits, products and slice sums on the bf16 matrix cores (7 to 14 launches).  Measured,
// float64 / bf16-exact weights / others: 256 x 256 32 / 43 / 94 us, 512 x 1024 50 / 47 / 106, 64 x
// 4096 62 / 75 / 153, 1024 x 256 82 / 44 / 98; dense 512 x 512 82 / 177 / 179, 768 x 2048 205 / 287 /
// 305, 512 x 8192 1235 / 1009 / 1054, 2048 x 256 323 / 215 / 221.
bool pullback_small(int64_t m_next, int64_t m, bool dense);

// Rows of the panel from row r0 of an M x N product held as `slices` float32 slices: the most, in whole
// 256-row tiles, whose slices take at most `budget` bytes, and one tile at least.  A symmetric
// product's panel holds the columns up to its last row.
int64_t panel_rows(int64_t M, int64_t N, bool symmetric, int64_t slices, int64_t r0, int64_t budget);
// The least budget that needs no more panels than `budget` does (within 1%): panels of about equal
// bytes, since the launches of a last panel of a few rows of tiles leave most of the chip idle
// (4096 weighted columns over 65536 tokens: 5.6 ms with a last panel of 256 rows, 4.6 ms in one).
int64_t even_budget(int64_t M, int64_t N, bool symmetric, int64_t slices, int64_t budget);
// Bytes of the slices of `rows` rows from r0.
constexpr int64_t panel_bytes(int64_t N, bool symmetric, int64_t slices, int64_t r0, int64_t rows) {
    return 4 * slices * rows * (symmetric ? r0 + rows : N);
}

// Places of the T tokens in the token-minor arrays of a Block-GD state (residual base, transposed
// inputs, token weights).  A chunk's operand rows must start on 16 bytes, 8 tokens: when the chunks of Tc
// tokens of the batches of Tb do not (`apart`), each chunk starts on the next multiple of 8
// places and the places between hold no token (zero inputs).  Only where that leaves at most a
// sixteenth more places than tokens: the GEMMs' checked register path is slower on an unaligned
// chunk, but the padding of a few tokens would multiply the arrays (16 places for a batch of 9).
// Otherwise, and when every chunk is aligned as it is, token t has place t.  Layers of 1024 x 1024,
// 4 steps a block, with and without places apart: 30001 tokens in chunks of 1003 46 and 110 ms, 65536
// in batches of 1001 6.1 and 9.4 ms, of 63 12.6 and 20.5 ms, of 100 10.6 and 10.6 ms (bound by its
// launches); batches of 33 (26 ms) and 9 (71 ms) stay in order.
struct Places {
    int64_t T = 0, Tb = 0, Tc = 0;
    int64_t chunk = 0, batch = 0;  // places of a whole chunk and of a whole batch
    int64_t count = 0;             // places in all
    bool apart = false;
};
Places place_tokens(int64_t T, int64_t Tb, int64_t Tc, bool may_part = true);
constexpr int64_t place_of(const Places& L, int64_t t) {
    return L.apart ? t / L.Tb * L.batch + t % L.Tb / L.Tc * L.chunk + t % L.Tb % L.Tc : t;
}
// The token at place p < count, or -1.
constexpr int64_t token_at(const Places& L, int64_t p) {
    if (!L.apart) return p;
    const int64_t b0 = p / L.batch * L.Tb, c0 = p % L.batch / L.chunk * L.Tc, u = p % L.batch % L.chunk;
    return u < L.Tc && c0 + u < L.Tb && b0 + c0 + u < L.T ? b0 + c0 + u : -1;
}

// One token chunk of a Block-GD step: tokens [t0, t0 + len) of the calibration set, and the
// range [parts_off, parts_off + parts) of the loss-partial workspace its residual launch (or,
// with the clip, its clip launch) writes.
struct Chunk {
    int64_t t0, len, parts_off, parts;
};

struct StepPlan {
    int64_t bt0 = 0, Tn = 0;   // tokens of the step: [bt0, bt0 + Tn)
    int64_t splits = 1;        // split factor passed to every chunk's gradient GEMM
    int64_t gp_slices = 1;     // gradient slices the split-K workspace must hold (max over chunks)
    int64_t parts_total = 0;   // loss partials over all chunks
    std::vector<Chunk> chunks;
};

// Step t (0-based count of earlier Adam steps of the module) of a Block-GD sweep over m rows,
// nJ trailing columns and T tokens, with batches of Tb tokens (Tb = T: full batch) cut into
// chunks of Tc tokens.  clip_parts > 0: each chunk writes that many partials (the clip
// launch) instead of one per residual block.
StepPlan plan_step(int64_t m, int64_t nJ, int64_t T, int64_t Tb, int64_t Tc, int64_t t, int cus,
                   int64_t clip_parts);
// Chunks of a residual-loss pass over all T tokens (one partial per residual block).
std::vector<Chunk> plan_loss(int64_t m, int64_t T, int64_t Tc, int64_t* parts_total);

}  // namespace plan
}  // namespace realq
