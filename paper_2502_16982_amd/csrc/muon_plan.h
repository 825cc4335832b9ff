// Host-side launch planner of the Muon step: plain C++, no HIP include, so that it also builds with the host
// compiler alone (the sanitizer build of the tests does that).
//
// A plan turns a list of matrix shapes into: the orientation and padded extents of every matrix, the chunking of
// the list against the workspace, and the host image of the device tables (matrix records, elementwise tiles, one
// grouped-GEMM problem table and tile table per Newton-Schulz product).  Pointers inside the image are computed from
// the workspace base address and never followed on the host.
#pragma once
#include <cstddef>
#include <cstdint>
#include <vector>

#include "../../include/muon.h"
#include "muon_tables.h"

namespace muon {

struct MatPlan {
  int64_t rows, cols;
  int m, n, mp, np, transposed;
  int w_dtype, g_dtype;
  int tile;         // fine GEMM block tile = padding granule, in elements
  int chunk;
  bool coarse;      // some of its outputs are computed in coarse tiles
  bool gram;        // takes the Gram route (gram_route)
  int ew_tr, ew_tc; // 64x64 tiles in U's orientation (padded)
  size_t ns_bytes;  // X + Xt[0] (+ Xt[1], see x_buffers) + Ag + Bp
  size_t part_off;  // first partial (floats)
};

// Tile tables of one launch level (byte offsets in the table region).
struct TileSet {
  size_t sym = 0, poly = 0, apply = 0;          // Gram, polynomial, apply
  int n_sym = 0, n_poly = 0, n_apply = 0;
  bool strips = false;    // the tables hold 512 x 128 tiles (the launch then needs the larger LDS allocation)
  // the K loops of the launch's tiles are of nearly the same length (Gram product: n_pad; the other two: m_pad), so
  // the launch, in plain bf16, runs persistent blocks that take the planner's static assignment of tiles
  bool persistent_n = false, persistent_m = false;
  bool long_n = false, long_m = false;    // fp32: some K (Gram product: n_pad; the other two: m_pad) is over kF32LongK
  int tail_sym = 0, tail_poly = 0, tail_apply = 0;      // fp32: the last entries of a launch in whole entries that run in quarters behind it
  bool quarter_sym = false, quarter_poly = false, quarter_apply = false;   // fine launches that run as one block per quarter of an entry
  int few_sym = 0, few_poly = 0, few_apply = 0;   // quarters on the matrix cores: 1 with the longer ring, 2 (plain bf16) as one wave per 32 x 32;
                                                  // 3 (plain bf16, not in quarters): 128-wide with a ring of four slabs
};

// The Gram route.  X' = P X with P = a I + b A + c A A, A = X X^T commutes with everything made of A, so the next iteration's Gram
// matrix is P A P and two iterations in a row are one product with Q = P_2 P_1:
//     A = X X^T;  P = a I + b A + c A A;  T = P A, A = T P;  D = b A + c A A;  Q = a P + D P;  X = Q X
// (the second iteration's a, b, c from D on).  Of m x m matrices a group takes 5 products instead of 2, of m x n ones one Gram and one
// apply product instead of two of each.  The first iteration is as it is written and in bf16: U is bf16 of any magnitude.  Then come
// groups of two, and at the end a single iteration where the number of iterations is even (gram_group).
// Everything between the first iteration and O is held in f16, scaled by a power of two: as wide as bf16, at the same rate, with 8 times its
// precision, which the route needs.  The identity that Q carries is what limits it: directions outside the range of X put
// a^2 = 12 on Q's diagonal where the directions that matter need values near 1.  Error of O against 64 bits (model of the arithmetic, N =
// 5, 384 x 3072; all of Eq. 2 in bf16 / groups of two and three from the first iteration on / these): Gaussian 1.4, 0.39, 0.38e-2; U
// zero outside 1 column 1.9, 6.2, 0.80e-2, 16 columns 1.2, 4.8, 0.66e-2, 96 columns 1.2, 4.1, 0.66e-2; singular values that fall like 1 / i
// 3.0, 2.5, 2.4e-2; equal columns 1.9, 6.6, 0.85e-2.  Groups of two from the first iteration on (its Q in bf16) 1.9e-2 with two columns, where
// Eq. 2 has 1.4.
// f16 holds 65504: coefficients under which a bound on some matrix could pass that (gram_coefficients_fit) take Eq. 2's products.
enum GramOp : int {
  kGramT = 0,      // T = Bp Ag -> U                    (U: an m x m matrix in the other buffer of the iterate)
  kGramA,          // A = U Bp -> Ag
  kGramD,          // D from Ag -> U
  kGramQ,          // Q = a Bp + U Bp -> Ag
  kGramParityOps   // each of the above for the two places of U
};
constexpr int kGramApply = 2 * kGramParityOps;       // X = Ag X: [parity * 2 + last]
constexpr int kGramOps = kGramApply + 4;
constexpr int kGramMinSteps = 4;                     // fewer iterations have nothing to gain
// Iterations of the group that starts with iteration `it` of n, and the number of groups.
inline int gram_group(int it, int n) { return it > 0 && n - it >= 2 ? 2 : 1; }
inline int gram_groups(int n) { return n / 2 + 1; }
// Powers of two by which the f16 matrices are larger than what they stand for: A and T; P, D and Q; X.
constexpr float kGramScaleA = 8192.f, kGramScaleP = 512.f, kGramScaleX = 8192.f;
bool gram_route(const MatPlan& q, int ns_dtype);
// Whether `steps` iterations with the coefficients coeff[3 * k] .. (a, b, c) stay inside f16 on the Gram route.  *gain: a bound on how much
// larger X gets, for store_norm.
bool gram_coefficients_fit(const double* coeff, int steps, double* gain);

// What a group contributes to a paired launch: nothing, its Gram product, another symmetric product, its apply product.
enum PairProduct : int { kPairNone = 0, kPairGram = 1, kPairSym = 2, kPairApply = 3 };
struct PairForm {
  bool persistent = false;                        // coarse launch
  bool quarters = false;                          // fine launch, as in TileSet
  int few = 0;
};

// Launch group: the matrices of one chunk that take one route.  Each product is one launch per level: the coarse launch (matrix-core
// paths only) runs 256 x 256 tiles over the part of every output that whole such tiles cover plus 512 x 128 tiles
// over the 128-wide column strip an odd multiple of 128 leaves; the fine launch (128 x 128 bf16, 64 x 64 fp32) takes
// what remains, so that nothing is padded beyond the fine tile.  (With several planes entries of the coarse tables run as four
// 128 x 128 blocks.)  A product whose coarse launch would leave much of the
// chip idle has no coarse launch: all its tiles are fine.
struct Group {
  int n_prob = 0;
  bool gram = false;                              // its matrices take the Gram route
  int64_t longest_n = 0, longest_m = 0;           // longest K of the Gram product, of the other two
  size_t prob_ops = 0;                            // Gram route: kGramOps tables of n_prob problems, one after the other
  std::vector<int> members;                       // problem index -> matrix index in the caller's list
  size_t prob_gram[2] = {0, 0}, prob_poly = 0, prob_apply[4] = {0, 0, 0, 0};  // byte offsets ([parity], [parity * 2 + last])
  TileSet fine, coarse;
  // Gram route: symmetric products that run without the other group's, where their own coarse tiles would be few or fill their rounds
  // badly: all tiles in a fine launch (n_lone = 0: no such table), alone or with the other group's apply product in fine tiles.
  size_t lone = 0;
  int n_lone = 0;
  PairForm lone_form[2];
};

struct Chunk {
  int first = 0, count = 0;
  size_t ew_tiles_off = 0;   // byte offset of the EwTile table
  int n_ew_tiles = 0;
  bool stream_w = true;      // no long list of bf16 weights whose rows end inside 128-byte lines
  bool fold_norm = false;    // the blocks of the first Gram launch add up the partial sums of squares themselves
  std::vector<Group> groups; // one, or the matrices iterated as Eq. 2 is written and then those of the Gram route
  // With a group of the Gram route: forms of the launches that pair a product of groups[0] with one of groups[1].
  // pair[i][j]: kPair* of the first and of the second group (kPairNone: nothing is left to do there, or there is no second group).
  bool paired = false;
  PairForm pair[4][4];
  // [group][kPair*]: the product can share a launch with the other group's apply product in coarse tiles, from its fine or its lone table
  bool beside[2][4] = {};
  // Where both groups have coarse symmetric tiles: one table of both for every pair of symmetric products, dealt as one.
  // [first group's Gram product / another][second group's Gram product / another]
  size_t shared_sym[2][2] = {};
  int n_shared_sym = 0;
  // Apply products of both groups in one launch of coarse tiles, where they read the same type: n_shared_app entries (0: no such table).  A
  // group without coarse apply tiles of its own has all of its product in here, the other its fine tiles in a launch of theirs.
  size_t shared_app = 0;
  int n_shared_app = 0;
  bool shared_app_strips = false, shared_app_steady = false;
};

struct Plan {
  int n = 0;
  int ns_dtype = MUON_BF16;
  std::vector<MatPlan> mats;
  std::vector<Chunk> chunks;
  std::vector<unsigned char> image;   // host image of the table region (what muon_init uploads)
  size_t off_mats = 0, off_ptrs = 0;  // byte offsets of the matrix records and of the per-step pointer table
  int coarse_blocks = 256;            // blocks of a persistent coarse launch (compute units of the device); set before plan_build
};

constexpr int kCoarse = 256;          // block tile of the large bf16 kernel
constexpr int64_t kMaxDim = 1 << 20;  // tile offsets are 16-bit in units of 64 elements

bool on_matrix_cores(int ns_dtype);
int planes_of(int ns_dtype);
bool folds_identity(const MatPlan& q, int ns_dtype);

// MUON_OK or the status muon_init would return for this list.
int validate_shapes(const muon_param* p, int32_t n, int32_t ns_dtype);

// Bytes to allocate for a list (see muon_workspace_bytes).  May throw std::bad_alloc.
int plan_workspace_bytes(const muon_param* shapes, int32_t n, int32_t ns_dtype, size_t max_bytes, size_t* out);

// Builds the plan for a workspace at address `ws_base` of `ws_bytes` bytes.  Returns MUON_OK,
// MUON_E_WORKSPACE_TOO_SMALL or a validation status.  May throw std::bad_alloc.
int plan_build(Plan& out, const muon_param* shapes, int32_t n, int32_t ns_dtype, uintptr_t ws_base, size_t ws_bytes);

// Tile table of one grouped launch as records {matrix, first row, first column, rows, columns (in elements),
// computed 32 x 32 blocks}
// (see muon_plan_tiles).  Returns the number of records of the table.
int64_t plan_tiles(const Plan& plan, int chunk, int product, int level, int32_t* out, int32_t cap_records);

}  // namespace muon
