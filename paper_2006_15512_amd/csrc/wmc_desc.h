// Device-visible plan descriptors, written by the host planner and read by
// the HIP kernels.  Plain C structs, identical layout on host and device.
#pragma once
#include <stdint.h>

#define WMC_MAX_RUNS 20       // runs of a bit-extraction (pext) map
#define WMC_LEAF_VARS 24      // distinct variables of a clause leaf
#define WMC_WAVE 64

// Per-tensor bookkeeping in device memory.  The stored entries t of a tensor
// represent t * 2^exp; maxbits holds the IEEE bits of max |t| (non-negative
// doubles order like their bit patterns, so an integer atomicMax works).
struct wmc_meta {
    unsigned long long maxbits;
    long long exp;
};

// Running slice sum (s + c) * 2^e with Neumaier compensation c, plus the
// last slice's value (mantissa, exponent) for per-slice inspection.
struct wmc_acc {
    double s;
    double c;
    long long e;
    long long n_added;
    double last_m;
    long long last_e;
    long long pad[2];
};

// Leaf tensors: a clause indicator table B_C (restricted to the current
// slice) or the weight vector [W(x,0), W(x,1)] of a variable.
enum { WMC_LEAF_CLAUSE = 0, WMC_LEAF_WEIGHT = 1, WMC_LEAF_WEIGHT_CLOSED = 2 };

struct LeafDesc {
    long long out;        // element offset of the table in the arena
    long long work_begin; // first work item (entries padded to a wave multiple)
    int tensor;           // meta index
    int kind;             // WMC_LEAF_*
    int rank;             // storage rank after slicing
    int k;                // clause: distinct variables
    int var;              // weight leaves: variable index (0-based)
    unsigned falsify;     // clause: the one falsifying assignment over its variables
    int taut;             // clause holds x and not-x: all ones
    int pad;
    // clause variable i (weight leaf: slot 0): storage bit >= 0, or
    // -(1 + b) when the variable is sliced and takes bit b of the slice id
    short pos[WMC_LEAF_VARS];
};

// One pairwise contraction C[beta,mu,nu] = sum_kappa A[beta,mu,kappa] B[beta,kappa,nu].
// Every operand's storage layout is [kappa bits | its C-variables in C's
// storage order], so for an output address r:
//   addr_A(r, j) = (pext(r, maskA) << nk) | j,   j over the 2^nk kappa values,
// where pext is given as runs packed in one word each:
//   src bit in r | length << 8 | dst bit << 16.
#define WMC_RUN(src, len, dst) ((unsigned)(src) | ((unsigned)(len) << 8) | ((unsigned)(dst) << 16))
struct NodeDesc {
    long long a, b, c;        // element offsets in the arena
    long long work_begin;     // first work item of this node in its launch
    int ta, tb, tc;           // meta indices
    int rc;                   // storage rank of C
    int nk;                   // |kappa| (after slicing)
    int nra, nrb;             // number of runs in ra / rb
    int cls;                  // node class
    unsigned ra[WMC_MAX_RUNS];
    unsigned rb[WMC_MAX_RUNS];
};

// A contraction run as a batched matrix product on MFMA:
//   C[beta, mu, nu] = sum_kappa A[beta, mu, kappa] * B[beta, kappa, nu]
// with rows (beta, mu) of the larger operand A and columns (beta, nu) of B.
// Logical indices list their variables in C's storage order; each deposit
// run list maps a logical index onto storage bits (src bit, length, dst bit):
//   row of A = dep(mu, 0) | dep(beta, 1)   -> A + (row << nk) + kappa
//   col of B = dep(nu, 2) | dep(beta, 3)   -> B + (col << nk) + kappa
//   address in C = dep(mu, 4) | dep(nu, 5) | dep(beta, 6)
#define WMC_GEMM_RUNS 12
enum { GR_MU_A = 0, GR_BETA_A, GR_NU_B, GR_BETA_B, GR_MU_C, GR_NU_C, GR_BETA_C, GR_N };

struct GemmDesc {
    long long a, b, c;
    int ta, tb, tc;
    int nk, nm, nn, nb;
    int nrun[GR_N];
    unsigned char run[GR_N][WMC_GEMM_RUNS][3];
    int pad;
};

// A chain: consecutive contractions F_i = F_{i-1} * G_i (i = 1 .. L) run by one
// launch.  F_0, the G_i and F_L are in the arena; F_1 .. F_{L-1} only exist
// as tiles in LDS.  A tile holds every combination of the inner variables
// (all variables summed after stage 1, and the lowest of F_L's order); the
// other variables of F_L number the tiles.  In a short chain the parts of the
// G_i and of F_0 that a tile reads are copied to LDS first.  Every
// address is a bit deposit of the tile index and of the entry index within
// the tile, so a chain is a list of 32-bit words: the header, the stages, the
// offsets of each tile index bit (CH_TILE_BITS words each) in F_0, C and every
// G_i, and the lists that copies refer to.
#define WMC_CHAIN_MAX 15        // stages
#define WMC_CHAIN_NK 3          // summed variables of a stage
#define WMC_CHAIN_BITS 13       // entry bits of a tile
#define WMC_CHAIN_LANE 9        // log2 of a workgroup's threads: short chains of one call,
#define WMC_CHAIN_LANE_MANY 8   // of many calls together,
#define WMC_CHAIN_LANE_BIG 8    // and chains of many tiles
// LDS bytes of a chain, its words included.  Short chains: four workgroups
// of 8 waves fill a compute unit's 32 wave slots, so its 160 KB are shared by
// four (512-instance batch FP64: 6.2 ms at 56 KB, 4.2 at 38, and 4.1 at 19
// with its shorter chains against 3.7 once 38 KB chains had a launch of their
// own); many tiles: three workgroups of 4 waves at 110 registers (min-fill
// lattice FP64: 54.6 ms at 30 KB, 48.7 at 38, 42.8 at 50, 42.9 at 72).
#define WMC_CHAIN_LDS_SHORT (38 * 1024)
#define WMC_CHAIN_LDS (50 * 1024)
// Where many short chains share a launch (batches, serving), those above this
// have a launch of their own: every workgroup of a launch reserves the most
// any of them needs, and eight of 256 threads fill a compute unit's wave
// slots at 19 KB each (512-instance batch FP64: 4.2 ms in one launch, 3.7 in
// two).
#define WMC_CHAIN_LDS_NARROW (19 * 1024)
#define WMC_CHAIN_TILE_BITS 11  // largest tile index of a short chain
// log2 of the bound of a chain's stored magnitudes.  Every operand entry is
// below 1 as it is read, so F_i stays below 2^(lift + summed variables up to
// stage i): the lift is this bound less all of the chain's summed variables.
// FP32: below the largest finite number.  FP64, and FP32 where a matrix node
// (K >= 16) reads the output: those multiply the operands as stored, in that
// type, so the product of two such tensors, summed, stays finite, too.
#define WMC_CHAIN_TOP_FP32 126
#define WMC_CHAIN_TOP_FP32_MATRIX 56
#define WMC_CHAIN_TOP_FP64 480
// A copied operand: log2 of its entries per tile, the lowest of them whose
// offset is the entry index itself, its first LDS entry, and the word where
// the offsets of the other index bits are listed.
enum { CX_BITS = 0, CX_LOW, CX_LDS, CX_LIST, CX_WORDS };
enum {
    CH_STAGES = 0, CH_TILE_BITS, CH_F, CH_F_HI, CH_C, CH_C_HI, CH_TF, CH_TC,
    CH_MASK,                    // meta entry that collects the stages' range bits
    CH_NT,                      // C is stored non-temporally
    CH_FCOPY,                   // F_0 is copied to LDS
    CH_TILES,                   // word where the tile index bits are listed
    CH_X,
    CH_OUT = CH_X + CX_WORDS,   // short chains: last outputs' offsets of the entry bits
    CH_SRC = CH_OUT + 16,       // and F_0's, where it is not copied
    CH_WORDS = CH_SRC + 16
};
// A stage: in a short chain, the offsets of the tile's entry bits in the
// source (low half of a word) and in G's copy (high half), then the copy; the
// entry index is the index of an output in LDS.  In a chain of many tiles the
// offsets have a word each, some bits are taken inside the thread (up to two
// that only the source has, with their source and output offsets, and up to
// two that only G has, with their G and output offsets), and the output
// offsets of the others are listed too.  Sources, copies and outputs are LDS
// entries except F_0 where it is not copied and the last output.
enum {
    CS_SHAPE = 0,               // nk | source-only register bits << 8 | G-only ones << 16
    CS_TBITS, CS_G, CS_G_HI, CS_TG, CS_SRC, CS_DST,
    CS_LIFT,                    // first stage: log2 of the factor F_1 .. F_L are stored larger by
    CS_BIT_SG,                  // short
    CS_X = CS_BIT_SG + 16,
    CS_WORDS = CS_X + CX_WORDS,
    CS_BIT_S = CS_BIT_SG,       // many tiles
    CS_BIT_G = CS_BIT_S + 16, CS_BIT_O = CS_BIT_G + 16,
    CS_PS = CS_BIT_O + 16, CS_PO = CS_PS + 2, CS_QG = CS_PO + 2, CS_QO = CS_QG + 2,
    CS_WORDS_BIG = CS_QO + 2
};
static_assert(CH_WORDS % 4 == 0 && CS_WORDS % 4 == 0 && CS_WORDS_BIG % 4 == 0 && WMC_CHAIN_BITS <= 16,
              "words are read four at a time");
// One workgroup of a chain launch: tiles [blk << jbits, (blk + 1) << jbits)
// of the chain at word `desc`, which has `words` words.
struct ChainRec {
    unsigned desc, blk, jbits, words;
};

static_assert(sizeof(LeafDesc) == 96, "LeafDesc layout");
static_assert(sizeof(GemmDesc) == 336, "GemmDesc layout");
static_assert(sizeof(NodeDesc) == 224, "NodeDesc layout");
