// bf16 MFMA GEMMs of the quantized linear layer (gfx950; fwd and dX on v_mfma_f32_32x32x16_bf16, dW on
// v_mfma_f32_16x16x32_bf16).
//
//   fwd :  Y [T,O]  = X [T,I]  * What[O,I]^T        (K = I)
//   dX  :  dX[T,I]  = dY[T,O]  * What[O,I]          (K = O)
//   dW  :  dWhat^T[I,O] = X[T,I]^T * dY[T,O]        (K = T), fused with the Eq.(3)-(5) epilogue
//
// What is never in HBM: the weight operand of fwd / dX is rebuilt per tile, in registers, from N-bit codes
// (working layout, see WorkCodes) and the (s, zbar) pair of each group, and written to LDS as bf16.
#include "common.h"
#include "gemm_bwd.h"
#include "kernels.h"
#include "prof.h"
#include "tile_gemm.h"

#include <algorithm>

namespace eqat {

template <int BITS, bool BT, int MODE, int BM, int BN, int BK, int WGM, int WGN>
__global__ __launch_bounds__(64 * WGM * WGN) void k_gemm_q(const GemmQArgs a)
{
    gemm_q_body<BITS, BT, MODE, BM, BN, BK, WGM, WGN>(a, (int)blockIdx.x, (int)gridDim.x);
}
template <int BITS, typename WT, bool BLOCK_AP, int BM, int BN, int BK, int NS, int WGM, int WGN, bool CUT>
__global__ __launch_bounds__(64 * WGM * WGN) void k_gemm_dw(const GemmDwArgs a)
{
    gemm_dw_body<BITS, WT, BLOCK_AP, BM, BN, BK, NS, WGM, WGN, CUT>(a, (int)blockIdx.x, (int)gridDim.x);
}

// ======================================================================================================
// host side
// ======================================================================================================
namespace {

// dW: a round of big tiles (one per compute unit) takes 12 us and 1.35 a K tile of 64 tokens, a round of small ones (two per compute
// unit, a quarter of the work each) 7 us and 0.88, and a small number of tiles beyond whole rounds costs most of a round unless
// the contraction is long (they are split then).  So the small tiles are taken where they fill one round, and, up to 2048 tokens,
// where the big ones leave at most a quarter of a second round while the small ones need two and a half at most; the big
// ones where the small ones would go into a second round (130 to 159 big tiles): up to 9 K tiles that is a draw, and with
// few more than 512 and a long contraction the split ones are level or ahead.  Measured, us, dW ds dz of Block-AP, g = 64, big / small:
// 2560 x 6912 (270 big tiles): 515 tokens 59 / 46, 1000 72 / 60, 2048 105 / 98; 4096 x 5120 (320): 1000 75 / 64, 2048 119 / 106, 4096 171 / 174;
// 5120 x 5120 (400): 1000 79 / 83; 3072 x 3072 (144): 300 26.4 / 25.8, 1000 37 / 39, 2048 51 / 66, 8192 143 / 163; 2560 x 3328 (130):
// 1536 tokens 15 % faster big, 8192 6 % slower.
bool use_small_dw_tile(int64_t m, int64_t n, int64_t tokens)
{
    const int64_t big = ((m + 255) / 256) * ((n + 255) / 256), small = ((m + 127) / 128) * ((n + 127) / 128);
    if (big >= 160) return big > 256 && big <= 320 && tokens <= 2048;
    return small <= 512 || tokens <= 576 || (small < 544 && tokens > 2048);
}

// Workgroups that a device of `cus` compute units runs at the same time (LDS is what limits these kernels), rounded down to a
// multiple of 8.
constexpr int kMaxCus = 256;            // compute units of an MI355X; the workspace is sized for this many
constexpr int kSkCounterWords = 2 * 2 * 2 * kMaxCus;  // 2 G arrival counters and 2 G flags, G <= 2 workgroups per compute unit
constexpr int per_cu(size_t smem) { return smem * 2 <= 160 * 1024 ? 2 : 1; }
int resident_workgroups(int cus, int per_cu) { return (cus * per_cu) & ~7; }
int current_cus()
{
    static int cus_of[64] = {0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev > 63) dev = 0;
    if (cus_of[dev] == 0) {
        int n = 0;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 8) n = kMaxCus;
        cus_of[dev] = n < kMaxCus ? n : kMaxCus;
    }
    return cus_of[dev];
}
// What a plan that cuts tiles of `tile` outputs may write: one part per resident workgroup if it splits tiles, two if it deals out
// runs.  The workspace is sized for the plans of kMaxCus compute units; with fewer of them another plan may cut where those do
// not, so every plan asks for the room it needs.
size_t parts_bytes(int resident, int tile, bool split) { return (size_t)resident * (split ? 1 : 2) * (size_t)tile * sizeof(float); }
bool parts_fit(const SkScratch &s, int resident, int tile, bool split)
{
    return s.partials != nullptr && s.counters != nullptr && s.bytes >= parts_bytes(resident, tile, split);
}

// fwd / dX with more tiles than k_gemm_ksplit takes: big tiles where they fill most of the chip, or where the small ones do not
// fit two per compute unit (dX of 5120 x 5120, 1792 tokens: 140 big tiles 99 us, 560 small ones 133; 2048 -> 5504: 154 big tiles 46,
// small 60), or, each shared by two or three workgroups, where the contraction is long enough to pay for the parts: small tiles
// take 0.9 us per K tile, a share of a big one 1.55 (the chip's power limit), 0.085 us per part comes on top (dX, 11008 -> 4096:
// 1280 tokens 157 -> 111 us, 2048 tokens 184 -> 164; 4096 -> 4096, 1280 tokens: 67 -> 64, 2048 tokens: 74, 80 if it were taken).
// The few small tiles beyond 512 are split eight ways where K is long, and a forward that reads few (s, z) pairs is faster on them
// than on 130 to 159 big tiles: 2-bit codes with at most 8 groups a row, each 16 K tiles or more, and from 48 K tiles on
// (513 to 544 tiles, 99 random sizes, from level to 12 % faster; us, small / big: one group per row, 532 tiles, 9792 inputs 176 / 195, 528 tiles,
// 4384 inputs 90 / 95; g = 1024, 516 tiles, 4096 inputs 81 / 85).  Shorter ones are level or slower (536 tiles, 2688 inputs 60 / 59), and so
// are g = 512 from 530 tiles on and 3-bit codes (one group, 540 tiles, 7968 inputs 159 / 156, 525 tiles, 15168 inputs 277 / 288).
enum class TileChoice { Small, Big, BigShared };
TileChoice q_tile(const Problem &p, bool bt, int cus, const SkScratch &scratch)
{
    const int64_t m = p.T, n = bt ? p.I : p.O, k = bt ? p.O : p.I;
    const int64_t big = ((m + 255) / 256) * ((n + 255) / 256), small = ((m + 127) / 128) * ((n + 127) / 128);
    if (!bt && big < 160 && small > 512 && small <= 544 && parts_fit(scratch, resident_workgroups(cus, 2), TileSmall::BM * TileSmall::BN, true)
        && p.bits == 2 && p.G <= 8 && p.g >= 1024 && k >= 48 * 64) return TileChoice::Small;
    if (big >= 160 || small > 512) return TileChoice::Big;
    const int64_t c = resident_workgroups(cus, 1) / 8 / ((big + 7) / 8), k_tiles = (k + 63) / 64;   // contributors per tile, as plan_tiles deals them out
    if (!parts_fit(scratch, resident_workgroups(cus, 1), TileBig::BM * TileBig::BN, true) || c < 2 || c > 3 || k_tiles < 32) return TileChoice::Small;
    return 5.0 + 1.55 * (double)((k_tiles + c - 1) / c) + 0.085 * (double)(big * c) < 4.0 + 0.9 * (double)k_tiles ? TileChoice::BigShared : TileChoice::Small;
}

// The kernels need more dynamic LDS than the default limit; the attribute is per kernel AND per device, so it is set
// once for every (instantiation, device) pair.  `done` is the caller's static mask of devices already served.
template <typename K> void allow_dynamic_lds(K kern, size_t smem, uint64_t &done)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev > 63) dev = 0;
    if ((done >> dev) & 1u) return;
    (void)hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    done |= (uint64_t)1 << dev;
}

// Tiles beyond whole rounds are split from this many pairs of K tiles on: two for every contributor there may be.
bool long_enough_to_split(int pairs) { return pairs >= 2 * kSkMaxSplit; }

// How `resident` workgroups share `ntiles` tiles of `tile` outputs and `pairs` K-tile pairs each (see SkPlan).  One workgroup per tile
// when they all fit; otherwise whole tiles, except that (K long enough)
//   - between one and two rounds of tiles, with more than half a round beyond the first, every tile is cut along K into
//     equal runs (with more rounds, cutting the last 1.x of them into runs measured slower than leaving the last round
//     partly filled: 7B gate, 5.4 rounds: -3 %; 13B gate, 3.4 rounds: -4 %);
//   - with at most half a round of tiles beyond the whole rounds, those few tiles are split among groups of workgroups.
SkPlan plan_tiles(int ntiles, int tile, int pairs, int resident, const SkScratch &scratch, bool runs = true, bool share = false)
{
    SkPlan sk{};
    sk.pairs = pairs; sk.slots = 2; sk.partials = scratch.partials; sk.counters = scratch.counters;
    const bool room = parts_fit(scratch, resident, tile, true), room_for_runs = parts_fit(scratch, resident, tile, false);
    if (ntiles <= resident) {                                // walk = 0: one workgroup per tile, unless they are to share
        if (share && room && 2 * ((ntiles + 7) / 8) <= resident / 8) { sk.walk = 1; sk.split = 1; sk.slots = 1; }
        return sk;
    }
    sk.walk = 1;
    const int W = resident / 8, per = ntiles / 8, full = per / W;
    const bool even = (per % W == 0) && (ntiles % 8 == 0);
    const bool may_cut = !even && pairs >= 4 && room;
    sk.dp_rounds = (may_cut && room_for_runs && runs && full == 1) ? 0 : (per + (ntiles % 8 ? 1 : 0) + W - 1) / W;
    // Few tiles beyond the whole rounds (at most half a round on every XCD): whole tiles first, then the rest split.
    // The tile arithmetic promises (1 - 1/c) of a round; measured, 5.4 rounds (7B gate, up) gain 2.6 %, 3.4 rounds (13B
    // gate) 1.5-2.3 %: the partly filled round that the split replaces ran at a higher clock, and the instantiation that
    // can cut is 1-5 % slower in its main loop.  Beyond six whole rounds the promise is smaller than that price.
    const int n_sk_max = per + (ntiles % 8 ? 1 : 0) - full * W;
    if (may_cut && full <= 6 && n_sk_max >= 1 && 2 * n_sk_max <= W && long_enough_to_split(pairs)) { sk.dp_rounds = full; sk.split = 1; sk.slots = 1; }
    return sk;
}

// Geometry of a fwd / dX launch: tiles, the XCD band, who computes what (SkPlan), the grid, and which instantiation runs.  A contraction of no whole
// K-tile pairs has one of its own: in that for cut tiles, which could serve it, two workgroups of small tiles do not fit a compute unit's registers
// (175 to 185 each) and big tiles spill: dX, 4104 -> 8960, 685 tokens 107 us there, 73 here, 4104 -> 11008, 515 tokens 104 and 71; forward 1 to 2.5 %.
struct QLaunchPlan { int tiles_m, tiles_n, band, ntiles, grid; SkPlan sk; QMode mode; };
int q_band(int tiles_m) { return std::max(2, std::min(8, tiles_m / 8)); }
template <bool BT, typename TS>
QLaunchPlan plan_q(int M, int N, int K, int cus, const SkScratch &scratch, bool share)
{
    QLaunchPlan q{};
    q.tiles_m = (M + TS::BM - 1) / TS::BM;
    q.tiles_n = (N + TS::BN - 1) / TS::BN;
    // Tile rows that one XCD walks together.  The activation panel of a tile row is eight times heavier than the code
    // panel of a tile column, so the 32 tiles an XCD holds at a time should span few rows and many columns (per K step
    // it fetches rows x 32 KB + columns x 6 KB: 4 rows x 8 columns 176 KB, 8 x 4 280 KB), and with an eighth of the tile
    // rows per band every XCD owns its rows outright, so that an activation panel is fetched by one XCD only.  Measured:
    // 4 (8192 tokens) and 2 (4096 tokens) are up to 2-4 % ahead of 8; 16 is 3 % behind.
    q.band = q_band(q.tiles_m);
    // At most as many workgroups as the chip holds at once; with more tiles than that every workgroup walks several
    // (grid a multiple of 8, one share per XCD).
    q.ntiles = q.tiles_m * q.tiles_n;
    const int resident = resident_workgroups(cus, per_cu(q_smem_bytes<BT, TS>()));
    q.sk = plan_tiles(q.ntiles, TS::BM * TS::BN, ((K + TS::BK - 1) / TS::BK + 1) / 2, resident, scratch, true, share);
    q.grid = q.sk.walk ? resident : q.ntiles;
    q.mode = q.sk.walk && (q.sk.dp_rounds == 0 || q.sk.split) ? kCut : K % (2 * TS::BK) != 0 ? kRagged : kWhole;
    return q;
}

template <int BITS, bool BT, typename TS>
void launch_q(const GemmQArgs &args, const SkScratch &scratch, hipStream_t st, bool share = false)
{
    constexpr size_t smem = q_smem_bytes<BT, TS>();
    static_assert(smem + 64 <= 160 * 1024, "LDS of one CU");
    GemmQArgs a = args;
    a.c_bytes = (uint32_t)((size_t)a.M * a.N * 2);
    const QLaunchPlan q = plan_q<BT, TS>(a.M, a.N, a.K, current_cus(), scratch, share);
    a.tiles_m = q.tiles_m; a.tiles_n = q.tiles_n; a.band = q.band; a.sk = q.sk;
    const dim3 grid(q.grid), block(64 * TS::WGM * TS::WGN);
    auto go = [&](auto kern, uint64_t &attr_done) {
        allow_dynamic_lds(kern, smem, attr_done);
        kern<<<grid, block, smem, st>>>(a);
    };
    static uint64_t done_cut = 0, done_ragged = 0, done_whole = 0;
    if (q.mode == kCut) go(k_gemm_q<BITS, BT, kCut, TS::BM, TS::BN, TS::BK, TS::WGM, TS::WGN>, done_cut);
    else if (q.mode == kRagged) go(k_gemm_q<BITS, BT, kRagged, TS::BM, TS::BN, TS::BK, TS::WGM, TS::WGN>, done_ragged);
    else go(k_gemm_q<BITS, BT, kWhole, TS::BM, TS::BN, TS::BK, TS::WGM, TS::WGN>, done_whole);
}

template <bool BT>
void launch_q_bits(const Problem &p, const GemmQArgs &a, const SkScratch &scratch, hipStream_t st)
{
    const TileChoice tile = q_tile(p, BT, current_cus(), scratch);
#define EQAT_GO(B) do { if (tile == TileChoice::Small) launch_q<B, BT, TileSmall>(a, scratch, st); else launch_q<B, BT, TileBig>(a, scratch, st, tile == TileChoice::BigShared); } while (0)
    if (p.bits == 2) EQAT_GO(2); else if (p.bits == 3) EQAT_GO(3); else EQAT_GO(4);
#undef EQAT_GO
}

// Geometry of a dW launch: tiles (rows: in-features, columns: out-features), and whether tiles are cut along T (then the
// grid is what the chip holds at once and sk says who computes what), or every tile has a workgroup of its own.
struct DwLaunchPlan { int tiles_m, tiles_n, ntiles, grid; SkPlan sk; bool cut; };
template <typename WT, bool AP, typename TS>
DwLaunchPlan plan_dw(int I, int O, int T, int cus, const SkScratch &scratch)
{
    DwLaunchPlan d{};
    d.tiles_m = (I + TS::BM - 1) / TS::BM;
    d.tiles_n = (O + TS::BN - 1) / TS::BN;
    d.ntiles = d.tiles_m * d.tiles_n;
    const int resident = resident_workgroups(cus, per_cu(dw_smem_bytes<WT, AP, TS::BM, TS::BN, TS::BK, TS::NS, TS::WGM, TS::WGN>()));
    d.sk = plan_tiles(d.ntiles, TS::BM * TS::BN, ((T + TS::BK - 1) / TS::BK + 1) / 2, resident, scratch, false);
    d.cut = d.sk.walk && (d.sk.dp_rounds == 0 || d.sk.split);
    if (!d.cut) d.sk = SkPlan{};
    d.grid = d.cut ? resident : d.ntiles;
    return d;
}

template <int BITS, typename WT, bool AP, typename TS>
void launch_dw_t(const GemmDwArgs &args, const SkScratch &scratch, hipStream_t st)
{
    constexpr size_t smem = dw_smem_bytes<WT, AP, TS::BM, TS::BN, TS::BK, TS::NS, TS::WGM, TS::WGN>();
    static_assert(smem + 64 <= 160 * 1024, "LDS of one CU");
    static_assert(per_cu(smem) == (TS::BM == TileSmall::BM ? 2 : 1), "plan_dw_of takes one pair of types for all");
    GemmDwArgs a = args;
    const DwLaunchPlan d = plan_dw<WT, AP, TS>(a.I, a.O, a.T, current_cus(), scratch);
    a.tiles_m = d.tiles_m;
    a.tiles_n = d.tiles_n;
    a.direct = (TS::BM % a.g == 0) ? 1 : 0;
    a.sk = d.sk;
    const dim3 grid(d.grid), block(64 * TS::WGM * TS::WGN);
    if (d.cut) {
        auto kern = k_gemm_dw<BITS, WT, AP, TS::BM, TS::BN, TS::BK, TS::NS, TS::WGM, TS::WGN, true>;
        static uint64_t attr_done = 0;
        allow_dynamic_lds(kern, smem, attr_done);
        kern<<<grid, block, smem, st>>>(a);
    } else {
        auto kern = k_gemm_dw<BITS, WT, AP, TS::BM, TS::BN, TS::BK, TS::NS, TS::WGM, TS::WGN, false>;
        static uint64_t attr_done = 0;
        allow_dynamic_lds(kern, smem, attr_done);
        kern<<<grid, block, smem, st>>>(a);
    }
}

template <typename WT, bool AP>
bool launch_dw_bits(int bits, const GemmDwArgs &a, const SkScratch &sk, hipStream_t st)   // returns whether per-segment partials were written
{
    const bool small = use_small_dw_tile(a.I, a.O, a.T);
#define EQAT_GO(B) do { if (small) launch_dw_t<B, WT, AP, DwTileSmall>(a, sk, st); else launch_dw_t<B, WT, AP, DwTileBig>(a, sk, st); } while (0)
    if (bits == 2) EQAT_GO(2); else if (bits == 3) EQAT_GO(3); else EQAT_GO(4);
#undef EQAT_GO
    return ((small ? TileSmall::BM : TileBig::BM) % a.g) != 0;
}

}  // namespace

// workspace reservation: either tile shape may be picked at launch
bool dw_needs_partials(const Problem &p) { return (TileSmall::BM % p.g) != 0; }

namespace {

// as much as any plan asks for; nothing is read or written through it
const SkScratch kAnyRoom{reinterpret_cast<float *>(16), ~(size_t)0, reinterpret_cast<uint32_t *>(16)};

QLaunchPlan plan_q_of(const Problem &p, bool bt, int cus, const SkScratch &sk, TileChoice *choice)
{
    const int M = (int)p.T, N = (int)(bt ? p.I : p.O), K = (int)(bt ? p.O : p.I);
    *choice = q_tile(p, bt, cus, sk);
    const bool small = *choice == TileChoice::Small, share = *choice == TileChoice::BigShared;
    if (bt) return small ? plan_q<true, TileSmall>(M, N, K, cus, sk, false) : plan_q<true, TileBig>(M, N, K, cus, sk, share);
    return small ? plan_q<false, TileSmall>(M, N, K, cus, sk, false) : plan_q<false, TileBig>(M, N, K, cus, sk, share);
}
// (weight type and phase make no difference to the plan: the LDS of both tiles allows the same workgroups per compute unit)
DwLaunchPlan plan_dw_of(const Problem &p, int cus, const SkScratch &sk, bool *small)
{
    *small = use_small_dw_tile(p.I, p.O, p.T);
    return *small ? plan_dw<bf16_t, true, DwTileSmall>((int)p.I, (int)p.O, (int)p.T, cus, sk)
                  : plan_dw<bf16_t, true, DwTileBig>((int)p.I, (int)p.O, (int)p.T, cus, sk);
}

// ---- what the launches of a backward take, in us, as the two rules below estimate it (fits to single calls, operands cold) ----------
int64_t tiles_of(int64_t m, int64_t n, int edge_m, int edge_n) { return ((m + edge_m - 1) / edge_m) * ((n + edge_n - 1) / edge_n); }
// Rounds that `tiles` one-per-compute-unit workgroups cost (workgroups go round the XCDs): a few beyond whole rounds are
// split where the contraction is long (plan_tiles; the parts of dW's cost more, its instantiation for them is slower); else a partly filled round costs less than
// its share, the clock rises.
double rounds_cost(int64_t tiles, int per_xcd, int k_tiles, bool dx)
{
    const double rounds = (double)((tiles + 7) / 8) / per_xcd, full = (double)(int64_t)rounds, part = rounds - full;
    if (full < 1.0) return 1.0;
    if (part == 0.0) return full;
    if (full <= 6.0 && part <= 0.5 && long_enough_to_split((k_tiles + 1) / 2)) return full + part + (dx ? 0.15 : 0.3);
    if (!dx) return full + std::max(0.8, __builtin_pow(part, 0.25));
    return full == 1.0 && k_tiles >= 8 ? 1.1 + part : full + __builtin_pow(part, 0.35);
}
// dX in a launch of its own; *tokens: token tile of k_gemm_mid_dx where it takes that, else 0
double dx_us(const Problem &p, int cus, const SkScratch &sk, int *tokens)
{
    const int64_t big = tiles_of(p.T, p.I, 256, 256), small = tiles_of(p.T, p.I, 128, 128);
    const int k_tiles = (int)((p.O + 63) / 64);
    double there;
    if (const int parts = ksplit_parts(p, true, sk)) {
        const double pairs = (double)(((p.O + 127) / 128 + parts - 1) / parts), groups = (double)(small * parts);
        there = (parts == 1 ? 5.8 : 6.5 + 0.03 * groups) + pairs * (0.8 + 0.5 * groups / 256.0 * std::min(1.0, pairs / 32.0));
    } else {
        switch (q_tile(p, true, cus, sk)) {
        case TileChoice::Small: there = 4.0 + 0.97 * k_tiles; break;       // operands cold; q_tile and the forward's rule weigh these tiles at 0.9, in fits of their own
        case TileChoice::Big: there = 5.0 + 1.38 * k_tiles * rounds_cost(big, cus / 8, k_tiles, true); break;
        default: {
            const int64_t c = resident_workgroups(cus, 1) / 8 / ((big + 7) / 8);
            there = 5.0 + 1.55 * (double)((k_tiles + c - 1) / c) + 0.085 * (double)(big * c);
        }
        }
    }
    int bm = 0;
    const double here = mid_dx_us(p, cus, &bm);
    *tokens = here < there ? bm : 0;
    return std::min(here, there);
}
// A 256 x 256 tile of dW with its epilogue
double dw_tile_us(const Problem &p, bool block_ap)
{
    const double k_tiles = (double)((p.T + 63) / 64);
    return !block_ap ? 12.0 + 1.37 * k_tiles : p.w_bf16 ? 14.5 + 1.38 * k_tiles : 24.0 + 1.65 * k_tiles;
}
double dw_us(const Problem &p, bool block_ap, int cus)
{
    const int k_tiles = (int)((p.T + 63) / 64);
    if (!use_small_dw_tile(p.I, p.O, p.T)) return rounds_cost(tiles_of(p.I, p.O, 256, 256), cus / 8, k_tiles, false) * dw_tile_us(p, block_ap);
    const int64_t small = tiles_of(p.I, p.O, 128, 128);
    const double extra = !block_ap ? 0.0 : p.w_bf16 ? 2.0 : 5.0;
    return small <= cus ? 6.0 + 0.62 * k_tiles + extra : (7.0 + 0.88 * k_tiles + extra) * rounds_cost(small, cus / 4, k_tiles, false);
}

// A backward that leaves compute units idle altogether, in one launch (every tile of both at once: the longer of them, dW's with the whole epilogue on few
// compute units) and in two (small tiles of dW); `dw_share`: tiles of dW per compute unit.
struct FewTiles { double start, per_share, g32, apart, apart_per_share; };
FewTiles few_tiles(const Problem &p, bool block_ap)
{
    if (!block_ap) return {10.0, 7.0, 1.0, 3.3, 2.3};
    return p.w_bf16 ? FewTiles{15.0, 16.0, 2.5, 5.2, 5.0} : FewTiles{16.5, 20.0, 2.5, 6.0, 8.0};
}
double bwd_one_round_us(const Problem &p, bool block_ap, int dx, double dw_share)
{
    const FewTiles f = few_tiles(p, block_ap);
    const double k_tiles = (double)((p.T + 63) / 64), steps = (double)((p.O + 127) / 128);
    const double dw = f.start + 0.96 * k_tiles + f.per_share * dw_share + (p.g == 32 ? f.g32 : 0.0);
    const double there = dx == kBwdBig ? 6.7 + 1.19 * (double)((p.O + 63) / 64) : dx == 64 ? 5.6 + 0.64 * steps : dx == 96 ? 6.2 + 0.75 * steps : 6.6 + 0.83 * steps;
    return std::max(dw, there) + (DwTileBig::BM % p.g != 0 ? 2.5 : 0.0);
}
double bwd_apart_few_us(const Problem &p, bool block_ap, double dx_alone_us, double dw_share)
{
    const FewTiles f = few_tiles(p, block_ap);
    return f.apart + 0.62 * (double)((p.T + 63) / 64) + 1.25 * dx_alone_us + f.apart_per_share * dw_share + (DwTileSmall::BM % p.g != 0 ? 2.0 : 0.0);
}

// Token tiles of k_gemm_mid_dx where dX alone takes that kernel, else 0: up to two rounds of its workgroups, where it is estimated to be faster
// than k_gemm_ksplit or the tiles of k_gemm_q.  196 random sizes, 50 to 2200 tokens, 768 to 12000 in-features, 768 to 16000 out-features: the rule
// takes no kernel more than 2 % slower than the one it leaves and is within 1 % of the best choice in the mean; 8 % faster in the mean, 25 to 50 %
// where one or two rounds are well filled.  us, that kernel / here: 515 tokens, 3 bit 4096 -> 4096 37.7 / 31.8, 11008 -> 4096 99 / 74; 1000
// tokens, 4 bit 11008 -> 4096 128 / 107, 4096 -> 4096 level.  830 more sizes, 1 to 20000 tokens and down to 64 in- and out-features: 4 % faster in the mean, five 2 to 5 % slower.
int mid_dx_tokens(const Problem &p, int cus, const SkScratch &sk)
{
    int tokens = 0;
    (void)dx_us(p, cus, sk, &tokens);
    return tokens;
}

// dX and dW in one launch (gemm_bwd.h): what computes dX then (kBwdBig ... 128), or -1: two launches.  Each of the two alone leaves compute units idle in its
// last round and starts and ends with the whole chip; together the tiles of dW, which come second, fill what those of dX leave.  The estimate deals
// `n1` tiles of dX and then `n2` of dW out to the compute units of an XCD, and lies between that and an even share.  us, two launches / one
// (147 random sizes, 256 to 8192 tokens: 11 % faster in the mean with this rule, 12 % with the best choice at each): 515 tokens, 3 bit, E2E-QP
// 11008 -> 4096 144 / 122; 1000 tokens, Block-AP, fp32 weights 4096 -> 11008 254 / 234; 4096 tokens, 3 bit, Block-AP 5120 -> 5120 380 / 351 (320 and 400
// tiles: 1.25 and 1.56 rounds), 13824 -> 5120 967 / 905.  Whole rounds of both gain 1 % (8192 tokens, 4096 -> 4096 410 / 407) or lose it (11008 -> 4096
// 1095 / 1101), and a single filled round of each does not care.  Where both together fill one round at most, the one launch takes as long as the longer of the
// two, and dW in big tiles, an epilogue on a quarter of the compute units, is longer than in small ones: estimates of their own (fits to 1420 random sizes,
// 1 to 9000 tokens, 200 to 14000 in-features, 64 to 14000 out-features; with the others in their place 163 calls were 5 to 39 % slower than two launches, now 19
// are, 13 % at most, and all are 8 % faster in the mean, 6 % before, 9 % with the best choice at each): 426 tokens, E2E-QP, 2752 -> 368 20.4 / 24.3 and 278 tokens, Block-AP, 1248 -> 448 22.2 / 25.7 stay apart.
int bwd_together(const Problem &p, bool block_ap, int cus, const SkScratch &sk)
{
    if (p.T < 1) return -1;
    // dW, ds and dz are bitwise the same whether or not dX is asked for: tiles of 256 that dW alone cuts along T are cut alike, as long as dX runs on such
    // tiles, too (from 1921 tokens on, 16 pairs of K tiles, which others are not for); no common launch where it cuts tiles of 128 or deals out runs
    bool small_dw;
    const DwLaunchPlan dw = plan_dw_of(p, cus, sk, &small_dw);
    const bool cut = dw.cut;
    if (cut && (small_dw || !dw.sk.split)) return -1;
    int alone = 0, best = -1;
    const double alone_us = dx_us(p, cus, sk, &alone), apart = 3.0 + alone_us + dw_us(p, block_ap, cus), t2 = dw_tile_us(p, block_ap);
    const int64_t n2 = (tiles_of(p.I, p.O, 256, 256) + 7) / 8, small = tiles_of(p.I, p.O, 128, 128);
    const int64_t per_xcd = cus / 8;
    double least = 1.0;                               // of the estimates with a margin, as shares of that of two launches
    for (const int dx : {64, 96, 128, (int)kBwdBig}) {
        int64_t n1 = dx == kBwdBig ? tiles_of(p.T, p.I, 256, 256) : tiles_of(p.T, p.I, dx, 128);
        if (dx != kBwdBig && (cut || n1 * 256 > 700 * (int64_t)cus)) continue;
        n1 = (n1 + 7) / 8;
        double est;
        if (small_dw && small <= cus && n1 + n2 <= per_xcd) {
            est = bwd_one_round_us(p, block_ap, dx, (double)n2 / (double)per_xcd) / (0.96 * bwd_apart_few_us(p, block_ap, alone_us, (double)small / cus));
        } else {
            const double t1 = dx == kBwdBig ? 4.6 + 1.26 * (double)((p.O + 63) / 64) : 4.0 + (double)((p.O + 127) / 128) * (dx == 64 ? 0.78 : dx == 96 ? 0.83 : 0.98);
            // n1 tiles on the compute units of an XCD: `late` of them are done after `a`, the others after `b`
            const int64_t late = n1 % per_xcd;
            const double b = (double)(n1 / per_xcd) * t1, a = late ? b + t1 : b, even = ((double)n1 * t1 + (double)n2 * t2) / (double)per_xcd;
            // the end of the last tile of dW: some whole number of them after a or b
            double end = 1e30;
            for (const double from : {a, b}) {
                const double first = from + t2 * std::max(0.0, (double)(int64_t)((even - from) / t2) - 2.0);
                for (int i = 0; i < 8; ++i) {
                    const double at = first + t2 * i;
                    const int64_t done = late * (int64_t)std::max(0.0, (at - a) / t2 + 1e-9) + (per_xcd - late) * (int64_t)std::max(0.0, (at - b) / t2 + 1e-9);
                    if (done >= n2 && at < end) end = at;
                }
            }
            if (cut) end = even + 0.4 * t2;           // the pieces of its last tiles are short
            est = (4.0 + 0.62 * std::max(end, a) + 0.38 * std::max(even, t1)) / (0.99 * apart);
        }
        if (est < least) { least = est; best = dx == kBwdBig && p.O % 128 != 0 ? kBwdBigRagged : dx; }
    }
    return best;
}

// Bytes from sk.partials on within which a launch of the forward (gemm = 0), the dX (1) or the dW (2) GEMM writes its parts.
size_t parts_written(const Problem &p, int gemm, int cus, const SkScratch &sk)
{
    constexpr int kSmall = TileSmall::BM * TileSmall::BN, kBig = TileBig::BM * TileBig::BN;
    if (gemm == 2) {
        bool small;
        const DwLaunchPlan d = plan_dw_of(p, cus, sk, &small);
        return d.cut ? parts_bytes(d.grid, small ? kSmall : kBig, d.sk.split != 0) : 0;
    }
    if (gemm == 1 && mid_dx_tokens(p, cus, sk)) return 0;
    if (const int parts = ksplit_parts(p, gemm == 1, sk)) return ksplit_bytes(p, gemm == 1, parts);
    TileChoice choice;
    const QLaunchPlan q = plan_q_of(p, gemm == 1, cus, sk, &choice);
    return q.sk.walk && (q.sk.dp_rounds == 0 || q.sk.split) ? parts_bytes(q.grid, choice == TileChoice::Small ? kSmall : kBig, q.sk.split != 0) : 0;
}

// Whether a launch takes parts that it can go without: it shares its tiles because they are few (k_gemm_ksplit, big tiles), or
// another choice of tiles needs none.
bool can_do_without_parts(const Problem &p, int gemm)
{
    if (gemm == 2) return false;
    if (ksplit_parts(p, gemm == 1, kAnyRoom)) return true;
    TileChoice choice, other;
    (void)plan_q_of(p, gemm == 1, kMaxCus, kAnyRoom, &choice);
    (void)plan_q_of(p, gemm == 1, kMaxCus, SkScratch{}, &other);
    return other != choice;
}

}  // namespace

// Scratch that cutting or sharing tiles needs, for whichever of the GEMMs of a problem may do so (fwd: the forward, bwd: dX and
// dW): the largest of their needs, with the full complement of compute units.
void sk_scratch_bytes(const Problem &p, bool fwd, bool bwd, size_t *partial_bytes, size_t *needed_bytes, size_t *counter_bytes)
{
    *partial_bytes = *needed_bytes = 0;
    *counter_bytes = p.act_bf16 ? (size_t)kSkCounterWords * sizeof(uint32_t) : 0;     // whatever the token count
    if (!p.act_bf16 || p.T == 0) return;
    for (int gemm = fwd ? 0 : 1; gemm < (bwd ? 3 : 1); ++gemm) {
        const size_t bytes = parts_written(p, gemm, kMaxCus, kAnyRoom);
        *partial_bytes = std::max(*partial_bytes, bytes);
        if (!can_do_without_parts(p, gemm)) *needed_bytes = std::max(*needed_bytes, bytes);
    }
}

size_t parts_written_for_test(const Problem &p, int gemm, int cus, const SkScratch &sk) { return parts_written(p, gemm, cus, sk); }

void dx_route_for_test(const Problem &p, bool block_ap, int32_t route[2])
{
    route[0] = mid_dx_tokens(p, current_cus(), kAnyRoom);
    route[1] = bwd_together(p, block_ap, current_cus(), kAnyRoom);
}

// Test aid: work item number j of workgroup `block` in the launch that the forward (gemm = 0), the dX (gemm = 1) or the dW
// (gemm = 2; tile rows: in-features, tile columns: out-features, K: tokens) GEMM of this problem makes, as the kernel
// itself works it out (the tile kernels' launch, also where the dispatch takes another route at that token count, or k_gemm_ksplit).
// item = {tile row, tile column, first and past-the-last K-tile pair, contributors of the tile, the first contributor's index in its XCD, 1 for a split tile, counter index, grid, K-tile pairs per tile, tile rows, tile
// columns}.  Returns 1, 0 past the workgroup's last item, -1 for a bad argument.
int plan_item_for_test(const Problem &p, int gemm, int block, int j, int32_t item[12])
{
    if (!p.act_bf16 || p.T < 1 || gemm < 0 || gemm > 2 || block < 0 || j < 0) return -1;
    if (gemm == 2) {
        bool small;
        const DwLaunchPlan d = plan_dw_of(p, current_cus(), kAnyRoom, &small);
        if (block >= d.grid) return -1;
        SkItem it{};
        bool ok;
        if (d.cut) {
            ok = sk_item_of(d.sk, d.ntiles, d.tiles_m, d.tiles_n, 8, block, d.grid, j, it);
        } else {        // one workgroup per tile
            ok = j == 0 && tile_of_xcd_slot(d.grid, block & 7, block >> 3, d.tiles_m, d.tiles_n, it.tm, it.tn, 8);
            it.kb = 0; it.ke = (((int)p.T + 63) / 64 + 1) / 2; it.parts = 1;
        }
        const int32_t v[12] = {it.tm, it.tn, it.kb, it.ke, it.parts, it.first, it.fixed, it.ctr, d.grid, (((int)p.T + 63) / 64 + 1) / 2, d.tiles_m, d.tiles_n};
        for (int k = 0; k < 12; ++k) item[k] = v[k];
        return ok ? 1 : 0;
    }
    TileChoice choice;
    const QLaunchPlan q = plan_q_of(p, gemm == 1, current_cus(), kAnyRoom, &choice);
    if (block >= q.grid) return -1;
    SkItem it{};
    bool ok;
    if (q.mode == kCut) {
        ok = sk_item_of(q.sk, q.ntiles, q.tiles_m, q.tiles_n, q.band, block, q.grid, j, it);
    } else {        // whole tiles only, as in the kernel's other instantiation
        const int loc_step = q.sk.walk ? q.grid >> 3 : q.ntiles;
        ok = tile_of_xcd_slot(q.sk.walk ? q.ntiles : q.grid, block & 7, (block >> 3) + j * loc_step, q.tiles_m, q.tiles_n, it.tm, it.tn, q.band);
        it.kb = 0; it.ke = q.sk.pairs; it.parts = 1;
    }
    const int32_t v[12] = {it.tm, it.tn, it.kb, it.ke, it.parts, it.first, it.fixed, it.ctr, q.grid, q.sk.pairs, q.tiles_m, q.tiles_n};
    for (int k = 0; k < 12; ++k) item[k] = v[k];
    return ok ? 1 : 0;
}

void launch_mfma_fwd(const Problem &p, const void *X, const void *codes, const void *sz, void *Y, const SkScratch &sk,
                     hipStream_t st)
{
    if (p.T == 0) return;
    if (const int parts = ksplit_parts(p, false, sk)) { launch_ksplit(p, false, X, codes, sz, Y, sk, parts, st); return; }
    GemmQArgs a{};
    a.A = (const bf16_t *)X; a.codes = (const uint32_t *)codes; a.sz = (const floatx2 *)sz; a.C = (bf16_t *)Y;
    a.M = (int)p.T; a.N = (int)p.O; a.K = (int)p.I; a.I = (int)p.I; a.G = (int)p.G; a.g = (int)p.g;
    a.a_bytes = (uint32_t)(p.T * p.I * 2); a.codes_bytes = (uint32_t)work_code_bytes(p); a.sz_bytes = (uint32_t)(p.O * p.G * 8);
    launch_q_bits<false>(p, a, sk, st);
}

namespace {

GemmQArgs dx_args(const Problem &p, const void *dY, const void *codes, const void *sz, void *dX)
{
    GemmQArgs a{};
    a.A = (const bf16_t *)dY; a.codes = (const uint32_t *)codes; a.sz = (const floatx2 *)sz; a.C = (bf16_t *)dX;
    a.M = (int)p.T; a.N = (int)p.I; a.K = (int)p.O; a.I = (int)p.I; a.G = (int)p.G; a.g = (int)p.g;
    a.a_bytes = (uint32_t)(p.T * p.O * 2); a.codes_bytes = (uint32_t)work_code_bytes(p); a.sz_bytes = (uint32_t)(p.O * p.G * 8);
    a.c_bytes = (uint32_t)(p.T * p.I * 2);
    return a;
}

GemmDwArgs dw_args(const Problem &p, const void *X, const void *dY, const void *W, const void *codes, const void *clampbits, const void *sz,
                   void *dW, float *ds, float *dz, float *part)
{
    GemmDwArgs a{};
    a.X = (const bf16_t *)X; a.dY = (const bf16_t *)dY; a.W = W; a.codes = (const uint32_t *)codes;
    a.clampbits = (const uint8_t *)clampbits; a.sz = (const floatx2 *)sz;
    a.dW = dW; a.ds = ds; a.dz = dz;
    a.T = (int)p.T; a.I = (int)p.I; a.O = (int)p.O; a.G = (int)p.G; a.g = (int)p.g;
    a.x_bytes = (uint32_t)(p.T * p.I * 2); a.dy_bytes = (uint32_t)(p.T * p.O * 2);
    a.w_bytes = (uint32_t)(p.O * p.I * (p.w_bf16 ? 2 : 4)); a.codes_bytes = (uint32_t)work_code_bytes(p);
    a.clamp_bytes = (uint32_t)(p.O * p.I / 8); a.sz_bytes = (uint32_t)(p.O * p.G * 8);
    a.part_ds = part; a.part_dz = part ? part + (size_t)p.O * (p.I / 32) : nullptr;
    return a;
}

void reduce_dw_partials(const Problem &p, const GemmDwArgs &a, const float *s, hipStream_t st)
{
    ProfScope ps(PK_REDUCE, st);
    if (a.ds != nullptr || a.dz != nullptr) launch_reduce_partials(a.part_ds, a.part_dz, a.ds, a.dz, s, (size_t)p.O * p.G, (uint32_t)(p.g / 32), st);
}

}  // namespace

void launch_mfma_dx(const Problem &p, const void *dY, const void *codes, const void *sz, void *dX, const SkScratch &sk,
                    hipStream_t st)
{
    if (p.T == 0) return;
    if (const int tokens = mid_dx_tokens(p, current_cus(), sk)) { launch_mid_dx(p, tokens, dY, codes, sz, dX, st); return; }
    if (const int parts = ksplit_parts(p, true, sk)) { launch_ksplit(p, true, dY, codes, sz, dX, sk, parts, st); return; }
    const GemmQArgs a = dx_args(p, dY, codes, sz, dX);
    launch_q_bits<true>(p, a, sk, st);
}

void launch_mfma_dw(const Problem &p, bool block_ap, const void *X, const void *dY, const void *W, const void *codes,
                    const void *clampbits, const void *sz, const float *s, void *dW, float *ds, float *dz, float *part,
                    const SkScratch &sk, hipStream_t st)
{
    const GemmDwArgs a = dw_args(p, X, dY, W, codes, clampbits, sz, dW, ds, dz, part);
    bool partials;
    {
        ProfScope ps(PK_GEMM_DW, st);
        if (block_ap) {
            if (p.w_bf16) partials = launch_dw_bits<bf16_t, true>(p.bits, a, sk, st);
            else partials = launch_dw_bits<float, true>(p.bits, a, sk, st);
        } else {
            partials = launch_dw_bits<bf16_t, false>(p.bits, a, sk, st);
        }
    }
    if (partials) reduce_dw_partials(p, a, s, st);
}

void launch_mfma_bwd(const Problem &p, bool block_ap, const void *X, const void *dY, const void *W, const void *codes, const void *clampbits,
                     const void *sz, const float *s, void *dX, void *dW, float *ds, float *dz, float *part, const SkScratch &sk, hipStream_t st)
{
    const bool want_w = dW != nullptr || ds != nullptr || dz != nullptr;
    const int dx = dX != nullptr && want_w ? bwd_together(p, block_ap, current_cus(), sk) : -1;
    if (dx < 0) {
        if (dX != nullptr) { ProfScope ps(PK_GEMM_DX, st); launch_mfma_dx(p, dY, codes, sz, dX, sk, st); }
        if (want_w) launch_mfma_dw(p, block_ap, X, dY, W, codes, clampbits, sz, s, dW, ds, dz, part, sk, st);
        return;
    }
    GemmDwArgs d = dw_args(p, X, dY, W, codes, clampbits, sz, dW, ds, dz, part);
    d.tiles_m = (d.I + DwTileBig::BM - 1) / DwTileBig::BM; d.tiles_n = (d.O + DwTileBig::BN - 1) / DwTileBig::BN;
    d.direct = DwTileBig::BM % d.g == 0 ? 1 : 0;
    GemmQArgs q{};
    MidArgs m{};
    int n_dx;
    if (dx >= 64) {
        m = mid_dx_args(p, dx, dY, codes, sz, dX);
        n_dx = m.tiles_m * m.tiles_n;
    } else {
        q = dx_args(p, dY, codes, sz, dX);
        q.tiles_m = (q.M + TileBig::BM - 1) / TileBig::BM; q.tiles_n = (q.N + TileBig::BN - 1) / TileBig::BN;
        q.band = q_band(q.tiles_m);
        n_dx = q.tiles_m * q.tiles_n;
    }
    {
        ProfScope ps(PK_GEMM_BWD, st);
        const DwLaunchPlan alone = block_ap ? p.w_bf16 ? plan_dw<bf16_t, true, DwTileBig>(d.I, d.O, d.T, current_cus(), sk) : plan_dw<float, true, DwTileBig>(d.I, d.O, d.T, current_cus(), sk)
                                            : plan_dw<bf16_t, false, DwTileBig>(d.I, d.O, d.T, current_cus(), sk);
        bool small;
        if (plan_dw_of(p, current_cus(), sk, &small).cut) d.sk = alone.sk;          // (of tiles of 256: bwd_together)
        const int n_dw = d.sk.walk ? alone.grid : d.tiles_m * d.tiles_n;
        if (!block_ap) launch_bwd_e2e(p.bits, dx, q, m, d, n_dx, n_dw, st);
        else if (p.w_bf16) launch_bwd_ap_bf16(p.bits, dx, q, m, d, n_dx, n_dw, st);
        else launch_bwd_ap_f32(p.bits, dx, q, m, d, n_dx, n_dw, st);
    }
    if (!d.direct) reduce_dw_partials(p, d, s, st);
}

}  // namespace eqat
