// Dispatch of the GEMM + TopK route kernel (rr_route_impl.hpp) by mode, input
// type and tile width.
#include "rr_route_impl.hpp"

namespace rr {

hipError_t launch_route_f32_full(const RouteArgs &a, int grid, hipStream_t stream);
hipError_t launch_route_f32_anchor(const RouteArgs &a, int grid, hipStream_t stream);
hipError_t launch_route_f32_reroute(const RouteArgs &a, int grid, hipStream_t stream);
hipError_t launch_route_bf16_full(const RouteArgs &a, int grid, hipStream_t stream);
hipError_t launch_route_bf16_anchor(const RouteArgs &a, int grid, hipStream_t stream);
hipError_t launch_route_bf16_reroute(const RouteArgs &a, int grid, hipStream_t stream);
hipError_t launch_route_f32_relay(const RouteArgs &a, int grid, hipStream_t stream);
hipError_t launch_route_bf16_relay(const RouteArgs &a, int grid, hipStream_t stream);

bool route_supported(int dtype, int d, int T)
{
    if (T < 1 || T > 128) return false;
    if (dtype == 0) return d == 32 || d == 64 || d == 128;
    if (dtype == 1) return d == 32 || d == 64 || d == 128 || d == 256;
    return false;
}

// Fewer 128-row tiles than compute units leave units idle and each tile's
// sweeps long (binary32 products run at 1/16 of the bf16 rate; a causal
// tile's key range is its last row's): 32-row tiles then spread the same
// rows over four times the workgroups.  With a tile per unit or more, the
// extra passes over each key head cost more than they save.
int route_tile_rows(int T, int n_heads, int n_q)
{
    if (T > 64) return kWideTileRows;
    const int64_t narrow = (int64_t)n_heads * ((n_q + kNarrowTileRows - 1) / kNarrowTileRows);
    return narrow < kFewTiles ? kSmallTileRows : kNarrowTileRows;
}

// Slots a tile of several panels may stage per row: its key rows' region takes 416
// (128 bytes each) beside the prefix counts, and 160 KB of LDS leave room for
// some more.
constexpr int kPanelSlots = 440;

// The resident-score kernel holds a 32-row tile's scores over the whole key
// range in registers: up to 1024 keys on four waves, 2048 on eight, and 4096 in
// panels on eight.  Eight lanes per row (four waves) sort 64 scores, sixteen
// sort 128.
int resident_shape(int n_k, int k, int m, int r, int n_mand)
{
    const int T = k + m;
    if (n_k > 4096 || T > 128) return 0;
    if (n_k > 2048) {
        const auto up = [](int x) { return (x + 3) & ~3; };
        return up(k) + up(m + r + n_mand) + up(r) <= kPanelSlots ? 386 : 0;
    }
    const int nw = (T > 64 || n_k > 1024) ? 8 : 4;
    const int kt = n_k <= 64 * nw ? 2 : (n_k <= 128 * nw ? 4 : 8);
    return 10 * nw + kt;
}

// Where that kernel is the faster one.  All times are of an anchor and three
// relays (two from 2049 keys) unless said otherwise, two-sweep tiles and split
// relays first, the resident tile second, at 32 heads and a drift of 0.3 (most
// rows rerouted) / 0.005 (a fifth).
//
// Panels (2049 to 4096 keys): with bf16 rows of up to 256 bytes and enough work
// for 128-row tiles (T <= 64) those read each key a quarter as often: 32 x 1024
// x 4096 969 against 1254 us, causal 32 x 4096 1138 against 1652.  With few of
// them panels win: 16 x 1024 x 4096 422 against 318 us.  Wider routes (64-row
// tiles) without the causal mask relay by rescoring and a compacted reroute,
// which at a low drift is the faster way where rows are many (32 x 4096, 9 % of
// the rows rerouted: 1796 against 2592 us; 32 x 1024: 649 against 668); causal
// 32 x 4096 at T = 96 takes 2653 against 2024 us.  Binary32 of d = 128: 2859
// against 1302 us at 32 x 1024 x 4096; 512-byte bf16 rows 1090 against 857.
static bool panels_pay(int dtype, int d, int64_t narrow, int64_t wide, bool causal, int T)
{
    if (dtype == 0 || d > 128) return true;
    if (T <= 64) return narrow < kFewTiles;
    return causal || wide < 2 * kFewTiles;
}

// Up to 2048 keys the tile wins under the causal mask (a tile reads the keys of
// its own rows only), for T > 64 (64-row tiles on the other side), for binary32
// products and where 128-row tiles would be few.  Left to the 128-row tiles,
// from a tile per compute unit (`many`) and two (`most`):
//   bf16, d <= 128, 1025 to 2048 keys, where a resident tile takes eight waves
//     and a compute unit to itself: T = 48, 2048 x 1280 592 / 458 against 685 /
//     651 us, 2048 x 2048 739 / 574 against 783 / 744, full routing at k = 32
//     103 against 132 and 138 against 156.  The line at T: 52 (2048 x 1536 679 /
//     531 against 750 / 725, 1024 x 2048 438 / 401 against 426 / 412), past it
//     their candidate lists overflow (T = 56: 1024 x 1536 442 / 392 against 391 /
//     380; with `most` 770 / 548 against 749 / 729; T = 60 854 / 618 against 728 /
//     695).  At 1024 keys the tile wins: 549 / 423 against 427 / 417.  So do
//     relays of d = 32 past 1536 keys without `most` (1024 x 1792 321 / 292
//     against 303 / 284; with it, 2048 x 2048, 609 / 473 against 605 / 568).
//   bf16, d = 256, more than 512 keys, T <= 24: full routing at k = 8 and 2048 x
//     1280 167 against 182 us (k = 32: 198 against 183); relays with `most`
//     only: T = 12, 2048 x 1536 988 / 695 against 960 / 918, 1024 x 1536 522 /
//     484 against 484 / 468.
//   binary32 relays of up to 256-byte rows in panels, T <= 56, with `most`: the
//     split schedule at 2048 x 2304, T = 48: d = 32 1139 / 765 against 1175 /
//     1138 us, d = 64 1753 / 1173 against 1528 / 1490.
bool resident_pays(int mode, int dtype, int d, int n_heads, int n_q, int n_k, bool causal, int T, bool one_pass)
{
    const auto tiles = [&](int rows) { return (int64_t)n_heads * ((n_q + rows - 1) / rows); };
    const int64_t narrow = tiles(kNarrowTileRows);
    if (n_k > 2048 && !panels_pay(dtype, d, narrow, tiles(kWideTileRows), causal, T)) return false;
    const bool relay = mode == MODE_RELAY, many = narrow >= kFewTiles, most = narrow >= 2 * kFewTiles;
    if (causal || T > 64 || !many || (relay && one_pass)) return true;
    if (dtype == 0) return !(relay && most && n_k > 2048 && d <= 64 && T <= 56);
    if (d <= 128) return n_k <= 1024 || T > (most ? 56 : 52) || (relay && !most && d == 32 && n_k > 1536);
    return n_k <= 512 || n_k > 2048 || T > 24 || (relay && !most);
}

int route_relay_max_bm_words(int dtype, int d, int T)
{
    using route_detail::relay_max_bm_words;
    switch (d) {
    case 32: return dtype == 0 ? relay_max_bm_words<float, 32>(T) : relay_max_bm_words<bf16_t, 32>(T);
    case 64: return dtype == 0 ? relay_max_bm_words<float, 64>(T) : relay_max_bm_words<bf16_t, 64>(T);
    case 128: return dtype == 0 ? relay_max_bm_words<float, 128>(T) : relay_max_bm_words<bf16_t, 128>(T);
    case 256: return dtype == 0 ? 0 : relay_max_bm_words<bf16_t, 256>(T);
    default: return 0;
    }
}

// One instance set per caller, input type and width (rr_resident_inst.hip).
#define RR_RESIDENT(mode) \
    hipError_t launch_resident_##mode##_float_32(const RouteArgs &, hipStream_t); \
    hipError_t launch_resident_##mode##_float_64(const RouteArgs &, hipStream_t); \
    hipError_t launch_resident_##mode##_float_128(const RouteArgs &, hipStream_t); \
    hipError_t launch_resident_##mode##_bf16_t_32(const RouteArgs &, hipStream_t); \
    hipError_t launch_resident_##mode##_bf16_t_64(const RouteArgs &, hipStream_t); \
    hipError_t launch_resident_##mode##_bf16_t_128(const RouteArgs &, hipStream_t); \
    hipError_t launch_resident_##mode##_bf16_t_256(const RouteArgs &, hipStream_t); \
    static hipError_t launch_resident_##mode(const RouteArgs &a, int dtype, hipStream_t s) \
    { \
        if (dtype == 0) { \
            switch (a.d) { \
            case 32: return launch_resident_##mode##_float_32(a, s); \
            case 64: return launch_resident_##mode##_float_64(a, s); \
            case 128: return launch_resident_##mode##_float_128(a, s); \
            default: return hipErrorInvalidValue; \
            } \
        } \
        switch (a.d) { \
        case 32: return launch_resident_##mode##_bf16_t_32(a, s); \
        case 64: return launch_resident_##mode##_bf16_t_64(a, s); \
        case 128: return launch_resident_##mode##_bf16_t_128(a, s); \
        case 256: return launch_resident_##mode##_bf16_t_256(a, s); \
        default: return hipErrorInvalidValue; \
        } \
    }
RR_RESIDENT(MODE_FULL)
RR_RESIDENT(MODE_ANCHOR)
RR_RESIDENT(MODE_RELAY)
#undef RR_RESIDENT

hipError_t launch_resident(const RouteArgs &a, int dtype, hipStream_t stream)
{
    switch (a.mode) {
    case MODE_FULL: return launch_resident_MODE_FULL(a, dtype, stream);
    case MODE_ANCHOR: return launch_resident_MODE_ANCHOR(a, dtype, stream);
    case MODE_RELAY: return launch_resident_MODE_RELAY(a, dtype, stream);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_route(const RouteArgs &a, int dtype, int grid, hipStream_t stream)
{
    if (a.resident) return launch_resident(a, dtype, stream);
    switch (a.mode) {
    case MODE_FULL: return dtype == 0 ? launch_route_f32_full(a, grid, stream) : launch_route_bf16_full(a, grid, stream);
    case MODE_ANCHOR:
        return dtype == 0 ? launch_route_f32_anchor(a, grid, stream) : launch_route_bf16_anchor(a, grid, stream);
    case MODE_REROUTE:
        return dtype == 0 ? launch_route_f32_reroute(a, grid, stream) : launch_route_bf16_reroute(a, grid, stream);
    case MODE_RELAY:
        return dtype == 0 ? launch_route_f32_relay(a, grid, stream) : launch_route_bf16_relay(a, grid, stream);
    default: break;
    }
    return hipErrorInvalidValue;
}

}  // namespace rr
